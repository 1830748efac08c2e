"""A decoder block's linears in one launch (decode_block.hip) against the separate launches, which
test_gpu_layer.py holds against the CPU oracle: the same bits for every stage, whoever does the
work -- with waits that run out at once (spin -1) every workgroup does what the others have not
finished, the way out on a busy or smaller device."""
import pytest
import torch

import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import DEV, build_packed, say, to_dev

pytestmark = pytest.mark.gpu

NAMES = ("qkv", "o", "gate_up", "down")


class Block:
    """Packed weights of a small block, its layer descriptor for given activation widths, and buffers."""

    def __init__(self, H, F, QKV, group, seed=1):
        self.H, self.F, self.QKV, self.group = H, F, QKV, group
        shapes = ((QKV, H), (H, H), (2 * F, H), (H, F))
        self.packed = [build_packed(n, k, 0.02, seed + i, group) for i, (n, k) in enumerate(shapes)]
        self.gains = [to_dev(synth.norm_gain(H, seed=seed + i)) for i in (10, 11)]

    def layer(self, bits):
        return fq.Layer(self.H, self.F, self.QKV, self.group, *self.packed, *self.gains, 1e-5, bits)

    def inputs(self, M, seed):
        return {k: to_dev(synth.activations(M, self.H, seed=seed + i, outlier_frac=0.02)) for i, k in enumerate(("x", "attn"))}

    def outputs(self, M):
        return {k: torch.full((M, n), float("nan"), dtype=torch.float16, device=DEV)
                for k, n in zip(NAMES, (self.QKV, self.H, 2 * self.F, self.H))}


def run(layer, M, ws, fuse, spin=0, first=0, last=3, **buffers):
    dev.set_fuse(fuse)
    dev.set_spin(spin)
    try:
        return dev.layer_linears(layer, M, ws, first, last, **buffers)
    finally:
        dev.set_fuse(0)
        dev.set_spin(0)


def equal(a, b):
    return [k for k in a if not torch.equal(a[k].view(torch.int16), b[k].view(torch.int16))] == []


# one row block per workgroup or none, several and a part; rows of one turn of tiles, of turns that do
# not divide, of more than one piece (4096) per token; turns of four and of five tiles
@pytest.mark.parametrize("group", [0, 128])
@pytest.mark.parametrize("H,F,QKV", [(128, 256, 96), (640, 1152, 800), (1024, 2816, 3072), (2048, 5632, 6144),
                                     (1280, 4224, 18464), (4224, 1152, 128), (4096, 4096, 4128)])
def test_one_launch_equals_the_separate_ones(H, F, QKV, group):
    block = Block(H, F, QKV, group)
    # with group-128 scales only where the streaming kernel adds in this one's order: every linear
    # unsplit (fewer row blocks of short rows are cut) and by eight wavefronts
    takes = group == 0 or (H, F, QKV) == (4096, 4096, 4128)
    for bits in ((6, 6, 6, 8), (8, 6, 8, 6)):
        layer = block.layer(bits)
        for M in (1, 2, 7, 8, 9, 16):
            say(f"one launch: H={H} F={F} QKV={QKV} group={group} A{bits} M={M}")
            ws, data, want = layer.make_workspace(M), block.inputs(M, 100 * M), block.outputs(M)
            assert not run(layer, M, ws, 2, x_ffn=want["o"], **data, **want)
            for spin in (0, -1):
                got = block.outputs(M)
                assert run(layer, M, ws, 1, spin, x_ffn=got["o"], **data, **got) == takes
                torch.cuda.synchronize()
                assert equal(got, want), (M, spin)
                assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
            # by the library's own choice only where a row block of the hidden size fills a turn
            got = block.outputs(M)
            assert run(layer, M, ws, 0, x_ffn=got["o"], **data, **got) == (takes and H >= 3072)
            assert equal(got, want)
            got = block.outputs(M)
            fq.layer_linears(layer, M, ws, x_ffn=got["o"], **data, **got)
            assert equal(got, want)


# Row blocks: one to four per workgroup.  Tiles per wavefront: 4 or 8 (whole turns of four), 10 or 11 (a part of
# the third), 5 (turns of five), 13 or 14 (a part of the third), 28; rows of two to seven pieces per token.  Where the
# launches are kept: sixteen or four wavefronts on some linear, or codes that do not fit LDS.
@pytest.mark.parametrize("H,F,QKV,takes,keeps", [(4096, 11008, 12288, (5, 8, 9, 11), (1, 4, 12)),
                                                 (5120, 13824, 15360, (5, 8, 9), (2, 4, 10, 16)),
                                                 (8192, 28672, 10240, (1, 5), (6,)),
                                                 (5120, 5120, 8192, (3, 15), (16,))])
def test_group_scales_of_whole_models(H, F, QKV, takes, keeps):
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    block = Block.__new__(Block)
    block.H, block.F, block.QKV, block.group = H, F, QKV, 128
    block.packed = [fq.pack_w6(*fq.quant_w6(torch.randn((n, k), generator=g, device=DEV).mul_(0.02), 128), 128)
                    for n, k in ((QKV, H), (H, H), (2 * F, H), (H, F))]
    block.gains = [to_dev(synth.norm_gain(H, seed=i)) for i in (10, 11)]
    layer = block.layer((6, 8, 6, 8))
    for M in takes + keeps:
        say(f"one launch, group scales: H={H} F={F} M={M}")
        ws, data, want = layer.make_workspace(M), block.inputs(M, 100 * M), block.outputs(M)
        assert not run(layer, M, ws, 2, x_ffn=want["o"], **data, **want)
        for spin in (0, -1):
            got = block.outputs(M)
            assert run(layer, M, ws, 1, spin, x_ffn=got["o"], **data, **got) == (M in takes), M
            torch.cuda.synchronize()
            assert equal(got, want), (M, spin)
            assert int(ws[:16384].view(torch.int32).abs().sum()) == 0


@pytest.mark.parametrize("first,last", [(0, 1), (0, 2), (1, 3), (2, 3), (0, 0), (3, 3)])
def test_ranges_of_stages_and_an_input_of_its_own(first, last):
    block, M = Block(1024, 2816, 3072, 0), 5
    layer = block.layer((6, 6, 6, 8))
    ws, data = layer.make_workspace(M), block.inputs(M, 3)
    data["x_ffn"] = to_dev(synth.activations(M, block.H, seed=9))
    gate_up = to_dev(synth.activations(M, 2 * block.F, seed=10))
    for spin in (0, -1):
        outs = []
        for fuse in (2, 1):
            outs.append(block.outputs(M))
            outs[-1]["gate_up"].copy_(gate_up)
            assert run(layer, M, ws, fuse, spin, first, last, **data, **outs[-1]) == (fuse == 1)
        assert equal(*outs), (first, last, spin)


def test_buffers_that_overlap_keep_the_separate_launches():
    block, M = Block(1024, 2816, 3072, 0), 2
    layer, H = block.layer((6, 6, 6, 8)), 1024
    ws, data = layer.make_workspace(M), block.inputs(M, 3)
    out = block.outputs(M)
    assert run(layer, M, ws, 1, x_ffn=out["o"], **data, **out)
    flat = out["qkv"].view(-1)
    inside = flat[:M * H].view(M, H)                       # of the qkv output, not all of it
    assert not run(layer, M, ws, 1, x_ffn=out["o"], x=data["x"], attn=inside, **out)
    assert not run(layer, M, ws, 1, x_ffn=inside, **data, **out)
    assert not run(layer, M, ws, 1, x_ffn=out["o"], **data, **dict(out, down=data["x"]))
    assert not run(layer, M, ws, 1, x_ffn=out["o"], **data, **dict(out, o=inside))
    assert not run(layer, M, ws, 1, x_ffn=out["o"], h_swiglu=torch.empty((M, block.F), dtype=torch.float16, device=DEV),
                   **data, **out)
    assert not run(layer, 17, layer.make_workspace(17), 1, x_ffn=(o := block.outputs(17))["o"], **block.inputs(17, 1), **o)
    torch.cuda.synchronize()


@pytest.mark.parametrize("M", [2, 20, 40])
def test_attention_output_inside_the_qkv_buffer(M):
    """Stage 1 then reads what stage 0 writes: one call gives what a call per stage gives, and so it does
    with buffers apart, where both inputs are quantized in one launch."""
    block = Block(1024, 2816, 3072, 0)
    layer = block.layer((6, 8, 6, 8))
    ws, data = layer.make_workspace(M), block.inputs(M, 3)
    for inside in (True, False):
        outs = []
        for calls in (((0, 3),), ((0, 0), (1, 1), (2, 3))):
            out = block.outputs(M)
            attn = out["qkv"].view(-1)[:M * block.H].view(M, block.H) if inside else data["attn"]
            for first, last in calls:
                fq.layer_linears(layer, M, ws, first, last, x=data["x"], attn=attn, x_ffn=out["o"], **out)
            outs.append(out)
        torch.cuda.synchronize()
        assert equal(*outs), inside


@pytest.mark.parametrize("group", [0, 128])
def test_fresh_inputs_on_one_workspace(group):
    """Two hundred back-to-back calls with eight sets of inputs in turn: no value of an earlier call,
    in the codes, the outputs or the words between workgroups, shows in a later one."""
    block, M = Block(2048, 5632, 6144, group) if group == 0 else Block(4096, 4096, 4128, group), 6
    layer = block.layer((6, 6, 6, 8))
    ws = layer.make_workspace(M)
    sets = [block.inputs(M, 50 * i) for i in range(8)]
    wants = []
    for data in sets:
        wants.append(block.outputs(M))
        run(layer, M, ws, 2, x_ffn=wants[-1]["o"], **data, **wants[-1])
    out, differs = block.outputs(M), torch.zeros(1, dtype=torch.int32, device=DEV)
    for rep in range(200):
        i = (5 * rep + rep // 8) % 8
        assert run(layer, M, ws, 1, x_ffn=out["o"], **sets[i], **out)
        for k in NAMES:
            differs += (out[k] != wants[i][k]).any()
        if rep % 50 == 49:
            assert int(differs.item()) == 0, rep
    assert int(ws[:16384].view(torch.int32).abs().sum()) == 0


def test_two_streams_at_once():
    """Two blocks on two streams, each with buffers of its own: whichever workgroups are resident, both
    give the bits they give alone."""
    block, M = Block(1024, 2816, 3072, 0), 4
    layer = block.layer((6, 6, 6, 8))
    lanes = []
    for i in range(2):
        data, want = block.inputs(M, 70 * i), block.outputs(M)
        ws = layer.make_workspace(M)
        run(layer, M, ws, 2, x_ffn=want["o"], **data, **want)
        lanes.append((torch.cuda.Stream(), ws, data, want, block.outputs(M)))
    torch.cuda.synchronize()
    for rep in range(20):
        for stream, ws, data, want, out in lanes:
            with torch.cuda.stream(stream):
                assert run(layer, M, ws, 1, x_ffn=out["o"], **data, **out)
    torch.cuda.synchronize()
    for stream, ws, data, want, out in lanes:
        assert equal(out, want)
        assert int(ws[:16384].view(torch.int32).abs().sum()) == 0


def test_beside_a_kernel_that_fills_the_chip():
    """A prefill GEMM on another stream holds every CU for a while: some workgroups of the block start late or
    find their partners missing, and the results stay the same."""
    block, M = Block(1024, 2816, 3072, 0), 4
    layer = block.layer((6, 6, 6, 8))
    ws, data, want, out = layer.make_workspace(M), block.inputs(M, 1), block.outputs(M), block.outputs(M)
    run(layer, M, ws, 2, x_ffn=want["o"], **data, **want)
    K, N, T = 4096, 8192, 2048
    packed = torch.zeros(fq.packed_bytes(N, K), dtype=torch.uint8, device=DEV)
    xq, sx = fq.quant_act(torch.ones((T, K), dtype=torch.float16, device=DEV), 8)
    big_ws, y = fq.make_workspace(T, N, K), torch.empty((T, N), dtype=torch.float16, device=DEV)
    differs = torch.zeros(1, dtype=torch.int32, device=DEV)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for rep in range(30):
        with torch.cuda.stream(a):
            for _ in range(3):
                fq.gemm_w6a8(packed, N, K, xq=xq, sx=sx, workspace=big_ws, out=y)
        with torch.cuda.stream(b):
            assert run(layer, M, ws, 1, x_ffn=out["o"], **data, **out)
            for k in NAMES:
                differs += (out[k] != want[k]).any()
    torch.cuda.synchronize()
    assert int(differs.item()) == 0
    assert int(ws[:16384].view(torch.int32).abs().sum()) == 0


def test_a_workgroup_that_comes_late_repeats_nothing():
    """A workgroup that starts when the others no longer wait for it finds its bit set in the linear's mask, set by
    one that did its row blocks: it leaves them alone.  Here the bits are set ahead of the launch, and what
    would have been stored there -- other values than the workgroups' own -- has to be there afterwards
    and in everything computed from it."""
    block, M = Block(1024, 2816, 3072, 0), 5
    layer, H, F = block.layer((6, 6, 6, 8)), 1024, 2816
    ws, data, other = layer.make_workspace(M), block.inputs(M, 3), block.inputs(M, 4)
    words = ws[:16384].view(torch.int32)
    plain, instead = block.outputs(M), block.outputs(M)
    run(layer, M, ws, 2, x_ffn=plain["o"], **data, **plain)
    run(layer, M, ws, 2, x_ffn=instead["o"], **other, **instead)
    # row block 0 of a linear is that of the workgroup behind the owner of the last linear's last one;
    # (linear, its first workgroup, row blocks): the attention output's 32, the gate and up projections' 176
    for stage, name, home, rows in ((1, "o", 3072 // 32, (0, 5, 31)), (2, "gate_up", (3072 + H) // 32, (1, 100, 127, 175))):
        for spin in (0, -1):
            got, want = block.outputs(M), {k: v.clone() for k, v in plain.items()}
            for b in rows:
                for out in (got, want):
                    out[name][:, 32 * b:32 * b + 32] = instead[name][:, 32 * b:32 * b + 32]
                slot = (home + b) % 256
                words[32 + (8 * stage + slot // 32) * 32] |= (1 << slot % 32) - (1 << 32 if slot % 32 == 31 else 0)
            run(layer, M, ws, 2, 0, stage + 1, 3, x_ffn=want["o"], **want)
            assert run(layer, M, ws, 1, spin, x_ffn=got["o"], **data, **got)
            torch.cuda.synchronize()
            assert int(words.abs().sum()) == 0
            assert not equal(want, plain) and equal(got, want), (name, spin)


def test_doing_what_is_missing_is_no_standstill():
    """LLaMA-2-7B's block at eight tokens with nobody waiting: every workgroup takes up what nobody has done yet,
    a different part where it can and with its tiles in flight.  1.6 times the separate launches' time;
    5.6 times before that was so; the line is twice what it takes."""
    H, F, QKV, M = 4096, 11008, 12288, 8
    packed = [torch.zeros(fq.packed_bytes(n, k), dtype=torch.uint8, device=DEV)
              for n, k in ((QKV, H), (H, H), (2 * F, H), (H, F))]
    gain = torch.ones(H, dtype=torch.float16, device=DEV)
    layer = fq.Layer(H, F, QKV, 0, *packed, gain, gain, 1e-5, (8, 8, 8, 8))
    ws, out = layer.make_workspace(M), {k: torch.empty((M, n), dtype=torch.float16, device=DEV)
                                        for k, n in zip(NAMES, (QKV, H, 2 * F, H))}
    x = torch.ones((M, H), dtype=torch.float16, device=DEV)
    best = {}
    for rep in range(7):
        for fuse, spin in ((2, 0), (1, -1)):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(10):
                assert run(layer, M, ws, fuse, spin, x=x, attn=x, x_ffn=out["o"], **out) == (fuse == 1)
            end.record()
            torch.cuda.synchronize()
            best[fuse] = min(best.get(fuse, 1e9), begin.elapsed_time(end))
    assert best[1] < 3.2 * best[2], best


def test_graph_replay():
    block, M = Block(1024, 2816, 3072, 0), 3
    layer = block.layer((6, 6, 6, 8))
    ws, data, out = layer.make_workspace(M), block.inputs(M, 1), block.outputs(M)
    assert run(layer, M, ws, 1, x_ffn=out["o"], **data, **out)
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            assert run(layer, M, ws, 1, x_ffn=out["o"], **data, **out)
    torch.cuda.synchronize()
    for rep in range(3):
        for k, v in block.inputs(M, 200 * rep + 7).items():
            data[k].copy_(v)
        graph.replay()
        torch.cuda.synchronize()
        got = {k: v.clone() for k, v in out.items()}
        run(layer, M, ws, 2, x_ffn=out["o"], **data, **out)
        torch.cuda.synchronize()
        assert equal(got, out), rep
    assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
