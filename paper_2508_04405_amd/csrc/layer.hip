// The linear layers of one decoder block as one call: each GEMM fed by the operator that
// produces its input with the activation quantizer fused in (paper Section 4.1.3), the
// activation width chosen per linear (Section 4.1.2: 8 bits for the down projection,
// 6 bits elsewhere).  Host code only: it strings together the library's own launches or, for a
// handful of tokens, prepares the one launch of decode_block.hip.
#include "api_internal.h"
#include "decode_block.h"
#include "flexq_kernels.h"

namespace {

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool bits_ok(int b) { return b == 6 || b == 8; }

struct Carve {
    int8_t *xq;      // [M, max(H, F)] codes of the stage being fed
    uint16_t *sx;    // [M]
    void *gemm;      // workspace of the GEMM calls (counter area first)
    size_t gemm_bytes;
};

size_t gemm_ws_bytes(const flexq_layer *L, int M)
{
    size_t need = 0;
    const int shapes[4][2] = {{L->QKV, L->H}, {L->H, L->H}, {2 * L->F, L->H}, {L->H, L->F}};
    for (const auto &s : shapes) {
        const size_t b = flexq_workspace_bytes(M, s[0], s[1]);
        if (b == 0) return 0;
        if (b > need) need = b;
    }
    return need;
}

struct Range {
    const uint8_t *p;
    size_t n;
};
inline bool overlap(const Range &a, const Range &b) { return a.p < b.p + b.n && b.p < a.p + a.n; }

}  // namespace

namespace flexq {

namespace {

// The one-launch form of the call (decode_block.hip), where it applies: fills its arguments.
//
// Where it is taken.  What it gains is the launches between linears that do not wait for each other, so
// it is for calls that hold stages 0 and 1: one launch over launches, LLaMA-2's 7B, 13B and 70B shapes at
// 1 .. 11 tokens, stages 0 to 3 0.86 .. 0.96 (7B at 8 tokens 54.1 -> 47.5 us, 13B's 69.0 -> 61.2, 70B's
// at one token 123 -> 113), stages 0 and 1 alone 0.84 .. 1.01.  A wait for another linear's outputs
// costs as much inside as two launches do: stages 2 and 3 0.93 .. 1.01, 1 and 2 0.90 .. 1.10, one stage
// 0.83 .. 1.31; those keep the launches.
// And for hidden sizes whose row block of tiles fills three quarters of a turn (24 of 32 tiles): below, fewer
// bytes are in flight and a wait covers less.  In replayed graphs, stages 0 to 3 at 1 .. 16 tokens, hidden
// size 512 1.10 .. 1.25, 1024 0.99 .. 1.10, 2048 0.92 .. 1.03, 2304 0.98 .. 1.12, 2560 0.96 .. 1.08, 3072 0.91 ..
// 1.01, 3584 0.84 .. 0.97.  (Called eagerly, 512 to 2048 take 0.85 .. 1.13 of the launches, whose seven calls
// are then the host's 26 us.)
constexpr int kLeastHidden = 24 * 128;

bool one_launch(const flexq_layer *L, int M, const flexq_layer_io *io, int first, int last, void *workspace,
                size_t room, bool forced, DecodeArgs &a, int &lds_bytes)
{
    if (!forced && (first > 0 || last < 1 || L->H < kLeastHidden)) return false;
    if (M > 16 || L->H > 8192 || L->F > 32768 || device_cu_count() != kDecodeGrid) return false;
    struct Stage {
        const void *w;
        const uint16_t *in, *gamma, *h;
        uint16_t *y;
        int N, K, row, bits, mode;
    };
    const Stage stages[4] = {
        {L->w_qkv, io->x, L->gamma_attn, io->h_attn_norm, io->qkv, L->QKV, L->H, L->H, L->bits_qkv, 0},
        {L->w_o, io->attn, nullptr, nullptr, io->o, L->H, L->H, L->H, L->bits_o, 2},
        {L->w_gate_up, io->x_ffn, L->gamma_ffn, io->h_ffn_norm, io->gate_up, 2 * L->F, L->H, L->H, L->bits_gate_up, 0},
        {L->w_down, io->gate_up, nullptr, io->h_swiglu, io->down, L->H, L->F, 2 * L->F, L->bits_down, 1}};
    a.n = last - first + 1;
    a.M = M;
    a.group = L->group;
    a.eps = L->eps;
    a.words = (unsigned *)workspace;
    // 41 us (0.16 us a poll).  Undisturbed no wait takes 128 polls: with bounds of 128, 256, 512 and 1024 the
    // 70B block takes 115 us, with 64 117; and beside another stream's GEMMs of 2048, 1000 and 300 tokens or
    // another block the four are equal within 1 %.
    a.spin = 256;
    // every linear's codes and token scales in a place of its own, behind the counters
    uint8_t *p = (uint8_t *)workspace + FLEXQ_WORKSPACE_COUNTER_BYTES, *const end = (uint8_t *)workspace + room;
    Range in[4], out[4];
    int taken = 0, pieces = 0;
    lds_bytes = 0;
    for (int i = 0; i < a.n; ++i) {
        const Stage &s = stages[first + i];
        const size_t tiles = (size_t)(s.N / 32) * (s.K / 128);
        if (s.h || tiles * 3072 > 0xFFFFF000u) return false;
        if (L->group != 0 && !streams_as_eight(M, s.N, s.K)) return false;
        DecodePhase &ph = a.ph[i];
        ph.packed = s.w;
        ph.scales = (const uint16_t *)((const uint8_t *)s.w + tiles * 3072);
        ph.y = s.y;
        ph.nb = s.N / 32;
        ph.kt = s.K / 128;
        ph.off = taken % kDecodeGrid;      // the next linear's row blocks begin where this one's ended
        taken += ph.nb;
        ph.inv = (unsigned)((1ull << 32) / (unsigned)(ph.kt * 8) + 1);
        ph.xq = (const int8_t *)p;
        p += round_up((size_t)M * s.K, 256);
        ph.sx = (uint16_t *)p;
        p += 256;
        const int lds = decode_block_lds(M, s.K);
        if (lds > lds_bytes) lds_bytes = lds;
        DecodeProducer &pr = a.pr[i];
        pr.in = s.in;
        pr.gamma = s.gamma;
        pr.xq = (int8_t *)ph.xq;
        pr.sx = ph.sx;
        pr.L = s.K;
        pr.mode = s.mode;
        pr.qmax = s.bits == 6 ? 31.0f : 127.0f;
        in[i] = Range{(const uint8_t *)s.in, (size_t)M * s.row * 2};
        out[i] = Range{(const uint8_t *)s.y, (size_t)M * s.N * 2};
        // an input is one of the outputs, all of it, or touches none
        pr.dep = -1;
        for (int q = 0; q < i; ++q) {
            if (overlap(out[q], out[i])) return false;
            if (in[i].p == out[q].p && in[i].n == out[q].n)
                pr.dep = q;
            else if (overlap(in[i], out[q]))
                return false;
        }
        for (int q = 0; q <= i; ++q)
            if (overlap(in[q], out[i])) return false;
        if (pr.dep >= 0 && pr.dep != i - 1) return false;
        pr.first = pr.dep < 0 ? pieces : 0;
        const int made = M * decode_pieces(pr.mode, pr.L);
        if (pr.first + made > kDecodeGrid) return false;        // a workgroup makes one piece of a producer
        if (pr.dep < 0) pieces += made;
    }
    if (p > end || lds_bytes > kDecodeLds) return false;
    return true;
}

}  // namespace

flexq_status layer_impl(const Tuning &tune, const flexq_layer *L, int M, const flexq_layer_io *io, int first_stage,
                        int last_stage, void *workspace, size_t workspace_bytes, void *stream, int *launched)
{
    if (!L || !io || M < 1) return FLEXQ_EINVAL;
    if (first_stage < 0 || last_stage > 3 || first_stage > last_stage) return FLEXQ_EINVAL;
    if (L->H < 1 || L->F < 1 || L->QKV < 1 || (L->group != 0 && L->group != 128) || !(L->eps > 0.0f))
        return FLEXQ_EINVAL;
    if (!bits_ok(L->bits_qkv) || !bits_ok(L->bits_o) || !bits_ok(L->bits_gate_up) || !bits_ok(L->bits_down))
        return FLEXQ_EINVAL;
    const size_t need = flexq_layer_workspace_bytes(L, M);
    if (need == 0) return FLEXQ_ESHAPE;
    // everything a stage in [first_stage, last_stage] touches is checked before any launch
    for (int s = first_stage; s <= last_stage; ++s) {
        const void *w = s == 0 ? L->w_qkv : s == 1 ? L->w_o : s == 2 ? L->w_gate_up : L->w_down;
        const void *in = s == 0 ? (const void *)io->x : s == 1 ? (const void *)io->attn
                       : s == 2 ? (const void *)io->x_ffn : (const void *)io->gate_up;
        const void *out = s == 0 ? (void *)io->qkv : s == 1 ? (void *)io->o : s == 2 ? (void *)io->gate_up
                                                                                     : (void *)io->down;
        const void *gamma = s == 0 ? L->gamma_attn : s == 2 ? L->gamma_ffn : (const void *)w;
        const void *h = s == 0 ? io->h_attn_norm : s == 2 ? io->h_ffn_norm : s == 3 ? io->h_swiglu : nullptr;
        if (!w || !in || !out || !gamma) return FLEXQ_EINVAL;
        if (!aligned16(w) || !aligned16(in) || !aligned16(out) || !aligned16(gamma) || (h && !aligned16(h)))
            return FLEXQ_EALIGN;
    }
    if (!workspace || workspace_bytes < need) return FLEXQ_EWORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return FLEXQ_EALIGN;

    Carve c;
    c.gemm_bytes = gemm_ws_bytes(L, M);
    c.gemm = workspace;                                       // its counter area leads the workspace
    uint8_t *p = (uint8_t *)workspace + c.gemm_bytes;
    const int widest = L->H > L->F ? L->H : L->F;
    c.xq = (int8_t *)p;
    c.sx = (uint16_t *)(p + round_up((size_t)(M < 32 ? 32 : M) * widest, 256));

    hipStream_t st = (hipStream_t)stream;
    DecodeArgs one;
    int lds_bytes = 0;
    const bool block = tune.fuse != 2 && one_launch(L, M, io, first_stage, last_stage, workspace, need,
                                                    tune.fuse == 1, one, lds_bytes);
    if (launched) *launched = block ? 1 : 0;
    if (block) {
        if (tune.spin != 0) one.spin = tune.spin < 0 ? 0 : tune.spin;
        return launch_decode_block(one, lds_bytes, st) == hipSuccess ? FLEXQ_OK : FLEXQ_EHIP;
    }
    const Tuning automatic{};
    auto gemm = [&](int bits, const void *w, const int8_t *xq, const uint16_t *sx, const uint16_t *x_fp16,
                    int N, int K, uint16_t *y, int xt) {
        return flexq::linear_impl(automatic, bits, w, L->group, xq, sx, x_fp16, M, N, K, y, nullptr, c.gemm,
                                  c.gemm_bytes, stream, nullptr, 0, nullptr, xt);
    };
    // batches of 11 to 32 tokens: the producers write their codes in tile order (packed at
    // 6 bits) where the streaming kernel reads them faster that way
    auto layout = [&](int bits, int N, int K) {
        return flexq::linear_wants_tiles(bits, M, N, K, L->group) ? bits : 0;
    };
    // Stages 0 and 1 do not wait for each other where the attention output is no part of what stage 0
    // writes: both are quantized in one launch then, the attention output into the place that the
    // linear call keeps for it (a single token is quantized by the linear itself).
    const size_t row = (size_t)M * L->H * 2;
    const Range attn{(const uint8_t *)io->attn, row};
    const bool both = M > 1 && first_stage == 0 && last_stage >= 1 &&
                      !overlap(attn, Range{(const uint8_t *)io->qkv, (size_t)M * L->QKV * 2}) &&
                      !(io->h_attn_norm && overlap(attn, Range{(const uint8_t *)io->h_attn_norm, row}));
    int8_t *const attn_q = (int8_t *)c.gemm + FLEXQ_WORKSPACE_COUNTER_BYTES;
    uint16_t *const attn_s = (uint16_t *)(attn_q + linear_codes_bytes(M, L->H));
    for (int s = first_stage; s <= last_stage; ++s) {
        flexq_status r = FLEXQ_OK;
        if (s == 0) {            // RMS norm + quantize -> fused QKV
            const int lay = layout(L->bits_qkv, L->QKV, L->H);
            if (both) {
                if (launch_norm_and_quant(io->x, L->gamma_attn, L->eps, L->bits_qkv, c.xq, c.sx, io->h_attn_norm, lay,
                                          io->attn, L->bits_o, attn_q, attn_s, layout(L->bits_o, L->H, L->H), M, L->H,
                                          st) != hipSuccess)
                    return FLEXQ_EHIP;
            } else if (flexq::launch_rmsnorm_quant(io->x, L->gamma_attn, L->eps, M, L->H, L->bits_qkv, c.xq, c.sx,
                                            io->h_attn_norm, st, lay) != hipSuccess)
                return FLEXQ_EHIP;
            r = gemm(L->bits_qkv, L->w_qkv, c.xq, c.sx, nullptr, L->QKV, L->H, io->qkv, lay);
        } else if (s == 1) {     // quantize node -> attention output projection (fp16 in: decode
                                 // batches quantize inside the streaming kernel)
            r = both ? gemm(L->bits_o, L->w_o, attn_q, attn_s, nullptr, L->H, L->H, io->o, layout(L->bits_o, L->H, L->H))
                     : gemm(L->bits_o, L->w_o, nullptr, nullptr, io->attn, L->H, L->H, io->o, 0);
        } else if (s == 2) {     // RMS norm + quantize -> fused gate | up
            const int lay = layout(L->bits_gate_up, 2 * L->F, L->H);
            if (flexq::launch_rmsnorm_quant(io->x_ffn, L->gamma_ffn, L->eps, M, L->H, L->bits_gate_up, c.xq,
                                            c.sx, io->h_ffn_norm, st, lay) != hipSuccess)
                return FLEXQ_EHIP;
            r = gemm(L->bits_gate_up, L->w_gate_up, c.xq, c.sx, nullptr, 2 * L->F, L->H, io->gate_up, lay);
        } else {                 // SiLU(gate) * up + quantize -> down projection
            const int lay = layout(L->bits_down, L->H, L->F);
            if (flexq::launch_swiglu_quant(io->gate_up, M, L->F, L->bits_down, c.xq, c.sx, io->h_swiglu, st,
                                           lay) != hipSuccess)
                return FLEXQ_EHIP;
            r = gemm(L->bits_down, L->w_down, c.xq, c.sx, nullptr, L->H, L->F, io->down, lay);
        }
        if (r != FLEXQ_OK) return r;
    }
    return FLEXQ_OK;
}

}  // namespace flexq

#pragma GCC visibility push(default)
extern "C" {

size_t flexq_layer_workspace_bytes(const flexq_layer *L, int M)
{
    if (!L || M < 1 || L->H < 1 || L->F < 1 || L->QKV < 1) return 0;
    const size_t g = gemm_ws_bytes(L, M);
    if (g == 0) return 0;
    const int widest = L->H > L->F ? L->H : L->F;
    // (fewer than 32 tokens: room for one block of 32-token tiles)
    return g + round_up((size_t)(M < 32 ? 32 : M) * widest, 256) + round_up((size_t)M * 2, 256);
}

flexq_status flexq_layer_linears(const flexq_layer *L, int M, const flexq_layer_io *io, int first_stage,
                                 int last_stage, void *workspace, size_t workspace_bytes, void *stream)
{
    return flexq::layer_impl(flexq::Tuning{}, L, M, io, first_stage, last_stage, workspace, workspace_bytes, stream,
                             nullptr);
}

}  // extern "C"
#pragma GCC visibility pop
