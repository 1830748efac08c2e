// Tiled i8-MFMA GEMM with BOTH operands through LDS: 256x256 tiles, 256x128 or 128x256.
//
// The 128x256 kernel is limited by power, and what costs power besides the
// MFMAs is every byte a wavefront brings in through the vector-memory path:
// timing probes put the packed-weight loads at about a fifth of its run time
// and the activation DMA at a tenth, while doubling the LDS operand reads
// costs 3 %.  This kernel therefore trades vector-memory bytes for LDS reads:
// one workgroup of eight wavefronts (2 along m x 4 along n, 128 x 32 NT each)
// owns a 256 x (128 NT) tile, and a packed weight tile is brought into LDS ONCE
// per workgroup (by DMA, like the activations) and read from there by the two
// wavefronts that share its columns: 0.875 KB through the vector-memory path
// per 32x32x128 block at NT = 2 instead of 1.25.
//
//   LDS: three weight stages (24 KiB for whole tiles), requested TWO stages ahead (a
//   packed weight panel is read by few workgroups, all at the same time, so its lines
//   come from HBM, well over a microsecond away), and activation stages of 32 KiB: for
//   whole tiles two of them, requested one stage ahead (an activation panel is shared by
//   every column tile of its row and mostly found in L2 or the Infinity Cache; a third
//   stage would not fit beside the weights), for half tiles, whose stages are shorter
//   than the memory latency, three, requested two ahead.  One workgroup per CU, two
//   wavefronts per SIMD.  The hand-over waits until at most the loads for the stage after
//   next are outstanding.
//
//   Where in a stage the requests are made matters as much as how far ahead (each
//   measured against the alternative on one box, alternating): whatever all eight
//   wavefronts do at the same moment -- right after the hand-over's barrier, at the
//   start of a stage -- is a burst that the matrix pipe waits out.  So the work beside
//   the MFMAs is dealt out over the eight steps of a stage (a step: the four MFMAs of one
//   k-step and column block):
//     step 0  activation requests (DMA); LDS reads: activation operands of k-step 1,
//             plane 1 of the stage's packed tiles
//     step 1  plane 2            step 2  activation operands of k-step 2
//     step 3  weight requests (DMA)       step 4  activation operands of k-step 3
//     step 6  hand-over: counted wait, barrier; plane 0 of the next stage's tiles
//     step 7  the next stage's first activation operands
//   Against everything at the stage's start and after the barrier: planes 1 and 2 later
//   +1.4 % (and the shorter register lifetimes end the spilling), weight requests later
//   +1.6 %, first activation operands a step after the barrier +0.9 %, one item per step
//   +1.4 %.  The activation requests stay at the start (a step later: -1.2 %; right after
//   the barrier, which would free their buffer a k-step earlier: -1.5 % to -3 %), and the
//   hand-over before the last k-step (a step earlier: -4.5 %, the requests have less time).
//   Letting the two wavefronts that share a pair of packed tiles expand one tile's fourth
//   k-step each and exchange the operands through LDS (a third fewer vector operations):
//   -1.4 %, the exchange costs more than the expansion.  Not
//   kept either: two weight buffers with a second barrier per stage to make room for a
//   third activation buffer (-3 %); raising one wavefront's priority over its SIMD-mate's,
//   for a k-step in turn or for part of a stage (-1 % to -40 %: a wavefront alone does not
//   keep the pipe busy, the two must interleave).
//
// Scales per channel; group-128 scales, on the weights or on both operands, run tiles of their
// own, 128x256 and 64x256 (group_item below).
//
// A launch is PERSISTENT: at most one workgroup per CU, each taking its items
// (tiles) one after the other, and the operands of the next item's first stages
// are already on their way into LDS while the finished tile is scaled and
// stored, so neither the first loads' latency nor the store burst stands
// between two tiles' MFMAs.  The wavefronts accumulate D^T (channels down the
// registers, one token per lane): a lane's four consecutive registers are four
// consecutive channels of one token, so the epilogue scales and converts in
// registers and sends 8-byte pieces of finished fp16 through a small LDS
// transpose, from which whole 128-byte lines are stored (Section 4.3.2's
// coalesced write-back, Section 4.3.4's fused dequantization).
//
// Launch forms.  Whole tiles.  Half tiles, 256x128: the tiles left over after
// the last whole round of 256, as twice as many items of half the work, so a
// round of up to 128 leftover tiles costs little more than half a round.
// And the cut tail (SK): the leftover tiles cut along K into contiguous runs of
// 128-k stages, one run per workgroup, whose int32 sums (exact, so the order of
// addition does not matter) meet in the workspace.  EVENLY (SK = 2): every tile
// into the same number of pieces, which end together and share the tile's
// reduction -- each piece stores the sums of the slabs it does not own, waits a
// bounded number of polls for the tile's stage count to be complete and
// finishes the slabs it owns; a piece whose wait runs out leaves its slabs to
// the piece that completed the count.  Or into 256 equal runs that begin and
// end inside tiles (SK = 1): the workgroups of a tile add their stage counts
// to the tile's counter, and the one that completes the count adds the others'
// sums to its own registers and runs the epilogue; nobody waits for anybody.
// And low tiles, 128x256, on their own: up to 128 tokens on a layer wide enough
// for them to fill the chip in one round, where the time is the one pass over
// the weights (about 37 GB/s per CU come through the DMA path, here as in the
// whole tiles); on narrower layers, from 65 tokens, each cut evenly along K; and
// above 128 tokens where they fill the chip more evenly than 256-row tiles
// (gemm_low_choose), those beyond the last whole round cut evenly.  And 192-row tiles, 192x256,
// whole, where their height fits the tokens or the rounds better (gemm_192_us).
#include "flexq_device.h"
#include "flexq_kernels.h"
#include "gemm_common.h"
#include <type_traits>

namespace {

constexpr int WAVES = 8;
// The outputs' stores in the last round of a launch go past the caches, those of the rounds before it do
// not.  Nothing follows the last round, and the lines that it leaves in the caches are written back while the
// chip waits: layers of K -> N 1536 -> 8960 at 1024 tokens 22.2 -> 20.4 us, 3584 -> 18944 at 300 28.1 -> 26.7, 8192 ->
// 10240 at 1024 83.0 -> 81.6, 4096 -> 12288 at 333 with group scales 34.6 -> 33.9; of 717 cells of one round the
// mean is 0.99 and none is slower by more than single cells differ from run to run (2.5 %).  Before that a
// workgroup waits for its stores together with its next item's first loads, and past the caches they take
// longer: 4096 -> 22016 at 1024 tokens with group scales 126 / 129 us, 5120 -> 27648 with both operands' 215 / 220,
// 5248 -> 13664 at 1300 (a round and half tiles) 102.6 / 104.5, a 13B block with group scales at 2048 850 / 863 (by
// this rule 853).  Pairs of pieces, a few items a workgroup, count as a last round (0.997 of the time).
constexpr int kLastRound = kNonTemporal;
constexpr int SLOT_BYTES = 256 * 256 * 4;      // one workgroup's int32 sums of a 256x256 tile

// The eight wavefronts share a whole tile 2 along m x 4 along n, 128 x 64 each (MT = 4 row
// blocks of 32, NT = 2 column blocks of 32: an expanded weight operand feeds four MFMAs,
// an activation operand two), and a half tile 4 along m x 2 along n, 64 x 64 each.  LDS
// delivers 128 bytes a clock to the CU and a 32x32x32 MFMA occupies a SIMD for 32, so a
// stage reads (MT + 0.75 NT) / (MT NT) KiB per MFMA of at most 1 KiB: 0.69 for the whole
// tile, 0.875 for 64 x 64.  (The whole tile's 128-row layout on half the columns, 128 x 32
// per wavefront, would ask for 1.19; measured, it runs the half tiles at the same speed --
// their stages are not bound by LDS reads -- and the lighter shape was kept.  For whole
// tiles, 1 x 8 wavefronts of 256 x 32 halve the expansion work per MFMA for twice the
// activation reads: measured 2-5 % slower on every layer.)
// TILE names the shape: 2 the whole tile (256 x 256), 1 the half tile (256 x 128), 3 the
// low tile (128 x 256, 2 x 4 wavefronts of 64 x 64: for up to 128 tokens on wide layers),
// 4 the group tile (128 x 256, eight wavefronts side by side of 128 x 32: group-128 scales),
// 5 the same at half the height (64 x 256), 6 the three-quarter tile (192 x 256, 2 x 4
// wavefronts of 96 x 64, 0.75 KiB of LDS reads per MFMA; its smaller stages leave room for both
// operands two stages ahead)
template <int TILE>
struct Shape {
    static_assert(TILE >= 1 && TILE <= 6, "half, whole, low, group or three-quarter tiles");
    static constexpr bool GROUPED = TILE == 4 || TILE == 5;
    static constexpr int WN = TILE == 1 ? 2 : GROUPED ? 8 : 4;
    static constexpr int MT = TILE == 2 || TILE == 4 ? 4 : TILE == 6 ? 3 : 2;
    static constexpr int NT = GROUPED ? 1 : 2;
    static constexpr int BN = WN * NT * 32;
    static constexpr int BM = WAVES / WN * MT * 32;
    static_assert(BN == 256 || BN == 128, "whole or half width");
    static_assert(BM == 256 || BM == 128 || (BM == 64 && TILE == 5) || (BM == 192 && TILE == 6),
                  "whole, half, quarter or three-quarter height");
    static constexpr int XSTAGE = BM * 128;               // bytes of one activation stage
    static constexpr int XDMA = BM / 8 / WAVES;           // 1 KiB activation DMA loads per wavefront and stage
    static constexpr int WTILES = BN / 32;                        // packed tiles per stage
    static constexpr int WSTAGE = WTILES * FLEXQ_TILE_BYTES;
    static constexpr int XA = TILE == 2 ? 1 : 2;                  // activation stages requested ahead
    static constexpr int XBUFS = XA + 1;
    static constexpr int WBASE = XBUFS * XSTAGE;
    // This wavefront's weight DMA loads per stage: plane p of a stage is fetched by
    // wavefront p % 4.  Wavefronts 0 .. 3 fetch all the weights: the two wavefronts of a SIMD
    // do not advance alike -- the older one (0 .. 3) wins the arbitration, runs ahead and
    // waits at the stage's barrier for the younger one, whose instruction stream sets the
    // pace -- and these loads are work that can move to the wavefronts that have the time
    // (measured A/B: about 1 % at 2048 and 4096 tokens, 3 % on the half tiles; moving the
    // activations' loads as well loses 1.3 %: eight more loads in a row per wavefront).
    static constexpr int WISSUERS = 4;
    static_assert(3 * WTILES % WISSUERS == 0, "equal shares");
    static constexpr int WDMA_LOW = 3 * WTILES / WISSUERS;               // wavefronts below WDMA_SPLIT
    static constexpr int WDMA_HIGH = 0;                                  // the others
    static constexpr int WDMA_SPLIT = WISSUERS;
    // Epilogue staging, 32 rows of fp16 per wavefront: it begins where the THIRD weight
    // stage does.  While a tile is stored, the next item's first stages are landing in
    // the activation stages below XA and in weight stages 0 and 1; weight stage 2 and what
    // lies beyond it are free until the next item's stage 0 asks for the weights of its
    // stage 2, after the barrier that ends the epilogue.
    static constexpr int STG = WBASE + 2 * WSTAGE;
    static constexpr int ESTRIDE = NT * 64 + 16;
    static constexpr int STG_END = STG + WAVES * 32 * ESTRIDE;
    // Group tiles: the scales of a stage follow everything else, a ring of four slots.
    static constexpr int SRING = STG_END > WBASE + 3 * WSTAGE ? STG_END : WBASE + 3 * WSTAGE;
    static constexpr int SSLOT = BN * 2 + 256;                    // weight scales, 128 token scales
    static constexpr int SF32 = SRING + 4 * SSLOT;                // the current stage's weight scales in fp32
    static constexpr int LDS_BYTES = GROUPED ? SF32 + BN * 4 : SRING;
    static_assert(LDS_BYTES + 1024 <= 160 * 1024, "LDS of one CU (plus the static part)");
};

// One item of a workgroup's list: stages [ks, ke) of the 256-wide tile `t256`
// (its half `half` when the items are half tiles); `tj` numbers the tile within a cut tail.
struct Item {
    int t256, half, ks, ke, tj;
};

// The stages of one item of group tiles: every 128-k stage's int32 sums, exact, are folded
// into the fp32 accumulators as acc = fma(float(sum), sw[n][g], acc), or, with scales on both
// operands, fma(float(sum) * sw[n][g], sx[m][g], acc).
//
// That is two (three) vector operations per accumulator and stage beside a quarter of an MFMA:
// the vector unit bounds this mode, and what the kernel can do is to keep it busy from the
// first stage to the last and to use cheap operations.  Eight wavefronts side by side, 128 x 32
// each, expand a weight operand once for four MFMAs (64 x 64 each would expand twice as
// often).  A block's four MFMAs are slots 4b .. 4b + 3, and quarter q of block c is scaled in
// slot 4c + q + 5, when its last MFMA has surely finished; three block buffers rotate (two, and
// a slot earlier, with scales on both operands, which need the registers).  Activation
// operands are read one block ahead, the next stage's weights and scales after the hand-over
// that opens the last block; the weight operand of a k-step is overwritten as soon as the last
// block has used it.
// The scaling avoids the slower operations of this machine: int -> float conversions, mixed-
// precision multiply-adds and any operand from a scalar register take twice the time of plain
// fp32 adds and multiply-adds on vector registers.  So the MFMA chain starts from the bits of
// 1.5 * 2^23 instead of zero -- the sum, read as a float, is then that constant plus the exact
// integer (at most 2^21 in magnitude), and one add takes the constant off -- and the weight
// scales are converted once per stage and wavefront, through LDS.  (With scales on both
// operands the constant could come off inside the multiplication, fma(bits, sw, -constant * sw),
// which is exact and saves one operation, 4 to 9 % on whole tiles, nothing on half ones: but an
// infinite scale then meets its own product, and the result is NaN instead of that infinity.)
// Measured against 128 x 128 tiles of four wavefronts, two workgroups a CU (conversions and
// mixed multiply-adds): 4096 x 8192 x 8192 297 us against 336; without any DMA it takes 268:
// the instruction stream and the clock it runs at are the bound.
//
// The half height, 64 x 256 with two blocks a stage and the same slots, is for layers that leave
// the chip short of items: it takes three quarters of a whole item's time (the expansion and
// the hand-over stay), but cuts the tokens, not the sums.  Cutting K of the last round's tiles alone
// was up to a fifth faster still (13824 x 5120 at 2048 tokens 172 us against 193), but then rows of
// one call were summed in one chain or in pieces by where they lay; where a layer has no whole
// round, group_split cuts all of its tiles alike.  LLaMA-2-13B's down projection at 2048 tokens 193
// us against 211, with scales on both operands 229 against 266, at 700 tokens, unsplit, 93 against 124.
template <int TILE, int GROUP, class DmaX, class DmaW, class DmaS>
__device__ __forceinline__ void group_item(v16f (&facc)[Shape<TILE>::MT][1], uint8_t *lds, int KN, int wave, int lane,
                                           const DmaX &dma_x, const DmaW &dma_w, const DmaS &dma_s)
{
    using S = Shape<TILE>;
    constexpr int MT = S::MT, NB = S::MT;
    static_assert(S::NT == 1 && (MT == 4 || MT == 2) && S::XBUFS == 3, "the slot tables below are written for these");
    const int arow = lane & 31, ahalf = lane >> 5;
    const int wfrag = S::WBASE + wave * FLEXQ_TILE_BYTES + lane * 16;

    PackedTile w;                      // the packed planes whose operands are not all expanded yet
    v4i bf[4], af[2][4];               // weight operands of the stage; activation operands of two blocks
    // int32 sums of the block in flight and of those before it that are not folded in yet
    constexpr int PB = GROUP == 2 ? 2 : 3;
    v16i part[PB];
    v4f sw[4];                         // this lane's sixteen channels' scales
    uint16_t sx_next[MT];              // GROUP == 2: this lane's token's scale of each block
    float sx[MT];
    // Constants in vector registers: an operand from a scalar register halves the rate.
    v16i magic;
    float minus_magic = -12582912.0f;
    int top6 = (int)0xFCFCFCFC, low2 = 0x03030303;
    asm volatile("" : "+v"(minus_magic), "+v"(top6), "+v"(low2));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        int m = 0x4B400000;
        asm volatile("" : "+v"(m));
        magic[r] = m;
    }
    auto read_planes = [&](int buf) {
        const v4i *t = reinterpret_cast<const v4i *>(lds + wfrag + buf * S::WSTAGE);
        w.q0 = t[0];
        w.q1 = t[64];
        w.q2 = t[128];
    };
    auto fourth = [&](int d) {          // a dword of the fourth k-step's operand
        int r = w.q0[d] & low2;
        r = (r << 2) | (w.q1[d] & low2);
        r = (r << 2) | (w.q2[d] & low2);
        return r << 2;
    };
    // the weight scales of stage kb from the ring to this wavefront's fp32 copy, in two halves
    auto scale_bits = [&](int kb) {
        return *reinterpret_cast<const uint16_t *>(lds + S::SRING + (kb & 3) * S::SSLOT + wave * 64 + 2 * arow);
    };
    float *const sw32 = reinterpret_cast<float *>(lds + S::SF32) + 32 * wave;
    auto read_sx = [&](int kb) {
        const uint8_t *slot = lds + S::SRING + (kb & 3) * S::SSLOT + S::BN * 2;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            sx_next[mt] = *reinterpret_cast<const uint16_t *>(slot + (32 * mt + arow) * 2);
    };
    auto read_act = [&](const uint8_t *xs, int mt, int j) {
        return *reinterpret_cast<const v4i *>(xs + lds_off(arow + 32 * mt, 2 * j + ahalf));
    };
    // quarter q of block mt, sums in p, folded in with the scales in registers
    auto scale = [&](const v16i &p, int mt, int q) {
        float f[4], t[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) f[r] = __int_as_float(p[4 * q + r]) + minus_magic;
        // (all four before the first is used: a dependent pair back to back waits)
        asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
        if (GROUP == 2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) f[r] *= sw[q][r];
            asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            t[r] = __builtin_fmaf(f[r], GROUP == 2 ? sx[mt] : sw[q][r], facc[mt][0][4 * q + r]);
        // (an empty statement that uses the results keeps the scaling in its slot)
        asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
#pragma unroll
        for (int r = 0; r < 4; ++r) facc[mt][0][4 * q + r] = t[r];
    };

    read_planes(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) af[0][j] = read_act(lds, 0, j);
    sw32[arow] = h2f(scale_bits(0));
    bf[0] = w.q0 & top6;
    bf[1] = w.q1 & top6;
#pragma unroll
    for (int i = 0; i < PB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[i][r] = 0;
    // "the stage before the first": finite sums times zero
#pragma unroll
    for (int q = 0; q < 4; ++q) sw[q] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sx[mt] = 0.0f;

    // STEADY: two more stages follow for certain (no branches but the wavefront's share of DMA)
    auto stage = [&](int kb, auto cur_tag, auto steady_tag) {
        constexpr int CUR = decltype(cur_tag)::value;      // kb % 3: the stage buffers it reads
        constexpr int NXT = (CUR + 1) % 3, NXT2 = (CUR + 2) % 3;
        constexpr bool STEADY = decltype(steady_tag)::value;
        const bool more1 = STEADY || kb + 1 < KN, more2 = STEADY || kb + 2 < KN;
        const uint8_t *xs = lds + CUR * S::XSTAGE, *xn = lds + NXT * S::XSTAGE;
        uint16_t sw_bits = 0;
#pragma unroll
        for (int s = 0; s < 4 * NB; ++s) {
            const int b = s >> 2, j = s & 3;
            if (s == 4 * NB - 4) {
                // stage kb + 1 (every wavefront's share) must have landed; the loads for stage
                // kb + 2 may be in flight.  Behind the barrier nobody reads this stage's buffers.
                if (!more2)
                    wait_vmcnt<0>();
                else if (wave < S::WDMA_SPLIT)
                    wait_vmcnt<S::XDMA + S::WDMA_LOW>();
                else if (wave < (GROUP == 2 ? 7 : 6))
                    wait_vmcnt<S::XDMA + 1>();
                else
                    wait_vmcnt<S::XDMA>();
                lds_barrier();
                if (more1) read_planes(NXT);
                __builtin_amdgcn_sched_barrier(0);
            }
            const int buf = (CUR * NB + b) % PB;
            part[buf] = mfma_i8(bf[j], af[b & 1][j], j == 0 ? magic : part[buf]);
            if (s == 0 && more2) dma_x(kb + 2, NXT2);
            if (s == 3 && more2) {
                dma_w(kb + 2, NXT2);
                dma_s(kb + 2);
            }
            if (b + 1 < NB) {
                if (j < 2) {
                    af[(b + 1) & 1][2 * j] = read_act(xs, b + 1, 2 * j);
                    af[(b + 1) & 1][2 * j + 1] = read_act(xs, b + 1, 2 * j + 1);
                }
            } else if (more1 && (j == 1 || j == 2)) {
                af[0][2 * (j - 1)] = read_act(xn, 0, 2 * (j - 1));
                af[0][2 * (j - 1) + 1] = read_act(xn, 0, 2 * (j - 1) + 1);
                if (j == 1) sw_bits = scale_bits(kb + 1);
            }
            // the quarter that is due; blocks before this stage's first belong to the one
            // before.  Its scales serve up to slot 4; behind the last use of a quarter's the
            // new ones are read, due four slots later.
            {
                const int c = PB == 2 || j != 0 ? b - 1 : b - 2, q = PB == 2 ? j : j == 0 ? 3 : j - 1;
                scale(part[(CUR * NB + c + 3 * PB) % PB], (c + NB) % NB, q);
            }
            constexpr int S0 = PB == 2 ? 0 : 1;        // the slot of the last use of the first quarter's
            if (s >= S0 && s < S0 + 4) {
                sw[s - S0] = *reinterpret_cast<const v4f *>(sw32 + 8 * (s - S0) + 4 * ahalf);
            }
            if (GROUP == 2) {
                if (s == 1) read_sx(kb);
                if (s == 3) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        sx[mt] = h2f(sx_next[mt]);
                        // (opaque: else the conversion moves into the multiply-adds, mixed
                        // precision then, at twice the time each)
                        asm volatile("" : "+v"(sx[mt]));
                    }
                }
            }
            // weight operands: the fourth k-step's, dearer, over the first three slots of its
            // stage; the next stage's first two once the last block has used this stage's
            if (s == 0) bf[2] = w.q2 & top6;
            if (s < 2) bf[3][s] = fourth(s);
            if (s == 2) {
                bf[3][2] = fourth(2);
                bf[3][3] = fourth(3);
            }
            if (s == 4 * NB - 2) bf[0] = w.q0 & top6;
            if (s == 4 * NB - 1) {
                bf[1] = w.q1 & top6;
                if (more1) sw32[arow] = h2f(sw_bits);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int kb = 0;
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    for (; kb + 5 <= KN; kb += 3) {
        stage(kb, c0, std::true_type{});
        stage(kb + 1, c1, std::true_type{});
        stage(kb + 2, c2, std::true_type{});
    }
    if (kb < KN) stage(kb, c0, std::false_type{});
    if (kb + 1 < KN) stage(kb + 1, c1, std::false_type{});
    if (kb + 2 < KN) stage(kb + 2, c2, std::false_type{});
    if (kb + 3 < KN) stage(kb + 3, c0, std::false_type{});
    // still unscaled: the last quarter of the block before the last, and the last block
    const int last = (KN * NB - 1) % PB, before = (KN * NB - 2) % PB;
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        if (PB == 3 && i == before) scale(part[i], NB - 2, 3);
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        if (i == last) {
#pragma unroll
            for (int q = 0; q < 4; ++q) scale(part[i], NB - 1, q);
        }
    }
}

// One phase of a launch: this workgroup's share of `item_count` items that begin at the
// 256-wide tile `item_begin` -- whole tiles (TILE = 2), half tiles (two items per tile),
// or, with SK, the stages of `item_count` tiles cut into `tail_wgs` runs.
// GROUP (group tiles only): 1 = weight scales per 128-k group, one scale per token; 2 = both
// operands' scales per group.
// YPOLICY, WPOLICY: cache policies of the outputs' stores and of the weights' DMA loads (the latter
// with per-channel scales).
template <int TILE, int SK, int GROUP = 0, int YPOLICY = 0, int WPOLICY = 0>
__device__ __forceinline__ void run_items(const flexq::LinearArgs &a, uint8_t *lds, int &s_last, int tiles_m,
                                          int tiles_n, int item_begin, int item_count, int tail_wgs)
{
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-resource builtins exist in the device pass only
    using S = Shape<TILE>;
    constexpr int MT = S::MT, NT = S::NT;
    constexpr bool WHOLE = S::BN == 256;
    static_assert(!SK || WHOLE, "the tail is cut in whole-width tiles");
    static_assert((GROUP != 0) == S::GROUPED && !(GROUP && SK == 1), "group scales run group tiles");
    static_assert(SK != 3 || (GROUP && NT == 1), "pairs of pieces are group tiles");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / S::WN, wn = wave % S::WN;
    const int M = a.M, N = a.N, K = a.K;
    const int KT = K / FLEXQ_TILE_K;

    // Workgroups 8 apart share an XCD.  Every XCD takes a contiguous share of the items
    // (or of the tail's runs), so the workgroups of one XCD work on neighbouring tiles
    // and find each other's operand panels in their L2.
    const int G = (int)gridDim.x;
    const int xcd = (int)(blockIdx.x % 8), slot = (int)(blockIdx.x / 8);
    int j_next = 0, j_end = 0;                      // !SK: this workgroup's items j_next, j_next + G/8, ...
    long u0 = 0, u1 = 0;                            // SK: this workgroup's run of stages
    int vt = -1;
    int j_stride = 0, pair_ks = 0, pair_ke = 0;     // SK == 3: this workgroup's stages of every tile of its own
    const long U = (long)item_count * KT;           // SK: 128-k stages of the tail
    if (!SK) {
        j_next = (int)((long)xcd * item_count / 8) + slot;
        j_end = (int)((long)(xcd + 1) * item_count / 8);
    } else if (SK == 3) {
        // an XCD's tiles, twice: their first pieces among its first workgroups, `tail_wgs` & 255 each,
        // their second pieces among the next ones, tail_wgs >> 8 each
        const int begin = (int)((long)xcd * item_count / 8), end = (int)((long)(xcd + 1) * item_count / 8);
        const int a1 = tail_wgs & 255, a2 = tail_wgs >> 8;
        const int n1 = (end - begin + a1 - 1) / a1, n2 = (end - begin + a2 - 1) / a2;
        const bool first = slot < n1;
        j_stride = first ? n1 : n2;
        j_next = begin + (first ? slot : slot - n1);
        j_end = slot < n1 + n2 ? end : begin;
        pair_ks = first ? 0 : item_begin;
        pair_ke = first ? item_begin : KT;
    } else {
        const int per = tail_wgs / 8, rem = tail_wgs % 8;
        if (slot < per + (xcd < rem ? 1 : 0)) vt = xcd * per + min(xcd, rem) + slot;
        if (vt >= 0) {
            u0 = (long)vt * U / tail_wgs;
            u1 = (long)(vt + 1) * U / tail_wgs;
        }
    }
    const long run_begin = u0;
    // the next item of this workgroup, if any (all values wavefront-uniform)
    auto take = [&](Item &it) -> bool {
        if (!SK) {
            if (j_next >= j_end) return false;
            const int j = j_next;
            j_next += G / 8;
            it.t256 = item_begin + (WHOLE ? j : j >> 1);
            it.half = WHOLE ? 0 : (j & 1);
            it.ks = 0;
            it.ke = KT;
            it.tj = 0;
            return true;
        } else if (SK == 3) {
            if (j_next >= j_end) return false;
            it.t256 = it.tj = j_next;
            j_next += j_stride;
            it.half = 0;
            it.ks = pair_ks;
            it.ke = pair_ke;
            return true;
        } else {
            if (u0 >= u1) return false;
            it.tj = (int)(u0 / KT);
            it.ks = (int)(u0 - (long)it.tj * KT);
            it.ke = (int)min((long)KT, it.ks + (u1 - u0));
            it.t256 = item_begin + it.tj;
            it.half = 0;
            u0 += it.ke - it.ks;
            return true;
        }
    };

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.xq, 0, (unsigned)((long)M * K), 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.packed, 0, (unsigned)((long)N * K / 4 * 3), 0x00020000);

    // ---- where an item's operands are, and the DMA loads of one stage -----------
    // The 32 tiles an XCD works on at a time share operand panels in its L2: a block of
    // 4 tiles along m x 8 along n fetches the fewest bytes (4 activation panels of 2 MB
    // per 8192 of K + 8 weight panels of 1.5 MB).
    struct Where {
        int bm0, bn0;
        unsigned xoff[S::XDMA];
    };
    auto locate = [&](const Item &it, Where &w) {
        int lane_l = lane;        // (opaque: recomputed per item rather than kept live, see the epilogue)
        asm volatile("" : "+v"(lane_l));
        // super-block: 4 tiles along m (8 of half the height, 16 of a quarter), then next n
        constexpr int SUP_M = TILE == 5 ? 16 : GROUP ? 8 : 4;
        const int bid = it.t256;
        const int sup = bid / (SUP_M * tiles_n);
        const int first_m = sup * SUP_M;
        const int span_m = min(SUP_M, tiles_m - first_m);
        const int in_sup = bid - sup * SUP_M * tiles_n;
        w.bm0 = (first_m + in_sup % span_m) * S::BM;
        w.bn0 = (in_sup / span_m) * 256 + it.half * S::BN;
#pragma unroll
        for (int i = 0; i < S::XDMA; ++i) {
            const int q = wave * S::XDMA + i;
            const int row = 8 * q + (lane_l >> 3);
            const int c = (lane_l & 7) ^ ((row >> 1) & 7);
            w.xoff[i] = (unsigned)(w.bm0 + row) * (unsigned)K + 16u * c;
        }
    };
    // activations: global -> LDS by DMA; rows beyond M read as zero (stage numbers count from ks)
    auto dma_x = [&](const Where &w, int ks, int kb, int buf) {
#pragma unroll
        for (int i = 0; i < S::XDMA; ++i) {
            uint8_t *dst = lds + buf * S::XSTAGE + (wave * S::XDMA + i) * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                xrsrc, (void __attribute__((address_space(3))) *)dst, 16, w.xoff[i],
                (ks + kb) * FLEXQ_TILE_K, 0, 0);
        }
    };
    // packed weights: the stage's WTILES tiles of three 1 KiB planes go into LDS exactly as
    // they lie in memory; plane p of the stage is fetched by wavefront p % 4.  The SGPR
    // offset is not range-checked: tiles past the last row block re-read the last one and
    // are never stored.
    const unsigned wlane = (unsigned)lane * 16u;
    auto dma_w = [&](const Where &w, int ks, int kb, int buf) {
        if constexpr (GROUP != 0) {
            // (whole tiles per wavefront: the planes are immediate offsets of one address)
            if (wave < S::WISSUERS) {
#pragma unroll
                for (int i = 0; i < S::WTILES / S::WISSUERS; ++i) {
                    const int t = wave * (S::WTILES / S::WISSUERS) + i;
                    const int wtile = min(w.bn0 / 32 + t, N / 32 - 1);
                    void __attribute__((address_space(3))) *dst =
                        (void __attribute__((address_space(3))) *)(lds + S::WBASE + buf * S::WSTAGE +
                                                                   t * FLEXQ_TILE_BYTES);
                    const unsigned soff = (unsigned)(wtile * KT + ks + kb) * FLEXQ_TILE_BYTES;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrsrc, dst, 16, wlane, soff, 0, 0);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrsrc, dst, 16, wlane, soff, 1024, 0);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrsrc, dst, 16, wlane, soff, 2048, 0);
                }
            }
            return;
        }
#pragma unroll
        for (int p0 = 0; p0 < 3 * S::WTILES; p0 += S::WISSUERS) {
            const int p = p0 + wave;
            if (wave < S::WISSUERS) {
                const int t = p / 3, plane = p - 3 * t;
                const int wtile = min(w.bn0 / 32 + t, N / 32 - 1);
                uint8_t *dst = lds + S::WBASE + buf * S::WSTAGE + p * 1024;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    wrsrc, (void __attribute__((address_space(3))) *)dst, 16, wlane,
                    (unsigned)(wtile * KT + ks + kb) * FLEXQ_TILE_BYTES + 1024u * plane, 0, WPOLICY);
            }
        }
    };
    // Group tiles: the stage's scales, two bytes each, by 4-byte DMA loads into a ring of four
    // slots: the eight weight tiles' 32 scales each (wavefronts 4 and 5, four tiles a load)
    // and, with group-wise token scales, the 128 rows' (wavefront 6).
    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.scales, 0, GROUP ? (unsigned)((long)N * KT * 2) : 0u, 0x00020000);
    const __amdgpu_buffer_rsrc_t xsrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(GROUP == 2 ? a.sxg : a.scales), 0, GROUP == 2 ? (unsigned)((long)KT * a.sxg_stride * 2) : 0u,
        0x00020000);
    auto dma_s = [&](const Where &w, int ks, int kb) {
        if constexpr (GROUP != 0) {
            uint8_t *slot = lds + S::SRING + (kb & 3) * S::SSLOT;
            if (wave == 4 || wave == 5) {
                const int t = 4 * (wave - 4) + (lane >> 4);
                const int wtile = min(w.bn0 / 32 + t, N / 32 - 1);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    srsrc, (void __attribute__((address_space(3))) *)(slot + (wave - 4) * 256), 4,
                    (unsigned)wtile * (unsigned)KT * 64u + (unsigned)(lane & 15) * 4u, (unsigned)(ks + kb) * 64u, 0, 0);
            }
            if (GROUP == 2 && wave == 6) {
                // (a pair of rows beyond M: an offset past the buffer reads as zero)
                const int row = w.bm0 + 2 * lane;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    xsrsrc, (void __attribute__((address_space(3))) *)(slot + S::BN * 2), 4,
                    row < M ? (unsigned)row * 2u : 0x80000000u,
                    (unsigned)(ks + kb) * (unsigned)a.sxg_stride * 2u, 0, 0);
            }
        }
    };
    // weights and activations of an item's stage 0, weights (and, where activations run
    // two stages ahead, activations) of its stage 1
    auto issue_prologue = [&](const Item &it, const Where &w) {
        dma_w(w, it.ks, 0, 0);
        dma_x(w, it.ks, 0, 0);
        dma_s(w, it.ks, 0);
        if (it.ke - it.ks > 1) {
            dma_s(w, it.ks, 1);
            dma_w(w, it.ks, 1, 1);
            if (S::XA == 2) dma_x(w, it.ks, 1, 1);
        }
    };

    const int arow = (wm * MT) * 32 + (lane & 31);
    const int ahalf = lane >> 5;
    const int wfrag = S::WBASE + (wn * NT) * FLEXQ_TILE_BYTES + lane * 16;   // this lane's piece of tile nt = 0

    Item cur;
    Where at;
    if (!take(cur)) return;
    locate(cur, at);
    issue_prologue(cur, at);
    wait_vmcnt<0>();
    lds_barrier();

    for (;;) {
        const int ks = cur.ks, KN = cur.ke - cur.ks;

        // int32 sums of 4 x the product, or (group scales) fp32 sums of the scaled group sums
        std::conditional_t<GROUP != 0, v16f, v16i> acc[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0;

        if constexpr (GROUP != 0) {
            group_item<TILE, GROUP>(acc, lds, KN, wave, lane, [&](int kb, int buf) { dma_x(at, ks, kb, buf); },
                              [&](int kb, int buf) { dma_w(at, ks, kb, buf); },
                              [&](int kb) { dma_s(at, ks, kb); });
        } else {
            // operands that live across stages: the stage's packed tiles, the activation
            // operands of two consecutive k-steps, the first weight operand of a stage
            PackedTile wreg[NT];
            v4i af[2][MT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const v4i *t = reinterpret_cast<const v4i *>(lds + wfrag + nt * FLEXQ_TILE_BYTES);
                wreg[nt].q0 = t[0];          // the other two planes follow at the start of the stage
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                af[0][mt] = *reinterpret_cast<const v4i *>(lds + lds_off(arow + 32 * mt, ahalf));
            v4i bf_first = unpack_kstep(wreg[0], 0);

            // One 128-k stage.  CUR = kb % XBUFS names the activation buffer (a constant, so that
            // the operand reads use immediate offsets), wcur = kb % 3 the weight buffer.
            // The MFMA takes the WEIGHT fragment as its row operand: the accumulators hold D^T.
            int wcur = 0;
            auto stage = [&](int kb, auto cur_tag) {
                constexpr int CUR = decltype(cur_tag)::value;
                const bool more1 = kb + 1 < KN, more2 = kb + 2 < KN;
                const int wnext = wcur == 2 ? 0 : wcur + 1, wnext2 = wcur == 0 ? 2 : wcur - 1;
                // First what the hand-over waits for (with everything older, the weights of
                // stage kb + 1 among it): the activations of stage kb + 1, where they run one
                // stage ahead.  Then, during step 3, what may stay in flight across it: the
                // loads for stage kb + 2.  All targets are free: an activation buffer was
                // last read before the previous stage's barrier, and the weight buffer is that
                // of stage kb - 1, whose last plane went to registers during that stage's first
                // k-step, before its barrier.
                if (S::XA == 1 && more1) dma_x(at, ks, kb + 1, (CUR + 1) % S::XBUFS);
                if (S::XA == 2 && more2) dma_x(at, ks, kb + 2, (CUR + 2) % S::XBUFS);

                const uint8_t *xs = lds + CUR * S::XSTAGE;
                const uint8_t *xn = lds + ((CUR + 1) % S::XBUFS) * S::XSTAGE;
                const uint8_t *wcb = lds + wfrag + wcur * S::WSTAGE;
                const uint8_t *wnb = lds + wfrag + wnext * S::WSTAGE;
                wcur = wnext;
                // The packed planes of this stage's tiles not yet in registers: only plane 0 (the
                // first k-step) is fetched after the hand-over, plane 1 during step 0 and plane 2
                // during step 1, well before the steps that expand them.
                auto rest_of_tiles = [&](int plane) {
#pragma unroll
                    for (int n2 = 0; n2 < NT; ++n2) {
                        const v4i *t = reinterpret_cast<const v4i *>(wcb + n2 * FLEXQ_TILE_BYTES);
                        if (plane == 1) wreg[n2].q1 = t[64];
                        if (plane == 2) wreg[n2].q2 = t[128];
                    }
                };
                // At the hand-over stage kb + 1 (weights and activations, every wavefront's
                // share) must have landed; the loads for stage kb + 2 may be in flight.
                auto hand_over = [&] {
                    constexpr int XFLY = S::XA == 2 ? S::XDMA : 0;
                    if (!more2)
                        wait_vmcnt<0>();
                    else if (wave < S::WDMA_SPLIT)
                        wait_vmcnt<XFLY + S::WDMA_LOW>();
                    else
                        wait_vmcnt<XFLY + S::WDMA_HIGH>();
                    lds_barrier();
                    if (more1) {
#pragma unroll
                        for (int n2 = 0; n2 < NT; ++n2) {
                            const v4i *t = reinterpret_cast<const v4i *>(wnb + n2 * FLEXQ_TILE_BYTES);
                            wreg[n2].q0 = t[0];
                        }
                    }
                };
                static_assert((MT == 4 || MT == 3 || MT == 2) && NT == 2, "the step tables below are written for these blockings");
                if constexpr (MT == 2) {
                    // 64 x 64 per wavefront: eight steps of two MFMAs, two dwords of the next
                    // step's operand expanded per MFMA; the dearer operands of the fourth k-step
                    // (steps 6 and 7) are spread over steps 2..5, one dword per MFMA
                    v4i bfc = bf_first, bf6 = {0, 0, 0, 0}, bf7 = {0, 0, 0, 0};
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        const int j = s >> 1, nt = s & 1;
                        if (nt == 0) {
                            if (j < 3) {
#pragma unroll
                                for (int mt = 0; mt < MT; ++mt)
                                    af[(j + 1) & 1][mt] = *reinterpret_cast<const v4i *>(
                                        xs + lds_off(arow + 32 * mt, 2 * (j + 1) + ahalf));
                                if (j == 0) rest_of_tiles(1);
                            } else {
                                hand_over();
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (s == 1) {
                            rest_of_tiles(2);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (s == 3 && more2) {
                            dma_w(at, ks, kb + 2, wnext2);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (s == 7 && more1) {   // the next stage's first activation operands
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt)
                                af[0][mt] = *reinterpret_cast<const v4i *>(xn + lds_off(arow + 32 * mt, ahalf));
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        const v4i cur_b = s == 6 ? bf6 : s == 7 ? bf7 : bfc;
                        v4i nxt = bfc;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            acc[mt][nt] = mfma_i8(cur_b, af[j & 1][mt], acc[mt][nt]);
#pragma unroll
                            for (int d = 2 * mt; d < 2 * mt + 2; ++d) {
                                if (s < 5) nxt[d] = unpack_kstep_dword(wreg[(s + 1) & 1], (s + 1) >> 1, d);
                                if (s == 7) nxt[d] = unpack_kstep_dword(wreg[0], 0, d);   // the next stage's first
                            }
                            if (s == 2) bf6[mt] = unpack_kstep_dword(wreg[0], 3, mt);
                            if (s == 3) bf6[2 + mt] = unpack_kstep_dword(wreg[0], 3, 2 + mt);
                            if (s == 4) bf7[mt] = unpack_kstep_dword(wreg[1], 3, mt);
                            if (s == 5) bf7[2 + mt] = unpack_kstep_dword(wreg[1], 3, 2 + mt);
                            {
                                int p0 = nxt[2 * mt], p1 = nxt[2 * mt + 1], p2 = bf6[(s & 1) * 2 + mt],
                                    p3 = bf7[(s & 1) * 2 + mt];
                                asm volatile("" : "+v"(p0), "+v"(p1), "+v"(p2), "+v"(p3));   // pins the expansion here
                                nxt[2 * mt] = p0;
                                nxt[2 * mt + 1] = p1;
                                bf6[(s & 1) * 2 + mt] = p2;
                                bf7[(s & 1) * 2 + mt] = p3;
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        bfc = nxt;
                    }
                    bf_first = bfc;
                } else {
                    v4i bfc = bf_first, bf6, bf7;
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        const int j = s >> 1, nt = s & 1;
                        if (nt == 0) {
                            if (j < 3) {
#pragma unroll
                                for (int mt = 0; mt < MT; ++mt)
                                    af[(j + 1) & 1][mt] = *reinterpret_cast<const v4i *>(
                                        xs + lds_off(arow + 32 * mt, 2 * (j + 1) + ahalf));
                                if (j == 0) rest_of_tiles(1);
                            } else {
                                hand_over();
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (s == 1) {
                            rest_of_tiles(2);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (s == 3 && more2) {
                            dma_w(at, ks, kb + 2, wnext2);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (s == 7 && more1) {   // the next stage's first activation operands
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt)
                                af[0][mt] = *reinterpret_cast<const v4i *>(xn + lds_off(arow + 32 * mt, ahalf));
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        const v4i cur_b = s == 6 ? bf6 : s == 7 ? bf7 : bfc;
                        v4i nxt = bfc;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            acc[mt][nt] = mfma_i8(cur_b, af[j & 1][mt], acc[mt][nt]);
                            // shadow work of this MFMA: one dword of an operand that is due later
                            // (three MFMAs a step: the first has two)
#pragma unroll
                            for (int d = MT == 3 && mt > 0 ? mt + 1 : mt; d < (MT == 3 ? mt + 2 : mt + 1); ++d) {
                                if (s < 5) nxt[d] = unpack_kstep_dword(wreg[(s + 1) & 1], (s + 1) >> 1, d);
                                if (s == 3) bf6[d] = unpack_kstep_dword(wreg[0], 3, d);
                                if (s == 4) bf7[d] = unpack_kstep_dword(wreg[1], 3, d);
                                if (s == 7) nxt[d] = unpack_kstep_dword(wreg[0], 0, d);   // the next stage's first
                                int p0 = nxt[d], p1 = bf6[d], p2 = bf7[d];
                                asm volatile("" : "+v"(p0), "+v"(p1), "+v"(p2));   // pins the expansion here
                                nxt[d] = p0;
                                bf6[d] = p1;
                                bf7[d] = p2;
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        bfc = nxt;
                    }
                    bf_first = bfc;
                }
            };

            int kb = 0;
            for (; kb + S::XBUFS <= KN; kb += S::XBUFS) {
                stage(kb, std::integral_constant<int, 0>{});
                stage(kb + 1, std::integral_constant<int, 1>{});
                if constexpr (S::XBUFS == 3) stage(kb + 2, std::integral_constant<int, 2>{});
            }
            if (kb < KN) stage(kb, std::integral_constant<int, 0>{});
            if (S::XBUFS == 3 && kb + 1 < KN) stage(kb + 1, std::integral_constant<int, 1>{});
        }
        // (every wavefront has passed the last stage's barrier with its LDS reads done: the
        // stage buffers are free)

        // ---- a run that is not a whole tile: leave the sums, or collect the others' ----
        bool finish = true;                              // this workgroup stores the tile
        unsigned fin_slabs = ~0u;                        // ... these 32-row slabs of each wavefront's part
        const int pieces = SK == 2 ? tail_wgs / item_count : 1;
        if (SK == 2 && KN != KT) {
            // EVEN CUT: every tile is cut into the same number of pieces, one per workgroup,
            // which therefore reach the end of their runs together.  The reduction is shared:
            // slab (wavefront w, row block mt) of the tile belongs to piece (w MT + mt) %
            // pieces.  A piece stores the sums of the slabs it does not own, adds its
            // stage count to the tile's counter, waits -- a bounded number of polls -- until
            // the count is complete, adds the other pieces' sums to the slabs it owns and
            // stores those.  No workgroup ever waits without a bound: a piece whose wait runs
            // out (its partners are not resident: a busy or smaller device) stores its own
            // slabs' sums as well, sets its bit in the tile's flag word and leaves; the piece
            // that completed the count closes the tile after its own slabs (one atomic OR)
            // and finishes the slabs of every piece whose bit it finds.  A piece that finds
            // the tile closed when it sets its bit finishes its slabs itself (all sums are
            // there by then).  Each piece ends with one add to the flag word's leave count;
            // the last to leave clears counter and flags for the next call.
            constexpr int kScopeAgent = 16;
            constexpr unsigned kClosed = 1u << 16, kLeave = 1u << 20;
            constexpr int PIECE_BYTES = S::BM * 256 * 4;      // one piece's int32 sums: slot `vt` of the area
            const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(
                a.partial, 0, (unsigned)tail_wgs * (unsigned)PIECE_BYTES, 0x00020000);
            // (the lane number passes through an opaque statement so that nothing derived
            // from it here is computed ahead of the main loop and kept in registers across it)
            int lane_m = lane;
            asm volatile("" : "+v"(lane_m));
            const unsigned in_slot = (unsigned)(wave * (PIECE_BYTES / WAVES) + lane_m * 16);
            const int tj = cur.tj;
            const int me = vt - tj * pieces;
            unsigned *flags = a.counters + 2048;
            auto owner = [&](int mt) { return (wave * MT + mt) % pieces; };      // uniform
            // Slabs of padding tokens alone are not added, and on 256-row tiles and in a single row of low tiles
            // not sent either: layers of K -> N 28672 -> 8192 at 140 tokens 66.1 -> 64.2 us, at 333 101.5 -> 97.8, 8192 ->
            // 10240 at 160 34.1 -> 32.5, 16384 -> 6144 at 66 (low) 30.9 -> 29.8.  Several rows of low tiles send them all
            // the same: without, 14336 -> 4096 at 200 tokens takes 30.6 us instead of 28.4, 11008 -> 4096 at 150 26.4 /
            // 25.0, 4096 -> 4096 at 180 18.2 / 16.7 (why is not known: dealing the slabs that are left evenly to the
            // pieces changes nothing), and left out of the additions alone they cost nothing that shows on 315 cells.
            auto live = [&](int mt) {
                if constexpr (GROUP != 0) return true;      // (those pad by less and gain nothing)
                else return at.bm0 + (wm * MT + mt) * 32 < M;
            };
            auto sent = [&](int mt) {
                if constexpr (TILE == 2 || GROUP != 0) return live(mt);
                else return tiles_m > 1 || live(mt);
            };
            auto store_slab = [&](int mt) {
                const unsigned mine = (unsigned)vt * PIECE_BYTES + in_slot;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        v4u piece;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const auto v = acc[mt][nt][4 * q + c];      // int or float
                            piece[c] = __builtin_bit_cast(unsigned, v);
                        }
                        __builtin_amdgcn_raw_buffer_store_b128(
                            piece, prsrc, mine + (unsigned)(((mt * NT + nt) * 4 + q) * 1024), 0, kScopeAgent);
                    }
            };
            auto load_slab = [&](v4u (&got)[NT * 4], int mt, int from) {
                const unsigned theirs = (unsigned)(tj * pieces + from) * PIECE_BYTES + in_slot;
#pragma unroll
                for (int i = 0; i < NT * 4; ++i)
                    got[i] = __builtin_amdgcn_raw_buffer_load_b128(
                        prsrc, theirs + (unsigned)((mt * NT * 4 + i) * 1024), 0, kScopeAgent);
            };
            auto sum_slab = [&](const v4u (&got)[NT * 4], int mt) {
#pragma unroll
                for (int i = 0; i < NT * 4; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const unsigned v = got[i][c];
                        if constexpr (GROUP != 0)
                            acc[mt][i >> 2][4 * (i & 3) + c] += __uint_as_float(v);
                        else
                            acc[mt][i >> 2][4 * (i & 3) + c] += (int)v;
                    }
            };
            // every other piece's sums of slab mt, the next piece's loads in flight while one
            // piece's sums are added (one round trip in all instead of one per piece).  fp32 sums
            // are added in the order of the pieces, this one's in its place, so that the result
            // does not depend on which piece finishes a slab.
            auto gather_slab = [&](int mt) {
                auto following = [&](int from) {
                    const int n = from + 1;
                    return n == me ? n + 1 : n;
                };
                v4u got_a[NT * 4], got_b[NT * 4];
                v16f own[GROUP ? NT : 1];
                if constexpr (GROUP != 0) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        own[nt] = acc[mt][nt];
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0.0f;
                    }
                }
                auto add_own = [&](int after) {     // this piece's sums follow piece `after`'s
                    if constexpr (GROUP != 0) {
                        if (after == me - 1) {
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] += own[nt];
                        }
                    }
                };
                int from = following(-1);
                load_slab(got_a, mt, from);
                add_own(-1);
                for (;;) {
                    int nxt = following(from);
                    if (nxt < pieces) load_slab(got_b, mt, nxt);
                    sum_slab(got_a, mt);
                    add_own(from);
                    if (nxt >= pieces) break;
                    from = following(nxt);
                    if (from < pieces) load_slab(got_a, mt, from);
                    sum_slab(got_b, mt);
                    add_own(nxt);
                    if (from >= pieces) break;
                }
            };
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                if (owner(mt) != me && sent(mt)) store_slab(mt);
            wait_vmcnt<0>();
            lds_barrier();
            if (tid == 0) {
                const unsigned prev = __hip_atomic_fetch_add(&a.counters[tj], (unsigned)KN, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                bool all = prev + (unsigned)KN == (unsigned)KT;
                const int completed = all ? 1 : 0;
                for (int poll = 0; !all && poll < a.spin; ++poll) {
                    __builtin_amdgcn_s_sleep(8);
                    all = __hip_atomic_load(&a.counters[tj], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                          (unsigned)KT;
                }
                s_last = all ? 1 + completed : 0;
            }
            lds_barrier();
            // 0 gave up, 1 all sums there, 2 and this piece completed the count
            int state = __builtin_amdgcn_readfirstlane(s_last);
            lds_barrier();                       // (read by all before it is written again)
            if (state == 0) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    if (owner(mt) == me && sent(mt)) store_slab(mt);
                wait_vmcnt<0>();
                lds_barrier();
                if (tid == 0) {
                    const unsigned old = __hip_atomic_fetch_or(&flags[tj], 1u << me, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                    s_last = (old & kClosed) ? 1 : 0;
                }
                lds_barrier();
                state = __builtin_amdgcn_readfirstlane(s_last);
                lds_barrier();
            }
            fin_slabs = 0;
            if (state != 0) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    if (owner(mt) == me && live(mt)) {
                        gather_slab(mt);
                        fin_slabs |= 1u << mt;
                    }
                if (state == 2) {
                    if (tid == 0) {
                        const unsigned old = __hip_atomic_fetch_or(&flags[tj], kClosed, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT);
                        s_last = (int)(old & 0xffffu);
                    }
                    lds_barrier();
                    const unsigned gone = (unsigned)__builtin_amdgcn_readfirstlane(s_last);
                    lds_barrier();
                    if (gone != 0) {
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            if (((gone >> owner(mt)) & 1u) && live(mt)) {
                                gather_slab(mt);
                                fin_slabs |= 1u << mt;
                            }
                    }
                }
            }
            if (tid == 0) {
                const unsigned old = __hip_atomic_fetch_add(&flags[tj], kLeave, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                if ((int)(old >> 20) + 1 == pieces) {
                    __hip_atomic_store(&a.counters[tj], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&flags[tj], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            finish = fin_slabs != 0;
        } else if constexpr (SK == 3) {
            // PAIRS: every tile in two pieces at the same stage, run at different times.  Whoever is
            // through first leaves its sums in its own slot and counts; the other, finding the count
            // or bringing it to two, adds them and finishes the tile.  Nobody waits, and of two
            // fp32 sums the order shows nowhere.
            constexpr int kScopeAgent = 16;
            constexpr int PIECE_BYTES = S::BM * 256 * 4;
            const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(
                a.partial, 0, (unsigned)(2 * item_count) * (unsigned)PIECE_BYTES, 0x00020000);
            int lane_m = lane;
            asm volatile("" : "+v"(lane_m));
            const unsigned in_slot = (unsigned)(wave * (PIECE_BYTES / WAVES) + lane_m * 16);
            const int tj = cur.tj, second = ks != 0 ? 1 : 0;
            auto broadcast = [&](auto value) {       // thread 0's answer to everybody
                if (tid == 0) s_last = value();
                lds_barrier();
                const bool yes = __builtin_amdgcn_readfirstlane(s_last) != 0;
                lds_barrier();                       // (read by all before it is written again)
                return yes;
            };
            finish = broadcast([&] {
                return __hip_atomic_load(&a.counters[tj], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u ? 1 : 0;
            });
            if (!finish) {
                const unsigned mine = (unsigned)(2 * tj + second) * PIECE_BYTES + in_slot;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        v4u piece;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const auto v = acc[mt][0][4 * q + c];
                            piece[c] = __builtin_bit_cast(unsigned, v);
                        }
                        __builtin_amdgcn_raw_buffer_store_b128(piece, prsrc, mine + (unsigned)((mt * 4 + q) * 1024), 0,
                                                               kScopeAgent);
                    }
                wait_vmcnt<0>();                     // acknowledged: visible device-wide
                lds_barrier();
                finish = broadcast([&] {
                    return __hip_atomic_fetch_add(&a.counters[tj], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u
                               ? 1 : 0;
                });
            }
            if (finish) {
                if (tid == 0)
                    __hip_atomic_store(&a.counters[tj], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const unsigned theirs = (unsigned)(2 * tj + 1 - second) * PIECE_BYTES + in_slot;
                v4u got[2][4];
                auto load = [&](int mt) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        got[mt & 1][q] = __builtin_amdgcn_raw_buffer_load_b128(
                            prsrc, theirs + (unsigned)((mt * 4 + q) * 1024), 0, kScopeAgent);
                };
                load(0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    if (mt + 1 < MT) load(mt + 1);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const unsigned v = got[mt & 1][q][c];
                            acc[mt][0][4 * q + c] += __uint_as_float(v);
                        }
                }
            }
        } else if constexpr (SK == 1) {
            if (KN != KT) {
                // [slot][wavefront][block mt, nt][quarter][lane] 16-byte pieces: every store and
                // load below is one contiguous KiB per wavefront.  Cache policy bit 4 = sc1 =
                // device scope: the access goes to memory all XCDs share.
                constexpr int kScopeAgent = 16;
                const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(
                    a.partial, 0, (unsigned)(2 * tail_wgs) * (unsigned)SLOT_BYTES, 0x00020000);
                const unsigned in_slot = (unsigned)(wave * (SLOT_BYTES / WAVES) + lane * 16);
                const int tj = cur.tj;
                const long tile_begin = (long)tj * KT;
                // a run leaves at most two partial tiles: slot 2 vt for the one it begins in,
                // 2 vt + 1 for the one it ends in
                const unsigned mine = (unsigned)(2 * vt + (run_begin < tile_begin ? 1 : 0)) * SLOT_BYTES + in_slot;
                // The tile a run ends in is begun by this workgroup and finished by its successor,
                // which reached it first thing: by now it has most likely arrived, and so has
                // everybody else.  One look at the counter tells (it only ever grows until the
                // last arrival; a workgroup adds to it after its stores are acknowledged): then
                // this workgroup is the last without storing its own sums first.
                int early = 0;
                if (run_begin < tile_begin) {
                    if (tid == 0) {
                        const unsigned seen = __hip_atomic_load(&a.counters[tj], __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT);
                        s_last = (seen + (unsigned)KN == (unsigned)KT);
                        if (s_last)
                            __hip_atomic_store(&a.counters[tj], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    lds_barrier();
                    early = __builtin_amdgcn_readfirstlane(s_last);
                }
                if (!early) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const v4u piece = {(unsigned)acc[mt][nt][4 * q], (unsigned)acc[mt][nt][4 * q + 1],
                                                   (unsigned)acc[mt][nt][4 * q + 2], (unsigned)acc[mt][nt][4 * q + 3]};
                                __builtin_amdgcn_raw_buffer_store_b128(
                                    piece, prsrc, mine + (unsigned)(((mt * NT + nt) * 4 + q) * 1024), 0, kScopeAgent);
                            }
                    // Once the stores are acknowledged (vmcnt 0) they are visible device-wide; the
                    // barrier plus one relaxed device-scope add to the tile's stage count publishes
                    // them.  Whoever brings the count to KT is the last and resets it.
                    wait_vmcnt<0>();
                    lds_barrier();
                    if (tid == 0) {
                        const unsigned prev = __hip_atomic_fetch_add(&a.counters[tj], (unsigned)KN, __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_AGENT);
                        s_last = (prev + (unsigned)KN == (unsigned)KT);
                        if (s_last)
                            __hip_atomic_store(&a.counters[tj], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    lds_barrier();
                    finish = __builtin_amdgcn_readfirstlane(s_last) != 0;   // wavefront-uniform
                }
                if (finish) {
                    // the runs that meet this tile: the one holding its first stage through the one
                    // holding its last (run w is [w U / W, (w + 1) U / W))
                    const long W = tail_wgs;
                    const int va = (int)(((tile_begin + 1) * W + U - 1) / U) - 1;
                    const int vb = (int)(((tile_begin + KT) * W + U - 1) / U) - 1;
                    for (int w2 = va; w2 <= vb; ++w2) {
                        if (w2 == vt) continue;
                        const long begin2 = (long)w2 * U / W;
                        const unsigned theirs =
                            (unsigned)(2 * w2 + (begin2 < tile_begin ? 1 : 0)) * SLOT_BYTES + in_slot;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            v4u got[NT * 4];
#pragma unroll
                            for (int i = 0; i < NT * 4; ++i)
                                got[i] = __builtin_amdgcn_raw_buffer_load_b128(
                                    prsrc, theirs + (unsigned)((mt * NT * 4 + i) * 1024), 0, kScopeAgent);
#pragma unroll
                            for (int i = 0; i < NT * 4; ++i)
#pragma unroll
                                for (int c = 0; c < 4; ++c) acc[mt][i >> 2][4 * (i & 3) + c] += (int)got[i][c];
                        }
                    }
                }
            }
        }

        // ---- the next item's first stages set out now, before this tile is stored ----
        Item nxt_item;
        Where nxt_at;
        const bool has_next = take(nxt_item);
        if (has_next) {
            locate(nxt_item, nxt_at);
            issue_prologue(nxt_item, nxt_at);
        }

        // ---- epilogue --------------------------------------------------------------
        // Register r of block (mt, nt) at lane l is token 32 mt' + (l & 31), channel
        // 32 nt' + 8 (r / 4) + 4 (l >> 5) + r % 4: four consecutive channels per register
        // quarter.  Scale (sx[m] * sw[n] in fp32, exact; the 1/4 of the 4x weights folded
        // into sx, a power of two) and convert in registers, pass 8-byte pieces of fp16
        // through this wavefront's own LDS rows (stride NT * 64 + 16 bytes), read 16-byte
        // pieces back so that the lanes of a row hold consecutive pieces, and store whole
        // lines.  Rows beyond M and column blocks beyond N are never stored.
        if (finish) {
            const int bm0 = at.bm0, bn0 = at.bn0;
            // (the lane number passes through an opaque statement: what the epilogue derives
            // from it is recomputed per tile, a handful of operations, instead of being kept
            // in registers -- or spilled -- across the main loop)
            int lane_e = lane;
            asm volatile("" : "+v"(lane_e));
            const int ml = lane_e & 31, hh = lane_e >> 5;
            const int n_wave = bn0 + wn * NT * 32;
            // (kept as packed fp16 and converted where used: sixteen registers, not thirty-two)
            uint2 sw4[NT][4];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const bool cvalid = !GROUP && n_wave + nt * 32 < N;       // uniform; N is a multiple of 32
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n_wave + nt * 32 + 8 * q + 4 * hh;
                    sw4[nt][q] = cvalid ? *reinterpret_cast<const uint2 *>(a.scales + n) : make_uint2(0u, 0u);
                }
            }
            float sxq[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = bm0 + (wm * MT + mt) * 32 + ml;
                if (GROUP == 2)
                    sxq[mt] = 0.25f;
                else
                    sxq[mt] = m < M ? 0.25f * h2f(a.sx[m]) : 0.0f;
            }
            uint8_t *stg = lds + S::STG + wave * (32 * S::ESTRIDE);
            constexpr int LPR = NT * 4;                 // lanes per staged row, 16 bytes (8 channels) each
            constexpr int RPI = 64 / LPR;               // rows per read instruction
            const int erow = lane_e / LPR, echunk = lane_e % LPR;
            const bool ecvalid = n_wave + echunk * 8 < N;
            // the output as a buffer from this wavefront's corner: a lane's offset is fixed,
            // the row offset is an SGPR
            const long corner = (long)(bm0 + wm * MT * 32) * N + n_wave;
            const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(a.y + corner), 0, (unsigned)(((long)(MT * 32 - 1) * N + NT * 32) * 2), 0x00020000);
            const unsigned yoff = (unsigned)((erow * N + echunk * 8) * 2);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m_slab = bm0 + (wm * MT + mt) * 32;
                if (m_slab >= M) break;                          // uniform: nothing below is stored
                if (SK == 2 && !((fin_slabs >> mt) & 1u)) continue;   // uniform: another piece stores this slab
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const unsigned swp[2] = {sw4[nt][q].x, sw4[nt][q].y};
                        uint16_t h[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const float swc = GROUP ? 1.0f : h2f((uint16_t)(swp[c >> 1] >> (16 * (c & 1))));
                            h[c] = f2h((float)acc[mt][nt][4 * q + c] * (sxq[mt] * swc));
                        }
                        uint2 out2;
                        out2.x = (unsigned)h[0] | ((unsigned)h[1] << 16);
                        out2.y = (unsigned)h[2] | ((unsigned)h[3] << 16);
                        *reinterpret_cast<uint2 *>(stg + ml * S::ESTRIDE + (nt * 32 + 8 * q + 4 * hh) * 2) = out2;
                    }
                if constexpr (!GROUP) {
                    if (a.acc_out) {     // the exact int32 sums, straight from the registers
                        const int m = m_slab + ml;
    #pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
    #pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const int n = n_wave + nt * 32 + 8 * q + 4 * hh;
                                if (m < M && n < N) {
                                    const v4i four = {acc[mt][nt][4 * q] >> 2, acc[mt][nt][4 * q + 1] >> 2,
                                                      acc[mt][nt][4 * q + 2] >> 2, acc[mt][nt][4 * q + 3] >> 2};
                                    *reinterpret_cast<v4i *>(a.acc_out + (long)m * N + n) = four;
                                }
                            }
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // own region only: no barrier
#pragma unroll
                for (int i = 0; i < 32 / RPI; ++i) {
                    const int row = i * RPI + erow;
                    const v4u piece = *reinterpret_cast<const v4u *>(stg + row * S::ESTRIDE + echunk * 16);
                    if (m_slab + row < M && ecvalid)
                        __builtin_amdgcn_raw_buffer_store_b128(piece, yrsrc, yoff,
                                                               (unsigned)((mt * 32 + i * RPI) * N * 2), YPOLICY);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // reads done before the next slab overwrites
            }
        }
        if (!has_next) break;
        // the next item's first stages (every wavefront's share) have landed
        wait_vmcnt<0>();
        lds_barrier();
        cur = nxt_item;
        at = nxt_at;
    }
#endif
}

// ONE_ROUND: no workgroup has more than one item.
// FORM 3: `full_count` low tiles (tiles_m counts 128-row tiles) and nothing else.  FORM 6: the
// same with 192-row tiles.  FORM 5:
// `full_count` low tiles, then `tail_count`, each cut along K into tail_wgs / tail_count pieces.
// FORM 0: `full_count` whole tiles.  FORM 1: then the `tail_count` tiles that follow them as
// 2 * tail_count half tiles.  FORM 2: then those tiles cut along K into `tail_wgs` runs
// across tile borders.  FORM 4: then those tiles each cut into tail_wgs / tail_count pieces.
// One launch: a second launch for the tail would cost the first one's drain and the
// end-of-kernel cache write-back in between (about 20 us, measured).
template <int FORM, bool ONE_ROUND = false>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_wlds_kernel(flexq::LinearArgs a, int tiles_m, int tiles_n, int full_count, int tail_count,
                      int tail_wgs)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ int s_last;
    constexpr int YPOLICY = ONE_ROUND ? kLastRound : 0;
    if (FORM == 3) {   // every item a low tile (128 x 256)
        run_items<3, 0, 0, YPOLICY>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
        return;
    }
    if (FORM == 7) {   // the same for one row of tiles, which uses a weight once
        run_items<3, 0, 0, YPOLICY, kNonTemporal>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
        return;
    }
    if (FORM == 6) {   // every item a tile of 192 x 256
        run_items<6, 0, 0, YPOLICY>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
        return;
    }
    if (FORM == 5) {   // whole rounds of low tiles, then the rest cut evenly along K
        if (full_count > 0) {
            run_items<3, 0>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
#if defined(__HIP_DEVICE_COMPILE__)
            lds_barrier();     // as below: the last epilogue's staging rows
#endif
        }
        run_items<3, 2, 0, kLastRound>(a, lds, s_last, tiles_m, tiles_n, full_count, tail_count, tail_wgs);
        return;
    }
    if (full_count > 0) run_items<2, 0, 0, YPOLICY>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
#if defined(__HIP_DEVICE_COMPILE__)
    // The two phases lay LDS out differently: every wavefront must be through with its last
    // epilogue's staging rows before anyone's first loads of the next phase land on them.
    if (FORM != 0) lds_barrier();
#endif
    if (FORM == 1)
        run_items<1, 0, 0, kLastRound>(a, lds, s_last, tiles_m, tiles_n, full_count, 2 * tail_count, 0);
    if (FORM == 2)
        run_items<2, 1, 0, kLastRound>(a, lds, s_last, tiles_m, tiles_n, full_count, tail_count, tail_wgs);
    if (FORM == 4)
        run_items<2, 2, 0, kLastRound>(a, lds, s_last, tiles_m, tiles_n, full_count, tail_count, tail_wgs);
}

// Group tiles, every tile (128 rows high) in two pieces, stages [0, cut) and [cut, K / 128): `per_wg` & 255
// first pieces a workgroup, per_wg >> 8 second pieces.  For layers of one to two rounds of tiles, whose last
// round would leave most of the chip idle: the two pieces' lengths are such that workgroups of either
// kind end together.
template <int GROUP>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_group_pair_kernel(flexq::LinearArgs a, int tiles_m, int tiles_n, int cut, int per_wg)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ int s_last;
    run_items<4, 3, GROUP, kLastRound>(a, lds, s_last, tiles_m, tiles_n, cut, tiles_m * tiles_n, per_wg);
}

// Group tiles (tiles_m counts 128-row tiles): `full_count` whole ones, then `tail_count` of
// shape TAIL: as many of the same (4), or those that follow at half the height (5).  Each of them
// is cut into tail_wgs / tail_count pieces.  TAIL 0: one round of whole ones.
template <int GROUP, int TAIL>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_group_kernel(flexq::LinearArgs a, int tiles_m, int tiles_n, int full_count, int tail_count, int tail_wgs)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ int s_last;
    if constexpr (TAIL == 0) {
        run_items<4, 0, GROUP, kLastRound>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
        return;
    }
    if (full_count > 0) run_items<4, 0, GROUP>(a, lds, s_last, tiles_m, tiles_n, 0, full_count, 0);
    if (tail_count == 0) return;
#if defined(__HIP_DEVICE_COMPILE__)
    lds_barrier();     // the last epilogue's staging rows, as above
#endif
    if constexpr (TAIL == 5)   // tile t is tiles 2 t and 2 t + 1 of half the height, in the same super-block order
        run_items<5, 2, GROUP, kLastRound>(a, lds, s_last, full_count > 0 ? 2 * tiles_m : (a.M + 63) / 64, tiles_n,
                                           2 * full_count, tail_count, tail_wgs);
    if constexpr (TAIL == 4)
        run_items<4, 2, GROUP, kLastRound>(a, lds, s_last, tiles_m, tiles_n, full_count, tail_count, tail_wgs);
}

}  // namespace

namespace flexq {

size_t low_cut_bytes(int pieces_in_all) { return (size_t)pieces_in_all * (128 * 256 * 4); }

// 65 to 128 tokens on a layer too narrow to fill the chip with 128x256 tiles: every tile
// cut along K into this many pieces (0: the form does not apply).  Measured on the
// LLaMA-2-7B and 70B layers at 96 and 128 tokens: fastest with 130 to 190 pieces in all
// (beyond that the partial sums of all pieces, which cross the memory system at the same
// moment, cost more than the shorter runs save) and runs of at least 13 stages; 5-22 %
// faster than 128x128 tiles with K splits in 11 cells of 12.
int low_cut_pieces(int M, int N, int K)
{
    if (M <= 64 || M > 128) return 0;
    const int tiles = (N + 255) / 256, KT = K / FLEXQ_TILE_K;
    int pieces = 176 / tiles;
    if (pieces > KT / 13) pieces = KT / 13;
    if (pieces > 8) pieces = 8;
    return pieces >= 2 ? pieces : 0;
}

StreamKPlan streamk_plan(int M, int N, int K)
{
    StreamKPlan p;
    p.tiles = ((M + 256 - 1) / 256) * ((N + 255) / 256);
    p.full_tiles = p.tiles / kStreamKGrid * kStreamKGrid;
    p.tail_tiles = p.tiles - p.full_tiles;
    // two slots per run; a run is at least one 128-k stage, and there are at most 256 runs
    const long stages = (long)p.tail_tiles * (K / FLEXQ_TILE_K);
    p.partial_bytes = (size_t)2 * (size_t)(stages < kStreamKGrid ? stages : kStreamKGrid) * SLOT_BYTES;
    return p;
}

// Estimated run time in microseconds of the fastest launch form, from measured constants
// of the MI355X.  A 128-k stage of a whole tile takes 1.50 us when every CU has a tile and
// 1.20 us when at most two thirds of them have (the chip is power-limited: idle CUs let
// the others clock higher), a half tile's stage 0.93 / 0.75 us; a tile costs 4 us more for
// its first loads and its epilogue.  Meeting in the workspace costs 7 to 27 us when every
// tile is cut into the same number of pieces (one partial tile per workgroup, the pieces of
// a tile share its reduction); about 45 us when the tail is simply cut into 256 equal
// runs, which then begin and end inside tiles (two partial tiles per workgroup, the last
// to arrive at a tile reads the others').
WldsChoice gemm_wlds_choose(int M, int N, int K, bool may_cut)
{
    const StreamKPlan p = streamk_plan(M, N, K);
    const int KT = K / FLEXQ_TILE_K;
    auto busy = [](double frac) { return frac <= 0.65 ? 0.0 : (frac - 0.65) / 0.35; };
    auto whole_us = [&](int tiles) { return (1.20 + 0.30 * busy(tiles / 256.0)) * KT + 4.0; };
    auto half_us = [&](int halves) { return (0.75 + 0.18 * busy(halves / 256.0)) * KT + 4.0; };
    const double rounds = (double)(p.full_tiles / kStreamKGrid) * whole_us(kStreamKGrid);
    WldsChoice best{rounds + (p.tail_tiles ? whole_us(p.tail_tiles) : 0.0), 0, 0};
    if (p.tail_tiles == 0) return best;
    {   // the tail as half tiles: one half round, or two
        const int halves = 2 * p.tail_tiles;
        const double t = rounds + (halves <= kStreamKGrid ? half_us(halves)
                                                          : half_us(kStreamKGrid) + half_us(halves - kStreamKGrid));
        if (t < best.us) best = WldsChoice{t, 1, halves};
    }
    if (!may_cut) return best;
    const double stage_us = 1.50;
    // every tile cut into S pieces that share its reduction: meeting costs by the pieces
    // per tile (a piece adds S - 1 others' sums) and by their number in all (the partial sums
    // of all pieces cross the memory system at the same moment); measured on the 8192- and
    // 28672-deep layers at 256 .. 3072 tokens, 2 .. 8 pieces per tile, 64 .. 256 in all
    for (int S = 2; S <= 16 && p.tail_tiles * S <= kStreamKGrid && S <= KT; ++S) {
        const int wgs = p.tail_tiles * S;
        const double meet = 1.0 + 2.0 * S + 0.03 * wgs + (wgs > 192 ? 0.03 * (wgs - 192) : 0.0);
        const double t = rounds + (1.15 + 0.35 * busy(wgs / 256.0)) * ((KT + S - 1) / S) + 4.0 + meet;
        if (t < best.us) best = WldsChoice{t, 2, wgs};
    }
    if ((long)p.tail_tiles * KT >= 2L * kStreamKGrid) {
        const double t = rounds + stage_us * KT * p.tail_tiles / kStreamKGrid + 4.0 + 45.0;
        if (t < best.us) best = WldsChoice{t, 2, kStreamKGrid};
    }
    return best;
}

// The same for 128x256 tiles above 128 tokens, where half the height fills the chip more
// evenly: whole (form 3), or those beyond the last whole round of 256 each cut into equal pieces
// (form 5).  A stage takes 0.60 us while at most half of the CUs have a tile and 0.91 us on a
// full chip -- 30 % more for the same work than a 256x256 tile's, which pays for itself where
// that would leave CUs idle.  Fitted on eighteen layers (512 .. 57344 wide, 512 .. 28672 deep)
// at 129 .. 2048 tokens; taken there it gains 5 to 45 % between 129 and 700 tokens (8192 x
// 8192 at 300 tokens: 44.5 -> 34.9 us, 4096 x 4096 at 220: 23.8 -> 16.4).  More than 192 pieces meet at
// little more than fewer do (15360 x 5120 at 129 .. 256 tokens, 240 pieces against 120 whole tiles: 26.7 .. 27.9
// us against 32.8; 16384 x 6144 at 129, 256 pieces: 30.6 against 35.7), but not for one more piece a tile alone
// (13824 x 5120 at 150: 160 pieces 29.1, 200 31.5).
WldsChoice gemm_low_choose(int M, int N, int K, size_t partial_bytes)
{
    const int tiles = ((M + 127) / 128) * ((N + 255) / 256), KT = K / FLEXQ_TILE_K;
    const int tail = tiles % kStreamKGrid;
    auto stage_us = [](int n) { return 0.60 + (n > 128 ? 0.31 * (n - 128) / 128.0 : 0.0); };
    const double rounds = tiles / kStreamKGrid * (stage_us(kStreamKGrid) * KT + 5.0);
    WldsChoice best{rounds + (tail ? stage_us(tail) * KT + 6.5 : 1.5), 3, 0};
    if (tail == 0 || device_cu_count() != kStreamKGrid) return best;
    for (int S = 2; S <= 16 && tail * S <= kStreamKGrid && S <= KT; ++S) {
        const int wgs = tail * S;
        if (partial_bytes < low_cut_bytes(wgs)) break;
        const double meet = 3.0 + 0.4 * S + 0.015 * wgs + (wgs > 192 ? 0.5 + 0.015 * (wgs - 192) : 0.0);
        const double t = rounds + stage_us(wgs) * ((KT + S - 1) / S) + 4.0 + meet;
        if (t < best.us) best = WldsChoice{t, 5, wgs};
    }
    return best;
}

// Estimated microseconds with 192-row tiles, all whole.  A stage takes 0.90 us while at most 150 CUs
// have a tile, 1.32 on a full chip (a 256-row tile's: 1.20, 1.50).  Within 7 % of the time, mostly 3, on
// fourteen layers (2048 .. 57344 wide, 4096 .. 28672 deep) at 256 .. 4096 tokens.
double gemm_192_us(int M, int N, int K)
{
    const int tiles = ((M + 191) / 192) * ((N + 255) / 256), KT = K / FLEXQ_TILE_K;
    auto round_us = [&](int n) { return (0.90 + (n > 150 ? 0.42 * (n - 150) / 106.0 : 0.0)) * KT + 5.0; };
    const int tail = tiles % kStreamKGrid;
    return tiles / kStreamKGrid * round_us(kStreamKGrid) + (tail ? round_us(tail) : 0.0) + 1.0;
}

namespace {

constexpr int kLdsMax(int a, int b) { return a > b ? a : b; }
constexpr int kLdsBytes = kLdsMax(Shape<2>::LDS_BYTES, kLdsMax(Shape<1>::LDS_BYTES, Shape<3>::LDS_BYTES));

template <int FORM, bool ONE_ROUND = false>
hipError_t launch_form(const LinearArgs &a, int tiles_m, int tiles_n, int full_count, int tail_count,
                       int tail_wgs, int grid, hipStream_t st)
{
    auto kern = gemm_wlds_kernel<FORM, ONE_ROUND>;
    static std::atomic<unsigned long long> lds_allowed{0};
    constexpr int lds_bytes = FORM == 6 ? Shape<6>::LDS_BYTES : kLdsBytes;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds_bytes, lds_allowed);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * WAVES), lds_bytes, st, a, tiles_m, tiles_n,
                       full_count, tail_count, tail_wgs);
    return hipGetLastError();
}

// every workgroup has one item at most
bool one_round(int items) { return items <= kStreamKGrid; }

// workgroups for `items` items: a multiple of 8 (one share per XCD), at most one per CU
// on the 256-CU device the persistent forms are laid out for, else one per item
int grid_for(int items)
{
    const int g = (items + 7) / 8 * 8;
    return device_cu_count() == kStreamKGrid && g > kStreamKGrid ? kStreamKGrid : g;
}

template <int GROUP, int TAIL>
hipError_t launch_group(const LinearArgs &a, int tiles_m, int tiles_n, int full, int tail, int tail_wgs, hipStream_t st)
{
    auto kern = gemm_group_kernel<GROUP, TAIL>;
    constexpr int lds_bytes = kLdsMax(Shape<4>::LDS_BYTES, Shape<TAIL == 0 ? 4 : TAIL>::LDS_BYTES);
    static std::atomic<unsigned long long> lds_allowed{0};
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds_bytes, lds_allowed);
        e != hipSuccess)
        return e;
    const int g_full = full ? grid_for(full) : 0, g_tail = (tail_wgs + 7) / 8 * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(g_full > g_tail ? g_full : g_tail)), dim3(64 * WAVES), lds_bytes, st, a,
                       tiles_m, tiles_n, full, tail, tail_wgs);
    return hipGetLastError();
}

}  // namespace

// Whole items for one K split.  Measured at 65 .. 2048 tokens on twenty layers (512 .. 28672
// deep, 1024 .. 57344 wide) against the 128x128 tiles: the half height takes 0.65 to 0.85 us a
// stage where the whole one takes 0.9 to 1.15, so it is the faster one wherever its items fit a
// round (13824 x 5120 at 97 tokens, 240 items in six splits: 24.4 us against 33.7; at 700, 220 whole
// items, 78.9 against 92.2, with both operands' scales 93 against 124; a tail of 128 behind a
// round, 2048 tokens, 193 against 211).  Else 128-row tiles: above 128 tokens always (8192 x
// 28672 at 333 tokens, two splits, 121 against 145), up to there unsplit (57344 x 8192 at 97:
// 84.5 against 102.5; with splits neither is ahead).  Of the forms that the workspace has room
// for, the choice is within 2 % of the fastest.
int group_form(int M, int N, int split_k, size_t partial_bytes)
{
    if (M <= 64 || split_k > 16) return 0;
    const int tiles_n = (N + 255) / 256, tiles = (M + 127) / 128 * tiles_n, tail = tiles % kStreamKGrid;
    const bool whole_chip = device_cu_count() == kStreamKGrid, rounds = tiles >= kStreamKGrid;
    if (split_k > 1 && (rounds || !whole_chip)) return 0;
    const int halves = rounds ? 2 * tail : (M + 63) / 64 * tiles_n;
    auto fits = [&](int items, size_t bytes) {
        return items * split_k <= kStreamKGrid && (split_k == 1 || bytes <= partial_bytes);
    };
    if (whole_chip && halves > 0 && fits(halves, low_cut_bytes(halves * split_k) / 2)) return 19;
    if (split_k == 1 || (M > 128 && fits(tiles, low_cut_bytes(tiles * split_k)))) return 18;
    return 0;
}

// K splits for group-128 scales above 128 tokens: `ks` (choose_gemm_split's, which bounds the partial
// sums by the weights' bytes), or more where that leaves most of the chip idle -- an item's chain of
// stages is then the whole time, and the sums are cheap.  Estimated as the time of one round: a
// stage of a 64x256 item takes 0.59 us while at most half of the CUs have one, 0.74 on a full chip,
// of a 128x256 item 0.86 and 1.08, plus 4.4 and 6.8 us; S pieces meet in 2.5 + 0.55 S us and what their
// number in all costs.  Measured on 170 random layers of 1024 .. 24448 deep and 512 .. 5120 wide at 150 ..
// 3667 tokens, scales on the weights and on both operands: 138 of the 340 cells are cut anew, in 0.31 ..
// 0.94 of the time (700 tokens of K 8576, N 512 44 -> 19 us, 1101 of 13824, 512 69 -> 24, 2000 of 24448, 512
// 120 -> 49, 500 of 13824, 5120 80 -> 54; both operands' scales, 700 of 13824, 5120 91 -> 81).  A function of
// the shape alone, for every row alike.  The splits show in the sums' last bits, so an
// unsplit layer is only cut for 7 % of the time, one that is cut already only cut anew for a quarter.
int group_split(int M, int N, int K, int ks, size_t partial_bytes)
{
    const int KT = K / FLEXQ_TILE_K, tiles_n = (N + 255) / 256;
    const int tiles = (M + 127) / 128 * tiles_n, halves = (M + 63) / 64 * tiles_n;
    if (M <= 128 || tiles >= kStreamKGrid) return ks;
    auto round_us = [&](int pieces) {       // in the form group_form takes; 0: neither fits
        const bool half = halves * pieces <= kStreamKGrid;
        if (!half && tiles * pieces > kStreamKGrid) return 0.0;
        const int n = (half ? halves : tiles) * pieces;
        const double busy = n > 128 ? (n - 128) / 128.0 : 0.0;
        const double stage = half ? 0.59 + 0.15 * busy : 0.86 + 0.22 * busy;
        const double meet = pieces > 1 ? 2.5 + 0.55 * pieces + (half ? 0.008 : 0.02) * n : 0.0;
        return stage * ((KT + pieces - 1) / pieces) + (half ? 4.4 : 6.8) + meet;
    };
    const double now = round_us(ks);
    if (now == 0.0) return ks;
    int best = ks;
    double t_best = (ks == 1 ? 0.93 : 0.76) * now;
    for (int s = ks + 1; s <= 16 && s <= KT / 4 && tiles * s <= kStreamKGrid; ++s) {
        const bool half = halves * s <= kStreamKGrid;
        const size_t area = half ? low_cut_bytes(halves * s) / 2 : low_cut_bytes(tiles * s);
        if (area > partial_bytes || (size_t)s * M * N * 4 > partial_bytes) break;
        if (const double t = round_us(s); t < t_best) {
            t_best = t;
            best = s;
        }
    }
    return best;
}

hipError_t launch_gemm_group(const LinearArgs &a, bool half, int pieces, hipStream_t st)
{
    if (a.group != 128 || a.split_k > 1) return hipErrorInvalidValue;
    const int tiles_m = (a.M + 127) / 128, tiles_n = (a.N + 255) / 256, tiles = tiles_m * tiles_n;
    int tail = tiles % kStreamKGrid;
    const int full = tiles - tail;
    if (pieces < 1) pieces = 1;
    if (half) tail = full ? 2 * tail : (a.M + 63) / 64 * tiles_n;
    if ((tail == 0 || (pieces == 1 && !half)) && tiles <= kStreamKGrid)
        return a.sxg ? launch_group<2, 0>(a, tiles_m, tiles_n, tiles, 0, 0, st)
                     : launch_group<1, 0>(a, tiles_m, tiles_n, tiles, 0, 0, st);
    if (tail == 0 || (pieces == 1 && !half))
        return a.sxg ? launch_group<2, 4>(a, tiles_m, tiles_n, tiles, 0, 0, st)
                     : launch_group<1, 4>(a, tiles_m, tiles_n, tiles, 0, 0, st);
    if (pieces > 16 || pieces > a.K / FLEXQ_TILE_K || tail * pieces > kStreamKGrid ||
        (pieces > 1 && a.partial_bytes < low_cut_bytes(tail * pieces) / (half ? 2 : 1)) ||
        device_cu_count() != kStreamKGrid)
        return hipErrorInvalidValue;
    if (half)
        return a.sxg ? launch_group<2, 5>(a, tiles_m, tiles_n, full, tail, tail * pieces, st)
                     : launch_group<1, 5>(a, tiles_m, tiles_n, full, tail, tail * pieces, st);
    return a.sxg ? launch_group<2, 4>(a, tiles_m, tiles_n, full, tail, tail * pieces, st)
                 : launch_group<1, 4>(a, tiles_m, tiles_n, full, tail, tail * pieces, st);
}

// How pairs of pieces are dealt out: of an XCD's 32 workgroups some run its tiles' first pieces, `first`
// each, the others its second pieces, `second` each, and the cut is where both take the same time.  A
// piece costs 8 us beside its stages: first loads, and sums left or collected (128 KiB of them), which
// nothing overlaps.  (The next piece's first loads ahead of that: no change, 190 us on the layer below.)
GroupPairs group_pairs(int tiles, int KT)
{
    constexpr double kStage = 1.08, kPiece = 8.0;       // us on a full chip
    GroupPairs best{0, 0, 0, 0.0};
    const int share = (tiles + 7) / 8;
    if (KT < 2) return best;
    for (int f = 1; f <= 4; ++f)
        for (int s = f; s <= 8; ++s) {
            if ((share + f - 1) / f + (share + s - 1) / s > kStreamKGrid / 8) continue;
            int cut = (int)((s * KT * kStage + (s - f) * kPiece) / ((f + s) * kStage) + 0.5);
            cut = cut < 1 ? 1 : cut > KT - 1 ? KT - 1 : cut;
            const double t1 = f * (cut * kStage + kPiece), t2 = s * ((KT - cut) * kStage + kPiece);
            const double t = t1 > t2 ? t1 : t2;
            if (best.first == 0 || t < best.us) best = GroupPairs{f, s, cut, t};
        }
    return best;
}

size_t group_pair_bytes(int tiles) { return 2 * low_cut_bytes(tiles); }

// Taken for one to two rounds of tiles, where the last round, whole or at half the height, would leave most
// of the chip idle, and for 10 % of the estimated time: layers of K -> N 13824 -> 5120 at 1692 tokens (280 tiles)
// 192 -> 153 us, with both operands' scales 221 -> 173, 8192 -> 8192 at 1052 (288) 117 -> 98 and 134 -> 111, 11008 ->
// 4096 at 2304 155 -> 129 and 179 -> 145.  Of 174 cells of 257 .. 416 tiles, either mode, the 48 that it takes
// need 0.77 to 0.93 of the fastest other form's time.  Beside the line 13824 -> 5120 at 1948 (320) 192 / 174 and
// 221 / 198 (a 13B block at 2048 876 / 865: there it is drawn too carefully), 8192 -> 10240 at 964 (320) 116 / 110 and
// 134 / 122, at 1147 (360) 119 / 120 and 136 / 137, 5120 -> 5120 at 1920 (300) 77 / 71, at 2176 (340) 77 / 80, 4096 ->
// 4096 at 2944 (368) 65 / 80.  Below 32 stages a piece is mostly its meeting.  A function of the shape alone: the cut shows in
// the sums' last bits.
bool group_pairs_pay(int M, int N, int K, size_t partial_bytes)
{
    const int tiles = (M + 127) / 128 * ((N + 255) / 256), KT = K / FLEXQ_TILE_K, tail = tiles - kStreamKGrid;
    if (tail <= 0 || tail >= kStreamKGrid || KT < 32 || device_cu_count() != kStreamKGrid ||
        group_pair_bytes(tiles) > partial_bytes)
        return false;
    const GroupPairs p = group_pairs(tiles, KT);
    if (p.first == 0) return false;
    const double round = 1.08 * KT + 6.8;
    auto busy = [](int n) { return n > 128 ? (n - 128) / 128.0 : 0.0; };
    const double last = 2 * tail <= kStreamKGrid ? (0.59 + 0.15 * busy(2 * tail)) * KT + 4.4
                                                 : (0.86 + 0.22 * busy(tail)) * KT + 6.8;
    return p.us < 0.90 * (round + last);
}

hipError_t launch_gemm_group_pairs(const LinearArgs &a, hipStream_t st)
{
    const int tiles_m = (a.M + 127) / 128, tiles_n = (a.N + 255) / 256, tiles = tiles_m * tiles_n;
    const GroupPairs p = group_pairs(tiles, a.K / FLEXQ_TILE_K);
    if (a.group != 128 || p.first == 0 || a.partial_bytes < group_pair_bytes(tiles) || tiles > 2048 ||
        device_cu_count() != kStreamKGrid)
        return hipErrorInvalidValue;
    static std::atomic<unsigned long long> allowed[2];
    const auto kern = a.sxg ? gemm_group_pair_kernel<2> : gemm_group_pair_kernel<1>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), Shape<4>::LDS_BYTES, allowed[a.sxg != nullptr]);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(kStreamKGrid), dim3(64 * WAVES), Shape<4>::LDS_BYTES, st, a, tiles_m, tiles_n, p.cut,
                       p.first | p.second << 8);
    return hipGetLastError();
}

hipError_t launch_gemm_wlds(const LinearArgs &a, int tail_form, int tail_wgs, hipStream_t st)
{
    if (a.group != 0 || a.split_k > 1 || a.sxg) return hipErrorInvalidValue;
    if (tail_form == 3) {   // low tiles throughout
        const int low_m = (a.M + 127) / 128, cols = (a.N + 255) / 256;
        // One row of tiles, up to 128 tokens on wide layers, uses a weight once: past the caches if the layer is
        // more than the Infinity Cache (256 MiB) holds from one call to the next.  K -> N 8192 -> 57344 (352 MB) at
        // 33 / 64 / 100 / 128 tokens 66 -> 64.5 us, 69.4 / 68.6, 74.9 / 74.5, 78.3 / 77; one layer called again and
        // again, 5760 -> 65536 (283 MB) at 64 52 / 49.8, but 5504 -> 65536 (271 MB) 46.6 / 47.9, 4096 -> 65536 (201 MB)
        // 34.6 / 43.6.  (Smaller layers gain 4 % among others that evict them and lose up to 26 % where they
        // stay; so do the 64-row tiles, of which those with six K splits or more lose up to 11 % either way.
        // Cut along K, 28672 -> 8192 at 97, it makes no difference from HBM, 57.5 / 58.  A kernel of its own: a branch in
        // the shared one costs 5248 -> 13664 at 333 tokens 3 %.)
        constexpr long kBeyondCaches = 280L * 1000 * 1000;
        if (low_m == 1 && one_round(cols) && (long)a.N * a.K / 4 * 3 > kBeyondCaches)
            return launch_form<7, true>(a, low_m, cols, cols, 0, 0, grid_for(cols), st);
        if (one_round(low_m * cols))
            return launch_form<3, true>(a, low_m, cols, low_m * cols, 0, 0, grid_for(low_m * cols), st);
        return launch_form<3>(a, low_m, cols, low_m * cols, 0, 0, grid_for(low_m * cols), st);
    }
    if (tail_form == 6) {   // 192-row tiles throughout
        const int rows = (a.M + 191) / 192, cols = (a.N + 255) / 256;
        return one_round(rows * cols) ? launch_form<6, true>(a, rows, cols, rows * cols, 0, 0, grid_for(rows * cols), st)
                                      : launch_form<6>(a, rows, cols, rows * cols, 0, 0, grid_for(rows * cols), st);
    }
    if (tail_form == 5) {   // low tiles, those beyond the last whole round cut into equal pieces
        const int low_m = (a.M + 127) / 128, cols = (a.N + 255) / 256, all = low_m * cols;
        const int tiles = all % kStreamKGrid, full = all - tiles;
        const int pieces = tiles ? tail_wgs / tiles : 0;
        if (pieces < 2 || tail_wgs % tiles != 0 || pieces > 16 || pieces > a.K / FLEXQ_TILE_K ||
            tail_wgs > kStreamKGrid || a.partial_bytes < low_cut_bytes(tail_wgs) ||
            device_cu_count() != kStreamKGrid)
            return hipErrorInvalidValue;
        const int g = (tail_wgs + 7) / 8 * 8, g_full = full ? grid_for(full) : 0;
        return launch_form<5>(a, low_m, cols, full, tiles, tail_wgs, g > g_full ? g : g_full, st);
    }
    const int tiles_m = (a.M + 256 - 1) / 256, tiles_n = (a.N + 255) / 256;
    const StreamKPlan p = streamk_plan(a.M, a.N, a.K);
    // without room for the partial sums, or on a device that is not 256 CUs wide, a tail
    // that was to be cut runs as whole tiles
    if (tail_form == 2 && (tail_wgs <= 0 || a.partial_bytes < p.partial_bytes ||
                           device_cu_count() != kStreamKGrid))
        tail_form = 0;
    if (tail_form == 0 || p.tail_tiles == 0)      // every tile whole
        return one_round(p.tiles) ? launch_form<0, true>(a, tiles_m, tiles_n, p.tiles, 0, 0, grid_for(p.tiles), st)
                                  : launch_form<0>(a, tiles_m, tiles_n, p.tiles, 0, 0, grid_for(p.tiles), st);
    // the whole rounds first, then the tiles of the last, partial round in their own form
    const int g_full = p.full_tiles ? grid_for(p.full_tiles) : 0;
    if (tail_form == 1) {
        const int g = grid_for(2 * p.tail_tiles);
        return launch_form<1>(a, tiles_m, tiles_n, p.full_tiles, p.tail_tiles, 0, g > g_full ? g : g_full, st);
    }
    // a run is at least one stage, and the tail has at most 256 runs
    const long stages = (long)p.tail_tiles * (a.K / FLEXQ_TILE_K);
    if (tail_wgs > kStreamKGrid) tail_wgs = kStreamKGrid;
    if (tail_wgs > stages) tail_wgs = (int)stages;
    const int g = (tail_wgs + 7) / 8 * 8;
    // every tile cut into the same number of pieces (each at least one stage): the pieces
    // of a tile end together and share its reduction
    const int pieces = tail_wgs / p.tail_tiles;
    if (tail_wgs % p.tail_tiles == 0 && pieces >= 2 && pieces <= 16 && pieces <= a.K / FLEXQ_TILE_K)
        return launch_form<4>(a, tiles_m, tiles_n, p.full_tiles, p.tail_tiles, tail_wgs, g > g_full ? g : g_full, st);
    return launch_form<2>(a, tiles_m, tiles_n, p.full_tiles, p.tail_tiles, tail_wgs, g > g_full ? g : g_full, st);
}

}  // namespace flexq
