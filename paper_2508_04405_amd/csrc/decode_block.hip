// A decoder block's linears for a handful of tokens in ONE launch.
//
// With few tokens every linear is one pass over its weights, and what the block loses between two
// launches -- the drain of one kernel, the dispatch of the next, its first loads' latency, and the
// same again for the small producer launch between two linears -- is a large share of its time.
// Here one workgroup per CU stays for the whole block.  It owns fixed row blocks of every linear,
// and its wavefronts keep the packed tiles of their NEXT turn of work in flight whatever it is:
// the next row block's, or the next linear's, whose weights depend on nothing.  So linears that do
// not wait for each other run as one stream, and a wait for activations (everybody's outputs
// stored, the producer's norm or gated SiLU, its codes read back) begins with the weights already
// on their way.
//
// Bound: HBM while it streams (LLaMA-2-70B's gate+up at one token: 6.9 TB/s), and the waits: 9 us from the
// last output of one linear to the first tile of the next, six round trips through memory and about
// 2 us of arithmetic in the producer, of which the 96 KB per CU in flight cover 3.8.  Tried: two
// turns in flight, 192 KB per CU (no gain: the producer's own loads then queue behind them, 13B's block
// at 8 tokens 64.4 -> 66 us); a norm by 256 lanes like the stand-alone kernel's (4.1 us instead of 3);
// one mask word polled by everybody instead of a copy for 32 (1 us more per wait).
//
// Order between workgroups.  A linear's outputs go to memory with device-scope stores; when they
// are acknowledged the workgroup sets its bit in the linear's mask (one atomic OR).  The pieces of
// a producer's tokens belong to fixed workgroups, which wait for the mask of the linear they read,
// write the codes with device-scope stores and set the piece's bit.  A linear starts when its
// producer's bits are there.  No workgroup waits without a bound: when its polls run out (somebody
// is not resident: a busy device, another launch of this kind) it does what is missing itself, in
// order, each beginning with a different part (with nobody waiting at all LLaMA-2-7B's block at 8
// tokens takes 83 us, 70B's at one token 168; with one tile a wavefront in flight, everybody walking
// the same way and a wait for every piece of a row 305 and 418).  That needs nobody else and changes
// nothing: every result is a function of buffers that no part of the launch overwrites -- the codes
// of every linear have a place of their own, and the host takes this path only for buffers that do
// not overlap -- so work done twice stores the same values.  A workgroup that starts late finds its
// bit set by whoever did its row blocks and leaves them alone (the bits are read with the words a
// wait looks at anyway: 0.2 us of a block, 115.3 -> 115.5).  The last one to leave clears the words.
//
// Who reads what from where.  Outputs are read back with device-scope loads.  The codes are read
// with ordinary loads, so that an XCD fetches them once: no cache can hold an older value of
// their lines, which nobody reads before the bits are there and whose rows are whole lines.
//
// Results equal the separate launches bit for bit for finite inputs, which the library asks for (a
// NaN hides its lane's other values from a row's maximum, and rows lie over lanes differently here):
// the sums are exact integers, or, with group-128 scales, fp32 sums in the order of the streaming
// kernel with eight wavefronts and one K split, and the producers are the same operations in the
// same order.
#include "../../include/flexq.h"
#include "decode_block.h"
#include "flexq_device.h"
#include "gemm_common.h"
#include "producer_math.h"
#include <type_traits>

namespace {

using flexq::DecodeArgs;
using flexq::kDecodeGrid;

typedef unsigned int v2u __attribute__((ext_vector_type(2)));

#define INLINE __attribute__((always_inline))

constexpr int WAVES = 8;
constexpr int THREADS = 64 * WAVES;
constexpr int kScopeAgent = 16;            // cache policy of buffer accesses: device scope
constexpr int kNoLoads = 0x0F70;          // s_waitcnt vmcnt(0), as the builtin encodes it
constexpr unsigned kNowhere = 0xFFFFF000u; // a lane offset beyond every buffer: loads zero, touches nothing

// The kernel's argument where it lies: indexed by the linear's number, a copy would go to scratch memory.
typedef const DecodeArgs __attribute__((address_space(4))) Args;

// Words of the counter area (zero between calls).  A linear's mask: eight words of 32 workgroups, each
// on a line of its own (256 arrivals at about the same time).  A producer's: eight copies, one for
// each eighth of the workgroups that wait for it, a word per piece of a token's row.  The pieces'
// largest magnitudes: eight words per token.
constexpr int kDone = 32, kCodes = kDone + 4 * 8 * 32, kTops = kCodes + 4 * 8 * 32, kLeave = kTops + 4 * 16 * 8;
static_assert((kLeave + 1) * 4 <= FLEXQ_WORKSPACE_COUNTER_BYTES, "the counter area");
__device__ __forceinline__ unsigned *done_word(Args &a, int k, int i) { return a.words + kDone + (k * 8 + i) * 32; }
__device__ __forceinline__ unsigned *codes_words(Args &a, int k, int copy) { return a.words + kCodes + (k * 8 + copy) * 32; }
__device__ __forceinline__ unsigned *top_words(Args &a, int k, int m) { return a.words + kTops + (k * 16 + m) * 8; }

__device__ __forceinline__ unsigned peek(const unsigned *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// GROUP: 0 = scales per output channel, 1 = weight scales per 128-k group.  MQ: eighths of a
// 32-token row block that hold tokens (M <= 8 MQ).  A wavefront's tiles of a row block come in turns
// of GS (the last one filled up with nothing), and a turn's tiles are in flight.
template <int GROUP, int MQ, int GS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_block_kernel(DecodeArgs)
{
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-resource builtins exist in the device pass only
    Args &a = *(Args *)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int RED = WAVES * 4 * MQ * 64;   // ints of one reduction buffer
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ float s_sx[8 * MQ], s_red[WAVES];
    __shared__ unsigned s_words[8];
    __shared__ int s_flag;
    __shared__ uint16_t s_sw[GROUP ? 1 : THREADS];     // scales of this workgroup's row blocks (at most 16)
    int *const red = reinterpret_cast<int *>(lds);
    uint8_t *const acts = lds + 2 * RED * 4;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int self = blockIdx.x;
    const int M = a.M, n = a.n;
    const unsigned all_tokens = (1u << M) - 1u;

    // ---- the weight stream, a turn ahead of the arithmetic -------------------------------------
    PackedTile st[GS];
    uint16_t gs[GS];        // GROUP: the scales of those tiles' channels
    // the turn to request next: linear (n: none), row block, turn of it
    int nk, nj = 0, nr = 0;
    int n_kt = 0, n_turns = 0, n_blocks = 0;
    const uint8_t *n_packed = nullptr;
    const uint16_t *n_scales = nullptr;
    auto first_block = [&](int k, int slot) INLINE {     // of workgroup `slot` in linear k, then every 256th
        const int j = slot - a.ph[k].off;
        return j < 0 ? j + kDecodeGrid : j;
    };
    auto turns_of = [&](int kt) INLINE { return ((kt + WAVES - 1) / WAVES + GS - 1) / GS; };   // per row block
    auto open = [&](int k) INLINE {
        n_kt = n_turns = n_blocks = nr = 0;
        for (nk = k; nk < n; ++nk) {
            nj = first_block(nk, self);
            if (nj >= a.ph[nk].nb) continue;
            n_blocks = a.ph[nk].nb;
            n_kt = a.ph[nk].kt;
            n_turns = turns_of(n_kt);
            n_packed = (const uint8_t *)a.ph[nk].packed;
            n_scales = a.ph[nk].scales;
            break;
        }
    };
    auto advance = [&]() INLINE {
        if (++nr < n_turns) return;
        nr = 0;
        nj += kDecodeGrid;
        if (nj >= n_blocks) open(nk + 1);
    };
    // (always the same number of loads: what is not wanted is asked for out of range)
    auto request = [&](int p, bool held) INLINE {
        const int t = (nr * GS + p) * WAVES + wave;
        const bool ok = t < n_kt && !held;
        const unsigned tiles = (unsigned)n_blocks * (unsigned)n_kt;
        const __amdgpu_buffer_rsrc_t w =
            __builtin_amdgcn_make_buffer_rsrc((void *)n_packed, 0, tiles * FLEXQ_TILE_BYTES, 0x00020000);
        const unsigned tile = ok ? (unsigned)(nj * n_kt + t) : 0u;
        const unsigned at = ok ? 16u * lane : kNowhere, base = tile * FLEXQ_TILE_BYTES;
        if (GROUP) {
            const __amdgpu_buffer_rsrc_t sc =
                __builtin_amdgcn_make_buffer_rsrc((void *)n_scales, 0, tiles * 64u, 0x00020000);
            gs[p] = __builtin_amdgcn_raw_buffer_load_b16(sc, ok ? 2u * (lane & 31) : kNowhere, tile * 64u, 0);
        }
        PackedTile &s = st[p];
        s.q0 = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w, at, base, kNonTemporal));
        s.q1 = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w, at + 1024u, base, kNonTemporal));
        s.q2 = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w, at + 2048u, base, kNonTemporal));
    };
    auto request_turn = [&]() INLINE {
#pragma unroll
        for (int p = 0; p < GS; ++p) {
            request(p, false);
            __builtin_amdgcn_sched_barrier(0);      // in this order: a wait counts the loads behind a tile's
        }
        advance();
    };

    // ---- arithmetic of one tile, and the end of a row block --------------------------------
    int xstride = 0;
    const uint8_t *xl = acts;
    v16i acc;
    float facc[4 * MQ];
    auto clear = [&] {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
        for (int r = 0; r < 4 * MQ; ++r) facc[r] = 0.0f;
    };
    auto consume = [&](const PackedTile &w, uint16_t g, int t) INLINE {
        v4i x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const v4i *>(xl + t * FLEXQ_TILE_K + 32 * j);
        if (GROUP) {
            v16i part;
#pragma unroll
            for (int r = 0; r < 16; ++r) part[r] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) part = mfma_i8(x[j], unpack_kstep(w, j), part);
            const float s = h2f(g);
#pragma unroll
            for (int r = 0; r < 4 * MQ; ++r) facc[r] = __builtin_fmaf((float)part[r], s, facc[r]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = mfma_i8(x[j], unpack_kstep(w, j), acc);
        }
    };
    int half = 0;           // reduction buffer in turn: one barrier per row block is enough
    auto finish = [&](int k, int j, uint16_t sw) INLINE {
        int *const r = red + half * RED;
#pragma unroll
        for (int q = 0; q < 4 * MQ; ++q)
            r[(wave * 4 * MQ + q) * 64 + lane] = GROUP ? __float_as_int(facc[q]) : acc[q];
        lds_barrier();
        if (wave == 0) {
            const int N = a.ph[k].nb * 32;
            uint16_t *const y = a.ph[k].y + 32 * j + (lane & 31);
#pragma unroll
            for (int first = 0; first < 4 * MQ; first += 4) {
                int part[4][WAVES];
                float sx[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sx[i] = s_sx[mfma_row(first + i, lane)];
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) part[i][w] = r[(w * 4 * MQ + first + i) * 64 + lane];
                }
                // (all of them ahead of the sums: else a read waits for the one before, 32 in a row)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = mfma_row(first + i, lane);
                    uint16_t h;
                    if (GROUP) {
                        float f = 0.0f;
#pragma unroll
                        for (int w = 0; w < WAVES; ++w) f += __int_as_float(part[i][w]);
                        h = f2h(f * 0.25f * sx[i]);
                    } else {
                        int v = 0;
#pragma unroll
                        for (int w = 0; w < WAVES; ++w) v += part[i][w];
                        h = f2h((float)(v >> 2) * (sx[i] * h2f(sw)));
                    }
                    if (m < M)
                        __hip_atomic_store(y + (long)m * N, h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        half ^= 1;
        clear();
    };

    // ---- waiting, with a bound; the answer (0: it ran out) goes to every wavefront ------------------
    auto wait_for = [&](auto ready, int polls) INLINE -> int {
        if (wave == 0) {
            int got = ready();
            for (int i = 0; got == 0 && i < polls; ++i) {
                __builtin_amdgcn_s_sleep(1);
                got = ready();
            }
            if (lane == 0) s_flag = got;
        }
        lds_barrier();
        const int got = __builtin_amdgcn_readfirstlane(s_flag);
        lds_barrier();
        return got;
    };
    auto pieces_of = [&](int i) INLINE { return flexq::decode_pieces(a.pr[i].mode, a.pr[i].L); };
    // What a wait is for may have been done in this workgroup's place, by one that no longer waited for
    // it: the last lane looks for that, on the first trip through memory.
    constexpr int kReady = 1, kDoneForUs = 2;
    auto bit_of_last_lane = [&](unsigned v, int bit) INLINE { return (__builtin_amdgcn_readlane((int)v, 63) >> bit) & 1; };
    auto codes_there = [&](int k) INLINE {
        const int pieces = pieces_of(k);
        const unsigned *const word = lane == 63 ? done_word(a, k, self >> 5) : codes_words(a, k, self & 7) + (lane & 7);
        bool look = lane < pieces || lane == 63;
        return wait_for([&] {
            unsigned v = lane == 63 ? 0u : all_tokens;
            if (look) v = peek(word);
            look = lane < pieces;
            if (bit_of_last_lane(v, self & 31)) return kDoneForUs;      // this workgroup's row blocks
            return __all(lane >= pieces || v == all_tokens) ? kReady : 0;
        }, a.spin);
    };
    auto outputs_there = [&](int k, int what) INLINE {                  // for piece `what` of the next linear's producer
        const unsigned *const word = lane == 63 ? codes_words(a, k + 1, self & 7) + (what >> 5) : done_word(a, k, lane & 7);
        bool look = lane < 8 || lane == 63;
        return wait_for([&] {
            unsigned v = lane == 63 ? 0u : ~0u;
            if (look) v = peek(word);
            look = lane < 8;
            if (bit_of_last_lane(v, what & 31)) return kDoneForUs;
            return __all(lane == 63 || v == ~0u) ? kReady : 0;
        }, a.spin);
    };
    auto meet = [&](float v, bool sum, int waves) INLINE {
        v = sum ? wave_sum(v) : wave_max(v);
        if (lane == 0) s_red[wave] = v;
        lds_barrier();
        float r = s_red[0];
        for (int w = 1; w < waves; ++w) r = sum ? r + s_red[w] : fmaxf(r, s_red[w]);
        lds_barrier();
        return r;
    };

    // ---- one piece of a producer's token: fp16 in, codes and scale out (as producer_kernel) ----
    auto produce_as = [&](auto mode_tag, int i, int m, int piece, int polls) INLINE {
        constexpr int MODE = decltype(mode_tag)::value;
        constexpr int CH = MODE == 0 ? 2 : 1;
        const auto &p = a.pr[i];
        const int L = p.L, chunks = L / 8;
        const int row_len = MODE == 1 ? 2 * L : L;
        const __amdgpu_buffer_rsrc_t in = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(p.in + (long)m * row_len), 0, (unsigned)row_len * 2u, 0x00020000);
        const __amdgpu_buffer_rsrc_t gamma = __builtin_amdgcn_make_buffer_rsrc(
            (void *)p.gamma, 0, MODE == 0 ? (unsigned)L * 2u : 0u, 0x00020000);
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(p.xq + (long)m * L), 0, (unsigned)L, 0x00020000);
        uint4 held[CH], other[CH];
        unsigned at[CH];
        // (lanes and chunks beyond the row read zeros, which change no sum and no maximum)
        auto load = [&](int first) INLINE {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int chunk = first + tid + THREADS * c;
                at[c] = chunk < chunks ? 16u * chunk : kNowhere;
                held[c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(in, at[c], 0, kScopeAgent));
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                other[c] = held[c];
                if (MODE == 0)
                    other[c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(gamma, at[c], 0, 0));
                if (MODE == 1)
                    other[c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                   in, at[c] == kNowhere ? kNowhere : at[c] + 2u * L, 0, kScopeAgent));
            }
        };
        float inv = 0.0f;
        auto largest = [&]() INLINE {
            unsigned best = 0;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                held[c] = produce_h<MODE>(held[c], other[c], inv);
                best = max_bits(held[c], best);
            }
            return h2f((uint16_t)best);
        };
        load(piece * THREADS);
        if (MODE == 0) {
            // The sum of squares in the order of the stand-alone kernel, whose 256 lanes take every
            // 256th chunk: four wavefronts read the other half of the row as well.
            float ss = 0.0f;
            if (wave < 4) {
                uint4 more[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const int chunk = tid + 256 + THREADS * c;
                    more[c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                            in, chunk < chunks ? 16u * chunk : kNowhere, 0, kScopeAgent));
                }
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    add_squares(held[c], ss);
                    add_squares(more[c], ss);
                }
            }
            inv = 1.0f / sqrtf(meet(ss, true, 4) / (float)L + a.eps);
        }
        float top = meet(largest(), false, WAVES);
        if (MODE != 0) {
            // the row's largest magnitude from all its pieces, or, if they do not come, from the row
            const int pieces = pieces_of(i);
            if (pieces > 1) {
                if (tid == 0)
                    __hip_atomic_store(top_words(a, i, m) + piece, 0x80000000u | f2h(top), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                unsigned seen = 0;
                const int ok = wait_for([&] {
                    seen = lane < pieces ? peek(top_words(a, i, m) + lane) : 0x80000000u;
                    return __all((int)seen < 0) ? kReady : 0;
                }, polls);
                if (ok != 0) {
                    top = meet(wave == 0 ? h2f((uint16_t)(seen & 0xffffu)) : 0.0f, false, 1);
                } else {
                    float all = 0.0f;
                    for (int q = 0; q < pieces; ++q) {
                        load(q * THREADS);
                        all = fmaxf(all, largest());
                    }
                    top = meet(all, false, WAVES);
                    load(piece * THREADS);
                    largest();
                }
            }
        }
        const uint16_t bits = token_scale(top, p.qmax);
        const float sf = h2f(bits), rf = 1.0f / sf;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const uint2 q = quant8(held[c], sf, rf, -p.qmax - 1.0f, p.qmax);
            __builtin_amdgcn_raw_buffer_store_b64((v2u){q.x, q.y}, out, at[c] == kNowhere ? kNowhere : at[c] / 2, 0,
                                                  kScopeAgent);
        }
        if (tid == 0 && piece == 0) __hip_atomic_store(p.sx + m, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(kNoLoads);
        lds_barrier();
        if (tid < 8)
            __hip_atomic_fetch_or(codes_words(a, i, tid) + piece, 1u << m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // `what`: piece * 32 + token; `polls`: how long to wait for the row's other pieces
    auto produce = [&](int i, int what, int polls) INLINE {
        const int mode = a.pr[i].mode, m = what & 31, piece = what >> 5;
        if (mode == 0)
            produce_as(std::integral_constant<int, 0>{}, i, m, piece, polls);
        else if (mode == 1)
            produce_as(std::integral_constant<int, 1>{}, i, m, piece, polls);
        else
            produce_as(std::integral_constant<int, 2>{}, i, m, piece, polls);
    };
    // Whose a producer's pieces are: numbered through (those of the producers that need no outputs one
    // after the other), they go to the workgroups that follow the owner of its linear's last row
    // block, which have a row block less there (or none); the host sees to it that there are no more of
    // them than workgroups.  This workgroup's piece of producer i as piece * 32 + token, or -1.
    auto my_piece = [&](int i) INLINE {
        const int home = a.pr[i].dep < 0 ? 0 : i, pieces = pieces_of(i);
        const int u = ((self - a.ph[home].off - a.ph[home].nb) & (kDecodeGrid - 1)) - a.pr[i].first;
        if (u < 0 || u >= M * pieces) return -1;
        const int m = u / pieces;
        return (u - m * pieces) * 32 + m;
    };

    // ---- linear k's codes and token scales into LDS --------------------------------------------
    auto stage = [&](int k) INLINE {
        const int K = a.ph[k].kt * FLEXQ_TILE_K, per_row = K / 16, total = M * per_row;
        const unsigned inv = a.ph[k].inv;
        const v4i *src = reinterpret_cast<const v4i *>(a.ph[k].xq);
        xstride = K + 16;
        xl = acts + ((lane & 31) < M ? (lane & 31) : 0) * xstride + 16 * (lane >> 5);
        uint16_t sx = 0, sw = 0;
        if (tid < M) sx = __hip_atomic_load(a.ph[k].sx + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!GROUP) {
            const int n = 32 * (first_block(k, self) + kDecodeGrid * (tid >> 5)) + (tid & 31);
            if (n < 32 * a.ph[k].nb) sw = a.ph[k].scales[n];
        }
        for (int base = tid; base < total; base += 8 * THREADS) {
            v4i got[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) got[i] = src[min(base + i * THREADS, total - 1)];
            // (the builtin, which the compiler counts: a load it took to be under way would make it
            // wait for the whole weight stream at every later use of that register)
            __builtin_amdgcn_s_waitcnt(kNoLoads);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = base + i * THREADS;
                if (c < total) {
                    const int row = (int)__umulhi((unsigned)c, inv);
                    *reinterpret_cast<v4i *>(acts + row * xstride + 16 * (c - row * per_row)) = got[i];
                }
            }
        }
        if (tid < 8 * MQ) s_sx[tid] = h2f(sx);
        if (!GROUP) s_sw[tid] = sw;
        lds_barrier();
    };
    auto set_done = [&](int k, int slot) INLINE {     // by wavefront 0, whose stores are acknowledged
        if (tid == 0)
            __hip_atomic_fetch_or(done_word(a, k, slot >> 5), 1u << (slot & 31), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    };
    auto feeds_later = [&](int k) INLINE {
        bool any = false;
        for (int i = k + 1; i < n; ++i) any = any || a.pr[i].dep == k;
        return any;
    };

    // ---- where a wait ran out: what nobody has done yet, by this workgroup ------------------------
    // One of the bits of `wanted` that are clear in a row of words, as word * 32 + bit, or -1: those
    // who ask at the same time get different ones where there are enough.  (Wavefront 0 set its own
    // bits: they are there once its stores are.)
    auto pick_missing = [&](const unsigned *word, int step, int words, unsigned wanted) INLINE {
        if (wave == 0) {
            __builtin_amdgcn_s_waitcnt(kNoLoads);
            if (lane < 8) s_words[lane] = lane < words ? ~peek(word + step * lane) & wanted : 0u;
        }
        lds_barrier();
        int total = 0, at = 0, before = 0;
        unsigned rest = 0;
        for (int i = 0; i < 8; ++i) total += __builtin_popcount(__builtin_amdgcn_readfirstlane((int)s_words[i]));
        const int rank = (self * total) >> 8;
        for (int i = 0, sum = 0; i < 8; ++i) {
            const unsigned w = (unsigned)__builtin_amdgcn_readfirstlane((int)s_words[i]);
            if (sum <= rank) {
                at = i;
                before = sum;
                rest = w;
            }
            sum += __builtin_popcount(w);
        }
        for (int i = before; i < rank; ++i) rest &= rest - 1u;
        lds_barrier();
        return total == 0 ? -1 : at * 32 + __builtin_ctz(rest);
    };
    // Linear q's row blocks, a workgroup's share at a time and a turn of tiles in flight.  The
    // registers are those of the stream, which begins anew, at linear k, afterwards.
    auto run_missing = [&](int q, int k) INLINE {
        int slot = pick_missing(done_word(a, q, 0), 32, 8, ~0u);
        if (slot < 0) return;
        stage(q);
        n_kt = a.ph[q].kt;
        n_blocks = a.ph[q].nb;
        n_packed = (const uint8_t *)a.ph[q].packed;
        n_scales = a.ph[q].scales;
        const int turns = turns_of(n_kt);
        int rounds = 0;
        do {                                    // (each sets a bit)
            for (nj = first_block(q, slot); nj < n_blocks; nj += kDecodeGrid) {
                for (nr = 0; nr < turns; ++nr) {
#pragma unroll
                    for (int p = 0; p < GS; ++p) request(p, false);
#pragma unroll
                    for (int p = 0; p < GS; ++p) {
                        const int t = (nr * GS + p) * WAVES + wave;
                        if (t < n_kt) consume(st[p], GROUP ? gs[p] : (uint16_t)0, t);
                    }
                }
                finish(q, nj, GROUP ? (uint16_t)0 : a.ph[q].scales[32 * nj + (lane & 31)]);
            }
            if (wave == 0) {
                __builtin_amdgcn_s_waitcnt(kNoLoads);
                set_done(q, slot);
            }
            slot = pick_missing(done_word(a, q, 0), 32, 8, ~0u);
        } while (slot >= 0 && ++rounds < kDecodeGrid);
        open(k);
        request_turn();
    };

    // ---- the block ------------------------------------------------------------------------
    // (the arguments' cache lines, all at once and ahead of their first use)
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" ::"s"(a.ph[k].nb), "s"(a.pr[k].L));
    clear();
    open(0);
    request_turn();
    unsigned left = 0;
    for (int k = 0; k < n; ++k) {
        const int kt = a.ph[k].kt, nb = a.ph[k].nb;
        int j = first_block(k, self);
        const bool feeds = feeds_later(k);
        bool mine = j < nb;      // row blocks of this linear are left for this workgroup
        // Step 0: this workgroup's share of the producers whose input is complete once linear
        // k - 1 is (k = 0: of those that need none).  Step 1: the codes of linear k.  Where a wait
        // ran out, first everything that is missing, in order.  (That part has a copy of the producers
        // of its own and lies behind the rest: in between, the longer way through the instructions cost
        // every launch 0.2 to 1 us.)
#pragma clang loop unroll(disable)
        for (int step = 0; step < 2; ++step) {
            int got = kReady;
            if (step == 0) {
                if (k > 0) {
                    if (a.pr[k].dep != k - 1 || my_piece(k) < 0) continue;
                    got = outputs_there(k - 1, my_piece(k));
                }
            } else if (mine) {
                got = codes_there(k);
                mine = got != kDoneForUs;
            }
            if (__builtin_expect(got == 0, 0)) {
                for (int i = 0; i < k + step; ++i) {
                    if (i < k && !feeds_later(i)) continue;
                    for (int round = 0; round < kDecodeGrid; ++round) {     // (each sets a bit)
                        const int what = pick_missing(codes_words(a, i, self & 7), 1, pieces_of(i), all_tokens);
                        if (what < 0) break;
                        produce(i, what, 0);
                    }
                    if (i < k) run_missing(i, k);
                }
            }
            if (step == 1 || got == kDoneForUs) continue;
            for (int i = k; i <= (k == 0 ? n - 1 : k); ++i)
                if (a.pr[i].dep == k - 1 && my_piece(i) >= 0) produce(i, my_piece(i), a.spin);
        }
        if (j < nb && !mine) {      // the tiles in flight are the next linear's instead
            open(k + 1);
            request_turn();
        }
        if (mine) {
            stage(k);
            // The masks are not looked at any more.  (Every bit this workgroup set is there: the loads
            // of `stage` were waited for, and with them all that wavefront 0 did before.)
            if (k == n - 1 && tid == 0)
                left = 1u + __hip_atomic_fetch_add(a.words + kLeave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int turns = turns_of(kt);
            for (; j < nb; j += kDecodeGrid) {
                for (int r = 0; r < turns; ++r) {
                    // wavefront 0 stores the last outputs and has to see them acknowledged: its next
                    // tiles are asked for behind that
                    const bool held = wave == 0 && feeds && j + kDecodeGrid >= nb && r == turns - 1;
#pragma unroll
                    for (int p = 0; p < GS; ++p) {
                        const int t = (r * GS + p) * WAVES + wave;
                        if (t < kt) consume(st[p], GROUP ? gs[p] : (uint16_t)0, t);
                        request(p, held);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (!held) advance();
                }
                finish(k, j, GROUP ? (uint16_t)0 : s_sw[(j / kDecodeGrid) * 32 + (lane & 31)]);
            }
        }
        if (feeds && wave == 0 && (mine || first_block(k, self) >= nb)) {
            __builtin_amdgcn_s_waitcnt(kNoLoads);
            set_done(k, self);
            if (first_block(k, self) < nb) request_turn();
        }
    }

    // ---- the last to leave clears the words -------------------------------------------------
    if (wave == 0) {
        __builtin_amdgcn_s_waitcnt(kNoLoads);
        if (tid == 0 && left == 0)
            left = 1u + __hip_atomic_fetch_add(a.words + kLeave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane((int)left) == kDecodeGrid) {
            auto zero = [&](unsigned *w) INLINE {
                __hip_atomic_store(w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            if (lane < 32) zero(done_word(a, 0, lane));
            for (int c = lane >> 3; c < 32; c += 8) zero(codes_words(a, 0, c) + (lane & 7));
            for (int w = lane; w < 4 * 16 * 8; w += 64) zero(a.words + kTops + w);
            if (lane == 0) zero(a.words + kLeave);
        }
    }
#endif
}

template <int GROUP, int MQ, int GS>
hipError_t launch_one(const DecodeArgs &a, int lds_bytes, hipStream_t st)
{
    auto kern = decode_block_kernel<GROUP, MQ, GS>;
    static std::atomic<unsigned long long> lds_allowed{0};
    if (hipError_t e = flexq::allow_dynamic_lds(reinterpret_cast<const void *>(kern), flexq::kDecodeLds, lds_allowed);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(kDecodeGrid), dim3(THREADS), lds_bytes, st, a);
    return hipGetLastError();
}

}  // namespace

namespace flexq {

int decode_block_lds(int M, int K) { return 2 * 8192 * ((M + 7) / 8) + M * (K + 16); }

hipError_t launch_decode_block(const DecodeArgs &a, int lds_bytes, hipStream_t st)
{
    if (a.M < 1 || a.M > 16 || a.n < 1 || a.n > 4 || lds_bytes > kDecodeLds) return hipErrorInvalidValue;
    // turns of four or five tiles, whichever leaves fewer empty places
    long empty[2] = {0, 0};
    for (int i = 0; i < a.n; ++i)
        for (int g = 4; g <= 5; ++g) {
            const int tiles = (a.ph[i].kt + WAVES - 1) / WAVES;
            empty[g - 4] += (long)a.ph[i].nb * ((tiles + g - 1) / g * g - tiles);
        }
    const bool five = empty[1] < empty[0];
    if (a.group)
        return a.M <= 8 ? (five ? launch_one<1, 1, 5>(a, lds_bytes, st) : launch_one<1, 1, 4>(a, lds_bytes, st))
                        : (five ? launch_one<1, 2, 5>(a, lds_bytes, st) : launch_one<1, 2, 4>(a, lds_bytes, st));
    return a.M <= 8 ? (five ? launch_one<0, 1, 5>(a, lds_bytes, st) : launch_one<0, 1, 4>(a, lds_bytes, st))
                    : (five ? launch_one<0, 2, 5>(a, lds_bytes, st) : launch_one<0, 2, 4>(a, lds_bytes, st));
}

}  // namespace flexq
