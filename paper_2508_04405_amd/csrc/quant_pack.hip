// Weight quantizer and the 6-bit packer (gfx950); the activation quantizer
// lives with the activation producers.
//
// Quantization is the symmetric, zero-point-free scheme of the paper's Section
// 2.1 with one scale per group of consecutive elements (Section 4.1.1); a whole
// row as one group is the per-channel / per-token case.  The scale is rounded
// to fp16 first and the SAME fp16 value divides the inputs, so quantize and
// dequantize agree; the division is the correctly rounded fp32 one and the
// rounding to an integer is v_rndne_f32 (half to even).
#include "flexq_device.h"
#include "flexq_kernels.h"

namespace {

// A row's floats and codes are moved four at a time; the caller's pointers need no more
// than the alignment of one element, which the types say and the hardware accepts.
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned codes4_any __attribute__((aligned(1)));

// fp16 scale of a group from its absmax, and the float the codes divide by.
__device__ __forceinline__ void make_scale(float amax, uint16_t &bits, float &sf)
{
    bits = f2h(amax / 31.0f);
    sf = h2f(bits);
    if (amax == 0.0f || sf == 0.0f) {
        bits = 0x3c00;
        sf = 1.0f;
    }
}

// Four codes clamp(rne(v / sf), -32, 31).  div_by gives the IEEE quotient of any float here:
// sf has eleven significant bits, so its remainder is exact and the quotient is never closer
// to a rounding boundary than 2^-12 ulp, far outside the correction's error (a quotient that
// underflows rounds to code 0 either way).  A scale that overflowed fp16 is infinite and
// every quotient 0: sf = 1, rf = 0 give that.
__device__ __forceinline__ unsigned quant4(const float4_any &v, float sf, float rf)
{
    unsigned out = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(div_by(v[i], sf, rf)), -32.0f, 31.0f);
        out = __builtin_amdgcn_cvt_pk_u8_f32(q + 128.0f, i, out);
    }
    return out ^ 0x80808080u;
}

__device__ __forceinline__ void reciprocal(float &sf, float &rf)
{
    rf = 1.0f / sf;
    if (rf == 0.0f) sf = 1.0f;
}

__device__ __forceinline__ float absmax4(const float4_any &v, float best)
{
    return fmaxf(fmaxf(best, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
}

// One scale per row: a workgroup of T lanes holds its row in registers, CH float4 a lane,
// between the absmax and the codes.  Bound by HBM: five bytes an element, each moved once
// (a loop over the row with one float a lane, read twice, took 139 us for 8192 x 8192, this
// with cached loads 64 us).  The floats, read once, come past the caches, which keep the codes
// for the packer: 57.8 us, 5.8 TB/s, and 75 us instead of 80 with the packer behind it.  (Stores
// of the codes past the caches too: the packer loses more than this kernel gains, 82 us for both.)
// Floats that another kernel has just written, quantizer and packer: 4096 x 11008 57.5 -> 50.6 us, 8192 x 8192
// 96 -> 73; long written, 89 -> 57 and 123 -> 82; the same floats again and again out of the Infinity Cache,
// which no program does, 47.6 / 52.5 and 80 / 74.
template <int CH, int T>
__global__ __launch_bounds__(T) void quant_w6_row_kernel(const float *__restrict__ w, int K,
                                                         int8_t *__restrict__ wq, uint16_t *__restrict__ sw)
{
    __shared__ float red[T / 64];
    const long row = blockIdx.x;
    const int chunks = K / 4;
    const float4_any *src = reinterpret_cast<const float4_any *>(w + row * K);
    codes4_any *dst = reinterpret_cast<codes4_any *>(wq + row * K);
    float4_any held[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = threadIdx.x + T * i;
        if (c < chunks) held[i] = __builtin_nontemporal_load(src + c);
    }
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < CH; ++i)
        if (threadIdx.x + T * i < chunks) amax = absmax4(held[i], amax);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < T / 64; ++i) amax = fmaxf(amax, red[i]);
    uint16_t bits;
    float sf, rf;
    make_scale(amax, bits, sf);
    if (threadIdx.x == 0) sw[row] = bits;
    reciprocal(sf, rf);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = threadIdx.x + T * i;
        if (c < chunks) dst[c] = quant4(held[i], sf, rf);
    }
}

// One scale per 128 consecutive k: 32 lanes own a group, four floats each, and the absmax
// meets by five shuffles.  Groups follow each other through the whole matrix, four KiB of a
// wavefront's loads in flight, past the caches as above (8192 x 8192: 53.4 us, with cached loads
// 59.8; with one wavefront per group and two floats a lane it took 189 us).
__global__ __launch_bounds__(256) void quant_w6_g128_kernel(const float *__restrict__ w, long chunks,
                                                            int8_t *__restrict__ wq, uint16_t *__restrict__ sw)
{
    constexpr int CH = 4;
    const float4_any *src = reinterpret_cast<const float4_any *>(w);
    codes4_any *dst = reinterpret_cast<codes4_any *>(wq);
    const long c0 = (long)blockIdx.x * (256 * CH) + threadIdx.x;    // the 32 lanes of a group leave together
    float4_any held[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i)
        if (c0 + 256 * i < chunks) held[i] = __builtin_nontemporal_load(src + c0 + 256 * i);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const long c = c0 + 256 * i;
        if (c >= chunks) return;
        float amax = absmax4(held[i], 0.0f);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        uint16_t bits;
        float sf, rf;
        make_scale(amax, bits, sf);
        if ((threadIdx.x & 31) == 0) sw[c >> 5] = bits;
        reciprocal(sf, rf);
        dst[c] = quant4(held[i], sf, rf);
    }
}

// One thread per (tile, lane): 64 codes in, 48 packed bytes out.
// The first threads copy the scales as well (there are at most half as many as threads),
// group ones from [N][K/128] to tile order [N/32][K/128][32]: a launch of its own for
// them took 4.7 us.
__global__ __launch_bounds__(256) void pack_w6_kernel(const int8_t *__restrict__ wq,
                                                      const uint16_t *__restrict__ sw, int N, int K, int group,
                                                      uint8_t *__restrict__ packed)
{
    const long gid = (long)blockIdx.x * 256 + threadIdx.x;
    const int kt = K / FLEXQ_TILE_K;
    const long tiles = (long)(N / FLEXQ_TILE_ROWS) * kt;
    uint16_t *scales = reinterpret_cast<uint16_t *>(packed + tiles * FLEXQ_TILE_BYTES);
    if (group == 0) {
        if (gid < N) scales[gid] = sw[gid];
    } else if (gid < (long)N * kt) {
        const long nb = gid / (32 * kt), in_nb = gid - nb * 32 * kt;
        scales[gid] = sw[(nb * 32 + (in_nb & 31)) * kt + (in_nb >> 5)];
    }
    const long tile = gid >> 6;
    const int lane = (int)(gid & 63);
    if (tile >= tiles) return;
    const long nb = tile / kt, kb = tile % kt;
    const int r = lane & 31, h = lane >> 5;
    const int8_t *row = wq + (nb * FLEXQ_TILE_ROWS + r) * (long)K + kb * FLEXQ_TILE_K + 16 * h;
    uint8_t c[4][16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint4 v = *reinterpret_cast<const uint4 *>(row + 32 * j);
        __builtin_memcpy(c[j], &v, 16);
    }
    uint8_t *dst = packed + tile * FLEXQ_TILE_BYTES + lane * 16;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        uint8_t o[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            unsigned code = c[j][t] & 63u;
            unsigned spare = ((c[3][t] & 63u) >> (4 - 2 * j)) & 3u;
            o[t] = (uint8_t)((code << 2) | spare);
        }
        uint4 v;
        __builtin_memcpy(&v, o, 16);
        *reinterpret_cast<uint4 *>(dst + 1024 * j) = v;
    }
}

__global__ __launch_bounds__(256) void unpack_w6_kernel(const uint8_t *__restrict__ packed, int N,
                                                        int K, int8_t *__restrict__ wq)
{
    const long gid = (long)blockIdx.x * 256 + threadIdx.x;
    const int kt = K / FLEXQ_TILE_K;
    const long tiles = (long)(N / FLEXQ_TILE_ROWS) * kt;
    const long tile = gid >> 6;
    const int lane = (int)(gid & 63);
    if (tile >= tiles) return;
    const long nb = tile / kt, kb = tile % kt;
    const int r = lane & 31, h = lane >> 5;
    PackedTile t = load_packed_tile_cached(
        reinterpret_cast<const v4i *>(packed + tile * FLEXQ_TILE_BYTES), lane);
    int8_t *row = wq + (nb * FLEXQ_TILE_ROWS + r) * (long)K + kb * FLEXQ_TILE_K + 16 * h;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v4i d = unpack_kstep(t, j);            // bytes hold 4*w
        int8_t b[16];
        __builtin_memcpy(b, &d, 16);
#pragma unroll
        for (int i = 0; i < 16; ++i) b[i] = (int8_t)(b[i] >> 2);
        uint4 v;
        __builtin_memcpy(&v, b, 16);
        *reinterpret_cast<uint4 *>(row + 32 * j) = v;
    }
}

// Activations in tile order (tiles of 32 tokens x 128 k: four 1 KiB planes of int8, or
// the three planes of the packed 6-bit format) back to row-major int8 codes [M][K].
__global__ __launch_bounds__(256) void untile_act_kernel(const uint8_t *__restrict__ xt, int bits, int M,
                                                         int K, int8_t *__restrict__ xq)
{
    const long gid = (long)blockIdx.x * 256 + threadIdx.x;
    const int kt = K / FLEXQ_TILE_K;
    const long tiles = (long)((M + 31) / 32) * kt;
    const long tile = gid >> 6;
    const int lane = (int)(gid & 63);
    if (tile >= tiles) return;
    const long mb = tile / kt, kb = tile % kt;
    const int r = lane & 31, h = lane >> 5;
    if (mb * 32 + r >= M) return;                       // a padding row of the last block
    int8_t *row = xq + (mb * 32 + r) * (long)K + kb * FLEXQ_TILE_K + 16 * h;
    if (bits == 8) {
        const uint4 *src = reinterpret_cast<const uint4 *>(xt + tile * 4096) + lane;
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<uint4 *>(row + 32 * j) = src[64 * j];
        return;
    }
    PackedTile t = load_packed_tile_cached(reinterpret_cast<const v4i *>(xt + tile * FLEXQ_TILE_BYTES), lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v4i d = unpack_kstep(t, j);            // bytes hold 4*x
        int8_t b[16];
        __builtin_memcpy(b, &d, 16);
#pragma unroll
        for (int i = 0; i < 16; ++i) b[i] = (int8_t)(b[i] >> 2);
        uint4 v;
        __builtin_memcpy(&v, b, 16);
        *reinterpret_cast<uint4 *>(row + 32 * j) = v;
    }
}

// Scales out of the packed buffer; group mode: tile order [N/32][K/128][32] back to [N][K/128].
__global__ void unpack_scales_kernel(const uint16_t *__restrict__ src, int N, int K, int group,
                                     uint16_t *__restrict__ dst)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (group == 0) {
        if (i < N) dst[i] = src[i];
        return;
    }
    const int kt = K / FLEXQ_TILE_K;
    if (i >= (long)N * kt) return;
    const long n = i / kt, g = i % kt;
    dst[i] = src[((n / 32) * kt + g) * 32 + (n % 32)];
}

__global__ void fill_zero_kernel(unsigned *p, long count)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

}  // namespace

namespace flexq {

hipError_t launch_quant_w6(const float *w, int N, int K, int group, int8_t *wq, uint16_t *sw,
                           hipStream_t st)
{
    if (group != 0) {
        const long chunks = (long)N * K / 4;
        hipLaunchKernelGGL(quant_w6_g128_kernel, dim3((unsigned)((chunks + 1023) / 1024)), dim3(256), 0, st, w,
                           chunks, wq, sw);
        return hipGetLastError();
    }
#define FLEXQ_QUANT_ROW(CH, T) \
    hipLaunchKernelGGL((quant_w6_row_kernel<CH, T>), dim3((unsigned)N), dim3(T), 0, st, w, K, wq, sw)
    // at most eight float4 a lane (sixteen for the longest rows), so that enough lanes are
    // resident to keep a CU's share of HBM busy
    if (K <= 2048)
        FLEXQ_QUANT_ROW(2, 256);
    else if (K <= 4096)
        FLEXQ_QUANT_ROW(4, 256);
    else if (K <= 8192)
        FLEXQ_QUANT_ROW(8, 256);
    else if (K <= 16384)
        FLEXQ_QUANT_ROW(8, 512);
    else if (K <= 32768)
        FLEXQ_QUANT_ROW(8, 1024);
    else if (K <= 65536)
        FLEXQ_QUANT_ROW(16, 1024);
    else
        return hipErrorInvalidValue;            // longer rows are refused by the caller
#undef FLEXQ_QUANT_ROW
    return hipGetLastError();
}

hipError_t launch_pack_w6(const int8_t *wq, const uint16_t *sw, int N, int K, int group,
                          void *packed, hipStream_t st)
{
    const long lanes = (long)(N / 32) * (K / 128) * 64;
    hipLaunchKernelGGL(pack_w6_kernel, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st, wq, sw,
                       N, K, group, (uint8_t *)packed);
    return hipGetLastError();
}

hipError_t launch_unpack_w6(const void *packed, int N, int K, int group, int8_t *wq, uint16_t *sw,
                            hipStream_t st)
{
    const long lanes = (long)(N / 32) * (K / 128) * 64;
    hipLaunchKernelGGL(unpack_w6_kernel, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st,
                       (const uint8_t *)packed, N, K, wq);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint16_t *src = (const uint16_t *)((const uint8_t *)packed + (size_t)N * K * 6 / 8);
    const long count = group == 0 ? N : (long)N * (K / 128);
    hipLaunchKernelGGL(unpack_scales_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, src,
                       N, K, group, sw);
    return hipGetLastError();
}

hipError_t launch_untile_act(const uint8_t *xt, int act_bits, int M, int K, int8_t *xq, hipStream_t st)
{
    const long lanes = (long)((M + 31) / 32) * (K / 128) * 64;
    hipLaunchKernelGGL(untile_act_kernel, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st, xt,
                       act_bits, M, K, xq);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t st)
{
    const long count = (long)(bytes / 4);
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                       (unsigned *)p, count);
    return hipGetLastError();
}

}  // namespace flexq
