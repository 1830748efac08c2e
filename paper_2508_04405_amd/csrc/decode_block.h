// Arguments of the one-launch decoder block (decode_block.hip).
#pragma once
#include "flexq_kernels.h"

namespace flexq {

constexpr int kDecodeGrid = 256;               // workgroups: one per CU of an MI355X
constexpr int kDecodeLds = 158 * 1024;         // dynamic LDS of a workgroup at most

struct DecodePhase {         // one linear
    const void *packed;
    const uint16_t *scales;
    const int8_t *xq;        // its codes [M, 128 kt] and token scales, written by its producer
    uint16_t *sx;
    uint16_t *y;             // [M, 32 nb]
    int nb, kt;              // row blocks of 32 channels, 128-k tiles per row block
    int off;                 // row block 0 belongs to this workgroup
    unsigned inv;            // 2^32 / (8 kt), rounded up
};
struct DecodeProducer {      // what makes its codes
    const uint16_t *in, *gamma;
    int8_t *xq;
    uint16_t *sx;
    int L, mode;             // row length; mode as in producers.hip
    int dep;                 // the linear whose outputs it reads, or -1
    int first;               // number of its first piece among those of all producers with dep -1, else 0
    float qmax;
};
struct DecodeArgs {
    DecodePhase ph[4];
    DecodeProducer pr[4];
    int n, M, group;
    float eps;
    unsigned *words;         // counter area of the workspace
    int spin;                // polls before a workgroup stops waiting
};

// Pieces of a token's row, one per workgroup: of 4096, or the whole row for the norm, whose fp32 sum of
// squares has the order of the stand-alone kernel's 256 or 512 lanes.
__host__ __device__ inline int decode_pieces(int mode, int L) { return mode == 0 ? 1 : (L + 4095) / 4096; }

int decode_block_lds(int M, int K);
hipError_t launch_decode_block(const DecodeArgs &a, int lds_bytes, hipStream_t st);

}  // namespace flexq
