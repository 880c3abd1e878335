// What the two large-M kernels (lords_prefill_kernel.h, lords_prefill_wide.hip) share: the arguments of a launch, code pairs.
#pragma once
#include "lords_decode_common.h"

namespace lords {

// One weight matrix of a launch.  Several matrices that read the same X (and are cut into tiles of the same shape) can
// share a launch: each gets a contiguous range of blockIdx.x, a multiple of eight long, and keeps the cut of the sums over K that it
// would have alone, so they are the same bit for bit.  Layers too small to fill the chip run beside each other and
// the last round of one is filled by the next; where a tile is cut into parts to fill the chip alone, one workgroup may take several
// of them.  q, k, v (4096 + 1024 + 1024 rows x 4096, 4 bits, rank 32) in one launch, us, no tiles in parts / in parts as alone / parts by
// workgroup and tiles chosen for the launch: 64 tokens 46 / 45 / 42, 256 40 / 48 / 33, 512 77 / 63 / 58, 1024 91 / 111 / 84,
// 2048 160 / 148 / 129; three of 1088 x 1088, 1360 tokens 31 / 63 / 38.
struct PfLayer {
    const uint8_t *codes;
    const void *B;         // N x rf, bf16 or fp32
    const void *A;         // rf x K, bf16 or fp32
    void *Y;
    const float *gate;     // M x N fp32 or null: Y = silu(gate) * (the product) instead of the product
    float *part;           // per workgroup: the accumulators of a part that does not start at the tile's first column
    uint32_t *arrived;     // per output tile: parts handed over so far, or lords_meet.h's count (zero before and after a launch)
    int N;
    int nt;                // tiles along N
    int per;               // work units (one K tile of one output tile) per workgroup, or per 2^meet; units are numbered tile by tile
    int meet;              // 0, or 1 .. 3: each tile is cut into 2^meet parts, one workgroup each, that finish it together
    int walk;              // 0, or 1 .. 3: each tile is cut into 2^(meet + walk) parts, 2^walk of them one workgroup's
    int xcd;               // tiles in parts: where those that do not go round evenly begin
    int x0, gx;            // first blockIdx.x of this matrix and how many it has (multiples of 8)
};

template <int NLAYERS>
struct PrefillArgsT {
    const uint16_t *X;
    const float *codebook;
    int M, K;
    int r;                 // contraction length of the scales: rf, or 3 rf for fp32 factors (hi/lo parts, see the kernel)
    int rf;                // rank of the factors
    int y_f32;
    int row_bytes;
    int mt;                // tiles along M
    int ntiles_k;          // ceil(K / 128)
    int tiled;             // codes in the slab-tile layout: tile (slab, K tile) contiguous, chunk = 16 g + c
    int L;                 // matrices
    int polls;             // how often a workgroup of a tile that meets looks for the others' parts before it leaves
    PfLayer layer[NLAYERS];
};

constexpr int kPfCopies = 8;                               // of the level table

template <int BITS>
__device__ __forceinline__ uint32_t pair_index(const uint32_t (&w)[BITS], int p)
{
    const int o = 2 * BITS * p, d = o >> 5, s = o & 31;
    uint32_t v = w[d] >> s;
    if (s + 2 * BITS > 32) v |= w[(d + 1) < BITS ? d + 1 : d] << (32 - s);
    return v & ((1u << (2 * BITS)) - 1u);
}

// Tile shape: padded contraction / 32, waves along the tokens and the rows, token blocks per wave.
struct PfShape {
    int ss, wm, wn, mb;
    bool f32fact;
};
hipError_t launch_prefill_2bit(const PrefillArgsT<1> &a, const PfShape &d, dim3 grid, hipStream_t st);
hipError_t launch_prefill_2bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st);
hipError_t launch_prefill_3bit(const PrefillArgsT<1> &a, const PfShape &d, dim3 grid, hipStream_t st);
hipError_t launch_prefill_3bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st);
hipError_t launch_prefill_4bit(const PrefillArgsT<1> &a, const PfShape &d, dim3 grid, hipStream_t st);
hipError_t launch_prefill_4bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st);
// The form of the kernel with one wave per SIMD: 256 x 256 tiles, bf16 factors of rank 33 .. 64 (lords_prefill_wide.hip).
hipError_t launch_prefill_wide(const PrefillArgsT<1> &a, dim3 grid, int bits, hipStream_t st);
hipError_t launch_prefill_wide(const PrefillArgsT<kMaxBatch> &a, dim3 grid, int bits, hipStream_t st);

}  // namespace lords
