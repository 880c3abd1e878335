// Large products in two passes:  Y = X W^T  with  W = C[Q] (.) (B A)  dequantised once.
//
// The large-M kernel (lords_prefill_kernel.h) dequantises a tile's weights again for every 256 tokens.  That is the larger part
// of what it does besides the product: on 16384 x 16384, 2048 tokens, a K tile of 256 x 256 takes 3.4 us, the same loop
// without table reads, scales and roundings (a timing-only build) 2.0 us.  Its matrix pipes are busy for 52 % of its cycles, those
// of pass 2 for 59 % (14336 x 4096, 2048 tokens, both at 2.0 to 2.2 GHz by the counters); a second form of it with half the LDS
// reads and one wave per SIMD took the same time.  With enough tokens it is cheaper to write W out once as bf16 and to read it
// back as MFMA operands:
//
//   pass 1  dequant_operand_kernel: codes, B, A -> W in scratch, in the order in which pass 2 wants it in its registers
//   pass 2  operand_gemm_kernel:    Y = X W^T, W straight from memory into registers, X through LDS
//
// The arithmetic is that of the large-M kernel on whole tiles, operation by operation (scales by MFMA over the rank, fp16
// level times fp32 scale, one rounding to bf16, products in the same order along K), so the results are the same bit for bit.
//
// W in scratch: slab s of 16 rows, K tile t of 128 columns, stage u = 0 .. 3: 1 KB at ((s * ntiles_k + t) * 4 + u) * 1024;
// lane l = (c = l % 16, g = l / 16) finds its a-operand of v_mfma_f32_16x16x32_bf16, row 16 s + c, columns 128 t + 32 g + 8 u .. + 8,
// at 16 l in it.  Columns beyond K and rows beyond N are zeros.
#include <algorithm>
#include <type_traits>
#include "lords_operand.h"

namespace lords {

// ---------------------------------------------------------------------------------------------
// pass 1
// ---------------------------------------------------------------------------------------------
struct OperandLayer {
    const uint8_t *codes;
    const void *B;         // N x rf
    const void *A;         // rf x K
    uint8_t *W;            // scratch
    int N, x0;             // rows; first workgroup
};
struct OperandArgs {
    const float *codebook;
    int K, r, rf;          // r: contraction length of the scales: rf, or 3 rf for fp32 factors
    int row_bytes, ntiles_k, tiled;
    int per_wave;          // slabs per wave
    int L;
    OperandLayer layer[kMaxBatch];
};

constexpr int kOpCopies = 16;                                  // of the level table

// A workgroup takes two neighbouring K tiles (waves 0, 1 and 2, 3: the code rows of both lie in the same cache lines) and
// 2 per_wave slabs.  A wave keeps the A operands of its K tile in registers (up to rank 64; above they are read again
// from LDS) and walks its slabs, the next one's codes requested before this one's are used.
// Bound by the writes: 14336 x 4096 at rank 32, 117 MB, 28 to 31 us (4.0 TB/s); at padded contraction 128 by the conversion as
// well (44 to 53 us), at six times 32 by the scale contraction (159).
template <int BITS, int SS, bool F32>
__global__ __launch_bounds__(256) void dequant_operand_kernel(OperandArgs a)
{
    constexpr int RP = 32 * SS, NL = 1 << BITS, NE = 1 << (2 * BITS);
    constexpr bool kKeepA = SS <= 2;
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    using Pair = std::conditional_t<F32, f32x2_t, uint32_t>;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *As = smem;                                   // [2][RP][256 B], chunks swizzled by row
    Pair *lut = reinterpret_cast<Pair *>(smem + 2 * RP * 256);  // [NE][kOpCopies]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, kh = wave >> 1;
    int li = 0;
    while (li + 1 < a.L && (int)blockIdx.x >= a.layer[li + 1].x0) ++li;
    const OperandLayer ly = a.layer[li];
    const int N = ly.N, K = a.K, nslabs = (N + 15) >> 4, npairs = (a.ntiles_k + 1) >> 1;
    const int bx = (int)blockIdx.x - ly.x0;
    const int kt = 2 * (bx % npairs) + kh, s0 = (bx / npairs) * 2 * a.per_wave;

    for (int id = tid; id < NE * kOpCopies; id += 256) {
        const int idx = id / kOpCopies;
        const float l0 = a.codebook[idx & (NL - 1)], l1 = a.codebook[idx >> BITS];
        if constexpr (F32) {
            lut[id] = Pair{l0, l1};
        } else {
            f16x2 h;
            h[0] = (_Float16)l0;
            h[1] = (_Float16)l1;
            lut[id] = __builtin_bit_cast(uint32_t, h);
        }
    }
    // ---- both A tiles: 16-byte chunk kc of rank row j in slot kc ^ (j & 15) of its 256 bytes; rows beyond the rank and
    //      columns beyond K are zeros
    for (int id = tid; id < 2 * (F32 ? RP / 3 : RP) * 16; id += 256) {
        const int h = id / ((F32 ? RP / 3 : RP) * 16), q = id % ((F32 ? RP / 3 : RP) * 16), j = q >> 4, kc = q & 15;
        const int k = (2 * (bx % npairs) + h) * 128 + 8 * kc;
        unsigned char *tile = As + h * RP * 256;
        const bool live = j < a.rf && k < K;
        if constexpr (F32) {
            if (j < a.rf) {
                f32x4 v[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
                if (live) {
                    const f32x4 *src = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(ly.A) + (size_t)j * K + k);
                    v[0] = src[0];
                    v[1] = src[1];
                }
                u32x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x0 = v[e >> 1][2 * (e & 1)], x1 = v[e >> 1][2 * (e & 1) + 1];
                    const uint16_t h0 = bf16_bits(x0), h1 = bf16_bits(x1);
                    hi[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                    lo[e] = (uint32_t)bf16_bits(x0 - bf16_to_f32(h0)) | ((uint32_t)bf16_bits(x1 - bf16_to_f32(h1)) << 16);
                }
#pragma unroll
                for (int seg = 0; seg < 3; ++seg) {
                    const int row = seg * a.rf + j;
                    *reinterpret_cast<u32x4 *>(tile + row * 256 + ((kc ^ (row & 15)) * 16)) = seg == 1 ? lo : hi;
                }
            }
        } else {
            u32x4 v = u32x4{0u, 0u, 0u, 0u};
            if (live) v = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint16_t *>(ly.A) + (size_t)j * K + k);
            *reinterpret_cast<u32x4 *>(tile + j * 256 + ((kc ^ (j & 15)) * 16)) = v;
        }
    }
    if constexpr (F32)
        for (int id = tid; id < 2 * (RP - a.r) * 16; id += 256) {
            const int h = id / ((RP - a.r) * 16), q = id % ((RP - a.r) * 16);
            *reinterpret_cast<u32x4 *>(As + h * RP * 256 + (a.r + (q >> 4)) * 256 + (q & 15) * 16) = u32x4{0u, 0u, 0u, 0u};
        }
    __syncthreads();
    if (kt >= a.ntiles_k) return;

    const unsigned char *Ap = As + kh * RP * 256;
    auto read_Aop = [&](int s, int t) __attribute__((always_inline)) -> bf16x8 {
        typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
        const int row0 = 32 * s + 8 * g + (c >> 2), kc = 4 * (c & 3) + (t >> 1);
        const unsigned char *p0 = Ap + row0 * 256 + ((kc ^ (row0 & 15)) * 16) + (t & 1) * 8;
        const unsigned char *p1 = Ap + (row0 + 4) * 256 + ((kc ^ ((row0 + 4) & 15)) * 16) + (t & 1) * 8;
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)p0);
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)p1);
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    bf16x8 Aop[kKeepA ? 8 : 1][SS];
    if constexpr (kKeepA) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int s = 0; s < SS; ++s) Aop[t][s] = read_Aop(s, t);
    }
    // Codes of a lane (row n, group g of this K tile), see lords_prefill_kernel.h; groups beyond K: the row's last one (their
    // weights are zeros).
    auto load_codes = [&](int s, uint32_t (&w)[BITS]) __attribute__((always_inline)) {
        const int n = min(16 * s + c, N - 1);
        const uint8_t *p = a.tiled ? ly.codes + ((((size_t)(n >> 4) * a.ntiles_k + kt) * 64) + 16 * g + (n & 15)) * (4 * BITS)
                                   : ly.codes + (size_t)n * a.row_bytes + (size_t)min(4 * kt + g, (K >> 5) - 1) * (4 * BITS);
        load_group<BITS>(p, w);
    };
    auto load_B = [&](int sl, u32x4 (&b)[SS]) __attribute__((always_inline)) {
        const int n = 16 * sl + c;
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            const int j0 = 32 * s + 8 * g;
            if constexpr (F32) {
                typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
                s16x8 t;
                const float *row = reinterpret_cast<const float *>(ly.B) + (size_t)min(n, N - 1) * a.rf;
                if ((a.rf & 3) == 0) {
                    // (four entries lie in one part: one load)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int jj = j0 + 4 * h, j = jj < a.rf ? jj : jj < 2 * a.rf ? jj - a.rf : jj - 2 * a.rf;
                        const bool live = n < N && jj < a.r;
                        const f32x4 x = *reinterpret_cast<const f32x4 *>(row + (live ? j : 0));
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint16_t hi = bf16_bits(x[e]), part = jj >= 2 * a.rf ? bf16_bits(x[e] - bf16_to_f32(hi)) : hi;
                            t[4 * h + e] = live ? (short)part : (short)0;
                        }
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int jj = j0 + e, j = jj < a.rf ? jj : jj < 2 * a.rf ? jj - a.rf : jj - 2 * a.rf;
                        t[e] = 0;
                        if (n < N && jj < a.r) {
                            const uint16_t hi = bf16_bits(row[j]);
                            t[e] = (short)(jj >= 2 * a.rf ? bf16_bits(row[j] - bf16_to_f32(hi)) : hi);
                        }
                    }
                }
                b[s] = __builtin_bit_cast(u32x4, t);
            } else {
                const uint16_t *B16 = reinterpret_cast<const uint16_t *>(ly.B);
                b[s] = rank8_fetch(B16, reinterpret_cast<const uint16_t *>(ly.A), min(n, N - 1), j0, N, a.r);
            }
        }
    };
    // G slabs at a time (above rank 64, where the A operands are read again for each, two)
    constexpr int G = kKeepA ? 1 : 2;
    const int slabs = min(s0 + 2 * a.per_wave, nslabs);
    int s = s0 + (wave & 1) * G;
    if (s >= slabs) return;
    uint32_t cw[G][BITS];
    u32x4 bw[G][SS];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        load_codes(min(s + i, nslabs - 1), cw[i]);
        load_B(min(s + i, nslabs - 1), bw[i]);
    }
    const uint32_t laneoff = lane & (kOpCopies - 1);
    for (; s < slabs; s += 2 * G) {
        uint32_t cn[G][BITS];
        u32x4 bn[G][SS];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            load_codes(min(s + 2 * G + i, nslabs - 1), cn[i]);
            if constexpr (G == 1) load_B(min(s + 2 * G + i, nslabs - 1), bn[i]);
        }
        bf16x8 Bop[G][SS];
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int q = 0; q < SS; ++q) {
                u32x4 t = bw[i][q];
                if constexpr (!F32) {
                    const int n = min(16 * (s + i) + c, N - 1);
                    t = rank8_fix(t, reinterpret_cast<const uint16_t *>(ly.B), n, 32 * q + 8 * g, N, a.r, 16 * (s + i) + 16 > N - 8);
                    if (16 * (s + i) + c >= N) t = u32x4{0u, 0u, 0u, 0u};
                }
                Bop[i][q] = __builtin_bit_cast(bf16x8, t);
            }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            f32x4 S[G][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < G; ++i) S[i][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < SS; ++q) {
                    const bf16x8 Aq = kKeepA ? Aop[kKeepA ? 2 * u + h : 0][q] : read_Aop(q, 2 * u + h);
#pragma unroll
                    for (int i = 0; i < G; ++i) S[i][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Aq, Bop[i][q], S[i][h], 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < G; ++i) {
                bf16x8 w;
#pragma unroll
                for (int pp = 0; pp < 4; ++pp) {
                    const int o = 2 * BITS * (4 * u + pp), d = o >> 5, sh = o & 31;
                    uint32_t v = cw[i][d] >> sh;
                    if (sh + 2 * BITS > 32) v |= cw[i][(d + 1) < BITS ? d + 1 : d] << (32 - sh);
                    const Pair lv = lut[(v & (NE - 1)) * kOpCopies + laneoff];
                    const float a0 = S[i][pp >> 1][2 * (pp & 1)], a1 = S[i][pp >> 1][2 * (pp & 1) + 1];
                    if constexpr (F32) {
                        w[2 * pp] = (__bf16)(lv.x * a0);
                        w[2 * pp + 1] = (__bf16)(lv.y * a1);
                    } else {
                        const f16x2 h = __builtin_bit_cast(f16x2, lv);
                        w[2 * pp] = (__bf16)__builtin_fmaf((float)h[0], a0, 0.0f);
                        w[2 * pp + 1] = (__bf16)__builtin_fmaf((float)h[1], a1, 0.0f);
                    }
                }
                if (G == 1 || s + i < slabs)
                    *reinterpret_cast<bf16x8 *>(ly.W + (((size_t)(s + i) * a.ntiles_k + kt) * 4 + u) * 1024 + 16 * lane) = w;
            }
        }
#pragma unroll
        for (int i = 0; i < G; ++i) {
#pragma unroll
            for (int q = 0; q < BITS; ++q) cw[i][q] = cn[i][q];
            if constexpr (G == 1) {
#pragma unroll
                for (int q = 0; q < SS; ++q) bw[i][q] = bn[i][q];
            } else {
                load_B(min(s + 2 * G + i, nslabs - 1), bw[i]);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// pass 2
// ---------------------------------------------------------------------------------------------
struct GemmLayer {
    const uint8_t *W;
    void *Y;
    int N, ld;             // rows of W, outputs per token of Y
    int n0;                // first column of tiles
};
struct GemmArgs {
    const uint16_t *X;
    int M, K, ntiles_k;
    int y_f32;
    int mt, nt;            // tiles along M, along N (all matrices)
    int group;             // tiles along M that neighbouring workgroups share
    int L;
    GemmLayer layer[kMaxBatch];
};

// R: slabs of 16 rows per wave; a tile is 64 R rows x 256 tokens, four waves side by side along the rows, one per SIMD.
// PAIR: matrices 0 and 1 are a gate/up pair; the wave's slabs are R / 2 of the gate and the same R / 2 of up, and
// Y[0] = silu(gate) * up.
template <int R, bool PAIR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void operand_gemm_kernel(GemmArgs a)
{
    constexpr int MB = 16, BN = (PAIR ? 32 : 64) * R, RS = PAIR ? R / 2 : R, BM = 256, XBUF = BM * 256;
    extern __shared__ __align__(16) unsigned char smem[];       // [2][64 token groups][1 KB]
    unsigned char *Xs = smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int M = a.M, K = a.K, ntk = a.ntiles_k, nk2 = (ntk + 1) & ~1;

    // ---- tiles of this workgroup: XCD x owns a contiguous eighth of them, its workgroups take turns
    const int total = a.mt * a.nt, per_xcd = (total + 7) >> 3, wgs_xcd = (int)gridDim.x >> 3;
    const int xcd = (int)blockIdx.x & 7, first = xcd * per_xcd, last = min(first + per_xcd, total);
    int T = first + ((int)blockIdx.x >> 3);
    if (T >= last) return;

    // ---- staging of X (layout as in lords_prefill_kernel.h)
    constexpr int XJ = 16;
    const int xt0 = 4 * wave + ((lane >> 3) & 3);
    const int xv = (lane & 7) ^ (xt0 & 7);
    const int xkcol = 32 * (xv & 3) + 8 * (xv >> 2) + 16 * (lane >> 5);
    uint32_t xo[XJ];
#pragma unroll
    for (int j = 0; j < XJ; ++j) xo[j] = ((uint32_t)(xt0 + 16 * j) * (uint32_t)K + (uint32_t)xkcol) * 2u;
    const uint32_t xl0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(Xs + wave * 1024));
    // (a ragged last K tile: chunks beyond K are fetched from further left, any finite data of the row will do)
    auto shift_X = [&](int kt) __attribute__((always_inline)) -> uint32_t { return (uint32_t)min(2 * (K - 8 - xkcol - kt * 128), 0); };
    const uint32_t wslab = (uint32_t)ntk * 4096u;               // bytes of a slab of W
    uint32_t wo[RS];
#pragma unroll
    for (int q = 0; q < RS; ++q) wo[q] = (uint32_t)q * wslab + 16u * (uint32_t)lane;

    // ---- where a tile's operands lie: X rows from m_blk on, the wave's slabs of W
    struct Src { uint64_t x, w[PAIR ? 2 : 1]; uint32_t xbytes, wbytes; };
    struct Tile { int m_blk, n_blk, li; };
    auto tile_of = [&](int t) __attribute__((always_inline)) -> Tile {
        const int in_group = a.group * a.nt, gr = t / in_group, rem = t - gr * in_group;
        const int gm = min(a.group, a.mt - gr * a.group), n = rem / gm;
        int li = 0;
        if (!PAIR)
            while (li + 1 < a.L && n >= a.layer[li + 1].n0) ++li;
        return Tile{(gr * a.group + rem - n * gm) * BM, (n - a.layer[li].n0) * BN, li};
    };
    auto src_of = [&](Tile t, bool live) __attribute__((always_inline)) -> Src {
        Src s;
        const GemmLayer &ly = a.layer[t.li];
        const int slab0 = (t.n_blk >> 4) + RS * wave, nslabs = (ly.N + 15) >> 4;
        s.x = (uint64_t)(uintptr_t)a.X + (uint64_t)t.m_blk * (uint64_t)K * 2u;
        s.xbytes = live ? (uint32_t)min(M - t.m_blk, BM) * (uint32_t)K * 2u : 0u;
        s.w[0] = (uint64_t)(uintptr_t)ly.W + (uint64_t)slab0 * wslab;
        if constexpr (PAIR) s.w[1] = (uint64_t)(uintptr_t)a.layer[1].W + (uint64_t)slab0 * wslab;
        s.wbytes = live ? (uint32_t)max(min(nslabs - slab0, RS), 0) * wslab : 0u;
        return s;
    };
    auto rsrc_X = [&](const Src &s, int kt) __attribute__((always_inline)) {
        return make_rsrc(s.x + (uint64_t)kt * 256u, kt < ntk && s.xbytes ? s.xbytes - (uint32_t)kt * 256u : 0u);
    };
    auto rsrc_W = [&](const Src &s, int i, int kt) __attribute__((always_inline)) -> __amdgpu_buffer_rsrc_t {
        const uint64_t b = s.w[i] + (uint64_t)kt * 4096u;
        return __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32) |
                                                                    (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b)), 0,
                                                 __builtin_amdgcn_readfirstlane(kt < ntk && s.wbytes ? s.wbytes - (uint32_t)kt * 4096u : 0u), 0x00020000);
    };

    f32x4 acc[R][MB];
    bf16x8 W[2][4][R], Xq[8];
    auto load_W = [&](__amdgpu_buffer_rsrc_t r, int i, int q, int u, bf16x8 &w) __attribute__((always_inline)) {
        w = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, wo[q] + u * 1024, 0, 0));
    };
    uint32_t xr = (uint32_t)((c >> 2) * 1024 + (c & 3) * 128 + ((g ^ (c & 7)) * 16));     // X operand of stage 0, block 0, buffer 0
    auto read_X = [&](int buf, int u, int mb) __attribute__((always_inline)) -> bf16x8 {
        return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>((uintptr_t)((xr ^ (uint32_t)((u & 1) * 64 + buf * XBUF)) + (u >> 1) * 512 + mb * 4096));
    };
    constexpr int kAhead = 4;

    Tile tile = tile_of(T);
    Src src = src_of(tile, true);
    {
        const BufferRsrc rX = rsrc_X(src, 0);
#pragma unroll
        for (int j = 0; j < XJ; ++j) lds_buffer_16(rX, xo[j], shift_X(0), xl0, j);
#pragma unroll
        for (int i = 0; i < (PAIR ? 2 : 1); ++i) {
            const __amdgpu_buffer_rsrc_t rW = rsrc_W(src, i, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < RS; ++q) load_W(rW, i, q, u, W[0][u][i * RS + q]);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAhead; ++i) Xq[i] = read_X(0, 0, i);

    for (;;) {
        const int Tn = T + wgs_xcd;
        const bool more = Tn < last;
        const Tile next = tile_of(more ? Tn : T);
        const Src src_next = src_of(next, more);
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[q][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

        // K tile kt from buffer and registers P; what is fetched meanwhile: the next K tile (one beyond the last is all zeros,
        // so that their number is even), after the last one the first of the next output tile.
        auto k_tile = [&](int kt, auto parity) __attribute__((always_inline)) {
            constexpr int P = decltype(parity)::value;
            const bool wrap = kt + 1 == nk2;
            const int kf = wrap ? 0 : kt + 1;
            const Src &sf = wrap ? src_next : src;
            const BufferRsrc rX = rsrc_X(sf, kf);
            const __amdgpu_buffer_rsrc_t rW0 = rsrc_W(sf, 0, kf), rW1 = rsrc_W(sf, PAIR ? 1 : 0, kf);
            const uint32_t sx = shift_X(kf), xl = xl0 + (P ^ 1) * XBUF;
            asm volatile("" : "+v"(xr));                        // (operand addresses are made where they are used: registers)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4 * MB; ++t) {
                const int u = t / MB, mb = t % MB, tn = t + kAhead;
                const bf16x8 Xop = Xq[t & 7];
                mfma_acc(acc[0][mb], W[P][u][0], Xop);
                if (t == 4 * MB - kAhead) {
                    // what was fetched has landed, for every wave; every wave has read the last of this tile's X
                    __builtin_amdgcn_s_waitcnt(0x0070);
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                Xq[tn & 7] = tn < 4 * MB ? read_X(P, tn / MB, tn % MB) : read_X(P ^ 1, 0, tn - 4 * MB);
                __builtin_amdgcn_sched_barrier(0);
                mfma_acc(acc[1][mb], W[P][u][1], Xop);
                if (t >= 8 && (t & 1) == 0 && t < 8 + 8 * R) {
                    const int v = ((t - 8) / 2) / R, q = ((t - 8) / 2) % R;
                    load_W(q < RS ? rW0 : rW1, q / RS, q % RS, v, W[P ^ 1][v][q]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (R == 4) mfma_acc(acc[R / 2][mb], W[P][u][R / 2], Xop);
                if ((t & 1) == 1 && t < 1 + 2 * XJ) lds_buffer_16(rX, xo[(t - 1) / 2], sx, xl, (t - 1) / 2);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (R == 4) mfma_acc(acc[R - 1][mb], W[P][u][R - 1], Xop);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        for (int kt = 0; kt < nk2; kt += 2) {
            k_tile(kt, std::integral_constant<int, 0>{});
            k_tile(kt + 1, std::integral_constant<int, 1>{});
        }
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");        // (results of the last matrix instructions)

        // ---- epilogue: lane (c, g) holds token 16 mb + c, rows 16 q + 4 g .. + 3 of the wave's slabs
        const GemmLayer &ly = a.layer[tile.li];
        const int N = ly.N, ld = ly.ld, n_wave = tile.n_blk + 16 * RS * wave;
        const bool full = tile.m_blk + BM <= M && tile.n_blk + BN <= N;
        void *Yp = ly.Y;
        constexpr int GB = 4;                                   // token blocks at a time
#pragma unroll
        for (int b0 = 0; b0 < MB; b0 += GB) {
            f32x4 v[GB * RS];
#pragma unroll
            for (int i = 0; i < GB * RS; ++i) {
                if constexpr (PAIR) {
                    const f32x4 ga = read_acc(acc[i % RS][b0 + i / RS]), up = read_acc(acc[RS + i % RS][b0 + i / RS]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[i][e] = ga[e] / (1.0f + __expf(-ga[e])) * up[e];
                } else {
                    v[i] = read_acc(acc[i % RS][b0 + i / RS]);
                }
            }
            int m0 = tile.m_blk + 16 * b0 + c, n0 = n_wave + 4 * g;
            asm volatile("" : "+v"(m0), "+v"(n0));              // (addresses of one batch at a time: registers)
            if (full) {
#pragma unroll
                for (int i = 0; i < GB * RS; ++i) store_out4(Yp, (size_t)(m0 + 16 * (i / RS)) * ld + n0 + 16 * (i % RS), v[i], a.y_f32);
            } else {
#pragma unroll
                for (int i = 0; i < GB * RS; ++i) {
                    const int m = m0 + 16 * (i / RS), n = n0 + 16 * (i % RS);
                    if (m >= M) continue;
                    if (n + 3 < N) {
                        store_out4(Yp, (size_t)m * ld + n, v[i], a.y_f32);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (n + e >= N) continue;
                            if (a.y_f32) reinterpret_cast<float *>(Yp)[(size_t)m * ld + n + e] = v[i][e];
                            else reinterpret_cast<uint16_t *>(Yp)[(size_t)m * ld + n + e] = bf16_bits(v[i][e]);
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!more) return;
        T = Tn;
        tile = next;
        src = src_next;
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
constexpr int kOpCUs = 256;

// Contraction length of the scales padded to 32 times 1, 2, 4 or, with fp32 factors (three parts of each), 6.
static int op_ss(const BatchedProblem &p)
{
    const int rp = ((p.f32fact ? 3 * p.r : p.r) + 31) / 32;
    return rp <= 1 ? 1 : rp <= 2 ? 2 : rp <= 4 ? 4 : rp <= 6 && p.f32fact ? 6 : 0;
}

static size_t op_slab_bytes(const BatchedProblem &p) { return (size_t)((p.K + 127) / 128) * 4096; }

// Rows of each matrix that are taken at once: all of them (0), or whole tiles of them in chunks of about one size that
// kTwoPassBytes of W hold (one tile each where that is too little: more than two_pass_supported lets through).
static int op_chunk_rows(const BatchedProblem &p)
{
    size_t slabs = 0;
    for (int l = 0; l < p.L; ++l) slabs += (size_t)(p.N[l] + 15) / 16;
    const size_t fit = kTwoPassBytes / op_slab_bytes(p);
    if (slabs <= fit) return 0;
    int most = 0;
    for (int l = 0; l < p.L; ++l) most = p.N[l] > most ? p.N[l] : most;
    const int cap = (int)std::max<size_t>(fit / p.L / 16, 1) * 256, chunks = (most + cap - 1) / cap;
    return (most + 256 * chunks - 1) / (256 * chunks) * 256;
}

size_t two_pass_workspace_bytes(const BatchedProblem &p)
{
    const int rows = op_chunk_rows(p);
    size_t slabs = 0;
    for (int l = 0; l < p.L; ++l) slabs += (size_t)((rows ? (rows < p.N[l] ? rows : p.N[l]) : p.N[l]) + 15) / 16;
    return slabs * op_slab_bytes(p);
}

bool two_pass_supported(const BatchedProblem &p)
{
    if (p.L < 1 || p.L > kMaxBatch || op_ss(p) == 0 || (p.f32fact && p.tiled)) return false;
    // (32-bit offsets: 256 rows of X, four slabs of W; a chunk must hold a tile of every matrix)
    if ((size_t)p.K * 512 >= ((size_t)1 << 32)) return false;
    return (size_t)p.L * 16 * op_slab_bytes(p) <= kTwoPassBytes;
}

template <int BITS, int SS, bool F32>
static hipError_t launch_operand_t(const OperandArgs &a, unsigned grid, hipStream_t st)
{
    const size_t smem = (size_t)2 * 32 * SS * 256 + (size_t)(1 << (2 * BITS)) * kOpCopies * (F32 ? 8 : 4);
    static LdsOptIn lds_opt_in;
    const hipError_t e = allow_dynamic_lds(lds_opt_in, reinterpret_cast<const void *>(&dequant_operand_kernel<BITS, SS, F32>), smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((dequant_operand_kernel<BITS, SS, F32>), dim3(grid), dim3(256), smem, st, a);
    return hipGetLastError();
}

template <int R, bool PAIR>
static hipError_t launch_gemm_t(const GemmArgs &a, hipStream_t st)
{
    const size_t smem = 2 * 65536;
    static LdsOptIn lds_opt_in;
    const hipError_t e = allow_dynamic_lds(lds_opt_in, reinterpret_cast<const void *>(&operand_gemm_kernel<R, PAIR>), smem);
    if (e != hipSuccess) return e;
    const int per_xcd = (a.mt * a.nt + 7) / 8;
    hipLaunchKernelGGL((operand_gemm_kernel<R, PAIR>), dim3(8 * (per_xcd < kOpCUs / 8 ? per_xcd : kOpCUs / 8)), dim3(256), smem, st, a);
    return hipGetLastError();
}

// Piecewise linear through (x0, y0), (x1, y1), constant outside.
static double op_between(double x, double x0, double y0, double x1, double y1)
{
    return x <= x0 ? y0 : x >= x1 ? y1 : y0 + (y1 - y0) * (x - x0) / (x1 - x0);
}

// Time of pass 2 in us as the planner sees it: rounds of tiles, one per CU, each of K tiles and a fixed part.  A K tile takes
// longer the more CUs are at work (clocks) and the longer the rows (us, measured on 1000 .. 20000 rows, 256 .. 4096 tokens):
//   256 rows, 112 / 172 / 256 tiles at once: 1.75 / 2.47 / 2.98 at 4096 columns, 2.4 / 2.6 / 3.1 beyond 6144
//   128 rows, 128 / 256 tiles: 1.75 / 2.1 at 4096 columns, 1.8 / 3.0 at 14336
static double op_gemm_us(long tiles, int ntiles_k, int R)
{
    const long rounds = (tiles + kOpCUs - 1) / kOpCUs;
    const double at_once = (double)tiles / (double)rounds;
    const double lo = op_between(ntiles_k, 32, 1.8, 48, 2.4), mid = op_between(ntiles_k, 32, 2.47, 48, 2.6), hi = op_between(ntiles_k, 32, 2.98, 48, 3.1);
    const double t = R == 2 ? op_between(at_once, 128, 1.78, 256, op_between(ntiles_k, 32, 2.1, 112, 3.0))
                            : at_once < 172 ? op_between(at_once, 112, lo, 172, mid) : op_between(at_once, 172, mid, 256, hi);
    return (double)rounds * (((ntiles_k + 1) & ~1) * t + 6.0) + 2.0;
}

// Time of pass 1: us per 58.7 M weights (14336 x 4096), measured at 2, 3 and 4 bits alike to a tenth.
static double op_dequant_us(const BatchedProblem &p, double weights)
{
    const int ss = op_ss(p);
    double t = p.f32fact ? (ss <= 1 ? 42.0 : ss == 2 ? 50.0 : ss == 4 ? 97.0 : 155.0) : (ss <= 1 ? 29.0 : ss == 2 ? 34.0 : 46.0);
    if (p.f32fact && (p.r & 3)) t *= 1.9;                      // (entries of B one by one)
    return 4.0 + t * weights / 58.7e6;
}

// Tiles of pass 2 for rows row0 .. row0 + rows (0: all) of every matrix, 64 R rows each (a pair's: half of each matrix).
static long op_tiles(const BatchedProblem &p, int row0, int rows, int R)
{
    const int bn = p.act ? 32 * R : 64 * R;
    long t = 0;
    for (int l = 0; l < (p.act ? 1 : p.L); ++l) {
        const int n = rows ? (p.N[l] - row0 < rows ? p.N[l] - row0 : rows) : p.N[l];
        if (n > 0) t += (n + bn - 1) / bn;
    }
    return t * ((p.M + 255) / 256);
}

double two_pass_cost(const BatchedProblem &p)
{
    const int rows = op_chunk_rows(p), ntk = (p.K + 127) / 128;
    int most = 0;
    double weights = 0, us = 0;
    for (int l = 0; l < p.L; ++l) {
        most = p.N[l] > most ? p.N[l] : most;
        weights += (double)p.N[l] * p.K;
    }
    const int step = rows ? rows : most;
    for (int row0 = 0; row0 < most; row0 += step) {
        const double four = op_gemm_us(op_tiles(p, row0, rows, 4), ntk, 4);
        us += 4.0 + (p.act ? four : std::min(four, op_gemm_us(op_tiles(p, row0, rows, 2), ntk, 2)));
    }
    return us + op_dequant_us(p, weights);
}

// A cut-off of the planner, not a limit of the device: a gate of more bytes than this is not counted in the large-M kernel's way (its
// output alone would be 32 GB in bf16), so that such a pair is served or refused as that way has the memory for it.
constexpr double kGateMost = 64.0 * (1 << 30);
// What the estimate of tiles that meet leaves out of each product of a pair, us.  Of 80 pairs (137 .. 539 tokens) that it had drawn
// from the two passes to the large-M kernel, 52 were up to 17 % slower for it; of 70 others (185 .. 2390 tokens) that this term sends the
// other way, two passes are faster for 53, by 7 % in the middle and 25 % at most, and slower for the rest, by 9 % at most.  6528 x 2496,
// rank 15, 330 tokens: 74.5 in two passes, 82.3 by the large-M kernel.
constexpr double kPairMeets = 2.5;
// The large-M kernel's estimate reads high or low by the padded contraction (measured / estimated, the middle of 10 to 40
// products each, whole tiles and runs: bf16 factors 32 columns 1.0, 64 0.85, 128 0.82; fp32 factors 0.95, 0.92, 0.9, six times 32 1.15).
double large_cost(const BatchedProblem &p)
{
    const int ss = op_ss(p);
    const double scale = p.f32fact ? (ss == 1 ? 0.95 : ss == 2 ? 0.92 : ss == 4 ? 0.9 : 1.15) : (ss == 1 ? 1.0 : ss == 2 ? 0.85 : 0.82);
    auto products = [&](int M) {
        double us = 0;
        for (int l = 0; l < p.L; ++l) {
            MatmulProblem m = matrix_of(p, l);
            m.M = M;
            us += prefill_fast_cost(m) + (p.act && prefill_cut(m, ~(size_t)0).meet ? kPairMeets : 0.0);
        }
        return us;
    };
    // A pair: 2048 tokens at a time; the gate's fp32 sums go through memory (14336 rows, 2048 tokens, 235 MB in about 62 us).
    // (up to kGateMost)
    if (p.act && (double)std::min(p.M, 2048) * p.N[0] * 4.0 <= kGateMost) {
        const int pieces = p.M / 2048, rest = p.M % 2048;
        return scale * (pieces * products(2048) + (rest ? products(rest) : 0.0)) + (double)p.M * p.N[0] * 8.0 / 3.8e6;
    }
    const double us = products(p.M);
    return scale * (p.act || p.L == 1 ? us : std::min(us, prefill_batched_cost(p)));
}

// Whether the weights are dequantised once, in a pass of their own, or for every tile of tokens again.  Decided by the
// two planners' estimates, not by what has been allocated; the last twentieth is the margin.
//   us, large-M kernel / two passes:   1024 tokens   2048          4096
//   14336 x 4096 bf16 rank 32          120 / 122     231 / 223     455 / 427
//                bf16 rank 48          133 / 125     253 / 230     513 / 437
//                bf16 rank 100         241 / 137     434 / 232     878 / 445
//                fp32 rank 16          194 / 130     361 / 233     706 / 445
//                fp32 rank 64          814 / 248     1627 / 342    3249 / 572
//   4096 x 14336 bf16 rank 48          147 / 216     248 / 286     428 / 399
//   4096 x 4096  bf16 rank 48          56 / 76       93 / 97       136 / 117      (1024: in two parts that meet)
//   3000 x 2048  fp32 rank 64          109 / 73      199 / 86      394 / 90
// A pair (us, two products by the large-M kernel with the gate through memory / two passes; of 36 drawn pairs that go here
// since the estimate counts the gate's way, 0.28 .. 0.87 of the time, none slower):
//   14336 x 4096 bf16 rank 32          2048 tokens 507 / 445, 4096 1014 / 814
//   4096 x 4096                        4096 tokens 370 / 215;  8192 x 2048, 2048 tokens 163 / 131;  28672 x 8192, 2048 1737 / 1581
//   19771 x 1664, 2 bits, rank 26, 1217 tokens 259 / 209;  1264 x 416, fp32 rank 11, 3887 tokens 79 / 34
bool two_pass_faster(const BatchedProblem &p)
{
    if (p.M <= 128 || !two_pass_supported(p)) return false;
    for (int l = 0; l < p.L; ++l)
        if (!prefill_fast_supported(matrix_of(p, l))) return false;
    return two_pass_cost(p) < 0.95 * large_cost(p);
}

static hipError_t launch_two_pass_rows(const BatchedProblem &p, int row0, int rows, void *scratch, hipStream_t st)
{
    const int ss = op_ss(p), ntk = (p.K + 127) / 128;
    const size_t row_bytes = (size_t)p.K / 8 * p.bits, esz = p.f32fact ? 4 : 2;
    OperandArgs o;
    GemmArgs g;
    o.codebook = p.codebook;
    o.K = p.K; o.rf = p.r; o.r = p.f32fact ? 3 * p.r : p.r;
    o.row_bytes = (int)row_bytes; o.ntiles_k = ntk; o.tiled = p.tiled ? 1 : 0;
    o.L = 0;
    const int npairs = (ntk + 1) / 2;
    long slabs = 0;
    for (int l = 0; l < p.L; ++l) {
        const int n = rows ? (p.N[l] - row0 < rows ? p.N[l] - row0 : rows) : p.N[l];
        if (n <= 0) continue;
        slabs += (n + 15) / 16;
    }
    // a wave's share: long enough to pay for its A operands, short enough for four workgroups and more per CU
    long per = slabs * npairs / (2 * 1024);
    o.per_wave = (int)(per < 2 ? 2 : per > 16 ? 16 : per);
    const int mt = (p.M + 255) / 256;
    const int R = p.act || op_gemm_us(op_tiles(p, row0, rows, 4), ntk, 4) <= op_gemm_us(op_tiles(p, row0, rows, 2), ntk, 2) ? 4 : 2, BN = p.act ? 128 : 64 * R;
    g.X = (const uint16_t *)p.X;
    g.M = p.M; g.K = p.K; g.ntiles_k = ntk;
    g.y_f32 = p.f32out ? 1 : 0;
    g.mt = mt; g.nt = 0;
    g.group = mt < 8 ? mt : 8;
    uint8_t *W = (uint8_t *)scratch;
    unsigned x0 = 0;
    for (int l = 0; l < p.L; ++l) {
        const int n = rows ? (p.N[l] - row0 < rows ? p.N[l] - row0 : rows) : p.N[l];
        if (n <= 0) continue;
        OperandLayer &ol = o.layer[o.L];
        GemmLayer &gl = g.layer[o.L];
        ol.codes = (const uint8_t *)p.codes[l] + (p.tiled ? (size_t)(row0 / 16) * ntk * 256 * p.bits : (size_t)row0 * row_bytes);
        ol.B = (const uint8_t *)p.B[l] + (size_t)row0 * p.r * esz;
        ol.A = p.A[l];
        ol.W = W;
        ol.N = n;
        ol.x0 = (int)x0;
        const int ns = (n + 15) / 16;
        x0 += (unsigned)(npairs * ((ns + 2 * o.per_wave - 1) / (2 * o.per_wave)));
        gl.W = W;
        gl.Y = (uint8_t *)p.Y[l] + (size_t)row0 * (p.f32out ? 4 : 2);
        gl.N = n;
        gl.ld = p.N[l];
        gl.n0 = g.nt;
        g.nt += p.act && l ? 0 : (n + BN - 1) / BN;
        W += (size_t)ns * op_slab_bytes(p);
        ++o.L;
    }
    g.L = p.act ? 1 : o.L;
    hipError_t e = hipErrorInvalidValue;
#define LORDS_OPCASE(B_, S_, F_) if (p.bits == B_ && ss == S_ && p.f32fact == F_) e = launch_operand_t<B_, S_, F_>(o, x0, st);
    LORDS_OPCASE(2, 1, false) LORDS_OPCASE(2, 2, false) LORDS_OPCASE(2, 4, false)
    LORDS_OPCASE(3, 1, false) LORDS_OPCASE(3, 2, false) LORDS_OPCASE(3, 4, false)
    LORDS_OPCASE(4, 1, false) LORDS_OPCASE(4, 2, false) LORDS_OPCASE(4, 4, false)
    LORDS_OPCASE(2, 1, true) LORDS_OPCASE(2, 2, true) LORDS_OPCASE(2, 4, true) LORDS_OPCASE(2, 6, true)
    LORDS_OPCASE(3, 1, true) LORDS_OPCASE(3, 2, true) LORDS_OPCASE(3, 4, true) LORDS_OPCASE(3, 6, true)
    LORDS_OPCASE(4, 1, true) LORDS_OPCASE(4, 2, true) LORDS_OPCASE(4, 4, true) LORDS_OPCASE(4, 6, true)
#undef LORDS_OPCASE
    if (e != hipSuccess) return e;
    return p.act ? launch_gemm_t<4, true>(g, st) : R == 4 ? launch_gemm_t<4, false>(g, st) : launch_gemm_t<2, false>(g, st);
}

hipError_t launch_two_pass(const BatchedProblem &p, void *scratch, hipStream_t st)
{
    if (!two_pass_supported(p)) return hipErrorInvalidValue;
    const int rows = op_chunk_rows(p);
    if (!rows) return launch_two_pass_rows(p, 0, 0, scratch, st);
    int most = 0;
    for (int l = 0; l < p.L; ++l) most = p.N[l] > most ? p.N[l] : most;
    for (int row0 = 0; row0 < most; row0 += rows) {
        const hipError_t e = launch_two_pass_rows(p, row0, rows, scratch, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lords
