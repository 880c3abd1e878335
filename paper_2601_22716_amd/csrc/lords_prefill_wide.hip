// The large-M kernel of lords_prefill_kernel.h in the form for bf16 factors of rank 33 .. 64: 256 x 256 tiles, four waves of 64 rows x
// 256 tokens, one per SIMD.  At these ranks the scales cost two matrix instructions where rank 32 costs one, and
// the eight waves of 128 registers for operands have room for 128 tokens only, so every weight was dequantised again for
// every 128 tokens; a wave that has a SIMD and its 512 registers to itself holds the sums of 256 tokens in its 256 accumulation
// registers and everything else in the other half.  (At ranks up to 32, where eight waves of 32 rows x 256 tokens do the
// same work per weight, this form is no faster: 2048 x 14336 x 4096 227 against 230 us.)
//
// Work division, hand-over of parts and the lane mapping are those of lords_prefill_kernel.h; so is a K tile of four stages
// u = 0 .. 3.  The whole K range is one software pipeline, also across K tiles: under the 64 product MFMAs of a stage
// (16 token blocks x 4 slabs) ride the conversion of the next stage's weights (one pair per token block), the table reads
// five blocks ahead of it, and the scale MFMAs of the stage after it.  Instructions follow an MFMA two by two at most, LDS and
// vector ones behind different MFMAs: what a lone wave issues in the shadow of one (three vector instructions behind one
// cost 4 clocks, a vector and an LDS instruction behind the same one 8).
// LDS, all 160 KB at 4 bits: X tile twice 64 KB, three half tiles of A (64 ranks x 64 columns, those of two stages) 24 KB, level
// table 8 KB.  Per K tile one barrier that waits for loads and one that only frees a half tile of A.
// us, 128-token tiles / this: 28672 x 8192, 2 bits, rank 64, 256 tokens 157 / 141, 512 303 / 241, 1000 591 / 447; 14336 x 4096, 4 bits,
// rank 48, 768 tokens 132 / 112; 4096 x 14336, 3 bits, rank 48, 1000 tokens 154 / 136, 2048 288 / 227.
#include "lords_operand.h"
#include "lords_prefill.h"

namespace lords {

template <int BITS, bool MULTI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void prefill_wide_kernel(PrefillArgsT<MULTI ? kMaxBatch : 1> a)
{
    constexpr int SS = 2, R = 4, MB = 16, NT = 256, BN = 64 * R, BM = 16 * MB, NL = 1 << BITS, NE = 1 << (2 * BITS);
    constexpr int XBUF = BM * 256, AHALF = 32 * SS * 128;      // bytes: an X tile, half an A tile
    constexpr int NP = 4 * R;                                  // pairs of weights per lane and stage
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *Xs = smem;                                   // [2][BM / 4 token groups][1 KB]
    unsigned char *As = smem + 2 * XBUF;                        // [3][32 SS][128 B]
    uint32_t *lut = reinterpret_cast<uint32_t *>(smem + 2 * XBUF + 3 * AHALF);   // [NE][8] pairs of levels

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    int li = 0;
    if (MULTI)
        while (li + 1 < a.L && (int)blockIdx.x >= a.layer[li + 1].x0) ++li;
    const PfLayer ly = a.layer[MULTI ? li : 0];
    const int M = a.M, N = ly.N, K = a.K;

    const int total_units = ly.nt * a.mt * a.ntiles_k;
    const int bx = (int)blockIdx.x - ly.x0;
    const int wg = (bx & 7) * (ly.gx >> 3) + (bx >> 3);
    int unit = wg * ly.per;
    const int unit_end = min(unit + ly.per, total_units);
    if (unit >= unit_end) return;
    const uint16_t *A16 = reinterpret_cast<const uint16_t *>(ly.A), *B16 = reinterpret_cast<const uint16_t *>(ly.B);

    for (int id = tid; id < NE * kPfCopies; id += NT) {
        const int idx = id / kPfCopies;
        f16x2 h;
        h[0] = (_Float16)a.codebook[idx & (NL - 1)];
        h[1] = (_Float16)a.codebook[idx >> BITS];
        lut[id] = __builtin_bit_cast(uint32_t, h);
    }

    while (unit < unit_end) {
    // ---- this part: K tiles kt0 .. kt1 - 1 of output tile T
    const int T = unit / a.ntiles_k;
    const int kt0 = unit - T * a.ntiles_k, kt1 = min(a.ntiles_k, kt0 + (unit_end - unit));
    unit += kt1 - kt0;
    const int m_blk = (T / ly.nt) * BM, n_blk = (T % ly.nt) * BN;
    const int n_wave = n_blk + 16 * R * wave;

    bf16x8 Bop[R][SS];
#pragma unroll
    for (int rho = 0; rho < R; ++rho) {
        const int n = n_wave + 16 * rho + c;
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            u32x4 t = rank8_fetch(B16, A16, min(n, N - 1), 32 * s + 8 * g, N, a.r);
            t = rank8_fix(t, B16, min(n, N - 1), 32 * s + 8 * g, N, a.r, n_wave + 16 * rho + 16 > N - 8);
            if (n >= N) t = u32x4{0u, 0u, 0u, 0u};
            Bop[rho][s] = __builtin_bit_cast(bf16x8, t);
        }
    }

    // ---- tile loads.  Through buffer descriptors whose bounds end with the matrix: rows beyond it read as zeros.
    // X tile: as in lords_prefill_kernel.h.  Half h of an A tile holds the columns 32 gg + 16 h .. + 16 of each rank row (stages
    // 2 h and 2 h + 1), 128 bytes: the 16-byte chunk 2 gg + uu in slot (2 gg + uu) ^ ((row >> 1) & 1), so that the rows of
    // a transposing read spread over the banks.
    constexpr int XJ = 16, AQ = 2;                             // loads of an X tile, of half an A tile, per wave
    const int xt0 = 4 * wave + ((lane >> 3) & 3);
    const int xv = (lane & 7) ^ (xt0 & 7);
    const int xkcol = 32 * (xv & 3) + 8 * (xv >> 2) + 16 * (lane >> 5);
    const int arow = 8 * wave + (lane >> 3);                   // (+ 32 for the second load: the same slots)
    const int av = (lane & 7) ^ ((arow >> 1) & 1);
    const int acol = 32 * (av >> 1) + 8 * (av & 1);            // (+ 16 h)
    uint32_t xo[XJ], ao[AQ];
#pragma unroll
    for (int j = 0; j < XJ; ++j) xo[j] = ((uint32_t)(xt0 + 16 * j) * (uint32_t)K + (uint32_t)xkcol) * 2u;
#pragma unroll
    for (int q = 0; q < AQ; ++q) ao[q] = ((uint32_t)(arow + 32 * q) * (uint32_t)K + (uint32_t)acol) * 2u;
    const uint32_t xl0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(Xs + wave * 1024));
    const uint32_t al0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(As + wave * 1024));
    const uint64_t xbase = (uint64_t)(uintptr_t)a.X + (uint64_t)m_blk * (uint64_t)K * 2u, abase = (uint64_t)(uintptr_t)A16;
    const uint32_t xbytes = (uint32_t)min(M - m_blk, BM) * (uint32_t)K * 2u, abytes = (uint32_t)a.r * (uint32_t)K * 2u;
    // (from column kt * 128 on: what lies in front of it is taken off the size, so that rows beyond the matrix stay outside)
    auto rsrc_X = [&](int kt) __attribute__((always_inline)) { return make_rsrc(xbase + (uint64_t)kt * 256u, xbytes - (uint32_t)kt * 256u); };
    auto rsrc_A = [&](int kt) __attribute__((always_inline)) { return make_rsrc(abase + (uint64_t)kt * 256u, abytes - (uint32_t)kt * 256u); };
    // What a lane adds to its offsets in tile kt: nothing but in a ragged last tile, where X chunks beyond K are fetched from
    // further left in their row (any finite data will do: their weights are zero) and A chunks beyond K from outside of the
    // descriptor, i.e. as zeros.
    auto shift_X = [&](int kt) __attribute__((always_inline)) -> uint32_t { return (uint32_t)min(2 * (K - 8 - xkcol - kt * 128), 0); };
    auto shift_A = [&](int kt, int h) __attribute__((always_inline)) -> uint32_t { return kt * 128 + acol + 16 * h < K ? 32u * (uint32_t)h : 0x80000000u; };

    // Codes of K tile kt, slab rho, of the lane's row and group (layouts: lords_prefill_kernel.h); rows beyond the matrix read as code 0,
    // groups beyond K as any code (their scales are zero).
    const uint32_t crho = a.tiled ? (uint32_t)a.ntiles_k * 64u * 4 * BITS : 16u * (uint32_t)a.row_bytes;     // a slab's codes
    const uint32_t cstep = a.tiled ? 64u * 4 * BITS : 4u * 4 * BITS;
    const uint32_t clane = a.tiled ? (uint32_t)(16 * g + c) * 4 * BITS : (uint32_t)c * (uint32_t)a.row_bytes + (uint32_t)g * 4 * BITS;
    const int slab0 = (n_blk >> 4) + R * wave, nslabs = (N + 15) >> 4;
    const uint64_t cbase = (uint64_t)(uintptr_t)ly.codes + (uint64_t)min(slab0, nslabs - 1) * crho;
    const uint32_t cbytes = a.tiled ? (uint32_t)max(min(nslabs - slab0, R), 0) * crho : (uint32_t)max(min(N - 16 * slab0, 16 * R), 0) * (uint32_t)a.row_bytes;
    // (readfirstlane gives an int: the words are put together unsigned)
    const __amdgpu_buffer_rsrc_t rC = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(uintptr_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(cbase >> 32)) << 32) |
                            (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)cbase)), 0,
        __builtin_amdgcn_readfirstlane(cbytes), 0x00020000);
    auto load_codes = [&](int kt, int rho, uint32_t (&w)[BITS]) __attribute__((always_inline)) {
        const uint32_t so = (uint32_t)min(kt, a.ntiles_k - 1) * cstep + (uint32_t)rho * crho;
        if constexpr (BITS == 4) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rC, clane + so, 0, 0);
            w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
        } else if constexpr (BITS == 3) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b96(rC, clane + so, 0, 0);
            w[0] = v[0]; w[1] = v[1]; w[2] = v[2];
        } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rC, clane + so, 0, 0);
            w[0] = v[0]; w[1] = v[1];
        }
    };

    f32x4 acc[R][MB];
#pragma unroll
    for (int rho = 0; rho < R; ++rho)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[rho][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int ktl = a.ntiles_k - 1;
    uint32_t cw[R][BITS], cn[R][BITS], cf[R][BITS];            // codes of this K tile, the next one, the one after
    __syncthreads();                                           // (table written; every wave has left the part before)
    {
        // half tiles 0, 1, 2 of A, counted from this part's first
        const BufferRsrc rX = rsrc_X(kt0), rA = rsrc_A(kt0), rA1 = rsrc_A(min(kt0 + 1, ktl));
#pragma unroll
        for (int j = 0; j < XJ; ++j) lds_buffer_16(rX, xo[j], shift_X(kt0), xl0, j);
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            lds_buffer_16(rA, ao[q], shift_A(kt0, 0), al0, q);
            lds_buffer_16(rA, ao[q], shift_A(kt0, 1), al0 + AHALF, q);
            lds_buffer_16(rA1, ao[q], shift_A(min(kt0 + 1, ktl), 0), al0 + 2 * AHALF, q);
        }
    }
#pragma unroll
    for (int rho = 0; rho < R; ++rho) {
        load_codes(kt0, rho, cw[rho]);
        load_codes(kt0 + 1, rho, cn[rho]);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    uint32_t xr = (uint32_t)((c >> 2) * 1024 + (c & 3) * 128 + ((g ^ (c & 7)) * 16));     // X operand of stage 0, block 0, in this tile's buffer
    const uint32_t lutoff = (uint32_t)(2 * XBUF + 3 * AHALF) + (uint32_t)((lane & (kPfCopies - 1)) * 4);
    auto pair_at = [&](const uint32_t (&w)[BITS], int p) __attribute__((always_inline)) -> uint32_t { return pair_index<BITS>(w, p) * (kPfCopies * 4) + lutoff; };
    auto load_pair = [&](uint32_t at) __attribute__((always_inline)) -> uint32_t {
        return *reinterpret_cast<const __attribute__((address_space(3))) uint32_t *>((uintptr_t)at);
    };
    // a-operand of scale MFMA t of a K tile: 8 rank entries of 16 A columns, transposed out of the half tile at `ar`
    const uint32_t ar0 = (uint32_t)(2 * XBUF + (8 * g + (c >> 2)) * 128 + (((2 * (c & 3)) ^ (((c >> 2) >> 1) & 1)) * 16));
    auto read_Aop = [&](uint32_t ar, int s, int t) __attribute__((always_inline)) -> bf16x8 {
        typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
        const uint32_t p = (ar ^ (uint32_t)(((t >> 1) & 1) * 16)) + (uint32_t)(s * 4096 + (t & 1) * 8);
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(uintptr_t)p);
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(uintptr_t)(p + 512));
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_X = [&](uint32_t x0, int u, int mb) __attribute__((always_inline)) -> bf16x8 {
        return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>((uintptr_t)((x0 ^ (uint32_t)((u & 1) * 64)) + (u >> 1) * 512 + mb * 4096));
    };

    // Pipeline state: weights of the stage being multiplied and of the next (W), scales of the next stage (S), table
    // entries of its first pairs (lv), the address of one more (ad), X operands of the next steps (Xq).
    constexpr int kAhead = 4, kLvAhead = 4;
    bf16x8 W[2][R], Xq[8], Ao[2][SS];
    f32x4 S[R][2];
    uint32_t lv[8], ad;
    float w0, w1;
    auto scale = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) S[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ao[h][0], Bop[q][0], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int h = 0; h < 2; ++h) S[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ao[h][1], Bop[q][1], S[q][h], 0, 0, 0);
    };
    // level times scale, rounded once
    auto weigh = [&](uint32_t l, f32x4 s, int pp) __attribute__((always_inline)) {
        const f16x2 h = __builtin_bit_cast(f16x2, l);
        w0 = __builtin_fmaf((float)h[0], s[(2 * pp) & 3], 0.0f);
        w1 = __builtin_fmaf((float)h[1], s[(2 * pp + 1) & 3], 0.0f);
        asm volatile("" : "+v"(w0), "+v"(w1));                     // (here, not where they are rounded)
    };
    auto round_to = [&](bf16x8 &w, int pp) __attribute__((always_inline)) {
        w[2 * pp] = (__bf16)w0;
        w[2 * pp + 1] = (__bf16)w1;
    };
    // stage 0 in the open, the scales of stage 1 and its first table entries
#pragma unroll
    for (int s = 0; s < SS; ++s) { Ao[0][s] = read_Aop(ar0, s, 0); Ao[1][s] = read_Aop(ar0, s, 1); }
#pragma unroll
    for (int q = 0; q < R; ++q) scale(q);
#pragma unroll
    for (int j = 0; j < NP; ++j) { weigh(load_pair(pair_at(cw[j >> 2], j & 3)), S[j >> 2][(j & 3) >> 1], j & 3); round_to(W[0][j >> 2], j & 3); }
#pragma unroll
    for (int s = 0; s < SS; ++s) { Ao[0][s] = read_Aop(ar0, s, 2); Ao[1][s] = read_Aop(ar0, s, 3); }
#pragma unroll
    for (int q = 0; q < R; ++q) scale(q);
#pragma unroll
    for (int j = 0; j < kLvAhead; ++j) lv[j] = load_pair(pair_at(cw[j >> 2], 4 + (j & 3)));
    ad = pair_at(cw[kLvAhead >> 2], 4 + (kLvAhead & 3));
#pragma unroll
    for (int i = 0; i < kAhead; ++i) Xq[i] = read_X(xr, 0, i);
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __syncthreads();                                           // (half tile 0 of A has been read: its place is free)

    uint32_t a1 = AHALF, a2 = 2 * AHALF, a3 = 0, xb = 0;       // half tiles of A: second of this K tile, first of the next, a free place; X buffer
    for (int kt = kt0; kt < kt1; ++kt) {
        const uint32_t xn = xb ^ XBUF;
        // (beyond the last tile: it once more, for nobody to read)
        const int kx = min(kt + 1, ktl), ka = min(kt + 2, ktl);
        const BufferRsrc rX = rsrc_X(kx), rA = rsrc_A(kx), rA2 = rsrc_A(ka);
        const uint32_t sx = shift_X(kx), sa = shift_A(kx, 1), sa2 = shift_A(ka, 0);
        uint32_t ar = ar0, arn = ar0;
        asm volatile("" : "+v"(xr), "+v"(ar), "+v"(arn));          // (operand addresses are made where they are used: registers)
        ar += a1;
        arn += a2;
        const uint32_t xl = xl0 + xn, al = al0 + a3, al2 = al0 + a1;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int cur = u & 1, nxt = cur ^ 1;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int t = MB * u + mb, tn = t + kAhead;
                const bf16x8 Xop = Xq[t & 7];
                mfma_acc(acc[0][mb], W[cur][0], Xop);
                if (t == 4 * MB - kAhead) {
                    // what was fetched has landed in LDS, for every wave; every wave has read the last of this tile's X
                    __builtin_amdgcn_s_waitcnt(0x0070);
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                lv[(mb + kLvAhead) & 7] = load_pair(ad);
                Xq[tn & 7] = tn < 4 * MB ? read_X(xr, tn / MB, tn % MB) : read_X(xr ^ XBUF, 0, tn - 4 * MB);
                __builtin_amdgcn_sched_barrier(0);
                mfma_acc(acc[1][mb], W[cur][1], Xop);
                weigh(lv[mb & 7], S[mb >> 2][(mb & 3) >> 1], mb & 3);              // pair mb of the next stage
                __builtin_amdgcn_sched_barrier(0);
                mfma_acc(acc[2][mb], W[cur][2], Xop);
                {
                    // table address of the pair kLvAhead + 1 steps on
                    const int j = mb + kLvAhead + 1, un = u + 1 + (j >> 4), q = (j & 15) >> 2, pp = j & 3;
                    ad = un < 4 ? pair_at(cw[q], 4 * un + pp) : pair_at(cn[q], 4 * (un - 4) + pp);
                    asm volatile("" : "+v"(ad));
                }
                __builtin_amdgcn_sched_barrier(0);
                mfma_acc(acc[3][mb], W[cur][3], Xop);
                round_to(W[nxt][mb >> 2], mb & 3);
                if ((t & 1) == 1 && t < 1 + 2 * XJ) lds_buffer_16(rX, xo[(t - 1) / 2], sx, xl, (t - 1) / 2);
                if (t == 2 || t == 4) lds_buffer_16(rA, ao[(t - 2) / 2], sa, al, (t - 2) / 2);
                if (t == 28) {
                    // every wave has read the second half of this tile's A (steps 4 .. 21): the first half of the one after
                    // the next takes its place
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                if (t == 30 || t == 32) lds_buffer_16(rA2, ao[(t - 30) / 2], sa2, al2, (t - 30) / 2);
                if (t >= 6 && t < 6 + 4 * R && (t & 3) == 2) load_codes(kt + 2, (t - 6) / 4, cf[(t - 6) / 4]);
                __builtin_amdgcn_sched_barrier(0);
                if (mb == 4 || mb == 5) {
                    const int v = u + 2, h = mb - 4;
#pragma unroll
                    for (int s = 0; s < SS; ++s) Ao[h][s] = read_Aop(v < 4 ? ar : arn, s, 2 * (v & 3) + h);
                }
                // (odd blocks: the last pair of the next stage has been converted when its scales are replaced)
                if (mb >= 8 && (mb & 1) == 1) scale((mb - 8) >> 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int rho = 0; rho < R; ++rho)
#pragma unroll
            for (int q = 0; q < BITS; ++q) { cw[rho][q] = cn[rho][q]; cn[rho][q] = cf[rho][q]; }
        const uint32_t old = a1;
        a1 = a3; a3 = a2; a2 = old;
        xb = xn;
        xr ^= XBUF;
    }
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");            // (results of the last matrix instructions)

    // ---- epilogue: lane (c, g) holds token 16 mb + c, rows 16 rho + 4 g + {0..3}; hand-over as in lords_prefill_kernel.h
    constexpr int kPartFloats = R * MB * NT * 4;
    if (kt0 != 0) {
        float *dst = ly.part + (size_t)wg * kPartFloats + tid * 4;
        asm volatile("" : "+v"(dst));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int rho = 0; rho < R; ++rho) store16_agent(dst + (mb * R + rho) * (NT * 4), read_acc(acc[rho][mb]));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(ly.arrived + T, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        continue;
    }
    int others = 0;
    if (kt1 != a.ntiles_k) {
        others = (a.ntiles_k - kt1 + ly.per - 1) / ly.per;                 // the workgroups after this one, up to the tile's end
        if (tid == 0) {
            // (bounded as in lords_prefill_kernel.h: the parts waited for are first parts of their workgroups and never wait themselves)
            int spins = 0;
            while ((int)__hip_atomic_load(ly.arrived + T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < others && ++spins < (1 << 21))
                __builtin_amdgcn_s_sleep(8);
            __hip_atomic_store(ly.arrived + T, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
    }
    const bool full = m_blk + BM <= M && n_blk + BN <= N;
    void *Yp = ly.Y;
    // Sixteen accumulator blocks at a time (four token blocks, all the wave's rows): the other parts are added, the
    // gate applied and the result stored from registers of their own, so that the accumulators are only read here.
    constexpr int GB = 4;
#pragma unroll
    for (int b0 = 0; b0 < MB; b0 += GB) {
        f32x4 v[GB * R];
#pragma unroll
        for (int i = 0; i < GB * R; ++i) v[i] = read_acc(acc[i % R][b0 + i / R]);
        // (two parts at a time: each wait is a round trip to memory; of an odd number the last is read twice and added once)
        for (int j = 1; j <= others; j += 2) {
            const float *src = ly.part + (size_t)(wg + j) * kPartFloats + tid * 4;
            const float *src2 = j < others ? src + kPartFloats : src;
            asm volatile("" : "+v"(src), "+v"(src2));
            f32x4 t[2 * GB * R];
#pragma unroll
            for (int i = 0; i < GB * R; ++i) t[i] = load16_agent(src + (b0 * R + i) * (NT * 4));
#pragma unroll
            for (int i = 0; i < GB * R; ++i) t[GB * R + i] = load16_agent(src2 + (b0 * R + i) * (NT * 4));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int i = 0; i < 2 * GB * R; ++i) asm volatile("" : "+v"(t[i]));           // (not before the wait)
#pragma unroll
            for (int i = 0; i < GB * R; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[i][e] += t[i][e];
                    v[i][e] = j < others ? v[i][e] + t[GB * R + i][e] : v[i][e];
                }
        }
        int m0 = m_blk + 16 * b0 + c, n0 = n_wave + 4 * g;
        asm volatile("" : "+v"(m0), "+v"(n0));                              // (addresses of one batch at a time: registers)
        if (ly.gate) {
            // This is the up product of a gate/up pair, the gate's fp32 sums lie in memory.  Addresses are clamped to the
            // matrix's rows; a load of its last columns may reach 12 bytes beyond them (the buffer is that much longer).
            f32x4_any t[GB * R];
#pragma unroll
            for (int i = 0; i < GB * R; ++i)
                t[i] = *reinterpret_cast<const f32x4_any *>(ly.gate + (size_t)min(m0 + 16 * (i / R), M - 1) * N + min(n0 + 16 * (i % R), N - 1));
#pragma unroll
            for (int i = 0; i < GB * R; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = t[i][e] / (1.0f + __expf(-t[i][e])) * v[i][e];
        }
        if (full) {
#pragma unroll
            for (int i = 0; i < GB * R; ++i) store_out4(Yp, (size_t)(m0 + 16 * (i / R)) * N + n0 + 16 * (i % R), v[i], a.y_f32);
        } else {
#pragma unroll
            for (int i = 0; i < GB * R; ++i) {
                const int m = m0 + 16 * (i / R), n = n0 + 16 * (i % R);
                if (m >= M) continue;
                if (n + 3 < N) {
                    store_out4(Yp, (size_t)m * N + n, v[i], a.y_f32);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (n + e >= N) continue;
                        if (a.y_f32) reinterpret_cast<float *>(Yp)[(size_t)m * N + n + e] = v[i][e];
                        else reinterpret_cast<uint16_t *>(Yp)[(size_t)m * N + n + e] = bf16_bits(v[i][e]);
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    }   // parts of this workgroup
}

template <int BITS, bool MULTI>
static hipError_t launch_wide_t(const PrefillArgsT<MULTI ? kMaxBatch : 1> &a, dim3 grid, hipStream_t st)
{
    const size_t smem = (size_t)2 * 65536 + (size_t)3 * 8192 + (size_t)(1 << (2 * BITS)) * kPfCopies * 4;
    static LdsOptIn lds_opt_in;
    {
        const hipError_t e = allow_dynamic_lds(lds_opt_in, reinterpret_cast<const void *>(&prefill_wide_kernel<BITS, MULTI>), smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((prefill_wide_kernel<BITS, MULTI>), grid, dim3(256), smem, st, a);
    return hipGetLastError();
}

hipError_t launch_prefill_wide(const PrefillArgsT<1> &a, dim3 grid, int bits, hipStream_t st)
{
    return bits == 2 ? launch_wide_t<2, false>(a, grid, st) : bits == 3 ? launch_wide_t<3, false>(a, grid, st) : launch_wide_t<4, false>(a, grid, st);
}
hipError_t launch_prefill_wide(const PrefillArgsT<kMaxBatch> &a, dim3 grid, int bits, hipStream_t st)
{
    return bits == 2 ? launch_wide_t<2, true>(a, grid, st) : bits == 3 ? launch_wide_t<3, true>(a, grid, st) : launch_wide_t<4, true>(a, grid, st);
}

}  // namespace lords
