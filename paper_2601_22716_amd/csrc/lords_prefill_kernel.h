// Large-M (prefill) kernel of  Y = X (C[Q] (.) (B A))^T  on gfx950: a bf16 MFMA GEMM whose weight
// operand is dequantised on the fly and never leaves the registers.
//
// Tiling.  A workgroup owns a (16*R*WN)-row x (16*MB*WM)-token tile of Y and walks K in tiles of
// 128 columns.  It has WN*WM waves: wave (wn, wm) owns rows 16R wn .. (R slabs of 16 rows) and
// tokens 16MB wm .., so each dequantised weight is reused for 16*MB tokens from registers; the
// accumulators (R slabs x MB token blocks x 4 registers, 128 in the large tiles) stay in
// registers over the whole K range.  The main shape is 256 x 256 with eight waves side by side
// along the rows (WN = 8, WM = 1, R = 2, MB = 16): every weight of the tile is dequantised by
// exactly one wave and meets all 256 tokens there.  (Waves of 64 rows x 128 tokens, two of
// which dequantise the same rows, were 9 % slower on the same tile although they read X from
// LDS half as often: the vector work and the scale MFMAs weigh more than the LDS reads.)  Two
// waves per SIMD, at most 256 registers each, so that every MFMA writes plain VGPRs (results of
// the scale MFMAs are read by vector ALU instructions, which cannot read the accumulation
// registers).  Smaller shapes for small problems and ranks above 32: see the launcher.
//
// Work division.  The launcher either gives every workgroup one whole output tile, or deals the
// K tiles of all output tiles, numbered tile by tile, to the workgroups in equal contiguous runs,
// so that every CU gets the same amount of work whatever the tile count.  A tile that a run
// boundary cuts is summed from its parts in column order: the parts that do not start at the
// tile's first column are written out as fp32 and counted in; the part that does adds them up
// in order and writes Y (see the epilogue).  The result does not depend on timing.
//
// Per K tile the X tile (BM x 128 bf16) and the A tile (padded rank x 128 bf16) are brought from
// global memory straight into LDS (global_load_lds_dwordx4, no registers), double-buffered, one
// barrier per tile.  16-byte chunks are XOR-swizzled by row so that the b-operand reads of X
// (ds_read_b128) and the transposing reads of A (ds_read_b64_tr_b16) are free of bank conflicts;
// the layouts are described where the tiles are staged.
//
// Lane mapping as in the decode kernels (v_mfma_f32_16x16x32_bf16, lane l = (c = l%16, g = l/16)):
// the lane holds the 32 codes of row n0+c at columns kb + 32g ..; scale MFMA t gives it the scales
// of codes 4t..4t+3; product MFMA u contracts columns 32g + 8u .. +8 with
// a-operand = the lane's 8 dequantised weights and b-operand = X[token c][same 8 columns].
// A K tile is processed in four stages u = 0..3 (scale MFMAs 2u, 2u+1 -> dequantise 8 weights per
// slab -> BM/16 x 4 product MFMAs); for ranks up to 32 the stages overlap as a software pipeline
// (stage u+1's dequantisation is spread over stage u's product MFMAs, see the K loop).
//
// Level look-up: two codes index an LDS table of fp16 pairs, 8 copies (address =
// index*32 + (lane%8)*4); v_fma_mix_f32 multiplies fp16 level by fp32 scale; one rounding to bf16.
// With fp32 factors the levels stay fp32 too (pairs of 8 bytes, 8 copies): level times scale is then
// rounded once, to bf16, and no level has to lie within the range of fp16.
#pragma once
#include <algorithm>
#include <type_traits>
#include "lords_prefill.h"
#include "lords_meet.h"

namespace lords {

constexpr int pf_pair_bytes(bool f32fact) { return f32fact ? 8 : 4; }
typedef float PfLevels __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void lds_direct_16(const void *gbase, uint32_t goff, uint32_t lds_wave_base)
{
    // Every active lane fetches 16 bytes from gbase + goff (gbase and lds_wave_base are the same
    // in all lanes and travel in scalar registers, goff is the lane's own byte offset); they land
    // at lds_wave_base + 16*lane (M0 holds the wave's LDS base).  With the row offsets of a tile
    // computed once, a tile load costs no vector instruction besides the load itself.
    // Written as assembly on purpose: when the compiler knows of an outstanding load into LDS it
    // makes the next LDS read wait for ALL outstanding memory loads, i.e. for the tile that was
    // just requested, which exposes the whole memory latency once per K tile.  The kernel orders
    // these loads itself: s_waitcnt vmcnt(0) and a barrier before a buffer is read.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_wave_base), "v"(goff), "s"(gbase) : "memory", "m0");
}

// F32: fp32 factors.  They are split x = hi + lo (two bf16) and the scale is the contraction of length
// 3 rf of [Bhi | Bhi | Blo] with [Ahi ; Alo ; Ahi] (lords_device.h).  The A tile then comes through
// registers: a thread requests 8 columns of a row with the codes of the next K tile, and splits them into
// the three LDS rows (rank rows j, rf + j, 2 rf + j) after this tile's products: about 20 vector
// instructions per thread and K tile at rank 16, no scratch and no launch of its own.
// 4096 x 4096, 4 bits, rank 16, 300 tokens: 47 us (general kernel of lords_fused.hip: 280); 1000 tokens 68 (352);
// 14336 x 4096, rank 40, 17 tokens 69 (602).
// MULTI: several matrices in the launch (a lone one is read from fixed offsets of a short argument block: through an
// index it cost 0.3 us a call).
// FORM: parts that meet (kMeet) or any other cut of the work (kRuns), a kernel each: in one, the code of the
// former cost the latter up to 2.5 % (333 tokens of 11008 x 4096, 3 bits, rank 48 61.5 -> 62.3 us).  Several matrices: kEither where
// those of some meet, kWalk where a workgroup takes several parts of a tile (PfLayer::walk; in one kernel the two cost launches without
// walk up to 1 us of 22).
enum PfForm { kRuns, kMeet, kEither, kWalk };
template <int BITS, int SS, int WM, int R, int WN = 4, int MB = 8, bool F32 = false, bool MULTI = false, PfForm FORM = kRuns>
__global__ __launch_bounds__(64 * WN * WM) __attribute__((amdgpu_waves_per_eu(WN * WM / 4, WN * WM / 4))) void prefill_kernel(PrefillArgsT<MULTI ? kMaxBatch : 1> a)
{
    constexpr int BN = 16 * R * WN, BM = 16 * MB * WM, NT = 64 * WN * WM, RP = 32 * SS, NL = 1 << BITS, NE = 1 << (2 * BITS);
    constexpr int RPP = 4 * WN * WM;                           // A tile rows one staging pass of the workgroup covers
    constexpr int XBUF = BM * 256, ABUF = RP * 256;            // bytes per buffer
    constexpr bool kPipe = (R == 2 && SS <= 2 && (MB == 8 || MB == 16));   // ranks up to 64: pipelined K loop
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *Xs = smem;                                   // [2][BM / 4 token groups][1 KB]
    unsigned char *As = smem + 2 * XBUF;                        // [2][RP][256 B]
    uint32_t *lut = reinterpret_cast<uint32_t *>(smem + 2 * XBUF + 2 * ABUF);   // [NE][8], a pair each

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    // the matrix this workgroup works on (the same in all lanes)
    int li = 0;
    if (MULTI)
        while (li + 1 < a.L && (int)blockIdx.x >= a.layer[li + 1].x0) ++li;
    const PfLayer ly = a.layer[MULTI ? li : 0];
    const int M = a.M, N = ly.N, K = a.K;

    // ---- work of this workgroup.  The work is cut into units, one K tile of one output tile each, numbered
    //      tile by tile (n fastest); workgroup w takes units w per .. w per + per - 1, so a workgroup walks a
    //      tail of one output tile, whole tiles, and a head of another.  Workgroups are dealt round-robin to
    //      the 8 XCDs, so each XCD gets a contiguous run of ranges: its workgroups then share X panels in its L2.
    const int total_units = ly.nt * a.mt * a.ntiles_k;
    const int bx = (int)blockIdx.x - ly.x0;
    // Parts that meet (see the epilogue): 2^meet workgroups share the `per` units of a tile, a unit more or less each.  With
    // walk, 2^(meet + walk) parts of a tile are shared in the same way by 2^meet workgroups, 2^walk parts each, one after the other.
    // A tile's workgroups are on one XCD, and tiles are dealt to the XCDs as evenly as they go, one more on the first ones from ly.xcd
    // on.  (Rounded up on all but the last, those of several matrices piled up on the first XCDs, and as workgroups are dispatched in
    // order the others then wait too.  Q/k/v of 4096 + 1024 + 1024 rows x 4096, 256 tokens: 42.4 us so, 33.4 now.)
    const int meet_log = FORM == kRuns ? 0 : ly.meet, walk = FORM == kWalk ? ly.walk : 0, cut_log = meet_log + walk;
    int wg = (bx & 7) * (ly.gx >> 3) + (bx >> 3), meet_part = 0;
    if (FORM == kMeet || (FORM >= kEither && cut_log)) {
        int tile;
        if (!meet_place(bx, ly.xcd, ly.nt * a.mt, meet_log, tile, meet_part)) return;
        wg = (tile << meet_log) + meet_part;
    }
    const int unit0 = (wg >> meet_log) * ly.per, unit_end = min(unit0 + (((meet_part + 1) << walk) * ly.per >> cut_log), total_units);
    int unit = unit0 + ((meet_part << walk) * ly.per >> cut_log);
    int walked = 0;
    if (unit >= unit_end) return;
    const int wn = wave % WN, wm = wave / WN;
    const uint16_t *A16 = reinterpret_cast<const uint16_t *>(ly.A), *B16 = reinterpret_cast<const uint16_t *>(ly.B);   // (bf16 factors)

    // ---- level table --------------------------------------------------------------------------------
    for (int id = tid; id < NE * kPfCopies; id += NT) {
        const int idx = id / kPfCopies;
        const float l0 = a.codebook[idx & (NL - 1)], l1 = a.codebook[idx >> BITS];
        if constexpr (F32) {
            reinterpret_cast<PfLevels *>(lut)[id] = PfLevels{l0, l1};
        } else {
            f16x2 h;
            h[0] = (_Float16)l0;
            h[1] = (_Float16)l1;
            lut[id] = __builtin_bit_cast(uint32_t, h);
        }
    }
    // ---- zero the A buffers once: rank rows >= r are never loaded and must read as zero --------------
    for (int id = tid; id < 2 * ABUF / 16; id += NT) reinterpret_cast<u32x4 *>(As)[id] = u32x4{0u, 0u, 0u, 0u};
    if (K & 127)                                               // ragged last K tile: stale X must at least be finite
        for (int id = tid; id < 2 * XBUF / 16; id += NT) reinterpret_cast<u32x4 *>(Xs)[id] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    while (unit < unit_end) {
    // ---- this part: K tiles kt0 .. kt1 - 1 of output tile T ------------------------------------------------
    const int T = unit / a.ntiles_k;
    const int kt0 = unit - T * a.ntiles_k;
    int kt1 = min(a.ntiles_k, kt0 + (unit_end - unit));
    if (FORM == kWalk && walk) kt1 = ((meet_part << walk) + ++walked) * ly.per >> cut_log;
    unit += kt1 - kt0;
    const int m_blk = (T / ly.nt) * BM, n_blk = (T % ly.nt) * BN;
    const int n_wave = n_blk + 16 * R * wn;
    const int m_wave = m_blk + 16 * MB * wm;

    // ---- B operands of the scale MFMAs: rows n_wave + 16 rho + c, rank entries 32 s + 8 g .. ----------
    bf16x8 Bop[R][SS];
#pragma unroll
    for (int rho = 0; rho < R; ++rho) {
        const int n = n_wave + 16 * rho + c;
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            const int jj0 = 32 * s + 8 * g;
            typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
            s16x8 t;
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = 0;
            if (n < N) {
                if constexpr (F32) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int jj = jj0 + e;
                        if (jj < a.r) {
                            const int j = jj < a.rf ? jj : jj < 2 * a.rf ? jj - a.rf : jj - 2 * a.rf;
                            const float x = reinterpret_cast<const float *>(ly.B)[(size_t)n * a.rf + j];
                            const uint16_t hi = bf16_bits(x);
                            t[e] = (short)(jj >= 2 * a.rf ? bf16_bits(x - bf16_to_f32(hi)) : hi);
                        }
                    }
                } else if ((a.r & 7) == 0) {
                    if (jj0 + 8 <= a.r) t = *reinterpret_cast<const s16x8 *>(B16 + (size_t)n * a.r + jj0);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (jj0 + e < a.r) t[e] = (short)B16[(size_t)n * a.r + jj0 + e];
                }
            }
            Bop[rho][s] = __builtin_bit_cast(bf16x8, t);
            if constexpr (F32) __builtin_amdgcn_sched_barrier(0);     // (eight gathered entries in flight, not all of them: registers)
        }
    }

    // ---- staging of one K tile into buffer p (direct to LDS) and of its codes into registers ---------
    // X tile in LDS: groups of four tokens, 1 KB each = [2 halves of 64 columns][4 tokens][128 B]; a
    // wave load fills one group, lane l landing in half l / 32, token (l / 8) % 4, slot l % 8, and
    // fetches whole 256-byte token rows from global memory (8 full cache lines per wave load).
    // Slot s of token t of half h holds the 8 columns 32 gg + 8 uu + 16 h with 4 uu + gg = s ^ (t & 7):
    // the four 16-byte chunks that the four lane groups g of an MFMA b-operand want at stage
    // u = 2 h + uu then sit in one 64-byte quarter-row, XOR-swizzled by token, and a wave's operand
    // read (16 tokens x 4 chunks) is free of bank conflicts (5.0 cycles per wave instruction; rows
    // of 256 bytes, one per token, cost 8.2 however they were swizzled).
    // A tile: row-major, 256 B per rank row, lane (wave, l) fetches chunk (l & 15) ^ (row & 15) of
    // row 4 wave + l / 16 (+ RPP per pass).  The byte offsets of a lane's chunks from the tile's
    // first element do not change along K and are kept in registers.
    constexpr int AQ = F32 ? 0 : (RP + RPP - 1) / RPP;         // (fp32 factors: the A tile takes the other way, below)
    constexpr int TPP = 4 * WN * WM, XJ = BM / TPP;             // tokens per staging pass, passes
    static_assert(BM % TPP == 0, "a staging pass covers whole token groups");
    const int xm0 = 4 * wave + (lane >> 4);
    const int xkc = (lane & 15) ^ (xm0 & 15);
    const int xt0 = 4 * wave + ((lane >> 3) & 3);             // the lane's token in pass 0 (then + TPP per pass)
    const int xv = (lane & 7) ^ (xt0 & 7);                    // (TPP is a multiple of 8: the same in every pass)
    const int xkcol = 32 * (xv & 3) + 8 * (xv >> 2) + 16 * (lane >> 5);
    uint32_t xo[XJ], ao[AQ + 1];
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
        const int m = min(m_blk + xt0 + TPP * j, M - 1);       // rows >= M: a copy of the last row, never stored
        xo[j] = ((uint32_t)(m - m_blk) * (uint32_t)K + (uint32_t)xkcol) * 2u;
    }
#pragma unroll
    for (int q = 0; q < AQ; ++q) ao[q] = ((uint32_t)min(xm0 + RPP * q, max(a.r - 1, 0)) * (uint32_t)K + 8u * xkc) * 2u;
    const uint32_t xl0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(Xs + wave * 1024));
    const uint32_t al0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(As + wave * 1024));
    const uint16_t *Xtile = a.X + (size_t)m_blk * K;
    auto stage = [&](int kt, int p) {
        const int kb = kt * 128;
        if (kb + 128 <= K) {
#pragma unroll
            for (int j = 0; j < XJ; ++j) lds_direct_16(Xtile + kb, xo[j], xl0 + p * XBUF + j * (TPP * 256));
#pragma unroll
            for (int q = 0; q < AQ; ++q)
                if (xm0 + RPP * q < a.r) lds_direct_16(A16 + kb, ao[q], al0 + p * ABUF + q * (RPP * 256));
        } else {
            // ragged last tile: X chunks beyond K are fetched from further left (any finite data will
            // do: their weights are zero), A columns beyond K of a live rank row must read as zero
            {
                const int over = kb + xkcol - (K - 8);
                const uint32_t back = over > 0 ? 2u * over : 0u;
#pragma unroll
                for (int j = 0; j < XJ; ++j) lds_direct_16(Xtile + kb, xo[j] - back, xl0 + p * XBUF + j * (TPP * 256));
            }
#pragma unroll
            for (int q = 0; q < AQ; ++q) {
                if (xm0 + RPP * q >= a.r) continue;
                if (kb + 8 * xkc < K) lds_direct_16(A16 + kb, ao[q], al0 + p * ABUF + q * (RPP * 256));
                else *reinterpret_cast<u32x4 *>(As + p * ABUF + wave * 1024 + q * (RPP * 256) + 16 * lane) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    };
    // Codes of K tile kt, row n, lane group g: canonical rows: n * row_bytes + (4 kt + g) * 4 BITS (clamped
    // into the row for a ragged last tile); slab-tile layout: the tile (n / 16, kt) is contiguous and the
    // lane's chunk is 16 g + n % 16.  Either way: a per-row base, a step per K tile, an offset per lane.
    const int ngroups = K >> 5;
    const uint8_t *crow[R];
#pragma unroll
    for (int rho = 0; rho < R; ++rho) {
        const int n = min(n_wave + 16 * rho + c, N - 1);
        crow[rho] = a.tiled ? ly.codes + ((size_t)(n >> 4) * a.ntiles_k * 64 + (n & 15)) * (4 * BITS)
                            : ly.codes + (size_t)n * a.row_bytes;
    }
    const uint32_t cstep = a.tiled ? 64u * 4 * BITS : 4u * 4 * BITS;
    const uint32_t cgoff = a.tiled ? (uint32_t)g * 16 * 4 * BITS : (uint32_t)g * 4 * BITS;
    const uint32_t cmax = a.tiled ? 0xffffffffu : (uint32_t)(ngroups - 1) * 4 * BITS;
    auto load_codes = [&](int kt, uint32_t (&cw)[R][BITS]) {
        const uint32_t off = min((uint32_t)kt * cstep + cgoff, cmax);
#pragma unroll
        for (int rho = 0; rho < R; ++rho) load_group<BITS>(crow[rho] + off, cw[rho]);
    };

    // fp32 A tile of K tile kt: item id = 16 j + kc is columns 8 kc .. +8 of factor row j (columns beyond K: zero)
    constexpr int AF = F32 ? ((RP / 3) * 16 + NT - 1) / NT : 0;
    f32x4 af[AF + 1][2];
    auto load_A32 = [&](int kt) {
#pragma unroll
        for (int q = 0; q < AF; ++q) {
            const int id = tid + NT * q, j = id >> 4, k = kt * 128 + 8 * (id & 15);
            af[q][0] = af[q][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (j < a.rf && k < K) {
                const f32x4 *src = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(ly.A) + (size_t)j * K + k);
                af[q][0] = src[0];
                af[q][1] = src[1];
            }
        }
    };
    auto store_A32 = [&](int p) {
#pragma unroll
        for (int q = 0; q < AF; ++q) {
            const int id = tid + NT * q, j = id >> 4, kc = id & 15;
            if (j >= a.rf) continue;
            u32x4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = af[q][e >> 1][2 * (e & 1)], x1 = af[q][e >> 1][2 * (e & 1) + 1];
                const uint16_t h0 = bf16_bits(x0), h1 = bf16_bits(x1);
                hi[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                lo[e] = (uint32_t)bf16_bits(x0 - bf16_to_f32(h0)) | ((uint32_t)bf16_bits(x1 - bf16_to_f32(h1)) << 16);
            }
#pragma unroll
            for (int seg = 0; seg < 3; ++seg) {
                const int row = seg * a.rf + j;
                *reinterpret_cast<u32x4 *>(As + p * ABUF + row * 256 + ((kc ^ (row & 15)) * 16)) = seg == 1 ? lo : hi;
            }
        }
    };

    f32x4 acc[R][MB];
#pragma unroll
    for (int rho = 0; rho < R; ++rho)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[rho][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    uint32_t cw[R][BITS], cwn[R][BITS];
    stage(kt0, 0);
    load_codes(kt0, cw);
    if constexpr (F32) { load_A32(kt0); store_A32(0); }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // per-lane LDS offsets
    uint32_t xoff[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        xoff[u] = (uint32_t)((u >> 1) * 512 + (c >> 2) * 1024 + (c & 3) * 128 + (((4 * (u & 1) + g) ^ (c & 7)) * 16));

    const uint32_t lutoff = (uint32_t)(2 * XBUF + 2 * ABUF) + (uint32_t)((lane & (kPfCopies - 1)) * pf_pair_bytes(F32));
    // a pair of levels: its LDS address, its load, its two weights (level times scale, rounded once)
    using Pair = std::conditional_t<F32, PfLevels, uint32_t>;
    auto pair_at = [&](uint32_t idx) __attribute__((always_inline)) -> uint32_t { return idx * (kPfCopies * pf_pair_bytes(F32)) + lutoff; };
    auto load_pair = [&](uint32_t at) __attribute__((always_inline)) -> Pair {
        return *reinterpret_cast<const __attribute__((address_space(3))) Pair *>((uintptr_t)at);
    };
    auto weights = [&](Pair lv, float s0, float s1, __bf16 &w0, __bf16 &w1) __attribute__((always_inline)) {
        if constexpr (F32) {
            w0 = (__bf16)(lv.x * s0);
            w1 = (__bf16)(lv.y * s1);
        } else {
            const f16x2 h = __builtin_bit_cast(f16x2, lv);
            w0 = (__bf16)__builtin_fmaf((float)h[0], s0, 0.0f);
            w1 = (__bf16)__builtin_fmaf((float)h[1], s1, 0.0f);
        }
    };

    for (int kt = kt0; kt < kt1; ++kt) {
        const int p = (kt - kt0) & 1;
        if (kt + 1 < kt1) {
            // (the main shape issues the loads of a whole next tile one by one from its pipeline steps)
            if (!kPipe || (kt + 2) * 128 > K) stage(kt + 1, p ^ 1);
            load_codes(kt + 1, cwn);
            if constexpr (F32) load_A32(kt + 1);
        }
        const unsigned char *Xp = Xs + p * XBUF + wm * (16 * MB * 256);
        const unsigned char *Ap = As + p * ABUF;

        // a-operand of scale MFMA t: 8 rank entries of 16 A columns, transposed out of LDS
        auto read_Aop = [&](int s, int t) -> bf16x8 {
            typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
            const int row0 = 32 * s + 8 * g + (c >> 2);                 // +4 for the second half
            const int kc = 4 * (c & 3) + (t >> 1);
            const unsigned char *p0 = Ap + row0 * 256 + ((kc ^ (row0 & 15)) * 16) + (t & 1) * 8;
            const unsigned char *p1 = Ap + (row0 + 4) * 256 + ((kc ^ ((row0 + 4) & 15)) * 16) + (t & 1) * 8;
            s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)p0);
            s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)p1);
            return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };

        // Stage u of the dequantisation, two slabs at a time.  The LDS reads of a pair of slabs
        // (table entries, transposed A columns) are all issued before the first use, so that the
        // wave pays two LDS round trips per pair rather than one per table entry.
        auto dequant_stage = [&](int u, bf16x8 (&W)[R]) {
            bf16x8 Aop0[SS], Aop1[SS];
#pragma unroll
            for (int s = 0; s < SS; ++s) { Aop0[s] = read_Aop(s, 2 * u); Aop1[s] = read_Aop(s, 2 * u + 1); }
#pragma unroll
            for (int hp = 0; hp < R / 2; ++hp) {
                Pair lv[2][4];
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int pp = 0; pp < 4; ++pp) lv[q][pp] = load_pair(pair_at(pair_index<BITS>(cw[2 * hp + q], 4 * u + pp)));
                f32x4 S0[2], S1[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    S0[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                    S1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < SS; ++s) {
                        S0[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Aop0[s], Bop[2 * hp + q][s], S0[q], 0, 0, 0);
                        S1[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Aop1[s], Bop[2 * hp + q][s], S1[q], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int pp = 0; pp < 4; ++pp) {
                        const float s0 = pp < 2 ? S0[q][2 * pp] : S1[q][2 * pp - 4];
                        const float s1 = pp < 2 ? S0[q][2 * pp + 1] : S1[q][2 * pp - 3];
                        __bf16 w0, w1;
                        weights(lv[q][pp], s0, s1, w0, w1);
                        W[2 * hp + q][2 * pp] = w0;
                        W[2 * hp + q][2 * pp + 1] = w1;
                    }
            }
        };

        if constexpr (kPipe) {
            // Ranks up to 64: the K tile as one software pipeline of 4 MB steps (4 stages x MB token
            // blocks), pinned step by step with scheduling barriers.  A step is the two product MFMAs
            // of one token block; riding on it are the X operand read of the block kAhead steps later
            // and a slice of the NEXT stage's dequantisation (with 16 token blocks: A columns and
            // table addresses in steps 0-3 of a stage, table reads in steps 1-4, scale MFMAs in step
            // 3, one pair of weights converted in each of steps 5-12; with 8 blocks the same slices at
            // twice the density), so that vector and LDS instructions issue in the shadow of MFMAs of
            // the same wave and every result is asked for several MFMAs before it is needed.  Only
            // stage 0 of a tile is dequantised in the open (its A tile arrives with the barrier).
            // The tile loads for the next K tile also ride on the steps, one each: issued in one
            // burst at the head of the tile they cost 3-4 % more.
            constexpr int H = MB / 8;                           // 1 or 2
            constexpr int NPS = 4 / H;                          // table addresses (and table reads) per step
            constexpr int kScaleStep = H == 2 ? 3 : 2;
            constexpr int kConv0 = H == 2 ? 5 : 4, CPS = 2 / H; // first converting step, weight pairs per step
            constexpr int kAhead = 3;
            constexpr int kLoad0 = 6, kLoads = XJ + AQ;      // steps kLoad0 .. of the tile carry its loads
            static_assert(kLoad0 + kLoads <= 4 * MB, "more tile loads than steps");
            const bool spread = kt + 1 < kt1 && (kt + 2) * 128 <= K;
            bf16x8 Wc[2], Wn[2];
            bf16x8 Xq[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) Xq[i] = *reinterpret_cast<const bf16x8 *>(Xp + i * 4096 + xoff[0]);
            __builtin_amdgcn_sched_barrier(0);
            dequant_stage(0, Wc);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                bf16x8 Aop0[SS], Aop1[SS];
                uint32_t ad[2][4];
                Pair lv[2][4];
                f32x4 S0[2], S1[2];
                const int un = u < 3 ? u + 1 : 3;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int t = MB * u + mb;
                    const bf16x8 Xop = Xq[t % kAhead];
                    acc[0][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wc[0], Xop, acc[0][mb], 0, 0, 0);
                    acc[1][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wc[1], Xop, acc[1][mb], 0, 0, 0);
                    if (t >= kLoad0 && t < kLoad0 + kLoads && spread) {
                        const int i = t - kLoad0, kbn = (kt + 1) * 128;
                        if (i < XJ) {
                            lds_direct_16(Xtile + kbn, xo[i], xl0 + (p ^ 1) * XBUF + i * (TPP * 256));
                        } else if (xm0 + RPP * (i - XJ) < a.r) {
                            lds_direct_16(A16 + kbn, ao[i - XJ], al0 + (p ^ 1) * ABUF + (i - XJ) * (RPP * 256));
                        }
                    }
                    if (t + kAhead < 4 * MB) {
                        const int tn = t + kAhead;
                        Xq[t % kAhead] = *reinterpret_cast<const bf16x8 *>(Xp + (tn % MB) * 4096 + xoff[tn / MB]);
                    }
                    if (u < 3) {
                        if (mb == 0) {
#pragma unroll
                            for (int ss = 0; ss < SS; ++ss) { Aop0[ss] = read_Aop(ss, 2 * un); Aop1[ss] = read_Aop(ss, 2 * un + 1); }
                        }
                        if (mb < 2 * H) {
#pragma unroll
                            for (int e = 0; e < NPS; ++e) {
                                const int lin = mb * NPS + e, q = lin >> 2, pp = lin & 3;
                                ad[q][pp] = pair_at(pair_index<BITS>(cw[q], 4 * un + pp));
                            }
                        }
                        if (mb >= 1 && mb < 1 + 2 * H) {
#pragma unroll
                            for (int e = 0; e < NPS; ++e) {
                                const int lin = (mb - 1) * NPS + e, q = lin >> 2, pp = lin & 3;
                                lv[q][pp] = load_pair(ad[q][pp]);
                            }
                        }
                        if (mb == kScaleStep) {
#pragma unroll
                            for (int q = 0; q < 2; ++q) {
                                S0[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                                S1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                                for (int ss = 0; ss < SS; ++ss) {
                                    S0[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Aop0[ss], Bop[q][ss], S0[q], 0, 0, 0);
                                    S1[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Aop1[ss], Bop[q][ss], S1[q], 0, 0, 0);
                                }
                            }
                        }
                        if (mb >= kConv0 && mb < kConv0 + 8 / CPS) {
#pragma unroll
                            for (int e = 0; e < CPS; ++e) {
                                const int j = (mb - kConv0) * CPS + e, q = j >> 2, pp = j & 3;
                                const float s0 = pp < 2 ? S0[q][2 * pp] : S1[q][2 * pp - 4];
                                const float s1 = pp < 2 ? S0[q][2 * pp + 1] : S1[q][2 * pp - 3];
                                __bf16 w0, w1;
                                weights(lv[q][pp], s0, s1, w0, w1);
                                Wn[q][2 * pp] = w0;
                                Wn[q][2 * pp + 1] = w1;
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                Wc[0] = Wn[0];
                Wc[1] = Wn[1];
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // X operands run kXAhead token blocks ahead of their MFMAs: the first ones of a stage
                // are requested before its dequantisation, each later one as the block kXAhead before
                // it is issued
                constexpr int kXAhead = 2;
                bf16x8 W[R];
                bf16x8 Xq[kXAhead];
#pragma unroll
                for (int i = 0; i < kXAhead; ++i)
                    Xq[i] = *reinterpret_cast<const bf16x8 *>(Xp + i * 4096 + xoff[u]);
                __builtin_amdgcn_sched_barrier(0);
                dequant_stage(u, W);
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const bf16x8 Xop = Xq[mb % kXAhead];
#pragma unroll
                    for (int rho = 0; rho < R; ++rho)
                        acc[rho][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[rho], Xop, acc[rho][mb], 0, 0, 0);
                    if (mb + kXAhead < MB) {
                        Xq[mb % kXAhead] =
                            *reinterpret_cast<const bf16x8 *>(Xp + (mb + kXAhead) * 4096 + xoff[u]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
        if constexpr (F32)
            if (kt + 1 < kt1) store_A32(p ^ 1);
        __builtin_amdgcn_s_waitcnt(0);          // the next tile has landed in LDS, the next codes in registers
        __syncthreads();
#pragma unroll
        for (int rho = 0; rho < R; ++rho)
#pragma unroll
            for (int q = 0; q < BITS; ++q) cw[rho][q] = cwn[rho][q];
    }

    // ---- epilogue: lane (c,g) holds token 16 mb + c, rows 16 rho + 4 g + {0..3} ------------------------
    // A part that does not start at the tile's first column hands its accumulators over in memory (it is
    // always the first part of its workgroup, so it waits for nothing); the part that does start there
    // is the last one of its workgroup, collects the others in column order and writes Y.  The sum of a
    // tile is therefore taken in a fixed order whatever the timing.
    // Of a 128-token tile that holds at most 64 tokens only the first four of the eight token blocks travel (the
    // buffers keep their size).  14336 x 4096, 4 bits, rank 32, 17 / 40 / 64 tokens, when these went in runs: 37.6 / 37.3 / 37.5 -> 30.4 / 30.2 /
    // 30.3 us (their parts meet now; 28672 x 8192 goes in runs at 17 to 64 tokens, 76 .. 79 us).
    // (Exactly the blocks in use, with a branch for each, was no faster there and cost 2-9 % at 100 and 128 tokens; in
    // 256-token tiles the second form cost registers: 10 % at 2048 tokens.)
    constexpr int kPartFloats = R * MB * NT * 4;
    void *Yp = ly.Y;
    auto store_at = [&](int m, int n, f32x4 v) __attribute__((always_inline)) {          // rows n .. n + 3 of token m
        if (m >= M) return;
        if (n + 3 < N) {
            store_out4(Yp, (size_t)m * N + n, v, a.y_f32);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (n + e >= N) continue;
                if (a.y_f32) reinterpret_cast<float *>(Yp)[(size_t)m * N + n + e] = v[e];
                else reinterpret_cast<uint16_t *>(Yp)[(size_t)m * N + n + e] = bf16_bits(v[e]);
            }
        }
    };
    auto store_block = [&](int rho, int mb, f32x4 v) __attribute__((always_inline)) { store_at(m_wave + 16 * mb + c, n_wave + 16 * rho + 4 * g, v); };
    // A tile that G workgroups share in equal parts, one each: every one of them finishes a slice of MB / G token blocks.  It
    // writes the other slices for their owners, counts itself in, waits for the others and adds what they have written of its
    // own, in column order (the sums are those of the form below).  All CUs then write, read and store Y, 1 / G of a tile each,
    // and only blocks with tokens in them travel.  us, before (one of them collected the tile) / this, 4 bits, rank 32 where
    // nothing else is said:
    //   4096 x 4096    32 tokens 24.1 / 19.1, 64 23.7 / 19.7, 128 28.5 / 21.6, 300 37.3 / 31.7, 512 39.4 / 33.1, 2048 80.2 / 73.0;
    //                  500 tokens, fp32 rank 16 49.2 / 42.3
    //   1024 x 4096    300 tokens 30.7 / 19.2;   4096 x 14336 2048 209.6 / 203.7
    // (of these 1 us where eight meet, and less where fewer do, is the first thread's word to the others in LDS.)
    // The wait is bounded (a.polls), and giving it up costs no more than time: the workgroup then also writes its own slice and
    // goes, and another finishes it (lords_meet.h).  So a tile needs no two of its workgroups to run at the same time.
    // That they do is what makes it fast: they are neighbours in the order of dispatch (blockIdx.x in steps of 8), so on an
    // idle chip all but the last few of a launch are resident together.
    // Parts and counter are agent-scope accesses (sc1: they pass the XCD's L2 by), the part's stores have been acknowledged by
    // all waves before the count, and nothing else is handed over, so neither a write-back nor an invalidation of an L2 is
    // wanted: with a release and an acquire at agent scope around the count, G of each per tile, 3 to 7 us more.
    if constexpr (FORM != kRuns) if (FORM == kMeet || __builtin_expect((ly.meet | walk) != 0, 0)) {       // (behind the other form in the code)
        // (what this wants of its thread is worked out again: registers of the K loop)
        int t_out = tid;
        asm volatile("" : "+v"(t_out));
        const int c_out = t_out & 15, g_out = (t_out >> 4) & 3, w_out = __builtin_amdgcn_readfirstlane(t_out >> 6);
        const int n_out = n_blk + 16 * R * (w_out % WN), m_out = m_blk + 16 * MB * (w_out / WN);
        // (... and of its workgroup: 150 to 200 instructions that the compiler would otherwise place in front of the first part,
        // 0.5 us of every launch)
        int own = meet_part, wg_first = wg - own, tokens = M;
        uint64_t part_base = (uint64_t)(uintptr_t)ly.part;
        uint32_t *counter = ly.arrived;
        asm volatile("" : "+s"(own), "+s"(wg_first), "+s"(tokens), "+s"(part_base), "+s"(counter));
        float *const parts_of_tile = (float *)(uintptr_t)part_base + ((size_t)wg_first << walk) * kPartFloats;
        counter += T;
        auto finish_at = [&](int m, int n, f32x4 v) __attribute__((always_inline)) {
            if (ly.gate) {
                const f32x4_any ga = *reinterpret_cast<const f32x4_any *>(ly.gate + (size_t)min(m, tokens - 1) * N + min(n, N - 1));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = ga[e] / (1.0f + __expf(-ga[e])) * v[e];
            }
            store_at(m, n, v);
        };
        if constexpr (FORM == kWalk) if (walk) {
            // Several of a tile's parts by one workgroup, one after the other: each is summed from zero and goes to memory, so that the
            // tile has the sum that it has where each part is a workgroup's own.  (In registers there is room for one part.)
            // (Added into the accumulators of the next part, which a K loop follows, they cost 900 to 1200 spilled registers.)
            if (!ly.meet) {
                // the tile is this workgroup's alone: the sum so far, which a thread reads back where it wrote it
                float *sum = parts_of_tile + t_out * 4;
                constexpr int TB = std::min(8, MB * R);
#pragma unroll
                for (int b0 = 0; b0 < MB * R; b0 += TB) {
                    if (m_out + 16 * (b0 / R) >= tokens) continue;
                    asm volatile("" : "+v"(sum));
                    f32x4 v[TB];
#pragma unroll
                    for (int b = 0; b < TB; ++b) v[b] = walked > 1 ? *reinterpret_cast<const f32x4 *>(sum + ((b0 + b) % R * MB + (b0 + b) / R) * (NT * 4)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[b][e] = walked > 1 ? v[b][e] + acc[(b0 + b) % R][(b0 + b) / R][e] : acc[(b0 + b) % R][(b0 + b) / R][e];
                        if (walked == 1 << walk) {
                            int m = m_out + 16 * ((b0 + b) / R) + c_out, n = n_out + 16 * ((b0 + b) % R) + 4 * g_out;
                            asm volatile("" : "+v"(m), "+v"(n));
                            finish_at(m, n, v[b]);
                        } else {
                            *reinterpret_cast<f32x4 *>(sum + ((b0 + b) % R * MB + (b0 + b) / R) * (NT * 4)) = v[b];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (walked == 1 << walk) return;
                continue;
            }
            // All parts to memory, and a slice of the tile added from there by each workgroup; who does not wait leaves its own, as below.
            float *dst = parts_of_tile + own * (kPartFloats << walk) + (walked - 1) * kPartFloats + t_out * 4;
            asm volatile("" : "+v"(dst));
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                if (m_out + 16 * mb >= tokens) continue;
#pragma unroll
                for (int rho = 0; rho < R; ++rho) store16_agent(dst + (rho * MB + mb) * (NT * 4), acc[rho][mb]);
                asm volatile("" : "+v"(dst));
            }
            if (walked != 1 << walk) continue;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            uint32_t *const verdict = reinterpret_cast<uint32_t *>(smem);
            const int log = ly.meet;
            if (t_out == 0) {
                __hip_atomic_fetch_add(counter, meet_unit(log), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                uint32_t now, mine = 0;
                for (int polls = a.polls;; --polls) {
                    now = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((now & kMeetAllThere) || polls <= 0) break;
                    __builtin_amdgcn_s_sleep(2);
                }
                const bool stays = (now & kMeetAllThere) != 0;
                if (!stays) now = __hip_atomic_fetch_add(counter, 1u << own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (now & kMeetAllThere) {
                    if (!stays || (now & kMeetSlices)) mine = __hip_atomic_fetch_and(counter, ~kMeetSlices, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kMeetSlices;
                    __hip_atomic_fetch_add(counter, meet_leave(log, mine, stays), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                *verdict = stays ? mine | 1u << own : mine;
            }
            __syncthreads();
            const int blocks = MB * R >> log;                  // of a slice
            auto add_up = [&](auto parts) __attribute__((always_inline)) {
                // (16 loads in flight)
                constexpr int G = decltype(parts)::value, TB = std::min(16, 2 * MB * R) / G;
                for (uint32_t left = __builtin_amdgcn_readfirstlane(*verdict); left != 0; left &= left - 1) {
                    const int b0 = __builtin_ctz(left) * blocks;
#pragma nounroll
                    for (int b = b0; b < b0 + blocks; b += TB) {
                        if (m_out + 16 * (b / R) >= tokens) break;
                        f32x4 t[G][TB];
#pragma unroll
                        for (int i = 0; i < G; ++i) {
                            const float *src = parts_of_tile + i * kPartFloats + b / R * (NT * 4) + t_out * 4;
                            asm volatile("" : "+v"(src));
#pragma unroll
                            for (int q = 0; q < TB; ++q) {
                                t[i][q] = load16_agent(src + (q % R * MB + q / R) * (NT * 4));
                                asm volatile("" : "+v"(src));
                            }
                        }
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
                        for (int q = 0; q < TB; ++q) {
#pragma unroll
                            for (int i = 0; i < G; ++i) {
                                asm volatile("" : "+v"(t[i][q]));                       // (not before the wait)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    if (i) t[0][q][e] += t[i][q][e];
                            }
                            int m = m_out + 16 * (b / R + q / R) + c_out, n = n_out + 16 * (q % R) + 4 * g_out;
                            asm volatile("" : "+v"(m), "+v"(n), "+v"(t[0][q]));
                            finish_at(m, n, t[0][q]);
                        }
                    }
                }
            };
            if (MB < 8 || cut_log == 2) add_up(std::integral_constant<int, 4>{});
            else add_up(std::integral_constant<int, MB < 8 ? 4 : 8>{});
            return;
        }
        auto meet = [&](auto parts) __attribute__((always_inline)) {
            constexpr int G = decltype(parts)::value, MS = MB / G, kLog = G == 2 ? 1 : G == 4 ? 2 : 3;
            float *dst = parts_of_tile + own * kPartFloats + t_out * 4;
            asm volatile("" : "+v"(dst));        // (addresses are made here, not kept in registers over the K loop)
#pragma unroll
            for (int s = 0; s < G; ++s) {
                if (s == own || m_out + 16 * s * MS >= tokens) continue;       // (tokens beyond M do not travel)
#pragma unroll
                for (int q = 0; q < MS; ++q) {
#pragma unroll
                    for (int rho = 0; rho < R; ++rho) store16_agent(dst + (rho * MB + s * MS + q) * (NT * 4), acc[rho][s * MS + q]);
                    asm volatile("" : "+v"(dst));                       // (addresses one by one: registers)
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            // (of the workgroup's first thread: its slice to finish, nothing, or slices that lie in memory; the tiles in LDS are done with)
            uint32_t *const verdict = reinterpret_cast<uint32_t *>(smem);
            if (t_out == 0) {
                __hip_atomic_fetch_add(counter, meet_unit(kLog), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                uint32_t now, taken = 0;
                for (int polls = a.polls;; --polls) {
                    now = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((now & kMeetAllThere) || polls <= 0) break;
                    __builtin_amdgcn_s_sleep(2);
                }
                if (now & kMeetAllThere) {
                    if (__builtin_expect((now & kMeetSlices) != 0, 0))
                        taken = __hip_atomic_fetch_and(counter, ~kMeetSlices, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kMeetSlices;
                    __hip_atomic_fetch_add(counter, meet_leave(kLog, taken, true), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    taken = kMeetAllThere;
                }
                *verdict = taken;
            }
            __syncthreads();
            uint32_t mine = __builtin_amdgcn_readfirstlane(*verdict);
            if (__builtin_expect(mine != 0, 0)) {
                const bool gave_up = mine == kMeetAllThere;
                if (gave_up) {
                    // waited long enough: the own slice goes to memory too
#pragma unroll
                    for (int s = 0; s < G; ++s) {
                        if (s != own || m_out + 16 * s * MS >= tokens) continue;
#pragma unroll
                        for (int q = 0; q < MS; ++q) {
#pragma unroll
                            for (int rho = 0; rho < R; ++rho) store16_agent(dst + (rho * MB + s * MS + q) * (NT * 4), acc[rho][s * MS + q]);
                            asm volatile("" : "+v"(dst));
                        }
                    }
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                    if (t_out == 0) {
                        uint32_t taken = 0;
                        if (__hip_atomic_fetch_add(counter, 1u << own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kMeetAllThere) {
                            taken = __hip_atomic_fetch_and(counter, ~kMeetSlices, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kMeetSlices;
                            __hip_atomic_fetch_add(counter, meet_leave(kLog, taken, false), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        *verdict = taken;
                    }
                    __syncthreads();
                    mine = __builtin_amdgcn_readfirstlane(*verdict);
                }
                // slices of which all parts lie in memory, a block at a time
                for (uint32_t left = mine; left != 0; left &= left - 1) {
                    const int b0 = __builtin_ctz(left) * MS;
                    if (m_out + 16 * b0 >= tokens) continue;
#pragma nounroll
                    for (int b = 0; b < MS * R; ++b) {
                        const int rho = b % R, mb = b0 + b / R;
                        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma nounroll
                        for (int i = 0; i < G; ++i) {
                            uint64_t *src = reinterpret_cast<uint64_t *>(parts_of_tile + (size_t)i * kPartFloats + (rho * MB + mb) * (NT * 4) + t_out * 4);
                            const uint64_t lo = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            const uint64_t hi = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            const f32x4 t = {__builtin_bit_cast(float, (uint32_t)lo), __builtin_bit_cast(float, (uint32_t)(lo >> 32)),
                                             __builtin_bit_cast(float, (uint32_t)hi), __builtin_bit_cast(float, (uint32_t)(hi >> 32))};
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = i == 0 ? t[e] : v[e] + t[e];
                        }
                        const int m = m_out + 16 * mb + c_out, n = n_out + 16 * rho + 4 * g_out;
                        finish_at(m, n, v);
                    }
                }
                if (gave_up) return;
            }
            if (m_out + 16 * own * MS >= tokens) return;
            // (accumulators are only read, where they are: blocks per round trip by the registers beside them)
            constexpr int TB = std::min(MS * R, G == 2 ? 16 : G == 4 ? 4 : 2);
#pragma unroll
            for (int b0 = 0; b0 < MS * R; b0 += TB) {
                f32x4 t[G - 1][TB];
#pragma unroll
                for (int i = 0; i < G - 1; ++i) {
                    const float *src = parts_of_tile + (i + (i >= own)) * kPartFloats + own * (MS * NT * 4) + t_out * 4;
                    asm volatile("" : "+v"(src));
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        t[i][b] = load16_agent(src + ((b0 + b) % R * MB + (b0 + b) / R) * (NT * 4));
                        asm volatile("" : "+v"(src));
                    }
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
                for (int i = 0; i < G - 1; ++i)
#pragma unroll
                    for (int b = 0; b < TB; ++b) asm volatile("" : "+v"(t[i][b]));       // (not before the wait)
#pragma unroll
                for (int s = 0; s < G; ++s) {
                    if (s != own) continue;
                    asm volatile("" ::: "memory");          // (a branch, not a choice between slices: registers)
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        const f32x4 mine = acc[(b0 + b) % R][s * MS + (b0 + b) / R];
                        f32x4 v = s == 0 ? mine : t[0][b];
#pragma unroll
                        for (int i = 1; i < G; ++i) {
                            const f32x4 next = i < s ? t[i < G - 1 ? i : 0][b] : i == s ? mine : t[i - 1][b];
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] += next[e];
                        }
                        asm volatile("" : "+v"(v));
                        t[0][b] = v;
                    }
                }
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    int m = m_out + 16 * (own * MS + (b0 + b) / R) + c_out, n = n_out + 16 * ((b0 + b) % R) + 4 * g_out;
                    asm volatile("" : "+v"(m), "+v"(n));
                    finish_at(m, n, t[0][b]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (ly.meet == 1) meet(std::integral_constant<int, 2>{});
        else if (MB < 8 || ly.meet == 2) meet(std::integral_constant<int, 4>{});
        else meet(std::integral_constant<int, MB < 8 ? 4 : 8>{});
        return;
    }
    if constexpr (FORM != kMeet) {
    const bool few = MB == 8 && M - m_wave <= 64;
    if (kt0 != 0) {
        float *dst = ly.part + (size_t)wg * kPartFloats + tid * 4;
        asm volatile("" : "+v"(dst));        // (addresses are made here, not kept in registers over the K loop)
#pragma unroll
        for (int half = 0; half < 2; ++half)
            if (half == 0 || !few)
#pragma unroll
                for (int rho = 0; rho < R; ++rho)
#pragma unroll
                    for (int mb = half * (MB / 2); mb < (half + 1) * (MB / 2); ++mb)
                        store16_agent(dst + (rho * MB + mb) * (NT * 4), acc[rho][mb]);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(ly.arrived + T, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        continue;
    }
    if (kt1 != a.ntiles_k) {
        const int others = (a.ntiles_k - kt1 + ly.per - 1) / ly.per;       // the workgroups after this one, up to the tile's end
        if (tid == 0) {
            // (The parts waited for are first parts of their workgroups and never wait themselves, so one free CU an XCD is enough for the
            // wait to end, whatever else waits.  The bound, some two seconds, is there so that every wave ends; a launch whose next
            // workgroup gets no CU for that long would have a wrong sum.)
            int spins = 0;
            while ((int)__hip_atomic_load(ly.arrived + T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < others && ++spins < (1 << 21))
                __builtin_amdgcn_s_sleep(8);
            __hip_atomic_store(ly.arrived + T, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        // (`few` is decided outside the loop: inside, the accumulators changed register files with every part)
        auto add_parts = [&](auto nr, auto nb) __attribute__((always_inline)) {
            constexpr int NR = decltype(nr)::value, NBK = decltype(nb)::value;
            for (int j = 1; j <= others; ++j) {
                const float *src = ly.part + (size_t)(wg + j) * kPartFloats + tid * 4;
                asm volatile("" : "+v"(src));
                // sixteen loads in flight (eight for half a tile): what the registers beside the accumulators
                // hold; each wait is a round trip to memory
#pragma unroll
                for (int rho0 = 0; rho0 < R; rho0 += NR) {
                    f32x4 t[NR * NBK];
#pragma unroll
                    for (int q = 0; q < NR * NBK; ++q) t[q] = load16_agent(src + ((rho0 + q / NBK) * MB + q % NBK) * (NT * 4));
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
                    for (int q = 0; q < NR * NBK; ++q) {
                        asm volatile("" : "+v"(t[q]));                                  // (not before the wait)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[rho0 + q / NBK][q % NBK][e] += t[q][e];
                    }
                }
            }
        };
        static_assert(R == 2 && (MB == 4 || MB == 8 || MB == 16), "at most sixteen accumulator blocks a round trip");
        if constexpr (MB == 16) {
            add_parts(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
        } else if (MB == 4 || few) {
            add_parts(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
        } else {
            add_parts(std::integral_constant<int, 2>{}, std::integral_constant<int, MB < 8 ? MB : 8>{});
        }
    }
    if (ly.gate) {
        // A gate/up pair: this is the up product, the gate's fp32 sums lie in memory.  Loads of eight token blocks in
        // flight; addresses are clamped to the matrix's rows, a load of its last columns may reach 12 bytes beyond
        // them (the buffer is that much longer), and what such loads bring is not stored.
        constexpr int GB = MB < 8 ? MB : 8;
#pragma unroll
        for (int rho = 0; rho < R; ++rho) {
            const float *col = ly.gate + min(n_wave + 16 * rho + 4 * g, N - 1);
#pragma unroll
            for (int b0 = 0; b0 < MB; b0 += GB) {
                int m0 = m_wave + 16 * b0 + c;
                asm volatile("" : "+v"(m0));                  // (addresses of one batch at a time: registers)
                f32x4_any t[GB];
#pragma unroll
                for (int i = 0; i < GB; ++i) t[i] = *reinterpret_cast<const f32x4_any *>(col + (size_t)min(m0 + 16 * i, M - 1) * N);
#pragma unroll
                for (int i = 0; i < GB; ++i) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = t[i][e] / (1.0f + __expf(-t[i][e])) * acc[rho][b0 + i][e];
                    store_block(rho, b0 + i, v);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int rho = 0; rho < R; ++rho) store_block(rho, mb, acc[rho][mb]);
    }
    }
    }   // parts of this workgroup
}

template <int BITS, int SS, int WM, int R, int WN, int MB, bool F32, bool MULTI, PfForm FORM = kRuns>
static hipError_t launch_pf_t(const PrefillArgsT<MULTI ? kMaxBatch : 1> &a, dim3 grid, hipStream_t st)
{
    if constexpr (FORM == kRuns) {
        int meet = 0, walk = 0;
        for (int l = 0; l < a.L; ++l) meet |= a.layer[l].meet, walk |= a.layer[l].walk;
        if (MULTI && walk) return launch_pf_t<BITS, SS, WM, R, WN, MB, F32, MULTI, MULTI ? kWalk : kMeet>(a, grid, st);
        if (meet) return launch_pf_t<BITS, SS, WM, R, WN, MB, F32, MULTI, MULTI ? kEither : kMeet>(a, grid, st);
    }
    const size_t smem = (size_t)2 * (16 * MB * WM) * 256 + (size_t)2 * (32 * SS) * 256 + (size_t)(1 << (2 * BITS)) * kPfCopies * pf_pair_bytes(F32);
    static LdsOptIn lds_opt_in;
    {
        const hipError_t e = allow_dynamic_lds(lds_opt_in, reinterpret_cast<const void *>(&prefill_kernel<BITS, SS, WM, R, WN, MB, F32, MULTI, FORM>), smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((prefill_kernel<BITS, SS, WM, R, WN, MB, F32, MULTI, FORM>), grid, dim3(64 * WN * WM), smem, st, a);
    return hipGetLastError();
}

// The launch of a.layer's matrices, all cut into tiles of one shape.
template <int BITS, bool MULTI>
static hipError_t launch_pf_bits(const PrefillArgsT<MULTI ? kMaxBatch : 1> &a, const PfShape &d, dim3 grid, hipStream_t st)
{
    if (d.ss == 6) return launch_pf_t<BITS, 6, 1, 2, 4, 4, true, MULTI>(a, grid, st);
    hipError_t e = hipErrorInvalidValue;
#define LORDS_PCASE(S_)                                                                                            \
    if (d.ss == S_) {                                                                                               \
        if (d.f32fact) e = S_ < 4 && d.wn == 8 ? launch_pf_t<BITS, (S_ < 4 ? S_ : 1), 1, 2, 8, 8, true, MULTI>(a, grid, st) \
                                               : launch_pf_t<BITS, S_, 1, 2, 4, 8, true, MULTI>(a, grid, st);       \
        else if (S_ == 1 && d.mb == 16) e = launch_pf_t<BITS, 1, 1, 2, 8, 16, false, MULTI>(a, grid, st);           \
        else if (S_ == 1 && d.wm == 2) e = launch_pf_t<BITS, 1, 2, 2, 4, 8, false, MULTI>(a, grid, st);             \
        else if (d.wn == 8) e = launch_pf_t<BITS, S_, 1, 2, 8, 8, false, MULTI>(a, grid, st);                       \
        else e = launch_pf_t<BITS, S_, 1, 2, 4, 8, false, MULTI>(a, grid, st);                                      \
    }
    LORDS_PCASE(1) LORDS_PCASE(2) LORDS_PCASE(4)
#undef LORDS_PCASE
    return e;
}

}  // namespace lords
