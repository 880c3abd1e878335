// Device-side building blocks shared by the LoRDS kernels (gfx950 only).
//
//  - bit-unpacking of 2/3/4-bit codes held in registers,
//  - bf16 helpers,
//  - the wave-level tile mapping used by the fused kernels, and
//  - access to the (possibly fp32) rank-r factors as bf16 MFMA operands.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lords {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// ---------------------------------------------------------------------------
// A group of 32 consecutive codes of one row occupies BITS dwords.
// code e (0..31) sits at bits [BITS*e, BITS*e+BITS) of that little-endian string.
// `e` is a compile-time constant after unrolling, so this becomes one v_bfe_u32
// (plus a v_alignbit_b32 for the two 3-bit codes that straddle a dword).
// ---------------------------------------------------------------------------
template <int BITS>
__device__ __forceinline__ uint32_t code_at(const uint32_t (&w)[BITS], int e)
{
    const int o = BITS * e, d = o >> 5, s = o & 31;
    uint32_t v = w[d] >> s;
    if (s + BITS > 32) v |= w[(d + 1) < BITS ? d + 1 : d] << (32 - s);
    return v & ((1u << BITS) - 1u);
}

// Load the BITS dwords of one 32-code group (4-byte aligned address).
template <int BITS>
__device__ __forceinline__ void load_group(const uint8_t *p, uint32_t (&w)[BITS])
{
    const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
#pragma unroll
    for (int i = 0; i < BITS; ++i) w[i] = q[i];
}

__device__ __forceinline__ uint16_t bf16_bits(float x)
{
    __bf16 h = (__bf16)x;                      // v_cvt_pk_bf16_f32, round-to-nearest-even
    return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b)
{
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// ---------------------------------------------------------------------------
// The rank-r factors as bf16 MFMA operands.
//
// bf16 factors are used as they are (contraction length r).  fp32 factors are
// split x = hi + lo with hi = bf16(x), lo = bf16(x - hi) and the scale is formed
// as  B A ~= Bhi Ahi + Bhi Alo + Blo Ahi,  i.e. one contraction of length 3r
// over the concatenated operands  B' = [Bhi | Bhi | Blo],  A' = [Ahi ; Alo ; Ahi].
// Every product of two bf16 values is exact in the fp32 accumulator, and the
// dropped Blo Alo term is below 2^-16 relative.
// ---------------------------------------------------------------------------
struct Factors {
    const void *B;   // N x r
    const void *A;   // r x K
    int N, K, r;
    int f32;         // 0: bf16 factors, 1: fp32 factors
    int r_eff;       // r (bf16) or 3r (fp32)
};

__device__ __forceinline__ uint16_t factorA_bits(const Factors &f, int jj, int k)
{
    if (jj >= f.r_eff || k >= f.K) return 0;
    if (!f.f32) return reinterpret_cast<const uint16_t *>(f.A)[(size_t)jj * f.K + k];
    const int seg = jj / f.r, j = jj - seg * f.r;
    const float x = reinterpret_cast<const float *>(f.A)[(size_t)j * f.K + k];
    const uint16_t hi = bf16_bits(x);
    return seg == 1 ? bf16_bits(x - bf16_to_f32(hi)) : hi;
}

__device__ __forceinline__ uint16_t factorB_bits(const Factors &f, int n, int jj)
{
    if (jj >= f.r_eff || n >= f.N) return 0;
    if (!f.f32) return reinterpret_cast<const uint16_t *>(f.B)[(size_t)n * f.r + jj];
    const int seg = jj / f.r, j = jj - seg * f.r;
    const float x = reinterpret_cast<const float *>(f.B)[(size_t)n * f.r + j];
    const uint16_t hi = bf16_bits(x);
    return seg == 2 ? bf16_bits(x - bf16_to_f32(hi)) : hi;
}

// Eight rank entries j0 .. j0 + 7 of row n of a bf16 factor with ANY number r of entries per row (row-major, N rows):
// one 16-byte load at the row's own alignment (2 bytes; global loads need none on gfx950) instead of eight 2-byte
// gathers, entries of the next row masked off afterwards.  At the array's end the load is moved back so that it stays
// inside and its entries are shifted into place.  The fetch can be issued far ahead; rank8_fix belongs to the use.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
// (A factor of fewer than eight entries in all has no 16 bytes to read: the fetch then reads them from `spare`, any
// readable 16 bytes, so that it stays one load without a branch, and rank8_fix gathers the entries.)
__device__ __forceinline__ bool rank8_tiny(int N, int r) { return N < 8 && N * r < 8; }
__device__ __forceinline__ u32x4 rank8_fetch(const uint16_t *B, const uint16_t *spare, int n, int j0, int N, int r)
{
    const uint16_t *base = rank8_tiny(N, r) ? spare : B;                     // (the same in all lanes, as is `last`)
    const uint64_t last = rank8_tiny(N, r) ? 0 : (uint64_t)N * (uint32_t)r - 8;
    const uint64_t at = (uint64_t)(uint32_t)n * (uint32_t)r + (uint32_t)(j0 < r ? j0 : 0);
    const u32x4_any w = *reinterpret_cast<const u32x4_any *>(base + (at < last ? at : last));
    return u32x4{w[0], w[1], w[2], w[3]};
}
// Entries of eight that lie beyond the row's end (v of them belong to it) become zero.
__device__ __forceinline__ u32x4 rank8_keep(u32x4 t, int v)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = v >= 2 * e + 2 ? t[e] : v == 2 * e + 1 ? t[e] & 0xffffu : 0u;
    return t;
}
// The entries of a load that was moved back by `back` (0 .. 7) come to the front.
__device__ __forceinline__ u32x4 rank8_shift(u32x4 t, int back)
{
    uint64_t lo = (uint64_t)t[0] | ((uint64_t)t[1] << 32), hi = (uint64_t)t[2] | ((uint64_t)t[3] << 32);
    if (back >= 4) { lo = hi; hi = 0; back -= 4; }
    if (back != 0) { lo = (lo >> (16 * back)) | (hi << (64 - 16 * back)); hi >>= 16 * back; }
    return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}
__device__ __forceinline__ u32x4 rank8_gather(const uint16_t *row, int j0, int r)
{
    u32x4 t = u32x4{0u, 0u, 0u, 0u};
#pragma unroll 1
    for (int e = 0; e < 8; ++e) {
        const uint32_t w = j0 + e < r ? (uint32_t)row[j0 + e] << (16 * (e & 1)) : 0u;
        t[0] |= (e >> 1) == 0 ? w : 0u;
        t[1] |= (e >> 1) == 1 ? w : 0u;
        t[2] |= (e >> 1) == 2 ? w : 0u;
        t[3] |= (e >> 1) == 3 ? w : 0u;
    }
    return t;
}
// `end`: true where a row within eight of the last may be among the lanes' (the shifting is skipped elsewhere).
__device__ __forceinline__ u32x4 rank8_fix(u32x4 t, const uint16_t *B, int n, int j0, int N, int r, bool end)
{
    if (end) {
        if (rank8_tiny(N, r)) return rank8_gather(B + (size_t)n * r, j0, r);
        const int rem = min(N - n, 8) * r - j0;              // entries from here to the array's end (or enough of them)
        t = rank8_shift(t, j0 < r && rem < 8 ? 8 - rem : 0);
    }
    return rank8_keep(t, r - j0);
}

// Four neighbouring outputs of one token, at the alignment their address happens to have (N need not be a multiple of
// four): one 16- or 8-byte store.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
__device__ __forceinline__ void store_out4(void *Y, size_t at, f32x4 v, int y_f32)
{
    if (y_f32) {
        *reinterpret_cast<f32x4_any *>(reinterpret_cast<float *>(Y) + at) = f32x4_any{v[0], v[1], v[2], v[3]};
    } else {
        u32x2_any o;
        o[0] = (uint32_t)bf16_bits(v[0]) | ((uint32_t)bf16_bits(v[1]) << 16);
        o[1] = (uint32_t)bf16_bits(v[2]) | ((uint32_t)bf16_bits(v[3]) << 16);
        *reinterpret_cast<u32x2_any *>(reinterpret_cast<uint16_t *>(Y) + at) = o;
    }
}

// fp32 sums that pass from one workgroup to another through memory: 16-byte stores and loads at
// agent scope (sc1: written through to, and read from, the level all XCDs share), so that the hand-over
// needs no write-back or invalidation of a whole L2.  Written as assembly because the language
// offers agent-scope atomic accesses of at most 8 bytes; the waits are placed by hand.
__device__ __forceinline__ void store16_agent(float *p, f32x4 v)
{
    // (A store of more than 8 bytes reads its data a cycle late: a vector instruction right behind it must not write those
    // registers.  The compiler keeps that distance for stores it knows, not for this one: a copy out of an accumulation
    // register right behind the store changed the first of its four floats.)
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ f32x4 load16_agent(const float *p)
{
    f32x4 v;
    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v) : "v"(p) : "memory");
    return v;
}

}  // namespace lords
