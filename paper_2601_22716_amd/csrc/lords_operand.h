// Buffer descriptors, direct loads into LDS through them, and sums kept in the accumulation registers: shared by the kernels with
// one wave per SIMD and all 512 registers of it (lords_prefill_wide.hip, lords_two_pass.hip).
#pragma once
#include "lords_decode_common.h"

namespace lords {

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int BufferRsrc;
// Buffer descriptor of `bytes` bytes from `base` (raw): loads beyond them return zeros and touch nothing.
__device__ __forceinline__ BufferRsrc make_rsrc(uint64_t base, uint32_t bytes)
{
    return BufferRsrc{(int)(uint32_t)base, (int)((uint32_t)(base >> 32) & 0xffffu), (int)bytes, 0x00020000};
}
// Every lane brings the 16 bytes at off + shift of the descriptor straight into LDS, at lds_wave_base + i * 4096 + 16 * lane
// (m0 holds the wave's base).  In assembly so that the compiler does not make later LDS reads wait for it; the kernel waits itself.
// The whole offset sits in the lane's register: that is what the descriptor's bounds are checked against.
__device__ __forceinline__ void lds_buffer_16(BufferRsrc r, uint32_t off, uint32_t shift, uint32_t lds_wave_base, int i)
{
    uint32_t at;
    asm volatile("s_add_u32 m0, %1, %5\n\tv_add_u32 %0, %2, %3\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds"
                 : "=&v"(at) : "s"(lds_wave_base), "v"(off), "v"(shift), "s"(r), "i"(i * 4096) : "memory", "m0", "scc");
}
// acc += w x in accumulation registers (all 256 of them hold the tile's sums; the vector registers are for operands).
__device__ __forceinline__ void mfma_acc(f32x4 &acc, bf16x8 w, bf16x8 x)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}
__device__ __forceinline__ f32x4 read_acc(f32x4 acc)
{
    float x[4];
    asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]) : "a"(acc[0]), "a"(acc[1]), "a"(acc[2]), "a"(acc[3]));
    return f32x4{x[0], x[1], x[2], x[3]};
}

}  // namespace lords
