// Integer instructions the verification kernels issue by name.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ej {

// s = a + b; the carry-out of every lane lands in one wave-wide mask.
__device__ inline uint32_t add_carry_mask(uint32_t a, uint32_t b, uint64_t &carry) {
    uint32_t s;
    asm("v_add_co_u32 %0, %1, %2, %3" : "=v"(s), "=s"(carry) : "v"(a), "v"(b));
    return s;
}

// s = a + b + (bit `lane` of cin); carry-outs of every lane in cout.
__device__ inline uint32_t add_carry_chain(uint32_t a, uint32_t b, uint64_t cin, uint64_t &cout) {
    uint32_t s;
    asm("v_addc_co_u32 %0, %1, %2, %3, %4" : "=v"(s), "=s"(cout) : "v"(a), "v"(b), "s"(cin));
    return s;
}

// popcount(x) + acc in one v_bcnt.
__device__ inline uint32_t popc_acc(uint32_t x, uint32_t acc) {
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

}  // namespace ej
