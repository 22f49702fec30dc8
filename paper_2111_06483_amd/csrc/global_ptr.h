// Pointers that kernels find in tables.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sar {

// A pointer into device memory that itself lies in LDS or in device memory (tables of the blocks' arrays).  Kept as a plain
// pointer, the compiler cannot tell what it points to and reads through it by FLAT instructions: their answers count in two
// counters and come in no order, so that a wavefront waits for all it has under way before it uses the first of them, and
// every address is a register pair that is tested for LDS.  (Kernel times over 140 steps of 10 us to 90 ms, geometric means: the
// sum's forward kernel 3% shorter by GLOBAL instructions, single-edge sources 3%, the generic attention kernel 2%, others 0 to 2%.)
template <typename T>
struct GlobalPtr {
    uint64_t bits;
    GlobalPtr() = default;
    __host__ __device__ inline GlobalPtr(T* p) : bits(reinterpret_cast<uint64_t>(p)) {}
    static __device__ inline GlobalPtr at(uint64_t address)
    {
        GlobalPtr p;
        p.bits = address;
        return p;
    }
    __host__ __device__ inline operator T*() const { return as<T>(); }
    template <typename U>
    __host__ __device__ inline U* as() const
    {
        return (U*)(__attribute__((address_space(1))) U*)bits;
    }
};

}  // namespace sar
