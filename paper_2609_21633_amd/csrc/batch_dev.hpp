// Device side of a batched launch (SlotBatch): copy blockIdx.z of the grid
// works on the buffers of slot z, at byte offset off[z] from the launch's
// pointers; a null pointer stays null.
#pragma once

#include <type_traits>

#include "tng_internal.hpp"

namespace tng {

// Byte-pointer arithmetic (not an integer round trip), so the compiler keeps
// the kernel argument's global address space and emits global, not flat,
// memory instructions.
template <class P>
__device__ __forceinline__ P* at_slot(P* p, long long off) {
    using B = typename std::conditional<std::is_const<P>::value, const char, char>::type;
    return p == nullptr ? p : reinterpret_cast<P*>(reinterpret_cast<B*>(p) + off);
}

__device__ __forceinline__ long long slot_off(const SlotBatch& sb) { return sb.off[blockIdx.z]; }

// vector count (or table index) of this copy: the per-slot one when given
__device__ __forceinline__ int slot_count(const SlotBatch& sb, int n) {
    return sb.has_cnt ? sb.cnt[blockIdx.z] : n;
}

// Division of 32-bit numbers by a launch constant: t / d = (umulhi(t, mul) + t) >> sh,
// exact for all t.
struct MagicDiv {
    unsigned mul;   // ceil(2^(32 + sh) / d) - 2^32
    int sh;         // ceil(log2 d)
};
inline MagicDiv magic_div(unsigned d) {
    MagicDiv m{0u, 0};
    while ((1ull << m.sh) < d) ++m.sh;
    const unsigned long long big = 1ull << (32 + m.sh);
    m.mul = (unsigned)((big + d - 1) / d - (1ull << 32));
    return m;
}
__device__ __forceinline__ unsigned mdiv(unsigned t, MagicDiv m) {
    return (unsigned)((((unsigned long long)__umulhi(t, m.mul)) + t) >> m.sh);
}

// Block number in XCD-aware order: the dispatcher deals consecutive workgroups to the eight
// XCDs in turn; each XCD takes a contiguous run of blocks instead, so that blocks that
// share data run under one L2.
__device__ __forceinline__ unsigned xcd_block() {
    const unsigned nbk = gridDim.x, q = nbk >> 3, r = nbk & 7, x = blockIdx.x & 7;
    return x * q + min(x, r) + (blockIdx.x >> 3);
}

// Lane l receives lane l + 1's value, lane 63 zero (DPP wavefront shift).
__device__ __forceinline__ float lane_above(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_above(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Lane l receives lane l - 1's value, lane 0 zero (DPP wavefront shift).
__device__ __forceinline__ float lane_below(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_below(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

}  // namespace tng
