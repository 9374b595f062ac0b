// Device helpers shared by the decode kernels.  Not part of the public ABI.
#pragma once
#include "fv_internal.h"

namespace fv {

// The engine reads its arguments from a copy in the workspace through the
// constant address space: field loads are scalar loads in every function.
typedef __attribute__((address_space(4))) const EngineArgs cargs_t;
// the argument block is the same for every lane: keep its address scalar
__device__ __forceinline__ cargs_t& uniform_args(cargs_t& a) {
    const uint64_t v = reinterpret_cast<uint64_t>(&a);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return *reinterpret_cast<cargs_t*>(((uint64_t)hi << 32) | lo);
}

// ---------------------------------------------------------------- access helpers
template <typename T>
__device__ __forceinline__ T ld_c(const T* p) {  // coherent across XCDs
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_c(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// st_c on a pointer known to address global memory: a global (not flat)
// store, so waiting for LDS results does not also wait for it
template <typename T>
__device__ __forceinline__ void st_cg(T* p, T v) {
    typedef __attribute__((address_space(1))) T gT;
    __hip_atomic_store(reinterpret_cast<gT*>(reinterpret_cast<uint64_t>(p)), v, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_cf(const float* p) {
    return __uint_as_float(ld_c(reinterpret_cast<const uint32_t*>(p)));
}
__device__ __forceinline__ void st_cf(float* p, float v) {
    st_c(reinterpret_cast<uint32_t*>(p), __float_as_uint(v));
}
__device__ __forceinline__ Row ld_row(const Row* p) {
    const uint64_t* q = reinterpret_cast<const uint64_t*>(p);
    uint64_t w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = ld_c(q + k);
    Row r;
    __builtin_memcpy(&r, w, sizeof r);
    return r;
}
__device__ __forceinline__ void st_row(Row* p, const Row& r) {
    uint64_t w[8];
    __builtin_memcpy(w, &r, sizeof r);
    uint64_t* q = reinterpret_cast<uint64_t*>(p);
#pragma unroll
    for (int k = 0; k < 8; ++k) st_c(q + k, w[k]);
}
__device__ __forceinline__ int32_t clampi(int32_t v, int32_t hi) { return v < 0 ? 0 : (v >= hi ? hi - 1 : v); }
// A value known to be the same in every lane, moved to a scalar register (so
// that the addresses and loops it controls are scalar too).
__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Explicit address spaces for the hot loops, which live in non-inlined
// functions (where pointers are generic): log A is never written during a
// decode, so a wave-uniform pointer to it may be read through the constant
// address space (scalar loads); per-lane data goes through the global one.
typedef __attribute__((address_space(4))) const float cfloat_t;
typedef __attribute__((address_space(1))) const float gfloat_t;
__device__ __forceinline__ cfloat_t* uniform_const(const float* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<cfloat_t*>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ gfloat_t* as_global(const float* p) {
    return reinterpret_cast<gfloat_t*>(reinterpret_cast<uint64_t>(p));
}
// coherent (agent-scope) load through the global address space
__device__ __forceinline__ float ld_cg(const float* p) {
    typedef __attribute__((address_space(1))) const uint32_t gu32_t;
    gu32_t* q = reinterpret_cast<gu32_t*>(reinterpret_cast<uint64_t>(p));
    return __uint_as_float(__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Final arg-max keys are combined by tiles and read by the finalize step
// with coherent loads, so the max is performed at the memory side (sc1).
__device__ __forceinline__ void key_max(unsigned long long* p, unsigned long long v) {
    __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ uint32_t my_xcd() {
    return __builtin_amdgcn_s_getreg((15 << 11) | (0 << 6) | 20) & (kXcd - 1);  // HW_REG_XCC_ID
}

__device__ __forceinline__ unsigned long long order_key(float v, int32_t j) {
    if (v == 0.0f) v = 0.0f;  // -0 and +0 compare equal; the lower index must win
    uint32_t b = __float_as_uint(v);
    uint32_t o = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return ((unsigned long long)o << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)j);
}

// Emission score of the Gaussian point model: state j's point xy[j] against
// observation t's point obs[t], in float64 with each operation rounded once
// (no contraction into fused multiply-adds), then rounded to float32:
// (float)(c2 * ((x - u)^2 + (y - v)^2) - c0).
__device__ __forceinline__ float gauss2d_score(const double* __restrict__ xy, const double* __restrict__ obs,
                                               double c2, double c0, int32_t t, int32_t j) {
#pragma clang fp contract(off)
    const double dx = xy[2 * (int64_t)j] - obs[2 * (int64_t)t];
    const double dy = xy[2 * (int64_t)j + 1] - obs[2 * (int64_t)t + 1];
    const double sx = dx * dx;
    const double sy = dy * dy;
    const double d2 = sx + sy;
    const double e = c2 * d2;
    return (float)(e - c0);
}

// log B_t(j) of a sequence whose emission data starts at lb: its table's
// entry lb[t * ld + j], or the Gaussian point model's score with lb
// addressing the observations (float64 [T][2]).  emit_kind is uniform.
__device__ __forceinline__ float emission_of(int32_t kind, const double* xy, double c2, double c0,
                                             const float* __restrict__ lb, int64_t ld, int32_t t, int32_t j) {
    if (kind == FV_EMIT_TABLE) return as_global(lb)[(int64_t)t * ld + j];
    return gauss2d_score(xy, reinterpret_cast<const double*>(lb), c2, c0, t, j);
}
__device__ __forceinline__ float emission(cargs_t& a, const float* lb, int64_t ld, int32_t t, int32_t j) {
    return emission_of(a.emit_kind, a.emit_xy, a.emit_c2, a.emit_c0, lb, ld, t, j);
}

// Waits for another block (decodes off the lock-step engine) end by count or
// once the decode has an error, which all of its blocks then see: true on a turn
// (counted from 0) that is the last one.  A wait that ends so leaves the error
// set, and the decode reports it whatever the block goes on to do.
// (The arguments are read on the turns that look at them: kept in scalar
// registers across the steps, others would be spilled.)
__device__ __forceinline__ bool wait_over(cargs_t& args, int64_t turn, bool pass) {
    if ((turn & 63) != 63) return false;
    uint64_t p = reinterpret_cast<uint64_t>(&args);
    asm volatile("" : "+s"(p));
    cargs_t& a = *reinterpret_cast<cargs_t*>(p);
    if (turn >= (pass ? a.pass_turns : a.step_turns)) {
        st_c(&a.st->error, 1);
        return true;
    }
    return uni(ld_c(&a.st->error)) != 0;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {   // zero where no lane is the source
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {   // in every lane
    v = max(v, dpp_u<0x111, 0xf>(v));   // row_shr:1
    v = max(v, dpp_u<0x112, 0xf>(v));
    v = max(v, dpp_u<0x114, 0xf>(v));
    v = max(v, dpp_u<0x118, 0xf>(v));
    v = max(v, dpp_u<0x142, 0xa>(v));   // row_bcast:15
    v = max(v, dpp_u<0x143, 0xc>(v));   // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 63);
}
// fmax would first quiet its operands, a second instruction for each
__device__ __forceinline__ double max64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double swap_max32(double a, double b) {   // low lanes: max of a's halves, high lanes: of b's
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return max64(__hiloint2double(h[0], l[0]), __hiloint2double(h[1], l[1]));
}
__device__ __forceinline__ double swap_max16(double a, double b) {   // even rows: max of a's row pair, odd rows: of b's
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    return max64(__hiloint2double(h[0], l[0]), __hiloint2double(h[1], l[1]));
}
// Merges the partial maxima of the lanes that scanned the same four columns
// (lanes equal modulo 16) and spreads the columns over them: row r of 16 lanes
// ends with column 4 (lane mod 16) + r.
__device__ __forceinline__ double merge_group(const double (&b)[4]) {
    return swap_max16(swap_max32(b[0], b[2]), swap_max32(b[1], b[3]));
}

}  // namespace fv
