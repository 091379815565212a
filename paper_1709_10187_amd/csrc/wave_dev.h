// Wave-level helpers of the cooperative walks, in which a whole wave advances one packet: lane
// reads and writes, and the packet's FP64 clock over a block of steps (one per lane) with the bits
// of adding the steps one after another.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rddmc {

__device__ __forceinline__ uint32_t rl(uint32_t v, int lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

__device__ __forceinline__ uint64_t rl64(uint64_t v, int lane)
{
    return ((uint64_t)rl((uint32_t)(v >> 32), lane) << 32) | rl((uint32_t)v, lane);
}

// v with `s` (wave-uniform) in lane `lane`: the compiler has no builtin for v_writelane_b32, and
// only the intrinsic lets it place the wait states after the instruction that wrote `s`
extern "C" __device__ int amdgcn_writelane_i32(int s, int lane, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ int write_lane(int s, int lane, int v) { return amdgcn_writelane_i32(s, lane, v); }

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double rl_f64(double v, int lane)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)(((uint64_t)rl((uint32_t)(b >> 32), lane) << 32) | rl((uint32_t)b, lane)));
}

// Clock of a block without the sequential chain, where that gives the same bits.  With
// t0 in [2^e, 2^(e+1)), ulp = 2^(e-52), and every partial sum below 2^(e+1), each
// addition t + d (d >= 0) rounds to t + ulp * rint(d / ulp), unless d / ulp lies exactly
// halfway between integers (then the rounding depends on the running sum).  Without such
// a tie the block's result is t0 + ulp * (sum of the rint values): an exact integer sum,
// reduced across the wave in any order.  Returns false (t unchanged) where the premises
// fail; the caller then adds in order.  The first form takes two steps per lane.
__device__ __forceinline__ bool clock_parallel(double &t, double da, double db)
{
    const uint64_t tbits = (uint64_t)__double_as_longlong(t);
    const int be = (int)((tbits >> 52) & 0x7ffu);
    if (be == 0 || be >= 0x7fe) return false;        // zero, subnormal or near the top
    const int e = be - 1023;
    const double qa = ldexp(da, 52 - e), qb = ldexp(db, 52 - e);   // exact: power-of-two scalings
    const bool tie = (qa - floor(qa)) == 0.5 || (qb - floor(qb)) == 0.5;
    if (__any(tie)) return false;
    double s = rint(qa) + rint(qb);                    // integers below 2^53: exact sums
    s += dpp_f64<0xb1>(s);                             // quad_perm [1,0,3,2]
    s += dpp_f64<0x4e>(s);                             // quad_perm [2,3,0,1]
    s += dpp_f64<0x124>(s);                            // row_ror:4
    s += dpp_f64<0x128>(s);                            // row_ror:8
    const double S = (rl_f64(s, 0) + rl_f64(s, 16)) + (rl_f64(s, 32) + rl_f64(s, 48));
    const double tf = t + ldexp(S, e - 52);
    if (!(tf < ldexp(1.0, e + 1))) return false;       // left the binade: add in order
    t = tf;
    return true;
}

__device__ __forceinline__ bool clock_parallel(double &t, double dd) { return clock_parallel(t, dd, 0.0); }

// Clock of a block: t += the FP64 path lengths of lanes 0, 1, ... in order (lanes at or
// beyond `done` hold +0, which leaves t unchanged).
template <int G>
__device__ __forceinline__ void clock_from(double &t, uint32_t dlo, uint32_t dhi, int done)
{
    double v[8];   // read the group's eight values first, then add them in order
#pragma unroll
    for (int u = 0; u < 8; ++u)
        v[u] = __longlong_as_double((long long)(((uint64_t)rl(dhi, 8 * G + u) << 32) | rl(dlo, 8 * G + u)));
#pragma unroll
    for (int u = 0; u < 8; ++u) t += v[u];
    if constexpr (G < 7) {
        if (done > 8 * (G + 1)) clock_from<G + 1>(t, dlo, dhi, done);
    }
}

}  // namespace rddmc
