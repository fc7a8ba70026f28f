// Device helpers shared by the HIP kernels of libscocg (not part of the C ABI).
#pragma once
#include "scocg_internal.h"

// No implicit contraction: every fused multiply-add is written out, so the arithmetic
// (and its rounding) is the same in every template instance.
#pragma clang fp contract(off)

namespace scocg {

static constexpr int WG = 256;

// a * b + c with explicit fused multiply-adds
__device__ inline double2 cfma(double2 a, double2 b, double2 c)
{
    return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ inline float2 cfma(float2 a, float2 b, float2 c)
{
    return make_float2(fmaf(a.x, b.x, fmaf(-a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(a.y, b.x, c.y)));
}
__device__ inline double rfma(double a, double b, double c) { return fma(a, b, c); }
__device__ inline float rfma(float a, float b, float c) { return fmaf(a, b, c); }

// Complex product, square, quotient and squared modulus with every rounding written out: the
// forms the compiler gives cmul, cdiv and cabs2 (which it may contract) in the seed kernels, so a
// kernel that takes over their work gives the same bits.
__device__ inline double2 cmul_f(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ inline double2 cdiv_f(double2 a, double2 b)
{
    // both cases of cdiv with their operands selected, so one chain of three divisions (the last
    // two independent) stands in one basic block
    const bool c = fabs(b.x) >= fabs(b.y);
    const double lo = c ? b.y : b.x, hi = c ? b.x : b.y;
    const double r = lo / hi, d = fma(lo, r, hi);
    const double p = c ? a.y : a.x, q = c ? a.x : a.y, u = c ? -a.x : a.y, v = c ? a.y : -a.x;
    return make_double2(fma(p, r, q) / d, fma(u, r, v) / d);
}
// r.r (bilinear) and |r|^2 of one row of the residual
__device__ inline double2 csq_f(double2 r)
{
    const double xx = r.x * r.x, xy = r.y * r.x;
    return make_double2(fma(-r.y, r.y, xx), xy + xy);
}
__device__ inline double cabs2_f(double2 r) { return fma(r.y, r.y, r.x * r.x); }

// Lane t receives lane t + S (lanes past the row, half or wave end receive something else):
// register moves instead of a trip through the LDS crossbar.
template <int S>
__device__ inline unsigned lane_down(unsigned x)
{
    static_assert(S == 32 || S == 16 || S == 8 || S == 4 || S == 2 || S == 1, "");
    if constexpr (S == 32) return __builtin_amdgcn_permlane32_swap(x, x, false, false)[1];
    else if constexpr (S == 16) return __builtin_amdgcn_permlane16_swap(x, x, false, false)[1];
    else return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x100 + S, 0xf, 0xf, true);  // row_shl
}
template <int S>
__device__ inline double lane_down(double x)
{
    const unsigned long long v = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = lane_down<S>((unsigned)v), hi = lane_down<S>((unsigned)(v >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double vadd(double a, double b) { return a + b; }
__device__ inline double2 vadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
template <int S>
__device__ inline double2 lane_down(double2 x)
{
    return make_double2(lane_down<S>(x.x), lane_down<S>(x.y));
}
// The narrow levels (those below TOP) of a sum over 64 lanes: the total in lane 0.  The
// additions and their order are those of a tree over LDS.
template <int TOP = 64, typename T>
__device__ inline T lane_tree(T x)
{
    if constexpr (TOP > 32) x = vadd(x, lane_down<32>(x));
    if constexpr (TOP > 16) x = vadd(x, lane_down<16>(x));
    if constexpr (TOP > 8) x = vadd(x, lane_down<8>(x));
    if constexpr (TOP > 4) x = vadd(x, lane_down<4>(x));
    if constexpr (TOP > 2) x = vadd(x, lane_down<2>(x));
    if constexpr (TOP > 1) x = vadd(x, lane_down<1>(x));
    return x;
}
__device__ inline double first_lane(double x)
{
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readfirstlane((int)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline double2 first_lane(double2 x) { return make_double2(first_lane(x.x), first_lane(x.y)); }

__device__ inline double2 keep_if(bool c, double2 v) { return make_double2(c ? v.x : 0.0, c ? v.y : 0.0); }

template <typename V>
__device__ inline V to_v(double2 a);
template <>
__device__ inline double2 to_v<double2>(double2 a) { return a; }
template <>
__device__ inline float2 to_v<float2>(double2 a) { return make_float2((float)a.x, (float)a.y); }

__device__ inline bool seed_running(const SeedState &st, int TB)
{
    return st.status == SEED_RUNNING && st.step < TB;
}

__device__ inline double2 *ring_slot(const SolveDev &s, int slot, const RhsDesc &d)
{
    return s.ring + (int64_t)slot * s.ntot + d.voff;
}

// Seed directions.  With two right-hand sides per SpMV thread (rhs 2i and 2i+1 share one
// matrix, so voff_{2i+1} = voff_{2i} + n) the pair is interleaved element by element from
// voff_{2i} on: one gather of 32 bytes serves both.  Otherwise p_j is the plain vector at voff_j.
__device__ inline int64_t p_index(const SolveDev &s, int64_t j, const RhsDesc &d, int64_t row)
{
    if (s.spmv_rb == 2) return d.voff - (j & 1) * d.n + 2 * row + (j & 1);
    return d.voff + row;
}

// Up-spin configuration of a workgroup of the tiled Hubbard products.  Workgroups go to the 8 XCDs in
// turn; each XCD takes a stretch of consecutive configurations, whose hops between low sites lead
// to configurations a short way off, read by the same L2 (grid: 8 times hub_stretch).
__host__ __device__ inline int64_t hub_stretch(int64_t Du) { return (Du + 7) / 8; }
__device__ inline int64_t hub_block(unsigned b, int64_t Du)
{
    return (int64_t)(b & 7) * hub_stretch(Du) + (b >> 3);
}

// A pointer that is the same in every lane, in scalar registers.
template <typename T>
__device__ inline T *first_lane(T *p)
{
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)v);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32));
    return (T *)(((unsigned long long)hi << 32) | lo);
}

// Matrix arrays reached through a descriptor are global memory; saying so lets the compiler
// use global (not flat) loads, which wait on the vector-memory counter only.
template <typename T>
__device__ inline const __attribute__((address_space(1))) T *gptr(const T *p)
{
    return (const __attribute__((address_space(1))) T *)p;
}

}  // namespace scocg
