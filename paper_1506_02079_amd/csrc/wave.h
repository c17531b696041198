// Device helpers shared by the multigrid kernels: lane shifts, wave-uniform
// copies and the storage types of a level's arrays.
#pragma once
#include "internal.h"

namespace gdf {

// Over-relaxation factor of the SOR instances of the fused finest pass
// (red-black order, level 0 only)
constexpr double kOmega = 1.2;

// ------------------------------------------------------------------ DPP ---

// lane i receives lane i-1's value (lane 0 receives 0)
__device__ __forceinline__ float wave_shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
// lane i receives lane i+1's value (lane 63 receives 0)
__device__ __forceinline__ float wave_shl1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ double wave_shr1(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x138, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_shl1(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x130, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Values every lane of the wave holds alike, moved into scalar registers (the
// work item and level descriptor are read with vector loads, so the compiler
// cannot tell they are uniform; scalar copies keep the address arithmetic on
// the scalar unit and allow scalar-base loads).
template <typename P> __device__ __forceinline__ P *uniform_ptr(P *p)
{
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return reinterpret_cast<P *>(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double uniform_d(double d)
{
    const unsigned long long v = (unsigned long long)__double_as_longlong(d);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ Item uniform_item(const Item &i)
{
    return Item{uniform(i.lev), uniform(i.x0), uniform(i.y0), uniform(i.y1), uniform(i.pidx)};
}
__device__ __forceinline__ LevelDesc uniform_level(const LevelDesc &d)
{
    LevelDesc r;
    r.u[0] = uniform_ptr(d.u[0]);
    r.u[1] = uniform_ptr(d.u[1]);
    r.b = uniform_ptr(d.b);
    r.ec = uniform_ptr(d.ec);
    r.bc = uniform_ptr(d.bc);
    r.H = uniform(d.H);
    r.W = uniform(d.W);
    r.pitch = uniform(d.pitch);
    r.Hc = uniform(d.Hc);
    r.Wc = uniform(d.Wc);
    r.pitch_c = uniform(d.pitch_c);
    r.sigma = uniform_d(d.sigma);
    r.wxL = uniform_d(d.wxL);
    r.wyL = uniform_d(d.wyL);
    r.bshift = uniform_ptr(d.bshift);
    r.slice = uniform(d.slice);
    r.pad_ = 0;
    r.bshift_fine = uniform_ptr(d.bshift_fine);
    return r;
}

// Storage of a level's arrays: the arithmetic type itself, or bfloat16 (raw
// 16-bit patterns, `unsigned short`) on the coarse levels of an FP32
// hierarchy.  Coarse levels only carry corrections, whose relative accuracy
// (2^-8 here) stays far below the cycle's convergence factor, so the cycle
// converges as with FP32 coarse levels while moving half the bytes there.
// Pair: two adjacent elements as one memory access.
template <typename S> struct Stor;
template <> struct Stor<float> {
    typedef float Pair __attribute__((ext_vector_type(2)));
    __device__ static float lo(Pair p) { return p.x; }
    __device__ static float hi(Pair p) { return p.y; }
    __device__ static float get(float s) { return s; }
    __device__ static float put(float v) { return v; }
    __device__ static Pair pair(float a, float b) { Pair p; p.x = a; p.y = b; return p; }
};
template <> struct Stor<double> {
    typedef double Pair __attribute__((ext_vector_type(2)));
    __device__ static double lo(Pair p) { return p.x; }
    __device__ static double hi(Pair p) { return p.y; }
    __device__ static double get(double s) { return s; }
    __device__ static double put(double v) { return v; }
    __device__ static Pair pair(double a, double b) { Pair p; p.x = a; p.y = b; return p; }
};
template <> struct Stor<unsigned short> {   // bfloat16
    typedef unsigned int Pair;
    typedef __bf16 BF2 __attribute__((ext_vector_type(2)));
    typedef float F2 __attribute__((ext_vector_type(2)));
    __device__ static float lo(Pair p) { return __uint_as_float(p << 16); }
    __device__ static float hi(Pair p) { return __uint_as_float(p & 0xFFFF0000u); }
    __device__ static float get(unsigned short s) { return __uint_as_float((unsigned)s << 16); }
    // round to nearest even (the hardware conversion)
    __device__ static unsigned short put(float v) { return __builtin_bit_cast(unsigned short, (__bf16)v); }
    __device__ static Pair pair(float a, float b)
    {
        F2 f;
        f.x = a;
        f.y = b;
        return __builtin_bit_cast(Pair, __builtin_convertvector(f, BF2));
    }
};

template <> struct Buf<Stor<float>::Pair> : BufBits<Stor<float>::Pair, U2> {};
template <> struct Buf<Stor<double>::Pair> : BufBits<Stor<double>::Pair, U4> {};

// storage of a level-0 pass (own arrays, coarse arrays) and of a coarse pass
template <typename T> struct LevelStor { typedef T Fine; typedef T Coarse; };
template <> struct LevelStor<float> { typedef float Fine; typedef unsigned short Coarse; };

}  // namespace gdf
