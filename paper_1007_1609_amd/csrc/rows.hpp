// Device-side pieces of the kernels that hold one vector's lattice rows in the
// lanes of a wavefront: lane shifts, buffer-resource accesses of 16 bytes per
// lane, the doubled stencil and the doubling sums of one site.
#pragma once

#include "stencil.hpp"

namespace cbdg {

namespace {

constexpr unsigned kOut = 0x80000000u;     // a byte offset past every buffer range
constexpr int kRsrcWord3 = 0x00020000;     // gfx9 buffer descriptor: 32-bit data format

// DPP controls of the whole-wavefront shifts by one lane
constexpr int kShl1 = 0x130;  // lane i <- lane i+1 (lane 63 <- 0)
constexpr int kRol1 = 0x134;  // lane i <- lane i+1 (lane 63 <- lane 0)
constexpr int kShr1 = 0x138;  // lane i <- lane i-1 (lane 0 <- 0)
constexpr int kRor1 = 0x13C;  // lane i <- lane i-1 (lane 0 <- lane 63)

template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL, typename T>
__device__ __forceinline__ Pair<T, false> dpp_pair(const Pair<T, false> &p)
{
    return Pair<T, false>{dpp<CTRL>(p.e), dpp<CTRL>(p.h)};
}

typedef unsigned U4 __attribute__((ext_vector_type(4)));
typedef unsigned U2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t vec_rsrc(const void *base, int64_t b, int64_t Dv)
{
    const char *p = reinterpret_cast<const char *>(base) + b * Dv * (int64_t)(2 * sizeof(T));
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, (int)(Dv * 2 * sizeof(T)), kRsrcWord3);
}

// Every access moves 16 bytes per lane: one FP64 pair or two FP32 pairs
// (kPer pairs).  Inside a row, chunk j of lane l (its pairs k = j*kPer ..
// j*kPer + kPer - 1) sits at (j*64 + l)*kPer, so the j-th chunks of all lanes
// are one contiguous 1 KB block.
template <typename T> constexpr int kPer = 16 / (2 * (int)sizeof(T));
template <typename T> __host__ __device__ constexpr int pair_pos(int lane, int k)
{
    return ((k / kPer<T>) * kWave + lane) * kPer<T> + k % kPer<T>;
}

// Cache policy of the vector streams: nontemporal (2) for FP64, where each
// row of a vector is read or written once per pass and the streams stay out
// of the caches' way (FP64, 256x256, one 1024-vector tile: 107.2 -> 99.3 ms);
// FP32 runs faster with ordinary accesses (136.2 ms against 160.9).
#ifndef CBDG_VC_NT_F64
#define CBDG_VC_NT_F64 2
#endif
#ifndef CBDG_VC_NT_F32
#define CBDG_VC_NT_F32 0
#endif
template <typename T> constexpr int kAux = sizeof(T) == 8 ? CBDG_VC_NT_F64 : CBDG_VC_NT_F32;

// the chunk of kPer pairs at byte offset off
template <typename T>
__device__ __forceinline__ void bld(__amdgpu_buffer_rsrc_t r, unsigned off, Pair<T, false> *p)
{
    const U4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kAux<T>);
    if constexpr (sizeof(T) == 8) {
        p[0].e = __hiloint2double((int)v[1], (int)v[0]);
        p[0].h = __hiloint2double((int)v[3], (int)v[2]);
    } else {
        p[0].e = __uint_as_float(v[0]); p[0].h = __uint_as_float(v[1]);
        p[1].e = __uint_as_float(v[2]); p[1].h = __uint_as_float(v[3]);
    }
}

template <typename T>
__device__ __forceinline__ void bst(__amdgpu_buffer_rsrc_t r, unsigned off, const Pair<T, false> *p)
{
    U4 v;
    if constexpr (sizeof(T) == 8) {
        v = U4{(unsigned)__double2loint(p[0].e), (unsigned)__double2hiint(p[0].e), (unsigned)__double2loint(p[0].h),
               (unsigned)__double2hiint(p[0].h)};
    } else {
        v = U4{__float_as_uint(p[0].e), __float_as_uint(p[0].h), __float_as_uint(p[1].e), __float_as_uint(p[1].h)};
    }
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, kAux<T>);
}

// Whether the passes of several steps fold the factor 2 of eq. (ref2) into
// their coefficients (2 de, 2 Delta/a and 2 t/a are exact): 2 Ht c - p of a
// component is then three fused multiply-adds after the neighbour sum
// instead of a product, two fused multiply-adds and the combination (FP32,
// 256x256, 16 tiles of 1024 vectors at N = 2048: 1203 -> 1148 ms; FP64 at
// N = 1024 unchanged within the run-to-run spread, 3189 / 3214 ms).
#ifndef CBDG_VC_FOLD
#define CBDG_VC_FOLD 1
#endif
template <typename T> constexpr T kCoefScale = CBDG_VC_FOLD ? T(2) : T(1);

// 2 Ht c - p at one site from the doubled coefficients cf = (2 de, 2 Delta/a)
// and th2 = 2 t/a (the hole diagonal is -2 de)
template <typename T>
__device__ __forceinline__ Pair<T, false> step_site(const typename Storage<T, false>::type &cf, T th2,
                                                     const Pair<T, false> &c, const Pair<T, false> &l,
                                                     const Pair<T, false> &r, const Pair<T, false> &d,
                                                     const Pair<T, false> &u, const Pair<T, false> &p)
{
#pragma clang fp contract(off)
    const T se = (l.e + r.e) + (d.e + u.e), sh = (l.h + r.h) + (d.h + u.h);
    Pair<T, false> y;
    y.e = fma_t(cf.x, c.e, fma_t(cf.y, c.h, fma_t(-th2, se, -p.e)));
    y.h = fma_t(-cf.x, c.h, fma_t(cf.y, c.e, fma_t(th2, sh, -p.h)));
    return y;
}

// <v|v>, <v|c> and B(v, c) of one site added to the partial sums, as two
// fused multiply-adds each (no other contraction: the sums do not depend on
// how the compiler schedules a pass)
__device__ __forceinline__ void dots3(double *acc, double e, double h, double ce, double ch)
{
    acc[0] = __builtin_fma(h, h, __builtin_fma(e, e, acc[0]));
    acc[1] = __builtin_fma(h, ch, __builtin_fma(e, ce, acc[1]));
    acc[2] = __builtin_fma(-h, ce, __builtin_fma(e, ch, acc[2]));
}

}  // namespace

}  // namespace cbdg
