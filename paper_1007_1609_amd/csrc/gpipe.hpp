// The row pipeline of vpipe.hpp for the other operators: complex order
// parameters, per-bond hopping and pairing, and the direct recursion that
// reads neighbour moments.
//
// One workgroup of S wavefronts takes one vector at a time through all its
// passes of L = S*K steps; stage s takes K steps, its lanes own W neighbouring
// columns, rows go from stage to stage through LDS (see vpipe.hpp for the
// trips, windows and row hand-over, which are the same).  A site's record
// holds the on-site block and, for per-bond operators, its four links, so a
// stage needs no other site's coefficients; columns past the row's end have
// zero records.  Rows outside the pass are skipped and set to zero.
//
// What bounds it: per-bond complex128 takes 96 operations per site and step
// beside its sums, against 96 bytes of vectors in the one-step passes, which
// stream at 5 TB/s; with L steps per crossing HBM is at 0.9 TB/s (48x40 neighbour
// moments), the vector units are busy 45 % of the time, and the rest waits for the
// records (160 bytes a site, from L2 into registers on every trip) and the barrier.
//
// The workgroups are persistent (vector b, then b + gridDim.x, ..): each owns
// its buffers in the workspace, which hold the vectors of the workgroups in
// flight instead of a whole tile and leave room for the records.
#pragma once

#include "vpipe.hpp"

namespace cbdg {

struct GPipeArgs {
    PipeArgs P;      // coef: the records; Dv, rowp in pairs
    int recs;        // T values per row of records
    double *nb_ee, *nb_he;  // neighbour moments (direct recursion) or null: doubling
};

__device__ __forceinline__ void global_pointers(GPipeArgs &G)
{
    global_pointers(G.P);
    G.nb_ee = as_global(G.nb_ee);
    G.nb_he = as_global(G.nb_he);
}

// Values of a site's record: {de, dh, Re Delta, Im Delta}, then the links
// +x, -x, +y, -y ({t, d}, complex ones as (re, im)).
template <bool CP, bool GEN> constexpr int kRec = GEN ? (CP ? 20 : 12) : 4;

namespace {

template <typename T, bool CP>
__device__ __forceinline__ Pair<T, CP> pair_at(const T *r, int k)
{
    Pair<T, CP> p;
    if constexpr (CP) { p.er = r[4 * k]; p.ei = r[4 * k + 1]; p.hr = r[4 * k + 2]; p.hi = r[4 * k + 3]; }
    else { p.e = r[2 * k]; p.h = r[2 * k + 1]; }
    return p;
}
template <typename T, bool CP>
__device__ __forceinline__ void put_pair(T *r, int k, const Pair<T, CP> &p)
{
    if constexpr (CP) { r[4 * k] = p.er; r[4 * k + 1] = p.ei; r[4 * k + 2] = p.hr; r[4 * k + 3] = p.hi; }
    else { r[2 * k] = p.e; r[2 * k + 1] = p.h; }
}
template <int CTRL, typename T, bool CP>
__device__ __forceinline__ Pair<T, CP> shift_pair(const Pair<T, CP> &p)
{
    if constexpr (CP) return Pair<T, true>{dpp<CTRL>(p.er), dpp<CTRL>(p.ei), dpp<CTRL>(p.hr), dpp<CTRL>(p.hi)};
    else return Pair<T, false>{dpp<CTRL>(p.e), dpp<CTRL>(p.h)};
}
template <typename T, bool CP>
__device__ __forceinline__ Pair<T, CP> lane_pair(const Pair<T, CP> &p, int lane)
{
    if constexpr (CP)
        return Pair<T, true>{lane_value(p.er, lane), lane_value(p.ei, lane), lane_value(p.hr, lane), lane_value(p.hi, lane)};
    else return Pair<T, false>{lane_value(p.e, lane), lane_value(p.h, lane)};
}
template <typename T>
__device__ __forceinline__ void unpack_row(const U4 &v, T *r)
{
    if constexpr (sizeof(T) == 8) {
        r[0] = __hiloint2double((int)v[1], (int)v[0]);
        r[1] = __hiloint2double((int)v[3], (int)v[2]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = __uint_as_float(v[i]);
    }
}
template <typename T>
__device__ __forceinline__ U4 pack_row(const T *r)
{
    if constexpr (sizeof(T) == 8)
        return U4{(unsigned)__double2loint(r[0]), (unsigned)__double2hiint(r[0]), (unsigned)__double2loint(r[1]),
                  (unsigned)__double2hiint(r[1])};
    else
        return U4{__float_as_uint(r[0]), __float_as_uint(r[1]), __float_as_uint(r[2]), __float_as_uint(r[3])};
}

// Neighbour d (+x, -x, +y, -y) of (x, y), or -1.
__device__ __forceinline__ int step_site_index(int x, int y, int d, int Lx, int Ly, int bcx, int bcy)
{
    if (d == 0) { if (++x == Lx) { if (!bcx) return -1; x = 0; } }
    else if (d == 1) { if (--x < 0) { if (!bcx) return -1; x = Lx - 1; } }
    else if (d == 2) { if (++y == Ly) { if (!bcy) return -1; y = 0; } }
    else { if (--y < 0) { if (!bcy) return -1; y = Ly - 1; } }
    return x + Lx * y;
}

// FP64 records of per-bond operators hold twice the coefficients (exact), so
// that the chains below add up to 2 Ht c: 96 operations a site for complex
// operators, a_{n-2} taken off included, 106 in the one-step kernels' form,
// which FP32 keeps (its vectors would differ in the seventh digit).  Uniform
// operators take apply_uniform in both types.
template <typename T, bool GEN> constexpr T kRecScale = GEN && sizeof(T) == 8 ? T(2) : T(1);

// 2 Ht c - p from a doubled per-bond record (FP64).  Every rounding of a sum has
// its magnitude: a neighbour's terms make a chain of their own, and p comes off
// last (rms error of neighbour moments against 80-bit vectors, 48x40, N = 256:
// 1.9e-17 so and in the one-step kernels, 2.3e-17 with one chain through all
// neighbours, 78 operations, 4.5e-17 with that chain begun with -p).
template <bool CP>
__device__ __forceinline__ Pair<double, CP> bond_site_f64(const double *r, const Pair<double, CP> &c,
                                                          const Pair<double, CP> *nb, const Pair<double, CP> &p)
{
#pragma clang fp contract(off)
    if constexpr (CP) {
        double er = fma_t(r[0], c.er, fma_t(r[2], c.hr, -(r[3] * c.hi)));
        double ei = fma_t(r[0], c.ei, fma_t(r[2], c.hi, r[3] * c.hr));
        double hr = fma_t(r[1], c.hr, fma_t(r[2], c.er, r[3] * c.ei));
        double hi = fma_t(r[1], c.hi, fma_t(r[2], c.ei, -(r[3] * c.er)));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const Pair<double, true> &a = nb[q];
            const double tr = r[4 + 4 * q], ti = r[5 + 4 * q], dr = r[6 + 4 * q], di = r[7 + 4 * q];
            er += fma_t(-tr, a.er, fma_t(ti, a.ei, fma_t(dr, a.hr, -(di * a.hi))));
            ei += fma_t(-tr, a.ei, fma_t(-ti, a.er, fma_t(dr, a.hi, di * a.hr)));
            hr += fma_t(dr, a.er, fma_t(di, a.ei, fma_t(tr, a.hr, ti * a.hi)));
            hi += fma_t(dr, a.ei, fma_t(-di, a.er, fma_t(tr, a.hi, -(ti * a.hr))));
        }
        return Pair<double, true>{er - p.er, ei - p.ei, hr - p.hr, hi - p.hi};
    } else {
        double e = fma_t(r[0], c.e, r[2] * c.h), h = fma_t(r[2], c.e, r[1] * c.h);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double t = r[4 + 2 * q], dl = r[5 + 2 * q];
            e += fma_t(dl, nb[q].h, -t * nb[q].e);
            h += fma_t(dl, nb[q].e, t * nb[q].h);
        }
        return Pair<double, false>{e - p.e, h - p.h};
    }
}

// Ht c at one site of a per-bond operator in FP32, with the roundings of the
// one-step kernels written out (their compiler fuses one product of each sum
// of two): FP32 vectors do not depend on which kernel advanced them.
template <bool CP>
__device__ __forceinline__ Pair<float, CP> bond_site_f32(const float *r, const Pair<float, CP> &c, const Pair<float, CP> *nb)
{
#pragma clang fp contract(off)
    Pair<float, CP> y;
    if constexpr (CP) {
        float er = fma_t(r[0], c.er, fma_t(r[2], c.hr, -(r[3] * c.hi)));
        float ei = fma_t(r[0], c.ei, fma_t(r[3], c.hr, r[2] * c.hi));
        float hr = fma_t(r[1], c.hr, fma_t(r[2], c.er, r[3] * c.ei));
        float hi = fma_t(r[1], c.hi, fma_t(r[2], c.ei, -(r[3] * c.er)));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const Pair<float, true> &a = nb[q];
            const float tr = r[4 + 4 * q], ti = r[5 + 4 * q], dr = r[6 + 4 * q], di = r[7 + 4 * q];
            er += fma_t(dr, a.hr, -(di * a.hi)) - fma_t(tr, a.er, -(ti * a.ei));
            ei += fma_t(di, a.hr, dr * a.hi) - fma_t(ti, a.er, tr * a.ei);
            hr += fma_t(dr, a.er, di * a.ei) + fma_t(tr, a.hr, ti * a.hi);
            hi += fma_t(dr, a.ei, -(di * a.er)) + fma_t(tr, a.hi, -(ti * a.hr));
        }
        y = Pair<float, true>{er, ei, hr, hi};
    } else {
        float e = fma_t(r[0], c.e, r[2] * c.h), h = fma_t(r[2], c.e, r[1] * c.h);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float t = r[4 + 2 * q], dl = r[5 + 2 * q];
            e += fma_t(dl, nb[q].h, -t * nb[q].e);
            h += fma_t(dl, nb[q].e, t * nb[q].h);
        }
        y = Pair<float, false>{e, h};
    }
    return y;
}

// A complex or real moment, stored as NaN beyond the bound.
__device__ __forceinline__ void put_moment(double *p, int64_t i, double re, double im, bool cplx, double lim)
{
    const double nan = __builtin_nan("");
    if (cplx) {
        const bool ok = re * re + im * im <= lim * lim;
        p[2 * i] = ok ? re : nan;
        p[2 * i + 1] = ok ? im : nan;
    } else {
        p[i] = fabs(re) <= lim ? re : nan;
    }
}

// Doubling moments 2m-1, 2m from the sums of step m (k_doubling_reduce).
template <bool CP>
__device__ __forceinline__ void gpipe_moments(const PipeArgs &A, int64_t mrow, int m, const double *s, double e1, double h1r,
                                              double h1i)
{
    if (m < 2) return;
    const double nan = __builtin_nan(""), sgn = (m & 1) ? -2.0 : 2.0;
    if (2 * m < A.N) {
        const double v = 2.0 * s[0] - 1.0;
        A.mu_ee[mrow + 2 * m] = fabs(v) <= A.lim ? v : nan;
        put_moment(A.mu_he, mrow + 2 * m, 0.0, 0.0, CP, A.lim);
    }
    if (2 * m - 1 < A.N) {
        const double v = 2.0 * s[1] - e1;
        A.mu_ee[mrow + 2 * m - 1] = fabs(v) <= A.lim ? v : nan;
        put_moment(A.mu_he, mrow + 2 * m - 1, sgn * s[2] - h1r, CP ? sgn * s[3] - h1i : 0.0, CP, A.lim);
    }
}

}  // namespace

template <typename T, bool CP, bool GEN> struct GPipeShape1 {
    // registers of a row and of its records, per owned column
    static constexpr int row = (CP ? 4 : 2) * (int)sizeof(T) / 4, rec = kRec<CP, GEN> * (int)sizeof(T) / 4;
};
// Steps a stage takes: as many as the windows (two rows a step, four more in
// work) and the records of its rows leave room for in 256 registers.
template <typename T, bool CP, bool GEN, int W> struct GPipeShape {
    static constexpr int row = W * GPipeShape1<T, CP, GEN>::row, rec = W * GPipeShape1<T, CP, GEN>::rec;
    static constexpr int regs(int k) { return 2 * k * row + 4 * row + k * rec + 8 * k; }
    static constexpr int K = regs(5) <= 160 ? 5 : regs(3) <= 180 ? 3 : regs(2) <= 215 ? 2 : 1;
    static constexpr int S = 4;
};

// PER: some direction is periodic.
template <typename T, bool CP, bool GEN, int W, int K, int S, bool PER>
__global__ __launch_bounds__(S * kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_gpipe(GPipeArgs G)
{
    using Q = Pair<T, CP>;
    constexpr int L = K * S, NC = CP ? 4 : 2;
    constexpr int NQ = (W * NC * (int)sizeof(T) + 15) / 16, NVP = NQ * 16 / (int)sizeof(T);
    constexpr int REC = kRec<CP, GEN>, CQ = (W * REC * (int)sizeof(T) + 15) / 16, CVP = CQ * 16 / (int)sizeof(T);
    constexpr int NF = (NQ + S / 2 - 1) / (S / 2);
    constexpr int U = 3, RC = K + kCoefAhead<K> - 1, XC = kCoefAhead<K>, UL = kRound<K>;
    constexpr int ND = CP ? 4 : 3;
    __shared__ U4 hand[S][2][2][NQ][kWave];
    __shared__ double sums[S][ND * K], first1[3];  // first1: mu_ee[1], mu_he[1]
    const PipeArgs &A = G.P;

    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int Lx = A.Lx, Ly = A.Ly, nl = A.nl;
    const bool bcx = PER && A.bcx != 0, bcy = PER && A.bcy != 0, direct = G.nb_ee != nullptr;
    const int lr = (Lx - 1) / W, kr = (Lx - 1) % W;
    const T th = T(A.th);
    const T *recs = reinterpret_cast<const T *>(A.coef);
    const unsigned cstep = (unsigned)nl * 16u;
    const int vbytes = (int)(A.Dv * (int64_t)(NC * sizeof(T)));
    const auto rrec = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(A.coef), (short)0,
                                                        (int)((int64_t)G.recs * Ly * (int64_t)sizeof(T)), kRsrcWord3);

    for (int b = blockIdx.x; b < A.Bt; b += gridDim.x) {
        const int si = __builtin_amdgcn_readfirstlane(A.sites[b]);
        if (si < 0 || si >= Lx * Ly) {
            const GPipeArgs B = cold_args<GPipeArgs>();
            const int64_t mrow = (int64_t)b * B.P.N;
            const double nan = __builtin_nan("");
            for (int n = threadIdx.x; n < B.P.N; n += S * kWave) {
                B.P.mu_ee[mrow + n] = nan;
                for (int c = 0; c < (CP ? 2 : 1); ++c) B.P.mu_he[(CP ? 2 : 1) * (mrow + n) + c] = nan;
            }
            if (direct)
                for (int64_t n = threadIdx.x; n < (int64_t)B.P.N * (CP ? 8 : 4); n += S * kWave) {
                    B.nb_ee[4 * mrow * (CP ? 2 : 1) + n] = nan;
                    B.nb_he[4 * mrow * (CP ? 2 : 1) + n] = nan;
                }
            continue;
        }
        const int yi = si / Lx, xi = si - yi * Lx;
        // this workgroup's buffers (pairs as in vpipe.hpp)
        const uint64_t vbase = reinterpret_cast<uint64_t>(A.buf) + (uint64_t)blockIdx.x * (uint64_t)vbytes, one = (uint64_t)A.one;
        const int flip = A.flip;
        auto vec_of = [&](int pass, int newer) -> __amdgpu_buffer_rsrc_t {
            const uint64_t at = vbase + (pass & flip ? 2 * one : 0) + (newer ? one : 0);
            return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char *>(at), (short)0, vbytes, kRsrcWord3);
        };
        // value i of site (x, y)'s record
        auto rec_at = [&](int x, int y, int i) -> T {
            const int e = x % W * REC + i;
            constexpr int per = 16 / (int)sizeof(T);
            return recs[(int64_t)y * G.recs + ((int64_t)(e / per) * nl + x / W) * per + e % per] * (T(1) / kRecScale<T, GEN>);
        };
        // a_0, a_1 and the moments that need no recursion
        __syncthreads();  // the last vector's rows are read no more
        {
            const GPipeArgs B = cold_args<GPipeArgs>();
            const PipeArgs &C = B.P;
            const int64_t mrow = (int64_t)b * C.N;
            const double lim = C.lim;
            T *v0 = reinterpret_cast<T *>(vbase), *v1 = reinterpret_cast<T *>(vbase + one);
            const int64_t rowv = (int64_t)nl * NVP;
            int nbs[4];
            for (int d = 0; d < 4; ++d) nbs[d] = step_site_index(xi, yi, d, Lx, Ly, bcx, bcy);
            constexpr int per = 16 / (int)sizeof(T);
            // component c of H|s,e> at the site, or at neighbour d (its link back, d ^ 1)
            auto h_at = [&](int d, int c) -> T {
                if (d < 0) {
                    if constexpr (CP) return c == 0 ? rec_at(xi, yi, 0) : c == 1 ? T(0) : c == 2 ? rec_at(xi, yi, 2) : -rec_at(xi, yi, 3);
                    else return rec_at(xi, yi, c == 0 ? 0 : 2);
                }
                if constexpr (!GEN) return c == 0 ? -th : T(0);
                const int x = nbs[d] % Lx, y = nbs[d] / Lx, i = 4 + (d ^ 1) * (CP ? 4 : 2);
                if constexpr (CP) {
                    const T v = rec_at(x, y, i + c);
                    return c == 2 ? v : -v;
                } else {
                    return c == 0 ? -rec_at(x, y, i) : rec_at(x, y, i + 1);
                }
            };
            for (int64_t i = threadIdx.x; i < 3 * rowv; i += S * kWave) {
                const int q = (int)(i / rowv);
                const int pos = (int)(i - q * rowv);
                const int y = q == 0 ? yi : nbs[q == 1 ? 2 : 3] < 0 ? -1 : nbs[q == 1 ? 2 : 3] / Lx;
                if (y < 0) continue;
                const int ch = pos / per, e = ch / nl * per + pos % per;
                const int x = ch % nl * W + e / NC, c = e % NC;
                const bool mine = e < W * NC;
                T a1 = T(0);
                if (mine) {
                    if (q == 0) {
                        if (x == xi) a1 = h_at(-1, c);
                        else if (nbs[0] >= 0 && x == nbs[0] % Lx) a1 = h_at(0, c);
                        else if (nbs[1] >= 0 && x == nbs[1] % Lx) a1 = h_at(1, c);
                        v0[(int64_t)y * rowv + pos] = x == xi && c == 0 ? T(1) : T(0);
                    } else if (x == xi) {
                        a1 = h_at(q + 1, c);
                    }
                } else if (q == 0) {
                    v0[(int64_t)y * rowv + pos] = T(0);
                }
                v1[(int64_t)y * rowv + pos] = a1;
            }
            if (threadIdx.x == 0) {
                C.mu_ee[mrow] = 1.0;
                put_moment(C.mu_he, mrow, 0.0, 0.0, CP, lim);
                double nrm = 0.0;
                for (int d = -1; d < 4; ++d) {
                    if (d >= 0 && nbs[d] < 0) continue;
                    for (int c = 0; c < NC; ++c) { const double v = (double)h_at(d, c); nrm += v * v; }
                }
                if (C.N > 1) {
                    put_moment(C.mu_ee, mrow + 1, (double)h_at(-1, 0), 0.0, false, lim);
                    put_moment(C.mu_he, mrow + 1, (double)h_at(-1, CP ? 2 : 1), CP ? (double)h_at(-1, 3) : 0.0, CP, lim);
                }
                if (!direct && C.N > 2) {
                    put_moment(C.mu_ee, mrow + 2, 2.0 * nrm - 1.0, 0.0, false, lim);
                    put_moment(C.mu_he, mrow + 2, 0.0, 0.0, CP, lim);
                }
            }
            if (direct) {
                for (int d = 0; d < 4; ++d) {
                    const int64_t at = 4 * mrow + (int64_t)d * C.N;
                    for (int n = threadIdx.x; n < (nbs[d] < 0 ? C.N : 1); n += S * kWave) {
                        put_moment(B.nb_ee, at + n, 0.0, 0.0, CP, lim);
                        put_moment(B.nb_he, at + n, 0.0, 0.0, CP, lim);
                    }
                    if (threadIdx.x == 0 && nbs[d] >= 0 && C.N > 1) {
                        put_moment(B.nb_ee, at + 1, (double)h_at(d, 0), CP ? (double)h_at(d, 1) : 0.0, CP, lim);
                        put_moment(B.nb_he, at + 1, (double)h_at(d, CP ? 2 : 1), CP ? (double)h_at(d, 3) : 0.0, CP, lim);
                    }
                }
            }
        }
        if (threadIdx.x == 0) {
            first1[0] = (double)rec_at(xi, yi, 0);
            first1[1] = (double)rec_at(xi, yi, 2);
            first1[2] = CP ? -(double)rec_at(xi, yi, 3) : 0.0;
        }
        for (int i = threadIdx.x; i < S * 2 * 2 * NQ * kWave; i += S * kWave) (&hand[0][0][0][0][0])[i] = U4{0, 0, 0, 0};
        __syncthreads();

        auto offset = [&](int v, int R) -> unsigned {
            const int ph = lattice_row(v, Ly, bcy), rr = R - row_dist(ph, yi, Ly, bcy);
            const unsigned at = (unsigned)((ph * NQ * nl + lane) * 16);
            bool ok = (lane < nl) & (rr >= 0) & (bcy | ((unsigned)v < (unsigned)Ly));
            ok = ok & (bcx | ((lane * W <= xi + rr) & (lane * W + W - 1 >= xi - rr)));
            const unsigned keep = 0u - (unsigned)ok;
            return (at & keep) | (kOut & ~keep);
        };
        auto rec_row = [&](int v, U4 *c) __attribute__((always_inline)) {
            const int ph = bcy ? lattice_row(v, Ly, true) : min(max(v, 0), Ly - 1);
            // lanes past the row get zeros: their columns stay zero
            const unsigned at = lane < nl ? (unsigned)((ph * CQ * nl + lane) * 16) : kOut;
#pragma unroll
            for (int j = 0; j < CQ; ++j) c[j] = __builtin_amdgcn_raw_buffer_load_b128(rrec, at + j * cstep, 0, 0);
        };

        const int fk = wv >= S / 2 ? 1 : 0, fw = wv - fk * (S / 2);
        int fp = 0, ft = -XC;
        PipeJob F = pipe_job<K, S, PER>(A, 0, yi, 0);
        U4 fd[U][NF];
        auto feed_load = [&](U4 *d) __attribute__((always_inline)) {
            const int c = ft + 1 - fk;
            const unsigned off = (unsigned)c < (unsigned)F.R ? offset(F.e0 + c, F.n - 1 - fk) : kOut;
            const auto rs = vec_of(fp, 1 - fk);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int j = fw + f * (S / 2);
                d[f] = __builtin_amdgcn_raw_buffer_load_b128(rs, j < NQ ? off + j * cstep : kOut, 0, 0);
            }
            if (++ft == F.P - XC) { ft = -XC; ++fp; F = pipe_job<K, S, PER>(A, fp, yi, 0); }
        };
        auto feed_store = [&](const U4 *d, int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int j = fw + f * (S / 2);
                if (j < NQ) hand[0][slot][fk][j][lane] = d[f];
            }
        };
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int f = 0; f < NF; ++f) fd[u][f] = U4{0, 0, 0, 0};

        int jp = 0, jt = -XC - kPipeAhead - wv * (K + 1);
        PipeJob J = F;
        int total = kPipeAhead + (S - 1) * (K + 1) + 2 * UL;
        for (int p = 0; p < A.n_pass; ++p) total += pipe_job<K, S, PER>(A, p, yi, 0).P;

        T in[3][NVP], lv[K > 1 ? K - 1 : 1][3][NVP];
        U4 cf[RC][CQ];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < NVP; ++k) {
                in[i][k] = T(0);
#pragma unroll
                for (int j = 0; j < K - 1; ++j) lv[j][i][k] = T(0);
            }
#pragma unroll
        for (int j = 0; j < RC; ++j)
#pragma unroll
            for (int q = 0; q < CQ; ++q) cf[j][q] = U4{0, 0, 0, 0};
        double d[ND * K];
#pragma unroll
        for (int i = 0; i < ND * K; ++i) d[i] = 0.0;

        // the moments of step n that row ph of a_n holds (direct recursion): the
        // start site's and its neighbours', written by the lanes that own them
        auto capture = [&](int ph, int n, const T *v) __attribute__((always_inline)) {
            const GPipeArgs B = cold_args<GPipeArgs>();
            const double lim = B.P.lim;
            const int64_t mrow = (int64_t)b * B.P.N;
            if (n >= B.P.N) return;
            const int above = yi + 1 < Ly ? yi + 1 : bcy ? 0 : -1;  // -1: no row
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int x = lane * W + k;
                int dx = x - xi;
                if (bcx) dx = dx == Lx - 1 ? -1 : dx == 1 - Lx ? 1 : dx;
                // place -1: the start site; 0 .. 3: its neighbour +x, -x, +y, -y
                const int t = ph == yi ? (dx == 0 ? -1 : dx == 1 ? 0 : dx == -1 ? 1 : -2) : dx == 0 ? (ph == above ? 2 : 3) : -2;
                if (t == -2 || x >= Lx) continue;
                const Q p = pair_at<T, CP>(v, k);
                double er, ei = 0.0, hr, hi = 0.0;
                if constexpr (CP) { er = p.er; ei = p.ei; hr = p.hr; hi = p.hi; }
                else { er = p.e; hr = p.h; }
                if (t < 0) {
                    put_moment(B.P.mu_ee, mrow + n, er, 0.0, false, lim);
                    put_moment(B.P.mu_he, mrow + n, hr, hi, CP, lim);
                } else {
                    const int64_t at = 4 * mrow + (int64_t)t * B.P.N + n;
                    put_moment(B.nb_ee, at, er, ei, CP, lim);
                    put_moment(B.nb_he, at, hr, hi, CP, lim);
                }
            }
        };

        auto trip = [&](auto place, int par, auto last) __attribute__((always_inline)) {
            constexpr int u = decltype(place)::value;
            constexpr int sa = u % 3, sb = (u + 1) % 3, sc = (u + 2) % 3;
            feed_store(fd[(u + 1) % U], par ^ 1);
            feed_load(fd[u % U]);
            T pr[NVP];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                unpack_row<T>(hand[wv][par][0][q][lane], in[sc] + q * (16 / (int)sizeof(T)));
                unpack_row<T>(hand[wv][par][1][q][lane], pr + q * (16 / (int)sizeof(T)));
            }
            T out[NVP];
#pragma unroll
            for (int i = 0; i < NVP; ++i) out[i] = T(0);
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const T *cc = j == 0 ? in[sb] : lv[j > 0 ? j - 1 : 0][sb];
                const T *dd = j == 0 ? in[sa] : lv[j > 0 ? j - 1 : 0][sa];
                const T *uu = j == 0 ? in[sc] : lv[j > 0 ? j - 1 : 0][sc];
                const T *pp = j == 0 ? pr : (j == 1 ? in[sa] : lv[j > 1 ? j - 2 : 0][sa]);
                T *v = j == K - 1 ? out : lv[j < K - 1 ? j : 0][sc];
                if ((unsigned)(jt - j) < (unsigned)J.R) {
                    T rc[CVP];
#pragma unroll
                    for (int q = 0; q < CQ; ++q) unpack_row<T>(cf[(u + RC - j) % RC][q], rc + q * (16 / (int)sizeof(T)));
                    const Q c0 = pair_at<T, CP>(cc, 0), cl = pair_at<T, CP>(cc, W - 1);
                    Q hl = shift_pair<kShr1, T, CP>(cl), hr = shift_pair<kShl1, T, CP>(c0), first = zero_pair<T, CP>();
                    if (bcx) {
                        first = lane_pair<T, CP>(c0, 0);
                        Q end = c0;
#pragma unroll
                        for (int k = 1; k < W; ++k) end = select_pair<T, CP>(k == kr, pair_at<T, CP>(cc, k), end);
                        end = lane_pair<T, CP>(end, lr);
                        hl = select_pair<T, CP>(lane == 0, end, hl);
                    }
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        const T *o4 = rc + k * REC;
                        const Q c = pair_at<T, CP>(cc, k), lo = k > 0 ? pair_at<T, CP>(cc, k > 0 ? k - 1 : 0) : hl;
                        Q hi = k < W - 1 ? pair_at<T, CP>(cc, k < W - 1 ? k + 1 : 0) : hr;
                        if (bcx) hi = select_pair<T, CP>(lane == lr && k == kr, first, hi);
                        const Q dn = pair_at<T, CP>(dd, k), up = pair_at<T, CP>(uu, k);
                        const T ths = lane * W + k < Lx ? th : T(0);
                        const Q nb[4] = {hi, lo, up, dn};
                        Q y;
                        if constexpr (GEN && sizeof(T) == 8) {
                            put_pair<T, CP>(v, k, bond_site_f64<CP>(o4, c, nb, pair_at<T, CP>(pp, k)));
                            continue;
                        } else if constexpr (GEN) {
                            y = bond_site_f32<CP>(o4, c, nb);
                        } else {
                            y = apply_uniform<T, CP>(OnSite<T>{o4[0], o4[1], o4[2], o4[3]}, ths, c, lo, hi, dn, up);
                        }
                        const Q w = cheb_combine<T, CP>(y, pair_at<T, CP>(pp, k), false);
                        put_pair<T, CP>(v, k, w);
                    }
                    const int s = J.e0 + jt - j;
                    if (s >= J.y0 && s < J.y1) {
                        if (direct) {
                            const int ph = lattice_row(s, Ly, bcy);
                            if (row_dist(ph, yi, Ly, bcy) <= 1) capture(ph, J.n + wv * K + j, v);
                        } else {
                            double t[ND];
#pragma unroll
                            for (int i = 0; i < ND; ++i) t[i] = 0.0;
#pragma unroll
                            for (int k = 0; k < W; ++k) {
                                const Q w = pair_at<T, CP>(v, k), c = pair_at<T, CP>(cc, k);
                                if constexpr (CP) {
                                    const double er = w.er, ei = w.ei, hr2 = w.hr, hi2 = w.hi;
                                    const double cer = c.er, cei = c.ei, chr = c.hr, chi = c.hi;
                                    t[0] += (er * er + ei * ei) + (hr2 * hr2 + hi2 * hi2);
                                    t[1] += (er * cer + ei * cei) + (hr2 * chr + hi2 * chi);
                                    t[2] += (er * chr - ei * chi) - (hr2 * cer - hi2 * cei);
                                    t[3] += (er * chi + ei * chr) - (hr2 * cei + hi2 * cer);
                                } else {
                                    const double e = w.e, h = w.h, ce = c.e, ch = c.h;
                                    t[0] += e * e + h * h;
                                    t[1] += e * ce + h * ch;
                                    t[2] += e * ch - h * ce;
                                }
                            }
#pragma unroll
                            for (int i = 0; i < ND; ++i) d[ND * j + i] += t[i];
                        }
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < NVP; ++i) v[i] = T(0);
                }
#pragma unroll
                for (int i = 0; i < ND; ++i) asm volatile("" : "+v"(d[ND * j + i]));
                if (j == K - 1) rec_row(J.e0 + jt + XC, cf[(u + XC) % RC]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const T *old = K == 1 ? in[sa] : lv[K > 1 ? K - 2 : 0][sa];
            if constexpr (!decltype(last)::value) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    hand[wv + 1][par ^ 1][0][q][lane] = pack_row<T>(out + q * (16 / (int)sizeof(T)));
                    hand[wv + 1][par ^ 1][1][q][lane] = pack_row<T>(old + q * (16 / (int)sizeof(T)));
                }
            } else {
                const int s1 = J.e0 + jt - (K - 1), s2 = J.e0 + jt - K;
                const bool l1 = (unsigned)(jt - (K - 1)) < (unsigned)J.R && s1 >= J.y0 && s1 < J.y1;
                const bool l2 = (unsigned)(jt - K) < (unsigned)J.R && s2 >= J.y0 && s2 < J.y1;
                const unsigned o1 = l1 ? offset(s1, J.n + L - 1) : kOut, o2 = l2 ? offset(s2, J.n + L - 2) : kOut;
                const auto r1 = vec_of(jp + 1, 1), r2 = vec_of(jp + 1, 0);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    __builtin_amdgcn_raw_buffer_store_b128(pack_row<T>(out + q * (16 / (int)sizeof(T))), r1, o1 + q * cstep, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(pack_row<T>(old + q * (16 / (int)sizeof(T))), r2, o2 + q * cstep, 0, 0);
                }
            }
            ++jt;
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
        };
        const int rounds = (total + UL - 1) / UL;
        auto stage = [&](auto last) __attribute__((always_inline)) {
            int par = 0, done = 0;
#pragma unroll 1
            for (int r = 0; r < rounds; ++r) {
                repeat<UL>([&](auto u) __attribute__((always_inline)) {
                    trip(u, par, last);
                    par ^= 1;
                });
                if (done) {
                    if (lane < K) {
                        const PipeArgs B = cold_args<GPipeArgs>().P;
                        gpipe_moments<CP>(B, (int64_t)b * B.N, done + lane, &sums[wv][ND * lane], first1[0], first1[1], first1[2]);
                    }
                    done = 0;
                }
                if (jt < J.R + K + 1) continue;
                if (!direct) {
#pragma unroll
                    for (int i = 0; i < ND * K; ++i) {
                        const double v = lane_sum(d[i]);
                        if (lane == kWave - 1) sums[wv][i] = v;
                        d[i] = 0.0;
                    }
                    done = jp < A.n_pass ? J.n + wv * K : 0;
                }
                jt -= J.P;
                ++jp;
                J = pipe_job<K, S, PER>(A, jp, yi, 0);
            }
        };
        if (wv == S - 1) stage(std::true_type{});
        else stage(std::false_type{});
    }
}

template <typename T, bool CP, bool GEN, int W>
static int launch_gpipe_w(const GPipeArgs &G, int grid, hipStream_t st)
{
    using Sh = GPipeShape<T, CP, GEN, W>;
    if (G.P.bcx || G.P.bcy)
        hipLaunchKernelGGL((k_gpipe<T, CP, GEN, W, Sh::K, Sh::S, true>), dim3(grid), dim3(Sh::S * kWave), 0, st, G);
    else
        hipLaunchKernelGGL((k_gpipe<T, CP, GEN, W, Sh::K, Sh::S, false>), dim3(grid), dim3(Sh::S * kWave), 0, st, G);
    CBDG_CHECK_LAUNCH("k_gpipe");
    return CBDG_OK;
}

}  // namespace cbdg
