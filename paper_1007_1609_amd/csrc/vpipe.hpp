// Pipelined Chebyshev recursion of eq. (ref2) with moment doubling for real
// operators with uniform hopping: one workgroup per start vector (or per row
// segment of one), its wavefronts the stages of a pipeline.
//
// Lane l of a wavefront owns the W neighbouring columns lW .. lW+W-1 of a
// lattice row (nl = ceil(Lx / W) lanes in use).  Stage s takes K consecutive
// recursion steps ("levels"), so a pass advances L = S*K steps while the
// vector crosses memory once in and once out: rows enter at stage 0, go from
// stage to stage through LDS and leave at stage S-1.  On trip r a stage
// computes row r - j of its level j, which needs rows r-j-1 .. r-j+1 of the
// level below and row r-j two levels below: each level keeps the two newest
// rows of the level below in registers.  A stage runs K + 1 rows behind the
// one before it (the row it needs ahead was written to LDS on the trip
// before), one barrier per trip.
//
// What bounds it: vector instructions (18 operations per site and step where
// the factor 2 is folded in, 20 elsewhere: additions and fused multiply-adds of
// the stencil, six of the doubling sums) and, where wavefronts are few or rows
// take two, the trip's barrier.  Vector units busy: 256x256 FP32 94 % of the
// time, FP64 59, 96x72 periodic 76 (a part of it selects and lane reads where
// rows close), 150x100 54, 400x500 34; HBM 0.8 to 1.4 TB/s.  One wavefront per
// vector and seven steps per launch, as the passes of vcstep.hip run it, is
// bound by HBM instead (4 vectors per 7 steps at 5 TB/s); here the vectors cross
// memory 4 times per L = 12, 20 or 24 steps (two wavefronts a row, rows of up to
// 8 registers, wider rows).
//
// The passes of a vector follow each other inside one launch: rows of pass
// p + 1 enter as soon as stage 0 has finished pass p, while later stages
// still work on it.  Pass p writes a_{n+L-2} and a_{n+L-1} over a_{n-2} and
// a_{n-1} in place (open y: a row is read long before its successor is
// written), so the working set of the launch is two buffers per resident
// workgroup.  Trips of a pass, P: all its rows, K + 1 rows of zeros that
// separate it from the next (every level's window is then zero where the next
// pass begins), and at least the time its first rows need to come out again.
//
// Rows outside the light cone of the pass's last step are zero and are not
// run through; rows outside the lattice or the pass come out zero because the
// hopping is switched off for them and every other term is zero already.
#pragma once

#include <type_traits>

#include "rows.hpp"
#include "step.hpp"

namespace cbdg {

// How the columns meet the edge of the row (template parameter XM):
//   0  open, every lane in use holds W columns (Lx = nl W)
//   1  open, the last lane holds fewer
//   2  periodic, Lx = 64 W: the halo is a rotation of the wavefront
//   3  periodic otherwise
enum PipeEdge { kOpenFull = 0, kOpenPart = 1, kRotate = 2, kWrap = 3 };

namespace {

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_rows(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the wavefront in a fixed order; the result is lane 63's.
__device__ __forceinline__ double lane_sum(double v)
{
    v += dpp_rows<0x111, 0xF>(v);  // row_shr:1
    v += dpp_rows<0x112, 0xF>(v);
    v += dpp_rows<0x114, 0xF>(v);
    v += dpp_rows<0x118, 0xF>(v);
    v += dpp_rows<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_rows<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// A lane shift whose outermost lane takes `edge` instead.
template <int CTRL>
__device__ __forceinline__ double dpp_or(double v, double edge)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_or(float v, float edge)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL, typename T>
__device__ __forceinline__ Pair<T, false> dpp_pair_or(const Pair<T, false> &v, const Pair<T, false> &edge)
{
    return Pair<T, false>{dpp_or<CTRL>(v.e, edge.e), dpp_or<CTRL>(v.h, edge.h)};
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

template <typename T>
__device__ __forceinline__ void unpack(const U4 &v, Pair<T, false> *p)
{
    if constexpr (sizeof(T) == 8) {
        p[0].e = __hiloint2double((int)v[1], (int)v[0]);
        p[0].h = __hiloint2double((int)v[3], (int)v[2]);
    } else {
        p[0].e = __uint_as_float(v[0]); p[0].h = __uint_as_float(v[1]);
        p[1].e = __uint_as_float(v[2]); p[1].h = __uint_as_float(v[3]);
    }
}
template <typename T>
__device__ __forceinline__ U4 pack(const Pair<T, false> *p)
{
    if constexpr (sizeof(T) == 8)
        return U4{(unsigned)__double2loint(p[0].e), (unsigned)__double2hiint(p[0].e),
                  (unsigned)__double2loint(p[0].h), (unsigned)__double2hiint(p[0].h)};
    else
        return U4{__float_as_uint(p[0].e), __float_as_uint(p[0].h), __float_as_uint(p[1].e), __float_as_uint(p[1].h)};
}

constexpr int cx_gcd(int a, int b) { return b == 0 ? a : cx_gcd(b, a % b); }
constexpr int cx_lcm(int a, int b) { return a / cx_gcd(a, b) * b; }

// f(0), f(1), .. f(N-1) with the index a constant: unrolled however long f is
template <int N, int I = 0, typename F>
__device__ __forceinline__ void repeat(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        repeat<N, I + 1>(f);
    }
}

// How many trips ahead a stage of K levels loads a coefficient row: its ring
// of rows and the three-row windows rotate with the unrolled trips of a round,
// so the ring's length is kept to a divisor or small multiple of three.
template <int K> constexpr int kCoefAhead = K == 2 || K == 5 ? 2 : K == 4 ? 3 : 1;
// Trips of a round.
template <int K> constexpr int kRound = cx_lcm(3, K + kCoefAhead<K> - 1);

// A pass as one vector (or row segment) sees it: its first step n, its rows
// e0 .. e0+R-1 (virtual rows on periodic y: taken modulo Ly), the rows y0 ..
// y1-1 whose sums and results are its own, and its trips P.
struct PipeJob {
    int n, e0, R, P, y0, y1;
};

// The lattice row of virtual row v (periodic y: modulo Ly).
__device__ __forceinline__ int lattice_row(int v, int Ly, bool bcy)
{
    if (bcy && (unsigned)v >= (unsigned)Ly) {
        v %= Ly;
        if (v < 0) v += Ly;
    }
    return v;
}

// Lattice distance in y of lattice rows ph and yi.
__device__ __forceinline__ int row_dist(int ph, int yi, int Ly, bool bcy)
{
    const int d = ph < yi ? yi - ph : ph - yi;
    return bcy ? min(d, Ly - d) : d;
}

// A pointer known to be to device memory (a generic access would make every
// later wait of the trips wait for all loads).
template <typename P> __device__ __forceinline__ P *as_global(P *p)
{
    return (P *)(__attribute__((address_space(1))) P *)p;
}
__device__ __forceinline__ const void *as_global(const void *p) { return as_global(reinterpret_cast<const char *>(p)); }

__device__ __forceinline__ void global_pointers(PipeArgs &A)
{
    A.buf = as_global(A.buf);
    A.coef = as_global(A.coef);
    A.onsite = as_global(A.onsite);
    A.mu_ee = as_global(A.mu_ee);
    A.mu_he = as_global(A.mu_he);
    A.part = as_global(A.part);
}

// The kernel's arguments, read from memory where they are used: for code that
// runs once a pass, whose pointers would otherwise take scalar registers from
// the trips.
template <typename A>
__device__ __forceinline__ A cold_args()
{
    using C = const __attribute__((address_space(4))) A;
    C *q = (C *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    A a;
    __builtin_memcpy(&a, (const void *)q, sizeof(A));
    global_pointers(a);
    return a;
}

template <int K, int S, bool SEG>
__device__ __forceinline__ PipeJob pipe_job(const PipeArgs &A, int p, int yi, int seg)
{
    constexpr int L = K * S;
    PipeJob J;
    if (p >= A.n_pass) {  // idle until every stage has finished
        J.n = 0; J.e0 = 0; J.R = 0; J.P = 1 << 28; J.y0 = J.y1 = 0;
        return J;
    }
    J.n = A.n0 + p * L;
    const int m = J.n + L - 1, Ly = A.Ly;
    int lo, hi;
    bool wrap = false;
    if (SEG && A.bcy) {
        wrap = 2 * m + 1 >= Ly;
        lo = wrap ? 0 : yi - m;
        hi = wrap ? Ly - 1 : yi + m;
    } else {
        lo = max(0, yi - m);
        hi = min(Ly - 1, yi + m);
    }
    J.y0 = lo; J.y1 = hi + 1;
    J.e0 = lo;
    int e1 = hi;
    if constexpr (SEG) {
        const int per = max(4, (hi - lo + A.n_segs) / A.n_segs);
        J.y0 = min(lo + seg * per, hi + 1);
        J.y1 = min(J.y0 + per, hi + 1);
        // each level computes one row less at either end correctly
        J.e0 = J.y0 - L;
        e1 = J.y1 - 1 + L;
        if (!wrap) { J.e0 = max(J.e0, lo); e1 = min(e1, hi); }
    }
    J.R = J.y0 < J.y1 ? e1 - J.e0 + 1 : 0;
    // A row may enter again once it has come out (its stage-to-stage and
    // prefetch lag is L + S + 3 trips).  Passes over the whole of a periodic
    // lattice start it at the same row; only the first of them may need a row
    // that the pass before it, which starts elsewhere, wrote last.
    const bool turn = SEG && A.bcy && !wrap && 2 * (m + L) + 1 >= Ly;
    J.P = turn ? J.R + K + L + S + 6 + kRound<K> : max(J.R + K + kCoefAhead<K> + kRound<K>, L + S + 6);
    return J;
}

}  // namespace

// a_0 = |s,e>, a_1 = Ht a_0 and the moments that need no recursion: mu[0],
// mu[1] and, by the doubling identities, mu[2].  Called by `nt` threads of
// one vector; whole rows are written (every pair a pass may read).
template <typename T>
__device__ __forceinline__ void pipe_seed(const PipeArgs &A, int b, int si, int tid, int nt)
{
    using V = typename Storage<T, false>::type;
    const int64_t mrow = (int64_t)b * A.N;
    const int Lx = A.Lx, Ly = A.Ly, W = A.W;
    if (si < 0 || si >= Lx * Ly) {
        const double nan = __builtin_nan("");
        for (int n = tid; n < A.N; n += nt) { A.mu_ee[mrow + n] = nan; A.mu_he[mrow + n] = nan; }
        return;
    }
    const int yi = si / Lx, xi = si - yi * Lx;
    const OnSite<T> o = reinterpret_cast<const OnSite<T> *>(A.onsite)[si];
    const T th = T(A.th);
    V *v0 = reinterpret_cast<V *>(A.buf) + b * A.Dv, *v1 = reinterpret_cast<V *>(A.buf + A.one) + b * A.Dv;
    const int xl = xi > 0 ? xi - 1 : (A.bcx ? Lx - 1 : -1), xr = xi + 1 < Lx ? xi + 1 : (A.bcx ? 0 : -1);
    const int yd = yi > 0 ? yi - 1 : (A.bcy ? Ly - 1 : -1), yu = yi + 1 < Ly ? yi + 1 : (A.bcy ? 0 : -1);
    const int rowp = A.rowp;
    for (int i = tid; i < 3 * rowp; i += nt) {
        const int q = i / rowp, pos = i - q * rowp;
        const int y = q == 0 ? yi : q == 1 ? yd : yu;
        if (y < 0) continue;
        // position -> column: chunk j of lane l holds pairs j*kPer .. of the lane
        const int ch = pos / kPer<T>, lane = ch % A.nl, k = ch / A.nl * kPer<T> + pos % kPer<T>;
        const int x = k < W ? lane * W + k : -2;
        V a1 = V{T(0), T(0)};
        if (q == 0) {
            if (x == xi) a1 = V{o.de, o.dr};
            else if (x == xl || x == xr) a1 = V{-th, T(0)};
            v0[(int64_t)y * rowp + pos] = V{x == xi ? T(1) : T(0), T(0)};
        } else if (x == xi) a1 = V{-th, T(0)};
        v1[(int64_t)y * rowp + pos] = a1;
    }
    if (tid == 0) {
        const double lim = A.lim, nan = __builtin_nan("");
        const double e = (double)o.de, h = (double)o.dr, t = (double)th;
        A.mu_ee[mrow] = 1.0;
        A.mu_he[mrow] = 0.0;
        if (A.N > 1) {
            A.mu_ee[mrow + 1] = fabs(e) <= lim ? e : nan;
            A.mu_he[mrow + 1] = fabs(h) <= lim ? h : nan;
        }
        if (A.N > 2) {
            const int nb = (xl >= 0) + (xr >= 0) + (yd >= 0) + (yu >= 0);
            const double m2 = 2.0 * (e * e + h * h + nb * (t * t)) - 1.0;
            A.mu_ee[mrow + 2] = fabs(m2) <= lim ? m2 : nan;
            A.mu_he[mrow + 2] = 0.0;
        }
    }
}

// Moments 2m-1 and 2m of a row from the doubling sums of step m (m >= 2),
// a moment beyond the bound stored as NaN:
//   mu_ee[2m] = 2 <a_m|a_m> - 1,  mu_he[2m] = 0,
//   mu_ee[2m-1] = 2 <a_m|a_{m-1}> - mu_ee[1],
//   mu_he[2m-1] = 2 (-1)^m B(a_m, a_{m-1}) - mu_he[1]
__device__ __forceinline__ void pipe_moments(const PipeArgs &A, int64_t mrow, int m, const double *s, double e1, double h1)
{
    const double lim = A.lim, nan = __builtin_nan("");
    if (m < 2) return;
    if (2 * m < A.N) {
        const double v = 2.0 * s[0] - 1.0;
        A.mu_ee[mrow + 2 * m] = fabs(v) <= lim ? v : nan;
        A.mu_he[mrow + 2 * m] = 0.0;
    }
    if (2 * m - 1 < A.N) {
        const double v = 2.0 * s[1] - e1, h = ((m & 1) ? -2.0 : 2.0) * s[2] - h1;
        A.mu_ee[mrow + 2 * m - 1] = fabs(v) <= lim ? v : nan;
        A.mu_he[mrow + 2 * m - 1] = fabs(h) <= lim ? h : nan;
    }
}

// Steps a stage takes, stages, and wavefronts per SIMD (which caps a lane's
// registers at 512 / waves), for lanes of W columns in C wavefronts per row.
// Rows of up to 8 registers: five steps in each of four stages, two workgroups
// per CU whose barriers do not meet (1024 vectors, N = 512, ms: 128x128 4.6
// against 5.1 with eight stages, one workgroup per CU, and 5.0 with two steps
// in each of eight stages; 64x64 1.6 / 2.2 / 2.0; FP32 128x128 3.6 / 4.8 / 3.9).
// Wider rows: three steps, as many as 256 registers hold, in eight stages
// (256x256, N = 1024: 36.3; four stages and two workgroups 41.2, two steps in
// four stages 50.4; rows split over two wavefronts of five steps 41.0).
template <typename T, int W, int C> struct PipeShape {
    static constexpr int kRegs = W * (int)sizeof(T) / 2;  // of one row
    static constexpr int K = kRegs > 8 || C > 1 ? 3 : 5;
    static constexpr int S = kRegs > 8 && C == 1 ? 8 : 4;
    static constexpr int waves = 2;
};

// Trips from the load of a row to the trip that stage 0 uses it on.
constexpr int kPipeAhead = 3;

// Most trips of a launch that are planned (a workgroup counts them in an int;
// half of what it holds).  10^9 trips take a quarter of an hour.
constexpr int64_t kMaxTrips = 1 << 30;

template <typename T, int W, int C, int K, int S, int XM, bool SEG, bool FOLD>
__global__ __launch_bounds__(S * C * kWave) __attribute__((amdgpu_waves_per_eu(PipeShape<T, W, C>::waves)))
void k_vpipe(PipeArgs A)
{
    static_assert(C == 1 || (C == 2 && XM != kRotate), "two column halves exchange their edges through LDS");
    using P = Pair<T, false>;
    using V = typename Storage<T, false>::type;
    constexpr int L = K * S, NW = S * C;
    constexpr int NQ = (W + kPer<T> - 1) / kPer<T>;   // 16-byte chunks per lane and row
    constexpr int WP = NQ * kPer<T>;
    constexpr int NF = (C * NQ + NW / 2 - 1) / (NW / 2);  // chunks of a row each wavefront feeds
    constexpr int U = 3;
    constexpr int RC = K + kCoefAhead<K> - 1;         // coefficient rows r-K+1 .. r and those on their way
    constexpr int XC = kCoefAhead<K>;
    constexpr int UL = kRound<K>;
    __shared__ U4 hand[S][2][2][C][NQ][kWave];  // slot 0: rows entering; slot s: stage s-1 -> s
    __shared__ double sums[S][C][3 * K];
    __shared__ P edge[C > 1 ? 2 : 1][S][K][2][2];  // [parity][stage][level][half][side] of the levels' centre rows

    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int stg = wv / C, half = wv % C;
    const int b = SEG ? blockIdx.x / A.n_segs : blockIdx.x;
    const int seg = SEG ? blockIdx.x % A.n_segs : 0;
    const int Lx = A.Lx, Ly = A.Ly, nl = A.nl;
    const int si = __builtin_amdgcn_readfirstlane(A.sites[b]);
    const bool bcy = SEG && A.bcy;
    if (A.seed) pipe_seed<T>(cold_args<PipeArgs>(), b, si, threadIdx.x, NW * kWave);
    if (si < 0 || si >= Lx * Ly) return;
    const int yi = si / Lx, xi = si - yi * Lx;
    for (int i = threadIdx.x; i < S * 2 * 2 * C * NQ * kWave; i += NW * kWave) (&hand[0][0][0][0][0][0])[i] = U4{0, 0, 0, 0};
    if constexpr (C > 1)
        for (int i = threadIdx.x; i < 2 * S * K * 4; i += NW * kWave) (&edge[0][0][0][0][0])[i] = zero_pair<T, false>();
    __syncthreads();

    // byte offset of lane g's first chunk in row v of a vector that vanishes
    // outside the diamond of radius R, past the buffer's range where it does
    const int gl = half * kWave + lane;
    auto offset = [&](int g, int v, int R) -> unsigned {
        const int ph = lattice_row(v, Ly, bcy), rr = R - row_dist(ph, yi, Ly, bcy);
        const unsigned at = (unsigned)((ph * NQ * nl + g) * 16);
        bool ok = (g < nl) & (rr >= 0) & (bcy | ((unsigned)v < (unsigned)Ly));
        if constexpr (XM == kOpenFull || XM == kOpenPart) ok = ok & (g * W <= xi + rr) & (g * W + W - 1 >= xi - rr);
        const unsigned keep = 0u - (unsigned)ok;
        return (at & keep) | (kOut & ~keep);
    };
    const unsigned cstep = (unsigned)nl * 16u;

    // the hopping of each owned column, zero past the row's end
    const T th2 = (FOLD ? T(2) : T(1)) * T(A.th);
    constexpr bool kMask = (XM == kOpenPart || XM == kWrap) && PipeShape<T, W, C>::kRegs > 8;  // registers are short
    T thl[!kMask && (XM == kOpenPart || XM == kWrap) ? W : 1];
    const int lr = (Lx - 1) / W - (C - 1) * kWave, kr = (Lx - 1) % W;  // (last half's) lane and column of the row's end
    if constexpr (kMask) {
        thl[0] = th2;
    } else if constexpr (XM == kOpenPart || XM == kWrap) {
#pragma unroll
        for (int k = 0; k < W; ++k) thl[k] = gl * W + k < Lx ? th2 : T(0);
    } else {
        thl[0] = (XM == kRotate || gl < nl) ? th2 : T(0);
    }
    const V *pc = reinterpret_cast<const V *>(A.coef);
    auto coef_row = [&](int v, U4 *c) __attribute__((always_inline)) {
        const int ph = bcy ? lattice_row(v, Ly, true) : min(max(v, 0), Ly - 1);
        const U4 *q = reinterpret_cast<const U4 *>(pc) + (int64_t)ph * NQ * nl + min(gl, nl - 1);
#pragma unroll
        for (int j = 0; j < NQ; ++j) c[j] = q[j * nl];
    };

    // Pass p reads pair (p + cur) & flip of buffers and writes the next one
    // (flip 0: in place); a pair is a_{n-2} and a_{n-1} of the whole tile.
    const int vbytes = (int)(A.Dv * (int64_t)(2 * sizeof(T)));
    const uint64_t vbase = reinterpret_cast<uint64_t>(A.buf) + (uint64_t)b * (uint64_t)vbytes, one = (uint64_t)A.one;
    const int flip = A.flip, cur = A.cur;
    auto vec_of = [&](int pass, int newer) -> __amdgpu_buffer_rsrc_t {
        const uint64_t at = vbase + ((pass + cur) & flip ? 2 * one : 0) + (newer ? one : 0);
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char *>(at), (short)0, vbytes, kRsrcWord3);
    };

    // half of the wavefronts feed a_{n-1}'s rows, the others a_{n-2}'s
    const int fk = wv >= NW / 2 ? 1 : 0, fw = wv - fk * (NW / 2);
    int fp = 0, ft = -XC;
    PipeJob F = pipe_job<K, S, SEG>(A, 0, yi, seg);
    U4 fd[U][NF];
    auto feed_load = [&](U4 *d) __attribute__((always_inline)) {
        const int c = ft + 1 - fk;
        const bool in = (unsigned)c < (unsigned)F.R;
        const auto rs = vec_of(fp, 1 - fk);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int j = fw + f * (NW / 2);
            const unsigned o = in && j < C * NQ ? offset(j / NQ * kWave + lane, F.e0 + c, F.n - 1 - fk) + j % NQ * cstep : kOut;
            d[f] = __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0);
        }
        if (++ft == F.P - XC) { ft = -XC; ++fp; F = pipe_job<K, S, SEG>(A, fp, yi, seg); }
    };
    auto feed_store = [&](const U4 *d, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int j = fw + f * (NW / 2);
            if (j < C * NQ) hand[0][slot][fk][j / NQ][j % NQ][lane] = d[f];
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int f = 0; f < NF; ++f) fd[u][f] = U4{0, 0, 0, 0};

    // this stage's pass and its trip in it
    int jp = 0, jt = -XC - kPipeAhead - stg * (K + 1);
    PipeJob J = F;
    int total = kPipeAhead + (S - 1) * (K + 1) + 2 * UL;
    for (int p = 0; p < A.n_pass; ++p) total += pipe_job<K, S, SEG>(A, p, yi, seg).P;

    P in[3][W], lv[K > 1 ? K - 1 : 1][3][W];
    U4 cf[RC][NQ];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < W; ++k) {
            in[i][k] = zero_pair<T, false>();
#pragma unroll
            for (int j = 0; j < K - 1; ++j) lv[j][i][k] = zero_pair<T, false>();
        }
#pragma unroll
    for (int j = 0; j < RC; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q) cf[j][q] = U4{0, 0, 0, 0};
    double d[3 * K];
#pragma unroll
    for (int i = 0; i < 3 * K; ++i) d[i] = 0.0;

    auto trip = [&](auto place, int par, auto last, auto hf) __attribute__((always_inline)) {
        constexpr int H = decltype(hf)::value, u = decltype(place)::value;
        constexpr int sa = u % 3, sb = (u + 1) % 3, sc = (u + 2) % 3;  // oldest, middle, newest slot of the windows
        feed_store(fd[(u + 1) % U], par ^ 1);
        feed_load(fd[u % U]);
        // rows r+1 of a_{n-1} and r of a_{n-2} as the stage before left them
        P pr[WP], nw[WP];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            unpack<T>(hand[stg][par][0][H][q][lane], nw + q * kPer<T>);
            unpack<T>(hand[stg][par][1][H][q][lane], pr + q * kPer<T>);
        }
#pragma unroll
        for (int k = 0; k < W; ++k) in[sc][k] = nw[k];
        // The edge columns of a row that becomes level j's centre on the next
        // trip, for the other half: its inner edge, and on periodic rows the
        // row's first and last column.
        auto publish = [&](int j, const P *v) __attribute__((always_inline)) {
            if constexpr (C > 1) {
                if constexpr (H == 0) {
                    if (lane == kWave - 1) edge[par ^ 1][stg][j][0][1] = v[W - 1];
                    if constexpr (XM == kWrap) { if (lane == 0) edge[par ^ 1][stg][j][0][0] = v[0]; }
                } else {
                    if (lane == 0) edge[par ^ 1][stg][j][1][0] = v[0];
                    if constexpr (XM == kWrap) {
#pragma unroll
                        for (int k = 0; k < W; ++k)
                            if (k == kr && lane == lr) edge[par ^ 1][stg][j][1][1] = v[k];
                    }
                }
            }
        };
        publish(0, in[sc]);
        // the other half's edge columns of every level's centre row
        P inner[K], far[K];
        if constexpr (C > 1) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                inner[j] = edge[par][stg][j][1 - H][H];
                if constexpr (XM == kWrap) far[j] = edge[par][stg][j][1 - H][1 - H];
            }
        }

        P out[WP];
        if constexpr (WP > W) out[WP - 1] = zero_pair<T, false>();
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const P *cc = j == 0 ? in[sb] : lv[j > 0 ? j - 1 : 0][sb];
            const P *dd = j == 0 ? in[sa] : lv[j > 0 ? j - 1 : 0][sa];
            const P *uu = j == 0 ? in[sc] : lv[j > 0 ? j - 1 : 0][sc];
            const P *pp = j == 0 ? pr : (j == 1 ? in[sa] : lv[j > 1 ? j - 2 : 0][sa]);
            P *v = j == K - 1 ? out : lv[j < K - 1 ? j : 0][sc];
            const bool live = (unsigned)(jt - j) < (unsigned)J.R;
            V cj[WP];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                P t[kPer<T>];
                unpack<T>(cf[(u + RC - j) % RC][q], t);
#pragma unroll
                for (int i = 0; i < kPer<T>; ++i) cj[q * kPer<T> + i] = V{t[i].e, t[i].h};
            }
            P hl, hr, first = zero_pair<T, false>();
            if constexpr (C == 1) {
                hl = dpp_pair<XM == kRotate ? kRor1 : kShr1>(cc[W - 1]);
                hr = dpp_pair<XM == kRotate ? kRol1 : kShl1>(cc[0]);
                if constexpr (XM == kWrap) {
                    // column 0 and the row's last column meet
                    first = P{lane_value(cc[0].e, 0), lane_value(cc[0].h, 0)};
                    P end = cc[0];
#pragma unroll
                    for (int k = 1; k < W; ++k) end = select_pair<T, false>(k == kr, cc[k], end);
                    end = P{lane_value(end.e, lr), lane_value(end.h, lr)};
                    hl = select_pair<T, false>(lane == 0, end, hl);
                }
            } else if constexpr (H == 0) {
                hr = dpp_pair_or<kShl1>(cc[0], inner[j]);
                if constexpr (XM == kWrap) hl = dpp_pair_or<kShr1>(cc[W - 1], far[j]);
                else hl = dpp_pair<kShr1>(cc[W - 1]);
            } else {
                hl = dpp_pair_or<kShr1>(cc[W - 1], inner[j]);
                hr = dpp_pair<kShl1>(cc[0]);
                if constexpr (XM == kWrap) first = far[j];
            }
#pragma unroll
            for (int k = 0; k < W; ++k) {
                P r = k < W - 1 ? cc[k + 1] : hr;
                if constexpr (XM == kWrap && H == C - 1) r = select_pair<T, false>(lane == lr && k == kr, first, r);
                T ths;
                if constexpr (kMask) ths = live && gl * W + k < Lx ? th2 : T(0);
                else ths = live ? thl[XM == kOpenPart || XM == kWrap ? k : 0] : T(0);
                const P &l = k > 0 ? cc[k - 1] : hl;
                if constexpr (FOLD) {
                    v[k] = step_site<T>(cj[k], ths, cc[k], l, r, dd[k], uu[k], pp[k]);
                } else {
                    const OnSite<T> o{cj[k].x, -cj[k].x, cj[k].y, T(0)};
                    v[k] = cheb_combine<T, false>(apply_uniform<T, false>(o, ths, cc[k], l, r, dd[k], uu[k]), pp[k], false);
                }
            }
            if (j < K - 1) publish(j + 1, v);
            const int s = J.e0 + jt - j;
            const bool own = !SEG || (live && s >= J.y0 && s < J.y1);
            if (own) {
                // a row's own sum first: the running sums take one addition per row
                double t[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    T ce = cc[k].e, ch = cc[k].h;
                    // FP32: convert again rather than keep every window row in FP64 as well
                    if constexpr (sizeof(T) == 4) asm("" : "+v"(ce), "+v"(ch));
                    dots3(t, (double)v[k].e, (double)v[k].h, (double)ce, (double)ch);
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) d[3 * j + i] += t[i];
            }
            // added up here and not put off to the end of the round
#pragma unroll
            for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(d[3 * j + i]));
            // the oldest coefficient row has had its last use: the next one takes its place
            if (j == K - 1) coef_row(J.e0 + jt + XC, cf[(u + XC) % RC]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // level K-1's newest row and the oldest row of level K-2's window
        // (what the next stage, K+1 rows behind, needs on its next trip)
        const P *old = K == 1 ? in[sa] : lv[K > 1 ? K - 2 : 0][sa];
        P oldp[WP];
#pragma unroll
        for (int k = 0; k < W; ++k) oldp[k] = old[k];
        if constexpr (WP > W) oldp[WP - 1] = zero_pair<T, false>();
        if constexpr (!decltype(last)::value) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                hand[stg + 1][par ^ 1][0][H][q][lane] = pack<T>(out + q * kPer<T>);
                hand[stg + 1][par ^ 1][1][H][q][lane] = pack<T>(oldp + q * kPer<T>);
            }
        } else {
            const int s1 = J.e0 + jt - (K - 1), s2 = J.e0 + jt - K;
            const bool l1 = (unsigned)(jt - (K - 1)) < (unsigned)J.R && s1 >= J.y0 && s1 < J.y1;
            const bool l2 = (unsigned)(jt - K) < (unsigned)J.R && s2 >= J.y0 && s2 < J.y1;
            const unsigned o1 = l1 ? offset(gl, s1, J.n + L - 1) : kOut, o2 = l2 ? offset(gl, s2, J.n + L - 2) : kOut;
            const auto r1 = vec_of(jp + 1, 1), r2 = vec_of(jp + 1, 0);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                __builtin_amdgcn_raw_buffer_store_b128(pack<T>(out + q * kPer<T>), r1, o1 + q * cstep, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(pack<T>(oldp + q * kPer<T>), r2, o2 + q * cstep, 0, 0);
            }
        }
        ++jt;
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
    };
    const int rounds = (total + UL - 1) / UL;
    auto stage = [&](auto last, auto hf) __attribute__((always_inline)) {
        int par = 0, done = 0;  // done: first step of a pass whose sums lie in LDS
#pragma unroll 1
        for (int r = 0; r < rounds; ++r) {
            repeat<UL>([&](auto u) __attribute__((always_inline)) {
                trip(u, par, last, hf);
                par ^= 1;
            });
            if (done) {
                // a barrier after both halves left their sums: one lane per level
                if (half == 0 && lane < K) {
                    double s[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        s[k] = sums[stg][0][3 * lane + k];
                        if constexpr (C > 1) s[k] += sums[stg][1][3 * lane + k];
                    }
                    // (two halves: the registers a fresh read takes cost more,
                    // 512x512, N = 512, factor 2 folded in: 43.5 ms against 49.6)
                    PipeArgs B;
                    if constexpr (C > 1) B = A;
                    else B = cold_args<PipeArgs>();
                    if (!SEG || B.n_segs == 1) {
                        const OnSite<T> o = reinterpret_cast<const OnSite<T> *>(B.onsite)[si];
                        pipe_moments(B, (int64_t)b * B.N, done + lane, s, (double)o.de, (double)o.dr);
                    } else {
#pragma unroll
                        for (int k = 0; k < 3; ++k)
                            B.part[(((int64_t)(stg * K + lane) * B.n_segs + seg) * 3 + k) * B.Bt + b] = s[k];
                    }
                }
                done = 0;
            }
            if (jt < J.R + K + 1) continue;
            // The stage has finished its pass: sums, and on to the next (P
            // leaves room for the round's end to come before its first row).
#pragma unroll
            for (int i = 0; i < 3 * K; ++i) {
                const double v = lane_sum(d[i]);
                if (lane == kWave - 1) sums[stg][half][i] = v;
                d[i] = 0.0;
            }
            done = jp < A.n_pass ? J.n + stg * K : 0;
            jt -= J.P;
            ++jp;
            J = pipe_job<K, S, SEG>(A, jp, yi, seg);
        }
    };
    // The last stage has a loop of its own: the others' waits for their
    // coefficient loads must not count its stores.
    using std::integral_constant;
    if constexpr (C == 1) {
        if (stg == S - 1) stage(std::true_type{}, integral_constant<int, 0>{});
        else stage(std::false_type{}, integral_constant<int, 0>{});
    } else {
        if (half == 0) {
            if (stg == S - 1) stage(std::true_type{}, integral_constant<int, 0>{});
            else stage(std::false_type{}, integral_constant<int, 0>{});
        } else {
            if (stg == S - 1) stage(std::true_type{}, integral_constant<int, 1>{});
            else stage(std::false_type{}, integral_constant<int, 1>{});
        }
    }
}

// Whether the recursion runs with doubled coefficients (2 de, 2 Delta/a,
// 2 t/a), one operation per component less, as the passes of vcstep.hip do on
// their widths.  Its sums begin with a_{n-2}, whose magnitude every rounding of
// the chain then has; elsewhere a_{n-2} comes off last, as in the one-step
// kernels (FP64, rms error against 80-bit vectors, folded / not: 16x16, N =
// 2000, 1.7e-16 / 1.3e-16; 150x40, N = 512, 1.2e-16 / 0.9e-16), and FP32
// vectors keep the bits they have there.
inline bool pipe_folds(int Lx, int W, bool f32) { return W > 0 && W == vc_width(Lx, f32); }

template <typename T, int W, int C, int XM>
static int launch_pipe_x(const PipeArgs &A, hipStream_t st)
{
    using Sh = PipeShape<T, W, C>;
    const int64_t nb = (int64_t)A.Bt * A.n_segs;
    if (nb > INT32_MAX) return fail(CBDG_EINVAL, "chebyshev_moments: launch grid too large");
    const dim3 g((unsigned)nb), bl(Sh::S * C * kWave);
    auto go = [&](auto fold) {
        constexpr bool FOLD = decltype(fold)::value;
        if (A.n_segs > 1 || A.bcy)
            hipLaunchKernelGGL((k_vpipe<T, W, C, Sh::K, Sh::S, XM, true, FOLD>), g, bl, 0, st, A);
        else
            hipLaunchKernelGGL((k_vpipe<T, W, C, Sh::K, Sh::S, XM, false, FOLD>), g, bl, 0, st, A);
    };
    // pipe_folds: only rows of 64 W columns, and of those the widths vc_width has
    constexpr bool can_fold = C == 1 && (XM == kRotate || XM == kOpenFull) && (W == 2 || W == 4 || (W == 1 && sizeof(T) == 8));
    if constexpr (can_fold) {
        if (pipe_folds(A.Lx, W, sizeof(T) == 4)) go(std::true_type{});
        else go(std::false_type{});
    } else {
        go(std::false_type{});
    }
    CBDG_CHECK_LAUNCH("k_vpipe");
    return CBDG_OK;
}

template <typename T, int W, int C>
static int launch_pipe_w(const PipeArgs &A, hipStream_t st)
{
    if (A.bcx) {
        if constexpr (C == 1) {
            if (A.Lx == kWave * W) return launch_pipe_x<T, W, C, kRotate>(A, st);
        }
        return launch_pipe_x<T, W, C, kWrap>(A, st);
    }
    if constexpr (W > 1) {
        if (A.Lx % W) return launch_pipe_x<T, W, C, kOpenPart>(A, st);
    }
    return launch_pipe_x<T, W, C, kOpenFull>(A, st);
}

}  // namespace cbdg
