// One recursion step of eq. (ref2) per launch for complex and per-bond
// operators on lattices too wide for the row pipeline (gpipe.hpp), each vector
// clipped to its own light cone.
//
// The tile is stored vector by vector, row by row (16-byte chunk j of column x
// at chunk j*Lx + x of its row).  A wavefront takes one vector, 64 columns and
// a run of rows; lane l owns one column, keeps rows y-1 .. y+1 of a_{n-1} and
// gets its x neighbours from the lanes beside it (the two columns beyond the
// block are loaded by its outer lanes).  a_n overwrites a_{n-2} in place.
//
// What bounds it: memory, 96 bytes of a complex128 site and step and, per bond,
// 160 of its record, inside the diamond of radius n around the start site only
// (records beside it in the wavefront's rows as well).  The vector-major kernels
// clip a tile to the bounding box of all its start sites, which for spread sites
// is the lattice: 512x512, N = 256, 256 vectors take 128 steps over 262144 sites
// each, the diamonds hold 9900 on average.  Of the 80 GB that makes, 59 cross HBM
// in 16.5 ms (3.6 TB/s; a large copy 4.75); the vector units are busy 17 %.
#include "gpipe.hpp"

#include <algorithm>

namespace cbdg {

struct GStepArgs {
    char *buf;       // a_{n-1} and a_{n-2} of the tile, `one` bytes each
    int64_t one;
    const void *recs;
    double th, lim;
    int Lx, Ly, bcx, bcy;
    int Bt, N, n;    // n: the step; a_n into buffer n & 1
    int n_blocks, n_runs;  // of the lattice
    const int32_t *sites;
    double *part;    // [steps of a batch][Bt * n_blocks * n_runs][4]
    double *mu_ee, *mu_he;
};

constexpr int kStepBatch = 8;   // steps whose sums are reduced together
// Shortest run of rows (512x512, N = 256, 256 vectors, ms: 8 rows 16.8, 16 16.5,
// 32 17.0; registers for four wavefronts on a SIMD instead of three change nothing).
constexpr int kStepRows = 16;

// Blocks of columns and runs of rows that step n's cone can touch: 2n + 1
// columns from anywhere in a block (one block more round a periodic row, whose
// last block may be short).  Wavefronts outside the cone are not launched: they
// took as long as the work (512x512, N = 256, 256 vectors: 182 us a launch of
// 65536 wavefronts, 129 us with the cone's own).
struct GStepGrid { int blocks, runs; };
__host__ __device__ inline GStepGrid gstep_grid(const GStepArgs &A, int n)
{
    const int b = (2 * n + 63) / kWave + (A.bcx ? 2 : 1), r = (2 * n + kStepRows) / kStepRows;
    return GStepGrid{b < A.n_blocks ? b : A.n_blocks, r < A.n_runs ? r : A.n_runs};
}

// Row y of a vector at column x (or zero), in the tile's layout.
template <typename T, bool CP>
struct GRow {
    static constexpr int NC = CP ? 4 : 2, NQ = NC * (int)sizeof(T) / 16 > 0 ? NC * (int)sizeof(T) / 16 : 1;
    static constexpr int NVP = NQ * 16 / (int)sizeof(T);
    __amdgpu_buffer_rsrc_t r;
    int Lx;
    __device__ __forceinline__ void load(T *v, int x, int y, bool ok) const
    {
        const unsigned at = ok ? (unsigned)((y * NQ * Lx + x) * 16) : kOut;
#pragma unroll
        for (int j = 0; j < NQ; ++j)
            unpack_row<T>(__builtin_amdgcn_raw_buffer_load_b128(r, at + (unsigned)(j * Lx * 16), 0, 0), v + j * (16 / (int)sizeof(T)));
    }
    __device__ __forceinline__ void store(const T *v, int x, int y, bool ok) const
    {
        const unsigned at = ok ? (unsigned)((y * NQ * Lx + x) * 16) : kOut;
#pragma unroll
        for (int j = 0; j < NQ; ++j)
            __builtin_amdgcn_raw_buffer_store_b128(pack_row<T>(v + j * (16 / (int)sizeof(T))), r, at + (unsigned)(j * Lx * 16), 0, 0);
    }
};

template <typename T, bool CP>
__device__ __forceinline__ GRow<T, CP> vector_rows(const GStepArgs &A, int which, int b)
{
    const int64_t bytes = (int64_t)A.Ly * A.Lx * GRow<T, CP>::NQ * 16;
    return GRow<T, CP>{__builtin_amdgcn_make_buffer_rsrc(A.buf + which * A.one + b * bytes, (short)0, (int)bytes, kRsrcWord3), A.Lx};
}

// A site's record (gpipe.hpp), loaded as it lies: 16-byte chunk j of column x
// at chunk j*Lx + x of its row, so that every load of a wavefront is one
// contiguous kilobyte (the operator's own arrays, 32 and 64 bytes a site, cost
// 64 lines an access: 512x512, N = 256, 256 vectors 25.6 ms).
template <typename T, bool CP, bool GEN> struct SiteCoef {
    static constexpr int REC = kRec<CP, GEN>, CQ = REC * (int)sizeof(T) / 16;
    T r[REC];
    __device__ __forceinline__ void load(const GStepArgs &A, int x, int y)
    {
        const U4 *q = reinterpret_cast<const U4 *>(A.recs) + (int64_t)y * CQ * A.Lx + x;
#pragma unroll
        for (int j = 0; j < CQ; ++j) unpack_row<T>(q[j * A.Lx], r + j * (16 / (int)sizeof(T)));
    }
    // 2 Ht c - p
    __device__ __forceinline__ Pair<T, CP> advance(T th, const Pair<T, CP> &c, const Pair<T, CP> &l, const Pair<T, CP> &rt,
                                                   const Pair<T, CP> &d, const Pair<T, CP> &u, const Pair<T, CP> &p) const
    {
        if constexpr (GEN) {
            static_assert(sizeof(T) == 8, "per-bond FP32 operators keep the one-step kernels");
            const Pair<T, CP> nb[4] = {rt, l, u, d};
            return bond_site_f64<CP>(r, c, nb, p);
        } else {
            return cheb_combine<T, CP>(apply_uniform<T, CP>(OnSite<T>{r[0], r[1], r[2], r[3]}, th, c, l, rt, d, u), p, false);
        }
    }
};

// a_0 and a_1 = Ht a_0 on the start site and its neighbours (all that later
// steps read of them), moments 0 .. 2; one thread per vector and site of the
// cross (thread 0 the start site).
template <typename T, bool CP, bool GEN>
__global__ __launch_bounds__(kWave) void k_gstep_seed(GStepArgs A)
{
    using Q = Pair<T, CP>;
    const int b = blockIdx.x, t = threadIdx.x;
    const int si = A.sites[b];
    const int64_t mrow = (int64_t)b * A.N;
    if (si < 0 || si >= A.Lx * A.Ly) {
        const double nan = __builtin_nan("");
        for (int n = t; n < A.N; n += kWave) {
            A.mu_ee[mrow + n] = nan;
            for (int c = 0; c < (CP ? 2 : 1); ++c) A.mu_he[(CP ? 2 : 1) * (mrow + n) + c] = nan;
        }
        return;
    }
    const int yi = si / A.Lx, xi = si - yi * A.Lx;
    double part = 0.0;
    if (t < 5) {
        const int s = t == 0 ? si : step_site_index(xi, yi, t - 1, A.Lx, A.Ly, A.bcx, A.bcy);
        if (s >= 0) {
            Q e = zero_pair<T, CP>(), z = zero_pair<T, CP>();
            if constexpr (CP) e.er = T(1);
            else e.e = T(1);
            const int y = s / A.Lx, x = s - y * A.Lx;
            // the start site as this site sees it: its own (0), or the neighbour
            // in the direction back, (t - 1) ^ 1
            const int back = t == 0 ? -1 : (t - 1) ^ 1;
            SiteCoef<T, CP, GEN> co;
            co.load(A, x, y);
            const Q v = co.advance(T(A.th), t == 0 ? e : z, back == 1 ? e : z, back == 0 ? e : z, back == 3 ? e : z,
                                   back == 2 ? e : z, z);
            T a[GRow<T, CP>::NVP] = {}, o[GRow<T, CP>::NVP] = {};
            put_pair<T, CP>(a, 0, v);
            for (int c = 0; c < GRow<T, CP>::NC; ++c) a[c] *= T(0.5);
            put_pair<T, CP>(o, 0, t == 0 ? e : z);
            vector_rows<T, CP>(A, 1, b).store(a, x, y, true);
            if (t == 0) vector_rows<T, CP>(A, 0, b).store(o, x, y, true);
            for (int c = 0; c < GRow<T, CP>::NC; ++c) part += (double)a[c] * (double)a[c];
            if (t == 0) {
                A.mu_ee[mrow] = 1.0;
                put_moment(A.mu_he, mrow, 0.0, 0.0, CP, A.lim);
                if (A.N > 1) {
                    put_moment(A.mu_ee, mrow + 1, (double)a[0], 0.0, false, A.lim);
                    put_moment(A.mu_he, mrow + 1, (double)a[CP ? 2 : 1], CP ? (double)a[3] : 0.0, CP, A.lim);
                }
            }
        }
    }
    double nrm = 0.0;
    for (int k = 0; k < 5; ++k) nrm += __shfl(part, k);
    if (t == 0 && A.N > 2) {
        put_moment(A.mu_ee, mrow + 2, 2.0 * nrm - 1.0, 0.0, false, A.lim);
        put_moment(A.mu_he, mrow + 2, 0.0, 0.0, CP, A.lim);
    }
}

template <typename T, bool CP, bool GEN>
__global__ __launch_bounds__(kBlock) void k_gstep(GStepArgs A)
{
    using Q = Pair<T, CP>;
    using R = GRow<T, CP>;
    const int lane = threadIdx.x % kWave;
    const GStepGrid grid = gstep_grid(A, A.n);
    const int per_vec = grid.blocks * grid.runs;
    const unsigned w = blockIdx.x * (kBlock / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (w >= (unsigned)(A.Bt * per_vec)) return;
    const int b = (int)(w / (unsigned)per_vec), at = (int)w - b * per_vec;
    const int run = at / grid.blocks;
    const int Lx = A.Lx, Ly = A.Ly, n = A.n;
    const bool bcx = A.bcx != 0, bcy = A.bcy != 0;
    double *part = A.part + ((int64_t)((n - 2) % kStepBatch) * A.Bt * A.n_blocks * A.n_runs + w) * 4;
    const int si = A.sites[b];
    const bool valid = si >= 0 && si < Lx * Ly;
    const int yi = valid ? si / Lx : 0, xi = valid ? si - yi * Lx : 0;
    // the wavefront's block of columns, counted from the cone's first
    int blk = at - run * grid.blocks;
    if (grid.blocks < A.n_blocks) {
        blk += (xi >= n ? xi - n : bcx ? xi - n + Lx : 0) / kWave;
        if (bcx && blk >= A.n_blocks) blk -= A.n_blocks;
        if (blk >= A.n_blocks) {
            if (lane < 4) part[lane] = 0.0;
            return;
        }
    }
    // rows of the vector's cone that reach these columns, shared out
    const int x0 = blk * kWave, x1 = min(x0 + kWave, Lx) - 1;
    int gap = xi < x0 ? x0 - xi : xi > x1 ? xi - x1 : 0;
    if (bcx && gap) gap = min(gap, xi < x0 ? xi + Lx - x1 : x0 + Lx - xi);
    const int m = n - gap;
    int lo = 0, hi = -1;
    if (valid && m >= 0) {
        if (bcy) {
            const bool all = 2 * m + 1 >= Ly;
            lo = all ? 0 : yi - m;
            hi = all ? Ly - 1 : yi + m;
        } else {
            lo = max(0, yi - m);
            hi = min(Ly - 1, yi + m);
        }
    }
    const int per = max(kStepRows, (hi - lo + grid.runs) / grid.runs);
    const int y0 = lo + run * per, y1 = min(y0 + per, hi + 1);
    if (y0 >= y1) {
        if (lane < 4) part[lane] = 0.0;
        return;
    }
    const auto prev = vector_rows<T, CP>(A, (n - 1) & 1, b), out = vector_rows<T, CP>(A, n & 1, b);
    // the lane's column; past a periodic row's end one lane holds column 0 for
    // its left neighbour.  The outer lanes also load the column beyond the block.
    const int xr = x0 + lane;
    const bool own = xr < Lx;
    const int x = own ? xr : 0;
    const bool has = own || (bcx && xr == Lx);
    int xe = lane == 0 ? x0 - 1 : x0 + kWave;
    if (bcx) xe = xe < 0 ? Lx - 1 : xe == Lx ? 0 : xe;
    const bool edge = (lane == 0 || lane == kWave - 1) && xe >= 0 && xe < Lx;
    auto dist = [&](int cx) -> int {
        const int d = cx < xi ? xi - cx : cx - xi;
        return bcx ? min(d, Lx - d) : d;
    };
    const int dx = dist(x), de = edge ? dist(xe) : 0;
    auto row = [&](int v, T *r) __attribute__((always_inline)) {
        const int y = lattice_row(v, Ly, bcy);
        const bool in = bcy || (unsigned)v < (unsigned)Ly;
        prev.load(r, x, in ? y : 0, in && has && dx + row_dist(y, yi, Ly, bcy) <= n - 1);
    };
    // Row v's inputs beside the window: a_{n-2}, the edge columns and the
    // coefficients.  They and row v + 2 of a_{n-1} are loaded while row v - 1 is
    // computed.
    struct Beside {
        T e[R::NVP], p[R::NVP];
        SiteCoef<T, CP, GEN> co;
    };
    auto beside = [&](int v, Beside &s) __attribute__((always_inline)) {
        const int y = lattice_row(v, Ly, bcy), dy = row_dist(y, yi, Ly, bcy);
        const bool in = bcy || (unsigned)v < (unsigned)Ly;
        prev.load(s.e, edge ? xe : 0, in ? y : 0, in && edge && de + dy <= n - 1);
        out.load(s.p, x, in ? y : 0, in && own && dx + dy <= n - 2);
        s.co.load(A, x, in ? y : 0);
    };
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    const T th = T(A.th);
    // one row: d, c, u its window; the window's next row goes to w
    auto step = [&](int v, const T *d, const T *c, const T *u, T *w, const Beside &s, Beside &nx) __attribute__((always_inline)) {
        row(v + 2, w);
        beside(v + 1, nx);
        __builtin_amdgcn_sched_barrier(0);
        const int y = lattice_row(v, Ly, bcy), dy = row_dist(y, yi, Ly, bcy);
        const Q cq = pair_at<T, CP>(c, 0), eq = pair_at<T, CP>(s.e, 0);
        Q l, r;
        if constexpr (CP) {
            l = Q{dpp_or<kShr1>(cq.er, eq.er), dpp_or<kShr1>(cq.ei, eq.ei), dpp_or<kShr1>(cq.hr, eq.hr), dpp_or<kShr1>(cq.hi, eq.hi)};
            r = Q{dpp_or<kShl1>(cq.er, eq.er), dpp_or<kShl1>(cq.ei, eq.ei), dpp_or<kShl1>(cq.hr, eq.hr), dpp_or<kShl1>(cq.hi, eq.hi)};
        } else {
            l = Q{dpp_or<kShr1>(cq.e, eq.e), dpp_or<kShr1>(cq.h, eq.h)};
            r = Q{dpp_or<kShl1>(cq.e, eq.e), dpp_or<kShl1>(cq.h, eq.h)};
        }
        const bool inside = own && v < y1 && dx + dy <= n;
        Q a = s.co.advance(th, cq, l, r, pair_at<T, CP>(d, 0), pair_at<T, CP>(u, 0), pair_at<T, CP>(s.p, 0));
        a = select_pair<T, CP>(inside, a, zero_pair<T, CP>());
        T o[R::NVP] = {};
        put_pair<T, CP>(o, 0, a);
        out.store(o, x, y, inside);
        if constexpr (CP) {
            const double er = a.er, ei = a.ei, hr = a.hr, hi2 = a.hi, cer = cq.er, cei = cq.ei, chr = cq.hr, chi = cq.hi;
            t[0] += (er * er + ei * ei) + (hr * hr + hi2 * hi2);
            t[1] += (er * cer + ei * cei) + (hr * chr + hi2 * chi);
            t[2] += (er * chr - ei * chi) - (hr * cer - hi2 * cei);
            t[3] += (er * chi + ei * chr) - (hr * cei + hi2 * cer);
        } else {
            const double ee = a.e, h = a.h, ce = cq.e, ch = cq.h;
            t[0] += ee * ee + h * h;
            t[1] += ee * ce + h * ch;
            t[2] += ee * ch - h * ce;
        }
    };
    // the window's four rows and the two sets beside it rotate by unrolling
    T win[4][R::NVP];
    Beside s[2];
    row(y0 - 1, win[0]);
    row(y0, win[1]);
    row(y0 + 1, win[2]);
    beside(y0, s[0]);
#pragma unroll 1
    for (int v = y0; v < y1; v += 4)
        repeat<4>([&](auto k) __attribute__((always_inline)) {
            constexpr int i = decltype(k)::value;
            step(v + i, win[i], win[(i + 1) % 4], win[(i + 2) % 4], win[(i + 3) % 4], s[i % 2], s[(i + 1) % 2]);
        });
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        t[k] = lane_sum(t[k]);
        if (lane == kWave - 1) part[k] = t[k];
    }
}

// Moments of the steps n0 .. n0 + steps - 1 from their partial sums: one
// wavefront per (vector, step), the partials added lane by lane and the lanes
// in a fixed order.
template <bool CP>
__global__ __launch_bounds__(kWave) void k_gstep_reduce(GStepArgs A, int n0)
{
    const int b = blockIdx.x, n = n0 + blockIdx.y, lane = threadIdx.x;
    const int si = A.sites[b];
    if (si < 0 || si >= A.Lx * A.Ly) return;
    const GStepGrid grid = gstep_grid(A, n);
    const int per_vec = grid.blocks * grid.runs;
    const double *p = A.part + ((int64_t)((n - 2) % kStepBatch) * A.Bt * A.n_blocks * A.n_runs + (int64_t)b * per_vec) * 4;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r = lane; r < per_vec; r += kWave)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] += p[4 * r + k];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = lane_sum(s[k]);
    if (lane != kWave - 1) return;
    PipeArgs P{};
    P.N = A.N; P.lim = A.lim; P.mu_ee = A.mu_ee; P.mu_he = A.mu_he;
    const int64_t mrow = (int64_t)b * A.N;
    gpipe_moments<CP>(P, mrow, n, s, A.mu_ee[mrow + 1], CP ? A.mu_he[2 * (mrow + 1)] : A.mu_he[mrow + 1],
                      CP ? A.mu_he[2 * (mrow + 1) + 1] : 0.0);
}

// Whether a tile takes these steps: more work than the light cones hold is
// saved, and the workspace holds two buffers and a batch's sums.
bool gstep_plan(const cbdg_op *op, int Bt, int N, bool f32, int64_t room)
{
    const bool cp = op->scalar == CBDG_COMPLEX;
    if (op->bounds.b != 0.0 || (!cp && !op->general)) return false;
    if (f32 && op->general) return false;  // the one-step kernels' roundings (gpipe.hip)
    // The cones cover at most half of the lattice on average over the steps:
    // past that the vector-major kernels move as few bytes, with scalar
    // coefficient loads.  Small tiles they leave waiting for three launches a
    // step (140x20, N = 260, 250 vectors 3.4 ms there, 1.9 here; 80x16, 600
    // vectors 3.8 / 3.2), but not where rows fill few lanes here (7x200, 1024
    // vectors 3.4 / 4.1).
    const double M = N / 2, L2 = (double)op->L2;
    const double bytes = L2 * (double)lane_stride(Bt) * (cp ? 4 : 2) * (f32 ? 4 : 8);
    if (2.0 * M * M / 3.0 > 0.5 * L2 && (op->Lx < 24 || bytes > 3e7)) return false;
    const int64_t vec = op->L2 * round_up((cp ? 4 : 2) * (f32 ? 4 : 8), 16);
    if (vec > INT32_MAX) return false;
    const int64_t per_vec = ceil_div(op->Lx, kWave) * std::max<int64_t>(1, op->Ly / kStepRows);
    const int64_t recs = op->L2 * (op->general ? (cp ? 20 : 12) : 4) * (f32 ? 4 : 8);
    return 2 * vec * Bt + kStepBatch * per_vec * Bt * 32 + recs + 512 <= room;
}

template <typename T, bool CP, bool GEN>
static int run_gstep_t(GStepArgs A, hipStream_t st)
{
    hipLaunchKernelGGL((k_gstep_seed<T, CP, GEN>), dim3(A.Bt), dim3(kWave), 0, st, A);
    CBDG_CHECK_LAUNCH("k_gstep_seed");
    if ((int64_t)A.Bt * A.n_blocks * A.n_runs > INT32_MAX) return fail(CBDG_EINVAL, "chebyshev_moments: launch grid too large");
    const int M = A.N / 2;
    for (int n0 = 2; n0 <= M; n0 += kStepBatch) {
        const int steps = std::min(kStepBatch, M - n0 + 1);
        for (int k = 0; k < steps; ++k) {
            A.n = n0 + k;
            const GStepGrid grid = gstep_grid(A, A.n);
            const int64_t waves = (int64_t)A.Bt * grid.blocks * grid.runs;
            hipLaunchKernelGGL((k_gstep<T, CP, GEN>), dim3((unsigned)ceil_div(waves, kBlock / kWave)), dim3(kBlock), 0, st, A);
            CBDG_CHECK_LAUNCH("k_gstep");
        }
        hipLaunchKernelGGL((k_gstep_reduce<CP>), dim3(A.Bt, steps), dim3(kWave), 0, st, A, n0);
        CBDG_CHECK_LAUNCH("k_gstep_reduce");
    }
    return CBDG_OK;
}

int run_gstep(const cbdg_op *op, bool f32, const int32_t *sites, int Bt, int N, void *ws, double *mu_ee, double *mu_he,
              hipStream_t st)
{
    const bool cp = op->scalar == CBDG_COMPLEX, gen = op->general;
    GStepArgs A{};
    A.buf = reinterpret_cast<char *>(ws);
    A.one = op->L2 * Bt * round_up((cp ? 4 : 2) * (f32 ? 4 : 8), 16);
    A.th = op->t / op->bounds.a;
    A.lim = moment_limit(f32);
    A.Lx = op->Lx; A.Ly = op->Ly; A.bcx = op->bc_x; A.bcy = op->bc_y;
    A.Bt = Bt; A.N = N;
    A.n_blocks = (int)ceil_div(op->Lx, kWave);
    A.n_runs = std::max(1, op->Ly / kStepRows);
    A.sites = sites;
    A.part = reinterpret_cast<double *>(A.buf + round_up(2 * A.one, 256));
    A.mu_ee = mu_ee; A.mu_he = mu_he;
    char *recs = A.buf + round_up(round_up(2 * A.one, 256) + (int64_t)kStepBatch * A.n_blocks * A.n_runs * Bt * 32, 256);
    A.recs = recs;
    const int rc = launch_gpipe_records(op, 1, op->Lx, op->Lx * (gen ? (cp ? 20 : 12) : 4), f32, recs, st);
    if (rc) return rc;
    if (f32) return run_gstep_t<float, true, false>(A, st);
    if (cp) return gen ? run_gstep_t<double, true, true>(A, st) : run_gstep_t<double, true, false>(A, st);
    return run_gstep_t<double, false, true>(A, st);
}

}  // namespace cbdg
