// Host side of the pipelined recursion: which tiles take it, its coefficients
// and launches, and the reduction of the row segments' sums.
#include "vpipe.hpp"

#include <algorithm>
#include <cmath>

namespace cbdg {

int launch_pipe_f64_11(const PipeArgs &A, hipStream_t st);
int launch_pipe_f64_21(const PipeArgs &A, hipStream_t st);
int launch_pipe_f64_31(const PipeArgs &A, hipStream_t st);
int launch_pipe_f64_41(const PipeArgs &A, hipStream_t st);
int launch_pipe_f64_32(const PipeArgs &A, hipStream_t st);
int launch_pipe_f64_42(const PipeArgs &A, hipStream_t st);
int launch_pipe_f32_11(const PipeArgs &A, hipStream_t st);
int launch_pipe_f32_21(const PipeArgs &A, hipStream_t st);
int launch_pipe_f32_41(const PipeArgs &A, hipStream_t st);
int launch_pipe_f32_42(const PipeArgs &A, hipStream_t st);

// The shapes that are built: lanes of W columns, C wavefronts per row, in the
// order of the widest row they take.  one, two: microseconds a trip takes with
// one and with two workgroups on a CU (two: where it holds them); wrap: how much
// longer where rows close across lanes (kWrap).
struct PipeWidth {
    int W, C, L, S, per_cu;  // columns, wavefronts per row, steps and stages of a pass, workgroups per CU
    int lead, drain;         // trips of a pass beside its rows, of a launch until its last stage has finished
    double one, two, wrap;
    int (*launch)(const PipeArgs &, hipStream_t);
};
template <typename T, int W, int C>
static constexpr PipeWidth pipe_width(int (*launch)(const PipeArgs &, hipStream_t), double one, double two, double wrap)
{
    using Sh = PipeShape<T, W, C>;
    return PipeWidth{W, C, Sh::K * Sh::S, Sh::S, 4 * Sh::waves / (Sh::S * C), Sh::K + kCoefAhead<Sh::K> + kRound<Sh::K>,
                     kPipeAhead + (Sh::S - 1) * (Sh::K + 1) + 2 * kRound<Sh::K>, one, two, wrap, launch};
}
static const PipeWidth kWidths64[] = {
    pipe_width<double, 1, 1>(launch_pipe_f64_11, 0.67, 0.82, 1.5),
    pipe_width<double, 2, 1>(launch_pipe_f64_21, 0.97, 1.28, 1.45),
    pipe_width<double, 3, 1>(launch_pipe_f64_31, 1.33, 0.0, 1.45),
    pipe_width<double, 4, 1>(launch_pipe_f64_41, 1.60, 0.0, 1.75),
    pipe_width<double, 3, 2>(launch_pipe_f64_32, 1.55, 0.0, 1.3),
    pipe_width<double, 4, 2>(launch_pipe_f64_42, 2.40, 0.0, 1.4),
};
static const PipeWidth kWidths32[] = {
    pipe_width<float, 1, 1>(launch_pipe_f32_11, 0.72, 0.94, 1.3),
    pipe_width<float, 2, 1>(launch_pipe_f32_21, 0.89, 1.10, 1.35),
    pipe_width<float, 4, 1>(launch_pipe_f32_41, 1.53, 2.12, 1.3),
    pipe_width<float, 4, 2>(launch_pipe_f32_42, 1.74, 0.0, 1.1),
};

static const PipeWidth *widths(bool f32, int *n)
{
    *n = f32 ? (int)(sizeof(kWidths32) / sizeof(*kWidths32)) : (int)(sizeof(kWidths64) / sizeof(*kWidths64));
    return f32 ? kWidths32 : kWidths64;
}

// The shape that was planned: steps of a pass and sums are sized for it.
static int launch_pipe(const PipePlan &p, const PipeArgs &A, bool f32, hipStream_t st)
{
    int n;
    const PipeWidth *w = widths(f32, &n);
    if (p.shape < 0 || p.shape >= n || w[p.shape].W != A.W || w[p.shape].L != p.L)
        return fail(CBDG_EUNSUPPORTED, "pipelined recursion: no shape for Lx = %d", A.Lx);
    return w[p.shape].launch(A, st);
}

static bool plan_width(const cbdg_op *op, const PipeWidth &w, int Bt, bool f32, bool cut, int64_t limit, PipePlan &p)
{
    // the row's end lies in its last wavefront (wrapping rows close there)
    if (kWave * w.W * w.C < op->Lx || kWave * w.W * (w.C - 1) >= op->Lx) return false;
    p = PipePlan{};
    p.W = w.W;
    p.L = w.L;
    p.nl = (int)ceil_div(op->Lx, w.W);
    p.rowp = p.nl * (int)round_up(w.W, f32 ? 2 : 1);
    // Row segments per vector, by the trips the slowest workgroup takes for a
    // pass.  One segment: the passes of a vector follow each other without a
    // gap, each taking its rows and those between two passes.  Segments: one
    // launch per pass; each fills and empties the pipeline and recomputes L
    // rows at either end, and the launches of a pass cost about 20 trips.
    // With one workgroup on a CU instead of two a trip is a little shorter
    // (256x256, N = 512, ms by segments; 64 vectors 1: 3.45, 2: 3.06, 4: 2.43,
    // 6: 4.11; 128 vectors 1: 3.52, 2: 3.13, 4: 4.77).
    const int rows = op->Ly, lag = 2 * p.L + 12, wrap = op->bc_y ? 2 * p.L : 0;
    auto rounds = [&](int64_t n) {
        return ceil_div(n, 256 * (int64_t)w.per_cu) - (w.per_cu > 1 && (n - 1) % 512 < 256 ? 0.1 : 0.0);
    };
    p.segs = 1;
    double best = rounds(Bt) * (std::max(rows + 12, p.L + 16) + wrap);
    for (int k = 2; cut && k <= rows / 4 && (int64_t)k * Bt <= 1024; ++k) {
        const double t = rounds((int64_t)k * Bt) * (ceil_div(rows, k) + 2 * p.L + lag) + 20;
        if (t < 0.95 * best) { best = t; p.segs = k; }
    }
    p.nbuf = p.segs > 1 || op->bc_y ? 4 : 2;
    const int64_t pair = f32 ? 8 : 16;
    p.Dv = (int64_t)op->Ly * p.rowp;
    if (p.Dv * pair > INT32_MAX) return false;
    p.coef_at = p.nbuf * p.Dv * Bt * pair;
    p.part_at = round_up(p.coef_at + p.Dv * pair, 256);
    p.bytes = p.part_at + (p.segs > 1 ? (int64_t)p.L * p.segs * 3 * Bt * 8 : 0);
    return p.bytes <= limit;
}

// Whether the pipeline is the faster way, by the time of either (us), both
// fitted to 43000 calls of 1 to 512 columns, 3 to 300 rows, 1 to 2000 vectors
// and N = 5 to 512, open and periodic.  Nine of ten times lie within 15 % (here,
// seven-step passes) and 35 % (vector-major passes) of these; the calls take
// 0.6 % more time, in the geometric mean, than with the faster way each time.
// Against the other passes alone they are 1.25 (FP64, 64, 128 and 256 columns),
// 1.53 (FP32), 1.94 and 1.74 times faster (other widths), with the pipeline
// alone 0.95, 1.25, 1.74 and 1.63 times.
//
// Here: trips.  A pass of L steps runs all of them however few are left (64x200
// periodic, 128 vectors, us here and in the seven-step passes: N = 48 207 / 150,
// N = 512 1597 / 1750), and on short lattices more trips than rows (256x6, N =
// 256, 1024 vectors 1622 / 669).  Rows beside a workgroup's own take no sums.
static double pipe_time(const cbdg_op *op, const PipePlan &p, const PipeWidth &w, int Bt, int N, bool f32)
{
    const int64_t Ly = op->Ly, L = w.L, slots = 256 * (int64_t)w.per_cu, nb = (int64_t)Bt * p.segs;
    double trips = 0.0, halo = 0.0;
    int passes = 0;
    for (int64_t n = 2; n <= N / 2; n += L, ++passes) {
        const int64_t cone = 2 * (n + L - 1) + 1, in = std::min(Ly, cone);
        const bool wrap = op->bc_y && cone >= Ly;
        const int64_t own = p.segs > 1 ? std::max<int64_t>(4, ceil_div(in, p.segs)) : in;
        const int64_t rows = wrap ? own + 2 * L : std::min(in, own + (p.segs > 1 ? 2 * L : 0));
        const int64_t t = std::max(rows + w.lead, L + w.S + 6);
        trips += (double)(t + (p.segs > 1 ? w.drain : 0));
        halo += (double)(t - own);
    }
    if (p.segs == 1) trips += w.drain;
    if (p.segs == 1 && trips > (double)kMaxTrips) return HUGE_VAL;
    trips -= (f32 ? 0.25 : 0.1) * halo;
    double trip = (double)(nb / slots) * (w.per_cu == 2 ? w.two : w.one);
    if (nb % slots) trip += w.per_cu == 2 && nb % slots > 256 ? w.two : w.one;
    if (op->bc_x && (w.C > 1 || op->Lx != kWave * w.W)) trip *= w.wrap;
    // (25 us in the fit: calls that are little more than launches stay there)
    return 35.0 + trips * trip + (p.segs > 1 ? 6.0 * passes : 0.0);
}

// The seven-step passes: launches, trips of a wavefront (1024 at a time), bytes.
static double vc_time(const cbdg_op *op, int vw, int Bt, int N, bool f32)
{
    // by lanes' width 1, 2, 4: us a launch, us a trip, bytes a us
    static const double kCost[2][3][3] = {{{6.4, 0.70, 1e9}, {3.8, 1.17, 11.5e6}, {3.4, 2.13, 12.6e6}},
                                          {{0, 0, 1e9}, {7.0, 0.88, 1e9}, {3.8, 1.57, 12.6e6}}};
    const double *c = kCost[f32][vw == 4 ? 2 : vw - 1];
    const int K = vc_steps(f32), M = N / 2, segs = vc_segments(op->Ly, Bt, K);
    const int64_t rounds = ceil_div((int64_t)Bt * segs, 1024);
    const double row = (double)op->Lx * Bt * (f32 ? 8 : 16), trip = c[1] * (op->bc_y ? 1.15 : 1.0);
    double us = 28.0;
    auto in = [&](int64_t m) { return (double)std::min<int64_t>(op->Ly, 2 * m + 1); };
    for (int n = 1; n <= M;) {
        const int left = M - n + 1, k = n == 1 ? 1 : left >= K ? K : left;
        const double rows = std::max(std::ceil(in(n + k - 1) / segs), 4.0) + 2.0 * (k - 1);
        us += c[0] + (segs > 1 ? 9.0 : 0.0) +
              std::hypot((double)rounds * rows * (k > 1 ? trip : 0.3 * c[1]), (2.0 * in(n) + 2.0 * in(n + k - 1)) * row / c[2]);
        n += k;
    }
    return us;
}

// The vector-major passes of three or two steps: launches and bytes, more of
// them where strips are narrow; the tile's start sites taken to lie in a run.
static double vm_time(const cbdg_op *op, int Bt, int N, bool f32)
{
    static const double kCost[2][4] = {{18.1, 4.7, 0.48, 3.3e6}, {20.7, 0.9, 1.38, 3.6e6}};
    const double *c = kCost[f32];
    const int k3 = Bt > 128 ? 3 : 2, M = N / 2;
    const int strip = k3 == 2 && op->Lx % 8 == 0 ? 8 : op->Lx % 4 == 0 ? 4 : op->Lx % 2 == 0 ? 2 : 1;
    const double row = (double)op->Lx * (double)lane_stride(Bt) * (f32 ? 8 : 16);
    double us = 30.0 + 3.0 * op->Ly * row / 20e6;
    for (int n = 1; n <= M;) {
        const int left = M - n + 1, k = n == 1 ? 1 : std::min(k3, left);
        const int64_t cone = ceil_div(Bt, op->Lx) + 2 * (int64_t)(n + k - 1);
        const double rows = n == 1 || op->bc_y ? op->Ly : (double)std::min<int64_t>(op->Ly, cone);
        us += c[0] + c[1] * (k - 1) + (n == 1 ? 2.0 : k > 1 ? 4.0 : 3.0) * rows * row * (1.0 + (k > 1 ? c[2] / strip : 0.0)) / c[3];
        n += k;
    }
    return us;
}

PipePlan pipe_plan(const cbdg_op *op, int Bt, int N, bool f32, int64_t limit)
{
    PipePlan p{};
    if (op->scalar != CBDG_REAL || op->general || op->bounds.b != 0.0) return p;
    int n;
    const PipeWidth *w = widths(f32, &n);
    for (int cut = 1; cut >= 0; --cut)
        for (int i = 0; i < n; ++i)
            if (plan_width(op, w[i], Bt, f32, cut != 0, limit, p)) {
                const int vw = vc_width(op->Lx, f32);
                const double there = vw ? vc_time(op, vw, Bt, N, f32) : vm_time(op, Bt, N, f32);
                p.shape = i;
                if (pipe_time(op, p, w[i], Bt, N, f32) > there) p.W = 0;
                return p;
            }
    p.W = 0;
    return p;
}

// scale * (de, Delta/a) of every site in the passes' row layout, zero past Lx
template <typename T>
__global__ void k_pipe_coef(const OnSite<T> *__restrict__ ons, typename Storage<T, false>::type *__restrict__ pc, int Lx,
                            int W, int nl, int rowp, int64_t Dv, T scale)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < Dv; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t y = i / rowp;
        const int pos = (int)(i - y * rowp), ch = pos / kPer<T>;
        const int k = ch / nl * kPer<T> + pos % kPer<T>, x = ch % nl * W + k;
        typename Storage<T, false>::type c{T(0), T(0)};
        if (k < W && x < Lx) {
            const OnSite<T> o = ons[y * Lx + x];
            c = typename Storage<T, false>::type{scale * o.de, scale * o.dr};
        }
        pc[i] = c;
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_pipe_seed(PipeArgs A)
{
    pipe_seed<T>(A, blockIdx.x, A.sites[blockIdx.x], threadIdx.x, kBlock);
}

// Moments of the steps n0 .. n0+L-1 from the segments' sums, added in order:
// one thread per (step, vector).
template <typename T>
__global__ void k_pipe_reduce(PipeArgs A, int L)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= (int64_t)L * A.Bt) return;
    const int lev = (int)(i / A.Bt), b = (int)(i - (int64_t)lev * A.Bt);
    const int32_t si = A.sites[b];
    if (si < 0 || si >= A.Lx * A.Ly) return;
    double s[3] = {0.0, 0.0, 0.0};
    for (int g = 0; g < A.n_segs; ++g)
        for (int k = 0; k < 3; ++k) s[k] += A.part[(((int64_t)lev * A.n_segs + g) * 3 + k) * A.Bt + b];
    const OnSite<T> o = reinterpret_cast<const OnSite<T> *>(A.onsite)[si];
    pipe_moments(A, (int64_t)b * A.N, A.n0 + lev, s, (double)o.de, (double)o.dr);
}

// The operator's part of a launch's arguments.
static PipeArgs pipe_args(const cbdg_op *op, const PipePlan &p, bool f32, int Bt, int N, const int32_t *sites, double *mu_ee,
                          double *mu_he)
{
    PipeArgs A{};
    A.flip = p.nbuf == 4 ? 1 : 0;
    A.onsite = f32 ? (const void *)op->onsite32 : (const void *)op->onsite64;
    A.th = op->t / op->bounds.a;
    A.lim = moment_limit(f32);
    A.Lx = op->Lx; A.Ly = op->Ly; A.bcx = op->bc_x; A.bcy = op->bc_y;
    A.W = p.W; A.nl = p.nl; A.rowp = p.rowp; A.Dv = p.Dv;
    A.Bt = Bt; A.N = N; A.n_segs = p.segs;
    A.n0 = 2;
    A.sites = sites; A.mu_ee = mu_ee; A.mu_he = mu_he;
    return A;
}

// Rows of 64 W columns lie as the seven-step passes keep them, so that those
// can take the recursion over at any step.
int run_pipe_prefix(const cbdg_op *op, const int32_t *sites, int Bt, int N, int steps, void *const *buf, const void *coef,
                    double *mu_ee, double *mu_he, int *done, int *at, hipStream_t st)
{
    *done = *at = 0;
    const PipePlan p = pipe_plan(op, Bt, N, false, INT64_MAX);
    if (!p.W || p.segs != 1 || p.nl * p.W != op->Lx || p.W != vc_width(op->Lx, false)) return CBDG_OK;
    const int passes = (steps - 1) / p.L;
    if (passes < 1) return CBDG_OK;
    PipeArgs A = pipe_args(op, p, false, Bt, N, sites, mu_ee, mu_he);
    A.buf = reinterpret_cast<char *>(buf[0]);
    A.one = reinterpret_cast<char *>(buf[1]) - A.buf;
    A.coef = coef;
    A.seed = 1;
    A.n_pass = passes;
    *done = 1 + passes * p.L;
    *at = passes & A.flip ? 2 : 0;
    return launch_pipe(p, A, false, st);
}

template <typename T>
static int run_pipe_t(const cbdg_op *op, const PipePlan &p, const int32_t *sites, int Bt, int N, char *ws, double *mu_ee,
                      double *mu_he, bool coef, hipStream_t st)
{
    using V = typename Storage<T, false>::type;
    constexpr bool f32 = sizeof(T) == 4;
    PipeArgs A = pipe_args(op, p, f32, Bt, N, sites, mu_ee, mu_he);
    A.buf = ws;
    A.one = p.Dv * Bt * (int64_t)sizeof(V);
    A.coef = ws + p.coef_at;
    A.part = reinterpret_cast<double *>(ws + p.part_at);
    if (coef) {
        hipLaunchKernelGGL((k_pipe_coef<T>), dim3((unsigned)std::min<int64_t>(ceil_div(p.Dv, kBlock), 4096)), dim3(kBlock),
                           0, st, reinterpret_cast<const OnSite<T> *>(A.onsite), reinterpret_cast<V *>(ws + p.coef_at),
                           A.Lx, A.W, A.nl, A.rowp, A.Dv, T(pipe_folds(A.Lx, A.W, f32) ? 2 : 1));
        CBDG_CHECK_LAUNCH("k_pipe_coef");
    }
    const int steps = N / 2 - 1, passes = (int)ceil_div(steps, p.L);
    if (p.segs == 1 && steps > 0) {
        A.seed = 1;
        A.n_pass = passes;
        return launch_pipe(p, A, f32, st);
    }
    hipLaunchKernelGGL((k_pipe_seed<T>), dim3(Bt), dim3(kBlock), 0, st, A);
    CBDG_CHECK_LAUNCH("k_pipe_seed");
    A.n_pass = 1;
    for (int i = 0; i < passes; ++i) {
        A.n0 = 2 + i * p.L;
        A.cur = i & 1;
        int rc = launch_pipe(p, A, f32, st);
        if (rc) return rc;
        hipLaunchKernelGGL((k_pipe_reduce<T>), dim3((unsigned)ceil_div((int64_t)p.L * Bt, kBlock)), dim3(kBlock), 0, st, A, p.L);
        CBDG_CHECK_LAUNCH("k_pipe_reduce");
    }
    return CBDG_OK;
}

int run_pipe(const cbdg_op *op, const PipePlan &p, bool f32, const int32_t *sites, int Bt, int N, void *ws, double *mu_ee,
             double *mu_he, bool coef, hipStream_t st)
{
    return f32 ? run_pipe_t<float>(op, p, sites, Bt, N, reinterpret_cast<char *>(ws), mu_ee, mu_he, coef, st)
               : run_pipe_t<double>(op, p, sites, Bt, N, reinterpret_cast<char *>(ws), mu_ee, mu_he, coef, st);
}

}  // namespace cbdg
