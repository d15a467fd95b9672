// Host side of the general row pipeline (gpipe.hpp): which tiles take it, the
// records, the launch.
#include "gpipe.hpp"

#include <algorithm>

namespace cbdg {

int launch_gpipe_f64_cg(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f64_cu(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f64_rg(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f64_ru(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f32_cg(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f32_cu(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f32_rg(const GPipeArgs &G, int grid, hipStream_t st);
int launch_gpipe_f32_ru(const GPipeArgs &G, int grid, hipStream_t st);

// Workgroups that run at once: two of four wavefronts per CU.
constexpr int kGPipeGrid = 512;

template <typename T, bool CP, bool GEN>
__global__ void k_gpipe_records(const OnSite<T> *__restrict__ ons, const void *__restrict__ bonds, T *__restrict__ out, int Lx,
                                int Ly, int bcx, int bcy, int W, int nl, int recs)
{
    constexpr int REC = kRec<CP, GEN>, per = 16 / (int)sizeof(T);
    const int cols = nl * W;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (int64_t)Ly * cols;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / cols), x = (int)(i - (int64_t)y * cols);
        T r[REC];
        for (int k = 0; k < REC; ++k) r[k] = T(0);
        if (x < Lx) {
            const int64_t s = (int64_t)y * Lx + x;
            const OnSite<T> o = ons[s];
            r[0] = o.de; r[1] = o.dh; r[2] = o.dr; r[3] = o.di;
            if constexpr (GEN) {
                const int64_t sl = x > 0 ? s - 1 : (bcx ? s + Lx - 1 : -1);
                const int64_t sd = y > 0 ? s - Lx : (bcy ? s + (int64_t)(Ly - 1) * Lx : -1);
                Link<T, CP> lk[4];
                links_of<T, CP>(bonds, s, sl, sd, lk);
                for (int q = 0; q < 4; ++q) {
                    T *l = r + 4 + q * (CP ? 4 : 2);
                    if constexpr (CP) { l[0] = lk[q].tr; l[1] = lk[q].ti; l[2] = lk[q].dr; l[3] = lk[q].di; }
                    else { l[0] = lk[q].t; l[1] = lk[q].d; }
                }
            }
        }
        for (int k = 0; k < REC; ++k) {
            const int e = x % W * REC + k;
            out[(int64_t)y * recs + ((int64_t)(e / per) * nl + x / W) * per + e % per] = kRecScale<T, GEN> * r[k];
        }
    }
}

// Steps of a pass, its trips beside its rows, and those until the last stage has finished.
struct GPipePass { int steps, lead, drain; };
static GPipePass gpipe_pass(int W, bool f32, bool cp, bool gen)
{
    auto shape = [&](auto t, auto c, auto g) -> GPipePass {
        using T = decltype(t);
        constexpr bool CP = decltype(c)::value, GEN = decltype(g)::value;
        auto of = [](auto sh) -> GPipePass {
            constexpr int K = decltype(sh)::K, S = decltype(sh)::S;
            return GPipePass{K * S, K + kCoefAhead<K> + kRound<K>, kPipeAhead + (S - 1) * (K + 1) + 2 * kRound<K>};
        };
        switch (W) {
        case 1: return of(GPipeShape<T, CP, GEN, 1>{});
        case 2: return of(GPipeShape<T, CP, GEN, 2>{});
        default: return of(GPipeShape<T, CP, GEN, 3>{});
        }
    };
    using yes = std::true_type;
    using no = std::false_type;
    return f32 ? (cp ? (gen ? shape(0.f, yes{}, yes{}) : shape(0.f, yes{}, no{}))
                     : (gen ? shape(0.f, no{}, yes{}) : shape(0.f, no{}, no{})))
               : (cp ? (gen ? shape(0., yes{}, yes{}) : shape(0., yes{}, no{}))
                     : (gen ? shape(0., no{}, yes{}) : shape(0., no{}, no{})));
}

// Whether the pipeline is the faster way, by a tenth at least, by the time of
// either (us).  Here: trips of a workgroup's vectors, more where rows wrap and with
// two workgroups on a CU.  The other kernels: launches (nearly all latency on small
// tiles) and the bytes of the tile.  Timed over 3600 calls of 3 to 400 columns, 2
// to 200 rows, 1 to 1024 vectors and N = 5 to 260.
//
// Neighbour moments: 1.27 times faster than with the one-step kernels alone, one
// call in 100 a tenth or more slower (25 us in place of 35: one in 70).  It is
// those of periodic-y lattices that stay there: the workspace holds two buffers a
// vector, the pipeline needs four of every workgroup's, and half of the tile has
// to wait (FP64, N = 260: 11x200, 100 vectors 2.4 ms there, 11.6 here; 34x80, N =
// 64, 1024 vectors 0.96 / 3.5).
static bool gpipe_pays_direct(const cbdg_op *op, const GPipePlan &p, int Bt, int N, bool f32)
{
    const bool cp = op->scalar == CBDG_COMPLEX, gen = op->general;
    const int L = gpipe_pass(p.W, f32, cp, gen).steps, M = N - 1;
    int64_t trips = 0;
    for (int n = 2; n <= M; n += L) {
        const int64_t cone = 2 * (int64_t)(n + L - 1) + 1;
        const int64_t rows = cone < op->Ly ? cone : op->Ly + (op->bc_y ? 2 * L : 0);
        trips += std::max<int64_t>(rows + L / 4 + 8, L + 12);
    }
    if (trips > kMaxTrips) return false;
    const double trip = 1.15 * (op->bc_x || op->bc_y ? 1.45 : 1.0) * (p.grid > 256 ? 1.35 : 1.0);
    const double here = 35.0 + (double)(trips * ceil_div(Bt, p.grid)) * trip;
    const int kind = gen ? (cp ? 2 : 1) : 0;
    static const double kLaunch[3] = {8, 12, 13};          // us a step
    static const double kRate[3] = {2.2e6, 1.9e6, 1.6e6};  // bytes of one vector a us
    const double bytes = (double)op->L2 * (double)lane_stride(Bt) * (cp ? 4 : 2) * (f32 ? 4 : 8);
    return here <= 0.9 * (20.0 + M * (kLaunch[kind] * (op->Ly < 8 ? 0.75 : 1.0) + bytes / kRate[kind]));
}

// Doubling: 2.2 times faster than with the other kernels alone, no call of 1200 a
// tenth slower.  Bytes and sites are those inside the cones, the tile's start
// sites taken to lie in a run; rows beside a workgroup's own take no sums.
static bool gpipe_pays_doubling(const cbdg_op *op, const GPipePlan &p, int Bt, int N, bool f32, int64_t room)
{
    const bool cp = op->scalar == CBDG_COMPLEX, gen = op->general;
    const int kind = (cp ? 1 + gen : 0), M = N / 2;  // per bond, complex, both
    static const double kTrip[3][2] = {{1.02, 1.09}, {1.14, 1.25}, {1.24, 1.38}};  // FP64, FP32
    const GPipePass s = gpipe_pass(p.W, f32, cp, gen);
    const int64_t Ly = op->Ly, L = s.steps;
    double trips = s.drain;
    for (int64_t n = 2; n <= M; n += L) {
        const int64_t cone = 2 * (n + L - 1) + 1, own = std::min(Ly, cone);
        const int64_t t = std::max(own + (op->bc_y && cone >= Ly ? 2 * L : 0) + s.lead, L + 10);
        trips += (double)t - 0.34 * (double)(t - own);
    }
    if (trips > (double)kMaxTrips) return false;
    const double two = p.grid > 256 ? 1.19 : 1.0;
    const int full = Bt / p.grid, rest = Bt % p.grid;
    const double here = 23.0 + trips * (full * two + (rest ? (rest > 256 ? two : 1.0) : 0.0)) * kTrip[kind][f32] *
                                   (p.W > 1 ? 1.07 : 1.0) * (op->bc_x ? 1.25 : 1.0) * (op->bc_y ? 1.28 : 1.0);
    static const double kLaunch[3] = {16.5, 13.5, 17.0};   // us a step, with its reductions
    static const double kRate[3] = {1.6e6, 1.8e6, 1.6e6};  // bytes of one vector a us
    // FP32 strips of four and eight complex columns take half as long again
    const double launch = kLaunch[kind] * (Ly < 8 ? 0.76 : 1.0) * (f32 && cp && op->Lx % 4 == 0 ? 1.6 : 1.0);
    const double row = (double)op->Lx * (double)lane_stride(Bt) * (cp ? 4 : 2) * (f32 ? 4 : 8);
    double rows = 2.0 * (double)Ly, sites = 0.0;  // cleared, written by the first step
    for (int64_t n = 1; n <= M; ++n) {
        rows += (double)(op->bc_y ? Ly : std::min(Ly, ceil_div(Bt, op->Lx) + 2 * n));
        sites += (double)std::min<int64_t>(op->L2, 2 * n * n);
    }
    double there = 30.0 + M * launch + rows * row / kRate[kind];
    // the steps inside each vector's cone: nearly all launches
    if (gstep_plan(op, Bt, N, f32, room))
        there = std::min(there, 20.0 + 20.0 * M + sites * Bt * ((gen ? (cp ? 20 : 12) : 4) + (cp ? 12 : 6)) * (f32 ? 4 : 8) / 14e6);
    return here <= 0.9 * there;
}

GPipePlan gpipe_plan(const cbdg_op *op, int Bt, int N, bool f32, bool direct, int64_t room)
{
    GPipePlan p{};
    const bool cp = op->scalar == CBDG_COMPLEX;
    if (!direct && (op->bounds.b != 0.0 || (!cp && !op->general))) return p;
    const int W = (int)ceil_div(op->Lx, kWave);
    if (W > (f32 ? 3 : 2)) return p;
    // FP32 per-bond sums: the one-step kernels' strips of two and more columns
    // round some of them differently by column, and keep those lattices.
    if (!direct && f32 && op->general && op->Lx % 2 == 0) return p;
    // A vector is one workgroup's: few vectors on a tall lattice are spread
    // better by the one-step passes.
    if (Bt < 64 && op->Ly > 128) return p;
    const int rec = op->general ? (cp ? 20 : 12) : 4, t = f32 ? 4 : 8, nc = cp ? 4 : 2;
    p.nl = (int)ceil_div(op->Lx, W);
    const int64_t row = p.nl * round_up(W * nc * t, 16);
    p.recs = (int)(p.nl * round_up(W * rec * t, 16) / t);
    const int nbuf = op->bc_y ? 4 : 2;
    const int64_t vec = row * op->Ly, recs = round_up((int64_t)p.recs * t * op->Ly, 256);
    if (vec > INT32_MAX || recs > INT32_MAX) return p;
    p.grid = (int)std::min<int64_t>({(int64_t)Bt, (int64_t)kGPipeGrid, (room - recs) / (nbuf * vec)});
    if (p.grid < 1 || 3 * (int64_t)p.grid < std::min(Bt, kGPipeGrid)) return p;
    p.Dv = vec / (nc * t);
    p.buf_at = recs;
    p.nbuf = nbuf;
    p.W = W;
    if (!(direct ? gpipe_pays_direct(op, p, Bt, N, f32) : gpipe_pays_doubling(op, p, Bt, N, f32, room))) p.W = 0;
    return p;
}

template <typename T, bool CP, bool GEN>
static int launch_records(const cbdg_op *op, int W, int nl, int recs, void *ws, hipStream_t st)
{
    const void *ons = sizeof(T) == 8 ? (const void *)op->onsite64 : (const void *)op->onsite32;
    const void *bonds = sizeof(T) == 8 ? op->bonds64 : op->bonds32;
    const unsigned grid = (unsigned)std::min<int64_t>(ceil_div((int64_t)op->Ly * nl * W, kBlock), 4096);
    hipLaunchKernelGGL((k_gpipe_records<T, CP, GEN>), dim3(grid), dim3(kBlock), 0, st,
                       reinterpret_cast<const OnSite<T> *>(ons), bonds, reinterpret_cast<T *>(ws), op->Lx, op->Ly, op->bc_x,
                       op->bc_y, W, nl, recs);
    CBDG_CHECK_LAUNCH("k_gpipe_records");
    return CBDG_OK;
}

int launch_gpipe_records(const cbdg_op *op, int W, int nl, int recs, bool f32, void *ws, hipStream_t st)
{
    const bool cp = op->scalar == CBDG_COMPLEX, gen = op->general;
    if (f32)
        return cp ? (gen ? launch_records<float, true, true>(op, W, nl, recs, ws, st) : launch_records<float, true, false>(op, W, nl, recs, ws, st))
                  : (gen ? launch_records<float, false, true>(op, W, nl, recs, ws, st) : launch_records<float, false, false>(op, W, nl, recs, ws, st));
    return cp ? (gen ? launch_records<double, true, true>(op, W, nl, recs, ws, st) : launch_records<double, true, false>(op, W, nl, recs, ws, st))
              : (gen ? launch_records<double, false, true>(op, W, nl, recs, ws, st) : launch_records<double, false, false>(op, W, nl, recs, ws, st));
}

int run_gpipe(const cbdg_op *op, const GPipePlan &p, bool f32, const int32_t *sites, int Bt, int N, void *ws, double *mu_ee,
              double *mu_he, double *nb_ee, double *nb_he, bool records, hipStream_t st)
{
    const bool cp = op->scalar == CBDG_COMPLEX, gen = op->general;
    if (records) {
        const int rc = launch_gpipe_records(op, p.W, p.nl, p.recs, f32, ws, st);
        if (rc) return rc;
    }
    GPipeArgs G{};
    PipeArgs &A = G.P;
    const int64_t one = p.Dv * (cp ? 4 : 2) * (f32 ? 4 : 8) * p.grid;
    A.buf = reinterpret_cast<char *>(ws) + p.buf_at;
    A.one = one;
    A.flip = p.nbuf == 4 ? 1 : 0;
    A.coef = ws;
    A.th = op->t / op->bounds.a;
    A.lim = moment_limit(f32);
    A.Lx = op->Lx; A.Ly = op->Ly; A.bcx = op->bc_x; A.bcy = op->bc_y;
    A.W = p.W; A.nl = p.nl; A.Dv = p.Dv;
    A.Bt = Bt; A.N = N; A.n0 = 2; A.n_segs = 1;
    A.sites = sites; A.mu_ee = mu_ee; A.mu_he = mu_he;
    G.recs = p.recs; G.nb_ee = nb_ee; G.nb_he = nb_he;
    const int steps = nb_ee ? N - 2 : N / 2 - 1;
    A.n_pass = steps > 0 ? (int)ceil_div(steps, gpipe_pass(p.W, f32, cp, gen).steps) : 0;
    if (f32) {
        if (cp) return gen ? launch_gpipe_f32_cg(G, p.grid, st) : launch_gpipe_f32_cu(G, p.grid, st);
        return gen ? launch_gpipe_f32_rg(G, p.grid, st) : launch_gpipe_f32_ru(G, p.grid, st);
    }
    if (cp) return gen ? launch_gpipe_f64_cg(G, p.grid, st) : launch_gpipe_f64_cu(G, p.grid, st);
    return gen ? launch_gpipe_f64_rg(G, p.grid, st) : launch_gpipe_f64_ru(G, p.grid, st);
}

}  // namespace cbdg
