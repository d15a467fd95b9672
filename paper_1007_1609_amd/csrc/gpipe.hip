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

// Steps of a pass.
static int gpipe_steps(int W, bool f32, bool cp, bool gen)
{
    auto shape = [&](auto t, auto c, auto g) -> int {
        using T = decltype(t);
        constexpr bool CP = decltype(c)::value, GEN = decltype(g)::value;
        switch (W) {
        case 1: return GPipeShape<T, CP, GEN, 1>::K * GPipeShape<T, CP, GEN, 1>::S;
        case 2: return GPipeShape<T, CP, GEN, 2>::K * GPipeShape<T, CP, GEN, 2>::S;
        default: return GPipeShape<T, CP, GEN, 3>::K * GPipeShape<T, CP, GEN, 3>::S;
        }
    };
    using yes = std::true_type;
    using no = std::false_type;
    return f32 ? (cp ? (gen ? shape(0.f, yes{}, yes{}) : shape(0.f, yes{}, no{}))
                     : (gen ? shape(0.f, no{}, yes{}) : shape(0.f, no{}, no{})))
               : (cp ? (gen ? shape(0., yes{}, yes{}) : shape(0., yes{}, no{}))
                     : (gen ? shape(0., no{}, yes{}) : shape(0., no{}, no{})));
}

// Whether the pipeline is the faster way, by the time of either (us).  Here:
// trips of a workgroup's vectors, 1.1 us each, more where rows wrap and with two
// workgroups on a CU.  The one-step kernels: per step a launch (under doubling
// with its reductions; nearly all latency on small tiles) and the tile's bytes.
// Over 490 calls of 3 to 192 columns, 3 to 200 rows, 1 to 1024 vectors and N = 24
// to 260 the middle 80 % of the times lie within 30 % of these.  It is the
// neighbour moments of periodic-y lattices that stay: the workspace holds two
// buffers a vector, the pipeline needs four of every workgroup's, and half of the
// tile has to wait (FP64, N = 260: 11x200, 100 vectors 2.4 ms there, 11.6 here;
// 34x80, N = 64, 1024 vectors 0.96 / 3.5; under doubling it is faster in 19 of 20
// calls, 2.1 times on average).
static bool gpipe_pays(const cbdg_op *op, const GPipePlan &p, int Bt, int N, bool f32, bool direct)
{
    const bool cp = op->scalar == CBDG_COMPLEX, gen = op->general;
    const int L = gpipe_steps(p.W, f32, cp, gen), M = direct ? N - 1 : N / 2;
    int64_t trips = 0;
    for (int n = 2; n <= M; n += L) {
        const int64_t cone = 2 * (int64_t)(n + L - 1) + 1;
        const int64_t rows = cone < op->Ly ? cone : op->Ly + (op->bc_y ? 2 * L : 0);
        trips += std::max<int64_t>(rows + L / 4 + 8, L + 12);
    }
    const double trip = (direct ? 1.15 : 1.1) * (op->bc_x || op->bc_y ? (direct ? 1.45 : 1.25) : 1.0) * (p.grid > 256 ? 1.35 : 1.0);
    const double here = 25.0 + (double)(trips * ceil_div(Bt, p.grid)) * trip;
    const int kind = gen ? (cp ? 2 : 1) : 0;
    static const double kLaunch[2][3] = {{14, 15, 16}, {8, 12, 13}};  // us a step
    static const double kRate[3] = {2.2e6, 1.9e6, 1.6e6};             // bytes of one vector a us
    const double launch = kLaunch[direct][kind] * (op->Ly < 8 ? 0.75 : 1.0);
    const double bytes = (double)op->L2 * (double)lane_stride(Bt) * (cp ? 4 : 2) * (f32 ? 4 : 8);
    return here <= 0.9 * (20.0 + M * (launch + bytes / kRate[kind]));
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
    if (!gpipe_pays(op, p, Bt, N, f32, direct)) p.W = 0;
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
    A.n_pass = steps > 0 ? (int)ceil_div(steps, gpipe_steps(p.W, f32, cp, gen)) : 0;
    if (f32) {
        if (cp) return gen ? launch_gpipe_f32_cg(G, p.grid, st) : launch_gpipe_f32_cu(G, p.grid, st);
        return gen ? launch_gpipe_f32_rg(G, p.grid, st) : launch_gpipe_f32_ru(G, p.grid, st);
    }
    if (cp) return gen ? launch_gpipe_f64_cg(G, p.grid, st) : launch_gpipe_f64_cu(G, p.grid, st);
    return gen ? launch_gpipe_f64_rg(G, p.grid, st) : launch_gpipe_f64_ru(G, p.grid, st);
}

}  // namespace cbdg
