// Asks the library's host code, without a GPU, which kernels a moments call
// takes.  The launches of the pipelined recursion are replaced by functions
// that say which shape was launched; every other launch does nothing.
//
//   launch Lx Ly bc_x bc_y Bt f32 limit   the pipelined plan within `limit`
//       bytes and what it launches: "W L segs" and the launched "W C" (or "none")
//   prefix Lx Ly bc_x bc_y Bt N           "done at": the steps that the forward part
//       of a reverse pass takes in the pipeline and the buffer pair they end in
//   route Lx Ly bc_x bc_y complex general Bt N f32 direct
//       "vpipe", "gpipe", "gstep" or "steps"
#include "step.hpp"

#include <cstdio>
#include <cstring>

static int launched_W = 0, launched_C = 0;

namespace cbdg {
#define SHAPE(type, w, c) \
    int launch_pipe_##type##_##w##c(const PipeArgs &, hipStream_t) { launched_W = w; launched_C = c; return CBDG_OK; }
SHAPE(f64, 1, 1) SHAPE(f64, 2, 1) SHAPE(f64, 3, 1) SHAPE(f64, 4, 1) SHAPE(f64, 3, 2) SHAPE(f64, 4, 2)
SHAPE(f32, 1, 1) SHAPE(f32, 2, 1) SHAPE(f32, 4, 1) SHAPE(f32, 4, 2)
}  // namespace cbdg

extern "C" hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

using namespace cbdg;

static cbdg_op make_op(int Lx, int Ly, int bcx, int bcy, int cplx, int general)
{
    cbdg_op op;
    op.Lx = Lx; op.Ly = Ly; op.bc_x = bcx; op.bc_y = bcy;
    op.scalar = cplx ? CBDG_COMPLEX : CBDG_REAL;
    op.general = general != 0;
    op.t = 1.0;
    op.bounds.a = 8.0;
    op.L2 = (int64_t)Lx * Ly;
    return op;
}

int main()
{
    char what[16];
    while (scanf("%15s", what) == 1) {
        int Lx, Ly, bcx, bcy, Bt, f32;
        if (!strcmp(what, "launch")) {
            long long limit;
            if (scanf("%d %d %d %d %d %d %lld", &Lx, &Ly, &bcx, &bcy, &Bt, &f32, &limit) != 7) return 1;
            const cbdg_op op = make_op(Lx, Ly, bcx, bcy, 0, 0);
            const PipePlan p = pipe_plan(&op, Bt, 20000, f32, limit);
            launched_W = launched_C = 0;
            if (!p.W) { printf("none\n"); continue; }
            static char ws[1];
            double mu[2];
            if (run_pipe(&op, p, f32, nullptr, Bt, 20000, ws, mu, mu, true, nullptr)) return 2;
            printf("%d %d %d %d %d %lld\n", p.W, p.L, p.segs, launched_W, launched_C, (long long)p.bytes);
        } else if (!strcmp(what, "prefix")) {
            int N, done = 0, at = 0;
            if (scanf("%d %d %d %d %d %d", &Lx, &Ly, &bcx, &bcy, &Bt, &N) != 6) return 1;
            const cbdg_op op = make_op(Lx, Ly, bcx, bcy, 0, 0);
            static char ws[4];
            void *const buf[4] = {ws, ws + 1, ws + 2, ws + 3};
            double mu[2];
            if (run_pipe_prefix(&op, nullptr, Bt, N, N / 2, buf, ws, mu, mu, &done, &at, nullptr)) return 2;
            printf("%d %d\n", done, at);
        } else if (!strcmp(what, "route")) {
            int cplx, general, N, direct;
            if (scanf("%d %d %d %d %d %d %d %d %d %d", &Lx, &Ly, &bcx, &bcy, &cplx, &general, &Bt, &N, &f32, &direct) != 10) return 1;
            const cbdg_op op = make_op(Lx, Ly, bcx, bcy, cplx, general);
            size_t bytes = 0;
            if (cbdg_moments_workspace_size(&op, Bt, f32 ? CBDG_FP32_ACC64 : CBDG_FP64, CBDG_ALG_DOUBLING, &bytes)) return 2;
            const int64_t room = direct ? 2 * op.L2 * lane_stride(Bt) * (cplx ? 4 : 2) * (f32 ? 4 : 8) : (int64_t)bytes;
            const char *r = "steps";
            if (!direct && pipe_plan(&op, Bt, N, f32, room).W) r = "vpipe";
            else if (gpipe_plan(&op, Bt, N, f32, direct, room).W) r = "gpipe";
            else if (!direct && gstep_plan(&op, Bt, N, f32, room)) r = "gstep";
            printf("%s\n", r);
        } else {
            return 1;
        }
        fflush(stdout);
    }
    return 0;
}
