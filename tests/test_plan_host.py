"""Host side of the row pipelines without a GPU: the shape that is launched is
the planned one, whatever workspace the plan was given."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1007_1609_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_host")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "native", "plan_host.cpp"), "-o", exe, "-L", PKG,
           "-lcbdg", "-Wl,-rpath," + PKG]
    subprocess.run(cmd, check=True)

    def run(lines):
        r = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True)
        return r.stdout.split("\n")[:len(lines)]

    return run


def _launched(ask, calls):
    return [None if s == "none" else tuple(int(v) for v in s.split()) for s in ask(["launch %d %d %d %d %d %d %d" % c for c in calls])]


@pytest.mark.parametrize("f32", [0, 1])
def test_the_planned_shape_is_launched(ask, f32):
    """Steps of a pass by shape: 20 where a row takes up to 8 registers (two
    wavefronts a row: 12), 24 on wider rows.  Limits from what the widest plan
    takes downwards, so that every shape that a plan can fall back to comes up."""
    calls = [(Lx, Ly, bcx, bcy, Bt, f32) for Lx in (64, 65, 128, 129, 192, 193, 256, 300, 384, 385, 512) for bcx in (0, 1)
             for bcy in (0, 1) for Ly in (40, 300, 1000) for Bt in (1, 8, 64)]
    full = _launched(ask, [c + (1 << 50,) for c in calls])
    calls = [c + (int(p[5] * k) - d,) for c, p in zip(calls, full) if p
             for k, d in ((1, 0), (1, 1), (0.99999, 0), (0.9999, 0), (0.999, 0), (0.99, 0), (0.9, 0), (0.6, 0))]
    seen = set()
    for c, plan in zip(calls, _launched(ask, calls)):
        if plan is None:
            continue
        W, L, _, lW, lC, _ = plan
        steps = 12 if lC == 2 else 20 if lW * (4 if f32 else 8) // 2 <= 8 else 24
        assert (lW, steps) == (W, L), (c, plan)
        # the columns of a row reach into the second wavefront
        assert 64 * lW * (lC - 1) < c[0] <= 64 * lW * lC, (c, plan)
        seen.add((lW, lC))
    assert len(seen) == (4 if f32 else 6)


def test_calls_take_the_faster_passes(ask):
    """Calls measured on either side of the line, by at least a fifth: few
    steps in a pass of many, few rows, a part of the GPU filled; and the ones
    that the pipeline is for."""
    call = "route %d %d %d %d 0 0 %d %d %d 0"  # Lx Ly bc_x bc_y Bt N f32
    steps = [(256, 6, 0, 0, 1024, 256, 0), (128, 64, 1, 1, 1024, 48, 0), (128, 300, 0, 0, 1024, 48, 0), (64, 80, 1, 1, 1024, 48, 0),
             (256, 96, 0, 0, 1024, 48, 1), (256, 3, 0, 0, 700, 256, 1), (200, 8, 1, 1, 1024, 12, 0), (130, 16, 1, 1, 1024, 5, 1),
             (390, 8, 1, 1, 1024, 5, 0), (256, 256, 0, 0, 64, 256, 1), (24, 128, 1, 1, 1024, 256, 1)]
    pipe = [(256, 256, 0, 0, 1024, 1024, 0), (256, 256, 0, 0, 1024, 2048, 1), (16, 16, 0, 0, 256, 256, 0), (96, 72, 1, 1, 1024, 384, 0),
            (150, 100, 0, 0, 441, 2048, 0), (400, 500, 0, 1, 64, 2000, 0), (128, 128, 0, 0, 1024, 512, 0), (64, 64, 1, 1, 1024, 512, 0),
            (128, 24, 0, 0, 128, 512, 0), (33, 130, 1, 1, 1024, 200, 1), (24, 8, 1, 1, 8, 200, 1)]
    for calls, want in ((steps, "steps"), (pipe, "vpipe")):
        assert ask([call % c for c in calls]) == [want] * len(calls)


def test_general_calls_take_the_faster_passes(ask):
    """The same for complex and per-bond operators and neighbour moments."""
    call = "route %d %d %d %d %d %d %d %d %d %d"  # Lx Ly bc_x bc_y complex per-bond Bt N f32 neighbours
    steps = [(11, 130, 1, 1, 0, 0, 100, 5, 0, 1), (16, 130, 1, 1, 1, 1, 512, 260, 0, 1), (11, 60, 1, 0, 0, 0, 512, 5, 0, 1),
             (95, 3, 0, 1, 1, 0, 285, 12, 0, 1), (47, 7, 1, 0, 0, 0, 100, 5, 1, 1), (33, 12, 1, 0, 1, 1, 250, 5, 1, 0)]
    pipe = [(48, 40, 0, 0, 1, 1, 1024, 256, 0, 1), (48, 40, 0, 0, 1, 1, 512, 256, 0, 0), (41, 20, 0, 0, 1, 0, 40, 256, 0, 1),
            (65, 9, 1, 1, 1, 1, 30, 100, 0, 1)]
    for calls, want in ((steps, "steps"), (pipe, "gpipe")):
        assert ask([call % c for c in calls]) == [want] * len(calls)


def test_the_parity_tests_reach_the_pipelines(ask):
    from tests import test_parity_gpipe as G
    from tests import test_parity_pipe as V
    kinds = [(int(c), int(b)) for c, b, _ in G.KINDS] + [(0, 0)]
    call = "route %d %d %d %d %d %d %d %d %d %d"
    nb = [call % (*c[:4], *kinds[k], c[4], c[5], p, 1) for c in G.NB_ROUTED for k, p in c[6]]
    dbl = [call % (*c[:4], *kinds[k], min(c[4], c[0] * c[1]), c[5], p, 0) for c in G.DOUBLING_ROUTED for p in (0, 1) for k in c[6 + p]]
    for calls in (nb, dbl):
        assert [(c, r) for c, r in zip(calls, ask(calls)) if r != "gpipe"] == []
    real = [(Lx, 31, bcx, Lx % 2, min(260, 31 * Lx), 90, p) for Lx in V.WIDTHS for bcx in (0, 1) for p in (0, 1) if not bcx or Lx >= 3]
    real += [(Lx, 40, 0, 0, 257, 2 * (k * L + 1) + off, 0) for Lx, L in ((64, 20), (192, 24), (384, 12)) for k in (1, 2)
             for off in (-2, -1, 0, 1, 2, 3)]
    real += [(*c, 161, p) for c in ((64, 200, 0, 0, 3), (64, 200, 0, 1, 3), (100, 150, 1, 1, 20), (256, 130, 0, 0, 1), (300, 90, 0, 1, 9),
                                    (16, 3, 1, 1, 48), (64, 61, 0, 1, 300), (128, 43, 1, 1, 300)) for p in (0, 1)]
    calls = [call % (*c[:4], 0, 0, *c[4:], 0) for c in real]
    assert [(c, r) for c, r in zip(calls, ask(calls)) if r != "vpipe"] == []


def test_the_reverse_pass_tests_begin_in_the_pipeline(ask):
    from tests.test_parity_vc_adjoint import PERIODIC
    calls = ["prefix %d %d %d 1 %d %d" % c[:5] for c in PERIODIC]
    assert ask(calls) == ["%d %d" % c[5:] for c in PERIODIC]


def test_calls_of_more_trips_than_an_int_counts(ask):
    """A long recursion on a long strip (hours of work): its trips overflowed
    the kernel's count, and nothing beyond the first moments was written."""
    call = "route 8 1000000 0 0 1 0 512 %d 0 1"
    assert ask([call % 20000, call % 200000]) == ["gpipe", "steps"]
