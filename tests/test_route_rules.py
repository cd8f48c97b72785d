"""Host checks of what the run calls route where, and of rules that the kernels'
sources have to keep."""
import os
import re
import time

import pytest

import paper_2303_08365_amd as st
import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2303_08365_amd", "csrc")


# the 1D strips hand their pieces from lane to lane through LDS without a barrier:
# the source orders every change between writing and reading
def test_1d_strips_order_their_lds_accesses():
    src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "stream1d.hip")).read())
    kinds = re.findall(r"(\blds\[[^;]*?\]\s*=[^=])|(=\s*lds\[)|(wave_lds_order\(\);)|(static __device__[^;{]*?u32x4\* lds)", src)
    ops = ["write" if w else "read" if r else "order" if o else "function" for w, r, o, _ in kinds]
    assert ops.count("write") == 2 and ops.count("read") == 2
    last = None  # the first access of a function follows those of whatever ran before
    for op in ops:
        if op == "function" and last != "start":
            last = "start" if last is None else "before"
        elif op in ("write", "read"):
            assert last in ("start", "order", op), f"{op} after {last} with nothing that orders them"
            last = op
        elif op == "order":
            last = "order"


# no heat leaves a periodic grid: an outflow run launches what a plain run does,
# register tiles and bricks and one step per launch included
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("pattern,shape", [(synth.star_offsets, (100, 256)), (synth.box_offsets, (66, 64)), (synth.star_offsets, (9, 9)),
                                           (synth.star_offsets, (32, 32, 64)), (synth.star_offsets, (12, 13, 14)),
                                           (synth.star_offsets, (89, 97, 101)), (synth.star_offsets, (512, 512, 512))])
def test_periodic_outflow_runs_launch_what_plain_runs_do(dtype, pattern, shape):
    plan = st.Plan(pattern(len(shape), 1), shape, dtype, "periodic")
    assert plan.launches("flux") == plan.launches("run")
    plan.select(variant=1)
    assert plan.launches("flux") == plan.launches("run")


# a chunk length asked for by the environment is what runs, on small grids too
@pytest.mark.parametrize("shape,kernel,axis", [((512, 512), st.KERNEL_STREAM2D, "tile_y"), ((64, 64, 64), st.KERNEL_STREAM3D, "tile_z"),
                                               ((20, 40, 70), st.KERNEL_STREAM3D, "tile_z")])
def test_chunk_length_from_the_environment_runs(monkeypatch, shape, kernel, axis):
    monkeypatch.setenv("STENCIL_CHUNK", "16")
    for dtype in ("f64", "f32", "bf16"):
        ran = st.Plan(synth.star_offsets(len(shape), 1), shape, dtype).launches()
        assert ran["kernel"] == kernel and ran[axis] == 16, (dtype, ran)


# making a plan searches a chunk length per tiling: against a plan that has nothing
# to search (one step per launch), 8 to 9 times the time where it was 19 to 24 with
# every trial length priced in full, for the transposed sweep's plan once more
@pytest.mark.parametrize("shape", [(512, 512, 512), (251, 319, 377)])
def test_a_plan_costs_a_bounded_search(shape):
    def least(**kw):
        best = float("inf")
        for _ in range(60):
            t = time.perf_counter()
            plan = st.Plan(synth.star_offsets(3, 1), shape, "f64", **kw)
            best = min(best, time.perf_counter() - t)
            plan.close()
        return best
    ratios = []
    for _ in range(5):  # a loaded machine: the least of a few
        ratios.append(least() / least(naive=True))
        if ratios[-1] < 14:
            return
    raise AssertionError(f"times a plan without a search: {ratios}")


# the transposed sweep takes the tilings that the plan's own choice takes, whatever
# the caller or the autotuner selects afterwards
def test_the_transposed_sweep_keeps_the_models_choice():
    for offs, shape in [(synth.star_offsets(3, 1), (96, 97, 98)), (synth.box_offsets(2, 2), (300, 900)), ([(0, 0), (0, 1), (-2, 0)], (50, 50))]:
        plan = st.Plan(offs, shape, "f32", "periodic")
        own = plan.launches()
        assert plan.launches("adjoint") == own
        plan.select(variant=len(plan.candidates()) - 1)
        assert plan.launches("adjoint") == own


# the two-step variable-coefficient passes try each count of chunks once: a call
# on a long grid spends microseconds there, not a division per plane (half a
# second at 10^8 planes)
def test_variable_coefficient_chunks_of_a_long_grid():
    plan = st.varcoef_plan((10 ** 8, 32, 64), "f32")
    best = float("inf")
    for _ in range(3):
        t = time.perf_counter()
        ran = plan.launches()
        best = min(best, time.perf_counter() - t)
    assert ran["tb"] == 2 and best < 0.02, best
    # every length that a search over all of them takes
    for nz in (1, 2, 7, 63, 64, 100, 257, 1000, 4099):
        for ny, nx in ((32, 64), (95, 512), (300, 1000)):
            got = {c: st.varcoef_plan((nz, ny, nx), "f32").launches(c)["tile_z"] for c in ("run", "adjoint")}
            for call, z in got.items():
                chunks = -(-nz // z)
                assert z == nz or -(-nz // (z + 1)) < chunks, (nz, call, z)  # the longest with that count


# what an outflow run takes is searched once per selection, not by every call: the
# question costs what it does for a plain run (several times that, searched)
@pytest.mark.parametrize("shape", [(512, 512), (64, 64, 64), (251, 319, 377)])
def test_outflow_runs_do_not_search_on_every_call(shape):
    plan = st.Plan(synth.star_offsets(len(shape), 1), shape, "f32")

    def least(call):
        best = float("inf")
        for _ in range(300):
            t = time.perf_counter()
            plan.launches(call)
            best = min(best, time.perf_counter() - t)
        return best
    before = plan.launches("flux")
    ratios = []
    for _ in range(5):  # a loaded machine: the least of a few
        ratios.append(least("flux") / least("run"))
        if ratios[-1] < 2.5:
            break
    else:
        raise AssertionError(ratios)
    plan.select(variant=5)
    assert plan.launches("flux") != before  # a selection is looked at again
    assert plan.launches("flux")["tb"] == plan.candidates()[5]["tb"]
