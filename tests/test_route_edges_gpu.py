"""Calls at the edges of the rules that choose a kernel."""
import ctypes

import numpy as np
import pytest

import synth
from gpu_helpers import gpu_sweep, to_device, to_host
from test_pipeline_edges_gpu import _offset_view, _varcoef, _weights

pytestmark = pytest.mark.gpu


# FP64 buffers at 4-byte boundaries (a caller's byte arithmetic): only the
# one-cell kernels take them, with the result that aligned buffers give
@pytest.mark.parametrize("shape", [(9, 95, 512), (60, 96, 130)])
def test_varcoef_buffers_off_the_element(shape):
    import torch
    import paper_2303_08365_amd as st
    lib, rng, n = st.library(), np.random.default_rng(91), int(np.prod(shape))
    plan = st.varcoef_plan(shape, "f64")
    fields = [rng.random(shape), 0.5 + rng.random(shape), rng.random(shape)]
    steps, every = 5, 3

    def run(off):
        bufs = [torch.zeros(8 * n + 8, dtype=torch.uint8, device="cuda") for _ in range(9)]  # u, k, lambda, work, grad, 2 checkpoints, 2 states
        seg = torch.zeros(16 * n + 8, dtype=torch.uint8, device="cuda")
        for b, f in zip(bufs, fields):
            b[off:off + 8 * n].copy_(torch.from_numpy(f.reshape(-1).view(np.uint8)))
        u, k, lam, work, grad, c0, c1 = (b.data_ptr() + off for b in bufs[:7])
        ck = (ctypes.c_void_p * 2)(c0, c1)
        print(f"varcoef {shape} buffers at +{off}", flush=True)
        assert lib.stencil_run_ckpt(plan._h, u, work, k, 0.1, steps, every, ck, None) == 0
        assert lib.stencil_adjoint_run(plan._h, k, 0.1, None, ck, every, steps, lam, grad, seg.data_ptr() + off, work, None) == 0
        torch.cuda.synchronize()
        return [b[off:off + 8 * n].cpu().numpy().view(np.float64) for b in (bufs[0], bufs[2], bufs[4], bufs[5], bufs[6])]

    for a, b in zip(run(4), run(0)):
        assert np.array_equal(a, b)


def _tiles_against_naive(shape, offs, dtype, bc, kernel, columns, depths):
    """Every depth of the register tiles at one lane width, selected by name, over
    step counts of one pass, two, an uneven last one and an odd count of passes."""
    import paper_2303_08365_amd as st
    w, u0 = _weights(offs, 92, dtype), synth.uniform_field(shape, seed=93)
    plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
    ref = {}
    for t in depths:
        plan.select(kernel=kernel, tb=t, variant=columns)
        ran = plan.launches()
        assert (ran["kernel"], ran["tb"], ran["pipeline"]) == (kernel, t, columns)
        for steps in (t, 2 * t, 3 * t, 2 * t + 1):
            print(f"tiles {kernel} {dtype} {bc} {len(offs)} points {shape} depth {t} columns {columns} steps {steps}", flush=True)
            if steps not in ref:
                ref[steps] = gpu_sweep(u0, offs, w, steps, bc, dtype, plan=naive)[0]
            got, _ = gpu_sweep(u0, offs, w, steps, bc, dtype, plan=plan)
            assert np.array_equal(got, ref[steps])
    plan.select(variant=0)
    assert plan.launches()["kernel"] != kernel


# every instance of the 2D register tiles: the smallest grids each takes, one row
# or column more, and several tiles with remainders (periodic rows are multiples
# of the lane's columns)
@pytest.mark.parametrize("dtype,radius,columns", [("f64", 1, 1), ("f64", 1, 2), ("f32", 1, 1), ("f32", 1, 2), ("bf16", 1, 4),
                                                  ("f64", 2, 2), ("f32", 2, 2), ("bf16", 2, 4)])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern", ["star", "box"])
def test_2d_register_tiles_every_instance(dtype, radius, columns, bc, pattern):
    import paper_2303_08365_amd as st
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(2, radius)
    wide = 64 * columns
    for ny, nx in [(64, wide), (65, wide + 1), (129, 2 * wide + 3), (200, 3 * wide - 5)]:
        nx -= nx % columns if bc == "periodic" else 0
        _tiles_against_naive((ny, nx), offs, dtype, bc, st.KERNEL_TILE2D, columns,
                             (1, 2, 5, 31) if radius == 1 else (1, 2, 7, 15))


# every instance of the 3D register bricks
@pytest.mark.parametrize("dtype,columns", [("f64", 1), ("f32", 1), ("f32", 2)])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
def test_3d_register_bricks_every_instance(dtype, columns, bc):
    import paper_2303_08365_amd as st
    wide = 64 * columns
    for nz, ny, nx in [(16, 16, wide), (17, 18, wide + 1), (40, 21, 2 * wide + 3), (33, 50, 3 * wide - 5)]:
        nx -= nx % columns if bc == "periodic" else 0
        _tiles_against_naive((nz, ny, nx), synth.star_offsets(3, 1), dtype, bc, st.KERNEL_BRICK3D, columns, (1, 2, 3, 7))


# register tiles asked for by name: refused where no instance takes the plan, and
# the calls that they do not take run on the candidate selected before
def test_register_tiles_refused_and_passed_by():
    import torch
    import paper_2303_08365_amd as st
    star = synth.star_offsets(2, 1)
    for plan, sel in [(st.Plan(star, (63, 64), "f64"), {"kernel": st.KERNEL_TILE2D}),
                      (st.Plan(star, (64, 64), "f64"), {"kernel": st.KERNEL_TILE2D, "variant": 2}),
                      (st.Plan(star, (64, 64), "f64"), {"kernel": st.KERNEL_TILE2D, "tb": 32}),
                      (st.Plan(star, (64, 258), "bf16", "periodic"), {"kernel": st.KERNEL_TILE2D}),
                      (st.Plan(star, (64, 64), "f64", naive=True), {"kernel": st.KERNEL_TILE2D}),
                      (st.Plan(star, (64, 64), "f64"), {"kernel": st.KERNEL_BRICK3D}),
                      (st.Plan(synth.star_offsets(3, 1), (16, 16, 64), "bf16"), {"kernel": st.KERNEL_BRICK3D}),
                      (st.BatchPlan(star, [(64, 64)], "f64"), {"kernel": st.KERNEL_TILE2D}),
                      (st.varcoef_plan((16, 16, 64), "f64"), {"kernel": st.KERNEL_BRICK3D})]:
        before = plan.launches()
        with pytest.raises(st.StencilError) as e:
            plan.select(**sel)
        assert e.value.status == -2 and plan.launches() == before
    shape, w = (97, 130), list(_weights(star, 94, "f32"))
    u0 = synth.uniform_field(shape, seed=95)
    plan = st.Plan(star, shape, "f32").select(variant=3).select(kernel=st.KERNEL_TILE2D)
    assert plan.launches("flux")["variant"] == 3 and plan.info()["variant"] == 3
    ref = to_device(u0, "f32")
    st.Plan(star, shape, "f32", naive=True).run(ref, w, 9)
    g, flux = to_device(u0, "f32"), torch.zeros(1, dtype=torch.float64, device="cuda")
    plan.run_flux(g, w, 9, flux)
    assert np.array_equal(to_host(g), to_host(ref)) and float(flux.cpu()[0]) > 0.0
    h, work = _offset_view(u0, "f32"), _offset_view(u0, "f32")
    plan.run(h, w, 9, work=work)
    assert np.array_equal(to_host(h), to_host(ref))


# the two-step variable-coefficient kernels at every lane width they run with,
# forward and adjoint, against the one-cell kernels: grids large enough that the
# planner takes that width, rows of any length, ragged tiles
@pytest.mark.parametrize("dtype,shape,forward,adjoint", [
    ("f32", (60, 190, 757), 4, 1), ("f32", (60, 190, 756), 4, 4), ("f32", (64, 90, 256), 1, 4), ("f32", (50, 64, 257), 1, 1),
    ("f64", (97, 64, 64), 1, 1), ("f64", (50, 70, 127), 1, 1), ("f64", (60, 190, 757), 2, 1), ("f64", (40, 127, 380), 2, 2)])
def test_varcoef_two_steps_every_lane_width(dtype, shape, forward, adjoint):
    import paper_2303_08365_amd as st
    plan = st.varcoef_plan(shape, dtype)
    for call, columns in (("run", forward), ("adjoint", adjoint)):
        ran = plan.launches(call)
        assert (ran["kernel"], ran["tb"], ran["pipeline"]) == (st.KERNEL_VARCOEF3D, 2, columns), (call, ran)
    rng = np.random.default_rng(96)
    u0, k, y = rng.random(shape), 0.5 + rng.random(shape), rng.random(shape)
    for steps, every in [(2, 2), (5, 2), (7, 3)]:
        print(f"varcoef {dtype} {shape} steps {steps} every {every}", flush=True)
        got, want = (_varcoef(u0, k, y, dtype, steps, every, naive) for naive in (False, True))
        for i, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b), f"buffer {i} of {len(got)}"


# what the register-tile and two-step tests of other files mean to run, runs
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_small_grids_run_in_register_tiles(dtype):
    import paper_2303_08365_amd as st
    for pattern in (synth.star_offsets, synth.box_offsets):
        for radius, shapes in ((1, [(66, 256), (256, 260)]), (2, [(66, 256), (130, 260)])):
            for shape in shapes:
                for bc in ("zero", "periodic"):
                    ran = st.Plan(pattern(2, radius), shape, dtype, bc).launches()
                    assert ran["kernel"] == st.KERNEL_TILE2D and ran["variant"] == -1, (shape, bc, ran)
    if dtype != "bf16":
        for shape in [(16, 16, 64), (17, 18, 65), (64, 64, 64), (30, 50, 190)]:
            for bc in ("zero", "periodic"):
                ran = st.Plan(synth.star_offsets(3, 1), shape, dtype, bc).launches()
                assert ran["kernel"] == st.KERNEL_BRICK3D, (shape, bc, ran)


# asking for autotuning must not give less than not asking: small grids keep the
# register tiles (twice the speed of the next tiling here), in the cache file too
@pytest.mark.parametrize("shape,kernel", [((512, 512), 6), ((64, 64, 64), 7)])
def test_autotuning_knows_the_register_tiles(tmp_path, shape, kernel):
    import paper_2303_08365_amd as st
    path = tmp_path / "tune.txt"
    offs, w, u0 = synth.star_offsets(len(shape), 1), synth.heat_weights(len(shape), 0.15, "f32"), synth.uniform_field(shape, seed=97)
    st.autotune_cache(str(path))
    try:
        tuned = st.Plan(offs, shape, "f32", autotune=True)
        print(f"autotuned {shape}: {tuned.launches()}", flush=True)
        assert tuned.launches()["kernel"] == kernel
        where = " grid " + "x".join(str(n) for n in (1,) * (3 - len(shape)) + shape) + " "
        line, = [ln for ln in path.read_text().splitlines() if where in ln and " t1 " in ln]
        key, idx, n = line.split("\t")
        base, tile = key.split(" tile ")
        assert [int(v) for v in tile.split()] == [tuned.launches()["pipeline"], tuned.launches()["tb"]]
        again = st.Plan(offs, shape, "f32", autotune=True)
        assert again.launches() == tuned.launches() and again.info() == tuned.info()
        naive = st.Plan(offs, shape, "f32", naive=True)
        want, _ = gpu_sweep(u0, offs, w, 25, "zero", "f32", plan=naive)
        for plan in (tuned, again):
            got, _ = gpu_sweep(u0, offs, w, 25, "zero", "f32", plan=plan)
            assert np.array_equal(got, want)
    finally:
        st.autotune_cache(None)


# stored choices of register tiles are taken as they are; ones that no instance
# can run are tuned anew
def test_autotune_cache_names_register_tiles(tmp_path):
    import paper_2303_08365_amd as st
    path, offs, shape = tmp_path / "tune.txt", synth.star_offsets(2, 1), (130, 257)
    st.autotune_cache(str(path))
    try:
        st.Plan(offs, shape, "f32", autotune=True)
        line, = [ln for ln in path.read_text().splitlines() if " grid 1x130x257 " in ln and " t1 " in ln]
        base, n = line.split("\t")[0].split(" tile ")[0], line.split("\t")[2]
        path.write_text(f"{base} tile 1 7\t2\t{n}\n")
        # a fresh table: what this process has tuned would come first
        import subprocess
        import sys
        code = (f"import sys; sys.path[:0] = {sys.path!r}\nimport synth, paper_2303_08365_amd as st\nst.autotune_cache({str(path)!r})\n"
                f"p = st.Plan(synth.star_offsets(2, 1), {shape}, 'f32', autotune=True); r = p.launches()\n"
                "print(r['kernel'], r['pipeline'], r['tb'], p.info()['variant'])")
        got = []
        for entry in ("tile 1 7", "tile 1 99", "tile 3 7", "tile x"):
            path.write_text(f"{base} {entry}\t2\t{n}\n")
            out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
            assert out.returncode == 0, out.stderr[-2000:]
            got.append(out.stdout.split()[-4:])
        print(f"from the file: {got}", flush=True)
        assert got[0] == ["6", "1", "7", "2"]
        assert all(g[:1] == ["6"] and g[1] in ("1", "2") and int(g[2]) < 32 for g in got[1:])
    finally:
        st.autotune_cache(None)


# a number from another library's candidate list means another tiling: lines of
# the format before, and of another list with as many entries, are not taken
def test_autotune_cache_of_another_list_is_not_taken(tmp_path):
    import paper_2303_08365_amd as st
    path, offs, shape = tmp_path / "tune.txt", synth.star_offsets(1, 1), (30011,)
    st.autotune_cache(str(path))
    try:
        tuned = st.Plan(offs, shape, "f64", autotune=True)
        line, = [ln for ln in path.read_text().splitlines() if " grid 1x1x30011 " in ln]
        key, idx, n = line.split("\t")
        version, listed, rest = key.split(" ", 2)
        assert version == "v2" and len(listed) == 16 and int(n) == tuned.info()["ncandidates"]
        st.Plan(offs, (30012,), "f64", autotune=True)  # the same list: the same name
        assert any(ln.startswith(f"v2 {listed} ") and " grid 1x1x30012 " in ln for ln in path.read_text().splitlines())
        # shape 30013 is not in the table: only what the file says could be taken
        other = rest.replace("1x1x30011", "1x1x30013")
        wrong = int(n) - 1  # one step per launch: the slowest by far
        path.write_text(f"v1 {other}\t{wrong}\t{n}\nv2 {listed[::-1]} {other}\t{wrong}\t{n}\n")
        st.autotune_cache(str(path))
        assert st.Plan(offs, (30013,), "f64", autotune=True).info()["kernel"] == st.KERNEL_STREAM1D
        other = rest.replace("1x1x30011", "1x1x30014")
        path.write_text(f"v2 {listed} {other}\t{wrong}\t{n}\n")
        st.autotune_cache(str(path))
        assert st.Plan(offs, (30014,), "f64", autotune=True).info()["variant"] == wrong
    finally:
        st.autotune_cache(None)
