"""GPU parity of the streaming pipelines at the places where their loops, tiles
and pass lists end: every fused depth with every remainder of the loop trip,
bit for bit against the one-step kernel (same point order, same chain), which
itself is checked against the FP64 oracle."""
import numpy as np
import pytest

import synth
from gpu_helpers import check, gpu_sweep, oracle_ref

pytestmark = pytest.mark.gpu


def _weights(offsets, seed, dtype):
    r = np.random.default_rng(seed).random(len(offsets))
    return synth.adjust_centre(r / r.sum(), "f64" if dtype == "f64" else "f32")


def _against_naive(plan, naive, u0, offs, w, steps, bc, dtype, select=None, what=""):
    print(f"{what} steps {steps}", flush=True)
    got, _ = gpu_sweep(u0, offs, w, steps, bc, dtype, select=select, plan=plan)
    one, _ = gpu_sweep(u0, offs, w, steps, bc, dtype, plan=naive)
    assert np.array_equal(got, one), f"{what} steps {steps}: differs from the one-step kernel"
    return one


# 2D: the rows of a chunk over the loop trip (4 rows, 6 at radius 2) leave every
# remainder, chunks that touch neither edge take the loop without ghost-row
# tests (several chunks of 8 rows), and the step counts bring every depth
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern,radius", [("star", 1), ("box", 1), ("star", 2), ("box", 2)])
@pytest.mark.parametrize("ny", [1, 6, 43, 90])
def test_2d_every_depth_and_row_remainder(dtype, bc, pattern, radius, ny):
    import paper_2303_08365_amd as st
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(2, radius)
    w = _weights(offs, 31, dtype)
    shape = (ny, 260)  # whole-vector rows, two strips
    u0 = synth.uniform_field(shape, seed=32)
    plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
    top = max(c["tb"] for c in plan.candidates() if not c["tessellated"])
    chunks = {c["tile_y"]: k for k, c in enumerate(plan.candidates())
              if c["kernel"] == st.KERNEL_STREAM2D and c["tb"] == top and not c["tessellated"]}
    for rows, k in sorted(chunks.items())[:3]:
        for steps in [top + d for d in range(1, top + 1)] + [2 * top]:
            one = _against_naive(plan, naive, u0, offs, w, steps, bc, dtype, {"variant": k},
                                 f"{dtype} {bc} {pattern}{radius} ny {ny} chunk {rows}")
    check(one, oracle_ref(u0, offs, w, steps, bc, dtype), dtype, steps, "one-step kernel")


def _offset_view(u0, dtype):
    """The field on the device, one element past the allocation's start."""
    import torch
    t = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    base = torch.zeros(u0.size + 1, dtype=t, device="cuda")
    g = base[1:].view(u0.shape)
    g.copy_(torch.from_numpy(u0).to(t))
    return g


# 2D rows whose length the lane width does not divide, in whole vectors: one
# column more and less than a strip (64 lanes x 2 or 4 columns) and than two,
# the last strip a lane wide or less, periodic rows too short for two strips
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern,radius", [("star", 1), ("box", 2)])
def test_2d_rows_of_any_length(dtype, bc, pattern, radius):
    import paper_2303_08365_amd as st
    import torch
    from gpu_helpers import to_host
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(2, radius)
    w = _weights(offs, 33, dtype)
    for nx in [19, 45, 127, 129, 131, 226, 241, 243, 255, 257, 259, 262, 381, 495, 511, 513, 517]:
        shape = (23, nx)
        u0 = synth.uniform_field(shape, seed=nx)
        plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
        depths = {c["tb"]: k for k, c in reversed(list(enumerate(plan.candidates())))
                  if c["kernel"] == st.KERNEL_STREAM2D and not c["tessellated"]}
        for tb, k in sorted(depths.items()):
            _against_naive(plan, naive, u0, offs, w, 2 * tb + 1, bc, dtype, {"variant": k}, f"{dtype} {bc} nx {nx} tb {tb}")
        # buffers that are aligned to an element only
        g, work, ref = _offset_view(u0, dtype), _offset_view(u0, dtype), _offset_view(u0, dtype)
        plan.run(g, list(w), 5, work=work)
        naive.run(ref, list(w), 5)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(g), to_host(ref)), f"{dtype} {bc} nx {nx}: element-aligned buffers"


# 3D rows whose length the lane width does not divide, in whole vectors: grids
# one register tile wide and high or a little more (64 lanes x 2 or 4 columns,
# 24 to 64 rows), several tiles, periodic rows too short for two tiles
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern,radius", [("star", 1), ("star", 4), ("box", 1)])
def test_3d_rows_of_any_length(dtype, bc, pattern, radius):
    import paper_2303_08365_amd as st
    import torch
    from gpu_helpers import to_host
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(3, radius)
    w = _weights(offs, 35, dtype)
    for nz, ny, nx in [(5, 33, 45), (9, 64, 129), (7, 49, 193), (10, 66, 257), (3, 35, 259), (6, 65, 395)]:
        shape = (nz, ny, nx)
        u0 = synth.uniform_field(shape, seed=nx)
        plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
        forms = {(c["kernel"], c["tb"], c["block"], c["tile_x"], c["tile_y"], c["pipeline"]): k
                 for k, c in reversed(list(enumerate(plan.candidates()))) if c["kernel"] != st.KERNEL_NAIVE}
        for form, k in sorted(forms.items()):
            _against_naive(plan, naive, u0, offs, w, 2 * form[1], bc, dtype, {"variant": k}, f"{dtype} {bc} {shape} {form}")
        g, work, ref = _offset_view(u0, dtype), _offset_view(u0, dtype), _offset_view(u0, dtype)
        plan.run(g, list(w), 5, work=work)
        naive.run(ref, list(w), 5)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(g), to_host(ref)), f"{dtype} {bc} {shape}: element-aligned buffers"


# 1D grids whose length the 16 cells of a lane do not divide: one strip (1024
# cells) and a little more, the last strip short, each fused depth
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("radius", [1, 2])
def test_1d_any_length(dtype, bc, radius):
    import paper_2303_08365_amd as st
    offs = synth.star_offsets(1, radius)
    w = _weights(offs, 37, dtype)
    for n in [1023, 1024, 1025, 1039, 1793, 1923, 2049, 5003]:
        u0 = synth.uniform_field((n,), seed=n)
        plan, naive = st.Plan(offs, (n,), dtype, bc), st.Plan(offs, (n,), dtype, bc, naive=True)
        for k, c in enumerate(plan.candidates()):
            _against_naive(plan, naive, u0, offs, w, 2 * c["tb"] + 1, bc, dtype, {"variant": k}, f"{dtype} {bc} n {n} tb {c['tb']}")


# the one-step kernel: rows of one, two and four columns a lane with remainders,
# point counts that leave every kind of last batch, offsets of a whole extent
# and beyond it under the periodic rule
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("npoints", [1, 2, 15, 17, 33, 125])
def test_one_step_kernel_rows_and_batches(dtype, bc, npoints):
    import paper_2303_08365_amd as st
    box = synth.box_offsets(3, 2)
    far = [(4, 0, 0), (0, -4, 0), (0, 0, 4), (-3, 2, -4)]
    offs = (box if npoints == 125 else box[:1] + (far + box[1:])[:npoints - 1])
    w = _weights(offs, 39, dtype)
    for shape in [(3, 5, 1), (2, 3, 63), (4, 6, 64), (5, 4, 65), (1, 9, 129), (6, 2, 257), (4, 4, 515)]:
        u0 = synth.uniform_field(shape, seed=shape[2])
        print(f"one step {dtype} {bc} {npoints} points {shape}", flush=True)
        got, _ = gpu_sweep(u0, offs, w, 3, bc, dtype, plan=st.Plan(offs, shape, dtype, bc, naive=True))
        check(got, oracle_ref(u0, offs, w, 3, bc, dtype), dtype, 3, f"{shape}")


# plans that choose for themselves, from grids of a few cells (one step per
# launch) to ones that fill the device with tiles: eager, replayed from a graph,
# and after a selection by the caller
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("pattern,radius,shapes", [
    ("star", 1, [(7,), (700,), (40000,), (9, 9), (200, 333), (1111, 640), (12, 13, 14), (40, 64, 131), (70, 130, 260)]),
    ("box", 1, [(64, 64), (513, 1027), (20, 30, 40), (33, 70, 200)]),
    ("star", 4, [(16, 20, 24), (30, 64, 300)])])
def test_plans_that_choose_for_themselves(dtype, pattern, radius, shapes):
    import paper_2303_08365_amd as st
    for shape in shapes:
        offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(len(shape), radius)
        w = _weights(offs, 41, dtype)
        u0 = synth.uniform_field(shape, seed=42)
        naive = st.Plan(offs, shape, dtype, "zero", naive=True)
        for graph in (False, True):
            plan = st.Plan(offs, shape, dtype, "zero", graph=graph)
            _against_naive(plan, naive, u0, offs, w, 13, "zero", dtype, what=f"{dtype} {shape} graph {graph}")
            _against_naive(plan, naive, u0, offs, w, 13, "zero", dtype, {"variant": 0}, f"{dtype} {shape} selected")


# grids where the edge tiles own their outer halo because that saves a tile: one
# cell around every such width and height, and the outflow account over them
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("pattern", ["star", "box"])
@pytest.mark.parametrize("shape", [(6, 34, 128), (9, 58, 248), (5, 60, 249), (7, 64, 256), (6, 90, 500), (4, 118, 505),
                                   (40, 128), (33, 248), (21, 256), (30, 500), (17, 737)])
def test_edge_tiles_own_their_outer_halo(dtype, pattern, shape):
    import torch
    import oracle
    import paper_2303_08365_amd as st
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(len(shape), 1)
    w = _weights(offs, 43, dtype)
    u0 = synth.uniform_field(shape, seed=44)
    plan, naive = st.Plan(offs, shape, dtype, "zero"), st.Plan(offs, shape, dtype, "zero", naive=True)
    forms = {(c["kernel"], c["tb"], c["block"], c["tile_x"], c["tile_y"], c["pipeline"]): k
             for k, c in reversed(list(enumerate(plan.candidates()))) if c["kernel"] != st.KERNEL_NAIVE and not c["tessellated"]}
    for form, k in sorted(forms.items()):
        _against_naive(plan, naive, u0, offs, w, 2 * form[1], "zero", dtype, {"variant": k}, f"{dtype} {shape} {form}")
    from gpu_helpers import to_device
    g, flux = to_device(u0, dtype), torch.zeros(1, dtype=torch.float64, device="cuda")
    st.Plan(offs, shape, dtype, "zero").run_flux(g, list(w), 7, flux)
    _, ref = oracle.sweep_flux(synth.round_to(u0, dtype), offs, synth.round_to(np.asarray(w), "f64" if dtype == "f64" else "f32"), 7)
    tol = {"f64": 1e-12, "f32": 1e-5, "bf16": 7 * 2.0 ** -8}[dtype]
    assert abs(float(flux.cpu()[0]) - ref) <= tol * max(abs(ref), 1.0), (float(flux.cpu()[0]), ref)


def _varcoef(u0, k, y, dtype, steps, every, naive):
    """Forward with checkpoints and both gradients, every buffer one element off."""
    import torch
    import paper_2303_08365_amd as st
    plan = st.varcoef_plan(u0.shape, dtype, naive=naive)
    g, kk, lam, gk = (_offset_view(f, dtype) for f in (u0, k, y, 0.1 * y))
    ck = [torch.full_like(g, float("nan")) for _ in range(-(-steps // every))]
    plan.run_ckpt(g, kk, 0.1, steps, torch.full_like(g, float("nan")), every=every, ckpts=ck)
    seg = torch.full((max(min(every, steps) - 1, 1),) + u0.shape, float("nan"), dtype=g.dtype, device="cuda")
    plan.adjoint(lam, steps, torch.full_like(g, float("nan")), k=kk, alpha=0.1, ckpts=ck, every=every, grad_k=gk, seg=seg)
    return [t.cpu().numpy() for t in (g, *ck, lam, gk)]


# two steps per pass against the one-cell-per-thread kernels, bit for bit (every
# kernel takes a cell's faces in the same order): the smallest grids of each
# lane width (4, 2, 1 columns; 16 or 32 rows), one plane, fewer planes than a
# pass re-streams, ragged tiles, rows of any length (forward only), and step
# counts and intervals that leave every mix of single and paired steps
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(1, 32, 64), (2, 33, 65), (3, 16, 128), (5, 62, 130), (9, 63, 256), (6, 95, 252),
                                   (17, 40, 509), (33, 32, 512)])
def test_varcoef_two_steps_per_pass(dtype, shape):
    rng = np.random.default_rng(5)
    u0, k, y = rng.random(shape), 0.5 + rng.random(shape), rng.random(shape)
    for steps, every in [(2, 2), (3, 1), (5, 2), (7, 3), (8, 8)]:
        print(f"varcoef {dtype} {shape} steps {steps} every {every}", flush=True)
        got = _varcoef(u0, k, y, dtype, steps, every, False)
        want = _varcoef(u0, k, y, dtype, steps, every, True)
        for i, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b), f"buffer {i} of {len(got)}"


# small 2D grids in register tiles (64 rows, 64 to 256 columns, up to 31 steps a
# pass): the smallest grids they take, one row or column more, tiles moved
# inward, edge tiles with their own halo, several tiles, rows off the lane grid,
# and step counts below, at and past a pass's depth, against the one-step kernel
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern", ["star", "box"])
@pytest.mark.parametrize("shape", [(64, 64), (65, 131), (66, 256), (97, 257), (256, 260), (130, 515)])
def test_2d_small_grids_in_register_tiles(dtype, bc, pattern, shape):
    import paper_2303_08365_amd as st
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(2, 1)
    w = _weights(offs, 51, dtype)
    u0 = synth.uniform_field(shape, seed=52)
    plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
    for steps in (1, 2, 5, 16, 33, 64):
        one = _against_naive(plan, naive, u0, offs, w, steps, bc, dtype, None, f"tiles {dtype} {bc} {pattern} {shape}")
    check(one, oracle_ref(u0, offs, w, steps, bc, dtype), dtype, steps, "one-step kernel")


# small 3D grids in register bricks (16 rows, 16 planes, 64 or 128 columns, up to 7
# steps a pass): the smallest grids they take, one cell more per axis, edge bricks
# with their own halo, several bricks, rows off the lane grid, against the
# one-step kernel
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("shape", [(16, 16, 64), (17, 18, 65), (16, 33, 128), (40, 21, 131), (64, 64, 64), (30, 50, 190)])
def test_3d_small_grids_in_register_bricks(dtype, bc, shape):
    import paper_2303_08365_amd as st
    offs = synth.star_offsets(3, 1)
    w = _weights(offs, 61, dtype)
    u0 = synth.uniform_field(shape, seed=62)
    plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
    for steps in (1, 2, 5, 7, 16, 30):
        one = _against_naive(plan, naive, u0, offs, w, steps, bc, dtype, None, f"bricks {dtype} {bc} {shape}")
    check(one, oracle_ref(u0, offs, w, steps, bc, dtype), dtype, steps, "one-step kernel")


# an infinite value inside the grid reaches the same cells, as the same values,
# through one pass of two steps as through two of one
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_varcoef_infinite_value_inside(dtype):
    shape = (9, 95, 512)
    rng = np.random.default_rng(7)
    u0, k, y = rng.random(shape), 0.5 + rng.random(shape), rng.random(shape)
    u0[4, 50, 200] = np.inf
    got, want = (_varcoef(u0, k, y, dtype, 2, 2, naive) for naive in (False, True))
    for i, (a, b) in enumerate(zip(got, want)):
        assert np.array_equal(a, b, equal_nan=True), f"buffer {i}"


# the same tiles at radius 2 (two edge rows a wave, two columns from the next lane)
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern", ["star", "box"])
@pytest.mark.parametrize("shape", [(64, 128), (65, 257), (66, 256), (130, 260), (256, 515)])
def test_2d_small_grids_in_register_tiles_radius_2(dtype, bc, pattern, shape):
    import paper_2303_08365_amd as st
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(2, 2)
    w = _weights(offs, 71, dtype)
    u0 = synth.uniform_field(shape, seed=72)
    plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
    for steps in (1, 2, 5, 15, 16, 31):
        one = _against_naive(plan, naive, u0, offs, w, steps, bc, dtype, None, f"tiles r2 {dtype} {bc} {pattern} {shape}")
    check(one, oracle_ref(u0, offs, w, steps, bc, dtype), dtype, steps, "one-step kernel")
