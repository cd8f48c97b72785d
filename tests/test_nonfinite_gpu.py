"""Infinite values reach the same cells, as the same values, through every tiling
and depth as through the kernels that take one step and one cell at a time:
nothing that lies outside the grid or another tile is multiplied by 0."""
import numpy as np
import pytest

import synth
from gpu_helpers import gpu_sweep

pytestmark = pytest.mark.gpu


def _weights(offsets, seed, dtype):
    r = np.random.default_rng(seed).random(len(offsets))
    return synth.adjust_centre(r / r.sum(), "f64" if dtype == "f64" else "f32")


# one infinity on a face, edge or corner of the grid or inside, at every fused
# depth: planes and rows beside it that lie outside the grid stay 0
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("pattern,radius,shape", [
    ("star", 1, (9, 66, 257)), ("star", 1, (33, 64, 256)), ("star", 4, (9, 66, 259)), ("box", 1, (9, 66, 257)),
    ("star", 1, (70, 259)), ("box", 2, (70, 259)), ("star", 2, (2049,))])
def test_infinite_values_at_the_faces(dtype, bc, pattern, radius, shape):
    import paper_2303_08365_amd as st
    offs = (synth.star_offsets if pattern == "star" else synth.box_offsets)(len(shape), radius)
    w = _weights(offs, 81, dtype)
    plan, naive = st.Plan(offs, shape, dtype, bc), st.Plan(offs, shape, dtype, bc, naive=True)
    forms = {(c["kernel"], c["tb"], c["block"], c["tile_x"], c["tile_y"], c["pipeline"], c["tessellated"]): k
             for k, c in reversed(list(enumerate(plan.candidates())))}
    mid = tuple(n // 2 for n in shape)
    places = [tuple(0 for _ in shape), tuple(n - 1 for n in shape), mid]
    for d in range(len(shape)):
        places += [mid[:d] + (0,) + mid[d + 1:], mid[:d] + (shape[d] - 1,) + mid[d + 1:]]
    for at in places:
        u0 = synth.uniform_field(shape, seed=82)
        u0[at] = np.inf
        print(f"infinity {dtype} {bc} {pattern}{radius} {shape} at {at}", flush=True)
        ref = {}
        for form, k in sorted(forms.items()):
            steps = 2 * min(form[1], 8)
            if steps not in ref:
                ref[steps] = gpu_sweep(u0, offs, w, steps, bc, dtype, plan=naive)[0]
            got, _ = gpu_sweep(u0, offs, w, steps, bc, dtype, select={"variant": k}, plan=plan)
            assert np.array_equal(got, ref[steps], equal_nan=True), f"{form} at {at}"
        own, _ = gpu_sweep(u0, offs, w, 8, bc, dtype, plan=st.Plan(offs, shape, dtype, bc))
        ref8 = ref.get(8, None)
        if ref8 is None:
            ref8 = gpu_sweep(u0, offs, w, 8, bc, dtype, plan=naive)[0]
        assert np.array_equal(own, ref8, equal_nan=True), f"the plan's own choice at {at}"


def _varcoef(u0, k, y, alpha, dtype, steps, naive):
    """Forward with a checkpoint at the start, and both gradients."""
    import torch
    import paper_2303_08365_amd as st
    t = {"f64": torch.float64, "f32": torch.float32}[dtype]
    plan = st.varcoef_plan(u0.shape, dtype, naive=naive)
    g, kk, lam = (torch.from_numpy(a).to("cuda", t) for a in (u0, k, y))
    gk, ck = torch.zeros_like(g), [torch.empty_like(g)]
    plan.run_ckpt(g, kk, alpha, steps, torch.empty_like(g), every=steps, ckpts=ck)
    seg = torch.empty((max(steps - 1, 1),) + u0.shape, dtype=t, device="cuda")
    plan.adjoint(lam, steps, torch.empty_like(g), k=kk, alpha=alpha, ckpts=ck, every=steps, grad_k=gk, seg=seg)
    return [a.cpu().numpy() for a in (g, lam, gk)]


# variable coefficients: an infinite state or cotangent on a face, edge or corner
# or inside, through single steps (1), pairs (2) and both (3).  The other field
# has an extremum in that cell, and the negative diffusion number keeps the
# infinity one, so that dL/dk there is an infinity that any stray 0 * inf or inf -
# inf would turn into NaN.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("what", ["u", "lambda"])
@pytest.mark.parametrize("shape", [(9, 95, 512), (7, 64, 100), (60, 96, 252)])
def test_varcoef_infinite_values_at_the_faces(dtype, what, shape):
    rng = np.random.default_rng(83)
    k = 0.5 + rng.random(shape)
    mid = tuple(n // 2 for n in shape)
    places = [tuple(0 for _ in shape), tuple(n - 1 for n in shape), mid]
    for d in range(3):
        places += [mid[:d] + (0,) + mid[d + 1:], mid[:d] + (shape[d] - 1,) + mid[d + 1:]]
    for at in places:
        u0, y = rng.random(shape), rng.random(shape)
        if what == "u":
            u0[at], y[at] = np.inf, 10.0
        else:
            u0[at], y[at] = -10.0, np.inf
        for steps in (1, 2, 3):
            print(f"varcoef infinity {dtype} {what} {shape} at {at} steps {steps}", flush=True)
            got, want = (_varcoef(u0, k, y, -0.1, dtype, steps, naive) for naive in (False, True))
            if what == "lambda" and steps == 1:
                assert np.isinf(want[2][at]), "the case tells nothing"
            for i, (a, b) in enumerate(zip(got, want)):
                assert np.array_equal(a, b, equal_nan=True), f"buffer {i}: {np.argwhere(~((a == b) | (np.isnan(a) & np.isnan(b))))[:4]}"


# conductivities whose sum overflows where their mean does not: the same bits as
# with k times 2^-8 and the diffusion number times 2^8, and as in the one-cell form
@pytest.mark.parametrize("dtype,big,small", [("f64", 1023, -300), ("f32", 127, -40)])
@pytest.mark.parametrize("shape", [(9, 95, 512), (7, 64, 100)])
def test_varcoef_largest_conductivities(dtype, big, small, shape):
    rng = np.random.default_rng(84)
    k = (1.0 + 0.999 * rng.random(shape)) * 2.0 ** big  # the type's last binade
    u0, y = rng.random(shape) * 2.0 ** small, rng.random(shape) * 2.0 ** small
    alpha = 2.0 ** (3 - big)
    for steps in (1, 2, 3):
        print(f"varcoef largest k {dtype} {shape} steps {steps}", flush=True)
        got, want = (_varcoef(u0, k, y, alpha, dtype, steps, naive) for naive in (False, True))
        scaled = _varcoef(u0, k * 2.0 ** -8, y, alpha * 2.0 ** 8, dtype, steps, False)
        for i in range(3):
            assert np.array_equal(got[i], want[i]), f"buffer {i}"
        for i in range(2):
            assert np.isfinite(got[i]).all() and np.array_equal(got[i], scaled[i]), f"buffer {i} of the scaled problem"
