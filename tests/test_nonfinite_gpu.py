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
