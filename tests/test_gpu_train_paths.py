"""The training kernels run other tiles (64 or 128 vertices a workgroup, one
launch or two) by the batch's size. A batch on either side of each switch
against the sum of its 64-vertex parts, which all take the smallest path.

A part's weights are the batch's w (1/B) times 64, so that every vertex's
gradient is the same float32 number in both and only the sums differ: a
workgroup's running sums (at most 16 products a tile and some tens of tiles)
and the tree over the workgroups. 512 units (2^-24) of the parts' magnitudes,
in the norm of each tensor, allow for all of it; a tile that is left out,
counted twice or read from another place is off by at least one part in the
number of tiles (1/800 here, 40 times that).
"""

import numpy as np
import pytest
import torch

from paper_2303_08064_amd import synth
from tests.helpers import make_guide, to_dev

pytestmark = pytest.mark.gpu

# batch sizes as (tiles of 64 per CU, vertices more): one round of 64-vertex
# tiles (or half of one), the first batch past it, two rounds and three
HALF, ONE, TWO, THREE = (0.5, 0), (1, 0), (2, 0), (2, 65)
CASES = {
    "c1_f32": [(0, 1), ONE, (1, 1), TWO, THREE],
    "c2_f32": [(0, 63), ONE, (1, 1), TWO, THREE, (3, 1)],
    "c2s_f32": [(1, 129)],
    "c3_f32": [(1, 1)],
    "c1_bf16": [(0, 65), HALF, (0.5, 1), (1, 1)],
    "c2_bf16": [HALF, (0.5, 1)],
    "c3_bf16": [(0.5, 1), ONE, (1, 1)],
    "c3s_bf16": [ONE, (1, 65)],
    "c5_bf16": [ONE, (1, 1), (2, 129)],
    "paper_bf16": [ONE, (1, 1), (2, 129)],
}


@pytest.mark.parametrize("name", CASES)
def test_gradient_is_the_sum_of_its_parts(name):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g, _ = make_guide(name, out_scale=2.0)
    for per_cu, more in CASES[name]:
        B = int(64 * cus * per_cu) + more
        rng = synth.rng_for(5)
        feat, dirs = to_dev(synth.features(B, rng)), to_dev(synth.unit_vectors(B, rng).T.astype(np.float32))
        w = synth.radiance_weights(B, rng).astype(np.float32)
        pfs = to_dev(rng.uniform(0.05, 1.0, B).astype(np.float32)) if g.selection else None
        g.loss_grad(feat, dirs, to_dev(w), pfs)
        got = [m.double() for m in g.split(g.grad.clone())]
        scaled = to_dev(w * (np.float32(1) / np.float32(B)) * np.float32(64))
        n = (B + 63) // 64
        at = torch.arange(64, device="cuda")
        total, mag = [torch.zeros_like(m) for m in got], [torch.zeros_like(m) for m in got]
        for t in range(n):
            i = (64 * t + at).clamp(max=B - 1)
            part_w = scaled[i] * (64 * t + at < B)      # weight 0: the part's padding adds nothing
            g.loss_grad(feat[:, i].contiguous(), dirs[:, i].contiguous(), part_w, None if pfs is None else pfs[i])
            for a, b, m in zip(total, mag, g.split(g.grad)):
                a += m.double()
                b += m.double().abs()
        for layer, (x, ref, s) in enumerate(zip(got, total, mag)):
            err, allowed = float((x - ref).norm()), 512 * 2.0 ** -24 * float(s.norm())
            assert err <= allowed, (name, B, layer, err, allowed)
