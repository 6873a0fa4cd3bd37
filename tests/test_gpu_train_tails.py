"""The vertices at the edges of the training kernels' tiles and batches: every
weight is 0 but those of the first and last vertices and of the two at each
switch, so that a vertex that is lost, counted twice or read from another place
is an error of the size of the gradient itself."""

import pytest
import torch

from paper_2303_08064_amd import synth
from tests.helpers import make_guide, to_dev
from tests.test_gpu_train_paths import CASES

pytestmark = pytest.mark.gpu


def _inputs(g, B, seed=6):
    rng = synth.rng_for(seed)
    feat, dirs = to_dev(synth.features(B, rng)), to_dev(synth.unit_vectors(B, rng).T.astype("float32"))
    pfs = to_dev(rng.uniform(0.05, 1.0, B).astype("float32")) if g.selection else None
    return feat, dirs, pfs


@pytest.mark.parametrize("name", CASES)
def test_gradient_of_the_tail_vertices(name):
    """Against the sum of the vertices' own gradients, each from a batch of 64
    with one nonzero weight (scaled so that dL/dlog q is the same float32
    number). A sum of at most eight vertices in another order: 16 units (2^-24)
    of the magnitudes."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g, _ = make_guide(name, out_scale=2.0)
    for per_cu, more in CASES[name] + [(4, 1), (5, 63)]:
        B = int(64 * cus * per_cu) + more
        feat, dirs, pfs = _inputs(g, B)
        switch = int(64 * cus * per_cu)
        picks = sorted({0, min(63, B - 1), B // 2, max(B - 2, 0), B - 1} | {v for v in (switch - 1, switch) if 0 <= v < B})
        w = torch.zeros(B, device="cuda")
        w[picks] = 0.5 + torch.arange(len(picks), device="cuda", dtype=torch.float32)
        g.loss_grad(feat, dirs, w, pfs)
        got, stats = [m.double() for m in g.split(g.grad.clone())], g.stats.clone()
        # 64 times the rounded product of the weight and 1 / B
        scaled = w * (torch.ones((), device="cuda") / B) * 64
        total, mag, loss = [torch.zeros_like(m) for m in got], [torch.zeros_like(m) for m in got], 0.0
        for v in picks:
            i = torch.full((64,), v, device="cuda")
            one = torch.zeros(64, device="cuda")
            one[v % 64] = scaled[v]
            g.loss_grad(feat[:, i].contiguous(), dirs[:, i].contiguous(), one, None if pfs is None else pfs[i])
            loss += float(g.stats[0])
            for a, b, m in zip(total, mag, g.split(g.grad)):
                a += m.double()
                b += m.double().abs()
        for layer, (x, ref, s) in enumerate(zip(got, total, mag)):
            err = (x - ref).abs() - 16 * 2.0 ** -24 * s
            assert float(err.max()) <= 1e-30, (name, B, layer, float((x - ref).abs().max()), float(s.max()))
        assert abs(float(stats[0]) - loss) <= 1e-6 * abs(loss) and abs(float(stats[1]) - float(w.sum())) <= 1e-6 * float(w.sum())
    g.close()


@pytest.mark.parametrize("name,four,eight", [("c1_f32", 1, 2), ("c2_f32", 1, 2), ("c2_f32", 3, 4), ("c2s_f32", 3, 4)])
def test_fp32_gradient_is_that_of_four_waves(name, four, eight):
    """FP32: a batch of `four` rounds of 64-vertex tiles runs four waves a
    workgroup, one of `eight` rounds eight. With the weights of the last rounds
    0 (and the others scaled by a power of two and the rounded 1 / B) both sum
    the same numbers, and do so in the same order: the same bits."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g, _ = make_guide(name, out_scale=2.0)
    n, B = 64 * cus * four, 64 * cus * eight
    assert B & (B - 1) == 0     # 1 / B exact
    feat, dirs, pfs = _inputs(g, B)
    w = to_dev(synth.radiance_weights(n, synth.rng_for(7)).astype("float32"))
    g.loss_grad(feat[:, :n].contiguous(), dirs[:, :n].contiguous(), w, None if pfs is None else pfs[:n].contiguous())
    small = g.grad.clone()
    padded = torch.zeros(B, device="cuda")
    padded[:n] = w * (torch.ones((), device="cuda") / n) * B
    g.loss_grad(feat, dirs, padded, pfs)
    assert torch.equal(g.grad, small)
    assert float(small.abs().max()) > 0
    g.close()
