"""Queries whose mixture leaves the float range: the density that a query
returns with a direction has to be that of its own records there (which sum
the mixture by its logarithm)."""

import numpy as np
import pytest
import torch

from paper_2303_08064_amd import synth
from tests.helpers import CONFIGS, make_guide, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,B", [(n, 1000) for n in CONFIGS if "nh" not in n] +
                         [("c3_bf16", 131072 + 100), ("c3_f32", 131072 + 100)])
def test_extreme_features(name, B):
    """A non-finite or huge feature in a vertex each: logits of 1e9 and more
    overflow or empty the softmax's sum, and NaN frames have no density. The
    query's pdf is 0 and NaN where that of its records is. The second size
    runs the four-block passes."""
    g, _ = make_guide(name, out_scale=8.0)
    rng = synth.rng_for(5)
    feat, xi = synth.features(B, rng), synth.uniforms(B, rng)
    at = []
    for row in range(9):
        for j, x in enumerate((np.nan, np.inf, -np.inf, 1e38, -1e38, 1e20, -1e20, 1e12)):
            at.append(B - 1 - 16 * row - j)
            feat[row, at[-1]] = x
    d, p, rec = g.query(to_dev(feat), to_dev(xi), records=True)
    q = g.pdf(rec, d.contiguous())
    torch.cuda.synchronize()
    p, q = p.cpu().numpy()[at], q.cpu().numpy()[at]
    assert np.any(q == 0) and np.all(np.isfinite(d.cpu().numpy()[:, :100]))
    assert np.array_equal(np.isnan(p), np.isnan(q)), (p, q)
    assert np.array_equal(p == 0, q == 0), (p, q)
    g.close()


@pytest.mark.parametrize("name", [n for n in CONFIGS if "nh" not in n])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_nan_pair(name, p):
    """A NaN in one raw output of a lobe's (cos, sin) pair leaves the pair
    (1, 0), as two zeros do: the same directions, densities, records and loss
    as with the pair's output rows zeroed. The Adam step skips its update (the
    pair's own gradient is NaN)."""
    K, sel = CONFIGS[name][2], "s_" in name or "paper" in name
    rng = synth.rng_for(6)
    feat, xi = to_dev(synth.features(1000, rng)), to_dev(synth.uniforms(1000, rng))
    f, d, w = synth.training_batch(999, rng, synth.VmfTarget(4, seed=1001))
    batch = [to_dev(x) for x in (f, d, w)] + ([to_dev(synth.lambert_pdf(d, f[6:9]))] if sel else [])
    out = []
    for value in (0.0, np.nan):
        g, mats = make_guide(name, out_scale=8.0)
        W = g.split(g.w)[-1]
        first = 1 if p < 3 else 3
        W[[first * K + 1, (first + 1) * K + 1]] = 0.0
        W[p * K + 1] = value
        g.repack()
        rec = torch.zeros(((1000 + 63) // 64) * 9 * K * 64, device="cuda")
        q = g.query(feat, xi, rec_out=rec)
        g.train_step(*batch)
        torch.cuda.synchronize()
        out.append([t.clone() for t in (*q, g.stats[:2])] + [int(g.flags) & 1])
        g.close()
    zero, nan = out
    for a, b in zip(zero[:4], nan[:4]):
        assert torch.equal(a, b)
    assert (zero[4], nan[4]) == (0, 1)
