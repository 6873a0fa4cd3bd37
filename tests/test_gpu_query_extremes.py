"""Queries whose mixture leaves the float range: the density that a query
returns with a direction has to be that of its own records there (which sum
the mixture by its logarithm)."""

import numpy as np
import pytest
import torch

from oracle import nasg as onasg
from paper_2303_08064_amd import synth
from tests.helpers import CONFIGS, ENCODED, make_guide, to_dev

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


@pytest.mark.parametrize("name,B", [(n, 20000) for n in CONFIGS if "nh" not in n] +
                         [("c3_bf16", 131072 + 100), ("c3_f32", 131072 + 100)])
def test_unlikely_lobe_beside_a_sharp_one(name, B):
    """xi_sel = 0 picks lobe 0 however small its weight (here e^-85), xi0 = 0
    the antipode of its axis. In a ring around a sharp lobe (lambda 148, a 7.4)
    the density is that lobe's, whose G is below the float range there while
    the density is not. Against float64 at the returned direction: where log G
    is -90, at angles of 0.4 (along x) and more, it moves by 180 / angle, some
    500, times the rounding of the frame and the direction, 1e-6 each."""
    K = CONFIGS[name][2]
    g, _ = make_guide(name)
    raw = np.zeros((8, K), np.float32)
    raw[2] = raw[4] = 1.0                       # phi = tau = 0
    raw[5], raw[6], raw[7] = -2.0, -2.0, -300.0
    raw[:, 0] = (-1.5, 1.0, 0.5, 0.25, 1.0, -2.0, -2.0, -85.0)
    raw[:, 1] = (1.0, 0.5, 2.0, 0.5, -1.0, 5.0, 2.0, 0.0)
    mats = g.split(g.w)
    for m in mats:
        m.zero_()
    mats[0][0, 63 if name in ENCODED else 9] = 1.0    # the constant one, handed through
    for m in mats[1:-1]:
        m[0, 0] = 1.0
    mats[-1][:8 * K, 0] = to_dev(raw.reshape(-1))
    g.repack()
    rng = synth.rng_for(8)
    feat, xi = synth.features(B, rng), synth.uniforms(B, rng)
    xi[0] = 0.0
    xi[1, ::7] = 0.0
    d, p = g.query(to_dev(feat), to_dev(xi))
    out = g.forward_raw(to_dev(feat[:, :1])).cpu().double()[:8 * K, 0]
    v = d.cpu().double().T
    lobes = onasg.decode(out.expand(B, 8 * K), K)
    ref = onasg.mixture_log_pdf(v, lobes).numpy()
    p = p.cpu().numpy().astype(np.float64)
    tiny, tol = float(np.log(np.finfo(np.float32).tiny)), 2e-3
    normal = ref > tiny + tol
    # directions of which the sharp lobe's share is beneath its float range
    log_g = onasg.lobe_log_g(v[:, None, :], lobes.z, lobes.x, lobes.lam, lobes.a)[:, 1].numpy()
    lost = normal & (log_g < tiny) & (onasg.component_log_terms(v, lobes)[:, 1].numpy() > ref - 0.7)
    assert lost.sum() > 50
    with np.errstate(divide="ignore"):
        err = np.abs(np.log(p) - ref)
    assert np.all(err[normal] <= tol), (err[normal].max(), int((err[normal] > tol).sum()))
    assert np.all(p[ref < tiny - tol] < 2 * np.finfo(np.float32).tiny)
    g.close()
