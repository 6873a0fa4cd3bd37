"""The hidden-64 queries run one or four 16-vertex blocks per wave pass by the
batch's size; both must give the same bits, vertex by vertex."""

import numpy as np
import pytest
import torch

from paper_2303_08064_amd import synth
from tests.helpers import CONFIGS, make_guide, rec_to_bk9, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["c1_bf16", "c2_bf16", "c3_bf16", "c3s_bf16", "c1_f32", "c2_f32", "c2s_f32", "c3_f32"])
def test_one_and_four_block_passes_agree_bitwise(name):
    """A batch of two full rounds of four-block passes less a ragged end (inside
    a block) against its vertices queried in batches of one-block passes: the
    first, a middle and the last ones, in batches that end inside a block, fill
    it, and hold a single vertex."""
    K = CONFIGS[name][2]
    g, _ = make_guide(name, out_scale=8.0)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    full = 1024 * cus - 37
    rng = synth.rng_for(77)
    feat, xi = to_dev(synth.features(full, rng)), to_dev(synth.uniforms(full, rng))
    sel = torch.empty(full, device="cuda") if g.selection else None
    d0, p0 = g.query(feat, xi, sel_out=sel)
    d1, p1, r0 = g.query(feat, xi, records=True)
    torch.cuda.synchronize()
    assert torch.equal(d0, d1) and torch.equal(p0, p1)   # with and without the record store
    rec = rec_to_bk9(r0, full, K)
    for start, n in ((0, 1), (0, 3001), (64 * 1000, 64), (full // 2, 1000), (full - 16, 16), (full - 777, 777)):
        f, x = feat[:, start:start + n].contiguous(), xi[:, start:start + n].contiguous()
        s = torch.empty(n, device="cuda") if g.selection else None
        d, p, r = g.query(f, x, records=True, sel_out=s)
        torch.cuda.synchronize()
        assert torch.equal(d, d0[:, start:start + n]) and torch.equal(p, p0[start:start + n]), (name, start, n)
        assert np.array_equal(rec_to_bk9(r, n, K), rec[start:start + n]), (name, start, n)
        if g.selection:
            assert torch.equal(s, sel[start:start + n]), (name, start, n)
    g.close()
