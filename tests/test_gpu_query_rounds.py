"""Queries whose waves take several passes: the passes' strides, the staging
buffers that they alternate between and the inputs requested ahead. A batch of
two to four rounds over the CUs with a ragged end, against the same vertices in
batches of one pass a wave: the same bits."""

import pytest
import torch

from paper_2303_08064_amd import synth
from paper_2303_08064_amd.nasg import record_elems
from tests.helpers import CONFIGS, make_guide, to_dev

pytestmark = pytest.mark.gpu

# vertices per CU of a batch: the hidden-64 networks' one-block passes (64, 128
# or 192 vertices a round and CU), the two-block kernel (256) and the streamed
# kernels (128); the four-block passes of the last column's sizes (512)
ROUNDS = {
    "c1_bf16": (640, 1536), "c2_bf16": (704, 1536), "c3_bf16": (448, 1536), "c3s_bf16": (448, 1536),
    "c1_f32": (448, 1536), "c2_f32": (384, 1536), "c3_f32": (384, 1536), "c3nh1_bf16": (448, 1536),
    "paper_bf16": (513,), "c5_bf16": (257,), "c5_f32": (257,), "paper_f32": (257,),
}
PIECE = 64 * 187     # vertices of a one-pass batch: whole record tiles, below 64 a CU


@pytest.mark.parametrize("name,per_cu", [(n, p) for n, ps in ROUNDS.items() for p in ps])
def test_rounds_agree_with_single_passes(name, per_cu):
    K = CONFIGS[name][2]
    g, _ = make_guide(name, out_scale=8.0)
    B = per_cu * torch.cuda.get_device_properties(0).multi_processor_count - 37
    rng = synth.rng_for(91)
    feat, xi = to_dev(synth.features(B, rng)), to_dev(synth.uniforms(B, rng))

    def run(f, x):
        n = f.shape[1]
        sel = torch.zeros(n, device="cuda") if g.selection else torch.zeros(0, device="cuda")
        rec = torch.zeros(record_elems(K, n), device="cuda")
        d, p = g.query(f, x, sel_out=sel if g.selection else None)
        dr, pr, _ = g.query(f, x, rec_out=rec)
        raw = g.forward_raw(f)
        assert torch.equal(d, dr) and torch.equal(p, pr)     # with and without the record store
        return d, p, sel, raw, rec.view(-1, 9, K, 64)

    whole = run(feat, xi)
    for start in range(0, B, PIECE):
        end = min(start + PIECE, B)
        part = run(feat[:, start:end], xi[:, start:end])     # views: their rows are B apart
        cut = [whole[0][:, start:end], whole[1][start:end], whole[2][start:end], whole[3][:, start:end],
               whole[4][start // 64:(end + 63) // 64]]
        for what, a, b in zip(("direction", "pdf", "selection", "raw outputs", "records"), cut, part):
            assert torch.equal(a, b), (name, B, start, what)
    g.close()
