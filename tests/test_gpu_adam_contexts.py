"""The Adam step takes its rate and betas from the context it is called on,
whatever ran before: another context's loss_grad on the same state (a
learning-rate schedule that makes a new context), or none (a gradient that the
caller wrote)."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import train as otrain
from paper_2303_08064_amd import synth
from paper_2303_08064_amd._lib import Config, check
from tests.helpers import make_guide, to_dev

pytestmark = pytest.mark.gpu


def _check(g, w0, m0, v0, t, lr, beta1, beta2):
    torch.cuda.synchronize()
    hyper = [float(np.float32(x)) for x in (lr, beta1, beta2, 1e-8)]
    ref = otrain.adam_step(w0, g.grad.cpu().double(), m0, v0, t, *hyper)[0]
    # a float32 weight below 1 and a float32 update below 2 lr, both rounded a few times
    assert int(g.step) == t + 1 and int(g.flags) == 0
    assert float((g.w.cpu().double() - ref).abs().max()) < 1e-7
    assert float((ref - w0).abs().max()) > lr / 2


@pytest.mark.parametrize("name", ["c2_f32", "c3_bf16", "c5_bf16"])
@pytest.mark.parametrize("lr,beta1,beta2", [(5e-3, 0.9, 0.999), (1e-3, 0.5, 0.999), (1e-3, 0.9, 0.9), (2e-3, 0.0, 0.0)])
def test_step_on_another_context(name, lr, beta1, beta2):
    g, _ = make_guide(name, max_batch=2048)
    f, d, w = synth.training_batch(2000, synth.rng_for(31), synth.VmfTarget(4, seed=1001))
    batch = [to_dev(x) for x in (f, d, w)]
    cfg = Config.from_buffer_copy(g.cfg)
    cfg.lr, cfg.beta1, cfg.beta2 = lr, beta1, beta2
    other = ctypes.c_void_p()
    check(g.lib.nasg_create(ctypes.byref(cfg), ctypes.byref(g._state), ctypes.byref(other)))
    for t in range(2):
        g.loss_grad(*batch)
        w0, m0, v0 = (x.cpu().double() for x in (g.w, g.adam_m, g.adam_v))
        check(g.lib.nasg_adam_step(other, g._stream()))
        _check(g, w0, m0, v0, t, lr, beta1, beta2)
    g.lib.nasg_destroy(other)
    g.close()


@pytest.mark.parametrize("name,beta", [("c2_f32", 0.9), ("c3_bf16", 0.9), ("paper_bf16", 0.9), ("c1_f32", 0.0)])
def test_step_from_a_written_gradient(name, beta):
    g, _ = make_guide(name, max_batch=2048, beta1=beta, beta2=beta)
    w0 = g.w.cpu().double()
    g.grad.copy_(torch.from_numpy(synth.rng_for(32).standard_normal(g.num_weights).astype(np.float32)))
    g.adam_step()
    _check(g, w0, torch.zeros_like(w0), torch.zeros_like(w0), 0, 1e-3, beta, beta)
    g.close()
