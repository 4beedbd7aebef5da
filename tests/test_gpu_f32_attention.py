"""The float32 decoder at every head dim and at window lengths around the
attention kernel's 64-key tiles: log-probabilities against the oracle, and the
decoding steps' tables bit for bit; and what windows shorter than a tile cost."""
import numpy as np
import pytest

from gpu_util import graph_us, log
from oracle import pipeline as opipe
from oracle.forward import Model as OracleModel
from paper_2409_17836_amd import binding as B
from synth.configs import ModelShape, hex_serial
from synth.gen import gen_values, gen_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [16, 32, 48, 64])
def test_head_dims_and_ragged_windows(hd):
    import torch
    shape = ModelShape(arch="llama", dtype="f32", n_layers=2, d_model=4 * hd, n_heads=4, n_kv_heads=4, d_ff=128,
                       vocab=256, max_pos=256)
    host = gen_weights(shape, 9, init="perturbed")
    cfg = B.model_config(shape)
    model = B.Model(cfg, [torch.from_numpy(host[n]).cuda() for n, _ in B.manifest(cfg)])
    om = OracleModel(shape, host)
    vals = gen_values("normal:1e-3", 60, hd)
    for W in (1, 5, 63, 64, 65, 130, 200):
        log(f"f32 attention hd={hd} W={W}")
        spec = hex_serial(window=W, bos_id=1)
        sp = B.serial_params(spec)
        n = min(2, -(-9 * vals.size // W))
        tok, _ = B.serialize(torch.from_numpy(vals).cuda(), sp, 0, n)
        cdf, logp = B.probs(model, tok, sp)
        otok, _ = opipe.serialize(vals, spec)
        lp = logp.cpu().numpy()
        for wi, (s, m) in enumerate(list(opipe.windows(otok.size, W))[:n]):
            ref = opipe.window_logprobs(om, otok[s:s + m], spec)
            assert np.abs(lp[wi, :m] - ref).max() <= 1e-4          # the float32 bar of the whole-model tests
        cdf2, logp2 = B.probs_stepwise(model, tok, sp)
        assert torch.equal(cdf, cdf2) and torch.equal(logp.view(torch.int32), logp2.view(torch.int32)), W
    model.close()


def test_short_windows_cost_no_more_than_long_ones():
    """The same tokens as windows of 4 and of 64.  (With 64 keys for every
    query 664 us against 319.)"""
    import torch
    shape = ModelShape(arch="llama", dtype="f32", n_layers=2, d_model=256, n_heads=4, n_kv_heads=4, d_ff=512,
                       vocab=256, max_pos=64)
    host = gen_weights(shape, 5, init="perturbed")
    cfg = B.model_config(shape)
    model = B.Model(cfg, [torch.from_numpy(host[n]).cuda() for n, _ in B.manifest(cfg)])
    us = []
    for W in (4, 64):
        log(f"f32 attention time W={W}")
        sp = B.serial_params(hex_serial(window=W, bos_id=1))
        tok = torch.full((4096 // W, W), 48, dtype=torch.int32, device="cuda")
        ws = B.workspace(model.probs_workspace(*tok.shape))
        cdf, logp = B.probs(model, tok, sp, ws=ws)
        us.append(graph_us(lambda: B.probs(model, tok, sp, ws=ws, cdf=cdf, logp=logp), reps=5))
    log(f"{us}")
    model.close()
    assert us[0] < 1.4 * us[1], us
