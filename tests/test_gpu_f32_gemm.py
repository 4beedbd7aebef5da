"""The float32 decoder's matrix kernel at the edges of its 64-row and
64-column tiles: both architectures (every epilogue), row counts around a
tile, windows that are no multiple of four rows, vocabularies that end inside
a tile; against the oracle, and the decoding steps bit for bit."""
import numpy as np
import pytest

from gpu_util import log
from oracle import pipeline as opipe
from oracle.forward import Model as OracleModel
from paper_2409_17836_amd import binding as B
from synth.configs import ModelShape, hex_serial
from synth.gen import gen_values, gen_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch", ["llama", "gpt2"])
@pytest.mark.parametrize("heads,hd,ff,vocab", [(4, 16, 64, 256), (4, 48, 128, 300), (6, 32, 192, 129)])
def test_tile_edges(arch, heads, hd, ff, vocab):
    import torch
    shape = ModelShape(arch=arch, dtype="f32", n_layers=2, d_model=heads * hd, n_heads=heads, n_kv_heads=heads,
                       d_ff=ff, vocab=vocab, max_pos=64)
    host = gen_weights(shape, 5, init="perturbed")
    cfg = B.model_config(shape)
    model = B.Model(cfg, [torch.from_numpy(host[n]).cuda() for n, _ in B.manifest(cfg)])
    om = OracleModel(shape, host)
    vals = gen_values("normal:1e-3", 60, ff)
    for W, nb in ((1, 1), (21, 3), (16, 4), (13, 5), (50, 2)):      # M = 1, 63, 64, 65, 100
        log(f"f32 gemm {arch} d={heads * hd} ff={ff} W={W} windows={nb}")
        spec = hex_serial(window=W, bos_id=1)
        sp = B.serial_params(spec)
        tok, _ = B.serialize(torch.from_numpy(vals).cuda(), sp, 0, nb)
        cdf, logp = B.probs(model, tok, sp)
        otok, _ = opipe.serialize(vals, spec)
        lp = logp.cpu().numpy()
        for wi, (s, m) in enumerate(list(opipe.windows(otok.size, W))[:nb]):
            ref = opipe.window_logprobs(om, otok[s:s + m], spec)
            assert np.abs(lp[wi, :m] - ref).max() <= 1e-4          # the float32 bar of the whole-model tests
        cdf2, logp2 = B.probs_stepwise(model, tok, sp)
        assert torch.equal(cdf, cdf2) and torch.equal(logp.view(torch.int32), logp2.view(torch.int32)), (W, nb)
    model.close()
