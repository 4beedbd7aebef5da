"""The float32 decoder's matrix kernel at the edges of its 64-row and
64-column tiles: both architectures (every epilogue), row counts around a
tile, windows that are no multiple of four rows, vocabularies that end inside
a tile; against the oracle, and the decoding steps bit for bit; and the product itself
against the host's fused multiply-adds."""
import ctypes

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


def test_product_is_one_fma_chain():
    """Every element is acc = fmaf(a[k], b[k], acc) over rising k from +0, all
    bits: what containers of the float32 decoder depend on.  Exponents from
    denormal products to 2^80, signed zeros, whole rows of zeros."""
    import torch
    M, N, K = 65, 64, 48
    rng = np.random.default_rng(2)

    def matrix(rows):
        x = rng.uniform(1, 2, (rows, K)) * np.exp2(rng.integers(-75, 40, (rows, K)).astype(np.float64))
        x[: rows // 2] = rng.normal(0, 1, (rows // 2, K))
        x[rng.random((rows, K)) < 0.05] = 0.0
        x[3] = 0.0
        x[4] = 1e-45 * rng.integers(0, 1000, K)
        return (x * rng.choice([-1.0, 1.0], (rows, K))).astype(np.float32)

    a, b = matrix(M), matrix(N)
    log(f"f32 product {M}x{N}x{K} against fmaf")
    got = B.op_gemm_f32(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()).cpu().numpy()
    fmaf = ctypes.CDLL("libm.so.6").fmaf
    fmaf.restype, fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    al, bl = a.tolist(), b.tolist()
    want = np.zeros((M, N), np.float32)
    for i in range(M):
        for j in range(N):
            acc = 0.0
            for x, y in zip(al[i], bl[j]):
                acc = fmaf(x, y, acc)
            want[i, j] = acc
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), int((got.view(np.uint32) != want.view(np.uint32)).sum())
    tiny = np.abs(want[want != 0]).min()
    assert tiny < 1.17e-38 and np.isfinite(want).all()       # denormal results are among them
