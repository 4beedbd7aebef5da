"""The smaller tiles of the bf16 matrix product: every row count gives the
rows, bit for bit, that a large batch gives (another tile), and the values of
a float64 product."""
import numpy as np
import pytest

from gpu_util import bf16_tensor, bf16_values, log
from paper_2409_17836_amd import binding as B
from synth.configs import ModelShape, hex_serial
from synth.gen import gen_normal, gen_weights

pytestmark = pytest.mark.gpu


# One row, one short of a tile, tiles and a remainder; (N, K) from one stage
# and fewer stages than a ring holds to many.
@pytest.mark.parametrize("N,K", [(256, 64), (768, 192), (2304, 768), (4096, 1024), (12288, 256)])
@pytest.mark.parametrize("kind", ["store", "resid", "swiglu"])
def test_rows_do_not_depend_on_the_tile(kind, N, K):
    import torch
    big = 8448
    a = bf16_tensor(bf16_values(gen_normal((big, K), 5)))
    b = B.op_block_weights(bf16_tensor(bf16_values(gen_normal((N, K), 6, 0.05))))

    def run(m):
        out = None
        if kind == "resid":
            out = torch.arange(m * N, device="cuda", dtype=torch.float32).reshape(m, N) % 7
        return B.op_gemm_bf16_blocked(a[:m].contiguous(), b, kind, out=out)

    ref = run(big)
    for m in (1, 31, 32, 33, 63, 65, 128, 257, 520, 1000, 3000):
        log(f"gemm tiles {kind} {m}x{N}x{K}")
        got = run(m)
        assert torch.equal(got.view(torch.int16), ref[:m].view(torch.int16)), m


@pytest.mark.parametrize("M,N,K", [(1, 256, 64), (33, 768, 192), (200, 2304, 768), (129, 4096, 512)])
def test_values(M, N, K):
    import torch
    a, b = bf16_values(gen_normal((M, K), 7)), bf16_values(gen_normal((N, K), 8))
    log(f"gemm tiles values {M}x{N}x{K}")
    got = B.op_gemm_bf16_blocked(bf16_tensor(a), B.op_block_weights(bf16_tensor(b)), "store")
    torch.cuda.synchronize()
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    # float32 accumulation of K products of size about 1
    np.testing.assert_allclose(got.cpu().numpy(), ref, rtol=1e-5, atol=2e-4 * np.sqrt(K))


@pytest.mark.parametrize("arch,heads,kv,d,vocab", [("gpt2", 8, 8, 512, 1000), ("llama", 2, 1, 256, 777),
                                                  ("llama", 16, 4, 1024, 5003)])
def test_tables_do_not_depend_on_the_batch(arch, heads, kv, d, vocab):
    """One window alone against the same window in a batch, through every
    product of a decoder (QKV, residual, FFN, head) and the norms of few and
    of many rows, whole and ragged windows."""
    import torch
    shape = ModelShape(arch=arch, dtype="bf16", n_layers=2, d_model=d, n_heads=heads, n_kv_heads=kv, d_ff=2 * d,
                       vocab=vocab, max_pos=1024)
    host = gen_weights(shape, 3, init="perturbed")
    cfg = B.model_config(shape)
    dw = [torch.from_numpy(host[n].view(np.int16)).cuda() for n, _ in B.manifest(cfg)]
    model = B.Model(cfg, dw)
    rng = np.random.default_rng(4)
    for W, many in ((8, 40), (40, 9), (136, 33), (264, 40), (1000, 17)):
        log(f"tables {arch} W={W} B=1/{many}")
        sp = B.serial_params(hex_serial(window=W, bos_id=1))
        tok = torch.from_numpy(rng.integers(0, vocab, (many, W), dtype=np.int32)).cuda()
        cdf, logp = B.probs(model, tok, sp)
        for b in (0, many - 1):
            c1, l1 = B.probs(model, tok[b:b + 1].contiguous(), sp)
            assert torch.equal(c1[0], cdf[b]) and torch.equal(l1[0].view(torch.int32), logp[b].view(torch.int32)), (W, b)
    model.close()
