"""The tiles of the bf16 matrix product: each tile by name, and the row counts
that take them by themselves, give the same rows bit for bit, and the values of a
float64 product."""
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


TILES = [t for t in B.TILES if t != "256x128"]       # (that one is the LM head's)


# Row counts that end inside every tile; one stage of 64 to seven, fewer and
# more than any ring holds; narrow and wide N (the 256x256 tile's ring holds B
# for N >= 2 K, else A).
@pytest.mark.parametrize("kind", ["store", "resid", "swiglu"])
@pytest.mark.parametrize("M,N,K", [(17, 256, 64), (300, 512, 128), (33, 768, 192), (129, 256, 320), (257, 1024, 448)])
def test_each_tile(kind, M, N, K):
    import torch
    a, b = bf16_values(gen_normal((M, K), 7)), bf16_values(gen_normal((N, K), 8))
    c0 = gen_normal((M, N), 9) if kind == "resid" else None
    acc = a.astype(np.float64) @ b.astype(np.float64).T
    if kind == "resid":
        acc += c0
    if kind == "swiglu":  # row 64 g + t is gate feature 32 g + t, row 64 g + 32 + t its up row
        g = acc.reshape(M, -1, 2, 32)
        acc = (g[:, :, 0] / (1 + np.exp(-g[:, :, 0])) * g[:, :, 1]).reshape(M, -1)
    at, bt = bf16_tensor(a), B.op_block_weights(bf16_tensor(b))
    first = None
    for tile in TILES:
        log(f"gemm tile {tile} {kind} {M}x{N}x{K}")
        got = B.op_gemm_bf16_blocked(at, bt, kind, out=None if c0 is None else torch.from_numpy(c0).cuda(), tile=tile)
        torch.cuda.synchronize()
        # float32 accumulation of K products of size about 1; bf16 results round by 2^-8 at most
        rtol, atol = (2.0 ** -8, 1e-3 * np.sqrt(K)) if kind == "swiglu" else (1e-5, 2e-4 * np.sqrt(K))
        np.testing.assert_allclose(got.float().cpu().numpy(), acc, rtol=rtol, atol=atol, err_msg=tile)
        first = got if first is None else first
        assert torch.equal(got.view(torch.int16), first.view(torch.int16)), tile


@pytest.mark.parametrize("arch", ["gpt2", "llama"])
@pytest.mark.parametrize("hd", [64, 128])
def test_each_tile_in_a_decoder(arch, hd):
    """Batches whose QKV product takes each tile in turn, and whose LM head
    takes each of the smaller ones, against windows alone (the smallest tile)."""
    import torch
    d, vocab, W = 1024, 5003, 8
    shape = ModelShape(arch=arch, dtype="bf16", n_layers=2, d_model=d, n_heads=d // hd, n_kv_heads=d // hd, d_ff=2 * d,
                       vocab=vocab, max_pos=64)
    host = gen_weights(shape, 3, init="perturbed")
    cfg = B.model_config(shape)
    model = B.Model(cfg, [torch.from_numpy(host[n].view(np.int16)).cuda() for n, _ in B.manifest(cfg)])
    sp = B.serial_params(hex_serial(window=W, bos_id=1))
    tok = torch.from_numpy(np.random.default_rng(4).integers(0, vocab, (351, W), dtype=np.int32)).cuda()
    ref = [B.probs(model, tok[b:b + 1].contiguous(), sp) for b in (0, 5, 7)]
    qkv, head = set(), set()
    for n in (8, 25, 51, 177, 351):
        log(f"decoder tiles {arch} hd={hd} windows={n}")
        qkv.add(B.gemm_tile(n * W, 3 * d, d))
        head.add(B.gemm_tile(n * W, 5120, d, head=True))
        cdf, logp = B.probs(model, tok[:n].contiguous(), sp)
        for b, (c1, l1) in zip((0, 5, 7), ref):
            assert torch.equal(c1[0], cdf[b]) and torch.equal(l1[0].view(torch.int32), logp[b].view(torch.int32)), (n, b)
        # the last rows of the batch
        c1, l1 = B.probs(model, tok[n - 1:n].contiguous(), sp)
        assert torch.equal(c1[0], cdf[-1]) and torch.equal(l1[0].view(torch.int32), logp[-1].view(torch.int32)), n
    model.close()
    assert qkv == set(TILES) and head == {"64x64", "128x64", "128x128", "256x128"}, (qkv, head)
