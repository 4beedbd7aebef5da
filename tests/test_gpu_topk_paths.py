"""Top-k against the oracle where its routes meet: the one-block kernel (its
tiles, and keys that crowd in one bin) and the passes, and around the number of
keys the candidate list holds (keys that share the threshold's leading 23 bits)."""
import numpy as np
import pytest

from gpu_util import graph_us, log
from oracle import lossy as olossy
from paper_2409_17836_amd import binding as B

pytestmark = pytest.mark.gpu


def _check(v, ks):
    import torch
    dv = torch.from_numpy(v).cuda()
    for k in ks:
        got = B.sparsify_topk(dv, k).cpu().numpy()
        assert got.tobytes() == olossy.sparsify_topk(v, k).tobytes(), (v.size, k)


@pytest.mark.parametrize("n", [4096, 4097, 8192, 8193, 16384, 16385, 24577, 32764, 32768, 32769, 36000, 131072, 131073,
                               200001])
def test_routes_by_size(n):
    log(f"top-k routes n={n}")
    rng = np.random.default_rng(n)
    v = rng.normal(0, 1e-3, n).astype(np.float32)
    _check(v, [1, n // 10, n // 2, n - 1, n])
    v[rng.random(n) < 0.7] = 0.0                     # the threshold is zero for large k
    _check(v, [n // 10, n // 2])
    _check(np.full(n, -2.5, np.float32), [1, n // 3, n])


@pytest.mark.parametrize("n", [8193, 12287, 16385, 24577, 32767, 40001, 131071])
def test_crowded_bins(n):
    """One magnitude among others, keys that share the first digit or both, runs
    of four alike, and a vector whose parts differ."""
    log(f"top-k crowded n={n}")
    rng = np.random.default_rng(n)
    v = rng.normal(0, 1e-3, n).astype(np.float32)
    clipped = np.clip(v, -7e-4, 7e-4)
    first = (1e-3 * (1 + 0.03 * rng.random(n))).astype(np.float32)
    both = (1e-3 * (1 + 2e-5 * rng.random(n))).astype(np.float32)
    runs = np.repeat(v, 4)[:n]
    parts = np.where(np.arange(n) < n // 2, v, np.float32(-3e-4)).astype(np.float32)
    for x in (clipped, first, both, runs, parts, np.sign(v)):
        _check(x, [1, n // 10, n // 2, n - 1])


def test_keys_alike_cost_little_more():
    """(With an LDS atomic for every key 97 us against 13.)"""
    import torch
    ws = B.workspace(B.lossy_workspace(1))
    for n, times in ((32768, 3.5), (16385, 3.5)):
        log(f"top-k time n={n}")
        x = torch.randn(n, device="cuda") * 1e-3
        out = torch.empty_like(x)
        us = [graph_us(lambda: B.sparsify_topk(y, n // 10, out=out, ws=ws)) for y in (x, torch.zeros_like(x), x.sign())]
        log(f"{us}")
        assert max(us[1:]) < times * us[0], (n, us)


@pytest.mark.parametrize("same", [1, 999, 1000, 1001, 5000])
def test_candidates_around_the_list(same):
    """`same` keys share their leading 23 bits: equal ones in one half (ties by
    index), ones that differ in the last 8 bits in the other."""
    n = 100003
    log(f"top-k candidates {same}")
    rng = np.random.default_rng(same)
    v = rng.normal(0, 1e-3, n).astype(np.float32)
    v[np.abs(np.abs(v) - 5e-4) < 1e-6] = 0.0
    bits = np.full(same, np.float32(5e-4).view(np.uint32) & 0xFFFFFF00, np.uint32)
    bits[: same // 2] |= rng.integers(0, 256, same // 2).astype(np.uint32)
    at = rng.choice(n, same, replace=False)
    v[at] = bits.view(np.float32) * rng.choice(np.array([-1, 1], np.float32), same)
    above = int((np.abs(v) > 5.001e-4).sum())
    _check(v, sorted({above + 1, above + same // 4 + 1, above + (3 * same) // 4 + 1, above + same}))


def test_smallest_workspace():
    """Workspaces of 25632 bytes, which every version has taken, hold a shorter
    candidate list: few candidates, more than it holds, ties; quantisation too."""
    import torch
    dev = lambda v: torch.from_numpy(v).cuda()
    ws = torch.empty(25632, dtype=torch.uint8, device="cuda")
    for n in (50003, 3_000_017):
        log(f"smallest workspace n={n}")
        rng = np.random.default_rng(n)
        v = rng.normal(0, 1e-3, n).astype(np.float32)
        coarse = (v.view(np.uint32) & 0xFFFFE000).view(np.float32)     # candidates by the hundred
        levels = np.round(v * 2e3).astype(np.float32)
        for x in (v, coarse, levels):
            for k in (n // 10, n // 2):
                got = B.sparsify_topk(dev(x), k, ws=ws).cpu().numpy()
                assert got.tobytes() == olossy.sparsify_topk(x, k).tobytes(), (n, k)
        got = B.quantize_linear(dev(v), 8, ws=ws)[0].cpu().numpy()
        assert np.array_equal(got, olossy.quantize_linear(v, 8)[0])
    for call in (lambda w: B.sparsify_topk(dev(v), 5, ws=w), lambda w: B.quantize_linear(dev(v), 8, ws=w)):
        with pytest.raises(B.LMGCError) as e:
            call(ws[:25631])
        assert e.value.code == -4


def test_ranking_many_candidates_of_a_short_vector():
    """(With no more waves than the vector has blocks for, 36 us against 17.)"""
    import torch
    n, same = 40000, 990
    x = torch.randn(n, device="cuda") * 1e-3
    few = torch.where((x.abs() - 5e-4).abs() < 1e-6, torch.zeros_like(x), x)
    many = few.clone()
    bits = (torch.arange(same, device="cuda", dtype=torch.int32) % 256) + (0x3A03126F & ~255)     # 5e-4
    many[torch.arange(0, n, n // same, device="cuda")[:same]] = bits.view(torch.float32)
    k = int((many.abs() > 5.001e-4).sum()) + same // 2
    out, ws = torch.empty_like(x), B.workspace(B.lossy_workspace(n))
    log("top-k ranking time")
    us = [graph_us(lambda: B.sparsify_topk(y, k, out=out, ws=ws)) for y in (few, many)]
    log(f"{us}")
    assert us[1] < 1.7 * us[0], us
