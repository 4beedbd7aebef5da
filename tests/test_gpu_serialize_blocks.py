"""Serialisation over whole blocks of tokens: every value width, byte order and
group length (also those that do not divide the value), ranges that start inside
a group, against the oracle; ranges around the change from four to sixteen tokens
per thread; and what the blocks at the end of the stream cost."""
import numpy as np
import pytest

from gpu_util import graph_us, log
from paper_2409_17836_amd import binding as B
from synth.configs import hex_serial
from test_gpu_serialize import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bpv", [1, 2, 4])
@pytest.mark.parametrize("bpg", [0, 1, 3, 4, 7, 255])
def test_blocks(bpv, bpg):
    n = 40009 // bpv
    log(f"serialize blocks bpv={bpv} bpg={bpg}")
    raw = np.random.default_rng(bpg + 10 * bpv).integers(0, 256, n * bpv, dtype=np.uint8)
    vals = raw.view({1: np.uint8, 2: np.int16, 4: np.float32}[bpv])
    for msb, sep2 in ((1, -1), (0, 44)):
        spec = hex_serial(window=1000, bos_id=1, bytes_per_value=bpv, bytes_per_group=bpg, msb_first=msb, sep2_id=sep2)
        _check(vals, spec)
        _check(vals, spec, first=7, count=30)


@pytest.mark.parametrize("windows", [4095, 4096, 4097])     # of 1024 tokens: 2^22 is the border
def test_short_and_long_ranges(windows):
    n = (windows * 1024 - 500) // 9
    log(f"serialize {windows} windows")
    vals = np.random.default_rng(windows).normal(0, 1e-3, n).astype(np.float32)
    _check(vals, hex_serial(window=1024, bos_id=1))
    _check(vals, hex_serial(window=1024, bos_id=1), first=1)


def test_the_end_of_the_stream_costs_no_more():
    """A short vector, whose last block is a good part of the launch, against as
    many windows from the middle of a long one.  (With a division per token in
    that block, 10 us against 4.)"""
    import torch
    sp = B.serial_params(hex_serial(window=2048, bos_id=1))
    v = torch.randn(1 << 20, device="cuda")
    for n in (455, 10000, 30000):
        log(f"serialize time n={n}")
        short = v[:n].clone()
        nw = B.num_windows(n, sp)
        tok = torch.empty((nw, 2048), dtype=torch.int32, device="cuda")
        sym = torch.empty((nw, 2048), dtype=torch.uint8, device="cuda")
        end = graph_us(lambda: B.serialize(short, sp, tokens=tok, sym=sym))
        middle = graph_us(lambda: B.serialize(v, sp, 100, nw, tokens=tok, sym=sym))
        assert end < 1.5 * middle, (n, end, middle)
