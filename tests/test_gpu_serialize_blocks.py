"""Serialisation over whole blocks of tokens: every value width, byte order and
group length (also those that do not divide the value), ranges that start inside
a group, against the oracle."""
import numpy as np
import pytest

from gpu_util import log
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
