"""Compression where its tiles and words end: escapes counted per tile of
2048 symbols, code words stored every two symbols in chunks of odd sizes,
track symbols stored 8 at a time.  Byte for byte the oracle's blob, on events
full of escapes and on tracks of every length modulo 8."""
import dataclasses

import numpy as np
import pytest

import synth
from test_gpu_compress import _check

pytestmark = pytest.mark.gpu


def noise(n):
    """n clusters anywhere: z steps and y beyond their byte range."""
    ev = synth.make_config1()
    g = np.random.Generator(np.random.PCG64(n))
    return dataclasses.replace(
        ev, row=g.integers(0, 152, n).astype(ev.row.dtype),
        y=g.uniform(-100, 100, n).astype(np.float32), z=g.uniform(0, 250, n).astype(np.float32),
        charge=g.integers(0, 1 << 17, n).astype(np.float32), label=np.full(n, -1, np.int32),
        sector_offsets=np.array([0, n], np.int64),
        sector_range=np.array([[-100, 100, 0, 250]], np.float32))


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 6000])
@pytest.mark.parametrize("chunk", [64, 101, 4096])
def test_escapes(n, chunk):
    _check(noise(n), chunk=chunk)


@pytest.mark.parametrize("chunk", [65, 128, 144, 1008])
@pytest.mark.parametrize("cbits", [2, 8])
def test_track_symbols(chunk, cbits):
    _check(synth.make_config2(seed=5, n_primary=60), cbits=cbits, chunk=chunk)
