"""Choices in a tuner's cache file hold for the version of the library that timed
them: a line stored by another one, whose kernels and defaults differ, is not
taken."""

import struct

import pytest

import gsvd_inputs as gi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = (160, 150, 96)


def _key(version, batch=0):
    """The FNV-1a hash that names a line, for default parameters with w = 16."""
    prop = torch.cuda.get_device_properties(0)
    p = [0, 1, 2, 16, 30, 1, 0, 0, 0]      # variant, orderings, w, sweeps, sort, lanes, splits, rows
    data = (b"dgsvd" + struct.pack("9i", *p) + struct.pack("d", 0.0) + struct.pack("i", 1)
            + struct.pack("3q", *N) + prop.gcnArchName.encode()
            + struct.pack("i", prop.multi_processor_count) + version)
    h = 14695981039346656037
    for b in data:
        h = ((h ^ b) * 1099511628211) & (2 ** 64 - 1)
    return h


@pytest.mark.parametrize("own", [True, False], ids=["own", "before"])
def test_cache_line_of_a_version(tmp_path, own):
    import paper_1909_00101_amd as hz
    version = hz.lib().hz_version() if own else b"hzgsvd 0.2 (gfx950)"
    cache = tmp_path / "tune.txt"
    line = "%016x 16 7 16 3 112 123.250000 1 2\n" % _key(version)
    cache.write_text(line)
    F, G, _ = gi.custom_pair(*N, kappa=10.0, seed=3)
    best, ms = hz.tune(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), cache=str(cache), w=16)
    taken = ms == 123.25 and best["gram_splits"] == 3 and best["update_rows"] == 112
    assert taken == own
    assert len(cache.read_text().splitlines()) == (1 if own else 2)
