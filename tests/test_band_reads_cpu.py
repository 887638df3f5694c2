"""Operand addresses of the kernels for long filters, followed on the host with the plans and the walk of the kernels (band_reads.hip): no
read outside what a stage has put into LDS, no product of a place that has no work, every product once."""
import os
import subprocess

import pytest

from paper_2604_25422_amd import _build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def reads(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("band_reads") / "band_reads")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    r = subprocess.run([hipcc, "--offload-host-only"] + _build.HIPCC_FLAGS + ["-O1", os.path.join(HERE, "band_reads.hip"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def run(exe, *args, shapes=()):
    r = subprocess.run([exe, *map(str, args)], input="".join("%d %d %d %d %d %d\n" % s for s in shapes), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-1000:]
    planned = int(r.stdout.split()[-6])
    return planned


# causal filters whose last window has fewer offsets than places, in several stages along a row (the places in front are then the empty ones)
DW_BAND = [(8, 256, 8192, 500, 499, 0), (32, 256, 4096, 257, 256, 0), (32, 256, 4096, 226, 225, 0), (1000, 64, 377, 100, 99, 0), (13, 582, 480, 8926, 8397, 0),
           (1, 317, 568, 1205, 1204, 0), (100, 64, 1500, 520, 519, 0), (64, 256, 2048, 500, 250, 0), (64, 256, 2048, 500, 0, 1), (8, 256, 8192, 500, 499, 1)]


def test_dw_band(reads):
    assert run(reads, "dw_band", "-", shapes=DW_BAND) == len(DW_BAND)
    assert run(reads, "dw_band", 1, 3000) > 2000


# nearly causal filters on rows of one item with fewer tiles than the waves have places for (the spare tile is then in front), forward and
# input gradient, one chunk of taps and several
CORR_BAND = [(1, 600, 3040, 600, 480, 0), (1, 1024, 3000, 600, 500, 0), (119, 47, 727, 1130, 117, 0), (456, 43, 709, 709, 6, 1), (1788, 128, 309, 309, 248, 0),
             (2048, 128, 256, 256, 255, 0), (8, 256, 8192, 8192, 8191, 0), (8, 256, 8192, 8192, 8191, 1), (2, 3, 40000, 39000, 30000, 0)]


def test_corr_band(reads):
    assert run(reads, "corr_band", "-", shapes=CORR_BAND) == 2 * len(CORR_BAND)
    assert run(reads, "corr_band", 1, 3000) > 4000


# one tile of lags per workgroup and two, lags that end in a spare tile, several chunks; chains of additions on both sides of B L = 65536
DW_TOEP = [(8, 256, 8192, 8192, 8191, 0), (7, 256, 8192, 8192, 8191, 0), (5, 256, 8192, 8192, 8191, 0), (32, 256, 4097, 4097, 4096, 1), (1, 300, 2049, 2050, 2049, 0),
           (1, 2, 8, 20, 9, 1), (9, 32, 3000, 3000, 2999, 0), (17, 736, 889, 889, 444, 0), (1, 2, 40000, 70000, 39000, 0)]


def test_dw_toep(reads):
    assert run(reads, "dw_toep", "-", shapes=DW_TOEP) == len(DW_TOEP)
    assert run(reads, "dw_toep", 1, 3000) > 2000
