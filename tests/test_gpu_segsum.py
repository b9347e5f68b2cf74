"""Sums of programs' rows at the edges of a wavefront's window of 2048 rows (256 in calls of few rows a program): programs
that fill it, cross it, take several of them or none, wavefronts that are not full, and both sides of the lines to
programs whose rows every lane reads for itself; every bit against the oracle."""
import numpy as np
import pytest

from paper_2201_00194_amd import workloads as W
from test_gpu_parity import api, check_family, run_families  # noqa: F401

pytestmark = pytest.mark.gpu

LENGTHS = {
    "one long": [5000],
    "a window and a row": [2047, 1, 2048, 1, 2049, 0, 0, 3],
    "nothing": [0] * 70,
    "first and last empty": [0, 5, 0, 0, 7, 0],
    "short": [1] * 130,
    "at window ends": [1024, 1023, 1, 2, 2046, 1, 1] * 3,
    "equal": [16] * 64 + [64] * 65 + [32],
    "uneven": 120,
    "long": [1000] * 64 + [144] * 64 + [96] * 64 + [97] * 63,
    "long and uneven": 400,
    "one or two": [1, 2] * 70,
    "two and one of three": [2] * 100 + [3] + [1, 0, 0] * 40,
    "four": [4] * 130,
    "short window's end": [4] * 64 + [4] * 63 + [5] + [3] * 63 + [67] + [1] * 63 + [193] + [1] * 63 + [194] + [0] * 700,
}


@pytest.mark.parametrize("kind", LENGTHS)
def test_program_lengths(api, oracle, kind):  # noqa: F811
    lengths = LENGTHS[kind]
    if isinstance(lengths, int):
        lengths = np.random.default_rng(3).integers(0, lengths, 700)
    off = np.concatenate(([0], np.cumsum(lengths))).astype(np.int32)
    rows = max(1, int(off[-1]))
    fam = W.make_small_family(seed=rows, n_programs=rows, stmts=(1, 1), n_trees=5, depth=3, k=4, n_features=9, bias=0.125)
    fam.features, fam.prog_off = fam.features[:int(off[-1])], off
    other = W.make_small_family(seed=2, n_programs=300, stmts=(1, 9), n_trees=5, depth=3, k=4, n_features=9)
    for fams in ([fam], [fam, other]):
        for f, dev in zip(fams, run_families(api, fams, api.FS_COLBLOCK64)):
            check_family(oracle, f, dev)
