"""Arenas are sized by a plan's footprint and kept by their callers, and the request loop admits by it: no plan asks
for more than the layout with the projector table over the whole sphere, the stick buffer of one batch and the split
partials of 64 x 64 tiles took (bytes below).  CPU only."""
import numpy as np
import pytest

from paper_2406_10765_amd import pw, synth

BF16, BF16_KB, GEN, LOBPCG = pw.PW_FLAG_BF16_ALL, pw.PW_FLAG_BF16_KB, pw.PW_FLAG_BETA_OTF, pw.PW_FLAG_LOBPCG
ONE_ATOM = synth.Cell(L=(26.0, 26.0, 12.0), tau=np.zeros((1, 3)), ecut=9.0, nbands=7)


def si(n, ecut, nb):
    return synth.silicon_cell(n, ecut, nbands=nb, disp_seed=1)


CASES = [
    # unequal sides: the pencil intermediate
    (si((1, 2, 3), 17, 101), pw.PW_MIXED, 0, 0),
    (si((1, 2, 3), 17, 101), pw.PW_MIXED, BF16, 0),
    (si((1, 2, 3), 17, 101), pw.PW_FP64, GEN, 0),
    (si((2, 1, 2), 8, 24), pw.PW_FP64, GEN, 0),
    (si((3, 1, 1), 10, 16), pw.PW_MIXED, GEN, 0),
    (si((3, 1, 1), 8, 1), pw.PW_FP64, GEN, 0),
    (si((4, 2, 1), 8, 5), pw.PW_FP64, GEN | LOBPCG, 0),
    (si((1, 2, 2), 17, 102), pw.PW_MIXED, 0, 34),
    # planes beyond LDS, rows padded to 16 bytes
    (si((1, 3, 1), 10, 1), pw.PW_MIXED, pw.PW_FLAG_PENCIL_FFT, 0),
    # many K splits
    (si((1, 1, 1), 10, 20), pw.PW_FP64, 0, 0),
    (si((1, 1, 1), 10, 20), pw.PW_MIXED, BF16, 0),
    (si((2, 2, 2), 20, 144), pw.PW_FP64, 0, 0),
    (synth.make_cell("si4096"), pw.PW_FP64, GEN, 0),
    # fewer projectors than a K tile
    (ONE_ATOM, pw.PW_MIXED, BF16, 0),
    (ONE_ATOM, pw.PW_MIXED, BF16_KB, 0),
]
BYTES = [146850048, 181988352, 213022208, 11966720, 4303360, 1081856, 11170304, 59730688,
         4623872, 4111104, 2635520, 657071872, 132697220096, 5680384, 5096192]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_footprint(i):
    cell, prec, flags, block = CASES[i]
    assert pw.plan(cell, prec, flags=flags, filter_block=block).footprint_bytes <= BYTES[i]
