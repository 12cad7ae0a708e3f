"""The viscous prepass where its plan changes, against the oracle's viscous right-hand side: block
sizes on both sides of 600k points (32 x 8 tiles below) and of 7M points (64 x 16 above), chosen
so that the shape does change between them and the last chunk along k is a shorter one; chunks of
several planes in the narrow tile, whose two LDS planes are then used in turn, also with the
one-sided closure and within the one launch of a small block.

Tolerances as for every viscous right-hand side of these flows: 5e-11 in FP64; in FP32 the
velocity enters rounded to 6e-8 of |u| ~ 0.7 and passes two sixth-order differences (together
< 4), the terms come from perturbations of 1e-3 per node, three such roundings: 5e-4.
"""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock, vector_norm_err

pytestmark = pytest.mark.gpu

VIS = 7 | B.CFD_TERM_VIS


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield


@pytest.mark.parametrize("size,precision", [
    ((81, 89, 82), B.CFD_FP64),     # 591k: narrow, 27 chunks of three planes and one of one
    ((61, 96, 103), B.CFD_FP64),    # 603k: wide, chunks of three, one of one
    ((151, 187, 247), B.CFD_FP64),  # 6.97M: narrow, chunks of 31, one of 30
    ((152, 188, 247), B.CFD_FP64),  # 7.06M: wide
    ((71, 101, 83), B.CFD_MIXED),   # 595k: narrow, chunks of four, one of three
    ((83, 89, 83), B.CFD_MIXED),    # 613k: wide, chunks of four, one of three
    ((138, 196, 257), B.CFD_MIXED),  # 6.95M: narrow, chunks of 33, one of 26
    ((139, 197, 257), B.CFD_MIXED)])  # 7.04M: wide
def test_viscous_rhs_where_the_plan_changes(size, precision):
    wl = W.vortex_wavy(size[0], nj=size[1], nk=size[2])
    c = O.cfg_from_workload(wl)
    dev = DevBlock(wl, precision=precision)
    try:
        err = vector_norm_err(dev.rhs(VIS), O.rhs(c, O.metrics(c, wl.blocks[0].xyz), wl.blocks[0].q, VIS))
    finally:
        dev.close()
    print(size, precision, err)
    assert err < (5e-11 if precision == B.CFD_FP64 else 5e-4)


@pytest.mark.parametrize("precision", [B.CFD_FP64, B.CFD_MIXED])
def test_closure_in_chunks_of_several_planes(precision):
    # walls along j, which tiles of eight rows cut unevenly (one row in the last)
    wl = dataclasses.replace(W.channel(81, 89, 82, reynolds=100.0), visc_closure=B.CFD_VISC_ONE_SIDED)
    c = O.cfg_from_workload(wl)
    q = O.bc_fill(c, O.periodic_wrap(c, O.wall_reset(c, wl.blocks[0].q)))
    dev = DevBlock(wl, q=q, precision=precision)
    try:
        err = vector_norm_err(dev.rhs(VIS), O.rhs(c, O.metrics(c, wl.blocks[0].xyz), q, VIS))
    finally:
        dev.close()
    print(precision, err)
    assert err < (5e-11 if precision == B.CFD_FP64 else 5e-4)


@pytest.mark.parametrize("size,precision", [
    ((33, 9, 367), B.CFD_FP64),     # chunks of two planes, one of one
    ((71, 101, 83), B.CFD_MIXED)])  # chunks of four, one of three
def test_prepass_within_the_launch_in_chunks_of_several_planes(size, precision):
    wl = W.vortex_wavy(size[0], nj=size[1], nk=size[2])
    dev = DevBlock(wl, precision=precision)
    try:
        assert B.cfd_block_sweep_forms(dev.h) == [B.CFD_SWEEP_ONE_LAUNCH] * 3
        got = dev.rhs().copy()
        B.cfd_block_set_tiles(dev.h, [5, 6, 6] if precision == B.CFD_FP64 else [5, 2, 2])
        np.testing.assert_array_equal(dev.rhs(), got)
    finally:
        dev.close()
