"""Workspace sizes stay within those of the previous layout (the figures here), so
that a caller's buffer of that size is still taken."""
import ctypes as C

import pytest

import paper_2605_26137_amd.bake as B


def batch_size(specs, save):
    A = (B.BakeAsset * len(specs))()
    for a, (hv, hf, lv, lf, res) in zip(A, specs):
        a.n_hi_v, a.n_hi_f, a.n_lo_v, a.n_lo_f, a.res, a.max_dist = hv, hf, lv, lf, res, 1.0
    o, n = B.make_options(2, save), C.c_size_t()
    assert B.lib().bake_batch_workspace_size(A, len(specs), C.byref(o), C.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("faces,tiny,before", [(2000, 100, 1459712), (2000, 10000, 105124352), (200000, 100, 36538368),
                                               (200000, 10000, 140207104), (200000, 65535, 721537792)])
def test_batches_of_tiny_assets(faces, tiny, before):
    """One asset of many tiles beside assets of a single face."""
    assert batch_size([(faces // 2, faces, 5, 4, 1)] + [(3, 1, 5, 4, 1)] * tiny, False) <= before


@pytest.mark.parametrize("sizes,before", [
    ((3, 1, 3, 1, 1), 99840), ((2562, 5120, 42, 80, 128), 7663104), ((12, 20, 42, 80, 4096), 2748890368),
    ((655362, 1310720, 10242, 20480, 2048), 1049435904), ((12, 20, 42, 80, 8192), 10492099840),
    ((12, 20, 42, 80, 16384), 41464937728)])
def test_saved_bakes(sizes, before):
    """Few faces onto large atlases above all: what the backward keeps per texel counts."""
    assert batch_size([sizes], True) <= before


def test_saved_batch():
    assert batch_size([(12, 20, 42, 80, 8192)] + [(3, 1, 5, 4, 1)] * 500, True) <= 10500167680


@pytest.mark.parametrize("n_v,n_f,before", [(3, 1, 11776), (12, 20, 16128), (10, 1000, 193792), (502, 1000, 351488),
                                            (10, 2560, 478720)])
def test_simplification(n_v, n_f, before):
    assert B.qem_workspace_size(n_v, n_f) <= before
