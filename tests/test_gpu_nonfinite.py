"""Infinities and NaN in single features and weights: an output is not finite exactly where its own pairs make it so, through
every feature kernel.  (A matrix instruction multiplies whole 32-row cells, and zero times infinity is NaN.)"""
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2511_20834_amd import binding as B
from paper_2511_20834_amd import synth

from gpu_common import assert_close, fit_desc, gpu_pack, oracle_layer, to_torch

pytestmark = pytest.mark.gpu

TOL = {torch.float16: 1e-2, torch.bfloat16: 1e-2, torch.float32: 1e-5}
INF, NAN = float("inf"), float("nan")


@functools.lru_cache(maxsize=None)
def _level(n, density, K, s_l):
    """(coordinates, M) of n uniformly random voxels and of the layer's map."""
    side = int(round((n / density) ** (1 / 3))) + 1
    lin = np.random.default_rng(n + K).choice(side ** 3, size=n, replace=False)
    c = np.stack([np.zeros_like(lin), lin // (side * side), lin // side % side, lin % side], 1).astype(np.int32)
    cs, _ = oracle.sort_coords(c)
    return cs, oracle_layer(cs, K, 1, s_l)[2]


def _check(got, ref, tol, relu, what):
    got = got.cpu().to(torch.float64).numpy()
    if relu:  # max(x, 0) of NaN is 0
        ref = np.where(np.isnan(ref), 0.0, np.maximum(ref, 0.0))
    assert np.array_equal(np.isnan(got), np.isnan(ref)), (what, int(np.isnan(got).sum()), int(np.isnan(ref).sum()))
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], ref[inf]), what
    ok = np.isfinite(ref)
    assert_close(np.where(ok, got, 0.0), np.where(ok, ref, 0.0), tol, what)


SPARSE, DENSE = (135_007, 0.0125), (6_001, 0.25)
OS, WS = B.DATAFLOW_OS, B.DATAFLOW_WS


@pytest.mark.parametrize("cloud,K,s_l,dtype,cin,cout,packed,dataflow,hybrid,flags", [
    (SPARSE, 3, 1, torch.float16, 32, 64, True, OS, None, B.CONV_OS_PHASE),            # pooled pairs
    (SPARSE, 3, 1, torch.bfloat16, 32, 64, False, OS, None, B.CONV_OS_PHASE | B.CONV_RELU),
    (DENSE, 3, 1, torch.float16, 32, 64, True, OS, None, B.CONV_OS_PHASE),             # phases, 64 and 32 columns
    (DENSE, 3, 1, torch.bfloat16, 16, 32, True, OS, None, B.CONV_OS_PHASE | B.CONV_RELU),
    (DENSE, 5, 1, torch.float16, 32, 64, False, OS, None, B.CONV_OS_PHASE),
    (DENSE, 3, 1, torch.float16, 24, 64, False, OS, None, B.CONV_OS_PHASE),            # padded copy of the rows
    (SPARSE, 3, 1, torch.float16, 32, 64, True, OS, None, B.CONV_OS_SPLITK),
    (DENSE, 3, 1, torch.float16, 256, 256, True, OS, None, B.CONV_OS_SPLITK | B.CONV_RELU),  # tiles shared by workgroups
    (DENSE, 3, 1, torch.bfloat16, 32, 256, True, OS, None, B.CONV_OS_SPLITK),
    (DENSE, 3, 1, torch.float16, 32, 64, True, OS, None, B.CONV_OS_SPLITK | 2 << 8),   # two row blocks per workgroup
    (DENSE, 3, 1, torch.bfloat16, 32, 40, False, OS, None, 0),
    (DENSE, 5, 1, torch.float16, 32, 32, True, OS, None, 0),
    (DENSE, 3, 1, torch.float32, 32, 64, False, OS, None, B.CONV_RELU),
    (DENSE, 3, 1, torch.float32, 6, 10, False, OS, None, 0),
    (DENSE, 3, 1, torch.float16, 24, 40, False, OS, None, 0),                          # channels that end inside a slab
    (DENSE, 3, 1, torch.float16, 24, 64, True, OS, None, 0),
    (DENSE, 3, 1, torch.bfloat16, 5, 33, False, OS, None, 0),                          # channel by channel
    (DENSE, 3, 1, torch.float16, 4, 32, True, OS, None, 0),                            # four offsets per slab
    (DENSE, 3, 1, torch.float16, 4, 32, False, WS, None, B.CONV_RELU),
    (DENSE, 3, 1, torch.float16, 32, 64, True, WS, None, 0),                           # lists
    (DENSE, 3, 1, torch.float32, 32, 32, False, WS, None, 0),
    (DENSE, 5, 1, torch.bfloat16, 32, 32, True, OS, 3, 0),
    (DENSE, 3, 1, torch.float16, 16, 48, False, OS, 2, B.CONV_RELU),
    (DENSE, 3, 2, torch.float16, 32, 64, True, OS, None, 0),                           # output count on the device only
    (DENSE, 3, 2, torch.float32, 32, 32, False, WS, None, 0),
])
def test_not_finite_only_where_its_pairs_are(cloud, K, s_l, dtype, cin, cout, packed, dataflow, hybrid, flags):
    cs, M = _level(*cloud, K, s_l)
    n, kvol = len(cs), K ** 3
    desc = fit_desc(cs, [(K, 1, s_l)])
    keys, _ = gpu_pack(cs, desc)
    F = synth.features(n, cin, np.float16, seed=71).astype(np.float32)
    W = synth.weights(kvol, cin, cout, np.float16, seed=72).astype(np.float32)
    bad_f, bad_w = F.copy(), W.copy()
    rows = np.random.default_rng(73).choice(n, size=9, replace=False)
    for r, v in zip(rows, [INF, -INF, NAN] * 3):
        bad_f[r, r % cin] = v
    bad_w[1, cin - 1, 0] = NAN          # (the last channel's weights may stand in for channels past the end)
    bad_w[kvol - 2, 0, cout - 1] = INF
    bad_w[kvol // 2 + 1, cin // 2, cout // 2] = -INF
    if hybrid is not None:
        layout = B.LAYOUT_BOTH | B.LAYOUT_HYBRID_T(hybrid)
    else:
        layout = B.LAYOUT_OS if dataflow == OS else B.LAYOUT_WS
    for what, f, w in (("features", bad_f, W), ("weights", F, bad_w), ("both", bad_f, bad_w)):
        Ft, F64 = to_torch(f, dtype)
        Wt, W64 = to_torch(w, dtype)
        with np.errstate(invalid="ignore"):
            ref = oracle.conv(M, F64, W64)
        km = B.spc_build_kmap(keys, desc, K, 1, s_l, 0, layout)
        out, fl = None, flags
        if s_l > 1:  # grids sized from an estimate, tiles walked with a stride
            km.set_size_hint(len(M) // 3)
            out = torch.empty((n, cout), dtype=dtype, device="cuda")
        if packed:
            Wt, fl = B.spc_conv_prepare_weights(Wt), flags | B.CONV_PACKED_WEIGHTS
        y = B.spc_conv_forward(km, Ft, Wt, dataflow, fl, out=out, hybrid_t=hybrid)[: len(M)]
        assert np.isfinite(ref).any() and not np.isfinite(ref).all()
        _check(y, ref, TOL[dtype], flags & B.CONV_RELU, what)
        km.destroy()


@pytest.mark.parametrize("K", [3, 5])
def test_not_finite_through_a_symmetric_half_map(K):
    cs, M = _level(*DENSE, K, 1)
    desc = fit_desc(cs, [(K, 1, 1)])
    keys, _ = gpu_pack(cs, desc)
    W = synth.weights(K ** 3, 16, 32, np.float16, seed=75).astype(np.float32)
    W[2, 3, 4], W[K ** 3 - 1, 0, 31], W[K ** 3 // 2, 5, 6] = NAN, INF, -INF  # stored half, mirrored half, centre
    Ft, F64 = to_torch(synth.features(len(cs), 16, np.float16, seed=74), torch.float16)
    Wt, W64 = to_torch(W, torch.float16)
    km = B.spc_build_kmap(keys, desc, K, 1, 1, 0, B.LAYOUT_WS | B.LAYOUT_WS_SYM)
    _check(B.spc_conv_forward(km, Ft, Wt, WS), oracle.conv(M, F64, W64), 1e-2, False, "weights")
    km.destroy()
