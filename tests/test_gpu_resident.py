"""The feature kernel that keeps a 3x3x3 layer's weights in LDS: every form of it (channel counts, types, dataflows, one or two waves to
a tile, rows that are stored in pieces or one channel at a time), NaN and infinities, and where it is taken by itself."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_20834_amd import binding as B
from paper_2511_20834_amd import synth

from gpu_common import assert_close, fit_desc, gpu_pack, oracle_layer, to_torch

pytestmark = pytest.mark.gpu

# the output's own rounding (2^-11, 2^-8), and fp32 sums of at most 27 * 64 products in another order
TOL = {torch.float16: 2e-3, torch.bfloat16: 1e-2, torch.float32: 1e-5}


def _cloud(n, density):
    side = max(3, int(round((n / density) ** (1 / 3))) + 1)
    lin = np.random.default_rng(n).choice(side ** 3, size=n, replace=False)
    return np.stack([np.zeros(n, np.int64), lin // (side * side), lin // side % side, lin % side], 1).astype(np.int32)


def _resident(km, F, W, waves=0, flags=0, **kw):
    """A forward pass that has to come to this kernel."""
    before = B.spc_resident_count()
    y = B.spc_conv_forward(km, F, W, flags=B.CONV_RESIDENT | waves << 8 | flags, **kw)
    assert B.spc_resident_count() == before + 1, "another kernel ran"
    return y


# (tiles: one that is not whole, the first of a chunk of the next XCD, several to a wave)
@pytest.mark.parametrize("n,density", [(1, 1.0), (33, 0.5), (4131, 0.3), (70_001, 0.05)])
@pytest.mark.parametrize("cin,cout", [(8, 32), (16, 64), (24, 40), (32, 32), (32, 128), (48, 96), (64, 64)])
def test_resident(n, density, cin, cout):
    c = _cloud(n, density)
    desc = fit_desc(c, [(3, 1, 1)])
    keys, _ = gpu_pack(c, desc)
    cs, _ = oracle.sort_coords(c)
    M = oracle.kernel_map(cs, cs, 3, 1)
    km = B.spc_build_kmap(keys, desc, 3, layout=B.LAYOUT_BOTH)
    km_h = B.spc_build_kmap(keys, desc, 3, layout=B.LAYOUT_BOTH | B.LAYOUT_HYBRID_T(2))
    for dtype in (torch.float16, torch.bfloat16, torch.float32):
        if dtype == torch.float32 and cin > 32:
            continue
        src = np.float32 if dtype == torch.float32 else np.float16
        F, F64 = to_torch(synth.features(n, cin, src, seed=91), dtype)
        W, W64 = to_torch(synth.weights(27, cin, cout, src, seed=92), dtype)
        ref = oracle.conv(M, F64, W64)
        Wp = B.spc_conv_prepare_weights(W) if dtype != torch.float32 and cout in (32, 64, 128) else None
        for waves in (1, 2):
            for kmap, kw in ((km, {"dataflow": B.DATAFLOW_OS}), (km, {"dataflow": B.DATAFLOW_WS}), (km_h, {"hybrid_t": 2})):
                y = _resident(kmap, F, W, waves, **kw)
                assert_close(y.cpu().to(torch.float64).numpy(), ref, TOL[dtype], (dtype, waves, kw))
                assert torch.equal(y, _resident(kmap, F, W, waves, **kw))
                if Wp is not None:
                    assert torch.equal(y, _resident(kmap, F, Wp, waves, B.CONV_PACKED_WEIGHTS, **kw))
                assert torch.equal(y.clamp_min(0), _resident(kmap, F, W, waves, B.CONV_RELU, **kw))
        # rows that no 16-byte store reaches: an odd pitch, and nothing between the rows is written
        wide = torch.full((n, cout + 3), 7.0, dtype=dtype, device="cuda")
        _resident(km, F, W, 2, out=wide[:, 1:1 + cout])
        assert torch.equal(wide[:, 1:1 + cout], _resident(km, F, W, 2))
        assert bool((wide[:, 0] == 7).all()) and bool((wide[:, 1 + cout:] == 7).all())
    km.destroy()
    km_h.destroy()


@pytest.mark.parametrize("cin,cout,dtype", [(32, 64, torch.float16), (64, 32, torch.bfloat16), (24, 40, torch.float16), (32, 32, torch.float32)])
@pytest.mark.parametrize("waves", [1, 2])
def test_resident_nonfinite(cin, cout, dtype, waves):
    """Infinities and NaN reach an output through its own pairs only, and ReLU makes 0 of NaN."""
    n = 5003
    c = _cloud(n, 0.3)
    desc = fit_desc(c, [(3, 1, 1)])
    keys, _ = gpu_pack(c, desc)
    cs, _ = oracle.sort_coords(c)
    M = oracle.kernel_map(cs, cs, 3, 1)
    src = np.float32 if dtype == torch.float32 else np.float16
    F, _ = to_torch(synth.features(n, cin, src, seed=3), dtype)
    W, _ = to_torch(synth.weights(27, cin, cout, src, seed=4), dtype)
    F[17, 3], F[4001, 0] = float("inf"), float("nan")
    W[2, 5, 7], W[20, 1, cout - 1] = float("-inf"), float("nan")
    Fd, Wd, j = F.double(), W.double(), torch.from_numpy(M.astype(np.int64)).cuda()
    want = torch.zeros(n, cout, dtype=torch.float64, device="cuda")
    for k in range(27):
        rows = torch.nonzero(j[:, k] >= 0)[:, 0]
        want[rows] += (Fd[j[rows, k]][:, :, None] * Wd[k][None]).sum(1)
    for layout, kw in ((B.LAYOUT_OS, {"dataflow": B.DATAFLOW_OS}), (B.LAYOUT_WS, {"dataflow": B.DATAFLOW_WS}),
                       (B.LAYOUT_BOTH | B.LAYOUT_HYBRID_T(2), {"hybrid_t": 2})):
        km = B.spc_build_kmap(keys, desc, 3, layout=layout)
        for relu in (0, B.CONV_RELU):
            y = _resident(km, F, W, waves, relu, **kw).double()
            ref = torch.where(torch.isnan(want), torch.zeros_like(want), want.clamp_min(0)) if relu else want
            assert torch.equal(torch.isnan(y), torch.isnan(ref)) and torch.equal(torch.isposinf(y), torch.isposinf(ref))
            assert torch.equal(torch.isneginf(y), torch.isneginf(ref))
            fin = torch.isfinite(ref)
            assert float((y[fin] - ref[fin]).abs().max() / ref[fin].abs().max()) <= TOL[dtype]
        km.destroy()


# (rows, density, cin, cout, type, dataflow, taken): on both sides of the lines; sums in another order than the split-k kernel's
@pytest.mark.parametrize("n,density,cin,cout,dtype,ws,want", [
    (95_000, 0.1, 64, 32, torch.float16, False, False), (97_000, 0.1, 64, 32, torch.float16, False, True),
    (79_000, 0.1, 64, 32, torch.float16, True, False), (81_000, 0.1, 64, 32, torch.float16, True, True),
    (50_000, 0.1, 48, 40, torch.bfloat16, False, True), (97_000, 0.1, 64, 64, torch.float16, False, False),
    (140_000, 0.1, 32, 64, torch.float16, False, True), (34_000, 0.1, 32, 64, torch.float32, False, True),
    (100_000, 0.1, 32, 32, torch.float32, False, False),
])
def test_resident_by_itself(n, density, cin, cout, dtype, ws, want):
    c = _cloud(n, density)
    desc = fit_desc(c, [(3, 1, 1)])
    keys, _ = gpu_pack(c, desc)
    km = B.spc_build_kmap(keys, desc, 3, layout=B.LAYOUT_WS if ws else B.LAYOUT_OS)
    src = np.float32 if dtype == torch.float32 else np.float16
    F, _ = to_torch(synth.features(n, cin, src, seed=5), dtype)
    W, _ = to_torch(synth.weights(27, cin, cout, src, seed=6), dtype)
    df = B.DATAFLOW_WS if ws else B.DATAFLOW_OS
    before = B.spc_resident_count()
    own = B.spc_conv_forward(km, F, W, df)
    assert B.spc_resident_count() - before == want
    assert torch.equal(own, B.spc_conv_forward(km, F, W, df, B.CONV_RESIDENT)) == want
    km.destroy()


def test_rows_that_lie_4_gib_apart():
    """Outputs whose pitch no 32-bit number holds: the split-k kernel's, also where this one is asked for."""
    c = np.array([[0, 0, 0, 0], [0, 0, 0, 1]], np.int32)
    desc = fit_desc(c, [(3, 1, 1)])
    keys, _ = gpu_pack(c, desc)
    km = B.spc_build_kmap(keys, desc, 3, layout=B.LAYOUT_OS)
    F, _ = to_torch(synth.features(2, 32, np.float16, seed=7), torch.float16)
    W, _ = to_torch(synth.weights(27, 32, 32, np.float16, seed=8), torch.float16)
    apart = torch.zeros((1 << 31) + 32, dtype=torch.float16, device="cuda")
    out = apart.as_strided((2, 32), (1 << 31, 1))
    B.spc_conv_forward(km, F, W, flags=B.CONV_RESIDENT, out=out)
    assert torch.equal(out, B.spc_conv_forward(km, F, W, flags=B.CONV_OS_SPLITK))
    assert int(torch.count_nonzero(apart)) == int(torch.count_nonzero(out))
    km.destroy()
    B.spc_release_cache()


@pytest.mark.parametrize("cin,cout,dtype", [(32, 32, torch.float16), (24, 40, torch.bfloat16), (64, 64, torch.float16), (32, 64, torch.float32)])
@pytest.mark.parametrize("stride,transposed", [(1, 0), (2, 0), (2, 1)])
def test_resident_levels_and_permuted_rows(cin, cout, dtype, stride, transposed):
    """Strided layers, by the level's bound, by an estimate of its rows and by their number; transposed ones; rows in the caller's order."""
    n = 30_011
    c = _cloud(n, 0.2)
    desc = fit_desc(c, [(3, 1, 2)])
    keys, perm = gpu_pack(c, desc)
    cs, _ = oracle.sort_coords(c)
    level_in, level_out, M = oracle_layer(cs, 3, 1, stride, transposed)
    src = np.float32 if dtype == torch.float32 else np.float16
    F, F64 = to_torch(synth.features(len(level_in), cin, src, seed=93), dtype)
    W, W64 = to_torch(synth.weights(27, cin, cout, src, seed=94), dtype)
    ref, n_out = oracle.conv(M, F64, W64), len(level_out)
    unsorted = torch.empty_like(F)
    if not transposed:
        unsorted[perm.long()] = F
    for layout, kw in ((B.LAYOUT_OS, {"dataflow": B.DATAFLOW_OS}), (B.LAYOUT_WS, {"dataflow": B.DATAFLOW_WS}),
                       (B.LAYOUT_BOTH | B.LAYOUT_HYBRID_T(2), {"hybrid_t": 2})):
        for waves in (1, 2):
            km = B.spc_build_kmap(keys, desc, 3, 1, stride, transposed, layout)

            def forward():
                out = torch.zeros((n, cout), dtype=dtype, device="cuda")
                _resident(km, F, W, waves, out=out, **kw)
                return out

            bound = forward()
            km.set_size_hint(n_out // 2)
            hinted = forward()
            assert km.n_out == n_out
            assert_close(bound[:n_out].cpu().to(torch.float64).numpy(), ref, TOL[dtype], (layout, waves))
            assert torch.equal(bound, hinted) and torch.equal(bound, forward()) and not bool(bound[n_out:].any())
            km.destroy()
            if not transposed:
                km = B.spc_build_kmap(keys, desc, 3, 1, stride, 0, layout, in_perm=perm)
                assert torch.equal(bound[:n_out], _resident(km, unsorted, W, waves, n_out=n_out, **kw))
                km.destroy()


@pytest.mark.parametrize("K,cin,cout,dtype", [(3, 96, 64, torch.float16), (5, 32, 32, torch.float16), (3, 20, 40, torch.float16), (3, 64, 32, torch.float32)])
@pytest.mark.parametrize("waves", [1, 2])
def test_layers_without_a_form_are_as_if_nothing_was_asked_for(K, cin, cout, dtype, waves):
    n = 9001
    c = _cloud(n, 0.3)
    desc = fit_desc(c, [(K, 1, 1)])
    keys, _ = gpu_pack(c, desc)
    km = B.spc_build_kmap(keys, desc, K, layout=B.LAYOUT_OS)
    src = np.float32 if dtype == torch.float32 else np.float16
    F, _ = to_torch(synth.features(n, cin, src, seed=9), dtype)
    W, _ = to_torch(synth.weights(K ** 3, cin, cout, src, seed=10), dtype)
    before = B.spc_resident_count()
    assert torch.equal(B.spc_conv_forward(km, F, W), B.spc_conv_forward(km, F, W, flags=B.CONV_RESIDENT | waves << 8))
    assert B.spc_resident_count() == before
    km.destroy()
