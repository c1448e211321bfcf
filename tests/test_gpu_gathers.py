"""How the feature kernels fetch rows: channel counts that end inside a piece, a slab or a group of lanes, lists of more
offsets than a wave has lanes, and features that lie beyond the reach of 32-bit byte offsets."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_20834_amd import binding as B
from paper_2511_20834_amd import synth

from gpu_common import assert_close, fit_desc, gpu_pack, to_torch

pytestmark = pytest.mark.gpu

# fp16 / bf16: the output's own rounding (2^-11, 2^-8) and fp32 sums in another order; fp32: at most 125 * 96 products, whose
# rounding errors of 2^-24 each add up like their square root to about 1e-5 of the largest sum at the worst, 1e-6 as measured
TOL = {torch.float16: 2e-3, torch.bfloat16: 1e-2, torch.float32: 1e-5}


def _level(n, density, K, layout=B.LAYOUT_OS):
    side = max(3, int(round((n / density) ** (1 / 3))) + 1)
    lin = np.random.default_rng(n + K).choice(side ** 3, size=n, replace=False)
    c = np.stack([np.zeros(n, np.int64), lin // (side * side), lin // side % side, lin % side], 1).astype(np.int32)
    desc = fit_desc(c, [(K, 1, 1)])
    keys, _ = gpu_pack(c, desc)
    cs, _ = oracle.sort_coords(c)
    return B.spc_build_kmap(keys, desc, K, layout=layout), oracle.kernel_map(cs, cs, K, 1)


def _tensors(n, kvol, cin, cout, dtype):
    src = np.float32 if dtype == torch.float32 else np.float16
    F = to_torch(synth.features(n, cin, src, seed=91), dtype)
    W = to_torch(synth.weights(kvol, cin, cout, src, seed=92), dtype)
    return *F, *W


@pytest.mark.parametrize("n,density,K", [(31, 0.5, 3), (4001, 0.3, 3), (2500, 0.6, 5)])
@pytest.mark.parametrize("cin,cout", [(16, 64), (24, 32), (32, 64), (48, 96), (64, 128), (96, 64), (192, 64)])
def test_phase_kernel_rows(n, density, K, cin, cout):
    km, M = _level(n, density, K)
    for dtype in (torch.float16, torch.bfloat16):
        F, F64, W, W64 = _tensors(n, K ** 3, cin, cout, dtype)
        y = B.spc_conv_forward(km, F, W, flags=B.CONV_OS_PHASE)
        assert_close(y.cpu().to(torch.float64).numpy(), oracle.conv(M, F64, W64), TOL[dtype], (cin, cout, dtype))
    km.destroy()


def _far_apart(F):
    """The same rows with a pitch that puts them on more than 2 GiB."""
    pitch = (((1 << 31) // F.element_size()) // F.shape[0] + 64) // 64 * 64
    wide = torch.empty((F.shape[0], pitch), dtype=F.dtype, device=F.device)
    wide[:, : F.shape[1]] = F
    assert wide.numel() * wide.element_size() > 1 << 31
    return wide[:, : F.shape[1]]


@pytest.mark.parametrize("cin", [32, 64])
def test_phase_kernel_far_rows(cin):
    n = 3001
    km, M = _level(n, 0.3, 3)
    F, F64, W, W64 = _tensors(n, 27, cin, 64, torch.float16)
    y = B.spc_conv_forward(km, _far_apart(F), W, flags=B.CONV_OS_PHASE)
    assert_close(y.cpu().to(torch.float64).numpy(), oracle.conv(M, F64, W64), TOL[torch.float16], cin)
    km.destroy()


# SPC_CONV_SPLITK_RB: 32-row blocks per workgroup, one (four waves share a block) or two; 0: by size
@pytest.mark.parametrize("n,density,K", [(1, 1.0, 3), (33, 0.5, 3), (4001, 0.3, 3), (2500, 0.6, 5)])
@pytest.mark.parametrize("cin,cout", [(4, 32), (8, 32), (16, 64), (24, 40), (32, 32), (40, 64), (48, 96), (64, 64), (96, 32)])
@pytest.mark.parametrize("rb", [0, 1, 2])
def test_splitk_rows(n, density, K, cin, cout, rb):
    km, M = _level(n, density, K, B.LAYOUT_BOTH)
    for dtype in (torch.float16, torch.bfloat16, torch.float32):
        F, F64, W, W64 = _tensors(n, K ** 3, cin, cout, dtype)
        ref = oracle.conv(M, F64, W64)
        flags = B.CONV_OS_SPLITK | rb << 8
        runs = [(W, B.DATAFLOW_OS, flags), (W, B.DATAFLOW_WS, rb << 8)]
        if dtype != torch.float32 and cout in (32, 64):
            Wp = B.spc_conv_prepare_weights(W)
            runs += [(Wp, B.DATAFLOW_OS, flags | B.CONV_PACKED_WEIGHTS), (Wp, B.DATAFLOW_WS, rb << 8 | B.CONV_PACKED_WEIGHTS)]
        for w, df, fl in runs:
            y = B.spc_conv_forward(km, F, w, df, fl)
            assert_close(y.cpu().to(torch.float64).numpy(), ref, TOL[dtype], (dtype, df, fl))
        y = B.spc_conv_forward(km, F, W, flags=rb << 8, hybrid_t=2)
        assert_close(y.cpu().to(torch.float64).numpy(), ref, TOL[dtype], (dtype, "hybrid"))
    km.destroy()


@pytest.mark.parametrize("n,cin,cout", [(41_003, 4, 32), (153_701, 32, 32), (16_411, 32, 32)])
def test_splitk_two_blocks_per_workgroup(n, cin, cout):
    """Sizes from which a workgroup takes two blocks by itself (and, of fp32, those from which rows pass through LDS)."""
    km, M = _level(n, 0.02, 3, B.LAYOUT_BOTH)
    for dtype in (torch.float16, torch.float32):
        F, F64, W, W64 = _tensors(n, 27, cin, cout, dtype)
        ref = oracle.conv(M, F64, W64)
        for df in (B.DATAFLOW_OS, B.DATAFLOW_WS):
            y = B.spc_conv_forward(km, F, W, df)
            assert_close(y.cpu().to(torch.float64).numpy(), ref, TOL[dtype], (dtype, df))
    km.destroy()


@pytest.mark.parametrize("dtype,cin,cout", [(torch.float16, 64, 64), (torch.float16, 24, 40), (torch.float16, 4, 32), (torch.float32, 32, 32),
                                            (torch.float16, 20, 40), (torch.float32, 30, 32)])
def test_splitk_far_rows(dtype, cin, cout):
    n = 3001
    km, M = _level(n, 0.3, 3, B.LAYOUT_BOTH)
    F, F64, W, W64 = _tensors(n, 27, cin, cout, dtype)
    ref, far = oracle.conv(M, F64, W64), _far_apart(F)
    runs = [(W, B.DATAFLOW_OS, B.CONV_OS_SPLITK), (W, B.DATAFLOW_WS, 0)]
    if cout % 32 == 0 and dtype != torch.float32:
        runs.append((B.spc_conv_prepare_weights(W), B.DATAFLOW_OS, B.CONV_OS_SPLITK | B.CONV_PACKED_WEIGHTS))
    for w, df, fl in runs:
        y = B.spc_conv_forward(km, far, w, df, fl)
        assert_close(y.cpu().to(torch.float64).numpy(), ref, TOL[dtype], (df, fl))
    km.destroy()


@pytest.mark.parametrize("dtype,cin,pitch,cout", [
    (torch.float16, 1001, 1001, 80_000),   # a channel count that ends inside a piece
    (torch.bfloat16, 1000, 1003, 80_000),  # rows that are not aligned
    (torch.float16, 1000, 1000, 80_000),
    (torch.float32, 501, 501, 80_000),
    (torch.float16, 64, 64, 1_250_016),    # channels of which the kernel with resident weights has a form, and tiles enough for it
    (torch.float32, 32, 32, 1_250_016),
])
def test_splitk_far_weights(dtype, cin, pitch, cout):
    """Weights of more than 4 GiB: neither their bytes nor their number of 16-bit channels fits 32 bits."""
    n = 40
    km, M = _level(n, 0.6, 3, B.LAYOUT_BOTH)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(cin)
    F = torch.randn(n, pitch, generator=gen, device="cuda").to(dtype)[:, pitch - cin:]
    W = torch.empty(27, cin, cout, dtype=dtype, device="cuda")
    assert W.numel() * W.element_size() > 1 << 32
    ref = torch.zeros(n, cout, dtype=torch.float64, device="cuda")
    for k in range(27):
        W[k] = (torch.randn(cin, cout, generator=gen, device="cuda") * cin ** -0.5).to(dtype)
        for c in range(0, cout, 16_000):  # (the products of an offset, in 64 bits)
            j = torch.from_numpy(M[:, k].astype(np.int64)).cuda()
            ref[:, c:c + 16_000] += (F[j.clamp_min(0)].double() * (j >= 0)[:, None]) @ W[k, :, c:c + 16_000].double()
    runs = [(W, B.DATAFLOW_OS, B.CONV_OS_SPLITK if dtype != torch.float32 else 0), (W, B.DATAFLOW_WS, 0), (W, B.DATAFLOW_OS, 0)]
    if dtype != torch.float32:
        runs.append((B.spc_conv_prepare_weights(W), B.DATAFLOW_OS, B.CONV_OS_SPLITK | B.CONV_PACKED_WEIGHTS))
    for w, df, fl in runs:
        y = B.spc_conv_forward(km, F, w, df, fl).double()
        scale = ref.abs().max()
        assert float((y - ref).abs().max() / scale) <= TOL[dtype], (df, fl)
        assert bool(((y - ref).abs() <= TOL[dtype] * (ref.abs() + ref.square().mean().sqrt())).all()), (df, fl)
    km.destroy()
    B.spc_release_cache()


# (more tiles than half the CUs: slabs of 128 columns; one and three slabs of channels per offset: odd numbers of entries per wave)
@pytest.mark.parametrize("density", [0.02, 0.3])
@pytest.mark.parametrize("cin", [16, 48])
def test_wide_slabs_of_large_kernels(density, cin):
    n, cout = 4203, 128
    for layout, dataflow in ((B.LAYOUT_OS, B.DATAFLOW_OS), (B.LAYOUT_WS, B.DATAFLOW_WS)):
        km, M = _level(n, density, 5, layout)
        F, F64, W, W64 = _tensors(n, 125, cin, cout, torch.float16)
        y = B.spc_conv_forward(km, F, B.spc_conv_prepare_weights(W), dataflow, B.CONV_PACKED_WEIGHTS)
        assert_close(y.cpu().to(torch.float64).numpy(), oracle.conv(M, F64, W64), TOL[torch.float16], (density, cin, layout))
        km.destroy()


# (grids whose bound of the output rows lies above the lines where two waves share a tile instead of four, and whose count lies below)
@pytest.mark.parametrize("side,K,cin,cout,dataflow", [(40, 2, 32, 32, B.DATAFLOW_OS), (40, 3, 4, 32, B.DATAFLOW_OS),
                                                      (40, 2, 32, 64, B.DATAFLOW_WS), (56, 3, 32, 32, B.DATAFLOW_OS)])
def test_sums_are_the_same_before_and_after_the_count_is_known(side, K, cin, cout, dataflow):
    """The same map, inputs and flags: bit by bit, whatever the host knows of the output count when the layer is enqueued."""
    c = synth.full_grid(side)
    n = len(c)
    desc = fit_desc(c, [(K, 1, 2)])
    keys, _ = gpu_pack(c, desc)
    F, _, W, _ = _tensors(n, K ** 3, cin, cout, torch.float16)
    km = B.spc_build_kmap(keys, desc, K, 1, 2, 0, B.LAYOUT_OS if dataflow == B.DATAFLOW_OS else B.LAYOUT_WS)
    flags = B.CONV_OS_SPLITK if dataflow == B.DATAFLOW_OS else 0

    def forward():
        out = torch.empty((n, cout), dtype=torch.float16, device="cuda")
        B.spc_conv_forward(km, F, W, dataflow, flags, out=out)
        return out

    bound = forward()
    km.set_size_hint((side // 2) ** 3 // 2)
    hinted = forward()
    assert km.n_out == (side // 2) ** 3
    known = forward()[: km.n_out]
    assert torch.equal(known, bound[: km.n_out]) and torch.equal(known, hinted[: km.n_out])
    km.destroy()
