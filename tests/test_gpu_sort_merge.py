"""The sort's merge pass where its workgroups' shares are uneven: bins that are shared between workgroups, repeated and rejected rows, empty
stretches of the key space, and the sizes at which shares and kernels change."""
import numpy as np
import pytest
import torch

from paper_2511_20834_amd import binding as B

from gpu_common import fit_desc, keys_to_u64

pytestmark = pytest.mark.gpu


def _dense(n, dims, seed, far):
    """n voxels of a box, all but a few of them in a few bins: one voxel lies `far` away."""
    lin = np.random.default_rng(seed).choice(int(np.prod(dims)), size=n - 1, replace=False)
    c = np.stack([np.zeros(n - 1, np.int64), lin // (dims[1] * dims[2]), lin // dims[2] % dims[1], lin % dims[2]], 1)
    return np.random.default_rng(seed + 1).permutation(np.concatenate([c, [[0, *far]]])).astype(np.int32)


def _check(c, desc):
    keys, perm = B.spc_pack_coords(torch.from_numpy(c).cuda(), desc)
    k = keys_to_u64(keys)
    assert np.all(k[1:] > k[:-1])
    assert np.array_equal(perm.cpu().numpy(), np.lexsort((c[:, 3], c[:, 2], c[:, 1])))
    m = B.spc_build_kmap(keys, desc, 3, 1, 2, 0, B.LAYOUT_OS)
    coarse = np.unique(c[:, 1:] // 2, axis=0)
    assert m.n_out == len(coarse)
    got = m.out_keys()
    m.destroy()
    half = np.concatenate([np.zeros((len(coarse), 1), np.int64), 2 * coarse], 1).astype(np.int32)
    half = half[np.lexsort((half[:, 3], half[:, 2], half[:, 1]))]
    want = keys_to_u64(B.spc_pack_coords(torch.from_numpy(half).cuda(), desc)[0])
    assert np.array_equal(got, want)


# (a bin of more than 2048 keys is shared, beyond 524 288 keys in all one of more than 4096)
@pytest.mark.parametrize("n,dims,far", [
    (20_000, (2, 150, 150), (4000, 4000, 200)),    # one bin holds nearly everything
    (20_000, (24, 30, 30), (2000, 10, 10)),        # bins of about 1000
    (20_000, (30, 30, 30), (1 << 19, 1 << 19, 1 << 19)),  # second bins, and theirs, are split again
    (150_000, (2, 400, 300), (1000, 1000, 300)),
    (260_000, (3, 500, 400), (4000, 4000, 400)),
    (524_288, (4, 700, 400), (4000, 4000, 400)),
    (524_289, (4, 700, 400), (4000, 4000, 400)),
    (600_001, (4, 700, 400), (4000, 4000, 400)),
])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_bins_beyond_the_lds(n, dims, far, key_bits):
    c = _dense(n, dims, n, far)
    _check(c, fit_desc(c, [(3, 1, 2)], key_bits))


# (a bin is a plane of x here)
@pytest.mark.parametrize("n,planes,most,q", [(20_000, 2000, 2048, 512), (530_000, 16_000, 4096, 2048)])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_bins_around_the_line(n, planes, most, q, key_bits):
    sizes = [most - 1, most, most + 1, q - 1, most - q + 2, 1, most + 1, q, q + 1, most + q]
    x = np.concatenate([np.full(s, p) for p, s in enumerate(sizes)] + [np.full(most + 1, planes - 1), np.full(most, planes - 3)])
    rest = np.random.default_rng(n).integers(len(sizes), planes - 3, size=n - len(x))
    x = np.concatenate([x, rest])
    yz = np.random.default_rng(n + 1).choice(300 * 200, size=n, replace=n > 300 * 200)
    c = np.unique(np.stack([np.zeros(n, np.int64), x, yz // 200, yz % 200], 1), axis=0)
    if len(c) < n:  # (the rows that met, in planes of their own)
        i = np.arange(n - len(c))
        c = np.concatenate([c, np.stack([0 * i, 20 + i // 50, 300 + 0 * i, i % 50], 1)])
    _check(np.random.default_rng(n + 2).permutation(c).astype(np.int32), fit_desc(c, [(3, 1, 2)], key_bits))


# (wide workgroups that read the totals, and 8192 bins: a plane of x each)
@pytest.mark.parametrize("n", [200_001, 300_000, 300_001, 524_288])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_bins_around_the_line_of_wide_merges(n, key_bits):
    test_bins_around_the_line(n, 8000, 4096, 2048, key_bits)


def _microseconds(f):
    f()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(5):
        start.record()
        f()
        f()
        end.record()
        end.synchronize()
        best = min(best, 500 * start.elapsed_time(end))
    return best


@pytest.mark.parametrize("kind", ["wall", "outlier", "slab"])
def test_crowded_bins_are_shared(kind):
    """120 k voxels, many or all of them in one bin, against as many spread over the key space.  A crowded bin is 2 to 6 times the time
    (levels: 2 to 7); with one workgroup to sort it, it was 24 to 900 times."""
    n = 120_000
    rng = np.random.default_rng(7)

    def box(m, dims, at=(0, 0, 0)):
        lin = rng.choice(int(np.prod(dims)), size=m, replace=False)
        return np.stack([np.zeros(m, np.int64), at[0] + lin // (dims[1] * dims[2]), at[1] + lin // dims[2] % dims[1], at[2] + lin % dims[2]], 1)

    spread = box(n, (2000, 2000, 100))
    if kind == "wall":  # a sixth of the scene in one plane of x
        c = np.concatenate([box(n // 6, (1, 1000, 200), (501, 0, 0)), box(n - n // 6, (500, 2000, 200))])
    elif kind == "outlier":  # all of it but one voxel
        c = np.concatenate([box(n - 1, (136, 136, 136)), [[0, 600_000, 0, 0]]])
    else:
        c = np.concatenate([box(n - 1, (2, 348, 348)), [[0, 60_000, 0, 0]]])
    times = []
    for cloud in (spread, c):
        cloud = rng.permutation(cloud).astype(np.int32)
        desc = fit_desc(cloud, [(2, 1, 2)], 64)
        if kind == "wall":
            desc.bits_x, desc.bits_y, desc.bits_z = 12, 12, 8
        d = torch.from_numpy(cloud).cuda()
        ws = torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device="cuda")
        keys, perm = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
        times.append((_microseconds(lambda: B.spc_pack_coords(d, desc, True, 0, None, ws, keys, perm)),
                      _microseconds(lambda: B.spc_build_kmap(keys, desc, 2, 1, 2, 0, B.LAYOUT_OS).destroy())))
        assert bool((keys[1:] > keys[:-1]).all())
    assert times[1][0] < 15 * times[0][0] and times[1][1] < 15 * times[0][1], times


# (the last workgroup takes what is left of the box and the far voxel's bin: a few second bins hold all its keys)
@pytest.mark.parametrize("n,dims,far", [(6000, (40, 20, 20), (4000, 0, 0)), (120_000, (60, 60, 60), (1500, 10, 10)), (200_001, (70, 70, 70), (2000, 10, 10)),
                                        (300_000, (80, 80, 80), (2000, 10, 10)), (300_001, (400, 400, 100), (4000, 4000, 100)),
                                        (524_288, (96, 96, 96), (500, 10, 10)), (700_000, (110, 110, 110), (2000, 10, 10))])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_second_bins_that_hold_many(n, dims, far, key_bits):
    c = _dense(n, dims, n, far)
    _check(c, fit_desc(c, [(3, 1, 2)], key_bits))


@pytest.mark.parametrize("key_bits", [0, 64])
def test_a_far_voxel_costs_no_more_than_a_spread_cloud(key_bits):
    """300 k voxels in a box beside one far away: 0.9 times as long as spread ones; 1.7 (64-bit keys 2.3) where the last workgroup compared all its keys with each other."""
    n, times = 300_000, []
    for c in (_dense(n, (350, 350, 200), 5, (0, 0, 0)), _dense(n, (80, 80, 80), 5, (2000, 10, 10))):
        c = np.unique(c, axis=0)
        c = np.random.default_rng(6).permutation(c).astype(np.int32)
        desc, d = fit_desc(c, [(3, 1, 2)], key_bits), torch.from_numpy(c).cuda()
        ws = torch.empty(B.spc_pack_workspace_bytes(len(c), desc), dtype=torch.uint8, device="cuda")
        keys, perm = B.spc_pack_coords(d, desc)
        times.append(_microseconds(lambda: [B.spc_pack_coords(d, desc, True, 0, None, ws, keys, perm) for _ in range(10)]))
    assert times[1] < 1.3 * times[0], times


@pytest.mark.parametrize("n", [4096, 5000, 70_000, 230_000, 524_289, 1_300_001])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_two_distant_clusters(n, key_bits):
    a, b = _dense(n // 2, (100, 120, 130), n, (99, 0, 0)), _dense(n - n // 2, (90, 110, 150), n + 1, (0, 0, 149))
    a, b = np.unique(a, axis=0), np.unique(b, axis=0)
    b[:, 1:3] += 1800
    c = np.random.default_rng(n).permutation(np.concatenate([a, b])).astype(np.int32)
    _check(c, fit_desc(c, [(3, 1, 2)], key_bits))


@pytest.mark.parametrize("n", [4096, 30_000, 300_000, 700_000])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_repeated_and_rejected_rows(n, key_bits):
    """Not a valid cloud, but the permutation stays a complete one, keys ascend and rejected rows come last."""
    rng = np.random.default_rng(n)
    c = np.concatenate([np.zeros((n, 1), np.int64), rng.integers(0, 12, (n, 3))], 1).astype(np.int32)  # 1728 distinct voxels
    desc = fit_desc(c, [(3, 1, 2)], key_bits)
    bad = rng.permutation(n)[:n // 3]
    c[bad, 2] = 1 << 20
    keys, perm = B.spc_pack_coords(torch.from_numpy(c).cuda(), desc)
    k, p = keys_to_u64(keys), perm.cpu().numpy()
    assert np.array_equal(np.sort(p), np.arange(n))
    assert np.all(k[1:] >= k[:-1])
    last = np.uint64(0xffffffffffffffff) if desc.key_bits == 64 else np.uint64(0xffffffff)
    assert np.all(k[n - len(bad):] == last) and np.all(k[:n - len(bad)] < last)
    assert np.array_equal(np.sort(p[n - len(bad):]), np.sort(bad))
    s = c[p[:n - len(bad)]].astype(np.int64)
    lin = (s[:, 1] * 4096 + s[:, 2]) * 4096 + s[:, 3]
    assert np.all(lin[1:] >= lin[:-1])


@pytest.mark.parametrize("n,dims", [(20_000, (2, 150, 150)), (40_000, (40, 40, 40)), (150_000, (2, 400, 300))])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_shared_bins_without_kept_totals(n, dims, key_bits):
    """On the thread's own stream (the table is summed, or the totals cleared first), and recorded (so are the levels' bins)."""
    c = _dense(n, dims, n, (4000, 4000, 400))
    desc, order = fit_desc(c, [(3, 1, 2)], key_bits), np.lexsort((c[:, 3], c[:, 2], c[:, 1]))
    coords = torch.from_numpy(c).cuda()
    torch.cuda.synchronize()
    keys, perm = B.spc_pack_coords(coords, desc, stream=2)  # (hipStreamPerThread)
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy(), order)
    m = B.spc_build_kmap(keys, desc, 3, 1, 2, 0, B.LAYOUT_OS)
    want = m.out_keys()
    m.destroy()
    ws = torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device="cuda")
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()

    def step():
        B.spc_pack_coords(coords, desc, True, 0, None, ws, keys, perm)
        return B.spc_build_kmap(keys, desc, 3, 1, 2, 0, B.LAYOUT_OS)

    with torch.cuda.stream(side):
        step().destroy()  # (warm)
    side.synchronize()
    with torch.cuda.graph(g, stream=side):
        m = step()
    for _ in range(3):
        keys.zero_()
        perm.zero_()
        ws.fill_(255)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(perm.cpu().numpy(), order)
        assert np.array_equal(m.out_keys(), want)
        B.spc_pack_coords(coords, desc)
    torch.cuda.synchronize()
    del g
    m.destroy()


@pytest.mark.parametrize("n", [4097, 40_000])
def test_on_the_threads_own_stream(n):
    """No totals are kept there: the table is summed, or the totals cleared first."""
    c = _dense(n, (60, 80, 90), n, (400, 5, 5))
    desc = fit_desc(c, [(3, 1, 2)])
    coords = torch.from_numpy(c).cuda()
    torch.cuda.synchronize()
    keys, perm = B.spc_pack_coords(coords, desc, stream=2)  # (hipStreamPerThread)
    torch.cuda.synchronize()
    assert np.all(np.diff(keys_to_u64(keys).astype(np.int64)) > 0)
    assert np.array_equal(perm.cpu().numpy(), np.lexsort((c[:, 3], c[:, 2], c[:, 1])))


# (beyond 2.9 M keys a split workgroup's share is the longest, 12 288 of them; beyond 6 M there are more regions than rows in the tables of
# recorded sorts, and the workspace has a term for them)
@pytest.mark.parametrize("n", [3_000_001, 6_500_000, 8192 * 1024])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_largest_sizes(n, key_bits):
    """With a workspace exactly as large as reported."""
    lin = np.random.default_rng(n).permutation(n).astype(np.int64) * 7 + 3
    c = np.stack([0 * lin, lin // 140_000, lin // 200 % 700, lin % 200], 1).astype(np.int32)
    desc = fit_desc(c, [(3, 1, 2)], key_bits)
    need = B.spc_pack_workspace_bytes(n, desc)
    block = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    keys = torch.empty(n, dtype=torch.int64 if desc.key_bits == 64 else torch.int32, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    B.spc_pack_coords(torch.from_numpy(c).cuda(), desc, True, 0, None, block[:need], keys, perm)
    assert np.array_equal(perm.cpu().numpy(), np.argsort(lin))
    k = keys_to_u64(keys)
    assert np.all(k[1:] > k[:-1])
    assert bool((block[need:] == 0xA5).all())
    m = B.spc_build_kmap(keys, desc, 2, 1, 2, 0, B.LAYOUT_OS)
    half = (c[:, 1] // 2).astype(np.int64) * 35_000 + c[:, 2] // 2 * 100 + c[:, 3] // 2
    assert m.n_out == np.count_nonzero(np.bincount(half))
    m.destroy()
