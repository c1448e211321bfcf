"""The sort's bin totals, which the library keeps cleared between its sorts: sizes around the lines where the workgroups' shares
change, sorts of different sizes one after the other, from several threads on one stream and on several, and in a graph that is
replayed between them."""
import threading

import numpy as np
import pytest
import torch

from paper_2511_20834_amd import binding as B

from gpu_common import fit_desc, keys_to_u64

pytestmark = pytest.mark.gpu


def _cloud(n, seed):
    side = int(round((n / 0.05) ** (1 / 3))) + 2
    lin = np.random.default_rng(seed).choice(side ** 3, size=n, replace=False)
    return np.stack([np.zeros(n, np.int64), lin // (side * side), lin // side % side, lin % side], 1).astype(np.int32)


def _check(c, keys, perm):
    k = keys_to_u64(keys)
    assert np.all(k[1:] > k[:-1])
    order = np.lexsort((c[:, 3], c[:, 2], c[:, 1]))
    assert np.array_equal(perm.cpu().numpy(), order)


@pytest.mark.parametrize("n", [4096, 4097, 65_535, 65_536, 65_537, 200_000, 200_001, 524_288, 524_289])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_sizes(n, key_bits):
    c = _cloud(n, n)
    desc = fit_desc(c, [(3, 1, 2)], key_bits)
    d = torch.from_numpy(c).cuda()
    for _ in range(3):
        keys, perm = B.spc_pack_coords(d, desc)
        _check(c, keys, perm)
        m = B.spc_build_kmap(keys, desc, 3, 1, 2, 0, B.LAYOUT_OS)  # the level of stride 2 is sorted on the same path
        assert m.n_out == len(np.unique(c[:, 1:] // 2, axis=0))
        m.destroy()


def test_threads_and_streams():
    clouds = [_cloud(n, i) for i, n in enumerate((5000, 30_011, 70_001, 121_003, 300_007))]
    descs = [fit_desc(c, [(3, 1, 1)]) for c in clouds]
    dev = [torch.from_numpy(c).cuda() for c in clouds]
    shared = torch.cuda.Stream()
    torch.cuda.synchronize()
    failed = []

    def work(stream, seed):
        try:
            got = []
            with torch.cuda.stream(stream):
                for i in np.random.default_rng(seed).integers(0, len(clouds), size=12):
                    got.append((i, *B.spc_pack_coords(dev[i], descs[i])))
            stream.synchronize()
            for i, keys, perm in got:
                _check(clouds[i], keys, perm)
        except Exception as e:  # (an assertion in a thread would go unnoticed)
            failed.append(repr(e))

    threads = [threading.Thread(target=work, args=(s, j)) for j, s in enumerate((shared, shared, torch.cuda.Stream(), torch.cuda.Stream()))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_replays_between_eager_sorts():
    a, b = _cloud(50_001, 1), _cloud(130_003, 2)
    da, db = fit_desc(a, [(3, 1, 2)]), fit_desc(b, [(3, 1, 2)])
    ta, tb = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    ws = torch.empty(B.spc_pack_workspace_bytes(len(a), da), dtype=torch.uint8, device="cuda")
    keys, perm = torch.empty(len(a), dtype=torch.int32, device="cuda"), torch.empty(len(a), dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):  # (warm)
        B.spc_pack_coords(ta, da, True, 0, None, ws, keys, perm)
    side.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        B.spc_pack_coords(ta, da, True, 0, None, ws, keys, perm)
    for _ in range(3):
        keys.zero_()
        perm.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            kb, pb = B.spc_pack_coords(tb, db)
        g.replay()  # on the current stream, while the other sort may still run
        torch.cuda.synchronize()
        _check(b, kb, pb)
        _check(a, keys, perm)


# (recorded sorts sum their workgroups' counts in the scatter pass up to 32 of them, 1024 keys each; they have 8192 bins above 200 k keys, a
# wave to a rank part from 400 k on, 16384 bins and a column scan above 524 288, and are split and merged from 600 k on)
@pytest.mark.parametrize("n", [4096, 4097, 9001, 32_767, 32_768, 32_769, 200_000, 200_001, 399_999, 400_001, 524_288, 524_289, 599_999, 600_000])
@pytest.mark.parametrize("key_bits", [0, 64])
def test_recorded_sizes(n, key_bits):
    c = _cloud(n, n + 1)
    desc = fit_desc(c, [(3, 1, 2)], key_bits)
    d = torch.from_numpy(c).cuda()
    ws = torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device="cuda")
    keys = torch.empty(n, dtype=torch.int64 if desc.key_bits == 64 else torch.int32, device="cuda")
    perm, side = torch.empty(n, dtype=torch.int32, device="cuda"), torch.cuda.Stream()

    def step():
        B.spc_pack_coords(d, desc, True, 0, None, ws, keys, perm)
        return B.spc_build_kmap(keys, desc, 3, 1, 2, 0, B.LAYOUT_OS)

    with torch.cuda.stream(side):
        step().destroy()  # (warm)
    side.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        m = step()
    for _ in range(3):
        keys.zero_()
        perm.zero_()
        ws.fill_(255)  # (nothing of an earlier replay is relied on)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        _check(c, keys, perm)
        assert m.n_out == len(np.unique(c[:, 1:] // 2, axis=0))
        B.spc_pack_coords(d, desc)
    torch.cuda.synchronize()
    del g
    m.destroy()


def test_first_sort_of_a_size_while_another_thread_records():
    """The sort asks for no memory, which would be refused and end the recording."""
    warm, c = _cloud(9001, 3), _cloud(400_009, 4)
    B.spc_pack_coords(torch.from_numpy(warm).cuda(), fit_desc(warm, [(3, 1, 1)]))  # (the library is loaded)
    B.spc_release_cache()
    desc, d = fit_desc(c, [(3, 1, 1)]), torch.from_numpy(c).cuda()
    ws = torch.empty(B.spc_pack_workspace_bytes(len(c), desc), dtype=torch.uint8, device="cuda")
    keys, perm = torch.empty(len(c), dtype=torch.int32, device="cuda"), torch.empty(len(c), dtype=torch.int32, device="cuda")
    x, side, own = torch.zeros(1000, device="cuda"), torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    failed = []

    def sort():
        try:
            B.spc_pack_coords(d, desc, True, 0, own, ws, keys, perm)
        except Exception as e:
            failed.append(repr(e))

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side, capture_error_mode="global"):
        x.add_(1.0)
        t = threading.Thread(target=sort)
        t.start()
        t.join()
    assert not failed, failed
    torch.cuda.synchronize()
    _check(c, keys, perm)
    for i in range(1, 4):
        g.replay()
        torch.cuda.synchronize()
        assert bool((x == i).all())
