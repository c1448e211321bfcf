"""The sort's kernels on the CPU (tests/host/emulated): bins that are shared between workgroups, in memory that ends where nothing may be
touched and in a workspace as large as reported, and what becomes of a sort whose totals or workspace another call has changed.  Every case
runs in a process of its own, with a time limit."""
import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
EMULATED = os.path.join(HERE, "host", "emulated")
PAD = 2


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    from paper_2511_20834_amd import build
    out = tmp_path_factory.mktemp("sort")
    text = open(os.path.join(build.CSRC, "bucket_sort.hip")).read()
    for pattern, by in (
            (r"__builtin_amdgcn_", "emu::"),
            (r"extern __shared__ __align__\(16\) unsigned bs_lds\[\];", "unsigned* bs_lds = emu::dynamic_lds;"),
            (r"extern __shared__ int lds_bins\[\];", "int* lds_bins = reinterpret_cast<int*>(emu::dynamic_lds);"),
            (r'asm volatile\("s_load_dwordx16.*?\);', "memcpy(&lo, q, 64), memcpy(&hi, static_cast<const char*>(q) + 64, 64);"),
            (r'asm volatile\("s_waitcnt.*?\);', ""),
            (r'asm volatile\("" : "\+[vs]"\(\w+\)\);', ""),
            (r"SPC_PIN_LOADED\(", "(void)("),
            # a kernel's arguments, where they are loaded anew
            (r"bs_args_anew\(const Args&\)", "bs_args_anew(const Args& a)"),
            (r"P p = \(P\)emu::kernarg_segment_ptr\(\);", "const Args* p = &a;"),
            (r"  using P = const Args __attribute__\(\(address_space\(4\)\)\)\*;\n", "")):
        text, n = re.subn(pattern, by, text)
        assert n > 0, pattern
    (out / "bucket_sort.inc").write_text(text)
    so = str(out / "sort.so")
    subprocess.check_call([os.path.join(os.path.dirname(build.HIPCC), "amdclang++"), "-std=c++17", "-O1", "-w", "-fPIC", "-shared",
                           "-fsanitize=bounds", "-fsanitize-trap=bounds", "-I", EMULATED, "-I", str(out), "-I", os.path.join(build.ROOT, "include"),
                           "-I", build.CSRC, os.path.join(EMULATED, "sort_entry.cpp"), os.path.join(EMULATED, "emulator.cpp"), "-o", so])
    return so


def in_child(lib, *args, timeout=120):
    p = subprocess.run([sys.executable, os.path.abspath(__file__), lib, *map(str, args)], timeout=timeout, capture_output=True, text=True)
    assert p.returncode == 0, (p.returncode, p.stdout, p.stderr)


# bits of x, y, z; a bin is the top 8 to 12 bits of them together
CLOUDS = {
    "wall": (6000, (12, 12, 8)),       # two thirds in one plane of x
    "slab": (7000, (12, 9, 9)),        # all but a voxel in two
    "cluster": (5000, (20, 20, 20)),   # all but one in a corner of the key space: second bins are split again
    "one": (5000, (10, 10, 10)),       # one voxel
    "few": (9000, (10, 10, 10)),       # four, and some others
    "rejected": (9000, (10, 10, 9)),   # half of the rows do not fit
    "band": (5200, (8, 12, 8)),        # bins that fit the LDS alone, but not beside others
    "outlier": (6000, (12, 9, 9)),     # the last workgroup's bins reach from a box to a voxel far away: all keys in a few second bins
    "large": (524_289, (11, 11, 8)),   # the smallest whose bins' starts a kernel of its own finds
}


def cloud(kind, rng):
    n, (bx, by, bz) = CLOUDS[kind]
    top = [(1 << b) - 2 * PAD for b in (bx, by, bz)]

    def box(m, dims, at=(0, 0, 0)):
        lin = rng.choice(int(np.prod(dims)), size=m, replace=False)
        return np.stack([at[0] + lin // (dims[1] * dims[2]), at[1] + lin // dims[2] % dims[1], at[2] + lin % dims[2]], 1)

    def anywhere(m):
        return np.stack([rng.integers(0, t, m) for t in top], 1)

    if kind == "wall":
        c = np.concatenate([box(4000, (1, 400, 60), (1000, 0, 0)), box(n - 4000, (900, 400, 60))])
    elif kind == "slab":
        c = np.concatenate([box(n - 1, (2, 300, 300)), [[top[0] - 1, 0, 0]]])
    elif kind == "cluster":
        c = np.concatenate([box(n - 1, (30, 30, 30)), [[t - 1 for t in top]]])
    elif kind == "outlier":
        c = np.concatenate([box(n - 1, (40, 20, 20)), [[top[0] - 1, 0, 0]]])
    elif kind == "one":
        c = np.tile([[5, 6, 7]], (n, 1))
    elif kind == "few":
        c = np.concatenate([rng.integers(100, 102, (n // 2, 3)) * [1, 1, 0], anywhere(n - n // 2)])
    elif kind == "rejected":
        c = anywhere(n)
        c[: n // 2, 0] = -5
    elif kind == "large":
        c = np.concatenate([box(9000, (1, 200, 200)), box(n - 15_000, (1500, 400, 200), (1, 0, 0)), np.full((6000, 3), -5)])
    else:
        c = np.concatenate([box(s, (1, 200, 200), (x, 0, 0)) for x, s in enumerate([500, 1900, 1, 400, 2048, 350, 1])])
    c = rng.permutation(np.concatenate([np.zeros((len(c), 1), np.int64), c], 1)).astype(np.int32)
    assert len(c) == n
    return np.ascontiguousarray(c), (bx, by, bz)


def run(so, kind, key_bits, keep, record, disturb, seed):
    L = ctypes.CDLL(so)
    L.emu_guarded.restype = ctypes.c_void_p
    L.emu_ws_bytes.restype = ctypes.c_size_t
    c, bits = cloud(kind, np.random.default_rng(seed))
    n, used, ktype = len(c), sum(bits), np.uint32 if key_bits == 32 else np.uint64

    def guarded(dtype, count, align=16):
        p = L.emu_guarded(ctypes.c_size_t(np.dtype(dtype).itemsize * count), ctypes.c_size_t(align))
        return p, np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(np.ctypeslib.as_ctypes_type(dtype))), (count,))

    need = L.emu_ws_bytes(key_bits, ctypes.c_int64(n))
    ws, (dc, coords) = guarded(np.uint8, need, 256)[0], guarded(np.int32, 4 * n)
    (dk, keys), (dp, perm) = guarded(ktype, n), guarded(np.int32, n)
    coords[:] = c.reshape(-1)
    L.emu_mode(keep, record, disturb, seed, ctypes.c_void_p(ws if disturb == 4 else None), ctypes.c_size_t(need if disturb == 4 else 0))
    args = [ctypes.c_void_p(p) for p in (dk, dp, ws)]
    assert L.emu_pack_sort(key_bits, ctypes.c_void_p(dc), ctypes.c_int64(n), (ctypes.c_int * 3)(*bits), PAD, *args) == 0
    if disturb < 0:
        x, y, z = (c[:, i].astype(np.uint64) + PAD for i in (1, 2, 3))
        k = x << np.uint64(bits[1] + bits[2]) | y << np.uint64(bits[2]) | z
        k = np.where(c[:, 1] < 0, np.uint64(2 ** key_bits - 1), k).astype(ktype)
        assert np.array_equal(np.sort(perm), np.arange(n))
        assert np.array_equal(keys, k[perm]) and np.all(keys[1:] >= keys[:-1])
        if key_bits == 32 and not record:
            assert np.array_equal(perm, np.argsort(k, kind="stable"))
    elif disturb == 4:
        return
    else:
        keys[:] = np.sort(np.random.default_rng(seed).integers(0, 2 ** min(used, 63), n).astype(ktype))
    masks = []
    for m in (1, 2, 6):
        fields = [((1 << b) - 1) & ~((1 << m) - 1) for b in bits]
        mask = fields[0] << (bits[1] + bits[2]) | fields[1] << bits[2] | fields[2]
        masks.append(mask | (2 ** key_bits - 1) >> used << used)
    outs, counts = [guarded(ktype, n) for _ in masks], guarded(np.int32, len(masks))
    pitch = (need + 255) // 256 * 256
    wide, _ = guarded(np.uint8, pitch * len(masks), 256)
    assert L.emu_levels(key_bits, ctypes.c_void_p(dk), ctypes.c_int64(n), used, len(masks), (ctypes.c_uint64 * len(masks))(*masks),
                        (ctypes.c_void_p * len(masks))(*[o[0] for o in outs]), ctypes.c_void_p(counts[0]), ctypes.c_void_p(wide),
                        ctypes.c_size_t(pitch)) == 0
    if disturb < 0:
        for mask, (_, out), count in zip(masks, outs, counts[1]):
            want = np.unique(keys & ktype(mask))
            assert count == len(want) and np.array_equal(out[:count], want)


@pytest.mark.parametrize("keep,record", [(1, 0), (0, 0), (0, 1)], ids=["kept totals", "no totals", "recorded"])
@pytest.mark.parametrize("kind,key_bits", [(k, b) for k in CLOUDS for b in (32, 64) if k != "large" and (b == 64 or sum(CLOUDS[k][1]) <= 32)])
def test_shared_bins(lib, kind, key_bits, keep, record):
    in_child(lib, kind, key_bits, keep, record, -1, 3)


@pytest.mark.parametrize("key_bits", [32, 64])
def test_shared_bins_of_a_large_cloud(lib, key_bits):
    in_child(lib, "large", key_bits, 0, 0, -1, 3)


# (totals twice as large, cleared, larger, halved, or words of the workspace changed; "large" has no totals)
@pytest.mark.parametrize("kind,key_bits,disturb", [(k, b, d) for k, b in (("wall", 32), ("few", 64), ("band", 32), ("large", 32), ("large", 64))
                                                   for d in range(5) if k != "large" or d == 4])
def test_totals_that_are_not_the_keys(lib, kind, key_bits, disturb):
    """As a caller that uses one workspace in two calls at once may leave them: the result is meaningless, but every loop ends and nothing
    outside is touched."""
    in_child(lib, kind, key_bits, 1, 0, disturb, 4, timeout=60)


if __name__ == "__main__":
    run(sys.argv[1], sys.argv[2], *map(int, sys.argv[3:]))
