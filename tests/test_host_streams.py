"""The library's host code on a stand-in for the HIP runtime (no GPU): which blocks of memory it hands to which stream, and
what it makes wait for what.  A stream handle alone does not name a stream: the default stream's is the same on every device
and hipStreamPerThread in every thread."""
import ctypes
import os
import subprocess
import threading
import time

import pytest

from paper_2511_20834_amd import binding as B
from paper_2511_20834_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
DEFAULT, PER_THREAD, OTHER = (ctypes.c_void_p(s) for s in (None, 2, 0x5000))
SOURCES = ["runtime.hip", "pack_sort.hip", "bucket_sort.hip", "kmap.hip", "conv.hip"]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = tmp_path_factory.mktemp("host")
    cmd = [build.HIPCC, "--offload-host-only", "-O0", "-std=c++17", "-fPIC", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
           "-Wno-unused-result", "-c"]
    objs, procs = [], []
    for src in [os.path.join(build.CSRC, s) for s in SOURCES] + [os.path.join(HERE, "host", "hip_standin.cpp")]:
        objs.append(str(out / (os.path.basename(src) + ".o")))
        procs.append(subprocess.Popen([*cmd, "-x", "hip", src, "-o", objs[-1]]))
    assert [p.wait() for p in procs] == [0] * len(procs)
    lib = str(out / "libspc_host.so")
    # (the device code's images, which nobody reads here)
    undefined = subprocess.run(["nm", "-u", *objs], check=True, capture_output=True, text=True).stdout.split()
    images = ["-Wl,--defsym=%s=0" % s for s in undefined if s.startswith("__hip_fatbin")]
    subprocess.check_call(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", *images, *objs, "-o", lib])
    L = ctypes.CDLL(lib)
    L.standin_log.restype = ctypes.c_char_p
    L.spc_kmap_os_map.restype = ctypes.c_void_p
    return Host(L)


class Host:
    def __init__(self, L):
        self.L = L
        self.desc = B.PackDesc()
        assert L.spc_pack_desc_fit((ctypes.c_int32 * 3)(0, 0, 0), (ctypes.c_int32 * 3)(500, 500, 100), 1, 4, 4, 32, ctypes.byref(self.desc)) == 0

    def log(self):
        return [l.split() for l in self.L.standin_log().decode().splitlines()]

    def on(self, device):
        self.L.standin_set_device(device)

    def device_of(self, p):
        return self.L.standin_device_of(ctypes.c_void_p(p))

    def pack(self, n, stream):
        """Sorts n coordinates; returns what was logged."""
        coords, keys = ctypes.create_string_buffer(16 * n), ctypes.create_string_buffer(4 * n)
        need = ctypes.c_size_t(0)
        args = (ctypes.byref(need), 0, stream)
        assert self.L.spc_pack_coords(coords, ctypes.c_int64(n), ctypes.byref(self.desc), keys, None, None, *args) == 0
        ws = ctypes.create_string_buffer(need.value)
        self.log()
        assert self.L.spc_pack_coords(coords, ctypes.c_int64(n), ctypes.byref(self.desc), keys, None, ws, *args) == 0
        return self.log()

    def build(self, n, stream, layer_stride=1, layout=B.LAYOUT_OS, K=3):
        m = ctypes.c_void_p()
        l = B.LayerDesc(K, 1, layer_stride, 0, layout)
        assert self.L.spc_build_kmap(ctypes.c_void_p(64), ctypes.c_int64(n), ctypes.byref(self.desc), ctypes.byref(l), ctypes.byref(m), stream) == 0
        return m

    def os_map(self, m):
        return self.L.spc_kmap_os_map(m)

    def forward(self, m, stream):
        p = ctypes.c_void_p(64)
        assert self.L.spc_conv_forward(m, p, ctypes.c_int64(32), p, p, ctypes.c_int64(32), 32, 32, 0, 0, 0, stream) == 0

    def destroy(self, m):
        self.L.spc_kmap_destroy(m)


def in_thread(f):
    """f's result, from a thread that has ended."""
    got = []
    t = threading.Thread(target=lambda: got.append(f()))
    t.start()
    t.join()
    while os.path.exists("/proc/self/task/%d" % t.native_id):  # (join returns a little before the thread's own data are torn down)
        time.sleep(0.001)
    return got[0]


def totals_of(log):
    return [int(l[4]) for l in log if l[0] == "launch" and "bs_count_kernel" in l[3]][0]


def cleared_first(log):
    return any(l[0] == "launch" and "clear" in l[3] for l in log)


@pytest.mark.parametrize("stream", [DEFAULT, PER_THREAD], ids=["default", "per thread"])
def test_maps_stay_on_their_device(host, stream):
    host.on(0)
    m = host.build(5000, stream)
    assert host.device_of(host.os_map(m)) == 0
    host.destroy(m)
    host.on(1)
    m = host.build(5000, stream)
    assert host.device_of(host.os_map(m)) == 1
    host.on(0)  # released while another device is the current one
    host.destroy(m)
    m = host.build(5000, stream)
    assert host.device_of(host.os_map(m)) == 0
    host.destroy(m)


def test_sort_totals_stay_on_their_device(host):
    for device in (0, 1, 0, 1):
        host.on(device)
        log = host.pack(20_000, DEFAULT)
        where = host.device_of(totals_of(log))
        assert where == device or (where < 0 and cleared_first(log))  # (the caller's workspace is host memory here)
    host.on(0)


def test_per_thread_streams_share_nothing(host):
    """Two threads' streams of the one handle have no order between them."""
    mine = host.build(7000, PER_THREAD)
    block = host.os_map(mine)
    host.destroy(mine)  # free, for this thread's stream
    go, done = threading.Event(), threading.Event()
    got = []

    def other():
        host.on(0)
        m = host.build(7000, PER_THREAD)
        got.append(host.os_map(m))
        host.destroy(m)
        done.set()
        go.wait()

    t = threading.Thread(target=other)
    t.start()
    done.wait()
    assert got[0] != block
    again = host.build(7000, PER_THREAD)
    assert host.os_map(again) == block
    host.destroy(again)
    go.set()
    t.join()


def test_sorts_on_per_thread_streams_share_no_totals(host):
    """Neither one after the other nor through a block that was left behind: there is no order to rely on."""
    for _ in range(2):
        for n, cleared in ((9000, False), (50_000, True)):  # (small sorts have no totals then)
            for log in (host.pack(n, PER_THREAD), in_thread(lambda: host.pack(n, PER_THREAD))):
                assert cleared_first(log) == cleared and host.device_of(totals_of(log)) < 0


@pytest.mark.parametrize("n,launches", [(4096, 3), (32_768, 3), (32_769, 4), (524_288, 4), (524_289, 4)])
def test_launches_of_recorded_sorts(host, n, launches):
    """A recorded sort keeps no totals from one replay to the next; small ones get by without clearing any."""
    host.on(0)
    host.L.standin_capture(OTHER)
    log = host.pack(n, OTHER)
    host.L.standin_capture(ctypes.c_void_p(2**64 - 1))
    assert [l[0] for l in log] == ["launch"] * launches and cleared_first(log) == (launches == 4 and n <= 524_288)


def test_blocks_of_ended_threads_come_back_after_a_drain(host):
    def left_behind():
        host.on(0)
        m = host.build(300_000, PER_THREAD)
        p = host.os_map(m)
        host.destroy(m)
        return p

    p = in_thread(left_behind)
    host.log()
    m = host.build(300_000, OTHER)
    assert host.os_map(m) == p and ["drain", "0"] in host.log()
    host.destroy(m)


def test_map_of_another_threads_stream_is_released_behind_a_drain(host):
    """Its stream, or a consumer's, cannot be waited for from here."""
    m = host.build(6000, OTHER)
    in_thread(lambda: host.forward(m, PER_THREAD))
    host.log()
    host.destroy(m)
    assert ["drain", "0"] in host.log()
    m = in_thread(lambda: host.build(6000, PER_THREAD))
    host.forward(m, OTHER)
    host.log()
    host.destroy(m)
    assert ["drain", "0"] in host.log()


def test_count_of_another_threads_level_is_waited_for(host):
    m = in_thread(lambda: host.build(6000, PER_THREAD, 2))
    host.log()
    host.L.spc_kmap_n_out.restype = ctypes.c_int64
    assert host.L.spc_kmap_n_out(m) == 0  # (nothing runs here: the count is the zero the memory started with)
    assert ["drain", "0"] in host.log()
    host.destroy(m)


def test_releases_on_two_devices_wait_each(host):
    """What the default stream of one device has been ordered behind says nothing about the other's."""
    for device in (0, 1):
        host.on(device)
        m = host.build(6000, DEFAULT)
        host.forward(m, OTHER)
        host.log()
        host.on(0)
        host.destroy(m)
        waits = [l for l in host.log() if l[0] == "wait"]
        assert len(waits) == 1 and waits[0][1] == str(device) and waits[0][2] == "0", waits


@pytest.mark.parametrize("stream", [DEFAULT, PER_THREAD], ids=["default", "per thread"])
def test_pipelined_maps_are_waited_for_once_per_stream(host, stream):
    """By the first layer on every stream but the build's, the default stream included."""
    layer, m, streams = B.LayerDesc(3, 1, 1, 0, B.LAYOUT_OS), ctypes.c_void_p(), (ctypes.c_void_p * 1)(OTHER)
    assert host.L.spc_build_kmaps_network(ctypes.c_void_p(64), ctypes.c_int64(5000), ctypes.byref(host.desc), ctypes.byref(layer), 1,
                                          ctypes.byref(m), streams, 1, B.NET_PIPELINED) == 0
    for waits in (1, 0):
        host.log()
        host.forward(m, stream)
        log = [l for l in host.log() if l[0] in ("wait", "launch")]
        assert [l[0] for l in log] == ["wait"] * waits + ["launch"] and int(log[0][2]) == (stream.value or 0)
    host.destroy(m)


def test_sorts_ask_for_no_memory(host):
    """The caller has brought a workspace.  Once the image's blocks are all in use on other streams, the totals lie in there."""
    host.on(2)
    streams = [ctypes.c_void_p(0x10000 + 16 * i) for i in range(80)]
    for n in (4096, 20_000, 200_000, 300_000, 524_288, 600_000):  # 1 to 32 KB of totals, and none (column scan)
        logs = [host.pack(n, s) for s in streams]
        assert not any(l[0] in ("malloc", "free", "drain") for log in logs for l in log)
        if n > 524_288:
            break
        for log in logs:
            assert host.device_of(totals_of(log)) == (-1 if cleared_first(log) else 2)
        held = [totals_of(log) for log in logs if not cleared_first(log)]
        assert len(set(held)) == len(held)  # a block of its own for every stream
    assert all(cleared_first(host.pack(300_000, s)) for s in streams[70:])  # (no room left)
    host.L.spc_release_cache()
    assert not any(cleared_first(host.pack(300_000, s)) for s in streams[70:])
    host.L.spc_release_cache()
    host.on(0)


# ---- which feature kernel a layer gets
F16, F32 = 0, 2


def feature_kernel(host, m, ld_in, cin, cout, dtype=F16, dataflow=B.DATAFLOW_OS, flags=0, ld_out=None):
    """The name of the feature kernel that a call enqueues."""
    p = ctypes.c_void_p(64)
    host.log()
    assert host.L.spc_conv_forward(m, p, ctypes.c_int64(ld_in), p, p, ctypes.c_int64(ld_out or cout), cin, cout, dtype, dataflow, flags, OTHER) == 0
    names = [l[3] for l in host.log() if l[0] == "launch"]
    return [k for k in ("resident", "phase", "splitk") if any("conv_%s_kernel" % k in n or "conv_os_%s_kernel" % k in n for n in names)][-1]


@pytest.mark.parametrize("flags", [0, B.CONV_RESIDENT])
@pytest.mark.parametrize("dtype,cin,cout", [(F16, 64, 1_250_000), (F16, 64, 700_000), (F32, 32, 1_250_000)])
def test_weights_beyond_32_bit_offsets_are_left_to_the_splitk_kernel(host, flags, dtype, cin, cout):
    """The kernel with resident weights reads plain ones at 32-bit offsets, of which the upper half is the mark of what is not there."""
    m = host.build(40, OTHER)
    assert feature_kernel(host, m, cin, cin, cout, dtype, flags=flags) == "splitk"
    assert feature_kernel(host, m, cin, cin, 40, dtype, flags=B.CONV_RESIDENT) == "resident"
    host.destroy(m)


def test_output_rows_beyond_32_bit_pitches_are_left_to_the_splitk_kernel(host):
    m = host.build(40, OTHER)
    for ld_out, kernel in ((2**31 - 1, "resident"), (2**31, "splitk"), (2**32 + 32, "splitk")):
        assert feature_kernel(host, m, 32, 32, 32, flags=B.CONV_RESIDENT, ld_out=ld_out) == kernel
    host.destroy(m)


def test_choice_does_not_follow_the_count(host):
    """Rows that lie beyond 32-bit offsets by the level's bound, and not by its count once the host has asked for it: every kernel has an
    order of sums of its own, so the layer keeps its kernel."""
    layers = (B.LayerDesc * 2)(B.LayerDesc(3, 2, 1, 0, B.LAYOUT_OS), B.LayerDesc(3, 2, 2, 0, B.LAYOUT_OS))
    m, streams = (ctypes.c_void_p * 2)(), (ctypes.c_void_p * 1)(OTHER)
    assert host.L.spc_build_kmaps_network(ctypes.c_void_p(64), ctypes.c_int64(300_000), ctypes.byref(host.desc), layers, 2, m, streams, 1, 0) == 0
    a, b = (ctypes.c_void_p(x) for x in m)
    before = feature_kernel(host, b, 4096, 32, 32, flags=B.CONV_RESIDENT)
    assert host.L.spc_kmap_n_out(a) == 0  # (the stride-2 level; nothing runs here)
    assert feature_kernel(host, b, 4096, 32, 32, flags=B.CONV_RESIDENT) == before == "splitk"
    assert feature_kernel(host, b, 32, 32, 32, flags=B.CONV_RESIDENT) == "resident"
    host.destroy(a)
    host.destroy(b)


def test_at_most_one_kernel_may_be_asked_for(host):
    m, p = host.build(40, OTHER), ctypes.c_void_p(64)
    for flags in (B.CONV_OS_PHASE | B.CONV_OS_SPLITK, B.CONV_OS_PHASE | B.CONV_RESIDENT, B.CONV_OS_SPLITK | B.CONV_RESIDENT):
        assert host.L.spc_conv_forward(m, p, ctypes.c_int64(32), p, p, ctypes.c_int64(32), 32, 32, F16, B.DATAFLOW_OS, flags, OTHER) == B.ERR_ARG
    host.destroy(m)


def test_layers_of_the_resident_kernel_are_counted(host):
    host.L.spc_resident_count.restype = ctypes.c_int64
    m = host.build(40, OTHER)
    for cin, kernel, more in ((32, "resident", 1), (128, "splitk", 0)):
        before = host.L.spc_resident_count()
        assert feature_kernel(host, m, cin, cin, 32, flags=B.CONV_RESIDENT) == kernel
        assert host.L.spc_resident_count() - before == more
    host.destroy(m)


# (33 and 64 slabs of columns: more than one round of workgroups; 17: half of the CUs; too few rows for all XCDs)
@pytest.mark.parametrize("n,dtype,cin,cout,taken", [
    (5000, F16, 64, 1056, False), (30_000, F16, 64, 544, False), (30_000, F32, 32, 544, False), (2000, F32, 32, 2048, False), (5000, F32, 32, 1024, False),
    (4000, F16, 32, 2048, False), (5000, F16, 32, 2048, True), (30_000, F16, 64, 800, True), (8200, F32, 32, 1024, True), (12_000, F16, 32, 1600, True)])
def test_layers_that_leave_cus_idle_are_not_the_resident_kernels(host, n, dtype, cin, cout, taken):
    m = host.build(n, OTHER)
    assert (feature_kernel(host, m, cin, cin, cout, dtype) == "resident") == taken
    host.destroy(m)


# (three slabs of 16 channels, fp32 of 8, are taken as four)
@pytest.mark.parametrize("n,dtype,cin,cout,ws,packed,taken", [
    (200_000, F32, 20, 64, False, False, False), (200_000, F32, 24, 32, True, False, False), (200_000, F32, 28, 64, False, False, True), (200_000, F32, 16, 64, True, False, True),
    (200_000, F16, 48, 64, True, True, False), (200_000, F16, 40, 128, True, True, False), (200_000, F16, 48, 64, True, False, True), (200_000, F16, 56, 64, True, True, True),
    (200_000, F16, 32, 64, True, True, True), (100_000, F16, 48, 32, True, True, False), (200_000, F16, 48, 32, True, True, True), (100_000, F16, 48, 32, True, False, True),
    (80_000, F16, 40, 8, False, False, False), (100_000, F16, 40, 8, False, False, True), (80_000, F16, 24, 8, False, False, True)])
def test_layers_of_three_slabs_of_channels_are_taken_where_four_pay(host, n, dtype, cin, cout, ws, packed, taken):
    m = host.build(n, OTHER, layout=B.LAYOUT_WS if ws else B.LAYOUT_OS)
    kernel = feature_kernel(host, m, cin, cin, cout, dtype, B.DATAFLOW_WS if ws else B.DATAFLOW_OS, B.CONV_PACKED_WEIGHTS if packed else 0)
    assert (kernel == "resident") == taken
    host.destroy(m)


# ---- how a map's tiles and lists are made
@pytest.mark.parametrize("K,n,layout,rows,scanned", [
    (1, 28_672, B.LAYOUT_WS, 64, False), (1, 28_673, B.LAYOUT_WS, 64, True), (1, 149_999, B.LAYOUT_OS, 64, False), (1, 150_000, B.LAYOUT_WS, 128, True),
    (1, 399_999, B.LAYOUT_OS, 128, False), (1, 400_000, B.LAYOUT_WS, 256, True), (3, 14_528, B.LAYOUT_WS, 64, False), (3, 14_592, B.LAYOUT_WS, 64, True),
    (3, 184_999, B.LAYOUT_WS, 64, True), (3, 185_000, B.LAYOUT_OS, 128, False), (3, 400_000, B.LAYOUT_WS, 128, True), (3, 400_000, B.LAYOUT_OS, 256, False)])
def test_tiles_of_a_search_and_who_adds_their_counts(host, K, n, layout, rows, scanned):
    """A column of one offset's counts is added by eight threads of every fill workgroup: not where it is long."""
    host.log()
    m = host.build(n, OTHER, layout=layout, K=K)
    names = [l[3] for l in host.log() if l[0] == "launch"]
    tile, window = ctypes.c_int32(0), ctypes.c_int32(0)
    assert host.L.spc_kmap_search_info(m, ctypes.byref(tile), ctypes.byref(window)) == 0
    assert tile.value == rows and any("ws_scan_kernel" in x for x in names) == scanned
    host.destroy(m)
