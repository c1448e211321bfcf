"""Configuration 4: the 25-layer UNet-style stack on the LiDAR-like cloud, with all kernel
maps built up front by the network-wide builder."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_20834_amd import binding as B
from paper_2511_20834_amd import synth
from paper_2511_20834_amd.network import SpcNetwork

from gpu_common import assert_close, oracle_keys, rel_err

pytestmark = pytest.mark.gpu


def _setup(cloud_name):
    coords = synth.cloud(cloud_name)
    layers = synth.unet_layers()
    W = synth.unet_weights(layers)
    desc = B.spc_pack_desc_fit(coords[:, 1:].min(0), coords[:, 1:].max(0), 1, 16, 16)
    assert desc.key_bits == 32
    keys, perm = B.spc_pack_coords(torch.from_numpy(coords).cuda(), desc, True, B.PACK_VALIDATE)
    cs, operm = oracle.sort_coords(coords)
    assert np.array_equal(perm.cpu().numpy(), operm)
    F0 = synth.features(len(coords), 4, np.float16, seed=synth.SEED_BASE + 300)
    Fs = B.spc_permute_rows(torch.from_numpy(F0).cuda(), perm)
    return coords, cs, operm, layers, W, desc, keys, F0, Fs


@pytest.mark.parametrize("cloud_name,mode", [("tiny", "streams"), ("lidar", "streams"), ("lidar", "sequential"),
                                             ("lidar", "pipelined")])
def test_network_maps_bit_exact_and_shared(cloud_name, mode):
    coords, cs, operm, layers, W, desc, keys, F0, Fs = _setup(cloud_name)
    net = SpcNetwork(layers, [torch.from_numpy(w).cuda() for w in W],
                     dataflow=[B.DATAFLOW_OS if j % 2 == 0 else B.DATAFLOW_WS for j in range(len(layers))])
    streams = [torch.cuda.current_stream()] + [torch.cuda.Stream() for _ in range(3)]
    searches = B.spc_search_count()
    maps = net.build_maps(keys, desc, streams, {"sequential": B.NET_SEQUENTIAL, "pipelined": B.NET_PIPELINED}.get(mode, 0))
    # 13 distinct maps; a transposed 2x2x2 map is derived from its strided twin's pairs instead of being searched
    # (its lists are the twin's, so the twin must have lists if the transposed layer wants them)
    ws_of = {}
    for l, df in zip(layers, net.dataflow):
        key = (l["K"], l["in_stride"], l["layer_stride"], l["transposed"])
        ws_of[key] = ws_of.get(key, False) or df == B.DATAFLOW_WS
    derived = sum(1 for key, ws in ws_of.items() if key[3] == 1 and (not ws or ws_of[key[:3] + (0,)]))
    assert B.spc_search_count() - searches == 13 - derived
    torch.cuda.synchronize()
    handles = {}
    for j, (l, m) in enumerate(zip(layers, maps)):
        key = (l["K"], l["in_stride"], l["layer_stride"], l["transposed"])
        handles.setdefault(key, set()).add(m.handle.value)
    assert len(handles) == 13 and all(len(v) == 1 for v in handles.values())  # one map per distinct layer geometry
    T, omaps = oracle.network_forward(cs, F0[operm], layers[:0], [])
    seen = set()
    for j, (l, m) in enumerate(zip(layers, maps)):
        key = (l["K"], l["in_stride"], l["layer_stride"], l["transposed"])
        if key in seen:
            continue
        seen.add(key)
        fine = cs if l["in_stride"] == 1 else oracle.downsample(cs, l["in_stride"])
        if l["layer_stride"] == 1:
            oc, M = fine, oracle.kernel_map(fine, fine, l["K"], l["in_stride"])
        elif not l["transposed"]:
            oc = oracle.downsample(cs, l["in_stride"] * 2)
            M = oracle.kernel_map(fine, oc, l["K"], l["in_stride"])
        else:
            oc = fine
            M = oracle.kernel_map_transposed(oracle.downsample(cs, l["in_stride"] * 2), fine, l["K"], l["in_stride"])
        assert m.n_out == len(oc), l["name"]
        assert np.array_equal(m.out_keys(), oracle_keys(oc, desc)), l["name"]
        ref = oracle.triples(M)
        # the shared map carries the union of the layouts its layers asked for
        for which in (B.LAYOUT_OS, B.LAYOUT_WS):
            try:
                got = m.export_triples(which)
            except B.SpcError:
                continue
            assert np.array_equal(got, ref), (l["name"], which)
    net.destroy_maps()


@pytest.mark.parametrize("cloud_name,dataflow", [("tiny", "os"), ("lidar", "os"), ("lidar", "mixed"), ("lidar", "hybrid"),
                                                 ("lidar", "os_pipelined")])
def test_network_forward_matches_oracle(cloud_name, dataflow):
    coords, cs, operm, layers, W, desc, keys, F0, Fs = _setup(cloud_name)
    net_flags = B.NET_PIPELINED if dataflow.endswith("_pipelined") else 0  # maps on one side stream, layers wait for their own
    df = [B.DATAFLOW_WS if l["K"] == 2 or l["in_stride"] >= 8 else B.DATAFLOW_OS for l in layers] if dataflow == "mixed" \
        else B.DATAFLOW_OS
    # hybrid: a different threshold on every 3x3x3 layer (1, 2, 3 in turn), single dataflows elsewhere
    ht = [(1 + j % 3 if l["K"] == 3 else None) for j, l in enumerate(layers)] if dataflow == "hybrid" else None
    net = SpcNetwork(layers, [torch.from_numpy(w).cuda() for w in W], dataflow=df, hybrid_t=ht)
    streams = [torch.cuda.current_stream()] + [torch.cuda.Stream() for _ in range(3)]
    net.build_maps(keys, desc, streams, net_flags)
    y, T = net.forward(Fs, keep=True)
    torch.cuda.synchronize()
    # (a) layer by layer: the oracle is fed the GPU's own (fp16) inputs, which isolates each layer's error
    gpu_in = []
    for l in layers:
        x = T[l["src"]].cpu().double().numpy()
        if l["skip"] is not None:
            x = np.concatenate([x, T[l["skip"]].cpu().double().numpy()], axis=1)
        gpu_in.append(x)
    Tl, _ = oracle.network_forward(cs, F0[operm], layers, W, inputs_override=gpu_in)
    for j, l in enumerate(layers):
        assert_close(T[l["save"]].cpu().double().numpy(), Tl[l["save"]], 1e-2, l["name"])
    # (b) end to end against the oracle's own chain
    To, _ = oracle.network_forward(cs, F0[operm], layers, W)
    assert_close(y.cpu().double().numpy(), To[layers[-1]["save"]], 1e-2, "end to end")
    net.destroy_maps()


@pytest.mark.parametrize("net_flags", [0, B.NET_PIPELINED])
def test_network_step_graph_replays_match_eager(net_flags):
    """The whole step captured into a HIP graph: every replay is compared with the eager result of the
    same input, with eager work and synchronisation between the replays, for the cloud the graph was
    recorded on and for two other clouds of the same size (other level sizes) written into its input
    buffers."""
    n0 = 20000
    clouds = [synth.random_cloud(n0, (90, 90, 24), seed=synth.SEED_BASE + 500 + i) for i in range(3)]
    lo = np.min([c[:, 1:].min(0) for c in clouds], axis=0)
    hi = np.max([c[:, 1:].max(0) for c in clouds], axis=0)
    desc = B.spc_pack_desc_fit(lo, hi, 1, 16, 16)
    layers = synth.unet_layers()
    W = [torch.from_numpy(w).cuda() for w in synth.unet_weights(layers)]
    feats = [synth.features(n0, 4, np.float16, seed=synth.SEED_BASE + 600 + i) for i in range(3)]
    side = [torch.cuda.Stream() for _ in range(3)]

    def eager(i):
        net = SpcNetwork(layers, W)
        keys, perm = B.spc_pack_coords(torch.from_numpy(clouds[i]).cuda(), desc, True)
        Fs = B.spc_permute_rows(torch.from_numpy(feats[i]).cuda(), perm)
        net.build_maps(keys, desc, [torch.cuda.current_stream()] + side)
        y = net.forward(Fs).clone()
        torch.cuda.synchronize()
        net.destroy_maps()
        return y

    refs = [eager(i) for i in range(3)]
    coords_buf = torch.from_numpy(clouds[0]).cuda()
    feats_buf = torch.from_numpy(feats[0]).cuda()
    net = SpcNetwork(layers, W)
    cap = net.capture_step(coords_buf, feats_buf, desc, side, net_flags)
    for rep, i in enumerate([0, 0, 1, 2, 0]):
        coords_buf.copy_(torch.from_numpy(clouds[i]).cuda())
        feats_buf.copy_(torch.from_numpy(feats[i]).cuda())
        cap.output.fill_(float("nan"))
        torch.cuda.synchronize()
        cap.replay()
        torch.cuda.synchronize()
        n_out = cap.n_out()
        assert n_out == refs[i].shape[0], (rep, i)
        got = cap.output[:n_out]
        # cloud 0 runs the very kernels of its eager run (sizes known exactly): bit-exact there;
        # the other clouds' kernels were chosen for cloud 0's level sizes
        if i == 0:
            assert torch.equal(got, refs[i]), rep
        else:
            assert rel_err(got.cpu().double().numpy(), refs[i].cpu().double().numpy()) <= 1e-2, (rep, i)
        # eager work between the replays
        _ = eager((i + 1) % 3)
    cap.destroy()


def test_capture_of_a_small_cloud_replays():
    """Below 4096 voxels the sort (and every downsampled level's) is a single-workgroup kernel: pack + sort and a
    strided map of a 1500-voxel cloud are recorded into a graph and replayed, with eager work in between, and every
    replay equals the eager result."""
    clouds = [synth.random_cloud(1500, (40, 40, 16), seed=synth.SEED_BASE + 700 + i) for i in range(2)]
    lo = np.min([c[:, 1:].min(0) for c in clouds], axis=0)
    hi = np.max([c[:, 1:].max(0) for c in clouds], axis=0)
    desc = B.spc_pack_desc_fit(lo, hi, 1, 2, 1)
    n = 1500
    coords = torch.from_numpy(clouds[0]).cuda()
    ws = torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device="cuda")
    keys = torch.empty(n, dtype=torch.int32 if desc.key_bits == 32 else torch.int64, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")

    def eager(c):
        k, p = B.spc_pack_coords(torch.from_numpy(c).cuda(), desc, True)
        km = B.spc_build_kmap(k, desc, 2, 1, 2, 0, B.LAYOUT_OS)
        t, ok = km.export_triples(B.LAYOUT_OS), km.out_keys()
        km.destroy()
        return k.clone(), p.clone(), t, ok

    refs = [eager(c) for c in clouds]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):  # warm the block cache on the capturing stream
        B.spc_pack_coords(coords, desc, True, 0, None, ws, keys, perm)
        B.spc_build_kmap(keys, desc, 2, 1, 2, 0, B.LAYOUT_OS).destroy()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
        B.spc_pack_coords(coords, desc, True, 0, None, ws, keys, perm)
        km = B.spc_build_kmap(keys, desc, 2, 1, 2, 0, B.LAYOUT_OS)
    for rep, i in enumerate([0, 1, 1, 0]):
        coords.copy_(torch.from_numpy(clouds[i]).cuda())
        keys.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(keys, refs[i][0]) and torch.equal(perm, refs[i][1]), rep
        assert np.array_equal(km.export_triples(B.LAYOUT_OS), refs[i][2]) and np.array_equal(km.out_keys(), refs[i][3]), rep
        eager(clouds[1 - i])  # eager work between the replays
    km.destroy()


def test_capture_of_a_large_cloud_replays():
    """The library's own sort runs up to 8 Mi keys (recorded from 600 k on by split and merge, as when it is called), so
    steps of that size can be recorded: pack + sort and a strided map (whose level is downsampled from 2.2 M voxels) go
    into a graph and are replayed; every replay equals the eager result."""
    n = 2_200_000
    clouds = [synth.scaled_random_cloud(n), None]
    rng = np.random.default_rng(synth.SEED_BASE + 710)
    clouds[1] = clouds[0][rng.permutation(n)].copy()
    clouds[1][:, 3] = np.where(clouds[1][:, 1] % 3 == 0, clouds[1][:, 3] ^ 1, clouds[1][:, 3])  # a different cloud of the same size
    clouds[1] = np.unique(clouds[1], axis=0)
    if len(clouds[1]) < n:  # top up with voxels outside the first cloud's z range
        extra = clouds[0][: n - len(clouds[1])].copy()
        extra[:, 3] += 400
        clouds[1] = np.concatenate([clouds[1], extra])
    lo = np.min([c[:, 1:].min(0) for c in clouds], axis=0)
    hi = np.max([c[:, 1:].max(0) for c in clouds], axis=0)
    desc = B.spc_pack_desc_fit(lo, hi, 1, 2, 1)
    coords = torch.from_numpy(clouds[0]).cuda()
    ws = torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device="cuda")
    keys = torch.empty(n, dtype=torch.int32 if desc.key_bits == 32 else torch.int64, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")

    def eager(c):
        k, p = B.spc_pack_coords(torch.from_numpy(c).cuda(), desc, True)
        km = B.spc_build_kmap(k, desc, 2, 1, 2, 0, B.LAYOUT_OS)
        t, ok = km.export_triples(B.LAYOUT_OS), km.out_keys()
        km.destroy()
        return k.clone(), p.clone(), t, ok

    refs = [eager(c) for c in clouds]
    cs, operm = oracle.sort_coords(clouds[0])
    assert np.array_equal(refs[0][1].cpu().numpy(), operm)  # the eager reference itself against the oracle
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):  # warm the block cache on the capturing stream
        B.spc_pack_coords(coords, desc, True, 0, None, ws, keys, perm)
        B.spc_build_kmap(keys, desc, 2, 1, 2, 0, B.LAYOUT_OS).destroy()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
        B.spc_pack_coords(coords, desc, True, 0, None, ws, keys, perm)
        km = B.spc_build_kmap(keys, desc, 2, 1, 2, 0, B.LAYOUT_OS)
    for rep, i in enumerate([0, 1, 0]):
        coords.copy_(torch.from_numpy(clouds[i]).cuda())
        keys.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(keys, refs[i][0]) and torch.equal(perm, refs[i][1]), rep
        assert np.array_equal(km.out_keys(), refs[i][3]), rep
        assert np.array_equal(km.export_triples(B.LAYOUT_OS), refs[i][2]), rep
    km.destroy()
    B.spc_release_cache()


def test_release_waits_for_replays_on_the_recorded_stream():
    """Feature calls on two maps are recorded into two graphs on one stream.  A replay enqueues nothing through the library,
    yet the release of the second map must order the build stream behind its replay, although the release of the first one
    has ordered the two streams before."""
    coords = synth.cloud("lidar")
    desc = B.spc_pack_desc_fit(coords[:, 1:].min(0), coords[:, 1:].max(0), 1, 1, 1)
    build, feature = torch.cuda.Stream(), torch.cuda.Stream()
    keys, _ = B.spc_pack_coords(torch.from_numpy(coords).cuda(), desc, False)
    F = torch.from_numpy(synth.features(len(coords), 64, np.float16, seed=5)).cuda()
    W = B.spc_conv_prepare_weights(torch.from_numpy(synth.weights(27, 64, 64, np.float16, seed=6)).cuda())
    torch.cuda.synchronize()
    maps = [B.spc_build_kmap(keys, desc, 3, layout=B.LAYOUT_OS, stream=build) for _ in range(2)]
    torch.cuda.synchronize()
    out, graphs = torch.empty_like(F), []
    for m, calls in zip(maps, (1, 400)):  # the second replay takes some 10 ms
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=feature, capture_error_mode="relaxed"):
            for _ in range(calls):
                B.spc_conv_forward(m, F, W, B.DATAFLOW_OS, B.CONV_PACKED_WEIGHTS, out=out)
    torch.cuda.synchronize()
    replayed, built = torch.cuda.Event(), torch.cuda.Event()
    with torch.cuda.stream(feature):
        graphs[0].replay()
        maps[0].destroy()
        graphs[1].replay()
        replayed.record()
    maps[1].destroy()
    built.record(build)  # (nothing takes the arrays again: only the order is looked at)
    built.synchronize()
    assert replayed.query()
    torch.cuda.synchronize()


def test_network_build_searches_nine_maps():
    """Configuration 4 in its default (all output-stationary) setting: 25 layers, 13 distinct maps, 9 searches."""
    coords, cs, operm, layers, W, desc, keys, F0, Fs = _setup("lidar")
    for flags in (0, B.NET_PIPELINED, B.NET_SEQUENTIAL):
        net = SpcNetwork(layers, [torch.from_numpy(w).cuda() for w in W])
        before = B.spc_search_count()
        net.build_maps(keys, desc, [torch.cuda.current_stream()] + [torch.cuda.Stream() for _ in range(2)], flags)
        assert B.spc_search_count() - before == 9
        torch.cuda.synchronize()
        net.destroy_maps()


def test_tuner_then_forward_matches_oracle():
    """One-time tuning of the hybrid dual dataflow (Section 5.4): every layer's threshold is chosen by
    timing on a sample cloud; whatever it picks, the stack must still give Eq. (2)."""
    coords, cs, operm, layers, W, desc, keys, F0, Fs = _setup("tiny")
    net = SpcNetwork(layers, [torch.from_numpy(w).cuda() for w in W])
    rows = net.tune(keys, desc, Fs, reps=2)
    assert len(rows) == len(layers)
    for (name, best, times), l in zip(rows, layers):
        l1_max = 3 if l["K"] == 2 else 3 * (l["K"] - 1) // 2
        assert name == l["name"] and 0 <= best <= l1_max + 1
        assert sorted(times) == list(range(l1_max + 2)) and all(t > 0 for t in times.values())
        assert times[best] == min(times.values())
    # force a mixed outcome as well, so that every kind of per-layer setting is exercised after tuning
    for trial in ("tuned", "forced"):
        if trial == "forced":
            net.dataflow = [B.DATAFLOW_WS if j % 3 == 0 else B.DATAFLOW_OS for j in range(len(layers))]
            net.hybrid_t = [(1 + j % 2) if j % 3 == 1 else None for j in range(len(layers))]
            net._packed = None
        net.build_maps(keys, desc)
        y = net.forward(Fs)
        torch.cuda.synchronize()
        To, _ = oracle.network_forward(cs, F0[operm], layers, W)
        assert_close(y.cpu().double().numpy(), To[layers[-1]["save"]], 1e-2, trial)
        net.destroy_maps()
