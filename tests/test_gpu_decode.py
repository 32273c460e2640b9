"""GPU parity: zm_decode_experts (through the C ABI) against the reference codec, bit for bit."""
import ctypes
import sys
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from oracle import oracle as zo
from paper_2601_21198_amd import synth, zipmoe as zm

pytestmark = pytest.mark.gpu

GUARD = 64          # int16 guard words on each side of every output buffer
GUARD_WORD = 0x5A5A


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def gpu_decode_tensors(blobs, repeat_ids=None, stores=None):
    """Decodes each blob as a one-tensor expert; returns the decoded uint16 arrays (with guard check).
    stores: None = zm_decode_experts, else the policy handed to zm_decode_experts_stores."""
    import torch
    layer = zm.ExpertLayer([[b] for b in blobs])
    ids = list(range(len(blobs))) if repeat_ids is None else repeat_ids
    outs = []
    ptrs = (ctypes.c_void_p * len(ids))()
    for j, e in enumerate(ids):
        n = int(layer.infos[e].n_values)
        buf = torch.full((n + 2 * GUARD,), GUARD_WORD, dtype=torch.int16, device="cuda")
        outs.append(buf)
        ptrs[j] = buf.data_ptr() + 2 * GUARD
    idarr = (ctypes.c_int32 * len(ids))(*ids)
    outp = ctypes.cast(ptrs, ctypes.POINTER(ctypes.c_void_p))
    stream = torch.cuda.current_stream().cuda_stream
    if stores is None:
        zm.decode_experts(layer._ptr_blobs, layer._ptr_tables, layer._ptr_infos, layer.n_experts, 1, idarr, len(ids), outp, stream)
    else:
        rc = zm.lib().zm_decode_experts_stores(layer._ptr_blobs, layer._ptr_tables, layer._ptr_infos, layer.n_experts, 1,
                                               idarr, len(ids), outp, stores, ctypes.c_void_p(stream))
        if rc != zm.OK:
            raise zm.ZipMoEError(rc, "zm_decode_experts_stores")
    torch.cuda.synchronize()
    res = []
    for buf in outs:
        a = buf.cpu().numpy().view(np.uint16)
        assert np.all(a[:GUARD] == GUARD_WORD) and np.all(a[-GUARD:] == GUARD_WORD), "guard words overwritten"
        res.append(a[GUARD:-GUARD].copy())
    return res


KINDS = ["all_equal", "two_exponents", "uniform_u16", "rare_last", "gauss", "wide", "many_long"]
SIZES = [0, 1, 7, 8, 9, 511, 512, 513, 4095, 4096, 4097, 9000, 3 * 16384 + 1234]


@pytest.mark.parametrize("C,W,max_len", [(4096, 4096, 8), (16384, 4096, 8), (4096, 1024, 12), (2048, 512, 8),
                                         (16384, 16384, 8), (8192, 2048, 12), (32768, 8192, 12),
                                         # streams so long that fewer of them share a workgroup
                                         (16384, 16384, 12), (32768, 32768, 12), (32768, 32768, 8)])
def test_edge_cases_bit_exact(C, W, max_len):
    tensors, blobs = [], []
    for kind in KINDS:
        for n in SIZES:
            w = synth.special_tensor(kind, n, seed=n + 3)
            blob, _ = zm.compress(w, C, W, max_len)
            tensors.append(w)
            blobs.append(blob)
    say(f"edge cases C={C} W={W} L<={max_len}: {len(blobs)} tensors in one call")
    refs = [zo.decode(blob) for blob in blobs]
    for stores in (None, zm.STORES_CACHED, zm.STORES_STREAMING):      # the library's own choice, and both kernels by name
        got = gpu_decode_tensors(blobs, stores=stores)
        for w, ref, g in zip(tensors, refs, got):
            assert np.array_equal(g, ref)                    # against the reference decoder
            assert np.array_equal(g, w)                      # and against the original: lossless


def test_all_bit_patterns_and_duplicates():
    w = np.random.default_rng(1).permutation(np.arange(65536, dtype=np.uint32)).astype(np.uint16)
    blob8, _ = zm.compress(w, 4096, 4096, 8)
    blob12, _ = zm.compress(w, 4096, 2048, 12)
    got = gpu_decode_tensors([blob8, blob12], repeat_ids=[1, 0, 1, 1])      # duplicate ids are decoded again
    for g in got:
        assert np.array_equal(g, w)
    assert np.array_equal(got[0], zo.decode(blob12))


def test_mixed_geometries_in_one_call():
    # tensors with different chunk lengths, stream lengths and code-length limits share a call: both round
    # lengths are launched, and the staging area is sized for the longest stream of each group.  Every other
    # blob comes from the reference encoder.
    rng = np.random.default_rng(77)
    geometries = [(4096, 512, 8), (4096, 4096, 8), (16384, 4096, 8), (16384, 2048, 11), (8192, 8192, 9),
                  (2048, 1024, 12), (16384, 16384, 8), (1024, 512, 10)]
    tensors, blobs = [], []
    for i in range(48):
        C, W, max_len = geometries[int(rng.integers(len(geometries)))]
        kind = KINDS[int(rng.integers(len(KINDS)))]
        n = int(rng.integers(1, 70000))
        w = synth.special_tensor(kind, n, seed=1000 + i)
        if i % 2:
            blob = zo.encode(w, C, W, zo.code_lengths(zo.histogram(zo.split(w)[0]), max_len))
        else:
            blob, _ = zm.compress(w, C, W, max_len)
        tensors.append(w)
        blobs.append(blob)
    say(f"mixed geometries: {len(blobs)} tensors in one call")
    got = gpu_decode_tensors(blobs)
    for w, blob, g in zip(tensors, blobs, got):
        assert np.array_equal(g, w) and np.array_equal(g, zo.decode(blob))


def chunk_modes(blob):
    """mode of every chunk (0 coded, 1 raw), read from the blob's chunk table"""
    h = zo.header(blob)
    table = np.asarray(blob[h["table_offset"]: h["table_offset"] + h["table_stride"] * h["n_chunks"]], np.uint8)
    return table.reshape(h["n_chunks"], h["table_stride"])[:, 0] & 15


def patchwork_tensor(rng, n):
    """segments of very different exponent statistics in one tensor: with one codebook for the whole tensor some
    chunks compress and others are stored raw, and streams differ widely in length"""
    parts, left = [], n
    while left > 0:
        m = int(min(left, rng.integers(1, 40000)))
        k = int(rng.integers(5))
        if k == 0:
            seg = rng.integers(0, 65536, m, dtype=np.uint16)                                     # incompressible
        elif k == 1:
            seg = np.full(m, 0x3F80, np.uint16) | rng.integers(0, 128, m, dtype=np.uint16)      # one exponent
        elif k == 2:
            seg = synth.bf16_round(rng.standard_normal(m, dtype=np.float32) * np.float32(10.0 ** rng.uniform(-4, 2)))
        elif k == 3:
            e = rng.geometric(0.5, m).clip(1, 40).astype(np.uint16) + 90                         # geometric exponents
            seg = (e << 7) | rng.integers(0, 128, m, dtype=np.uint16) | (rng.integers(0, 2, m, dtype=np.uint16) << 15)
        else:
            e = rng.choice(np.array([1, 2, 127, 128, 254, 255], np.uint16), m, p=[0.5, 0.25, 0.12, 0.07, 0.04, 0.02])
            seg = (e << 7) | rng.integers(0, 128, m, dtype=np.uint16)
        parts.append(seg.astype(np.uint16))
        left -= m
    return np.concatenate(parts) if parts else np.zeros(0, np.uint16)


@pytest.mark.parametrize("seed", [11, 12, 13])
def test_random_patchwork_tensors(seed):
    rng = np.random.default_rng(seed)
    geometries = [(4096, 512, 8), (4096, 4096, 8), (16384, 4096, 8), (16384, 4096, 12), (16384, 2048, 9), (8192, 8192, 8),
                  (2048, 1024, 12), (16384, 16384, 10), (1024, 512, 8), (32768, 4096, 8)]
    tensors, blobs, n_raw, n_coded = [], [], 0, 0
    for i in range(64):
        C, W, max_len = geometries[int(rng.integers(len(geometries)))]
        w = patchwork_tensor(rng, int(rng.integers(1, 150000)))
        n_present = np.unique(zo.split(w)[0]).size
        while (1 << max_len) < n_present:
            max_len += 1
        if i % 2:
            blob = zo.encode(w, C, W, zo.code_lengths(zo.histogram(zo.split(w)[0]), max_len))
        else:
            blob, _ = zm.compress(w, C, W, max_len)
        modes = chunk_modes(blob)
        n_raw += int((modes == 1).sum())
        n_coded += int((modes == 0).sum())
        tensors.append(w)
        blobs.append(blob)
    say(f"patchwork seed {seed}: {len(blobs)} tensors, {n_coded} coded and {n_raw} raw chunks")
    assert n_raw > 20 and n_coded > 20
    for stores in (None, zm.STORES_STREAMING):
        got = gpu_decode_tensors(blobs, stores=stores)
        for w, blob, g in zip(tensors, blobs, got):
            assert np.array_equal(g, w)
    for blob, w in list(zip(blobs, tensors))[::4]:
        assert np.array_equal(zo.decode(blob), w)


@pytest.mark.parametrize("kind,W,max_len", [("gauss", 4096, 8), ("wide", 4096, 12), ("wide", 16384, 12),
                                            ("wide", 32768, 12), ("gauss", 32768, 8)])
def test_outputs_larger_than_the_last_level_cache(kind, W, max_len):
    """a call that writes more than 256 MB takes the launch variant with non-temporal stores; every workgroup
    width is covered (streams of 16384 and 32768 values leave room for fewer streams per workgroup)"""
    import torch
    unit = synth.special_tensor(kind, (1 << 20) + 12345, seed=W + max_len)
    tensors = [np.tile(unit, 45)[: 45 * (1 << 20) + 777 * i] for i in range(3)]          # 3 x 47 M values: 283 MB of bf16
    say(f"{kind} W={W} L<={max_len}: compressing 3 x {tensors[0].size} values")
    with ThreadPoolExecutor(3) as ex:
        blobs = list(ex.map(lambda w: zm.compress(w, 32768, W, max_len)[0], tensors))
    assert sum(2 * w.size for w in tensors) > 256 << 20
    layer = zm.ExpertLayer([blobs], validate=False)
    for b in blobs:
        zm.validate_blob(b)
        assert (zm.blob_info(b[:384]).max_len > 8) == (kind == "wide")       # "wide" takes the long-code kernels
    bufs, starts, vals = layer.alloc_outputs(1)
    bufs[0].fill_(0x3333)
    layer.decode([0], bufs, starts, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = bufs[0].cpu().numpy().view(np.uint16)
    say("decoding with the reference codec")
    for m, (w, blob) in enumerate(zip(tensors, blobs)):
        g = got[starts[m]: starts[m] + vals[m]]
        assert np.array_equal(g, w)
        h = zo.header(blob)
        ref = np.zeros(w.size, np.uint16)
        step = -(-h["n_chunks"] // 64)
        with ThreadPoolExecutor(16) as ex:
            list(ex.map(lambda c0: zo.decode_chunks(blob, c0, min(h["n_chunks"], c0 + step), ref), range(0, h["n_chunks"], step)))
        assert np.array_equal(g, ref)


def test_bad_arguments_are_refused_on_the_host():
    import torch
    w = synth.special_tensor("gauss", 5000, 0)
    blob, _ = zm.compress(w, 4096, 4096)
    layer = zm.ExpertLayer([[blob]])
    out = torch.empty(5008, dtype=torch.int16, device="cuda")
    ptrs = (ctypes.c_void_p * 1)(out.data_ptr())
    P = ctypes.POINTER(ctypes.c_void_p)
    call = lambda ids, outs=ptrs, n=1: zm.decode_experts(layer._ptr_blobs, layer._ptr_tables, layer._ptr_infos, 1, 1,
                                                         (ctypes.c_int32 * 1)(ids), n, ctypes.cast(outs, P), 0)
    call(0)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint16)[:5000], w)
    for bad_id in (-1, 1):
        with pytest.raises(zm.ZipMoEError):
            call(bad_id)
    with pytest.raises(zm.ZipMoEError):
        call(0, (ctypes.c_void_p * 1)(out.data_ptr() + 2))        # misaligned output
    with pytest.raises(zm.ZipMoEError):
        call(0, (ctypes.c_void_p * 1)(None))
    call(0, n=0)                                                   # nothing selected: no launch, no error


def oracle_decode_parallel(blobs, workers=16):
    with ThreadPoolExecutor(workers) as ex:
        return list(ex.map(zo.decode, blobs))


def compress_expert(wl, layer, expert, stream_values=4096):
    return [zm.compress(m, wl.chunk_values, stream_values)[0] for m in synth.expert_tensors(wl, layer, expert)]


def test_config1_single_matrix():
    w = synth.expert_matrix(synth.CFG1, 0, 0, 0)
    lengths = zo.code_lengths(zo.histogram(zo.split(w)[0]), 8)
    ref_blob = zo.encode(w, 4096, 4096, lengths)             # the reference encoder's own blob
    got = gpu_decode_tensors([ref_blob])[0]
    assert np.array_equal(got, zo.decode(ref_blob)) and np.array_equal(got, w.reshape(-1))


def test_config2_one_expert_with_outliers():
    import torch
    wl = synth.CFG2
    tensors = synth.expert_tensors(wl, 0, 0)
    blobs = compress_expert(wl, 0, 0)
    layer = zm.ExpertLayer([blobs])
    bufs, starts, vals = layer.alloc_outputs(1)
    layer.decode([0], bufs, starts, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = bufs[0].cpu().numpy().view(np.uint16)
    ref = oracle_decode_parallel(blobs)
    for m in range(3):
        g = got[starts[m]: starts[m] + vals[m]]
        assert np.array_equal(g, ref[m]) and np.array_equal(g, tensors[m].reshape(-1))


def test_config3_layer_top8_zipf():
    import torch
    wl = synth.CFG3
    say("config 3: generating and compressing 64 experts")
    with ThreadPoolExecutor(16) as ex:
        all_blobs = list(ex.map(lambda e: compress_expert(wl, 0, e), range(wl.n_experts)))
    layer = zm.ExpertLayer(all_blobs, validate=False)
    bufs, starts, vals = layer.alloc_outputs(wl.top_k)
    stream = torch.cuda.current_stream().cuda_stream
    for call in range(6):
        ids = synth.route(wl, 0, call)
        assert len(set(ids.tolist())) == wl.top_k
        for b in bufs:
            b.fill_(0x1111)
        layer.decode(ids, bufs, starts, stream)
        torch.cuda.synchronize()
        say(f"config 3 call {call}: experts {ids.tolist()}")
        flat = [all_blobs[e][m] for e in ids for m in range(3)]
        ref = oracle_decode_parallel(flat) if call < 2 else None
        for j, e in enumerate(ids):
            got = bufs[j].cpu().numpy().view(np.uint16)
            orig = synth.expert_tensors(wl, 0, int(e))
            for m in range(3):
                g = got[starts[m]: starts[m] + vals[m]]
                assert np.array_equal(g, orig[m].reshape(-1))
                if ref is not None:
                    assert np.array_equal(g, ref[3 * j + m])


def test_decode_tensors_with_parts_in_separate_allocations():
    """zm_decode_tensors: decode table, chunk table, SM section and E-chunks each in an allocation of its own"""
    import torch
    tensors = [synth.special_tensor(k, n, seed=n) for k, n in (("gauss", 3 * 16384 + 700), ("wide", 20000),
                                                               ("uniform_u16", 9000), ("two_exponents", 4096))]
    blobs = [zm.compress(w, 16384, 4096, 12 if i == 1 else 8)[0] for i, w in enumerate(tensors)]
    n = len(blobs)
    parts, infos, outs = (zm.TensorParts * n)(), (zm.TensorInfo * n)(), (ctypes.c_void_p * n)()
    keep = []
    for i, b in enumerate(blobs):
        info = zm.blob_info(b)
        infos[i] = info
        cut = lambda lo, hi: torch.from_numpy(b[lo:hi].copy()).cuda()
        pieces = [cut(info.lut_offset, info.table_offset), cut(info.table_offset, info.table_offset + info.table_stride * (info.n_chunks + 1)),
                  cut(info.sm_offset, info.e_offset), cut(info.e_offset, info.blob_size)]
        out = torch.full((int(info.n_values) + 2 * GUARD,), GUARD_WORD, dtype=torch.int16, device="cuda")
        keep.append((pieces, out))
        parts[i] = zm.TensorParts(*[p.data_ptr() for p in pieces])
        outs[i] = out.data_ptr() + 2 * GUARD
    zm.decode_tensors(parts, infos, n, ctypes.cast(outs, ctypes.POINTER(ctypes.c_void_p)), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for (pieces, out), w, b in zip(keep, tensors, blobs):
        a = out.cpu().numpy().view(np.uint16)
        assert np.all(a[:GUARD] == GUARD_WORD) and np.all(a[-GUARD:] == GUARD_WORD)
        assert np.array_equal(a[GUARD:-GUARD], zo.decode(b)) and np.array_equal(a[GUARD:-GUARD], w)


def test_limits_of_one_call():
    """256 tensors in one call is the most a call takes (six launches); one more is refused; a stream too long to
    stage in LDS is refused on the host; the longest stream one wave can stage decodes correctly"""
    import torch
    small = [synth.special_tensor("gauss", 600 + i, seed=i) for i in range(256)]
    blobs = [zm.compress(w, 1024, 512)[0] for w in small]
    got = gpu_decode_tensors(blobs)
    for w, g in zip(small, got):
        assert np.array_equal(g, w)
    with pytest.raises(zm.ZipMoEError):
        gpu_decode_tensors(blobs + blobs[:1])
    # streams of 32768 values: only one fits the LDS of a workgroup
    w = synth.special_tensor("gauss", 2 * 32768 + 999, seed=3)
    blob, _ = zm.compress(w, 32768, 32768)
    assert np.array_equal(gpu_decode_tensors([blob])[0], w) and np.array_equal(zo.decode(blob), w)
    # streams of 131072 values can not be staged: refused, nothing launched
    big, _ = zm.compress(synth.special_tensor("gauss", 131072, seed=4), 131072, 131072)
    with pytest.raises(zm.ZipMoEError):
        gpu_decode_tensors([big])
    assert np.array_equal(zo.decode(big), synth.special_tensor("gauss", 131072, seed=4))
    torch.cuda.synchronize()


def test_layer_handle_decodes_like_the_array_call():
    """zm_layer_create / zm_layer_decode: the library's own handle for a layer's resident experts"""
    import torch
    rng = np.random.default_rng(5)
    n_experts, per = 5, 3
    tensors = [[synth.special_tensor(KINDS[int(rng.integers(len(KINDS)))], int(rng.integers(1, 90000)), seed=50 + 3 * e + m)
                for m in range(per)] for e in range(n_experts)]
    blobs = [[(zm.compress(w, 16384, 4096, 8)[0] if (e + m) % 2 else zo.encode_tensor(w, 16384, 4096, 8)[0])
              for m, w in enumerate(ts)] for e, ts in enumerate(tensors)]
    layer = zm.Layer(blobs)
    for e in range(n_experts):
        for m in range(per):
            a, b = layer.tensor_info(e, m), zm.blob_info(blobs[e][m][:384])
            assert bytes(a) == bytes(b)
    ids = [3, 0, 3, 4]                                           # a duplicate is decoded twice
    outs = [[torch.full((tensors[e][m].size + 2 * GUARD,), GUARD_WORD, dtype=torch.int16, device="cuda") for m in range(per)]
            for e in ids]
    ptrs = [o.data_ptr() + 2 * GUARD for row in outs for o in row]
    for stores in (zm.STORES_AUTO, zm.STORES_STREAMING):
        layer.decode(ids, ptrs, torch.cuda.current_stream().cuda_stream, stores)
        torch.cuda.synchronize()
        for j, e in enumerate(ids):
            for m in range(per):
                a = outs[j][m].cpu().numpy().view(np.uint16)
                assert np.all(a[:GUARD] == GUARD_WORD) and np.all(a[-GUARD:] == GUARD_WORD)
                assert np.array_equal(a[GUARD:-GUARD], tensors[e][m])
                assert np.array_equal(a[GUARD:-GUARD], zo.decode(blobs[e][m]))
                outs[j][m][GUARD:-GUARD].zero_()
    with pytest.raises(zm.ZipMoEError):
        layer.decode([n_experts], ptrs[:per])                    # id out of range
    layer.close()


def test_decode_call_can_be_captured_in_a_hip_graph():
    """the hot call allocates nothing and copies nothing, so it can be recorded into a graph; every replay,
    with eager work and synchronisations in between, must give the eager result"""
    import torch
    wl = synth.CFG2
    tensors = synth.expert_tensors(wl, 0, 0)
    blobs = compress_expert(wl, 0, 0)
    layer = zm.ExpertLayer([blobs, blobs])
    bufs, starts, vals = layer.alloc_outputs(2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    call = layer.make_call([1, 0], bufs, starts)
    with torch.cuda.stream(side):
        call(side.cuda_stream)                                  # eager warm-up on the capture stream
    side.synchronize()
    eager = [b.clone() for b in bufs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(torch.cuda.current_stream().cuda_stream)
    for replay in range(4):
        for b in bufs:
            b.fill_(0x2222 + replay)                            # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for b, e in zip(bufs, eager):
            assert torch.equal(b, e), replay
    got = bufs[0].cpu().numpy().view(np.uint16)
    for m in range(3):
        assert np.array_equal(got[starts[m]: starts[m] + vals[m]], tensors[m].reshape(-1))


def layer_calls(tensors_by_expert, chunk, stream_values, max_len, stores=None):
    """all experts of a layer in one call; returns the decoded arrays, expert by expert"""
    import torch
    flat = [w for ts in tensors_by_expert for w in ts]
    with ThreadPoolExecutor(16) as ex:
        blobs = list(ex.map(lambda w: zm.compress(w, chunk, stream_values, max_len)[0], flat))
    per = len(tensors_by_expert[0])
    layer = zm.Layer([blobs[i: i + per] for i in range(0, len(blobs), per)])
    outs = [torch.full((w.size + 2 * GUARD,), GUARD_WORD, dtype=torch.int16, device="cuda") for w in flat]
    shapes = zm.decode_launch_shapes([layer.tensor_info(e, m) for e in range(len(tensors_by_expert)) for m in range(per)],
                                     zm.STORES_AUTO if stores is None else stores)
    layer.decode(list(range(len(tensors_by_expert))), [o.data_ptr() + 2 * GUARD for o in outs],
                 torch.cuda.current_stream().cuda_stream, zm.STORES_AUTO if stores is None else stores)
    torch.cuda.synchronize()
    res = []
    for o in outs:
        a = o.cpu().numpy().view(np.uint16)
        assert np.all(a[:GUARD] == GUARD_WORD) and np.all(a[-GUARD:] == GUARD_WORD), "guard words overwritten"
        res.append(a[GUARD:-GUARD])
    layer.close()
    return flat, blobs, res, shapes


@pytest.mark.parametrize("n_tensors,max_len,stream_values,launches", [(48, 8, 4096, [48]), (49, 8, 4096, [49]), (240, 8, 1024, [240]),
                                                                      (241, 8, 4096, [121, 120]), (60, 12, 4096, [60]),
                                                                      (50, 8, 16384, [50])])
def test_many_tensors_share_a_launch(n_tensors, max_len, stream_values, launches):
    """blobs of few layouts and 64 Ki values or more travel in 16 bytes each, up to 240 of them in a launch"""
    n = (1 << 16) + 4099
    kinds = ["gauss", "rare_last"] if max_len == 8 else ["gauss"]
    tensors = [[synth.special_tensor(kinds[i % len(kinds)], n + (i % 2), seed=i % 4)] for i in range(n_tensors)]
    flat, blobs, got, shapes = layer_calls(tensors, 16384, stream_values, max_len)
    assert [s.tensors for s in shapes] == launches
    for i, (w, g) in enumerate(zip(flat, got)):
        assert np.array_equal(g, w), i
    assert np.array_equal(got[-1], zo.decode(blobs[-1]))


@pytest.mark.parametrize("count,stores,through", [(7, zm.STORES_AUTO, True), (48, zm.STORES_STREAMING, True), (3, zm.STORES_AUTO, True),
                                                  (6, zm.STORES_STREAMING, True), (2, zm.STORES_CACHED, False)])
@pytest.mark.parametrize("max_len", [8, 12])
def test_launches_numbered_through_tensors_of_very_different_lengths(count, stores, through, max_len):
    """one long tensor beside short ones: the launch counts through the workgroups of all of them, unless few would be idle"""
    lengths = [(9 << 20) + 5] + [(1 if max_len == 8 else 3000) + 1237 * i for i in range(count - 1)]
    order = np.random.default_rng(count).permutation(count)
    tensors = [[synth.special_tensor("gauss" if max_len == 8 else "wide", lengths[i], seed=3 + int(i))] for i in order]
    flat, blobs, got, shapes = layer_calls(tensors, 16384, 4096, max_len, stores)
    assert all((zm.blob_info(b).max_len > 8) == (max_len > 8) for b in blobs)
    workgroups = [-(-(-(-n // 4096)) // 2) for n in lengths]
    assert [(s.tensors, s.workgroups) for s in shapes] == [(count, sum(workgroups) if through else max(workgroups))]
    for w, g in zip(flat, got):
        assert np.array_equal(g, w)


@pytest.mark.parametrize("n", [4 * 4096 * 4, 8 * 16384 + 512, 16384 + 8191, 2 * 16384 + 3])
@pytest.mark.parametrize("W", [1024, 8192, 16384])
def test_raw_and_long_streams_in_groups_of_tiles(n, W):
    """streams of one and of several groups of tiles, whole and cut off, coded and raw, under every store kind"""
    tensors = [synth.special_tensor(k, n, seed=W + n) for k in ("gauss", "uniform_u16", "wide", "all_equal")]
    blobs = [zm.compress(w, 32768, W, 12 if k == 2 else 8)[0] for k, w in enumerate(tensors)]
    for stores in (None, zm.STORES_CACHED, zm.STORES_STREAMING):
        for w, b, g in zip(tensors, blobs, gpu_decode_tensors(blobs, stores=stores)):
            assert np.array_equal(g, w) and np.array_equal(g, zo.decode(b))


@pytest.mark.parametrize("layouts,stores,max_len,launches", [(4, zm.STORES_CACHED, 8, [60]), (4, zm.STORES_STREAMING, 8, [60]), (4, zm.STORES_CACHED, 12, [60]),
                                                             (4, zm.STORES_STREAMING, 12, [60]), (5, zm.STORES_CACHED, 8, [48, 12])])
def test_many_tensors_share_a_launch_with_every_kind_of_store(layouts, stores, max_len, launches):
    """more than 36 MiB in a launch, where ordinary stores take over from device-scope ones; and more layouts than a shared launch has room for"""
    tensors = [[synth.special_tensor("gauss" if max_len == 8 else "wide", 340_000 + 4099 * (i % layouts), seed=i % 4)] for i in range(60)]
    flat, _, got, shapes = layer_calls(tensors, 16384, 4096, max_len, stores)
    assert sum(2 * w.size for w in flat[:48]) <= 36 << 20 < sum(2 * w.size for w in flat)
    assert [s.tensors for s in shapes] == launches
    for i, (w, g) in enumerate(zip(flat, got)):
        assert np.array_equal(g, w), i


def test_more_tensors_of_long_codes_than_one_launch_takes():
    tensors = [[synth.special_tensor("wide", (1 << 16) + 4099 + i % 3, seed=i % 4)] for i in range(241)]
    flat, _, got, shapes = layer_calls(tensors, 16384, 4096, 12)
    assert [(s.tensors, s.round_symbols) for s in shapes] == [(121, 2), (120, 2)]
    for i, (w, g) in enumerate(zip(flat, got)):
        assert np.array_equal(g, w), i


@pytest.mark.parametrize("lengths", [[7168 * 4096], [7168 * 4096 + 1], [14_000_003] * 3, [38_000_001, 5, 70_000], [5_000_011] * 8,
                                     [660_007] * 60], ids=["at the line", "above it", "three", "numbered", "eight", "shared"])
def test_launches_of_many_streams_with_streaming_stores(lengths):
    """up to 7168 streams of 4096 values and more of them: one tensor, row launches of few and of many, a numbered one and a shared one"""
    w = synth.special_tensor("gauss", max(lengths), seed=5)
    tensors = [[w[7 * i: 7 * i + n] if 7 * i + n <= w.size else w[:n]] for i, n in enumerate(lengths)]
    flat, _, got, shapes = layer_calls(tensors, 16384, 4096, 8, zm.STORES_STREAMING)
    assert len(shapes) == 1 and shapes[0].streaming_stores == 1
    for a, g in zip(flat, got):
        assert np.array_equal(g, a)


@pytest.mark.parametrize("max_len", [8, 12])
@pytest.mark.parametrize("lengths", [[7168 * 4096], [7168 * 4096 + 1], [11_000_003] * 3, [31_000_001, 5, 70_000], [660_007] * 60],
                         ids=["at the line", "above it", "three", "numbered", "shared"])
def test_launches_of_many_streams_that_stay_cached(lengths, max_len):
    """up to 7168 streams of 4096 values and more of them, with stores that leave their lines cached"""
    w = synth.special_tensor("gauss" if max_len == 8 else "wide", max(lengths), seed=6)
    tensors = [[w[7 * i: 7 * i + n] if 7 * i + n <= w.size else w[:n]] for i, n in enumerate(lengths)]
    flat, _, got, shapes = layer_calls(tensors, 16384, 4096, max_len, zm.STORES_CACHED)
    assert sum(s.tensors for s in shapes) == len(lengths) and all(s.streaming_stores == 0 for s in shapes)
    for a, g in zip(flat, got):
        assert np.array_equal(g, a)


def test_a_launch_of_many_streams_holds_tensors_of_every_kind():
    """raw chunks, cut-off streams and streams shorter than a group beside whole ones, in one launch of more than 7168 streams"""
    tensors = [synth.special_tensor("gauss", 40_000_003, 5)] + [synth.special_tensor(kind, n, n) for kind in ("uniform_u16", "rare_last", "all_equal")
                                                               for n in (1, 9, 511, 4095, 4097, 50_001)]
    blobs = [zm.compress(w, 16384, 4096 if i % 2 == 0 else 512, 8)[0] for i, w in enumerate(tensors)]
    for w, g in zip(tensors, gpu_decode_tensors(blobs, stores=zm.STORES_STREAMING)):
        assert np.array_equal(g, w)


@pytest.mark.parametrize("n", [(18 << 20) - 1, 18 << 20, (18 << 20) + 1])
def test_outputs_at_the_line_between_the_store_kinds(n):
    """36 MiB in one launch"""
    w = synth.special_tensor("gauss", n, seed=n & 7)
    blob, _ = zm.compress(w, 16384, 4096)
    assert np.array_equal(gpu_decode_tensors([blob], stores=zm.STORES_CACHED)[0], w)


def test_outputs_between_the_store_kinds():
    """a launch of up to 7168 streams that writes more than 36 MiB, where it takes ordinary stores, and less than the last-level cache"""
    w = synth.special_tensor("gauss", (20 << 20) + 777, seed=9)
    blob, _ = zm.compress(w, 16384, 4096)
    assert np.array_equal(gpu_decode_tensors([blob])[0], w)


def bursts(n, n_rare, burst, gap, seed):
    """exponents of short codes, with runs of `burst` rare ones every `gap` values: few bits a value, but four codes in a
    row that do not fit a 32-bit window"""
    rng = np.random.default_rng(seed)
    e = (120 - rng.geometric(0.6, n).clip(1, 9)).astype(np.uint16)
    for at in range(seed % 7, n, gap):
        m = min(burst, n - at)
        e[at: at + m] = 121 + rng.integers(0, n_rare, m)
    return (e << 7) | rng.integers(0, 128, n, dtype=np.uint16)


@pytest.mark.parametrize("W", [512, 2048, 4096, 16384])
@pytest.mark.parametrize("n_rare,burst,gap", [(100, 8, 400), (100, 6, 4000), (100, 300, 20000), (60, 12, 300), (120, 1, 50)])
def test_long_codes_in_a_row(W, n_rare, burst, gap):
    """streams whose four-symbol windows overflow in some rounds, from the first pair of tiles to the last"""
    tensors, blobs = [], []
    for k, max_len in enumerate((9, 10, 11, 12)):
        w = bursts(3 * 16384 + 4096 * k + 77, n_rare, burst, gap, 5 + k)
        while (1 << max_len) < np.unique(zo.split(w)[0]).size:
            max_len += 1
        tensors.append(w)
        blobs.append(zm.compress(w, 16384, W, max_len)[0])
        assert zm.blob_info(blobs[-1][:384]).max_len > 8
        assert blobs[-1].size < 0.78 * 2 * w.size           # few enough bits a value for the four-symbol rounds
    for stores in (None, zm.STORES_STREAMING):
        for w, b, g in zip(tensors, blobs, gpu_decode_tensors(blobs, stores=stores)):
            assert np.array_equal(g, w) and np.array_equal(g, zo.decode(b))


@pytest.mark.parametrize("n_symbols", [3, 9, 17, 64, 129, 200, 256])
def test_long_code_tables_of_every_width(n_symbols):
    """exponent counts that fall off geometrically or not at all: from one shared eight-bit beginning to all that fit"""
    rng = np.random.default_rng(n_symbols)
    tensors, blobs = [], []
    for max_len in (9, 10, 11, 12):
        for p in (0.55, 0.85, 0.98):
            if (1 << max_len) < n_symbols:
                continue
            e = np.minimum(rng.geometric(1 - p, 40000) - 1, n_symbols - 1).astype(np.uint16)
            e[:n_symbols] = np.arange(n_symbols)
            w = (e << 7) | rng.integers(0, 128, e.size, dtype=np.uint16)
            tensors.append(w)
            blobs.append(zm.compress(w, 16384, 4096, max_len)[0])
    for w, b, g in zip(tensors, blobs, gpu_decode_tensors(blobs)):
        assert np.array_equal(g, w) and np.array_equal(g, zo.decode(b))


def test_longest_stream_of_long_codes_beside_the_widest_table():
    """the longest stream that one wave can stage, of a tensor with every exponent: its table comes on top"""
    w = synth.special_tensor("many_long", 40960 + 700, seed=2)
    blob, _ = zm.compress(w, 40960, 40960, 12)
    assert zm.blob_info(blob[:384]).max_len > 8
    assert np.array_equal(gpu_decode_tensors([blob])[0], w)
    big, _ = zm.compress(synth.special_tensor("many_long", 45056, seed=4), 45056, 45056, 12)
    with pytest.raises(zm.ZipMoEError):
        gpu_decode_tensors([big])


@pytest.mark.parametrize("n_present", [0, 9, 40, 300, 1 << 31])
@pytest.mark.parametrize("C,W,max_len", [(16384, 4096, 12), (16384, 4096, 9), (4096, 1024, 11), (32768, 32768, 12)])
def test_long_codes_do_not_depend_on_the_count_of_symbols_in_a_description(monkeypatch, n_present, C, W, max_len):
    """the LDS table is sized by it, the values come from the blob's own table all the same"""
    tensors = [synth.special_tensor(kind, n, seed=n) for kind in ("many_long", "wide", "gauss", "uniform_u16") for n in (3 * 16384 + 1234, 32768, 513)]
    blobs = [zm.compress(w, C, W, max_len)[0] for w in tensors]
    assert max(zm.blob_info(b).max_len for b in blobs) == max_len and max(zm.blob_info(b).n_present for b in blobs) == 256
    describe = zm.blob_info

    def with_another_count(blob):
        info = describe(blob)
        info.n_present = n_present
        return info

    monkeypatch.setattr(zm, "blob_info", with_another_count)
    # each by itself, so that no other tensor of the launch makes room for it, then all in one launch
    for w, b in zip(tensors, blobs):
        assert np.array_equal(gpu_decode_tensors([b], stores=zm.STORES_STREAMING)[0], w)
    for w, g in zip(tensors, gpu_decode_tensors(blobs)):
        assert np.array_equal(g, w)


def decode_at(blobs, ids, stores, shift, gap, backwards):
    """Decodes blobs[i] for i in ids from one arena in which every blob starts `shift` bytes past a multiple of 256 and `gap` bytes
    past the last, with outputs in the order of ids or backwards."""
    import torch
    at, starts = 0, []
    for b in blobs:
        starts.append(-(-at // 256) * 256 + shift)
        at = starts[-1] + b.size + gap
    arena = torch.zeros(at, dtype=torch.uint8, device="cuda")
    infos = (zm.TensorInfo * len(blobs))()
    blob_ptrs, table_ptrs = (ctypes.c_void_p * len(blobs))(), (ctypes.c_void_p * len(blobs))()
    for k, b in enumerate(blobs):
        arena[starts[k]: starts[k] + b.size].copy_(torch.from_numpy(np.ascontiguousarray(b)))
        infos[k] = zm.blob_info(b[:384])
        blob_ptrs[k] = arena.data_ptr() + starts[k]
        table_ptrs[k] = blob_ptrs[k] + infos[k].table_offset
    order = list(range(len(ids)))[::-1] if backwards else list(range(len(ids)))
    rooms, end = [0] * len(ids), GUARD
    for j in order:
        rooms[j] = end
        end += -(-int(infos[ids[j]].n_values) // 8) * 8 + GUARD
    out = torch.full((end,), GUARD_WORD, dtype=torch.int16, device="cuda")
    ptrs = (ctypes.c_void_p * len(ids))(*[out.data_ptr() + 2 * r for r in rooms])
    cast = lambda a, t=ctypes.c_void_p: ctypes.cast(a, ctypes.POINTER(t))
    rc = zm.lib().zm_decode_experts_stores(cast(blob_ptrs), cast(table_ptrs), cast(infos, zm.TensorInfo), len(blobs), 1,
                                           (ctypes.c_int32 * len(ids))(*ids), len(ids), cast(ptrs), stores,
                                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == zm.OK
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint16)
    untouched = np.ones(end, bool)
    for j, e in enumerate(ids):
        untouched[rooms[j]: rooms[j] + int(infos[e].n_values)] = False
    assert np.all(got[untouched] == GUARD_WORD)
    return [got[rooms[j]: rooms[j] + int(infos[e].n_values)] for j, e in enumerate(ids)]


@pytest.mark.parametrize("C,W,max_len", [(16384, 4096, 8), (12288, 4096, 8), (2560, 512, 8), (4096, 1024, 3), (1 << 17, 512, 8), (16384, 16384, 12),
                                         (32768, 32768, 12), (65536, 4096, 11)])
@pytest.mark.parametrize("count,shift,backwards", [(1, 0, False), (2, 16, False), (3, 0, True), (6, 0, False), (6, 208, True), (7, 0, False)])
def test_calls_of_few_tensors(C, W, max_len, count, shift, backwards):
    # up to six blobs cut alike travel in their own kind of arguments: those, and what does not fit it (chunks of other than 2^k
    # streams, addresses that are no multiple of 256, seven tensors, one of another length or codebook)
    n = 2 * C + C // 2 + 777
    kinds = ["two_exponents" if max_len < 8 else "gauss" if max_len == 8 else "wide"] * count
    tensors = [synth.special_tensor(kind, n, seed=50 + i) for i, kind in enumerate(kinds)]
    tensors.append(synth.special_tensor("gauss", n - 1, seed=7))
    tensors.append(synth.special_tensor("all_equal", n, seed=8))
    blobs = [zm.compress(w, C, W, max_len if i < count else max(max_len, 8))[0] for i, w in enumerate(tensors)]
    refs = [zo.decode(b) for b in blobs]
    for ids in (list(range(count)), list(range(count))[::-1], list(range(count - 1)) + [count], list(range(count - 1)) + [count + 1], [0] * count):
        for stores in (zm.STORES_CACHED, zm.STORES_STREAMING):
            for e, g in zip(ids, decode_at(blobs, ids, stores, shift, 4096, backwards)):
                assert np.array_equal(g, refs[e]) and np.array_equal(g, tensors[e])


@pytest.mark.parametrize("W", [8192, 20480, 24576, 32768])
@pytest.mark.parametrize("bits", [1, 2, 3, 5, 7])
def test_long_streams_of_every_density(W, bits):
    # streams of several groups of tiles that take between a kilobyte and thrice what a wave holds in registers, whole, cut off in
    # front of a group's end and within a tile; every exponent's code has `bits` bits, or (long codes) around twice as many
    rng = np.random.default_rng(W + bits)
    blobs, tensors = [], []
    for n in (3 * W, 2 * W + W // 2, W + 4096, 2 * W - 4095, W + 8 * 512 + 3):
        e = 100 + rng.permutation(np.arange(n, dtype=np.uint32) % (1 << bits)).astype(np.uint16)
        tensors.append((e << 7) | rng.integers(0, 128, n, dtype=np.uint16))
        blobs.append(zm.compress(tensors[-1], 2 * W, W, 8)[0])
        tensors.append(bursts(n, 60, 300, 20000 >> bits, bits))
        blobs.append(zm.compress(tensors[-1], W, W, 12)[0])
    for stores in (zm.STORES_CACHED, zm.STORES_STREAMING):
        for w, b, g in zip(tensors, blobs, gpu_decode_tensors(blobs, stores=stores)):
            assert np.array_equal(g, w) and np.array_equal(g, zo.decode(b))


@pytest.mark.parametrize("streams,count", [(7168, 1), (7169, 1), (1024, 7), (1024, 8), (1025, 8), (512, 14), (512, 15), (180, 48)])
@pytest.mark.parametrize("stores,max_len", [(zm.STORES_CACHED, 8), (zm.STORES_STREAMING, 8), (zm.STORES_STREAMING, 12)])
def test_launches_around_the_lines_between_wave_counts(streams, count, stores, max_len):
    """as many streams as find a place at once and more, in one tensor and in many"""
    n = streams * 4096 - 5
    w = synth.special_tensor("gauss" if max_len == 8 else "wide", n + 64, seed=streams)
    tensors = [[w[k % 8: k % 8 + n]] for k in range(count)]
    flat, _, got, shapes = layer_calls(tensors, 16384, 4096, max_len, stores)
    assert len(shapes) == 1
    for a, g in zip(flat, got):
        assert np.array_equal(g, a)


@pytest.mark.parametrize("max_len", [8, 12])
@pytest.mark.parametrize("W", [4608, 6144, 7680, 10240, 14336])
def test_streams_of_no_whole_groups(W, max_len):
    """longer than a group of tiles and no multiple of it, with last streams that are whole groups all the same or end inside a tile"""
    lengths = [3 * W, 2 * W + 4096, 5 * W + 8192 if W > 8192 else 5 * W + 512, W + 1, 2 * W - 511, 4096, 40 * W - 5]
    tensors = [synth.special_tensor("gauss" if max_len == 8 else "wide", n, seed=n) for n in lengths]
    tensors.append(bursts(3 * W, 60, 300, 5000, W))
    blobs = [zm.compress(w, 2 * W, W, max_len)[0] for w in tensors]
    for stores in (zm.STORES_CACHED, zm.STORES_STREAMING):
        for w, b, g in zip(tensors, blobs, gpu_decode_tensors(blobs, stores=stores)):
            assert np.array_equal(g, w) and np.array_equal(g, zo.decode(b))
        for i in range(3):
            assert np.array_equal(gpu_decode_tensors(blobs[i: i + 1], stores=stores)[0], tensors[i])


@pytest.mark.parametrize("streams", [[8192, 4096, 4096, 4096], [8192, 8192, 8192, 4096], [8192, 1024, 1024, 512], [16384, 4096, 1024, 4096],
                                     [4096, 4096, 4096, 1024], [4096, 1024, 512, 1024], [6144, 4096, 4096, 12288], [10240, 4096, 8192, 10240]])
@pytest.mark.parametrize("count", [5, 12, 60])
@pytest.mark.parametrize("max_len", [8, 12])
def test_launches_of_several_stream_lengths(streams, count, max_len):
    """one launch decodes streams of one group of tiles, of several, of none, of each length in the majority: up to six tensors, more, and many that
    share a launch; every fourth one is cut off inside a tile"""
    n = (1 << 16) + 12288
    tensors, blobs = [], []
    for i in range(count):
        kind = "gauss" if max_len == 8 else ("wide", "gauss")[i % 2]
        tensors.append(synth.special_tensor(kind, n - 5 * (i % 4 == 3 and count < 60), seed=i % 5))
        blobs.append(zm.compress(tensors[-1], 2 * streams[i % 4], streams[i % 4], max_len)[0])
    for stores in (zm.STORES_CACHED, zm.STORES_STREAMING):
        for w, b, g in zip(tensors, blobs, gpu_decode_tensors(blobs, stores=stores)):
            assert np.array_equal(g, w)
    assert np.array_equal(gpu_decode_tensors(blobs[:1], stores=zm.STORES_CACHED)[0], zo.decode(blobs[0]))


@pytest.mark.parametrize("streams,count", [(3072, 1), (3073, 1), (512, 6), (513, 6), (256, 12), (257, 12), (64, 48), (65, 48), (1024, 1), (1025, 1), (128, 8), (129, 8)])
@pytest.mark.parametrize("max_len", [8, 12])
def test_launches_around_the_lines_of_few_streams(streams, count, max_len):
    """with stores that leave their lines cached, as many streams as ask for their bytes early and one more"""
    n = streams * 4096 - 5
    w = synth.special_tensor("gauss" if max_len == 8 else "wide", n + 64, seed=streams)
    tensors = [[w[k % 8: k % 8 + n]] for k in range(count)]
    flat, _, got, shapes = layer_calls(tensors, 16384, 4096, max_len, zm.STORES_CACHED)
    assert len(shapes) == 1
    for a, g in zip(flat, got):
        assert np.array_equal(g, a)


@pytest.mark.parametrize("W,max_len", [(512, 8), (4096, 8), (4096, 12), (16384, 8)])
@pytest.mark.parametrize("damage", ["start", "chunk behind", "chunk in front", "raw"])
def test_streams_that_a_table_places_outside_are_left_alone(W, max_len, damage):
    """entries of one chunk whose places wrap in 32 or 64 bits: its streams write nothing (the words before stay), the others are decoded"""
    import torch
    C, n = 2 * W, 7 * W + 5
    w = synth.special_tensor("gauss" if max_len == 8 else "wide", n, seed=W)
    blob = zm.compress(w, C, W, max_len)[0].copy()
    assert chunk_modes(blob)[1] == 0
    info = zm.blob_info(blob)
    entry = info.table_offset + info.table_stride * 1
    places = {"start": (entry + 12, "<u4", (1 << 32) - 16), "chunk behind": (entry, "<u8", (1 << 64) - 16), "chunk in front": (entry, "<u8", 0),
              "raw": (entry, "<u8", (1 << 64) - 16 | 1)}
    at, kind, value = places[damage]
    blob[at: at + int(kind[2])] = np.array([value], kind).view(np.uint8)
    layer = zm.ExpertLayer([[blob]], validate=False)
    bufs, starts, _ = layer.alloc_outputs(1)
    bufs[0].fill_(GUARD_WORD)
    layer.decode([0], bufs, starts, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = bufs[0].cpu().numpy().view(np.uint16)
    assert np.all(got[C: 2 * C] == GUARD_WORD)
    assert np.array_equal(got[:C], w[:C]) and np.array_equal(got[2 * C: n], w[2 * C:])


def bundle_tensor(n, W, max_len, seed):
    """Gaussian weights with streams that a bundle has to treat apart: a chunk and four chunks that are stored raw, half a stream and two streams of
    rare exponents, and lanes whose symbols all have the longest codes"""
    rng = np.random.default_rng(seed)
    w = synth.special_tensor("gauss", n, seed).copy()

    def rare(at, count):
        at = max(0, min(at, n - count))
        w[at: at + count] = (rng.integers(0x90, 0xa8, count).astype(np.uint16) << 7) | (w[at: at + count] & 0x807F)

    for k in range(5):
        rare((n * (k + 1) // 7) // 8 * 8, 8)
    rare(n // 3 // W * W + W // 2, min(W // 2, n // 64))
    if n > 256 * W:
        rare(n // 2 // (4 * W) * 4 * W, 4 * W)
        rare(n // 5 // (16 * W) * 16 * W, 16 * W)
        rare(n // 4 // (4 * W) * 4 * W, 2 * W)
    return w


@pytest.mark.parametrize("count,ragged,stores", [(1, False, zm.STORES_CACHED), (7, True, zm.STORES_STREAMING), (60, False, zm.STORES_CACHED)])
@pytest.mark.parametrize("W,max_len,streams,cached,streaming", [
    (512, 8, 9180, 1, 1), (512, 8, 9217, 8, 8), (512, 12, 9217, 8, 8), (512, 12, 30000, 8, 8), (1024, 8, 10241, 4, 4), (1024, 8, 16385, 1, 1), (1024, 12, 7169, 4, 4),
    (1024, 12, 16385, 4, 4), (2048, 8, 6145, 2, 2), (2048, 8, 9217, 1, 1), (2048, 8, 9180, 2, 2), (2048, 12, 6145, 2, 2), (2048, 12, 9217, 2, 2)])
def test_waves_that_take_several_short_streams(W, max_len, streams, cached, streaming, count, ragged, stores):
    """at the lines from which on they do: tensors of no whole bundle and a cut-off last stream, with streams in between that are treated apart; whole
    blobs alike, tensors of very different lengths, many in a launch; and what a damaged chunk table places outside stays as it was"""
    import torch
    lengths = [max(1, (streams // (2 ** k if k else 1)) // 2) for k in range(count)] if ragged else [-(-streams // count)] * count
    lengths[0] += max(0, streams - sum(lengths))
    cut = [5 if k % 2 or count == 1 else 0 for k in range(count)]
    tensors = [[bundle_tensor(s * W - cut[k], W, max_len, seed=k % 3)] for k, s in enumerate(lengths)]
    flat, blobs, got, shapes = layer_calls(tensors, 4 * W, W, max_len, stores)
    assert {int(zm.blob_info(b).max_len > 8) for b in blobs} == {int(max_len > 8)} and len(shapes) == 1
    # the launch is one of bundles, or is not: a wave for each whole bundle and for each other stream, two waves a workgroup
    bundle = streaming if stores == zm.STORES_STREAMING else cached
    whole = [s - (c > 0) for s, c in zip(lengths, cut)]
    blocks = [(w // bundle + w % bundle + (c > 0) + 1) // 2 for w, c in zip(whole, cut)]
    assert shapes[0].workgroups in (max(blocks), sum(blocks))
    assert count == 60 or set(chunk_modes(blobs[0])) == {0, 1}
    for a, g in zip(flat, got):
        assert np.array_equal(g, a)
    assert np.array_equal(got[-1], zo.decode(blobs[-1]))
    if count > 1:
        return
    blob, (w,) = blobs[0].copy(), flat
    info = zm.blob_info(blob)
    at = info.table_offset + info.table_stride * 5
    assert chunk_modes(blob)[5] == 0
    blob[at + 12: at + 16] = np.array([(1 << 32) - 16], "<u4").view(np.uint8)         # the first two streams of chunk 5
    layer = zm.ExpertLayer([[blob]], validate=False)
    bufs, starts, _ = layer.alloc_outputs(1)
    bufs[0].fill_(GUARD_WORD)
    layer.decode([0], bufs, starts, torch.cuda.current_stream().cuda_stream, stores)
    torch.cuda.synchronize()
    back, lost = bufs[0].cpu().numpy().view(np.uint16)[: w.size], slice(20 * W, 22 * W)
    assert np.all(back[lost] == GUARD_WORD)
    back[lost] = w[lost]
    assert np.array_equal(back, w)
