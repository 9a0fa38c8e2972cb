"""Parity of the HIP Huffman stage with the CPU oracle (Section 4.4.1: the quantisation codes
of the predictive form are encoded with Huffman coding; restoring begins with Huffman
decoding).  Bar: the stream -- length bytes, chunk offsets, payload words -- and the totals
bit-exact; decoding restores the input bytes."""
from __future__ import annotations

import huffman_streams as HS
import numpy as np
import pytest

import oracle
from paper_2510_11400_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    from paper_2510_11400_amd import api as _api
    return _api


def _check(api, data, name=""):
    print(f"[huffman] {name} n={data.size}", flush=True)
    want, bits = oracle.huffman_encode(data)
    d = torch.from_numpy(data).cuda() if data.size else torch.empty(0, dtype=torch.uint8, device="cuda")
    stream, totals = api.fh_huffman_encode(d)
    torch.cuda.synchronize()
    used, got_bits = (int(v) for v in totals.cpu().tolist())
    assert (used, got_bits) == (want.size, bits), f"{name}: totals {(used, got_bits)} vs {(want.size, bits)}"
    got = stream.cpu().numpy()[:used]
    assert np.array_equal(got[:256], want[:256]), f"{name}: code lengths differ"
    chunks = (data.size + 255) // 256
    end = 256 + 4 * (chunks + 1)
    assert np.array_equal(got[256:end], want[256:end]), f"{name}: chunk offsets differ"
    bad = np.flatnonzero(got[end:] != want[end:])
    assert bad.size == 0, f"{name}: payload differs first at byte {bad[:4]}"
    back = api.fh_huffman_decode(stream[:used], data.size)
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy(), data), f"{name}: decoded bytes differ"
    return want


@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 255, 256, 257, 4095, 65535, 65536, 65537, 1 << 20, (1 << 22) + 13])
def test_sizes_around_vectors_chunks_and_groups(api, n):
    rng = np.random.default_rng(n)
    data = np.clip(np.rint(rng.normal(128, 2.5, n)), 0, 255).astype(np.uint8)
    _check(api, data, "normal around 128")


@pytest.mark.parametrize("n", [224 * 131072 - 1, 224 * 131072 + 16, 256 * 131072 - 1, 256 * 131072, 257 * 131072 + 5])
def test_sizes_around_a_histogram_workgroup_for_each_unit(api, n):
    rng = np.random.default_rng(n)
    _check(api, (rng.standard_normal(n, dtype=np.float32) * np.float32(9.5) + np.float32(128)).clip(0, 255).astype(np.uint8), "histogram workgroups")


@pytest.mark.parametrize("spread", [2.5, 14.0, 20.0, -1.0, 0.0])
def test_streams_long_enough_that_a_workgroup_decodes_several_groups(api, spread):
    # Beyond 256 * 488 chunks the decoder has a workgroup of 1024 threads per compute unit and deals the chunks out evenly: 1026
    # each here, so a workgroup takes a pass with every thread at work (34 words per chunk fit the LDS stage then; spread
    # 2.5 gives 27) and another of two chunks, the last one fewer and a ragged chunk.
    # spread 14: codes longer than the decoder's fast table occur; 14 and 20: more words per chunk than the stage
    # holds for 1024 (and for 768) chunks, so its passes seat fewer; -1: a clustered first half and noise behind it, whose words
    # go through the per-thread rings; 0: uniform bytes, all codes eight bits long, which are copied
    n = 256 * (256 * 1024 + 300) + 77
    rng = np.random.default_rng(int(abs(spread) * 10))
    if spread > 0:
        data = np.clip(np.rint(rng.normal(128, spread, n)), 0, 255)
    elif spread < 0:
        data = np.concatenate([np.clip(np.rint(rng.normal(128, 3.0, n // 2)), 0, 255), rng.integers(0, 256, n - n // 2)])
    else:
        data = rng.integers(0, 256, n)
    want = _check(api, data.astype(np.uint8), f"spread {spread}")
    (_, (threads, stage)), seats = HS.decoder_shapes()[0].items(), HS.decoder_shapes()[1]
    chunks = -(-n // 256)
    share = -(-chunks // 256)
    assert chunks > 256 * seats and share > threads
    offsets = HS.offsets_of(want, n)
    kinds = {staged for b in range(256) for _, staged in HS.passes(offsets, b * share, min((b + 1) * share, chunks), threads, stage)}
    assert bool((want[:256] == 8).all()) == (spread == 0.0)
    assert spread == 0.0 or kinds == ({True, False} if spread < 0 else {True})


@pytest.mark.parametrize("more", [0, 1])
def test_streams_on_both_sides_of_the_scan(api, more):
    # up to 4096 groups of 65536 symbols every workgroup of the write pass adds up the group sums before its own, beyond
    # that a scan kernel does; the stream's groups differ in size, so a sum left out or taken twice moves the payload
    rng = np.random.default_rng(7)
    piece = np.clip(np.rint(rng.normal(128, 3.0, 99991)), 0, 255).astype(np.uint8)
    data = np.resize(piece, 4096 * 65536 + more)
    _check(api, data, f"{data.size} symbols")


@pytest.mark.parametrize("groups", [[4000, 95, 1], [4000, 95, 2], [1, 0, 1, 4093, 1]])
def test_launches_of_several_streams_on_both_sides_of_the_scan(api, groups):
    # 4096 groups of a launch, and 4097, an empty stream has a workgroup too; scanned launches with short streams in them
    rng = np.random.default_rng(8)
    piece = np.clip(np.rint(rng.normal(128, 3.0, 99991)), 0, 255).astype(np.uint8)
    datas = [np.resize(piece, g * 65536 - (17 if g else 0)) for g in groups]
    print(f"[huffman] streams of {groups} groups", flush=True)
    batch = api.HuffmanBatch([torch.from_numpy(d).cuda() if d.size else torch.empty(0, dtype=torch.uint8, device="cuda") for d in datas])
    api.fh_huffman_encode_batch(batch)
    torch.cuda.synchronize()
    for d, stream, total in zip(datas, batch.streams, batch.totals.cpu().tolist()):
        want, bits = oracle.huffman_encode(d)
        assert total == [want.size, bits] and np.array_equal(stream[:want.size].cpu().numpy(), want), f"{d.size} symbols"


@pytest.mark.parametrize("kind", ["2.5", "14", "mixed"])
def test_outputs_stored_in_whole_cache_lines(api, kind):
    # a call of 384 MiB and more, as two streams that end inside a line, inside a half of one and inside a vector; 14: passes
    # that seat fewer chunks; mixed: noise behind the clustered half, whose words go through the rings
    rng = np.random.default_rng(3)
    sizes = [(200 << 20) + 256 * 77 + 64 + 48 + 5, (184 << 20) + 70]
    assert sum(sizes) >= 384 << 20
    piece = np.clip(np.rint(rng.normal(128, 2.5 if kind == "mixed" else float(kind), 9999991)), 0, 255).astype(np.uint8)
    datas = []
    for n in sizes:
        data = np.resize(piece, n)
        if kind == "mixed":
            data[n // 2:] = np.resize(rng.integers(0, 256, 9999973, dtype=np.uint8), n - n // 2)
        datas.append(data)
    print(f"[huffman] whole lines, {kind}", flush=True)
    batch = api.HuffmanBatch([torch.from_numpy(d).cuda() for d in datas])
    for o in batch.out:
        o.fill_(0xEE)
    api.fh_huffman_encode_batch(batch)
    api.fh_huffman_decode_batch(batch)
    torch.cuda.synchronize()
    for d, o in zip(batch.data, batch.out):
        assert torch.equal(o, d)


@pytest.mark.parametrize("kind", ["deep", "flat", "nearly flat"])
@pytest.mark.parametrize("n", [5, 16411, 256 * 488 * 256, 256 * 488 * 256 + 3])
def test_decoder_forms(api, n, kind):
    # 488 chunks per compute unit are the most that workgroups of 512 threads take.  deep: code lengths up to the limit of
    # 24 and long codes side by side, so that a window of the stream runs out between four symbols; flat: eight bits each, which are copied
    # (the last word a part of one); nearly flat: lengths 7 to 9, 64 words per chunk and all of them decoded.
    rng = np.random.default_rng(n % 1000)
    if kind == "deep":
        data = np.minimum(rng.geometric(0.5, n) - 1, 255)
        for at in range(0, min(n, 3000) - 40, 97):            # symbols that occur a few times, side by side
            data[at:at + 33] = 40 + rng.permutation(33)
    else:
        data = np.arange(n) % 256
        if kind == "nearly flat":
            data = np.where(rng.random(n) < 0.01, 7, data)
    _check(api, data.astype(np.uint8), f"{kind}")


@pytest.mark.parametrize("kind", ["2.5", "14", "nearly flat"])
@pytest.mark.parametrize("counts_on", ["host", "device"])
def test_decoder_on_both_sides_of_the_wide_workgroups(api, counts_on, kind):
    """Workgroups of 512 threads take up to 488 chunks per compute unit where the count is the host's, up to 512 where it is
    on the device and the host knows a bound; one symbol more and the launch has workgroups of 1024.  Counts on the
    device: the bound itself, and two thirds of it, as the whole chain has them.  Nearly flat: 64 words per chunk, of which
    the narrow workgroup's stage does not hold 512 chunks, so that its share takes a second pass."""
    shapes, seats = HS.decoder_shapes()
    (narrow, stage), _ = shapes.items()
    limit = 256 * (seats if counts_on == "host" else narrow) * 256
    rng = np.random.default_rng(limit % 1000)
    full = rng.integers(0, 256, limit + 1) if kind == "nearly flat" else np.clip(np.rint(rng.normal(128, float(kind), limit + 1)), 0, 255)
    full = full.astype(np.uint8)
    if kind == "nearly flat":
        full[rng.random(full.size) < 0.01] = 7
    for n in (limit, limit + 1):
        if counts_on == "host":
            _check(api, full[:n], f"{n} symbols, {kind}")
            continue
        d = torch.from_numpy(full[:n].copy()).cuda()
        for count in (n, n * 2 // 3 + 5):
            print(f"[huffman] {count} of {n} symbols, {kind}", flush=True)
            batch = api.HuffmanBatch([d], n_device=[torch.tensor([count], dtype=torch.int64, device="cuda")])
            batch.out[0].fill_(0xEE)
            api.fh_huffman_encode_batch(batch)
            api.fh_huffman_decode_batch(batch)
            torch.cuda.synchronize()
            want, bits = oracle.huffman_encode(full[:count])
            assert batch.totals.cpu().tolist() == [[want.size, bits]]
            assert np.array_equal(batch.streams[0].cpu().numpy()[:want.size], want)
            back = batch.out[0].cpu().numpy()
            assert np.array_equal(back[:count], full[:count])
            assert np.all(back[-(-count // 16) * 16:] == 0xEE)
            if kind == "nearly flat" and count == limit:
                assert HS.passes(HS.offsets_of(want, count), 0, narrow, narrow, stage)[1:], "one pass is enough"


def test_rings_of_the_narrow_workgroups(api):
    """Symbols that are rare in the stream and stand together have codes of some 16 bits: 128 words per chunk, of which the
    stage of a workgroup of 512 threads holds a half of its 488 chunks.  Such passes go through the rings: a
    workgroup in the middle, and the last one with a ragged chunk.  Then codes of 24 bits, the longest there are."""
    shapes, seats = HS.decoder_shapes()
    (threads, stage), _ = shapes.items()
    n = 256 * seats * 256 - 37
    rng = np.random.default_rng(31)
    data = np.clip(np.rint(rng.normal(128, 2.5, n)), 0, 255).astype(np.uint8)
    for b in (100, 255):
        part = data[b * seats * 256: (b + 1) * seats * 256]
        part[:] = rng.integers(0, 256, part.size)
    want = _check(api, data, "noise in two workgroups")
    offsets = HS.offsets_of(want, n)
    for b in (0, 99, 100, 255):
        kinds = {staged for _, staged in HS.passes(offsets, b * seats, (b + 1) * seats, threads, stage)}
        assert kinds == {b not in (100, 255)}, f"workgroup {b}"
    n = 700 * 256 - 37                                        # three workgroups of 234 chunks
    data, stream = HS.long_codes(rng, n, [(234, 700)])
    offsets = HS.offsets_of(stream, n)
    assert [HS.passes(offsets, a, min(a + 234, 700), threads, stage)[0][1] for a in (0, 234, 468)] == [True, False, False]
    print("[huffman] codes of 24 bits", flush=True)
    back = api.fh_huffman_decode(torch.from_numpy(stream).cuda(), n)
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy(), data)


@pytest.mark.parametrize("kind", ["uniform", "one", "two", "geometric", "all-once", "ties"])
def test_distributions(api, kind):
    rng = np.random.default_rng(1)
    n = 300001
    data = {"uniform": lambda: rng.integers(0, 256, n),
            "one": lambda: np.full(n, 77),
            "two": lambda: rng.integers(0, 2, n) * 200 + 3,
            "geometric": lambda: rng.geometric(0.05, n) % 256,
            "all-once": lambda: np.arange(256),
            "ties": lambda: np.tile(np.arange(37), 1000)}[kind]().astype(np.uint8)
    _check(api, data, kind)


@pytest.mark.parametrize("used", [2, 3, 4, 63, 64, 65, 66, 127, 128, 129, 191, 255, 256])
@pytest.mark.parametrize("kind", ["equal", "pairs", "doubling", "alternating", "random"])
def test_code_construction_in_rounds(api, used, kind):
    """Histograms around the 64 nodes of either queue that a round of merges looks at: all counts equal (full windows,
    odd numbers of candidates), equal pairs, groups that double (leaves tie with nodes made of them), leaves that
    alternate with the nodes, and counts that rarely tie."""
    rng = np.random.default_rng(used)
    i = np.arange(used)
    counts = {"equal": np.full(used, 7), "pairs": 3 + i // 2, "doubling": 1 << (i * 12 // used),
              "alternating": 1 + i + (i % 3) * used // 2, "random": rng.integers(1, 4000, used)}[kind]
    symbols = rng.permutation(256)[:used].astype(np.uint8)
    _check(api, rng.permutation(np.repeat(symbols, counts)), f"{kind} counts of {used} symbols")


def test_codes_that_would_exceed_24_bits(api):
    fib = [1, 1]
    while len(fib) < 28:
        fib.append(fib[-1] + fib[-2])
    data = np.repeat(np.arange(10, 38, dtype=np.uint8), fib)          # a 27-deep comb: counts are halved
    rng = np.random.default_rng(2)
    rng.shuffle(data)
    assert _check(api, data, "comb").size < data.size


def test_index_stream_of_the_predictive_form_end_to_end(api):
    """sparse storage with an error bound -> Huffman on its code bytes -> back -> restored maps
    equal the oracle's, and the code bytes shrink."""
    maps, h, w, n, eps = 64, 56, 56, 4, 0.02
    x = W.salient_feature_maps(maps, h, w, seed=4, zero_level=0.0)
    b = api.fh_sparse_encode(torch.from_numpy(x).cuda(), maps, h, w, n, 0.3, eps=eps)
    torch.cuda.synchronize()
    nv, ni = (int(v) for v in b.totals.cpu().tolist()[:2])
    idx = b.indices[:ni].contiguous()
    stream, totals = api.fh_huffman_encode(idx)
    torch.cuda.synchronize()
    used = int(totals[0])
    want, _ = oracle.huffman_encode(idx.cpu().numpy())
    assert np.array_equal(stream.cpu().numpy()[:used], want)
    print(f"[huffman] index stream {ni} -> {used} bytes", flush=True)
    assert used < 0.9 * ni
    idx_back = api.fh_huffman_decode(stream[:used], ni)
    out = api.fh_sparse_decode(b.info, b.values[:nv], idx_back, maps, h, w, n, eps=eps)
    torch.cuda.synchronize()
    info, v, i, _ = oracle.sparse_encode(x, maps, h, w, n, 0.3, eps=eps)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), oracle.sparse_decode(info, v, i, maps, h, w, n, eps=eps).view(np.uint32))


def test_decoder_stays_inside_truncated_or_foreign_streams(api):
    rng = np.random.default_rng(3)
    data = np.clip(np.rint(rng.normal(128, 6, 200000)), 0, 255).astype(np.uint8)
    stream, totals = api.fh_huffman_encode(torch.from_numpy(data).cuda())
    torch.cuda.synchronize()
    used = int(totals[0])
    chunks = (data.size + 255) // 256
    header = 256 + 4 * (chunks + 1)
    # payload cut in half: the chunks that are still there come back exactly
    cut = header + ((used - header) // 8) * 4
    out = api.fh_huffman_decode(stream[:cut], data.size).cpu().numpy()
    torch.cuda.synchronize()
    assert np.array_equal(out[: data.size // 4], data[: data.size // 4]) and not np.array_equal(out, data)
    # random bytes as a stream (lengths, offsets and payload): must simply finish
    junk = torch.randint(0, 256, (used,), dtype=torch.uint8, device="cuda")
    out = api.fh_huffman_decode(junk, data.size)
    torch.cuda.synchronize()
    assert out.numel() == data.size
    # a stream too short to hold the lengths and the offsets is refused on the host
    with pytest.raises(api.FedHybridError):
        api.fh_huffman_decode(stream[: header - 4], data.size)


def test_buffers_can_be_reused_and_errors_reach_the_caller(api):
    a = (np.arange(100000) % 7).astype(np.uint8)
    b = (np.arange(50000) % 200).astype(np.uint8)
    out = torch.empty(api.huffman_stream_bytes(a.size), dtype=torch.uint8, device="cuda")
    tot = torch.zeros(2, dtype=torch.int64, device="cuda")
    ws = torch.empty(api.huffman_workspace_bytes(a.size), dtype=torch.uint8, device="cuda")
    for data in (a, b, a):
        api.fh_huffman_encode(torch.from_numpy(data).cuda(), stream_out=out, totals=tot, workspace=ws)
        torch.cuda.synchronize()
        want, bits = oracle.huffman_encode(data)
        assert tot.cpu().tolist() == [want.size, bits]
        assert np.array_equal(out.cpu().numpy()[: want.size], want)
    with pytest.raises(api.FedHybridError):
        api.fh_huffman_encode(torch.from_numpy(a).cuda(), stream_out=out[:1000], totals=tot, workspace=ws)
    with pytest.raises(api.FedHybridError):
        api.fh_huffman_encode(torch.from_numpy(a).cuda()[1:], stream_out=out, totals=tot, workspace=ws)   # misaligned


def test_batched_calls_match_the_oracle_for_every_stream(api, per_launch):
    """More streams than one launch holds, an empty one among them, sizes from one symbol to a few groups."""
    rng = np.random.default_rng(9)
    sizes = [1, 0, 300, 65536, 200001, 77] + [1000 + 4099 * (i % 14) + i for i in range(2 * per_launch + 1)]
    datas = []
    for i, n in enumerate(sizes):
        spread = 1.0 + (i % 5) * 3.0
        datas.append(np.clip(np.rint(rng.normal(128, spread, n)), 0, 255).astype(np.uint8))
    dev = [torch.from_numpy(d).cuda() if d.size else torch.empty(0, dtype=torch.uint8, device="cuda") for d in datas]
    batch = api.HuffmanBatch(dev)
    api.fh_huffman_encode_batch(batch)
    torch.cuda.synchronize()
    used = batch.refresh()
    api.fh_huffman_decode_batch(batch)
    torch.cuda.synchronize()
    totals = batch.totals.cpu().tolist()
    for i, d in enumerate(datas):
        want, bits = oracle.huffman_encode(d)
        assert totals[i] == [want.size, bits], f"stream {i}: totals"
        assert np.array_equal(batch.streams[i].cpu().numpy()[: used[i]], want), f"stream {i}: bytes"
        assert np.array_equal(batch.out[i].cpu().numpy(), d), f"stream {i}: decoded"


def test_symbol_count_taken_from_device_memory(api):
    """The buffer's length is the output of an earlier call on the stream: buffers and launches are
    sized for an upper bound, the count comes from device memory, and nothing is read back between
    encode and decode."""
    rng = np.random.default_rng(5)
    cap = 300_000
    full = np.clip(np.rint(rng.normal(128.0, 5.0, cap)), 0, 255).astype(np.uint8)
    counts = [0, 1, 255, 256, 257, 65_536, 65_537, 200_001, cap, cap + 999]        # the last: clipped to the bound
    data = [torch.from_numpy(full.copy()).cuda() for _ in counts]
    n_dev = [torch.tensor([c], dtype=torch.int64, device="cuda") for c in counts]
    batch = api.HuffmanBatch(data, n_device=n_dev)
    for o in batch.out:
        o.fill_(0xEE)
    torch.cuda.synchronize()
    api.fh_huffman_encode_batch(batch)
    api.fh_huffman_decode_batch(batch)                       # no refresh: stream capacities bound the reads
    torch.cuda.synchronize()
    totals = batch.totals.cpu().numpy()
    for k, c in enumerate(counts):
        n = min(c, cap)
        print(f"[huffman] device count {c} of capacity {cap}", flush=True)
        want, bits = oracle.huffman_encode(full[:n])
        assert (int(totals[k, 0]), int(totals[k, 1])) == (want.size, bits)
        assert np.array_equal(batch.streams[k].cpu().numpy()[:want.size], want)
        back = batch.out[k].cpu().numpy()
        assert np.array_equal(back[:n], full[:n])
        assert np.all(back[-(-n // 16) * 16:] == 0xEE)          # nothing written past the count's last 16-byte vector
