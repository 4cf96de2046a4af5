"""GPU parity of formats v2 and v3 (codec 2: per-chunk canonical Huffman
codes of the exponent plane in 512 streams; codec 3: the same of the high
byte plane, the bf16 byte-plane split) against the oracle: payload bytes,
decoded bytes, verdict words and record status are equal (tolerance 0) on
the tiny cache, dirty lists, edge-case states, flipped bits and the
production-size cache."""
import numpy as np
import pytest
import torch

import oracle
import wm_inputs

from gpu_helpers import ORACLE_THREADS, host_bytes, random_bytes, say, u32

pytestmark = pytest.mark.gpu

CH = 65536


@pytest.fixture(scope="module")
def wm():
    from paper_2607_10389_amd import _wm
    _wm.init(-1)
    return _wm


@pytest.fixture(params=[2, 3], ids=["v2", "v3"])
def codec(request):
    return request.param


def mover(nbytes, kind=0, codec=2):
    from paper_2607_10389_amd import Mover
    return Mover(nbytes, kind, codec=codec)


def dev(a: np.ndarray) -> torch.Tensor:
    t = torch.empty(max(a.size, 16), dtype=torch.uint8, device="cuda")
    t[: a.size] = torch.from_numpy(a).cuda()
    return t


def ship(wm, state_h: np.ndarray, kind=0, label="", codec=2):
    """Full v2 ship of a host state through the GPU; checks payload, decode
    and verdict against the oracle.  Returns the payload."""
    st = dev(state_h)
    m = mover(state_h.size, kind, codec)
    m.encode(st, with_crc=False)
    torch.cuda.synchronize()
    got = m.payload_host()
    want = oracle.encode(kind, state_h, CH, None, ORACLE_THREADS, codec=codec)
    assert got.size == want.size, (label, got.size, want.size)
    if not np.array_equal(got, want):
        bad = np.nonzero(got != want)[0]
        raise AssertionError(f"{label}: {bad.size} payload bytes differ, first {bad[:8].tolist()}")
    m.decode()
    assert m.commit(None, scatter=False) == wm.WM_OK, label
    torch.cuda.synchronize()
    assert np.array_equal(m.staging[: state_h.size].cpu().numpy(), state_h), label
    return got, m


@pytest.mark.parametrize("kind", [0, 1])
def test_tiny_full_ship(wm, kind, codec):
    state = host_bytes(wm_inputs.make_cache(wm_inputs.TINY))
    got, _ = ship(wm, state, kind, f"tiny kind={kind}", codec)
    say(f"[v{codec}] tiny ratio {got.size / state.size:.4f}")


def _edge_states():
    rng = np.random.default_rng(7)
    n = 3 * CH // 2
    out = {}
    out["constant"] = np.full(n, 0x3F80, np.uint16).view(np.uint8)
    out["random_bits"] = rng.integers(0, 1 << 16, n, dtype=np.uint16).view(np.uint8)
    out["all_patterns"] = np.arange(1 << 16, dtype=np.uint16).view(np.uint8).copy()
    sp = np.array([0x0000, 0x8000, 0x7F80, 0xFF80, 0x7FC1, 0x0001, 0x8001, 0x3F80], np.uint16)
    out["special"] = sp[rng.integers(0, sp.size, n)].view(np.uint8)
    t = (rng.standard_t(3, n) * 10).astype(np.float32)
    out["student_t"] = (t.view(np.uint32) >> 16).astype(np.uint16).view(np.uint8)
    x = (rng.standard_normal(n) * 2).astype(np.float32)
    bf = (x.view(np.uint32) >> 16).astype(np.uint16).view(np.uint8)
    out["tail_5536"] = bf[: 2 * CH + 5536].copy()
    out["tail_4098"] = bf[: 2 * CH + 4098].copy()  # a row piece straddles the end
    out["one_word_tail"] = bf[: CH + 2].copy()
    out["two_exponents"] = np.where(rng.random(n) < 0.9, 0x3F80, 0x4000).astype(np.uint16).view(np.uint8)
    # more than 64 distinct exponents in a chunk that still codes as HUF (the
    # plan's code construction past one wave's 64 lanes, and the length cap)
    for scale in (6, 20):
        e = np.clip(127 + np.round(rng.laplace(0, scale, n)), 0, 255).astype(np.int64)
        sm = rng.integers(0, 256, n)
        w = (((sm >> 7) << 15) | (e << 7) | (sm & 127)).astype(np.uint16)
        out[f"laplace_{scale}"] = w.view(np.uint8)
    # exactly 64 and 65 distinct exponents in every chunk, with geometric
    # counts (codes past the length cap, several capping passes): the two
    # sides of the 64-symbol limit of the register-resident construction
    rng2 = np.random.default_rng(11)
    for m_sym in (64, 65):
        g = np.minimum(rng2.geometric(0.12, n) - 1, m_sym - 1)
        for cw in range(0, n, CH // 2):
            g[cw:cw + m_sym] = np.arange(m_sym)
        e = 60 + g
        sm = rng2.integers(0, 256, n)
        w = (((sm >> 7) << 15) | (e << 7) | (sm & 127)).astype(np.uint16)
        out[f"exact_{m_sym}_exponents"] = w.view(np.uint8)
    return out


@pytest.mark.parametrize("scale,min_distinct", [(6, 100), (20, 240)])
def test_wide_alphabet_states_plan_huf(scale, min_distinct):
    """The wide-alphabet edge states really have more than 64 symbols per
    chunk and plan HUF (so the GPU test of them exercises that path)."""
    state = _edge_states()[f"laplace_{scale}"]
    for c in range(0, state.size, CH):
        ch = state[c:c + CH]
        e = (ch.view(np.uint16) >> 7) & 255
        assert np.unique(e).size >= min_distinct
        plan = oracle.plan_chunk_v2(ch)
        assert plan["mode"] == 2 and plan["k"] == 11, plan


@pytest.mark.parametrize("m_sym", [64, 65])
def test_boundary_alphabet_states_plan_huf(m_sym):
    """The boundary states have exactly 64 or 65 exponents in every chunk
    and plan HUF at the length cap (so their GPU test exercises both sides
    of the 64-symbol limit, with capping passes)."""
    state = _edge_states()[f"exact_{m_sym}_exponents"]
    for c in range(0, state.size, CH):
        ch = state[c:c + CH]
        assert np.unique((ch.view(np.uint16) >> 7) & 255).size == m_sym
        plan = oracle.plan_chunk_v2(ch)
        assert plan["mode"] == 2 and plan["k"] == 11, plan


@pytest.mark.parametrize("name", list(_edge_states().keys()))
def test_edge_cases(wm, name, codec):
    state = _edge_states()[name]
    got, _ = ship(wm, state, 0, name, codec)
    modes = got[64]
    say(f"[v{codec}] {name}: {state.size} B -> {got.size} B, first record mode {modes}")


def test_empty_state(wm, codec):
    m = mover(0, 0, codec)
    state = torch.zeros(16, dtype=torch.uint8, device="cuda")
    m.encode(state, with_crc=False)
    torch.cuda.synchronize()
    want = oracle.encode(0, np.zeros(0, np.uint8), CH, None, 1, codec=codec)
    assert np.array_equal(m.payload_host(), want)
    m.decode()
    assert m.commit(None, scatter=False) == wm.WM_OK


def test_dirty_list(wm, codec):
    prev, cur, ids = wm_inputs.tiny_step("cuda")
    h = host_bytes(cur)
    m = mover(h.size, 0, codec)
    m.checksum(cur)
    m.diff(cur, prev)
    m.encode(cur, dirty_only=True)
    torch.cuda.synchronize()
    idx = m.dirty_host()
    want = oracle.encode(0, h, CH, idx, ORACLE_THREADS, codec=codec)
    assert np.array_equal(m.payload_host(), want)
    live = prev.clone().view(-1).view(torch.uint8)
    m.decode()
    assert m.commit(live, scatter=True) == wm.WM_OK
    torch.cuda.synchronize()
    assert torch.equal(live, cur.view(-1).view(torch.uint8))


def test_bit_flips_match_oracle(wm, codec):
    state = _edge_states()["tail_4098"]
    good, m = ship(wm, state, 0, "flips", codec)
    n_rec = int(good[24:28].view(np.uint32)[0])
    total = int(good[32:40].view(np.uint64)[0])
    table = total - 16 * n_rec
    rng = np.random.default_rng(11)
    # header, table, every record's header, tables, streams and planes
    positions = [3, 30, 45, 61, table + 5, table + 16 * (n_rec - 1) + 9]
    positions += list(rng.integers(64, table, 40))
    for pos in positions:
        for bit in (0, 5):
            bad = good.copy()
            bad[pos] ^= 1 << bit
            m.payload[: bad.size] = torch.from_numpy(bad).cuda()
            m.decode()
            torch.cuda.synchronize()
            v = int(m.verdict.item())
            v_o, _, rs_o = oracle.decode_verify(0, bad, state.size, CH, m.staging.numel(),
                                                ORACLE_THREADS, codec=codec)
            assert v == v_o and v != 0, (pos, bit, v, v_o)
            if v_o & 3 == 0:
                assert np.array_equal(u32(m.rec_status)[:n_rec], rs_o[:n_rec]), (pos, bit)


def test_production_full_ship(wm, codec):
    state = wm_inputs.make_cache(wm_inputs.PRODUCTION, "cuda")
    nbytes = state.numel() * 2
    m = mover(nbytes, 0, codec)
    m.checksum(state)
    m.encode(state)
    torch.cuda.synchronize()
    got = m.payload_host()
    h = host_bytes(state)
    want = oracle.encode(0, h, CH, None, ORACLE_THREADS, codec=codec)
    assert got.size == want.size
    if not np.array_equal(got, want):
        bad = np.nonzero(got != want)[0]
        raise AssertionError(f"{bad.size} bytes differ, first {bad[:8].tolist()}")
    say(f"[v{codec}] production ratio {got.size / nbytes:.5f}")
    del want, h
    m.decode()
    assert m.commit(None, scatter=False) == wm.WM_OK
    torch.cuda.synchronize()
    assert torch.equal(m.staging[:nbytes], state.view(-1).view(torch.uint8))


def test_huf_record_longer_than_raw_is_rejected(wm, codec):
    from test_oracle_codec_v2 import _huf_payload
    from test_oracle_codec_v3 import _payload
    rng = np.random.default_rng(13)
    st = rng.integers(0, 1 << 16, 3000, dtype=np.uint16).view(np.uint8)
    p = np.frombuffer(_huf_payload(st) if codec == 2 else _payload(st, True), np.uint8)
    m = mover(st.size, 0, codec)
    m.payload[: p.size] = torch.from_numpy(p.copy()).cuda()
    m.decode()
    torch.cuda.synchronize()
    assert int(m.verdict.item()) == 4
    assert int(u32(m.rec_status)[0]) == 4


@pytest.mark.parametrize("kind", [0, 1])
def test_v2_encode_step(wm, kind, codec):
    """Format v2 through the fused call: full ship and the tiny 75%-dirty
    step give the oracle's CRCs, global CRC, dirty list and payload, and the
    step's scatter install leaves live equal to the source."""
    prev, cur, ids = wm_inputs.tiny_step("cuda")
    hc, hp = host_bytes(cur), host_bytes(prev)
    n = hc.size
    m = mover(n, kind, codec)
    m.encode_step(cur, None)
    torch.cuda.synchronize()
    assert np.array_equal(m.payload_host(), oracle.encode(kind, hc, CH, None, 1, codec=codec))
    assert np.array_equal(m.dirty_host(), np.arange(n // CH, dtype=np.uint32))
    crcs, g = oracle.checksum_chunks(kind, hc, CH)
    assert np.array_equal(m.crc_host(), crcs)
    assert int(u32(m.global_crc)[0]) == g
    m.encode_step(cur, prev)
    torch.cuda.synchronize()
    idx = oracle.diff_dirty(hc, hp, CH)
    assert np.array_equal(m.dirty_host(), idx)
    assert np.array_equal(m.crc_host(), crcs)
    assert np.array_equal(m.payload_host(), oracle.encode(kind, hc, CH, idx, 1, codec=codec))
    live = prev.clone()
    m.decode()
    assert m.commit(live, scatter=True) == wm.WM_OK
    assert torch.equal(live, cur)
    # no dirty_idx, n_dirty or crc_out from the caller: the workspace holds them
    m2 = mover(n, kind, codec)
    wm.encode_step(cur, prev, n, m2.p, None, None, None, None, m2.payload, m2.payload_bytes,
                   m2.ws_src)
    torch.cuda.synchronize()
    assert np.array_equal(m2.payload_host(), m.payload_host())


@pytest.mark.parametrize("batch", [0, 200_000, 1 << 40])
def test_v2_pipelined_receive(wm, batch, codec):
    """Format v2 received in record batches: verdict, record status and
    staging equal the oracle's decode of the same bytes, also with a flipped
    bit in a record and in the table."""
    prev, cur, _ = wm_inputs.tiny_step("cuda")
    hc, hp = host_bytes(cur), host_bytes(prev)
    idx = oracle.diff_dirty(hc, hp, CH)
    good = oracle.encode(0, hc, CH, idx, 1, codec=codec)
    n = hc.size
    m = mover(n, 0, codec)
    for label, flip in (("clean", None), ("record", 64 + 300), ("table", good.size - 20)):
        bad = good.copy()
        if flip is not None:
            bad[flip] ^= 0x10
        host = torch.empty(bad.size, dtype=torch.uint8, pin_memory=True)
        host[:] = torch.from_numpy(bad)
        cs = torch.cuda.Stream()
        m.payload.fill_(0xA7)
        torch.cuda.synchronize()
        m.receive(host, bad.size, batch, cs)
        torch.cuda.synchronize()
        v = int(m.verdict.item())
        v_o, st_o, rs_o = oracle.decode_verify(0, bad, n, CH, m.staging.numel(), 1, codec=codec)
        assert v == v_o, (label, v, v_o)
        if v_o & 3 == 0:
            k = idx.size
            assert np.array_equal(u32(m.rec_status)[:k], rs_o[:k]), label
        if v_o == 0:
            got = m.staging[: idx.size * CH].cpu().numpy()
            assert np.array_equal(got, st_o[: idx.size * CH]), label
        else:
            assert flip is not None


def test_v2_precopy_rounds(wm, codec):
    """Pre-copy rounds in format v2: each round's dirty list and payload
    equal the oracle's, and the destination ends equal to the source."""
    spec = wm_inputs.TINY
    cur = wm_inputs.make_cache(spec, "cuda")
    n = spec.nbytes
    shipped = torch.zeros(n, dtype=torch.uint8, device="cuda")
    dest = torch.zeros_like(shipped)
    m = mover(n, 0, codec)
    for k in range(4):
        cur_h, shp_h = host_bytes(cur), shipped.cpu().numpy()
        st, nd = m.precopy_round(cur, shipped, dest)
        assert st == wm.WM_OK, k
        got = m.dirty_host()
        assert np.array_equal(got, oracle.diff_dirty(cur_h, shp_h, CH)), k
        assert np.array_equal(m.payload_host(), oracle.encode(0, cur_h, CH, got, 1, codec=codec)), k
        crcs, g = oracle.checksum_chunks(0, cur_h, CH)
        assert np.array_equal(m.crc_host(), crcs), k
        assert torch.equal(dest, shipped)
        writes = wm_inputs.chunk_writes(n // CH, 9, seed=70 + k, device="cuda")
        wm_inputs.rewrite_chunks(cur, spec, writes, seed=80 + k)
    st, nd = m.precopy_round(cur, shipped, dest)
    assert st == wm.WM_OK
    assert torch.equal(dest, cur.view(-1).view(torch.uint8))


@pytest.mark.parametrize("symbols", [90, 108, 128, 200])
def test_wide_streams(wm, codec, symbols):
    """Plane A uniform over `symbols` values: streams on either side of what
    the decoder's stage holds (54 bytes each) and of the RAW limit."""
    rng = np.random.default_rng(symbols)
    n = 4 * CH // 2 + 2000
    a = rng.integers(20, 20 + symbols, n)
    b = rng.integers(0, 256, n)
    w = (a << 8 | b) if codec == 3 else ((b >> 7) << 15 | a << 7 | (b & 127))
    ship(wm, w.astype(np.uint16).view(np.uint8), 0, f"{symbols} symbols", codec)


@pytest.mark.parametrize("records", [1, 255, 257, 4095, 4097])
def test_record_per_wave_counts(wm, codec, records):
    """Record counts around the CU count and the waves of the whole grid; the
    last record short."""
    n = records * CH - 2 * (records % 1000)
    say(f"[v{codec}] {records} records, {n} bytes")
    spec = wm_inputs.CacheSpec("waves", (1, 2, 1, -(-n // 512), 128), seed=records)
    state = host_bytes(wm_inputs.make_cache(spec, "cuda"))[:n].copy()
    ship(wm, state, 1, f"{records} records", codec)


@pytest.mark.parametrize("chunks", [1, 3, 511, 513, 1100])
@pytest.mark.parametrize("tail", [2, 14, 18, 1024, 65534, 65536])
def test_step_scan_dirty_list_and_crcs(wm, chunks, tail):
    """The dirty list and the CRCs of a format v2 step (one pass over both
    states) where one byte differs: the first or last of a chunk, or any of
    a lane's row edges, over less and more than the grid's chunks."""
    n = (chunks - 1) * 65536 + tail
    gen = torch.Generator(device="cuda").manual_seed(chunks + tail)
    prev = torch.randint(0, 256, (n,), generator=gen, device="cuda", dtype=torch.uint8)
    cur = prev.clone()
    spots = [0, 65535, 1023, 1024, 8191, 8192, 40961]
    for i, c in enumerate(range(0, chunks, 5)):
        at = c * 65536 + spots[i % len(spots)]
        cur[min(at, n - 1)] ^= 0x80
    cur[n - 1] ^= 1  # the tail's last byte
    m = mover(n, kind=chunks & 1)
    m.encode_step(cur, prev)
    torch.cuda.synchronize()
    hc, hp = cur.cpu().numpy(), prev.cpu().numpy()
    crcs, g = oracle.checksum_chunks(chunks & 1, hc)
    assert np.array_equal(m.crc_host(), crcs)
    assert int(m.global_crc.cpu().numpy().view("uint32")[0]) == g
    assert np.array_equal(m.dirty_host(), oracle.diff_dirty(hc, hp))


@pytest.mark.parametrize("order", ["first", "last", "alternate"])
def test_uneven_groups(wm, codec, order):
    """Chunks whose eight groups of 64 streams differ most in length: most at
    one bit a word, others at eight to ten (their streams pass the
    decoder's stage), at the record's start, at its end and by turns."""
    rng = np.random.default_rng(5)
    wide = {"first": [0], "last": [7], "alternate": [1, 4, 6]}[order]
    chunks = []
    for c in range(3):
        a = np.where(rng.random(CH // 2) < 0.97, 60, 61)
        for q in wide:
            a[4096 * q:4096 * (q + 1)] = 70 + rng.integers(0, 120, 4096)
        b = rng.integers(0, 256, CH // 2)
        chunks.append((a << 8 | b) if codec == 3 else ((b >> 7) << 15 | a << 7 | (b & 127)))
    state = np.concatenate(chunks)[: 5 * CH // 4 + 3000].astype(np.uint16).view(np.uint8)
    for kind in (0, 1):
        got, _ = ship(wm, state, kind, f"uneven groups {order}", codec)
        assert got[64] == 2  # the first record is Huffman-coded


def test_wide_streams_take_the_staged_path(wm, codec):
    """Records whose groups fill the decoder's stage almost to its end (62
    bytes a stream) decode about as fast as narrower ones: 7.2 bits a word
    carry a third more stream bytes than 5.4, and took twice the time where
    the stage was too small for them."""
    n = 6144 * CH
    gen = torch.Generator(device="cuda").manual_seed(3)
    best = {}
    for symbols in (40, 150):
        state = torch.empty(n, dtype=torch.uint8, device="cuda")
        w = state.view(torch.int16)
        for s in range(0, n // 2, 1 << 25):
            m = min(1 << 25, n // 2 - s)
            a = torch.randint(20, 20 + symbols, (m,), generator=gen, device="cuda",
                              dtype=torch.int32)
            b = torch.randint(0, 256, (m,), generator=gen, device="cuda", dtype=torch.int32)
            w[s:s + m] = ((a << 8 | b) if codec == 3
                          else ((b >> 7) << 15 | a << 7 | (b & 127))).to(torch.int16)
        m = mover(n, codec=codec)
        m.encode(state, with_crc=False)
        times = []
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda._sleep(1_000_000)  # the host's launches lie behind it
            e[0].record()
            m.decode()
            e[1].record()
            torch.cuda.synchronize()
            times.append(e[0].elapsed_time(e[1]))
        assert int(m.verdict.item()) == 0
        assert torch.equal(m.staging[:n], state)
        best[symbols] = min(times)
    say(f"[v{codec}] decode of {n} bytes: 40 symbols {best[40]:.3f} ms, 150 {best[150]:.3f} ms")
    assert best[150] < 1.5 * best[40]


@pytest.mark.parametrize("records", [2, 256, 512, 513, 1025, 3841])
def test_record_counts_at_launch_shapes(wm, codec, records):
    """Record counts on both sides of another wave per workgroup; the last
    record short."""
    n = records * CH - 2 * (records % 1000)
    spec = wm_inputs.CacheSpec("shapes", (1, 2, 1, -(-n // 512), 128), seed=records)
    state = host_bytes(wm_inputs.make_cache(spec, "cuda"))[:n].copy()
    ship(wm, state, 0, f"{records} records", codec)


def test_v2_rounds_keep_the_crcs_of_what_was_compared(wm, codec):
    """While another stream writes single bytes of the source, a round that
    succeeds leaves the CRCs of what the destination now holds: a chunk
    changed after it was found clean keeps the CRC of the bytes that were
    compared (it is dirty in the next round)."""
    chunks, batches, per = 2048, 400, 4
    gen = torch.Generator(device="cuda").manual_seed(9)
    cur = torch.randint(0, 256, (chunks * CH,), generator=gen, device="cuda", dtype=torch.uint8)
    shipped, dest = cur.clone(), cur.clone()
    m = mover(cur.numel(), 0, codec)
    st, nd = m.precopy_round(cur, shipped, dest)  # the kept CRCs
    assert st == wm.WM_OK and nd == 0
    at = torch.randperm(chunks, generator=gen, device="cuda")[:batches * per].view(batches, per)
    at = at * CH + torch.randint(0, CH, (batches, per), generator=gen, device="cuda")
    value = cur[at] ^ 1
    writer = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(writer):
        torch.cuda._sleep(20_000_000)  # the writes' launches lie behind it
        for b in range(batches):
            cur.index_copy_(0, at[b], value[b])
    kept = []
    while not writer.query() and len(kept) < 24:
        st, nd = m.precopy_round(cur, shipped, dest)
        if st == wm.WM_OK and nd:  # (rounds that end before the writes begin hold nothing)
            kept.append((shipped.clone(), m.crc.clone(), nd))
    writer.synchronize()
    assert kept, "no round ran while the source was written"
    for state, crc, nd in kept:
        want, _ = oracle.checksum_chunks(0, host_bytes(state), CH, ORACLE_THREADS)
        bad = np.nonzero(u32(crc)[:chunks] != want)[0]
        assert bad.size == 0, (len(kept), nd, bad[:8].tolist())
    say(f"[v{codec}] rounds beside the writer: {[k[2] for k in kept]} dirty")
    while nd:
        st, nd = m.precopy_round(cur, shipped, dest)
        assert st == wm.WM_OK
    assert torch.equal(dest, cur) and torch.equal(shipped, cur)
