"""GPU parity of the re-verifying install (wm_commit_reverify) with the
oracle's: the verdict word and the installed state are equal, on the right
base (installed, equal to the source), on a base that differs in a chunk the
payload does not carry, on staging changed after verification, on a full
ship, with a short last chunk, and on the production-size active step."""
import numpy as np
import pytest
import torch

import oracle
import wm_inputs
from gpu_helpers import ORACLE_THREADS, host_bytes, say

pytestmark = pytest.mark.gpu

CH = 65536


@pytest.fixture(scope="module")
def wm():
    from paper_2607_10389_amd import _wm
    _wm.init(-1)
    return _wm


def _pair(seed, n_bytes, dirty):
    g = torch.Generator(device="cuda").manual_seed(seed)
    prev = torch.randint(0, 256, (n_bytes,), generator=g, device="cuda",
                         dtype=torch.int32).to(torch.uint8)
    cur = prev.clone()
    for c in dirty:
        lo, hi = c * CH, min((c + 1) * CH, n_bytes)
        cur[lo:hi] = torch.randint(0, 256, (hi - lo,), generator=g, device="cuda",
                                   dtype=torch.int32).to(torch.uint8)
    return prev, cur


def _check(m, live, kind, want_status, label):
    """Run the GPU install and the oracle's on the same bytes."""
    from paper_2607_10389_amd import _wm
    pb = int(m.payload_bytes.item())
    payload = m.payload[:pb].cpu().numpy()
    staging = m.staging.cpu().numpy()
    v0 = int(m.verdict.item())
    host_live = host_bytes(live).copy()
    v_orc = oracle.commit_reverify(kind, host_live, CH, staging, payload, v0)
    st = m.commit_reverify(live)
    torch.cuda.synchronize()
    assert st == want_status, (label, st)
    assert int(m.verdict.item()) == v_orc, (label, int(m.verdict.item()), v_orc)
    assert np.array_equal(host_bytes(live), host_live), label


@pytest.mark.parametrize("kind", [0, 1])
def test_reverify_dirty_ship(wm, kind):
    from paper_2607_10389_amd import Mover
    n = 6 * CH + 1000  # chunk 6 is a 1,000-byte tail
    prev, cur = _pair(11 + kind, n, [1, 4, 6])
    m = Mover(n, kind)
    m.encode_step(cur, prev)
    m.decode()
    torch.cuda.synchronize()
    assert m.dirty_host().tolist() == [1, 4, 6]
    # the right base: installed, bit-identical to the source
    live = prev.clone()
    _check(m, live, kind, wm.WM_OK, "right base")
    assert torch.equal(live, cur)
    # a base differing in a clean chunk: refused, live untouched
    live = prev.clone()
    live[2 * CH + 7] ^= 1
    before = live.clone()
    _check(m, live, kind, wm.WM_VERIFY_FAILED, "other base")
    assert torch.equal(live, before)
    assert int(m.verdict.item()) == wm.V_REVERIFY
    # staging changed after verification: refused
    m.verdict.zero_()
    m.staging[CH + 5] ^= 0x80
    live = prev.clone()
    _check(m, live, kind, wm.WM_VERIFY_FAILED, "stale staging")
    assert torch.equal(live, prev)
    # a failed verification passes through: nothing installed
    m.verdict.fill_(wm.V_DATA)
    live = prev.clone()
    st = m.commit_reverify(live)
    assert st == wm.WM_VERIFY_FAILED and int(m.verdict.item()) == wm.V_DATA
    assert torch.equal(live, prev)


def test_reverify_full_ship_and_empty_dirty_set(wm):
    from paper_2607_10389_amd import Mover
    state = wm_inputs.make_cache(wm_inputs.TINY, "cuda")
    n = state.numel() * 2
    m = Mover(n)
    m.encode_step(state, None)
    m.decode()
    live = torch.zeros(n, dtype=torch.uint8, device="cuda")
    _check(m, live, 0, wm.WM_OK, "full ship")
    assert torch.equal(live, state.view(-1).view(torch.uint8))
    # no dirty chunk: installs nothing, and succeeds only on the right base
    m.encode_step(state, state)
    m.decode()
    torch.cuda.synchronize()
    assert int(m.n_dirty.item()) == 0
    live = state.view(-1).view(torch.uint8).clone()
    _check(m, live, 0, wm.WM_OK, "empty, right base")
    live[5] ^= 2
    _check(m, live, 0, wm.WM_VERIFY_FAILED, "empty, other base")


def test_reverify_production_step(wm):
    from paper_2607_10389_amd import Mover
    prev = wm_inputs.make_cache(wm_inputs.PRODUCTION, "cuda")
    cur, ids = wm_inputs.production_step(prev)
    n = prev.numel() * 2
    say(f"[reverify] production step, {ids.numel()} dirty chunks")
    m = Mover(n)
    m.encode_step(cur, prev)
    m.decode()
    live = prev.view(-1).view(torch.uint8).clone()
    assert m.commit_reverify(live) == wm.WM_OK
    assert torch.equal(live, cur.view(-1).view(torch.uint8))
    live = prev.view(-1).view(torch.uint8).clone()
    clean = int(np.setdiff1d(np.arange(n // CH), ids.cpu().numpy())[17])
    live[clean * CH + 100] ^= 1
    before = live.clone()
    assert m.commit_reverify(live) == wm.WM_VERIFY_FAILED
    assert int(m.verdict.item()) == wm.V_REVERIFY
    assert torch.equal(live, before)


@pytest.mark.parametrize("n_chunks,dirty", [
    (1, []), (1, [0]), (40, [0]), (40, [39]), (40, list(range(0, 40, 2))), (40, list(range(40))),
    (70, [5, 6, 7, 68]), (1500, [0, 3, 9, 700, 1499]), (1500, list(range(0, 1500, 6))),
    (1500, list(range(1, 1500)))])
def test_reverify_reads_the_chunks_that_stay(wm, n_chunks, dirty):
    """Gaps of every kind between the installed records (none, short, longer
    than a wave, the ends): a flipped byte in any chunk that stays is seen,
    one in a chunk that is overwritten does not matter."""
    from paper_2607_10389_amd import Mover
    n = (n_chunks - 1) * CH + 4098
    prev, cur = _pair(n_chunks + len(dirty), n, dirty)
    m = Mover(n)
    m.encode_step(cur, prev)
    m.decode()
    torch.cuda.synchronize()
    assert m.dirty_host().tolist() == dirty
    live = prev.clone()
    for c in dirty:
        live[c * CH + 77] ^= 4
    _check(m, live, 0, wm.WM_OK, "overwritten chunks differ")
    assert torch.equal(live, cur)
    stay = sorted(set(range(n_chunks)) - set(dirty))
    for c in sorted(set(stay[:2] + stay[len(stay) // 2:][:1] + stay[-2:])):
        m.verdict.zero_()
        live = prev.clone()
        live[min(c * CH + CH - 1, n - 1)] ^= 1
        before = live.clone()
        _check(m, live, 0, wm.WM_VERIFY_FAILED, f"chunk {c}")
        assert torch.equal(live, before)
    if len(dirty) > 2:  # the table changed after the verdict, out of order
        m.verdict.zero_()
        at = int(m.payload_bytes.item()) - 16 * len(dirty)
        t = m.payload[at:at + 32].clone()
        m.payload[at:at + 16], m.payload[at + 16:at + 32] = t[16:], t[:16]
        live = prev.clone()
        _check(m, live, 0, wm.WM_VERIFY_FAILED, "table out of order")
        assert torch.equal(live, prev)


def _step(n_chunks, stay, kind=0):
    """A decoded step that ships every chunk but `stay`, its last one short."""
    from paper_2607_10389_amd import Mover
    n = (n_chunks - 1) * CH + 4098
    dirty = sorted(set(range(n_chunks)) - set(stay))
    prev, cur = _pair(n_chunks + len(stay), n, [])
    for c in dirty:
        cur[c * CH + 9] ^= 1
    m = Mover(n, kind)
    m.encode_step(cur, prev)
    m.decode()
    torch.cuda.synchronize()
    assert m.dirty_host().tolist() == dirty
    return m, prev, cur, dirty


def _written_words(m, live):
    """Workspace words that a re-verifying install of `live` changes."""
    m.ws_dst.fill_(0xA5)
    st = m.commit_reverify(live)
    torch.cuda.synchronize()
    words = m.ws_dst[:m.ws_dst.numel() // 4 * 4].view(-1, 4)
    return st, int((words != 0xA5).any(1).sum())


@pytest.mark.parametrize("n_chunks,records", [(1500, 1), (1500, 1400), (2400, 2248)])
def test_reverify_of_few_records_makes_no_list(wm, n_chunks, records):
    """Below the line where a list of the chunks that stay pays, an install
    writes the CRC of every chunk and staged record and the control words,
    and no list."""
    m, prev, cur, dirty = _step(n_chunks, range(n_chunks - records))
    st, words = _written_words(m, prev.clone())
    assert st == wm.WM_OK
    assert words <= n_chunks + records + 16, words


# 2,400 chunks: a list from 2,249 records on
@pytest.mark.parametrize("kind,stay", [
    (0, list(range(151))),                       # 2,249 records, one long gap
    (1, list(range(1, 302, 2))),                 # short gaps
    (0, [0, 5, 6] + list(range(1000, 1100)) + [2399]),
    (1, list(range(2249, 2399)) + [7, 9]),       # 2,248: no list
    (0, [])])
def test_reverify_on_both_sides_of_the_list(wm, kind, stay):
    """The right base installs, a byte flipped in a chunk that stays is
    refused.  Where the table has changed since it was verified (two entries
    and their staged records swapped: every record still matches its receipt)
    the outcome depends on the chunks that were checksummed, and equals the
    oracle's."""
    m, prev, cur, dirty = _step(2400, stay, kind)
    n = prev.numel()

    def check(want, label, flip=None):
        m.verdict.zero_()
        live = prev.clone()
        if flip is not None:
            live[min(flip * CH + CH - 1, n - 1)] ^= 1
        before = live.clone()
        _check(m, live, kind, want, label)
        assert torch.equal(live, cur if want == wm.WM_OK else before), label

    check(wm.WM_OK, "right base")
    for c in sorted({stay[0], stay[len(stay) // 2], stay[-1]}) if stay else []:
        check(wm.WM_VERIFY_FAILED, f"chunk {c}", c)
    at = int(m.payload_bytes.item()) - 16 * len(dirty)
    for buf, a, b in ((m.payload, at + 16, 16), (m.staging, CH, CH)):
        t = buf[a - b:a].clone()
        buf[a - b:a] = buf[a:a + b]
        buf[a:a + b] = t
    check(wm.WM_OK, "two records swapped")
    if stay:
        check(wm.WM_VERIFY_FAILED, "two records swapped, another base", stay[-1])
