"""GPU: the cut alone (Sec. 3.1; the ranking of Sec. 3.2) on crafted cache states.

Scores, positions and K/V rows are written straight into the cache, the
context is rebuilt on that state (bm_resume) and bm_evict_compact runs the
select and the compaction.  The sum rule ranks by the stored float itself, so
the oracle's float64 order is exactly the device's and kept sets must agree
entry for entry, with no near-tie allowance.

The score patterns put the decision in every digit of the 64-bit key: the
evicted and the kept entries part in the first, second, third or fourth byte
of the float; all scores equal (the positions decide); a few tied values with
the cut inside a tie; uniform and log-spread values with exact zeros.
Positions reach past 2^16, so three position digits can take part.  Cache
sizes cover the four select instantiations (3, 4 and 16 keys per thread, and
the streaming form above 4096 entries), with 1 to 1024 entries removed.
The paper's own rule (the average) is checked the same way on scores built so
that every quotient is exact.
"""
import numpy as np
import pytest
import torch

from oracle import pd as opd
from paper_2412_05693_amd.batchmax import PDAttention

pytestmark = pytest.mark.gpu

HEAD_DIM = 64
CURR_ID = 70_000


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _bits(lo, hi, size, rng):
    """float32 values whose bit patterns are drawn from [lo, hi)."""
    return rng.integers(lo, hi, size=size, dtype=np.uint64).astype(np.uint32).view(np.float32)


def _scores(kind, n, e, rng):
    """n float32 scores of which the e smallest (ties by position) are the cut."""
    kept = n - e
    if kind == "byte0":      # [1, 2) against [2, 8): top byte 0x3f against 0x40
        ev, kp = rng.uniform(1, 2, e), rng.uniform(2, 8, kept)
    elif kind == "byte1":    # 0x4000xxxx against 0x4020xxxx and up
        ev, kp = _bits(0x40000000, 0x40010000, e, rng), _bits(0x40200000, 0x40800000, kept, rng)
    elif kind == "byte2":    # 0x400000xx against 0x400080xx and up
        ev, kp = _bits(0x40000000, 0x40000100, e, rng), _bits(0x40008000, 0x40010000, kept, rng)
    elif kind == "byte3":    # last byte below 0x40 against at or above it (many float ties)
        ev, kp = _bits(0x40000000, 0x40000040, e, rng), _bits(0x40000040, 0x40000100, kept, rng)
    elif kind == "equal":    # one value: the positions alone decide
        return np.full(n, 1.0, dtype=np.float32)
    elif kind == "ties":     # zeros, then a tie group that the cut splits, then ones
        z = e // 2
        half = min(n - z, e - z + max(1, kept // 2))
        out = np.concatenate([np.zeros(z), np.full(half, 0.5), np.ones(n - z - half)])
        return rng.permutation(out).astype(np.float32)
    elif kind == "uniform":  # [0, 1) with exact zeros
        x = rng.uniform(0, 1, n)
        x[rng.random(n) < 0.05] = 0.0
        return x.astype(np.float32)
    elif kind == "spread":   # many exponents
        return np.exp(rng.uniform(-60, 20, n)).astype(np.float32)
    else:
        raise ValueError(kind)
    return rng.permutation(np.concatenate([ev, kp])).astype(np.float32)


PATTERNS = (("byte0", "byte1", "byte2", "byte3"), ("equal", "ties", "uniform", "spread"))


def _run_cut(n, e, rule, make_unit, tags):
    """Write a crafted state into a 2 x 2-unit cache, cut it, compare with the oracle.
    make_unit(rng, unit_index) -> (positions, float32 scores) of the unit's n entries."""
    _need_gpu()
    b, hk = 2, 2
    kv_max = n - e
    pd = PDAttention(b=b, s=CURR_ID + 1, kv_max=kv_max, block=e, max_gen=0, n_heads=hk,
                     n_kv_heads=hk, head_dim=HEAD_DIM, dtype="f32", device="cuda", init=False)
    assert pd.cap == n
    rng = np.random.default_rng(n * 7919 + e)
    units = [(bi, h) for bi in range(b) for h in range(hk)]
    score = np.zeros((b, hk, n), np.float32)
    pos = np.zeros((b, hk, n), np.int32)
    k = rng.standard_normal((b, hk, n, HEAD_DIM)).astype(np.float32)
    v = rng.standard_normal((b, hk, n, HEAD_DIM)).astype(np.float32)
    for i, (bi, h) in enumerate(units):
        pos[bi, h], score[bi, h] = make_unit(rng, i)
    pd.score.copy_(torch.from_numpy(score))
    pd.pos.copy_(torch.from_numpy(pos))
    pd.k.copy_(torch.from_numpy(k))
    pd.v.copy_(torch.from_numpy(v))
    pd.len.fill_(n)
    pd.resume(n, CURR_ID + 1)
    pd.set_rank_rule(rule)
    print(f"[select] n={n} e={e} rule={rule} patterns={tags}", flush=True)
    pd.evict_compact(CURR_ID)
    torch.cuda.synchronize()
    assert pd.length == kv_max
    g_len = pd.len.cpu().numpy()
    g_pos = pd.pos.cpu().numpy()
    g_score = pd.score.cpu().numpy()
    g_k, g_v = pd.k.cpu().numpy(), pd.v.cpu().numpy()
    for i, (bi, h) in enumerate(units):
        tag = f"unit {(bi, h)} {tags[i]}"
        assert g_len[bi, h] == kv_max, tag
        orc = opd.UnitOracle(head_dim=HEAD_DIM, group=1, kv_max=kv_max, sm_scale=1.0, rule=rule)
        orc.pos = pos[bi, h].astype(np.int64)
        orc.score = score[bi, h].astype(np.float64)
        orc.k = np.zeros((n, HEAD_DIM))
        orc.v = np.zeros((n, HEAD_DIM))
        orc.last_w = np.zeros(n)
        ev = orc.evict(CURR_ID, "prefill")
        kept = g_pos[bi, h, :kv_max]
        assert np.array_equal(np.sort(kept), ev.kept_pos), tag
        # every kept entry carries its own score and K/V rows
        slot_of = {int(p): j for j, p in enumerate(pos[bi, h])}
        src = np.array([slot_of[int(p)] for p in kept])
        assert np.array_equal(g_score[bi, h, :kv_max], score[bi, h, src]), tag
        assert np.array_equal(g_k[bi, h, :kv_max], k[bi, h, src]), tag
        assert np.array_equal(g_v[bi, h, :kv_max], v[bi, h, src]), tag
        # survivors already below kv_max stay in their slots (only holes are filled)
        stay = np.isin(pos[bi, h, :kv_max], kept)
        assert np.array_equal(kept[stay], pos[bi, h, :kv_max][stay]), tag
    pd.close()


def _positions(rng, n):
    return rng.permutation(np.sort(rng.choice(CURR_ID + 1, size=n, replace=False))).astype(np.int32)


SIZES = [(700, 188), (768, 256), (1000, 1), (1000, 999), (3000, 1024), (4096, 512), (5000, 777)]


@pytest.mark.parametrize("n,e", SIZES, ids=lambda x: str(x))
@pytest.mark.parametrize("patterns", PATTERNS, ids=("bytes", "ties"))
def test_cut_on_crafted_state(n, e, patterns):
    def unit(rng, i):
        return _positions(rng, n), _scores(patterns[i], n, e, rng)

    _run_cut(n, e, "sum", unit, patterns)


@pytest.mark.parametrize("n,e", [
    (2048, 128), (2048, 129),                         # 64 KB of moves: one launch, and two
    (2049, 64), (2049, 65),                           # 32 KB past 2048 entries
    (4096, 64), (4096, 65), (4096, 2), (70, 69),      # the most entries; few; one kept
], ids=lambda x: str(x))
def test_cut_at_the_edges_of_one_launch(n, e):
    patterns = ("uniform", "ties", "spread", "byte2")

    def unit(rng, i):
        return _positions(rng, n), _scores(patterns[i], n, e, rng)

    _run_cut(n, e, "sum", unit, patterns)


AVE_PATTERNS = ("equal", "ties", "dyadic", "dyadic_small")


@pytest.mark.parametrize("n,e", SIZES, ids=lambda x: str(x))
def test_cut_ave_rule_exact_quotients(n, e):
    """The paper's rule (Sec. 3.2: sum_weights / (curr_id + 1 - kv_ids)) with
    scores built as target x (curr_id + 1 - pos) exactly, for targets with few
    mantissa bits: the quotient is the target itself in any correctly rounded
    float32 division, so the device's keys equal the oracle's float64 averages
    and the kept sets must match exactly (many exact ties: positions decide)."""
    def unit(rng, i):
        p = _positions(rng, n)
        kind = AVE_PATTERNS[i]
        if kind == "equal":
            t = np.full(n, 0.25)
        elif kind == "ties":
            t = rng.choice([0.0, 0.125, 0.5], size=n)
        elif kind == "dyadic":
            t = rng.integers(0, 64, size=n) / 64.0
        else:
            t = rng.integers(1, 64, size=n) * 2.0 ** -30
        den = (CURR_ID + 1 - p.astype(np.int64)).astype(np.float64)
        sc = (t * den).astype(np.float32)
        assert np.array_equal(sc.astype(np.float64), t * den)          # exact products
        assert np.array_equal(sc.astype(np.float64) / den, t)           # exact quotients
        return p, sc

    _run_cut(n, e, "ave", unit, AVE_PATTERNS)


@pytest.mark.parametrize("kv_max", [511, 1023, 4095])
def test_decode_eviction_exact_ties(kv_max):
    """One decode step (append, attend, one eviction; Algorithm 1's decoding
    loop, one removal per step) on a crafted full cache.  A zero query gives
    every one of the kv_max + 1 entries the weight 1 / (kv_max + 1), a power of
    two, so the updated scores (multiples of 2^-12 below 2) are exact on both
    sides; under the sum rule the smallest score is held by many entries (the
    cached ones that had none, and the new one) and the oldest of them must go.
    Scores, kept sets and outputs against the oracle."""
    _need_gpu()
    b, hk, G = 2, 2, 2
    H, p = hk * G, CURR_ID + 1
    pd = PDAttention(b=b, s=p, kv_max=kv_max, block=256, max_gen=1, n_heads=H, n_kv_heads=hk,
                     head_dim=HEAD_DIM, dtype="f32", device="cuda", init=False)
    rng = np.random.default_rng(kv_max)
    cap = pd.cap
    score = np.zeros((b, hk, cap), np.float32)
    pos = np.zeros((b, hk, cap), np.int32)
    k = rng.standard_normal((b, hk, cap, HEAD_DIM)).astype(np.float32)
    v = rng.standard_normal((b, hk, cap, HEAD_DIM)).astype(np.float32)
    for bi in range(b):
        for h in range(hk):
            pos[bi, h, :kv_max] = _positions(rng, kv_max)
            # zero scores tie, after the update, with the new entry's own weight
            score[bi, h, :kv_max] = rng.choice([0, 3, 5, 900], size=kv_max) * 2.0 ** -12
    q = torch.zeros((b, H, 1, HEAD_DIM), dtype=torch.float32, device="cuda")
    kn = rng.standard_normal((b, hk, 1, HEAD_DIM)).astype(np.float32)
    vn = rng.standard_normal((b, hk, 1, HEAD_DIM)).astype(np.float32)
    o = torch.zeros_like(q)
    for dst, src in ((pd.score, score), (pd.pos, pos), (pd.k, k), (pd.v, v)):
        dst.copy_(torch.from_numpy(src))
    pd.len.fill_(kv_max)
    pd.resume(kv_max, p)
    pd.set_rank_rule("sum")
    print(f"[select] decode step kv_max={kv_max}", flush=True)
    pd.decode_step(p, q, torch.from_numpy(kn).cuda(), torch.from_numpy(vn).cuda(), o, row=0)
    torch.cuda.synchronize()
    assert pd.length == kv_max
    g_pos, g_score = pd.pos.cpu().numpy(), pd.score.cpu().numpy()
    g_o = o.cpu().numpy()
    for bi in range(b):
        for h in range(hk):
            tag = f"unit {(bi, h)}"
            orc = opd.UnitOracle(head_dim=HEAD_DIM, group=G, kv_max=kv_max, sm_scale=1.0,
                                 rule="sum")
            orc.pos = pos[bi, h, :kv_max].astype(np.int64)
            orc.score = score[bi, h, :kv_max].astype(np.float64)
            orc.k = k[bi, h, :kv_max].astype(np.float64)
            orc.v = v[bi, h, :kv_max].astype(np.float64)
            orc.last_w = np.zeros(kv_max)
            ref, ev = orc.decode_step(p, np.zeros((G, HEAD_DIM)), kn[bi, h, 0], vn[bi, h, 0])
            assert ev is not None and ev.gap == 0.0, tag      # the cut falls inside a tie
            kept = g_pos[bi, h, :kv_max]
            assert np.array_equal(np.sort(kept), ev.kept_pos), tag
            by_pos = dict(zip(orc.pos.tolist(), orc.score.tolist()))
            assert all(float(g_score[bi, h, j]) == by_pos[int(kept[j])] for j in range(kv_max)), tag
            err = np.max(np.abs(g_o[bi, h * G:(h + 1) * G, 0] - ref))
            assert err <= 1e-4, (tag, err)
    pd.close()


def _cut_us(units, n, removed):
    """Median time of the cut of n entries by themselves down to n - removed."""
    att = PDAttention(b=units, s=n + 100, kv_max=n - removed, block=removed, max_gen=0, n_heads=1,
                      n_kv_heads=1, head_dim=128, dtype="bf16")
    att.set_rank_rule("sum")
    att.k.zero_()
    att.v.zero_()
    score = torch.rand(att.score.shape, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    pos = torch.arange(att.cap, device="cuda", dtype=torch.int32).expand(score.shape).contiguous()
    wait = torch.empty(1 << 28, device="cuda")
    times = []
    for _ in range(7):
        att.score.copy_(score)
        att.pos.copy_(pos)
        att.resume(n, n + 100)
        wait.zero_()                # work ahead of the cut, so that the host is not what is timed
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        att.evict_compact(n + 99)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    att.close()
    return sorted(times)[3]


def test_time_of_large_cuts_grows_with_their_entries():
    # the same moves with twice the entries to rank: the latter is reading twice the
    # scores, not waiting for a place on a compute unit (2.3 to 2.4 times the time when
    # one workgroup of the larger cut took a unit's LDS; 1.4 to 1.5 now, six runs each)
    _need_gpu()
    t1, t2 = _cut_us(2048, 2048, 32), _cut_us(2048, 4096, 32)
    print(f"[select] 2048 units, 32 removed: {t1:.1f} us of 2048 entries, {t2:.1f} us of 4096", flush=True)
    assert t2 < 2 * t1
