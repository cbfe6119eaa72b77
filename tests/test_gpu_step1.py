"""GPU parity: energies, flip deltas, the first-step walker and the pool,
through the C ABI, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import labs_inputs as li

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_07222_amd import labs
    labs.lib()
    return labs


def _dev(packed):
    import torch
    return torch.from_numpy(np.ascontiguousarray(packed).view(np.int32)).cuda()


def _host_seqs(t, L):
    return li.unpack(t.cpu().numpy().view(np.uint32), L)


# ------------------------------------------------------------------ energies
@pytest.mark.parametrize("L", [1, 2, 3, 5, 31, 32, 33, 37, 64, 101, 255, 501, 527, 1023])
def test_energy_parity(lb, orc, L):
    S = li.random_pm1(100 + L, 40, L)
    edge = np.stack([np.ones(L, np.int8), np.array([(-1) ** i for i in range(L)], np.int8),
                     -np.ones(L, np.int8)])
    S = np.concatenate([S, edge])
    E, C = lb.energy(L, _dev(li.pack(S)), want_c=True)
    Eo, Co = orc.energy_batch(S, with_c=True)
    assert np.array_equal(E.cpu().numpy(), Eo)
    assert np.array_equal(C.cpu().numpy(), Co)


def test_energy_empty(lb):
    import torch
    E = lb.energy(37, torch.zeros((0, 2), dtype=torch.int32, device="cuda"))
    assert E.numel() == 0


@pytest.mark.parametrize("L", [2, 3, 7, 37, 64, 101, 501])
def test_flip_deltas_single(lb, orc, L):
    S = li.random_pm1(7 * L, 12, L)
    dE = lb.flip_deltas(L, _dev(li.pack(S))).cpu().numpy()
    for j in range(len(S)):
        assert np.array_equal(dE[j], orc.deltas_single(S[j]))


@pytest.mark.parametrize("L,p", [(3, 0), (5, 1), (37, 0), (101, 8), (501, 16), (527, 16)])
def test_flip_deltas_skew(lb, orc, L, p):
    S = np.concatenate([li.random_skew(L, 6, L, p), li.random_pm1(L + 1, 2, L)])
    dE = lb.flip_deltas(L, _dev(li.pack(S)), skew=True, p=p).cpu().numpy()
    for j in range(len(S)):
        assert np.array_equal(dE[j], orc.deltas_skew(S[j], p))


@pytest.mark.parametrize("L", [1, 16, 17, 31, 32, 33, 48, 49, 255, 256, 257, 511, 513, 767, 768, 769, 1008, 1009, 1023])
def test_flip_deltas_edges(lb, orc, L):
    """Word, 16-element, 64-element and tile edges of the flips' products; the constant
    sequences reach the largest C (two bytes), and bits behind the last element are
    not read."""
    S = np.concatenate([li.random_pm1(5 * L, 4, L), np.ones((1, L), np.int8), -np.ones((1, L), np.int8)])
    words = li.pack(S).view(np.uint32).copy()
    if L % 32:
        words[:, -1] |= np.uint32(0xFFFFFFFF >> (L % 32))
    E, C = lb.energy(L, _dev(words), want_c=True)
    Eo, Co = orc.energy_batch(S, with_c=True)
    assert np.array_equal(E.cpu().numpy(), Eo)
    if L > 1:
        assert np.array_equal(C.cpu().numpy(), Co)
    dE = lb.flip_deltas(L, _dev(words)).cpu().numpy()
    for j in range(len(S)):
        assert np.array_equal(dE[j], orc.deltas_single(S[j]))
    if L % 2 and L >= 3:
        for p in {0, (L - 1) // 4, (L - 1) // 2}:
            dE = lb.flip_deltas(L, _dev(words), skew=True, p=p).cpu().numpy()
            for j in range(len(S)):
                assert np.array_equal(dE[j], orc.deltas_skew(S[j], p))


def test_cfg1_exhaustive(lb, orc):
    """All 2^19 skew-symmetric sequences at L = 37: min E and its argmin set."""
    L = 37
    S = li.skew_all(L)
    E = lb.energy(L, _dev(li.pack(S))).cpu().numpy()
    m, allE = orc.skew_exhaustive(L, want_all=True)
    assert E.min() == m
    assert np.array_equal(np.nonzero(E == E.min())[0], np.nonzero(allE == m)[0])
    assert np.array_equal(E, allE)


# ------------------------------------------------------------------ walker
def _compare_walk(lb, orc, L, p, steps, lo, hi, seed, n, begin=0):
    r = lb.walk_step1(L, p, steps, lo, hi, seed, n, walker_begin=begin, want_traj=True)
    o = orc.walk(L, p, steps, lo, hi, seed, range(begin, begin + n))
    traj = r.traj_E.cpu().numpy()
    for j in range(n):
        assert np.array_equal(traj[j], o["traj"][j]), "walker %d" % (begin + j)
    assert np.array_equal(_host_seqs(r.final_seqs, L), o["final"])
    assert np.array_equal(r.final_E.cpu().numpy(), o["final_E"])
    assert np.array_equal(r.best_E.cpu().numpy(), o["best_E"])
    assert np.array_equal(r.best_step.cpu().numpy(), o["best_step"])
    assert np.array_equal(_host_seqs(r.best_seqs, L), o["best"])
    k = (L - 1) // 2
    halted = (o["traj"] < 0).sum(axis=1)
    assert int(r.flip_evals.item()) == int(((steps - halted) * (k + 1 - p)).sum())
    return r


def test_walk_cfg1_trajectories(lb, orc):
    """The first configuration: L = 37, p = 0, tenure 8, 256 walkers x 4096 steps."""
    _compare_walk(lb, orc, 37, 0, 4096, 8, 8, 1, 256)


@pytest.mark.parametrize("L,p,steps,lo,hi,n", [
    (5, 0, 40, 0, 2, 8),          # smallest length, zero tenure allowed
    (7, 2, 30, 0, 1, 4),
    (13, 0, 200, 2, 2, 16),
    (63, 3, 300, 4, 9, 8),        # k = 31: one full even-lag word
    (65, 0, 300, 5, 11, 8),       # k = 32: free count 33, second slot partly used
    (101, 8, 600, 10, 20, 12),    # the second configuration's shape
    (131, 1, 400, 13, 26, 4),     # k = 65: two chunks of 64 lags, 65 free positions
    (301, 12, 60, 30, 60, 2),     # third configuration's range
    (301, 120, 40, 3, 6, 2),      # long prefix: 31 free positions in the smallest slot group
    (385, 12, 30, 38, 77, 2),     # k = 192: six even-lag words, three slot groups
    (387, 12, 30, 38, 77, 2),     # k = 193: one lag into a seventh word, still three groups
    (389, 12, 30, 38, 77, 2),     # k = 194: two lags in the seventh word, backward word in use
    (133, 4, 200, 13, 26, 4),     # k = 66: three words, two lags in the last, backward word in use
    (141, 2, 200, 14, 28, 4),     # k = 70: six lags in the last word
    (143, 2, 200, 14, 28, 4),     # k = 71: seven lags in the last word
    (259, 8, 100, 25, 50, 2),     # k = 129: five words, one lag in the last
    (527, 16, 20, 52, 105, 2),    # k = 263: nine words, four slot groups
    (409, 12, 30, 40, 81, 2),     # k = 204: seven words, four slot groups (the half tile, held to four waves)
    (449, 12, 30, 44, 89, 2),     # k = 224: seven full words, four slot groups
])
def test_walk_shapes(lb, orc, L, p, steps, lo, hi, n):
    _compare_walk(lb, orc, L, p, steps, lo, hi, 7 + L, n)


def test_walk_L501_cfg4_shape(lb, orc):
    _compare_walk(lb, orc, 501, 16, 40, 50, 100, 4, 3)


def test_walk_long_no_pool(lb, orc):
    """9,000 steps without a pool run as three launches of up to 4,096 steps; the
    whole trajectories, final and best sequences equal the oracle's."""
    L, p, steps, n = 37, 0, 9000, 12
    r = lb.walk_step1(L, p, steps, 8, 8, 21, n, want_traj=True)
    o = orc.walk(L, p, steps, 8, 8, 21, range(n))
    assert np.array_equal(r.traj_E.cpu().numpy(), o["traj"])
    assert np.array_equal(_host_seqs(r.final_seqs, L), o["final"])
    assert np.array_equal(_host_seqs(r.best_seqs, L), o["best"])
    assert np.array_equal(r.best_step.cpu().numpy(), o["best_step"])


def test_walk_L501_across_pool_segments(lb, orc):
    """L = 501 with the pool on: the walk runs in segments of 256, 512, ... steps
    with a compaction between them.  Two walkers' 1,200-step trajectories equal the
    oracle's linear-time walker (pinned to the definitional one in the CPU suite),
    and the pool holds exactly the distinct sequences the walkers reached at
    E <= e_max, each at an energy their trajectories show."""
    L, p, steps, n = 501, 16, 1200, 2
    em = orc.e_max_for_tau(L, 4, 1)
    pool = lb.PoolBuffers.empty(L, 1 << 16)
    r = lb.walk_step1(L, p, steps, 50, 100, 4, n, e_max=em, pool=pool, want_traj=True)
    b = orc.baseline_walk(L, p, steps, 50, 100, 4, 0, n, threads=2, want_traj=True)
    traj = r.traj_E.cpu().numpy()
    assert np.array_equal(traj, b["traj"])
    assert np.array_equal(r.final_E.cpu().numpy(), b["final_E"])
    assert np.array_equal(r.best_E.cpu().numpy(), b["best_E"])
    cnt = int(pool.count.item())
    assert cnt > 0 and int(pool.dropped.item()) == 0
    pw, ps, pe = (pool.walker[:cnt].cpu().numpy(), pool.step[:cnt].cpu().numpy(),
                  pool.E[:cnt].cpu().numpy())
    assert np.array_equal(traj[pw, ps - 1], pe)
    assert np.array_equal(orc.energy_batch(_host_seqs(pool.seqs[:cnt], L)), pe)
    # every step at or below e_max was offered; distinct sequences, so at most that many
    assert cnt <= int((traj <= em).sum()) and pe.max() <= em


def test_walk_halts(lb, orc):
    """Tenure = free count - 1 with p = k-1 leaves 2 free positions: the walker
    alternates; tenure equal to the free count is rejected, so check the edge
    where every move becomes tabu is unreachable and the trajectory has no -1."""
    _compare_walk(lb, orc, 9, 3, 20, 1, 1, 5, 3)


def test_walk_sharding_invariance(lb, orc):
    """Any split of the walker range gives the same per-walker results."""
    L, p, steps = 101, 8, 300
    a = lb.walk_step1(L, p, steps, 10, 20, 99, 64, want_traj=True)
    b1 = lb.walk_step1(L, p, steps, 10, 20, 99, 21, walker_begin=0, want_traj=True)
    b2 = lb.walk_step1(L, p, steps, 10, 20, 99, 43, walker_begin=21, want_traj=True)
    import torch
    assert torch.equal(a.traj_E, torch.cat([b1.traj_E, b2.traj_E]))
    assert torch.equal(a.final_seqs, torch.cat([b1.final_seqs, b2.final_seqs]))


def test_walk_default_steps(lb):
    r = lb.walk_step1(37, 0, 0, 8, 8, 1, 2, want_traj=True)
    assert r.traj_E.shape[1] == 4 * 38


def test_walk_invalid_args(lb):
    with pytest.raises(lb.LabsError):
        lb.walk_step1(36, 0, 10, 1, 1, 1, 4)          # even L
    with pytest.raises(lb.LabsError):
        lb.walk_step1(37, 0, 10, 19, 19, 1, 4)        # tenure >= free count
    with pytest.raises(lb.LabsError):
        lb.walk_step1(37, 18, 10, 0, 0, 1, 4)         # p > k-1


# ------------------------------------------------------------------ pool
def test_pool_sieve_cfg2_shape(lb, orc):
    """Second configuration's shape (L = 101, p = 8) at reduced size; the
    threshold is lowered to F >= 4.4 so that 500 steps produce offers."""
    L, p, steps, n = 101, 8, 500, 24
    em = orc.e_max_for_tau(L, 22, 5)
    for cap in (1 << 20, 50):
        pool = lb.PoolBuffers.empty(L, cap)
        r = lb.walk_step1(L, p, steps, 10, 20, 2, n, e_max=em, pool=pool, want_traj=True)
        o = orc.walk(L, p, steps, 10, 20, 2, range(n), e_max=em)
        assert np.array_equal(r.traj_E.cpu().numpy(), o["traj"])
        ref, dropped = orc.pool(o["emits"], cap)
        cnt = int(pool.count.item())
        assert len(ref) >= 20
        assert cnt == len(ref)
        assert int(pool.dropped.item()) == dropped
        got_E = pool.E[:cnt].cpu().numpy()
        got_S = _host_seqs(pool.seqs[:cnt], L)
        assert [int(e) for e in got_E] == [e for e, _ in ref]
        assert [orc.seq_key(s) for s in got_S] == [k for _, k in ref]
        # walker/step of the earliest offer of each sequence
        first = {}
        for E, s, w, t in o["emits"]:
            key = orc.seq_key(s)
            if key not in first or (w, t) < first[key]:
                first[key] = (w, t)
        gw = pool.walker[:cnt].cpu().numpy()
        gt = pool.step[:cnt].cpu().numpy()
        for i, (_, key) in enumerate(ref):
            assert (int(gw[i]), int(gt[i])) == first[key]


def test_pool_dropped_repeats_across_segments(lb, orc):
    """At L = 21 the walkers revisit sequences often, so the same sequence is
    offered in several compaction segments (the pool path starts with 256-step
    segments) and is cut each time the capacity is reached: `dropped` counts it
    once.  A second call on the same pool counts the distinct sequences of (its
    previous contents) U (the new offers) beyond the capacity."""
    L, p, steps, n, cap = 21, 0, 3000, 48, 30
    em = orc.e_max_for_tau(L, 3, 1)
    pool = lb.PoolBuffers.empty(L, cap)
    lb.walk_step1(L, p, steps, 1, 3, 7, n, e_max=em, pool=pool)
    o = orc.walk(L, p, steps, 1, 3, 7, range(n), e_max=em, want_traj=False)
    ref, dropped = orc.pool(o["emits"], cap)
    assert len(o["emits"]) > 2 * (len(ref) + dropped)      # the case has many repeats
    assert dropped > 0
    cnt = int(pool.count.item())
    assert cnt == cap
    assert int(pool.dropped.item()) == dropped
    assert [orc.seq_key(s) for s in _host_seqs(pool.seqs[:cnt], L)] == [k for _, k in ref]
    # a second call adds to the same pool
    lb.walk_step1(L, p, 700, 1, 3, 8, n, e_max=em, pool=pool)
    o2 = orc.walk(L, p, 700, 1, 3, 8, range(n), e_max=em, want_traj=False)
    prev = [(E, orc.key_seq(k, L)) for E, k in ref]
    ref2, dropped2 = orc.pool(prev + o2["emits"], cap)
    assert int(pool.dropped.item()) == dropped + dropped2
    assert [orc.seq_key(s) for s in _host_seqs(pool.seqs[:cap], L)] == [k for _, k in ref2]


def test_pool_topk_edges(lb, orc):
    """k beyond the pool's distinct sequences returns all of them, in order; an
    empty pool returns none."""
    L, p, steps, n = 63, 4, 200, 40
    pool = lb.PoolBuffers.empty(L, 1000)
    lb.walk_step1(L, p, steps, 4, 9, 11, n, e_max=-1, pool=pool, pool_walker_best=True)
    o = orc.walk(L, p, steps, 4, 9, 11, range(n))
    ref, _ = orc.pool([(int(o["best_E"][j]), o["best"][j]) for j in range(n)], 1000)
    s, E = lb.pool_topk(pool, len(ref) + 25)
    assert [int(e) for e in E.cpu().numpy()] == [e for e, _ in ref]
    assert [orc.seq_key(x) for x in _host_seqs(s, L)] == [k for _, k in ref]
    s, E = lb.pool_topk(lb.PoolBuffers.empty(L, 16), 4)
    assert len(E) == 0 and len(s) == 0


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 9000])
@pytest.mark.parametrize("run", [1, 2, 31, 32, 33, 400])
def test_pool_topk_shared_leading_words(lb, n, run):
    """Entries that agree in E and their leading words and differ behind them, in
    runs up to and beyond the longest that is put in order in place, some twice: the
    distinct ones in the order of (E, words)."""
    import torch
    L, W = 501, 16
    g = np.random.default_rng(31 * n + run)
    words = g.integers(0, 2 ** 32, (n, W), dtype=np.uint32)
    words[:, -1] &= np.uint32(0xFFFFFFFF << (32 * W - L) & 0xFFFFFFFF)
    E = g.integers(20000, 20200, n).astype(np.int32)
    head = (np.arange(n) // run) * run            # every run takes its first entry's lead
    words[:, :3] = words[head, :3]
    E[:] = E[head]
    twice = np.arange(n) % 7 == 3
    twice[0] = False
    words[twice] = words[np.flatnonzero(twice) - 1]
    E[twice] = E[np.flatnonzero(twice) - 1]
    order = g.permutation(n)
    pool = lb.PoolBuffers.empty(L, n + 3)
    pool.seqs[:n] = torch.from_numpy(words[order].view(np.int32)).cuda()
    pool.E[:n] = torch.from_numpy(E[order]).cuda()
    pool.count.fill_(n)
    want = np.unique(np.concatenate([E[:, None].astype(np.uint32), words], 1), axis=0)
    for k in (5, n + 1):
        s, e = lb.pool_topk(pool, k)
        got = np.concatenate([e.cpu().numpy()[:, None].view(np.uint32), s.cpu().numpy().view(np.uint32)], 1)
        assert np.array_equal(got, want[:k])


def test_pool_topk_and_walker_best(lb, orc):
    L, p, steps, n = 63, 4, 200, 40
    pool = lb.PoolBuffers.empty(L, 1000)
    lb.walk_step1(L, p, steps, 4, 9, 11, n, e_max=-1, pool=pool, pool_walker_best=True)
    o = orc.walk(L, p, steps, 4, 9, 11, range(n))
    entries = [(int(o["best_E"][j]), o["best"][j]) for j in range(n)]
    ref, _ = orc.pool(entries, 1000)
    assert int(pool.count.item()) == len(ref)
    s, E = lb.pool_topk(pool, 10)
    assert [int(e) for e in E.cpu().numpy()] == [e for e, _ in ref[:10]]
    assert [orc.seq_key(x) for x in _host_seqs(s, L)] == [k for _, k in ref[:10]]


@pytest.mark.parametrize("L,p,n", [(5, 0, 4097), (37, 0, 4098), (101, 8, 4099), (105, 1, 4096), (107, 8, 8193),
                                   (125, 0, 8194), (127, 0, 8193), (127, 3, 8195), (129, 8, 8192), (201, 16, 8193),
                                   (231, 0, 8192), (233, 16, 8193)])
def test_several_walkers_a_wave_equal_one(lb, L, p, n):
    """Short sequences walk four or two to a wave where there are many walkers: energies,
    final and best states against the logging walk (a wave a walker), at the lengths where
    the lags, the indices or a class row stop to fit, with a last wave that is not full."""
    nf = (L - 1) // 2 + 1 - p
    steps, lo, hi = 90, max(1, nf // 8), max(1, nf // 3)
    a = lb.walk_step1(L, p, steps, lo, hi, 23, n, want_traj=True)
    b = lb.learned_walk(L, p, steps, lo, hi, 23, n, mode=lb.PROPOSE_RANDOM, top_m=1, fallback_every=1, want_traj=True)
    for key in ("traj_E", "final_seqs", "final_E", "best_seqs", "best_E", "best_step"):
        assert np.array_equal(getattr(a, key).cpu().numpy(), b[key].cpu().numpy()), key


@pytest.mark.parametrize("L,p", [(101, 8), (201, 12)])
def test_several_walkers_a_wave_fill_the_same_pool(lb, L, p):
    """The sieve of 8,192 walkers in one launch (several a wave) against four launches of
    2,048 (a wave a walker) into one pool."""
    lo, hi, steps, e_max = L // 10, L // 5, 150, L * L // 9
    one, four = lb.PoolBuffers.empty(L, 1 << 18), lb.PoolBuffers.empty(L, 1 << 18)
    lb.walk_step1(L, p, steps, lo, hi, 3, 8192, e_max=e_max, pool=one)
    for q in range(4):
        lb.walk_step1(L, p, steps, lo, hi, 3, 2048, walker_begin=2048 * q, e_max=e_max, pool=four)
    c = int(one.count.item())
    assert c > 100 and c == int(four.count.item())
    assert int(one.dropped.item()) == int(four.dropped.item()) == 0
    for key in ("E", "seqs", "walker", "step"):
        assert np.array_equal(getattr(one, key)[:c].cpu().numpy(), getattr(four, key)[:c].cpu().numpy()), key


@pytest.mark.parametrize("L,p,n", [(37, 2, 4098), (101, 8, 4097), (107, 8, 8193), (201, 12, 8193)])
def test_several_walkers_a_wave_go_on_in_the_next_launch(lb, L, p, n):
    """More steps than one launch holds: walkers that share a wave take up tabu deadlines,
    correlations and bests where the launch before left them, as walkers alone do."""
    steps, lo, hi = 4200, L // 10, L // 5
    a = lb.walk_step1(L, p, steps, lo, hi, 29, n)
    b = lb.learned_walk(L, p, steps, lo, hi, 29, n, mode=lb.PROPOSE_RANDOM, top_m=1, fallback_every=1)
    for key in ("final_seqs", "final_E", "best_seqs", "best_E", "best_step"):
        assert np.array_equal(getattr(a, key).cpu().numpy(), b[key].cpu().numpy()), key
    if L > 100:                          # shorter walks have their optimum long before
        assert int((a.best_step > 4096).sum().item()) > 0


@pytest.mark.parametrize("L,p", [(101, 8), (201, 12)])
def test_several_walkers_a_wave_fill_the_same_pool_over_segments(lb, L, p):
    """With a pool a launch holds 256 steps at first: 900 steps of 8,192 walkers in shared
    waves against four calls of 2,048 walkers a wave each."""
    lo, hi, steps, e_max = L // 10, L // 5, 900, L * L // 10
    one, four = lb.PoolBuffers.empty(L, 1 << 18), lb.PoolBuffers.empty(L, 1 << 18)
    lb.walk_step1(L, p, steps, lo, hi, 3, 8192, e_max=e_max, pool=one, pool_walker_best=True)
    for q in range(4):
        lb.walk_step1(L, p, steps, lo, hi, 3, 2048, walker_begin=2048 * q, e_max=e_max, pool=four,
                      pool_walker_best=True)
    c = int(one.count.item())
    assert c > 8000 and c == int(four.count.item())
    assert int(one.dropped.item()) == int(four.dropped.item()) == 0
    assert int(one.step[:c].max().item()) > 256
    for key in ("E", "seqs", "walker", "step"):
        assert np.array_equal(getattr(one, key)[:c].cpu().numpy(), getattr(four, key)[:c].cpu().numpy()), key


# ------------------------------------------------------------------ edges of the walk kernel
# Lengths on both sides of every size the matrix-core scan is instantiated at: the class
# rows grow by 32 indices where k + 12 passes a multiple of 32 (L = 105/107, 169/171, ...,
# 617/619), a second group of lags starts at k > 256 (L = 513/515), a second tile of slots
# where more than 128 indices are scanned (p = 0 against p = 16 from L = 511 on), and long
# prefixes leave two free positions.  Even and odd k read the partner lags differently.
_EDGES = [(5, 0), (7, 1), (9, 0), (31, 0), (33, 2), (105, 0), (107, 0), (169, 3), (171, 1), (233, 12), (235, 12),
          (297, 12), (299, 5), (361, 1), (363, 12), (425, 16), (427, 2), (489, 16), (491, 7), (501, 0), (501, 248),
          (509, 0), (511, 16), (513, 16), (513, 255), (515, 2), (515, 17), (527, 8), (527, 0), (553, 2), (553, 40),
          (555, 1), (617, 16), (617, 0), (619, 0), (619, 60), (637, 1), (639, 0), (639, 16), (639, 317)]


@pytest.mark.parametrize("L,p", _EDGES)
def test_walk_scan_edges(lb, orc, L, p):
    nf = (L - 1) // 2 + 1 - p
    hi = min(L // 5, nf - 1)
    lo = min(L // 10, hi)
    n, steps = 40, 150
    r = lb.walk_step1(L, p, steps, lo, hi, 70 + L, n, want_traj=True)
    o = orc.baseline_walk(L, p, steps, lo, hi, 70 + L, 0, n, want_traj=True)
    assert np.array_equal(r.traj_E.cpu().numpy(), o["traj"])
    assert np.array_equal(r.best_E.cpu().numpy(), o["best_E"])
    # the packed results, rebuilt from the class rows, carry these energies
    for seqs, E in ((r.final_seqs, r.final_E), (r.best_seqs, r.best_E)):
        assert np.array_equal(orc.energy_batch(_host_seqs(seqs, L)), E.cpu().numpy())


@pytest.mark.parametrize("L,p", [(105, 0), (301, 12), (513, 16), (515, 2), (527, 0), (553, 2), (619, 16)])
def test_bloom_scan_edges(lb, orc, L, p):
    steps, n = 12, 2
    r = lb.walk_step1(L, p, steps, 0, 0, 5 + L, n, want_traj=True, bloom=(10, 5))
    o = orc.walk_bloom(L, p, steps, 10, 5, 5 + L, range(n))
    assert np.array_equal(r.traj_E.cpu().numpy(), o["traj"])


def test_batched_scan_edges(lb):
    """The persistent form at the same edges, against one launch per length."""
    import torch
    cfgs = []
    for L, p in _EDGES:
        nf = (L - 1) // 2 + 1 - p
        hi = min(L // 5, nf - 1)
        cfgs.append(dict(L=L, p=p, steps=90, tenure_lo=min(L // 10, hi), tenure_hi=hi, seed=9, n_walkers=24))
    res, _ = lb.walk_step1_batch(cfgs, want_traj=True)
    torch.cuda.synchronize()
    for c, r in zip(cfgs, res):
        one = lb.walk_step1(c["L"], c["p"], c["steps"], c["tenure_lo"], c["tenure_hi"], c["seed"], c["n_walkers"],
                            want_traj=True)
        assert torch.equal(r.traj_E, one.traj_E), (c["L"], c["p"])
        assert torch.equal(r.best_seqs, one.best_seqs) and torch.equal(r.final_seqs, one.final_seqs), (c["L"], c["p"])
