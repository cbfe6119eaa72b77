"""GPU parity of the walk with a proposer (labs_learned_walk) through the C ABI:
full-scan and covering configurations equal the plain walker; the random
proposer's whole trajectory equals the CPU reference; with the network, every
step's move and energy are replayed exactly by the oracle on the logged
candidate sets, and each set is the top-m of the CPU reference logits up to the
logit tolerance; the training log holds the plain walker's states and moves."""
import numpy as np
import pytest

import labs_inputs as li
from oracle import learned as ol
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_07222_amd import labs
    labs.lib()
    return labs


def _np(t):
    return t.cpu().numpy()


def _net(lb, L, hidden, seed):
    import torch
    lay = lb.mlp_layout(L, hidden)
    P = li.mlp_init(seed, lay.d_in, hidden, lay.d_out)
    blob = torch.from_numpy(lb.mlp_blob_from_dict(lay, P)).cuda()
    pb = torch.empty(lay.n_params, dtype=torch.bfloat16, device="cuda")
    lb.mlp_cast(lay, blob, pb)
    return lay, P, blob, pb


@pytest.mark.parametrize("L,p,lo,hi,steps", [(37, 0, 3, 6, 300), (101, 8, 10, 20, 257)])
def test_full_scan_every_step_equals_plain_walker(lb, orc, L, p, lo, hi, steps):
    n = 96
    plain = lb.walk_step1(L, p, steps, lo, hi, 21, n, want_traj=True)
    r = lb.learned_walk(L, p, steps, lo, hi, 21, n, mode=lb.PROPOSE_RANDOM, top_m=4,
                        fallback_every=1, want_traj=True)
    assert np.array_equal(_np(r["traj_E"]), _np(plain.traj_E))
    assert np.array_equal(_np(r["final_seqs"]), _np(plain.final_seqs))
    assert np.array_equal(_np(r["best_E"]), _np(plain.best_E))
    assert np.array_equal(_np(r["best_step"]), _np(plain.best_step))
    # the plain walker counts every free position per step; this walk evaluates
    # only the admissible ones: nf - min(t-1, tenure) at step t (the last `tenure`
    # moved positions are distinct and still tabu)
    nf = (L - 1) // 2 + 1 - p
    want = 0
    for w in range(n):
        ten = orc.walker_init(21, L, p, w, lo, hi)[1]
        want += sum(nf - min(t - 1, ten) for t in range(1, steps + 1))
    assert int(r["flip_evals"].item()) == want
    assert int(plain.flip_evals.item()) == n * steps * nf


def test_covering_top_m_equals_plain_walker_with_network(lb):
    L, p, lo, hi, steps, n = 101, 8, 10, 20, 200, 64
    lay, P, blob, pb = _net(lb, L, 64, 55)
    plain = lb.walk_step1(L, p, steps, lo, hi, 5, n, want_traj=True)
    r = lb.learned_walk(L, p, steps, lo, hi, 5, n, mode=lb.PROPOSE_MLP, top_m=64,
                        fallback_every=8, hidden=64, params=blob, params_bf16=pb, want_traj=True)
    assert np.array_equal(_np(r["traj_E"]), _np(plain.traj_E))


@pytest.mark.parametrize("L,p,m,F,steps", [(37, 0, 3, 5, 200), (101, 8, 8, 16, 300)])
def test_random_proposer_matches_oracle(lb, orc, L, p, m, F, steps):
    lo, hi, seed, ps, n = L // 10, L // 5, 17, 99, 24
    e_max = orc.e_max_for_tau(L, 4)
    r = lb.learned_walk(L, p, steps, lo, hi, seed, n, mode=lb.PROPOSE_RANDOM, top_m=m,
                        fallback_every=F, prop_seed=ps, e_max=e_max, want_traj=True,
                        want_cands=True)
    traj, moves, cands = _np(r["traj_E"]), _np(r["moves"]), _np(r["cands"])
    hit, bestE = _np(r["hit_step"]), _np(r["best_E"])
    for w in (0, 7, n - 1):
        ref = ol.proposal_walk(L, p, steps, lo, hi, seed, w, F, ol.random_proposer(ps, L, w, m),
                               e_max=e_max)
        assert np.array_equal(traj[w], np.array(ref["traj"])), w
        assert np.array_equal(moves[w], np.array(ref["moves"])), w
        for t, c in enumerate(ref["cands"]):
            got = [int(x) for x in cands[w, t] if x >= 0]
            assert got == (c if c is not None else []), (w, t)
        assert hit[w] == ref["hit_step"] and bestE[w] == ref["best_E"]
    assert int(r["flip_evals"].item()) > 0


def test_network_proposer_replay(lb, orc):
    """Each move is the exact best of its logged set (definitional energies), and
    each set holds the top-m admissible positions by the CPU reference logits up
    to the 1e-2 logit tolerance."""
    L, p, m, F, steps, n, hidden = 101, 8, 8, 16, 96, 8, 64
    lo, hi, seed = 10, 20, 23
    lay, P, blob, pb = _net(lb, L, hidden, 56)
    r = lb.learned_walk(L, p, steps, lo, hi, seed, n, mode=lb.PROPOSE_MLP, top_m=m,
                        fallback_every=F, hidden=hidden, params=blob, params_bf16=pb,
                        want_traj=True, want_cands=True)
    traj, moves, cands = _np(r["traj_E"]), _np(r["moves"]), _np(r["cands"])
    for w in range(0, n, 3):
        logged = {}

        def propose(t, s, adm, w=w):
            c = [int(x) for x in cands[w, t - 1] if x >= 0]
            C = orc.energy(s, with_c=True)[1][1::2]
            z, _ = omlp.forward(P, omlp.features(s[None, :], C[None, :]), exact=False)
            z = z[0]
            tol = 1e-2 * max(1.0, np.abs(z).max())
            assert len(c) == min(m, len(adm)) and set(c) <= set(adm)
            rest = [a for a in adm if a not in c]
            if rest:
                assert min(z[a - 1] for a in c) >= max(z[a - 1] for a in rest) - 2 * tol
            logged[t] = c
            return c

        ref = ol.proposal_walk(L, p, steps, lo, hi, seed, w, F, propose)
        assert np.array_equal(traj[w], np.array(ref["traj"])), w
        assert np.array_equal(moves[w], np.array(ref["moves"])), w
        assert len(logged) == steps - (steps + F - 1) // F


def test_training_log_is_plain_walker_data(lb, orc):
    L, p, lo, hi, steps, n, every = 37, 2, 3, 6, 60, 16, 4
    r = lb.learned_walk(L, p, steps, lo, hi, 8, n, mode=lb.PROPOSE_RANDOM, top_m=1,
                        fallback_every=1, log_every=every, want_traj=True)
    seqs, mask, label = _np(r["log_seqs"]), _np(r["log_mask"]), _np(r["log_label"])
    n_log = steps // every
    for w in (0, 9):
        ref = ol.proposal_walk(L, p, steps, lo, hi, 8, w, 1, None)
        for q in range(n_log):
            t = (q + 1) * every
            rec = q * n + w
            st = li.unpack(seqs[rec:rec + 1].view(np.uint32), L)[0]
            assert np.array_equal(st, ref["states"][t - 1])
            adm = [a for a in range(1, (L - 1) // 2 + 2)
                   if (int(mask[rec, (a - 1) // 32]) >> ((a - 1) % 32)) & 1]
            assert adm == ref["admissible"][t - 1]
            assert label[rec] == ref["moves"][t - 1] - 1


def test_repeat_call_reuses_graph_identically(lb):
    L, p, lo, hi, steps, n = 101, 8, 10, 20, 200, 32
    lay, P, blob, pb = _net(lb, L, 64, 57)
    a = lb.learned_walk(L, p, steps, lo, hi, 3, n, mode=lb.PROPOSE_MLP, top_m=8,
                        fallback_every=16, hidden=64, params=blob, params_bf16=pb, want_traj=True)
    b = lb.learned_walk(L, p, steps, lo, hi, 3, n, mode=lb.PROPOSE_MLP, top_m=8,
                        fallback_every=16, hidden=64, params=blob, params_bf16=pb, want_traj=True,
                        workspace=a["workspace"])
    assert np.array_equal(_np(a["traj_E"]), _np(b["traj_E"]))


@pytest.mark.parametrize("L,p,m,F,n,steps", [(5, 0, 2, 3, 1, 12), (37, 0, 9, 2, 17, 40), (255, 10, 16, 4, 3, 14),
                                             (257, 0, 8, 7, 5, 16), (511, 16, 17, 5, 2, 12),
                                             (513, 3, 64, 4, 2, 10), (639, 0, 7, 6, 33, 10)])
def test_narrow_step_edges(lb, orc, L, p, m, F, n, steps):
    """The narrow step where its shape changes (128, 256 and 320 lags; lists of 8, 16
    and beyond; workgroups of 16 walkers with a remainder): moves, energies,
    candidates and the log against the oracle with the random proposer."""
    lo, hi, seed, ps, every = max(1, L // 10), max(2, L // 5), 19, 77, 3
    r = lb.learned_walk(L, p, steps, lo, hi, seed, n, mode=lb.PROPOSE_RANDOM, top_m=m, fallback_every=F,
                        prop_seed=ps, log_every=every, want_traj=True, want_cands=True)
    traj, moves, cands = _np(r["traj_E"]), _np(r["moves"]), _np(r["cands"])
    seqs, mask, label = _np(r["log_seqs"]), _np(r["log_mask"]), _np(r["log_label"])
    for w in {0, n // 2, n - 1}:
        ref = ol.proposal_walk(L, p, steps, lo, hi, seed, w, F, ol.random_proposer(ps, L, w, m))
        done = len(ref["moves"])
        assert np.array_equal(traj[w, :done], np.array(ref["traj"])[:done]), w
        assert np.array_equal(moves[w, :done], np.array(ref["moves"])), w
        for t, c in enumerate(ref["cands"]):
            assert [int(x) for x in cands[w, t] if x >= 0] == (c if c is not None else []), (w, t)
        for q in range(steps // every):
            t, rec = (q + 1) * every, q * n + w
            if t > done or ref["moves"][t - 1] < 0:
                break
            st = li.unpack(seqs[rec:rec + 1].view(np.uint32), L)[0]
            assert np.array_equal(st, ref["states"][t - 1])
            adm = [a for a in range(1, (L - 1) // 2 + 2)
                   if (int(mask[rec, (a - 1) // 32]) >> ((a - 1) % 32)) & 1]
            assert adm == ref["admissible"][t - 1]
            assert label[rec] == ref["moves"][t - 1] - 1


@pytest.mark.parametrize("L,hidden,n", [(5, 64, 3), (101, 64, 17), (255, 128, 40), (257, 256, 64),
                                        (513, 256, 70), (639, 192, 33)])
def test_network_features_from_the_walk_state(lb, L, hidden, n):
    """The forward pass that builds its features from the walk's state against the
    features kernel and the separate products: the network widened to 320 hidden
    units with zero weights gives the same logits bit for bit, so the walks are equal."""
    import torch
    p, steps, lo, hi = 0, 20, 1, 2
    lay, P, blob, pb = _net(lb, L, hidden, 58)
    wide = lb.mlp_layout(L, 320)
    Q = {key: np.zeros(s, np.float32) for key, s in
         (("W1", (320, lay.d_in)), ("b1", 320), ("W2", (320, 320)), ("b2", 320),
          ("W3", (lay.d_out, 320)), ("b3", lay.d_out))}
    for key in Q:
        Q[key][tuple(slice(0, d) for d in P[key].shape)] = P[key]
    wblob = torch.from_numpy(lb.mlp_blob_from_dict(wide, Q)).cuda()
    wpb = torch.empty(wide.n_params, dtype=torch.bfloat16, device="cuda")
    lb.mlp_cast(wide, wblob, wpb)
    a, b = (lb.learned_walk(L, p, steps, lo, hi, 6, n, mode=lb.PROPOSE_MLP, top_m=8, fallback_every=8,
                            hidden=h, params=x, params_bf16=y, want_traj=True, want_cands=True)
            for h, x, y in ((hidden, blob, pb), (320, wblob, wpb)))
    for key in ("traj_E", "moves", "cands"):
        assert np.array_equal(_np(a[key]), _np(b[key])), key


@pytest.mark.parametrize("m", [5, 12, 20])
def test_equal_scores_take_the_lower_positions(lb, orc, m):
    """A network of zeros scores every position alike: the candidates are the first
    m admissible positions."""
    import torch
    L, p, steps, n, F = 101, 8, 40, 18, 16
    lay = lb.mlp_layout(L, 64)
    blob = torch.zeros(lay.n_params, dtype=torch.float32, device="cuda")
    pb = torch.zeros(lay.n_params, dtype=torch.bfloat16, device="cuda")
    r = lb.learned_walk(L, p, steps, 10, 20, 4, n, mode=lb.PROPOSE_MLP, top_m=m, fallback_every=F, hidden=64,
                        params=blob, params_bf16=pb, want_traj=True, want_cands=True)
    for w in (0, n - 1):
        ref = ol.proposal_walk(L, p, steps, 10, 20, 4, w, F, lambda t, s, adm: sorted(adm)[:m])
        assert np.array_equal(_np(r["traj_E"])[w], np.array(ref["traj"]))
        assert np.array_equal(_np(r["moves"])[w], np.array(ref["moves"]))
        for t, c in enumerate(ref["cands"]):
            assert [int(x) for x in _np(r["cands"])[w, t] if x >= 0] == (c if c is not None else [])


def _admissible(mask_words, d_out):
    mk = mask_words.cpu().numpy().view(np.uint32)
    adm = np.zeros((mk.shape[0], d_out), bool)
    for j in range(d_out):
        adm[:, j] = (mk[:, j // 32] >> np.uint32(j % 32)) & 1
    return adm


def _recall(z, adm, labels, m=8):
    z = np.where(adm, z[:, :adm.shape[1]], -np.inf)
    top = np.argsort(-z, axis=1, kind="stable")[:, :m]
    return float(np.mean([labels[i] in top[i] for i in range(len(labels))]))


def test_trained_network_gains_over_untrained_and_random(lb):
    """What training buys, on held-out plain-walker states at L = 101 (p = 8): the
    trained network's top-8 admissible positions hold the plain walker's move more
    often than an untrained network's or a random top-8, and its held-out
    cross-entropy is lower than the untrained network's.  The gain is small."""
    from paper_2409_07222_amd import learn
    L, p, lo, hi, hidden = 101, 8, 10, 20, 128
    seqs, mask, lab = learn.log_plain(L, p, 400, lo, hi, 5, 4096, 2)
    hs, hm, hl = learn.log_plain(L, p, 400, lo, hi, 6, 512, 20)
    lay = lb.mlp_layout(L, hidden)
    net = learn.Network(L, li.mlp_init(55, lay.d_in, hidden, lay.d_out), hidden)
    untrained = net.clone()
    learn.train(net, seqs, mask, lab, batch=4096, epochs=3, lr=1e-3)
    adm, labels = _admissible(hm, lay.d_out), hl.cpu().numpy()
    r_tr = _recall(net.logits(hs).cpu().numpy(), adm, labels)
    r_un = _recall(untrained.logits(hs).cpu().numpy(), adm, labels)
    r_rand = _recall(li.rng(3).random(adm.shape), adm, labels)
    Xh = lb.mlp_features(L, hs)
    _, loss_tr = lb.mlp_grads(lay, net.params, net.params_bf16, Xh, hm, hl)
    _, loss_un = lb.mlp_grads(lay, untrained.params, untrained.params_bf16, Xh, hm, hl)
    print("recall@8 trained %.3f untrained %.3f random %.3f; held-out loss %.3f vs %.3f"
          % (r_tr, r_un, r_rand, float(loss_tr.item()), float(loss_un.item())))
    # measured: recall 0.360 / 0.283 / 0.301, loss 3.295 / 3.320 (close to the
    # log of the admissible count: the network learns little of the argmin)
    assert r_tr >= max(r_un, r_rand) + 0.03
    assert float(loss_tr.item()) < float(loss_un.item()) - 0.01


def test_single_walker_default_steps(lb):
    """steps = 0 means T_i = 4(L+1), as for the plain walker; one walker, top-1."""
    L, p, lo, hi = 37, 2, 3, 6
    plain = lb.walk_step1(L, p, 0, lo, hi, 9, 1, want_traj=True)
    r = lb.learned_walk(L, p, 0, lo, hi, 9, 1, mode=lb.PROPOSE_RANDOM, top_m=1,
                        fallback_every=1, want_traj=True)
    assert r["traj_E"].shape[1] == 4 * (L + 1)
    assert np.array_equal(_np(r["traj_E"]), _np(plain.traj_E))
    narrow = lb.learned_walk(L, p, 0, lo, hi, 9, 1, mode=lb.PROPOSE_RANDOM, top_m=1,
                             fallback_every=4, want_traj=True)
    assert int(narrow["flip_evals"].item()) < int(r["flip_evals"].item())


@pytest.mark.parametrize("L,p,steps,every", [(7, 1, 9, 2), (101, 8, 24, 5), (301, 12, 12, 4), (513, 255, 10, 3),
                                             (515, 2, 9, 4), (527, 0, 9, 3), (639, 16, 6, 5)])
def test_logging_walk_edges(lb, orc, L, p, steps, every):
    """Every step a full scan (the plain walk's kernel with the log's outputs): records,
    moves, hits, evaluations and candidate rows at the scan kernel's size edges."""
    nf = (L - 1) // 2 + 1 - p
    hi = min(L // 5, nf - 1)
    lo = min(L // 10, hi)
    n, seed = 3, 31 + L
    E0 = [orc.energy(orc.walker_init(seed, L, p, w, lo, hi)[0]) for w in range(n)]
    e_max = min(E0) - 1                      # some walkers hit it on the way down
    r = lb.learned_walk(L, p, steps, lo, hi, seed, n, mode=lb.PROPOSE_RANDOM, top_m=2, fallback_every=1,
                        log_every=every, e_max=e_max, want_traj=True, want_cands=True)
    traj, moves, hit = _np(r["traj_E"]), _np(r["moves"]), _np(r["hit_step"])
    seqs, mask, label = _np(r["log_seqs"]), _np(r["log_mask"]), _np(r["log_label"])
    assert (_np(r["cands"]) == -1).all()
    evals = 0
    for w in range(n):
        ref = ol.proposal_walk(L, p, steps, lo, hi, seed, w, 1, None, e_max=e_max)
        assert np.array_equal(traj[w], np.array(ref["traj"])), w
        assert np.array_equal(moves[w], np.array(ref["moves"])), w
        assert hit[w] == ref["hit_step"]
        evals += sum(len(a) for a in ref["admissible"])
        for q in range(steps // every):
            t, rec = (q + 1) * every, q * n + w
            assert np.array_equal(li.unpack(seqs[rec:rec + 1].view(np.uint32), L)[0], ref["states"][t - 1])
            adm = [a for a in range(1, (L - 1) // 2 + 2)
                   if (int(mask[rec, (a - 1) // 32]) >> ((a - 1) % 32)) & 1]
            assert adm == ref["admissible"][t - 1]
            assert label[rec] == ref["moves"][t - 1] - 1
    assert int(r["flip_evals"].item()) == evals


def test_logging_walk_across_segments(lb):
    """More steps than one launch holds: trajectory, best and records as the plain walk's."""
    L, p, lo, hi, steps, n = 37, 2, 3, 6, 9000, 8
    plain = lb.walk_step1(L, p, steps, lo, hi, 5, n, want_traj=True)
    r = lb.learned_walk(L, p, steps, lo, hi, 5, n, mode=lb.PROPOSE_RANDOM, top_m=1, fallback_every=1,
                        log_every=700, want_traj=True)
    assert np.array_equal(_np(r["traj_E"]), _np(plain.traj_E))
    assert np.array_equal(_np(r["best_step"]), _np(plain.best_step))
    assert np.array_equal(_np(r["best_seqs"]), _np(plain.best_seqs))
    # record q is the state before step 700 (q + 1): its energy is the trajectory's
    E = lb.energy(L, r["log_seqs"]).cpu().numpy().reshape(steps // 700, n)
    traj = _np(plain.traj_E)
    for q in range(steps // 700):
        assert np.array_equal(E[q], traj[:, 700 * (q + 1) - 2])
