"""The dispatch rules' branches against the oracle, each at the sizes where it
can go wrong: the smallest it takes, remainders, and either side of its line."""
import numpy as np
import pytest

from gpu_util import SCORE_REL, assert_argmin, device_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qlm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_00047_amd import qlm as q
    q.library()
    return q


def make(G, I, P, seed, M=4, evict=True, loaded=True, sizes=(16, 128), ld=None):
    """A random problem and plans of any size (fields as workload.make_problem)."""
    from paper_2407_00047_amd import workload
    rng = np.random.default_rng(seed)
    C = min(3, I)
    f = np.float32
    swap = rng.uniform(5.0, 40.0, (C, M, M)).astype(f)
    pr = {"seed": seed, "n_groups": G, "n_instances": I, "n_models": M, "n_classes": C,
          "grp_count": rng.integers(sizes[0], sizes[1] + 1, G).astype(np.int32),
          "grp_mu": rng.uniform(50, 600, G).astype(f), "grp_var": rng.uniform(1e3, 1e5, G).astype(f),
          "grp_model": rng.integers(0, M, G).astype(np.int32),
          "grp_slo": np.where(rng.random(G) < 0.3, 20.0, rng.uniform(100, 2000, G)).astype(f),
          "inst_tput": rng.choice([800.0, 1500.0, 6000.0], I).astype(f),
          "inst_class": rng.integers(0, C, I).astype(np.int32),
          "inst_model0": rng.integers(-1, M, I).astype(np.int32) if loaded else None,
          "swap_cost": swap.reshape(-1), "evict_cost": 2.0 if evict else 0.0,
          "n_evict": max(1, G // 20) if evict else 0}
    return pr, workload.make_plans(pr, 0, P, ld=ld)


# Wavefronts per tile (1 to 16 parts of a plan) and per workgroup: from plans
# too short to split to sixteen parts, one tile to more tiles than wavefronts fit
@pytest.mark.parametrize("G,I,P,evict", [
    (31, 3, 65, True), (64, 2, 200, False), (96, 3, 4100, True), (128, 4, 5000, False),
    (160, 5, 700, True), (511, 8, 300, True), (545, 17, 2049, False), (1024, 16, 130, True),
    (1000, 16, 9001, True), (2048, 16, 70, False), (2051, 5, 333, True), (4096, 64, 1030, True)])
def test_score_parts(qlm, orc, G, I, P, evict):
    import torch
    pr, pl = make(G, I, P, 1000 + G, evict=evict)
    dpr, dpl = device_inputs(pr, pl)
    print("case parts", G, I, P, flush=True)
    res = qlm.rwt_score(dpr, dpl, penalty=True)
    bi, bs = qlm.best_plan(dpr, dpl)
    torch.cuda.synchronize()
    osc, ope = orc.score_plans(pr, pl)
    err = np.abs(res["score"].cpu().numpy() - osc)
    assert np.all(err <= SCORE_REL * dpr.total_requests), err.max()
    # the bound of test_gpu_parity.test_scores_match_oracle
    mag = (ope + pr["grp_slo"].astype(np.float64).sum()) + np.abs(pr["grp_slo"]).sum()
    perr = np.abs(res["penalty"].cpu().numpy() - ope)
    assert np.all(perr <= 2.0 * (2.0 ** -36 + (2 * G + 4) * 2.0 ** -53) * mag), perr.max()
    _, obs = assert_argmin(int(bi.item()), osc, (G, I, P))
    assert abs(float(bs.item()) - obs) <= 1e-12 * abs(obs)


# Seeds: a queue per lane up to 64 queues and the LDS form past them; chunks of
# 512 groups and batches of 64; equal drain times (identical instances and
# groups, groups without tokens) and negative tokens, which the approximate
# comparison leaves to the full one
@pytest.mark.parametrize("G,I,kind", [
    (1, 1, "plain"), (63, 3, "plain"), (65, 64, "plain"), (130, 65, "plain"), (511, 7, "plain"),
    (513, 63, "ties"), (1027, 64, "plain"), (700, 16, "negative"), (600, 5, "no swap"),
    (300, 130, "ties")])
def test_seed_lanes(qlm, orc, G, I, kind):
    import torch
    pr, _ = make(G, I, 1, 77 + G, evict=False)
    rng = np.random.default_rng(G)
    if kind == "ties":
        pr["inst_tput"][:] = 1500.0
        pr["inst_class"][:] = 0
        pr["grp_count"] = rng.choice([0, 8], G).astype(np.int32)
        pr["grp_mu"][:] = 100.0
        pr["swap_cost"][:] = 7.0
    if kind == "negative":
        pr["grp_mu"] = rng.uniform(-300.0, 600.0, G).astype(np.float32)
    if kind == "no swap":
        pr["swap_cost"] = None
    dpr, _ = device_inputs(pr, {"perm": np.zeros((G, 1), np.int32),
                                "qoff": np.zeros((I + 1, 1), np.int32)})
    print("case seeds", G, I, kind, flush=True)
    sp = qlm.seed_plans(dpr, (0, 1))
    torch.cuda.synchronize()
    for k in (0, 1):
        perm, qoff = orc.seed_plan(pr, k)
        assert np.array_equal(sp.perm[:, k].cpu().numpy(), perm)
        assert np.array_equal(sp.qoff[:, k].cpu().numpy(), qoff)


# Per-request screen: segments of 32, 64 and 128 slots; groups of 0 to 3 blocks
# of 32 requests and a remainder; spreads from none to wider than the waits (every
# group sure, some, none); SLOs met exactly, infinite or far apart within a
# group; negative tokens (no sure side)
@pytest.mark.parametrize("G,I,P,kind", [
    (1, 1, 3, "plain"), (40, 3, 130, "plain"), (130, 4, 65, "ragged"), (257, 16, 200, "ragged"),
    (300, 5, 64, "wide"), (200, 6, 70, "none"), (150, 4, 100, "half"), (90, 3, 64, "infinite"),
    (120, 4, 64, "negative"), (600, 9, 9000, "plain"), (513, 64, 26000, "plain")])
def test_fcfs_lists(qlm, orc, G, I, P, kind):
    import torch
    pr, pl = make(G, I, P, 300 + G, sizes=(0, 100) if kind == "ragged" else (32, 64))
    rng = np.random.default_rng(G)
    if kind == "wide":
        pr["grp_var"] = (pr["grp_var"] * 1e4).astype(np.float32)
    if kind == "none":
        pr["grp_var"][:] = 0.0
        pr["grp_mu"] = rng.integers(1, 9, G).astype(np.float32) * 100.0
        pr["inst_tput"][:] = 800.0
    if kind == "half":
        pr["grp_var"][rng.random(G) < 0.5] = 0.0
    if kind == "negative":
        pr["grp_mu"] = rng.uniform(-200.0, 600.0, G).astype(np.float32)
    N = int(pr["grp_count"].sum())
    req = rng.uniform(0.0, 3000.0, N).astype(np.float32)
    if kind == "none":
        req = rng.integers(0, 3000, N).astype(np.float32)       # waits met exactly among them
    if kind == "infinite":
        req[rng.random(N) < 0.2] = np.inf
    dpr, dpl = device_inputs(pr, pl)
    dreq = qlm.device_requests(req)
    print("case fcfs lists", G, I, P, kind, flush=True)
    F = qlm.fcfs_score(dpr, dpl, dreq).cpu().numpy()
    n = min(P, 400)
    S = orc.score_plans_fcfs(pr, pl, req, 0, n) if n < P else orc.score_plans_fcfs(pr, pl, req)
    err = np.abs(F[:n] - S[:n])
    assert np.all(err <= SCORE_REL * N + 1e-9), err.max()
    # chunks of 64 plans change no bit
    m = min(P, 700)
    sub = qlm.DevicePlans(dpl.perm, dpl.qoff, dpl.evict_bits, m)
    whole = qlm.fcfs_score(dpr, sub, dreq)
    small = qlm.fcfs_score(dpr, sub, dreq,
                           ws=qlm.fcfs_workspace(dpr, m, N, chunk_plans=64))
    bi, bs = qlm.fcfs_best_plan(dpr, dpl, dreq)
    some = qlm.fcfs_score_exact(dpr, dpl, dreq, np.arange(n))
    torch.cuda.synchronize()
    assert torch.equal(whole, small)
    X = some.cpu().numpy()
    assert np.all(np.abs(X - S[:n]) <= 1e-12 * (np.abs(S[:n]) + 1.0))
    # one task, several and many: the same bits
    one = qlm.fcfs_score_exact(dpr, dpl, dreq, [int(bi.item())])
    assert float(one[0]) == float(bs[0])
    assert float(one[0]) <= X.min()


# Per-request tails with every request evaluated: groups on either side of a step of
# 8, a half of 16 and a block of 32 requests, of one size and of all of them
@pytest.mark.parametrize("sizes", [(1, 1), (2, 2), (8, 8), (9, 9), (10, 10), (16, 18), (24, 26),
                                   (32, 32), (33, 33), (34, 34), (64, 66), (97, 97), (0, 130)])
def test_fcfs_blocks(qlm, orc, sizes):
    import torch
    G, I, P = 150, 5, 70
    pr, pl = make(G, I, P, 60 + sizes[0], sizes=sizes)
    pr["grp_var"] = (pr["grp_var"] * 1e5).astype(np.float32)
    pr["grp_var"][::7] = 0.0
    N = int(pr["grp_count"].sum())
    req = np.random.default_rng(N).uniform(0.0, 3000.0, N).astype(np.float32)
    dpr, dpl = device_inputs(pr, pl)
    print("case fcfs blocks", sizes, flush=True)
    F = qlm.fcfs_score(dpr, dpl, qlm.device_requests(req))
    torch.cuda.synchronize()
    err = np.abs(F.cpu().numpy() - orc.score_plans_fcfs(pr, pl, req))
    assert np.all(err <= SCORE_REL * N), err.max()


# Per-request sums: tails of some 1e-9 keep their bits, alone in their block (a
# group of one request each) and as the first of 33 requests of which the others are
# late.  The table's lines follow so small a tail to 3e-4 of it (a cell is 0.0117
# wide, Q'' = z Q' there); a sum that rounds each block to 2^-32 or adds it to 32 in
# single precision loses percent of them, or all.
@pytest.mark.parametrize("n", [1, 33])
def test_fcfs_small_tails(qlm, orc, n):
    import torch
    from cases import plans, problem
    I, rng = 300, np.random.default_rng(n)
    theta, head, mu, var = 1000.0, 4, 500.0, 1e5
    groups = [(head, mu, var, 0, 1e9) for _ in range(I)] + [(n, 1.0, 1.0, 0, 1e9) for _ in range(I)]
    pr = problem(groups, [(theta, 0)] * I)
    pl = plans([[[g, I + g] for g in range(I)]] * 3, 2 * I)
    req = np.full(I * (head + n), 1e9, np.float32)
    z = rng.uniform(5.6, 5.95, I)
    mine = np.full((I, n), -1e6, np.float32)             # late, but for the first
    mine[:, 0] = head * mu / theta + z * np.sqrt(head * var) / theta
    req[I * head:] = mine.reshape(-1)
    dpr, dpl = device_inputs(pr, pl)
    print("case fcfs small tails", n, flush=True)
    F = qlm.fcfs_score(dpr, dpl, qlm.device_requests(req))
    torch.cuda.synchronize()
    late = float(I * (n - 1))
    want = orc.score_plans_fcfs(pr, pl, req) - late
    got = F.cpu().numpy() - late
    assert np.all(want > 3e-7)
    assert np.all(np.abs(got - want) <= 2e-3 * want), (got, want)


# Exact per-request scores of many plans: groups of fewer requests than slices,
# queues of more positions than lanes; and the pick among more candidates than a
# wavefront each is right for (every plan tied)
@pytest.mark.parametrize("G,I,P,sizes", [(70, 1, 130, (1, 1)), (200, 3, 300, (0, 9)),
                                         (150, 2, 64, (63, 65)), (64, 64, 129, (16, 130))])
def test_fcfs_exact_many(qlm, orc, G, I, P, sizes):
    import torch
    pr, pl = make(G, I, P, 90 + G, sizes=sizes)
    N = int(pr["grp_count"].sum())
    req = np.random.default_rng(G).uniform(0.0, 3000.0, N).astype(np.float32)
    dpr, dpl = device_inputs(pr, pl)
    print("case fcfs exact many", G, I, P, flush=True)
    X = qlm.fcfs_score_exact(dpr, dpl, qlm.device_requests(req), np.arange(P))
    never = qlm.device_requests(np.full(N, 1e9, np.float32))
    bi, bs = qlm.fcfs_best_plan(dpr, dpl, never)
    torch.cuda.synchronize()
    S = orc.score_plans_fcfs(pr, pl, req)
    assert np.all(np.abs(X.cpu().numpy() - S) <= 1e-12 * (np.abs(S) + 1.0))
    assert int(bi.item()) == 0 and float(bs.item()) == 0.0


# Validation: 1 to 64 plans a workgroup (by plan count and by the bitmaps' size) and
# a smaller workgroup per plan past them; each kind of malformed plan at the tile's edges
@pytest.mark.parametrize("G,I,P,ld", [
    (1, 1, 5, 5), (33, 4, 4097, 4100), (64, 1, 9000, 9000), (500, 9, 16500, 16501),
    (300, 9, 33000, 33000), (5000, 16, 70, 70), (25000, 3, 33, 40), (170000, 2, 3, 3),
    (25000, 5, 1, 1), (16001, 5, 17, 17), (9000, 3, 127, 127), (9000, 3, 128, 130),
    (170000, 2, 129, 129)])
def test_validate_tiles(qlm, G, I, P, ld):
    import torch
    pr, pl = make(G, I, P, 900 + G, ld=ld)
    rng = np.random.default_rng(G)
    want = np.zeros(P, np.int32)
    for p in {0, P - 1, P // 2, min(63, P - 1), min(64, P - 1)}:
        if G > 1:
            kind = int(rng.integers(0, 4))
            if kind == 0:
                pl["perm"][G - 1, p] = pl["perm"][0, p]
            elif kind == 1:
                pl["perm"][int(rng.integers(0, G)), p] = [-1, G][int(rng.integers(0, 2))]
            if kind <= 1:
                want[p] |= 2
            if kind == 2:
                pl["qoff"][I, p] = G - 1
                want[p] |= 1
        if G % 32 and (G == 1 or kind == 3):
            pl["evict_bits"][-1, p] |= np.uint32(1) << np.uint32(G % 32)
            want[p] |= 4
    dpr, dpl = device_inputs(pr, pl)
    print("case validate", G, I, P, flush=True)
    n, status = qlm.validate_plans(dpr, dpl)
    torch.cuda.synchronize()
    assert np.array_equal(status.cpu().numpy(), want)
    assert int(n.item()) == int((want != 0).sum())


# Search: after the first step only the two changed queues are screened.  Every
# step equals a search of one step (which screens everything) from the plan it
# left: relocations that set flags, emptied and skewed queues (workgroups that loop),
# one queue of nearly all groups (more workgroups than a mean queue's), more queues
# and wider windows than a wavefront, one queue, no window
@pytest.mark.parametrize("G,I,W,steps,kind", [
    (1, 1, 2, 2, "plain"), (30, 3, 4, 14, "evict"), (64, 9, 0, 10, "empty"), (90, 1, 70, 6, "plain"),
    (200, 70, 3, 8, "evict"), (300, 4, 8, 12, "skewed"), (500, 12, 16, 8, "evict"),
    (1500, 16, 2, 5, "heavy")])
def test_search_incremental(qlm, G, I, W, steps, kind):
    import torch
    P = 3
    pr, pl = make(G, I, P, 500 + G, evict=kind != "plain")
    rng = np.random.default_rng(G)
    pr["evict_cost"] = 0.5
    pr["grp_slo"] = rng.choice([5.0, 20.0, 60.0, 400.0], G).astype(np.float32)
    if kind == "heavy":                          # nearly all groups in one queue
        for p in range(P):
            pl["qoff"][1:I, p] = np.where(np.arange(1, I) <= 5 * p, np.arange(1, I), G - I +
                                          np.arange(1, I))
    if kind in ("empty", "skewed"):
        for p in range(P):
            cuts = np.sort(rng.integers(0, G + 1, I - 1)) if kind == "empty" else \
                np.minimum(G, np.arange(1, I) * 2)
            pl["qoff"][1:I, p] = cuts
    dpr, dpl = device_inputs(pr, pl)
    print("case search", G, I, W, kind, flush=True)
    whole = qlm.local_search(dpr, dpl, W, steps, trace=True)
    torch.cuda.synchronize()
    cur, trace = dpl, []
    for _ in range(steps):
        one = qlm.local_search(dpr, cur, W, 1, trace=True)
        torch.cuda.synchronize()
        cur = one["plans"]
        trace.append(one["trace"][:, 0].cpu().numpy())
    assert np.array_equal(whole["trace"].cpu().numpy(), np.stack(trace, 1))
    for name in ("perm", "qoff", "evict_bits"):
        assert torch.equal(getattr(whole["plans"], name), getattr(cur, name)), name
    assert torch.equal(whole["score"], one["score"])
    exact = qlm.rwt_score_exact(dpr, cur, np.arange(P))
    assert torch.equal(exact, whole["score"])
    if kind == "evict":
        assert int((whole["trace"] >= G * (W + I)).sum()) > 0       # a relocation among them


# Placements at the line where queues become many (the group's queue by a search, the
# queue scores' running sums kept) and past it
@pytest.mark.parametrize("I", [1024, 1025, 2100])
def test_place_many_queues(qlm, orc, I):
    import torch
    G, P = 3000, 2
    pr, pl = make(G, I, P, 800 + I)
    dpr, dpl = device_inputs(pr, pl)
    for group in (0, 1, G // 2, G - 1):
        print("case place many", I, group, flush=True)
        r = qlm.place_group(dpr, dpl, group)
        torch.cuda.synchronize()
        out = r["plans"]
        for p in range(P):
            o = orc.place_group(pr, pl, p, group)
            assert int(r["queue"][p]) == o["queue"]
            assert np.array_equal(out.perm[:, p].cpu().numpy(), o["perm"])
            assert np.array_equal(out.qoff[:, p].cpu().numpy(), o["qoff"])
        assert torch.equal(qlm.rwt_score_exact(dpr, out, np.arange(P)), r["score"])


# The general walk in parts: groups without requests or variance, counts and
# models beyond the compact records; penalties and detail across the parts
@pytest.mark.parametrize("G,I,P,kind", [
    (31, 3, 65, "zero"), (128, 4, 5000, "zero"), (1000, 16, 300, "zero"), (1024, 1, 70, "zero"),
    (2051, 5, 333, "counts"), (600, 1, 130, "models"), (512, 16, 20000, "zero"),
    (700, 64, 200, "same")])
def test_general_parts(qlm, orc, G, I, P, kind):
    import torch
    many = kind == "models"                  # (their costs leave LDS for one class)
    pr, pl = make(G, I, P, 700 + G, M=66 if many else 4, evict=not many)
    rng = np.random.default_rng(G)
    if kind == "zero":
        pr["grp_count"][rng.random(G) < 0.1] = 0
        pr["grp_var"][rng.random(G) < 0.3] = 0.0
    if kind == "counts":
        pr["grp_count"][0] = 5000
    if kind == "same":                       # whole-second waits that meet SLOs exactly
        pr["grp_var"][:] = 0.0
        pr["grp_count"][:] = 8
        pr["grp_mu"][:] = 750.0
        pr["inst_tput"][:] = 6000.0
        pr["swap_cost"][:] = 4.0
        pr["grp_slo"] = rng.integers(0, 60, G).astype(np.float32)
    dpr, dpl = device_inputs(pr, pl)
    print("case general", G, I, P, kind, flush=True)
    assert qlm.score_form(dpr, not many) == 0
    d = min(P, 66)
    res = qlm.rwt_score(dpr, dpl, penalty=True, detail=(P - d, d))
    bi, bs = qlm.best_plan(dpr, dpl)
    torch.cuda.synchronize()
    osc, ope = orc.score_plans(pr, pl)
    err = np.abs(res["score"].cpu().numpy() - osc)
    assert np.all(err <= SCORE_REL * dpr.total_requests), err.max()
    mag = (ope + pr["grp_slo"].astype(np.float64).sum()) + np.abs(pr["grp_slo"]).sum()
    perr = np.abs(res["penalty"].cpu().numpy() - ope)
    assert np.all(perr <= 2.0 * (2 * G + 4) * 2.0 ** -53 * mag + 1e-300), perr.max()
    from gpu_util import assert_close_detail
    out = [res[k].cpu().numpy() for k in ("wait_mean", "wait_sd", "prob")]
    for q in (0, d // 2, d - 1):
        ref = orc.plan_detail(pr, pl, P - d + q)
        assert_close_detail([x[:, q] for x in out], ref, G, (G, I, q))
        zero = ref["wait_sd"] == 0
        assert np.array_equal(out[2][zero, q], ref["prob"][zero])
    _, obs = assert_argmin(int(bi.item()), osc, (G, I, P))
    assert abs(float(bs.item()) - obs) <= 1e-12 * abs(obs)


# The best plan's candidates: few and many, selected by the re-score itself (up to
# 1024 plans) or listed before; every plan tied, one best, none (NaN scores); a
# workspace whose queue sums hold fewer candidates than there are
@pytest.mark.parametrize("G,I,P,kind", [
    (8, 1, 1, "tie"), (8, 1, 256, "tie"), (40, 3, 1024, "tie"), (40, 3, 1025, "tie"),
    (40, 3, 1024, "one"), (64, 64, 700, "one"), (64, 64, 1500, "tie"), (20, 2, 300, "nan"),
    (20, 2, 2000, "nan")])
def test_best_plan_candidates(qlm, orc, G, I, P, kind):
    import torch
    pr, pl = make(G, I, P, 40 + P + G)
    if kind == "tie":
        pr["grp_slo"][:] = 1e9               # no plan violates anything
    if kind == "nan":
        pr["grp_mu"][:] = np.nan
    dpr, dpl = device_inputs(pr, pl)
    print("case candidates", G, I, P, kind, flush=True)
    for _ in range(3):                       # (the counts start anew in every call)
        bi, bs = qlm.best_plan(dpr, dpl)
        si, ss = qlm.best_plan_static(dpr, dpl)
    torch.cuda.synchronize()
    assert int(bi.item()) == int(si.item()) and (float(bs) == float(ss) or kind == "nan")
    if kind == "nan":
        return                               # (unspecified, and it returns)
    osc, _ = orc.score_plans(pr, pl)
    _, obs = assert_argmin(int(bi.item()), osc, (G, I, P))
    assert abs(float(bs.item()) - obs) <= 1e-12 * abs(obs)


# The grid's occupancies are kept by sizes, and no more than 4096 of them: group counts
# past that many, then an early one again
def test_many_group_counts(qlm, orc):
    import ctypes
    import torch
    G = 6000
    pr, pl = make(G, 1, 64, 5, evict=False)
    dpr, dpl = device_inputs(pr, pl)
    # the identity order, of which a problem of n groups takes the first n
    dpl.perm.copy_(torch.arange(G, dtype=torch.int32, device="cuda")[:, None].expand(G, 64))
    lib, ws = qlm.library(), qlm.workspace(dpr, 64)
    out = (torch.empty(1, dtype=torch.int64, device="cuda"),
           torch.empty(1, dtype=torch.float64, device="cuda"))
    first = None
    for n in [40] + list(range(41, 4600)) + [40]:
        sub = qlm.Problem.from_buffer_copy(dpr.struct)
        sub.n_groups = n
        dpl.qoff[1:] = n
        assert lib.qlm_best_plan(ctypes.byref(sub), ctypes.byref(dpl.struct), ws.data_ptr(),
                                 ws.numel(), out[0].data_ptr(), out[1].data_ptr(), None) == 0
        if n == 40:
            torch.cuda.synchronize()
            score = float(out[1].item())
            assert first is None or score == first
            first = score
    torch.cuda.synchronize()
