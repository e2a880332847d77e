"""Parity of the HIP library against the CPU oracle, through the C ABI.

Tolerances: 1e-5 relative (denominator max(|ref|, 1e-6)) on expected
accuracies, keys, scores and utilities for float32 features; for the bfloat16
config 2e-3 on posteriors (absolute) and on EA.  Decisions must match exactly
or be tolerance ties as defined in tests/parity.py.
"""
import copy

import numpy as np
import pytest

from oracle import sneakpeek_oracle as orc
from paper_2505_06641_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

TOL = 1e-5
BF16_EA_DERIVED = 1e-5      # bound on EA and key errors of the bf16 kernels that follows from their arithmetic


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu-marked tests need a real MI355X")
    from paper_2505_06641_amd import binding
    binding.load_library()
    return torch, binding


def run_window(gpu, w, max_rounds, ctx=None, want_cube=False, policy=None, n_groups=None):
    """Score + schedule one workload through the C ABI; everything back on the host."""
    torch, binding = gpu
    p, rq = w.profile, w.requests
    n = rq.n
    own = ctx is None
    if own:
        ctx = binding.Context(p, max(n, 1), policy=policy)
    x, app, D, wt = binding.to_device(rq)
    ea = torch.full((n, ctx.m_max), -7.0, device="cuda:0")
    key = torch.full((n,), -7.0, device="cuda:0")
    ctx.sp_score(x, app, D, wt, ea_out=ea, key_out=key)
    out = {"ctx": ctx}
    order = torch.zeros(max(n, 1), dtype=torch.int32, device="cuda:0")
    seg = torch.zeros(p.n_apps + 1, dtype=torch.int32, device="cuda:0")
    ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
    ctx.sp_debug_dump(binding.SP_DUMP_SEGMENTS, seg)
    out["order"], out["seg"] = order.cpu().numpy()[:n], seg.cpu().numpy()
    if want_cube:
        cube = torch.zeros((n_groups or p.n_apps, ctx.m_max, p.max_batch), device="cuda:0")
        ctx.sp_debug_dump(binding.SP_DUMP_SCORE_CUBE, cube)
        out["cube"] = cube.cpu().numpy()
    model = torch.full((max(n, 1),), 99, dtype=torch.int32, device="cuda:0")
    rnd = torch.full((max(n, 1),), 99, dtype=torch.int32, device="cuda:0")
    ordr = torch.full((max(n, 1),), 99, dtype=torch.int32, device="cuda:0")
    util = torch.full((max(n, 1),), -7.0, device="cuda:0")
    rc, summ, log = ctx.sp_schedule(max_rounds, model, rnd, ordr, util, log_capacity=max(n, 1))
    out.update(rc=rc, summary=summ, log=log, ea=ea.cpu().numpy(), key=key.cpu().numpy(),
               model=model.cpu().numpy()[:n], round_of=rnd.cpu().numpy()[:n], order_of=ordr.cpu().numpy()[:n],
               util=util.cpu().numpy()[:n], x=x, app=app)
    if own:
        out["close"] = ctx.close
    return out


def full_parity(gpu, w, max_rounds, tol=TOL, ea_tol=None, want_cube=False, policy=None):
    torch, binding = gpu
    p, rq = w.profile, w.requests
    sub, n_groups, border = None, None, []
    if policy is not None and getattr(policy, "split_groups", 0):
        # Subgroup labels (Sec. 5.3.2) from the head's own posterior.  The library sees every request.  Rule
        # for labels: they must equal the oracle's, except for requests whose largest oracle probability is
        # within 1e-4 of one half, where float32 and float64 may legitimately fall on different sides: for
        # those (`border`) either label is accepted, and the one the library took is read off its order.
        plain = copy.copy(p)
        plain.prior_alpha = None
        _, _, thetas = orc.score_requests(plain, rq, return_theta=True)
        top = np.array([float(np.max(t)) for t in thetas])
        arg = np.array([int(np.argmax(t)) for t in thetas])
        border = [int(i) for i in np.nonzero(np.abs(top - 0.5) <= 1e-4)[0]]
        assert len(border) <= 10, "too many requests at the labelling threshold for this test to resolve"
        sub = orc.split_labels(thetas)
        n_groups = len(set(zip(rq.app.tolist(), sub.tolist()))) + len(border)
    ea_ref, key_ref = orc.score_requests(p, rq)
    got = run_window(gpu, w, max_rounds, want_cube=want_cube, policy=policy, n_groups=n_groups)
    if border:
        # the labelling of the borderline requests that reproduces the library's order, if there is one
        def order_of(labels):
            w0 = orc.Window(p, rq, ea=ea_ref, key=key_ref, policy=policy, sub=labels)
            return np.concatenate([w0.order[g] for a in range(p.n_apps) for g in range(w0.G) if w0.gapp[g] == a])
        found = None
        for bits in range(1 << len(border)):
            trial = sub.copy()
            for k, i in enumerate(border):
                trial[i] = 1 + arg[i] if (bits >> k) & 1 else 0
            if np.array_equal(order_of(trial), got["order"][:got["seg"][p.n_apps]]):
                found = trial
                break
        assert found is not None, "no admissible labelling of the borderline requests gives the library's order"
        sub = found
    if sub is not None:
        n_groups = len(set(zip(rq.app.tolist(), sub.tolist())))
        if want_cube:
            got["cube"] = got["cube"][:n_groups]
    stats = {}
    stats["ea_rel"] = parity.assert_close("EA", got["ea"], ea_ref, ea_tol or tol)
    stats["key_rel"] = parity.assert_close("key", got["key"], key_ref, ea_tol or tol, floor=1e-30)
    # bfloat16 configs are allowed 2e-3 (ea_tol), but the arithmetic says they do as well as float32 ones:
    # bf16 features and weights are exact in both implementations, layer 1 multiplies them exactly and
    # accumulates in float32, the hidden activations stay float32, so only float32 roundings remain
    assert stats["ea_rel"] <= BF16_EA_DERIVED and stats["key_rel"] <= BF16_EA_DERIVED, stats
    edf = policy is not None and policy.order == wl.ORDER_EDF
    omega = -orc.widen(rq.deadline_rel_ms) if edf else key_ref
    if sub is None:
        stats["order_swaps"] = parity.check_order(got["order"], got["seg"], rq.app, omega, p.n_apps, tol)
    else:
        # inside an application: subgroups in ascending order, each by descending ordering value
        w0 = orc.Window(p, rq, ea=ea_ref, key=key_ref, policy=policy, sub=sub)
        for a in range(p.n_apps):
            want = np.concatenate([w0.order[g] for g in range(w0.G) if w0.gapp[g] == a] or [np.zeros(0, dtype=np.int64)])
            have = got["order"][got["seg"][a]:got["seg"][a + 1]]
            assert np.array_equal(have, want), f"app {a}: order inside the subgroups differs"
        stats["order_swaps"] = 0
    if want_cube:
        ref_cube = orc.Window(p, rq, ea=ea_ref, key=key_ref, policy=policy, sub=sub).score_cube()
        valid = np.isfinite(ref_cube)
        assert np.array_equal(got["cube"] >= 0, valid), "candidate sets differ"
        stats["cube_rel"] = parity.assert_close("score cube", got["cube"][valid], ref_cube[valid], tol, floor=1e-12)
    members = parity.members_by_round(got["round_of"], got["order_of"], len(got["log"]))
    win, rstats = parity.replay(p, rq, ea_ref, key_ref, got["log"], members, got["summary"]["done"] == 1, tol,
                                policy=policy, sub=sub)
    stats.update(rstats)
    stats["util_rel"] = parity.check_outputs(win, got["model"], got["round_of"], got["order_of"], got["util"],
                                             got["summary"], tol)
    got["close"]()
    got["workload"] = w
    print(w.name, stats)
    return got, stats


def test_cfg1_scoring_cube_and_one_round(gpu):
    torch, binding = gpu
    w = wl.make("cfg1")
    got, stats = full_parity(gpu, w, max_rounds=1, want_cube=True)
    assert got["rc"] == binding.SP_OK and got["summary"]["n_rounds"] == 1
    assert stats["ties"] == 0 and stats["order_swaps"] == 0


def test_cfg2_full_schedule(gpu):
    torch, binding = gpu
    w = wl.make("cfg2")
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
    assert got["rc"] == binding.SP_DONE and got["summary"]["done"] == 1
    assert stats["exact"] + stats["ties"] == got["summary"]["n_rounds"] > 10
    assert stats["ties"] <= 2


def test_cfg3_full_schedule_tight_deadlines(gpu):
    torch, binding = gpu
    w = wl.make("cfg3")
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
    assert got["rc"] == binding.SP_DONE
    assert got["summary"]["n_dropped"] > 0 and got["summary"]["n_scheduled"] > 0
    assert stats["ties"] <= 2


def test_cfg4_bf16_posteriors_and_rounds(gpu):
    torch, binding = gpu
    w = wl.make("cfg4")
    p, rq = w.profile, w.requests
    got, stats = full_parity(gpu, w, max_rounds=64, ea_tol=2e-3, want_cube=True)
    # the queue may run dry before the 64th round (replay has already checked that it really is dry)
    assert got["summary"]["n_rounds"] == 64 or (got["rc"] == binding.SP_DONE and 0 < got["summary"]["n_rounds"] < 64)
    # posteriors from the library's logits against the oracle's, on a sample of requests
    ctx = binding.Context(p, rq.n)
    x, app, D, wt = binding.to_device(rq)
    ctx.sp_score(x, app, D, wt)
    z = torch.zeros((rq.n, ctx.c_max), device="cuda:0")
    ctx.sp_debug_dump(binding.SP_DUMP_LOGITS, z, x=x, app=app)
    z = z.cpu().numpy()
    ctx.close()
    sample = np.random.default_rng(0).choice(rq.n, 2048, replace=False)
    for a in range(p.n_apps):
        ids = sample[rq.app[sample] == a]
        th_ref = orc.posterior(orc.head_logits(rq.x[ids], p.W1[a], p.b1[a], p.W2[a], p.b2[a]))
        th_got = orc.posterior(z[ids, : p.n_classes[a]])
        assert np.max(np.abs(th_got - th_ref)) <= 2e-3


@pytest.mark.parametrize("kind", [wl.PEN_STEP, wl.PEN_LINEAR, wl.PEN_SIGMOID])
def test_ragged_applications_all_penalties(gpu, kind):
    w = wl.tiny(seed=40 + kind, n=3000, classes=(5, 1, 130, 2), models=(3, 1, 16, 7), max_batch=37, feat_dim=19,
                hidden_dim=0, penalty=kind, deadline=(4.0, 60.0), fractions=(0.4, 0.1, 0.3, 0.2))
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
    assert got["summary"]["done"] == 1


def test_ragged_mlp_head(gpu):
    w = wl.tiny(seed=50, n=1500, classes=(3, 70), models=(2, 5), max_batch=8, feat_dim=33, hidden_dim=17,
                deadline=(4.0, 80.0))
    full_parity(gpu, w, max_rounds=0, want_cube=True)


def test_bf16_ragged(gpu):
    w = wl.tiny(seed=51, n=700, classes=(3, 9), models=(2, 3), max_batch=5, feat_dim=24, hidden_dim=10,
                feat_dtype=wl.BF16, deadline=(4.0, 80.0))
    full_parity(gpu, w, max_rounds=0, ea_tol=2e-3)


@pytest.mark.parametrize("head", ["logistic", "mlp_f32", "mlp_bf16"])
def test_dirichlet_priors_on_every_scoring_kernel(gpu, head):
    """Sec. 4.2 eq. (10)-(11): priors of the three kinds of Sec. 6.3 and one application without a prior."""
    kw = dict(classes=(5, 12, 130, 2), models=(3, 1, 16, 7), max_batch=9, deadline=(4.0, 60.0), fractions=(0.4, 0.1, 0.3, 0.2))
    if head == "logistic":
        w = wl.tiny(seed=90, n=2500, feat_dim=19, hidden_dim=0, **kw)
    elif head == "mlp_f32":
        w = wl.tiny(seed=91, n=1200, feat_dim=33, hidden_dim=17, **kw)
    else:
        w = wl.tiny(seed=92, n=1500, feat_dim=24, hidden_dim=10, feat_dtype=wl.BF16, **kw)
    wl.attach_priors(w.profile, seed=93)
    plain, _ = orc.score_requests(wl.tiny(seed=w.seed, n=w.requests.app.shape[0], feat_dim=w.profile.feat_dim,
                                          hidden_dim=w.profile.hidden_dim, feat_dtype=w.profile.feat_dtype, **kw).profile,
                                  w.requests)
    smooth, _ = orc.score_requests(w.profile, w.requests)
    assert np.max(np.abs(plain - smooth)) > 1e-3          # the priors do move the estimates
    full_parity(gpu, w, max_rounds=0, ea_tol=2e-3 if head == "mlp_bf16" else None, want_cube=head != "mlp_bf16")


@pytest.mark.parametrize("name", ["sneakpeek", "alg1"])
def test_data_oblivious_baselines_are_a_prior_without_evidence(gpu, name):
    """Sec. 6.1: the data-oblivious approaches use the profiled accuracy under the profiling label mix for
    every request of an application: a prior equal to that mix and no evidence (Sec. 4.1, fallback of eq. 9)."""
    w = wl.tiny(seed=96, n=1800, classes=(5, 12, 40), models=(3, 2, 6), max_batch=7, feat_dim=21, deadline=(4.0, 90.0))
    wl.attach_priors(w.profile, seed=97, kinds=("weak", "strong"))
    w.profile.evidence_k[:] = 0.0
    ea_ref, _ = orc.score_requests(w.profile, w.requests)
    for a in range(3):
        rows = ea_ref[w.requests.app == a]
        assert np.ptp(rows, axis=0).max() == 0.0          # one row per application, whatever the request holds
    full_parity(gpu, w, max_rounds=0, policy=wl.named_policy(name), want_cube=True)


def test_prior_can_be_removed_and_bad_priors_are_rejected(gpu):
    torch, binding = gpu
    w = wl.tiny(seed=94, n=300, classes=(4, 6), models=(2, 3), max_batch=4, feat_dim=8)
    ea_plain, _ = orc.score_requests(w.profile, w.requests)
    ctx = binding.Context(w.profile, 300)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_set_prior(1, np.array([2.0, 0.5, 0.5, 1.0, 3.0, 0.25], dtype=np.float32), 5.0)
    ea = torch.zeros((300, ctx.m_max), device="cuda:0")
    ctx.sp_score(x, app, D, wt, ea_out=ea)
    ea1 = ea.cpu().numpy()
    ctx.sp_set_prior(1, None, 0.0)
    ctx.sp_score(x, app, D, wt, ea_out=ea)
    ea2 = ea.cpu().numpy()
    assert np.max(np.abs(ea1 - ea_plain)) > 1e-3
    parity.assert_close("EA", ea2, ea_plain, TOL)
    for bad_alpha, k in (([1.0, -0.1, 1.0, 1.0], 1.0), ([1.0, float("nan"), 1.0, 1.0], 1.0), ([0.0] * 4, 0.0),
                         ([1.0] * 4, -1.0)):
        with pytest.raises(binding.SneakPeekError) as e:
            ctx.sp_set_prior(0, np.asarray(bad_alpha, dtype=np.float32), k)
        assert e.value.status == binding.SP_EINVAL
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_set_prior(2, np.ones(4, dtype=np.float32), 1.0)
    assert e.value.status == binding.SP_EINVAL
    ctx.close()


def test_batch_of_one(gpu):
    w = wl.tiny(seed=52, n=200, classes=(4, 3), models=(3, 2), max_batch=1, feat_dim=8, deadline=(3.0, 40.0))
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
    assert all(r["batch"] == 1 for r in got["log"])


def test_fewer_requests_than_batch_and_single_request(gpu):
    for n in (1, 3):
        w = wl.tiny(seed=60 + n, n=n, classes=(4,), models=(2,), max_batch=16, feat_dim=8, deadline=(50.0, 90.0))
        got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
        assert got["summary"]["n_scheduled"] == n


def test_empty_window(gpu):
    torch, binding = gpu
    w = wl.tiny(seed=70, n=0, classes=(4, 2), models=(2, 2))
    got = run_window(gpu, w, max_rounds=0)
    assert got["rc"] == binding.SP_DONE
    assert got["summary"] == {"total_weighted_utility": 0.0, "mean_utility": 0.0, "total_violation_ms": 0.0,
                              "n_rounds": 0, "n_scheduled": 0, "n_dropped": 0, "done": 1}
    rc, dec = got["ctx"].sp_greedy_round()
    assert rc == binding.SP_DONE and dec is None
    got["close"]()


def test_all_dead_queue(gpu):
    torch, binding = gpu
    w = wl.tiny(seed=71, n=50, classes=(4,), models=(2,), penalty=wl.PEN_STEP, deadline=(0.01, 0.02))
    got, stats = full_parity(gpu, w, max_rounds=0)
    assert got["summary"]["n_scheduled"] == 0 and got["summary"]["n_dropped"] == 50 and got["rc"] == binding.SP_DONE
    assert np.all(got["model"] == -1) and np.all(got["round_of"] == -1) and np.all(got["order_of"] == 0)


def test_duplicate_keys_fall_back_to_request_id(gpu):
    w = wl.tiny(seed=72, n=400, classes=(3, 2), models=(2, 2), max_batch=6, feat_dim=4, deadline=(30.0, 30.0))
    rq = w.requests
    rq.x[:] = rq.x[0]                       # identical features -> identical EA within an application
    rq.deadline_rel_ms[:] = 30.0
    rq.weight[:] = np.float32(0.5)
    got, stats = full_parity(gpu, w, max_rounds=0)
    for a in range(2):
        mine = got["order"][got["seg"][a]:got["seg"][a + 1]]
        assert np.all(np.diff(mine) > 0)     # equal keys: ascending request id


@pytest.mark.parametrize("head", ["generic", "mfma"])
def test_weight_of_negative_zero_sorts_with_the_zeros(gpu, head):
    # a weight of -0.0 gives the key 0 like +0.0: such requests are served last in their application, by id
    if head == "generic":
        w = wl.tiny(seed=73, n=300, classes=(3, 2), models=(2, 2), max_batch=6, feat_dim=4, hidden_dim=3)
    else:
        w = wl.tiny(seed=74, n=300, classes=(5, 2), models=(3, 2), max_batch=6, feat_dim=8)
    rq = w.requests
    rq.weight[1::7] = np.float32(0.0)
    rq.weight[::5] = np.float32(-0.0)
    zero = rq.weight == 0
    assert np.signbit(rq.weight[::5]).all() and not np.signbit(rq.weight[1::35][rq.weight[1::35] == 0]).all()
    got, stats = full_parity(gpu, w, max_rounds=0)
    assert np.all(got["key"] == 0.0) or np.any(got["key"] > 0)
    assert not np.signbit(got["key"]).any()
    for a in range(2):
        mine = got["order"][got["seg"][a]:got["seg"][a + 1]]
        nz = int(np.sum(zero[mine]))
        assert nz > 0 and zero[mine[-nz:]].all() and not zero[mine[:-nz]].any()
        assert np.all(np.diff(mine[-nz:]) > 0)


def test_exact_score_ties_pick_smallest_candidate(gpu):
    w = wl.tiny(seed=900, n=6, classes=(3, 3), models=(2, 2), max_batch=2, deadline=(1e3, 1e3))
    p, r = w.profile, w.requests
    r.app[:] = [0, 1, 0, 1, 0, 1]
    r.x[1::2] = r.x[0::2]
    r.deadline_rel_ms[:] = 1e3
    r.weight[:] = 0.5
    p.W1[1][:] = p.W1[0]
    p.acc[0][1] = p.acc[0][0]
    p.acc[1][:] = p.acc[0]
    p.lat_ms[1][:] = p.lat_ms[0]
    got, stats = full_parity(gpu, w, max_rounds=1, want_cube=True)
    c = got["cube"]
    assert c[0, 0, 1] == c[0, 1, 1] == c[1, 0, 1] == c[1, 1, 1]
    assert (got["log"][0]["app"], got["log"][0]["model"], got["log"][0]["batch"]) == (0, 0, 2)


def test_short_circuit_variant(gpu):
    w = wl.tiny(seed=800, n=4, classes=(3,), models=(2,), max_batch=2, penalty=wl.PEN_STEP, deadline=(10.0, 10.0))
    w.requests.deadline_rel_ms[:] = 10.0
    w.profile.acc[0][0, :] = 0.9
    w.profile.acc[0][1, :] = 0.4
    w.profile.lat_ms[0][1, :] = 0.0
    w.profile.lat_ms[0][0, :] = [50.0, 60.0]
    got, stats = full_parity(gpu, w, max_rounds=1)
    assert got["log"][0]["model"] == 1 and got["log"][0]["t_end_ms"] == 0.0


def test_round_by_round_equals_schedule_and_is_deterministic(gpu):
    torch, binding = gpu
    w = wl.make("cfg2", n_requests=1500)
    a = run_window(gpu, w, max_rounds=0)
    b = run_window(gpu, w, max_rounds=0)
    for k in ("ea", "key", "order", "model", "round_of", "order_of", "util"):
        assert np.array_equal(a[k], b[k]), k
    assert a["log"] == b["log"] and a["summary"] == b["summary"]
    # the same window stepped one round at a time, with the member ids of every round
    ctx = b["ctx"]
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt)
    ids = torch.zeros(w.profile.max_batch, dtype=torch.int32, device="cuda:0")
    members = parity.members_by_round(a["round_of"], a["order_of"], len(a["log"]))
    for r, rec in enumerate(a["log"]):
        rc, dec = ctx.sp_greedy_round(req_ids_out=ids)
        assert rc == binding.SP_OK and dec == rec
        assert np.array_equal(ids.cpu().numpy()[: rec["batch"]], members[r])
    rc, dec = ctx.sp_greedy_round()
    assert rc == binding.SP_DONE
    # resumable: a limited run followed by an unlimited one gives the same log
    ctx.sp_score(x, app, D, wt)
    rc, s1, log1 = ctx.sp_schedule(5, log_capacity=4096)
    assert rc == binding.SP_OK and s1["n_rounds"] == 5 and log1 == a["log"][:5]
    rc, s2, log2 = ctx.sp_schedule(0, log_capacity=4096)
    assert rc == binding.SP_DONE and log2 == a["log"] and s2 == a["summary"]
    a["close"]()
    b["close"]()


@pytest.mark.parametrize("name", ["alg1", "lo_priority", "lo_edf", "maxacc_edf", "edf_batched", "capped"])
def test_policies_of_the_evaluation_on_both_round_paths(gpu, name):
    """Sec. 6.1 "Baselines and Metrics" and Alg. 1 as printed, as knobs on the same kernels."""
    torch, binding = gpu
    policy = {"edf_batched": wl.Policy(order=wl.ORDER_EDF, weight=wl.WEIGHT_UNIT),
              "capped": wl.Policy(batch_cap=5, choice=wl.CHOICE_MAX_ACCURACY)}.get(name) or wl.named_policy(name)
    n = 600 if policy.batch_cap == 1 else 2400
    w = wl.tiny(seed=97, n=n, classes=(5, 3, 40, 2), models=(3, 2, 8, 5), max_batch=19, feat_dim=19,
                penalty=wl.PEN_LINEAR, deadline=(6.0, 150.0), fractions=(0.4, 0.1, 0.3, 0.2))
    w.profile.penalty[:] = [wl.PEN_LINEAR, wl.PEN_STEP, wl.PEN_SIGMOID, wl.PEN_LINEAR]
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True, policy=policy)      # rounds in one launch
    assert got["summary"]["done"] == 1 and stats["rounds"] > 10
    if policy.batch_cap:
        assert max(r["batch"] for r in got["log"]) <= policy.batch_cap
    # the same window one round per call (two kernels per round)
    ctx = binding.Context(w.profile, n, policy=policy)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt)
    for rec in got["log"]:
        rc, dec = ctx.sp_greedy_round()
        assert rc == binding.SP_OK and dec == rec
    assert ctx.sp_greedy_round()[0] == binding.SP_DONE
    # back to the default policy: the window has to be scored again, and then runs as without a policy
    ctx.sp_set_policy(None)
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_schedule(0)
    assert e.value.status == binding.SP_ESTATE
    ctx.sp_score(x, app, D, wt)
    rc, summ, log = ctx.sp_schedule(0, log_capacity=4096)
    plain = run_window(gpu, w, 0)
    assert log == plain["log"] and summ == plain["summary"]
    plain["close"]()
    bad = wl.Policy(order=7)
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_set_policy(bad)
    assert e.value.status == binding.SP_EINVAL
    ctx.close()


@pytest.mark.parametrize("head", ["logistic", "mlp_f32", "mlp_bf16"])
@pytest.mark.parametrize("name", ["sneakpeek", "alg1"])
def test_data_aware_group_splitting(gpu, head, name):
    """Sec. 5.3.2: subgroups per predicted class, labelled by every scoring kernel, ordered and scheduled as
    groups of their own."""
    torch, binding = gpu
    kw = dict(classes=(2, 5, 33, 3), models=(3, 2, 6, 4), max_batch=11, deadline=(6.0, 150.0), fractions=(0.3, 0.2, 0.3, 0.2))
    if head == "logistic":
        w = wl.tiny(seed=98, n=2200, feat_dim=19, hidden_dim=0, **kw)
    elif head == "mlp_f32":
        w = wl.tiny(seed=99, n=1100, feat_dim=33, hidden_dim=17, **kw)
    else:
        w = wl.tiny(seed=100, n=1300, feat_dim=24, hidden_dim=10, feat_dtype=wl.BF16, **kw)
    for a in range(4):                          # sharper heads: a good share of confident requests
        if w.profile.feat_dtype == wl.BF16:
            w.profile.W1[a] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(w.profile.W1[a]) * 2.0)
        else:
            w.profile.W1[a] = (w.profile.W1[a] * 3.0).astype(np.float32)
    policy = wl.named_policy(name)
    policy.split_groups = 1
    got, stats = full_parity(gpu, w, max_rounds=0, ea_tol=2e-3 if head == "mlp_bf16" else None, want_cube=True,
                             policy=policy)
    assert got["summary"]["done"] == 1 and stats["rounds"] > 10
    # round by round gives the same schedule (on the window full_parity actually ran)
    w = got["workload"]
    ctx = binding.Context(w.profile, w.requests.n, policy=policy)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt)
    # sp_schedule above ran the rounds in one launch (a resident workgroup serves all groups of its application);
    # one round per call below takes the two-kernel path: the two must agree decision for decision
    assert ctx.lib.sp_rounds_in_one_launch(ctx.h)
    for rec in got["log"]:
        rc, dec = ctx.sp_greedy_round()
        assert rc == binding.SP_OK and dec == rec
    assert ctx.sp_greedy_round()[0] == binding.SP_DONE
    ctx.close()


def test_group_splitting_beyond_what_a_resident_workgroup_serves(gpu):
    """More than 64 non-empty subgroups in one application: sp_schedule takes two kernels per round, with the
    same parity; an application with few subgroups beside it changes nothing."""
    torch, binding = gpu
    w = wl.tiny(seed=101, n=4000, classes=(120, 3), models=(3, 2), max_batch=9, feat_dim=24, deadline=(6.0, 150.0),
                fractions=(0.8, 0.2))
    w.profile.W1[0] = (w.profile.W1[0] * 8.0).astype(np.float32)       # sharp head: most requests are confident
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = 1
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True, policy=policy)
    assert got["summary"]["done"] == 1 and stats["rounds"] > 10
    ctx = binding.Context(w.profile, w.requests.n, policy=policy)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt)
    assert not ctx.lib.sp_rounds_in_one_launch(ctx.h)
    ctx.close()


@pytest.mark.parametrize("kind", [wl.PEN_STEP, wl.PEN_LINEAR, wl.PEN_SIGMOID])
def test_swap_in_costs_on_both_round_paths(gpu, kind):
    """Sec. 3.1 "context switch time" / Sec. 5.2 model locality: a batch pays its variant's swap-in cost
    unless the previous batch ran the same variant."""
    torch, binding = gpu
    w = wl.tiny(seed=95 + kind, n=2600, classes=(5, 3, 40, 2), models=(3, 2, 8, 5), max_batch=21, feat_dim=19,
                penalty=kind, deadline=(4.0, 120.0), fractions=(0.4, 0.1, 0.3, 0.2))
    wl.attach_swap_costs(w.profile, seed=96, lo=0.5, hi=9.0, skip_every=3)
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)       # sp_schedule: rounds in one launch
    # swap costs do show in the clock: some batch starts computing later than the previous one ended
    L = w.profile.lat_ms
    paid = [r for r in got["log"] if r["t_end_ms"] - r["t_start_ms"] > float(L[r["app"]][r["model"], r["batch"] - 1]) * (1 + 1e-6)]
    free = [r for r in got["log"] if r not in paid]
    assert paid and free
    # the same window one round per call (two kernels per round)
    ctx = binding.Context(w.profile, 2600)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt)
    for rec in got["log"]:
        rc, dec = ctx.sp_greedy_round()
        assert rc == binding.SP_OK and dec == rec
    assert ctx.sp_greedy_round()[0] == binding.SP_DONE
    # costs can be taken away again, and bad ones are rejected
    for a in range(4):
        ctx.sp_set_swap_cost(a, None)
    ctx.sp_score(x, app, D, wt)
    rc, summ, log = ctx.sp_schedule(0, log_capacity=4096)
    assert all(r["t_end_ms"] - r["t_start_ms"] == pytest.approx(float(L[r["app"]][r["model"], r["batch"] - 1]), rel=1e-6) for r in log)
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_set_swap_cost(0, np.array([1.0, -2.0, 0.0], dtype=np.float32))
    assert e.value.status == binding.SP_EINVAL
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_set_swap_cost(9, np.array([1.0], dtype=np.float32))
    assert e.value.status == binding.SP_EINVAL
    ctx.close()


def test_profile_too_large_for_the_one_launch_rounds_takes_the_two_kernel_path(gpu):
    """More (application, variant) pairs than resident workgroups fit: sp_schedule falls back to two kernels
    per round and takes the same decisions the oracle does."""
    torch, binding = gpu
    A = 90
    w = wl.tiny(seed=101, n=5000, classes=tuple(2 + (a % 5) for a in range(A)), models=tuple(9 + (a % 4) for a in range(A)),
                max_batch=7, feat_dim=12, deadline=(5.0, 90.0))
    assert int(np.sum(w.profile.n_models)) > 900
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=False)
    assert stats["rounds"] > 20 and got["summary"]["done"] == 1
    ctx = binding.Context(w.profile, 5000)
    assert not ctx.rounds_in_one_launch
    ctx.close()


def test_more_than_255_applications_two_pass_grouping(gpu):
    """Two radix passes over the application id, segment starts by search, many empty and tiny groups."""
    A = 300
    rng = np.random.default_rng(7)
    frac = rng.dirichlet(np.full(A, 0.3))
    w = wl.tiny(seed=102, n=4000, classes=tuple(2 + (a % 3) for a in range(A)), models=tuple(1 + (a % 3) for a in range(A)),
                max_batch=6, feat_dim=10, deadline=(5.0, 90.0), fractions=tuple(frac / frac.sum()))
    counts = np.bincount(w.requests.app, minlength=A)
    assert (counts == 0).any() and counts.max() > 50
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
    assert got["summary"]["done"] == 1 and stats["rounds"] >= 20


def test_more_applications_than_the_segment_table_holds(gpu):
    """Beyond 1024 applications k_segments places tiles and units without its LDS tables, the scan's
    digit totals are one row per application, and the rounds run over more than a thousand groups."""
    A = 1100
    rng = np.random.default_rng(11)
    frac = rng.dirichlet(np.full(A, 0.5))
    w = wl.tiny(seed=103, n=6000, classes=tuple(2 + (a % 4) for a in range(A)), models=tuple(1 + (a % 2) for a in range(A)),
                max_batch=4, feat_dim=6, deadline=(5.0, 60.0), fractions=tuple(frac / frac.sum()))
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=False)
    assert stats["rounds"] >= 20 and got["summary"]["done"] == 1


def test_largest_batch_variant_and_class_counts(gpu):
    """B = 256 and M = 16 (the library's limits) with C well beyond one class tile, on the matrix-core kernel."""
    w = wl.tiny(seed=103, n=900, classes=(1500, 700), models=(16, 16), max_batch=256, feat_dim=64, deadline=(20.0, 900.0),
                alpha=(0.5, 3.0), beta=(0.05, 0.4))
    got, stats = full_parity(gpu, w, max_rounds=0, want_cube=True)
    assert max(r["batch"] for r in got["log"]) > 64 and got["summary"]["done"] == 1


def test_bf16_logistic_head_and_wide_fp32_head(gpu):
    """Heads of the streaming kernel: bf16 without a hidden layer, fp32 wider than 256 features."""
    w = wl.tiny(seed=104, n=500, classes=(6, 11), models=(3, 4), max_batch=7, feat_dim=40, hidden_dim=0,
                feat_dtype=wl.BF16, deadline=(5.0, 90.0))
    full_parity(gpu, w, max_rounds=0, ea_tol=2e-3)
    w = wl.tiny(seed=105, n=300, classes=(9, 4), models=(2, 5), max_batch=5, feat_dim=300, hidden_dim=0, deadline=(5.0, 90.0))
    full_parity(gpu, w, max_rounds=0, want_cube=True)


def test_context_reuse_with_a_smaller_second_window(gpu):
    torch, binding = gpu
    big = wl.make("cfg2", n_requests=3000)
    small = wl.make("cfg2", n_requests=700, seed=5)
    small.profile = big.profile
    ctx = binding.Context(big.profile, 3000)
    first = run_window(gpu, big, 0, ctx=ctx)
    second = run_window(gpu, small, 0, ctx=ctx)
    alone = run_window(gpu, small, 0)
    for k in ("ea", "key", "order", "model", "round_of", "order_of", "util"):
        assert np.array_equal(second[k], alone[k]), k
    assert second["log"] == alone["log"] and first["summary"]["n_rounds"] > 0
    ctx.close()
    alone["close"]()


def test_error_paths(gpu):
    torch, binding = gpu
    w = wl.tiny(seed=80, n=100, classes=(4, 2), models=(2, 2), max_batch=4, feat_dim=8)
    ctx = binding.Context(w.profile, 100)
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_greedy_round()
    assert e.value.status == binding.SP_ESTATE
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_schedule(0)
    assert e.value.status == binding.SP_ESTATE
    x, app, D, wt = binding.to_device(w.requests)
    big = torch.zeros((101, 8), device="cuda:0")
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_score(big, torch.zeros(101, dtype=torch.int32, device="cuda:0"), torch.ones(101, device="cuda:0"),
                     torch.ones(101, device="cuda:0"))
    assert e.value.status == binding.SP_ECAPACITY
    for what in ("app_hi", "app_neg", "deadline", "deadline_nan", "weight"):
        a2, D2, w2 = app.clone(), D.clone(), wt.clone()
        if what == "app_hi":
            a2[17] = 2
        elif what == "app_neg":
            a2[3] = -1
        elif what == "deadline":
            D2[5] = 0.0
        elif what == "deadline_nan":
            D2[5] = float("nan")
        else:
            w2[99] = -0.5
        ctx.sp_score(x, a2, D2, w2)
        with pytest.raises(binding.SneakPeekError) as e:
            ctx.sp_schedule(0)
        assert e.value.status == binding.SP_EINVAL, what
        with pytest.raises(binding.SneakPeekError) as e:
            ctx.sp_greedy_round()
        assert e.value.status == binding.SP_EINVAL, what
    # the context recovers with a good window
    ctx.sp_score(x, app, D, wt)
    rc, summ, _ = ctx.sp_schedule(0)
    assert rc == binding.SP_DONE and summ["n_scheduled"] + summ["n_dropped"] == 100
    ctx.close()


def random_case(seed):
    """A small workload, a policy and the optional profile extras, all drawn from the seed."""
    rng = np.random.Generator(np.random.PCG64(7000 + seed))
    A = int(rng.integers(1, 6))
    classes = tuple(int(c) for c in np.where(rng.random(A) < 0.15, rng.integers(100, 300, A), rng.integers(2, 70, A)))
    models = tuple(int(m) for m in rng.integers(1, 17, A))
    head = ["logistic", "mlp_f32", "mlp_bf16", "logistic_bf16"][int(rng.integers(0, 4))]
    bf16 = head.endswith("bf16")
    wide = rng.random() < 0.12                      # beyond the widths the matrix-core kernels take
    d = int(rng.integers(1, 6)) * 8 if bf16 else int(rng.integers(1, 41))
    hidden = 0 if head.startswith("logistic") else int(rng.integers(3, 41))
    if wide:
        d = int(rng.integers(33, 41)) * 8
        hidden = 0 if hidden == 0 else int(rng.integers(257, 300))
    lo = float(rng.uniform(2.0, 20.0))
    frac = rng.dirichlet(np.full(A, 2.0))
    frac = tuple(float(f) for f in frac / frac.sum())
    n = int(rng.integers(1, 1500)) if rng.random() < 0.6 else int(rng.integers(1500, 6000))
    w = wl.tiny(seed=7100 + seed, n=n, classes=classes, models=models,
                max_batch=int(rng.integers(1, 25)), feat_dim=d, hidden_dim=hidden,
                feat_dtype=wl.BF16 if bf16 else wl.F32, penalty=int(rng.integers(0, 3)),
                deadline=(lo, lo * float(rng.uniform(1.5, 12.0))), fractions=frac)
    if rng.random() < 0.5:
        wl.attach_priors(w.profile, seed=7200 + seed)
    if rng.random() < 0.5:
        wl.attach_swap_costs(w.profile, seed=7300 + seed, lo=0.2, hi=6.0, skip_every=int(rng.integers(0, 4)))
    names = ["sneakpeek", "alg1", "lo_priority", "lo_edf", "maxacc_edf", "capped", "unit", "split", "split_alg1"]
    name = names[int(rng.integers(0, len(names)))]
    if name == "capped":
        policy = wl.Policy(batch_cap=int(rng.integers(1, 9)))
    elif name == "unit":
        policy = wl.Policy(weight=wl.WEIGHT_UNIT, order=wl.ORDER_EDF if rng.random() < 0.5 else wl.ORDER_PRIORITY)
    elif name.startswith("split"):
        policy = copy.copy(wl.named_policy("alg1" if name == "split_alg1" else "sneakpeek"))
        policy.split_groups = 1
    else:
        policy = wl.named_policy(name)
    return w, policy, bf16, name


@pytest.mark.parametrize("seed", range(64))
def test_random_shapes_policies_and_profile_extras(gpu, seed):
    """Random small workloads (ragged class / variant counts, every head kind and penalty, priors, swap-in
    costs, every policy) through the whole path, against the oracle."""
    w, policy, bf16, name = random_case(seed)
    p = w.profile
    print(f"seed {seed}: n={w.requests.n} classes={tuple(int(c) for c in p.n_classes)} models={tuple(int(m) for m in p.n_models)} "
          f"B={p.max_batch} d={p.feat_dim} H={p.hidden_dim} bf16={bf16} policy={name}", flush=True)
    full_parity(gpu, w, max_rounds=60, policy=policy, ea_tol=2e-3 if bf16 else None, want_cube=not bf16)


@pytest.mark.parametrize("d", [64, 65, 100, 128, 129, 201, 252, 256])
def test_logistic_widths_of_the_matrix_core_kernel(gpu, d):
    """Every padded feature width of the matrix-core logistic kernel (64, 128, 256), at and next to the
    boundaries, with and without rows that are multiples of 16 bytes; several class tiles, a ragged last
    class tile, several request tiles with a ragged tail."""
    w = wl.tiny(seed=7400 + d, n=1100, classes=(70, 33, 5, 129), models=(3, 16, 1, 7), max_batch=9, feat_dim=d,
                deadline=(5.0, 80.0), fractions=(0.45, 0.25, 0.05, 0.25))
    wl.attach_priors(w.profile, seed=7500 + d, kinds=(None, "weak"))
    full_parity(gpu, w, max_rounds=20, want_cube=True)


@pytest.mark.parametrize("d,H", [(8, 3), (72, 33), (136, 128), (192, 64), (264, 200), (448, 96), (512, 256), (40, 255)])
def test_bf16_mlp_widths_of_the_matrix_core_kernel(gpu, d, H):
    """Input widths across the 64-channel slices of layer 1 (a ragged last slice included; slice counts of
    every remainder modulo three, the depth of the kernel's feature ring) and hidden widths up to the
    kernel's 256."""
    w = wl.tiny(seed=7600 + d, n=900, classes=(70, 33, 5), models=(3, 16, 1), max_batch=9, feat_dim=d, hidden_dim=H,
                feat_dtype=wl.BF16, deadline=(5.0, 80.0), fractions=(0.5, 0.3, 0.2))
    full_parity(gpu, w, max_rounds=20, ea_tol=2e-3)


def test_matrix_core_rate_diagnostic(gpu):
    torch, binding = gpu
    tf_c, ghz_c = binding.sp_debug_mfma_rate(False, iters=2048)
    tf_r, ghz_r = binding.sp_debug_mfma_rate(True, iters=2048)
    # one instruction per 32 cycles and SIMD is the most the hardware does (2048 wavefronts on 1024 SIMDs);
    # how the workgroups spread over the CUs and what clock the device picks are not this library's to fix
    for tf, ghz in ((tf_c, ghz_c), (tf_r, ghz_r)):
        assert 100.0 < tf < 2600.0 and 0.5 < ghz < 3.0
        ceiling = 1024 * 32768 / 32 * ghz * 1e9 / 1e12
        assert 0.3 * ceiling < tf < 1.15 * ceiling
    with pytest.raises(binding.SneakPeekError) as e:
        binding.sp_debug_mfma_rate(True, iters=0)
    assert e.value.status == binding.SP_EINVAL
    with pytest.raises(binding.SneakPeekError) as e:
        binding.sp_debug_mfma_rate(True, iters=64, idle=3)
    assert e.value.status == binding.SP_EINVAL
    # with idle gaps (one wavefront per SIMD) the matrix cores cannot be busier than without
    for idle in (1, 8):
        tf, ghz = binding.sp_debug_mfma_rate(True, iters=2048, idle=idle)
        ceiling = 1024 * 32768 / 32 * ghz * 1e9 / 1e12
        assert 0.05 * ceiling < tf < 1.15 * ceiling
        if idle == 8:
            assert tf < 0.6 * ceiling            # 256 busy cycles, then some 512 idle ones


def test_copy_rate_diagnostic_and_stage_timing(gpu):
    torch, binding = gpu
    gbs = binding.sp_debug_copy_rate(1 << 26)
    assert 100.0 < gbs < 16000.0                 # read + written; the data sheet says 8,000 GB/s
    lib = binding.load_library()
    import ctypes as C
    out = C.c_double(0.0)
    assert lib.sp_debug_copy_rate(0, 8, None, C.byref(out)) == binding.SP_EINVAL
    assert lib.sp_debug_copy_rate(0, 1 << 20, None, None) == binding.SP_EINVAL
    # the timing record: stage times are consistent, the evaluation count is the triangle's
    w = wl.tiny(seed=7700, n=600, classes=(4, 3), models=(2, 3), max_batch=7, deadline=(50.0, 90.0))
    ctx = binding.Context(w.profile, 600)
    ctx.sp_set_timing(1)
    x, app, D, wt = binding.to_device(w.requests)
    model = torch.zeros(600, dtype=torch.int32, device="cuda:0")
    for one_launch in (True, False):
        ctx.sp_score(x, app, D, wt)
        if one_launch:
            rc, summ, _ = ctx.sp_schedule(3, model_out=model)
        else:
            for _ in range(3):
                ctx.sp_greedy_round()
            rc, summ, _ = ctx.sp_schedule(0 if False else 1, model_out=model)    # brings the state to the host
        tm = ctx.sp_get_timing()
        assert 0.0 < tm["finish_order_ms"] <= tm["order_ms"] and tm["copy_outputs_ms"] > 0.0
        # loose deadlines: every round sees full windows of 7 requests in both applications
        rounds = summ["n_rounds"]
        assert tm["utility_evaluations"] == rounds * (2 + 3) * 7 * 8 // 2
    # level 3: the two events around the scoring kernel only; the other fields stay 0
    ctx.sp_set_timing(3)
    ctx.sp_score(x, app, D, wt)
    ctx.sp_schedule(3, model_out=model)
    tm = ctx.sp_get_timing()
    assert tm["score_kernel_ms"] > 0.0
    assert tm["group_ms"] == 0.0 and tm["order_ms"] == 0.0 and tm["rounds_ms"] == 0.0 and tm["copy_outputs_ms"] == 0.0
    ctx.close()


def test_a_caller_stream_is_honoured(gpu):
    """Everything a window launches goes to the stream the caller names: the same window on a stream of the
    caller's own (default priority), behind other work queued on that stream, gives bit-identical results."""
    torch, binding = gpu
    w = wl.tiny(seed=7700, n=3000, classes=(40, 7, 90), models=(5, 16, 3), max_batch=12, feat_dim=48, deadline=(4.0, 90.0))
    ref = run_window(gpu, w, 0, want_cube=True)
    side = torch.cuda.Stream()
    noise = torch.randn(2048, 2048, device="cuda:0")
    with torch.cuda.stream(side):
        for _ in range(3):
            noise = noise @ noise * 1e-3               # unrelated work ahead of the window on the same stream
        got = run_window(gpu, w, 0, want_cube=True)
    side.synchronize()
    torch.cuda.synchronize()
    assert got["log"] == ref["log"] and got["summary"] == ref["summary"]
    for k in ("ea", "key", "order", "seg", "cube", "model", "round_of", "order_of", "util"):
        assert np.array_equal(got[k], ref[k], equal_nan=True), k
    ref["close"]()
    got["close"]()


def test_two_contexts_interleaved_are_independent(gpu):
    """Separate contexts share nothing: windows of two contexts scheduled in alternating chunks end exactly
    as when each runs alone."""
    torch, binding = gpu
    wa = wl.tiny(seed=7800, n=2500, classes=(30, 8), models=(4, 9), max_batch=10, feat_dim=40, deadline=(4.0, 120.0))
    wb = wl.tiny(seed=7801, n=1800, classes=(5, 60, 12), models=(16, 2, 7), max_batch=6, feat_dim=24, hidden_dim=12,
                 feat_dtype=wl.BF16, deadline=(3.0, 80.0))
    alone = [run_window(gpu, w, 0) for w in (wa, wb)]
    ctxs = [binding.Context(w.profile, w.requests.n) for w in (wa, wb)]
    devs = [binding.to_device(w.requests) for w in (wa, wb)]
    outs = []
    for ctx, (x, app, D, wt), w in zip(ctxs, devs, (wa, wb)):
        ctx.sp_score(x, app, D, wt)
        n = w.requests.n
        outs.append([torch.full((n,), 99, dtype=torch.int32, device="cuda:0") for _ in range(3)] +
                    [torch.full((n,), -7.0, device="cuda:0")])
    done = [False, False]
    logs = [[], []]
    summ = [None, None]
    while not all(done):
        for i, ctx in enumerate(ctxs):
            if done[i]:
                continue
            rc, sm, _ = ctx.sp_schedule(3, *outs[i], log_capacity=0)
            summ[i] = sm
            done[i] = rc == binding.SP_DONE
    for i in range(2):
        assert summ[i] == alone[i]["summary"]
        for t, k in zip(outs[i], ("model", "round_of", "order_of", "util")):
            assert np.array_equal(t.cpu().numpy(), alone[i][k]), (i, k)
        ctxs[i].close()
        alone[i]["close"]()


@pytest.mark.parametrize("name", ["sneakpeek", "alg1"])
def test_many_rounds_across_several_launches(gpu, name):
    """Several hundred rounds in one sp_schedule call: the one-launch kernel is launched again every 64
    rounds and has to pick up clock, resident variant (swap-in costs), head pointers and generation
    numbers where the previous launch left them."""
    w = wl.tiny(seed=7900, n=700, classes=(6, 20, 3), models=(3, 5, 2), max_batch=3, feat_dim=16, penalty=wl.PEN_LINEAR,
                deadline=(200.0, 2500.0), alpha=(1.0, 4.0), beta=(0.2, 1.0), fractions=(0.5, 0.3, 0.2))
    wl.attach_swap_costs(w.profile, seed=7901, lo=0.5, hi=5.0)
    got, stats = full_parity(gpu, w, max_rounds=0, policy=wl.named_policy(name), want_cube=True)
    assert stats["rounds"] > 150 and got["summary"]["done"] == 1
    assert got["summary"]["n_scheduled"] + got["summary"]["n_dropped"] == 700 and got["summary"]["total_violation_ms"] > 0


def test_round_generations_start_over_cleanly(gpu):
    """The exchange words of the one-launch rounds kernel carry generation numbers that start over after
    2^23 - 1 rounds in the life of a context: a window placed across that point is scheduled exactly as
    one that is not."""
    torch, binding = gpu
    w = wl.tiny(seed=7900, n=700, classes=(6, 20, 3), models=(3, 5, 2), max_batch=3, feat_dim=16, penalty=wl.PEN_LINEAR,
                deadline=(200.0, 2500.0), alpha=(1.0, 4.0), beta=(0.2, 1.0), fractions=(0.5, 0.3, 0.2))
    ref = run_window(gpu, w, 0)
    assert ref["summary"]["n_rounds"] > 150
    ctx = binding.Context(w.profile, 700)
    if not ctx.rounds_in_one_launch:
        pytest.skip("this device does not hold the one-launch rounds kernel")
    ctx.sp_debug_set_generation((1 << 23) - 1 - 100)         # the second launch of the window reaches the limit
    got = run_window(gpu, w, 0, ctx=ctx)
    assert got["log"] == ref["log"] and got["summary"] == ref["summary"]
    for k in ("model", "round_of", "order_of", "util"):
        assert np.array_equal(got[k], ref[k]), k
    got2 = run_window(gpu, w, 0, ctx=ctx)                     # and the context goes on normally afterwards
    assert got2["log"] == ref["log"] and got2["summary"] == ref["summary"]
    with pytest.raises(binding.SneakPeekError):
        ctx.sp_debug_set_generation(1 << 23)
    ctx.close()
    ref["close"]()


def test_a_wait_that_runs_out_fails_the_call_and_the_context_carries_on_with_two_kernels(gpu):
    """The bounded waits of the one-launch rounds kernel, forced to run out from the host (a poll limit of
    one; every kernel still ends normally): sp_schedule reports SP_EDEVICE, the window has to be scored
    again, and from then on the context schedules with two kernels per round, with the same decisions."""
    torch, binding = gpu
    w = wl.tiny(seed=7950, n=2000, classes=(9, 30), models=(4, 7), max_batch=8, feat_dim=20, deadline=(4.0, 90.0))
    ref = run_window(gpu, w, 0)
    ctx = binding.Context(w.profile, 2000)
    if not ctx.rounds_in_one_launch:
        pytest.skip("this device does not hold the one-launch rounds kernel")
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_debug_set_spin_limit(1)
    ctx.sp_score(x, app, D, wt)
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_schedule(0, log_capacity=16)
    assert e.value.status == binding.SP_EDEVICE
    assert not ctx.lib.sp_rounds_in_one_launch(ctx.h)
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_schedule(0, log_capacity=16)                   # the window's state is not to be trusted any more
    assert e.value.status == binding.SP_ESTATE
    ctx.sp_debug_set_spin_limit(0)
    got = run_window(gpu, w, 0, ctx=ctx)                      # scored again, two kernels per round
    assert got["log"] == ref["log"] and got["summary"] == ref["summary"]
    for k in ("model", "round_of", "order_of", "util"):
        assert np.array_equal(got[k], ref[k]), k
    ctx.close()
    ref["close"]()


def test_a_look_back_that_runs_out_fails_the_window_and_the_context_carries_on(gpu):
    """The bounded look-back of the radix passes, forced to give up from the host (every kernel still ends
    normally): the rounds report SP_EDEVICE, the window has to be scored again, and then all is as before."""
    torch, binding = gpu
    # one application with three sort tiles, one with a single tile (which never looks back)
    w = wl.tiny(seed=7955, n=12000, classes=(9, 5), models=(3, 2), max_batch=8, feat_dim=12, deadline=(4.0, 90.0),
                fractions=(0.85, 0.15))
    ref = run_window(gpu, w, 0)
    ctx = binding.Context(w.profile, 12000)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_debug_set_sort_spin_limit(-1)
    ctx.sp_score(x, app, D, wt)
    for call in (ctx.sp_greedy_round, lambda: ctx.sp_schedule(0, log_capacity=16)):
        with pytest.raises(binding.SneakPeekError) as e:
            call()
        assert e.value.status in (binding.SP_EDEVICE, binding.SP_ESTATE)
    assert b"look-back" in ctx.lib.sp_last_hip_error(ctx.h)
    ctx.sp_debug_set_sort_spin_limit(0)
    got = run_window(gpu, w, 0, ctx=ctx)
    assert got["log"] == ref["log"] and got["summary"] == ref["summary"]
    for k in ("model", "round_of", "order_of", "util", "order"):
        assert np.array_equal(got[k], ref[k]), k
    ctx.close()
    ref["close"]()


@pytest.mark.parametrize("path", ["one launch", "two kernels"])
def test_timing_aid_changes_nothing_and_reports_sane_times(gpu, path):
    """sp_set_timing: the same schedule with stage and per-round timing on, on both rounds paths; the
    times are positive, one per round, and add up to no more than the whole."""
    torch, binding = gpu
    if path == "one launch":
        w = wl.tiny(seed=7960, n=2500, classes=(9, 30), models=(4, 7), max_batch=8, feat_dim=20, deadline=(4.0, 90.0))
    else:
        A = 90                                               # too many (application, variant) pairs to stay resident
        w = wl.tiny(seed=7961, n=4000, classes=tuple(2 + (a % 5) for a in range(A)), models=tuple(9 + (a % 4) for a in range(A)),
                    max_batch=7, feat_dim=12, deadline=(5.0, 90.0))
    ref = run_window(gpu, w, 0)
    ctx = binding.Context(w.profile, w.requests.n)
    if (path == "one launch") != ctx.rounds_in_one_launch:
        pytest.skip("this device runs the rounds of this profile the other way")
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_get_timing()
    assert e.value.status == binding.SP_ESTATE
    ctx.sp_set_timing(2)
    got = run_window(gpu, w, 0, ctx=ctx)
    assert got["log"] == ref["log"] and got["summary"] == ref["summary"]
    tm = ctx.sp_get_timing()
    per_round = ctx.sp_get_round_times()
    n_rounds = ref["summary"]["n_rounds"]
    assert tm["n_rounds_timed"] == len(per_round) == n_rounds
    assert all(0.0 < t < 5.0 for t in per_round)             # milliseconds
    assert 0.0 < tm["score_kernel_ms"] < 50.0 and 0.0 < tm["group_ms"] < 50.0 and 0.0 < tm["order_ms"] < 50.0
    assert sum(per_round) <= tm["rounds_ms"] * 1.05 + 0.05
    ctx.sp_set_timing(0)
    ctx.close()
    ref["close"]()


def test_optional_outputs_short_log_and_calls_after_the_end(gpu):
    """sp_schedule with only some outputs, a log shorter than the schedule, and further calls once nothing
    is live: the same schedule, the log's first entries, SP_DONE with the same summary."""
    torch, binding = gpu
    w = wl.tiny(seed=7970, n=1500, classes=(9, 30), models=(4, 7), max_batch=8, feat_dim=20, deadline=(4.0, 90.0))
    ref = run_window(gpu, w, 0)
    assert ref["summary"]["n_rounds"] > 8
    ctx = binding.Context(w.profile, 1500)
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt)                              # no EA / key outputs asked for
    util = torch.full((1500,), -7.0, device="cuda:0")
    rc, summ, log = ctx.sp_schedule(0, util_out=util, log_capacity=5)
    assert rc == binding.SP_DONE and summ == ref["summary"]
    assert log == ref["log"][:5]
    assert np.array_equal(util.cpu().numpy(), ref["util"])
    model = torch.full((1500,), 99, dtype=torch.int32, device="cuda:0")
    rc, summ2, log2 = ctx.sp_schedule(0, model_out=model, log_capacity=1500)     # nothing left to do
    assert rc == binding.SP_DONE and summ2 == ref["summary"] and log2 == ref["log"]
    assert np.array_equal(model.cpu().numpy(), ref["model"])
    rc, dec = ctx.sp_greedy_round()
    assert rc == binding.SP_DONE
    ctx.close()
    ref["close"]()


@pytest.mark.parametrize("d", [1, 3, 4, 7, 8, 63, 90, 95, 97, 150, 161, 191, 194, 223, 225, 255])
def test_logistic_rows_that_end_inside_a_piece(gpu, d):
    """Every padded width of the logistic kernel that walks the classes (64 to 256 in steps of 32), rows whose last
    16-byte piece is partial or whose start is not aligned, rows shorter than a piece."""
    w = wl.tiny(seed=8100 + d, n=700, classes=(140, 33, 5), models=(3, 16, 1), max_batch=5, feat_dim=d,
                deadline=(5.0, 80.0), fractions=(0.5, 0.3, 0.2))
    full_parity(gpu, w, max_rounds=10)


STREAM_SHAPES = [  # dtype, d, H, classes: rows held (1, 2, 4, 8 blocks of 32, at and next to their edges), steps of 32 or 64
    (wl.F32, 8, 0, (32, 2)), (wl.F32, 9, 0, (33, 5)), (wl.F32, 257, 0, (64, 7)), (wl.F32, 300, 0, (65, 128)),
    (wl.F32, 289, 0, (129, 300)), (wl.F32, 513, 0, (256, 257, 9)),
    (wl.F32, 8, 1, (5, 40)), (wl.F32, 31, 32, (33, 3)), (wl.F32, 33, 33, (5, 64)), (wl.F32, 65, 64, (70, 2)),
    (wl.F32, 128, 65, (10, 7, 2)), (wl.F32, 130, 128, (97, 4)), (wl.F32, 63, 129, (5, 9)), (wl.F32, 97, 256, (40, 3)),
    (wl.BF16, 8, 0, (32, 2)), (wl.BF16, 9, 0, (33, 5)), (wl.BF16, 63, 0, (64, 7)), (wl.BF16, 65, 0, (128, 3)),
    (wl.BF16, 129, 0, (129, 300)), (wl.BF16, 512, 0, (100, 31)),
    (wl.BF16, 9, 5, (5, 40)), (wl.BF16, 64, 32, (33, 3)), (wl.BF16, 71, 64, (10, 70)), (wl.BF16, 200, 128, (100, 37)),
    (wl.BF16, 127, 129, (9, 33)), (wl.BF16, 61, 255, (40, 3))]


@pytest.mark.parametrize("shape", STREAM_SHAPES, ids=lambda s: f"{'bf16' if s[0] else 'f32'}-d{s[1]}-h{s[2]}-c{max(s[3])}")
def test_heads_of_the_streaming_kernel(gpu, shape):
    """The kernel that streams the features, at the edges of its tiles: one to nine steps with whole and partial last
    steps, rows at any alignment, groups of classes, a workgroup with one request and one that is full."""
    dtype, d, H, classes = shape
    A = len(classes)
    w = wl.tiny(seed=8200 + d + H, n=129 * A + 300, classes=classes, models=(3, 16, 1)[:A], max_batch=5, feat_dim=d, hidden_dim=H,
                feat_dtype=dtype, deadline=(5.0, 80.0), fractions=(0.5, 0.3, 0.2)[:A] if A == 3 else (0.7, 0.3))
    wl.attach_priors(w.profile, seed=8300 + d, kinds=(None, "weak"))
    full_parity(gpu, w, max_rounds=10, ea_tol=2e-3 if dtype == wl.BF16 else None)


@pytest.mark.parametrize("dtype,d,C", [(wl.F32, 160, 32), (wl.F32, 161, 33), (wl.F32, 195, 64), (wl.F32, 225, 65), (wl.F32, 260, 128), (wl.F32, 1003, 5),
                                       (wl.BF16, 320, 64), (wl.BF16, 321, 100), (wl.BF16, 391, 32), (wl.BF16, 455, 33), (wl.BF16, 512, 128)])
def test_rows_shared_by_two_teams(gpu, dtype, d, C):
    """Five to thirty-two slices of a row, even and odd numbers, whole and partial last ones, taken by one team of wavefronts (windows of more
    tiles than compute units, or of five slices) or two: the same requests in a long window and in short ones, logits, labels and
    rows that bring their largest value in either team's share."""
    torch, binding = gpu
    tiles = torch.cuda.get_device_properties(0).multi_processor_count
    n, few = tiles * 128 + 1, 389
    w = wl.tiny(seed=8250 + d, n=few, classes=(C, 3), models=(5, 16), feat_dim=d, feat_dtype=dtype, fractions=(0.7, 0.3))
    x = w.requests.x
    if dtype == wl.F32:
        x[0::5, :40] *= np.float32(30.0)
        # (a product is held to 2^-22, so 32 of about 20 * 0.1 leave 3e-6 of a logit; at a thousand times a feature's usual size it is 1e-4, beyond
        # the tolerance, in any float32 sum)
        x[1::5, 32:64] *= np.float32(20.0)
        x[2::5, d - 1] = np.float32(50.0)
        x[3::5, 32:] = 0.0
    ref_ea, ref_key = orc.score_requests(w.profile, w.requests)
    tol = 2e-3 if dtype == wl.BF16 else TOL
    ctx = binding.Context(w.profile, n, policy=wl.Policy(split_groups=1))
    short = binding.to_device(w.requests)
    long = [torch.cat([t.repeat(*([n // few + 1] + [1] * (t.dim() - 1)))[: n - few], t]) for t in short]
    got = []
    for args, m in ((short, few), (long, n), ([t[: n - 1] for t in long], n - 1)):
        ea, key = torch.zeros((m, ctx.m_max), device="cuda:0"), torch.zeros(m, device="cuda:0")
        logits = torch.zeros((m, C), device="cuda:0")
        ctx.sp_score(*args, ea_out=ea, key_out=key)
        ctx.sp_debug_dump(binding.SP_DUMP_LOGITS, logits, x=args[0])
        got.append([v[:few].cpu().numpy() for v in (ea, key, logits)])
    ctx.close()
    for ea, key, logits in got:
        parity.assert_close("EA", ea, ref_ea, tol)
        parity.assert_close("key", key, ref_key, tol, floor=1e-30)
        # sums of up to 1,003 products of 22 bits and more, in another order
        parity.assert_close("logits", logits, got[1][2], 1e-5, floor=float(np.abs(logits).max()))


@pytest.mark.parametrize("hidden", [0, 24])
def test_streamed_rows_of_any_scale(gpu, hidden):
    """float32 rows are scaled by a running maximum: rows whose large values come first, last, or not at all, rows of zeros,
    and an infinity, which makes its own request's results NaN and no other's."""
    torch, binding = gpu
    w = wl.tiny(seed=8400 + hidden, n=300, classes=(20, 6), models=(4, 3), feat_dim=300, hidden_dim=hidden)
    x = w.requests.x
    x[0::7] *= np.float32(1e-12)
    x[1::7, 200:] *= np.float32(40.0)
    x[2::7, :40] *= np.float32(30.0)
    x[3::7] = 0.0
    x[4::7] *= np.float32(1e-3)
    x[4::7, 299] = 25.0
    ref_ea, ref_key = orc.score_requests(w.profile, w.requests)
    x[13, 150] = np.inf
    ctx = binding.Context(w.profile, 300)
    ea = torch.zeros((300, ctx.m_max), device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
    ea = ea.cpu().numpy()
    ctx.close()
    a = int(w.requests.app[13])
    assert np.all(np.isnan(ea[13, :int(w.profile.n_models[a])]))
    keep = np.arange(300) != 13
    parity.assert_close("EA", ea[keep], ref_ea[keep], TOL)


def _service_order(w, key, edf=False):
    """Requests of each application by descending key (ascending deadline), equal ones by id: whole numbers, no tolerance."""
    out = []
    for a in range(int(w.profile.n_apps)):
        ids = np.nonzero(w.requests.app == a)[0]
        by = w.requests.deadline_rel_ms[ids] if edf else -key[ids].astype(np.float64)
        out.append(ids[np.argsort(by, kind="stable")])
    return np.concatenate(out)


@pytest.mark.parametrize("A", [1, 2, 7, 8])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1025, 2048, 2049, 2051, 8190, 8192, 8193, 16384, 16387, 32767, 32768, 32769])
def test_short_windows_counted_and_placed_in_one_launch(gpu, n, A):
    """Window lengths around the ids per thread of the kernel that counts for itself, up to one application more than it takes; ids
    that start at any four bytes, so that the last quad of a window ends at the end of the array.  Whole numbers, no tolerance."""
    torch, binding = gpu
    rng = np.random.default_rng(100 * n + A)
    frac = rng.pareto(1.0, A) + 0.01
    w = wl.tiny(seed=8700 + A, n=n, classes=(2,) * A, models=(1,) * A, max_batch=2, feat_dim=8, fractions=tuple(frac / frac.sum()))
    ctx = binding.Context(w.profile, n)
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    seg = torch.zeros(A + 1, dtype=torch.int32, device="cuda:0")
    x, app, D, wt = binding.to_device(w.requests)
    for lead in (0, 1, 3):
        shifted = torch.full((n + lead,), A - 1, dtype=torch.int32, device="cuda:0")
        shifted[lead:] = app
        ctx.sp_score(x, shifted[lead:], D, wt, key_out=key)
        ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
        assert np.array_equal(order.cpu().numpy(), _service_order(w, key.cpu().numpy()))
        ctx.sp_debug_dump(binding.SP_DUMP_SEGMENTS, seg)
        assert np.array_equal(seg.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(w.requests.app, minlength=A))]))
    # ids outside [0, A) are counted apart and refused
    bad = app.clone()
    bad[n // 2] = -1
    bad[n - 1] = 1 << 30
    ctx.sp_score(x, bad, D, wt, key_out=key)
    with pytest.raises(binding.SneakPeekError):
        ctx.sp_schedule()
    ctx.sp_score(x, app, D, wt, key_out=key)              # and leave nothing behind
    ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
    assert np.array_equal(order.cpu().numpy(), _service_order(w, key.cpu().numpy()))
    ctx.close()


@pytest.mark.parametrize("n,A", [(1, 8), (1023, 8), (1025, 31), (2049, 32), (32769, 7), (40000, 1), (131072, 31), (131073, 30), (262144, 9)])
def test_windows_whose_tiles_hand_each_other_their_counts(gpu, n, A):
    """One tile to 128, one application more than are counted in this way: windows one after the other with other ids and lengths, waits that run
    out (all or every other tile counted from the ids), and a recorded window played again with ids changed in place.  Whole numbers."""
    torch, binding = gpu
    rng = np.random.default_rng(9100 + n + A)
    w = wl.tiny(seed=9100 + A, n=n, classes=(2,) * A, models=(1,) * A, max_batch=2, feat_dim=8)
    x, app, D, wt = binding.to_device(w.requests)
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    seg = torch.zeros(A + 1, dtype=torch.int32, device="cuda:0")
    ctx = binding.Context(w.profile, n)

    def draw(m):
        p = rng.random(A) ** 3 + 1e-3
        ids = rng.choice(A, m, p=p / p.sum()).astype(np.int32)
        app[:m].copy_(torch.from_numpy(ids))
        return ids

    def check(ids):
        ctx.sp_debug_dump(binding.SP_DUMP_SEGMENTS, seg)
        assert np.array_equal(seg.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(ids, minlength=A))]))
        ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
        m = ids.size
        assert np.array_equal(order[:m].cpu().numpy(), np.lexsort((np.arange(m), -key[:m].cpu().numpy().astype(np.float64), ids)))

    for m in (n, max(1, n // 2), n):
        ids = draw(m)
        ctx.sp_score(x[:m], app[:m], D[:m], wt[:m], key_out=key)
        check(ids)
    for polls in (1, 2, 1):                             # (nothing waited for; every other tile's counts do not come)
        ctx.sp_debug_set_spin_limit(polls)
        for m in (n, max(1, n - 1100)):
            ids = draw(m)
            ctx.sp_score(x[:m], app[:m], D[:m], wt[:m], key_out=key)
            check(ids)
    ctx.sp_debug_set_spin_limit(0)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        ctx.sp_score(x, app, D, wt, key_out=key)
    for _ in range(3):
        ids = draw(n)
        graph.replay()
        torch.cuda.synchronize()
        check(ids)
        ids = draw(n)
        ctx.sp_score(x, app, D, wt, key_out=key)
        check(ids)
    ctx.close()


@pytest.mark.parametrize("policy", ["sneakpeek", "lo_edf"])
@pytest.mark.parametrize("n,A,ties", [
    (1, 1, 0), (255, 2, 0), (1023, 1, 0), (1024, 1, 0), (1025, 1, 0), (3000, 1, 3), (4097, 3, 0), (16384, 1, 0), (16385, 1, 2),
    (17000, 40, 0), (131072, 5, 0), (131073, 200, 5), (262144, 1, 1), (262145, 2, 0), (300001, 255, 4), (5000, 256, 0), (5000, 700, 2)])
def test_grouping_and_ordering_at_the_edges_of_their_plans(gpu, n, A, ties, policy):
    """Window lengths at which the number of launches, the tiles or the method change, with the keys the library itself
    computed: applications of very different sizes (one empty), many equal keys, zero weights (the largest sort key)."""
    torch, binding = gpu
    rng = np.random.default_rng(n + A)
    frac = rng.pareto(1.0, A) + 0.01
    if A > 2:
        frac[1] = 0.0
    w = wl.tiny(seed=8500 + A, n=n, classes=(2,) * A, models=(1,) * A, max_batch=2, feat_dim=8, fractions=tuple(frac / frac.sum()))
    if ties:
        w.requests.x[:] = 0.0
        w.requests.deadline_rel_ms[:] = 10.0 + rng.integers(0, ties, n).astype(np.float32)
        w.requests.weight[:] = rng.integers(0, 3, n).astype(np.float32)
    ctx = binding.Context(w.profile, n, policy=wl.named_policy(policy))
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    x, app, D, wt = binding.to_device(w.requests)
    for _ in range(2):                                  # the second window reuses every buffer
        ctx.sp_score(x, app, D, wt, key_out=key)
        ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
        assert np.array_equal(order.cpu().numpy(), _service_order(w, key.cpu().numpy(), edf=policy == "lo_edf"))
    seg = torch.zeros(A + 1, dtype=torch.int32, device="cuda:0")
    ctx.sp_debug_dump(binding.SP_DUMP_SEGMENTS, seg)
    assert np.array_equal(seg.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(w.requests.app, minlength=A))]))
    ctx.close()


@pytest.mark.parametrize("n", [900, 5000, 20000, 270000])
def test_ordering_by_subgroup_and_key(gpu, n):
    """With data-aware subgroups the order inside an application is (subgroup, key, id) on every plan of the ordering."""
    torch, binding = gpu
    w = wl.tiny(seed=8600, n=n, classes=(300, 3), models=(2, 1), max_batch=2, feat_dim=8, fractions=(0.8, 0.2))
    for a in range(2):
        w.profile.W1[a] = (w.profile.W1[a] * 12.0).astype(np.float32)          # confident heads: most requests in a subgroup
    pol = wl.Policy(split_groups=1)
    ctx = binding.Context(w.profile, n, policy=pol)
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt, key_out=key)
    ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
    z = torch.zeros((n, ctx.c_max), device="cuda:0")
    ctx.sp_debug_dump(binding.SP_DUMP_LOGITS, z, x=x, app=app)
    z, key, order = z.cpu().numpy().astype(np.float64), key.cpu().numpy(), order.cpu().numpy()
    ctx.close()
    at = 0
    for a in range(2):
        ids = np.nonzero(w.requests.app == a)[0]
        th = orc.posterior(z[ids, :int(w.profile.n_classes[a])])
        top = th.max(axis=1)
        label = np.where(top > 0.5, 1 + th.argmax(axis=1), 0)
        clear = np.abs(top - 0.5) > 1e-4                # (at the threshold either label is right)
        got = order[at:at + ids.shape[0]]
        at += ids.shape[0]
        assert np.array_equal(np.sort(got), ids)
        keep = np.isin(got, ids[clear])
        want = ids[clear][np.lexsort((ids[clear], -key[ids[clear]].astype(np.float64), label[clear]))]
        assert np.array_equal(got[keep], want)


@pytest.mark.parametrize("classes", [(2,), (1000, 22), (1000, 23), (40, 3, 500)])
def test_subgroups_up_to_the_slots_of_one_workgroup_and_beyond(gpu, classes):
    """Groups formed from 3 possible pairs of application and label, from 1,024 (one thread each) and from 1,025: their ranges, their number
    and what the rounds make of them."""
    A = len(classes)
    w = wl.tiny(seed=9300 + classes[-1], n=500, classes=classes, models=(3, 2, 4)[:A], max_batch=6, feat_dim=16, deadline=(6.0, 150.0),
                fractions=(0.6, 0.3, 0.1) if A == 3 else (0.7, 0.3)[:A] if A == 2 else (1.0,))
    for a in range(A):
        w.profile.W1[a] *= np.float32(8.0)               # (decided heads: most requests have a label)
    full_parity(gpu, w, max_rounds=12, want_cube=True, policy=wl.Policy(split_groups=1))


@pytest.mark.parametrize("n", [1023, 1024, 1025, 3100])
@pytest.mark.parametrize("rounds", [1, 3])
def test_outputs_of_unserved_requests_at_the_fill_edges(gpu, n, rounds):
    """The workgroup that commits the rounds fills the outputs of requests that no round serves, 1,024 per round: windows
    it covers exactly, by one request too few and by more than the rounds allow (those are written behind the rounds)."""
    w = wl.tiny(seed=8700, n=n, classes=(5, 3), models=(3, 2), max_batch=7, feat_dim=16, deadline=(6.0, 150.0), fractions=(0.7, 0.3))
    full_parity(gpu, w, max_rounds=rounds)


@pytest.mark.parametrize("big", [63, 64, 65])
def test_subgroups_at_the_edge_of_the_lds_copy(gpu, big):
    """Subgroups of up to 64 requests are kept in LDS, 512 requests in all: sizes at that edge, one that is larger, and
    more small ones than fit."""
    sizes = [150, big, 1, 64, 65, 63] + [64] * 8
    C = len(sizes)
    n = sum(sizes)
    w = wl.tiny(seed=8710, n=n, classes=(C,), models=(3,), max_batch=9, feat_dim=16, deadline=(6.0, 400.0), fractions=(1.0,))
    lab = np.random.default_rng(8711).permutation(np.repeat(np.arange(C), sizes))
    w.requests.x[:] = 0.0
    w.requests.x[np.arange(n), lab] = 1.0
    w.profile.W1[0] = np.zeros((16, C), dtype=np.float32)
    w.profile.W1[0][np.arange(C), np.arange(C)] = 6.0              # class posterior 0.97: every request in its class's subgroup
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = 1
    got, stats = full_parity(gpu, w, max_rounds=0, policy=policy)
    assert got["summary"]["done"] == 1 and stats["rounds"] > 10


def test_empty_window_right_behind_a_split_one(gpu):
    """The number of groups reaches the host in stream order: an empty window scored while a split window of a single group
    is still on the stream has its own number of groups (every application), and nothing to serve."""
    torch, binding = gpu
    w = wl.tiny(seed=8720, n=30000, classes=(3,) * 12, models=(2,) * 12, max_batch=4, feat_dim=64)
    w.requests.app[:] = 0
    w.requests.x[:] = 0.0
    w.profile.b1[0][:] = np.array([9.0, 0.0, 0.0], np.float32)           # one subgroup of one application
    ctx = binding.Context(w.profile, 30000, policy=wl.Policy(split_groups=1))
    args = binding.to_device(w.requests)
    none = tuple(t[:0] for t in args)
    for one_launch in (True, False):
        for _ in range(3):
            ctx.sp_score(*args)
            ctx.sp_score(*none)
            if one_launch:
                rc, summ, _ = ctx.sp_schedule(4)
                assert rc == binding.SP_DONE and summ["n_rounds"] == 0
            else:
                rc, dec = ctx.sp_greedy_round()
                assert rc == binding.SP_DONE and dec is None
            cube = torch.zeros((12, ctx.m_max, 4), device="cuda:0")
            ctx.sp_debug_dump(binding.SP_DUMP_SCORE_CUBE, cube)          # one slab per group of the empty window
            assert torch.all(cube == -1.0)
    ctx.close()


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("d,at", [(72, 71), (71, 64), (9, 8), (100, 95), (128, 120), (300, 299)])
def test_infinite_feature_in_front_of_a_hidden_layer(gpu, dtype, d, at):
    """An infinite feature, also among the last ones of a row that ends inside a step, acts as in plain arithmetic: hidden units
    it drives to +inf make the request's expected accuracies NaN, units it drives to -inf are zero and leave the head's
    output bias.  No other request notices."""
    torch, binding = gpu
    w = wl.tiny(seed=8730 + d, n=200, classes=(9, 4), models=(3, 2), feat_dim=d, hidden_dim=20, feat_dtype=dtype)
    inf = np.uint16(0x7f80) if dtype == wl.BF16 else np.float32(np.inf)
    sign = np.uint16(0x8000)
    for a in range(2):                                   # every unit's weight of that feature is negative
        row = w.profile.W1[a][at]
        row[:] = (row | sign) if dtype == wl.BF16 else -np.abs(row)
    ref_ea, _ = orc.score_requests(w.profile, w.requests)
    w.requests.x[7, at] = inf                            # +inf: every unit at -inf
    w.requests.x[90, at] = -inf if dtype == wl.F32 else inf | sign      # -inf: every unit at +inf
    ctx = binding.Context(w.profile, 200)
    ea = torch.zeros((200, ctx.m_max), device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
    ea = ea.cpu().numpy()
    ctx.close()
    M = [int(w.profile.n_models[int(a)]) for a in w.requests.app]
    assert np.all(np.isnan(ea[90, :M[90]]))
    a = int(w.requests.app[7])
    z = w.profile.b2[a].astype(np.float64)
    parity.assert_close("EA without hidden units", ea[7, :M[7]], w.profile.acc[a].astype(np.float64) @ orc.posterior(z[None])[0], TOL)
    keep = ~np.isin(np.arange(200), (7, 90))
    parity.assert_close("EA", ea[keep], ref_ea[keep], 2e-3 if dtype == wl.BF16 else TOL)


def test_a_wait_that_runs_out_is_reported_by_its_own_call(gpu):
    """Bounds on the waits from far too short to enough, in steps of 2%, one round per launch, an application that takes about
    a hundred times longer than the others to find its window: whichever workgroup loses patience, and whether or not the commit
    got its batch, a call that returns SP_OK has left nothing behind for the next one to fail on."""
    torch, binding = gpu
    n = 400000
    w = wl.tiny(seed=8740, n=n, classes=(5,) * 6, models=(4, 4, 4, 4, 4, 4), max_batch=16, feat_dim=8, deadline=(4.0, 90.0),
                fractions=(0.99, 0.002, 0.002, 0.002, 0.002, 0.002))
    w.requests.deadline_rel_ms[w.requests.app == 0] = 1e-3           # dead from the start, all but the last in service order
    w.requests.weight[:] = 1.0
    first = np.nonzero(w.requests.app == 0)[0]
    w.requests.weight[first[-5:]] = 1e-6
    w.requests.deadline_rel_ms[first[-5:]] = 500.0
    args = binding.to_device(w.requests)
    ctx, lost, polls = None, 0, 20.0
    while polls < 600.0:
        if ctx is None:
            ctx = binding.Context(w.profile, n)
            if not ctx.rounds_in_one_launch:
                pytest.skip("this device does not hold the one-launch rounds kernel")
        ctx.sp_score(*args)
        torch.cuda.synchronize()
        ctx.sp_debug_set_spin_limit(int(polls))
        try:
            rc, summ, _ = ctx.sp_schedule(1)
        except binding.SneakPeekError as e:
            assert e.status == binding.SP_EDEVICE
            lost += 1
            ctx.close()                                  # (this one takes two kernels per round from here on)
            ctx = None
        else:
            ctx.sp_debug_set_spin_limit(0)
            assert rc == binding.SP_OK and summ["n_rounds"] == 1
            rc, summ, _ = ctx.sp_schedule(1)
            assert rc == binding.SP_OK and summ["n_rounds"] == 2
        polls *= 1.02
    assert lost > 0
    if ctx is not None:
        ctx.close()


@pytest.mark.parametrize("dtype,d,H,C", [(wl.F32, 300, 0, 100), (wl.F32, 40, 24, 30), (wl.F32, 40, 0, 150), (wl.BF16, 64, 0, 100), (wl.BF16, 72, 40, 20),
                                         (wl.BF16, 64, 200, 20)])
def test_small_accuracies_keep_their_bits(gpu, dtype, d, H, C):
    """Accuracy tables with values down to 1e-6, whole variants of small ones among them: expected accuracies relative to
    themselves, at the general float32 tolerance (the halves hold 22 bits: 2.4e-7 each)."""
    torch, binding = gpu
    w = wl.tiny(seed=8750 + d, n=300, classes=(C, 7), models=(8, 3), feat_dim=d, hidden_dim=H, feat_dtype=dtype)
    rng = np.random.default_rng(8751)
    for a in range(2):
        M, Ca = w.profile.acc[a].shape
        w.profile.acc[a] = (w.profile.acc[a] * 10.0 ** -np.linspace(0.0, 6.0, M)[:, None] * 10.0 ** rng.uniform(-0.3, 0.0, (M, Ca))).astype(np.float32)
    ref_ea, _ = orc.score_requests(w.profile, w.requests)
    ctx = binding.Context(w.profile, 300)
    ea = torch.zeros((300, ctx.m_max), device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
    parity.assert_close("EA", ea.cpu().numpy(), ref_ea, TOL, floor=1e-12)
    ctx.close()


@pytest.mark.parametrize("dtype,d,H,C", [(wl.F32, 300, 0, 20), (wl.F32, 770, 0, 100), (wl.F32, 289, 0, 300), (wl.F32, 40, 0, 50), (wl.F32, 130, 24, 30),
                                         (wl.F32, 33, 60, 5), (wl.F32, 150, 128, 40), (wl.F32, 97, 256, 40), (wl.BF16, 70, 40, 20), (wl.BF16, 64, 128, 9)])
def test_features_and_hidden_units_of_very_different_ranges(gpu, dtype, d, H, C):
    """Features that are not normalised (scales 10^-5 to 10^5, the weights making up for it), hidden units likewise, inputs that a
    head ignores at values of 10^9: as accurate as normalised ones (float32 tolerance; a float32 product does not care)."""
    torch, binding = gpu
    w = wl.tiny(seed=8760 + d, n=300, classes=(C, 7), models=(5, 3), feat_dim=d, hidden_dim=H, feat_dtype=dtype)
    p, rng = w.profile, np.random.default_rng(8761)
    up = (lambda v: v) if dtype == wl.F32 else wl.f32_to_bf16_bits
    down = (lambda v: np.asarray(v, np.float32)) if dtype == wl.F32 else (lambda v: orc.widen(v).astype(np.float32))
    if dtype == wl.F32:                                  # (bfloat16 features carry their own exponents)
        s = (10.0 ** rng.uniform(-5.0, 5.0, d)).astype(np.float32)
        w.requests.x = (w.requests.x * s).astype(np.float32)
        w.requests.x[:, d // 2] = rng.uniform(1e9, 2e9, 300)
        for a in range(2):
            p.W1[a] = (p.W1[a] / s[:, None]).astype(np.float32)
            p.W1[a][d // 2] = 0.0
    if H:
        for a in range(2):
            t = (10.0 ** rng.uniform(-5.0, 5.0, H)).astype(np.float32)
            p.W1[a], p.b1[a] = up(down(p.W1[a]) * t), (p.b1[a] * t).astype(np.float32)
            p.W2[a] = up(down(p.W2[a]) / t[:, None])
    ref_ea, ref_key = orc.score_requests(p, w.requests)
    ctx = binding.Context(p, 300)
    ea = torch.zeros((300, ctx.m_max), device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
    parity.assert_close("EA", ea.cpu().numpy(), ref_ea, TOL)
    ctx.close()


@pytest.mark.parametrize("dtype,d,H,C", [(wl.F32, 300, 0, 100), (wl.F32, 40, 0, 20), (wl.F32, 40, 24, 300), (wl.BF16, 64, 0, 100), (wl.BF16, 72, 40, 70)])
@pytest.mark.parametrize("size", [3e5, 4e7, 6e9, 1e20, 3.3e38])
def test_logits_of_millions_and_more(gpu, dtype, d, H, C, size):
    """Logits so large that the softmax is a choice: the largest logit's row of the table, in whatever tile of classes it lies
    and whatever came before it."""
    torch, binding = gpu
    n = 200
    w = wl.tiny(seed=8770 + d, n=n, classes=(C, 7), models=(5, 3), max_batch=4, feat_dim=d, hidden_dim=H, feat_dtype=dtype)
    p, rng = w.profile, np.random.default_rng(8771)
    last = p.W2 if H else p.W1
    for a in range(2):
        Ca = int(p.n_classes[a])
        b = (size * rng.permutation(np.linspace(-1.0, 1.0, Ca))).astype(np.float32)     # what decides: every other class is far below
        if H:
            p.b2[a] = b
        else:
            p.b1[a] = b
        last[a] = last[a] * 0 if dtype == wl.F32 else np.zeros_like(last[a])
    ctx = binding.Context(p, n)
    ea = torch.zeros((n, ctx.m_max), device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
    ctx.close()
    for i in range(n):
        a = int(w.requests.app[i])
        top = int(np.argmax((p.b2 if H else p.b1)[a]))
        want = p.acc[a][:, top].astype(np.float64)
        parity.assert_close("EA", ea[i, :want.size].cpu().numpy(), want, TOL)


@pytest.mark.parametrize("size", [3e5, 6e9])
def test_subgroup_labels_of_large_logits(gpu, size):
    """The subgroup label of logits of millions is the largest one's class: the service order is by label, then key."""
    torch, binding = gpu
    w = wl.tiny(seed=8775, n=400, classes=(40,), models=(2,), max_batch=4, feat_dim=300)
    w.profile.W1[0][:] = 0.0
    w.profile.W1[0][0, 30] = w.profile.W1[0][1, 4] = np.float32(size)
    w.requests.x[:] = 0.0
    w.requests.x[np.arange(400), np.arange(400) % 2] = 1.0
    ctx = binding.Context(w.profile, 400, policy=wl.Policy(split_groups=1))
    key = torch.zeros(400, device="cuda:0")
    order = torch.zeros(400, dtype=torch.int32, device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), key_out=key)
    ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
    ctx.close()
    ids = np.arange(400)
    want = ids[np.lexsort((ids, -key.cpu().numpy().astype(np.float64), np.where(ids % 2 == 0, 31, 5)))]
    assert np.array_equal(order.cpu().numpy(), want)


@pytest.mark.parametrize("dtype,d,H", [(wl.F32, 300, 0), (wl.F32, 40, 24), (wl.BF16, 64, 0), (wl.BF16, 71, 40)])
def test_infinite_weights(gpu, dtype, d, H):
    """A weight of -inf excludes a class (or turns a hidden unit off) for requests with a positive input there."""
    torch, binding = gpu
    w = wl.tiny(seed=8780 + d, n=200, classes=(12, 7), models=(5, 3), feat_dim=d, hidden_dim=H, feat_dtype=dtype)
    p = w.profile
    ninf = np.float32(-np.inf) if dtype == wl.F32 else np.uint16(0xff80)
    one = np.float32(1.0) if dtype == wl.F32 else np.uint16(0x3f80)
    w.requests.x[:, 3] = one
    ref = copy.deepcopy(w)                               # the same with a weight that is large enough
    big = np.float32(-1e6) if dtype == wl.F32 else wl.f32_to_bf16_bits(np.float32([-1e6]))[0]
    for q, v in ((w, ninf), (ref, big)):
        for a in range(2):
            q.profile.W1[a][3, 2] = v
            if H:
                q.profile.W1[a][:, 5], q.profile.b1[a][5] = 0, 1.0       # a unit that is always on
                q.profile.W2[a][5, 4] = v
    ref_ea, _ = orc.score_requests(ref.profile, ref.requests)
    ctx = binding.Context(p, 200)
    ea = torch.zeros((200, ctx.m_max), device="cuda:0")
    ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
    ctx.close()
    parity.assert_close("EA", ea.cpu().numpy(), ref_ea, TOL if dtype == wl.F32 else 2e-3)


@pytest.mark.parametrize("B", [128, 211, 213, 256])
def test_subgroup_rounds_of_the_largest_batches(gpu, B):
    """Subgroups in one launch with the windows of the largest batches in LDS (more than 64 KB per workgroup from 212 on)."""
    torch, binding = gpu
    w = wl.tiny(seed=8790 + B, n=3000, classes=(12, 3), models=(3, 2), max_batch=B, feat_dim=24, deadline=(20.0, 900.0),
                beta=(0.05, 0.3), fractions=(0.8, 0.2))
    w.profile.W1[0] = (w.profile.W1[0] * 6.0).astype(np.float32)
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = 1
    got, stats = full_parity(gpu, w, max_rounds=12, policy=policy)
    assert stats["rounds"] > 3 and max(r["batch"] for r in got["log"]) > 64
    ctx = binding.Context(w.profile, 3000, policy=policy)
    ctx.sp_score(*binding.to_device(w.requests))
    assert ctx.lib.sp_rounds_in_one_launch(ctx.h)
    ctx.close()


@pytest.mark.parametrize("single", [3, 64, 70])
def test_log_of_single_rounds_and_scheduled_ones(gpu, single):
    """The log of a window that single rounds began and sp_schedule ended, below and beyond the decisions that the host keeps
    (64 without an allocation; otherwise the log is read back from the device)."""
    torch, binding = gpu
    w = wl.tiny(seed=8800, n=900, classes=(5, 3), models=(3, 2), max_batch=4, feat_dim=16, alpha=(0.1, 0.3), beta=(0.01, 0.05), deadline=(40.0, 300.0))
    args = binding.to_device(w.requests)
    ctx = binding.Context(w.profile, 900)
    ctx.sp_score(*args)
    _, want, log = ctx.sp_schedule(0, log_capacity=900)
    assert len(log) > 100
    ctx.sp_score(*args)
    for k in range(single):
        rc, dec = ctx.sp_greedy_round()
        assert rc == binding.SP_OK and dec == log[k]
    rc, got, again = ctx.sp_schedule(0, log_capacity=900)
    assert got == want and again == log
    rc, got, short = ctx.sp_schedule(0, log_capacity=single)            # after the end: the log once more
    assert got == want and short == log[:single]
    ctx.close()


OTHER_HEADS = {  # the scoring kernels that the heads of the two tests of priors and of subgroups do not reach
    "generic f32": dict(feat_dim=33, hidden_dim=260), "generic bf16": dict(feat_dim=24, hidden_dim=257, feat_dtype=wl.BF16),
    "generic narrow": dict(feat_dim=5, hidden_dim=9), "wide bf16 mlp": dict(feat_dim=24, hidden_dim=200, feat_dtype=wl.BF16),
    "classes walked": dict(feat_dim=40, hidden_dim=0)}


@pytest.mark.parametrize("split", [False, True], ids=["priors", "priors and subgroups"])
@pytest.mark.parametrize("head", OTHER_HEADS)
def test_priors_and_subgroups_on_the_other_scoring_kernels(gpu, head, split):
    kw = OTHER_HEADS[head]
    bf16 = kw.get("feat_dtype") == wl.BF16
    w = wl.tiny(seed=8820, n=1200, classes=(5, 12, 135, 2), models=(3, 1, 16, 7), max_batch=9, deadline=(6.0, 150.0),
                fractions=(0.4, 0.1, 0.3, 0.2), **kw)
    for a in range(4):                                   # sharper heads: a good share of confident requests
        w.profile.W1[a] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(w.profile.W1[a]) * 2.0) if bf16 else (w.profile.W1[a] * 3.0).astype(np.float32)
    wl.attach_priors(w.profile, seed=8821)
    full_parity(gpu, w, max_rounds=25, ea_tol=2e-3 if bf16 else None, want_cube=not bf16,
                policy=wl.Policy(split_groups=1) if split else None)


@pytest.mark.parametrize("dtype,d,H", [(wl.F32, 300, 0), (wl.F32, 40, 0), (wl.F32, 40, 24), (wl.F32, 97, 200), (wl.BF16, 64, 0), (wl.BF16, 71, 40)])
@pytest.mark.parametrize("f", [1e36, 1e-36])
def test_weights_and_features_at_the_ends_of_the_range(gpu, dtype, d, H, f):
    """Large weights on small inputs and the other way round, features and hidden units: products of ordinary size."""
    torch, binding = gpu
    up = (lambda v: np.asarray(v, np.float32)) if dtype == wl.F32 else wl.f32_to_bf16_bits
    val = (lambda v: v) if dtype == wl.F32 else wl.bf16_bits_to_f32
    for hidden in ([False, True] if H else [False]):
        w = wl.tiny(seed=8830 + d, n=200, classes=(20, 6), models=(5, 3), feat_dim=d, hidden_dim=H, feat_dtype=dtype)
        p = w.profile
        if not hidden:
            w.requests.x = up(val(w.requests.x) * np.float32(1.0 / f))
        for a in range(2):
            p.W1[a] = up(val(p.W1[a]) * np.float32(f))
            if hidden:
                p.b1[a] = (p.b1[a] * np.float32(f)).astype(np.float32)
                p.W2[a] = up(val(p.W2[a]) * np.float32(1.0 / f))
        ref_ea, _ = orc.score_requests(p, w.requests)
        ctx = binding.Context(p, 200)
        ea = torch.zeros((200, ctx.m_max), device="cuda:0")
        ctx.sp_score(*binding.to_device(w.requests), ea_out=ea)
        ctx.close()
        parity.assert_close("EA", ea.cpu().numpy(), ref_ea, TOL if dtype == wl.F32 else 2e-3)


@pytest.mark.parametrize("n,classes,hidden", [
    (5, (2, 300, 40), 0), (1021, (300, 2, 33, 161, 64, 1, 97), 0), (20011, (4, 700, 4, 130), 0), (68011, (4, 300, 4, 130), 0),
    (3000, tuple(2 + 37 * (a % 9) for a in range(300)), 0), (3000, tuple(2 + 37 * (a % 9) for a in range(253)), 0), (2500, (5, 400, 60), 24),
    (40003, (5, 140, 60), 24)],
    ids=["fewer tiles than dies", "one or two tiles each", "fewer tiles than compute units", "many tiles", "more than 255 applications",
         "253 applications", "hidden layer", "hidden layer, many tiles"])
def test_scoring_tiles_dealt_by_their_cost(gpu, n, classes, hidden):
    """Applications of very different class counts: beyond a tile per compute unit (256) tiles are numbered from the costliest
    application to the cheapest."""
    A = len(classes)
    f = np.array([3.0 if a % 3 == 0 else 0.02 if a % 3 == 1 else 1.0 for a in range(A)])
    w = wl.tiny(seed=900 + A, n=n, classes=classes, models=tuple(1 + a % 4 for a in range(A)), max_batch=8, feat_dim=40,
                hidden_dim=hidden, deadline=(4.0, 80.0), fractions=tuple(f / f.sum()))
    full_parity(gpu, w, max_rounds=4)


@pytest.mark.parametrize("n,A", [(3, 16), (2048, 16), (68007, 16), (5000, 304)])
def test_scoring_tiles_in_even_eighths(gpu, n, A):
    """Large and small heads by turns: the dies' contiguous eighths cost the same although the tiles do not."""
    w = wl.tiny(seed=950 + A, n=n, classes=(300, 20) * (A // 2), models=(2,) * A, max_batch=8, feat_dim=40, deadline=(4.0, 80.0))
    full_parity(gpu, w, max_rounds=4)


@pytest.mark.parametrize("name", ["sneakpeek", "alg1", "maxacc_edf", "group first"])
@pytest.mark.parametrize("A,M,B,n,due,fractions", [
    (1, 1, 1, 40, (5.0, 60.0), None), (3, 4, 31, 3000, (5.0, 150.0), (0.9, 0.09, 0.01)), (2, 6, 64, 5000, (30.0, 400.0), None),
    (15, 2, 33, 4000, (20.0, 300.0), None), (2, 3, 20, 30000, (4.0, 200.0), (0.97, 0.03)), (1, 16, 58, 63, (50.0, 500.0), None)],
    ids=["one of each", "short windows", "batches of 64", "fifteen applications", "mostly dead", "fewer than a wavefront"])
def test_single_rounds_in_one_workgroup(gpu, name, A, M, B, n, due, fractions):
    """A round per call in one launch of one workgroup against two kernels per round: the same decisions and members to the last
    bit, also with swap-in costs, from the first round until nothing is live."""
    torch, binding = gpu
    policy = wl.Policy(select=wl.SELECT_GROUP_FIRST) if name == "group first" else wl.named_policy(name)
    w = wl.tiny(seed=9100 + n, n=n, classes=(3,) * A, models=tuple(max(1, M - a % 3) for a in range(A)), max_batch=B, feat_dim=16, deadline=due,
                alpha=(0.5, 20.0), beta=(0.05, 2.5), fractions=fractions)
    w.profile.penalty[:] = [(wl.PEN_SIGMOID, wl.PEN_LINEAR, wl.PEN_STEP)[a % 3] for a in range(A)]
    wl.attach_swap_costs(w.profile, 9100, skip_every=2)
    args = binding.to_device(w.requests)
    ctxs = [binding.Context(w.profile, n, policy=policy) for _ in range(2)]
    ctxs[1].sp_debug_set_spin_limit(1 << 19)            # (any bound but the default keeps this kernel out)
    assert [c.lib.sp_rounds_in_one_workgroup(c.h) for c in ctxs] == [1, 0]
    ids = [torch.full((B,), -1, dtype=torch.int32, device="cuda:0") for _ in range(2)]
    for c in ctxs:
        c.sp_score(*args)
    for k in range(60):
        got = [c.sp_greedy_round(req_ids_out=i) for c, i in zip(ctxs, ids)]
        assert got[0] == got[1], f"round {k}"
        assert torch.equal(*ids), f"round {k}"
        if got[0][0] == binding.SP_DONE:
            break
    assert k > 0
    # what is left in one launch, from the state that either kernel has left
    ends = [c.sp_schedule(0, log_capacity=n) for c in ctxs]
    assert ends[0] == ends[1]
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("n", [1, 700, 16384, 16385])
def test_one_scheduled_round_fills_the_outputs(gpu, n):
    """sp_schedule of one round: the outputs of the requests it does not serve, below and beyond what its kernel fills itself."""
    w = wl.tiny(seed=9200 + n, n=n, classes=(4, 2), models=(3, 2), max_batch=16, feat_dim=16, deadline=(20.0, 90.0))
    full_parity(gpu, w, max_rounds=1)


@pytest.mark.parametrize("B,sizes", [(40, (300, 16, 17, 15, 1, 40, 2)), (64, (16, 17, 64, 9, 200)), (65, (16, 17, 8, 100))],
                         ids=["B40", "B64", "B65"])
def test_subgroups_of_a_few_requests(gpu, B, sizes):
    """Secondary subgroups around the sixteen requests up to which batch sizes are evaluated four at a time."""
    C, n = len(sizes), sum(sizes)
    w = wl.tiny(seed=9300 + B, n=n, classes=(C,), models=(3,), max_batch=B, feat_dim=16, deadline=(20.0, 500.0), fractions=(1.0,))
    lab = np.random.default_rng(9301).permutation(np.repeat(np.arange(C), sizes))
    w.requests.x[:] = 0.0
    w.requests.x[np.arange(n), lab] = 1.0
    w.profile.W1[0] = np.zeros((16, C), dtype=np.float32)
    w.profile.W1[0][np.arange(C), np.arange(C)] = 8.0
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = 1
    full_parity(gpu, w, max_rounds=0, policy=policy)


@pytest.mark.parametrize("split", [0, 1], ids=["plain", "subgroups"])
@pytest.mark.parametrize("B", [12, 70])
@pytest.mark.parametrize("A,M", [(32, 16), (30, 16), (15, 16)], ids=["512 pairs", "480 pairs", "240 pairs"])
def test_rounds_of_many_pairs(gpu, A, M, B, split):
    """The kernel with room for three workgroups per compute unit (more than 254 pairs on 256) and for two, batches below and beyond
    64."""
    torch, binding = gpu
    w = wl.tiny(seed=9400 + A, n=6000, classes=(4,) * A, models=(M,) * A, max_batch=B, feat_dim=16, deadline=(15.0, 200.0))
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = split
    ctx = binding.Context(w.profile, 6000, policy=policy)
    assert ctx.rounds_in_one_launch
    ctx.close()
    full_parity(gpu, w, max_rounds=12, policy=policy)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 255, 257, 511, 513, 1023, 1024, 1025, 2047])
@pytest.mark.parametrize("split", [0, 1], ids=["plain", "subgroups"])
def test_runs_of_every_stage_of_the_network(gpu, n, split):
    """Ordering of one application around the powers of two where the sorting network takes another stage, with many equal keys."""
    w = wl.tiny(seed=9500 + n, n=n, classes=(3,), models=(2,), max_batch=8, feat_dim=16, deadline=(20.0, 90.0), fractions=(1.0,))
    same = np.random.default_rng(9501).random(n) < 0.5
    w.requests.x[same] = w.requests.x[0]
    w.requests.weight[same] = w.requests.weight[0]
    w.requests.deadline_rel_ms[same] = w.requests.deadline_rel_ms[0]
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = split
    full_parity(gpu, w, max_rounds=2, policy=policy)


@pytest.mark.parametrize("A,M,B,edf", [(1, 3, 16, 0), (3, 4, 32, 0), (2, 4, 64, 1), (1, 4, 15, 1)])
def test_scores_that_are_no_numbers_win_on_every_route(gpu, A, M, B, edf):
    """An infinite weight whose request is lost inside the larger batches (infinity times zero), or, earliest deadline first with unit
    weights, a request with NaN features behind the first half of the window: some sizes' scores are NaN.  A NaN is above every
    number in a round's maximum, whichever kernel takes it; ties go to the smallest size."""
    torch, binding = gpu
    n = 400
    w = wl.tiny(seed=9600 + B, n=n, classes=(3,) * A, models=(M,) * A, max_batch=B, feat_dim=16, deadline=(30.0, 300.0), alpha=(1.0, 1.1),
                beta=(0.5, 0.55))
    policy = wl.Policy(order=wl.ORDER_EDF, weight=wl.WEIGHT_UNIT) if edf else wl.Policy()
    rng = np.random.default_rng(9601)
    for a in range(A):
        mine = np.nonzero(w.requests.app == a)[0]
        if edf:                                       # in the last quarter of the first window in service order
            at = np.argsort(w.requests.deadline_rel_ms[mine], kind="stable")[3 * B // 4]
            w.requests.x[mine[at]] = np.nan
        else:                                         # first in service order, lost in the last quarter of the batch sizes
            i = mine[rng.integers(mine.size)]
            w.requests.weight[i] = np.inf
            w.requests.deadline_rel_ms[i] = float(w.profile.lat_ms[a][:, 3 * B // 4].max())
            w.profile.penalty[a] = wl.PEN_STEP
    args = binding.to_device(w.requests)
    ctxs = [binding.Context(w.profile, n, policy=policy) for _ in range(3)]
    ctxs[1].sp_debug_set_spin_limit(1 << 19)          # (two kernels per round)
    assert [c.lib.sp_rounds_in_one_workgroup(c.h) for c in ctxs] == [1, 0, 1]
    ids = [torch.full((B,), -1, dtype=torch.int32, device="cuda:0") for _ in range(2)]
    for c in ctxs:
        c.sp_score(*args)
    cube = torch.zeros((A, ctxs[0].m_max, B), device="cuda:0")
    ctxs[1].sp_debug_dump(binding.SP_DUMP_SCORE_CUBE, cube)
    first = cube.cpu().numpy()
    assert np.isnan(first).any() and not np.isnan(first[..., : (B + 1) // 2]).any()
    log = []
    decided = lambda d: None if d is None else (d["app"], d["model"], d["batch"], d["t_start_ms"], d["t_end_ms"])
    for k in range(12):
        got = [c.sp_greedy_round(req_ids_out=i) for c, i in zip(ctxs[:2], ids)]
        if k == 0:                                    # from the scores themselves
            a, m, b = np.unravel_index(int(np.nonzero(np.isnan(first).ravel())[0][0]), first.shape)
            assert decided(got[1][1])[:3] == (a, m, b + 1)
        assert got[0][0] == got[1][0] and decided(got[0][1]) == decided(got[1][1]), f"round {k}"
        if got[0][0] == binding.SP_DONE:
            break
        assert torch.equal(*ids), f"round {k}"
        log.append(decided(got[1][1]))
    assert ctxs[2].rounds_in_one_launch
    _, _, one_launch = ctxs[2].sp_schedule(len(log), log_capacity=len(log))
    assert [decided(d) for d in one_launch] == log
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("density", [0.0004, 0.01, 0.2])
@pytest.mark.parametrize("n,A,B", [(1030, 1, 16), (5125, 1, 64), (20000, 2, 33), (70001, 1, 20)])
def test_single_rounds_past_long_stretches_of_the_dead(gpu, n, A, B, density):
    """Queues of which few are live, anywhere in service order: the walk of the one-workgroup round, 2,048 positions a step,
    against two kernels per round, to the last bit, and sp_schedule of one round against both.  The dead ones miss the first
    round by one float, half of the live ones just make it."""
    torch, binding = gpu
    w = wl.tiny(seed=9700 + n, n=n, classes=(3,) * A, models=(3,) * A, max_batch=B, feat_dim=16, deadline=(40.0, 900.0))
    rng = np.random.default_rng(int(9701 + n + 1e5 * density))
    dead = rng.random(n) >= density
    dead[-1] = False
    w.profile.penalty[:] = [(wl.PEN_SIGMOID, wl.PEN_STEP)[(a + n) % 2] for a in range(A)]
    due = w.requests.deadline_rel_ms
    for a in range(A):
        step = w.profile.penalty[a] == wl.PEN_STEP
        e0 = np.float32(w.profile.lat_ms[a][:, 0].min())                 # dead: e0 > D, or e0 >= 2 D
        lost = np.nextafter(e0, np.float32(0)) if step else e0 / np.float32(2)
        mine = w.requests.app == a
        due[mine & dead] = lost
        due[mine & ~dead & (rng.random(n) < 0.5)] = np.nextafter(lost, np.float32(np.inf))
    args = binding.to_device(w.requests)
    ctxs = [binding.Context(w.profile, n) for _ in range(3)]
    ctxs[1].sp_debug_set_spin_limit(1 << 19)            # (two kernels per round)
    assert [c.lib.sp_rounds_in_one_workgroup(c.h) for c in ctxs] == [1, 0, 1]
    ids = [torch.full((B,), -1, dtype=torch.int32, device="cuda:0") for _ in range(2)]
    for c in ctxs:
        c.sp_score(*args)
    for k in range(40):
        got = [c.sp_greedy_round(req_ids_out=i) for c, i in zip(ctxs, ids)]
        assert got[0] == got[1] and torch.equal(*ids), f"round {k}"
        rc, _, log = ctxs[2].sp_schedule(1, log_capacity=k + 1)
        assert rc == got[0][0]
        if rc == binding.SP_DONE:
            break
        assert log[k] == got[0][1], f"round {k}"
    assert k > 0
    for c in ctxs:
        c.close()


def test_windows_of_several_contexts_side_by_side(gpu):
    """Contexts of 300 and 500 pairs on streams and threads of their own, whose resident grids do not fit the device together: a call
    waits for room.  Decisions and outputs as of each context alone; no wait on the device runs out."""
    import threading
    torch, binding = gpu
    n, reps = 8000, 12
    kinds = [(30, 10, 0), (31, 16, 0), (30, 10, 1)]
    work, errors = [], []
    for i, (A, M, split) in enumerate(kinds):
        w = wl.tiny(seed=9800 + i, n=n, classes=(4,) * A, models=(M,) * A, max_batch=12, feat_dim=16, deadline=(15.0, 400.0))
        policy = wl.named_policy("sneakpeek")
        policy.split_groups = split
        ctx = binding.Context(w.profile, n, policy=policy)
        assert ctx.rounds_in_one_launch
        args = binding.to_device(w.requests)
        ctx.sp_score(*args)
        model = torch.zeros(n, dtype=torch.int32, device="cuda:0")
        ref = ctx.sp_schedule(0, model_out=model, log_capacity=n)
        work.append((ctx, args, ref, model.clone(), torch.cuda.Stream()))
    torch.cuda.synchronize()
    start = threading.Barrier(len(work))

    def serve(ctx, args, ref, ref_model, stream):
        try:
            with torch.cuda.stream(stream):
                model = torch.full((n,), 99, dtype=torch.int32, device="cuda:0")
                start.wait()
                for _ in range(reps):
                    ctx.sp_score(*args, stream=stream)
                    got = ctx.sp_schedule(0, model_out=model, log_capacity=n, stream=stream)
                    assert got == ref
                    assert torch.equal(model, ref_model)
        except BaseException as e:
            errors.append(e)

    threads = [threading.Thread(target=serve, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for w in work:
        assert w[0].lib.sp_rounds_in_one_launch(w[0].h)
        w[0].close()


@pytest.mark.parametrize("A,M,split", [(15, 16, 0), (31, 16, 0), (31, 16, 1)], ids=["240 pairs", "496 pairs", "496 pairs, subgroups"])
def test_rounds_beside_another_stream_of_kernels(gpu, A, M, split):
    """Matrix products without end on two other streams: the resident grid finds its places, no wait runs out."""
    import threading
    torch, binding = gpu
    n = 8000
    w = wl.tiny(seed=9850 + A, n=n, classes=(4,) * A, models=(M,) * A, max_batch=12, feat_dim=16, deadline=(15.0, 400.0))
    policy = wl.named_policy("sneakpeek")
    policy.split_groups = split
    ctx = binding.Context(w.profile, n, policy=policy)
    args = binding.to_device(w.requests)
    ctx.sp_score(*args)
    ref = ctx.sp_schedule(0, log_capacity=n)
    torch.cuda.synchronize()
    stop = threading.Event()

    def busy():
        with torch.cuda.stream(torch.cuda.Stream()):
            a, b = (torch.randn(2048, 2048, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
            while not stop.is_set():
                for _ in range(20):
                    a @ b
                torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=busy) for _ in range(2)]
    for t in threads:
        t.start()
    try:
        stream = torch.cuda.Stream()
        for _ in range(20):
            ctx.sp_score(*args, stream=stream)
            assert ctx.sp_schedule(0, log_capacity=n, stream=stream) == ref
    finally:
        stop.set()
        for t in threads:
            t.join()
    ctx.close()


@pytest.mark.parametrize("classes,models,B,select,one", [
    (2, (16, 16), 32, wl.SELECT_JOINT, 1), (1, (16,), 64, wl.SELECT_JOINT, 1), (11, (16,) * 11, 15, wl.SELECT_JOINT, 0),
    (15, (8,) * 15, 20, wl.SELECT_JOINT, 0), (15, (8,) * 15, 20, wl.SELECT_GROUP_FIRST, 1), (4, (16,) * 4, 64, wl.SELECT_GROUP_FIRST, 0),
    (13, (16,) * 13, 4, wl.SELECT_JOINT, 1), (15, (16,) * 15, 4, wl.SELECT_JOINT, 0), (16, (1,) * 16, 2, wl.SELECT_JOINT, 0), (1, (1,), 65, wl.SELECT_JOINT, 0)],
    ids=["two of 16", "one of 16, 64", "many pairs", "many pairs, 20", "group first", "group first, 64", "small batches", "too much LDS", "16 applications", "65"])
def test_which_rounds_run_in_one_workgroup(gpu, classes, models, B, select, one):
    """Either side of the lines by evaluations and pairs of batch sizes, LDS, applications and batches; the decisions are the oracle's."""
    torch, binding = gpu
    A, n = classes, 700
    w = wl.tiny(seed=9900 + A + B, n=n, classes=(3,) * A, models=models, max_batch=B, feat_dim=16, deadline=(20.0, 300.0))
    policy = wl.Policy(select=select)
    ctx = binding.Context(w.profile, n, policy=policy)
    assert ctx.lib.sp_rounds_in_one_workgroup(ctx.h) == one
    ctx.close()
    full_parity(gpu, w, max_rounds=1, policy=policy)


@pytest.mark.parametrize("route", ["one workgroup", "resident workgroups", "two kernels"])
def test_outputs_are_there_for_other_streams_when_a_call_returns(gpu, route):
    """A call has waited for its stream when it returns: what it wrote is read at once on another stream, whether the work in front
    of it is short or longer than the host polls, and the next call may come on that stream."""
    torch, binding = gpu
    w = wl.make("cfg2", n_requests=2048)
    p, rq = w.profile, w.requests
    ctx = binding.Context(p, rq.n)
    if route == "two kernels":
        ctx.sp_debug_set_spin_limit(1 << 19)           # (no rounds in one workgroup)
    args = binding.to_device(rq)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    big = torch.randn((4096, 4096), device="cuda:0")
    torch.cuda.synchronize()
    want = None
    for i in range(40):
        a, b = streams[i % 2], streams[(i + 1) % 2]
        ids = torch.full((4, p.max_batch), -1, dtype=torch.int32, device="cuda:0")
        outs = [torch.full((rq.n,), 99, dtype=torch.int32, device="cuda:0") for _ in range(3)] + [torch.full((rq.n,), -7.0, device="cuda:0")]
        torch.cuda.synchronize()
        if i % 10 == 9:
            with torch.cuda.stream(a):
                for _ in range(60):                    # (about 10 ms)
                    torch.mm(big, big)
        ctx.sp_score(*args, stream=a)
        got = []
        if route == "resident workgroups":
            got.append(ctx.sp_schedule(3, *outs, log_capacity=8, stream=a)[2])
            with torch.cuda.stream(b):
                got.append(torch.stack([o.view(torch.int32) for o in outs]).cpu().numpy())
            got.append(ctx.sp_schedule(2, *outs, log_capacity=8, stream=b)[2])
        else:
            for k in range(4):
                s, other = (a, b) if k % 2 else (b, a)
                if k == 0:
                    s, other = a, b
                got.append(ctx.sp_greedy_round(req_ids_out=ids[k], stream=s)[1])
                with torch.cuda.stream(other):
                    got.append(ids[k].cpu().numpy())
        torch.cuda.synchronize()
        if want is None:
            want = got
            assert route == "resident workgroups" or (got[1] >= 0).any()
        for g, h in zip(got, want):
            assert np.array_equal(g, h) if isinstance(g, np.ndarray) else g == h
    ctx.close()


def _sampled_positions(n):
    return ((n - 16) * np.repeat(np.arange(512), 16)) // 511 + np.tile(np.arange(16), 512)


def _weights(shape, n, rng):
    """Weights that make priority keys of one variant and one deadline: as they are, but for rounding that keeps their order."""
    u = rng.random(n)
    if shape == "equal":
        return np.ones(n)
    if shape == "three":
        return rng.integers(1, 4, n) * 0.25
    if shape == "zeros":
        return np.where(u < 0.5, 0.0, u)
    if shape == "two scales":
        return np.where(rng.random(n) < 0.5, u, 1e-30 * (1.0 + u))
    if shape == "rising":
        return np.arange(1, n + 1) / n
    if shape == "almost equal":
        return 1.0 + rng.integers(0, 5, n) * 2.0 ** -23
    if shape == "sample apart" and n > 8192:            # the requests that are sampled say nothing about the others
        w = 0.25 + 0.5 * u
        w[_sampled_positions(n)] = 1.0
        return w
    return u


@pytest.mark.parametrize("shape", ["spread", "equal", "three", "zeros", "two scales", "rising", "almost equal", "sample apart"])
@pytest.mark.parametrize("n,A", [(512, 1), (513, 1), (1024, 2), (1025, 2), (1025, 5), (1025, 1), (4096, 1), (4097, 1), (8192, 1), (8193, 1), (20011, 1), (65536, 1), (65537, 1), (65536, 2),
                                 (65536, 8), (106496, 3), (106497, 3)])
def test_ordering_in_one_launch(gpu, n, A, shape):
    """Window lengths around the steps of the one-launch ordering, keys that are evenly spread, equal, clustered, sorted or unlike
    what its sample tells.  Whole numbers, no tolerance."""
    torch, binding = gpu
    rng = np.random.default_rng(n + A)
    w = wl.tiny(seed=8800 + A, n=n, classes=(2,) * A, models=(1,) * A, max_batch=2, feat_dim=8)
    w.requests.deadline_rel_ms[:] = 10.0
    w.requests.weight[:] = _weights(shape, n, rng).astype(np.float32)
    ctx = binding.Context(w.profile, n)
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    x, app, D, wt = binding.to_device(w.requests)
    for _ in range(2):
        ctx.sp_score(x, app, D, wt, key_out=key)
        ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
        assert np.array_equal(order.cpu().numpy(), _service_order(w, key.cpu().numpy()))
    ctx.close()


@pytest.mark.parametrize("shape", ["spread", "three", "equal"])
@pytest.mark.parametrize("n,C", [(9000, 300), (9000, 5000), (40000, 40), (3000, 5000)])
def test_ordering_by_subgroup_in_one_launch(gpu, n, C, shape):
    """The same by (subgroup, key, id): few and many subgroups (more than there are bins), keys evenly spread and equal."""
    torch, binding = gpu
    rng = np.random.default_rng(n + C)
    w = wl.tiny(seed=8900, n=n, classes=(C, 3), models=(1, 1), max_batch=2, feat_dim=8, fractions=(0.9, 0.1))
    for a in range(2):
        w.profile.W1[a] = (w.profile.W1[a] * 40.0).astype(np.float32)          # confident heads: most requests in a subgroup
    w.requests.deadline_rel_ms[:] = 10.0
    w.requests.weight[:] = _weights(shape, n, rng).astype(np.float32)
    ctx = binding.Context(w.profile, n, policy=wl.Policy(split_groups=1))
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt, key_out=key)
    ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
    z = torch.zeros((n, ctx.c_max), device="cuda:0")
    ctx.sp_debug_dump(binding.SP_DUMP_LOGITS, z, x=x, app=app)
    z, key, order = z.cpu().numpy().astype(np.float64), key.cpu().numpy(), order.cpu().numpy()
    ctx.close()
    at = 0
    for a in range(2):
        ids = np.nonzero(w.requests.app == a)[0]
        th = orc.posterior(z[ids, :int(w.profile.n_classes[a])])
        top = th.max(axis=1)
        label = np.where(top > 0.5, 1 + th.argmax(axis=1), 0)
        clear = np.abs(top - 0.5) > 1e-4                # (at the threshold either label is right)
        got = order[at:at + ids.shape[0]]
        at += ids.shape[0]
        assert np.array_equal(np.sort(got), ids)
        keep = np.isin(got, ids[clear])
        want = ids[clear][np.lexsort((ids[clear], -key[ids[clear]].astype(np.float64), label[clear]))]
        assert np.array_equal(got[keep], want)


def _rare_labels_window(n, C, rare, shape, many=False):
    """One application whose requests' classes are set by hand: all but the `rare` greatest at random, and one to three requests of each of
    those (many: 300), early, in the middle and late among the requests that the ordering does not sample."""
    rng = np.random.default_rng(n + C)
    w = wl.tiny(seed=8950 + C, n=n, classes=(C,), models=(1,), max_batch=2, feat_dim=16)
    w.profile.W1[0] = np.zeros((16, C), np.float32)
    w.profile.W1[0][np.arange(C), np.arange(C)] = 40.0
    w.profile.b1[0] = np.zeros(C, np.float32)
    label = rng.integers(0, C - rare, n)
    free = np.setdiff1d(np.arange(n), _sampled_positions(n))
    for k in range(rare):
        some = rng.choice(free, 300 if many else 1 + (C + k) % 3, replace=False)
        label[some] = C - 1 - k
        free = np.setdiff1d(free, some)
    w.requests.x[:] = np.eye(16, dtype=np.float32)[label]
    w.requests.deadline_rel_ms[:] = 10.0
    if shape == "two deadlines":
        w.requests.weight[:] = 1.0
        w.requests.deadline_rel_ms[:] = rng.choice([10.0, 25.0], n)
    else:
        w.requests.weight[:] = np.where(rng.random(n) < 0.4, 0.0, rng.random(n)) if shape == "zeros" else rng.integers(1, 4, n) * 0.25
    return w, label


@pytest.mark.parametrize("shape", ["zeros", "three", "two deadlines"])
@pytest.mark.parametrize("n,C,rare", [(8700, 2, 1), (20000, 2, 1), (20000, 3, 1), (20000, 12, 2), (60000, 2, 1), (60000, 4, 1), (60000, 8, 1), (60000, 12, 2),
                                      (60000, 5, 3)])
def test_ordering_by_subgroup_with_labels_that_are_not_sampled(gpu, n, C, rare, shape):
    """The greatest subgroups consist of a few requests outside the ordering's sample, of 60,000 also of hundreds.  Whole numbers, no tolerance."""
    for many in (False, True) if n == 60000 else (False,):
        _check_rare_labels(gpu, n, C, rare, shape, many)


def _check_rare_labels(gpu, n, C, rare, shape, many):
    torch, binding = gpu
    w, label = _rare_labels_window(n, C, rare, shape, many)
    ctx = binding.Context(w.profile, n, policy=wl.Policy(split_groups=1))
    key = torch.zeros(n, device="cuda:0")
    order = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    x, app, D, wt = binding.to_device(w.requests)
    ctx.sp_score(x, app, D, wt, key_out=key)
    ctx.sp_debug_dump(binding.SP_DUMP_ORDER, order)
    key = key.cpu().numpy().astype(np.float64)
    assert np.array_equal(order.cpu().numpy(), np.lexsort((np.arange(n), -key, label)))
    ctx.close()


def test_rounds_over_subgroups_with_labels_that_are_not_sampled(gpu):
    w, _ = _rare_labels_window(20000, 2, 1, "two deadlines")
    full_parity(gpu, w, 4, policy=wl.Policy(split_groups=1))


def test_ordering_of_equal_keys_finds_its_range(gpu):
    """Where all keys are equal no workgroup of the one-launch ordering has to find its places digit by digit, which takes ten times as
    long as all of the rest: the device time of the ordering is of the same order as for keys that are spread (bound: four times)."""
    torch, binding = gpu
    n, took = 65536, {}
    for shape in ("spread", "equal"):
        w = wl.tiny(seed=8990, n=n, classes=(2,), models=(1,), max_batch=2, feat_dim=8)
        w.requests.deadline_rel_ms[:] = 10.0
        w.requests.weight[:] = _weights(shape, n, np.random.default_rng(1)).astype(np.float32)
        ctx = binding.Context(w.profile, n)
        ctx.sp_set_timing(1)
        data = binding.to_device(w.requests)
        times = []
        for _ in range(20):
            ctx.sp_score(*data)
            times.append(ctx.sp_get_timing()["order_ms"])
        ctx.close()
        took[shape] = min(times)
    assert took["equal"] < 4 * took["spread"], took


@pytest.mark.parametrize("call", ["round", "schedule"])
def test_a_call_that_meets_an_error_of_the_program_still_waits(gpu, call):
    """An earlier HIP call of the program has failed: a call reports that as it did before, and what it has launched has ended by then."""
    import ctypes
    torch, binding = gpu
    n = 20000
    w = wl.tiny(seed=9300, n=n, classes=(1000,), models=(2,), max_batch=4, feat_dim=256)
    ctx = binding.Context(w.profile, n)
    data = binding.to_device(w.requests)
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    torch.cuda.synchronize()
    for _ in range(20):                                 # (more than a millisecond)
        ctx.sp_score(*data)
    assert hip.hipSetDevice(4096) != 0
    with pytest.raises(binding.SneakPeekError) as e:
        ctx.sp_greedy_round() if call == "round" else ctx.sp_schedule(1)
    assert e.value.status == binding.SP_EDEVICE
    assert torch.cuda.current_stream().query()
    ctx.sp_score(*data)
    assert ctx.sp_greedy_round()[0] == binding.SP_OK
    ctx.close()
