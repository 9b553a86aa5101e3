"""GPU parity of Algorithm 1 end to end (star_plan_migrations) against the
oracle's plan: the same moves in the same order with the same exact gains, the
same final placement and the same final curves.

The cases cover:
* the two rules for the underloaded set;
* both memory rules;
* the remaining-length filter and thresholds;
* invalid requests;
* many instance counts;
* plans that stop early (balanced start, no improving move);
* plans that hit max_moves.
At the largest workload, each executed move is checked against properties
that hold at any size: its gain as the oracle scores it, the filters, the
final curves, and no better feasible move among sampled requests.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_13668_amd import star, synth
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu


def gpu_plan(cur, rem, inst, load, beta, n, b, K, max_moves, **kw):
    N = len(cur)
    pp = star.plan_params(N, n, b, K, max_moves, **kw)
    ws = star.Workspace(star.plan_workspace_size(pp))
    inst_d = to_dev(inst.copy())
    load_d = to_dev(load.copy())
    moves = torch.full((max(max_moves, 1) * star.MOVE_FIELDS,), -7, dtype=torch.int32, device=DEV)
    cnt = torch.full((1,), -7, dtype=torch.int32, device=DEV)
    star.plan_migrations(pp, to_dev(cur), to_dev(rem), inst_d, load_d,
                         to_dev(np.ascontiguousarray(beta, np.uint16).view(np.int16)), moves, cnt,
                         ws)
    torch.cuda.synchronize()
    m = int(cnt.cpu()[0])
    mv = moves.cpu().numpy().reshape(-1, star.MOVE_FIELDS)[:m]
    gains = [star.i128_to_int(w[2], w[3]) for w in mv.view(np.int64).reshape(-1, 4)]
    return {"moves": [(int(x[0]), int(x[1]), int(x[2])) for x in mv], "gains": gains,
            "inst_of": inst_d.cpu().numpy(), "load": load_d.cpu().numpy(),
            "error": ws.read_device_error()}


def _check(cur, rem, inst, beta, n, b, K, max_moves, label="", **kw):
    print(f"plan {label} N={len(cur)} n={n} b={b} K={K} moves<={max_moves} {kw}", flush=True)
    load, flags = oracle.project_load(cur, rem, inst, n_inst=n, bucket=b, n_buckets=K)
    okw = dict(kw)
    if "u_rule" in okw:
        okw["u_mode"] = okw.pop("u_rule")
    if "mem_rule" in okw:
        okw["mem_mode"] = okw.pop("mem_rule")
    ref = oracle.plan(cur, rem, inst, beta, n_inst=n, bucket=b, n_buckets=K, max_moves=max_moves,
                      **okw)
    gpu = gpu_plan(cur, rem, inst, load, beta, n, b, K, max_moves, **kw)
    assert gpu["moves"] == ref["moves"]
    assert gpu["gains"] == ref["gains"]
    np.testing.assert_array_equal(gpu["inst_of"], ref["inst_of"])
    np.testing.assert_array_equal(gpu["load"], ref["load"])
    assert gpu["error"] == flags
    return gpu


def _crowded(rng, N, n, b, K, frac=0.5, cur_hi=4000):
    cur, rem, inst = synth.random_requests(rng, N, n, cur_hi=cur_hi, len_hi=b * K + 50)
    inst[: int(N * frac)] = 0
    return cur, rem, inst


@pytest.mark.parametrize("N,n,b,K,moves,kw", [
    (40, 3, 1, 6, 6, {}),
    (200, 4, 4, 20, 12, dict(theta=(1, 10))),
    (300, 8, 64, 16, 16, dict(u_rule=1, theta=(1, 20))),
    (333, 5, 3, 30, 10, dict(min_rem=40, mem_rule=1, mem_cap=400000)),
    (120, 17, 2, 9, 20, dict(mem_cap=30000)),
    (500, 64, 8, 12, 8, dict(theta=(1, 4))),
    (90, 2, 16, 5, 30, {}),
    (64, 1, 4, 8, 3, {}),
])
def test_small_plans(N, n, b, K, moves, kw):
    rng = np.random.default_rng(N + 13 * n)
    cur, rem, inst = _crowded(rng, N, n, b, K)
    beta = rng.integers(0, 65536, size=K).astype(np.uint16)
    gpu = _check(cur, rem, inst, beta, n, b, K, moves, "small", **kw)
    if n > 1:
        assert len(gpu["moves"]) >= 1


def test_invalid_requests_and_early_stops():
    rng = np.random.default_rng(4)
    N, n, b, K = 300, 6, 8, 24
    cur, rem, inst = _crowded(rng, N, n, b, K)
    inst[3], cur[10], rem[20] = n + 1, 0, -4
    gpu = _check(cur, rem, inst, synth.bucket_weights(K), n, b, K, 10, "invalid")
    assert gpu["error"] == oracle.BAD_INST | oracle.BAD_CUR | oracle.BAD_REM
    # balanced start: identical instances, nothing to do
    cur = np.tile(np.array([300, 80, 1200], np.int32), 4)
    rem = np.tile(np.array([40, 5, 150], np.int32), 4)
    inst = np.repeat(np.arange(4, dtype=np.int32), 3)
    gpu = _check(cur, rem, inst, synth.bucket_weights(K), 4, b, K, 5, "balanced")
    assert gpu["moves"] == []
    # max_moves = 0 leaves everything as it was
    gpu = _check(cur, rem, inst, synth.bucket_weights(K), 4, b, K, 0, "zero")
    assert gpu["moves"] == []


@pytest.mark.parametrize("name,moves", [("continuous", 16), ("8b_batch", 12)])
def test_workload_plans(name, moves):
    """The workload's requests with true remaining lengths, half of them
    crowded onto instance 0."""
    wl = synth.WORKLOADS[name]
    x = synth.make_inputs(wl, steps=1, n_req=1)
    inst = x.inst_of.copy()
    inst[: wl.n_req // 2] = 0
    gpu = _check(x.cur_len, x.true_len, inst, synth.bucket_weights(wl.n_buckets), wl.n_inst,
                 wl.bucket, wl.n_buckets, moves, name, theta=(1, 10), min_rem=64)
    assert len(gpu["moves"]) == moves


@pytest.mark.parametrize("N,n,b,K,moves,cur_hi,kw", [
    (1, 2, 1, 1, 3, 50, {}),                                # one request, one bucket
    (17, 2, 1, 3, 40, 50, {}),                              # requests that move again; stops early
    (255, 6, 4, 12, 1, 4000, {}),                           # one move: first and last launch only
    (3841, 16, 8, 130, 9, 4000, {}),                        # a ragged last run of requests
    (61441, 3, 1, 5, 6, 4000, {}),                          # two rounds of requests per workgroup
    (700, 530, 2, 4, 3, 4000, dict(theta=(1, 4))),         # more instances than threads
    (300, 5, 64, 64, 12, 2**31 - 1, dict(mem_rule=1)),      # terms beyond the short products
    (200, 7, 64, 40, 12, 4000, dict(theta=(3, 2))),         # theta above one
    (200, 7, 64, 40, 12, 4000, dict(theta=(3, 2), u_rule=1)),
])
def test_plan_dispatch_edges(N, n, b, K, moves, cur_hi, kw):
    """Sizes where the passes' layout can go wrong (one workgroup, ragged and
    repeated rounds, more instances than threads, long products)."""
    rng = np.random.default_rng(N + n)
    cur, rem, inst = _crowded(rng, N, n, b, K, cur_hi=cur_hi)
    _check(cur, rem, inst, synth.bucket_weights(K), n, b, K, moves, "edges", **kw)


def test_rebalance_scan_plan_properties():
    """32768 requests on 64 instances: four moves, each checked on its own."""
    wl = synth.WORKLOADS["rebalance_scan"]
    x = synth.make_inputs(wl, steps=1, n_req=1)
    n, b, K = wl.n_inst, wl.bucket, wl.n_buckets
    inst = x.inst_of.copy()
    inst[: wl.n_req // 4] = 3
    beta = synth.bucket_weights(K)
    load, _ = oracle.project_load(x.cur_len, x.true_len, inst, n_inst=n, bucket=b, n_buckets=K)
    print("plan rebalance_scan full size", flush=True)
    gpu = gpu_plan(x.cur_len, x.true_len, inst, load, beta, n, b, K, 4, theta=(1, 10))
    assert len(gpu["moves"]) == 4
    place = inst.copy()
    rng = np.random.default_rng(2)
    for (r, s, t), g in zip(gpu["moves"], gpu["gains"]):
        cur_load, _ = oracle.project_load(x.cur_len, x.true_len, place, n_inst=n, bucket=b,
                                          n_buckets=K)
        assert place[r] == s
        one = oracle.score_variance(x.cur_len[[r]], x.true_len[[r]], place[[r]], cur_load, beta,
                                    bucket=b)
        assert int(one[0, t]) == g and g < 0
        # classification of this pass (theta = 1/10), exactly
        w = [sum(int(beta[k]) * int(cur_load[i, k]) for k in range(K)) for i in range(n)]
        now = np.bincount(place, weights=x.cur_len.astype(np.float64), minlength=n)
        assert 10 * n * w[s] > 11 * sum(w)
        assert 10 * n * int(now[t]) < 11 * sum(w)
        # no sampled feasible candidate beats it
        over = [10 * n * wi > 11 * sum(w) for wi in w]
        under = [10 * n * int(now[i]) < 11 * sum(w) for i in range(n)]
        pool = [q for q in rng.choice(wl.n_req, 300, replace=False) if over[place[q]]]
        if pool:
            gs = oracle.score_variance(x.cur_len[pool], x.true_len[pool], place[pool], cur_load,
                                       beta, bucket=b)
            for qi, q in enumerate(pool):
                for tt in range(n):
                    if tt != place[q] and under[tt]:
                        assert (int(gs[qi, tt]), int(q), tt) >= (g, r, t)
        place[r] = t
    np.testing.assert_array_equal(gpu["inst_of"], place)
    final, _ = oracle.project_load(x.cur_len, x.true_len, place, n_inst=n, bucket=b, n_buckets=K)
    np.testing.assert_array_equal(gpu["load"], final)
