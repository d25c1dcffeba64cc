"""GPU parity: the HIP pipeline, called through the C ABI, against the CPU oracle.

Small and adversarial windows are compared element by element on every output; the
benchmark workloads are compared exactly on every plan array and on sampled collate
outputs (plus whole-output properties), in the launch configuration the benchmark uses.
"""
import numpy as np
import pytest

import oracle
import synth
from _parity import (collate_properties, compare_collate_by_rank, compare_collate_full, compare_collate_sampled,
                     compare_loss_weights, compare_plan, log, run_gpu)

pytestmark = pytest.mark.gpu


def win(per_rank, budget, **kw):
    return synth.window_from_ranks("t", [np.asarray(x, dtype=np.int64) for x in per_rank], budget, **kw)


def check_full(w, pad_id=0):
    log(f"case {w.name}: W={w.W} n={w.n} budget={w.budget} mode={w.mode} quota={w.quota} "
        f"cap={None if w.capacity is None else list(w.capacity)}")
    ref = oracle.plan_window(w)
    pipe, outs = run_gpu(w, pad_id=pad_id)
    compare_plan(w, pipe, ref)
    compare_collate_full(w, outs, ref, pad_id)
    compare_loss_weights(pipe, ref)
    return pipe, ref


def adversarial_windows():
    rng = np.random.default_rng(100)
    out = []
    add = lambda name, per, budget, **kw: out.append(
        synth.window_from_ranks(name, [np.asarray(x, dtype=np.int64) for x in per], budget, **kw))
    add("worked_example", [[100, 200, 500, 800]], 1000)
    add("all_equal", [[64] * 700, [64] * 513], 4096)
    add("ascending", [np.arange(1, 3001), np.arange(5, 900)], 8192)
    add("descending", [np.arange(3000, 0, -1)], 5000)
    add("heavy_ties", [rng.integers(1, 4, 5000) for _ in range(3)], 64)
    add("single_sample_ranks", [[7], [9], [1]], 100)
    add("empty_ranks", [[], rng.integers(1, 500, 300), [], rng.integers(1, 500, 40), []], 2000)
    add("longer_than_budget", [rng.integers(900, 3000, 200), rng.integers(1, 100, 900)], 1000)
    add("budget_below_min", [rng.integers(50, 300, 400), rng.integers(50, 300, 10)], 49)
    add("one_rank", [rng.integers(1, 4000, 10000)], 16384)
    add("tiny_budget_one", [rng.integers(1, 5, 300)], 1)
    add("capacity_overflow", [rng.integers(1, 600, 900), rng.integers(1, 600, 500), rng.integers(1, 600, 50)], 3000,
        capacity=np.array([5, 0, 3]))
    add("capacity_one", [rng.integers(1, 300, 120), rng.integers(1, 300, 80)], 600, capacity=np.array([1, 1]))
    add("unequal_buffers", [rng.integers(1, 2000, 4000), rng.integers(1, 2000, 37), rng.integers(1, 2000, 1)], 8192)
    n4 = 4000 + 800 + 3
    for q in (1, 777, n4 - 1, n4, n4 + 1):
        add(f"nonjoin_q{q}", [rng.integers(1, 3000, 4000), rng.integers(1, 3000, 800), rng.integers(1, 3000, 3)],
            12000, mode="nonjoin", quota=q)
    add("nonjoin_capacity", [rng.integers(1, 900, 700), rng.integers(1, 900, 600)], 2500, mode="nonjoin",
        quota=1000, capacity=np.array([2, 4]))
    add("nonjoin_empty_rank", [rng.integers(1, 900, 70), [], rng.integers(1, 900, 5)], 2500, mode="nonjoin", quota=10)
    add("empty_window", [[], []], 100)
    # group discovery: a huge budget with a wide length range takes the pointer-jumping
    # path; a 4M budget with lengths up to 5000 gives ~4000 distinct steps, close to the
    # run walk's LDS table
    add("huge_budget_jumping", [rng.integers(1, 20000, 9000), rng.integers(1, 20000, 5000)], 1 << 40)
    add("many_step_runs", [rng.integers(1, 5000, 12000), rng.integers(1, 5000, 7000)], 4_000_000)
    per = [rng.integers(100, 3000, 47 - r) for r in range(15)] + [np.zeros(0, np.int64)]
    add("empty_rank_audit_w16", per, 8192)
    # narrow tiles (widths 3..9, a few rows each): groups straddle tile edges at every
    # offset, the next tile's first row is sometimes shorter than the group's remainder,
    # and an empty rank leaves zero-size IDLE tiles between non-empty ones
    add("narrow_tile_edges", [rng.integers(3, 10, 3000), [], rng.integers(3, 10, 1500), rng.integers(1, 4, 700)], 24)
    add("narrow_tile_edges_nonjoin", [rng.integers(3, 10, 3000), rng.integers(3, 10, 1501)], 31, mode="nonjoin",
        quota=2500)
    # more ranks than the LDS rank table (1024) and than a block's threads, some empty
    add("many_ranks_w1500", [rng.integers(1, 2000, int(rng.integers(0, 12))) for _ in range(1500)], 8192)
    per = [rng.integers(1, 2000, int(rng.integers(1, 9))) for _ in range(700)]
    add("many_ranks_w700_nonjoin", per, 6000, mode="nonjoin", quota=sum(len(x) for x in per) // 2)
    return out


@pytest.mark.parametrize("idx", range(len(adversarial_windows())))
def test_adversarial_window(idx):
    w = adversarial_windows()[idx]
    check_full(w, pad_id=idx + 3)


@pytest.mark.parametrize("kind", synth.AUDIT_KINDS)
def test_audit_distributions(kind):
    for W, mode in ((3, "join"), (8, "join"), (3, "nonjoin")):
        w = synth.audit_window(kind, W, budget=4096, mode=mode, quota=1000)
        pipe, ref = check_full(w)
        if mode == "join":
            _, q, P = synth.sampler_views(1000, W, seed=1)
            assert pipe.info["missing_ids"] == 0 and pipe.info["duplicate_ids"] == P


def test_random_small_windows():
    rng = np.random.default_rng(7)
    for t in range(40):
        W = int(rng.integers(1, 6))
        per = [rng.integers(1, int(rng.integers(2, 3000)), size=int(rng.integers(0, 400))) for _ in range(W)]
        n = sum(len(x) for x in per)
        mode = "nonjoin" if t % 3 == 2 else "join"
        cap = rng.integers(0, 6, size=W) if t % 4 == 1 else None
        w = win(per, int(rng.integers(1, 20000)), mode=mode, quota=int(rng.integers(1, n + 2)), capacity=cap)
        w.name = f"random_{t}"
        check_full(w, pad_id=int(rng.integers(0, 5)))


def test_random_medium_windows():
    # windows past the one-block-per-rank limit (ranks of up to 60,000 samples) in random
    # shapes: 1-24 ranks of unequal sizes, uniform, lognormal and bimodal lengths, budgets
    # from below the longest sample to 2^23 (where a wide length range sends group
    # discovery to pointer jumping), join and non-join modes, per-rank slot capacities
    import torch

    rng = np.random.default_rng(2025)
    for t in range(14):
        W = int(rng.integers(1, 25))
        big = int(rng.integers(0, W))
        kind = t % 3
        per = []
        for r in range(W):
            m = int(rng.integers(16385, 60000)) if r == big else int(rng.integers(0, 9000))
            if kind == 0:
                x = rng.integers(1, int(rng.integers(2, 3000)), size=m)
            elif kind == 1:
                x = np.clip(np.rint(synth.lognormal(rng, 200, 1.5, m)), 1, 8000).astype(np.int64)
            else:
                x = np.where(rng.random(m) < 0.9, rng.integers(8, 300, size=m), rng.integers(2000, 8000, size=m))
            per.append(x)
        jump = t % 5 == 4
        if jump:   # lengths 1 and 8000 in the window: more distinct steps than the run table holds
            per[big] = np.concatenate([per[big], [1, 8000]])
        n = sum(len(x) for x in per)
        budget = 1 << 23 if jump else int(rng.integers(2000, 300000))
        mode = "nonjoin" if t % 4 == 3 else "join"
        cap = rng.integers(0, 40, size=W) if t % 6 == 1 else None
        w = win(per, budget, mode=mode, quota=int(rng.integers(1, n + 2)), capacity=cap)
        w.name = f"random_medium_{t}"
        if jump:
            log(f"case {w.name}: W={w.W} n={w.n} budget={w.budget} mode={w.mode} (plan only)")
            ref = oracle.plan_window(w)
            pipe, _ = run_gpu(w, tokens=torch.zeros(64, dtype=torch.int32, device="cuda"), collate=False)
            compare_plan(w, pipe, ref)
            compare_loss_weights(pipe, ref)
        else:
            check_full(w, pad_id=int(rng.integers(0, 5)))


def test_sampler_padding_identity_coverage():
    # identity-coverage audit arithmetic: N = 57,284 over 8 ranks leaves P = 4 padding views
    views, q, P = synth.sampler_views(57284, 8, seed=3)
    rng = np.random.default_rng(3)
    lens = rng.integers(16, 12110, size=57284)
    w = win([lens[v] for v in views], 12288, identity=np.concatenate(views), num_identities=57284)
    w.name = "sampler_padding_57284"
    pipe, ref = check_full(w)
    assert pipe.info["missing_ids"] == 0 and pipe.info["duplicate_ids"] == P == 4


def test_workload_small_full():
    w = synth.WORKLOADS["ln512_w2x2048"].window()
    check_full(w)


@pytest.mark.parametrize("name", ["text_w8x65536", "bimodal_w16x65536", "mm_w8x262144", "ln480_w64x262144"])
def test_workload_full_size(name):
    # the launch configuration the benchmark times; every output element is compared
    w = synth.WORKLOADS[name].window()
    log(f"workload {name}: n={w.n} tokens={w.total_tokens}")
    ref = oracle.plan_window(w)
    log(f"  oracle plan done: steps={ref.steps} padded={ref.padded_elems}")
    pipe, outs = run_gpu(w)
    log("  gpu pipeline done")
    compare_plan(w, pipe, ref)
    compare_loss_weights(pipe, ref)
    log("  plan and loss weights equal")
    compare_collate_sampled(w, outs, ref)
    collate_properties(outs, ref)
    compare_collate_by_rank(w, outs, ref, pipe.win.tokens)
    log("  every output element equal")
    del pipe, outs
    import torch
    torch.cuda.empty_cache()


@pytest.mark.parametrize("case", ["at_block_limit", "past_block_limit", "wide_lengths", "one_length_per_rank",
                                  "long_rank", "tile_edges", "many_ranks", "many_ranks_jump", "max_lengths",
                                  "max_lengths_one_block", "budget_int64_max", "budget_int64_max_jump"])
def test_grouping_paths(case):
    # The two grouping paths (one block per rank up to 16,384 samples per rank, the
    # multi-block sort and run-table walk beyond) at the limit; lengths up to 2^25 (all
    # four byte digits of the one-block sort in use) with the collate left out (the token
    # stream of such lengths would not fit); equal lengths within each rank (no digit
    # varies); a rank of 700,000 samples (342 sort tiles: the per-rank scan of the tiles'
    # run counts takes two passes of its block) beside one of 3; ranks one position past,
    # at and one short of a tile edge, with empty and one-sample ranks; 1,100 ranks (more
    # than the rank table kernels stage in LDS) with one past the one-block limit, grouped
    # by the run-table walk and, at budget 2^23 with lengths 1..8000, by pointer jumping;
    # lengths over the whole valid range [1, 2^31 - 1] (31-bit keys: four radix passes of
    # 8-bit digits; with ranks of at most 16,384 samples, the one-block sort's top byte)
    # at a budget of 2^40 (64-bit batch sizes), plan only; a budget of 2^63 - 1 (batch
    # sizes past any rank: every group after the first takes the rest of its rank), on the
    # one-block path and on pointer jumping (plan only there)
    import torch

    rng = np.random.default_rng(61)
    if case == "at_block_limit":
        per = [rng.integers(1, 5000, 16384), rng.integers(1, 5000, 100), rng.integers(1, 5000, 16384)]
        w = win(per, 20000)
    elif case == "past_block_limit":
        per = [rng.integers(1, 5000, 16385), rng.integers(1, 5000, 5)]
        w = win(per, 20000)
    elif case == "wide_lengths":
        per = [np.concatenate([rng.integers(1, 1 << 25, 3000), rng.integers(1, 300, 1000)]) for _ in range(3)]
        w = win(per, 1 << 21)
    elif case == "long_rank":
        per = [rng.integers(1, 3000, 700000), rng.integers(1, 3000, 3)]
        w = win(per, 20000)
    elif case == "tile_edges":
        per = [rng.integers(1, 5000, 10 * 2048 + 1), rng.integers(1, 5000, 10 * 2048),
               np.zeros(0, np.int64), rng.integers(1, 5000, 10 * 2048 - 1), rng.integers(1, 5000, 1),
               rng.integers(1, 5000, 2)]
        w = win(per, 20000)
    elif case in ("many_ranks", "many_ranks_jump"):
        per = [rng.integers(1, 3000, 20000)] + [rng.integers(1, 3000, int(rng.integers(0, 21))) for _ in range(1099)]
        if case == "many_ranks_jump":
            per[0] = np.concatenate([per[0], [1, 8000]])
        w = win(per, (1 << 23) if case == "many_ranks_jump" else 20000)
    elif case == "max_lengths":
        top = (1 << 31) - 1
        per = [np.concatenate([rng.integers(1, top, 17000), [top, 1, top]]), rng.integers(1, top, 3),
               np.zeros(0, np.int64), np.concatenate([rng.integers(1, top, 2000), [top, top, 1]])]
        w = win(per, 1 << 40)
    elif case == "budget_int64_max":
        per = [rng.integers(1, 3000, 2000), rng.integers(1, 3000, 500), np.array([1, 1, 2])]
        w = win(per, (1 << 63) - 1)
    elif case == "budget_int64_max_jump":
        per = [rng.integers(1, 20000, 17000), rng.integers(1, 100, 5)]
        w = win(per, (1 << 63) - 1)
    elif case == "max_lengths_one_block":
        top = (1 << 31) - 1
        per = [np.concatenate([rng.integers(1, top, 2000), [top, 1, top]]), rng.integers(1, top, 3)]
        w = win(per, 1 << 40)
    else:
        per = [np.full(3000, 77), np.full(10, 5000), np.full(1, 1)]
        w = win(per, 9000)
    w.name = f"paths_{case}"
    log(f"case {w.name}: W={w.W} n={w.n} budget={w.budget}")
    ref = oracle.plan_window(w)
    if case in ("wide_lengths", "long_rank", "many_ranks_jump", "max_lengths", "max_lengths_one_block",
                "budget_int64_max_jump"):
        pipe, _ = run_gpu(w, tokens=torch.zeros(64, dtype=torch.int32, device="cuda"), collate=False)
        compare_plan(w, pipe, ref)
        compare_loss_weights(pipe, ref)
    else:
        pipe, outs = run_gpu(w)
        compare_plan(w, pipe, ref)
        compare_collate_full(w, outs, ref)
        compare_loss_weights(pipe, ref)


def _numpy_coverage(ids, n, identity=None, nid=0):
    cnt = np.bincount(ids, minlength=n)
    bad = int((cnt != 1).sum())
    if identity is None:
        return bad, int((cnt == 0).sum()), int(np.maximum(cnt - 1, 0).sum())
    icnt = np.bincount(identity[ids], minlength=nid)
    return bad, int((icnt == 0).sum()), int(np.maximum(icnt - 1, 0).sum())


@pytest.mark.parametrize("case", ["permutation", "duplicates", "missing_and_dup", "identity_map"])
def test_check_coverage_entry_point(case):
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(21)
    n = 100_003
    w = win([rng.integers(1, 50, 60_000), rng.integers(1, 50, n - 60_000)], 4096)
    ids = rng.permutation(n).astype(np.int32)
    identity, nid = None, 0
    if case == "duplicates":
        ids[5] = ids[6]
    elif case == "missing_and_dup":
        ids[:100] = ids[100:200]
    elif case == "identity_map":
        nid = 70_000
        identity = np.concatenate([np.arange(nid), rng.integers(0, nid, n - nid)]).astype(np.int64)
        w.identity, w.num_identities = identity, nid
    tok_off, toks, ident = synth.device_tensors(w, "cuda")
    dwin = odb.DeviceWindow(w.rank_off, tok_off, toks, ident, nid)
    ws = torch.empty(odb.odb_workspace_size(dwin), dtype=torch.uint8, device="cuda")
    emitted = torch.from_numpy(ids[:70_000].copy()).cuda()
    left = torch.from_numpy(ids[70_000:].copy()).cuda()
    log(f"coverage case {case}")
    info = odb.odb_check_coverage(dwin, emitted, emitted.numel(), left, left.numel(), ws)
    bad, miss, dup = _numpy_coverage(ids.astype(np.int64), n, identity, nid)
    assert (info["bad_views"], info["missing_ids"], info["duplicate_ids"]) == (bad, miss, dup)


SKETCH_CV_RTOL = 1e-15   # both sides: a few correctly rounded fp64 operations on exact integers


def _compare_sketch(got, want):
    for f in ("samples", "short_samples", "sum_len", "sum_sq", "min_len", "max_len", "high_roi"):
        assert got[f] == want[f], (f, got[f], want[f])
    assert got["short_fraction"] == want["short_fraction"]
    assert abs(got["mean"] - want["mean"]) <= 2.0 ** -52 * want["mean"]
    assert abs(got["cv"] - want["cv"]) <= SKETCH_CV_RTOL * max(want["cv"], 1e-300), (got["cv"], want["cv"])


@pytest.mark.parametrize("name", list(synth.WORKLOADS))
def test_length_sketch(name):
    # the screen the practical-guidance section prescribes: a 1k-5k sketch (ids drawn
    # without replacement), plus leading prefixes of the window
    import torch
    import paper_2606_19989_amd as odb

    w = synth.WORKLOADS[name].window()
    tok_off = torch.from_numpy(w.tok_off).cuda()
    win = odb.DeviceWindow(w.rank_off, tok_off, torch.zeros(4, dtype=torch.int32, device="cuda"), None, 0)
    ws = torch.empty(odb.odb_workspace_size(win), dtype=torch.uint8, device="cuda")
    rng = np.random.default_rng(51)
    log(f"sketch {name}: n={w.n}")
    for k in (1000, 5000):
        ids = rng.choice(w.n, size=min(k, w.n), replace=False).astype(np.int32)
        got = odb.odb_length_sketch(win, torch.from_numpy(ids).cuda(), len(ids), w.budget, ws)
        _compare_sketch(got, oracle.length_sketch(w.tok_off, ids, w.budget))
    for count in (0, 1, min(w.n, 100_000)):
        got = odb.odb_length_sketch(win, None, count, w.budget, ws)
        _compare_sketch(got, oracle.length_sketch(w.tok_off, np.arange(count), w.budget))
    del ws, tok_off


def test_length_sketch_whole_window_and_edge_cases():
    import torch
    import paper_2606_19989_amd as odb

    w = synth.WORKLOADS["text_w8x65536"].window()
    tok_off = torch.from_numpy(w.tok_off).cuda()
    win = odb.DeviceWindow(w.rank_off, tok_off, torch.zeros(4, dtype=torch.int32, device="cuda"), None, 0)
    ws = torch.empty(odb.odb_workspace_size(win), dtype=torch.uint8, device="cuda")
    log("sketch whole window text_w8x65536")
    got = odb.odb_length_sketch(win, None, w.n, w.budget, ws)
    _compare_sketch(got, oracle.length_sketch(w.tok_off, None, w.budget))
    for budget in (1, 4, 700 * 4, 700 * 4 + 1, 1 << 40):
        ids = np.array([0, 0, 5, w.n - 1, 5], dtype=np.int32)   # repeated ids count every time
        got = odb.odb_length_sketch(win, torch.from_numpy(ids).cuda(), len(ids), budget, ws)
        _compare_sketch(got, oracle.length_sketch(w.tok_off, ids, budget))
    # an id outside the window is caught by the kernel's own bounds check
    bad = torch.tensor([3, w.n], dtype=torch.int32, device="cuda")
    with pytest.raises(odb.OdbError) as e:
        odb.odb_length_sketch(win, bad, 2, w.budget, ws)
    assert e.value.status == odb.ODB_E_INVALID_DATA


@pytest.mark.parametrize("count", [16384, 16385, 20480, 20481, 1 << 20, (1 << 20) + 4097])
def test_length_sketch_block_edges(count):
    """One block, the fewest and the most small blocks, the fewest large ones, one per compute
    unit and a grid that strides, with and without ids."""
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(count)
    n = (1 << 20) + 5000
    off = np.concatenate([[0], np.cumsum(rng.integers(1, 40000, n))]).astype(np.int64)
    win = odb.DeviceWindow(np.array([0, n], np.int64), torch.from_numpy(off).cuda(),
                           torch.zeros(1, dtype=torch.int32, device="cuda"), None, 0)
    ws = torch.empty(odb.odb_workspace_size(win), dtype=torch.uint8, device="cuda")
    log(f"sketch edge {count}")
    ids = rng.integers(0, n, count).astype(np.int32)
    got = odb.odb_length_sketch(win, torch.from_numpy(ids).cuda(), count, 1 << 16, ws)
    _compare_sketch(got, oracle.length_sketch(off, ids, 1 << 16))
    got = odb.odb_length_sketch(win, None, count, 1 << 16, ws)
    _compare_sketch(got, oracle.length_sketch(off, np.arange(count), 1 << 16))


def test_length_sketch_sums_past_64_bits():
    # lengths near 2^31: the sum of squares passes 2^64 (the 128-bit accumulation), at a
    # budget of 2^40 (the short-sample test 4 l < L_max in 64 bits)
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(53)
    n = 6000
    lens = np.concatenate([rng.integers(1 << 30, 1 << 31, n - 4), [(1 << 31) - 1, 1, (1 << 31) - 1, 7]])
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    tok_off = torch.from_numpy(off).cuda()
    win = odb.DeviceWindow(np.array([0, n], np.int64), tok_off, torch.zeros(4, dtype=torch.int32, device="cuda"),
                           None, 0)
    ws = torch.empty(odb.odb_workspace_size(win), dtype=torch.uint8, device="cuda")
    want = oracle.length_sketch(off, None, 1 << 40)
    assert want["sum_sq"] >= 1 << 64
    log("sketch past 64 bits")
    _compare_sketch(odb.odb_length_sketch(win, None, n, 1 << 40, ws), want)
    ids = rng.integers(0, n, 5000).astype(np.int32)   # with repeats
    for budget in (1 << 40, 1 << 33, 7):
        got = odb.odb_length_sketch(win, torch.from_numpy(ids).cuda(), len(ids), budget, ws)
        _compare_sketch(got, oracle.length_sketch(off, ids, budget))


def test_collate_tile_width_at_the_length_limit():
    # tiles 2^31 - 1 and 2^31 - 2 elements wide (the longest valid samples): a 4-element
    # group that starts 1 to 3 columns before a row's end must still take the row-edge
    # path there (column + 4 is past 2^31); every element around each row edge and a
    # random sample are checked against the oracle's per-element rule
    import torch

    top = (1 << 31) - 1
    for lens, name in (([top, top, top - 1], "width_2p31m1"), ([top - 1, top - 1, 5, top - 2], "width_2p31m2")):
        w = win([np.array(lens, np.int64)], 1 << 40)
        w.name = name
        log(f"collate at the length limit: {name}, {int(w.tok_off[-1])} tokens")
        ref = oracle.plan_window(w)
        pipe, outs = run_gpu(w)
        compare_plan(w, pipe, ref)
        P = ref.padded_elems
        edges = []
        for k in range(len(ref.slot_rows)):
            t0, ml, rows = int(ref.slot_tile_off[k]), int(ref.slot_maxlen[k]), int(ref.slot_rows[k])
            for r in range(1, rows + 1):
                edges.append(np.arange(t0 + r * ml - 24, t0 + r * ml + 24))
        idx = np.concatenate(edges + [np.random.default_rng(5).integers(0, P, 20000), [0, P - 1]])
        idx = np.unique(idx[(idx >= 0) & (idx < P)])
        want = oracle.collate_elements(ref, w.tok_off, synth.token_ids, idx, 0)
        ti = torch.from_numpy(idx).cuda()
        for label, g, e in zip(["input_ids", "labels", "attention_mask", "position_ids"], outs, want):
            got = g[ti].cpu().numpy()
            bad = np.nonzero(got != e)[0]
            assert len(bad) == 0, f"{name} {label}: {len(bad)} mismatches, first at {idx[bad[0]]}"
        del pipe, outs, ti
        torch.cuda.synchronize()
        torch.cuda.empty_cache()


def test_collate_from_emit_order():
    # odb_collate without row records gathers them from the emitted ids itself; both
    # routes give the oracle's outputs
    import torch
    import paper_2606_19989_amd as odb

    for w in (synth.WORKLOADS["ln512_w2x2048"].window(), adversarial_windows()[4], adversarial_windows()[16]):
        log(f"collate from emit order: {w.name}")
        ref = oracle.plan_window(w)
        pipe, outs = run_gpu(w, pad_id=3)
        P = int(pipe.info["padded_elems"])
        alt = tuple(torch.empty(max(P, 1), dtype=torch.int32, device="cuda") for _ in range(4))
        odb.odb_collate(pipe.win, pipe.num_slots, pipe.emit_order, pipe.slot_rows, pipe.slot_maxlen,
                        pipe.slot_row_off, pipe.slot_tile_off, 3, P, *alt, pipe.ws)
        torch.cuda.synchronize()
        odb.odb_collate_status(pipe.ws)
        compare_collate_full(w, tuple(a[:P] for a in alt), ref, 3)
        for a, b in zip(alt, outs):
            assert torch.equal(a[:P], b)


def test_collate_output_capacity():
    # outputs shorter than the padded size: the first out_capacity elements are the
    # oracle's and nothing at or past out_capacity is written, with and without row
    # records, at capacities that end inside a group, a step and a run of steps
    import torch
    import paper_2606_19989_amd as odb

    w = synth.WORKLOADS["ln512_w2x2048"].window()
    ref = oracle.plan_window(w)
    pipe, outs = run_gpu(w, pad_id=5)
    compare_collate_full(w, outs, ref, 5)
    P = int(pipe.info["padded_elems"])
    assert P > 70000
    sentinel = -12345
    for cap in (0, 1, 3, 1023, 1025, 65 * 1024 + 7, P - 1):
        for records in (True, False):
            log(f"collate with out_capacity={cap} of {P}, row records={records}")
            alt = tuple(torch.full((P + 64,), sentinel, dtype=torch.int32, device="cuda") for _ in range(4))
            rec = dict(row_token_start=pipe.row_token_start, row_len=pipe.row_len) if records else {}
            odb.odb_collate(pipe.win, pipe.num_slots, pipe.emit_order, pipe.slot_rows, pipe.slot_maxlen,
                            pipe.slot_row_off, pipe.slot_tile_off, 5, cap, *alt, pipe.ws, **rec)
            torch.cuda.synchronize()
            odb.odb_collate_status(pipe.ws)
            for a, b in zip(alt, outs):
                assert torch.equal(a[:cap], b[:cap])
                assert bool((a[cap:] == sentinel).all())


def test_concurrent_collates():
    # two collates in flight at once on two streams, each with its own workspace (and so
    # its own run counter) and outputs, repeated: both give the oracle's outputs
    import torch
    import paper_2606_19989_amd as odb

    w = synth.WORKLOADS["ln512_w2x2048"].window()
    ref = oracle.plan_window(w)
    pipes = []
    for pad in (2, 9):
        pipe, outs = run_gpu(w, pad_id=pad)
        compare_collate_full(w, outs, ref, pad)
        pipes.append((pipe, outs, pad))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    P = int(pipes[0][0].info["padded_elems"])
    alts = [tuple(torch.full((P,), -1, dtype=torch.int32, device="cuda") for _ in range(4)) for _ in pipes]
    torch.cuda.synchronize()
    for rep in range(3):
        log(f"two concurrent collates, repetition {rep}")
        for (pipe, _, pad), alt, st in zip(pipes, alts, streams):
            odb.odb_collate(pipe.win, pipe.num_slots, pipe.emit_order, pipe.slot_rows, pipe.slot_maxlen,
                            pipe.slot_row_off, pipe.slot_tile_off, pad, P, *alt, pipe.ws, st,
                            row_token_start=pipe.row_token_start, row_len=pipe.row_len)
        torch.cuda.synchronize()
        for (pipe, outs, _), alt in zip(pipes, alts):
            odb.odb_collate_status(pipe.ws)
            for a, b in zip(alt, outs):
                assert torch.equal(a, b)
            for a in alt:
                a.fill_(-1)
        torch.cuda.synchronize()


def _formed(w):
    import torch
    import paper_2606_19989_amd as odb

    tok_off, toks, ident = synth.device_tensors(w, "cuda")
    win_ = odb.DeviceWindow(w.rank_off, tok_off, toks, ident, w.num_identities)
    pipe = odb.Pipeline(win_, w.budget, mode=w.mode, quota=w.quota, capacity=w.capacity)
    pipe.form()
    torch.cuda.synchronize()
    return pipe


@pytest.mark.parametrize("mode", ["join", "nonjoin"])
def test_align_rejects_a_wrong_sorted_length(mode):
    # a stage-1 sorted length that keeps the order valid but is not the sample's CSR
    # length is found once the plan is built (emitted rows, or leftovers in non-join)
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(31)
    w = win([rng.integers(10, 3000, 5000), rng.integers(10, 3000, 3000)], 8192, mode=mode,
            quota=2000 if mode == "nonjoin" else 0)
    pipe = _formed(w)
    ref = oracle.plan_window(w)
    slen = pipe.sorted_len.cpu().numpy()
    # a position strictly inside a run of descending lengths: lowering its length by one
    # keeps (length desc, id asc).  Non-join emits the shortest samples first, so a long
    # one (an early position) is left over and checked on that path
    cand = [p for p in range(1, 4999) if slen[p - 1] > slen[p] > slen[p + 1] + 1]
    p = cand[len(cand) // 2] if mode == "join" else cand[0]
    order = pipe.order.cpu().numpy()
    if mode == "nonjoin":
        assert order[p] in set(ref.leftover.tolist())
    bad = pipe.sorted_len.clone()
    bad[p] -= 1
    pipe.sorted_len.copy_(bad)
    log(f"wrong sorted length at position {p} ({mode}); the oracle leaves {ref.info['leftover_samples']} over")
    with pytest.raises(odb.OdbError) as e:
        pipe.align()
    assert e.value.status == odb.ODB_E_INVALID_DATA
    assert "sorted length" in str(e.value)


def test_collate_flags_a_bad_row_record():
    # a row record outside the token stream is written as padding and reported
    import torch
    import paper_2606_19989_amd as odb

    w = synth.WORKLOADS["ln512_w2x2048"].window()
    pipe, outs = run_gpu(w)
    P = int(pipe.info["padded_elems"])
    pipe.row_token_start[5] = int(w.tok_off[-1])   # starts at the end of the stream
    pipe.collate()
    torch.cuda.synchronize()
    with pytest.raises(odb.OdbError) as e:
        odb.odb_collate_status(pipe.ws)
    assert e.value.status == odb.ODB_E_INVALID_DATA
    pipe.row_token_start[5] = int(w.tok_off[int(pipe.emit_order[5])])
    pipe.collate()
    torch.cuda.synchronize()
    odb.odb_collate_status(pipe.ws)
    ref = oracle.plan_window(w)
    compare_collate_full(w, tuple(o[:P] for o in pipe.outputs), ref)


def test_two_stream_schedule():
    # the benchmark's schedule: step i+1's plan on one stream beside step i's collate on
    # another, two plan buffers, one set of outputs; after several steps the outputs and
    # both plans are the oracle's
    import torch
    import paper_2606_19989_amd as odb
    import bench

    w = synth.WORKLOADS["text_w8x65536"].window()
    log(f"two-stream schedule on {w.name}")
    plan_stream, collate_stream = torch.cuda.Stream(), torch.cuda.Stream()
    tok_off, toks, ident = synth.device_tensors(w, "cuda")
    dwin = odb.DeviceWindow(w.rank_off, tok_off, toks, ident, w.num_identities)
    pipes = [odb.Pipeline(dwin, w.budget, mode=w.mode, quota=w.quota) for _ in range(2)]
    for p in pipes:
        p.run()
        pipes[1].outputs = pipes[0].outputs
    torch.cuda.synchronize()
    pipes[0].outputs[0].fill_(-7)
    sec, coll, _ = bench.pipelined_steps(pipes, plan_stream, collate_stream, 5)
    assert len(coll) == 5 and sec > 0
    ref = oracle.plan_window(w)
    for p in pipes:
        odb.odb_collate_status(p.ws)
        compare_plan(w, p, ref)
    P = ref.padded_elems
    outs = tuple(o[:P] for o in pipes[0].outputs)
    compare_collate_sampled(w, outs, ref)
    collate_properties(outs, ref)
    compare_collate_by_rank(w, outs, ref, toks)


def one_round_windows():
    """Windows aligned in one round, and the edges of that path: ranks at the edges of a
    block's tile (1,024 positions, 4 per thread), ranks dealt to the XCDs (8 and more) or not,
    empty ranks, one slot per sample and one slot per rank (lanes per slot 1 to 64), more
    slot ranges than blocks, splits with X = 0 and at the last group, quotas inside and at a
    step's end, an identity map, and windows that turn out to overflow and start over."""
    rng = np.random.default_rng(91)
    U = lambda lo, hi, n: rng.integers(lo, hi, size=n)
    win = synth.window_from_ranks
    out = []
    for n in (1, 3, 4, 5, 1023, 1024, 1025, 2049):
        out.append(win(f"tile_{n}", [U(50, 60, n), U(50, 60, max(n - 1, 1))], 240))
    out.append(win("xcd_ranks", [U(20, 900, 1500 + 7 * r) for r in range(11)], 8192))
    out.append(win("empty_ranks", [U(5, 50, 400), U(1, 2, 0), U(5, 50, 399), U(1, 2, 0)], 300))
    out.append(win("singletons", [U(100, 900, 3000) for _ in range(9)], 100))
    out.append(win("one_group", [U(1, 9, 5000), U(1, 9, 4000)], 1 << 20))
    out.append(win("few_rows", [U(30, 60, 70000)], 130))
    out.append(win("deep_split", [U(1000, 1001, 900), U(1, 3, 900)], 1000))
    out.append(win("split_last", [U(10, 11, 40), np.concatenate([U(90, 91, 3), U(1, 2, 37)])], 100))
    out.append(win("overflow_restart", [U(500, 900, 300), U(10, 20, 7)], 1000))
    out.append(win("very_ragged", [U(10, 400, 60000)] + [U(10, 400, 200 + r) for r in range(70)], 2000))
    for q in (1, 2, 700, 2999, 3000, 5000):
        out.append(win(f"quota_{q}", [U(10, 700, 1000 + 13 * r) for r in range(3)], 4096, mode="nonjoin", quota=q))
    # equal lengths: every step but the first holds the same samples, so the quota can fall on
    # a step's end
    for q in (2, 3 * 16 + 2, 3 * 16 + 3):
        out.append(win(f"quota_even_{q}", [np.full(333, 100), np.full(333, 100)], 800, mode="nonjoin", quota=q))
    # ranks split from 64, 66, about 2,000 and about 6,000 groups (the split is searched 64 places
    # at a time), towards one of 7,000
    split = [U(1000, 1001, 7000)] + [np.concatenate([U(400, 1000, g), U(1, 9, 7000 - g)]) for g in (60, 62, 2000, 6000)]
    for q in (500, 20000):
        out.append(win(f"quota_split_{q}", split, 1000, mode="nonjoin", quota=q))
    out.append(win("quota_overflow", [U(500, 900, 300), U(10, 20, 7)], 1000, mode="nonjoin", quota=250))
    out.append(win("quota_empty_rank", [U(10, 20, 100), U(1, 2, 0)], 100, mode="nonjoin", quota=50))
    for mode, q in (("join", 0), ("nonjoin", 900)):
        ident = rng.permutation(1990)
        ident = np.concatenate([ident, ident[:10]]).astype(np.int64)
        out.append(win(f"identities_{mode}", [U(10, 400, 500) for _ in range(4)], 2048, mode=mode, quota=q,
                       identity=ident, num_identities=1990))
    out.append(win("capacity_free", [U(10, 300, 400), U(10, 300, 500)], 2000, capacity=np.array([500, 0])))
    return out


@pytest.mark.parametrize("idx", range(len(one_round_windows())))
def test_one_round_windows(idx):
    w = one_round_windows()[idx]
    log(f"one round: {w.name}")
    ref = oracle.plan_window(w)
    pipe, outs = run_gpu(w, pad_id=idx)
    compare_plan(w, pipe, ref)
    compare_loss_weights(pipe, ref)
    compare_collate_full(w, outs, ref, pad_id=idx)


def overflow_windows():
    """A rank of one sample per group beside one that holds as many samples, one fewer (the window
    overflows and goes round by round) or one more; short ranks, and more than 16 tiles."""
    rng = np.random.default_rng(94)
    out = []
    for n in (50, 17000):
        for d in (0, -1, 1):
            for mode, q in (("join", 0), ("nonjoin", n + n // 3)):
                ident = np.concatenate([rng.permutation(2 * n + d - 2), [0, 1]]).astype(np.int64)
                out.append(synth.window_from_ranks(f"groups_{n}{d:+d}_{mode}", [
                    np.full(n, 100), rng.integers(1, 90, size=n + d)], 100, mode=mode, quota=q, identity=ident,
                    num_identities=2 * n + d - 2))
    return out


@pytest.mark.parametrize("idx", range(len(overflow_windows())))
def test_one_round_overflow_edge(idx):
    check_full(overflow_windows()[idx])


@pytest.mark.parametrize("mode", ["join", "nonjoin"])
@pytest.mark.parametrize("where", ["overflowing_rank", "other_rank", "groups"])
def test_overflow_reports_the_first_bad_position(where, mode):
    """Stage-1 arrays that are inconsistent in two places, in a window that overflows: the first place
    is named, whichever ranks the one-round attempt looked at."""
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(97)
    w = win([rng.integers(500, 900, 3000), rng.integers(10, 20, 700)], 1000, mode=mode, quota=1500 if mode == "nonjoin" else 0)
    pipe = _formed(w)
    assert int(pipe.groups_per_rank[0]) > 700
    first = {"overflowing_rank": 1200, "other_rank": 3100, "groups": 2000}[where]
    a = pipe.group_index if where == "groups" else pipe.order
    for p in (first, 3500):
        a[p] = -5 if where == "groups" else 0 if p >= 3000 else w.n - 1   # a group or an id of no rank of its own
    log(f"bad stage-1 arrays in an overflowing window: {where}, {mode}")
    with pytest.raises(odb.OdbError) as e:
        pipe.align()
    assert e.value.status == odb.ODB_E_INVALID_DATA
    assert f"first inconsistent position {first})" in str(e.value), str(e.value)


def short_round_windows():
    """Join windows of short ranks that take several rounds: rank sizes at the edges of the
    kernels (1, 1,023 .. 1,025, 16,383 and 16,384 positions; 16,385 takes the general path),
    rounds past the first chunk, the last group kept and returned, ranks that end early, a
    rank without capacity, an identity map, and steps listed from the budget or the samples."""
    rng = np.random.default_rng(92)
    U = lambda lo, hi, n: rng.integers(lo, hi, size=n)
    win = synth.window_from_ranks
    out = []
    for n in (1, 2, 1023, 1024, 1025, 16383, 16384, 16385):
        out.append(win(f"ranks_{n}", [U(10, 900, n), U(10, 900, max(1, n // 3))], 9000,
                       capacity=np.array([max(1, n // 90), 3 + n // 50])))
    out.append(win("one_slot", [U(10, 300, 700), U(10, 300, 650)], 2000, capacity=np.array([1, 0])))
    out.append(win("many_ranks", [U(10, 900, 300 + 5 * r) for r in range(67)], 4096,
                   capacity=np.arange(67) % 5 * 9))
    out.append(win("empty_and_small", [U(10, 900, 900), U(1, 2, 0), U(10, 900, 40), U(10, 900, 1)], 4096,
                   capacity=np.array([11, 4, 0, 2])))
    # equal lengths: the last group is one short of, equal to and one past a full one
    for n in (1 + 8 * 12 - 1, 1 + 8 * 12, 1 + 8 * 12 + 1, 9, 10):
        out.append(win(f"equal_{n}", [np.full(n, 100), U(50, 150, n + 5)], 800, capacity=np.array([4, 0])))
    out.append(win("tail_kept", [np.concatenate([U(400, 500, 60), U(10, 20, 90)]) for _ in range(3)], 1000,
                   capacity=np.array([7, 9, 0])))
    out.append(win("no_capacity", [U(500, 900, 900), U(10, 20, 5), U(100, 200, 300)], 1000))
    ident = np.concatenate([rng.permutation(1990), np.arange(10)]).astype(np.int64)
    out.append(win("identities", [U(10, 400, 500) for _ in range(4)], 2048, capacity=np.array([9, 0, 30, 12]),
                   identity=ident, num_identities=1990))
    out.append(win("by_sample", [U(1, 20000, 3000), U(1, 20000, 3500)], 1 << 40, capacity=np.array([1, 1])))
    out.append(win("general_steps", [U(1, 20000, 9000), U(1, 20000, 3500)], 1 << 40, capacity=np.array([1, 1])))
    return out


@pytest.mark.parametrize("idx", range(len(short_round_windows())))
def test_short_rank_rounds(idx):
    w = short_round_windows()[idx]
    log(f"short ranks: {w.name}")
    ref = oracle.plan_window(w)
    pipe, outs = run_gpu(w, pad_id=idx)
    compare_plan(w, pipe, ref)
    compare_loss_weights(pipe, ref)
    compare_collate_full(w, outs, ref, pad_id=idx)


def _align_reference(lens, groups, caps, budget):
    """Algorithm 1 over given first-round groups (lists of group sizes per rank, formation order
    over samples sorted by length desc, id asc): per rank the steps' (rows, longest, tokens)."""
    buf, steps = [], [[] for _ in lens]
    for r, l in enumerate(lens):
        o = np.lexsort((np.arange(len(l)), -l))
        buf.append((list(l[o]), np.cumsum([0] + list(groups[r]))[:-1].tolist() if len(l) else []))
    while any(b for b, _ in buf):
        T = max(len(g) for _, g in buf)
        T = max(1, min([T] + [len(b) for b, _ in buf if b] + [c for c, (b, _) in zip(caps, buf) if c > 0 and b]))
        nxt = []
        for r, (b, g) in enumerate(buf):
            parts = [b[x:y] for x, y in zip(g, g[1:] + [len(b)])]
            back = []
            if b and len(parts) < T:
                k, split = T - len(parts), []
                for p in parts:
                    while k and len(p) > 1:
                        split.append(p[:1])
                        p, k = p[1:], k - 1
                    split.append(p)
                parts = split
            elif len(parts) > T:
                keep = set(sorted(range(len(parts)), key=lambda i: (-len(parts[i]), -i))[:T])
                back = [x for i, p in enumerate(parts) if i not in keep for x in p]
                parts = [p for i, p in enumerate(parts) if i in keep]
            for j in range(T):
                p = parts[T - 1 - j] if parts else []
                steps[r].append((len(p), p[0] if p else 0, sum(p)))
            g2, p = [], 0
            while p < len(back):
                g2.append(p)
                p += 1 if p == 0 else max(budget // int(back[p - 1]), 1)
            nxt.append((back, g2))
        buf = nxt
    return np.array(steps)


@pytest.mark.parametrize("sizes", ["uneven", "falling", "fixed"])
@pytest.mark.parametrize("capped", [False, True])
def test_align_takes_any_consistent_groups(sizes, capped):
    """Group indices that odb_form_groups would not write (sizes that go up and down, or fall)
    are accepted as long as they step by 0 or 1, with and without overflow."""
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(93)
    lens = [rng.integers(1, 500, size=n) for n in (700, 655)]
    groups = []
    for l in lens:
        left, s = len(l), []
        while left:
            c = {"uneven": int(rng.integers(1, 30)), "falling": max(1, 40 - len(s)), "fixed": 7}[sizes]
            s.append(min(c, left))
            left -= s[-1]
        groups.append(s)
    caps = np.array([9, 14]) if capped else None
    w = synth.window_from_ranks("custom_groups", lens, 4000, capacity=caps)
    tok_off, toks, _ = synth.device_tensors(w, "cuda")
    win_ = odb.DeviceWindow(w.rank_off, tok_off, toks)
    pipe = odb.Pipeline(win_, w.budget, capacity=caps)
    pipe.form()
    gidx = np.concatenate([np.repeat(np.arange(len(s)), s) for s in groups]).astype(np.int32)
    pipe.group_index.copy_(torch.from_numpy(gidx))
    pipe.groups_per_rank.copy_(torch.tensor([len(s) for s in groups], dtype=torch.int32))
    info = pipe.align()
    ref = _align_reference(lens, groups, [0, 0] if caps is None else caps, w.budget)
    K = 2 * ref.shape[1]
    assert info["steps"] == ref.shape[1] and info["emitted_samples"] == w.n and info["bad_views"] == 0
    assert np.array_equal(pipe.slot_rows[:K].cpu().numpy(), ref[:, :, 0].reshape(-1))
    assert np.array_equal(pipe.slot_maxlen[:K].cpu().numpy(), ref[:, :, 1].reshape(-1))
    assert np.array_equal(pipe.slot_tokens[:K].cpu().numpy(), ref[:, :, 2].reshape(-1))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384])
def test_one_block_grouping_sizes(n):
    """Ranks at the edges of the one-block grouping's variants (positions per thread 1 to 16),
    beside a shorter rank, with one digit, two digits and four digits of lengths, and all equal."""
    rng = np.random.default_rng(n)
    m = max(1, n - 3)
    for lo, hi, budget in ((7, 8, 64), (1, 200, 900), (1, 20000, 60000), (1, 2 ** 31 - 1, 2 ** 40)):
        w = synth.window_from_ranks(f"form_{n}_{hi}", [rng.integers(lo, hi, n), rng.integers(lo, hi, m)], budget)
        ref = oracle.plan_window(w)
        import torch
        pipe, _ = run_gpu(w, tokens=torch.zeros(1, dtype=torch.int32, device="cuda"), collate=False)
        compare_plan(w, pipe, ref)


@pytest.mark.parametrize("span", [256, 257, 1 << 17, (1 << 17) + 1])
@pytest.mark.parametrize("per_rank", [1 << 15, (1 << 15) + 1])
def test_sort_word_widths(per_rank, span):
    """Key and position in exactly 32 bits (15 + 17) and in one more, in one, two and three passes;
    both ends of the range of lengths occur, at the last positions of a rank, too."""
    import torch
    rng = np.random.default_rng(96)
    lens = [rng.integers(1, span + 1, n) for n in (per_rank, 17, per_rank - 5)]
    lens[0][-2:] = 1, span
    lens[0][:2] = 1, span
    w = synth.window_from_ranks("sort_words", lens, 1 << 20)
    ref = oracle.plan_window(w)
    pipe, _ = run_gpu(w, tokens=torch.zeros(1, dtype=torch.int32, device="cuda"), collate=False)
    compare_plan(w, pipe, ref)


@pytest.mark.parametrize("longest,budget", [(3000, 20000), (3, 1 << 18), (40000, 1 << 17)])
@pytest.mark.parametrize("per_rank", [1 << 19, (1 << 19) + 1])
def test_chain_remainder_widths(per_rank, longest, budget):
    """The largest rank whose group chain is carried in fp32 and one sample more (integers), with
    hundreds of runs, with steps of up to half the rank, and with few samples a group."""
    import torch
    rng = np.random.default_rng(98)
    w = synth.window_from_ranks("chain_widths", [rng.integers(1, longest + 1, per_rank), rng.integers(1, longest + 1, 90)],
                                budget)
    ref = oracle.plan_window(w)
    pipe, _ = run_gpu(w, tokens=torch.zeros(1, dtype=torch.int32, device="cuda"), collate=False)
    compare_plan(w, pipe, ref)


@pytest.mark.parametrize("per_rank", [(1 << 22) // 3 + 1, (1 << 22) // 3])
def test_sort_tile_lengths(per_rank):
    """Windows just at and just below 4 Mi samples: the longer and the shorter radix tile, ragged
    against both, with a one-sample and an empty rank between."""
    import torch
    rng = np.random.default_rng(95)
    sizes = [per_rank, 0, per_rank - 1, 1, per_rank + 1]
    w = synth.window_from_ranks("sort_tiles", [rng.integers(1, 5000, n) for n in sizes], 1 << 20)
    ref = oracle.plan_window(w)
    pipe, _ = run_gpu(w, tokens=torch.zeros(1, dtype=torch.int32, device="cuda"), collate=False)
    compare_plan(w, pipe, ref)


@pytest.mark.parametrize("W,S", [(1, 32767), (1, 32768), (2, 40001), (3, 100003), (8, 32768), (10, 32767), (10, 32768),
                                 (11, 49151), (11, 49152), (12, 65536), (24, 196608), (24, 262144), (25, 300001), (32, 196607), (32, 196608), (33, 200000)])
def test_loss_weights_few_ranks(W, S):
    # both sides of the line between one thread per step and the waves over the ranks; the reference adds
    # the ranks in order, one fp64 operation each, as the library states
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(W)
    rows = rng.integers(0, 50, (W, S)).astype(np.int32)
    rows[:, ::97] = 0   # steps without a sample: zero weights
    tokens = rows.astype(np.int64) * rng.integers(1, 3000, (W, S))
    approx = rows * rng.uniform(1.0, 3000.0, (W, S))
    d = [torch.from_numpy(x).cuda() for x in (rows, tokens, approx)]
    a_sum = np.zeros(S)
    for r in range(W):
        a_sum = a_sum + approx[r]
    t_sum, n_sum = tokens.sum(0), rows.sum(0, dtype=np.int64)
    for mode, x, total in ((oracle.WEIGHT_SAMPLE, rows, n_sum), (oracle.WEIGHT_TOKEN_APPROX, approx, a_sum),
                           (oracle.WEIGHT_TOKEN_EXACT, tokens, t_sum)):
        log(f"loss weights {W} x {S}, mode {mode}")
        wt = torch.empty(W * S, dtype=torch.float64, device="cuda")
        st, ss = (torch.empty(S, dtype=torch.int64, device="cuda") for _ in range(2))
        odb.odb_loss_weights(W, S, mode, *d, wt, st, ss)
        den = total.astype(np.float64)
        want = np.where(total > 0, x.astype(np.float64) / np.where(total > 0, den, 1.0), 0.0)
        assert np.array_equal(wt.cpu().numpy().reshape(W, S).view(np.int64), want.view(np.int64)), mode
        assert np.array_equal(st.cpu().numpy(), t_sum) and np.array_equal(ss.cpu().numpy(), n_sum)


@pytest.mark.parametrize("W", [63, 64, 65, 128, 129, 700])
def test_quota_cut_of_many_ranks(W):
    # one slice of 64 ranks, several, and a last one of a single rank; of unequal size, so that most are split
    rng = np.random.default_rng(W)
    ranks = [rng.integers(1, 3000, 200 + r % 60) for r in range(W)]
    n = sum(map(len, ranks))
    for q in (1, W, n // 2, n - 1, n + 1):
        w = win(ranks, 20000, mode="nonjoin", quota=q)
        log(f"quota {q} of {n} over {W} ranks")
        ref = oracle.plan_window(w)
        pipe, _ = run_gpu(w, collate=False)
        compare_plan(w, pipe, ref)
        compare_loss_weights(pipe, ref)
