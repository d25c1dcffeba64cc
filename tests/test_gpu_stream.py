"""GPU parity of the unified streaming loop (odb_stream_plan) with the oracle: every plan
array, the per-round trace, the summary, the loss weights bit for bit and, on small
cases, every collate element."""
import numpy as np
import pytest

import oracle
import synth
from _parity import compare_row_records, log

pytestmark = pytest.mark.gpu

STREAM_INFO_EXACT = ["steps", "rounds", "emit_rounds", "skip_rounds", "stop_reason", "views", "emitted_views",
                     "undelivered_views", "pending_views", "real_tokens", "padded_elems", "max_step_samples",
                     "splits", "overflow_groups", "missing_ids", "duplicate_ids", "bad_views",
                     "second_gather_rounds", "max_outstanding"]


def offsets(lens):
    return np.concatenate([[0], np.cumsum(np.asarray(lens, dtype=np.int64))])


def run_case(name, lens, perm, W, budget, buffer_size, depth, rate, mode="join", quota=0, cap=None, pad_id=0,
             full_collate=True, tokens=None, max_rounds=None, device_perm=None, slot_capacity=None):
    import torch
    import paper_2606_19989_amd as odb

    N = len(lens)
    log(f"stream case {name}: N={N} W={W} budget={budget} buffer={buffer_size} depth={depth} mode={mode} "
        f"quota={quota} rate={list(rate)[:8]}")
    tok_off = offsets(lens)
    m_mode = oracle.MODE_NONJOIN if mode == "nonjoin" else oracle.MODE_JOIN
    ref = oracle.stream(tok_off, perm, W, budget, mode=m_mode, quota=quota, buffer_size=buffer_size, depth=depth,
                        rate=rate, capacity=cap)
    rank_off = np.linspace(0, N, W + 1).astype(np.int64)   # not used by the streaming loop
    d_tok_off = torch.from_numpy(tok_off).cuda()
    toks = tokens if tokens is not None else synth.fill_tokens_torch(int(tok_off[-1]), "cuda")
    win = odb.DeviceWindow(rank_off, d_tok_off, toks, None, 0)
    dperm = perm if device_perm is None else device_perm
    sp = odb.StreamPipeline(win, torch.from_numpy(np.asarray(dperm, dtype=np.int32)).cuda(), budget,
                            buffer_size=buffer_size, depth=depth, rate=rate, mode=mode, quota=quota, capacity=cap,
                            pad_id=pad_id, max_rounds=max_rounds, slot_capacity=slot_capacity)
    info = sp.plan()
    torch.cuda.synchronize()
    for f in STREAM_INFO_EXACT:
        assert info[f] == ref.sinfo[f], (f, info[f], ref.sinfo[f])
    assert abs(info["pad_fraction"] - ref.sinfo["pad_fraction"]) <= 1e-12 * max(ref.sinfo["pad_fraction"], 1e-300)
    assert np.array_equal(sp.trace_array(), ref.trace), "trace"
    S, K, M = ref.steps, W * ref.steps, ref.sinfo["views"]
    E = ref.sinfo["emitted_views"]
    h = lambda t, k: t[:k].cpu().numpy()
    assert np.array_equal(h(sp.slot_rows, K), ref.slot_rows), "slot_rows"
    assert np.array_equal(h(sp.slot_maxlen, K), ref.slot_maxlen), "slot_maxlen"
    assert np.array_equal(h(sp.slot_tokens, K), ref.slot_tokens), "slot_tokens"
    assert np.array_equal(h(sp.slot_tokens_approx, K).view(np.int64), ref.slot_tokens_approx.view(np.int64))
    assert np.array_equal(h(sp.slot_row_off, K + 1), ref.slot_row_off), "slot_row_off"
    assert np.array_equal(h(sp.slot_tile_off, K + 1), ref.slot_tile_off), "slot_tile_off"
    assert np.array_equal(h(sp.emit_views, E), ref.emit_views), "emit_views"
    assert np.array_equal(h(sp.emit_order, E), ref.emit_order), "emit_order"
    compare_row_records(tok_off, sp, ref.emit_order)
    assert np.array_equal(h(sp.left_views, M - E), ref.left_views), "left_views"
    assert np.array_equal(h(sp.left_off, W + 1), ref.left_off), "left_off"
    for m in (oracle.WEIGHT_SAMPLE, oracle.WEIGHT_TOKEN_APPROX, oracle.WEIGHT_TOKEN_EXACT):
        wt, st, ss = sp.loss_weights(m)
        ewt, est, ess = ref.loss_weights(m)
        assert np.array_equal(wt.cpu().numpy().view(np.int64), ewt.view(np.int64)), ("weights", m)
        assert np.array_equal(st.cpu().numpy(), est) and np.array_equal(ss.cpu().numpy(), ess)
    if full_collate:
        outs = sp.collate()
        torch.cuda.synchronize()
        odb.odb_collate_status(sp.ws)
        want = ref.collate(tok_off, toks.cpu().numpy(), pad_id)
        for name_, g, e in zip(["input_ids", "labels", "attention_mask", "position_ids"], outs, want):
            assert np.array_equal(g.cpu().numpy(), e), name_
    return sp, ref


def edge_cases():
    rng = np.random.default_rng(71)
    out = []
    add = lambda name, lens, W, budget, buf, depth, rate, **kw: out.append(
        (name, np.asarray(lens, dtype=np.int64), W, budget, buf, depth, np.asarray(rate, dtype=np.int32), kw))
    add("empty", [], 3, 100, 4, 4, [4, 4, 4])
    add("one_sample_four_ranks", [7], 4, 100, 2, 3, [1, 2, 3, 1])           # padding wraps N = 1 times 3
    add("fewer_samples_than_ranks", [5, 9, 2], 5, 12, 1, 1, [1] * 5)
    add("buffer_one", rng.integers(1, 50, 40), 3, 30, 1, 1, [1, 1, 1])
    add("slow_rank", rng.integers(1, 900, 700), 4, 4096, 64, 64, [1, 64, 64, 64])
    add("deep_envelope", rng.integers(1, 900, 3000), 3, 8192, 128, 1024, [300, 17, 128])
    add("tiny_budget", rng.integers(1, 9, 500), 2, 1, 50, 80, [20, 80])
    add("overflow_capacity", rng.integers(1, 600, 1500), 3, 3000, 200, 256, [256, 100, 50], cap=np.array([3, 0, 5]))
    add("max_depth", rng.integers(1, 3000, 20000), 2, 16384, 4096, 4096, [4096, 4096])
    # depth 1500: four sort keys per thread; skip rounds while the slow rank fills
    add("depth_1500", rng.integers(1, 5000, 12000), 3, 12000, 1200, 1500, [1500, 700, 1500])
    # one rank with 600,000 views: its emitted-view bits exceed the LDS budget and are set
    # in global memory
    add("long_rank", rng.integers(1, 12, 600000), 1, 64, 1024, 1024, [1024])
    # more ranks than a round block has threads (the round decision loops over them)
    add("many_ranks", rng.integers(1, 300, 4000), 600, 2000, 4, 4, [2] * 600)
    n = 2003
    for q in (1, 500, n + 1):
        add(f"nonjoin_q{q}", rng.integers(1, 2000, n), 4, 6000, 100, 150, [150, 90, 40, 150], mode="nonjoin",
            quota=q)
    add("nonjoin_capacity", rng.integers(1, 900, 900), 2, 2500, 64, 64, [64, 7], mode="nonjoin", quota=700,
        cap=np.array([2, 4]))
    return out


@pytest.mark.parametrize("idx", range(len(edge_cases())))
def test_stream_edge_cases(idx):
    name, lens, W, budget, buf, depth, rate, kw = edge_cases()[idx]
    perm = np.random.default_rng(idx).permutation(len(lens)).astype(np.int32)
    run_case(name, lens, perm, W, budget, buf, depth, rate, pad_id=idx, **kw)


def test_stream_random_small():
    rng = np.random.default_rng(72)
    for t in range(30):
        N = int(rng.integers(1, 3000))
        W = int(rng.integers(1, 9))
        lens = rng.integers(1, int(rng.integers(2, 4000)), size=N)
        buf = int(rng.integers(1, 300))
        depth = buf + int(rng.integers(0, 200))
        rate = rng.integers(1, depth + 1, size=W).astype(np.int32)
        mode = "nonjoin" if t % 3 == 2 else "join"
        cap = rng.integers(0, 6, size=W) if t % 4 == 1 else None
        run_case(f"random_{t}", lens, rng.permutation(N).astype(np.int32), W, int(rng.integers(1, 30000)), buf, depth,
                 rate, mode=mode, quota=int(rng.integers(1, N + 2)), cap=cap, pad_id=t % 5)


def _stream_pipeline(lens, perm, W, budget, buffer_size, depth, rate, **kw):
    import torch
    import paper_2606_19989_amd as odb

    tok_off = offsets(lens)
    win = odb.DeviceWindow(np.linspace(0, len(lens), W + 1).astype(np.int64), torch.from_numpy(tok_off).cuda(),
                           synth.fill_tokens_torch(int(tok_off[-1]), "cuda"), None, 0)
    return odb.StreamPipeline(win, torch.from_numpy(np.asarray(perm, dtype=np.int32)).cuda(), budget,
                              buffer_size=buffer_size, depth=depth, rate=np.asarray(rate, dtype=np.int32), **kw)


@pytest.mark.parametrize("mode", ["join", "nonjoin"])
def test_stream_round_limit(mode):
    # rounds are enqueued in chunks sized by a lower bound on the rounds left (a slow rank
    # makes the first bound short, so later chunks follow): a limit equal to the rounds
    # the iteration takes passes and matches the oracle, one round fewer is a capacity
    # error, and so is a limit of one round
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(76)
    N, W = 700, 4
    lens = rng.integers(1, 900, N)
    perm = rng.permutation(N).astype(np.int32)
    rate = np.array([3, 64, 64, 64], np.int32)
    kw = dict(mode=mode, quota=N // 2 if mode == "nonjoin" else 0)
    m_mode = oracle.MODE_NONJOIN if mode == "nonjoin" else oracle.MODE_JOIN
    ref = oracle.stream(offsets(lens), perm, W, 4096, mode=m_mode, quota=kw["quota"], buffer_size=64, depth=64,
                        rate=rate)
    R = int(ref.sinfo["rounds"])
    log(f"round limit {mode}: the iteration takes {R} rounds")
    assert R > 20
    run_case(f"round_limit_{mode}", lens, perm, W, 4096, 64, 64, rate, max_rounds=R, **kw)
    for limit in (R - 1, 1):
        sp = _stream_pipeline(lens, perm, W, 4096, 64, 64, rate, max_rounds=limit, **kw)
        with pytest.raises(odb.OdbError) as e:
            sp.plan()
        assert e.value.status == odb.ODB_E_CAPACITY, limit


@pytest.mark.parametrize("bad", ["perm", "length"])
def test_stream_rejects_bad_data(bad):
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(77)
    N, W = 60, 3
    lens = rng.integers(1, 50, N)
    perm = rng.permutation(N).astype(np.int32)
    if bad == "perm":
        perm[17] = N       # outside [0, N)
    else:
        lens[perm[17]] = 0
    sp = _stream_pipeline(lens, perm, W, 200, 4, 4, [4, 4, 4])
    with pytest.raises(odb.OdbError) as e:
        sp.plan()
    assert e.value.status == odb.ODB_E_INVALID_DATA


def test_stream_ignores_views_after_the_stop():
    # the grouping of the round after the one that meets a non-join quota runs before the
    # quota is known, and must leave no trace: a perm entry outside [0, N) for a view only
    # that round fetches does not fail the call, and the plan is the one of the valid perm
    rng = np.random.default_rng(78)
    N, W = 40, 2
    lens = rng.integers(1, 30, N)
    perm = rng.permutation(N).astype(np.int32)
    bad = perm.copy()
    bad[8] = N          # view 8: rank 0's first view of the second round
    sp, ref = run_case("stop_then_bad_view", lens, perm, W, 100, 4, 4, [4, 4], mode="nonjoin", quota=1,
                       device_perm=bad)
    assert ref.sinfo["rounds"] == 1 and ref.sinfo["stop_reason"] == oracle.STOP_QUOTA


def test_stream_window_workload():
    # the multimodal window's samples as a dataset streamed through 8 ranks with the
    # paper's default buffer of 1024 and unequal worker throughput
    w = synth.WORKLOADS["mm_w8x262144"].window()
    lens = np.diff(w.tok_off)
    rng = np.random.default_rng(73)
    perm = rng.permutation(len(lens)).astype(np.int32)
    rate = np.array([1024, 512, 1024, 256, 1024, 1024, 768, 1024], dtype=np.int32)
    import torch
    import paper_2606_19989_amd as odb

    from _parity import compare_collate_by_rank_whole_stream

    toks = synth.fill_tokens_torch(int(w.tok_off[-1]), "cuda")
    sp, ref = run_case("mm_stream", lens, perm, 8, w.budget, 1024, 1024, rate, full_collate=False, tokens=toks)
    outs = sp.collate()
    torch.cuda.synchronize()
    odb.odb_collate_status(sp.ws)
    compare_collate_by_rank_whole_stream(w.tok_off, outs, ref, toks)
    log("  every stream collate element equal")
    del sp, outs, toks
    torch.cuda.empty_cache()


@pytest.mark.parametrize("quota_div", [1, 3])
def test_stream_bimodal_nonjoin(quota_div):
    # the bimodal 16-rank window's 1.05M samples streamed in non-join mode with two worker
    # rates and a depth of 2048 (four sort keys per thread): quota N stops when the fast
    # ranks finish, quota N/3 at the quota; plan, trace, weights and every collate element
    # exact
    import torch
    import paper_2606_19989_amd as odb

    from _parity import compare_collate_by_rank_whole_stream, compare_collate_sampled

    w = synth.WORKLOADS["bimodal_w16x65536"].window()
    lens = np.diff(w.tok_off)
    perm = np.random.default_rng(79).permutation(len(lens)).astype(np.int32)
    toks = synth.fill_tokens_torch(int(w.tok_off[-1]), "cuda")
    sp, ref = run_case(f"bimodal_nonjoin_q{quota_div}", lens, perm, 16, 32768, 1024, 2048,
                       np.array([1024, 512] * 8, np.int32), mode="nonjoin", quota=len(lens) // quota_div,
                       full_collate=False, tokens=toks)
    assert ref.sinfo["stop_reason"] == (oracle.STOP_RANK_FINISHED if quota_div == 1 else oracle.STOP_QUOTA)
    outs = sp.collate()
    torch.cuda.synchronize()
    odb.odb_collate_status(sp.ws)
    compare_collate_sampled(w, outs, ref)
    compare_collate_by_rank_whole_stream(w.tok_off, outs, ref, toks)
    log("  every stream collate element equal")
    del sp, outs, toks
    torch.cuda.empty_cache()


def test_stream_full_size():
    # the largest window's 16.7M samples streamed by 64 ranks with the paper's buffer
    # of 1024 and a budget in its L_max range; the benchmark times this configuration.
    # Plan, trace, weights and every collate element (8.5 G per output) are compared
    # exactly
    import torch

    from _parity import collate_properties, compare_collate_by_rank_whole_stream, compare_collate_sampled

    w = synth.WORKLOADS["ln480_w64x262144"].window()
    lens = np.diff(w.tok_off)
    perm = np.random.default_rng(74).permutation(len(lens)).astype(np.int32)
    toks = synth.fill_tokens_torch(int(w.tok_off[-1]), "cuda")
    sp, ref = run_case("ln480_stream", lens, perm, 64, 16384, 1024, 1024, np.full(64, 1024, np.int32),
                       full_collate=False, tokens=toks)
    outs = sp.collate()
    torch.cuda.synchronize()
    import paper_2606_19989_amd as odb
    odb.odb_collate_status(sp.ws)
    compare_collate_sampled(w, outs, ref)
    collate_properties(outs, ref)
    log("  stream collate sampled and properties equal")
    compare_collate_by_rank_whole_stream(w.tok_off, outs, ref, toks)
    log("  every stream collate element equal")
    del sp, outs, toks
    torch.cuda.empty_cache()


def test_stream_two_stream_schedule():
    # the benchmark's streaming schedule: iteration i+1's odb_stream_plan on one stream
    # beside iteration i's collate on another, two plan buffers, one set of outputs
    import torch
    import paper_2606_19989_amd as odb
    import bench

    from _parity import collate_properties, compare_collate_sampled

    w = synth.WORKLOADS["text_w8x65536"].window()
    lens = np.diff(w.tok_off)
    N, W = len(lens), 8
    perm = np.random.default_rng(75).permutation(N).astype(np.int32)
    log(f"two-stream streaming schedule: N={N} W={W}")
    ref = oracle.stream(w.tok_off, perm, W, 16384, buffer_size=1024, depth=1024, rate=np.full(W, 1024))
    plan_stream, collate_stream = torch.cuda.Stream(), torch.cuda.Stream()
    toks = synth.fill_tokens_torch(int(w.tok_off[-1]), "cuda")
    win = odb.DeviceWindow(np.linspace(0, N, W + 1).astype(np.int64), torch.from_numpy(w.tok_off).cuda(), toks,
                           None, 0)
    d_perm = torch.from_numpy(perm).cuda()
    sps = [odb.StreamPipeline(win, d_perm, 16384, buffer_size=1024, depth=1024, rate=np.full(W, 1024, np.int32))
           for _ in range(2)]
    for sp in sps:
        sp.plan()
        sp.collate()
        sps[1].outputs = sps[0].outputs
    torch.cuda.synchronize()
    sps[0].outputs[0].fill_(-7)
    sec, coll, _ = bench.pipelined_steps(sps, plan_stream, collate_stream, 5, plan=bench.stream_plan,
                                         weights=bench.stream_weights)
    assert len(coll) == 5 and sec > 0
    S, E = ref.steps, ref.sinfo["emitted_views"]
    for sp in sps:
        odb.odb_collate_status(sp.ws)
        assert sp.info["steps"] == S
        assert np.array_equal(sp.slot_tile_off[:W * S + 1].cpu().numpy(), ref.slot_tile_off)
        assert np.array_equal(sp.emit_order[:E].cpu().numpy(), ref.emit_order)
        compare_row_records(w.tok_off, sp, ref.emit_order)
    outs = tuple(o[:ref.padded_elems] for o in sps[0].outputs)
    compare_collate_sampled(w, outs, ref)
    collate_properties(outs, ref)
    wt, st, ss = sps[0].loss_weights(oracle.WEIGHT_TOKEN_EXACT)
    ewt, est, ess = ref.loss_weights(oracle.WEIGHT_TOKEN_EXACT)
    assert np.array_equal(wt.cpu().numpy().view(np.int64), ewt.view(np.int64))


def test_stream_quota_cut_retry_at_the_reported_capacity():
    # room for one step per rank first: the call reports W * S and the retry at exactly
    # that capacity must succeed even though the round that reaches the quota stages more
    # steps than the cut keeps
    rng = np.random.default_rng(79)
    N, W = 6007, 5
    lens = np.clip(np.rint(synth.lognormal(rng, 300.0, 1.0, N)), 1, 4000).astype(np.int64)
    perm = rng.permutation(N).astype(np.int32)
    rate = rng.integers(8, 40, W).astype(np.int32)
    sp, ref = run_case("quota_cut_retry", lens, perm, W, 8192, 64, 96, rate, mode="nonjoin", quota=N // 3,
                       slot_capacity=W)
    assert sp.slot_capacity == W * ref.steps


@pytest.mark.parametrize("mode", ["join", "nonjoin"])
def test_stream_max_lengths(mode):
    # lengths over the whole valid range [1, 2^31 - 1] (31-bit sort keys: seven 5-bit
    # digit passes) at a budget of 2^40 (64-bit batch sizes); plan and weights only, the
    # token stream would not fit
    import torch

    rng = np.random.default_rng(78)
    top = (1 << 31) - 1
    lens = np.concatenate([rng.integers(1, top, 600), [top, 1, top], rng.integers(1, 50, 300)])
    perm = rng.permutation(len(lens)).astype(np.int32)
    run_case(f"max_lengths_{mode}", lens, perm, 3, 1 << 40, 64, 96, [64, 30, 64], mode=mode,
             quota=len(lens) // 2 if mode == "nonjoin" else 0, full_collate=False,
             tokens=torch.zeros(64, dtype=torch.int32, device="cuda"))


def test_stream_budget_int64_max():
    # a budget of 2^63 - 1: every group after a round's first takes the rest of the buffer
    rng = np.random.default_rng(80)
    lens = rng.integers(1, 3000, 2500)
    perm = rng.permutation(len(lens)).astype(np.int32)
    run_case("budget_int64_max", lens, perm, 3, (1 << 63) - 1, 128, 200, [128, 50, 128])


def together_cases():
    """Rounds formed together: buffer sizes at the edges of the block variants (256, 512, 1024
    and 4096 views), 64 rounds and more (dealt to the XCDs), tile offsets scanned ahead, a capacity that never binds, and
    the ways such a run ends: drained, in a round that overflows (the rest goes round by
    round), at a quota inside and at the end of a round, and at the first finished rank."""
    rng = np.random.default_rng(83)
    out = []
    for buf in (1, 255, 256, 257, 512, 513, 1024, 1025, 4096):
        out.append((f"buffer_{buf}", rng.integers(1, 5000, 3 * 2 * buf + 5), 2, 16384, buf, buf, [buf, buf], {}))
    out.append(("rounds_64", rng.integers(1, 700, 64 * 3 * 40), 3, 4000, 40, 40, [40] * 3, {}))
    out.append(("rounds_65_long", rng.integers(1, 2 ** 31 - 1, 65 * 40 - 3), 1, 2 ** 40, 40, 64, [64], {}))
    # more than 1,024 rounds, and rank-rounds, drained and cut in the last round
    many = rng.integers(1, 700, 2 * 2 * 1100 - 1)
    out.append(("rounds_1100", many, 2, 1400, 2, 2, [2] * 2, {}))
    out.append(("rounds_1100_quota", many, 2, 1400, 2, 2, [2] * 2, dict(mode="nonjoin", quota=4398)))
    out.append(("wide_digits", rng.integers(2 ** 16, 2 ** 24, 2000), 2, 2 ** 25, 300, 300, [300] * 2, {}))
    out.append(("free_capacity", rng.integers(1, 900, 3000), 3, 6000, 128, 128, [128] * 3,
                dict(cap=np.array([128, 0, 500]))))
    # uneven rates: the fast rank's last buffer is small, so a late round overflows
    out.append(("resume", rng.integers(1, 900, 3 * 1003), 3, 3000, 100, 300, [100, 129, 250], {}))
    out.append(("resume_skips", rng.integers(1, 900, 3 * 905), 3, 3000, 100, 300, [13, 17, 40], {}))
    for quota in (1950, 3000):
        out.append((f"resume_quota_{quota}", rng.integers(1, 900, 3 * 1003), 3, 3000, 100, 300, [100, 129, 250],
                    dict(mode="nonjoin", quota=quota)))
    for quota in (1, 600, 601, 1799, 1800, 3000):
        out.append((f"quota_{quota}", rng.integers(1, 2000, 3000), 3, 6000, 200, 200, [200] * 3,
                    dict(mode="nonjoin", quota=quota)))
    # identities carried by two views, both, one or none of them emitted
    for quota in (1700, 2900, 2998):
        out.append((f"shared_{quota}", rng.integers(1, 2000, 2998), 3, 6000, 200, 200, [200] * 3,
                    dict(mode="nonjoin", quota=quota)))
    # the stop round still fetches: one rank ready (its views count as fetched), one not
    out.append(("finished", rng.integers(900, 1000, 3 * 400), 3, 1000, 50, 200, [50, 100, 200],
                dict(mode="nonjoin", quota=10 ** 6)))
    # the most ranks formed together (64 KB of splits at the cut) and one more (round by round);
    # schedules of more ranks than one launch's arguments hold
    for ranks in (8192, 8193):
        out.append((f"ranks_{ranks}", np.full(4 * ranks, 100), ranks, 100, 2, 2, [2] * ranks,
                    dict(mode="nonjoin", quota=3 * ranks)))
    out.append(("uneven_130", rng.integers(1, 300, 130 * 40), 130, 900, 8, 32, [4 + r % 3 for r in range(130)], {}))
    return out


@pytest.mark.parametrize("idx", range(len(together_cases())))
def test_stream_rounds_together(idx):
    name, lens, W, budget, buf, depth, rate, kw = together_cases()[idx]
    perm = np.random.default_rng(100 + idx).permutation(len(lens)).astype(np.int32)
    small = int(lens.sum()) < 1 << 24
    run_case(name, lens, perm, W, budget, buf, depth, np.asarray(rate, dtype=np.int32), full_collate=small,
             tokens=None if small else _one_token(), **kw)


def cut_cases():
    """The quota cut of rounds formed together: ranks at the edges of the split search (a wave or a
    thread per rank, 32 and 33) and of the tries of the cut's search (512 for 8 ranks down to 8 for 512 and
    more), a few to over a thousand steps in the last round, quotas reached by its first step, its last and in
    between, even and uneven rates."""
    rng = np.random.default_rng(87)
    out = []
    for W, n, top in ((1, 1500, 900), (3, 2000, 9000), (8, 2000, 9000), (9, 700, 900), (32, 300, 900), (33, 300, 900), (64, 200, 9000),
                      (511, 60, 900), (513, 40, 9000), (1100, 24, 900)):
        lens = rng.integers(1, top, 2 * n * W)
        for rate in ([n], [n, n + n // 4]):
            first = sum(min(2 * n, rate[r % len(rate)]) for r in range(W))   # views of the first round
            for quota in (1, W + 1, first // 2, first - 1, first, first + 1, int(1.5 * first)):
                out.append((f"{W}x{n}_{len(rate)}_{quota}", lens, W, 4000, n, 2 * n, [rate[r % len(rate)] for r in range(W)],
                            quota))
    return out


@pytest.mark.parametrize("W", sorted({c[2] for c in cut_cases()}))
def test_stream_quota_cut_of_rounds_together(W):
    for name, lens, ranks, budget, buf, depth, rate, quota in cut_cases():
        if ranks != W:
            continue
        perm = np.random.default_rng(W).permutation(len(lens)).astype(np.int32)
        run_case(f"cut_{name}", lens, perm, W, budget, buf, depth, np.asarray(rate, dtype=np.int32), mode="nonjoin",
                 quota=quota, full_collate=False, tokens=_one_token())


@pytest.mark.parametrize("rounds", [1, 2, 3, 255, 256, 257, 511, 512, 513, 1025])
def test_stream_uneven_rounds_together(rounds):
    # rounds share the block's threads by powers of two, up to 512 rounds a pass; the fast ranks finish early
    W = 5
    lens = np.random.default_rng(88).integers(1, 40, W * rounds * 16)
    perm = np.random.default_rng(rounds).permutation(len(lens)).astype(np.int32)
    rate = np.asarray([16, 18, 17, 20, 16], dtype=np.int32)
    for mode, quota in (("join", 0), ("nonjoin", len(lens))):
        _, ref = run_case(f"uneven_{rounds}_{mode}", lens, perm, W, 200, 16, 20, rate, mode=mode, quota=quota,
                          full_collate=False, tokens=_one_token())
    assert mode == "join" or ref.sinfo["emit_rounds"] <= rounds


def early_overflow_cases():
    """Iterations formed together in which a round overflows early and hundreds of rounds, most of whose
    blocks then end at once, come after it: the first round, one a few rounds later (short samples at
    first, so that the fast rank forms few groups), 64 rounds and more or fewer, join and quota."""
    rng = np.random.default_rng(86)
    out = []
    for N, depth in ((3 * 14001, 300), (3 * 700, 300), (64 * 3000, 1024)):
        W = 64 if N > 10 ** 5 else 3
        rate = [depth] + [20] * (W - 1)
        for mode, quota in (("join", 0), ("nonjoin", N // 3)):
            out.append((f"first_{N}_{mode}", rng.integers(300, 900, N), W, 3000, rate, depth, dict(mode=mode, quota=quota)))
    lens = rng.integers(300, 900, 3 * 14001)
    lens[:3 * 1000] = rng.integers(1, 9, 3 * 1000)
    out.append(("later", lens, 3, 3000, [300, 20, 20], 300, dict(identity=True)))
    return out


@pytest.mark.parametrize("idx", range(len(early_overflow_cases())))
def test_stream_early_overflow(idx):
    name, lens, W, budget, rate, depth, kw = early_overflow_cases()[idx]
    perm = np.arange(len(lens), dtype=np.int32)
    if not kw.pop("identity", False):
        np.random.default_rng(87 + idx).shuffle(perm)
    _, ref = run_case(name, lens, perm, W, budget, 20, depth, np.asarray(rate, dtype=np.int32), tokens=_one_token(),
                      full_collate=False, **kw)
    assert ref.sinfo["overflow_groups"] > 0


@pytest.mark.parametrize("bad", ["perm", "length"])
def test_stream_early_overflow_meets_bad_data(bad):
    """Bad data in a late round of such an iteration is still met."""
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(88)
    N = 3 * 14001
    lens = rng.integers(300, 900, N)
    perm = rng.permutation(N).astype(np.int32)
    sp = _stream_pipeline(lens, perm, 3, 3000, 20, 300, [300, 20, 20])
    sp.plan()
    if bad == "perm":
        sp.perm[N - 7] = N
    else:
        sp.win.token_offsets[int(perm[N - 7]) + 1] = int(sp.win.token_offsets[int(perm[N - 7])])
    for _ in range(2):
        with pytest.raises(odb.OdbError) as e:
            sp.plan()
        assert e.value.status == odb.ODB_E_INVALID_DATA


def capacity_cases():
    """Iterations drained and cut at a quota, formed together, with a round that overflows after some of
    them, and round by round from the start."""
    rng = np.random.default_rng(84)
    L = rng.integers(1, 900, 3 * 1003)
    return [
        ("drained", L, 3, 3000, 100, 100, [100] * 3, {}),
        ("drained_many_ranks", rng.integers(1, 900, 130 * 70), 130, 3000, 16, 16, [16] * 130, {}),
        ("cut", L, 3, 3000, 100, 100, [100] * 3, dict(mode="nonjoin", quota=1234)),
        ("uneven_cut", L, 3, 3000, 100, 300, [100, 129, 250], dict(mode="nonjoin", quota=1234)),
        ("resume", L, 3, 3000, 100, 300, [100, 129, 250], {}),
        ("resume_cut", L, 3, 3000, 100, 300, [100, 129, 250], dict(mode="nonjoin", quota=3000)),
        ("rounds", L, 3, 3000, 100, 300, [100, 129, 250], dict(cap=np.array([9, 0, 8]))),
        # more steps in a round than the block has threads; more ranks, and a cut
        ("long_rounds", rng.integers(1, 9000, 3 * 4000), 3, 4000, 2000, 2000, [2000] * 3, {}),
        ("many_ranks_cut", rng.integers(1, 900, 600 * 40), 600, 3000, 16, 16, [16] * 600, dict(mode="nonjoin", quota=15000)),
    ]


@pytest.mark.parametrize("idx", range(len(capacity_cases())))
def test_stream_capacity_error_fills_the_summary(idx):
    """An iteration that needs more slots than there are reports the same summary, the largest step
    among it, whether its rounds were formed together or not."""
    import paper_2606_19989_amd as odb

    name, lens, W, budget, buf, depth, rate, kw = capacity_cases()[idx]
    perm = np.random.default_rng(85).permutation(len(lens)).astype(np.int32)
    rate = np.asarray(rate, dtype=np.int32)
    mode, quota, cap = kw.get("mode", "join"), kw.get("quota", 0), kw.get("cap")
    ref = oracle.stream(offsets(lens), perm, W, budget, quota=quota, buffer_size=buf, depth=depth, rate=rate, capacity=cap,
                        mode=oracle.MODE_NONJOIN if mode == "nonjoin" else oracle.MODE_JOIN)
    log(f"stream capacity summary {name}: steps {ref.steps}, overflow {ref.sinfo['overflow_groups']}")
    for steps in (1, ref.steps // 2, ref.steps - 1):
        sp = _stream_pipeline(lens, perm, W, budget, buf, depth, rate, mode=mode, quota=quota, capacity=cap,
                              slot_capacity=W * steps)
        st, info = sp._call(None)
        assert st == odb.ODB_E_CAPACITY and info["required_slot_capacity"] == W * ref.steps
        for f in ("steps", "rounds", "emit_rounds", "skip_rounds", "stop_reason", "views", "emitted_views", "splits",
                  "overflow_groups", "second_gather_rounds", "max_outstanding", "max_step_samples"):
            assert info[f] == ref.sinfo[f], (steps, f, info[f], ref.sinfo[f])


def _one_token():
    import torch
    return torch.zeros(1, dtype=torch.int32, device="cuda")
