"""GPU tests of the window path's data-error, capacity and status branches, called
through the C ABI: bad CSR lengths are reported with the first bad sample, a slot
capacity below W * S is reported with the capacity the plan needs (and Pipeline.align
then reallocates and matches the oracle), and the collate status word survives later
plan calls on the same workspace."""
import numpy as np
import pytest

import oracle
import synth
from _parity import compare_collate_full, compare_loss_weights, compare_plan, log, run_gpu

pytestmark = pytest.mark.gpu


def _window_with_offsets(tok_off, W):
    """A device window over explicit CSR offsets (possibly invalid); the token stream is a
    small array the grouping and alignment stages never read."""
    import torch
    import paper_2606_19989_amd as odb

    n = len(tok_off) - 1
    rank_off = np.linspace(0, n, W + 1).astype(np.int64)
    d_off = torch.from_numpy(np.ascontiguousarray(tok_off, dtype=np.int64)).cuda()
    toks = torch.zeros(64, dtype=torch.int32, device="cuda")
    return odb.DeviceWindow(rank_off, d_off, toks, None, 0)


def _bad_offsets(kind, rng):
    lens = rng.integers(1, 3000, 6000).astype(np.int64)
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    if kind == "zero_length":
        first = 777
        off[first + 1:] -= lens[first]           # sample 777 has length 0
        off[4001 + 1:] -= lens[4001]              # and a later one
    elif kind == "decreasing_offset":
        first = 1000
        off[first + 1] = off[first] - 5           # sample 1000 has length -5
    elif kind == "length_2p31":
        first = 2500
        off[first + 1:] += (1 << 31) - lens[first]    # sample 2500 has length exactly 2^31
    elif kind == "negative_offset":
        first = 0
        off[:] -= 3                               # sample 0 starts at token -3
    else:
        raise ValueError(kind)
    return off, first


@pytest.mark.parametrize("span", [1, 200, 20000, 1 << 30])
def test_long_ranks_reject_bad_lengths(span):
    """Ranks longer than one block groups: the form's first digit pass is under way when the host
    learns of the bad length; the call fails and the workspace then serves a valid window (equal
    lengths, one pass, two in a word, four with a position beside the key)."""
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(42)
    lens = rng.integers(1, span + 1, 50000).astype(np.int64)
    lens[:2] = 1, span
    off = np.concatenate([[0], np.cumsum(lens)])
    bad = off.copy()
    bad[30000] = bad[29999] - 7
    pipe = odb.Pipeline(_window_with_offsets(bad, 2), 1 << 20)
    for _ in range(2):
        with pytest.raises(odb.OdbError) as e:
            pipe.form()
        assert e.value.status == odb.ODB_E_INVALID_DATA, str(e.value)
        assert "sample 29999 " in str(e.value), str(e.value)
    pipe.win.token_offsets.copy_(torch.from_numpy(off))
    pipe.form()
    pipe.align()
    w = synth.window_from_ranks("after_bad", [lens[:25000], lens[25000:]], 1 << 20)
    compare_plan(w, pipe, oracle.plan_window(w))


@pytest.mark.parametrize("budget,longest,by_form", [
    (3682560, 5000, False), (3682561, 5000, True), (4194303, 5000, True), (4194304, 5000, True),
    (1 << 40, 3840, False), (1 << 40, 3841, True), (1 << 40, 4096, True), (1 << 40, 4097, True)])
def test_which_call_reports_a_bad_length(budget, longest, by_form):
    """Where the one-block grouping ends (batch sizes of 3,840 table entries, ranks of 3,840 samples):
    up to there odb_align_groups reports a bad length, beyond it odb_form_groups itself; the plans
    on both sides equal the oracle's."""
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(44)
    lens = rng.integers(1, 3000, longest + 100).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(lens)])
    bad = off.copy()
    bad[78:] -= lens[77]                          # sample 77 has length 0
    toks = torch.zeros(64, dtype=torch.int32, device="cuda")
    rank_off = np.array([0, longest, longest + 100])
    pipe = odb.Pipeline(odb.DeviceWindow(rank_off, torch.from_numpy(bad).cuda(), toks), budget)
    with pytest.raises(odb.OdbError) as e:
        pipe.form()
        assert not by_form, "odb_form_groups took the bad length"
        pipe.align()
    assert e.value.status == odb.ODB_E_INVALID_DATA and "sample 77 " in str(e.value), str(e.value)
    if not by_form:
        pipe.form()
    pipe.win.token_offsets.copy_(torch.from_numpy(off))
    pipe.form()
    pipe.align()
    w = synth.window_from_ranks("after_bad", [lens[:longest], lens[longest:]], budget)
    compare_plan(w, pipe, oracle.plan_window(w))


@pytest.mark.parametrize("kind", ["zero_length", "decreasing_offset", "length_2p31", "negative_offset"])
def test_window_rejects_bad_lengths(kind):
    # l < 1, l >= 2^31 and negative token offsets are invalid data (a length the batch
    # size rule of Eq. 1 cannot take); the first such sample is named, and the same
    # workspace then serves a valid window
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(41)
    off, first = _bad_offsets(kind, rng)
    log(f"bad lengths: {kind}, first bad sample {first}")
    dwin = _window_with_offsets(off, 3)
    pipe = odb.Pipeline(dwin, 16384)
    with pytest.raises(odb.OdbError) as e:
        pipe.form()
        pipe.align()
    assert e.value.status == odb.ODB_E_INVALID_DATA, str(e.value)
    assert f"sample {first} " in str(e.value), str(e.value)
    torch.cuda.synchronize()
    # the workspace recovers: a valid window of the same shape on it
    lens = rng.integers(1, 3000, 6000)
    w = synth.window_from_ranks("after_error", [lens[:2000], lens[2000:4000], lens[4000:]], 16384)
    tok_off, toks, _ = synth.device_tensors(w, "cuda")
    good = odb.DeviceWindow(w.rank_off, tok_off, toks, None, 0)
    pipe2 = odb.Pipeline(good, w.budget)
    pipe2.ws = pipe.ws
    pipe2.form()
    pipe2.align()
    compare_plan(w, pipe2, oracle.plan_window(w))


@pytest.mark.parametrize("mode", ["join", "nonjoin"])
def test_align_reports_capacity_and_pipeline_retries(mode):
    # slot arrays below W * S: ODB_E_CAPACITY with the capacity the plan needs; the
    # Pipeline then reallocates and its plan and outputs equal the oracle's
    import torch
    import paper_2606_19989_amd as odb

    rng = np.random.default_rng(43)
    per = [rng.integers(1, 3000, 4000), rng.integers(1, 3000, 900), rng.integers(1, 3000, 2500)]
    n = sum(len(x) for x in per)
    w = synth.window_from_ranks(f"capacity_{mode}", per, 12000, mode=mode, quota=n // 2 if mode == "nonjoin" else 0)
    ref = oracle.plan_window(w)
    need = w.W * ref.steps
    log(f"capacity: {mode}, plan needs {need} slots")
    tok_off, toks, _ = synth.device_tensors(w, "cuda")
    dwin = odb.DeviceWindow(w.rank_off, tok_off, toks, None, 0)
    for cap in (1, need - 1):
        pipe = odb.Pipeline(dwin, w.budget, mode=w.mode, quota=w.quota, slot_capacity=cap)
        pipe.form()
        st, info = odb.odb_align_groups(dwin, w.budget, pipe.mode, pipe.quota, None, pipe.order, pipe.sorted_len,
                                        pipe.group_index, pipe.groups_per_rank, pipe.slot_capacity, pipe.emit_order,
                                        pipe.slot_rows, pipe.slot_maxlen, pipe.slot_row_off, pipe.slot_tile_off,
                                        pipe.slot_tokens, pipe.leftover, pipe.leftover_off, pipe.ws,
                                        raise_on_capacity=False, slot_tokens_approx=pipe.slot_tokens_approx,
                                        row_token_start=pipe.row_token_start, row_len=pipe.row_len)
        assert st == odb.ODB_E_CAPACITY
        assert info["required_slot_capacity"] == need and info["steps"] == ref.steps
        with pytest.raises(odb.OdbError) as e:
            odb.odb_align_groups(dwin, w.budget, pipe.mode, pipe.quota, None, pipe.order, pipe.sorted_len,
                                 pipe.group_index, pipe.groups_per_rank, pipe.slot_capacity, pipe.emit_order,
                                 pipe.slot_rows, pipe.slot_maxlen, pipe.slot_row_off, pipe.slot_tile_off,
                                 pipe.slot_tokens, pipe.leftover, pipe.leftover_off, pipe.ws)
        assert e.value.status == odb.ODB_E_CAPACITY and str(need) in str(e.value)
        # Pipeline.align reallocates the slot arrays to the reported size and retries
        pipe.align()
        assert pipe.slot_capacity == need
        outs = pipe.collate()
        torch.cuda.synchronize()
        odb.odb_collate_status(pipe.ws)
        compare_plan(w, pipe, ref)
        compare_collate_full(w, outs, ref)
        compare_loss_weights(pipe, ref)


def capacity_windows():
    """One window per path of the alignment: one round (ranks on both sides of 16 tiles, join and with
    quotas inside and past the window), rounds of short ranks, and round by round."""
    rng = np.random.default_rng(45)
    U = lambda n: rng.integers(1, 3000, size=n)
    win = synth.window_from_ranks
    return [
        win("one_round", [U(900), U(1025), U(700)], 12000),
        win("one_round_long", [U(20000), U(30), U(18000)], 1 << 22),
        win("one_round_quota", [U(900), U(1025), U(700)], 12000, mode="nonjoin", quota=1111),
        win("one_round_quota_all", [U(900), U(1025), U(700)], 12000, mode="nonjoin", quota=1 << 40),
        win("short_rounds", [U(900), U(1025), U(700)], 12000, capacity=np.array([40, 0, 33])),
        win("rounds", [U(17000), U(1025), U(700)], 12000, capacity=np.array([400, 0, 330])),
        win("rounds_quota", [U(900), U(1025), U(7)], 12000, mode="nonjoin", quota=100),
        # the steps summed over slices of 64 ranks
        win("slices", [U(90) for _ in range(65)], 12000),
        win("slices_quota", [U(60 + r % 7) for r in range(700)], 12000, mode="nonjoin", quota=20000),
    ]


@pytest.mark.parametrize("idx", range(len(capacity_windows())))
def test_capacity_error_fills_the_summary(idx):
    """A plan that needs more slots than there are still reports what it is: steps, rounds, stop reason,
    splits, overflow and the largest step, whichever way it was aligned."""
    import torch
    import paper_2606_19989_amd as odb

    w = capacity_windows()[idx]
    ref = oracle.plan_window(w)
    log(f"capacity summary: {w.name}, rounds {ref.info['rounds']}")
    toks = torch.zeros(1, dtype=torch.int32, device="cuda")
    dwin = odb.DeviceWindow(w.rank_off, torch.from_numpy(w.tok_off).cuda(), toks)
    for cap in (1, w.W * ref.steps - 1):
        pipe = odb.Pipeline(dwin, w.budget, mode=w.mode, quota=w.quota, capacity=w.capacity, slot_capacity=cap)
        pipe.form()
        st, info = odb.odb_align_groups(dwin, w.budget, pipe.mode, pipe.quota, w.capacity, pipe.order, pipe.sorted_len,
                                        pipe.group_index, pipe.groups_per_rank, cap, pipe.emit_order, pipe.slot_rows,
                                        pipe.slot_maxlen, pipe.slot_row_off, pipe.slot_tile_off, pipe.slot_tokens,
                                        pipe.leftover, pipe.leftover_off, pipe.ws, raise_on_capacity=False)
        assert st == odb.ODB_E_CAPACITY
        assert info["required_slot_capacity"] == w.W * ref.steps
        for f in ("steps", "rounds", "stop_reason", "splits", "overflow_groups", "second_gather_rounds",
                  "max_step_samples"):
            assert info[f] == ref.info[f], (f, info[f], ref.info[f])


def test_collate_status_survives_plan_calls():
    # a collate error stays readable after grouping and alignment calls on the same
    # workspace; reading it clears it; a fresh workspace full of ones reports no error
    import torch
    import paper_2606_19989_amd as odb

    w = synth.WORKLOADS["ln512_w2x2048"].window()
    tok_off, toks, ident = synth.device_tensors(w, "cuda")
    dwin = odb.DeviceWindow(w.rank_off, tok_off, toks, ident, w.num_identities)
    pipe = odb.Pipeline(dwin, w.budget)
    pipe.ws.fill_(255)
    pipe.run()
    torch.cuda.synchronize()
    odb.odb_collate_status(pipe.ws)
    ref = oracle.plan_window(w)
    good = int(pipe.row_token_start[5])
    pipe.row_token_start[5] = int(w.tok_off[-1])   # a row record past the end of the stream
    pipe.collate()
    pipe.row_token_start[5] = good
    pipe.form()
    pipe.align()
    torch.cuda.synchronize()
    with pytest.raises(odb.OdbError) as e:
        odb.odb_collate_status(pipe.ws)
    assert e.value.status == odb.ODB_E_INVALID_DATA
    odb.odb_collate_status(pipe.ws)          # cleared by the read
    outs = pipe.collate()
    torch.cuda.synchronize()
    odb.odb_collate_status(pipe.ws)
    compare_plan(w, pipe, ref)
    compare_collate_full(w, outs, ref)


def test_pointer_jumping_full_size():
    # group discovery by pointer jumping over the next-group-start links on the largest
    # window (64 ranks x 262,144 samples, lengths 8..16384): a budget of 2^26 gives more
    # distinct batch sizes per rank than the run walk's table holds, so every rank's chain
    # is found by doubling rounds.  Every plan array and the loss weights are compared
    # exactly (groups of up to 2^26 padded elements: the collate is not run here)
    import torch

    w = synth.WORKLOADS["ln480_w64x262144"].window()
    w.budget = 1 << 26
    lens = np.diff(w.tok_off)
    rng_len = int(lens.max() - lens.min() + 1)
    runs_bound = min(2 * (int(np.sqrt(w.budget)) + 1) + 1, rng_len)
    assert runs_bound > 4096, runs_bound
    log(f"pointer jumping: n={w.n} budget={w.budget} distinct-step bound {runs_bound}")
    ref = oracle.plan_window(w)
    log(f"  oracle plan done: steps={ref.steps} groups={int(ref.groups_per_rank.sum())}")
    pipe, _ = run_gpu(w, collate=False)
    compare_plan(w, pipe, ref)
    compare_loss_weights(pipe, ref)
    log("  plan and loss weights equal")
    del pipe
    torch.cuda.empty_cache()
