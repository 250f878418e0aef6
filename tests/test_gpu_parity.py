"""GPU parity: every C-ABI entry point against the CPU oracle on seeded synthetic inputs.

Sizes span several key chunks and MFMA tiles with ragged tails; the full-size workloads run in the
benchmark's launch configuration (all layers in one batch) and are checked on sampled problems.
"""
import numpy as np
import pytest

from paper_2609_30738_amd import _lib, workloads
from tests import gpu_cases

pytestmark = pytest.mark.gpu


def _all(run, heads=None, certified=False):
    """Compare every problem of a run with the oracle; certified=True: every head's inputs are
    margin-certified, so every head must reproduce the oracle exactly."""
    reports = gpu_cases.check_all(run, heads=heads)
    print("  ", gpu_cases.summarize(reports), flush=True)
    if certified:
        assert all(r.certified for r in reports), gpu_cases.summarize(reports)
        assert all(r.identical_steps == r.steps for r in reports)
    return reports


def _all_of(run, js):
    """Compare problems js of a run (None: all)."""
    print("  ", gpu_cases.summarize(gpu_cases.check_all(run, js=js)), flush=True)


def test_tiny_f32_unfused_with_attention():
    """fp32 path, 2 query heads on 1 kv head, d=64, W=8 (general window reduction); certified."""
    _all(gpu_cases.run_case("tiny_f32", want_attn=True), certified=True)


def test_tiny_f32_fused_exact_greedy_over_all_candidates():
    """cand_mult = 0: the greedy runs over every prefix position; certified."""
    _all(gpu_cases.run_case("tiny_f32_all_candidates", fused=True), certified=True)


@pytest.mark.parametrize("case", ["tiny_f32_no_tail", "tiny_f32_tail3"])
def test_tiny_f32_keep_tail(case):
    _all(gpu_cases.run_case(case), certified=True)


def test_mistral_layer_unfused():
    """One Mistral-7B layer, bf16, L=4096, W=32, B=64, lambda1=0.3, lambda2=-0.8; certified inputs,
    so every admission is the oracle's."""
    _all(gpu_cases.run_case("mistral_layer"), certified=True)


def test_mistral_layer_timed_calls():
    """The benchmark's calls (kv_window_mu_sigma, kv_mmr_select_compact) on certified inputs."""
    _all(gpu_cases.run_case("mistral_layer", timed=True), certified=True)


def test_exact_duplicate_keys_ties_to_lower_position():
    """Clusters of bitwise identical keys: exact ties at the candidate cut and in the greedy argmax
    are decided by the lower position on both sides (R10), through the default and the benchmark
    calls."""
    for timed in (False, True):
        _all(gpu_cases.run_case("exact_duplicates", fused=True, timed=timed), certified=True)


def test_nonfinite_inputs_keep_indices_valid():
    """NaN and Inf planted in keys and in window queries (results unspecified, R21): every call
    succeeds, and every selection is B distinct candidate positions."""
    wl = workloads.mistral_layer()
    wl.seq_lens = [3000]
    wl.n_seq = 1
    pk = workloads.draw_packed(wl)
    L, d, G = 3000, wl.d, wl.h_q // wl.h_kv
    k = pk.k.reshape(wl.h_kv, L, d)
    nan, inf, ninf = np.uint16(0x7FC0), np.uint16(0x7F80), np.uint16(0xFF80)
    k[0, 100] = nan                 # a NaN key row
    k[1, 200, :5] = inf             # a key with infinite entries
    k[2, 300:310] = ninf            # ten keys of -inf entries
    k[3, :, 7] = nan                # a NaN component in every key of a head
    pk.q_win[0, 5 * G, 3] = nan     # a NaN window query of kv head 5's group
    pk.q_win[0, 6 * G + 1, :] = inf  # an infinite window query of kv head 6's group
    for fused in (True, False):
        run = gpu_cases.run_gpu(wl, fused=fused, packed=pk)
        for timed in (False, True):
            if timed:
                run = gpu_cases.run_gpu(wl, packed=pk, timed=True)
            B = run.budget
            sel = run.host["sel_idx"].reshape(wl.h_kv, B)
            for g in range(wl.h_kv):
                s = sel[g]
                assert len(set(s.tolist())) == B, f"g={g}: repeated positions {s}"
                assert np.all((s >= 0) & (s < L - wl.w)), f"g={g}: out of range {s}"


def test_mistral_layer_fused_with_attention_short_context():
    """Ragged context (L=1337: partial chunk and partial tile) with the attention output."""
    wl = workloads.mistral_layer()
    wl.seq_lens = [1337]
    _all(gpu_cases.run_gpu(wl, want_attn=True))


@pytest.mark.parametrize("budget", [32, 64, 128])
def test_segments_profile_budget_sweep_scaled(budget):
    """Three-segment lambda2 over 3 layers (one per segment), L=2048, B in {32, 64, 128}."""
    _all(gpu_cases.run_case(f"segments_scaled_B{budget}", fused=True))


def test_curve_profile_scaled():
    """Quadratic lambda2 profile with passages repeated twice, 4 layers of L=6000; certified."""
    _all(gpu_cases.run_case("curve_scaled", fused=True), certified=True)


@pytest.mark.parametrize("run", ["dispersion_only", "redundancy_only", "both"])
def test_ragged_batch_scaled(run):
    """Three sequences of different lengths x 2 layers, B=128, the three term-ablation runs."""
    _all(gpu_cases.run_case(f"ragged_scaled_{run}", fused=True))


def _plant_rising_keys(wl, pk, plants):
    """Per kv group, keys along head 0's mean query direction (orthogonal to the other heads'
    mean directions) with window logits of about alpha nats at the given positions of problem 0."""
    from oracle import evict
    q = evict.decode(pk.q_win[0], wl.dtype).astype(np.float64)  # [h_q, w, d]
    L = int(pk.lens[0])
    G = wl.h_q // wl.h_kv
    k = pk.k[: wl.h_kv * L * wl.d].reshape(wl.h_kv, L, wl.d)
    for g in range(wl.h_kv):
        dirs = [q[g * G + h].mean(axis=0) for h in range(G)]
        u = dirs[0].copy()
        basis = []
        for v in dirs[1:]:
            for b_ in basis:
                v = v - (v @ b_) * b_
            basis.append(v / np.linalg.norm(v))
        for b_ in basis:
            u = u - (u @ b_) * b_
        u /= np.linalg.norm(u)
        nu = float((q[g * G] @ u).mean())
        for pos, alpha in plants:
            k[g, pos] = workloads.f32_to_bf16_bits((alpha / (wl.scale * nu) * u).astype(np.float32))


@pytest.mark.parametrize("fused", [True, False])
def test_rising_logits_move_the_running_offset(fused):
    """Keys whose logits rise far above the earlier ones, in later tiles and segments of the unit:
    about 9 nats (kept against the running offset), 40 nats (a rebase) and 100 nats (2^x of the
    difference overflows; a rebase).  Row statistics, mu and sigma must still match."""
    wl = workloads.mistral_layer()
    wl.seq_lens = [5000]
    pk = workloads.draw_packed(wl)
    _plant_rising_keys(wl, pk, [(777, 9.0), (2222, 40.0), (4444, 100.0)])
    _all(gpu_cases.run_gpu(wl, fused=fused, packed=pk))


@pytest.mark.parametrize("pool", [3, 7, 31])
def test_max_pooled_scores(pool):
    """kv_mmr_select_ex with a max-pool over positions (the window stops at the end of the
    candidate range): two ragged sequences x 2 layers, B=64."""
    wl = workloads.ragged_batch("both", n_seq=2, n_layers=2, len_range=(700, 3100))
    wl.budget = 64
    _all(gpu_cases.run_gpu(wl, fused=True, pool=pool))


def test_max_pooled_scores_across_pooling_chunks():
    """bf16 keys, L = 20000: the in-place pooling of the staged keys runs in three chunks of
    8192 positions, so windows straddle chunk ends (pool 31)."""
    wl = workloads.mistral_layer()
    wl.seq_lens = [20000]
    _all(gpu_cases.run_gpu(wl, fused=True, pool=31), heads=[0, 3, 7])


def test_max_pooled_scores_fp32_chunks():
    """fp32 keys (256 threads, chunks of 2048 positions), L = 5000, pool 9."""
    wl = workloads.tiny_f32()
    wl.seq_lens = [5000]
    _all(gpu_cases.run_gpu(wl, fused=True, pool=9))


def test_max_pooled_scores_fp32_keep_all():
    """fp32 keys (256-thread select), every position a candidate (keep_tail = 0) and pool 5."""
    _all(gpu_cases.run_gpu(workloads.tiny_f32(), fused=True, keep_tail=0, pool=5))


@pytest.mark.parametrize("case", ["mean_free_dispersion_only", "mean_free"])
def test_mean_free_score(case):
    """w_mu = 0: the score without the mean term (dispersion and redundancy only)."""
    _all(gpu_cases.run_case(case, fused=True))


def test_mean_free_max_pooled_unfused():
    """w_mu = 0.5 and pool 9 together, through the two-call scoring path."""
    wl = workloads.mistral_layer()
    wl.seq_lens = [3000]
    _all(gpu_cases.run_gpu(wl, fused=False, w_mu=0.5, pool=9))


@pytest.mark.parametrize("fused", [True, False])
def test_dispersion_over_all_group_rows(fused):
    """KV_SIGMA_ALL_ROWS, 4 query heads per kv head: streaming pass 2 (fused) and the generic
    w = 32 kernel with the attention output (unfused), L = 3000."""
    _all(gpu_cases.run_case("sigma_all_rows", fused=fused, want_attn=not fused), certified=True)


@pytest.mark.parametrize("sigma_rows", ["group_mean", "all_rows"])
def test_three_query_heads_per_kv_head(sigma_rows):
    """G = 3 (w = 32): 96 window rows in four 32-row blocks, the last one padding; generic
    kernels, both dispersion readings, L = 2100."""
    _all(gpu_cases.run_case(f"g3_{sigma_rows}", fused=True), certified=True)


def test_dispersion_over_all_group_rows_general_window():
    """KV_SIGMA_ALL_ROWS through the LDS reduction of other window sizes (fp32, G = 2, w = 8)."""
    _all(gpu_cases.run_gpu(workloads.tiny_f32(), fused=True, sigma_rows="all_rows"))


def test_depth_decreasing_budgets():
    """Per-problem budgets from the depth schedule (B = 64 over 4 layers, beta = 20: 125, 85, 43,
    3), two sequences x 4 layers of L = 3000 and 2200: ragged greedy lengths, candidate counts and
    compacted blocks, padded steps."""
    from oracle import budgets
    from tests import certified_cases
    sched = budgets.pyramid_budgets(64, 4, 20.0)
    assert sched == [125, 85, 43, 3]
    assert certified_cases.options("depth_budgets").budgets == tuple(sched * 2)
    _all(gpu_cases.run_case("depth_budgets", fused=True))


def test_depth_decreasing_budgets_fp32_with_options():
    """fp32 keys (256-thread select), budgets 40 and 16 in one batch, with pool 3 and w_mu 0.5."""
    wl = workloads.tiny_f32()
    wl.n_seq, wl.seq_lens = 2, [512, 700]
    _all(gpu_cases.run_gpu(wl, fused=True, budgets=[40, 16], pool=3, w_mu=0.5))


def test_compaction_of_oracle_selection():
    """kv_compact_cache fed with the oracle's admissions reproduces the oracle's compacted rows."""
    import torch
    from oracle import evict
    from paper_2609_30738_amd import _lib, api
    wl = workloads.mistral_layer()
    wl.seq_lens = [900]
    print(f"[gpu case] compaction {wl.name} L=900", flush=True)
    pk = workloads.draw_packed(wl)
    q, k, v = pk.q_win[0], pk.k.reshape(wl.h_kv, 900, wl.d), pk.v.reshape(wl.h_kv, 900, wl.d)
    res = evict.evict_problem(q, k, v, wl.dtype, wl.scale, 0.3, -0.8, wl.budget)
    sel = np.array([res.heads[g].trace.selected for g in range(wl.h_kv)], dtype=np.int32)
    inp = api.upload(wl.dtype, wl.h_q, wl.h_kv, wl.d, wl.w, pk.q_win, pk.k, pk.v, pk.lens,
                     pk.tok_off, [0.3], [-0.8])
    rows = wl.budget + wl.w
    k_out = torch.empty(wl.h_kv * rows * wl.d, dtype=inp.k.dtype, device=inp.k.device)
    v_out = torch.empty_like(k_out)
    _lib.compact_cache(inp.batch, inp.k, inp.v, api.to_device(sel.reshape(-1)), wl.budget, wl.w,
                       k_out, v_out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(api.to_host_bits(k_out).reshape(res.k_out.shape), res.k_out)
    np.testing.assert_array_equal(api.to_host_bits(v_out).reshape(res.v_out.shape), res.v_out)


def test_deterministic_repeat():
    """Two runs on the same inputs give bitwise-identical outputs (no races in the reductions)."""
    wl = workloads.mistral_pass_32k(n_layers=2, L=5000, n_clusters=16, n_passages=4)
    a = gpu_cases.run_gpu(wl, fused=True)
    b = gpu_cases.run_gpu(wl, fused=True, packed=a.packed)
    for name in ("row_max", "row_sum", "mu", "sigma", "sel_idx", "sel_score", "cand_idx",
                 "cand_corr", "k_out", "v_out"):
        np.testing.assert_array_equal(a.host[name], b.host[name], err_msg=name)


@pytest.mark.parametrize("fused", [True, False])
def test_short_contexts_near_the_window(fused):
    """Contexts of 33, 64, 65, 95 and 287 keys in one bf16 batch with per-problem budgets: one
    candidate, partial tiles, the causal triangle of the window across two tiles, tiles with no
    unmasked key for some rows."""
    wl = workloads.Workload(
        "short_contexts_W32", 1, workloads.BF16, 32, 8, 128, 32, 64, 5, 1, [33, 64, 65, 95, 287],
        workloads.Layout(cluster_density=0.02),
        workloads.ProfileSpec(workloads.PROFILE_GLOBAL, (float(np.arcsinh(0.3)),)),
        workloads.ProfileSpec(workloads.PROFILE_GLOBAL, (float(np.arcsinh(-0.8)),)))
    _all(gpu_cases.run_gpu(wl, fused=fused, budgets=[1, 8, 8, 16, 64]))


def _one_segment_per_unit(wl) -> bool:
    """Whether the streaming plan gives every unit a single segment (both passes of a unit then
    run in one workgroup): about one segment per compute unit, 1024 keys at least, in whole
    256-key steps, never longer than the longest context."""
    total = int(wl.lens.astype(np.int64).sum()) * wl.h_kv
    seg = max(1024, -(-(-(-total // 256)) // 256) * 256)
    seg = min(seg, -(-int(wl.lens.max()) // 256) * 256)
    return seg >= int(wl.lens.max())


@pytest.mark.parametrize("sigma_rows", ["group_mean", "all_rows"])
def test_both_passes_in_one_workgroup_ragged(sigma_rows):
    """256 units of 1024, 1000, 700 and 513 keys (8 layers of 4 sequences): each unit is one
    segment, so the fused entry point runs pass 1, the normalisers and pass 2 of a unit in one
    workgroup; ragged tails, whole tiles and the window's causal triangle."""
    wl = workloads.Workload(
        "one_segment_units_W32", 1, workloads.BF16, 32, 8, 128, 32, 32, 4, 8, [1024, 1000, 700, 513],
        workloads.Layout(cluster_density=0.02),
        workloads.ProfileSpec(workloads.PROFILE_GLOBAL, (float(np.arcsinh(0.3)),)),
        workloads.ProfileSpec(workloads.PROFILE_GLOBAL, (float(np.arcsinh(-0.8)),)))
    assert wl.n_prob * wl.h_kv == 256 and _one_segment_per_unit(wl)
    _all(gpu_cases.run_gpu(wl, fused=True, sigma_rows=sigma_rows))


@pytest.mark.parametrize("sigma_rows", ["group_mean", "all_rows"])
def test_segments_computed_by_a_waiting_workgroup(sigma_rows, monkeypatch):
    """Units of 4096 keys in 4 segments (one Mistral-shaped layer): both passes run in one launch,
    and a workgroup that stops waiting for its unit's other segments computes their partials
    itself.  A poll limit of 0, set from the host, sends every workgroup down that path: the
    results match the oracle and are bit-identical to those of the default path."""
    wl = workloads.mistral_layer()
    monkeypatch.delenv("KVEVICT_SPIN_LIMIT", raising=False)
    ref = gpu_cases.run_gpu(wl, fused=True, sigma_rows=sigma_rows)
    monkeypatch.setenv("KVEVICT_SPIN_LIMIT", "0")
    run = gpu_cases.run_gpu(wl, fused=True, sigma_rows=sigma_rows)
    for name in ("row_max", "row_sum", "mu", "sigma", "sel_idx", "k_out", "v_out"):
        assert np.array_equal(run.host[name], ref.host[name]), name
    _all(run)


def _shape_workload(h_q, h_kv, d, n_seq, n_layers, lens, budget=16):
    return workloads.Workload(
        f"bf16_hq{h_q}_hkv{h_kv}_d{d}_W32", 1, workloads.BF16, h_q, h_kv, d, 32, budget, n_seq,
        n_layers, list(lens), workloads.Layout(cluster_density=0.02),
        workloads.ProfileSpec(workloads.PROFILE_GLOBAL, (float(np.arcsinh(0.3)),)),
        workloads.ProfileSpec(workloads.PROFILE_GLOBAL, (float(np.arcsinh(-0.8)),)))


STREAM_SHAPES = [(8, 8, 64), (16, 8, 128), (8, 2, 64), (16, 8, 64), (8, 8, 128)]


@pytest.mark.parametrize("h_q,h_kv,d", STREAM_SHAPES)
@pytest.mark.parametrize("fused", [True, False])
def test_stream_shapes_several_segments(h_q, h_kv, d, fused):
    """bf16, W = 32, every head layout and head size the streaming kernels take (G = 1, 2, 4;
    d = 64, 128), units of 3000 and 2100 keys in several segments: both passes in one launch
    (fused) or as the two entry points."""
    wl = _shape_workload(h_q, h_kv, d, 2, 2, [3000, 2100])
    _all(gpu_cases.run_gpu(wl, fused=fused))


@pytest.mark.parametrize("h_q,h_kv,d", STREAM_SHAPES)
def test_stream_shapes_one_segment_per_unit(h_q, h_kv, d):
    """The same layouts with 256 units of at most 1024 keys: each unit is one segment, so both
    passes of a unit run in one workgroup."""
    n_prob = 256 // h_kv
    wl = _shape_workload(h_q, h_kv, d, 2, n_prob // 2, [1024, 777])
    assert _one_segment_per_unit(wl)
    _all(gpu_cases.run_gpu(wl, fused=True))


@pytest.mark.parametrize("h_q,h_kv,d,w", [(8, 2, 128, 8), (14, 2, 64, 8), (2, 2, 128, 8),
                                          (4, 2, 64, 16), (6, 2, 128, 16), (8, 2, 64, 16)])
@pytest.mark.parametrize("lens,n_layers", [([1000, 531, 41], 1), ([5003, 300], 2), ([3001], 80)])
def test_short_windows(h_q, h_kv, d, w, lens, n_layers, monkeypatch):
    """bf16 windows of 8 and 16 rows, whole and padded 32-row blocks (G w = 8 .. 56), both
    dispersion readings: units of one segment and of several (ragged, partial tiles), the
    workgroup that computes late segments itself, and 160 units over the chip's CUs."""
    import dataclasses
    wl = dataclasses.replace(_shape_workload(h_q, h_kv, d, len(lens), n_layers, lens), w=w,
                             name=f"bf16_hq{h_q}_d{d}_W{w}_L{lens}")
    probs = [0] if n_layers > 2 else None
    for sigma_rows in ("group_mean", "all_rows"):
        monkeypatch.delenv("KVEVICT_SPIN_LIMIT", raising=False)
        run = gpu_cases.run_gpu(wl, timed=True, sigma_rows=sigma_rows)
        _all_of(run, probs)
        if n_layers > 2:
            continue
        monkeypatch.setenv("KVEVICT_SPIN_LIMIT", "0")
        late = gpu_cases.run_gpu(wl, timed=True, sigma_rows=sigma_rows)
        for name in ("row_max", "row_sum", "score", "sel_idx", "k_out", "v_out"):
            assert np.array_equal(run.host[name], late.host[name]), name


def test_segments_merged_by_the_second_launch():
    """192 units of 5000 keys in two segments each: 384 workgroups do not fit the chip at once, so
    the fused entry point takes two launches, the second merging the first's segment partials
    from the workspace."""
    wl = _shape_workload(32, 8, 128, 3, 8, [5000, 5000, 5000], budget=32)
    total = int(wl.lens.sum()) * wl.h_kv
    seg = min(max(1024, -(-(-(-total // 256)) // 256) * 256), -(-int(wl.lens.max()) // 256) * 256)
    n_seg = -(-int(wl.lens.max()) // seg)
    assert n_seg == 2 and n_seg * wl.n_prob * wl.h_kv > 256
    _all(gpu_cases.run_gpu(wl, fused=True))


@pytest.mark.parametrize("n_seq,n_layers,lens,h_q,d,exact", [
    (1, 24, [5000], 32, 128, True), (1, 24, [1500], 16, 64, True), (1, 14, [9000], 32, 128, True), (1, 10, [9000], 32, 128, True),
    (1, 10, [9000], 8, 64, True), (2, 16, [2500, 700], 32, 128, True),
    (38, 1, [300] * 37 + [6000], 8, 128, False)])
def test_workgroups_of_several_segments(n_seq, n_layers, lens, h_q, d, exact):
    """Batches whose segments do not fit the chip at once: 192 units of two segments and
    112 of three in one workgroup each (also with no tile of the last for some waves), 80 units of four segments in
    two workgroups, ragged units of one and two, and 304 units of up to six, which take two
    launches.  The statistics are merged segment by segment whatever the workgroups, so the row
    statistics equal those of kv_window_scores (one workgroup per segment, merged by its combine
    kernel in segment order, which for up to four segments is the same order) bit for bit."""
    wl = _shape_workload(h_q, 8, d, n_seq, n_layers, lens, budget=32)
    run = gpu_cases.run_gpu(wl, timed=True)
    _all_of(run, [0, wl.n_prob - 1])
    if exact:
        plain = gpu_cases.run_gpu(wl, fused=False)
        for name in ("row_max", "row_sum"):
            assert np.array_equal(run.host[name].view(np.uint32), plain.host[name].view(np.uint32)), name


@pytest.mark.parametrize("h_q,h_kv,d", STREAM_SHAPES)
def test_stream_shapes_late_segments_computed_by_the_waiting_workgroup(h_q, h_kv, d, monkeypatch):
    """Every head layout and head size with a poll limit of 0: each workgroup computes the other
    segments' partials itself; the results are bit-identical to the default path's."""
    wl = _shape_workload(h_q, h_kv, d, 2, 2, [3000, 2100])
    monkeypatch.delenv("KVEVICT_SPIN_LIMIT", raising=False)
    ref = gpu_cases.run_gpu(wl, fused=True)
    monkeypatch.setenv("KVEVICT_SPIN_LIMIT", "0")
    run = gpu_cases.run_gpu(wl, fused=True)
    for name in ("row_max", "row_sum", "mu", "sigma", "sel_idx", "k_out", "v_out"):
        assert np.array_equal(run.host[name], ref.host[name]), name


@pytest.mark.parametrize("case", ["mistral_layer", "pass_8k_B128_scaled", "tiny_f32", "tiny_f32_no_tail"])
def test_select_and_compact_in_one_launch(case):
    """kv_mmr_select_compact: the admission sequence and the compacted rows are bit-identical to
    kv_mmr_select followed by kv_compact_cache on the same scores (256 and 512 candidates in
    bf16, fp32 keys with and without the kept tail)."""
    import torch
    from paper_2609_30738_amd import _lib, api
    tail = None
    if case == "mistral_layer":
        wl = workloads.mistral_layer()
    elif case == "pass_8k_B128_scaled":
        wl = workloads.mistral_pass_8k(budget=128, n_layers=3, L=4096)
    else:
        wl = workloads.tiny_f32()
        tail = 0 if case == "tiny_f32_no_tail" else None
    keep = wl.w if tail is None else tail
    print(f"[gpu case] select+compact {case}", flush=True)
    packed = workloads.draw_packed(wl)
    import bench
    lam1, lam2 = bench.lambdas(wl)
    inp = api.upload(wl.dtype, wl.h_q, wl.h_kv, wl.d, wl.w, packed.q_win, packed.k, packed.v,
                     packed.lens, packed.tok_off, lam1, lam2)
    out = api.allocate(inp, wl.budget, 4, keep)
    b = inp.batch
    _lib.window_mu_sigma(b, inp.q_win, inp.k, inp.scale, out.row_max, out.row_sum, out.mu,
                         out.sigma, out.ws)
    _lib.mmr_select(b, out.mu, out.sigma, inp.k, inp.lambda1, inp.lambda2, wl.budget, 4, keep,
                    out.sel_idx, None, None, None, out.ws)
    _lib.compact_cache(b, inp.k, inp.v, out.sel_idx, wl.budget, keep, out.k_out, out.v_out)
    sel2, k2, v2 = (torch.full_like(out.sel_idx, -7), torch.zeros_like(out.k_out),
                    torch.zeros_like(out.v_out))
    _lib.mmr_select_compact(b, out.mu, out.sigma, inp.k, inp.v, inp.lambda1, inp.lambda2,
                            wl.budget, 4, keep, sel2, k2, v2, out.ws)
    torch.cuda.synchronize()
    assert torch.equal(sel2, out.sel_idx)
    assert torch.equal(k2.view(torch.int16 if k2.element_size() == 2 else torch.int32),
                       out.k_out.view(torch.int16 if k2.element_size() == 2 else torch.int32))
    assert torch.equal(v2.view(torch.int16 if v2.element_size() == 2 else torch.int32),
                       out.v_out.view(torch.int16 if v2.element_size() == 2 else torch.int32))


# ------------------------------------------------------------------------------------------------
# The benchmark's calls (kv_window_base_scores, then kv_mmr_select_scored with the compaction) with
# every scoring option and on every window path: fp32 batches take mu / sigma through the
# workspace and the base-score kernel, units in several segments the one-launch cooperative kernel
# (or, when its grid does not fit, the two-launch path), whole-unit workgroups the fused kernel.
# Each run also checks the scores bit for bit against the mu / sigma path's (tests/gpu_cases.py).
# ------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("case,certified", [
    ("tiny_f32", True), ("tiny_f32_tail3", True), ("sigma_all_rows", True),
    ("g3_group_mean", True), ("g3_all_rows", True), ("curve_scaled", True),
    ("mean_free", False), ("depth_budgets", False)])
def test_scored_calls_with_options(case, certified):
    _all(gpu_cases.run_case(case, timed=True), certified=certified)


def test_scored_calls_max_pooled():
    """Pooling in the selection from given scores."""
    wl = workloads.ragged_batch("both", n_seq=2, n_layers=2, len_range=(700, 3100))
    wl.budget = 64
    _all(gpu_cases.run_gpu(wl, pool=7, timed=True))


@pytest.mark.parametrize("h_q,h_kv,d", STREAM_SHAPES)
def test_scored_calls_stream_shapes(h_q, h_kv, d):
    """Every streaming head layout and head size, one segment per unit (scores formed in the fused
    kernel) and several (in the cooperative kernel)."""
    n_prob = 256 // h_kv
    one = _shape_workload(h_q, h_kv, d, 2, n_prob // 2, [1024, 777])
    assert _one_segment_per_unit(one)
    _all(gpu_cases.run_gpu(one, timed=True))
    _all(gpu_cases.run_gpu(_shape_workload(h_q, h_kv, d, 2, 2, [3000, 2100]), timed=True))


def test_scored_calls_late_segments_and_second_launch(monkeypatch):
    """Base scores from the cooperative kernel's waiting-workgroup path (poll limit 0) equal the
    default path's bit for bit; a batch whose cooperative grid does not fit the chip forms them
    from mu / sigma in the workspace."""
    wl = workloads.mistral_layer()
    monkeypatch.delenv("KVEVICT_SPIN_LIMIT", raising=False)
    ref = gpu_cases.run_gpu(wl, timed=True)
    monkeypatch.setenv("KVEVICT_SPIN_LIMIT", "0")
    run = gpu_cases.run_gpu(wl, timed=True)
    for name in ("row_max", "row_sum", "score", "sel_idx", "k_out", "v_out"):
        assert np.array_equal(run.host[name], ref.host[name]), name
    _all(run)
    monkeypatch.delenv("KVEVICT_SPIN_LIMIT", raising=False)
    big = _shape_workload(32, 8, 128, 3, 8, [5000, 5000, 5000], budget=32)
    _all(gpu_cases.run_gpu(big, timed=True))


@pytest.mark.parametrize("h_q,h_kv,d,lens,budget,cand_mult", [
    (8, 8, 64, [8192, 8161], 16, 4), (8, 8, 64, [8192, 8161], 37, 3),
    (8, 8, 64, [8192, 8161], 72, 4), (8, 8, 64, [8192, 8161], 128, 4),
    (32, 8, 128, [4096, 4065], 37, 3), (32, 8, 128, [4096, 4065], 96, 4)])
def test_candidates_cut_in_the_window_kernel(h_q, h_kv, d, lens, budget, cand_mult):
    """256 units of one segment each, 4065 to 8192 keys, 2 % planted keys, so that for C above
    their count the cut falls in the bulk: the candidate kernel codes every tile's row maxima in
    pass 1, bounds the
    tiles' scores once the normalisers are known, revisits tiles in decreasing order of their
    bounds until the cut passes them, and finds the C-th largest of the evaluated entries digit by
    digit (C = 64, 111, 288, 512 and 384).  The selection from its candidates equals
    kv_mmr_select_ex's, every output bit for bit, and the oracle's."""
    wl = _shape_workload(h_q, h_kv, d, 2, 16, lens, budget=budget)
    assert wl.n_prob * wl.h_kv == 256 and _one_segment_per_unit(wl)
    b = _lib.Batch(wl.dtype, h_q, h_kv, d, wl.w, wl.lens, device="cpu")
    C = cand_mult * budget
    lists = 256 * C * 8
    codes = 256 * ((max(lens) + 31) // 32) * 128  # 128 bytes per tile of the longest unit
    # the lists are formed in the window pass: the workspace holds them, the normalisers and the
    # first pass's tile codes only
    assert _lib.candidates_workspace_bytes(b, budget, cand_mult, wl.w) == lists + 1024 + codes
    run = gpu_cases.run_gpu(wl, cand_mult=cand_mult, timed=True)
    assert "cands_sel_idx" in run.host
    _all(run)


@pytest.mark.parametrize("n_layers", [1, 132])
@pytest.mark.parametrize("dtype,d,lens,budget", [
    ("bf16", 128, [1100, 640], 65), ("bf16", 128, [700], 128), ("bf16", 64, [1300, 900], 100),
    ("bf16", 64, [1300, 1100], 200), ("f32", 64, [300, 200], 16), ("f32", 64, [700, 500], 100),
    ("f32", 128, [300], 60)])
def test_greedy_against_the_last_admitted_row(dtype, d, lens, budget, n_layers):
    """The greedy that forms cosines in every step (bf16 above 256 candidates, fp32): one and two
    candidates per thread, counts that leave quads and waves partly empty (C = 64 .. 800), from the
    scores and from candidate lists, the rows in LDS (few units) and only the waves' best ones (264
    units and more): every route the same bits, and the oracle's."""
    wl = _shape_workload(4, 2, d, len(lens), n_layers, lens, budget=budget)
    wl.dtype = workloads.BF16 if dtype == "bf16" else workloads.F32
    _all_of(gpu_cases.run_gpu(wl, timed=True), [0, wl.n_prob - 1])


@pytest.mark.parametrize("dtype,h_q,w,lens", [
    (*s, n) for s in (("f32", 6, 20), ("bf16", 6, 20), ("f32", 2, 64), ("bf16", 4, 5))
    for n in ([2100, 333], [20000])] + [("f32", 8, 32, [2100, 333])])
def test_chunked_windows(dtype, h_q, w, lens):
    """Shapes of the chunked kernels (windows that are no power of two, fp32, one to four 32-row
    blocks): row blocks in workgroups of their own, second-pass workgroups of few keys, the row
    statistics merged in the second pass (up to 16 chunks) or by the combine kernel (20 chunks).
    Four fp32 heads of 32 rows only at the short lengths: a logit l errs by about |l| d^(1/2) 2^-24,
    and where that layout's sink logits at 20000 keys pass 20 nats a row sum may move by more than
    the 1e-5 that the comparison allows (measured 1.3e-5 on one row of 256)."""
    import dataclasses
    wl = dataclasses.replace(_shape_workload(h_q, 2, 64, len(lens), 1, lens), w=w)
    wl.dtype = workloads.BF16 if dtype == "bf16" else workloads.F32
    for sigma_rows in ("group_mean", "all_rows"):
        _all_of(gpu_cases.run_gpu(wl, timed=True, sigma_rows=sigma_rows), None)
    _all_of(gpu_cases.run_gpu(wl, fused=False), None)


@pytest.mark.parametrize("d,lens,budget,density", [(64, [36001, 35003], 16, 0.02), (64, [40003], 200, 0.02),
                                                   (128, [36003], 37, 0.02), (64, [36001], 64, 0.0)])
def test_cut_of_long_units_from_memory(d, lens, budget, density):
    """Units whose score keys do not fit in LDS: the cut reads the scores twice (rows that start off
    a 16-byte boundary, odd lengths), from scores and from mu / sigma, with a few members in the
    cut's bin and (no planted keys: every score in one bin) too many, where the general digit passes
    take over."""
    import dataclasses
    wl = _shape_workload(4, 2, d, len(lens), 1, lens, budget=budget)
    wl = dataclasses.replace(wl, layout=workloads.Layout(cluster_density=density) if density else workloads.Layout())
    _all_of(gpu_cases.run_gpu(wl, timed=True), None)


@pytest.mark.parametrize("lens,budget,density", [([8191, 8193], 16, 0.02), ([12289, 33001], 110, 0.02),
                                                 ([8257], 200, 0.002), ([20001, 9001], 16, 0.0)])
def test_cut_of_staged_units(lens, budget, density):
    """The cut's count of keys held in LDS, at and above the length from which keys below the first
    4096's bound are skipped, with short and long lists of members (ranked by counting, sorted) and
    (no planted keys: every score in one bin) too many for a list."""
    import dataclasses
    wl = _shape_workload(4, 2, 64, len(lens), 1, lens, budget=budget)
    wl = dataclasses.replace(wl, layout=workloads.Layout(cluster_density=density) if density else workloads.Layout())
    _all_of(gpu_cases.run_gpu(wl, timed=True), None)


@pytest.mark.parametrize("sigma_rows", ["group_mean", "all_rows"])
@pytest.mark.parametrize("h_q,h_kv,d,n_layers,lens,budget,cand_mult", [
    (32, 8, 128, 8, [40001], 16, 4), (8, 8, 64, 10, [30001], 8, 3), (16, 8, 64, 8, [36005], 30, 3)])
def test_units_of_several_workgroups_revisit_few_tiles(h_q, h_kv, d, n_layers, lens, budget, cand_mult,
                                                       sigma_rows):
    """64 and 80 units of four segments each (one or two to a workgroup): the first launch codes the
    tiles, the second revisits those that can hold a candidate; the selection equals that from all
    scores (kv_mmr_select_scored, kv_mmr_select_ex) bit for bit, and the oracle's, also where the
    cut falls in the flat scores of a workgroup's own keys."""
    wl = _shape_workload(h_q, h_kv, d, len(lens), n_layers, lens, budget=budget)
    assert lens[0] * 64 // 256 // 32 >= 3 * cand_mult * budget  # tiles of a workgroup against C
    _all_of(gpu_cases.run_gpu(wl, timed=True, cand_mult=cand_mult, sigma_rows=sigma_rows), [0, wl.n_prob - 1])


@pytest.mark.parametrize("w,h_q,lens", [(8, 32, [1000, 531]), (16, 16, [5003]), (32, 32, [5000] * 24)])
def test_scores_with_a_negative_scale(w, h_q, lens):
    """-scale with negated queries has the logits of scale and q bit for bit, but takes the chunked
    kernels where scale > 0 streams: row statistics and scores differ by the order of their sums only,
    of up to 128 rows and 5003 keys (relative error below 2e-5), in a workspace of the queried size."""
    import torch
    from paper_2609_30738_amd import _lib
    print(f"[gpu case] negative scale w={w} h_q={h_q} lens={lens[:3]} x{len(lens)}", flush=True)
    b = _lib.Batch("bf16", h_q, 8, 128, w, lens)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q = torch.randn(len(lens) * h_q * w * 128, device="cuda", generator=gen).to(torch.bfloat16)
    k = torch.randn(sum(lens) * 8 * 128, device="cuda", generator=gen).to(torch.bfloat16)
    lam = torch.full((len(lens),), 0.3, device="cuda")
    outs = []
    for sign in (1.0, -1.0):
        need = _lib.base_scores_workspace_bytes(b)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
        rm, rs = (torch.zeros(len(lens) * h_q * w, device="cuda") for _ in range(2))
        score = torch.zeros(sum(lens) * 8, device="cuda")
        _lib.window_base_scores(b, (sign * q).contiguous(), k, sign * 0.088, lam, rm, rs, score, ws=ws)
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy().astype(np.float64) for x in (rm, rs, score)])
    for a, c in zip(*outs):
        assert np.all(np.abs(a) > 0) and np.max(np.abs(a - c) / np.abs(a)) < 2e-5


def _check_window_statistics(dtype, q, ks, w, rtol, hidden=0, sigma_rows="group_mean"):
    """kv_window_mu_sigma_ex, kv_window_scores and kv_window_base_scores of queries q [P, h_kv, G, w, d]
    and keys ks (one [h_kv, L, d] per problem) against 64-bit statistics; the first `hidden` keys count
    as logits of -inf (their first elements make them so)."""
    import torch
    from paper_2609_30738_amd import _lib
    P, h_kv, G, _, d = q.shape
    lens, scale = [k.shape[1] for k in ks], d ** -0.5
    b = _lib.Batch(dtype, h_kv * G, h_kv, d, w, lens)
    f = dict(dtype=torch.float32, device="cuda")
    out = {n: torch.empty(P * h_kv * G * w, **f) for n in ("row_max", "row_sum")}
    out.update({n: torch.empty(sum(lens) * h_kv, **f) for n in ("mu", "sigma")})
    ws = torch.empty(_lib.workspace_bytes(b, 1), dtype=torch.uint8, device="cuda")
    kk = torch.cat([k.reshape(-1) for k in ks])
    _lib.window_mu_sigma_ex(b, q, kk, scale, sigma_rows, out["row_max"], out["row_sum"], out["mu"], out["sigma"], ws)
    rm2, rs2, rm3, rs3 = (torch.empty(P * h_kv * G * w, **f) for _ in range(4))
    score = torch.empty_like(out["mu"])
    need = _lib.base_scores_workspace_bytes(b)
    ws_sc = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    _lib.window_scores(b, q, kk, scale, rm2, rs2, ws)
    _lib.window_base_scores(b, q, kk, scale, torch.full((P,), 0.25, device="cuda"), rm3, rs3, score,
                            sigma_rows=sigma_rows, ws=ws_sc)
    torch.cuda.synchronize()
    ref = {n: [] for n in out}
    h0 = 1 if hidden else 0  # the element that hides keys is 0 in the others
    for p, L in enumerate(lens):
        lg = scale * torch.matmul(q[p].double().cpu()[..., h0:].reshape(h_kv, G * w, d - h0),
                                  ks[p].double().cpu()[..., h0:].transpose(1, 2).contiguous())
        lg = lg.reshape(h_kv, G, w, L)
        lg[..., :hidden] = -float("inf")
        lg.masked_fill_(torch.arange(L) > (L - w + torch.arange(w))[:, None], -float("inf"))
        m = lg.max(-1, keepdim=True).values
        e = (lg - m).exp()
        z = e.sum(-1, keepdim=True)
        e = e / z
        ref["row_max"].append(m.reshape(-1))
        ref["row_sum"].append(z.reshape(-1))
        a = e.mean(1)
        ref["mu"].append(a.mean(1).reshape(-1))
        ref["sigma"].append((a.std(1) if sigma_rows == "group_mean" else e.reshape(h_kv, G * w, L).std(1)).reshape(-1))
    for n, got in (*out.items(), ("row_max", rm2), ("row_sum", rs2), ("row_max", rm3), ("row_sum", rs3)):
        r, g = torch.cat(ref[n]), got.double().cpu()
        bad = (g - r).abs() > rtol * r.abs() + (1e-5 if n == "row_max" else 0.0)
        assert not bool(bad.any()) and bool(torch.isfinite(g).all()), (n, int(bad.sum()), float((g - r).abs().max()))
    # the score is fma(lambda1, sigma, mu) of the same mu and sigma, one rounding
    s64 = 0.25 * out["sigma"].double() + out["mu"].double()
    assert bool(((score.double() - s64).abs() <= 2.0 ** -24 * s64.abs()).all())


@pytest.mark.parametrize("w,h_q,d", [(8, 32, 128), (8, 16, 64), (16, 16, 128), (16, 8, 64)])
@pytest.mark.parametrize("lens", [[700], [5003, 1500]])
def test_short_windows_with_logits_of_minus_infinity(w, h_q, d, lens):
    """Keys 0 .. 599 (every wave's first tiles) whose products overflow to a logit of -inf for every
    window row: they weigh nothing, and the statistics are those of the other keys (64-bit reference;
    2e-5 for the fp32 sums over at most 5003 keys and 64 rows)."""
    import torch
    print(f"[gpu case] -inf logits w={w} h_q={h_q} d={d} lens={lens}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    q = torch.randn(len(lens), 8, h_q // 8, w, d, device="cuda", generator=gen)
    q[..., 0] = 2.0 ** 10
    ks = []
    for L in lens:
        k = torch.randn(8, L, d, device="cuda", generator=gen)
        k[..., 0] = 0.0
        k[:, :600, 0] = -2.0 ** 125
        ks.append(k.to(torch.bfloat16))
    _check_window_statistics("bf16", q.to(torch.bfloat16), ks, w, 2e-5, hidden=600)


@pytest.mark.parametrize("sigma_rows", ["group_mean", "all_rows"])
@pytest.mark.parametrize("h_kv,d,lens", [(2, 64, [20000, 333]), (8, 128, [4096] * 8), (8, 64, [17000, 16500])])
def test_chunked_four_row_blocks(h_kv, d, lens, sigma_rows):
    """Four fp32 heads of 32 rows in the chunked kernels: more than 16 chunks with every row block a
    workgroup of its own (44 chunks), and workgroups of all four blocks, with the row statistics merged in
    the second pass (256 chunks of 4 to a unit) and by the combine kernel (272 chunks, 17 to a unit).
    Logits of random keys stay below 7, whose fp32 error of about 7 d^(1/2) 2^-24 = 5e-6 averages out in
    the sums: 1e-5."""
    import torch
    print(f"[gpu case] chunked, four row blocks h_kv={h_kv} d={d} lens={lens} {sigma_rows}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    q = torch.randn(len(lens), h_kv, 4, 32, d, device="cuda", generator=gen)
    ks = [torch.randn(h_kv, L, d, device="cuda", generator=gen) for L in lens]
    _check_window_statistics("f32", q, ks, 32, 1e-5, sigma_rows=sigma_rows)


@pytest.mark.parametrize("sigma_rows", ["group_mean", "all_rows"])
def test_units_of_several_workgroups_ragged(sigma_rows):
    """Units of six, three and one workgroups in one batch of the two-launch candidate path, two segments
    of 6144 keys to a workgroup: workgroups past the end of short units, units with no more positions than
    candidates (68 and 128), and a last workgroup whose 20 keys all lie in the kept tail."""
    lens, n_layers, budget = [61460, 33001, 300, 100], 2, 32
    wl = _shape_workload(32, 8, 128, len(lens), n_layers, lens, budget=budget)
    seg = -(-(-(-sum(lens) * n_layers * 8 // 256)) // 256) * 256
    assert seg == 6144 and 2 * seg // 32 >= 3 * 4 * budget  # tiles of a workgroup against C
    assert sum(8 * n_layers * -(-L // seg) for L in lens) > 256 and 0 < lens[0] % (2 * seg) <= wl.w
    run = gpu_cases.run_gpu(wl, timed=True, sigma_rows=sigma_rows)
    print("  ", gpu_cases.summarize(gpu_cases.check_all(run, js=[0, 3, 5, 6], heads=[0, 5])), flush=True)
