"""Parity of the HIP path (through the C ABI) with the CPU oracle.  Needs an MI355X.

Discrete results (candidate order, first crossings, r*, eviction sets, the
committed bank layout, densities, baselines, K/V bytes) must be bit-identical;
attention must be within the row-normalised max error 2e-2 (bf16) / 1e-5 (fp32).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import (Q23, BankState, attention, candidate_scores, density_from_scratch, pair_d2,  # noqa: E402
                    update_layer, weight_q23)
from paper_2608_27922_amd import api, synth  # noqa: E402
from gpu_util import (TORCH_DT, assert_bank_equal, assert_trace_equal, attention_error, dev, host,  # noqa: E402
                      mirror, oracle_params, oracle_step)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    api.lib()


def _log(msg):
    print(msg, flush=True)


# ----------------------------------------------------------------------------- per-pair contract

@pytest.mark.parametrize("s,p", [(6, 2), (5, 2), (6, 1), (6, 4), (4, 2), (8, 2), (0, 1)])
def test_pair_weight_exhaustive(s, p):
    """Every squared distance the key grid can produce (d2 * 2^12 in [0, 8258048])."""
    _log(f"pair weight sweep s={s} p={p}")
    n = np.arange(0, 8_258_049, dtype=np.float64)
    d2 = n / 4096.0
    ref = weight_q23(d2, oracle_params(api.Params(sigma2_log2=s, p=p)))
    got = api.pair_weight_q23(torch.from_numpy(d2.astype(np.float32)).cuda(), api.Params(sigma2_log2=s, p=p))
    got = got.cpu().numpy().astype(np.int64)
    bad = np.nonzero(got != ref)[0]
    assert bad.size == 0, f"{bad.size} mismatches, first d2*4096={n[bad[:5]]} got {got[bad[:5]]} ref {ref[bad[:5]]}"


# ----------------------------------------------------------------------------- rollouts

def _run_rollout(cfg, blocks, prm, budgets=None, dup_every=0, trace=True, init_full=False, check_every=1,
                 grid_values=False, seq_groups=None):
    """Rollout over one layer of `cfg`: GPU update + oracle update per block, compared
    (seq_groups: workspace for that many groups' pairwise weights, sequential policy)."""
    B, gs, d, dt = cfg.heads, cfg.group_size, cfg.d, cfg.dtype
    if budgets is None:
        budgets = np.full(B, cfg.budget, np.int32)
    Mcap = int(max(budgets))
    bank = api.Bank(B, Mcap, d, dtype=torch.bfloat16 if dt == "bf16" else torch.float32, group_size=gs,
                    budget=torch.from_numpy(np.asarray(budgets, np.int32)))
    obanks = [BankState.empty(int(budgets[b]), d) for b in range(B)]
    op = oracle_params(prm)
    streams = [synth.HeadStream(cfg, 0, h) for h in range(B)]
    ws = None
    if seq_groups is not None:
        n_max = max(Mcap if init_full else cfg.n_cand, cfg.n_cand)
        ws = api.alloc_workspace(bank, n_max, prm.flags, seq_groups=seq_groups)
    for t in range(blocks):
        n = Mcap if (init_full and t == 0) else cfg.n_cand
        K = np.stack([s.keys(t, n) for s in streams])
        V = np.stack([s.values(t, n) for s in streams])
        if grid_values:  # the [K; V] geometry needs values on the key grid too (exact descriptor Gram)
            V = (np.clip(np.rint(V * 64.0), -127, 127) / 64.0).astype(np.float32)
        if dup_every and t > 0 and t % dup_every == 0:
            for h in range(B):
                if obanks[h].m:
                    K[h] = streams[h].near_duplicates(K[h], obanks[h].K.astype(np.float32), t)
        out = api.UpdateOut(bank, n, trace=trace)
        api.update_bank(bank, dev(K, dt), dev(V, dt), t, prm, workspace=ws, out=out)
        torch.cuda.synchronize()
        new, recs = oracle_step(obanks, K, V, t, op, gs)
        if t % check_every == 0 or t == blocks - 1:
            if trace:
                assert_trace_equal(out, recs, gs, obanks, n, ctx=f"block {t}",
                                   sequential=bool(prm.flags & api.POLICY_SEQUENTIAL))
            for b in range(B):
                assert_bank_equal(bank, b, new[b], ctx=f"block {t}", kv=bool(prm.flags & api.POLICY_KV_DESCRIPTOR))
        obanks = new
    return bank, obanks


SMALL = dict(seed_id=77, name="small", layers=1, n_query=40, n_window=24, clusters=6, blocks=6, sigma2_log2=4,
             drift=0.05)


@pytest.mark.parametrize("dt,d", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
def test_rollout_small_shared_prefix(dt, d):
    """6 banks in 2 groups of 3, budget 300 (ragged tiles), 200 candidates per block,
    near-duplicate blocks to force mandatory evictions."""
    _log(f"rollout small dt={dt} d={d}")
    cfg = synth.Config(heads=6, d=d, dtype=dt, n_cand=200, budget=300, group_size=3, **SMALL)
    _run_rollout(cfg, 6, api.Params(sigma2_log2=4 if d == 64 else 5), dup_every=2)


@pytest.mark.parametrize("trace", [True, False])
def test_rollout_checkpoint_tiles(trace):
    """N = 700 > 256 candidates: prefix checkpoints plus a partial tile at r*
    (without the trace outputs the crossing search may end after its first part)."""
    _log(f"rollout checkpoint tiles trace={trace}")
    cfg = synth.Config(heads=4, d=128, dtype="bf16", n_cand=700, budget=1000, group_size=2, **SMALL)
    _run_rollout(cfg, 4, api.Params(sigma2_log2=5), dup_every=2, trace=trace)


@pytest.mark.parametrize("n,trace", [(1, True), (64, True), (65, True), (256, False), (257, False), (512, True),
                                     (513, True), (513, False), (1025, True), (1025, False)])
def test_rollout_candidate_count_boundaries(n, trace):
    """Candidate counts at the edges of the 64-candidate chunks, the 256-candidate
    first part of the crossing search, the 512-key sort chunks, the 128-row Gram
    blocks and the runs of the symmetric admitted x admitted Gram (budget 1,100: the first
    blocks admit everything, later ones evict); without the trace outputs the
    crossing search may end after its first part."""
    _log(f"rollout candidate count n={n} trace={trace}")
    cfg = synth.Config(heads=2, d=128, dtype="bf16", n_cand=n, budget=1100, group_size=2, **SMALL)
    _run_rollout(cfg, 4, api.Params(sigma2_log2=5), dup_every=2, trace=trace)


def test_rollout_ragged_budgets_independent_heads():
    """group_size = 1 with per-head budgets (the independent per-head variant)."""
    _log("rollout ragged budgets")
    cfg = synth.Config(heads=5, d=128, dtype="bf16", n_cand=150, budget=400, group_size=1, **SMALL)
    _run_rollout(cfg, 6, api.Params(sigma2_log2=5), budgets=np.array([120, 400, 260, 150, 333], np.int32),
                 dup_every=2)


def test_rollout_group_ragged_budgets():
    """Shared prefix over a group whose budgets differ: r <= min budget, e_r per head."""
    _log("rollout group ragged budgets")
    cfg = synth.Config(heads=4, d=64, dtype="f32", n_cand=90, budget=200, group_size=4, **SMALL)
    _run_rollout(cfg, 5, api.Params(sigma2_log2=4), budgets=np.array([200, 130, 170, 90], np.int32),
                 dup_every=2)


@pytest.mark.parametrize("tau,p,s", [((3, 1), 2, 5), ((3, 0), 1, 6), ((2, 0), 4, 6)])
def test_rollout_parameter_sweep(tau, p, s):
    """tau in {1.5, 3}, p in {1, 4}, sigma^2 in {32, 64} (the paper's sweeps)."""
    _log(f"rollout params tau={tau} p={p} s={s}")
    cfg = synth.Config(heads=3, d=128, dtype="bf16", n_cand=120, budget=250, group_size=3, **SMALL)
    _run_rollout(cfg, 5, api.Params(sigma2_log2=s, p=p, tau_num=tau[0], tau_log2_den=tau[1]), dup_every=2)


POLICY_FLAGS = {"source_order": api.POLICY_SOURCE_ORDER, "refresh_base": api.POLICY_REFRESH_BASE,
                "densest_only": api.POLICY_DENSEST_ONLY, "source_fill": api.POLICY_SOURCE_FILL,
                "source_order+refresh": api.POLICY_SOURCE_ORDER | api.POLICY_REFRESH_BASE}


@pytest.mark.parametrize("dt,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("policy", list(POLICY_FLAGS))
def test_rollout_policy_ablations(policy, dt, d):
    """The policy ablations of Table 1(b): same rollout shape as the default test,
    near-duplicate blocks (mandatory evictions) and full banks (fills), every
    intermediate and the committed bank bit-exact against the oracle run with the
    same policy."""
    _log(f"rollout policy {policy} dt={dt} d={d}")
    cfg = synth.Config(heads=6, d=d, dtype=dt, n_cand=200, budget=300, group_size=3, **SMALL)
    _run_rollout(cfg, 6, api.Params(sigma2_log2=4 if d == 64 else 5, flags=POLICY_FLAGS[policy]), dup_every=2)


@pytest.mark.parametrize("policy", sorted(POLICY_FLAGS))
def test_rollout_policy_ablations_no_trace(policy):
    """Every policy ablation with 600 candidates per block (more than the 256 of
    the crossing search's first part) and without trace outputs, so that the
    search may end after its first part: the committed banks bit-exact against
    the oracle run with the same policy."""
    _log(f"rollout policy {policy} no trace")
    cfg = synth.Config(heads=4, d=128, dtype="bf16", n_cand=600, budget=1000, group_size=2, **SMALL)
    _run_rollout(cfg, 5, api.Params(sigma2_log2=5, flags=POLICY_FLAGS[policy]), dup_every=2, trace=False)


@pytest.mark.parametrize("dt,d", [("bf16", 128), ("bf16", 64)])
def test_rollout_kv_descriptor(dt, d):
    """The [K; V] retention geometry (descriptor dimension 2 d: 256 and 128) on the
    near-duplicate rollout, every intermediate and the committed bank bit-exact against
    the oracle run on the concatenated descriptors."""
    _log(f"rollout kv descriptor dt={dt} d={d}")
    cfg = synth.Config(heads=6, d=d, dtype=dt, n_cand=200, budget=300, group_size=3, **SMALL)
    _run_rollout(cfg, 6, api.Params(sigma2_log2=5 if d == 64 else 6, flags=api.POLICY_KV_DESCRIPTOR), dup_every=2,
                 grid_values=True)


@pytest.mark.parametrize("trace", [True, False])
def test_rollout_kv_descriptor_multi_split(trace):
    """The [K; V] geometry at descriptor dimension 256 across the tiling edges: banks of
    2,600 states filled by the empty-bank rule (three 1,024-column score splits), then
    1,100 candidates per block (three 512-key sort chunks, 18 prefix chunks, admitted x
    admitted in three half-splits of 512 columns) into full banks, every block releasing
    1,100 states by the densest fill (survivors x evicted 1,500 x 1,100); every
    intermediate (with trace outputs) and the committed bank bit-exact against the
    oracle on the concatenated descriptors."""
    _log(f"rollout kv descriptor multi-split trace={trace}")
    cfg = synth.Config(heads=2, d=128, dtype="bf16", n_cand=1100, budget=2600, group_size=2, **SMALL)
    bank, obanks = _run_rollout(cfg, 4, api.Params(sigma2_log2=6, flags=api.POLICY_KV_DESCRIPTOR), dup_every=2,
                                init_full=True, grid_values=True, trace=trace)
    assert all(b.m == 2600 for b in obanks)


@pytest.mark.parametrize("dt,d,tau", [("bf16", 128, 3), ("bf16", 64, 3), ("bf16", 128, 2)])
def test_rollout_sequential_competition(dt, d, tau):
    """Within-block sequential competition (DKV_POLICY_SEQUENTIAL): 6 banks in 2
    groups of 3, budget 300, 200 candidates per block with near-duplicate blocks;
    the first block fills the empty banks (empty-bank rule), then every step of
    every block is decided on the device.  Order, scores, steps taken, admitted and
    released lists, and the committed banks (layout, K/V, rho, base, knorm) are
    bit-exact against the oracle."""
    _log(f"rollout sequential dt={dt} d={d} tau={tau}")
    cfg = synth.Config(heads=6, d=d, dtype=dt, n_cand=200, budget=300, group_size=3, **SMALL)
    prm = api.Params(sigma2_log2=4 if d == 64 else 5, tau_num=tau, flags=api.POLICY_SEQUENTIAL)
    _run_rollout(cfg, 5, prm, dup_every=2)


@pytest.mark.parametrize("seq_groups", [1, 2])
def test_sequential_batches_of_groups(seq_groups):
    """The sequential competition with a workspace that holds the pairwise
    weights of 1 or 2 groups: 9 banks in 3 groups of 3 (ragged budgets 300 /
    260 / 300) are walked in batches of 1 group (three batches) or 2 groups (a
    full batch and a ragged one), every result bit-exact against the oracle.
    The workspace is smaller than the size query's by 2 or 1 groups of weights."""
    _log(f"sequential batches of {seq_groups} groups")
    cfg = synth.Config(heads=9, d=128, dtype="bf16", n_cand=200, budget=300, group_size=3, **SMALL)
    prm = api.Params(sigma2_log2=5, tau_num=3, flags=api.POLICY_SEQUENTIAL)
    budgets = np.array([300, 260, 300] * 3, np.int32)
    bank = api.Bank(9, 300, 128, dtype=torch.bfloat16, group_size=3)
    full = api.workspace_size(bank, 200, prm.flags)
    per = api.seq_group_weight_bytes(bank, 200)
    assert api.alloc_workspace(bank, 200, prm.flags, seq_groups=seq_groups).numel() == full - (3 - seq_groups) * per
    _run_rollout(cfg, 5, prm, budgets=budgets, dup_every=2, seq_groups=seq_groups)


def test_sequential_workspace_below_one_group_is_rejected():
    """A sequential workspace without room for one group's pairwise weights is
    DKV_ERR_WORKSPACE, and the bank is left as it was."""
    _log("sequential workspace below one group")
    bank = api.Bank(6, 300, 128, dtype=torch.bfloat16, group_size=3)
    prm = api.Params(sigma2_log2=5, flags=api.POLICY_SEQUENTIAL)
    full = api.workspace_size(bank, 200, prm.flags)   # fixed part + both groups' weights (256-byte aligned)
    per = api.seq_group_weight_bytes(bank, 200)
    fixed = full - (2 * per + 255) // 256 * 256
    ws = torch.empty(fixed + per - 1, dtype=torch.uint8, device="cuda")
    K = torch.zeros(6, 200, 128, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(api.DkvError):
        api.update_bank(bank, K, K.clone(), 0, prm, workspace=ws)
    torch.cuda.synchronize()
    assert int(bank.occupancy.sum()) == 0


def test_sequential_banks_spanning_workgroups():
    """Sequential competition on banks of 2,500-2,600 slots (ragged budgets 2,600 /
    2,500 / 2,560): each bank's slots span two workgroups of the multi-workgroup
    walk, so every step merges the records of six workgroups.  The first block
    fills the banks from empty with 2,300 keys and exact copies of 200 of them
    (sigma^2 = 1/2, d = 128); then 100 copies of bank keys and 100 fresh keys per
    block, in source order (rejected steps on banks that are not full) and in
    score order (steps that release a violator).  Every block bit-exact against
    the oracle, which must see both kinds of steps."""
    _log("sequential banks spanning workgroups")
    rng = np.random.default_rng(7)
    budgets = np.array([2600, 2500, 2560], np.int32)
    B, gs, d = 3, 3, 128
    bank = api.Bank(B, int(budgets.max()), d, dtype=torch.bfloat16, group_size=gs,
                    budget=torch.from_numpy(budgets))
    obanks = [BankState.empty(int(M), d) for M in budgets]
    taken_with_violator = rejected = 0
    for t, flags in enumerate([0, api.POLICY_SOURCE_ORDER, 0]):
        prm = api.Params(sigma2_log2=-1, flags=api.POLICY_SEQUENTIAL | flags)
        if t == 0:
            K = np.stack([np.concatenate([k, k[:200]])
                          for k in (synth.random_grid_keys(rng, (2300, d)) for _ in range(B))])
        else:
            K = np.stack([np.concatenate([obanks[h].K[rng.choice(obanks[h].m, 100, replace=False)].astype(np.float32),
                                          synth.random_grid_keys(rng, (100, d))]) for h in range(B)])
            for h in range(B):
                rng.shuffle(K[h])
        V = synth.random_grid_keys(rng, K.shape)
        n = K.shape[1]
        out = api.UpdateOut(bank, n, trace=True)
        api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), t, prm, out=out)
        torch.cuda.synchronize()
        new, recs = oracle_step(obanks, K, V, t, oracle_params(prm), gs)
        assert_trace_equal(out, recs, gs, obanks, n, ctx=f"block {t}", sequential=True)
        for b in range(B):
            assert_bank_equal(bank, b, new[b], ctx=f"block {t}")
        if t > 0:
            rec = recs[0]
            rejected += int((~rec.steps).sum())
            taken_with_violator += sum(int(((hr.c > 0) & rec.steps).sum()) for hr in rec.heads)
        obanks = new
    assert rejected > 0 and taken_with_violator > 0


def test_sequential_part_boundary_and_empty_bank():
    """Sequential competition in a group whose banks have budgets 2,049, 0 and
    2,100: the first bank's last slot (2,048) belongs to the second workgroup of
    the bank, so states enter a part that held none; the budget-0 bank stays
    empty, takes the empty-bank rule every block and stays out of the shared
    test.  d = 64, sigma^2 = 1/2, exact copies of bank keys among fresh keys,
    source order then score order; bit-exact against the oracle, which must see
    rejected steps and steps that release a violator."""
    _log("sequential part boundary and empty bank")
    rng = np.random.default_rng(11)
    budgets = np.array([2049, 0, 2100], np.int32)
    B, gs, d = 3, 3, 64
    bank = api.Bank(B, int(budgets.max()), d, dtype=torch.bfloat16, group_size=gs,
                    budget=torch.from_numpy(budgets))
    obanks = [BankState.empty(int(M), d) for M in budgets]
    taken_with_violator = rejected = 0
    for t, flags in enumerate([0, api.POLICY_SOURCE_ORDER, 0]):
        prm = api.Params(sigma2_log2=-1, flags=api.POLICY_SEQUENTIAL | flags)
        if t == 0:
            K = np.stack([np.concatenate([k, k[:100]])
                          for k in (synth.random_grid_keys(rng, (1900, d)) for _ in range(B))])
        else:
            K = np.stack([np.concatenate([obanks[h].K[rng.choice(obanks[h].m, 100, replace=False)].astype(np.float32)
                                          if obanks[h].m else synth.random_grid_keys(rng, (100, d)),
                                          synth.random_grid_keys(rng, (100, d))]) for h in range(B)])
            for h in range(B):
                rng.shuffle(K[h])
        V = synth.random_grid_keys(rng, K.shape)
        n = K.shape[1]
        out = api.UpdateOut(bank, n, trace=True)
        api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), t, prm, out=out)
        torch.cuda.synchronize()
        new, recs = oracle_step(obanks, K, V, t, oracle_params(prm), gs)
        assert_trace_equal(out, recs, gs, obanks, n, ctx=f"block {t}", sequential=True)
        for b in range(B):
            assert_bank_equal(bank, b, new[b], ctx=f"block {t}")
        if t > 0:
            rec = recs[0]
            rejected += int((~rec.steps).sum())
            taken_with_violator += sum(int(((hr.c > 0) & rec.steps).sum()) for hr in rec.heads)
        obanks = new
    assert int(bank.occupancy[0].item()) == 2049 and int(bank.occupancy[1].item()) == 0
    assert rejected > 0 and taken_with_violator > 0


@pytest.mark.parametrize("n", [1, 65])
def test_sequential_candidate_counts(n):
    """Sequential competition with 1 and 65 candidates per block into banks that
    the first block fills (budget 150, three banks per group), then an empty
    segment, which must leave the banks unchanged and report no step."""
    _log(f"sequential candidate count n={n}")
    cfg = synth.Config(heads=3, d=128, dtype="bf16", n_cand=n, budget=150, group_size=3, **SMALL)
    prm = api.Params(sigma2_log2=5, tau_num=3, flags=api.POLICY_SEQUENTIAL)
    bank, _ = _run_rollout(cfg, 5, prm, dup_every=2, init_full=True)
    before = bank.state_dict()
    out = api.UpdateOut(bank, 0)
    out.r_star.fill_(-7)
    api.update_bank(bank, None, None, 9, prm, out=out)
    torch.cuda.synchronize()
    for name, t in bank.state_dict().items():
        assert torch.equal(t, before[name]), name
    assert int(out.r_star[0].item()) == 0


def test_sequential_sixteen_slots_per_thread():
    """Sequential competition in a group of 33 banks of budget 2,100: at 2,048
    slots per workgroup the group would need 66 workgroups, more than the walk
    takes, so it runs with 16 slots per thread (4,096 per workgroup, 33
    workgroups) and states enter slots past 2,048 of a workgroup.  d = 64,
    sigma^2 = 1/2, exact copies of bank keys among fresh keys, source order
    (every step rejected: some bank of the group has a violator) then score
    order (steps that release a violator); bit-exact against the oracle."""
    _log("sequential sixteen slots per thread")
    rng = np.random.default_rng(13)
    B, gs, d, M = 33, 33, 64, 2100
    bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=gs)
    obanks = [BankState.empty(M, d) for _ in range(B)]
    taken_with_violator = rejected = 0
    for t, flags in enumerate([0, api.POLICY_SOURCE_ORDER, 0]):
        prm = api.Params(sigma2_log2=-1, flags=api.POLICY_SEQUENTIAL | flags)
        if t == 0:
            K = np.stack([np.concatenate([k, k[:100]])
                          for k in (synth.random_grid_keys(rng, (1900, d)) for _ in range(B))])
        else:
            K = np.stack([np.concatenate([obanks[h].K[rng.choice(obanks[h].m, 60, replace=False)].astype(np.float32),
                                          synth.random_grid_keys(rng, (100, d))]) for h in range(B)])
            for h in range(B):
                rng.shuffle(K[h])
        V = synth.random_grid_keys(rng, K.shape)
        n = K.shape[1]
        out = api.UpdateOut(bank, n, trace=True)
        api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), t, prm, out=out)
        torch.cuda.synchronize()
        new, recs = oracle_step(obanks, K, V, t, oracle_params(prm), gs)
        assert_trace_equal(out, recs, gs, obanks, n, ctx=f"block {t}", sequential=True)
        for b in range(B):
            assert_bank_equal(bank, b, new[b], ctx=f"block {t}")
        if t > 0:
            rec = recs[0]
            rejected += int((~rec.steps).sum())
            taken_with_violator += sum(int(((hr.c > 0) & rec.steps).sum()) for hr in rec.heads)
        obanks = new
    assert int(bank.occupancy.min().item()) == M
    assert rejected > 0 and taken_with_violator > 0


def test_sequential_wide_group():
    """Sequential competition with 72 banks sharing each step (more banks than
    the multi-workgroup walk takes, so one workgroup walks the group): budget 120,
    80 candidates per block, near-duplicate blocks; bit-exact against the oracle."""
    _log("sequential wide group")
    cfg = synth.Config(heads=72, d=64, dtype="bf16", n_cand=80, budget=120, group_size=72, **SMALL)
    prm = api.Params(sigma2_log2=4, tau_num=3, flags=api.POLICY_SEQUENTIAL)
    _run_rollout(cfg, 4, prm, dup_every=2)


def test_sequential_violators_and_rejected_steps():
    """Sequential competition with exact duplicates of bank keys among sparse grid
    keys (sigma^2 = 4, d = 128), on two bank sets that both start empty.  Score
    order fills the banks and then takes steps that release a violator; source
    order on a bank that is not full rejects the steps whose candidate makes a
    state violate.  Every block bit-exact against the oracle, which must see both
    kinds of steps."""
    _log("sequential violators and rejected steps")
    B, gs, d, M = 3, 3, 128, 300
    taken_with_violator = rejected = 0
    for schedule in ([0, 0, 0], [0, api.POLICY_SOURCE_ORDER]):
        rng = np.random.default_rng(5)
        bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=gs)
        obanks = [BankState.empty(M, d) for _ in range(B)]
        for t, flags in enumerate(schedule):
            prm = api.Params(sigma2_log2=2, flags=api.POLICY_SEQUENTIAL | flags)
            if t == 0:
                # 230 keys and exact copies of the first 20 of them
                K = np.stack([np.concatenate([k, k[:20]])
                              for k in (synth.random_grid_keys(rng, (230, d)) for _ in range(B))])
            else:
                # 100 copies of bank keys and 100 fresh keys, shuffled
                K = np.stack([np.concatenate([obanks[h].K[rng.choice(obanks[h].m, 100, replace=False)].astype(np.float32),
                                              synth.random_grid_keys(rng, (100, d))]) for h in range(B)])
                for h in range(B):
                    rng.shuffle(K[h])
            V = synth.random_grid_keys(rng, K.shape)
            n = K.shape[1]
            out = api.UpdateOut(bank, n, trace=True)
            api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), t, prm, out=out)
            torch.cuda.synchronize()
            new, recs = oracle_step(obanks, K, V, t, oracle_params(prm), gs)
            ctx = f"schedule {schedule} block {t}"
            assert_trace_equal(out, recs, gs, obanks, n, ctx=ctx, sequential=True)
            for b in range(B):
                assert_bank_equal(bank, b, new[b], ctx=ctx)
            if t > 0:
                rec = recs[0]
                rejected += int((~rec.steps).sum())
                taken_with_violator += sum(int(((hr.c > 0) & rec.steps).sum()) for hr in rec.heads)
            obanks = new
    assert rejected > 0 and taken_with_violator > 0


def test_rollout_sequential_with_source_order_and_refresh():
    """The sequential competition combined with source-order candidates and
    refreshed baselines (the combinations it admits), independent heads."""
    _log("rollout sequential + source order + refresh")
    cfg = synth.Config(heads=4, d=128, dtype="bf16", n_cand=150, budget=250, group_size=1, **SMALL)
    prm = api.Params(sigma2_log2=5, tau_num=3,
                     flags=api.POLICY_SEQUENTIAL | api.POLICY_SOURCE_ORDER | api.POLICY_REFRESH_BASE)
    _run_rollout(cfg, 4, prm, dup_every=2)


def test_kv_descriptor_score_and_density():
    """densitykv_score with the [K; V] geometry: candidate scores and the bank's own
    densities against the oracle on concatenated descriptors."""
    _log("score kv descriptor")
    rng = np.random.default_rng(12)
    B, M, N, d = 3, 200, 150, 128
    grid = lambda a: np.clip(np.rint(a * 64.0), -127, 127) / 64.0
    Kb, Vb = grid(rng.standard_normal((B, M, d)) * 0.4), grid(rng.standard_normal((B, M, d)) * 0.4)
    Kc, Vc = grid(rng.standard_normal((B, N, d)) * 0.4), grid(rng.standard_normal((B, N, d)) * 0.4)
    prm = api.Params(sigma2_log2=6, flags=api.POLICY_KV_DESCRIPTOR)
    op = oracle_params(prm)
    bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=1)
    # build the banks through the update (empty-bank rule), then score a second segment
    api.update_bank(bank, dev(Kb, "bf16"), dev(Vb, "bf16"), 0, prm)
    sq, _, dens = api.score(bank, dev(Kc, "bf16"), dev(Vc, "bf16"), prm, want_density=True)
    torch.cuda.synchronize()
    for b in range(B):
        ob = BankState.empty(M, d)
        (ob,), _ = update_layer([ob], [Kb[b]], [Vb[b].astype(np.float32)], 0, op)
        desc_b = np.hstack([ob.K, ob.V.astype(np.float64)])
        S, _, _ = candidate_scores(desc_b, ob.base, np.hstack([Kc[b], Vc[b]]), op)
        assert np.array_equal(sq[b].cpu().numpy(), S), f"bank {b}: scores differ"
        assert np.array_equal(dens[b, :ob.m].cpu().numpy(), density_from_scratch(desc_b, op)), f"bank {b}: density"


def test_empty_bank_more_candidates_than_budget():
    """Alg. 1 first branch: first min(N, M) source-ordered candidates, N > M."""
    _log("empty bank N > M")
    cfg = synth.Config(heads=2, d=128, dtype="bf16", n_cand=300, budget=170, group_size=2, **SMALL)
    _run_rollout(cfg, 1, api.Params(sigma2_log2=5))


def test_zero_candidates_and_determinism():
    """N = 0 leaves a valid bank unchanged; the same update twice gives identical bits."""
    _log("zero candidates + determinism")
    cfg = synth.Config(heads=3, d=128, dtype="bf16", n_cand=100, budget=150, group_size=3, **SMALL)
    bank, obanks = _run_rollout(cfg, 3, api.Params(sigma2_log2=5), dup_every=2)
    before = bank.state_dict()
    api.update_bank(bank, None, None, 9, api.Params(sigma2_log2=5))
    torch.cuda.synchronize()
    for n, t in bank.state_dict().items():
        assert torch.equal(t, before[n]), n
    # determinism: replay one update from a checkpoint twice
    s = synth.HeadStream(cfg, 0, 0)
    K = np.stack([synth.HeadStream(cfg, 0, h).keys(11, 100) for h in range(3)])
    V = np.stack([synth.HeadStream(cfg, 0, h).values(11, 100) for h in range(3)])
    results = []
    for _ in range(2):
        bank.load_state_dict(before)
        api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), 11, api.Params(sigma2_log2=5))
        torch.cuda.synchronize()
        results.append(bank.state_dict())
    for n in results[0]:
        assert torch.equal(results[0][n], results[1][n]), n
    del s


def test_all_duplicate_candidates():
    """Every candidate is an exact copy of one bank key: weights of exactly 1 everywhere."""
    _log("all-duplicate candidates")
    prm = api.Params(sigma2_log2=5)
    B, d, M, N = 2, 128, 64, 40
    rng = np.random.default_rng(4)
    bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=2)
    K0 = synth.random_grid_keys(rng, (B, M, d))
    V0 = synth.to_storage(rng.standard_normal((B, M, d)), "bf16")
    api.update_bank(bank, dev(K0, "bf16"), dev(V0, "bf16"), 0, prm)
    obanks, _ = oracle_step([BankState.empty(M, d) for _ in range(B)], K0, V0, 0, oracle_params(prm), 2)
    K1 = np.repeat(K0[:, 3:4], N, axis=1)
    V1 = synth.to_storage(rng.standard_normal((B, N, d)), "bf16")
    out = api.UpdateOut(bank, N, trace=True)
    api.update_bank(bank, dev(K1, "bf16"), dev(V1, "bf16"), 1, prm, out=out)
    torch.cuda.synchronize()
    new, recs = oracle_step(obanks, K1, V1, 1, oracle_params(prm), 2)
    assert_trace_equal(out, recs, 2, obanks, N)
    for b in range(B):
        assert_bank_equal(bank, b, new[b])


def test_corrupted_bank_is_compacted():
    """Outside the paper's precondition (states already violating): r* = 0, violators
    are evicted and the survivors beyond the new occupancy close the holes."""
    _log("corrupted bank")
    prm = api.Params(sigma2_log2=5)
    B, d, M = 2, 64, 100
    rng = np.random.default_rng(8)
    bank = api.Bank(B, M, d, dtype=torch.float32, group_size=1)
    K0 = synth.random_grid_keys(rng, (B, 60, d))
    V0 = synth.to_storage(rng.standard_normal((B, 60, d)), "f32")
    api.update_bank(bank, dev(K0, "f32"), dev(V0, "f32"), 0, prm)
    torch.cuda.synchronize()
    for b in range(B):
        for s in (2, 7, 30):
            bank.base[b, s] = bank.rho[b, s] // 4
    obanks = [mirror(bank, b) for b in range(B)]
    K1 = synth.random_grid_keys(rng, (B, 10, d))
    V1 = synth.to_storage(rng.standard_normal((B, 10, d)), "f32")
    out = api.UpdateOut(bank, 10, trace=True)
    api.update_bank(bank, dev(K1, "f32"), dev(V1, "f32"), 1, prm, out=out)
    torch.cuda.synchronize()
    new, recs = oracle_step(obanks, K1, V1, 1, oracle_params(prm), 1)
    assert all(r.r_star == 0 for r in recs)
    assert_trace_equal(out, recs, 1, obanks, 10)
    for b in range(B):
        assert_bank_equal(bank, b, new[b])


def _spread_case(d, kv, seed):
    """Two banks of 600 grid states (five 128-state workgroups and a partial one)
    and 1,000 candidates (15 whole 64-candidate chunks and one of 40), with every
    state's baseline set so that its bound lies a uniform fraction U in
    [-0.15, 1.15] of its total weight to the candidates above rho (tau = 2:
    2 b - rho = U T): first crossings spread over every chunk, and some states
    never cross (U > 1) or already violate (U < 0)."""
    prm = api.Params(sigma2_log2=5, flags=api.POLICY_KV_DESCRIPTOR if kv else 0)
    op = oracle_params(prm)
    B, m0, N, M = 2, 600, 1000, 2600
    rng = np.random.default_rng(seed)
    bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=1)
    vals = (lambda shape: synth.random_grid_keys(rng, shape)) if kv else \
        (lambda shape: synth.to_storage(rng.standard_normal(shape), "bf16"))
    K0, V0 = synth.random_grid_keys(rng, (B, m0, d)), vals((B, m0, d))
    api.update_bank(bank, dev(K0, "bf16"), dev(V0, "bf16"), 0, prm)
    torch.cuda.synchronize()
    K1, V1 = synth.random_grid_keys(rng, (B, N, d)), vals((B, N, d))
    for b in range(B):
        ob = mirror(bank, b)
        db = np.hstack([ob.K, ob.V.astype(np.float64)]) if kv else ob.K
        dc = np.hstack([K1[b], V1[b]]) if kv else K1[b]
        T = weight_q23(pair_d2(db, dc.astype(np.float64)), op).sum(axis=1)
        U = rng.uniform(-0.15, 1.15, ob.m)
        base = np.maximum(op.delta_q, np.floor((ob.rho + U * T) / 2)).astype(np.int64)
        bank.base[b, :ob.m] = torch.from_numpy(base).to(bank.base.device)
    torch.cuda.synchronize()
    return prm, op, bank, K1, V1


@pytest.mark.parametrize("budgets,decided", [((3000, 3000), (True, True)), ((1191, 1191), (False, False)),
                                             ((1195, 1191), (True, False))])
@pytest.mark.parametrize("trace", [False, True])
def test_crossing_search_first_part(budgets, decided, trace):
    """Two banks of one group, d = 128, three blocks of 600 candidates from one
    cluster: the states admitted in block 1 carry baselines from a half-full bank,
    so in block 2 all 600 cross within the first 256 ordered candidates.  A bank
    with more crossings there than the evictions it could make at any tested
    length, max(0, m + R - M), rules out every prefix past 256 (Eqs. 9-11):
    budget 3,000 (E = 0) and 1,195 (E = 596) decide the group in the first part
    (r* < 256), 1,191 (E = 600) does not (the search goes on; r* = 600 with
    600 releases); one bank of each kind in a group decides it.  The
    scenario is checked on the oracle's records, the banks against the oracle,
    and with trace outputs every record too."""
    _log(f"crossing search first part budgets={budgets} trace={trace}")
    d, N, H = 128, 600, 2
    rng = np.random.default_rng(91)
    snap = lambda x: (np.clip(np.rint(x * 64.0), -127, 127) / 64.0).astype(np.float32)
    c0 = rng.standard_normal(d)
    c0 /= np.linalg.norm(c0)
    prm = api.Params(sigma2_log2=5)
    op = oracle_params(prm)
    bank = api.Bank(H, max(budgets), d, dtype=torch.bfloat16, group_size=H,
                    budget=torch.tensor(budgets, dtype=torch.int32))
    obanks = [BankState.empty(b, d) for b in budgets]
    for t in range(3):
        K = np.stack([snap(c0 + 0.3 * rng.standard_normal((N, d))) for _ in range(H)])
        V = torch.from_numpy(rng.standard_normal((H, N, d)).astype(np.float32)).to(torch.bfloat16).float().numpy()
        out = api.UpdateOut(bank, N, trace=trace)
        api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), t, prm, out=out)
        torch.cuda.synchronize()
        new, recs = oracle_step(obanks, K, V, t, op, H)
        if t == 2:  # the scenario, on the oracle
            R = recs[0].R
            got = tuple(bool(np.count_nonzero(recs[0].heads[h].first_cross <= 256) > max(0, obanks[h].m + R - budgets[h]))
                        for h in range(H))
            assert R > 256 and got == decided, f"scenario: first part decides {got}, expected {decided}"
            assert (recs[0].r_star < 256) if any(decided) else (recs[0].r_star == 600), f"scenario: r* {recs[0].r_star}"
        if trace:
            assert_trace_equal(out, recs, H, obanks, N, ctx=f"block {t}")
        assert int(out.r_star[0]) == recs[0].r_star, f"block {t}: r*"
        for b in range(H):
            assert_bank_equal(bank, b, new[b], ctx=f"block {t}")
        obanks = new


@pytest.mark.parametrize("d,kv", [(128, False), (64, False), (64, True), (128, True)])
def test_crossing_search_spread_bounds(d, kv):
    """First crossings over every 64-candidate chunk, the partial last chunk, the
    never-crossing sentinel R + 1 and the already-violating 0 (Eqs. 8-9), with many
    distinct crossing chunks inside one workgroup of states; then the rest of the
    update, also in the [K; V] geometry (descriptor dimensions 128 and 256)."""
    _log(f"crossing search spread bounds d={d} kv={kv}")
    prm, op, bank, K1, V1 = _spread_case(d, kv, 23 + d + int(kv))
    B, N = K1.shape[0], K1.shape[1]
    obanks = [mirror(bank, b) for b in range(B)]
    out = api.UpdateOut(bank, N, trace=True)
    api.update_bank(bank, dev(K1, "bf16"), dev(V1, "bf16"), 1, prm, out=out)
    torch.cuda.synchronize()
    new, recs = oracle_step(obanks, K1, V1, 1, op, 1)
    for b, rec in enumerate(recs):  # the case exercises what it is for
        fc, R = rec.heads[0].first_cross, rec.R
        cross = (fc > 0) & (fc <= R)
        ch = np.where(cross, (fc - 1) // 64, -1)
        most = max(np.unique(ch[i:i + 128][ch[i:i + 128] >= 0]).size for i in range(0, fc.size, 128))
        assert most >= 12 and (fc == 0).any() and (fc == R + 1).any() and (ch == (R - 1) // 64).any(), \
            f"bank {b}: {most} distinct chunks per 128 states"
    assert_trace_equal(out, recs, 1, obanks, N)
    for b in range(B):
        assert_bank_equal(bank, b, new[b], kv=kv)


# ----------------------------------------------------------------------------- score entry point

def test_score_and_bank_density():
    _log("score + density")
    prm = api.Params(sigma2_log2=5)
    cfg = synth.Config(heads=3, d=128, dtype="bf16", n_cand=130, budget=260, group_size=3, **SMALL)
    bank, obanks = _run_rollout(cfg, 3, prm, trace=False)
    K = np.stack([synth.HeadStream(cfg, 0, h).keys(9, 130) for h in range(3)])
    V = np.stack([synth.HeadStream(cfg, 0, h).values(9, 130) for h in range(3)])
    sq, sf, dens = api.score(bank, dev(K, "bf16"), dev(V, "bf16"), prm, want_density=True)
    torch.cuda.synchronize()
    op = oracle_params(prm)
    for b in range(3):
        S, E, s_real = candidate_scores(obanks[b].K, obanks[b].base, K[b].astype(np.float64), op)
        assert np.array_equal(sq[b].cpu().numpy(), S)
        assert np.allclose(sf[b].cpu().numpy(), s_real, rtol=1e-6, atol=0)
        m = obanks[b].m
        assert np.array_equal(dens[b, :m].cpu().numpy(), density_from_scratch(obanks[b].K, op))
        assert np.array_equal(dens[b, :m].cpu().numpy(), obanks[b].rho)


# ----------------------------------------------------------------------------- configs 1 and 2

def _starts_full_case(name):
    cfg = synth.WORKLOADS[name]
    prm = api.Params(sigma2_log2=cfg.sigma2_log2)
    case = synth.single_update_case(cfg)
    return cfg, prm, case


@pytest.mark.parametrize("name", ["tiny", "single_layer"])
def test_workload_update_and_attention(name):
    """tiny (1 layer x 2 heads, d 64, fp32, budget 256, 64 candidates) and single_layer (1 layer x
    12 heads, d 128, bf16, N = M = 4680, 30% near-duplicates): bank built by the empty-bank rule,
    one update, then attention."""
    _log(f"workload {name}")
    cfg, prm, case = _starts_full_case(name)
    B, gs, d, dt, M, N = cfg.heads, cfg.group_size, cfg.d, cfg.dtype, cfg.budget, cfg.n_cand
    op = oracle_params(prm)
    bank = api.Bank(B, M, d, dtype=torch.bfloat16 if dt == "bf16" else torch.float32, group_size=gs)
    ob = [BankState.empty(M, d) for _ in range(B)]
    for blk, (Kn, Vn) in enumerate([("init_K", "init_V"), ("seg_K", "seg_V")]):
        K, V = case[Kn], case[Vn]
        out = api.UpdateOut(bank, K.shape[1], trace=True)
        api.update_bank(bank, dev(K, dt), dev(V, dt), blk, prm, out=out)
        torch.cuda.synchronize()
        _log(f"  block {blk}: GPU done, running oracle")
        new, recs = oracle_step(ob, K, V, blk, op, gs)
        assert_trace_equal(out, recs, gs, ob, K.shape[1], ctx=f"{name} block {blk}")
        for b in range(B):
            assert_bank_equal(bank, b, new[b], ctx=f"{name} block {blk}")
        ob = new
        _log(f"  block {blk}: r* = {recs[0].r_star}, evicted {[int(x) for x in out.n_evicted.cpu()][:4]}")
    q, wk, wv = case["q"], case["win_K"], case["win_V"]
    o = api.bank_attention(bank, dev(q, dt), dev(wk, dt), dev(wv, dt))
    torch.cuda.synchronize()
    got = host(o)
    tol = 2e-2 if dt == "bf16" else 1e-5
    worst = 0.0
    for b in range(B):
        ref = attention(q[b], ob[b].K, ob[b].V, wk[b], wv[b], 1.0 / np.sqrt(d))
        worst = max(worst, attention_error(got[b], ref))
    _log(f"  attention max row-normalised error {worst:.3e} (tol {tol})")
    assert worst <= tol


# ----------------------------------------------------------------------------- attention edge cases

@pytest.mark.parametrize("dt,d", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
def test_attention_edge_cases(dt, d):
    _log(f"attention edges {dt} {d}")
    rng = np.random.default_rng(21)
    B, M = 4, 300
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    bank = api.Bank(B, M, d, dtype=tdt, group_size=1, budget=torch.tensor([300, 0, 77, 5], dtype=torch.int32))
    occ = [300, 0, 77, 5]
    Kb = synth.to_storage(rng.standard_normal((B, M, d)), dt)
    Vb = synth.to_storage(rng.standard_normal((B, M, d)), dt)
    bank.k.copy_(dev(Kb, dt))
    bank.v.copy_(dev(Vb, dt))
    bank.occupancy.copy_(torch.tensor(occ, dtype=torch.int32))
    tol = 2e-2 if dt == "bf16" else 1e-5
    for nq, nw in [(97, 33), (1, 0), (130, 1), (64, 200)]:
        q = synth.to_storage(rng.standard_normal((B, nq, d)), dt)
        wk = synth.to_storage(rng.standard_normal((B, nw, d)), dt)
        wv = synth.to_storage(rng.standard_normal((B, nw, d)), dt)
        o = api.bank_attention(bank, dev(q, dt), dev(wk, dt) if nw else None, dev(wv, dt) if nw else None)
        torch.cuda.synchronize()
        got = host(o)
        for b in range(B):
            m = occ[b]
            if m + nw == 0:
                assert np.all(got[b] == 0)
                continue
            ref = attention(q[b], Kb[b, :m], Vb[b, :m], wk[b], wv[b], 1.0 / np.sqrt(d))
            err = attention_error(got[b], ref)
            assert err <= tol, (nq, nw, b, err)


# ----------------------------------------------------------------------------- sink + window + bank

@pytest.mark.parametrize("dt,d", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
def test_sink_attention_edge_cases(dt, d):
    """[bank; window; sink] with every segment present or absent, ragged lengths and
    occupancies, against the fp64 oracle over the concatenated keys."""
    _log(f"sink attention edges {dt} {d}")
    rng = np.random.default_rng(33)
    B, M = 4, 200
    occ = [200, 0, 77, 5]
    bank = api.Bank(B, M, d, dtype=TORCH_DT[dt], group_size=1, budget=torch.tensor([200, 0, 77, 5], dtype=torch.int32))
    Kb = synth.to_storage(rng.standard_normal((B, M, d)), dt)
    Vb = synth.to_storage(rng.standard_normal((B, M, d)), dt)
    bank.k.copy_(dev(Kb, dt))
    bank.v.copy_(dev(Vb, dt))
    bank.occupancy.copy_(torch.tensor(occ, dtype=torch.int32))
    tol = 2e-2 if dt == "bf16" else 1e-5
    for nq, nw, ns in [(70, 33, 65), (1, 0, 1), (130, 64, 0), (64, 0, 129), (5, 1, 64)]:
        q = synth.to_storage(rng.standard_normal((B, nq, d)), dt)
        seg = lambda n: synth.to_storage(rng.standard_normal((B, n, d)), dt)
        wk, wv, sk, sv = seg(nw), seg(nw), seg(ns), seg(ns)
        o = api.bank_attention_sink(bank, dev(q, dt), dev(sk, dt) if ns else None, dev(sv, dt) if ns else None,
                                    dev(wk, dt) if nw else None, dev(wv, dt) if nw else None)
        torch.cuda.synchronize()
        got = host(o)
        for b in range(B):
            m = occ[b]
            if m + nw + ns == 0:
                assert np.all(got[b] == 0)
                continue
            ref = attention(q[b], Kb[b, :m], Vb[b, :m], np.concatenate([wk[b], sk[b]]), np.concatenate([wv[b], sv[b]]),
                            1.0 / np.sqrt(d))
            err = attention_error(got[b], ref)
            assert err <= tol, (nq, nw, ns, b, err)


def test_sink_attention_without_sink_is_bank_attention():
    """n_sink = 0 is the two-segment call (the same kernel, bit for bit)."""
    _log("sink attention n_sink=0")
    cfg = synth.WORKLOADS["tiny"]
    rng = np.random.default_rng(5)
    B, M, d = 3, 150, 128
    bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=3)
    bank.k.copy_(dev(synth.to_storage(rng.standard_normal((B, M, d)), "bf16"), "bf16"))
    bank.v.copy_(dev(synth.to_storage(rng.standard_normal((B, M, d)), "bf16"), "bf16"))
    bank.occupancy.fill_(131)
    q = dev(synth.to_storage(rng.standard_normal((B, 77, d)), "bf16"), "bf16")
    wk = dev(synth.to_storage(rng.standard_normal((B, 90, d)), "bf16"), "bf16")
    wv = dev(synth.to_storage(rng.standard_normal((B, 90, d)), "bf16"), "bf16")
    a = api.bank_attention(bank, q, wk, wv)
    b2 = api.bank_attention_sink(bank, q, None, None, wk, wv)
    torch.cuda.synchronize()
    assert torch.equal(a, b2)


def test_sink_attention_deployment_shape():
    """The paper's deployment context at full size: 12 heads, d = 128, bf16, a
    1,560-token sink, a 7,800-token window and banks of up to 9,360 retained states
    (ragged occupancy), 4,680 queries; 64 sampled query rows per head against the
    fp64 oracle (clustered keys on the grid, as in the rollout workloads)."""
    _log("sink attention deployment shape")
    cfg = synth.Config(seed_id=41, name="deploy", layers=1, heads=12, d=128, dtype="bf16", n_cand=4680,
                       n_query=4680, n_window=7800, budget=9360, clusters=64, blocks=1, group_size=12,
                       sigma2_log2=6, drift=0.0)
    B, d, M = cfg.heads, cfg.d, cfg.budget
    occ = np.array([9360, 9360, 9001, 4680, 9360, 64, 9360, 9359, 1, 9360, 7777, 9360], np.int32)
    bank = api.Bank(B, M, d, dtype=torch.bfloat16, group_size=B)
    kb, vb = synth.torch_layer_block(cfg, 0, 0, M, "cuda", seed=1)
    sk, sv = synth.torch_layer_block(cfg, 0, 1, 1560, "cuda", seed=1)
    wk, wv = synth.torch_layer_block(cfg, 0, 2, 7800, "cuda", seed=1)
    q, _ = synth.torch_layer_block(cfg, 0, 3, cfg.n_query, "cuda", seed=1)
    bank.k.copy_(kb)
    bank.v.copy_(vb)
    bank.occupancy.copy_(torch.from_numpy(occ))
    o = api.bank_attention_sink(bank, q, sk, sv, wk, wv)
    torch.cuda.synchronize()
    rows = np.random.default_rng(3).choice(cfg.n_query, 64, replace=False)
    rows[:2] = [0, cfg.n_query - 1]
    for b in range(B):
        m = int(occ[b])
        ref = attention(host(q[b])[rows], host(bank.k[b, :m]), host(bank.v[b, :m]),
                        np.concatenate([host(wk[b]), host(sk[b])]), np.concatenate([host(wv[b]), host(sv[b])]),
                        1.0 / np.sqrt(d))
        err = attention_error(host(o[b])[rows], ref)
        assert err <= 2e-2, (b, m, err)
