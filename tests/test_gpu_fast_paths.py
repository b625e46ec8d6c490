"""Size- and state-dependent routes of the update and the attention against the oracle (needs an MI355X).

Each test runs the sizes where a route begins and ends; decisions and committed
banks are compared bit for bit, attention within the row-normalised error of
the path (2e-2 bf16, 1e-5 fp32).
"""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2608_27922_amd import api, synth  # noqa: E402
from gpu_util import (TORCH_DT, assert_bank_equal, assert_trace_equal, attention_error, dev, host,  # noqa: E402
                      oracle_params, oracle_step)
from oracle import BankState, attention, pair_d2, weight_q23  # noqa: E402
from test_gpu_parity import POLICY_FLAGS, SMALL, _log, _run_rollout  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    api.lib()


@pytest.mark.parametrize("policy", [""] + sorted(POLICY_FLAGS))
@pytest.mark.parametrize("dt,d,n,budgets,gs", [
    ("bf16", 128, 300, (300, 300), 2),            # budget = block: all candidates enter, no order needed
    ("bf16", 64, 300, (299, 299, 120), 1),        # budgets below the block: the first M of the order enter
    ("bf16", 128, 300, (300, 120, 300), 3),       # unequal budgets in a group: R = 120, the general search
    ("bf16", 128, 300, (300, 301, 0), 1),         # one short of a whole replacement; a bank of budget 0
    ("f32", 64, 200, (200, 150), 1),
])
def test_banks_of_at_most_one_block(policy, dt, d, n, budgets, gs):
    """Banks whose budget is at most the block are replaced whole in every update (r* = R), which the
    update uses when no trace output is requested; the others take the general search."""
    _log(f"whole replacement dt={dt} d={d} n={n} budgets={budgets} gs={gs} policy={policy}")
    cfg = synth.Config(heads=len(budgets), d=d, dtype=dt, n_cand=n, budget=max(budgets), group_size=gs, **SMALL)
    flags = POLICY_FLAGS[policy] if policy else 0
    _run_rollout(cfg, 3, api.Params(sigma2_log2=4 if d == 64 else 5, flags=flags),
                 budgets=np.array(budgets, np.int32), dup_every=2, trace=False)


@pytest.mark.parametrize("dt,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("nq,cap,m,nw,ns", [
    (1, 1200, 1200, 70, 33),      # one query, every segment with a partial last tile
    (33, 4000, 0, 65, 0),         # empty bank: all but one of the splits sized by the capacity hold no key
    (257, 900, 130, 0, 1),        # a second query block of one query; a sink of one key
    (70, 640, 640, 0, 0),
    (40, 640, 0, 0, 0),           # no key at all: zeros
])
def test_attention_key_splits(dt, d, nq, cap, m, nw, ns):
    """Few queries: the keys are split over workgroups and the partial results combined."""
    _log(f"attention splits dt={dt} d={d} nq={nq} cap={cap} m={m} nw={nw} ns={ns}")
    rng = np.random.default_rng(nq + d)
    B = 2
    bank = api.Bank(B, cap, d, dtype=TORCH_DT[dt])
    draw = lambda n: synth.to_storage(rng.standard_normal((B, n, d)).astype(np.float32), dt)
    K, V, wk, wv, sk, sv, q = (draw(n) for n in (m, m, nw, nw, ns, ns, nq))
    bank.k[:, :m] = dev(K, dt)
    bank.v[:, :m] = dev(V, dt)
    bank.k[:, m:] = float("nan")  # slots beyond the occupancy are not read
    bank.v[:, m:] = float("nan")
    bank.occupancy.fill_(m)
    opt = lambda a: dev(a, dt) if a.shape[1] else None
    out = host(api.bank_attention_sink(bank, dev(q, dt), opt(sk), opt(sv), opt(wk), opt(wv)))
    tol = 2e-2 if dt == "bf16" else 1e-5
    for b in range(B):
        if m + nw + ns == 0:
            assert not out[b].any()
            continue
        ref = attention(q[b], np.concatenate([K[b], sk[b]]), np.concatenate([V[b], sv[b]]), wk[b], wv[b], 1 / np.sqrt(d))
        assert attention_error(out[b], ref) <= tol


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("m", [0, 1, 192, 193, 384, 385, 5000])  # bf16: 1 split up to 6 tiles of 64 keys, then 2
def test_attention_splits_of_banks_below_their_capacity(dt, m):
    """The host sizes the splits by the capacity; a bank takes those that its keys fill, and the partial results
    of the others, left as the workspace held them (NaN here), are not read."""
    _log(f"attention splits below capacity dt={dt} m={m}")
    rng = np.random.default_rng(m)
    B, cap, d, nq, nw = 3, 18720, 64, 5, 0 if m else 40
    bank = api.Bank(B, cap, d, dtype=TORCH_DT[dt])
    draw = lambda n: synth.to_storage(rng.standard_normal((B, n, d)).astype(np.float32), dt)
    K, V, wk, wv, q = (draw(n) for n in (m, m, nw, nw, nq))
    bank.k.fill_(float("nan"))
    bank.v.fill_(float("nan"))
    bank.k[:, :m], bank.v[:, :m] = dev(K, dt), dev(V, dt)
    bank.occupancy.fill_(m)
    out, cb, size = torch.empty(B, nq, d, device="cuda", dtype=TORCH_DT[dt]), bank.c(), ctypes.c_size_t(0)
    lib = api.lib()
    assert lib.densitykv_attention_workspace_size(ctypes.byref(cb), nq, nw, 0, ctypes.byref(size)) == 0 and size.value
    ws = torch.full((size.value // 4,), float("nan"), device="cuda")
    qd, w = dev(q, dt), [dev(x, dt) if nw else None for x in (wk, wv)]
    assert lib.densitykv_bank_attention_ws(ctypes.byref(cb), qd.data_ptr(), nq, None, None, 0,
                                           *(None if x is None else x.data_ptr() for x in w), nw, out.data_ptr(),
                                           1 / d ** 0.5, ws.data_ptr(), size.value, api._stream()) == 0
    for b in range(B):
        ref = attention(q[b], K[b], V[b], wk[b], wv[b], 1 / np.sqrt(d))
        assert attention_error(host(out)[b], ref) <= (2e-2 if dt == "bf16" else 1e-5)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_attention_without_a_fitting_workspace(dt):
    """No workspace, one byte too little, or an address that is not a multiple of 16: the bits of the unsplit call,
    and nothing written to the workspace."""
    d, m, nq = 64, 2000, 9
    g = torch.Generator(device="cuda").manual_seed(1)
    bank = api.Bank(2, m, d, dtype=TORCH_DT[dt])
    bank.k.normal_(generator=g)
    bank.v.normal_(generator=g)
    bank.occupancy.fill_(m)
    q = torch.randn(2, nq, d, device="cuda", generator=g).to(TORCH_DT[dt])
    lib, cb, size = api.lib(), bank.c(), ctypes.c_size_t(0)
    assert lib.densitykv_attention_workspace_size(ctypes.byref(cb), nq, 0, 0, ctypes.byref(size)) == 0 and size.value
    ws = torch.full((size.value + 64,), 7, device="cuda", dtype=torch.uint8)

    def run(offset, nbytes):
        out = torch.empty_like(q)
        assert lib.densitykv_bank_attention_ws(ctypes.byref(cb), q.data_ptr(), nq, None, None, 0, None, None, 0,
                                               out.data_ptr(), 1 / d ** 0.5,
                                               None if offset is None else ws.data_ptr() + offset, nbytes,
                                               api._stream()) == 0
        return out

    ref = run(None, 0)
    for offset, nbytes in ((0, size.value - 1), (4, size.value), (8, size.value)):
        assert torch.equal(run(offset, nbytes), ref)
        assert bool((ws == 7).all())
    split = run(16, size.value)
    assert torch.equal(run(16, size.value), split)  # equal calls, equal bits
    assert attention_error(host(split), host(ref)) <= (2e-2 if dt == "bf16" else 1e-5)
    assert not bool((ws == 7).all())


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_attention_key_splits_of_infinite_scores(dt):
    """A split whose scores are all -inf weighs nothing beside finite ones; a row of such scores alone is
    NaN, as softmax gives; a NaN key makes its row NaN in whatever split it lies."""
    d, m = 64, 2000
    bank = api.Bank(1, m, d, dtype=TORCH_DT[dt])
    bank.k.zero_()
    bank.v.fill_(1.0)
    bank.v[:, 1500:] = 3.0
    bank.occupancy.fill_(m)
    bank.k[:, :1500, 0] = -float("inf")
    q = torch.zeros(1, 3, d, device="cuda", dtype=TORCH_DT[dt])
    q[:, 0, 0] = 1.0
    q[:, 1, 1] = 1.0
    bank.k[:, 1500:, 2] = 1.0
    q[:, 2, 0] = 1.0
    out = api.bank_attention(bank, q, None, None).float()
    assert torch.allclose(out[0, 0], torch.full_like(out[0, 0], 3.0), rtol=1e-2)
    assert out[0, 1].isnan().all()       # 0 * -inf
    bank.k[:, 1500:, 0] = -float("inf")
    assert api.bank_attention(bank, q, None, None).float()[0, 0].isnan().all()
    bank.k[:, :, 0] = 0.0
    bank.k[:, 3, 5] = float("nan")
    assert api.bank_attention(bank, q, None, None).isnan().all()


@pytest.mark.parametrize("d,kv", [(64, False), (128, False), (128, True)])
@pytest.mark.parametrize("m", [1, 63, 128, 129, 896, 897, 1793])  # blocks of 128 (256) held items, runs of 768 streamed ones
def test_densities_at_run_edges(d, kv, m):
    """From-scratch densities as a symmetric Gram against direct sums over pairs: every pair once, whatever
    number of held blocks and streamed runs the list has (whole numbers: keys on the grid, t exact)."""
    _log(f"densities d={d} kv={kv} m={m}")
    g = torch.Generator(device="cuda").manual_seed(7 * m + d)
    prm = api.Params(sigma2_log2=5, flags=api.POLICY_KV_DESCRIPTOR if kv else 0)
    bank = api.Bank(2, 1800, d)
    rows = (torch.randint(-40, 41, (2, m, 2, d), generator=g, device="cuda") / 64.0).to(torch.bfloat16)
    bank.k[:, :m], bank.v[:, :m] = rows[:, :, 0], rows[:, :, 1]
    desc = rows.flatten(2) if kv else rows[:, :, 0]
    bank.knorm[:, :m] = desc.float().square().sum(-1)
    bank.base.fill_(1 << 23)
    bank.occupancy.fill_(m)
    seg = torch.zeros(2, 1, d, device="cuda", dtype=torch.bfloat16)
    dens = api.score(bank, seg, seg, prm, want_density=True)[2]
    for b in range(2):
        x = desc[b].double().cpu()
        d2 = (x * x).sum(-1)[:, None] + (x * x).sum(-1)[None] - 2.0 * x @ x.T  # exact on the grid
        t = (1.0 + d2.float() / 32.0)  # exact in binary32
        w = (1.0 / (t * t).double()).float()  # correctly rounded reciprocal of the rounded square
        W = torch.round(w.double() * 2.0 ** 23).long()
        W.fill_diagonal_(0)
        assert torch.equal(dens[b, :m].cpu(), W.sum(-1)), f"bank {b}"


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 256, 511, 512, 513, 1025, 2048, 2049])
@pytest.mark.parametrize("source_order", [False, True])
def test_order_at_sort_edges(n, source_order):
    """The candidates' order and its committed update at the sizes where the sort changes its route or its
    number of stages; the first block meets empty banks, so all its scores tie."""
    _log(f"order n={n} source_order={source_order}")
    cfg = synth.Config(heads=2, d=64, dtype="bf16", n_cand=n, budget=max(600, n), group_size=2, **SMALL)
    flags = api.POLICY_SOURCE_ORDER if source_order else 0
    _run_rollout(cfg, 2, api.Params(sigma2_log2=4, flags=flags), dup_every=1)


@pytest.mark.parametrize("kv,B,gs,n,budgets", [
    (False, 40, 4, 8191, (300, 700, 300, 300)),   # unequal budgets: the general search up to R = 300
    (False, 40, 2, 8191, (300, 300)),             # replaced whole: the order matters across position 300 only
    (False, 320, 2, 1000, (1400, 1500)),          # growing, then at its budget: every order position may matter
    (True, 320, 2, 1000, (1400, 1500)),
])
def test_approximate_scores_give_the_exact_order(kv, B, gs, n, budgets):
    """Calls of at least 1e10 pairs (by capacity) that ask for no scores may order their candidates by approximate
    ones; asking for them takes the exact route.  Same decisions and banks, with duplicated and nearly
    duplicated candidates so that many neighbours in the order are closer than the error bound."""
    _log(f"approximate scores kv={kv} B={B} n={n} budgets={budgets}")
    d, cap = 64, 32767
    assert B * cap * n >= 1e10
    prm = api.Params(sigma2_log2=5, flags=api.POLICY_KV_DESCRIPTOR if kv else 0)
    bud = torch.tensor([budgets[b % gs] for b in range(B)], dtype=torch.int32)
    banks = [api.Bank(B, cap, d, group_size=gs, budget=bud) for _ in range(2)]
    g = torch.Generator(device="cuda").manual_seed(n + B)
    for t in range(4):
        centres = torch.randn(B, 16, d, generator=g, device="cuda") / d ** 0.5
        pick = torch.randint(0, 16, (B, n, 1), generator=g, device="cuda").expand(B, n, d)
        k = torch.gather(centres, 1, pick) + 0.1 * torch.randn(B, n, d, generator=g, device="cuda")
        k = (torch.clamp(torch.round(k * 64), -127, 127) / 64)
        k[:, 1::2] = k[:, 0::2][:, : n // 2]                     # exact ties ...
        k[:, 3::4, 0] = torch.clamp(k[:, 3::4, 0] + 1 / 64, -1.9, 1.9)  # ... half of them moved by one grid step
        k = (torch.round(k * 64) / 64).to(torch.bfloat16).contiguous()
        v = (torch.round(torch.randn(B, n, d, generator=g, device="cuda") * 16) / 64).to(torch.bfloat16)
        outs = [api.UpdateOut(banks[i], n, trace=i == 1) for i in range(2)]
        for i in range(2):
            api.update_bank(banks[i], k, v, t, prm, out=outs[i])
        assert torch.equal(outs[0].r_star, outs[1].r_star), f"block {t}"
        for name in ("admitted", "evicted"):
            assert torch.equal(getattr(outs[0], name), getattr(outs[1], name)), f"block {t} {name}"
        assert torch.equal(banks[0].occupancy, banks[1].occupancy)
        m = int(banks[0].occupancy.max())
        live = torch.arange(m, device="cuda")[None] < banks[0].occupancy[:, None]
        for name in ("k", "v", "knorm", "rho", "base", "prov"):
            x, y = (getattr(bk, name)[:, :m][live] for bk in banks)
            assert torch.equal(x, y), f"block {t} {name}"


@pytest.mark.parametrize("d,kv", [(64, False), (128, False), (64, True)])
def test_approximate_scores_read_no_stale_scale(d, kv):
    """Approximate scores (calls of at least 1e10 pairs by capacity, banks replaced whole by a larger block) where
    the banks end inside a tile of 32 states and what lies behind them, in the bank and in the workspace, is NaN."""
    _log(f"stale workspace d={d} kv={kv}")
    B, cap, n, check = 40, 32767, 8191, (0, 19, 39)
    assert B * cap * n >= 1e10
    rng = np.random.default_rng(d)
    prm = api.Params(sigma2_log2=5, flags=api.POLICY_KV_DESCRIPTOR if kv else 0)
    bank = api.Bank(B, cap, d, budget=torch.full((B,), 300, dtype=torch.int32))
    for x in (bank.k, bank.v, bank.knorm):
        x.fill_(float("nan"))
    obanks = [BankState.empty(300, d) for _ in check]
    for t in range(2):
        K, V = _spread_rows(rng, B, n, d), _spread_rows(rng, B, n, d)
        ws = api.alloc_workspace(bank, n, prm.flags).fill_(255)
        api.update_bank(bank, dev(K, "bf16"), dev(V, "bf16"), t, prm, workspace=ws, out=api.UpdateOut(bank, n))
        obanks, _ = oracle_step(obanks, K[list(check)], V[list(check)], t, oracle_params(prm), 1)
        for b, ob in zip(check, obanks):
            assert_bank_equal(bank, b, ob, ctx=f"block {t}", kv=kv)


def _spread_rows(rng, B, n, d):
    """[B, n, d] float32 rows on the key grid whose distances to one another, and so their scores, vary widely."""
    c = rng.standard_normal((B, 12, d)) / 3.0
    x = c[np.arange(B)[:, None], rng.integers(0, 12, (B, n))] * rng.uniform(0.2, 1.0, (B, n, 1))
    x += rng.uniform(0.05, 0.4, (B, n, 1)) * rng.standard_normal((B, n, d))
    return (np.clip(np.rint(x * 64), -127, 127) / 64).astype(np.float32)


def _near_banks(B, cap, m, d, prm, candidates, reach, seed):
    """Banks of m states that all stand near their bound (next to their densities), so that calls may approximate
    their scores; the nearest takes `reach` candidates of mean weight.  Returns the bank and the oracle's."""
    rng = np.random.default_rng(seed)
    bank = api.Bank(B, cap, d, group_size=2)
    K, V = _spread_rows(rng, B, m, d), _spread_rows(rng, B, m, d)
    obanks, op = [], oracle_params(prm)
    for b in range(B):
        k = K[b].astype(np.float64)
        w = weight_q23(pair_d2(k, candidates[b, ::16].astype(np.float64)), op).mean(1)  # mean weight to the block
        thr = (w * reach * rng.uniform(1.0, 2.0, m)).astype(np.int64) // 2 * 2 + 2
        rho = np.full(m, 1 << 38, np.int64)
        obanks.append(BankState(budget=cap, K=k, V=V[b], rho=rho, base=(rho + thr) // 2,
                                prov=np.arange(m, dtype=np.int64)))
        for name in ("rho", "base", "prov"):
            getattr(bank, name)[b, :m] = torch.from_numpy(getattr(obanks[b], name)).cuda()
    bank.k[:, :m], bank.v[:, :m] = dev(K, "bf16"), dev(V, "bf16")
    bank.knorm[:, :m] = torch.from_numpy((K.astype(np.float64) ** 2).sum(-1).astype(np.float32)).cuda()
    bank.occupancy.fill_(m)
    return bank, obanks


@pytest.mark.parametrize("reach", [20, 900])  # the first part of the crossing search decides; it leaves the groups open
@pytest.mark.parametrize("rows", ["spread", "triples", "hidden run", "tied"])
def test_approximate_order_against_the_oracle(rows, reach):
    """The order from approximate scores at m > 0: distinct scores, short clusters, one cluster of 8,063 candidates
    that the 128 sampled ones do not show (the list is sorted), all scores tied (the exact scores at once)."""
    _log(f"approximate order rows={rows} reach={reach}")
    B, cap, m, d, n = 40, 32767, 1001, 64, 8191
    assert B * cap * n >= 1e10
    prm = api.Params(sigma2_log2=5)
    rng = np.random.default_rng(reach)
    k, v = _spread_rows(rng, B, n, d), _spread_rows(rng, B, n, d)
    if rows == "triples":
        k[:, 1::3], k[:, 2::3] = k[:, 0::3][:, : k[:, 1::3].shape[1]], k[:, 0::3][:, : k[:, 2::3].shape[1]]
    elif rows != "spread":
        keep = np.arange(128) * n // 128 if rows == "hidden run" else np.zeros(0, int)
        same = np.repeat(k[:, 5:6], n, 1)
        same[:, keep] = k[:, keep]
        k = same
    bank, obanks = _near_banks(B, cap, m, d, prm, k, reach, 3)
    out = api.UpdateOut(bank, n)
    api.update_bank(bank, dev(k, "bf16"), dev(v, "bf16"), 1, prm, out=out)
    for i in (0, 7, B // 2 - 1):  # groups
        b = [2 * i, 2 * i + 1]
        new, (rec,) = oracle_step([obanks[x] for x in b], k[b], v[b], 1, oracle_params(prm), 2)
        assert (rec.r_star < 256) == (reach == 20) and int(out.r_star[i]) == rec.r_star, f"group {i}"
        for j in range(2):
            got = out.admitted[b[j]].cpu().numpy()
            assert np.array_equal(got[got >= 0], rec.heads[j].admitted), f"bank {b[j]}: admitted"
            assert_bank_equal(bank, b[j], new[j])


def test_first_crossings_within_short_prefixes():
    """First crossings wanted, more than 256 candidates, R <= 256 (a small bank in each group) and banks whose
    crossings rule r* out at once: states of workgroups that start after that was known (2,000 workgroups of 128
    states, more than the chip holds at a time) get theirs as well."""
    _log("first crossings of short prefixes")
    G, m, d, n, R = 12, 20001, 64, 300, 200
    rng = np.random.default_rng(5)
    grid = lambda *s: (np.clip(np.rint(rng.standard_normal(s) * 8), -127, 127) / 64).astype(np.float32)
    prm = api.Params(sigma2_log2=5)
    budgets = np.tile(np.array([R, m + 300], np.int32), G)  # E = max(0, m + R - M) = 0: one crossing decides a bank
    bank = api.Bank(2 * G, m + 300, d, group_size=2, budget=torch.from_numpy(budgets))
    base = rng.integers(1 << 30, 1 << 31, (G, m))
    rho = 2 * base - rng.integers(1, 220 << 23, (G, m))      # spread over the first 256 candidates and past them
    prov = np.broadcast_to(np.arange(m, dtype=np.int64), (G, m))
    K, V = grid(G, m, d), grid(G, m, d)
    obanks = [BankState.empty(R, d) for _ in range(2 * G)]
    for i in range(G):
        obanks[2 * i + 1] = BankState(budget=m + 300, K=K[i].astype(np.float64), V=V[i], rho=rho[i], base=base[i],
                                      prov=prov[i])
    bank.k[1::2, :m], bank.v[1::2, :m] = dev(K, "bf16"), dev(V, "bf16")
    bank.knorm[1::2, :m] = torch.from_numpy((K.astype(np.float64) ** 2).sum(-1).astype(np.float32)).cuda()
    for name, x in (("rho", rho), ("base", base), ("prov", prov)):
        getattr(bank, name)[1::2, :m] = torch.from_numpy(x.copy()).cuda()
    bank.occupancy[1::2] = m
    sk, sv = grid(2 * G, n, d), grid(2 * G, n, d)
    out = api.UpdateOut(bank, n, trace=True)
    api.update_bank(bank, dev(sk, "bf16"), dev(sv, "bf16"), 1, prm, out=out)
    new, recs = oracle_step(obanks, sk, sv, 1, oracle_params(prm), 2)
    first = np.concatenate([r.heads[1].first_cross for r in recs])
    assert len(np.unique((first[first <= R] + 63) // 64)) == 4  # crossings in every chunk of the prefix
    assert_trace_equal(out, recs, 2, obanks, n)
    for b in range(2 * G):
        assert_bank_equal(bank, b, new[b])
