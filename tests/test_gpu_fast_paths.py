"""Size- and state-dependent routes of the update and the attention against the oracle (needs an MI355X).

Each test runs the sizes where a route begins and ends; decisions and committed
banks are compared bit for bit, attention within the row-normalised error of
the path (2e-2 bf16, 1e-5 fp32).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2608_27922_amd import api, synth  # noqa: E402
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
