"""GPU parity of the single-site forward on both sides of its rule for one or
two tokens per wave (past 2048 tokens, where a workgroup no longer splits one
token, and past 4352): odd and even numbers of sources (two a batch), ragged
rows and token groups, narrow and wide rows, scalar rows, both storages.
"""
import pytest

import oracle
import paper_2607_09694_amd as lr
from paper_2607_09694_amd.inputs import PROJECTED, SLICED, make_host_problem
from test_gpu_parity import _id, check_values, dev, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (mode, dtype, S, N, d, r)
CASES = [
    (PROJECTED, "bf16", 2, 2049, 64, 8),
    (SLICED, "bf16", 5, 4352, 200, 24),
    (SLICED, "bf16", 5, 4353, 200, 24),
    (PROJECTED, "bf16", 1, 2051, 520, 16),
    (PROJECTED, "bf16", 3, 2050, 2000, 16),   # four chunks a row
    (SLICED, "f32", 4, 2050, 1000, 20),
    (PROJECTED, "bf16", 7, 3001, 101, 5),     # scalar rows
    (SLICED, "f32", 65, 2049, 72, 8),
]


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_forward_of_few_thousand_tokens_matches_oracle(dev, case):  # noqa: F811
    mode, dtype, S, N, d, r = case
    p = make_host_problem(mode, S, N, d, r, dtype=dtype, seed=S * 1000 + N)
    H = lr.route_fwd(to_dev(p.V, dev), to_dev(p.K, dev), to_dev(p.q, dev), mode)
    torch.cuda.synchronize()
    check_values("H", dtype, to_host(H), oracle.route_fwd(p.V, p.K, p.q, mode, r=p.r))
