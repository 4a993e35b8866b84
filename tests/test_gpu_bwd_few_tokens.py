"""GPU parity of the single-site backward on both sides of its rules for few
tokens: up to 512 a workgroup splits each token's sources over its four waves
(two sources to more than one batch per wave, sources that don't divide by the
waves, ragged rows), above that one token per wave takes them alone, and from
there the tokens per wave double as the grid fills the chip.
"""
import pytest

import oracle
import paper_2607_09694_amd as lr
from paper_2607_09694_amd.inputs import FULL, PROJECTED, SLICED, make_host_problem
from test_gpu_parity import _id, check_dq, check_key_grad, check_value_grad, dev, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (mode, dtype, S, N, d, r)
CASES = [
    (PROJECTED, "bf16", 2, 512, 64, 8),
    (PROJECTED, "bf16", 2, 513, 64, 8),     # the first size past the split
    (SLICED, "bf16", 5, 512, 200, 24),
    (SLICED, "bf16", 5, 513, 200, 24),
    (PROJECTED, "f32", 37, 511, 100, 12),   # ten sources a wave, the last one seven
    (SLICED, "f32", 6, 1, 1028, 20),        # one token
    (PROJECTED, "bf16", 65, 40, 1000, 5),   # scalar key path, more than 64 sources
    (PROJECTED, "bf16", 3, 2049, 64, 16),   # past one token per wave
    (SLICED, "bf16", 3, 4097, 72, 8),       # past two
    (FULL, "f32", 3, 4097, 40, 40),
]

# Both sides of the least sources of a split: 9 (waves of 3, 3, 3 and none) and
# 10 (3, 3, 3, 1) beside 8.
CASES += [
    (PROJECTED, "bf16", 8, 512, 64, 8),
    (PROJECTED, "bf16", 9, 512, 64, 8),
    (SLICED, "bf16", 10, 512, 200, 24),
    (PROJECTED, "f32", 9, 511, 100, 12),
    (SLICED, "f32", 13, 1, 1028, 20),
]


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_backward_of_few_tokens_matches_oracle(dev, case):  # noqa: F811
    mode, dtype, S, N, d, r = case
    p = make_host_problem(mode, S, N, d, r, dtype=dtype, seed=S * 1000 + N + 1, with_dH=True)
    dV, dK, dq = lr.route_bwd(to_dev(p.V, dev), to_dev(p.K, dev), to_dev(p.q, dev),
                              to_dev(p.dH, dev), mode)
    torch.cuda.synchronize()
    dV_ref, dK_ref, dq_ref = oracle.route_bwd(p.V, p.K, p.q, p.dH, mode, r=p.r)
    check_value_grad(mode, dtype, to_host(dV), dV_ref, p.r)
    if mode == PROJECTED:
        check_key_grad("dK", dtype, to_host(dK), dK_ref)
    check_dq("dq", to_host(dq), dq_ref, tol=1e-5 if dtype == "f32" else 1e-4)
