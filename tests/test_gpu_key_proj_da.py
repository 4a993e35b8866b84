"""GPU parity of the key producer's backward where dA takes the 256 x 256 tiles
of the forward: 256 or more tiles, d a multiple of 64, the token sum split (so
that the workspace has room for the transposed W).  The stages of its reduction
come from two tensors: values only, one ragged stage of keys, a full stage and
a ragged one; ragged rows and columns; and one case beside the line each for
the tiles' fill and for d.  Bars as in the backward's own test.
"""
import pytest

import oracle
import paper_2607_09694_amd as lr
from paper_2607_09694_amd.inputs import bf16_tensor_to_bits, f32_from_bf16_bits
from parity import check_sum_by_terms
from test_gpu_key_proj_bwd import check_dA, dev, host_operands, magnitudes, splits, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (N, m, d, r)
CASES = [
    (2040, 8200, 64, 0),    # 256 tiles: values only, ragged rows and columns
    (1793, 8224, 64, 8),    # one row in the last row tile, a ragged stage of keys
    (2048, 8192, 128, 72),  # a full and a ragged stage of keys
    (2100, 8192, 64, 8),    # 288 tiles, rounds filled to 0.56: the backward's own tiles
    (2040, 8200, 72, 8),    # d not a multiple of 64: likewise
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N{}-m{}-d{}-r{}".format(*c))
def test_da_tiles_match_oracle(dev, case):  # noqa: F811
    N, m, d, r = case
    A, W, dO, dK = host_operands(N, m, d, r, seed=N + m + d + r)
    out = torch.full((N + 1, m), 7.0, dtype=torch.bfloat16, device=dev)
    dW = torch.empty((d + r, m), dtype=torch.float32, device=dev)
    lr.key_proj_bwd(to_dev(A, dev), to_dev(W, dev), to_dev(dO, dev), to_dev(dK, dev),
                    out=(out[:N], dW))
    torch.cuda.synchronize()
    refA, refW = oracle.key_projection_bwd(A, W, dO, dK)
    tA, tW = oracle.key_projection_bwd(*magnitudes(A, W, dO, dK))
    check_dA(f32_from_bf16_bits(bf16_tensor_to_bits(out[:N])), refA, tA, d + r)
    check_sum_by_terms("dW", dW.cpu().numpy(), refW, tW, N + splits(N, m, d + r), 0.0)
    assert bool((out[N] == 7.0).all())
