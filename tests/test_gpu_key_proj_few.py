"""GPU parity of the key producer on both sides of its choice of tiles: the
few-token tiles (16, 32 or 64 tokens by 16 columns, 64 by 64, a quarter of k
per wave, ragged in every direction) and the 256 x 256 tiles with ragged rows,
columns and k stages above that line.
"""
import pytest

import oracle
import paper_2607_09694_amd as lr
from test_gpu_key_proj import bits_to_dev, check_projection, dev, operands, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (N, m, d, r)
CASES = [
    (15, 8, 24, 8),         # three waves without k, one token tile
    (17, 136, 50, 6),       # two row tiles, ragged columns split inside a vector
    (33, 264, 104, 12),     # four row tiles, a k range that ends inside a step
    (65, 1000, 296, 16),    # a second token tile of one row
    (500, 200, 1032, 20),   # 64 x 64 tiles, ragged in both
    (2049, 72, 1040, 12),   # 256 x 256 tiles: ragged rows, columns and k stage
    (2305, 128, 960, 6),    # d + r not a multiple of 8, one row in the last tile
    (4097, 40, 520, 24),
]

# Both sides of the tiles up to which the few-token form is taken, by width and
# sum: narrow outputs (63 tiles and 192), wide ones (256 and 512).
CASES += [
    (4032, 64, 48, 16), (4033, 64, 48, 16),
    (12288, 512, 40, 20), (12289, 512, 40, 20),
    (1024, 72, 1000, 24), (1025, 72, 1000, 24),
    (2048, 512, 1000, 24), (2049, 512, 1000, 24),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N{}-m{}-d{}-r{}".format(*c))
def test_key_projection_tiles_match_oracle(dev, case):  # noqa: F811
    N, m, d, r = case
    Ab, Wb = operands(N, m, d + r, seed=N + m + d + r)
    guard = 7.0
    O = torch.full((N + 1, d), guard, dtype=torch.bfloat16, device=dev)
    K = torch.full((N + 1, r), guard, dtype=torch.bfloat16, device=dev)
    lr.key_proj_fwd(bits_to_dev(Ab, dev), bits_to_dev(Wb, dev), d, out=(O, K))
    torch.cuda.synchronize()
    Or, Kr = oracle.key_projection(Ab, Wb, d)
    check_projection("O", to_host(O[:N]), Or, Ab, Wb[:d])
    check_projection("K", to_host(K[:N]), Kr, Ab, Wb[d:])
    assert bool((O[N] == guard).all()) and bool((K[N] == guard).all())
