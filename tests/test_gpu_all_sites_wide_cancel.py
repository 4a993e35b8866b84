"""Cancelling sums of the all-sites calls with sliced keys wider than 64
columns: the routed states and the value gradients as exact as weights in fp32
make them.

Sources whose weighted values cancel to 2^-18 of their terms leave nothing of
the bf16 rounding of H, so what shows is the error of the weights alone: fp32
softmax weights of a few sources with scores around 1 carry about ten
roundings (score, norm, exponential, sum, quotient), and the sum over the
sources one per term at most.  Bar per entry: (16 + S) 2^-24 sum |alpha v| +
2^-8 |H|, the latter bf16's half-ulp.  Weights in two bf16 terms (2^-18 each
at most) miss it nearly threefold at 8 sources; what is measured is 0.2 of it.
The value gradient sums weights times upstream rows over the sites, T terms,
and is held to the same bar.
"""
import numpy as np
import pytest

import oracle
import paper_2607_09694_amd as lr
from paper_2607_09694_amd.inputs import SLICED, bf16_bits_from_f32, f32_from_bf16_bits
from test_gpu_all_sites_bwd import dev, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 2.0 ** -24


def bf16(x):
    return f32_from_bf16_bits(bf16_bits_from_f32(np.asarray(x, dtype=np.float32))).astype(np.float64)


def weights(V, Q, first, r):
    """fp64 weights [T, S, N], zero past each site's prefix."""
    T, (S, N, _) = Q.shape[0], V.shape
    a = np.zeros((T, S, N))
    for j in range(T):
        a[j, :first + j] = oracle.route_weights(V[:first + j], None, Q[j].astype(np.float64), SLICED,
                                                r=r).T
    return a


# (S, T, first, N, d, r): one to four site tiles
CASES = [(8, 7, 2, 40, 328, 72), (12, 11, 2, 9, 1000, 256), (33, 32, 2, 5, 520, 128),
         (49, 48, 2, 3, 328, 72), (64, 64, 1, 3, 200, 72)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S{}-T{}-f{}-N{}-d{}-r{}".format(*c))
def test_cancelling_states_keep_fp32_weights(dev, case):  # noqa: F811
    S, T, first, N, d, r = case
    rng = np.random.default_rng(S + N + d)
    V = bf16(rng.standard_normal((S, N, d)))
    # scores of about 1: |kbar| = sqrt(r)
    Q = (rng.standard_normal((T, r)) / np.sqrt(r)).astype(np.float32)
    a = weights(bf16_bits_from_f32(V.astype(np.float32)), Q, first, r)
    # the last two sources cancel the last site's sum in the value columns
    for i in (S - 2, S - 1):
        rest = (a[T - 1, :, :, None] * V)[:i].sum(0)
        V[i, :, :d - r] = bf16(-rest[:, :d - r] / a[T - 1, i][:, None])[:, :d - r]
    Vb = bf16_bits_from_f32(V.astype(np.float32))
    ref = np.einsum("jin,inc->jnc", a, V)[..., :d - r]
    mag = np.einsum("jin,inc->jnc", a, np.abs(V))[..., :d - r]
    assert np.median(np.abs(ref[-1]) / mag[-1]) < 2.0 ** -16
    H, _ = lr.route_all_fwd(to_dev(Vb, dev), None, to_dev(Q, dev), SLICED, first)
    torch.cuda.synchronize()
    err = np.abs(to_host(H)[..., :d - r].astype(np.float64) - ref)
    # sites whose sums do not cancel are bound by the bf16 rounding of H
    worst = (err / ((16 + S) * U * mag + 2.0 ** -8 * np.abs(ref))).max(axis=(1, 2))
    assert worst.max() <= 1.0, f"error / bar by site: {worst}"


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S{}-T{}-f{}-N{}-d{}-r{}".format(*c))
@pytest.mark.parametrize("accumulate", [False, True], ids=["write", "add"])
def test_cancelling_value_gradients_keep_fp32_weights(dev, case, accumulate):  # noqa: F811
    """The last two sites' upstream rows cancel source 0's sum over the sites."""
    S, T, first, N, d, r = case
    rng = np.random.default_rng(S * N + d)
    Vb = bf16_bits_from_f32(rng.standard_normal((S, N, d)).astype(np.float32))
    Q = (rng.standard_normal((T, r)) / np.sqrt(r)).astype(np.float32)
    a = weights(Vb, Q, first, r)
    dH = bf16(rng.standard_normal((T, N, d)))
    for j in (T - 2, T - 1):
        dH[j] = bf16(-(a[:, 0, :, None] * dH)[:j].sum(0) / a[j, 0][:, None])
    ref = np.einsum("jin,jnc->inc", a, dH)[..., :d - r]
    mag = np.einsum("jin,jnc->inc", a, np.abs(dH))[..., :d - r]
    assert np.median(np.abs(ref[0]) / mag[0]) < 2.0 ** -16
    dHd = to_dev(bf16_bits_from_f32(dH.astype(np.float32)), dev)
    V, Qd = to_dev(Vb, dev), to_dev(Q, dev)
    out = (torch.zeros_like(V), None, torch.zeros_like(Qd)) if accumulate else None
    dV, _, _ = lr.route_all_bwd(V, None, Qd, dHd, SLICED, first, out=out, accumulate=accumulate)
    torch.cuda.synchronize()
    err = np.abs(to_host(dV)[..., :d - r].astype(np.float64) - ref)
    worst = (err / ((16 + T) * U * mag + 2.0 ** -8 * np.abs(ref))).max(axis=(1, 2))
    assert worst.max() <= 1.0, f"error / bar by source: {worst}"


def dq64(V, Q, dH, first, r, eps=1e-6):
    """dQ [T, r] in fp64 by torch, one site at a time."""
    X = V.double().transpose(0, 1).contiguous()          # [N, S, d]
    k = X[..., X.shape[2] - r:]
    kb = k / (k.square().mean(-1, keepdim=True) + eps).sqrt()
    out = []
    for j in range(Q.shape[0]):
        x, b = X[:, :first + j], kb[:, :first + j]
        a = torch.softmax((b * Q[j].double()).sum(-1), dim=1)
        g = (x * dH[j].double()[:, None]).sum(-1)
        ds = a * (g - (a * g).sum(1, keepdim=True))
        out.append((ds[..., None] * b).sum((0, 1)))
    return torch.stack(out)


@pytest.mark.parametrize("S,N,d,r", [(64, 1500, 128, 72), (49, 2048, 256, 128)])
def test_dq_is_no_further_off_than_site_by_site(dev, S, N, d, r):  # noqa: F811
    """dQ of the one pass against the single-site calls' own distance from 64
    bits: the same fp32 operations, the sum over sources and tokens split
    differently (at these sizes 0.9 of their distance; with one chain of
    additions over a token's sources and fp32 sums of the shares 1.05)."""
    gen = torch.Generator().manual_seed(S + N)
    T, first = S - 1, 2
    scale = torch.exp2(torch.rand((S, 1, 1), generator=gen) * 3.0 - 1.5)
    V = (torch.randn((S, N, d), generator=gen) * scale).to(torch.bfloat16).to(dev)
    Q = (torch.randn((T, r), generator=gen) * 1.5 * r ** -0.5).to(dev)
    dH = torch.randn((T, N, d), generator=gen).to(torch.bfloat16).to(dev)
    ref = dq64(V, Q, dH, first, r)
    _, _, dQ = lr.route_all_bwd(V, None, Q, dH, SLICED, first)
    sites = torch.stack([lr.route_bwd(V[:first + j], None, Q[j], dH[j], SLICED)[2] for j in range(T)])
    far, far_sites = (float((x.double() - ref).norm() / ref.norm()) for x in (dQ, sites))
    assert far <= far_sites
