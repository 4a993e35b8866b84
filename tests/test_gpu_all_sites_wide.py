"""GPU parity of the all-sites calls with full-rank keys and with sliced keys wider than 64 columns
(bf16 storage), forward and backward, against the fp64 oracle: one to four
site tiles and source tiles, keys that end inside a 32-column step or start
inside one, ragged slabs, sources that no site reads, one token and more
tokens than dQ shares, accumulation, bitwise reruns, and non-finite values
confined to the sites that read them.
"""
import numpy as np
import pytest

import oracle
import paper_2607_09694_amd as lr
from paper_2607_09694_amd.inputs import FULL, SLICED, bf16_bits_from_f32, f32_from_bf16_bits, \
    make_host_problem
from parity import check_bf16_grown, check_bf16_key_grad, check_bf16_value, check_dq, check_f32
from test_gpu_all_sites_bwd import _queries, _upstream, dev, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (S, T, first, N, d, r)
CASES = [
    (9, 8, 2, 13, 256, 72),       # one tile; the key starts inside a 32-column step
    (33, 32, 2, 5, 200, 128),     # two site tiles, three source tiles, ragged slab
    (49, 48, 2, 7, 1024, 256),    # the paper's model, r = 256
    (64, 64, 1, 3, 520, 256),     # every limit
    (20, 6, 3, 9, 128, 128),      # the whole row; sources 8..19 read by no site
    (17, 1, 17, 1, 136, 80),      # one site, one token, one source past a tile
    (5, 4, 2, 1100, 96, 96),      # fewer than 128 columns, several tokens per share
]


def _run(dev, case, seed, accumulate=False):
    S, T, first, N, d, r = case
    p = make_host_problem(SLICED, S, N, d, r, dtype="bf16", seed=seed)
    Q, dH = _queries(T, r, seed + 1), _upstream(T, N, d, seed + 2)
    V, Qd, dHd = to_dev(p.V, dev), to_dev(Q, dev), to_dev(dH, dev)
    return p, Q, dH, V, Qd, dHd


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S{}-T{}-f{}-N{}-d{}-r{}".format(*c))
@pytest.mark.parametrize("accumulate", [False, True], ids=["write", "add"])
def test_wide_keys_match_oracle(dev, case, accumulate):  # noqa: F811
    S, T, first, N, d, r = case
    p, Q, dH, V, Qd, dHd = _run(dev, case, seed=S + T + N)
    Q64 = Q.astype(np.float64)
    rV, _, rQ = oracle.route_all_bwd(p.V, None, Q64, dH, SLICED, first, r=r)
    out = None
    if accumulate:
        rng = np.random.default_rng(5)
        dV0 = bf16_bits_from_f32(rng.standard_normal((S, N, d)).astype(np.float32))
        dQ0 = rng.standard_normal((T, r)).astype(np.float32)
        out = (to_dev(dV0, dev), None, to_dev(dQ0, dev))
        rV, rQ = rV + f32_from_bf16_bits(dV0), rQ + dQ0
    dV, dK, dQ = lr.route_all_bwd(V, None, Qd, dHd, SLICED, first, out=out, accumulate=accumulate)
    H, ne = lr.route_all_fwd(V, None, Qd, SLICED, first)
    torch.cuda.synchronize()
    Hr, NEr = oracle.route_all_fwd(p.V, None, Q64, SLICED, first, r=r)
    check_bf16_value("H", to_host(H), Hr)
    check_f32("neff", to_host(ne), NEr)
    assert dK is None
    gV = to_host(dV)
    check_bf16_grown("dV", gV[..., :d - r], rV[..., :d - r])
    check_bf16_key_grad("dV key columns", gV[..., d - r:], rV[..., d - r:])
    if first > 1 or T > 1:
        check_dq("dQ", to_host(dQ), rQ)
    if not accumulate and first + T - 1 < S:
        assert not bool(dV[first + T - 1:].float().abs().max() > 0)


def test_wide_keys_rerun_bitwise_and_unaligned_workspace(dev):  # noqa: F811
    case = (33, 20, 3, 70, 264, 136)
    _, _, _, V, Qd, dHd = _run(dev, case, seed=3)
    a = lr.route_all_bwd(V, None, Qd, dHd, SLICED, case[2])
    need = lr.route_all_bwd_workspace_bytes(*case[:1], *case[3:], case[2], case[1], SLICED,
                                            torch.bfloat16)
    ws = torch.empty((need + 4,), dtype=torch.uint8, device=dev)[4:]
    out = (torch.full_like(a[0], 7.0), None, torch.full_like(a[2], 7.0))
    b = lr.route_all_bwd(V, None, Qd, dHd, SLICED, case[2], out=out, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(a[0].view(torch.int16), b[0].view(torch.int16)) and torch.equal(a[2], b[2])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("column", [0, 250], ids=["value", "key"])
def test_wide_keys_confine_non_finite_values(dev, value, column):  # noqa: F811
    """A non-finite value of source 11 at token 2 reaches the sites that read
    it and no other (their own single-site results stay what they were), and
    a source that no site reads is not read at all; a non-finite upstream
    value of the first site reaches only the sources that this site reads."""
    S, T, first, N, d, r = 14, 12, 2, 5, 256, 128
    _, _, _, V, Qd, dHd = _run(dev, (S, T, first, N, d, r), seed=9)
    H0, ne0 = lr.route_all_fwd(V, None, Qd, SLICED, first)
    dV0, _, dQ0 = lr.route_all_bwd(V, None, Qd, dHd, SLICED, first)
    Vb = V.clone()
    Vb[13] = float("nan")  # past every prefix
    Vb[11, 2, column] = value
    H, ne = lr.route_all_fwd(Vb, None, Qd, SLICED, first)
    dV, _, dQ = lr.route_all_bwd(Vb, None, Qd, dHd, SLICED, first)
    readers = [j for j in range(T) if first + j > 11]
    others = [j for j in range(T) if first + j <= 11]
    other_tokens = [0, 1, 3, 4]
    assert torch.equal(H[:, other_tokens], H0[:, other_tokens])
    assert torch.allclose(H[others].float(), H0[others].float(), rtol=2.0 ** -7, atol=1e-6)
    assert torch.equal(ne[others], ne0[others])
    assert not bool(torch.isfinite(H[readers][:, 2, column].float()).any())
    if column >= d - r:
        assert not bool(torch.isfinite(H[readers][:, 2].float()).any())
    assert torch.equal(dV[:, other_tokens], dV0[:, other_tokens])
    assert torch.allclose(dQ[others], dQ0[others], rtol=1e-4, atol=1e-4)
    assert not bool(torch.isfinite(dQ[readers]).any())
    assert not bool(dV[13].float().abs().max() > 0)
    dHb = dHd.clone()
    dHb[0, 2, column] = value
    dV, _, dQ = lr.route_all_bwd(V, None, Qd, dHb, SLICED, first)
    torch.cuda.synchronize()
    assert torch.allclose(dV[first:].float(), dV0[first:].float(), rtol=2.0 ** -7, atol=1e-4)
    assert not bool(torch.isfinite(dV[:first, 2, column].float()).any())
    assert torch.allclose(dQ[1:], dQ0[1:], rtol=1e-4, atol=1e-4)


# Full-rank keys: (S, T, first, N, d).  Every width of the single-site kernel
# that keeps its rows in registers (256, 512, 1024 columns, ragged), rows wider
# than those, and more tokens than run site by site in the forward.
FULL_CASES = [(33, 20, 3, 9, 200), (12, 11, 2, 5, 488), (49, 48, 2, 6, 1000), (9, 8, 2, 6, 1544),
              (18, 3, 16, 1030, 136)]
# (S, N, d) of single sites with many tokens: a wave per token, or per 2 or 4.
MANY_TOKENS = [(2, 2051, 1000), (4, 2049, 136), (7, 2050, 512), (16, 2053, 776), (30, 2049, 264),
               (64, 2049, 96)]


@pytest.mark.parametrize("case", FULL_CASES, ids=lambda c: "S{}-T{}-f{}-N{}-d{}".format(*c))
def test_full_rank_sites_match_oracle_and_single_sites(dev, case):  # noqa: F811
    S, T, first, N, d = case
    p, Q, dH, V, Qd, dHd = _run(dev, (S, T, first, N, d, d), seed=S + T + N)
    Q64 = Q.astype(np.float64)
    dV, _, dQ = lr.route_all_bwd(V, None, Qd, dHd, FULL, first)
    H, ne = lr.route_all_fwd(V, None, Qd, FULL, first)
    torch.cuda.synchronize()
    Hr, NEr = oracle.route_all_fwd(p.V, None, Q64, FULL, first, r=d)
    rV, _, rQ = oracle.route_all_bwd(p.V, None, Q64, dH, FULL, first, r=d)
    check_bf16_value("H", to_host(H), Hr)
    check_f32("neff", to_host(ne), NEr)
    check_bf16_key_grad("dV", to_host(dV), rV)
    check_dq("dQ", to_host(dQ), rQ)
    for j in sorted({0, T // 2, T - 1}):
        sV, _, sq = lr.route_bwd(V[:first + j], None, Qd[j].contiguous(), dHd[j], FULL)
        torch.cuda.synchronize()
        if d <= 1024:
            assert torch.equal(dQ[j], sq), f"dQ row {j}"
        oV, _, _ = oracle.route_bwd(p.V[:first + j], None, Q64[j], dH[j], FULL, r=d)
        check_bf16_value("single-site dV", to_host(sV), oV)


@pytest.mark.parametrize("case", MANY_TOKENS, ids=lambda c: "S{}-N{}-d{}".format(*c))
@pytest.mark.parametrize("accumulate", [False, True], ids=["write", "add"])
def test_full_rank_single_site_of_many_tokens(dev, case, accumulate):  # noqa: F811
    S, N, d = case
    p, Q, dH, V, Qd, dHd = _run(dev, (S, 1, S, N, d, d), seed=S + N)
    rV, _, rQ = oracle.route_bwd(p.V, None, Q[0].astype(np.float64), dH[0], FULL, r=d)
    out = None
    if accumulate:
        dV0 = bf16_bits_from_f32(np.random.default_rng(5).standard_normal((S, N, d)).astype(np.float32))
        out = (to_dev(dV0, dev), None, torch.zeros((d,), device=dev))
        rV = rV + f32_from_bf16_bits(dV0)
    dV, _, dq = lr.route_bwd(V, None, Qd[0].contiguous(), dHd[0], FULL, out=out, accumulate=accumulate)
    _, _, dQ = lr.route_all_bwd(V, None, Qd, dHd, FULL, S)
    torch.cuda.synchronize()
    # Few sources leave |dV| past 5.12, where a correctly rounded bf16 is up to
    # 2^-8 |dV| off: the bar for grown values.
    check_bf16_grown("dV", to_host(dV), rV)
    check_dq("dq", to_host(dq), rQ)
    assert torch.equal(dQ[0], dq)


# (N, d): both sides of the tokens from which a single site takes a wave per
# token, with one tile of sources (320) and with more (1024), for every width.
SINGLE_SITES = [(319, 136), (321, 1000), (321, 264), (1024, 200), (1025, 200), (1025, 456),
                (2053, 1024)]


@pytest.mark.parametrize("N,d", SINGLE_SITES)
def test_full_rank_rows_of_one_pass_are_the_single_sites(dev, N, d):  # noqa: F811
    """Every dQ row of one pass over the stack is bit for bit the single-site
    dq of its site: 2 to 4 sources (a wave shared by four tokens), to 8, to 16,
    to 32 and above."""
    S, first = 50, 2
    T = S - first + 1
    _, _, _, V, Qd, dHd = _run(dev, (S, T, first, N, d, d), seed=N + d)
    _, _, dQ = lr.route_all_bwd(V, None, Qd, dHd, FULL, first)
    for n_src in (2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 48, 49, 50):
        j = n_src - first
        _, _, dq = lr.route_bwd(V[:n_src], None, Qd[j].contiguous(), dHd[j], FULL)
        torch.cuda.synchronize()
        assert torch.equal(dQ[j], dq), f"{n_src} sources"


@pytest.mark.parametrize("mode,N,r", [(SLICED, 5, 128), (FULL, 1030, 256)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_values_stay_with_their_readers_when_adding(dev, value, mode, N, r):  # noqa: F811
    """As test_wide_keys_confine_non_finite_values, gradients added to what is
    there, and with full-rank keys, where a non-finite value is a key too."""
    S, T, first, d, n, column = 14, 12, 2, 256, 2, 40
    _, _, _, V, Qd, dHd = _run(dev, (S, T, first, N, d, r), seed=19)
    base = torch.randn((S, N, d), device=dev).to(torch.bfloat16)

    def add(V, dH):
        out = (base.clone(), None, torch.ones_like(Qd))
        lr.route_all_bwd(V, None, Qd, dH, mode, first, out=out, accumulate=True)
        return out[0], out[2]

    dV0, dQ0 = add(V, dHd)
    # an upstream value of the first site: sources that this site reads
    dHb = dHd.clone()
    dHb[0, n, column] = value
    dV, dQ = add(V, dHb)
    torch.cuda.synchronize()
    tokens = [t for t in range(N) if t != n]
    assert torch.equal(dV[:, tokens], dV0[:, tokens])
    assert torch.allclose(dV[first:].float(), dV0[first:].float(), rtol=2.0 ** -7, atol=1e-3)
    assert not bool(torch.isfinite(dV[:first, n, column].float()).any())
    assert torch.allclose(dQ[1:], dQ0[1:], rtol=1e-4, atol=1e-3)
    # a source value: the sites that read it, and through them all they read
    Vb = V.clone()
    Vb[11, n, column] = value
    H0, _ = lr.route_all_fwd(V, None, Qd, mode, first)
    H, _ = lr.route_all_fwd(Vb, None, Qd, mode, first)
    dV, dQ = add(Vb, dHd)
    torch.cuda.synchronize()
    readers = [j for j in range(T) if first + j > 11]
    others = [j for j in range(T) if first + j <= 11]
    assert torch.equal(H[:, tokens], H0[:, tokens])
    assert torch.allclose(H[others].float(), H0[others].float(), rtol=2.0 ** -7, atol=1e-6)
    assert not bool(torch.isfinite(H[readers][:, n, column].float()).any())
    assert torch.equal(dV[:, tokens], dV0[:, tokens])
    assert torch.allclose(dQ[others], dQ0[others], rtol=1e-4, atol=1e-3)
    assert not bool(torch.isfinite(dQ[readers]).any())
    assert torch.equal(dV[13, n], dV0[13, n])  # read by no site


def _dq64(V, q, dH, r, eps=1e-6):
    """dq [r] of one site in fp64 by torch, in chunks of tokens."""
    out = torch.zeros((r,), dtype=torch.float64, device=V.device)
    for b in range(0, V.shape[1], 2000):
        x = V[:, b:b + 2000].double()
        k = x[..., x.shape[2] - r:]
        kb = k / (k.square().mean(-1, keepdim=True) + eps).sqrt()
        a = torch.softmax((kb * q.double()).sum(-1), dim=0)
        g = (x * dH[b:b + 2000].double()).sum(-1)
        ds = a * (g - (a * g).sum(0))
        out += (ds[..., None] * kb).sum((0, 1))
    return out.cpu().numpy()


def test_stack_beyond_2_31_elements(dev):  # noqa: F811
    """64-bit plane offsets in the one pass over the stack and in the register
    form of one full-rank site: sampled tokens against the oracle, the last
    ones among them, and rows of dQ over all tokens."""
    S, T, first, N, d, r = 33, 32, 2, 66000, 1000, 72
    assert S * N * d > 2 ** 31
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    V = torch.empty((S, N, d), dtype=torch.bfloat16, device=dev)
    dH = torch.empty((T, N, d), dtype=torch.bfloat16, device=dev)
    for i in range(S):
        V[i].copy_(torch.randn((N, d), generator=g, device=dev))
    for j in range(T):
        dH[j].copy_(torch.randn((N, d), generator=g, device=dev))
    Q = torch.randn((T, r), generator=g, device=dev) * (2.0 / r ** 0.5)
    H, ne = lr.route_all_fwd(V, None, Q, SLICED, first)
    dV, _, dQ = lr.route_all_bwd(V, None, Q, dH, SLICED, first)
    torch.cuda.synchronize()
    toks = torch.as_tensor([0, 1, 32768, N // 2 + 1, N - 2, N - 1], device=dev)

    def host(x):
        return x[:, toks].contiguous()

    def bits(x):
        return host(x).view(torch.int16).cpu().numpy().view(np.uint16)

    Qh = Q.cpu().numpy().astype(np.float64)
    rH, rne = oracle.route_all_fwd(bits(V), None, Qh, SLICED, first, r=r)
    rV, _, _ = oracle.route_all_bwd(bits(V), None, Qh, bits(dH), SLICED, first, r=r)
    check_bf16_grown("H", to_host(host(H)), rH)
    check_f32("neff", to_host(host(ne)), rne)
    check_bf16_grown("dV", to_host(host(dV))[..., :d - r], rV[..., :d - r])
    check_bf16_key_grad("dV key columns", to_host(host(dV))[..., d - r:], rV[..., d - r:])
    for j in (0, T - 1):
        check_dq(f"dQ row {j}", to_host(dQ[j]), _dq64(V[:first + j], Q[j], dH[j], r))
    del H, ne
    q = torch.randn((d,), generator=g, device=dev) * (2.0 / d ** 0.5)
    _, _, dq = lr.route_bwd(V, None, q, dH[0], FULL, out=(dV, None, torch.empty_like(q)))
    torch.cuda.synchronize()
    oV, _, _ = oracle.route_bwd(bits(V), None, q.cpu().numpy().astype(np.float64), bits(dH)[0], FULL,
                                r=d)
    check_bf16_grown("single-site dV", to_host(host(dV)), oV)
    check_dq("single-site dq", to_host(dq), _dq64(V, q, dH[0], d))
