"""What the all-sites calls accept with sliced keys wider than 64 columns,
checked on the host: the wide launch takes no problem that the sites refuse
one by one, and needs no workspace without tokens."""
import ctypes

import pytest

import paper_2607_09694_amd as lr

BF16, F32 = 1, 0


def _workspace(S, N, d, r, first, T, dtype):
    return lr.load_library().lr_attnres_route_all_bwd_workspace_bytes(S, N, d, r, first, T,
                                                                      lr.SLICED, dtype)


@pytest.mark.parametrize("S,N,d,r,first,T,dtype,wide", [
    (49, 100, 1024, 256, 2, 48, BF16, True),
    (64, 100, 1024, 72, 1, 64, BF16, True),
    (49, 100, 1024, 260, 2, 48, BF16, None),    # r above the backward's 256: refused
    (49, 100, 1024, 100, 2, 48, BF16, False),   # r % 8 != 0
    (49, 100, 1024, 256, 2, 48, F32, False),    # fp32 storage
    (65, 100, 1024, 256, 2, 40, BF16, False),   # S > 64
    (49, 0, 1024, 256, 2, 48, BF16, None),      # no tokens
])
def test_workspace_names_the_route(S, N, d, r, first, T, dtype, wide):
    need = _workspace(S, N, d, r, first, T, dtype)
    coefficients = N * T * 64 * 4
    assert need == 0 if wide is None else (need > coefficients) == wide


def test_rank_above_the_backward_limit_stays_refused():
    lib = lr.load_library()
    a = [0x10_0000_0000 * k for k in range(1, 7)]
    rc = lib.lr_attnres_route_all_bwd(a[0], None, a[1], a[2], a[3], None, a[4], a[5], 1 << 34, 49,
                                      100, 1024, 264, 2, 48, lr.SLICED, BF16,
                                      ctypes.c_float(1e-6), 0, None)
    assert rc == 2 and b"site by site" in lib.lr_attnres_last_error()


@pytest.mark.parametrize("N,wide", [((1 << 24) - 1, True), (1 << 24, False), (1 << 30, False)])
def test_tokens_past_one_launch_run_site_by_site(N, wide):
    """The wide kernels take a 256-thread workgroup per token and a launch less
    than 2^32 threads; calls with more tokens stay accepted."""
    need = _workspace(32, N, 72, 72, 1, 32, BF16)
    assert need > 0 and (need > N * 32 * 64 * 4) == wide
    lib = lr.load_library()
    a = [0x1000_0000_0000 * k for k in range(1, 7)]
    rc = lib.lr_attnres_route_all_bwd(a[0], None, a[1], a[2], a[3], None, a[4], a[5], need - 1, 32,
                                      N, 72, 72, 1, 32, lr.SLICED, BF16, ctypes.c_float(1e-6), 0,
                                      None)
    assert rc == 1 and b"workspace" in lib.lr_attnres_last_error()


@pytest.mark.parametrize("S,N,first,T,wide", [
    (12, 2048, 9, 4, True), (12, 2049, 9, 4, False),      # 42 reads, 4 sites
    (12, 2049, 2, 11, True),
    (6, 1280, 2, 5, True), (6, 1281, 2, 5, False), (4, 1280, 2, 3, False),
    (64, 2048, 63, 2, False), (64, 2048, 64, 1, False),   # fewer than three sites
    (49, 8192, 47, 3, True), (24, 2049, 22, 3, False),
])
def test_few_sites_run_one_by_one(S, N, first, T, wide):
    """One pass over the stack only where it is ahead of the sites: few reads
    of the stack keep the single site's workspace."""
    need = _workspace(S, N, 1024, 256, first, T, BF16)
    single = lr.load_library().lr_attnres_route_bwd_workspace_bytes(S, N, 1024, 256, lr.SLICED, BF16)
    assert (need == single) != wide and (need > N * T * 64 * 4) == wide


def _single(S, N, d, r, mode, dtype):
    return lr.load_library().lr_attnres_route_bwd_workspace_bytes(S, N, d, r, mode, dtype)


@pytest.mark.parametrize("S,N,d,shares", [
    (49, 16384, 1024, 64), (2, 16384, 1000, 64), (64, 100000, 64, 1024), (100, 1000, 512, 128),
])
def test_one_full_rank_site_asks_for_one_site(S, N, d, shares):
    """The softmax gradients of each token at one site and the dq shares, or
    the dq partials of a workgroup per 16 (few tokens: 4 or 8) tokens."""
    rows = 16 + (N * 64 + shares * d) * 4
    assert rows <= _single(S, N, d, d, lr.FULL, BF16) <= max(rows, -(-N // 4) * d * 4)


@pytest.mark.parametrize("S,N,d,dtype", [(64, 16384, 2048, BF16), (49, 16384, 1020, BF16), (49, 16385, 1024, BF16),
                                         (49, 16384, 1024, F32), (49, 1 << 24, 64, BF16)])
def test_full_rank_sites_of_other_forms_ask_for_dq_partials(S, N, d, dtype):
    assert _single(S, N, d, d, lr.FULL, dtype) == -(-N // 16) * d * 4


@pytest.mark.parametrize("mode,d,r,dtype", [(lr.PROJECTED, 256, 16, BF16), (lr.SLICED, 256, 16, F32),
                                            (lr.FULL, 512, 512, BF16), (lr.FULL, 512, 512, F32)])
@pytest.mark.parametrize("N", [1, 300, 512, 513, 5000])
def test_workspace_is_the_same_for_every_number_of_sources(mode, d, r, dtype, N):
    """A buffer sized for the first site of a pass serves the later ones."""
    assert len({_single(S, N, d, r, mode, dtype) for S in (1, 2, 3, 64, 65, 512)}) == 1
