"""Grouped FFN kernels for few and for middling rows per expert, on group sizes at the edges of their tiles.

The expert FFN is called with offsets written by hand and compared with a float64 product on the CPU: all rows together
(fp32 1e-5, bf16 2e-2 of the largest value) and each row by itself, against its own norm.

Bound of a row.  A value y = sum_f h_f w_f has the norm |h||w| to go by, and a row of them about sqrt(d) times that, which
is the row's own norm for weights drawn at random.  bf16 (u = 2^-9, the largest relative error of one rounding): the hidden
activation and the result are rounded, errors that are independent from entry to entry, so a row is off by sqrt(2) u = 0.28 %
of its norm at most; fp32 sums of up to 1536 terms and the fast exponential add less than 1e-5.  fp32: a sum of K terms in
four parts is off by sqrt(K) 2^-24 of its norm where roundings are independent, twice in a row (gate/up, down), 4.7e-6 in
all at K = 1536, 5.5e-6 at K = 3600 and then 1024; the bounds below are about twice these."""
import numpy as np
import pytest
import torch

import paper_2503_04398_amd as S
from tests import harness as H

pytestmark = pytest.mark.gpu
ROW_TOL = {"fp32": 1e-5, "bf16": 6e-3}  # see above


def _ffn(rows, d, F, dtype, D=1, rank=-1, knobs=(), seed=0):
    """(Y, its float64 reference, rows of the rank, poison) of one expert_ffn call with `rows` rows per expert"""
    r = np.random.default_rng(seed)
    E, P = len(rows), int(sum(rows))
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    X = torch.from_numpy(r.standard_normal((P, d), dtype=np.float32)).to(act)
    W_gu = torch.from_numpy(0.05 * r.standard_normal((E, 2 * F, d), dtype=np.float32)).to(act)
    W_dn = torch.from_numpy(0.05 * r.standard_normal((E, d, F), dtype=np.float32)).to(act)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    of_phys = r.permutation(E).astype(np.int32)
    m = S.SemMoE(S.Config(T=P, d=d, E=E, k=1, F=F, D=D, dtype=dtype, cap=P))
    Y = torch.full((P, d), 512.0, dtype=act, device=H.DEV)
    m.ws.fill_(0xff)  # NaN: a hidden activation that nobody writes does not pass for one left by another call
    try:
        for key, value in knobs:
            m.set_tuning(key, value)
        m.expert_ffn(rank, X.to(H.DEV), torch.from_numpy(off).to(H.DEV), torch.from_numpy(of_phys).to(H.DEV), W_gu.to(H.DEV),
                     W_dn.to(H.DEV), Y)
        torch.cuda.synchronize()
    finally:
        for key, _ in knobs:
            m.set_tuning(key, -1)
    lo, hi = (0, E) if rank < 0 else (rank * (E // D), (rank + 1) * (E // D))
    want = np.full((P, d), 512.0)
    for q in range(lo, hi):
        x = X[off[q]:off[q + 1]].double().numpy()
        gu, dn = W_gu[of_phys[q]].double().numpy(), W_dn[of_phys[q]].double().numpy()
        gate, up = x @ gu[:F].T, x @ gu[F:].T
        want[off[q]:off[q + 1]] = (gate / (1.0 + np.exp(-gate)) * up) @ dn.T
    return H.to_np(Y), want, slice(int(off[lo]), int(off[hi]))


def _check(got, want, mine, dtype):
    H.assert_close(got[mine], want[mine], dtype, "Y")
    assert (np.delete(got, np.r_[mine], axis=0) == 512.0).all()  # rows of other ranks stay as they were
    off = np.linalg.norm(got[mine] - want[mine], axis=1) / np.linalg.norm(want[mine], axis=1)
    assert off.max() <= ROW_TOL[dtype], "row %d of the rank: |a-b|/|b| = %.3e" % (off.argmax(), off.max())


RAGGED = (0, 1, 15, 16, 17, 33, 64, 65, 0, 130, 31, 48)


# d / F: whole slices for every wave (256 / 512: K = 512, 256 and more); K with a partial slice (264 / 296: 8 elements in
# the last one); K so short that some waves have no slice (72, 8); F below a feature tile (8, 24)
@pytest.mark.parametrize("d,F", [(256, 512), (264, 296), (72, 24), (512, 8), (8, 72)])
@pytest.mark.parametrize("tile,cap", [(30, -1), (31, -1), (32, -1), (30, 8), (32, 3), (34, -1), (34, 3), (35, -1), (35, 8)])
def test_streamed_tiles_bf16(tile, cap, d, F):
    got, want, mine = _ffn(RAGGED, d, F, "bf16", knobs=((0, tile), (1, tile), (4, cap)), seed=tile + d)
    _check(got, want, mine, "bf16")


# one hot group and small ones on grids of 8 and 16 workgroups, of which the hot group's tiles take some: by the width of
# the shape itself (one or both products have so few tiles), and by a cap on a wider one with 2, 3, 4 and 5 large tiles
@pytest.mark.parametrize("rows,d,F", [((70, 10, 10, 10), 64, 256), ((66, 4), 128, 256), ((66, 12), 128, 192),
                                      ((70, 10, 10, 6), 256, 32), ((65, 9, 0, 7), 8, 8)])
def test_hot_group_on_a_small_grid(rows, d, F):
    got, want, mine = _ffn(rows, d, F, "bf16", seed=d + F)
    _check(got, want, mine, "bf16")


@pytest.mark.parametrize("rows", [(65, 3, 17), (130, 9, 64, 1), (65, 20, 65, 33), (200, 9, 5), (65, 8, 130, 40)])
@pytest.mark.parametrize("tile", [34, 35])
@pytest.mark.parametrize("cap", [8, 16])
def test_hot_group_under_a_cap(cap, tile, rows):
    got, want, mine = _ffn(rows, 64, 64, "bf16", knobs=((0, tile), (1, tile), (4, cap)), seed=len(rows))
    _check(got, want, mine, "bf16")


@pytest.mark.parametrize("d,F", [(256, 512), (264, 296), (72, 24), (512, 8), (8, 72)])
@pytest.mark.parametrize("rows,cap", [(RAGGED, -1), (RAGGED, 8), ((3,) * 12, -1), ((140,) * 12, 5)])
def test_fp32(rows, cap, d, F):
    got, want, mine = _ffn(rows, d, F, "fp32", knobs=((4, cap),), seed=d)
    _check(got, want, mine, "fp32")


# every fp32 form by its id; 37 holds 64-bit addresses, which the library takes for panels of 2 GiB
@pytest.mark.parametrize("d,F", [(256, 512), (264, 296), (72, 24), (512, 8), (8, 72)])
@pytest.mark.parametrize("tile,cap", [(30, -1), (31, 5), (32, -1), (36, -1), (37, -1), (37, 5)])
def test_fp32_forms(tile, cap, d, F):
    got, want, mine = _ffn(RAGGED, d, F, "fp32", knobs=((0, tile), (1, tile), (4, cap)), seed=tile + d)
    _check(got, want, mine, "fp32")


@pytest.mark.parametrize("T,d,E", [(70, 72, 24), (130, 512, 50), (17, 8, 7), (33, 264, 256)])
@pytest.mark.parametrize("tile", [-1, 30, 31, 32, 36, 37])
def test_fp32_router_forms(tile, T, d, E):
    r = np.random.default_rng(T)
    X, W = torch.from_numpy(r.standard_normal((T, d), dtype=np.float32)), torch.from_numpy(0.1 * r.standard_normal((E, d), dtype=np.float32))
    b_g, bias = (torch.from_numpy(r.standard_normal(n, dtype=np.float32)) for n in (E, (3, E)))
    cls = torch.from_numpy(r.integers(-1, 3, T).astype(np.int32))
    m = S.SemMoE(S.Config(T=T, d=d, E=E, k=2, F=8, D=1, dtype="fp32", cap=T, num_classes=3))
    ids, w = torch.empty(T, 2, dtype=torch.int32, device=H.DEV), torch.empty(T, 2, device=H.DEV)
    logits = torch.full((T, E), 512.0, device=H.DEV)
    try:
        m.set_tuning(0, tile)
        m.route(X.to(H.DEV), W.to(H.DEV), ids, w, b_g=b_g.to(H.DEV), token_class=cls.to(H.DEV), class_bias=bias.to(H.DEV),
                logits_out=logits)
        torch.cuda.synchronize()
    finally:
        m.set_tuning(0, -1)
    want = X.double() @ W.double().t() + b_g.double() + torch.cat([bias, torch.zeros(1, E)]).double()[cls.long()]  # -1: the zeros
    H.assert_close(H.to_np(logits), want.numpy(), "fp32", "logits")


# gate and up of one set of weights in 2 GiB and a little more: beyond 32-bit offsets.  fp32 takes 64-bit addresses, the
# streamed bf16 tiles hand over to the 128 x 64 ones; the down projection (half as large) stays as it is
@pytest.mark.parametrize("dtype,d,F", [("fp32", 16384, 16392), ("bf16", 16384, 32776)])
@pytest.mark.parametrize("grouped", [False, True])
def test_weights_of_two_gib(dtype, d, F, grouped):
    act, n = (torch.float32 if dtype == "fp32" else torch.bfloat16), 5
    g = torch.Generator(device=H.DEV).manual_seed(d + F)
    def randn(*shape, std):
        return torch.empty(shape, dtype=act, device=H.DEV).normal_(0.0, std, generator=g)
    X, gu, dn = randn(n, d, std=1.0), randn(2 * F, d, std=0.01), randn(d, F, std=0.01)
    assert gu.numel() * gu.element_size() >= 2 ** 31
    m = S.SemMoE(S.Config(T=n, d=d, E=1, k=1, F=F, D=1, dtype=dtype, cap=n))
    Y = torch.empty(n, d, dtype=act, device=H.DEV)
    if grouped:
        m.expert_ffn(-1, X, torch.tensor([0, n], dtype=torch.int32, device=H.DEV),
                     torch.zeros(1, dtype=torch.int32, device=H.DEV), gu, dn, Y)
    else:
        m.shared_ffn(X, n, gu, dn, Y)
    got = H.to_np(Y)
    hidden = torch.empty(n, F, dtype=torch.float64, device=H.DEV)
    for lo in range(0, F, 4096):  # float64 a slice at a time
        hi = min(lo + 4096, F)
        gate, up = X.double() @ gu[lo:hi].double().t(), X.double() @ gu[F + lo:F + hi].double().t()
        hidden[:, lo:hi] = gate * torch.sigmoid(gate) * up
    want = torch.cat([hidden @ dn[lo:lo + 4096].double().t() for lo in range(0, d, 4096)], dim=1)
    H.assert_close(got, want.cpu().numpy(), dtype, "Y")


# grid caps: 1 and 3 workgroups walk many tiles (the load stream crosses tile ends, a tile end every 3 slices at K = 192);
# 16 leaves a few tiles over, which run as pieces; F = 320 fills two and a half feature tiles
@pytest.mark.parametrize("cap", [-1, 1, 3, 16])
@pytest.mark.parametrize("d,F", [(256, 320), (192, 448), (448, 192)])
def test_256x128_tiles(cap, d, F):
    rows = (0, 1, 127, 128, 129, 300, 64, 65)
    got, want, mine = _ffn(rows, d, F, "bf16", D=2, rank=1, knobs=((0, 33), (1, 33), (4, cap)), seed=d)
    _check(got, want, mine, "bf16")


# the same tiles uncut (knob 5 at 0), and the workgroups per compute unit of the tiles that run two kernels in a launch
@pytest.mark.parametrize("tile,knob", [(33, (5, 0)), (34, (2, 1)), (35, (2, 4))])
@pytest.mark.parametrize("cap", [-1, 3, 16])
@pytest.mark.parametrize("d,F", [(256, 320), (448, 192)])
def test_knobs_of_the_default_tiles(cap, tile, knob, d, F):
    rows = (0, 1, 127, 128, 129, 300, 64, 65)
    got, want, mine = _ffn(rows, d, F, "bf16", knobs=((0, tile), (1, tile), (4, cap), knob), seed=d)
    _check(got, want, mine, "bf16")


# the library's own choice over its range of rows per expert, many experts and few, whole slices of K and not
@pytest.mark.parametrize("rows_per_expert", [1, 9, 10, 19, 20, 39, 40, 191, 192, 383, 384])
@pytest.mark.parametrize("E,D,d,F", [(32, 1, 256, 192), (4, 2, 200, 136), (2, 1, 384, 256)])
def test_own_choice(rows_per_expert, E, D, d, F):
    r = np.random.default_rng(rows_per_expert)
    rows = np.full(E, rows_per_expert) + r.integers(0, 3, E)
    rows[0] += int(rows[1]) - 1
    rows[1] = 1
    got, want, mine = _ffn(tuple(rows), d, F, "bf16", D=D, rank=D - 1 if D > 1 else -1, seed=rows_per_expert)
    _check(got, want, mine, "bf16")


# ... on both sides of its lines in K and in the number of tiles: streamed (1 and 12 rows per expert), 256 x 128 tiles, and
# more experts than those have room for.  One expert has most of its neighbour's rows as well
@pytest.mark.parametrize("rows_per_expert,E,d,F", [
    (1, 8, 184, 192), (1, 8, 192, 384), (1, 64, 384, 376), (1, 96, 64, 960), (1, 128, 640, 632), (1, 128, 1536, 64),
    (12, 4, 640, 576), (12, 64, 320, 960), (12, 128, 960, 128), (25, 16, 1408, 64), (25, 16, 64, 1408), (25, 8, 2048, 64),
    (35, 4, 64, 4096), (12, 8, 64, 2048), (35, 128, 1408, 512), (35, 127, 1408, 512), (34, 32, 2048, 1024),
    (45, 64, 640, 512), (45, 40, 1408, 256), (130, 16, 192, 1408), (200, 32, 640, 512), (100, 382, 192, 192), (100, 384, 192, 64),
    (192, 384, 64, 192)])
def test_own_choice_by_depth_and_tiles(rows_per_expert, E, d, F):
    rows = np.full(E, rows_per_expert + 1)
    rows[0] += int(rows[1]) - 1
    rows[1] = 1
    got, want, mine = _ffn(tuple(rows), d, F, "bf16", seed=d)
    _check(got, want, mine, "bf16")


# fp32, both sides of the lines between 16 tokens a tile, 32 x 32 and 64 x 64 tiles: 8 and 16 tiles of 64 weight rows a compute unit
# (of 256) in gate and up, 8, 9, 16, 17, 48 and 49 rows expected
@pytest.mark.parametrize("rows_per_expert,E", [(8, 128), (9, 127), (9, 128), (17, 127), (17, 128), (48, 128), (49, 128), (3, 256), (4, 256)])
def test_own_choice_fp32(rows_per_expert, E):
    rows = np.full(E, rows_per_expert)
    rows[0] += int(rows[1]) - 1
    rows[1] = 1
    got, want, mine = _ffn(tuple(rows), 16, 512, "fp32", seed=E)
    _check(got, want, mine, "fp32")


# ... and by K: 64 x 64 tiles from 12, 6 and 4 a compute unit on (gate and up, K below 1024, below 3600 and from there), one tile less
@pytest.mark.parametrize("rows_per_expert,E,d,F", [(1024, 3, 1016, 2048), (1024, 3, 1016, 2016), (1024, 2, 1024, 1536), (1024, 2, 1024, 1504),
                                                   (1024, 2, 3592, 1024), (1024, 2, 3600, 1024), (1024, 2, 3600, 992)])
def test_own_choice_fp32_by_depth(rows_per_expert, E, d, F):
    rows = np.full(E, rows_per_expert)
    rows[0] += int(rows[1]) - 1
    rows[1] = 1
    got, want, mine = _ffn(tuple(rows), d, F, "fp32", seed=d)
    _check(got, want, mine, "fp32")


# sums are formed in one order: a second call gives the same bits
@pytest.mark.parametrize("dtype,tile", [("bf16", t) for t in (30, 31, 32, 33, 34, 35)] + [("fp32", t) for t in (30, 31, 32, 36, 37)])
def test_same_bits_again(dtype, tile):
    args = ((150, 3, 70, 0, 17, 64, 1, 40), 448, 320, dtype)
    (first, _, mine), (again, _, _) = (_ffn(*args, knobs=((0, tile), (1, tile)), seed=tile) for _ in range(2))
    assert (first[mine] == again[mine]).all()


@pytest.mark.parametrize("n", [1, 64, 160, 161, 256, 257, 400])
def test_one_set_of_weights(n):
    """the shared expert on n rows, on both sides of the lines between its tiles"""
    r = np.random.default_rng(n)
    d, F = 448, 320
    X, gu, dn = (torch.from_numpy(s * r.standard_normal(shape, dtype=np.float32)).bfloat16()
                 for s, shape in ((1.0, (n, d)), (0.05, (2 * F, d)), (0.05, (d, F))))
    m = S.SemMoE(S.Config(T=n, d=d, E=2, k=1, F=F, D=1, dtype="bf16", cap=n))
    Y = torch.empty(n, d, dtype=torch.bfloat16, device=H.DEV)
    m.shared_ffn(X.to(H.DEV), n, gu.to(H.DEV), dn.to(H.DEV), Y)
    gate, up = X.double() @ gu[:F].double().t(), X.double() @ gu[F:].double().t()
    H.assert_close(H.to_np(Y), ((gate * torch.sigmoid(gate) * up) @ dn.double().t()).numpy(), "bf16", "Y_shared")


# eight waves a workgroup: whole slices for every wave (512 / 1024), a partial one, fewer slices than waves; by id on ragged
# groups, so that tiles of many sizes follow each other, and as the shared expert's own choice on both sides of its lines
@pytest.mark.parametrize("d,F", [(512, 1024), (264, 296), (72, 24), (1032, 8)])
@pytest.mark.parametrize("tile,cap", [(38, -1), (38, 3), (39, -1), (39, 8), (40, -1), (40, 5)])
def test_eight_waves(tile, cap, d, F):
    knobs = ((0, tile), (1, tile), (4, cap))
    got, want, mine = _ffn(RAGGED, d, F, "bf16", knobs=knobs, seed=tile + d)
    _check(got, want, mine, "bf16")
    again, _, _ = _ffn(RAGGED, d, F, "bf16", knobs=knobs, seed=tile + d)
    assert (got[mine] == again[mine]).all()


@pytest.mark.parametrize("n,d,F", [(1, 1024, 1032), (129, 1024, 1032), (130, 1000, 2048), (256, 1024, 2048), (257, 1024, 4096),
                                   (520, 4096, 2048), (128, 256, 8200), (130, 200, 8200), (700, 256, 2600)])
def test_one_set_of_weights_by_tiles(n, d, F):
    g = torch.Generator().manual_seed(n + d)
    X, gu, dn = (torch.empty(shape).normal_(0, std, generator=g).bfloat16()
                 for std, shape in ((1.0, (n, d)), (0.05, (2 * F, d)), (0.05, (d, F))))
    m = S.SemMoE(S.Config(T=n, d=d, E=2, k=1, F=F, D=1, dtype="bf16", cap=n))
    Y = torch.empty(n, d, dtype=torch.bfloat16, device=H.DEV)
    m.shared_ffn(X.to(H.DEV), n, gu.to(H.DEV), dn.to(H.DEV), Y)
    x, w, v = (t.to(H.DEV).double() for t in (X, gu, dn))
    gate, up = x @ w[:F].t(), x @ w[F:].t()
    want = (gate * torch.sigmoid(gate) * up) @ v.t()
    H.assert_close(H.to_np(Y), want.cpu().numpy(), "bf16", "Y_shared")
    off = ((Y.double() - want).norm(dim=1) / want.norm(dim=1)).max().item()
    assert off <= ROW_TOL["bf16"], off


# rows of a multiple of 4 KB: every group begins its walk over K at another place (12 groups: first, last and middle slices),
# by the tiles with a ring, with a load stream across tiles (grids of few workgroups: the walk wraps in the middle of a tile and
# at its end), in pieces and streamed; fp32 rows of 4 KB
@pytest.mark.parametrize("d,F", [(2048, 64), (64, 2048)])
@pytest.mark.parametrize("dtype,tile,cap", [("bf16", t, c) for t in (16, 22, 26, 28, 33, 34, 35, 40) for c in (-1, 3)] +
                         [("fp32", 30, -1), ("fp32", 32, 3)])
def test_walks_that_begin_anywhere(dtype, tile, cap, d, F):
    if dtype == "fp32":
        d, F = d // 2, F // 2
    got, want, mine = _ffn(RAGGED, d, F, dtype, knobs=((0, tile), (1, tile), (4, cap)), seed=tile)
    _check(got, want, mine, dtype)


def test_one_rank_gives_the_bits_of_all():
    """a rank's launch numbers its groups from the first one it has; the walks are those of the whole launch"""
    rows, knobs = (30, 64, 17, 40, 9, 33, 128, 50), ((0, 33), (1, 33))
    every, _, _ = _ffn(rows, 2048, 128, "bf16", D=2, rank=-1, knobs=knobs, seed=5)
    second, _, mine = _ffn(rows, 2048, 128, "bf16", D=2, rank=1, knobs=knobs, seed=5)
    assert (every[mine] == second[mine]).all()


def _placed(place, rows, X, W_gu, W_dn, F, dtype, knobs):
    """{expert: its rows of Y} with expert place[q] at physical position q"""
    d, E, P = W_dn.shape[1], len(rows), int(sum(rows))
    off = np.concatenate([[0], np.cumsum([rows[e] for e in place])]).astype(np.int32)
    m = S.SemMoE(S.Config(T=P, d=d, E=E, k=1, F=F, D=1, dtype=dtype, cap=P))
    Y = torch.empty(P, d, dtype=W_dn.dtype, device=H.DEV)
    try:
        for key, value in knobs:
            m.set_tuning(key, value)
        m.expert_ffn(-1, torch.cat([X[e] for e in place]), torch.from_numpy(off).to(H.DEV),
                     torch.tensor(place, dtype=torch.int32, device=H.DEV), W_gu, W_dn, Y)
        torch.cuda.synchronize()
    finally:
        for key, _ in knobs:
            m.set_tuning(key, -1)
    return {e: Y[off[q]:off[q + 1]] for q, e in enumerate(place)}


# rows of 4 KB, where the experts begin their walks at different columns: an expert's rows have the same bits wherever it
# is placed, by every kernel that spreads the starts and by the library's own choice
@pytest.mark.parametrize("d,F", [(2048, 64), (64, 2048)])
@pytest.mark.parametrize("dtype,tile", [("bf16", t) for t in (-1, 16, 22, 26, 28, 33, 34, 35, 40)] + [("fp32", -1), ("fp32", 32)])
def test_bits_of_an_expert_wherever_it_is_placed(dtype, tile, d, F):
    if dtype == "fp32":
        d, F = d // 2, F // 2
    g = torch.Generator().manual_seed(tile + d)
    act, rows = (torch.bfloat16 if dtype == "bf16" else torch.float32), (30, 64, 17, 0, 40, 9, 65, 128, 300, 1)
    new = lambda std, *shape: torch.empty(shape).normal_(0, std, generator=g).to(act).to(H.DEV)
    X, W_gu, W_dn = [new(1.0, n, d) for n in rows], new(0.05, len(rows), 2 * F, d), new(0.05, len(rows), d, F)
    first = _placed(list(range(len(rows))), rows, X, W_gu, W_dn, F, dtype, ((0, tile), (1, tile)))
    other = _placed([7, 0, 8, 5, 1, 9, 2, 3, 6, 4], rows, X, W_gu, W_dn, F, dtype, ((0, tile), (1, tile)))
    for e in first:
        assert torch.equal(first[e], other[e]), "expert %d: %d of %d values" % (e, (first[e] != other[e]).sum(), first[e].numel())
