"""Router: the selection on ties, on rows with fewer experts than it asks for and on groups of equal score, and the GEMM where
its form changes (parts of K, tokens per workgroup, tile), with the workspace it asks for and with the logits' alone."""
import numpy as np
import pytest
import torch

import paper_2503_04398_amd as S
import workloads as WL
from oracle import semmoe_oracle as O
from tests import harness as H

pytestmark = pytest.mark.gpu
NONE = 0x7fffffff  # an expert that is not there


def _select(L, k, sb=None, **kw):
    T, E = L.shape
    m = S.SemMoE(S.Config(T=T, d=8, E=E, k=k, F=8, D=1, cap=T, **kw), allocate_workspace=False)
    ids, w = torch.empty(T, k, dtype=torch.int32, device=H.DEV), torch.empty(T, k, device=H.DEV)
    m.route_from_logits(H.to_dev(L), ids, w, sel_bias=None if sb is None else H.to_dev(sb))
    torch.cuda.synchronize()
    return H.to_np(ids), H.to_np(w)


# a round per winner (1), lists of 4, 8 and 16 per lane, 1 to 16 slots a lane, a last slot that is partly there
@pytest.mark.parametrize("E", [1, 7, 16, 33, 64, 100, 128, 130, 250, 256])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16])
def test_ties_and_absent_experts(E, k):
    if k > E:
        pytest.skip("more experts asked for than there are")
    r = np.random.default_rng(E * 17 + k)
    L = r.integers(-3, 3, (41, E)).astype(np.float32)
    L[1::4] += r.standard_normal((len(L[1::4]), E)).astype(np.float32)
    L[2, :] = 0.0
    L[2, ::2] = -0.0  # equal to +0: the lower expert first, whatever the sign
    for i in range(5, 41, 5):  # so many experts are there, the others' logits are -inf
        L[i, r.permutation(E)[1 + i % k:]] = -np.inf
    ids, w = _select(L, k, renorm=True)
    order = np.argsort(-L, axis=1, kind="stable")[:, :k]
    top = np.take_along_axis(L, order, 1)
    there = np.isfinite(top)
    assert (ids == np.where(there, order, NONE)).all()
    e = np.where(there, np.exp(top - top[:, :1]), 0.0)
    assert np.abs(w - e / e.sum(1, keepdims=True)).max() < 1e-6  # a few roundings of numbers up to 1


def _check_groups(E, n, tg, k):
    r = np.random.default_rng(E + tg)
    k = min(k, tg * (E // n))
    L = np.round(2 * r.standard_normal((70, E))).astype(np.float32)  # equal scores in and across groups
    L[0] = 0.0
    L[1] = np.repeat(np.arange(n)[::-1], E // n)
    L[2] = r.standard_normal(E)
    sb = np.round(4 * r.standard_normal(E)).astype(np.float32) / 4
    for bias in (None, sb):
        ids, w = _select(L, k, sb=bias, score="sigmoid", renorm=True, n_group=n, topk_group=tg, routed_scale=2.5)
        want_ids, want_w = O.select_topk(L, k, "sigmoid", True, n, tg, 2.5, bias)
        assert (ids == want_ids).all()
        assert O.max_rel_err(w, want_w) <= 1e-5


# (1 and 2 a token by sigmoid: a round per winner)
@pytest.mark.parametrize("E", [128, 256, 64])
@pytest.mark.parametrize("tg", [1, 3, 4, 7, 8])
@pytest.mark.parametrize("k", [1, 2, 8])
def test_best_of_8_groups(E, tg, k):
    _check_groups(E, 8, tg, k)


# other numbers of groups, and 8 of other sizes: whole slots of 16 experts (16, 48, 64, 80 a group), and groups that share one (1 to 12)
@pytest.mark.parametrize("E,n", [(16, 16), (32, 16), (96, 16), (128, 16), (160, 16), (192, 16), (256, 16), (96, 2), (256, 4), (160, 2),
                                 (40, 4), (60, 12), (72, 8), (96, 8)])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("k", [1, 2, 4, 8])
def test_best_of_any_groups(E, n, half, k):
    _check_groups(E, n, n // 2 if half else 1, k)


# up to 512 tokens in parts of K, beyond in one where K is short (what is in parts there: the next test); 32 (4097), 64 (8193) tokens
# a workgroup, ragged last tiles; more than 128 experts: two workgroups a tile (40 to 500 tokens in parts of K, 1030 and 4095 not), one
# (4096 and 4100), 64 tokens a workgroup from 8193 on
@pytest.mark.parametrize("T,d,E,k", [(257, 512, 128, 8), (512, 1000, 64, 4), (513, 1000, 128, 8), (1024, 2048, 128, 8),
                                     (4096, 264, 128, 8), (4097, 264, 128, 8), (8193, 136, 96, 4), (40, 1984, 160, 8), (200, 1024, 252, 8),
                                     (500, 264, 256, 8), (1030, 2048, 256, 8), (4095, 2056, 132, 4), (4096, 136, 132, 4), (4100, 136, 132, 4),
                                     (8193, 136, 256, 8), (8300, 1024, 160, 6), (130, 72, 16, 1), (300, 2048, 128, 1), (700, 264, 64, 1),
                                     (1030, 2048, 256, 1), (4100, 136, 100, 2)])
def test_gemm_where_its_form_changes(T, d, E, k):
    w = WL.small(T=T, d=d, E=E, k=k, D=1, C=4, dtype="bf16")
    inp = H.make_inputs(w)
    lay = H.Layer(w)
    logits, ids, tw = lay.route(inp)
    want = O.route_logits(inp.X, inp.W_r, None, inp.token_class, inp.class_bias)
    assert O.max_rel_err(logits, want) <= 1e-5  # exact inputs; the order of fp32 sums
    want_ids, want_w = H.oracle_select(w, logits)
    assert (ids == want_ids).all() and O.max_rel_err(tw, want_w) <= 1e-5


# Beyond 512 tokens, on 256 compute units: as many parts of K as the 32-token tiles leave units for, at least 6 slices each, at most 8
# and 512 / tiles (the workspace), and one where the walk gets shorter by less than 20 slices.  513 tokens are 17 tiles (K 2048: 32 / 6 =
# 5 parts), 1024 32 (8), 1025 33 (7), 1500 47 (5), 2049 65 (3), 4096 128 (2), 4097 129 (none).  More than 128 experts: sums of one
# part, by two workgroups a tile, up to 4096 tokens from 32 slices on.  100 experts are no whole tile, 90 no whole quads.
@pytest.mark.parametrize("T,d,E,parts", [(512, 2048, 128, 16), (513, 2048, 128, 5), (1024, 4096, 128, 8), (1025, 4096, 64, 7),
                                         (1500, 1992, 100, 5), (2049, 4096, 90, 3), (4096, 4096, 128, 2), (4096, 2048, 128, 0),
                                         (4097, 4096, 128, 0), (1030, 2048, 256, 1), (4096, 2048, 132, 1), (4097, 2048, 132, 0),
                                         (1030, 1984, 256, 0)])
def test_parts_of_K(T, d, E, parts):
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256, "the parts above are those of 256 compute units"
    w = WL.small(T=T, d=d, E=E, k=8, D=1, C=4, F=8, dtype="bf16")
    inp = H.make_inputs(w)
    lay = H.Layer(w)
    need = lay.m.ws_bytes
    lay.m.ws = torch.full((need + 65536,), 0x5a, dtype=torch.uint8, device=H.DEV)
    want = O.route_logits(inp.X, inp.W_r, None, inp.token_class, inp.class_bias)

    def routed():
        logits, ids, tw = lay.route(inp)
        assert O.max_rel_err(logits, want) <= 1e-5
        want_ids, want_w = H.oracle_select(w, logits)
        assert (ids == want_ids).all() and O.max_rel_err(tw, want_w) <= 1e-5
        return logits

    routed()
    used = lay.m.ws.view(torch.int32) != 0x5a5a5a5a  # which words of the workspace were written: what the sums took
    sets = parts + (1 if E % 4 != 0 and parts else 0)  # no whole quads: the logits too
    assert round(used.sum().item() / (T * E)) == sets
    assert not used[(sets * T * E * 4 + 511) // 4:].any()
    if T > 512:  # a workspace for one set of logits, and with more than 128 experts none at all, is enough: the fused kernel
        lay.m.ws_bytes = T * E * 4 + 512 if E <= 128 and parts else (0 if E > 128 else need)
        lay.m.ws.fill_(0x5a)
        short = routed()
        assert (lay.m.ws == 0x5a).all()
        lay.m.set_tuning(7, 0)
        try:
            assert (routed() == short).all()
        finally:
            lay.m.set_tuning(7, -1)


# 129 to 256 experts while two workgroups share a tile (sigmoid: 513 to 4096 tokens, d from 1473 on), and beside that: logits, ids and
# weights have the bits of the fused kernel's, with either bias and both; arrays off a 16-byte boundary take the fused kernel's
# bias terms one after the other
@pytest.mark.parametrize("T,d,E", [(300, 136, 256), (513, 1480, 132), (1030, 2048, 256), (4096, 1536, 252), (1024, 1472, 160)])
@pytest.mark.parametrize("biases", ["b_g", "class", "both"])
@pytest.mark.parametrize("odd", ["", "b_g", "logits"])
def test_shared_tile_has_the_bits_of_the_fused_kernel(T, d, E, biases, odd):
    g = torch.Generator().manual_seed(T + E)
    new = lambda *shape: torch.empty(shape).normal_(0, 1, generator=g)
    X, W = new(T, d).bfloat16().to(H.DEV), (0.1 * new(E, d)).bfloat16().to(H.DEV)
    off = lambda name: 1 if odd == name else 0  # floats past a 16-byte boundary
    b_g = new(E + 1).to(H.DEV)[off("b_g"):][:E] if biases != "class" else None
    cb, cls = (new(5, E).to(H.DEV), torch.randint(0, 5, (T,), generator=g).int().to(H.DEV)) if biases != "b_g" else (None, None)
    m = S.SemMoE(S.Config(T=T, d=d, E=E, k=8, F=8, D=1, dtype="bf16", cap=T, num_classes=5, score="sigmoid"), device=H.DEV)
    got = {}
    for split in (-1, 0):  # the library's choice, the fused kernel
        ids, w = torch.empty(T, 8, dtype=torch.int32, device=H.DEV), torch.empty(T, 8, device=H.DEV)
        logits = torch.empty(T * E + 1, device=H.DEV)[off("logits"):][:T * E].view(T, E)
        m.set_tuning(7, split)
        try:
            m.route(X, W, ids, w, b_g=b_g, token_class=cls, class_bias=cb, logits_out=logits)
            torch.cuda.synchronize()
        finally:
            m.set_tuning(7, -1)
        got[split] = logits, ids, w
    for name, a, b in zip(("logits", "ids", "weights"), got[-1], got[0]):
        assert torch.equal(a, b), "%s: %d of %d differ" % (name, (a != b).sum(), a.numel())


def test_sigmoid_is_the_oracles_bit_for_bit():
    """1 / (1 + z) is formed from the hardware's reciprocal and two Newton steps, which give the correctly rounded quotient or
    not depending on that first value: of 1 / (2 - 2^-23), half way between two results to first order, two steps from 0.5 stay
    at 0.5.  So: logits for every mantissa that 1 + z takes in [1, 8), the all-ones one among them, those around zero,
    and the ones clamped.  A weight of one expert, not renormalised, is its sigmoid."""
    x = [-np.log(np.maximum(np.arange(lo, lo + (1 << 23), dtype=np.uint32).view(np.float32).astype(np.float64) - 1, 1e-14)).astype(np.float32)
         for lo in (0x3f800000, 0x40000000, 0x40800000)]
    tiny = np.arange(1 << 16, dtype=np.uint32) << 15 | 1
    x += [tiny.view(np.float32), (tiny | 0x80000000).view(np.float32),
          np.array([0.0, -0.0, 30.0, -30.0, 31.0, -31.0, 88.8, -88.8, 104.0, -104.0, np.inf, -np.inf], np.float32)]
    x = np.concatenate(x)
    x = x[~np.isnan(x)]
    t = -np.clip(x, np.float32(-30), np.float32(30)) * O._LOG2E  # the denominators, to see which there are
    n = np.rint(t)
    z = np.full_like(t, O._EXP2_COEF[6])
    for c in O._EXP2_COEF[5::-1]:
        z = z * (t - n) + c
    q = np.float32(1) + np.ldexp(z, n.astype(np.int32))
    s = O.sigmoid_f32(x)
    assert q.dtype == np.float32 and (np.float32(1) / q == s).all()
    mantissas = np.unique(q.view(np.uint32) & 0x7fffff)
    assert mantissas[-1] == 0x7fffff and len(mantissas) > 0.997 * 2 ** 23
    for at in range(0, len(x), 1 << 23):
        part = x[at:at + (1 << 23)]
        ids, w = _select(part[:, None], 1, score="sigmoid", renorm=False)
        bad = np.flatnonzero(w[:, 0].view(np.uint32) != s[at:at + (1 << 23)].view(np.uint32))
        assert len(bad) == 0, "%d of %d, the first at %r" % (len(bad), len(part), part[bad[0]])
        assert (ids == 0).all()


# not a number: with the sign bit clear it is above every number (equal ones: the lower expert first), with it set it is like
# an expert that is not there, and a row of nothing else has none.  Scores by sigmoid take it for the lowest logit, -30.
@pytest.mark.parametrize("E", [16, 100, 128, 250, 256])
@pytest.mark.parametrize("k", [1, 2, 4, 8, 16])
def test_not_a_number(E, k):
    r = np.random.default_rng(E + k)
    L = r.standard_normal((40, E)).astype(np.float32)
    up, down = np.array([0x7fc00000, 0xffc00000], np.uint32).view(np.float32)
    for i in range(1, 40):
        L[i, r.permutation(E)[:i % 5]] = up
        L[i, r.permutation(E)[:i % 7]] = down
    L[39] = down
    ids, _ = _select(L, k, renorm=True)
    bits = L.view(np.uint32)
    rank = np.where(bits == 0x7fc00000, np.inf, np.where(bits == 0xffc00000, -np.inf, L))
    order = np.argsort(-rank, axis=1, kind="stable")[:, :k]
    assert (ids == np.where(np.take_along_axis(rank, order, 1) > -np.inf, order, NONE)).all()
    ids, w = _select(L, k, score="sigmoid", renorm=False)
    want_ids, want_w = O.select_topk(np.where(np.isnan(L), np.float32(-30), L), k, "sigmoid")
    assert (ids == want_ids).all() and (w == want_w.astype(np.float32)).all()
