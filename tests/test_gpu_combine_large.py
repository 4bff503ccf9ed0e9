"""combine on a result larger than half of the memory-side cache, which is stored past the caches: the same bits as from
calls on parts of the tokens, each small enough for ordinary stores."""
import pytest
import torch

import paper_2503_04398_amd as S
from tests import harness as H

pytestmark = pytest.mark.gpu
LINE = 128 << 20  # bytes of the result from which on it is stored past the caches


# widths with a last pass of fewer chunks than threads, k that is and is not one of the unrolled widths
@pytest.mark.parametrize("dtype,d,k", [("fp32", 4104, 2), ("fp32", 1000, 3), ("bf16", 7176, 2), ("bf16", 2880, 5)])
@pytest.mark.parametrize("shared", [False, True])
def test_large_result_equals_its_parts(dtype, d, k, shared):
    act = torch.float32 if dtype == "fp32" else torch.bfloat16
    parts = 3
    n = (LINE // (d * act.itemsize) + 7 + parts) // parts  # tokens of a part
    T = parts * n
    assert T * d * act.itemsize > LINE > n * d * act.itemsize
    g = torch.Generator(device=H.DEV).manual_seed(d)
    Y = torch.empty(T * k, d, dtype=act, device=H.DEV).normal_(generator=g)
    w = torch.rand(T, k, device=H.DEV, generator=g)
    Y_sh = torch.empty(T, d, dtype=act, device=H.DEV).normal_(generator=g) if shared else None
    # the rows of a part's tokens lie in its own share of Y, in any order
    slot = torch.cat([torch.randperm(n * k, device=H.DEV, generator=g).to(torch.int32) for _ in range(parts)])

    def combine(lo, tokens):
        m = S.SemMoE(S.Config(T=tokens, d=d, E=8, k=k, F=8, D=1, dtype=dtype, cap=tokens))
        out = torch.full((tokens, d), 512.0, dtype=act, device=H.DEV)
        base = torch.arange(T, device=H.DEV).div(n, rounding_mode="floor").repeat_interleave(k).to(torch.int32) * (n * k)
        s = (slot + base)[lo * k:(lo + tokens) * k] - lo * k
        m.combine(Y[lo * k:(lo + tokens) * k], s.contiguous(), w[lo:lo + tokens], out,
                  Y_shared=None if Y_sh is None else Y_sh[lo:lo + tokens])
        return out

    whole = combine(0, T)
    for p in range(parts):
        assert torch.equal(whole[p * n:(p + 1) * n], combine(p * n, n)), p
    # and against the definition, in float64 on a few tokens of every part
    pick = torch.cat([torch.arange(p * n, p * n + 5) for p in range(parts)] + [torch.arange(T - 5, T)]).to(H.DEV)
    base = pick.div(n, rounding_mode="floor") * (n * k)
    rows = slot.view(T, k)[pick].long() + base[:, None]
    want = (w[pick][:, :, None].double() * Y[rows].double()).sum(1)
    if Y_sh is not None:
        want = want + Y_sh[pick].double()
    H.assert_close(H.to_np(whole[pick]), want.cpu().numpy(), dtype, "Out")
