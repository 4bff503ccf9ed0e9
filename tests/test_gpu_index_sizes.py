"""reshuffle and dispatch index where their kernels change form: one workgroup of 256, 512 or 1024 threads, two launches, one
kernel per phase; 4, 8 and 16 registers for a token's experts; ids in quads or one by one (k, alignment); the send matrix
in quads or not.  All outputs bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2503_04398_amd as S
from oracle import semmoe_oracle as O
from tests import harness as H

pytestmark = pytest.mark.gpu


def _odd(a):
    """the same values in device memory that starts 4 bytes off a 16-byte boundary"""
    flat = torch.empty(a.size + 1, dtype=torch.int32, device=H.DEV)[1:]
    flat.copy_(torch.from_numpy(np.ascontiguousarray(a)).reshape(-1))
    return flat.view(a.shape)


def _check_index(T, E, D, k, odd):
    r = np.random.default_rng(T + E + k)
    ids = np.argsort(r.random((T, E)) - 0.4 * (np.arange(E)[None, :] < E // 2), axis=1)[:, :k].astype(np.int32)
    e2r = r.permutation(np.repeat(np.arange(D), E // D)).astype(np.int32)
    phys = np.argsort(np.argsort(e2r, kind="stable"), kind="stable").astype(np.int32)
    cap = -(-T // D)
    m = S.SemMoE(S.Config(T=T, d=8, E=E, k=k, F=8, D=D, cap=cap), device=H.DEV)
    new = lambda *shape: (_odd if odd else H.to_dev)(np.full(shape, -7, dtype=np.int32))
    ids_d, e2r_d, phys_d = ((_odd if odd else H.to_dev)(a) for a in (ids, e2r, phys))
    want = O.reshuffle(ids, e2r, D, cap)
    wd = O.dispatch(None, ids, want[0], want[2], phys, D)
    for path in (-1, 1, 2, 3):
        print("index", dict(T=T, E=E, D=D, k=k, odd=odd, path=path), flush=True)
        rs = [new(T), new(T), new(T), new(D)]
        dp = dict(slot_of_pair=new(T * k), pair_of_slot=new(T * k), expert_offsets=new(E + 1), rank_offsets=new(D + 1),
                  send_matrix=new(D, D))
        remote = torch.full((1,), -7, dtype=torch.int64, device=H.DEV)
        m.set_tuning(3, path)
        try:
            m.reshuffle(ids_d, e2r_d, *rs)
            m.dispatch_index(ids_d, rs[0], rs[1], phys_d, *dp.values(), remote)
            torch.cuda.synchronize()
        finally:
            m.set_tuning(3, -1)
        for g, w, name in zip(rs, want, ("token_rank", "shf", "inv_shf", "rank_count")):
            assert (H.to_np(g) == w).all(), name
        for name, g in dp.items():
            assert (H.to_np(g) == wd[name]).all(), name
        assert int(remote.item()) == int(wd["remote_pairs"])


@pytest.mark.parametrize("T", [1, 255, 256, 257, 511, 512, 513, 1025, 2047])
@pytest.mark.parametrize("E,D,k", [(6, 3, 3), (16, 4, 4), (32, 8, 8), (40, 5, 12), (128, 64, 16), (512, 32, 8), (510, 2, 5)])
@pytest.mark.parametrize("odd", [False, True])
def test_index_at_the_edges_of_its_forms(T, E, D, k, odd):
    _check_index(T, E, D, k, odd)


# few pairs: one workgroup of 1024 threads up to 1024 tokens (one expert a token) or 768 (two), and where it is asked for (path 2)
@pytest.mark.parametrize("T", [513, 768, 769, 1000, 1024, 1025])
@pytest.mark.parametrize("E,D,k", [(8, 2, 1), (510, 2, 1), (512, 64, 2), (6, 3, 2), (12, 4, 4), (512, 64, 4)])
@pytest.mark.parametrize("odd", [False, True])
def test_index_of_few_pairs(T, E, D, k, odd):
    _check_index(T, E, D, k, odd)
