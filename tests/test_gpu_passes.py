"""Batches that a key-switch or a multiplication takes in one pass or several: every ciphertext as in a call of its own, and nothing
written behind the workspace that was asked for."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, workspace

pytestmark = pytest.mark.gpu

GUARD = 4096


@pytest.mark.parametrize("bits", [36, 28])
@pytest.mark.parametrize("L,Kk,dnum,ell", [(6, 2, 3, 6), (6, 2, 3, 2), (6, 6, 1, 5), (5, 2, 4, 5)])
@pytest.mark.parametrize("batch", [8, 9, 12, 13, 14, 15, 16, 27])
def test_batches_in_passes(bits, L, Kk, dnum, ell, batch):
    st = Setup(12, L, Kk, dnum, bits=bits)
    q = list(range(ell))
    evk = st.uniform(51, 1, (dnum, 2), list(range(L + Kk)))
    d, cta, ctb = st.uniform(51, 2, (batch,), q), st.uniform(51, 3, (batch, 2), q), st.uniform(51, 4, (batch, 2), q)
    for op, fn, args, limbs in ((K.KS_OP_KEYSWITCH, K.ks_keyswitch, (d,), ell),
                                (K.KS_OP_HMULT_RELIN_RESCALE, K.hmult_relin_rescale, (cta, ctb), ell - 1)):
        words = K.ks_workspace_bytes(st.ctx, op, ell, batch, 0) // 8
        buf = torch.full((words + GUARD,), -7, dtype=torch.int64, device="cuda")
        out = torch.full((batch, 2, limbs, st.N), -1, dtype=torch.int64, device="cuda")
        fn(st.ctx, *args, ell, evk, out, buf[:words])
        one, ws = torch.empty_like(out[:1]), workspace(st.ctx, op, ell, 1)
        for b in range(batch):
            fn(st.ctx, *(a[b:b + 1] for a in args), ell, evk, one, ws)
            assert torch.equal(out[b:b + 1], one), b
        assert bool((buf[words:] == -7).all())
