"""Batches that a key-switch or a multiplication takes in one pass or several: every ciphertext as in a call of its own, and nothing
written behind the workspace that was asked for."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host, workspace

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


@pytest.mark.parametrize("logN,L,Kk,dnum,batch,passes", [
    (12, 5, 2, 3, 9, 1),       # vector conversions
    (14, 12, 4, 3, 29, 3),
    (15, 20, 7, 3, 15, 2),     # matrix cores, eight and seven
    (16, 24, 8, 3, 17, 2),     # 16-column tiles, nine and eight
    (16, 24, 8, 3, 15, 2),     # eight and seven: 16- and 8-column tiles
    (16, 16, 4, 4, 27, 2),     # fourteen and thirteen, vector conversions
])
def test_passes_of_a_key_switch(logN, L, Kk, dnum, batch, passes):
    """The number of passes, with either conversion kernel; every ciphertext as in a call of its own, the last one of each pass against the
    reference."""
    st = Setup(logN, L, Kk, dnum)
    evk, d = st.uniform(53, 1, (dnum, 2), list(range(L + Kk))), st.uniform(53, 2, (batch,), list(range(L)))
    out = torch.full((batch, 2, L, st.N), -1, dtype=torch.int64, device="cuda")
    ws = workspace(st.ctx, K.KS_OP_KEYSWITCH, L, batch)
    K.ks_profile_enable(True)
    K.ks_keyswitch(st.ctx, d, L, evk, out, ws)
    launches = {r["kernel"]: r["launches"] for r in K.ks_profile_report()}
    K.ks_profile_enable(False)
    assert launches.get("rows_inner_product", 0) + launches.get("rows_inner_product_split", 0) == passes
    one = torch.empty_like(out[:1])
    for b in range(batch):
        K.ks_keyswitch(st.ctx, d[b:b + 1], L, evk, one, ws)
        assert torch.equal(out[b:b + 1], one), b
    size = 8 if passes == -(-batch // 8) else -(-batch // passes)
    for last in sorted({min((p + 1) * size, batch) - 1 for p in range(passes)}):
        assert_equal(out[last:last + 1], st.ref.keyswitch(host(d[last:last + 1]), host(evk), L))


@pytest.mark.parametrize("logN,L,Kk,dnum,batch,passes", [(14, 9, 3, 3, 27, 3), (15, 20, 7, 3, 13, 1), (16, 12, 6, 2, 15, 2)])
def test_passes_of_a_multiplication(logN, L, Kk, dnum, batch, passes):
    st = Setup(logN, L, Kk, dnum)
    q = list(range(L))
    cta, ctb, rlk = st.uniform(54, 1, (batch, 2), q), st.uniform(54, 2, (batch, 2), q), st.uniform(54, 3, (dnum, 2), list(range(L + Kk)))
    ws = workspace(st.ctx, K.KS_OP_HMULT_RELIN_RESCALE, L, batch)
    for fn, ref in ((K.hmult_relin_rescale, st.ref.hmult_relin_rescale), (K.hmult_relin_rescale_merged, st.ref.hmult_relin_rescale_merged)):
        out = torch.full((batch, 2, L - 1, st.N), -1, dtype=torch.int64, device="cuda")
        K.ks_profile_enable(True)
        fn(st.ctx, cta, ctb, L, rlk, out, ws)
        launches = {r["kernel"]: r["launches"] for r in K.ks_profile_report()}
        K.ks_profile_enable(False)
        assert launches["tensor_inv_rows"] == passes
        one = torch.empty_like(out[:1])
        for b in range(batch):
            fn(st.ctx, cta[b:b + 1], ctb[b:b + 1], L, rlk, one, ws)
            assert torch.equal(out[b:b + 1], one), b
        assert_equal(out[-1:], ref(host(cta[-1:]), host(ctb[-1:]), host(rlk), L))


@pytest.mark.parametrize("bits", [36, 28])
@pytest.mark.parametrize("L,Kk,dnum,ell", [(6, 2, 3, 6), (6, 6, 1, 2), (5, 2, 4, 5)])
@pytest.mark.parametrize("batch,n_rot", [(1, 5), (1, 16), (3, 8), (8, 7), (8, 17), (9, 20)])
def test_rotations_in_groups(bits, L, Kk, dnum, ell, batch, n_rot):
    st = Setup(12, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: t.to(torch.int32))
    fn, op = (K.ks_rotate_hoisted, K.KS_OP_ROTATE_HOISTED) if wide else (K.ks_rotate_hoisted_u32, K.KS_OP_ROTATE_HOISTED_U32)
    galois = [pow(5, r + 1, 2 * st.N) if r % 3 else 2 * st.N - pow(5, r + 1, 2 * st.N) for r in range(n_rot)]
    keys = [word(st.uniform(52, 10 + r, (dnum, 2), list(range(L + Kk)))) for r in range(n_rot)]
    ct = word(st.uniform(52, 1, (batch, 2), list(range(ell))))
    words = K.ks_workspace_bytes(st.ctx, op, ell, batch, n_rot) // 8
    buf = torch.full((words + GUARD,), -7, dtype=torch.int64, device="cuda")
    out = torch.full((batch, n_rot, 2, ell, st.N), -1, dtype=ct.dtype, device="cuda")
    fn(st.ctx, ct, ell, galois, keys, out, buf[:words])
    one, ws = torch.empty((batch, 1, 2, ell, st.N), dtype=ct.dtype, device="cuda"), workspace(st.ctx, op, ell, batch, 1)
    for r in range(n_rot):
        fn(st.ctx, ct, ell, galois[r:r + 1], keys[r:r + 1], one, ws)
        assert torch.equal(out[:, r:r + 1], one), r
    assert bool((buf[words:] == -7).all())
