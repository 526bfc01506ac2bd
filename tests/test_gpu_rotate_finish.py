"""Hoisted rotations whose sums meet the division in registers."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [36, 32, 28])
@pytest.mark.parametrize("logN,L,Kk,dnum,ell,batch,n_rot", [
    (16, 5, 2, 3, 5, 8, 4),       # two halves of four; a short last digit
    (16, 6, 3, 2, 6, 7, 4),       # halves of four and three
    (16, 7, 2, 4, 7, 6, 5),       # halves of four and two; a group of one rotation, whose sums go through memory
    (16, 9, 9, 1, 9, 5, 6),       # a launch for four and one for one; one digit
    (15, 14, 2, 7, 14, 7, 5),     # seven digits
    (16, 37, 13, 3, 37, 1, 5),    # more workgroups than are resident: rotations of a group shared among them
    (16, 9, 3, 3, 9, 4, 4),
    (16, 11, 4, 3, 10, 3, 5),
    (15, 17, 6, 3, 17, 2, 8),     # rotations of a group shared among workgroups
    (16, 24, 8, 3, 24, 1, 16),
    (14, 14, 5, 3, 13, 8, 14),
    (13, 24, 8, 3, 23, 8, 16),
])
def test_rotations_meet_the_division(bits, logN, L, Kk, dnum, ell, batch, n_rot):
    st = Setup(logN, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: torch.where(t >= 1 << 31, t - (1 << 32), t).to(torch.int32))
    fn, op = (K.ks_rotate_hoisted, K.KS_OP_ROTATE_HOISTED) if wide else (K.ks_rotate_hoisted_u32, K.KS_OP_ROTATE_HOISTED_U32)
    galois = [pow(5, r + 1, 2 * st.N) if r % 3 else 2 * st.N - pow(5, r + 1, 2 * st.N) for r in range(n_rot)]
    keys64 = [st.uniform(81, 10 + r, (dnum, 2), list(range(L + Kk))) for r in range(n_rot)]
    ct64 = st.uniform(81, 1, (batch, 2), list(range(ell)))
    keys, ct = [word(k) for k in keys64], word(ct64)
    words = K.ks_workspace_bytes(st.ctx, op, ell, batch, n_rot) // 8
    ws = torch.full((words + 4096,), -7, dtype=torch.int64, device="cuda")
    out = torch.full((batch, n_rot, 2, ell, st.N), -1, dtype=ct.dtype, device="cuda")
    K.ks_profile_enable(True)
    fn(st.ctx, ct, ell, galois, keys, out, ws[:words])
    ran = {r["kernel"] for r in K.ks_profile_report()}
    K.ks_profile_enable(False)
    assert "rotate_finish" in ran
    assert bool((ws[words:] == -7).all())
    one, small = torch.empty((1, 1, 2, ell, st.N), dtype=ct.dtype, device="cuda"), workspace(st.ctx, op, ell, 1, 1)
    for b in range(batch):
        for r in range(n_rot):      # a rotation of one ciphertext: sums in memory
            fn(st.ctx, ct[b:b + 1], ell, galois[r:r + 1], keys[r:r + 1], one, small)
            assert torch.equal(out[b:b + 1, r:r + 1], one), (b, r)
    got = out[-1:] if wide else torch.where(out[-1:] < 0, out[-1:].long() + (1 << 32), out[-1:].long())
    want = st.ref.rotate_hoisted(host(ct64[-1:]), galois[-2:], [host(k) for k in keys64[-2:]], ell)
    assert_equal(got[:, -2:], want)


@pytest.mark.parametrize("bits", [36, 28])
@pytest.mark.parametrize("logN,L,Kk,dnum,ell,batch,n_rot,meets", [
    (14, 10, 2, 5, 10, 8, 8, {}),             # below N = 2^15: few wavefronts, many digits
    (14, 15, 3, 5, 14, 7, 8, {}),             # many digits
    (14, 14, 5, 3, 13, 8, 10, {}),            # three digits, few wavefronts
    (13, 24, 8, 3, 23, 8, 12, {}),
    (16, 7, 7, 1, 7, 5, 6, {}),               # five ciphertexts, few wavefronts
    (16, 6, 1, 6, 6, 6, 4, {}),               # six ciphertexts, six digits
    (15, 12, 3, 4, 12, 5, 8, {}),             # five ciphertexts: more than three digits, or few wavefronts
    (15, 7, 3, 3, 7, 5, 8, {}),
    (15, 9, 3, 3, 9, 5, 8, {36, 28}),
])
def test_forms_that_sums_in_memory_serve_better(bits, logN, L, Kk, dnum, ell, batch, n_rot, meets):
    st = Setup(logN, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: t.to(torch.int32))
    fn, op = (K.ks_rotate_hoisted, K.KS_OP_ROTATE_HOISTED) if wide else (K.ks_rotate_hoisted_u32, K.KS_OP_ROTATE_HOISTED_U32)
    galois = [pow(5, r + 1, 2 * st.N) for r in range(n_rot)]
    keys64 = [st.uniform(82, 10 + r, (dnum, 2), list(range(L + Kk))) for r in range(n_rot)]
    ct64 = st.uniform(82, 1, (batch, 2), list(range(ell)))
    out = torch.full((batch, n_rot, 2, ell, st.N), -1, dtype=torch.int64 if wide else torch.int32, device="cuda")
    K.ks_profile_enable(True)
    fn(st.ctx, word(ct64), ell, galois, [word(k) for k in keys64], out, workspace(st.ctx, op, ell, batch, n_rot))
    ran = {r["kernel"] for r in K.ks_profile_report()}
    K.ks_profile_enable(False)
    assert ("rotate_finish" in ran) == (bits in meets) and ("rows_moddown_finish" in ran) == (bits not in meets)
    want = st.ref.rotate_hoisted(host(ct64[-1:]), galois[-2:], [host(k) for k in keys64[-2:]], ell)
    assert_equal(out[-1:, -2:].long(), want)
