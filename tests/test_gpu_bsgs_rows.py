"""Inner sums of a baby-step giant-step transform formed for several giant steps at a time."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [36, 32, 28])
@pytest.mark.parametrize("L,Kk,dnum,ell,batch,n1,n2", [
    (4, 2, 2, 4, 8, 3, 4),      # two halves of four
    (6, 2, 3, 5, 7, 3, 7),      # halves of four and three; four, two and one giant steps; a short last digit
    (4, 1, 4, 4, 5, 17, 4),     # halves of four and one; more baby steps than a launch takes
    (4, 4, 1, 3, 4, 2, 5),      # one digit: two ciphertexts at most
    (4, 4, 1, 4, 2, 3, 5),
    (5, 1, 5, 5, 8, 2, 4),      # more digits than there are sets of operands
    (3, 2, 2, 3, 3, 4, 3),
    (3, 2, 2, 1, 2, 2, 6),
    (4, 2, 2, 4, 1, 6, 4),
    (4, 2, 2, 4, 3, 2, 2),      # below the number of products from which the bundle holds c0
    (5, 2, 3, 5, 6, 3, 3),      # three giant steps one by one: two halves
])
def test_giant_steps_together(bits, L, Kk, dnum, ell, batch, n1, n2):
    st = Setup(12, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: torch.where(t >= 1 << 31, t - (1 << 32), t).to(torch.int32))
    every = list(range(L + Kk))
    baby = [pow(5, r, 2 * st.N) if r % 3 != 2 else 2 * st.N - pow(5, r, 2 * st.N) for r in range(n1)]
    baby[-1], baby[0] = baby[0], baby[-1]     # the identity is the last baby step
    giant = [pow(5, n1 * r + 1, 2 * st.N) for r in range(n2 - 1)] + [1]
    bkeys64, gkeys64 = ([st.uniform(71, 100 * i + r, (dnum, 2), every) for r in range(n)] for i, n in ((1, n1), (2, n2)))
    pts64 = [[None if (g + b) % 5 == 4 else st.uniform(71, 1000 + g * n1 + b, (), every) for b in range(n1)] for g in range(n2)]
    ct64 = st.uniform(71, 1, (batch, 2), list(range(ell)))
    fn, op = (K.ks_bsgs_linear_transform, K.KS_OP_BSGS) if wide else (K.ks_bsgs_linear_transform_u32, K.KS_OP_BSGS_U32)
    ws = workspace(st.ctx, op, ell, batch)
    guard = torch.full((ws.numel() + 4096,), -7, dtype=torch.int64, device="cuda")
    out = torch.full((batch, 2, ell, st.N), -1, dtype=torch.int64 if wide else torch.int32, device="cuda")
    K.ks_profile_enable(True)
    fn(st.ctx, word(ct64), ell, baby, [word(k) for k in bkeys64], giant, [word(k) for k in gkeys64],
       [[None if p is None else word(p) for p in row] for row in pts64], out, guard[:ws.numel()])
    ran = {r["kernel"] for r in K.ks_profile_report()}
    K.ks_profile_enable(False)
    one_digit = ell <= -(-L // dnum)
    assert ("rotate_mac_rows" in ran) == (n1 * n2 >= 6 and (batch <= 2 if one_digit else n2 >= 4 or batch <= 4))
    assert bool((guard[ws.numel():] == -7).all())
    got = out if wide else torch.where(out < 0, out.long() + (1 << 32), out.long())
    for b in sorted({0, min(3, batch - 1), batch - 1}):
        want = st.ref.bsgs_linear_transform(host(ct64[b:b + 1]), baby, [host(k) for k in bkeys64], giant, [host(k) for k in gkeys64],
                                            [[None if p is None else host(p) for p in row] for row in pts64], ell)
        assert_equal(got[b:b + 1], want)
