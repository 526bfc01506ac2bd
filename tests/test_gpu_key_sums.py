"""The forms of the inner product with the key: sums that meet the division in registers, and sums in memory."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [36, 28])
@pytest.mark.parametrize("logN,L,Kk,dnum,ell,batch", [
    (16, 5, 5, 1, 5, 6),      # one digit: no raised ciphertext limb
    (16, 6, 2, 3, 6, 8),
    (16, 7, 3, 3, 7, 6),      # short last digit
    (16, 7, 3, 3, 4, 9),      # a digit of one limb
    (15, 10, 3, 4, 10, 9),
    (15, 24, 4, 6, 23, 8),    # more digits than a wavefront for each takes
])
def test_sums_meet_the_division(bits, logN, L, Kk, dnum, ell, batch):
    """Every ciphertext of a batch as in a call of its own, whose sums go through memory; the first and the last against the reference."""
    st = Setup(logN, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: t.to(torch.int32))
    evk = word(st.uniform(61, 1, (dnum, 2), list(range(L + Kk))))
    d, cta, ctb = (word(st.uniform(61, 2 + i, lead, list(range(ell)))) for i, lead in enumerate(((batch,), (batch, 2), (batch, 2))))
    fns = (K.ks_keyswitch, K.hmult_relin_rescale, K.hmult_relin_rescale_merged) if wide else \
        (K.ks_keyswitch_u32, K.hmult_relin_rescale_u32, K.hmult_relin_rescale_merged_u32)
    refs = (st.ref.keyswitch, st.ref.hmult_relin_rescale, st.ref.hmult_relin_rescale_merged)
    for i, (fn, ref) in enumerate(zip(fns, refs)):
        args, limbs, op = ((d,), ell, K.KS_OP_KEYSWITCH) if i == 0 else ((cta, ctb), ell - 1, K.KS_OP_HMULT_RELIN_RESCALE)
        out = torch.full((batch, 2, limbs, st.N), -1, dtype=evk.dtype, device="cuda")
        K.ks_profile_enable(True)
        fn(st.ctx, *args, ell, evk, out, workspace(st.ctx, op, ell, batch))
        ran = {r["kernel"] for r in K.ks_profile_report()}
        K.ks_profile_enable(False)
        assert "rows_key_finish" in ran and "rows_moddown_finish" not in ran
        one, ws = torch.empty_like(out[:1]), workspace(st.ctx, op, ell, 1)
        for b in range(batch):
            fn(st.ctx, *(a[b:b + 1] for a in args), ell, evk, one, ws)
            assert torch.equal(out[b:b + 1], one), b
        for b in (0, batch - 1):
            assert_equal(out[b:b + 1].long(), ref(*(host(a[b:b + 1].long()) for a in args), host(evk.long()), ell))


@pytest.mark.parametrize("bits", [36, 28])
@pytest.mark.parametrize("logN,L,Kk,dnum,ell,batch,in_memory", [
    (15, 14, 14, 1, 2, 8, (True, True, True)),        # few limbs stay
    (16, 8, 8, 1, 3, 8, (False, True, True)),         # a multiplication leaves one less
    (16, 10, 2, 5, 10, 5, (True, True, True)),        # many digits
    (15, 18, 3, 6, 17, 6, (True, True, True)),
])
def test_calls_that_sums_in_memory_serve_better(bits, logN, L, Kk, dnum, ell, batch, in_memory):
    st = Setup(logN, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: t.to(torch.int32))
    evk = word(st.uniform(63, 1, (dnum, 2), list(range(L + Kk))))
    d, cta, ctb = (word(st.uniform(63, 2 + i, lead, list(range(ell)))) for i, lead in enumerate(((batch,), (batch, 2), (batch, 2))))
    fns = (K.ks_keyswitch, K.hmult_relin_rescale, K.hmult_relin_rescale_merged) if wide else \
        (K.ks_keyswitch_u32, K.hmult_relin_rescale_u32, K.hmult_relin_rescale_merged_u32)
    refs = (st.ref.keyswitch, st.ref.hmult_relin_rescale, st.ref.hmult_relin_rescale_merged)
    for i, (fn, ref) in enumerate(zip(fns, refs)):
        args, limbs, op = ((d,), ell, K.KS_OP_KEYSWITCH) if i == 0 else ((cta, ctb), ell - 1, K.KS_OP_HMULT_RELIN_RESCALE)
        out = torch.full((batch, 2, limbs, st.N), -1, dtype=evk.dtype, device="cuda")
        K.ks_profile_enable(True)
        fn(st.ctx, *args, ell, evk, out, workspace(st.ctx, op, ell, batch))
        ran = {r["kernel"] for r in K.ks_profile_report()}
        K.ks_profile_enable(False)
        assert ("rows_moddown_finish" in ran) == in_memory[i] and ("rows_key_finish" in ran) != in_memory[i]
        for b in (0, batch - 1):
            assert_equal(out[b:b + 1].long(), ref(*(host(a[b:b + 1].long()) for a in args), host(evk.long()), ell))


@pytest.mark.parametrize("bits", [36, 28])
@pytest.mark.parametrize("logN,L,Kk,dnum,ell,batch,split", [
    (12, 4, 2, 2, 4, 1, True),
    (12, 3, 3, 1, 3, 2, True),      # one digit
    (12, 7, 2, 4, 7, 3, True),      # as many digits as the form takes, a short last one
    (12, 7, 2, 4, 3, 14, True),
    (13, 5, 2, 3, 2, 1, True),      # launches padded to eight workgroups
    (14, 4, 4, 1, 1, 3, True),      # one limb, 240 workgroups
    (15, 8, 4, 3, 8, 2, True),      # 768 workgroups
    (15, 9, 4, 3, 9, 2, False),     # the form with a wavefront for everything
    (14, 4, 4, 1, 1, 9, False),
])
def test_a_wavefront_per_digit_and_component(bits, logN, L, Kk, dnum, ell, batch, split):
    st = Setup(logN, L, Kk, dnum, bits=bits)
    wide = bits == 36
    word = (lambda t: t) if wide else (lambda t: t.to(torch.int32))
    evk = word(st.uniform(62, 1, (dnum, 2), list(range(L + Kk))))
    d, cta, ctb = (word(st.uniform(62, 2 + i, lead, list(range(ell)))) for i, lead in enumerate(((batch,), (batch, 2), (batch, 2))))
    fns = (K.ks_keyswitch, K.hmult_relin_rescale, K.hmult_relin_rescale_merged) if wide else \
        (K.ks_keyswitch_u32, K.hmult_relin_rescale_u32, K.hmult_relin_rescale_merged_u32)
    refs = (st.ref.keyswitch, st.ref.hmult_relin_rescale, st.ref.hmult_relin_rescale_merged)
    for i, (fn, ref) in enumerate(zip(fns, refs)):
        if i and ell < 2:
            continue
        args, limbs, op = ((d,), ell, K.KS_OP_KEYSWITCH) if i == 0 else ((cta, ctb), ell - 1, K.KS_OP_HMULT_RELIN_RESCALE)
        out = torch.full((batch, 2, limbs, st.N), -1, dtype=evk.dtype, device="cuda")
        K.ks_profile_enable(True)
        fn(st.ctx, *args, ell, evk, out, workspace(st.ctx, op, ell, batch))
        ran = {r["kernel"] for r in K.ks_profile_report()}
        K.ks_profile_enable(False)
        assert ("rows_inner_product_split" in ran) == split and ("rows_inner_product" in ran) != split
        for b in sorted({0, batch - 1}):
            assert_equal(out[b:b + 1].long(), ref(*(host(a[b:b + 1].long()) for a in args), host(evk.long()), ell))
