"""The rotation gathers lay the sources of the ciphertexts of a call side by side, up to eight at a time: every group size and a batch
of more than one group, with Galois elements of both kinds (powers of 5 permute the slots inside each half of a limb, -5^r swaps
the halves), bit-exact against the plain-C reference, in both word sizes."""

import pytest
import torch

import ks_inputs
import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host, workspace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[12, 13], ids=lambda n: "N2^%d" % n)
def st(request):
    return Setup(request.param, 5, 2, 3)


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11])
def test_every_group_size(st, batch):
    ell, all_ids = 4, list(range(st.L + st.K))
    g = ks_inputs.galois_elements(st.logN, 2)
    galois = [g[0], 2 * st.N - g[1], 2 * st.N - 1]
    ct = st.uniform(4001, batch, (batch, 2), list(range(ell)))
    keys = [st.uniform(4001, 50 + r, (st.ctx.dnum, 2), all_ids) for r in range(3)]
    pts = [st.uniform(4001, 70 + r, (), all_ids) for r in range(4)]
    ws = workspace(st.ctx, K.KS_OP_ROTATE_HOISTED, ell, batch, 4)
    out = torch.empty((batch, 3, 2, ell, st.N), dtype=torch.int64, device="cuda")
    K.ks_rotate_hoisted(st.ctx, ct, ell, galois, keys, out, ws)
    assert_equal(out, st.ref.rotate_hoisted(host(ct), galois, [host(k) for k in keys], ell))
    mac = torch.empty((batch, 2, ell, st.N), dtype=torch.int64, device="cuda")
    K.ks_rotate_mac_hoisted(st.ctx, ct, ell, [galois[0], 1] + galois[1:], [keys[0], None] + keys[1:], pts, mac, ws)
    assert_equal(mac, st.ref.rotate_mac_hoisted(host(ct), [galois[0], 1] + galois[1:], [host(keys[0]), None] + [host(k) for k in keys[1:]],
                                                [host(w) for w in pts], ell))


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 6, 7, 8, 13])
def test_every_group_size_words32(batch):
    st = Setup(12, 5, 2, 3, bits=28)
    ell, all_ids = 5, list(range(st.L + st.K))
    g = ks_inputs.galois_elements(st.logN, 1)
    galois = [2 * st.N - g[0], g[0]]
    word = lambda t: t.to(torch.int32)
    ct = st.uniform(4002, batch, (batch, 2), list(range(ell)))
    keys = [st.uniform(4002, 50 + r, (st.ctx.dnum, 2), all_ids) for r in range(2)]
    pts = [st.uniform(4002, 70 + r, (), all_ids) for r in range(3)]
    ws = workspace(st.ctx, K.KS_OP_ROTATE_HOISTED_U32, ell, batch, 3)
    out = torch.empty((batch, 2, 2, ell, st.N), dtype=torch.int32, device="cuda")
    K.ks_rotate_hoisted_u32(st.ctx, word(ct), ell, galois, [word(k) for k in keys], out, ws)
    assert_equal(out.to(torch.int64), st.ref.rotate_hoisted(host(ct), galois, [host(k) for k in keys], ell))
    mac = torch.empty((batch, 2, ell, st.N), dtype=torch.int32, device="cuda")
    K.ks_rotate_mac_hoisted_u32(st.ctx, word(ct), ell, [1] + galois, [None] + [word(k) for k in keys], [word(w) for w in pts], mac, ws)
    assert_equal(mac.to(torch.int64), st.ref.rotate_mac_hoisted(host(ct), [1] + galois, [None] + [host(k) for k in keys], [host(w) for w in pts], ell))


@pytest.mark.parametrize("n_rot", [1, 5, 6])
@pytest.mark.parametrize("bits,batch", [(36, 1), (36, 3), (36, 8), (28, 2), (28, 7)])
def test_addend_from_the_ciphertexts_and_from_the_bundle(bits, batch, n_rot):
    """Up to five rotations gather c0 from the ciphertexts, six read a copy; an identity and a unit plaintext among them."""
    st = Setup(12, 5, 2, 3, bits=bits)
    ell, all_ids = 4, list(range(st.L + st.K))
    g = ks_inputs.galois_elements(st.logN, n_rot)
    galois = [2 * st.N - g[0]] + [1 if r == 2 else g[r] for r in range(1, n_rot)]
    ct = st.uniform(4003, batch, (batch, 2), list(range(ell)))
    keys = [None if e == 1 else st.uniform(4003, 50 + r, (st.ctx.dnum, 2), all_ids) for r, e in enumerate(galois)]
    pts = [None if r == 3 else st.uniform(4003, 70 + r, (), all_ids) for r in range(n_rot)]
    want = st.ref.rotate_mac_hoisted(host(ct), galois, [k if k is None else host(k) for k in keys],
                                     [w if w is None else host(w) for w in pts], ell)
    word = (lambda t: t) if bits == 36 else (lambda t: t if t is None else t.to(torch.int32))
    op, fn = (K.KS_OP_ROTATE_HOISTED, K.ks_rotate_mac_hoisted) if bits == 36 else (K.KS_OP_ROTATE_HOISTED_U32, K.ks_rotate_mac_hoisted_u32)
    out = word(torch.zeros((batch, 2, ell, st.N), dtype=torch.int64, device="cuda"))
    fn(st.ctx, word(ct), ell, galois, [word(k) for k in keys], [word(w) for w in pts], out, workspace(st.ctx, op, ell, batch, n_rot))
    assert_equal(out.to(torch.int64), want)


@pytest.mark.parametrize("bits,op", [(36, K.KS_OP_ROTATE_HOISTED), (28, K.KS_OP_ROTATE_HOISTED_U32)])
def test_workspace_holds_no_ciphertexts_beyond_the_batch(bits, op):
    """Everything a rotation keeps is per ciphertext but the words of the bits above 32, of which two to eight ciphertexts share one
    of 1, 2 or 4 bytes (0.8 bytes a residue for five, 0.5 for eight)."""
    ctx = Setup(12, 5, 2, 3, bits=bits).ctx
    one = K.ks_workspace_bytes(ctx, op, 5, 1, 1)
    for batch in range(2, 9):
        assert K.ks_workspace_bytes(ctx, op, 5, batch, 1) <= batch * one
