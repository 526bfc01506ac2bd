"""The two base-conversion kernel families -- vector fp64 accumulation and int8 matrix cores (one or three targets per
lane half) -- forced through the context option, each against the plain-C reference, bit-exact on every residue: the
standalone conversion, and the fused conversion + column transform inside ks_keyswitch / hmult_relin_rescale_merged.
Source counts 1 .. 17 cover every operand-slot shape of the matrix-core tables (1, 2 or 3 instructions per position, 1 to 9
sources a lane half), including digits of different sizes in one launch."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host, workspace

pytestmark = pytest.mark.gpu

KERNELS = [(1, 0), (2, 1), (2, 3)]     # (KS_OPT_BCONV_KERNEL, KS_OPT_BCONV_TARGETS)


def _select(st, kernel, targets):
    st.ctx.set_option(K.KS_OPT_BCONV_KERNEL, kernel)
    st.ctx.set_option(K.KS_OPT_BCONV_TARGETS, targets)


@pytest.fixture(scope="module")
def small():
    return Setup(12, 9, 3, 3)        # digits of 3 limbs; 12 moduli to draw conversions from


@pytest.fixture(scope="module")
def boot():
    return Setup(16, 24, 8, 3)


@pytest.mark.parametrize("kernel,targets", KERNELS)
@pytest.mark.parametrize("which,src,dst,batch", [
    ("small", [4], [0, 11], 2),
    ("small", [0, 1], [2, 3, 4, 5, 6, 7, 8], 1),
    ("small", [9, 10, 11], list(range(9)), 3),
    ("small", [0, 2, 4, 6, 8], [1, 3, 5, 7, 9, 10, 11], 1),
    ("small", list(range(7)), [7, 8, 9, 10, 11], 2),
    ("small", list(range(1, 11)), [0, 11], 1),
    ("boot", list(range(8)), list(range(8, 32)), 2),
    ("boot", list(range(24, 32)), list(range(24)), 1),
    ("boot", list(range(13)), list(range(13, 32)), 1),
    ("boot", list(range(16, 32)), [0, 5, 15], 1),
])
def test_standalone_conversion(kernel, targets, which, src, dst, batch, request):
    st = request.getfixturevalue(which)
    _select(st, kernel, targets)
    x = st.uniform(31, 2, (batch,), src)
    out = torch.full((batch, len(dst), st.N), -1, dtype=torch.int64, device="cuda")
    K.bconv_prepare(st.ctx, src, dst)
    K.bconv(st.ctx, x, src, out, dst)
    assert_equal(out, st.ref.bconv(host(x), src, dst))


def test_standalone_conversion_extreme_residues(boot):
    """All-zero and all (modulus - 1) sources: the ends of the byte-cutting range."""
    src, dst = list(range(8)), list(range(8, 32))
    x = torch.zeros((2, 8, boot.N), dtype=torch.int64, device="cuda")
    for i, m in enumerate(src):
        x[1, i, :] = boot.moduli[m] - 1
    K.bconv_prepare(boot.ctx, src, dst)
    for kernel, targets in KERNELS:
        _select(boot, kernel, targets)
        out = torch.full((2, 24, boot.N), -1, dtype=torch.int64, device="cuda")
        K.bconv(boot.ctx, x, src, out, dst)
        assert_equal(out, boot.ref.bconv(host(x), src, dst))
        assert int(out[0].abs().max()) == 0


@pytest.mark.parametrize("kernel,targets", KERNELS)
@pytest.mark.parametrize("logN,L,Kk,dnum,ells", [
    (12, 5, 2, 3, (5, 4, 1)),        # digits 2 / 2 / 1
    (12, 9, 3, 3, (9, 7)),           # 3-limb digits, short last digit at level 7
    (12, 6, 6, 1, (6, 5)),           # one digit of 6 (and 7 sources in the merged ModDown)
    (13, 4, 2, 2, (4,)),
    (14, 6, 3, 2, (6,)),
    (15, 4, 2, 2, (3,)),
    (16, 24, 8, 3, (24, 17)),        # configuration 2; level 17 has digits 8 / 8 / 1
    (16, 13, 13, 1, (13,)),          # 13 sources: three matrix instructions per position
])
def test_fused_conversion_in_keyswitch(kernel, targets, logN, L, Kk, dnum, ells):
    st = Setup(logN, L, Kk, dnum)
    _select(st, kernel, targets)
    evk = st.uniform(32, 2, (dnum, 2), list(range(L + Kk)))
    for ell in ells:
        batch = 1 if logN == 16 else 3
        d = st.uniform(32, 10 + ell, (batch,), list(range(ell)))
        out = torch.full((batch, 2, ell, st.N), -1, dtype=torch.int64, device="cuda")
        K.ks_keyswitch(st.ctx, d, ell, evk, out, workspace(st.ctx, K.KS_OP_KEYSWITCH, ell, batch))
        assert_equal(out, st.ref.keyswitch(host(d), host(evk), ell))


@pytest.mark.parametrize("kernel,targets", KERNELS)
def test_fused_conversion_in_merged_multiplication(kernel, targets):
    st = Setup(12, 6, 6, 1)
    _select(st, kernel, targets)
    rlk = st.uniform(33, 3, (1, 2), list(range(12)))
    for ell in (6, 3):
        cta = st.uniform(33, 20 + ell, (2, 2), list(range(ell)))
        ctb = st.uniform(33, 40 + ell, (2, 2), list(range(ell)))
        out = torch.full((2, 2, ell - 1, st.N), -1, dtype=torch.int64, device="cuda")
        K.hmult_relin_rescale_merged(st.ctx, cta, ctb, ell, rlk, out, workspace(st.ctx, K.KS_OP_HMULT_RELIN_RESCALE, ell, 2))
        assert_equal(out, st.ref.hmult_relin_rescale_merged(host(cta), host(ctb), host(rlk), ell))


def test_option_values_are_checked(small):
    with pytest.raises(K.KsError):
        small.ctx.set_option(K.KS_OPT_BCONV_KERNEL, 3)
    with pytest.raises(K.KsError):
        small.ctx.set_option(99, 0)
    small.ctx.set_option(K.KS_OPT_BCONV_KERNEL, 0)
    small.ctx.set_option(K.KS_OPT_BCONV_TARGETS, 0)


@pytest.mark.parametrize("kernel,targets", KERNELS)
def test_rescale_with_the_most_sources(kernel, targets):
    """K = 16: the conversion of a multiplication's division by P and the rescale takes seventeen sources, the last one signed."""
    st = Setup(12, 17, 16, 2)
    _select(st, kernel, targets)
    for ell, batch in ((17, 2), (2, 3)):
        cta, ctb = (st.uniform(35 + i, 1, (batch, 2), list(range(ell))) for i in range(2))
        rlk = st.uniform(37, 2, (st.ctx.dnum, 2), list(range(33)))
        out = torch.empty((batch, 2, ell - 1, st.N), dtype=torch.int64, device="cuda")
        K.hmult_relin_rescale(st.ctx, cta, ctb, ell, rlk, out, workspace(st.ctx, K.KS_OP_HMULT_RELIN_RESCALE, ell, batch))
        assert_equal(out, st.ref.hmult_relin_rescale(host(cta), host(ctb), host(rlk), ell))


@pytest.mark.parametrize("merged", [False, True])
def test_rescale_with_many_sources_and_several_polynomials_a_workgroup(merged):
    """Nine sources a lane half, twelve pairs at N = 2^16: a workgroup of the last conversion takes five polynomials in turn; the signed
    source of the rescale (K = 16) and the unsigned one of the merged form (K = 15)."""
    Kk = 15 if merged else 16
    st, batch = Setup(16, Kk, Kk, 1), 12
    cta, ctb = (st.uniform(48 + i, 1, (batch, 2), list(range(Kk))) for i in range(2))
    rlk = st.uniform(50, 2, (1, 2), list(range(2 * Kk)))
    out = torch.full((batch, 2, Kk - 1, st.N), -1, dtype=torch.int64, device="cuda")
    fn, ref = (K.hmult_relin_rescale_merged, st.ref.hmult_relin_rescale_merged) if merged else (K.hmult_relin_rescale, st.ref.hmult_relin_rescale)
    ws = workspace(st.ctx, K.KS_OP_HMULT_RELIN_RESCALE, Kk, batch)
    fn(st.ctx, cta, ctb, Kk, rlk, out, ws)
    one = torch.empty_like(out[:1])
    for b in range(batch):
        fn(st.ctx, cta[b:b + 1], ctb[b:b + 1], Kk, rlk, one, ws)
        assert torch.equal(out[b:b + 1], one), b
    assert_equal(out[-1:], ref(host(cta[-1:]), host(ctb[-1:]), host(rlk), Kk))


@pytest.mark.parametrize("logN,L,Kk,dnum", [(12, 5, 2, 3), (13, 9, 3, 3), (15, 2, 1, 2), (15, 9, 3, 3), (16, 10, 5, 2), (16, 14, 7, 2)])
def test_every_number_of_targets(logN, L, Kk, dnum):
    """KS_OPT_BCONV_TARGETS: all numbers of targets that either fused kernel can be set to."""
    st = Setup(logN, L, Kk, dnum)
    evk, d = st.uniform(51, 1, (dnum, 2), list(range(L + Kk))), st.uniform(51, 2, (2,), list(range(L)))
    want = st.ref.keyswitch(host(d), host(evk), L)
    for kernel, targets in ((1, 1), (1, 2), (1, 3), (1, 4), (2, 1), (2, 3)):
        _select(st, kernel, targets)
        out = torch.full((2, 2, L, st.N), -1, dtype=torch.int64, device="cuda")
        K.ks_keyswitch(st.ctx, d, L, evk, out, workspace(st.ctx, K.KS_OP_KEYSWITCH, L, 2))
        assert_equal(out, want)


@pytest.mark.parametrize("batch", [31, 32, 33, 127, 128, 129])
def test_standalone_conversion_positions_per_wavefront(small, batch):
    """N = 2^12 has 32 wavefront tiles of 128 positions per polynomial: 1, 2 and 4 position groups per wavefront, at the batch sizes
    where the count changes."""
    src, dst = [0, 2, 4, 6, 8], [1, 3, 5, 7, 9, 10, 11]
    x = small.uniform(41, batch, (batch,), src)
    out = torch.full((batch, len(dst), small.N), -1, dtype=torch.int64, device="cuda")
    K.bconv_prepare(small.ctx, src, dst)
    K.bconv(small.ctx, x, src, out, dst)
    assert_equal(out, small.ref.bconv(host(x), src, dst))


@pytest.mark.parametrize("bits,n_src", [(36, 7), (36, 13), (28, 8), (28, 16)])
@pytest.mark.parametrize("batch", [3, 32, 128])
def test_standalone_conversion_positions_and_instructions(bits, n_src, batch):
    """1, 2 and 4 position groups with two and three matrix instructions per position, both word sizes."""
    st = Setup(12, 18, 3, 3, bits=bits)
    src, dst = list(range(n_src)), [17, 18, 20, 16, 19]
    x = st.uniform(46, batch, (batch,), src)
    K.bconv_prepare(st.ctx, src, dst)
    dtype = torch.int64 if bits == 36 else torch.int32
    out = torch.full((batch, len(dst), st.N), -1, dtype=dtype, device="cuda")
    (K.bconv if bits == 36 else K.bconv_u32)(st.ctx, x.to(dtype), src, out, dst)
    assert_equal(out.to(torch.int64), st.ref.bconv(host(x), src, dst))


@pytest.mark.parametrize("batch", [3, 32, 128])
def test_standalone_conversion_positions_per_wavefront_words32(batch):
    st = Setup(12, 9, 3, 3, bits=28)
    _select(st, 2, 0)
    src, dst = [0, 2, 4, 6, 8], [1, 3, 5, 7, 9, 10, 11]
    x = st.uniform(42, batch, (batch,), src)
    out = torch.full((batch, len(dst), st.N), -1, dtype=torch.int32, device="cuda")
    K.bconv_prepare(st.ctx, src, dst)
    K.bconv_u32(st.ctx, x.to(torch.int32), src, out, dst)
    assert_equal(out.to(torch.int64), st.ref.bconv(host(x), src, dst))


@pytest.mark.parametrize("logN,L,Kk,dnum,batch", [
    (16, 16, 4, 4, 8),    # 4 sources: vector or 8 columns; tiles of 16 columns with 6, 8, 12 and 13 sources (3, 4, 6 and 7 a lane half)
    (16, 24, 6, 4, 8),
    (16, 24, 8, 3, 9),    # 16-column tiles, all nine in one pass
    (16, 24, 8, 3, 15),   # passes of eight and seven: 16- and 8-column tiles in one call
    (16, 36, 12, 3, 8),
    (16, 39, 13, 3, 8),
    (16, 30, 15, 2, 1),   # nine a lane half: one target per half, three in tiles of 8 and of 16 columns
    (16, 30, 15, 2, 8),
    (16, 30, 15, 2, 12),
    (15, 20, 7, 3, 5),    # N = 2^15: one target per lane half, and three
    (15, 30, 15, 2, 5),
])
def test_conversion_tiles_of_large_launches(logN, L, Kk, dnum, batch):
    """The kernel that is chosen, the vector kernel and the matrix cores against each other on every residue, and against the
    reference on the last item."""
    st = Setup(logN, L, Kk, dnum)
    evk = st.uniform(43, 1, (dnum, 2), list(range(L + Kk)))
    d = st.uniform(43, 2, (batch,), list(range(L)))
    ws = workspace(st.ctx, K.KS_OP_KEYSWITCH, L, batch)
    out = []
    for kernel in (0, 1, 2):
        _select(st, kernel, 0)
        out.append(torch.full((batch, 2, L, st.N), -1, dtype=torch.int64, device="cuda"))
        K.ks_keyswitch(st.ctx, d, L, evk, out[-1], ws)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    assert_equal(out[0][-1:], st.ref.keyswitch(host(d[-1:]), host(evk), L))


@pytest.mark.parametrize("bits,logN,L,Kk,dnum,batch,want", [
    (36, 16, 16, 4, 4, 6, "vector"),     # 4 -> 16: few sources, groups of six targets that are not full
    (28, 16, 16, 4, 4, 6, "vector"),
    (36, 16, 24, 8, 3, 1, "matrix"),
    (28, 16, 24, 8, 3, 7, "matrix"),
    (28, 16, 36, 12, 3, 6, "vector"),    # seven rounds of workgroups: too many for 8 columns, too few for 16
    (36, 16, 36, 12, 3, 8, "matrix"),
    (36, 16, 3, 3, 1, 2, "vector"),      # a single round
    (36, 15, 21, 7, 3, 3, "matrix"),
    (36, 15, 9, 3, 3, 3, "vector"),      # 288 workgroups on 256 compute units
    (36, 14, 12, 4, 3, 3, "vector"),
])
def test_conversion_kernel_that_is_chosen(bits, logN, L, Kk, dnum, batch, want):
    """Both conversions of a call run on the kernel that measured faster at this size; its outputs are those of the other one."""
    st = Setup(logN, L, Kk, dnum, bits=bits)
    evk = st.uniform(44, 1, (dnum, 2), list(range(L + Kk)))
    d = st.uniform(44, 2, (batch,), list(range(L)))
    ws = workspace(st.ctx, K.KS_OP_KEYSWITCH, L, batch)
    out = [torch.full((batch, 2, L, st.N), -1, dtype=torch.int64, device="cuda") for _ in range(2)]
    K.ks_profile_enable(True)
    K.ks_keyswitch(st.ctx, d, L, evk, out[0], ws)
    launches = {r["kernel"]: r["launches"] for r in K.ks_profile_report()}
    K.ks_profile_enable(False)
    assert launches.get("bconv_mfma_ntt_cols" if want == "matrix" else "bconv_ntt_cols") == 2
    _select(st, 1 if want == "matrix" else 2, 0)
    K.ks_keyswitch(st.ctx, d, L, evk, out[1], ws)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("bits,n_src,n_dst,want", [
    (36, 1, 1, "vector"), (36, 1, 12, "vector"), (36, 1, 13, "matrix"), (36, 2, 4, "vector"), (36, 2, 5, "matrix"), (36, 3, 4, "vector"),
    (36, 3, 5, "matrix"), (36, 4, 2, "vector"), (36, 4, 3, "matrix"), (36, 5, 2, "vector"), (36, 5, 3, "matrix"), (36, 6, 1, "matrix"),
    (28, 1, 12, "vector"), (28, 1, 13, "matrix"), (28, 4, 6, "vector"), (28, 5, 10, "vector"), (28, 6, 1, "matrix"),
])
@pytest.mark.parametrize("batch", [1, 5])
def test_standalone_conversion_of_few_sources(bits, n_src, n_dst, want, batch):
    """Both sides of the line between the two standalone kernels, 28-bit moduli in both word sizes."""
    st = Setup(12, 15, 1, 3, bits=bits)
    src, dst = list(range(1, 1 + n_src)), [m for m in range(16) if not 1 <= m <= n_src][:n_dst]
    x = st.uniform(45, n_src, (batch,), src)
    ref = st.ref.bconv(host(x), src, dst)
    K.bconv_prepare(st.ctx, src, dst)
    for words in (64,) if bits == 36 else (64, 32):
        dtype = torch.int64 if words == 64 else torch.int32
        out = torch.full((batch, len(dst), st.N), -1, dtype=dtype, device="cuda")
        K.ks_profile_enable(True)
        (K.bconv if words == 64 else K.bconv_u32)(st.ctx, x.to(dtype), src, out, dst)
        ran = {r["kernel"] for r in K.ks_profile_report()}
        K.ks_profile_enable(False)
        assert ran == {"bconv" if want == "vector" else "bconv_mfma"}
        assert_equal(out.to(torch.int64), ref)


def test_sixteen_column_tiles_on_28_bit_moduli():
    """Four hoisted rotations of eight ciphertexts: the ModDown conversion of 64 polynomials takes whole-line tiles in this word size
    too; every residue against the vector kernel."""
    st = Setup(16, 24, 8, 3, bits=28)
    g = [pow(5, r, 2 * st.N) for r in range(1, 5)]
    word = lambda t: t.to(torch.int32)
    ct = word(st.uniform(47, 1, (8, 2), list(range(24))))
    keys = [word(st.uniform(47, 10 + r, (3, 2), list(range(32)))) for r in range(4)]
    ws = workspace(st.ctx, K.KS_OP_ROTATE_HOISTED_U32, 24, 8, 4)
    out = []
    for kernel in (0, 1):
        _select(st, kernel, 0)
        out.append(torch.full((8, 4, 2, 24, st.N), -1, dtype=torch.int32, device="cuda"))
        K.ks_rotate_hoisted_u32(st.ctx, ct, 24, g, keys, out[-1], ws)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("bits,pieces", [(36, 3), (28, 2)])
def test_operations_that_are_reported(bits, pieces):
    """The report's work of the fused conversions: per coefficient a multiply-add per source, target and piece (vector kernel), then the
    reduction and column stages of each target.  Digits of 2, 2 and 1 sources with 5, 5 and 6 targets, and 2 -> 5 for both components."""
    st = Setup(12, 5, 2, 3, bits=bits)
    evk, d = st.uniform(52, 1, (3, 2), list(range(7))), st.uniform(52, 2, (1,), list(range(5)))
    ws, out = workspace(st.ctx, K.KS_OP_KEYSWITCH, 5, 1), torch.empty((1, 2, 5, st.N), dtype=torch.int64, device="cuda")
    pairs, targets = 2 * 5 + 2 * 5 + 1 * 6 + 2 * (2 * 5), 5 + 5 + 6 + 2 * 5
    for kernel, name, ops in ((1, "bconv_ntt_cols", pieces * pairs + 19 * targets), (2, "bconv_mfma_ntt_cols", 28 * targets)):
        _select(st, kernel, 0)
        K.ks_profile_enable(True)
        K.ks_keyswitch(st.ctx, d, 5, evk, out, ws)
        report = {r["kernel"]: r for r in K.ks_profile_report()}
        K.ks_profile_enable(False)
        assert report[name]["total_ops"] == ops * st.N
