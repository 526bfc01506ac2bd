"""64-bit transforms keep a limb packed or as doubles between their two passes, by the size of the data: both sides of every line, against
the reference."""

import pytest
import torch

import paper_2512_11269_amd as K
from gpu_util import Setup, assert_equal, host

pytestmark = pytest.mark.gpu

MIB = 1 << 20


@pytest.mark.parametrize("logN,inverse,least,most", [
    (12, False, 19, 26), (13, False, 19, 25), (14, False, 19, 33),
    (12, True, 19, 28), (13, True, 19, 35), (14, True, 19, 35),
    (15, False, None, None), (15, True, None, None), (16, True, None, None),
])
def test_form_between_the_passes(logN, inverse, least, most):
    st = Setup(logN, 3, 1, 3)
    limb = 8 * st.N
    sizes = [24] if least is None else [least, most]
    for mib in sizes:
        for limbs in (mib * MIB // limb - 1, mib * MIB // limb, mib * MIB // limb + 1):
            x = st.uniform(61, limbs, (limbs,), [2])
            y = x.clone()
            K.ks_profile_enable(True)
            (K.ntt_inv if inverse else K.ntt_fwd)(st.ctx, y, [2])
            moved = {r["kernel"]: r["total_bytes"] for r in K.ks_profile_report()}
            K.ks_profile_enable(False)
            doubles = least is not None and least * MIB <= limbs * limb <= most * MIB
            assert len(moved) == 2 and set(moved.values()) == {(16 if doubles else 13) * limbs * st.N}
            assert_equal(y, (st.ref.ntt_inv if inverse else st.ref.ntt_fwd)(host(x), [2]))
