"""The ring kernel of the projections multiplies k-tiles of 32 in pairs: every launcher refuses a reduction with an odd
number of them, and one shorter than its ring, before anything is launched (no GPU).  The launchers are not part of the C
ABI; they are called by their C++ names.  Where a GPU is present the test is left out: the pointers are host memory."""
import ctypes as C

import pytest
import torch

from paper_2602_06412_amd import binding as B

P, I, Z = C.c_void_p, C.c_int, C.c_size_t
BUF = C.create_string_buffer(4096)
PTR = (C.addressof(BUF) + 255) // 256 * 256


def _call(name, *args):
    f = getattr(B.lib(), name)
    f.restype = I
    return f(*args)


LAUNCHERS = {
    "plain": lambda k, s: _call("_Z16slk_gemm_mfma256P12ihipStream_tPKviS2_PKiiiiiPfPvS4_m", P(0), P(PTR), I(0), P(PTR), P(PTR),
                                I(64), I(256), I(k), I(s), P(PTR), P(0), P(0), Z(256)),
    "probe": lambda k, s: _call("_Z22slk_gemm_mfma256_probeP12ihipStream_tPKviS2_PKiiiiPvS4_mPx", P(0), P(PTR), I(0), P(PTR),
                                P(PTR), I(256), I(256), I(k), P(PTR), P(0), Z(256), P(PTR)),
    "swiglu": lambda k, s: _call("_Z23slk_gemm_mfma256_swigluP12ihipStream_tPKvS2_PKiiiiPv", P(0), P(PTR), P(PTR), P(PTR), I(64),
                                 I(128), I(k), P(PTR)),
    "qkv_rope": lambda k, s: _call("_Z25slk_gemm_mfma256_qkv_ropeP12ihipStream_tPKvS2_PKiiiiS4_iiS2_PvS5_S5_", P(0), P(PTR), P(PTR),
                                   P(PTR), I(64), I(2), I(k), P(PTR), I(64), I(64), P(PTR), P(PTR), P(PTR), P(PTR)),
    "residual": lambda k, s: _call("_Z25slk_gemm_mfma256_residualP12ihipStream_tPKvS2_PKiiiiPv", P(0), P(PTR), P(PTR), P(PTR), I(64),
                                   I(256), I(k), P(PTR)),
}


@pytest.mark.skipif(torch.cuda.is_available(), reason="a launch that is wrongly accepted must have no device to run on")
@pytest.mark.parametrize("name,k,splits", [(n, k, 1) for n in LAUNCHERS for k in (288, 352, 192)] +
                         [("plain", 544, 2), ("plain", 576, 2), ("plain", 256, 2)])
def test_refused(name, k, splits):
    assert LAUNCHERS[name](k, splits) == B.SL_EINVAL
