"""The minimisers' quotients and roots on the device, from v_rcp_f32 and v_sqrt_f32,
against the compiler's division and sqrtf, bit for bit: every significand of the
divisor and of the root's operand (all ones with powers of two among them, where
the refinement rests on the estimate), over the exponents the minimisers use."""
import ctypes as ct

import pytest

pytestmark = pytest.mark.gpu


# quotients of these stay in [2^-92, 2^95], inside the range the refinement is for
@pytest.mark.parametrize("exponent", [-85, -30, -1, 0, 9, 60])
def test_every_significand(exponent):
    import torch
    from paper_1311_4527_amd import twa as T
    num = [2.0 ** e for e in (-30, -1, 0, 1, 9)] + [1.9999998807907104, 1.0000001192092896, 1.5, 4.0 / 3.0, -0.7, 3.1415927]
    n = torch.tensor(num, dtype=torch.float32, device="cuda")
    bad = torch.zeros(2, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream()
    st = T.load_library().twa_debug_quotients(ct.c_void_p(n.data_ptr()), ct.c_int(len(n)), ct.c_float(2.0 ** exponent),
                                              ct.c_void_p(bad.data_ptr()), ct.c_void_p(stream.cuda_stream))
    assert st == T.TWA_OK
    assert bad.tolist() == [0, 0]
