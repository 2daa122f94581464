"""The two forms of the packed product, sums held until the launch ends and sums written as they come, on the same words: every output
word the same, for any count of giant steps (blocks, parts of a block), partly filled rounds (n = 4096) and several launches."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 65536])
def test_forms_agree(n):
    from paper_2602_11470_amd import binding as B
    f = B.lib._Z19launch_vmm_mac_formP6cm_ctxPmPKmS3_iiiimP12ihipStream_tb
    f.argtypes, f.restype = [C.c_void_p] * 4 + [C.c_int] * 4 + [C.c_size_t, C.c_void_p, C.c_bool], None
    for bits in ((50, 50, 60), (58, 58, 61)):
        ctx = B.Context(n, 14, 2, 2, *bits, 2.0 ** 40, hamming=64)
        try:
            for level, r_i, r_o in ((3, 8, 1), (3, 16, 2), (4, 16, 4), (6, 32, 8), (13, 8, 16), (4, 32, 16), (9, 16, 32), (13, 8, 4)):
                limbs, gen = level + 3, torch.Generator(device="cuda").manual_seed(level + r_o)
                ct = 2 * limbs * n
                babies = torch.randint(0, 1 << 49, (r_i * ct,), generator=gen, device="cuda")
                pts = torch.randint(-(1 << 63), (1 << 63) - 1, (r_i * r_o * limbs * n,), generator=gen, device="cuda")
                if bits[2] > 60:
                    pts &= (1 << 58) - 1                 # 64-bit words under the special primes: residues
                outs = [torch.zeros(r_o * ct, dtype=torch.int64, device="cuda") for _ in range(2)]
                for held, out in enumerate(outs):
                    f(ctx.h, out.data_ptr(), babies.data_ptr(), pts.data_ptr(), r_i, r_o, limbs, level, ct, None, bool(held))
                torch.cuda.synchronize()
                assert outs[0].any() and torch.equal(*outs), (bits, level, r_i, r_o)
        finally:
            ctx.close()
