"""What a grouped-query object takes of the device: the area of the passes that read the cache together stops growing at four passes."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_area_of_the_joint_passes_is_bounded():
    from paper_2602_11470_amd import binding as B
    ctx, dim, lv = B.llama_ring(6, 4), 128, 3
    try:
        kv = ctx.kv_create(8, dim, lv, r_i=16, unrolled_ladders=True)
        limb = 8 * ctx.n

        def taken(group):
            torch.cuda.synchronize()
            before = torch.cuda.mem_get_info()[0]
            gqa = ctx.gqa(kv, group)
            after = torch.cuda.mem_get_info()[0]
            del gqa
            return before - after

        taken(2)
        two, four, eight, sixteen = (taken(g) for g in (2, 4, 8, 16))
        turn = 9 * limb * ((lv + 2) + lv)                      # an inner rotation of the query and one of a result
        area = (16 + 12) * 2 * (lv + 1) * limb                 # baby steps and tensor sums of a pass
        slack = 1 << 25                                        # the allocator's granularity
        assert four - two >= 2 * area                          # the joint form is the one in use
        assert eight - four <= 4 * turn + slack
        assert sixteen - eight <= 8 * turn + slack
    finally:
        ctx.close()
