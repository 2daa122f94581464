"""The rules that choose between two forms of a launch, at the sizes whose both forms were timed (the figures stand beside each rule):
no call is sent to the slower one.  The functions are called in the library; no GPU is needed."""
import ctypes

import pytest


def _rule(name):
    from paper_2602_11470_amd import binding as B
    f = getattr(B.lib, name)
    f.restype = ctypes.c_bool
    return f


@pytest.mark.parametrize("n,limbs,cnt,groups,passes,pays", [
    (65536, 10, 16, 8, 2, True), (65536, 4, 16, 4, 2, True), (65536, 10, 16, 1, 2, False), (65536, 21, 8, 8, 2, False), (65536, 10, 1, 2, 2, False),
    (65536, 10, 16, 8, 4, True), (65536, 10, 16, 1, 4, True), (65536, 10, 4, 1, 4, False), (65536, 21, 8, 1, 4, False), (65536, 21, 2, 8, 4, False),
    (65536, 10, 1, 2, 4, True), (65536, 21, 4, 8, 4, True), (4096, 5, 1, 1, 2, True), (4096, 5, 1, 8, 2, True), (4096, 13, 16, 8, 2, True),
    (4096, 25, 8, 4, 2, False), (4096, 5, 1, 8, 4, True)])
def test_joint_passes_where_they_are_faster(n, limbs, cnt, groups, passes, pays):
    assert _rule("_Z22tensor_sum_passes_paysiiiii")(n, limbs, cnt, groups, passes) == pays


@pytest.mark.parametrize("n,limbs,cnt,groups,held", [
    (65536, 3, 1, 2, True), (4096, 25, 1, 2, True), (65536, 6, 2, 4, True), (65536, 5, 2, 2, False), (65536, 4, 16, 2, False), (65536, 4, 4, 8, False),
    (65536, 4, 16, 8, True), (65536, 10, 8, 8, True), (65536, 10, 8, 2, False), (65536, 10, 2, 8, False), (65536, 21, 16, 2, True), (65536, 21, 8, 2, False),
    (65536, 21, 1, 2, False), (65536, 13, 4, 4, False), (65536, 8, 2, 8, False)])
def test_tensor_sums_held_where_that_is_faster(n, limbs, cnt, groups, held):
    assert _rule("_Z15tensor_sum_heldiiii")(n, limbs, cnt, groups) == held


@pytest.mark.parametrize("n,limbs,r_i,r_o,held", [
    (65536, 28, 32, 16, True), (65536, 9, 32, 16, True), (65536, 8, 64, 32, True), (65536, 28, 8, 1, False), (65536, 28, 8, 32, False),
    (65536, 9, 64, 1, False), (65536, 9, 16, 8, True), (65536, 9, 16, 2, False), (65536, 6, 16, 8, False), (65536, 14, 16, 16, False),
    (65536, 18, 16, 16, True), (65536, 6, 16, 64, True), (65536, 4, 16, 8, False), (65536, 8, 32, 4, False), (4096, 6, 16, 8, False),
    (4096, 6, 8, 1, False), (4096, 14, 32, 64, True)])
def test_packed_products_held_where_that_is_faster(n, limbs, r_i, r_o, held):
    assert _rule("_Z12vmm_mac_heldiiii")(n, limbs, r_i, r_o) == held


@pytest.mark.parametrize("split,bits,ns,joined,pays", [(0, 50, 1, False, False), (0, 50, 8, False, False), (0, 50, 4, False, True), (0, 50, 1, True, True),
                                                       (0, 60, 1, False, True), (0, 60, 8, False, True), (1, 50, 1, False, True), (2, 60, 1, False, True)])
def test_cut_weights_where_they_are_faster(split, bits, ns, joined, pays):
    """split: how the sources' words are split (0: all below 2^50); bits: of the largest target modulus."""
    assert _rule("_Z14conv_near_paysimib")(split, ctypes.c_ulong((1 << bits) - 1), ns, ctypes.c_bool(joined)) == pays
