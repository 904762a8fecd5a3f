"""Rules of the dispatch that rest on measured times, asked of the library itself (host code, no GPU): calls that a route made slower keep
off it, calls that it serves stay on it.  The functions are internal, so their mangled names are used."""
import ctypes

import pytest

from paper_2504_11681_amd import binding

ll, ci, cb = ctypes.c_longlong, ctypes.c_int, ctypes.c_bool


def rule(name, *types, result=cb):
    fn = getattr(binding.lib(), name)
    fn.restype, fn.argtypes = result, types
    return fn


# (real, B, C_in, C_out, K): 1024 points, three kernels with spectra in y instead of the fused one
@pytest.mark.parametrize("case,on", [((True, 13, 1, 1, 5), False), ((True, 134, 1, 1, 2), False), ((True, 7, 3, 2, 22), False), ((False, 3, 2, 1, 6), False),
                                     ((False, 1, 7, 2, 2), False), ((True, 16, 8, 15, 8), False), ((False, 8, 8, 8, 43), False),
                                     ((False, 4, 4, 12, 64), True), ((True, 3, 2, 20, 30), True), ((False, 4, 9, 5, 16), True), ((True, 4, 9, 5, 16), True),
                                     ((False, 48, 128, 128, 64), True), ((True, 90, 128, 128, 64), True)], ids=str)
def test_rows_of_1024_points_held_in_y(case, on):
    real, B, Ci, Co, K = case
    assert rule("_ZN4tfno23pruned1d_in_y_supportedEbxiiii", cb, ll, ci, ci, ci, ci)(real, B, Ci, Co, 1024, K) == on


# (B, C_in, C_out, N, kernels' K, modes): own weights per mode, contraction and inverse in one kernel
@pytest.mark.parametrize("case,on", [((3, 186, 2, 256, 128, 90), False), ((5, 106, 12, 256, 128, 90), False), ((25, 89, 29, 128, 64, 37), False), ((8, 636, 45, 64, 16, 3), False),
                                     ((9, 373, 76, 128, 16, 7), False), ((2, 1800, 3, 256, 16, 12), False),
                                     ((6, 64, 25, 256, 128, 69), True), ((20, 166, 10, 64, 16, 15), True), ((7, 365, 31, 128, 16, 7), True), ((32, 64, 64, 1024, 64, 16), True),
                                     ((6, 65, 25, 256, 128, 69), False), ((30, 192, 16, 128, 16, 1), True), ((30, 193, 16, 128, 16, 1), False),
                                     ((7, 512, 31, 128, 16, 7), True), ((7, 513, 31, 128, 16, 7), False)], ids=str)
def test_small_layers_with_own_weights_in_one_kernel(case, on):
    assert rule("_ZN4tfno22pruned1d_permode_fusedExiiiii", ll, ci, ci, ci, ci, ci)(*case) == on


# (K, rows, C_in, C_out): real rows of 256 points, slabs of a workgroup of eight waves (0: four waves)
@pytest.mark.parametrize("case,slabs", [((64, 14, 2, 1), 0), ((64, 2, 16, 32), 0), ((128, 1, 7, 2), 0), ((128, 8, 8, 33), 0),
                                        ((64, 23, 17, 7), 1), ((128, 8, 9, 33), 1), ((32, 2, 3, 2), 1), ((64, 64, 64, 64), 1), ((64, 200, 9, 64), 2), ((128, 200, 64, 64), 0),
                                        ((64, 257, 64, 64), 0), ((16, 4, 64, 64), 0)], ids=str)
def test_eight_waves_for_few_real_rows_of_256_points(case, slabs):
    assert rule("_ZN4tfno24fused1d_real_eight_wavesEixii", ci, ll, ci, ci, result=ci)(*case) == slabs


# (B, C_in, N, K): lengths that are no powers of two, forward kernel of 16 pencils per workgroup
@pytest.mark.parametrize("case,on", [((76, 166, 581, 241), False), ((83, 73, 1026, 262), False), ((139, 89, 434, 179), False), ((459, 33, 476, 133), False), ((33, 33, 398, 195), False),
                                     ((11, 99, 2411, 200), False), ((103, 43, 203, 35), False), ((29, 163, 130, 55), False), ((189, 52, 304, 50), False),
                                     ((67, 34, 977, 152), True), ((67, 34, 400, 152), False), ((64, 128, 500, 64), True), ((64, 40, 1000, 50), True), ((5, 71, 162, 9), True),
                                     ((64, 128, 50, 12), True), ((64, 64, 300, 128), False), ((32, 64, 300, 128), True), ((64, 64, 130, 60), True), ((65, 64, 130, 60), False),
                                     ((128, 64, 130, 16), True), ((129, 64, 130, 16), False), ((256, 64, 600, 50), False), ((255, 64, 600, 50), True)], ids=str)
def test_forward_transform_of_few_pencils_of_odd_length(case, on):
    assert rule("_ZN4tfno24matrow_forward_supportedExiii", ll, ci, ci, ci)(*case) == on


# (B, C_in, C_out, N, K): lengths that are no powers of two, contraction and inverse in one kernel
@pytest.mark.parametrize("case,on", [((617, 1, 1, 1713, 121), False), ((208, 1, 2, 3169, 117), False), ((282, 3, 10, 1307, 153), False), ((88, 1, 33, 1286, 184), False),
                                     ((895, 7, 3, 338, 116), False), ((547, 224, 269, 77, 4), False), ((985, 111, 221, 46, 1), False),
                                     ((571, 1, 5, 291, 2), False), ((3, 257, 13, 551, 169), False), ((1, 129, 32, 551, 169), False), ((2, 1100, 32, 1000, 20), False),
                                     ((42, 44, 1, 1954, 74), True), ((145, 3, 244, 447, 98), True), ((228, 68, 172, 215, 34), True), ((453, 2, 17, 273, 50), True), ((64, 40, 56, 1000, 50), True), ((8, 69, 72, 116, 12), True), ((2, 3, 5, 600, 192), True),
                                     ((1, 128, 32, 551, 169), True), ((2, 1024, 32, 1000, 20), True), ((2, 3, 5, 600, 257), False), ((2, 4, 5, 31, 9), False)], ids=str)
def test_contraction_and_inverse_of_odd_lengths_in_one_kernel(case, on):
    assert rule("_ZN4tfno24matrow_inverse_supportedExiiii", ll, ci, ci, ci, ci)(*case) == on


# (direction, fields, N1, N2, K1, K2): both sides odd, both axes of a field in one kernel; many narrow fields with few kept columns as well
@pytest.mark.parametrize("case,on", [((-1, 1805, 77, 141, 18, 10), False), ((-1, 585, 99, 147, 23, 2), False), ((-1, 3270, 33, 136, 3, 18), False), ((-1, 3780, 45, 51, 19, 2), False),
                                     ((+1, 320, 273, 133, 28, 8), False), ((+1, 640, 93, 142, 32, 7), False), ((+1, 1040, 240, 52, 31, 9), False), ((+1, 1525, 272, 37, 29, 1), False),
                                     ((+1, 1142, 71, 149, 20, 12), False), ((-1, 8, 300, 300, 12, 12), False), ((-1, 100, 40, 40, 33, 9), False), ((-1, 100, 29, 40, 9, 9), False),
                                     ((-1, 1024, 85, 85, 12, 12), True), ((+1, 1024, 85, 85, 12, 12), True), ((-1, 8, 85, 85, 12, 12), True), ((-1, 594, 158, 131, 12, 12), True),
                                     ((+1, 342, 158, 131, 12, 12), True), ((-1, 126, 200, 120, 32, 17), True), ((-1, 3250, 54, 39, 2, 2), True), ((-1, 3320, 198, 38, 26, 3), True)], ids=str)
def test_fields_with_odd_sides_in_one_kernel(case, on):
    assert rule("_ZN4tfno17matgrid_supportedEixiiii", ci, ll, ci, ci, ci, ci)(*case) == on
