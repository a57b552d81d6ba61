"""The launch rules that are arithmetic on sizes, on the host: the shapes of the GPU tests take the kernels they are there for."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_dword as dword
import test_gpu_interleaved as interleaved
import test_gpu_kgroup as kgroup
import test_gpu_narrow as narrow
import test_gpu_output_stage as output_stage
import test_gpu_product_tile as product_tile
from paper_2505_18574_amd import ops

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18574_amd", "csrc")
SHIM = """
#include "gemm_rules.hpp"
extern "C" int product_tile(int M, int N, int K, int st160, int st320) { return ac::choose_product_tile_i8(M, N, K, st160, st320); }
extern "C" int kgroup(int ragged, int M, int N, int K, int eb, int conv, int a_along_k, int b_along_k, int splits, int workspace, int Cin, int raw) {
  const ac::KGroupCall c = {M, N, K, eb, conv != 0, a_along_k != 0, b_along_k != 0, (int64_t)N * eb, splits, workspace != 0, Cin, raw != 0};
  return ragged ? ac::kgroup_ragged_rule(c) : ac::kgroup_rule(c);
}
extern "C" int one_wave(int M, int N, int K) { return !ac::kgroup_instead_of_one_wave(M, N, K); }
extern "C" int narrow_product(int M, int N, int K) { return ac::narrow_product_rule(M, N, K); }
extern "C" int narrow_conv(int M, int N, int K, int taps, int stride, int one_wave, int stationary) { return ac::narrow_conv_rule(M, N, K, taps, stride, one_wave, stationary); }
extern "C" int narrow_tile(int M, int N, int K, int taps, int stride) { return ac::narrow_conv_tile(M, N, K, taps, stride); }
extern "C" int narrow_not_patch(int M, int N, int stride) { return ac::narrow_conv_instead_of_patch(M, N, stride); }
extern "C" int interleaved(int M, int N, int kbytes, int eb, int out_bytes, int ta, int tb) { return ac::interleaved_rule(M, N, kbytes, eb, out_bytes, ta != 0, tb != 0); }
extern "C" int interleaved_128x256(int M, int N, int K) { return ac::interleaved_128x256_rule(M, N, K); }
extern "C" int interleaved_at_bt(int M, int N, int K) { return ac::interleaved_at_bt_rule(M, N, K); }
extern "C" int wide_trans(int M, int N, int K, int ta, int tb, int dw) { return ac::wide_trans_rule(M, N, K, ta != 0, tb != 0, dw != 0); }
extern "C" int wide_product(int M, int N, int kbytes, int eb, int dw, int splits) { return ac::wide_product_rule(M, N, kbytes, eb, dw != 0, splits); }
extern "C" int tile(int M, int N) { return ac::choose_tile(M, N); }
extern "C" int dword_tiles(int M, int N, int kbytes, int both_along_k) { return ac::dword_tiles_rule(M, N, kbytes, both_along_k != 0); }
"""
TILE_128X256 = 129


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    folder = tmp_path_factory.mktemp("rules")
    (folder / "shim.cpp").write_text(SHIM)
    so = str(folder / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(folder / "shim.cpp")], check=True)
    return ctypes.CDLL(so)


def product_tile_of(rules, M, N, K, matrix_bias):
    """The tile of an int8 product on aligned operands whose plan the caller does not name."""
    tiles = -(-M // 64) * -(-N // 64)
    assert tiles > 512 or (tiles > 256 and K < 4096)
    assert ops.ac_gemm_i8_auto_plan(M, N, K, False)[0] != 32
    return rules.product_tile(M, N, K, *(1 <= K <= limit and not matrix_bias for limit in (2048, 1536)))


def test_product_tile_shapes(rules):
    for matrix in (False, True):
        for shape in product_tile.TILE_128X256:
            assert product_tile_of(rules, *shape, matrix) == TILE_128X256, shape
        for M, N, K in product_tile.SEVERAL_TO_A_WORKGROUP:
            assert product_tile_of(rules, M, N, K, matrix) == TILE_128X256 and -(-M // 128) * -(-N // 256) > 512, (M, N, K)
    assert [product_tile_of(rules, *shape, False) for shape in product_tile.OTHER_CODES] == [320, 128]


def last_trips(kb, dw):
    """K tiles of 64 bytes that the interleaved loop multiplies outside its rounds of four, the very last one apart: a round needs the
    four tiles behind its own to be whole, which on dwords the last tile never is."""
    tiles, whole = -(-kb // 64), (kb - dw) // 64
    kt = 0
    while kt + 7 < min(tiles, whole):
        kt += 4
    return tiles - kt - 1


def test_interleaved_shapes(rules):
    """The shapes of the interleaved loop's tests take it, and run each count of last trips in each form."""
    for form, (eb, ta, tb, out, dw) in interleaved.FORMS.items():
        for rounds, (tiles, _, _) in interleaved.ROUNDS.items():
            seen = set()
            for kb in interleaved.K_BYTES[dw]:
                M, N, K = interleaved.shape_of(form, rounds, kb)
                assert -(-M // 256) * -(-N // 256) == tiles and (tiles > 256) == (rounds == "several")
                assert rules.interleaved(M, N, kb, eb, 1 if out == "i8" else 4, ta, tb), (form, rounds, kb)
                if out == "i32":
                    assert rules.tile(M, N) == 256
                elif eb == 2:
                    assert tuple(ops.ac_gemm_bf16_auto_plan(M, N, K)) == (256, 1)
                else:
                    assert tuple(ops.ac_gemm_i8_auto_plan(M, N, K, False)) == (256, 1)
                if form == "i8":
                    assert product_tile_of(rules, M, N, K, False) == 256
                if ta and not dw:
                    assert not rules.interleaved_at_bt(M, N, K)
                if dw:
                    assert rules.dword_tiles(M, N, kb, not ta and tb)
                if ta or tb:
                    assert not rules.wide_trans(M, N, K, ta, tb, dw)
                else:
                    assert not rules.wide_product(M, N, kb, eb, dw, 1)
                assert not rules.kgroup(0, M, N, K, eb, 0, not ta, tb, 1, 0, 0, out == "i32")
                seen.add(last_trips(kb, dw))
            assert seen == ({4, 5, 6, 7} if dw else {3, 4, 5, 6, 7}), (form, rounds, seen)
    for M, N, K, dw in interleaved.SHORT_AT_BT:
        assert rules.interleaved(M, N, K, 1, 1, 1, 1) and not rules.wide_trans(M, N, K, 1, 1, dw)
        assert rules.dword_tiles(M, N, K, 0) if dw else not rules.interleaved_at_bt(M, N, K)
        assert tuple(ops.ac_gemm_i8_auto_plan(M, N, K, False)) == (256, 1) and -(-M // 256) * -(-N // 256) > 256
    # whole K tiles: with eight a prefetched item runs a whole round of trips, with seven none
    assert {(dw, (K - dw) // 64) for _, _, K, dw in interleaved.SHORT_AT_BT} == {(False, 8), (False, 9), (True, 7), (True, 8), (True, 9)}
    assert {(-(-M // 128) * -(-N // 256) > 256, last_trips(K, False)) for M, N, K in interleaved.CHOSEN_128X256} >= {(True, t) for t in (4, 5, 6, 7, 3)} | {(False, 4)}
    for M, N, K in interleaved.CHOSEN_128X256:
        assert rules.interleaved_128x256(M, N, K) and product_tile_of(rules, M, N, K, False) == product_tile_of(rules, M, N, K, True) == TILE_128X256
    assert not rules.interleaved_128x256(1334, 3456, 2512) and not rules.interleaved_128x256(1386, 3328, 2192)
    assert not rules.interleaved_128x256(3648, 1344, 1024) and not rules.interleaved_128x256(5088, 3520, 1024)
    for M, N, K in interleaved.CHOSEN_AT_BT:
        assert rules.interleaved_at_bt(M, N, K) and not rules.wide_trans(M, N, K, 1, 1, 0)
    assert not rules.interleaved_at_bt(3792, 784, 4096) and not rules.interleaved_at_bt(3008, 5824, 1536) and not rules.interleaved_at_bt(6240, 576, 768) and not rules.interleaved_at_bt(1216, 3136, 5120)
    assert not any(rules.interleaved(M, N, kb, 1, 1, 1, 0) for M, N in ((3601, 4080), (5393, 5392)) for kb in (1024, 4096, 8192))  # A^T alone
    assert not any(rules.interleaved(3136, 3296, k, 1, 1, 0, tb) or rules.interleaved(3136, 3296, k, 2, 4, 0, 0) for k in (1024, 2048, 4096) for tb in (0, 1))  # 169 tiles
    assert not rules.interleaved(8192, 8192, 1024, 1, 1, 0, 0) and not rules.interleaved(4096, 4096, 2048, 1, 4, 0, 0) and not rules.interleaved(4096, 4096, 512, 2, 4, 0, 0)


def test_interleaved_needs_longer_k_where_units_idle(rules):
    """Products that the loop slows down by 4 to 9 %: few K tiles for the compute units that have none in the last round."""
    for M, N, K, eb, out, tb in [(3674, 6792, 616, 2, 4, 0), (8380, 5032, 616, 2, 4, 0), (7032, 3680, 928, 2, 4, 0), (13449, 908, 758, 2, 4, 0), (3388, 7192, 888, 2, 4, 0),
                                 (5203, 5376, 2272, 1, 1, 0), (7150, 5632, 2256, 1, 1, 0), (2639, 5412, 1224, 1, 1, 0), (15212, 1740, 1440, 1, 1, 1), (14288, 2320, 2512, 1, 4, 0)]:
        assert not rules.interleaved(M, N, K * eb, eb, out, 0, tb), (M, N, K)
    for M, N, K, eb, out, tb in [(8192, 8192, 8192, 1, 1, 0), (4096, 4096, 4096, 2, 4, 0), (8192, 8192, 1024, 2, 4, 0), (4096, 4096, 2048, 1, 1, 0), (4096, 8192, 1024, 1, 1, 1), (8192, 4096, 2048, 1, 4, 0)]:
        assert rules.interleaved(M, N, K * eb, eb, out, 0, tb), (M, N, K)
        # the line rises with the units that idle: one tile more than a round's
        assert not rules.interleaved(2048, 8448, 1024 * eb if out == 4 else 1024, eb, out, 0, tb)


def shared_tile(rules, M, N, K, eb=1, conv=False, ragged=False, workspace=True, Cin=0, a_along_k=True, b_along_k=False, raw=False):
    """Whether the waves of a workgroup share the call's tiles (dense operands)."""
    need = (ops.ac_gemm_i8_workspace_bytes if eb == 1 else ops.ac_gemm_bf16_workspace_bytes)(M, N, K)
    splits = need // (4 * M * N) if need and (workspace or eb == 2) else 1
    if ragged and eb == 2:
        splits = 1  # never cut
    return bool(rules.kgroup(ragged, M, N, K, eb, conv, a_along_k, b_along_k, splits, workspace, Cin, raw))


def test_shared_tiles_leave_cut_products_that_they_would_slow_down(rules):
    """Products and convolutions that the other kernels cut over workgroups and run faster, from HBM or at all."""
    for M, N, K in [(16, 4096, 4096), (31, 1792, 2896 + 512), (16, 2048, 2048), (128, 128, 4096), (26, 896, 3520), (235, 64, 5568), (264, 64, 6856)]:
        assert not shared_tile(rules, M, N, K), (M, N, K)
        assert shared_tile(rules, M, N, K, workspace=False)
    for M, N, K in [(16, 2064, 2048), (344, 480, 3136), (58, 512, 2144), (128, 1024, 3072), (1400, 32, 4352), (49, 512, 2304)]:
        assert shared_tile(rules, M, N, K), (M, N, K)
    for M, N, K in [(16, 896, 2432), (60, 512, 1984), (23, 336, 2176), (93, 208, 2064)]:
        assert not shared_tile(rules, M, N, K, eb=2), (M, N, K)
    assert shared_tile(rules, 150, 576, 1184, eb=2) and shared_tile(rules, 64, 96, 2400, eb=2, workspace=False)
    for M, N, K in [(49, 512, 4608), (64, 256, 6272), (200, 576, 6400), (100, 64, 5040)]:
        assert not shared_tile(rules, M, N, K, conv=True), (M, N, K)
    assert shared_tile(rules, 196, 256, 2304, conv=True) and shared_tile(rules, 338, 64, 4176, conv=True)
    for M, N, K in [(20, 485, 3244), (317, 262, 3123), (14, 3779, 3482)]:
        assert not shared_tile(rules, M, N, K, ragged=True), (M, N, K)
    assert shared_tile(rules, 25, 1000, 2557, ragged=True) and shared_tile(rules, 20, 39, 3064, ragged=True)
    for M, N, K, Cin in [(2048, 148, 13965, 285), (1764, 237, 8624, 176), (2160, 126, 5650, 226), (5600, 36, 7007, 143), (11236, 15, 9457, 193)]:
        assert not shared_tile(rules, M, N, K, conv=True, ragged=True, Cin=Cin), (M, N, K)
        assert shared_tile(rules, M, N, K, conv=True, ragged=True, Cin=Cin, workspace=False)


def test_two_rounds_of_shared_tiles_end_where_wider_tiles_are_ahead(rules):
    """257 to 448 tiles of any alignment, K uncut: which operands' rows run along K decides how deep."""
    forms = {"plain": (True, False), "ta": (False, False), "tb": (True, True), "tab": (False, True)}
    for M, N, K, form, takes in [(621, 509, 2394, "plain", False), (361, 871, 8134, "plain", False), (195, 1599, 233, "plain", True),
                                 (361, 1101, 1542, "ta", False), (387, 623, 3283, "ta", False), (194, 1737, 203, "ta", True),
                                 (156, 1897, 6132, "tab", False), (915, 349, 3444, "tab", True), (2294, 127, 7027, "tb", True)]:
        a, b = forms[form]
        assert shared_tile(rules, M, N, K, ragged=True, workspace=False, a_along_k=a, b_along_k=b) == takes, (M, N, K, form)
    assert not shared_tile(rules, 1383, 293, 6769, eb=2, ragged=True) and shared_tile(rules, 2526, 105, 3140, eb=2, ragged=True)


def test_two_rounds_of_shared_tiles_of_convolutions_end_where_their_weights_are_many(rules):
    for M, N, K, takes in [(2448, 128, 6800, False), (3072, 128, 7344, False), (3757, 128, 7344, False), (3024, 128, 6192, False), (3200, 112, 7056, False), (3179, 112, 6768, False),
                           (2304, 112, 5616, False), (3456, 96, 7056, False), (3520, 96, 6800, False), (3920, 128, 3600, False), (3888, 128, 2448, False), (722, 464, 3168, False), (576, 496, 3920, False),
                           (960, 448, 2592, False), (588, 512, 2880, False), (3528, 112, 5488, True), (3211, 112, 5200, True), (4056, 96, 4800, True), (3528, 128, 4704, True), (2800, 128, 3136, True), (4608, 96, 5488, True),
                           (5200, 80, 6272, True), (4800, 64, 7840, True), (12167, 32, 7840, True), (1100, 320, 2880, True), (648, 400, 2800, True)]:
        assert 256 < -(-M // 32) * -(-N // 32) <= 512
        assert shared_tile(rules, M, N, K, conv=True) == takes, (M, N, K)


def test_shared_tiles_where_k_is_short(rules):
    assert [rules.one_wave(*s) for s in [(57, 64, 64), (190, 64, 64), (30, 64, 256), (100, 256, 64), (256, 256, 256), (700, 400, 64)]] == [1, 1, 0, 0, 0, 1]
    assert shared_tile(rules, 64, 5584, 336, a_along_k=False) and not shared_tile(rules, 1328, 352, 448, a_along_k=False)
    assert shared_tile(rules, 528, 736, 432) and not shared_tile(rules, 224, 1920, 624)


def test_small_convolutions_of_few_columns_keep_the_row_copying_kernel(rules):
    for M, N, K, Cin, takes in [(6728, 6, 288, 32, False), (640, 11, 200, 8, False), (576, 15, 300, 12, False), (300, 20, 576, 64, False),
                                (363, 174, 245, 5, True), (1058, 21, 700, 28, True), (1863, 20, 392, 8, True), (169, 51, 600, 24, True), (1600, 198, 1200, 48, False), (6075, 54, 1210, 54, True)]:
        assert shared_tile(rules, M, N, K, conv=True, ragged=True, workspace=False, Cin=Cin) == takes, (M, N, K)


def test_dword_products_leave_the_direct_tiles_where_the_unaligned_ones_are_ahead(rules):
    """(M, N, bytes of K, both operands' rows along K)"""
    for M, N, kb, both, takes in [(828, 2276, 4028, 0, False), (904, 1380, 2668, 0, False), (1420, 1032, 2560, 0, False), (1600, 980, 940, 1, False),
                                  (2639, 212, 64, 0, False), (2107, 1120, 72, 0, False), (535, 1672, 28, 1, False), (1564, 536, 772, 1, False), (7077, 460, 156, 1, False),
                                  (1000, 1000, 1000, 0, True), (2584, 2040, 160, 0, True), (1146, 2564, 2076, 0, True), (5426, 4740, 148, 1, True),
                                  (3513, 788, 1032, 1, True), (935, 2092, 3968, 1, True)]:
        assert bool(rules.dword_tiles(M, N, kb, both)) == takes, (M, N, kb)


def test_dword_shapes(rules):
    for tile, shapes in dword.DIRECT_TILES.items():
        for M, N, K in shapes:
            assert ops.ac_gemm_i8_auto_plan(M, N, K, False) == (tile, 1), (M, N, K)
            assert all(rules.dword_tiles(M, N, K, both) for both in (0, 1)) and not shared_tile(rules, M, N, K, workspace=False), (M, N, K)
            assert (K % 16 or N % 16) and M % 16  # each form meets the rule's operands


def shapes_of(test):
    """The last parametrised sizes of a GPU test."""
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and "," in m.args[0])


def conv_sizes(nb, edge, cin, cout, k, stride):
    out = (edge + 2 * (k // 2) - k) // stride + 1
    return nb * out * out, cout, k * k * cin


def test_shared_tile_shapes(rules):
    """The sizes of the GPU tests lie on the side of each line that they are there for."""
    taken = [(M, N, K) for M, N, K in shapes_of(kgroup.test_int32_on_two_rounds) if shared_tile(rules, M, N, K, workspace=False, raw=True)]
    assert taken == [(8193, 32, 624), (16384, 16, 1408), (288, 928, 960), (511, 1008, 944), (300, 932, 956), (4099, 60, 1404)]
    assert all(256 < -(-M // 32) * -(-N // 32) <= 512 for M, N, K in shapes_of(kgroup.test_int32_on_two_rounds))
    convs = shapes_of(kgroup.test_convolutions_beside_a_workspace)
    left = [c for c in convs if not shared_tile(rules, *conv_sizes(*c), conv=True, Cin=c[2])]
    assert left == [(2, 9, 432, 16, 5, 1), (1, 14, 384, 32, 5, 1), (1, 20, 160, 64, 7, 1), (3, 19, 208, 80, 5, 2), (1, 7, 208, 144, 5, 1), (4, 37, 336, 48, 5, 1), (7, 14, 176, 240, 5, 1),
                    (33, 9, 272, 160, 3, 1), (3, 31, 208, 128, 5, 1), (13, 16, 224, 112, 5, 1), (17, 15, 272, 96, 5, 1), (5, 28, 112, 128, 5, 1), (14, 7, 400, 416, 3, 1)]


def test_narrow_shapes(rules):
    products = shapes_of(narrow.test_products)
    assert [s for s in products if not rules.narrow_product(*s)] == [(131073, 16, 112), (40000, 32, 2064)]
    for c in shapes_of(narrow.test_convolutions):
        (M, N, K), taps, stride = conv_sizes(*c), c[4] ** 2, c[5]
        one_wave = K % 64 == 0 and K <= 640 and -(-M // 32) * -(-N // 32) <= 2048
        assert one_wave == (c == (70, 31, 64, 32, 3, 2)), c  # this one is planned with a wave to a tile
        # whatever else is planned; not the patch kernel, which needs whole 32s of channels, a stride of 1 and at most 32 taps
        assert one_wave or all(rules.narrow_conv(M, N, K, taps, stride, 0, stationary) for stationary in (0, 1)), c
        assert rules.narrow_tile(M, N, K, taps, stride) == (c != (35, 96, 144, 16, 3, 3)) or one_wave, c
        assert c[2] % 32 != 0 or stride > 1 or taps > 32, c


def test_narrow_tiles_leave_what_they_would_slow_down(rules):
    for M, N, K, takes in [(753035, 16, 128, False), (902968, 16, 128, False), (574609, 32, 352, False), (1837930, 16, 176, False), (401408, 16, 80, False),
                           (48529, 32, 2192, False), (36048, 32, 2960, False), (38364, 16, 3792, False), (70643, 16, 2288, False), (39018, 32, 1184, False),
                           (137103, 32, 128, True), (282133, 32, 208, True), (290715, 32, 544, True), (96366, 32, 16, True), (38235, 32, 160, True),
                           (40867, 16, 1088, True), (87408, 32, 2304, True), (153392, 16, 1280, True), (51937, 32, 1600, True), (50176, 48, 1024, False), (16384, 32, 1024, False)]:
        assert bool(rules.narrow_product(M, N, K)) == takes, (M, N, K)
    # beside the weight-stationary kernel: pixels, columns, K, taps, stride
    for M, N, K, taps, stride, takes in [(1052025, 16, 48, 1, 2, False), (625931, 16, 128, 1, 2, False), (1018464, 32, 16, 1, 2, False), (811008, 32, 64, 4, 2, False),
                                         (1177254, 16, 256, 4, 2, False), (960000, 32, 704, 4, 2, False), (835200, 16, 720, 9, 3, False), (349856, 16, 1008, 4, 2, False), (349856, 16, 1408, 4, 2, True),
                                         (1802493, 32, 1200, 25, 2, True), (578654, 32, 432, 9, 1, True), (137275, 32, 352, 1, 3, True), (100719, 16, 48, 1, 2, True)]:
        assert bool(rules.narrow_conv(M, N, K, taps, stride, 0, 1)) == takes, (M, N, K, taps, stride)
        assert rules.narrow_conv(M, N, K, taps, stride, 0, 0) and not rules.narrow_conv(M, N, K, taps, stride, 1, 0)
    assert not rules.narrow_tile(35525, 16, 3312, 9, 3) and rules.narrow_tile(35525, 16, 3312, 9, 2) and rules.narrow_tile(35525, 16, 1008, 9, 3) and not rules.narrow_tile(50176, 48, 4608, 9, 1) and not rules.narrow_tile(349856, 16, 1408, 4, 2)
    assert rules.narrow_not_patch(1441557, 16, 2) and not rules.narrow_not_patch(284350, 32, 1)


def test_output_stage_shapes(rules):
    """The shapes of the 4-byte output stages' tests make each tile, none of them on the interleaved loop."""
    codes = {"64": 64, "128": 128, "256x128": 192, "256": 256, "256, several": 256}
    for name, (M, N, K) in output_stage.SHAPES.items():
        for dword in (False, True):
            n, k = (N, K - 4) if dword else (N + 4 & ~15, K)
            assert rules.tile(M, n) == codes[name], name
            assert not rules.interleaved(M, n, k, 1, 4, 0, 0) and not rules.wide_product(M, n, k, 1, dword, 1)
            assert not rules.kgroup(0, M, n, k, 1, 0, 1, 0, 1, 0, 0, 1)
            assert not dword or rules.dword_tiles(M, n, k, 0), (name, dword)
    assert -(-5393 // 256) * -(-5388 // 256) > 256
