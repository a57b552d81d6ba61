"""GPU parity of the interleaved K loop: each operand form that has it, on one round of tiles and with several tiles to a workgroup
(the next one's prefetch), every count of last trips (3 to 7; on dwords 4 to 7), a partial last K tile, last rows and columns that
are missing, shifts at both ends of its output stage's range, a bias row, a bias matrix and none.  Every element of every output is
compared: int8 and int32 bit for bit with exact sums, bf16 with the bound of fp32 sums.  test_gemm_rules.py holds each shape to the
loop and the counts of last trips to what is said here."""
import pytest
import torch

from gpu_util import check_bf16_product, check_equal, product_i64, requantise
from paper_2505_18574_amd import ops

pytestmark = pytest.mark.gpu

# form: bytes of an element, A^T, B^T, output, operands on dwords
FORMS = {"i8": (1, False, False, "i8", False), "bt": (1, False, True, "i8", False), "at_bt": (1, True, True, "i8", False),
         "i32": (1, False, False, "i32", False), "bf16": (2, False, False, "f32", False),
         "i8_dw": (1, False, False, "i8", True), "bt_dw": (1, False, True, "i8", True), "at_bt_dw": (1, True, True, "i8", True),
         "i32_dw": (1, False, False, "i32", True), "bf16_dw": (2, False, False, "f32", True)}
# 240 tiles of 256 x 256: one round of them; 484: a second and a part of one
ROUNDS = {"one": (240, 3601, 4080), "several": (484, 5393, 5392)}
# K in bytes: whole 16 bytes, and whole dwords (4096 of those are dwords by the columns alone)
K_BYTES = {False: [4096, 4160, 4224, 4288, 4304], True: [4096, 4100, 4164, 4228, 4348]}


def shape_of(form, rounds, kb):
    """M, N, K: no side a whole number of MFMA tiles where the form leaves it free."""
    eb, ta, tb, out, dw = FORMS[form]
    _, M, N = ROUNDS[rounds]
    if ta:
        M = M - 1 if not dw else M + 3
    if dw:
        N += 4
    return M, N, kb // eb


CASES = [(form, rounds, kb) for form in FORMS for rounds in ROUNDS for kb in K_BYTES[FORMS[form][4]]]
# (M, N, K, on dwords) of A^T B^T: short K loops behind a prefetch, eight to ten K tiles, the last whole, of part of a chunk and of several
SHORT_AT_BT = [(8208, 8208, 512, False), (8208, 8208, 592, False), (8204, 8212, 512, True), (8204, 8212, 516, True), (8204, 8212, 596, True)]
# the 128 x 256 tiles that a product without a plan takes: on one round of them and on more; and A^T B^T products on one round
CHOSEN_128X256 = [(1617, 4544, 2064), (1361, 4736, 2176), (2257, 3232, 3136), (3297, 6960, 1296), (6049, 3008, 2240), (3297, 6960, 1408), (3297, 6960, 1520), (3297, 6960, 1536)]
CHOSEN_AT_BT = [(1712, 3584, 512), (2128, 2192, 592), (1040, 4112, 1136), (4464, 1744, 704)]


def matrix(rows, cols, dtype, seed, dword=False):
    """Random values; on dwords, a view one dword into longer rows, whose surroundings would show in a sum."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    pad = 0 if not dword else 4 if dtype == torch.int8 else 2
    if dtype == torch.int8:
        m = torch.randint(-128, 128, (rows, cols + 2 * pad), dtype=dtype, device="cuda", generator=g)
    else:
        m = torch.randn((rows, cols + 2 * pad), dtype=torch.float32, device="cuda", generator=g).to(dtype)
    if dword:
        m[:, :pad], m[:, pad + cols:] = (77, 77) if dtype == torch.int8 else (float("nan"), float("nan"))
    return m[:, pad:pad + cols]


def operands(M, N, K, dtype, seed, ta=False, tb=False, dword=False):
    """A and B as the call takes them, and as the product reads them."""
    A = matrix(K, M, dtype, seed, dword) if ta else matrix(M, K, dtype, seed, dword)
    B = matrix(N, K, dtype, seed + 1, dword) if tb else matrix(K, N, dtype, seed + 1, dword)
    return A, B, A.T if ta else A, B.T if tb else B


def bias_of(kind, M, N, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = {"none": None, "row": (N,), "matrix": (M, N)}[kind]
    return None if shape is None else torch.randint(-(1 << 15), 1 << 15, shape, dtype=torch.int32, device="cuda", generator=g)


def output(M, N, dtype, fill):
    """M rows, and one behind them that stays."""
    return torch.full((M + 1, N), fill, dtype=dtype, device="cuda")


@pytest.mark.parametrize("form,rounds,kb", CASES)
def test_forms(form, rounds, kb):
    eb, ta, tb, out, dw = FORMS[form]
    M, N, K = shape_of(form, rounds, kb)
    if eb == 2:
        A, B, Am, Bm = operands(M, N, K, torch.bfloat16, kb + len(form), dword=dw)
        C = output(M, N, torch.float32, float("nan"))
        ops.ac_gemm_bf16(A, B, C[:M])
        check_bf16_product(Am, Bm, C[:M])
        assert torch.isnan(C[M]).all()
        return
    A, B, Am, Bm = operands(M, N, K, torch.int8, kb + len(form), ta, tb, dw)
    b = bias_of("row", M, N, kb)
    acc = product_i64(Am, Bm) + b
    C = output(M, N, torch.int32 if out == "i32" else torch.int8, 9)
    if out == "i32":
        ops.ac_gemm_i8_acc32(A, B, b, C[:M])
        check_equal(C[:M], acc)
    else:
        if ta or tb:
            ops.ac_gemm_i8_t(A, B, b, C[:M], 11, 0, trans_a=ta, trans_b=tb)
        else:
            ops.ac_gemm_i8(A, B, b, C[:M], 11, 0)
        check_equal(C[:M], requantise(acc, 11, 0))
    assert (C[M] == 9).all()


@pytest.mark.parametrize("M,N,K,dw", SHORT_AT_BT)
def test_short_at_bt(M, N, K, dw):
    A, B, Am, Bm = operands(M, N, K, torch.int8, K, True, True, dw)
    b = bias_of("row", M, N, K)
    C = output(M, N, torch.int8, 9)
    ops.ac_gemm_i8_t(A, B, b, C[:M], 10, 0, trans_a=True, trans_b=True)
    check_equal(C[:M], requantise(product_i64(Am, Bm) + b, 10, 0))
    assert (C[M] == 9).all()


@pytest.mark.parametrize("rounds", ROUNDS)
@pytest.mark.parametrize("shift,kind", [(1, "row"), (17, "row"), (9, "none"), (9, "matrix"), (18, "row"), (0, "row")])
def test_output_stage_i8(rounds, shift, kind):
    """Shifts and biases that the loop's output stage has and, around them, those that it leaves to the ping-pong loop."""
    M, N, K = shape_of("i8", rounds, 4304)
    A, B, _, _ = operands(M, N, K, torch.int8, shift)
    b = bias_of(kind, M, N, shift)
    acc = product_i64(A, B) + (0 if b is None else b)
    for act in (0, 1):
        C = output(M, N, torch.int8, 9)
        ops.ac_gemm_i8_planned(A, B, b, C[:M], shift, act, 256, 1)
        check_equal(C[:M], requantise(acc, shift, act))
        assert (C[M] == 9).all()


@pytest.mark.parametrize("rounds", ROUNDS)
@pytest.mark.parametrize("kind", ["none", "matrix"])
@pytest.mark.parametrize("form", ["i32", "i32_dw"])
def test_output_stage_i32(form, kind, rounds):
    M, N, K = shape_of(form, rounds, 4228 if FORMS[form][4] else 4304)
    A, B, Am, Bm = operands(M, N, K, torch.int8, 3, dword=FORMS[form][4])
    b = bias_of(kind, M, N, 4)
    C = output(M, N, torch.int32, 9)
    ops.ac_gemm_i8_acc32(A, B, b, C[:M])
    check_equal(C[:M], product_i64(Am, Bm) + (0 if b is None else b))
    assert (C[M] == 9).all()


@pytest.mark.parametrize("rounds", ROUNDS)
@pytest.mark.parametrize("form", ["bf16", "bf16_dw"])
def test_output_stage_bf16(form, rounds):
    M, N, K = shape_of(form, rounds, 4164 if FORMS[form][4] else 4160)
    A, B, Am, Bm = operands(M, N, K, torch.bfloat16, 5, dword=FORMS[form][4])
    old = matrix(M, N, torch.bfloat16, 6).float()
    C = old.clone()
    ops.ac_gemm_bf16(A, B, C, 0.5, -2.0)
    check_bf16_product(Am, Bm, C, 0.5, -2.0, old)


@pytest.mark.parametrize("shift,kind", [(1, "row"), (17, "none"), (11, "matrix"), (18, "row")])
@pytest.mark.parametrize("M,N,K", CHOSEN_128X256)
def test_128x256(M, N, K, shift, kind):
    A, B, _, _ = operands(M, N, K, torch.int8, M + shift)
    b = bias_of(kind, M, N, shift)
    C = output(M, N, torch.int8, 9)
    ops.ac_gemm_i8(A, B, b, C[:M], shift, 1)
    check_equal(C[:M], requantise(product_i64(A, B) + (0 if b is None else b), shift, 1))
    assert (C[M] == 9).all()


@pytest.mark.parametrize("shift,kind", [(2, "row"), (17, "none"), (11, "matrix")])
@pytest.mark.parametrize("M,N,K", CHOSEN_AT_BT)
def test_128x256_at_bt(M, N, K, shift, kind):
    A, B, Am, Bm = operands(M, N, K, torch.int8, M + shift, True, True)
    b = bias_of(kind, M, N, shift)
    C = output(M, N, torch.int8, 9)
    ops.ac_gemm_i8_t(A, B, b, C[:M], shift, 1, trans_a=True, trans_b=True)
    check_equal(C[:M], requantise(product_i64(Am, Bm) + (0 if b is None else b), shift, 1))
    assert (C[M] == 9).all()


def test_output_beside_other_columns():
    """C with a pitch of its own: the columns behind N stay."""
    M, N, K = shape_of("i8", "one", 4288)
    A, B, _, _ = operands(M, N, K, torch.int8, 7)
    b = bias_of("row", M, N, 8)
    C = torch.full((M, N + 16), 9, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8_planned(A, B, b, C[:, :N], 9, 1, 256, 1)
    check_equal(C[:, :N], requantise(product_i64(A, B) + b, 9, 1))
    assert (C[:, N:] == 9).all()
