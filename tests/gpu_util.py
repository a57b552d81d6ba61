"""Helpers shared by the GPU parity tests (device upload, error norms)."""
import numpy as np
import torch


def dev(a):
    """numpy -> device tensor; uint16 arrays are taken as bf16 bit patterns."""
    if a is None:
        return None
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16).copy()).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


def rel_fro(got, want):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    den = np.linalg.norm(want.ravel())
    num = np.linalg.norm((got - want).ravel())
    return num / den if den > 0 else num


def requantise(acc, shift, act):
    """The int8 output stage on a tensor of int64 sums: acc / 2^shift to nearest, halves to even, clamped, then ReLU."""
    q = acc
    if shift > 0:
        low, rem, half = acc >> shift, acc & ((1 << shift) - 1), 1 << (shift - 1)
        q = low + ((rem > half) | ((rem == half) & (low & 1 == 1))).to(acc.dtype)
    return q.clamp(0 if act else -128, 127).to(torch.int8)


def product_i64(A, B):
    """Every sum of an int8 product, exact: fp64 holds the integers up to 2^53."""
    return (A.double() @ B.double()).to(torch.int64)


def check_equal(got, want):
    """Two whole matrices on the device, element by element."""
    assert got.shape == want.shape
    if not torch.equal(got, want.to(got.dtype)):
        bad = (got != want.to(got.dtype)).nonzero()
        r, c = bad[0].tolist()
        raise AssertionError(f"{len(bad)} of {got.numel()} elements differ, first at ({r}, {c}): {got[r, c].item()} for {want[r, c].item()}; "
                             f"rows % 16 {sorted(set((bad[:, 0] % 16).tolist()))}, bands of 16 rows {sorted(set((bad[:, 0] // 16 % 16).tolist()))}")


def check_bf16_product(A, B, got, alpha=1.0, beta=0.0, old=None):
    """Every element of got = alpha A . B + beta old on the device (A, B bf16, got and old fp32) against fp64.  A sum of K exact products
    in fp32 in any order is off by at most (K + 2) 2^-24 sum_k |a_k b_k| to first order; the two scalings and the addition round three
    times more.  Four times that is allowed."""
    K = A.shape[1]
    want, mag = alpha * (A.double() @ B.double()), abs(alpha) * (A.double().abs() @ B.double().abs())
    bound = (K + 2) * mag
    if beta != 0.0:
        want += beta * old.double()
        bound += 3 * (mag + abs(beta) * old.double().abs())
    bad = ~((got.double() - want).abs() <= 4 * 2.0 ** -24 * bound + 1e-30)  # NaN fails
    assert not bad.any(), f"{int(bad.sum())} of {got.numel()} elements beyond the bound, first at {bad.nonzero()[0].tolist()}"


def check_bf16_product_in_full(A_bits, B_bits, got, block_rows=2048):
    """Every element of got (fp32, M x N) against the fp64 oracle of the bf16 product A . B, in blocks of rows so
    that the fp64 copies stay small: relative Frobenius error <= 1e-3 over the whole matrix, and element by element
    |err| <= 4 (K + 2) 2^-24 sum_k |a_k b_k| (fp32 accumulation in any order)."""
    import oracle
    from paper_2505_18574_amd import inputs

    M, K = A_bits.shape
    num = den = 0.0
    Ba = np.abs(inputs.bf16_bits_to_f32(B_bits).astype(np.float64))
    for r0 in range(0, M, block_rows):
        r1 = min(M, r0 + block_rows)
        want = oracle.gemm_bf16(A_bits[r0:r1], B_bits)
        g = got[r0:r1].astype(np.float64)
        assert np.isfinite(g).all()
        err = np.abs(g - want)
        mag = np.abs(inputs.bf16_bits_to_f32(A_bits[r0:r1]).astype(np.float64)) @ Ba
        bad = err > 4.0 * (K + 2) * 2.0 ** -24 * mag + 1e-30
        assert not bad.any(), f"rows {r0}..{r1}: {int(bad.sum())} elements beyond the bound, first at {np.argwhere(bad)[0]}"
        num += float((err * err).sum())
        den += float((want * want).sum())
    assert np.sqrt(num) <= 1e-3 * np.sqrt(den)
