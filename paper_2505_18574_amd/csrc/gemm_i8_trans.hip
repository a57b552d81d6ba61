// int8 GEMM with transposed operands (the A_transpose / B_transpose fields of the accelerator's config_ex,
// Appendix C Fig. 14): A may be given as A^T (K x M row-major) and B as B^T (N x K row-major).
//
// Either operand of the product is, in memory, "K-contiguous" (a row holds consecutive k: plain A, transposed
// B) or "K-strided" (a row holds consecutive m or n: transposed A, plain B), and is staged in LDS in its memory order;
// the fragment read that matches does the rest.
//
// Operands that qualify for the direct-to-LDS kernels (16-byte aligned bases and pitches, M, N and K in whole
// 16-byte chunks) run on those, with the transposed operand in the other operand's LDS role (TA / TB of
// gemm_dtl_kernel): the same tiles, pipeline and output stage as the untransposed product.  Everything else runs on
// the ragged kernel.
#include <algorithm>

#include "gemm_kgroup.hpp"

namespace ac {

template <bool TA, bool TB, bool DW>
static hipError_t launch_trans_dtl(const GemmParams& p0, hipStream_t stream) {
  GemmParams p = p0;
  p.splits = 1;
  p.kt_per_split = 0;
  if (kgroup_takes<TypeI8, TA, TB>(p, false, 1)) return launch_kgroup<TypeI8, KGroupI8, 0, TA, TB, DW>(p, stream);
  if constexpr (TA || !DW)  // (B^T on dwords never does)
    if (wide_trans_rule(p.M, p.N, p.K, TA, TB, DW)) return launch_dtl_wide<TypeI8, EpilogueI8, 0, DW, TA, TB>(p, stream);
  if constexpr (TA && TB && !DW)
    if (interleaved_at_bt_rule(p.M, p.N, p.K) && EpilogueI8::takes16(p.shift, p.bias, p.bias_ld)) return launch_dtl<TypeI8, EpilogueI8, 128, 256, 2, 2, 0, 4, 64, DTL_INTERLEAVED, TA, TB>(p, stream);
  switch (choose_tile_i8(p.M, p.N, p.K, false)) {  // no tile but the wide ones is other than square: the 256 x 128 code falls to 128
    case 256: return launch_dtl_256<TypeI8, EpilogueI8, 0, TA, TB, DW>(p, stream);
    case 192:
    case 128: return launch_dtl<TypeI8, EpilogueI8, 128, 128, 2, 4, 0, 3, 128, DTL_ROLLING, TA, TB, DW>(p, stream);
    default: return launch_dtl<TypeI8, EpilogueI8, 64, 64, 2, 2, 0, 4, 128, DTL_ROLLING, TA, TB, DW>(p, stream);
  }
}

// A is K x M when trans_a, B is N x K when trans_b (both row-major with their own leading dimension).
hipError_t launch_gemm_i8_trans(const GemmParams& p, bool trans_a, bool trans_b, hipStream_t stream) {
  if (!trans_a && !trans_b) return launch_gemm_i8(p, stream);
  // direct-to-LDS kernels: whole 16-byte chunks along every contiguous dimension, and row pitches that keep a lane's
  // offset from its tile's first row in 32 bits (a K-contiguous operand spans up to 320 rows, a K-strided one 128)
  const int64_t pitch_kc = std::max<int64_t>(trans_a ? 0 : p.lda, trans_b ? p.ldb : 0);
  const int64_t pitch_ks = std::max<int64_t>(trans_a ? p.lda : 0, trans_b ? 0 : p.ldb);
  const bool fast = (((uintptr_t)p.A | (uintptr_t)p.B) & 15) == 0 && p.lda % 16 == 0 && p.ldb % 16 == 0 && ((uintptr_t)p.C & 3) == 0 &&
                    p.ldc % 4 == 0 && p.K % 16 == 0 && p.N % 16 == 0 && (!trans_a || p.M % 16 == 0) && p.K > 0 &&
                    lane_offsets_fit(pitch_kc, pitch_ks);
  if (fast) {
    if (trans_a && trans_b) return launch_trans_dtl<true, true, false>(p, stream);
    if (trans_a) return launch_trans_dtl<true, false, false>(p, stream);
    return launch_trans_dtl<false, true, false>(p, stream);
  }
  if (dword_operands(p, 1, trans_a, trans_b, 4, 1) && (dword_tiles(p, 1, trans_a, trans_b) || wide_trans_rule(p.M, p.N, p.K, trans_a, trans_b, true) || kgroup_rule({p.M, p.N, p.K, 1, false, !trans_a, trans_b, p.ldb, 1, false, 0}))) {
    if (trans_a && trans_b) {
      if (!ragged_tiny<TypeI8, false, true, false>(p)) return launch_trans_dtl<true, true, true>(p, stream);
    } else if (trans_a) {
      if (!ragged_tiny<TypeI8, false, false, false>(p)) return launch_trans_dtl<true, false, true>(p, stream);
    } else if (!ragged_tiny<TypeI8, true, true, false>(p)) {
      return launch_trans_dtl<false, true, true>(p, stream);
    }
  }
  const int tile = ragged_tile(p.M, p.N);
  GemmParams q = p;
  q.splits = 1;
  q.kt_per_split = 0;
  auto ragged = [&](auto ta, auto tb) {
    constexpr bool AKC = !decltype(ta)::value, BKC = decltype(tb)::value;
    if (!ragged_tiny<TypeI8, AKC, BKC, false>(q) && kgroup_ragged_takes<TypeI8, AKC, BKC>(q, 1)) return launch_kgroup_ragged<TypeI8, KGroupI8, AKC, BKC>(q, stream);
    return launch_ragged<TypeI8, EpilogueI8Any, AKC, BKC>(tile, q, stream);
  };
  if (trans_a && trans_b) return ragged(std::true_type{}, std::true_type{});
  return trans_a ? ragged(std::true_type{}, std::false_type{}) : ragged(std::false_type{}, std::true_type{});
}

}  // namespace ac
