// The error bounds of the RVQ screen (k_rvq.hip).  Plain C++ (no device
// code), so the host-side tests check the constants that the kernels use.
//
// Screening margin for residual width R.  Everything is in the round's scaled
// units: codewords times a power of two that puts the codebook's larger
// coordinates near 2^RVQ_CB_EXP (see prep_codebook_block), residuals times
// that and a power of two of the token's own (tsc, RVQ_TOK_SCALE for most).
// With R~ = fp16(R), C~_j = fp16(C_j) (saturated; the matrix unit takes
// subnormals as they are), eR = ||R - R~|| and e_j = ||C_j - C~_j||, each
// plus RVQ_TINY for squares that underflow, the screen's score s~_j =
// ||C_j||^2 - 2 R~.C~_j (the squared norm exact after the first k-step: three
// bf16 pieces that sum to it exactly, times ones) satisfies
//   |s~_j - s_j| <= 2 (||R|| + eR) e_j + 2 eR (1 + 2^-8) ||C_j||
//                   + ka ||R|| ||C_j|| + k2 ||C_j||^2  =: Delta_j, where
// 2 R.C_j - 2 R~.C~_j = 2 R.(C_j - C~_j) + 2 (R - R~).C~_j gives the first
// two terms (Cauchy-Schwarz; ||C~_j|| <= ||C_j|| + e_j), and
//   ka = (8 R 2^-24            (fp32 accumulation of 2R~.C~, any order,
//                               relative error up to 2 u per addition)
//        + 2^-20 + 2^-16) (1 + 2^-7)  (norm rounding; an index tag in the
//                               low 4 mantissa bits, which moves a score by
//                               less than 2^-19 of |s~_j| <= ||C_j||^2 +
//                               2.02 ||R|| ||C_j||, doubled; ||R~|| ||C~||
//                               against ||R|| ||C||)
//   k2 = 4 (R + 4) 2^-24 + 2^-17 (accumulation and fp32 rounding of
//                               ||C_j||^2; the index tag, doubled)
// fp16 pieces (11 significant bits) keep the margin at about 2^-10
// ||R|| ||C_j||, a seventh of what bf16 pieces leave: on data-drawn
// codebooks a third of the token-rounds was undecided with bf16 (1B-model
// boundary, K = 1024) and 7 % is with fp16.
//
// The screen computes, per codeword, a certified lower bound of the exact
// score s_j = ||C_j||^2 - 2 R . C_j rather than the score itself: the norm
// columns of a codeword row hold (1 - RVQ_K2_SLACK k2) ||C_j||^2 (three bf16
// pieces, exact), ||C_j|| rounded up (two bf16 pieces) and e_j rounded up
// (one piece); the token's operand multiplies them by ones, by -b with
// b = (2 eR (1 + 2^-7) + ka ||R||) RVQ_K1_SLACK and by -c with
// c = 2 (||R|| + eR) RVQ_K1_SLACK, each rounded up to bf16, so that the
// accumulator ends at
//   L_j = s~_j - k2' ||C_j||^2 - b ||C_j||' - c e_j'  <=  s_j.
// The subtracted amount is at most RVQ_SUB_FACTOR Delta_j (bf16 rounding up
// of the coefficients and of e_j, 2^-7 each, and the slack), so
// s_j <= L_j + (RVQ_SUB_FACTOR + 1) Delta_j.
#pragma once

namespace mapl {

constexpr float rvq_margin_ka(int R) {
  return (8.0f * R / 16777216.0f + 1.0f / 1048576.0f + 1.0f / 65536.0f) * 1.0078125f;
}
constexpr float rvq_margin_k2(int R) { return 4.0f * (R + 4) / 16777216.0f + 1.0f / 131072.0f; }
constexpr float RVQ_K1_SLACK = 1.0002f * 1.01f;
constexpr float RVQ_K2_SLACK = 1.01f;
constexpr float RVQ_SUB_FACTOR = 1.03f;
// sqrt(1024) 2^-75, rounded up: what squares below 2^-150 can take from a norm
constexpr float RVQ_TINY = 0x1p-66f;
// The larger codebook coordinates land in [2^10, 2^11): fp16 has all its
// eleven bits down to 2^-24 of them (and loses one per power of two
// below) and saturates from 2^5 times them.  Tokens keep to 2^-5 of that, so
// that one 2^9 times the codebook's size still fits, or take a power of
// their own.
constexpr int RVQ_CB_EXP = 10;
constexpr float RVQ_TOK_SCALE = 0x1p-5f;

}  // namespace mapl
