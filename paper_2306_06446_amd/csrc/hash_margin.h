// What the matrix-core hash (binarize_mfma.hip, and in the projection's launches norm_hash.hip and linear_hash.hip) may get wrong
// before it asks the defining chain, in one place, so that its margin is a proof and not a measurement.  The three add their
// products in different orders; the bound on the accumulation holds for any.  Plain C++: the test suite compiles it on the host.
//
// With X = |x| and a column r of which the kernel holds r^ = r / |r| in units of 1 / 1024, z~ = xh rh + xh rl + xl rh in
// fp16 terms with fp32 sums.  The sign of z~ is that of the chain if |z~| exceeds X times the sum of, each relative to
// X |r^| (Cauchy-Schwarz: sum |x_k r^_k| <= X |r^|):
//   * the fp32 accumulation of the 3 d products: 3 d 2^-23, even if every addition truncates;
//   * the defining chain: d roundings, d 2^-24;
//   * the terms.  Rounding an operand to fp16 twice leaves 2^-22 of it, or 2^-25 where the lower term is below fp16's normal
//     range: with the row's d elements together 2^-22 + sqrt(d) 2^-25 / X, with the column's 2^-22 + sqrt(d) 2^-35.  The
//     product of the lower terms is dropped: about 2^-22;
//   * the rounding of r_k / |r|: 2^-24 of each element.
// Everything of second order (the roundings of the two norms and of the threshold itself, at most 70 * 2^-24 of it; the growth of
// the partial sums, 2^-9; chain sums in denormal range, 2^-32) is covered by 2^-7 of the total.
#pragma once

namespace sa {

// |z~| > theta |x| keeps the sign of z~.
constexpr float hash_theta(int d) { return d == 32 ? 0x1p-16f : (d == 64 ? 0x1p-15f : 0x1p-14f); }

// Rows with |x|^2 in this range split as they are: nothing overflows fp16, and the lower terms lose little to its subnormals.
// Others are brought to |x| in 0.5 .. 1.42 first (a power of two: exact).
constexpr float kOrdinaryMin2 = 0x1p-4f, kOrdinaryMax2 = 0x1p24f;
constexpr double kSplitMin = 0.25;              // the smallest |x| that is split: the square root of kOrdinaryMin2, below 0.5

// Columns whose |r|^2 is below that (its squares may have underflowed) or not finite are left to the chain altogether.
constexpr float kColumnMin2 = 0x1p-100f;
constexpr float kColumnScale = 1024.0f;         // |r^| as staged: its lower terms are then normal fp16 numbers
constexpr float kKeepFloor = 3.2e-19f;          // |z| below that: products and sums of the chain may be denormal

constexpr double hash_sqrt_bound(int d) { return d == 32 ? 5.66 : (d == 64 ? 8.0 : 11.32); }

// The terms of a row of length x against a column, over x |r^|.
constexpr double hash_split_error(int d, double x) {
    const double s = hash_sqrt_bound(d), l = 0x1p-11 * (1.0 + 0x1p-11);
    const double row = 0x1p-22 + s * 0x1p-25 / x, column = 0x1p-22 + s * 0x1p-35;
    return row + column * (1.0 + 0x1p-10) + (l + s * 0x1p-23 / x) * (l + s * 0x1p-33);
}
constexpr double hash_error(int d) {
    return (3.0 * d * 0x1p-23 + d * 0x1p-24 + hash_split_error(d, kSplitMin) + 0x1p-24) * (1.0 + 0x1p-7);
}
static_assert(kSplitMin <= 0.5 && kSplitMin * kSplitMin <= (double)kOrdinaryMin2, "every row that is split is at least that long");
static_assert(hash_error(32) < (double)hash_theta(32) && hash_error(64) < (double)hash_theta(64) &&
                  hash_error(128) < (double)hash_theta(128),
              "the margin covers every error");

}  // namespace sa
