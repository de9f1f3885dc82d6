// When two scores of the k-means assignment are too close for the matrix cores to tell which is larger, in one place and
// as plain functions, so that they can be checked on the host.
//
// A score is s = x.c - |c|^2/2 = (|x|^2 - |x - c|^2) / 2; with M = max(|x|^2, max_j |c_j|^2) it lies between -1.5 M and
// M/2, and so does every partial sum of it (in any order; bounded by |x||c| + |c|^2/2 <= 1.5 M).  Model of the hardware:
// the products of bf16 values are exact, and each of the accumulation steps (128, in the tiled kernel 131: it adds the
// offset as three more products) loses at most one unit in the last place of such a partial sum, 2^-23 of it.  That is at
// most 1.54 * 2^-16 M a score, and |c|^2/2 itself is a dozen fp32 roundings off, 0.05 * 2^-16 M.
// While the scores are compared, a few of their lowest mantissa bits carry an index: a change of less than 2^bits units in
// the last place of the score.
#pragma once

namespace mp {

constexpr int kTiledSlotBits = 4;
constexpr int kResidentSlotBits = 6;

// Below the normal range of fp32 all of this is absolute: a step loses at most 2^-126 even if subnormal numbers are flushed, some
// 140 steps and a product each 2^-117 a score, the index bits far less.  kNearFloor covers two scores of it (keys smaller than
// 1e-14 then go to the exact pass, all of them).
constexpr float kNearFloor = 0x1p-110f;

// Scores whose index bits are four (2^-19 of at most 1.5 M each), or that carry none: two of them are off by less than
// 3.6 * 2^-16 M (3.2 without index bits) together.  M is an fp32 sum, less than 2^-16 of it off.
constexpr float near_margin(float m) { return m * (4.0f / 65536.0f) + kNearFloor; }

// Scores that carry six bits: 2^-17 of their size each, of which the size matters: of two scores, only one that is no
// further from the best than the margin can have been confused with it, so 2^-16 |best| covers both.  3.2 * 2^-16 M +
// 2^-16 |best| in all, which for a best score above zero (at most M/2) is still less than the margin of four bits; but a
// point far from every centroid has scores down to -1.5 M.
constexpr float near_margin_of_best(float m, float best)
{
    return (3.25f * m + (best < 0.0f ? -best : best)) * (1.0f / 65536.0f) + kNearFloor;
}

// What a step keeps as the score of the centroid it chose, for a later step to compare with the scores of others.  The best score
// is that centroid's own unless it was a near tie: then another one's, whose error goes with an M it may take with it when it
// moves away.  The chosen one's true score is no lower than that one's, which is at least the best less its error, so the best less
// the margin (more than twice that error) is below it with nothing left to allow for.
constexpr float kept_score(bool near, float best, float margin) { return near ? best - margin : best; }

}  // namespace mp
