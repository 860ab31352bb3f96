// The softmax reference of the bf16 attention kernels, scheduled and plain (attn_bf16.hip, attn_bf16_group.hip): a weight is
// exp2(logit - reference) in log2 units, and both kernels take the reference by the same rule, so that a column set that names every key gives
// the weights of dense attention.  It is taken from the maximum of the first 32 keys and raised, from the maximum of the running ones and
// by a whole number of units, where the sum of 16 weights of a lane exceeds kAttnGrowthLimit.
//
// Headroom.  The first 32 kept keys say little about the largest logit of a row: against their maximum alone some lane of a wave outgrew its
// reference in most of the first tiles of a block, at some 2000 ticks for all four waves of the scheduled kernel.  Sums and accumulators are
// floats that carry the same power of two as the weights, so only small weights are lost: below 2^-117 of a row's largest (a raise leaves the
// reference up to nine units above the maximum), 2^-125 without headroom.  A whole number, so that a weight is rounded to sixteen bits as without, but for the fp32
// rounding of reference and shifted logit.  Outputs are as far from 64 bits as without (differences below 0.02%).  The row log-sum-exp of dense attention takes
// the exponent of the sum into the reference (log2_of: the logarithm of a sum of 2^-8 and less is rounded more coarsely than a short row's
// was): rms error against 64 bits without headroom / with it / and log2_of, unit logits, 17 rows 1.7 / 2.0 / 1.6e-7, 256 rows 3.1 / 2.8 / 2.6e-7, 8192 rows
// 4.7 / 4.1 / 3.9e-7, three times as steep at D = 64, 64 rows 5.3 / 6.0 / 5.3e-7, 8192 rows 1.35 / 1.41 / 1.35e-6.  Two unit logits 0.5 / 2.0 / 1.2e-7: the shifted
// logits, eight instead of none, are rounded to 5e-7 where nothing averages that.
// 0 / 3 / 5 / 8 units, us: scheduled kernel, 64K rows, keep 10%, 5348 / 5187 / 5123 / 5107, 32K, keep 20%, 2698 / 2609 / 2559 / 2546, refresh_dense of 16K 5089 /
// 5011 / 4959 / 4934.  0 / 8 units: plain kernel, 32 heads of 4096 rows, keep 10%, 37.6 / 35.3, 4 heads of 8192 20.4 / 18.6, groups of 128 at 32
// heads of 8192 138.6 / 132.7.
#pragma once

namespace pulsecol {

constexpr float kAttnGrowthLimit = 256.0f;
constexpr float kAttnHeadroom = 8.0f;

}  // namespace pulsecol
