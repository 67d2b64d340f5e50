// What the host decides about a backward launch, from what it knows of a bag.  Plain C++, so that a test can compare it with the
// queues the kernels build (tests/queue_model.cpp).
#pragma once

#include <stdint.h>

namespace knap {

// The dK/dV kernel takes 2 or 4 wave pairs per workgroup and this many workgroups on each CU: two waves per SIMD is what
// its registers allow, three with two pairs at d = 64.
constexpr int dkdv_workgroups_per_cu(int d, int pairs) { return d == 64 && pairs == 2 ? 3 : 4 / pairs; }
constexpr int dkdv_waves_per_simd(int d, int pairs) { return d == 64 && pairs == 2 ? 3 : 2; }

// Rounds of `slots` workgroups that a bag's items take without the mask, its sequences taken to be of one length: whole ones
// where there are few, and as many as the items fill where there are so many that the shorter sequences even out the last.
inline double rounds(int64_t total_tokens, int n_seq, int H, int tile, int64_t slots) {
  const int64_t items = ((total_tokens + n_seq - 1) / n_seq + tile - 1) / tile * n_seq * H;
  return items >= 8 * slots ? (double)items / slots : (double)((items + slots - 1) / slots);
}

// Wave pairs per workgroup of the dK/dV kernel where it is a launch of its own (2 or 4, see there), from what the host knows of
// a bag: its tokens, heads and number of sequences.  Both sides measured on bags that bwd_joint() leaves to two launches,
// four pairs | two, forward and backward in us at 24 heads of 128 where nothing else is said.
//  * At most half a 256-key tile per CU: two, which spread the keys over twice as many CUs (hundreds of sequences of a few
//    tokens each).
//  * Short sequences: two, which hide the start and the end of every item: 60 of 350 tokens 730 | 671, 32 of 450 548 | 545; under
//    the mask 128 of 450 1654 | 1592.  The average does not show one long sequence among many short ones, where two pairs lose as
//    soon as the long one's tiles fill the GPU (half of 60000 tokens in one, under the mask, 23359 | 24010); the bounds on the
//    whole bag are a compromise between such bags and those of like lengths.
//  * Without the mask, where four pairs would have six rounds or more: two at averages below 3000 (60 of 800 2563 | 2474, 20 of
//    2600 6881 | 6887; 20 of 3000 8818 | 8877, 16 of 4096 12526 | 12689), but not from 512 to 640.  That band is kept for one long
//    sequence among short ones (half of 60000 tokens in one 42090 | 42985; 65536 and 200 short, dK/dV alone, 81.4 | 84.4 ms), and
//    bags of like lengths pay for it: 60 of 600 1565 | 1494, 80 of 560 1910 | 1821.  By tokens and number of sequences they
//    are the same bags.
//  * Fewer than six rounds: two where the smaller tiles save one (a single sequence of 2680 tokens: 465 | 373).
//  * d = 64, where three workgroups of two pairs share a CU: always two (dK/dV alone, 32 of 450 tokens, 48 heads, 289 | 246; 65536
//    103.3 | 98.1 ms).
//  * Otherwise four: one of 30000, 12 heads, 21968 | 22633; of 4292, 14 heads, 540 | 555; of 4825 under the mask 638 | 658.
inline int dkdv_pairs(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  if (d == 64 || total_tokens * H <= (int64_t)cus / 2 * 256) return 2;
  const int64_t n = n_seq;
  if (causal) return total_tokens <= 65536 && total_tokens < 4096 * n ? 2 : 4;
  if (total_tokens < 512 * n && total_tokens <= 16384) return 2;
  const double four = rounds(total_tokens, n_seq, H, 256, cus);
  if (four >= 6.0)
    return total_tokens < 512 * n || (total_tokens >= 640 * n && total_tokens < 3000 * n) ? 2 : 4;
  return total_tokens >= 640 * n && rounds(total_tokens, n_seq, H, 128, 2 * (int64_t)cus) < 0.9 * four ? 2 : 4;
}

// Whether both kinds of items go out in one launch (knap_attn_joint.h), behind the kernel that forms delta, or the dQ kernel
// and then the dK/dV kernel.  One launch has one last round to fill where two have two, spreads every sequence over the XCDs,
// and takes two wave pairs per workgroup for the keys.  Two launches | one, forward and backward in us at 24 heads of 128 where
// nothing else is said, n rounds of 128-row tiles: 4 sequences of up to 311 tokens, 2 x 64, 29.6 | 23.5; 4000, 3 x 128 (0.2), 229 |
// 188; one of 3000 (1.1) 578 | 489, of 4292 (1.6) 1077 | 944; 5 of up to 4346 (4.2) 1617 | 1600; 40 of 600 (9.4) 1080 | 1025; 10 of
// up to 6795, 48 x 64 (11), 5936 | 5814; 17 of 328..4533 (12) 4354 | 4353, under the mask (6.4) 2566 | 2527.  Two where
//  * the rounds are many, above 13, where one launch no longer gains on every kind of bag: 16 of 4096 (24) 12534 | 12681, images and
//    videos (25) 25844 | 26058, but 23 of 328..4533 (17) 6444 | 6416, half of 40000 tokens in one (16) 19838 | 18615;
//    and at d = 128, where four wave pairs are the better ones for long sequences, above 4 of those: 131072, 32768 and 4 of 8192,
//    3 heads (9), 101.3 ms | 106.2; but 40000, 12 heads (7.3), 37.7 | 37.4, and 60000, 3 heads (2.7), 22.3 | 21.5;
//  * short sequences fill several: 128 of 450 under the mask, 12 heads (6), 822 | 850; 32 of 450 (6) 547 | 546;
//  * each kernel has one round that is nearly full, of one sequence: 4000, 15 heads (0.9), 503 | 547; 4825, 12 heads (0.9), 585 | 632,
//    under the mask, 24 heads, 636 | 668.
// One launch loses where a long sequence's 256-key tiles just fill the GPU once, beside short ones (9000 tokens and 30 short, 6 heads,
// 1081 | 1200; 4500 and 15 short 406 | 319): by tokens and number of sequences these are the same bags as others that gain.
inline bool bwd_joint(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  const int64_t tiles = ((total_tokens + n_seq - 1) / n_seq + 127) / 128;
  const double r = (double)((causal ? (tiles + 1) / 2 : tiles) * n_seq * H) / (double)((int64_t)cus * dkdv_workgroups_per_cu(d, 2));
  if (r > 13.0 || (r > 4.5 && total_tokens < 500 * (int64_t)n_seq)) return false;
  if (d == 128 && r > 4.0 && total_tokens > 16384 * (int64_t)n_seq) return false;
  return !(n_seq == 1 && r > 0.8 && r <= 1.0);
}

// Whether that launch takes items of 64 rows (knap_attn_bwd_small.hip), twice as many, of half the length each, and single tiles under the
// mask: up to as many rounds of 128-row tiles as leave a workgroup for every one of them, a quarter; under the mask, where pairs of
// 128-row tiles leave more of the GPU idle, somewhat more.  128 rows | 64, backward in us, n the rounds.  Without the mask: one of 4776, 3 x
// 128 (0.22), 162 | 123; one of 10784, 2 x 64 (0.22), 273 | 219; 2021 in 10, 6 x 128 (0.23), 24.0 | 21.4; one of 1500, 12 x 128 (0.28), 64 | 72;
// one of 544, 48 x 64 (0.31), 25.9 | 28.7.  Under it: one of 4776, 3 x 128 (0.22), 176 | 104; one of 16682, 2 x 64 (0.34), 470 | 429, of 19631
// (0.40) 547 | 560; 9960 in 3, 3 x 128 (0.46), 172 | 137; 4536 in 10, 6 x 128 (0.47), 47 | 37; one of 10019, 3 x 128 (0.46), 346 | 375; 10525 in 19, half
// of them in one, 3 x 128 (0.56), 201 | 131; 1862 in 4, 24 x 128 (0.75), 50 | 54.  Without the mask bags of one long and many short sequences gain up to a
// half (8352 in 14, 3 x 128, 165 | 118), and bags of like lengths of the same numbers lose up to 8 %.  Bags of other lengths than the average's lose
// by it: small_pays() takes those back.
inline bool bwd_small(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  const int64_t tiles = ((total_tokens + n_seq - 1) / n_seq + 127) / 128;
  const double r = (double)(tiles * n_seq * H) / (double)((int64_t)cus * dkdv_workgroups_per_cu(d, 2));
  return r <= (!causal ? 0.25 : n_seq == 1 ? 0.375 : 0.55);
}

// Whether items of 64 rows pay after all: decided in front of that launch on the device, which knows the lengths.  tiles: of 64 rows, of
// all sequences of a head; longest: those of the longest.  Where not, the launch takes items of 128 rows.  Backward in us, 128 rows | 64, n
// the workgroups' worth of 64-row items of both kinds; 583 bags without the mask and 623 under it.
//  * Without the mask: where each item has a workgroup.  Sequences of 1 and 200 tokens in turn, 3 x 128: 34 (n = 1.0) 23.7 | 21.1, 40 (1.17) 25.3 |
//    26.9; 92, 2 x 64 (1.2), 20.3 | 25.9.
//  * Under it items of half the average length fill in behind the long ones, so that more than one worth pays, but not
//    - of one long sequence, alone or beside a few short ones, where the longer walks count and not the starts: one of 7864, 3 x 128 (1.44), 285 |
//      273, 9175 and 1 (1.7) 320 | 338; 24576 and 1, 2 x 64 (2.0), 725 | 911; but 18432 and 20 of 300 (2.0) 533 | 516;
//    - of sequences up to 128 tokens, each one item of 128 rows, from one worth on until those need a second round as well: 32 of 128, 6 x
//      128 (1.5), 23.6 | 27.7, 46 (2.16) 36.2 | 35.2; 24 of 96, 12 x 64 (1.5), 16.4 | 23.9; 46 of 64, 6 x 128 (1.08), 29.5 | 24.5;
//    - at d = 64, where a 128-row item of two tiles is short as well, up to 192 tokens, and up to 256 from one and a half on: 24 of 160, 6 x 64
//      (1.12), 18.9 | 20.8; 24 of 256 (1.5) 26.5 | 26.4, 35 (2.19) 28.4 | 33.9; but 23 of 320 (1.8) 31.2 | 29.8, and 32 of 192, 6 x 128 (1.12), 28.3 | 24.0.
constexpr bool small_pays(int tiles, int longest, int H, int slots, int d, bool causal) {
  const int64_t both = 2 * (int64_t)tiles * H, n = slots;
  if (!causal) return both <= n;
  if (longest > 128 && 4 * (int64_t)longest >= 3 * (int64_t)tiles) return 5 * both <= 8 * n;
  if (longest == 2) return 10 * both <= 11 * n || (d == 128 && both > 2 * n);
  if (d == 64 && longest == 3) return 10 * both <= 11 * n;
  if (d == 64 && longest == 4) return 50 * both <= 76 * n;
  return true;
}

// Whether that is so whatever the lengths are (L tokens have at most (L + 63) / 64 tiles, and the longest sequence the average): such bags
// take a kernel without the other form, whose prologue and code are shorter: half a us of 10 to 60 (134 bags, 2.7 %).
inline bool small_sure(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  const int64_t slots = (int64_t)cus * dkdv_workgroups_per_cu(d, 2), most = 2 * ((total_tokens + 63 * (int64_t)n_seq) / 64) * H;
  if (!causal) return most <= slots;
  if (10 * most <= 11 * slots) return true;
  return total_tokens > (d == 128 ? 128 : 256) * (int64_t)n_seq && (total_tokens <= 8192 || 5 * most <= 8 * slots);
}

// Counter sets of the forward's work queues.  The forward entry points have no workspace: a launch draws from one of these sets
// (8 counters each, at zero in the device image), which it leaves at zero.  Eager calls take the first 3 kSetsPerThird in
// rotation.  Calls that share a set because too many were enqueued while one ran lose items and may leave the set at
// another value than zero; so that this ends, and does not spoil a launch of every later turn, the call that
// enters a third clears the one that follows.  Nobody draws from that one as long as no call runs beside one that is
// kSetsPerThird calls younger: it was left that many calls ago, and is entered that many later.  One launch of 128
// workgroups in 4096 calls.  The sets behind belong to launches recorded under stream capture, which keep theirs for every
// replay.
constexpr unsigned kSetsPerThird = 4096, kCapturedSets = 4096, kQueueSets = 3 * kSetsPerThird + kCapturedSets;

struct EagerSet {
  unsigned set;
  int clear;        // the first of kSetsPerThird sets to clear on the call's stream before its launch, or -1
};

inline EagerSet eager_set(uint64_t call) {
  const uint64_t third = call / kSetsPerThird;
  return {(unsigned)(call % (3 * kSetsPerThird)), call % kSetsPerThird == 0 ? (int)((third + 1) % 3 * kSetsPerThird) : -1};
}

inline unsigned captured_set(uint64_t call) { return 3 * kSetsPerThird + (unsigned)(call % kCapturedSets); }

}  // namespace knap
