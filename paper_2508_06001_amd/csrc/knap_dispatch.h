// What the host decides about a backward launch, from what it knows of a bag.  Plain C++, so that a test can compare it with the
// queues the kernels build (tests/queue_model.cpp).
#pragma once

#include <stdint.h>

namespace knap {

// The dK/dV kernel takes 2 or 4 wave pairs per workgroup and this many workgroups on each CU: two waves per SIMD is what
// its registers allow, three with two pairs at d = 64.
constexpr int dkdv_workgroups_per_cu(int d, int pairs) { return d == 64 && pairs == 2 ? 3 : 4 / pairs; }
constexpr int dkdv_waves_per_simd(int d, int pairs) { return d == 64 && pairs == 2 ? 3 : 2; }

// Rounds of `slots` workgroups that a bag's items take, its sequences taken to be of one length: whole ones where there
// are few, and as many as the items fill where there are so many that the shorter sequences even out the last.
inline double rounds(int64_t total_tokens, int n_seq, int H, bool causal, int tile, int64_t slots) {
  const int64_t tiles = ((total_tokens + n_seq - 1) / n_seq + tile - 1) / tile;
  const int64_t items = (causal ? (tiles + 1) / 2 : tiles) * n_seq * H;
  return items >= 8 * slots ? (double)items / slots : (double)((items + slots - 1) / slots);
}

// Wave pairs per workgroup of the dK/dV kernel (2 or 4, see there), from what the host knows of a bag: its tokens, heads
// and number of sequences.  Both sides measured, two pairs against four: times of that kernel where nothing else is said.
//  * At most half a 256-key tile per CU: two, which spread the keys over twice as many CUs (3 causal sequences of up to
//    391 tokens, 6 x 128: 38 against 51 us; 2 of up to 4362, 2 x 64: 104 against 150 us).
//  * Many short sequences: two, which hide the start and the end of every item (32 of 450 tokens, 24 x 128: 249 against
//    276 us; 17 causal ones of 328..4533 tokens: 1125 against 1240 us).
//    The average does not show one long sequence among many short ones, where two pairs lose as soon as the long one's
//    tiles fill the GPU; the bounds on the whole bag are a compromise between such bags and those of like lengths.  Causal,
//    d = 128, whole backward in us: 20 of 3000 tokens, 24 heads 3904 against 4023; 128 of 450, 24 heads 1227 against 1332; 30 of
//    1100, 3 heads 158 against 225; but 30000 and 30 of 300, 12 heads 8752 against 8394; half of 60000 tokens in one
//    sequence, 24 heads 17234 against 16973, 3 heads 2627 against 2464 (of 30000, 12 heads 3047 against 2930; of 20000, 6 heads,
//    where the GPU is not full, 686 against 755).
//    Without the mask at d = 128: up to 16384 tokens at an average below 512 (32 of 450, 24 x 128: 233 against 267 us; but
//    4405, 619 and 371: 490 against 463; 4200 and seven of 450, 12 x 128: 247 against 229).  Where four pairs would have six
//    rounds or more, at averages below 3000 (12 of 2600, 24 x 128: 1704 against 1818 us; 17 of 328..4533: 1806 against
//    1837; 60 of 800: 1011 against 1154; 64 of 450: 409 against 433, with 6 heads and three rounds 122 against 114; 20 of
//    3000: 3796 against 3778) but those from 512 to 640, which are mostly one long sequence among short ones (16384 and
//    30 of 300: 5358 against 5117; 65536 and 200 short 84.4 against 81.4 ms; but 60 of 600: 592 against 700 us).  And where
//    the smaller tiles save a round (15 of 640: 174 against 216 us).
//  * d = 64, where three workgroups of two pairs share a CU: always two (the bags that leave it to be chosen have many
//    rounds or short sequences.  32 of 450 tokens, 48 x 64: 246 against 289 us; 16 of 4096: 6389 against 7163; 65536: 98.1
//    against 103.3 ms; causal, 20 of 3000: 2637 against 2970 us, 65536: 51.6 against 52.1 ms).
//  * Otherwise four (65536 and 200 short, 24 x 128: 80.3 against 82.4 ms; 30000 tokens, 3 x 128: 2.90 against 3.13 ms).
inline int dkdv_pairs(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  if (d == 64 || total_tokens * H <= (int64_t)cus / 2 * 256) return 2;
  const int64_t n = n_seq;
  if (causal) return total_tokens <= 65536 && total_tokens < 4096 * n ? 2 : 4;
  if (total_tokens < 512 * n && total_tokens <= 16384) return 2;
  const double four = rounds(total_tokens, n_seq, H, causal, 256, cus);
  if (four >= 6.0)
    return total_tokens < 512 * n || (total_tokens >= 640 * n && total_tokens < 3000 * n) ? 2 : 4;
  return total_tokens >= 640 * n && rounds(total_tokens, n_seq, H, causal, 128, 2 * (int64_t)cus) < 0.9 * four ? 2 : 4;
}

// Whether both kinds of items go out in one launch (knap_attn_joint.h), behind the kernel that forms delta, or the dQ kernel
// and then the dK/dV kernel.  One launch has one last round to fill where two have two, spreads every sequence over the XCDs,
// and takes two wave pairs per workgroup for the keys.  Backward in us, two launches against one, at n rounds of 128-row
// tiles: 4 sequences of up to 311 tokens, 2 x 64, 28 against 22; 4000, 3 x 128 (0.2): 184 against 145; one of 4292, 24 x 128
// (1.6): 828 against 762; 3000 (1.1): 506 against 369; 5 of up to 4346 (2.9): 951 against 851; 21 of up to 6108 (4.6): 1805
// against 1451; 17 of 328..4533 (11.5): 3356 against 3306, causal (6): 2036 against 1952; 10 of up to 6795, 48 x 64 (11):
// 4559 against 4477; 16 of up to 4393 (15.6): 4931 against 4865.  Two where
//  * the rounds are many: 20 of up to 4479 (20.9): 7016 against 7029; 16 causal ones of up to 25431 (13.9): 17860 against 18017,
//    and at d = 128, where four wave pairs are the better ones for long sequences, fewer of those: 131072, 32768 and 4 of 8192,
//    3 heads (9) 76.8 ms against 80.5; but 60000, 3 heads (2.7) 16.7 against 16.0;
//  * short sequences fill several: 32 of 450 (6): 423 against 437, 128 of 450, 12 x 128, causal (7): 643 against 660;
//  * each kernel has one round that is nearly full, of one sequence: 4825 causal (0.9): 487 against 510.
inline bool bwd_joint(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  const int64_t tiles = ((total_tokens + n_seq - 1) / n_seq + 127) / 128;
  const double r = (double)((causal ? (tiles + 1) / 2 : tiles) * n_seq * H) / (double)((int64_t)cus * dkdv_workgroups_per_cu(d, 2));
  if (r > 13.0 || (r > 4.5 && total_tokens < 500 * (int64_t)n_seq)) return false;
  if (d == 128 && r > 4.0 && total_tokens > 16384 * (int64_t)n_seq) return false;
  return !(n_seq == 1 && r > 0.8 && r <= 1.0);
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
