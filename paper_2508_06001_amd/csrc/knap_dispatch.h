// What the host decides about a backward launch, from what it knows of a bag.  Plain C++, so that a test can compare it with the
// queues the kernels build (tests/queue_model.cpp).
#pragma once

#include <stdint.h>

namespace knap {

// The dK/dV kernel takes 2 or 4 wave pairs per workgroup and this many workgroups on each CU (two waves per SIMD is what
// its registers allow).
constexpr int dkdv_workgroups_per_cu(int pairs) { return 4 / pairs; }

// Wave pairs per workgroup of the dK/dV kernel (2 or 4, see there), from what the host knows of a bag: its tokens, heads
// and number of sequences.  Both sides measured, two pairs against four: times of that kernel where nothing else is said.
//  * At most half a 256-key tile per CU: two, which spread the keys over twice as many CUs (3 causal sequences of up to
//    391 tokens, 6 x 128: 38 against 51 us; 2 of up to 4362, 2 x 64: 104 against 150 us).
//  * Many short sequences: two, which hide the start and the end of every item (32 of 450 tokens, 24 x 128: 249 against
//    276 us; 17 causal ones of 328..4533 tokens: 1125 against 1240 us; 10 of 310..6795 tokens, 48 x 64: 2806 against
//    3057 us).  The causal kernel at d = 64 has little of either to hide and is up to 8 % slower.
//    The average does not show one long sequence among many short ones, where two pairs lose as soon as the long one's
//    tiles fill the GPU; the bounds on the whole bag are a compromise between such bags and those of like lengths.  Causal,
//    d = 128, whole backward in us: 20 of 3000 tokens, 24 heads 3904 against 4023; 128 of 450, 24 heads 1227 against 1332; 30 of
//    1100, 3 heads 158 against 225; but 30000 and 30 of 300, 12 heads 8752 against 8394; half of 60000 tokens in one
//    sequence, 24 heads 17234 against 16973, 3 heads 2627 against 2464 (of 30000, 12 heads 3047 against 2930; of 20000, 6 heads,
//    where the GPU is not full, 686 against 755).  Without the mask at d = 64: 28000 and 8 of 500, 48 heads 31872 against
//    32436; half of 32000 in one, 48 heads 10575 against 11002, 12 heads 2816 against 2766.
//    Without the mask at d = 128 the line is at an average of 512: above it two pairs win where they pad less and lose
//    where the lengths are multiples of 256 or one sequence stands out (forward and backward, two against four: 15 of 640
//    tokens, 24 x 128: 471 against 506 us; but 10 of 1024: 669 against 652; 8 of 1200: 742 against 721; 4405, 619 and 371:
//    1135 against 1107; 4200 and seven of 300..600, 12 x 128: 611 against 582; 18 of 512: 208 both).  And at 16384 tokens:
//    beyond, short sequences gain nothing from two pairs (64 of 450, backward, 24 heads 835 against 827, 6 heads 226 against
//    220; 128 of 450, 24 heads 1619 against 1620), and a long one among them loses (8192 and 45 of 300, 6 heads 779 against 723).
//  * Otherwise four (65536 and 200 short, 24 x 128: 80.3 against 82.4 ms; 30000 tokens, 3 x 128: 2.90 against 3.13 ms).
inline int dkdv_pairs(int64_t total_tokens, int n_seq, int H, int d, bool causal, int cus) {
  if (total_tokens * H <= (int64_t)cus / 2 * 256) return 2;
  const int64_t longest_average = d == 128 && !causal ? 512 : 4096;
  const int64_t largest_bag = d == 64 ? (causal ? 0 : 32768) : (causal ? 65536 : 16384);
  if (total_tokens <= largest_bag && total_tokens < longest_average * n_seq) return 2;
  return 4;
}

// Whether some queue of the backward's kernels may hold more items than workgroups, so that the counters are used and
// have to be zeroed first.  A bag has at most T / tile + n_seq tiles per head.  Few enough that all parts of all items
// (four each under the mask, two without) find a workgroup: the dQ kernel deals out parts and draws none (see
// ItemQueue).  The dK/dV kernel's items, at most half as many as its workgroups, fill at most per / 2 tickets of a
// queue in whole rounds and a chunk of at most as many in the last.  Without the clearing launch: 4 sequences of up
// to 311 tokens, 2 x 64, forward and backward 36.1 -> 34.2 us; a bag past the line keeps it.
inline bool bwd_draws(int64_t total_tokens, int n_seq, int H, bool causal, int pairs, int cus, int grid_dq) {
  const int64_t items_dq = (total_tokens / 128 + n_seq) * H;
  const int64_t items_dkdv = (total_tokens / (64 * pairs) + n_seq) * H;
  return items_dq * (causal ? 4 : 2) > grid_dq || items_dkdv * 2 > cus * dkdv_workgroups_per_cu(pairs);
}

}  // namespace knap
