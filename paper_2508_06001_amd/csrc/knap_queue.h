// Work queues of the persistent attention kernels: which workgroup takes which item of the descending-cost item list.
// Integer arithmetic on the schedule alone, so that the host can walk through it as well (tests/queue_model.cpp).
#pragma once

namespace knap {

// Items of a sequence and head: its tiles, or pairs of them (causal attention).
template <bool PAIRED>
__device__ __forceinline__ int items_per_head(int tiles) { return PAIRED ? (tiles + 1) >> 1 : tiles; }

// Items of the sequences at least half as long as the longest one, or `enough` if there are that many:
// the band of dear items that has to be spread over the whole GPU.  Items per sequence fall along the order.
__device__ __forceinline__ int dear_items(const int* s_start, int n_seq, int enough) {
  const int top = s_start[1];
  if (top >= enough) return enough;
  int lo = 0, hi = n_seq - 1;     // largest rank with at least half the items of rank 0
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (2 * (s_start[mid + 1] - s_start[mid]) >= top) lo = mid; else hi = mid - 1;
  }
  return min(enough, s_start[lo + 1]);
}

// Rank of the sequence that item w belongs to: the largest r with s_start[r] <= w (sequences without items share their
// successor's start).
__device__ __forceinline__ int rank_of_item(const int* s_start, int n_seq, int w) {
  int lo = 0, hi = n_seq - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_start[mid] <= w) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Whether item w belongs to a sequence with at least three quarters of the longest one's items.
__device__ __forceinline__ bool long_tail(const int* s_start, int n_seq, int w) {
  const int r = rank_of_item(s_start, n_seq, w);
  return 4 * (s_start[r + 1] - s_start[r]) >= 3 * s_start[1];
}

// Dynamic assignment for kernels that are handed counters at zero (one unsigned per XCD, 8 in
// all): the descending-cost item list is cut into chunks of consecutive items, every XCD takes one
// chunk of each round of 8 (so that the workgroups of an XCD keep meeting on the same K and V in its
// L2), and the workgroups of an XCD draw that XCD's items in order from its counter: list
// scheduling, longest first, within the XCD.  The first ticket past the queue's items ends the workgroup.
//
// Chunks are G / 8 items (smaller ones cost long sequences up to 7 %: fewer workgroups meet in an L2),
// except where the dear items are fewer than G: those are then dealt evenly, an eighth to every XCD,
// instead of filling the first XCDs and leaving the others idle (eight sequences of up to 2101 tokens, two
// heads of 64: forward 54 -> 41 us, dQ 64 -> 45 us).  Rounds run through the XCDs alternately
// upwards and downwards: an item costs at most what the one before it costs, and always upwards the first
// XCD would get the dearest chunk of every round (17 sequences of 328..4533 tokens, 24 heads of 128: forward
// 1104 -> 1087 us, dQ 1511 -> 1482 us).
//
// SPLIT > 0: where the last, partly filled round is at most a 1 / SPLIT full and of long items, its items are dealt
// out in SPLIT parts each (the kernels' narrow items), so that the round takes the GPU and not one workgroup in
// SPLIT: tickets from `wide` on stand for parts.  A bag of so few items has no full round at all.  (Short items fill
// the gaps that long ones leave, and cutting them up only adds work: 6293 tokens in 4 sequences of up to 4385,
// 24 x 128, forward 283 -> 294 us.)
template <int SPLIT>
struct ItemQueue {
  unsigned* ctr;
  int q, n_q, per, chunk;
  int n_wide, wide;         // items dealt out whole, and how many of them this queue has
  int part0, parts;         // this queue's share of the parts
  bool draws;               // more tickets than workgroups: somebody has to draw
  __device__ __forceinline__ void init(unsigned* counters, const int* s_start, int n_seq, int n_items) {
    const int G = (int)gridDim.x;
    n_q = (G % 8 == 0) ? 8 : 1;
    q = (int)(blockIdx.x % n_q);                  // workgroups go to the XCDs round-robin
    per = G / n_q;
    const int dear = dear_items(s_start, n_seq, G);
    chunk = __builtin_amdgcn_readfirstlane(max(1, (dear + n_q - 1) / n_q));
    ctr = counters + q;
    n_wide = n_items;
    part0 = parts = 0;
    if constexpr (SPLIT > 0) {
      const int last = n_items % G;
      if (last * SPLIT <= G && (n_items == last || (chunk == per && long_tail(s_start, n_seq, n_items - last)))) {
        n_wide = n_items - last;
        const int share = (last * SPLIT + n_q - 1) / n_q;
        part0 = q * share;
        parts = max(0, min(share, last * SPLIT - part0));
      }
      n_wide = __builtin_amdgcn_readfirstlane(n_wide);
      part0 = __builtin_amdgcn_readfirstlane(part0);
      parts = __builtin_amdgcn_readfirstlane(parts);
    }
    // items before n_wide: whole rounds, and the part of this queue's chunk that the last round holds
    const int round = n_wide / (n_q * chunk);
    const int in_last = n_wide - (round * n_q + chunk_of(round)) * chunk;
    wide = __builtin_amdgcn_readfirstlane(round * chunk + max(0, min(chunk, in_last)));
    draws = wide + parts > per;
  }
  // a workgroup's first item needs no draw: the first G / n_q tickets go to the queue's workgroups in order,
  // and the counter deals out the ones after them
  __device__ __forceinline__ int first_ticket() const { return (int)blockIdx.x / n_q; }
  __device__ __forceinline__ int later_ticket(unsigned drawn) const { return per + (int)drawn; }
  __device__ __forceinline__ int chunk_of(int round) const { return (round & 1) ? n_q - 1 - q : q; }
  __device__ __forceinline__ int item(int ticket) const {     // ticket < wide
    const int round = ticket / chunk;
    return (round * n_q + chunk_of(round)) * chunk + ticket % chunk;
  }
};

// Even shares: every XCD gets an eighth of each sequence's items and takes them by falling length.  Of a sequence that fills the
// GPU several times the XCDs take a round's worth of chunks in turn, so that they meet on the same heads (an eighth of its
// heads for each instead cost one of 65536 and 200 short 2.9 %, forward); what is left of it, or all of a shorter one, is cut
// in eight.  Chunks of the whole list, as above, can give one XCD the long sequences of a small bag and another the short
// ones.  Forward in us, chunks -> shares: 3512 tokens in 2 sequences, 24 x 128, 121 -> 95; 12417 in 21 of up to 6290 613 -> 491;
// 12 of up to 2673, 12 x 128, 190 -> 151; one of 4292, 24 x 128, 273 -> 259; 17 of 328..4533 1070 -> 1052; 10 of up to 6795,
// 48 x 64, 1514 -> 1491.
//
// KINDS = 2: the launch holds two kinds of items, every sequence as many of one as of the other (knap_attn_joint.h); a queue
// takes its first kind before its second.  (4096, 2300, 1024, 256 and 256 tokens, 12 x 128, backward 572 us in chunks, 472 in
// shares.)  Parts stand for items of the last kind: for all of them, where they find a workgroup each, or for those of a
// thin last round that would end late: long ones, and behind a single round of one kind also those that together with the
// round's shortest item, whose workgroup takes them, are longer than the longest (by a sixteenth: whole -> in parts at a sum of
// n longest, forward in us: 1.06, 2 of 8192 and 2 of 4300, 3 x 128, 252 -> 262; 1.09, 8192, 6000, 4500 and 4400 229 -> 220;
// 1.33, 1536 and 1000, 27 x 128, 63.7 -> 60.0; under the mask 81 -> 72).
template <int SPLIT, int KINDS>
struct EvenQueue {
  unsigned* ctr;
  int q, n_q, per;
  int mine;                 // items of each kind that are this queue's
  int wide, parts;          // items dealt out whole, and parts
  bool draws;               // more tickets than workgroups: somebody has to draw
  __device__ __forceinline__ void init(unsigned* counters) {
    n_q = (gridDim.x % 8 == 0) ? 8 : 1;
    q = (int)(blockIdx.x % n_q);
    per = (int)gridDim.x / n_q;
    ctr = counters + q;
  }
  // how many of the `count` items of the sequence of rank r are this queue's (the odd ones go round with the rank) ...
  __device__ __forceinline__ int share(int count, int r) const {
    const int k = (q + r) % n_q, whole = count / (n_q * per), rest = count - whole * n_q * per;
    return whole * per + rest * (k + 1) / n_q - rest * k / n_q;
  }
  // ... and which of them its i-th is
  __device__ __forceinline__ int locate(int count, int r, int i) const {
    const int k = (q + r) % n_q, whole = count / (n_q * per), rest = count - whole * n_q * per;
    if (i < whole * per) return (i / per * n_q + k) * per + i % per;
    return whole * n_q * per + rest * k / n_q + i - whole * per;
  }
  // s_mine[r]: this queue's items of the ranks before r; s_mine[n_seq] all of them.  length(r): of the sequence of rank r, in
  // tiles or in items, all of them (a queue's shares are too few to tell three quarters).
  template <class Length>
  __device__ __forceinline__ void deal(const int* s_mine, int n_seq, Length length) {
    mine = s_mine[n_seq];
    int last = 0;           // items of the last kind that parts stand for (SPLIT = 0: none)
    if (SPLIT == 0) {
    } else if (mine * (KINDS - 1 + SPLIT) <= per) {
      last = mine;
    } else {
      const int thin = KINDS * mine % per;
      if (thin > 0 && thin <= mine && thin * SPLIT <= per) {
        const int top = length(0), own = length(rank_of_item(s_mine, n_seq, mine - thin));
        const bool late = KINDS == 1 && mine < 2 * per && 16 * (length(rank_of_item(s_mine, n_seq, per - 1)) + own) > 17 * top;
        if (late || 4 * own >= 3 * top) last = thin;
      }
    }
    mine = __builtin_amdgcn_readfirstlane(mine);
    wide = __builtin_amdgcn_readfirstlane(KINDS * mine - last);
    parts = __builtin_amdgcn_readfirstlane(last * SPLIT);
    draws = wide + parts > per;
  }
  // the item's number among this queue's items of its kind
  __device__ __forceinline__ bool first_kind(int ticket) const { return ticket < mine; }
  __device__ __forceinline__ int item(int ticket) const { return KINDS == 1 || ticket < mine ? ticket : ticket - mine; }
  __device__ __forceinline__ int item_of_part(int part) const { return wide - (KINDS - 1) * mine + part / SPLIT; }
  __device__ __forceinline__ int first_ticket() const { return (int)blockIdx.x / n_q; }
  __device__ __forceinline__ int later_ticket(unsigned drawn) const { return per + (int)drawn; }
  // Every workgroup of a queue that draws draws until a ticket is past the queue's, so its draws are as many as its tickets:
  // whoever draws the last one can put the counter back to zero, and no launch in front of the kernel has to (5 us on a busy
  // stream)
  __device__ __forceinline__ bool last_draw(unsigned drawn) const { return (int)drawn == wide + parts - 1; }
};

// Pairs: two items of an even queue that follow each other go out as one ticket, in front of the single ones, where the kernel has a
// cheaper form for two query tiles of a sequence and head (knap_attn_fwd_full.hip).  Which items: from the first one on, as long as
// they are of sequences of at least kPairTiles tiles (shorter ones lose about as much by the longer start and end of a pair as their loop
// gains) and the items behind them have the work of a tail of two rounds of theirs (three at d = 64, where pairs gain less: one of
// 6000 tokens, 48 x 64, 468 -> 490 with two): the list has to end evenly.  Forward in us, all single ->
// pairs down to a tail of one, 1.5 and 2.5 rounds: 24 heads, one of 16384 2855 -> 2634, 2709, 2766; 8 of 4096 1482 -> 1424, 1420, 1420; 6 of
// up to 4388 567 -> 598, 602, 571; of 4267, 841 and 216 243 -> 276, 245, 247.  Counted in items and not by their work, 12000 tokens and 40 of
// 300, 12 heads, took 879 (848 single).  The limit decides on sequences of up to 1408 tokens alone.  From 6 | 8 | 12 tiles on, 24 x 128: 64 of 1024 tokens 848 |
// 858 | 862, 16 of 1024 219 | 220 | 224, 32 of 900 394 | 394 | 380, 64 of 800 620 | 617 | 605; 48 x 64: 64 of 1024 940 | 943 | 973, 24 of 1400 642 | 647 | 664,
// 32 of 900 429 | 427 | 424; from 8 against from 12, 48 bags of 600 to 1500 tokens, 1.002 at d = 128 (0.96 to 1.04), 1.008 at d = 64.
constexpr int kPairTiles = 12;
constexpr int pair_tail_rounds(int d) { return d == 64 ? 3 : 2; }
// ... and fewer than these are none.  At d = 64 a few pairs gain nothing, and the list ends less evenly behind them: 6000 tokens and 10 of 250, 48 x
// 64 (7 pairs for 96 workgroups), 465 without pairs, 476 with, and 460; 20 such bags 1.008.  At d = 128 a few are better than none: 6000 and 20 of 250, 24 x
// 128, 431 with, 437 without (and 424 without any before there were pairs).
constexpr int least_pairs(int d, int per) { return d == 64 ? (per + 3) / 4 : 0; }
// units of work of an item: a bag's work has to fit an int
__device__ __forceinline__ int item_work(int tiles) { return (tiles + 7) >> 3; }
// how many of the first of a sequence's `share` items, of `work` units each, may be paired; `behind`: the units of the queue's items
// of shorter sequences
__device__ __forceinline__ int pairable(int share, int tiles, int work, int behind, int tail) {
  return tiles < kPairTiles ? 0 : max(0, min(share, share + behind / work - tail));
}
// the pairs of a queue whose first `paired` items may be paired and whose first `whole` are dealt out whole; a tail of those stays
// single also where a few items behind them go out in parts (one of 5939 tokens, 24 heads, 411 -> 418 with five pairs)
__device__ __forceinline__ int item_pairs(int paired, int whole, int tail, int least) {
  const int pairs = max(0, min(paired, whole - tail)) / 2;
  return pairs < least ? 0 : pairs;
}

}  // namespace knap
