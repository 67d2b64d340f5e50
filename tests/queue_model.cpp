// The device's work queues (csrc/knap_queue.h) and the host's rules about them (csrc/knap_dispatch.h) compiled for the
// CPU: the same text, with the few device words it uses defined here.
#include <algorithm>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_readfirstlane(x) (x)
using std::max;
using std::min;
static struct { int x; } gridDim, blockIdx;

#include "knap_dispatch.h"
#include "knap_queue.h"

namespace {

struct Walk {
  int items, parts, per, most, draws, wrong;
};

template <int SPLIT>
Walk walk(int grid, const std::vector<int>& start, int n_seq, int n_items) {
  Walk r = {n_items, 0, 0, 0, 0, 0};
  std::vector<int> whole(n_items, 0), part((size_t)n_items * max(SPLIT, 1), 0);
  std::vector<unsigned> counters(8, 0);
  gridDim.x = grid;
  const int n_q = grid % 8 == 0 ? 8 : 1;
  int n_wide = -1;
  for (int q = 0; q < n_q; ++q) {
    blockIdx.x = q;
    knap::ItemQueue<SPLIT> queue;
    queue.init(counters.data(), start.data(), n_seq, n_items);
    if (q == 0) n_wide = queue.n_wide;
    r.wrong += queue.n_wide != n_wide || queue.ctr != counters.data() + q;
    const int tickets = queue.wide + queue.parts;
    // the tickets 0 .. per - 1 come from the workgroups' indexes, `per` and up from the counter, which starts at zero
    for (int i = 0; i < queue.per; ++i) {
      blockIdx.x = q + i * n_q;
      r.wrong += queue.first_ticket() != i;
    }
    r.wrong += queue.later_ticket(0u) != queue.per || queue.later_ticket(3u) != queue.per + 3;
    r.wrong += !queue.draws && tickets > queue.per;
    for (int t = 0; t < queue.wide; ++t) {
      const int w = queue.item(t);
      if (w < 0 || w >= n_wide) ++r.wrong; else ++whole[w];
    }
    for (int p = 0; p < queue.parts; ++p) {
      const int at = n_wide * SPLIT + queue.part0 + p;
      if (at < 0 || at >= n_items * SPLIT) ++r.wrong; else ++part[at];
    }
    r.per = queue.per;
    r.most = max(r.most, tickets);
    r.draws |= queue.draws;
    r.parts += queue.parts;
  }
  for (int w = 0; w < n_items; ++w) {
    r.wrong += whole[w] != (w < n_wide ? 1 : 0);
    for (int i = 0; i < SPLIT; ++i) r.wrong += part[(size_t)w * SPLIT + i] != (w < n_wide ? 0 : 1);
  }
  return r;
}

// even shares: every item of a first kind of two whole, every one of the last kind whole or all its parts
template <int SPLIT, int KINDS>
Walk walk_even(int grid, const std::vector<int>& start, int n_seq, int n_items) {
  Walk r = {n_items, 0, 0, 0, 0, 0};
  std::vector<int> first(n_items, 0), second(n_items, 0), part((size_t)n_items * SPLIT, 0), mine(n_seq + 1);
  std::vector<unsigned> counters(8, 0);
  gridDim.x = grid;
  const int n_q = grid % 8 == 0 ? 8 : 1;
  for (int q = 0; q < n_q; ++q) {
    blockIdx.x = q;
    knap::EvenQueue<SPLIT, KINDS> queue;
    queue.init(counters.data());
    mine[0] = 0;
    for (int s = 0; s < n_seq; ++s) mine[s + 1] = mine[s] + queue.share(start[s + 1] - start[s], s);
    queue.deal(mine.data(), n_seq, [&](int k) { return start[k + 1] - start[k]; });
    const int tickets = queue.wide + queue.parts;
    auto global = [&](int i) {        // item i of this queue's
      const int k = knap::rank_of_item(mine.data(), n_seq, i);
      const int w = start[k] + queue.locate(start[k + 1] - start[k], k, i - mine[k]);
      return i < 0 || i >= mine[n_seq] || w < start[k] || w >= start[k + 1] ? -1 : w;
    };
    for (int t = 0; t < queue.wide; ++t) {
      const int w = global(queue.item(t));
      if (w < 0) ++r.wrong; else ++(KINDS == 2 && queue.first_kind(t) ? first : second)[w];
    }
    if constexpr (SPLIT > 0) {
      for (int p = 0; p < queue.parts; ++p) {
        const int w = global(queue.item_of_part(p));
        if (w < 0) ++r.wrong; else ++part[(size_t)w * SPLIT + p % SPLIT];
      }
    } else {
      r.wrong += queue.parts != 0;
    }
    for (int i = 0; i < queue.per; ++i) {
      blockIdx.x = q + i * n_q;
      r.wrong += queue.first_ticket() != i;
    }
    r.wrong += queue.later_ticket(0u) != queue.per || queue.ctr != counters.data() + q || (!queue.draws && tickets > queue.per);
    // every workgroup of a queue that draws draws until a ticket is past the queue's: the last draw, which puts the counter
    // back to zero, is known as such, and nobody draws after it
    if (queue.draws) {
      int at_work = queue.per;
      for (unsigned drawn = 0; at_work > 0 && drawn <= (unsigned)tickets; ++drawn) {
        if (queue.later_ticket(drawn) >= tickets) --at_work;
        r.wrong += queue.last_draw(drawn) != (at_work == 0);
      }
      r.wrong += at_work != 0;
    }
    r.per = queue.per;
    r.most = max(r.most, tickets);
    r.draws |= queue.draws;
    r.parts += queue.parts;
  }
  for (int w = 0; w < n_items; ++w) {
    int parts = 0;
    for (int i = 0; i < SPLIT; ++i) parts += part[(size_t)w * SPLIT + i] == 1 ? 1 : part[(size_t)w * SPLIT + i] == 0 ? 0 : 100;
    r.wrong += first[w] != KINDS - 1 || !((second[w] == 1 && parts == 0) || (second[w] == 0 && parts == SPLIT));
  }
  return r;
}

}  // namespace

extern "C" {

// lens: the sequences' lengths.  out: items, parts dealt, workgroups per queue, most tickets of a queue, whether some queue
// draws, and how many items or parts were not dealt exactly once (or tickets not served).
void queue_walk(const int* lens, int n_seq, int H, int tile, int causal, int split, int grid, int* out) {
  std::vector<int> sorted(lens, lens + n_seq);
  std::sort(sorted.begin(), sorted.end(), [](int a, int b) { return a > b; });
  std::vector<int> start(n_seq + 1, 0);
  for (int r = 0; r < n_seq; ++r) {
    const int tiles = (sorted[r] + tile - 1) / tile;
    start[r + 1] = start[r] + H * (causal ? knap::items_per_head<true>(tiles) : knap::items_per_head<false>(tiles));
  }
  const int n = start[n_seq];
  const Walk w = split == 0 ? walk<0>(grid, start, n_seq, n) : split == 2 ? walk<2>(grid, start, n_seq, n) : walk<4>(grid, start, n_seq, n);
  const int values[] = {w.items, w.parts, w.per, w.most, w.draws, w.wrong};
  std::copy(values, values + 6, out);
}

// the same for even shares (tiles of 128) of one kind of items (the forward) or of two (the backward in one launch)
void queue_walk_even(const int* lens, int n_seq, int H, int causal, int kinds, int grid, int* out) {
  std::vector<int> sorted(lens, lens + n_seq);
  std::sort(sorted.begin(), sorted.end(), [](int a, int b) { return a > b; });
  std::vector<int> start(n_seq + 1, 0);
  for (int r = 0; r < n_seq; ++r) {
    const int tiles = (sorted[r] + 127) / 128;
    start[r + 1] = start[r] + H * (causal ? knap::items_per_head<true>(tiles) : knap::items_per_head<false>(tiles));
  }
  const int n = start[n_seq];
  const Walk w = kinds == 2 ? (causal ? walk_even<4, 2>(grid, start, n_seq, n) : walk_even<2, 2>(grid, start, n_seq, n))
                            : (causal ? walk_even<4, 1>(grid, start, n_seq, n) : walk_even<2, 1>(grid, start, n_seq, n));
  const int values[] = {w.items, w.parts, w.per, w.most, w.draws, w.wrong};
  std::copy(values, values + 6, out);
}

// ... and of both kinds in tiles of 64, none in parts (the backward of small bags)
void queue_walk_small(const int* lens, int n_seq, int H, int grid, int* out) {
  std::vector<int> sorted(lens, lens + n_seq);
  std::sort(sorted.begin(), sorted.end(), [](int a, int b) { return a > b; });
  std::vector<int> start(n_seq + 1, 0);
  for (int r = 0; r < n_seq; ++r) start[r + 1] = start[r] + H * ((sorted[r] + 63) / 64);
  const Walk w = walk_even<0, 2>(grid, start, n_seq, start[n_seq]);
  const int values[] = {w.items, w.parts, w.per, w.most, w.draws, w.wrong};
  std::copy(values, values + 6, out);
}

int queue_bwd_small(long long tokens, int n_seq, int H, int d, int causal, int cus) {
  return knap::bwd_small(tokens, n_seq, H, d, causal != 0, cus);
}

// What the host knows about the items of 64 rows of that launch (2: taken whatever the lengths are, 1: the device decides), and the
// device's decision.
void queue_small_items(const int* lens, int n_seq, int H, int d, int causal, int cus, int* out) {
  long long tokens = 0;
  int tiles = 0, longest = 0;
  for (int s = 0; s < n_seq; ++s) {
    tokens += lens[s];
    tiles += (lens[s] + 63) / 64;
    longest = max(longest, (lens[s] + 63) / 64);
  }
  out[0] = !knap::bwd_small(tokens, n_seq, H, d, causal != 0, cus) ? 0 : knap::small_sure(tokens, n_seq, H, d, causal != 0, cus) ? 2 : 1;
  out[1] = knap::small_pays(tiles, longest, H, cus * knap::dkdv_workgroups_per_cu(d, 2), d, causal != 0);
}

int queue_bwd_joint(long long tokens, int n_seq, int H, int d, int causal, int cus) {
  return knap::bwd_joint(tokens, n_seq, H, d, causal != 0, cus);
}

int queue_dkdv_pairs(long long tokens, int n_seq, int H, int d, int causal, int cus) {
  return knap::dkdv_pairs(tokens, n_seq, H, d, causal != 0, cus);
}

// the forward without the mask, whose tickets stand for pairs of items, single ones and parts (knap_attn_fwd_full.hip): out as above, with
// the pairs of all queues in place of the items
void queue_walk_pairs(const int* lens, int n_seq, int H, int d, int grid, int* out) {
  const int rounds = knap::pair_tail_rounds(d);
  std::vector<int> sorted(lens, lens + n_seq);
  std::sort(sorted.begin(), sorted.end(), [](int a, int b) { return a > b; });
  std::vector<int> start(n_seq + 1, 0), mine(n_seq + 1);
  for (int r = 0; r < n_seq; ++r) start[r + 1] = start[r] + H * ((sorted[r] + 127) / 128);
  const int n = start[n_seq];
  std::vector<int> whole(n, 0), part((size_t)n * 2, 0);
  std::vector<unsigned> counters(8, 0);
  Walk w = {0, 0, 0, 0, 0, 0};
  gridDim.x = grid;
  const int n_q = grid % 8 == 0 ? 8 : 1;
  for (int q = 0; q < n_q; ++q) {
    blockIdx.x = q;
    knap::EvenQueue<2, 1> queue;
    queue.init(counters.data());
    mine[0] = 0;
    int behind = 0, paired = 0;
    bool stop = n <= rounds * grid;
    for (int s = 0; s < n_seq; ++s) {
      const int items = start[s + 1] - start[s];
      mine[s + 1] = mine[s] + queue.share(items, s);
      behind += queue.share(items, s) * knap::item_work(items / H);
    }
    for (int s = 0; s < n_seq && !stop; ++s) {
      const int share = mine[s + 1] - mine[s], tiles = (start[s + 1] - start[s]) / H, work = max(1, knap::item_work(tiles));
      behind -= share * work;
      const int some = knap::pairable(share, tiles, work, behind, rounds * queue.per);
      paired = mine[s] + some;
      stop = some < share;
    }
    queue.deal(mine.data(), n_seq, [&](int k) { return start[k + 1] - start[k]; });
    const int pairs = knap::item_pairs(paired, queue.wide, rounds * queue.per, knap::least_pairs(d, queue.per)), singles = queue.wide - pairs, tickets = singles + queue.parts;
    auto global = [&](int i) {
      const int k = knap::rank_of_item(mine.data(), n_seq, i);
      return start[k] + queue.locate(start[k + 1] - start[k], k, i - mine[k]);
    };
    w.wrong += pairs < 0 || singles < pairs;
    for (int t = 0; t < pairs; ++t) { ++whole[global(2 * t)]; ++whole[global(2 * t + 1)]; }
    for (int t = pairs; t < singles; ++t) ++whole[global(t + pairs)];
    for (int t = singles; t < tickets; ++t) {
      const int p = t - singles;
      ++part[(size_t)global(queue.item_of_part(p)) * 2 + (p & 1)];
    }
    w.items += pairs;
    w.parts += queue.parts;
    w.per = queue.per;
    w.most = max(w.most, tickets);
    w.draws |= tickets > queue.per;
    // all parts: one for a workgroup, none drawn
    w.wrong += singles == 0 && tickets > queue.per;
  }
  for (int i = 0; i < n; ++i) w.wrong += !((whole[i] == 1 && part[2 * i] == 0 && part[2 * i + 1] == 0) || (whole[i] == 0 && part[2 * i] == 1 && part[2 * i + 1] == 1));
  const int values[] = {w.items, w.parts, w.per, w.most, w.draws, w.wrong};
  std::copy(values, values + 6, out);
}

// set of eager forward call `call`, and the first of the sets it clears (-1: none)
void queue_eager_set(unsigned long long call, int* out) {
  const knap::EagerSet s = knap::eager_set(call);
  out[0] = (int)s.set;
  out[1] = s.clear;
}

int queue_captured_set(unsigned long long call) { return (int)knap::captured_set(call); }

int queue_dkdv_workgroups_per_cu(int d, int pairs) { return knap::dkdv_workgroups_per_cu(d, pairs); }

}  // extern "C"
