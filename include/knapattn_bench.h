/* libknapattn: hooks for benchmarks and tests.  Not part of the attention
 * interface (include/knapattn.h) and of no use to a training loop: they let a
 * benchmark time one kernel of the backward with events on the launch stream,
 * and read the size of the persistent launches.  Same conventions as
 * knapattn.h (plain C ABI, nothing allocates or synchronises).
 */
#ifndef KNAPATTN_BENCH_H
#define KNAPATTN_BENCH_H

#ifdef __cplusplus
extern "C" {
#endif

/* While both are non-NULL, every backward call made by this thread records
 * `start` right before and `stop` right after its dK/dV kernel (the longest
 * kernel of the path) on the call's stream; the dQ kernel, which runs before
 * it, stays outside the pair.  Where the items of both kernels share one launch
 * (bags that fill the GPU a few times), the pair brackets that launch and the
 * small one in front of it.  hipEvent_t passed as void*, owned by the
 * caller.  Pass NULLs to switch it off.  Not for use under graph capture. */
void knap_bwd_profile_events(void* start, void* stop);

/* Number of persistent workgroups the forward / backward kernels are launched
 * with on the current device (<= 0 on error); for the dK/dV kernel at d = 128
 * those of its four-pair form (256 keys per workgroup; the two-pair form, 128
 * keys, has twice as many), at d = 64 of the two-pair form, its only one there. */
int knap_launch_workgroups(int which /* d = 128: 0 = forward, 1 = backward dK/dV, 2 = backward dQ; d = 64: 3, 4, 5 */);

/* Device address of the counters that forward launches draw their work items
 * from, on the current device (NULL on error), and their number.  All zero
 * while no forward runs. */
unsigned* knap_fwd_queue_counters(int* count);

#ifdef __cplusplus
}
#endif
#endif /* KNAPATTN_BENCH_H */
