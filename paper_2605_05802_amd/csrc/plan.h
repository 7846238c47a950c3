// Host-side rules that decide how work is laid out over the chip, in plain C++ so that they can be evaluated (and tested)
// without a GPU or the HIP headers; kernels use the parts marked SR_HD.
#pragma once

#ifdef __HIPCC__
#define SR_HD __host__ __device__
#else
#define SR_HD
#endif

namespace sr {

SR_HD inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
SR_HD inline int round_up(int a, int b) { return ceil_div(a, b) * b; }

// Attention whose query tiles share K/V blocks: workgroup `wg` -> set (unit, kv head, split) and which of the set's `per_set`
// workgroups.  Consecutive workgroups go to consecutive XCDs.  Of every eight sets each goes to one XCD, whose L2 then
// serves the set's workgroups; the last n_sets % 8 sets are dealt out over all XCDs, because whole sets would leave
// XCDs idle (one group's prompt of 5000 tokens and two kv heads of 128: 549 us on two XCDs, 202 on eight).
SR_HD inline void shared_tiles_of(int wg, int n_sets, int per_set, int *set, int *part) {
    const int rest0 = (n_sets & ~7) * per_set, t = wg - rest0;
    *set = t < 0 ? (wg >> 3) / per_set * 8 + (wg & 7) : (n_sets & ~7) + t / per_set;
    *part = t < 0 ? (wg >> 3) % per_set : t % per_set;
}

}  // namespace sr
