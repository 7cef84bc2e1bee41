// donate.h -- the queue of donated tasks: sequence numbers, slots and ready words.
//
// Task s (s = 0, 1, ... in the order of reservation) takes slot s mod cap (a
// power of two), as that slot's use u = s / cap.  The slot's ready word steps through its uses:
//   3u      free (0 at the start of a launch)
//   3u + 1  published: the donor has written the task's words
//   3u + 2  claimed by a waiting wave
//   3u + 3  read: the taker has its words; free for use u + 1
// A word never takes a value twice, so a claim of a task that is gone fails.
// The head moves past read tasks only, and a task is reserved only while it is
// less than cap ahead of the head: its slot is then free.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define XM_HD __host__ __device__
#else
#define XM_HD
#endif

namespace xm {

constexpr uint32_t kDonLast = 0xFFFF0000u;  // sequence numbers end here (no wrap; donation stops)

XM_HD inline uint32_t don_slot(uint32_t s, uint32_t cap) { return s & (cap - 1u); }
XM_HD inline uint32_t don_published(uint32_t s, uint32_t cap) { return 3u * (s >> __builtin_ctz(cap)) + 1u; }
XM_HD inline uint32_t don_read(uint32_t s, uint32_t cap) { return 3u * (s >> __builtin_ctz(cap)) + 3u; }
// Whether k tasks may be reserved behind `tail` (head: the head or an earlier one).
XM_HD inline bool don_fits(uint32_t head, uint32_t tail, uint32_t k, uint32_t cap) {
    return tail <= kDonLast - k && tail + k - head <= cap;
}

// Whether a reserved task of [head, tail) was never read: slots' words at don,
// `words` a slot, the ready word second; looks at every step-th task from `first` on.
XM_HD inline bool don_left(const uint32_t* don, uint32_t words, uint32_t cap, uint32_t head, uint32_t tail,
                           uint32_t first, uint32_t step) {
    bool left = false;
    for (uint64_t s = (uint64_t)head + first; s < tail; s += step)
        left = left || don[(uint64_t)don_slot((uint32_t)s, cap) * words + 1] != don_read((uint32_t)s, cap);
    return left;
}

}  // namespace xm
