// Host build of the donated-task queue's slot arithmetic
// (paper_2404_11105_amd/csrc/donate.h) for tests/test_donation_queue.py.
#include "../../paper_2404_11105_amd/csrc/donate.h"

extern "C" {

uint32_t t_slot(uint32_t s, uint32_t cap) { return xm::don_slot(s, cap); }
uint32_t t_published(uint32_t s, uint32_t cap) { return xm::don_published(s, cap); }
uint32_t t_read(uint32_t s, uint32_t cap) { return xm::don_read(s, cap); }
int t_fits(uint32_t head, uint32_t tail, uint32_t k, uint32_t cap) { return xm::don_fits(head, tail, k, cap) ? 1 : 0; }
int t_left(const uint32_t* don, uint32_t words, uint32_t cap, uint32_t head, uint32_t tail, uint32_t first, uint32_t step) {
    return xm::don_left(don, words, cap, head, tail, first, step) ? 1 : 0;
}
uint32_t t_last() { return xm::kDonLast; }
}
