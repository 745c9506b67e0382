// Polls that a bounded wait still has, counted down in the limit's own 64 bits: the
// test against zero and the decrement are scalar instructions, where comparing a
// count with the limit is a vector one.
#pragma once

// Takes one poll; false when the limit's polls are all taken.
__host__ __device__ inline bool take_poll(unsigned long long* left) {
  if (*left == 0ull) return false;
  --*left;
  return true;
}
