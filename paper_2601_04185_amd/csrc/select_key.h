// select_key.h -- the order in which a query's candidates are chosen: (msac
// asc, count desc, sample asc, solution asc), a strict total order.
#pragma once

#include <cstdint>

namespace imloc {

// Solutions of one minimal sample, at most: P3P gives four, generalised P3P
// (rig queries) eight.
constexpr int kMaxSolutions = 8;

struct Key {
  double ms;
  long long hj;   // sample index and solution index: hj_order
  int cnt, idx;
};

// Different for every solution of every sample, and in their order.
__host__ __device__ inline long long hj_order(int64_t h, int j) { return (long long)h * kMaxSolutions + j; }

__host__ __device__ inline bool key_less(const Key& a, const Key& b) {
  if (a.ms != b.ms) return a.ms < b.ms;
  if (a.cnt != b.cnt) return a.cnt > b.cnt;
  return a.hj < b.hj;
}

// Place of key e of a list: how many precede it, equal ones by their position,
// so that the places of n keys are 0 .. n - 1 whatever the keys are.
__host__ __device__ inline int key_place(const Key* keys, int n, int e) {
  const Key mine = keys[e];
  int before = 0;
  for (int i = 0; i < n; ++i) {
    const Key x = keys[i];
    before += key_less(x, mine) || (i < e && !key_less(mine, x)) ? 1 : 0;
  }
  return before;
}

}  // namespace imloc
