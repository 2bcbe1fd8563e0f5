// Classes of equal work items and their schedule (host code, plain C++; the
// table is also read by the kernels).
//
// A launch runs items of every chunk of a call; the items of one chunk take
// equally long.  Items are grouped into classes of equal length and dispatched
// longest class first, which is longest-first list scheduling.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace fastvr {

constexpr int kMaxClasses = 32;

// Passed by value as a kernel argument.  Class k holds items first[k] ..
// first[k + 1] - 1 of chunks c0[k] .. c0[k] + nc[k] - 1; the last chunk of a call,
// whose tile count may differ, is always a class of its own.
struct ClassTable {
  int32_t n;
  int32_t c0[kMaxClasses], nc[kMaxClasses], kind[kMaxClasses];
  int32_t first[kMaxClasses + 1];
};

// Workgroups go to the 8 XCDs round-robin; within each round of 256 workgroups
// of a class (the last one may be shorter), each XCD gets consecutive units
// (neighbouring tiles of one stream share its L2).  i: index within the class of
// n units.  Rounds over all units instead would give whole XCDs to one class.
// (Kernel code; constexpr compiles it for the host as well.)
constexpr int xcd_unit(int i, int n) {
  constexpr int kRound = 256;
  const int r0 = i / kRound * kRound, w = i - r0;
  const int m = (n - r0 < kRound) ? n - r0 : kRound;  // units of this round
  const int x = w & 7, per = m >> 3, rem = m & 7;
  return r0 + x * per + (x < rem ? x : rem) + (w >> 3);
}

struct WorkClass {
  int64_t cost, units;  // cost of one item, items
  int32_t c0, nc, kind;
};

// The classes of n chunks in chunk order, `per` items a chunk (`per_last` in the
// last one), cost(c) the cost of an item of chunk c, which up to chunk `peak` does
// not fall and after it does not rise (the last chunk aside).  Runs of equal
// chunks share a class; with more runs than `room` allows, neighbouring chunks are
// grouped (at their longest chunk's cost).  Returns the number of classes.
// Equal ends of a run make equal chunks between them, so a run's end is found by
// doubling steps and bisection, not chunk by chunk: this is on the path of every
// call, and a window makes nearly all chunks equal (65280 chunks of one token, W =
// 1: forward 284 -> 0.3 us, backward 572 -> 0.6 us on the host).
template <typename Cost>
inline int make_classes(int64_t n, int64_t per, int64_t per_last, int kind, int room, int64_t peak, WorkClass* out,
                        Cost cost) {
  if (n <= 0) return 0;
  int k = 0;
  const int64_t body = n - 1;
  // end of the run of chunks like c (cost w) in [c, end)
  auto run_end = [&](int64_t c, int64_t end, int64_t w) {
    int64_t like = c, step = 1;
    while (step < end - like && cost(like + step) == w) {
      like += step;
      step *= 2;
    }
    int64_t other = std::min(like + step, end);  // costs more or less, or the end
    while (other - like > 1) {
      const int64_t mid = like + (other - like) / 2;
      (cost(mid) == w ? like : other) = mid;
    }
    return other;
  };
  for (int64_t step = 1;; step = std::max<int64_t>(2 * step, (body + room - 2) / (room - 1))) {
    k = 0;
    bool fits = true;
    for (int64_t c = 0, nc; c < body; c += nc) {
      int64_t w = cost(c);
      if (step == 1) {
        nc = run_end(c, c <= peak ? std::min(body, peak + 1) : body, w) - c;
      } else {
        nc = std::min(step, body - c);
        // longest of the group: costs are monotone in the chunk up to the window's ends
        if (nc > 1) w = std::max(std::max(w, cost(c + nc - 1)), cost(c + nc / 2));
      }
      if (k > 0 && out[k - 1].cost == w) {
        out[k - 1].nc += (int32_t)nc;
        out[k - 1].units += nc * per;
      } else if (k < room - 1) {
        out[k++] = WorkClass{w, nc * per, (int32_t)c, (int32_t)nc, kind};
      } else {
        fits = false;
        break;
      }
    }
    if (fits) break;
  }
  out[k++] = WorkClass{cost(n - 1), per_last, (int32_t)(n - 1), 1, kind};
  return k;
}

// Longest first; equal classes keep their order.
inline void sort_classes(WorkClass* cls, int n) {
  for (int i = 1; i < n; ++i) {  // a few classes, on the path of every call: no allocation
    const WorkClass x = cls[i];
    int j = i;
    for (; j > 0 && cls[j - 1].cost < x.cost; --j) cls[j] = cls[j - 1];
    cls[j] = x;
  }
}

// Makespan of dispatching the classes in order on n_cu CUs (each unit on the CU
// that frees up first), with CUs of equal load kept as one group.
inline int64_t class_makespan(const WorkClass* cls, int n, int n_cu) {
  constexpr int kMaxGroups = 512;
  int64_t load[kMaxGroups];
  int count[kMaxGroups];
  int head = 0, tail = 1;  // groups head .. tail - 1, ascending load
  load[0] = 0;
  count[0] = n_cu;
  for (int k = 0; k < n; ++k) {
    int64_t m = cls[k].units;
    while (m > 0) {
      const int64_t l = load[head] + cls[k].cost;
      int take = count[head];
      if (m < take) {
        take = (int)m;
        count[head] -= take;
      } else {
        ++head;
      }
      m -= take;
      // insert (l, take)
      int i = tail;
      while (i > head && load[i - 1] > l) --i;
      if (i > head && load[i - 1] == l) {
        count[i - 1] += take;
        continue;
      }
      if (tail == kMaxGroups) {  // close the gap at the front
        std::copy(load + head, load + tail, load);
        std::copy(count + head, count + tail, count);
        tail -= head;
        i -= head;
        head = 0;
      }
      for (int j = tail; j > i; --j) {
        load[j] = load[j - 1];
        count[j] = count[j - 1];
      }
      load[i] = l;
      count[i] = take;
      ++tail;
    }
  }
  return load[tail - 1];
}

// Fills the table; returns the number of items (the grid).
inline int64_t fill_table(const WorkClass* cls, int n, ClassTable* tab) {
  tab->n = n;
  int64_t units = 0;
  for (int k = 0; k < n; ++k) {
    tab->first[k] = (int32_t)units;
    tab->c0[k] = cls[k].c0;
    tab->nc[k] = cls[k].nc;
    tab->kind[k] = cls[k].kind;
    units += cls[k].units;
  }
  tab->first[n] = (int32_t)units;
  return units;
}

}  // namespace fastvr
