// How an operation by whole chunks learns that a workgroup is its last one:
// lines of arrivals in the plan's memory.  A chunk adds its arrival (low half)
// and its bit (high half) to its bitmap word's line in one atomic; whoever
// brings the last arrival of a word thereby holds all its bits, writes them,
// and adds the word's arrival and count to its group's line (of kArriveGroup
// words, where there are more) and then to the first line the same way.  The
// data ride in the atomics, so nothing has to be ordered or flushed between
// XCDs.
//
// Lines that are kept from one call to the next (kKept) are zero whenever no
// call is running: whoever finds a line full takes off again exactly what it
// found.  That holds too where calls of one plan overlapped, which a caller
// must not do and whose own results are undefined: while a line holds a full
// count or more, the one that found it full goes on taking full counts off it
// (and passing them on), so that every call's arrivals are taken off once and
// later calls start from zero.  (Clearing a full line instead dropped the
// arrivals that another call had added in between, and the line stayed off by
// them for the life of the plan: no later call wrote its count.)  Lines that
// an earlier kernel of the same call has cleared are left as they end.
//
// The atomic is a parameter (Mem::add(line, x): adds x, returns the value
// before), so that the protocol also runs on a CPU, in any order of its steps.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define FR_DEVICE __device__ __forceinline__
#else
#define FR_DEVICE inline
#endif

namespace fr {

// Every line has 128 bytes of its own: atomics on one line follow each other at
// about 7 ns (16 words to a line: 6,300 chunks of 4 KiB unpacked in 37 us
// instead of 31).
constexpr uint32_t kArriveLine = 128, kArriveGroup = 64;
// Bytes of the lines for n chunks: one for all, one per bitmap word and one per
// group of words.
inline uint64_t arrive_bytes(uint64_t n) {
  const uint64_t words = (n + 31) / 32;
  return (1 + words + (words + kArriveGroup - 1) / kArriveGroup) * kArriveLine;
}

struct Arrivals {
  uint64_t* lines;   // line 0: everything; lines 1 ...: bitmap words; behind them: groups of them
  uint32_t* bitmap;
  uint64_t* count;
  uint64_t n;        // chunks the lines are laid out for
};

FR_DEVICE uint64_t* arrive_line(const Arrivals& a, uint32_t i) {
  return a.lines + uint64_t(i) * (kArriveLine / sizeof(uint64_t));
}
FR_DEVICE uint64_t* group_line(const Arrivals& a, uint32_t g) {
  return arrive_line(a, 1 + uint32_t((a.n + 31) / 32) + g);
}

// `now`: a line's value with its `of`-th arrival, as its bringer found it;
// full(data) is called with the data of every `of` arrivals.
template <class Mem, bool kKept, class Full>
FR_DEVICE void line_full(uint64_t* line, uint64_t now, uint32_t of, Full full) {
  for (;;) {
    // in flight beside what full() adds further up
    const uint64_t rest = kKept ? Mem::add(line, 0 - now) - now : 0;
    full(uint32_t(now >> 32));
    if (uint32_t(rest) < of) return;
    now = (rest >> 32 << 32) | of;  // only where calls overlap
  }
}

// A word's arrival with `set` bits set, of a call of `words` words: at its
// group's line, where there is one, and at the first.
template <class Mem, bool kKept>
FR_DEVICE void arrive_word(const Arrivals& a, uint32_t w, uint32_t words, uint32_t set) {
  const bool grouped = words > kArriveGroup;
  const uint32_t g = w / kArriveGroup, left = words - g * kArriveGroup;
  uint64_t* const line = grouped ? group_line(a, g) : arrive_line(a, 0);
  const uint32_t of = left < kArriveGroup ? left : kArriveGroup;
  const uint64_t add = (uint64_t(set) << 32) + 1, now = Mem::add(line, add) + add;
  if (uint32_t(now) != of) return;
  line_full<Mem, kKept>(line, now, of, [&](uint32_t count) {
    if (grouped) {
      const uint32_t groups = (words + kArriveGroup - 1) / kArriveGroup;
      const uint64_t one = (uint64_t(count) << 32) + 1, all = Mem::add(arrive_line(a, 0), one) + one;
      if (uint32_t(all) == groups)
        line_full<Mem, kKept>(arrive_line(a, 0), all, groups, [&](uint32_t c) { *a.count = c; });
    } else {
      *a.count = count;
    }
  });
}

// One thread's call for the chunks c[k] with on[k], of the n chunks of the
// call, each of which arrives once: bit[k] goes to the bitmap, and the last
// arrival of all writes the count.
template <class Mem, bool kKept, int N>
FR_DEVICE void arrive_chunks(const Arrivals& a, uint64_t n, const uint64_t (&c)[N],
                             const uint32_t (&bit)[N], const bool (&on)[N]) {
  uint64_t now[N];
#pragma unroll
  for (int k = 0; k < N; k++) {  // all in flight together
    now[k] = 0;
    if (!on[k]) continue;
    const uint64_t add = (uint64_t(bit[k]) << (32 + (c[k] & 31))) + 1;
    now[k] = Mem::add(arrive_line(a, 1 + uint32_t(c[k] >> 5)), add) + add;
  }
  const uint32_t words = uint32_t((n + 31) / 32), last = uint32_t(n - 1) % 32 + 1;
  auto here = [&](uint32_t w) { return w + 1 == words ? last : 32u; };
  for (;;) {  // one copy of what follows a full word, whichever of the chunks filled it
    uint32_t w = 0;
    uint64_t full = 0;
#pragma unroll
    for (int k = 0; k < N; k++)
      if (!full && uint32_t(now[k]) == here(uint32_t(c[k] >> 5))) {
        w = uint32_t(c[k] >> 5);
        full = now[k];
        now[k] = 0;
      }
    if (!full) return;
    line_full<Mem, kKept>(arrive_line(a, 1 + w), full, here(w), [&](uint32_t bits) {
      a.bitmap[w] = bits;
      arrive_word<Mem, kKept>(a, w, words, uint32_t(__builtin_popcount(bits)));
    });
    if (N == 1) return;
  }
}

}  // namespace fr
