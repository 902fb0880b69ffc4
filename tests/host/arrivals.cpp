// The arrival lines by which the last workgroup of an operation writes its
// bitmap and count (csrc/arrive.h), run on the CPU step by step: every chunk's
// thread is a coroutine that yields before each of its atomics, and a seeded
// scheduler picks who goes next, so that steps of one call, and of calls of
// one plan that overlap (which callers must not do), come in any order.
// A call alone has to write its own bits and count; after any calls, also
// overlapping ones, the lines have to be zero, so that the next call is right.
// Built and run by tests/test_arrivals_cpu.py.
#include <ucontext.h>

#include <cstdio>
#include <deque>
#include <memory>
#include <random>
#include <vector>

#include "arrive.h"

namespace {

constexpr size_t kStack = 32 * 1024;
std::mt19937_64 rng(1);
uint64_t U(uint64_t n) { return rng() % n; }

ucontext_t scheduler;
struct Thread;
Thread* running = nullptr;

struct Call {
  uint64_t n;
  std::vector<uint32_t> bit, bitmap;
  uint64_t count;
  fr::Arrivals a;
};
struct Thread {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack{new char[kStack]};
  bool done = false;
  Call* call;
  uint64_t c[3];
  bool on[3];
};

// The atomic: another thread may run first.
struct Step {
  static uint64_t add(uint64_t* line, uint64_t x) {
    swapcontext(&running->ctx, &scheduler);
    const uint64_t before = *line;
    *line = before + x;
    return before;
  }
};

void body() {
  Thread* t = running;
  const uint32_t bit[3] = {t->call->bit[t->c[0]], t->on[1] ? t->call->bit[t->c[1]] : 0,
                           t->on[2] ? t->call->bit[t->c[2]] : 0};
  fr::arrive_chunks<Step, true, 3>(t->call->a, t->call->n, t->c, bit, t->on);
  t->done = true;
  swapcontext(&t->ctx, &scheduler);
}

// Runs the calls' chunks, up to `most` threads at a time, in random order.
void run(std::vector<Call>& calls, size_t most) {
  struct Work {
    Call* call;
    uint64_t c;
    int k;
  };
  std::deque<Work> todo;
  for (auto& call : calls)
    for (uint64_t c = 0; c < call.n;) {  // one chunk, or up to three
      const int k = int(std::min<uint64_t>(call.n - c, U(4) ? 1 : 3));
      todo.push_back({&call, c, k});
      c += k;
    }
  for (size_t i = todo.size(); i > 1; i--) std::swap(todo[i - 1], todo[U(i)]);
  std::vector<std::unique_ptr<Thread>> live;
  while (!todo.empty() || !live.empty()) {
    while (live.size() < most && !todo.empty()) {
      auto t = std::make_unique<Thread>();
      const Work w = todo.front();
      todo.pop_front();
      t->call = w.call;
      for (int k = 0; k < 3; k++) {
        t->on[k] = k < w.k;
        t->c[k] = t->on[k] ? w.c + k : 0;
      }
      getcontext(&t->ctx);
      t->ctx.uc_stack.ss_sp = t->stack.get();
      t->ctx.uc_stack.ss_size = kStack;
      t->ctx.uc_link = nullptr;
      makecontext(&t->ctx, body, 0);
      live.push_back(std::move(t));
    }
    const size_t i = U(live.size());
    running = live[i].get();
    swapcontext(&scheduler, &running->ctx);
    if (running->done) {
      std::swap(live[i], live.back());
      live.pop_back();
    }
  }
}

std::vector<Call> make_calls(uint64_t n, int how_many, uint64_t* lines) {
  std::vector<Call> calls(how_many);
  for (auto& c : calls) {
    c.n = n;
    const uint64_t share = U(3);  // none, some, all set
    for (uint64_t i = 0; i < n; i++) c.bit.push_back(share == 2 || (share == 1 && U(4) == 0));
    c.bitmap.assign((n + 31) / 32, 0xDEADBEEF);
    c.count = ~0ull;
    c.a = fr::Arrivals{lines, c.bitmap.data(), &c.count, n};
  }
  return calls;
}

}  // namespace

int main() {
  int wrong = 0, left = 0, runs = 0;
  for (uint64_t n : {1, 2, 31, 32, 33, 64, 65, 100, 2048, 2049, 2080, 4097}) {
    std::vector<uint64_t> lines(fr::arrive_bytes(n) / 8, 0);
    for (int it = 0; it < (n > 1000 ? 12 : 200); it++) {
      const int overlap = 1 + it % 3;
      for (int how_many : {overlap, 1}) {
        auto calls = make_calls(n, how_many, lines.data());
        run(calls, it % 2 ? 1 + U(8) : 300);
        runs++;
        if (how_many == 1) {
          uint64_t set = 0;
          bool ok = true;
          for (uint64_t i = 0; i < n; i++) {
            set += calls[0].bit[i];
            ok = ok && ((calls[0].bitmap[i / 32] >> (i % 32)) & 1u) == calls[0].bit[i];
          }
          if (n % 32) ok = ok && (calls[0].bitmap.back() >> (n % 32)) == 0;
          if (!ok || calls[0].count != set) wrong++;
        }
        for (uint64_t x : lines)
          if (x) {
            left++;
            break;
          }
      }
    }
  }
  std::printf("%d runs, %d with wrong bits or counts, %d that left lines set\n", runs, wrong, left);
  return wrong || left;
}
