// Every order of the shared-memory operations of two claiming wavefronts and
// the poller on a small id queue, with the protocol of mc_queue.h.  Each actor
// is a coroutine that stops before every operation on shared memory; the
// orders are enumerated by running again with the next choice.  A claimed id
// has to be the one put in at its position.  argv: slots, ids in the queue at the start,
// ids the poller adds, the smallest claim, first position, read order (1: read, then
// claim; 0: claim, then read, which loses ids).  Prints orders tried, wrong
// claims seen, ids delivered in the order that delivered most.
#include <ucontext.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "mc_queue.h"

namespace {

constexpr int kActors = 3;
ucontext_t g_main, g_ctx[kActors];
char g_stack[kActors][1 << 16];
bool g_over[kActors];
int g_now;

unsigned g_slots, g_start, g_adds, g_per, g_first;
bool g_read_first;
unsigned g_ids[8], g_head, g_tail, g_done, g_wrong, g_claimed;

void step() { swapcontext(&g_ctx[g_now], &g_main); }   // the next operation may wait for others

struct Claimer {
  std::vector<unsigned> got;
  unsigned head() { step(); return g_head; }
  void fetch(unsigned h) {
    got.clear();
    for (unsigned k = 0; k < g_slots; ++k) got.push_back(g_ids[(h + k) % g_slots]);
  }
  void read(unsigned h) { if (g_read_first) { step(); fetch(h); } }
  unsigned take(unsigned h, unsigned to) {
    step();
    const unsigned found = g_head;
    if (found == h) { g_head = to; at = h; }
    return found;
  }
  unsigned at = 0;
};

void claimer() {
  Claimer q;
  step();
  const unsigned tail = g_tail;
  const unsigned c = mc::claim_ids(q, tail, g_per, 2);
  if (c) {
    if (!g_read_first) { step(); q.fetch(q.at); }
    for (unsigned k = 0; k < c; ++k) g_wrong += q.got[k] != q.at + k;
    g_claimed += c;
    step();
    g_done += c;
  }
  g_over[g_now] = true;
  step();
}

void poller() {
  unsigned tail = g_first + g_start;
  for (unsigned put = 0, tries = 0; put < g_adds && tries < g_adds + 1; ++tries) {
    step();
    const unsigned gone = g_done;
    if ((int)mc::queue_room(g_slots, tail, gone) < 1) continue;
    step();
    g_ids[tail % g_slots] = tail;
    ++tail;
    ++put;
    step();
    g_tail = tail;
  }
  g_over[g_now] = true;
  step();
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 7) return 2;
  g_slots = (unsigned)atoi(argv[1]); g_start = (unsigned)atoi(argv[2]); g_adds = (unsigned)atoi(argv[3]);
  g_per = (unsigned)atoi(argv[4]); g_first = (unsigned)strtoul(argv[5], nullptr, 10); g_read_first = atoi(argv[6]) != 0;
  if (g_slots > 8 || g_start > g_slots || g_first % g_slots) return 2;
  std::vector<int> choice, width;                   // of every operation: which actor, of how many
  long long orders = 0;
  unsigned wrong = 0, most = 0;
  for (;;) {
    g_head = g_done = g_first;                      // (as if that many had gone through before)
    g_tail = g_first + g_start;
    for (unsigned k = 0; k < g_start; ++k) g_ids[(g_first + k) % g_slots] = g_first + k;
    g_wrong = g_claimed = 0;
    for (int a = 0; a < kActors; ++a) {
      g_over[a] = false;
      getcontext(&g_ctx[a]);
      g_ctx[a].uc_stack.ss_sp = g_stack[a];
      g_ctx[a].uc_stack.ss_size = sizeof g_stack[a];
      g_ctx[a].uc_link = &g_main;
      makecontext(&g_ctx[a], a < 2 ? claimer : poller, 0);
      g_now = a;
      swapcontext(&g_main, &g_ctx[a]);              // up to its first operation
    }
    for (size_t n = 0;; ++n) {
      int ready[kActors], r = 0;
      for (int a = 0; a < kActors; ++a)
        if (!g_over[a]) ready[r++] = a;
      if (r == 0) break;
      if (n == choice.size()) { choice.push_back(0); width.push_back(r); }
      g_now = ready[choice[n]];
      swapcontext(&g_main, &g_ctx[g_now]);
    }
    ++orders;
    wrong += g_wrong;
    most = std::max(most, g_claimed);
    while (!choice.empty() && choice.back() + 1 == width.back()) { choice.pop_back(); width.pop_back(); }
    if (choice.empty()) break;
    ++choice.back();
  }
  std::printf("%lld %u %u\n", orders, wrong, most);
  return 0;
}
