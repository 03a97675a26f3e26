// Runs the lanes of one workgroup on the CPU, one after the other from each
// fence or barrier to the next, in ascending or descending order.  Code whose
// lanes exchange values gives the right result in both orders only if every
// exchange has a fence between the store and the load, and between the load
// and the next store to the same place.
#pragma once
#include <ucontext.h>

#include <functional>
#include <vector>

namespace lanes {
struct Fiber {
  ucontext_t ctx;
  std::vector<char> stack;
  bool done = false;
};
inline std::vector<Fiber>* g_all = nullptr;
inline int g_now = -1;
inline ucontext_t g_main;
inline const std::function<void(int)>* g_body = nullptr;

inline void entry() {
  (*g_body)(g_now);
  (*g_all)[g_now].done = true;
  swapcontext(&(*g_all)[g_now].ctx, &g_main);
}

// body(lane) for `n` lanes in lockstep between fences
inline void run(int n, bool descending, const std::function<void(int)>& body) {
  std::vector<Fiber> all(n);
  g_all = &all;
  g_body = &body;
  for (auto& f : all) {
    f.stack.resize(256 * 1024);
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = f.stack.data();
    f.ctx.uc_stack.ss_size = f.stack.size();
    f.ctx.uc_link = nullptr;
    makecontext(&f.ctx, entry, 0);
  }
  for (int left = n; left > 0;)
    for (int q = 0; q < n; ++q) {
      const int i = descending ? n - 1 - q : q;
      if (all[i].done) continue;
      g_now = i;
      swapcontext(&g_main, &all[i].ctx);
      if (all[i].done) --left;
    }
}
}  // namespace lanes

void lane_yield() {
  ucontext_t& me = (*lanes::g_all)[lanes::g_now].ctx;
  swapcontext(&me, &lanes::g_main);
}
