// Runs the meeting rules of csrc/team.h with workgroups as coroutines, in random
// orders of their accesses, each wait ending at a random moment.  Prints how many
// runs ended with a projector that stands, without one, and with one that stands
// though a workgroup left before its blocks were written (must be 0).
#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "team.h"

namespace {

constexpr int kMaxGroups = 4, kStack = 64 << 10;
ucontext_t g_main, g_ctx[kMaxGroups];
char g_stack[kMaxGroups][kStack];
std::mt19937 g_rng(1);
int g_cur = 0, g_groups = 0, g_meetings = 0, g_late_in = 0;
bool g_ended[kMaxGroups], g_wrote[kMaxGroups];
struct {
  unsigned arrived;
  uint32_t lost;
  int32_t booked;
} g_mem;

void step() { swapcontext(&g_ctx[g_cur], &g_main); }  // another workgroup may run here

struct Ctl {
  void arrive() { step(); ++g_mem.arrived; }
  unsigned arrived() { step(); return g_mem.arrived; }
  bool lost() { step(); return g_mem.lost != 0; }
  bool late() { return g_late_in > 0 && static_cast<int>(g_rng() % g_late_in) == 0; }
  void lose() { step(); g_mem.lost = 1; }
};

void group() {
  const int g = g_cur;
  Ctl c;
  bool on = true;
  for (int k = 1; k <= g_meetings && on; ++k) on = rpca::meet_team(c, static_cast<unsigned>(k * g_groups));
  if (on) {
    step();
    g_wrote[g] = true;
    if (g == 0) g_mem.booked = 1;
  }
  g_ended[g] = true;
  step();
}

}  // namespace

int main(int argc, char** argv) {
  const int runs = argc > 1 ? std::atoi(argv[1]) : 1000;
  long stands = 0, falls = 0, wrong = 0;
  for (int r = 0; r < runs; ++r) {
    g_groups = 2 + static_cast<int>(g_rng() % (kMaxGroups - 1));
    g_meetings = 1 + static_cast<int>(g_rng() % 3);
    g_late_in = static_cast<int>(g_rng() % 3) * 20;  // 0: nobody is ever late
    g_mem.arrived = 0;
    g_mem.lost = 0;
    g_mem.booked = 0;
    std::vector<int> on;
    for (int g = 0; g < g_groups; ++g) {
      g_ended[g] = g_wrote[g] = false;
      getcontext(&g_ctx[g]);
      g_ctx[g].uc_stack.ss_sp = g_stack[g];
      g_ctx[g].uc_stack.ss_size = kStack;
      g_ctx[g].uc_link = nullptr;
      makecontext(&g_ctx[g], group, 0);
      on.push_back(g);
    }
    const int slow = static_cast<int>(g_rng() % (g_groups + 1));  // one that seldom runs (or none)
    while (!on.empty()) {
      size_t i = g_rng() % on.size();
      if (on[i] == slow && on.size() > 1 && g_rng() % 16 != 0) i = (i + 1) % on.size();
      g_cur = on[i];
      swapcontext(&g_main, &g_ctx[g_cur]);
      if (g_ended[g_cur]) on.erase(on.begin() + static_cast<long>(i));
    }
    bool all = true;
    for (int g = 0; g < g_groups; ++g) all = all && g_wrote[g];
    const bool ok = rpca::steps_stand(g_mem.lost, g_mem.booked, 1);
    if (ok && !all) ++wrong;
    if (g_late_in == 0 && !ok) ++wrong;  // nobody late: it has to stand
    if (ok) ++stands;
    else ++falls;
  }
  std::printf("%ld %ld %ld\n", stands, falls, wrong);
  return 0;
}
