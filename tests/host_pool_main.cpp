// Driver of csrc/host_pool.h for the sanitizers (see test_host_pool.py): every check aborts with a message.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../paper_2301_08895_amd/csrc/host_pool.h"

using namespace abs_impl;

static thread_local long t_allocs_left = -1;       // >= 0: that many allocations of this thread still succeed
void* operator new(std::size_t n) {
  if (t_allocs_left == 0) throw std::bad_alloc();
  if (t_allocs_left > 0) --t_allocs_left;
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "line %d: %s\n", __LINE__, #c); std::abort(); } } while (0)

// phases in which item i belongs to thread i % T: every item is taken exactly once, whatever T becomes
struct Call {
  std::vector<int> items = std::vector<int>(37, 0);
  void work(int k, int T) { for (size_t i = (size_t)k; i < items.size(); i += (size_t)T) ++items[i]; }
  void phases(Team& team, int n) {
    for (int p = 0; p < n; ++p) team.phase([] {});
  }
  void done(int n) { for (int v : items) CHECK(v == n); }
};

static void alone(HostPool& pool, SpinBudget& budget) {
  for (int call = 0; call < 40; ++call) {
    Call c;
    Team team(&pool, budget, 2, 8, [&](int k, int T) { c.work(k, T); });
    CHECK(team.size() == 8 && budget.used() == 8);
    c.phases(team, 5);
    if (call % 3 == 0) { team.keep_least(); CHECK(team.size() == 2 && budget.used() == 2); }
    c.phases(team, 5);
    c.done(10);
  }
  CHECK(budget.used() == 0);
}

// Four calls at once: each keeps its least once all of them are there, and the sum stays at the budget.
static void together() {
  SpinBudget budget(8);
  std::atomic<int> here{0}, settled{0}, checked{0};
  auto meet = [](std::atomic<int>& at, int call) {          // all four callers get here
    ++at;
    while (at.load() < 4 * (call + 1)) { cpu_relax(); std::this_thread::yield(); }
  };
  auto caller = [&] {
    HostPool pool(7);
    for (int call = 0; call < 10; ++call) {
      Call c;
      {
        Team team(&pool, budget, 2, 8, [&](int k, int T) { c.work(k, T); });
        meet(here, call);
        c.phases(team, 1);
        meet(settled, call);
        CHECK(team.size() == 2);
        CHECK(budget.used() == 8);
        meet(checked, call);                         // (a call that ends and begins anew may take more for one phase)
        c.phases(team, 20);
      }
      c.done(21);
    }
  };
  std::vector<std::thread> t;
  for (int i = 0; i < 4; ++i) t.emplace_back(caller);
  for (std::thread& x : t) x.join();
  CHECK(budget.used() == 0);
}

static void thrown(HostPool& pool, SpinBudget& budget) {
  for (int i = 0; i < 20; ++i) {
    bool caught = false;
    try {
      Team team(&pool, budget, 2, 8, [&](int k, int) { if (k == 0) throw std::bad_alloc(); });
      team.phase([] {});
    } catch (const std::bad_alloc&) { caught = true; }
    CHECK(caught && budget.used() == 0);
  }
}

static void short_of_memory(SpinBudget& budget) {
  for (long left = 0; left < 12; ++left) {
    t_allocs_left = left;
    HostPool pool(7);
    t_allocs_left = -1;
    CHECK(pool.size() <= 7);
    Call c;
    Team team(&pool, budget, 2, 8, [&](int k, int T) { c.work(k, T); });
    CHECK(team.size() == 1 + pool.size());
    c.phases(team, 3);
    c.done(3);
  }
}

// One thread held up now and then leaves the batch its threads; threads that do not run much of the time do not,
// and not for ever.
static void watched() {
  using namespace std::chrono;
  StarvedWatch::Clock::time_point t = StarvedWatch::Clock::now();
  StarvedWatch once, seldom, often, slow;
  CHECK(!once.starved(t) && !once.phase_took(t, 5.0) && !once.starved(t));
  for (int i = 0; i < 100000; ++i) {
    t += microseconds(50);
    CHECK(!once.phase_took(t, 20e-6));
  }
  for (int i = 0; i < 200; ++i) {                    // 5 ms in every 100
    t += milliseconds(100);
    CHECK(!seldom.phase_took(t, 6e-3));
  }
  int phases = 1;
  for (; !often.phase_took(t, 10e-3); ++phases) { CHECK(phases < 10); t += milliseconds(12); }
  CHECK(phases >= 3 && often.starved(t) && often.starved(t + seconds(9)) && !often.starved(t + seconds(11)));
  t += seconds(11);
  CHECK(!often.phase_took(t, 10e-3));                // starts anew
  for (phases = 1; !slow.phase_took(t, 6e-3); ++phases) { CHECK(phases < 20); t += milliseconds(20); }
}

int main() {
  SpinBudget budget(8);
  HostPool pool(7);
  alone(pool, budget);
  thrown(pool, budget);
  alone(pool, budget);
  short_of_memory(budget);
  together();
  watched();
  {
    Call c;                                         // no pool at all
    Team team(nullptr, budget, 1, 1, [&](int k, int T) { c.work(k, T); });
    c.phases(team, 4);
    c.done(4);
  }
  std::puts("ok");
  return 0;
}
