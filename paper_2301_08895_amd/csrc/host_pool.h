// Host threads of a batch: they sleep between calls, and inside a call run its short parallel phases side
// by side with the caller, spinning from one phase to the next (a phase lasts microseconds).
#pragma once
#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <exception>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

namespace abs_impl {

inline void cpu_relax() {
#if defined(__x86_64__)
  __builtin_ia32_pause();
#endif
}

// Threads 1 .. size(), asleep until start() hands them a job; joined by the destructor.
class HostPool {
 public:
  explicit HostPool(int n) {
    try {                                            // fewer threads than asked for (perhaps none) also do
      threads_.reserve((size_t)n);
      for (int k = 1; k <= n; ++k) threads_.emplace_back([this, k] { loop(k); });
    } catch (const std::exception&) {}
  }
  ~HostPool() {
    { std::lock_guard<std::mutex> g(m_); stop_ = true; }
    wake_.notify_all();
    for (std::thread& t : threads_) t.join();
  }
  int size() const { return (int)threads_.size(); }
  // threads 1 .. n (<= size()) run job(k); returns at once, `job` must live until wait() has returned
  void start(const std::function<void(int)>& job, int n) {
    { std::lock_guard<std::mutex> g(m_); job_ = &job; running_ = wanted_ = n; ++calls_; }
    wake_.notify_all();
  }
  void wait() {
    std::unique_lock<std::mutex> g(m_);
    idle_.wait(g, [this] { return running_ == 0; });
    job_ = nullptr;
  }

 private:
  void loop(int k) {
    uint64_t seen = 0;
    std::unique_lock<std::mutex> g(m_);
    for (;;) {
      wake_.wait(g, [&] { return stop_ || calls_ != seen; });
      if (stop_) return;
      seen = calls_;
      if (k > wanted_) continue;
      const std::function<void(int)>* job = job_;
      g.unlock();
      (*job)(k);
      g.lock();
      if (--running_ == 0) idle_.notify_one();
    }
  }
  std::mutex m_;
  std::condition_variable wake_, idle_;
  const std::function<void(int)>* job_ = nullptr;
  uint64_t calls_ = 0;
  int running_ = 0, wanted_ = 0;
  bool stop_ = false;
  std::vector<std::thread> threads_;
};

// How many threads of the process spin in such calls at the moment, against how many may.  A thread that
// spins takes a whole CPU: with more of them than the process may use, each waits for threads that are not
// running (four batches of eight threads on 16 CPUs: 57 us a round -> up to 30 ms).  So a call that is
// alone has as many as it wishes, and gives the further ones back, down to its least, once others come.
class SpinBudget {
 public:
  explicit SpinBudget(int most) : most_(most) {}
  int take(int least, int wish) {
    const int others = used_.load(std::memory_order_relaxed);
    const int n = std::max(least, std::min(wish, most_ - others));
    used_.fetch_add(n, std::memory_order_relaxed);
    return n;
  }
  int trim(int have, int least) {                    // what of `have` may stay (at least `least`)
    const int over = used_.load(std::memory_order_relaxed) - most_;
    const int n = over > 0 ? std::max(least, have - over) : have;
    if (n < have) give(have - n);
    return n;
  }
  void give(int n) { used_.fetch_sub(n, std::memory_order_relaxed); }
  int used() const { return used_.load(std::memory_order_relaxed); }

 private:
  const int most_;
  std::atomic<int> used_{0};
};

// CPUs that other processes use, or a quota, can be short all the same.  Told of every phase that waits for nothing
// but its threads, this says when they did not get to run for a share of the time that fewer threads would win back:
// phases of kLong and more for over a tenth of the time, at least three close together.  A thread that was held up
// once costs that one phase, not ten seconds with two threads for eight (64 simulations: linear 25 -> 30 us a
// round, softmax 52 -> 64).
class StarvedWatch {
 public:
  using Clock = std::chrono::steady_clock;
  // true: from now on, for kFew, the least threads do
  bool phase_took(Clock::time_point now, double seconds) {
    if (last_ != Clock::time_point{}) lost_ = std::max(0.0, lost_ - kShare * std::chrono::duration<double>(now - last_).count());
    last_ = now;
    if (seconds > kLong) lost_ += std::min(seconds, kMost);
    if (lost_ <= kEnough) return false;
    lost_ = 0.0;
    until_ = now + kFew;
    return true;
  }
  bool starved(Clock::time_point now) const { return now < until_; }

 private:
  static constexpr double kLong = 5e-3, kMost = 8e-3, kEnough = 20e-3, kShare = 0.1;      // seconds; share of the time
  static constexpr std::chrono::seconds kFew{10};
  Clock::time_point last_{}, until_{};
  double lost_ = 0.0;
};

// The threads of one call: the caller (thread 0) and helpers 1 .. size() - 1 of a pool.
class Team {
 public:
  // work(k, size()): thread k's part of a phase.  least <= size() <= wish, and <= 1 + pool->size().
  Team(HostPool* pool, SpinBudget& budget, int least, int wish, std::function<void(int, int)> work)
      : pool_(pool), budget_(budget), work_(std::move(work)), helper_([this](int k) { help(k); }) {
    const int most = 1 + (pool ? pool->size() : 0);
    least_ = std::min(least, most);
    had_ = budget_.take(least_, std::min(wish, most));
    n_.store(had_, std::memory_order_relaxed);
    if (had_ > 1) pool_->start(helper_, had_ - 1);
  }
  ~Team() {                                          // the helpers go back to sleep
    stop_.store(true, std::memory_order_relaxed);
    phase_.fetch_add(1, std::memory_order_release);
    if (had_ > 1) pool_->wait();
    budget_.give(size());
  }
  Team(const Team&) = delete;
  Team& operator=(const Team&) = delete;
  int size() const { return n_.load(std::memory_order_relaxed); }
  void keep_least() {                                // from the next phase on
    const int n = size();
    if (n > least_) { budget_.give(n - least_); n_.store(least_, std::memory_order_relaxed); }
  }
  // One phase on every thread; poll() is called now and then while the others are waited for.
  template <typename Poll>
  void phase(Poll poll) {
    int n = size();
    if (n > least_) n_.store(n = budget_.trim(n, least_), std::memory_order_relaxed);
    done_.store(0, std::memory_order_relaxed);
    phase_.fetch_add(1, std::memory_order_release);
    work_(0, n);
    for (uint64_t spin = 1; done_.load(std::memory_order_acquire) != n - 1; ++spin) {
      if ((spin & 0x3FFF) == 0) poll();
      cpu_relax();
    }
  }

 private:
  void help(int k) {
    int seen = 0;
    for (;;) {
      int p;
      while ((p = phase_.load(std::memory_order_acquire)) == seen) cpu_relax();
      seen = p;
      const int n = size();                          // only ever falls: a thread left out stays out
      if (stop_.load(std::memory_order_relaxed) || k >= n) return;
      work_(k, n);
      done_.fetch_add(1, std::memory_order_release);
    }
  }
  HostPool* const pool_;
  SpinBudget& budget_;
  const std::function<void(int, int)> work_;
  const std::function<void(int)> helper_;
  std::atomic<int> n_{1}, phase_{0}, done_{0};
  std::atomic<bool> stop_{false};
  int least_ = 1, had_ = 1;
};

}  // namespace abs_impl
