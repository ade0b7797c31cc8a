// Host threads of one pass over a batch.
#pragma once

#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace celeste {

// A wait that lasts a few microseconds on an idle host and any time on a busy one: some turns of looking, then asleep.
// (Threads that only look take the processors from those they wait for.)
class Signal {
 public:
  template <class P>
  void wait(P done) {
    for (int k = 0; k < 500; ++k) {
      if (done()) return;
      std::this_thread::yield();
    }
    std::unique_lock<std::mutex> l(m_);
    cv_.wait(l, done);
  }
  // f changes what done() looks at
  template <class F>
  void set(F f) {
    {
      std::lock_guard<std::mutex> l(m_);
      f();
    }
    cv_.notify_all();
  }

 private:
  std::mutex m_;
  std::condition_variable cv_;
};

// Barrier of the threads of a team.  Once one of them has failed, wait() throws on the others.
class Barrier {
 public:
  struct Broken {};
  void wait() {
    const int g = gen_.load(std::memory_order_acquire);
    if (in_.fetch_add(1, std::memory_order_acq_rel) + 1 == total_) {
      in_.store(0, std::memory_order_relaxed);
      signal_.set([&] { gen_.store(g + 1, std::memory_order_release); });
      return;
    }
    signal_.wait([&] { return gen_.load(std::memory_order_acquire) != g || broken_.load(std::memory_order_acquire); });
    if (gen_.load(std::memory_order_acquire) == g) throw Broken{};
  }
  void set_total(int n) { total_ = n; }
  void fail() {
    signal_.set([&] { broken_.store(true, std::memory_order_release); });
  }

 private:
  int total_ = 1;
  std::atomic<int> in_{0}, gen_{0};
  std::atomic<bool> broken_{false};
  Signal signal_;
};

// Threads for a pass over n items of `ns` nanoseconds each.  A thread takes about 15 us to start, one after the other, so that n
// threads end after work / n + 15 n us: least at the root of the work in units of 15 us.  The checks of 10,000 images'
// records take 95 us, and 105 in each of eight processes on 16 processors (125 and 250 with a thread per
// 2,048 images, which wait spinning; 230 and 235 with one per 8,192); of 40,000 200 and 670 us (605 and 1,830; 580
// and 1,830); a colour's 4,000 patches are found disjoint in 70 us (220..290 on 15 threads, 125 on one).
constexpr int TEAM_MAX = 16;
inline int team_size(int64_t n, int ns) {
  const int nt = (int)std::min<double>(TEAM_MAX, std::max(1.0, std::sqrt((double)n * ns / 15e3)));
  return std::min<int>(nt, std::max(1u, std::thread::hardware_concurrency()));
}

// fn(t, n, barrier) on n threads, the calling one (t = 0) among them: nt, or as many as can be started.  The first
// exception that one of them leaves fn with is thrown here once all have ended.
template <class F>
void team(int nt, F fn) {
  Barrier bar;
  std::exception_ptr error;
  std::mutex m;
  const auto run = [&](int t, int n) {
    try {
      fn(t, n, bar);
    } catch (const Barrier::Broken&) {
    } catch (...) {
      {
        std::lock_guard<std::mutex> l(m);
        if (!error) error = std::current_exception();
      }
      bar.fail();
    }
  };
  if (nt <= 1) {
    fn(0, 1, bar);
    return;
  }
  Signal start;
  std::atomic<int> go{0};   // the number of threads, once all have been started
  std::vector<std::thread> th;
  th.reserve(nt);
  for (int t = 1; t < nt; ++t) {
    try {
      th.emplace_back([&, t] {
        start.wait([&] { return go.load(std::memory_order_acquire) != 0; });
        run(t, go.load(std::memory_order_relaxed));
      });
    } catch (const std::exception&) {
      break;
    }
  }
  const int n = (int)th.size() + 1;
  bar.set_total(n);
  start.set([&] { go.store(n, std::memory_order_release); });
  run(0, n);
  for (auto& x : th) x.join();
  if (error) std::rethrow_exception(error);
}

// The first index of [0, n) for which ok(i), of `ns` nanoseconds, is false, or n.
template <class F>
int64_t first_failure(int64_t n, int ns, F ok) {
  std::atomic<int64_t> bad{n};
  team(team_size(n, ns), [&](int t, int nt, Barrier&) {
    for (int64_t i = n * t / nt; i < n * (t + 1) / nt; ++i)
      if (!ok(i)) {
        int64_t cur = bad.load();
        while (i < cur && !bad.compare_exchange_weak(cur, i)) {
        }
        break;
      }
  });
  return bad.load();
}

}  // namespace celeste
