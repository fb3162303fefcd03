// Checks of the encoder's thread pool, built against the CPU build of the
// library: a call that throws, on the calling thread or in a worker, reaches
// the caller as the exception once no thread is in the loop any more, and the
// pool goes on working; work is dealt out whole when threads cannot be started.
#include "../../paper_2606_24531_amd/csrc/encoder.cpp"

#include <sys/resource.h>

#include <chrono>
#include <stdexcept>

static int g_bad = 0;
static void expect(bool ok, const char* what) {
  printf("%s: %s\n", ok ? "ok" : "FAILED", what);
  fflush(stdout);
  if (!ok) g_bad = 1;
}

// Every index below 64 is slow but for `at`, which throws at once.
static void throwing(Pool& pool, bool in_caller, const char* what) {
  const std::thread::id caller = std::this_thread::get_id();
  std::atomic<int> inside{0}, thrown{0};
  bool caught = false;
  int left_inside = -1;
  try {
    pool.run(64, [&](uint64_t) {
      inside++;
      std::this_thread::sleep_for(std::chrono::milliseconds(2));
      if ((std::this_thread::get_id() == caller) == in_caller && thrown++ == 0) {
        inside--;
        throw std::runtime_error("planted");
      }
      std::this_thread::sleep_for(std::chrono::milliseconds(5));
      inside--;
    });
  } catch (const std::runtime_error&) {
    caught = true;
    left_inside = inside;
  }
  expect(caught && left_inside == 0, what);
  std::atomic<uint64_t> sum{0};
  pool.run(1000, [&](uint64_t i) { sum += i; });
  expect(sum == 499500, "the next loop is whole");
}

int main() {
  {
    Pool pool(4);
    throwing(pool, true, "thrown on the calling thread");
    throwing(pool, false, "thrown in a worker");
  }
  {
    Pool pool(1);
    throwing(pool, true, "thrown with no workers");
  }
  rlimit r{};
  getrlimit(RLIMIT_AS, &r);
  const rlim_t was = r.rlim_cur;
  Pool pool(64);
  std::atomic<uint64_t> sum{0};
  r.rlim_cur = 1;  // no further mapping, so no further thread
  setrlimit(RLIMIT_AS, &r);
  bool threw = false;
  try {
    pool.run(1000, [&](uint64_t i) { sum += i; });
  } catch (...) {
    threw = true;
  }
  r.rlim_cur = was;
  setrlimit(RLIMIT_AS, &r);
  expect(!threw && sum == 499500, "no thread could be started");
  return g_bad;
}
