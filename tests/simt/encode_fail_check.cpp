// Allocation failures inside an encode, built against the CPU build of the
// library: the k-th allocation of a call fails, alone or with all that follow
// it, for every k.  The call then returns ACE_E_NOMEM (or gets by), leaves no
// device buffer behind and lets no exception out.
#include <atomic>
#include <cstdlib>
#include <new>

static std::atomic<long> g_left{-1};  // allocations that still succeed; below 0: all do
static std::atomic<bool> g_once{false};
static thread_local int t_quiet = 0;

void* operator new(size_t n) {
  if (!t_quiet && g_left >= 0 && g_left-- <= 0) {
    if (g_once) g_left = -1;
    else g_left = 0;
    throw std::bad_alloc();
  }
  void* p = malloc(n ? n : 1);
  if (!p) abort();
  return p;
}
void* operator new[](size_t n) { return operator new(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete[](void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
void operator delete[](void* p, size_t) noexcept { free(p); }

#include "../../paper_2606_24531_amd/csrc/common.h"

static std::atomic<int> g_buffers{0};
static hipError_t counted_malloc(void** p, size_t n) {
  g_buffers++;
  t_quiet++;  // the stand-in runtime's own allocations
  const hipError_t r = hipMalloc(p, n);
  t_quiet--;
  return r;
}
static hipError_t counted_free(void* p) {
  g_buffers--;
  return hipFree(p);
}
namespace ace {
static hipError_t quiet_launch(const EncArgs& e, hipStream_t s) {
  const long was = g_left.exchange(-1);  // the stand-in runtime's own allocations
  const hipError_t r = launch_rans_encode(e, s);
  g_left = was;
  return r;
}
}  // namespace ace
#define launch_rans_encode quiet_launch
#define hipMalloc counted_malloc
#define hipFree counted_free
#include "../../paper_2606_24531_amd/csrc/encoder.cpp"

int main() {
  std::vector<uint8_t> x(70'000);
  uint32_t r = 1;
  for (size_t i = 0; i < x.size(); i++) {
    r = r * 1664525u + 1013904223u;
    x[i] = i >= 300 && (i / 50) % 3 ? x[i - 300] : (uint8_t)(r >> 24);
  }
  int bad = 0;
  for (uint32_t flags : {0u, 8u})
    for (uint32_t threads : {1u, 5u})
      for (bool once : {true, false}) {
        ace_encode_params p{20'000, 8, 8, 8, 8, 3, flags, threads};
        std::vector<uint8_t> want(200'000), got(200'000);
        uint64_t n_want = 0, n_got = 0;
        if (ace_encode_archive(x.data(), x.size(), &p, want.data(), want.size(), &n_want) != ACE_OK) return 2;
        long k = 0, nomem = 0;
        for (bool whole = false; !whole; k += k < 60 ? 1 : 1 + k / 16) {
          g_once = once;
          g_left = k;
          const int rc = ace_encode_archive(x.data(), x.size(), &p, got.data(), got.size(), &n_got);
          whole = g_left > 0;  // the call had allocations to spare
          g_left = -1;
          nomem += rc == ACE_E_NOMEM;
          if (rc != ACE_E_NOMEM && (rc != ACE_OK || n_got != n_want || memcmp(got.data(), want.data(), n_want)))
            printf("FAILED: flags %u, %u threads, allocation %ld: %d\n", flags, threads, k, rc), bad = 1;
          if (g_buffers) printf("FAILED: %d device buffers left at %ld\n", (int)g_buffers, k), bad = 1, g_buffers = 0;
        }
        printf("flags %u, %u threads, %s: up to allocation %ld, %ld times out of memory\n", flags, threads,
               once ? "one fails" : "all fail from there", k, nomem);
        fflush(stdout);
        if (!nomem) bad = 1;
      }
  return bad;
}
