// Scene creation's host side (scene_host.h) when the system refuses memory or threads:
// with the k-th allocation refused, for every k, the build throws std::bad_alloc and
// leaves nothing allocated (an exception that left one of its threads, or its caller
// beside a running one, would end the process); where no thread can be started, the
// scene is the same.  Prints one line per case; exit status 1 on failure.

#include <dlfcn.h>
#include <pthread.h>

#include <atomic>
#include <cerrno>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>
#include <vector>

#include "../../paper_1811_03510_amd/csrc/scene_host.h"

namespace {

std::atomic<long> g_live{0}, g_count{0}, g_refuse{-1};
std::atomic<bool> g_no_threads{false};
std::atomic<int> g_started{0};

void* take(std::size_t n) {
  if (g_count.fetch_add(1) == g_refuse.load()) throw std::bad_alloc();
  void* p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  g_live.fetch_add(1);
  return p;
}

void give(void* p) {
  if (!p) return;
  g_live.fetch_sub(1);
  std::free(p);
}

}  // namespace

void* operator new(std::size_t n) { return take(n); }
void* operator new[](std::size_t n) { return take(n); }
void operator delete(void* p) noexcept { give(p); }
void operator delete[](void* p) noexcept { give(p); }
void operator delete(void* p, std::size_t) noexcept { give(p); }
void operator delete[](void* p, std::size_t) noexcept { give(p); }

extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* x) {
  using Fn = int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
  static const Fn real = reinterpret_cast<Fn>(dlsym(RTLD_NEXT, "pthread_create"));
  if (g_no_threads.load()) return EAGAIN;
  g_started.fetch_add(1);
  return real(t, a, f, x);
}

int main() {
  int failures = 0;
  for (uint32_t n : {1u, 700u, 33000u}) {  // the largest builds on several threads, its plan on one
    std::mt19937 g(n);
    std::uniform_real_distribution<float> U(-100.0f, 100.0f);
    std::vector<float> cp(60 * (size_t)n);
    std::vector<uint8_t> types(n);
    for (uint32_t k = 0; k < n; ++k) {
      const float c[3] = {U(g), U(g), U(g)};
      for (int q = 0; q < 20; ++q)
        for (int a = 0; a < 3; ++a) cp[60 * (size_t)k + 3 * q + a] = c[a] + 0.01f * U(g);
      types[k] = (uint8_t)(k % 3 == 0);
    }
    auto build = [&]() { return ccs::make_host_scene(cp, types, 48, 4, 64, 1024); };
    const long before = g_live.load();
    g_started.store(0);
    const ccs::HostScene want = build();
    const bool threaded = g_started.load() > 0;
    if (threaded != (n >= 32768)) {
      std::printf("FAIL: n=%u started %d threads\n", n, g_started.load());
      ++failures;
    }
    auto same = [&](const ccs::HostScene& s) {
      return s.recs == want.recs && s.inv_perm == want.inv_perm && s.bvh.perm == want.bvh.perm &&
             s.refit.words == want.refit.words;
    };
    const long held = g_live.load();
    long refused = 0;
    bool done = false;
    for (long k = 0; !done; ++k) {
      g_count.store(0);
      g_refuse.store(k);
      try {
        const ccs::HostScene s = build();
        g_refuse.store(-1);
        done = g_count.load() <= k;  // fewer allocations than k: none was refused
        if (!same(s)) {
          std::printf("FAIL: n=%u differs at allocation %ld\n", n, k);
          ++failures;
        }
      } catch (const std::bad_alloc&) {
        ++refused;
      }
      g_refuse.store(-1);
      if (g_live.load() != held) {
        std::printf("FAIL: n=%u leaves %ld allocations after %ld\n", n, g_live.load() - held, k);
        ++failures;
        break;
      }
    }
    g_no_threads.store(true);
    if (!same(build())) {
      std::printf("FAIL: n=%u without threads\n", n);
      ++failures;
    }
    g_no_threads.store(false);
    if (refused < 8) {
      std::printf("FAIL: n=%u saw only %ld refusals\n", n, refused);
      ++failures;
    }
    std::printf("n=%u: %ld refusals, threads %s, %ld live before\n", n, refused, threaded ? "yes" : "no", before);
  }
  std::printf("%d failure(s)\n", failures);
  return failures ? 1 : 0;
}
