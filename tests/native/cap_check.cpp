// Calls that CCS_MAX_DEVICE_BYTES=1 refuses, on four threads, while the bytes in use are
// read: they never change.  argv[1]: the library.  Exit status 1 on failure.

#include <dlfcn.h>

#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

int main(int, char** argv) {
  setenv("CCS_MAX_DEVICE_BYTES", "1", 1);  // refuses before anything is launched or read
  void* lib = dlopen(argv[1], RTLD_NOW);
  if (!lib) {
    std::printf("%s\n", dlerror());
    return 2;
  }
  auto infer = reinterpret_cast<int (*)(const float*, const float*, uint32_t, float*, void*)>(dlsym(lib, "ccs_policy_infer"));
  auto in_use = reinterpret_cast<uint64_t (*)()>(dlsym(lib, "ccs_device_bytes_in_use"));
  const uint64_t held = in_use();
  std::atomic<int> running{4}, wrong_status{0};
  std::vector<std::thread> threads;
  for (int t = 0; t < 4; ++t)
    threads.emplace_back([&]() {
      float word[4] = {0, 0, 0, 0};
      for (int k = 0; k < 100000; ++k)
        if (infer(word, word, 1, word, nullptr) != 2) wrong_status.fetch_add(1);  // CCS_ERR_OOM
      running.fetch_sub(1);
    });
  uint64_t reads = 0, changed = 0;
  while (running.load() > 0) {
    changed += in_use() != held;
    ++reads;
  }
  for (std::thread& t : threads) t.join();
  std::printf("%llu of %llu reads changed, %d calls not refused\n", (unsigned long long)changed, (unsigned long long)reads,
              wrong_status.load());
  return changed != 0 || wrong_status.load() != 0 || reads < 10000;
}
