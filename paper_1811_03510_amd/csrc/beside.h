// Two pieces of host work at once.
#pragma once

#include <exception>
#include <system_error>
#include <thread>

namespace ccs {

// Runs `a` on a thread of its own beside `b`, or before it where the system has no thread
// to give.  Both have ended when this returns or throws; what either throws is thrown here
// (an exception that left the thread itself would end the process, and so would one that
// left `b` while the thread was still to be joined).
template <class A, class B>
void beside(A a, B b) {
  std::exception_ptr failed_a, failed_b;
  std::thread t;
  try {
    t = std::thread([&]() {
      try {
        a();
      } catch (...) {
        failed_a = std::current_exception();
      }
    });
  } catch (const std::system_error&) {
    a();
    b();
    return;
  }
  try {
    b();
  } catch (...) {
    failed_b = std::current_exception();
  }
  t.join();
  if (failed_a) std::rethrow_exception(failed_a);
  if (failed_b) std::rethrow_exception(failed_b);
}

}  // namespace ccs
