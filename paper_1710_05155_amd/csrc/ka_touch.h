// ka_touch.h -- host memory made resident ahead of a large copy into it.
#pragma once

#include <stddef.h>

#include <thread>
#include <vector>

// Touches the pages of arrays that are about to be written whole, so that a large export is not
// bound by their first use on one thread (fresh memory is copied to at 4 GB/s, touched memory at
// 17).  A touch writes nothing that was not there, so a call that fails before it comes to an array
// leaves that array alone.  Ends with the object.
class PageToucher {
 public:
  static constexpr size_t kWorth = (size_t)4 << 20;   // smaller arrays are left to the copy
  static constexpr int kThreads = 4;

  void add(void *p, size_t bytes)
  {
    if (!p || bytes < kWorth) return;
    char *base = static_cast<char *>(p);
    for (int k = 0; k < kThreads; ++k) {
      const size_t a = bytes / kThreads * k, b = k + 1 < kThreads ? bytes / kThreads * (k + 1) : bytes;
      try {
        threads_.emplace_back([base, a, b] {
          const auto touch = [base](size_t q) {
            char held = 0;   // writes 0 over 0 or what it found: one page fault, a read and a store take two
            (void)__atomic_compare_exchange_n(base + q, &held, (char)0, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED);
          };
          for (size_t q = a; q < b; q += 4096) touch(q);
          if (a < b) touch(b - 1);   // the last page of a part need not begin a multiple of 4096 after its start
        });
      } catch (...) {
        return;   // no more threads: the copy touches the rest itself
      }
    }
  }
  void wait()
  {
    for (std::thread &t : threads_) t.join();
    threads_.clear();
  }
  ~PageToucher() { wait(); }

 private:
  std::vector<std::thread> threads_;
};
