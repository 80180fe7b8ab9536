// Touches an array that holds values and one that was never written, both past the size from which
// arrays are touched, and looks at every byte; the second takes one fault a page, and writing it then none.
// Argument: bytes beyond that size.
#include <sys/mman.h>
#include <sys/resource.h>

#include <cstdio>
#include <cstdlib>
#include <vector>

#include "ka_touch.h"

int main(int argc, char **argv)
{
  const size_t bytes = PageToucher::kWorth + (argc > 1 ? std::strtoull(argv[1], nullptr, 10) : 0);
  std::vector<unsigned char> held(bytes + 64);
  for (size_t k = 0; k < held.size(); ++k) held[k] = (unsigned char)(k * 37 + 11);
  unsigned char *fresh = static_cast<unsigned char *>(mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  if (fresh == MAP_FAILED) return 2;
  (void)madvise(fresh, bytes, MADV_NOHUGEPAGE);
  rusage before, after;
  {
    PageToucher touch[2];
    touch[0].add(held.data() + 8, bytes);
    touch[0].wait();
    getrusage(RUSAGE_SELF, &before);
    touch[1].add(fresh, bytes);
  }
  getrusage(RUSAGE_SELF, &after);
  // (a thread's start and end take some of their own)
  const long pages = (long)((bytes + 4095) / 4096);
  if (after.ru_minflt - before.ru_minflt > pages + pages / 2) return std::printf("%ld faults for %ld pages\n", after.ru_minflt - before.ru_minflt, pages), 1;
  getrusage(RUSAGE_SELF, &before);
  volatile unsigned char *const w = fresh;
  for (size_t k = 0; k < bytes; k += 4096) w[k] = 0;
  getrusage(RUSAGE_SELF, &after);
  if (after.ru_minflt - before.ru_minflt > 8) return std::printf("%ld pages were not touched\n", after.ru_minflt - before.ru_minflt), 1;
  for (size_t k = 0; k < held.size(); ++k)
    if (held[k] != (unsigned char)(k * 37 + 11)) return std::printf("byte %zu changed\n", k), 1;
  for (size_t k = 0; k < bytes; ++k)
    if (fresh[k] != 0) return std::printf("fresh byte %zu changed\n", k), 1;
  std::puts("ok");
  return 0;
}
