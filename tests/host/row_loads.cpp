// Row loads of the kernels (rows.h), built for the host: every row is laid
// out so that the aligned 16-byte words that hold its entries end at, or start
// after, a page that may not be read.  A load of any other word ends the
// program.
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))

#include <sys/mman.h>
#include <unistd.h>

#include <cstdio>
#include <cstring>

#include "rows.h"

namespace {

constexpr uint32_t kFill = 0xABCD0123u;

// [unreadable page][kPages pages][unreadable page]
constexpr int kPages = 2;
char *guarded(long page) {
  char *p = static_cast<char *>(mmap(nullptr, (kPages + 2) * page, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  if (p == MAP_FAILED || mprotect(p + page, kPages * page, PROT_READ | PROT_WRITE)) return nullptr;
  return p + page;
}

// A row of d entries whose first lies `sh` entries into a 16-byte word, read
// from position b of an array that starts b entries before it.
template <int D, bool V4>
bool check(char *mem, long page, int d, int sh, bool at_end) {
  const int64_t words = d > 0 ? (sh + d + 3) / 4 : 0;  // 16-byte words that hold the row
  char *first = at_end ? mem + kPages * page - 16 * words : mem;
  const uint32_t *row = reinterpret_cast<uint32_t *>(first) + sh;
  uint32_t *fill = reinterpret_cast<uint32_t *>(first);
  for (int k = 0; k < 4 * words; ++k) fill[k] = 1000u + k;
  const int64_t b = 4096 + sh;
  uint32_t r[D];
  gsl::load_row<D, V4>(row - b, b, d, kFill, r);
  for (int k = 0; k < D; ++k)
    if (r[k] != (k < d ? 1000u + sh + k : kFill)) return false;
  return true;
}

template <int D>
bool check_rows(char *mem, long page) {
  for (int d = 0; d <= D; ++d)
    for (int sh = 0; sh < 4; ++sh)
      for (int at_end = 0; at_end < 2; ++at_end) {
        printf("D %d d %d shift %d end %d\n", D, d, sh, at_end);
        fflush(stdout);
        if (!check<D, true>(mem, page, d, sh, at_end) || !check<D, false>(mem, page, d, sh, at_end)) return false;
      }
  return true;
}

}  // namespace

int main() {
  const long page = sysconf(_SC_PAGESIZE);
  char *mem = guarded(page);
  if (!mem) return 2;
  if (!check_rows<8>(mem, page) || !check_rows<16>(mem, page) || !check_rows<32>(mem, page) || !check_rows<64>(mem, page))
    return 1;
  printf("all rows\n");
  return 0;
}
