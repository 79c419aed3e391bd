// Drives DisjointRanges beside a plain list of ranges that is compared pair by
// pair: every answer and every later answer has to be the same.  Prints the
// number of groups taken and refused.
#include <cstdio>
#include <random>
#include <vector>

#include "disjoint_ranges.h"

using edit::ByteRange;

static bool meet(const ByteRange& a, const ByteRange& b) { return a.lo < b.hi && b.lo < a.hi; }

int main() {
  std::mt19937 gen(1);
  long taken = 0, refused = 0;
  for (int round = 0; round < 20000; ++round) {
    edit::DisjointRanges<96> set;
    std::vector<ByteRange> list;
    const uintptr_t span = 20 + gen() % 3000;  // crowded to sparse
    for (int group = 0; group < 40; ++group) {
      std::vector<ByteRange> r;
      const int want = 1 + gen() % 4;
      for (int tries = 0; tries < 20 && static_cast<int>(r.size()) < want; ++tries) {
        const uintptr_t lo = gen() % span;
        const ByteRange x{lo, lo + 1 + gen() % 40};  // touching ends are common
        bool own = false;
        for (const ByteRange& y : r) own = own || meet(x, y);
        if (!own) r.push_back(x);
      }
      if (list.size() + r.size() > 96 || gen() % 16 == 0) {
        set.clear();
        list.clear();
      }
      bool fits = true;
      for (const ByteRange& x : r)
        for (const ByteRange& y : list) fits = fits && !meet(x, y);
      if (set.meets(r.data(), static_cast<int>(r.size())) == fits) {
        std::printf("round %d group %d: the set disagrees\n", round, group);
        return 1;
      }
      if (fits) {
        set.add(r.data(), static_cast<int>(r.size()));
        list.insert(list.end(), r.begin(), r.end());
      }
      ++(fits ? taken : refused);
    }
  }
  std::printf("%ld %ld\n", taken, refused);
  return 0;
}
