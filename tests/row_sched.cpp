// Every (head, item) of a one-row grid once, on the XCDs' even shares.
#include <cstdio>
#include <vector>

#include "wise_device.hpp"

int main() {
  using namespace wise;
  for (int heads : {1, 2, 3, 5, 7, 8, 9, 17, 22, 25, 29, 33, 36, 40, 57, 88, 131})
    for (int items : {1, 3, 7, 8, 9, 32, 65, 128})
      for (size_t kv : {(size_t)16384, (size_t)1 << 20, (size_t)2 << 20, (size_t)5 << 20})
        for (bool one : {false, true}) {
          const RowSched s = make_row_sched(heads, items, kv, one);
          if (!s.split) continue;
          std::vector<int> seen((size_t)heads * items);
          int on[8] = {};
          const unsigned grid = row_grid(s);
          for (unsigned b = 0; b < grid; ++b) {
            int h = -1, i = -1;
            if (!split_slot(s, (int)b, h, i)) continue;
            if (h < 0 || h >= heads || i < 0 || i >= items) return 1;
            ++seen[(size_t)h * items + i];
            ++on[b & 7];
          }
          for (int x : seen)
            if (x != 1) return 2;
          for (int x : on)
            if (items % 8 == 0 && x != heads * items / 8) return 3;
        }
  std::puts("ok");
}
