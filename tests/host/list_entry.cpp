// Host check of the entries of the list of tiles (fbg_kernels.h; built by
// tests/test_host_parts.py): tile and position come back from every entry, up
// to the last tile of 2^37 and the most models before a tile of a block.
#include <stdio.h>

#include "fbg_kernels.h"

int main() {
  const uint64_t tiles[] = {0, 1, 0xFFFFFFFFull, 1ull << 32, (1ull << 32) + 5, (1ull << 33) - 1, (1ull << 37) - 1};
  const uint32_t before[] = {0, 1, 65536, 2047u * 65536u};
  for (uint64_t t : tiles)
    for (uint32_t b : before) {
      const uint64_t e = fbg::list_entry(t, b);
      if (fbg::list_tile(e) != t || fbg::list_before(e) != b) {
        printf("entry of tile %llu, %u before\n", (unsigned long long)t, b);
        return 1;
      }
    }
  return 0;
}
