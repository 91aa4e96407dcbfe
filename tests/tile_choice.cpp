// The products' tile choice (csrc/ee_tiles.h) as a filter: lines
// "bytes resid qkv P N K ws_floats n_cu" in, "tile splits" out; first the
// number of tiles of bf16 and of fp32.
#include <stdio.h>

#include "ee_tiles.h"

int main() {
  printf("%zu %zu\n", sizeof(ee::MmTiles<uint16_t>::t) / sizeof(ee::MmTile), sizeof(ee::MmTiles<float>::t) / sizeof(ee::MmTile));
  int bytes, resid, qkv, P, N, K, n_cu;
  long long ws;
  while (scanf("%d %d %d %d %d %d %lld %d", &bytes, &resid, &qkv, &P, &N, &K, &ws, &n_cu) == 8) {
    const ee::MmChoice c = bytes == 2 ? ee::mm_choose<uint16_t>(resid, qkv, P, N, K, ws, n_cu)
                                      : ee::mm_choose<float>(resid, qkv, P, N, K, ws, n_cu);
    printf("%zu %d\n", c.tile, c.splits);
  }
  return 0;
}
