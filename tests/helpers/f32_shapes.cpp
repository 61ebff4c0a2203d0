// The tile shapes that fp32 calls take (zo_common.hpp's rule, as the launchers
// call it): per input line "L V H N B fd C", the row tiles per sign and 16-column
// tiles of a gate launch over all L layers and over one, the head's row tiles (of a
// whole chunk), and the 16-row tiles of a pass.
#include <cstdio>

#include "../../paper_2505_17852_amd/csrc/zo_common.hpp"

int main() {
  int L, V, H, N, B, fd, C;
  while (std::scanf("%d %d %d %d %d %d %d", &L, &V, &H, &N, &B, &fd, &C) == 7) {
    const zo_config c{L, V, 32, H, ZO_WFP32, ZO_RADEMACHER};
    const zo::Rows r = zo::make_rows(N, B, zo::row_granule(c, N, B, fd), fd);
    const zo::RowMap rm = zo::row_map(r);
    const int ns = fd ? 1 : 2, nvt = zo::vocab_tiles(c), T = zo::time_chunk(c, r.M, nvt, C);
    const zo::Pick all = zo::pick_shape(rm, r.M, ns, 4 * (int64_t)H, L, true);
    const zo::Pick one = zo::pick_shape(rm, r.M, ns, 4 * (int64_t)H, 1, true);
    const zo::Pick head = zo::pick_shape(rm, r.M, ns, (int64_t)nvt * zo::kVocabTile, T, false);
    std::printf("%d %d %d %d %d %d\n", all.rt, all.ct, one.rt, one.ct, head.rt, r.Bp / 16);
  }
  return 0;
}
