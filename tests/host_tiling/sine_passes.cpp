// Prints the shapes of the transform passes of the sine-basis solver. For every line
// "nx member ragged lines" on stdin (member: the grid whose lines the launch meets,
// nx itself unless ragged):
//   parts nq items threads per_wave lds64 lds32 steps served | member's parts nq, items
//   of its forward and inverse transforms, lane logarithms of the two
#include <cstdio>
#include "../../paper_1205_1864_amd/csrc/sg_internal.h"

int main() {
  int nx, member, ragged, lines;
  while (std::scanf("%d %d %d %d", &nx, &member, &ragged, &lines) == 4) {
    const sgk::SinePass p(nx, ragged != 0);
    const sgk::SineSizes m = sgk::sine_sizes(member);
    const int f = sgk::sine_items(member, m.parts, false), i = sgk::sine_items(member, m.parts, true);
    std::printf("%d %d %d %d %d %zu %zu %d %d %d %d %d %d %d %d\n", p.parts, p.nq, p.items, p.threads(), p.per_wave(),
                p.lds(8, lines), p.lds(4, lines), p.steps(member, m.parts, lines),
                (int)(p.served(member, m.parts, lines, 8) && p.served(member, m.parts, lines, 4)), m.parts, m.nq, f, i,
                sgk::sine_lane_log(f), sgk::sine_lane_log(i));
  }
  return 0;
}
