// line_table.h -- line grids of the counting kernel by grain-density bucket
// (the buckets of cell_table.h): edge of a plane's cells and thickness of a
// slab, in units, and slope bins an axis. Larger cells, thicker slabs and
// fewer bins mean fewer words to fill and fewer slabs to walk, and more grains
// tested per line. The fastest of five to eight settings for 8 views of 350 x
// 350 x 50 um at each bucket's middle density (seed, count and member stages):
//   bucket 0: (250, 1000, 2) 0.81 ms, (400, 1600, 1) 1.40 ms
//   bucket 1: (250, 800, 2) 0.80 ms, (200, 800, 3) 0.86 ms
//   bucket 2: (250, 800, 2) 1.11 ms, (200, 800, 4) 1.27 ms
//   bucket 3: (200, 600, 3) 2.84 ms, (150, 600, 4) 3.30 ms
//   bucket 4: (130, 500, 4) 10.21 ms, (200, 800, 4) 10.41 ms; 8 c5 views
//     (11 per 1000 um^3) 19.3 against 19.9 ms with (150, 600, 4)
//   bucket 5: (110, 400, 4) 27.7 ms, (150, 600, 4) 29.3 ms (4 views)
//   bucket 6: (100, 250, 4) 133 ms, (130, 500, 4) 146 ms (4 views)
#ifndef EMT_LINE_TABLE_H
#define EMT_LINE_TABLE_H

namespace emt {

constexpr int kLineTable[8][3] = {
    {250, 1000, 2},  // bucket 0
    {250, 800, 2},  // bucket 1
    {250, 800, 2},  // bucket 2
    {200, 600, 3},  // bucket 3
    {130, 500, 4},  // bucket 4
    {110, 400, 4},  // bucket 5
    {100, 250, 4},  // bucket 6
    {100, 250, 4},  // bucket 7
};

}  // namespace emt

#endif
