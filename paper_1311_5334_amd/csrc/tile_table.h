// tile_table.h -- queue sizes and launch shapes of the counting kernel and
// the cell budget per grain, chosen by paper_1311_5334_amd/autotune.py
// --tiles from timings of the whole path; -D on the compiler line overrides
// each value.
//   Against each value's neighbours, in ms a call for one c2 view, 8 c5 views
//   and 16 c3 views (here 0.774, 20.39, 3.535): 3 or 6 slabs a step 0.783,
//   20.56, 3.583 and 0.775, 20.36, 3.525; 1024 or 4096 seeds a chunk 0.777,
//   20.48, 3.533 and 0.777, 20.60, 3.604; 768 workgroups of 512 threads 0.805,
//   20.59, 3.624; 512 of 1024 at eight waves a SIMD 0.848, 22.75, 3.960.
#ifndef EMT_TILE_TABLE_H
#define EMT_TILE_TABLE_H

#ifndef EMT_COUNT_FETCH
#define EMT_COUNT_FETCH 4  // slabs a lane walks per step
#endif
#ifndef EMT_CHUNK_SEEDS
#define EMT_CHUNK_SEEDS 2048  // seeds a workgroup takes at a time
#endif
#ifndef EMT_COUNT_THREADS
#define EMT_COUNT_THREADS 768  // threads of a counting workgroup
#endif
#ifndef EMT_COUNT_BLOCKS
#define EMT_COUNT_BLOCKS 512  // workgroups of the counting kernel
#endif
#ifndef EMT_COUNT_OCCUPANCY
#define EMT_COUNT_OCCUPANCY 6  // waves per SIMD the counting kernel is compiled for
#endif
#ifndef EMT_MERGE_WIDE
#define EMT_MERGE_WIDE 16  // grid-wide merge rounds at most before the per-view tails
#endif
#ifndef EMT_CELLS_PER_GRAIN
#define EMT_CELLS_PER_GRAIN 4  // cells a view may use per grain (plus 4096)
#endif

#endif
