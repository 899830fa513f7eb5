// tile_table.h -- queue sizes and launch shapes of the counting kernel and
// the cell budget per grain, chosen by paper_1311_5334_amd/autotune.py
// --tiles from timings of the whole path; -D on the compiler line overrides
// each value.
//   starting tiles {'EMT_COUNT_FETCH': 4, 'EMT_CHUNK_SEEDS': 2048, 'EMT_COUNT_THREADS': 768, 'EMT_COUNT_BLOCKS': 512, 'EMT_COUNT_OCCUPANCY': 6, 'EMT_MERGE_WIDE': 16, 'EMT_CELLS_PER_GRAIN': 4}: c2 0.771 ms, c5x8 20.128 ms, c3x16 3.569 ms
//   chosen tiles {'EMT_COUNT_FETCH': 4, 'EMT_CHUNK_SEEDS': 2048, 'EMT_COUNT_THREADS': 768, 'EMT_COUNT_BLOCKS': 512, 'EMT_COUNT_OCCUPANCY': 6, 'EMT_MERGE_WIDE': 16, 'EMT_CELLS_PER_GRAIN': 4} (each constant's best one-at-a-time variation)
//   13 builds timed; one value changed:
//     EMT_COUNT_FETCH 3: c2 0.780 ms, c5x8 20.425 ms, c3x16 3.572 ms
//     EMT_COUNT_FETCH 6: c2 0.767 ms, c5x8 20.151 ms, c3x16 3.573 ms
//     EMT_CHUNK_SEEDS 1024: c2 0.772 ms, c5x8 20.407 ms, c3x16 3.541 ms
//     EMT_CHUNK_SEEDS 4096: c2 0.770 ms, c5x8 20.351 ms, c3x16 3.654 ms
//     EMT_COUNT_THREADS 512: c2 0.816 ms, c5x8 22.764 ms, c3x16 4.037 ms
//     EMT_COUNT_THREADS 1024: c2 0.845 ms, c5x8 22.509 ms, c3x16 3.984 ms
//     EMT_COUNT_BLOCKS 256: c2 0.873 ms, c5x8 25.727 ms, c3x16 4.471 ms
//     EMT_COUNT_BLOCKS 768: c2 0.802 ms, c5x8 20.289 ms, c3x16 3.648 ms
//     EMT_COUNT_OCCUPANCY 4: c2 0.770 ms, c5x8 20.288 ms, c3x16 3.556 ms
//     EMT_COUNT_OCCUPANCY 8: c2 0.771 ms, c5x8 20.192 ms, c3x16 3.560 ms
//     EMT_MERGE_WIDE 12: c2 0.766 ms, c5x8 20.204 ms, c3x16 3.556 ms
//     EMT_CELLS_PER_GRAIN 8: c2 0.782 ms, c5x8 20.495 ms, c3x16 3.596 ms
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
