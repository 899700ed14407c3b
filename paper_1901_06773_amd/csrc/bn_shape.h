// Host-side arithmetic of batch norm's sums: how the workgroups of the pass that sums cover a rows x c tensor
// (no device code here).
#pragma once

namespace acc {

constexpr int kBnThreads = 256;              // threads of a workgroup
constexpr int kBnMaxSlabs = 1024;            // largest number of row slabs that a statistics pass adds up
// Workgroups of a pass that sums, over all column slices: three per compute unit, all of them at once, and a quarter fewer partial sums for the
// finishing kernel than four (1024).  768 against 1024 on 38 shapes of each storage type that it changes (forward, backward, storing the masked
// gradient; replayed from a graph, equal shapes differ by 0.3 %), by how many would give every thread its rows:
//   up to 896 (a fifth trip for what are four): sums alone 1.03 times as fast (0.98 to 1.09), sums that store 0.99 (0.93 to 1.05; 1568
//     rows of 2048 fp32 26.0 -> 27.8 us, 25088 of 256 bf16 28.1 -> 29.4): those stay as wanted;
//   up to 2048: 1.02 (0.97 to 1.07);
//   more: fp32 1.01 (0.99 to 1.05), bf16 storing 1.02 (1.00 to 1.04; 200704 rows of 512 276 -> 268 us), but bf16 sums alone 0.99 (0.95
//     to 1.01; 12544 rows of 2048 67.8 -> 70.5 us, 135424 of 100 30.3 -> 31.7): those take 1024.
constexpr int kBnWorkgroups = 768;
constexpr int kBnRowsPerThread = 4;          // rows a thread of the reduction sums at least (else fewer slabs)
constexpr int kSliceMaxSlabs = 512;          // finish and apply in one launch up to here; beyond, the separate finishing launch
constexpr long kSliceMaxRows = 16384;        // ... and, with 2-byte storage, larger tensors: a slice's row segment is 64 bytes
                                             // there (ResNet-152 bf16 at minibatch 512: 3320 with, 3909 images/s without the
                                             // slice kernels; fp32 at minibatch 128: 1326 with, 1310 without)
constexpr bool slice_takes(int elem_size, long rows, long slabs) {
  return slabs <= kSliceMaxSlabs && (elem_size == 4 || rows <= kSliceMaxRows);
}

// tpr threads of v channels each across a row, rpi rows per trip; col_slices workgroups (grid.y) where a row is wider than one
// covers; slabs of rows (grid.x).
struct SumShape {
  int tpr, rpi, col_slices, slabs;
};

// as many slabs as give every thread kBnRowsPerThread rows
inline long slabs_wanted(long rows, int rpi) { return (rows + (long)rpi * kBnRowsPerThread - 1) / ((long)rpi * kBnRowsPerThread); }

// elem_size: bytes of a stored value; v: channels per thread; stores: the pass stores the masked gradient as it sums.
// A function of the shape only.
inline SumShape bn_sum_shape(long rows, int c, int v, int elem_size, bool backward, bool stores) {
  const int groups = c / v;
  SumShape s;
  s.col_slices = (groups + 63) / 64;
  // Eight channels per thread, or two slices that store gradients: slices of like width (65 groups as 33 + 32; bf16 520 channels, 41 images of
  // 28x28 backward 53 -> 47 us; fp32 storing the masked gradient, 25088 rows of 264 channels 63.5 -> 47.9, of 320 61.0 -> 51.3, of 384
  // 65.6 -> 58.9), else as wide as can be (65 as 64 + 1; fp32 516 channels 107 us against 110; storing, 25088 rows of 1028 180 against 191)
  const bool even = v == 8 || (stores && s.col_slices == 2);
  s.tpr = even ? (groups + s.col_slices - 1) / s.col_slices : groups < 64 ? groups : 64;
  // Small tensors: two slices, where they halve the slabs (every workgroup of the slice kernels reads its channels of all of them again).
  // They do between 129 slabs of one slice, below which the sums only get shorter rows, and 512, from where one slice goes to the
  // finishing launch.  One slice -> two, fp32, forward / backward (us): 128 channels, 2000 rows 6.3 -> 6.9 / 7.8 -> 9.1 (not taken), 8036 rows
  // 9.3 -> 8.3 / 12.0 -> 11.0, 16384 rows 11.3 -> 10.6 / 16.6 -> 16.1; 256 channels, 4096 rows 9.7 -> 8.4 / 12.5 -> 11.1; bf16, four channels
  // per thread, 200 channels, 8036 rows 13.2 -> 12.0 / 15.8 -> 14.9, 12544 rows (628 slabs) 13.9 -> 15.3 / 16.2 -> 20.3 (not taken).
  // Beyond 512 slabs fp32 still gains forward (132 to 256 channels, 10000 to 16384 rows: 1.02 to 1.36 times as fast) and backward where rows
  // come in whole 128-byte lines (160 channels, 13000 rows 17.6 -> 15.9, 192, 16000 rows 22.6 -> 20.7, 256, 12544 rows 24.2 -> 22.1; 252 channels,
  // 14500 rows 0.82 times as fast, 200 0.83), but for the pass that stores the masked gradient as it sums at 256 channels only (12544 rows
  // 26.7 -> 25.6; 192 channels, 16384 rows 0.94 times as fast, 224 0.93 to 1.03).
  // Below 32 groups a slice's rows get too short to gain.
  const long one = slabs_wanted(rows, kBnThreads / s.tpr);
  const bool finish_too = elem_size == 4 && (!backward || c % (stores ? 256 : 32) == 0);
  if (v == 4 && rows <= kSliceMaxRows && s.col_slices == 1 && groups >= 32 && one > 128 && (one <= kSliceMaxSlabs || finish_too)) {
    s.col_slices = 2;
    s.tpr = (groups + 1) / 2;
  }
  // tpr need not divide kBnThreads: the leftover threads idle
  s.rpi = kBnThreads / s.tpr;
  // at least kBnRowsPerThread rows per thread and slab (the partials the finishing kernel has to read grow with slabs * c)
  long n = slabs_wanted(rows, s.rpi);
  const long wanted = n * s.col_slices;
  const bool four = stores ? wanted <= kBnWorkgroups / 6 * 7 : elem_size == 2 && wanted > 2 * kBnMaxSlabs;
  const int most = four ? kBnMaxSlabs : kBnWorkgroups;
  const long cap = most / s.col_slices > 0 ? most / s.col_slices : 1;
  if (n > cap) n = cap;
  // few enough for the slice kernels: then as few as one batch of their partial loads
  // (128 slabs of doubles), as long as that leaves a workgroup per compute unit
  if (slice_takes(elem_size, rows, n)) {
    const long one_batch = 128 > 256 / s.col_slices ? 128 : 256 / s.col_slices;
    if (n > one_batch) n = one_batch;
  }
  s.slabs = n < 1 ? 1 : (int)n;
  return s;
}

// Whether the pass that sums stores the masked gradient that is wanted anyway, and the next one reads it in the place of dy and y: a tensor
// less (fp32 256 channels, 295750 rows 489 -> 416 us, 1024 channels, 6936 rows 52 -> 45; bf16 512 channels, 200704 rows 324 -> 272).
// Below a million elements the store costs as much (8.2 -> 8.5 us for 128 rows of 1024).  In an iteration, where a weight gradient runs beside
// and the caches hold smaller tensors, fp32 from 20 million on: ResNet-152, 41 images 30.0 ms from one million on, 29.6 from 12, 29.4 from 20
// or never; 128 images 78.6, 78.2, 78.3, 78.7; ResNet-101, 32 images 16.97, 16.83, 16.78, 16.83.  (bf16, ResNet-50, 128 images 13.0 ms from
// one million on, 13.3 never.)  A function of the shape only: with or without the other stream an iteration gives the same bits.
inline bool bn_stores_early(long rows, int c, int elem_size, bool in_iteration) {
  return rows * c >= (in_iteration && elem_size == 4 ? 20L << 20 : 1L << 20);
}

}  // namespace acc
