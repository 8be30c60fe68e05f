// How a segmented batch is walked and how its slices are cut (k_segmented in
// segmented.hip): the arithmetic of the choices, with no HIP call in it, so
// that a test without a GPU evaluates what the kernel evaluates.
#pragma once

#include <stdint.h>

#include <algorithm>

#ifdef __HIP__
#define RED_HD __host__ __device__ __forceinline__
#else
#define RED_HD inline
#endif

namespace redsum {

// How the slices are cut and walked.
enum SegForm : int {
  kSegAuto = 0,        // chosen on the device
  kSegWorkgroup = 1,   // workgroup slices
  kSegWavePieces = 2,  // wavefront slices, one combine per piece
  kSegWaveRuns = 3,    // wavefront slices, reduce-by-key over lane runs
};

// Batches whose mean segment holds fewer values than this take wavefront
// slices, the others workgroup slices, where the reduce-by-key form is not
// chosen (measured on MI355X: 64- to 4096-value segments run 2 to 8 times
// faster on wavefront slices, long ones about 10 to 30 % faster on workgroup
// slices).
constexpr int64_t kWaveSliceMeanLen = 16384;

RED_HD int long_form(int64_t E, int64_t nseg) {
  return E >= kWaveSliceMeanLen * nseg ? kSegWorkgroup : kSegWavePieces;
}

// Batches whose mean segment holds fewer values than kRunsMeanLen always
// take the reduce-by-key form (plans of at most 4 loads per thread), ragged
// ones up to kRunsRaggedLen.  us per call against one combine per piece, 60 M
// values: equal segments of 512 values 50.2 against 62.0, of 1024 47.5
// against 48.2, of 2048 46.3 against 44.9; of random length (mean 512) 50.2
// against 72.8, (mean 1024) 48.0 against 53.8, (mean 4096) 46.3 against 45.2.
// Log-uniform lengths of mean 65536 take the same in both (10 M values 18.5
// us), since there the pieces of one segment count on one ticket.
constexpr int64_t kRunsMeanLen = 1024;
constexpr int64_t kRunsRaggedLen = 65536;

// Short segments, or less than one value per thread (100,000 values in equal
// segments of 65536: 16.7 us in the other forms, 7.9 in this one).
RED_HD bool short_batch(int64_t E, int64_t nseg, int64_t threads) {
  return E < kRunsMeanLen * nseg || E < threads;
}

// A segment of the sample, [x, y), the next one of the sample starting at
// `next`, against the batch's mean length.
struct SampledSegment {
  bool is_short;   // shorter than a quarter of the mean
  bool is_filled;  // not empty
  bool is_joined;  // only empty segments up to the next sampled one
  bool is_long;    // twice the mean or longer
};

RED_HD SampledSegment sampled_segment(int64_t E, int64_t nseg, int64_t x, int64_t y, int64_t next) {
  const float len = (float)(y - x) * (float)nseg;
  return SampledSegment{4.0f * len < (float)E, y != x, y == x && next == x, len >= 2.0f * (float)E};
}

// How many of the 64 sampled segments are what sampled_segment() tells.
struct SegSample {
  int n_short, n_short_filled, n_filled, n_joined, n_long;
};

// Whether a batch of mean length kRunsMeanLen to kRunsRaggedLen is so ragged
// that the reduce-by-key form, which takes segments of any mix of lengths
// 64 at a time, beats the forms that walk one after another.  us per call,
// the other form / reduce-by-key:
//   * half of the sample short and a quarter short and not empty.  10 M
//     values, log-uniform lengths of mean 1024 27.5 / 16.5, 4096 19.8 / 15.4,
//     32768 20.3 / 15.4; one segment of nearly all values among ones of 100,
//     3e8 values, mean 60000 1905 / 209;
//   * up to twice kRunsMeanLen, one sampled segment long and half of them not
//     empty: random cuts of mean 1024 19.0 / 17.0 (2048 16.8 / 17.0; equal
//     lengths of 4096 13.7 / 14.7);
//   * empty segments in long stretches, where the other forms step over them
//     one by one: equal lengths and then as many empty segments, 10 M values,
//     mean 17000 47.8 / 13.3, 3e8 values 1388 / 187.  One segment of all
//     values among few empty ones is worse here, since its pieces are counted
//     on one ticket, 14 ns each, and there are more of them: 10 M values in
//     588 segments 52.6 / 70.8, in 166 24.9 / 51.1 (60 M in 1000 98 / 93, in
//     3529 264 / 95);
//   * empty segments spread among the others cost the other forms little: 60
//     M values, three of four segments empty, mean 1100 46.1 / 47.5, 4000
//     43.6 / 45.0; 10 M, mean 60000 12.2 / 13.7; 3e8, mean 17000 183.4 / 189.9.
//     Small batches are faster here all the same (1 M values, mean 4000 10.4 /
//     7.5; 10 M 14.1 / 13.7), from kWaveSliceMeanLen up those of at most 64
//     segments, whose slices of a sixteenth of the mean are not more than the
//     other form's, unless half of them hold values (1 M values, mean 60000,
//     three of four empty 12.3 / 9.2, half 8.4 / 9.1).
constexpr int64_t kSpreadEmptyMaxValues = 1 << 24;

RED_HD bool ragged_batch(int64_t E, int64_t nseg, const SegSample& c) {
  if (c.n_long > 0 && c.n_filled >= 32 && E < 2 * kRunsMeanLen * nseg) return true;
  if (c.n_short < 32) return false;
  if (c.n_short_filled >= 16) return true;
  if (c.n_joined >= 16 && (nseg >= 1024 || (nseg >= 512 && c.n_filled >= 8))) return true;
  return E < kWaveSliceMeanLen * nseg ? E < kSpreadEmptyMaxValues : nseg <= 64 && c.n_filled < 32;
}

// Slices of at least this many values: below, more wavefronts do not shorten
// a call, and shorter slices cut more segments (1 M values in segments of
// about 200: 8.4 us per call against 10.0 with slices down to 64).  Long
// segments take slices of a sixteenth of the mean segment, up to
// kRunsLongChunk, so that not too many pieces of one count on one ticket (1 M
// values in 15 log-uniform segments: 10.7 us against 18.9).
constexpr int64_t kRunsMinChunk = 512;
constexpr int64_t kRunsLongChunk = 4096;
// The least where the values start `shift` > 0 elements past a 16-byte
// boundary: 512 of them lie in one vector more than a tile of 2 rows holds, and
// that vector costs a tile (random cuts of mean 2000, 270,000 values 7.2 us per
// call against 8.0, 1.7 M 9.9 against 10.4).
constexpr int64_t kRunsMinChunkShifted = 448;

// Values of a slice of the reduce-by-key form over W wavefronts.
RED_HD int64_t runs_slice(int64_t E, int64_t nseg, int64_t W, int shift) {
  const int64_t mean = (int64_t)((float)E / (float)nseg);
  return std::max<int64_t>({shift ? kRunsMinChunkShifted : kRunsMinChunk, (((E + W - 1) / W) + 63) & ~(int64_t)63,
                            std::min<int64_t>(mean / 16, kRunsLongChunk) & ~(int64_t)63});
}

// Rows of the largest tile.  The wide kernels keep 16 wavefronts per CU (123
// VGPRs with 8 rows), the others 20 and more; the host takes a wide one for a
// grid that is then wholly resident.
constexpr int runs_max_rows(int ipt, bool wide) { return ipt == 4 ? (wide ? 8 : 4) : ipt == 2 && wide ? 4 : 2; }

// Rows (64 vectors of 4 values) of the tiles that a slice is walked in: 8
// (2048 values) for slices of more than 7168 values (three and a half such
// tiles), so that a tile's fixed work is spread over more values (32 M values
// in segments of 64: 31.0 us against 32.8 with 4 rows); 4 rows below, so that a
// short slice is still several tiles, the last of them nearly full, and one
// loads while the other is walked (20 M values: 21.5 us against 23.8 with 8
// rows); 2 rows for slices of 512.
constexpr int64_t kRows8Above = 7168, kRows4Above = 512;
RED_HD int runs_rows(int max_rows, int64_t slice) {
  return max_rows >= 8 && slice > kRows8Above ? 8 : max_rows >= 4 && slice > kRows4Above ? 4 : 2;
}

// Vectors of a tile buffer, and the place in it of the tile's vector i: one
// vector of padding after every 8, so that the run reads (lane l, vector
// ROWS l + j) of neighbouring lanes fall in distinct banks, as do the writes of
// a row, and every read and write of a lane lies at a fixed distance from its
// first.
constexpr int run_tile_vectors(int rows) { return 64 * rows * 9 / 8; }
RED_HD constexpr int run_place(int i) { return i + (i >> 3); }

// A tile with more non-empty segments than this holds more sums than its LDS
// has room for, and is walked in halves.
constexpr int run_max_starts(int rows) { return 2 * 64 * rows; }

}  // namespace redsum
