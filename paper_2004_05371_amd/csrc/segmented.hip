// Batched segmented sum reduction over a fixed grid (gfx950).
//
// The paper's persistent-kernel reduction (Section VII-C, explicit
// synchronization) keeps one grid of blocks alive for the whole job.  Here a
// fixed grid handles a whole CSR batch of uneven segments:
//
//   * the concatenated values are cut into equal slices (chunk = ceil(E / S)
//     rounded up to 64 values), one per workgroup or, when the batch's mean
//     segment is short, one per wavefront, so every slice streams the same
//     number of bytes whatever the segment lengths;
//   * a slice finds its first segment by binary search in the offsets
//     (read through the scalar cache), then streams its values as one
//     sequence of tiles of 16-byte vectors (the next tile in flight while
//     the current one is added into fp32 TwoSum-compensated accumulators,
//     or, in the reduce-by-key form, into binary64 per-lane runs);
//   * the segments are finished in one of three forms, chosen on the device
//     from the mean segment length and a sample of lengths (seg_rules.h): a
//     piece that ends in a tile is finished by a wavefront combine per wave,
//     completed in batches of 64 pieces after one workgroup barrier (workgroup
//     slices); by one DPP wavefront combine (wavefront slices); or, for short
//     or ragged ones, the wavefront reduces by key over per-lane runs of
//     consecutive values with a segmented scan across its lanes
//     (seg_wave_runs);
//   * a segment that lies inside the slice is written directly (binary64);
//     a piece of a segment that crosses a slice boundary goes to a carry
//     slot, and the pieces of that segment are summed in slice order in
//     binary64 by one wavefront: by the wavefront that publishes the last
//     piece (atomic ticket per owning slice, the default), in a second
//     kernel after the launch boundary (relaunch fix-up), or by the owning
//     slice after a grid barrier (co-resident grid); within one launch the
//     pieces are published with device-scope atomic stores, so neither the
//     ticket nor the barrier needs an L2 write-back or invalidation.
//
// Workgroup slices keep few concurrent streams (better DRAM locality) and
// suit long segments; wavefront slices let every wave walk its own pieces
// without barriers and suit short ones.  Empty segments write 0.  The
// result is deterministic for a given grid and workgroup size, and the
// three fix-ups give the same bits.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "device_prims.h"
#include "internal.h"
#include "seg_rules.h"

namespace redsum {

struct SegArgs {
  const float* x;
  const int64_t* offsets;
  int64_t nseg;
  double* out;
  SegCarry* carry_in;   // piece of a segment that started before the slice
  SegCarry* carry_out;  // piece of a segment that starts in the slice and continues
  unsigned* tickets;    // per owning slice: pieces published so far
  BarrierWords* words;
  unsigned spin_limit;
  unsigned bar_groups;
  int form;  // SegForm: automatic, or one form forced
  // Workgroups of the slice kernel and threads per workgroup.  The kernels
  // take the sizes from here: blockDim.x costs a dependent load through
  // vector memory, 0.2 to 0.4 us per call where a wavefront has little to do.
  int grid;
  int wg;
};

// How the pieces of a segment cut by slice boundaries are summed.
enum SegFix : int {
  kFixTicket = 0,    // the wavefront that publishes the last piece (atomic ticket)
  kFixBarrier = 1,   // the owning slice, after a grid barrier (co-resident grid)
  kFixRelaunch = 2,  // a second kernel, after the implicit barrier between launches
};

// offsets[i] through the scalar data cache (the offsets are read-only for
// the whole launch), so the segment walk waits on scalar loads only and
// never on the vector loads of the stream in flight.
__device__ __forceinline__ int64_t offset_at(const int64_t* offsets, int64_t i) {
  return ((const __attribute__((address_space(4))) int64_t*)offsets)[i];
}

// offsets[i] and offsets[i + 1] in one load (offsets are 8-byte aligned).
typedef long long v2l __attribute__((ext_vector_type(2), aligned(8)));

// Sum of the np pieces of a cut segment (owning slice o: carry_out[o], then
// carry_in[o+1 .. o+np-1]) by one wavefront: lane l adds pieces o+l,
// o+l+64, ... in order, then the fixed binary64 wavefront combine
// (returned to every lane).  The pieces are read with device-scope atomic
// loads: the ticket and grid-barrier fix-ups read them in the launch that
// published them, with no acquire.
__device__ __forceinline__ double combine_pieces(const SegArgs& a, int64_t o, int64_t np) {
  double v = 0.0;
  for (int64_t k = o + __lane_id(); k < o + np; k += kWave)
    v += load_published(k == o ? &a.carry_out[o].val : &a.carry_in[k].val);
  return wave_reduce_dpp<OpF64>(v);
}

// A carry slot published to the other workgroups of the same launch.
__device__ __forceinline__ void publish_carry(SegCarry* slot, int64_t s, double v, int64_t np) {
  publish(&slot->seg, (long long)s);
  publish(&slot->val, v);
  publish(&slot->np, (long long)np);
}

// Completes, by one wavefront, the piece [max(sa, lo), min(sb, hi)) of
// segment s whose total is v: a whole segment is written; a piece of a cut
// segment is published in its carry slot (slice w), and the wavefront that
// completes the segment's ticket sums all of its pieces (ticket fix-up), or
// the owning wavefront does so after the grid barrier (barrier fix-up:
// *own_fix records the segment), or the fix-up kernel that follows does
// (relaunch fix-up: the slot is an ordinary store, made visible by the
// kernel boundary).  Within one launch the slots are published with
// device-scope atomic stores, waited for before the ticket or the barrier,
// so no workgroup writes back its L2 or invalidates it.
template <int FIX>
__device__ __forceinline__ void finish_piece(const SegArgs& a, int64_t s, int64_t sa, int64_t sb, double v,
                                             int64_t lo, int64_t hi, int64_t w, int64_t chunk, int64_t* own_fix) {
  const int lane = __lane_id();
  if (sa >= lo && sb <= hi) {
    if (lane == 0) a.out[s] = v;
    return;
  }
  const int64_t o = sa / chunk;
  const int64_t np = (sb - 1) / chunk - o + 1;
  if constexpr (FIX == kFixRelaunch) {
    if (lane == 0) {
      if (sa < lo)
        a.carry_in[w] = SegCarry{s, v, np};
      else
        a.carry_out[w] = SegCarry{s, v, np};
    }
  } else if constexpr (FIX == kFixBarrier) {
    if (lane == 0) publish_carry(sa < lo ? &a.carry_in[w] : &a.carry_out[w], s, v, np);
    if (sa >= lo) *own_fix = s;
  } else {
    int last = 0;
    if (lane == 0) {
      publish_carry(sa < lo ? &a.carry_in[w] : &a.carry_out[w], s, v, np);
      drain_stores();
      const unsigned tk = __hip_atomic_fetch_add(&a.tickets[o], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = tk == (unsigned)(np - 1);
    }
    if (__builtin_amdgcn_readfirstlane(last)) {  // this wave published the last piece
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      const double t = combine_pieces(a, o, np);
      if (lane == 0) {
        a.out[s] = t;
        __hip_atomic_store(&a.tickets[o], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// Moves the segment cursor s to the next non-empty segment that starts
// before hi, writing 0 (if `writer`) for the empty segments passed on the
// way (those at positions in [lo, hi), and, for the slice that ends at E,
// those at E).  Returns false when the slice holds no further segment.
__device__ __forceinline__ bool seek_segment(const SegArgs& a, int64_t& s, int64_t hi, int64_t E, bool end_slice,
                                             int64_t& sa, int64_t& sb, bool writer) {
  for (; s < a.nseg; ++s) {
    sa = offset_at(a.offsets, s);
    sb = offset_at(a.offsets, s + 1);
    if (sa >= hi && !(end_slice && sa == E)) return false;
    if (sa != sb) return true;
    if (writer) a.out[s] = 0.0;
  }
  return false;
}

// The first s in [0, nseg] with offsets[s] >= pos (0 <= pos <= E =
// offsets[nseg], nseg > 0), by one wavefront: 64 lanes probe at a time, so a
// batch of two million segments takes 4 dependent loads and not 21; the last
// 128 candidates are read at once (5333 segments: two dependent loads, not
// three; 8 M values in equal segments 13.0 us per call against 13.7).  Eight
// candidates a lane instead of two cost 0.3 us: 16 wavefronts of a CU search at
// once, and what counts is how many lanes' addresses they send.
__device__ __forceinline__ int64_t first_at_or_after(const int64_t* offsets, int64_t nseg, int64_t pos) {
  const int lane = __lane_id();
  int64_t L = 0, R = nseg;  // the answer lies in [L, R]; offsets[R] >= pos
  while (R - L > 2 * kWave) {
    const int64_t d = R - L;
    // Probe l at L + (l + 1) d / 64; the last one is R itself.
    const bool below = offsets[L + (((int64_t)(lane + 1) * d) >> 6)] < pos;
    const int c = __popcll(__ballot(below));  // probes 0 .. c-1 lie below; c < 64
    R = L + (((int64_t)(c + 1) * d) >> 6);
    if (c > 0) L = L + (((int64_t)c * d) >> 6) + 1;
  }
  const int64_t i = L + 2 * lane;
  v2l e = {pos, pos};
  if (i < R) e = *reinterpret_cast<const v2l*>(offsets + i);
  return L + __popcll(__ballot(e.x < pos)) + __popcll(__ballot(i + 1 < R && e.y < pos));
}

// The segment that holds element lo of a non-empty slice, or for an empty
// slice the first one that starts at or after lo: the first s with
// offsets[s] >= lo, stepped back by one when segment s-1 crosses lo.
__device__ __forceinline__ int64_t first_segment(const SegArgs& a, int64_t lo) {
  const int64_t L = first_at_or_after(a.offsets, a.nseg, lo);
  return (L > 0 && offset_at(a.offsets, L) > lo) ? L - 1 : L;
}

// Adds to acc the elements of the thread's IPT vectors of one tile that lie
// in the tile-relative range [ra, rb) (0 <= ra <= rb <= 4 T): vector u of
// thread idx (0 <= idx < bs) starts at element 4 (u bs + idx) of the tile.
// A wave whose 256 elements of row u miss the range skips that row (the
// test is wave-uniform).  32-bit unsigned range test: r in [ra, rb) iff
// r - ra < rb - ra.
template <int IPT>
__device__ __forceinline__ void add_masked(CompF32* acc, const v4f* v, int bs, int idx, int ra, int rb) {
  const unsigned w = (unsigned)(rb - ra);
  const int wave0 = __builtin_amdgcn_readfirstlane(idx & ~(kWave - 1));
#pragma unroll
  for (int u = 0; u < IPT; ++u) {
    const int wb = 4 * (u * bs + wave0);  // first element of this wave's part of row u
    if (wb >= rb || wb + 4 * kWave <= ra) continue;
    const unsigned r = (unsigned)(4 * (u * bs + idx) - ra);
    v4f x = v[u];
    x.x = r < w ? x.x : 0.0f;
    x.y = r + 1u < w ? x.y : 0.0f;
    x.z = r + 2u < w ? x.z : 0.0f;
    x.w = r + 3u < w ? x.w : 0.0f;
    ModeF32Comp::add_vec(acc[u], x);
  }
}

// Whether any of the calling wave's rows of a workgroup tile meets [ra, rb).
template <int IPT>
__device__ __forceinline__ bool wave_touches(int bs, int ra, int rb) {
  const int wave0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~(kWave - 1));
  bool t = false;
#pragma unroll
  for (int u = 0; u < IPT; ++u) {
    const int wb = 4 * (u * bs + wave0);
    t = t || (wb < rb && wb + 4 * kWave > ra);
  }
  return t;
}

// Pieces whose workgroup combine is finished together, after one barrier.
constexpr int kBatch = 64;

struct PieceInfo {
  int64_t s, sa, sb;  // segment id and its bounds
};

// At most 512 threads per workgroup: a thread keeps two tiles of IPT
// 16-byte vectors and IPT compensated accumulators in registers, which for
// IPT = 8 needs more than the 128 VGPRs a 1024-thread workgroup allows.
constexpr int kSegMaxWG = 512;

// Wavefront-granular slices (short segments: every wave walks its own
// pieces, with no workgroup barrier): wavefront w of the grid owns slice
// w and streams it as tiles of 64 x IPT vectors.
template <int IPT, bool NT, int FIX>
__device__ __forceinline__ void seg_wave_slices(const SegArgs& a) {
  // Barrier fix-up: thread 0 holds the barrier generation of this launch.
  unsigned gen = FIX == kFixBarrier ? grid_barrier_gen(a.words) : 0u;
  using M = ModeF32Comp;
  const int nwaves = a.wg / kWave;
  const int lane = __lane_id();
  const int64_t w = (int64_t)blockIdx.x * nwaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t W = (int64_t)a.grid * nwaves;
  const int64_t nseg = a.nseg;
  const int64_t E = offset_at(a.offsets, nseg);
  const int64_t chunk = std::max<int64_t>(64, (((E + W - 1) / W) + 63) & ~(int64_t)63);
  const int64_t lo = std::min(w * chunk, E);
  const int64_t hi = std::min(lo + chunk, E);
  // The slice that ends at E also writes the empty segments that sit at
  // position E (for E == 0: slice 0).
  const bool end_slice = E > 0 ? (lo < E && hi == E) : (w == 0);
  // Relaunch fix-up: the slot says "no cut segment starts here" unless a
  // later store by the same lane replaces it.
  if constexpr (FIX == kFixRelaunch)
    if (lane == 0) a.carry_out[w] = SegCarry{-1, 0.0, 0};

  int64_t s = first_segment(a, lo);
  int64_t sa = 0, sb = 0;
  bool have = seek_segment(a, s, hi, E, end_slice, sa, sb, lane == 0);
  int64_t A = std::max(sa, lo), B = std::min(sb, hi);  // current piece

  // The slice is streamed as one sequence of tiles (64 x IPT 16-byte
  // vectors of the 16-byte-aligned base, the next tile's loads issued
  // before the current tile is added), whatever the segment boundaries.
  const int shift = (int)((reinterpret_cast<uintptr_t>(a.x) & 15) >> 2);
  const v4f* xa = reinterpret_cast<const v4f*>(a.x - shift);
  const int64_t vlo = (lo + shift) >> 2;
  const int64_t vhi = (hi + shift + 3) >> 2;  // vectors [vlo, vhi) hold the slice
  constexpr int64_t T = kWave * IPT;
  const int64_t ntiles = lo < hi ? (vhi - vlo + T - 1) / T : 0;

  CompF32 acc[IPT];
#pragma unroll
  for (int u = 0; u < IPT; ++u) acc[u] = M::zero();
  v4f cur[IPT], nxt[IPT];
  auto load_tile = [&](v4f* v, int64_t t) {
    const int64_t v0 = vlo + t * T + lane;
    if (vlo + (t + 1) * T <= vhi) {
#pragma unroll
      for (int u = 0; u < IPT; ++u) v[u] = load_vec<NT>(xa + v0 + u * kWave);
    } else {
#pragma unroll
      for (int u = 0; u < IPT; ++u)
        v[u] = v0 + u * kWave < vhi ? load_vec<NT>(xa + v0 + u * kWave) : v4f{0, 0, 0, 0};
    }
  };

  int64_t own_fix = -1;  // barrier form: the cut segment this slice owns
  if (ntiles > 0) load_tile(cur, 0);
  for (int64_t t = 0; t < ntiles; ++t) {
    // The current tile is complete before the next one is requested, so
    // nothing below waits on the loads in flight (on this target a wait
    // with stores and loads both pending would drain every load).
    __builtin_amdgcn_s_waitcnt(0);
    if (t + 1 < ntiles) load_tile(nxt, t + 1);
    __builtin_amdgcn_sched_barrier(0);
    const int64_t e0 = 4 * (vlo + t * T) - shift;        // first element of the tile
    const int64_t e1 = 4 * (vlo + (t + 1) * T) - shift;  // one past its last
    auto rel = [&](int64_t e) { return (int)std::min(std::max(e - e0, (int64_t)0), 4 * T); };
    // Pieces that end in this tile.
    while (have && B <= e1) {
      add_masked<IPT>(acc, cur, kWave, lane, rel(A), rel(B));
      CompF32 tot = acc[0];
#pragma unroll
      for (int u = 1; u < IPT; ++u) tot = OpComp::add(tot, acc[u]);
#pragma unroll
      for (int u = 0; u < IPT; ++u) acc[u] = M::zero();
      tot = wave_reduce_dpp<OpComp>(tot);
      finish_piece<FIX>(a, s, sa, sb, comp_to_double(tot), lo, hi, w, chunk, &own_fix);
      ++s;
      have = seek_segment(a, s, hi, E, end_slice, sa, sb, lane == 0);
      A = std::max(sa, lo);
      B = std::min(sb, hi);
    }
    // The piece that continues past this tile.
    if (have) {
      if (A <= e0 && vlo + (t + 1) * T <= vhi) {
#pragma unroll
        for (int u = 0; u < IPT; ++u) M::add_vec(acc[u], cur[u]);
      } else {
        add_masked<IPT>(acc, cur, kWave, lane, rel(A), rel(B));
      }
    }
#pragma unroll
    for (int u = 0; u < IPT; ++u) cur[u] = nxt[u];
  }
  if constexpr (FIX == kFixBarrier) {
    grid_barrier_published(a.words, a.grid, a.bar_groups, a.spin_limit, gen);
    if (own_fix >= 0) {
      __atomic_signal_fence(__ATOMIC_SEQ_CST);  // the pieces are loaded as published
      const int64_t o = offset_at(a.offsets, own_fix) / chunk;
      const int64_t np = (offset_at(a.offsets, own_fix + 1) - 1) / chunk - o + 1;
      const double v = combine_pieces(a, o, np);
      if (lane == 0) a.out[own_fix] = v;
    }
  }
}

// Reduce-by-key form of the wavefront slices, for short segments of any mix
// of lengths.
//
// Each tile of 64 x ROWS 16-byte vectors (256 ROWS contiguous values) comes
// in by coalesced loads, one tile ahead, and is turned over in LDS so that
// lane l holds the run of RL = 4 ROWS consecutive values from RL l on.  Then
//   * 64 offsets at a time, lane k takes the segment q + k that starts in the
//     tile: a non-empty one sets the bit of its start in a mask word per
//     run, and its rank among the tile's non-empty segments is its place in
//     the ballot;
//   * each lane adds up its run in binary64; at a start it puts the sum so
//     far in LDS (where the tile was) at the start's rank and begins again,
//     so a run may hold any number of starts;
//   * a segmented scan of what is left at the runs' ends gives each lane the
//     partial of the segment open at its left edge, which it adds to the sum
//     at its first start;
//   * the sum at rank j + 1 belongs to the segment of rank j: the lanes that
//     took the segments write them out in their order, 64 neighbouring sums
//     at a time, and 0 for the empty ones.
// The sum at rank 0 closes the segment that was open before the tile, which
// may have begun before the slice and then goes through finish_piece.  A
// tile without a start adds to per-lane sums of the open segment and needs
// no scan.  A tile with more starts than its LDS holds sums (half its
// values) is walked in two halves, which cannot.
//
// What bounds it is latency that four wavefronts per SIMD do not hide: the
// steps of a tile depend on one another through LDS and memory.  By the
// counters a wavefront waits for one of these 47 % of its time (32 M values in
// segments of 16 on average) or 41 % (67 M in segments of 512), for its turn to
// issue 27 and 32 %; the VALU is busy about a quarter of the time, LDS 23 and
// 29 %, 9 and 0.4 % of that with bank conflicts.  So the runs are as long as
// four wavefronts have registers for, to spread a tile's fixed steps, about 250
// operations, over more values (about 10 operations per row of 64; smaller
// tiles with five or six wavefronts were slower).  The walk it replaced finished every
// tile with an empty segment, or with two starts in one run, piece by piece,
// bound by the chain of dependent steps of each piece.  64 M values, us per
// call now and before: segments of random length (empty ones among them) of
// mean 4 118 / 3631, 16 69 / 1148, 64 59 / 402, 512 54 / 64; equal lengths
// of 4 114 / 2864, 16 66 / 72, 64 56 / 61, 512 52 / 57.
template <int ROWS>
struct RunLds {
  v4f tile[run_tile_vectors(ROWS)];  // one tile of up to ROWS rows, padded; then sums by rank
  unsigned mask[kWave];              // per lane run: bit i set when a segment starts at its value i
};

constexpr int kChunks = 4;  // chunks of 64 offsets loaded a tile ahead

// The wavefront's LDS instructions execute in program order, so words that
// one lane writes and another reads need no wait, only an order that the
// compiler keeps.
template <class T>
using LdsPtr = __attribute__((address_space(3))) T*;

template <class T>
__device__ __forceinline__ LdsPtr<T> lds_ptr(T* p) {
  return (LdsPtr<T>)p;
}

__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Lanes of the ballot b below the calling one.
__device__ __forceinline__ int lanes_below(uint64_t b) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
}

// The slice [lo, hi) of wavefront w, by tiles of ROWS rows.
template <int ROWS, bool NT, int FIX>
__device__ __forceinline__ void seg_walk_runs(const SegArgs& a, const LdsPtr<v4f> tile, const LdsPtr<unsigned> mask,
                                              int64_t w, int64_t chunk, int64_t lo, int64_t hi, int64_t E,
                                              bool end_slice, int64_t& own_fix) {
  static_assert(ROWS <= 8, "runs of at most 32 values");
  const LdsPtr<double> sums = (LdsPtr<double>)tile;
  const int lane = __lane_id();
  const int nseg = (int)a.nseg;  // below 2^31
  const int shift = (int)((reinterpret_cast<uintptr_t>(a.x) & 15) >> 2);
  const v4f* xa = reinterpret_cast<const v4f*>(a.x - shift);
  const int64_t vlo = (lo + shift) >> 2;
  const int64_t vhi = (hi + shift + 3) >> 2;  // vectors [vlo, vhi) hold the slice
  constexpr int64_t T = kWave * ROWS;
  const int64_t ntiles = lo < hi ? (vhi - vlo + T - 1) / T : 0;
  // Past the slice's last vector that vector is read again (its values lie
  // at or past hi there and are masked out): one path and one place in the
  // loop, so that the loads go straight to the registers that the next
  // tile is taken from (where paths meet, a register that a load is still
  // to fill is copied, which waits for the load).
  v4f cur[ROWS];
  auto load_tile = [&](int64_t t) {
    const int64_t v0 = vlo + t * T + lane;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) cur[u] = load_vec<NT>(xa + std::min(v0 + u * kWave, vhi - 1));
  };
  if (ntiles > 0) load_tile(0);

  // q: the first segment that starts at or after the position reached.
  // so: the non-empty segment open there (-1: none), which began before
  // the slice if `cut`; its sum so far is Cs, plus the sum of cl over the
  // lanes if `spread`.
  int q = (int)first_at_or_after(a.offsets, nseg, lo);
  double Cs = 0.0, cl = 0.0;
  bool spread = false;

  // Entry c 64 + lane from q on: its start and the next one's (past the
  // last segment, the last segment's again: take() tells by the count).
  auto entry = [&](int at, int c) -> v2l {
    const int i = std::min(c * kWave + lane, nseg - at - 1);
    return *reinterpret_cast<const v2l*>(a.offsets + at + i);
  };
  // Chunks loaded ahead: as many as the mean segment length makes a tile
  // need (further ones are loaded when they turn out to be needed).
  const int ahead = (int)std::min<int64_t>(
      kChunks, 1 + (4 * T * nseg / std::max<int64_t>(E, 1) + kWave / 2) / kWave);
  v2l ent[kChunks];
  auto load_entries = [&]() {
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
      if (c < ahead) ent[c] = entry(q, c);
  };
  if (ntiles > 0) load_entries();
  mask[lane] = 0u;
  // Every load completes before the stores that follow it are issued, on
  // every path: with loads and stores pending together the compiler can
  // only wait for all of them.
  auto loads_done = [] { __builtin_amdgcn_s_waitcnt(0); };
  loads_done();
  // The segment before q crosses lo unless q starts there.
  int so = ntiles > 0 && q > 0 && (q == nseg || read_lane(ent[0].x, 0) > lo) ? q - 1 : -1;
  bool cut = so >= 0;

  // Walks the part of the tile that starts at value f0 and whose run values
  // are xv; returns false, with nothing changed, when it holds too many
  // starts for LDS.
  auto part = [&](auto rl_tag, const float* xr, int64_t f0) -> bool {
    constexpr int RL = decltype(rl_tag)::value;
    const int64_t f1 = f0 + (int64_t)kWave * RL;
    const int64_t fe = std::min(f1, hi);
    if (f0 >= hi) return true;

    // The segments that start in the part, by chunks of 64: R non-empty
    // ones, cnt in all, the last non-empty one s_last.
    int R = 0, cnt = 0, s_last = 0;
    // Rank of the lane's segment: -1 not in the part, -2 empty.  Returns
    // whether the next chunk may hold more.
    auto take = [&](v2l e, int s0, int& rank) -> bool {
      const bool in = e.x < fe && lane < nseg - s0;
      const bool full = in && e.y != e.x;
      const uint64_t b = __ballot(full);
      const int r = R + lanes_below(b);
      rank = in ? (full ? r : -2) : -1;
      if (full) {
        const unsigned p = (unsigned)e.x - (unsigned)f0;
        __hip_atomic_fetch_or(mask + p / RL, 1u << (p % RL), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      }
      s_last = b ? s0 + 63 - __builtin_clzll(b) : s_last;
      R += __popcll(b);
      const int n = __popcll(__ballot(in));
      cnt += n;
      return n == kWave;
    };
    int rank[kChunks];
    bool more = true;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      rank[c] = -1;
      if (more && c < ahead) more = take(ent[c], q + c * kWave, rank[c]);
    }
    const int R_ahead = R, cnt_ahead = cnt;
    while (more) {
      v2l e[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) e[c] = entry(q + cnt, c);
      const int s0 = q + cnt;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        int unused;
        if (more) more = take(e[c], s0 + c * kWave, unused);
      }
      __builtin_amdgcn_s_waitcnt(0);  // those not taken, so that no later use of the registers waits
    }
    wave_order();
    const unsigned word = mask[lane];
    mask[lane] = 0u;
    wave_order();
    if constexpr (RL == 4 * ROWS)
      if (R > run_max_starts(ROWS)) return false;
    const int q0 = q;
    q += cnt;
    load_entries();

    float xv[RL];
#pragma unroll
    for (int i = 0; i < RL; ++i) xv[i] = xr[i];
    if (f0 < lo || f1 > hi) {  // values outside the slice are not its own
      const int64_t p = f0 + (int64_t)RL * lane;
#pragma unroll
      for (int i = 0; i < RL; ++i) xv[i] = (p + i >= lo && p + i < hi) ? xv[i] : 0.0f;
    }
    if (R == 0) {
#pragma unroll
      for (int i = 0; i < RL; ++i) cl += (double)xv[i];
      spread = true;
      loads_done();
      return true;
    }
    if (spread) {
      Cs += wave_reduce_dpp<OpF64>(cl);
      cl = 0.0;
      spread = false;
    }
    const int own = __popc(word);
    const LdsPtr<double> first = sums + (wave_scan_add(own) - own);  // the lane's first start
    LdsPtr<double> at = first;
    double acc = lane == 0 ? Cs : 0.0;  // the open segment enters with the first run
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      if (word & (1u << i)) {
        *at++ = acc;
        acc = 0.0;
      }
      acc += (double)xv[i];
    }
    int f = word != 0u;
    wave_segscan(acc, f);
    const double left = dpp_move<kWaveShr1, 0xF, 0xF>(acc);  // lane - 1's scan; 0 in lane 0
    if (word != 0u) *first = left + *first;
    Cs = read_lane(acc, kWave - 1);
    wave_order();

    // Results.
    loads_done();
    if (so >= 0) {
      if (!cut) {
        if (lane == 0) a.out[so] = sums[0];
      } else {
        finish_piece<FIX>(a, so, offset_at(a.offsets, so), offset_at(a.offsets, so + 1), sums[0], lo, hi, w, chunk,
                          &own_fix);
      }
    }
    so = s_last;
    cut = false;
    auto put = [&](int s0, int rk) {
      if (rk != -1 && rk + 1 < R) {
        const double v = sums[std::max(rk + 1, 0)];
        a.out[s0 + lane] = rk >= 0 ? v : 0.0;
      }
    };
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
      if (c < ahead) put(q0 + c * kWave, rank[c]);
    if (cnt > cnt_ahead) {  // the chunks beyond: their ranks again
      int Rc = R_ahead;
      for (int d = cnt_ahead; d < cnt; d += kWave) {
        const v2l e = entry(q0 + d, 0);
        const bool in = e.x < fe && lane < nseg - (q0 + d), full = in && e.y != e.x;
        const uint64_t b = __ballot(full);
        put(q0 + d, in ? (full ? Rc + lanes_below(b) : -2) : -1);
        Rc += __popcll(b);
      }
    }
    wave_order();
    return true;
  };

  // Batches whose mean segment is under 2.25 values are walked in halves
  // from the start.
  const bool dense = 4 * E < 9 * (int64_t)nseg;
  constexpr int RL = 4 * ROWS, RH = 2 * ROWS;  // values per lane run of a tile, of a half
  for (int64_t t = 0; t < ntiles; ++t) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u) tile[run_place(u * kWave) + run_place(lane)] = cur[u];
    wave_order();
    load_tile(t + 1);
    const int64_t e0 = 4 * (vlo + t * T) - shift;
    float xr[RL];
    // The lane's run of `rows` vectors in the half (or whole) tile whose
    // first vector is i0, to xr[at ..].
    auto read_runs = [&](auto rows_tag, int i0, int at) {
      constexpr int N = decltype(rows_tag)::value;
      const LdsPtr<v4f> run = tile + run_place(i0) + run_place(N * lane);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const v4f y = run[j];
        xr[at + 4 * j] = y.x, xr[at + 4 * j + 1] = y.y, xr[at + 4 * j + 2] = y.z, xr[at + 4 * j + 3] = y.w;
      }
    };
    bool done = false;
    if (!dense) {
      read_runs(std::integral_constant<int, ROWS>{}, 0, 0);
      wave_order();
      done = part(std::integral_constant<int, RL>{}, xr, e0);
    }
    if (!done) {
      read_runs(std::integral_constant<int, ROWS / 2>{}, 0, 0);
      read_runs(std::integral_constant<int, ROWS / 2>{}, kWave * ROWS / 2, RH);
      wave_order();
      part(std::integral_constant<int, RH>{}, xr, e0);
      part(std::integral_constant<int, RH>{}, xr + RH, e0 + kWave * RH);
    }
    wave_order();
  }
  if (so >= 0) {  // the segment open at the slice's end ends at or after hi
    if (spread) Cs += wave_reduce_dpp<OpF64>(cl);
    finish_piece<FIX>(a, so, offset_at(a.offsets, so), offset_at(a.offsets, so + 1), Cs, lo, hi, w, chunk, &own_fix);
  }
  if (end_slice)  // the empty segments at E
    for (int64_t i = (int64_t)q + lane; i < nseg; i += kWave) a.out[i] = 0.0;
}

// The reduce-by-key form over the slices of runs_slice() values, in tiles of
// runs_rows() rows.
template <int MAX_ROWS, bool NT, int FIX>
__device__ __forceinline__ void seg_wave_runs(const SegArgs& a, RunLds<MAX_ROWS>* lds_all) {
  // Barrier fix-up: thread 0 holds the barrier generation of this launch.
  unsigned gen = FIX == kFixBarrier ? grid_barrier_gen(a.words) : 0u;
  const int nwaves = a.wg / kWave;
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t w = (int64_t)blockIdx.x * nwaves + wv;
  const int64_t W = (int64_t)a.grid * nwaves;
  const int64_t E = offset_at(a.offsets, a.nseg);
  const int64_t chunk = runs_slice(E, a.nseg, W, (int)((reinterpret_cast<uintptr_t>(a.x) & 15) >> 2));
  const int64_t lo = std::min(w * chunk, E);
  const int64_t hi = std::min(lo + chunk, E);
  const bool end_slice = E > 0 ? (lo < E && hi == E) : (w == 0);
  // Relaunch fix-up: the slot says "no cut segment starts here" unless a
  // later store by the same lane replaces it.
  if constexpr (FIX == kFixRelaunch)
    if (lane == 0) a.carry_out[w] = SegCarry{-1, 0.0, 0};
  int64_t own_fix = -1;
  if (lo < hi || end_slice) {
    const LdsPtr<v4f> tile = lds_ptr(lds_all[wv].tile);
    const LdsPtr<unsigned> mask = lds_ptr(lds_all[wv].mask);
    if (MAX_ROWS >= 8 && chunk > kRows8Above)  // runs_rows(), with no value to keep
      seg_walk_runs<MAX_ROWS, NT, FIX>(a, tile, mask, w, chunk, lo, hi, E, end_slice, own_fix);
    else if (MAX_ROWS >= 4 && chunk > kRows4Above)
      seg_walk_runs<MAX_ROWS >= 4 ? 4 : 2, NT, FIX>(a, tile, mask, w, chunk, lo, hi, E, end_slice, own_fix);
    else
      seg_walk_runs<2, NT, FIX>(a, tile, mask, w, chunk, lo, hi, E, end_slice, own_fix);
  }
  if constexpr (FIX == kFixBarrier) {
    grid_barrier_published(a.words, a.grid, a.bar_groups, a.spin_limit, gen);
    if (own_fix >= 0) {
      __atomic_signal_fence(__ATOMIC_SEQ_CST);  // the pieces are loaded as published
      const int64_t o = offset_at(a.offsets, own_fix) / chunk;
      const int64_t np = (offset_at(a.offsets, own_fix + 1) - 1) / chunk - o + 1;
      const double v = combine_pieces(a, o, np);
      if (lane == 0) a.out[own_fix] = v;
    }
  }
}

// Workgroup-granular slices (long segments: few streams, little per-piece
// work): workgroup g owns slice g, streams it as tiles of blockDim x IPT
// vectors, and finishes the pieces that end in a tile in batches of
// kBatch after one workgroup barrier, wave w finishing pieces w,
// w + nwaves, ...
// Per-wave partials of up to kBatch finished pieces, completed together
// after one barrier.  Two buffers used alternately: a wave writes a buffer
// again only after the next batch's barrier, which every wave reaches after
// its reads of that buffer.
struct WorkgroupLds {
  CompF32 part[2][kBatch][kMaxWavesPerWG];
  PieceInfo info[2][kBatch];
  int64_t own_fix;  // barrier form: cut segment this workgroup owns
};

template <int IPT, bool NT, int FIX>
__device__ __forceinline__ void seg_workgroup_slices(const SegArgs& a, WorkgroupLds& lds) {
  // Barrier fix-up: thread 0 holds the barrier generation of this launch.
  unsigned gen = FIX == kFixBarrier ? grid_barrier_gen(a.words) : 0u;
  using M = ModeF32Comp;
  auto& part = lds.part;
  auto& info = lds.info;
  int64_t& own_fix = lds.own_fix;
  int buf = 0, nb = 0;
  const int64_t nseg = a.nseg;
  const int64_t E = offset_at(a.offsets, nseg);
  const int64_t G = a.grid;
  const int64_t g = blockIdx.x;
  const int64_t chunk = std::max<int64_t>(64, (((E + G - 1) / G) + 63) & ~(int64_t)63);
  const int64_t lo = std::min(g * chunk, E);
  const int64_t hi = std::min(lo + chunk, E);
  // The workgroup whose slice ends at E also writes the empty segments that
  // sit at position E (for E == 0: workgroup 0).
  const bool end_wg = E > 0 ? (lo < E && hi == E) : (g == 0);

  int64_t s = first_segment(a, lo);
  int64_t sa = 0, sb = 0;
  bool have = seek_segment(a, s, hi, E, end_wg, sa, sb, threadIdx.x == 0);
  int64_t A = std::max(sa, lo), B = std::min(sb, hi);  // current piece

  // The slice is streamed as one sequence of tiles (blockDim x IPT 16-byte
  // vectors of the 16-byte-aligned base, the next tile's loads issued
  // before the current tile is added), whatever the segment boundaries: a
  // piece that ends inside a tile is finished (workgroup combine and
  // publication) while the next tile is in flight.
  const int shift = (int)((reinterpret_cast<uintptr_t>(a.x) & 15) >> 2);
  const v4f* xa = reinterpret_cast<const v4f*>(a.x - shift);
  const int64_t vlo = (lo + shift) >> 2;
  const int64_t vhi = (hi + shift + 3) >> 2;  // vectors [vlo, vhi) hold the slice
  const int64_t bs = a.wg;
  const int64_t T = bs * IPT;
  const int64_t ntiles = lo < hi ? (vhi - vlo + T - 1) / T : 0;
  const int tid = threadIdx.x;
  const int wave = tid / kWave;
  const int lane = tid % kWave;
  const int nwaves = (int)bs / kWave;
  if (tid == 0) own_fix = -1;
  // Relaunch fix-up: "no cut segment starts here" unless a store after the
  // first batch barrier replaces it.  The fix-up kernel looks at one slot
  // per wavefront of the grid, so the other waves also clear the slots
  // [G, G * nwaves) that workgroup slices do not use.
  if constexpr (FIX == kFixRelaunch) {
    if (tid == 0) a.carry_out[g] = SegCarry{-1, 0.0, 0};
    if (wave > 0 && lane == 0) a.carry_out[G + g * (nwaves - 1) + (wave - 1)] = SegCarry{-1, 0.0, 0};
  }

  // Completes the batched pieces: wave w finishes pieces w, w + nwaves, ...
  auto flush = [&]() {
    __syncthreads();
    for (int j = wave; j < nb; j += nwaves) {
      CompF32 v = lane < nwaves ? part[buf][j][lane] : OpComp::zero();
      v = wave_reduce_dpp<OpComp>(v);
      const PieceInfo& pi = info[buf][j];
      finish_piece<FIX>(a, pi.s, pi.sa, pi.sb, comp_to_double(v), lo, hi, g, chunk, &own_fix);
    }
    buf ^= 1;
    nb = 0;
  };

  CompF32 acc[IPT];
#pragma unroll
  for (int u = 0; u < IPT; ++u) acc[u] = M::zero();
  v4f cur[IPT], nxt[IPT];
  auto load_tile = [&](v4f* v, int64_t t) {
    const int64_t v0 = vlo + t * T + tid;
    if (vlo + (t + 1) * T <= vhi) {
#pragma unroll
      for (int u = 0; u < IPT; ++u) v[u] = load_vec<NT>(xa + v0 + u * bs);
    } else {
#pragma unroll
      for (int u = 0; u < IPT; ++u) v[u] = v0 + u * bs < vhi ? load_vec<NT>(xa + v0 + u * bs) : v4f{0, 0, 0, 0};
    }
  };

  if (ntiles > 0) load_tile(cur, 0);
  for (int64_t t = 0; t < ntiles; ++t) {
    // The current tile is complete before the next one is requested, so
    // nothing below waits on the loads in flight (on this target a wait
    // with stores and loads both pending would drain every load).
    __builtin_amdgcn_s_waitcnt(0);
    if (t + 1 < ntiles) load_tile(nxt, t + 1);
    __builtin_amdgcn_sched_barrier(0);
    const int64_t e0 = 4 * (vlo + t * T) - shift;        // first element of the tile
    const int64_t e1 = 4 * (vlo + (t + 1) * T) - shift;  // one past its last
    const int64_t span = e1 - e0;  // 4 T elements
    auto rel = [&](int64_t e) { return (int)std::min(std::max(e - e0, (int64_t)0), span); };
    // Pieces that end in this tile: each wave's share goes to the batch.
    while (have && B <= e1) {
      const int ra = rel(A), rb = rel(B);
      add_masked<IPT>(acc, cur, (int)bs, tid, ra, rb);
      CompF32 tot = acc[0];
#pragma unroll
      for (int u = 1; u < IPT; ++u) tot = OpComp::add(tot, acc[u]);
#pragma unroll
      for (int u = 0; u < IPT; ++u) acc[u] = M::zero();
      // A piece that started in this tile has nothing in the waves whose
      // rows miss it: they skip the wavefront combine.
      if (A < e0 || wave_touches<IPT>((int)bs, ra, rb)) tot = wave_reduce_dpp<OpComp>(tot);
      else tot = OpComp::zero();
      if (lane == 0) part[buf][nb][wave] = tot;
      if (tid == 0) info[buf][nb] = PieceInfo{s, sa, sb};
      if (++nb == kBatch) flush();
      ++s;
      have = seek_segment(a, s, hi, E, end_wg, sa, sb, threadIdx.x == 0);
      A = std::max(sa, lo);
      B = std::min(sb, hi);
    }
    // The piece that continues past this tile.
    if (have) {
      if (A <= e0 && vlo + (t + 1) * T <= vhi) {
#pragma unroll
        for (int u = 0; u < IPT; ++u) M::add_vec(acc[u], cur[u]);
      } else {
        add_masked<IPT>(acc, cur, (int)bs, tid, rel(A), rel(B));
      }
    }
#pragma unroll
    for (int u = 0; u < IPT; ++u) cur[u] = nxt[u];
  }
  if (nb > 0) flush();
  if constexpr (FIX == kFixBarrier) {
    grid_barrier_published(a.words, a.grid, a.bar_groups, a.spin_limit, gen);  // also a workgroup barrier
    const int64_t os = own_fix;
    if (os >= 0 && wave == 0) {
      __atomic_signal_fence(__ATOMIC_SEQ_CST);  // the pieces are loaded as published
      const int64_t o = offset_at(a.offsets, os) / chunk;
      const int64_t np = (offset_at(a.offsets, os + 1) - 1) / chunk - o + 1;
      const double v = combine_pieces(a, o, np);
      if (lane == 0) a.out[os] = v;
    }
  }
}

// One form runs per launch, so the forms share the workgroup's LDS, which
// is dynamic: the reduce-by-key form needs one RunLds per wavefront, so a
// small workgroup does not reserve the space of a 512-thread one.
template <int MAX_ROWS>
union SegLds {
  WorkgroupLds wg;
  RunLds<MAX_ROWS> runs[kSegMaxWG / kWave];
};

size_t run_lds_bytes(int max_rows) {
  return max_rows == 8 ? sizeof(RunLds<8>) : max_rows == 4 ? sizeof(RunLds<4>) : sizeof(RunLds<2>);
}

size_t seg_lds_bytes(int wg, int max_rows) {
  return std::max(sizeof(WorkgroupLds), (size_t)(wg / kWave) * run_lds_bytes(max_rows));
}

// The form of a launch: forced, or from the batch's mean segment length and,
// for plans of at most 4 loads per thread, from the lengths of 64 segments
// evenly spaced over the batch (the same decision in every workgroup; the
// rules and their figures are in seg_rules.h).  One wavefront per workgroup
// takes the sample, 64 cache lines: taken by each of a CU's 16 wavefronts it
// held up the loads behind it.
template <int IPT>
__device__ __forceinline__ int seg_form(const SegArgs& a, int* shared) {
  if (a.form != kSegAuto) return a.form;
  const bool sampler = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) == 0;
  v2l sample = {0, 0};
  if (IPT <= 4 && sampler)
    sample = *reinterpret_cast<const v2l*>(a.offsets + (((int64_t)__lane_id() * a.nseg) >> 6));
  const int64_t E = offset_at(a.offsets, a.nseg);
  if constexpr (IPT <= 4) {
    if (short_batch(E, a.nseg, (int64_t)a.grid * a.wg)) return kSegWaveRuns;
    if (E < kRunsRaggedLen * a.nseg) {
      if (sampler) {
        const long long next = dpp_move<kWaveShl1, 0xF, 0xF>((long long)sample.x);
        const SampledSegment l = sampled_segment(E, a.nseg, sample.x, sample.y, next);
        auto lanes = [](bool p) { return (int)__popcll(__ballot(p)); };
        const SegSample c{lanes(l.is_short), lanes(l.is_short && l.is_filled), lanes(l.is_filled), lanes(l.is_joined),
                          lanes(l.is_long)};
        if (__lane_id() == 0) *shared = ragged_batch(E, a.nseg, c) ? kSegWaveRuns : long_form(E, a.nseg);
      }
      __syncthreads();
      return __builtin_amdgcn_readfirstlane(*shared);
    }
  }
  return long_form(E, a.nseg);
}

template <int IPT, bool NT, int FIX, bool WIDE>
__global__ __launch_bounds__(kSegMaxWG) void k_segmented(SegArgs a) {
  extern __shared__ __align__(16) unsigned char seg_lds[];
  constexpr int MAX_ROWS = runs_max_rows(IPT, WIDE);
  SegLds<MAX_ROWS>& lds = *reinterpret_cast<SegLds<MAX_ROWS>*>(seg_lds);
  __shared__ int shared_form;
  const int form = seg_form<IPT>(a, &shared_form);
  if (form == kSegWorkgroup) {
    seg_workgroup_slices<IPT, NT, FIX>(a, lds.wg);
  } else if (form == kSegWaveRuns) {
    if constexpr (IPT <= 4) seg_wave_runs<MAX_ROWS, NT, FIX>(a, lds.runs);
  } else {
    seg_wave_slices<IPT, NT, FIX>(a);
  }
}

// Relaunch fix-up: wavefront w of this grid looks at carry slot w, which
// the slice kernel wrote for every w below its grid's wavefront count
// (slice w's slot in the wavefront forms; in the workgroup form, the slots
// past the grid say "none"); if a cut segment starts in slice w, it sums
// the segment's pieces in slice order (the same combine as the ticket and
// barrier fix-ups) and writes it.  The slot holds the segment and its
// piece count, so the fix-up reads no offsets.
constexpr int kFixupWG = 256;

__global__ __launch_bounds__(kFixupWG) void k_seg_fixup(SegArgs a) {
  const int64_t w = (int64_t)blockIdx.x * (kFixupWG / kWave) + threadIdx.x / kWave;
  if (w >= (int64_t)a.grid * (a.wg / kWave)) return;
  const SegCarry c = a.carry_out[w];
  if (c.seg < 0) return;
  const double v = combine_pieces(a, w, c.np);
  if (__lane_id() == 0) a.out[c.seg] = v;
}

namespace {

int ipt_index(int ipt) { return ipt == 1 ? 0 : ipt == 2 ? 1 : ipt == 4 ? 2 : ipt == 8 ? 3 : -1; }

struct SegTable {
  const void* k[3][2][4][2];  // SegFix, nontemporal, ipt index, wide
  template <int F, bool NT>
  void fill() {
    k[F][NT][0][0] = k[F][NT][0][1] = reinterpret_cast<const void*>(&k_segmented<1, NT, F, false>);
    k[F][NT][1][0] = reinterpret_cast<const void*>(&k_segmented<2, NT, F, false>);
    k[F][NT][1][1] = reinterpret_cast<const void*>(&k_segmented<2, NT, F, true>);
    k[F][NT][2][0] = reinterpret_cast<const void*>(&k_segmented<4, NT, F, false>);
    k[F][NT][2][1] = reinterpret_cast<const void*>(&k_segmented<4, NT, F, true>);
    k[F][NT][3][0] = k[F][NT][3][1] = reinterpret_cast<const void*>(&k_segmented<8, NT, F, false>);
  }
  SegTable() {
    fill<kFixTicket, false>();
    fill<kFixTicket, true>();
    fill<kFixBarrier, false>();
    fill<kFixBarrier, true>();
    fill<kFixRelaunch, false>();
    fill<kFixRelaunch, true>();
  }
};

const SegTable& seg_table() {
  static const SegTable t;
  return t;
}

}  // namespace

// Default (measured on MI355X over uniform segment lengths and 10,000
// log-uniform ones): the atomic-ticket fix-up.  With the cut pieces
// published by device-scope atomic stores it is one kernel and 1 to 4 %
// faster than the relaunch fix-up's two (768-value segments, every slice
// boundary a cut: 188 against 196 us; with a release fence per cut piece
// it had taken 405 us).  Four 256-thread workgroups per CU: 16 wavefronts,
// the most the reduce-by-key form keeps resident, which beat two 512-thread
// workgroups by up to 8 % on 16-value segments and 2 to 4 % at 512 values
// and on the drawn batch; 4 loads of 16 bytes per thread per tile.
red_plan default_seg_plan(int64_t nseg, const DeviceInfo& dev) {
  (void)nseg;
  red_plan p;
  p.variant = RED_VARIANT_ATOMIC;
  p.wg = 256;
  p.ipt = 4;
  p.grid = 4 * dev.cus;
  p.flags = RED_FLAG_NONTEMPORAL;
  return p;
}

namespace {
// Workgroups of wg threads per CU of the (wide or other) grid-barrier kernel
// with `ipt` loads per thread: asked once.
int seg_per_cu(int ii, int wg, bool wide, int* per_cu) {
  static std::atomic<int> known[4][kSegMaxWG / kWave + 1][2];  // 0: not asked yet
  std::atomic<int>& c = known[ii][wg / kWave][wide ? 1 : 0];
  int v = c.load(std::memory_order_relaxed);
  if (v == 0) {
    RED_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, seg_table().k[kFixBarrier][0][ii][wide ? 1 : 0], wg,
                                                         seg_lds_bytes(wg, runs_max_rows(1 << ii, wide))));
    c.store(v, std::memory_order_relaxed);
  }
  *per_cu = v;
  return RED_OK;
}
}  // namespace

int seg_max_coresident(int ipt, int wg, const DeviceInfo& dev, int* n_wg) {
  const int ii = ipt_index(ipt);
  if (ii < 0) return set_error(RED_EINVAL, "bad ipt %d", ipt);
  int narrow = 0, wide = 0;
  int rc = seg_per_cu(ii, wg, false, &narrow);
  if (!rc) rc = seg_per_cu(ii, wg, true, &wide);
  if (rc) return rc;
  *n_wg = std::max(narrow, wide) * dev.cus;
  return RED_OK;
}

int seg_launch(const SegLaunch& sl, const float* x, const int64_t* offsets, int64_t nseg, double* out,
               Workspace* ws, hipStream_t s, const DeviceInfo& dev) {
  const red_plan& p = sl.plan;
  const int ii = ipt_index(p.ipt);
  if (ii < 0) return set_error(RED_EINVAL, "bad ipt %d", p.ipt);
  if (p.wg > kSegMaxWG) return set_error(RED_EINVAL, "segmented: at most %d threads per workgroup", kSegMaxWG);
  const bool barrier = p.variant == RED_VARIANT_PERSISTENT;
  const int fix = barrier ? kFixBarrier : p.variant == RED_VARIANT_RELAUNCH ? kFixRelaunch : kFixTicket;
  if (!barrier && p.variant != RED_VARIANT_ATOMIC && p.variant != RED_VARIANT_RELAUNCH)
    return set_error(RED_EINVAL, "segmented: variant must be RELAUNCH, ATOMIC (ticket) or PERSISTENT (barrier)");
  int grid = p.grid > 0 ? p.grid : 4 * dev.cus;
  grid = std::max(1, std::min(grid, RED_MAX_GRID));
  // One carry slot and one ticket per wavefront slice.
  grid = std::min<int>(grid, (int)(kMaxChunks / (p.wg / kWave)));
  if (barrier) {
    int maxg = 0;
    int rc = seg_max_coresident(p.ipt, p.wg, dev, &maxg);
    if (rc) return rc;
    if (grid > maxg)
      return set_error(RED_EINVAL, "segmented persistent: grid %d exceeds %d co-resident workgroups",
                       grid, maxg);
  }
  // The wide kernel if all of the grid is resident with it.  The rule is the
  // same for the three fix-ups, so that they walk the same tiles and give the
  // same bits.
  int wide_per_cu = 0;
  int wrc = seg_per_cu(ii, p.wg, true, &wide_per_cu);
  if (wrc) return wrc;
  const bool wide = grid <= wide_per_cu * dev.cus;
  SegArgs a;
  a.x = x;
  a.offsets = offsets;
  a.nseg = nseg;
  a.out = out;
  a.carry_in = ws->carry_in;
  a.carry_out = ws->carry_out;
  a.tickets = ws->seg_tickets;
  a.words = ws->words;
  a.spin_limit = watchdog_spins();
  a.bar_groups = ((p.flags & RED_FLAG_XCD) && xcd_tree_fits(dev.nxcc)) ? (kBarrierXcd | (unsigned)dev.nxcc)
                                                            : barrier_groups(grid);
  a.form = (p.flags & RED_FLAG_SEG_WORKGROUP) ? kSegWorkgroup
           : (p.flags & RED_FLAG_SEG_PIECES)  ? kSegWavePieces
           : (p.flags & RED_FLAG_SEG_RUNS)    ? kSegWaveRuns
                                              : kSegAuto;
  if (a.form == kSegWaveRuns && p.ipt > 4)
    return set_error(RED_EINVAL, "segmented: the reduce-by-key form takes at most 4 loads per thread");
  a.grid = grid;
  a.wg = p.wg;
  void* args[] = {&a};
  const bool nt = (p.flags & RED_FLAG_NONTEMPORAL) != 0;
  const bool coop = barrier && (p.flags & RED_FLAG_PLAIN_LAUNCH) == 0;
  const int slot = timer_begin(s);
  int rc = launch(seg_table().k[fix][nt ? 1 : 0][ii][wide ? 1 : 0], grid, p.wg, args, s, coop,
                  seg_lds_bytes(p.wg, runs_max_rows(p.ipt, wide)));
  if (rc == RED_OK && fix == kFixRelaunch) {
    // One wavefront per possible slice (the wavefront-slice count bounds the
    // workgroup-slice count).
    const int64_t waves = (int64_t)grid * (p.wg / kWave);
    const int fix_grid = (int)((waves + kFixupWG / kWave - 1) / (kFixupWG / kWave));
    rc = launch(reinterpret_cast<const void*>(&k_seg_fixup), fix_grid, kFixupWG, args, s, false);
  }
  timer_end(s, slot);
  return rc;
}

}  // namespace redsum
