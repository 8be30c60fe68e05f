// Lane-level CPU emulation of the reduce-by-key form of the segmented batch
// (seg_wave_runs, seg_walk_runs, finish_piece and k_seg_fixup in
// paper_2004_05371_amd/csrc/segmented.hip) over whole launches.  The slice
// length, the tile's rows, the places in a tile buffer and their bounds come
// from csrc/seg_rules.h, which the kernel takes them from; the walk, the carry
// slots, the tickets and the three fix-ups are restated here, one wavefront at
// a time, with per-lane values as arrays of 64.
//
// Checked: every global access (value vectors that overlap the batch, offsets,
// results, carry slots and tickets below the wavefront count), every LDS
// access against the buffer of the rows in use (tile vectors and which vector
// each place holds, mask words, sums by rank and that a sum read was written
// for this part), each start inside its part, the carry slots (each written
// at most once per launch, each piece read written by this launch for this
// segment, in slices that follow one another), tickets that end at zero, every
// segment written exactly once with the exact integer sum of its values.
//
// -DMUTATION=k plants a mistake that the checks must catch: 1 no half tiles
// for tiles with too many starts, 2 the sum at rank j (not j + 1) taken for
// rank j, 3 a chunk's end taken for the part's end, 4 no mask for values
// outside the slice, 5 the mask words not cleared, 6 a piece count one short,
// 7 a padding vector after every 4 vectors of a tile, 8 no "none" in a slice's
// outgoing slot, 9 slices as long as the mean asks, however many wavefronts
// there are.
//
// Usage: seg_slices_emu E mean layout grid wg ipt wide fix shift seed
//   layout 0: equal lengths; 1: uniform on [0, 2 mean]; 2: half of the
//   segments empty; 3: stretches of length 1, of empties, and long ones;
//   4: one segment of nearly all values among empty ones and ones
//   fix 0: ticket, 1: grid barrier, 2: second kernel
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "../../paper_2004_05371_amd/csrc/seg_rules.h"

#ifndef MUTATION
#define MUTATION 0
#endif

namespace {
using namespace redsum;
constexpr int kWave = 64, kChunks = 4;
constexpr int64_t kMaxChunks = 65536;
enum Fix { kTicket, kBarrier, kRelaunch };

[[noreturn]] void fail(const char* what, long long a, long long b = 0, long long c = 0) {
  printf("{\"ok\": false, \"violation\": \"%s\", \"a\": %lld, \"b\": %lld, \"c\": %lld}\n", what, a, b, c);
  fflush(stdout);
  exit(1);
}

int64_t value(int64_t i) {
  uint64_t h = (uint64_t)i * 0x9E3779B97F4A7C15ull;
  h ^= h >> 29;
  h *= 0xBF58476D1CE4E5B9ull;
  h ^= h >> 32;
  return (int64_t)(h % 15) - 7;
}

int place_of(int i) { return MUTATION == 7 ? i + (i >> 2) : run_place(i); }

struct Slot {
  int64_t seg = 0, val = 0, np = 0;
  int launch = 0;  // that wrote it
};

struct Machine {
  int64_t E = 0, nseg = 0, W = 0;
  int shift = 0, fix = 0, launch = 0, max_rows = 0;
  std::vector<int64_t> off, out;
  std::vector<uint8_t> writes;
  std::vector<Slot> in, outgoing;  // carry_in, carry_out
  std::vector<int64_t> tickets;
  std::vector<int64_t> own;  // barrier: cut segment that slice w owns
  long long halves = 0, scanned = 0, plain = 0, late_chunks = 0, cut = 0;
  int rows_used = 0;
  int64_t max_tiles = 0;

  int64_t offset(int64_t i) {
    if (i < 0 || i > nseg) fail("offsets read out of bounds", i, nseg);
    return off[i];
  }
  void write(int64_t s, int64_t v) {
    if (s < 0 || s >= nseg) fail("out write out of bounds", s, nseg);
    out[s] = v;
    if (writes[s] < 255) ++writes[s];
  }
  Slot& slot(std::vector<Slot>& v, int64_t w) {
    if (w < 0 || w >= W || w >= kMaxChunks) fail("carry slot out of bounds", w, W);
    return v[w];
  }
  void put_slot(std::vector<Slot>& v, int64_t w, int64_t s, int64_t val, int64_t np) {
    Slot& c = slot(v, w);
    if (c.launch == launch && c.seg >= 0) fail("carry slot written twice", w, c.seg, s);
    c = Slot{s, val, np, launch};
  }
  int64_t combine(int64_t o, int64_t np, int64_t s) {
    int64_t v = 0;
    for (int64_t k = o; k < o + np; ++k) {
      const Slot& c = slot(k == o ? outgoing : in, k);
      if (c.launch != launch || c.seg != s) fail("piece of another segment or launch", k, c.seg, s);
      v += c.val;
    }
    return v;
  }
  void finish_piece(int64_t s, int64_t v, int64_t lo, int64_t hi, int64_t w, int64_t chunk) {
    const int64_t sa = offset(s), sb = offset(s + 1);
    if (sa >= lo && sb <= hi) {
      write(s, v);
      return;
    }
    ++cut;
    const int64_t o = sa / chunk;
    int64_t np = (sb - 1) / chunk - o + 1;
    if (np < 2) fail("a cut segment of one piece", s, o, np);
    if (MUTATION == 6) --np;
    put_slot(sa < lo ? in : outgoing, w, s, v, np);
    if (fix == kBarrier && sa >= lo) own[w] = s;
    if (fix == kTicket) {
      if (o < 0 || o >= W || o >= kMaxChunks) fail("ticket out of bounds", o);
      if (++tickets[o] == np) {
        write(s, combine(o, np, s));
        tickets[o] = 0;
      }
    }
  }
  void wave(int64_t w, int64_t chunk, int ROWS);
  void run_launch();
};

struct Entry {
  int64_t x, y;
};

int64_t first_at_or_after(Machine& b, int64_t pos) {
  int64_t L = 0, R = b.nseg;
  while (R - L > 2 * kWave) {
    const int64_t d = R - L;
    int c = 0;
    for (int l = 0; l < kWave; ++l) {
      const bool below = b.offset(L + (((int64_t)(l + 1) * d) >> 6)) < pos;
      if (below && c != l) fail("probes are not a prefix", l);
      c += below;
    }
    if (c == kWave) fail("the last probe lies below", L, R);
    R = L + (((int64_t)(c + 1) * d) >> 6);
    if (c > 0) L = L + (((int64_t)c * d) >> 6) + 1;
  }
  int c = 0;
  for (int64_t i = L; i < R && i < L + 2 * kWave; i += 2) {
    const int64_t x = b.offset(i), y = b.offset(i + 1);
    c += (x < pos) + (i + 1 < R && y < pos);
  }
  return L + c;
}

void Machine::wave(int64_t w, int64_t chunk, int ROWS) {
  const int64_t lo = std::min(w * chunk, E), hi = std::min(lo + chunk, E);
  const bool end_slice = E > 0 ? (lo < E && hi == E) : (w == 0);
  if (fix == kRelaunch && MUTATION != 8) put_slot(outgoing, w, -1, 0, 0);
  if (!(lo < hi || end_slice)) return;
  const int64_t vlo = (lo + shift) >> 2, vhi = (hi + shift + 3) >> 2;
  const int64_t T = (int64_t)kWave * ROWS;
  const int64_t ntiles = lo < hi ? (vhi - vlo + T - 1) / T : 0;
  max_tiles = std::max(max_tiles, ntiles);

  const int tile_size = run_tile_vectors(ROWS), max_sums = 2 * tile_size;  // 16-byte vectors, 8-byte sums
  if (tile_size > run_tile_vectors(max_rows)) fail("rows beyond the launch's buffer", ROWS, max_rows);
  std::vector<int64_t> tile(tile_size, -2);  // vector of the batch at each place (-2: none, or a sum)
  std::vector<int64_t> sums(max_sums, 0), sums_part(max_sums, -1);
  unsigned mask[kWave] = {};
  long long part_no = 0;

  int64_t q = first_at_or_after(*this, lo);
  if (offset(q) < lo || (q > 0 && offset(q - 1) >= lo)) fail("search", q, lo);
  auto entry = [&](int64_t at, int c, int l) {
    const int64_t i = at + std::min<int64_t>(c * kWave + l, nseg - at - 1);
    return Entry{offset(i), offset(i + 1)};
  };
  const int ahead = (int)std::min<int64_t>(kChunks, 1 + (4 * T * nseg / std::max<int64_t>(E, 1) + kWave / 2) / kWave);
  Entry ent[kChunks][kWave];
  auto load_entries = [&]() {
    for (int c = 0; c < ahead; ++c)
      for (int l = 0; l < kWave; ++l) ent[c][l] = entry(q, c, l);
  };
  if (ntiles > 0) load_entries();
  int64_t so = ntiles > 0 && q > 0 && (q == nseg || ent[0][0].x > lo) ? q - 1 : -1;
  bool is_cut = so >= 0;
  int64_t Cs = 0, cl[kWave] = {};
  bool spread = false;

  std::vector<int64_t> xr;  // the runs read from the tile: lane l's from l RL on, per part
  auto read_runs = [&](int N, int i0, int64_t t) {
    for (int l = 0; l < kWave; ++l)
      for (int j = 0; j < N; ++j) {
        const int place = place_of(i0) + place_of(N * l) + j;
        const int64_t v = std::min(vlo + t * T + i0 + N * l + j, vhi - 1);
        if (place < 0 || place >= tile_size) fail("tile read out of bounds", place, tile_size);
        if (tile[place] != v) fail("tile place holds another vector", place, tile[place], v);
        for (int k = 0; k < 4; ++k) {
          const int64_t i = 4 * v - shift + k;
          xr.push_back((i >= 0 && i < E) ? value(i) : (int64_t)1 << 40);
        }
      }
  };
  auto part = [&](int RL, const int64_t* x, int64_t f0) -> bool {
    const int64_t f1 = f0 + (int64_t)kWave * RL, fe = std::min(f1, hi);
    if (f0 >= hi) return true;
    int R = 0;
    int64_t cnt = 0, o_first = 0, s_last = 0;
    auto take = [&](const Entry* e, int64_t s0, int* rank) -> bool {
      int n = 0, in_chunk = 0, last = -1;
      for (int l = 0; l < kWave; ++l) {
        const bool is_in = e[l].x < fe && l < nseg - s0, full = is_in && e[l].y != e[l].x;
        rank[l] = full ? R + in_chunk : is_in ? -2 : -1;
        if (full) {
          const int64_t p = e[l].x - f0;
          if (p < 0 || p >= (int64_t)kWave * RL) fail("start outside its part", e[l].x, f0, f1);
          if (mask[p / RL] & (1u << (p % RL))) fail("two starts at one value", e[l].x);
          mask[p / RL] |= 1u << (p % RL);
          if (R + in_chunk == 0) o_first = e[l].x;
          last = l;
          ++in_chunk;
        }
        n += is_in;
      }
      if (in_chunk) s_last = s0 + last;
      R += in_chunk;
      cnt += n;
      return n == kWave;
    };
    int rank[kChunks][kWave];
    bool more = true;
    for (int c = 0; c < kChunks; ++c) {
      std::fill(rank[c], rank[c] + kWave, -1);
      if (more && c < ahead) more = take(ent[c], q + c * kWave, rank[c]);
    }
    const int R_ahead = R;
    const int64_t cnt_ahead = cnt;
    if (MUTATION == 3) more = false;
    while (more) {
      const int64_t s0 = q + cnt;
      for (int c = 0; c < 4 && more; ++c) {
        Entry e[kWave];
        int unused[kWave];
        for (int l = 0; l < kWave; ++l) e[l] = entry(s0, c, l);
        ++late_chunks;
        more = take(e, s0 + c * kWave, unused);
      }
    }
    unsigned word[kWave];
    for (int l = 0; l < kWave; ++l) {
      word[l] = mask[l];
      if (MUTATION != 5) mask[l] = 0;
    }
    if (RL == 4 * ROWS && R > run_max_starts(ROWS) && MUTATION != 1) return false;
    const int64_t q0 = q;
    q += cnt;
    load_entries();
    ++part_no;
    std::vector<int64_t> xv(x, x + (size_t)kWave * RL);
    if (MUTATION != 4 && (f0 < lo || f1 > hi))
      for (int i = 0; i < kWave * RL; ++i)
        if (!(f0 + i >= lo && f0 + i < hi)) xv[i] = 0;
    if (R == 0) {
      if (cnt) fail("empty segments in a part without a start", q0, cnt);
      for (int l = 0; l < kWave; ++l)
        for (int i = 0; i < RL; ++i) cl[l] += xv[(size_t)l * RL + i];
      spread = true;
      ++plain;
      return true;
    }
    ++scanned;
    if (spread) {
      for (int l = 0; l < kWave; ++l) Cs += cl[l], cl[l] = 0;
      spread = false;
    }
    int64_t acc[kWave];
    int r0[kWave], f[kWave], scan = 0;
    for (int l = 0; l < kWave; ++l) {
      r0[l] = scan;
      scan += __builtin_popcount(word[l]);
    }
    if (scan != R) fail("mask words do not hold the starts", scan, R);
    for (int l = 0; l < kWave; ++l) {
      acc[l] = l == 0 ? Cs : 0;
      int at = r0[l];
      for (int i = 0; i < RL; ++i) {
        if (word[l] & (1u << i)) {
          if (at < 0 || at >= max_sums) fail("sum out of bounds", at, max_sums);
          tile[at / 2] = -2;
          sums[at] = acc[l];
          sums_part[at++] = part_no;
          acc[l] = 0;
        }
        acc[l] += xv[(size_t)l * RL + i];
      }
      f[l] = word[l] != 0;
    }
    auto step = [&](auto src_of) {
      int64_t pv[kWave];
      int pf[kWave];
      for (int l = 0; l < kWave; ++l) {
        const int s = src_of(l);
        pv[l] = s >= 0 ? acc[s] : 0;
        pf[l] = s >= 0 ? f[s] : 0;
      }
      for (int l = 0; l < kWave; ++l) {
        acc[l] = f[l] ? acc[l] : pv[l] + acc[l];
        f[l] |= pf[l];
      }
    };
    for (int k : {1, 2, 4, 8}) step([k](int l) { return (l % 16) >= k ? l - k : -1; });
    step([](int l) { return ((l / 16) & 1) ? (l / 16) * 16 - 1 : -1; });
    step([](int l) { return (l / 16) >= 2 ? 31 : -1; });
    for (int l = 0; l < kWave; ++l)
      if (word[l]) sums[r0[l]] += l == 0 ? 0 : acc[l - 1];
    Cs = acc[kWave - 1];
    auto sum_at = [&](int r) {
      if (r < 0 || r >= max_sums) fail("sum read out of bounds", r, max_sums);
      if (sums_part[r] != part_no) fail("sum read was not written for this part", r);
      return sums[r];
    };
    if (so >= 0) {
      if (o_first != offset(so + 1)) fail("the open segment does not end at the first start", so, o_first);
      if (is_cut != (offset(so) < lo)) fail("cut flag wrong", so);
      if (!is_cut)
        write(so, sum_at(0));
      else
        finish_piece(so, sum_at(0), lo, hi, w, chunk);
    }
    so = s_last;
    is_cut = false;
    auto put = [&](int64_t s, int rk) {
      if (rk == -2)
        write(s, 0);
      else if (rk >= 0 && rk + 1 < R)
        write(s, sum_at(MUTATION == 2 ? rk : rk + 1));
    };
    for (int c = 0; c < ahead; ++c)
      for (int l = 0; l < kWave; ++l)
        if (rank[c][l] != -1) put(q0 + c * kWave + l, rank[c][l]);
    int Rc = R_ahead;
    for (int64_t d = cnt_ahead; d < cnt; d += kWave) {
      int in_chunk = 0;
      for (int l = 0; l < kWave; ++l) {
        const Entry e = entry(q0 + d, 0, l);
        const bool is_in = e.x < fe && l < nseg - (q0 + d), full = is_in && e.y != e.x;
        if (is_in) put(q0 + d + l, full ? Rc + in_chunk : -2);
        in_chunk += full;
      }
      Rc += in_chunk;
    }
    return true;
  };

  const bool dense = 4 * E < 9 * nseg;
  for (int64_t t = 0; t < ntiles; ++t) {
    for (int i = 0; i < kWave * ROWS; ++i) {
      const int64_t v = std::min(vlo + t * T + i, vhi - 1);
      const int64_t e = 4 * v - shift;
      if (e + 3 < 0 || e >= E) fail("vector load out of bounds", v, e, E);
      const int place = place_of(i / kWave * kWave) + place_of(i % kWave);
      if (place < 0 || place >= tile_size) fail("tile write out of bounds", place, tile_size);
      tile[place] = v;
    }
    const int64_t e0 = 4 * (vlo + t * T) - shift;
    bool done = false;
    xr.clear();
    if (!dense) {
      read_runs(ROWS, 0, t);
      done = part(4 * ROWS, xr.data(), e0);
    }
    if (!done) {
      ++halves;
      xr.clear();
      read_runs(ROWS / 2, 0, t);
      read_runs(ROWS / 2, kWave * ROWS / 2, t);
      part(2 * ROWS, xr.data(), e0);
      part(2 * ROWS, xr.data() + kWave * 2 * ROWS, e0 + kWave * 2 * ROWS);
    }
  }
  if (so >= 0) {
    if (spread)
      for (int l = 0; l < kWave; ++l) Cs += cl[l];
    finish_piece(so, Cs, lo, hi, w, chunk);
  }
  if (end_slice)
    for (int64_t i = q; i < nseg; ++i) write(i, 0);
}

void Machine::run_launch() {
  ++launch;
  out.assign(nseg, 0);
  writes.assign(nseg, 0);
  own.assign(W, -1);
  const int64_t chunk = MUTATION == 9 ? std::max<int64_t>(kRunsMinChunk, E / nseg / 16 / 64 * 64) : runs_slice(E, nseg, W, shift);
  rows_used = runs_rows(max_rows, chunk);
  // The wavefronts in an order of their own per launch.
  std::vector<int64_t> order(W);
  std::iota(order.begin(), order.end(), 0);
  uint64_t st = 88172645463325252ull + launch;
  for (int64_t i = W - 1; i > 0; --i) {
    st ^= st << 13, st ^= st >> 7, st ^= st << 17;
    std::swap(order[i], order[st % (uint64_t)(i + 1)]);
  }
  for (int64_t w : order) wave(w, chunk, rows_used);
  if (fix == kBarrier)
    for (int64_t w : order)
      if (own[w] >= 0) {
        const int64_t o = offset(own[w]) / chunk, np = (offset(own[w] + 1) - 1) / chunk - o + 1;
        write(own[w], combine(o, np, own[w]));
      }
  if (fix == kRelaunch)
    for (int64_t w : order) {
      const Slot c = slot(outgoing, w);
      if (c.launch != launch) fail("outgoing slot not written by this launch", w);
      if (c.seg >= 0) write(c.seg, combine(w, c.np, c.seg));
    }
  for (int64_t t : tickets)
    if (t) fail("a ticket is left", t);
  int64_t e = 0;
  for (int64_t s = 0; s < nseg; ++s) {
    int64_t want = 0;
    for (; e < off[s + 1]; ++e) want += value(e);
    if (writes[s] != 1) fail("segment not written exactly once", s, writes[s]);
    if (out[s] != want) fail("wrong segment sum", s, out[s], want);
  }
}
}  // namespace

int main(int argc, char** argv) {
  if (argc != 11) return 2;
  Machine m;
  m.E = atoll(argv[1]);
  const int64_t mean = std::max<int64_t>(1, atoll(argv[2]));
  const int layout = atoi(argv[3]), grid = atoi(argv[4]), wg = atoi(argv[5]), ipt = atoi(argv[6]), wide = atoi(argv[7]);
  m.fix = atoi(argv[8]);
  m.shift = atoi(argv[9]);
  m.W = (int64_t)grid * (wg / kWave);
  m.max_rows = runs_max_rows(ipt, wide != 0);
  m.in.resize(kMaxChunks);
  m.outgoing.resize(kMaxChunks);
  m.tickets.assign(kMaxChunks, 0);
  uint64_t st = strtoull(argv[10], nullptr, 10) * 0x9E3779B97F4A7C15ull + 12345;
  auto rnd = [&]() {
    st ^= st << 13;
    st ^= st >> 7;
    st ^= st << 17;
    return st;
  };
  m.off.push_back(0);
  for (int64_t e = 0, k = 0; e < m.E || (layout >= 2 && k < 300); ++k) {
    int64_t len = mean;
    if (layout == 1) len = (int64_t)(rnd() % (uint64_t)(2 * mean + 1));
    if (layout == 2) len = (rnd() & 1) ? 0 : (int64_t)(rnd() % (uint64_t)(4 * mean + 1));
    if (layout == 3) {
      const int64_t phase = (k / 700) % 4;
      len = phase == 0 ? 1 : phase == 1 ? 0 : phase == 2 ? (int64_t)(rnd() % 9) : (int64_t)(rnd() % (uint64_t)(8 * mean));
    }
    if (layout == 4) len = k == 90 ? std::max<int64_t>(1, m.E - 300) : (int64_t)(k & 1);
    e = std::min(m.E, e + len);
    m.off.push_back(e);
  }
  if (m.off.size() == 1) m.off.push_back(m.E);
  m.nseg = (int64_t)m.off.size() - 1;
  // Twice: the second launch finds what the first left in the slots.
  m.run_launch();
  m.run_launch();
  printf("{\"ok\": true, \"segments\": %lld, \"rows\": %d, \"max_tiles\": %lld, \"halves\": %lld, \"scanned\": %lld, \"plain\": %lld, "
         "\"late_chunks\": %lld, \"cut\": %lld}\n",
         (long long)m.nseg, m.rows_used, (long long)m.max_tiles, m.halves, m.scanned, m.plain, m.late_chunks, m.cut);
  return 0;
}
