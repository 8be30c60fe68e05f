// Lane-level CPU emulation of the segmented batch's reduce-by-key walk
// (seg_wave_runs in paper_2004_05371_amd/csrc/segmented.hip): mask words per
// lane run, sums by rank in the tile's own LDS, chunks of 64 offsets, half
// tiles where a tile holds more starts than sums fit.  Test infrastructure only: nothing of the
// library is linked or included.  Its slices and rows are its own (slices down
// to 64 values, 2 ipt rows); seg_slices_emu.cpp runs whole launches with those
// of the kernel.
//
// Per-lane values are arrays of 64.  Checked: every global access (value
// vectors that overlap the batch, offsets[0 .. nseg], out[0 .. nseg)), every
// LDS access (tile vectors and which vector each place holds, mask words,
// sums by rank and that a sum read was written for this part), each start
// inside its part, every segment written exactly once with the exact integer
// sum of its values.  Cut segments are summed here by segment id.
//
// -DMUTATION=k plants a mistake that the checks must catch: 1 no half
// tiles for tiles with too many starts, 2 the sum at rank j (not j + 1) taken for
// rank j, 3 a chunk's end taken for the part's end, 4 no mask for values
// outside the slice, 5 the mask words not cleared.
//
// Usage: seg_keys_emu E mean layout grid wg ipt shift seed
//   layout 0: equal lengths; 1: uniform on [0, 2 mean]; 2: half of the
//   segments empty; 3: stretches of length 1, of empties, and long ones
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <map>
#include <vector>

#ifndef MUTATION
#define MUTATION 0
#endif

namespace {
constexpr int kWave = 64, kChunks = 4;

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

struct Batch {
  int64_t E = 0, nseg = 0;
  int shift = 0;
  std::vector<int64_t> off, out;
  std::vector<uint8_t> writes;
  std::map<int64_t, int64_t> cut;  // sums of pieces of cut segments
  long long dense_tiles = 0, scanned = 0, plain = 0, late_chunks = 0;
  int64_t offset(int64_t i) {
    if (i < 0 || i > nseg) fail("offsets read out of bounds", i, nseg);
    return off[i];
  }
  void write(int64_t s, int64_t v) {
    if (s < 0 || s >= nseg) fail("out write out of bounds", s, nseg);
    out[s] = v;
    if (writes[s] < 255) ++writes[s];
  }
};

struct Entry {
  int64_t x, y;
};

int64_t first_at_or_after(Batch& b, int64_t pos) {
  int64_t L = 0, R = b.nseg;
  while (R - L > kWave) {
    const int64_t d = R - L;
    int c = 0;
    bool prefix = true;
    for (int l = 0; l < kWave; ++l) {
      const bool below = b.offset(L + (((int64_t)(l + 1) * d) >> 6)) < pos;
      if (below && !prefix) fail("probes are not a prefix", l);
      prefix = below;
      c += below;
    }
    if (c == kWave) fail("the last probe lies below", L, R);
    R = L + (((int64_t)(c + 1) * d) >> 6);
    if (c > 0) L = L + (((int64_t)c * d) >> 6) + 1;
  }
  int c = 0;
  for (int l = 0; l < kWave; ++l) c += L + l < R && b.offset(L + l) < pos;
  return L + c;
}

void finish_piece(Batch& b, int64_t s, int64_t sa, int64_t sb, int64_t v, int64_t lo, int64_t hi) {
  if (sb <= sa || sa != b.offset(s) || sb != b.offset(s + 1)) fail("segment bounds wrong", s, sa, sb);
  if (sa >= lo && sb <= hi)
    b.write(s, v);
  else
    b.cut[s] += v;
}

void wave(Batch& b, int IPT, int64_t w, int64_t W) {
  const int64_t nseg = b.nseg, E = b.offset(nseg);
  const int64_t chunk = std::max<int64_t>(64, (((E + W - 1) / W) + 63) & ~(int64_t)63);
  const int64_t lo = std::min(w * chunk, E), hi = std::min(lo + chunk, E);
  const bool end_slice = E > 0 ? (lo < E && hi == E) : (w == 0);
  if (!(lo < hi || end_slice)) return;
  const int64_t vlo = (lo + b.shift) >> 2, vhi = (hi + b.shift + 3) >> 2;
  const int ROWS = 2 * IPT;
  const int64_t T = (int64_t)kWave * ROWS;
  const int64_t ntiles = lo < hi ? (vhi - vlo + T - 1) / T : 0;
  auto place_of = [&](int i) { return i + (i >> 3); };

  std::vector<int64_t> tile_vec(kWave * 9, -2);  // vector of the batch at each place (-2: none, or a sum)
  const int max_sums = kWave * 9 * 2;            // 8-byte sums in the tile's LDS
  std::vector<int64_t> sums(max_sums, 0), sums_part(max_sums, -1);
  unsigned mask[kWave] = {};
  long long part_no = 0;

  int64_t q = first_at_or_after(b, lo);
  for (int64_t k = 0; k < 1; ++k)
    if (b.offset(q) < lo || (q > 0 && b.offset(q - 1) >= lo)) fail("search", q, lo);
  int64_t so = -1;
  if (q > 0 && b.offset(q) > lo) so = q - 1;
  bool cut = so >= 0;
  int64_t Cs = 0;
  int64_t cl[kWave] = {};
  bool spread = false;
  // Past the last segment the last one's entry again; take() tells by the count.
  auto entry = [&](int64_t at, int c, int l) {
    const int64_t i = at + std::min<int64_t>(c * kWave + l, nseg - at - 1);
    return Entry{b.offset(i), b.offset(i + 1)};
  };
  const int ahead = (int)std::min<int64_t>(kChunks, 1 + (4 * T * nseg / std::max<int64_t>(E, 1) + kWave / 2) / kWave);
  Entry ent[kChunks][kWave];
  auto load_entries = [&]() {
    for (int c = 0; c < ahead; ++c)
      for (int l = 0; l < kWave; ++l) ent[c][l] = entry(q, c, l);
  };
  if (ntiles > 0) load_entries();

  std::vector<int64_t> runs;  // values read from the tile: lane l's run from l RL on (per half)
  auto read_runs = [&](int N, int i0, int64_t t) {
    for (int l = 0; l < kWave; ++l)
      for (int j = 0; j < N; ++j) {
        const int place = place_of(i0) + place_of(N * l) + j;
        const int64_t v = std::min(vlo + t * T + i0 + N * l + j, vhi - 1);
        if (place < 0 || place >= kWave * 9) fail("tile read out of bounds", place);
        if (tile_vec[place] != v) fail("tile place holds another vector", place, tile_vec[place], v);
        for (int k = 0; k < 4; ++k) {
          const int64_t i = 4 * v - b.shift + k;
          runs.push_back((i >= 0 && i < E) ? value(i) : (int64_t)1 << 40);
        }
      }
  };
  auto part = [&](int RL, const int64_t* xr, int64_t f0) -> bool {
    const int64_t f1 = f0 + (int64_t)kWave * RL, fe = std::min(f1, hi);
    if (f0 >= hi) return true;
    int R = 0;
    int64_t cnt = 0, o_first = 0, s_last = 0;
    auto take = [&](const Entry* e, int64_t s0, int* rank) -> bool {
      int n = 0, in_chunk = 0, first = -1, last = -1;
      for (int l = 0; l < kWave; ++l) {
        const bool in = e[l].x < fe && l < nseg - s0, full = in && e[l].y != e[l].x;
        rank[l] = full ? R + in_chunk : in ? -2 : -1;
        if (full) {
          const int64_t p = e[l].x - f0;
          if (p < 0 || p >= (int64_t)kWave * RL) fail("start outside its part", e[l].x, f0, f1);
          if (mask[p / RL] & (1u << (p % RL))) fail("two starts at one value", e[l].x);
          mask[p / RL] |= 1u << (p % RL);
          if (first < 0) first = l;
          last = l;
          ++in_chunk;
        }
        n += in;
      }
      if (in_chunk) {
        if (R == 0) o_first = e[first].x;
        s_last = s0 + last;
        R += in_chunk;
      }
      cnt += n;
      return n == kWave;
    };
    int rank[kChunks][kWave];
    bool more = true;
    for (int c = 0; c < kChunks; ++c) {
      for (int l = 0; l < kWave; ++l) rank[c][l] = -1;
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
        ++b.late_chunks;
        more = take(e, s0 + c * kWave, unused);
      }
    }
    unsigned word[kWave];
    for (int l = 0; l < kWave; ++l) {
      word[l] = mask[l];
      if (MUTATION != 5) mask[l] = 0;
    }
    if (RL == 4 * ROWS && R > 2 * kWave * ROWS && MUTATION != 1) return false;
    const int64_t q0 = q;
    q += cnt;
    load_entries();
    ++part_no;
    std::vector<int64_t> xv(xr, xr + (size_t)kWave * RL);
    if (MUTATION != 4 && (f0 < lo || f1 > hi))
      for (int l = 0; l < kWave; ++l)
        for (int i = 0; i < RL; ++i) {
          const int64_t p = f0 + (int64_t)RL * l + i;
          if (!(p >= lo && p < hi)) xv[(size_t)l * RL + i] = 0;
        }
    if (R == 0) {
      for (int l = 0; l < kWave; ++l)
        for (int i = 0; i < RL; ++i) cl[l] += xv[(size_t)l * RL + i];
      spread = true;
      ++b.plain;
      return true;
    }
    ++b.scanned;
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
          if (at < 0 || at >= 2 * kWave * ROWS) fail("sum out of bounds", at);
          tile_vec[at / 2] = -2;
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
      if (r < 0 || r >= max_sums) fail("sum read out of bounds", r);
      if (sums_part[r] != part_no) fail("sum read was not written for this part", r);
      return sums[r];
    };
    if (so >= 0) {
      if (o_first != b.offset(so + 1)) fail("the open segment does not end at the first start", so, o_first);
      if (cut != (b.offset(so) < lo)) fail("cut flag wrong", so);
      if (!cut)
        b.write(so, sum_at(0));
      else
        finish_piece(b, so, b.offset(so), b.offset(so + 1), sum_at(0), lo, hi);
    }
    so = s_last;
    cut = false;
    auto put = [&](int64_t s, int rk) {
      if (rk == -2)
        b.write(s, 0);
      else if (rk >= 0 && rk + 1 < R)
        b.write(s, sum_at(MUTATION == 2 ? rk : rk + 1));
    };
    for (int c = 0; c < ahead; ++c)
      for (int l = 0; l < kWave; ++l)
        if (rank[c][l] != -1) put(q0 + c * kWave + l, rank[c][l]);
    int Rc = R_ahead;
    for (int64_t d = cnt_ahead; d < cnt; d += kWave) {
      int in_chunk = 0;
      for (int l = 0; l < kWave; ++l) {
        const Entry e = entry(q0 + d, 0, l);
        const bool in = e.x < fe && l < nseg - (q0 + d), full = in && e.y != e.x;
        if (in) put(q0 + d + l, full ? Rc + in_chunk : -2);
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
      const int64_t e = 4 * v - b.shift;
      if (e + 3 < 0 || e >= E) fail("vector load out of bounds", v, e, E);
      const int place = place_of(i / kWave * kWave) + place_of(i % kWave);
      if (place < 0 || place >= kWave * 9) fail("tile write out of bounds", place);
      tile_vec[place] = v;
    }
    const int64_t e0 = 4 * (vlo + t * T) - b.shift;
    bool done = false;
    runs.clear();
    if (!dense) {
      read_runs(ROWS, 0, t);
      done = part(4 * ROWS, runs.data(), e0);
    }
    if (!done) {
      ++b.dense_tiles;
      runs.clear();
      read_runs(IPT, 0, t);
      read_runs(IPT, kWave * IPT, t);
      part(2 * ROWS, runs.data(), e0);
      part(2 * ROWS, runs.data() + kWave * 2 * ROWS, e0 + kWave * 2 * ROWS);
    }
  }
  if (so >= 0) {
    if (spread)
      for (int l = 0; l < kWave; ++l) Cs += cl[l];
    finish_piece(b, so, b.offset(so), b.offset(so + 1), Cs, lo, hi);
  }
  if (end_slice)
    for (int64_t i = q; i < nseg; ++i) b.write(i, 0);
}
}  // namespace

int main(int argc, char** argv) {
  if (argc != 9) return 2;
  Batch b;
  b.E = atoll(argv[1]);
  const int64_t mean = std::max<int64_t>(1, atoll(argv[2]));
  const int layout = atoi(argv[3]), grid = atoi(argv[4]), wg = atoi(argv[5]), ipt = atoi(argv[6]);
  b.shift = atoi(argv[7]);
  uint64_t st = strtoull(argv[8], nullptr, 10) * 0x9E3779B97F4A7C15ull + 12345;
  auto rnd = [&]() {
    st ^= st << 13;
    st ^= st >> 7;
    st ^= st << 17;
    return st;
  };
  b.off.push_back(0);
  for (int64_t e = 0, k = 0; e < b.E || (layout >= 2 && k < 300); ++k) {
    int64_t len = mean;
    if (layout == 1) len = (int64_t)(rnd() % (uint64_t)(2 * mean + 1));
    if (layout == 2) len = (rnd() & 1) ? 0 : (int64_t)(rnd() % (uint64_t)(4 * mean + 1));
    if (layout == 3) {
      const int64_t phase = (k / 700) % 4;
      len = phase == 0 ? 1 : phase == 1 ? 0 : phase == 2 ? (int64_t)(rnd() % 9) : (int64_t)(rnd() % (uint64_t)(8 * mean));
    }
    e = std::min(b.E, e + len);
    b.off.push_back(e);
  }
  if (b.off.size() == 1) b.off.push_back(b.E);
  b.nseg = (int64_t)b.off.size() - 1;
  b.out.assign(b.nseg, 0);
  b.writes.assign(b.nseg, 0);
  const int64_t W = (int64_t)grid * (wg / kWave);
  for (int64_t w = 0; w < W; ++w) wave(b, ipt, w, W);
  for (auto& c : b.cut) b.write(c.first, c.second);
  int64_t e = 0;
  for (int64_t s = 0; s < b.nseg; ++s) {
    int64_t want = 0;
    for (; e < b.off[s + 1]; ++e) want += value(e);
    if (b.writes[s] != 1) fail("segment not written exactly once", s, b.writes[s]);
    if (b.out[s] != want) fail("wrong segment sum", s, b.out[s], want);
  }
  printf("{\"ok\": true, \"segments\": %lld, \"dense_tiles\": %lld, \"scanned\": %lld, \"plain\": %lld, "
         "\"late_chunks\": %lld}\n",
         (long long)b.nseg, b.dense_tiles, b.scanned, b.plain, b.late_chunks);
  return 0;
}
