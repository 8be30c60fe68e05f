// Prints the form (SegForm) that a batch takes under the default plan: the
// rules of csrc/seg_rules.h over the 64 segments that the kernel samples.
// Usage: seg_form_main FILE (nseg + 1 int64 offsets) THREADS
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "../../paper_2004_05371_amd/csrc/seg_rules.h"

using namespace redsum;

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  FILE* f = fopen(argv[1], "rb");
  if (!f) return 2;
  std::vector<int64_t> off;
  for (int64_t v; fread(&v, sizeof v, 1, f) == 1;) off.push_back(v);
  fclose(f);
  const int64_t nseg = (int64_t)off.size() - 1, E = off[nseg], threads = atoll(argv[2]);
  int form = long_form(E, nseg);
  if (short_batch(E, nseg, threads)) {
    form = kSegWaveRuns;
  } else if (E < kRunsRaggedLen * nseg) {
    auto at = [&](int lane) { return (lane * nseg) >> 6; };
    SegSample c{};
    for (int l = 0; l < 64; ++l) {
      const SampledSegment s = sampled_segment(E, nseg, off[at(l)], off[at(l) + 1], l < 63 ? off[at(l + 1)] : 0);
      c.n_short += s.is_short;
      c.n_short_filled += s.is_short && s.is_filled;
      c.n_filled += s.is_filled;
      c.n_joined += s.is_joined;
      c.n_long += s.is_long;
    }
    if (ragged_batch(E, nseg, c)) form = kSegWaveRuns;
  }
  printf("%d\n", form);
  return 0;
}
