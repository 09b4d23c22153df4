// Prints the library's default schedules: a line of input per question,
//   kind row_bytes phase rows owned runs terms values jobs bytes source identity fresh
// a line of output per answer,
//   tile_rows block_threads blocks_per_cu nontemporal unroll push_pack lds_window pair_rows
#include <cstdio>

#include "common.h"

int main() {
  int kind, rb, phase, values, identity, fresh;
  long long rows, owned, runs, terms, jobs, bytes, source;
  while (std::scanf("%d %d %d %lld %lld %lld %lld %d %lld %lld %lld %d %d", &kind, &rb, &phase, &rows, &owned, &runs, &terms,
                    &values, &jobs, &bytes, &source, &identity, &fresh) == 13) {
    hx::SchedFor w;
    w.phase = phase;
    w.rows = rows;
    w.owned = owned;
    w.runs = runs;
    w.terms = terms;
    w.values = values;
    w.jobs = jobs;
    w.bytes = bytes;
    w.source = source;
    w.identity = identity != 0;
    w.fresh = fresh != 0;
    const hx::Sched s = hx::default_sched(kind, rb, w);
    std::printf("%d %d %d %d %d %d %d %d\n", s.tile_rows, s.block_threads, s.blocks_per_cu, s.nontemporal, s.unroll,
                s.push_pack, s.lds_window, s.pair_rows);
  }
  return 0;
}
