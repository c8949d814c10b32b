// Reads launches "nq kmax per_query m n longest planes", one a line, and prints for each what the
// rules choose: kernel, bucketed, lanes per query, queries per wavefront (8192 resident).
#include <cstdio>

#include "launch_rule.h"

int main() {
  long long nq, m, n, longest;
  int kmax, per_query, planes;
  while (std::scanf("%lld %d %d %lld %lld %lld %d", &nq, &kmax, &per_query, &m, &n, &longest, &planes) == 7) {
    mknn::LaunchSize l;
    l.nq = nq;
    l.kmax = kmax;
    l.per_query = per_query != 0;
    l.m = m;
    l.n = n;
    l.longest = longest;
    const mknn::WaveShape w = mknn::wave_shape(l, 8192);
    static const char *const name[] = {"rows", "waves", "scan"};
    std::printf("%s %d %d %d\n", name[(int)mknn::walk_for(l)],
                nq >= mknn::wave_sort_min(l, planes != 0) ? 1 : 0, w.lanes, w.per_wave);
  }
  return 0;
}
