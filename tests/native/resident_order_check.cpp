// Host check of the order of resident launches: random launches on random streams, queued at random times and
// running for random times, start when their stream's launch before them and all they wait for are over.  Prints, for
// `streams` from the command line, the most blocks that ran together, and the launches that waited for nobody.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "resident_order.hpp"

int main(int argc, char** argv) {
  const int cus = 256, streams = std::atoi(argv[1]), launches = 20000, most = argc > 2 ? std::atoi(argv[2]) : cus;
  std::mt19937 rng(7 + streams);
  struct Launch { double start, end; int blocks; };
  std::vector<Launch> all;
  std::vector<int> last(streams, -1);     // newest launch per stream
  dd::ResFlights<int, int> flights;       // events: launch numbers
  double now = 0.0;
  int free_runs = 0;
  std::exponential_distribution<double> gap(1.0), length(0.5);
  for (int i = 0; i < launches; ++i) {
    now += gap(rng) * (rng() % 16 ? 0.2 : 20.0);
    const int st = rng() % streams, blocks = 4 + (int)(rng() % (most - 3));
    double start = now;
    if (last[st] >= 0) start = std::max(start, all[last[st]].end);
    const double alone = start;
    const int counts = flights.admit(
        st, blocks, cus, [&](int e) { return all[e].end <= now && rng() % 4; },
        [&](int e) { start = std::max(start, all[e].end); }, [](int) {});
    free_runs += start == alone;
    all.push_back({start, start + length(rng), blocks});
    last[st] = i;
    flights.add(st, i, counts);
  }
  // the most blocks at once: at the start of some launch
  int worst = 0;
  for (size_t i = 0; i < all.size(); ++i) {
    int sum = 0;
    for (const Launch& l : all) sum += l.start <= all[i].start && all[i].start < l.end ? l.blocks : 0;
    worst = std::max(worst, sum);
  }
  std::printf("%d %d %d\n", worst, free_runs, launches);
  return 0;
}
