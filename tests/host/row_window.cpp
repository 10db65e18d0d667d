// The range-query planner's window of row counts, by the kernel's order of
// barriers, reads and loads: which rows a load may overwrite while another
// wave, on the same side of the barrier, still reads the batch just taken.
// Prints "<reads of a row not held> <loads over a row being read> <loads>".
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "row_window.h"

using namespace fmdp;

struct Window {
    int held[kCountRows], since[kCountRows];           // row in each slot, barrier interval of its load
    int wb = 0, now = 0;                               // first row; barriers passed
    std::vector<int> reading;                          // rows read in this interval by waves other than the loading one
    long missing = 0, overwritten = 0, loads = 0;

    void load(int first) {
        ++loads;
        for (int r = first; r < first + kCountLoad; ++r) {
            for (int q : reading) overwritten += count_slot(q) == count_slot(r) && q != r;
            held[count_slot(r)] = r;
            since[count_slot(r)] = now;
        }
    }
    void start(int row) {
        wb = row;
        load(wb);
        load(wb + kCountLoad);
        barrier();
    }
    void barrier() {
        ++now;
        reading.clear();
    }
    void read(int row) {                               // a wave reads it before or after a load of this interval
        missing += held[count_slot(row)] != row || since[count_slot(row)] >= now;
        reading.push_back(row);
    }
};

int main(int argc, char **argv) {
    const bool planted = argc > 1 && std::atoi(argv[1]) != 0;        // shift a batch too early
    auto due = [&](int wb, int row) { return planted ? row - wb >= kCountLoad : count_load_due(wb, row); };
    std::mt19937 rng(7);
    Window total;
    for (int flight = 0; flight < 400; ++flight) {
        Window w;
        int row = 1 + (int)(rng() % 200);
        w.start(row);
        auto shift = [&]() {
            if (due(w.wb, row)) {
                w.load(w.wb + kCountRows);
                w.wb += kCountLoad;
            }
        };
        const int longest = flight % 3 == 0 ? kRunSteps : 1 + (int)(rng() % kRunSteps);
        while (row < 4000) {
            shift();
            if (rng() % 8 == 0) {                      // a single step: its row before the barrier
                w.read(row);
                w.barrier();
                row += 1;
                continue;
            }
            for (bool more = true; more && row < 4000; more = rng() % 6 != 0) {      // batches of a run
                const int nb = longest, f = rng() % 4 ? nb : (int)(rng() % (nb + 1));
                for (int i = 0; i < nb; ++i) w.read(row + i);
                w.barrier();
                for (int i = 0; i < f; ++i) w.read(row + i);         // the taken steps' records
                row += f;
                if (f < nb) break;
                shift();
            }
            w.barrier();
        }
        total.missing += w.missing;
        total.overwritten += w.overwritten;
        total.loads += w.loads;
    }
    std::printf("%ld %ld %ld\n", total.missing, total.overwritten, total.loads);
    return 0;
}
