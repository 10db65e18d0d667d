// row_window.h -- the rows whose entry counts the range-query planner holds
// in LDS (internal; plain arithmetic, also compiled for the host).
//
// The counts of kCountRows rows from row wb on, row r in slot r mod kCountRows.
// Once the flight has come far enough, one wave loads the kCountLoad rows
// behind the window over the slots of the window's first kCountLoad rows, and
// the window moves on.  The load has no barrier of its own: another wave may
// still be reading, after the last barrier, the rows of the batch just taken,
// up to kRunSteps rows before the flight's, so the load waits until those
// rows, too, lie past the slots that it overwrites.
#pragma once

namespace fmdp {

constexpr int kRunSteps = 16;                          // most steps of a batch
constexpr int kCountRows = 128, kCountLoad = 64;

constexpr int count_slot(int row) { return row & (kCountRows - 1); }

// Rows wb + kCountRows .. wb + kCountRows + kCountLoad - 1 are to be loaded
// before the batch whose first row is `row`.
constexpr bool count_load_due(int wb, int row) { return row - wb >= kCountLoad + kRunSteps; }

static_assert(2 * kCountLoad == kCountRows, "a load replaces half the window");
// a batch that just misses the load still ends inside the window, and the
// batches before the barrier that shows a load's rows do not reach them
static_assert(kCountLoad + 3 * kRunSteps <= kCountRows, "the window covers the batches until the next load");

}  // namespace fmdp
