// Rules by which the C ABI picks a kernel or the shape of a launch, as plain
// functions of sizes: they can be evaluated without a GPU.
#pragma once

#include <stdint.h>

namespace janus {

// ---- page demand: one block for all of it, or three launches -----------------

constexpr int PD_ROWS = 4;          // rows in flight per block
constexpr int RUN_THREADS = 1024;   // the one block, and the list and run kernel's
constexpr int PD_SMALL_STEPS = 2;

// Steps that one block takes over the ids, one after another: PD_ROWS rows at
// a time, four ids of each row per thread.
constexpr int64_t pd_steps(int64_t total_q, int64_t k)
{
    return ((total_q + PD_ROWS - 1) / PD_ROWS) * ((k + 4 * RUN_THREADS - 1) / (4 * RUN_THREADS));
}

// A step is a chain of dependent loads, about 2 us however few ids it has, and
// many rows would be walked by one block alone.  Measured, one block against
// three launches: 8 rows of 2048 ids 12.9 against 13 us (and two launches
// less for the host), 12 of 1024 14.9 against 12.9, 64 of 256 46 against 14,
// 256 of 64 162 against 18.  (The one block has a word of the bitmap per thread.)
constexpr bool pd_one_block(int64_t total_q, int64_t k, int nwords)
{
    return total_q > 0 && nwords > 0 && nwords <= RUN_THREADS && pd_steps(total_q, k) <= PD_SMALL_STEPS;
}

// ---- decode indexer: blocks of a batch ----------------------------------------

// First block of session s, whose keys start at ctx_start, in chunks of 2^shift
// keys: each session has as many blocks as chunks, or one more, and no block
// needs the sessions before its own.
constexpr int rows_first(int ctx_start, int s, int shift) { return (ctx_start >> shift) + s; }

} // namespace janus
