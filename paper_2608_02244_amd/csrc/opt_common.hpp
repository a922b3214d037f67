// Launch descriptor of the exact-optimum search kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fsched.h"

namespace fs {

constexpr int OPT_MAX_JOBS = 8;
constexpr int OPT_LEN_LIMIT = 255;   // every length <= 255 (one byte of progress)
constexpr int OPT_ARR_LIMIT = 4095;  // every arrival <= 4095 (12-bit key field)

struct OptArgs {
  int64_t n_inst;
  int32_t n;
  int32_t B;          // effective capacity (n when unlimited)
  int32_t alpha;      // INT32_MAX = infinite
  int64_t M;          // 0 = no KV budget
  const int32_t* arrival;
  const int32_t* prompt;
  const int32_t* output;
  int64_t* T;         // in: ISJL makespan (incumbent) or marker; out: optimum
  int32_t* start;     // in: ISJL schedule; out: an optimal schedule (nullable)
  // Scratch for the searches that one launch leaves to the next: OPT_LISTS lists
  // of n_inst instance indices, OPT_COUNTERS counters (per list its length and
  // the claim counter of the launch that takes it) and the second search pass's
  // memo (OPT_FB_WAVES regions of OPT_FB_MEMO_ENTRIES 16-byte entries).  Null
  // lists: one search launch over the batch, and a capped search reports
  // FSCHED_T_INTERNAL.
  int32_t* lists;
  int32_t* counters;
  uint32_t* fb_memo;
  // Set by launch_opt: the list that the search takes (null: the whole batch),
  // and the list of the searches that reach the first pass's step cap, which the
  // second pass solves again with its large memo.
  int32_t* todo_list;
  int32_t* todo_count;
  int32_t* fb_list;
  int32_t* fb_count;
};

constexpr int OPT_LISTS = 3;
constexpr int OPT_COUNTERS = 2 * OPT_LISTS;
constexpr int OPT_FB_WAVES = 16;                // waves of the second pass
constexpr int OPT_FB_MEMO_ENTRIES = 1 << 20;    // memo entries per wave (16 MiB)
constexpr int OPT_FB_GUARD = 1 << 28;           // DFS pushes per search in the second pass

// The two-worker tables, the search and its second pass (a.T and a.start hold
// the incumbent).
hipError_t launch_opt(const OptArgs& a, hipStream_t s);

}  // namespace fs
