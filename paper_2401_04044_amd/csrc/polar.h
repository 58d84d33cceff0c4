// Internal: the polar iteration of the remainder factorisation (polar.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include "polar_steps.h"

namespace ffsplit {

// Steps launched product by product (all of a fixed plan): a step that is not needed costs 3 launches (10 us), one in
// the queue 135 us at rank 512 instead of 65.  Flat spectra take 4 or 5 steps, i^-1/2 6.
inline int polar_launched(const PolarPlan& p) { return p.fixed ? p.max_steps : 6; }
constexpr int POLAR_SHARDS = 16, POLAR_SHARD_WORDS = 16;   // counters of the steps after those, 64 bytes apart

// `mats` matrices X [r8, dk] fp32 (r valid rows, d valid columns, the rest zero) one after the other at off_x,
// twice: the caller fills the first copies, zeroes the queue_words at off_queue, and finds the result in the copy that the
// state's parity names.
struct PolarWs {
  int mats, r, d, r8, rk, dk;
  int queue_words;
  int side, tri;   // tiles of the symmetric products: side x side, `tri` of a triangle
  int64_t nx;   // elements of one X
  size_t off_x, off_s, off_t, off_queue, off_share, off_rows, off_state, bytes;
};
PolarWs make_polar_ws(int mats, int r, int d);
// state: [mats] on the device, valid behind the launches
int launch_polar(const PolarWs& w, char* ws, const PolarState** state, hipStream_t st);
// moves every result to the first copy
int launch_polar_settle(const PolarWs& w, char* ws, const PolarState* state, hipStream_t st);

}  // namespace ffsplit
