// Internal: the polar iteration of the remainder factorisation (polar.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include "polar_steps.h"

namespace ffsplit {

// `mats` matrices X [r8, dk] fp32 (r valid rows, d valid columns, the rest zero) one after the other at off_x,
// twice: the caller fills the first copies and finds the result in the copy that the state's parity names.
struct PolarWs {
  int mats, r, d, r8, rk, dk;
  int side, tri;   // tiles of X X^T: side x side, `tri` of a triangle
  int64_t nx;   // elements of one X
  size_t off_x, off_s, off_t, off_share, off_rows, off_state, off_ended, bytes;
};
PolarWs make_polar_ws(int mats, int r, int d);
// state: [mats] on the device, valid behind the launches
int launch_polar(const PolarWs& w, char* ws, const PolarState** state, hipStream_t st);
// moves every result to the first copy
int launch_polar_settle(const PolarWs& w, char* ws, const PolarState* state, hipStream_t st);

}  // namespace ffsplit
