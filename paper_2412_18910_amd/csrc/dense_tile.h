// Which activation tiles the waves of a prompt GEMM load: device code, and host code of the tests that count them.
#pragma once
#include <hip/hip_runtime.h>

namespace ae {

// The DM row-blocks of a workgroup are 2 * DM tiles of 1 KB a k-tile (hi, lo), each in an LDS slot of its own.  Wave w of NW fills slots
// w + NW * i; every wave loads as often as the others (loads are waited for by count), one too many fills the last slot again.
__host__ __device__ inline int dense_slot(int w, int i, int NW, int DM) {
  const int t = w + NW * i;
  return DM * 2 % NW == 0 || t < DM * 2 ? t : DM * 2 - 1;
}

// The tile that goes there, counted from row-block rb0: where DM does not divide the RB row-blocks of the buffer, slots behind its end
// repeat the last one (nothing of theirs is stored).
__host__ __device__ inline int dense_source(int slot, int rb0, int RB) {
  const int last = (RB - rb0) * 2 - 1;
  return slot < last ? slot : last;
}

}  // namespace ae
