// What a call sets up before its first kernel that computes: the plan in the workspace, the rows of its rollouts
// and the arrays that start at zero (SetupArgs), as device functions: in a launch of their own
// (launch_setup), by workgroups of the fused path's prepare_kernel or by one of a launch of logits rows.
// Every launch costs about 4.7 us however little it does; as separate launches the upload, the fills and the
// row expansion were 6 of the 19 launches of a small fused call (two rollouts of 128 rows,
// V = 4,096: 112 -> 105 us).  A plan that fits the argument block (up to about 90 rollouts) is read by
// every workgroup from there, block 0 writing it to the workspace; a larger one is uploaded first
// and read from the workspace.
#pragma once
#include <cstring>

#include "device_utils.h"
#include "plan_device.h"

namespace adwin {

constexpr int kUploadChunk = 3072;   // bytes per launch (the argument block stays below 4 KiB)
struct SetupBlob {
  int n16 = 0;
  uint4 data[kUploadChunk / 16];
  bool take(const std::vector<unsigned char>& blob) {        // false: too large
    if (blob.size() > (size_t)kUploadChunk) return false;
    n16 = (int)(blob.size() / 16);
    memcpy(data, blob.data(), blob.size());
    return true;
  }
};

inline unsigned setup_blocks(const SetupArgs& a, int threads) {
  int64_t most = a.n_pad > 1 ? a.n_pad : 1;
  for (int z = 0; z < a.n_zero; ++z) most = a.zero_n[z] > most ? a.zero_n[z] : most;
  const int64_t blocks = (most + threads - 1) / threads;
  return (unsigned)(blocks < 1024 ? blocks : 1024);
}

// Workgroup `block` of `blocks`; `plan`: the plan's bytes, in the arguments (blob) or in the workspace.
__device__ __forceinline__ void setup_body(const SetupArgs& a, const SetupBlob* blob, const unsigned char* plan,
                                           int block, int blocks, int threads) {
  if (blob && block == 0 && (int)threadIdx.x < blob->n16) ((uint4*)a.plan)[threadIdx.x] = blob->data[threadIdx.x];
  const int64_t* offsets = (const int64_t*)plan;
  const int64_t* comp_off = (const int64_t*)(plan + a.o_comp_off);
  const int64_t first = (int64_t)block * threads + threadIdx.x, step = (int64_t)blocks * threads;
  for (int64_t r = first; r < a.n_pad; r += step) {
    const int64_t rr = r < a.n_rows ? r : a.n_rows - 1;
    const int i = last_le<int64_t>(comp_off, a.B + 1, rr);
    a.row_idx[r] = (int32_t)(offsets[i] + (rr - comp_off[i]));
    a.row_seq[r] = i;
  }
  for (int z = 0; z < a.n_zero; ++z)
    for (int64_t q = first; q < a.zero_n[z]; q += step) a.zero[z][q] = 0u;
}

// The packed positions of computed rows [row0, row0 + n) into `table`, from the plan itself: for a launch that
// also writes row_idx.  n <= blockDim.x.
__device__ __forceinline__ void plan_rows(const SetupArgs& a, const unsigned char* plan, int64_t row0, int n, int32_t* table) {
  const int64_t* offsets = (const int64_t*)plan;
  const int64_t* comp_off = (const int64_t*)(plan + a.o_comp_off);
  const int64_t first = row0 + (threadIdx.x & ~63u), last = a.n_rows - 1;
  int i = wave_last_le(comp_off, a.B + 1, first < last ? first : last);      // of the wave's first row
  if ((int)threadIdx.x < n) {
    int64_t r = row0 + threadIdx.x;
    if (r > last) r = last;                          // padding repeats the last computed row
    while (comp_off[i + 1] <= r) ++i;                // comp_off[B] = n_rows
    table[threadIdx.x] = (int32_t)(offsets[i] + (r - comp_off[i]));
  }
  __syncthreads();
}

}  // namespace adwin
