// Workspace of the chunked fast-weight kernels (fmm_fastweight.hip).
#pragma once

#include <stddef.h>

#include <algorithm>

#include "fmm_launch.h"

namespace fmm {

constexpr int kFwChunk = 16;  // positions of a chunk: one matrix-core tile

// Floats one chunk of a slice takes: the row arrays of 16 rows of d floats
// each (p(k), p(q), X, Y; the backward adds U and Dn), the state W and the sum
// z at the chunk's start, and the rows' scalars (two inverse sums; the
// backward adds the same state for G and ds and one sum).
inline size_t fw_chunk_floats(int d, bool bwd) {
  const size_t rows = (size_t)kFwChunk * d, state = (size_t)d * d + d;
  return bwd ? 6 * rows + 2 * state + 3 * kFwChunk + 4 : 5 * rows + state + 2 * kFwChunk;
}
inline long long fw_chunks(int N) { return ((long long)N + kFwChunk - 1) / kFwChunk; }

// The forward runs in passes of at most `bytes` of chunks (whole slices, or,
// where one slice alone has more, ranges of its chunks with W and z carried from
// one range to the next): up to kFwPassBytes, or what is to be had.  A position
// takes 5 d + d (d + 1) / 16 + 2 floats (378 at d = 32, 1674 at d = 128).
constexpr size_t kFwPassBytes = (size_t)1 << 30;
struct FwPlan {
  long long slices;  // slices per pass
  long long chunks;  // chunks of a slice per pass
};
inline FwPlan fw_plan(long long bh, int N, int d, size_t bytes) {
  const long long most = std::max<long long>(
      1, (long long)(bytes / (fw_chunk_floats(d, false) * sizeof(float))));
  const long long nc = fw_chunks(N);
  FwPlan p;
  p.chunks = std::min(nc, most);
  p.slices = nc > most ? 1 : std::min(bh, most / nc);
  return p;
}
inline size_t fw_forward_bytes(long long bh, int N, int d, size_t bytes) {
  const FwPlan p = fw_plan(bh, N, d, bytes);
  // (the carried state of one slice at the end)
  return ((size_t)(p.slices * p.chunks) * fw_chunk_floats(d, false) + (size_t)d * d + d) *
         sizeof(float);
}
// The backward keeps every chunk.
inline unsigned __int128 fw_backward_bytes(long long bh, int N, int d) {
  return (unsigned __int128)bh * (unsigned long long)fw_chunks(N) * fw_chunk_floats(d, true) *
         sizeof(float);
}

}  // namespace fmm
