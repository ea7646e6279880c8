// First and last work of a step, done by the kernels that stand there anyway: the upload of the step's description and its
// rotary table beside the embedding, the approval walk inside the compaction.  Each was a launch of its own, and what a
// launch of this size costs is its place in the chain (about 5 us).  Both ends reach into the context's pinned host
// memory, which kernels read and write directly: the description is fetched from where the host wrote it, the verdict is
// stored where the host reads it.
#pragma once
#include <hip/hip_runtime.h>

#include "ded_kernels.h"

namespace ded {

// Angle pos * base^(-2i/hd), formed in fp64 so that long contexts do not lose phase accuracy; the rotation itself is applied in
// fp32 by the consumers.
__device__ inline float2 rope_entry(int pos, int i, double neg2_over_hd_log2base) {
  const double ang = (double)pos * exp2((double)i * neg2_over_hd_log2base);
  return make_float2((float)cos(ang), (float)sin(ang));
}

// Workgroup `block` (256 threads) of step_front_blocks(f): first the rotary table, then the copy of the description.
__device__ inline void step_front(const StepFront& f, int block) {
  const int rope_blocks = (f.rows * f.half + 255) / 256;
  if (block < rope_blocks) {
    const int idx = block * 256 + threadIdx.x;
    if (idx < f.rows * f.half) f.tab[idx] = rope_entry(f.pos[idx / f.half], idx % f.half, f.neg2_over_hd_log2base);
    return;
  }
  const int u = (block - rope_blocks) * 256 + threadIdx.x;
  if (u < f.units) f.meta_dst[u] = f.meta_src[u];
}
inline int step_front_blocks(const StepFront& f) { return (f.rows * f.half + 255) / 256 + (f.units + 255) / 256; }

// Approval walk of sequence b, by all threads of a workgroup.  Node i is approved iff every node v on the path root .. i (v !=
// root) carries the model's token of its parent; the end node is the deepest approved one, lowest index among equals.  Returns
// the path's length (its nodes are in sh.path), or 0 for every sequence if a real node of any of them has a non-finite logit:
// such a step has no verdict, nothing is compacted.  The trees are walked in LDS: through memory every step up costs a round
// trip (256 nodes: 22 us).
struct WalkShared {
  int32_t tok[256], par[256], am[256], path[256];  // (a tree has at most 256 nodes)
  int best, len;
};
__device__ inline int approval_walk(const ApprovalWalk& w, int b, WalkShared& sh) {
  const int n = w.seq_n[b], row0 = w.row0[b], tid = threadIdx.x, threads = blockDim.x;
  int bad = 0;
  for (int b2 = 0; b2 < w.batch; ++b2)
    for (int i = tid; i < w.seq_n[b2]; i += threads) bad |= w.row_flag[w.row0[b2] + i];
  for (int i = tid; i < n; i += threads) {
    sh.tok[i] = w.token[row0 + i];
    sh.par[i] = w.parent[row0 + i];
    sh.am[i] = w.amax[row0 + i];
  }
  if (tid == 0) sh.best = -1;
  if (__syncthreads_or(bad)) return 0;
  if (w.mode == 1) {  // a chain, as the caller has checked: its nodes in order
    for (int i = tid; i < n; i += threads) sh.path[i] = i;
    __syncthreads();
    return n;
  }
  for (int i = tid; i < n; i += threads) {
    int v = i, depth = 0;
    bool ok = true;
    for (int p = sh.par[v]; p >= 0 && ok; p = sh.par[v], ++depth) {
      ok = sh.tok[v] == sh.am[p];
      v = p;
    }
    if (ok) atomicMax(&sh.best, depth * 1024 + (1023 - i));
  }
  __syncthreads();
  if (tid == 0) {
    const int end = 1023 - (sh.best & 1023), len = (sh.best >> 10) + 1;
    for (int j = len - 1, v = end; j >= 0; --j, v = sh.par[v]) sh.path[j] = v;
    sh.len = len;
  }
  __syncthreads();
  return sh.len;
}
// the verdict, to the host: path, and the tokens of its nodes after the first, then the model's own at its end
__device__ inline void report_walk(const ApprovalWalk& w, int b, const WalkShared& sh, int len) {
  for (int j = threadIdx.x; j < len; j += blockDim.x) {
    w.out_path[(int64_t)b * w.stride + j] = sh.path[j];
    w.out_tok[(int64_t)b * w.stride + j] = j + 1 < len ? sh.tok[sh.path[j + 1]] : sh.am[sh.path[j]];
  }
  if (threadIdx.x == 0) {
    w.out_n[b] = len;
    w.out_flag[b] = len == 0;
  }
}

}  // namespace ded
