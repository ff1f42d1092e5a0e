// Backup and root correction, one workgroup per root.
//
//  * Backup (Eq. 1 / Alg. 1, final steps): a leaf's value is its discounted
//    return plus gamma^d max_a Q(leaf, a); the leaves of root action a0 are
//    the contiguous block [a0 A^(d-1), (a0+1) A^(d-1)) of the root's leaves
//    (blocks of leaf_blk leaves when a beam cut the tree: the surviving
//    leaves stay grouped by root action), so Q_d(a0) is a max-reduction over
//    that block.
//  * Correction (Eq. 3 with B of Eq. 6 or the exact gap of Lemma 3.2):
//    pi_o = argmax of the network at the root, the depth-1 Bellman errors
//    delta(a) = r_a + gamma V(s_1^a) - Q_0(a) (Prop. 3.6), d_o = |delta(pi_o)|,
//    d_e = mean of |delta(a)| over the other actions, B = pen_e d_e - pen_o d_o
//    (pen_e, pen_o fixed by A and d, computed on the host); every a != pi_o
//    loses c gamma^d B.
//  * Action: argmax of the returned vector, lowest index on ties (Eq. 4).
// Everything is FP32; max is exact, so the result does not depend on the
// reduction order.
//
// Bound by latency: a root's leaves are a few KB.  A workgroup of eight
// wavefronts, one per root action in turn, with the correction's operands
// fetched meanwhile, takes 8.4 us for one root of A = 18, d = 3 (5,832 leaves)
// where one wavefront took 36, and 11 us for 64 roots of 5,184 leaves where it
// took 54; roots with few leaves keep one wavefront (1,501 roots of depth 0
// 4.1 us, 8.2 before the correction's rows were read by an action a lane).
#include "bcts_internal.h"

namespace bcts {
namespace {

__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

constexpr int kMaxThreads = 512;
constexpr long long kWideLeaves = 512;        // leaves a root from which a workgroup is eight wavefronts

__global__ void __launch_bounds__(kMaxThreads)
backup_kernel(int n_roots, const RootInfo* __restrict__ roots, const float* __restrict__ V,
              const float* __restrict__ q0, LevelRet level_ret, float gamma, float corr_scale, int* __restrict__ out_action,
              float* __restrict__ out_q) {
  const int r = blockIdx.x;
  if (r >= n_roots) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const RootInfo& ri = roots[r];
  const int A = ri.A, d = ri.d;
  const bool corr = ri.corr;
  __shared__ float q[kMaxA], Q0[kMaxA], delta[kMaxA];

  // the correction's rows, an action a thread
  if (tid < A && (corr || d == 0)) {
    const float x = q0[(long long)r * kMaxA + tid];
    if (d == 0) q[tid] = x;
    if (corr) {
      const float* r1 = level_ret.ret[1] + ri.base[1];          // depth-1 returns = rewards
      const float* v1 = V + (ri.d1_item >= 0 ? ri.d1_item : ri.leaf_item);
      Q0[tid] = x;
      delta[tid] = fabsf(r1[tid] + gamma * v1[tid] - x);
    }
  }
  if (d > 0) {
    const long long blk = ri.leaf_blk;          // A^(d-1), fewer when a beam cut the tree
    const float* ret = level_ret.ret[d] + ri.base[d];
    const float* v = V + ri.leaf_item;
    const float gamma_d = ri.gamma_d;
    for (int a0 = tid >> 6; a0 < A; a0 += blockDim.x >> 6) {
      float m = -INFINITY;
#pragma unroll 4
      for (long long j = a0 * blk + lane; j < (a0 + 1) * blk; j += 64)
        m = fmaxf(m, ret[j] + gamma_d * v[j]);
      m = wave_max(m);
      if (lane == 0) q[a0] = m;
    }
  }
  __syncthreads();

  if (tid == 0) {
    if (corr) {
      int pi_o = 0;
      for (int a = 1; a < A; ++a)
        if (Q0[a] > Q0[pi_o]) pi_o = a;
      float d_o = 0.f, d_e = 0.f;
      for (int a = 0; a < A; ++a) {
        const float dl = delta[a];
        if (a == pi_o) d_o = dl; else d_e += dl;
      }
      d_e /= (float)(A - 1);
      const float B = ri.pen_e * d_e - ri.pen_o * d_o;
      const float shift = corr_scale * ri.gamma_d * B;
      for (int a = 0; a < A; ++a)
        if (a != pi_o) q[a] = q[a] - shift;
    }
    int best = 0;
    for (int a = 1; a < A; ++a)
      if (q[a] > q[best]) best = a;
    out_action[r] = best;
  }
  __syncthreads();
  for (int a = tid; a < ri.q_stride; a += blockDim.x)
    out_q[(long long)r * ri.q_stride + a] = a < A ? q[a] : -INFINITY;
}

}  // namespace

void launch_backup_correct(int n_roots, const RootInfo* roots, const float* V, const float* q0,
                           const LevelRet& level_ret, float gamma, float corr_scale,
                           long long leaves, int* out_action, float* out_q, hipStream_t s) {
  if (n_roots <= 0) return;
  hipLaunchKernelGGL(backup_kernel, dim3(n_roots), dim3(leaves >= kWideLeaves ? kMaxThreads : 64), 0, s, n_roots, roots, V, q0,
                     level_ret, gamma, corr_scale, out_action, out_q);
}

}  // namespace bcts
