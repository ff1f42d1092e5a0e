// Batch-BFS over a learned forward model: the fully connected stand-in for a
// learned simulator of the paper's runtime study (Sec. 4.1: three hidden
// layers of width 100 fed a 100-dimensional state and a one-hot action).
//
// The model maps x = [s ; onehot(a)] through three ReLU layers of width 100
// to a linear output of 101 units (next state, then reward); a leaf state is
// valued by the linear head Q(s, .) = Wq s + bq.  All roots of one call share
// A and the depth, so child c of level k has parent c / A at level k - 1 and
// the leaves of root r, root action a0 form the contiguous block
// [(r A + a0) A^(d-1), (r A + a0 + 1) A^(d-1)).
//
// FP32 throughout, on the FP32 matrix cores: v_mfma_f32_16x16x4_f32 adds its
// four products to the accumulator as a chain of fused multiply-adds in K
// order (every bit of 1 M random results, subnormal operands among them,
// equals the chain), so a layer's sum -- bias, the action column, then k =
// 0..99 -- has the same bits here, in a scalar loop and on the host, and
// results do not depend on batching.  Without packed instructions the vector
// units reach half the matrix cores' 157 TFLOP/s.
//
// A layer is computed transposed, D[unit][child] = W[unit][k] X[k][child]:
// the weights are the A operand, the activations the B operand.  Row i of
// unit fragment f holds unit 16 f + 4 (i % 4) + i / 4, so lane group g's
// result register q is unit 16 f + 4 q + g, which is exactly the B operand of
// K step 4 f + q of the next layer: a wavefront's results feed its next
// layer from the registers they are in, in K order, with no data movement.
#include "bcts_internal.h"

namespace bcts {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kS = 100;          // state / hidden width
constexpr int kSteps = kS / 4;   // K steps of a layer
constexpr int kF = kMlpFrags;    // unit fragments of 16: 7, covering 112 units
constexpr int kG4 = kMlpSteps4;  // weight loads of 4 K steps: 7, the last 3 steps of padding unused

// One unit fragment's weights of a layer: 7 16-byte loads per lane.
__device__ __forceinline__ void load_frag(const float* __restrict__ W, int f, int lane, f32x4 (&w)[kG4]) {
#pragma unroll
  for (int j = 0; j < kG4; ++j) w[j] = reinterpret_cast<const f32x4*>(W)[(f * kG4 + j) * 64 + lane];
}

// max over the A actions of a child's head values: lane group g's registers
// hold actions 16 f + 4 q + g
__device__ __forceinline__ float head_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}

// ---- large levels ----------------------------------------------------------
// One workgroup per CU holds the weights of all four layers in LDS for the
// whole launch (160,400 bytes: fragments without their padding, see
// kMlpImage*) and its wavefronts loop over tiles of 16 C children, each
// keeping its children's activations in registers from the parent state to
// the head value; they never wait for one another.
//   ps    parent states [n / A][100] (the roots at level 1), pret their
//         returns (null at level 1: the root's return is 0)
//   gpow  gamma^(k-1), the discount of this level's reward
//   os    child states (null: not kept), oret child returns (null: not kept)
//   ov    max_a Q(child, a) (null: not needed)
//   oleaf return + gamma^d max_a Q (null: not a leaf level)
// Bound by the matrix cores.
// Measured on 64 roots at A = 10, depth 5 (7.1 M children): 19.75 ms a search
// with the layers as FMA loops on the vector units (29 TFLOP/s), 6.0 with the
// weights streamed from L2 (C = 4, one wavefront per SIMD), 4.9 with them in
// LDS (119 TFLOP/s of 154 that a large FP32 matrix product reaches; the
// padding of 100 units to 112 takes 11%); C = 3 or 12 wavefronts 5.0, 5.1.
template <int C, int NW>
__global__ void __launch_bounds__(64 * NW, NW / 4)
mlp_level_kernel(MlpDev m, long long n, const float* __restrict__ ps, const float* __restrict__ pret, float gpow,
                 float* __restrict__ os, float* __restrict__ oret, float* __restrict__ ov, float* __restrict__ oleaf,
                 float gamma_d) {
  __shared__ __attribute__((aligned(16))) float img[kMlpImage];
  for (int e = threadIdx.x; e < kMlpImage / 4; e += 64 * NW)
    reinterpret_cast<f32x4*>(img)[e] = reinterpret_cast<const f32x4*>(m.image)[e];
  __syncthreads();
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, A = m.A;
  const long long tiles = (n + 16 * C - 1) / (16 * C);
  for (long long tile = (long long)blockIdx.x * NW + (threadIdx.x >> 6); tile < tiles; tile += (long long)gridDim.x * NW) {
  const long long c0 = tile * (16 * C);
  long long child[C], par[C];
  const float* w1a[C];                 // the child's action column of layer 1
  float x[C][kF * 4];                  // activations: x[c][s] is unit 4 s + g of child r
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const long long at = c0 + 16 * c + r;
    child[c] = at < n ? at : n - 1;    // columns past n repeat the last child (computed, never stored)
    par[c] = child[c] / A;
    w1a[c] = m.w1a + (int)(child[c] - par[c] * A) * kMlpPad;
    const float* p = ps + par[c] * kS + g;
#pragma unroll
    for (int s = 0; s < kSteps; ++s) x[c][s] = p[4 * s];
  }
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    const float* W = img + l * kS * kS;
    const float* bias = img + kMlpImageBias + l * kS;
    float y[C][kF * 4];
    f32x4 col[2][C];                   // layer 1: the action columns, requested a fragment ahead
    auto fetch = [&](int f, int b) {
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) col[b][c][q] = w1a[c][16 * f + 4 * q + g];
    };
    if (l == 0) fetch(0, 0);
#pragma unroll
    for (int f = 0; f < kF; ++f) {
      // the fragment's weights: 6 loads of 4 K steps and one of the 25th; the
      // last fragment holds its 4 units only (5 in the output layer)
      const int row = f + 1 < kF ? 64 : l < 3 ? 16 : 20;
      const int slot = f + 1 < kF ? lane : l < 3 ? g * 4 + (r >> 2) : g * 5 + (r == 1 ? 4 : r >> 2);
      const float* wf = W + f * 16 * kS;
      f32x4 acc[C], w[2];
      w[0] = *reinterpret_cast<const f32x4*>(wf + slot * 4);
      f32x4 b;
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = bias[16 * f + 4 * q + g];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[c][q] = b[q] + (l == 0 ? col[f & 1][c][q] : 0.f);
      if (l == 0 && f + 1 < kF) fetch(f + 1, (f + 1) & 1);
#pragma unroll
      for (int j = 0; j < kG4; ++j) {
        if (j + 1 < kG4 - 1) w[(j + 1) & 1] = *reinterpret_cast<const f32x4*>(wf + ((j + 1) * row + slot) * 4);
        else if (j + 1 == kG4 - 1) w[(j + 1) & 1][0] = wf[(kG4 - 1) * row * 4 + slot];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (4 * j + t < kSteps)
#pragma unroll
            for (int c = 0; c < C; ++c)
              acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j & 1][t], x[c][4 * j + t], acc[c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) y[c][4 * f + q] = l < 3 ? fmaxf(acc[c][q], 0.f) : acc[c][q];
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int s = 0; s < kF * 4; ++s) x[c][s] = y[c][s];
  }
  // x: units 0..99 next state, 100 reward

  float ret[C];                        // valid in lane group 0, which holds unit 100
#pragma unroll
  for (int c = 0; c < C; ++c) {
    ret[c] = fmaf(gpow, x[c][kS / 4], pret ? pret[par[c]] : 0.f);
    const bool in = c0 + 16 * c + r < n;
    if (oret && g == 0 && in) oret[child[c]] = ret[c];
    if (os && in) {
      float* o = os + child[c] * kS + g;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) o[4 * s] = x[c][s];
    }
  }
  if (!ov && !oleaf) continue;
  float v[C];
#pragma unroll
  for (int c = 0; c < C; ++c) v[c] = -INFINITY;
  for (int f = 0; f * 16 < A; ++f) {
    f32x4 w[kG4], acc[C];
    load_frag(m.fq, f, lane, w);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float b = m.bqp[16 * f + 4 * q + g];
#pragma unroll
      for (int c = 0; c < C; ++c) acc[c][q] = b;
    }
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
      for (int c = 0; c < C; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s >> 2][s & 3], x[c][s], acc[c], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (16 * f + 4 * q + g < A) {
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = fmaxf(v[c], acc[c][q]);
      }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    v[c] = head_max(v[c]);
    if (g == 0 && c0 + 16 * c + r < n) {
      if (ov) ov[child[c]] = v[c];
      if (oleaf) oleaf[child[c]] = fmaf(gamma_d, v[c], ret[c]);
    }
  }
  }
}

// ---- small levels ----------------------------------------------------------
// One workgroup of 7 wavefronts takes 16 children at a time, wavefront f the
// units of fragment f, with that fragment's weights of all four layers in
// registers for the whole launch; the layers exchange activations through
// LDS.  A level of few children is bound by the serial chain of one child
// (four layers of 25 dependent matrix instructions), which this splits seven
// ways.
// With `m` > 1 levels a workgroup runs a whole sub-tree, from node blockIdx.x
// of level k - 1 down m levels (A^m <= 16 children at the last one), and only
// the last level's states and returns go to memory: a shallow tree takes a
// few launches instead of one per level.  One root at A = 2, depth 10: 142 us
// a search with a launch per level (13.6 us each), 57 us now.
constexpr int kSmallThreads = 64 * kF;
constexpr int kXR = 4 * kF * 4 + 4;    // LDS floats per child: [lane group][K step], padded

struct MlpSmall {
  long long n;                         // children of the (first) level, over all roots
  int levels;                          // levels of the sub-tree; 1: tiles of 16 children, any parents
  const float *ps, *pret;
  float gpow[4];                       // discount of each level's reward
  float *os, *oret;                    // last level
  float *ret1, *ov;                    // first level: returns and head values (null: not kept)
  float* oleaf;                        // last level
  float gamma_d;
};

__global__ void __launch_bounds__(kSmallThreads, 1) mlp_small_kernel(MlpDev m, MlpSmall a) {
  __shared__ __attribute__((aligned(16))) float xs[2][16 * kXR];
  __shared__ float rets[2][16];
  const int tid = threadIdx.x, lane = tid & 63, f = tid >> 6, r = lane & 15, g = lane >> 4, A = m.A;
  f32x4 w[4][kG4];
  load_frag(m.f1, f, lane, w[0]);
  load_frag(m.f2, f, lane, w[1]);
  load_frag(m.f3, f, lane, w[2]);
  load_frag(m.fo, f, lane, w[3]);
  f32x4 bias[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int u = 16 * f + 4 * q + g;
    bias[0][q] = m.b1[u];
    bias[1][q] = m.b2[u];
    bias[2][q] = m.b3[u];
    bias[3][q] = m.bo[u];
  }
  const long long tiles = a.levels > 1 ? a.n / A : (a.n + 15) / 16;
  for (long long t = blockIdx.x; t < tiles; t += gridDim.x) {
    long long first = a.levels > 1 ? t * A : t * 16;      // the tile's first child in its level
    int cnt = a.levels > 1 ? A : (int)(a.n - first < 16 ? a.n - first : 16);
    for (int lv = 0; lv < a.levels; ++lv, first *= A, cnt *= A) {
      const int rr = r < cnt ? r : cnt - 1;               // columns past the tile repeat its last child
      const long long child = first + rr, par = child / A;
      float x[kG4 * 4];
      float pret = 0.f;
      if (lv == 0) {
        const float* p = a.ps + par * kS + g;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) x[s] = p[4 * s];
        if (a.pret) pret = a.pret[par];
      } else {
        // the previous level's states are in xs[1], its returns in rets
#pragma unroll
        for (int j = 0; j < kG4; ++j)
          *reinterpret_cast<f32x4*>(&x[4 * j]) = *reinterpret_cast<const f32x4*>(&xs[1][(rr / A) * kXR + g * 4 * kF + 4 * j]);
        pret = rets[(lv - 1) & 1][rr / A];
      }
      const float* w1a = m.w1a + (int)(child - par * A) * kMlpPad;
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        f32x4 acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = bias[l][q] + (l == 0 ? w1a[16 * f + 4 * q + g] : 0.f);
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[l][s >> 2][s & 3], x[s], acc, 0, 0, 0);
        if (l < 3)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q] = fmaxf(acc[q], 0.f);
        // layers write xs[0], xs[1], xs[0], xs[1] in turn: a buffer is
        // written again only after the barrier that follows its last reads
        *reinterpret_cast<f32x4*>(&xs[l & 1][r * kXR + g * 4 * kF + 4 * f]) = acc;
        if (l == 3 && f == kF - 1 && g == 0) rets[lv & 1][r] = fmaf(a.gpow[lv], acc[1], pret);   // unit 100
        __syncthreads();
        if (l < 3) {
#pragma unroll
          for (int j = 0; j < kG4; ++j)
            *reinterpret_cast<f32x4*>(&x[4 * j]) = *reinterpret_cast<const f32x4*>(&xs[l & 1][r * kXR + g * 4 * kF + 4 * j]);
        }
      }
      const bool last = lv + 1 == a.levels;
      float* oret = last ? a.oret : nullptr;
      if (f == kF - 1 && lane < cnt) {
        if (oret) oret[first + lane] = rets[lv & 1][lane];
        if (lv == 0 && a.ret1) a.ret1[first + lane] = rets[lv & 1][lane];
      }
      if (last && a.os)
        for (int e = tid; e < cnt * kS; e += kSmallThreads) {
          const int c = e / kS, u = e - c * kS;
          a.os[first * kS + e] = xs[1][c * kXR + (u & 3) * 4 * kF + (u >> 2)];
        }
      float* ov = lv == 0 ? a.ov : nullptr;
      float* oleaf = last ? a.oleaf : nullptr;
      if (f == 0 && (ov || oleaf)) {                      // the head: wavefront 0
#pragma unroll
        for (int j = 0; j < kG4; ++j)
          *reinterpret_cast<f32x4*>(&x[4 * j]) = *reinterpret_cast<const f32x4*>(&xs[1][r * kXR + g * 4 * kF + 4 * j]);
        float v = -INFINITY;
        for (int h = 0; h * 16 < A; ++h) {
          f32x4 wq[kG4], acc;
          load_frag(m.fq, h, lane, wq);
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q] = m.bqp[16 * h + 4 * q + g];
#pragma unroll
          for (int s = 0; s < kSteps; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wq[s >> 2][s & 3], x[s], acc, 0, 0, 0);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (16 * h + 4 * q + g < A) v = fmaxf(v, acc[q]);
        }
        v = head_max(v);
        if (lane < cnt) {
          if (ov) ov[first + lane] = v;
          if (oleaf) oleaf[first + lane] = fmaf(a.gamma_d, v, rets[lv & 1][lane]);
        }
      }
      __syncthreads();     // xs and rets may be written again
    }
  }
}

// q_d[b] = max over leaf block b (block elements contiguous)
constexpr int kThreads = 256;
__global__ void __launch_bounds__(kThreads) mlp_blockmax_kernel(long long block, const float* __restrict__ leaf,
                                                                float* __restrict__ qd) {
  __shared__ float red[kThreads];
  const long long b = blockIdx.x;
  float v = -INFINITY;
  for (long long i = threadIdx.x; i < block; i += kThreads) v = fmaxf(v, leaf[b * block + i]);
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) qd[b] = red[0];
}

// Per root (one workgroup): the maxima of its leaf blocks (`leaf` given:
// `block` values per root action; else qd holds them), Q0 = Wq s + bq, then
// for d >= 1 the BCTS correction (Eq. 3 with B = pen_e d_e - pen_o d_o of Eq.
// 6 or Lemma 3.2): pi_o = argmax Q0 (lowest index), delta_a = r_a + gamma max
// Q(s1^a) - Q0_a from the level-1 returns and head values, d_o =
// |delta_pi_o|, d_e the mean of |delta_a| over a != pi_o (summed in index
// order); every a != pi_o moves by scale gamma^d B.  Output q [n][A] and the
// argmax action (lowest index).
__global__ void __launch_bounds__(kThreads) mlp_root_kernel(MlpDev m, int d, const float* __restrict__ states,
                                                            const float* __restrict__ ret1,
                                                            const float* __restrict__ v1,
                                                            const float* __restrict__ leaf, long long block,
                                                            const float* __restrict__ qd, float gamma, float gamma_d,
                                                            float pen_e, float pen_o, int corr, float scale,
                                                            int32_t* __restrict__ act, float* __restrict__ q) {
  __shared__ float q0s[kMaxA], dels[kMaxA], outs[kMaxA], st[kS], red[kMaxA][kThreads / 64];
  const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, A = m.A;
  if (tid < kS) st[tid] = states[(size_t)r * kS + tid];
  if (leaf) {
    const float* mine = leaf + (size_t)r * A * block;
    for (int a = 0; a < A; ++a) {
      float v = -INFINITY;
      for (long long i = tid; i < block; i += kThreads) v = fmaxf(v, mine[a * block + i]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
      if (lane == 0) red[a][tid >> 6] = v;
    }
  }
  __syncthreads();
  if (tid < A) {
    const f32x4* wr = reinterpret_cast<const f32x4*>(m.wq + (size_t)tid * kS);
    f32x4 w[kSteps];
#pragma unroll
    for (int k4 = 0; k4 < kSteps; ++k4) w[k4] = wr[k4];
    float acc = m.bq[tid];
#pragma unroll
    for (int k = 0; k < kS; ++k) acc = fmaf(w[k >> 2][k & 3], st[k], acc);
    q0s[tid] = acc;
    if (d >= 1 && corr) dels[tid] = fmaf(gamma, v1[(size_t)r * A + tid], ret1[(size_t)r * A + tid]) - acc;
    float v = acc;
    if (leaf) v = fmaxf(fmaxf(red[tid][0], red[tid][1]), fmaxf(red[tid][2], red[tid][3]));
    else if (d >= 1) v = qd[(size_t)r * A + tid];
    outs[tid] = v;
  }
  __syncthreads();
  if (tid == 0) {
#pragma clang fp contract(off)
    float o[kMaxA];
#pragma unroll
    for (int a = 0; a < kMaxA; ++a) o[a] = a < A ? outs[a] : 0.f;
    if (d >= 1 && corr) {
      float q0[kMaxA], dl[kMaxA];
#pragma unroll
      for (int a = 0; a < kMaxA; ++a) {
        q0[a] = a < A ? q0s[a] : 0.f;
        dl[a] = a < A ? fabsf(dels[a]) : 0.f;
      }
      int pi = 0;
      float top = q0[0], dobs = dl[0];
#pragma unroll
      for (int a = 1; a < kMaxA; ++a)
        if (a < A && q0[a] > top) {
          pi = a;
          top = q0[a];
          dobs = dl[a];
        }
      float se = 0.f;
#pragma unroll
      for (int a = 0; a < kMaxA; ++a)
        if (a < A && a != pi) se += dl[a];
      const float de = se / (float)(A - 1);
      // one rounding of pen_e d_e - pen_o d_o, and none of the others fused
      // (the host search does the same)
      const float shift = scale * gamma_d * fmaf(pen_e, de, -(pen_o * dobs));
#pragma unroll
      for (int a = 0; a < kMaxA; ++a)
        if (a != pi) o[a] -= shift;
    }
    int best = 0;
    float top = o[0];
#pragma unroll
    for (int a = 1; a < kMaxA; ++a)
      if (a < A && top < o[a]) {
        best = a;
        top = o[a];
      }
    act[r] = best;
#pragma unroll
    for (int a = 0; a < kMaxA; ++a)
      if (a < A) q[(size_t)r * A + a] = o[a];
  }
}

}  // namespace

void launch_mlp_level(const MlpDev& m, long long n, const float* ps, const float* pret, float gpow, float* os,
                      float* oret, float* ov, float* oleaf, float gamma_d, hipStream_t s) {
  if (n <= 0) return;
  if (n < kMlpLarge) {
    launch_mlp_levels(m, n, 1, ps, pret, &gpow, os, oret, nullptr, ov, oleaf, gamma_d, s);
    return;
  }
  // Below kMlpLarge the small kernel is faster (8,000 children: 28 us against
  // 63, which the LDS fill and one tile take; 32,760: 78 and 75; 65,530: 142
  // and 90; times of a depth-1 search).
  constexpr int C = 2, NW = 8;
  const long long groups = (n + 16LL * C * NW - 1) / (16LL * C * NW);
  hipLaunchKernelGGL((mlp_level_kernel<C, NW>), dim3((unsigned)(groups < 256 ? groups : 256)), dim3(64 * NW), 0, s, m,
                     n, ps, pret, gpow, os, oret, ov, oleaf, gamma_d);
}

void launch_mlp_levels(const MlpDev& m, long long n, int levels, const float* ps, const float* pret,
                       const float* gpow, float* os, float* oret, float* ret1, float* ov, float* oleaf, float gamma_d,
                       hipStream_t s) {
  if (n <= 0) return;
  MlpSmall a{};
  a.n = n;
  a.levels = levels;
  a.ps = ps;
  a.pret = pret;
  for (int i = 0; i < levels; ++i) a.gpow[i] = gpow[i];
  a.os = os;
  a.oret = oret;
  a.ret1 = ret1;
  a.ov = ov;
  a.oleaf = oleaf;
  a.gamma_d = gamma_d;
  const long long tiles = levels > 1 ? n / m.A : (n + 15) / 16;
  const unsigned grid = (unsigned)(tiles < 256 ? tiles : 256);   // one per CU, each looping over tiles
  hipLaunchKernelGGL(mlp_small_kernel, dim3(grid), dim3(kSmallThreads), 0, s, m, a);
}

void launch_mlp_blockmax(long long n_blocks, long long block, const float* leaf, float* qd, hipStream_t s) {
  if (n_blocks <= 0) return;
  hipLaunchKernelGGL(mlp_blockmax_kernel, dim3((unsigned)n_blocks), dim3(kThreads), 0, s, block, leaf, qd);
}

void launch_mlp_root(const MlpDev& m, int n, int d, const float* states, const float* ret1, const float* v1,
                     const float* leaf, long long block, const float* qd, float gamma, float gamma_d, float pen_e,
                     float pen_o, int corr, float scale, int32_t* act, float* q, hipStream_t s) {
  hipLaunchKernelGGL(mlp_root_kernel, dim3((unsigned)n), dim3(kThreads), 0, s, m, d, states, ret1, v1, leaf, block,
                     qd, gamma, gamma_d, pen_e, pen_o, corr, scale, act, q);
}

}  // namespace bcts
