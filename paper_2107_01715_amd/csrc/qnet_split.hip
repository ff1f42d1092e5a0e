// The FP32 Q-network on the FP16 matrix cores: every operand as the sum of two
// FP16 values.
//
// An FP32 value v scaled into FP16's range is hi + lo / 2^11, hi = fp16(v), lo =
// fp16((v - hi) 2^11): 22 to 23 bits of the 24, and a product w x is w_hi x_hi +
// (w_hi x_lo + w_lo x_hi) / 2^11, each exact in FP32, summed in FP32.  Left out is
// w_lo x_lo (2^-22 of w x at most, of either sign).  The pixels of conv1 are
// whole numbers, exact in FP16: two products there.  A sum over K = 32 is one
// v_mfma_f32_16x16x32_f16 and one rounding where v_mfma_f32_16x16x4_f32 makes
// 32.  It rounds within, too, every 4 to 8 values, so long sums are cut: the
// small products have sums of their own, and K runs in slices summed from zero
// (conv2 4 steps a slice, conv3 3, fc1 14).  The sums' error then falls by more
// than the operands' rises.  Against 64 bits, of a root's largest |Q| over 1,024
// searches of A = 6, d = 3 with Kaiming-uniform weights: 2.9e-7 on average and
// 2.0e-6 at most, where the FP32 instruction has 6.5e-7 and 3.4e-6 (one sum for
// all products and no slices in the conv layers: 1.5 times the error, 3% faster).
// Of a stack's largest |Q| over 768 stacks: heavy-tailed weights (Student's t, 4
// degrees) 2.8e-7 and 6.0e-7, channels uneven by a normal of two bits 2.8e-7 and
// 6.0e-7.
//
// Time, 256 searches of A = 6, d = 3 (57,088 stacks): conv layers 2.3 ms where
// layer-by-layer kernels on v_mfma_f32_16x16x4_f32 took 5.86 (the FP32
// instruction alone 4.2 at the card's 154 TFLOP/s), fc1 0.56 (1.65).
//
// Scaling is by powers of two, exact, a power for every output channel and every
// row of weights (split_scales.cpp): a channel's outputs are held with what it can
// reach at most at 2^14 to 2^15, the next layer's weights on it divided by the
// same.  FP16's normal values end at 2^-14 and the low plane is held 2^11 times as
// large, so a value keeps its 22 bits down to 2^-29 of that bound (2^-17 with the
// low plane as it is; the median positive output of conv3 lies at 2^-15, since the
// bound grows with each layer).  conv1's planes share one sum, its low one is held
// as it is.  Weights of which the planes would hold too few bits run on the FP32
// instruction (qnet.hip).
#include "bcts_internal.h"
#include "qnet_groups.h"

namespace bcts {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) _Float16 h16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 h16x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

__device__ __forceinline__ void lds_barrier() { __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ void load_lds16(const unsigned char* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds(src, (void __attribute__((address_space(3)))*)dst, 16, 0, 0);
}

__device__ __forceinline__ f32x4 mma(h16x8 a, h16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// a, b, held times 2^11, as two FP16 pairs: hi = fp16(a / 2^11), lo = fp16(a -
// 2^11 hi), which is exact in FP32.  One instruction a value and plane, with
// its rounding to FP16.
__device__ __forceinline__ void split2(float a, float b, unsigned& hi, unsigned& lo) {
  const float down = 1.f / kSplitLow, up = -kSplitLow;
  __asm__("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel_hi:[0,0,0]" : "=v"(hi) : "v"(a), "s"(down));
  __asm__("v_fma_mixhi_f16 %0, %1, %2, 0 op_sel_hi:[0,0,0]" : "+v"(hi) : "v"(b), "s"(down));
  __asm__("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(hi), "s"(up), "v"(a));
  __asm__("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(lo) : "v"(hi), "s"(up), "v"(b));
}

// ---- conv1 -> conv2 -> conv3 --------------------------------------------
// A workgroup takes runs of siblings (stacks that share channels 0..2), NI at
// a time: conv1's sum over the shared channels stays in registers for the
// run, x1 and x2 in LDS, x3 leaves as fc1's operand rows.  Two barriers a turn:
// x1 complete (and the last turn's conv3 done with x2), x2 complete (and conv2
// done with x1).  Wavefronts split a
// layer as (4 / NF channel groups of NF fragments) x (2 NF row groups): the
// weights stream from L2, a wavefront's copy serving its row tiles of all NI
// stacks.  Bound by the weights' way through L1 and by issue: 24.6k clocks a
// stack where its matrix instructions take 9.3k.  Two workgroups of one stack on a CU
// (four wavefronts a SIMD) take 3.4 ms for 2.8, one channel fragment a wavefront 3.0.
//
// LDS: x1 [400] positions x 128 bytes (32 channels hi, lo), even columns of a
// row before odd ones so that a stride-2 window reads consecutive positions;
// x2 [81] x 256 bytes (64 hi, 64 lo).  16-byte chunk c of position p is at
// chunk c ^ (p & 7): consecutive positions start in different banks.
constexpr int kX1 = 400 * 128, kX2 = 81 * 256;

// keeps the compiler from computing what follows from v before this point
__device__ __forceinline__ int fresh(int v) {
  __asm__ volatile("" : "+v"(v));
  return v;
}

// 1 KB block `blk` of a layer's weights: 16 bytes at this lane's offset
__device__ __forceinline__ h16x8 ldw(const void* w, int blk, unsigned off) {
  return *reinterpret_cast<const h16x8*>(reinterpret_cast<const char*>(w) + blk * 1024 + off);
}

// One K step of a wavefront's tiles: w_lo x_hi and w_hi x_lo in sums of their
// own, 2^11 times as large as they count
template <int T, int NF>
__device__ __forceinline__ void step(f32x4 (&acc)[T][NF], f32x4 (&low)[T][NF], const h16x8 (&w)[NF][2],
                                     const h16x8 (&x)[T][2]) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int f = 0; f < NF; ++f) low[t][f] = mma(w[f][1], x[t][0], low[t][f]);
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int f = 0; f < NF; ++f) low[t][f] = mma(w[f][0], x[t][1], low[t][f]);
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[t][f] = mma(w[f][0], x[t][0], acc[t][f]);
}

// The end of a slice of K: its sums join the total, the next slice starts from zero
template <int T, int NF>
__device__ __forceinline__ void take(f32x4 (&tot)[T][NF], f32x4 (&acc)[T][NF], bool first) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      tot[t][f] = first ? acc[t][f] : tot[t][f] + acc[t][f];
      acc[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// ReLU(acc scale + bias) of a wavefront's row tiles, split: st(row, channel / 8,
// byte offset in the chunk, hi, lo) for each 8 (NF 2) or 4 (NF 1) channels
template <int NF, int M, int RG, int T, class St>
__device__ __forceinline__ void store_rows(const f32x4 (&acc)[T][NF], const f32x4 (&low)[T][NF], const float* __restrict__ scale,
                                           const float* __restrict__ bias, int ng, int rg, int r16, int g, St st) {
  // fragment f holds channels 32 (f / 2) + 8 g + 4 (f & 1) + 0..3
  constexpr int C = 4 * NF;
  const int f0 = ng * NF, ch = fresh(32 * (f0 >> 1) + 8 * g + 4 * (f0 & 1));
  float sc[C], b[C];
#pragma unroll
  for (int e = 0; e < C; ++e) {
    sc[e] = scale[ch + e];
    b[e] = bias[ch + e];
  }
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int m = (rg + RG * t) * 16 + r16;
    __attribute__((ext_vector_type(C / 2))) unsigned hi, lo;
#pragma unroll
    for (int e = 0; e < C; e += 2) {
      float v[2];
#pragma unroll
      for (int k = 0; k < 2; ++k)
        v[k] = fmaxf(fmaf(fmaf(low[t][(e + k) >> 2][(e + k) & 3], 1.f / kSplitLow, acc[t][(e + k) >> 2][(e + k) & 3]),
                          sc[e + k], b[e + k]), 0.f);
      unsigned h, l;
      split2(v[0], v[1], h, l);
      hi[e / 2] = h;
      lo[e / 2] = l;
    }
    if (m < M) st(m, ch >> 3, (ch & 7) * 2, hi, lo);
  }
}

template <int NI, int NF>
__global__ void __launch_bounds__(512) conv_split_kernel(SplitConvArgs a) {
  constexpr int NG = 4 / NF, RG = 8 / NG;
  // K steps of weights and pixels held: what fits the registers (256 a lane)
  constexpr int WD = NI == 1 ? 3 : 2, XD = NI == 1 ? 2 : 1;
  constexpr int M2 = NI * 81, T2 = ((M2 + 15) / 16 + RG - 1) / RG;       // row tiles per wavefront
  constexpr int M3 = NI * 49, T3 = ((M3 + 15) / 16 + RG - 1) / RG;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NI * (kX1 + kX2)];
  unsigned char* const x1 = lds;
  unsigned char* const x2 = lds + NI * kX1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, g = lane >> 4;
  const int ng = wave % NG, rg = wave / NG;
  for (long long u = blockIdx.x; u < a.units; u += gridDim.x) {
    const long long run = u / a.n_groups, gi = u - run * a.n_groups;     // runs past a group's end come last
    const int sub = (int)run * a.per_run;
    long long item = gi;                                  // chunk-relative first item
    int count = 1;
    if (a.groups) {
      const FusedGroup gr = a.groups[gi];
      item = gr.item0 - a.item_base;
      count = gr.count;
    }
    const int end = sub + a.per_run < count ? sub + a.per_run : count;
    if (sub >= end) continue;

    // conv1 over the shared channels: this wavefront's pixel tiles wave, wave + 8, ..
    int xo[4];
    unsigned off[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int p = (wave + 8 * t) * 16 + r16;
      const int y = (p < 400 ? p : 399) / 20, x = (p < 400 ? p : 399) % 20, q = y * 20 + (x >> 1) + 10 * (x & 1);
      off[t] = (y * 4 + g) * kFrame + x * 4;
      xo[t] = q * 128 + ((g ^ (q & 7)) << 4);
    }
    auto pixels = [&](const uint8_t* f, int t, int half) {
      const unsigned* q = reinterpret_cast<const unsigned*>(f + half * 4 * kFrame + off[t]);
      return make_uint2(q[0], q[1]);
    };
    auto operand = [](uint2 w) {                          // 8 pixels: 1024 + b is 0x6400 | b
      const h16x2 k = {(_Float16)-1024.f, (_Float16)-1024.f};
      const h16x2 p0 = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(0x64646464u, w.x, 0x04010400u)) + k;
      const h16x2 p1 = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(0x64646464u, w.x, 0x04030402u)) + k;
      const h16x2 p2 = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(0x64646464u, w.y, 0x04010400u)) + k;
      const h16x2 p3 = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(0x64646464u, w.y, 0x04030402u)) + k;
      return h16x8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
    };
    f32x4 part[4][2];
    {
      const ItemDesc& d = a.desc[item + sub];
      const unsigned lo16 = (unsigned)fresh(lane * 16);
      uint2 raw[6][4];
#pragma unroll
      for (int ks = 0; ks < 6; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t) raw[ks][t] = pixels(d.frame[ks >> 1], t, ks & 1);
#pragma unroll
      for (int t = 0; t < 4; ++t) part[t][0] = part[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 6; ++ks) {
        h16x8 w[2][2];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int pl = 0; pl < 2; ++pl) w[f][pl] = ldw(a.w[0], (ks * 2 + f) * 2 + pl, lo16);
        h16x8 x[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = operand(raw[ks][t]);
#pragma unroll
        for (int pl = 1; pl >= 0; --pl)
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int f = 0; f < 2; ++f) part[t][f] = mma(w[f][pl], x[t], part[t][f]);
      }
    }
    uint2 own[NI][2][4];
    auto load_own = [&](int s) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint8_t* f = a.desc[item + (s + i < end ? s + i : end - 1)].frame[3];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int t = 0; t < 4; ++t) own[i][h][t] = pixels(f, t, h);
      }
    };
    load_own(sub);

    for (int s = sub; s < end; s += NI) {
      // conv1: channel 3 on a copy of the shared sums
      {
        const unsigned lo16 = (unsigned)fresh(lane * 16);
        h16x8 w[2][2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) w[h][f][pl] = ldw(a.w[0], ((6 + h) * 2 + f) * 2 + pl, lo16);
        const int ch = fresh(8 * g);
        float sc[8], b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          sc[e] = a.scale[0][ch + e];
          b[e] = a.bias[0][ch + e];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          f32x4 acc[4][2];
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int f = 0; f < 2; ++f) acc[t][f] = part[t][f];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            h16x8 x[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) x[t] = operand(own[i][h][t]);
#pragma unroll
            for (int pl = 1; pl >= 0; --pl)
#pragma unroll
              for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int f = 0; f < 2; ++f) acc[t][f] = mma(w[h][f][pl], x[t], acc[t][f]);
          }
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            if (t == 3 && wave > 0) continue;             // 25 tiles
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = fmaxf(fmaf(acc[t][e >> 2][e & 3], sc[e], b[e]), 0.f);
            u32x4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              unsigned h, l;
              split2(v[2 * e], v[2 * e + 1], h, l);
              hi[e] = h;
              lo[e] = l;
            }
            const int o = i * kX1 + xo[t];
            *reinterpret_cast<u32x4*>(x1 + o) = hi;
            *reinterpret_cast<u32x4*>(x1 + (o ^ 64)) = lo;
          }
        }
      }
      lds_barrier();

      // conv2: 16 taps of 32 channels
      {
        int p0[T2], base[T2];
#pragma unroll
        for (int t = 0; t < T2; ++t) {
          int m = fresh((rg + RG * t) * 16 + r16);
          m = m < M2 ? m : M2 - 1;
          const int i = m / 81, q = m - i * 81;
          p0[t] = q / 9 * 40 + q % 9;
          base[t] = i * kX1;
        }
        f32x4 acc[T2][NF], low[T2][NF], tot[T2][NF];
#pragma unroll
        for (int t = 0; t < T2; ++t)
#pragma unroll
          for (int f = 0; f < NF; ++f) acc[t][f] = low[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
        unsigned wo = (ng * NF * 128 + lane) * 16 - 8192;
        h16x8 w[WD][NF][2];
        auto load_w = [&](int ks) {
          wo = (unsigned)fresh((int)wo + 8192);
#pragma unroll
          for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) w[ks % WD][f][pl] = ldw(a.w[1], f * 2 + pl, wo);
        };
        h16x8 x[XD][T2][2];
        auto load_x = [&](int ks) {
          const int kh = ks >> 2, kw = ks & 3, d = kh * 20 + (kw >> 1) + 10 * (kw & 1);
#pragma unroll
          for (int t = 0; t < T2; ++t) {
            const int p = p0[t] + d, o = base[t] + p * 128 + ((g ^ (p & 7)) << 4);
            x[ks % XD][t][0] = *reinterpret_cast<const h16x8*>(x1 + o);
            x[ks % XD][t][1] = *reinterpret_cast<const h16x8*>(x1 + (o ^ 64));
          }
        };
#pragma unroll
        for (int ks = 0; ks < WD - 1; ++ks) load_w(ks);
        if (XD > 1) load_x(0);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
          if (ks + WD - 1 < 16) load_w(ks + WD - 1);
          if (ks + XD - 1 < 16) load_x(ks + XD - 1);
          step<T2, NF>(acc, low, w[ks % WD], x[ks % XD]);
          if (ks % 4 == 3) take<T2, NF>(tot, acc, ks < 4);
          __builtin_amdgcn_sched_barrier(0);
        }
        store_rows<NF, M2, RG, T2>(tot, low, a.scale[1], a.bias[1], ng, rg, r16, g, [&](int m, int c8, int half, auto hi, auto lo) {
          const int i = m / 81, q = m - i * 81;
          unsigned char* o = x2 + i * kX2 + q * 256 + ((c8 ^ (q & 7)) << 4) + half;
          *reinterpret_cast<decltype(hi)*>(o) = hi;
          *reinterpret_cast<decltype(lo)*>(o + 128) = lo;
        });
      }
      lds_barrier();
      if (s + NI < end) load_own(s + NI);

      // conv3: 9 taps of 64 channels
      {
        int p0[T3], base[T3];
#pragma unroll
        for (int t = 0; t < T3; ++t) {
          int m = fresh((rg + RG * t) * 16 + r16);
          m = m < M3 ? m : M3 - 1;
          const int i = m / 49, q = m - i * 49;
          p0[t] = q / 7 * 9 + q % 7;
          base[t] = i * kX2;
        }
        f32x4 acc[T3][NF], low[T3][NF], tot[T3][NF];
#pragma unroll
        for (int t = 0; t < T3; ++t)
#pragma unroll
          for (int f = 0; f < NF; ++f) acc[t][f] = low[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
        unsigned wo = (ng * NF * 128 + lane) * 16 - 8192;
        h16x8 w[WD][NF][2];
        auto load_w = [&](int ks) {
          wo = (unsigned)fresh((int)wo + 8192);
#pragma unroll
          for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) w[ks % WD][f][pl] = ldw(a.w[2], f * 2 + pl, wo);
        };
        h16x8 x[XD][T3][2];
        auto load_x = [&](int ks) {
          const int tap = ks >> 1, d = tap / 3 * 9 + tap % 3;
#pragma unroll
          for (int t = 0; t < T3; ++t) {
            const int p = p0[t] + d, o = base[t] + p * 256 + (((4 * (ks & 1) + g) ^ (p & 7)) << 4);
            x[ks % XD][t][0] = *reinterpret_cast<const h16x8*>(x2 + o);
            x[ks % XD][t][1] = *reinterpret_cast<const h16x8*>(x2 + o + 128);
          }
        };
#pragma unroll
        for (int ks = 0; ks < WD - 1; ++ks) load_w(ks);
        if (XD > 1) load_x(0);
#pragma unroll
        for (int ks = 0; ks < 18; ++ks) {
          if (ks + WD - 1 < 18) load_w(ks + WD - 1);
          if (ks + XD - 1 < 18) load_x(ks + XD - 1);
          step<T3, NF>(acc, low, w[ks % WD], x[ks % XD]);
          if (ks % 3 == 2) take<T3, NF>(tot, acc, ks < 3);
          __builtin_amdgcn_sched_barrier(0);
        }
        store_rows<NF, M3, RG, T3>(tot, low, a.scale[2], a.bias[2], ng, rg, r16, g, [&](int m, int c8, int half, auto hi, auto lo) {
          const int i = m / 49, q = m - i * 49;
          if (s + i >= end) return;
          unsigned char* o = a.x3 + (item + s + i) * kSplitRow + (q * 2 + (c8 >> 2)) * 128 + (c8 & 3) * 16 + half;
          *reinterpret_cast<decltype(hi)*>(o) = hi;
          *reinterpret_cast<decltype(lo)*>(o + 64) = lo;
        });
      }
    }
  }
}

// ---- fc1 ----------------------------------------------------------------
// H = ReLU(X W^T scale + b) in FP32 from BM x BN tiles of (NWM x NWN)
// wavefronts.  X and W rows hold, per K stage of 32, 32 values hi and 32 lo: a
// stage of a row is one 128-byte line, copied straight to LDS, three stages in
// the ring.  K is summed in kFc1Split slices, each from zero, and the slices in
// order, whatever the tile: a row's bits do not depend on the batch.  SLICES:
// a workgroup per slice, its sums in part[slice][n][512] for the fc2 kernel.
template <int BM, int BN, int NWM, int NWN, bool SLICES>
__global__ void __launch_bounds__(64 * NWM * NWN)
fc1_split_kernel(long long n, const unsigned char* __restrict__ X, const unsigned char* __restrict__ W,
                 const float* __restrict__ scale, const float* __restrict__ bias, float* __restrict__ H,
                 float* __restrict__ part) {
  constexpr int T = 64 * NWM * NWN, SB = (BM + BN) * 128, PER = SB / (T * 16), D = 3;
  constexpr int FM = BM / NWM / 16, FN = BN / NWN / 16;
  constexpr int NST = kFc1K / 32, SS = NST / kFc1Split;
  static_assert(SB % (T * 16) == 0 && FN % 2 == 0 && NST % kFc1Split == 0, "tile shape");
  __shared__ __attribute__((aligned(1024))) unsigned char ring[D][SB];
  // the neuron tiles of a stack tile run on one XCD, close in time
  constexpr int NT = 512 / BN;
  const long long bid = blockIdx.x, mt = bid / (8 * NT) * 8 + bid % 8;
  const long long m0 = mt * BM;
  const int n0 = (int)(bid / 8 % NT) * BN;
  if (m0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, g = lane >> 4;
  const int wm = wave / NWN, wn = wave % NWN;

  // LDS slot ps = tid + j T holds row ps / 8, chunk (ps % 8) ^ (row & 7) of the stage
  const unsigned char* src[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int ps = tid + j * T, row = ps >> 3, c = (ps & 7) ^ (row & 7);
    const long long m = m0 + row < n ? m0 + row : n - 1;
    src[j] = row < BM ? X + m * kSplitRow + c * 16 : W + (long long)(n0 + row - BM) * kSplitRow + c * 16;
  }
  const int st0 = SLICES ? (int)blockIdx.y * SS : 0, st1 = SLICES ? st0 + SS : NST;
  auto issue = [&](int st) {
    unsigned char* base = ring[st % D] + wave * 1024;
#pragma unroll
    for (int j = 0; j < PER; ++j) load_lds16(src[j] + st * 128, base + j * T * 16);
  };
  f32x4 acc[FN][FM], low[FN][FM], tot[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = low[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  issue(st0);
  issue(st0 + 1);
  for (int z = st0; z < st1; z += SS) {
    for (int st = z; st < z + SS; ++st) {
      if (st + 1 < st1) __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
      else __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_barrier();
      if (st + 2 < st1) issue(st + 2);
      const unsigned char* Xs = ring[st % D];
      const unsigned char* Ws = Xs + BM * 128;
      auto ld = [&](const unsigned char* b, int row, int c) {
        return *reinterpret_cast<const h16x8*>(b + row * 128 + ((c ^ (row & 7)) << 4));
      };
      h16x8 x[FM][2];
#pragma unroll
      for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) x[j][pl] = ld(Xs, (wm * FM + j) * 16 + r16, 4 * pl + g);
#pragma unroll
      for (int i = 0; i < FN; ++i) {
        const h16x8 wh = ld(Ws, (wn * FN + i) * 16 + r16, g), wl = ld(Ws, (wn * FN + i) * 16 + r16, 4 + g);
#pragma unroll
        for (int j = 0; j < FM; ++j) low[i][j] = mma(wl, x[j][0], low[i][j]);
#pragma unroll
        for (int j = 0; j < FM; ++j) low[i][j] = mma(wh, x[j][1], low[i][j]);
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = mma(wh, x[j][0], acc[i][j]);
      }
    }
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[i][j][q] = fmaf(low[i][j][q], 1.f / kSplitLow, acc[i][j][q]);
        tot[i][j] = z == st0 ? acc[i][j] : tot[i][j] + acc[i][j];
        acc[i][j] = low[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  }
#pragma unroll
  for (int k = 0; k < FN / 2; ++k) {
    const int nb = n0 + wn * FN * 16 + 32 * k + 8 * g;
    float sc[8], b[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sc[e] = scale[nb + e];
      b[e] = bias[nb + e];
    }
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      const long long m = m0 + (wm * FM + j) * 16 + r16;
      if (m >= n) continue;
      float* o = SLICES ? part + ((long long)blockIdx.y * n + m) * 512 + nb : H + m * 512 + nb;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 v = tot[2 * k + h][j];
        if (!SLICES) {
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = fmaxf(fmaf(v[q], sc[4 * h + q], b[4 * h + q]), 0.f);
        }
        *reinterpret_cast<f32x4*>(o + 4 * h) = v;
      }
    }
  }
}

// ---- fc2 ----------------------------------------------------------------
// Q = h W2^T + b in FP32 (v_mfma_f32_16x16x4_f32), V = max over the stack's A
// actions, the q0 rows of root items.  IPB stacks a workgroup, an eighth of K a
// wavefront, the eight sums added in pairs.  SLICES: H holds fc1's slices, of
// which h is formed as fc1_split_kernel forms it; 14 KB a stack, so few stacks a
// workgroup.
template <bool SLICES, int IPB>
__global__ void __launch_bounds__(512) fc2_split_kernel(long long n, const float* __restrict__ H,
                                                        const float* __restrict__ scale1, const float* __restrict__ bias1,
                                                        const float* __restrict__ W2, const float* __restrict__ bias,
                                                        const ItemDesc* __restrict__ desc, float* __restrict__ V,
                                                        float* __restrict__ q0) {
  __shared__ f32x4 sums[8][2][64];
  const int lane = threadIdx.x & 63, c = threadIdx.x >> 6, r16 = lane & 15, g = lane >> 4;
  const long long first = (long long)blockIdx.x * IPB, m = r16 < IPB ? first + r16 : n;
  const long long mm = m < n ? m : first;
  const int A = desc[mm].A, root = desc[mm].q0_root;
  f32x4 h[4], w[2][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = 64 * c + 16 * j + 4 * g;
    w[0][j] = *reinterpret_cast<const f32x4*>(W2 + r16 * 512 + k);
    w[1][j] = *reinterpret_cast<const f32x4*>(W2 + (16 + r16 < kMaxA ? 16 + r16 : kMaxA - 1) * 512 + k);   // rows past the last: unused
  }
  if constexpr (SLICES) {
    f32x4 p[kFc1Split][4], sc[4], b[4];                    // every load in flight at once
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 64 * c + 16 * j + 4 * g;
#pragma unroll
      for (int z = 0; z < kFc1Split; ++z) p[z][j] = *reinterpret_cast<const f32x4*>(H + (z * n + mm) * 512 + k);
      sc[j] = *reinterpret_cast<const f32x4*>(scale1 + k);
      b[j] = *reinterpret_cast<const f32x4*>(bias1 + k);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      h[j] = p[0][j];
#pragma unroll
      for (int z = 1; z < kFc1Split; ++z) h[j] += p[z][j];
#pragma unroll
      for (int q = 0; q < 4; ++q) h[j][q] = fmaxf(fmaf(h[j][q], sc[j][q], b[j][q]), 0.f);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = *reinterpret_cast<const f32x4*>(H + mm * 512 + 64 * c + 16 * j + 4 * g);
  }
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int af = 0; af < 2; ++af)
        acc[af] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[af][j][q], h[j][q], acc[af], 0, 0, 0);
  sums[c][0][lane] = acc[0];
  sums[c][1][lane] = acc[1];
  __syncthreads();
  if (c) return;
  float best = -INFINITY;
  f32x4 qv[2];
#pragma unroll
  for (int af = 0; af < 2; ++af)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int x = 16 * af + 4 * g + q;
      float p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = sums[2 * i][af][lane][q] + sums[2 * i + 1][af][lane][q];
      qv[af][q] = (p[0] + p[1]) + (p[2] + p[3]) + (x < kMaxA ? bias[x] : 0.f);
      if (x < A) best = fmaxf(best, qv[af][q]);
    }
  best = fmaxf(best, __shfl_xor(best, 16));
  best = fmaxf(best, __shfl_xor(best, 32));
  if (m >= n) return;
  if (g == 0) V[m] = best;
  if (root >= 0) {
#pragma unroll
    for (int af = 0; af < 2; ++af)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (16 * af + 4 * g + q < kMaxA) q0[(long long)root * kMaxA + 16 * af + 4 * g + q] = qv[af][q];
  }
}

// W[N][K] FP32, row o times rs[o], weight k times cs[k % C], as operand planes, the low one times `low`
// (2^11; conv1's 1, whose planes share one sum).  Rows are paired so that
// a lane's sums of two fragments are 8 consecutive channels: row r of fragment
// f is channel 32 (f / 2) + 8 (r / 4) + 4 (f & 1) + r % 4.  Conv layers:
// [K / 32][N / 16][plane][64 lanes][8]; fc1 (rows): [N][K / 32][plane][32].
__global__ void split_weights_kernel(const float* __restrict__ w, const float* __restrict__ rs,
                                     const float* __restrict__ cs, int C, int N, int K, int rows, float low,
                                     _Float16* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)N * K) return;
  const int row = (int)(i / K), k = (int)(i % K), f = row >> 4, r = row & 15;
  const int o = 32 * (f >> 1) + 8 * (r >> 2) + 4 * (f & 1) + (r & 3);
  const float v = w[(long long)o * K + k] * (cs[k % C] * rs[o]);
  const _Float16 hi = (_Float16)v, lo = (_Float16)((v - (float)hi) * low);
  const int ks = k >> 5, g = (k >> 3) & 3, e = k & 7;
  _Float16* d = rows ? out + ((long long)row * (K / 32) + ks) * 64 + (k & 31)
                     : out + (((long long)ks * (N / 16) + f) * 2 * 64 + 16 * g + r) * 8 + e;
  d[0] = hi;
  d[rows ? 32 : 512] = lo;
}

}  // namespace

void launch_split_weights(int layer, const float* w, const float* row_scale, const float* col_scale, int C, int N, int K,
                          void* out, hipStream_t s) {
  const long long n = (long long)N * K;
  hipLaunchKernelGGL(split_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, row_scale, col_scale,
                     C, N, K, layer == 3 ? 1 : 0, layer == 0 ? 1.f : kSplitLow, reinterpret_cast<_Float16*>(out));
}

// Rules, with both sides measured (us; FP32 searches of A = 18 and A = 6, d = 1).
// Two stacks at a time (half the weight traffic, less padding of the row
// tiles) from kPairItems: 56 stacks 33 against 28 one at a time, 304 37 / 45,
// 3,584 107 / 121, 38,912 635 / 758.  Runs of about n / kRunItems stacks (each
// sums the shared channels again) so that the chip is full: 2,432 stacks 102
// with 256, 115 with 512, 125 with 1,024; 4,864 168 / 175 / 193; 9,728 345 /
// 328 / 343.
constexpr int kRunItems = 256, kPairItems = 256;
// fc1 + fc2: K's slices as workgroups (32 x 32 tiles) up to kSplitFc1Small, 512
// stacks 17 + 10 against 30 + 9 in 64 x 64 tiles, 1,024 26 + 10 / 31 + 8; then
// 64 x 64 tiles, and 256 x 128 ones for whole rounds of the chip (256 tiles,
// kSplitFc1Round stacks) and for a rest past kSplitFc1Medium: 8,192 stacks 102
// in 64 x 64 against 124 in 256 x 128, 14,336 143 / 132, 16,384 206 / 134;
// 19,456 180 against 239 as one launch.
constexpr long long kSplitFc1Small = 768, kSplitFc1Medium = 12288, kSplitFc1Round = 16384;

void launch_qnet_split(const QnetDev& q, const ItemDesc* desc, long long n, const ChunkGroups& cg, void* ws, float* V,
                       float* q0, hipStream_t s, hipEvent_t* ev) {
  if (n <= 0) return;
  unsigned char* x3 = reinterpret_cast<unsigned char*>(ws);
  float* h = reinterpret_cast<float*>(x3 + n * kSplitRow);
  float* part = h + n * 512;
  if (ev) (void)hipEventRecord(ev[0], s);
  SplitConvArgs a{};
  a.groups = cg.n > 0 ? cg.groups : nullptr;
  a.item_base = cg.item_base;
  a.desc = desc;
  for (int l = 0; l < 3; ++l) {
    a.w[l] = q.wsplit[l];
    a.scale[l] = q.ssplit[l];
    a.bias[l] = q.bsplit[l];
  }
  a.x3 = x3;
  a.n_groups = cg.n > 0 ? cg.n : n;
  const int most = cg.n > 0 ? cg.max_group : 1;
  const bool pairs = most > 1 && n >= kPairItems;
  const long long per = n / kRunItems;
  a.per_run = (int)(per < 1 ? 1 : per > most ? most : per);
  if (pairs) a.per_run += a.per_run & 1;
  a.units = a.n_groups * ((most + a.per_run - 1) / a.per_run);
  // a workgroup per run, dealt as CUs come free, where runs are few and uneven
  // (a mixed batch of 1,032 roots, 2,064 runs: the call 6,070 us, 6,160 with
  // 1,024 looping workgroups); 9,728 runs loop (2,640 us against 2,670)
  const unsigned blocks = (unsigned)(a.units < 4096 ? a.units : 1024);
  if (pairs) hipLaunchKernelGGL((conv_split_kernel<2, 2>), dim3(blocks), dim3(512), 0, s, a);
  else hipLaunchKernelGGL((conv_split_kernel<1, 1>), dim3(blocks), dim3(512), 0, s, a);
  for (int k = 1; ev && k <= 3; ++k) (void)hipEventRecord(ev[k], s);

  const unsigned char* w = reinterpret_cast<const unsigned char*>(q.wsplit[3]);
  auto grid = [](long long m, int bm, int bn) { return (unsigned)(((m + bm - 1) / bm + 7) / 8 * 8 * (512 / bn)); };
  const bool slices = n <= kSplitFc1Small;
  if (slices) {
    hipLaunchKernelGGL((fc1_split_kernel<32, 32, 2, 1, true>), dim3(grid(n, 32, 32), kFc1Split), dim3(128), 0, s, n, x3,
                       w, q.ssplit[3], q.bsplit[3], h, part);
  } else {
    const long long rest = n % kSplitFc1Round, full = rest <= kSplitFc1Medium ? n - rest : n;
    if (full > 0)
      hipLaunchKernelGGL((fc1_split_kernel<256, 128, 4, 2, false>), dim3(grid(full, 256, 128)), dim3(512), 0, s, full,
                         x3, w, q.ssplit[3], q.bsplit[3], h, part);
    if (full < n)
      hipLaunchKernelGGL((fc1_split_kernel<64, 64, 2, 2, false>), dim3(grid(n - full, 64, 64)), dim3(256), 0, s,
                         n - full, x3 + full * kSplitRow, w, q.ssplit[3], q.bsplit[3], h + full * 512, part);
  }
  if (ev) (void)hipEventRecord(ev[4], s);
  if (slices)
    hipLaunchKernelGGL((fc2_split_kernel<true, 4>), dim3((unsigned)((n + 3) / 4)), dim3(512), 0, s, n, part,
                       q.ssplit[3], q.bsplit[3], q.w2split, q.b[4], desc, V, q0);
  else
    hipLaunchKernelGGL((fc2_split_kernel<false, 16>), dim3((unsigned)((n + 15) / 16)), dim3(512), 0, s, n, h,
                       q.ssplit[3], q.bsplit[3], q.w2split, q.b[4], desc, V, q0);
  if (ev) (void)hipEventRecord(ev[5], s);
}

}  // namespace bcts
