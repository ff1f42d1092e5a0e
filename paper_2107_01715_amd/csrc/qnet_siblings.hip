// conv1 -> conv2 -> conv3 of the Nature-DQN for the leaves of a search (BF16
// and FP8 operands), sibling group by sibling group: the A children of one
// node, whose own frames the kernel forms itself.
//
// The children of a node share stack channels 0..2 (their parent's last three
// frames), and in the sprite world their own frames differ in the agent only:
// every other sprite moves the same way whatever the action.  So the kernel
// works on the group's background -- the shared frames and a frame without
// the agent -- plus, per child, the few outputs of each layer whose window
// meets the child's 6x6 agent square: at most 4x4 of conv1's 20x20, 4x4 of
// conv2's 9x9 and 6x6 of conv3's 7x7.  Every output sees the matrix
// instructions of a child computed by itself, in the same order, on the same
// operands, so the results are the same bits; an output that no agent square
// meets is the background's.  For 18 children that is 572 rows of conv1 on average
// instead of 7,200, 210 of conv2 instead of 1,458 and 259 of conv3 instead
// of 882, and the layers' weights are read once per group instead of once
// per 3 stacks.  A leaf's frame is never read, and expand.hip renders none.
//
// Work of a group (8 wavefronts, two per SIMD; one workgroup per CU, looping
// over groups):
//   * rows: conv1's list is the background's 400 pixels, then the children's
//     affected ones; conv2's 81 and conv3's 49 likewise.  A fragment is 16
//     consecutive rows of a list.  In conv1 a wavefront takes every eighth
//     fragment, in conv2 / conv3 every fourth for half the channels: all
//     channels per wavefront read the weights 8 times per group through the
//     CU's 64-byte vector-memory path, which then took longer than the matrix
//     instructions (conv2 9.7k clocks a group against 7.7k).
//   * a layer's result of list row r is entry r of the next layer's input
//     in LDS (conv1's background split in stride-2 phases as conv2 reads it).
//     A tap of child t at (y, x) is an affected entry of that child when both
//     y and x are among its affected rows and columns, else the background's:
//     two per-child tables of byte offsets from the background pixel to the
//     entry, one by row, one by column, very negative where unaffected;
//     background + max(row + column, 0) is the address.
//   * conv3's background rows stay in LDS; children's affected pixels go to
//     x3 in fc1's tiles directly, then every child's other pixels are copied
//     from the background.
//
// Measured on 1.49 M leaves of 256 roots (A = 18, depth 3), BF16: 17.1 ms in
// the group kernel of qnet_fused.hip, 5.8 ms here; FP8 13.8 and 4.4;
// the expansion, without the leaves' frames, 2.05 and 0.17 ms.  A group of 18
// takes 37k clocks, of which the matrix cores are busy 14k, vector
// instructions issue for 19k and LDS is active 21k: conv1 7k, conv2 7k and
// conv3 11k with the waits at their ends, the next group's lists, tables and
// frames 5k, the copies of unaffected pixels 3k.  What it learned on the
// way: one wavefront per SIMD with 512 registers was slower (it can issue one
// instruction per 4 clocks, and accumulators in the upper registers are
// moved), as was any code past the 64 KB instruction cache that two CUs
// share (with every fragment count its own unrolled copy a group took 99k
// clocks); a load or a register spill read back behind the stores of x3
// waits for them.
#include "bcts_internal.h"
#include "qnet_operand.h"

#include <atomic>

namespace bcts {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int kList1 = kMaxA * 16, kList2 = kMaxA * 16, kList3 = kMaxA * 36;   // affected outputs of a group, at most
constexpr int kBack = kMaxA;                            // table row of the background: nothing affected
constexpr int kNone = -(1 << 20);                       // table entry of an unaffected row or column

// Sizes by operand type.  LDS: x1 pixels (32 channels) X1P bytes apart, the
// background's as [phase (y & 1) * 2 + (x & 1)][y / 2][x / 2], then the
// children's entries; x2 pixels (64 channels) X2P apart.
template <int P> struct Geo {
  typedef Operand<P> Op;
  typedef typename Op::V V;
  static constexpr int EB = Op::EB, UB = Op::UB;
  static constexpr int X1P = EB == 2 ? 80 : 32, X2P = EB == 2 ? 144 : 80;
  static constexpr int FRB = kFrameBytes * EB;           // a staged frame
  static constexpr int X1B = (400 + kList1) * X1P, X2B = (81 + kList2) * X2P;
  static constexpr int UX = X2B > 3 * FRB ? X2B : 3 * FRB;
};
// FP8: conv2 / conv3 on the K = 128 instruction, their weights in LDS for the
// whole launch: per (layer, channel fragment cf, step s) two 1 KB blocks, the
// low and high 16 bytes of each lane's 32, conv2 at 0, conv3 at 32 KB, then
// conv3's two K = 32 tail units per fragment (512 bytes each).
constexpr int kWk3 = 32768, kWkTail = 65536, kWkBytes = 69632;

// A set of rows or columns is at most two runs of bits, one of them from bit
// 0 (a wrapping square): its n-th member, and the rank of a member.
struct Runs {
  unsigned m;
  int first, second;                     // length of the run from bit 0, start of the other
  __device__ explicit Runs(unsigned mask) : m(mask) {
    first = __builtin_ctz(~m);
    second = __builtin_ctz((m >> first << first) | 0x80000000u);
  }
  __device__ int count() const { return __builtin_popcount(m); }
  __device__ int nth(int n) const { return n < first ? n : second + n - first; }
  __device__ bool has(int b) const { return (m >> b) & 1u; }
  __device__ int rank(int b) const { return __builtin_popcount(m & ((1u << b) - 1u)); }
};
// i / c for i < 36, c = 1..6: by the rounded-up reciprocal in 256ths, exact there
__device__ __forceinline__ int quot(int i, int c) {
  constexpr unsigned long long k = 257ull | 129ull << 9 | 86ull << 18 | 65ull << 27 | 52ull << 36 | 43ull << 45;
  return (i * (int)((k >> (9 * c - 9)) & 511u)) >> 8;
}

// conv1 outputs (of 20) whose window [4 o, 4 o + 7] meets [a, a + 5] modulo 84
__device__ __forceinline__ unsigned hit1(int a) {
  const int lo = a >= 4 ? (a - 4) >> 2 : 0, hi = (a + 5) >> 2 < 19 ? (a + 5) >> 2 : 19;
  unsigned m = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
  if (a + 5 >= kFrame) m |= (2u << ((a + 5 - kFrame) >> 2)) - 1u;
  return m;
}
// conv2 outputs (of 9) whose window [2 o, 2 o + 3] meets the set m
__device__ __forceinline__ unsigned hit2(unsigned m) {
  unsigned r = 0;
#pragma unroll
  for (int o = 0; o < 9; ++o) r |= ((m >> (2 * o)) & 15u) ? 1u << o : 0u;
  return r;
}
// conv3 outputs (of 7) whose window [o, o + 2] meets the set m
__device__ __forceinline__ unsigned hit3(unsigned m) { return (m | (m >> 1) | (m >> 2)) & 127u; }

template <int P> struct Shared {
  typedef Geo<P> G;
  unsigned char x1[G::X1B];
  unsigned char ux[G::UX];               // the shared frames' operands during conv1, then x2
  unsigned char wk[P == P_FP8 ? kWkBytes : 16];
  unsigned char w1[16 * 64 * G::UB];     // conv1's weights, operand-major: unit (h2, s, lane)
  unsigned char noagent[G::FRB];         // operands of the children's frame without the agent
  unsigned char back3[49 * 64 * G::EB];  // conv3's background rows
  unsigned nrow[kFrame][4];              // columns covered by sprites 1..7, per frame row
  int rt1[kMaxA + 1][20], ct1[kMaxA + 1][20], rt2[kMaxA + 1][9], ct2[kMaxA + 1][9];
  // conv1's rows, the background's first: window origin in the frame's
  // pixels / 4 (11 bits), then the agent's square relative to the window,
  // column + 5 (4 bits) and row + 5 (5 bits; 31: none), and the entry's
  // offset in x1 / 16 (12 bits); conv2's and conv3's affected outputs: index
  // of the window's first row and column in the row and column tables (9 bits
  // each), then the window's origin in the background / 16
  unsigned list1[400 + kList1], list2[kList2];
  uint2 list3[kList3];                   // and the output's offset in x3 from the group's tile
  uint2 hits[kFrame];                    // per agent coordinate: conv1's set | conv2's << 20, conv3's
  unsigned long long own3[2][kMaxA];     // conv3's affected pixels of a child, bit y * 7 + x (two groups in turn)
  float bias[3][64];                     // conv1's 32 first
};
static_assert(sizeof(Shared<P_BF16>) <= 160 * 1024 && sizeof(Shared<P_FP8>) <= 160 * 1024, "one workgroup's LDS");

constexpr int kAhead = 2;                                // BF16: K steps of conv2 / conv3 weights in flight

// The lane index as a value the compiler cannot carry addresses across phases
// by: they are cheap to form again, and the registers are full in conv3.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A row of conv2's or conv3's list: child t's output (y, x).
template <int P, bool CONV3> __device__ __forceinline__ unsigned row_entry(int t, int y, int x) {
  const int n = CONV3 ? 9 : 20, s = CONV3 ? 1 : 2;
  return (unsigned)(t * n + s * y) | (unsigned)(t * n + s * x) << 9 |
         (unsigned)((CONV3 ? y * 9 + x : y * 10 + x) * ((CONV3 ? Geo<P>::X2P : Geo<P>::X1P) / 16)) << 18;
}

// BF16: the first K steps' weights of a layer (the wavefront's two channel
// fragments), requested before the barrier that opens it; FP8 keeps all
// weights in LDS.
template <int P> struct First {
  bf16x8 w[kAhead][2];
  __device__ void ask(__amdgpu_buffer_rsrc_t W, int lane, int wave, int steps) {
    const int ln = fresh(lane);
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        w[s][j] = Operand<P_BF16>::ldw(W, ln * 16 + (wave & 1) * steps * 2048, (j * steps + s) * 1024);
  }
};
template <> struct First<P_FP8> {
  __device__ void ask(__amdgpu_buffer_rsrc_t, int, int, int) {}
};

// One layer of conv2 / conv3 over NF fragments of a wavefront, its f0-th on
// (fragments wave / 2 + 4 i), for channel half wave % 2.  K step s is kernel
// row s / U, U steps per row (conv2: 4 columns; conv3: 3 columns x 2 channel
// halves of the input).  The weights of a step load kAhead steps ahead; a
// fragment's next pixels are read into the registers its matrix instructions
// have just used.
template <int NF, bool CONV3>
__device__ __forceinline__ void conv_rows(Shared<P_BF16>& sh, __amdgpu_buffer_rsrc_t W, const First<P_BF16>& first,
                                          int lane_, int wave, int f0, int total, f32x4 (&acc)[NF][2]) {
  typedef Operand<P_BF16> Op;
  typedef Op::V V;
  constexpr int kX1P = Geo<P_BF16>::X1P, kX2P = Geo<P_BF16>::X2P;
  constexpr int KW = CONV3 ? 3 : 4, PER = CONV3 ? 2 : 1, U = KW * PER, STEPS = KW * U, R = kAhead + 1;
  constexpr int SPAN = CONV3 ? 49 : 81, SIDE = CONV3 ? 7 : 9, PIX = CONV3 ? kX2P : kX1P;
  const int lane = fresh(lane_), r16 = lane & 15, g = lane >> 4;
  const unsigned char* src = CONV3 ? sh.ux : sh.x1;
  const int* rows = CONV3 ? &sh.rt2[0][0] : &sh.rt1[0][0];
  const int* cols = CONV3 ? &sh.ct2[0][0] : &sh.ct1[0][0];
  // offset of kernel row / column k from a window's origin
  auto row_off = [](int k) { return (CONV3 ? k * 9 : (k & 1) * 200 + (k >> 1) * 10) * PIX; };
  auto col_off = [](int k) { return (CONV3 ? k : (k & 1) * 100 + (k >> 1)) * PIX; };
  int base[NF], rt[NF][KW], ct[NF][KW];
  unsigned entry[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    int r = ((wave >> 1) + 4 * (f0 + i)) * 16 + r16;
    r = r < total ? r : total - 1;
    const int oy = r / SIDE;
    entry[i] = row_entry<P_BF16, CONV3>(kBack, oy, r - oy * SIDE);
    if (r >= SPAN) entry[i] = CONV3 ? sh.list3[r - SPAN].x : sh.list2[r - SPAN];
  }
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    base[i] = (int)(entry[i] >> 18) * 16 + 16 * g;
    const int* rp = rows + (entry[i] & 511u);
    const int* cp = cols + ((entry[i] >> 9) & 511u);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      rt[i][k] = rp[k];
      ct[i][k] = cp[k] + base[i];
    }
    acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int wl = lane * 16 + (wave & 1) * STEPS * 2048;
  V w[R][2], pv[NF];
#pragma unroll
  for (int s = 0; s < kAhead; ++s) {
    w[s][0] = first.w[s][0];
    w[s][1] = first.w[s][1];
  }
  auto pixel = [&](int s, int i) {
    const int kr = s / U, kc = s % U / PER, d = rt[i][kr] + ct[i][kc];
    return Op::ld(src + (d > base[i] ? d : base[i]) + row_off(kr) + col_off(kc) + (s % PER) * 64);
  };
#pragma unroll
  for (int i = 0; i < NF; ++i) pv[i] = pixel(0, i);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    if (s + kAhead < STEPS) {
#pragma unroll
      for (int j = 0; j < 2; ++j) w[(s + kAhead) % R][j] = Op::ldw(W, wl, (j * STEPS + s + kAhead) * 1024);
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      acc[i][0] = Op::mma(w[s % R][0], pv[i], acc[i][0]);
      acc[i][1] = Op::mma(w[s % R][1], pv[i], acc[i][1]);
      if (s + 1 < STEPS) pv[i] = pixel(s + 1, i);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The same for FP8: conv2 step s is kernel row s, lane group g its column g
// (32 channels); conv3 step s is tap 2 s + (g & 1), channels 32 (g >> 1) ..
// +31, and the ninth tap two K = 32 steps (the order of the group kernel's
// K = 128 path).  A lane's tap is its own, so its addresses are formed whole
// before the steps.
template <int NF, bool CONV3>
__device__ __forceinline__ void conv_rows(Shared<P_FP8>& sh, __amdgpu_buffer_rsrc_t, const First<P_FP8>&, int lane_,
                                          int wave, int f0, int total, f32x4 (&acc)[NF][2]) {
  typedef Operand<P_FP8> Op;
  constexpr int X1P = Geo<P_FP8>::X1P, X2P = Geo<P_FP8>::X2P;
  constexpr int SPAN = CONV3 ? 49 : 81, SIDE = CONV3 ? 7 : 9;
  const int lane = fresh(lane_), r16 = lane & 15, g = lane >> 4, half = wave & 1;
  const unsigned char* src = CONV3 ? sh.ux : sh.x1;
  int at[NF][4], at8[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    int r = ((wave >> 1) + 4 * (f0 + i)) * 16 + r16;
    r = r < total ? r : total - 1;
    const int oy = r / SIDE;
    unsigned e = row_entry<P_FP8, CONV3>(kBack, oy, r - oy * SIDE);
    if (r >= SPAN) e = CONV3 ? sh.list3[r - SPAN].x : sh.list2[r - SPAN];
    const int base = (int)(e >> 18) * 16, ri = e & 511u, ci = (e >> 9) & 511u;
    if (!CONV3) {
      const int col = (&sh.ct1[0][0])[ci + g], off = base + ((g & 1) * 100 + (g >> 1)) * X1P;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int d = (&sh.rt1[0][0])[ri + s] + col;
        at[i][s] = off + (d > 0 ? d : 0) + ((s & 1) * 200 + (s >> 1) * 10) * X1P;
      }
    } else {
      int row[3], col[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        row[k] = (&sh.rt2[0][0])[ri + k];
        col[k] = (&sh.ct2[0][0])[ci + k];
      }
      auto tap = [&](int kr, int kc) {
        const int d = row[kr] + col[kc];
        return base + (d > 0 ? d : 0) + (kr * 9 + kc) * X2P;
      };
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int even = tap(2 * s / 3, 2 * s % 3), odd = tap((2 * s + 1) / 3, (2 * s + 1) % 3);
        at[i][s] = ((g & 1) ? odd : even) + 32 * (g >> 1);
      }
      at8[i] = tap(2, 2) + 8 * g;
    }
    acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto ld32 = [](const unsigned char* q, int hi_at) {
    const u32x4 lo = *reinterpret_cast<const u32x4*>(q);
    const u32x4 hi = *reinterpret_cast<const u32x4*>(q + hi_at);
    return v8i{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
  };
  auto weights = [&](int s, int j) {
    return ld32(&sh.wk[(CONV3 ? kWk3 : 0) + (((2 * half + j) * 4 + s) * 2) * 1024 + lane * 16], 1024);
  };
  v8i w[2][2], pv[2];
  w[0][0] = weights(0, 0);
  w[0][1] = weights(0, 1);
  pv[0] = ld32(src + at[0][0], 16);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s + 1 < 4) {
      w[(s + 1) & 1][0] = weights(s + 1, 0);
      w[(s + 1) & 1][1] = weights(s + 1, 1);
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int n = s * NF + i;                          // pixel operand slot n & 1
      if (i + 1 < NF) pv[(n + 1) & 1] = ld32(src + at[i + 1][s], 16);
      else if (s + 1 < 4) pv[(n + 1) & 1] = ld32(src + at[0][s + 1], 16);
      __builtin_amdgcn_sched_barrier(0);                 // the next fragment's read goes out before these
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[s & 1][j], pv[n & 1], acc[i][j], 0, 0, 0, 127, 0, 127);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the sums materialise here: else the compiler sinks a fragment's whole
    // chain into its conditional store, which keeps every step's operands live
#pragma unroll
    for (int i = 0; i < NF; ++i) asm volatile("" : "+v"(acc[i][0]), "+v"(acc[i][1]));
  }
  if constexpr (CONV3) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      long wt[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) wt[j] = Op::ld(&sh.wk[kWkTail + (2 * half + j) * 1024 + (t * 64 + lane) * 8]);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        const long px = Op::ld(src + at8[i] + 32 * t);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = Op::mma(wt[j], px, acc[i][j]);
      }
    }
  }
}

// the lane's 8 consecutive channels 32 h + 8 g .. +7 of one row
template <int P>
__device__ __forceinline__ void out8(void* p, const f32x4& a, const f32x4& b, float sc, const float (&bb)[2][4], float o8) {
  typedef Operand<P> Op;
  const typename Op::PK lo = Op::pk4(fmaxf(a[0] * sc + bb[0][0], 0.f), fmaxf(a[1] * sc + bb[0][1], 0.f),
                            fmaxf(a[2] * sc + bb[0][2], 0.f), fmaxf(a[3] * sc + bb[0][3], 0.f), o8);
  const typename Op::PK hi = Op::pk4(fmaxf(b[0] * sc + bb[1][0], 0.f), fmaxf(b[1] * sc + bb[1][1], 0.f),
                            fmaxf(b[2] * sc + bb[1][2], 0.f), fmaxf(b[3] * sc + bb[1][3], 0.f), o8);
  Op::st8(p, lo, hi);
}

// conv2 (rows -> x2) and conv3 (the background's rows -> back3, the
// children's -> x3 in fc1's tiles)
template <int P, int NF, bool CONV3>
__device__ __forceinline__ void conv_group(Shared<P>& sh, const FusedConvArgs& a, __amdgpu_buffer_rsrc_t W,
                                           const First<P>& first, int lane, int wave, int f0, int total,
                                           long long item0) {
  typedef Geo<P> G;
  f32x4 acc[NF][2];
  conv_rows<NF, CONV3>(sh, W, first, lane, wave, f0, total, acc);
  lane = fresh(lane);
  const int r16 = lane & 15, g = lane >> 4, half = wave & 1;
  const int ch = (32 * half + 8 * g) * G::EB;            // the lane's channels within a pixel
  // within x3's 64-byte slices of a pixel (2 in BF16)
  const unsigned slice = (unsigned)((ch >> 6) * kFc1StageBytes + (ch & 63));
  unsigned char* x3 = reinterpret_cast<unsigned char*>(a.x3) + (item0 / kFc1Rows) * fc1_tile_bytes(G::EB);
  const float sc = a.acc_scale[CONV3 ? 2 : 1], o8 = a.out_s8[CONV3 ? 2 : 1];
  float bb[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) bb[j][q] = sh.bias[CONV3 ? 2 : 1][32 * half + 8 * g + 4 * j + q];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int r = ((wave >> 1) + 4 * (f0 + i)) * 16 + r16;
    if (r >= total) continue;
    if (!CONV3) out8<P>(&sh.ux[r * G::X2P + ch], acc[i][0], acc[i][1], sc, bb, o8);
    else if (r < 49) out8<P>(&sh.back3[r * 64 * G::EB + ch], acc[i][0], acc[i][1], sc, bb, o8);
    else out8<P>(x3 + (sh.list3[r - 49].y + slice), acc[i][0], acc[i][1], sc, bb, o8);
  }
}

template <int P>
__global__ void __launch_bounds__(kThreads, 2) conv_siblings_kernel(FusedConvArgs a) {
  typedef Geo<P> G;
  typedef typename G::Op Op;
  typedef typename G::V V;
  constexpr int EB = G::EB;
  __shared__ __attribute__((aligned(16))) Shared<P> sh;
  typedef const __attribute__((address_space(1))) u32x4 GV;
  typedef const __attribute__((address_space(1))) unsigned long long GQ;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grid = (int)gridDim.x;
  const __amdgpu_buffer_rsrc_t W2r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w[1]), (short)0, 64 * 512 * EB, 0x00020000);
  const __amdgpu_buffer_rsrc_t W3r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w[2]), (short)0, 64 * 576 * EB, 0x00020000);

  // ---- once per launch: conv1's weights (rows paired), the background's
  // table rows, biases ----
  const unsigned char* W1 = reinterpret_cast<const unsigned char*>(a.w[0]);
  for (int k = tid; k < 16 * 64; k += kThreads) {
    const int h2 = k >> 9, s = (k >> 6) & 7, l = k & 63, row = 8 * ((l & 15) >> 2) + 4 * h2 + (l & 3);
    *reinterpret_cast<V*>(&sh.w1[k * G::UB]) = Op::ld(W1 + (row * 256 + 32 * s + 8 * (l >> 4)) * EB);
  }
  if constexpr (P == P_FP8) {
    // the K = 128 weight copies (per fragment 16 rows x K bytes: 32 bytes per
    // lane and step, then K = 32 units of 8) into the layout above
    const unsigned char* W2 = reinterpret_cast<const unsigned char*>(a.w[1]);
    const unsigned char* W3 = reinterpret_cast<const unsigned char*>(a.w[2]);
    for (int c = tid; c < kWkBytes / 16; c += kThreads) {
      const unsigned char* src;
      int dst;
      if (c < 4096) {                                    // c = ((cf * 4 + s) * 64 + lane) * 2 + part of conv2, then conv3
        const int c3 = c >= 2048, cc = c & 2047, part = cc & 1, ln = (cc >> 1) & 63, us = cc >> 7;
        src = c3 ? W3 + (us >> 2) * 16 * 576 + ((us & 3) * 64 + ln) * 32 + part * 16 : W2 + cc * 16;
        // conv3: lane group g takes tap offset g & 1 and channel half g >> 1,
        // in memory lane group 2 (g & 1) + (g >> 1)
        const int lg = c3 ? ((((ln >> 4) & 1) << 1) | (ln >> 5)) : (ln >> 4);
        dst = (c3 ? kWk3 : 0) + (us * 2 + part) * 1024 + ((ln & 15) + 16 * lg) * 16;
      } else {
        const int cc = c - 4096;
        src = W3 + (cc >> 6) * 16 * 576 + 4 * 2048 + (cc & 63) * 16;
        dst = kWkTail + cc * 16;
      }
      *reinterpret_cast<u32x4*>(&sh.wk[dst]) = *reinterpret_cast<const u32x4*>(src);
    }
  }
  // a background sprite's pixel (128) and the agent's (255) as operands, in
  // every element of a 32-bit word
  unsigned sprite_op, agent_op;
  if constexpr (P == P_BF16) {
    sprite_op = 0x43004300u;
    agent_op = 0x437F437Fu;
  } else {
    const float s128 = 128.f * a.pix_s8, s255 = 255.f * a.pix_s8;
    sprite_op = (unsigned)__builtin_amdgcn_readfirstlane((int)fp8_pack4(s128, s128, s128, s128));
    agent_op = (unsigned)__builtin_amdgcn_readfirstlane((int)fp8_pack4(s255, s255, s255, s255));
  }
  // all-ones elements of word k of 8 pixels' operands where `on` has their bit
  auto word_mask = [](unsigned on, int k) {
    if constexpr (P == P_BF16)
      return (((int)(on << (31 - 2 * k)) >> 31) & 0xFFFFu) | (((int)(on << (30 - 2 * k)) >> 31) & 0xFFFF0000u);
    else
      return (((on >> (4 * k)) & 15u) * 0x00204081u & 0x01010101u) * 255u;
  };
  if (tid < kFrame) {
    const unsigned m1 = hit1(tid), m2 = hit2(m1);
    sh.hits[tid] = make_uint2(m1 | m2 << 20, hit3(m2));
  }
  for (int p = tid; p < 400; p += kThreads) {
    const int y = p / 20, x = p - y * 20, at = ((y & 1) * 2 + (x & 1)) * 100 + (y >> 1) * 10 + (x >> 1);
    sh.list1[p] = (unsigned)(y * kFrame + x) | 31u << 15 | (unsigned)(at * (G::X1P / 16)) << 20;
  }
  if (tid < 20) sh.rt1[kBack][tid] = sh.ct1[kBack][tid] = kNone;
  else if (tid < 29) sh.rt2[kBack][tid - 20] = sh.ct2[kBack][tid - 20] = kNone;
  if (tid >= kThreads - 192) {
    const int l = (tid - (kThreads - 192)) >> 6, c = tid & 63;
    if (l > 0 || c < 32) sh.bias[l][c] = a.bias[l][c];
  }
  // ---- a group's inputs, requested ahead of their use: its header and first
  // descriptor (frame pointers, position rows) two groups ahead, its 3
  // shared frames and its children's positions one ahead.  Vector loads: a
  // scalar load would make the next LDS read wait for it too. ----
  struct Head { int count, leaf; long long i0; };
  auto clampg = [&](int q) { return q < a.n_groups ? q : a.n_groups - 1; };
  auto word = [](unsigned long long v, int l) {          // lane l's 64-bit value
    return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)v, l) |
           (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32;
  };
  auto ask_head = [&](int q) { return ((GQ*)(a.groups + clampg(q)))[fresh(lane) & 1]; };
  auto head = [&](unsigned long long v) {
    const unsigned long long hi = word(v, 1);
    return Head{(int)(unsigned)hi, (int)(hi >> 32), (long long)word(v, 0) - a.item_base};
  };
  auto ask_desc = [&](long long i0) { return ((GQ*)(a.desc + i0))[fresh(lane) & 3]; };
  constexpr int kChunks = kFrameBytes / 16, kLoads = (3 * kChunks + kThreads - 1) / kThreads;
  u32x4 fv[kLoads], pv;                                  // flat chunk 441 frame + chunk, 512 threads x 3
  auto request = [&](unsigned long long d, int cnt) {
    const uint8_t* f[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) f[c] = reinterpret_cast<const uint8_t*>(word(d, c));
    const uint8_t* pos = reinterpret_cast<const uint8_t*>(word(d, 3));
    const int ft = fresh(tid);
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int e0 = ft + j * kThreads, e = e0 < 3 * kChunks ? e0 : 3 * kChunks - 1;
      const int c = e >= 2 * kChunks ? 2 : e >= kChunks ? 1 : 0;
      const uint8_t* p = c == 2 ? f[2] : c == 1 ? f[1] : f[0];
      fv[j] = ((GV*)p)[e - c * kChunks];
    }
    const int fl = ft & 63;
    pv = ((GV*)pos)[fl < cnt ? fl : cnt - 1];        // positions of child `lane`
  };

  // The frames of a group go to LDS, its affected sets become lists and tables
  // (par: the group's parity, for own3); returns the three lists' lengths.
  struct Counts { int n1, n2, n3; };
  auto prepare = [&](int G, long long i0, int par) {
    const int first_row = (int)(i0 & (kFc1Rows - 1));
    const int tid = fresh(threadIdx.x), lane = tid & 63;
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int e0 = tid + j * kThreads, e = e0 < 3 * kChunks ? e0 : 3 * kChunks - 1;
      // threads past the end store the last chunk again
      Op::stage16(&sh.ux[e * 16 * EB], make_uint4(fv[j][0], fv[j][1], fv[j][2], fv[j][3]), a.pix_s8);
    }
    // child `lane`'s affected rows and columns, in every wavefront alike
    const int ax = pv[0] & 255, ay = (pv[0] >> 8) & 255;
    const uint2 hx = sh.hits[ax], hy = sh.hits[ay];
    const int mine = __builtin_popcount(hy.x & 0xFFFFFu) * __builtin_popcount(hx.x & 0xFFFFFu) |
                     __builtin_popcount(hy.x >> 20) * __builtin_popcount(hx.x >> 20) << 10 |
                     __builtin_popcount(hy.y) * __builtin_popcount(hx.y) << 20;
    // inclusive sums over the children (lanes 0..17), three 10-bit counts in one word
    int scan = lane < G ? mine : 0;
    scan += __builtin_amdgcn_update_dpp(0, scan, 0x111, 0xF, 0xF, false);      // row_shr:1, 2, 4, 8
    scan += __builtin_amdgcn_update_dpp(0, scan, 0x112, 0xF, 0xF, false);
    scan += __builtin_amdgcn_update_dpp(0, scan, 0x114, 0xF, 0xF, false);
    scan += __builtin_amdgcn_update_dpp(0, scan, 0x118, 0xF, 0xF, false);
    scan += lane >= 16 ? __builtin_amdgcn_readlane(scan, 15) : 0;
    const int all = __builtin_amdgcn_readlane(scan, G - 1), before = scan - mine;
    // 28 threads per child
    const int t = tid / 28, sub = tid - t * 28;
    const int at = __shfl(before, t), xy = __shfl(ax | ay << 8, t);
    if (t < G) {
      const int cx = xy & 255, cy = xy >> 8;
      const uint2 ux = sh.hits[cx], uy = sh.hits[cy];
      const Runs y1(uy.x & 0xFFFFFu), x1(ux.x & 0xFFFFFu), y2(uy.x >> 20), x2(ux.x >> 20), y3(uy.y), x3(ux.y);
      const int o1 = at & 1023, o2 = (at >> 10) & 1023, o3 = at >> 20;
      const int c1 = x1.count(), c2 = x2.count(), c3 = x3.count();
      // tables: the entry's offset by row plus by column, less the background
      // pixel's; adding the background address gives the entry's
      if (sub < 20) {
        const int half = sub >> 1, odd = sub & 1;
        sh.rt1[t][sub] = y1.has(sub) ? (400 + o1 + y1.rank(sub) * c1 - odd * 200 - half * 10) * G::X1P : kNone;
        sh.ct1[t][sub] = x1.has(sub) ? (x1.rank(sub) - odd * 100 - half) * G::X1P : kNone;
      } else if (sub == 20) {
        unsigned long long m = 0;
#pragma unroll
        for (int y = 0; y < 7; ++y) m |= y3.has(y) ? (unsigned long long)x3.m << (7 * y) : 0ull;
        sh.own3[par][t] = m;
      }
      if (sub < 9) {
        sh.rt2[t][sub] = y2.has(sub) ? (81 + o2 + y2.rank(sub) * c2 - sub * 9) * G::X2P : kNone;
        sh.ct2[t][sub] = x2.has(sub) ? (x2.rank(sub) - sub) * G::X2P : kNone;
      }
      if (sub < y1.count() * c1) {
        const int q = quot(sub, c1), y = y1.nth(q), x = x1.nth(sub - q * c1);
        int ex = cx - 4 * x, ey = cy - 4 * y;            // past the frame's end: a wrapping square
        ex -= ex > 7 ? kFrame : 0;
        ey -= ey > 7 ? kFrame : 0;
        sh.list1[400 + o1 + sub] = (unsigned)(y * kFrame + x) | (unsigned)(ex + 5) << 11 | (unsigned)(ey + 5) << 15 |
                                   (unsigned)((400 + o1 + sub) * (G::X1P / 16)) << 20;
      }
      if (sub < y2.count() * c2) {
        const int q = quot(sub, c2);
        sh.list2[o2 + sub] = row_entry<P, false>(t, y2.nth(q), x2.nth(sub - q * c2));
      }
      for (int l = sub; l < y3.count() * c3; l += 28) {
        const int q = quot(l, c3);
        const int y = y3.nth(q), x = x3.nth(l - q * c3);
        // x3 rows of a group lie in at most two of fc1's tiles
        const int row = first_row + t;
        sh.list3[o3 + l] = make_uint2(row_entry<P, true>(t, y, x), (unsigned)((row >> 8) * (int)fc1_tile_bytes(EB) + (row & 255) * 64 +
                                                                           (y * 7 + x) * EB * kFc1StageBytes));
      }
    }
    // columns covered by sprites 1..7 (the same for every child: child 0's)
    unsigned pw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) pw[k] = (unsigned)__builtin_amdgcn_readfirstlane((int)pv[k]);
    if (tid >= kThreads - kFrame) {
      const int y = tid - (kThreads - kFrame);
      unsigned m[3] = {0u, 0u, 0u};
#pragma unroll
      for (int i = 1; i < kSprites; ++i) {
        const int sx = (pw[i >> 1] >> ((i & 1) * 16)) & 255, sy = (pw[i >> 1] >> ((i & 1) * 16 + 8)) & 255;
        int dy = y - sy;
        dy += dy < 0 ? kFrame : 0;
        if (dy < 6) {
          // columns 32 k .. 32 k + 31 of [sx, sx + 5], and of its wrapped part
          const unsigned long long w = 0x3Full << (sx & 31);
          const int j = sx >> 5;
#pragma unroll
          for (int k = 0; k < 3; ++k) m[k] |= j == k ? (unsigned)w : j + 1 == k ? (unsigned)(w >> 32) : 0u;
          if (sx + 6 > kFrame) m[0] |= (1u << (sx + 6 - kFrame)) - 1u;
        }
      }
      *reinterpret_cast<u32x4*>(sh.nrow[y]) = u32x4{m[0], m[1], m[2] & 0xFFFFFu, 0u};   // columns 0..83
    }
    return Counts{all & 1023, (all >> 10) & 1023, all >> 20};
  };

  // Everything a group needs is in LDS when its iteration begins.  A load in
  // flight there would be waited for behind the previous group's stores (one
  // counter, in order), so none is: the next group's frames are requested
  // before conv1 and staged at the end of the same iteration.
  if ((int)blockIdx.x >= a.n_groups) return;
  lds_barrier();                                         // the launch's tables are in LDS
  int gi = (int)blockIdx.x - grid;                       // the first iteration only stages the first group
  Head cur{0, 0, 0}, nxt = head(ask_head(blockIdx.x));
  unsigned long long next_desc = ask_desc(nxt.i0), next2_head = ask_head(blockIdx.x + grid);
  int par = 0;
  Counts cn{};
  for (;;) {
    const bool has_next = gi + grid < a.n_groups;
    const Head nxt2 = head(next2_head);
    const unsigned long long next2_desc = ask_desc(nxt2.i0), next3_head = ask_head(gi + 3 * grid);
    if (cur.leaf) {
    lds_barrier();
    // the background frame's operands, 16 pixels a thread
    for (int e = fresh(tid); e < kChunks; e += kThreads) {
      const int y0 = (e * 16) / kFrame, x0 = e * 16 - y0 * kFrame;
      const u32x4 r0 = *reinterpret_cast<const u32x4*>(sh.nrow[y0]);
      const u32x4 r1 = *reinterpret_cast<const u32x4*>(sh.nrow[y0 + 1 < kFrame ? y0 + 1 : y0]);
      const unsigned long long lo = (unsigned long long)r0[1] << 32 | r0[0], hi = r0[2];
      // bits x0 .. x0 + 15 of row y0, continued by row y0 + 1 from column 84 on
      unsigned v = (unsigned)(x0 < 64 ? lo >> x0 | (x0 ? hi << (64 - x0) : 0ull) : hi >> (x0 - 64));
      if (x0 > kFrame - 16) v = (v & ((1u << (kFrame - x0)) - 1u)) | r1[0] << (kFrame - x0);
#pragma unroll
      for (int h = 0; h < 2; ++h) {                      // 8 pixels: UB bytes
        unsigned o[2 * EB];
#pragma unroll
        for (int k = 0; k < 2 * EB; ++k) o[k] = word_mask((v >> (8 * h)) & 255u, k) & sprite_op;
        __builtin_memcpy(&sh.noagent[e * 16 * EB + h * G::UB], o, G::UB);
      }
    }
    if (has_next) request(next_desc, nxt.count);
    lds_barrier();

    // ---- conv1: rows of the background, then the children's ----
    {
      const float sc = a.acc_scale[0], o8 = a.out_s8[0];
      const int ln = fresh(lane), l16 = ln & 15, lg = ln >> 4;
      V w1[2][8];
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
        for (int s = 0; s < 8; ++s) w1[h2][s] = Op::ld(&sh.w1[((h2 * 8 + s) * 64 + ln) * G::UB]);
      // A fragment's sums run while the next one's operands are read and the
      // previous one's outputs stored; rows past the list repeat its last one
      // (same bits, same entry).
      const int rows1 = 400 + cn.n1, nf = (rows1 + 16 * kWaves - 1) / (16 * kWaves);
      V pix[2][8];
      int entry[2];
      f32x4 acc[2][2];
      unsigned le;
      auto ask = [&](int i) {                            // list entry of the wavefront's i-th fragment
        const int r = (i * kWaves + wave) * 16 + l16;
        le = sh.list1[r < rows1 ? r : rows1 - 1];
      };
      auto read = [&](int b) {
        const int off = ((le & 2047u) * 4u + lg * kFrame) * EB;
        entry[b] = (le >> 20) * 16 + G::UB * lg;
#pragma unroll
        for (int s = 0; s < 8; ++s)
          pix[b][s] = Op::ld_pix((s < 6 ? &sh.ux[(s >> 1) * G::FRB] : sh.noagent) + off + (s & 1) * 4 * kFrame * EB);
      };
      auto overlay = [&](int b, unsigned e) {            // the agent's pixels: 255
        const int ey = (int)((e >> 15) & 31u) - 5;
        const unsigned sq = ((0x3Fu << (((e >> 11) & 15u) + 1u)) >> 6) & 255u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const unsigned on = (unsigned)(4 * h + lg - ey) < 6u ? sq : 0u;
          unsigned v[2 * EB];
          __builtin_memcpy(v, &pix[b][6 + h], G::UB);
#pragma unroll
          for (int q = 0; q < 2 * EB; ++q) {
            const unsigned m = word_mask(on, q);
            v[q] = (m & agent_op) | (~m & v[q]);
          }
          __builtin_memcpy(&pix[b][6 + h], v, G::UB);
        }
      };
      auto store = [&](int b) {
        float b1[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) b1[j][q] = sh.bias[0][8 * lg + 4 * j + q];
        out8<P>(&sh.x1[entry[b]], acc[b][0], acc[b][1], sc, b1, o8);
      };
      ask(0);
      unsigned lc = le;
      read(0);
      ask(1);
      auto step = [&](int i, int b, bool stores) {
        if (i * kWaves + wave >= 25) overlay(b, lc);     // wave-uniform: the background's fragments have none
        lc = le;
        if (stores) store(b ^ 1);
        read(b ^ 1);                                     // past the last fragment: its rows again, unused
        ask(i + 2);
        acc[b][0] = acc[b][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2) acc[b][h2] = Op::mma(w1[h2][s], pix[b][s], acc[b][h2]);
      };
      step(0, 0, false);
#pragma unroll 1
      for (int i = 1; i < nf; i += 2) {
        step(i, 1, true);
        if (i + 1 < nf) step(i + 1, 0, true);
      }
      if (nf & 1) store(0);
      else store(1);
    }
    First<P> first;
    first.ask(W2r, lane, wave, 16);
    lds_barrier();       // x1 complete; the frames are read: conv2 may write x2 over them

    // ---- conv2 and conv3: 64 rows per fragment of a wavefront, unrolled code
    // for several counts; the largest leaves what is past it to a second turn.
    // A group of 18 has 2 to 5 fragments of conv2 and 2 to 9 of conv3 (3.7 and
    // 4.5 on average): with code for 3 and 5, 4 and 8 only, which run 4.2 and
    // 5.8, 256 searches of A = 18, d = 3 take 3% longer (53 KB of code: two
    // CUs' 64 KB of instruction cache hold it) ----
    const int rows2 = 81 + cn.n2, rows3 = 49 + cn.n3, frags2 = (rows2 + 63) >> 6, frags3 = (rows3 + 63) >> 6;
    if (frags2 > 4) conv_group<P, 5, false>(sh, a, W2r, first, lane, wave, 0, rows2, 0);
    if (frags2 > 5) first.ask(W2r, lane, wave, 16);
    if (frags2 <= 4 || frags2 > 5) {
      const int f0 = frags2 > 5 ? 5 : 0, left = frags2 - f0;
      if (left <= 2) conv_group<P, 2, false>(sh, a, W2r, first, lane, wave, f0, rows2, 0);
      else if (left <= 3) conv_group<P, 3, false>(sh, a, W2r, first, lane, wave, f0, rows2, 0);
      else conv_group<P, 4, false>(sh, a, W2r, first, lane, wave, f0, rows2, 0);
    }
    first.ask(W3r, lane, wave, 18);
    lds_barrier();
    if (frags3 > 6) conv_group<P, 8, true>(sh, a, W3r, first, lane, wave, 0, rows3, cur.i0);
    if (frags3 > 8) first.ask(W3r, lane, wave, 18);
    if (frags3 <= 6 || frags3 > 8) {
      const int f0 = frags3 > 8 ? 8 : 0, left = frags3 - f0;
      if (left <= 2) conv_group<P, 2, true>(sh, a, W3r, first, lane, wave, f0, rows3, cur.i0);
      else if (left <= 3) conv_group<P, 3, true>(sh, a, W3r, first, lane, wave, f0, rows3, cur.i0);
      else if (left <= 4) conv_group<P, 4, true>(sh, a, W3r, first, lane, wave, f0, rows3, cur.i0);
      else conv_group<P, 6, true>(sh, a, W3r, first, lane, wave, f0, rows3, cur.i0);
    }
    lds_barrier();       // the background's rows are in LDS; x2 is read

    // ---- every child's unaffected pixels: a thread copies 16-byte chunk c of
    // child t's 64-byte slices (EB a pixel), consecutive threads along a
    // slice's children, 512 / 4 G slices at a time ----
    {
      const int per = 4 * cur.count, step = kThreads / per, tid_ = fresh(tid);
      const int first_sl = tid_ / per, rem = tid_ - first_sl * per, t = rem >> 2, c = rem & 3;
      if (first_sl < step) {
        const unsigned long long own = sh.own3[par][t];
        unsigned char* to = reinterpret_cast<unsigned char*>(a.x3) + fc1_tiled_offset(cur.i0 + t, 16 * c, EB);
        const unsigned char* from = &sh.back3[16 * c];
#pragma unroll 4
        for (int sl = first_sl; sl < 49 * EB; sl += step) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(from + sl * 64);
          if (!((own >> (sl / EB)) & 1ull)) *reinterpret_cast<u32x4*>(to + sl * kFc1StageBytes) = v;
        }
      }
    }
    par ^= 1;
    } else if (has_next) {
      request(next_desc, nxt.count);                     // before the first group, or another kernel's group
    }
    if (!has_next) break;
    if (nxt.leaf) cn = prepare(nxt.count, nxt.i0, par);
    gi += grid;
    cur = nxt;
    nxt = nxt2;
    next_desc = next2_desc;
    next2_head = next3_head;
  }
}

}  // namespace

void launch_conv_siblings(int prec, const FusedConvArgs& args, int n_groups, hipStream_t s) {
  if (n_groups <= 0) return;
  constexpr int kDevs = 64;
  static std::atomic<int> cus[kDevs];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
  int n = dev < kDevs ? cus[dev].load(std::memory_order_relaxed) : 0;
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    if (dev < kDevs) cus[dev].store(n, std::memory_order_relaxed);
  }
  FusedConvArgs a = args;
  a.n_groups = n_groups;
  const dim3 blocks((unsigned)(n_groups < n ? n_groups : n)), threads(kThreads);
  if (prec == P_BF16) hipLaunchKernelGGL(conv_siblings_kernel<P_BF16>, blocks, threads, 0, s, a);
  else hipLaunchKernelGGL(conv_siblings_kernel<P_FP8>, blocks, threads, 0, s, a);
}

}  // namespace bcts
