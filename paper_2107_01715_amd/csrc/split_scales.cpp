// Scales of the FP32 network's split form (see split_scales.h).
//
// Every conv output channel is held times a power of two of its own: the one
// that brings what the channel can reach at most, b = sum max(w, 0) b_in +
// bias over inputs of [0, b_in], into [2^14, 2^15).  The next layer's weights
// on the channel are divided by it, then every row of weights is held times the
// power of two that brings its largest into [2^13, 2^14).  So sizes that a
// network shifts between a channel and the weights that read it do not count:
// such networks give the same bits.
//
// What FP16 cannot hold is then a matter of how far below those limits a layer
// works.  The smallest values' error is absolute: 2^-36 of a held activation or
// weight (half of FP16's last place, the low plane held 2^11 times as large),
// 2^-25 of a weight of conv1, whose low plane is held as it is.  It has to stay
// below FP32's own 2^-24 of a channel's typical output.  Typical: of its
// positive contributions, one an input channel (conv1: a pixel) at the input's
// typical value, the lower quartile times the square root of their number.  A
// few inputs that could be large but never are raise the bound and not the
// quartile, and so turn a network down rather than take its bits.  And on a dark
// stack, whose outputs come from the biases alone: the errors of a layer's
// outputs, weighted by the weights that read them, stay below 2^-22 of them.
// Kaiming and heavier-tailed weights (Student's t, 4 degrees) pass with 2^8 to
// spare; biases of 1e-5 throughout pass, of 1e-6 do not.
#include "split_scales.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "layout.h"

namespace bcts {

bool split_scales(const std::vector<float>* W, const std::vector<float>* B, SplitScales* sp) {
  constexpr int kMost = 60;                      // of an exponent; weights of a size no trained network has are past it
  const double fine = std::ldexp(1.0, -25) / kSplitLow, need = std::ldexp(1.0, -24);
  // the inputs' largest and typical values, their values on a dark stack and
  // their exponents, by channel (conv1: by pixel of the window)
  std::vector<double> bound(256, 255.0), typical(256, 128.0), dark(256, 0.0);
  std::vector<int> e_in(256, 0);
  for (int l = 0; l < 4; ++l) {
    const size_t N = B[l].size(), K = W[l].size() / N, C = bound.size();
    const double acc = l == 0 ? (double)(1.f / 255.f) : 1.0;   // as the FP32 path multiplies it
    std::vector<double> col(C), readers(C, 0.0);   // readers: sum over the rows of their largest weight's square
    double held = 0.0;                           // sum over a row of the typical inputs' squares, as held
    for (size_t c = 0; c < C; ++c) {
      col[c] = bound[c] > 0.0 ? std::ldexp(1.0, -e_in[c]) : 0.0;   // a channel that is always zero
      held += std::pow(std::ldexp(typical[c], e_in[c]), 2.0) * (double)(K / C);
      sp->col[l].push_back((float)col[c]);
    }
    std::vector<double> b_out(N), t_out(N), d_out(N);
    std::vector<int> e_out(N, 0);
    std::vector<double> part;
    float sum[256], positive[256], most[256], largest[256];
    for (size_t o = 0; o < N; ++o) {
      const float* w = &W[l][o * K];
      const double bias = B[l][o];
      // of the row's weights on each channel (a lane a channel: 1.6 M weights in fc1)
      for (size_t c = 0; c < C; ++c) sum[c] = positive[c] = most[c] = largest[c] = 0.f;
      for (size_t k = 0; k < K; k += C)
        for (size_t c = 0; c < C; ++c) {
          const float v = w[k + c], up = v > 0.f ? v : 0.f, size = std::fabs(v);
          sum[c] += v;
          positive[c] += up;
          most[c] = most[c] > up ? most[c] : up;
          largest[c] = largest[c] > size ? largest[c] : size;
        }
      double top = 0.0, reach = 0.0, at_dark = 0.0;
      part.clear();
      for (size_t c = 0; c < C; ++c) {
        top = std::max(top, largest[c] * col[c]);
        reach += positive[c] * bound[c];
        at_dark += sum[c] * dark[c];
        readers[c] += (double)largest[c] * largest[c];
        if (most[c] > 0.f && typical[c] > 0.0) part.push_back(most[c] * typical[c]);
      }
      b_out[o] = std::max(0.0, reach * acc + bias);
      if (b_out[o] == 0.0) {                     // never positive: zeros
        sp->row[l].push_back(0.f);
        sp->out[l].push_back(0.f);
        sp->bias[l].push_back(0.f);
        continue;
      }
      double t = std::max(bias, 0.0);
      if (!part.empty()) {
        std::nth_element(part.begin(), part.begin() + part.size() / 4, part.end());
        t = std::max(t, part[part.size() / 4] * std::sqrt((double)part.size()) * acc);
      }
      t_out[o] = t = std::min(t, b_out[o]);
      d_out[o] = std::max(0.0, at_dark * acc + bias);

      const int er = top > 0.0 ? 13 - std::ilogb(top) : 0;
      if (l < 3) e_out[o] = 14 - std::ilogb(b_out[o]);   // fc1's outputs stay FP32, unscaled
      const int eo = e_out[o];
      bool ok = std::abs(er) <= kMost && std::abs(eo) <= kMost && std::abs(eo - er) <= 100;
      if (top > 0.0) ok = ok && (l == 0 ? fine * kSplitLow : fine) * std::sqrt(held) <= need * std::ldexp(t / acc, er);
      if (l < 3) ok = ok && fine <= need * std::ldexp(t, eo);
      if (!ok) return false;
      // a conv layer's outputs are split from kSplitLow times what the planes hold
      const double up = l < 3 ? (double)kSplitLow : 1.0;
      sp->row[l].push_back((float)std::ldexp(1.0, er));
      sp->out[l].push_back((float)std::ldexp(up * acc, eo - er));
      sp->bias[l].push_back((float)std::ldexp(up * bias, eo));
    }
    double values = 0.0, errors = 0.0;           // of the layer's inputs on a dark stack
    for (size_t c = 0; c < C; ++c) {
      if (dark[c] == 0.0) continue;              // held without error
      values += readers[c] * dark[c] * dark[c];
      errors += readers[c] * std::pow(fine * col[c], 2.0);
    }
    if (errors > std::pow(4.0 * need, 2.0) * values) return false;
    bound = b_out;
    typical = t_out;
    dark = d_out;
    e_in = e_out;
  }
  return true;
}

}  // namespace bcts
