// Operands split in three bf16 parts: the split itself and the weight fragments every split kernel
// reads (included by lirpa.hip, ahead of k_setup, which writes them).

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));

// Two floats as a pair of bf16 (round to nearest even), the first in the low half.
__device__ __forceinline__ unsigned pk_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(float2v{a, b}, bf16x2));
}

// The three bf16 parts of a pair of floats.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& m,
                                           unsigned& l) {
  h = pk_bf16(a, b);
  a -= __builtin_bit_cast(float, h << 16);
  b -= __builtin_bit_cast(float, h & 0xffff0000u);
  m = pk_bf16(a, b);
  a -= __builtin_bit_cast(float, m << 16);
  b -= __builtin_bit_cast(float, m & 0xffff0000u);
  l = pk_bf16(a, b);
}

// Split weights of one layer in the order of the matrix operand: dst[(mt ks + k) 3 + part][lane],
// 8 bf16 each, for M tile mt and K step k.  Lane l holds row mt 16 + l % 16, entries
// 8 (l / 16) .. + 7 of the step's 32.
//   kind 0, T^T:  row (phase py s ex + px, input channel ci of 4 Cqi), entry (j = jy tx + jx,
//                 output channel of 4 Cqo); ex = 2 (unit stride, 8 channels or fewer) takes two
//                 neighbouring output columns as phases, over tx = t + 1 input columns, so that
//                 the tile's 16 rows are used;
//   kind 1, T:    row (column phase p, output channel of 4 Cqo), entry (tap ky kw + kx, input
//                 channel of 4 Cqi), kw = k + s (ex - 1); ex = 2 (8 channels or fewer) takes two
//                 neighbouring output columns, the second at the taps from kx = s on.
struct FragJob {
  const float* W;  // [out_c][in_c][k][k]
  int in_c, out_c, k, s, t, ex, Cqi, Cqo, kind, nmt, nks, blk;
  uint4v* dst;
};
constexpr int kFragJobs = 16;  // in one launch

// Entry idx = (M tile, K step, lane) of a job.
template <class Job>
__device__ __forceinline__ void frag_entry(const Job& f, int idx) {
  const int lane = idx & 63, step = idx >> 6;
  const int mt = step / f.nks, ks = step - mt * f.nks;
  const int M = mt * 16 + (lane & 15);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int kk = ks * 32 + (lane >> 4) * 8 + e;
    v[e] = 0.f;
    if (f.kind == 0) {
      const int ci = M % (4 * f.Cqi), ph = M / (4 * f.Cqi);
      const int co = kk % (4 * f.Cqo), j = kk / (4 * f.Cqo);
      const int sx = f.s * f.ex, tx = f.t + f.ex - 1;
      const int ky = ph / sx + f.s * (j / tx), kx = ph % sx + f.s * (j % tx - (f.ex - 1));
      if (ph < f.s * sx && j < f.t * tx && ci < f.in_c && co < f.out_c && ky < f.k && kx >= 0 &&
          kx < f.k)
        v[e] = f.W[(((long)co * f.in_c + ci) * f.k + ky) * f.k + kx];
    } else {
      const int ci = kk % (4 * f.Cqi), tap = kk / (4 * f.Cqi), kw = f.k + f.s * (f.ex - 1);
      const int co = M % (4 * f.Cqo), p = M / (4 * f.Cqo);
      const int ky = tap / kw, kx = tap % kw - f.s * p;
      if (co < f.out_c && p < f.ex && ky < f.k && kx >= 0 && kx < f.k && ci < f.in_c)
        v[e] = f.W[(((long)co * f.in_c + ci) * f.k + ky) * f.k + kx];
    }
  }
  uint4v h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    unsigned a, b, c;
    split_pair(v[2 * e], v[2 * e + 1], a, b, c);
    h[e] = a;
    m[e] = b;
    l[e] = c;
  }
  uint4v* d = f.dst + (size_t)step * 192 + lane;
  d[0] = h;
  d[64] = m;
  d[128] = l;
}
