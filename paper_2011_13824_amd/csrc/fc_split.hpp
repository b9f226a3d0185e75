// Fully connected stages on split operands (included by lirpa.hip, after win_pass.hpp): the
// backward stage T^T with its relaxation or concretisation, and the witness forward over x.
//
// A block holds NT tiles of 16 rows q: their inputs stay split in LDS for the whole kernel
// ([chunk of 8 inputs][row], 16 bytes a part), and the waves take two tiles of 16 outputs at a
// time, streaming the weight fragments from the cache one K step ahead.  Two output tiles per
// operand read keep the LDS at half its rate; NT = 4 row tiles per fragment read keep the cache
// at a quarter of its own.  Measured on a 784-256 layer and 102,400 rows (41 GFLOP): T^T with its
// sign tape 1.03 ms with the fp32 kernel, 0.31 here (0.25 without the tape; matrix cores 35 % and
// VALU 23 % busy, 1.9 conflict cycles an LDS read, 0.7 TB/s: latency at three waves a SIMD);
// witness forward 2.61 and 0.26 (21 %, 26 %, 3.8, 1.1 TB/s).

constexpr int kFcThreads = 512;

struct FcSplit {
  int nin, nout;  // of the stage: inputs (K), outputs (M)
  int nks, nmt;
  int plane;      // bytes of one part of the panel
  const uint4v* frag;
};

// T^T: out[i] = sum_o W[o][i] in[o].  (SYM: a relaxing stage of a pass with one row per neuron,
// see Sink)
template <int MODE, int NT, bool SYM>
__global__ void __launch_bounds__(kFcThreads)
    k_fcT_split(FcSplit c, const float* __restrict__ in, unsigned ldq, unsigned Q, Sink s) {
  extern __shared__ char fsm[];
  constexpr int NQ = 16 * NT, NW = kFcThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), n = lane & 15, G = lane >> 4;
  const unsigned q0 = xcd_range(blockIdx.x) * (unsigned)NQ;
  if (q0 >= Q) return;  // grid padding, uniform per block
  float* red = reinterpret_cast<float*>(fsm + 3 * c.plane);  // [NW][4][NQ]
  for (int e = tid; e < c.nks * 8 * (NQ / 4); e += kFcThreads) {
    const int q4 = e % (NQ / 4), k4 = e / (NQ / 4);  // four inputs of four rows
    float4v v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 4 * k4 + r;
      v[r] = float4v{0.f, 0.f, 0.f, 0.f};
      if (o < c.nin) v[r] = *reinterpret_cast<const float4v*>(in + (size_t)o * ldq + q0 + 4 * q4);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      put_split(fsm, c.plane, (((k4 >> 1) * NQ + 4 * q4 + j) * 2 + (k4 & 1)) * 8,
                float4v{v[0][j], v[1][j], v[2][j], v[3][j]});
  }
  __syncthreads();
  unsigned qn[NT];
  bool qok[NT];
  long pb[NT];
  RowBias<SYM> rb[NT];
  float lin[NT], l1[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    qn[t] = q0 + 16 * t + n;
    qok[t] = qn[t] < Q;
    pb[t] = (long)(qok[t] ? qn[t] / (unsigned)s.R : 0u) * s.pstride;
    lin[t] = l1[t] = 0.f;
  }
  const char* bp = fsm + n * 16;
  for (int mp = wave; 2 * mp < c.nmt; mp += NW) {
    const bool two = 2 * mp + 1 < c.nmt;  // (the last pair may be one tile: it reads it twice)
    const uint4v* f0 = c.frag + (size_t)(2 * mp) * c.nks * 192 + lane;
    const uint4v* f1 = two ? f0 + (size_t)c.nks * 192 : f0;
    float4v hi[2][NT], lo[2][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t) hi[u][t] = lo[u][t] = float4v{0.f, 0.f, 0.f, 0.f};
    uint4v A[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      A[0][p] = f0[p * 64];
      A[1][p] = f1[p * 64];
    }
    for (int k = 0; k < c.nks; ++k) {
      uint4v N[2][3];
      const int kn = k + 1 < c.nks ? k + 1 : k;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        N[0][p] = f0[(kn * 3 + p) * 64];
        N[1][p] = f1[(kn * 3 + p) * 64];
      }
      const char* bk = bp + (size_t)(k * 4 + G) * (NQ * 16);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        uint4v B[3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
          B[p] = *reinterpret_cast<const uint4v*>(bk + p * c.plane + t * 256);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          lo[u][t] = mfma_b(A[u][2], B[0], lo[u][t]);
          lo[u][t] = mfma_b(A[u][0], B[2], lo[u][t]);
          lo[u][t] = mfma_b(A[u][1], B[1], lo[u][t]);
          lo[u][t] = mfma_b(A[u][1], B[0], lo[u][t]);
          lo[u][t] = mfma_b(A[u][0], B[1], lo[u][t]);
          hi[u][t] = mfma_b(A[u][0], B[0], hi[u][t]);
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int p = 0; p < 3; ++p) A[u][p] = N[u][p];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && !two) break;
      const int i0 = (2 * mp + u) * 16 + 4 * G;
      if (i0 >= c.nout) continue;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (!qok[t]) continue;
        const float4v d = hi[u][t] + lo[u][t];
        float4v pl, pu, pc, pz;
        if constexpr (MODE == MODE_SLAB) {
          // (segments of the relaxation are padded to four neurons and 16-byte aligned)
          pl = *reinterpret_cast<const float4v*>(s.a_lo + pb[t] + i0);
          pu = *reinterpret_cast<const float4v*>(s.a_up + pb[t] + i0);
          pc = *reinterpret_cast<const float4v*>(s.b_up + pb[t] + i0);
          pz = *reinterpret_cast<const float4v*>(s.bias + i0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (i0 + r >= c.nout) continue;
          const float a = d[r];
          const size_t idx = (size_t)(unsigned)(i0 + r) * ldq + qn[t];
          if constexpr (MODE == MODE_SLAB) {
            if (s.tape) s.tape[idx] = a;
            const float ah = a * rb[t].slope(a, pl[r], pu[r]);
            rb[t].add(a, fminf(a, 0.f), ah, pc[r], pz[r]);
            s.out[idx] = ah;
          } else {
            if (s.tsign) s.tsign[idx] = sign8(a);
            if (s.x0) lin[t] = fmaf(a, s.x0[i0 + r], lin[t]);
            l1[t] += fabsf(a);
          }
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    float v[4] = {rb[t].lo, lin[t], l1[t], rb[t].up};
#pragma unroll
    for (int e = 0; e < (SYM ? 4 : 3); ++e) {
      v[e] += __shfl_xor(v[e], 16, 64);
      v[e] += __shfl_xor(v[e], 32, 64);
      if (lane < 16) red[(wave * 4 + e) * NQ + 16 * t + lane] = v[e];
    }
  }
  __syncthreads();
  const unsigned q = q0 + tid;
  if (tid >= NQ || q >= Q) return;
  Acc tot{0.f, 0.f, 0.f};
  for (int w = 0; w < NW; ++w) {
    tot.beta += red[(w * 4 + 0) * NQ + tid];
    tot.lin += red[(w * 4 + 1) * NQ + tid];
    tot.l1 += red[(w * 4 + 2) * NQ + tid];
    if constexpr (SYM) tot.up += red[(w * 4 + 3) * NQ + tid];
  }
  sink_finish<MODE>(s, tot, q, q / (unsigned)s.R, q % (unsigned)s.R, false);
}

// Witness forward through a first fully connected layer: G = z1 - eps W sign over the sign
// tape (bias = z1), with the outputs of k_conv_split (part: the adjoint sums of each group of 8
// rows instead of G).  The panel holds the signs as the high bytes of bf16 +-2,
// [quad of inputs][row], four bytes each.
template <int NT>
__global__ void __launch_bounds__(kFcThreads)
    k_fc_sign(FcSplit c, const int8_t* __restrict__ sg, unsigned ldq, unsigned Q, long R,
              const float* __restrict__ w, float eps, const float* __restrict__ tape,
              const float* __restrict__ a_lo, const float* __restrict__ a_up,
              const float* __restrict__ b_up, const float* __restrict__ bias, long pstride,
              float* __restrict__ Gs, float* __restrict__ zout, float* __restrict__ part,
              unsigned char* __restrict__ gflag) {
  extern __shared__ char fsm[];
  constexpr int NQ = 16 * NT, NW = kFcThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), n = lane & 15, G = lane >> 4;
  const unsigned q0 = xcd_range(blockIdx.x) * (unsigned)NQ;
  if (q0 >= Q) return;  // grid padding, uniform per block
  // the rows' weights; a group of 8 rows without any only writes its flag
  const unsigned qw = q0 + (lane & (NQ - 1));
  const float wl = qw < Q ? w[qw] : 0.f;
  const unsigned long long live = __ballot(wl != 0.f);
  if (part && tid < NQ / 8) gflag[q0 / 8 + tid] = (live >> (8 * tid)) & 0xffull ? 1 : 0;
  if (live == 0) return;  // uniform: every wave sees the same rows
  for (int e = tid; e < c.nks * 8 * (NQ / 4); e += kFcThreads) {
    const int q4 = e % (NQ / 4), k4 = e / (NQ / 4);
    unsigned u[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 4 * k4 + r;
      unsigned v = 0;
      if (o < c.nin)
        v = *reinterpret_cast<const unsigned*>(sg + (size_t)o * ldq + q0 + 4 * q4);
      u[r] = ((v & 0x01010101u) << 6) | (v & 0x80808080u);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<unsigned*>(fsm + (k4 * NQ + 4 * q4 + j) * 4) =
          ((u[0] >> (8 * j)) & 0xffu) | (((u[1] >> (8 * j)) & 0xffu) << 8) |
          (((u[2] >> (8 * j)) & 0xffu) << 16) | (((u[3] >> (8 * j)) & 0xffu) << 24);
  }
  __syncthreads();
  unsigned qn[NT];
  float wq[NT];
  long pb[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    qn[t] = q0 + 16 * t + n;
    wq[t] = qn[t] < Q ? w[qn[t]] : 0.f;
    pb[t] = (long)(qn[t] < Q ? qn[t] / (unsigned)R : 0u) * pstride;
  }
  for (int mp = wave; 2 * mp < c.nmt; mp += NW) {
    const bool two = 2 * mp + 1 < c.nmt;
    const uint4v* f0 = c.frag + (size_t)(2 * mp) * c.nks * 192 + lane;
    const uint4v* f1 = two ? f0 + (size_t)c.nks * 192 : f0;
    float4v hi[2][NT], lo[2][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t) hi[u][t] = lo[u][t] = float4v{0.f, 0.f, 0.f, 0.f};
    uint4v A[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      A[0][p] = f0[p * 64];
      A[1][p] = f1[p * 64];
    }
    for (int k = 0; k < c.nks; ++k) {
      uint4v N[2][3];
      const int kn = k + 1 < c.nks ? k + 1 : k;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        N[0][p] = f0[(kn * 3 + p) * 64];
        N[1][p] = f1[(kn * 3 + p) * 64];
      }
      const char* bk = fsm + (size_t)((k * 4 + G) * 2 * NQ + n) * 4;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        uint4v B;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const unsigned v = *reinterpret_cast<const unsigned*>(bk + (h * NQ + 16 * t) * 4);
          B[2 * h] = __builtin_amdgcn_perm(v, 0u, 0x05000400u);
          B[2 * h + 1] = __builtin_amdgcn_perm(v, 0u, 0x07000600u);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          lo[u][t] = mfma_b(A[u][2], B, lo[u][t]);
          lo[u][t] = mfma_b(A[u][1], B, lo[u][t]);
          hi[u][t] = mfma_b(A[u][0], B, hi[u][t]);
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int p = 0; p < 3; ++p) A[u][p] = N[u][p];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && !two) break;
      const int i0 = (2 * mp + u) * 16 + 4 * G;
      const bool ok = i0 < c.nout;
      float4v bz = {0.f, 0.f, 0.f, 0.f};
      if (ok) bz = *reinterpret_cast<const float4v*>(bias + i0);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bool on = wq[t] != 0.f && ok;
        const float4v d = hi[u][t] + lo[u][t];
        float4v pl = {0.f, 0.f, 0.f, 0.f}, pu = pl, pc = pl, sa = pl, da = pl, db = pl;
        if (zout && on) {
          pl = *reinterpret_cast<const float4v*>(a_lo + pb[t] + i0);
          pu = *reinterpret_cast<const float4v*>(a_up + pb[t] + i0);
          pc = *reinterpret_cast<const float4v*>(b_up + pb[t] + i0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool onr = on && i0 + r < c.nout;
          const float gv = fmaf(-0.5f * eps, d[r], bz[r]);  // (the signs are stored as +-2)
          const size_t idx = (size_t)(unsigned)(i0 + r) * ldq + qn[t];
          float tp = 0.f;
          if (onr && (zout || part)) tp = tape[idx];
          if (onr && zout) zout[idx] = tp >= 0.f ? pl[r] * gv : fmaf(pu[r], gv, pc[r]);
          if (onr && !part) Gs[idx] = gv;
          const float tpos = fmaxf(tp, 0.f), tneg = fminf(tp, 0.f);
          sa[r] = onr ? (wq[t] * tpos) * gv : 0.f;
          da[r] = onr ? (wq[t] * tneg) * gv : 0.f;
          db[r] = onr ? wq[t] * tneg : 0.f;
        }
        if (part) {  // (every lane takes part in the sums)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            sa[r] = sum8(sa[r]);
            da[r] = sum8(da[r]);
            db[r] = sum8(db[r]);
          }
          if ((n & 7) == 0 && ok) {  // (outputs in whole quads)
            float* dst = part + (size_t)(q0 / 8 + 2 * t + (n >> 3)) * 3 * c.nout + i0;
            *reinterpret_cast<float4v*>(dst) = sa;
            *reinterpret_cast<float4v*>(dst + c.nout) = da;
            *reinterpret_cast<float4v*>(dst + 2 * c.nout) = db;
          }
        }
      }
    }
  }
}
