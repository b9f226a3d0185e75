// Dense stages of a convolution of any geometry over slabs [n][ldq] (included by lirpa.hip): one
// backward stage (T^T with the relaxation or the concretisation) and one witness forward stage.
// Operands are split in three bf16 parts as in win_pass.hpp, with the same weight fragments.
//
// A block takes 16 rows q.  The rows of the input map a step needs sit split in an LDS ring,
// [slot][part][x][row][channel], channels padded to eight; the next step's are loaded into
// registers before the step's matrix work and parked after it, one barrier a step.  Each wave
// keeps the fragments of its M tile in registers as long as the tile does not change.
// What bounds them: latency at two waves a SIMD (213 VGPRs with four K steps of fragments): the
// epilogue's loads and stores, four bytes a lane (rows of 16 are half a line), and the LDS reads,
// with 3.7 conflict cycles each.  On the net below the relaxing stage keeps the matrix cores 21 %
// and the VALU 44 % busy at 1.6 TB/s, the concretising one 12 % and 40 % at 1.4.  Measured, 255
// sub-domains of a 28x28 1-16-32-channel net with two rows per neuron: T_2^T of pass 3 70 ms per
// lane, 0.31 here (41 GFLOP), T_1^T 7.4 and 0.22.  Witness forward of the four-convolution net's
// pass 5 (12,800 rows, 8 channels): 0.275 ms a layer with the fp32 kernel of those shapes, 0.18
// here with two columns a tile.

// Input row loader: task = (column x, quad of channels, quad of rows q): four 16-byte loads,
// transposed into four 8-byte stores per part.
struct RowTask {
  float4v v[4];
};
__device__ __forceinline__ void row_fetch(RowTask& t, const float* __restrict__ in, unsigned ldq,
                                          unsigned q0, int task, int Cq, int C, int HW, int y,
                                          int W) {
  const int q4 = task & 3, xc = task >> 2;
  const int cq = xc % Cq, x = xc / Cq;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = 4 * cq + r;
    t.v[r] = float4v{0.f, 0.f, 0.f, 0.f};
    if (c < C)
      t.v[r] = *reinterpret_cast<const float4v*>(
          in + (size_t)(unsigned)(c * HW + y * W + x) * ldq + q0 + 4 * q4);
  }
}
__device__ __forceinline__ void row_park(const RowTask& t, char* slot, int rowb, int task, int Cq) {
  const int q4 = task & 3, xc = task >> 2;
  const int cq = xc % Cq, x = xc / Cq;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    put_split(slot, rowb, ((x * 16 + 4 * q4 + j) * Cq + cq) * 8,
              float4v{t.v[0][j], t.v[1][j], t.v[2][j], t.v[3][j]});
}

struct ConvSplit {
  int C, Cq, H, W;      // input map of the stage (channels in quads)
  int Cd, Cqd, Hd, Wd;  // output map
  int K, s, t, ex, pad, nks, nmt, NS, rowb;  // (ex: FragJob)
  const uint4v* frag;
};

// acc of one (M tile, position): KS > 0 fragments in registers, else read here.
template <int KS, bool SIGN, class Load>
__device__ __forceinline__ float4v conv_dot(const uint4v (&A)[KS ? KS : 1][3], const uint4v* fm,
                                            int nks, Load load) {
  if constexpr (KS > 0) {
    uint4v B[KS][3];
#pragma unroll
    for (int k = 0; k < KS; ++k) load(k, B[k]);
    return win_dot<KS, SIGN>(A, B);
  } else {
    float4v d = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < nks; ++k) {
      uint4v a[1][3], B[1][3];
#pragma unroll
      for (int p = 0; p < 3; ++p) a[0][p] = fm[(k * 3 + p) * 64];
      load(k, B[0]);
      d += win_dot<1, SIGN>(a, B);
    }
    return d;
  }
}

constexpr int kRowTasks = 2;  // prefetched tasks a thread

// T_m^T: output (iy, ix) = (s ay + py - pad, s ex ax + px - pad), inputs (ay - jy,
// ex ax + ex - 1 - jx).
// (SYM: a relaxing stage of a pass with one row per neuron, see Sink)
template <int MODE, int KS, bool SYM>
__global__ void __launch_bounds__(512) k_convT_split(ConvSplit c, const float* __restrict__ in,
                                                     unsigned ldq, unsigned Q, Sink s) {
  extern __shared__ char csm[];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = wave_id(), nw = nt >> 6;
  const int n = lane & 15, G = lane >> 4;
  const unsigned q0 = xcd_tile(blockIdx.x) * 16u;
  if (q0 >= Q) return;  // grid padding, uniform per block
  const unsigned q = q0 + n;
  const bool qok = q < Q;
  const unsigned b = qok ? q / (unsigned)s.R : 0u;
  const long pb = (long)b * s.pstride;
  const int slotb = 3 * c.rowb, NS = c.NS, c2 = c.Cq / 2;
  float* red = reinterpret_cast<float*>(csm + NS * slotb);  // [nw][4][16]
  for (int e = tid; e < NS * 3; e += nt)  // the zero chunk that ends each part of a row
    *reinterpret_cast<uint4v*>(csm + (e + 1) * c.rowb - 16) = uint4v{0, 0, 0, 0};
  const int ntask = c.W * c.Cq * 4, HW = c.H * c.W;
  RowTask pf[kRowTasks];
  auto fetch = [&](int y) {
    if (y < c.H)
#pragma unroll
      for (int k = 0; k < kRowTasks; ++k)
        if (tid + k * nt < ntask) row_fetch(pf[k], in, ldq, q0, tid + k * nt, c.Cq, c.C, HW, y, c.W);
  };
  auto park = [&](int y) {
    if (y >= c.H) return;
    char* slot = csm + (y % NS) * slotb;
#pragma unroll
    for (int k = 0; k < kRowTasks; ++k)
      if (tid + k * nt < ntask) row_park(pf[k], slot, c.rowb, tid + k * nt, c.Cq);
    for (int e = tid + kRowTasks * nt; e < ntask; e += nt) {
      RowTask r;
      row_fetch(r, in, ldq, q0, e, c.Cq, c.C, HW, y, c.W);
      row_park(r, slot, c.rowb, e, c.Cq);
    }
  };
  fetch(0);
  park(0);
  __syncthreads();

  const int sx = c.s * c.ex, tx = c.t + c.ex - 1;
  const int nay = (c.Hd - 1 + c.pad) / c.s + 1, nax = (c.Wd - 1 + c.pad) / sx + 1;
  // M tiles dealt to the waves; with fewer tiles than waves, nw / nmt waves share a tile's columns
  const int share = nw / c.nmt > 1 ? nw / c.nmt : 1;
  const int mt0 = wave / share, xs0 = wave - mt0 * share, mstep = (nw + share - 1) / share;
  RowBias<SYM> rb;
  float lin = 0.f, l1 = 0.f;
  uint4v A[KS ? KS : 1][3];
  int cur = -1;
  for (int ay = 0; ay < nay; ++ay) {
    fetch(ay + 1);
    const int sy = ay % NS;
    for (int mt = mt0; mt < c.nmt; mt += mstep) {
      const uint4v* fm = c.frag + (size_t)mt * c.nks * 192 + lane;
      if constexpr (KS > 0) {
        if (mt != cur) {
          cur = mt;
#pragma unroll
          for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int p = 0; p < 3; ++p) A[k][p] = fm[(k * 3 + p) * 64];
        }
      }
      const int qd = mt * 4 + G, ph = qd / c.Cqd, cq = qd - ph * c.Cqd;
      const int iy = c.s * ay + ph / sx - c.pad;
      const bool oky = ph < c.s * sx && iy >= 0 && iy < c.Hd && qok;
      for (int ax = xs0; ax < nax; ax += share) {
        const int ix = sx * ax + ph % sx - c.pad;
        const bool ok = oky && ix >= 0 && ix < c.Wd;
        unsigned i[4];
        float lo[4], up[4], bu[4], bz[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          i[r] = ((unsigned)(4 * cq + r) * c.Hd + iy) * c.Wd + ix;
          lo[r] = up[r] = bu[r] = bz[r] = 0.f;
          if constexpr (MODE == MODE_SLAB) {
            if (ok && 4 * cq + r < c.Cd) {
              lo[r] = s.a_lo[pb + i[r]];
              up[r] = s.a_up[pb + i[r]];
              bu[r] = s.b_up[pb + i[r]];
              bz[r] = s.bias[i[r]];
            }
          }
        }
        const float4v d = conv_dot<KS, false>(A, fm, c.nks, [&](int ks, uint4v (&B)[3]) {
          const int ck = ks * 4 + G, j = ck / c2, cc = ck - j * c2;
          const int jy = j / tx, yy = ay - jy, xx = c.ex * ax + (c.ex - 1) - (j - jy * tx);
          const bool in_ = j < c.t * tx && yy >= 0 && yy < c.H && xx >= 0 && xx < c.W;
          int sl = sy - jy;
          sl += sl < 0 ? NS : 0;
          const int o = in_ ? sl * slotb + ((xx * 16 + n) * c2 + cc) * 16 : c.rowb - 16;
#pragma unroll
          for (int p = 0; p < 3; ++p) B[p] = *reinterpret_cast<const uint4v*>(csm + o + p * c.rowb);
        });
        if (!ok) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (4 * cq + r >= c.Cd) continue;
          const float a = d[r];
          const unsigned idx = i[r] * ldq + q;
          if constexpr (MODE == MODE_SLAB) {
            if (s.tape) s.tape[idx] = a;
            const float ah = a * rb.slope(a, lo[r], up[r]);
            rb.add_any(a, ah, bu[r], bz[r]);
            s.out[idx] = ah;
          } else {
            if (s.tsign) s.tsign[idx] = sign8(a);
            if (s.x0) lin = fmaf(a, s.x0[i[r]], lin);
            l1 += fabsf(a);
          }
        }
      }
    }
    park(ay + 1);
    __syncthreads();
  }
  float beta = rb.lo, up = 0.f;
  if constexpr (SYM) {
    up = rb.up;
    up += __shfl_xor(up, 16, 64);
    up += __shfl_xor(up, 32, 64);
  }
  beta += __shfl_xor(beta, 16, 64);
  lin += __shfl_xor(lin, 16, 64);
  l1 += __shfl_xor(l1, 16, 64);
  beta += __shfl_xor(beta, 32, 64);
  lin += __shfl_xor(lin, 32, 64);
  l1 += __shfl_xor(l1, 32, 64);
  if (lane < 16) {
    red[(wave * 4 + 0) * 16 + lane] = beta;
    red[(wave * 4 + 1) * 16 + lane] = lin;
    red[(wave * 4 + 2) * 16 + lane] = l1;
    if constexpr (SYM) red[(wave * 4 + 3) * 16 + lane] = up;
  }
  __syncthreads();
  if (tid >= 16 || !qok) return;
  Acc tot{0.f, 0.f, 0.f};
  for (int w = 0; w < nw; ++w) {
    tot.beta += red[(w * 4 + 0) * 16 + tid];
    tot.lin += red[(w * 4 + 1) * 16 + tid];
    tot.l1 += red[(w * 4 + 2) * 16 + tid];
    if constexpr (SYM) tot.up += red[(w * 4 + 3) * 16 + tid];
  }
  sink_finish<MODE>(s, tot, q, b, q % (unsigned)s.R, false);
}

// Witness forward through a convolution (see k_fwd_mfma).  WITNESS: the input is the sign tape
// and G = z1 - eps W sign (bias = z1); otherwise the z slab and G = b + W z (bias per channel in
// the layout of the relaxation parameters).  part (rows in whole groups of 8 per sub-domain,
// output channels in whole quads): the adjoint sums of each group instead of G, as k_fwd_conv.
template <bool WITNESS, int KS>
__global__ void __launch_bounds__(512)
    k_conv_split(ConvSplit c, const float* __restrict__ in, unsigned ldq, unsigned Q, long R,
                 const float* __restrict__ w, float eps, const float* __restrict__ tape,
                 const float* __restrict__ a_lo, const float* __restrict__ a_up,
                 const float* __restrict__ b_up, const float* __restrict__ bias, long pstride,
                 float* __restrict__ Gs, float* __restrict__ zout, float* __restrict__ part,
                 unsigned char* __restrict__ gflag) {
  extern __shared__ char csm[];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = wave_id(), nw = nt >> 6;
  const int n = lane & 15, G = lane >> 4;
  const unsigned q0 = xcd_tile(blockIdx.x) * 16u;
  if (q0 >= Q) return;  // grid padding, uniform per block
  const unsigned q = q0 + n;
  const bool qok = q < Q;
  const float wq = qok ? w[q] : 0.f;
  if (part) {
    const bool live = __syncthreads_or(wq != 0.f && n < 8) != 0;
    const bool live2 = __syncthreads_or(wq != 0.f && n >= 8) != 0;
    if (tid == 0) {
      gflag[q0 / 8] = live ? 1 : 0;
      gflag[q0 / 8 + 1] = live2 ? 1 : 0;
    }
  }
  if (__syncthreads_or(wq != 0.f) == 0) return;  // uniform: the whole block is idle
  const unsigned b = qok ? q / (unsigned)R : 0u;
  const long pb = (long)b * pstride;
  constexpr int NPL = WITNESS ? 1 : 3;
  const int slotb = NPL * c.rowb, NS = c.NS, c2 = c.Cq / 2, HW = c.H * c.W;
  if constexpr (!WITNESS)
    for (int e = tid; e < NS * 3; e += nt)
      *reinterpret_cast<uint4v*>(csm + (e + 1) * c.rowb - 16) = uint4v{0, 0, 0, 0};
  const int ntask = c.W * c.Cq * 4;
  RowTask pf[2];
  const int8_t* sg = reinterpret_cast<const int8_t*>(in);
  // sign rows: the four channels' words of four rows each, transposed bytewise
  auto sfetch = [&](RowTask& t, int task, int y) {
    const int q4 = task & 3, xc = task >> 2, cq = xc % c.Cq, x = xc / c.Cq;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      unsigned u = 0;
      if (4 * cq + r < c.C)
        u = *reinterpret_cast<const unsigned*>(
            sg + (size_t)(unsigned)((4 * cq + r) * HW + y * c.W + x) * ldq + q0 + 4 * q4);
      t.v[0][r] = __builtin_bit_cast(float, u);
    }
  };
  auto spark = [&](const RowTask& t, char* slot, int task) {
    const int q4 = task & 3, xc = task >> 2, cq = xc % c.Cq, x = xc / c.Cq;
    unsigned u[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // +1 -> 0x40, -1 -> 0xc0, 0 -> 0 per byte: the high byte of a bf16 +-2
      // (a scalar first: a bit cast of a vector element reads element 0)
      const float f = t.v[0][r];
      const unsigned v = __builtin_bit_cast(unsigned, f);
      u[r] = ((v & 0x01010101u) << 6) | (v & 0x80808080u);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned o = ((u[0] >> (8 * j)) & 0xffu) | (((u[1] >> (8 * j)) & 0xffu) << 8) |
                         (((u[2] >> (8 * j)) & 0xffu) << 16) | (((u[3] >> (8 * j)) & 0xffu) << 24);
      *reinterpret_cast<unsigned*>(slot + ((x * 16 + 4 * q4 + j) * c.Cq + cq) * 4) = o;
    }
  };
  auto load_row = [&](RowTask& t, int e, int y) {
    if constexpr (WITNESS) sfetch(t, e, y);
    else row_fetch(t, in, ldq, q0, e, c.Cq, c.C, HW, y, c.W);
  };
  auto put_row = [&](const RowTask& t, char* slot, int e) {
    if constexpr (WITNESS) spark(t, slot, e);
    else row_park(t, slot, c.rowb, e, c.Cq);
  };
  auto fetch = [&](RowTask& t, int y) {  // this thread's first task of input row y
    if (y >= 0 && y < c.H && tid < ntask) load_row(t, tid, y);
  };
  auto park = [&](const RowTask& t, int y) {  // ... into the ring, with its other tasks
    if (y < 0 || y >= c.H) return;
    char* slot = csm + (y % NS) * slotb;
    if (tid < ntask) put_row(t, slot, tid);
    for (int e = tid + nt; e < ntask; e += nt) {
      RowTask r;
      load_row(r, e, y);
      put_row(r, slot, e);
    }
  };
  for (int y = -c.pad; y < c.K - c.pad; ++y) {
    fetch(pf[0], y);
    park(pf[0], y);
  }
  __syncthreads();
  const int share = nw / c.nmt > 1 ? nw / c.nmt : 1;
  const int mt0 = wave / share, xs0 = wave - mt0 * share, mstep = (nw + share - 1) / share;
  const int npos = c.Hd * c.Wd;
  const bool fz = (zout || part) && qok && wq != 0.f;
  uint4v A[KS ? KS : 1][3];
  int cur = -1;
  for (int oy = 0; oy < c.Hd; ++oy) {
    // the rows output row oy + 1 adds: the first two in flight over the matrix work
    const int yn = oy * c.s - c.pad + c.K, y1 = oy + 1 < c.Hd ? c.s : 0;
    if (y1 > 0) fetch(pf[0], yn);
    if (y1 > 1) fetch(pf[1], yn + 1);
    for (int mt = mt0; mt < c.nmt; mt += mstep) {
      const uint4v* fm = c.frag + (size_t)mt * c.nks * 192 + lane;
      if constexpr (KS > 0) {
        if (mt != cur) {
          cur = mt;
#pragma unroll
          for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int p = 0; p < 3; ++p) A[k][p] = fm[(k * 3 + p) * 64];
        }
      }
      const int qd = mt * 4 + G, ph = qd / c.Cqd, cq = qd - ph * c.Cqd;
      const int kw = c.K + c.s * (c.ex - 1), nbx = (c.Wd + c.ex - 1) / c.ex;
      for (int bx = xs0; bx < nbx; bx += share) {
        const int ox = c.ex * bx + ph;
        const bool okx = ph < c.ex && ox < c.Wd;  // (the same for the lanes a sum runs over)
        float lo[4], up[4], bu[4], bz[4], tp[4];
        unsigned i[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int co = 4 * cq + r;
          i[r] = ((unsigned)co * c.Hd + oy) * c.Wd + ox;
          lo[r] = up[r] = bu[r] = bz[r] = tp[r] = 0.f;
          if (co < c.Cd && qok && okx) {
            bz[r] = bias[i[r]];
            if (fz) tp[r] = tape[(size_t)i[r] * ldq + q];
            if (fz && zout) {
              lo[r] = a_lo[pb + i[r]];
              up[r] = a_up[pb + i[r]];
              bu[r] = b_up[pb + i[r]];
            }
          }
        }
        const float4v d = conv_dot<KS, WITNESS>(A, fm, c.nks, [&](int ks, uint4v (&B)[3]) {
          if constexpr (WITNESS) {
            uint4v v;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int qi = (ks * 4 + G) * 2 + h, tap = qi / c.Cq, cc = qi - tap * c.Cq;
              const int ky = tap / kw, yy = oy * c.s - c.pad + ky;
              const int xx = c.ex * bx * c.s - c.pad + tap - ky * kw;
              const bool in_ = tap < c.K * kw && yy >= 0 && yy < c.H && xx >= 0 && xx < c.W;
              const int o = in_ ? (yy % NS) * slotb + ((xx * 16 + n) * c.Cq + cc) * 4 : 0;
              const unsigned u = in_ ? *reinterpret_cast<const unsigned*>(csm + o) : 0u;
              v[2 * h] = __builtin_amdgcn_perm(u, 0u, 0x05000400u);
              v[2 * h + 1] = __builtin_amdgcn_perm(u, 0u, 0x07000600u);
            }
            B[0] = v;
            B[1] = v;
            B[2] = v;
          } else {
            const int ck = ks * 4 + G, tap = ck / c2, cc = ck - tap * c2;
            const int ky = tap / kw, yy = oy * c.s - c.pad + ky;
            const int xx = c.ex * bx * c.s - c.pad + tap - ky * kw;
            const bool in_ = tap < c.K * kw && yy >= 0 && yy < c.H && xx >= 0 && xx < c.W;
            const int o = in_ ? (yy % NS) * slotb + ((xx * 16 + n) * c2 + cc) * 16 : c.rowb - 16;
#pragma unroll
            for (int p = 0; p < 3; ++p)
              B[p] = *reinterpret_cast<const uint4v*>(csm + o + p * c.rowb);
          }
        });
        const float gs = WITNESS ? -0.5f * eps : 1.f;  // (the signs are stored as +-2)
        float gv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) gv[r] = fmaf(gs, d[r], bz[r]);
        if (part) {
          float4v sa, da, db;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float tpos = fmaxf(tp[r], 0.f), tneg = fminf(tp[r], 0.f);
            sa[r] = sum8(fz ? (wq * tpos) * gv[r] : 0.f);
            da[r] = sum8(fz ? (wq * tneg) * gv[r] : 0.f);
            db[r] = sum8(fz ? wq * tneg : 0.f);
          }
          if ((n & 7) == 0 && 4 * cq < c.Cd && okx) {
            float* dst = part + (size_t)(q0 / 8 + (n >> 3)) * 3 * (npos * c.Cd) +
                         (size_t)(oy * c.Wd + ox) * c.Cd + 4 * cq;
            *reinterpret_cast<float4v*>(dst) = sa;
            *reinterpret_cast<float4v*>(dst + npos * c.Cd) = da;
            *reinterpret_cast<float4v*>(dst + 2 * npos * c.Cd) = db;
          }
        }
        if (!qok || wq == 0.f || !okx) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (4 * cq + r >= c.Cd) continue;
          const size_t idx = (size_t)i[r] * ldq + q;
          if (!part) Gs[idx] = gv[r];
          if (zout) zout[idx] = tp[r] >= 0.f ? lo[r] * gv[r] : fmaf(up[r], gv[r], bu[r]);
        }
      }
    }
    if (y1 > 0) park(pf[0], yn);
    if (y1 > 1) park(pf[1], yn + 1);
    for (int j = 2; j < y1; ++j) {
      RowTask r;
      fetch(r, yn + j);
      park(r, yn + j);
    }
    __syncthreads();
  }
}
