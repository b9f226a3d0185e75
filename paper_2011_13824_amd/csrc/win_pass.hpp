// Receptive-field passes of a chain of convolutions, any geometry (included by lirpa.hip).
//
// A pass that opens at a convolution k (rows +-e_j over h^(k)) only ever touches, on each map
// g^(m) below, the square window its neuron can see: side w_(k-1) = K_k,
// w_(m-1) = (w_m - 1) s_m + K_m, origin y S_m - P_m for position y.  One block takes 16 rows of
// one position of one sub-domain and carries them from W_k to the bounds without leaving LDS;
// the reverse sweep rebuilds the same coefficients, runs the rows' witnesses forward over the
// same windows and sums the 16 rows' adjoint terms per window neuron.
//
// Arithmetic.  The contractions run on bf16 matrix cores with every fp32 operand split into
// three bf16 parts (8 + 8 + 8 bits, round to nearest, which hold the fp32 value) and the six
// products of weight >= 2^-16 accumulated in fp32, the leading product on its own accumulator.
// Measured on normal data against 64-bit sums: relative error 0.6e-7 / 1.5e-7 / 2.9e-7 at
// K = 64 / 512 / 2048, where the fp32 matrix instruction gives 1.4e-7 / 3.9e-7 / 8.1e-7; and
// 358 TFLOP/s of fp32 products instead of 139.  A witness sign is exact in bf16, so the
// forward step over x takes three products.
//
// T_m^T in gather form: output i = s a + p of the window below takes the taps
// ky = p + s j of the inputs a - j, j < t = ceil(K / s), for every phase p < s alike.  So one
// GEMM per block position a serves all s^2 phases: M = (phase, input channel of T_m),
// K = (tap pair j, output channel), N = the 16 rows.
//
// What bounds it: instructions, the relaxation and split of every window entry and the operand
// addresses before the matrix work (VALU 78 % and matrix cores 20 % of the SIMD cycles in the bound
// of a 28x28 net's pass 2, 65 and 16 in the reverse sweep of the four-convolution net's pass 3, 49
// and 13 in its pass 4; LDS reads with 1 to 2.6 conflict cycles each; a block of that net's pass 3
// issues about 1,700 per wave beside 120 matrix instructions; more positions in flight change
// nothing).  In its pass 4 also the LDS, 108 KB for a bound and 153 KB for the reverse sweep: one
// block of eight waves a CU, where the registers would hold two.
// Measured (ms, before and after): 64 sub-domains of the four-convolution net, ten reverse sweeps
// of passes 3 and 4 with their bounds, dense slabs 209, here 12.2; 255 sub-domains of a 28x28
// 1-16-32-channel net, pass 2, per-lane gathers 57, here 0.215 (0.127 with one row per neuron).

constexpr int kWinMax = 6;   // most layers below the pass's own
constexpr int kWinLds = 160 * 1024;

__device__ __forceinline__ float4v mfma_b(uint4v a, uint4v b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// One map of the chain.  Index m = 0 is x; T_m leads from g^(m) down to g^(m-1).
struct WinLayer {
  int w, H, W;      // window side; map
  int Cq;           // channels in quads of four (m >= 1: an even number of quads)
  int C;
  int S, P;         // window origin y S - P
  int K, s, t;      // of T_m
  int ex, exf;      // output columns a position of T_m^T, T_m takes (FragJob)
  int nks, nmt;     // T_m^T fragments
  const uint4v* fb;
  int nksf, nmtf;   // T_m fragments
  const uint4v* ff;
  int o_prm;        // LDS: float4 (a_lo, a_up, b_up, bias) per (position, channel)
  int o_pl, plane;  // LDS: split coefficients [part][position][row][channel], bytes per part
  int o_at;         // LDS, reverse sweep: coefficients before relaxation, [position][quad][row][4]
  long poff, noff;
  int part;         // reverse sweep: offset of this map's sums in a block's partial sums
};
struct WinDesc {
  int k;            // the pass
  int H, W, C, G;   // h^(k); groups of rows per position
  int K;            // of T_k
  int nwin;         // windows a block (SYM)
  const float* Wk;
  const float* bk;
  int o_red, o_x;   // LDS: reductions; reverse sweep: signs of A_x, [position][row][quad][4] bytes
  int npart;        // partial sums per block
  WinLayer L[kWinMax];
};
struct WinArgs {
  const float* a_lo;
  const float* a_up;
  const float* b_up;
  const float* bias;
  long pstride, n_relu, noff_k;
  float eps;
  float* lo;        // bounds of the chunk (whole rows of n_relu)
  float* hi;
  const float* gl;  // adjoints of the bounds (whole rows)
  const float* gu;
  float* part;
  unsigned char* pflag;
};

// acc = sum over the K steps of A B, both split in three.
template <int KS, bool SIGN>
__device__ __forceinline__ float4v win_dot(const uint4v (&A)[KS][3], const uint4v (&B)[KS][3]) {
  float4v hi = {0.f, 0.f, 0.f, 0.f}, lo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    lo = mfma_b(A[k][2], B[k][0], lo);
    if constexpr (!SIGN) {
      lo = mfma_b(A[k][0], B[k][2], lo);
      lo = mfma_b(A[k][1], B[k][1], lo);
    }
    lo = mfma_b(A[k][1], B[k][0], lo);
    if constexpr (!SIGN) lo = mfma_b(A[k][0], B[k][1], lo);
    hi = mfma_b(A[k][0], B[k][0], hi);
  }
  return hi + lo;
}

// Every (M tile, position) of a stage: positions ny x nx dealt to the waves, an M tile's
// fragments held in registers over them.  load(ks, y, x, B) fetches this lane's B operand of
// a K step; emit(mt, y, x, d) takes the 4 x 1 results of a lane.
template <int KS, bool SIGN, class Load, class Emit>
__device__ __forceinline__ void win_tiles(const uint4v* __restrict__ frag, int nmt, int ny, int nx,
                                          int wave, int nw, Load load, Emit emit) {
  const int lane = threadIdx.x & 63;
  for (int mt = 0; mt < nmt; ++mt) {
    const uint4v* fm = frag + (size_t)mt * KS * 192 + lane;
    uint4v A[KS][3];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int p = 0; p < 3; ++p) A[k][p] = fm[(k * 3 + p) * 64];
    int y = 0, x = wave;
    while (x >= nx) {
      x -= nx;
      ++y;
    }
    while (y < ny) {
      uint4v B[KS][3];
#pragma unroll
      for (int k = 0; k < KS; ++k) load(k, y, x, B[k]);
      emit(mt, y, x, win_dot<KS, SIGN>(A, B));
      x += nw;
      while (x >= nx) {
        x -= nx;
        ++y;
      }
    }
  }
}

// The same for any number of K steps, the fragments read again at every position.
template <bool SIGN, class Load, class Emit>
__device__ __forceinline__ void win_tiles_any(const uint4v* __restrict__ frag, int nmt, int nks,
                                              int ny, int nx, int wave, int nw, Load load,
                                              Emit emit) {
  const int lane = threadIdx.x & 63;
  for (int it = wave; it < nmt * ny * nx; it += nw) {
    const int mt = it % nmt, pos = it / nmt;
    const int y = pos / nx, x = pos - y * nx;
    const uint4v* fm = frag + (size_t)mt * nks * 192 + lane;
    float4v d = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < nks; ++k) {
      uint4v A[1][3], B[1][3];
#pragma unroll
      for (int p = 0; p < 3; ++p) A[0][p] = fm[(k * 3 + p) * 64];
      load(k, y, x, B[0]);
      d += win_dot<1, SIGN>(A, B);
    }
    emit(mt, y, x, d);
  }
}

// (MAXKS: the most K steps whose fragments the kernel's registers hold)
template <int MAXKS, bool SIGN, class Load, class Emit>
__device__ __forceinline__ void win_stage(const uint4v* __restrict__ frag, int nmt, int nks, int ny,
                                          int nx, int wave, int nw, Load load, Emit emit) {
  switch (nks) {
    case 1: return win_tiles<1, SIGN>(frag, nmt, ny, nx, wave, nw, load, emit);
    case 2: return win_tiles<2, SIGN>(frag, nmt, ny, nx, wave, nw, load, emit);
    case 3:
      if constexpr (MAXKS >= 3) return win_tiles<3, SIGN>(frag, nmt, ny, nx, wave, nw, load, emit);
      break;
    case 4:
      if constexpr (MAXKS >= 4) return win_tiles<4, SIGN>(frag, nmt, ny, nx, wave, nw, load, emit);
      break;
    default:
      if constexpr (MAXKS >= 4)
        return win_tiles_any<SIGN>(frag, nmt, nks, ny, nx, wave, nw, load, emit);
  }
}

// Splits a lane's four values (consecutive channels) and stores them at byte `o` of the planes.
__device__ __forceinline__ void put_split(char* pl, int plane, int o, const float4v& v) {
  unsigned h0, m0, l0, h1, m1, l1;
  split_pair(v[0], v[1], h0, m0, l0);
  split_pair(v[2], v[3], h1, m1, l1);
  *reinterpret_cast<uint2v*>(pl + o) = uint2v{h0, h1};
  *reinterpret_cast<uint2v*>(pl + plane + o) = uint2v{m0, m1};
  *reinterpret_cast<uint2v*>(pl + 2 * plane + o) = uint2v{l0, l1};
}

// One pass over the windows.  GRAD = false: the bounds l, u of the block's 8 neurons (rows r
// and r + 8 of a block are +-e_j of channel 8 g + r).  GRAD = true: the reverse sweep of the
// pass; the rows with weight of a position are numbered in the order (channel, sign) and group
// g takes rows 16 g .. 16 g + 15; a block without any stops after its flag.
// SYM (bounds without given slopes): one row per neuron gives both bounds (Sink::up), so the 16
// rows are 16 channels of a position, or, with 8 channels or fewer, those of two neighbouring
// positions (nwin = 2: rows 0-7 and 8-15, each in its own window's coordinates; the windows'
// relaxations stand one behind the other).
template <bool GRAD, bool SYM, int MAXKS>
__global__ void __launch_bounds__(512) k_win_pass(WinDesc d_, WinArgs a) {
  // (kernel arguments are read in place: a by-value struct indexed at run time would be copied
  // to scratch)
  const __attribute__((address_space(4))) WinDesc& d =
      *(const __attribute__((address_space(4))) WinDesc*)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ char wsm[];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = wave_id(), nw = nt >> 6;
  const int n = lane & 15, G = lane >> 4;
  const int nwin = SYM ? d.nwin : 1, nbx = (d.W + nwin - 1) / nwin;  // blocks along x
  const int win = SYM && nwin == 2 ? n >> 3 : 0;  // this row's window
  unsigned blk = xcd_range(blockIdx.x);
  const unsigned blk0 = blk;
  const int px = (int)(blk % (unsigned)nbx) * nwin; blk /= (unsigned)nbx;
  const int py = (int)(blk % (unsigned)d.H); blk /= (unsigned)d.H;
  const int g = (int)(blk % (unsigned)d.G); blk /= (unsigned)d.G;
  const long b = blk;
  const int k = d.k;
  float* red = reinterpret_cast<float*>(wsm + d.o_red);   // [nw][3][16]
  float* wrow = red + nw * 48;                            // GRAD: [16] row weights
  int* rid = reinterpret_cast<int*>(wrow + 16);           // GRAD: [16] 2 channel + (sign -)

  if constexpr (GRAD) {
    if (wave == 0) {
      int base = 0;
      for (int c0 = 0; c0 < 2 * d.C; c0 += 64) {
        const int ci = c0 + lane;
        float wgt = 0.f;
        if (ci < 2 * d.C) {
          const long j = b * a.n_relu + a.noff_k + ((long)(ci >> 1) * d.H + py) * d.W + px;
          wgt = (ci & 1) ? -a.gu[j] : a.gl[j];
        }
        const unsigned long long m = __ballot(wgt != 0.f);
        const int r = base + (int)__builtin_amdgcn_mbcnt_hi(
                                 (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)) -
                      16 * g;
        if (wgt != 0.f && r >= 0 && r < 16) {
          wrow[r] = wgt;
          rid[r] = ci;
        }
        base += __popcll(m);
      }
      if (lane < 16 && 16 * g + lane >= base) {
        wrow[lane] = 0.f;
        rid[lane] = 0;
      }
      if (lane == 0) a.pflag[blk0] = base > 16 * g ? 1 : 0;
      if (lane == 0) reinterpret_cast<int*>(red)[0] = base > 16 * g;
    }
    __syncthreads();
    if (reinterpret_cast<int*>(red)[0] == 0) return;  // uniform
  }

  // the relaxation of every window (zeros outside the maps), and the zero chunk that ends each
  // plane of split coefficients
  for (int m = 1; m < k; ++m) {
    const int w = d.L[m].w, C = d.L[m].C, Cp = 4 * d.L[m].Cq, H = d.L[m].H, W = d.L[m].W;
    const int oy = py * d.L[m].S - d.L[m].P, ox = px * d.L[m].S - d.L[m].P;
    float4v* prm = reinterpret_cast<float4v*>(wsm + d.L[m].o_prm);
    const long pb = b * a.pstride + d.L[m].poff, po = d.L[m].poff;
    const int ent = w * w * Cp;
    for (int e2 = tid; e2 < nwin * ent; e2 += nt) {
      // (columns fastest: neighbouring threads read neighbouring neurons)
      const int wi = SYM && e2 >= ent, e = e2 - wi * ent;
      const int xx = e % w, yy = (e / w) % w, c = e / (w * w);
      const int y = oy + yy, x = ox + xx + wi * d.L[m].S;
      float4v v = {0.f, 0.f, 0.f, 0.f};
      if (c < C && y >= 0 && y < H && x >= 0 && x < W) {
        const long i = ((long)c * H + y) * W + x;
        v = float4v{a.a_lo[pb + i], a.a_up[pb + i], a.b_up[pb + i], a.bias[po + i]};
      }
      prm[wi * ent + (yy * w + xx) * Cp + c] = v;
    }
  }
  __syncthreads();

  // the rows of W_k, relaxed onto g^(k-1): thread = (row, quad of channels of a position)
  RowBias<SYM> rb;
  {
    const int m = k - 1;
    const int w = d.K, Cq = d.L[m].Cq, C = d.L[m].C, plane = d.L[m].plane;
    char* pl = wsm + d.L[m].o_pl;
    const float4v* prm =
        reinterpret_cast<const float4v*>(wsm + d.L[m].o_prm) + win * (w * w * 4 * Cq);
    if (tid < 3) *reinterpret_cast<uint4v*>(pl + (tid + 1) * plane - 16) = uint4v{0, 0, 0, 0};
    const int row = tid & 15;
    int ch;
    float sgn;
    if constexpr (GRAD) {
      ch = rid[row] >> 1;
      sgn = (rid[row] & 1) ? -1.f : 1.f;
    } else if constexpr (SYM) {
      ch = min(nwin == 2 ? row & 7 : 16 * g + row, d.C - 1);
      sgn = 1.f;
    } else {
      ch = min(8 * g + (row & 7), d.C - 1);
      sgn = row >= 8 ? -1.f : 1.f;
    }
    const int ww = w * w;
    const float* wk = d.Wk + (long)ch * C * ww;
    for (int e = tid >> 4; e < ww * Cq; e += nt >> 4) {
      const int cq = e % Cq, pos = e / Cq;
      float4v at, v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = 4 * cq + r;
        at[r] = c < C ? sgn * wk[c * ww + pos] : 0.f;
        const float4v p = prm[pos * 4 * Cq + c];
        v[r] = at[r] * rb.slope(at[r], p[0], p[1]);
        if constexpr (!GRAD) {
          rb.add_any(at[r], v[r], p[2], p[3]);
        }
      }
      put_split(pl, plane, ((pos * 16 + row) * Cq + cq) * 8, v);
      if constexpr (GRAD)
        *reinterpret_cast<float4v*>(wsm + d.L[m].o_at + ((pos * Cq + cq) * 16 + row) * 16) = at;
    }
  }
  __syncthreads();

  // T_m^T down the chain
  float l1 = 0.f;
  for (int m = k - 1; m >= 1; --m) {
    const int w = d.L[m].w, s = d.L[m].s, t = d.L[m].t, Cq = d.L[m].Cq, plane = d.L[m].plane;
    const char* src = wsm + d.L[m].o_pl;
    const int wd = d.L[m - 1].w, Cqd = d.L[m - 1].Cq;
    const int ex = d.L[m].ex, sx = s * ex, tx = t + ex - 1;
    const int na = w + t - 1, nax = (na + ex - 1) / ex;
    const int c2 = Cq / 2;  // 16-byte chunks per (position, row)
    // this lane's chunk of K step ks: tap pair (jy, jx), 8 output channels
    auto load = [&](int ks, int y, int x, uint4v (&B)[3]) {
      const int ck = ks * 4 + G, j = ck / c2, cc = ck - j * c2;
      const int yy = y - j / tx, xx = ex * x + (ex - 1) - j % tx;
      const bool ok = j < t * tx && yy >= 0 && yy < w && xx >= 0 && xx < w;
      const int o = ok ? (((yy * w + xx) * 16 + n) * c2 + cc) * 16 : plane - 16;
#pragma unroll
      for (int p = 0; p < 3; ++p) B[p] = *reinterpret_cast<const uint4v*>(src + p * plane + o);
    };
    if (m > 1) {
      const float4v* prm =
          reinterpret_cast<const float4v*>(wsm + d.L[m - 1].o_prm) + win * (wd * wd * 4 * Cqd);
      char* pl = wsm + d.L[m - 1].o_pl;
      const int pld = d.L[m - 1].plane, oat = d.L[m - 1].o_at;
      if (tid < 3) *reinterpret_cast<uint4v*>(pl + (tid + 1) * pld - 16) = uint4v{0, 0, 0, 0};
      win_stage<MAXKS, false>(d.L[m].fb, d.L[m].nmt, d.L[m].nks, na, nax, wave, nw, load,
                       [&](int mt, int y, int x, const float4v& dv) {
                         const int qd = mt * 4 + G, ph = qd / Cqd, cq = qd - ph * Cqd;
                         const int iy = s * y + ph / sx, ix = sx * x + ph % sx;
                         if (ph >= s * sx || iy >= wd || ix >= wd) return;
                         const int pos = iy * wd + ix;
                         float4v v;
#pragma unroll
                         for (int r = 0; r < 4; ++r) {
                           const float4v p = prm[(pos * Cqd + cq) * 4 + r];
                           v[r] = dv[r] * rb.slope(dv[r], p[0], p[1]);
                           if constexpr (!GRAD)
                             rb.add_any(dv[r], v[r], p[2], p[3]);
                         }
                         put_split(pl, pld, ((pos * 16 + n) * Cqd + cq) * 8, v);
                         if constexpr (GRAD)
                           *reinterpret_cast<float4v*>(
                               wsm + oat + ((pos * Cqd + cq) * 16 + n) * 16) = dv;
                       });
    } else {
      const int H = d.L[0].H, W = d.L[0].W;
      const int oy = py * d.L[0].S - d.L[0].P, ox = (px + win) * d.L[0].S - d.L[0].P;
      unsigned* xs = reinterpret_cast<unsigned*>(wsm + d.o_x);
      win_stage<MAXKS, false>(
          d.L[m].fb, d.L[m].nmt, d.L[m].nks, na, nax, wave, nw, load,
          [&](int mt, int y, int x, const float4v& dv) {
            const int qd = mt * 4 + G, ph = qd / Cqd, cq = qd - ph * Cqd;
            const int iy = s * y + ph / sx, ix = sx * x + ph % sx;
            if (ph >= s * sx || iy >= wd || ix >= wd) return;
            const bool in = oy + iy >= 0 && oy + iy < H && ox + ix >= 0 && ox + ix < W;
            if constexpr (GRAD) {
              // sign in the high byte of a bf16 +-2 (0x40, 0xc0)
              unsigned sv = 0;
#pragma unroll
              for (int r = 0; r < 4; ++r)
                sv |= (dv[r] > 0.f ? 0x40u : (dv[r] < 0.f ? 0xc0u : 0u)) << (8 * r);
              xs[((iy * wd + ix) * 16 + n) * Cqd + cq] = in ? sv : 0u;
            } else if (in) {
              l1 += (fabsf(dv[0]) + fabsf(dv[1])) + (fabsf(dv[2]) + fabsf(dv[3]));
            }
          });
    }
    __syncthreads();
  }

  if constexpr (!GRAD) {
    // a thread's bias terms: row tid % 16 in the fill and n in the stages are the same row
    float v3[3] = {rb.lo, l1, rb.up};
#pragma unroll
    for (int e = 0; e < (SYM ? 3 : 2); ++e) {
      v3[e] += __shfl_xor(v3[e], 16, 64);
      v3[e] += __shfl_xor(v3[e], 32, 64);
      if (lane < 16) red[(wave * 3 + e) * 16 + lane] = v3[e];
    }
    __syncthreads();
    if (tid >= 16) return;
    const bool neg = !SYM && tid >= 8;
    const int ch = SYM ? (nwin == 2 ? tid & 7 : 16 * g + tid) : 8 * g + (tid & 7);
    if (ch >= d.C || px + win >= d.W) return;
    float tb = (neg ? -1.f : 1.f) * d.bk[ch], ta = 0.f, tu = tb;
    for (int w = 0; w < nw; ++w) {
      tb += red[(w * 3 + 0) * 16 + tid];
      ta += red[(w * 3 + 1) * 16 + tid];
      if constexpr (SYM) tu += red[(w * 3 + 2) * 16 + tid];
    }
    const float v = tb - a.eps * ta;
    const long j = b * a.n_relu + a.noff_k + ((long)ch * d.H + py) * d.W + px + win;
    if constexpr (SYM) {
      a.lo[j] = v;
      a.hi[j] = tu + a.eps * ta;
    } else if (neg) {
      a.hi[j] = -v;
    } else {
      a.lo[j] = v;
    }
  } else {
    // the witness x0 - eps sign(A_x) forward: G_1 = z1 - eps W_1 sign(A_x), G_m = b_m + W_m z,
    // each G's adjoint terms summed over the 16 rows, z = the row's line applied to G
    const float wn = wrow[n];
    for (int m = 1; m < k; ++m) {
      const int w = d.L[m].w, s = d.L[m].s, K = d.L[m].K, Cq = d.L[m].Cq;
      const int wb = d.L[m - 1].w, Cqb = d.L[m - 1].Cq;
      const int H = d.L[m].H, W = d.L[m].W;
      const int oy = py * d.L[m].S - d.L[m].P, ox = px * d.L[m].S - d.L[m].P;
      const float4v* prm = reinterpret_cast<const float4v*>(wsm + d.L[m].o_prm);
      char* pl = wsm + d.L[m].o_pl;
      const int pld = d.L[m].plane;
      const float* atb = reinterpret_cast<const float*>(wsm + d.L[m].o_at);
      const float gs = m == 1 ? -0.5f * a.eps : 1.f;  // (the signs are stored as +-2)
      float* out = a.part + (long)blk0 * d.npart + d.L[m].part;
      const int ex = d.L[m].exf, kw = K + s * (ex - 1), nbx = (w + ex - 1) / ex;
      auto emit = [&](int mt, int y, int bx, const float4v& dv) {
        const int qd = mt * 4 + G, p = qd / Cq, cq = qd - p * Cq;
        const int x = ex * bx + p, yy = oy + y, xx = ox + x;
        // (the same for the 16 lanes that a sum runs over)
        const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
        const bool okq = p < ex && x < w;
        const int pos = y * w + x;
        float4v at = {0.f, 0.f, 0.f, 0.f}, z = at, sa = at, da = at, db = at;
        if (okq) {
          at = *reinterpret_cast<const float4v*>(atb + ((pos * Cq + cq) * 16 + n) * 4);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float4v p = prm[(pos * Cq + cq) * 4 + r];
            const float gv = fmaf(gs, dv[r], p[3]);
            z[r] = at[r] >= 0.f ? p[0] * gv : fmaf(p[1], gv, p[2]);
            const float tp = fmaxf(at[r], 0.f), tn = fminf(at[r], 0.f);
            sa[r] = wn != 0.f ? (wn * tp) * gv : 0.f;
            da[r] = wn != 0.f ? (wn * tn) * gv : 0.f;
            db[r] = wn != 0.f ? wn * tn : 0.f;
          }
          if (m + 1 < k) put_split(pl, pld, ((pos * 16 + n) * Cq + cq) * 8, z);
        }
        if (!in || !okq) return;  // (positions outside the map have no neuron)
#pragma unroll
        for (int r = 0; r < 4; ++r) sa[r] = row_sum16(sa[r]);
        if (m > 1) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            da[r] = row_sum16(da[r]);
            db[r] = row_sum16(db[r]);
          }
        }
        if (n == 0 && okq) {
          const int nt_ = w * w * 4 * Cq;
          *reinterpret_cast<float4v*>(out + (pos * Cq + cq) * 4) = sa;
          if (m > 1) {
            *reinterpret_cast<float4v*>(out + nt_ + (pos * Cq + cq) * 4) = da;
            *reinterpret_cast<float4v*>(out + 2 * nt_ + (pos * Cq + cq) * 4) = db;
          }
        }
      };
      if (m == 1) {
        const unsigned* xs = reinterpret_cast<const unsigned*>(wsm + d.o_x);
        win_stage<MAXKS, true>(d.L[m].ff, d.L[m].nmtf, d.L[m].nksf, w, nbx, wave, nw,
                        [&](int ks, int y, int x, uint4v (&B)[3]) {
                          uint4v v;
#pragma unroll
                          for (int h = 0; h < 2; ++h) {
                            const int qi = (ks * 4 + G) * 2 + h;
                            const int tap = min(qi / Cqb, K * kw - 1), cq = qi % Cqb;
                            const int iy = y * s + tap / kw;
                            const int ix = min(ex * x * s + tap % kw, wb - 1);
                            const unsigned u = xs[((iy * wb + ix) * 16 + n) * Cqb + cq];
                            // bytes to the high halves of bf16 pairs
                            v[2 * h] = __builtin_amdgcn_perm(u, 0u, 0x05000400u);
                            v[2 * h + 1] = __builtin_amdgcn_perm(u, 0u, 0x07000600u);
                          }
                          B[0] = v;
                          B[1] = v;
                          B[2] = v;
                        },
                        emit);
      } else {
        const char* src = wsm + d.L[m - 1].o_pl;
        const int plane = d.L[m - 1].plane, c2 = Cqb / 2;
        win_stage<MAXKS, false>(d.L[m].ff, d.L[m].nmtf, d.L[m].nksf, w, nbx, wave, nw,
                         [&](int ks, int y, int x, uint4v (&B)[3]) {
                           const int ck = ks * 4 + G, tap = min(ck / c2, K * kw - 1), cc = ck % c2;
                           const int iy = y * s + tap / kw;
                           const int ix = min(ex * x * s + tap % kw, wb - 1);
                           const int o = (((iy * wb + ix) * 16 + n) * c2 + cc) * 16;
#pragma unroll
                           for (int p = 0; p < 3; ++p)
                             B[p] = *reinterpret_cast<const uint4v*>(src + p * plane + o);
                         },
                         emit);
      }
      __syncthreads();
    }
  }
}

// Adjoint accumulation of layer m from the window partial sums of pass k: for each unstable
// neuron the flagged blocks of every position whose window holds it, in the order (y, x, group),
// then as k_grad_reduce.  A thread per (sub-domain, neuron).
__global__ void __launch_bounds__(kBlock)
    k_win_gather(long nb, WinLayer L, int m, int H, int W, int G, int npart,
                 const float* __restrict__ part, const unsigned char* __restrict__ pflag,
                 const int8_t* __restrict__ code, const float* __restrict__ l,
                 const float* __restrict__ u, long n_relu, float* __restrict__ ga,
                 float* __restrict__ gl, float* __restrict__ gu) {
  const long idx = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nm = (long)L.C * L.H * L.W;
  if (idx >= nb * nm) return;
  const long b = idx / nm;
  const int j = (int)(idx - b * nm);
  const long p = b * n_relu + L.noff + j;
  if (code[p] != 5) return;
  const int x = j % L.W, y = (j / L.W) % L.H, c = j / (L.W * L.H);
  // positions y_k with y_k S - P <= y < y_k S - P + w
  auto first = [&](int v) { const int q = v + L.P - L.w + 1; return q > 0 ? (q + L.S - 1) / L.S : 0; };
  const int y0 = first(y), y1 = min((y + L.P) / L.S, H - 1);
  const int x0 = first(x), x1 = min((x + L.P) / L.S, W - 1);
  const int nt = L.w * L.w * 4 * L.Cq;
  float sa = 0.f, da = 0.f, db = 0.f;
  for (int yk = y0; yk <= y1; ++yk)
    for (int xk = x0; xk <= x1; ++xk) {
      const int pos = (y - (yk * L.S - L.P)) * L.w + x - (xk * L.S - L.P);
      for (int g = 0; g < G; ++g) {
        const long blk = ((b * G + g) * H + yk) * W + xk;
        if (!pflag[blk]) break;  // (the groups of a position fill in order)
        const float* e = part + blk * npart + L.part + pos * 4 * L.Cq + c;
        sa += e[0];
        if (m > 1) {
          da += e[nt];
          db += e[2 * nt];
        }
      }
    }
  ga[p] += sa;
  if (m > 1) {
    const float lj = l[p], uj = u[p], dd = uj - lj, d2 = dd * dd;
    gl[p] += (da * uj - db * uj * uj) / d2;
    gu[p] += (-da * lj + db * lj * lj) / d2;
  }
}
