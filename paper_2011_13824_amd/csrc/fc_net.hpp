// A whole bound of a small fully connected net in one launch (included by lirpa.hip).
//
// At widths of a few wavefronts every stage is launch latency (seven launches, 33 us for a
// 4-32-32-2 net with 64 sub-domains, none of them over 3 us of work).  A block takes one
// sub-domain through layer 1, every intermediate pass and the final pass with the weights, the
// bounds and the relaxations in LDS; a row is carried by 16 lanes, 32 rows at a time.  What
// bounds it is the LDS latency of the rows' dot products (reads eight at a time: 19.9 -> 12.5 us
// at 64 sub-domains, of which the host's share is most).

constexpr int kNetWidth = 64;   // widest layer
constexpr int kNetLayers = 8;
constexpr int kNetWeights = 8192;  // floats of all W and b
constexpr int kNetThreads = 512;

struct FcNet {
  int L, S;
  int n[kNetLayers + 1];   // widths
  int w[kNetLayers + 1];   // W_m and b_m in the LDS copy
  int bo[kNetLayers + 1];
  int off[kNetLayers + 1]; // ReLU layer offsets
  const float* W[kNetLayers + 1];
  const float* b[kNetLayers + 1];
  const float* x0;
  const float* C;
  float eps;
  long n_relu;
  const int8_t* split;
  const float* alpha;
  const float* lpar;
  const float* upar;
  float* lb;
  float* l;       // optional, whole rows
  float* u;
  int8_t* code;   // optional
};

__global__ void __launch_bounds__(kNetThreads) k_fc_net(FcNet d_) {
  const __attribute__((address_space(4))) FcNet& d =
      *(const __attribute__((address_space(4))) FcNet*)__builtin_amdgcn_kernarg_segment_ptr();
  __shared__ float wt[kNetWeights];
  __shared__ float x0s[kNetWidth];
  // (a_lo, a_up, b_up, constant) of ReLU layer m: the bias, and of layer 1 z1 = W_1 x0 + b_1, which
  // holds the rows' terms in x0 (summed over x they would overflow where the bound does not)
  __shared__ float4v rel[kNetLayers][kNetWidth];
  __shared__ float z1[kNetWidth];
  __shared__ float lu[2][kNetWidth];
  __shared__ float4v buf[kNetThreads / 16][2][kNetWidth / 4];
  const int tid = threadIdx.x, grp = tid >> 4, ln = tid & 15;
  const long b = blockIdx.x;
  const int L = d.L;
  for (int m = 1; m <= L; ++m) {
    const int nw = d.n[m] * d.n[m - 1];
    for (int e = tid; e < nw; e += kNetThreads) wt[d.w[m] + e] = d.W[m][e];
    for (int e = tid; e < d.n[m]; e += kNetThreads) wt[d.bo[m] + e] = d.b[m][e];
  }
  for (int e = tid; e < d.n[0]; e += kNetThreads) x0s[e] = d.x0[e];
  __syncthreads();

  // bounds of ReLU layer m (in lu) to its relaxation
  auto relax = [&](int m) {
    for (int j = tid; j < d.n[m]; j += kNetThreads) {
      const long p = b * d.n_relu + d.off[m] + j;
      float lj = lu[0][j], uj = lu[1][j];
      parent_clip(lj, uj, d.lpar, d.upar, p);
      const Relax1 r = relax_neuron(lj, uj, d.split ? d.split[p] : 0,
                                    d.alpha ? d.alpha + p : nullptr);
      rel[m][j] = float4v{r.lo, r.up, r.bu, m == 1 ? z1[j] : wt[d.bo[m] + j]};
      if (d.l) {
        d.l[p] = lj;
        d.u[p] = uj;
      }
      if (d.code) d.code[p] = (int8_t)r.code;
    }
  };
  auto lane_sum = [](float v) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
  // layer 1: exact over the box
  for (int j0 = 0; j0 < d.n[1]; j0 += kNetThreads / 16) {  // (every wave runs every turn)
    const int j = min(j0 + grp, d.n[1] - 1);
    float z = 0.f, r = 0.f;
    for (int i = ln; i < d.n[0]; i += 16) {
      const float w = wt[d.w[1] + j * d.n[0] + i];
      z = fmaf(w, x0s[i], z);
      r += fabsf(w);
    }
    z = lane_sum(z) + wt[d.bo[1] + j];
    r = lane_sum(r);
    if (ln == 0) {
      z1[j] = z;
      lu[0][j] = z - d.eps * r;
      lu[1][j] = z + d.eps * r;
    }
  }
  __syncthreads();
  if (L > 1) relax(1);
  __syncthreads();

  for (int k = 2; k <= L; ++k) {
    // rows +-e_j of h^(k), or the spec rows of the last layer
    const bool last = k == L;
    const int nk = d.n[k], rows = last ? d.S : 2 * nk, nb = d.n[k - 1];
    // (every wave runs every turn: the sums shuffle)
    for (int r0 = 0; r0 < rows; r0 += kNetThreads / 16) {
      const int r = min(r0 + grp, rows - 1);
      const int j = r >> 1;
      const float sg = (r & 1) ? -1.f : 1.f;
      float beta = 0.f, l1 = 0.f;
      if (last) {
        if (ln == 0)
          for (int o = 0; o < nk; ++o) beta = fmaf(d.C[r * nk + o], wt[d.bo[k] + o], beta);
      } else if (ln == 0) {
        beta = sg * wt[d.bo[k] + j];
      }
      auto put = [&](int m, float* dst, int i, float a) {  // relaxed onto layer m
        const float4v p = rel[m][i];
        const float ah = a * (a >= 0.f ? p[0] : p[1]);
        beta = fmaf(fminf(a, 0.f), p[2], beta);
        beta = fmaf(ah, p[3], beta);
        dst[i] = ah;
      };
      float* cur = reinterpret_cast<float*>(buf[grp][0]);
      float* nxt = reinterpret_cast<float*>(buf[grp][1]);
      for (int i = ln; i < nb; i += 16) {
        float a;
        if (last) {
          a = 0.f;
          for (int o = 0; o < nk; ++o) a = fmaf(d.C[r * nk + o], wt[d.w[k] + o * nb + i], a);
        } else {
          a = sg * wt[d.w[k] + j * nb + i];
        }
        put(k - 1, cur, i, a);
      }
      for (int m = k - 1; m >= 1; --m) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the row's 16 lanes share a wave
        const int no = d.n[m], ni = d.n[m - 1];
        const float* W = wt + d.w[m];
        for (int i = ln; i < ni; i += 16) {
          // two sums of eight products in flight, so that the LDS latency is paid once per eight
          float a = 0.f, a2 = 0.f;
          int o = 0;
          for (; o + 8 <= no; o += 8) {
            const float4v c0 = *reinterpret_cast<const float4v*>(cur + o);
            const float4v c1 = *reinterpret_cast<const float4v*>(cur + o + 4);
            float w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = W[(o + e) * ni + i];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              a = fmaf(c0[e], w[e], a);
              a2 = fmaf(c1[e], w[e + 4], a2);
            }
          }
          for (; o < no; ++o) a = fmaf(cur[o], W[o * ni + i], a);
          a += a2;
          if (m > 1) {
            put(m - 1, nxt, i, a);
          } else {
            l1 += fabsf(a);
          }
        }
        float* t = cur;
        cur = nxt;
        nxt = t;
      }
      beta = fmaf(-d.eps, lane_sum(l1), lane_sum(beta));
      if (ln == 0 && r0 + grp < rows) {
        if (last)
          d.lb[b * d.S + r] = beta;
        else
          lu[r & 1][j] = sg * beta;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // before the buffers are refilled
    }
    __syncthreads();
    if (!last) {
      relax(k);
      __syncthreads();
    }
  }
}
