// The layers of an MLP one after the other, each contraction a launch of its own over output
// tiles of the whole matrix: the general route of the critic's calls and the policy gradient, for
// networks and row counts at which the row tiles of sim_gemm.h are slower (layer_route below).  A
// row tile reads every weight, so few row tiles of a wide network are a long chain on a few CUs,
// and many of them read the weights again and again; here a launch spreads the columns over the
// GPU as well.
//
// 32x64 output tiles staged through LDS in K-slices of 32, four wavefronts per tile, each
// wavefront a 1x2 block of 16x16x4 MFMA accumulators; the next slice is loaded into registers
// while the current one is multiplied.  Row reductions (K = rows) are split into fixed chunks
// whose partial tiles are summed in a fixed order, so every result is bitwise reproducible.
//
// Included inside a namespace with `real` defined as float or double, after sim_gemm.h.

#define GT_M 32
#define GT_MI (GT_M / 32)   // 16-row accumulator blocks per wavefront
#define GT_N 64
#define GT_K 32
#define GT_THREADS 256

enum { EPI_STORE = 0, EPI_BIAS_ELU = 1, EPI_DELU = 2, EPI_BIAS = 3 };

// C(m, n) = sum_k A(m, k) B(k, n) over k in this split's chunk, with element strides
// A(m, k) = A[m * sam + k * sak], B(k, n) = B[k * sbk + n * sbn].
struct GemmArgs {
  const real* A;
  long sam, sak;
  const real* B;
  long sbk, sbn;
  int M, N, K;
  int ones_col;      // column N-1 of B is all ones (bias gradient); B holds N-1 columns
  int k_chunk;       // K rows per split (multiple of GT_K); split z = blockIdx.z
  real* C;
  long ldc, split_stride;
  int epi;
  const real* bias;  // EPI_BIAS_ELU: C = elu(acc + bias[n]); EPI_BIAS: C = acc + bias[n]
  const real* Hm;    // EPI_DELU: C = acc * elu'(z), z > 0 <=> Hm > 0, else elu'(z) = Hm + 1
  long ldh;
  // optional per-column affine on the operand loads (observation normalisation of a first
  // layer's input): A(m, k) -> (A(m, k) - a_shift[k]) * a_scale[k], B(k, n) likewise by n
  const real* a_shift;
  const real* a_scale;
  const real* b_shift;
  const real* b_scale;
};

// one K-slice of A and B into registers (zero outside the matrices and the split's chunk)
#define GT_RA (GT_M * GT_K / GT_THREADS)
#define GT_RB (GT_N * GT_K / GT_THREADS)
__device__ __forceinline__ void gemm_load_slice(const GemmArgs& g, int tid, int m0, int n0, int k0, int ke, int bcols,
                                                real (&ra)[GT_RA], real (&rb)[GT_RB]) {
  const bool a_kfast = (g.sak == 1), b_kfast = (g.sbk == 1);
#pragma unroll
  for (int r = 0; r < GT_RA; ++r) {
    const int e = tid + r * GT_THREADS;
    const int m = m0 + (a_kfast ? e / GT_K : e % GT_M), k = k0 + (a_kfast ? e % GT_K : e / GT_M);
    real v = RL(0.0);
    if (m < g.M && k < ke) {
      v = g.A[(long)m * g.sam + (long)k * g.sak];
      if (g.a_shift) v = (v - g.a_shift[k]) * g.a_scale[k];
    }
    ra[r] = v;
  }
#pragma unroll
  for (int r = 0; r < GT_RB; ++r) {
    const int e = tid + r * GT_THREADS;
    const int n = n0 + (b_kfast ? e / GT_K : e % GT_N), k = k0 + (b_kfast ? e % GT_K : e / GT_N);
    real v = RL(0.0);
    if (k < ke) {
      if (n < bcols) {
        v = g.B[(long)k * g.sbk + (long)n * g.sbn];
        if (g.b_shift) v = (v - g.b_shift[n]) * g.b_scale[n];
      } else if (g.ones_col && n == g.N - 1) v = RL(1.0);
    }
    rb[r] = v;
  }
}

__global__ __launch_bounds__(GT_THREADS) void k_gemm(GemmArgs g) {
  __shared__ real As[GT_K][GT_M + 4];
  __shared__ real Bs[GT_K][GT_N + 4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m0 = blockIdx.x * GT_M, n0 = blockIdx.y * GT_N;
  const int kb = blockIdx.z * g.k_chunk;
  const int ke = min(g.K, kb + g.k_chunk);
  const int wm = (wv >> 1) * (16 * GT_MI), wn = (wv & 1) * 32;
  const int bcols = g.ones_col ? g.N - 1 : g.N;
  mfma_v4 acc[GT_MI][2];
#pragma unroll
  for (int i = 0; i < GT_MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = mfma_v4{RL(0.0), RL(0.0), RL(0.0), RL(0.0)};

  const bool a_kfast = (g.sak == 1), b_kfast = (g.sbk == 1);
  real ra[GT_RA], rb[GT_RB];
  if (kb < ke) gemm_load_slice(g, tid, m0, n0, kb, ke, bcols, ra, rb);
  for (int k0 = kb; k0 < ke; k0 += GT_K) {
#pragma unroll
    for (int r = 0; r < GT_RA; ++r) {
      const int e = tid + r * GT_THREADS;
      As[a_kfast ? e % GT_K : e / GT_M][a_kfast ? e / GT_K : e % GT_M] = ra[r];
    }
#pragma unroll
    for (int r = 0; r < GT_RB; ++r) {
      const int e = tid + r * GT_THREADS;
      Bs[b_kfast ? e % GT_K : e / GT_N][b_kfast ? e / GT_K : e % GT_N] = rb[r];
    }
    __syncthreads();
    // the next slice's loads are in flight while this one is multiplied
    if (k0 + GT_K < ke) gemm_load_slice(g, tid, m0, n0, k0 + GT_K, ke, bcols, ra, rb);
#pragma unroll
    for (int k4 = 0; k4 < GT_K; k4 += 4) {
      const int kr = k4 + (lane >> 4);
      real b0 = Bs[kr][wn + (lane & 15)], b1 = Bs[kr][wn + 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < GT_MI; ++i) {
        const real a = As[kr][wm + 16 * i + (lane & 15)];
        acc[i][0] = mfma_16x16x4(a, b0, acc[i][0]);
        acc[i][1] = mfma_16x16x4(a, b1, acc[i][1]);
      }
    }
    __syncthreads();
  }
  real* C = g.C + (long)blockIdx.z * g.split_stride;
#pragma unroll
  for (int i = 0; i < GT_MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + i * 16 + mfma_row(RL(0.0), lane, r);
        const int n = n0 + wn + j * 16 + (lane & 15);
        if (m < g.M && n < g.N) {
          real v = acc[i][j][r];
          if (g.epi == EPI_BIAS_ELU) {
            v += g.bias[n];
            v = v > RL(0.0) ? v : m_expm1(v);
          } else if (g.epi == EPI_BIAS) {
            v += g.bias[n];
          } else if (g.epi == EPI_DELU) {
            const real hv = g.Hm[(long)m * g.ldh + n];
            v *= hv > RL(0.0) ? RL(1.0) : hv + RL(1.0);
          }
          C[(long)m * g.ldc + n] = v;
        }
      }
}

__global__ void k_theta_seed(const real* __restrict__ da, const real* __restrict__ a, real* __restrict__ d, long n,
                             int mtu) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = squash_seed(da[i], a[i], mtu);
}

// sum of the split partials in split order; column `in` of each row is the bias gradient
__global__ void k_split_reduce(const real* __restrict__ part, int splits, long stride, int rows, int cols,
                               real* __restrict__ gW, real* __restrict__ gb) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)rows * cols) return;
  real s = RL(0.0);
  for (int z = 0; z < splits; ++z) s += part[z * stride + idx];
  const int o = (int)(idx / cols), i = (int)(idx % cols);
  if (i < cols - 1) gW[(long)o * (cols - 1) + i] = s;
  else gb[o] = s;
}

// ---- layer normalisation of the hidden layers (App. A.2) in the policy-gradient pass
// the normalised layer inputs from the window's ELU outputs and per-row statistics (the window's
// own expression, so the values are those its actor consumed)
__global__ void k_ln_apply(const real* __restrict__ E, long lde, const real* __restrict__ st, long ldst, int j,
                           const real* __restrict__ g, const real* __restrict__ b, real* __restrict__ Y, long M,
                           int n) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= M * n) return;
  const long r = idx / n;
  const int c = (int)(idx % n);
  const real mu = st[r * ldst + 2 * j], is = st[r * ldst + 2 * j + 1];
  Y[idx] = m_fma(g[c], (E[r * lde + c] - mu) * is, b[c]);
}

// Layer normalisation of hidden layer j row by row, computing its statistics (the critic's
// passes, which have no window activations): one wavefront per row; lane c sums columns c,
// c + 64, ... and a butterfly over the wavefront gives the row's mean and population
// variance; st[r ldst + 2 j] / [.. + 1] receive the mean and 1 / sqrt(var + eps), and
// Y [M][n] = g (E - mean) / sqrt(var + eps) + b as k_ln_apply forms it.
__global__ __launch_bounds__(256) void k_ln_forward(const real* __restrict__ E, long lde, real* __restrict__ st,
                                                    long ldst, int j, const real* __restrict__ g,
                                                    const real* __restrict__ b, real* __restrict__ Y, long M, int n,
                                                    real eps) {
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const long r = (long)blockIdx.x * 4 + wave;
  if (r >= M) return;   // uniform over the wavefront
  const real* e = E + r * lde;
  real sm = RL(0.0);
  for (int c = lane; c < n; c += SIM_WAVE) sm += e[c];
#pragma unroll
  for (int o = SIM_WAVE / 2; o > 0; o >>= 1) sm += __shfl_xor(sm, o);
  const real mu = sm / (real)n;
  real sv2 = RL(0.0);
  for (int c = lane; c < n; c += SIM_WAVE) {
    const real d = e[c] - mu;
    sv2 = m_fma(d, d, sv2);
  }
#pragma unroll
  for (int o = SIM_WAVE / 2; o > 0; o >>= 1) sv2 += __shfl_xor(sv2, o);
  const real is = RL(1.0) / m_sqrt(sv2 / (real)n + eps);
  for (int c = lane; c < n; c += SIM_WAVE) Y[r * n + c] = m_fma(g[c], (e[c] - mu) * is, b[c]);
  if (lane == 0) {
    st[r * ldst + 2 * j] = mu;
    st[r * ldst + 2 * j + 1] = is;
  }
}

// Adjoint through the normalisation and the ELU of hidden layer j, row by row: dY [M][n] (the
// adjoint of the normalised outputs) -> D [M][n] (the adjoint of the pre-activations), with
// a = (e - mean) r and u = g dY, ebar = r (u - mean(u) - a mean(u a)), D = ebar ELU'(z).  One
// wavefront per row at a time (lane c holds columns c, c + 64, ...); each block also sums, over
// its rows in a fixed order, dY a (the gain gradient) and dY (the bias gradient) per column
// into part[block][0 / 1][n], reduced across blocks in block order by k_ln_reduce.
#define SIM_LN_Q (SIM_MAXHID / SIM_WAVE)
__global__ __launch_bounds__(256) void k_ln_backward(const real* __restrict__ dY, const real* __restrict__ E, long lde,
                                                     const real* __restrict__ st, long ldst, int j,
                                                     const real* __restrict__ g, real* __restrict__ D, long M, int n,
                                                     real* __restrict__ part) {
  __shared__ real red[4][2][SIM_MAXHID];
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  real pg[SIM_LN_Q], pb[SIM_LN_Q];
#pragma unroll
  for (int q = 0; q < SIM_LN_Q; ++q) { pg[q] = RL(0.0); pb[q] = RL(0.0); }
  for (long r = (long)blockIdx.x * 4 + wave; r < M; r += (long)gridDim.x * 4) {
    const real mu = st[r * ldst + 2 * j], is = st[r * ldst + 2 * j + 1];
    real u[SIM_LN_Q], a[SIM_LN_Q], ev[SIM_LN_Q];
    real su = RL(0.0), sua = RL(0.0);
#pragma unroll
    for (int q = 0; q < SIM_LN_Q; ++q) {
      const int c = lane + SIM_WAVE * q;
      u[q] = a[q] = ev[q] = RL(0.0);
      if (c < n) {
        const real dy = dY[r * n + c];
        ev[q] = E[r * lde + c];
        a[q] = (ev[q] - mu) * is;
        u[q] = g[c] * dy;
        su += u[q];
        sua = m_fma(u[q], a[q], sua);
        pg[q] = m_fma(dy, a[q], pg[q]);
        pb[q] += dy;
      }
    }
    const real mu_u = wave_sum(su) / (real)n, mu_ua = wave_sum(sua) / (real)n;
#pragma unroll
    for (int q = 0; q < SIM_LN_Q; ++q) {
      const int c = lane + SIM_WAVE * q;
      if (c < n) {
        const real eb = is * (u[q] - mu_u - a[q] * mu_ua);
        D[r * n + c] = eb * ((ev[q] > RL(0.0)) ? RL(1.0) : ev[q] + RL(1.0));
      }
    }
  }
#pragma unroll
  for (int q = 0; q < SIM_LN_Q; ++q) {
    const int c = lane + SIM_WAVE * q;
    if (c < n) { red[wave][0][c] = pg[q]; red[wave][1][c] = pb[q]; }
  }
  __syncthreads();
  for (int c = (int)threadIdx.x; c < n; c += 256) {
    part[((long)blockIdx.x * 2 + 0) * n + c] = ((red[0][0][c] + red[1][0][c]) + red[2][0][c]) + red[3][0][c];
    part[((long)blockIdx.x * 2 + 1) * n + c] = ((red[0][1][c] + red[1][1][c]) + red[2][1][c]) + red[3][1][c];
  }
}

__global__ void k_ln_reduce(const real* __restrict__ part, int nb, int n, real* __restrict__ gg,
                            real* __restrict__ gb) {
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= n) return;
  real s0 = RL(0.0), s1 = RL(0.0);
  for (int z = 0; z < nb; ++z) {
    s0 += part[((long)z * 2 + 0) * n + c];
    s1 += part[((long)z * 2 + 1) * n + c];
  }
  gg[c] = s0;
  gb[c] = s1;
}

static void launch_gemm(const GemmArgs& g, int splits, hipStream_t s) {
  dim3 grid((g.M + GT_M - 1) / GT_M, (g.N + GT_N - 1) / GT_N, splits);
  hipLaunchKernelGGL(k_gemm, grid, dim3(GT_THREADS), 0, s, g);
}

// the hidden layers of a critic on T.M rows of T.x0 (H[l + 1] = elu(H[l] W_l^T + b_l))
static void theta_hidden(const ThetaArgsT<real>& T, hipStream_t s) {
  const int M = T.M, L = T.nl;
  for (int l = 0; l + 1 < L; ++l) {
    const int ni = T.dims[l], no = T.dims[l + 1];
    GemmArgs g = {};
    g.A = (l == 0) ? T.x0 : (T.ln ? T.Y[l] : T.H[l]);
    g.sam = ni; g.sak = 1;
    g.B = T.W[l]; g.sbk = 1; g.sbn = ni;
    g.M = M; g.N = no; g.K = ni;
    g.k_chunk = (ni + GT_K - 1) / GT_K * GT_K;
    g.C = T.H[l + 1]; g.ldc = no;
    g.epi = EPI_BIAS_ELU; g.bias = T.b[l];
    if (l == 0) { g.a_shift = T.x_shift; g.a_scale = T.x_scale; }
    launch_gemm(g, 1, s);
    if (T.ln)
      hipLaunchKernelGGL(k_ln_forward, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, s, T.H[l + 1], (long)no, T.st,
                         T.ldst, l, T.lng[l], T.lnb[l], T.Y[l + 1], (long)M, no, T.ln_eps);
  }
}

// the linear output layer on the rows (out [M][dims[L]] = H[L-1] W^T + b)
static void theta_output(const ThetaArgsT<real>& T, real* out, hipStream_t s) {
  const int L = T.nl, ni = T.dims[L - 1], no = T.dims[L];
  GemmArgs g = {};
  g.A = (L == 1) ? T.x0 : (T.ln ? T.Y[L - 1] : T.H[L - 1]);
  g.sam = ni; g.sak = 1;
  g.B = T.W[L - 1]; g.sbk = 1; g.sbn = ni;
  g.M = T.M; g.N = no; g.K = ni;
  g.k_chunk = (ni + GT_K - 1) / GT_K * GT_K;
  g.C = out; g.ldc = no;
  g.epi = EPI_BIAS; g.bias = T.b[L - 1];
  if (L == 1) { g.a_shift = T.x_shift; g.a_scale = T.x_scale; }
  launch_gemm(g, 1, s);
}

// given the output adjoint in T.d0, every layer's weight and bias gradient (flat in T.out)
static void theta_backward(const ThetaArgsT<real>& T, hipStream_t s) {
  const int M = T.M, L = T.nl;
  real* dcur = T.d0;
  real* dnext = T.d1;
  const int chunk = ((M + T.splits - 1) / T.splits + GT_K - 1) / GT_K * GT_K;
  const int splits = (M + chunk - 1) / chunk;
  for (int l = L - 1; l >= 0; --l) {
    const int ni = T.dims[l], no = T.dims[l + 1];
    // layer l's input: the observations, the hidden activations, or their normalisations
    const real* xin = (l == 0) ? T.x0 : (T.ln ? T.Y[l] : T.H[l]);
    const long ldx = (l > 0 && !T.ln && T.ldH[l]) ? T.ldH[l] : ni;
    const long ldh = (l > 0 && T.ldH[l]) ? T.ldH[l] : ni;
    GemmArgs g = {};
    g.A = dcur; g.sam = 1; g.sak = no;
    g.B = xin; g.sbk = ldx; g.sbn = 1; g.ones_col = 1;
    g.M = no; g.N = ni + 1; g.K = M; g.k_chunk = chunk;
    g.C = T.part; g.ldc = ni + 1; g.split_stride = (long)no * (ni + 1);
    g.epi = EPI_STORE;
    if (l == 0) { g.b_shift = T.x_shift; g.b_scale = T.x_scale; }
    launch_gemm(g, splits, s);
    const long nr = (long)no * (ni + 1);
    hipLaunchKernelGGL(k_split_reduce, dim3((unsigned)((nr + 255) / 256)), dim3(256), 0, s, T.part, splits,
                       (long)no * (ni + 1), no, ni + 1, T.out + T.off_w[l], T.out + T.off_b[l]);
    if (l > 0) {
      GemmArgs g2 = {};
      g2.A = dcur; g2.sam = no; g2.sak = 1;
      g2.B = T.W[l]; g2.sbk = ni; g2.sbn = 1;
      g2.M = M; g2.N = ni; g2.K = no;
      g2.k_chunk = (no + GT_K - 1) / GT_K * GT_K;
      g2.C = dnext; g2.ldc = ni;
      if (!T.ln) {
        g2.epi = EPI_DELU; g2.Hm = T.H[l]; g2.ldh = ldh;
        launch_gemm(g2, 1, s);
        real* t = dcur; dcur = dnext; dnext = t;
      } else {
        // the adjoint of the normalised outputs, then through the normalisation and the ELU
        // into dcur (whose layer-l adjoint has been consumed)
        g2.epi = EPI_STORE;
        launch_gemm(g2, 1, s);
        hipLaunchKernelGGL(k_ln_backward, dim3(SIM_LN_BLOCKS), dim3(256), 0, s, dnext, T.H[l], ldh, T.st, T.ldst, l - 1,
                           T.lng[l - 1], dcur, (long)M, ni, T.lnpart);
        hipLaunchKernelGGL(k_ln_reduce, dim3((ni + 255) / 256), dim3(256), 0, s, T.lnpart, SIM_LN_BLOCKS, ni,
                           T.out + T.off_g[l - 1], T.out + T.off_beta[l - 1]);
      }
    }
  }
}

// ---------------------------------------------------------------- the choice
// Loads a wave of a row tile waits for one after the other in a forward pass: 32 values of k for two
// column tiles (one below 128 columns) at a time
static int row_chain(const ThetaArgsT<real>& T) {
  int c = 0;
  for (int l = 0; l + 1 < T.nl; ++l) {
    const int cols = MR_WAVES * 16 * (T.dims[l + 1] >= 128 ? 2 : 1);
    c += (T.dims[l + 1] + cols - 1) / cols * ((T.dims[l] + 31) / 32);
  }
  return c;
}

// Whether the rows of a call go layer by layer, or as row tiles (sim_gemm.h).  A block of row tiles
// streams all weights: with few rows a wide network is a chain of loads on a few CUs, and with many
// rows its weights are read once per tile.  Layer by layer a call is three to fifteen launches, whose
// contractions take any width well.  So the lines lie by the rows M and, for values, by the chain c
// of loads, with weights that are not in L2 (a program asks for values once per episode, behind a
// window); for fits and the policy gradient by the network's parameters np and, with layer
// normalisation, whose passes over the hidden layers cost the tiles most, the sum hs of the hidden
// widths; FP64 streams twice the bytes.  Measured, as time layer by layer over time in tiles (above
// one: tiles), at 12 to 15 row counts of 12 networks for each line; the muscle critic is 280-400-200-1
// (193 k parameters, c 62), the other inputs 76 or named:
//   values  FP32 256-128 (c 14) 1.35 to 2.1 from 64 rows on; 280-256-128 (26) 1.07 to 2.0, 0.78 at one row;
//           300-200 (29) 0.80 to 0.94 to 4096 rows, 1.24 at 5000; 400-200 (38) 0.70 to 0.90 and 1.06; muscle
//           critic 0.58 to 0.80, 0.94 at 6144, 1.36 at 8000.  Normalised 280-512 (36) 1.12 from 64 rows on, 0.90
//           at one; muscle critic 1.01 to 2.2, 0.83 at one; 37-512-512 (72) 0.76 to 0.91 to 2048, 1.02 at 2560.  FP64
//           280-256-128 1.27, 5-400-200 (30) 0.91 to 0.98 to 2048 rows and 1.14 at 2560; muscle critic 0.77 to
//           0.82, 1.12 at 2560, 0.84 at 4500, 1.17 at 8000.  Normalised FP64 400-200 0.90 to 0.95 to 1024 and 1.02
//           at 1536, muscle critic 0.80 to 0.88 to 2048 and 1.16 at 2560.
//   fit     FP32 to 111 k parameters 0.98 to 2.1; muscle critic 0.87 at 64, 1.05 at 512, 1.1 to 1.3 from 1024
//           on; 512-512 0.62 to 0.93.  FP64 53 k 1.13 to 1.57 to 4096 rows, 0.99 at 6144, 0.73 at 32768; 76 k
//           0.88 at 64, 1.07 to 1.16 from 512 to 4096; 83 k 0.80 to 1.05 to 2048, 1.08 to 1.20 at 3072 and
//           4096; 111 k below 0.93.  Normalised: FP32 1.15 to 3.9 to 2048 rows, then 256-256 1.13 at 8192, 400-200
//           1.20 at 4096 and 0.95 at 6144, 512-512 0.76 at 3072; FP64 256-256 1.28 at 4096, 400-200 1.45 at 2048
//           and 0.91 at 3072, 512-512 below 0.91.
//   theta   FP32 policies 76-256-128-21 (58 k) 1.28 to 3.4, 83 k 1.07 to 2.4, muscle (280-400-200-152, 223 k)
//           1.06 at 8192 rows and 0.90 at 16384, 512-512 0.69 to 1.1.  FP64 83 k 1.09 at 16384, 0.89 at 32768;
//           muscle 0.79 at 64.  Normalised: FP32 83 k 1.22 at 8192 and 0.95 at 16384, FP64 1.03 and 0.87.
static bool layered(const ThetaArgsT<real>& T, int mode) {
  constexpr bool f64 = sizeof(real) == 8;
  const double np = (double)mlp_params(T), M = T.M;
  double hs = 0;
  for (int l = 1; l < T.nl; ++l) hs += T.dims[l];
  if (mode == ROWS_VALUES) {
    const int c = row_chain(T);
    if (M < 16 && c > (!f64 && T.ln ? 35 : 17)) return true;
    if (f64) return (c > 60 && (M < 2300 || (M > 4096 && M < 7000))) || (T.ln ? c > 33 && M < 1300 : c > 28 && M < 2300);
    return T.ln ? c > 64 && M < 2560 : (c > 28 && M < 4608) || (c > 60 && M < 7000);
  }
  if (mode == ROWS_FIT) {
    if (T.ln) return M > (f64 ? 8192 : 16384) || (M > 2048 && hs * hs * hs * M > (f64 ? 5.6e11 : 1.2e12)) || (f64 && np > 200e3);
    if (f64) return M > 4096 || np > 106e3 || (np > 80e3 && M < 3072) || (np > 55e3 && M < 512);
    return np > 200e3 || (np > 120e3 && M < 384);
  }
  if (T.ln) return np * M > (f64 ? 0.7e9 : 1.2e9);
  return np * M > (f64 ? 1.0e9 : 2.0e9) || np > (f64 ? 100e3 : 250e3);
}

// ---------------------------------------------------------------- policy gradient
static void theta_layers(const ThetaArgsT<real>& T, hipStream_t s) {
  if (T.ln)
    for (int l = 1; l < T.nl; ++l) {
      const long n = (long)T.M * T.dims[l];
      hipLaunchKernelGGL(k_ln_apply, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, T.H[l], T.ldH[l], T.st,
                         T.ldst, l - 1, T.lng[l - 1], T.lnb[l - 1], T.Y[l], (long)T.M, T.dims[l]);
    }
  const long n = (long)T.M * T.dims[T.nl];
  hipLaunchKernelGGL(k_theta_seed, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, T.da, T.act, T.d0, n, T.mtu);
  theta_backward(T, s);
}

static int theta_tiles(const ThetaArgsT<real>& T, hipStream_t s) {
  RowsArgs R = {};
  int blocks = 0;
  if (T.nl > 1 && launch_rows<ROWS_THETA>(R, T, &blocks, nullptr, s)) return -1;
  WgradArgs W = {};
  W.N = mlp_net(T);
  launch_wgrad(W, T, s);
  if (W.splits > 1 || T.ln) {
    ReduceArgs Q = {};
    reduce_args(Q, T, W.part, W.splits, blocks, true);
    Q.out = T.out;
    hipLaunchKernelGGL(k_mlp_reduce, dim3((unsigned)((Q.np + SIM_WAVE - 1) / SIM_WAVE)), dim3(RD_WAVES * SIM_WAVE), 0, s, Q);
  }
  return 0;
}

int launch_theta(const ThetaArgsT<real>& T, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (T.noise && T.out_log_std)
    hipLaunchKernelGGL(k_log_std_grad, dim3(T.dims[T.nl]), dim3(256), 0, s, T.da, T.act, T.noise, T.log_std, (long)T.M,
                       T.dims[T.nl], T.mtu, T.out_log_std);
  if (layered(T, ROWS_THETA)) theta_layers(T, s);
  else if (theta_tiles(T, s)) return -1;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}
