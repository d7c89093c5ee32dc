// Policy-parameter gradient of the short-horizon actor loss (App. A.1, the dL/dtheta
// term): given dL/da_t of every environment and frame, the gradient is the sum over all
// h*N (frame, env) rows of (d pi(o_t) / d theta)^T dL/da_t.  The layer inputs are the
// observations and the hidden activations that the forward window stored for every frame
// and env; the action adjoint is carried back through the squash and every ELU layer, and
// the weight gradient of a layer is the contraction of its output adjoint with its input
// over all rows.  The critic's calls (values, minibatch fit) use the same kernels and
// compute their hidden layers themselves.  Networks and row counts for which these tiles of rows
// are the slower form go layer by layer (sim_layers.h).
//
// Kernels, each one launch whatever the depth of the network:
//   k_mlp_fit     a minibatch's 16 or 32 rows per block through every layer, back, and into the
//                 block's own weight gradient, all in LDS (networks that fit),
//   k_mlp_rows    the same rows without the weight gradient (values; larger networks; dL/dtheta),
//   k_mlp_wgrad   every layer's weight and bias gradient from k_mlp_rows's arrays,
//   k_mlp_reduce  the sum of the partial gradients in a fixed order, with the Adam step of a fit.
// The argument structures are flat, without arrays indexed at run time: kernel arguments come
// from a memory far from the GPU, and with arrays a kernel waited for them once per layer
// (128 rows of a 5-64-64-1 critic: 13.4 us in k_mlp_rows with arrays, 8 us without).
// Every contraction runs on the 16x16x4 matrix instructions in the precision of the path;
// all sums have a fixed order, so the gradient is bitwise reproducible.
//
// Included inside a namespace with `real` defined as float or double.

typedef float mfma_v4f __attribute__((__vector_size__(4 * sizeof(float))));
typedef double mfma_v4d __attribute__((__vector_size__(4 * sizeof(double))));
typedef real mfma_v4 __attribute__((__vector_size__(4 * sizeof(real))));
typedef real mlp_r4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mfma_v4f mfma_16x16x4(float a, float b, mfma_v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ mfma_v4d mfma_16x16x4(double a, double b, mfma_v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Row of a 16x16 accumulator block held by lane l in element r (the column is l % 16).
// The two instructions lay their results out differently: FP32 keeps four consecutive
// rows per 16-lane group, FP64 interleaves the groups.
__device__ __forceinline__ int mfma_row(float, int l, int r) { return 4 * (l >> 4) + r; }
__device__ __forceinline__ int mfma_row(double, int l, int r) { return (l >> 4) + 4 * r; }

#define MR_THREADS 256
#define MR_WAVES (MR_THREADS / SIM_WAVE)
#define MR_MAXHIDL 2     // hidden layers (sim_create accepts at most two)
enum { ROWS_VALUES = 0, ROWS_FIT = 1, ROWS_THETA = 2 };

__host__ __device__ __forceinline__ int mlp_pad16(int n) { return (n + 15) & ~15; }

// One network and one set of rows.  D1 / D2 / H1 / H2 / Y1 / Y2 belong to the first / second
// hidden layer: adjoint of its pre-activations, ELU outputs, normalised outputs (layer
// normalisation), [M][d1] and [M][d2] (H1 / H2 with row strides ldh1 / ldh2).
struct MlpNet {
  int M, L;                    // rows, linear layers (1 .. 3)
  int d0, d1, d2, d3;          // widths: input, then each layer's outputs
  int vec;                     // bit l: rows of W_l can be read four values at a time
  int mtu;
  const real *W0, *W1, *W2, *b0, *b1, *b2;
  const real *x0, *shift, *scale;
  real *H1, *H2, *D1, *D2;
  int ldh1, ldh2;
  const real *da, *act;        // policy gradient: dL/da and the actions [M][d_L]
  const real *g1, *be1, *g2, *be2;   // layer normalisation
  real *Y1, *Y2;
  const real* st;              // the window's statistics, row stride ldst
  int ldst;
  real eps;
};
__device__ __forceinline__ int net_dim(const MlpNet& n, int l) { return l == 0 ? n.d0 : (l == 1 ? n.d1 : (l == 2 ? n.d2 : n.d3)); }

// acc(row, n) = sum_k A(row, k) W(n, k) for the block's rows (A in LDS, zero past K up to a
// multiple of 16) and every output n, handed to epi(row, n, acc) for n < pad16(N).  Wave wv of nw
// takes CT column tiles of 16 at a time.  The four values of k a lane holds per 16 are consecutive
// (one vector load each of A and W); the same permutation of k on both operands leaves the
// product unchanged.  W comes from L2, the next 32 values of k requested before the present ones
// are multiplied.
template <int RT, int CT, class F>
__device__ __forceinline__ void rows_fwd(const real* A, int ld, const real* __restrict__ W, int K, int N, bool vec,
                                         int wv, int nw, F epi) {
  const int lane = threadIdx.x & 63, q = lane >> 4, c16 = lane & 15;
  const int nt = (N + 15) >> 4, Kp = mlp_pad16(K);
  for (int t0 = wv * CT; t0 < nt; t0 += nw * CT) {
    mfma_v4 acc[RT][CT];
    const real* wp[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int n = (t0 + c) * 16 + c16;
      wp[c] = W + (long)(n < N ? n : 0) * K;
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i][c] = mfma_v4{RL(0.0), RL(0.0), RL(0.0), RL(0.0)};
    }
    auto load = [&](mlp_r4 (&b)[2][CT], int k0) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          const int k = k0 + 16 * h + 4 * q;
          mlp_r4 v = {RL(0.0), RL(0.0), RL(0.0), RL(0.0)};
          if (vec) {
            if (k < K) v = *reinterpret_cast<const mlp_r4*>(wp[c] + k);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (k + j < K) v[j] = wp[c][k + j];
          }
          b[h][c] = v;
        }
    };
    mlp_r4 b[2][CT], bn[2][CT];
    load(b, 0);
    for (int k0 = 0; k0 < Kp; k0 += 32) {
      if (k0 + 32 < Kp) load(bn, k0 + 32);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (k0 + 16 * h < Kp) {
          mlp_r4 a[RT];
#pragma unroll
          for (int i = 0; i < RT; ++i) a[i] = *reinterpret_cast<const mlp_r4*>(A + (16 * i + c16) * ld + k0 + 16 * h + 4 * q);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
              for (int c = 0; c < CT; ++c) acc[i][c] = mfma_16x16x4(a[i][j], b[h][c][j], acc[i][c]);
        }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < CT; ++c) b[h][c] = bn[h][c];
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
      if (t0 + c < nt) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) epi(16 * i + mfma_row(RL(0.0), lane, r), (t0 + c) * 16 + c16, acc[i][c][r]);
      }
  }
}

// acc(row, n) = sum_k A(row, k) W(k, n), W [K][N]: a layer's input adjoint (see rows_fwd)
template <int RT, int CT, class F>
__device__ __forceinline__ void rows_dgrad(const real* A, int ld, const real* __restrict__ W, int K, int N, int wv, int nw,
                                           F epi) {
  const int lane = threadIdx.x & 63, q = lane >> 4, c16 = lane & 15;
  const int nt = (N + 15) >> 4, Kp = mlp_pad16(K);
  for (int t0 = wv * CT; t0 < nt; t0 += nw * CT) {
    mfma_v4 acc[RT][CT];
    const real* wp[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int n = (t0 + c) * 16 + c16;
      wp[c] = W + (n < N ? n : 0);
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i][c] = mfma_v4{RL(0.0), RL(0.0), RL(0.0), RL(0.0)};
    }
    auto load = [&](real (&b)[2][CT][4], int k0) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = k0 + 16 * h + 4 * q + j;
#pragma unroll
          for (int c = 0; c < CT; ++c) b[h][c][j] = (k < K) ? wp[c][k * N] : RL(0.0);
        }
    };
    real b[2][CT][4], bn[2][CT][4];
    load(b, 0);
    for (int k0 = 0; k0 < Kp; k0 += 32) {
      if (k0 + 32 < Kp) load(bn, k0 + 32);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (k0 + 16 * h < Kp) {
          mlp_r4 a[RT];
#pragma unroll
          for (int i = 0; i < RT; ++i) a[i] = *reinterpret_cast<const mlp_r4*>(A + (16 * i + c16) * ld + k0 + 16 * h + 4 * q);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
              for (int c = 0; c < CT; ++c) acc[i][c] = mfma_16x16x4(a[i][j], b[h][c][j], acc[i][c]);
        }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) b[h][c][j] = bn[h][c][j];
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
      if (t0 + c < nt) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) epi(16 * i + mfma_row(RL(0.0), lane, r), (t0 + c) * 16 + c16, acc[i][c][r]);
      }
  }
}

// the adjoint of the pre-squash policy output: dL/dy = dL/da da/dy with a = tanh(y) (1 - a^2)
// or, for muscle excitations, u = (tanh(y) + 1) / 2 (2 u (1 - u))
__device__ __forceinline__ real squash_seed(real da, real av, int mtu) {
  return da * (mtu ? RL(2.0) * av * (RL(1.0) - av) : RL(1.0) - av * av);
}

// sum over the 16 lanes of a row group (butterfly; every lane of the group receives it)
__device__ __forceinline__ real sum16(real x) {
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) x += __shfl_xor(x, o, SIM_WAVE);
  return x;
}

// mean and inverse deviation of each row of E (LDS, n columns) into st[row][2], 16 lanes a row
template <int RT, int NW>
__device__ __forceinline__ void rows_ln_stats(const real* E, int ld, int n, real eps, real (*st)[2]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c16 = lane & 15;
  for (int r = 4 * wv + (lane >> 4); r < 16 * RT; r += 4 * NW) {
    const real* e = E + r * ld;
    real s = RL(0.0);
    for (int c = c16; c < n; c += 16) s += e[c];
    const real mu = sum16(s) / (real)n;
    real v = RL(0.0);
    for (int c = c16; c < n; c += 16) {
      const real d = e[c] - mu;
      v = m_fma(d, d, v);
    }
    v = sum16(v);
    if (c16 == 0) {
      st[r][0] = mu;
      st[r][1] = RL(1.0) / m_sqrt(v / (real)n + eps);
    }
  }
}

// columns of a layer-normalisation pass: thread tid takes column c (and, with 256 threads, c + 256)
// of the rows of its group; narrow layers split the rows over several groups
template <int NW>
__device__ __forceinline__ int ln_groups(int n) { return NW / (n <= 64 ? 1 : (n <= 128 ? 2 : (n <= 256 ? 4 : NW))); }

// The adjoint through the normalisation and the ELU of one hidden layer for the block's rows:
// dY (LDS) -> D (LDS, in place, and global unless null), with a = (e - mean) r, u = g dY,
// ebar = r (u - mean(u) - a mean(u a)), D = ebar ELU'(z); pg / pb gain the row sums of dY a and
// dY of this thread's columns.  E: the layer's ELU outputs (LDS or global).
template <int RT, int NW>
__device__ __forceinline__ void rows_ln_backward(real* dY, int ld, const real* E, int lde,
                                                 const real* __restrict__ g, int n, int rows, const real (*st)[2],
                                                 real (*su)[2], real* D, real (&pg)[2], real (&pb)[2]) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c16 = lane & 15;
  for (int r = 4 * wv + (lane >> 4); r < 16 * RT; r += 4 * NW) {
    real s0 = RL(0.0), s1 = RL(0.0);
    if (r < rows) {
      const real mu = st[r][0], is = st[r][1];
      for (int c = c16; c < n; c += 16) {
        const real u = g[c] * dY[r * ld + c];
        s0 += u;
        s1 = m_fma(u, (E[r * lde + c] - mu) * is, s1);
      }
    }
    s0 = sum16(s0);
    s1 = sum16(s1);
    if (c16 == 0) {
      su[r][0] = s0 / (real)n;
      su[r][1] = s1 / (real)n;
    }
  }
  __syncthreads();
  const int G = ln_groups<NW>(n), cw = NW * SIM_WAVE / G, grp = tid / cw, nr = 16 * RT / G;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = tid % cw + h * NW * SIM_WAVE;
    if (c < n) {
      const real gc = g[c];
      for (int r = grp * nr; r < (grp + 1) * nr; ++r) {
        if (r >= rows) break;
        const real dy = dY[r * ld + c], e = E[r * lde + c];
        const real a = (e - st[r][0]) * st[r][1];
        pg[h] = m_fma(dy, a, pg[h]);
        pb[h] += dy;
        const real eb = st[r][1] * (gc * dy - su[r][0] - a * su[r][1]);
        const real d = eb * ((e > RL(0.0)) ? RL(1.0) : e + RL(1.0));
        dY[r * ld + c] = d;
        if (D) D[r * n + c] = d;
      }
    }
  }
}

// this block's gain / bias sums of a layer-normalised hidden layer (n columns) to dst[2 n]; the
// row groups of a narrow layer are added in order (buf: 1024 values of LDS)
template <int NW>
__device__ __forceinline__ void ln_flush(real* buf, real* dst, int n, const real (&pg)[2], const real (&pb)[2]) {
  const int tid = threadIdx.x, G = ln_groups<NW>(n), cw = NW * SIM_WAVE / G, grp = tid / cw;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = tid % cw + h * NW * SIM_WAVE;
    if (c < n) {
      buf[grp * 2 * n + c] = pg[h];
      buf[grp * 2 * n + n + c] = pb[h];
    }
  }
  __syncthreads();
  for (int c = tid; c < 2 * n; c += NW * SIM_WAVE) {
    real s = buf[c];
    for (int q = 1; q < G; ++q) s += buf[q * 2 * n + c];
    dst[c] = s;
  }
  __syncthreads();
}

// the block's rows of the network's input into LDS (zero past the rows and up to a multiple of 16
// columns); xs, if given, receives them
template <int R, int NW>
__device__ __forceinline__ void rows_input(const MlpNet& N, const int* perm, long m0, int rows, real* x, int ld, real* xs) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, K = N.d0, Kp = mlp_pad16(K);
  // every row number first, then the rows: two memory latencies for the block's rows
  long src[R / NW];
#pragma unroll
  for (int i = 0; i < R / NW; ++i) {
    const int r = wv + i * NW;
    src[i] = (r < rows) ? (perm ? (long)perm[m0 + r] : m0 + r) : 0;
  }
  for (int c = lane; c < Kp; c += SIM_WAVE) {
    real v[R / NW];
#pragma unroll
    for (int i = 0; i < R / NW; ++i) v[i] = (wv + i * NW < rows && c < K) ? N.x0[src[i] * K + c] : RL(0.0);
    const real sh = (N.shift && c < K) ? N.shift[c] : RL(0.0), sc = (N.shift && c < K) ? N.scale[c] : RL(1.0);
#pragma unroll
    for (int i = 0; i < R / NW; ++i) {
      const int r = wv + i * NW;
      const bool in = r < rows && c < K;
      if (N.shift && in) v[i] = (v[i] - sh) * sc;
      if (xs && in) xs[(m0 + r) * K + c] = v[i];
      x[r * ld + c] = v[i];
    }
  }
}

// the linear output of a critic for row r, V = w . x + b: TP lanes a row, every one gets it
template <int TP>
__device__ __forceinline__ real rows_output(const real* cur, int ld, const real* w, const real* b, int K, int r) {
  const int p = threadIdx.x % TP;
  real s = RL(0.0);
  for (int k = p; k < K; k += TP) s = m_fma(cur[r * ld + k], w[k], s);
#pragma unroll
  for (int o = TP / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o, SIM_WAVE);
  return s + b[0];
}

// The rows pass.  ROWS_VALUES: V[r] of the critic.  ROWS_FIT: the same on the minibatch's rows
// perm[0 .. M), then the adjoint of (1/M) sum (V - y)^2 back to every hidden layer; xs, H1 / H2
// (and Y1 / Y2) receive the layer inputs, V the output adjoint, D1 / D2 the hidden layers'
// adjoints.  ROWS_THETA: the hidden layers' adjoints from dL/da, with the window's activations.
struct RowsArgs {
  MlpNet N;
  const int* perm;
  const real* tgt;
  real *xs, *V;
  real* loss_part;   // [tiles] sums of squared errors
  real* lnpart;      // [blocks][lnw] gain / bias sums
  int lnw;
  int ld;            // row stride of an LDS buffer: pad16(widest layer) + 4
};

// What bounds the rows pass: the matrix instructions (a 32-row block of the 76-128-128-1 critic
// issues 208 of them per wave forward) and, with few rows, the chain of memory latencies
// (arguments, rows, each layer's first weights).  Keeping a tile's rows in LDS through all layers
// replaces one launch and one round trip of the activations per layer: 33792 rows of that
// critic's values take 33 us (54 TFLOP/s of the 150 a large FP32 product reaches), 92 us before (in
// cache; 85 and 142 us on rows and weights that are not).
// waves per SIMD the register allocation aims at
constexpr int rows_waves(int rt, int mode, bool ln) {
  if (sizeof(real) == 8) return mode == ROWS_VALUES ? 2 : 1;
  return mode == ROWS_VALUES ? (rt == 3 ? 3 : 4) : (ln ? 1 : 2);
}
template <int RT, int MODE, bool LN>
__global__ __launch_bounds__(MR_THREADS, rows_waves(RT, MODE, LN)) void k_mlp_rows(RowsArgs g) {
  extern __shared__ __attribute__((aligned(16))) char rows_lds[];
  constexpr int R = 16 * RT;
  __shared__ real stat[MR_MAXHIDL][R][2], su[R][2], red[R];
  const MlpNet& N = g.N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, ld = g.ld, L = N.L, M = N.M;
  real* const lds = reinterpret_cast<real*>(rows_lds);
  real pg1[2] = {RL(0.0), RL(0.0)}, pb1[2] = {RL(0.0), RL(0.0)}, pg2[2] = {RL(0.0), RL(0.0)}, pb2[2] = {RL(0.0), RL(0.0)};
  const int tiles = (M + R - 1) / R;
  // one tile a block, but where the gain / bias sums bound the blocks
  for (int tile = blockIdx.x; tile < tiles; tile += (LN && MODE != ROWS_VALUES) ? (int)gridDim.x : tiles) {
    const long m0 = (long)tile * R;
    const int rows = (int)((M - m0) < R ? (M - m0) : R);
    // the two buffers take turns: layer l's input and output are buffers l % 2 and (l + 1) % 2
    if constexpr (MODE != ROWS_THETA) {
      rows_input<R, MR_WAVES>(N, MODE == ROWS_FIT ? g.perm : nullptr, m0, rows, lds, ld, MODE == ROWS_FIT ? g.xs : nullptr);
      __syncthreads();
      auto forward = [&](int l, const real* W, const real* bias, int K, int no, real* Hg, const real* lg, const real* lb,
                         real* Yg) __attribute__((always_inline)) {
        const real* cur = lds + (l & 1) * R * ld;
        real* nxt = lds + ((l + 1) & 1) * R * ld;
        real* H = (MODE == ROWS_FIT) ? Hg + m0 * no : nullptr;
        auto epi = [&](int row, int n, real v) __attribute__((always_inline)) {
          if (n < no) {
            v += bias[n];
            v = v > RL(0.0) ? v : m_expm1(v);
            if (MODE == ROWS_FIT && row < rows) H[row * no + n] = v;
          } else {
            v = RL(0.0);
          }
          nxt[row * ld + n] = v;
        };
        if (no >= 128) rows_fwd<RT, 2>(cur, ld, W, K, no, (N.vec >> l) & 1, wv, MR_WAVES, epi);
        else rows_fwd<RT, 1>(cur, ld, W, K, no, (N.vec >> l) & 1, wv, MR_WAVES, epi);
        __syncthreads();
        if constexpr (LN) {
          rows_ln_stats<RT, MR_WAVES>(nxt, ld, no, N.eps, stat[l]);
          __syncthreads();
          for (int r = wv; r < rows; r += MR_WAVES)
            for (int c = lane; c < no; c += SIM_WAVE) {
              const real y = m_fma(lg[c], (nxt[r * ld + c] - stat[l][r][0]) * stat[l][r][1], lb[c]);
              nxt[r * ld + c] = y;
              if (MODE == ROWS_FIT) Yg[(m0 + r) * no + c] = y;
            }
          __syncthreads();
        }
      };
      if (L > 1) forward(0, N.W0, N.b0, N.d0, N.d1, N.H1, N.g1, N.be1, N.Y1);
      if (L > 2) forward(1, N.W1, N.b1, N.d1, N.d2, N.H2, N.g2, N.be2, N.Y2);
      {
        // (in a block of 48 rows the lanes past them repeat the last row)
        constexpr int TP = RT == 1 ? 16 : (RT == 2 ? 8 : 4);
        const int r = (tid / TP < R) ? tid / TP : R - 1, p = tid % TP;
        const real* cur = lds + ((L - 1) & 1) * R * ld;
        real* nxt = lds + (L & 1) * R * ld;
        const real V = rows_output<TP>(cur, ld, L == 1 ? N.W0 : (L == 2 ? N.W1 : N.W2), L == 1 ? N.b0 : (L == 2 ? N.b1 : N.b2),
                                      net_dim(N, L - 1), r);
        if constexpr (MODE == ROWS_VALUES) {
          if (p == 0 && tid / TP < rows) g.V[m0 + r] = V;
        } else {
          real d = RL(0.0), e2 = RL(0.0);
          if (r < rows) {
            const real e = V - g.tgt[g.perm[m0 + r]];
            d = RL(2.0) / (real)M * e;
            e2 = e * e;
            if (p == 0) g.V[m0 + r] = d;
          }
          for (int c = p; c < 16; c += TP) nxt[r * ld + c] = (c == 0) ? d : RL(0.0);
          if (p == 0) red[r] = e2;
        }
      }
      __syncthreads();
      if constexpr (MODE == ROWS_FIT) {
        if (wv == 0) {
          const real s = wave_sum(lane < R ? red[lane] : RL(0.0));
          if (lane == 0) g.loss_part[tile] = s;
        }
      }
    } else {
      const int na = net_dim(N, L), nap = mlp_pad16(na);
      for (int r = wv; r < R; r += MR_WAVES)
        for (int c = lane; c < nap; c += SIM_WAVE) {
          const long i = (m0 + r) * na + c;
          lds[(L & 1) * R * ld + r * ld + c] = (r < rows && c < na) ? squash_seed(N.da[i], N.act[i], N.mtu) : RL(0.0);
        }
      if constexpr (LN) {
        // the window's statistics, and the normalised layer inputs it consumed
        for (int i = tid; i < (L - 1) * R; i += MR_THREADS) {
          const int j = i / R, r = i % R;
          if (r < rows) {
            stat[j][r][0] = N.st[(m0 + r) * N.ldst + 2 * j];
            stat[j][r][1] = N.st[(m0 + r) * N.ldst + 2 * j + 1];
          }
        }
        __syncthreads();
        auto normalised = [&](int j, int n, const real* H, int ldh, const real* lg, const real* lb, real* Y)
            __attribute__((always_inline)) {
          for (int r = wv; r < rows; r += MR_WAVES)
            for (int c = lane; c < n; c += SIM_WAVE)
              Y[(m0 + r) * n + c] = m_fma(lg[c], (H[(m0 + r) * ldh + c] - stat[j][r][0]) * stat[j][r][1], lb[c]);
        };
        if (L > 1) normalised(0, N.d1, N.H1, N.ldh1, N.g1, N.be1, N.Y1);
        if (L > 2) normalised(1, N.d2, N.H2, N.ldh2, N.g2, N.be2, N.Y2);
      }
      __syncthreads();
    }
    if constexpr (MODE != ROWS_VALUES) {
      // back to hidden layer l (1-based) from the adjoint of layer l + 1's pre-activations
      auto back = [&](int l, const real* W, int K, int n, const real* Hg, int ldh, const real* lg, real* Dg, real (&pg)[2],
                      real (&pb)[2]) __attribute__((always_inline)) {
        const real* H = Hg + m0 * ldh;
        real* D = Dg + m0 * n;
        const real* cur = lds + ((l + 1) & 1) * R * ld;
        real* nxt = lds + (l & 1) * R * ld;
        const bool to_lds = LN || l > 1 || MODE == ROWS_FIT;
        auto epi = [&](int row, int c, real v) __attribute__((always_inline)) {
          if (to_lds) {
            nxt[row * ld + c] = c < n ? v : RL(0.0);
          } else if (c < n && row < rows) {
            const real hv = H[row * ldh + c];
            D[row * n + c] = v * (hv > RL(0.0) ? RL(1.0) : hv + RL(1.0));
          }
        };
        if (n >= 128) rows_dgrad<RT, 2>(cur, ld, W, K, n, wv, MR_WAVES, epi);
        else rows_dgrad<RT, 1>(cur, ld, W, K, n, wv, MR_WAVES, epi);
        __syncthreads();
        if (!LN && to_lds) {
          for (int r = wv; r < rows; r += MR_WAVES)
            for (int c = lane; c < n; c += SIM_WAVE) {
              const real hv = H[r * ldh + c];
              const real v = nxt[r * ld + c] * (hv > RL(0.0) ? RL(1.0) : hv + RL(1.0));
              nxt[r * ld + c] = v;
              D[r * n + c] = v;
            }
          __syncthreads();
        }
        if constexpr (LN) {
          rows_ln_backward<RT, MR_WAVES>(nxt, ld, H, ldh, lg, n, rows, stat[l - 1], su, D, pg, pb);
          __syncthreads();
        }
      };
      if (L > 2) back(2, N.W2, N.d3, N.d2, N.H2, N.ldh2, N.g2, N.D2, pg2, pb2);
      if (L > 1) back(1, N.W1, N.d2, N.d1, N.H1, N.ldh1, N.g1, N.D1, pg1, pb1);
    }
    __syncthreads();
  }
  if constexpr (LN && MODE != ROWS_VALUES) {
    real* dst = g.lnpart + (long)blockIdx.x * g.lnw;
    if (L > 1) ln_flush<MR_WAVES>(lds, dst, N.d1, pg1, pb1);
    if (L > 2) ln_flush<MR_WAVES>(lds, dst + 2 * N.d1, N.d2, pg2, pb2);
  }
}

// One minibatch tile of a critic fit: forward, loss adjoint, and per layer the weight gradient
// and the way back, all from LDS.  Each block leaves its own gradient (flat, in part), so the
// layer inputs and adjoints never reach memory; the traffic is the 256 blocks' gradients (27 MB
// written here, read by k_mlp_reduce).  Bound by the chain of memory latencies of a tile (rows,
// weights from another XCD's L2, gradients out) over the matrix instructions' 8 us: eight waves a
// block, two to a SIMD, against four: 32 us against 42.  A minibatch of 8192 rows of the
// 76-128-128-1 critic takes 40 us with its sum (a launch per layer and step: 140 us), 128 rows of a
// 5-64-64-1 critic 15 us (58 us), 5000 rows of a layer-normalised 37-64-64-1 critic 29 us (242 us).
struct FitArgs {
  MlpNet N;
  const int* perm;
  const real* tgt;
  real* part;        // [tiles][np]
  real* loss_part;   // [tiles]
  int np;
  int ow1, ow2, ob0, ob1, ob2, og1, og2;   // flat offsets (W_0 at 0; a bias beta follows its gain)
  int ld0, ld1, ld2;                       // row strides of the LDS buffers
  int p1, p2, e1, e2, pd;                  // their offsets: layer outputs, ELU outputs, output adjoint
};

// part[off_w + m ni + n] = sum over the block's rows of D[row][m] X[row][n], part[off_b + m] = sum
// of D[row][m]; D, X in LDS, zero in rows past the tile's (D) and in the padding columns
template <int RT, int NW>
__device__ __forceinline__ void rows_wgrad(const real* D, int ldd, const real* X, int ldx, int no, int ni, real* part,
                                           int off_w, int off_b) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, q = lane >> 4, c16 = lane & 15;
  const int tm = (no + 15) >> 4, tn = (ni + 15) >> 4;
  // ws rows of tiles at a time, NW / ws waves sharing one
  const int ws = tm >= NW ? NW : (tm >= NW / 2 ? NW / 2 : 1), wr = NW / ws;
  for (int mt = wv / wr; mt < tm; mt += ws) {
    real a[4 * RT], bs = RL(0.0);
#pragma unroll
    for (int s = 0; s < 4 * RT; ++s) {
      a[s] = D[(4 * s + q) * ldd + mt * 16 + c16];
      bs += a[s];
    }
    for (int t = wv % wr; t < tn; t += wr) {
      mfma_v4 acc = {RL(0.0), RL(0.0), RL(0.0), RL(0.0)};
      real b[4 * RT];
#pragma unroll
      for (int s = 0; s < 4 * RT; ++s) b[s] = X[(4 * s + q) * ldx + t * 16 + c16];
#pragma unroll
      for (int s = 0; s < 4 * RT; ++s) acc = mfma_16x16x4(a[s], b[s], acc);
      const int n = t * 16 + c16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = mt * 16 + mfma_row(RL(0.0), lane, r);
        if (m < no && n < ni) part[off_w + m * ni + n] = acc[r];
      }
    }
    bs += __shfl_xor(bs, 16, SIM_WAVE);
    bs += __shfl_xor(bs, 32, SIM_WAVE);
    if (q == 0 && wv % wr == 0 && mt * 16 + c16 < no) part[off_b + mt * 16 + c16] = bs;
  }
}

#define FIT_WAVES 8
template <int RT, bool LN>
__global__ __launch_bounds__(FIT_WAVES * SIM_WAVE) void k_mlp_fit(FitArgs g) {
  extern __shared__ __attribute__((aligned(16))) char rows_lds[];
  constexpr int R = 16 * RT, NW = FIT_WAVES;
  __shared__ real stat[MR_MAXHIDL][R][2], su[R][2], red[R], lnbuf[LN ? 1024 : 1];
  const MlpNet& N = g.N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, L = N.L, M = N.M;
  real* const lds = reinterpret_cast<real*>(rows_lds);
  const long m0 = (long)blockIdx.x * R;
  const int rows = (int)((M - m0) < R ? (M - m0) : R);
  real* part = g.part + (long)blockIdx.x * g.np;
  // x0 | y1 (layer inputs; y1, y2 turn into the adjoints D1, D2) | e1 | y2 | e2 | output adjoint
  real* y1 = lds + g.p1;
  real* y2 = lds + g.p2;
  real* e1 = LN ? lds + g.e1 : y1;
  real* e2 = LN ? lds + g.e2 : y2;
  real* dv = lds + g.pd;
  constexpr int LDV = 20;
  // this lane's row target, and a word of every 128-byte line of the weights: the weights were
  // written by other CUs a launch ago, and coming from there in one go they cost one latency, not
  // one per layer
  constexpr int TP = NW * SIM_WAVE / R;
  const real yr = (tid / TP < rows) ? g.tgt[g.perm[m0 + tid / TP]] : RL(0.0);
  real touch = RL(0.0);
  auto warm = [&](const real* W, int n) __attribute__((always_inline)) {
    for (int i = tid * (128 / (int)sizeof(real)); i < n; i += NW * SIM_WAVE * (128 / (int)sizeof(real))) touch += W[i];
  };
  if (L > 1) warm(N.W1, N.d1 * N.d2);
  rows_input<R, NW>(N, g.perm, m0, rows, lds, g.ld0, nullptr);
  __syncthreads();
  auto forward = [&](int l, const real* cur, int ldc, const real* W, const real* bias, int K, int no, real* e, real* y, int ldn,
                     const real* lg, const real* lb) __attribute__((always_inline)) {
    auto epi = [&](int row, int n, real v) __attribute__((always_inline)) {
      if (n < no) {
        v += bias[n];
        v = v > RL(0.0) ? v : m_expm1(v);
      } else {
        v = RL(0.0);
      }
      e[row * ldn + n] = v;
    };
    // eight column tiles give every wave one; below, the waves split the rows as well
    if (RT == 1 || no > 64) rows_fwd<RT, 1>(cur, ldc, W, K, no, (N.vec >> l) & 1, wv, NW, epi);
    else
      rows_fwd<1, 1>(cur + (wv & 1) * 16 * ldc, ldc, W, K, no, (N.vec >> l) & 1, wv >> 1, NW / 2,
                     [&](int row, int n, real v) __attribute__((always_inline)) { epi(row + (wv & 1) * 16, n, v); });
    __syncthreads();
    if constexpr (LN) {
      rows_ln_stats<RT, NW>(e, ldn, no, N.eps, stat[l]);
      __syncthreads();
      const int np16 = mlp_pad16(no);
      for (int r = wv; r < R; r += NW)
        for (int c = lane; c < np16; c += SIM_WAVE)
          y[r * ldn + c] = c < no ? m_fma(lg[c], (e[r * ldn + c] - stat[l][r][0]) * stat[l][r][1], lb[c]) : RL(0.0);
      __syncthreads();
    }
  };
  if (L > 1) forward(0, lds, g.ld0, N.W0, N.b0, N.d0, N.d1, e1, y1, g.ld1, N.g1, N.be1);
  if (L > 2) forward(1, y1, g.ld1, N.W1, N.b1, N.d1, N.d2, e2, y2, g.ld2, N.g2, N.be2);
  const real* top = L == 1 ? lds : (L == 2 ? y1 : y2);
  const int ldt = L == 1 ? g.ld0 : (L == 2 ? g.ld1 : g.ld2), dtop = L == 1 ? N.d0 : (L == 2 ? N.d1 : N.d2);
  {
    const int r = tid / TP, p = tid % TP;
    const real V = rows_output<TP>(top, ldt, L == 1 ? N.W0 : (L == 2 ? N.W1 : N.W2), L == 1 ? N.b0 : (L == 2 ? N.b1 : N.b2), dtop, r);
    real d = RL(0.0), s2 = RL(0.0);
    if (r < rows) {
      const real err = V - yr;
      d = RL(2.0) / (real)M * err;
      s2 = err * err;
    }
    for (int c = p; c < 16; c += TP) dv[r * LDV + c] = (c == 0) ? d : RL(0.0);
    if (p == 0) red[r] = s2;
  }
  __syncthreads();
  if (wv == 0) {
    const real s = wave_sum(lane < R ? red[lane] : RL(0.0));
    if (lane == 0) g.loss_part[blockIdx.x] = s;
  }
  rows_wgrad<RT, NW>(dv, LDV, top, ldt, 1, dtop, part, L == 1 ? 0 : (L == 2 ? g.ow1 : g.ow2),
                 L == 1 ? g.ob0 : (L == 2 ? g.ob1 : g.ob2));
  auto back = [&](int l, const real* cur, int ldc, const real* W, int K, int n, const real* e, real* y, int ldn, const real* lg,
                  int og) __attribute__((always_inline)) {
    __syncthreads();   // the weight gradient has read y before it turns into the adjoint
    auto epi = [&](int row, int c, real v) __attribute__((always_inline)) {
      if constexpr (!LN) {
        const real hv = e[row * ldn + c];
        v *= hv > RL(0.0) ? RL(1.0) : hv + RL(1.0);
      }
      y[row * ldn + c] = c < n ? v : RL(0.0);
    };
    if (RT == 1 || n > 64) rows_dgrad<RT, 1>(cur, ldc, W, K, n, wv, NW, epi);
    else
      rows_dgrad<1, 1>(cur + (wv & 1) * 16 * ldc, ldc, W, K, n, wv >> 1, NW / 2,
                       [&](int row, int c, real v) __attribute__((always_inline)) { epi(row + (wv & 1) * 16, c, v); });
    __syncthreads();
    if constexpr (LN) {
      real pg[2] = {RL(0.0), RL(0.0)}, pb[2] = {RL(0.0), RL(0.0)};
      rows_ln_backward<RT, NW>(y, ldn, e, ldn, lg, n, rows, stat[l - 1], su, nullptr, pg, pb);
      __syncthreads();
      ln_flush<NW>(lnbuf, part + og, n, pg, pb);
    }
  };
  if (L > 2) {
    back(2, dv, LDV, N.W2, 1, N.d2, e2, y2, g.ld2, N.g2, g.og2);
    rows_wgrad<RT, NW>(y2, g.ld2, y1, g.ld1, N.d2, N.d1, part, g.ow1, g.ob1);
  }
  if (L > 1) {
    back(1, L > 2 ? y2 : dv, L > 2 ? g.ld2 : LDV, N.W1, N.d2, N.d1, e1, y1, g.ld1, N.g1, g.og1);
    rows_wgrad<RT, NW>(y1, g.ld1, lds, g.ld0, N.d1, N.d0, part, 0, g.ob0);
  }
  if (touch != touch && M < 0) g.loss_part[0] = touch;   // never: keeps the loads
}

// Weight and bias gradients of every layer, one launch: G_l [no][ni + 1] = sum over rows of
// D_{l+1}[row][no] (X_l[row][ni], 1).  A wave owns a 32x32 tile of one layer and one chunk of the
// rows; its operands come straight from global memory in the matrix instruction's own layout
// (16 consecutive columns of four rows), eight row quads requested ahead of their products; the
// four waves of a block are neighbouring tiles of one chunk and share rows through L1.  Blocks of
// one chunk run on one XCD (chunk mod 8), so that its rows come into one L2 only.
#define WG_T SIM_WG_T   // tile side
#define WG_ST 8      // row quads per stage (the bias sum is written for eight)
#define WG_XCD 8
struct WgradArgs {
  MlpNet N;
  const real* dv;               // adjoint of the network's output; null: formed from dL/da
  const real* xs;               // layer 0's input rows as gathered (a fit), else null: N.x0 with its affine
  int t1, t2, t3;               // first tile of layers 1, 2, and the tile count
  int ow1, ow2, ob0, ob1, ob2;  // flat offsets
  int chunk, splits;            // rows per chunk (a multiple of 4), chunks
  real* part;                   // [chunks][np]
  long np;
};

__global__ __launch_bounds__(MR_THREADS) void k_mlp_wgrad(WgradArgs g) {
  const MlpNet& N = g.N;
  const int lane = threadIdx.x & 63, q = lane >> 4, c16 = lane & 15, L = N.L;
  const int tb = (g.t3 + MR_WAVES - 1) / MR_WAVES;   // blocks of one chunk
  const int slot = (int)blockIdx.x / WG_XCD;
  const int z = (int)blockIdx.x % WG_XCD + WG_XCD * (slot / tb);
  const int u = __builtin_amdgcn_readfirstlane((slot % tb) * MR_WAVES + ((int)threadIdx.x >> 6));
  if (z >= g.splits || u >= g.t3) return;
  const int l = u >= g.t2 ? 2 : (u >= g.t1 ? 1 : 0);
  const int ni = l == 0 ? N.d0 : (l == 1 ? N.d1 : N.d2), no = l == 0 ? N.d1 : (l == 1 ? N.d2 : N.d3);
  const int tn = (ni + WG_T - 1) / WG_T, t = u - (l == 0 ? 0 : (l == 1 ? g.t1 : g.t2));
  const int m0 = (t / tn) * WG_T, n0 = (t % tn) * WG_T;
  const int kb = z * g.chunk, ke = min(N.M, kb + g.chunk);
  const bool ln = N.g1 != nullptr;
  const real* X = l == 0 ? (g.xs ? g.xs : N.x0) : (l == 1 ? (ln ? N.Y1 : N.H1) : (ln ? N.Y2 : N.H2));
  const long ldx = (l == 0 || ln) ? ni : (l == 1 ? N.ldh1 : N.ldh2);
  const bool seed = l == L - 1 && !g.dv;
  const real* D = l == L - 1 ? (seed ? N.da : g.dv) : (l == 0 ? N.D1 : N.D2);
  const bool aff = l == 0 && !g.xs && N.shift;
  bool mok[2], nok[2];
  int mc[2], nc[2];
  real sh[2] = {RL(0.0), RL(0.0)}, sc[2] = {RL(1.0), RL(1.0)};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + 16 * i + c16, n = n0 + 16 * i + c16;
    mok[i] = m < no;
    mc[i] = mok[i] ? m : 0;
    nok[i] = n < ni;
    nc[i] = nok[i] ? n : 0;
    if (aff) { sh[i] = N.shift[nc[i]]; sc[i] = N.scale[nc[i]]; }
  }
  mfma_v4 acc[2][2];
  real accb[2] = {RL(0.0), RL(0.0)};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = mfma_v4{RL(0.0), RL(0.0), RL(0.0), RL(0.0)};
  // SEED: D from dL/da and the actions; AFF: X through the input's affine.  Fixed per wave and
  // compiled apart: a test inside the loads' loop made the compiler wait for every load (a stage
  // of 32 rows took 6.8 us instead of one memory latency)
  auto run = [&](auto SEED, auto AFF) __attribute__((always_inline)) {
    // one stage's operands: row quad s of the stage holds rows k + 4 s + q
    auto load = [&](real (&a)[WG_ST][2], real (&b)[WG_ST][2], int k) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < WG_ST; ++s) {
        const int row = k + 4 * s + q;
        const bool ok = row < ke;
        const long rr = ok ? row : kb;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const long ai = rr * no + mc[i];
          real av = D[ai];
          if constexpr (SEED) av = squash_seed(av, N.act[ai], N.mtu);
          real bv = X[rr * ldx + nc[i]];
          if constexpr (AFF) bv = (bv - sh[i]) * sc[i];
          a[s][i] = (ok && mok[i]) ? av : RL(0.0);
          b[s][i] = (ok && nok[i]) ? bv : RL(0.0);
        }
      }
    };
    real a[WG_ST][2], b[WG_ST][2], an[WG_ST][2], bn[WG_ST][2];
    load(a, b, kb);
    for (int k = kb; k < ke; k += 4 * WG_ST) {
      if (k + 4 * WG_ST < ke) load(an, bn, k + 4 * WG_ST);
#pragma unroll
      for (int s = 0; s < WG_ST; ++s) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma_16x16x4(a[s][i], b[s][j], acc[i][j]);
        }
      }
      // the bias column in stage sums of eight rows a lane
#pragma unroll
      for (int i = 0; i < 2; ++i)
        accb[i] += ((a[0][i] + a[1][i]) + (a[2][i] + a[3][i])) + ((a[4][i] + a[5][i]) + (a[6][i] + a[7][i]));
#pragma unroll
      for (int s = 0; s < WG_ST; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          a[s][i] = an[s][i];
          b[s][i] = bn[s][i];
        }
    }
  };
  if (seed && aff) run(std::true_type{}, std::true_type{});
  else if (seed) run(std::true_type{}, std::false_type{});
  else if (aff) run(std::false_type{}, std::true_type{});
  else run(std::false_type{}, std::false_type{});
  // the bias gradient: this lane's column of D over its row quads' rows, then over the four of them
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    accb[i] += __shfl_xor(accb[i], 16, SIM_WAVE);
    accb[i] += __shfl_xor(accb[i], 32, SIM_WAVE);
  }
  real* out = g.part + (long)z * g.np;
  const int ow = l == 0 ? 0 : (l == 1 ? g.ow1 : g.ow2), ob = l == 0 ? g.ob0 : (l == 1 ? g.ob1 : g.ob2);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 16 * i + mfma_row(RL(0.0), lane, r);
      if (m < no) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int n = n0 + 16 * j + c16;
          if (n < ni) out[ow + (long)m * ni + n] = acc[i][j][r];
        }
      }
    }
  if (n0 == 0 && q == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (mok[i]) out[ob + m0 + 16 * i + c16] = accb[i];
  }
}

// Adam (Kingma and Ba): m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2,
// p -= lr (m / bc1) / (sqrt(v / bc2) + eps) with bc = 1 - b^t; element i of the flat gradient and
// moments belongs to the tensor whose range of the list holds it.  LIST_END: the search ends with
// the list, which is right for millions of elements; without it the whole list is requested at once,
// one memory latency for a block that has only this to wait for (0.7 us of a fit's minibatch).
template <bool LIST_END>
__device__ __forceinline__ void adam_element(const LearnAdamT<real>& A, long i, real gi) {
  real* p = A.p[0] + i;
  long base = 0;
#pragma unroll
  for (int t = 1; t < SIM_MAX_TENSORS; ++t) {
    if (LIST_END && t >= A.n) break;
    base += A.size[t - 1];
    if (t < A.n && i >= base) p = A.p[t] + (i - base);
  }
  const real m = A.b1 * A.m[i] + (RL(1.0) - A.b1) * gi;
  const real v = A.b2 * A.v[i] + (RL(1.0) - A.b2) * gi * gi;
  A.m[i] = m;
  A.v[i] = v;
  *p -= A.lr * (m / A.bc1) / (m_sqrt(v / A.bc2) + A.eps);
}

// Sum of the partial gradients (and, with layer normalisation, of the row blocks' gain and bias
// sums where those are kept apart) into T.out or straight into the Adam step of a fit.  A block
// takes 64 parameters; its 16 waves each sum every 16th partial, four loads in flight, and the
// wave sums are added in order.  The last block of a fit forms the minibatch's mean squared error
// from the row tiles' sums.
#define RD_WAVES 16
struct ReduceArgs {
  const real* part;
  int splits;
  long np;
  const real* lnpart;             // gain / bias sums of the row blocks (null: part holds them)
  int lnw, ln_blocks;
  long og1, og2;                  // flat offsets of the hidden layers' gains
  int n1, n2;                     // their widths, twice
  real* out;                      // the gradient, or
  int fit;                        // the Adam step
  LearnAdamT<real> A;
  const real* loss_part;
  int n_loss, rows;
  real* loss_out;
};

__global__ __launch_bounds__(RD_WAVES * SIM_WAVE) void k_mlp_reduce(ReduceArgs g) {
  __shared__ real red[RD_WAVES][SIM_WAVE];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const bool loss = g.fit && blockIdx.x == gridDim.x - 1;
  const long i = (long)blockIdx.x * SIM_WAVE + lane;
  const real* p = g.part + i;
  int n = g.splits, z = wv;
  long stride = g.np;
  if (loss) {
    p = g.loss_part;
    n = g.n_loss;
    z = (int)threadIdx.x;
  } else if (g.lnpart) {
    if (i >= g.og1 && i < g.og1 + g.n1) { p = g.lnpart + (i - g.og1); n = g.ln_blocks; stride = g.lnw; }
    if (i >= g.og2 && i < g.og2 + g.n2) { p = g.lnpart + g.n1 + (i - g.og2); n = g.ln_blocks; stride = g.lnw; }
  }
  const int step = loss ? RD_WAVES * SIM_WAVE : RD_WAVES;
  if (loss) stride = 1;
  real s[4] = {RL(0.0), RL(0.0), RL(0.0), RL(0.0)};
  if (loss || i < g.np) {
    for (; z + 3 * step < n; z += 4 * step) {
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += p[(z + u * step) * stride];
    }
    for (; z < n; z += step) s[0] += p[z * stride];
  }
  red[wv][lane] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (wv != 0) return;
  real t = red[0][lane];
#pragma unroll
  for (int w = 1; w < RD_WAVES; ++w) t += red[w][lane];
  if (loss) {
    t = wave_sum(t);
    if (lane == 0 && g.loss_out) *g.loss_out = t / (real)g.rows;
  } else if (i < g.np) {
    if (g.fit) adam_element<false>(g.A, i, t);
    else g.out[i] = t;
  }
}

// dL/dlog_std[i] = sum over rows of dL/dy[row][i] exp(log_std[i]) eps[row][i] (the
// reparameterised sample y = mu + exp(log_std) eps); one block per action, a fixed-order
// tree over 256 per-thread partial sums, so the result is reproducible
__global__ __launch_bounds__(256) void k_log_std_grad(const real* __restrict__ da, const real* __restrict__ act,
                                                      const real* __restrict__ eps, const real* __restrict__ log_std,
                                                      long rows, int na, int mtu, real* __restrict__ out) {
  __shared__ real part[256];
  const int i = blockIdx.x, tid = threadIdx.x;
  real s = RL(0.0);
#pragma unroll 4
  for (long r = tid; r < rows; r += 256) s += squash_seed(da[r * na + i], act[r * na + i], mtu) * eps[r * na + i];
  part[tid] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) part[tid] += part[tid + w];
    __syncthreads();
  }
  if (tid == 0) out[i] = part[0] * m_exp(log_std[i]);
}

// ---------------------------------------------------------------- launches
#define MR_CUS SIM_CUS
static MlpNet mlp_net(const ThetaArgsT<real>& T) {
  MlpNet N = {};
  N.M = T.M;
  N.L = T.nl;
  N.d0 = T.dims[0]; N.d1 = T.dims[1]; N.d2 = T.nl > 1 ? T.dims[2] : 0; N.d3 = T.nl > 2 ? T.dims[3] : 0;
  for (int l = 0; l < T.nl; ++l)
    if (T.dims[l] % 4 == 0 && reinterpret_cast<uintptr_t>(T.W[l]) % (4 * sizeof(real)) == 0) N.vec |= 1 << l;
  N.mtu = T.mtu;
  N.W0 = T.W[0]; N.W1 = T.W[1]; N.W2 = T.W[2];
  N.b0 = T.b[0]; N.b1 = T.b[1]; N.b2 = T.b[2];
  N.x0 = T.x0; N.shift = T.x_shift; N.scale = T.x_scale;
  N.H1 = T.H[1]; N.H2 = T.H[2];
  N.ldh1 = (int)(T.ldH[1] ? T.ldH[1] : N.d1);
  N.ldh2 = (int)(T.ldH[2] ? T.ldH[2] : N.d2);
  N.D1 = T.d0; N.D2 = T.d1;
  N.da = T.da; N.act = T.act;
  if (T.ln) {
    N.g1 = T.lng[0]; N.be1 = T.lnb[0]; N.g2 = T.lng[1]; N.be2 = T.lnb[1];
    N.Y1 = T.Y[1]; N.Y2 = T.Y[2];
    N.st = T.st;
    N.ldst = (int)T.ldst;
    N.eps = T.ln_eps;
  }
  return N;
}
static int mlp_ln_width(const ThetaArgsT<real>& T) {
  int w = 0;
  if (T.ln)
    for (int l = 1; l < T.nl; ++l) w += 2 * T.dims[l];
  return w;
}
static long mlp_params(const ThetaArgsT<real>& T) {
  long n = mlp_ln_width(T);
  for (int l = 0; l < T.nl; ++l) n += (long)T.dims[l + 1] * (T.dims[l] + 1);
  return n;
}

// above 64 KB of dynamic LDS a kernel must be allowed it
template <class K>
static int allow_lds(K* kernel, size_t lds) {
  if (lds <= 65536) return 0;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) ==
                 hipSuccess ? 0 : -1;
}
template <int RT, int MODE, bool LN>
static int launch_rows_as(const RowsArgs& g, int blocks, size_t lds, hipStream_t s) {
  if (allow_lds(&k_mlp_rows<RT, MODE, LN>, lds)) return -1;
  hipLaunchKernelGGL((k_mlp_rows<RT, MODE, LN>), dim3(blocks), dim3(MR_THREADS), lds, s, g);
  return 0;
}

// 32 rows a block where that still gives every CU a block, else 16 (also where 32 rows of the
// widest layer take more than 64 KB of LDS: with up to 144 KB a CU has one block, and values of
// 32768 rows took 1.1 times as long for 512 columns and 1.5 for 400); with layer normalisation the blocks are as many as
// the partial-sum buffer holds.  *n_blocks: the blocks launched (rows of lnpart), *n_tiles: the row
// tiles (entries of loss_part).
template <int MODE>
static int launch_rows(RowsArgs& g, const ThetaArgsT<real>& T, int* n_blocks, int* n_tiles, hipStream_t s) {
  int w = 16;
  // (the policy gradient's way back starts at the actions and leaves its last layer in memory)
  for (int l = (MODE == ROWS_THETA) ? (T.ln ? 1 : 2) : 0; l <= T.nl; ++l)
    if (l < T.nl || MODE == ROWS_THETA) w = w > T.dims[l] ? w : T.dims[l];
  g.N = mlp_net(T);
  g.ld = mlp_pad16(w) + 4;
  g.lnw = mlp_ln_width(T);
  g.lnpart = T.lnpart;
  const size_t row_bytes = 2 * (size_t)g.ld * sizeof(real);
  int rt = (T.M >= 32 * MR_CUS && 32 * row_bytes <= 65536) ? 2 : 1;
  // A CU holds four 32-row tiles of values or three of 48 rows (FP64: two of either), and a round of
  // tiles takes about as long as it has rows: 48 rows where their rounds hold no more rows.  A
  // 76-128-128-1 critic in FP32: 33792 rows 44 us with 32 rows a block (two rounds) and 33 us with 48
  // (one), 69632 rows 1.10 and 73728 rows 1.14 times faster, 40960 rows 5 % slower (two rounds of either).
  constexpr int b2 = sizeof(real) == 8 ? 2 : 4, b3 = sizeof(real) == 8 ? 2 : 3;
  auto round_rows = [&](int r, int b) { return (T.M + 16L * r * b * MR_CUS - 1) / (16L * r * b * MR_CUS) * r * b; };
  if (MODE == ROWS_VALUES && rt == 2 && 48 * row_bytes <= 53248 && round_rows(3, b3) <= round_rows(2, b2)) rt = 3;
  const int tiles = (T.M + 16 * rt - 1) / (16 * rt);
  int blocks = tiles;
  if (T.ln && MODE != ROWS_VALUES && g.lnw > 0 && blocks > T.lnpart_cap / g.lnw) blocks = (int)(T.lnpart_cap / g.lnw);
  if (n_blocks) *n_blocks = blocks;
  if (n_tiles) *n_tiles = tiles;
  const size_t lds = 16 * rt * row_bytes;
  if (rt == 3) {
    if constexpr (MODE == ROWS_VALUES)
      return T.ln ? launch_rows_as<3, MODE, true>(g, blocks, lds, s) : launch_rows_as<3, MODE, false>(g, blocks, lds, s);
  }
  if (T.ln) return rt == 2 ? launch_rows_as<2, MODE, true>(g, blocks, lds, s) : launch_rows_as<1, MODE, true>(g, blocks, lds, s);
  return rt == 2 ? launch_rows_as<2, MODE, false>(g, blocks, lds, s) : launch_rows_as<1, MODE, false>(g, blocks, lds, s);
}

// Row chunks of the weight gradient: as many as sim_wgrad_chunks has use for and the partial buffer
// holds; one chunk writes its gradient straight to T.out.
static void launch_wgrad(WgradArgs& g, const ThetaArgsT<real>& T, hipStream_t s) {
  g.t1 = sim_wgrad_tiles(T.dims[1], T.dims[0]);
  g.t2 = g.t1 + (T.nl > 1 ? sim_wgrad_tiles(T.dims[2], T.dims[1]) : 0);
  g.t3 = g.t2 + (T.nl > 2 ? sim_wgrad_tiles(T.dims[3], T.dims[2]) : 0);
  g.ow1 = (int)T.off_w[1]; g.ow2 = (int)T.off_w[2];
  g.ob0 = (int)T.off_b[0]; g.ob1 = (int)T.off_b[1]; g.ob2 = (int)T.off_b[2];
  g.np = mlp_params(T);
  const long cap = T.part_cap / g.np;
  long n = sim_wgrad_chunks(T.dims, T.nl, T.M);
  n = n < cap ? n : cap;
  if (n >= WG_XCD) n = n / WG_XCD * WG_XCD;
  if (n < 1) n = 1;
  g.chunk = (int)(((T.M + n - 1) / n + 3) / 4 * 4);
  g.splits = (T.M + g.chunk - 1) / g.chunk;
  g.part = (g.splits > 1) ? T.part : T.out;
  const int tb = (g.t3 + MR_WAVES - 1) / MR_WAVES, zs = (g.splits + WG_XCD - 1) / WG_XCD;
  hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)(WG_XCD * tb * zs)), dim3(MR_THREADS), 0, s, g);
}

// every field but the step's own (a caller may use Q again for a minibatch that takes another
// route): the gain / bias sums lie apart from the partial gradients or among them
static void reduce_args(ReduceArgs& Q, const ThetaArgsT<real>& T, const real* part, int splits, int ln_blocks, bool ln_apart) {
  const bool apart = T.ln && ln_apart;
  Q.part = part;
  Q.splits = splits;
  Q.np = mlp_params(T);
  Q.lnpart = apart ? T.lnpart : nullptr;
  Q.lnw = apart ? mlp_ln_width(T) : 0;
  Q.ln_blocks = apart ? ln_blocks : 0;
  Q.og1 = apart ? T.off_g[0] : 0;
  Q.n1 = apart ? 2 * T.dims[1] : 0;
  Q.og2 = apart && T.nl > 2 ? T.off_g[1] : 0;
  Q.n2 = apart && T.nl > 2 ? 2 * T.dims[2] : 0;
}
