// The learning-episode update that follows a window (Sec. 3.3, Algorithm "SHAC"): one Adam
// step of the policy, TD-lambda value estimates of the window's states from the target
// critic, the critic's mean-squared-error fit over shuffled minibatches with Adam, and the
// smooth update of the target critic.  The contractions run on the matrix cores through the
// kernels of the policy-parameter gradient (sim_gemm.h, sim_layers.h).
//
// Included inside a namespace with `real` defined as float or double, after sim_math.h,
// sim_gemm.h and sim_layers.h.

// one Adam step (adam_element) over every tensor of a list in one launch
__global__ void k_adam_multi(LearnAdamT<real> A, long total) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  adam_element<true>(A, i, A.g[i]);
}

// target <- alpha target + (1 - alpha) online over every tensor of a list in one launch (a
// launch per tensor spent 20 us on the six tensors of a 27 k-parameter critic); element i of
// the list belongs to the tensor whose range holds it
__global__ void k_soft_update(SoftUpdateT<real> A, long total) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  real* t = A.t[0] + i;
  const real* o = A.o[0] + i;
  long base = 0;
#pragma unroll
  for (int k = 1; k < SIM_MAX_TENSORS; ++k) {
    if (k >= A.n) break;
    base += A.size[k - 1];
    if (i >= base) {
      t = A.t[k] + (i - base);
      o = A.o[k] + (i - base);
    }
  }
  *t = A.alpha * *t + (RL(1.0) - A.alpha) * *o;
}

// TD-lambda estimates, one thread per env, by the backward recursion
// G_t = r_t + gamma ((1 - lambda) V_{t+1} + lambda G_{t+1}) from G_h = V_h, which equals the
// lambda-weighted average of the k-step returns of the definition.
// r [h][N], v [h+1][N] (values of s_0 .. s_h; s_0's is not used), out [h][N]
#define TD_BATCH 8
__global__ void k_td_lambda(const real* __restrict__ r, const real* __restrict__ v, const uint8_t* __restrict__ done,
                            int h, int N, real gamma, real lam, real* __restrict__ out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  real G = v[(size_t)h * N + e];
  // The recursion is serial but its inputs are not: TD_BATCH frames are requested at a time, so
  // a thread waits for one memory latency per batch instead of one per frame.
  for (int t1 = h - 1; t1 >= 0; t1 -= TD_BATCH) {
    real rt[TD_BATCH], vt[TD_BATCH];
    bool dn[TD_BATCH];
#pragma unroll
    for (int u = 0; u < TD_BATCH; ++u) {
      const size_t t = (size_t)(t1 - u > 0 ? t1 - u : 0);
      rt[u] = r[t * N + e];
      vt[u] = v[(t + 1) * N + e];
      dn[u] = done && done[t * N + e];
    }
#pragma unroll
    for (int u = 0; u < TD_BATCH; ++u) {
      if (t1 - u < 0) break;
      // a frame that ended in termination returns its reward alone: every k-step return from
      // it stops there and the fallen state has no value (s_{t+1} is already the reset state)
      if (dn[u]) G = rt[u];
      else G = rt[u] + gamma * ((RL(1.0) - lam) * vt[u] + lam * G);
      out[(size_t)(t1 - u) * N + e] = G;
    }
  }
}

// minibatch rows: x[b] = obs[perm[b]], y[b] = targets[perm[b]]
// (normalised with the running statistics when given: x = (o - mean) * inv_std)
__global__ void k_gather_rows(const real* __restrict__ obs, const real* __restrict__ tgt, const int* __restrict__ perm,
                              int B, int od, const real* __restrict__ mean, const real* __restrict__ inv_std,
                              real* __restrict__ x, real* __restrict__ y) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)B * od) return;
  const int b = (int)(i / od), c = (int)(i % od);
  const int r = perm[b];
  real v = obs[(long)r * od + c];
  if (mean) v = (v - mean[c]) * inv_std[c];
  x[i] = v;
  if (c == 0) y[b] = tgt[r];
}

// Running observation statistics (Sec. 3.3): merges a batch of rows into the count, mean
// and (population) variance of every observation seen before, by the pairwise update of
// Chan, Golub and LeVeque: with the batch's own mean m_b and sum of squared deviations
// M2_b, delta = m_b - mean, n = count + rows,
//   mean' = mean + delta rows / n,   var' = (var count + M2_b + delta^2 count rows / n) / n,
// and inv_std = 1 / sqrt(var' + eps).  All sums in FP64, in a fixed order.
__device__ __forceinline__ void os_merge(real* mean, real* var, real* inv_std, int c, double count, double rows,
                                         double bm, double m2b, double eps) {
  const double n = count + rows;
  const double m0 = count > 0.0 ? (double)mean[c] : 0.0;
  const double v0 = count > 0.0 ? (double)var[c] : 0.0;
  const double delta = bm - m0;
  const double mn = m0 + delta * (rows / n);
  const double vn = (v0 * count + m2b + delta * delta * (count * rows / n)) / n;
  mean[c] = (real)mn;
  var[c] = (real)vn;
  inv_std[c] = (real)(1.0 / sqrt(vn + eps));
}

// Without a workspace: a block owns 64 columns; its 16 row groups read consecutive columns of a
// row (coalesced), twice (the mean, then the deviations).  Each thread keeps eight independent
// partial sums so that eight loads are in flight at once.
#define OS_COLS 64
#define OS_GROUPS 16
#define OS_UNROLL 8

// sum over rows r = grp, grp + OS_GROUPS, ... of f(x[r][c]), in a fixed order
template <class F>
__device__ __forceinline__ double os_column_sum(const real* __restrict__ x, long rows, int od, int c, int grp, F f) {
  double p[OS_UNROLL];
#pragma unroll
  for (int u = 0; u < OS_UNROLL; ++u) p[u] = 0.0;
  long r = grp;
  for (; r + (long)(OS_UNROLL - 1) * OS_GROUPS < rows; r += (long)OS_UNROLL * OS_GROUPS) {
#pragma unroll
    for (int u = 0; u < OS_UNROLL; ++u) p[u] += f((double)x[(r + (long)u * OS_GROUPS) * od + c]);
  }
  for (; r < rows; r += OS_GROUPS) p[0] += f((double)x[r * od + c]);
  return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
}
__global__ __launch_bounds__(OS_COLS * OS_GROUPS) void k_obs_stats(const real* __restrict__ x, long rows, int od,
                                                                    double count, real* __restrict__ mean,
                                                                    real* __restrict__ var, real* __restrict__ inv_std,
                                                                    double eps) {
  __shared__ double red[OS_GROUPS][OS_COLS];
  __shared__ double bmean[OS_COLS];
  const int cl = threadIdx.x % OS_COLS, grp = threadIdx.x / OS_COLS;
  const int c = blockIdx.x * OS_COLS + cl;
  const bool ok = c < od;
  double s = 0.0, q = 0.0;
  if (ok) s = os_column_sum(x, rows, od, c, grp, [](double v) { return v; });
  red[grp][cl] = s;
  __syncthreads();
  if (grp == 0) {
    double t = 0.0;
    for (int g = 0; g < OS_GROUPS; ++g) t += red[g][cl];
    bmean[cl] = t / (double)rows;
  }
  __syncthreads();
  const double bm = bmean[cl];
  if (ok) q = os_column_sum(x, rows, od, c, grp, [bm](double v) { const double d = v - bm; return d * d; });
  red[grp][cl] = q;
  __syncthreads();
  if (grp == 0 && ok) {
    double m2b = 0.0;
    for (int g = 0; g < OS_GROUPS; ++g) m2b += red[g][cl];
    os_merge(mean, var, inv_std, c, count, (double)rows, bm, m2b, eps);
  }
}

// With a workspace: the rows are read once, by as many blocks as there are chunks of them.  The
// column blocks above leave 2 of 256 CUs working on a 76-column batch: 32768 rows of it take
// 221 us there and 12.4 us here (10 MB read, two launches; the rows still in cache).  A block of
// OSP_THREADS threads
// takes OSP_UNROLL rows for each of its row groups and w consecutive columns, so that its threads
// read consecutive words, holds them in registers, and leaves its rows' column sums and sums of
// squared deviations from its own column means; k_obs_stats_merge joins the chunks:
//   M2 = sum_b (M2_b + n_b (mean_b - mean)^2).
#define OSP_THREADS SIM_OSP_THREADS
#define OSP_UNROLL SIM_OSP_UNROLL
__global__ __launch_bounds__(OSP_THREADS) void k_obs_stats_part(const real* __restrict__ x, long rows, int od, int w,
                                                                 int groups, double* __restrict__ part) {
  __shared__ double red[OSP_THREADS];
  const int tid = threadIdx.x, grp = tid / w, cl = tid % w;
  const int c = blockIdx.y * w + cl;
  const bool on = grp < groups && c < od;
  const long r0 = (long)blockIdx.x * groups * OSP_UNROLL;
  const long nb = min((long)groups * OSP_UNROLL, rows - r0);
  real v[OSP_UNROLL];
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < OSP_UNROLL; ++u) {
    const long r = r0 + (long)u * groups + grp;
    v[u] = (on && r < rows) ? x[r * od + c] : RL(0.0);
  }
#pragma unroll
  for (int u = 0; u < OSP_UNROLL; ++u) s += (double)v[u];
  red[tid] = s;
  __syncthreads();
  double sum = 0.0;
  for (int g = 0; g < groups; ++g) sum += red[g * w + cl];
  const double bm = sum / (double)nb;
  double q = 0.0;
#pragma unroll
  for (int u = 0; u < OSP_UNROLL; ++u) {
    const double d = (double)v[u] - bm;
    if (r0 + (long)u * groups + grp < rows) q += d * d;
  }
  __syncthreads();
  red[tid] = q;
  __syncthreads();
  if (grp == 0 && on) {
    double m2 = 0.0;
    for (int g = 0; g < groups; ++g) m2 += red[g * w + cl];
    part[(size_t)blockIdx.x * od + c] = sum;
    part[((size_t)gridDim.x + blockIdx.x) * od + c] = m2;
  }
}
// A block joins the chunks of 16 columns, 64 groups of chunks side by side (a few chunks each:
// the join is a chain of memory latencies, 18 us with the column blocks' 64 x 16 split).
#define OSM_COLS 16
#define OSM_GROUPS 64
__device__ __forceinline__ double osm_sum(double (*red)[OSM_COLS], double s, int cl, int grp) {
  __syncthreads();
  red[grp][cl] = s;
  __syncthreads();
  for (int w = OSM_GROUPS / 2; w > 0; w >>= 1) {
    if (grp < w) red[grp][cl] += red[grp + w][cl];
    __syncthreads();
  }
  return red[0][cl];
}
__global__ __launch_bounds__(OSM_COLS * OSM_GROUPS) void k_obs_stats_merge(const double* __restrict__ part, int chunks,
                                                                            long chunk_rows, long rows, int od,
                                                                            double count, real* __restrict__ mean,
                                                                            real* __restrict__ var,
                                                                            real* __restrict__ inv_std, double eps) {
  __shared__ double red[OSM_GROUPS][OSM_COLS];
  const int cl = threadIdx.x % OSM_COLS, grp = threadIdx.x / OSM_COLS;
  const int c = blockIdx.x * OSM_COLS + cl;
  const bool ok = c < od;
  const double* sp = part + (ok ? c : 0);
  const double* mp = sp + (size_t)chunks * od;
  double s = 0.0, q = 0.0;
  for (int b0 = grp; b0 < chunks; b0 += OSM_GROUPS * 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = (b0 + u * OSM_GROUPS < chunks) ? sp[(size_t)(b0 + u * OSM_GROUPS) * od] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  const double bm = osm_sum(red, s, cl, grp) / (double)rows;
  for (int b0 = grp; b0 < chunks; b0 += OSM_GROUPS * 4) {
    double v[4], m2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = b0 + u * OSM_GROUPS < chunks;
      v[u] = in ? sp[(size_t)(b0 + u * OSM_GROUPS) * od] : 0.0;
      m2[u] = in ? mp[(size_t)(b0 + u * OSM_GROUPS) * od] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long b = b0 + u * OSM_GROUPS;
      if (b < chunks) {
        const double nb = (double)min(chunk_rows, rows - b * chunk_rows);
        const double d = v[u] / nb - bm;
        q += m2[u] + nb * d * d;
      }
    }
  }
  const double m2b = osm_sum(red, q, cl, grp);
  if (grp == 0 && ok) os_merge(mean, var, inv_std, c, count, (double)rows, bm, m2b, eps);
}

// output adjoint of the mean squared error (1/B) sum (V - y)^2
__global__ void k_mse_seed(const real* __restrict__ V, const real* __restrict__ y, int B, real* __restrict__ d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < B) d[i] = RL(2.0) / (real)B * (V[i] - y[i]);
}

// the minibatch's mean squared error before the step, by a fixed-order tree (one block)
__global__ __launch_bounds__(256) void k_mse_loss(const real* __restrict__ V, const real* __restrict__ y, int B,
                                                  real* __restrict__ out) {
  __shared__ real part[256];
  real s = RL(0.0);
  for (int i = threadIdx.x; i < B; i += 256) {
    const real d = V[i] - y[i];
    s += d * d;
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = part[0] / (real)B;
}

static void launch_adam_multi(const LearnAdamT<real>& A, hipStream_t s) {
  long total = 0;
  for (int i = 0; i < A.n; ++i) total += A.size[i];
  hipLaunchKernelGGL(k_adam_multi, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, A, total);
}

int launch_adam(const LearnAdamT<real>& A, void* stream) {
  launch_adam_multi(A, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_soft_update(const SoftUpdateT<real>& A, void* stream) {
  long total = 0;
  for (int i = 0; i < A.n; ++i) total += A.size[i];
  hipLaunchKernelGGL(k_soft_update, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, A, total);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_td_lambda(const real* r, const real* v, const uint8_t* done, int h, int N, real gamma, real lam,
                     real* out, void* stream) {
  hipLaunchKernelGGL(k_td_lambda, dim3((unsigned)((N + 63) / 64)), dim3(64), 0, (hipStream_t)stream, r, v, done, h,
                     N, gamma, lam, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_obs_stats(const real* x, long rows, int od, double count, real* mean, real* var, real* inv_std,
                     double eps, double* ws, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const dim3 cols((unsigned)((od + OS_COLS - 1) / OS_COLS));
  if (!ws) {
    hipLaunchKernelGGL(k_obs_stats, cols, dim3(OS_COLS * OS_GROUPS), 0, s, x, rows, od, count, mean, var, inv_std, eps);
  } else {
    const ObsStatsPlan P = obs_stats_plan(rows, od);
    hipLaunchKernelGGL(k_obs_stats_part, dim3((unsigned)P.chunks, (unsigned)((od + P.width - 1) / P.width)),
                       dim3(OSP_THREADS), 0, s, x, rows, od, P.width, P.groups, ws);
    hipLaunchKernelGGL(k_obs_stats_merge, dim3((unsigned)((od + OSM_COLS - 1) / OSM_COLS)), dim3(OSM_COLS * OSM_GROUPS), 0, s, ws, (int)P.chunks, P.chunk_rows, rows,
                       od, count, mean, var, inv_std, eps);
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_critic_values(const ThetaArgsT<real>& T, real* out, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (layered(T, ROWS_VALUES)) {
    theta_hidden(T, s);
    theta_output(T, out, s);
  } else {
    RowsArgs R = {};
    R.V = out;
    if (launch_rows<ROWS_VALUES>(R, T, nullptr, nullptr, s)) return -1;
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int RT, bool LN>
static int launch_fit_as(const FitArgs& g, int tiles, size_t lds, hipStream_t s) {
  if (allow_lds(&k_mlp_fit<RT, LN>, lds)) return -1;
  hipLaunchKernelGGL((k_mlp_fit<RT, LN>), dim3(tiles), dim3(FIT_WAVES * SIM_WAVE), lds, s, g);
  return 0;
}

// Whether a minibatch of M rows runs as k_mlp_fit with rt x 16 rows a block: the tile's layers
// within a CU's LDS, the tiles' gradients within the scratch, and at most FIT_PARAMS_PER_ROW
// gradient values written per row (beyond that the gradients are more traffic than the layer
// inputs and adjoints that k_mlp_rows and k_mlp_wgrad exchange).  32 rows a block once they give
// every CU a block, if two such blocks fit a CU; else 16 rows if three fit; else whatever fits:
// a block alone on its CU still beats the three launches and the layers (76-256-128-1, 8192 rows:
// 59 us fused with 32 rows in 63 KB, 105 and 168 us; FP64 280-64-64-1, 256 rows: 29 us with 16 rows in
// 57 KB, 43 us in three launches), but 12288 rows of a normalised 76-128-128-1 take 85 us as 32-row
// blocks of 86 KB and 68 us as 16-row blocks of 45 KB.
#define FIT_PARAMS_PER_ROW 2048
static bool fit_plan(const CriticFitT<real>& F, int M, FitArgs& g, int& rt, size_t& lds) {
  const ThetaArgsT<real>& T = F.G;
  const long np = mlp_params(T);
  auto ld = [&](int l) { return l < T.nl ? mlp_pad16(T.dims[l]) + 4 : 0; };
  g.ld0 = ld(0); g.ld1 = ld(1); g.ld2 = ld(2);
  const struct { int rt; size_t lds; } form[] = {{2, 80 << 10}, {1, 160 * 1024 / 3}, {2, 160 << 10}, {1, 160 << 10}};
  for (const auto& f : form) {
    rt = f.rt;
    if (rt == 2 && M < 32 * MR_CUS) continue;
    const int R = 16 * rt, copies = T.ln ? 2 : 1;
    g.p1 = R * g.ld0;
    g.e1 = g.p1 + R * g.ld1;
    g.p2 = g.p1 + copies * R * g.ld1;
    g.e2 = g.p2 + R * g.ld2;
    g.pd = g.p2 + copies * R * g.ld2;
    lds = (size_t)(g.pd + R * 20) * sizeof(real);
    // with the kernel's own arrays: statistics, row sums, the normalisation's column sums
    const size_t all = lds + ((MR_MAXHIDL * 2 + 3) * R + (T.ln ? 1024 : 1)) * sizeof(real);
    if (all <= f.lds && np <= (long)FIT_PARAMS_PER_ROW * R && (long)((M + R - 1) / R) * np <= F.scratch_cap) return true;
  }
  return false;
}

// One minibatch layer by layer: gather, forward, loss adjoint, layer gradients, Adam step.
static void fit_layers(const CriticFitT<real>& F, const ThetaArgsT<real>& G, const int* perm, const LearnAdamT<real>& A,
                       real* loss_out, hipStream_t s) {
  const int B = G.M;
  const long nx = (long)B * G.dims[0];
  hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)((nx + 255) / 256)), dim3(256), 0, s, F.obs, F.targets, perm, B,
                     G.dims[0], F.obs_mean, F.obs_inv_std, F.x, F.y);
  ThetaArgsT<real> T = G;
  T.x0 = F.x;
  T.x_shift = T.x_scale = nullptr;
  theta_hidden(T, s);
  theta_output(T, F.vbuf, s);
  if (loss_out) hipLaunchKernelGGL(k_mse_loss, dim3(1), dim3(256), 0, s, F.vbuf, F.y, B, loss_out);
  hipLaunchKernelGGL(k_mse_seed, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, F.vbuf, F.y, B, T.d0);
  theta_backward(T, s);
  launch_adam_multi(A, s);
}

// n_iter passes over the rows in the order of perm[it], n_mb minibatches each.  A minibatch is
// two launches where its tiles fit (fit_plan): the tiles' gradients, and their sum with the Adam
// step.  Others take three, the rows pass, every layer's weight gradient, and the sum with the
// Adam step, or go layer by layer (layered).
int launch_critic_fit(const CriticFitT<real>& F, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  ThetaArgsT<real> T = F.G;
  T.x0 = F.obs;
  T.x_shift = F.obs_mean;
  T.x_scale = F.obs_inv_std;
  ReduceArgs Q = {};
  Q.fit = 1;
  Q.loss_part = F.y;
  LearnAdamT<real> A = {};
  // the flat gradient holds W_0, b_0, W_1, ... in order; with layer normalisation a hidden
  // layer's gain and bias follow its W, b
  for (int l = 0; l < T.nl; ++l) {
    A.p[A.n] = F.W[l];
    A.size[A.n++] = (long)T.dims[l] * T.dims[l + 1];
    A.p[A.n] = F.bvec[l];
    A.size[A.n++] = T.dims[l + 1];
    if (T.ln && l + 1 < T.nl) {
      A.p[A.n] = F.lng[l];
      A.size[A.n++] = T.dims[l + 1];
      A.p[A.n] = F.lnb[l];
      A.size[A.n++] = T.dims[l + 1];
    }
  }
  A.g = T.out; A.m = F.m; A.v = F.v;
  A.lr = F.lr; A.b1 = F.b1; A.b2 = F.b2; A.eps = F.eps;
  int step = F.adam_step;
  for (int it = 0; it < F.n_iter; ++it) {
    for (int mb = 0; mb < F.n_mb; ++mb) {
      const int r0 = (int)((long)mb * F.rows / F.n_mb), r1 = (int)((long)(mb + 1) * F.rows / F.n_mb);
      if (r1 <= r0) continue;
      T.M = r1 - r0;
      const int* perm = F.perm + (long)it * F.rows + r0;
      real* loss_out = F.loss_out ? F.loss_out + it * F.n_mb + mb : nullptr;
      ++step;
      A.bc1 = RL(1.0) - (real)pow((double)F.b1, (double)step);
      A.bc2 = RL(1.0) - (real)pow((double)F.b2, (double)step);
      FitArgs g = {};
      int rt;
      size_t lds;
      if (fit_plan(F, T.M, g, rt, lds)) {
        g.N = mlp_net(T);
        g.perm = perm;
        g.tgt = F.targets;
        g.part = F.scratch;
        g.loss_part = F.y;
        g.np = (int)mlp_params(T);
        g.ow1 = (int)T.off_w[1]; g.ow2 = (int)T.off_w[2];
        g.ob0 = (int)T.off_b[0]; g.ob1 = (int)T.off_b[1]; g.ob2 = (int)T.off_b[2];
        g.og1 = (int)T.off_g[0]; g.og2 = (int)T.off_g[1];
        const int tiles = (T.M + 16 * rt - 1) / (16 * rt);
        const int bad = T.ln ? (rt == 2 ? launch_fit_as<2, true>(g, tiles, lds, s) : launch_fit_as<1, true>(g, tiles, lds, s))
                             : (rt == 2 ? launch_fit_as<2, false>(g, tiles, lds, s) : launch_fit_as<1, false>(g, tiles, lds, s));
        if (bad) return -1;
        reduce_args(Q, T, F.scratch, tiles, 0, false);
        Q.n_loss = tiles;
      } else if (layered(T, ROWS_FIT)) {
        fit_layers(F, T, perm, A, loss_out, s);
        continue;
      } else {
        RowsArgs R = {};
        R.perm = perm;
        R.tgt = F.targets;
        R.xs = F.x;
        R.V = F.vbuf;
        R.loss_part = F.y;
        int blocks = 0;
        if (launch_rows<ROWS_FIT>(R, T, &blocks, &Q.n_loss, s)) return -1;
        WgradArgs W = {};
        W.N = R.N;
        W.dv = F.vbuf;
        W.xs = F.x;
        launch_wgrad(W, T, s);
        reduce_args(Q, T, W.part, W.splits, blocks, true);
      }
      Q.rows = T.M;
      Q.loss_out = loss_out;
      Q.A = A;
      hipLaunchKernelGGL(k_mlp_reduce, dim3((unsigned)((Q.np + SIM_WAVE - 1) / SIM_WAVE) + 1), dim3(RD_WAVES * SIM_WAVE), 0, s, Q);
    }
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}
