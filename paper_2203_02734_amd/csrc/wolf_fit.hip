// Gradient kernels for fitting a source to an observed spectral density.
//
// Model (eq. W_def with a Gaussian degree of coherence): W_A[p1; p2] = a(p1) a(p2) mu_g(p1, p2),
// with a = sqrt(I) and mu_g = exp(-|xi1 - xi2|^2 / (2 sg^2)). The loss depends on S_B = Re diag(W_B)
// (Algorithm 4). With g = dL/dS_B, the gradient with respect to W_B is diag(g)
// (k_diag_embed). The adjoint propagation maps it to G_A (wolf_propagate_adjoint). For each real
// parameter theta, dL/dtheta = sum Re(conj(G_A) dW_A/dtheta):
//   dL/dI(p) = [R(p) + K(p)] / (2 a(p)),  R(p) = sum_q Re(conj(G_A[p; q])) a(q) mu_g(p, q)
//                                          K(p) = sum_q Re(conj(G_A[q; p])) a(q) mu_g(q, p)
//   dL/dsg   = sum_{p, q} Re(conj(G_A[p; q]) W_A[p; q]) |xi_p - xi_q|^2 / sg^3
// Workgroups own a group of slabs and a part of the N^2 columns (at most 4096 of them: one part below
// N = 128, four at N = 128). Each gives a partial row sum R per slab and part, a partial column sum K
// per column and group, and a partial of dL/dsg; the finishing kernel adds the parts in a fixed order.
#include "wolf_device.hpp"
#include "wolf_internal.hpp"

namespace wolf {

template <class T>
__global__ __launch_bounds__(256) void k_diag_embed(const typename real_of<T>::type* __restrict__ g, int n,
                                                    T* __restrict__ out) {
  using R = typename real_of<T>::type;
  const long long nn = (long long)n * n;
  const long long p1 = blockIdx.x;
  T* slab = out + p1 * nn;
  for (long long e = threadIdx.x; e < nn; e += blockDim.x) slab[e] = T{e == p1 ? g[p1] : (R)0, (R)0};
}

// Partials of one (group of slabs, part of the columns): rows[part][p] (a slab's row sum over the
// part's columns), colpart[group][q] (q in the part), sgpart[group][part]. A thread owns the columns
// q = part * COLS_PER_THREAD * 256 + k 256 + tid, k < COLS_PER_THREAD (at most 16, so that the column
// sums stay in registers), issues their loads before it uses any, and computes a(q) of its columns once.
// N divides 256 (both powers of two, N <= 128 here), so q has the fixed second index qj = tid mod N.
// The row sum of a slab is reduced by a butterfly within each wavefront and then over the four
// wavefronts in order.
template <class T, int COLS_PER_THREAD>
__global__ __launch_bounds__(256) void k_fit_partials(const T* __restrict__ ga, const float* __restrict__ imap, int n,
                                                      double inv2g2_px, int slabs_per_group, int parts,
                                                      typename real_of<T>::type* __restrict__ rows,
                                                      typename real_of<T>::type* __restrict__ colpart,
                                                      double* __restrict__ sgpart) {
  using R = typename real_of<T>::type;
  constexpr int CPT = COLS_PER_THREAD;
  __shared__ R red[2][4];  // wavefront sums of the row, double-buffered by slab parity
  __shared__ double redd[256];
  __shared__ R gx[256];  // exp(-d^2 pitch^2 / (2 sg^2)) for d = 0..N-1; mu_g = gx[|di|] gx[|dj|]
  const int nn = n * n;
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  for (int d = tid; d < n; d += 256) gx[d] = (R)exp(-(double)d * (double)d * inv2g2_px);
  const long long group = blockIdx.x / parts;
  const int part = (int)(blockIdx.x - group * parts);
  const int q0 = part * CPT * 256;
  const int qj = tid % n, qi0 = (q0 + tid) / n, qstep = 256 / n;
  R aqs[CPT];  // a(q) = sqrt(I(q)) of this thread's columns, the same for every slab
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int q = q0 + k * 256 + tid;
    aqs[k] = q < nn ? sqrt((R)imap[q]) : (R)0;
  }
  __syncthreads();
  R colacc[CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) colacc[k] = (R)0;
  double sgacc = 0.0;
  for (int s = 0; s < slabs_per_group; ++s) {
    const long long p = group * slabs_per_group + s;
    const int pi = (int)(p / n), pj = (int)(p % n);
    const R ap = sqrt((R)imap[p]);
    const T* row = ga + p * nn + q0;
    const int dj = pj - qj;
    const R muj = gx[dj < 0 ? -dj : dj];
    T gv[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) gv[k] = load_or_first(row, q0 + k * 256 + tid < nn, k * 256 + tid);
    R racc = (R)0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const bool ok = q0 + k * 256 + tid < nn;
      const int di = pi - (qi0 + k * qstep);
      const int ai = di < 0 ? -di : di;
      const double d2 = (double)(di * di + dj * dj);
      const R mu = gx[ok ? ai : 0] * muj;
      const R gre = ok ? gv[k].x : (R)0;
      const R w = gre * aqs[k] * mu;               // Re(conj(G) a(q) mu), a and mu real
      racc += w;
      colacc[k] += gre * ap * mu;                  // contribution to K(q)
      sgacc += (double)(w * ap) * d2;              // Re(conj(G) W_A) |d|^2 in pixel units
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) racc += __shfl_xor(racc, off);
    if (lane == 0) red[s & 1][wave] = racc;
    __syncthreads();
    if (tid == 0) rows[(long long)part * nn + p] = ((red[s & 1][0] + red[s & 1][1]) + red[s & 1][2]) + red[s & 1][3];
  }
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int q = q0 + k * 256 + tid;
    if (q < nn) colpart[group * nn + q] = colacc[k];
  }
  redd[tid] = sgacc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) redd[tid] += redd[tid + h];
    __syncthreads();
  }
  if (tid == 0) sgpart[blockIdx.x] = redd[0];
}

// dL/dI from the row sums (added over the column parts) and the column partials, and dL/dsg from the
// group partials. A workgroup
// owns 32 columns; its eight slices of 32 threads each add every eighth group in order, and the slices
// are combined in order. Workgroup 0 also adds the sg partials: 256 strided sums, then a fixed tree.
template <class T>
__global__ __launch_bounds__(256) void k_fit_finish(const float* __restrict__ imap, int n, int groups, int parts,
                                                    const typename real_of<T>::type* __restrict__ rows,
                                                    const typename real_of<T>::type* __restrict__ colpart,
                                                    const double* __restrict__ sgpart, double sg_scale,
                                                    float* __restrict__ d_imap, double* __restrict__ d_sigma) {
  using R = typename real_of<T>::type;
  __shared__ R part[8][32];
  __shared__ double sred[256];
  const long long nn = (long long)n * n;
  const int cx = threadIdx.x % 32, sl = threadIdx.x / 32;
  const long long q = (long long)blockIdx.x * 32 + cx;
  R k = (R)0;
  if (q < nn) {
#pragma unroll 8
    for (int g = sl; g < groups; g += 8) k += colpart[(long long)g * nn + q];  // loads in flight, sums in order
  }
  part[sl][cx] = k;
  if (blockIdx.x == 0) {
    double t = 0.0;
    for (int g = threadIdx.x; g < groups * parts; g += 256) t += sgpart[g];
    sred[threadIdx.x] = t;
  }
  __syncthreads();
  if (sl == 0 && q < nn) {
    R kk = part[0][cx];
#pragma unroll
    for (int j = 1; j < 8; ++j) kk += part[j][cx];
    R rsum = rows[q];
    for (int j = 1; j < parts; ++j) rsum += rows[(long long)j * nn + q];
    const R a = sqrt((R)imap[q]);
    d_imap[q] = (float)((rsum + kk) / ((R)2 * a));
  }
  if (blockIdx.x == 0) {
    for (int h = 128; h > 0; h >>= 1) {
      if ((int)threadIdx.x < h) sred[threadIdx.x] += sred[threadIdx.x + h];
      __syncthreads();
    }
    if (threadIdx.x == 0) *d_sigma = sred[0] * sg_scale;
  }
}

template <class T>
hipError_t launch_diag_embed(int n, const typename real_of<T>::type* g, T* out, hipStream_t st) {
  hipLaunchKernelGGL(k_diag_embed<T>, dim3((unsigned)(n * n)), dim3(256), 0, st, g, n, out);
  return hipGetLastError();
}

// Columns per part: 256 threads x at most 16 columns each.
static int fit_parts(int n) {
  const long long nn = (long long)n * n;
  return nn > 4096 ? (int)(nn / 4096) : 1;
}

template <class T>
hipError_t launch_fit_gradient(int n, const T* ga, const float* imap, double inv2g2_px, double sg_scale, void* work,
                               float* d_imap, double* d_sigma, hipStream_t st) {
  using R = typename real_of<T>::type;
  const long long nn = (long long)n * n;
  const int slabs_per_group = fit_slabs_per_group(n);
  const int groups = (int)(nn / slabs_per_group);
  const int parts = fit_parts(n);
  R* rows = reinterpret_cast<R*>(work);
  R* colpart = rows + parts * nn;
  double* sgpart = reinterpret_cast<double*>(colpart + (long long)groups * nn + 1);
  sgpart = reinterpret_cast<double*>((reinterpret_cast<uintptr_t>(sgpart) + 7) & ~(uintptr_t)7);
  const dim3 grid((unsigned)(groups * parts));
  switch (nn / parts > 256 ? (nn / parts + 255) / 256 : 1) {
    case 1: hipLaunchKernelGGL((k_fit_partials<T, 1>), grid, dim3(256), 0, st, ga, imap, n, inv2g2_px, slabs_per_group, parts, rows, colpart, sgpart); break;
    case 4: hipLaunchKernelGGL((k_fit_partials<T, 4>), grid, dim3(256), 0, st, ga, imap, n, inv2g2_px, slabs_per_group, parts, rows, colpart, sgpart); break;
    case 16: hipLaunchKernelGGL((k_fit_partials<T, 16>), grid, dim3(256), 0, st, ga, imap, n, inv2g2_px, slabs_per_group, parts, rows, colpart, sgpart); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fit_finish<T>, dim3((unsigned)((nn + 31) / 32)), dim3(256), 0, st, imap, n, groups, parts,
                     (const R*)rows, (const R*)colpart, (const double*)sgpart, sg_scale, d_imap, d_sigma);
  return hipGetLastError();
}

int fit_slabs_per_group(int n) {
  const long long nn = (long long)n * n;
  // About 512 groups of slabs: two workgroups per CU, and a partial buffer of 512 x N^2 reals.
  long long s = nn / 512;
  return (int)(s < 1 ? 1 : s);
}

size_t fit_work_bytes(int n, int real_bytes) {
  const long long nn = (long long)n * n;
  const long long groups = nn / fit_slabs_per_group(n);
  const long long parts = fit_parts(n);
  return (size_t)(parts * nn + groups * nn + 1) * real_bytes + 8 + (size_t)(groups * parts) * 8;
}

template hipError_t launch_diag_embed<float2>(int, const float*, float2*, hipStream_t);
template hipError_t launch_diag_embed<double2>(int, const double*, double2*, hipStream_t);
template hipError_t launch_fit_gradient<float2>(int, const float2*, const float*, double, double, void*, float*,
                                                double*, hipStream_t);
template hipError_t launch_fit_gradient<double2>(int, const double2*, const float*, double, double, void*, float*,
                                                 double*, hipStream_t);

// ---------------------------------------------------------------------------------------------
// The same model's S_B and its gradient without any N^4 array. With t = q(z, xi) (1 in the far field), b = a t and
// the difference delta = p - q in (-N, N)^2, both the forward and the adjoint operator act on functions of delta:
//   S_B[m] = s sum_d e^{2 pi i <m - c, d>/N} D[d],   D[d] = sum_{delta = d mod N} mu_g(delta) C[delta],
//            C[delta] = sum_p conj(b(p)) b(p - delta),
//   G_A[p; q] = s t(p) conj(t(q)) G[p - q mod N],   G[d] = sum_m g(m) e^{-2 pi i <m - c, d>/N},
//   dL/dI(p)  = s / a(p) Re( t(p) sum_q conj(b(q)) mu_g(p - q) G[p - q] )   (G_A is Hermitian: R = K above),
//   dL/dsg    = s pitch^2 / sg^3 sum_d Re( G[d] conj(D2[d]) ),  D2[d] = sum_{delta = d mod N} |delta|^2 mu_g(delta) C[delta].
// N^4 / 2 and N^4 complex multiply-adds on N^2 operands in FP64, where the propagated array took three passes over N^4
// elements each way. D and D2 obey X[-d] = conj(X[d]), so d_i runs over [0, N/2].
// Bound: launches and LDS reads. One optimisation step in complex128: N = 64 0.78 -> 0.23 ms (68 us of it in these
// kernels), N = 128 10.8 -> 0.36 ms (245 us; the sums 72 and 114 us).
// ---------------------------------------------------------------------------------------------
constexpr int kFitThreads = 128;
constexpr int kFitRows = 8;  // rows of one operand per workgroup

struct FitModel {
  const float* imap;
  int n;
  double alpha;      // source chirp rate pitch^2 / (lambda z), 0 in the far field
  double inv2g2_px;  // pitch^2 / (2 sg^2)
  double scale;      // s = C pitch^4
};

__host__ __device__ __forceinline__ int fit_rows(int n) { return n < kFitRows ? n : kFitRows; }
// Outputs per thread of the two sums: four neighbours share all but one of the operand reads of a step.
__host__ __device__ __forceinline__ int fit_outputs(int n) { return n >= 64 ? 4 : 1; }

// tx[i] = t along one axis, g[d] = exp(-d^2 pitch^2 / (2 sg^2)), d = 0 .. n.
__device__ __forceinline__ void fit_tables(const FitModel& f, double2* tx, double* g) {
  for (int i = threadIdx.x; i < f.n; i += blockDim.x) tx[i] = chirp_entry<double2>(Chirp{f.alpha, 1.0, +1, 0}, i, f.n);
  if (g != nullptr)
    for (int d = threadIdx.x; d <= f.n; d += blockDim.x) g[d] = exp(-(double)d * (double)d * f.inv2g2_px);
}

__device__ __forceinline__ double2 fit_b(const FitModel& f, const double2* tx, int i, int j) {
  return cscale(cmul(tx[i], tx[j]), sqrt((double)f.imap[i * f.n + j]));
}

// e^{2 pi i j / n}, j = 0 .. n - 1.
__device__ __forceinline__ void fit_roots(double2* w, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)i / (double)n, &s, &c);
    w[i] = double2{c, s};
  }
}

// The two transforms and the sums over parts carry their roundings (add_compensated): they are the last chains before the results,
// and plain ones left S_B 2.8e-16 to 4.4e-16 off in the 2-norm at N = 16 to 64, where the propagated array gave 1.1e-16 to 2.8e-16.
__device__ __forceinline__ void cmac(double2& a, const double2& x, const double2& y) {
  a.x += x.x * y.x - x.y * y.y;
  a.y += x.x * y.y + x.y * y.x;
}

// Parts of D and D2: part[0 / 1][chunk][d_i][d_j] over the kFitRows rows p_i of a chunk. A workgroup owns d_i and a chunk;
// thread (sub, tj) the outputs d_j = K tj .. K tj + K - 1 of the rows sub, sub + subs, ... As p_j rises, the operands
// b(p_i - d_i, p_j - d_j) of the K outputs slide by one. The sum up to p_j = d_j - 1 belongs to delta_j = d_j - N, the
// rest to d_j; likewise in p_i by whole rows.
template <int K>
__global__ __launch_bounds__(kFitThreads) void k_fit_corr(FitModel f, double2* __restrict__ part) {
  extern __shared__ double2 fit_lds[];
  const int n = f.n, rows = fit_rows(n), nm = n - 1;
  double2* u = fit_lds;            // conj(b) of the chunk's rows, then the sums of the row groups
  double2* v = u + rows * n;       // b of the rows p_i - d_i
  double2* tx = v + rows * n;
  double* g = reinterpret_cast<double*>(tx + n);
  const int di = blockIdx.x, i0 = blockIdx.y * rows;
  fit_tables(f, tx, g);
  __syncthreads();
  for (int e = threadIdx.x; e < rows * n; e += kFitThreads) {
    const int r = e / n, j = e % n;
    u[e] = cconj(fit_b(f, tx, i0 + r, j));
    v[e] = fit_b(f, tx, (i0 + r - di) & nm, j);
  }
  __syncthreads();
  const int tjs = n / K, subs = kFitThreads / tjs > 0 ? kFitThreads / tjs : 1;
  const int tj = threadIdx.x % tjs, sub = threadIdx.x / tjs, dj0 = K * tj;
  double2 d1[K], d2[K];
#pragma unroll
  for (int k = 0; k < K; ++k) d1[k] = d2[k] = double2{0.0, 0.0};
  for (int r = sub; r < rows; r += subs) {
    const double2* ur = u + r * n;
    const double2* vr = v + r * n;
    double2 run[K], low[K], w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      run[k] = low[k] = double2{0.0, 0.0};
    }
    // Step p_j: slot (p_j - k) mod K of w holds b(p_j - d_j0 - k); each step replaces the oldest.
#pragma unroll
    for (int k = 1; k < K; ++k) w[K - k] = vr[(-dj0 - k) & nm];
    for (int p0 = 0; p0 < n; p0 += K) {
      const bool here = p0 == dj0;  // the block that holds the switch of every output of this thread
#pragma unroll
      for (int i = 0; i < K; ++i) {
        w[i] = vr[(p0 + i - dj0) & nm];
        const double2 a = ur[p0 + i];
        if (here) {  // p_j = d_j of output k = i
          low[i] = run[i];
          run[i] = double2{0.0, 0.0};
        }
#pragma unroll
        for (int k = 0; k < K; ++k) cmac(run[k], a, w[(i - k + K) % K]);
      }
    }
    const int pi = i0 + r, ai = pi >= di ? di : n - di;  // |delta_i|
    const double gi = g[ai];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int dj = dj0 + k;
      const double wu = gi * g[dj], wl = gi * g[n - dj];
      const double qu = wu * (double)(ai * ai + dj * dj), ql = wl * (double)(ai * ai + (n - dj) * (n - dj));
      d1[k].x += wu * run[k].x + wl * low[k].x;
      d1[k].y += wu * run[k].y + wl * low[k].y;
      d2[k].x += qu * run[k].x + ql * low[k].x;
      d2[k].y += qu * run[k].y + ql * low[k].y;
    }
  }
  // The row groups' sums, added in order.
  const long long plane = (long long)(n / 2 + 1) * n;
  const int active = subs < rows ? subs : rows;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
    if (sub < active)
#pragma unroll
      for (int k = 0; k < K; ++k) u[sub * n + dj0 + k] = which ? d2[k] : d1[k];
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += kFitThreads) {
      double2 a = u[j], lost{0.0, 0.0};
      for (int q = 1; q < active; ++q) add_compensated(a, lost, u[q * n + j]);
      part[((long long)which * gridDim.y + blockIdx.y) * plane + (long long)di * n + j] = a;
    }
  }
}

// E[d_i][m_j] = sum_{d_j} e^{2 pi i (m_j - c) d_j / N} D[d_i][d_j], D the sum of its parts over the chunks, in order; D2's
// sum goes to `corr` for the backward pass. One workgroup per d_i.
__global__ __launch_bounds__(kFitThreads) void k_fit_dft_rows(const double2* __restrict__ part, int n, int chunks,
                                                              double2* __restrict__ e, double2* __restrict__ corr) {
  extern __shared__ double2 fit_lds[];
  double2* row = fit_lds;
  double2* w = row + n;
  const long long plane = (long long)(n / 2 + 1) * n, at = (long long)blockIdx.x * n;
  fit_roots(w, n);
  for (int j = threadIdx.x; j < 2 * n; j += kFitThreads) {
    const int which = j / n, jj = j % n;
    double2 a{0.0, 0.0}, lost{0.0, 0.0};
#pragma unroll 8
    for (int q = 0; q < chunks; ++q) add_compensated(a, lost, part[((long long)which * chunks + q) * plane + at + jj]);
    if (which)
      corr[at + jj] = a;
    else
      row[jj] = a;
  }
  __syncthreads();
  for (int m = threadIdx.x; m < n; m += kFitThreads) {
    double2 a{0.0, 0.0}, lost{0.0, 0.0};
#pragma unroll 4
    for (int d = 0; d < n; ++d) add_compensated(a, lost, cmul(w[((m - n / 2) * d) & (n - 1)], row[d]));
    e[at + m] = a;
  }
}

// S[m] = s Re sum_{d_i = 0}^{N/2} weight e^{2 pi i (m_i - c) d_i / N} E[d_i][m_j]; the rows 0 < d_i < N/2 count for -d_i too.
__global__ __launch_bounds__(256) void k_fit_dft_s(const double2* __restrict__ e, int n, double scale,
                                                   double* __restrict__ s) {
  extern __shared__ double2 fit_lds[];
  fit_roots(fit_lds, n);
  __syncthreads();
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m >= n * n) return;
  const int mi = m / n, mj = m % n;
  double a = 0.0, lost = 0.0;
#pragma unroll 8
  for (int d = 0; d <= n / 2; ++d) {
    const double2 x = fit_lds[((mi - n / 2) * d) & (n - 1)], y = e[(long long)d * n + mj];
    add_compensated(a, lost, (d == 0 || d == n / 2 ? 1.0 : 2.0) * (x.x * y.x - x.y * y.y));
  }
  s[m] = scale * a;
}

// A[m_i][d_j] = sum_{m_j} g(m) e^{-2 pi i (m_j - c) d_j / N}: one workgroup per m_i.
__global__ __launch_bounds__(kFitThreads) void k_fit_g_rows(const double* __restrict__ g, int n,
                                                            double2* __restrict__ a) {
  extern __shared__ double2 fit_lds[];
  double2* w = fit_lds;
  double* row = reinterpret_cast<double*>(w + n);
  fit_roots(w, n);
  for (int j = threadIdx.x; j < n; j += kFitThreads) row[j] = g[(long long)blockIdx.x * n + j];
  __syncthreads();
  for (int d = threadIdx.x; d < n; d += kFitThreads) {
    double2 t{0.0, 0.0}, lost{0.0, 0.0};
#pragma unroll 4
    for (int m = 0; m < n; ++m) add_compensated(t, lost, cscale(w[(-(m - n / 2) * d) & (n - 1)], row[m]));
    a[(long long)blockIdx.x * n + d] = t;
  }
}

// G[d_i][d_j] = sum_{m_i} e^{-2 pi i (m_i - c) d_i / N} A[m_i][d_j].
__global__ __launch_bounds__(kFitThreads) void k_fit_g_cols(const double2* __restrict__ a, int n, double2* __restrict__ gd) {
  extern __shared__ double2 fit_lds[];
  fit_roots(fit_lds, n);
  __syncthreads();
  const int e = blockIdx.x * kFitThreads + threadIdx.x;
  if (e >= n * n) return;
  const int di = e / n, dj = e % n;
  double2 t{0.0, 0.0}, lost{0.0, 0.0};
#pragma unroll 8
  for (int m = 0; m < n; ++m)
    add_compensated(t, lost, cmul(fit_lds[(-(m - n / 2) * di) & (n - 1)], a[(long long)m * n + dj]));
  gd[e] = t;
}

// part[chunk][p] = Re( t(p) sum_{q_i in chunk} sum_{q_j} conj(b(q)) mu_g(p - q) G[p - q] ). A workgroup owns p_i and kFitRows
// rows q_i; thread (sub, tj) the outputs p_j = K tj .. K tj + K - 1, whose operands mu_g G at p_j - q_j slide by one as q_j
// rises.
template <int K>
__global__ __launch_bounds__(kFitThreads) void k_fit_conv(FitModel f, const double2* __restrict__ gd,
                                                          double* __restrict__ part) {
  extern __shared__ double2 fit_lds[];
  const int n = f.n, rows = fit_rows(n), nm = n - 1;
  double2* br = fit_lds;             // conj(b) of the chunk's rows, then the sums of the row groups
  double2* mr = br + rows * n;       // mu_g(delta_j) G[p_i - q_i][delta_j] at delta_j + N, delta_j in (-N, N)
  double2* tx = mr + rows * 2 * n;
  double* g = reinterpret_cast<double*>(tx + n);
  const int pi = blockIdx.x, i0 = blockIdx.y * rows;
  fit_tables(f, tx, g);
  __syncthreads();
  for (int e = threadIdx.x; e < rows * n; e += kFitThreads) {
    const int r = e / n, j = e % n, di = pi - (i0 + r), ai = di < 0 ? -di : di;
    br[e] = cscale(cconj(fit_b(f, tx, i0 + r, j)), g[ai]);
    const double2 x = gd[(long long)(di & nm) * n + j];
    mr[r * 2 * n + n + j] = cscale(x, g[j]);  // delta_j = j
    mr[r * 2 * n + j] = cscale(x, g[n - j]);  // delta_j = j - N (its entry 0 is not used)
  }
  __syncthreads();
  const int tjs = n / K, subs = kFitThreads / tjs > 0 ? kFitThreads / tjs : 1;
  const int tj = threadIdx.x % tjs, sub = threadIdx.x / tjs, pj0 = K * tj;
  double2 acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = double2{0.0, 0.0};
  for (int r = sub; r < rows; r += subs) {
    const double2* b = br + r * n;
    const double2* m = mr + r * 2 * n + n + pj0;  // delta_j = p_j0 + k - q_j
    double2 w[K];  // step q_j: slot (k - q_j) mod K holds the operand of output k
#pragma unroll
    for (int k = 1; k < K; ++k) w[k] = m[k];
    for (int q0 = 0; q0 < n; q0 += K) {
#pragma unroll
      for (int i = 0; i < K; ++i) {
        w[(K - i) % K] = m[-(q0 + i)];
        const double2 x = b[q0 + i];
#pragma unroll
        for (int k = 0; k < K; ++k) cmac(acc[k], x, w[(k - i + K) % K]);
      }
    }
  }
  __syncthreads();
  const int active = subs < rows ? subs : rows;
  if (sub < active)
#pragma unroll
    for (int k = 0; k < K; ++k) br[sub * n + pj0 + k] = acc[k];
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += kFitThreads) {
    double2 a = br[j];
    for (int q = 1; q < active; ++q) a = cadd(a, br[q * n + j]);
    const double2 t = cmul(tx[pi], tx[j]);
    part[((long long)blockIdx.y * n + pi) * n + j] = t.x * a.x - t.y * a.y;
  }
}

// dL/dI from the parts, added in order; the workgroup past the last point adds dL/dsg: 256 strided sums, then a fixed tree.
__global__ __launch_bounds__(256) void k_fit_grad(FitModel f, const double* __restrict__ part, int chunks,
                                                  const double2* __restrict__ gd, const double2* __restrict__ corr,
                                                  double sg_scale, float* __restrict__ d_imap,
                                                  double* __restrict__ d_sigma) {
  __shared__ double red[256];
  const int n = f.n, nn = n * n;
  if (blockIdx.x + 1 == gridDim.x) {
    double a = 0.0, lost = 0.0;
    for (int e = threadIdx.x; e < (n / 2 + 1) * n; e += 256) {
      const int di = e / n;
      const double2 x = gd[e], y = corr[e];
      add_compensated(a, lost, (di == 0 || di == n / 2 ? 1.0 : 2.0) * (x.x * y.x + x.y * y.y));
    }
    red[threadIdx.x] = a;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
      __syncthreads();
    }
    if (threadIdx.x == 0) *d_sigma = f.scale * sg_scale * red[0];
    return;
  }
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= nn) return;
  double a = 0.0;
#pragma unroll 8
  for (int q = 0; q < chunks; ++q) a += part[(long long)q * nn + p];
  d_imap[p] = (float)(f.scale * a / sqrt((double)f.imap[p]));
}

static FitModel fit_model(int n, const float* imap, double alpha, double inv2g2_px, double scale) {
  return FitModel{imap, n, alpha, inv2g2_px, scale};
}

// Forward: the parts [2][chunks][N/2 + 1][N] and E. Backward: A, G and the parts [chunks][N^2].
size_t fit_sums_work_bytes(int n) {
  const size_t nn = (size_t)n * n, plane = (size_t)(n / 2 + 1) * n, chunks = (size_t)(n / fit_rows(n));
  const size_t forward = (2 * chunks + 1) * plane * sizeof(double2);
  const size_t backward = 2 * nn * sizeof(double2) + chunks * nn * sizeof(double);
  return forward > backward ? forward : backward;
}

hipError_t launch_fit_forward(int n, const float* imap, double alpha, double inv2g2_px, double scale, void* work,
                              double2* corr, double* s, hipStream_t st) {
  const FitModel f = fit_model(n, imap, alpha, inv2g2_px, scale);
  const int rows = fit_rows(n), chunks = n / rows, half = n / 2 + 1;
  double2* part = reinterpret_cast<double2*>(work);
  double2* e = part + 2ll * chunks * half * n;
  const size_t lds = (size_t)(2 * rows * n + n) * sizeof(double2) + (size_t)(n + 1) * sizeof(double);
  const dim3 grid((unsigned)half, (unsigned)chunks);
  if (fit_outputs(n) == 4)
    hipLaunchKernelGGL(k_fit_corr<4>, grid, dim3(kFitThreads), lds, st, f, part);
  else
    hipLaunchKernelGGL(k_fit_corr<1>, grid, dim3(kFitThreads), lds, st, f, part);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_fit_dft_rows, dim3((unsigned)half), dim3(kFitThreads), 2 * n * sizeof(double2), st, part, n,
                     chunks, e, corr);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  hipLaunchKernelGGL(k_fit_dft_s, dim3((unsigned)((n * n + 255) / 256)), dim3(256), n * sizeof(double2), st, e, n,
                     scale, s);
  return hipGetLastError();
}

hipError_t launch_fit_backward(int n, const double* g_s, const float* imap, double alpha, double inv2g2_px,
                               double scale, double sg_scale, const double2* corr, void* work, float* d_imap,
                               double* d_sigma, hipStream_t st) {
  const FitModel f = fit_model(n, imap, alpha, inv2g2_px, scale);
  const int rows = fit_rows(n), chunks = n / rows;
  const long long nn = (long long)n * n;
  double2* a = reinterpret_cast<double2*>(work);
  double2* gd = a + nn;
  double* part = reinterpret_cast<double*>(gd + nn);
  hipLaunchKernelGGL(k_fit_g_rows, dim3((unsigned)n), dim3(kFitThreads), n * (sizeof(double2) + sizeof(double)), st,
                     g_s, n, a);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_fit_g_cols, dim3((unsigned)((nn + kFitThreads - 1) / kFitThreads)), dim3(kFitThreads),
                     n * sizeof(double2), st, a, n, gd);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  const size_t lds = (size_t)(3 * rows * n + n) * sizeof(double2) + (size_t)(n + 1) * sizeof(double);
  const dim3 grid((unsigned)n, (unsigned)chunks);
  if (fit_outputs(n) == 4)
    hipLaunchKernelGGL(k_fit_conv<4>, grid, dim3(kFitThreads), lds, st, f, gd, part);
  else
    hipLaunchKernelGGL(k_fit_conv<1>, grid, dim3(kFitThreads), lds, st, f, gd, part);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  hipLaunchKernelGGL(k_fit_grad, dim3((unsigned)((nn + 255) / 256 + 1)), dim3(256), 0, st, f, part, chunks, gd, corr,
                     sg_scale, d_imap, d_sigma);
  return hipGetLastError();
}

}  // namespace wolf
