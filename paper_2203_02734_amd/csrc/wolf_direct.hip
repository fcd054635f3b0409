// Propagation with the exact free-space kernel (eq. h_free), summed directly: the check of the
// approximation Lambda/r ~ Lambda/R (eq. approx_L) and of the Fresnel expansion (eq. W_fresnel).
//
// h(x, xi) = Lambda(r) exp(i k r) / r with r = sqrt(z^2 + |x - xi|^2). A secondary source at normal
// incidence has Lambda = (k / (4 pi i)) (1 + z / r); a primary one Lambda = 1 / (4 pi). The factor 1/i
// and the common phase exp(i k z) cancel between h* and h and are left out, so
//   H[m][p] = |Lambda(r)| exp(2 pi i (r - z) / lambda) / r,   r - z = rho^2 / (r + z)  (no cancellation),
// on the output grid of the Fresnel operator (pitch lambda z / (N pitch)) and the source grid.
// The kernel does not factorise over x and y, so the sum is a dense contraction over N^2 source
// points for each point: W_B = pitch^4 conj(H) W_A H^T.
//
// Mirrored form (N >= 16). H depends on |x_k - xi_m| per axis only through its square, and both grids are symmetric
// about their middle c = N/2, except that they end at c - 1: h(-k, -m) = h(k, m). Per axis, with z[c] = 0,
//   e[m] = z[m] + z[-m] (m = 0: z[0]; m = c: z[-c]),  o[m] = z[m] - z[-m],
//   E[k] = sum_{m=0}^{c} (h(k, m) + h(k, -m)) / 2 e[m],   O[k] = sum_{m=1}^{c} (h(k, m) - h(k, -m)) / 2 o[m],
//   out[k] = E[k] + O[k],   out[-k] = E[k] - O[k],
// so each point's product splits into four (even or odd per axis) of about N^2 / 4 rows and columns: 3.7 times
// fewer operations at N = 64, and shorter sums. Slots: e[m] and E[k] at c - m, o[m] and O[k] at c + m, the positions of the
// points they mix, so folding W and unfolding the result work in place. O[c] needs one slot more than the
// grid (N), and o[c] = -e[c] is read from slot 0, with the sign in the matrix.
#include "wolf_device.hpp"
#include "wolf_internal.hpp"
#include "wolf_mfma.hpp"

namespace wolf {

// The kernel between grid points at (k, l) and (m, n) pixels from the middles, in FP64.
__device__ __forceinline__ double2 rs_entry(int k, int l, int m, int n, double pitch, double dx, double z, double lam,
                                            int primary) {
  const double ddx = dx * k - pitch * m, ddy = dx * l - pitch * n;
  const double rho2 = ddx * ddx + ddy * ddy;
  const double r = sqrt(z * z + rho2);
  const double cyc = rho2 / ((r + z) * lam);  // (r - z) / lambda
  const double red = cyc - rint(cyc);          // cycles mod 1, exact
  double s, c;
  sincospi(2.0 * red, &s, &c);
  const double amp = (primary ? 1.0 / (4.0 * M_PI) : (1.0 + z / r) / (2.0 * lam)) / r;
  return double2{amp * c, amp * s};
}

// The products of one operand split: per class an index set of `len` slots from `start` on each axis, for rows and
// contraction alike, and its matrix [la lb][la lb] at `h`. One class (0, N) is the plain product.
struct RsClass {
  int sa, la, sb, lb;
  long long h;
  int tile;  // first 64-row tile
};
struct RsClasses {
  RsClass c[4];
  int count, tiles;
  int n, slots;  // slots per axis of the products: N, or N + 1 when mirrored
};

static RsClasses rs_classes(int n, bool mirrored) {
  RsClasses s{};
  s.n = n;
  s.slots = mirrored ? n + 1 : n;
  const int c = n / 2;
  const int start[2] = {0, c + 1}, len[2] = {c + 1, c};
  long long h = 0;
  for (int a = 0; a < (mirrored ? 2 : 1); ++a)
    for (int b = 0; b < (mirrored ? 2 : 1); ++b) {
      RsClass& k = s.c[s.count++];
      k = mirrored ? RsClass{start[a], len[a], start[b], len[b], h, s.tiles} : RsClass{0, n, 0, n, h, s.tiles};
      const long long m = (long long)k.la * k.lb;
      h += m * m;
      s.tiles += (int)((m + 63) / 64);
    }
  return s;
}

// The plain matrix H[m][p].
template <class T>
__global__ __launch_bounds__(256) void k_rs_kernel(T* __restrict__ h, int n, double pitch, double dx, double z,
                                                   double lam, int primary) {
  using R = typename real_of<T>::type;
  const long long nn = (long long)n * n, total = nn * nn;
  const int c = n / 2;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int m = (int)(e / nn), p = (int)(e - m * nn);
    // x = d (i - N/2), y = d (N/2 - j) on both grids; the y flip enters both coordinates alike.
    const double2 v = rs_entry(m / n - c, m % n - c, p / n - c, p % n - c, pitch, dx, z, lam, primary);
    h[e] = T{(R)v.x, (R)v.y};
  }
}

// The four matrices of the mirrored form: a thread evaluates the kernel at (k, l) against (+-m, +-n) and writes its
// entry of every class that has one. blockIdx.y is the output (k, l), threads run along (m, n).
template <class T>
__global__ __launch_bounds__(256) void k_rs_mirror(T* __restrict__ h, RsClasses cs, double pitch, double dx, double z,
                                                   double lam, int primary) {
  using R = typename real_of<T>::type;
  const int c = cs.n / 2, w = c + 1;
  const int k = (int)blockIdx.y / w, l = (int)blockIdx.y % w;
  const int e = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (e >= w * w) return;
  const int m = c - e / w, n = c - e % w;  // slots of the even class ascend with e
  const double2 f00 = rs_entry(k, l, m, n, pitch, dx, z, lam, primary);
  const double2 f01 = rs_entry(k, l, m, -n, pitch, dx, z, lam, primary);
  const double2 f10 = rs_entry(k, l, -m, n, pitch, dx, z, lam, primary);
  const double2 f11 = rs_entry(k, l, -m, -n, pitch, dx, z, lam, primary);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool oi = q / 2, oj = q % 2;
    if ((oi && (k == 0 || m == 0)) || (oj && (l == 0 || n == 0))) continue;
    const RsClass& cl = cs.c[q];
    // Slots c - k (even) or c + k (odd); an odd m = c is stored as -e[c].
    const int row = ((oi ? c + k : c - k) - cl.sa) * cl.lb + (oj ? c + l : c - l) - cl.sb;
    const int col = ((oi ? c + m : c - m) - cl.sa) * cl.lb + (oj ? c + n : c - n) - cl.sb;
    const double si = oi ? -1.0 : 1.0, sj = oj ? -1.0 : 1.0;
    const double f = 0.25 * ((oi && m == c) ? -1.0 : 1.0) * ((oj && n == c) ? -1.0 : 1.0);
    const double re = f * ((f00.x + sj * f01.x) + si * (f10.x + sj * f11.x));
    const double im = f * ((f00.y + sj * f01.y) + si * (f10.y + sj * f11.y));
    h[cl.h + (long long)row * cl.la * cl.lb + col] = T{(R)re, (R)im};
  }
}

// Entry (U, V) of the mirrored result, U and V pairs of slots in [0, N]: the grid's own positions in `out`, the
// others (a slot N among them) in `extra`: first the rows with such a U, then the columns of the other rows.
__host__ __device__ __forceinline__ long long rs_extra_col(int n, int vi, int vj) { return vi == n ? vj : n + 1 + vi; }
template <class T>
__device__ __forceinline__ T* rs_result(T* out, T* extra, int n, int ui, int uj, int vi, int vj) {
  const long long n1 = n + 1, x = 2 * n + 1;
  if (ui == n || uj == n) return extra + rs_extra_col(n, ui, uj) * n1 * n1 + vi * n1 + vj;
  const long long u = (long long)ui * n + uj;
  if (vi == n || vj == n) return extra + x * n1 * n1 + u * x + rs_extra_col(n, vi, vj);
  return out + (u * n + vi) * n + vj;
}
static long long rs_extra_elems(long long n) { return (2 * n + 1) * ((n + 1) * (n + 1) + n * n); }

// Sums and differences of mirrored points, both points at once (in == out allowed): a thread owns the 16 entries that
// mirrors of its (a, b, m, n), each in [0, c], map to each other.
template <class T, bool UNFOLD>
__global__ __launch_bounds__(256) void k_rs_fold(const T* in, T* out, T* extra, int n) {
  const int c = n / 2, w = c + 1;
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)w * w * w * w) return;
  int q[4];
  {
    long long r = e;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
      q[i] = (int)(r % w);
      r /= w;
    }
  }
  // Bit i of s: slot (position) c + q[i] instead of c - q[i]. The upper one is missing at q = 0, and at q = c it is
  // outside the grid (a zero going in, the extra slot coming out).
  T v[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    int p[4];
    bool has = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool up = (s >> i) & 1;
      p[i] = up ? c + q[i] : c - q[i];
      has = has && !(up && (q[i] == 0 || (!UNFOLD && q[i] == c)));
    }
    using R = typename real_of<T>::type;
    v[s] = T{(R)0, (R)0};
    if (has) v[s] = UNFOLD ? *rs_result(out, extra, n, p[0], p[1], p[2], p[3]) : in[((p[0] * n + p[1]) * (long long)n + p[2]) * n + p[3]];
  }
  // Along each axis (lower, upper) -> (upper + lower, upper - lower) going in, (E, O) -> (E - O, E + O) coming out. A
  // middle row (q = 0) has no upper entry and stays.
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      if ((s >> i) & 1) continue;
      const T lo = v[s], hi = v[s | (1 << i)];
      v[s] = UNFOLD ? csub(lo, hi) : cadd(hi, lo);
      v[s | (1 << i)] = UNFOLD ? cadd(lo, hi) : csub(hi, lo);
    }
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    int p[4];
    bool has = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool up = (s >> i) & 1;
      p[i] = up ? c + q[i] : c - q[i];
      has = has && !(up && (q[i] == 0 || q[i] == c));
    }
    if (has) out[((p[0] * n + p[1]) * (long long)n + p[2]) * n + p[3]] = v[s];
  }
}

// The two products. FIRST: T1[p][V] = sum_kk F[p][slot(kk)] H[V][kk] over the second point's slots, rows p the N^2 slots of
// the first point. Otherwise R[U][V] = alpha sum_kk conj(H[U][kk]) T1[slot(kk)][V] over the first point's slots, stored by
// rs_result. Per class of outputs (U or V); slot N of the contraction reads slot 0.
// On the matrix cores (FP32 for complex64, FP64 for complex128) in the 3M form: 64 x 64 outputs per
// workgroup of four wavefronts (32 x 32 blocks), kk staged through double-buffered LDS 16 at a time, the
// loads of step s + 1 issued before the products of step s. Out-of-range elements load as zero and are not stored.
// Workgroups: the pairs of a 64-wide panel of F (or T1) and a matrix tile are listed by groups of an eighth of the panels,
// each group tile by tile, and each XCD takes an equal contiguous share of the list: it streams the matrices through its
// L2 about once, and its consecutive workgroups share a matrix tile.
// Bound: the matrix cores. N = 64: 1.07 and 1.16 ms in complex64 (103 and 98 TFLOP/s executed of 154), 2.04 and 2.28 ms in
// complex128 (54 and 50 of 72); the plain products took 4.2 and 10.7 ms each. Stores of the operands that run along kk
// are swizzled over the LDS banks (before: 3.45 and 3.18 ms in complex128).
// !MIRRORED (N < 16): one class whose slots are its indices; a launch is one tile and a chain of at most four steps, which the
// walk of the slots would lengthen (a call at N = 8: 23.8 us with it, 18.8 without in complex64, 30.3 and 24.4 in complex128).
template <class T, bool FIRST, bool MIRRORED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 2))) void k_rs_gemm(
    const T* __restrict__ x, const T* __restrict__ h, T* __restrict__ y, T* __restrict__ extra, RsClasses cs,
    int panels, int per_xcd, double alpha) {
  using R = typename real_of<T>::type;
  using G = MTile<64>;
  constexpr int TK = 16;
  __shared__ R ar[2][TK][G::LDA], ai[2][TK][G::LDA], br[2][TK][G::LDB], bi[2][TK][G::LDB];
  const int tid = threadIdx.x, lane = tid % 64;
  const int wv = __builtin_amdgcn_readfirstlane(tid / 64);  // wavefront-uniform
  const int row0 = (wv / G::WC) * 32, col0 = (wv % G::WC) * 32;
  const int xcd = (int)blockIdx.x % 8, total = panels * cs.tiles;
  const int unit = (int)((long long)total * xcd / 8) + (int)blockIdx.x / 8;
  if (unit >= (int)((long long)total * (xcd + 1) / 8)) return;
  const int group = unit / (per_xcd * cs.tiles), first = group * per_xcd, in_group = unit - first * cs.tiles;
  const int width = panels - first < per_xcd ? panels - first : per_xcd;
  const int panel = first + in_group % width, tile = in_group / width;
  RsClass cl = cs.c[0];
  if constexpr (MIRRORED) {
#pragma unroll
    for (int q = 1; q < 4; ++q)
      if (tile >= cs.c[q].tile) cl = cs.c[q];
  }
  const int n = cs.n, nn = n * n, kk_n = cl.la * cl.lb, vs = cs.slots, vv = vs * vs;
  const int o0 = (tile - cl.tile) * 64, p0 = panel * 64;  // first output of the class, first line of the panel
  const int p_n = FIRST ? nn : vv;
  const T* const hm = h + cl.h;
  auto slot = [&](int mi, int mj) {  // of the contraction index (mi, mj) within the class
    const int si = cl.sa + mi, sj = cl.sb + mj;
    return (si == n ? 0 : si) * n + (sj == n ? 0 : sj);
  };
  // Element q of thread tid in a step. The matrix, and F: (row e / 16, kk e % 16), 16 consecutive kk of one row; T1:
  // (kk e / 64, column e % 64), 64 consecutive columns. (mi, mj) of this thread's kk advance with the steps.
  constexpr int NI = FIRST ? 1 : 4;
  int mi[NI], mj[NI];
  if constexpr (MIRRORED) {
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const int kk = FIRST ? tid % TK : wv + 4 * q;
      mi[q] = kk / cl.lb;
      mj[q] = kk - mi[q] * cl.lb;
    }
  }
  T rh[4], rx[4];
  auto fetch = [&](int k0) {  // called for k0 = 0, 16, 32, ... in turn
    const int kh = k0 + tid % TK;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int o = o0 + tid / TK + 16 * q;
      rh[q] = load_or_first(hm, o < kk_n && kh < kk_n, (long long)o * kk_n + kh);
    }
    if constexpr (FIRST) {
      const int s = kh >= kk_n ? 0 : MIRRORED ? slot(mi[0], mj[0]) : kh;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p = p0 + tid / TK + 16 * q;
        rx[q] = load_or_first(x, p < p_n, (long long)p * nn + s);
      }
    } else {
      const int v = p0 + lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int kx = k0 + wv + 4 * q, s = kx >= kk_n ? 0 : MIRRORED ? slot(mi[q], mj[q]) : kx;
        rx[q] = load_or_first(x, v < p_n, (long long)s * vv + v);
      }
    }
    if constexpr (MIRRORED) {
#pragma unroll
      for (int q = 0; q < NI; ++q) {
        mj[q] += TK;
        while (mj[q] >= cl.lb) {
          mj[q] -= cl.lb;
          ++mi[q];
        }
      }
    }
  };
  auto stage = [&](int buf, int k0) {
    const int kk = tid % TK;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int ii = tid / TK + 16 * q, at = swizzled(kk, ii);
      const T v = keep_or_zero(o0 + ii < kk_n && k0 + kk < kk_n, rh[q]);
      if constexpr (FIRST) {
        const T u = keep_or_zero(p0 + ii < p_n && k0 + kk < kk_n, rx[q]);
        ar[buf][kk][at] = u.x;
        ai[buf][kk][at] = u.y;
        br[buf][kk][at] = v.x;
        bi[buf][kk][at] = v.y;
      } else {
        const int kx = wv + 4 * q;
        const T u = keep_or_zero(p0 + lane < p_n && k0 + kx < kk_n, rx[q]);
        ar[buf][kk][at] = v.x;
        ai[buf][kk][at] = -v.y;
        br[buf][kx][lane] = u.x;
        bi[buf][kx][lane] = u.y;
      }
    }
  };
  CTile<T> acc;
  ctile_zero(acc);
  fetch(0);
  stage(0, 0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < kk_n; k0 += TK) {
    const bool more = k0 + TK < kk_n;
    if (more) fetch(k0 + TK);
    ctile_mfma16<T, G::LDA, G::LDB, true, FIRST>(acc, ar[buf], ai[buf], br[buf], bi[buf], row0, col0, lane);
    if (more) stage(buf ^ 1, k0 + TK);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int gi = row0 + 16 * r + Mfma<T>::row(lane, i), gj = col0 + 16 * q + lane % 16;
        const T v{(R)(alpha * acc.re(r, q, i)), (R)(alpha * acc.im(r, q, i))};
        const int o = o0 + (FIRST ? gj : gi), p = p0 + (FIRST ? gi : gj);
        if (o < kk_n && p < p_n) {
          if constexpr (!MIRRORED) {
            y[FIRST ? (long long)p * nn + o : (long long)o * nn + p] = v;
            continue;
          }
          const int oi = o / cl.lb, oj = o - oi * cl.lb;
          if constexpr (FIRST) {
            y[(long long)p * vv + (cl.sa + oi) * vs + cl.sb + oj] = v;
          } else {
            const int pi = p / vs;
            *rs_result(y, extra, n, cl.sa + oi, cl.sb + oj, pi, p - pi * vs) = v;
          }
        }
      }
}

template <class T, bool FIRST, bool MIRRORED>
static hipError_t launch_rs_gemm(const T* x, const T* h, T* y, T* extra, const RsClasses& cs, double alpha,
                                 hipStream_t st) {
  const int lines = FIRST ? cs.n * cs.n : cs.slots * cs.slots;
  const int panels = (lines + 63) / 64, per_xcd = (panels + 7) / 8;
  hipLaunchKernelGGL((k_rs_gemm<T, FIRST, MIRRORED>), dim3((unsigned)(8 * ((panels * cs.tiles + 7) / 8))), dim3(256), 0, st, x, h, y, extra,
                     cs, panels, per_xcd, alpha);
  return hipGetLastError();
}

// Elements of `work` that the mirrored form takes: the four matrices, T1 (N^2 x (N + 1)^2) and the extra entries.
static long long rs_mirror_elems(long long n) {
  const long long c = n / 2, m = (c + 1) * (c + 1) + c * c;
  return m * m + n * n * (n + 1) * (n + 1) + rs_extra_elems(n);
}

template <class T>
hipError_t launch_direct(int n, const T* in, T* out, void* work, double pitch, double lam, double z, int primary,
                         hipStream_t st) {
  const long long nn = (long long)n * n, total = nn * nn;
  const double dx = lam * z / ((double)n * pitch);
  const double s = pitch * pitch * pitch * pitch;
  // The mirrored form wherever it fits the work buffer of two N^4 arrays (N >= 16). N = 64: 8.4 ms plain, 2.36 mirrored
  // in complex64, 21.4 and 4.6 ms in complex128; below N = 16 the products are a few tiles.
  const bool mirrored = rs_mirror_elems(n) <= 2 * total;
  const RsClasses cs = rs_classes(n, mirrored);
  T* h = reinterpret_cast<T*>(work);
  hipError_t e;
  if (!mirrored) {
    T* t1 = h + total;
    hipLaunchKernelGGL(k_rs_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, h, n, pitch, dx, z, lam,
                       primary);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_rs_gemm<T, true, false>(in, h, t1, (T*)nullptr, cs, 1.0, st)) != hipSuccess) return e;
    return launch_rs_gemm<T, false, false>(t1, h, out, (T*)nullptr, cs, s, st);
  }
  const int c = n / 2, w = c + 1;
  const long long m = (long long)w * w + (long long)c * c;
  T* t1 = h + m * m;
  T* extra = t1 + nn * (n + 1) * (n + 1);
  hipLaunchKernelGGL(k_rs_mirror<T>, dim3((unsigned)((w * w + 255) / 256), (unsigned)(w * w)), dim3(256), 0, st, h, cs,
                     pitch, dx, z, lam, primary);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const dim3 orbits((unsigned)(((long long)w * w * w * w + 255) / 256));
  hipLaunchKernelGGL((k_rs_fold<T, false>), orbits, dim3(256), 0, st, in, out, extra, n);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_rs_gemm<T, true, true>(out, h, t1, extra, cs, 1.0, st)) != hipSuccess) return e;
  if ((e = launch_rs_gemm<T, false, true>(t1, h, out, extra, cs, s, st)) != hipSuccess) return e;
  hipLaunchKernelGGL((k_rs_fold<T, true>), orbits, dim3(256), 0, st, (const T*)out, out, extra, n);
  return hipGetLastError();
}

size_t direct_work_bytes(int n, int elem) { return 2 * (size_t)n * n * n * n * (size_t)elem; }

template hipError_t launch_direct<float2>(int, const float2*, float2*, void*, double, double, double, int, hipStream_t);
template hipError_t launch_direct<double2>(int, const double2*, double2*, void*, double, double, double, int,
                                           hipStream_t);

}  // namespace wolf
