// Coarse-space transfer of the two-level method.
//
// Blocks (Two level preconditioner section): 4D boxes of bx*by*bz*bt sites
// tiling the lattice, each taken with all Ls slices.  On even-parity fields a
// block holds nsb = bx*by*bz*bt/2 even sites, listed in `bsite[b * nsb + j]`
// (half-lattice index, block-local lexicographic order).  On fields of both
// parities (packed "both" layout: the even halves of all n fields, then the
// odd halves) a block lists all nsb = bx*by*bz*bt sites, an odd site h as
// h + V4h; its data lies n half fields further on (the parity stride).  The
// blocked basis phi_k^b is a field phi_k restricted to block b.
//
// * chiral_split: P+- v = (v +- Gamma_5 v)/2 with (Gamma_5 v)_s = gamma_5
//   v_{Ls-1-s}: the five-dimensional chirality used when the domain-wall
//   operator is coarsened (Deflation basis setup section).
// * block_dot: c[r][b][k] = <phi_k^b, v_r>, the restrictor applied to nrhs
//   fields.
// * prolong: out_r = sum_k c[r][b][k] phi_k^b, FP64 and FP32 fields.
// * block_combine: the same for FP16 + scale fields, and the in-place map
//   phi_k <- sum_{j<=k} W[b][j][k] phi_j^b that orthonormalises them
//   (W = R^{-1} of the block's Cholesky factor); that map for the other
//   precisions and the Gram matrices are in gram.hip.
// * block_cholesky: per block G = R^dag R, then W = R^{-1}.
//
// One workgroup owns one block; its lane p = j * Ls + s holds one 5D site of
// the block (blocks of more than 512 5D sites: lane p also holds site
// p + 512).  Spinor loads are contiguous along s as in every other kernel.
// Sums over a block are reduced in a fixed order (wavefront shuffles, then
// the waves in index order), so results are reproducible run to run.
#include <algorithm>

#include "dwf_internal.hpp"
#include "kernels.hpp"

namespace dwf {

constexpr int KG = 4;  // basis vectors per reduction batch of block_dot

// (P+ v, P- v) for one lane: upper spins take (v_s + v_r)/2 and (v_s - v_r)/2,
// lower spins (gamma_5 = -1) the other way round; r = Ls - 1 - s
template <int P>
__global__ void __launch_bounds__(256) chiral_split_kernel(Geom g, const char* __restrict__ in, char* __restrict__ out,
                                                            size_t stride) {
  using R = typename Store<P>::real;
  const long long n = g.V4h * g.Ls;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k = blockIdx.y;
  const long long h = i / g.Ls;
  const int s = (int)(i - h * g.Ls);
  const char* v = in + (size_t)k * stride;
  cplx<R> a[12], b[12], p[12], m[12];
  Store<P>::load(v, g.V4h, g.Ls, h, s, a);
  Store<P>::load(v, g.V4h, g.Ls, h, g.Ls - 1 - s, b);
  const R half = (R)0.5;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const cplx<R> sum = {(a[c].re + b[c].re) * half, (a[c].im + b[c].im) * half};
    const cplx<R> dif = {(a[c].re - b[c].re) * half, (a[c].im - b[c].im) * half};
    p[c] = c < 6 ? sum : dif;
    m[c] = c < 6 ? dif : sum;
  }
  Store<P>::store(out + (size_t)(2 * k) * stride, g.V4h, g.Ls, h, s, p);
  Store<P>::store(out + (size_t)(2 * k + 1) * stride, g.V4h, g.Ls, h, s, m);
}

// Fixed-order sum of NV doubles over the workgroup; thread 0 gets the totals.
// red holds (blockDim / 64) * NV doubles.
template <int NV>
__device__ __forceinline__ void group_sum(double (&v)[NV], double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double x = v[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    v[i] = x;
  }
  __syncthreads();  // red is free
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) red[i * nw + wave] = v[i];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double t = 0;
      for (int w = 0; w < nw; ++w) t += red[i * nw + w];
      v[i] = t;
    }
  }
}

struct BlockArgs {
  Geom g;
  const int* bsite;  // [nb][nsb]; odd sites (fields of both parities) as h + V4h
  int nsb, nb;
  size_t basis_ps, v_ps, out_ps;  // byte offset of the odd halves (fields of both parities)
  const char* basis;  // nvec fields, stride `stride`
  int nvec;
  size_t stride;
  const char* v;  // block_dot: nrhs fields, stride `stride`
  char* out;      // block_combine: output fields (or the basis itself, in place)
  int nrhs;
  double* coef;        // block_dot output / block_combine input, complex [nrhs][nb][nvec]
  const double* wmat;  // block_combine in-place mode: complex [nb][nvec][nvec], W[j][k] at (j * nvec + k)
};

// Half-lattice site and parity of a block-table entry.
__device__ __forceinline__ int split_site(long long V4h, long long& h) {
  const int par = h >= V4h ? 1 : 0;
  h -= par * V4h;
  return par;
}

// c[r][b][k] = <phi_k^b, v_r> for the RT right-hand sides r = blockIdx.y * RT + ...
// A lane holds PP of the block's 5D sites (p = lane + q * blockDim.x), so a block
// may have up to PP * 512 of them.
template <int P, int RT, int PP>
__global__ void __launch_bounds__(512) block_dot_kernel(BlockArgs a) {
  using R = typename Store<P>::real;
  extern __shared__ double red[];
  const int b = blockIdx.x;
  const int r0 = blockIdx.y * RT;
  const int np = a.nsb * a.g.Ls;
  bool live[PP];
  long long h[PP];
  int s[PP], par[PP];
#pragma unroll
  for (int q = 0; q < PP; ++q) {
    const int p = threadIdx.x + q * blockDim.x;
    live[q] = p < np;
    h[q] = 0;
    s[q] = 0;
    par[q] = 0;
    if (live[q]) {
      const int j = p / a.g.Ls;
      s[q] = p - j * a.g.Ls;
      h[q] = a.bsite[(size_t)b * a.nsb + j];
      par[q] = split_site(a.g.V4h, h[q]);
    }
  }
  cplx<R> v[PP][RT][12];
#pragma unroll
  for (int q = 0; q < PP; ++q)
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const bool use = live[q] && (r0 + r < a.nrhs);
#pragma unroll
      for (int c = 0; c < 12; ++c) v[q][r][c] = {0, 0};
      if (use) Store<P>::load(a.v + par[q] * a.v_ps + (size_t)(r0 + r) * a.stride, a.g.V4h, a.g.Ls, h[q], s[q], v[q][r]);
    }
  const int kend = a.nvec;
  for (int k0 = blockIdx.z * KG; k0 < kend; k0 += KG * gridDim.z) {
    double acc[2 * RT * KG];
#pragma unroll
    for (int i = 0; i < 2 * RT * KG; ++i) acc[i] = 0;
#pragma unroll
    for (int kk = 0; kk < KG; ++kk) {
#pragma unroll
      for (int q = 0; q < PP; ++q) {
        if (live[q] && k0 + kk < kend) {
          cplx<R> f[12];
          Store<P>::load(a.basis + par[q] * a.basis_ps + (size_t)(k0 + kk) * a.stride, a.g.V4h, a.g.Ls, h[q], s[q], f);
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            double re = acc[2 * (r * KG + kk)], im = acc[2 * (r * KG + kk) + 1];
#pragma unroll
            for (int c = 0; c < 12; ++c) {  // conj(f) v
              re = fma((double)f[c].re, (double)v[q][r][c].re, re);
              re = fma((double)f[c].im, (double)v[q][r][c].im, re);
              im = fma((double)f[c].re, (double)v[q][r][c].im, im);
              im = fma(-(double)f[c].im, (double)v[q][r][c].re, im);
            }
            acc[2 * (r * KG + kk)] = re;
            acc[2 * (r * KG + kk) + 1] = im;
          }
        }
      }
    }
    group_sum<2 * RT * KG>(acc, red);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int kk = 0; kk < KG; ++kk)
          if (r0 + r < a.nrhs && k0 + kk < kend) {
            const size_t row = (size_t)(r0 + r) * a.nb + b;
            double* o = a.coef + 2 * (row * a.nvec + k0 + kk);
            o[0] = acc[2 * (r * KG + kk)];
            o[1] = acc[2 * (r * KG + kk) + 1];
          }
    }
  }
}

// Pair j of component pairs (2j, 2j + 1) at (h, s): 16 bytes of an FP32 field, twice 16 of an FP64 one.
template <class R>
__device__ __forceinline__ void load_pair(const char* f, long long row, int Ls, int s, cplx<R> v[2]) {
  if constexpr (sizeof(R) == 8) {
    const double2* q = reinterpret_cast<const double2*>(f) + 2 * row * Ls + s;
    const double2 x = q[0], y = q[Ls];
    v[0] = {x.x, x.y};
    v[1] = {y.x, y.y};
  } else {
    const float4 x = reinterpret_cast<const float4*>(f)[row * Ls + s];
    v[0] = {x.x, x.y};
    v[1] = {x.z, x.w};
  }
}
template <class R>
__device__ __forceinline__ void store_pair(char* f, long long row, int Ls, int s, const cplx<R> v[2]) {
  if constexpr (sizeof(R) == 8) {
    double2* q = reinterpret_cast<double2*>(f) + 2 * row * Ls + s;
    q[0] = make_double2(v[0].re, v[0].im);
    q[Ls] = make_double2(v[1].re, v[1].im);
  } else {
    reinterpret_cast<float4*>(f)[row * Ls + s] = make_float4(v[0].re, v[0].im, v[1].re, v[1].im);
  }
}

// out_r = sum_k coef[r][b][k] phi_k^b for the KT right-hand sides r = blockIdx.y * KT + ... of FP64
// and FP32 fields; a lane holds NP of a spinor's six component pairs, 6 / NP workgroups a block.
// Bound by the read of the basis.  8^3 x 16, Ls 8, 2^4 blocks of the even sites, 24 FP64 vectors:
// 51 -> 24 us for one rhs, 56 -> 34 for eight; 16^3 x 32, Ls 16, 40 FP32 vectors: 750 us for one
// (5.3 TB/s), 3290 -> 1850 for eight.
template <class R, int KT, int NP>
__global__ void __launch_bounds__(512) prolong_kernel(BlockArgs a) {
  constexpr int U = NP == 1 ? 4 : 1;  // vectors in flight
  extern __shared__ double cs[];      // complex coefficients [KT][nvec] of the block
  const int b = blockIdx.x, first = blockIdx.z * NP;
  const int np = a.nsb * a.g.Ls;
  const int n = a.nvec;
  const int r0 = blockIdx.y * KT;
  for (int i = threadIdx.x; i < KT * n; i += blockDim.x) {
    const int r = i / n, k = i - r * n;
    double re = 0, im = 0;
    if (r0 + r < a.nrhs) {
      const double* c = a.coef + 2 * (((size_t)(r0 + r) * a.nb + b) * n + k);
      re = c[0];
      im = c[1];
    }
    cs[2 * i] = re;
    cs[2 * i + 1] = im;
  }
  __syncthreads();
  for (int p = threadIdx.x; p < np; p += blockDim.x) {
    const int jsite = p / a.g.Ls;
    const int s = p - jsite * a.g.Ls;
    long long h = a.bsite[(size_t)b * a.nsb + jsite];
    const int par = split_site(a.g.V4h, h);
    const long long row = 6 * h + first;
    const char* bb = a.basis + par * a.basis_ps;
    cplx<double> acc[KT][2 * NP];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int c = 0; c < 2 * NP; ++c) acc[t][c] = {0, 0};
    auto load = [&](int j, cplx<R> f[2 * NP]) {
#pragma unroll
      for (int k = 0; k < NP; ++k) load_pair<R>(bb + (size_t)j * a.stride, row + k, a.g.Ls, s, f + 2 * k);
    };
    auto add = [&](int j, const cplx<R> f[2 * NP]) {
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const double cr = cs[2 * (t * n + j)], ci = cs[2 * (t * n + j) + 1];
#pragma unroll
        for (int c = 0; c < 2 * NP; ++c) {
          acc[t][c].re = fma(cr, (double)f[c].re, fma(-ci, (double)f[c].im, acc[t][c].re));
          acc[t][c].im = fma(cr, (double)f[c].im, fma(ci, (double)f[c].re, acc[t][c].im));
        }
      }
    };
    int j = 0;
    for (; j + U <= n; j += U) {
      cplx<R> f[U][2 * NP];
#pragma unroll
      for (int k = 0; k < U; ++k) load(j + k, f[k]);
#pragma unroll
      for (int k = 0; k < U; ++k) add(j + k, f[k]);
    }
    for (; j < n; ++j) {
      cplx<R> f[2 * NP];
      load(j, f);
      add(j, f);
    }
    char* ob = a.out + par * a.out_ps;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      if (r0 + t >= a.nrhs) continue;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const cplx<double>*v = acc[t] + 2 * k;
        const cplx<R> o[2] = {{(R)v[0].re, (R)v[0].im}, {(R)v[1].re, (R)v[1].im}};
        store_pair<R>(ob + (size_t)(r0 + t) * a.stride, row + k, a.g.Ls, s, o);
      }
    }
  }
}

// FP16 + scale: a lane owns whole spinors, whose largest number it needs for the stored form (the
// matrix-core combination and the lane-per-pair prolongation spread a spinor over lanes).
// INPLACE = false: out_r = sum_k coef[r][b][k] phi_k^b for the KT right-hand
//   sides r = blockIdx.y * KT + ...
// INPLACE = true: phi_k <- sum_{j<=k} W[b][j][k] phi_j^b for every k, one
//   workgroup per block taking the k tiles from the top down, so that the
//   phi_j a tile still needs (j below the tile) are not yet overwritten; every
//   lane reads and writes only its own 5D site.
template <int KT, bool INPLACE>
__global__ void __launch_bounds__(512) block_combine_kernel(BlockArgs a) {
  extern __shared__ double cs[];  // complex coefficients of the workgroup
  const int b = blockIdx.x;
  const int np = a.nsb * a.g.Ls;
  const int n = a.nvec;
  if (INPLACE) {
    for (int i = threadIdx.x; i < n * n; i += blockDim.x) {
      cs[2 * i] = a.wmat[2 * ((size_t)b * n * n + i)];
      cs[2 * i + 1] = a.wmat[2 * ((size_t)b * n * n + i) + 1];
    }
  } else {
    const int r0 = blockIdx.y * KT;
    for (int i = threadIdx.x; i < KT * n; i += blockDim.x) {
      const int r = i / n, k = i - r * n;
      double re = 0, im = 0;
      if (r0 + r < a.nrhs) {
        const double* c = a.coef + 2 * (((size_t)(r0 + r) * a.nb + b) * n + k);
        re = c[0];
        im = c[1];
      }
      cs[2 * i] = re;
      cs[2 * i + 1] = im;
    }
  }
  __syncthreads();
  // every lane handles the block's 5D sites p = lane, lane + blockDim.x, ...
  for (int p = threadIdx.x; p < np; p += blockDim.x) {
    const int jsite = p / a.g.Ls;
    const int s = p - jsite * a.g.Ls;
    long long h = a.bsite[(size_t)b * a.nsb + jsite];
    const int par = split_site(a.g.V4h, h);
    const char* bb = a.basis + par * a.basis_ps;
    char* ob = a.out + par * a.out_ps;
    const int ntiles = INPLACE ? (n + KT - 1) / KT : 1;
    for (int tile = ntiles - 1; tile >= 0; --tile) {
      const int k0 = tile * KT;                         // INPLACE: outputs k0 .. k0+KT-1
      const int jmax = INPLACE ? min(n, k0 + KT) : n;  // inputs j < jmax
      cplx<double> acc[KT][12];
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[t][c] = {0, 0};
      for (int j = 0; j < jmax; ++j) {
        cplx<float> f[12];
        Store<DWF_F16S>::load(bb + (size_t)j * a.stride, a.g.V4h, a.g.Ls, h, s, f);
#pragma unroll
        for (int t = 0; t < KT; ++t) {
          // coefficient of phi_j in output t
          const int idx = INPLACE ? (j * n + k0 + t) : (t * n + j);
          if (INPLACE && (k0 + t >= n || j > k0 + t)) continue;
          const double cr = cs[2 * idx], ci = cs[2 * idx + 1];
#pragma unroll
          for (int c = 0; c < 12; ++c) {
            acc[t][c].re = fma(cr, (double)f[c].re, fma(-ci, (double)f[c].im, acc[t][c].re));
            acc[t][c].im = fma(cr, (double)f[c].im, fma(ci, (double)f[c].re, acc[t][c].im));
          }
        }
      }
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const int k = INPLACE ? k0 + t : blockIdx.y * KT + t;
        if (k >= (INPLACE ? n : a.nrhs)) continue;
        cplx<float> o[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) o[c] = {(float)acc[t][c].re, (float)acc[t][c].im};
        Store<DWF_F16S>::store(ob + (size_t)k * a.stride, a.g.V4h, a.g.Ls, h, s, o);
      }
    }
  }
}

// Per block: Cholesky G = R^dag R of the Hermitian Gram matrix
// G[k][j] = <phi_j, phi_k> (only j <= k is read), then W = R^{-1}, upper
// triangular, stored W[j][k] at (j * n + k).  One wave per block, lane k owning
// column k: row j of R is R[j][k] = (G_jk - sum_{i<j} conj(R[i][j]) R[i][k]) / R[j][j],
// computed by all lanes k >= j at once, the diagonal among them; column k of
// R^{-1} then needs only R and the lane's own column.  R and W stay in LDS: a
// column read back from memory at every step made this a chain of memory
// round trips (0.44 ms for 2048 blocks of 40 vectors).  A non-positive or
// non-finite pivot raises *flag.
__global__ void __launch_bounds__(64) block_cholesky_kernel(const double2* __restrict__ gram, double2* __restrict__ w,
                                                            int nb, int n, int* flag) {
  extern __shared__ double2 rs[];  // R [n][n], then W [n][n]
  double2* ws = rs + n * n;
  const int b = blockIdx.x;
  const int k = threadIdx.x;
  const double2* G = gram + (size_t)b * n * n;
  for (int i = k; i < n * n; i += 64) ws[i] = G[i];  // G waits where W will be, entry (k, j) at k * n + j
  __syncthreads();
  for (int j = 0; j < n; ++j) {
    double re = 0, im = 0;
    if (k >= j && k < n) {
      const double2 g = ws[k * n + j];  // G_jk = <phi_j, phi_k>
      re = g.x;
      im = g.y;
      for (int i = 0; i < j; ++i) {
        const double2 c = rs[i * n + j], r = rs[i * n + k];  // conj(R[i][j]) R[i][k]
        re -= c.x * r.x + c.y * r.y;
        im -= c.x * r.y - c.y * r.x;
      }
    }
    double d = __shfl(re, j);
    if (!(d > 0.0) || !isfinite(d)) {
      if (k == j) *flag = 1;
      d = 1.0;
    }
    const double root = sqrt(d), inv = 1.0 / root;
    if (k >= j && k < n) rs[j * n + k] = k == j ? make_double2(root, 0.0) : make_double2(re * inv, im * inv);
    __syncthreads();
  }
  // column k of R^{-1}: W[k][k] = 1 / R[k][k]; W[j][k] = -(sum_{i=j+1..k} R[j][i] W[i][k]) / R[j][j]
  if (k < n) {
    for (int j = k + 1; j < n; ++j) ws[j * n + k] = make_double2(0.0, 0.0);
    ws[k * n + k] = make_double2(1.0 / rs[k * n + k].x, 0.0);
    for (int j = k - 1; j >= 0; --j) {
      double re = 0, im = 0;
      for (int i = j + 1; i <= k; ++i) {
        const double2 r = rs[j * n + i], v = ws[i * n + k];
        re += r.x * v.x - r.y * v.y;
        im += r.x * v.y + r.y * v.x;
      }
      const double inv = -1.0 / rs[j * n + j].x;
      ws[j * n + k] = make_double2(re * inv, im * inv);
    }
  }
  __syncthreads();
  double2* W = w + (size_t)b * n * n;
  for (int i = k; i < n * n; i += 64) W[i] = ws[i];
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static int lanes_of(const dwf_context* c) { return c->nsb * c->g.Ls; }
// workgroup of a per-block kernel: one lane per 5D site of the block, at most 512
static int group_of(int lanes) { return std::min(512, (lanes + 63) / 64 * 64); }

hipError_t launch_chiral_split(dwf_context* c, int prec, const char* in, char* out, int nvec) {
  const long long n = c->g.V4h * c->g.Ls;
  dim3 grid((unsigned)((n + 255) / 256), nvec);
  const size_t st = field_bytes_rhs(c, prec);
  // fields of both parities: the even halves, then the odd halves (nvec in, 2 nvec out)
  for (int par = 0; par < (c->coarse_both ? 2 : 1); ++par) {
    const char* i = in + (size_t)par * nvec * st;
    char* o = out + (size_t)par * 2 * nvec * st;
    switch (prec) {
      case DWF_F64: hipLaunchKernelGGL(chiral_split_kernel<DWF_F64>, grid, dim3(256), 0, c->stream, c->g, i, o, st); break;
      case DWF_F32: hipLaunchKernelGGL(chiral_split_kernel<DWF_F32>, grid, dim3(256), 0, c->stream, c->g, i, o, st); break;
      default: hipLaunchKernelGGL(chiral_split_kernel<DWF_F16S>, grid, dim3(256), 0, c->stream, c->g, i, o, st); break;
    }
  }
  return hipGetLastError();
}

static BlockArgs block_args(const dwf_context* c, int prec, const char* basis, int nvec) {
  BlockArgs a{};
  a.g = c->g;
  a.bsite = c->bsite;
  a.nsb = c->nsb;
  a.nb = c->nb;
  a.basis = basis;
  a.nvec = nvec;
  a.stride = field_bytes_rhs(c, prec);
  a.basis_ps = c->coarse_both ? (size_t)nvec * a.stride : 0;
  return a;
}

template <int P, int RT, int PP>
static void dot_t(const dwf_context* c, const BlockArgs& a) {
  const int lanes = group_of(lanes_of(c));
  const size_t lds = (size_t)(lanes / 64) * 2 * RT * KG * sizeof(double);
  // Up to a wave a SIMD (1024) the batches of basis vectors go to several workgroups, each with its
  // own copy of v: 8^3 x 16, Ls 8, 24 FP64 vectors, one rhs 39 -> 25 us; with more waves the copies
  // cost more than they hide (three rhs of 4 x 4 x 2 x 4 blocks, 1536 waves: 32 -> 39 us).
  const long long waves = (long long)a.nb * ((a.nrhs + RT - 1) / RT) * (lanes / 64);
  const int groups = (a.nvec + KG - 1) / KG;
  const int split = waves <= 1024 ? (int)std::min<long long>(groups, 4096 / waves) : 1;
  hipLaunchKernelGGL((block_dot_kernel<P, RT, PP>), dim3(a.nb, (a.nrhs + RT - 1) / RT, split), dim3(lanes), lds,
                     c->stream, a);
}

// blocks of up to 512 5D sites: one site and one or two rhs per lane; up to 1024: two sites and one rhs
template <int P>
static void dot_p(const dwf_context* c, const BlockArgs& a) {
  if (lanes_of(c) > 512)
    dot_t<P, 1, 2>(c, a);
  else if (a.nrhs == 1)
    dot_t<P, 1, 1>(c, a);
  else
    dot_t<P, 2, 1>(c, a);
}

hipError_t launch_block_dot(dwf_context* c, int prec, const char* basis, int nvec, const char* v, int nrhs,
                            double* coef) {
  BlockArgs a = block_args(c, prec, basis, nvec);
  a.v = v;
  a.nrhs = nrhs;
  a.v_ps = c->coarse_both ? (size_t)nrhs * a.stride : 0;
  a.coef = coef;
  switch (prec) {
    case DWF_F64: dot_p<DWF_F64>(c, a); break;
    case DWF_F32: dot_p<DWF_F32>(c, a); break;
    default: dot_p<DWF_F16S>(c, a); break;
  }
  return hipGetLastError();
}

template <int KT, bool INPLACE>
static void combine_t(const dwf_context* c, const BlockArgs& a) {
  const int lanes = group_of(lanes_of(c));
  const size_t lds = (INPLACE ? (size_t)a.nvec * a.nvec : (size_t)KT * a.nvec) * 2 * sizeof(double);
  const unsigned gy = INPLACE ? 1 : (unsigned)((a.nrhs + KT - 1) / KT);
  hipLaunchKernelGGL((block_combine_kernel<KT, INPLACE>), dim3(a.nb, gy), dim3(lanes), lds, c->stream, a);
}

template <class R, int KT, int NP>
static void prolong_t(const dwf_context* c, const BlockArgs& a) {
  const size_t lds = (size_t)KT * a.nvec * 2 * sizeof(double);
  hipLaunchKernelGGL((prolong_kernel<R, KT, NP>),
                     dim3(a.nb, (unsigned)((a.nrhs + KT - 1) / KT), 6 / NP), dim3(group_of(lanes_of(c))),
                     lds, c->stream, a);
}

template <class R>
static void prolong_r(const dwf_context* c, const BlockArgs& a) {
  // Below four waves a SIMD a lane per spinor leaves the chip waiting on its chain of vectors, so a
  // lane takes a sixth of one; for three or more rhs the small accumulators of that form also let
  // four share a read of the basis.  Else the lane per spinor reads each site's lines together.
  // Up to three FP32 vectors that also holds for three and more rhs: the outputs are then most of
  // the bytes, and six workgroups a block write them in pieces (16^3 x 32, 2^4 blocks, four rhs: one
  // vector 98 us whole and 130 in sixths at Ls 16, 74 and 137 at Ls 12, three vectors 182 and 157,
  // 137 and 170; four vectors 220 and 165, 167 and 163; FP64 of one 228 and 200, 177 and 159).
  const bool whole = (long long)a.nb * (group_of(lanes_of(c)) / 64) >= 4096;
  const bool few = sizeof(R) == 4 && a.nvec <= 3;
  if (a.nrhs > 2 && !(whole && few))
    prolong_t<R, 4, 1>(c, a);
  else if (whole)
    prolong_t<R, 2, 6>(c, a);
  else if (a.nrhs == 2)
    prolong_t<R, 2, 1>(c, a);
  else
    prolong_t<R, 1, 1>(c, a);
}

hipError_t launch_block_prolong(dwf_context* c, int prec, const char* basis, int nvec, const double* coef, int nrhs,
                                char* out) {
  BlockArgs a = block_args(c, prec, basis, nvec);
  a.coef = const_cast<double*>(coef);
  a.nrhs = nrhs;
  a.out = out;
  a.out_ps = c->coarse_both ? (size_t)nrhs * a.stride : 0;
  switch (prec) {
    case DWF_F64: prolong_r<double>(c, a); break;
    case DWF_F32: prolong_r<float>(c, a); break;
    default: combine_t<2, false>(c, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_block_apply(dwf_context* c, int prec, char* basis, int nvec, const double* wmat) {
  if (prec != DWF_F16S) return launch_block_apply_mfma(c, prec, basis, nvec, wmat);
  BlockArgs a = block_args(c, prec, basis, nvec);
  a.wmat = wmat;
  a.out = basis;
  a.out_ps = a.basis_ps;
  combine_t<2, true>(c, a);
  return hipGetLastError();
}

hipError_t launch_block_cholesky(dwf_context* c, const double* gram, double* w, int nvec, int* flag) {
  hipLaunchKernelGGL(block_cholesky_kernel, dim3(c->nb), dim3(64), (size_t)nvec * nvec * 2 * sizeof(double2), c->stream,
                     reinterpret_cast<const double2*>(gram), reinterpret_cast<double2*>(w), c->nb, nvec, flag);
  return hipGetLastError();
}

}  // namespace dwf
