// Gram matrices and in-place triangular combinations of up to 64 fields on the
// FP64 matrix cores: the two halves of a Cholesky QR round, for every block of
// the coarse space (block orthonormalisation) and for the whole lattice
// (Gram-Schmidt).
//
// Both work on sets of 4D sites: a site's 12 Ls complex values are contiguous in
// every vector (FP16 + scale: its 3 Ls groups of 16 bytes, and its Ls scales).
// A workgroup takes one set -- a block's sites, or an equal range of the lattice --
// and its waves take every fourth site.
//
// Gram: with X the real matrix of a set's values, one row per complex value and
// columns (vector, re / im) interleaved, X^T X holds every product the complex
// Gram matrix needs, Re G = S_rr + S_ii and Im G = S_ri - S_ir.  As real columns
// n = 40 vectors are exactly five tiles of 16, and the 15 upper tiles cost 15
// 16x16x4 MFMAs per four rows where complex tiles of 16 vectors cost 24.  The
// left and right operands of X^T X are the same registers, so a lane loads 16
// bytes of its vector per tile (both halves of a 128-byte line back to back),
// converts its part to FP64 and feeds it to every tile of the row: no LDS.
//
// Combination: v_k <- sum_{j <= k} W[j][k] v_j as the transposed product
// W^T X^T, so that the 16 columns of a tile are 16 consecutive values of a vector
// (whole lines) and a lane ends with both parts of its vectors.  All vectors of a
// wave's 16 values are in registers before the first is written, which makes
// the update in place safe; W is laid out in LDS in the order the lanes read it.
#include <algorithm>

#include "dwf_internal.hpp"
#include "kernels.hpp"

namespace dwf {
namespace {

typedef double d4v __attribute__((ext_vector_type(4)));
// 16 bytes of a vector, which Gram-Schmidt takes at any multiple of 8 (as the combination's
// accesses of one complex value do); the loads are global_load_dwordx4 all the same
typedef float f4v __attribute__((ext_vector_type(4), aligned(8)));
typedef double d2v __attribute__((ext_vector_type(2), aligned(8)));

constexpr int GW = 4;  // waves of a workgroup

struct SetArgs {
  char* V;            // n fields, `stride` bytes apart (the odd halves `odd` bytes on)
  size_t stride, odd;
  const int* bsite;   // [sets][nsites] (odd sites as h + V4h), or null: set g is sites g * nsites ..
  int nsites;
  int sets, set8;     // number of sets; sets per XCD
  long long V4h;
  int Ls, n;
};

// Site i of set g: byte offset of its half field, and its index.
__device__ __forceinline__ long long set_site(const SetArgs& a, const int* __restrict__ bsite, int g, int i, int& par) {
  long long h = bsite ? (long long)bsite[(size_t)g * a.nsites + i] : (long long)g * a.nsites + i;
  par = h >= a.V4h ? 1 : 0;
  return h - par * a.V4h;
}
// number of sites of set g (the last range of the lattice may be short)
__device__ __forceinline__ int set_size(const SetArgs& a, int g) {
  if (a.bsite) return a.nsites;
  const long long left = a.V4h - (long long)g * a.nsites;
  return left < a.nsites ? (left > 0 ? (int)left : 0) : a.nsites;
}

// Complex values per 16-byte unit of a site.
template <int P>
struct Unit;
template <>
struct Unit<DWF_F64> {
  static constexpr int values = 1;
};
template <>
struct Unit<DWF_F32> {
  static constexpr int values = 2;
};
template <>
struct Unit<DWF_F16S> {
  static constexpr int values = 4;
};

// One 16-byte unit as loaded, and its part (re or im) of value v in FP64.
template <int P>
struct Loaded {
  f4v q;
  __device__ __forceinline__ void load(const char* site, const char*, int u, int) {
    q = *reinterpret_cast<const f4v*>(site + (size_t)u * 16);
  }
  __device__ __forceinline__ double part(int v, bool im) const { return (double)(im ? q[2 * v + 1] : q[2 * v]); }
};
template <>
struct Loaded<DWF_F64> {
  d2v q;
  __device__ __forceinline__ void load(const char* site, const char*, int u, int) {
    q = *reinterpret_cast<const d2v*>(site + (size_t)u * 16);
  }
  __device__ __forceinline__ double part(int, bool im) const { return im ? q.y : q.x; }
};
template <>
struct Loaded<DWF_F16S> {
  half8v q;
  float scale;
  __device__ __forceinline__ void load(const char* site, const char* scales, int u, int Ls) {
    q = *reinterpret_cast<const half8v*>(site + (size_t)u * 16);
    const int s = u < Ls ? u : (u < 2 * Ls ? u - Ls : u - 2 * Ls);
    scale = reinterpret_cast<const float*>(scales)[s];
  }
  __device__ __forceinline__ double part(int v, bool im) const {
    return (double)((float)(im ? q[2 * v + 1] : q[2 * v]) * scale);
  }
};

// G[g][k][j] = <v_j, v_k> over set g, j <= k.  T = ceil(n / 8) tiles of 16 real columns;
// the launch forms the upper tile pairs FIRST .. LAST - 1, counted row by row.
template <int P, int T, int FIRST, int LAST>
__global__ void __launch_bounds__(64 * GW) __attribute__((amdgpu_waves_per_eu(T <= 5 ? 2 : 1)))
gram_kernel(SetArgs a, const int* __restrict__ bsite, double2* __restrict__ G) {
  constexpr int NT = LAST - FIRST;
  constexpr bool AHEAD = T <= (P == DWF_F16S ? 4 : 6);  // beyond, the registers hold the tiles and one step
  __shared__ double red[GW][4][64];
  const int g = (blockIdx.x & 7) * a.set8 + (blockIdx.x >> 3);  // neighbouring sets on one XCD
  if (g >= a.sets) return;                                      // whole workgroup leaves together
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int col = lane & 15, q = lane >> 4;
  const bool im = (col & 1) != 0;
  const int units = 12 * a.Ls / Unit<P>::values;
  const int count = set_size(a, g);
  // lanes past the last vector repeat it; their products are not stored
  auto vec_of = [&](int t) { return min(8 * t + (col >> 1), a.n - 1); };

  d4v acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) acc[i] = d4v{0, 0, 0, 0};
  // a step: eight units (a 128-byte line) of one site, four lanes by two
  Loaded<P> cur[T][2], nxt[T][2];
  auto fetch = [&](Loaded<P> (&x)[T][2], int i, int u0) {
    int par;
    const long long h = set_site(a, bsite, g, i, par);
    const size_t site = par * a.odd + (size_t)h * units * 16;
    const size_t scales = par * a.odd + (size_t)a.V4h * a.Ls * 48 + (size_t)h * a.Ls * 4;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const char* f = a.V + (size_t)vec_of(t) * a.stride;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) x[t][hf].load(f + site, f + scales, min(u0 + 4 * hf + q, units - 1), a.Ls);
    }
  };
  int i = wave, u0 = 0;
  if (i < count) fetch(cur, i, 0);
  while (i < count) {
    int ni = i, nu = u0 + 8;
    if (nu >= units) {
      nu = 0;
      ni += GW;
    }
    if (AHEAD && ni < count) fetch(nxt, ni, nu);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const bool in = u0 + 4 * hf + q < units;  // a site of no whole number of lines: idle lanes count as zero
#pragma unroll
      for (int v = 0; v < Unit<P>::values; ++v) {
        double x[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const double w = cur[t][hf].part(v, im);
          x[t] = in ? w : 0.0;
        }
        int p = 0;
#pragma unroll
        for (int ta = 0; ta < T; ++ta)
#pragma unroll
          for (int tb = ta; tb < T; ++tb, ++p)
            if (p >= FIRST && p < LAST)
              acc[p - FIRST] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[ta], x[tb], acc[p - FIRST], 0, 0, 0);
      }
    }
    if (AHEAD) {
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) cur[t][hf] = nxt[t][hf];
    } else if (ni < count) {
      fetch(cur, ni, nu);
    }
    i = ni;
    u0 = nu;
  }
  // the waves' sums in wave order, tile by tile; element (r, lane) of a tile is row
  // q + 4 r, column col, so the four parts of a complex entry sit in lanes l, l ^ 1, l ^ 16, l ^ 17
  double2* out = G + (size_t)g * a.n * a.n;
  int p = 0;
#pragma unroll
  for (int ta = 0; ta < T; ++ta)
#pragma unroll
    for (int tb = ta; tb < T; ++tb, ++p) {
      if (p < FIRST || p >= LAST) continue;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[p - FIRST][r];
      __syncthreads();
      const int r = wave;
      double s = 0;
#pragma unroll
      for (int w = 0; w < GW; ++w) s += red[w][r][lane];
      const double ri = __shfl_xor(s, 1), ir = __shfl_xor(s, 16), ii = __shfl_xor(s, 17);
      const int j = (16 * ta + q + 4 * r) >> 1, k = (16 * tb + col) >> 1;
      if (!im && !(q & 1) && j <= k && k < a.n) out[(size_t)k * a.n + j] = make_double2(s + ii, ri - ir);
    }
}

// G[e] = sum over the sets, in a fixed order, of part[set][e] (n * n entries, 16 per workgroup;
// entry k * n + j with j > k is not used)
__global__ void __launch_bounds__(256) gram_sum_kernel(const double2* __restrict__ part, int sets, int n,
                                                       double2* __restrict__ G) {
  __shared__ double2 red[16][16];
  const int e = threadIdx.x & 15, w = threadIdx.x >> 4;
  const int idx = blockIdx.x * 16 + e, nn = n * n;
  double2 s = make_double2(0, 0);
  if (idx < nn && idx % n <= idx / n)
    for (int k = w; k < sets; k += 16) {
      const double2 x = part[(size_t)k * nn + idx];
      s.x += x.x;
      s.y += x.y;
    }
  red[w][e] = s;
  __syncthreads();
  if (w == 0 && idx < nn) {
    for (int k = 1; k < 16; ++k) {
      s.x += red[k][e].x;
      s.y += red[k][e].y;
    }
    G[idx] = s;
  }
}

// v_k <- sum_{j <= k} W[j][k] v_j over set g, W (complex, [j][k], per set `wstride` entries
// apart) upper triangular.  T = ceil(n / 8) output tiles of 8 vectors.
template <class R, int T>
__global__ void __launch_bounds__(64 * GW) __attribute__((amdgpu_waves_per_eu(T <= 5 ? 2 : 1)))
combine_kernel(SetArgs a, const int* __restrict__ bsite, const double2* __restrict__ W, size_t wstride) {
  constexpr int NG = 2 * T;           // groups of four input vectors
  constexpr bool AHEAD = T <= 5;      // beyond, the registers hold one step's values
  extern __shared__ double wt[];      // [T (T + 1) * 2][64]
  const int g = (blockIdx.x & 7) * a.set8 + (blockIdx.x >> 3);
  if (g >= a.sets) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int e = lane & 15, q = lane >> 4;
  const int n = a.n;
  // Operand (tile t, group m, part pi) of W^T: row rho of the tile is part (rho / 4) % 2 of vector
  // 8 t + 4 (rho / 8) + rho % 4, inner index q is part pi of vector 4 m + q; groups m <= 2 t + 1
  // reach the tile, at ((t (t + 1) + m) * 2 + pi).
  const double2* Wg = W + (size_t)g * wstride;
  for (int t = 0, idx = 0; t < T; ++t)
    for (int m = 0; m <= 2 * t + 1; ++m)
      for (int pi = 0; pi < 2; ++pi, ++idx) {
        if ((idx & (GW - 1)) != wave) continue;
        const int rho = e, vo = 8 * t + 4 * (rho >> 3) + (rho & 3), po = (rho >> 2) & 1, vi = 4 * m + q;
        double w = 0.0;
        if (vi <= vo && vo < n) {
          const double2 c = Wg[(size_t)vi * n + vo];
          w = po == pi ? c.x : (po ? c.y : -c.y);
        }
        wt[idx * 64 + lane] = w;
      }
  __syncthreads();
  const int values = 12 * a.Ls;
  const int count = set_size(a, g);
  cplx<R> cur[NG], nxt[NG];
  auto fetch = [&](cplx<R> (&x)[NG], int i, int e0) {
    int par;
    const long long h = set_site(a, bsite, g, i, par);
    const size_t at = par * a.odd + ((size_t)h * values + min(e0 + e, values - 1)) * sizeof(cplx<R>);
#pragma unroll
    for (int m = 0; m < NG; ++m)
      x[m] = *reinterpret_cast<const cplx<R>*>(a.V + (size_t)min(4 * m + q, n - 1) * a.stride + at);
  };
  int i = wave, e0 = 0;
  if (i < count) fetch(cur, i, 0);
  while (i < count) {
    int ni = i, ne = e0 + 16;
    if (ne >= values) {
      ne = 0;
      ni += GW;
    }
    if (AHEAD && ni < count) fetch(nxt, ni, ne);
    int par;
    const long long h = set_site(a, bsite, g, i, par);
    char* site = a.V + par * a.odd + ((size_t)h * values + e0 + e) * sizeof(cplx<R>);
    const bool in = e0 + e < values;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      d4v acc = d4v{0, 0, 0, 0};
#pragma unroll
      for (int m = 0; m <= 2 * t + 1; ++m) {
        const double* w = wt + ((t * (t + 1) + m) * 2) * 64 + lane;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(w[0], (double)cur[m].re, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(w[64], (double)cur[m].im, acc, 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int v = 8 * t + 4 * k + q;
        if (in && v < n)
          *reinterpret_cast<cplx<R>*>(site + (size_t)v * a.stride) = cplx<R>{(R)acc[2 * k], (R)acc[2 * k + 1]};
      }
    }
    if (AHEAD) {
#pragma unroll
      for (int m = 0; m < NG; ++m) cur[m] = nxt[m];
    } else if (ni < count) {
      fetch(cur, ni, ne);
    }
    i = ni;
    e0 = ne;
  }
}

template <int P, int T, int FIRST = 0, int LAST = T * (T + 1) / 2>
hipError_t gram_t(dwf_context* c, const SetArgs& a, double* G) {
  hipLaunchKernelGGL((gram_kernel<P, T, FIRST, LAST>), dim3((unsigned)a.set8 * 8), dim3(64 * GW), 0, c->stream, a,
                     a.bsite, reinterpret_cast<double2*>(G));
  return hipGetLastError();
}

template <int P>
hipError_t gram_p(dwf_context* c, const SetArgs& a, double* G) {
  switch ((a.n + 7) / 8) {
    case 1: return gram_t<P, 1>(c, a, G);
    case 2: return gram_t<P, 2>(c, a, G);
    case 3: return gram_t<P, 3>(c, a, G);
    case 4: return gram_t<P, 4>(c, a, G);
    case 5: return gram_t<P, 5>(c, a, G);
    case 6: return gram_t<P, 6>(c, a, G);
    case 7: return gram_t<P, 7>(c, a, G);
    default: {  // 36 tiles do not fit the 256 registers the products can address: two launches
      const hipError_t e = gram_t<P, 8, 0, 18>(c, a, G);
      return e != hipSuccess ? e : gram_t<P, 8, 18, 36>(c, a, G);
    }
  }
}

hipError_t gram_sets(dwf_context* c, int prec, const SetArgs& a, double* G) {
  switch (prec) {
    case DWF_F64: return gram_p<DWF_F64>(c, a, G);
    case DWF_F32: return gram_p<DWF_F32>(c, a, G);
    default: return gram_p<DWF_F16S>(c, a, G);
  }
}

template <class R, int T>
hipError_t combine_t(dwf_context* c, const SetArgs& a, const double* W, size_t wstride) {
  const size_t lds = (size_t)T * (T + 1) * 2 * 64 * sizeof(double);
  hipLaunchKernelGGL((combine_kernel<R, T>), dim3((unsigned)a.set8 * 8), dim3(64 * GW), lds, c->stream, a, a.bsite,
                     reinterpret_cast<const double2*>(W), wstride);
  return hipGetLastError();
}

template <class R>
hipError_t combine_r(dwf_context* c, const SetArgs& a, const double* W, size_t wstride) {
  switch ((a.n + 7) / 8) {
    case 1: return combine_t<R, 1>(c, a, W, wstride);
    case 2: return combine_t<R, 2>(c, a, W, wstride);
    case 3: return combine_t<R, 3>(c, a, W, wstride);
    case 4: return combine_t<R, 4>(c, a, W, wstride);
    case 5: return combine_t<R, 5>(c, a, W, wstride);
    case 6: return combine_t<R, 6>(c, a, W, wstride);
    case 7: return combine_t<R, 7>(c, a, W, wstride);
    default: return combine_t<R, 8>(c, a, W, wstride);
  }
}

SetArgs set_args(const dwf_context* c, int prec, const char* V, int n) {
  SetArgs a{};
  a.V = const_cast<char*>(V);
  a.stride = field_bytes_rhs(c, prec);
  a.V4h = c->g.V4h;
  a.Ls = c->g.Ls;
  a.n = n;
  return a;
}

SetArgs block_sets(const dwf_context* c, int prec, const char* basis, int n) {
  SetArgs a = set_args(c, prec, basis, n);
  a.odd = c->coarse_both ? (size_t)n * a.stride : 0;
  a.bsite = c->bsite;
  a.nsites = c->nsb;
  a.sets = c->nb;
  a.set8 = (c->nb + 7) / 8;
  return a;
}

// the lattice (one parity) as about `sets` equal ranges of sites
SetArgs lattice_sets(const dwf_context* c, int prec, const char* V, int n, int sets) {
  SetArgs a = set_args(c, prec, V, n);
  a.nsites = (int)((a.V4h + sets - 1) / sets);
  a.sets = (int)((a.V4h + a.nsites - 1) / a.nsites);
  a.set8 = (a.sets + 7) / 8;
  return a;
}

}  // namespace

hipError_t launch_block_gram(dwf_context* c, int prec, const char* basis, int nvec, double* gram) {
  return gram_sets(c, prec, block_sets(c, prec, basis, nvec), gram);
}

hipError_t launch_block_apply_mfma(dwf_context* c, int prec, char* basis, int nvec, const double* wmat) {
  const SetArgs a = block_sets(c, prec, basis, nvec);
  const size_t nn = (size_t)nvec * nvec;
  return prec == DWF_F64 ? combine_r<double>(c, a, wmat, nn) : combine_r<float>(c, a, wmat, nn);
}

hipError_t ts_gram(dwf_context* ctx, int prec, const char* V, int n, double* partial, int nwg, double* G) {
  if (n < 1 || n > TS_NMAX || nwg < 1 || prec < DWF_F64 || prec > DWF_F16S) return hipErrorInvalidValue;
  const SetArgs a = lattice_sets(ctx, prec, V, n, nwg);
  const hipError_t e = gram_sets(ctx, prec, a, partial);
  if (e != hipSuccess) return e;
  const int nn = n * n;
  hipLaunchKernelGGL(gram_sum_kernel, dim3((unsigned)((nn + 15) / 16)), dim3(256), 0, ctx->stream,
                     reinterpret_cast<const double2*>(partial), a.sets, n, reinterpret_cast<double2*>(G));
  return hipGetLastError();
}

hipError_t ts_combine_mfma(dwf_context* ctx, int prec, char* V, int n, const double* W) {
  // 4096 ranges: several for every resident workgroup, so that a slow one does not end the pass
  const SetArgs a = lattice_sets(ctx, prec, V, n, 4096);
  return prec == DWF_F64 ? combine_r<double>(ctx, a, W, 0) : combine_r<float>(ctx, a, W, 0);
}

}  // namespace dwf
