// The little Dirac operator of the two-level method (Two level preconditioner
// section): A^{ab}_{jk} = <phi_j^a | H_DW | phi_k^b> on a blocked basis, FP64, as
// the 9-point stencil [nb][9][n][n] with entry (j, k) at k * n + j (points as in
// dwf_hdcr_coarse_data).
//
// One workgroup owns a block.  Its waves are four directions times KW tiles of 16
// columns k; every wave keeps the 16 x 16 tiles of the FP64 matrix cores of its
// direction's face and of its part of the block itself, for JT tiles of rows j.
// The workgroup walks the block's sites, eight slices (a 128-byte line of FP64
// spinors) at a time: the site's own vectors phi_j pass through LDS, where all
// waves read them as left operands, and each wave loads the neighbour's spinors
// phi_k straight into registers, projects and rotates them there and uses them as
// right operands.  Every spin-colour component is then one step of the product's
// inner index; no intermediate field is written, and every line of the basis that
// is fetched is used whole.
//
// Two identities keep the work small.  Across a face the hop needs only half
// spinors: phi_j^dag gamma_5 (1 + sigma g_mu) chi = (u_j - sigma B l_j)^dag (u + sigma B l)_chi,
// six inner steps instead of twelve.  And H_DW is Hermitian, so the backward
// points are the conjugate transposes of the neighbouring blocks' forward ones:
// four face products and one for the block itself instead of nine.
//
// What bounds it: the fabric, then the matrix cores.  16^3 x 32, Ls 16, 32 vectors on
// 2^4 blocks takes 21.5 ms: 0.62 TFLOP (36 complex inner steps per 5D site, 9 ms at the
// 69 TFLOP/s the FP64 matrix cores reach) and 108 GB of line reads by the L1s, 100 GB of
// them from beyond L2, with 8.4 GB written where the stencil is 1.2 GB, together 5.0 TB/s --
// own vectors once, neighbours four times, the site-local part twice (it could come from the
// staged vectors); a block's 1.6 MB of vectors do not stay in an L2 that 32 workgroups share.
// The two-tile forms spill 58 registers (228 bytes a lane), the three-tile form 81 (328), part
// of them in the site loop: scratch traffic and the waits for it are in these figures.  Measured before: a workgroup
// per stencil point and block with both operands loaded 64 bytes of a line at a time,
// 41.9 ms (285 GB, 6.3 TB/s); nine fields written per basis vector and each restricted
// onto the whole basis, 389 ms.
#include "dwf_internal.hpp"
#include "kernels.hpp"

namespace dwf {
namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int SL = 8;  // slices of a step: one 128-byte line of an FP64 component

struct StencilArgs {
  Geom g;
  int blk[4];
  int nsb, nb, nb8, n;
  double d, mf;         // 5 - M5, mass
  const int* bnbr;      // [nb][8]
  const char* basis;    // n fields of both parities: even halves, then odd halves
  size_t fb;            // bytes of a half field
};

// acc += conj(a) b over one inner step (4 slices) of a 16 x 16 tile
__device__ __forceinline__ void tile_step(cplx<double> a, cplx<double> b, d4v& re, d4v& im) {
  re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.re, re, 0, 0, 0);
  im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.im, im, 0, 0, 0);
  re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.im, b.im, re, 0, 0, 0);
  im = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.im, b.re, im, 0, 0, 0);
}

// A wave's direction mu is a run-time value: one code path for the four directions.
// Upper half of (1 + sigma g_mu) psi = u + sigma B_mu l: for upper spin sp, B_mu takes the
// lower spin whose first component is lo[sp], times cr[sp] + i ci[sp], one of the two being
// zero (so the fmas below round once, as an add).
struct Direction {
  int mu, lo[2];
  double cr[2], ci[2];
  __device__ __forceinline__ explicit Direction(int m) : mu(m) {
    lo[0] = m < 2 ? 9 : 6;
    lo[1] = m < 2 ? 6 : 9;
    cr[0] = m == 1 ? -1.0 : (m == 3 ? 1.0 : 0.0);
    cr[1] = m == 1 || m == 3 ? 1.0 : 0.0;
    ci[0] = m == 0 || m == 2 ? 1.0 : 0.0;
    ci[1] = m == 0 ? 1.0 : (m == 2 ? -1.0 : 0.0);
  }
  template <int SIGMA>
  __device__ __forceinline__ cplx<double> half(int sp, double2 u, double2 l) const {
    const double r = SIGMA * cr[sp], i = SIGMA * ci[sp];
    return {fma(r, l.x, fma(-i, l.y, u.x)), fma(r, l.y, fma(i, l.x, u.y))};
  }
};

// Spin sp of the forward hop at one site, for the two slices of this lane: chi = U
// (1 - g_mu)-half of phi_k (ul: the spinors' two components per colour).  The link is the
// same for the whole wave.
__device__ __forceinline__ void rotate_spin(const Direction& d, int sp, const double2* __restrict__ lk, long long V4h,
                                            const double2 (&ul)[2][2][3], const bool (&in)[2],
                                            cplx<double> (&chi)[2][3]) {
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    cplx<double> hs[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) hs[c] = d.half<-1>(sp, ul[hf][0][c], ul[hf][1][c]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double2 u0 = lk[(3 * i + 0) * V4h], u1 = lk[(3 * i + 1) * V4h], u2 = lk[(3 * i + 2) * V4h];
      cplx<double> v = cmul(cplx<double>{u0.x, u0.y}, hs[0]);
      v = cfma(cplx<double>{u1.x, u1.y}, hs[1], v);
      v = cfma(cplx<double>{u2.x, u2.y}, hs[2], v);
      chi[hf][i] = in[hf] ? v : cplx<double>{0, 0};  // Ls no multiple of SL: idle slices count as zero
    }
  }
}

// acc += conj((1 + g_mu)-half of phi_j) chi, phi_j from LDS ([12][SL][stride], this lane's
// slice and vector at own)
template <int JT>
__device__ __forceinline__ void hop_steps(const Direction& d, int sp, const double2* own, int stride,
                                          const cplx<double> (&chi)[2][3], d4v (&re)[JT], d4v (&im)[JT]) {
  const double2* up = own + 3 * sp * SL * stride;
  const double2* lo = own + d.lo[sp] * SL * stride;
#pragma unroll
  for (int hf = 0; hf < 2; ++hf)
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int t = 0; t < JT; ++t) {
        const int o = (c * SL + 4 * hf) * stride + 16 * t;
        tile_step(d.half<+1>(sp, up[o], lo[o]), chi[hf][c], re[t], im[t]);
      }
}

__device__ __forceinline__ void put(double2* p, double re, double im) { *p = make_double2(re, im); }
__device__ __forceinline__ void put(float2* p, double re, double im) { *p = make_float2((float)re, (float)im); }

// Vectors come in groups of JT row tiles and KW column tiles, taken one after another;
// the block's own n x n matrix waits in LDS (X) for its conjugate transpose.
// Neighbouring blocks share an XCD.  NBUF = 2 buffers of staged vectors let a wave run
// a step ahead of the others; where they do not fit (JT = 3) one is used.
template <int JT, int KW, int NBUF, class E>
__global__ void __launch_bounds__(256 * KW) __attribute__((amdgpu_waves_per_eu(2)))
stencil_kernel(StencilArgs a, const double2* __restrict__ links, const int* __restrict__ bsite,
               const int* __restrict__ nbr, E* __restrict__ A) {
  extern __shared__ double2 smem[];
  constexpr int NJ = 16 * JT, STRIDE = NJ + 1;  // padded: the staging writes go down columns
  constexpr int BUF = 12 * SL * STRIDE;
  constexpr int PER = NJ * 12 * SL / (256 * KW);  // staged values per thread
  const int n = a.n, Ls = a.g.Ls;
  const long long V4h = a.g.V4h;
  double2* X = smem;  // [k][j]
  double2* st = smem + n * n;
  const int b = (blockIdx.x & 7) * a.nb8 + (blockIdx.x >> 3);
  if (b >= a.nb) return;  // whole workgroup leaves together
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int mu = wave & 3, kw = wave >> 2;
  const int col = lane & 15, q = lane >> 4;
  const int tiles = (n + 15) / 16;
  const int chunks = (Ls + SL - 1) / SL;
  const int nsteps = a.nsb * chunks;
  const Direction dir(mu);
  // local coordinate along mu of site i of the block: i / along % thick; a hop from the last
  // one leaves the block unless the block wraps round the lattice
  const int thick = a.blk[mu];
  const int along = (mu > 0 ? a.blk[0] : 1) * (mu > 1 ? a.blk[1] : 1) * (mu > 2 ? a.blk[2] : 1);
  const bool wraps = thick == (mu == 0 ? a.g.X : mu == 1 ? a.g.Y : mu == 2 ? a.g.Z : a.g.T);
  // A step: a site and its first slice.
  struct Step {
    int i, p, s0;
    long long h, nh;  // the site and its forward neighbour
    int face;
  };
  auto at_site = [&](int i) {
    Step w;
    w.i = i;
    w.s0 = 0;
    const long long e = __builtin_amdgcn_readfirstlane(bsite[(size_t)b * a.nsb + i]);
    w.p = e >= V4h ? 1 : 0;
    w.h = e - w.p * V4h;
    w.nh = __builtin_amdgcn_readfirstlane(nbr[((size_t)w.p * 8 + 2 * mu) * V4h + w.h]);
    w.face = !wraps && i / along % thick == thick - 1 ? 1 : 0;
    return w;
  };
  auto step_after = [&](Step w) {
    w.s0 += SL;
    return w.s0 < Ls ? w : at_site(w.i + 1);
  };
  const size_t nn = (size_t)n * n;
  E* Ab = A + (size_t)b * 9 * nn;

  for (int j0 = 0; j0 < tiles * 16; j0 += NJ)
    for (int k0 = 0; k0 < tiles * 16; k0 += 16 * KW) {
      const bool active = k0 + 16 * kw < n;  // uniform over the wave
      const int vk = min(k0 + 16 * kw + col, n - 1);  // lanes past the last vector repeat it and store nothing
      d4v fre[JT], fim[JT], ore[JT], oim[JT];
#pragma unroll
      for (int t = 0; t < JT; ++t) fre[t] = fim[t] = ore[t] = oim[t] = d4v{0, 0, 0, 0};
      // This thread's share of a step's own vectors: one slice (consecutive threads,
      // consecutive slices), vectors row % 16 + 16 t, every (2 KW)-th component
      double2 pre[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) pre[u] = make_double2(0, 0);
      const int s8 = threadIdx.x & (SL - 1), row = threadIdx.x / SL;
      const int fv = row & 15, fc = row >> 4;
      auto fetch = [&](const Step& w) {
        if (w.s0 + s8 >= Ls) return;  // an idle slice keeps the values of an earlier one, which meet zeros
#pragma unroll
        for (int t = 0; t < JT; ++t) {
          const char* f = a.basis + ((size_t)w.p * n + min(j0 + 16 * t + fv, n - 1)) * a.fb;
          const double2* o = reinterpret_cast<const double2*>(f) + (w.h * 12 + fc) * Ls + w.s0 + s8;
#pragma unroll
          for (int u = 0; u < PER / JT; ++u) pre[t * (PER / JT) + u] = o[2 * KW * u * Ls];
        }
      };
      auto mirrored = [&](int s0, int hf, bool& in) {
        const int s = s0 + 4 * hf + q;
        in = s < Ls;
        return in ? Ls - 1 - s : 0;
      };
      // the two components per colour of spin sp of the forward neighbour's phi_k, for this lane's two slices
      double2 ul[2][2][3];
      auto load_spin = [&](const Step& w, int sp) {
        const double2* f =
            reinterpret_cast<const double2*>(a.basis + ((size_t)(1 - w.p) * n + vk) * a.fb) + w.nh * 12 * Ls;
        const int lo = dir.lo[sp];
        bool unused;
        const int m0 = mirrored(w.s0, 0, unused), m1 = mirrored(w.s0, 1, unused);
#pragma unroll
        for (int c = 0; c < 3; ++c) {  // both slices of a line together
          ul[0][0][c] = f[(3 * sp + c) * Ls + m0];
          ul[1][0][c] = f[(3 * sp + c) * Ls + m1];
          ul[0][1][c] = f[(lo + c) * Ls + m0];
          ul[1][1][c] = f[(lo + c) * Ls + m1];
        }
      };
      Step cur = at_site(0), next = nsteps > 1 ? step_after(cur) : cur;
      fetch(cur);
      if (active) load_spin(cur, 0);
      for (int step = 0; step < nsteps; ++step) {
        const bool face = cur.face != 0;
        int sr[2];
        bool in[2];
        sr[0] = mirrored(cur.s0, 0, in[0]);
        sr[1] = mirrored(cur.s0, 1, in[1]);
        double2* buf = st + (NBUF == 2 ? (step & 1) * BUF : 0);
        {
          double2* o = buf + (fc * SL + s8) * STRIDE + fv;
#pragma unroll
          for (int t = 0; t < JT; ++t)
#pragma unroll
            for (int u = 0; u < PER / JT; ++u) o[2 * KW * u * SL * STRIDE + 16 * t] = pre[t * (PER / JT) + u];
        }
        __syncthreads();
        fetch(next);
        if (active) {
          const double2* own = buf + q * STRIDE + col;
          const double2* lk = links + ((size_t)(cur.p * 8 + 2 * mu) * 9) * V4h + cur.h;
          // a fetch always has a spin's products to hide behind
          cplx<double> chi[2][3];
          rotate_spin(dir, 0, lk, V4h, ul, in, chi);
          load_spin(cur, 1);
          if (face)
            hop_steps<JT>(dir, 0, own, STRIDE, chi, fre, fim);
          else
            hop_steps<JT>(dir, 0, own, STRIDE, chi, ore, oim);
          rotate_spin(dir, 1, lk, V4h, ul, in, chi);
          load_spin(next, 0);
          if (face)
            hop_steps<JT>(dir, 1, own, STRIDE, chi, fre, fim);
          else
            hop_steps<JT>(dir, 1, own, STRIDE, chi, ore, oim);
          // components 3 mu .. 3 mu + 2 of the site-local part -gamma_5 M5D phi_k at the mirrored
          // slice: (5 - M5) v_s - P_- v_{s+1} - P_+ v_{s-1}, the ends wrapping round with +mf
          // instead of -1; P_+ (upper spins) from below, P_- from above.  The block's tiles are
          // scaled by -1/2 and added to their conjugate transpose at the end: hence the sign.
          const double2* phik =
              reinterpret_cast<const double2*>(a.basis + ((size_t)cur.p * n + vk) * a.fb) + (cur.h * 12 + 3 * mu) * Ls;
          const bool upper = mu < 2;
          int s1[2];
          double c0[2], c1[2];
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            s1[hf] = upper ? (sr[hf] > 0 ? sr[hf] - 1 : Ls - 1) : (sr[hf] + 1 < Ls ? sr[hf] + 1 : 0);
            const bool wrap = upper ? sr[hf] == 0 : sr[hf] + 1 == Ls;
            const double sg = in[hf] ? (upper ? -1.0 : 1.0) : 0.0;
            c0[hf] = sg * a.d;
            c1[hf] = wrap ? sg * a.mf : -sg;
          }
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            double2 v0[2], v1[2];  // one line, but for the slice beyond its end
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
              v0[hf] = phik[k * Ls + sr[hf]];
              v1[hf] = phik[k * Ls + s1[hf]];
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
              const cplx<double> m = {c0[hf] * v0[hf].x + c1[hf] * v1[hf].x, c0[hf] * v0[hf].y + c1[hf] * v1[hf].y};
#pragma unroll
              for (int t = 0; t < JT; ++t) {
                const double2 f = own[((3 * mu + k) * SL + 4 * hf) * STRIDE + 16 * t];
                tile_step(cplx<double>{f.x, f.y}, m, ore[t], oim[t]);
              }
            }
          }
        }
        cur = next;
        if (step + 2 < nsteps) next = step_after(next);
        if (NBUF == 1) __syncthreads();
      }
      // register r of a tile: row j = lane / 16 + 4 r, column k = lane % 16
      const int k = k0 + 16 * kw + col;
      E* own = Ab + (size_t)(2 * mu) * nn;
      E* back = A + ((size_t)a.bnbr[(size_t)b * 8 + 2 * mu] * 9 + 2 * mu + 1) * nn;
#pragma unroll
      for (int t = 0; t < JT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = j0 + 16 * t + q + 4 * r;
          if (j < n && k < n) {
            put(own + (size_t)k * n + j, -0.5 * fre[t][r], -0.5 * fim[t][r]);
            put(back + (size_t)j * n + k, -0.5 * fre[t][r], 0.5 * fim[t][r]);
          }
        }
      for (int m = 0; m < 4; ++m) {  // the directions' parts of the block itself, added in order
        if (mu == m) {
#pragma unroll
          for (int t = 0; t < JT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int j = j0 + 16 * t + q + 4 * r;
              if (j < n && k < n) {
                double2 x = m ? X[(size_t)k * n + j] : make_double2(0, 0);
                X[(size_t)k * n + j] = make_double2(x.x - 0.5 * ore[t][r], x.y - 0.5 * oim[t][r]);
              }
            }
        }
        __syncthreads();
      }
    }
  for (int idx = threadIdx.x; idx < (int)nn; idx += 256 * KW) {
    const int k = idx / n, j = idx - k * n;
    const double2 x = X[idx], y = X[j * n + k];
    put(Ab + 8 * nn + idx, x.x + y.x, x.y - y.y);
  }
}

// The same for N = 1 or 2 vectors, whose products would leave a 16 x 16 tile all but empty: on the
// vector units, a lane per (site, s) of the block, bound by the loads' latency at the one or two
// waves a SIMD that its registers allow.  16^4, Ls 8, 2^4 blocks: one vector 102 us against 1.05 ms in
// a tile (and 0.54 ms with a field per stencil point, each restricted), two 0.52 against 1.03 (1.28);
// 4^4, where a block's chain of sites is all there is, 26 against 93 us (40) and 43 against 94 (65).
constexpr int FEW = 256;  // lanes

template <int N, class E>
__global__ void __launch_bounds__(FEW)
stencil_few_kernel(StencilArgs a, const double2* __restrict__ links, const int* __restrict__ bsite,
                   const int* __restrict__ nbr, E* __restrict__ A) {
  constexpr int NN = N * N, SUMS = 5 * NN;  // per (j, k): the four forward faces, the block itself
  __shared__ double2 red[FEW / 64][SUMS];
  const int b = (blockIdx.x & 7) * a.nb8 + (blockIdx.x >> 3);
  if (b >= a.nb) return;  // whole workgroup leaves together
  const int Ls = a.g.Ls;
  const long long V4h = a.g.V4h;
  const int ext[4] = {a.g.X, a.g.Y, a.g.Z, a.g.T};
  cplx<double> acc[SUMS];  // [point][j][k]
#pragma unroll
  for (int i = 0; i < SUMS; ++i) acc[i] = {0, 0};
  auto add = [](cplx<double> x, cplx<double> y, cplx<double>& s) {  // s += conj(x) y
    s.re = fma(x.re, y.re, fma(x.im, y.im, s.re));
    s.im = fma(x.re, y.im, fma(-x.im, y.re, s.im));
  };
  for (int p = threadIdx.x; p < a.nsb * Ls; p += FEW) {
    const int i = p / Ls, s = p - i * Ls, sr = Ls - 1 - s;
    const long long e = bsite[(size_t)b * a.nsb + i];
    const int par = e >= V4h ? 1 : 0;
    const long long h = e - par * V4h;
    auto field = [&](int q, int k, long long site) {
      return reinterpret_cast<const double2*>(a.basis + ((size_t)q * N + k) * a.fb) + site * 12 * Ls;
    };
    double2 own[N][12];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int c = 0; c < 12; ++c) own[j][c] = field(par, j, h)[c * Ls + s];
    // the forward hops from the mirrored slice, across a face or inside
    int along = 1;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      const Direction dir(mu);
      const bool face = a.blk[mu] != ext[mu] && i / along % a.blk[mu] == a.blk[mu] - 1;
      along *= a.blk[mu];
      const long long nh = nbr[((size_t)par * 8 + 2 * mu) * V4h + h];
      const double2* lk = links + ((size_t)(par * 8 + 2 * mu) * 9) * V4h + h;
      double2 u[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) u[c] = lk[c * V4h];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const double2* f = field(1 - par, k, nh);
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
          cplx<double> hs[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) hs[c] = dir.half<-1>(sp, f[(3 * sp + c) * Ls + sr], f[(dir.lo[sp] + c) * Ls + sr]);
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            cplx<double> chi = cmul(cplx<double>{u[3 * r].x, u[3 * r].y}, hs[0]);
            chi = cfma(cplx<double>{u[3 * r + 1].x, u[3 * r + 1].y}, hs[1], chi);
            chi = cfma(cplx<double>{u[3 * r + 2].x, u[3 * r + 2].y}, hs[2], chi);
#pragma unroll
            for (int j = 0; j < N; ++j) {
              const cplx<double> x = dir.half<+1>(sp, own[j][3 * sp + r], own[j][dir.lo[sp] + r]);
              if (face)
                add(x, chi, acc[mu * NN + j * N + k]);
              else
                add(x, chi, acc[4 * NN + j * N + k]);
            }
          }
        }
      }
    }
    // the site-local part at the mirrored slice, with the signs of stencil_kernel
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const bool upper = c < 6;
      const int s1 = upper ? (sr > 0 ? sr - 1 : Ls - 1) : (sr + 1 < Ls ? sr + 1 : 0);
      const bool wrap = upper ? sr == 0 : sr + 1 == Ls;
      const double sg = upper ? -1.0 : 1.0, c0 = sg * a.d, c1 = wrap ? sg * a.mf : -sg;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const double2 v0 = field(par, k, h)[c * Ls + sr], v1 = field(par, k, h)[c * Ls + s1];
        const cplx<double> m = {c0 * v0.x + c1 * v1.x, c0 * v0.y + c1 * v1.y};
#pragma unroll
        for (int j = 0; j < N; ++j) add(cplx<double>{own[j][c].x, own[j][c].y}, m, acc[4 * NN + j * N + k]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < SUMS; ++i) {
    const double re = wave_sum(acc[i].re), im = wave_sum(acc[i].im);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][i] = make_double2(re, im);
  }
  __syncthreads();
  if ((int)threadIdx.x >= SUMS) return;
  auto total = [&](int i) {  // the waves in order, times -1/2
    double2 t = red[0][i];
    for (int w = 1; w < FEW / 64; ++w) {
      t.x += red[w][i].x;
      t.y += red[w][i].y;
    }
    return make_double2(-0.5 * t.x, -0.5 * t.y);
  };
  const int point = threadIdx.x / NN, j = threadIdx.x % NN / N, k = threadIdx.x % N;
  const double2 t = total(threadIdx.x);
  E* Ab = A + (size_t)b * 9 * NN;
  if (point < 4) {
    put(Ab + 2 * point * NN + k * N + j, t.x, t.y);
    put(A + ((size_t)a.bnbr[(size_t)b * 8 + 2 * point] * 9 + 2 * point + 1) * NN + j * N + k, t.x, -t.y);
  } else {
    const double2 y = total(4 * NN + k * N + j);
    put(Ab + 8 * NN + k * N + j, t.x + y.x, t.y - y.y);
  }
}

template <int N, class E>
hipError_t launch_few(dwf_context* c, const StencilArgs& a, E* A) {
  hipLaunchKernelGGL((stencil_few_kernel<N, E>), dim3((unsigned)a.nb8 * 8), dim3(FEW), 0, c->stream, a,
                     reinterpret_cast<const double2*>(c->links64), c->bsite, c->nbr, A);
  return hipGetLastError();
}

template <int JT, int KW, int NBUF, class E>
hipError_t launch_s(dwf_context* c, const StencilArgs& a, E* A) {
  const size_t lds = ((size_t)a.n * a.n + (size_t)NBUF * 12 * SL * (16 * JT + 1)) * sizeof(double2);
  hipLaunchKernelGGL((stencil_kernel<JT, KW, NBUF, E>), dim3((unsigned)a.nb8 * 8), dim3(256 * KW), lds, c->stream, a,
                     reinterpret_cast<const double2*>(c->links64), c->bsite, c->nbr, A);
  return hipGetLastError();
}

// Row tiles per group: up to three, which the registers of two waves per SIMD hold but for the
// spills above; 49 to 64 vectors take two groups of two.  A tile is 16 x 16 whatever the number of
// vectors, so the time hardly falls below 16 of them (16^4, Ls 8, 4, 8 and 16 vectors 1.15, 1.20
// and 1.80 ms), and one and two vectors take the vector units.  LDS: 56, 117, 112 and 116 KB of a CU's 160 at
// n = 16, 32, 48 and 64.
template <class E>
hipError_t launch_t(dwf_context* c, const StencilArgs& a, E* A) {
  if (a.n == 1) return launch_few<1>(c, a, A);
  if (a.n == 2) return launch_few<2>(c, a, A);
  switch ((a.n + 15) / 16) {
    case 1: return launch_s<1, 1, 2>(c, a, A);
    case 2: return launch_s<2, 2, 2>(c, a, A);
    case 3: return launch_s<3, 2, 1>(c, a, A);
    default: return launch_s<2, 2, 1>(c, a, A);
  }
}

}  // namespace

hipError_t launch_stencil(dwf_context* c, const char* basis, int nvec, int prec, void* A) {
  StencilArgs a{};
  a.g = c->g;
  for (int i = 0; i < 4; ++i) a.blk[i] = c->blk[i];
  a.nsb = c->nsb;
  a.nb = c->nb;
  a.nb8 = (c->nb + 7) / 8;
  a.n = nvec;
  a.d = 5.0 - c->M5;
  a.mf = c->mf;
  a.bnbr = c->bnbr;
  a.basis = basis;
  a.fb = field_bytes_rhs(c, DWF_F64);
  return prec == DWF_F32 ? launch_t(c, a, reinterpret_cast<float2*>(A)) : launch_t(c, a, reinterpret_cast<double2*>(A));
}

}  // namespace dwf
