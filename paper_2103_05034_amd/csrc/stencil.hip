// The little Dirac operator of the two-level method (Two level preconditioner
// section): A^{ab}_{jk} = <phi_j^a | H_DW | phi_k^b> on a blocked basis, FP64, as
// the 9-point stencil [nb][9][n][n] with entry (j, k) at k * n + j (points as in
// dwf_hdcr_coarse_data).
//
// One workgroup forms one stencil point of one block as a matrix product over the
// block's 5D sites: rows j, columns k, in 16 x 16 tiles of the FP64 matrix cores.
// The operands come straight from the fields.  A lane holds one vector and one
// slice (16 vectors x 4 slices per wave), so it loads whole spinors, projects and
// rotates them in its registers, and every spin-colour component is then one
// step of the product's inner index; nothing is staged and no intermediate
// field is written.
//
// Two identities keep the work small.  Across a face the hop needs only half
// spinors: phi_j^dag gamma_5 (1 + sigma g_mu) chi = (u_j - sigma B l_j)^dag (u + sigma B l)_chi,
// six inner steps instead of twelve.  And H_DW is Hermitian, so the backward
// points are the conjugate transposes of the neighbouring blocks' forward ones:
// four face products and one for the block itself instead of nine.
//
// What bounds it: the fabric.  16^3 x 32, Ls 16, 32 vectors on 2^4 blocks is 0.41
// TFLOP (24 complex inner steps per 5D site, 6 ms of matrix core time) and takes
// 41.9 ms: the vectors of a workgroup's loads are 64-byte pieces of 128-byte lines
// that are gone from L1 and L2 when their other half is wanted, 2.2e9 line reads
// (285 GB, 6.3 TB/s) where 13 GB of basis are needed.  The form before this one
// wrote nine fields per basis vector and restricted each onto the whole basis,
// which read the basis five times per vector: 392 ms.
#include "dwf_internal.hpp"
#include "kernels.hpp"

namespace dwf {
namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int WAVES = 4;  // waves of a workgroup; each takes every fourth site of the block

struct StencilArgs {
  Geom g;
  int blk[4];
  int nsb, nb, nb8, n;
  int groups;           // tile groups along each of j and k
  double d, mf;         // 5 - M5, mass
  const double2* links; // [2][8][9][V4h]
  const int* nbr;       // [2][8][V4h]
  const int* bsite;     // [nb][nsb], odd sites as h + V4h
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

// chi = U (1 + sigma g_mu)-half of psi; the link is the same for the whole wave
template <int D>
__device__ __forceinline__ void rotated_half(const double2* __restrict__ lk, long long V4h, const cplx<double> psi[12],
                                             cplx<double> chi[6]) {
  constexpr int MU = D / 2;
  constexpr int SIGMA = (D % 2) ? +1 : -1;
  cplx<double> hs[6];
  project<MU, SIGMA>(psi, hs);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double2 u0 = lk[(size_t)(3 * i + 0) * V4h], u1 = lk[(size_t)(3 * i + 1) * V4h],
                  u2 = lk[(size_t)(3 * i + 2) * V4h];
#pragma unroll
    for (int sp = 0; sp < 2; ++sp) {
      cplx<double> v = cmul(cplx<double>{u0.x, u0.y}, hs[3 * sp + 0]);
      v = cfma(cplx<double>{u1.x, u1.y}, hs[3 * sp + 1], v);
      v = cfma(cplx<double>{u2.x, u2.y}, hs[3 * sp + 2], v);
      chi[3 * sp + i] = v;
    }
  }
}

// Component 3 sp + a of (1 + g_mu) psi's upper half, u + B_mu l, from u = component
// 3 sp + a and the lower component that B_mu pairs with it (project<MU, +1> one
// component at a time).
template <int MU>
__device__ __forceinline__ constexpr int lower_of(int c6) {
  return MU < 2 ? (c6 < 3 ? 9 + c6 : 3 + c6) : 6 + c6;
}
template <int MU>
__device__ __forceinline__ cplx<double> project_one(double2 u, double2 l, int c6) {
  const bool first = c6 < 3;
  if (MU == 0) return {u.x - l.y, u.y + l.x};                                                  // (i l1, i l0)
  if (MU == 1) return first ? cplx<double>{u.x - l.x, u.y - l.y} : cplx<double>{u.x + l.x, u.y + l.y};  // (-l1, l0)
  if (MU == 2) return first ? cplx<double>{u.x - l.y, u.y + l.x} : cplx<double>{u.x + l.y, u.y - l.x};  // (i l0, -i l1)
  return {u.x + l.x, u.y + l.y};                                                               // (l0, l1)
}

// Does hop direction D lead from coordinate c out of its block?
template <int D>
__device__ __forceinline__ bool leaves_block(const StencilArgs& a, const int c[4]) {
  constexpr int MU = D / 2;
  const int ext[4] = {a.g.X, a.g.Y, a.g.Z, a.g.T};
  const int cn = (D % 2) ? (c[MU] + ext[MU] - 1) % ext[MU] : (c[MU] + 1) % ext[MU];
  return cn / a.blk[MU] != c[MU] / a.blk[MU];
}

// Wave-uniform site i of block b: its half-lattice index, parity and coordinates.
__device__ __forceinline__ void block_site(const StencilArgs& a, int b, int i, long long& h, int& p, int c[4]) {
  long long e = __builtin_amdgcn_readfirstlane(a.bsite[(size_t)b * a.nsb + i]);
  p = e >= a.g.V4h ? 1 : 0;
  h = e - p * a.g.V4h;
  site_coords(a.g, p, h, c[0], c[1], c[2], c[3]);
}

__device__ __forceinline__ const char* half_of(const StencilArgs& a, int vec, int p) {
  return a.basis + ((size_t)p * a.n + vec) * a.fb;
}

// Forward face in direction MU: sum over the sites whose hop leaves the block of
// conj((1 + g_mu)-half of phi_j(x, s)) U (1 - g_mu)-half of phi_k(x + mu, Ls-1-s).
template <int MU, int T>
__device__ __forceinline__ void face_product(const StencilArgs& a, int b, const int (&vj)[T], const int (&vk)[T],
                                             d4v (&re)[T][T], d4v (&im)[T][T]) {
  const int q = (threadIdx.x & 63) >> 4;
  const int Ls = a.g.Ls;
  const long long V4h = a.g.V4h;
  for (int i = threadIdx.x >> 6; i < a.nsb; i += WAVES) {
    long long h;
    int p, c[4];
    block_site(a, b, __builtin_amdgcn_readfirstlane(i), h, p, c);
    if (!leaves_block<2 * MU>(a, c)) continue;
    const long long nh = __builtin_amdgcn_readfirstlane(a.nbr[((size_t)p * 8 + 2 * MU) * V4h + h]);
    const double2* lk = a.links + ((size_t)(p * 8 + 2 * MU) * 9) * V4h + h;
    for (int s0 = 0; s0 < Ls; s0 += 4) {
      const bool in = s0 + q < Ls;  // Ls not a multiple of four: the last step's idle slices count as zero
      const int s = in ? s0 + q : Ls - 1;
      cplx<double> hk[T][6];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        cplx<double> psi[12];
        Store<DWF_F64>::load(half_of(a, vk[t], 1 - p), V4h, Ls, nh, Ls - 1 - s, psi);
        rotated_half<2 * MU>(lk, V4h, psi, hk[t]);
      }
      const double2* pj[T];  // phi_j is read as its components are needed: holding it would cost a wave per SIMD
#pragma unroll
      for (int t = 0; t < T; ++t)
        pj[t] = reinterpret_cast<const double2*>(half_of(a, vj[t], p)) + h * 12 * Ls + s;
#pragma unroll
      for (int c6 = 0; c6 < 6; ++c6) {
#pragma unroll
        for (int t = 0; t < T; ++t)
          if (!in) hk[t][c6] = {0, 0};
#pragma unroll
        for (int tj = 0; tj < T; ++tj) {
          cplx<double> g = project_one<MU>(pj[tj][(size_t)c6 * Ls], pj[tj][(size_t)lower_of<MU>(c6) * Ls], c6);
          if (!in) g = {0, 0};
#pragma unroll
          for (int tk = 0; tk < T; ++tk) tile_step(g, hk[tk][c6], re[tj][tk], im[tj][tk]);
        }
      }
    }
  }
}

// -D_hop term of direction D added to `in` where it stays inside the block
template <int D>
__device__ __forceinline__ void inside_term(const StencilArgs& a, int vec, int p, long long h, int sr, const int c[4],
                                            cplx<double> in[12]) {
  if (leaves_block<D>(a, c)) return;
  constexpr int MU = D / 2;
  constexpr int SIGMA = (D % 2) ? +1 : -1;
  const long long V4h = a.g.V4h;
  const long long nh = __builtin_amdgcn_readfirstlane(a.nbr[((size_t)p * 8 + D) * V4h + h]);
  cplx<double> psi[12], chi[6];
  Store<DWF_F64>::load(half_of(a, vec, 1 - p), V4h, a.g.Ls, nh, sr, psi);
  rotated_half<D>(a.links + ((size_t)(p * 8 + D) * 9) * V4h + h, V4h, psi, chi);
  reconstruct<MU, SIGMA>(chi, in);
}

// The block itself: conj(phi_j(x, s)) gamma_5 [M5D phi_k - D_hop^{inside} phi_k / 2](x, Ls-1-s).
template <int T>
__device__ __forceinline__ void block_product(const StencilArgs& a, int b, const int (&vj)[T], const int (&vk)[T],
                                              d4v (&re)[T][T], d4v (&im)[T][T]) {
  const int q = (threadIdx.x & 63) >> 4;
  const int Ls = a.g.Ls;
  const long long V4h = a.g.V4h;
  for (int i = threadIdx.x >> 6; i < a.nsb; i += WAVES) {
    long long h;
    int p, c[4];
    block_site(a, b, __builtin_amdgcn_readfirstlane(i), h, p, c);
    for (int s0 = 0; s0 < Ls; s0 += 4) {
      const bool in = s0 + q < Ls;
      const int s = in ? s0 + q : Ls - 1;
      const int sr = Ls - 1 - s;
      // M5D at the mirrored slice: (5 - M5) v_s - P_- v_{s+1} - P_+ v_{s-1}, the
      // ends wrapping round with +mf instead of -1
      const int su = sr + 1 < Ls ? sr + 1 : 0, sd = sr > 0 ? sr - 1 : Ls - 1;
      const double cu = sr + 1 < Ls ? -1.0 : a.mf, cd = sr > 0 ? -1.0 : a.mf;
      const double2* pj[T];  // phi_j is read as its components are needed: holding it would cost a wave per SIMD
#pragma unroll
      for (int t = 0; t < T; ++t)
        pj[t] = reinterpret_cast<const double2*>(half_of(a, vj[t], p)) + h * 12 * Ls + s;
#pragma unroll
      for (int tk = 0; tk < T; ++tk) {
        cplx<double> hop[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) hop[k] = {0, 0};
        inside_term<0>(a, vk[tk], p, h, sr, c, hop);
        inside_term<1>(a, vk[tk], p, h, sr, c, hop);
        inside_term<2>(a, vk[tk], p, h, sr, c, hop);
        inside_term<3>(a, vk[tk], p, h, sr, c, hop);
        inside_term<4>(a, vk[tk], p, h, sr, c, hop);
        inside_term<5>(a, vk[tk], p, h, sr, c, hop);
        inside_term<6>(a, vk[tk], p, h, sr, c, hop);
        inside_term<7>(a, vk[tk], p, h, sr, c, hop);
        __builtin_amdgcn_sched_barrier(0);  // the loads below, moved up, would not fit the registers
        const double2* own = reinterpret_cast<const double2*>(half_of(a, vk[tk], p)) + h * 12 * Ls;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
          const double2 v0 = own[(size_t)k * Ls + sr];
          const double2 v1 = own[(size_t)k * Ls + (k < 6 ? sd : su)];  // P_+ (upper spins) from below, P_- from above
          const double c1 = k < 6 ? cd : cu;
          cplx<double> m = {a.d * v0.x, a.d * v0.y};
          m.re += c1 * v1.x;
          m.im += c1 * v1.y;
          m.re -= 0.5 * hop[k].re;
          m.im -= 0.5 * hop[k].im;
          const double sg = k < 6 ? 1.0 : -1.0;
          m = {sg * m.re, sg * m.im};
          if (!in) m = {0, 0};
#pragma unroll
          for (int tj = 0; tj < T; ++tj) {
            const double2 f = pj[tj][(size_t)k * Ls];
            tile_step(in ? cplx<double>{f.x, f.y} : cplx<double>{0, 0}, m, re[tj][tk], im[tj][tk]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

__device__ __forceinline__ void put(double2* p, double re, double im) { *p = make_double2(re, im); }
__device__ __forceinline__ void put(float2* p, double re, double im) { *p = make_float2((float)re, (float)im); }

// The workgroups of a block's five products follow each other on one XCD, so the
// block's vectors are fetched into its L2 once; neighbouring blocks share an XCD.
// The waves' sums are added in wave order through LDS.
template <int T, class E>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(T == 3 ? 1 : 2)))
stencil_kernel(StencilArgs a, E* __restrict__ A) {
  __shared__ double red[WAVES][8][64];
  const int slot = blockIdx.x >> 3;
  const int point = slot % 5;  // 0..3 the forward faces, 4 the block itself
  const int b = (blockIdx.x & 7) * a.nb8 + slot / 5;
  if (b >= a.nb) return;  // whole workgroup leaves together
  const int gj = blockIdx.y % a.groups, gk = blockIdx.y / a.groups;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int vj[T], vk[T];  // vectors of this lane; lanes past the last vector repeat it and store nothing
#pragma unroll
  for (int t = 0; t < T; ++t) {
    vj[t] = min((gj * T + t) * 16 + (lane & 15), a.n - 1);
    vk[t] = min((gk * T + t) * 16 + (lane & 15), a.n - 1);
  }
  d4v re[T][T], im[T][T];
#pragma unroll
  for (int tj = 0; tj < T; ++tj)
#pragma unroll
    for (int tk = 0; tk < T; ++tk) re[tj][tk] = im[tj][tk] = d4v{0, 0, 0, 0};
  switch (point) {
    case 0: face_product<0, T>(a, b, vj, vk, re, im); break;
    case 1: face_product<1, T>(a, b, vj, vk, re, im); break;
    case 2: face_product<2, T>(a, b, vj, vk, re, im); break;
    case 3: face_product<3, T>(a, b, vj, vk, re, im); break;
    default: block_product<T>(a, b, vj, vk, re, im); break;
  }
  const size_t nn = (size_t)a.n * a.n;
  const double w = point < 4 ? -0.5 : 1.0;
  E* own = A + ((size_t)b * 9 + (point < 4 ? 2 * point : 8)) * nn;
  E* back = point < 4 ? A + ((size_t)a.bnbr[(size_t)b * 8 + 2 * point] * 9 + 2 * point + 1) * nn : nullptr;
#pragma unroll
  for (int tj = 0; tj < T; ++tj)
#pragma unroll
    for (int tk = 0; tk < T; ++tk) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        red[wave][r][lane] = re[tj][tk][r];
        red[wave][4 + r][lane] = im[tj][tk][r];
      }
      __syncthreads();
      // thread (r, lane) of the tile: row j = lane / 16 + 4 r, column k = lane % 16
      const int r = wave;
      double sr = 0, si = 0;
#pragma unroll
      for (int v = 0; v < WAVES; ++v) {
        sr += red[v][r][lane];
        si += red[v][4 + r][lane];
      }
      const int j = (gj * T + tj) * 16 + (lane >> 4) + 4 * r;
      const int k = (gk * T + tk) * 16 + (lane & 15);
      if (j < a.n && k < a.n) {
        put(own + (size_t)k * a.n + j, w * sr, w * si);
        if (back) put(back + (size_t)j * a.n + k, w * sr, -(w * si));
      }
    }
}

template <class E>
hipError_t launch_t(dwf_context* c, StencilArgs& a, E* A) {
  // one group of T x T tiles holds up to 48 vectors in registers; 49 to 64 take four groups of 2 x 2
  const int tiles = (a.n + 15) / 16;
  const int T = tiles == 4 ? 2 : tiles;
  a.groups = (tiles + T - 1) / T;
  const dim3 grid((unsigned)a.nb8 * 8 * 5, (unsigned)(a.groups * a.groups)), block(64 * WAVES);
  switch (T) {
    case 1: hipLaunchKernelGGL((stencil_kernel<1, E>), grid, block, 0, c->stream, a, A); break;
    case 2: hipLaunchKernelGGL((stencil_kernel<2, E>), grid, block, 0, c->stream, a, A); break;
    default: hipLaunchKernelGGL((stencil_kernel<3, E>), grid, block, 0, c->stream, a, A); break;
  }
  return hipGetLastError();
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
  a.links = reinterpret_cast<const double2*>(c->links64);
  a.nbr = c->nbr;
  a.bsite = c->bsite;
  a.bnbr = c->bnbr;
  a.basis = basis;
  a.fb = field_bytes_rhs(c, DWF_F64);
  return prec == DWF_F32 ? launch_t(c, a, reinterpret_cast<float2*>(A)) : launch_t(c, a, reinterpret_cast<double2*>(A));
}

}  // namespace dwf
