// ov_kernels.hpp -- HIP kernels of the overlap hot path (gfx950).
//
// Every kernel works on a *batch* of systems: one system is one right-hand
// side on one lattice.  A launch covers sum_s nblk_s workgroups; workgroup b
// is remapped XCD-contiguously to a logical block L, which belongs to system
// s with sys[s].blk0 <= L < sys[s].blk0 + sys[s].nblk.  Systems may live on
// lattices of different sizes (uneven batches) and carry their own scalars,
// iteration counts and convergence flags.
//
// Multi-shift CG, Krylov-basis form.  For (H^2 + b_k) y_k = psi the shifted
// solutions are linear combinations of the base residuals r_j, with scalar
// coefficients that follow from the base CG scalars alone (Jegerlehner's
// recurrences).  The pole sum needed by the sign function is
//     eps = H sum_k a_k y_k = sum_j d_j t_j,   t_j = H P_j,
// so one pass of the base CG on H^2 that keeps every t_j (HBM is 288 GB) plus
// one combination pass replaces the n_poles shifted search directions of the
// textbook algorithm.  Per iteration only two vectors are read and one written
// in each of the two stencil kernels:
//     k_ms_t:  t_n = H r_n + beta_{n-1} t_{n-1}         (= H P_n, P never stored)
//     k_ms_r:  r_{n+1} = r_n - alpha_n H t_n
// The scalar reductions are finished redundantly by every workgroup of the
// next kernel (fixed summation order -> identical bits in every workgroup), so
// no grid barrier, atomic or host round trip is needed inside an iteration.
#pragma once

#include "ov_common.hpp"

namespace ov {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int MAXP = 32;      // max poles
constexpr int NTHREADS = 256; // default workgroup size (4 waves)

// Device descriptor of one system for one phase of a solve.
struct SysDev {
  Geo g;
  int nblk;    // workgroups of this system in a launch
  int blk0;    // first logical workgroup
  int spb;     // sites per workgroup
  int pad0;
  int* active;              // host-controlled on/off flag (batched solves); may be null
  // multi-shift
  void* basis;              // t_j slots, slot stride 4V complex
  void* r;                  // r_n, n >= 1
  const void* src;          // r_0
  double* part_a;           // [nblk] |t_n|^2 partials
  double* part_b;           // [nblk] |r_n|^2 partials (source partials for n = 0)
  double* h_rho;            // [cap+1]
  double* h_alpha;          // [cap+1]
  double* h_zeta;           // [(cap+1) * MAXP]
  unsigned int* h_active;   // [cap+1] shift masks
  int* h_ctl;               // [4]: done, n_done, status, sticky error (host-reset)
  long long* stat;          // [4]: inner iterations, multi-shift solves, max N, max N of the
                            //      current outer iteration (cleared by k_cg_p)
  double* dstat;            // [2]: max shift residual of the last multi-shift, (unused)
  double* coef_term;        // [MAXP * cap]
  double* coef_c;           // [cap+1]
  double* coef_d;           // [cap]
  double* coef_d2;          // [cap] non-null: also the coefficients of H r(A)^2 psi (k_ms_coef)
  double* coef_sq;          // [(2 MAXP + 2) cap] scratch of those coefficients
  // epilogue / CG
  const double2* phi;       // [V] background scalar
  const void* e_in;         // operator input psi (spin-planar, kernel precision)
  void* e_out;              // operator output
  void* e_out2;             // optional g5 * output (next multi-shift source)
  double* part_c;           // [nblk] partials of |e_out|^2 or |r|^2
  void* cg_x;               // CG vectors (kernel precision)
  void* cg_p;
  void* cg_r;
  void* cg_z;               // preconditioned residual z = P r (PCG); null: z = r
  const double2* cg_b;      // FP64 right-hand side (true residual)
  void* cg_r64;             // FP64 true residual out
  void* cg_x64;             // FP64 solution (reliable updates)
  double* cg_s;             // per-system CG scalars (see CG_* below)
  double m_re, m_im;        // fermion mass
  double pc_re, pc_im;      // mass of the preconditioner M0 (m, or the RMS of c = m + g phi)
  double shift;             // sigma of a shifted solve (MdagM + sigma) x = b; 0 otherwise
  double g_re, g_im;        // Yukawa coupling
  double2* shx;             // multi-shift CG on MdagM: nshift solutions (FP64 planar)
  double2* shp;             //   and nshift search directions
  const double* shc;        //   per-shift coefficients (SHC_* layout)
  int nshift;
  void* fft_tmp;            // momentum-space scratch field (kernel precision)
  int off_xy, off_z, off_t, off_zt; // first workgroup of this system in each transform pass
  int xc;                   // x values per workgroup in the t pass (divides X, xc T <= 256)
  double* pcs;              // [V] preconditioner scale per momentum (k_pcg_table), or null
  // the caller's fields (complex128, spin innermost) and their planar twins of a call:
  // k_pack io_in -> io_pin, k_unpack io_pout -> io_out
  const double2* io_in;
  void* io_pin;
  void* io_pout;
  double2* io_out;
  int src_io;               // resident multi-shift source: 1 io_in, 2 g5 io_in (0: src)
};

// CG scalar slots
// CG_RR holds rho = <r, z> (= |r|^2 without a preconditioner); CG_R2 holds |r|^2 of
// the preconditioned recursion.
enum { CG_RR = 0, CG_RR_OLD, CG_PAP, CG_ALPHA, CG_BETA, CG_BB, CG_RTRUE, CG_R2, CG_NSLOT = 8 };

struct MsParams {
  int np;               // poles
  int cap;              // basis capacity (max iterations)
  double tol;           // shift tolerance
  double diag;          // 4 - M0
  double sigma[MAXP];   // shifts b_k
  double coef[MAXP];    // residues a_k
  int zm;               // > 0: z-marching passes over zm planes per workgroup (ZmMarch)
  int share;            // the XCDs share every system (xcd_share), not the launch
  int nt;               // t_n and r_{n+1} are stored past the caches (launch_ms_tab)
  unsigned long long* tstamp;  // non-null: per workgroup (start, end, sites) stamps
};

__device__ __forceinline__ int find_sys(const SysDev* __restrict__ sys, int nsys, int L) {
  int s = 0;
  for (int k = 1; k < nsys; ++k)
    if (sys[k].blk0 <= L) s = k;
  return s;
}

// ------------------------------------------------------------------ pack
// The caller's complex128 (V, 4) <-> spin-planar R.
template <class R>
__global__ void k_pack(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                       int nb_total) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int V = S.g.V;
  const int lb = L - S.blk0;
  const double2* in = S.io_in;
  c2<R>* out = (c2<R>*)S.io_pin;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 v = in[(size_t)i * 4 + k];
      out[(size_t)k * V + i] = c2<R>{(R)v.x, (R)v.y};
    }
  }
}

template <class R>
__global__ void k_unpack(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                         int nb_total) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int V = S.g.V;
  const int lb = L - S.blk0;
  const c2<R>* in = (const c2<R>*)S.io_pout;
  double2* out = S.io_out;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const c2<R> v = in[(size_t)k * V + i];
      out[(size_t)i * 4 + k] = double2{(double)v.x, (double)v.y};
    }
  }
}

// out = a * in over n complex128 values (ABI layout).
__global__ void k_scale_copy(double2* __restrict__ out, const double2* __restrict__ in, double a,
                             size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const double2 v = in[i];
    out[i] = double2{a * v.x, a * v.y};
  }
}

// io_out += a io_pout: planar FP64 added into the caller's field.
__global__ void k_unpack_axpy(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                              int nb_total, double a) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int V = S.g.V;
  const int lb = L - S.blk0;
  const double2* in = (const double2*)S.io_pout;
  double2* out = S.io_out;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 v = in[(size_t)k * V + i];
      double2& o = out[(size_t)i * 4 + k];
      o = double2{o.x + a * v.x, o.y + a * v.y};
    }
  }
}

// ---------------------------------------------------------- plain stencil
// out = H_W in; optional |out|^2 partials.  in/out per system from e_in/e_out.
template <class R>
__global__ void __launch_bounds__(256) k_hw(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                             int nb_total, double diag, int want_norm) {
  __shared__ double lds[17];
  const int L = xcd_logical_block(nb_total);
  const int s = bmap[L];
  const SysDev& S = sys[s];
  const Geo g = S.g;
  const int lb = L - S.blk0;
  const c2<R>* in = (const c2<R>*)S.e_in;
  c2<R>* out = (c2<R>*)S.e_out;
  const int i0 = lb * S.spb;
  const int i1 = min(g.V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    c2<R> o[4];
    hw_site<R>(in, g, i, (R)diag, o);
    store_sp<R>(out, g.V, i, o);
    if (want_norm) acc += norm2_sp(o);
  }
  if (want_norm) {
    const double tot = block_sum(acc, lds);
    if (threadIdx.x == 0) S.part_c[lb] = tot;
  }
}

// out = H_W in with the block's own sites staged in LDS: a block of spb
// consecutive sites covers whole x rows (and, at 16^4 with 256 sites, a whole
// xy plane), so its x and y neighbours are read from LDS and only the centre
// and the z and t neighbours come through the vector cache (5 of 9 spinor
// loads).  Neighbours outside the block fall back to global loads.
// Dynamic LDS: 4 * spb complex values.
template <class R>
__device__ __forceinline__ void nb_lds(const c2<R>* __restrict__ f, const c2<R>* sh, int V, int spb,
                                       int i0, int i1, int j, c2<R> v[4]) {
  if (j >= i0 && j < i1) {
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = sh[s * spb + (j - i0)];
  } else {
    load_sp<R>(f, V, j, v);
  }
}

template <class R>
__device__ __forceinline__ void load_nbr_staged(const c2<R>* __restrict__ f, const Geo& g, int i,
                                                const c2<R>* sh, int spb, int i0, int i1,
                                                Nbr<R>& nb) {
  const int X = g.X, Y = g.Y, Z = g.Z, T = g.T, V = g.V;
  int r = i;
  const int x = r % X; r /= X;
  const int y = r % Y; r /= Y;
  const int z = r % Z;
  const int t = r / Z;
  const int XY = X * Y, XYZ = XY * Z;
  load_sp<R>(f, V, (z + 1 < Z) ? i + XY : i + XY - XYZ, nb.zf);
  load_sp<R>(f, V, (z > 0) ? i - XY : i - XY + XYZ, nb.zb);
  load_sp<R>(f, V, (t + 1 < T) ? i + XYZ : i + XYZ - V, nb.tf);
  load_sp<R>(f, V, (t > 0) ? i - XYZ : i - XYZ + V, nb.tb);
#pragma unroll
  for (int s = 0; s < 4; ++s) nb.c[s] = sh[s * spb + (i - i0)];
  nb_lds<R>(f, sh, V, spb, i0, i1, (x + 1 < X) ? i + 1 : i + 1 - X, nb.xf);
  nb_lds<R>(f, sh, V, spb, i0, i1, (x > 0) ? i - 1 : i - 1 + X, nb.xb);
  nb_lds<R>(f, sh, V, spb, i0, i1, (y + 1 < Y) ? i + X : i + X - XY, nb.yf);
  nb_lds<R>(f, sh, V, spb, i0, i1, (y > 0) ? i - X : i - X + XY, nb.yb);
}

// Stage the block's sites [i0, i1) of f into sh (planar, 4 * spb values).
template <class R>
__device__ __forceinline__ void stage_block(const c2<R>* __restrict__ f, int V, int spb, int i0,
                                            int i1, c2<R>* sh) {
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
#pragma unroll
    for (int s = 0; s < 4; ++s) sh[s * spb + (i - i0)] = f[(size_t)s * V + i];
  }
  __syncthreads();
}

template <class R>
__global__ void __launch_bounds__(256) k_hw_lds(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                 int nb_total, double diag) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  c2<R>* sh = (c2<R>*)dyn_lds;
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const Geo g = S.g;
  const int lb = L - S.blk0;
  const c2<R>* in = (const c2<R>*)S.e_in;
  c2<R>* out = (c2<R>*)S.e_out;
  const int spb = S.spb;
  const int i0 = lb * spb;
  const int i1 = min(g.V, i0 + spb);
  stage_block<R>(in, g.V, spb, i0, i1, sh);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    Nbr<R> nb;
    load_nbr_staged<R>(in, g, i, sh, spb, i0, i1, nb);
    c2<R> o[4];
    hw_compute<R>(nb, g, i, (R)diag, o);
    store_sp<R>(out, g.V, i, o);
  }
}

// out = H_W in, z-marching form: a workgroup owns one xy plane (X Y <= 256
// sites, one per thread) of one time slice and walks ZC consecutive z planes.
// The z neighbours stay in registers (the plane below, the current one, the
// plane above), the x and y neighbours come from the current plane staged in
// LDS, so each output site reads (ZC + 2)/ZC centre spinors plus its two time
// neighbours from the memory hierarchy instead of nine spinors.  Every system
// of the table has the same lattice.  Grid: nsys * T * (Z / ZC) workgroups.
// Streaming store of a site's spinor: marked non-temporal so that the output lines do
// not push the input planes, which neighbouring workgroups still read, out of L2.
template <class R>
__device__ __forceinline__ void store_sp_nt(c2<R>* __restrict__ f, int V, int i, const c2<R> v[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const ev2<R> e = {v[s].x, v[s].y};
    __builtin_nontemporal_store(e, (OV_GLOBAL ev2<R>*)(f + (size_t)s * V + i));
  }
}

// The multi-shift passes' stores: the next pass reads them, from the caches if they can hold them.
template <class R>
__device__ __forceinline__ void store_ms(int nt, c2<R>* __restrict__ f, int V, int i, const c2<R> v[4]) {
  if (nt)
    store_sp_nt<R>(f, V, i, v);
  else
    store_sp<R>(f, V, i, v);
}

template <class R, int ZC>
__global__ void __launch_bounds__(256) k_hw_zm(const SysDev* __restrict__ sys, double diag) {
  __shared__ c2<R> sh[4 * 256];
  const Geo g = sys[0].g;
  const int X = g.X, Y = g.Y, Z = g.Z, T = g.T, V = g.V;
  const int XY = X * Y, XYZ = XY * Z;
  const int nzc = Z / ZC;
  // XCD-contiguous order: the workgroups of neighbouring time slices share an L2,
  // which then serves the time-neighbour reads.  FP64 takes the time slices fastest
  // (time neighbours in consecutive workgroups, loaded together: 48 fields at 16^4 read
  // 1.14x instead of 1.23x the algorithmic bytes, 5.14 -> 5.43 TB/s); FP32, with more
  // workgroups resident, reuses them as well with the z chunks fastest (1.04x; 1.09x
  // the other way round).
  const int b = xcd_logical_block(gridDim.x);
  const int s = b / (T * nzc);
  constexpr bool t_fast = sizeof(R) == sizeof(double);
  const int t = t_fast ? b % T : (b / nzc) % T;
  const int z0 = (t_fast ? (b / T) % nzc : b % nzc) * ZC;
  const SysDev& S = sys[s];
  const c2<R>* in = (const c2<R>*)S.e_in;
  c2<R>* out = (c2<R>*)S.e_out;
  const int j = threadIdx.x;
  const bool on = j < XY;
  const int x = on ? j % X : 0, y = on ? j / X : 0;
  const int tf_off = (t + 1 < T) ? XYZ : XYZ - V;
  const int tb_off = (t > 0) ? -XYZ : V - XYZ;
  const int jxf = y * X + ((x + 1 < X) ? x + 1 : 0);
  const int jxb = y * X + ((x > 0) ? x - 1 : X - 1);
  const int jyf = ((y + 1 < Y) ? y + 1 : 0) * X + x;
  const int jyb = ((y > 0) ? y - 1 : Y - 1) * X + x;
  auto site = [&](int z) { return j + XY * (z + Z * t); };
  auto zwrap = [&](int z) { return z < 0 ? z + Z : (z >= Z ? z - Z : z); };
  // software pipeline: the plane above and the time neighbours of the next plane
  // are loaded one step ahead
  c2<R> prev[4], cur[4], next[4], tf[4], tb[4];
  if (on) {
    load_sp<R>(in, V, site(zwrap(z0 - 1)), prev);
    load_sp<R>(in, V, site(z0), cur);
    load_sp<R>(in, V, site(zwrap(z0 + 1)), next);
    load_sp<R>(in, V, site(z0) + tf_off, tf);
    load_sp<R>(in, V, site(z0) + tb_off, tb);
  }
#pragma unroll
  for (int zi = 0; zi < ZC; ++zi) {
    const int z = z0 + zi;
    const int i = site(z);
    c2<R> next2[4], tf2[4], tb2[4];
    if (on && zi + 1 < ZC) {
      load_sp<R>(in, V, site(zwrap(z + 2)), next2);
      load_sp<R>(in, V, site(z + 1) + tf_off, tf2);
      load_sp<R>(in, V, site(z + 1) + tb_off, tb2);
    }
    __syncthreads();  // the previous plane's LDS reads are done
    if (on) {
#pragma unroll
      for (int q = 0; q < 4; ++q) sh[q * 256 + j] = cur[q];
    }
    __syncthreads();
    if (on) {
      Nbr<R> nb;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        nb.c[q] = cur[q];
        nb.xf[q] = sh[q * 256 + jxf];
        nb.xb[q] = sh[q * 256 + jxb];
        nb.yf[q] = sh[q * 256 + jyf];
        nb.yb[q] = sh[q * 256 + jyb];
        nb.zf[q] = next[q];
        nb.zb[q] = prev[q];
        nb.tf[q] = tf[q];
        nb.tb[q] = tb[q];
      }
      c2<R> o[4];
      hw_compute<R>(nb, g, i, (R)diag, o);
      store_sp_nt<R>(out, V, i, o);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        prev[q] = cur[q];
        cur[q] = next[q];
        next[q] = next2[q];
        tf[q] = tf2[q];
        tb[q] = tb2[q];
      }
    }
  }
}

// ---------------------------------------------------- H_W on the caller's fields
// io_out = H_W io_in on complex128 fields with the spin innermost (ov_apply OV_OP_HW): the
// stencil reads and writes the caller's layout itself, one pass over memory instead of
// pack, stencil and unpack.  A site is 64 contiguous bytes, so a wave's four loads of a
// component each share their cache lines.  Bound by memory: 128 bytes per site; 48 fields of
// 16^4 take 80 us (5.0 TB/s; pack, k_hw and unpack took 92 + 127 + 155).
__device__ __forceinline__ void load_io(const double2* __restrict__ f, int i, double2 v[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) v[s] = ldg2<double>(f, (size_t)i * 4 + s);
}

// Any lattice: one site per thread, nine spinors through the caches.
__global__ void __launch_bounds__(256) k_hw_io(const SysDev* __restrict__ sys,
                                               const int* __restrict__ bmap, int nb_total,
                                               double diag) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const Geo g = S.g;
  const int lb = L - S.blk0;
  const double2* in = S.io_in;
  double2* out = S.io_out;
  const int XY = g.X * g.Y, XYZ = XY * g.Z;
  const int i0 = lb * S.spb;
  const int i1 = min(g.V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    int r = i;
    const int x = r % g.X; r /= g.X;
    const int y = r % g.Y; r /= g.Y;
    const int z = r % g.Z;
    const int t = r / g.Z;
    Nbr<double> nb;
    load_io(in, i, nb.c);
    load_io(in, (x + 1 < g.X) ? i + 1 : i + 1 - g.X, nb.xf);
    load_io(in, (x > 0) ? i - 1 : i - 1 + g.X, nb.xb);
    load_io(in, (y + 1 < g.Y) ? i + g.X : i + g.X - XY, nb.yf);
    load_io(in, (y > 0) ? i - g.X : i - g.X + XY, nb.yb);
    load_io(in, (z + 1 < g.Z) ? i + XY : i + XY - XYZ, nb.zf);
    load_io(in, (z > 0) ? i - XY : i - XY + XYZ, nb.zb);
    load_io(in, (t + 1 < g.T) ? i + XYZ : i + XYZ - g.V, nb.tf);
    load_io(in, (t > 0) ? i - XYZ : i - XYZ + g.V, nb.tb);
    double2 o[4];
    hw_compute<double>(nb, g, i, diag, o);
#pragma unroll
    for (int k = 0; k < 4; ++k) stg2<double>(out, (size_t)i * 4 + k, o[k]);
  }
}

// z-marching form (k_hw_zm): xy planes of at most 256 sites, ZC planes per workgroup, every
// system on one lattice.  The results of a plane go through LDS, so that a wave stores
// whole lines.
template <int ZC>
__global__ void __launch_bounds__(256) k_hw_io_zm(const SysDev* __restrict__ sys, double diag) {
  constexpr int P = 257;  // plane pitch: the transposed reads of a site fall on four banks
  __shared__ double2 sh[4 * P];
  const Geo g = sys[0].g;
  const int X = g.X, Y = g.Y, Z = g.Z, T = g.T, V = g.V;
  const int XY = X * Y, XYZ = XY * Z;
  const int nzc = Z / ZC;
  const int b = xcd_logical_block(gridDim.x);
  const SysDev& S = sys[b / (T * nzc)];
  const int t = b % T;  // time slices fastest, as in k_hw_zm in FP64
  const int z0 = ((b / T) % nzc) * ZC;
  const double2* in = S.io_in;
  double2* out = S.io_out;
  const int j = threadIdx.x;
  const bool on = j < XY;
  const int x = on ? j % X : 0, y = on ? j / X : 0;
  const int tf_off = (t + 1 < T) ? XYZ : XYZ - V;
  const int tb_off = (t > 0) ? -XYZ : V - XYZ;
  const int jxf = y * X + ((x + 1 < X) ? x + 1 : 0);
  const int jxb = y * X + ((x > 0) ? x - 1 : X - 1);
  const int jyf = ((y + 1 < Y) ? y + 1 : 0) * X + x;
  const int jyb = ((y > 0) ? y - 1 : Y - 1) * X + x;
  auto site = [&](int z) { return j + XY * ((z < 0 ? z + Z : (z >= Z ? z - Z : z)) + Z * t); };
  Nbr<double> nb;
  double2 next2[4], tf2[4], tb2[4];
  if (on) {
    load_io(in, site(z0 - 1), nb.zb);
    load_io(in, site(z0), nb.c);
    load_io(in, site(z0 + 1), nb.zf);
    load_io(in, site(z0) + tf_off, nb.tf);
    load_io(in, site(z0) + tb_off, nb.tb);
  }
#pragma unroll
  for (int zi = 0; zi < ZC; ++zi) {
    const int z = z0 + zi;
    if (on && zi + 1 < ZC) {
      load_io(in, site(z + 2), next2);
      load_io(in, site(z + 1) + tf_off, tf2);
      load_io(in, site(z + 1) + tb_off, tb2);
    }
    if (zi > 0) __syncthreads();  // the previous plane's results have been stored
    if (on) {
#pragma unroll
      for (int q = 0; q < 4; ++q) sh[q * P + j] = nb.c[q];
    }
    __syncthreads();
    double2 o[4];
    if (on) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        nb.xf[q] = sh[q * P + jxf];
        nb.xb[q] = sh[q * P + jxb];
        nb.yf[q] = sh[q * P + jyf];
        nb.yb[q] = sh[q * P + jyb];
      }
      hw_compute<double>(nb, g, site(z), diag, o);
    }
    __syncthreads();
    if (on) {
#pragma unroll
      for (int q = 0; q < 4; ++q) sh[q * P + j] = o[q];
    }
    __syncthreads();
    double2* plane = out + (size_t)4 * XY * (z + Z * t);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = q * 256 + j;
      if (e < 4 * XY) {
        const double2 v = sh[(e & 3) * P + (e >> 2)];
        const ev2<double> w = {v.x, v.y};
        __builtin_nontemporal_store(w, (OV_GLOBAL ev2<double>*)(plane + e));
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      nb.zb[q] = nb.c[q];
      nb.c[q] = nb.zf[q];
      nb.zf[q] = next2[q];
      nb.tf[q] = tf2[q];
      nb.tb[q] = tb2[q];
    }
  }
}

// H_W of f on the sites of a workgroup that owns zc consecutive z planes of one
// time slice (X Y == blockDim.x; the block's sites i0 .. i0 + zc X Y - 1, zc
// dividing Z), in the z-marching order of k_hw_zm: plane z below and above in
// registers, the current plane in LDS (sh: 4 X Y values) for the x and y
// neighbours.  Next to the stencil operands each site may take one more spinor
// of its own (the epilogue operand, from ep).  begin() issues the loads of the
// first plane, so that a caller puts them in flight before its scalar work (a
// workgroup whose system has converged reads no more than that); with PIPE, run()
// loads the operands of plane k + 1 while plane k is computed (two register sets),
// else after it.  For each site, epi(i, w, e) receives w = (H_W f)_i and the epilogue
// operand e and returns a partial sum; run() returns the total.  Every thread of the
// block must call run().
template <class R, bool PIPE>
struct ZmMarch {
  const c2<R>* f;
  const c2<R>* ep;
  int V, XY, Z, base, z0, tf_off, tb_off, jxf, jxb, jyf, jyb;
  c2<R> prev[4], cur[4], next[4], tf[4], tb[4], e[4];
  c2<R> next2[4], tf2[4], tb2[4], e2[4];  // PIPE: operands of the following plane

  __device__ __forceinline__ int plane(int z) const { return base + XY * (z < Z ? z : z - Z); }

  // operands of the plane after the one at site index i (z index z of that plane)
  __device__ __forceinline__ void load_ahead(int i, int z) {
    const int i2 = i + XY;  // plane z + 1 < Z
    load_sp<R>(f, V, plane(z + 2), next2);
    load_sp<R>(f, V, i2 + tf_off, tf2);
    load_sp<R>(f, V, i2 + tb_off, tb2);
    if (ep) load_sp<R>(ep, V, i2, e2);
  }

  __device__ __forceinline__ void begin(const c2<R>* __restrict__ f_, const c2<R>* __restrict__ ep_,
                                        const Geo& g, int i0) {
    f = f_;
    ep = ep_;
    const int X = g.X, Y = g.Y, T = g.T;
    V = g.V;
    Z = g.Z;
    XY = X * Y;
    const int XYZ = XY * Z;
    const int j = threadIdx.x;
    const int x = j % X, y = j / X;
    const int p0 = i0 / XY;  // z0 + Z t
    const int t = p0 / Z;
    z0 = p0 - Z * t;
    tf_off = (t + 1 < T) ? XYZ : XYZ - V;
    tb_off = (t > 0) ? -XYZ : V - XYZ;
    jxf = y * X + ((x + 1 < X) ? x + 1 : 0);
    jxb = y * X + ((x > 0) ? x - 1 : X - 1);
    jyf = ((y + 1 < Y) ? y + 1 : 0) * X + x;
    jyb = ((y > 0) ? y - 1 : Y - 1) * X + x;
    base = j + XYZ * t;
    const int i = plane(z0);
    load_sp<R>(f, V, plane(z0 > 0 ? z0 - 1 : Z - 1), prev);
    load_sp<R>(f, V, i, cur);
    load_sp<R>(f, V, plane(z0 + 1), next);
    load_sp<R>(f, V, i + tf_off, tf);
    load_sp<R>(f, V, i + tb_off, tb);
    if (ep) load_sp<R>(ep, V, i, e);
  }

  template <class Epi>
  __device__ __forceinline__ double run(int zc, const Geo& g, R diag, c2<R>* sh, Epi epi) {
    const int j = threadIdx.x;
    double acc = 0.0;
    for (int k = 0; k < zc; ++k) {
      const int i = plane(z0 + k);
      if (PIPE && k + 1 < zc) load_ahead(i, z0 + k);
      __syncthreads();  // reads of the previous plane are done
#pragma unroll
      for (int q = 0; q < 4; ++q) sh[q * XY + j] = cur[q];
      __syncthreads();
      Nbr<R> nb;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        nb.c[q] = cur[q];
        nb.xf[q] = sh[q * XY + jxf];
        nb.xb[q] = sh[q * XY + jxb];
        nb.yf[q] = sh[q * XY + jyf];
        nb.yb[q] = sh[q * XY + jyb];
        nb.zf[q] = next[q];
        nb.zb[q] = prev[q];
        nb.tf[q] = tf[q];
        nb.tb[q] = tb[q];
      }
      c2<R> w[4];
      hw_compute<R>(nb, g, i, diag, w);
      acc += epi(i, w, e);
      if (PIPE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          prev[q] = cur[q];
          cur[q] = next[q];
          next[q] = next2[q];
          tf[q] = tf2[q];
          tb[q] = tb2[q];
          e[q] = e2[q];
        }
      } else if (k + 1 < zc) {
        const int i2 = i + XY;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          prev[q] = cur[q];
          cur[q] = next[q];
        }
        load_sp<R>(f, V, plane(z0 + k + 2), next);
        load_sp<R>(f, V, i2 + tf_off, tf);
        load_sp<R>(f, V, i2 + tb_off, tb);
        if (ep) load_sp<R>(ep, V, i2, e);
      }
    }
    return acc;
  }
};

// First site of z-marching workgroup lb of a system (lb < T Z / zc).  As in k_hw_zm, FP64
// takes the time slices fastest, so that time-neighbouring planes belong to consecutive
// workgroups (loaded together, served by one L2); FP32 keeps the z chunks fastest.
template <class R>
__device__ __forceinline__ int zm_first_site(const SysDev& S, int lb) {
  if (sizeof(R) == sizeof(double)) {
    const int nzc = (S.g.Z * S.g.X * S.g.Y) / S.spb;  // z chunks per time slice
    return ((lb % S.g.T) * nzc + lb / S.g.T) * S.spb;
  }
  return lb * S.spb;
}

// The z-marching passes prefetch the next plane's operands in FP32 only (ZM = 2): in
// FP64 the second register set would halve the co-resident workgroups of large launches
// and measured no faster on small ones.

// ------------------------------------------------------- multi-shift: t pass
// Iteration n.  Finishes rho_n = |r_n|^2 (partials of the previous kernel),
// advances the shift recurrences, decides convergence, then
//   t_n = H r_n + beta_{n-1} t_{n-1}  -> basis slot n,  partial |t_n|^2.
// Latency layout: every independent load (control word, partials, scalar
// history, the nine stencil operands and t_{n-1}) is issued before any of them
// is consumed, and each wave finishes the reduction and the shift recurrences
// on its own (identical bits in every wave), so the only barrier is the final
// block reduction.
// ZM: 0 plain passes, 1 z-marching, 2 z-marching with the next plane prefetched.
// CF: read the system's on/off flag and the done word before the stencil operands, so
// that a workgroup with nothing to do returns without reading them (large batched
// launches, where other workgroups hide the extra round trip); else the operands go out
// first and the check follows (a single system's launch waits for memory once).
template <class R, int ZM, bool CF>
__device__ __forceinline__ int ms_t_block(const SysDev& S, int lb, int n, const MsParams* mp,
                                          double* lds, c2<R>* sh) {
  const int lane = threadIdx.x & 63;
  const Geo g = S.g;
  const int np = mp->np;
  const int nblk = S.nblk;

  const int act_sys = S.active ? *S.active : 1;
  const int done = (n > 0) ? S.h_ctl[0] : 0;
  // partials of rho_n (this lane's share, summed in a fixed order)
  double pr = 0.0;
  for (int j = lane; j < nblk; j += 64) pr += ldg(S.part_b, j);
  // scalar history for lane k = shift k
  const int k = lane;
  double zk1 = 1.0, zk2 = 1.0, a1 = 0.0, a2 = 1.0, rho_m1 = 1.0, rho_m2 = 1.0, rho0 = 0.0;
  unsigned int act_prev = 0xffffffffu;
  if (n > 0) {
    act_prev = S.h_active[n - 1];
    rho_m1 = S.h_rho[n - 1];
    a1 = S.h_alpha[n - 1];
    rho0 = S.h_rho[0];
    if (k < np) zk1 = S.h_zeta[(size_t)(n - 1) * MAXP + k];
    if (n >= 2) {
      a2 = S.h_alpha[n - 2];
      rho_m2 = S.h_rho[n - 2];
      if (k < np) zk2 = S.h_zeta[(size_t)(n - 2) * MAXP + k];
    }
  }
  // stencil operands
  const size_t slot = (size_t)4 * g.V;
  const c2<R>* rin = (const c2<R>*)(n == 0 ? S.src : S.r);
  c2<R>* tn = (c2<R>*)S.basis + (size_t)n * slot;
  const c2<R>* tp = (const c2<R>*)S.basis + (size_t)(n > 0 ? n - 1 : 0) * slot;
  const int i0 = ZM ? zm_first_site<R>(S, lb) : lb * S.spb;
  const int i1 = min(g.V, i0 + S.spb);
  int i = i0 + threadIdx.x;
  constexpr bool zm = ZM > 0;  // z-marching (mp->zm planes per workgroup)
  const bool have = !zm && i < i1;
  Nbr<R> nb;
  c2<R> q[4];
  ZmMarch<R, ZM == 2> zmm;
  if (CF && (!act_sys || done)) return 0;
  if (zm) zmm.begin(rin, n > 0 ? tp : nullptr, g, i0);
  if (have) {
    load_nbr<R>(rin, g, i, nb);
    if (n > 0) load_sp<R>(tp, g.V, i, q);
  }
  if (!act_sys || done) return 0;

  // rho_n and the shift recurrences, per wave
  const double rho = wave_sum_all(pr);
  const double srho = sqrt(rho);
  if (n == 0) rho0 = rho;
  const double thr = mp->tol * sqrt(rho0);
  bool act = false;
  double zn = 1.0;
  if (n == 0) {
    act = (k < np) && (srho > thr);
  } else if (k < np) {
    zn = zk1;
    if (act_prev & (1u << k)) {
      const double b2 = (n >= 2) ? rho_m1 / rho_m2 : 0.0;  // beta_{n-2}
      const double den = a2 * zk2 * (1.0 + a1 * mp->sigma[k]) + a1 * b2 * (zk2 - zk1);
      zn = zk1 * zk2 * a2 / den;
      act = fabs(zn) * srho > thr;
    }
  }
  const unsigned int amask = (unsigned int)__ballot(act);
  int status = 0;
  if (n > 0 && (!(rho >= 0.0) || !isfinite(rho))) status = 1;  // breakdown
  int stop = (amask == 0) || status != 0;
  if (!stop && n >= mp->cap) { stop = 1; status = 2; }            // basis exhausted
  if (lb == 0 && threadIdx.x < 64) {
    if (k < np) S.h_zeta[(size_t)n * MAXP + k] = zn;
    if (k == 0) {
      S.h_rho[n] = rho;
      S.h_active[n] = amask;
      if (stop) {
        S.h_ctl[1] = n;
        S.h_ctl[2] = status;
      }
      // one word: 0 while iterating, n + 1 once finished at iteration n
      __hip_atomic_store(&S.h_ctl[0], stop ? n + 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (stop) return 0;
  const R beta = (R)((n > 0) ? rho / rho_m1 : 0.0);

  double acc = 0.0;
  if (zm) {
    acc = zmm.run(mp->zm, g, (R)mp->diag, sh, [&](int ii, c2<R>* o, const c2<R>* qq) -> double {
      if (n > 0) {
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2)
          o[k2] = c2<R>{o[k2].x + beta * qq[k2].x, o[k2].y + beta * qq[k2].y};
      }
      store_ms<R>(mp->nt, tn, g.V, ii, o);
      return norm2_sp(o);
    });
    i = i1;  // every site done
  }
  if (have) {
    c2<R> o[4];
    hw_compute<R>(nb, g, i, (R)mp->diag, o);
    if (n > 0) {
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) o[k2] = c2<R>{o[k2].x + beta * q[k2].x, o[k2].y + beta * q[k2].y};
    }
    store_ms<R>(mp->nt, tn, g.V, i, o);
    acc = norm2_sp(o);
  }
  // remaining sites of this block (sites per thread > 1)
  for (i += blockDim.x; !zm && i < i1; i += blockDim.x) {
    c2<R> o[4];
    hw_site<R>(rin, g, i, (R)mp->diag, o);
    if (n > 0) {
      load_sp<R>(tp, g.V, i, q);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) o[k2] = c2<R>{o[k2].x + beta * q[k2].x, o[k2].y + beta * q[k2].y};
    }
    store_ms<R>(mp->nt, tn, g.V, i, o);
    acc += norm2_sp(o);
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_a[lb] = tot;
  return i1 - i0;
}

template <class R, int ZM, bool CF>
__device__ __forceinline__ int ms_r_block(const SysDev& S, int lb, int n, const MsParams* mp,
                                          double* lds, c2<R>* sh) {
  const int lane = threadIdx.x & 63;
  const Geo g = S.g;
  const int nblk = S.nblk;
  const int act_sys = S.active ? *S.active : 1;
  const int done = S.h_ctl[0];
  double pg = 0.0;
  for (int j = lane; j < nblk; j += 64) pg += ldg(S.part_a, j);
  const double rho = S.h_rho[n];
  const size_t slot = (size_t)4 * g.V;
  const c2<R>* tn = (const c2<R>*)S.basis + (size_t)n * slot;
  const c2<R>* rin = (const c2<R>*)(n == 0 ? S.src : S.r);
  c2<R>* rout = (c2<R>*)S.r;
  const int i0 = ZM ? zm_first_site<R>(S, lb) : lb * S.spb;
  const int i1 = min(g.V, i0 + S.spb);
  int i = i0 + threadIdx.x;
  constexpr bool zm = ZM > 0;
  const bool have = !zm && i < i1;
  Nbr<R> nb;
  c2<R> r[4];
  ZmMarch<R, ZM == 2> zmm;
  if (CF && (!act_sys || done)) return 0;
  if (zm) zmm.begin(tn, rin, g, i0);
  if (have) {
    load_nbr<R>(tn, g, i, nb);
    load_sp<R>(rin, g.V, i, r);
  }
  if (!act_sys || done) return 0;
  const double gam = wave_sum_all(pg);
  const double alpha_d = rho / gam;
  const int stop = !(gam > 0.0) || !isfinite(alpha_d);
  if (lb == 0 && threadIdx.x == 0) {
    S.h_alpha[n] = alpha_d;
    if (stop) {
      S.h_ctl[1] = n;
      S.h_ctl[2] = 1;
      __hip_atomic_store(&S.h_ctl[0], n + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (stop) return 0;
  const R alpha = (R)alpha_d;
  double acc = 0.0;
  if (zm) {
    acc = zmm.run(mp->zm, g, (R)mp->diag, sh, [&](int ii, c2<R>* w, const c2<R>* r0) -> double {
      c2<R> rr[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) rr[k] = r0[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) rr[k] = c2<R>{rr[k].x - alpha * w[k].x, rr[k].y - alpha * w[k].y};
      store_ms<R>(mp->nt, rout, g.V, ii, rr);
      return norm2_sp(rr);
    });
    i = i1;
  }
  if (have) {
    c2<R> w[4];
    hw_compute<R>(nb, g, i, (R)mp->diag, w);
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = c2<R>{r[k].x - alpha * w[k].x, r[k].y - alpha * w[k].y};
    store_ms<R>(mp->nt, rout, g.V, i, r);
    acc = norm2_sp(r);
  }
  for (i += blockDim.x; !zm && i < i1; i += blockDim.x) {
    c2<R> w[4];
    hw_site<R>(tn, g, i, (R)mp->diag, w);
    load_sp<R>(rin, g.V, i, r);
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = c2<R>{r[k].x - alpha * w[k].x, r[k].y - alpha * w[k].y};
    store_ms<R>(mp->nt, rout, g.V, i, r);
    acc += norm2_sp(r);
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_b[lb] = tot;
  return i1 - i0;
}

// Kernel-duration sampling: once every wave of the workgroup is done, thread 0 stores
// the workgroup's start and end wall-clock stamps and the sites it processed (0 for a
// system that sat the launch out) in its own three words (vector stores, no atomics); the
// host takes max(end) - min(start) over the workgroups and counts the processed sites' bytes.
__device__ __forceinline__ void stamp_block(unsigned long long* ts, unsigned long long t0,
                                            int sites) {
  __syncthreads();
  if (threadIdx.x == 0) {
    ts[3 * blockIdx.x] = t0;
    ts[3 * blockIdx.x + 1] = wall_clock64();
    ts[3 * blockIdx.x + 2] = (unsigned long long)(sites > 0 ? sites : 0);
  }
}

// Iteration n, t pass: finishes rho_n = |r_n|^2 from the previous kernel's
// partials, advances the shift recurrences, decides convergence, then
//   t_n = H r_n + beta_{n-1} t_{n-1}  -> basis slot n,  partial |t_n|^2.
// Latency layout: every independent load (control word, partials, scalar
// history, the nine stencil operands and t_{n-1}) is issued before any of them
// is consumed, and each wave finishes the reduction and the shift recurrences
// on its own (identical bits in every wave), so the only barrier is the final
// block reduction.  The stores of t_n and r_{n+1} go through the caches where those can hold
// them for the next pass, which reads both (MsParams nt; launch_ms_tab).
template <class R, int ZM, bool CF>
__global__ void __launch_bounds__(256) k_ms_t(const SysDev* __restrict__ sys,
                                              const int* __restrict__ bmap, int nb_total, int n,
                                              const MsParams mp_) {
  __shared__ double lds[17];
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  unsigned long long t0 = 0;
  if (mp_.tstamp && threadIdx.x == 0) t0 = wall_clock64();
  const int L = mp_.share ? (int)blockIdx.x : xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = mp_.share ? xcd_share(L - S.blk0, S.nblk) : L - S.blk0;
  const int sites = ms_t_block<R, ZM, CF>(S, lb, n, &mp_, lds, ZM ? (c2<R>*)dyn_lds : nullptr);
  if (mp_.tstamp) stamp_block(mp_.tstamp, t0, sites);
}

// Iteration n, r pass:
//   alpha_n = rho_n / |t_n|^2;  r_{n+1} = r_n - alpha_n H t_n;  partial |r_{n+1}|^2.
template <class R, int ZM, bool CF>
__global__ void __launch_bounds__(256) k_ms_r(const SysDev* __restrict__ sys,
                                              const int* __restrict__ bmap, int nb_total, int n,
                                              const MsParams mp_) {
  __shared__ double lds[17];
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  unsigned long long t0 = 0;
  if (mp_.tstamp && threadIdx.x == 0) t0 = wall_clock64();
  const int L = mp_.share ? (int)blockIdx.x : xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = mp_.share ? xcd_share(L - S.blk0, S.nblk) : L - S.blk0;
  const int sites = ms_r_block<R, ZM, CF>(S, lb, n, &mp_, lds, ZM ? (c2<R>*)dyn_lds : nullptr);
  if (mp_.tstamp) stamp_block(mp_.tstamp, t0, sites);
}

// ------------------------------------------------ multi-shift: resident form
// Every iteration of a multi-shift solve in one launch, for lattices whose r_n and t_n fit
// the chip's registers: one workgroup per CU owns a block of bx by bz bt sites of one
// entry; its compute waves keep r and t of their sites in registers (K sites per thread)
// and the field the stencil reads in LDS, one more wave (the service wave) handles the
// exchange with the other workgroups and the CG scalars.  Per pass
//   1. the compute waves publish the field: their sites to LDS, and the projected half
//      spinors (1 -+ g_mu) psi (two of four components: the hop needs no more) of the
//      block's faces to the neighbouring workgroups by device-scope (sc1) stores;
//   2. while these travel they apply the hops inside the block out of LDS, then read the
//      neighbours' faces (device-scope loads) until every value is there (res_empty);
//      meanwhile the service wave sends the block's partial norm and collects everybody's:
//      words that carry the pass's epoch, so one exchange is the reduction and the barrier;
//   3. with the sum they update t or r, while the service wave advances the recurrences.
// Nothing else crosses workgroups, so no cache is written back or invalidated, and t_n goes
// to the basis with streaming stores (no workgroup reads them, but they share the wait counter
// of the face loads behind them, and the next publication waits for both).  Bound by latency:
// an FP64 pass at 16^4 (one source, 128 workgroups of 512 sites) takes 2.9 us, a third of it
// update and publish, a third the hops out of LDS, the rest waits for faces and the sum (the
// per-pass kernels: 10 us and the launch gap; with a flag per workgroup for its faces and the
// partials read one after the other 3.7); 8^4 takes 1.8 us (4.5 us), 4^4, one workgroup and no
// exchange, 1.4 us (3.3 us). Two sources of 16^4 at once, 256 workgroups, 3.9 us; 16^3 x 32, all
// of them in one sum, 4.0 us.
struct ResRun {          // consecutive entries on one lattice
  int e0, ne;            // table entries
  int wg0;               // first workgroup of the launch
  int G;                 // workgroups per entry
  int b[4], nb[4];       // block extents, blocks per axis
  int FT;                // complex values of one workgroup's faces (one field)
  long long face0;       // first byte of this run's faces
};
constexpr int RES_RUNS = 8;
constexpr int RES_WGS = 256;      // workgroups of a launch at most
// Compute waves of a workgroup at most: with the service wave four per SIMD, 128 registers
// each (FP64 one site per thread, FP32 two).  The same block on half the waves with twice
// the sites each takes a fifth longer (12^4, 216 sites: 2.84 -> 3.41 us per pass).
constexpr int RES_WAVES = 15;
constexpr int RES_THREADS = 64 * (RES_WAVES + 1);
// Device words of the exchange, zero at first: epochs only grow, so nothing is cleared
// between launches.
struct ResShared {
  unsigned epoch, abort;                    // epoch base of the next launch; a wait ran out
  unsigned pad[62];
  // per workgroup one 64-byte line each: words of one line written by several workgroups
  // cost the exchange a quarter more (128 workgroups: 2.37 us, 1.73 us apart)
  struct {
    u32x4 word, pad[3];
  } part[2][RES_WGS];                       // tagged partial sums by the epoch's parity
};
struct ResArgs {
  int nrun, L;                     // runs; iterations at most
  int nap, nap_face;               // first looks, in 128 and 64 cycles (ResLaunch)
  unsigned eoff;                   // epoch offset of this launch
  ResShared* sh;
  int* abort_host;                 // pinned host word, set with sh->abort
  char* face;
  long long spin;                  // wall-clock ticks a wait may take
  ResRun run[RES_RUNS];
};
// What k_ms_coef, which follows every resident multi-shift, does to the epochs.
struct ResEpoch {
  ResShared* sh = nullptr;         // null: no resident launch
  unsigned bump = 0;               // epochs the launches used
};

// A face value that has not arrived: the faces hold this pattern when a launch starts and when
// it ends, and a reader puts it back.  Each value's first word (FP32), high word (FP64) tells
// whether its eight bytes are there, so faces need no flag of their own (waiting for the
// stores' end, a flag and its polling took a microsecond of every pass).  Both words are
// signalling NaNs of their type, which no arithmetic returns, whatever NaN the caller's fields
// hold (a published value is a sum; the kernels run in IEEE mode, where a sum quiets them).
constexpr unsigned RES_EMPTY32 = 0x7fa45a5au;  // a float; even words
constexpr unsigned RES_EMPTY64 = 0x7ff45a5au;  // the high word of a double; odd words
__device__ __forceinline__ u32x4 res_empty() {
  return u32x4{RES_EMPTY32, RES_EMPTY64, RES_EMPTY32, RES_EMPTY64};
}
constexpr unsigned RES_OOB = 0x80000000u;  // beyond every buffer: loads 0, stores nothing
constexpr int RES_SC1 = 16;                // device-scope cache policy of a buffer access
constexpr int RES_VOLATILE = (int)0x80000000;

template <class R>
struct Half {
  c2<R> a, b;
};

// Two components of a face site at byte offset o of the field that starts at byte so: FP64
// one 16-byte access per component (components Fb bytes apart), FP32 both in one access.
__device__ __forceinline__ Half<double> face_ld(__amdgpu_buffer_rsrc_t rs, unsigned o, unsigned so,
                                                unsigned Fb, double) {
  const u32x4 p = __builtin_amdgcn_raw_buffer_load_b128(rs, o, so, RES_SC1);
  const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rs, o, so + Fb, RES_SC1);
  return Half<double>{__builtin_bit_cast(double2, p), __builtin_bit_cast(double2, q)};
}
__device__ __forceinline__ Half<float> face_ld(__amdgpu_buffer_rsrc_t rs, unsigned o, unsigned so,
                                               unsigned, float) {
  return __builtin_bit_cast(
      Half<float>, __builtin_amdgcn_raw_buffer_load_b128(rs, o, so, RES_SC1));
}
// Every eight bytes of the two values have arrived.
__device__ __forceinline__ bool face_in(const Half<double>& h) {
  const u32x4 p = __builtin_bit_cast(u32x4, h.a), q = __builtin_bit_cast(u32x4, h.b);
  return p.y != RES_EMPTY64 && p.w != RES_EMPTY64 && q.y != RES_EMPTY64 && q.w != RES_EMPTY64;
}
__device__ __forceinline__ bool face_in(const Half<float>& h) {
  const u32x4 p = __builtin_bit_cast(u32x4, h);
  return p.x != RES_EMPTY32 && p.z != RES_EMPTY32;
}
// Stores add the field's byte to the vector offset: behind a 16-byte store with an offset in
// a scalar register the compiler leaves no wait state before it reuses the data registers,
// and the store then took the new values here.
__device__ __forceinline__ void face_st(__amdgpu_buffer_rsrc_t rs, unsigned o, unsigned Fb,
                                        const Half<double>& h) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h.a), rs, o, 0, RES_SC1);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h.b), rs, o + Fb, 0, RES_SC1);
}
__device__ __forceinline__ void face_st(__amdgpu_buffer_rsrc_t rs, unsigned o, unsigned,
                                        const Half<float>& h) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h), rs, o, 0, RES_SC1);
}

// The field in LDS: a site's four components side by side, 16 bytes of padding behind them
// (FP64 80, FP32 48 bytes a site: 16 lanes of consecutive sites fall on different banks, and
// one address serves every component).  Site S, the last, stays zero: a neighbour that is
// another workgroup's.
template <class R>
constexpr int RES_SITE = 4 * (int)sizeof(c2<R>) + 16;
__device__ __forceinline__ void lds_get(const unsigned char* sh, unsigned j, double2 v[4]) {
  const u32x4* p = (const u32x4*)(sh + j * RES_SITE<double>);
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = __builtin_bit_cast(double2, p[q]);
}
__device__ __forceinline__ void lds_get(const unsigned char* sh, unsigned j, float2 v[4]) {
  const f32x4* p = (const f32x4*)(sh + j * RES_SITE<float>);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const f32x4 x = p[q];
    v[2 * q] = float2{x.x, x.y};
    v[2 * q + 1] = float2{x.z, x.w};
  }
}
__device__ __forceinline__ void lds_put(unsigned char* sh, unsigned j, const double2 v[4]) {
  u32x4* p = (u32x4*)(sh + j * RES_SITE<double>);
#pragma unroll
  for (int q = 0; q < 4; ++q) p[q] = __builtin_bit_cast(u32x4, v[q]);
}
__device__ __forceinline__ void lds_put(unsigned char* sh, unsigned j, const float2 v[4]) {
  f32x4* p = (f32x4*)(sh + j * RES_SITE<float>);
#pragma unroll
  for (int q = 0; q < 2; ++q)
    p[q] = f32x4{v[2 * q].x, v[2 * q].y, v[2 * q + 1].x, v[2 * q + 1].y};
}

__device__ __forceinline__ void face_clear(__amdgpu_buffer_rsrc_t rs, unsigned o, unsigned Fb,
                                           double) {
  const u32x4 e = res_empty();
  __builtin_amdgcn_raw_buffer_store_b128(e, rs, o, 0, RES_SC1);
  __builtin_amdgcn_raw_buffer_store_b128(e, rs, o + Fb, 0, RES_SC1);
}
__device__ __forceinline__ void face_clear(__amdgpu_buffer_rsrc_t rs, unsigned o, unsigned, float) {
  const u32x4 e = res_empty();
  __builtin_amdgcn_raw_buffer_store_b128(e, rs, o, 0, RES_SC1);
}

// Sum over the wave in lane 63, on the vector ALU alone (a shuffle tree through LDS takes
// three times as long, on the critical path of every pass): rows of 16 by row_shr 1, 2, 4,
// 8, then row_bcast 15 and 31.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_term(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum_last(double v) {
  v += dpp_term<0x111, 0xf>(v);
  v += dpp_term<0x112, 0xf>(v);
  v += dpp_term<0x114, 0xf>(v);
  v += dpp_term<0x118, 0xf>(v);
  v += dpp_term<0x142, 0xa>(v);
  v += dpp_term<0x143, 0xc>(v);
  return v;
}

// Upper two components of (1 + s g_mu) psi: s = -1 the hop from x + mu, s = 1 from x - mu.
// With g_mu = [[0, B], [B^dag, 0]] they are u + s B l, and the lower two s B^dag of them.
template <class R, int MU>
__device__ __forceinline__ Half<R> hop_project(const c2<R> v[4], R s) {
  using C = c2<R>;
  C p, q;  // B l
  if (MU == 0) { p = cmul_i(v[3]); q = cmul_i(v[2]); }
  if (MU == 1) { p = v[3]; q = C{-v[2].x, -v[2].y}; }
  if (MU == 2) { p = cmul_i(v[2]); q = C{v[3].y, -v[3].x}; }
  if (MU == 3) { p = v[2]; q = v[3]; }
  return Half<R>{C{v[0].x + s * p.x, v[0].y + s * p.y}, C{v[1].x + s * q.x, v[1].y + s * q.y}};
}

// acc += f (h, s B^dag h), with fs = f s.
template <class R, int MU>
__device__ __forceinline__ void hop_add(const Half<R>& h, R f, R fs, c2<R> acc[4]) {
  using C = c2<R>;
  C p, q;  // B^dag h
  if (MU == 0) { p = C{h.b.y, -h.b.x}; q = C{h.a.y, -h.a.x}; }
  if (MU == 1) { p = C{-h.b.x, -h.b.y}; q = h.a; }
  if (MU == 2) { p = C{h.a.y, -h.a.x}; q = cmul_i(h.b); }
  if (MU == 3) { p = h.a; q = h.b; }
  acc[0] = C{acc[0].x + f * h.a.x, acc[0].y + f * h.a.y};
  acc[1] = C{acc[1].x + f * h.b.x, acc[1].y + f * h.b.y};
  acc[2] = C{acc[2].x + fs * p.x, acc[2].y + fs * p.y};
  acc[3] = C{acc[3].x + fs * q.x, acc[3].y + fs * q.y};
}

// One site of a block as its thread sees it, set up once.  An axis that is cut (split over
// workgroups) has at least two sites in the block, so a site lies on at most one of the two
// faces: one half spinor per axis goes out and one comes in.
struct ResSite {
  int j, gi;        // index in the block and on the lattice
  unsigned fl;      // bits 2 mu, 2 mu + 1: the hop from above / below comes from another
                    // workgroup; 8, 9: the time hop above / below takes the phase -1
  unsigned nb[4];   // LDS sites of the neighbours: above | below << 16 (S: another's)
  unsigned st[4];   // byte offset of the half spinor the site sends, RES_OOB for none
  unsigned ld[4];   // byte offset of the one it receives
};

// Site index jj (of the block's S = prod b, or beyond: a thread without a site gets the last
// one's fields and no faces) of workgroup w of its entry.
template <class R>
__host__ __device__ inline ResSite res_site(const ResRun& U, const Geo& g, int w, int jj) {
  const int S = U.b[0] * U.b[1] * U.b[2] * U.b[3];
  const bool have = jj < S;
  const int j = have ? jj : S - 1;
  int c[4], wc[4], q = j, r = w;
  for (int mu = 0; mu < 4; ++mu) {
    c[mu] = q % U.b[mu];
    q /= U.b[mu];
    wc[mu] = r % U.nb[mu];
    r /= U.nb[mu];
  }
  ResSite s;
  s.j = jj;
  s.gi = wc[0] * U.b[0] + c[0] +
         g.X * (wc[1] * U.b[1] + c[1] +
                g.Y * (wc[2] * U.b[2] + c[2] + g.Z * (wc[3] * U.b[3] + c[3])));
  s.fl = 0;
  int ss = 1, ws = 1;  // strides of the axis in the block and among the workgroups
  unsigned o = 0;      // first face value of the axis
  for (int mu = 0; mu < 4; ++mu) {
    const int b = U.b[mu], n = U.nb[mu];
    const bool top = c[mu] == b - 1, bot = c[mu] == 0, cut = n > 1;
    const unsigned F = (unsigned)(S / b);
    s.nb[mu] = (unsigned)(!top ? j + ss : cut ? S : j - ss * (b - 1)) |
               (unsigned)(!bot ? j - ss : cut ? S : j + ss * (b - 1)) << 16;
    s.st[mu] = s.ld[mu] = RES_OOB;
    if (cut && top) s.fl |= 1u << 2 * mu;
    if (cut && bot) s.fl |= 2u << 2 * mu;
    if (cut && have && (top || bot)) {
      const unsigned f = (unsigned)(j % ss + ss * (j / (ss * b)));  // site of the face
      // own face: the lower one, or 2 F values on, the upper; the neighbour's is the other
      const int wn = top ? w + (wc[mu] + 1 < n ? ws : ws - n * ws)
                         : w - (wc[mu] > 0 ? ws : ws - n * ws);
      const unsigned own = (unsigned)(w * U.FT) + o + (top ? 2 * F : 0u);
      const unsigned oth = (unsigned)(wn * U.FT) + o + (top ? 0u : 2 * F);
      const unsigned e = sizeof(R) == sizeof(double) ? f : 2 * f;  // FP32: interleaved
      s.st[mu] = (own + e) * (unsigned)sizeof(c2<R>);
      s.ld[mu] = (oth + e) * (unsigned)sizeof(c2<R>);
    }
    if (mu == 3 && g.bc < 0) {
      if (top && wc[3] == n - 1) s.fl |= 256u;
      if (bot && wc[3] == 0) s.fl |= 512u;
    }
    if (cut) o += 4 * F;
    ss *= b;
    ws *= n;
  }
  return s;
}

template <class R>
struct ResHalo {
  Half<R> h[4];     // per axis (0 where nothing is received)
};

// The field's uniform data of a compute wave.
template <class R>
struct ResBlock {
  int S;                     // sites of the block
  unsigned Fb[4];            // bytes between the two components of a face site (FP64)
  unsigned char* sh;         // LDS
  __amdgpu_buffer_rsrc_t rs;

  // Keeps what follows from a value (addresses of eight neighbours per site) from being
  // hoisted out of the iteration loop, where it would spill.
  __device__ __forceinline__ static unsigned opaque(unsigned c) {
    asm volatile("" : "+v"(c));
    return c;
  }
  // the forward hop of the block below, (1 - g) psi, or the backward hop of the one above
  template <int MU>
  __device__ __forceinline__ void put(const c2<R> v[4], const ResSite& s, unsigned fl,
                                      unsigned fld) const {
    face_st(rs, opaque(s.st[MU]) + fld, Fb[MU], hop_project<R, MU>(v, fl & (1u << 2 * MU) ? R(1) : R(-1)));
  }
  // The site holds v: to the faces and to LDS.
  __device__ __forceinline__ void publish(const c2<R> v[4], const ResSite& s, unsigned fld) const {
    const unsigned fl = opaque(s.fl);
    put<0>(v, s, fl, fld);
    put<1>(v, s, fl, fld);
    put<2>(v, s, fl, fld);
    put<3>(v, s, fl, fld);
    if (s.j < S) lds_put(sh, (unsigned)s.j, v);
  }
  // the half spinors received, and whether all of them are there
  __device__ __forceinline__ bool halo(ResHalo<R>& h, const ResSite& s, unsigned fld) const {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) h.h[mu] = face_ld(rs, s.ld[mu], fld, Fb[mu], R());
    bool in = true;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) in &= face_in(h.h[mu]);
    return in;
  }
  // empties the places of a site's received half spinors (o = s.ld), or of the sent ones
  __device__ __forceinline__ void clear(const unsigned (&o)[4], unsigned fld) const {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) face_clear(rs, opaque(o[mu]) + fld, Fb[mu], R());
  }

  // hops of an axis from inside the block
  template <int MU>
  __device__ __forceinline__ void hop_in(unsigned nb, unsigned fl, c2<R> acc[4]) const {
    R ff = R(1), fb = R(1);
    if (MU == 3) {
      ff = fl & 256u ? R(-1) : R(1);
      fb = fl & 512u ? R(-1) : R(1);
    }
    c2<R> n[4], m[4];
    lds_get(sh, nb & 0xffffu, n);
    lds_get(sh, nb >> 16, m);
    hop_add<R, MU>(hop_project<R, MU>(n, R(-1)), ff, -ff, acc);
    hop_add<R, MU>(hop_project<R, MU>(m, R(1)), fb, fb, acc);
  }
  // acc = sum of the hops from inside the block (the field in LDS)
  __device__ __forceinline__ void inside(const ResSite& s, c2<R> acc[4]) const {
    const unsigned fl = opaque(s.fl);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = c2<R>{R(0), R(0)};
    // two axes at a time: more LDS reads in flight would spill
    hop_in<0>(opaque(s.nb[0]), fl, acc);
    hop_in<1>(opaque(s.nb[1]), fl, acc);
    __builtin_amdgcn_sched_barrier(0);
    hop_in<2>(opaque(s.nb[2]), fl, acc);
    hop_in<3>(opaque(s.nb[3]), fl, acc);
    // computed here, before the barrier that follows: the compiler would sink the
    // arithmetic to its use behind it and keep every LDS operand alive
#pragma unroll
    for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(acc[q].x), "+v"(acc[q].y));
    __builtin_amdgcn_sched_barrier(0);
  }
  template <int MU>
  __device__ __forceinline__ void hop_out(const ResHalo<R>& h, unsigned fl, c2<R> acc[4]) const {
    R f = R(1);
    const bool top = fl & (1u << 2 * MU);
    if (MU == 3) f = fl & (top ? 256u : 512u) ? R(-1) : R(1);
    hop_add<R, MU>(h.h[MU], f, top ? -f : f, acc);
  }
  // acc += the hops from other workgroups' sites
  __device__ __forceinline__ void outside(const ResHalo<R>& h, const ResSite& s,
                                          c2<R> acc[4]) const {
    const unsigned fl = opaque(s.fl);
    hop_out<0>(h, fl, acc);
    hop_out<1>(h, fl, acc);
    hop_out<2>(h, fl, acc);
    hop_out<3>(h, fl, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(acc[q].x), "+v"(acc[q].y));
    __builtin_amdgcn_sched_barrier(0);
  }
  // out = H_W f at a site: g5 (diag v - 1/2 sum of the hops), v its own value.
  __device__ __forceinline__ static void finish(R diag, const c2<R> v[4], const c2<R> acc[4],
                                                c2<R> out[4]) {
    const R hh = R(0.5);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const c2<R> d = c2<R>{diag * v[q].x - hh * acc[q].x, diag * v[q].y - hh * acc[q].y};
      out[q] = q < 2 ? c2<R>{-d.x, -d.y} : d;
    }
  }
};

// Faces before the first resident launch of a call.
__global__ void __launch_bounds__(256) k_res_empty(u32x4* __restrict__ face, size_t n) {
  const u32x4 e = res_empty();
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    face[i] = e;
}

// What the service wave and the compute waves tell each other.
struct ResLds {
  double red[RES_WAVES];  // wave sums of the field just published
  double total;           // the entry's sum
  int stop;               // leave after the field is out (converged, broke down)
  int gone;               // a wait ran out
};

// A wait has run out: every workgroup leaves, the host runs the call again (one lane).
__device__ __forceinline__ void res_give_up(const ResArgs& A, ResLds& X) {
  __hip_atomic_store(&A.sh->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(A.abort_host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&X.gone, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The service wave's exchange: send the workgroup's partial s and wait for the G partials
// of the entry; their sum (lane 63) in a fixed order, the same bits in every workgroup.
// Each half of a 16-byte word carries the epoch, so that it need not arrive whole.
// Partials alternate between two slots: a workgroup writes epoch e + 2 only after every
// workgroup has sent e + 1, that is, has read e.  The wait is bounded: when `spin` ticks pass,
// or another workgroup has given up, the abort words are raised, false is returned and every
// workgroup leaves.
__device__ __forceinline__ bool res_exchange(const ResArgs& A, ResLds& X, int slot0, int w, int G,
                                             unsigned epoch, double s, double* total) {
  const int lane = threadIdx.x & 63;
  // scalar by construction, but not to the compiler, which would access the words in a loop
  // over the lanes' descriptors
  epoch = (unsigned)__builtin_amdgcn_readfirstlane((int)epoch);
  const int first = (int)(epoch & 1) * RES_WGS + __builtin_amdgcn_readfirstlane(slot0);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      &A.sh->part[0][0] + first, 0,
      __builtin_amdgcn_readfirstlane(G) * (int)sizeof(A.sh->part[0][0]), 0x00020000);
  if (lane == 0) {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(s);
    const u32x4 x = {(unsigned)bits, epoch, (unsigned)(bits >> 32), epoch};
    __builtin_amdgcn_raw_buffer_store_b128(x, rs, w * 64, 0, RES_SC1);
  }
  // nothing arrives sooner; polls in the meantime slow the stores that are on their way
  for (int n = 0; n < A.nap; ++n) __builtin_amdgcn_s_sleep(2);
  long long t0 = 0;
  for (int n = 0;; ++n) {
    // the lane's words (up to four) all in flight at once: a trip to memory is the cost, and
    // one after the other they made G > 64 half a microsecond slower, G > 192 two; words
    // beyond G read as zero
    u32x4 x[4] = {};
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u == 0 || G > 64 * u)
        x[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, (lane + 64 * u) * 64, 0,
                                                     RES_SC1 | RES_VOLATILE);
    bool ready = true;
    double p = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ready &= lane + 64 * u >= G || (x[u].y == epoch && x[u].w == epoch);
      p += __longlong_as_double((long long)(((unsigned long long)x[u].z << 32) | x[u].x));
    }
    if (__all(ready)) {
      *total = wave_sum_last(p);
      return true;
    }
    if ((n & 15) == 0) {
      const long long now = (long long)wall_clock64();
      if (n == 0) t0 = now;
      if (now - t0 >= A.spin ||
          __hip_atomic_load(&A.sh->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        if (lane == 0) res_give_up(A, X);
        return false;
      }
    }
  }
}

template <class R, int K>
__global__ void __launch_bounds__(RES_THREADS) k_ms_res(const SysDev* __restrict__ tab,
                                                        const ResArgs A, const MsParams mp) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ ResLds X;
  int ir = 0;
  for (int k = 1; k < A.nrun; ++k)
    if (A.run[k].wg0 <= (int)blockIdx.x) ir = k;
  const ResRun& U = A.run[ir];
  const int lw = (int)blockIdx.x - U.wg0;
  const int G = U.G;
  const SysDev& S = tab[U.e0 + lw / G];
  const int w = lw % G;
  const int slot0 = (int)blockIdx.x - w;
  if (S.active && *S.active == 0) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwc = (int)(blockDim.x >> 6) - 1;  // compute waves; the last wave serves
  if (threadIdx.x == 0) {
    X.stop = X.gone = 0;
  }
  unsigned ep = A.sh->epoch + A.eoff;

  if (wave == nwc) {
    // ---------------------------------------------------------- service wave
    const int np = mp.np;
    const double sigma = lane < np ? mp.sigma[lane] : 0.0;
    const bool keep = w == 0;  // records the history
    double* const h_zeta = S.h_zeta;
    double* const h_rho = S.h_rho;
    double* const h_alpha = S.h_alpha;
    unsigned* const h_active = S.h_active;
    // scalar history of lane = shift, as in the per-pass kernels
    double zk1 = 1.0, zk2 = 1.0, a1 = 1.0, a2 = 1.0, rho_m1 = 1.0, rho_m2 = 1.0, thr = 0.0;
    unsigned act_prev = 0xffffffffu;
    int n_stop = 0, status = 0, done = 0;
    auto exchange = [&](double* tot) -> bool {
      double s = 0.0;
      for (int k = 0; k < nwc; ++k) s += X.red[k];
      ++ep;
      bool ok = true;
      if (G > 1)
        ok = res_exchange(A, X, slot0, w, G, ep, s, &s);
      if (lane == 63) X.total = s;
      *tot = __longlong_as_double(
          ((long long)__builtin_amdgcn_readlane((int)(__double_as_longlong(s) >> 32), 63) << 32) |
          (unsigned)__builtin_amdgcn_readlane((int)__double_as_longlong(s), 63));
      return ok;
    };
    bool ok = true;
    for (int n = 0; n < A.L; ++n) {
      __syncthreads();  // r_n is out
      if (done) break;  // the previous r pass broke down
      double rho, gam;
      ok = exchange(&rho);
      __syncthreads();  // total is in
      ok &= X.gone == 0;
      if (!ok) break;
      const double srho = sqrt(rho);
      if (n == 0) thr = mp.tol * srho;
      bool act = false;
      double zn = 1.0;
      if (n == 0) {
        act = lane < np && srho > thr;
      } else if (lane < np) {
        zn = zk1;
        if (act_prev & (1u << lane)) {
          const double b2 = n >= 2 ? rho_m1 / rho_m2 : 0.0;
          const double den = a2 * zk2 * (1.0 + a1 * sigma) + a1 * b2 * (zk2 - zk1);
          zn = zk1 * zk2 * a2 / den;
          act = fabs(zn) * srho > thr;
        }
      }
      const unsigned amask = (unsigned)__ballot(act);
      if (n > 0 && (!(rho >= 0.0) || !isfinite(rho))) status = 1;
      bool stop = amask == 0 || status != 0;
      if (!stop && n >= mp.cap) {
        stop = true;
        status = 2;
      }
      if (keep) {
        if (lane < np) h_zeta[(size_t)n * MAXP + lane] = zn;
        if (lane == 0) {
          h_rho[n] = rho;
          h_active[n] = amask;
        }
      }
      if (stop) {
        n_stop = n;
        done = n + 1;
        if (lane == 0) X.stop = 1;
      }
      __syncthreads();  // t_n is out
      if (stop) break;
      ok = exchange(&gam);
      __syncthreads();  // total is in
      ok &= X.gone == 0;
      if (!ok) break;
      const double alpha = rho / gam;
      if (keep && lane == 0) h_alpha[n] = alpha;
      if (!(gam > 0.0) || !isfinite(alpha)) {
        status = 1;
        n_stop = n;
        done = n + 1;
        if (lane == 0) X.stop = 1;
      }
      zk2 = zk1;
      zk1 = zn;
      a2 = a1;
      a1 = alpha;
      rho_m2 = rho_m1;
      rho_m1 = rho;
      act_prev = amask;
    }
    if (keep && lane == 0 && ok) {
      if (done) {
        S.h_ctl[1] = n_stop;
        S.h_ctl[2] = status;
      }
      S.h_ctl[0] = done;  // 0: not finished within L
    }
    return;
  }

  // ------------------------------------------------------------ compute waves
  const Geo g = S.g;
  ResBlock<R> B;
  B.S = U.b[0] * U.b[1] * U.b[2] * U.b[3];
  B.sh = dyn_lds;
  if (threadIdx.x < RES_SITE<R> / 4)  // the zero site
    ((unsigned*)(dyn_lds + B.S * RES_SITE<R>))[threadIdx.x] = 0u;
  const unsigned fb = (unsigned)(G * U.FT * sizeof(c2<R>));  // bytes of one field's faces
  B.rs = __builtin_amdgcn_make_buffer_rsrc(A.face + U.face0 + (size_t)(lw / G) * 2 * fb, 0,
                                           (int)(2 * fb), 0x00020000);
  const R diag = (R)mp.diag;
  ResSite site[K];
#pragma unroll
  for (int k = 0; k < K; ++k) site[k] = res_site<R>(U, g, w, (int)threadIdx.x + k * 64 * nwc);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu)
    B.Fb[mu] = (unsigned)(B.S / U.b[mu]) * (unsigned)sizeof(c2<R>);
  c2<R>* basis = (c2<R>*)S.basis;
  const size_t slot = (size_t)4 * g.V;

  c2<R> r[K][4], t[K][4], hops[K][4];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if constexpr (sizeof(R) == sizeof(double)) {
      if (S.src_io) {  // the caller's field: no packed copy, no pass that makes g5 times it
        load_io(S.io_in, site[k].gi, r[k]);
        if (S.src_io == 2)
#pragma unroll
          for (int q = 0; q < 2; ++q) r[k][q] = c2<R>{-r[k][q].x, -r[k][q].y};
      } else {
        load_sp<R>((const c2<R>*)S.src, g.V, site[k].gi, r[k]);
      }
    } else {
      load_sp<R>((const c2<R>*)S.src, g.V, site[k].gi, r[k]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) t[k][q] = c2<R>{R(0), R(0)};
  }
  // The field v of the next pass goes out; false: leave.  Places emptied since the last one
  // are so before it goes out: their writers write them again only after a sum that this
  // workgroup's next partial is part of.
  auto send = [&](c2<R>(&v)[K][4], unsigned fo) -> bool {
    if (G > 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      B.publish(v[k], site[k], fo);
      acc += site[k].j < B.S ? norm2_sp(v[k]) : 0.0;
      __builtin_amdgcn_sched_barrier(0);
    }
    acc = wave_sum_last(acc);
    if (lane == 63) X.red[wave] = acc;
    __syncthreads();
    if (X.stop == 0) return true;
    // every workgroup stops here: nobody reads what has just gone out
#pragma unroll
    for (int k = 0; k < K; ++k) B.clear(site[k].st, fo);
    return false;
  };
  // hops = sum of the hops of the field just sent, its faces in the half at fo
  auto gather = [&](unsigned fo) {
#pragma unroll
    for (int k = 0; k < K; ++k) B.inside(site[k], hops[k]);
    if (G == 1) return;
    ResHalo<R> h[K];
    for (int n = 0; n < A.nap_face; ++n) __builtin_amdgcn_s_sleep(1);
    long long t0 = 0;
    for (int n = 0;; ++n) {
      asm volatile("" ::: "memory");  // every turn loads again
      bool in = true;
#pragma unroll
      for (int k = 0; k < K; ++k) in &= B.halo(h[k], site[k], fo);
      // the service wave ends the wait when it gives up
      if (__all(in) ||
          __hip_atomic_load(&X.gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
        break;
      if ((n & 15) == 0) {
        const long long now = (long long)wall_clock64();
        if (n == 0) t0 = now;
        if (now - t0 > A.spin) {
          if (lane == 0) res_give_up(A, X);
          break;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      B.clear(site[k].ld, fo);
      B.outside(h[k], site[k], hops[k]);
    }
  };
  double rho_m1 = 1.0;
  bool on = send(r, 0);
  for (int n = 0; n < A.L && on; ++n) {
    // ---- t pass: t_n = H r_n + beta_{n-1} t_{n-1}
    gather(0);
    __syncthreads();
    const double rho = X.total;
    if (X.gone) return;
    const R beta = (R)(n > 0 ? rho / rho_m1 : 0.0);
    rho_m1 = rho;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      c2<R> o[4];
      B.finish(diag, r[k], hops[k], o);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        t[k][q] = c2<R>{o[q].x + beta * t[k][q].x, o[q].y + beta * t[k][q].y};
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!send(t, fb)) return;  // converged at n
    // ---- r pass: alpha_n = rho_n / |t_n|^2, r_{n+1} = r_n - alpha_n H t_n
    c2<R>* tn = basis + (size_t)n * slot;
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (site[k].j < B.S)
        store_sp_nt<R>(tn, g.V, (int)B.opaque((unsigned)site[k].gi), t[k]);
    gather(fb);
    __syncthreads();
    const R alpha = (R)(rho / X.total);
    if (X.gone) return;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      c2<R> o[4];
      B.finish(diag, t[k], hops[k], o);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        r[k][q] = c2<R>{r[k][q].x - alpha * o[q].x, r[k][q].y - alpha * o[q].y};
      __builtin_amdgcn_sched_barrier(0);
    }
    if (n + 1 < A.L) on = send(r, 0);
  }
}

// Sites times iterations of the ne entries of a sampled resident launch (its t_n written), as
// the stamp of one workgroup without a time.
__global__ void __launch_bounds__(64) k_res_sites(const SysDev* __restrict__ tab, int ne, int L,
                                                  unsigned long long* __restrict__ stamp) {
  double sum = 0.0;
  for (int e = threadIdx.x; e < ne; e += 64) {
    const SysDev& S = tab[e];
    if (S.active && *S.active == 0) continue;
    sum += (double)S.g.V * (S.h_ctl[0] ? S.h_ctl[1] : L);
  }
  sum = wave_sum_last(sum);
  if (threadIdx.x == 63) {
    stamp[0] = stamp[1] = 0;
    stamp[2] = (unsigned long long)sum;
  }
}

// n > 0 values to LDS, four loads of a thread in flight: get(e) reads one (a thread without
// a value reads the last one), put(e, v) stores it, `between` runs while the first four are on
// their way.
template <class Get, class Put, class F>
__device__ __forceinline__ void stage_in(int n, Get get, Put put, F between) {
  const int bd = blockDim.x;
  int e0 = threadIdx.x;
  decltype(get(0)) v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = get(min(e0 + u * bd, n - 1));
  between();
  for (;;) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e0 + u * bd < n) put(e0 + u * bd, v[u]);
    e0 += 4 * bd;
    if (e0 >= n) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = get(min(e0 + u * bd, n - 1));
  }
}

// ------------------------------------------------- multi-shift: coefficients
// One workgroup per system.  Shift k ran N_k iterations (first n with its bit
// clear in h_active).  With z^j = zeta_k^j, alpha_{j,k} = alpha_j z^{j+1}/z^j,
// beta_{j,k} = beta_j (z^{j+1}/z^j)^2 and p_k^j = sum_{i<=j} z^i prod beta_{.,k} r_i:
//   y_k = sum_j z^j S_k^j r_j,  S_k^j = alpha_{j,k} + beta_{j,k} S_k^{j+1},  S_k^{N_k} = 0,
//   acc = sum_j c_j r_j,  c_j = sum_k a_k z^j S_k^j,
//   eps = H acc = sum_j d_j t_j,  d_j = c_j - beta_j c_{j+1}   (H r_j = t_j - beta_{j-1} t_{j-1}).
constexpr int COEF_THREADS = 512;
constexpr int COEF_LDS_ITERS = 160;  // history rows staged in LDS (larger N reads global)

// LDS of k_ms_coef.  The staged path works on these arrays only (no pointer that may
// point to either LDS or global memory: such accesses compile to flat instructions, and
// each of them waits for every global store in flight).
struct CoefLds {
  int N;
  int nk[MAXP];
  double res[MAXP];
  double rho[COEF_LDS_ITERS + 1], alpha[COEF_LDS_ITERS + 1], c[COEF_LDS_ITERS + 1];
  unsigned int act[COEF_LDS_ITERS + 1];
  double zeta[(COEF_LDS_ITERS + 1) * MAXP];
  double u[MAXP][COEF_LDS_ITERS + 1];   // recurrence factors, then the terms (k, j)
  double cp[MAXP][COEF_LDS_ITERS + 1];
  double g[COEF_LDS_ITERS + 1], td[COEF_LDS_ITERS + 1], to[COEF_LDS_ITERS + 1];
};

// Second function of the same Krylov space (entries with coef_d2 set):
//   w = H r(A)^2 psi = sum_j d2_j t_j,   so that eps^2 psi = A r(A)^2 psi = H w.
// The CG scalars give the Lanczos tridiagonal of A on v_j = (-1)^j r_j / |r_j|:
//   T_jj = 1/alpha_j + beta_{j-1}/alpha_{j-1},  T_j,j+1 = sqrt(beta_j)/alpha_j,
// and r(A)^2 psi ~ |psi| V r(T)^2 e_1 with r(T)^2 e_1 = sum_l a_l (T + b_l)^-1 g,
// g = sum_k a_k (T + b_k)^-1 e_1: 2 np tridiagonal solves (T + b is positive definite,
// elimination without pivoting is stable), one thread per shift.  Coefficients on r_j:
// c2_j = |psi| (-1)^j h_j / |r_j|; on t_j: d2_j = c2_j - beta_j c2_{j+1}.
// Work arrays U, CP ([MAXP][ld]), G, TD, TO ([N]) all in LDS or all in global memory.
__device__ __forceinline__ void coef_second(const SysDev& S, const MsParams* mp, int N,
                                            const double* rho, const double* alph, double* U,
                                            double* CP, double* G, double* TD, double* TO,
                                            int ld) {
  const int np = mp->np;
  for (int j = threadIdx.x; j < N; j += blockDim.x) {
    TD[j] = 1.0 / alph[j] + (j > 0 ? (rho[j] / rho[j - 1]) / alph[j - 1] : 0.0);
    TO[j] = sqrt(rho[j + 1] / rho[j]) / alph[j];
  }
  __syncthreads();
  auto solve = [&](int k, bool from_g) {
    double* u = U + (size_t)k * ld;
    double* cp = CP + (size_t)k * ld;
    const double bk = mp->sigma[k];
    // forward elimination; the next row's operands are read ahead of the division
    double cprev = 0.0, dprev = 0.0, ol = 0.0;
    double td = TD[0], rhs = from_g ? G[0] : 1.0;
    for (int j = 0; j < N; ++j) {
      const double to = TO[j];
      double td_n = 0.0, rhs_n = 0.0;
      if (j + 1 < N) {
        td_n = TD[j + 1];
        rhs_n = from_g ? G[j + 1] : 0.0;
      }
      const double inv = 1.0 / (td + bk - ol * cprev);
      const double cj = j + 1 < N ? to * inv : 0.0;
      const double dj = (rhs - ol * dprev) * inv;
      cp[j] = cj;
      u[j] = dj;
      cprev = cj;
      dprev = dj;
      ol = to;
      td = td_n;
      rhs = rhs_n;
    }
    double un = dprev;
    for (int j = N - 2; j >= 0; --j) {
      un = u[j] - cp[j] * un;
      u[j] = un;
    }
  };
  if (threadIdx.x < np) solve(threadIdx.x, false);
  __syncthreads();
  for (int j = threadIdx.x; j < N; j += blockDim.x) {
    double g = 0.0;
    for (int k = 0; k < np; ++k) g += mp->coef[k] * U[(size_t)k * ld + j];
    G[j] = g;
  }
  __syncthreads();
  if (threadIdx.x < np) solve(threadIdx.x, true);
  __syncthreads();
  const double sr0 = sqrt(rho[0]);
  for (int j = threadIdx.x; j < N; j += blockDim.x) {
    double h = 0.0;
    for (int k = 0; k < np; ++k) h += mp->coef[k] * U[(size_t)k * ld + j];
    G[j] = sr0 * ((j & 1) ? -h : h) / sqrt(rho[j]);  // c2_j
  }
  __syncthreads();
  for (int j = threadIdx.x; j < N; j += blockDim.x) {
    const double cn = (j + 1 < N) ? G[j + 1] : 0.0;
    S.coef_d2[j] = G[j] - (rho[j + 1] / rho[j]) * cn;
  }
}

__global__ void __launch_bounds__(COEF_THREADS) k_ms_coef(const SysDev* __restrict__ sys, int nsys,
                                                 int launched, const MsParams mp_,
                                                 const ResEpoch re) {
  __shared__ CoefLds L;
  const int s = blockIdx.x;
  if (s >= nsys) return;
  if (s == 0 && re.sh) {  // the next resident launch's epochs
    const unsigned e = re.sh->epoch;
    __syncthreads();
    if (e > 0x70000000u) {  // start over: no word may hold an epoch that returns
      unsigned* q = (unsigned*)re.sh->part;
      constexpr int n = (sizeof(ResShared) - offsetof(ResShared, part)) / sizeof(unsigned);
      for (int k = threadIdx.x; k < n; k += blockDim.x) q[k] = 0u;
      if (threadIdx.x == 0) re.sh->epoch = 0u;
    } else if (threadIdx.x == 0) {
      re.sh->epoch = e + re.bump;
    }
  }
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const MsParams* mp = &mp_;
  const int np = mp->np;
  const int cap = mp->cap;
  if (threadIdx.x == 0) {
    int N;
    if (S.h_ctl[0]) {
      N = S.h_ctl[1];
      if (S.h_ctl[2]) S.h_ctl[3] |= 1 << S.h_ctl[2];
    } else {  // not finished within the launched iterations: use what exists
      N = launched > 0 ? launched - 1 : 0;
      S.h_ctl[1] = N;
      S.h_ctl[3] |= 1 << 2;
    }
    L.N = N;
  }
  for (int k = threadIdx.x; k < MAXP; k += blockDim.x) L.res[k] = 0.0;
  __syncthreads();
  const int N = L.N;
  if (N <= COEF_LDS_ITERS) {
    // stage rows 0..N of the history (coalesced)
    const double* zeta = S.h_zeta;
    stage_in((N + 1) * MAXP, [&](int q) { return ldg(zeta, q); },
             [&](int q, double v) { L.zeta[q] = v; },
             [&]() {
               for (int j = threadIdx.x; j <= N; j += blockDim.x) {
                 L.rho[j] = S.h_rho[j];
                 L.alpha[j] = S.h_alpha[j];
                 L.act[j] = S.h_active[j];
               }
             });
    __syncthreads();
    // N_k, the first iteration with shift k inactive: one wave per shift, a ballot per
    // 64 iterations
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    for (int k = threadIdx.x >> 6; k < np; k += nw) {
      int nk = N;
      for (int j0 = 0; j0 < N; j0 += 64) {
        const int j = j0 + lane;
        const unsigned long long m = __ballot(j < N && !(L.act[j] & (1u << k)));
        if (m) {
          nk = j0 + __ffsll((long long)m) - 1;
          break;
        }
      }
      if (lane == 0) L.nk[k] = nk;
    }
    for (int j = threadIdx.x; j < N; j += blockDim.x) L.g[j] = L.rho[j + 1] / L.rho[j];
    __syncthreads();
    // the recurrence factors alpha_{j,k}, beta_{j,k} for every (k, j) at once; the
    // per-shift chains below are then multiply-adds on LDS operands, read eight
    // iterations at a time (one by one, each waited for, N = 111 took 14 us, not 6)
    for (int q = threadIdx.x; q < np * N; q += blockDim.x) {
      const int k = q / N, j = q - k * N;
      const double zj = L.zeta[j * MAXP + k];
      const double zr = L.zeta[(j + 1) * MAXP + k] / zj;
      L.u[k][j] = L.alpha[j] * zr;
      L.cp[k][j] = L.g[j] * zr * zr;
    }
    __syncthreads();
    const double rho0 = L.rho[0];
    for (int k = threadIdx.x; k < np; k += blockDim.x) {
      const int Nk = L.nk[k];
      const double ck = mp->coef[k];
      double Sk = 0.0;
      for (int j = Nk - 1; j >= 0; j -= 8) {  // the last eight may reach below 0
        double u[8], b[8], z[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int q = max(j - i, 0);
          u[i] = L.u[k][q];
          b[i] = L.cp[k][q];
          z[i] = L.zeta[q * MAXP + k];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          Sk = u[i] + b[i] * Sk;
          u[i] = ck * z[i] * Sk;  // term (k, j - i)
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (j >= i) L.u[k][j - i] = u[i];
      }
      for (int j = Nk; j < N; ++j) L.u[k][j] = 0.0;
      if (rho0 > 0.0) L.res[k] = fabs(L.zeta[Nk * MAXP + k]) * sqrt(L.rho[Nk] / rho0);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < N; j += blockDim.x) {
      double c = 0.0;
      for (int k = 0; k < np; ++k) c += L.u[k][j];
      L.c[j] = c;
      S.coef_c[j] = c;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < N; j += blockDim.x) {
      const double cn = (j + 1 < N) ? L.c[j + 1] : 0.0;
      S.coef_d[j] = L.c[j] - L.g[j] * cn;
    }
    if (S.coef_d2 && N > 0)
      coef_second(S, mp, N, L.rho, L.alpha, &L.u[0][0], &L.cp[0][0], L.g, L.td, L.to,
                  COEF_LDS_ITERS + 1);
  } else {
    // long histories read global memory (terms through the entry's coef_term)
    const double* rho = S.h_rho;
    const double* alph = S.h_alpha;
    const double* zeta = S.h_zeta;
    const double rho0 = rho[0];
    for (int k = threadIdx.x; k < np; k += blockDim.x) {
      int Nk = N;
      for (int j = 0; j < N; ++j)
        if (!(S.h_active[j] & (1u << k))) { Nk = j; break; }
      double Sk = 0.0;
      for (int j = Nk - 1; j >= 0; --j) {
        const double zj = zeta[(size_t)j * MAXP + k];
        const double zr = zeta[(size_t)(j + 1) * MAXP + k] / zj;
        const double aj = alph[j] * zr;
        const double bj = (rho[j + 1] / rho[j]) * zr * zr;
        Sk = aj + bj * Sk;
        S.coef_term[(size_t)k * cap + j] = mp->coef[k] * zj * Sk;
      }
      for (int j = Nk; j < N; ++j) S.coef_term[(size_t)k * cap + j] = 0.0;
      if (rho0 > 0.0) L.res[k] = fabs(zeta[(size_t)Nk * MAXP + k]) * sqrt(rho[Nk] / rho0);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < N; j += blockDim.x) {
      double c = 0.0;
      for (int k = 0; k < np; ++k) c += S.coef_term[(size_t)k * cap + j];
      S.coef_c[j] = c;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < N; j += blockDim.x) {
      const double cn = (j + 1 < N) ? S.coef_c[j + 1] : 0.0;
      S.coef_d[j] = S.coef_c[j] - (rho[j + 1] / rho[j]) * cn;
    }
    if (S.coef_d2 && N > 0) {
      __syncthreads();  // the terms are consumed: coef_term becomes TO
      coef_second(S, mp, N, rho, alph, S.coef_sq, S.coef_sq + (size_t)MAXP * cap,
                  S.coef_sq + (size_t)2 * MAXP * cap, S.coef_sq + (size_t)2 * MAXP * cap + cap,
                  S.coef_term, cap);
    }
  }
  if (threadIdx.x == 0) {  // statistics, off the critical path
    double mx = 0.0;
    for (int k = 0; k < np; ++k) mx = fmax(mx, L.res[k]);
    S.dstat[0] = mx;
    S.stat[0] += N;
    S.stat[1] += 1;
    if (N > S.stat[2]) S.stat[2] = N;
    if (N > S.stat[3]) S.stat[3] = N;  // max N since the host last cleared it
  }
}

// ---------------------------------------------- combination + epilogues
enum EpiMode {
  EPI_SIGN = 0,     // out = eps
  EPI_DOV = 1,      // out = psi + g5 eps
  EPI_DOVDAG = 2,   // out = psi + eps            (multi-shift source was g5 psi)
  EPI_M = 3,        // out = psi + g5 eps + Y psi;   out2 = g5 out;  partial |out|^2
  EPI_MDAG = 4,     // out = psi + eps + Y^dag psi
  EPI_MDAG_CG = 5,  // q = psi + eps + Y^dag psi;  x += alpha p;  r -= alpha q;  partial |r|^2
  EPI_MDAG_RES = 6  // r64 = b - (psi + eps + Y^dag psi) (+ low-precision copy in cg_r); partial |r64|^2
};

// c+ = m + g phi, c- = m* + g* phi*;  Y psi = c- psi_{0,1} (P-) + c+ psi_{2,3} (P+).
// Like the other kernels without neighbours, k_ms_combine takes its workgroups as dispatched,
// round-robin over the XCDs: in a batch whose members finish one by one, contiguous shares
// leave the XCDs of the finished ones idle.
// A site's sum runs over jw groups of threads, each with every jw-th pair of basis fields,
// added up in LDS (jw > 1 for small lattices, whose one thread per site leaves the chip idle
// and waits for memory N / 2 times: launch_combine).  aos: 1 psi is the caller's io_in,
// 2 the result goes to io_out.
template <class R>
__global__ void __launch_bounds__(512) k_ms_combine(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                     int mode, int jw, int aos) {
  __shared__ double lds[17];
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const Geo g = S.g;
  const int V = g.V;
  const size_t slot = (size_t)4 * V;
  const int N = S.h_ctl[1];
  const double* __restrict__ d = S.coef_d;
  const c2<R>* basis = (const c2<R>*)S.basis;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double alpha = 0.0;
  if (mode == EPI_MDAG_CG) alpha = S.cg_s[CG_ALPHA];
  double acc = 0.0;
  const int nt = blockDim.x / jw;  // sites at a time
  const int grp = threadIdx.x / nt, tl = threadIdx.x - grp * nt;
  for (int ib = i0; ib < i1; ib += nt) {
    const bool on = ib + tl < i1;
    const int i = on ? ib + tl : i1 - 1;
    double2 e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = double2{0.0, 0.0};
    int j = 2 * grp;
    for (; j + 1 < N; j += 2 * jw) {
      const double d0 = d[j], d1 = d[j + 1];
      const c2<R>* b0 = basis + (size_t)j * slot;
      const c2<R>* b1 = b0 + slot;
      c2<R> v0[4], v1[4];
      load_sp<R>(b0, V, i, v0);
      load_sp<R>(b1, V, i, v1);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        e[k].x += d0 * (double)v0[k].x + d1 * (double)v1[k].x;
        e[k].y += d0 * (double)v0[k].y + d1 * (double)v1[k].y;
      }
    }
    if (j < N) {
      const double d0 = d[j];
      c2<R> v0[4];
      load_sp<R>(basis + (size_t)j * slot, V, i, v0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        e[k].x += d0 * (double)v0[k].x;
        e[k].y += d0 * (double)v0[k].y;
      }
    }
    if (jw > 1) {
      double2* part = (double2*)dyn_lds;  // [group - 1][component][site]
      if (ib > i0) __syncthreads();
      if (grp > 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) part[((grp - 1) * 4 + k) * nt + tl] = e[k];
      __syncthreads();
      if (grp > 0) continue;
      for (int q = 0; q < jw - 1; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double2 v = part[(q * 4 + k) * nt + tl];
          e[k].x += v.x;
          e[k].y += v.y;
        }
    }
    if (!on) continue;
    auto write = [&](const c2<R> v[4]) {
      if constexpr (sizeof(R) == sizeof(double)) {
        if (aos & 2) {
#pragma unroll
          for (int k = 0; k < 4; ++k) stg2<double>(S.io_out, (size_t)i * 4 + k, v[k]);
          return;
        }
      }
      store_sp<R>((c2<R>*)S.e_out, V, i, v);
    };
    if (mode == EPI_SIGN) {
      c2<R> o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = c2<R>{(R)e[k].x, (R)e[k].y};
      write(o);
      continue;
    }
    c2<R> p[4];
    if constexpr (sizeof(R) == sizeof(double)) {
      if (aos & 1)
        load_io(S.io_in, i, p);
      else
        load_sp<R>((const c2<R>*)S.e_in, V, i, p);
    } else {
      load_sp<R>((const c2<R>*)S.e_in, V, i, p);
    }
    double2 o[4];
    if (mode == EPI_DOV || mode == EPI_M) {
      o[0] = double2{(double)p[0].x - e[0].x, (double)p[0].y - e[0].y};
      o[1] = double2{(double)p[1].x - e[1].x, (double)p[1].y - e[1].y};
      o[2] = double2{(double)p[2].x + e[2].x, (double)p[2].y + e[2].y};
      o[3] = double2{(double)p[3].x + e[3].x, (double)p[3].y + e[3].y};
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = double2{(double)p[k].x + e[k].x, (double)p[k].y + e[k].y};
    }
    if (mode >= EPI_M) {
      const double2 ph = S.phi[i];
      // c+ = m + g phi ; c- = conj(m) + conj(g) conj(phi)
      double cpr = S.m_re + S.g_re * ph.x - S.g_im * ph.y;
      double cpi = S.m_im + S.g_re * ph.y + S.g_im * ph.x;
      double cmr = S.m_re + S.g_re * ph.x - S.g_im * ph.y;
      double cmi = -S.m_im - (S.g_re * ph.y + S.g_im * ph.x);
      if (mode != EPI_M) { cpi = -cpi; cmi = -cmi; }  // adjoint: conjugate coefficients
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double cr = (k < 2) ? cmr : cpr, ci = (k < 2) ? cmi : cpi;
        const double pr = (double)p[k].x, pi = (double)p[k].y;
        o[k].x += cr * pr - ci * pi;
        o[k].y += cr * pi + ci * pr;
      }
    }
    if (mode == EPI_MDAG_CG) {
      // x += alpha p ; r -= alpha q
      c2<R> xv[4], pv[4], rv[4];
      load_sp<R>((const c2<R>*)S.cg_x, V, i, xv);
      load_sp<R>((const c2<R>*)S.cg_p, V, i, pv);
      load_sp<R>((const c2<R>*)S.cg_r, V, i, rv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        xv[k] = c2<R>{(R)((double)xv[k].x + alpha * (double)pv[k].x),
                      (R)((double)xv[k].y + alpha * (double)pv[k].y)};
        rv[k] = c2<R>{(R)((double)rv[k].x - alpha * o[k].x), (R)((double)rv[k].y - alpha * o[k].y)};
      }
      store_sp<R>((c2<R>*)S.cg_x, V, i, xv);
      store_sp<R>((c2<R>*)S.cg_r, V, i, rv);
      acc += norm2_sp(rv);
      continue;
    }
    if (mode == EPI_MDAG_RES) {
      double2 rr[4];
      const double2* b = S.cg_b;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double2 bv = b[(size_t)i * 4 + k];
        rr[k] = double2{bv.x - o[k].x, bv.y - o[k].y};
      }
      store_sp<double>((double2*)S.cg_r64, V, i, rr);
      if (S.cg_r) {
        c2<R> lo[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) lo[k] = c2<R>{(R)rr[k].x, (R)rr[k].y};
        store_sp<R>((c2<R>*)S.cg_r, V, i, lo);
      }
      acc += norm2_sp(rr);
      continue;
    }
    c2<R> ov[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) ov[k] = c2<R>{(R)o[k].x, (R)o[k].y};
    write(ov);
    if (mode == EPI_M) {
      acc += norm2_sp(ov);
      if (S.e_out2) {
        c2<R> g5o[4] = {c2<R>{-ov[0].x, -ov[0].y}, c2<R>{-ov[1].x, -ov[1].y}, ov[2], ov[3]};
        store_sp<R>((c2<R>*)S.e_out2, V, i, g5o);
      }
    }
  }
  if (mode == EPI_M || mode == EPI_MDAG_CG || mode == EPI_MDAG_RES) {
    const double tot = block_sum(acc, lds);
    if (threadIdx.x == 0) {
      if (S.part_c) S.part_c[lb] = tot;
      if (mode == EPI_M && S.part_b) S.part_b[lb] = tot;  // rho_0 of the next multi-shift
    }
  }
}

// ------------------------------------------------------- multi-shift setup
// Source partials |src|^2 -> part_b (and src = g5 e_in when g5_src).
template <class R>
__global__ void __launch_bounds__(256) k_ms_prep(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                  int nb_total, int g5_src) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  // optional: src = g5 * e_in  (writes the multi-shift source buffer)
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    c2<R> v[4];
    if (g5_src) {
      load_sp<R>((const c2<R>*)S.e_in, V, i, v);
      v[0] = c2<R>{-v[0].x, -v[0].y};
      v[1] = c2<R>{-v[1].x, -v[1].y};
      store_sp<R>((c2<R>*)S.src, V, i, v);
    } else {
      load_sp<R>((const c2<R>*)S.src, V, i, v);
    }
    acc += norm2_sp(v);
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_b[lb] = tot;
}

// Deterministic synthetic field for tuning runs: a hash of the site and spin
// mapped to [-1, 1) in both components, written to src.
template <class R>
__global__ void __launch_bounds__(256) k_fill(const SysDev* __restrict__ sys,
                                              const int* __restrict__ bmap, int nb_total) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  c2<R>* out = (c2<R>*)S.src;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      unsigned int h = (unsigned int)(i * 4 + k) * 2654435761u + 0x9e3779b9u;
      h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
      const unsigned int h2 = h * 3266489917u + 374761393u;
      out[(size_t)k * V + i] = c2<R>{(R)((double)(h & 0xffffff) / 8388608.0 - 1.0),
                                     (R)((double)(h2 & 0xffffff) / 8388608.0 - 1.0)};
    }
  }
}

// ------------------------------------------------- momentum-space operators
// The theory has no gauge field, so every translation-invariant operator built
// from H_W is diagonal in momentum space (the FFT route of Sec. 7.2).  For a
// field ~ exp(+i p.x), D_W(p) = w + i gamma.s with w = 4 - M0 - sum cos p_mu,
// s_mu = sin p_mu, H_W(p)^2 = s2 = w^2 + |s|^2.  Every Dirac operator form is
//   D(p) = a0 + i c gamma.s :
//   overlap, rational sign R = sum_k a_k / (s2 + b_k):  a0 = 1 + R w, c = R;
//   overlap, exact sign R = 1 / sqrt(s2):                a0 = 1 + R w, c = R;
//   Dslash = (1 - D_ov/2)^-1 D_ov (exact sign, Sec. 2.2): a0 = 0,
//     c = 2 / (sqrt(s2) - w) = 2 (sqrt(s2) + w) / |s|^2  (finite when no momentum
//     has every component in {0, pi}: antiperiodic time, T even).
// The free fermion matrix of the preconditioner (Sec. 7.3),
//   M0 = D + m P+ + m* P- = a + i mu g5 + i c gamma.s,  a = a0 + Re m, mu = Im m,
// has M0^-1 = (a - i mu g5 - i c gamma.s) / (a^2 + mu^2 + c^2 |s|^2), and M0^-dag
// the same with + signs.
// Fields go through per-axis DFTs of L <= 64 points: forward e^{-2 pi i j k/L},
// inverse e^{+2 pi i j k/L} with 1/V.  Antiperiodic time is handled by the
// twist e^{-i pi t/T} before the forward and e^{+i pi t/T} after the inverse
// transform, which puts p_t on (2n+1) pi / T.
// SYM_PCG: the scalar (M0^dag M0)^-1 = M0^-1 M0^-dag of the free-field operator, the
// preconditioner of CG on MdagM (Sec. 7.3 in its split form; same iterates).
enum SymKind { SYM_D = 0, SYM_D_DAG = 1, SYM_M0INV = 2, SYM_M0INV_DAG = 3, SYM_BOSON = 4,
               SYM_PCG = 5 };
enum DiracForm { DIRAC_RATIONAL = 0, DIRAC_EXACT = 1, DIRAC_DSLASH = 2 };

struct SymParams {
  int kind;
  int form;           // DiracForm
  int periodic;       // 1: periodic time (scalar fields) whatever the fermion boundary
  int np;
  double diag;        // 4 - M0
  double a[MAXP];     // residues a_k of the sign rational
  double b[MAXP];     // shifts b_k
};

// System of workgroup b in a transform pass (which: 0 xy, 1 z, 2 t).
__device__ __forceinline__ int find_sys(const SysDev* __restrict__ sys, int nsys, int b, int which) {
  int s = 0;
  for (int k = 1; k < nsys; ++k) {
    const int o = which == 0   ? sys[k].off_xy
                  : which == 1 ? sys[k].off_z
                  : which == 2 ? sys[k].off_t
                               : sys[k].off_zt;
    if (o <= b) s = k;
  }
  return s;
}

// Twiddle table e^{sgn 2 pi i j / L}, evaluated in FP64 and stored in the transform's
// precision (an FP32 transform reads 8-byte entries from LDS).
template <class R>
__device__ __forceinline__ void twiddles(c2<R>* tw, int L, double sgn) {
  for (int j = threadIdx.x; j < L; j += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * (double)j / (double)L, &sn, &cs);
    tw[j] = c2<R>{(R)cs, (R)(sgn * sn)};
  }
}

// W' = m phi + g phi^2 / 2 at a site.
__device__ __forceinline__ double2 w_prime(const SysDev& S, double2 f) {
  const double lr = 0.5 * S.g_re, li = 0.5 * S.g_im;
  const double f2r = f.x * f.x - f.y * f.y, f2i = 2.0 * f.x * f.y;
  return double2{S.m_re * f.x - S.m_im * f.y + lr * f2r - li * f2i,
                 S.m_re * f.y + S.m_im * f.x + lr * f2i + li * f2r};
}

// What a transform reads and writes.
struct SymIo {
  int in = 0;   // 0: planar e_in; 1: the caller's io_in; 2: phi, W', conj W' of phi
  int out = 0;  // 0: planar e_out; 1: the caller's io_out
  int yuk = 0;  // 1, 2: adds Y psi, Y^dag psi, psi the field read (k_yuk)
  int zt = 0;   // fft_tmp holds a site line (z, t) after the other (k_fft_zt), else planes
};

// e / d for 0 <= e < 2^16, 1 <= d < 2^16 by a multiplication (e (d - 1) < 2^32).
struct SmallDiv {
  unsigned m;
  int d;
  __device__ __forceinline__ explicit SmallDiv(int d_) : m(0xffffffffu / (unsigned)d_ + 1u), d(d_) {}
  __device__ __forceinline__ int div(int e) const {
    return d == 1 ? e : (int)__umulhi((unsigned)e, m);
  }
};

// Values k = g, N - g, N/2 - g and N/2 + g of the transform of one line of even length N
// (elements a[j st] in LDS, twiddles tw[m] = (cos, sin) 2 pi m / N, sgn the exponent's sign),
// 0 <= g <= N/4 (all values over all g; the ends of the range give two values twice).  With
// s_j = a_j + a_{N-j}, d_j = a_j - a_{N-j} the four share their sums over even and odd j,
//   X_k = a_0 + (-1)^k a_{N/2} + sum_j s_j cos(2 pi j k / N) + i sgn sum_j d_j sin(2 pi j k / N):
// 3 N / 8 LDS reads and N / 2 real multiplications per value, where the plain sum takes 2 N
// and 4 N (LDS reads bound these passes).
template <class R>
__host__ __device__ __forceinline__ void line_dft(const c2<R>* a, int st, int N, const c2<R>* tw, int g,
                                         R sgn, c2<R> o[4]) {
  const int h = N >> 1;
  const c2<R> a0 = a[0], ah = a[h * st];
  c2<R> ce{R(0), R(0)}, co = ce, de = ce, dd = ce;
  const c2<R>* p = a + st;
  const c2<R>* q = a + (N - 1) * st;
  int m = 0;
#pragma unroll 2
  for (int j = 1; j < h; j += 2) {
    m += g;
    if (m >= N) m -= N;
    {
      const c2<R> u = *p, v = *q, w = tw[m];
      co.x += (u.x + v.x) * w.x;
      co.y += (u.y + v.y) * w.x;
      dd.x += (u.x - v.x) * w.y;
      dd.y += (u.y - v.y) * w.y;
    }
    if (j + 1 < h) {
      m += g;
      if (m >= N) m -= N;
      const c2<R> u = p[st], v = q[-st], w = tw[m];
      ce.x += (u.x + v.x) * w.x;
      ce.y += (u.y + v.y) * w.x;
      de.x += (u.x - v.x) * w.y;
      de.y += (u.y - v.y) * w.y;
    }
    p += 2 * st;
    q -= 2 * st;
  }
  const R s0 = g & 1 ? R(-1) : R(1), s1 = (h - g) & 1 ? R(-1) : R(1);
  const c2<R> c0{a0.x + s0 * ah.x + (ce.x + co.x), a0.y + s0 * ah.y + (ce.y + co.y)};
  const c2<R> c1{a0.x + s1 * ah.x + (ce.x - co.x), a0.y + s1 * ah.y + (ce.y - co.y)};
  const c2<R> d0{sgn * (de.x + dd.x), sgn * (de.y + dd.y)};
  const c2<R> d1{sgn * (dd.x - de.x), sgn * (dd.y - de.y)};
  o[0] = c2<R>{c0.x - d0.y, c0.y + d0.x};
  o[1] = c2<R>{c0.x + d0.y, c0.y - d0.x};
  o[2] = c2<R>{c1.x - d1.y, c1.y + d1.x};
  o[3] = c2<R>{c1.x + d1.y, c1.y - d1.x};
}
__host__ __device__ inline int dft_groups(int N) { return N / 4 + 1; }
// The four places of group g in the line (stride st).
__host__ __device__ __forceinline__ void dft_places(int N, int g, int st, int k[4]) {
  k[0] = g * st;
  k[1] = g > 0 ? (N - g) * st : 0;
  k[2] = (N / 2 - g) * st;
  k[3] = (N / 2 + g) * st;
}

// LDS of the xy pass: the rows of a plane one value longer than X (lanes of different rows
// read different banks), the components' planes 2 mod 8 values apart (so do the four
// components of a site).
__host__ __device__ inline int fft_xy_plane(int X, int Y) { return Y * (X + 1) + (10 - Y * (X + 1) % 8) % 8; }

// x and y axes of one (z, t) plane, all NS components.  inv = 0: the field -> fft_tmp; inv = 1:
// fft_tmp -> the result; either with the time twist of the direction, the inverse with
// 1/V.  Needs X, Y <= 64, X Y <= 1024, and 2 NS fft_xy_plane + X + Y + 1 values of LDS.  All
// components, so that the caller's layout is read and written here, in whole lines.  Bound
// by latency: 12.3 us in a kernel trace on 16^3 x 32 in FP64 (512 workgroups), 8.5 of them by
// the clocks of a workgroup: 2 until the field is there, 1.8 for each axis, 2.5 for the store;
// one component per workgroup and plain sums took 15, and pack, k_yuk and unpack 19 more.
template <class R, int NS>
__global__ void __launch_bounds__(512) k_fft_xy(const SysDev* __restrict__ sys, int nsys, int inv,
                                                int periodic, const SymIo io) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const SysDev& S = sys[find_sys(sys, nsys, blockIdx.x, 0)];
  if (S.active && *S.active == 0) return;
  const int X = S.g.X, Y = S.g.Y, Z = S.g.Z, T = S.g.T, V = S.g.V;
  const int zt = blockIdx.x - S.off_xy;  // z + Z t
  const int t = zt / Z;
  const int XY = X * Y, ZT = Z * T, P = X + 1, SP = fft_xy_plane(X, Y);
  const SmallDiv dX(X), dXY(XY);
  const size_t base = (size_t)zt * XY;
  c2<R>* A = (c2<R>*)dyn_lds;
  c2<R>* B = A + NS * SP;
  c2<R>* twx = B + NS * SP;
  c2<R>* twy = twx + X;
  double2* const tws = (double2*)(twy + Y);  // e^{-+ i pi t / T}, 1 / V
  auto between = [&]() {
    for (int j = threadIdx.x; j < X + Y; j += blockDim.x) {
      double sn, cs;
      sincospi(j < X ? 2.0 * j / X : 2.0 * (j - X) / Y, &sn, &cs);
      twx[j] = c2<R>{(R)cs, (R)sn};
    }
    if (threadIdx.x == blockDim.x - 1) {  // the last wave: the first ones are busy above
      double2 w{1.0, 0.0};
      if (S.g.bc < 0 && !periodic) sincospi((inv ? 1.0 : -1.0) * t / T, &w.y, &w.x);
      const double f = inv ? 1.0 / V : 1.0;
      *tws = double2{w.x * f, w.y * f};
    }
  };
  auto cell = [&](int k, int i) -> c2<R>& {
    const int y = dX.div(i);
    return A[k * SP + y * P + (i - y * X)];
  };
  // value e of a plane whose sites hold their components side by side
  auto comp = [](int e) { return e % NS; };
  auto spot = [](int e) { return e / NS; };
  if (NS == 3 && !inv) {
    stage_in(XY, [&](int i) { return S.phi[base + i]; },
             [&](int i, double2 f) {
               const double2 w = w_prime(S, f);
               cell(0, i) = c2<R>{(R)f.x, (R)f.y};
               cell(1, i) = c2<R>{(R)w.x, (R)w.y};
               cell(2, i) = c2<R>{(R)w.x, -(R)w.y};
             },
             between);
  } else if (!inv && io.in == 1) {
    const double2* in = S.io_in + NS * base;
    stage_in(NS * XY, [&](int e) { return ldg2<double>(in, e); },
             [&](int e, double2 v) { cell(comp(e), spot(e)) = c2<R>{(R)v.x, (R)v.y}; }, between);
  } else if (inv && io.zt) {
    const c2<R>* in = (const c2<R>*)S.fft_tmp;
    stage_in(NS * XY,
             [&](int e) { return ldg2<R>(in, ((size_t)spot(e) * ZT + zt) * NS + comp(e)); },
             [&](int e, c2<R> v) { cell(comp(e), spot(e)) = v; }, between);
  } else {
    const c2<R>* in = (const c2<R>*)(inv ? S.fft_tmp : S.e_in) + base;
    stage_in(NS * XY,
             [&](int e) {
               const int k = dXY.div(e);
               return ldg2<R>(in, (size_t)k * V + (e - k * XY));
             },
             [&](int e, c2<R> v) {
               const int k = dXY.div(e);
               cell(k, e - k * XY) = v;
             },
             between);
  }
  __syncthreads();
  const R sgn = inv ? R(1) : R(-1);
  const SmallDiv dY(Y), dlx(NS * Y), dly(NS * X);
  int at[4];
  c2<R> o[4];
  for (int it = threadIdx.x; it < NS * Y * dft_groups(X); it += blockDim.x) {  // x axis
    const int g = dlx.div(it), ln = it - g * (NS * Y);
    const int k = dY.div(ln), row = k * SP + (ln - k * Y) * P;
    line_dft<R>(A + row, 1, X, twx, g, sgn, o);
    dft_places(X, g, 1, at);
#pragma unroll
    for (int q = 0; q < 4; ++q) B[row + at[q]] = o[q];
  }
  __syncthreads();
  const bool staged = inv ? io.out == 1 || io.yuk : io.zt;  // out through LDS
  c2<R>* out = (c2<R>*)(inv ? S.e_out : S.fft_tmp) + base;
  const double2 w = *tws;
  for (int it = threadIdx.x; it < NS * X * dft_groups(Y); it += blockDim.x) {  // y axis
    const int g = dly.div(it), ln = it - g * (NS * X);
    const int k = dX.div(ln), kx = ln - k * X;
    line_dft<R>(B + k * SP + kx, P, Y, twy, g, sgn, o);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      o[q] = c2<R>{(R)(o[q].x * w.x - o[q].y * w.y), (R)(o[q].x * w.y + o[q].y * w.x)};
    c2<R>* to = staged ? A + k * SP + kx : out + (size_t)k * V + kx;
    dft_places(Y, g, staged ? P : X, at);
    if (staged) {
#pragma unroll
      for (int q = 0; q < 4; ++q) A[k * SP + kx + at[q]] = o[q];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) to[at[q]] = o[q];
    }
  }
  if (!staged) return;
  __syncthreads();
  if (!inv) {
    c2<R>* tmp = (c2<R>*)S.fft_tmp + (size_t)zt * NS;
    for (int e = threadIdx.x; e < NS * XY; e += blockDim.x)
      tmp[(size_t)spot(e) * (ZT * NS) + comp(e)] = cell(comp(e), spot(e));
    return;
  }
  if constexpr (sizeof(R) == sizeof(double) && NS == 4) {  // operator calls on the caller's fields
    const bool aos = io.out == 1;
    auto k_of = [&](int e) { return aos ? e & 3 : dXY.div(e); };
    auto i_of = [&](int e) { return aos ? e >> 2 : e - XY * dXY.div(e); };
    auto write = [&](int e, double2 v) {
      if (aos)
        S.io_out[4 * base + e] = v;
      else
        ((double2*)out)[(size_t)k_of(e) * V + i_of(e)] = v;
    };
    if (!io.yuk) {
      for (int e = threadIdx.x; e < 4 * XY; e += blockDim.x) write(e, cell(k_of(e), i_of(e)));
      return;
    }
    struct PsiPhi {
      double2 psi, phi;
    };
    stage_in(4 * XY,
             [&](int e) {
               const size_t i = base + i_of(e);
               return PsiPhi{io.in == 1 ? ldg2<double>(S.io_in, 4 * i + k_of(e))
                                        : ldg2<double>((const double2*)S.e_in, k_of(e) * (size_t)V + i),
                             ldg2<double>(S.phi, i)};
             },
             [&](int e, const PsiPhi& p) {
               const int k = k_of(e);
               const double2 v = cell(k, i_of(e));
               const double cr = S.m_re + S.g_re * p.phi.x - S.g_im * p.phi.y;
               double ci = S.m_im + S.g_re * p.phi.y + S.g_im * p.phi.x;
               if ((k < 2) != (io.yuk == 2)) ci = -ci;
               write(e, double2{v.x + cr * p.psi.x - ci * p.psi.y, v.y + cr * p.psi.y + ci * p.psi.x});
             },
             []() {});
  }
}

// z axis of the (x, z) slab of one (y, t), all components, in place on fft_tmp.
// Needs Z <= 64, X Z <= 1024, and NS X Z + Z values of LDS.
template <class R, int NS>
__global__ void __launch_bounds__(512) k_fft_z(const SysDev* __restrict__ sys, int nsys, int inv) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const SysDev& S = sys[find_sys(sys, nsys, blockIdx.x, 1)];
  if (S.active && *S.active == 0) return;
  const int X = S.g.X, Y = S.g.Y, Z = S.g.Z, V = S.g.V;
  const int yt = blockIdx.x - S.off_z;  // y + Y t
  const int t = yt / Y, y = yt - t * Y;
  const int XZ = X * Z, XY = X * Y;
  const SmallDiv dX(X), dZ(Z), dl(NS * X);
  c2<R>* A = (c2<R>*)dyn_lds;
  c2<R>* tw = A + NS * XZ;
  c2<R>* f = (c2<R>*)S.fft_tmp + X * (y + Y * Z * t);
  stage_in(NS * XZ,
           [&](int e) {  // (k Z + z) X + x
             const int q = dX.div(e), k = dZ.div(q);
             return ldg2<R>((const c2<R>*)f, (size_t)k * V + (e - q * X) + XY * (q - k * Z));
           },
           [&](int e, c2<R> v) { A[e] = v; }, [&]() { twiddles<R>(tw, Z, 1.0); });
  __syncthreads();  // every read of f happens before it
  int at[4];
  c2<R> o[4];
  for (int it = threadIdx.x; it < NS * X * dft_groups(Z); it += blockDim.x) {
    const int g = dl.div(it), ln = it - g * (NS * X);
    const int k = dX.div(ln), x = ln - k * X;
    line_dft<R>(A + k * XZ + x, X, Z, tw, g, inv ? R(1) : R(-1), o);
    dft_places(Z, g, XY, at);
#pragma unroll
    for (int q = 0; q < 4; ++q) f[(size_t)k * V + x + at[q]] = o[q];
  }
}

// Free-field Dirac operator at one momentum: D = a0 + i c gamma.s (s_mu = sin p_mu,
// w the Wilson term), for the form's sign function.
__device__ __forceinline__ void free_symbol(const SymParams& sp, double s2sin, double w,
                                            double& a0, double& c) {
  const double s2 = w * w + s2sin;
  if (sp.form == DIRAC_DSLASH) {
    const double sq = sqrt(s2);
    a0 = 0.0;
    c = (w > 0.0) ? 2.0 * (sq + w) / s2sin : 2.0 / (sq - w);
  } else {
    double Rr = 0.0;
    if (sp.form == DIRAC_EXACT) {
      Rr = 1.0 / sqrt(s2);
    } else {
      for (int k = 0; k < sp.np; ++k) Rr += sp.a[k] / (s2 + sp.b[k]);
    }
    a0 = 1.0 + Rr * w;
    c = Rr;
  }
}

// The preconditioner of CG on MdagM at one momentum: M0^dag M0 = (a^2 + mu^2 + c^2 |s|^2) 1
// is a scalar (a shifted solve takes the free shifted operator, M0^dag M0 + sigma), so
// P = (M0^dag M0 + sigma)^-1 is one number per momentum.
__device__ __forceinline__ double pcg_scale(const SymParams& sp, double m_re, double m_im,
                                            double shift, double s2sin, double w) {
  double a0, c;
  free_symbol(sp, s2sin, w, a0, c);
  const double A = a0 + m_re;
  return 1.0 / (A * A + m_im * m_im + c * c * s2sin + shift);
}

// Momentum-space operator on the four spin components v of one momentum.
__device__ __forceinline__ void apply_symbol(const SymParams& sp, double m_re, double m_im,
                                             double shift, double sx, double sy, double sz,
                                             double st, double w, double2 v[4]) {
  const double s2sin = sx * sx + sy * sy + sz * sz + st * st;
  if (sp.kind == SYM_PCG) {
    const double sc = pcg_scale(sp, m_re, m_im, shift, s2sin, w);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = double2{v[k].x * sc, v[k].y * sc};
    return;
  }
  double a0, c;
  free_symbol(sp, s2sin, w, a0, c);
  // out = (A v + i (cg gamma.s v + c5 g5 v)) * scale
  double A = a0, cg = c, c5 = 0.0, scale = 1.0;
  if (sp.kind == SYM_D_DAG) {
    cg = -c;
  } else if (sp.kind == SYM_M0INV || sp.kind == SYM_M0INV_DAG) {
    A = a0 + m_re;
    const double sg = sp.kind == SYM_M0INV ? -1.0 : 1.0;
    cg = sg * c;
    c5 = sg * m_im;
    scale = 1.0 / (A * A + m_im * m_im + c * c * s2sin);
  }
  // G = gamma.s v in the basis of Sec. 2.1 (the one of the Wilson stencil)
  double2 G[4];
  G[0] = double2{-sx * v[3].y + sy * v[3].x - sz * v[2].y + st * v[2].x,
                 sx * v[3].x + sy * v[3].y + sz * v[2].x + st * v[2].y};
  G[1] = double2{-sx * v[2].y - sy * v[2].x + sz * v[3].y + st * v[3].x,
                 sx * v[2].x - sy * v[2].y - sz * v[3].x + st * v[3].y};
  G[2] = double2{sx * v[1].y - sy * v[1].x + sz * v[0].y + st * v[0].x,
                 -sx * v[1].x - sy * v[1].y - sz * v[0].x + st * v[0].y};
  G[3] = double2{sx * v[0].y + sy * v[0].x - sz * v[1].y + st * v[1].x,
                 -sx * v[0].x + sy * v[0].y + sz * v[1].x + st * v[1].y};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double g5 = k < 2 ? -1.0 : 1.0;
    const double hr = cg * G[k].x + c5 * g5 * v[k].x;
    const double hi = cg * G[k].y + c5 * g5 * v[k].y;
    v[k] = double2{(A * v[k].x - hi) * scale, (A * v[k].y + hr) * scale};
  }
}

// The operator of a transform pass at one momentum, from (sin, cos) of its components.
__device__ __forceinline__ void site_symbol(const SymParams& sp, const SysDev& S, double2 px,
                                            double2 py, double2 pz, double2 pt, double2 v[4]) {
  const double w = sp.diag - (px.y + py.y + pz.y + pt.y);
  if (sp.kind == SYM_BOSON) {
    // scalar fields in planes 0-2: D_2 = 1 + w/s (scalar part of the exact overlap
    // operator), then 1 - D_2/2 twice
    const double d2 =
        1.0 + w / sqrt(w * w + px.x * px.x + py.x * py.x + pz.x * pz.x + pt.x * pt.x);
    v[0] = double2{d2 * v[0].x, d2 * v[0].y};
    const double k2 = 1.0 - 0.5 * d2;
    v[1] = double2{k2 * v[1].x, k2 * v[1].y};
    v[2] = double2{k2 * v[2].x, k2 * v[2].y};
  } else {
    const bool m0 = sp.kind == SYM_M0INV || sp.kind == SYM_M0INV_DAG || sp.kind == SYM_PCG;
    apply_symbol(sp, m0 ? S.pc_re : S.m_re, m0 ? S.pc_im : S.m_im, S.shift, px.x, py.x, pz.x,
                 pt.x, w, v);
  }
}

// t axis forward, the momentum-space operator on all components, t axis
// inverse, in place on fft_tmp.  Workgroup: (chunk of xc x values, y, z);
// needs T <= 64 and xc T <= 256.
template <class R, int NS>
__global__ void __launch_bounds__(256) k_fft_t_sym(const SysDev* __restrict__ sys, int nsys,
                                                   const SymParams sp) {
  __shared__ c2<R> A[1024], B[1024];
  __shared__ c2<R> tw[64];
  __shared__ double2 csx[64], cst[64];  // (sin, cos) of the block's x momenta and of every t momentum
  const SysDev& S = sys[find_sys(sys, nsys, blockIdx.x, 2)];
  if (S.active && *S.active == 0) return;
  const int X = S.g.X, Y = S.g.Y, Z = S.g.Z, T = S.g.T, V = S.g.V;
  const int XC = S.xc;
  const int loc = blockIdx.x - S.off_t;
  const int nxc = X / XC;
  const int xb = (loc % nxc) * XC;
  const int yz = loc / nxc;  // y + Y z
  const int z = yz / Y, y = yz - z * Y;
  const SmallDiv dC(XC), dT(T), dl(NS * XC);
  c2<R>* f = (c2<R>*)S.fft_tmp + xb + X * (y + Y * z);
  const int XYZ = X * Y * Z;
  double2 py, pz;
  stage_in(NS * XC * T,  // element e = (k T + t) XC + xl
           [&](int e) {
             const int q = dC.div(e), k = dT.div(q);
             return ldg2<R>((const c2<R>*)f,
                            (size_t)k * V + (e - q * XC) + (size_t)XYZ * (q - k * T));
           },
           [&](int e, c2<R> v) { A[e] = v; },
           [&]() {
             const double shift = S.g.bc < 0 && !sp.periodic ? 1.0 : 0.0;
             for (int j = threadIdx.x; j < 2 * T + XC; j += blockDim.x) {
               double2 sc;
               const double a = j < T       ? 2.0 * j / T
                                : j < 2 * T ? (2.0 * (j - T) + shift) / T
                                            : 2.0 * (xb + j - 2 * T) / X;
               sincospi(a, &sc.x, &sc.y);
               if (j < T) tw[j] = c2<R>{(R)sc.y, (R)sc.x};
               else if (j < 2 * T) cst[j - T] = sc;
               else csx[j - 2 * T] = sc;
             }
             sincospi(2.0 * y / Y, &py.x, &py.y);
             sincospi(2.0 * z / Z, &pz.x, &pz.y);
           });
  __syncthreads();
  int at[4];
  c2<R> o[4];
  const int lines = NS * XC, items = lines * dft_groups(T);
  for (int it = threadIdx.x; it < items; it += blockDim.x) {  // forward t
    const int g = dl.div(it), ln = it - g * lines;
    const int k = dC.div(ln), l0 = k * T * XC + (ln - k * XC);
    line_dft<R>(A + l0, XC, T, tw, g, R(-1), o);
    dft_places(T, g, XC, at);
#pragma unroll
    for (int q = 0; q < 4; ++q) B[l0 + at[q]] = o[q];
  }
  __syncthreads();
  for (int q = threadIdx.x; q < XC * T; q += blockDim.x) {  // operator at (kx, ky, kz, kt)
    const int kt = dC.div(q), xl = q - kt * XC;
    double2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const c2<R> u = k < NS ? B[(k * T + kt) * XC + xl] : c2<R>{R(0), R(0)};
      v[k] = double2{(double)u.x, (double)u.y};
    }
    site_symbol(sp, S, csx[xl], py, pz, cst[kt], v);
#pragma unroll
    for (int k = 0; k < NS; ++k) A[(k * T + kt) * XC + xl] = c2<R>{(R)v[k].x, (R)v[k].y};
  }
  __syncthreads();
  for (int it = threadIdx.x; it < items; it += blockDim.x) {  // inverse t
    const int g = dl.div(it), ln = it - g * lines;
    const int k = dC.div(ln), xl = ln - k * XC;
    line_dft<R>(A + k * T * XC + xl, XC, T, tw, g, R(1), o);
    dft_places(T, g, XYZ, at);
#pragma unroll
    for (int q = 0; q < 4; ++q) f[(size_t)k * V + xl + at[q]] = o[q];
  }
}

// z and t axes of one (x, y) line, all components: forward, the momentum-space operator,
// inverse, in place on fft_tmp in the site-line order ((x y) T + t) Z + z with a site's
// components side by side.  One pass instead of three (k_fft_z twice and k_fft_t_sym): the
// line stays in LDS, 2 NS fft_xy_plane(Z, T) + Z + T values and 2 (Z + T) doubles.  Bound by
// the LDS reads of its sums: 16^3 x 32 in FP64 (256 workgroups) 17.6 us in a kernel trace, 14
// by the clocks of a workgroup: 3 for each t axis, 2 for each z axis, 1.3 for the operator; the
// three passes took 44.
template <class R, int NS>
__global__ void __launch_bounds__(1024) k_fft_zt(const SysDev* __restrict__ sys, int nsys,
                                                 const SymParams sp) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const SysDev& S = sys[find_sys(sys, nsys, blockIdx.x, 3)];
  if (S.active && *S.active == 0) return;
  const int X = S.g.X, Y = S.g.Y, Z = S.g.Z, T = S.g.T;
  const int xy = blockIdx.x - S.off_zt;
  const int ZT = Z * T, P = Z + 1, SP = fft_xy_plane(Z, T);
  const SmallDiv dZ(Z), dT(T), dlz(NS * T), dlt(NS * Z);
  double2* csz = (double2*)dyn_lds;  // (sin, cos) of every z and t momentum
  double2* cst = csz + Z;
  c2<R>* A = (c2<R>*)(cst + T);
  c2<R>* B = A + NS * SP;
  c2<R>* twz = B + NS * SP;
  c2<R>* twt = twz + Z;
  c2<R>* f = (c2<R>*)S.fft_tmp + (size_t)xy * ZT * NS;
  auto cell = [&](int e) -> c2<R>& {
    const int i = e / NS, k = e - i * NS, t = dZ.div(i);
    return A[k * SP + t * P + (i - t * Z)];
  };
  double2 px, py;
  stage_in(NS * ZT, [&](int e) { return ldg2<R>((const c2<R>*)f, e); },
           [&](int e, c2<R> v) { cell(e) = v; },
           [&]() {
             const double shift = S.g.bc < 0 && !sp.periodic ? 1.0 : 0.0;
             for (int j = threadIdx.x; j < Z + 2 * T; j += blockDim.x) {
               double2 sc;
               const double a = j < Z       ? 2.0 * j / Z
                                : j < Z + T ? 2.0 * (j - Z) / T
                                            : (2.0 * (j - Z - T) + shift) / T;
               sincospi(a, &sc.x, &sc.y);
               if (j < Z) csz[j] = sc;
               if (j < Z + T) twz[j] = c2<R>{(R)sc.y, (R)sc.x};
               else cst[j - Z - T] = sc;
             }
             const int y = xy / X;
             sincospi(2.0 * (xy - y * X) / X, &px.x, &px.y);
             sincospi(2.0 * y / Y, &py.x, &py.y);
           });
  int at[4];
  c2<R> o[4];
  // z lines (row (k, t)) and t lines (column (k, z)), from one buffer to the other
  auto z_axis = [&](const c2<R>* from, c2<R>* to, R sgn) {
    __syncthreads();
    for (int it = threadIdx.x; it < NS * T * dft_groups(Z); it += blockDim.x) {
      const int g = dlz.div(it), ln = it - g * (NS * T);
      const int k = dT.div(ln), row = k * SP + (ln - k * T) * P;
      line_dft<R>(from + row, 1, Z, twz, g, sgn, o);
      dft_places(Z, g, 1, at);
#pragma unroll
      for (int q = 0; q < 4; ++q) to[row + at[q]] = o[q];
    }
  };
  auto t_axis = [&](const c2<R>* from, c2<R>* to, R sgn) {
    __syncthreads();
    for (int it = threadIdx.x; it < NS * Z * dft_groups(T); it += blockDim.x) {
      const int g = dlt.div(it), ln = it - g * (NS * Z);
      const int k = dZ.div(ln), col = k * SP + (ln - k * Z);
      line_dft<R>(from + col, P, T, twt, g, sgn, o);
      dft_places(T, g, P, at);
#pragma unroll
      for (int q = 0; q < 4; ++q) to[col + at[q]] = o[q];
    }
  };
  z_axis(A, B, R(-1));
  t_axis(B, A, R(-1));
  __syncthreads();
  for (int i = threadIdx.x; i < ZT; i += blockDim.x) {  // operator at (kx, ky, kz, kt)
    const int kt = dZ.div(i), kz = i - kt * Z;
    c2<R>* a = A + kt * P + kz;
    double2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const c2<R> u = k < NS ? a[k * SP] : c2<R>{R(0), R(0)};
      v[k] = double2{(double)u.x, (double)u.y};
    }
    site_symbol(sp, S, px, py, csz[kz], cst[kt], v);
#pragma unroll
    for (int k = 0; k < NS; ++k) a[k * SP] = c2<R>{(R)v[k].x, (R)v[k].y};
  }
  t_axis(A, B, R(1));
  z_axis(B, A, R(1));
  __syncthreads();
  for (int e = threadIdx.x; e < NS * ZT; e += blockDim.x) f[e] = cell(e);
}

// ------------------------------------------- transforms of fixed length
// Lines of compile-time length N (N = 2^a 3^b) transformed in registers: mixed-radix
// Cooley-Tukey, decimation in time, every index a constant after unrolling, twiddles
// e^{sgn 2 pi i m / N} folded into the code from a constant table.

// cos and sin of 2 pi j / n at compile time: reduction to |r| <= pi/4 by quadrants,
// then the Taylor series (terms to r^25: below 1e-17 there).
struct CS {
  double c, s;
};
constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr CS ce_cossin(long long j, long long n) {
  j %= n;
  if (j < 0) j += n;
  // quadrant q = round(4 j / n), r = 2 pi (j / n - q / 4)
  const long long q = (8 * j + n) / (2 * n);
  const double r = kTwoPi * ((double)(4 * j - q * n) / (double)(4 * n));
  const double r2 = r * r;
  double sn = r, cs = 1.0, ts = r, tc = 1.0;
  for (int k = 1; k <= 12; ++k) {
    ts *= -r2 / (double)((2 * k) * (2 * k + 1));
    tc *= -r2 / (double)((2 * k - 1) * (2 * k));
    sn += ts;
    cs += tc;
  }
  switch (q & 3) {
    case 0: return CS{cs, sn};
    case 1: return CS{-sn, cs};
    case 2: return CS{-cs, -sn};
    default: return CS{sn, -cs};
  }
}

template <int N>
struct TwTable {
  double c[N], s[N];
  constexpr TwTable() : c(), s() {
    for (int j = 0; j < N; ++j) {
      const CS v = ce_cossin(j, N);
      c[j] = v.c;
      s[j] = v.s;
    }
  }
};
template <int N>
constexpr TwTable<N> kTw{};

template <class R>
__host__ __device__ __forceinline__ c2<R> cmul(c2<R> a, R wr, R wi) {
  return c2<R>{a.x * wr - a.y * wi, a.x * wi + a.y * wr};
}

// out[k] = sum_j a[j] e^{SGN 2 pi i j k / N}, in place, natural order in and out.
template <class R, int N, int SGN>
struct LineFft {
  static_assert(N >= 1, "length");
  static constexpr int P = (N % 2 == 0) ? 2 : 3;
  static constexpr int Q = N / P;
  static_assert(N == 1 || N % P == 0, "lengths are 2^a 3^b");
  __host__ __device__ static __forceinline__ void run(c2<R> (&a)[N]) {
    if constexpr (N == 1) {
      return;
    } else {
      c2<R> sub[P][Q];
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int q = 0; q < Q; ++q) sub[p][q] = a[q * P + p];
#pragma unroll
      for (int p = 0; p < P; ++p) LineFft<R, Q, SGN>::run(sub[p]);
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        c2<R> t[P];
        t[0] = sub[0][k];
#pragma unroll
        for (int p = 1; p < P; ++p) {
          const int m = (p * k) % N;
          t[p] = cmul<R>(sub[p][k], (R)kTw<N>.c[m], (R)(SGN * kTw<N>.s[m]));
        }
        if constexpr (P == 2) {
          a[k] = c2<R>{t[0].x + t[1].x, t[0].y + t[1].y};
          a[k + Q] = c2<R>{t[0].x - t[1].x, t[0].y - t[1].y};
        } else {
          // radix 3: w3 = e^{SGN 2 pi i / 3} = -1/2 + SGN i sqrt(3)/2
          const R h = (R)0.8660254037844386467637231707529 * (R)SGN;
          const c2<R> sp{t[1].x + t[2].x, t[1].y + t[2].y};
          const c2<R> sm{t[1].x - t[2].x, t[1].y - t[2].y};
          const c2<R> m0{t[0].x - (R)0.5 * sp.x, t[0].y - (R)0.5 * sp.y};
          a[k] = c2<R>{t[0].x + sp.x, t[0].y + sp.y};
          a[k + Q] = c2<R>{m0.x - h * sm.y, m0.y + h * sm.x};
          a[k + 2 * Q] = c2<R>{m0.x + h * sm.y, m0.y - h * sm.x};
        }
      }
    }
  }
};

// Forward (inverse) transform of the x, y and z axes of one (time slice, spin) of a
// system, through LDS: e_in -> fft_tmp with the time twist (fft_tmp -> e_out with the
// untwist and 1/V).  Replaces k_fft_xy + k_fft_z for lattices whose spatial extents
// have templates.  Workgroup b of the run starting at system s0: system s0 + b / (4 T),
// spin b % 4, time slice (b / 4) % T.  LDS rows padded by one value against bank
// conflicts of the x lines.
template <class R, int NX, int NY, int NZ, int INV>
__global__ void __launch_bounds__(256) k_fft_xyz(const SysDev* __restrict__ sys, int s0,
                                                 int periodic) {
  constexpr int PX = NX + 1;
  constexpr int NV = NX * NY * NZ;
  constexpr int SGN = INV ? 1 : -1;
  __shared__ c2<R> A[PX * NY * NZ];
  const int T = sys[s0].g.T;
  const int b = blockIdx.x;
  const SysDev& S = sys[s0 + b / (4 * T)];
  if (S.active && *S.active == 0) return;
  const int spin = b & 3;
  const int t = (b >> 2) % T;
  const int V = S.g.V;
  const size_t off = (size_t)spin * V + (size_t)t * NV;
  const c2<R>* in = (const c2<R>*)(INV ? S.fft_tmp : S.e_in) + off;
  c2<R>* out = (c2<R>*)(INV ? S.e_out : S.fft_tmp) + off;
  double tr = 1.0, ti = 0.0;  // twist (forward) / untwist and normalisation (inverse)
  if (S.g.bc < 0 && !periodic) sincospi((double)SGN * (double)t / (double)T, &ti, &tr);
  if (INV) {
    tr /= (double)V;
    ti /= (double)V;
  }
  const R rr = (R)tr, ri = (R)ti;
  {
    // every load of the volume in flight before the first LDS store (256 threads)
    constexpr int NL = (NV + 255) / 256;
    c2<R> v[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int i = q * 256 + (int)threadIdx.x;
      if (i < NV) v[q] = ldg2<R>(in, i);
    }
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int i = q * 256 + (int)threadIdx.x;
      if (i < NV) A[i % NX + PX * (i / NX)] = INV ? v[q] : cmul<R>(v[q], rr, ri);
    }
  }
  __syncthreads();
  for (int l = threadIdx.x; l < NY * NZ; l += blockDim.x) {  // x lines
    c2<R> a[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) a[x] = A[x + PX * l];
    LineFft<R, NX, SGN>::run(a);
#pragma unroll
    for (int x = 0; x < NX; ++x) A[x + PX * l] = a[x];
  }
  __syncthreads();
  for (int l = threadIdx.x; l < NX * NZ; l += blockDim.x) {  // y lines
    const int x = l % NX, z = l / NX;
    c2<R> a[NY];
#pragma unroll
    for (int y = 0; y < NY; ++y) a[y] = A[x + PX * (y + NY * z)];
    LineFft<R, NY, SGN>::run(a);
#pragma unroll
    for (int y = 0; y < NY; ++y) A[x + PX * (y + NY * z)] = a[y];
  }
  __syncthreads();
  for (int l = threadIdx.x; l < NX * NY; l += blockDim.x) {  // z lines
    c2<R> a[NZ];
#pragma unroll
    for (int z = 0; z < NZ; ++z) a[z] = A[l % NX + PX * (l / NX + NY * z)];
    LineFft<R, NZ, SGN>::run(a);
#pragma unroll
    for (int z = 0; z < NZ; ++z) A[l % NX + PX * (l / NX + NY * z)] = a[z];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < NV; i += blockDim.x) {
    const c2<R> v = A[i % NX + PX * (i / NX)];
    stg2<R>(out, i, INV ? cmul<R>(v, rr, ri) : v);
  }
}

// The preconditioner's scale per momentum of every system (sites of the table's
// partition; momentum (kx, ky, kz, kt) at the site index of (x, y, z, t)), for
// k_fft_t_pcg: the same arithmetic as the SYM_PCG symbol.
__global__ void __launch_bounds__(256) k_pcg_table(const SysDev* __restrict__ sys,
                                                   const int* __restrict__ bmap, int nb_total,
                                                   const SymParams sp) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int X = S.g.X, Y = S.g.Y, Z = S.g.Z, T = S.g.T, V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  const double tshift = (S.g.bc < 0 && !sp.periodic) ? 1.0 : 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    int r = i;
    const int kx = r % X; r /= X;
    const int ky = r % Y; r /= Y;
    const int kz = r % Z;
    const int kt = r / Z;
    double sx, cx, sy, cy, sz, cz, st, ct;
    sincospi(2.0 * (double)kx / (double)X, &sx, &cx);
    sincospi(2.0 * (double)ky / (double)Y, &sy, &cy);
    sincospi(2.0 * (double)kz / (double)Z, &sz, &cz);
    sincospi((2.0 * kt + tshift) / (double)T, &st, &ct);
    const double w = sp.diag - (cx + cy + cz + ct);
    const double s2sin = sx * sx + sy * sy + sz * sz + st * st;
    S.pcs[i] = pcg_scale(sp, S.pc_re, S.pc_im, S.shift, s2sin, w);
  }
}

// t axis forward, the preconditioner's scale, t axis inverse, in place on fft_tmp: the
// t pass of z = P r.  P does not mix spins, so one thread owns one (site, spin) line of
// NT values in registers; a wave reads 64 consecutive sites of one time slice per load
// (coalesced), and no LDS is needed.  Workgroup (64 threads) b of the run starting at
// system s0: system s0 + b / (4 nchunk), chunk of 64 sites (b / 4) % nchunk, spin b % 4
// (the four spins of a chunk are neighbours, so they share the scale lines in L2).
template <class R, int NT>
__global__ void __launch_bounds__(64) k_fft_t_pcg(const SysDev* __restrict__ sys, int s0,
                                                  int nchunk) {
  const int b = blockIdx.x;
  const SysDev& S = sys[s0 + b / (4 * nchunk)];
  if (S.active && *S.active == 0) return;
  const int XYZ = S.g.X * S.g.Y * S.g.Z;
  const int site = ((b >> 2) % nchunk) * 64 + (int)threadIdx.x;
  if (site >= XYZ) return;
  c2<R>* f = (c2<R>*)S.fft_tmp + (size_t)(b & 3) * S.g.V + site;
  const double* sc = S.pcs + site;
  c2<R> a[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) a[t] = ldg2<R>(f, (size_t)t * XYZ);
  LineFft<R, NT, -1>::run(a);
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const double m = ldg(sc, (size_t)k * XYZ);
    a[k] = c2<R>{(R)((double)a[k].x * m), (R)((double)a[k].y * m)};
  }
  LineFft<R, NT, 1>::run(a);
#pragma unroll
  for (int t = 0; t < NT; ++t) stg2<R>(f, (size_t)t * XYZ, a[t]);
}

// Yukawa epilogue of a momentum-space D (psi = e_in, D psi already in e_out):
//   mode 0:  e_out = D psi + Y psi,           partial |e_out|^2 -> part_c, part_b
//   mode 1:  e_out = D^dag psi + Y^dag psi
//   mode 2:  r64 = b - (D^dag psi + Y^dag psi)  (+ copy in cg_r when set),
//            partial |r64|^2 -> part_c   (FP64 only)
// c+ = m + g phi, c- = m* + g* phi*;  Y psi = c- P- psi + c+ P+ psi (spins 0,1 / 2,3).
template <class R>
__global__ void __launch_bounds__(256) k_yuk(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                              int nb_total, int mode) {
  __shared__ double lds[17];
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    c2<R> p[4], w[4];
    load_sp<R>((const c2<R>*)S.e_in, V, i, p);
    load_sp<R>((const c2<R>*)S.e_out, V, i, w);
    const double2 ph = S.phi[i];
    double cpr = S.m_re + S.g_re * ph.x - S.g_im * ph.y;
    double cpi = S.m_im + S.g_re * ph.y + S.g_im * ph.x;
    const double cmr = cpr;
    double cmi = -cpi;
    if (mode != 0) {  // adjoint: conjugate coefficients
      cpi = -cpi;
      cmi = -cmi;
    }
    double2 o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double cr = (k < 2) ? cmr : cpr, ci = (k < 2) ? cmi : cpi;
      const double pr = (double)p[k].x, pi = (double)p[k].y;
      o[k] = double2{(double)w[k].x + cr * pr - ci * pi, (double)w[k].y + cr * pi + ci * pr};
    }
    if (S.shift != 0.0 && mode == 1) {  // (MdagM + sigma) p: p = cg_p
      c2<R> q[4];
      load_sp<R>((const c2<R>*)S.cg_p, V, i, q);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        o[k] = double2{o[k].x + S.shift * (double)q[k].x, o[k].y + S.shift * (double)q[k].y};
    }
    if (mode == 2) {
      double2 rr[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double2 bv = S.cg_b[(size_t)i * 4 + k];
        rr[k] = double2{bv.x - o[k].x, bv.y - o[k].y};
      }
      if (S.shift != 0.0) {  // (MdagM + sigma) x: x = cg_x64
        double2 x[4];
        load_sp<double>((const double2*)S.cg_x64, V, i, x);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          rr[k] = double2{rr[k].x - S.shift * x[k].x, rr[k].y - S.shift * x[k].y};
      }
      store_sp<double>((double2*)S.cg_r64, V, i, rr);
      if (S.cg_r) {
        c2<R> lo[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) lo[k] = c2<R>{(R)rr[k].x, (R)rr[k].y};
        store_sp<R>((c2<R>*)S.cg_r, V, i, lo);
      }
      acc += norm2_sp(rr);
      continue;
    }
    c2<R> ov[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) ov[k] = c2<R>{(R)o[k].x, (R)o[k].y};
    store_sp<R>((c2<R>*)S.e_out, V, i, ov);
    if (mode == 0) acc += norm2_sp(ov) + S.shift * norm2_sp(p);  // <p, (MdagM + sigma) p>
  }
  if (mode != 1) {
    const double tot = block_sum(acc, lds);
    if (threadIdx.x == 0) {
      S.part_c[lb] = tot;
      if (mode == 0 && S.part_b) S.part_b[lb] = tot;
    }
  }
}

// ------------------------------------------------ locality probe (Sec. 3.2)
// norm[i] = ||psi_i|| (psi = e_in, FP64 planar) for the sites of one system.
__global__ void __launch_bounds__(256) k_site_norm(const SysDev* __restrict__ sys,
                                                    const int* __restrict__ bmap, int nb_total,
                                                    double* __restrict__ norm) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 v[4];
    load_sp<double>((const double2*)S.e_in, V, i, v);
    norm[i] = sqrt(norm2_sp(v));
  }
}

// f[r] = max norm[i] over the sites at taxi-driver distance r from the origin,
// r = sum_mu min(x_mu, L_mu - x_mu).  One workgroup per r.
__global__ void __launch_bounds__(256) k_shell_max(const Geo g, const double* __restrict__ norm,
                                                    double* __restrict__ f) {
  __shared__ double red[256];
  const int r = blockIdx.x;
  double m = 0.0;
  for (int i = threadIdx.x; i < g.V; i += blockDim.x) {
    int q = i;
    const int x = q % g.X; q /= g.X;
    const int y = q % g.Y; q /= g.Y;
    const int z = q % g.Z;
    const int t = q / g.Z;
    const int d = min(x, g.X - x) + min(y, g.Y - y) + min(z, g.Z - z) + min(t, g.T - t);
    if (d == r) m = fmax(m, norm[i]);
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) f[r] = red[0];
}

// ----------------------------------------- multi-shift CG on MdagM (RHMC layers)
// (MdagM + beta_i) X_i = b for every shift on the Krylov space of the base CG
// (beta = 0), with Jegerlehner's zeta recurrences (the rational functions of
// MdagM of Sec. 7.3).  Per system the coefficient block shc holds, per shift i,
// (a_i, z_i, b_i, act_i) at 4 i: x_i += a_i p_i; p_i = z_i r + b_i p_i while
// act_i != 0; the residues alpha_i at SHC_RES + i and a0 at SHC_A0.
enum { SHC_RES = 4 * MAXP, SHC_A0 = 5 * MAXP, SHC_LEN = 5 * MAXP + 1 };

// mode 0: x_i = 0, p_i = r (cg_r, FP64).  mode 1: the update above.
__global__ void __launch_bounds__(256) k_shift(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                int nb_total, int mode) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const size_t slot = (size_t)4 * V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  const double* cf = S.shc;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 r[4];
    load_sp<double>((const double2*)S.cg_r, V, i, r);
    for (int k = 0; k < S.nshift; ++k) {
      double2* xk = S.shx + (size_t)k * slot;
      double2* pk = S.shp + (size_t)k * slot;
      if (mode == 0) {
        double2 z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) z[q] = double2{0.0, 0.0};
        store_sp<double>(xk, V, i, z);
        store_sp<double>(pk, V, i, r);
        continue;
      }
      if (cf[4 * k + 3] == 0.0) continue;
      const double a = cf[4 * k], zz = cf[4 * k + 1], bb = cf[4 * k + 2];
      double2 x[4], pv[4];
      load_sp<double>(xk, V, i, x);
      load_sp<double>(pk, V, i, pv);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[q] = double2{x[q].x + a * pv[q].x, x[q].y + a * pv[q].y};
        pv[q] = double2{zz * r[q].x + bb * pv[q].x, zz * r[q].y + bb * pv[q].y};
      }
      store_sp<double>(xk, V, i, x);
      store_sp<double>(pk, V, i, pv);
    }
  }
}

// e_out = a0 b + sum_i alpha_i x_i (b = cg_b, complex128 AoS; e_out FP64 planar).
__global__ void __launch_bounds__(256) k_rat_combine(const SysDev* __restrict__ sys,
                                                      const int* __restrict__ bmap, int nb_total) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const size_t slot = (size_t)4 * V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  const double a0 = S.shc[SHC_A0];
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double2 bv = S.cg_b[(size_t)i * 4 + q];
      o[q] = double2{a0 * bv.x, a0 * bv.y};
    }
    for (int k = 0; k < S.nshift; ++k) {
      const double al = S.shc[SHC_RES + k];
      double2 x[4];
      load_sp<double>(S.shx + (size_t)k * slot, V, i, x);
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = double2{o[q].x + al * x[q].x, o[q].y + al * x[q].y};
    }
    store_sp<double>((double2*)S.e_out, V, i, o);
  }
}

// e_out *= f (FP64 planar).
__global__ void __launch_bounds__(256) k_scale(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                int nb_total, double f) {
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 v[4];
    load_sp<double>((const double2*)S.e_out, V, i, v);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = double2{f * v[q].x, f * v[q].y};
    store_sp<double>((double2*)S.e_out, V, i, v);
  }
}

// ----------------------------- inner MdagM in Ginsparg-Wilson form (Sec. 2.2)
// With D = 1 + g5 eps and eps^2 = 1, D^dag D = D + D^dag (the Ginsparg-Wilson
// relation at a = 1), so with the site-local Y = c- P- + c+ P+
//   MdagM v = (1 + |1 + c|^2) v + (1 + c*) g5 eps(v) + eps(g5 (1 + Y) v)
// per spin component (c = c- on spins 0,1 and c+ on spins 2,3).  The two signs
// are independent, so one two-source multi-shift solve replaces the two
// dependent ones of M then M^dag.  For the rational eps the result differs from
// MdagM by (1 - eps^2) v, i.e. by the approximation error: the inner solver
// uses it, the FP64 true residuals use M then M^dag.
//
// prep (entries A = ta[s], B = tb[s]; v = A.e_in): B.src = g5 (1 + Y) v, the
// source partials |v|^2 -> A.part_b and |B.src|^2 -> B.part_b (rho_0 of both
// multi-shift solves), and B's per-outer-iteration counter stat[3] cleared.
template <class R>
__global__ void __launch_bounds__(512) k_gw_prep(const SysDev* __restrict__ ta,
                                                  const SysDev* __restrict__ tb,
                                                  const int* __restrict__ bmap, int nb_total) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& A = ta[s];
  const SysDev& B = tb[s];
  if (A.active && *A.active == 0) return;
  const int lb = L - A.blk0;
  const int V = A.g.V;
  const int i0 = lb * A.spb;
  const int i1 = min(V, i0 + A.spb);
  if (lb == 0 && threadIdx.x == 0) B.stat[3] = 0;
  double av = 0.0, as = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    c2<R> v[4];
    load_sp<R>((const c2<R>*)A.e_in, V, i, v);
    const double2 ph = A.phi[i];
    const double cpr = A.m_re + A.g_re * ph.x - A.g_im * ph.y;
    const double cpi = A.m_im + A.g_re * ph.y + A.g_im * ph.x;
    c2<R> o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double cr = cpr, ci = (k < 2) ? -cpi : cpi;  // c- = conj(c+)
      const double vr = (double)v[k].x, vi = (double)v[k].y;
      const double g5 = k < 2 ? -1.0 : 1.0;
      o[k] = c2<R>{(R)(g5 * (vr + cr * vr - ci * vi)), (R)(g5 * (vi + cr * vi + ci * vr))};
    }
    store_sp<R>((c2<R>*)B.src, V, i, o);
    av += norm2_sp(v);
    as += norm2_sp(o);
  }
  const double tv = block_sum(av, lds);
  const double ts = block_sum(as, lds);
  if (threadIdx.x == 0) {
    A.part_b[lb] = tv;
    B.part_b[lb] = ts;
  }
}

// e = sum_{j < N} d_j t_j at site i (FP64 accumulation, two slots per step).
template <class R>
__device__ __forceinline__ void basis_sum(const c2<R>* __restrict__ basis,
                                          const double* __restrict__ d, int N, size_t slot, int V,
                                          int i, double2 e[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) e[k] = double2{0.0, 0.0};
  int j = 0;
  for (; j + 1 < N; j += 2) {
    const double d0 = d[j], d1 = d[j + 1];
    const c2<R>* b0 = basis + (size_t)j * slot;
    c2<R> v0[4], v1[4];
    load_sp<R>(b0, V, i, v0);
    load_sp<R>(b0 + slot, V, i, v1);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      e[k].x += d0 * (double)v0[k].x + d1 * (double)v1[k].x;
      e[k].y += d0 * (double)v0[k].y + d1 * (double)v1[k].y;
    }
  }
  if (j < N) {
    const double d0 = d[j];
    c2<R> v0[4];
    load_sp<R>(basis + (size_t)j * slot, V, i, v0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      e[k].x += d0 * (double)v0[k].x;
      e[k].y += d0 * (double)v0[k].y;
    }
  }
}

// combine: e1 = sum_j dA_j tA_j (entry A: eps(v)), e23 = sum_j dB_j tB_j (entry
// B: eps(g5 (1 + Y) v)), w = (1 + |1 + c|^2) v + (1 + c*) g5 e1 + e23 -> A.e_out;
// partial Re <v, w> -> A.part_a (the passes' partials are dead by then; k_cg_misc op 7
// reduces them while it writes part_c).  v = A.e_in.
template <class R>
__global__ void __launch_bounds__(512) k_gw_combine(const SysDev* __restrict__ ta,
                                                     const SysDev* __restrict__ tb,
                                                     const int* __restrict__ bmap, int nb_total) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& A = ta[s];
  const SysDev& B = tb[s];
  if (A.active && *A.active == 0) return;
  const int lb = L - A.blk0;
  const int V = A.g.V;
  const size_t slot = (size_t)4 * V;
  const int NA = A.h_ctl[1], NB = B.h_ctl[1];
  const int i0 = lb * A.spb;
  const int i1 = min(V, i0 + A.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 e1[4], e2[4];
    basis_sum<R>((const c2<R>*)A.basis, A.coef_d, NA, slot, V, i, e1);
    basis_sum<R>((const c2<R>*)B.basis, B.coef_d, NB, slot, V, i, e2);
    c2<R> v[4];
    load_sp<R>((const c2<R>*)A.e_in, V, i, v);
    const double2 ph = A.phi[i];
    const double cpr = A.m_re + A.g_re * ph.x - A.g_im * ph.y;
    const double cpi = A.m_im + A.g_re * ph.y + A.g_im * ph.x;
    c2<R> w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double cr = cpr, ci = (k < 2) ? -cpi : cpi;
      const double g5 = k < 2 ? -1.0 : 1.0;
      const double a = 1.0 + (1.0 + cr) * (1.0 + cr) + ci * ci + A.shift;  // 1 + |1 + c|^2 + sigma
      // (1 + c*) g5 e1
      const double br = 1.0 + cr, bi = -ci;
      const double fr = g5 * (br * e1[k].x - bi * e1[k].y);
      const double fi = g5 * (br * e1[k].y + bi * e1[k].x);
      const double vr = (double)v[k].x, vi = (double)v[k].y;
      const double wr = a * vr + fr + e2[k].x, wi = a * vi + fi + e2[k].y;
      w[k] = c2<R>{(R)wr, (R)wi};
      acc += vr * wr + vi * wi;
    }
    store_sp<R>((c2<R>*)A.e_out, V, i, w);
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) A.part_a[lb] = tot;  // part_a: free once the passes are done
}

// ------------------------ FP64 true residual in Ginsparg-Wilson form (Sec. 2.2)
// For any Hermitian eps, D = 1 + g5 eps gives D^dag D = 1 + g5 eps + eps g5 + eps^2, so
//   MdagM x = |1 + c|^2 x + (1 + c*) g5 eps(x) + eps(g5 (1 + Y) x) + eps^2 x
// exactly (rational eps included).  One multi-shift with the two sources x (entry A)
// and g5 (1 + Y) x (entry B) provides eps(x), eps(g5 (1 + Y) x) and, from the Krylov
// space of x, w = H r(A)^2 x (coef_d2), with eps^2 x = H w: the true residual needs one
// multi-shift depth instead of two (M, then M^dag).
// combine: P = |1 + c|^2 x + (1 + c*) g5 e1 + e23 -> A.e_out, w -> A.e_out2; x = A.e_in.
__global__ void __launch_bounds__(512) k_truth_combine(const SysDev* __restrict__ ta,
                                                       const SysDev* __restrict__ tb,
                                                       const int* __restrict__ bmap, int nb_total) {
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& A = ta[s];
  const SysDev& B = tb[s];
  if (A.active && *A.active == 0) return;
  const int lb = L - A.blk0;
  const int V = A.g.V;
  const size_t slot = (size_t)4 * V;
  const int NA = A.h_ctl[1], NB = B.h_ctl[1];
  const int i0 = lb * A.spb;
  const int i1 = min(V, i0 + A.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 e1[4], w[4], e2[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e1[k] = w[k] = double2{0.0, 0.0};
    for (int j = 0; j < NA; ++j) {
      const double d = A.coef_d[j], d2 = A.coef_d2[j];
      double2 t[4];
      load_sp<double>((const double2*)A.basis + (size_t)j * slot, V, i, t);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        e1[k] = double2{e1[k].x + d * t[k].x, e1[k].y + d * t[k].y};
        w[k] = double2{w[k].x + d2 * t[k].x, w[k].y + d2 * t[k].y};
      }
    }
    basis_sum<double>((const double2*)B.basis, B.coef_d, NB, slot, V, i, e2);
    double2 x[4];
    load_sp<double>((const double2*)A.e_in, V, i, x);
    const double2 ph = A.phi[i];
    const double cpr = A.m_re + A.g_re * ph.x - A.g_im * ph.y;
    const double cpi = A.m_im + A.g_re * ph.y + A.g_im * ph.x;
    double2 P[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double cr = cpr, ci = (k < 2) ? -cpi : cpi;
      const double g5 = k < 2 ? -1.0 : 1.0;
      const double a = (1.0 + cr) * (1.0 + cr) + ci * ci;  // |1 + c|^2
      const double br = 1.0 + cr, bi = -ci;                // 1 + c*
      const double fr = g5 * (br * e1[k].x - bi * e1[k].y);
      const double fi = g5 * (br * e1[k].y + bi * e1[k].x);
      P[k] = double2{a * x[k].x + fr + e2[k].x, a * x[k].y + fi + e2[k].y};
    }
    store_sp<double>((double2*)A.e_out, V, i, P);
    store_sp<double>((double2*)A.e_out2, V, i, w);
  }
}

// finish, P = e_out, w = e_out2 (H w = eps^2 x):
//   mode 0 (true residual): r64 = b - P - H w -> cg_r64 (b = cg_b, AoS), low-precision
//          copy in cg_r when set, partial |r64|^2 -> part_c;
//   mode 1 (product): W = P + H w = MdagM x -> cg_r64, partial Re <x, W> -> part_c, x = e_in.
template <class R>
__global__ void __launch_bounds__(512) k_truth_finish(const SysDev* __restrict__ sys,
                                                      const int* __restrict__ bmap, int nb_total,
                                                      double diag, int mode) {
  __shared__ double lds[17];
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const Geo g = S.g;
  const int V = g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 hw[4], P[4], rr[4];
    hw_site<double>((const double2*)S.e_out2, g, i, diag, hw);
    load_sp<double>((const double2*)S.e_out, V, i, P);
    if (mode == 1) {
      double2 x[4];
      load_sp<double>((const double2*)S.e_in, V, i, x);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        rr[k] = double2{P[k].x + hw[k].x, P[k].y + hw[k].y};
        acc += x[k].x * rr[k].x + x[k].y * rr[k].y;
      }
      store_sp<double>((double2*)S.cg_r64, V, i, rr);
      continue;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 bv = S.cg_b[(size_t)i * 4 + k];
      rr[k] = double2{bv.x - P[k].x - hw[k].x, bv.y - P[k].y - hw[k].y};
    }
    if (S.shift != 0.0) {  // (MdagM + sigma) x: x = e_in
      double2 x[4];
      load_sp<double>((const double2*)S.e_in, V, i, x);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        rr[k] = double2{rr[k].x - S.shift * x[k].x, rr[k].y - S.shift * x[k].y};
    }
    store_sp<double>((double2*)S.cg_r64, V, i, rr);
    if (S.cg_r) {
      c2<R> lo[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) lo[k] = c2<R>{(R)rr[k].x, (R)rr[k].y};
      store_sp<R>((c2<R>*)S.cg_r, V, i, lo);
    }
    acc += norm2_sp(rr);
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_c[lb] = tot;
}

// From the transformed planes (e_out: D_2 phi, K W', K conj(W'), K = 1 - D_2/2):
//   S partials  2 Re conj(phi) D_2 phi + Re conj(W') K W'  -> part_c
//   G = 2 [2 D_2 phi + conj(m + g phi) K W']   (G_out, may be null)
//   F = -K conj(W')                            (F_out, may be null)
__global__ void __launch_bounds__(256) k_boson_finish(const SysDev* __restrict__ sys,
                                                       const int* __restrict__ bmap, int nb_total,
                                                       double2* __restrict__ G_out,
                                                       double2* __restrict__ F_out) {
  __shared__ double lds[17];
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 t[3];  // D_2 phi, K W', K conj W'
#pragma unroll
    for (int k = 0; k < 3; ++k) t[k] = ldg2<double>((const double2*)S.e_out, (size_t)k * V + i);
    const double2 f = S.phi[i], w = w_prime(S, f);
    acc += 2.0 * (f.x * t[0].x + f.y * t[0].y) + (w.x * t[1].x + w.y * t[1].y);
    if (G_out) {
      // conj(m + g phi)
      const double cr = S.m_re + S.g_re * f.x - S.g_im * f.y;
      const double ci = -(S.m_im + S.g_re * f.y + S.g_im * f.x);
      const double pr = cr * t[1].x - ci * t[1].y, pi = cr * t[1].y + ci * t[1].x;
      G_out[i] = double2{2.0 * (2.0 * t[0].x + pr), 2.0 * (2.0 * t[0].y + pi)};
    }
    if (F_out) F_out[i] = double2{-t[2].x, -t[2].y};
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_c[lb] = tot;
}

// Molecular-dynamics updates on complex128 [n] arrays: y += a (x1 + x2) (x2 may be
// null); optional partial |y|^2 per workgroup into part (null: none).
__global__ void __launch_bounds__(256) k_md_axpy(double2* __restrict__ y, double a,
                                                  const double2* __restrict__ x1,
                                                  const double2* __restrict__ x2, int n,
                                                  double* __restrict__ part) {
  __shared__ double lds[17];
  double acc = 0.0;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    double2 v = y[i];
    if (x1) {
      double2 d = x1[i];
      if (x2) d = double2{d.x + x2[i].x, d.y + x2[i].y};
      v = double2{v.x + a * d.x, v.y + a * d.y};
      y[i] = v;
    }
    acc = v.x * v.x + v.y * v.y;
  }
  if (part) {
    const double tot = block_sum(acc, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
  }
}

// ------------------------------------------------------------ CG kernels
// CG scalars of system s from partial sums (part_c; part_b for rho = <r, z>):
//   op 0: start, rho = |r|^2;  1: alpha = rho / <p, w>;  2: beta, rho = |r|^2;
//   3 / 7: reliable update (true |r|^2 replaces the recursive one; 7 restarts);
//   4: |b|^2;  5: true |r|^2 only;
//   preconditioned (PCG, z = P r):  9: beta, rho = <r, z>, |r|^2;  10: start;
//   11 / 12: reliable update from the true residual (|r|^2 set by op 5; 12 restarts);
//   13: the part_b sum alone -> RTRUE.
__global__ void k_cg_scalar(const SysDev* __restrict__ sys, int nsys, int op) {
  __shared__ double lds[17];
  const int s = blockIdx.x;
  if (s >= nsys) return;
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const double v = (op >= 10) ? 0.0 : sum_partials(S.part_c, S.nblk, lds);
  const double rz = (op >= 9) ? sum_partials(S.part_b, S.nblk, lds) : 0.0;
  if (threadIdx.x == 0) {
    double* c = S.cg_s;
    if (op == 0) {
      c[CG_RR] = v;
      c[CG_RR_OLD] = v;
      c[CG_BETA] = 0.0;
      c[CG_R2] = v;
    } else if (op == 1) {
      c[CG_PAP] = v;
      c[CG_ALPHA] = c[CG_RR] / v;
    } else if (op == 2) {
      c[CG_RR_OLD] = c[CG_RR];
      c[CG_RR] = v;
      c[CG_BETA] = v / c[CG_RR_OLD];
      c[CG_R2] = v;
    } else if (op == 3 || op == 7) {  // reliable update: recursive |r|^2 -> true one
      // Keep the search direction unless the true residual exceeds the recursive
      // one by more than 2x (the recursion drifted) or a restart is forced (op 7,
      // a stalled recursion): then restart with p = r.
      const double rec = c[CG_RR];
      c[CG_RTRUE] = v;
      c[CG_RR] = v;
      c[CG_R2] = v;
      c[CG_BETA] = (op == 7 || v > 4.0 * rec) ? 0.0 : v / c[CG_RR_OLD];
    } else if (op == 5) {  // true residual only (no CG state change)
      c[CG_RTRUE] = v;
    } else if (op == 9) {
      c[CG_RR_OLD] = c[CG_RR];
      c[CG_RR] = rz;
      c[CG_BETA] = rz / c[CG_RR_OLD];
      c[CG_R2] = v;
    } else if (op == 10) {  // start from r = b (|b|^2 set by op 4)
      c[CG_RR] = rz;
      c[CG_RR_OLD] = rz;
      c[CG_BETA] = 0.0;
      c[CG_R2] = c[CG_BB];
    } else if (op == 11 || op == 12) {
      const double rec = c[CG_R2];
      const double rt = c[CG_RTRUE];
      c[CG_R2] = rt;
      c[CG_RR] = rz;
      c[CG_BETA] = (op == 12 || rt > 4.0 * rec) ? 0.0 : rz / c[CG_RR_OLD];
    } else if (op == 4) {  // norm of b
      c[CG_BB] = v;
    } else if (op == 13) {
      c[CG_RTRUE] = rz;
    }
  }
}

// stat[3] = 0 for the nsys entries (the per-update maximum of multi-shift iterations).
__global__ void k_stat3_clear(const SysDev* __restrict__ sys, int nsys) {
  for (int s = threadIdx.x; s < nsys; s += blockDim.x)
    if (sys[s].stat) sys[s].stat[3] = 0;
}

// h_ctl[3] = 0 (the sticky multi-shift error bits) for the nsys entries, so that the
// next multi-shift solves can be checked on their own.
__global__ void k_ctl3_clear(const SysDev* __restrict__ sys, int nsys) {
  for (int s = threadIdx.x; s < nsys; s += blockDim.x)
    if (sys[s].h_ctl) sys[s].h_ctl[3] = 0;
}

// Zero n 32-bit words (a fill kernel rather than a memset node, so that the clear is
// an ordinary kernel also when a caller captures the stream into a graph).
__global__ void __launch_bounds__(256) k_zero32(unsigned int* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// p = z + beta p (z = cg_z, or r without a preconditioner; beta from cg_s;
// use_beta = 0 -> p = z); partial |p|^2 -> part_b.
template <class R>
__global__ void __launch_bounds__(512) k_cg_p(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                               int nb_total, int use_beta) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const double beta = use_beta ? S.cg_s[CG_BETA] : 0.0;
  use_beta = use_beta && beta != 0.0;  // restart: p = r, the old p is never read
  if (lb == 0 && threadIdx.x == 0) S.stat[3] = 0;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    c2<R> r[4], p[4];
    load_sp<R>((const c2<R>*)(S.cg_z ? S.cg_z : S.cg_r), V, i, r);
    if (use_beta) {
      load_sp<R>((const c2<R>*)S.cg_p, V, i, p);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        p[k] = c2<R>{(R)((double)r[k].x + beta * (double)p[k].x),
                     (R)((double)r[k].y + beta * (double)p[k].y)};
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) p[k] = r[k];
    }
    store_sp<R>((c2<R>*)S.cg_p, V, i, p);
    acc += norm2_sp(p);
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_b[lb] = tot;
}

// k_cg_p followed by k_gw_prep in one pass (the Ginsparg-Wilson inner operator):
// p = z + beta p -> cg_p; the second multi-shift source g5 (1 + Y) p -> B.src; partials
// |p|^2 -> part_b (the CG table's and entry A's, one buffer) and |g5 (1 + Y) p|^2 ->
// B.part_b.  S: CG table, A and B: the two entries of the inner multi-shift.
template <class R>
__global__ void __launch_bounds__(512) k_cg_p_gw(const SysDev* __restrict__ sys,
                                                 const SysDev* __restrict__ ta,
                                                 const SysDev* __restrict__ tb,
                                                 const int* __restrict__ bmap, int nb_total,
                                                 int use_beta) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& S = sys[s];
  const SysDev& A = ta[s];
  const SysDev& B = tb[s];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const double beta = use_beta ? S.cg_s[CG_BETA] : 0.0;
  use_beta = use_beta && beta != 0.0;  // restart: p = z, the old p is never read
  if (lb == 0 && threadIdx.x == 0) {
    S.stat[3] = 0;
    B.stat[3] = 0;
  }
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double av = 0.0, as = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    c2<R> r[4], p[4];
    load_sp<R>((const c2<R>*)(S.cg_z ? S.cg_z : S.cg_r), V, i, r);
    if (use_beta) {
      load_sp<R>((const c2<R>*)S.cg_p, V, i, p);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        p[k] = c2<R>{(R)((double)r[k].x + beta * (double)p[k].x),
                     (R)((double)r[k].y + beta * (double)p[k].y)};
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) p[k] = r[k];
    }
    store_sp<R>((c2<R>*)S.cg_p, V, i, p);
    const double2 ph = A.phi[i];
    const double cpr = A.m_re + A.g_re * ph.x - A.g_im * ph.y;
    const double cpi = A.m_im + A.g_re * ph.y + A.g_im * ph.x;
    c2<R> o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double cr = cpr, ci = (k < 2) ? -cpi : cpi;  // c- = conj(c+)
      const double vr = (double)p[k].x, vi = (double)p[k].y;
      const double g5 = k < 2 ? -1.0 : 1.0;
      o[k] = c2<R>{(R)(g5 * (vr + cr * vr - ci * vi)), (R)(g5 * (vi + cr * vi + ci * vr))};
    }
    store_sp<R>((c2<R>*)B.src, V, i, o);
    av += norm2_sp(p);
    as += norm2_sp(o);
  }
  const double tv = block_sum(av, lds);
  const double ts = block_sum(as, lds);
  if (threadIdx.x == 0) {
    S.part_b[lb] = tv;
    B.part_b[lb] = ts;
  }
}

// Fill / axpy helpers used by the reliable-update solver.
//   op 0: x64 += x (low precision), x = 0
//   op 1: r = b (FP64 AoS -> planar R), partial |b|^2 -> part_c
//   op 2: x = 0
//   op 3: x64 += e_out (low precision), x = 0        (preconditioned fold-in)
//   op 4: partial |r|^2 -> part_c
//   op 5: x += alpha p, r -= alpha e_in, partial |r|^2 -> part_c
//   op 6: partial Re <r, z> -> part_b  (z = cg_z)
//   op 7: op 5 with alpha = rho / Re <p, w> from the partials in part_a, reduced by every
//         workgroup in the fixed order of k_cg_scalar (identical bits everywhere);
//         workgroup 0 records PAP and ALPHA
template <class R>
__global__ void __launch_bounds__(512) k_cg_misc(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                  int nb_total, int op) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double alpha7 = 0.0;
  const bool own_alpha = op == 7;
  if (own_alpha) {
    const double pap = sum_partials(S.part_a, S.nblk, lds);
    alpha7 = S.cg_s[CG_RR] / pap;
    if (lb == 0 && threadIdx.x == 0) {
      S.cg_s[CG_PAP] = pap;
      S.cg_s[CG_ALPHA] = alpha7;
    }
    op = 5;
  }
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    if (op == 0) {
      c2<R> xv[4];
      double2 xh[4];
      load_sp<R>((const c2<R>*)S.cg_x, V, i, xv);
      load_sp<double>((const double2*)S.cg_x64, V, i, xh);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        xh[k] = double2{xh[k].x + (double)xv[k].x, xh[k].y + (double)xv[k].y};
        xv[k] = c2<R>{(R)0, (R)0};
      }
      store_sp<double>((double2*)S.cg_x64, V, i, xh);
      store_sp<R>((c2<R>*)S.cg_x, V, i, xv);
    } else if (op == 1) {
      c2<R> rv[4];
      double2 bv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        bv[k] = S.cg_b[(size_t)i * 4 + k];
        rv[k] = c2<R>{(R)bv[k].x, (R)bv[k].y};
      }
      store_sp<R>((c2<R>*)S.cg_r, V, i, rv);
      acc += norm2_sp(bv);
    } else if (op == 2) {
      c2<R> z[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) z[k] = c2<R>{(R)0, (R)0};
      store_sp<R>((c2<R>*)S.cg_x, V, i, z);
    } else if (op == 3) {
      c2<R> xv[4];
      double2 xh[4];
      load_sp<R>((const c2<R>*)S.e_out, V, i, xv);
      load_sp<double>((const double2*)S.cg_x64, V, i, xh);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        xh[k] = double2{xh[k].x + (double)xv[k].x, xh[k].y + (double)xv[k].y};
        xv[k] = c2<R>{(R)0, (R)0};
      }
      store_sp<double>((double2*)S.cg_x64, V, i, xh);
      store_sp<R>((c2<R>*)S.cg_x, V, i, xv);
    } else if (op == 4) {
      c2<R> rv[4];
      load_sp<R>((const c2<R>*)S.cg_r, V, i, rv);
      acc += norm2_sp(rv);
    } else if (op == 5) {
      const double alpha = own_alpha ? alpha7 : S.cg_s[CG_ALPHA];
      c2<R> xv[4], pv[4], rv[4], qv[4];
      load_sp<R>((const c2<R>*)S.cg_x, V, i, xv);
      load_sp<R>((const c2<R>*)S.cg_p, V, i, pv);
      load_sp<R>((const c2<R>*)S.cg_r, V, i, rv);
      load_sp<R>((const c2<R>*)S.e_in, V, i, qv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        xv[k] = c2<R>{(R)((double)xv[k].x + alpha * (double)pv[k].x),
                      (R)((double)xv[k].y + alpha * (double)pv[k].y)};
        rv[k] = c2<R>{(R)((double)rv[k].x - alpha * (double)qv[k].x),
                      (R)((double)rv[k].y - alpha * (double)qv[k].y)};
      }
      store_sp<R>((c2<R>*)S.cg_x, V, i, xv);
      store_sp<R>((c2<R>*)S.cg_r, V, i, rv);
      acc += norm2_sp(rv);
    } else if (op == 6) {
      c2<R> rv[4], zv[4];
      load_sp<R>((const c2<R>*)S.cg_r, V, i, rv);
      load_sp<R>((const c2<R>*)S.cg_z, V, i, zv);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        acc += (double)rv[k].x * (double)zv[k].x + (double)rv[k].y * (double)zv[k].y;
    }
  }
  if (op == 1 || op == 4 || op == 5) {
    const double tot = block_sum(acc, lds);
    if (threadIdx.x == 0) S.part_c[lb] = tot;
  } else if (op == 6) {
    const double tot = block_sum(acc, lds);
    if (threadIdx.x == 0) S.part_b[lb] = tot;
  }
}

// ------------------------------------------------------------------ force
// dS/dphi_x = -g [ Y_x^dag P+ X_x + X_x^dag P- Y_x ]  and  G_x = 2 conj(dS/dphi_x),
// summed over the nsys right-hand sides (same lattice, same phi) in index order.
// X = e_in, Y = e_out (FP64 planar) per system; G complex128 [V].
__global__ void __launch_bounds__(256) k_force(const SysDev* __restrict__ sys, int nsys,
                                                int nb0, double2* __restrict__ G) {
  const int L = xcd_logical_block(nb0);
  const SysDev& S0 = sys[0];
  const int V = S0.g.V;
  const int i0 = L * S0.spb;
  const int i1 = min(V, i0 + S0.spb);
  const double g_re = S0.g_re, g_im = S0.g_im;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double gr = 0.0, gi = 0.0;
    for (int s = 0; s < nsys; ++s) {
      double2 X[4], Y[4];
      load_sp<double>((const double2*)sys[s].e_in, V, i, X);
      load_sp<double>((const double2*)sys[s].e_out, V, i, Y);
      // t = sum_{s=2,3} conj(Y_s) X_s + sum_{s=0,1} conj(X_s) Y_s
      double tr = 0.0, ti = 0.0;
#pragma unroll
      for (int k = 2; k < 4; ++k) {
        tr += Y[k].x * X[k].x + Y[k].y * X[k].y;
        ti += Y[k].x * X[k].y - Y[k].y * X[k].x;
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        tr += X[k].x * Y[k].x + X[k].y * Y[k].y;
        ti += X[k].x * Y[k].y - X[k].y * Y[k].x;
      }
      // dS/dphi = -g t ;  G = 2 conj(dS/dphi)
      const double fr = -(g_re * tr - g_im * ti);
      const double fi = -(g_re * ti + g_im * tr);
      gr += 2.0 * fr;
      gi += -2.0 * fi;
    }
    G[i] = double2{gr, gi};
  }
}

// Partials of |c_x|^2 = |m + g phi_x|^2 over the sites of each system -> part_c.
__global__ void __launch_bounds__(256) k_c_norm(const SysDev* __restrict__ sys,
                                                const int* __restrict__ bmap, int nb_total) {
  __shared__ double lds[17];
  const int L = xcd_logical_block(nb_total);
  const SysDev& S = sys[bmap[L]];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    const double2 ph = S.phi[i];
    const double cr = S.m_re + S.g_re * ph.x - S.g_im * ph.y;
    const double ci = S.m_im + S.g_re * ph.y + S.g_im * ph.x;
    acc += cr * cr + ci * ci;
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_c[lb] = tot;
}

// Re <xi, X> partials (xi AoS complex128 from cg_b, X planar FP64 e_in) -> part_c
__global__ void __launch_bounds__(256) k_dot_re(const SysDev* __restrict__ sys, const int* __restrict__ bmap,
                                                 int nb_total) {
  __shared__ double lds[17];
  const int L = blockIdx.x;
  const int s = bmap[L];
  const SysDev& S = sys[s];
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  double acc = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 X[4];
    load_sp<double>((const double2*)S.e_in, V, i, X);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 b = S.cg_b[(size_t)i * 4 + k];
      acc += b.x * X[k].x + b.y * X[k].y;
    }
  }
  const double tot = block_sum(acc, lds);
  if (threadIdx.x == 0) S.part_c[lb] = tot;
}

}  // namespace ov
