// ov_lib.hip -- host orchestration and the C ABI of libov.so (gfx950).
//
// Layers:
//   kernels (ov_kernels.hpp)  -> Engine (batched systems, tables, launch
//   sequences for sign / apply / solve / force)  -> extern "C" ov_* (ov.h).
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/ov.h"
#include "ov_gate.hpp"
#include "ov_host.hpp"
#include "ov_kernels.hpp"

using namespace ov;
static_assert(ov::HOST_MAXP == ov::MAXP, "host and kernel pole limits");

struct ov_ctx {
  ov_params p;
  hipStream_t stream = nullptr;  // caller's stream: work is ordered after it
  hipStream_t priv = nullptr;    // private non-blocking stream all work runs on
  hipEvent_t ev_in = nullptr;    // caller-stream marker the private stream waits for
  std::map<std::string, hipGraphExec_t> graphs;  // captured launch sequences
  bool use_graphs = false;
  bool fft_fixed = true;          // fixed-length transforms for z = P r (OV_FFT_FIXED=0 at
                                  // context creation: the generic passes)
  // resident multi-shift kernel (k_ms_res): see ResGeom
  int res_cus = 0;               // compute units: workgroups of a resident launch
  bool resident = true;          // OV_PERSISTENT=0 at context creation: per-pass kernels only
  ResGeom rg[2];                 // block decomposition of this lattice, FP64 / FP32
  ResShared* res_sh = nullptr;   // device words of the exchange
  int* res_abort = nullptr;      // pinned: raised by a resident launch whose wait ran out
  long long res_spin = 0;        // wall-clock ticks a resident wait may take
  int res_aborts = 0;
  hipEvent_t ev_res = nullptr;   // marks this context's work for another context's launch
  hipError_t gate_err = hipSuccess;  // that wait failed
  bool capturing = false;        // inside a graph capture of the private stream
  std::map<long long, int> n_est;  // (precision, tolerance) -> iterations the last multi-shift needed
  int device = 0;
  std::string err;
  double a[MAXP], b[MAXP], delta = 0;
  double smin = 0, smax = 0;     // analytic free |H_W| range on this lattice
  int block = NTHREADS;          // threads per workgroup
  int spt = 0;                   // sites per thread (0 = automatic)
  // workspace
  void* user_ws = nullptr;
  size_t user_ws_bytes = 0;
  void* own_ws = nullptr;
  size_t own_ws_bytes = 0;
  char* host_block = nullptr;    // pinned: what a context starts with (the four below)
  double* pinned = nullptr;      // host staging of per-system scalars
  int pinned_n = 0;
  bool noalloc = false;          // inside ov_apply_noalloc: scratch array, no allocation
  int* pinned_flags = nullptr;
  char* stage = nullptr;         // pinned: a call's tables on their way to the device
  size_t stage_cap = 0;
  bool stage_busy = false;       // a copy from it may still run
  // kernel-duration sampling (see ov_kernel_sampling)
  int sample_max = 0;
  std::vector<hipEvent_t> ev_pool;             // pairs
  struct EvUse {
    int kernel;
    double bytes;          // bytes of the whole launch
    int ts_blocks;         // workgroups that stamped region ts_index (0: none)
    double sites;          // sites of the launch (all systems): its stamped site count
                           // scales bytes to the systems that took part
  };
  std::vector<EvUse> ev_use;
  // kernels: 0 / 1 FP32 t / r pass, 2 resident, 3 / 4 FP64 t / r pass
  int ev_call_count[5] = {0, 0, 0, 0, 0};
  double ksum_ms[5] = {0, 0, 0, 0, 0}, ksum_bytes[5] = {0, 0, 0, 0, 0};
  double ksum_kernel_ms[5] = {0, 0, 0, 0, 0};  // device-stamped kernel spans
  long long kcount[5] = {0, 0, 0, 0, 0}, kcount_kernel[5] = {0, 0, 0, 0, 0};
  unsigned long long* ts_dev = nullptr;  // stamp regions, ts_region u64 each
  size_t ts_regions = 0, ts_region = 0;
  double wall_khz = 0;                   // wall-clock rate of the stamps
};

// Scratch of ov_apply_noalloc: one array per device, held until the process ends.
// Host code never uses its name as an address (on the host it is only a stand-in for
// the symbol); the device address comes from hipGetSymbolAddress, once per device,
// at context creation (noalloc_scratch_setup).
static __device__ __align__(256) unsigned char scratch[OV_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};  // device address of `scratch` per device
// Host staging (pinned scalars) allocated at context creation, so that the
// no-allocation entry point never allocates it: systems it serves per call.
constexpr int kNoAllocSystems = 16;
// ... and bytes of tables: two per system, and a workgroup map that the scratch array bounds
// (each workgroup's sites hold basis fields in it).
constexpr size_t kNoAllocStage = 64 << 10;

thread_local std::string g_err;

#define HIPCHK(ctx, call)                                                        \
  do {                                                                           \
    hipError_t e_ = (call);                                                      \
    if (e_ != hipSuccess) {                                                      \
      (ctx)->err = std::string(#call) + ": " + hipGetErrorString(e_);            \
      return OV_ERR_DEVICE;                                                      \
    }                                                                            \
  } while (0)

#define TRY(x)                 \
  do {                         \
    ov_status s_ = (x);        \
    if (s_ != OV_OK) return s_; \
  } while (0)

// Test hook: every mixed solve hands its systems to the FP64 solver at the first
// reliable update (exercises the stagnation fallback).
bool force_fallback_env() {
  const char* e = std::getenv("OV_FORCE_FALLBACK");
  return e && *e == '1';
}

// ROCTX range for the life of a scope: the phases of a call show up in a marker trace
// (rocprofv3 --marker-trace); without a tool attached the calls return at once.
struct Range {
  explicit Range(const char* what) { roctxRangePushA(what); }
  ~Range() { roctxRangePop(); }
  Range(const Range&) = delete;
  Range& operator=(const Range&) = delete;
};

bool ov_log() {
  static int v = -1;
  if (v < 0) {
    const char* e = std::getenv("OV_LOG");
    v = (e && *e && *e != '0') ? 1 : 0;
  }
  return v == 1;
}

// z-marching multi-shift passes (OV_MS_ZM=0 switches them off).
// Large multi-shift launches read their flags before their operands; OV_MS_CF=0 keeps
// the operands first everywhere.
bool ms_cf_enabled() {
  static int v = -1;
  if (v < 0) {
    const char* e = std::getenv("OV_MS_CF");
    v = (e && *e == '0') ? 0 : 1;
  }
  return v == 1;
}

bool ms_zm_enabled() {
  static int v = -1;
  if (v < 0) {
    const char* e = std::getenv("OV_MS_ZM");
    v = (e && *e == '0') ? 0 : 1;
  }
  return v == 1;
}

double now_s() {
  using namespace std::chrono;
  return duration<double>(steady_clock::now().time_since_epoch()).count();
}


int capacity(const ov_ctx* c, double tol) {
  const int cap = cg_bound(c->smin, c->smax, tol) + 6;
  return std::max(4, std::min(cap, c->p.max_inner));
}

// 256-byte aligned bump allocator over a device buffer.
struct Bump {
  char* base;
  size_t off = 0, cap;
  bool dry;  // sizing pass: only count
  Bump(void* b, size_t c, bool d) : base((char*)b), cap(c), dry(d) {}
  void* take(size_t bytes) {
    off = (off + 255) & ~size_t(255);
    void* p = dry ? nullptr : base + off;
    off += bytes;
    return p;
  }
};

// Per-system device buffers.
struct SysBuf {
  const ov_ctx* ctx;
  int V, nblk, blk0, spb;
  double2 *basis64, *r64ms, *src64b, *u64, *x64, *r64;
  void *basisR, *rR, *srcR2, *uR, *xR, *pR, *rcgR;
  double *part_a, *part_b, *part_c;
  double *h_rho, *h_alpha, *h_zeta;
  unsigned* h_active;
  int* h_ctl;
  long long* stat;
  double* dstat;
  double *coef_term, *coef_c, *coef_d, *cg_s;
  double* pcs = nullptr;  // preconditioner scale per momentum (preconditioned solves)
  int *act_cg, *act_ru;
  void *vR, *fftR;              // preconditioned solve: M0^-1 p / M^dag u, transform scratch
  // second multi-shift entry of the inner operator in Ginsparg-Wilson form (ms_b*)
  void *ms_b_basis = nullptr, *ms_b_r = nullptr, *ms_b_src = nullptr;
  double *ms_b_part_a = nullptr, *ms_b_part_b = nullptr, *ms_b_part_c = nullptr;
  double *ms_b_h_rho = nullptr, *ms_b_h_alpha = nullptr, *ms_b_h_zeta = nullptr;
  unsigned* ms_b_h_active = nullptr;
  int* ms_b_h_ctl = nullptr;
  double* ms_b_dstat = nullptr;
  double *ms_b_coef_term = nullptr, *ms_b_coef_c = nullptr, *ms_b_coef_d = nullptr;
  long long* ms_b_stat = nullptr;
  // FP64 true residual in Ginsparg-Wilson form: entry B twins (tb_*) and entry A's
  // coefficients of H r(A)^2 x with their scratch
  double2 *tb_basis = nullptr, *tb_r = nullptr, *tb_src = nullptr;
  double *tb_part_a = nullptr, *tb_part_b = nullptr, *tb_part_c = nullptr;
  double *tb_h_rho = nullptr, *tb_h_alpha = nullptr, *tb_h_zeta = nullptr;
  unsigned* tb_h_active = nullptr;
  int* tb_h_ctl = nullptr;
  double* tb_dstat = nullptr;
  double *tb_coef_term = nullptr, *tb_coef_c = nullptr, *tb_coef_d = nullptr;
  long long* tb_stat = nullptr;
  double *coef_d2 = nullptr, *coef_sq = nullptr;
  double2 *shx = nullptr, *shp = nullptr;  // multi-shift CG on MdagM: solutions, directions
  double* shc = nullptr;        //   per-shift coefficients
  int nshift = 0;
  int xc = 1, off_xy = 0, off_z = 0, off_t = 0, off_zt = 0;  // momentum-space pass geometry
};

// Sites per workgroup of `block` threads.  Automatic choice (spt = 0) from the sites of the
// whole launch: one site per thread while every workgroup can start at once (latency-bound
// single systems), beyond 1024 workgroups as many as leave about two per CU: a workgroup
// of a multi-shift pass first sums the partials of all of them (24^3 x 48, FP64 sign, us per
// pass: 2592 workgroups 80, 1296 49, 648 40, 432 39, 260 57; 16^2 x 32 x 48: 1536
// 37, 768 28, 512 23; the FP32 passes of the mixed solve likewise).  Where the xy plane is
// one workgroup and four sites divide Z it takes those, z-marching.  Workgroups of fewer
// threads keep more of them (8^4, 32 mixed solves: 18.6 ms with two sites, 20.3 with four).
int sites_per_block(const ov_ctx* c, int block, int V, long long total_sites) {
  int spt = c->spt;
  if (spt <= 0) {
    const long long blocks1 = (std::max<long long>(total_sites, V) + block - 1) / block;
    const int* d = c->p.dims;
    const bool plane = d[0] * d[1] == block;
    spt = blocks1 <= 1024 ? 1 : (int)std::min<long long>(6, (blocks1 + 511) / 512);
    if (spt > 1 && plane) spt = d[2] % 4 == 0 ? 4 : 2;
    if (block < 256 && spt > 1) spt = blocks1 <= 4096 ? 2 : 4;
    spt = std::max(spt, (int)(((V + block - 1) / block + 2047) / 2048));
    // two sites per thread turn on the z-marching passes (a workgroup per xy plane,
    // two z planes each), which beat one site per thread while every launch still
    // has at least 64 workgroups per system (16^4: 25.2 -> 22.3 ms per mixed solve)
    if (spt == 1 && plane && d[2] % 2 == 0 && V / (2 * block) >= 64) spt = 2;
  }
  return block * spt;
}

// What a call needs: FP64 ms basis capacity cap64, inner precision buffers.
struct Plan {
  int cap64 = 0;   // FP64 basis slots
  int capR = 0;    // inner basis slots (0 = inner is FP64 and shares)
  bool mixed = false;
  bool solve = false;
  bool pc = false;   // free-field preconditioned solve
  bool fft = false;  // momentum-space Dirac operator (no multi-shift)
  int nshift = 0;    // shifted systems of a multi-shift CG on MdagM (rational layers)
  bool gw = false;   // inner MdagM in Ginsparg-Wilson form: one two-source multi-shift
  bool gwx = false;  // exact Ginsparg-Wilson MdagM (true residuals, rational layers): tb_* twins
};

template <class R>
size_t cplx_bytes() { return sizeof(c2<R>); }

// Carve one system's buffers (dry run computes the size).
void carve(Bump& bp, SysBuf& s, const Plan& pl) {
  const size_t v64 = (size_t)4 * s.V * sizeof(double2);
  const size_t v32 = (size_t)4 * s.V * sizeof(float2);
  const int capmax = std::max(pl.cap64, pl.capR);
  s.basis64 = (double2*)bp.take(v64 * pl.cap64);
  s.r64ms = (double2*)bp.take(v64);
  s.src64b = (double2*)bp.take(v64);
  s.u64 = (double2*)bp.take(v64);
  s.x64 = (double2*)bp.take(v64);
  s.r64 = (double2*)bp.take(v64);
  if (pl.solve) {
    if (pl.mixed) {
      s.basisR = bp.take(v32 * pl.capR);
      s.rR = bp.take(v32);
      s.srcR2 = bp.take(v32);
      s.uR = bp.take(v32);
      s.xR = bp.take(v32);
      s.pR = bp.take(v32);
      s.rcgR = bp.take(v32);
    } else {
      s.basisR = s.basis64;
      s.rR = s.r64ms;
      s.srcR2 = s.src64b;
      s.uR = s.u64;
      s.xR = bp.take(v64);
      s.pR = bp.take(v64);
      s.rcgR = bp.take(v64);
    }
  } else {
    s.basisR = s.rR = s.srcR2 = s.uR = s.xR = s.pR = s.rcgR = nullptr;
  }
  s.vR = s.fftR = nullptr;
  if (pl.solve && (pl.pc || pl.fft || pl.nshift > 0 || pl.gw)) {
    s.vR = bp.take(pl.mixed ? v32 : v64);
    s.fftR = bp.take(pl.mixed ? v32 : v64);
  }
  s.pcs = (pl.solve && pl.pc) ? (double*)bp.take(sizeof(double) * s.V) : nullptr;
  s.shx = s.shp = nullptr;
  s.shc = nullptr;
  s.nshift = (pl.solve && pl.nshift > 0) ? pl.nshift : 0;
  if (pl.solve && pl.nshift > 0) {
    s.shx = (double2*)bp.take(v64 * pl.nshift);
    s.shp = (double2*)bp.take(v64 * pl.nshift);
    s.shc = (double*)bp.take(sizeof(double) * SHC_LEN);
  }
  s.part_a = (double*)bp.take(sizeof(double) * s.nblk);
  s.part_b = (double*)bp.take(sizeof(double) * s.nblk);
  s.part_c = (double*)bp.take(sizeof(double) * s.nblk);
  s.h_rho = (double*)bp.take(sizeof(double) * (capmax + 1));
  s.h_alpha = (double*)bp.take(sizeof(double) * (capmax + 1));
  s.h_zeta = (double*)bp.take(sizeof(double) * (capmax + 1) * MAXP);
  s.h_active = (unsigned*)bp.take(sizeof(unsigned) * (capmax + 1));
  s.coef_term = (double*)bp.take(sizeof(double) * MAXP * capmax);
  s.coef_c = (double*)bp.take(sizeof(double) * (capmax + 1));
  s.coef_d = (double*)bp.take(sizeof(double) * capmax);
  if (pl.solve && pl.gw) {
    const size_t vR = pl.mixed ? v32 : v64;
    s.ms_b_basis = bp.take(vR * pl.capR);
    s.ms_b_r = bp.take(vR);
    s.ms_b_src = bp.take(vR);
    s.ms_b_part_a = (double*)bp.take(sizeof(double) * s.nblk);
    s.ms_b_part_b = (double*)bp.take(sizeof(double) * s.nblk);
    s.ms_b_part_c = (double*)bp.take(sizeof(double) * s.nblk);
    s.ms_b_h_rho = (double*)bp.take(sizeof(double) * (capmax + 1));
    s.ms_b_h_alpha = (double*)bp.take(sizeof(double) * (capmax + 1));
    s.ms_b_h_zeta = (double*)bp.take(sizeof(double) * (capmax + 1) * MAXP);
    s.ms_b_h_active = (unsigned*)bp.take(sizeof(unsigned) * (capmax + 1));
    s.ms_b_coef_term = (double*)bp.take(sizeof(double) * MAXP * capmax);
    s.ms_b_coef_c = (double*)bp.take(sizeof(double) * (capmax + 1));
    s.ms_b_coef_d = (double*)bp.take(sizeof(double) * capmax);
  }
  if (pl.solve && pl.gwx) {
    s.tb_basis = (double2*)bp.take(v64 * pl.cap64);
    s.tb_r = (double2*)bp.take(v64);
    s.tb_src = (double2*)bp.take(v64);
    s.tb_part_a = (double*)bp.take(sizeof(double) * s.nblk);
    s.tb_part_b = (double*)bp.take(sizeof(double) * s.nblk);
    s.tb_part_c = (double*)bp.take(sizeof(double) * s.nblk);
    s.tb_h_rho = (double*)bp.take(sizeof(double) * (capmax + 1));
    s.tb_h_alpha = (double*)bp.take(sizeof(double) * (capmax + 1));
    s.tb_h_zeta = (double*)bp.take(sizeof(double) * (capmax + 1) * MAXP);
    s.tb_h_active = (unsigned*)bp.take(sizeof(unsigned) * (capmax + 1));
    s.tb_coef_term = (double*)bp.take(sizeof(double) * MAXP * capmax);
    s.tb_coef_c = (double*)bp.take(sizeof(double) * (capmax + 1));
    s.tb_coef_d = (double*)bp.take(sizeof(double) * capmax);
    s.coef_d2 = (double*)bp.take(sizeof(double) * capmax);
    s.coef_sq = (double*)bp.take(sizeof(double) * (2 * MAXP + 2) * capmax);
  }
}

enum Table {
  T_APPLY = 0, T_APPLY2, T_IN_M, T_IN_MDAG, T_TR_M, T_TR_MDAG, T_CG, T_CG_RU,
  T_PC_Z,     // z = P r, P = (M0^dag M0)^-1 (systems iterating)
  T_PC_ZRU,   // the same for the systems taking a reliable update
  T_F_M,      // momentum-space D: inner M v
  T_F_MD,     // inner M^dag u
  T_F_TM,     // FP64 true residual: M x64
  T_F_TMD,    // r64 = b - M^dag (M x64)
  T_NT
};

// LDS a transform pass may take (of 160 KiB); the xy and z passes of the largest lattices
// (X Y = X Z = 1024, extents up to 64) need 141 KiB.
constexpr size_t FFT_LDS = 148 * 1024;

// x values per workgroup of the t pass: the largest divisor of X with xc T <= 256 (the
// kernel's LDS; MdagM of the 24^3 x 48 fermion with 64, 128, 256: 621, 509, 453 us).
int pick_xc(int X, int T) {
  int best = 1;
  for (int d = 1; d <= X; ++d)
    if (X % d == 0 && d * T <= 256) best = d;
  return best;
}

// The resident launches of one multi-shift solve over a table: entries in order, as many per
// launch as there are CUs for.
struct ResLaunch {
  ResRun run[RES_RUNS];
  int nrun = 0, grid = 0, threads = 64, K = 1;
  int S = 0, G = 0;  // largest block and workgroups of an entry
  size_t lds = 0;
  // When a pass first looks for the partials and the faces.  Partials, in 128 cycles: a look
  // that comes too early costs a whole trip to memory more, and a line through the best of
  // 8 to 24 stays below it (8^4, 32 workgroups of 128 sites: 2.15 us per pass with 8, 1.89 with
  // 11, 2.29 with 20; 16^4 twice, 256 of 512: 4.47, 3.94 with 18, 3.89).  Faces: at once, but
  // for entries on all CUs, whose stores take longer than the hops inside (16^3 x 32: 4.01 us
  // at once, 3.96 after 4 times 64 cycles; 12^4 twice 2.40 and 2.43).
  int nap() const { return std::max(11, (int)(9.6 + 0.01 * S + 0.016 * grid)); }
  int nap_face() const { return G >= 192 ? 4 : 0; }
};
struct ResPlan {
  std::vector<ResLaunch> launches;
  size_t face_bytes = 0;  // the largest launch's faces
  bool use = false;
};

// Lattices the momentum-space kernels handle (LDS tiles of <= 1024 complex values).
// A batch of systems sharing poles, tolerances and precision.
struct Engine {
  std::vector<ov_ctx*> ctxs;        // per system
  std::vector<int> rhs_of;          // rhs index inside its ctx call
  std::vector<SysBuf> sb;
  ov_ctx* lead;
  hipStream_t st;
  Plan pl;
  int nsys = 0, nb_total = 0;
  int block = NTHREADS;             // threads per workgroup: the largest of the members' (a
                                    // small one in front of a batch does not set it for all)
  SysDev* tables = nullptr;         // device: ntab * nsys
  std::vector<SysDev> htab;         // host copy
  size_t up_bytes = 0;              // bytes from `tables` to the end of the uploaded region
  size_t up_head = 0;               // bytes from stat_all to `tables`
  int ntab = T_NT;                  // tables this engine has: the first two, or all (solves)
  int* bmap = nullptr;              // device: logical workgroup -> system
  // the caller's fields and their planar twins per system (SysDev io_*), copied into the
  // T_APPLY entries
  struct Io {
    const void* in = nullptr;
    void *pin = nullptr, *pout = nullptr, *out = nullptr;
  };
  std::vector<Io> io;
  double* cg_all = nullptr;         // device: nsys * CG_NSLOT scalars (one copy to the host)
  long long* stat_all = nullptr;    // device: 3 nsys * 4 multi-shift counters (entries A, B, B')
  double* dstat_all = nullptr;      // device: 3 nsys * 2 shift residuals
  int* ctl_all = nullptr;           // device: 3 nsys * 4 control words
  size_t ctl_words = 0;             // 32-bit words from stat_all to the end of ctl_all
  std::string geo_key;              // launch geometry of every system (graph cache key)
  bool size_worst = false;          // sizing only: the smallest workgroup partition any
                                    // launch shape gives (64 sites per workgroup)
  int* act_all = nullptr;           // device: act_cg[nsys] then act_ru[nsys]
  std::vector<int> last_flags;      // last uploaded flags (upload only on change)
  MsParams mp64{}, mpR{};
  int L64 = 0, LR = 0;              // multi-shift launch counts
  bool no_relax = false;            // fixed inner tolerance (the FP64 fallback solver)
  double shift = 0.0;               // solve (MdagM + shift) x = b (rational layers)
  bool guess = false;               // solve: pack the caller's guesses (io) into x64 first
  int max_outer = 0;                // > 0: outer iteration cap instead of max_outer (the
                                    // fallback solver gets what the mixed one left)
  bool force_fallback = false;      // hand every system to the FP64 solver at its first
                                    // reliable update (OV_FORCE_FALLBACK=1; tests)
  int nb_xy = 0, nb_z = 0, nb_t = 0, nb_zt = 0;  // workgroups of the momentum-space passes
  SysDev* ftab = nullptr;           // device: (system, shift) table of the rational force
  SysDev* gwtab = nullptr;          // device: 2 nsys multi-shift entries of the GW inner operator
  int* gwbmap = nullptr;            // device: 2 nb_total workgroups -> entry
  std::vector<SysDev> hgwtab;       // host copy of gwtab
  SysDev* trgwtab = nullptr;        // device: 2 nsys entries of the FP64 true residual (same map)
  std::vector<SysDev> htrgw;        // host copy

  ResPlan res[2][2];                // resident launches: [FP64, FP32][copies of the systems - 1]
  bool no_res = false;              // per-pass kernels only (tuning, a tight workspace)
  char* face = nullptr;             // device: faces of the largest resident launch
  size_t face_bytes = 0;
  bool shifts = true;               // this call runs multi-shift solves

  template <class R>
  const ResPlan* resident(int copies) const {
    const ResPlan& p = res[sizeof(R) == sizeof(float)][copies - 1];
    return p.use ? &p : nullptr;
  }
  bool resident_any() const {
    return res[0][0].use || res[0][1].use || res[1][0].use || res[1][1].use;
  }

  // Resident launches for `copies` entries per system in a precision, and whether they beat
  // the per-pass kernels: those cost two launches and three field passes per iteration at
  // about 7 us + bytes / 4.6 TB/s each (16^4, two FP64 sources: 12.5 us), a resident pass
  // what res_geom models for it, once per launch.
  void plan_resident(int fp32, int copies) {
    ResPlan& P = res[fp32][copies - 1];
    P = ResPlan{};
    if (no_res || !lead->resident) return;
    const int esize = fp32 ? 8 : 16;
    double t_res = 0.0, t_pass = 7.0;
    double us = 0.0;  // slowest block of the open launch
    size_t faces = 0;
    auto close = [&]() {
      t_res += us;
      us = 0.0;
      P.face_bytes = std::max(P.face_bytes, faces);
      faces = 0;
    };
    for (int e = 0; e < copies * nsys; ++e) {
      const ov_ctx* c = ctxs[e % nsys];
      const ResGeom& q = c->rg[fp32];
      if (q.G == 0) return;
      t_pass += 12.0 * esize * q.S * q.G / 4.6e6;
      const size_t fb = (size_t)2 * q.G * q.FT * esize;
      ResLaunch* l = P.launches.empty() ? nullptr : &P.launches.back();
      const ov_ctx* prev = e > 0 ? ctxs[(e - 1) % nsys] : nullptr;
      const bool same = l && std::equal(c->p.dims, c->p.dims + 4, prev->p.dims);
      if (!l || l->grid + q.G > lead->res_cus || (!same && l->nrun == RES_RUNS)) {
        close();
        P.launches.emplace_back();
        l = &P.launches.back();
      }
      if (l->nrun > 0 && same) {
        ++l->run[l->nrun - 1].ne;
      } else {
        ResRun& r = l->run[l->nrun++];
        r.e0 = e;
        r.ne = 1;
        r.wg0 = l->grid;
        r.G = q.G;
        r.FT = q.FT;
        std::copy(q.b, q.b + 4, r.b);
        std::copy(q.nb, q.nb + 4, r.nb);
        r.face0 = (long long)faces;
      }
      l->grid += q.G;
      l->threads = std::max(l->threads, q.threads);
      l->K = std::max(l->K, q.K);
      l->S = std::max(l->S, q.S);
      l->G = std::max(l->G, q.G);
      l->lds = std::max(l->lds, (size_t)(q.S + 1) * (4 * esize + 16));
      faces += fb;
      us = std::max(us, q.us);
    }
    close();
    P.use = t_res < t_pass;
    if (!P.use) P = ResPlan{};
  }

  // The plans of the tables this engine runs: sign / apply and M, M^dag forms one entry per
  // system, the Ginsparg-Wilson forms two.
  size_t plan_residents() {
    for (auto& row : res)
      for (ResPlan& p : row) p = ResPlan{};
    if (!pl.fft && pl.cap64 > 0) {
      plan_resident(0, 1);
      if (pl.gwx || (pl.gw && !pl.mixed)) plan_resident(0, 2);
      if (pl.solve && pl.mixed) plan_resident(1, pl.gw ? 2 : 1);
    }
    size_t fb = 0;
    for (const auto& row : res)
      for (const ResPlan& p : row) fb = std::max(fb, p.face_bytes);
    return fb;
  }

  size_t layout(void* base, size_t cap, bool dry) {
    Bump bp(base, cap, dry);
    const size_t fb = plan_residents();
    face = fb ? (char*)bp.take(fb) : nullptr;
    face_bytes = fb;
    act_all = (int*)bp.take(sizeof(int) * 2 * nsys);
    int blk = 0, nxy = 0, nz = 0, nt = 0, nzt = 0;
    long long total_sites = 0;
    for (int s = 0; s < nsys; ++s) {
      const ov_params& p = ctxs[s]->p;
      total_sites += (long long)p.dims[0] * p.dims[1] * p.dims[2] * p.dims[3];
    }
    for (int s = 0; s < nsys; ++s) {
      SysBuf& b = sb[s];
      b.ctx = ctxs[s];
      const ov_params& p = ctxs[s]->p;
      b.V = p.dims[0] * p.dims[1] * p.dims[2] * p.dims[3];
      b.spb = size_worst ? 64 : sites_per_block(ctxs[s], block, b.V, total_sites);
      b.nblk = (b.V + b.spb - 1) / b.spb;
      b.blk0 = blk;
      blk += b.nblk;
      carve(bp, b, pl);
      const int X = p.dims[0], Y = p.dims[1], Z = p.dims[2], T = p.dims[3];
      b.xc = pick_xc(X, T);
      b.off_xy = nxy;
      nxy += Z * T;
      b.off_z = nz;
      nz += Y * T;
      b.off_t = nt;
      nt += (X / b.xc) * Y * Z;
      b.off_zt = nzt;
      nzt += X * Y;
      b.act_cg = dry ? nullptr : act_all + s;
      b.act_ru = dry ? nullptr : act_all + nsys + s;
    }
    nb_total = blk;
    nb_xy = nxy;
    nb_z = nz;
    nb_t = nt;
    nb_zt = nzt;
    // everything a captured launch sequence bakes in besides the table and workspace
    // addresses: per system its lattice, boundary, partition and transform chunking
    geo_key.clear();
    for (int s = 0; s < nsys; ++s) {
      const ov_params& p = ctxs[s]->p;
      if (!lead->use_graphs) break;
      char g[96];
      std::snprintf(g, sizeof g, "%dx%dx%dx%d/%d/%d/%d;", p.dims[0], p.dims[1], p.dims[2],
                    p.dims[3], p.bc_t, sb[s].spb, sb[s].xc);
      geo_key += g;
    }
    ftab = pl.nshift > 0 ? (SysDev*)bp.take(sizeof(SysDev) * nsys * pl.nshift) : nullptr;
    // the CG scalars and, right after them, the counters of entries A, B (inner) and
    // B (true residual) -- read back with one copy -- then the entries' shift residuals
    // and control words: everything from stat_all on is cleared together
    const size_t ctl_bytes = sizeof(long long) * 12 * nsys + sizeof(double) * 6 * nsys +
                             sizeof(int) * 12 * nsys;
    cg_all = (double*)bp.take(sizeof(double) * CG_NSLOT * nsys + ctl_bytes);
    const size_t stat0 = bp.off - ctl_bytes;
    stat_all = dry ? nullptr : (long long*)(cg_all + (size_t)CG_NSLOT * nsys);
    dstat_all = dry ? nullptr : (double*)(stat_all + (size_t)12 * nsys);
    ctl_all = dry ? nullptr : (int*)(dstat_all + (size_t)6 * nsys);
    ctl_words = ctl_bytes / sizeof(int);
    for (int s = 0; s < nsys; ++s) {
      SysBuf& b = sb[s];
      b.cg_s = dry ? nullptr : cg_all + (size_t)s * CG_NSLOT;
      b.stat = dry ? nullptr : stat_all + (size_t)s * 4;
      b.ms_b_stat = (dry || !pl.gw) ? nullptr : stat_all + (size_t)(nsys + s) * 4;
      b.tb_stat = (dry || !pl.gwx) ? nullptr : stat_all + (size_t)(2 * nsys + s) * 4;
      b.dstat = dry ? nullptr : dstat_all + (size_t)s * 2;
      b.h_ctl = dry ? nullptr : ctl_all + (size_t)s * 4;
      b.ms_b_dstat = (dry || !pl.gw) ? nullptr : dstat_all + (size_t)(nsys + s) * 2;
      b.ms_b_h_ctl = (dry || !pl.gw) ? nullptr : ctl_all + (size_t)(nsys + s) * 4;
      b.tb_dstat = (dry || !pl.gwx) ? nullptr : dstat_all + (size_t)(2 * nsys + s) * 2;
      b.tb_h_ctl = (dry || !pl.gwx) ? nullptr : ctl_all + (size_t)(2 * nsys + s) * 4;
    }
    // one region, uploaded with one copy (upload_tables)
    ntab = pl.solve ? T_NT : 2;
    tables = (SysDev*)bp.take(sizeof(SysDev) * ntab * nsys);
    const size_t up0 = bp.off - sizeof(SysDev) * ntab * nsys;
    bmap = (int*)bp.take(sizeof(int) * (size_t)nb_total);
    gwtab = pl.gw ? (SysDev*)bp.take(sizeof(SysDev) * 2 * nsys) : nullptr;
    trgwtab = pl.gwx ? (SysDev*)bp.take(sizeof(SysDev) * 2 * nsys) : nullptr;
    gwbmap = (pl.gw || pl.gwx) ? (int*)bp.take(sizeof(int) * 2 * (size_t)nb_total) : nullptr;
    up_bytes = bp.off - up0;
    up_head = up0 - stat0;
    return bp.off + 256;
  }
};

void clear_graphs(ov_ctx* c) {
  for (auto& kv : c->graphs) (void)hipGraphExecDestroy(kv.second);
  c->graphs.clear();
}

ov_status ensure_ws(ov_ctx* c, size_t need, void** base) {
  if (c->noalloc) {  // ov_apply_noalloc: the device's scratch array, never an allocation
    void* p = (c->device >= 0 && c->device < kMaxDevices) ? g_scratch_dev[c->device] : nullptr;
    if (!p) {
      c->err = "no-allocation scratch has no device address on this device";
      return OV_ERR_DEVICE;
    }
    if (need > (size_t)OV_NOALLOC_SCRATCH_BYTES) {
      char buf[200];
      std::snprintf(buf, sizeof buf,
                    "no-allocation scratch of %zu bytes is too small: this call needs %zu",
                    (size_t)OV_NOALLOC_SCRATCH_BYTES, need);
      c->err = buf;
      return OV_ERR_WORKSPACE;
    }
    *base = p;
    return OV_OK;
  }
  if (c->user_ws) {  // a caller-owned workspace is never supplemented by a hidden allocation
    if (c->user_ws_bytes < need) {
      char buf[160];
      std::snprintf(buf, sizeof buf, "workspace of %zu bytes is too small: this call needs %zu",
                    c->user_ws_bytes, need);
      c->err = buf;
      return OV_ERR_WORKSPACE;
    }
    *base = c->user_ws;
    return OV_OK;
  }
  if (c->own_ws_bytes < need) {
    clear_graphs(c);
    if (c->own_ws) (void)hipFree(c->own_ws);
    c->own_ws = nullptr;
    c->own_ws_bytes = 0;
    HIPCHK(c, hipMalloc(&c->own_ws, need));
    c->own_ws_bytes = need;
  }
  *base = c->own_ws;
  return OV_OK;
}

// Pinned memory a context starts with, one allocation: scalars and flags of kNoAllocSystems
// systems, the staging, and the abort word of the resident launches.
constexpr size_t kHostScalars = sizeof(double) * (CG_NSLOT + 24) * kNoAllocSystems;
constexpr size_t kHostFlags = 256;  // two ints per system
static_assert(2 * kNoAllocSystems * sizeof(int) <= kHostFlags, "flags");
static_assert(kNoAllocSystems * (2 * sizeof(SysDev) + 256) + 16384 <= kNoAllocStage, "tables");
constexpr size_t kHostBlock = kHostScalars + kHostFlags + kNoAllocStage + 64;
ov_status host_setup(ov_ctx* c) {
  HIPCHK(c, hipHostMalloc((void**)&c->host_block, kHostBlock));
  c->pinned = (double*)c->host_block;
  c->pinned_flags = (int*)(c->host_block + kHostScalars);
  c->pinned_n = kNoAllocSystems;
  c->stage = c->host_block + kHostScalars + kHostFlags;
  c->stage_cap = kNoAllocStage;
  c->res_abort = (int*)(c->stage + kNoAllocStage);
  *c->res_abort = 0;
  return OV_OK;
}

// Frees pinned memory a context has grown (not its first block).
void host_free(ov_ctx* c, void* p) {
  if (p && !((char*)p >= c->host_block && (char*)p < c->host_block + kHostBlock))
    (void)hipHostFree(p);
}

ov_status ensure_pinned(ov_ctx* c, int nsys) {
  if (c->pinned_n >= nsys) return OV_OK;
  if (c->noalloc) {
    char buf[120];
    std::snprintf(buf, sizeof buf, "no-allocation calls take at most %d right-hand sides",
                  c->pinned_n);
    c->err = buf;
    return OV_ERR_WORKSPACE;
  }
  host_free(c, c->pinned);
  host_free(c, c->pinned_flags);
  c->pinned = nullptr;
  c->pinned_flags = nullptr;
  HIPCHK(c, hipHostMalloc((void**)&c->pinned, sizeof(double) * (CG_NSLOT + 24) * nsys));
  HIPCHK(c, hipHostMalloc((void**)&c->pinned_flags, sizeof(int) * 2 * nsys + 64));
  c->pinned_n = nsys;
  return OV_OK;
}

// Device address of the no-allocation scratch array on the context's device: looked
// up once per device (with that device current: contexts are created on the current
// device) and kept for the life of the process.
ov_status noalloc_scratch_setup(ov_ctx* c) {
  if (c->device < 0 || c->device >= kMaxDevices) {
    c->err = "device ordinal beyond the no-allocation scratch table";
    return OV_ERR_DEVICE;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[c->device]) return OV_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    c->err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
    return OV_ERR_DEVICE;
  }
  g_scratch_dev[c->device] = ptr;
  return OV_OK;
}

MsParams make_mp(const ov_ctx* c, double tol, int cap) {
  MsParams m{};
  m.np = c->p.n_poles;
  m.cap = cap;
  m.tol = tol;
  m.diag = 4.0 - c->p.M0;
  for (int k = 0; k < MAXP; ++k) {
    m.sigma[k] = k < m.np ? c->b[k] : 0.0;
    m.coef[k] = k < m.np ? c->a[k] : 0.0;
  }
  return m;
}

ResGate<ov_ctx> g_res_gate[kMaxDevices];

// Enqueues context c's resident work in the order of its device's gate.  An event on the
// other stream costs nothing while one context launches; without it, wait on the host.
template <class F>
auto res_ordered(ov_ctx* c, F&& enqueue) {
  if (c->device < 0 || c->device >= kMaxDevices) return enqueue();
  return g_res_gate[c->device].pass(
      c,
      [c](ov_ctx* last) {
        hipError_t e = hipEventRecord(last->ev_res, last->priv);
        if (e == hipSuccess) e = hipStreamWaitEvent(c->priv, last->ev_res, 0);
        if (e != hipSuccess) e = hipStreamSynchronize(last->priv);
        if (e != hipSuccess) c->gate_err = e;  // check_launch
      },
      enqueue);
}

template <class R>
const void* res_kernel(int K) {
  if constexpr (sizeof(R) == sizeof(float))  // FP64 with two sites per thread would spill
    if (K > 1) return (const void*)k_ms_res<R, 2>;
  return (const void*)k_ms_res<R, 1>;
}

// Set-up of the resident multi-shift kernel: the lattice's decompositions, the epoch word,
// abort word and slots, and the wait limit (OV_RES_WAIT_US at context creation; half a
// second is far beyond any pass and short enough for a caller that lost the race with
// another process for the chip).
ov_status res_setup(ov_ctx* c) {
  const char* ep = std::getenv("OV_PERSISTENT");
  c->resident = !(ep && *ep == '0');
  int cus = 0, khz = 0;
  HIPCHK(c, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device));
  HIPCHK(c, hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, c->device));
  c->res_cus = std::min(cus, RES_WGS);
  const char* ew = std::getenv("OV_RES_WAIT_US");
  const double us = ew ? std::atof(ew) : 5e5;
  c->res_spin = (long long)(us * khz * 1e-3);
  c->rg[0] = res_geom(c->p.dims, 16, c->res_cus, 1);
  c->rg[1] = res_geom(c->p.dims, 8, c->res_cus, 2);
  const void* kern[] = {res_kernel<double>(1), res_kernel<float>(1), res_kernel<float>(2)};
  for (const void* k : kern)
    HIPCHK(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, RES_MAX_LDS));
  const void* fft[] = {(const void*)k_fft_xy<double, 4>, (const void*)k_fft_xy<float, 4>,
                       (const void*)k_fft_xy<double, 3>, (const void*)k_fft_z<double, 4>,
                       (const void*)k_fft_z<float, 4>,   (const void*)k_fft_z<double, 3>,
                       (const void*)k_fft_zt<double, 4>, (const void*)k_fft_zt<float, 4>,
                       (const void*)k_fft_zt<double, 3>};
  for (const void* k : fft)
    HIPCHK(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, FFT_LDS));
  HIPCHK(c, hipMalloc((void**)&c->res_sh, sizeof(ResShared)));
  HIPCHK(c, hipMemsetAsync(c->res_sh, 0, sizeof(ResShared), c->priv));
  HIPCHK(c, hipEventCreateWithFlags(&c->ev_res, hipEventDisableTiming));
  return OV_OK;
}

// Run a call; when a resident launch gave up waiting (another process held part of the
// chip), run it again with the per-pass kernels.  The calls write no output that may lie on
// an input before they know of the expiry.  A batch's engine is led by its first member, the
// FP64 solver that finishes some of its members by the first of those: any of the call's
// contexts may have given up.
template <class F>
ov_status res_retry(ov_ctx* const* cs, size_t n, F&& call) {
  const ov_status rc = call();
  bool gave_up = false;
  for (size_t k = 0; k < n; ++k) gave_up |= cs[k] && *cs[k]->res_abort;
  if (!gave_up) return rc;
  std::vector<std::pair<ov_ctx*, bool>> was;  // (context, resident) of each, once
  for (size_t k = 0; k < n; ++k) {
    ov_ctx* c = cs[k];
    bool seen = false;
    for (const auto& w : was) seen |= w.first == c;
    if (!c || seen) continue;
    was.push_back({c, c->resident});
    if (*c->res_abort) {
      HIPCHK(c, hipStreamSynchronize(c->priv));
      *c->res_abort = 0;
      k_zero32<<<1, 64, 0, c->priv>>>(&c->res_sh->abort, 1);
      if (++c->res_aborts >= 3) was.back().second = false;
    }
  }
  for (const auto& w : was) w.first->resident = false;
  const ov_status again = call();
  for (const auto& w : was) w.first->resident = w.second;
  return again;
}
template <class F>
ov_status res_retry(ov_ctx* c, F&& call) {
  return res_retry(&c, 1, std::forward<F>(call));
}

// The plan of a call (buffers, basis capacities, multi-shift parameters) for `ctxs`
// (one entry per system).  Host only: engine_init carves it, the workspace queries size it.
void plan_engine(Engine& E, const std::vector<ov_ctx*>& ctxs, bool solve, bool mixed,
                 double tol64, double tolR, int nshift) {
  E.ctxs = ctxs;
  E.nsys = (int)ctxs.size();
  E.sb.assign(E.nsys, SysBuf{});
  E.lead = ctxs[0];
  E.block = 0;
  for (const ov_ctx* c : ctxs) E.block = std::max(E.block, c->block);
  E.st = E.lead->priv;
  E.pl.solve = solve;
  E.pl.mixed = mixed;
  E.pl.nshift = solve ? nshift : 0;
  // the shifted systems of the rational layers are not preconditioned
  E.pl.pc = solve && nshift == 0 && E.lead->p.precondition != 0;
  E.pl.fft = solve && E.lead->p.dirac != OV_DIRAC_OVERLAP_MS;
  E.pl.gw = solve && !E.pl.fft && nshift == 0 && E.lead->p.inner_form == 1;
  E.pl.gwx = solve && !E.pl.fft && E.lead->p.inner_form == 1;
  // capacities from the loosest spectral bound over the batch (no multi-shift
  // basis for a momentum-space operator).  The exact Ginsparg-Wilson product runs its
  // multi-shift ten times tighter than the tolerance it serves (truth_ms_tol), so the
  // FP64 basis is sized for that.
  const double cap_tol64 = E.pl.gwx ? 0.1 * tol64 : tol64;
  int cap64 = 0, capR = 0;
  for (auto* c : ctxs) {
    cap64 = std::max(cap64, capacity(c, cap_tol64));
    if (solve) capR = std::max(capR, capacity(c, tolR));
  }
  E.pl.cap64 = solve && !mixed ? std::max(cap64, capR) : cap64;
  E.pl.capR = solve ? (mixed ? capR : E.pl.cap64) : 0;
  if (E.pl.fft) E.pl.cap64 = E.pl.capR = 0;
  E.mp64 = make_mp(E.lead, tol64, E.pl.cap64);
  E.mpR = make_mp(E.lead, tolR, solve ? E.pl.capR : E.pl.cap64);
  E.L64 = E.pl.cap64;
  E.LR = solve ? E.pl.capR : E.pl.cap64;
}

// Tolerances of the solve plan (ov_solve, ov_solve_batch, ov_force).
double solve_tol64(const ov_ctx* c) { return std::min(c->p.inner_tol, c->p.truth_tol); }
double solve_tolR(const ov_ctx* c) {
  return c->p.precision == OV_MIXED ? c->p.mixed_inner_tol : c->p.inner_tol;
}

// Build the engine for `ctxs` (one entry per system) and carve the workspace.
ov_status engine_init(Engine& E, const std::vector<ov_ctx*>& ctxs, bool solve, bool mixed,
                      double tol64, double tolR, int nshift = 0) {
  plan_engine(E, ctxs, solve, mixed, tol64, tolR, nshift);
  for (int& k : E.lead->ev_call_count) k = 0;
  HIPCHK(E.lead, hipEventRecord(E.lead->ev_in, E.lead->stream));
  HIPCHK(E.lead, hipStreamWaitEvent(E.st, E.lead->ev_in, 0));
  size_t need = E.layout(nullptr, 0, true);
  const size_t limit = E.lead->noalloc   ? (size_t)OV_NOALLOC_SCRATCH_BYTES
                       : E.lead->user_ws ? E.lead->user_ws_bytes
                                         : (size_t)-1;
  if (need > limit && E.resident_any()) {  // no room for the faces: the per-pass kernels
    E.no_res = true;
    need = E.layout(nullptr, 0, true);
  }
  void* base = nullptr;
  TRY(ensure_ws(E.lead, need, &base));
  E.layout(base, need, false);
  TRY(ensure_pinned(E.lead, E.nsys));
  return OV_OK;
}

SysDev base_dev(const SysBuf& b) {
  SysDev d{};
  const ov_params& p = b.ctx->p;
  d.g = Geo{p.dims[0], p.dims[1], p.dims[2], p.dims[3], b.V, p.bc_t};
  d.nblk = b.nblk;
  d.blk0 = b.blk0;
  d.spb = b.spb;
  d.part_a = b.part_a;
  d.part_b = b.part_b;
  d.part_c = b.part_c;
  d.h_rho = b.h_rho;
  d.h_alpha = b.h_alpha;
  d.h_zeta = b.h_zeta;
  d.h_active = b.h_active;
  d.h_ctl = b.h_ctl;
  d.stat = b.stat;
  d.dstat = b.dstat;
  d.coef_term = b.coef_term;
  d.coef_c = b.coef_c;
  d.coef_d = b.coef_d;
  d.cg_s = b.cg_s;
  d.m_re = p.m_re;
  d.m_im = p.m_im;
  d.pc_re = p.m_re;  // the free-field operator of the action's mass (ov_apply M0INV)
  d.pc_im = p.m_im;
  d.g_re = p.g_re;
  d.g_im = p.g_im;
  d.shx = b.shx;
  d.shp = b.shp;
  d.shc = b.shc;
  d.nshift = b.nshift;
  d.pcs = b.pcs;
  d.xc = b.xc;
  d.off_xy = b.off_xy;
  d.off_z = b.off_z;
  d.off_t = b.off_t;
  d.off_zt = b.off_zt;
  return d;
}

// Pinned staging of at least `bytes`, free to be written.
ov_status ensure_stage(ov_ctx* c, size_t bytes) {
  if (c->stage_busy) HIPCHK(c, hipStreamSynchronize(c->priv));
  c->stage_busy = false;
  if (c->stage_cap >= bytes) return OV_OK;
  if (c->noalloc) {
    c->err = "no-allocation call: the host staging is too small";
    return OV_ERR_WORKSPACE;
  }
  host_free(c, c->stage);
  c->stage = nullptr;
  c->stage_cap = 0;
  HIPCHK(c, hipHostMalloc((void**)&c->stage, bytes));
  c->stage_cap = bytes;
  return OV_OK;
}

// The engine's host tables to the device: one asynchronous copy from pinned memory (a copy
// per table, each waited for, took 20 us of a call that runs 60 us of kernels).
// With `clear` it zeroes the counters and control words in front of them as well (reset_stats).
ov_status upload_tables(Engine& E, bool clear = false) {
  ov_ctx* c = E.lead;
  const size_t head = clear ? E.up_head : 0;
  TRY(ensure_stage(c, head + E.up_bytes));
  std::memset(c->stage, 0, head);
  char* const base = c->stage + head;
  auto at = [&](const void* dev) { return base + ((const char*)dev - (const char*)E.tables); };
  std::memcpy(base, E.htab.data(), sizeof(SysDev) * (size_t)E.ntab * E.nsys);
  if (!E.io.empty())
    for (int s = 0; s < E.nsys; ++s) {
      for (int t : {(int)T_APPLY, (int)T_APPLY2}) {
        SysDev& d = ((SysDev*)base)[(size_t)t * E.nsys + s];
        d.io_in = (const double2*)E.io[s].in;
        d.io_pin = E.io[s].pin;
        d.io_pout = E.io[s].pout;
        d.io_out = (double2*)E.io[s].out;
      }
    }
  int* m = (int*)at(E.bmap);
  for (int s = 0; s < E.nsys; ++s)
    for (int b = 0; b < E.sb[s].nblk; ++b) *m++ = s;
  if (E.pl.gw && E.hgwtab.size() == 2 * (size_t)E.nsys)
    std::memcpy(at(E.gwtab), E.hgwtab.data(), sizeof(SysDev) * E.hgwtab.size());
  if (E.pl.gwx && E.htrgw.size() == 2 * (size_t)E.nsys)
    std::memcpy(at(E.trgwtab), E.htrgw.data(), sizeof(SysDev) * E.htrgw.size());
  if (E.gwbmap) {
    m = (int*)at(E.gwbmap);
    for (int s = 0; s < 2 * E.nsys; ++s)
      for (int b = 0; b < E.sb[s % E.nsys].nblk; ++b) *m++ = s;
  }
  HIPCHK(c, hipMemcpyAsync((char*)E.tables - head, c->stage, head + E.up_bytes,
                           hipMemcpyHostToDevice, E.st));
  c->stage_busy = true;
  if (E.shifts && E.face_bytes) {  // a multiple of 64 bytes: whole face values of a block
    const size_t n = E.face_bytes / sizeof(u32x4);
    k_res_empty<<<(unsigned)std::min<size_t>((n + 255) / 256, 1024), 256, 0, E.st>>>((u32x4*)E.face, n);
  }
  return OV_OK;
}

const SysDev* tab(const Engine& E, int t) { return E.tables + (size_t)t * E.nsys; }

// ----------------------------------------------------------------- launches
// Event pair around one launch when sampling is on (first sample_max per kernel and call).
struct Sample {
  ov_ctx* c;
  int k;
  bool on = false;
  Sample(ov_ctx* c_, int k_, double bytes) : c(c_), k(k_) {
    if (c->sample_max <= 0 || c->ev_call_count[k] >= c->sample_max) return;
    const size_t idx = c->ev_use.size();
    if (2 * idx + 2 > c->ev_pool.size()) {
      hipEvent_t a, b;
      if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return;
      c->ev_pool.push_back(a);
      c->ev_pool.push_back(b);
    }
    c->ev_use.push_back({k, bytes, 0, 0.0});
    c->ev_call_count[k]++;
    on = hipEventRecord(c->ev_pool[2 * idx], c->priv) == hipSuccess;
  }
  ~Sample() {
    if (on) (void)hipEventRecord(c->ev_pool[2 * (c->ev_use.size() - 1) + 1], c->priv);
  }
};

// Stamp regions (start, end, sites per workgroup) for the sampled launches of a call.
void ensure_stamps(ov_ctx* c, int blocks) {
  const size_t region = 3 * (size_t)blocks;
  const size_t regions = 4 * (size_t)c->sample_max + 2;
  if (c->ts_region < region || c->ts_regions < regions) {
    if (c->ts_dev) (void)hipFree(c->ts_dev);  // synchronises the device
    c->ts_dev = nullptr;
    c->ts_region = std::max(region, c->ts_region);
    c->ts_regions = std::max(regions, c->ts_regions);
    if (hipMalloc((void**)&c->ts_dev, sizeof(unsigned long long) * c->ts_region * c->ts_regions) !=
        hipSuccess) {
      c->ts_dev = nullptr;
      c->ts_region = c->ts_regions = 0;
    }
  }
  if (c->wall_khz <= 0) {
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, c->device) == hipSuccess)
      c->wall_khz = khz;
  }
}

// Collect the sampled durations after the stream has been synchronised.
void collect_samples(ov_ctx* c) {
  for (size_t i = 0; i < c->ev_use.size(); ++i) {
    const auto& u = c->ev_use[i];
    // device stamps: (start, end, sites processed) per workgroup
    double frac = 1.0;  // share of the launch's sites that were processed
    if (u.ts_blocks > 0 && c->ts_dev && c->wall_khz > 0 && i < c->ts_regions) {
      std::vector<unsigned long long> h(3 * (size_t)u.ts_blocks);
      if (hipMemcpy(h.data(), c->ts_dev + i * c->ts_region, sizeof(unsigned long long) * h.size(),
                    hipMemcpyDeviceToHost) == hipSuccess) {
        unsigned long long lo = ~0ull, hi = 0, sites = 0;
        for (int b = 0; b < u.ts_blocks; ++b) {
          lo = std::min(lo, h[3 * b]);
          hi = std::max(hi, h[3 * b + 1]);
          sites += h[3 * b + 2];
        }
        if (u.sites > 0) frac = std::min(1.0, (double)sites / u.sites);
        if (hi > lo) {
          c->ksum_kernel_ms[u.kernel] += (double)(hi - lo) / c->wall_khz;
          c->kcount_kernel[u.kernel]++;
        }
      }
    }
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev_pool[2 * i], c->ev_pool[2 * i + 1]) == hipSuccess) {
      c->ksum_ms[u.kernel] += ms;
      c->ksum_bytes[u.kernel] += u.bytes * frac;
      c->kcount[u.kernel]++;
    }
  }
  c->ev_use.clear();
  for (int& k : c->ev_call_count) k = 0;
}

template <class R>
void launch_resident(const Engine& E, const SysDev* T, const ResPlan& P, const MsParams& mp,
                     int L) {
  ov_ctx* c = E.lead;
  if (c->sample_max > 0) ensure_stamps(c, 2 * E.nb_total);
  const unsigned range = 2 * (unsigned)L + 4;  // epochs of one launch
  auto enqueue = [&]() {
    unsigned eoff = 0;
    int nent = 0;
    for (const ResLaunch& l : P.launches) {
      ResArgs a{};
      a.nrun = l.nrun;
      a.L = L;
      a.eoff = eoff;
      a.nap = l.nap();
      a.nap_face = l.nap_face();
      a.sh = c->res_sh;
      a.abort_host = c->res_abort;
      a.face = E.face;
      a.spin = c->res_spin;
      std::copy(l.run, l.run + l.nrun, a.run);
      MsParams m = mp;
      const SysDev* Tp = T;
      void* args[] = {(void*)&Tp, (void*)&a, (void*)&m};
      const int e0 = nent;
      double vol = 0.0;
      for (int k = 0; k < l.nrun; ++k) {
        nent += l.run[k].ne;
        vol += (double)l.run[k].ne * E.sb[l.run[k].e0 % E.nsys].V;
      }
      bool sampled;
      {
        Sample smp(c, 2, 0.0);
        (void)hipLaunchKernel(res_kernel<R>(l.K), dim3(l.grid), dim3(l.threads + 64), args, l.lds, E.st);
        sampled = smp.on;
      }
      const size_t idx = c->ev_use.size() - 1;
      if (sampled && c->ts_dev && idx < c->ts_regions) {
        // written per iteration: t_n of every entry that still iterates, counted behind it
        auto& u = c->ev_use[idx];
        u.ts_blocks = 1;
        u.sites = vol * L;
        u.bytes = 4.0 * sizeof(c2<R>) * u.sites;
        k_res_sites<<<1, 64, 0, E.st>>>(T + e0, nent - e0, L, c->ts_dev + idx * c->ts_region);
      }
      eoff += range;
    }
    k_ms_coef<<<nent, COEF_THREADS, 0, E.st>>>(T, nent, L, mp, ResEpoch{c->res_sh, eoff});
  };
  if (c->capturing)
    enqueue();  // run_graph has the gate
  else
    res_ordered(c, enqueue);
}

template <class R>
// Multi-shift solves of `nent` table entries (nent / E.nsys entries per system,
// laid out system-major per copy) over nbt workgroups mapped by bmap.
void launch_ms_tab(const Engine& E, const SysDev* T, const int* bmap_, int nbt_, int nent,
                   const MsParams& mp, int L) {
  const int copies = nent / E.nsys;
  double vol = 0.0;  // sites in this launch (all entries)
  for (const auto& b : E.sb) vol += (double)b.V * copies;
  const double bytes = 3.0 * 4.0 * sizeof(c2<R>) * vol;  // per pass
  ov_ctx* c = E.lead;
  if (const ResPlan* pl = E.resident<R>(copies)) {
    launch_resident<R>(E, T, *pl, mp, L);
    return;
  }
  // z-marching passes when every system's workgroup owns whole xy planes of one
  // time slice (X Y == threads per workgroup, sites per thread zc >= 2 dividing Z);
  // OV_MS_ZM=0 switches them off
  MsParams mps = mp;
  // t_n and r_{n+1} past the caches where the three fields of a pass exceed the 256 MiB
  // last-level cache (FP64 sign, cached against streaming stores: 24^3 x 48, 127 MB, 6.99
  // and 7.03 ms, 20^3 x 40, 61 MB, 3.57 and 3.76; 12 fields of 16^3 x 32, 302 MB, 12.7 and
  // 12.2, 8 of 16^2 x 32^2, 403 MB, 16.9 and 15.2, 8 of 16^3 x 64 17.4 and 16.2, two of 32^4
  // 23.0 and 21.6; at 201 and 255 MB either by 3 % or less)
  mps.nt = bytes > 256.0 * (1 << 20);
  size_t shb = 0;
  {
    int zc = 0;
    bool ok = ms_zm_enabled();
    for (const auto& b : E.sb) {
      const ov_params& p = b.ctx->p;
      const int XY = p.dims[0] * p.dims[1];
      const int k = b.spb / E.block;
      ok &= XY == E.block && b.spb == k * E.block && k >= 2 && p.dims[2] % k == 0 &&
            (zc == 0 || zc == k);
      zc = k;
    }
    mps.zm = ok ? zc : 0;
    shb = ok ? (size_t)4 * E.block * sizeof(c2<R>) : 0;
  }
  if (c->sample_max > 0) ensure_stamps(c, nbt_);
  auto stamped = [&](Sample& smp) -> MsParams {
    MsParams m = mps;
    const size_t idx = c->ev_use.size() - 1;
    if (smp.on && c->ts_dev && idx < c->ts_regions) {
      m.tstamp = c->ts_dev + idx * c->ts_region;
      c->ev_use[idx].ts_blocks = nbt_;
      c->ev_use[idx].sites = vol;
    }
    return m;
  };
  // z-marching (with the next plane prefetched in FP32), else the plain passes
  const bool zmode = mps.zm > 0;
  constexpr int ZMF = sizeof(R) == sizeof(float) ? 2 : 1;  // the z-marching form of R
  // batched launches check their flags before reading operands: the plain ones of any size
  // (the uneven batch of 8^4 to 24^3 x 48, mixed: 229 -> 217 ms), z-marching ones when large
  const bool cf = (zmode ? nbt_ >= 2048 : E.nsys > 1) && ms_cf_enabled();
  // lattices of several sizes converge at different times: every XCD takes a share of each
  // (same batch: 217 -> 195 ms); equal ones stay whole in an XCD's L2 (24^3 x 48, one
  // mixed solve: 159 against 162)
  for (const ov_ctx* o : E.ctxs) mps.share |= !std::equal(o->p.dims, o->p.dims + 4, c->p.dims);
  for (int n = 0; n < L; ++n) {
    {
      Sample smp(c, sizeof(R) == sizeof(double) ? 3 : 0, bytes);
      if (zmode && cf)
        k_ms_t<R, ZMF, true><<<nbt_, E.block, shb, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
      else if (zmode)
        k_ms_t<R, ZMF, false><<<nbt_, E.block, shb, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
      else if (cf)
        k_ms_t<R, 0, true><<<nbt_, E.block, 0, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
      else
        k_ms_t<R, 0, false><<<nbt_, E.block, 0, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
    }
    {
      Sample smp(c, sizeof(R) == sizeof(double) ? 4 : 1, bytes);
      if (zmode && cf)
        k_ms_r<R, ZMF, true><<<nbt_, E.block, shb, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
      else if (zmode)
        k_ms_r<R, ZMF, false><<<nbt_, E.block, shb, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
      else if (cf)
        k_ms_r<R, 0, true><<<nbt_, E.block, 0, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
      else
        k_ms_r<R, 0, false><<<nbt_, E.block, 0, E.st>>>(T, bmap_, nbt_, n, stamped(smp));
    }
  }
  k_ms_coef<<<nent, COEF_THREADS, 0, E.st>>>(T, nent, L, mp, ResEpoch{});
}

template <class R>
void launch_ms(const Engine& E, int t, const MsParams& mp, int L) {
  launch_ms_tab<R>(E, tab(E, t), E.bmap, E.nb_total, E.nsys, mp, L);
}

template <class R>
void launch_combine(const Engine& E, int t, int mode, int aos = 0) {
  // groups per site: as many as fit 512 threads, four at most (whole calls with 1, 2, 4, 8
  // groups: sign 4^4 120, 113, 106, 111 us, M 8^4 476, 462, 457, 457; 16^4 in 256 threads,
  // MdagM, 1648, 1609 with 1 and 2)
  const int jw = std::min(4, 512 / E.block);
  k_ms_combine<R><<<E.nb_total, E.block * jw, sizeof(double2) * 4 * E.block * (jw - 1), E.st>>>(
      tab(E, t), E.bmap, mode, jw, aos);
}

SymParams sym_params(const ov_ctx* c, int kind) {
  SymParams sp{};
  sp.kind = kind;
  sp.form = c->p.dirac == OV_DIRAC_OVERLAP_EXACT ? DIRAC_EXACT
            : c->p.dirac == OV_DIRAC_DSLASH      ? DIRAC_DSLASH
                                                 : DIRAC_RATIONAL;
  sp.np = c->p.n_poles;
  sp.diag = 4.0 - c->p.M0;
  for (int k = 0; k < MAXP; ++k) {
    sp.a[k] = k < sp.np ? c->a[k] : 0.0;
    sp.b[k] = k < sp.np ? c->b[k] : 0.0;
  }
  sp.periodic = kind == SYM_BOSON ? 1 : 0;  // scalar fields are periodic in time
  return sp;
}

// x, y, z transforms of systems [s0, s0 + ns) of spatial extents d through one
// fixed-length kernel; false when no kernel has these extents (FP64 24^3 does not fit
// in LDS).
template <class R, int NX, int NY, int NZ>
void xyz_launch(const Engine& E, const SysDev* T, int s0, int ns, int nt, int inv, int periodic) {
  const unsigned grid = (unsigned)(4 * nt * ns);
  if (inv)
    k_fft_xyz<R, NX, NY, NZ, 1><<<grid, 256, 0, E.st>>>(T, s0, periodic);
  else
    k_fft_xyz<R, NX, NY, NZ, 0><<<grid, 256, 0, E.st>>>(T, s0, periodic);
}

template <class R>
bool xyz_fixed(const Engine* E, const SysDev* T, int s0, int ns, const int* d, int inv,
               int periodic) {
  struct Shape {
    int x, y, z;
    void (*go)(const Engine&, const SysDev*, int, int, int, int, int);
  };
  static const Shape shapes[] = {
      {4, 4, 4, xyz_launch<R, 4, 4, 4>},       {8, 8, 8, xyz_launch<R, 8, 8, 8>},
      {12, 12, 12, xyz_launch<R, 12, 12, 12>}, {16, 16, 16, xyz_launch<R, 16, 16, 16>},
      {16, 16, 8, xyz_launch<R, 16, 16, 8>},
  };
  for (const Shape& sh : shapes)
    if (d[0] == sh.x && d[1] == sh.y && d[2] == sh.z) {
      if (E) sh.go(*E, T, s0, ns, d[3], inv, periodic);
      return true;
    }
  if (sizeof(R) == sizeof(float) && d[0] == 24 && d[1] == 24 && d[2] == 24) {
    if (E) xyz_launch<float, 24, 24, 24>(*E, T, s0, ns, d[3], inv, periodic);
    return true;
  }
  return false;
}

template <class R, int NT>
void tpcg_launch(const Engine& E, const SysDev* T, int s0, int ns, int xyz) {
  const int nchunk = (xyz + 63) / 64;
  k_fft_t_pcg<R, NT><<<(unsigned)(4 * nchunk * ns), 64, 0, E.st>>>(T, s0, nchunk);
}

template <class R>
bool tpcg_fixed(const Engine* E, const SysDev* T, int s0, int ns, const int* d) {
  const int xyz = d[0] * d[1] * d[2];
  switch (d[3]) {
    case 4: if (E) tpcg_launch<R, 4>(*E, T, s0, ns, xyz); return true;
    case 8: if (E) tpcg_launch<R, 8>(*E, T, s0, ns, xyz); return true;
    case 12: if (E) tpcg_launch<R, 12>(*E, T, s0, ns, xyz); return true;
    case 16: if (E) tpcg_launch<R, 16>(*E, T, s0, ns, xyz); return true;
    case 24: if (E) tpcg_launch<R, 24>(*E, T, s0, ns, xyz); return true;
    case 32: if (E) tpcg_launch<R, 32>(*E, T, s0, ns, xyz); return true;
    case 48:
      if (sizeof(R) != sizeof(float)) return false;  // 48 FP64 values per thread spill
      if (E) tpcg_launch<float, 48>(*E, T, s0, ns, xyz);
      return true;
    default: return false;
  }
}

// Runs of consecutive systems on one lattice (same extents and time boundary).
void lattice_runs(const Engine& E, std::vector<std::pair<int, int>>& runs) {
  runs.clear();
  for (int s = 0; s < E.nsys; ++s) {
    const ov_params& p = E.sb[s].ctx->p;
    if (!runs.empty()) {
      const ov_params& q = E.sb[runs.back().first].ctx->p;
      if (std::equal(p.dims, p.dims + 4, q.dims) && p.bc_t == q.bc_t) {
        ++runs.back().second;
        continue;
      }
    }
    runs.push_back({s, 1});
  }
}

// z = P r of the preconditioned CG by the fixed-length kernels (three passes: x y z,
// t with the scale table, x y z inverse) when every system's extents have one.
template <class R>
bool pcg_fixed(const Engine& E, int t) {
  if (!E.lead->fft_fixed) return false;
  std::vector<std::pair<int, int>> runs;
  lattice_runs(E, runs);
  for (const auto& r : runs) {
    const int* d = E.sb[r.first].ctx->p.dims;
    if (!E.sb[r.first].pcs || !xyz_fixed<R>(nullptr, nullptr, 0, 0, d, 0, 0) ||
        !tpcg_fixed<R>(nullptr, nullptr, 0, 0, d))
      return false;
  }
  const SysDev* T = tab(E, t);
  for (const auto& r : runs)
    xyz_fixed<R>(&E, T, r.first, r.second, E.sb[r.first].ctx->p.dims, 0, 0);
  for (const auto& r : runs) tpcg_fixed<R>(&E, T, r.first, r.second, E.sb[r.first].ctx->p.dims);
  for (const auto& r : runs)
    xyz_fixed<R>(&E, T, r.first, r.second, E.sb[r.first].ctx->p.dims, 1, 0);
  return true;
}

// The preconditioner's scale per momentum of every system (once per solve: it depends
// on the preconditioner mass and the shift only).
void pcg_table(const Engine& E) {
  if (!E.pl.pc) return;
  k_pcg_table<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_PC_Z), E.bmap, E.nb_total,
                                                      sym_params(E.lead, SYM_PCG));
}

// Threads per workgroup of the site kernels of the solve (basis combinations, CG vector
// updates, true-residual finish): one site per thread up to 512, so that a single
// system's partition (two sites per thread of the passes' 256) keeps twice the waves in
// flight (16^4 mixed solve 15.1 -> 14.6 ms with the combinations alone).
int site_block(const Engine& E) {
  int spb = 0;
  for (const auto& b : E.sb) spb = std::max(spb, b.spb);
  spb = (spb + 63) / 64 * 64;
  return std::max(E.block, std::min(512, spb));
}

// e_out = op(e_in) for a momentum-space operator (forward DFTs, symbol, inverse
// DFTs through fft_tmp); e_out may alias e_in.
template <class R, int NS = 4>
void launch_sym(const Engine& E, int t, int kind, SymIo io = {}) {
  if (kind == SYM_PCG && pcg_fixed<R>(E, t)) return;
  const SymParams sp = sym_params(E.lead, kind);
  const SysDev* T = tab(E, t);
  // threads: the groups of a workgroup's lines in as few equal rounds as `most` threads allow
  auto threads = [](int items, int most) {
    const int rounds = (items + most - 1) / most;
    return ((items + rounds - 1) / rounds + 63) / 64 * 64;
  };
  int nxy = 64, nz = 64, nt = 64, nzt = 64;
  size_t lxy = 0, lz = 0, lzt = 0;
  for (const SysBuf& b : E.sb) {
    const int* d = b.ctx->p.dims;
    const int gx = dft_groups(d[0]), gy = dft_groups(d[1]), gz = dft_groups(d[2]), gt = dft_groups(d[3]);
    nxy = std::max(nxy, threads(NS * std::max(d[1] * gx, d[0] * gy), 512));
    nz = std::max(nz, threads(NS * d[0] * gz, 512));
    nt = std::max(nt, threads(std::max(NS * b.xc * gt, b.xc * d[3]), 256));
    nzt = std::max(nzt, threads(NS * std::max(d[3] * gz, d[2] * gt), 1024));
    lxy = std::max(lxy, sizeof(c2<R>) * (2 * NS * fft_xy_plane(d[0], d[1]) + d[0] + d[1]) + sizeof(double2));
    lz = std::max(lz, sizeof(c2<R>) * (NS * d[0] * d[2] + d[2]));
    lzt = std::max(lzt, sizeof(c2<R>) * (2 * NS * fft_xy_plane(d[2], d[3]) + d[2] + d[3]) +
                            sizeof(double2) * (d[2] + d[3]));
  }
  // the (z, t) line in one pass where LDS holds it; three passes over planes else (M of the
  // overlap_exact form: 22x14x10x26 103 against 124 us, 16^3 x 32 85 against 101, 4^2 x
  // 24 x 48, of 16 workgroups, 69 against 69)
  io.zt = lzt <= FFT_LDS;
  k_fft_xy<R, NS><<<E.nb_xy, nxy, lxy, E.st>>>(T, E.nsys, 0, sp.periodic, io);
  if (io.zt) {
    k_fft_zt<R, NS><<<E.nb_zt, nzt, lzt, E.st>>>(T, E.nsys, sp);
  } else {
    k_fft_z<R, NS><<<E.nb_z, nz, lz, E.st>>>(T, E.nsys, 0);
    k_fft_t_sym<R, NS><<<E.nb_t, nt, 0, E.st>>>(T, E.nsys, sp);
    k_fft_z<R, NS><<<E.nb_z, nz, lz, E.st>>>(T, E.nsys, 1);
  }
  k_fft_xy<R, NS><<<E.nb_xy, nxy, lxy, E.st>>>(T, E.nsys, 1, sp.periodic, io);
}

ov_status check_launch(ov_ctx* c) {
  hipError_t e = hipGetLastError();
  if (c->gate_err != hipSuccess) e = c->gate_err;
  c->gate_err = hipSuccess;
  if (e != hipSuccess) {
    c->err = std::string("kernel launch: ") + hipGetErrorString(e);
    return OV_ERR_DEVICE;
  }
  return OV_OK;
}

ov_status sync(Engine& E) {
  TRY(check_launch(E.lead));
  HIPCHK(E.lead, hipStreamSynchronize(E.st));
  E.lead->stage_busy = false;
  if (!E.lead->ev_use.empty()) collect_samples(E.lead);
  if (*E.lead->res_abort) {  // the caller runs again with the per-pass kernels (res_retry)
    E.lead->err = "resident multi-shift: a wait ran out";
    return OV_ERR_DEVICE;
  }
  return OV_OK;
}

// CG scalars, multi-shift counters, shift residuals and control words of every entry
// (the engine's contiguous scalar block) to the pinned host copy, then synchronise.
ov_status read_scalars(Engine& E) {
  static_assert(sizeof(long long) == sizeof(double), "counters share the scalar block");
  HIPCHK(E.lead, hipMemcpyAsync(E.lead->pinned, E.cg_all,
                                sizeof(double) * CG_NSLOT * E.nsys + sizeof(int) * E.ctl_words,
                                hipMemcpyDeviceToHost, E.st));
  return sync(E);
}

// Sticky multi-shift error bits (h_ctl[3]: bit 1 breakdown, bit 2 not converged within
// the launched iterations or the basis) of system s's entries, from the last
// read_scalars.
int sticky_bits(const Engine& E, int s) {
  const int* ctl = (const int*)((const double*)E.lead->pinned + (size_t)CG_NSLOT * E.nsys +
                                (size_t)18 * E.nsys);
  int b = 0;
  for (int e = 0; e < 3; ++e) b |= ctl[(size_t)(e * E.nsys + s) * 4 + 3];
  return b;
}

// Error bits, multi-shift iterations (every entry) and shift residual of system s, from the
// last read_scalars.
struct SysCtl {
  int bits;
  long long inner;
  double shift_res;
};
SysCtl sys_ctl(const Engine& E, int s) {
  const size_t ns = E.nsys;
  const long long* st = (const long long*)(E.lead->pinned + CG_NSLOT * ns);
  const double* ds = E.lead->pinned + (CG_NSLOT + 12) * ns;
  const int* ctl = (const int*)(E.lead->pinned + (CG_NSLOT + 18) * ns);
  SysCtl c{ctl[4 * s + 3], st[4 * s], ds[2 * s]};
  if (E.sb[s].ms_b_stat) {  // second multi-shift entry of the inner operator
    c.bits |= ctl[4 * (ns + s) + 3];
    c.inner += st[4 * (ns + s)];
  }
  if (E.sb[s].tb_stat) c.inner += st[4 * (2 * ns + s)];  // and of the true residuals
  return c;
}

// Counters, shift residuals and control words of every entry: one fill kernel.
ov_status reset_stats(Engine& E) {
  const size_t n = E.ctl_words;
  k_zero32<<<(unsigned)std::min<size_t>((n + 255) / 256, 64), 256, 0, E.st>>>(
      (unsigned int*)E.stat_all, n);
  return check_launch(E.lead);
}

// Zero a device buffer (a multiple of 4 bytes) with the fill kernel.
void zero_dev(const Engine& E, void* p, size_t bytes) {
  const size_t n = bytes / sizeof(unsigned int);
  const unsigned nb = (unsigned)std::max<size_t>(1, std::min<size_t>((n + 255) / 256, 4096));
  k_zero32<<<nb, 256, 0, E.st>>>((unsigned int*)p, n);
}

// The caller's fields to their planar twins and back (E.io, in the uploaded tables).
ov_status pack64(Engine& E) {
  k_pack<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  return check_launch(E.lead);
}

ov_status unpack64(Engine& E) {
  k_unpack<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  return check_launch(E.lead);
}

// --------------------------------------------------------- apply / sign
// Tables of an operator on x64 (planar FP64) with the result in r64.
ov_status run_apply(Engine& E, int op, const void* phi, bool direct, bool clear) {
  E.htab.assign((size_t)E.ntab * E.nsys, SysDev{});
  for (int s = 0; s < E.nsys; ++s) {
    SysBuf& b = E.sb[s];
    SysDev d = base_dev(b);
    d.phi = (const double2*)phi;
    d.basis = b.basis64;
    d.r = b.r64ms;
    SysDev d1 = d, d2 = d;
    // phase 1: operator on psi = x64
    d1.e_in = b.x64;
    d1.src = (op == OV_OP_DOV_DAG || op == OV_OP_M_DAG) ? (const void*)b.src64b
                                                        : (const void*)b.x64;
    d1.e_out = (op == OV_OP_MDAGM) ? (void*)b.u64 : (void*)b.r64;  // H_W: x64 -> r64 too
    d1.e_out2 = (op == OV_OP_MDAGM) ? (void*)b.src64b : nullptr;
    d1.fft_tmp = b.src64b;  // momentum-space ops: transform scratch
    d2.fft_tmp = b.src64b;
    // phase 2 (MdagM only): M^dag on u64, source g5 u64 = src64b
    d2.e_in = b.u64;
    d2.src = b.src64b;
    d2.e_out = b.r64;
    if (direct) d1.src_io = op == OV_OP_DOV_DAG || op == OV_OP_M_DAG ? 2 : 1;
    E.htab[(size_t)T_APPLY * E.nsys + s] = d1;
    E.htab[(size_t)T_APPLY2 * E.nsys + s] = d2;
  }
  return upload_tables(E, clear);
}

// H_W on the caller's fields (every system of an operator call is on one lattice).  The
// marching form reads a plane's neighbours once, from registers and LDS, but holds 228
// VGPRs, so it needs planes that fill its 256 threads and three workgroups per CU: whole
// calls, marching against plain, 16^4: 4 systems (256 workgroups) 64 against 59 us, 12
// (768) 89 against 103, 48 174 against 268; 6x22 planes, 12 systems 78 against 101; 4x4
// planes, 40 systems of 4^2x24x48 184 against 120.
void launch_hw_io(const Engine& E, double diag) {
  const int* d = E.lead->p.dims;
  const int plane = d[0] * d[1];
  const int zc = d[2] % 4 == 0 ? 4 : 2;
  const long nzm = (long)E.nsys * d[3] * (d[2] / zc);
  const SysDev* T = tab(E, T_APPLY);
  if (plane >= 128 && plane <= 256 && nzm >= 768) {
    if (zc == 4)
      k_hw_io_zm<4><<<nzm, 256, 0, E.st>>>(T, diag);
    else
      k_hw_io_zm<2><<<nzm, 256, 0, E.st>>>(T, diag);
  } else {
    k_hw_io<<<E.nb_total, E.block, 0, E.st>>>(T, E.bmap, E.nb_total, diag);
  }
}

ov_status apply_sequence(Engine& E, int op, bool direct) {
  const ov_ctx* c = E.lead;
  const double diag = 4.0 - c->p.M0;
  if (c->p.dirac != OV_DIRAC_OVERLAP_MS && op >= OV_OP_DOV && op <= OV_OP_MDAGM) {
    // momentum-space D and Y, on the caller's fields unless they overlap: then on the planar
    // copies (x64 -> r64); MdagM through u64
    const int nb = E.nb_total, bl = E.block;
    const bool dag = op == OV_OP_DOV_DAG || op == OV_OP_M_DAG;
    const int kind = dag ? SYM_D_DAG : SYM_D;
    const bool yuk = op >= OV_OP_M;
    SymIo io;
    io.in = direct;
    io.out = direct && op != OV_OP_MDAGM;
    io.yuk = direct && yuk ? 1 + dag : 0;
    launch_sym<double>(E, T_APPLY, kind, io);
    if (yuk && !direct) k_yuk<double><<<nb, bl, 0, E.st>>>(tab(E, T_APPLY), E.bmap, nb, dag);
    if (op == OV_OP_MDAGM) {
      io.in = 0;
      io.out = direct;
      io.yuk = direct ? 2 : 0;
      launch_sym<double>(E, T_APPLY2, SYM_D_DAG, io);
      if (!direct) k_yuk<double><<<nb, bl, 0, E.st>>>(tab(E, T_APPLY2), E.bmap, nb, 1);
    }
    return check_launch(E.lead);
  }
  switch (op) {
    case OV_OP_HW:  // in place, the stencil reads a planar copy
      if (direct)
        launch_hw_io(E, diag);
      else
        k_hw<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, diag, 0);
      break;
    case -1:  // sign
    case OV_OP_DOV:
    case OV_OP_M:
    case OV_OP_DOV_DAG:
    case OV_OP_M_DAG: {
      // on the caller's fields, a resident multi-shift takes its source from them too
      const bool dag = op == OV_OP_DOV_DAG || op == OV_OP_M_DAG;
      if (!direct)
        k_ms_prep<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, dag);
      launch_ms<double>(E, T_APPLY, E.mp64, E.L64);
      launch_combine<double>(E, T_APPLY,
                             op == -1              ? EPI_SIGN
                             : op == OV_OP_DOV     ? EPI_DOV
                             : op == OV_OP_M       ? EPI_M
                             : op == OV_OP_DOV_DAG ? EPI_DOVDAG
                                                   : EPI_MDAG,
                             direct ? 3 : 0);
      break;
    }
    case OV_OP_M0INV:
    case OV_OP_M0INV_DAG:
    {
      SymIo io;
      io.in = io.out = direct;
      launch_sym<double>(E, T_APPLY, op == OV_OP_M0INV ? SYM_M0INV : SYM_M0INV_DAG, io);
    }
      break;
    case OV_OP_MDAGM:
      if (!direct)
        k_ms_prep<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
      launch_ms<double>(E, T_APPLY, E.mp64, E.L64);
      launch_combine<double>(E, T_APPLY, EPI_M, direct);  // u64, src64b = g5 u64, part_b
      launch_ms<double>(E, T_APPLY2, E.mp64, E.L64);
      launch_combine<double>(E, T_APPLY2, EPI_MDAG, direct ? 2 : 0);
      break;
    default:
      return OV_ERR_INVALID_ARG;
  }
  return check_launch(E.lead);
}

// ------------------------------------------------------------------ solve
// Every pointer a kernel dereferences through a table must be set: which
// kernels run on which table is fixed by solve_engine / true_residual.
ov_status check_roles(Engine& E, bool fp64_inner) {
  auto need = [&](int t, int s, const void* p, const char* what) -> bool {
    if (p) return true;
    char buf[160];
    std::snprintf(buf, sizeof buf, "internal: table %d system %d lacks %s", t, s, what);
    E.lead->err = buf;
    return false;
  };
  for (int s = 0; s < E.nsys; ++s) {
    const SysDev* T[T_NT];
    for (int t = 0; t < T_NT; ++t) T[t] = &E.htab[(size_t)t * E.nsys + s];
    bool ok = true;
    for (int t : {T_CG, T_CG_RU}) {
      ok &= need(t, s, T[t]->part_a, "part_a") && need(t, s, T[t]->part_b, "part_b") &&
            need(t, s, T[t]->part_c, "part_c") && need(t, s, T[t]->cg_s, "cg_s") &&
            need(t, s, T[t]->h_ctl, "h_ctl") && need(t, s, T[t]->active, "active");
    }
    if (E.pl.fft) {
      // momentum-space D + k_yuk on the F tables
      for (int t : {T_F_M, T_F_MD, T_F_TM, T_F_TMD})
        ok &= need(t, s, T[t]->e_in, "e_in") && need(t, s, T[t]->e_out, "e_out") &&
              need(t, s, T[t]->fft_tmp, "fft_tmp") && need(t, s, T[t]->active, "active") &&
              need(t, s, T[t]->phi, "phi") && need(t, s, T[t]->part_c, "part_c") &&
              need(t, s, T[t]->cg_s, "cg_s");
      ok &= need(T_F_TMD, s, T[T_F_TMD]->cg_b, "cg_b") &&
            need(T_F_TMD, s, T[T_F_TMD]->cg_r64, "cg_r64");
      if (fp64_inner) ok &= need(T_F_TMD, s, T[T_F_TMD]->cg_r, "cg_r");
      ok &= need(T_CG, s, T[T_CG]->e_in, "e_in");
    }
    // multi-shift + combine tables
    if (!E.pl.fft) {
    for (int t : {T_IN_M, T_IN_MDAG, T_TR_M, T_TR_MDAG}) {
      ok &= need(t, s, T[t]->part_a, "part_a") && need(t, s, T[t]->part_b, "part_b") &&
            need(t, s, T[t]->part_c, "part_c") && need(t, s, T[t]->cg_s, "cg_s") &&
            need(t, s, T[t]->h_ctl, "h_ctl") && need(t, s, T[t]->active, "active");
    }
    for (int t : {T_IN_M, T_IN_MDAG, T_TR_M, T_TR_MDAG})
      ok &= need(t, s, T[t]->basis, "basis") && need(t, s, T[t]->r, "r") &&
            need(t, s, T[t]->src, "src") && need(t, s, T[t]->e_in, "e_in") &&
            need(t, s, T[t]->phi, "phi") && need(t, s, T[t]->h_rho, "h_rho") &&
            need(t, s, T[t]->coef_d, "coef_d") && need(t, s, T[t]->stat, "stat");
    ok &= need(T_IN_M, s, T[T_IN_M]->e_out, "e_out") && need(T_IN_M, s, T[T_IN_M]->e_out2, "e_out2");
    ok &= need(T_TR_M, s, T[T_TR_M]->e_out, "e_out") && need(T_TR_M, s, T[T_TR_M]->e_out2, "e_out2");
    // EPI_MDAG_CG
    ok &= need(T_IN_MDAG, s, T[T_IN_MDAG]->cg_x, "cg_x") && need(T_IN_MDAG, s, T[T_IN_MDAG]->cg_p, "cg_p") &&
          need(T_IN_MDAG, s, T[T_IN_MDAG]->cg_r, "cg_r");
    // EPI_MDAG_RES (cg_r only for an FP64 inner solver)
    ok &= need(T_TR_MDAG, s, T[T_TR_MDAG]->cg_b, "cg_b") && need(T_TR_MDAG, s, T[T_TR_MDAG]->cg_r64, "cg_r64");
    if (fp64_inner) ok &= need(T_TR_MDAG, s, T[T_TR_MDAG]->cg_r, "cg_r");
    }
    // k_cg_p / k_cg_misc / k_ms_prep on T_CG and T_CG_RU, k_r64_to_r32 on T_CG_RU
    for (int t : {T_CG, T_CG_RU})
      ok &= need(t, s, T[t]->cg_x, "cg_x") && need(t, s, T[t]->cg_p, "cg_p") &&
            need(t, s, T[t]->cg_r, "cg_r") && need(t, s, T[t]->cg_b, "cg_b") &&
            need(t, s, T[t]->cg_x64, "cg_x64") && need(t, s, T[t]->src, "src");
    ok &= need(T_CG_RU, s, T[T_CG_RU]->cg_r64, "cg_r64");
    if (E.pl.pc) {
      // z = P r (momentum-space passes), EPI_MDAG into w, k_cg_misc ops 5 and 6
      for (int t : {T_PC_Z, T_PC_ZRU})
        ok &= need(t, s, T[t]->e_in, "e_in") && need(t, s, T[t]->e_out, "e_out") &&
              need(t, s, T[t]->fft_tmp, "fft_tmp") && need(t, s, T[t]->active, "active");
      if (!E.pl.fft) ok &= need(T_IN_MDAG, s, T[T_IN_MDAG]->e_out, "e_out");
      ok &= need(T_CG, s, T[T_CG]->e_in, "e_in");
      for (int t : {T_CG, T_CG_RU}) ok &= need(t, s, T[t]->cg_z, "cg_z");
    }
    if (E.pl.gw) {
      // k_cg_p_gw / multi-shift / k_gw_combine over both entries
      for (int e = 0; e < 2; ++e) {
        const SysDev* G = &E.hgwtab[(size_t)e * E.nsys + s];
        const int t = 100 + e;
        ok &= need(t, s, G->basis, "basis") && need(t, s, G->r, "r") && need(t, s, G->src, "src") &&
              need(t, s, G->part_a, "part_a") && need(t, s, G->part_b, "part_b") &&
              need(t, s, G->part_c, "part_c") && need(t, s, G->h_rho, "h_rho") &&
              need(t, s, G->h_alpha, "h_alpha") && need(t, s, G->h_zeta, "h_zeta") &&
              need(t, s, G->h_active, "h_active") && need(t, s, G->h_ctl, "h_ctl") &&
              need(t, s, G->coef_term, "coef_term") && need(t, s, G->coef_c, "coef_c") &&
              need(t, s, G->coef_d, "coef_d") && need(t, s, G->stat, "stat") &&
              need(t, s, G->dstat, "dstat") && need(t, s, G->active, "active") &&
              need(t, s, G->phi, "phi");
      }
      const SysDev* A = &E.hgwtab[s];
      ok &= need(100, s, A->e_in, "e_in") && need(100, s, A->e_out, "e_out") &&
            need(100, s, A->cg_s, "cg_s") && need(T_CG, s, T[T_CG]->e_in, "e_in");
    }
    if (E.pl.gwx) {
      // the exact form's two entries, its combine and finish
      for (int e = 0; e < 2; ++e) {
        const SysDev* G = &E.htrgw[(size_t)e * E.nsys + s];
        const int t = 110 + e;
        ok &= need(t, s, G->basis, "basis") && need(t, s, G->r, "r") && need(t, s, G->src, "src") &&
              need(t, s, G->part_a, "part_a") && need(t, s, G->part_b, "part_b") &&
              need(t, s, G->part_c, "part_c") && need(t, s, G->h_rho, "h_rho") &&
              need(t, s, G->h_alpha, "h_alpha") && need(t, s, G->h_zeta, "h_zeta") &&
              need(t, s, G->h_active, "h_active") && need(t, s, G->h_ctl, "h_ctl") &&
              need(t, s, G->coef_term, "coef_term") && need(t, s, G->coef_c, "coef_c") &&
              need(t, s, G->coef_d, "coef_d") && need(t, s, G->stat, "stat") &&
              need(t, s, G->dstat, "dstat") && need(t, s, G->active, "active") &&
              need(t, s, G->phi, "phi");
      }
      const SysDev* TA = &E.htrgw[s];
      ok &= need(110, s, TA->e_in, "e_in") && need(110, s, TA->e_out, "e_out") &&
            need(110, s, TA->e_out2, "e_out2") && need(110, s, TA->coef_d2, "coef_d2") &&
            need(110, s, TA->coef_sq, "coef_sq") && need(110, s, TA->cg_b, "cg_b") &&
            need(110, s, TA->cg_r64, "cg_r64");
    }
    if (!ok) return OV_ERR_DEVICE;
  }
  return OV_OK;
}

// Preconditioner masses (pc_mass = 1): the RMS over the lattice of the site-local
// coefficient c = m + g phi, in the direction of m (real when m = 0).
ov_status pc_masses(Engine& E, const std::vector<const void*>& phi, std::vector<double2>& pcm) {
  ov_ctx* c = E.lead;
  const int ns = E.nsys;
  pcm.assign(ns, double2{0.0, 0.0});
  E.htab.assign((size_t)E.ntab * ns, SysDev{});
  for (int s = 0; s < ns; ++s) {
    SysDev d = base_dev(E.sb[s]);
    d.phi = (const double2*)phi[s];
    E.htab[(size_t)T_APPLY * ns + s] = d;
  }
  TRY(upload_tables(E));
  k_c_norm<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  TRY(check_launch(c));
  k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_APPLY), ns, 4);
  TRY(read_scalars(E));
  for (int s = 0; s < ns; ++s) {
    const SysBuf& b = E.sb[s];
    const double acc = c->pinned[(size_t)s * CG_NSLOT + CG_BB];
    const ov_params& p = b.ctx->p;
    const double rms = std::sqrt(acc / b.V);
    const double am = std::hypot(p.m_re, p.m_im);
    pcm[s] = am > 0.0 ? double2{rms * p.m_re / am, rms * p.m_im / am} : double2{rms, 0.0};
  }
  return OV_OK;
}

template <class R>
ov_status build_solve_tables(Engine& E, const std::vector<const void*>& bvec,
                             const std::vector<const void*>& phi) {
  std::vector<double2> pcm;
  const bool rms_pc = E.pl.pc && E.lead->p.pc_mass == 1;
  if (rms_pc) TRY(pc_masses(E, phi, pcm));
  E.htab.assign((size_t)E.ntab * E.nsys, SysDev{});
  E.hgwtab.assign(E.pl.gw ? 2 * (size_t)E.nsys : 0, SysDev{});
  E.htrgw.assign(E.pl.gwx ? 2 * (size_t)E.nsys : 0, SysDev{});
  for (int s = 0; s < E.nsys; ++s) {
    SysBuf& b = E.sb[s];
    SysDev d = base_dev(b);
    d.phi = (const double2*)phi[s];
    d.cg_b = (const double2*)bvec[s];
    d.shift = E.shift;
    if (rms_pc) {
      d.pc_re = pcm[s].x;
      d.pc_im = pcm[s].y;
    }
    // inner M p
    SysDev im = d;
    im.active = b.act_cg;
    im.basis = b.basisR;
    im.r = b.rR;
    im.src = b.pR;
    im.e_in = b.pR;
    im.e_out = b.uR;
    im.e_out2 = b.srcR2;
    // inner M^dag u with the CG update
    SysDev imd = d;
    imd.active = b.act_cg;
    imd.basis = b.basisR;
    imd.r = b.rR;
    imd.src = b.srcR2;
    imd.e_in = b.uR;
    imd.cg_x = b.xR;
    imd.cg_p = b.pR;
    imd.cg_r = b.rcgR;
    imd.e_out = b.vR;  // preconditioned: w = M^dag u -> v (EPI_MDAG), then the CG update
    // FP64 true residual: M x64, then r64 = b - M^dag (M x64)
    SysDev tm = d;
    tm.active = b.act_ru;
    tm.basis = b.basis64;
    tm.r = b.r64ms;
    tm.src = b.x64;
    tm.e_in = b.x64;
    tm.e_out = b.u64;
    tm.e_out2 = b.src64b;
    SysDev tmd = d;
    tmd.active = b.act_ru;
    tmd.basis = b.basis64;
    tmd.r = b.r64ms;
    tmd.src = b.src64b;
    tmd.e_in = b.u64;
    tmd.cg_r64 = b.r64;
    // FP64 inner solver: copy of r64 in cg_r; FP32: k_r64_to_r32
    tmd.cg_r = (sizeof(R) == sizeof(double)) ? b.rcgR : nullptr;
    // CG vector ops
    SysDev cg = d;
    cg.active = b.act_cg;
    cg.cg_x = b.xR;
    cg.cg_p = b.pR;
    cg.cg_r = b.rcgR;
    cg.cg_x64 = b.x64;
    cg.src = b.x64;
    cg.e_in = b.vR;   // w = MdagM p of the update (preconditioned and GW forms)
    cg.cg_z = E.pl.pc ? b.vR : nullptr;  // z = P r, in v once w has been used
    SysDev cgr = cg;
    cgr.active = b.act_ru;
    cgr.cg_r64 = b.r64;
    if (E.pl.pc) {  // z = P r: rcgR -> vR through the transform scratch
      SysDev pz = d;
      pz.active = b.act_cg;
      pz.fft_tmp = b.fftR;
      pz.e_in = b.rcgR;
      pz.e_out = b.vR;
      SysDev pzr = pz;
      pzr.active = b.act_ru;
      E.htab[(size_t)T_PC_Z * E.nsys + s] = pz;
      E.htab[(size_t)T_PC_ZRU * E.nsys + s] = pzr;
    }
    if (E.pl.fft) {
      SysDev fm = d;  // inner: u = D p + Y p
      fm.active = b.act_cg;
      fm.fft_tmp = b.fftR;
      fm.e_in = b.pR;
      fm.e_out = b.uR;
      SysDev fmd = fm;  // inner: w = D^dag u + Y^dag u (+ shift p) -> v
      fmd.e_in = b.uR;
      fmd.e_out = b.vR;
      fmd.cg_p = b.pR;
      SysDev ftm = d;  // FP64 truth: u64 = M x64
      ftm.active = b.act_ru;
      ftm.fft_tmp = b.src64b;
      ftm.e_in = b.x64;
      ftm.e_out = b.u64;
      SysDev ftmd = ftm;  // r64 = b - M^dag u64 (- shift x64)
      ftmd.e_in = b.u64;
      ftmd.cg_x64 = b.x64;
      ftmd.e_out = b.r64ms;
      ftmd.cg_r64 = b.r64;
      ftmd.cg_r = (sizeof(R) == sizeof(double)) ? b.rcgR : nullptr;
      E.htab[(size_t)T_F_M * E.nsys + s] = fm;
      E.htab[(size_t)T_F_MD * E.nsys + s] = fmd;
      E.htab[(size_t)T_F_TM * E.nsys + s] = ftm;
      E.htab[(size_t)T_F_TMD * E.nsys + s] = ftmd;
    }
    if (E.pl.gw) {
      // entry A: eps(v) on the system's inner buffers, MdagM v -> vR; entry B:
      // eps(g5 (1 + Y) v) on the twin buffers, workgroups after all of A's
      SysDev ga = im;
      ga.e_out = b.vR;
      SysDev gb = d;
      gb.active = b.act_cg;
      gb.blk0 = b.blk0 + E.nb_total;
      gb.basis = b.ms_b_basis;
      gb.r = b.ms_b_r;
      gb.src = b.ms_b_src;
      gb.part_a = b.ms_b_part_a;
      gb.part_b = b.ms_b_part_b;
      gb.part_c = b.ms_b_part_c;
      gb.h_rho = b.ms_b_h_rho;
      gb.h_alpha = b.ms_b_h_alpha;
      gb.h_zeta = b.ms_b_h_zeta;
      gb.h_active = b.ms_b_h_active;
      gb.h_ctl = b.ms_b_h_ctl;
      gb.stat = b.ms_b_stat;
      gb.dstat = b.ms_b_dstat;
      gb.coef_term = b.ms_b_coef_term;
      gb.coef_c = b.ms_b_coef_c;
      gb.coef_d = b.ms_b_coef_d;
      gb.cg_s = nullptr;
      E.hgwtab[s] = ga;
      E.hgwtab[E.nsys + s] = gb;
    }
    if (E.pl.gwx) {
      // exact MdagM: entry A on x64 (also the finish: r64 = b - P - H w), entry B on
      // g5 (1 + Y) x64 with the FP64 twins.  The rational layers' CG applies it to p
      // instead (W = MdagM p -> vR, Re <p, W>).
      SysDev ta = tm;
      ta.coef_d2 = b.coef_d2;
      ta.coef_sq = b.coef_sq;
      ta.cg_b = (const double2*)bvec[s];
      ta.cg_r64 = b.r64;
      ta.cg_r = tmd.cg_r;
      if (E.pl.nshift > 0) {
        ta.active = b.act_cg;
        ta.src = b.pR;
        ta.e_in = b.pR;
        ta.cg_r64 = b.vR;
        ta.cg_r = nullptr;
      }
      SysDev tbb = d;
      tbb.active = b.act_ru;
      tbb.blk0 = b.blk0 + E.nb_total;
      tbb.basis = b.tb_basis;
      tbb.r = b.tb_r;
      tbb.src = b.tb_src;
      tbb.part_a = b.tb_part_a;
      tbb.part_b = b.tb_part_b;
      tbb.part_c = b.tb_part_c;
      tbb.h_rho = b.tb_h_rho;
      tbb.h_alpha = b.tb_h_alpha;
      tbb.h_zeta = b.tb_h_zeta;
      tbb.h_active = b.tb_h_active;
      tbb.h_ctl = b.tb_h_ctl;
      tbb.stat = b.tb_stat;
      tbb.dstat = b.tb_dstat;
      tbb.coef_term = b.tb_coef_term;
      tbb.coef_c = b.tb_coef_c;
      tbb.coef_d = b.tb_coef_d;
      tbb.cg_s = nullptr;
      if (E.pl.nshift > 0) tbb.active = b.act_cg;
      E.htrgw[s] = ta;
      E.htrgw[E.nsys + s] = tbb;
    }
    E.htab[(size_t)T_IN_M * E.nsys + s] = im;
    E.htab[(size_t)T_IN_MDAG * E.nsys + s] = imd;
    E.htab[(size_t)T_TR_M * E.nsys + s] = tm;
    E.htab[(size_t)T_TR_MDAG * E.nsys + s] = tmd;
    E.htab[(size_t)T_CG * E.nsys + s] = cg;
    E.htab[(size_t)T_CG_RU * E.nsys + s] = cgr;
    SysDev ap = d;  // pack/unpack geometry
    E.htab[(size_t)T_APPLY * E.nsys + s] = ap;
  }
  TRY(check_roles(E, sizeof(R) == sizeof(double)));
  return upload_tables(E);
}

ov_status set_flags(Engine& E, const std::vector<int>& cg, const std::vector<int>& ru) {
  std::vector<int> f(2 * E.nsys);
  for (int s = 0; s < E.nsys; ++s) {
    f[s] = cg[s];
    f[E.nsys + s] = ru[s];
  }
  if (f == E.last_flags) return OV_OK;
  int* h = E.lead->pinned_flags;
  // the pinned staging may still feed an earlier copy
  HIPCHK(E.lead, hipStreamSynchronize(E.st));
  std::memcpy(h, f.data(), sizeof(int) * f.size());
  HIPCHK(E.lead, hipMemcpyAsync(E.act_all, h, sizeof(int) * f.size(), hipMemcpyHostToDevice, E.st));
  E.last_flags = f;
  return OV_OK;
}

// Clear every entry's control words before multi-shift solves that are checked on their own.
void clear_ctl(const Engine& E) {
  k_zero32<<<1, 256, 0, E.st>>>((unsigned int*)E.ctl_all, (size_t)12 * E.nsys);
}

// OV_OK, or the status a set of sticky bits stands for (with the reason in err).
ov_status sticky_status(ov_ctx* c, int bits, const char* what) {
  if (bits & (1 << 1)) {
    c->err = std::string(what) + ": multi-shift breakdown (non-finite or non-positive scalar)";
    return OV_ERR_BREAKDOWN;
  }
  if (bits & (1 << 2)) {
    c->err = std::string(what) + ": multi-shift did not converge within its basis (max_inner)";
    return OV_ERR_NOT_CONVERGED;
  }
  return OV_OK;
}

// Largest iteration count of the FP64 multi-shift solves of the last reliable
// update (stat[3] of the systems' own entries, cleared at the update's start).
int last_truth_iters(const Engine& E) {
  const long long* st = (const long long*)(E.lead->pinned + (size_t)CG_NSLOT * E.nsys);
  long long m = 0;
  for (int s = 0; s < E.nsys; ++s) {
    m = std::max(m, st[(size_t)s * 4 + 3]);
    if (E.pl.gwx) m = std::max(m, st[(size_t)(2 * E.nsys + s) * 4 + 3]);  // its entry B
  }
  return (int)m;
}

// Largest multi-shift iteration count of the current outer iteration (stat[3]).
int last_ms_iters(const Engine& E) {
  const long long* st = (const long long*)(E.lead->pinned + (size_t)CG_NSLOT * E.nsys);
  long long m = 0;
  for (int s = 0; s < 2 * E.nsys; ++s) m = std::max(m, st[(size_t)s * 4 + 3]);  // A and B
  return (int)m;
}

long long n_est_key(size_t rsize, double tol) {
  return (long long)rsize * 1000 + (long long)std::lround(-std::log10(tol) * 10.0);
}

// The cached graph of `key`, captured now if there is none, on the engine's stream.
template <class F>
ov_status graph_launch(Engine& E, const std::string& key, F&& enqueue) {
  ov_ctx* c = E.lead;
  char buf[160];
  std::snprintf(buf, sizeof buf, "|%p|%p|%p|%d|%d|%d|%d|%d|%d|", (void*)E.tables, (void*)E.bmap,
                (void*)E.gwtab, E.nb_total, E.nsys, E.block, E.nb_xy, E.nb_z, E.nb_t);
  const std::string k = key + buf + E.geo_key;
  auto it = c->graphs.find(k);
  if (it == c->graphs.end()) {
    if (c->graphs.size() >= 64) clear_graphs(c);
    HIPCHK(c, hipStreamBeginCapture(E.st, hipStreamCaptureModeThreadLocal));
    c->capturing = true;
    enqueue();
    c->capturing = false;
    hipGraph_t g = nullptr;
    const hipError_t ec = hipStreamEndCapture(E.st, &g);
    TRY(check_launch(c));
    if (ec != hipSuccess) {
      c->err = std::string("hipStreamEndCapture: ") + hipGetErrorString(ec);
      return OV_ERR_DEVICE;
    }
    hipGraphExec_t ge = nullptr;
    const hipError_t ei = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ei != hipSuccess) {
      c->err = std::string("hipGraphInstantiate: ") + hipGetErrorString(ei);
      return OV_ERR_DEVICE;
    }
    it = c->graphs.emplace(k, ge).first;
  }
  HIPCHK(c, hipGraphLaunch(it->second, E.st));
  return OV_OK;
}

// Run `enqueue` (kernel launches only) through a cached hipGraph keyed by
// everything its launches bake in; direct launches while kernel sampling is on.  Capture and
// launch are under the gate: an event of another context on a stream that is being captured
// would draw that context into the capture.
template <class F>
ov_status run_graph(Engine& E, const std::string& key, F&& enqueue) {
  ov_ctx* c = E.lead;
  if (!c->use_graphs || c->sample_max > 0) {
    enqueue();
    return check_launch(c);
  }
  auto run = [&]() { return graph_launch(E, key, enqueue); };
  if (E.resident_any()) return res_ordered(c, run);
  if (c->device < 0 || c->device >= kMaxDevices) return run();
  return g_res_gate[c->device].alone(run);
}

}  // namespace

// The float inner solver needs r (FP32) = r64 after a true residual; a small
// conversion kernel keeps the FP64 combine generic.
namespace ov {
__global__ void __launch_bounds__(512) k_r64_to_r32(const SysDev* __restrict__ sys,
                                                    const int* __restrict__ bmap, int nb_total) {
  const int L = xcd_logical_block(nb_total);
  const int s = bmap[L];
  const SysDev& S = sys[s];
  if (S.active && *S.active == 0) return;
  const int lb = L - S.blk0;
  const int V = S.g.V;
  const int i0 = lb * S.spb;
  const int i1 = min(V, i0 + S.spb);
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    double2 v[4];
    load_sp<double>((const double2*)S.cg_r64, V, i, v);
    float2 w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = float2{(float)v[k].x, (float)v[k].y};
    store_sp<float>((float2*)S.cg_r, V, i, w);
  }
}
}  // namespace ov

namespace {

// Reliable update for the systems with act_ru set: x64 += xR, xR = 0, then the
// FP64 true residual r64 = b - MdagM x64 (inner-precision copy into rcgR) with
// multi-shift tolerance tol, and its norm through k_cg_scalar(scalar_op).
// The tolerance is rounded down to a power of ten so that few graphs exist.
// Multi-shift tolerance of a true residual at tolerance tol: the Ginsparg-Wilson form
// takes eps^2 x from the Krylov space of x, about ten times less accurate than the
// shifted solutions themselves, so the final check (tol = truth_tol) runs ten times
// tighter; intermediate updates tolerate that much by construction (truth_relax).
double truth_ms_tol(const Engine& E, double tol) {
  const bool final_check = tol <= E.lead->p.truth_tol * 1.0000001;
  return (E.pl.gwx && final_check) ? 0.1 * tol : tol;
}

template <class R>
ov_status reliable_update_L(Engine& E, double tol, int scalar_op, int L) {
  const ov_ctx* c = E.lead;
  const MsParams mp = make_mp(c, truth_ms_tol(E, tol), E.pl.cap64);
  const bool pc = E.pl.pc;
  char key[96];
  std::snprintf(key, sizeof key, "ru|%zu|%.3e|%d|%d|%d|%d", sizeof(R), tol, L, scalar_op, (int)pc,
                (int)E.pl.fft);
  return run_graph(E, key, [&]() {
    if (!E.pl.fft)  // per-update maximum of the FP64 multi-shift iteration counts
      k_stat3_clear<<<1, 64, 0, E.st>>>(tab(E, T_TR_M), E.nsys);
    // x64 += x, x = 0
    k_cg_misc<R><<<E.nb_total, site_block(E), 0, E.st>>>(tab(E, T_CG_RU), E.bmap, E.nb_total, 0);
    // the residual table: EPI_MDAG_RES (multi-shift) or k_yuk mode 2 (momentum
    // space) writes r64 (FP64) and, for an FP64 inner solver, its copy in cg_r; an
    // FP32 inner solver gets its copy from k_r64_to_r32.
    const int tres = E.pl.fft ? T_F_TMD : T_TR_MDAG;
    if (E.pl.fft) {
      launch_sym<double>(E, T_F_TM, SYM_D);
      k_yuk<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_F_TM), E.bmap, E.nb_total, 0);
      launch_sym<double>(E, T_F_TMD, SYM_D_DAG);
      k_yuk<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_F_TMD), E.bmap, E.nb_total, 2);
    } else if (E.pl.gwx) {  // one two-source multi-shift (see k_truth_combine)
      const int nb = E.nb_total, ns = E.nsys;
      k_stat3_clear<<<1, 64, 0, E.st>>>(E.trgwtab, 2 * ns);
      k_gw_prep<double><<<nb, site_block(E), 0, E.st>>>(E.trgwtab, E.trgwtab + ns, E.bmap, nb);
      launch_ms_tab<double>(E, E.trgwtab, E.gwbmap, 2 * nb, 2 * ns, mp, L);
      k_truth_combine<<<nb, site_block(E), 0, E.st>>>(E.trgwtab, E.trgwtab + ns, E.bmap, nb);
      k_truth_finish<R><<<nb, site_block(E), 0, E.st>>>(E.trgwtab, E.bmap, nb, 4.0 - c->p.M0, 0);
    } else {
      k_ms_prep<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_TR_M), E.bmap, E.nb_total, 0);
      launch_ms<double>(E, T_TR_M, mp, L);
      launch_combine<double>(E, T_TR_M, EPI_M);
      launch_ms<double>(E, T_TR_MDAG, mp, L);
      launch_combine<double>(E, T_TR_MDAG, EPI_MDAG_RES);
    }
    if (pc) {
      // |r64|^2, then the recursion restarts from r = r64 with z = P r and
      // rho = <r, z> in the CG state
      k_cg_scalar<<<E.nsys, 256, 0, E.st>>>(tab(E, tres), E.nsys, 5);
      if (sizeof(R) != sizeof(double))
        k_r64_to_r32<<<E.nb_total, site_block(E), 0, E.st>>>(tab(E, T_CG_RU), E.bmap, E.nb_total);
      if (scalar_op == 3 || scalar_op == 7) {
        launch_sym<R>(E, T_PC_ZRU, SYM_PCG);
        k_cg_misc<R><<<E.nb_total, site_block(E), 0, E.st>>>(tab(E, T_CG_RU), E.bmap, E.nb_total, 6);
        k_cg_scalar<<<E.nsys, 256, 0, E.st>>>(tab(E, T_CG_RU), E.nsys, scalar_op == 3 ? 11 : 12);
      }
    } else {
      k_cg_scalar<<<E.nsys, 256, 0, E.st>>>(tab(E, tres), E.nsys, scalar_op);
      if (sizeof(R) != sizeof(double))
        k_r64_to_r32<<<E.nb_total, site_block(E), 0, E.st>>>(tab(E, T_CG_RU), E.bmap, E.nb_total);
    }
  });
}

// Reliable update (above) followed by the scalar read-back.  The FP64 multi-shift
// solves launch as many iterations as the last update at this tolerance needed plus
// a margin; when an update may have been cut short by that (its largest iteration
// count reached the launched count) it is repeated with the full Chebyshev bound.
// The repeat is exact: the fold-in adds the (now zero) inner solution again and the
// residual, its norm and the CG state update are recomputed from x64 alone.
template <class R>
ov_status reliable_update(Engine& E, double tol, int scalar_op) {
  ov_ctx* c = E.lead;
  Range range("ov reliable update (FP64 true residual)");
  tol = std::pow(10.0, std::floor(std::log10(tol) + 1e-9));
  int Lfull = 0;
  for (int s = 0; s < E.nsys; ++s)
    Lfull = std::max(Lfull, capacity(E.ctxs[s], truth_ms_tol(E, tol)));
  Lfull = std::min(E.pl.cap64, Lfull);
  if (E.pl.fft) {
    TRY(reliable_update_L<R>(E, tol, scalar_op, Lfull));
    return read_scalars(E);
  }
  const long long key = n_est_key(1000 + sizeof(R), tol);  // FP64 truth solves of this solver
  // the last count at this tolerance plus max(4, n/8): a true residual cut short is
  // repeated in full, so this margin stays wider than the inner solves' one (max(3, n/16)
  // saved 0.13 ms per 16^4 solve but repeated four true residuals per uneven-batch solve,
  // +4%: a batch's count is the maximum over its systems, which moves between calls);
  // a resident launch stops by itself
  int L = Lfull;
  {
    auto it = c->n_est.find(key);
    if (it != c->n_est.end() && !E.resident<double>(E.pl.gwx ? 2 : 1))
      L = std::min(Lfull, it->second + std::max(4, it->second / 8));
  }
  clear_ctl(E);
  TRY(reliable_update_L<R>(E, tol, scalar_op, L));
  TRY(read_scalars(E));
  int nobs = last_truth_iters(E);
  if (L < Lfull && nobs >= L - 1) {
    if (ov_log())
      std::fprintf(stderr, "[ov] truth multi-shift at tol %.0e cut at %d of %d: repeated\n", tol, L,
                   Lfull);
    clear_ctl(E);
    TRY(reliable_update_L<R>(E, tol, scalar_op, Lfull));
    TRY(read_scalars(E));
    nobs = last_truth_iters(E);
  }
  c->n_est[key] = nobs;
  // The final check certifies the solution: its multi-shift solves must have converged
  // within their basis (a basis capped by max_inner, or a breakdown, leaves an
  // uncertified residual).
  if (tol <= c->p.truth_tol * 1.0000001) {
    int bits = 0;
    for (int s = 0; s < E.nsys; ++s) bits |= sticky_bits(E, s);
    TRY(sticky_status(c, bits, "true residual"));
  }
  return OV_OK;
}

struct SolveOut {
  std::vector<int> outer, ru;
  std::vector<double> res;
  std::vector<int> conv;
  std::vector<int> stag;      // restarts forced by a stagnating recursion
  std::vector<int> fallback;  // mixed solve handed to the FP64 solver (stagnating cycles)
};

// Reliable-update CG on MdagM x = b.  Inner iterations run in precision R with
// multi-shift tolerance tol_in; every time the recursive residual has dropped
// by `delta` relative to the last true residual (or meets the target) the
// inner solution is folded into the FP64 x64 and the FP64 true residual
// replaces the recursive one (Sleijpen & van der Vorst; Clark et al. for
// mixed precision).  Convergence is declared only on the FP64 true residual
// computed with multi-shift tolerance truth_tol.
template <class R>
ov_status solve_engine(Engine& E, const std::vector<const void*>& bvec,
                       const std::vector<const void*>& phi, double tol_in, double delta,
                       SolveOut& out) {
  ov_ctx* c = E.lead;
  const ov_params& P = c->p;
  const int ns = E.nsys;
  const int max_outer = E.max_outer > 0 ? E.max_outer : P.max_outer;
  Range range(sizeof(R) == sizeof(double) ? "ov solve engine FP64" : "ov solve engine mixed");
  TRY((build_solve_tables<R>(E, bvec, phi)));
  if (E.guess) TRY(pack64(E));
  pcg_table(E);
  TRY(reset_stats(E));
  std::vector<int> fcg(ns, 1), fru(ns, 1);
  TRY(set_flags(E, fcg, fru));
  // x64 <- guess was packed by the caller; xR = 0; rcgR = b, |b|^2
  k_cg_misc<R><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_CG), E.bmap, E.nb_total, 2);
  k_cg_misc<R><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_CG), E.bmap, E.nb_total, 1);
  k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 4);  // BB
  const bool pc = E.pl.pc;
  if (pc) {  // z = P b, rho = <b, z>, beta = 0
    launch_sym<R>(E, T_PC_Z, SYM_PCG);
    k_cg_misc<R><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_CG), E.bmap, E.nb_total, 6);
    k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 10);
  } else {
    k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 0);  // rho = |b|^2, beta = 0
  }
  // |x0|^2 -> part_b via prep on x64 (src = x64 in T_CG)
  k_ms_prep<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_CG), E.bmap, E.nb_total, 0);
  k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 13);
  TRY(read_scalars(E));
  std::vector<double> x0n(ns);
  for (int s = 0; s < ns; ++s) x0n[s] = c->pinned[(size_t)s * CG_NSLOT + CG_RTRUE];
  // rmax: residual norm at the last restart (the recursion's |r| is slot CG_R2,
  // with or without the preconditioner).
  std::vector<double> bn(ns), rmax(ns);
  std::vector<int> last_ru(ns, 0);  // outer iteration of the last reliable update
  // Stagnation.  Within a cycle: a recursion that has not dropped by delta in kStall
  // iterations, or, under a relaxed (inexact) inner sign in a preconditioned solve,
  // has made no new minimum of
  // |r| for kStagnate iterations or gained less than kCrawl of the decades its best
  // kStagnate-iteration window of this solve gained -> reliable update and restart.  At an update: a true
  // residual more than 10x the recursive one (the inexact sign's error has decoupled
  // the recursion) tightens that system's relaxation tenfold.  Across cycles: a true
  // residual that fell by less than half since the last update, kCycleStag times in a
  // row -> a mixed solve hands the system to the FP64 solver (fixed inner tolerance).
  constexpr int kStall = 250, kStagnate = 8, kCycleStag = 2;
  constexpr double kCrawl = 0.25;
  const bool relaxed = !E.pl.fft && P.inner_relax > 0.0 && !E.no_relax;
  // the within-cycle checks need an even convergence rate: preconditioned solves only
  // (unpreconditioned CG on MdagM has plateaus that a restart would throw away)
  const bool watch = relaxed && E.pl.pc;
  std::vector<double> rbest(ns, 1e300), rt_prev(ns, 0.0), rec_last(ns, 1.0);
  std::vector<double> relax_scale(ns, 1.0);
  std::vector<int> it_best(ns, 0), nstag(ns, 0);
  std::vector<std::vector<double>> hist(ns);  // recursive |r| since the last update
  std::vector<double> gain_best(ns, 0.0);     // most decades gained in kStagnate iterations
  const bool can_fall_back = sizeof(R) != sizeof(double);
  out.outer.assign(ns, 0);
  out.ru.assign(ns, 0);
  out.res.assign(ns, 1.0);
  out.conv.assign(ns, 0);
  out.stag.assign(ns, 0);
  out.fallback.assign(ns, 0);
  bool any_guess = false;
  for (int s = 0; s < ns; ++s) {
    bn[s] = std::sqrt(c->pinned[(size_t)s * CG_NSLOT + CG_BB]);
    if (bn[s] == 0.0 || !std::isfinite(bn[s])) {
      if (!std::isfinite(bn[s])) {
        c->err = "non-finite right-hand side";
        return OV_ERR_BREAKDOWN;
      }
      out.conv[s] = 1;  // b = 0: x = 0
      fcg[s] = 0;
    }
    fru[s] = (x0n[s] > 0.0 && fcg[s]) ? 1 : 0;
    if (fru[s]) any_guess = true;
    rmax[s] = bn[s];
  }
  if (any_guess) {  // r = b - A x0 for warm starts; the recursion restarts from it
    TRY(set_flags(E, fcg, fru));
    TRY(reliable_update<R>(E, P.truth_tol, 7));
    for (int s = 0; s < ns; ++s)
      if (fru[s]) {
        rmax[s] = std::sqrt(c->pinned[(size_t)s * CG_NSLOT + CG_RTRUE]);
        out.ru[s]++;
      }
  }
  int iter = 0;
  while (true) {
    bool any = false;
    for (int s = 0; s < ns; ++s) any |= (fcg[s] != 0);
    if (!any) break;
    std::fill(fru.begin(), fru.end(), 0);
    TRY(set_flags(E, fcg, fru));
    // Inner multi-shift tolerance of this iteration.  With relaxation the sign
    // may be as inexact as inner_relax * ||r_cycle|| / ||r_j|| (the error it
    // adds to the residual gap stays a fixed fraction of the cycle's start,
    // van den Eshof & Sleijpen's inexact-Krylov bound); the tightest system
    // sets it, rounded down to a power of ten.
    double tol_it = tol_in;
    if (P.inner_relax > 0.0 && !E.no_relax) {
      double t = P.inner_tol_max;
      for (int s = 0; s < ns; ++s) {
        if (!fcg[s]) continue;
        const double rr = c->pinned[(size_t)s * CG_NSLOT + CG_R2];
        const double rn = std::sqrt(std::max(rr, 0.0));
        t = std::min(t, rn > 0.0 ? P.inner_relax * relax_scale[s] * rmax[s] / rn
                                 : P.inner_tol_max);
      }
      tol_it = std::max(tol_in, std::pow(10.0, std::floor(std::log10(t) + 1e-9)));
    }
    const MsParams mpR = make_mp(c, tol_it, E.pl.capR);
    int LR = 0;
    for (int s = 0; s < ns; ++s) LR = std::max(LR, capacity(E.ctxs[s], tol_it));
    LR = std::min(E.pl.capR, LR);
    // launch what the last multi-shift at this tolerance needed, plus one iteration (each
    // launch past convergence is an empty pass of ~5 us; a multi-shift cut one iteration
    // short ends a fraction above its relaxed tolerance, which the relaxation bound
    // absorbs, and widens the estimate for the next one: 16^4 15.3 -> 15.1 ms, same
    // outer iterations, against a margin of two); a resident launch stops by itself
    const long long nkey = n_est_key(sizeof(R), tol_it);
    {
      auto it = c->n_est.find(nkey);
      if (it != c->n_est.end() && !E.resident<R>(E.pl.gw ? 2 : 1)) LR = std::min(LR, it->second + 1);
    }
    char ikey[96];
    std::snprintf(ikey, sizeof ikey, "in|%zu|%.6e|%d|%d|%d|%d", sizeof(R), tol_it, LR, (int)pc,
                  (int)E.pl.fft, (int)E.pl.gw);
    // p = z + beta p (beta = 0 right after a (re)start; z = P r preconditioned, else
    // r) ; w = MdagM p ; alpha ; x += alpha p, r -= alpha w ; z = P r ; beta -- one
    // captured graph per iteration.  Preconditioned CG with P = (M0^dag M0)^-1, a
    // scalar per momentum: the iterates of CG on (M M0^-1)^dag (M M0^-1) x~ = M0^-dag b,
    // x = M0^-1 x~ (Sec. 7.3), with one transform per iteration instead of two.
    Range it_range("ov CG iteration");
    TRY(run_graph(E, ikey, [&]() {
      const int nb = E.nb_total, bl = E.block;
      if (E.pl.gw && !E.pl.fft)  // p = z + beta p and the second inner source in one pass
        k_cg_p_gw<R><<<nb, site_block(E), 0, E.st>>>(tab(E, T_CG), E.gwtab, E.gwtab + ns, E.bmap, nb, 1);
      else
        k_cg_p<R><<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 1);
      bool fused_update = false;  // EPI_MDAG_CG did the update and the beta scalar
      int update_op = 5;          // k_cg_misc: x += alpha p, r -= alpha w
      if (E.pl.fft) {  // momentum-space D: M = D + Y exactly, no inner solve
        launch_sym<R>(E, T_F_M, SYM_D);
        k_yuk<R><<<nb, bl, 0, E.st>>>(tab(E, T_F_M), E.bmap, nb, 0);
        k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_F_M), ns, 1);
        launch_sym<R>(E, T_F_MD, SYM_D_DAG);
        k_yuk<R><<<nb, bl, 0, E.st>>>(tab(E, T_F_MD), E.bmap, nb, 1);
      } else if (E.pl.gw) {  // w = MdagM p in Ginsparg-Wilson form: both signs in one multi-shift
        launch_ms_tab<R>(E, E.gwtab, E.gwbmap, 2 * nb, 2 * ns, mpR, LR);
        k_gw_combine<R><<<nb, site_block(E), 0, E.st>>>(E.gwtab, E.gwtab + ns, E.bmap, nb);
        update_op = 7;  // alpha = rho / Re<p, w> inside the update
      } else {
        launch_ms<R>(E, T_IN_M, mpR, LR);
        launch_combine<R>(E, T_IN_M, EPI_M);
        k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_IN_M), ns, 1);
        launch_ms<R>(E, T_IN_MDAG, mpR, LR);
        if (pc) {
          launch_combine<R>(E, T_IN_MDAG, EPI_MDAG);
        } else {
          launch_combine<R>(E, T_IN_MDAG, EPI_MDAG_CG);
          k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_IN_MDAG), ns, 2);
          fused_update = true;
        }
      }
      if (fused_update) return;
      k_cg_misc<R><<<nb, site_block(E), 0, E.st>>>(tab(E, T_CG), E.bmap, nb, update_op);
      if (pc) {
        launch_sym<R>(E, T_PC_Z, SYM_PCG);
        k_cg_misc<R><<<nb, site_block(E), 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 6);
        k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 9);
      } else {
        k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 2);
      }
    }));
    TRY(read_scalars(E));
    ++iter;
    {
      // learn the iteration count; a multi-shift that ran out of launches
      // (sticky flag) widens the estimate for the next iteration
      const int nobs = last_ms_iters(E);
      int& est = c->n_est[nkey];
      if (nobs >= LR - 1) {
        est = std::max(est, LR + 6);
      } else {
        est = nobs;
      }
    }
    bool need_ru = false, final_check = false, restart = false;
    double best_rec = 1e300;  // the tightest residual among the systems updated now
    if (ov_log()) {
      std::fprintf(stderr, "[ov] iter %d:", iter);
      for (int s = 0; s < ns; ++s)
        if (fcg[s])
          std::fprintf(stderr, " s%d rec=%.3e pap=%.3e", s,
                       std::sqrt(c->pinned[(size_t)s * CG_NSLOT + CG_R2]) / bn[s],
                       c->pinned[(size_t)s * CG_NSLOT + CG_PAP]);
      std::fprintf(stderr, "\n");
    }
    for (int s = 0; s < ns; ++s) {
      if (!fcg[s]) continue;
      out.outer[s]++;
      const double* cs = c->pinned + (size_t)s * CG_NSLOT;
      const double rr = cs[CG_R2];
      if (!std::isfinite(rr) || !std::isfinite(cs[CG_RR]) || !std::isfinite(cs[CG_ALPHA]) ||
          cs[CG_PAP] <= 0.0 || cs[CG_RR] < 0.0) {
        c->err = "CG breakdown (non-finite or non-positive scalar)";
        return OV_ERR_BREAKDOWN;
      }
      const double rec = std::sqrt(rr) / bn[s];
      rec_last[s] = rec;
      const bool at_target = rec <= P.outer_tol;
      const bool dropped = delta > 0.0 && std::sqrt(rr) < delta * rmax[s];
      if (std::sqrt(rr) < rbest[s]) {
        rbest[s] = std::sqrt(rr);
        it_best[s] = iter;
      }
      hist[s].push_back(std::sqrt(rr));
      const size_t nh = hist[s].size();
      bool crawling = false;
      if (watch && nh > (size_t)kStagnate && hist[s][nh - 1] > 0.0) {
        // decades the recursion gained over the last kStagnate iterations, against the
        // best such window of this solve: far slower than before is a crawl
        const double gain = std::log10(hist[s][nh - 1 - kStagnate] / hist[s][nh - 1]);
        crawling = gain < kCrawl * gain_best[s];
        gain_best[s] = std::max(gain_best[s], gain);
      }
      // a recursion that has made no progress for kStagnate iterations, or has not
      // dropped by delta in kStall, has stalled (lost conjugacy in the inner precision
      // or under the inexact inner sign): update and restart
      const bool stalled = delta > 0.0 && ((watch && iter - it_best[s] >= kStagnate) ||
                                           crawling || iter - last_ru[s] >= kStall);
      if (stalled) {
        restart = true;
        out.stag[s]++;
      }
      if (at_target || dropped || stalled || iter >= max_outer) {
        fru[s] = 1;
        need_ru = true;
        if (at_target || iter >= max_outer) final_check = true;
        best_rec = std::min(best_rec, rec);
      }
    }
    if (need_ru && ns > 1 && delta > 0.0) {
      // Batched systems drop by delta at different iterations; each update launches the
      // FP64 multi-shift passes over the whole batch however few systems take part.  A
      // system that is more than halfway there (in log scale) joins now, which keeps the
      // updates of a batch together and cuts the number of update launch sequences.
      const double half = std::sqrt(delta);
      for (int s = 0; s < ns; ++s) {
        if (!fcg[s] || fru[s]) continue;
        const double rr = c->pinned[(size_t)s * CG_NSLOT + CG_R2];
        if (std::sqrt(rr) < half * rmax[s]) {
          fru[s] = 1;
          best_rec = std::min(best_rec, std::sqrt(rr) / bn[s]);
        }
      }
    }
    if (need_ru) {
      TRY(set_flags(E, fcg, fru));
      // One multi-shift tolerance serves every updated system, so it follows the
      // smallest residual: its operator error must stay ~1% of that residual.
      const double ttol = final_check
                              ? P.truth_tol
                              : std::max(P.truth_tol, std::min(1e-6, P.truth_relax * best_rec));
      TRY(reliable_update<R>(E, ttol, restart ? 7 : 3));
      for (int s = 0; s < ns; ++s) {
        if (!fru[s]) continue;
        out.ru[s]++;
        last_ru[s] = iter;
        const double rt = std::sqrt(c->pinned[(size_t)s * CG_NSLOT + CG_RTRUE]);
        if (relaxed && rt > 10.0 * rec_last[s] * bn[s]) relax_scale[s] *= 0.1;
        // cycles whose true residual fell by less than half
        nstag[s] = (rt_prev[s] > 0.0 && rt > 0.5 * rt_prev[s]) ? nstag[s] + 1 : 0;
        rt_prev[s] = rt;
        rmax[s] = rt;
        rbest[s] = rt;
        it_best[s] = iter;
        hist[s].clear();
        out.res[s] = rt / bn[s];
        if (ov_log())
          std::fprintf(stderr,
                       "[ov] reliable update s%d at iter %d: true res %.3e (ms tol %.1e, %d "
                       "FP64 multi-shift iterations)\n",
                       s, iter, out.res[s], ttol, last_truth_iters(E));
        if (out.res[s] <= P.outer_tol) {
          // a momentum-space operator is exact at every tolerance
          if (E.pl.fft || ttol <= P.truth_tol * 1.0000001) {
            out.conv[s] = 1;
            fcg[s] = 0;
          }
        } else if (can_fall_back && (nstag[s] >= kCycleStag || E.force_fallback)) {
          out.fallback[s] = 1;  // x64 holds the best iterate; the FP64 solver finishes
          fcg[s] = 0;
        }
      }
      if (iter >= max_outer) break;
    }
  }
  return OV_OK;
}


// Statistics from the last read_scalars.
void fill_stats(ov_stats* st, int n, Engine* E, const SolveOut* so, double secs, int prec_bytes) {
  if (!st) return;
  for (int s = 0; s < n; ++s) {
    ov_stats& o = st[s];
    std::memset(&o, 0, sizeof(o));
    if (E) {
      const SysCtl k = sys_ctl(*E, s);
      o.inner_iters = k.inner;
      o.stencil_apps = 2 * k.inner;
      o.max_shift_res = k.shift_res;
      const double V = E->sb[s].V;
      o.model_bytes = 7.0 * (double)k.inner * 4.0 * V * prec_bytes;
    }
    if (so) {
      o.outer_iters = so->outer[s];
      o.reliable_updates = so->ru[s];
      o.true_rel_res = so->res[s];
      o.stagnations = so->stag.empty() ? 0 : so->stag[s];
    }
    o.seconds = secs;
  }
}

}  // namespace

namespace {
template <class R>
ov_status tune_run(ov_ctx* c, int nrhs, int iters, float* us) {
  Engine E;
  std::vector<ov_ctx*> v(nrhs, c);
  const bool fp32 = sizeof(R) == sizeof(float);
  E.no_res = true;  // the launch shape is the per-pass kernels'
  TRY(engine_init(E, v, true, fp32, solve_tol64(c), fp32 ? c->p.mixed_inner_tol : c->p.inner_tol));
  E.htab.assign((size_t)E.ntab * nrhs, SysDev{});
  for (int s = 0; s < nrhs; ++s) {
    SysBuf& b = E.sb[s];
    SysDev d = base_dev(b);
    d.basis = fp32 ? b.basisR : (void*)b.basis64;
    d.r = fp32 ? b.rR : (void*)b.r64ms;
    d.src = fp32 ? b.pR : (void*)b.x64;
    E.htab[(size_t)T_APPLY * nrhs + s] = d;
  }
  TRY(upload_tables(E));
  TRY(reset_stats(E));
  const int cap = fp32 ? E.pl.capR : E.pl.cap64;
  const int L = std::min(iters, cap);
  MsParams mp = make_mp(c, 1e-300, cap);  // never converges: every iteration works
  k_fill<R><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  k_ms_prep<R><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
  launch_ms<R>(E, T_APPLY, mp, std::min(4, L));  // warm-up
  k_ms_prep<R><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
  hipEvent_t e0, e1;
  HIPCHK(c, hipEventCreate(&e0));
  HIPCHK(c, hipEventCreate(&e1));
  HIPCHK(c, hipEventRecord(e0, E.st));
  launch_ms<R>(E, T_APPLY, mp, L);
  HIPCHK(c, hipEventRecord(e1, E.st));
  TRY(sync(E));
  float ms = 0.f;
  HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *us = 1000.f * ms / (float)L;
  return OV_OK;
}

}  // namespace

// =================================================================== C ABI
extern "C" {

void ov_params_default(ov_params* p) {
  std::memset(p, 0, sizeof(*p));
  p->dims[0] = p->dims[1] = p->dims[2] = p->dims[3] = 4;
  p->bc_t = -1;
  p->M0 = 1.0;
  p->m_re = 0.05;
  p->g_re = 0.3;
  p->n_poles = 20;
  p->lambda_min = 1e-3;
  p->lambda_max = 8.0;
  p->inner_tol = 1e-12;
  p->outer_tol = 1e-10;
  p->truth_tol = 1e-13;
  p->mixed_inner_tol = 1e-6;
  p->reliable_delta = 3e-4;
  p->max_inner = 400;
  p->max_outer = 2000;
  p->precision = OV_MIXED;
  p->inner_relax = 3e-4;
  p->inner_tol_max = 1e-2;
  p->precondition = 1;
  p->truth_relax = 0.01;
  p->inner_form = 1;
  p->pc_mass = 1;
}

const char* ov_status_string(ov_status s) {
  switch (s) {
    case OV_OK: return "ok";
    case OV_ERR_INVALID_ARG: return "invalid argument";
    case OV_ERR_NOT_CONVERGED: return "not converged";
    case OV_ERR_BREAKDOWN: return "breakdown";
    case OV_ERR_SPECTRUM: return "spectrum outside the approximation interval";
    case OV_ERR_WORKSPACE: return "workspace too small";
    case OV_ERR_DEVICE: return "device error";
  }
  return "unknown status";
}

const char* ov_last_error(const ov_ctx* ctx) { return ctx ? ctx->err.c_str() : g_err.c_str(); }

ov_status ov_zolotarev(int n, double lmin, double lmax, double* a, double* b, double* delta) {
  if (!a || !b || n < 1 || n > MAXP) return OV_ERR_INVALID_ARG;
  return zolotarev_coeffs(n, lmin, lmax, a, b, delta) == 0 ? OV_OK : OV_ERR_INVALID_ARG;
}

ov_status ov_ctx_create(const ov_params* p, void* hip_stream, ov_ctx** out) {
  if (!out) return OV_ERR_INVALID_ARG;
  *out = nullptr;
  if (!p) {
    g_err = "null params";
    return OV_ERR_INVALID_ARG;
  }
  std::string err;
  ov_status s = validate(p, err);
  if (s != OV_OK) {
    g_err = err;
    return s;
  }
  ov_ctx* c = new ov_ctx();
  c->p = *p;
  // Small lattices take 64 threads per workgroup, so that a launch still has enough
  // workgroups to spread over the chip (8^4, two sources per pass: 128 instead of 32;
  // mixed solve 8.45 -> 7.74 ms); ov_set_launch overrides it.
  if ((long long)p->dims[0] * p->dims[1] * p->dims[2] * p->dims[3] <= 8192) c->block = 64;
  c->stream = (hipStream_t)hip_stream;
  if (zolotarev_coeffs(p->n_poles, p->lambda_min, p->lambda_max, c->a, c->b, &c->delta) != 0) {
    g_err = "Zolotarev coefficients failed";
    delete c;
    return OV_ERR_INVALID_ARG;
  }
  free_spectrum(p, c->smin, c->smax);
  if (c->smin < p->lambda_min * (1 - 1e-12) || c->smax > p->lambda_max * (1 + 1e-12)) {
    char buf[200];
    std::snprintf(buf, sizeof buf, "free |H_W| in [%.6g, %.6g] not inside [%.6g, %.6g]", c->smin,
                  c->smax, p->lambda_min, p->lambda_max);
    g_err = buf;
    delete c;
    return OV_ERR_SPECTRUM;
  }
  if (hipGetDevice(&c->device) != hipSuccess) {
    g_err = "no HIP device";
    delete c;
    return OV_ERR_DEVICE;
  }
  if (hipStreamCreateWithFlags(&c->priv, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&c->ev_in, hipEventDisableTiming) != hipSuccess) {
    g_err = "stream/event creation failed";
    if (c->priv) (void)hipStreamDestroy(c->priv);
    delete c;
    return OV_ERR_DEVICE;
  }
  // set-up of the no-allocation entry point: the scratch array's device address and
  // host staging for kNoAllocSystems systems
  if (noalloc_scratch_setup(c) != OV_OK || host_setup(c) != OV_OK) {
    g_err = c->err;
    (void)hipEventDestroy(c->ev_in);
    (void)hipStreamDestroy(c->priv);
    if (c->host_block) (void)hipHostFree(c->host_block);
    delete c;
    return OV_ERR_DEVICE;
  }
  const char* eg = std::getenv("OV_GRAPHS");
  c->use_graphs = (eg && *eg == '1');
  const char* ef = std::getenv("OV_FFT_FIXED");
  c->fft_fixed = !(ef && *ef == '0');
  if (res_setup(c) != OV_OK) {
    g_err = c->err;
    (void)ov_ctx_destroy(c);
    return OV_ERR_DEVICE;
  }
  *out = c;
  return OV_OK;
}

ov_status ov_ctx_destroy(ov_ctx* c) {
  if (!c) return OV_ERR_INVALID_ARG;
  if (c->priv) (void)hipStreamSynchronize(c->priv);
  if (c->device >= 0 && c->device < kMaxDevices) g_res_gate[c->device].forget(c);
  clear_graphs(c);
  if (c->ev_res) (void)hipEventDestroy(c->ev_res);
  if (c->res_sh) (void)hipFree(c->res_sh);
  for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
  if (c->ev_in) (void)hipEventDestroy(c->ev_in);
  if (c->priv) (void)hipStreamDestroy(c->priv);
  if (c->own_ws) (void)hipFree(c->own_ws);
  if (c->ts_dev) (void)hipFree(c->ts_dev);
  host_free(c, c->pinned);
  host_free(c, c->pinned_flags);
  host_free(c, c->stage);
  if (c->host_block) (void)hipHostFree(c->host_block);
  delete c;
  return OV_OK;
}

// Workspace bytes of a plan for nrhs systems of this context, for any launch shape
// (the partial-sum arrays are sized for 64 sites per workgroup).
static size_t plan_bytes(const ov_ctx* c, int nrhs, bool solve, bool mixed, double tol64,
                         double tolR, int nshift) {
  Engine E;
  std::vector<ov_ctx*> v(nrhs, const_cast<ov_ctx*>(c));
  plan_engine(E, v, solve, mixed, tol64, tolR, nshift);
  E.size_worst = true;
  return E.layout(nullptr, 0, true);
}

size_t ov_workspace_bytes(const ov_ctx* c, int nrhs) {
  if (!c || nrhs < 1) return 0;
  // the solve plan (solve, force) covers every other call without shifted systems
  // (sign, apply, locality, boson, pack, the tuning probe in the context's precision)
  const size_t solve = plan_bytes(c, nrhs, true, c->p.precision == OV_MIXED, solve_tol64(c),
                                  solve_tolR(c), 0);
  const size_t apply = plan_bytes(c, nrhs, false, false, c->p.inner_tol, c->p.inner_tol, 0);
  // a mixed solve whose cycles stagnate is finished by the FP64 solver
  const size_t fallback = c->p.precision == OV_MIXED
                              ? plan_bytes(c, nrhs, true, false, solve_tol64(c), c->p.inner_tol, 0)
                              : 0;
  return std::max(std::max(solve, apply), fallback);
}

static bool shifted_pc_on(const ov_ctx* c);

size_t ov_workspace_bytes_rational(const ov_ctx* c, int nrhs, int nshift) {
  if (!c || nrhs < 1 || nshift < 1 || nshift > MAXP) return 0;
  size_t need = plan_bytes(c, nrhs, true, false, solve_tol64(c), c->p.inner_tol, nshift);
  if (shifted_pc_on(c))  // shifts solved one by one: the solve plans (and the FP64 retry)
    need = std::max(need, ov_workspace_bytes(c, nrhs));
  return need;
}

ov_status ov_set_workspace(ov_ctx* c, void* ptr, size_t bytes) {
  if (!c) return OV_ERR_INVALID_ARG;
  if (ptr && ((uintptr_t)ptr & 255)) {
    c->err = "workspace must be 256-byte aligned";
    return OV_ERR_INVALID_ARG;
  }
  if (c->priv) (void)hipStreamSynchronize(c->priv);
  clear_graphs(c);
  c->user_ws = ptr;
  c->user_ws_bytes = ptr ? bytes : 0;
  return OV_OK;
}

ov_status ov_get_coeffs(const ov_ctx* c, double* a, double* b, double* delta) {
  if (!c || !a || !b) return OV_ERR_INVALID_ARG;
  for (int k = 0; k < c->p.n_poles; ++k) {
    a[k] = c->a[k];
    b[k] = c->b[k];
  }
  if (delta) *delta = c->delta;
  return OV_OK;
}

ov_status ov_set_launch(ov_ctx* c, int block, int spt) {
  if (!c) return OV_ERR_INVALID_ARG;
  if (block) {
    if (block < 64 || block > 256 || (block & 63)) return OV_ERR_INVALID_ARG;
    c->block = block;
  }
  if (spt < 0 || spt > 16) return OV_ERR_INVALID_ARG;
  if (spt) c->spt = spt;
  return OV_OK;
}

ov_status ov_get_launch(const ov_ctx* c, int* block, int* spt) {
  if (!c) return OV_ERR_INVALID_ARG;
  if (block) *block = c->block;
  if (spt) *spt = c->spt;
  return OV_OK;
}

// na bytes at a and nb at b share some.
static bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

// A gradient on top of xi or phi is written only once the launches of Y = M X are known to
// have ended well: the call runs again, from its inputs, when one has given up waiting.
static ov_status before_gradient(Engine& E, const void* grad, const void* xi, const void* phi) {
  const size_t sb = (size_t)E.sb[0].V * sizeof(double2);
  if (E.resident<double>(1) && (overlap(grad, sb, xi, 4 * sb * E.nsys) || overlap(grad, sb, phi, sb)))
    return sync(E);
  return OV_OK;
}

static ov_status apply_impl(ov_ctx* c, int op, void* out, const void* in, const void* phi,
                            int nrhs, ov_stats* st) {
  if (!c || !out || !in || nrhs < 1) return OV_ERR_INVALID_ARG;
  if ((op == OV_OP_M || op == OV_OP_M_DAG || op == OV_OP_MDAGM) && !phi) {
    c->err = "phi required for M, M^dag, MdagM";
    return OV_ERR_INVALID_ARG;
  }
  const double t0 = now_s();
  Engine E;
  std::vector<ov_ctx*> v(nrhs, c);
  TRY(engine_init(E, v, false, false, c->p.inner_tol, c->p.inner_tol));
  // Operators without a multi-shift, and those whose multi-shift runs in resident launches,
  // work on the caller's fields themselves, unless the result overlaps one that is read; the
  // former report nothing from the device.
  const bool shifts = op != OV_OP_HW && op != OV_OP_M0INV && op != OV_OP_M0INV_DAG &&
                      (op < OV_OP_DOV || c->p.dirac == OV_DIRAC_OVERLAP_MS);
  E.shifts = shifts;
  if (!shifts)
    std::memset(c->pinned, 0, sizeof(double) * CG_NSLOT * E.nsys + sizeof(int) * E.ctl_words);
  const size_t vb = (size_t)E.sb[0].V * 4 * sizeof(double2);
  E.io.resize(nrhs);
  for (int r = 0; r < nrhs; ++r)
    E.io[r] = {(const char*)in + r * vb, E.sb[r].x64, E.sb[r].r64, (char*)out + r * vb};
  // phi: a site's result may land on another site's phi
  const bool yuk = op == OV_OP_M || op == OV_OP_M_DAG || op == OV_OP_MDAGM;
  const bool apart = !overlap(out, nrhs * vb, in, nrhs * vb) &&
                     !(yuk && overlap(out, nrhs * vb, phi, vb / 4));
  const bool direct = apart && (!shifts || E.resident<double>(1));
  TRY(run_apply(E, op, phi, direct && shifts, shifts));
  if (!direct) TRY(pack64(E));
  TRY(apply_sequence(E, op, direct));
  if (!direct) {
    // overlapping fields: out may be in, which a call whose resident launch gave up
    // waiting needs again, so it is written only once the launch is known to have ended well
    if (shifts && E.resident<double>(1)) TRY(read_scalars(E));
    TRY(unpack64(E));
  }
  TRY(shifts ? read_scalars(E) : sync(E));
  ov_status rc = OV_OK;
  for (int s = 0; s < nrhs; ++s) {
    const int bits = sys_ctl(E, s).bits;
    if (bits & (1 << 1)) rc = OV_ERR_BREAKDOWN;
    else if ((bits & (1 << 2)) && rc == OV_OK) rc = OV_ERR_NOT_CONVERGED;
  }
  if (rc == OV_ERR_BREAKDOWN) c->err = "multi-shift breakdown (non-finite input?)";
  if (rc == OV_ERR_NOT_CONVERGED) c->err = "multi-shift did not converge within its basis";
  fill_stats(st, nrhs, &E, nullptr, now_s() - t0, 16);
  return rc;
}

ov_status ov_sign(ov_ctx* c, void* out, const void* in, int nrhs, ov_stats* st) {
  Range range("ov_sign");
  return res_retry(c, [&] { return apply_impl(c, -1, out, in, nullptr, nrhs, st); });
}

ov_status ov_apply(ov_ctx* c, ov_op op, void* out, const void* in, const void* phi, int nrhs,
                   ov_stats* st) {
  Range range("ov_apply");
  if ((int)op < 0 || (int)op > OV_OP_M0INV_DAG) return OV_ERR_INVALID_ARG;
  if (c && (op == OV_OP_M0INV || op == OV_OP_M0INV_DAG) && !fft_ok(&c->p, c->err))
    return OV_ERR_INVALID_ARG;
  return res_retry(c, [&] { return apply_impl(c, (int)op, out, in, phi, nrhs, st); });
}

ov_status ov_apply_noalloc(ov_ctx* c, ov_op op, void* out, const void* in, const void* phi,
                           int nrhs, ov_stats* st) {
  Range range("ov_apply_noalloc");
  if (!c || nrhs < 1) return OV_ERR_INVALID_ARG;
  if (nrhs > c->pinned_n) {
    char buf[120];
    std::snprintf(buf, sizeof buf, "no-allocation calls take at most %d right-hand sides",
                  c->pinned_n);
    c->err = buf;
    return OV_ERR_WORKSPACE;
  }
  // kernel-duration sampling creates events and stamp buffers: off for this call
  const int sample_max = c->sample_max;
  c->sample_max = 0;
  c->noalloc = true;
  const ov_status rc = ov_apply(c, op, out, in, phi, nrhs, st);
  c->noalloc = false;
  c->sample_max = sample_max;
  return rc;
}

static bool same_solver(const ov_params& a, const ov_params& b) {
  return a.n_poles == b.n_poles && a.lambda_min == b.lambda_min && a.lambda_max == b.lambda_max &&
         a.inner_tol == b.inner_tol && a.outer_tol == b.outer_tol && a.truth_tol == b.truth_tol &&
         a.mixed_inner_tol == b.mixed_inner_tol && a.reliable_delta == b.reliable_delta &&
         a.precision == b.precision && a.M0 == b.M0 && a.inner_relax == b.inner_relax &&
         a.inner_tol_max == b.inner_tol_max && a.precondition == b.precondition &&
         a.dirac == b.dirac && a.truth_relax == b.truth_relax && a.inner_form == b.inner_form &&
         a.pc_mass == b.pc_mass;
}

static ov_status solve_systems(std::vector<ov_ctx*>& sysctx, std::vector<const void*>& bv,
                               std::vector<void*>& xv, std::vector<const void*>& phv,
                               ov_stats* st) {
  ov_ctx* c = sysctx[0];
  const double t0 = now_s();
  const bool mixed = c->p.precision == OV_MIXED;
  const double tolR = mixed ? c->p.mixed_inner_tol : c->p.inner_tol;
  Engine E;
  TRY(engine_init(E, sysctx, true, mixed, solve_tol64(c), tolR));
  const int ns = E.nsys;
  E.force_fallback = mixed && force_fallback_env();
  E.io.resize(ns);
  for (int s = 0; s < ns; ++s) E.io[s] = {xv[s], E.sb[s].x64, E.sb[s].x64, xv[s]};
  E.guess = true;
  SolveOut so;
  const double delta = c->p.reliable_delta;
  ov_status rc = mixed ? solve_engine<float>(E, bv, phv, tolR, delta, so)
                       : solve_engine<double>(E, bv, phv, tolR, delta, so);
  if (rc != OV_OK && rc != OV_ERR_NOT_CONVERGED) return rc;
  TRY(unpack64(E));
  TRY(read_scalars(E));
  fill_stats(st, ns, &E, &so, now_s() - t0, mixed ? 8 : 16);
  if (rc != OV_OK) return rc;  // x holds the best iterate; err says why
  // Systems whose mixed-precision cycles stagnated: the FP64 solver (fixed inner
  // tolerance inner_tol, no relaxation) finishes them from the iterate just written to x.
  std::vector<int> fb;
  int used = 0;  // outer iterations the mixed solver spent on the systems handed over
  for (int s = 0; s < ns; ++s)
    if (so.fallback[s]) {
      fb.push_back(s);
      used = std::max(used, so.outer[s]);
    }
  if (!fb.empty() && used < c->p.max_outer) {
    if (ov_log()) std::fprintf(stderr, "[ov] %zu system(s) handed to the FP64 solver\n", fb.size());
    std::vector<ov_ctx*> c2;
    std::vector<const void*> b2, p2;
    std::vector<void*> x2;
    for (int s : fb) {
      c2.push_back(sysctx[s]);
      b2.push_back(bv[s]);
      p2.push_back(phv[s]);
      x2.push_back(xv[s]);
    }
    Engine F;
    TRY(engine_init(F, c2, true, false, solve_tol64(c), c->p.inner_tol));
    F.no_relax = true;
    F.max_outer = c->p.max_outer - used;
    F.io.resize(F.nsys);
    for (int k = 0; k < F.nsys; ++k) F.io[k] = {x2[k], F.sb[k].x64, F.sb[k].x64, x2[k]};
    F.guess = true;
    SolveOut so2;
    rc = solve_engine<double>(F, b2, p2, c->p.inner_tol, delta, so2);
    if (rc != OV_OK && rc != OV_ERR_NOT_CONVERGED) return rc;
    TRY(unpack64(F));
    TRY(read_scalars(F));
    std::vector<ov_stats> st2(F.nsys);
    fill_stats(st2.data(), F.nsys, &F, &so2, now_s() - t0, 16);
    for (int k = 0; k < F.nsys; ++k) {
      const int s = fb[k];
      so.conv[s] = so2.conv[k];
      so.res[s] = so2.res[k];
      if (st) {
        st[s].outer_iters += st2[k].outer_iters;
        st[s].reliable_updates += st2[k].reliable_updates;
        st[s].inner_iters += st2[k].inner_iters;
        st[s].stencil_apps += st2[k].stencil_apps;
        st[s].model_bytes += st2[k].model_bytes;
        st[s].true_rel_res = st2[k].true_rel_res;
        st[s].max_shift_res = st2[k].max_shift_res;
        st[s].stagnations += so2.stag[k];
        st[s].fp64_fallback = 1;
      }
    }
    if (st)
      for (int s = 0; s < ns; ++s) st[s].seconds = now_s() - t0;
    if (rc != OV_OK) return rc;
  }
  for (int s = 0; s < ns; ++s)
    if (!so.conv[s]) {
      c->err = "outer CG did not reach outer_tol within max_outer";
      return OV_ERR_NOT_CONVERGED;
    }
  return OV_OK;
}

ov_status ov_solve(ov_ctx* c, void* x, const void* b, const void* phi, int nrhs, ov_stats* st) {
  Range range("ov_solve");
  if (!c || !x || !b || !phi || nrhs < 1) return OV_ERR_INVALID_ARG;
  const size_t vb = (size_t)c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3] * 4 *
                    sizeof(double2);
  std::vector<ov_ctx*> sc(nrhs, c);
  std::vector<const void*> bv(nrhs), ph(nrhs, phi);
  std::vector<void*> xv(nrhs);
  for (int r = 0; r < nrhs; ++r) {
    bv[r] = (const char*)b + r * vb;
    xv[r] = (char*)x + r * vb;
  }
  return res_retry(c, [&] { return solve_systems(sc, bv, xv, ph, st); });
}

ov_status ov_solve_batch(int n, ov_ctx* const* ctx, void* const* x, const void* const* b,
                         const void* const* phi, const int* nrhs, ov_stats* st) {
  Range range("ov_solve_batch");
  if (n < 1 || !ctx || !x || !b || !phi || !nrhs) return OV_ERR_INVALID_ARG;
  std::vector<ov_ctx*> sc;
  std::vector<const void*> bv, ph;
  std::vector<void*> xv;
  for (int i = 0; i < n; ++i) {
    if (!ctx[i] || !x[i] || !b[i] || !phi[i] || nrhs[i] < 1) return OV_ERR_INVALID_ARG;
    if (!same_solver(ctx[i]->p, ctx[0]->p)) {
      ctx[0]->err = "batched contexts must share poles, interval, tolerances and precision";
      return OV_ERR_INVALID_ARG;
    }
    const size_t vb = (size_t)ctx[i]->p.dims[0] * ctx[i]->p.dims[1] * ctx[i]->p.dims[2] *
                      ctx[i]->p.dims[3] * 4 * sizeof(double2);
    for (int r = 0; r < nrhs[i]; ++r) {
      sc.push_back(ctx[i]);
      bv.push_back((const char*)b[i] + r * vb);
      xv.push_back((char*)x[i] + r * vb);
      ph.push_back(phi[i]);
    }
  }
  return res_retry(sc.data(), sc.size(), [&] { return solve_systems(sc, bv, xv, ph, st); });
}

static ov_status force_impl(ov_ctx* c, void* grad_phi, double* S_host, const void* xi, const void* phi,
                   int nrhs, ov_stats* st) {
  if (!c || !grad_phi || !S_host || !xi || !phi || nrhs < 1) return OV_ERR_INVALID_ARG;
  const double t0 = now_s();
  const size_t V = (size_t)c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3];
  const size_t vb = V * 4 * sizeof(double2);
  std::vector<ov_ctx*> sc(nrhs, c);
  std::vector<const void*> bv(nrhs), ph(nrhs, phi);
  std::vector<void*> xv(nrhs);
  // X = (MdagM)^-1 xi, cold start, kept in the engine's x64 buffers
  const bool mixed = c->p.precision == OV_MIXED;
  Engine E;
  TRY(engine_init(E, sc, true, mixed, std::min(c->p.inner_tol, c->p.truth_tol),
                  mixed ? c->p.mixed_inner_tol : c->p.inner_tol));
  E.force_fallback = mixed && force_fallback_env();
  // zero guess directly in x64
  for (int r = 0; r < nrhs; ++r) {
    bv[r] = (const char*)xi + r * vb;
    zero_dev(E, E.sb[r].x64, vb);
  }
  SolveOut so;
  const double tolR = mixed ? c->p.mixed_inner_tol : c->p.inner_tol;
  ov_status rc = mixed ? solve_engine<float>(E, bv, ph, tolR, c->p.reliable_delta, so)
                       : solve_engine<double>(E, bv, ph, tolR, c->p.reliable_delta, so);
  if (rc != OV_OK) return rc;
  bool fell_back = false;
  for (int r = 0; r < nrhs; ++r) fell_back |= so.fallback[r] != 0;
  if (fell_back) {
    // the force's FP64 solve starts cold: it gets the whole max_outer
    // a stagnating mixed solve: the FP64 solver (fixed inner tolerance) solves again
    // from a cold start in an engine of its own (X must sit in that engine's buffers)
    if (ov_log()) std::fprintf(stderr, "[ov] force solve handed to the FP64 solver\n");
    E = Engine{};
    TRY(engine_init(E, sc, true, false, std::min(c->p.inner_tol, c->p.truth_tol),
                    c->p.inner_tol));
    E.no_relax = true;
    for (int r = 0; r < nrhs; ++r) zero_dev(E, E.sb[r].x64, vb);
    SolveOut so2;
    rc = solve_engine<double>(E, bv, ph, c->p.inner_tol, c->p.reliable_delta, so2);
    if (rc != OV_OK) return rc;
    for (int r = 0; r < nrhs; ++r) {
      so2.outer[r] += so.outer[r];
      so2.ru[r] += so.ru[r];
      so2.stag[r] += so.stag[r];
    }
    so = so2;
  }
  for (int r = 0; r < nrhs; ++r)
    if (!so.conv[r]) {
      c->err = "force solve did not converge";
      return OV_ERR_NOT_CONVERGED;
    }
  // Y = M X (FP64, recomputed: no shifted vector was kept)
  E.htab.assign((size_t)E.ntab * nrhs, SysDev{});
  for (int s = 0; s < nrhs; ++s) {
    SysBuf& b = E.sb[s];
    SysDev d = base_dev(b);
    d.phi = (const double2*)phi;
    d.basis = b.basis64;
    d.r = b.r64ms;
    d.src = b.x64;
    d.e_in = b.x64;
    d.e_out = b.u64;
    d.fft_tmp = b.src64b;
    d.cg_b = (const double2*)bv[s];
    E.htab[(size_t)T_APPLY * nrhs + s] = d;
  }
  TRY(upload_tables(E));
  if (E.pl.fft) {
    launch_sym<double>(E, T_APPLY, SYM_D);
    k_yuk<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
  } else {
    MsParams mp = make_mp(c, c->p.truth_tol, E.pl.cap64);
    const int L = std::min(E.pl.cap64, capacity(c, c->p.truth_tol));
    clear_ctl(E);  // the sticky bits below then belong to the Y = M X multi-shift alone
    k_ms_prep<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
    launch_ms<double>(E, T_APPLY, mp, L);
    launch_combine<double>(E, T_APPLY, EPI_M);
  }
  // S_r = Re <xi_r, X_r>
  k_dot_re<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  TRY(before_gradient(E, grad_phi, xi, phi));
  // G summed over right-hand sides in order (one launch over the sites)
  k_force<<<E.sb[0].nblk, E.block, 0, E.st>>>(tab(E, T_APPLY), nrhs, E.sb[0].nblk,
                                               (double2*)grad_phi);
  k_cg_scalar<<<nrhs, 256, 0, E.st>>>(tab(E, T_APPLY), nrhs, 4);  // S_r -> BB
  TRY(read_scalars(E));
  if (!E.pl.fft) {
    int bits = 0;
    for (int s = 0; s < nrhs; ++s) bits |= sticky_bits(E, s);
    TRY(sticky_status(c, bits, "ov_force, Y = M X"));
  }
  for (int s = 0; s < nrhs; ++s) S_host[s] = c->pinned[(size_t)s * CG_NSLOT + CG_BB];
  fill_stats(st, nrhs, &E, &so, now_s() - t0, (mixed && !fell_back) ? 8 : 16);
  if (st && fell_back)
    for (int r = 0; r < nrhs; ++r) st[r].fp64_fallback = 1;
  return OV_OK;
}

ov_status ov_force(ov_ctx* c, void* grad_phi, double* S_host, const void* xi, const void* phi,
                   int nrhs, ov_stats* st) {
  Range range("ov_force");
  return res_retry(c, [&] {
    return force_impl(c, grad_phi, S_host, xi, phi, nrhs, st);
  });
}

// ------------------------------------------------ rational layers (Sec. 7.3)
// One multi-shift CG on MdagM (FP64) for (MdagM + beta_i) X_i = b, i < n, for
// every system of E; the base CG has shift 0.  Leaves X_i in shx and
// r64 = a0 b + sum_i alpha_i X_i.  Shift i stops once |zeta_i| |r| <= outer_tol |b|.
static ov_status rational_core(ov_ctx* c, Engine& E, double a0, int n, const double* al,
                               const double* be, const std::vector<const void*>& bv,
                               const std::vector<const void*>& phv, std::vector<int>& iters) {
  const int ns = E.nsys;
  TRY(build_solve_tables<double>(E, bv, phv));
  TRY(reset_stats(E));
  // coefficients: residues and a0 once; per-iteration blocks below
  std::vector<double> blk((size_t)ns * SHC_LEN, 0.0);
  auto upload = [&]() -> ov_status {
    TRY(sync(E));  // the staging vector feeds the copies below
    for (int s = 0; s < ns; ++s)
      HIPCHK(c, hipMemcpyAsync(E.sb[s].shc, blk.data() + (size_t)s * SHC_LEN,
                               sizeof(double) * SHC_LEN, hipMemcpyHostToDevice, E.st));
    return OV_OK;
  };
  for (int s = 0; s < ns; ++s) {
    double* b = blk.data() + (size_t)s * SHC_LEN;
    for (int k = 0; k < n; ++k) b[SHC_RES + k] = al[k];
    b[SHC_A0] = a0;
  }
  TRY(upload());
  std::vector<int> fcg(ns, 1), fru(ns, 0);
  TRY(set_flags(E, fcg, fru));
  const int nb = E.nb_total, bl = E.block;
  k_cg_misc<double><<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 2);  // x = 0
  k_cg_misc<double><<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 1);  // r = b, |b|^2
  k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 4);
  k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 0);
  k_cg_p<double><<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 1);     // p = r
  k_shift<<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 0);             // x_i = 0, p_i = r
  TRY(read_scalars(E));
  std::vector<double> bn(ns);
  // per system and shift: zeta_{n-1}, zeta_n; per system alpha_{n-1}, beta_{n-1}
  std::vector<double> zo((size_t)ns * n, 1.0), zc((size_t)ns * n, 1.0), aold(ns, 1.0),
      bold(ns, 0.0);
  std::vector<char> act((size_t)ns * n, 1);
  iters.assign(ns, 0);
  for (int s = 0; s < ns; ++s) {
    bn[s] = std::sqrt(c->pinned[(size_t)s * CG_NSLOT + CG_BB]);
    if (!std::isfinite(bn[s])) {
      c->err = "non-finite right-hand side";
      return OV_ERR_BREAKDOWN;
    }
    if (bn[s] == 0.0) {
      fcg[s] = 0;
      for (int k = 0; k < n; ++k) act[(size_t)s * n + k] = 0;
    }
  }
  const double tol = c->p.outer_tol;
  const MsParams mp = make_mp(c, c->p.inner_tol, E.pl.cap64);
  // the exact Ginsparg-Wilson product takes eps^2 p from the Krylov space of p, about
  // ten times less accurate than the shifted solutions: its multi-shift runs ten times
  // tighter
  const double tol_ms = E.pl.gwx ? 0.1 * c->p.inner_tol : c->p.inner_tol;
  const MsParams mpx = make_mp(c, tol_ms, E.pl.cap64);
  int L = 0;
  for (int s = 0; s < ns; ++s) L = std::max(L, capacity(E.ctxs[s], tol_ms));
  L = std::min(E.pl.cap64, L);
  int Lrun = L;
  // w = MdagM p (vR for the multi-shift forms), alpha = rho / Re <p, w>
  auto product = [&](int Ln) {
    if (E.pl.fft) {
      launch_sym<double>(E, T_F_M, SYM_D);
      k_yuk<double><<<nb, bl, 0, E.st>>>(tab(E, T_F_M), E.bmap, nb, 0);
      k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_F_M), ns, 1);
      launch_sym<double>(E, T_F_MD, SYM_D_DAG);
      k_yuk<double><<<nb, bl, 0, E.st>>>(tab(E, T_F_MD), E.bmap, nb, 1);
    } else if (E.pl.gwx) {
      // w = MdagM p exactly in Ginsparg-Wilson form: one two-source multi-shift
      // (eps^2 p from the Krylov space of p) -> vR, alpha = rho / Re <p, w>
      k_stat3_clear<<<1, 64, 0, E.st>>>(E.trgwtab, 2 * ns);
      k_gw_prep<double><<<nb, bl, 0, E.st>>>(E.trgwtab, E.trgwtab + ns, E.bmap, nb);
      launch_ms_tab<double>(E, E.trgwtab, E.gwbmap, 2 * nb, 2 * ns, mpx, Ln);
      k_truth_combine<<<nb, site_block(E), 0, E.st>>>(E.trgwtab, E.trgwtab + ns, E.bmap, nb);
      k_truth_finish<double><<<nb, bl, 0, E.st>>>(E.trgwtab, E.bmap, nb, 4.0 - c->p.M0, 1);
      k_cg_scalar<<<ns, 256, 0, E.st>>>(E.trgwtab, ns, 1);
    } else {
      k_ms_prep<double><<<nb, bl, 0, E.st>>>(tab(E, T_IN_M), E.bmap, nb, 0);
      launch_ms<double>(E, T_IN_M, mp, Ln);
      launch_combine<double>(E, T_IN_M, EPI_M);
      k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_IN_M), ns, 1);
      launch_ms<double>(E, T_IN_MDAG, mp, Ln);
      launch_combine<double>(E, T_IN_MDAG, EPI_MDAG);
    }
  };
  for (int it = 0; it < c->p.max_outer; ++it) {
    bool any = false;
    for (int s = 0; s < ns; ++s) any |= fcg[s] != 0;
    if (!any) break;
    const std::vector<int> live = fcg;  // the systems this iteration advances
    TRY(set_flags(E, fcg, fru));
    if (E.pl.fft) {
      product(0);
    } else {
      // The launch count follows the last iteration's need plus a margin; a product
      // cut short by it is recomputed with the full count before the CG update uses
      // it (the product of p is exact to the multi-shift tolerance in every iteration).
      clear_ctl(E);
      product(Lrun);
      TRY(read_scalars(E));
      int nobs = E.pl.gwx ? last_truth_iters(E) : last_ms_iters(E);
      if (Lrun < L && nobs >= Lrun - 1) {
        clear_ctl(E);
        product(L);
        TRY(read_scalars(E));
        nobs = E.pl.gwx ? last_truth_iters(E) : last_ms_iters(E);
      }
      int bits = 0;
      for (int s = 0; s < ns; ++s) bits |= live[s] ? sticky_bits(E, s) : 0;
      TRY(sticky_status(c, bits, "multi-shift CG on MdagM, product MdagM p"));
      if (!E.resident<double>(E.pl.gwx ? 2 : 1)) Lrun = std::min(L, nobs + 4);
    }
    k_cg_misc<double><<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 5);  // r -= alpha w
    k_cg_scalar<<<ns, 256, 0, E.st>>>(tab(E, T_CG), ns, 2);                // rho, beta
    TRY(read_scalars(E));
    for (int s = 0; s < ns; ++s) {
      if (!fcg[s]) continue;
      iters[s]++;
      const double* cs = c->pinned + (size_t)s * CG_NSLOT;
      const double a = cs[CG_ALPHA], bt = cs[CG_BETA], rho = cs[CG_RR];
      if (!std::isfinite(a) || !std::isfinite(rho) || cs[CG_PAP] <= 0.0) {
        c->err = "multi-shift CG on MdagM: breakdown (non-finite or non-positive scalar)";
        return OV_ERR_BREAKDOWN;
      }
      double* b = blk.data() + (size_t)s * SHC_LEN;
      bool alive = false;
      for (int k = 0; k < n; ++k) {
        const size_t j = (size_t)s * n + k;
        if (!act[j]) {
          b[4 * k + 3] = 0.0;
          continue;
        }
        const double zn = zc[j] * zo[j] * aold[s] /
                          (a * bold[s] * (zo[j] - zc[j]) + zo[j] * aold[s] * (1.0 + be[k] * a));
        const double ratio = zn / zc[j];
        b[4 * k] = a * ratio;               // alpha_i
        b[4 * k + 1] = zn;                  // zeta_i of r_{n+1}
        b[4 * k + 2] = bt * ratio * ratio;  // beta_i
        b[4 * k + 3] = 1.0;
        zo[j] = zc[j];
        zc[j] = zn;
        if (std::fabs(zn) * std::sqrt(std::max(rho, 0.0)) <= tol * bn[s]) act[j] = 0;
        alive |= act[j] != 0;
      }
      aold[s] = a;
      bold[s] = bt;
      if (!alive) fcg[s] = 0;
    }
    TRY(upload());
    // The shifted update of this iteration applies to the systems it advanced (a shift
    // that converged just now still takes its last step); systems that had converged
    // before are left alone.
    TRY(set_flags(E, live, fru));
    k_shift<<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 1);
    TRY(set_flags(E, fcg, fru));
    k_cg_p<double><<<nb, bl, 0, E.st>>>(tab(E, T_CG), E.bmap, nb, 1);  // p = r + beta p
  }
  for (int s = 0; s < ns; ++s)
    if (fcg[s]) {
      c->err = "multi-shift CG on MdagM did not converge within max_outer";
      return OV_ERR_NOT_CONVERGED;
    }
  // r64 = a0 b + sum_i alpha_i X_i
  for (int s = 0; s < ns; ++s) E.htab[(size_t)T_APPLY * ns + s].e_out = E.sb[s].r64;
  TRY(upload_tables(E));
  k_rat_combine<<<nb, bl, 0, E.st>>>(tab(E, T_APPLY), E.bmap, nb);
  return check_launch(c);
}

// Whether a context's rational layers solve their small shifts one by one with the
// preconditioned solver (shift_pc_cutoff): the shifted operator needs the Ginsparg-Wilson
// inner form or a momentum-space D.
static bool shifted_pc_on(const ov_ctx* c) {
  return c->p.shift_pc_cutoff > 0.0 && c->p.precondition != 0 &&
         (c->p.inner_form == 1 || c->p.dirac != OV_DIRAC_OVERLAP_MS);
}

// (MdagM + sigma) X = b for every right-hand side bv (cold start) with the solver of the
// context's precision and the free shifted preconditioner, then outs[r] += alpha X_r (ABI
// layout).  A mixed solve whose cycles stagnate is solved again in FP64.  Adds the outer
// iterations, reliable updates and multi-shift iterations to the totals.
static ov_status shifted_solve_acc(ov_ctx* c, double sigma, double alpha,
                                   const std::vector<const void*>& bv,
                                   const std::vector<const void*>& ph,
                                   const std::vector<void*>& outs, std::vector<int>& outer,
                                   std::vector<int>& ru, std::vector<long long>& inner) {
  const int ns = (int)bv.size();
  const size_t vb = (size_t)c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3] * 4 *
                    sizeof(double2);
  std::vector<ov_ctx*> sc(ns, c);
  const bool mixed = c->p.precision == OV_MIXED;
  for (int attempt = 0; attempt < 2; ++attempt) {
    const bool m = mixed && attempt == 0;
    const double tolR = m ? c->p.mixed_inner_tol : c->p.inner_tol;
    Engine F;
    TRY(engine_init(F, sc, true, m, solve_tol64(c), tolR));
    F.shift = sigma;
    F.io.resize(ns);
    for (int r = 0; r < ns; ++r) F.io[r] = {nullptr, nullptr, F.sb[r].x64, outs[r]};
    F.no_relax = attempt == 1;
    for (int r = 0; r < ns; ++r) zero_dev(F, F.sb[r].x64, vb);
    SolveOut so;
    ov_status rc = m ? solve_engine<float>(F, bv, ph, tolR, c->p.reliable_delta, so)
                     : solve_engine<double>(F, bv, ph, tolR, c->p.reliable_delta, so);
    if (rc != OV_OK) return rc;
    TRY(read_scalars(F));
    bool fell_back = false;
    for (int r = 0; r < ns; ++r) {
      outer[r] += so.outer[r];
      ru[r] += so.ru[r];
      inner[r] += sys_ctl(F, r).inner;
      fell_back |= so.fallback[r] != 0;
    }
    if (fell_back && m) continue;
    for (int r = 0; r < ns; ++r)
      if (!so.conv[r]) {
        c->err = "shifted solve of the rational layer did not converge within max_outer";
        return OV_ERR_NOT_CONVERGED;
      }
    k_unpack_axpy<<<F.nb_total, F.block, 0, F.st>>>(tab(F, T_APPLY), F.bmap, F.nb_total, alpha);
    return sync(F);
  }
  c->err = "shifted solve of the rational layer: FP64 retry did not finish";
  return OV_ERR_NOT_CONVERGED;
}

static ov_status rational_impl(ov_ctx* c, double a0, int n, const double* alpha, const double* beta,
                      void* out, const void* in, const void* phi, int nrhs, ov_stats* st) {
  if (!c || !alpha || !beta || !out || !in || !phi || nrhs < 1 || n < 1 || n > MAXP)
    return OV_ERR_INVALID_ARG;
  for (int k = 0; k < n; ++k)
    if (!(beta[k] >= 0.0) || !std::isfinite(alpha[k]) || !std::isfinite(beta[k])) {
      c->err = "ov_rational: need finite alpha_i and beta_i >= 0";
      return OV_ERR_INVALID_ARG;
    }
  const double t0 = now_s();
  const size_t vb = (size_t)c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3] * 4 *
                    sizeof(double2);
  std::vector<ov_ctx*> sc(nrhs, c);
  std::vector<const void*> bv(nrhs), ph(nrhs, phi);
  std::vector<void*> ov(nrhs);
  for (int r = 0; r < nrhs; ++r) {
    bv[r] = (const char*)in + r * vb;
    ov[r] = (char*)out + r * vb;
  }
  // Shifts at or below shift_pc_cutoff: one preconditioned solve each (the paper's
  // heatbath, Sec. 7.3); the rest: one multi-shift CG on MdagM.
  std::vector<double> al_hi, be_hi, al_lo, be_lo;
  const bool split = shifted_pc_on(c);
  for (int k = 0; k < n; ++k) {
    const bool lo = split && beta[k] <= c->p.shift_pc_cutoff;
    (lo ? al_lo : al_hi).push_back(alpha[k]);
    (lo ? be_lo : be_hi).push_back(beta[k]);
  }
  std::vector<int> outer(nrhs, 0), ru(nrhs, 0);
  std::vector<long long> inner(nrhs, 0);
  std::vector<double> shift_res(nrhs, 0.0);
  if (!al_hi.empty()) {
    Engine E;
    TRY(engine_init(E, sc, true, false, solve_tol64(c), c->p.inner_tol, (int)al_hi.size()));
    E.io.resize(nrhs);
    for (int r = 0; r < nrhs; ++r) E.io[r] = {nullptr, nullptr, E.sb[r].r64, ov[r]};
    std::vector<int> iters;
    TRY(rational_core(c, E, a0, (int)al_hi.size(), al_hi.data(), be_hi.data(), bv, ph, iters));
    TRY(unpack64(E));
    TRY(read_scalars(E));
    for (int r = 0; r < nrhs; ++r) {
      const SysCtl k = sys_ctl(E, r);
      outer[r] += iters[r];
      inner[r] += k.inner;
      shift_res[r] = k.shift_res;
    }
  } else {  // out = a0 in, ordered after the caller's stream like every other launch
    HIPCHK(c, hipEventRecord(c->ev_in, c->stream));
    HIPCHK(c, hipStreamWaitEvent(c->priv, c->ev_in, 0));
    const size_t nel = (size_t)nrhs * vb / sizeof(double2);
    k_scale_copy<<<(unsigned)std::min<size_t>((nel + 255) / 256, 4096), 256, 0, c->priv>>>(
        (double2*)out, (const double2*)in, a0, nel);
    TRY(check_launch(c));
  }
  for (size_t k = 0; k < al_lo.size(); ++k)
    TRY(shifted_solve_acc(c, be_lo[k], al_lo[k], bv, ph, ov, outer, ru, inner));
  if (st) {
    for (int r = 0; r < nrhs; ++r) {
      ov_stats& o = st[r];
      std::memset(&o, 0, sizeof(o));
      o.outer_iters = outer[r];
      o.reliable_updates = ru[r];
      o.inner_iters = inner[r];
      o.stencil_apps = 2 * inner[r];
      o.max_shift_res = shift_res[r];
      o.seconds = now_s() - t0;
    }
  }
  return OV_OK;
}

ov_status ov_rational(ov_ctx* c, double a0, int n, const double* alpha, const double* beta,
                      void* out, const void* in, const void* phi, int nrhs, ov_stats* st) {
  Range range("ov_rational");
  return res_retry(c, [&] {
    return rational_impl(c, a0, n, alpha, beta, out, in, phi, nrhs, st);
  });
}

static ov_status rational_force_impl(ov_ctx* c, double a0, int n, const double* alpha,
                            const double* beta, void* grad_phi, double* S_host, const void* xi,
                            const void* phi, int nrhs, ov_stats* st) {
  if (!c || !alpha || !beta || !grad_phi || !S_host || !xi || !phi || nrhs < 1 || n < 1 ||
      n > MAXP)
    return OV_ERR_INVALID_ARG;
  for (int k = 0; k < n; ++k)
    if (!(beta[k] >= 0.0) || !std::isfinite(alpha[k]) || !std::isfinite(beta[k])) {
      c->err = "ov_rational_force: need finite alpha_i and beta_i >= 0";
      return OV_ERR_INVALID_ARG;
    }
  const double t0 = now_s();
  const size_t V = (size_t)c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3];
  const size_t vb = V * 4 * sizeof(double2);
  std::vector<ov_ctx*> sc(nrhs, c);
  std::vector<const void*> bv(nrhs), ph(nrhs, phi);
  for (int r = 0; r < nrhs; ++r) bv[r] = (const char*)xi + r * vb;
  Engine E;
  TRY(engine_init(E, sc, true, false, solve_tol64(c), c->p.inner_tol, n));
  std::vector<int> iters;
  TRY(rational_core(c, E, a0, n, alpha, beta, bv, ph, iters));
  // S_r = Re xi_r^dag (a0 xi_r + sum_i alpha_i X_i) from the combined field in r64
  for (int s = 0; s < nrhs; ++s) E.htab[(size_t)T_APPLY * nrhs + s].e_in = E.sb[s].r64;
  TRY(upload_tables(E));
  k_dot_re<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  TRY(sync(E));
  for (int s = 0; s < nrhs; ++s) {
    std::vector<double> tmp(E.sb[s].nblk);
    HIPCHK(c, hipMemcpy(tmp.data(), E.sb[s].part_c, sizeof(double) * tmp.size(),
                        hipMemcpyDeviceToHost));
    double acc = 0;
    for (double v : tmp) acc += v;
    S_host[s] = acc;
  }
  // Y_i = alpha_i M X_i into the (no longer needed) search directions, FP64
  const MsParams mp = make_mp(c, c->p.truth_tol, E.pl.cap64);
  const int L = std::min(E.pl.cap64, capacity(c, c->p.truth_tol));
  const size_t slot = V * 4;
  std::vector<int> on(nrhs, 1), off(nrhs, 0);
  TRY(set_flags(E, on, off));
  clear_ctl(E);  // the sticky bits checked below then belong to the Y_i multi-shifts
  for (int k = 0; k < n; ++k) {
    for (int s = 0; s < nrhs; ++s) {
      SysDev& d = E.htab[(size_t)T_APPLY * nrhs + s];
      d.e_in = E.sb[s].shx + (size_t)k * slot;
      d.src = d.e_in;
      d.e_out = E.sb[s].shp + (size_t)k * slot;
      d.e_out2 = nullptr;
      d.fft_tmp = E.sb[s].src64b;
      d.basis = E.sb[s].basis64;
      d.r = E.sb[s].r64ms;
      d.active = nullptr;
    }
    TRY(upload_tables(E));
    if (E.pl.fft) {
      launch_sym<double>(E, T_APPLY, SYM_D);
      k_yuk<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
    } else {
      k_ms_prep<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, 0);
      launch_ms<double>(E, T_APPLY, mp, L);
      launch_combine<double>(E, T_APPLY, EPI_M);
    }
    k_scale<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total, alpha[k]);
  }
  // G = sum over (system, shift) of the force density of (X_i, alpha_i M X_i)
  std::vector<SysDev> ft((size_t)nrhs * n);
  for (int s = 0; s < nrhs; ++s)
    for (int k = 0; k < n; ++k) {
      SysDev d = base_dev(E.sb[s]);
      d.e_in = E.sb[s].shx + (size_t)k * slot;
      d.e_out = E.sb[s].shp + (size_t)k * slot;
      ft[(size_t)s * n + k] = d;
    }
  HIPCHK(c, hipMemcpyAsync(E.ftab, ft.data(), sizeof(SysDev) * ft.size(), hipMemcpyHostToDevice,
                           E.st));
  TRY(before_gradient(E, grad_phi, xi, phi));
  k_force<<<E.sb[0].nblk, E.block, 0, E.st>>>(E.ftab, nrhs * n, E.sb[0].nblk,
                                               (double2*)grad_phi);
  TRY(read_scalars(E));
  if (!E.pl.fft) {
    int bits = 0;
    for (int s = 0; s < nrhs; ++s) bits |= sticky_bits(E, s);
    TRY(sticky_status(c, bits, "ov_rational_force, Y_i = M X_i"));
  }
  SolveOut so;
  so.outer = iters;
  so.ru.assign(nrhs, 0);
  so.res.assign(nrhs, 0.0);
  so.conv.assign(nrhs, 1);
  fill_stats(st, nrhs, &E, &so, now_s() - t0, 16);
  return OV_OK;
}

ov_status ov_rational_force(ov_ctx* c, double a0, int n, const double* alpha,
                            const double* beta, void* grad_phi, double* S_host, const void* xi,
                            const void* phi, int nrhs, ov_stats* st) {
  Range range("ov_rational_force");
  return res_retry(c, [&] {
    return rational_force_impl(c, a0, n, alpha, beta, grad_phi, S_host, xi, phi, nrhs, st);
  });
}

// ------------------------------------------------------------ RHMC (Sec. 7.3)
ov_status ov_boson(ov_ctx* c, const void* phi, double* S_host, void* G, void* F) {
  Range range("ov_boson");
  if (!c || !phi || !S_host) return OV_ERR_INVALID_ARG;
  std::string why;
  if (!fft_ok(&c->p, why)) {
    c->err = "ov_boson: " + why;
    return OV_ERR_INVALID_ARG;
  }
  Engine E;
  std::vector<ov_ctx*> v(1, c);
  TRY(engine_init(E, v, false, false, c->p.inner_tol, c->p.inner_tol));
  SysBuf& b = E.sb[0];
  E.htab.assign((size_t)E.ntab, SysDev{});
  SysDev d = base_dev(b);
  d.phi = (const double2*)phi;
  const size_t sb = (size_t)b.V * sizeof(double2);
  if (overlap(G, G ? sb : 0, phi, sb) || overlap(F, F ? sb : 0, phi, sb)) {
    // the last pass reads phi beside its results
    k_scale_copy<<<(unsigned)std::min((b.V + 255) / 256, 4096), 256, 0, E.st>>>(
        b.x64, (const double2*)phi, 1.0, (size_t)b.V);
    d.phi = b.x64;
  }
  E.shifts = false;
  d.e_out = b.r64;     // transformed planes of phi, W', conj W'
  d.fft_tmp = b.src64b;
  E.htab[T_APPLY] = d;
  TRY(upload_tables(E));
  SymIo io;
  io.in = 2;
  launch_sym<double, 3>(E, T_APPLY, SYM_BOSON, io);
  k_boson_finish<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total,
                                                    (double2*)G, (double2*)F);
  k_cg_scalar<<<1, 256, 0, E.st>>>(tab(E, T_APPLY), 1, 4);  // S_B -> BB
  TRY(read_scalars(E));
  *S_host = c->pinned[CG_BB];
  return OV_OK;
}

namespace {
// sum of |y|^2 over n complex values after y += a (x1 + x2), on the caller's stream
ov_status md_axpy(ov_ctx* c, double2* y, double a, const double2* x1, const double2* x2, int n,
                  double* part, double* norm2) {
  const int nb = (n + 255) / 256;
  k_md_axpy<<<nb, 256, 0, c->stream>>>(y, a, x1, x2, n, norm2 ? part : nullptr);
  TRY(check_launch(c));
  if (norm2) {
    std::vector<double> h(nb);
    HIPCHK(c, hipMemcpyAsync(h.data(), part, sizeof(double) * nb, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    double acc = 0;
    for (double v : h) acc += v;
    *norm2 = acc;
  }
  return OV_OK;
}
}  // namespace

ov_status ov_rhmc_trajectory(ov_ctx* c, void* phi, const void* pi0, const void* R, int nsteps,
                             double tau, double a18, int n18, const double* al18,
                             const double* be18, double a14, int n14, const double* al14,
                             const double* be14, double u, double* dH, int* accepted,
                             ov_stats* st) {
  Range range("ov_rhmc_trajectory");
  if (!c || !phi || !pi0 || !R || nsteps < 1 || !(tau > 0) || !al18 || !be18 || !al14 ||
      !be14 || !dH || !accepted)
    return OV_ERR_INVALID_ARG;
  const double t0 = now_s();
  const int V = c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3];
  const size_t sb = (size_t)V * sizeof(double2);
  // trajectory state: eta (4V), phi and pi working copies, G_B, G_F, partial sums
  char* buf = nullptr;
  const size_t nbytes = 8 * sb + sizeof(double) * ((V + 255) / 256 + 64);
  HIPCHK(c, hipMalloc((void**)&buf, nbytes));
  struct Free {
    char* p;
    ~Free() { if (p) (void)hipFree(p); }
  } guard{buf};
  double2* eta = (double2*)buf;
  double2* ph = (double2*)(buf + 4 * sb);
  double2* pi = ph + V;
  double2* Gb = pi + V;
  double2* Gf = Gb + V;
  double* part = (double*)(Gf + V);
  HIPCHK(c, hipMemcpyAsync(ph, phi, sb, hipMemcpyDeviceToDevice, c->stream));
  HIPCHK(c, hipMemcpyAsync(pi, pi0, sb, hipMemcpyDeviceToDevice, c->stream));
  // heatbath eta = r18(MdagM) R
  TRY(ov_rational(c, a18, n18, al18, be18, eta, R, phi, 1, nullptr));
  const double eps = tau / nsteps;
  double Sb = 0, Sf = 0, p2 = 0;
  auto forces = [&]() -> ov_status {
    TRY(ov_boson(c, ph, &Sb, Gb, nullptr));
    TRY(ov_rational_force(c, a14, n14, al14, be14, Gf, &Sf, eta, ph, 1, nullptr));
    return OV_OK;
  };
  TRY(forces());
  TRY(md_axpy(c, pi, 0.0, nullptr, nullptr, V, part, &p2));
  const double H0 = 0.5 * p2 + Sb + Sf;
  for (int k = 0; k < nsteps; ++k) {
    TRY(md_axpy(c, pi, -0.5 * eps, Gb, Gf, V, part, nullptr));
    TRY(md_axpy(c, ph, eps, pi, nullptr, V, part, nullptr));
    TRY(forces());
    TRY(md_axpy(c, pi, -0.5 * eps, Gb, Gf, V, part, k + 1 == nsteps ? &p2 : nullptr));
  }
  const double H1 = 0.5 * p2 + Sb + Sf;
  *dH = H1 - H0;
  *accepted = (u < std::exp(-*dH)) ? 1 : 0;
  if (*accepted) HIPCHK(c, hipMemcpyAsync(phi, ph, sb, hipMemcpyDeviceToDevice, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  if (st) {
    std::memset(st, 0, sizeof(*st));
    st->outer_iters = nsteps;
    st->seconds = now_s() - t0;
  }
  return OV_OK;
}

static ov_status locality_impl(ov_ctx* c, int spin, double* f, int nr, ov_stats* st) {
  if (!c || !f || spin < 0 || spin > 3) return OV_ERR_INVALID_ARG;
  const int* d = c->p.dims;
  const int rmax = d[0] / 2 + d[1] / 2 + d[2] / 2 + d[3] / 2;
  if (nr < rmax + 1) {
    c->err = "ov_locality: nr must be at least sum_mu L_mu/2 + 1";
    return OV_ERR_INVALID_ARG;
  }
  const double t0 = now_s();
  Engine E;
  std::vector<ov_ctx*> v(1, c);
  TRY(engine_init(E, v, false, false, c->p.inner_tol, c->p.inner_tol));
  TRY(reset_stats(E));
  TRY(run_apply(E, OV_OP_DOV, nullptr, false, false));  // e_in = x64, result in r64
  SysBuf& b = E.sb[0];
  const size_t V = b.V;
  // unit point source at the origin: x64 = 0, plane `spin` of site 0 = 1
  zero_dev(E, b.x64, V * 4 * sizeof(double2));
  static const double2 one = {1.0, 0.0};
  HIPCHK(c, hipMemcpyAsync(b.x64 + (size_t)spin * V, &one, sizeof(double2),
                           hipMemcpyHostToDevice, E.st));
  TRY(apply_sequence(E, OV_OP_DOV, false));
  // norms of r64 into u64 (as doubles), then one workgroup per distance into basis64
  SysDev dn = E.htab[T_APPLY];
  dn.e_in = b.r64;
  E.htab[T_APPLY2] = dn;
  TRY(upload_tables(E));
  double* norm = (double*)b.u64;
  double* fd = (double*)b.basis64;
  k_site_norm<<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY2), E.bmap, E.nb_total, norm);
  k_shell_max<<<rmax + 1, 256, 0, E.st>>>(dn.g, norm, fd);
  TRY(check_launch(c));
  std::vector<double> h(rmax + 1);
  HIPCHK(c, hipMemcpyAsync(h.data(), fd, sizeof(double) * h.size(), hipMemcpyDeviceToHost, E.st));
  TRY(read_scalars(E));
  for (int r = 0; r < nr; ++r) f[r] = r <= rmax ? h[r] : 0.0;
  fill_stats(st, 1, &E, nullptr, now_s() - t0, 16);
  if (sys_ctl(E, 0).bits & (1 << 2)) {
    c->err = "multi-shift did not converge within its basis";
    return OV_ERR_NOT_CONVERGED;
  }
  return OV_OK;
}

ov_status ov_locality(ov_ctx* c, int spin, double* f, int nr, ov_stats* st) {
  Range range("ov_locality");
  return res_retry(c, [&] {
    return locality_impl(c, spin, f, nr, st);
  });
}

ov_status ov_pack(ov_ctx* c, int prec, void* dst, const void* src, int nrhs) {
  if (!c || !dst || !src || nrhs < 1 || (prec != 0 && prec != 1)) return OV_ERR_INVALID_ARG;
  Engine E;
  std::vector<ov_ctx*> v(nrhs, c);
  TRY(engine_init(E, v, false, false, c->p.inner_tol, c->p.inner_tol));
  E.htab.assign((size_t)E.ntab * nrhs, SysDev{});
  for (int s = 0; s < nrhs; ++s) E.htab[(size_t)T_APPLY * nrhs + s] = base_dev(E.sb[s]);
  const size_t V = E.sb[0].V;
  E.io.resize(nrhs);
  for (int r = 0; r < nrhs; ++r)
    E.io[r] = {(const char*)src + r * V * 4 * sizeof(double2),
               (char*)dst + r * V * 4 * (prec ? sizeof(float2) : sizeof(double2)), nullptr, nullptr};
  TRY(upload_tables(E));
  if (prec)
    k_pack<float><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  else
    k_pack<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  return sync(E);
}

ov_status ov_unpack(ov_ctx* c, int prec, void* dst, const void* src, int nrhs) {
  if (!c || !dst || !src || nrhs < 1 || (prec != 0 && prec != 1)) return OV_ERR_INVALID_ARG;
  Engine E;
  std::vector<ov_ctx*> v(nrhs, c);
  TRY(engine_init(E, v, false, false, c->p.inner_tol, c->p.inner_tol));
  E.htab.assign((size_t)E.ntab * nrhs, SysDev{});
  for (int s = 0; s < nrhs; ++s) E.htab[(size_t)T_APPLY * nrhs + s] = base_dev(E.sb[s]);
  const size_t V = E.sb[0].V;
  E.io.resize(nrhs);
  for (int r = 0; r < nrhs; ++r)
    E.io[r] = {nullptr, nullptr,
               (char*)const_cast<void*>(src) + r * V * 4 * (prec ? sizeof(float2) : sizeof(double2)),
               (char*)dst + r * V * 4 * sizeof(double2)};
  TRY(upload_tables(E));
  if (prec)
    k_unpack<float><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  else
    k_unpack<double><<<E.nb_total, E.block, 0, E.st>>>(tab(E, T_APPLY), E.bmap, E.nb_total);
  return sync(E);
}

ov_status ov_tune_ms(ov_ctx* c, int prec, int nrhs, int block, int spt, int iters, float* us) {
  if (!c || !us || nrhs < 1 || iters < 1 || (prec != 0 && prec != 1) || block < 64 ||
      block > 256 || (block & 63) || spt < 1 || spt > 16)
    return OV_ERR_INVALID_ARG;
  const int ob = c->block, os = c->spt;
  c->block = block;
  c->spt = spt;
  const ov_status st = prec ? tune_run<float>(c, nrhs, iters, us) : tune_run<double>(c, nrhs, iters, us);
  c->block = ob;
  c->spt = os;
  return st;
}

ov_status ov_kernel_sampling(ov_ctx* c, int max_per_call) {
  if (!c || max_per_call < 0) return OV_ERR_INVALID_ARG;
  c->sample_max = max_per_call;
  return OV_OK;
}

ov_status ov_kernel_times(ov_ctx* c, int k, double* total_ms, long long* count, double* bytes,
                          double* kernel_ms, long long* kernel_count, int reset) {
  if (!c || k < 0 || k > 4) return OV_ERR_INVALID_ARG;
  if (total_ms) *total_ms = c->ksum_ms[k];
  if (count) *count = c->kcount[k];
  if (bytes) *bytes = c->ksum_bytes[k];
  if (kernel_ms) *kernel_ms = c->ksum_kernel_ms[k];
  if (kernel_count) *kernel_count = c->kcount_kernel[k];
  if (reset) {
    c->ksum_ms[k] = 0;
    c->ksum_bytes[k] = 0;
    c->kcount[k] = 0;
    c->ksum_kernel_ms[k] = 0;
    c->kcount_kernel[k] = 0;
  }
  return OV_OK;
}

ov_status ov_stencil_bench(ov_ctx* c, int prec, void* out, const void* in, int nrhs, int reps,
                           float* ms_per_launch) {
  if (!c || !out || !in || nrhs < 1 || reps < 1 || (prec != 0 && prec != 1))
    return OV_ERR_INVALID_ARG;
  Engine E;
  std::vector<ov_ctx*> v(nrhs, c);
  std::vector<int> hbmap;
  // only tables / partials are needed: a tiny plan
  E.ctxs = v;
  E.nsys = nrhs;
  E.sb.assign(nrhs, SysBuf{});
  E.lead = c;
  E.st = c->priv;
  HIPCHK(c, hipEventRecord(c->ev_in, c->stream));
  HIPCHK(c, hipStreamWaitEvent(E.st, c->ev_in, 0));
  E.pl.cap64 = 1;
  E.pl.capR = 0;
  E.pl.solve = false;
  // carve without the big vectors: use a dedicated small layout
  {
    Bump dry(nullptr, 0, true);
    int blk = 0;
    for (int s = 0; s < nrhs; ++s) {
      SysBuf& b = E.sb[s];
      b.ctx = c;
      b.V = c->p.dims[0] * c->p.dims[1] * c->p.dims[2] * c->p.dims[3];
      b.spb = sites_per_block(c, c->block, b.V, (long long)b.V * nrhs);
      b.nblk = (b.V + b.spb - 1) / b.spb;
      b.blk0 = blk;
      blk += b.nblk;
      b.part_c = (double*)dry.take(sizeof(double) * b.nblk);
    }
    E.nb_total = blk;
    dry.take(sizeof(SysDev) * nrhs);
    dry.take(sizeof(int) * (size_t)blk);
    void* base = nullptr;
    TRY(ensure_ws(c, dry.off + 1024, &base));
    Bump bp(base, dry.off + 1024, false);
    for (int s = 0; s < nrhs; ++s) E.sb[s].part_c = (double*)bp.take(sizeof(double) * E.sb[s].nblk);
    E.tables = (SysDev*)bp.take(sizeof(SysDev) * nrhs);
    E.bmap = (int*)bp.take(sizeof(int) * (size_t)blk);
    hbmap.assign(blk, 0);
    for (int s = 0; s < nrhs; ++s)
      for (int b = 0; b < E.sb[s].nblk; ++b) hbmap[E.sb[s].blk0 + b] = s;
  }
  const size_t V = E.sb[0].V;
  const size_t es = prec ? sizeof(float2) : sizeof(double2);
  E.htab.assign(nrhs, SysDev{});
  for (int s = 0; s < nrhs; ++s) {
    SysDev d = base_dev(E.sb[s]);
    d.e_in = (const char*)in + s * V * 4 * es;
    d.e_out = (char*)out + s * V * 4 * es;
    E.htab[s] = d;
  }
  HIPCHK(c, hipMemcpyAsync(E.tables, E.htab.data(), sizeof(SysDev) * nrhs, hipMemcpyHostToDevice,
                           E.st));
  HIPCHK(c, hipMemcpyAsync(E.bmap, hbmap.data(), sizeof(int) * hbmap.size(),
                           hipMemcpyHostToDevice, E.st));
  HIPCHK(c, hipStreamSynchronize(E.st));
  hipEvent_t e0, e1;
  HIPCHK(c, hipEventCreate(&e0));
  HIPCHK(c, hipEventCreate(&e1));
  const double diag = 4.0 - c->p.M0;
  // Stencil form: z-marching (xy plane in LDS, z neighbours in registers) where
  // the plane fits a workgroup, else the LDS-staged block form; OV_HW_LDS=0
  // selects the plain form, OV_HW_LDS=1 the block form (measurement switches).
  const int spb = E.sb[0].spb;
  const size_t lds_bytes = (size_t)4 * spb * (prec ? sizeof(float2) : sizeof(double2));
  const char* ev = std::getenv("OV_HW_LDS");
  const int* dm = c->p.dims;
  const int zc = (dm[2] % 4 == 0) ? 4 : (dm[2] % 2 == 0 ? 2 : 1);
  const int nzm = nrhs * dm[3] * (dm[2] / zc);
  // z-marching needs enough workgroups (one per xy plane and z chunk) to fill the chip
  const bool use_zm = !(ev && (*ev == '0' || *ev == '1')) && dm[0] * dm[1] <= 256 && zc >= 2 &&
                      nzm >= 512;
  const bool use_lds = !use_zm && !(ev && *ev == '0') && lds_bytes <= 64 * 1024;
  HIPCHK(c, hipEventRecord(e0, E.st));
  for (int r = 0; r < reps; ++r) {
    if (use_zm) {
      if (prec)
        zc == 4 ? k_hw_zm<float, 4><<<nzm, 256, 0, E.st>>>(E.tables, diag)
                : k_hw_zm<float, 2><<<nzm, 256, 0, E.st>>>(E.tables, diag);
      else
        zc == 4 ? k_hw_zm<double, 4><<<nzm, 256, 0, E.st>>>(E.tables, diag)
                : k_hw_zm<double, 2><<<nzm, 256, 0, E.st>>>(E.tables, diag);
    } else if (use_lds) {
      if (prec)
        k_hw_lds<float><<<E.nb_total, c->block, lds_bytes, E.st>>>(E.tables, E.bmap, E.nb_total, diag);
      else
        k_hw_lds<double><<<E.nb_total, c->block, lds_bytes, E.st>>>(E.tables, E.bmap, E.nb_total, diag);
    } else if (prec) {
      k_hw<float><<<E.nb_total, c->block, 0, E.st>>>(E.tables, E.bmap, E.nb_total, diag, 0);
    } else {
      k_hw<double><<<E.nb_total, c->block, 0, E.st>>>(E.tables, E.bmap, E.nb_total, diag, 0);
    }
  }
  HIPCHK(c, hipEventRecord(e1, E.st));
  TRY(check_launch(c));
  HIPCHK(c, hipEventSynchronize(e1));
  float ms = 0;
  HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (ms_per_launch) *ms_per_launch = ms / reps;
  return OV_OK;
}

}  // extern "C"
