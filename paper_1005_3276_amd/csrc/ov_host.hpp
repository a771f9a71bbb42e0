// ov_host.hpp -- host-only functions of libov.so (ov_host.cpp, ov_zolotarev.cpp).
#pragma once
#include <string>

#include "../../include/ov.h"

namespace ov {

constexpr int HOST_MAXP = 32;  // poles (the kernels' MAXP)

// Worst-case CG iterations on H_W^2 (spectrum [smin^2, smax^2]) for the shifted
// residuals to reach tol (Chebyshev bound).
int cg_bound(double smin, double smax, double tol);
// The momentum-space kernels' lattice limits; why receives the reason when false.
bool fft_ok(const ov_params* p, std::string& why);
// OV_OK or OV_ERR_INVALID_ARG with the reason in err.
ov_status validate(const ov_params* p, std::string& err);
// Range of the free |H_W| over the lattice momenta (antiperiodic time: p_t = (2n+1) pi/T).
void free_spectrum(const ov_params* p, double& smin, double& smax);
// Zolotarev coefficients of sign(x) ~ x sum_k a_k/(x^2 + b_k) on [lmin, lmax]; 0 on success.
int zolotarev_coeffs(int n, double lmin, double lmax, double* a, double* b, double* delta);

// Block decomposition of one lattice for the resident multi-shift kernel (k_ms_res): one
// workgroup per block of b[0] b[1] b[2] b[3] sites, all G of them resident at once.
struct ResGeom {
  int G = 0;               // workgroups (0: the lattice does not fit)
  int b[4], nb[4];         // block extents, blocks per axis
  int S = 0;               // sites per block
  int FT = 0;              // complex values of one workgroup's faces of one field
  int threads = 0, K = 0;  // workgroup size, sites per thread
  double us = 0;           // modelled time of one pass
};
constexpr int RES_MAX_THREADS = 960;     // compute threads: 15 waves and the service wave
constexpr int RES_MAX_LDS = 144 * 1024;  // the block's field; the rest of 160 KiB is spare
// The decomposition of the least modelled pass time for complex values of esize bytes (16
// FP64, 8 FP32) on ncu compute units with at most maxK sites per thread.
ResGeom res_geom(const int dims[4], int esize, int ncu, int maxK);

}  // namespace ov
