// HIP kernel (gfx950) of the detector inputs of the demodulation: detector
// position and velocity per SFT from a circular-orbit and rotating-Earth
// model, and the antenna-pattern factors a, b per (sky, SFT) as the plus and
// cross projections of the detector tensor on the wave frame.  All FP64
// (hardware sin/cos of arguments below 1e4 rad), a and b stored as FP32.
#include "fstat_internal.h"

namespace fstat {

// Sky points of a block at most; with few SFTs (up to kFewSfts) kSkyChunkFew.
constexpr int kSkyChunk = 64;
constexpr int kSkyChunkFew = 256;
constexpr int kFewSfts = 128;

// A block takes 256 SFTs, one per thread, at up to kSkyChunk sky points; of
// few SFTs, the lanes of the next power of two take every (256 / lanes)-th of
// its sky points (1 SFT x 1e6 points 66 us with one lane busy, so 14).  Each
// thread forms r, v (sum of the orbital and the diurnal parts; written by the
// first chunk's blocks) and the six unique components of its detector tensor
// D = (u u^T - w w^T) / 2; the first threads form, per sky point, the wave
// frame X, Y and from it the coefficients of a = X^T D X - Y^T D Y and
// b = 2 X^T D Y as linear forms in D's components.  A pair then costs twelve
// FP64 FMAs and its 8 bytes of output, which bound the kernel: 2000 SFTs x
// 2000 points (32 MB) in 28 us as two kernels that rebuilt the frame (two
// square roots, two divisions) per pair and passed the tensors through memory.
// The wave frame of n = (cos d cos al, cos d sin al, sin d) is formed from the
// components directly: with rho = sqrt(nx^2 + ny^2), X = (ny, -nx, 0) / rho,
// Y = (-nz nx / rho, -nz ny / rho, rho); at the poles (rho = 0) al = 0.
template <bool FEW>
__global__ __launch_bounds__(256) void detector_kernel(EarthModel m, int64_t n_sft, const double* t_mid,
                                                       const int32_t* site_of_sft, int64_t n_sky, const double* sky,
                                                       int chunk, int lg_lanes, double* pos, double* vel, float* a,
                                                       float* b) {
  __shared__ double form[FEW ? kSkyChunkFew : kSkyChunk][12];
  const int64_t n_sb = FEW ? 1 : (n_sft + 255) / 256;
  const int64_t sb = blockIdx.x % n_sb, kb = blockIdx.x / n_sb;
  const int64_t s0 = kb * chunk;
  const int ns = (int)(n_sky - s0 < chunk ? n_sky - s0 : chunk);
  const int tid = threadIdx.x;
  if (tid < ns) {
    const double* n = sky + 3 * (s0 + tid);
    const double nx = n[0], ny = n[1];
    const double nz = n[2] > 1.0 ? 1.0 : (n[2] < -1.0 ? -1.0 : n[2]);
    const double rho = sqrt(nx * nx + ny * ny);
    double X[3] = {0.0, -1.0, 0.0}, Y[3] = {-nz, 0.0, 0.0};
    if (rho > 0.0) {
      const double ca = nx / rho, sa = ny / rho;
      const double cd = sqrt(1.0 - nz * nz);       // cos of the declination from sin d = nz
      X[0] = sa; X[1] = -ca;
      Y[0] = -nz * ca; Y[1] = -nz * sa; Y[2] = cd;
    }
    double* f = form[tid];                         // components xx, yy, zz, xy, xz, yz
    const int p[6] = {0, 1, 2, 0, 0, 1}, q[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const double k = c < 3 ? 1.0 : 2.0;
      f[c] = k * (X[p[c]] * X[q[c]] - Y[p[c]] * Y[q[c]]);
      f[6 + c] = c < 3 ? 2.0 * (X[p[c]] * Y[q[c]]) : 2.0 * (X[p[c]] * Y[q[c]] + X[q[c]] * Y[p[c]]);
    }
  }
  const int lane = FEW ? tid & ((1 << lg_lanes) - 1) : tid, group = FEW ? tid >> lg_lanes : 0;
  const int groups = FEW ? 256 >> lg_lanes : 1;
  const int64_t al = sb * 256 + lane;
  const bool live = al < n_sft;
  double d[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (live) {
    const int si = site_of_sft[al];
    const bool known = si >= 0 && si < m.n_sites;
    const SiteModel st = m.sites[known ? si : 0];
    const double dt = t_mid[al] - m.t0;
    double sp, cp, sth, cth;
    sincos(m.orbit_phase + m.orbit_rate * dt, &sp, &cp);
    sincos(st.lon + m.sidereal_phase + m.sidereal_rate * dt, &sth, &cth);
    if (kb == 0 && group == 0) {
      const double nan = __builtin_nan("");
      const double R = m.orbit_radius, RW = m.orbit_radius * m.orbit_rate;
      const double Re = m.earth_radius, ReW = m.earth_radius * m.sidereal_rate;
      pos[3 * al + 0] = known ? R * cp + Re * st.cla * cth : nan;
      pos[3 * al + 1] = known ? R * sp * m.ce + Re * st.cla * sth : nan;
      pos[3 * al + 2] = known ? R * sp * m.se + Re * st.sla : nan;
      vel[3 * al + 0] = known ? -RW * sp - ReW * st.cla * sth : nan;
      vel[3 * al + 1] = known ? RW * cp * m.ce + ReW * st.cla * cth : nan;
      vel[3 * al + 2] = known ? RW * cp * m.se : nan;
    }
    // local east and north, then the arms
    const double e[3] = {-sth, cth, 0.0};
    const double nn[3] = {-st.sla * cth, -st.sla * sth, st.cla};
    double u[3], w[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      u[c] = st.cx * nn[c] + st.sx * e[c];
      w[c] = st.cy * nn[c] + st.sy * e[c];
    }
    d[0] = 0.5 * (u[0] * u[0] - w[0] * w[0]);
    d[1] = 0.5 * (u[1] * u[1] - w[1] * w[1]);
    d[2] = 0.5 * (u[2] * u[2] - w[2] * w[2]);
    d[3] = 0.5 * (u[0] * u[1] - w[0] * w[1]);
    d[4] = 0.5 * (u[0] * u[2] - w[0] * w[2]);
    d[5] = 0.5 * (u[1] * u[2] - w[1] * w[2]);
    if (!known) d[0] = __builtin_nan("");
  }
  __syncthreads();
  if (!live) return;
  for (int s = group; s < ns; s += groups) {
    const double* f = form[s];
    double x = d[0] * f[0], y = d[0] * f[6];
#pragma unroll
    for (int c = 1; c < 6; ++c) {
      x = __builtin_fma(d[c], f[c], x);
      y = __builtin_fma(d[c], f[6 + c], y);
    }
    a[(s0 + s) * n_sft + al] = (float)x;
    b[(s0 + s) * n_sft + al] = (float)y;
  }
}

hipError_t launch_detector_inputs(const EarthModel& m, int64_t n_sft, const double* t_mid, const int32_t* site_of_sft,
                                  int64_t n_sky, const double* sky, double* pos, double* vel, float* a, float* b,
                                  hipStream_t st) {
  if (n_sft <= 0 || n_sky <= 0) return hipErrorInvalidValue;
  // sky points per block: enough blocks to fill the device first (about four
  // per CU), then as many points per block as share its tensors
  const int64_t n_sb = (n_sft + 255) / 256;
  const bool few = n_sft <= kFewSfts;
  const int64_t most = few ? kSkyChunkFew : kSkyChunk;
  int64_t chunk = (n_sky * n_sb + 1023) / 1024;
  chunk = chunk < 1 ? 1 : (chunk > most ? most : chunk);
  int lg_lanes = 8;
  if (few) {
    for (lg_lanes = 0; (1 << lg_lanes) < n_sft; ++lg_lanes) {
    }
    const int64_t groups = 256 >> lg_lanes;        // every group of lanes has a sky point
    chunk = (chunk + groups - 1) / groups * groups;
  }
  const int64_t blocks = n_sb * ((n_sky + chunk - 1) / chunk);
  if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(few ? detector_kernel<true> : detector_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, m,
                     n_sft, t_mid, site_of_sft, n_sky, sky, (int)chunk, lg_lanes, pos, vel, a, b);
  return hipGetLastError();
}

}  // namespace fstat
