// Per-antenna planes: a_ps = e_ps K_ps (and, WITH_K3, the beam-gradient factor)
// of a range of sources, once per (timestep, channel, source, antenna), for the
// staging of rime_main.
#include "rime_device.h"

namespace rime {

// ---------------------------------------------------------------------------
// Planes: thread = (source, antenna) of one timestep and one block of
// p.phase_nc channels; the phase argument and the beam radius are formed once
// per block.  Bound by its stores (500 sources x 64 antennas x 6400
// (timestep, channel): 0.52 ms, 3.2 TB/s; with k3 0.66 ms, 3.7 TB/s).
// ---------------------------------------------------------------------------
template <bool WITH_K3>
__global__ __launch_bounds__(256) void plane_phase(const KParams p) {
  const int tt = blockIdx.y;
  const int t = p.pme_t0 + tt;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t plane = static_cast<int64_t>(p.pl_ns) * p.nap;
  if (idx >= plane) return;
  const int cb = blockIdx.z * p.phase_nc;
  const int ce = min(p.nchan, cb + p.phase_nc);
  const int s = static_cast<int>(idx / p.nap);
  const int a = static_cast<int>(idx - static_cast<int64_t>(s) * p.nap);
  if (a >= p.na) return;  // padding, never read
  const int64_t at = static_cast<int64_t>(tt) * p.nchan * plane + idx;
  float2 *pa = p.pl_a + at;
  float *pk = p.pl_k3 + at;
  const double4 g = p.src_geo[p.one.src_off + p.pl_s0 + s];
  const double *x = p.uvw + (static_cast<int64_t>(t) * p.na + a) * 3;
  const PhaseArg<false> tau(x[0], x[1], x[2], g.x, g.y, g.z);
  double r2b = 0.0, rb = 0.0;
  if (p.beam) {
    const double *q = p.pointing + (static_cast<int64_t>(t) * p.na + a) * 2;
    r2b = sumsq_rn(g.x - q[0], g.y - q[1]);
    rb = sqrt(r2b);
  }
  for (int c = cb; c < ce; ++c) {
    float2 v;
    float k3;
    antenna_term<float, WITH_K3>(p, tau, r2b, rb, c, v, k3);
    pa[c * plane] = v;
    if (WITH_K3) pk[c * plane] = k3;
  }
}

// Timesteps [p.pme_t0, p.pme_t0 + p.pme_nt).  Channels per workgroup by the
// rule of the fp16 engine's phase planes (planes of 1 MiB and more write
// fastest in blocks of 4 channels, smaller ones in blocks of 16).
hipError_t launch_planes(const KParams &p, hipStream_t stream) {
  const int64_t plane = static_cast<int64_t>(p.pl_ns) * p.nap;
  KParams q = p;
  q.phase_nc = plane * static_cast<int64_t>(sizeof(float2)) >= (int64_t(1) << 20) ? 4 : 16;
  const dim3 g(static_cast<unsigned>((plane + 255) / 256), static_cast<unsigned>(p.pme_nt),
               static_cast<unsigned>((p.nchan + q.phase_nc - 1) / q.phase_nc));
  if (p.pl_k3)
    hipLaunchKernelGGL(plane_phase<true>, g, dim3(256), 0, stream, q);
  else
    hipLaunchKernelGGL(plane_phase<false>, g, dim3(256), 0, stream, q);
  return hipGetLastError();
}

}  // namespace rime
