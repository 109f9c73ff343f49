// Velocity Verlet (constant N, V, E) around the energy+force path: the MD
// step the method is used in (Sec. 4, MD proxy application with energy
// conservation checks).  Per step, with a = F / m:
//   v <- v + (dt/2) a(t);  x <- x + dt v;  F <- F(x);  v <- v + (dt/2) a(t + dt).
// Units: A, fs, eV, amu; accel_conv turns eV/(A amu) into A/fs^2 and
// ke_conv turns amu A^2/fs^2 into eV.  Updates are done in FP64 and rounded
// once to the positions' type; positions are wrapped back into [0, L).
#include <algorithm>

#include "kernels.h"

namespace nnp {
namespace {

constexpr int MD_THREADS = 256, MD_BLOCKS = 1024;

__device__ inline int clamp_type(int t) { return t < 0 ? 0 : (t >= MAX_EL ? MAX_EL - 1 : t); }

// The kinetic energy of a step from its per-block partial sums, in block order.
__device__ inline void ke_total(const double* partial, int nb, double conv, double* out) {
  __shared__ double all[MD_BLOCKS];
  for (int b = threadIdx.x; b < nb; b += MD_THREADS) all[b] = partial[b];
  __syncthreads();
  if (threadIdx.x != 0) return;
  double s = 0.0;
  for (int b = 0; b < nb; ++b) s += all[b];
  *out = s * conv;
}

// All that lies between two evaluations of the forces: the second half-kick of a
// step (kick), its kinetic energy as one FP64 partial sum per block, and the first
// half-kick and the drift of the next one (drift).  One launch, where the two
// half-kicks and the sum of the partials were one each (a step of 12,288 atoms has
// some 15 launches of about 4.5 us beside the pair passes): the velocity between
// the half-kicks is rounded to its type as it was when it was stored.  The first
// workgroup also adds up the partials of the step before (prev) and clears the
// flags[0..3] of the neighbour list.
template <class IO>
__global__ void __launch_bounds__(MD_THREADS) k_md_step(int64_t n, IO* pos, IO* vel, const IO* F, const int32_t* types,
                                                        MdArgs m, int kick, int drift, double* partial,
                                                        const double* prev, double* ke_prev, int* flags) {
  __shared__ double red[MD_THREADS];
  if (blockIdx.x == 0) {
    if (threadIdx.x < 4) flags[threadIdx.x] = 0;
    if (prev) ke_total(prev, gridDim.x, m.ke_conv, ke_prev);
  }
  const int64_t stride = (int64_t)gridDim.x * MD_THREADS;
  double ke = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * MD_THREADS + threadIdx.x; i < n; i += stride) {
    const int t = clamp_type(types[i]);
    const double h = m.half_kick[t], h2 = kick ? h : 0.0;
    double v2 = 0.0;
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      const double f = (double)F[3 * i + x];
      const IO vr = (IO)((double)vel[3 * i + x] + h2 * f);
      v2 += (double)vr * (double)vr;
      if (drift) {
        const double v = (double)vr + h * f;
        double p = (double)pos[3 * i + x] + m.dt * v;
        p -= m.L[x] * floor(p * m.invL[x]);
        vel[3 * i + x] = (IO)v;
        pos[3 * i + x] = (IO)p;
      } else if (kick) {
        vel[3 * i + x] = vr;
      }
    }
    ke += m.half_mass[t] * v2;
  }
  red[threadIdx.x] = ke;
  __syncthreads();
  for (int s = MD_THREADS / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(MD_THREADS) k_ke_total(const double* partial, int nb, double conv, double* out) {
  ke_total(partial, nb, conv, out);
}

}  // namespace

int md_blocks(int64_t n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((n + MD_THREADS - 1) / MD_THREADS, MD_BLOCKS));
}

template <class IO>
void launch_md_step(int64_t n, IO* pos, IO* vel, const IO* F, const int32_t* types, const MdArgs& m, bool kick, bool drift,
                    double* partial, const double* prev, double* ke_prev, int* flags, hipStream_t stream) {
  hipLaunchKernelGGL(k_md_step<IO>, dim3(md_blocks(n)), dim3(MD_THREADS), 0, stream, n, pos, vel, F, types, m,
                     kick ? 1 : 0, drift ? 1 : 0, partial, prev, ke_prev, flags);
}

void launch_ke_total(int64_t n, const double* partial, const MdArgs& m, double* out, hipStream_t stream) {
  hipLaunchKernelGGL(k_ke_total, dim3(1), dim3(MD_THREADS), 0, stream, partial, md_blocks(n), m.ke_conv, out);
}

template void launch_md_step<float>(int64_t, float*, float*, const float*, const int32_t*, const MdArgs&, bool, bool,
                                    double*, const double*, double*, int*, hipStream_t);
template void launch_md_step<double>(int64_t, double*, double*, const double*, const int32_t*, const MdArgs&, bool, bool,
                                     double*, const double*, double*, int*, hipStream_t);

}  // namespace nnp
