// Fills, (un)permutation to the caller's atom order and the deterministic
// FP64 energy sums E_b = sum_i E_i (Fig. 1(b), the E_system loop).
#include "kernels.h"

namespace nnp {

template <class T>
__global__ void __launch_bounds__(256) k_fill(T* __restrict__ p, int64_t n, T v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

template <class T>
void launch_fill(T* p, int64_t n, T v, hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n, v);
}
template void launch_fill<float>(float*, int64_t, float, hipStream_t);
template void launch_fill<double>(double*, int64_t, double, hipStream_t);
template void launch_fill<int>(int*, int64_t, int, hipStream_t);

void launch_fill_int(int* p, int64_t n, int v, hipStream_t stream) { launch_fill<int>(p, n, v, stream); }

template <class IO, class FAcc>
__global__ void __launch_bounds__(256) k_unpermute(int64_t n, const int* __restrict__ perm, const IO* __restrict__ Ei_s,
                                                   const FAcc* __restrict__ F_s, double* __restrict__ Ei_o,
                                                   IO* __restrict__ Ei_out, IO* __restrict__ F_out, Gate gate) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n || gate_closed(gate)) return;
  const int64_t i = perm[s];
  const IO e = Ei_s[s];
  Ei_o[i] = (double)e;
  if (Ei_out) Ei_out[i] = e;
  if (F_out) {
    F_out[3 * i + 0] = (IO)F_s[s];  // sorted accumulator: component planes [3][n]
    F_out[3 * i + 1] = (IO)F_s[n + s];
    F_out[3 * i + 2] = (IO)F_s[2 * n + s];
  }
}

template <class IO, class FAcc>
void launch_unpermute(int64_t n, const int* perm, const IO* Ei_s, const FAcc* F_s, double* Ei_o, IO* Ei_out,
                      IO* F_out, const Gate& gate, hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_unpermute<IO, FAcc>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, n, perm, Ei_s,
                     F_s, Ei_o, Ei_out, F_out, gate);
}
template void launch_unpermute<double, double>(int64_t, const int*, const double*, const double*, double*, double*,
                                               double*, const Gate&, hipStream_t);
template void launch_unpermute<float, float>(int64_t, const int*, const float*, const float*, double*, float*, float*,
                                             const Gate&, hipStream_t);
template void launch_unpermute<float, double>(int64_t, const int*, const float*, const double*, double*, float*,
                                              float*, const Gate&, hipStream_t);

// out[s] = in[perm[s]] for rows of 3 (caller order -> sorted order).
template <class IO>
__global__ void __launch_bounds__(256) k_permute_rows3(int64_t n, const int* __restrict__ perm, const IO* __restrict__ in,
                                                       IO* __restrict__ out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int64_t i = perm[s];
  out[3 * s + 0] = in[3 * i + 0];
  out[3 * s + 1] = in[3 * i + 1];
  out[3 * s + 2] = in[3 * i + 2];
}

template <class IO>
void launch_permute_rows3(int64_t n, const int* perm, const IO* in, IO* out, hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_permute_rows3<IO>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, n, perm, in, out);
}
template void launch_permute_rows3<float>(int64_t, const int*, const float*, float*, hipStream_t);
template void launch_permute_rows3<double>(int64_t, const int*, const double*, double*, hipStream_t);

// Block tree sum of a range in a fixed order.
template <int N>
__device__ inline double block_sum(double v) {
  __shared__ double sh[N];
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int o = N / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  return sh[0];
}

// 16 values a thread: one chunk of 16,384 atoms takes as long as one of 4,096 did
// with 256 threads (6 us), and boxes of up to 16,384 atoms need no second launch.
__global__ void __launch_bounds__(1024) k_chunk_sum(const double* __restrict__ x, const int64_t* __restrict__ lo,
                                                   const int64_t* __restrict__ hi, double* __restrict__ partial,
                                                   double* __restrict__ host, Gate gate) {
  if (gate_closed(gate)) return;
  const int c = blockIdx.x;
  double s = 0.0;
  for (int64_t i = lo[c] + threadIdx.x; i < hi[c]; i += 1024) s += x[i];
  s = block_sum<1024>(s);
  if (threadIdx.x == 0) {
    partial[c] = s;
    if (host && c == 0) __hip_atomic_store(host, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__global__ void __launch_bounds__(256) k_struct_sum(const double* __restrict__ partial, const int* __restrict__ sc,
                                                    double* __restrict__ out, double* __restrict__ host, Gate gate) {
  if (gate_closed(gate)) return;
  const int b = blockIdx.x;
  double s = 0.0;
  for (int c = sc[b] + threadIdx.x; c < sc[b + 1]; c += 256) s += partial[c];
  s = block_sum<256>(s);
  if (threadIdx.x == 0) {
    out[b] = s;
    if (host && b == 0) __hip_atomic_store(host, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

template <class IO>
__global__ void __launch_bounds__(256) k_copy_inputs(int64_t n, const IO* __restrict__ pos,
                                                     const int32_t* __restrict__ types, IO* __restrict__ pos_out,
                                                     int32_t* __restrict__ types_out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 3 * n) pos_out[i] = pos[i];
  if (i < n) types_out[i] = types[i];
}

template <class IO>
void launch_copy_inputs(int64_t n, const IO* pos, const int32_t* types, IO* pos_out, int32_t* types_out,
                        hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_copy_inputs<IO>, dim3((unsigned)((3 * n + 255) / 256)), dim3(256), 0, stream, n, pos, types,
                     pos_out, types_out);
}
template void launch_copy_inputs<float>(int64_t, const float*, const int32_t*, float*, int32_t*, hipStream_t);
template void launch_copy_inputs<double>(int64_t, const double*, const int32_t*, double*, int32_t*, hipStream_t);

void launch_energy(const double* Ei_o, const int64_t* chunk_lo, const int64_t* chunk_hi, int nchunk,
                   const int* struct_chunk, int n_struct, bool one_chunk_each, double* partial, double* energies,
                   double* host, const Gate& gate, hipStream_t stream) {
  if (one_chunk_each) {  // a chunk's sum is its structure's energy
    hipLaunchKernelGGL(k_chunk_sum, dim3(nchunk), dim3(1024), 0, stream, Ei_o, chunk_lo, chunk_hi, energies, host,
                       gate);
    return;
  }
  if (nchunk > 0)
    hipLaunchKernelGGL(k_chunk_sum, dim3(nchunk), dim3(1024), 0, stream, Ei_o, chunk_lo, chunk_hi, partial, nullptr,
                       gate);
  hipLaunchKernelGGL(k_struct_sum, dim3(n_struct), dim3(256), 0, stream, partial, struct_chunk, energies, host,
                     gate);
}

}  // namespace nnp
