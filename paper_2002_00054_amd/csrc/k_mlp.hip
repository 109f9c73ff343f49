// Per-element atomic networks (Sec. 3.1 step 2, Fig. 1(c)) and their
// derivatives:
//   forward   h1 = tanh(W1 x + b1), h2 = tanh(W2 h1 + b2), E_i = w3 . h2 + b3
//             on the scaled descriptors x = G~;
//   dE/dG     c = diag(1/scale) W1^T [(1 - h1^2) o W2^T [(1 - h2^2) o w3]]
//             (the network part of step 3, counted with the forces in the
//             paper's Fig. 5);
//   weights   differentiation form: gradient of sum_i [a_i E_i - <dE_i/dx_i, t_i>]
//             with a tangent t_i per atom (forward-over-reverse).
// Sorted atoms of one element are contiguous, so every workgroup works on
// rows of a single element and reads that element's weights with uniform
// loads.
#include <algorithm>

#include "kernels.h"

namespace nnp {

// Workgroup b -> (element, first row) for tiles of `rows` rows per element.
__device__ inline bool element_tile(int b, int rows, int n_el, const int* __restrict__ eoff, int& e, int64_t& r0,
                                    int64_t& r1) {
  int acc = 0;
  for (int f = 0; f < n_el; ++f) {
    const int64_t lo = eoff[f], hi = eoff[f + 1];
    const int nt = (int)((hi - lo + rows - 1) / rows);
    if (b < acc + nt) {
      e = f;
      r0 = lo + (int64_t)(b - acc) * rows;
      r1 = hi;
      return true;
    }
    acc += nt;
  }
  return false;
}

__device__ inline float tanh_t(float x) { return tanhf(x); }
__device__ inline double tanh_t(double x) { return tanh(x); }

// ------------------------------------------------------------------ MFMA
// Network forward + input gradient on the matrix cores, one 16-atom tile per
// wave step.  Activations are kept transposed (units x atoms) and used as the
// B operand, weights as the A operand, so the accumulator layout of one layer
// is directly the B operand of the next layer: no LDS transposes.  Each lane
// carries 8 values of a 32-wide vector; slot s = 4 t + r of lane group
// g = lane / 16 stands for unit kin_acc(g, s) (accumulator order: the FP32
// 16x16 accumulators hold rows 4 g + r of tile t, the FP64 ones rows g + 4 r,
// as measured on gfx950) or for unit 8 g + s (the input rows read from G~).
// Any bijection works for the reduction as long as the A operand uses the
// same one.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <class T>
__device__ inline int kin_acc(int g, int s) {
  if constexpr (sizeof(T) == 8) return 16 * (s >> 2) + g + 4 * (s & 3);
  else return 16 * (s >> 2) + 4 * g + (s & 3);
}
__device__ inline int kin_row(int g, int s) { return 8 * g + s; }

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline f64x4 mfma4(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

template <class T> struct Acc4;
template <> struct Acc4<float> { using type = f32x4; };
template <> struct Acc4<double> { using type = f64x4; };

// y = W x for one tile with 16x16x4 MFMA (FP32 or FP64).  w(o, k) gives the
// weight of output unit o and input unit k; in_row selects the input slot map.
template <class T, class WF>
__device__ inline void layer_k4(const T (&in)[8], bool in_row, WF w, T (&out)[8]) {
  using V = typename Acc4<T>::type;
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    V acc = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int s = 0; s < 8; ++s) acc = mfma4(w(16 * t + col, in_row ? kin_row(g, s) : kin_acc<T>(g, s)), in[s], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) out[4 * t + r] = acc[r];
  }
}

// y = W x with 16x16x32 BF16 MFMA and FP32 accumulation; split = BF16x3
// (x = x_hi + x_lo, W = W_hi + W_lo, products hi*hi + hi*lo + lo*hi).
template <class WF>
__device__ inline void layer_bf16(const float (&in)[8], bool in_row, WF w, bool split, float (&out)[8]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  bf16x8 bh, bl;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const __bf16 h = (__bf16)in[s];
    bh[s] = h;
    bl[s] = (__bf16)(in[s] - (float)h);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    bf16x8 ah, al;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float x = w(16 * t + col, in_row ? kin_row(g, s) : kin_acc<float>(g, s));
      const __bf16 h = (__bf16)x;
      ah[s] = h;
      al[s] = (__bf16)(x - (float)h);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
    if (split) {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) out[4 * t + r] = acc[r];
  }
}

template <int P, class T, class WF>
__device__ inline void layer(const T (&in)[8], bool in_row, WF w, bool first, T (&out)[8]) {
  if constexpr (P == P_BF16) layer_bf16(in, in_row, w, first, out);
  else layer_k4<T>(in, in_row, w, out);
}

// flags[2] = the largest of itself and cmax[0 .. ncells); the host's copy of flags[0..3].
__device__ inline void report_flags(int* flags, const int* cmax, int ncells, int* host_flags) {
  __shared__ int red[4];
  int m = 0;
  for (int i = threadIdx.x; i < ncells; i += 256) m = max(m, cmax[i]);
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x != 0) return;
  m = max(max(flags[2], max(red[0], red[1])), max(red[2], red[3]));
  flags[2] = m;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    __hip_atomic_store(&host_flags[i], i == 2 ? m : flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Workgroups of 4 waves (and one that reports the flags), shared among the
// elements by their 16-atom tiles; the waves of an element's workgroups stride
// over its tiles, and its padded weights are staged in LDS once per workgroup.
template <int P>
__global__ void __launch_bounds__(256, 2) k_mlp_mfma(MlpArgs<P> a, int blocks) {
  using T = typename Types<P>::T;
  using IO = typename Types<P>::IO;
  __shared__ T W[NET_STRIDE];
  __shared__ T isc[HID];
  if ((int)blockIdx.x == blocks) {  // the extra workgroup (MlpArgs::host_flags)
    report_flags(a.flags, a.cmax, a.ncells, a.host_flags);
    return;
  }
  // one workgroup for each element that has atoms, the others in proportion
  const int all = (a.eoff[a.n_el] + 15) / 16 + a.n_el;
  int e = -1, b = blockIdx.x, wpe = 0;
  for (int f = 0; f < a.n_el; ++f) {
    const int nt = (a.eoff[f + 1] - a.eoff[f] + 15) / 16;
    wpe = nt > 0 ? 1 + (int)((int64_t)(blocks - a.n_el) * nt / all) : 0;
    if (b < wpe) {
      e = f;
      break;
    }
    b -= wpe;
  }
  if (e < 0) return;
  const T* __restrict__ src = a.nets + (size_t)e * NET_STRIDE;
  for (int i = threadIdx.x; i < NET_STRIDE; i += 256) W[i] = src[i];
  if (threadIdx.x < HID) isc[threadIdx.x] = threadIdx.x < MAX_SF ? (T)a.tab->inv_scale_d[e][threadIdx.x] : T(0);
  __syncthreads();
  const int64_t lo = a.eoff[e], hi = a.eoff[e + 1];
  const int64_t ntiles = (hi - lo + 15) / 16;
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const int wv = threadIdx.x >> 6;
  T b1[8], b2[8], w3[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int u = kin_acc<T>(g, s);
    b1[s] = W[OFF_B1 + u];
    b2[s] = W[OFF_B2 + u];
    w3[s] = W[OFF_W3 + u];
  }
  const T b3 = W[OFF_B3];
  auto W1 = [&](int o, int k) { return W[OFF_W1 + o * HID + k]; };
  auto W2 = [&](int o, int k) { return W[OFF_W2 + o * HID + k]; };
  auto W2t = [&](int o, int k) { return W[OFF_W2 + k * HID + o]; };
  auto W1t = [&](int o, int k) { return W[OFF_W1 + k * HID + o]; };
  for (int64_t tile = (int64_t)b * 4 + wv; tile < ntiles; tile += (int64_t)wpe * 4) {
    const int64_t atom = lo + tile * 16 + col;
    const bool valid = atom < hi;
    T x[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) x[s] = valid ? (T)a.G[atom * LD + kin_row(g, s)] : T(0);
    T h1[8], h2[8], d[8], y[8];
    layer<P>(x, true, W1, true, y);
#pragma unroll
    for (int s = 0; s < 8; ++s) h1[s] = tanh_t(y[s] + b1[s]);
    layer<P>(h1, false, W2, false, y);
    T pe = T(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      h2[s] = tanh_t(y[s] + b2[s]);
      pe += w3[s] * h2[s];
      d[s] = w3[s] * (T(1) - h2[s] * h2[s]);
    }
    pe += __shfl_xor(pe, 16, 64);
    pe += __shfl_xor(pe, 32, 64);
    if (g == 0 && valid) a.Ei[atom] = (IO)(pe + b3);
    // the force pass's accumulator, cleared here (one launch fewer per call)
    if (g < 3 && valid) a.F[g * a.n + atom] = typename Types<P>::FAcc(0);
    layer<P>(d, false, W2t, false, y);
#pragma unroll
    for (int s = 0; s < 8; ++s) d[s] = y[s] * (T(1) - h1[s] * h1[s]);
    layer<P>(d, false, W1t, true, y);
    if (valid) {
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int k = kin_acc<T>(g, s);
        a.C[atom * LD + k] = (IO)(y[s] * isc[k]);
      }
    }
  }
}

// As many workgroups as the 256 CUs hold at once (three each, in FP64 two, which
// takes a limit of 256 VGPRs): the pass is short, and a second set of workgroups
// pays for its weights and its latencies again.  Against 512 per element, whatever
// its share of the atoms: 255,552 water atoms in FP64 161 -> 123 us, 98,304 in BF16
// 23 -> 18 us, 34,440 fcc atoms in FP64 42 -> 33 us, 1.5M fcc atoms 181 -> 167 us,
// 2M water atoms 219 -> 218 us (768 shared equally by the two elements: 240 us).
template <int P> constexpr int MLP_BLOCKS = P == P_FP64 ? 512 : 768;

template <int P>
void launch_mlp(const MlpArgs<P>& a, hipStream_t stream) {
  if (a.n == 0) return;
  const int blocks = (int)std::min<int64_t>(MLP_BLOCKS<P>, (a.n + 63) / 64 + a.n_el);
  hipLaunchKernelGGL(k_mlp_mfma<P>, dim3((unsigned)(blocks + (a.host_flags ? 1 : 0))), dim3(256), 0, stream, a, blocks);
}

// ------------------------------------------------------------ weight gradient
// One workgroup per chunk of atoms of one element: eight atoms at a time go
// through the forward-over-reverse pass (a.chunk / 8 rounds), and their outer
// products are added to the chunk's partial gradient, all parameters in FP64.
//
// Pass: one atom per 32 lanes, lane l owning hidden unit l with its rows of W1
// and W2 in registers for the whole chunk (and its column of W2 in LDS), so that
// every layer is one 32-term product per lane whose inputs come from the atom's
// other lanes through LDS (broadcast reads of two (value, tangent) pairs each).  With t
// the tangent (JVP row / scale): dh the tangent of h, zb / dzb the adjoints of
// the pre-activations of the primal and the tangent chain.
//
// Sums (W1: zb1 x^T + dzb1 t^T, W2: zb2 h1^T + dzb2 dh1^T): thread t owns the 2 x
// 2 tile at (o, k) = (2 (t / 16), 2 (t % 16)) of both matrices, threads 0-31 also
// b1, b2 and w3 at index t, thread 32 b3, and threads 33-63 the padding (zero).
//
// The eleven vectors of an atom stay in LDS: written to memory by a kernel of
// their own and read back by one per (chunk, element), with the rows of W read by
// every atom and one chunk's atoms loaded one after another, the two took 42 + 60
// us for 30,108 atoms (FP32); this one takes 38 us (FP64 110 -> 64).
template <class T> struct PairOf;
template <> struct PairOf<float> { using type = float2; };
template <> struct PairOf<double> { using type = double2; };

// w . v and w . dv over an atom's 32 (v, dv) pairs, added to z and dz in order
template <class T>
__device__ inline void dot_pairs(const T (&w)[HID], const typename Vec4<T>::type* pairs, T& z, T& dz) {
#pragma unroll
  for (int k = 0; k < HID; k += 2) {
    const typename Vec4<T>::type p = pairs[k / 2];
    z += w[k] * p.x;
    dz += w[k] * p.y;
    z += w[k + 1] * p.z;
    dz += w[k + 1] * p.w;
  }
}

template <int P>
__global__ void __launch_bounds__(256, 2) k_wgrad(WGradArgs<P> a) {
  using T = typename Types<P>::T;
  using T2 = typename PairOf<T>::type;
  using V4 = typename Vec4<T>::type;
  constexpr int ATOMS = 256 / HID;  // atoms per round
  static_assert(HID == 32 && NET_STRIDE == OFF_B3 + HID, "tile map covers the padded layout exactly");
  __shared__ V4 xt[ATOMS][HID / 2], hh[ATOMS][HID / 2], zz1[ATOMS][HID / 2], zz2[ATOMS][HID / 2];  // pairs
  __shared__ T w3g[ATOMS][HID], alphas[ATOMS], W2[HID][HID];
  if (gate_closed(a.gate)) return;
  int e;
  int64_t lo, hi;
  if (!element_tile(blockIdx.x, a.chunk, a.n_el, a.eoff, e, lo, hi)) return;
  hi = lo + a.chunk < hi ? lo + a.chunk : hi;
  e = uniform(e);
  const int t = threadIdx.x, l = t & (HID - 1), g = t / HID;
  const T* __restrict__ W = a.nets + (size_t)e * NET_STRIDE;
  T r1[HID], r2[HID];  // row l of W1 and of W2
#pragma unroll
  for (int k = 0; k < HID; k += 4) {
    const V4 u = *reinterpret_cast<const V4*>(W + OFF_W1 + l * HID + k);
    const V4 v = *reinterpret_cast<const V4*>(W + OFF_W2 + l * HID + k);
    r1[k] = u.x, r1[k + 1] = u.y, r1[k + 2] = u.z, r1[k + 3] = u.w;
    r2[k] = v.x, r2[k + 1] = v.y, r2[k + 2] = v.z, r2[k + 3] = v.w;
  }
  for (int i = t; i < HID * HID; i += 256) W2[i / HID][i % HID] = W[OFF_W2 + i];
  __syncthreads();
  const T b1 = W[OFF_B1 + l], b2 = W[OFF_B2 + l], w3 = W[OFF_W3 + l];
  const T inv_scale = l < MAX_SF ? (T)a.tab->inv_scale_d[e][l] : T(0);
  const int to = t >> 4, tk = t & 15;  // the tile's pairs
  double w1s[2][2] = {{0.0, 0.0}, {0.0, 0.0}}, w2s[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  double b1s = 0.0, b2s = 0.0, w3s = 0.0, b3s = 0.0;
  for (int64_t base = lo; base < hi; base += ATOMS) {
    const int64_t r = base + g;
    if (r < hi) {
      T2 pair;
      pair.x = (T)a.G[r * LD + l];
      pair.y = (T)a.V[r * LD + l] * inv_scale;
      reinterpret_cast<T2*>(xt[g])[l] = pair;
      const T alpha = a.gE ? (T)a.gE[struct_of(a.pos4[r].w)] : T(0);
      __builtin_amdgcn_wave_barrier();
      // layer 1: z = W1 x + b1 and its tangent W1 t
      T z = b1, dz1 = T(0);
      dot_pairs<T>(r1, xt[g], z, dz1);
      const T h1 = tanh_t(z);
      const T dh1 = (T(1) - h1 * h1) * dz1;
      pair.x = h1;
      pair.y = dh1;
      reinterpret_cast<T2*>(hh[g])[l] = pair;
      __builtin_amdgcn_wave_barrier();
      // layer 2.  Objective J = alpha E - w3 . dh2, dh2 = (1 - h2^2) dz2.
      T z2 = b2, dz2 = T(0);
      dot_pairs<T>(r2, hh[g], z2, dz2);
      const T h2 = tanh_t(z2);
      const T g2 = T(1) - h2 * h2;
      // adjoint of h2: alpha w3 from E, and from -w3 . (1 - h2^2) dz2: +2 w3 h2 dz2
      const T h2bar = alpha * w3 + T(2) * w3 * h2 * dz2;
      pair.x = g2 * h2bar;
      pair.y = -g2 * w3;
      reinterpret_cast<T2*>(zz2[g])[l] = pair;
      const T dh2 = g2 * dz2;
      w3g[g][l] = alpha * h2 - dh2;
      if (l == 0) alphas[g] = alpha;
      __builtin_amdgcn_wave_barrier();
      // back through W2 (lane = input unit of layer 2)
      T c2[HID], hb = T(0), dhb = T(0);
#pragma unroll
      for (int o = 0; o < HID; ++o) c2[o] = W2[o][l];
      dot_pairs<T>(c2, zz2[g], hb, dhb);
      const T g1 = T(1) - h1 * h1;
      // dh1 = (1 - h1^2) dz1 contributes -2 h1 dz1 dhb to the adjoint of h1
      hb += dhb * (T(-2) * h1 * dz1);
      pair.x = g1 * hb;
      pair.y = g1 * dhb;
      reinterpret_cast<T2*>(zz1[g])[l] = pair;
    }
    __syncthreads();
    const int na = (int)(hi - base < ATOMS ? hi - base : ATOMS);
    for (int q = 0; q < na; ++q) {
      const V4 zo = zz1[q][to], xk = xt[q][tk], po = zz2[q][to], hk = hh[q][tk];
      const T a_o[2] = {zo.x, zo.z}, c_o[2] = {zo.y, zo.w}, b_k[2] = {xk.x, xk.z}, d_k[2] = {xk.y, xk.w};
      const T p_o[2] = {po.x, po.z}, q_o[2] = {po.y, po.w}, u_k[2] = {hk.x, hk.z}, v_k[2] = {hk.y, hk.w};
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          w1s[i][j] += (double)(a_o[i] * b_k[j] + c_o[i] * d_k[j]);
          w2s[i][j] += (double)(p_o[i] * u_k[j] + q_o[i] * v_k[j]);
        }
      if (t < HID) {
        b1s += (double)reinterpret_cast<const T2*>(zz1[q])[t].x;
        b2s += (double)reinterpret_cast<const T2*>(zz2[q])[t].x;
        w3s += (double)w3g[q][t];
      } else if (t == HID) {
        b3s += (double)alphas[q];
      }
    }
    __syncthreads();  // the round's vectors are read
  }
  const int ch = (int)((lo - a.eoff[e]) / a.chunk);
  double* out = a.partial + ((size_t)e * a.nch + ch) * NET_STRIDE;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      out[OFF_W1 + (2 * to + i) * HID + 2 * tk + j] = w1s[i][j];
      out[OFF_W2 + (2 * to + i) * HID + 2 * tk + j] = w2s[i][j];
    }
  if (t < HID) {
    out[OFF_B1 + t] = b1s;
    out[OFF_B2 + t] = b2s;
    out[OFF_W3 + t] = w3s;
  } else if (t == HID) {
    out[OFF_B3] = b3s;
  }
}

// The gradient in the caller's layout: for each parameter the sum over the
// chunks of its element in a fixed order: eight running sums, chunk ch going to
// sum ch % 8 in chunk order, then the eight in order.  A block covers 32
// parameters with 8 threads each.
__global__ void __launch_bounds__(256) k_wgrad_final(int64_t np, const int* __restrict__ map,
                                                     const int* __restrict__ eoff, int chunk, int nch,
                                                     const double* __restrict__ partial, double* __restrict__ out,
                                                     Gate gate) {
  __shared__ double red[8][32];
  if (gate_closed(gate)) return;
  const int pl = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int64_t i = (int64_t)blockIdx.x * 32 + pl;
  double s = 0.0;
  if (i < np) {
    const int e = map[i] / NET_STRIDE, used = min(nch, (eoff[e + 1] - eoff[e] + chunk - 1) / chunk);
    const double* p = partial + (size_t)e * nch * NET_STRIDE + (map[i] - e * NET_STRIDE);
    // eight loads in flight per thread
#pragma unroll 8
    for (int ch = g; ch < used; ch += 8) s += p[(size_t)ch * NET_STRIDE];
  }
  red[g][pl] = s;
  __syncthreads();
  if (g == 0 && i < np) {
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) tot += red[k][pl];
    out[i] = tot;
  }
}

template <int P>
void launch_wgrad(const WGradArgs<P>& a, hipStream_t stream) {
  if (a.n > 0)  // an element's last chunk may be short: at most one more each
    hipLaunchKernelGGL(k_wgrad<P>, dim3((unsigned)((a.n + a.chunk - 1) / a.chunk + a.n_el)), dim3(256), 0, stream, a);
  hipLaunchKernelGGL(k_wgrad_final, dim3((unsigned)((a.n_params + 31) / 32)), dim3(256), 0, stream, a.n_params, a.flatmap,
                     a.eoff, a.chunk, a.nch, a.partial, a.out, a.gate);
}

template void launch_mlp<P_FP64>(const MlpArgs<P_FP64>&, hipStream_t);
template void launch_mlp<P_FP32>(const MlpArgs<P_FP32>&, hipStream_t);
template void launch_mlp<P_BF16>(const MlpArgs<P_BF16>&, hipStream_t);
template void launch_wgrad<P_FP64>(const WGradArgs<P_FP64>&, hipStream_t);
template void launch_wgrad<P_FP32>(const WGradArgs<P_FP32>&, hipStream_t);

}  // namespace nnp
