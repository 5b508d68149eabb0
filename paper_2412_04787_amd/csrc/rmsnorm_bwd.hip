// Backward of the RMSNorm that feeds a group of DQT linears, for the model
// step: the linears' dX (the activation quantiser passes the gradient
// through) summed, then the norm's own backward, in one pass pair over the
// rows.  For row m of X [M, K] with r_m from dqt_rmsnorm_act_quant:
//   dn_mk = sum_i dY_i[m, k]                       (fp32, i in order)
//   g_mk  = dn_mk gamma_k
//   c_m   = (sum_k g_mk x_mk) / K
//   dX_mk = r_m g_mk - x_mk r_m^3 c_m              (rounded to bf16)
//   gpart[b, k] = sum over the rows m of block b of dn_mk x_mk r_m
// so dgamma_k = sum_b gpart[b, k] (the caller sums, in a fixed order).
//
// One wave per row, 4 waves per block; block b takes rows 4 b + w,
// 4 b + w + 4 B, ... (B blocks).  The block adds its waves' gamma gradients in
// order at the end.  HBM traffic per element: 2 bytes per dY_i and 2 for x,
// 2 bytes of dX written; bound by it.
//
// Rows of up to 64 x 8 x 8 elements are held in registers (the row read once,
// all its loads in flight together), as are gamma (up to 2048 elements) and
// the wave's share of the gamma gradient; longer rows are read twice, with
// the gamma gradient in LDS.  Same operations in the same order either way.
// Reading every row twice with an LDS read-modify-write per element took 108
// us at 16384 x 2048 with three dY (3.1 TB/s), this 65 us (5.2 TB/s).
#include "dqt_launch.h"

namespace dqt {

namespace {

constexpr int kWaves = 4;

struct DyArgs {
  const uint16_t* p[kMaxNormDy];
};

__device__ __forceinline__ void decode8(uint4 u, float (&v)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = bf16_bits_to_f32(w[i] & 0xFFFFu);
    v[2 * i + 1] = bf16_bits_to_f32(w[i] >> 16);
  }
}

__device__ __forceinline__ void load8_bf16(const uint16_t* p, float (&v)[8]) {
  decode8(*reinterpret_cast<const uint4*>(p), v);
}

template <int NDY>
__global__ __launch_bounds__(kWaves * kWave) void rmsnorm_bwd_kernel(
    DyArgs dy, const uint16_t* __restrict__ X, const float* __restrict__ gamma,
    const float* __restrict__ rinv, int64_t M, int K, uint16_t* __restrict__ dX,
    float* __restrict__ gpart) {
  extern __shared__ float gsh[];              // [kWaves][K]
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  const int nchunk = K / 8;
  float* mine = gsh + (size_t)w * K;
  for (int k = lane; k < K; k += kWave) mine[k] = 0.0f;
  const float invK = __fdiv_rn(1.0f, (float)K);
  auto dn8 = [&](int64_t off, float (&dn)[8]) {
    load8_bf16(dy.p[0] + off, dn);
#pragma unroll
    for (int i = 1; i < NDY; ++i) {
      float t[8];
      load8_bf16(dy.p[i] + off, t);
#pragma unroll
      for (int j = 0; j < 8; ++j) dn[j] = dn[j] + t[j];
    }
  };
  for (int64_t row = (int64_t)blockIdx.x * kWaves + w; row < M; row += (int64_t)gridDim.x * kWaves) {
    const int64_t base = row * (int64_t)K;
    const float r = rinv[row];
    float dot = 0.0f;
    for (int c = lane; c < nchunk; c += kWave) {
      float dn[8], x[8];
      dn8(base + 8 * c, dn);
      load8_bf16(X + base + 8 * c, x);
      const float4 g0 = *reinterpret_cast<const float4*>(gamma + 8 * c);
      const float4 g1 = *reinterpret_cast<const float4*>(gamma + 8 * c + 4);
      const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) dot = dot + (dn[j] * g[j]) * x[j];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) dot = dot + __shfl_xor(dot, d, kWave);
    const float cr3 = ((dot * invK) * r) * (r * r);
    for (int c = lane; c < nchunk; c += kWave) {
      float dn[8], x[8];
      dn8(base + 8 * c, dn);
      load8_bf16(X + base + 8 * c, x);
      const float4 g0 = *reinterpret_cast<const float4*>(gamma + 8 * c);
      const float4 g1 = *reinterpret_cast<const float4*>(gamma + 8 * c + 4);
      const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
      uint32_t o[4];
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float a = r * (dn[j] * g[j]) - x[j] * cr3;
        const float b = r * (dn[j + 1] * g[j + 1]) - x[j + 1] * cr3;
        o[j >> 1] = f32_to_bf16_bits(a) | (f32_to_bf16_bits(b) << 16);
      }
      *reinterpret_cast<uint4*>(dX + base + 8 * c) = make_uint4(o[0], o[1], o[2], o[3]);
#pragma unroll
      for (int j = 0; j < 8; ++j) mine[8 * c + j] += (dn[j] * x[j]) * r;
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += kWaves * kWave) {
    float s = gsh[k];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) s = s + gsh[(size_t)i * K + k];
    gpart[(int64_t)blockIdx.x * K + k] = s;
  }
}

// Rows of at most 512 NCH elements, NCH chunks of 8 per lane.  (NCH = 6: in 256
// registers, so that two blocks fit a compute unit.)
template <int NDY, int NCH>
__global__ __launch_bounds__(kWaves * kWave, NCH == 6 ? 2 : 1) void rmsnorm_bwd_reg_kernel(
    DyArgs dy, const uint16_t* __restrict__ X, const float* __restrict__ gamma,
    const float* __restrict__ rinv, int64_t M, int K, uint16_t* __restrict__ dX,
    float* __restrict__ gpart) {
  extern __shared__ float gsh[];              // [kWaves][K]
  constexpr bool kHoldG = NCH <= 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  const int nchunk = K / 8;
  const float invK = __fdiv_rn(1.0f, (float)K);
  auto load_g = [&](int c, float (&g)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(gamma + 8 * c);
    const float4 b = *reinterpret_cast<const float4*>(gamma + 8 * c + 4);
    g[0] = a.x; g[1] = a.y; g[2] = a.z; g[3] = a.w;
    g[4] = b.x; g[5] = b.y; g[6] = b.z; g[7] = b.w;
  };
  // (lanes without a chunk c load the last one and do not use it)
  int idx[NCH];
  float acc[NCH][8], gam[kHoldG ? NCH : 1][8];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    idx[c] = lane + kWave * c < nchunk ? lane + kWave * c : nchunk - 1;
    if constexpr (kHoldG) load_g(idx[c], gam[c]);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[c][j] = 0.0f;
  }
  for (int64_t row = (int64_t)blockIdx.x * kWaves + w; row < M; row += (int64_t)gridDim.x * kWaves) {
    const int64_t base = row * (int64_t)K;
    const float r = rinv[row];
    uint4 xr[NCH], yr[NCH][NDY];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      xr[c] = *reinterpret_cast<const uint4*>(X + base + 8 * idx[c]);
#pragma unroll
      for (int i = 0; i < NDY; ++i) yr[c][i] = *reinterpret_cast<const uint4*>(dy.p[i] + base + 8 * idx[c]);
    }
    float dn[NCH][8];
    float dot = 0.0f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      float x[8], g[8];
      decode8(xr[c], x);
      decode8(yr[c][0], dn[c]);
#pragma unroll
      for (int i = 1; i < NDY; ++i) {
        float t[8];
        decode8(yr[c][i], t);
#pragma unroll
        for (int j = 0; j < 8; ++j) dn[c][j] = dn[c][j] + t[j];
      }
      if constexpr (!kHoldG) load_g(idx[c], g);
      const bool in = lane + kWave * c < nchunk;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float d = dot + (dn[c][j] * (kHoldG ? gam[kHoldG ? c : 0][j] : g[j])) * x[j];
        dot = in ? d : dot;
      }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) dot = dot + __shfl_xor(dot, d, kWave);
    const float cr3 = ((dot * invK) * r) * (r * r);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (lane + kWave * c >= nchunk) continue;
      float x[8], g[8];
      decode8(xr[c], x);
      if constexpr (!kHoldG) load_g(idx[c], g);
      uint32_t o[4];
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float ga = kHoldG ? gam[kHoldG ? c : 0][j] : g[j], gb = kHoldG ? gam[kHoldG ? c : 0][j + 1] : g[j + 1];
        const float a = r * (dn[c][j] * ga) - x[j] * cr3;
        const float b = r * (dn[c][j + 1] * gb) - x[j + 1] * cr3;
        o[j >> 1] = f32_to_bf16_bits(a) | (f32_to_bf16_bits(b) << 16);
      }
      *reinterpret_cast<uint4*>(dX + base + 8 * idx[c]) = make_uint4(o[0], o[1], o[2], o[3]);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[c][j] += (dn[c][j] * x[j]) * r;
    }
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if (lane + kWave * c >= nchunk) continue;
    float4* const d = reinterpret_cast<float4*>(gsh + (size_t)w * K + 8 * idx[c]);
    d[0] = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
    d[1] = make_float4(acc[c][4], acc[c][5], acc[c][6], acc[c][7]);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += kWaves * kWave) {
    float s = gsh[k];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) s = s + gsh[(size_t)i * K + k];
    gpart[(int64_t)blockIdx.x * K + k] = s;
  }
}

template <int NDY>
hipError_t launch_ndy(const DyArgs& a, const uint16_t* x, const float* gamma, const float* rinv, int64_t M, int K,
                      uint16_t* dx, float* gpart, int blocks, hipStream_t stream) {
  const size_t lds = (size_t)kWaves * K * sizeof(float);
  const dim3 grid((unsigned)blocks), block(kWaves * kWave);
  const int nch = (K / 8 + kWave - 1) / kWave;
  if constexpr (NDY == 1) {
    // One dY over more than 2048 elements: so many blocks that they do not
    // all fit beside each other in registers, with few rows each, are better
    // in the kernel that keeps the gradient in LDS (1024 blocks: 1024 x 4096
    // 15.1 against 16.1 us, 4096 x 2560 21.3 against 23.9; 4096 x 4096 42 against
    // 35 us); two blocks a compute unit up to 3072 elements (4096 x 2064 21.7
    // us, one 24.2; with two dY that spills, 27.5 -> 35 us).
    if (nch > 4 && blocks > 2 * current_device_cus() && M < (int64_t)kWaves * blocks * (nch == 5 ? 2 : 1))
      return launch_kernel_lds(rmsnorm_bwd_kernel<1>, grid, block, lds, stream, a, x, gamma, rinv, M, K, dx, gpart);
    if (nch > 4 && nch <= 6)
      return launch_kernel_lds(rmsnorm_bwd_reg_kernel<1, 6>, grid, block, lds, stream, a, x, gamma, rinv, M, K, dx, gpart);
  }
  const auto k = nch <= 1 ? rmsnorm_bwd_reg_kernel<NDY, 1> : nch <= 2 ? rmsnorm_bwd_reg_kernel<NDY, 2>
               : nch <= 3 ? rmsnorm_bwd_reg_kernel<NDY, 3> : nch <= 4 ? rmsnorm_bwd_reg_kernel<NDY, 4>
               : nch <= 8 ? rmsnorm_bwd_reg_kernel<NDY, 8> : rmsnorm_bwd_kernel<NDY>;
  return launch_kernel_lds(k, grid, block, lds, stream, a, x, gamma, rinv, M, K, dx, gpart);
}

}  // namespace

hipError_t launch_rmsnorm_backward(int n_dy, const void* const* dY, const void* X, const float* gamma,
                                   const float* rinv, int64_t M, int K, void* dX, float* gpart,
                                   int blocks, hipStream_t stream) {
  DyArgs a{};
  for (int i = 0; i < n_dy; ++i) a.p[i] = static_cast<const uint16_t*>(dY[i]);
  const uint16_t* x = static_cast<const uint16_t*>(X);
  uint16_t* dx = static_cast<uint16_t*>(dX);
  switch (n_dy) {
    case 1: return launch_ndy<1>(a, x, gamma, rinv, M, K, dx, gpart, blocks, stream);
    case 2: return launch_ndy<2>(a, x, gamma, rinv, M, K, dx, gpart, blocks, stream);
    case 3: return launch_ndy<3>(a, x, gamma, rinv, M, K, dx, gpart, blocks, stream);
    default: return launch_ndy<4>(a, x, gamma, rinv, M, K, dx, gpart, blocks, stream);
  }
}

}  // namespace dqt
