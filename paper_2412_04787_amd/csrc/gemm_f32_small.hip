// fp32-environment backward products (Sec. 3.2) of small linears, dX and dW
// of every linear of a call in one launch:
//   dX[m, k] = alpha sum_n dY[m, n] q[n, k]
//   dW[n, k] = sum_m dY[m, n] X~[m, k],   X~ = value(Xq) * xdq in fp32
// on the fp32 matrix cores (v_mfma_f32_32x32x2_f32).
//
// gemm_f32.hip's 128 x 128 tiles leave a small product on a handful of
// compute units, each with a chain of load, barrier and multiply per 16
// reduction elements: a 256 x 256 linear with 512 tokens took 42 us for dX
// and 99 us for dW on four blocks, for 0.13 GFLOP.  Here a block owns one
// 32 x 32 tile and its eight waves take every eighth group of 16 reduction
// elements, straight from memory into registers with the next group in
// flight; their sums are added through LDS in wave order.  Lane half h of a
// wave holds elements 8 h .. 8 h + 7 of a group for both operands.  Bound by
// latency and, for the larger ones, by the operand reads from the caches (per
// 32768 flop a tile reads 2 KB of dY and 128 to 512 bytes of codes for dX, or
// 576 bytes of Xq and scales for dW); 64 x 64 tiles halve those reads but lose
// more blocks than that gives.  Measured, a whole fp32 step (quantise,
// forward, backward, SR update), 128 x 128 tiles -> 32 x 32 (64 x 64), us:
//   256 -> 256, 512 tokens      150 -> 30 (46)
//   512 -> 512, 2048 tokens     210 -> 62 (139)
//   1024 -> 1024, 1024 tokens   292 -> 99 (143)
//   1024 -> 1024, 4096 tokens   353 -> 312 (493)
// (30 us was the host's time for the three calls then; 24 us now.)  With four
// waves a block
// 512 -> 512 with 512 tokens took 35 us instead of 31, 672 -> 192 with 1627
// tokens 61 instead of 47.
#include "gemm_common.h"
#include "sr_rule.h"

namespace dqt {

namespace {

constexpr int kW = 8;      // waves per block
constexpr int kR = 16;     // reduction elements per group

// One product of a launch: C [I][J], tiles in row-major order from block b0.
struct SmallProd {
  const float* dY;         // [M][d_out]
  const uint8_t* p;        // dX: codes [d_out][d_in]; dW: Xq [M][d_in]
  const float* xdq;        // dW: [M]
  void* out;
  float alpha;
  int64_t I, J, R;         // dX: M, d_in, d_out; dW: d_out, d_in, M
  int32_t nj;              // tiles along J
  bool dw, bf16;
};
struct SmallProds {
  SmallProd p[2 * kMaxBatch];
  int32_t b0[2 * kMaxBatch + 1];
  int32_t n;
};

// Code (n, k) of a row of K codes, as fp32.
template <int CF>
struct CodeAt {
  uint32_t v[CF == CF_I3 ? 2 : 1];
  __device__ __forceinline__ void load(const uint8_t* row, int64_t k) {
    if constexpr (CF == CF_T2) v[0] = row[k >> 2];
    else if constexpr (CF == CF_I4) v[0] = row[k >> 1];
    else if constexpr (CF == CF_I3) {
      // bits 3 (k mod 8) of the 24-bit group: one byte, or two neighbours
      const int b = (int)(3 * (k & 7)) >> 3;
      v[0] = row[3 * (k >> 3) + b];
      v[1] = row[3 * (k >> 3) + (b < 2 ? b + 1 : 2)];
    } else v[0] = row[k];
  }
  __device__ __forceinline__ float value(int64_t k) const {
    if constexpr (CF == CF_T2) return code_to_f32((v[0] >> (2 * (k & 3))) & 3u);
    else if constexpr (CF == CF_I4) return (float)((int)(v[0] << (28 - 4 * (k & 1))) >> 28);
    else if constexpr (CF == CF_I3) return (float)((int)(((v[0] | (v[1] << 8)) >> ((3 * (k & 7)) & 7)) << 29) >> 29);
    else return (float)(int)(int8_t)v[0];
  }
};

// Group operands as loaded (converted when used, so the loads stay in
// flight).
template <int CF>
struct DxGroup {
  f32x4 a[2];
  CodeAt<CF> q[8];
};
struct DwGroup {
  float a[8];
  uint32_t x[8];
  float d[8];
};

template <int CF, bool E4M3>
__global__ __launch_bounds__(64 * kW) void gemm_f32_small_kernel(const SmallProds tab) {
  __shared__ f32x4 red[kW][4][64];
  int s = 0;
  while (s + 1 < tab.n && (int)blockIdx.x >= tab.b0[s + 1]) ++s;
  const SmallProd& P = tab.p[s];
  const int tile = (int)blockIdx.x - tab.b0[s];
  const int64_t i0 = (int64_t)(tile / P.nj) * 32, j0 = (int64_t)(tile % P.nj) * 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r32 = lane & 31, h = lane >> 5;
  const int64_t I = P.I, J = P.J, R = P.R;
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
  // this lane's row and column, inside the operands
  const int64_t ci = i0 + r32 < I ? i0 + r32 : I - 1, cj = j0 + r32 < J ? j0 + r32 : J - 1;
  const int64_t ng = (R + kR - 1) / kR;
  // (a wave past its last group loads that group again and does not use it)
  const int64_t last = ng - 1 - ((ng - 1 - wave) & (kW - 1));
  if (wave < ng) {
    if (!P.dw) {
      // dX: R = d_out is a multiple of 16, so every group is whole
      const int64_t ldw = J / 8 * chunk_code_bytes<CF>();
      auto load = [&](int64_t g, DxGroup<CF>& G) {
        const int64_t n = g * kR + 8 * h;
        const f32x4* pa = reinterpret_cast<const f32x4*>(P.dY + ci * R + n);
        G.a[0] = pa[0];
        G.a[1] = pa[1];
#pragma unroll
        for (int e = 0; e < 8; ++e) G.q[e].load(P.p + (n + e) * ldw, cj);
      };
      auto use = [&](const DxGroup<CF>& G) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(G.a[e >> 2][e & 3], G.q[e].value(cj), acc, 0, 0, 0);
      };
      DxGroup<CF> G0, G1;
      load(wave, G0);
      for (int64_t g = wave; g <= last; g += 2 * kW) {
        load(g + kW < last ? g + kW : last, G1);
        use(G0);
        if (g + kW > last) break;
        load(g + 2 * kW < last ? g + 2 * kW : last, G0);
        use(G1);
      }
    } else {
      auto load = [&](int64_t g, DwGroup& G) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int64_t m = g * kR + 8 * h + e < R ? g * kR + 8 * h + e : R - 1;
          G.d[e] = P.xdq[m];
          G.a[e] = P.dY[m * I + ci];
          G.x[e] = P.p[m * J + cj];
        }
      };
      auto use = [&](int64_t g, const DwGroup& G) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool ok = g * kR + 8 * h + e < R;       // tokens past the end count as zeros
          const float v = E4M3 ? e4m3_to_f32(G.x[e]) : (float)(int)(int8_t)G.x[e];
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ok ? G.a[e] : 0.0f, ok ? v * G.d[e] : 0.0f, acc, 0, 0, 0);
        }
      };
      DwGroup G0, G1;
      load(wave, G0);
      for (int64_t g = wave; g <= last; g += 2 * kW) {
        load(g + kW < last ? g + kW : last, G1);
        use(g, G0);
        if (g + kW > last) break;
        load(g + 2 * kW < last ? g + 2 * kW : last, G0);
        use(g + kW, G1);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    red[wave][k][lane] = f32x4{acc[4 * k], acc[4 * k + 1], acc[4 * k + 2], acc[4 * k + 3]};
  __syncthreads();
  // wave k: rows 8 k + 4 h .. + 3 of column r32
  if (wave >= 4) return;
  f32x4 v = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < kW; ++w)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] + red[w][wave][lane][e];
  const int64_t j = j0 + r32;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int64_t i = i0 + 8 * wave + 4 * h + e;
    if (i >= I || j >= J) continue;
    if (P.dw) {
      static_cast<float*>(P.out)[i * J + j] = v[e];
    } else {
      const float o = P.alpha * v[e];
      if (P.bf16) static_cast<uint16_t*>(P.out)[i * J + j] = (uint16_t)f32_to_bf16_bits(o);
      else static_cast<float*>(P.out)[i * J + j] = o;
    }
  }
}

template <int CF, bool E4M3>
hipError_t launch_t(SmallProds& tab, hipStream_t stream) {
  int32_t blocks = 0;
  for (int s = 0; s < tab.n; ++s) {
    SmallProd& p = tab.p[s];
    p.nj = (int32_t)((p.J + 31) / 32);
    tab.b0[s] = blocks;
    blocks += p.nj * (int32_t)((p.I + 31) / 32);
  }
  tab.b0[tab.n] = blocks;
  return timed_launch(stream, [&] {
    return launch_kernel(gemm_f32_small_kernel<CF, E4M3>, dim3((unsigned)blocks), dim3(64 * kW), stream, tab);
  });
}

}  // namespace

// The rule, for each product of a linear by the linear's own shape: few
// outputs (64 x 64 tiles of dX and dW together: 1280 of them 313 against 353
// us, 1536 631 against 670 us, 3072 1205 against 1065 us), and a reduction
// over tokens that one block's waves get through (256 -> 256: 512 tokens 30
// against 150 us; 16384 tokens, which the 128 x 128 kernel splits over blocks,
// 290 against 193 us).  Many tiles of a reduction too short for the eight
// waves are better in 128 x 128 (dX of 4096 -> 64: 512 tokens, 512 tiles, 12.2
// against 15.2 us, 1000 tokens 20.3 against 16.4; dW of 16 tokens: 1024 ->
// 1024, 256 tiles, 7.0 against 7.8 us, 2048 -> 2048 20.2 against 9.5), as are
// those of dW with so many tokens that the other kernel splits them (1024 ->
// 2048, 512 tiles: 1536 tokens 122 against 154 us, 4096 321 against 294).  The
// two kernels add in different orders, and a batch gives the results of its
// linears one by one: so neither the other linears of the call nor which of
// dX and dW it asks for count.
static int64_t tiles64(int64_t rows, int64_t cols) { return ((rows + 63) / 64) * ((cols + 63) / 64); }
static bool f32_small_linear(int64_t d_in, int64_t d_out, int64_t M) {
  return M >= 1 && M <= kF32SmallM && tiles64(M, d_in) + tiles64(d_out, d_in) <= kF32SmallTiles;
}
bool f32_small_dx(int64_t d_in, int64_t d_out, int64_t M) {
  return f32_small_linear(d_in, d_out, M) && tiles64(M, d_in) <= (d_out > 32 ? 8 * d_out : 256);
}
bool f32_small_dw(int64_t d_in, int64_t d_out, int64_t M) {
  const int64_t t = tiles64(d_out, d_in);
  return f32_small_linear(d_in, d_out, M) && t <= (M > 42 ? 6 * M : 256) &&
         (dw_splits_f32(d_out, d_in, M) == 1 || t * M <= 3 << 18);
}

hipError_t launch_bwd_f32_small(int cf, bool e4m3, bool dx_bf16, int n, const LinearIO* io, int64_t M,
                                hipStream_t stream) {
  SmallProds tab{};
  // the longer reductions first
  for (int l = 0; l < n; ++l)
    if (io[l].dW != nullptr)
      tab.p[tab.n++] = SmallProd{static_cast<const float*>(io[l].dY), static_cast<const uint8_t*>(io[l].Xq), io[l].xdq,
                                 io[l].dW, 1.0f, io[l].d_out, io[l].d_in, M, 0, true, false};
  for (int l = 0; l < n; ++l)
    if (io[l].dX != nullptr)
      tab.p[tab.n++] = SmallProd{static_cast<const float*>(io[l].dY), static_cast<const uint8_t*>(io[l].Wq), nullptr,
                                 io[l].dX, io[l].alpha, M, io[l].d_in, io[l].d_out, 0, false, dx_bf16};
  switch (cf) {
    case CF_T2: return e4m3 ? launch_t<CF_T2, true>(tab, stream) : launch_t<CF_T2, false>(tab, stream);
    case CF_I4: return e4m3 ? launch_t<CF_I4, true>(tab, stream) : launch_t<CF_I4, false>(tab, stream);
    case CF_I3: return e4m3 ? launch_t<CF_I3, true>(tab, stream) : launch_t<CF_I3, false>(tab, stream);
    default: return e4m3 ? launch_t<CF_I8, true>(tab, stream) : launch_t<CF_I8, false>(tab, stream);
  }
}

}  // namespace dqt
