// Forward of DQT linears for few tokens (decoding, prompts, short
// micro-batches), Sec. 3.2: Y = fl(fl(Xq q^T) fl(xdq alpha)).
//
// The persistent 256 x 256 GEMM (gemm_v3.hip) expands every weight code into
// the workspace first and then needs enough tokens to fill its tiles.  With
// few tokens both are the cost: at hidden 4096 and 8 tokens the block's
// forward took 28 us of expansion and 116 us of GEMM, where the packed codes
// (51 MB) stream in 11 us.  The two kernels here read the packed codes
// themselves, expand them in registers, and need no workspace:
//  * fwd_skinny_kernel: bound by the stream of codes;
//  * fwd_mid_kernel: bound by the matrix cores and the LDS traffic of its
//    64 x 64 wave tiles.
// Measured, whole block with the activation quantisation (one launch), the
// persistent GEMM -> these kernels, us:
//   tokens                        1        16        64       256       512       777
//   h4096 ternary, e4m3   152 -> 18  153 -> 21  153 -> 50  157 -> 73  207 -> 126  217 -> 205
//   h2048 4-bit, int8      86 -> 15   87 -> 17   88 -> 35   89 -> 37   91 -> 49   120 -> 77
//   h2048 8-bit, int8      72 -> 15   73 -> 22   74 -> 34   75 -> 37   77 -> 47   106 -> 73
//   h768 ternary, int8     40 -> 14   40 -> 15   41 -> 18   41 -> 19   41 -> 24    43 -> 25
// (14 us is two launches from the Python binding.)
#include <algorithm>

#include "gemm_common.h"
#include "sr_rule.h"

namespace dqt {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
using lds_i32x4 = __attribute__((address_space(3))) i32x4;

// 64 consecutive codes of one weight row as stored: 16 bytes of ternary
// codes, 24 of 3-bit, 32 of 4-bit, 64 of 8-bit.
template <int CF>
struct Raw64 {
  static constexpr int NB = 8 * chunk_code_bytes<CF>();
  static constexpr int ND = NB / 4;
  uint32_t w[ND];

  // Loads the codes k .. k + 63 of the row at p (K codes); those past K hold
  // codes of the row's start until mask().  VEC: K is a multiple of 64, so
  // the row and the 64 codes are aligned for wide loads and all valid or
  // none; otherwise 16 codes at a time, at the alignment that K a multiple of
  // 16 leaves.  (Masking where the codes are used, not here, keeps the loads
  // in flight: a select right after them waited for every one.)
  template <bool VEC>
  __device__ __forceinline__ void load(const uint8_t* p, int k, int K) {
    if constexpr (VEC) {
      const uint8_t* s = p + (int64_t)((k < K ? k : 0) / 8 * chunk_code_bytes<CF>());
      if constexpr (CF == CF_I3) {
#pragma unroll
        for (int i = 0; i < ND / 2; ++i) {
          const u32x2 v = reinterpret_cast<const u32x2*>(s)[i];
          w[2 * i] = v[0];
          w[2 * i + 1] = v[1];
        }
      } else {
#pragma unroll
        for (int i = 0; i < ND / 4; ++i) {
          const i32x4 v = reinterpret_cast<const i32x4*>(s)[i];
#pragma unroll
          for (int j = 0; j < 4; ++j) w[4 * i + j] = (uint32_t)v[j];
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint8_t* s = p + (int64_t)((k + 16 * q < K ? k + 16 * q : 0) / 8 * chunk_code_bytes<CF>());
        if constexpr (CF == CF_T2) {
          w[q] = *reinterpret_cast<const uint32_t*>(s);
        } else if constexpr (CF == CF_I4) {
          const u32x2 v = *reinterpret_cast<const u32x2*>(s);
          w[2 * q] = v[0];
          w[2 * q + 1] = v[1];
        } else if constexpr (CF == CF_I3) {
          const uint16_t* h = reinterpret_cast<const uint16_t*>(s);
          h3[q][0] = h[0];
          h3[q][1] = h[1];
          h3[q][2] = h[2];
        } else {
          const i32x4 v = *reinterpret_cast<const i32x4*>(s);
#pragma unroll
          for (int j = 0; j < 4; ++j) w[4 * q + j] = (uint32_t)v[j];
        }
      }
    }
  }
  uint16_t h3[CF == CF_I3 ? 4 : 1][3];   // 3-bit codes of the narrow form, as loaded
  // Codes past K become zero (once, before bytes16).
  template <bool VEC>
  __device__ __forceinline__ void mask(int k, int K) {
    constexpr uint32_t kZero = CF == CF_T2 ? 0x55555555u : 0u;
    if constexpr (VEC) {
#pragma unroll
      for (int i = 0; i < ND; ++i) w[i] = k < K ? w[i] : kZero;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool ok = k + 16 * q < K;
        if constexpr (CF == CF_I3) {
          const uint32_t a = ok ? h3[q][0] : 0u, b = ok ? h3[q][1] : 0u, c = ok ? h3[q][2] : 0u;
          // 48 bits at bit 48 q of the six words
          if ((q & 1) == 0) {
            w[3 * (q >> 1)] = a | (b << 16);
            w[3 * (q >> 1) + 1] = c;
          } else {
            w[3 * (q >> 1) + 1] |= a << 16;
            w[3 * (q >> 1) + 2] = b | (c << 16);
          }
        } else {
#pragma unroll
          for (int j = 0; j < ND / 4; ++j) w[ND / 4 * q + j] = ok ? w[ND / 4 * q + j] : kZero;
        }
      }
    }
  }

  // Four codes (one per byte of x, as stored fields) -> operand bytes.
  template <bool E4M3>
  __device__ static __forceinline__ uint32_t conv(uint32_t x) {
    if constexpr (CF == CF_I3) {
      // fields 0..3 -> 0..3, 4..7 -> -4..-1
      if constexpr (E4M3) return __builtin_amdgcn_perm(0xB8C0C4C8u, 0x44403800u, x);
      else return ((x ^ 0x04040404u) + 0x7C7C7C7Cu) ^ 0x80808080u;
    } else {
      // nibbles 0..7 -> 0..7, 8..15 -> -8..-1
      if constexpr (E4M3) {
        const uint32_t sel = x & 0x07070707u;
        const uint32_t lo = __builtin_amdgcn_perm(0x4E4C4A48u, 0x44403800u, sel);
        const uint32_t hi = __builtin_amdgcn_perm(0xB8C0C4C8u, 0xCACCCED0u, sel);
        const uint32_t m = ((x >> 3) & 0x01010101u) * 255u;
        return (lo & ~m) | (hi & m);
      } else {
        return ((x ^ 0x08080808u) + 0x78787878u) ^ 0x80808080u;
      }
    }
  }
  // Codes 16 q .. 16 q + 15 as 16 operand bytes (int8, or e4m3) in order.
  template <bool E4M3>
  __device__ __forceinline__ i32x4 bytes16(int q) const {
    if constexpr (CF == CF_I8) {
      return i32x4{(int)w[4 * q], (int)w[4 * q + 1], (int)w[4 * q + 2], (int)w[4 * q + 3]};
    } else if constexpr (CF == CF_T2) {
      return expand16(w[q], E4M3 ? 0x003800B8u : 0x000100FFu);
    } else if constexpr (CF == CF_I4) {
      i32x4 o;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t lo = w[2 * q + i] & 0x0F0F0F0Fu, hi = (w[2 * q + i] >> 4) & 0x0F0F0F0Fu;
        o[2 * i] = (int)conv<E4M3>(__builtin_amdgcn_perm(hi, lo, 0x05010400u));
        o[2 * i + 1] = (int)conv<E4M3>(__builtin_amdgcn_perm(hi, lo, 0x07030602u));
      }
      return o;
    } else {
      // 48 bits: four groups of 12
      const uint32_t x0 = (q & 1) == 0 ? w[3 * (q >> 1)] : (w[3 * (q >> 1) + 1] >> 16) | (w[3 * (q >> 1) + 2] << 16);
      const uint32_t x1 = (q & 1) == 0 ? w[3 * (q >> 1) + 1] & 0xFFFFu : w[3 * (q >> 1) + 2] >> 16;
      const uint32_t g[4] = {x0 & 0xFFFu, (x0 >> 12) & 0xFFFu, (x0 >> 24) | ((x1 & 0xFu) << 8), (x1 >> 4) & 0xFFFu};
      i32x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = (int)conv<E4M3>((g[i] & 7u) | ((g[i] & 0x38u) << 5) | ((g[i] & 0x1C0u) << 10) | ((g[i] & 0xE00u) << 15));
      return o;
    }
  }
};

// One linear of a launch.
struct SmallLin {
  const uint8_t* wq;
  const uint8_t* xq;
  const float* xdq;
  void* y;
  float alpha;
  int32_t K, N;
};
struct SmallTab {
  SmallLin p[kMaxBatch];
  int32_t b0[kMaxBatch + 1];   // skinny: first block; mid: tiles of each linear
  int32_t n;
  int32_t M;
  int32_t mt;                  // mid: row tiles
  int32_t bf16;
};

template <bool E4M3> struct Acc4 { using type = i32x4; };
template <> struct Acc4<true> { using type = f32x4; };

// Few tokens.  A wave multiplies 16 RG rows of W (first operand of the
// 16 x 16 matrix instructions) by up to 16 MT tokens; lane (r, g) holds row
// r's 64 codes at 256 i + 64 g of reduction step i, one wide load of the
// packed codes (16 rows x 64 contiguous bytes per instruction for ternary
// codes) that expands to the operands of four sub-steps.  The tokens' codes
// come straight from the caches with the same lane-to-element map.  The eight
// waves of a block take every eighth step of the same rows and add their
// sums through LDS in wave order (int32: exact; fp32: a fixed order), so a
// block's work is short and thousands of waves are in flight: what bounds
// the kernel is the stream of codes and, with more tokens, the tokens' codes
// from L2 (M / (16 RG) bytes per weight).
//
// RG (which no result depends on): 2; 4 where that leaves two blocks for
// every compute unit (h4096 ternary, 8 tokens 22.7 -> 19.8 us, 48 tokens 50
// -> 39 us; at hidden 2048 with 4-bit codes 1 token 14.5 -> 16.6 us); 1 for
// up to 16 tokens of 8-bit codes, whose loads are four times the bytes (h2048,
// 1 token 19.1 -> 14.6 us).
constexpr int kSkW = 8;
template <int CF, bool E4M3, int MT, int RG, bool VEC>
__global__ __launch_bounds__(64 * kSkW) void fwd_skinny_kernel(const SmallTab tab) {
  using Acc = typename Acc4<E4M3>::type;
  __shared__ Acc red[kSkW][RG * MT][64];
  int s = 0;
  while (s + 1 < tab.n && (int)blockIdx.x >= tab.b0[s + 1]) ++s;
  const SmallLin& L = tab.p[s];
  const int K = L.K, N = L.N, M = tab.M;
  const int n0 = ((int)blockIdx.x - tab.b0[s]) * (16 * RG);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const uint8_t* wrow[RG];
#pragma unroll
  for (int t = 0; t < RG; ++t) {
    const int n = n0 + 16 * t + r;
    wrow[t] = L.wq + (int64_t)(n < N ? n : N - 1) * (K / 8 * chunk_code_bytes<CF>());
  }
  const uint8_t* xrow[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int m = 16 * t + r;
    xrow[t] = L.xq + (int64_t)(m < M ? m : M - 1) * K;
  }
  Acc acc[RG][MT];
#pragma unroll
  for (int a = 0; a < RG; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) acc[a][b] = Acc{0, 0, 0, 0};

  const int nit = (K + 255) / 256;
  struct Step {
    Raw64<CF> w[RG];
    i32x4 x[MT][4];
  };
  auto fetch = [&](int it, Step& S) {
    const int k = it * 256 + 64 * g;
#pragma unroll
    for (int t = 0; t < RG; ++t) S.w[t].template load<VEC>(wrow[t], k, K);
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // (past the end of the row: any codes of the row, they meet zeros)
        const int kx = k + 16 * q < K ? k + 16 * q : 0;
        S.x[t][q] = *reinterpret_cast<const i32x4*>(xrow[t] + kx);
      }
  };
  auto mult = [&](int it, Step& S) {
    const int k = it * 256 + 64 * g;
#pragma unroll
    for (int a = 0; a < RG; ++a) {
      S.w[a].template mask<VEC>(k, K);
      if constexpr (!E4M3) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const i32x4 wv = S.w[a].template bytes16<false>(q);
#pragma unroll
          for (int b = 0; b < MT; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, S.x[b][q], acc[a][b], 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
          const i32x4 w0 = S.w[a].template bytes16<true>(q), w1 = S.w[a].template bytes16<true>(q + 1);
          const i32x8 wv = {w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3]};
#pragma unroll
          for (int b = 0; b < MT; ++b) {
            const i32x4 x0 = S.x[b][q], x1 = S.x[b][q + 1];
            const i32x8 xv = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wv, xv, acc[a][b], 0, 0, 0, 127, 0, 127);
          }
        }
      }
    }
  };
  if (wave < nit) {
    // (a step past this wave's last is fetched again and not used: the loads
    // stay free of branches, so none of them is waited for early)
    const int last = nit - 1 - ((nit - 1 - wave) & (kSkW - 1));
    Step S0, S1;
    fetch(wave, S0);
    for (int it = wave; it <= last; it += 2 * kSkW) {
      fetch(it + kSkW < last ? it + kSkW : last, S1);
      mult(it, S0);
      if (it + kSkW > last) break;
      fetch(it + 2 * kSkW < last ? it + 2 * kSkW : last, S0);
      mult(it + kSkW, S1);
    }
  }
#pragma unroll
  for (int a = 0; a < RG; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) red[wave][a * MT + b][lane] = acc[a][b];
  __syncthreads();
  // lane (m = r, g) of block (a, b): rows n = 16 a + 4 g .. + 3 of token 16 b + r
  for (int q = wave; q < RG * MT; q += kSkW) {
    Acc v = red[0][q][lane];
#pragma unroll
    for (int w = 1; w < kSkW; ++w) v += red[w][q][lane];
    const int m = 16 * (q % MT) + r, n = n0 + 16 * (q / MT) + 4 * g;
    if (m < M && n < N) {
      const float sc = L.xdq[m] * L.alpha;
      const float o0 = (float)v[0] * sc, o1 = (float)v[1] * sc, o2 = (float)v[2] * sc, o3 = (float)v[3] * sc;
      const int64_t at = (int64_t)m * N + n;
      if (tab.bf16)
        *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(L.y) + at) = u32x2{pack_bf16x2(o0, o1), pack_bf16x2(o2, o3)};
      else
        *reinterpret_cast<f32x4*>(static_cast<float*>(L.y) + at) = f32x4{o0, o1, o2, o3};
    }
  }
}

// Some hundred tokens: 128 x 128 output tiles, 4 waves of 64 x 64 (2 x 2
// matrix blocks of 32 x 32), 128 reduction elements a step, two blocks a
// compute unit.  Both operands go through registers (16-byte loads two steps
// ahead, so a step's latency from HBM is spread over two steps of two
// blocks; the weights are expanded on the way into LDS, each code once per
// tile, between the matrix instructions of the step before).  KS = 2: two
// groups of 4 waves take every other step of one tile, each with its own
// stages (one block a compute unit), and the second group's sums are added
// through LDS; a tile then takes half the steps, which counts while the
// launch has about as many tiles as compute units (h4096 at 128 tokens 75 ->
// 57 us; at 512 tokens 131 -> 138 us, so the rule stops at kMidSplitM).  LDS rows are 128 bytes, 16-byte chunk c of row i at chunk
// c ^ ((i >> 1) & 7), conflict-free for the fragment reads.
constexpr int MTI = 128;                    // tile edge
constexpr int kMidStage = 2 * MTI * 128;    // A then B, bytes
__device__ __forceinline__ int mid_at(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }
__device__ __forceinline__ void mid_barrier() {
  __asm__ volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((15) | (3 << 14) | (7 << 4) | (0 << 8));   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
}

template <int CF, bool E4M3, bool VEC, int KS>
__global__ __launch_bounds__(256 * KS, 2) void fwd_mid_kernel(const SmallTab tab) {
  using Acc = typename AccT<E4M3 ? Mfma::F8 : Mfma::I8>::type;
  __shared__ __attribute__((aligned(1024))) uint8_t stages[KS * 2 * kMidStage];
  const int kg = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
  lds_u8* const smem = (lds_u8*)stages + kg * 2 * kMidStage;
  // XCD x (blocks are dispatched round-robin) takes a contiguous eighth of
  // every linear's tiles, row tiles of one weight panel next to each other
  const int x = blockIdx.x & 7;
  int j = blockIdx.x >> 3, s = 0, local = -1;
  for (; s < tab.n; ++s) {
    const int nt = tab.b0[s];
    const int first = (x * nt) >> 3, cnt = (((x + 1) * nt) >> 3) - first;
    if (j < cnt) {
      local = first + j;
      break;
    }
    j -= cnt;
  }
  if (local < 0) return;
  const SmallLin& L = tab.p[s];
  const int K = L.K, N = L.N, M = tab.M;
  const int m0 = (local % tab.mt) * MTI, n0 = (local / tab.mt) * MTI;
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 1, wj = wave & 1;
  const int h = lane >> 5, fr = lane & 31;

  // A: chunks tid + 256 q: row (tid >> 3) + 32 q, 16-byte chunk tid & 7
  const int ac = tid & 7;
  const uint8_t* arow[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int m = m0 + (tid >> 3) + 32 * q;
    arow[q] = L.xq + (int64_t)(m < M ? m : M - 1) * K;
  }
  // B: row tid / 2, 64 codes from 64 (tid & 1)
  const int bn = n0 + (tid >> 1);
  const uint8_t* const brow = L.wq + (int64_t)(bn < N ? bn : N - 1) * (K / 8 * chunk_code_bytes<CF>());
  // this group's steps: kg, kg + KS, ... (the same number for every group;
  // those past K multiply zeros)
  const int nst = (K + KS * 128 - 1) / (KS * 128);
  struct Regs {
    i32x4 a[4];
    Raw64<CF> b;
  };
  auto fetch = [&](int st, Regs& R) {
    const int k = (st * KS + kg) * 128;
    // (past the end of the row: any codes of the row, they meet zero weights)
    const int ka = k + 16 * ac < K ? k + 16 * ac : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) R.a[q] = *reinterpret_cast<const i32x4*>(arow[q] + ka);
    R.b.template load<VEC>(brow, k + 64 * (tid & 1), K);
  };
  // quarter q of step st's operands from registers to LDS
  auto put = [&](Regs& R, int slot, int q) {
    lds_u8* const la = smem + slot * kMidStage;
    lds_u8* const lb = la + MTI * 128;
    *(lds_i32x4*)(la + mid_at((tid >> 3) + 32 * q, ac)) = R.a[q];
    *(lds_i32x4*)(lb + mid_at(tid >> 1, 4 * (tid & 1) + q)) = R.b.template bytes16<E4M3>(q);
  };
  auto mask = [&](int st, Regs& R) {
    if (!VEC || st >= nst - 1) R.b.template mask<VEC>((st * KS + kg) * 128 + 64 * (tid & 1), K);
  };
  Acc acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0;
  // one step from LDS stage `slot`; the next step's operands R go to the
  // other stage between its matrix instructions
  auto compute = [&](int slot, Regs& R) {
    const lds_u8* la = smem + slot * kMidStage + wi * 64 * 128;
    const lds_u8* lb = smem + slot * kMidStage + MTI * 128 + wj * 64 * 128;
    auto rd = [&](const lds_u8* p, int t, int kk) { return *(const lds_i32x4*)(p + mid_at(32 * t + fr, 2 * kk + h)); };
    // (scheduling barriers keep the reads of the next sub-step ahead of the
    // matrix instructions of this one)
    if constexpr (!E4M3) {
      i32x4 fa[2][2], fb[2][2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        fa[0][t] = rd(la, t, 0);
        fb[0][t] = rd(lb, t, 0);
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kk < 3) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            fa[(kk + 1) & 1][t] = rd(la, t, kk + 1);
            fb[(kk + 1) & 1][t] = rd(lb, t, kk + 1);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[kk & 1][b], fa[kk & 1][a], acc[a][b], 0, 0, 0);
        put(R, slot ^ 1, kk);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      auto rd2 = [&](const lds_u8* p, int t, int kk) {
        const i32x4 u = rd(p, t, kk), v = rd(p, t, kk + 1);
        return i32x8{u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
      };
      i32x8 fa[2][2], fb[2][2];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          fa[kk][t] = rd2(la, t, 2 * kk);
          fb[kk][t] = rd2(lb, t, 2 * kk);
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[kk][b], fa[kk][a], acc[a][b], 0, 0, 0, 127, 0, 127);
        put(R, slot ^ 1, 2 * kk);
        put(R, slot ^ 1, 2 * kk + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // LDS stage s mod 2 holds step s; registers hold steps s + 1 and s + 2
  // (past the last step: its operands again, not used, so that no load or
  // store sits behind a branch and the waits stay exact)
  auto fetch_c = [&](int st, Regs& R) { fetch(st < nst ? st : nst - 1, R); };
  Regs R0, R1;
  fetch(0, R0);
  fetch_c(1, R1);
  mask(0, R0);
#pragma unroll
  for (int q = 0; q < 4; ++q) put(R0, 0, q);
  mid_barrier();
  for (int st = 0; st < nst; st += 2) {
    fetch_c(st + 2, R0);
    mask(st + 1, R1);
    compute(0, R1);
    mid_barrier();
    if (st + 1 >= nst) break;
    fetch_c(st + 3, R1);
    mask(st + 2, R0);
    compute(1, R0);
    mid_barrier();
  }
  if constexpr (KS == 2) {
    // the second group's sums through its stages (64 KB) to the first, which
    // adds them and alone goes on; a lane's 64 values 16 bytes at a time
    using Quad = typename Acc4<E4M3>::type;
    __attribute__((address_space(3))) Quad* const ex =
        (__attribute__((address_space(3))) Quad*)((lds_u8*)stages + 2 * kMidStage) + wave * 16 * 64 + lane;
    if (kg == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const Acc& v = acc[i >> 3][(i >> 2) & 1];
        ex[i * 64] = Quad{v[4 * (i & 3)], v[4 * (i & 3) + 1], v[4 * (i & 3) + 2], v[4 * (i & 3) + 3]};
      }
    }
    mid_barrier();
    if (kg == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const Quad w = ex[i * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i >> 3][(i >> 2) & 1][4 * (i & 3) + e] += w[e];
      }
    }
  }
  // Lane (token fr, h) of block (a, b) holds columns 8 (e / 4) + 4 h + e mod 4:
  // the tile goes through LDS (a row at a time, 16-byte chunks XORed with
  // the row) and out in whole 16-byte chunks of output rows.
  float sc[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int m = m0 + wi * 64 + 32 * a + fr;
    sc[a] = L.xdq[m < M ? m : M - 1] * L.alpha;
  }
  const int eb = tab.bf16 ? 2 : 4;
  lds_u8* const out = (lds_u8*)stages;
  if (kg == 0)
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float v0 = (float)acc[a][b][4 * k] * sc[a], v1 = (float)acc[a][b][4 * k + 1] * sc[a];
        const float v2 = (float)acc[a][b][4 * k + 2] * sc[a], v3 = (float)acc[a][b][4 * k + 3] * sc[a];
        const int row = wi * 64 + 32 * a + fr, col = wj * 64 + 32 * b + 8 * k + 4 * h;
        if (tab.bf16) {
          const int c = (col >> 3) ^ (row & 15);
          *(__attribute__((address_space(3))) u32x2*)(out + row * 256 + 16 * c + 2 * (col & 7)) =
              u32x2{pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
        } else {
          const int c = (col >> 2) ^ (row & 31);
          *(__attribute__((address_space(3))) f32x4*)(out + row * 512 + 16 * c) = f32x4{v0, v1, v2, v3};
        }
      }
  mid_barrier();
  const int cpr = MTI * eb / 16;              // chunks per row: 16 (bf16) or 32
  for (int i = threadIdx.x; i < MTI * cpr; i += 256 * KS) {
    const int row = i / cpr, c = i % cpr;
    const int m = m0 + row, n = n0 + c * (16 / eb);
    if (m < M && n < N)
      *reinterpret_cast<i32x4*>(static_cast<uint8_t*>(L.y) + ((int64_t)m * N + n) * eb) =
          *(const lds_i32x4*)(out + row * (MTI * eb) + 16 * (c ^ (row & (cpr - 1))));
  }
}

template <int CF, bool E4M3, int RG, bool VEC>
hipError_t launch_skinny(SmallTab& tab, hipStream_t stream) {
  int32_t blocks = 0;
  for (int s = 0; s < tab.n; ++s) {
    tab.b0[s] = blocks;
    blocks += (tab.p[s].N + 16 * RG - 1) / (16 * RG);
  }
  tab.b0[tab.n] = blocks;
  const dim3 grid((unsigned)blocks), block(64 * kSkW);
  // (8-bit codes come with RG = 1 up to 16 tokens, with RG = 2 for 17 to 48)
  constexpr bool k8 = CF == CF_I8;
  if constexpr (!k8 || RG == 1)
    if (tab.M <= 16) return launch_kernel(fwd_skinny_kernel<CF, E4M3, 1, RG, VEC>, grid, block, stream, tab);
  if constexpr (!k8 || RG > 1) {
    if (tab.M <= 32) return launch_kernel(fwd_skinny_kernel<CF, E4M3, 2, RG, VEC>, grid, block, stream, tab);
    if (tab.M <= 48) return launch_kernel(fwd_skinny_kernel<CF, E4M3, 3, RG, VEC>, grid, block, stream, tab);
  }
  if constexpr (!k8) return launch_kernel(fwd_skinny_kernel<CF, E4M3, 4, RG, VEC>, grid, block, stream, tab);
  return hipErrorInvalidValue;   // (not reached: the rule above)
}

template <int CF, bool E4M3, bool VEC>
hipError_t launch_small_v(SmallTab& tab, hipStream_t stream) {
  return timed_launch(stream, [&] {
    int64_t rows = 0;
    for (int s = 0; s < tab.n; ++s) rows += tab.p[s].N;
    const bool wide = rows >= 2 * 64 * current_device_cus();
    if (tab.M <= (CF != CF_I8 ? kSkinnyM : wide ? kSkinnyM8Wide : kSkinnyM8)) {
      if constexpr (CF == CF_I8) {
        if (tab.M <= 16) return launch_skinny<CF, E4M3, 1, VEC>(tab, stream);
      } else {
        if (wide) return launch_skinny<CF, E4M3, 4, VEC>(tab, stream);
      }
      return launch_skinny<CF, E4M3, 2, VEC>(tab, stream);
    }
    tab.mt = (tab.M + MTI - 1) / MTI;
    for (int s = 0; s < tab.n; ++s) tab.b0[s] = tab.mt * ((tab.p[s].N + MTI - 1) / MTI);
    int32_t per_xcd = 0;
    for (int x = 0; x < 8; ++x) {
      int32_t c = 0;
      for (int s = 0; s < tab.n; ++s) c += (((x + 1) * tab.b0[s]) >> 3) - ((x * tab.b0[s]) >> 3);
      if (c > per_xcd) per_xcd = c;
    }
    const dim3 grid((unsigned)(8 * per_xcd));
    if (tab.M <= kMidSplitM) return launch_kernel(fwd_mid_kernel<CF, E4M3, VEC, 2>, grid, dim3(512), stream, tab);
    return launch_kernel(fwd_mid_kernel<CF, E4M3, VEC, 1>, grid, dim3(256), stream, tab);
  });
}

template <int CF, bool E4M3>
hipError_t launch_small(SmallTab& tab, bool vec, hipStream_t stream) {
  return vec ? launch_small_v<CF, E4M3, true>(tab, stream) : launch_small_v<CF, E4M3, false>(tab, stream);
}

}  // namespace

// The rule.  Up to kSkinnyM tokens the stream of codes is the cost, and the
// skinny kernel's token operand traffic grows with the tokens: at 64 tokens
// it and the mid kernel meet (h4096 ternary 47 and 49 us, h2048 4-bit 28 and
// 32 us, h768 13 and 16 us; h4096 4-bit 61 and 55 us); with 8-bit codes
// at 48 (h2048 29 and 31 us), or 16 where the launch has so many rows that
// the mid kernel fills the chip (h4096: 16 tokens 73 and 70 us, 24 tokens 93
// and 71 us).
// Above, the persistent GEMM's tile takes a step in half the time that four
// tiles of the mid kernel need, but there are a quarter as many of them to
// fill the compute units with, and its codes are expanded first.  Which of
// the two is ahead turns on how full the last round of tiles is (one 4096 ->
// 4096 linear, 8-bit codes: 777 tokens, 64 tiles, 48 against 25 us; 4096
// tokens, 256 tiles, 65 against 91 us), so both are estimated: rounds of tiles
// whose steps slow down as the compute units fill up (bandwidth and clock),
// with constants fitted to 1800 calls of both (one linear to whole blocks,
// d_in 16 to 65536, 65 to 4096 tokens, all formats).  Over those calls the
// choice is at most 3 % slower than the persistent GEMM, and 0.1 % slower than
// the better one on average; limits in tiles or tokens alone were up to 1.7
// times slower where the GEMM's rounds are full.
// The estimates stop where the mid kernel never wins by much: 512 of the 256 x
// 256 tiles (384 with 8-bit codes), 800 tokens with e4m3 activations.
// With e4m3 activations the fp32 sums come out the same on either side above
// kMidSplitM tokens (both add 64 products per instruction, in the same order),
// and a batch gives the results of its linears one by one; the reduction in
// two halves, and the packed form that the persistent GEMM takes without a
// workspace for the expansion, round differently: there the rule is on the
// tokens alone.
static bool codes8(const BatchCfg& c) { return !c.w_ternary && !c.w_int4 && !c.w_int3; }

// us of n tiles in rounds of `slots`: a tile of `steps` takes steps * step *
// (1 + fill * share of the slots taken) + tile, in a round at most half full
// `half` of that; at least as long as the longest tile.
struct TileTime {
  double step, tile, fill, half;
  double round(double steps, double share) const {
    return (steps * step * (1 + fill * share) + tile) * (share <= 0.5 ? half : 1.0);
  }
  double us(int64_t n, int64_t sum_steps, int64_t longest, int64_t slots) const {
    const double mean = (double)sum_steps / (double)n;
    const int64_t rem = n % slots;
    const double t = (double)(n / slots) * round(mean, 1.0) + (rem > 0 ? round(mean, (double)rem / (double)slots) : 0.0);
    return std::max(t, round((double)longest, n < slots ? (double)n / (double)slots : 1.0));
  }
};

static bool mid_is_ahead(const BatchCfg& c, const LinearIO* io) {
  const int64_t cus = current_device_cus();
  const bool split = c.M <= kMidSplitM;
  bool fp4 = c.w_ternary && c.act_e4m3;
  for (int l = 0; l < c.n; ++l) fp4 &= io[l].d_in % 64 == 0;
  int64_t np = 0, sp = 0, lp = 0, nm = 0, sm = 0, lm = 0;
  double weights = 0;
  for (int l = 0; l < c.n; ++l) {
    const int64_t k = io[l].d_in, n = io[l].d_out;
    const int64_t tp = ((c.M + 255) / 256) * ((n + 255) / 256), kp = (k + 127) / 128;
    const int64_t tm = ((c.M + MTI - 1) / MTI) * ((n + MTI - 1) / MTI), km = split ? (k + 255) / 256 : kp;
    np += tp;
    sp += tp * kp;
    lp = std::max(lp, kp);
    nm += tm;
    sm += tm * km;
    lm = std::max(lm, km);
    weights += (double)(k * n);
  }
  // the persistent GEMM, after the pass that expands its codes (4.4 TB/s)
  double big = 7.6 + TileTime{!c.act_e4m3 ? 1.1 : fp4 ? 0.93 : 1.21, 3.4, 0.41, 1.0}.us(np, sp, lp, cus);
  if (!codes8(c)) big += 3.7 + weights * ((c.w_ternary ? 0.25 : c.w_int4 ? 0.5 : 0.375) + (fp4 ? 0.5 : 1.0)) / 4.4e6;
  const double fmt = c.w_ternary ? 0.93 : c.w_int4 ? 1.08 : c.w_int3 ? 1.22 : 1.0;
  const TileTime mid = split ? TileTime{0.87 * fmt, 3.1, 0.46, 1.0} : TileTime{0.78 * fmt, 3.25, 0.46, 0.69};
  return 1.02 * (3.4 + mid.us(nm, sm, lm, split ? cus : 2 * cus)) <= big;
}

bool fwd_small_applies(const BatchCfg& c, const LinearIO* io, bool packed) {
  if (c.M <= kSkinnyM) return true;
  if (c.act_e4m3) {
    if (c.M > kMidMaxE4M3) return false;
    // (the second half of a reduction of at most 128 elements is empty)
    bool halves = false;
    for (int l = 0; l < c.n; ++l) halves |= c.M <= kMidSplitM && io[l].d_in > 128;
    if (packed || halves) return true;
  } else {
    int64_t tiles = 0;
    for (int l = 0; l < c.n; ++l) tiles += ((c.M + 255) / 256) * ((io[l].d_out + 255) / 256);
    if (tiles > (codes8(c) ? kMidMaxTiles8 : kMidMaxTiles)) return false;
  }
  return mid_is_ahead(c, io);
}

hipError_t launch_fwd_small(const BatchCfg& c, const LinearIO* io, hipStream_t stream) {
  SmallTab tab{};
  tab.n = c.n;
  tab.M = (int32_t)c.M;
  tab.bf16 = c.out_bf16;
  bool vec = true;
  for (int l = 0; l < c.n; ++l) {
    // longest reduction first (stable)
    int at = l;
    while (at > 0 && tab.p[at - 1].K < io[l].d_in) {
      tab.p[at] = tab.p[at - 1];
      --at;
    }
    tab.p[at] = SmallLin{static_cast<const uint8_t*>(io[l].Wq), static_cast<const uint8_t*>(io[l].Xq), io[l].xdq,
                         io[l].Y, io[l].alpha, (int32_t)io[l].d_in, (int32_t)io[l].d_out};
    vec &= io[l].d_in % 64 == 0;
  }
  if (c.w_ternary)
    return c.act_e4m3 ? launch_small<CF_T2, true>(tab, vec, stream) : launch_small<CF_T2, false>(tab, vec, stream);
  if (c.w_int4)
    return c.act_e4m3 ? launch_small<CF_I4, true>(tab, vec, stream) : launch_small<CF_I4, false>(tab, vec, stream);
  if (c.w_int3)
    return c.act_e4m3 ? launch_small<CF_I3, true>(tab, vec, stream) : launch_small<CF_I3, false>(tab, vec, stream);
  return launch_small<CF_I8, false>(tab, vec, stream);
}

}  // namespace dqt
