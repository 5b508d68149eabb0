// MFMA GEMM for the int8 / e4m3 / bf16 contractions of the DQT linear step
// (Sec. 3.2), written for gfx950:
//   C[i, j] = sum_r A(i, r) B(j, r)
// Each operand is either K-contiguous (stored [rows][R], the reduction runs
// along a row) or K-major (stored [R][rows], bf16 only).
//
// Design (measured on MI355X):
//  * Block tile 256 x 256, 8 waves in a 2 x 4 grid, each wave 128 x 64 as
//    4 x 2 MFMA 32x32 blocks.  Two waves share each SIMD, so one wave's LDS
//    and barrier waits are covered by the other's matrix instructions.  At
//    this tile size a full-rate MFMA loop needs ~32 B/clk/CU of operands.
//  * Operands move global -> LDS with direct-to-LDS DMA
//    (global_load_lds_dwordx4, no VGPR staging) in steps of one 128-byte
//    cache line per tile row (128 int8 / e4m3 or 64 bf16 reduction
//    elements): streaming whole lines delivers ~35 B/clk/CU, half lines only
//    ~21.  Two stages of 64 KB.  A copy's address is a wave-uniform base in
//    scalar registers plus one 32-bit offset per lane.
//  * Two-phase loop: a step is four quarters of the wave's outputs, each a
//    memory part (fragment reads, then the copies of one half-tile of a
//    later step) and a compute part (8 matrix instructions); the two waves
//    of a SIMD run half a phase apart, so one's memory part always runs
//    beside the other's matrix instructions, and five half-tiles of copies
//    stay in flight.  Bound by the board's power: the matrix cores are busy
//    77 % of the cycles (60 % with all waves in the same phase and the copies
//    in one burst per step), and the clock falls from 1.87 to about 1.6 GHz
//    under it.  Measured, that form -> this: hidden-4096 backward + SR 5.85
//    -> 5.06 ms (1310 TFLOP/s), hidden-2048 3.05 -> 2.70 ms, hidden-768 282
//    -> 263 us; forward hidden-4096 (FP4 x e4m3) 1.41 -> 1.30 ms, hidden-2048
//    int8 908 -> 863 us.  Of that, moving the copies behind the fragment
//    reads gave 4 %, scalar base addresses 8 % (64-bit vector addresses cost
//    issue slots and registers), reading one half-tile of B a step early 1.5
//    %; raised wave priority in the compute part cost 0.5 %.
//  * One-phase loop, for packed codes and for forward tiles of few steps (the
//    rule and both sides' times stand at one_phase()): all waves run the same
//    phase, a step's copies go out in one burst after its barrier, two stages or
//    the three that fit with packed codes and FP4 values.
//  * Persistent grid, one block per CU.  XCD x (workgroups are dispatched
//    round-robin over the 8 XCDs, each with its own L2) owns a contiguous
//    share of every problem's tiles, problems sorted longest reduction first;
//    its blocks take tiles from that list through an atomic counter, so a
//    block that finishes early takes the next one (longest-first list
//    scheduling).  Before a tile's epilogue the
//    block issues the first DMA stage of its next tile, so the load latency
//    hides behind the epilogue.
//  * Fragments come from LDS with ds_read_b128 (K-contiguous) or with the
//    transposing ds_read_b64_tr_b16 (K-major), which hands each lane eight
//    reduction-consecutive bf16 of one row straight from a [R][rows] tile, so
//    dW = dY^T X~ and dX = dY Q need no register transposes.
//
// LDS layouts (per stage, per operand), free of bank conflicts for the
// fragment reads:
//   K-contiguous: [256 rows][128 B]; 16-byte chunk c of row r sits at
//     position c ^ ((r >> 1) & 7).
//   K-major (bf16): four 64-column regions, each [64 reduction rows][128 B];
//     the 32-byte segment s of row k sits at position s ^ (k & 3).
// Each DMA wave instruction fills 1 KB of consecutive LDS positions, so each
// lane loads the global chunk that belongs at its position.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "gemm_common.h"
#include "sr_rule.h"

namespace dqt {
namespace v3 {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int NW = 8;                 // waves per block: a 2 x 4 grid
constexpr int NTH = 64 * NW;
constexpr int NTD = NTH;             // threads issuing global -> LDS copies
constexpr int TILE = 256;             // block tile edge (outputs)
constexpr int WI = 4;                 // MFMA 32x32 blocks per wave along rows
constexpr int WJ = 2;                 // ... and along columns
constexpr int WGC = TILE / (32 * WJ); // waves per row of the wave grid
// Step geometry: KB reduction bytes per tile row per step (one cache line).
// K-contiguous tiles are [256 rows][KB bytes]; K-major (bf16) tiles are KR
// reduction rows of 256 columns, stored as four 64-column regions.  Packed
// ternary codes are PKB bytes per row per step (four codes a byte).
constexpr int KB = 128;
constexpr int PKB = KB / 4;
struct Geo {
  static constexpr int OPB = TILE * KB;       // bytes per operand per stage
  static constexpr int NL = OPB / 16 / NTD;   // DMA chunks per thread per operand
  static constexpr int CPR = KB / 16;         // K-contiguous 16-byte chunks per row
  static constexpr int KR = KB / 2;           // K-major rows per step
  // K-contiguous swizzle: chunk c of row r sits at c ^ swz(r) (conflict-free
  // ds_read_b128)
  __device__ static int swz(int r) { return (r >> 1) & 7; }
};


// EF4B: e4m3 A with ternary B as FP4 (E2M1) values formed from the packed
// codes in registers (B must be packed codes)
enum Elem { EI8 = 0, EF8 = 1, EBF16 = 2, EF4B = 3 };
// KCP: K-contiguous packed ternary codes (B only); KF4: K-contiguous FP4
// (E2M1) values, two per byte (B only, with e4m3 A), expanded from the codes
// by a pass into the workspace
enum Mode { KC = 0, KM = 1, KCP = 2, KF4 = 3 };

// bytes per stage: A, then B (bf16 / 8-bit operand, FP4 values or packed codes)
template <int MB>
constexpr int slot_bytes() { return Geo::OPB + (MB == KCP ? TILE * PKB : MB == KF4 ? TILE * KB / 2 : Geo::OPB); }


// Global operand: base of element (row 0, reduction 0), row stride in bytes,
// extent of the tile dimension.
struct Opnd {
  const uint8_t* p;
  int64_t ld;
  int64_t n;
};

// One GEMM problem of a grouped launch: nbx x nby x nbz tiles (column tiles,
// row tiles, reduction splits).
template <class Epi>
struct Prob {
  Opnd A, B;
  Epi epi;
  int64_t I, J, R, split_len;
  int32_t nbx, nby, nbz, ntiles;
  int32_t xb[9];               // XCD x owns tiles xb[x] .. xb[x + 1] - 1
};
constexpr int MAXG = 8;
template <class Epi>
struct Group {
  Prob<Epi> p[MAXG];
  int32_t ng;
  // tile counters: sched[x] is the next tile of XCD x's list to hand out
  int* sched;
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
// Transposing LDS read: each lane receives four 16-bit values of one column
// from four consecutive rows of a row-major tile (ds_read_b64_tr_b16).
__device__ __forceinline__ u32x2 tr_read(const lds_u8* base, int off) {
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(base + off));
  return __builtin_bit_cast(u32x2, v);
}
__device__ __forceinline__ i32x4 join(u32x2 lo, u32x2 hi) {
  return i32x4{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
}
// 16 packed ternary codes (code q + 1 at bits 2k) -> 16 FP4 (E2M1) values,
// value k in nibble k of the 64-bit result (low nibble of each byte first):
// q = -1 -> 0xA (-1.0), 0 -> 0x0, +1 -> 0x2 (+1.0).  Each 8-code half: its
// two bytes to bytes 0 and 2, their nibbles to bytes 0..3, the 2-bit codes
// to nibbles; then nibble = (code bit 1) * 2 + (code == 0) * 0xA.
__device__ __forceinline__ u32x2 expand16_fp4(uint32_t x) {
  auto half = [](uint32_t v) {
    v = (v | (v << 4)) & 0x0F0F0F0Fu;
    const uint32_t u = v | (v << 2);             // codes at nibble bits 0-1 (bits 2-3: junk)
    const uint32_t z = ~u & ~(u >> 1) & 0x11111111u;
    const uint32_t w = z | (z << 2);
    return (u & 0x22222222u) | (w << 1);
  };
  return u32x2{half(__builtin_amdgcn_perm(0u, x, 0x0C010C00u)), half(__builtin_amdgcn_perm(0u, x, 0x0C030C02u))};
}
// Barrier that keeps the compiler from moving memory accesses across it; it
// waits for this wave's LDS accesses but not for outstanding DMA.
__device__ __forceinline__ void block_barrier() {
  __asm__ volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((15) | (3 << 14) | (7 << 4) | (0 << 8));   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
}

// The value x, hidden from the optimiser: per-lane indices derived from it
// are recomputed where they are used instead of being hoisted out of the
// tile loop, where they would hold registers across the main loop.
__device__ __forceinline__ int opaque(int x) {
  __asm__ volatile("" : "+v"(x));
  return x;
}

// Per-thread DMA plan of one operand of one tile (the one-phase loop): the
// global address of each of its NL chunks at step 0; the reduction offset
// (elements, within a step) the chunks cover, which is the same for all of
// them; and the distance back from a chunk's address to a safe one in the
// same row for loads past the end of the reduction.
template <int MODE, int EB>
struct Plan {
  using G = Geo;
  static constexpr int CH = TILE * PKB / 16;   // packed 16-byte chunks per stage
  static constexpr int NL = MODE == KCP ? CH / NTD : MODE == KF4 ? G::NL / 2 : G::NL;
  static_assert(CH % NTD == 0, "every thread copies packed codes");
  const uint8_t* g[NL];
  int64_t back;
  int64_t inc;
  int rk;

  __device__ void init(const Opnd& o, int64_t row0, int64_t r_begin, int tid) {
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int p = q * NTD + tid;                  // physical 16-byte position
      if constexpr (MODE == KCP) {
        // 32-byte rows: two chunks of 64 codes, swapped on odd groups of 8 rows
        const int row = p >> 1;
        const int c = (p & 1) ^ ((row >> 3) & 1);
        int64_t gr = row0 + row;
        if (gr > o.n - 1) gr = o.n - 1;
        g[q] = o.p + gr * o.ld + r_begin / 4 + 16 * c;
        back = r_begin / 4 + 16 * c;
        rk = 64 * c;
      } else if constexpr (MODE == KF4) {
        // rows of 64 bytes: chunk c of row r at position c ^ ((r >> 2) & 3)
        const int row = p >> 2;
        const int c = (p & 3) ^ ((row >> 2) & 3);
        int64_t gr = row0 + row;
        if (gr > o.n - 1) gr = o.n - 1;
        g[q] = o.p + gr * o.ld + r_begin / 2 + 16 * c;
        back = r_begin / 2 + 16 * c;
        rk = 32 * c;
      } else {
        const int row = p / G::CPR;
        const int c = (p % G::CPR) ^ G::swz(row);   // logical chunk (same for every q)
        int64_t gr = row0 + row;
        if (gr > o.n - 1) gr = o.n - 1;
        g[q] = o.p + gr * o.ld + r_begin * EB + 16 * c;
        back = r_begin * EB + 16 * c;
        rk = 16 * c / EB;
      }
    }
    inc = MODE == KC ? KB : MODE == KF4 ? KB / 2 : PKB;
  }
};

// Copy plan of one operand of the two-phase loop (kPP): a wave's copy q
// moves 8 rows (K-contiguous; 8 reduction rows of 64 columns when K-major) of
// 128 bytes, so its address is a wave-uniform base, kept in scalar registers,
// plus a 32-bit offset per lane, within 8 rows.  B32: copies q = 2 j + u
// cover the rows whose bit 5 is j (the waves' column block j); such an
// operand's rows are weights' rows, a multiple of 16, so a copy's rows are
// all inside or all outside and one offset serves every copy.
template <int MODE, int EB, bool B32>
struct PPlan {
  static_assert(MODE == KC || MODE == KM || (MODE == KF4 && B32), "operands of the two-phase loop");
  static constexpr int NV = B32 && MODE != KM ? 1 : 4;
  static constexpr int NB = MODE == KC ? 4 : MODE == KF4 ? 2 : 1;
  const uint8_t* b[NB];
  int64_t inc;
  uint32_t vo[NV];
  __device__ static int row_of(int q, int w) {       // first row of copy q of wave w
    return B32 ? 64 * (2 * (q & 1) + (w >> 2)) + 32 * (q >> 1) + 8 * (w & 3) : 64 * q + 8 * w;
  }
  // position of this lane's 16 bytes in its row (K-contiguous) and its row
  __device__ static int chunk(int w, int lane) { return (lane & 7) ^ Geo::swz(8 * w + (lane >> 3)); }
  // first row (K-contiguous) of copy q, inside the operand
  __device__ static int64_t first_row(const Opnd& o, int64_t row0, int q, int w) {
    const int64_t gr = row0 + (MODE == KF4 ? 64 * (w >> 1) + 32 * q + 16 * (w & 1) : row_of(q, w));
    const int64_t last = MODE == KF4 ? o.n - 16 : B32 ? o.n - 8 : o.n - 1;
    return gr < last ? gr : last;
  }
  // this lane's distance from copy q's base (init has it in 32 bits)
  __device__ static int64_t lane_off(const Opnd& o, int64_t row0, int q, int w, int lane) {
    if constexpr (MODE == KC) {
      const int64_t rest = o.n - 1 - first_row(o, row0, q, w);   // rows of the copy past its first
      const int64_t r = B32 || (lane >> 3) < rest ? lane >> 3 : rest;
      return r * o.ld + 16 * chunk(w, lane);
    } else if constexpr (MODE == KF4) {
      // rows of 64 bytes: copy j moves 16 rows of the waves' column block j
      return (lane >> 2) * o.ld + 16 * chunk4(lane);
    } else {
      const int pc = lane & 7, k = lane >> 3;
      int64_t col = row0 + 64 * q + 16 * ((pc >> 1) ^ (k & 3)) + 8 * (pc & 1);
      if (col > o.n - 8) col = o.n - 8;
      return k * o.ld + 2 * (col - row0);
    }
  }
  // 32 bits hold every lane's distance (16 rows) below this row stride;
  // wider operands take 64-bit addresses at every step
  __device__ static bool wide(const Opnd& o) { return o.ld >= (int64_t)1 << 27; }
  __device__ void init(const Opnd& o, int64_t row0, int64_t r_begin, int w, int lane) {
    inc = MODE == KC ? KB : MODE == KF4 ? KB / 2 : Geo::KR * o.ld;
    if constexpr (MODE == KM) {
      b[0] = o.p + (r_begin + 8 * w) * o.ld + 2 * row0;
      // (columns from the tile's first: at most 256 of them)
      const int last = (int)(o.n - 8 - row0 < TILE ? o.n - 8 - row0 : TILE);
      const int pc = lane & 7, k = lane >> 3;
      const uint32_t at = (uint32_t)k * (uint32_t)o.ld;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int col = 64 * q + 16 * ((pc >> 1) ^ (k & 3)) + 8 * (pc & 1);
        vo[q] = at + 2u * (uint32_t)(col < last ? col : last);
      }
    } else {
      int64_t fr[4];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        fr[q] = first_row(o, row0, q, w);
        b[q] = o.p + fr[q] * o.ld + (MODE == KF4 ? r_begin / 2 : r_begin * EB);
      }
      if constexpr (NV == 1) {
        vo[0] = MODE == KF4 ? (uint32_t)(lane >> 2) * (uint32_t)o.ld + 16u * (uint32_t)chunk4(lane)
                            : (uint32_t)(lane >> 3) * (uint32_t)o.ld + 16u * (uint32_t)chunk(w, lane);
      } else {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          const int rest = (int)(o.n - 1 - fr[q] < 7 ? o.n - 1 - fr[q] : 7);
          const int r = (lane >> 3) < rest ? lane >> 3 : rest;
          vo[q] = (uint32_t)r * (uint32_t)o.ld + 16u * (uint32_t)chunk(w, lane);
        }
      }
    }
  }
  // reduction element (within the step) of this lane's chunk, and what takes
  // its address back to reduction element 0 of the step
  __device__ static int chunk4(int lane) { return (lane & 3) ^ ((lane >> 4) & 3); }
  __device__ static int rk(int w, int lane) {
    return MODE == KC ? 16 * chunk(w, lane) / EB : MODE == KF4 ? 32 * chunk4(lane) : 8 * w + (lane >> 3);
  }
  __device__ static int64_t back(int rk, int64_t ld) { return MODE == KC ? rk * EB : MODE == KF4 ? rk / 2 : rk * ld; }
  __device__ const uint8_t* base(int q, int s) const { return b[q < NB ? q : 0] + (int64_t)s * inc; }
  __device__ uint32_t off(int q) const { return vo[q < NV ? q : 0]; }
};

// Tile order within one problem: reduction split bz outermost; within a
// split, bands of kGroupRows tile rows, and within a band column by column
// (problems more than 8 tiles wide; narrower ones stay row-major).  An XCD
// owns a contiguous run of this order, so the 32 tiles its compute units
// hold at once span about 4 tile rows and 8 tile columns, where row-major
// order would span 1-2 rows and 16-32 columns: they share more of their
// operand panels in the XCD's L2 (12 panels per step instead of 18; hidden
// 4096 block: forward -2 %, backward + SR -1.5 %).
constexpr int kGroupRows = 4;
__host__ __device__ __forceinline__ void tile_coords(int local, int nbx, int nby, int& bx, int& by,
                                                     int& bz) {
  const int per_z = nbx * nby;
  bz = local / per_z;
  const int r = local - bz * per_z;
  const int gr = nbx > 8 ? kGroupRows : 1;
  const int band = r / (gr * nbx);
  const int in = r - band * (gr * nbx);
  const int rows = nby - band * gr < gr ? nby - band * gr : gr;
  by = band * gr + in % rows;
  bx = in / rows;
}

// Tile j of XCD x's list: its tiles of every problem, problems in launch
// order.  False past the end.
template <class Epi>
__device__ __forceinline__ bool locate(const Group<Epi>& grp, int x, int j, int& g, int& local) {
  for (g = 0; g < grp.ng; ++g) {
    const int s0 = grp.p[g].xb[x], cnt = grp.p[g].xb[x + 1] - s0;
    if (j < cnt) {
      local = s0 + j;
      return true;
    }
    j -= cnt;
  }
  return false;
}

using lds_f32 = __attribute__((address_space(3))) float;
using lds_u32 = __attribute__((address_space(3))) uint32_t;
using lds_i32 = __attribute__((address_space(3))) int;

// Stage geometry of one instantiation: bytes per stage and stages (two, or
// in the one-phase loop the three that fit with packed codes or FP4 values).
template <int MB, bool ONE>
struct StageGeo {
  static constexpr int SLOTB = slot_bytes<MB>();
  static constexpr int NS = ONE && MB != KC ? 3 : 2;
  static constexpr int kBytes = NS * SLOTB;
};
static_assert(StageGeo<KCP, true>::kBytes + TILE * 4 + 16 <= 160 * 1024, "stages fit in LDS");
static_assert(StageGeo<KF4, true>::kBytes + TILE * 4 + 16 <= 160 * 1024, "stages fit in LDS");

// The persistent grouped GEMM over the tiles of `grp`, with its LDS passed
// in (stages, 256 row factors, the next-tile slot), so that two groups can
// run one after the other in one launch.  ONE: the one-phase loop, where all
// waves run the same phase and a step's copies go out in one burst, for packed
// codes and for tiles of few steps (one_phase() has the rule).
template <int ELEM, int MA, int MB, class Epi, bool ONE = MB == KCP>
__device__ __forceinline__ void gemm_v3_body(const Group<Epi>& grp, lds_u8* smem, lds_f32* row_scale,
                                             lds_i32* next_tile_p) {
  using G = Geo;
  constexpr int EB = ELEM == EBF16 ? 2 : 1;
  constexpr int BK = KB / EB;               // reduction elements per step
  constexpr int OPB = G::OPB;
  constexpr int NL = G::NL;
  constexpr int SLOTB = StageGeo<MB, ONE>::SLOTB;
  constexpr int NS = StageGeo<MB, ONE>::NS;
  static_assert(NW * 32 * 128 <= SLOTB, "epilogue staging (32 rows of 128 bytes per wave) fits in one stage");
  constexpr bool kPP = !ONE;
  constexpr int CB = MB == KF4 ? 1 : 2;     // copies per wave of a half-tile of B
  static_assert(!kPP || MB != KCP, "packed codes are expanded in the one-phase loop");
  static_assert(kPP || (MA == KC && ELEM != EBF16), "8-bit activations in the one-phase loop");
  static_assert(MB == KF4 || MB == KCP || ELEM != EF4B, "FP4 B comes from ternary codes");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int wi = wave_u / WGC, wj = wave_u % WGC;
  const int h = lane >> 5;
  const int xcd = blockIdx.x & 7;

  // ---- state of the tile being computed
  struct TileState {
    int g;
    int64_t i0, j0, rlen;
    int bz, nsteps;
    bool tail, wide;
  };
  std::conditional_t<kPP, PPlan<MA, EB, false>, Plan<KC, EB>> pa;
  std::conditional_t<kPP, PPlan<kPP ? MB : KC, EB, true>, Plan<MB, EB>> pb;
  TileState cur;
  float my_scale = 0.0f;

  auto setup = [&](int g, int local, TileState& T) {
    const Prob<Epi>& P = grp.p[g];
    int bx, by, bz;
    tile_coords(local, P.nbx, P.nby, bx, by, bz);
    T.g = g;
    T.i0 = (int64_t)by * TILE;
    T.j0 = (int64_t)bx * TILE;
    T.bz = bz;
    const int64_t r_begin = (int64_t)bz * P.split_len;
    int64_t r_end = r_begin + P.split_len;
    if (r_end > P.R) r_end = P.R;
    T.rlen = r_end > r_begin ? r_end - r_begin : 0;
    T.nsteps = (int)((T.rlen + BK - 1) / BK);
    T.tail = (T.rlen % BK) != 0;
    T.wide = false;
    const int tid_s = opaque(tid);
    if constexpr (kPP) {
      T.wide = pa.wide(P.A) || pb.wide(P.B);
      pa.init(P.A, T.i0, r_begin, wave_u, tid_s & 63);
      pb.init(P.B, T.j0, r_begin, wave_u, tid_s & 63);
    } else {
      pa.init(P.A, T.i0, r_begin, tid_s);
      pb.init(P.B, T.j0, r_begin, tid_s);
    }
    if constexpr (Epi::kRowScale) {
      if (tid < TILE) {
        int64_t i = T.i0 + tid;
        if (i > P.I - 1) i = P.I - 1;
        my_scale = P.epi.scale_raw(i);     // used only in the epilogue
      }
    }
  };

  // (one-phase loop) DMA of step s of the current plans into stage `slot`
  auto issue = [&](int s, int slot, const TileState& T) {
    if constexpr (!kPP) {
      constexpr int NL = decltype(pa)::NL, NLB = decltype(pb)::NL;
      lds_u8* la = smem + slot * SLOTB + wave_u * 1024;
      lds_u8* lb = la + OPB;
      // (a chunk past the end of the reduction loads the first of its row)
      int64_t da = (int64_t)s * pa.inc, db = (int64_t)s * pb.inc;
      if (T.tail && s == T.nsteps - 1) {
        const int left = (int)(T.rlen - (int64_t)s * BK);
        if (pa.rk >= left) da = -pa.back;
        if (pb.rk >= left) db = -pb.back;
      }
#pragma unroll
      for (int q = 0; q < NL; ++q) dma16(pa.g[q] + da, la + q * (NTD * 16));
#pragma unroll
      for (int q = 0; q < NLB; ++q) dma16(pb.g[q] + db, lb + q * (NTD * 16));
    }
  };
  // Half-tiles of a step (kPP): 0: A rows whose bit 6 is 0, 1: B columns of
  // the waves' first column block, 2: of their second, 3: A rows whose bit 6
  // is 1.  Two copies per wave each: chunk index and place of copy u.
  auto half_q = [&](int w, int u) { return w == 0 || w == 3 ? (w == 3) + 2 * u : CB * (w == 2) + u; };
  auto half_dst = [&](int w, int u, int slot) {
    lds_u8* const st = smem + slot * SLOTB;
    if (w == 0 || w == 3) return st + half_q(w, u) * (NTD * 16) + wave_u * 1024;
    if (MB == KM) return st + OPB + half_q(w, u) * (NTD * 16) + wave_u * 1024;
    if (MB == KF4) return st + OPB + (wave_u >> 1) * 4096 + (w == 2 ? 2048 : 0) + (wave_u & 1) * 1024;
    return st + OPB + u * 16384 + (wave_u >> 2) * 8192 + (w == 2 ? 4096 : 0) + (wave_u & 3) * 1024;
  };
  // Copy u of half-tile w of step s.  maybe_tail: the step may end past the
  // reduction; lanes past it then load the step's first chunk of their row
  // (or its first reduction row), which is inside.
  auto issue_copy = [&](int w, int u, int s, int slot, const TileState& T, auto maybe_tail) {
    if constexpr (kPP) {
    const bool is_a = w == 0 || w == 3;
    const int q = half_q(w, u);
    const uint8_t* const b = is_a ? pa.base(q, s) : pb.base(q, s);
    if constexpr (decltype(maybe_tail)::value) {
      if (T.wide || (T.tail && s == T.nsteps - 1)) {
        const int lane_s = opaque(lane);
        const Opnd& o = is_a ? grp.p[T.g].A : grp.p[T.g].B;
        const int rk = is_a ? pa.rk(wave_u, lane_s) : pb.rk(wave_u, lane_s);
        const int64_t back = is_a ? pa.back(rk, o.ld) : pb.back(rk, o.ld);
        const int64_t off = is_a ? pa.lane_off(o, T.i0, q, wave_u, lane_s) : pb.lane_off(o, T.j0, q, wave_u, lane_s);
        dma16(b + off - ((int64_t)s * BK + rk >= T.rlen ? back : 0), half_dst(w, u, slot));
        return;
      }
    }
    dma16s(b, is_a ? pa.off(q) : pb.off(q), half_dst(w, u, slot));
    }
  };
  auto issue_half = [&](int w, int s, int slot, const TileState& T) {
    issue_copy(w, 0, s, slot, T, std::true_type{});
    if (w == 0 || w == 3 || CB == 2) issue_copy(w, 1, s, slot, T, std::true_type{});
  };
  auto zero_half = [&](int w, int s, int slot, const TileState& T) {
    // (FP4 values past the end need no zeroing: they meet zeroed A, and FP4
    // has no NaN and no infinity)
    if constexpr (kPP) {
    if (MB == KF4 && (w == 1 || w == 2)) return;
    const int left = (int)(T.rlen - (int64_t)s * BK);   // whole steps aside, elements of the last one
    const int lane_s = opaque(lane);
    const i32x4 z = {0, 0, 0, 0};
    const int rk = w == 0 || w == 3 ? pa.rk(wave_u, lane_s) : pb.rk(wave_u, lane_s);
    if (rk >= left) {
#pragma unroll
      for (int u = 0; u < 2; ++u) *(__attribute__((address_space(3))) i32x4*)(half_dst(w, u, slot) + lane_s * 16) = z;
    }
    }
  };
  // (one-phase loop) zero the chunks of A this thread loaded past the end of
  // the reduction (its own DMA for that stage has completed); the weights
  // there need no zeroing: they meet zeroed A, and hold no NaN or infinity
  auto zero_tail = [&](int s, int slot, const TileState& T) {
    if constexpr (!kPP) {
      lds_u8* la = smem + slot * SLOTB;
      const i32x4 z = {0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < decltype(pa)::NL; ++q)
        if ((int64_t)s * BK + pa.rk >= T.rlen) *(__attribute__((address_space(3))) i32x4*)(la + (q * NTD + tid) * 16) = z;
    }
  };

  // first column of this wave's column block t: the two blocks are adjacent,
  // or (K-major B, whose halves are 128 columns) 128 apart
  auto col_of = [&](int t) { return MB == KM ? 128 * t + 32 * wj : wj * 32 * WJ + t * 32; };
  using AccV = typename AccT<ELEM == EI8 ? Mfma::I8 : Mfma::BF16>::type;
  AccV acc[WI][WJ];

  // fragment address parts
  const int frow = lane & 31;
  const int t4 = (lane >> 2) & 3, u4 = lane & 3, ch = (lane >> 4) & 1;

  // (one-phase loop) Fragments of one reduction sub-step kk (0..3; 32 bytes of
  // reduction per tile row).  pq, with packed codes: this lane's 16-byte half
  // of each B row (64 codes, read once per step; sub-step kk in word kk).  Lane
  // half h then
  // takes reduction elements 64 h .. 64 h + 63 of the step, sub-step kk the 16
  // from 64 h + 16 kk, and its A chunks follow the same order: chunk 4 h + kk
  // instead of 2 kk + h.  (One 16-byte read per row half is free of bank
  // conflicts; four 4-byte reads of words 2 kk + h, all lanes at one word
  // offset in 32-byte rows, conflicted 4-way and cost the e4m3 forward 9 %.)
  struct Frags {
    i32x4 fa[WI], fb[WJ];
    uint32_t pb[WJ];          // packed codes (16 per lane), expanded at use
  };
  auto read_frags = [&](const lds_u8* la, int kk, Frags& F, const i32x4* pq) {
#pragma unroll
    for (int t = 0; t < WI; ++t) {
      const int row = wi * 32 * WI + t * 32 + frow;
      const int c = (MB == KCP ? 4 * h + kk : 2 * kk + h) ^ G::swz(row);
      F.fa[t] = *(const __attribute__((address_space(3))) i32x4*)(la + row * KB + 16 * c);
    }
    const lds_u8* const lb = la + OPB;
#pragma unroll
    for (int t = 0; t < WJ; ++t) {
      const int row = wj * 32 * WJ + t * 32 + frow;
      if constexpr (MB == KCP) {
        F.pb[t] = (uint32_t)pq[t][kk];
      } else if constexpr (MB == KF4) {
        // sub-step pair kk / 2: lane half h takes the row's 32 values from
        // 64 (kk / 2) + 32 h, which its e4m3 partner lanes pair them with
        if ((kk & 1) == 0)
          F.fb[t] = *(const __attribute__((address_space(3))) i32x4*)(lb + row * 64 + 16 * ((kk + h) ^ ((row >> 2) & 3)));
      } else {
        F.fb[t] = *(const __attribute__((address_space(3))) i32x4*)(lb + row * KB + 16 * ((2 * kk + h) ^ G::swz(row)));
      }
    }
  };
  // MFMAs of one sub-step (int8), or of two (e4m3, whose instruction reduces
  // 64 elements: sub-step pairs (0, 1) and (2, 3)).
  auto mfma1 = [&](const Frags& F) {
    if constexpr (!kPP && ELEM == EI8) {
#pragma unroll
      for (int ta = 0; ta < WI; ++ta)
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb) {
          const i32x4 b = MB == KCP ? expand16(F.pb[tb], 0x000100FFu) : F.fb[tb];
          acc[ta][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b, F.fa[ta], acc[ta][tb], 0, 0, 0);
        }
    }
  };
  auto mfma2 = [&](const Frags& F0, const Frags& F1) {
    if constexpr (!kPP && ELEM != EI8) {
#pragma unroll
      for (int ta = 0; ta < WI; ++ta)
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb) {
          const i32x4 a0 = F0.fa[ta], a1 = F1.fa[ta];
          const i32x8 av = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
          if constexpr (MB == KC) {
            const i32x4 b0 = F0.fb[tb], b1 = F1.fb[tb];
            const i32x8 bv = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
            acc[ta][tb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bv, av, acc[ta][tb], 0, 0, 0, 127, 0, 127);
            continue;
          }
          if constexpr (MB == KF4) {
            const i32x4 f = F0.fb[tb];
            const i32x8 bv4 = {f[0], f[1], f[2], f[3], 0, 0, 0, 0};
            acc[ta][tb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bv4, av, acc[ta][tb], 4, 0, 0, 127, 0, 127);
            continue;
          }
          // B as FP4 (format 4: 32 values in the first four registers), A
          // e4m3 (format 0), unit E8M0 scales (127 = 2^0).  With FP4 the
          // first operand's lane half h holds reduction elements 16 h ..
          // 16 h + 15 and 32 + 16 h .. 32 + 16 h + 15 of the instruction
          // (the e4m3 operand: 32 h .. 32 h + 31).  The A chunks cover
          // elements 64 h' + 32 m .. + 31 of the step (m: the sub-step
          // pair), so half h takes the codes of word 2 m + h from both lane
          // halves: one swap of the halves' upper and lower lanes gives
          // them (lanes 0-31 keep their word 2 m and get word 2 m of lanes
          // 32-63, which keep word 2 m + 1 and get that of lanes 0-31).
          const auto sw = __builtin_amdgcn_permlane32_swap(F0.pb[tb], F1.pb[tb], false, false);
          const u32x2 f0 = expand16_fp4(sw[0]), f1 = expand16_fp4(sw[1]);
          const i32x8 bv4 = {(int)f0[0], (int)f0[1], (int)f1[0], (int)f1[1], 0, 0, 0, 0};
          acc[ta][tb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bv4, av, acc[ta][tb], 4, 0, 0, 127, 0, 127);
        }
    }
  };
  auto stage_ptr = [&](int slot) { return smem + slot * SLOTB; };

  // ---- persistent loop over this block's tiles (the counters were cleared
  // on the stream before this launch: by its pre-pass, or sched_clear_kernel)
  lds_i32& next_tile = *next_tile_p;
  int* const next_ctr = grp.sched + xcd;
  if (tid == 0) next_tile = atomicAdd(next_ctr, 1);
  __syncthreads();
  int g0, local0;
  if (!locate(grp, xcd, next_tile, g0, local0)) return;
  setup(g0, local0, cur);
  // Stage of step s of the current tile: (slot0 + s) mod NS.  Before a tile
  // starts, its steps 0 .. NS-2 are in flight.
  int slot0 = 0;
  auto prefetch = [&](int slot) {
    if constexpr (kPP) {
      if (cur.nsteps > 0) {
#pragma unroll
        for (int w = 0; w < 4; ++w) issue_half(w, 0, slot, cur);
      }
    } else {
      for (int s = 0; s < NS - 1 && s < cur.nsteps; ++s) issue(s, (slot + s) % NS, cur);
    }
  };
  prefetch(0);

  // (one-phase loop) One step from stage `slot`: sub-step kk+1's fragments load
  // while kk's MFMAs run (e4m3: sub-steps are consumed in pairs); mid() comes
  // after the first group of MFMAs.
  auto compute = [&](int slot, auto&& mid) {
    const lds_u8* la = stage_ptr(slot);
    const lds_u8* lb = la + OPB;
    // (the DMA stores logical 16-byte half c of row r at half c ^ ((r >> 3) & 1))
    i32x4 pq[WJ];
    if constexpr (MB == KCP) {
#pragma unroll
      for (int t = 0; t < WJ; ++t) {
        const int row = wj * 32 * WJ + t * 32 + frow;
        pq[t] = *(const __attribute__((address_space(3))) i32x4*)(lb + row * PKB + 16 * (h ^ ((row >> 3) & 1)));
      }
    }
    Frags F0, F1;
    if constexpr (ELEM == EI8) {
      // (scheduling barriers keep each group of reads ahead of the MFMAs that
      // precede their use; left alone, the compiler sinks every read next to
      // its first use and exposes the LDS latency)
      read_frags(la, 0, F0, pq);
      read_frags(la, 1, F1, pq);
      __builtin_amdgcn_sched_barrier(0);
      mfma1(F0);
      __builtin_amdgcn_sched_barrier(0);
      mid();
      __builtin_amdgcn_sched_barrier(0);
      read_frags(la, 2, F0, pq);
      __builtin_amdgcn_sched_barrier(0);
      mfma1(F1);
      __builtin_amdgcn_sched_barrier(0);
      read_frags(la, 3, F1, pq);
      __builtin_amdgcn_sched_barrier(0);
      mfma1(F0);
      __builtin_amdgcn_sched_barrier(0);
      mfma1(F1);
    } else {
      // (e4m3 keeps the compiler's own order: a pair of sub-steps per
      // instruction leaves no registers for a further pair in flight)
      Frags F2, F3;
      read_frags(la, 0, F0, pq);
      read_frags(la, 1, F1, pq);
      read_frags(la, 2, F2, pq);
      mfma2(F0, F1);
      mid();
      read_frags(la, 3, F3, pq);
      mfma2(F2, F3);
    }
  };

  // vector stores one thread issues in an epilogue (every chunk is stored;
  // chunks outside the output go to a dummy slot in the workspace)
  constexpr int kStoresBf16 = WI * 32 * (32 * WJ * 2 / 16) / 64;
  constexpr int kStoresF32 = WI * 32 * (32 * WJ * 4 / 16) / 64;
  constexpr int kStoresSR = WI * WJ * 2;      // two 8-weight code chunks per 32 x 32 block
  // the wave's vmcnt counts at most 63 operations in flight (the wave waits
  // at issue beyond that), so "at most 63 newer" is a correct, if
  // conservative, wait when more were issued
  constexpr int kVmMax = 63;
  uint8_t* const dummy = reinterpret_cast<uint8_t*>(grp.sched) + 128;
  bool first_tile = true;
  int stores_prev = 0;                 // stores per thread of the previous epilogue
  // SR epilogue: changed and non-finite counts of each wave, kept in LDS
  // (the row-scale area, which that epilogue does not use) so that nothing
  // extra stays live in registers across the main loop
  lds_u32* const sr_cnt = (lds_u32*)row_scale;
  if constexpr (Epi::kSR) {
    if (lane == 0) {
      sr_cnt[2 * wave_u] = 0;
      sr_cnt[2 * wave_u + 1] = 0;
    }
  }
  int fetched = 0;                     // thread 0: index of the next tile
  // The main loop of kPP: a step's 128 x 64 outputs per wave as four quarters
  // (64 rows x 32 columns: A half x B half), each a phase of
  //   memory: fragments of the half-tile the quarter needs new, copies of one
  //           half-tile of a later step, the wait for a half-tile needed next;
  //   compute: 8 matrix instructions.
  // The second four waves (each shares its SIMD with one of the first four)
  // run one half-phase behind, so on every SIMD one wave's memory part always
  // runs beside the other's matrix instructions, and the copies are spread
  // over the step, five half-tiles (80 KB) in flight.
  auto pp_loop = [&]() {
    const int n = cur.nsteps;
    if (n == 0) return;
    const bool g2 = wave_u >= NW / 2;
    {
      // step 0's copies were issued before the previous epilogue's stores
      if (first_tile) wait_vm<0>();
      else if (Epi::kSR) wait_vm<kStoresSR>();
      else if (stores_prev == kStoresBf16) wait_vm<kStoresBf16>();
      else wait_vm<kStoresF32 < kVmMax ? kStoresF32 : kVmMax>();
      first_tile = false;
    }
    if (cur.tail && n == 1) {
#pragma unroll
      for (int w = 0; w < 4; ++w) zero_half(w, 0, slot0, cur);
    }
    block_barrier();                   // step 0 complete; the other stage is free
    if (n > 1) {
#pragma unroll
      for (int w = 0; w < 3; ++w) issue_half(w, 1, slot0 ^ 1, cur);
    }
    // (opaque: for an address known to be the same in every lane the compiler
    // combines the lanes' adds and waits for the result on the spot, which
    // held the whole tile until its predecessor's stores were out: dW alone of
    // the hidden-2048 block at 128 tokens 59 us, 51 without; with the SR update
    // the wait is the faster form, 4-bit codes at 1531 tokens 116 against 125)
    if (tid == 0) fetched = atomicAdd(next_ctr + (Epi::kSR ? 0 : opaque(0)), 1);
    if (g2) block_barrier();
    // (e4m3: a pair of sub-steps is one operand of eight registers)
    constexpr bool kF8 = ELEM == EF8 || ELEM == EF4B;
    struct HA { i32x4 f[2][4]; u32x2 k[2][4][2]; i32x8 p[2][2]; };
    struct HB { i32x4 f[4]; u32x2 k[4][2]; i32x8 p[2]; };
    auto put4 = [](i32x8& d, int hi, i32x4 v) {
#pragma unroll
      for (int e = 0; e < 4; ++e) d[4 * hi + e] = v[e];
    };
    auto read_a = [&](const lds_u8* la, int hf, HA& F) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          if constexpr (MA == KC) {
            const int row = wi * 128 + 64 * hf + 32 * t + frow;
            const i32x4 v = *(const __attribute__((address_space(3))) i32x4*)(la + row * KB + 16 * ((2 * kk + h) ^ G::swz(row)));
            if constexpr (kF8) put4(F.p[t][kk >> 1], kk & 1, v);
            else F.f[t][kk] = v;
          } else {
            const int col = wi * 128 + 64 * hf + 32 * t + 16 * ch + 4 * u4;
            const int seg = ((col & 63) >> 4) ^ t4;
            const int a0 = (col >> 6) * (G::KR * 128) + (16 * kk + 8 * h + t4) * 128 + 32 * seg + 8 * u4;
            F.k[t][kk][0] = tr_read(la, a0);
            F.k[t][kk][1] = tr_read(la, a0 + 512);
          }
        }
    };
    auto read_b = [&](const lds_u8* lb, int t, HB& F) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if constexpr (MB == KF4) {
          // sub-step pair kk / 2: lane half h takes the row's 32 values from
          // 64 (kk / 2) + 32 h, which its e4m3 partner lanes pair them with
          const int row = wj * 64 + t * 32 + frow;
          if ((kk & 1) == 0)
            F.f[kk >> 1] = *(const __attribute__((address_space(3))) i32x4*)(lb + row * 64 + 16 * ((kk + h) ^ ((row >> 2) & 3)));
        } else if constexpr (MB == KC) {
          const int row = wj * 64 + t * 32 + frow;
          const i32x4 v = *(const __attribute__((address_space(3))) i32x4*)(lb + row * KB + 16 * ((2 * kk + h) ^ G::swz(row)));
          if constexpr (kF8) put4(F.p[kk >> 1], kk & 1, v);
          else F.f[kk] = v;
        } else {
          const int col = col_of(t) + 16 * ch + 4 * u4;
          const int seg = ((col & 63) >> 4) ^ t4;
          const int a0 = (col >> 6) * (G::KR * 128) + (16 * kk + 8 * h + t4) * 128 + 32 * seg + 8 * u4;
          F.k[kk][0] = tr_read(lb, a0);
          F.k[kk][1] = tr_read(lb, a0 + 512);
        }
      }
    };
    auto quarter = [&](const HA& A, const HB& B, int hf, int tb) {
      __builtin_amdgcn_sched_barrier(0);
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (ELEM == EF8 || ELEM == EF4B) {
        // unit E8M0 scales (127 = 2^0); B e4m3 (format 0) or FP4 (format 4)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const i32x8 av = A.p[t][m];
            AccV& c = acc[2 * hf + t][tb];
            if constexpr (ELEM == EF4B) {
              const i32x4 f = B.f[m];
              const i32x8 bv = {f[0], f[1], f[2], f[3], 0, 0, 0, 0};
              c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bv, av, c, 4, 0, 0, 127, 0, 127);
            } else {
              c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(B.p[m], av, c, 0, 0, 0, 127, 0, 127);
            }
          }
      } else {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const i32x4 a = MA == KC ? A.f[t][kk] : join(A.k[t][kk][0], A.k[t][kk][1]);
          const i32x4 b = MB == KC ? B.f[kk] : join(B.k[kk][0], B.k[kk][1]);
          AccV& c = acc[2 * hf + t][tb];
          if constexpr (ELEM == EI8)
            c = __builtin_amdgcn_mfma_i32_32x32x32_i8(b, a, c, 0, 0, 0);
          else if constexpr (Epi::kTrans)
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
          else
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    // One step.  Each phase: its fragment reads first, then one half-tile's
    // copies (issued ahead of the reads they delayed them: hidden-4096
    // backward + SR 6.3 against 5.6 ms; one copy in the compute part held up
    // the matrix instructions: 6.2 ms), then the wait for the half-tile that
    // the next phase reads: all but the copies newer than it.  The first
    // half-tile of B is read a step ahead, in the fourth phase, so that the
    // phases read 8, 4, 8 and 4 fragments (read in the first phase: 5.14
    // against 5.06 ms).  STEADY: steps s + 1 and s + 2 exist and are whole.
    // (e4m3 B keeps it in the first phase: its eight-register operands would
    // be copied from one step to the next)
    // Step 0 is in LDS as a whole when it begins: it waits for nothing in its
    // first two phases, least of all for the last tile's stores.
    constexpr bool kEarlyB = ELEM != EF8;
    HB B0;
    if constexpr (kEarlyB) read_b(stage_ptr(slot0) + OPB, 0, B0);
    auto step = [&](int s, auto steady) {
      constexpr bool ST = decltype(steady)::value;
      constexpr std::bool_constant<!ST> mt{};
      const int rem = n - 1 - s;
      const bool f1 = ST || rem >= 1, f2 = ST || rem >= 2;
      const bool ztail = !ST && cur.tail && n > 1;
      const int slot = slot0 ^ (s & 1);
      const lds_u8* la = stage_ptr(slot);
      const lds_u8* lb = la + OPB;
      auto copies = [&](int w, int at, int to) {
#pragma unroll
        for (int u = 0; u < (w == 0 || w == 3 ? 2 : CB); ++u) issue_copy(w, u, at, to, cur, mt);
      };
      HA A;
      HB B1;
      read_a(la, 0, A);
      if constexpr (!kEarlyB) read_b(lb, 0, B0);
      if (f1) {
        copies(3, s + 1, slot ^ 1);
        if (s > 0) wait_vm<6 + 2 * CB>();
      } else if (s > 0) {
        wait_vm<2>();
        if (ztail) zero_half(2, s, slot, cur);
      }
      quarter(A, B0, 0, 0);
      read_b(lb, 1, B1);
      if (f2) {
        copies(0, s + 2, slot);
        if (s > 0) wait_vm<6 + 2 * CB>();
      } else if (f1) {
        if (s > 0) wait_vm<4 + 2 * CB>();
      } else if (s > 0) {
        wait_vm<0>();
        if (ztail) zero_half(3, s, slot, cur);
      }
      quarter(A, B1, 0, 1);
      read_a(la, 1, A);
      if (f2) {
        copies(1, s + 2, slot);
        wait_vm<4 + 2 * CB>();
      } else if (f1) {
        wait_vm<2 + CB>();
        if (ztail) {
          zero_half(0, s + 1, slot ^ 1, cur);
          zero_half(1, s + 1, slot ^ 1, cur);
        }
      }
      quarter(A, B1, 1, 1);
      HB Bn;
      if (kEarlyB && f1) read_b(stage_ptr(slot ^ 1) + OPB, 0, Bn);
      if (f2) copies(2, s + 2, slot);
      quarter(A, B0, 1, 0);
      if (kEarlyB && f1) B0 = Bn;
    };
    int s = 0;
    for (const int ns = cur.wide ? 0 : n - 2 - (cur.tail ? 1 : 0); s < ns; ++s) step(s, std::true_type{});
    for (; s < n; ++s) step(s, std::false_type{});
    if (!g2) block_barrier();
  };
  for (;;) {
    fetched = 0;
#pragma unroll
    for (int a = 0; a < WI; ++a)
#pragma unroll
      for (int b = 0; b < WJ; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;

    if constexpr (kPP) {
      pp_loop();
    } else {
      // step it computes from stage (slot0 + it) mod NS while the next NS - 1
      // steps load into the other stages.  Step 0's loads were issued before
      // the previous epilogue's stores (a fixed number per thread), which may
      // stay in flight, as may the tile's later prefetched steps.
      constexpr int LPS = decltype(pa)::NL + decltype(pb)::NL;   // copies per thread per stage
      static_assert(NS * LPS < kVmMax, "vmcnt range");
      for (int it = 0; it < cur.nsteps; ++it) {
        const int slot = (slot0 + it) % NS;
        if (it == 0) {
          const int ahead = (cur.nsteps < NS - 1 ? cur.nsteps : NS - 1) - 1;
          int n = ahead * LPS + (first_tile ? 0 : stores_prev);
          if (n > kVmMax) n = kVmMax;
          wait_vm_le<kVmMax>(__builtin_amdgcn_readfirstlane(n));
          first_tile = false;
        } else {
          // copies of steps it + 1 .. it + NS - 2 (those issued) may stay in flight
          const int newer = cur.nsteps - 1 - it < NS - 2 ? cur.nsteps - 1 - it : NS - 2;
          wait_vm_le<(NS - 2) * LPS>(__builtin_amdgcn_readfirstlane(newer * LPS));
        }
        if (cur.tail && it == cur.nsteps - 1) zero_tail(it, slot, cur);
        block_barrier();                 // stage `slot` complete; step it - 1's stage is free
        // int8: one of the two waves of each SIMD copies after its first group
        // of MFMAs
        const bool copy_now = ELEM != EI8 || wave_u < NW / 2;
        if (copy_now && it + NS - 1 < cur.nsteps) issue(it + NS - 1, (slot + NS - 1) % NS, cur);
        // fetch the next tile early; its value is needed only at the epilogue
        if (it == 0 && tid == 0) fetched = atomicAdd(next_ctr + opaque(0), 1);
        compute(slot, [&]() {
          if (!copy_now && it + NS - 1 < cur.nsteps) issue(it + NS - 1, (slot + NS - 1) % NS, cur);
        });
      }
    }

    // epilogue parameters of this tile, then the next tile's first stage
    const Prob<Epi>& P = grp.p[cur.g];
    const Epi epi = P.epi;
    const int64_t I = P.I, J = P.J;
    const int64_t i0 = cur.i0, j0 = cur.j0;
    const int bz = cur.bz;
    const int last = (slot0 + cur.nsteps + NS - 1) % NS;   // stage of the last step (staging area)
    if constexpr (Epi::kRowScale) {
      const int tid_e = opaque(tid);
      if (tid_e < TILE) row_scale[tid_e] = epi.scale_fin(my_scale);
    }
    // SR epilogue: this lane's code chunks, rows sr_r + 16 u of each 32-row
    // block and columns 8 sr_c .. 8 sr_c + 7 of each 32-column block (8
    // weights per chunk: one Philox block, since d_in is a multiple of 8).
    // Loaded here, after the main loop, and waited for before the next
    // tile's copies are issued, so the wait drains nothing else.
    const int sr_r = lane >> 2, sr_c = lane & 3;
    // ternary: both chunks of a 32 x 32 block in one register (u = 0 low
    // half); int8: two words per chunk
    [[maybe_unused]] uint32_t srt[Epi::kSR ? WI : 1][Epi::kSR ? WJ : 1];
    [[maybe_unused]] uint32_t sr8[Epi::kSR && !Epi::kTern ? WI : 1][Epi::kSR && !Epi::kTern ? WJ : 1][2][2];
    auto sr_pos = [&](int ta, int tb, int u, int64_t& n, int64_t& k) {
      // block (ta, tb) of dW^T holds dW rows j0 + col_of(tb) + .. (d_out) and
      // columns i0 + .. + 32 ta (d_in), laid out as a block of dW
      n = j0 + col_of(tb) + sr_r + 16 * u;
      k = i0 + wi * 32 * WI + ta * 32 + 8 * sr_c;
      return n < J && k < I;
    };
    if constexpr (Epi::kSR) {
#pragma unroll
      for (int ta = 0; ta < WI; ++ta)
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            int64_t n, k;
            const bool ok = sr_pos(ta, tb, u, n, k);
            if constexpr (Epi::kTern) {
              const uint8_t* src = ok ? epi.wq + n * epi.ldc + (k >> 2) : dummy;
              const uint32_t v = *reinterpret_cast<const uint16_t*>(src);
              if (u == 0) srt[ta][tb] = v;
              else srt[ta][tb] |= v << 16;
            } else if constexpr (Epi::kCF == CF_I4) {
              const uint8_t* src = ok ? epi.wq + n * epi.ldc + (k >> 1) : dummy;
              sr8[ta][tb][u][0] = *reinterpret_cast<const uint32_t*>(src);
              sr8[ta][tb][u][1] = 0;
            } else if constexpr (Epi::kCF == CF_I3) {
              // three bytes (k / 8 chunks of 3 bytes into the row)
              uint32_t w[4];
              ChunkIO<CF_I3>::load(ok ? epi.wq + n * epi.ldc : dummy, ok ? (k >> 3) : 0, w);
              sr8[ta][tb][u][0] = w[0];
              sr8[ta][tb][u][1] = 0;
            } else {
              const uint8_t* src = ok ? epi.wq + n * epi.ldc + k : dummy;
              const uint2 v = *reinterpret_cast<const uint2*>(src);
              sr8[ta][tb][u][0] = v.x;
              sr8[ta][tb][u][1] = v.y;
            }
          }
    }
    if (tid == 0) next_tile = cur.nsteps > 0 ? fetched : atomicAdd(next_ctr, 1);
    block_barrier();                   // every wave is done with every stage
    int gn, localn;
    const bool more = locate(grp, xcd, next_tile, gn, localn);
    if constexpr (Epi::kSR) wait_vm<0>();   // the codes (nothing else is in flight)
    if (more) {
      const int slotn = (last + 1) % NS;      // the next tile's stages avoid `last`
      setup(gn, localn, cur);
      prefetch(slotn);
      slot0 = slotn;
    }

    // The MFMAs take the B fragment as their first operand, so lane
    // (j = lane mod 32, h) of block (ta, tb) holds row 32 ta + j, columns
    // 32 tb + 8 (r / 4) + 4 h + (r mod 4), r = 0..15: four consecutive
    // columns per group of four entries.  Each wave stages 32 rows of 128
    // bytes at a time in its own part of stage `last` (bf16: both column
    // blocks of a pair; fp32: one column block), 16-byte chunk c of row
    // r at chunk c ^ ((r >> 1) & 7), then writes whole 16-byte chunks of
    // output rows.
    const int lane_e = opaque(lane), h_e = lane_e >> 5, j_e = lane_e & 31;
    lds_u8* stage = smem + last * SLOTB + wave * (32 * 128);
    const bool obf = epi.out_bf16();
    const int sw_w = (j_e >> 1) & 7;
    const int rd_row = lane_e >> 3, rd_chunk = lane_e & 7;
    // one row block (32 rows of the wave): its values in LDS, then its rows
    auto epi_block = [&](int ta, auto ebytes_tag) {
      constexpr int EBY = decltype(ebytes_tag)::value;
      const float sc = Epi::kRowScale ? row_scale[wi * 32 * WI + ta * 32 + j_e] : epi.scale(0);
      auto value = [&](int tb, int r) {
        float v;
        if constexpr (ELEM == EI8) v = (float)acc[ta][tb][r];
        else v = acc[ta][tb][r];
        return v * sc;
      };
      // stores the staged 32 x 128 bytes: columns from `col0` (elements)
      // (every lane stores every time, chunks outside the output to a dummy
      // slot, so the number of stores in flight is known)
      auto store_staged = [&](int col0) {
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int64_t jj = j0 + wj * 32 * WJ + col0 + rd_chunk * (16 / EBY);
        const int rows_left = (int)__builtin_amdgcn_readfirstlane(
            (int)(I - (i0 + wi * 32 * WI + ta * 32) < 32 ? I - (i0 + wi * 32 * WI + ta * 32) : 32));
        uint8_t* const p0 = epi.row(i0 + wi * 32 * WI + ta * 32 + rd_row, bz) + jj * EBY;
        const int64_t rstride = 8 * epi.row_bytes();
        const bool col_ok = jj < J;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = rd_row + 8 * u;
          const i32x4 d = *(const __attribute__((address_space(3))) i32x4*)(
              stage + row * 128 + ((rd_chunk ^ ((row >> 1) & 7)) << 4));
          uint8_t* dst = (col_ok && row < rows_left) ? p0 + u * rstride : dummy;
          *reinterpret_cast<i32x4*>(dst) = d;
        }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      };
      if constexpr (EBY == 2) {
#pragma unroll
        for (int tp = 0; tp < WJ / 2; ++tp) {
#pragma unroll
          for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int tb = 2 * tp + t2;
              const u32x2 w = {pack_bf16x2(value(tb, 4 * k), value(tb, 4 * k + 1)),
                               pack_bf16x2(value(tb, 4 * k + 2), value(tb, 4 * k + 3))};
              *(__attribute__((address_space(3))) u32x2*)(
                  stage + j_e * 128 + (((4 * t2 + k) ^ sw_w) << 4) + 8 * h_e) = w;
            }
          store_staged(64 * tp);
        }
      } else {
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const f32x4 w = {value(tb, 4 * k), value(tb, 4 * k + 1), value(tb, 4 * k + 2), value(tb, 4 * k + 3)};
            *(__attribute__((address_space(3))) f32x4*)(stage + j_e * 128 + (((2 * k + h_e) ^ sw_w) << 4)) = w;
          }
          store_staged(32 * tb);
        }
      }
    };
    if constexpr (Epi::kSR) {
      // each 32 x 32 block of dW staged in LDS as fp32, then read back as
      // two chunks of 8 consecutive entries of a row per lane, which update
      // their 8 codes; out-of-range chunks count nothing and store their
      // codes to the dummy slot (a fixed number of stores per thread)
      SRArgs sa;
      sa.c = epi.c;
      sa.L = epi.L;
      sa.qmin = epi.qmin;
      sa.qmax = epi.qmax;
      sa.k0 = epi.k0;
      sa.k1 = epi.k1;
      sa.step = epi.step;
      sa.tid = epi.tid;
      uint32_t tc = 0, tn = 0;   // this tile's counts
      // 32 rows x 64 columns (both column blocks of a row block) per wave:
      // two 32 x 128-byte areas, laid out as the fp32 staging above
      static_assert(NW * 32 * 256 <= SLOTB, "SR staging (32 rows of 256 bytes per wave) fits in one stage");
      lds_u8* const st2 = smem + last * SLOTB + wave * (32 * 256);
#pragma unroll
      for (int ta = 0; ta < WI; ++ta) {
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const f32x4 w = {(float)acc[ta][tb][4 * k], (float)acc[ta][tb][4 * k + 1],
                             (float)acc[ta][tb][4 * k + 2], (float)acc[ta][tb][4 * k + 3]};
            *(__attribute__((address_space(3))) f32x4*)(st2 + tb * (32 * 128) + j_e * 128 +
                                                          (((2 * k + h_e) ^ sw_w) << 4)) = w;
          }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // the row block's 2 WJ chunks from LDS, one at a time (not
        // unrolled: short code, few live registers)
#pragma unroll 1
        for (int cq = 0; cq < 2 * WJ; ++cq) {
          const int tb = cq >> 1, u = cq & 1;
          const int row = sr_r + 16 * u;
          const int sw = (row >> 1) & 7;
          const lds_u8* sb = st2 + tb * (32 * 128) + row * 128;
          f32x4 gv[2];
          gv[0] = *(const __attribute__((address_space(3))) f32x4*)(sb + (((2 * sr_c) ^ sw) << 4));
          gv[1] = *(const __attribute__((address_space(3))) f32x4*)(sb + (((2 * sr_c + 1) ^ sw) << 4));
          int64_t n, k;
          const bool ok = sr_pos(ta, tb, u, n, k);
          uint32_t win[4] = {0u, 0u, 0u, 0u};
          if constexpr (Epi::kTern) {
            uint32_t w2 = srt[ta][0];
#pragma unroll
            for (int t = 1; t < WJ; ++t) w2 = tb == t ? srt[ta][t] : w2;
            win[0] = (w2 >> (16 * u)) & 0xFFFFu;
          } else {
            uint32_t x0 = sr8[ta][0][0][0], x1 = sr8[ta][0][0][1];
#pragma unroll
            for (int t = 0; t < WJ; ++t)
#pragma unroll
              for (int v = 0; v < 2; ++v)
                if (cq == 2 * t + v) {
                  x0 = sr8[ta][t][v][0];
                  x1 = sr8[ta][t][v][1];
                }
            win[0] = x0;
            win[1] = x1;
          }
          uint32_t wout[4];
          uint32_t ch = 0, nf = 0;
          sr_chunk<Epi::kCF, 8>(win, gv, (uint64_t)(n * epi.d_in + k) >> 3, sa, wout, ch, nf);
          if (ok) {
            tc += ch;
            tn += nf;
          }
          if constexpr (Epi::kTern) {
            uint8_t* dst = ok ? epi.wq + n * epi.ldc + (k >> 2) : dummy;
            *reinterpret_cast<uint16_t*>(dst) = (uint16_t)wout[0];
          } else if constexpr (Epi::kCF == CF_I4) {
            uint8_t* dst = ok ? epi.wq + n * epi.ldc + (k >> 1) : dummy;
            *reinterpret_cast<uint32_t*>(dst) = wout[0];
          } else if constexpr (Epi::kCF == CF_I3) {
            // (three single-byte stores: the vmcnt accounting above counts
            // one per chunk, a lower bound, which only makes waits stricter)
            ChunkIO<CF_I3>::store(ok ? epi.wq + n * epi.ldc : dummy, ok ? (k >> 3) : 0, wout);
          } else {
            uint8_t* dst = ok ? epi.wq + n * epi.ldc + k : dummy;
            *reinterpret_cast<uint2*>(dst) = make_uint2(wout[0], wout[1]);
          }
        }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      tc = wave_sum_u32(tc);
      tn = wave_sum_u32(tn);
      if (lane == 0) {
        sr_cnt[2 * wave_u] += tc;
        sr_cnt[2 * wave_u + 1] += tn;
      }
      stores_prev = kStoresSR;
    } else {
      if (obf) {
#pragma unroll
        for (int ta = 0; ta < WI; ++ta) epi_block(ta, std::integral_constant<int, 2>{});
      } else {
#pragma unroll
        for (int ta = 0; ta < WI; ++ta) epi_block(ta, std::integral_constant<int, 4>{});
      }
      stores_prev = obf ? kStoresBf16 : kStoresF32;
    }
    if (!more) break;
    // a tile without reduction steps has no main-loop barrier before the
    // next epilogue reuses the staging area and the row scales
    if (cur.nsteps == 0) block_barrier();
  }
  if constexpr (Epi::kSR) {
    unsigned long long* const cnt = grp.p[0].epi.counters;
    if (cnt != nullptr && lane == 0) {
      const unsigned long long c = sr_cnt[2 * wave_u], f = sr_cnt[2 * wave_u + 1];
      if (c) atomicAdd(cnt, c);
      if (f) atomicAdd(cnt + 1, f);
    }
  }
}

template <int ELEM, int MA, int MB, class Epi, bool ONE>
__global__ __launch_bounds__(NTH) void gemm_v3_kernel(const Group<Epi> grp) {
  __shared__ __attribute__((aligned(1024))) uint8_t stages[StageGeo<MB, ONE>::kBytes];
  __shared__ float row_scale[TILE];
  __shared__ int next_tile;
  gemm_v3_body<ELEM, MA, MB, Epi, ONE>(grp, (lds_u8*)stages, (lds_f32*)row_scale, (lds_i32*)&next_tile);
}

// Two groups of bf16 products in one launch: every block takes tiles of the
// first group until its lists are empty, then tiles of the second, so blocks
// left without a tile of the first start on the second at once.
template <int MA1, int MB1, class Epi1, int MA2, int MB2, class Epi2>
__global__ __launch_bounds__(NTH) void gemm_v3_dual_kernel(const Group<Epi1> g1, const Group<Epi2> g2) {
  static_assert(StageGeo<MB1, false>::kBytes == StageGeo<MB2, false>::kBytes, "one stage area");
  __shared__ __attribute__((aligned(1024))) uint8_t stages[StageGeo<MB1, false>::kBytes];
  __shared__ float row_scale[TILE];
  __shared__ int next_tile;
  gemm_v3_body<EBF16, MA1, MB1, Epi1>(g1, (lds_u8*)stages, (lds_f32*)row_scale, (lds_i32*)&next_tile);
  __syncthreads();
  gemm_v3_body<EBF16, MA2, MB2, Epi2>(g2, (lds_u8*)stages, (lds_f32*)row_scale, (lds_i32*)&next_tile);
}

}  // namespace v3
}  // namespace dqt

// ------------------------------------------------------------ pre-passes
namespace dqt {
namespace v3 {

// Up to MAXG independent element ranges handled by one launch.  Segment s
// owns blocks [b0[s], b0[s+1]); each thread of a block handles one 16-element
// chunk; chunks past n16[s] do nothing.
struct SegTab {
  const void* src[MAXG];
  void* dst[MAXG];
  const float* scale[MAXG];   // per-row scales (activation dequantisation)
  int64_t n16[MAXG];
  int32_t k16[MAXG];          // 16-element chunks per row (activation dequantisation)
  int32_t b0[MAXG + 1];
  int32_t n;
  int* sched;                 // the GEMM's tile counters to zero, or NULL
};

// The persistent GEMM's tile counters (both 64-byte slots) are zeroed by
// block 0 of the pass before it, so a workspace needs no particular contents
// (a launch of their own took 5 us).
__device__ __forceinline__ void sched_clear(int* sched) {
  if (blockIdx.x == 0 && threadIdx.x < 32) sched[threadIdx.x] = 0;
}

__device__ __forceinline__ int seg_of_block(const SegTab& t) {
  if (t.sched != nullptr) sched_clear(t.sched);
  int s = 0;
  while (s + 1 < t.n && (int)blockIdx.x >= t.b0[s + 1]) ++s;
  return s;
}

// Packed ternary codes -> one operand byte (int8 or e4m3) per weight, same
// [d_out][d_in] row-major order.
// Four chunks of 16 weights per thread (16 bytes in, 64 out), the last
// thread of a tensor whatever chunks remain.
template <int OUT>
__device__ __forceinline__ uint4 unpack16_ternary(uint32_t w) {
  uint32_t o[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint32_t sp = spread_codes((w >> (8 * b)) & 0xFFu);
    o[b] = OUT == 1 ? codes_to_e4m3x4(sp) : codes_to_i8x4(sp);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}
template <int OUT>   // 0: int8, 1: e4m3
__global__ __launch_bounds__(256) void unpack_ternary_kernel(const SegTab tab) {
  const int s = seg_of_block(tab);
  const int64_t t = (int64_t)(blockIdx.x - tab.b0[s]) * 256 + threadIdx.x;
  const int64_t g0 = 4 * t, n16 = tab.n16[s];
  if (g0 >= n16) return;
  uint4* const dst = static_cast<uint4*>(tab.dst[s]);
  if (g0 + 4 <= n16) {
    const uint4 w = static_cast<const uint4*>(tab.src[s])[t];
    dst[g0] = unpack16_ternary<OUT>(w.x);
    dst[g0 + 1] = unpack16_ternary<OUT>(w.y);
    dst[g0 + 2] = unpack16_ternary<OUT>(w.z);
    dst[g0 + 3] = unpack16_ternary<OUT>(w.w);
  } else {
    for (int64_t g = g0; g < n16; ++g) dst[g] = unpack16_ternary<OUT>(static_cast<const uint32_t*>(tab.src[s])[g]);
  }
}

// Packed ternary codes -> FP4 (E2M1) values, two per byte in weight order
// (weight k in the low nibble of byte k / 2 when k is even): the B operand of
// the e4m3 forward.  64 weights per thread (16 bytes in, 32 out: with 16
// weights a thread the pass was held by the few bytes each had in flight);
// n16 a multiple of 4.
__global__ __launch_bounds__(256) void expand_fp4_kernel(const SegTab tab) {
  const int s = seg_of_block(tab);
  const int64_t t = (int64_t)(blockIdx.x - tab.b0[s]) * 256 + threadIdx.x;
  if (t >= tab.n16[s] / 4) return;
  const uint4 w = static_cast<const uint4*>(tab.src[s])[t];
  const u32x2 a = expand16_fp4(w.x), b = expand16_fp4(w.y), c = expand16_fp4(w.z), d = expand16_fp4(w.w);
  uint4* const dst = static_cast<uint4*>(tab.dst[s]) + 2 * t;
  dst[0] = make_uint4(a[0], a[1], b[0], b[1]);
  dst[1] = make_uint4(c[0], c[1], d[0], d[1]);
}

// int4 codes (two's-complement nibbles, weight k at bits 4 (k mod 2) of byte
// k / 2) -> one operand byte per weight (int8, or e4m3, exact for |q| <= 8),
// same order; 16 weights per thread.
template <int OUT>   // 0: int8, 1: e4m3
__global__ __launch_bounds__(256) void unpack_int4_kernel(const SegTab tab) {
  const int s = seg_of_block(tab);
  const int64_t t = (int64_t)(blockIdx.x - tab.b0[s]) * 256 + threadIdx.x;
  if (t >= tab.n16[s]) return;
  const uint2 w2 = static_cast<const uint2*>(tab.src[s])[t];
  const uint32_t w[2] = {w2.x, w2.y};
  uint32_t o[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int q = (int)(w[e >> 3] << (28 - 4 * (e & 7))) >> 28;
    const uint32_t b = OUT == 1 ? f32_to_e4m3((float)q) : ((uint32_t)q & 0xFFu);
    o[e >> 2] |= b << (8 * (e & 3));
  }
  static_cast<uint4*>(tab.dst[s])[t] = make_uint4(o[0], o[1], o[2], o[3]);
}

// 3-bit codes (8 weights in 3 bytes, weight k at bits 3 (k mod 8) of its
// group) -> one operand byte per weight (int8, or e4m3, exact for |q| <= 4),
// same order; 16 weights (6 bytes, read as three 2-byte words) per thread.
template <int OUT>   // 0: int8, 1: e4m3
__global__ __launch_bounds__(256) void unpack_int3_kernel(const SegTab tab) {
  const int s = seg_of_block(tab);
  const int64_t t = (int64_t)(blockIdx.x - tab.b0[s]) * 256 + threadIdx.x;
  if (t >= tab.n16[s]) return;
  const uint16_t* src = static_cast<const uint16_t*>(tab.src[s]) + 3 * t;
  const uint64_t bits = (uint64_t)src[0] | ((uint64_t)src[1] << 16) | ((uint64_t)src[2] << 32);
  uint32_t o[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int q = (int)((uint32_t)(bits >> (3 * e)) << 29) >> 29;
    const uint32_t b = OUT == 1 ? f32_to_e4m3((float)q) : ((uint32_t)q & 0xFFu);
    o[e >> 2] |= b << (8 * (e & 3));
  }
  static_cast<uint4*>(tab.dst[s])[t] = make_uint4(o[0], o[1], o[2], o[3]);
}

// Weights q [d_out][d_in] (3-bit, 4-bit or 8-bit codes) -> the B operand of
// dX with the reduction contiguous: W~T[k][n] = bf16(q[n][k]) (exact), rows of
// d_out elements.  One 64 x 64 tile per block, transposed through LDS.
struct TrTab {
  const uint8_t* src[MAXG];
  uint16_t* dst[MAXG];
  int32_t d_out[MAXG], d_in[MAXG];
  int32_t tn[MAXG];           // tiles along n (d_out / 64, rounded up)
  int32_t b0[MAXG + 1];
  int32_t n;
};
using TLds = uint16_t[64][72];   // a transposed tile
template <int CF>
__device__ __forceinline__ void unpack_t_block(const TrTab& tab, int block, TLds& t_lds) {
  int s = 0;
  while (s + 1 < tab.n && block >= tab.b0[s + 1]) ++s;
  const int tile = block - tab.b0[s];
  const int n0 = (tile % tab.tn[s]) * 64, k0 = (tile / tab.tn[s]) * 64;
  const int d_out = tab.d_out[s], d_in = tab.d_in[s];
  const int t = threadIdx.x;
  {
    // thread t: row n0 + t / 4, reduction elements k0 + 16 (t mod 4) .. + 15
    const int nl = t >> 2, kl = (t & 3) * 16;
    const int n = n0 + nl, k = k0 + kl;
    uint16_t v[16];
    if (n < d_out && k < d_in) {
      if constexpr (CF == CF_I3) {
        // 16 weights: 6 bytes at 3 k / 8 (k a multiple of 16: 2-byte aligned)
        const uint16_t* w3 = reinterpret_cast<const uint16_t*>(tab.src[s] + (int64_t)n * (3 * d_in / 8) + 3 * k / 8);
        const uint64_t bits = (uint64_t)w3[0] | ((uint64_t)w3[1] << 16) | ((uint64_t)w3[2] << 32);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float f = (float)((int)((uint32_t)(bits >> (3 * e)) << 29) >> 29);
          v[e] = (uint16_t)(__float_as_uint(f) >> 16);   // exact: |q| <= 4
        }
      } else if constexpr (CF == CF_I4) {
        const uint2 w2 = *reinterpret_cast<const uint2*>(tab.src[s] + (int64_t)n * (d_in / 2) + k / 2);
        const uint32_t w[2] = {w2.x, w2.y};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float f = (float)((int)(w[e >> 3] << (28 - 4 * (e & 7))) >> 28);
          v[e] = (uint16_t)(__float_as_uint(f) >> 16);   // exact: |q| <= 8
        }
      } else {
        const uint4 w4 = *reinterpret_cast<const uint4*>(tab.src[s] + (int64_t)n * d_in + k);
        const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float f = (float)(int)(int8_t)((w[e >> 2] >> (8 * (e & 3))) & 0xFFu);
          v[e] = (uint16_t)(__float_as_uint(f) >> 16);   // exact: |q| <= 128
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = 0;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) t_lds[kl + e][nl] = v[e];
  }
  __syncthreads();
#pragma unroll
  for (int c = t; c < 64 * 8; c += 256) {
    const int kl = c >> 3, ch = c & 7;
    const int k = k0 + kl, n = n0 + ch * 8;
    if (k < d_in && n < d_out)
      *reinterpret_cast<uint4*>(tab.dst[s] + (int64_t)k * d_out + n) =
          *reinterpret_cast<const uint4*>(&t_lds[kl][ch * 8]);
  }
}

// Ternary codes -> W~T as unpack_t_block, one block per strip of 64 rows x
// 512 reduction elements: the strip's codes (whole 128-byte lines of each
// row) come into LDS in one pass, eight loads in flight per thread, then its
// eight 64 x 64 tiles are transposed through LDS in turn.  (One block per
// tile read 16 bytes of each row's line and fetched about 4 times the code
// bytes.)
using CodeLds = uint32_t[64][33];   // [row][word of 16 codes]
__device__ __forceinline__ void unpack_t2_strip_block(const TrTab& tab, int block, TLds& t_lds, CodeLds& codes) {
  int s = 0;
  while (s + 1 < tab.n && block >= tab.b0[s + 1]) ++s;
  const int strip = block - tab.b0[s];
  const int n0 = (strip % tab.tn[s]) * 64, ks0 = (strip / tab.tn[s]) * 512;
  const int d_out = tab.d_out[s], d_in = tab.d_in[s];
  const int t = threadIdx.x;
  {
    // thread t: row n0 + t / 4, words 8 (t mod 4) .. + 7 of the strip
    const int row = t >> 2, n = n0 + row;
    const int wrow = d_in / 16;                       // words of a row
    const uint32_t* src = reinterpret_cast<const uint32_t*>(tab.src[s]) + (int64_t)n * wrow;
    uint32_t w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kw = ks0 / 16 + 8 * (t & 3) + e;
      w[e] = (n < d_out && kw < wrow) ? src[kw] : 0u;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) codes[row][8 * (t & 3) + e] = w[e];
  }
  __syncthreads();
  const int nl = t >> 2, kl = (t & 3) * 16;
  for (int j = 0; j < 8; ++j) {
    const int k0 = ks0 + 64 * j;
    if (k0 >= d_in) break;                            // (uniform)
    const uint32_t w = codes[nl][4 * j + (t & 3)];
#pragma unroll
    for (int e = 0; e < 16; ++e) t_lds[kl + e][nl] = (uint16_t)code_to_bf16_bits((w >> (2 * e)) & 3u);
    __syncthreads();
#pragma unroll
    for (int c = t; c < 64 * 8; c += 256) {
      const int kr = c >> 3, ch = c & 7;
      const int k = k0 + kr, n = n0 + ch * 8;
      if (k < d_in && n < d_out)
        *reinterpret_cast<uint4*>(tab.dst[s] + (int64_t)k * d_out + n) =
            *reinterpret_cast<const uint4*>(&t_lds[kr][ch * 8]);
    }
    __syncthreads();
  }
}

// X~T[k, m] = bf16(fl(value(Xq[m, k]) * xdq[m])): the dequantised
// activations transposed (the reduction of dW, over tokens, contiguous).
// One 64 x 64 tile per block, transposed through LDS.
struct DqTab {
  const uint8_t* src[MAXG];   // Xq [M][K]
  uint16_t* dst[MAXG];        // X~T [K][Mp]
  const float* scale[MAXG];   // xdq [M]
  int32_t K[MAXG];
  int32_t tm[MAXG];           // tiles along m
  int32_t b0[MAXG + 1];
  int32_t n;
  int64_t M, Mp;              // tokens, and the row stride of X~T (a multiple of 64)
};
template <bool E4M3>
__device__ __forceinline__ void dequant_t_block(const DqTab& tab, int block, TLds& t_lds) {
  int s = 0;
  while (s + 1 < tab.n && block >= tab.b0[s + 1]) ++s;
  const int tile = block - tab.b0[s];
  const int64_t M = tab.M;
  const int K = tab.K[s];
  const int64_t m0 = (int64_t)(tile % tab.tm[s]) * 64;
  const int k0 = (tile / tab.tm[s]) * 64;
  const int t = threadIdx.x;
  {
    // thread t: token m0 + t / 4, features k0 + 16 (t mod 4) .. + 15
    const int ml = t >> 2, kl = (t & 3) * 16;
    const int64_t m = m0 + ml;
    const int k = k0 + kl;
    uint32_t o[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (m < M && k < K) {
      const float d = tab.scale[s][m];
      const uint4 v = *reinterpret_cast<const uint4*>(tab.src[s] + m * K + k);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t two = w[j >> 1] >> (16 * (j & 1));
        float a, b;
        if constexpr (E4M3) {
          a = e4m3_to_f32(two & 0xFFu);
          b = e4m3_to_f32((two >> 8) & 0xFFu);
        } else {
          a = (float)(int)(int8_t)(two & 0xFFu);
          b = (float)(int)(int8_t)((two >> 8) & 0xFFu);
        }
        o[j] = pack_bf16x2(a * d, b * d);
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      t_lds[kl + 2 * j][ml] = (uint16_t)(o[j] & 0xFFFFu);
      t_lds[kl + 2 * j + 1][ml] = (uint16_t)(o[j] >> 16);
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = t; c < 64 * 8; c += 256) {
    const int kl = c >> 3, ch = c & 7;
    const int k = k0 + kl;
    const int64_t m = m0 + ch * 8;
    if (k < K && m < M)
      *reinterpret_cast<uint4*>(tab.dst[s] + (int64_t)k * tab.Mp + m) =
          *reinterpret_cast<const uint4*>(&t_lds[kl][ch * 8]);
  }
}

// What the products of a backward call need before them, in one launch: W~T
// for dX (the first n_tr blocks), X~T for dW, and the cleared tile counters.
// (As three launches, backward + SR of the hidden-768 block at 8192 tokens
// took 258 us instead of 250.)
struct PrepTab {
  TrTab tr;
  DqTab dq;
  int32_t n_tr, n_dq;
  int* sched;
};
template <int CF, bool E4M3>
__global__ __launch_bounds__(256) void bwd_prep_kernel(const PrepTab tab) {
  __shared__ __attribute__((aligned(16))) TLds t_lds;
  sched_clear(tab.sched);
  const int b = (int)blockIdx.x;
  if (b < tab.n_tr) {
    if constexpr (CF == CF_T2) {
      __shared__ CodeLds codes;
      unpack_t2_strip_block(tab.tr, b, t_lds, codes);
    } else {
      unpack_t_block<CF>(tab.tr, b, t_lds);
    }
  } else {
    dequant_t_block<E4M3>(tab.dq, b - tab.n_tr, t_lds);
  }
}

// dW[l] = sum over splits of the fp32 partials of linear l, in split order
// (deterministic), for every linear of a batch in one launch.
struct RedTab {
  const float* src[MAXG];     // [splits][n] partials
  float* dst[MAXG];           // [n]
  int64_t n4[MAXG];           // n / 4
  int32_t b0[MAXG + 1];
  int32_t n, splits;
};
__global__ __launch_bounds__(256) void split_reduce_batch_kernel(const RedTab tab) {
  int s = 0;
  while (s + 1 < tab.n && (int)blockIdx.x >= tab.b0[s + 1]) ++s;
  const int64_t t = (int64_t)(blockIdx.x - tab.b0[s]) * 256 + threadIdx.x;
  const int64_t n4 = tab.n4[s];
  if (t >= n4) return;
  const f32x4* src = reinterpret_cast<const f32x4*>(tab.src[s]);
  f32x4 acc = __builtin_nontemporal_load(src + t);
  for (int k = 1; k < tab.splits; ++k) {
    const f32x4 v = __builtin_nontemporal_load(src + (int64_t)k * n4 + t);
    acc[0] = acc[0] + v[0];
    acc[1] = acc[1] + v[1];
    acc[2] = acc[2] + v[2];
    acc[3] = acc[3] + v[3];
  }
  reinterpret_cast<f32x4*>(tab.dst[s])[t] = acc;
}

// The split-K sum of dW (the same order as split_reduce_batch_kernel, so the
// same dW bits) consumed by the SR update of the codes, 8 weights per
// thread; dW is never stored.
struct RedSRTab {
  const float* src[MAXG];     // [splits][n] partials
  uint8_t* wq[MAXG];          // codes, updated in place
  int64_t n8[MAXG];           // n / 8
  float c[MAXG], L[MAXG];
  int32_t qmin[MAXG], qmax[MAXG];
  uint32_t tid[MAXG];
  int32_t b0[MAXG + 1];
  int32_t n, splits;
  uint32_t k0, k1, step;
  unsigned long long* counters;
};
template <int CF>
__global__ __launch_bounds__(256) void split_reduce_sr_kernel(const RedSRTab tab) {
  int s = 0;
  while (s + 1 < tab.n && (int)blockIdx.x >= tab.b0[s + 1]) ++s;
  const int64_t t = (int64_t)(blockIdx.x - tab.b0[s]) * 256 + threadIdx.x;
  uint32_t ch = 0, nf = 0;
  if (t < tab.n8[s]) {
    const int64_t n4 = 2 * tab.n8[s];
    const f32x4* src = reinterpret_cast<const f32x4*>(tab.src[s]);
    f32x4 gv[2];
    gv[0] = __builtin_nontemporal_load(src + 2 * t);
    gv[1] = __builtin_nontemporal_load(src + 2 * t + 1);
    for (int k = 1; k < tab.splits; ++k) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const f32x4 v = __builtin_nontemporal_load(src + (int64_t)k * n4 + 2 * t + e);
        gv[e][0] = gv[e][0] + v[0];
        gv[e][1] = gv[e][1] + v[1];
        gv[e][2] = gv[e][2] + v[2];
        gv[e][3] = gv[e][3] + v[3];
      }
    }
    SRArgs a;
    a.c = tab.c[s];
    a.L = tab.L[s];
    a.qmin = tab.qmin[s];
    a.qmax = tab.qmax[s];
    a.k0 = tab.k0;
    a.k1 = tab.k1;
    a.step = tab.step;
    a.tid = tab.tid[s];
    uint32_t win[4] = {0u, 0u, 0u, 0u}, wout[4];
    ChunkIO<CF>::load(tab.wq[s], t, win);
    sr_chunk<CF, 8>(win, gv, (uint64_t)t, a, wout, ch, nf);
    ChunkIO<CF>::store(tab.wq[s], t, wout);
  }
  if (tab.counters != nullptr) {
    // one atomic per block (atomics of every wave on one address serialise)
    __shared__ uint32_t red[2][256 / kWave];
    const uint32_t c = wave_sum_u32(ch), f = wave_sum_u32(nf);
    if ((threadIdx.x & (kWave - 1)) == 0) {
      red[0][threadIdx.x / kWave] = c;
      red[1][threadIdx.x / kWave] = f;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long ct = 0, ft = 0;
#pragma unroll
      for (int w = 0; w < 256 / kWave; ++w) {
        ct += red[0][w];
        ft += red[1][w];
      }
      if (ct) atomicAdd(tab.counters, ct);
      if (ft) atomicAdd(tab.counters + 1, ft);
    }
  }
}

static int32_t seal(SegTab& t) {
  int32_t b = 0;
  for (int s = 0; s < t.n; ++s) {
    t.b0[s] = b;
    b += (int32_t)((t.n16[s] + 255) / 256);
  }
  t.b0[t.n] = b;
  return b;
}

// Zeroes the persistent GEMM's tile counters before its launch where no pass
// that does so precedes it.
__global__ __launch_bounds__(64) void sched_clear_kernel(int* sched) { sched_clear(sched); }

// XCD shares of a launch's tiles: contiguous, since the tiles an XCD's
// compute units hold at once share operand panels in its L2 only if they are
// neighbours.  A launch of at most one tile per compute unit gives its tiles,
// problem after problem, to the XCDs in eight equal runs (an eighth of every
// problem each left 2-3 neighbours of a small problem, and the misses held
// the launch at 4.4 TB/s: hidden-672 block, 8-bit codes, 1423 tokens, 249
// tiles: backward + SR 102 -> 75 us).  A larger one gives every XCD an eighth
// of every problem, longest reductions first, so that all eight stay equally
// long (whole problems on fewer XCDs were 2-10 % faster where they happened
// to balance and up to 20 % slower where not).
struct XcdShares {
  int64_t total, at = 0;       // tiles of the launch; shared out so far
  int32_t cus;
  int32_t tiles[8] = {};
  explicit XcdShares(int64_t n) : total(n), cus(std::max(8, current_device_cus())) {}

  // the shares of a problem of n tiles
  void take(int64_t n, int32_t (&xb)[9]) {
    for (int x = 0; x <= 8; ++x)
      xb[x] = (int32_t)(total <= cus ? std::min(std::max(total * x / 8 - at, (int64_t)0), n) : n * x / 8);
    at += n;
    for (int x = 0; x < 8; ++x) tiles[x] += xb[x + 1] - xb[x];
  }
  // blocks per XCD: one per tile, at most one per compute unit
  int32_t blocks() const { return std::min(*std::max_element(tiles, tiles + 8), cus / 8); }
};

template <class Epi>
static int64_t group_tiles(Group<Epi>& grp) {
  int64_t n = 0;
  for (int g = 0; g < grp.ng; ++g) {
    Prob<Epi>& p = grp.p[g];
    p.nbx = (int32_t)((p.J + TILE - 1) / TILE);
    p.nby = (int32_t)((p.I + TILE - 1) / TILE);
    p.ntiles = p.nbx * p.nby * p.nbz;
    n += p.ntiles;
  }
  return n;
}
// Longest-first order and XCD shares of a group; `slot` picks its 64 bytes of
// tile counters among the workspace's first 128.
template <int ELEM, class Epi>
static void prep_group(Group<Epi>& grp, uint8_t* ws, int slot, XcdShares& sh) {
  grp.sched = reinterpret_cast<int*>(ws + 64 * slot);
  constexpr int64_t BK = KB / (ELEM == EBF16 ? 2 : 1);
  auto steps = [&](int g) { return (std::min(grp.p[g].split_len, grp.p[g].R) + BK - 1) / BK; };
  for (int a = 1; a < grp.ng; ++a)          // stable insertion sort, descending
    for (int b = a; b > 0 && steps(b) > steps(b - 1); --b) std::swap(grp.p[b], grp.p[b - 1]);
  for (int g = 0; g < grp.ng; ++g) sh.take(grp.p[g].ntiles, grp.p[g].xb);
}

// Persistent grid over one group: 8 x (blocks per XCD), one block per
// compute unit at most.
template <int ELEM, int MA, int MB, class Epi, bool ONE = MB == KCP>
static hipError_t launch_group(Group<Epi>& grp, uint8_t* ws, hipStream_t s, bool cleared) {
  XcdShares sh(group_tiles(grp));
  if (sh.total == 0) return hipSuccess;
  prep_group<ELEM>(grp, ws, 0, sh);
  const int32_t bpx = sh.blocks();
  LaunchStatus st;
  if (!cleared) st << launch_kernel(sched_clear_kernel, dim3(1), dim3(64), s, reinterpret_cast<int*>(ws));
  st << timed_launch(s, [&] {
    return launch_kernel(gemm_v3_kernel<ELEM, MA, MB, Epi, ONE>, dim3((unsigned)(8 * bpx)), dim3(NTH), s, grp);
  });
  return st.e;
}

// Groups g1 and g2 in one launch (tile counters in slots 1 and 0).
template <int MA1, int MB1, class Epi1, int MA2, int MB2, class Epi2>
static hipError_t launch_dual(Group<Epi1>& g1, Group<Epi2>& g2, uint8_t* ws, hipStream_t s, bool cleared) {
  XcdShares sh(group_tiles(g1) + group_tiles(g2));
  if (sh.total == 0) return hipSuccess;
  prep_group<EBF16>(g1, ws, 1, sh);
  prep_group<EBF16>(g2, ws, 0, sh);
  const int32_t bpx = sh.blocks();
  LaunchStatus st;
  if (!cleared) st << launch_kernel(sched_clear_kernel, dim3(1), dim3(64), s, reinterpret_cast<int*>(ws));
  // The group with the longest tile goes first, so that the launch ends on
  // short tiles: with few tokens dX's tiles (reduction d_out) are longer than
  // dW's (reduction M), and left to the end they ran with most compute units
  // idle (backward + SR: hidden-2496 block, 237 tokens 370 -> 230 us;
  // hidden-2048, 256 tokens 214 -> 147 us; hidden-768, 512 tokens 86 -> 61 us).
  // dX goes first only where its longest tile is 1.5 times dW's, whose SR update
  // counts like 8 steps: dX's other tiles are shorter, and closer to the line
  // they and the update's end cost more (hidden 640, 1562 tokens 79 us with dW
  // first, 117 with dX; hidden 768, 2048 tokens 95 and 132; hidden 2048, 1280
  // tokens 352 and 319; of 339 calls none is slower by this rule than with dW
  // first on the one-phase loop).  Over many rounds of tiles the end matters
  // little, and dW first is the better neighbour for the caches (hidden-4096,
  // 8192 tokens, 29 rounds: 5.09 against 5.14 ms; 1024 tokens, 14 rounds: 907
  // against 889 us).  Each order is a kernel of its own: one kernel with the
  // order as an argument spilled more and was 1-2 % slower on large blocks.
  constexpr int64_t kOrderRounds = 16;
  constexpr int64_t kSrTile = Epi1::kSR ? 8 * (KB / 2) : 0;
  auto longest = [](const auto& g) { return g.ng > 0 ? std::min(g.p[0].split_len, g.p[0].R) : 0; };
  const dim3 grid((unsigned)(8 * bpx));
  st << timed_launch(s, [&] {
    if (2 * longest(g2) > 3 * longest(g1) + 2 * kSrTile && sh.total <= kOrderRounds * 8 * bpx)
      return launch_kernel(gemm_v3_dual_kernel<MA2, MB2, Epi2, MA1, MB1, Epi1>, grid, dim3(NTH), s, g2, g1);
    return launch_kernel(gemm_v3_dual_kernel<MA1, MB1, Epi1, MA2, MB2, Epi2>, grid, dim3(NTH), s, g1, g2);
  });
  return st.e;
}

}  // namespace v3

using namespace v3;

static size_t align256(size_t n) { return (n + 255) / 256 * 256; }

hipError_t launch_unpack_int3(const void* src, int8_t* dst, int64_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  SegTab tab{};
  tab.n = 1;
  tab.src[0] = src;
  tab.dst[0] = dst;
  tab.n16[0] = n / 16;
  const int32_t blocks = seal(tab);
  return launch_kernel(unpack_int3_kernel<0>, dim3(blocks), dim3(256), stream, tab);
}

hipError_t launch_unpack_int4(const void* src, int8_t* dst, int64_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  SegTab tab{};
  tab.n = 1;
  tab.src[0] = src;
  tab.dst[0] = dst;
  tab.n16[0] = n / 16;
  const int32_t blocks = seal(tab);
  return launch_kernel(unpack_int4_kernel<0>, dim3(blocks), dim3(256), stream, tab);
}

// Ternary weights reach the forward GEMM as packed codes when every d_in of
// the batch is a multiple of 64 (16-byte aligned packed rows); otherwise
// they are first unpacked into the workspace.
static bool fwd_packed(int n, const LinearIO* io) {
  for (int l = 0; l < n; ++l)
    if (io[l].d_in % 64 != 0) return false;
  return true;
}

// Forward workspace: the tile counters, then per linear the operand bytes
// its codes are expanded into (one byte per weight; FP4 uses half).  Ternary
// codes with d_in a multiple of 64 can also run straight from the packed
// codes, expanded in registers, with the counters alone: that form needs
// only fwd_batch_workspace_min, the expanded one (measured faster: the
// expansion in the main loop costs more than a pass and the extra copies)
// is taken whenever the workspace holds it.
size_t fwd_batch_workspace(int n, const LinearIO* io, int cf, size_t* offs) {
  size_t total = kSchedBytes;
  const bool unpack = cf == CF_T2 || cf == CF_I4 || cf == CF_I3;
  for (int l = 0; l < n; ++l) {
    if (offs) offs[l] = total;
    if (unpack) total += align256((size_t)(io[l].d_out * io[l].d_in));
  }
  return total;
}
size_t fwd_batch_workspace_min(int n, const LinearIO* io, int cf) {
  if (cf == CF_T2 && fwd_packed(n, io)) return kSchedBytes;
  return fwd_batch_workspace(n, io, cf, nullptr);
}

// The two-phase loop's steps are shorter, but its tiles start and end slower
// (the first step's copies and its eight barriers have nothing to overlap
// with), and a ragged last step costs it more: with few steps a tile the
// one-phase loop is ahead.  The persistent GEMM with the one-phase loop alone
// -> with two phases alone -> by this rule, us, blocks of 8192 tokens: hidden
// 256 4-bit e4m3 32.1 -> 37.6 -> 32.0, 768 4-bit e4m3 81.4 -> 93.3 -> 81.6, 1344
// (ragged) 4-bit int8 230 -> 242 -> 229, 1536 8-bit 258 -> 250 -> 250 (one phase:
// 264).  Both loops give the same bits.
static bool one_phase(const BatchCfg& c, const LinearIO* io) {
  int64_t tiles = 0, steps = 0;
  for (int l = 0; l < c.n; ++l) {
    const int64_t t = ((c.M + TILE - 1) / TILE) * ((io[l].d_out + TILE - 1) / TILE);
    tiles += t;
    steps += t * ((io[l].d_in + KB - 1) / KB - (io[l].d_in % KB != 0 ? 5 : 0));
  }
  return 2 * steps < (c.act_e4m3 ? 22 : 17) * tiles;
}

hipError_t launch_fwd_batch(const BatchCfg& c, const LinearIO* io, uint8_t* ws, size_t ws_bytes,
                           hipStream_t stream) {
  if (c.M == 0 || c.n == 0) return hipSuccess;
  LaunchStatus st;
  size_t offs[kMaxBatch];
  const size_t full =
      fwd_batch_workspace(c.n, io, c.w_ternary ? CF_T2 : c.w_int4 ? CF_I4 : c.w_int3 ? CF_I3 : CF_I8, offs);
  const bool aligned = c.w_ternary && fwd_packed(c.n, io);
  // ternary codes straight from the packed form only when the workspace
  // cannot hold their expansion
  const bool packed = aligned && ws_bytes < full;
  if (fwd_small_applies(c, io, packed)) return launch_fwd_small(c, io, stream);
  // FP4 values of ternary codes in the workspace (e4m3 activations)
  const bool fp4 = aligned && !packed && c.act_e4m3;
  // int8 (or e4m3) copy of the codes in the workspace
  const bool unpacked = (c.w_ternary && !packed && !fp4) || c.w_int4 || c.w_int3;
  if (c.w_int3) {
    SegTab tab{};
    tab.n = c.n;
    tab.sched = reinterpret_cast<int*>(ws);
    for (int l = 0; l < c.n; ++l) {
      tab.src[l] = io[l].Wq;
      tab.dst[l] = ws + offs[l];
      tab.n16[l] = io[l].d_out * io[l].d_in / 16;
    }
    const int32_t blocks = seal(tab);
    if (c.act_e4m3)
      st << launch_kernel(unpack_int3_kernel<1>, dim3(blocks), dim3(256), stream, tab);
    else
      st << launch_kernel(unpack_int3_kernel<0>, dim3(blocks), dim3(256), stream, tab);
  } else if (c.w_int4) {
    SegTab tab{};
    tab.n = c.n;
    tab.sched = reinterpret_cast<int*>(ws);
    for (int l = 0; l < c.n; ++l) {
      tab.src[l] = io[l].Wq;
      tab.dst[l] = ws + offs[l];
      tab.n16[l] = io[l].d_out * io[l].d_in / 16;
    }
    const int32_t blocks = seal(tab);
    if (c.act_e4m3)
      st << launch_kernel(unpack_int4_kernel<1>, dim3(blocks), dim3(256), stream, tab);
    else
      st << launch_kernel(unpack_int4_kernel<0>, dim3(blocks), dim3(256), stream, tab);
  } else if (fp4) {
    SegTab tab{};
    tab.n = c.n;
    tab.sched = reinterpret_cast<int*>(ws);
    for (int l = 0; l < c.n; ++l) {
      tab.src[l] = io[l].Wq;
      tab.dst[l] = ws + offs[l];
      tab.n16[l] = io[l].d_out * io[l].d_in / 16;   // a multiple of 4 (d_in of 64)
    }
    // one thread per 4 chunks
    int32_t blocks = 0;
    for (int l = 0; l < c.n; ++l) {
      tab.b0[l] = blocks;
      blocks += (int32_t)((tab.n16[l] / 4 + 255) / 256);
    }
    tab.b0[c.n] = blocks;
    st << launch_kernel(expand_fp4_kernel, dim3(blocks), dim3(256), stream, tab);
  } else if (c.w_ternary && !packed) {
    SegTab tab{};
    tab.n = c.n;
    tab.sched = reinterpret_cast<int*>(ws);
    for (int l = 0; l < c.n; ++l) {
      tab.src[l] = io[l].Wq;
      tab.dst[l] = ws + offs[l];
      tab.n16[l] = io[l].d_out * io[l].d_in / 16;
    }
    // one thread per 4 chunks
    int32_t blocks = 0;
    for (int l = 0; l < c.n; ++l) {
      tab.b0[l] = blocks;
      blocks += (int32_t)(((tab.n16[l] + 3) / 4 + 255) / 256);
    }
    tab.b0[c.n] = blocks;
    if (c.act_e4m3)
      st << launch_kernel(unpack_ternary_kernel<1>, dim3(blocks), dim3(256), stream, tab);
    else
      st << launch_kernel(unpack_ternary_kernel<0>, dim3(blocks), dim3(256), stream, tab);
  }
  Group<EpiFwd> grp{};
  grp.ng = c.n;
  for (int l = 0; l < c.n; ++l) {
    Prob<EpiFwd>& p = grp.p[l];
    p.A = Opnd{static_cast<const uint8_t*>(io[l].Xq), io[l].d_in, c.M};
    if (packed)
      p.B = Opnd{static_cast<const uint8_t*>(io[l].Wq), io[l].d_in / 4, io[l].d_out};
    else if (fp4)
      p.B = Opnd{ws + offs[l], io[l].d_in / 2, io[l].d_out};
    else if (unpacked)
      p.B = Opnd{ws + offs[l], io[l].d_in, io[l].d_out};
    else
      p.B = Opnd{static_cast<const uint8_t*>(io[l].Wq), io[l].d_in, io[l].d_out};
    p.epi = EpiFwd{io[l].Y, io[l].d_out, c.out_bf16, io[l].xdq, io[l].alpha};
    p.I = c.M;
    p.J = io[l].d_out;
    p.R = io[l].d_in;
    p.split_len = io[l].d_in;
    p.nbz = 1;
  }
  if (packed) {
    if (c.act_e4m3) st << launch_group<EF4B, KC, KCP>(grp, ws, stream, false);
    else st << launch_group<EI8, KC, KCP>(grp, ws, stream, false);
  } else if (one_phase(c, io)) {
    if (fp4) st << launch_group<EF4B, KC, KF4, EpiFwd, true>(grp, ws, stream, true);
    else if (c.act_e4m3) st << launch_group<EF8, KC, KC, EpiFwd, true>(grp, ws, stream, unpacked);
    else st << launch_group<EI8, KC, KC, EpiFwd, true>(grp, ws, stream, unpacked);
  } else {
    if (fp4) st << launch_group<EF4B, KC, KF4>(grp, ws, stream, true);
    else if (c.act_e4m3) st << launch_group<EF8, KC, KC>(grp, ws, stream, unpacked);
    else st << launch_group<EI8, KC, KC>(grp, ws, stream, unpacked);
  }
  return st.e;
}

// Backward plan for a batch in the bf16 environment: one split count for
// every dW product of the batch, and the workspace layout
//   per linear: [bf16 weights d_in x d_out][bf16 X~T d_in x Mp][fp32 partials]
// (Mp: M rounded up to a multiple of 64, the row stride of X~T)
// (partials sized for the larger of this plan's and the fp32 kernels' split).
// The split count minimises an estimate of rounds of the persistent grid x
// steps per tile plus the traffic of the partial sums.
static int64_t xt_stride(int64_t M) { return (M + 63) / 64 * 64; }

BwdPlan plan_bwd_batch(int n, const LinearIO* io, int64_t M) {
  BwdPlan P{};
  P.wi = 4;
  P.wj = 4;
  P.splits = 1;
  P.splits_dual = 1;
  const int cus = current_device_cus();
  // a step of a 256 x 256 bf16 tile is 2048 MFMA cycles, at ~2.1 GHz, plus ~2
  // us of per-tile prologue / epilogue; partials move at ~4 TB/s.  (A lower
  // bound since the power limit counts: full launches take about 1.6 us a step
  // and 12 us for the end of an SR tile.)
  constexpr double kStepUs = 2048.0 / 2100.0, kTileUs = 2.0;
  auto tiles_of = [](int64_t I, int64_t J) { return ((I + TILE - 1) / TILE) * ((J + TILE - 1) / TILE); };
  double dx_us = 0;     // dX work of the whole batch, summed over its tiles
  for (int l = 0; l < n; ++l)
    dx_us += (double)tiles_of(M, io[l].d_in) * ((double)((io[l].d_out + 63) / 64) * kStepUs + kTileUs);
  double best = 1e300, best_dual = 1e300;
  for (int64_t s = 1; s <= 32; ++s) {
    if (s > 1 && M / s < 256) break;
    int64_t tiles = 0;
    double part_bytes = 0;
    for (int l = 0; l < n; ++l) {
      tiles += tiles_of(io[l].d_out, io[l].d_in) * s;
      if (s > 1) part_bytes += (2.0 * s + 1.0) * (double)(io[l].d_out * io[l].d_in * 4);
    }
    const double rounds = (double)((tiles + cus - 1) / cus);
    const double tile_us = (double)(((M + s - 1) / s + 63) / 64) * kStepUs + kTileUs;
    // dW alone: whole rounds of equal tiles
    const double t_us = rounds * tile_us + part_bytes / 4.0e6;
    if (t_us < best * 0.999) { best = t_us; P.splits = s; }
    // dW then dX in one launch: the dW rounds, or the total work spread
    // over every compute unit, whichever is longer
    const double t_dual = std::max(rounds * tile_us, ((double)tiles * tile_us + dx_us) / cus) +
                          part_bytes / 4.0e6;
    if (t_dual < best_dual * 0.999) { best_dual = t_dual; P.splits_dual = s; }
  }
  // The SR update in the dW epilogue saves dW's store and a streaming pass
  // over it, at the price of ~173 vector instructions per 8 weights in the
  // dW tiles.  Measured per call it is the faster form on every LLaMA block
  // (hidden 768, where those tiles are the launch's critical path: 265 us
  // against 256 us of products and 12 us of update), so it is the default;
  // DQT_SR_EPILOGUE=staged in the environment stages dW in the workspace and
  // updates it in a pass of its own (same dW bits, same codes), e.g. to test
  // both forms.
  bool fuse = true;
  if (const char* f = getenv("DQT_SR_EPILOGUE")) fuse = strcmp(f, "staged") != 0;
  P.sr_fused = P.splits == 1 && fuse;
  P.sr_fused_dual = P.splits_dual == 1 && fuse;
  const bool stage_dw = (P.splits == 1 && !P.sr_fused) || (P.splits_dual == 1 && !P.sr_fused_dual);
  size_t off = kSchedBytes;
  for (int l = 0; l < n; ++l) {
    const size_t wn = (size_t)(io[l].d_out * io[l].d_in);
    const int64_t s32 = dw_splits_f32(io[l].d_out, io[l].d_in, M);
    const int64_t sp = std::max(std::max(P.splits, P.splits_dual), s32);
    P.q_off[l] = off;
    off += align256(wn * 2);
    P.xt_off[l] = off;
    off += align256((size_t)xt_stride(M) * (size_t)io[l].d_in * 2);
    P.part_off[l] = off;
    off += sp > 1 ? align256((size_t)sp * wn * 4) : stage_dw ? align256(wn * 4) : 0;
  }
  P.total = off;
  return P;
}

// dX[m, k] = alpha sum_n dY[m, n] q[n, k]: I = M, J = d_in, R = d_out.
// Fills the problems of the group and the part of the pre-pass that writes
// its B operand into the workspace.
static void prep_dx(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                    Group<EpiScale>& grp, PrepTab& prep) {
  grp.ng = c.n;
  for (int l = 0; l < c.n; ++l) {
    Prob<EpiScale>& p = grp.p[l];
    p.A = Opnd{static_cast<const uint8_t*>(io[l].dY), io[l].d_out * 2, c.M};
    p.epi = EpiScale{io[l].dX, io[l].d_in, c.out_bf16, io[l].alpha};
    p.I = c.M;
    p.J = io[l].d_in;
    p.R = io[l].d_out;
    p.split_len = io[l].d_out;
    p.nbz = 1;
  }
  // bf16 weights transposed (reduction contiguous), so both operands are
  // read without the transposing LDS reads
  TrTab& tab = prep.tr;
  tab.n = c.n;
  int32_t blocks = 0;
  for (int l = 0; l < c.n; ++l) {
    tab.src[l] = static_cast<const uint8_t*>(io[l].Wq);
    tab.dst[l] = reinterpret_cast<uint16_t*>(ws + P.q_off[l]);
    tab.d_out[l] = (int32_t)io[l].d_out;
    tab.d_in[l] = (int32_t)io[l].d_in;
    tab.tn[l] = (int32_t)((io[l].d_out + 63) / 64);
    tab.b0[l] = blocks;
    // ternary: strips of 512 reduction elements; else 64 x 64 tiles
    const int kspan = c.w_ternary ? 512 : 64;
    blocks += tab.tn[l] * (int32_t)((io[l].d_in + kspan - 1) / kspan);
    grp.p[l].B = Opnd{ws + P.q_off[l], io[l].d_out * 2, io[l].d_in};
  }
  tab.b0[c.n] = blocks;
  prep.n_tr = blocks;
}

template <int CF>
static hipError_t launch_prep_cf(const BatchCfg& c, const PrepTab& prep, hipStream_t stream) {
  const dim3 grid((unsigned)(prep.n_tr + prep.n_dq));
  if (c.act_e4m3) return launch_kernel(bwd_prep_kernel<CF, true>, grid, dim3(256), stream, prep);
  return launch_kernel(bwd_prep_kernel<CF, false>, grid, dim3(256), stream, prep);
}
// The pre-pass; `cleared` tells whether it ran (and so cleared the counters).
static hipError_t launch_prep(const BatchCfg& c, PrepTab& prep, uint8_t* ws, hipStream_t stream, bool* cleared) {
  *cleared = prep.n_tr + prep.n_dq > 0;
  if (!*cleared) return hipSuccess;
  prep.sched = reinterpret_cast<int*>(ws);
  if (c.w_ternary) return launch_prep_cf<CF_T2>(c, prep, stream);
  if (c.w_int4) return launch_prep_cf<CF_I4>(c, prep, stream);
  if (c.w_int3) return launch_prep_cf<CF_I3>(c, prep, stream);
  return launch_prep_cf<CF_I8>(c, prep, stream);
}

hipError_t launch_dx_batch(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                           hipStream_t stream) {
  if (c.M == 0 || c.n == 0) return hipSuccess;
  Group<EpiScale> grp{};
  PrepTab prep{};
  LaunchStatus st;
  bool cleared;
  prep_dx(c, io, ws, P, grp, prep);
  st << launch_prep(c, prep, ws, stream, &cleared);
  st << launch_group<EBF16, KC, KC>(grp, ws, stream, cleared);
  return st.e;
}

// X~T once per distinct quantised input (the dequantising transpose of the
// pre-pass); first[l] is the linear whose X~T linear l reads.
static void prep_xt(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                    int* first, PrepTab& prep) {
  DqTab& tab = prep.dq;
  tab.M = c.M;
  tab.Mp = xt_stride(c.M);
  int32_t blocks = 0;
  for (int l = 0; l < c.n; ++l) {
    first[l] = l;
    for (int m = 0; m < l; ++m)
      if (io[m].Xq == io[l].Xq && io[m].d_in == io[l].d_in) { first[l] = first[m]; break; }
    if (first[l] == l && c.M > 0) {
      const int s = tab.n++;
      tab.src[s] = static_cast<const uint8_t*>(io[l].Xq);
      tab.dst[s] = reinterpret_cast<uint16_t*>(ws + P.xt_off[l]);
      tab.scale[s] = io[l].xdq;
      tab.K[s] = (int32_t)io[l].d_in;
      tab.tm[s] = (int32_t)((c.M + 63) / 64);
      tab.b0[s] = blocks;
      blocks += tab.tm[s] * (int32_t)((io[l].d_in + 63) / 64);
    }
  }
  tab.b0[tab.n] = blocks;
  prep.n_dq = blocks;
}

// dW[n, k] = sum_m dY[m, n] X~T[k, m]: I = d_out, J = d_in, R = M, split over
// the batch into P.splits parts; make(l) gives linear l's epilogue.
template <class Epi, class MakeEpi>
static void fill_dw(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                    const int* first, Group<Epi>& grp, MakeEpi make) {
  const int64_t splits = P.splits;
  int64_t len = splits > 1 ? (c.M + splits - 1) / splits : (c.M > 0 ? c.M : 1);
  len = (len + 63) / 64 * 64;
  grp.ng = c.n;
  for (int l = 0; l < c.n; ++l) {
    Prob<Epi>& p = grp.p[l];
    const int64_t I = io[l].d_out, J = io[l].d_in;
    p.A = Opnd{static_cast<const uint8_t*>(io[l].dY), I * 2, I};
    p.B = Opnd{ws + P.xt_off[first[l]], xt_stride(c.M) * 2, J};
    p.epi = make(l);
    p.I = I;
    p.J = J;
    p.R = c.M;
    p.split_len = len;
    p.nbz = (int32_t)splits;
  }
}

// dW into dW (one split) or into the workspace partials (several).
static void prep_dw(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                    Group<EpiPartial>& grp, PrepTab& prep) {
  int first[kMaxBatch];
  prep_xt(c, io, ws, P, first, prep);
  fill_dw(c, io, ws, P, first, grp, [&](int l) {
    const int64_t I = io[l].d_out, J = io[l].d_in;
    float* target = P.splits > 1 ? reinterpret_cast<float*>(ws + P.part_off[l]) : io[l].dW;
    return EpiPartial{target, J, I * J};
  });
}

// Sum of the batch-split dW partials into dW.
static hipError_t reduce_dw(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                            hipStream_t stream) {
  if (P.splits == 1) return hipSuccess;
  LaunchStatus st;
  RedTab red{};
  red.n = c.n;
  red.splits = (int32_t)P.splits;
  int32_t blocks = 0;
  for (int l = 0; l < c.n; ++l) {
    red.src[l] = reinterpret_cast<const float*>(ws + P.part_off[l]);
    red.dst[l] = io[l].dW;
    red.n4[l] = io[l].d_out * io[l].d_in / 4;
    red.b0[l] = blocks;
    blocks += (int32_t)((red.n4[l] + 255) / 256);
  }
  red.b0[c.n] = blocks;
  st << launch_kernel(split_reduce_batch_kernel, dim3((unsigned)blocks), dim3(256), stream, red);
  return st.e;
}

hipError_t launch_dw_batch(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                           hipStream_t stream) {
  if (c.n == 0) return hipSuccess;
  Group<EpiPartial> grp{};
  PrepTab prep{};
  LaunchStatus st;
  bool cleared;
  prep_dw(c, io, ws, P, grp, prep);
  st << launch_prep(c, prep, ws, stream, &cleared);
  st << launch_group<EBF16, KM, KC>(grp, ws, stream, cleared);
  if (st.e != hipSuccess) return st.e;
  return reduce_dw(c, io, ws, P, stream);
}

// dW and dX of a batch in one persistent launch: the tiles of one product,
// then the other's (launch_dual has the order), so compute units that draw no
// tile of the first, or finish theirs early, go on with the second at once.
hipError_t launch_dxdw_batch(const BatchCfg& c, const LinearIO* io, uint8_t* ws, const BwdPlan& P,
                             hipStream_t stream) {
  if (c.n == 0) return hipSuccess;
  if (c.M == 0) {
    const hipError_t e = launch_dx_batch(c, io, ws, P, stream);
    return e != hipSuccess ? e : launch_dw_batch(c, io, ws, P, stream);
  }
  Group<EpiScale> gx{};
  Group<EpiPartial> gw{};
  BwdPlan Q = P;
  Q.splits = P.splits_dual;
  PrepTab prep{};
  LaunchStatus st;
  bool cleared;
  prep_dx(c, io, ws, Q, gx, prep);
  prep_dw(c, io, ws, Q, gw, prep);
  st << launch_prep(c, prep, ws, stream, &cleared);
  st << launch_dual<KM, KC, EpiPartial, KC, KC, EpiScale>(gw, gx, ws, stream, cleared);
  if (st.e != hipSuccess) return st.e;
  return reduce_dw(c, io, ws, Q, stream);
}

// Partials of a batch-split dW summed and consumed by the SR update.
static hipError_t reduce_sr(const BatchCfg& c, const LinearIO* io, const SRTensor* t, uint64_t seed,
                            uint32_t step, unsigned long long* counters, uint8_t* ws,
                            const BwdPlan& P, hipStream_t stream) {
  LaunchStatus st;
  RedSRTab red{};
  red.n = c.n;
  red.splits = (int32_t)P.splits;
  red.k0 = (uint32_t)seed;
  red.k1 = (uint32_t)(seed >> 32);
  red.step = step;
  red.counters = counters;
  int32_t blocks = 0;
  for (int l = 0; l < c.n; ++l) {
    red.src[l] = reinterpret_cast<const float*>(ws + P.part_off[l]);
    red.wq[l] = t[l].wq;
    red.n8[l] = io[l].d_out * io[l].d_in / 8;
    red.c[l] = t[l].c;
    red.L[l] = (float)(t[l].qmax - t[l].qmin + 1);
    red.qmin[l] = t[l].qmin;
    red.qmax[l] = t[l].qmax;
    red.tid[l] = t[l].tensor_id;
    red.b0[l] = blocks;
    blocks += (int32_t)((red.n8[l] + 255) / 256);
  }
  red.b0[c.n] = blocks;
  if (c.w_ternary)
    st << launch_kernel(split_reduce_sr_kernel<CF_T2>, dim3((unsigned)blocks), dim3(256), stream, red);
  else if (c.w_int4)
    st << launch_kernel(split_reduce_sr_kernel<CF_I4>, dim3((unsigned)blocks), dim3(256), stream, red);
  else if (c.w_int3)
    st << launch_kernel(split_reduce_sr_kernel<CF_I3>, dim3((unsigned)blocks), dim3(256), stream, red);
  else
    st << launch_kernel(split_reduce_sr_kernel<CF_I8>, dim3((unsigned)blocks), dim3(256), stream, red);
  return st.e;
}

// dW of every linear consumed by the SR update of its codes in the GEMM
// epilogue (one split) or in the reduction of the partials (several), with
// dX of every linear in the same launch when with_dx.
template <int CF>
static hipError_t launch_dw_sr_group(const BatchCfg& c, const LinearIO* io, const SRTensor* t, uint64_t seed,
                               uint32_t step, unsigned long long* counters, uint8_t* ws,
                               const BwdPlan& P, const int* first, Group<EpiScale>* gx,
                               bool cleared, hipStream_t stream) {
  Group<EpiSR<CF>> gw{};
  fill_dw(c, io, ws, P, first, gw, [&](int l) {
    EpiSR<CF> e;
    e.wq = t[l].wq;
    e.ldc = io[l].d_in / 8 * chunk_code_bytes<CF>();
    e.d_in = io[l].d_in;
    e.c = t[l].c;
    e.L = (float)(t[l].qmax - t[l].qmin + 1);
    e.qmin = t[l].qmin;
    e.qmax = t[l].qmax;
    e.k0 = (uint32_t)seed;
    e.k1 = (uint32_t)(seed >> 32);
    e.step = step;
    e.tid = t[l].tensor_id;
    e.counters = counters;
    return e;
  });
  // dW^T = X~^T dY: X~^T [d_in][Mp] (K-contiguous) as the first operand,
  // dY [M][d_out] (K-major) as the second
  for (int l = 0; l < c.n; ++l) {
    Prob<EpiSR<CF>>& p = gw.p[l];
    const int64_t I = io[l].d_in, J = io[l].d_out;
    p.A = Opnd{ws + P.xt_off[first[l]], xt_stride(c.M) * 2, I};
    p.B = Opnd{static_cast<const uint8_t*>(io[l].dY), J * 2, J};
    p.I = I;
    p.J = J;
  }
  if (gx != nullptr) return launch_dual<KC, KM, EpiSR<CF>, KC, KC, EpiScale>(gw, *gx, ws, stream, cleared);
  return launch_group<EBF16, KC, KM, EpiSR<CF>>(gw, ws, stream, cleared);
}

hipError_t launch_bwd_sr_batch(const BatchCfg& c, const LinearIO* io, const SRTensor* t, uint64_t seed,
                               uint32_t step, unsigned long long* counters, bool with_dx, uint8_t* ws,
                               const BwdPlan& P, hipStream_t stream) {
  if (c.n == 0 || c.M == 0) return hipSuccess;
  BwdPlan Q = P;
  Q.splits = with_dx ? P.splits_dual : P.splits;
  const bool fused = with_dx ? P.sr_fused_dual : P.sr_fused;
  Group<EpiScale> gx{};
  PrepTab prep{};
  LaunchStatus st;
  bool cleared;
  if (with_dx) prep_dx(c, io, ws, Q, gx, prep);
  int first[kMaxBatch];
  prep_xt(c, io, ws, Q, first, prep);
  st << launch_prep(c, prep, ws, stream, &cleared);
  if (Q.splits == 1 && fused) {
    Group<EpiScale>* const pgx = with_dx ? &gx : nullptr;
    if (c.w_ternary) st << launch_dw_sr_group<CF_T2>(c, io, t, seed, step, counters, ws, Q, first, pgx, cleared, stream);
    else if (c.w_int4) st << launch_dw_sr_group<CF_I4>(c, io, t, seed, step, counters, ws, Q, first, pgx, cleared, stream);
    else if (c.w_int3) st << launch_dw_sr_group<CF_I3>(c, io, t, seed, step, counters, ws, Q, first, pgx, cleared, stream);
    else st << launch_dw_sr_group<CF_I8>(c, io, t, seed, step, counters, ws, Q, first, pgx, cleared, stream);
    return st.e;
  }
  Group<EpiPartial> gw{};
  fill_dw(c, io, ws, Q, first, gw, [&](int l) {
    const int64_t I = io[l].d_out, J = io[l].d_in;
    return EpiPartial{reinterpret_cast<float*>(ws + Q.part_off[l]), J, I * J};
  });
  if (with_dx)
    st << launch_dual<KM, KC, EpiPartial, KC, KC, EpiScale>(gw, gx, ws, stream, cleared);
  else
    st << launch_group<EBF16, KM, KC, EpiPartial>(gw, ws, stream, cleared);
  if (st.e != hipSuccess) return st.e;
  return reduce_sr(c, io, t, seed, step, counters, ws, Q, stream);
}

}  // namespace dqt
