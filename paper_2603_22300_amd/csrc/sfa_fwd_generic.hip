// SFA forward (Sec. 3.1-3.2) on the matrix cores for the shapes that the tuned
// forward does not take: any head dimension d <= 256 and any group size, with
// no workspace, at float32 accuracy.
//
// Scores: the code values (queries with scale * log2(e) folded in, so that a
// score is a base-2 exponent) are densified as three bfloat16 pieces
// x0 = bf16(x) (the largest bf16 for a float32 past it), x1 = bf16(x - x0), x2 =
// bf16(x - x0 - x1), which hold any float32 of magnitude 2^-109 or more, smaller
// ones to 2^-134, and every product of order <= 2 is kept (~2^-24).  16-bit code values with bf16 V (KX) are their own operands: one
// exact product, the scale (bf16: but its power of two) applied to the float32 score.  P.V: V in bf16 is
// exact (float32 V: three pieces), P enters as three bf16 pieces.  Error against 64
// bits (float32 O, 2-norm; the vector-unit kernel this replaced in brackets): with
// codes of three times the usual size, 1535 rows at d = 128 O 2.6e-7 (4.5e-7), 1000
// at d = 192 2.7e-7 (4.2e-7); LSE 4.1e-8 and 5.1e-8 (4.6e-8, 5.4e-8).
//
// A workgroup takes R = 32 NW / KG query rows: gs heads of one KV head (the
// largest power of two <= 4 in the group) times BR = R / gs positions, so that a
// wavefront's 32 rows are one head.  Per tile of 32 KG keys the workgroup
// densifies the codes and copies V into LDS, both straight from the caller's
// arrays, rows of V kept row-major and read transposed (sfa_tile.h); wavefront
// (rg, kg) works on rows 32 rg.. and keys 32 kg.. of the tile.  With KG = 2 the
// two wavefronts of a row group split the keys and merge by their LSE at the
// end: that halves the serial chain of the longest causal block, which sets
// the time of sequences of a few thousand tokens, and gives each SIMD two
// waves.  d > 128 (KG = 1, 4 wavefronts) has one wave per SIMD for its operands
// and still spills with 32-bit codes: 73 registers (292 bytes of scratch a lane) with
// bf16 V, 96 (388) with float32 V; 16-bit codes spill none, and at d in (96, 128]
// float32 V spills 16.  Rows, V and O of any alignment (vec: 16-byte loads where d and
// the arrays allow).
//
// Bound by the chain of one tile (stage, scores, softmax, P.V, barrier: about
// 5.3 us with 48 + 24 MFMAs per wavefront and 32 x 32 tile at d = 128, 4 with
// 16-bit codes' 8 + 24) at two waves per SIMD.  Measured against the float32
// vector-unit kernel it replaces (k + 2d multiply-adds per pair, 32 rows per
// workgroup), us per call: batch 2, 12 query over 2 KV heads, n = 1535, d = 128, k =
// 16: 2528 -> 150 (16-bit codes 2536 -> 110, float32 V and O 2573 -> 204); batch 4, 8
// heads, n = 1000, d = 96: 974 -> 68; 8 heads, n = 1000: d = 256 1546 -> 230, d = 192
// with float32 V 1269 -> 297; 5 heads, n = 100: 82 -> 14.5.  Of these the third piece of
// P, the sums that keep the error at the other kernel's and the exact maximum take 5%
// (16-bit codes 15%).  Letting one wavefront of a SIMD stage while the other
// computes changed nothing.
#include <math.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "sfa_device.h"
#include "sfa_launch.h"
#include "sfa_tile.h"

namespace sfa {
namespace {

constexpr int kGDmax = 256;
constexpr float kBf16Max = 0x1.fep127f;

struct GenParams {
  const void* q_idx;
  const void* q_val;
  const void* k_idx;
  const void* k_val;
  const void* v;
  void* o;
  float* lse;
  int Hq, Hkv, n, d, k, causal, window, n_global;
  // The factors of the query values and of the scores; their product is scale *
  // log2(e), so that a score is a base-2 exponent (launch_attn_fwd_generic).
  float q_mul, s_mul;
  int ifmt, vfmt, obf16;
  int G, gs, BR, nqb;  // group size; heads and positions of a workgroup; blocks per head group
  float inv_k;
  int vec;  // d % 8 == 0 and V, O 16-byte aligned
};

// D: head dimension padded; NV: bf16 pieces of V (1: bf16 V, 3: float32 V);
// KX: 0, or the 16-bit code value type (one raw piece).
template <int D_, int NW_, int KG_, int NV_, int KX_>
struct GGeo {
  static constexpr int D = D_, NW = NW_, KG = KG_, NV = NV_, KX = KX_;
  static constexpr int NT = 64 * NW, RG = NW / KG, R = 32 * RG, KT = 32 * KG;
  static constexpr int NP = KX ? 1 : 3, NKB = D / 16, NDB = D / 32;
  static constexpr int QP = D + 8;       // pitch of a densified query row (setup), 16-bit
  static constexpr int KR = NP * D + 8;  // pitch of a key row, 16-bit: conflict-free 16-byte reads
  // pitch of a V row, bytes: the least with 16 or 48 banks modulo 64 (sfa_tile.h)
  static constexpr int V0 = NV * D * 2;
  static constexpr int VR = V0 - V0 % 256 + (V0 % 256 <= 64 ? 64 : V0 % 256 <= 192 ? 192 : 320);
  static constexpr int SB = KT * (2 * KR + VR);             // a stage
  static constexpr int NS = 2 * SB <= 160 * 1024 ? 2 : 1;   // stages
  static constexpr int MERGE = KG == 2 ? RG * 64 * (16 * NDB + 2) * 4 : 0;
  static constexpr int LDS = std::max(std::max(NS * SB, R * QP * 2), MERGE);
  static_assert(LDS <= 160 * 1024, "fits LDS");
  static constexpr int KW = KT / NW;                         // key rows a wavefront densifies
  static constexpr int VCH = KT * (D / 8);                   // 8-value chunks of a V tile
  static constexpr int VI = (VCH + NT - 1) / NT;             // of them per thread
  static constexpr int VW = NV == 1 ? 1 : 2;                 // 16-byte loads per chunk
};

// N code entries as stored, then one of them as (coordinate, value): the loads
// carry no arithmetic, so that nothing waits for them before they are used.
// The coordinate is clamped into [0, d): a violated precondition cannot
// address outside the tables.
template <int N>
__device__ __forceinline__ void load_entries(const void* idx, const void* val, const int64_t (&at)[N],
                                             int ifmt, int vfmt, uint32_t (&ri)[N], uint32_t (&rv)[N]) {
  if (ifmt == kIdxI16) {
#pragma unroll
    for (int r = 0; r < N; ++r) ri[r] = ((const uint16_t*)idx)[at[r]];
  } else if (ifmt == kIdxU8) {
#pragma unroll
    for (int r = 0; r < N; ++r) ri[r] = ((const uint8_t*)idx)[at[r]];
  } else {
#pragma unroll
    for (int r = 0; r < N; ++r) ri[r] = ((const uint32_t*)idx)[at[r]];
  }
  if (vfmt == kValF32) {
#pragma unroll
    for (int r = 0; r < N; ++r) rv[r] = ((const uint32_t*)val)[at[r]];
  } else {
#pragma unroll
    for (int r = 0; r < N; ++r) rv[r] = ((const uint16_t*)val)[at[r]];
  }
}
__device__ __forceinline__ int entry_idx(uint32_t raw, int ifmt, int d) {
  const int u = ifmt == kIdxI16 ? (int)(int16_t)raw : (int)raw;
  return min(max(u, 0), d - 1);
}
__device__ __forceinline__ float entry_val(uint32_t raw, int vfmt) {
  if (vfmt == kValF32) return __uint_as_float(raw);
  return vfmt == kValBF16 ? bf16_bits_to_f32(raw) : f16_bits_to_f32(raw);
}

// bf16 piece `pc` of x (0: nearest finite bf16; 1, 2: bf16 of the remaining error)
__device__ __forceinline__ uint16_t gen_piece(float x, int pc) {
  const uint32_t h = f32_to_bf16_rne(__builtin_amdgcn_fmed3f(x, -kBf16Max, kBf16Max));
  if (pc == 0) return (uint16_t)h;
  const float r1 = x - bf16_bits_to_f32(h);
  const uint32_t m = f32_to_bf16_rne(r1);
  if (pc == 1) return (uint16_t)m;
  return (uint16_t)f32_to_bf16_rne(r1 - bf16_bits_to_f32(m));
}

template <class Ge>
__global__ __launch_bounds__(Ge::NT) void sfa_fwd_generic_kernel(GenParams p) {
  constexpr int D = Ge::D, NW = Ge::NW, KG = Ge::KG, NV = Ge::NV, KX = Ge::KX, NT = Ge::NT;
  constexpr int RG = Ge::RG, R = Ge::R, KT = Ge::KT, NP = Ge::NP, NKB = Ge::NKB, NDB = Ge::NDB;
  constexpr int QP = Ge::QP, KR = Ge::KR, VR = Ge::VR, SB = Ge::SB, NS = Ge::NS, KW = Ge::KW;
  constexpr int VCH = Ge::VCH, VI = Ge::VI, VW = Ge::VW;
  constexpr int PP = 3;  // bf16 pieces of P
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hh = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave % RG, kg = wave / RG;
  const int n = p.n, d = p.d, k = p.k;
  // XCD-aware placement as the tuned forward's: with the head groups a
  // multiple of 8, XCD x runs those congruent to x; longest causal blocks first
  int qb = (int)blockIdx.x, hg = (int)blockIdx.y;
  if (gridDim.y % 8 == 0) {
    const int id = qb + hg * p.nqb, j = id >> 3;
    qb = j % p.nqb;
    hg = (id & 7) + 8 * (j / p.nqb);
  }
  qb = p.nqb - 1 - qb;
  const int ngs = p.Hq / p.gs;
  const int b = hg / ngs, hq0 = (hg - b * ngs) * p.gs, hkv = hq0 / p.G;
  const int i0 = qb * p.BR;
  const int hq = hq0 + rg * 32 / p.BR, pos0 = i0 + rg * 32 % p.BR;
  const int my_i = pos0 + l32;
  const bool row_ok = my_i < n;
  const int wave_last = min(n, pos0 + 32) - 1;
  const int64_t kv_row0 = ((int64_t)b * p.Hkv + hkv) * n;

  // key tiles of the block: up to the causal limit, or with a token window (and
  // no global row here) the global tiles [0, gt_end) and those from wt_begin on
  const bool win = p.window > 0;
  const int blk_last = min(n, i0 + p.BR) - 1;
  int n_keys = p.causal ? blk_last + 1 : n, gt_end = 0, wt_begin = 0;
  if (win && i0 >= p.n_global) {
    if (!p.causal) n_keys = (int)min((int64_t)n, (int64_t)blk_last + p.window);
    gt_end = (p.n_global + KT - 1) / KT;
    wt_begin = max(0, i0 - p.window + 1) / KT;
    if (wt_begin <= gt_end) gt_end = wt_begin = 0;
  }
  const int ntiles = gt_end + (n_keys + KT - 1) / KT - wt_begin;
  auto tile_at = [&](int t) { return t < gt_end ? t : wt_begin + (t - gt_end); };

  // ---- one tile: global -> registers -> LDS stage ------------------------
  // Each wavefront densifies KW key rows (the first two code entries of a lane
  // are loaded a tile ahead: all of them for k <= 16) and the workgroup copies V.
  int k_row[2], k_off[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int el = lane + 64 * r;
    k_row[r] = el < KW * k ? wave * KW + (int)(((float)el + 0.5f) * p.inv_k) : -1;
    k_off[r] = wave * KW * k + el;
  }
  uint32_t ki[2], kv[2];
  uint4 vr[VI][VW];
  auto load_tile = [&](int jt) {
    const int j0 = jt * KT;
    int64_t at[2];  // (entries past the sequence or the wave's rows re-read the head's first)
#pragma unroll
    for (int r = 0; r < 2; ++r)
      at[r] = kv_row0 * k + (k_row[r] >= 0 && j0 + k_row[r] < n ? (int64_t)j0 * k + k_off[r] : 0);
    load_entries(p.k_idx, p.k_val, at, p.ifmt, p.vfmt, ki, kv);
    if (p.vec) {
#pragma unroll
      for (int r = 0; r < VI; ++r) {
        const int c = tid + r * NT, j = c / (D / 8), c8 = c % (D / 8) * 8;
#pragma unroll
        for (int w = 0; w < VW; ++w) {
          const int64_t at_v = c < VCH && j0 + j < n && c8 < d ? (int64_t)(j0 + j) * d + c8 : 0;
          vr[r][w] = *(const uint4*)((const unsigned char*)p.v +
                                     (kv_row0 * d + at_v) * (NV == 1 ? 2 : 4) + 16 * w);
        }
      }
    }
  };
  auto write_tile = [&](int stage, int jt) {
    const int j0 = jt * KT;
    uint16_t* Kd = (uint16_t*)(smem + stage * SB);
    unsigned char* Vt = smem + stage * SB + KT * KR * 2;
    constexpr int RU4 = NP * D / 8;  // uint4 per key row, padding excluded
    for (int x = lane; x < KW * RU4; x += 64)
      *(uint4*)(Kd + (wave * KW + x / RU4) * KR + x % RU4 * 8) = make_uint4(0u, 0u, 0u, 0u);
    // (entries past the sequence go to the row's padding, never read)
    auto put = [&](int row, bool ok, uint32_t ri, uint32_t rv) {
      const int f = entry_idx(ri, p.ifmt, d);
      const float x = KX != 0 ? 0.f : entry_val(rv, p.vfmt);
#pragma unroll
      for (int pc = 0; pc < NP; ++pc)
        Kd[row * KR + (ok ? pc * D + f : NP * D + pc)] = KX != 0 ? (uint16_t)rv : gen_piece(x, pc);
    };
#pragma unroll
    for (int r = 0; r < 2; ++r)
      put(max(k_row[r], wave * KW), k_row[r] >= 0 && j0 + k_row[r] < n, ki[r], kv[r]);
    for (int el = lane + 128; el < KW * k; el += 64) {
      const int row = wave * KW + (int)(((float)el + 0.5f) * p.inv_k);
      const int64_t at[1] = {(kv_row0 + j0) * k + wave * KW * k + el};
      uint32_t ri[1], rv[1];
      if (j0 + row < n) {
        load_entries(p.k_idx, p.k_val, at, p.ifmt, p.vfmt, ri, rv);
        put(row, true, ri[0], rv[0]);
      }
    }
#pragma unroll
    for (int r = 0; r < VI; ++r) {
      const int c = tid + r * NT, j = c / (D / 8), c8 = c % (D / 8) * 8;
      if (VCH % NT != 0 && c >= VCH) break;
      if constexpr (NV == 1) {
        uint4 w = j0 + j < n && c8 < d ? vr[r][0] : make_uint4(0u, 0u, 0u, 0u);
        if (!p.vec) {
          uint32_t h[8];
#pragma unroll
          for (int e = 0; e < 8; ++e)
            h[e] = j0 + j < n && c8 + e < d ? ((const uint16_t*)p.v)[(kv_row0 + j0 + j) * d + c8 + e] : 0u;
          w = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
        }
        *(uint4*)(Vt + img_pos<VR>(j, c8)) = w;
      } else {
        const uint4 w0 = vr[r][0], w1 = vr[r][VW - 1];
        const uint32_t w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = j0 + j < n && c8 < d ? __uint_as_float(w[e]) : 0.f;
        if (!p.vec) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            x[e] = j0 + j < n && c8 + e < d ? ((const float*)p.v)[(kv_row0 + j0 + j) * d + c8 + e] : 0.f;
        }
#pragma unroll
        for (int pc = 0; pc < 3; ++pc) {
          uint32_t h[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) h[e] = gen_piece(x[e], pc);
          *(uint4*)(Vt + img_pos<VR>(j, pc * D + c8)) =
              make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
        }
      }
    }
  };

  // ---- query operand: the densified rows' pieces, through LDS -------------
  bf16x8 qB[NP][NKB];
  {
    uint16_t* Qs = (uint16_t*)smem;
    for (int x = tid; x < R * QP / 8; x += NT) ((uint4*)Qs)[x] = make_uint4(0u, 0u, 0u, 0u);
    const int lbr = __builtin_ctz(p.BR);
    // code entry e of the block: row e / k; -1 where it has none.  The first QE
    // of a thread (all of them for k <= 16) are loaded once, for every piece.
    constexpr int QE = R * 16 / NT;
    auto entry_at = [&](int e, int& row) -> int64_t {
      row = (int)(((float)e + 0.5f) * p.inv_k);
      const int i = i0 + (row & (p.BR - 1));
      const bool ok = e < R * k && i < n;
      const int64_t at = (((int64_t)b * p.Hq + hq0 + (row >> lbr)) * n + i) * k + (e - row * k);
      if (!ok) row = -1;
      return ok ? at : 0;
    };
    int qrow[QE];
    int64_t at[QE];
    uint32_t qi[QE], qv[QE];
#pragma unroll
    for (int u = 0; u < QE; ++u) at[u] = entry_at(tid + NT * u, qrow[u]);
    load_entries(p.q_idx, p.q_val, at, p.ifmt, p.vfmt, qi, qv);
    auto put = [&](int row, uint32_t ri, uint32_t rv, int pc) {
      if (row < 0) return;
      const float x = p.q_mul * entry_val(rv, p.vfmt);
      Qs[row * QP + entry_idx(ri, p.ifmt, d)] =
          KX == kValF16 ? __builtin_bit_cast(uint16_t, (_Float16)x) : gen_piece(x, pc);
    };
#pragma unroll
    for (int pc = 0; pc < NP; ++pc) {
      __syncthreads();  // zeroed, or the previous piece is read
#pragma unroll
      for (int u = 0; u < QE; ++u) put(qrow[u], qi[u], qv[u], pc);
      for (int e = tid + NT * QE; e < R * k; e += NT) {
        int row;
        const int64_t at1[1] = {entry_at(e, row)};
        uint32_t ri[1], rv[1];
        load_entries(p.q_idx, p.q_val, at1, p.ifmt, p.vfmt, ri, rv);
        put(row, ri[0], rv[0], pc);
      }
      __syncthreads();
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
        qB[pc][kb] = *(const bf16x8*)(Qs + (rg * 32 + l32) * QP + kb * 16 + 8 * hh);
    }
    __syncthreads();  // Qs overlaps the stages
  }

  float m_run = -INFINITY, l_run = 0.f;
  floatx16 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
  const LaneOff<VR> vo(lane);

  // ---- this wavefront's 32 x 32 scores of a tile, softmax, P.V ------------
  auto compute = [&](int stage, int jt) {
    const int j0 = jt * KT + 32 * kg;
    const bool seen = pos0 < n && j0 < n && (!p.causal || j0 <= wave_last) &&
                      (!win || j0 < p.n_global || pos0 < p.n_global ||
                       (j0 + 31 > pos0 - p.window && j0 < (int64_t)wave_last + p.window));
    if (!seen) return;  // uniform per wavefront
    const uint16_t* Kd = (const uint16_t*)(smem + stage * SB) + (32 * kg + l32) * KR + 8 * hh;
    const unsigned char* Vt = smem + stage * SB + KT * KR * 2 + 32 * kg * VR;
    // S^T: lane = row my_i, register r = key j0 + 8 (r / 4) + 4 hh + r % 4
    // in two sums, the products of the first pieces and the rest (s_lo): what the
    // large terms round off is then as much as in a sum of full products
    floatx16 s, s_lo;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = s_lo[r] = 0.f;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      bf16x8 a[NP];
#pragma unroll
      for (int pc = 0; pc < NP; ++pc) a[pc] = *(const bf16x8*)(Kd + pc * D + kb * 16);
      if constexpr (KX == kValF16) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a[0]),
                                                   __builtin_bit_cast(f16x8, qB[0][kb]), s, 0, 0, 0);
      } else {
#pragma unroll
        for (int o = NP - 1; o > 0; --o)
#pragma unroll
          for (int pc = o; pc >= 0; --pc)
            s_lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pc], qB[o - pc][kb], s_lo, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], qB[0][kb], s, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = KX != 0 ? s[r] * p.s_mul : s[r] + s_lo[r];
    // every (row, key) pair of the sub-tile allowed: no element mask
    const bool wcut = win && j0 + 32 > p.n_global &&
                      (pos0 < p.n_global || wave_last - j0 >= p.window || j0 + 31 - pos0 >= p.window);
    const bool full = pos0 + 32 <= n && j0 + 32 <= n && (!p.causal || j0 + 31 <= pos0) && !wcut;
    uint32_t pw[2][PP][4];  // [16-key block][piece], as bf16 pairs
    auto softmax = [&](auto full_c) {
      float mt = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if constexpr (!decltype(full_c)::value) {
          const int j = j0 + 8 * (r >> 2) + 4 * hh + (r & 3);
          // (bitwise: no branch per element)
          const bool ok = row_ok & (j < n) & (!p.causal | (j <= my_i)) &
                          (!win | (abs(my_i - j) < p.window) | (j < p.n_global) | (my_i < p.n_global));
          s[r] = ok ? s[r] : -INFINITY;
        }
        mt = fmaxf(mt, s[r]);
      }
      mt = pair_max(mt);
      const bool upd = mt > m_run;
      if (__builtin_amdgcn_ballot_w64(upd)) {
        const float alpha = upd ? __builtin_amdgcn_exp2f(m_run - mt) : 1.f;
        m_run = upd ? mt : m_run;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[db][r] *= alpha;
      }
      const float m_use = m_run == -INFINITY ? 0.f : m_run;
      // (the tile's sum apart from the running one: a rounding of the large sum
      // per tile, not per key)
      float lt = 0.f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        float x[2];
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          x[y] = __builtin_amdgcn_exp2f(s[r + y] - m_use);
          lt += x[y];
        }
#pragma unroll
        for (int pc = 0; pc < PP; ++pc) {
          const f32x2 v = {x[0], x[1]};
          const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
          pw[r >> 3][pc][(r & 7) >> 1] = w;
          x[0] -= __uint_as_float(w << 16);
          x[1] -= __uint_as_float(w & 0xffff0000u);
        }
      }
      l_run += lt;
    };
    if (full) softmax(std::true_type{});
    else softmax(std::false_type{});
    // O^T += V^T P^T, products of order < max(NV, PP), smaller terms first
    constexpr int ORD = NV > PP ? NV : PP;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      bf16x8 pb[PP];
#pragma unroll
      for (int pc = 0; pc < PP; ++pc) {
        const u32x4 w = {pw[kk][pc][0], pw[kk][pc][1], pw[kk][pc][2], pw[kk][pc][3]};
        pb[pc] = __builtin_bit_cast(bf16x8, w);
      }
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        bf16x8 va[NV];
#pragma unroll
        for (int pc = 0; pc < NV; ++pc) va[pc] = tr_operand(Vt, vo, kk, pc * D / 8 + 4 * db);
#pragma unroll
        for (int o = ORD - 1; o >= 0; --o)
#pragma unroll
          for (int pc = NV - 1; pc >= 0; --pc)
            if (o - pc >= 0 && o - pc < PP)
              acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[pc], pb[o - pc], acc[db], 0, 0, 0);
      }
    }
  };

  if (ntiles > 0) {
    load_tile(tile_at(0));
    write_tile(0, tile_at(0));
  }
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int jt = tile_at(t), stage = NS == 2 ? t & 1 : 0;
    const bool more = t + 1 < ntiles;
    if (more) load_tile(tile_at(t + 1));  // in flight during this tile
    compute(stage, jt);
    if constexpr (NS == 1) __syncthreads();
    if (more) write_tile(NS == 2 ? stage ^ 1 : 0, tile_at(t + 1));
    __syncthreads();
  }
  l_run = pair_sum(l_run);

  // ---- merge the key groups (through LDS, the stages are free) ------------
  if constexpr (KG == 2) {
    float* M = (float*)smem + rg * 64 * (16 * NDB + 2) + lane;
    if (kg == 1) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) M[(db * 16 + r) * 64] = acc[db][r];
      M[16 * NDB * 64] = m_run;
      M[(16 * NDB + 1) * 64] = l_run;
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = M[16 * NDB * 64], l1 = M[(16 * NDB + 1) * 64];
    const float m = fmaxf(m_run, m1), mu = m == -INFINITY ? 0.f : m;
    const float a0 = __builtin_amdgcn_exp2f(m_run - mu), a1 = __builtin_amdgcn_exp2f(m1 - mu);
    m_run = m;
    l_run = l_run * a0 + l1 * a1;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[db][r] = acc[db][r] * a0 + M[(db * 16 + r) * 64] * a1;
  }

  if (!row_ok) return;
  const float inv = 1.f / l_run;
  const int64_t orow = ((int64_t)b * p.Hq + hq) * n + my_i;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int dim = db * 32 + 8 * g + 4 * hh;
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = acc[db][4 * g + e] * inv;
      if (p.vec) {
        if (dim >= d) continue;
        if (p.obf16) {
          uint2 w;
          w.x = f32_to_bf16_rne(x[0]) | (f32_to_bf16_rne(x[1]) << 16);
          w.y = f32_to_bf16_rne(x[2]) | (f32_to_bf16_rne(x[3]) << 16);
          *(uint2*)((uint16_t*)p.o + orow * d + dim) = w;
        } else {
          *(float4*)((float*)p.o + orow * d + dim) = make_float4(x[0], x[1], x[2], x[3]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (dim + e < d) {
            if (p.obf16) ((uint16_t*)p.o)[orow * d + dim + e] = (uint16_t)f32_to_bf16_rne(x[e]);
            else ((float*)p.o)[orow * d + dim + e] = x[e];
          }
      }
    }
  if (p.lse && hh == 0) p.lse[orow] = (m_run + __log2f(l_run)) * kLn2;
}

template <class Ge>
hipError_t launch_gen(GenParams p, int B, hipStream_t stream) {
  if (Ge::LDS > 65536) {
    // once per device and instantiation (a bit per device; past the 64th on each call)
    static std::atomic<uint64_t> configured{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    const uint64_t bit = dev < 64 ? 1ull << dev : 0;
    if (e == hipSuccess && !(configured.load(std::memory_order_relaxed) & bit)) {
      e = hipFuncSetAttribute((const void*)sfa_fwd_generic_kernel<Ge>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, Ge::LDS);
      if (e == hipSuccess) configured.fetch_or(bit, std::memory_order_relaxed);
    }
    if (e != hipSuccess) return e;
  }
  p.BR = Ge::R / p.gs;
  p.nqb = (p.n + p.BR - 1) / p.BR;
  hipLaunchKernelGGL((sfa_fwd_generic_kernel<Ge>), dim3(p.nqb, B * p.Hq / p.gs), dim3(Ge::NT),
                     Ge::LDS, stream, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_gen_d(const GenParams& p, int B, int vbf16, hipStream_t stream) {
  constexpr int NW = D <= 128 ? 8 : 4, KG = D <= 128 ? 2 : 1;
  if (!vbf16) return launch_gen<GGeo<D, NW, KG, 3, 0>>(p, B, stream);
  auto go = [&](auto kx) { return launch_gen<GGeo<D, NW, KG, 1, decltype(kx)::value>>(p, B, stream); };
  if (p.vfmt == kValBF16) return go(std::integral_constant<int, kValBF16>{});
  if (p.vfmt == kValF16) return go(std::integral_constant<int, kValF16>{});
  return go(std::integral_constant<int, 0>{});
}

}  // namespace

bool fwd_generic_supported(int d, int k) { return d >= 1 && d <= kGDmax && k >= 1 && k <= d; }

hipError_t launch_attn_fwd_generic(const void* q_idx, const void* q_val, const void* k_idx,
                                   const void* k_val, const void* v, int B, int Hq, int Hkv,
                                   int n, int d, int k, int causal, int window, int n_global,
                                   float scale, int ifmt, int vfmt, int vbf16, int obf16, void* o,
                                   float* lse, hipStream_t stream) {
  GenParams p;
  p.q_idx = q_idx; p.q_val = q_val; p.k_idx = k_idx; p.k_val = k_val; p.v = v;
  p.o = o; p.lse = lse;
  p.Hq = Hq; p.Hkv = Hkv; p.n = n; p.d = d; p.k = k;
  p.causal = causal; p.window = window; p.n_global = n_global;
  const float scale_log2 = (float)((double)scale * 1.4426950408889634);
  p.q_mul = scale_log2;
  p.s_mul = 1.f;
  if (vbf16 && vfmt != kValF32) {
    // raw 16-bit operands: the scores take |scale_log2|.  Its power of two goes to bf16
    // queries (exact; a product then overflows where that of scaled queries would), its
    // sign to either kind, and a zero scale as zero queries
    int e = 0;
    if (vfmt == kValBF16 && scale_log2 != 0.f) e = std::min(std::max(ilogbf(scale_log2), -126), 127);
    p.q_mul = scale_log2 == 0.f ? 0.f : copysignf(ldexpf(1.f, e), scale_log2);
    p.s_mul = scale_log2 == 0.f ? 1.f : ldexpf(fabsf(scale_log2), -e);
  }
  p.ifmt = ifmt; p.vfmt = vfmt; p.obf16 = obf16;
  p.G = Hq / Hkv;
  p.gs = p.G % 4 == 0 ? 4 : p.G % 2 == 0 ? 2 : 1;
  p.BR = p.nqb = 0;  // set by launch_gen
  p.inv_k = 1.0f / (float)k;
  p.vec = d % 8 == 0 && ((uintptr_t)v | (uintptr_t)o) % 16 == 0;
  // head dimensions padded to the next kernel's (zero coordinates and values)
  if (d <= 64) return launch_gen_d<64>(p, B, vbf16, stream);
  if (d <= 96) return launch_gen_d<96>(p, B, vbf16, stream);
  if (d <= 128) return launch_gen_d<128>(p, B, vbf16, stream);
  return launch_gen_d<256>(p, B, vbf16, stream);
}

}  // namespace sfa
