// SFA decode step (App. B, KV-cache attention) on gfx950: launchers of the
// decode kernel (sfa_decode_kernel.h) for bf16 / float32 V caches, and the
// merge of the context chunks' partials by their LSE.
#include <algorithm>

#include "../../include/sfa.h"
#include "sfa_decode_kernel.h"

namespace sfa {

// Merge the chunk partials of each (b, h): O = sum_c w_c o_c / sum_c w_c l_c,
// w_c = 2^(m_c - M), LSE = (M + log2 sum_c w_c l_c) ln 2.  A few KB of
// dependent loads per row: each wave takes the maximum and the sum with
// lanes over the chunks.  The output sum (thread = dimension) is kMergeThreads / D
// sums, each over the chunks of one residue, added in order: by as many groups of
// threads (T = kMergeThreads; launch_decode_combine), or in turn by one (T = D).  Which
// of the two runs follows the cache's capacity; the order of the sums, and so the
// bits, do not.
constexpr int kMergeThreads = 512;
template <int D, int T>
__global__ __launch_bounds__(T) void sfa_decode_combine_kernel(
    const float* __restrict__ ws_m, const float* __restrict__ ws_l, const float* __restrict__ ws_o,
    const int32_t* seq_len, int Hq, int Lmax, int nch, int window, int n_global, int aim, void* o,
    int obf16, float* lse) {
  constexpr int NG = kMergeThreads / D;
  static_assert(T == D || T == kMergeThreads, "one group of threads, or one per sum");
  __shared__ float part[T == D ? 1 : NG][D];
  const int bh = blockIdx.x;
  const int b = bh / Hq;
  const int dd = threadIdx.x % D, grp = threadIdx.x / D, lane = threadIdx.x & 63;
  const int L = seq_len_of(seq_len, b, Lmax);
  const int nc = decode_plan(L, window, n_global, aim).count;
  const int64_t s0 = (int64_t)bh * nch;
  float M = -INFINITY;
  for (int c = lane; c < nc; c += 64) M = fmaxf(M, ws_m[s0 + c]);
  M = wave_max_dpp(M);
  const float Mu = (M == -INFINITY) ? 0.f : M;
  float lsum = 0.f;
  for (int c = lane; c < nc; c += 64) lsum = fmaf(exp2f(ws_m[s0 + c] - Mu), ws_l[s0 + c], lsum);
  lsum = wave_sum(lsum);
  float osum = 0.f;
  if constexpr (T == D) {
    float os[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) os[g] = 0.f;
    for (int c0 = 0; c0 < nc; c0 += NG) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {  // (past the last chunk: read, not added)
        const int c = min(c0 + g, nc - 1);
        const float x = ws_o[(s0 + c) * D + dd], w = exp2f(ws_m[s0 + c] - Mu);
        os[g] = c0 + g < nc ? fmaf(w, x, os[g]) : os[g];
      }
    }
    osum = os[0];
#pragma unroll
    for (int g = 1; g < NG; ++g) osum += os[g];
  } else {
#pragma unroll 4
    for (int c = grp; c < nc; c += NG) osum = fmaf(exp2f(ws_m[s0 + c] - Mu), ws_o[(s0 + c) * D + dd], osum);
    part[grp][dd] = osum;
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int g = 1; g < NG; ++g) osum += part[g][dd];
  }
  const float out = lsum > 0.f ? osum / lsum : 0.f;
  if (obf16) ((uint16_t*)o)[(int64_t)bh * D + dd] = (uint16_t)f32_to_bf16_rne(out);
  else ((float*)o)[(int64_t)bh * D + dd] = out;
  if (lse && dd == 0) lse[bh] = lsum > 0.f ? (M + __log2f(lsum)) * kLn2 : -INFINITY;
}

static size_t slot_bytes(int B, int Hq, size_t slots, int d) {
  return (size_t)B * Hq * slots * (size_t)(d + 2) * sizeof(float);
}

size_t decode_workspace_bytes_min(int B, int Hq, int Lmax, int d) {
  return slot_bytes(B, Hq, (size_t)((Lmax + kDecodeChunk - 1) / kDecodeChunk), d);
}

// The most partial slots of a step over Lmax keys with that aim, windowed or not: a
// sequence has at most aim + 2 chunks below kDecodeChunk keys (decode_plan; under a
// window the global keys' last chunk and the window's first are partly filled), or
// its whole chunks of kDecodeChunk.
static int most_slots(int Lmax, int aim) {
  const int fine = Lmax / kDecodeMinChunk + (Lmax % kDecodeMinChunk != 0);
  return aim == 0 ? decode_slots(Lmax, 0) : std::min(fine, std::max(decode_slots(Lmax, 0), aim + 2));
}

// For any group (a group of kDecMaxG heads and a window have the largest aim),
// cache format and token window.  A finer cut never needs more than the
// allocation-free decode's scratch has: B * Hq * (aim + 2) <= 24 * kDecodeTargetWindow.  So
// that entry point cuts as the others do, and whether a cut is made does not
// depend on the capacity.
size_t decode_workspace_bytes(int B, int Hq, int Lmax, int d) {
  static_assert(kDecodeTarget <= kDecodeTargetWindow && kDecodeTargetQ8 <= kDecodeTargetWindow, "largest aim");
  static_assert((size_t)3 * kDecMaxG * kDecodeTargetWindow * (128 + 2) * sizeof(float) <=
                    SFA_DECODE_NOALLOC_MAX_BYTES, "a finer cut fits the scratch");
  if (d != 64 && d != 128) return decode_workspace_bytes_min(B, Hq, Lmax, d);
  return slot_bytes(B, Hq, most_slots(Lmax, decode_chunks_aim(B, (Hq + kDecMaxG - 1) / kDecMaxG, true, 1)), d);
}

int decode_aim(int B, int Hq, int Hkv, int Lmax, int d, int window, size_t ws_bytes, bool q8) {
  return ws_bytes >= decode_workspace_bytes(B, Hq, Lmax, d) ? decode_chunks_aim(B, Hkv, q8, window) : 0;
}

template <int D, int G, bool VBF16, int KC8, bool C8>
static void launch_dec_t(const DecParams& p, int B, hipStream_t stream) {
  const dim3 grid(p.nch, B * p.Hkv), block(kDecThreads);
  if (p.table)
    hipLaunchKernelGGL((sfa_decode_kernel<D, G, VBF16, KC8, C8, true>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((sfa_decode_kernel<D, G, VBF16, KC8, C8, false>), grid, block, 0, stream, p);
}

template <int D, int G, bool VBF16>
static void launch_dec_kc(const DecParams& p, int B, hipStream_t stream) {
  if constexpr (VBF16) {
    if (p.kifmt == kIdxI16 && p.kvfmt == kValBF16) {
      if (p.k == 8) return launch_dec_t<D, G, VBF16, 1, false>(p, B, stream);
      if (p.k == 16) return launch_dec_t<D, G, VBF16, 2, false>(p, B, stream);
      if (p.k == 32) return launch_dec_t<D, G, VBF16, 4, false>(p, B, stream);
    }
    if (p.kifmt == kIdxU8 && p.kvfmt == kValF16) {
      if (p.k == 8) return launch_dec_t<D, G, VBF16, 1, true>(p, B, stream);
      if (p.k == 16) return launch_dec_t<D, G, VBF16, 2, true>(p, B, stream);
      if (p.k == 32) return launch_dec_t<D, G, VBF16, 4, true>(p, B, stream);
    }
  }
  launch_dec_t<D, G, VBF16, 0, false>(p, B, stream);
}

template <int D, bool VBF16>
static void launch_dec_g(const DecParams& p, int G, int B, hipStream_t stream) {
  if (G == 1) launch_dec_kc<D, 1, VBF16>(p, B, stream);
  else if (G == 2) launch_dec_kc<D, 2, VBF16>(p, B, stream);
  else if (G <= 4) launch_dec_kc<D, 4, VBF16>(p, B, stream);
  else launch_dec_kc<D, 8, VBF16>(p, B, stream);
}

int decode_max_group() { return kDecMaxG; }

DecParams make_dec_params(const DecodeArgs& a) {
  DecParams p;
  p.q_idx = a.q_idx; p.q_val = a.q_val; p.kc_idx = a.kc_idx; p.kc_val = a.kc_val; p.v = a.v;
  p.seq_len = a.seq_len;
  p.Hq = a.Hq; p.Hkv = a.Hkv; p.Lmax = a.Lmax; p.k = a.k;
  p.G = a.Hq / a.Hkv;
  p.aim = a.aim;
  p.window = a.window; p.n_global = a.n_global;
  const int64_t wspan = (int64_t)a.window + a.n_global;
  p.nch = decode_slots(a.Lmax, a.aim);
  if (a.window > 0 && wspan < a.Lmax) {
    // a sequence still inside the window, or whose query is a global token,
    // is cut as without one: its length is at most wspan
    p.nch = std::min(decode_slots((int)wspan, a.aim) + 2, most_slots(a.Lmax, a.aim));
  }
  // The 8-bit cache's step is bound by its arithmetic, and slots that a sequence does
  // not have, dispatched among the others, leave compute units with fewer workgroups: by
  // slot they come last (24 x 8 heads of 16,384 keys, four of five slots in use: 134 ->
  // 118 us, 117 with four slots; 12 x 8 mixed lengths to 12,000 47.7 -> 41.5).  Not with few
  // heads, whose workgroups are all resident: there it puts the chunks of one sequence
  // on one compute unit (8 x 8 mixed lengths to 5000: 17.8 -> 20.7).  Over bf16 caches,
  // bound by memory, it was up to 2.5% slower.
  p.by_slot = a.kc_scale != nullptr && a.B * a.Hkv >= 96 && p.nch <= 65535;
  const size_t nslot = (size_t)a.B * a.Hq * p.nch;
  p.ws_m = (float*)a.ws;
  p.ws_l = p.ws_m + nslot;
  p.ws_o = p.ws_l + nslot;
  p.scale_log2 = (float)((double)a.scale * 1.4426950408889634);
  p.qifmt = a.qifmt; p.qvfmt = a.qvfmt; p.kifmt = a.kifmt; p.kvfmt = a.kvfmt;
  p.q_dense = a.q_dense;
  p.table = a.table;
  p.max_pages = a.max_pages; p.log2P = a.log2P; p.num_pages = a.num_pages;
  p.kc_scale = a.kc_scale;
  p.v_scale = a.v_scale;
  return p;
}

hipError_t launch_decode_combine(const DecParams& p, const DecodeArgs& a, hipStream_t stream) {
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(a.B * a.Hq), dim3(threads), 0, stream, p.ws_m, p.ws_l, p.ws_o,
                       a.seq_len, a.Hq, a.Lmax, p.nch, p.window, p.n_global, p.aim, a.o, a.obf16,
                       a.lse);
  };
  // Groups of threads where one's sum is a long serial chain (64,000 keys of one
  // sequence, 63 chunks: 38.0 -> 35.3 us a step; 4000 keys, 16: 14.0 -> 11.2), one group
  // where the rows fill the chip (2048 rows of 1 to 8 chunks: 4 us less).
  const bool many = p.nch > 16 || (p.nch > 4 && a.B * a.Hq <= 1024);
  if (a.d == 64) {
    if (many) go(sfa_decode_combine_kernel<64, kMergeThreads>, kMergeThreads);
    else go(sfa_decode_combine_kernel<64, 64>, 64);
  } else {
    if (many) go(sfa_decode_combine_kernel<128, kMergeThreads>, kMergeThreads);
    else go(sfa_decode_combine_kernel<128, 128>, 128);
  }
  return hipGetLastError();
}

hipError_t launch_attn_decode(const DecodeArgs& a, hipStream_t stream) {
  const DecParams p = make_dec_params(a);
  const int G = a.Hq / a.Hkv, B = a.B;
  if (a.d == 64) {
    if (a.vbf16) launch_dec_g<64, true>(p, G, B, stream); else launch_dec_g<64, false>(p, G, B, stream);
  } else {
    if (a.vbf16) launch_dec_g<128, true>(p, G, B, stream); else launch_dec_g<128, false>(p, G, B, stream);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_decode_combine(p, a, stream);
}

}  // namespace sfa
