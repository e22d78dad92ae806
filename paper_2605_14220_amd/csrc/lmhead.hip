// Fused LM-head log-softmax kernels for gfx950 (CDNA4).
//
// The per-row quantity is the token log-probability of Section 2 of the paper
// (the terms of Eq. 1) plus the entropy of the same distribution. Every row is
// computed with one fixed sequence of floating-point operations that depends
// only on d and V, never on how many rows share a launch, on a row's position
// among them, or on the launch grid: the batch-invariance principle of
// Section 3.1 (fixed tiling and reduction order, no atomics).
//
// Kernel 1, lmhead_partials: (vocab tile of 256, row tile) output tiles.
//   z^T = W_tile . h_tile^T on MFMA (v_mfma_f32_16x16x32_bf16, fp32
//   accumulate, hidden dimension in ascending 32-element steps, one
//   accumulation chain per logit). W is the A operand and the hidden states
//   the B operand: a lane's 4 accumulator registers of a 16x16 block hold 4
//   consecutive vocabulary entries of ONE row. Of the two MFMA shapes with
//   the full bf16 rate, this one moves fewer accumulator bytes per flop and
//   sustains a higher clock under the card's power limit.
//   Operands are staged HBM -> LDS with direct global->LDS DMA loads
//   (buffer_load_dwordx4 into LDS), double buffered, XOR-swizzled against LDS
//   bank conflicts. The epilogue turns the 256 logits of each row into one
//   partial (m, s, u) = (max z, sum e^(z-m), sum e^(z-m) (z-m)) and captures
//   the sampled token's logit from the same register value. Logits never
//   reach HBM.
//
// Decode batches may run lmhead_half_partials instead: the same pass over
//   128-entry halves of the vocab tiles, writing each half's partial where
//   the whole-tile epilogue merges the two; the merge pairs them up again. Up
//   to 64 rows lmhead_half_stream forms the same partials, a wave per half.
//
// Kernel 2, lmhead_merge: one wavefront per row (four for launches of at most
//   512 rows) merges that row's partials with a fixed balanced binary tree
//   over the tile index, then logp = z_tok - (M + log S) and H = log S - U / S.
//
// Reduction structure inside one vocab tile, for one row (fixed): each of the
// two vocab waves holds 128 entries of the row, 32 per lane in 4 lanes; per
// wave, the max and then the sums against it go lane-local in (block, register)
// order, then over the lane groups (lane ^ 16, then lane ^ 32); the two waves'
// partials are then merged, lower vocabulary half first.


#include <atomic>

#include "tilepass.h"

namespace tim {
namespace {

struct MSU {
  float m, s, u;
};

// (m, s, u) of the union of two disjoint vocab sets; `a` is the lower-index set.
__device__ __forceinline__ MSU merge2(MSU a, MSU b) {
  if (b.m == kNegInf) return a;  // empty set: exact identity
  if (a.m == kNegInf) return b;
  const float M = fmaxf(a.m, b.m);
  const float da = a.m - M, db = b.m - M;
  const float ea = exp2_hw(da * kLog2e), eb = exp2_hw(db * kLog2e);
  MSU r;
  r.m = M;
  r.s = a.s * ea + b.s * eb;
  r.u = (a.u + da * a.s) * ea + (b.u + db * b.s) * eb;
  return r;
}

// z[i] for the i with 16 (i / 4) + i % 4 == tl (there is one: tl < 128,
// tl % 16 < 4), as a chain of compare-selects. Each compare takes its own
// opaque copy of tl, so none is hoisted ahead of the chain (which would hold
// all 32 conditions in scalar registers at once).
__device__ __forceinline__ float select_entry(const float (&z)[32], int tl) {
  float zf = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    int t = tl;
    asm volatile("" : "+v"(t));
    if ((i >> 2) * 16 + (i & 3) == t) zf = z[i];
  }
  return zf;
}

// One tile's per-row results from its accumulators. Each wave holds 128 of
// the tile's 256 vocabulary entries of its rows: for row block bj, lane l holds
// row (l % 16) and, in register r of W block bi, the entry
// wv * 128 + bi * 16 + 4 (l / 16) + r. With NV = 1 the workgroup covers one
// 128-entry half of a vocabulary tile (v0 its first entry, vt its index among
// the halves) and writes that half's partial as it is. Per row block the wave takes the logits
// z = acc * inv_tau (a multiply by exactly 1 is skipped, which changes
// nothing), masks entries past V to -inf (tail tile only), forms its half's
// partial (m, s, u) -- max first, then the sums against that max, lane-local
// in (bi, r) order, then over lane ^ 16 and lane ^ 32 -- and captures the
// sampled token's logit from the same register value. The two vocab halves
// are merged in a fixed order (lower half first) into the tile's Partial.
// `scratch` holds 7 * BT floats of LDS; with `tok_lds` the tile's tokens come
// from LDS.
template <int NTB, int WT, bool DUMP, int NV = 2>
__device__ __forceinline__ void tile_epilogue(const LmHeadArgs& a, int n_vt, int vt, int64_t v0, int64_t t0,
                                              f32x4 (&acc)[8][2 * NTB], float* scratch, const int* tok_lds, int wave,
                                              int lane) {
  constexpr int BT = Tile<NTB, WT, NV>::BT;
  constexpr int NJ = 2 * NTB;
  static_assert(NV == 2 || (NV == 1 && !DUMP), "half tiles form partials only");
  const int wv = NV == 2 ? (wave & 1) : 0, wt = NV == 2 ? (wave >> 1) : wave;
  const int V = a.V;
  const int64_t rows = a.rows;
  const int g = lane >> 4, c16 = lane & 15;
  const float inv_tau = a.inv_tau;
  const int64_t vlane = v0 + wv * 128 + 4 * g;  // + bi * 16 + r
  float* red_m = scratch;                // [2][BT]
  float* red_s = red_m + 2 * BT;         // [2][BT]
  float* red_u = red_s + 2 * BT;         // [2][BT]
  float* zt_l = red_u + 2 * BT;          // [BT]
  // Whether a tile is the tail depends only on (v0, V), so a tile takes the
  // same path in every launch shape; a half takes its vocabulary tile's path.
  const bool full = (NV == 2 ? v0 : v0 - v0 % kVocabTile) + kVocabTile <= V;

#pragma unroll
  for (int bj = 0; bj < NJ; ++bj) {
    const int t_loc = wt * NTB * 32 + bj * 16 + c16;
    const int64_t tg = t0 + t_loc;
    const bool row_ok = tg < rows;
    // A row block of padding only writes nothing, so it skips the exponentials (a wave-uniform branch). Few rows per
    // call gain most, as their tile's end is not hidden: 5 rows at d = 2048, V = 151936 127.9 -> 127.4 us a call, 643
    // rows at d = 4096 726 -> 722; calls of whole tiles the same.
    if (t0 + wt * NTB * 32 + bj * 16 >= rows) continue;
    float z[32];  // z[4 bi + r]: entry vlane + 16 bi + r
#pragma unroll
    for (int bi = 0; bi < 8; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) z[bi * 4 + r] = acc[bi][bj][r];
    if (inv_tau != 1.0f) {
#pragma unroll
      for (int i = 0; i < 32; ++i) z[i] = z[i] * inv_tau;
    }
    if (!full) {
      const int lim = (int)(V - vlane);  // entries past V: (i / 4) 16 + i % 4 >= lim (32-bit: V < 2^31)
#pragma unroll
      for (int i = 0; i < 32; ++i)
        if ((i >> 2) * 16 + (i & 3) >= lim) z[i] = kNegInf;
    }
    if constexpr (DUMP) {
      if (row_ok) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          const int64_t v = vlane + (i >> 2) * 16 + (i & 3);
          if (v < V) a.logits[tg * (int64_t)V + v] = z[i];
        }
      }
      continue;
    }
    // the half's max, then e^(z - m) and e^(z - m) (z - m) summed against it
    // (z - m is exact 0 at the max, which so adds exactly 1 and 0); masked
    // entries add exactly zero to both. Lane groups combine as
    // (g0 + g1) + (g2 + g3): each permlane swap leaves one operand pair in the
    // same order in all four lanes, so they agree bit for bit.
    float m = kNegInf;
#pragma unroll
    for (int i = 0; i < 32; ++i) m = fmaxf(m, z[i]);
    m = group_max(m);
    float sv = 0.f, uv = 0.f;
    if (full) {
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const float x = z[i] - m;
        const float e = exp2_hw(x * kLog2e);
        sv = sv + e;
        uv = __builtin_fmaf(e, x, uv);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        float x = z[i] - m;
        float e = exp2_hw(x * kLog2e);
        if (z[i] == kNegInf) { x = 0.f; e = 0.f; }
        sv = sv + e;
        uv = __builtin_fmaf(e, x, uv);
      }
    }
    sv = group_sum(sv);
    uv = group_sum(uv);
    if constexpr (NV == 2) {
      if (g == 0) {
        red_m[wv * BT + t_loc] = m;
        red_s[wv * BT + t_loc] = sv;
        red_u[wv * BT + t_loc] = uv;
      }
    }
    // Token gather: the lane holding the row's token has tl = token - vlane
    // in [0, 128) with tl % 16 < 4 (entry z[4 (tl / 16) + tl % 16]). Rare, so
    // the 32-way select runs under a divergent branch.
    const int tok = row_ok ? (tok_lds != nullptr ? tok_lds[t_loc] : a.tokens[tg]) : -1;
    const int tl = (tok >= 0) ? (int)((int64_t)tok - vlane) : -1000000;
    if constexpr (NV == 2) {
      if (tl >= 0 && tl < 128 && (tl & 15) < 4) zt_l[t_loc] = select_entry(z, tl);
    } else {
      float zf = 0.f;
      if (tl >= 0 && tl < 128 && (tl & 15) < 4) zf = select_entry(z, tl);
      // the half's Partial, with the token's logit from the lane holding it
      // (lane group ((token - v0) % 16) / 4 of the row's four)
      const int64_t th = (int64_t)tok - v0;
      const bool mine = tok >= 0 && th >= 0 && th < 128;
      const float zt = __shfl(zf, c16 + (mine ? 16 * (int)((th & 15) >> 2) : 0));
      if (g == 0 && row_ok) {
        Partial p;
        p.m = m;
        p.s = sv;
        p.u = uv;
        p.ztok = mine ? zt : 0.f;
        a.part[tg * n_vt + vt] = p;
      }
    }
  }
  if constexpr (DUMP || NV == 1) return;
  __syncthreads();

  // the tile's Partial: lower vocab half merged with the upper one
  if (wv == 0 && g == 0) {
#pragma unroll
    for (int bj = 0; bj < NJ; ++bj) {
      const int t_loc = wt * NTB * 32 + bj * 16 + c16;
      const int64_t tg = t0 + t_loc;
      if (tg >= rows) continue;
      const MSU h = merge2(MSU{red_m[t_loc], red_s[t_loc], red_u[t_loc]},
                           MSU{red_m[BT + t_loc], red_s[BT + t_loc], red_u[BT + t_loc]});
      const int tok = tok_lds != nullptr ? tok_lds[t_loc] : a.tokens[tg];
      const int64_t tv = (int64_t)tok - v0;
      Partial p;
      p.m = h.m;
      p.s = h.s;
      p.u = h.u;
      p.ztok = (tv >= 0 && tv < kVocabTile) ? zt_l[t_loc] : 0.f;
      a.part[tg * n_vt + vt] = p;
    }
  }
}

// Epilogue policies of a tile pass. Each one names the pass's operands (and
// whether they are in the packed layout), how the stage loads are placed in a
// k-step, the LDS it needs beside the stage buffers, the per-row data it wants
// staged in LDS with each tile, how the accumulators start, and what it does
// with them.
//
// EpiPartials: the LM head forward. A = W [V, d], B = hidden states, K = d;
// the epilogue forms the tile's softmax partials (or, DUMP, writes logits);
// with NV = 1, those of half tiles.
template <bool DUMP, int NV = 2>
struct EpiPartials {
  using Args = LmHeadArgs;
  static constexpr bool kTokens = !DUMP;
  static constexpr bool kCoef = false;
  static constexpr bool kPacked = false;  // W and h as the caller holds them
  static constexpr int kLoadSpacing = 0;  // stage loads spread evenly over a k-step's MFMAs
  static constexpr int kGroupA = kGroupV;
  static constexpr int kNV = NV;
  template <int BT>
  static constexpr int scratch_bytes() { return NV == 2 ? 7 * BT * 4 : 0; }
  __device__ static TileOps ops(const Args& a) {
    return TileOps{a.w, a.hidden, a.tokens, nullptr, a.rows, a.V, a.d};
  }
  template <int NTB, int WT>
  __device__ static void init(const Args&, int64_t, int64_t, f32x4 (&acc)[8][2 * NTB], int, int) {
#pragma unroll
    for (int bi = 0; bi < 8; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2 * NTB; ++bj) acc[bi][bj] = f32x4{};
  }
  template <int NTB, int WT>
  __device__ static void epilogue(const Args& a, int n_vt, int vt, int64_t v0, int64_t t0, f32x4 (&acc)[8][2 * NTB],
                                  float* scratch, const int* tok_lds, const f32x4*, int wave, int lane) {
    tile_epilogue<NTB, WT, DUMP, NV>(a, n_vt, vt, v0, t0, acc, scratch, tok_lds, wave, lane);
  }
};

// Softmax partials (or, DUMP, logits) of every (vocab tile, row tile).
template <int NTB, int WT, bool SPLITK4, bool DUMP>
__global__ __launch_bounds__(128 * WT, (Shape<NTB, WT, SPLITK4>::PER_CU))
void lmhead_partials(LmHeadArgs a, int n_vt, int n_tt) {
  tile_pass<NTB, WT, SPLITK4, EpiPartials<DUMP>>(a, n_vt, n_tt);
}

// Softmax partials of every (half vocabulary tile, row tile), for decode
// batches: one vocab wave per workgroup along the vocabulary (WT waves along
// the rows), a third or half of the LDS of a CU each, so that several
// workgroups share a CU and the vocabulary's 2 * ceil(V / 256) halves fill the
// chip more evenly than its ceil(V / 256) tiles. A half's partial is the one
// the whole-tile epilogue forms for that half before merging the two.
// (PER_CU workgroups of WT waves put up to ceil(PER_CU * WT / 4) waves on
// one SIMD, which bounds each wave's registers.)
template <int NTB, int WT>
__global__ __launch_bounds__(64 * WT)
__attribute__((amdgpu_waves_per_eu((Shape<NTB, WT, false, 1>::PER_CU * WT + 3) / 4)))
void lmhead_half_partials(LmHeadArgs a, int n_ht, int n_tt) {
  tile_pass<NTB, WT, false, EpiPartials<false, 1>>(a, n_ht, n_tt);
}

// The same half-tile partials for batches of at most 16 NH rows, W streamed
// through wave-private rings: one wave per half tile, no barriers.
//
// A wave walks its half in groups of GB W blocks of 16 entries, each over all
// of K in stages of 64. A stage is cut into units of 16 rows x 128 bytes, 2 KB
// of LDS: first the NH row blocks, whose operands stay in registers for the
// stage, then the group's W blocks. The ring holds RU units; each consumed
// unit's slot takes the unit RU further on at once, so close to the whole ring
// is always in flight, and vmcnt (loads return in order) says when a unit has
// landed. An accumulator takes its k-steps in ascending order as everywhere.
//
// Bound by HBM where there are enough halves (stream_shape says where it is
// taken). What it gains over lmhead_half_partials: no stage barrier drains the
// loads, and with 24 KB a wave all of a 150k vocabulary's 1187 halves are
// resident at once (4.6 per CU) instead of 768 and a thin second round. Calls with the merge, before and after: 64 rows at d = 5120,
// V = 152064 319 -> 291 us (5.35 TB/s of W), at d = 2560 174 -> 154, at
// d = 4096 245 -> 239; 5 rows at d = 5120 288 -> 270. A bare stream of W
// through the same rings takes 256 us at d = 5120 and 222 at d = 4096.
template <int NH, int GB, int RU>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void lmhead_half_stream(LmHeadArgs a, int n_ht) {
  constexpr int NTB = (NH + 1) / 2, NJ = 2 * NTB, U = NH + GB, NG = 8 / GB, kUnit = 16 * kRowBytes;
  static_assert(RU > NH && 2 * RU < 64, "a stage's row blocks and a W block fit the ring; vmcnt counts it");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[RU * kUnit + 256];
  int* tok_lds = (int*)(lds + RU * kUnit);
  const int lane = threadIdx.x;
  const int64_t v0 = (int64_t)blockIdx.x * kHalfTile;
  const int w_rows = (a.V - v0) < kHalfTile ? (int)(a.V - v0) : kHalfTile;
  const rsrc_t wr = make_rsrc((const __bf16*)a.w + v0 * a.d, (uint64_t)w_rows * a.d * 2);
  const rsrc_t hr = make_rsrc(a.hidden, (uint64_t)a.rows * a.d * 2);
  const int nk = a.d / kKS;

  // this lane's 16 bytes of a unit's two 1 KB loads (rows 0-7 and 8-15), relative to the unit's first row
  const int r8 = lane >> 3;
  const uint32_t off0 = (uint32_t)(r8 * a.d + ((lane & 7) ^ swz(r8)) * 8) * 2u;
  const uint32_t off1 = (uint32_t)((r8 + 8) * a.d + ((lane & 7) ^ swz(r8 + 8)) * 8) * 2u;
  const uint32_t block = (uint32_t)a.d * 32u;  // bytes of 16 rows
  // Unit x of group g's stage s (s may run into the next group's) into the slot at `buf`. The unit's rows are in the
  // lane's offset, so rows past the operand's end lie outside its resource's range and load zeros. Past the last
  // group: its last stage again, never used.
  auto issue = [&](unsigned char* buf, int x, int g, int s) {
#if defined(__HIP_DEVICE_COMPILE__)
    const bool over = s >= nk;
    const int gg = over && g + 1 < NG ? g + 1 : g;
    const int ss = !over ? s : g + 1 < NG ? s - nk : nk - 1;
    const uint32_t o = (uint32_t)(x < NH ? x : gg * GB + x - NH) * block;
    const int soff = ss * kRowBytes;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(x < NH ? hr : wr, (lds_void*)buf, 16, off0 + o, soff, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(x < NH ? hr : wr, (lds_void*)(buf + 1024), 16, off1 + o, soff, 0, 0);
#endif
  };
  auto fence = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
#if defined(__HIP_DEVICE_COMPILE__)
  // the rows' tokens, landed before the first units (lanes past the batch read zeros, never used)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(a.tokens, (uint64_t)a.rows * 4), (lds_void*)tok_lds, 4,
                                           (uint32_t)lane * 4u, 0, 0, 0);
#endif
#pragma unroll
  for (int u = 0; u < RU; ++u) issue(lds + u * kUnit, u % U, 0, u / U);

  f32x4 acc[8][NJ];
#pragma unroll
  for (int bi = 0; bi < 8; ++bi)
#pragma unroll
    for (int bj = 0; bj < NJ; ++bj) acc[bi][bj] = f32x4{};
  bf16x8 fb[2][NH], fa[2][2];
  int slot = 0;  // the next unit's
  auto next = [](int p) { return p + kUnit == RU * kUnit ? 0 : p + kUnit; };
#pragma unroll
  for (int g = 0; g < NG; ++g) {
#pragma unroll 1
    for (int s = 0; s < nk; ++s) {
      // the stage's row blocks and its first W block
      fence();
      wait_vmem<2 * (RU - NH - 1)>();
      fence();
      const int first = slot;
#pragma unroll
      for (int bj = 0; bj < NH; ++bj, slot = next(slot))
#pragma unroll
        for (int k = 0; k < 2; ++k) fb[k][bj] = read_operand(lds + slot, lane & 15, k, lane);
#pragma unroll
      for (int k = 0; k < 2; ++k) fa[0][k] = read_operand(lds + slot, lane & 15, k, lane);
      slot = first;
#pragma unroll
      for (int bi = 0; bi < GB; ++bi) {
        fence();
        wait_lgkm0_vmem<63>();  // unit bi (and the row blocks) in registers, the slots free
        fence();
        if (bi == 0) {
#pragma unroll
          for (int bj = 0; bj < NH; ++bj, slot = next(slot)) issue(lds + slot, (bj + RU) % U, g, s + (bj + RU) / U);
        }
        issue(lds + slot, (NH + bi + RU) % U, g, s + (NH + bi + RU) / U);
        slot = next(slot);
        if (bi + 1 < GB) {
          fence();
          wait_vmem<2 * (RU - 1)>();  // unit bi + 1 landed
          fence();
#pragma unroll
          for (int k = 0; k < 2; ++k) fa[(bi + 1) & 1][k] = read_operand(lds + slot, lane & 15, k, lane);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int bj = 0; bj < NH; ++bj)
            acc[g * GB + bi][bj] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[bi & 1][k], fb[k][bj], acc[g * GB + bi][bj], 0, 0, 0);
      }
    }
  }
  wait_vmem<0>();  // no global->LDS request may outlive the workgroup
  fence();
  tile_epilogue<NTB, 1, false, 1>(a, n_ht, blockIdx.x, v0, 0, acc, nullptr, tok_lds, 0, lane);
}

// ---------------------------------------------------------------- merge

// TW: vocabulary entries per partial (whole or half tiles)
template <int TW>
__device__ __forceinline__ void finish_row(MSU v, const Partial* p, int tok, int V, int64_t row,
                                           float* logp, float* ent, float* lse) {
  const float logS = logf(v.s);
  const float L = v.m + logS;
  const bool ok = tok >= 0 && tok < V;
  logp[row] = ok ? p[tok / TW].ztok - L : __builtin_nanf("");
  if (ent) ent[row] = logS - v.u / v.s;
  if (lse) lse[row] = L;
}

// The balanced pairwise tree over 64 L consecutive leaves of a row, from
// leaf `first`: lane l owns leaves [first + l L, first + l L + L), merged in a
// tree within the lane, then across lanes by index (lane ^ 1, ^ 2, ... ^ 32),
// lower index first at every node. Leaves at or past n_vt are the identity, so
// the tree is the same whatever L is. With HALVES the row holds the partials of
// half tiles, and leaf jt is merge2(half 2 jt, half 2 jt + 1), as the
// whole-tile epilogue forms tile jt's partial (a missing upper half is the
// identity there too). Every lane returns the subtree's value.
template <int L, bool HALVES>
__device__ __forceinline__ MSU wave_subtree(const Partial* p, int n_vt, int n_ht, int first, int lane) {
  MSU leaf[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int jt = first + lane * L + i;
    if (jt < n_vt) {
      if constexpr (HALVES) {
        const Partial q0 = p[2 * jt];
        leaf[i] = MSU{q0.m, q0.s, q0.u};
        if (2 * jt + 1 < n_ht) {
          const Partial q1 = p[2 * jt + 1];
          leaf[i] = merge2(leaf[i], MSU{q1.m, q1.s, q1.u});
        }
      } else {
        const Partial q = p[jt];
        leaf[i] = MSU{q.m, q.s, q.u};
      }
    } else {
      leaf[i] = MSU{kNegInf, 0.f, 0.f};
    }
  }
#pragma unroll
  for (int wdt = 1; wdt < L; wdt *= 2)
#pragma unroll
    for (int i = 0; i < L; i += 2 * wdt) leaf[i] = merge2(leaf[i], leaf[i + wdt]);
  MSU v = leaf[0];
#pragma unroll
  for (int off = 1; off < 64; off *= 2) {
    MSU o;
    o.m = __shfl_xor(v.m, off);
    o.s = __shfl_xor(v.s, off);
    o.u = __shfl_xor(v.u, off);
    v = (lane & off) ? merge2(o, v) : merge2(v, o);
  }
  return v;
}

// One wavefront per row: the balanced pairwise tree over the tile index.
template <int L, bool HALVES = false>
__global__ __launch_bounds__(256) void lmhead_merge_tree(const Partial* __restrict__ part,
                                                         const int32_t* __restrict__ tokens,
                                                         int64_t rows, int n_vt, int V, float* logp,
                                                         float* ent, float* lse) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int n_ht = (V + kHalfTile - 1) / kHalfTile;
  const Partial* p = part + row * (HALVES ? n_ht : n_vt);
  const MSU v = wave_subtree<L, HALVES>(p, n_vt, n_ht, 0, lane);
  if (lane == 0) finish_row<HALVES ? kHalfTile : kVocabTile>(v, p, tokens[row], V, row, logp, ent, lse);
}

// Few rows (decode batches): four wavefronts per row, wave w reducing the
// quarter [w 64 LQ, (w + 1) 64 LQ) of the leaves as above, the quarters then
// merged as (q0 + q1) + (q2 + q3): the top two levels of the same balanced
// tree over 256 LQ leaves, so the same bits as lmhead_merge_tree<4 LQ> with a
// quarter of the serial work per lane.
template <int LQ, bool HALVES>
__global__ __launch_bounds__(256) void lmhead_merge_quad(const Partial* __restrict__ part,
                                                         const int32_t* __restrict__ tokens,
                                                         int64_t rows, int n_vt, int V, float* logp,
                                                         float* ent, float* lse) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = blockIdx.x;
  const int n_ht = (V + kHalfTile - 1) / kHalfTile;
  const Partial* p = part + row * (HALVES ? n_ht : n_vt);
  const MSU v = wave_subtree<LQ, HALVES>(p, n_vt, n_ht, wave * 64 * LQ, lane);
  __shared__ MSU q[4];
  if (lane == 0) q[wave] = v;
  __syncthreads();
  if (threadIdx.x == 0)
    finish_row<HALVES ? kHalfTile : kVocabTile>(merge2(merge2(q[0], q[1]), merge2(q[2], q[3])), p, tokens[row], V,
                                                row, logp, ent, lse);
}

// merge2 without branches, the same value: a row's maxima and exponentials do
// not depend on its sums, so a run of merges computes them ahead of the sums'
// chain (2048 rows of 594 partials: 79 us with branches, 50-56 without).
__device__ __forceinline__ MSU merge2_flat(MSU a, MSU b) {
  const float M = fmaxf(a.m, b.m);
  const float da = a.m - M, db = b.m - M;
  const float ea = exp2_hw(da * kLog2e), eb = exp2_hw(db * kLog2e);
  const float s = a.s * ea + b.s * eb;
  const float u = (a.u + da * a.s) * ea + (b.u + db * b.s) * eb;
  const bool no_a = a.m == kNegInf, no_b = b.m == kNegInf;
  return MSU{no_b ? a.m : no_a ? b.m : M, no_b ? a.s : no_a ? b.s : s, no_b ? a.u : no_a ? b.u : u};
}

// SPLITK4 engine: partials folded left to right, kFoldRows rows per workgroup.
// The fold is a serial chain of n_vt merges per row, so it is bound by that
// chain's latency once the partials are at hand: the workgroup brings them in
// chunks of kFoldTiles per row into LDS with coalesced loads, the next chunk's
// loads in flight while the first kFoldRows lanes fold the current one. With a
// thread per row loading its own partials, 2048 rows of 594 took 302 us (4
// partials a row 0.4 us less than this).
constexpr int kFoldRows = 16;
constexpr int kFoldTiles = 64;
__global__ __launch_bounds__(256) void lmhead_merge_fold(const Partial* __restrict__ part,
                                                         const int32_t* __restrict__ tokens,
                                                         int64_t rows, int n_vt, int V, float* logp,
                                                         float* ent, float* lse) {
  constexpr int kLoads = kFoldRows * kFoldTiles / 256;
  // one partial of padding per row: the folding lanes' rows fall on different banks
  __shared__ float4 buf[kFoldRows][kFoldTiles + 1];
  const int64_t row0 = (int64_t)blockIdx.x * kFoldRows;
  const int tid = threadIdx.x;
  float4 next[kLoads];
  auto fetch = [&](int first) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r = (tid + 256 * i) / kFoldTiles, jt = first + (tid + 256 * i) % kFoldTiles;
      next[i] = float4{};  // past the row's tiles: not folded
      if (row0 + r < rows && jt < n_vt) next[i] = ((const float4*)part)[(row0 + r) * n_vt + jt];
    }
  };
  MSU v = MSU{kNegInf, 0.f, 0.f};
  fetch(0);
  for (int first = 0; first < n_vt; first += kFoldTiles) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) buf[(tid + 256 * i) / kFoldTiles][(tid + 256 * i) % kFoldTiles] = next[i];
    __syncthreads();
    if (first + kFoldTiles < n_vt) fetch(first + kFoldTiles);
    if (tid < kFoldRows) {
      auto leaf = [&](int i) { const float4 q = buf[tid][i]; return MSU{q.x, q.y, q.z}; };
      v = first == 0 ? leaf(0) : merge2_flat(v, leaf(0));
      const int n = n_vt - first < kFoldTiles ? n_vt - first : kFoldTiles;
#pragma unroll 8
      for (int i = 1; i < n; ++i) v = merge2_flat(v, leaf(i));
    }
    __syncthreads();
  }
  const int64_t row = row0 + tid;
  if (tid < kFoldRows && row < rows) finish_row<kVocabTile>(v, part + row * n_vt, tokens[row], V, row, logp, ent, lse);
}

}  // namespace

// Compute units of the current device (cached per device).
int device_cu_count() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
  // atomic: host threads may launch on one device at once (a racing first
  // call only queries the same attribute twice)
  static std::atomic<int> cache[64];
  if (dev < 64) {
    const int c = cache[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (dev < 64) cache[dev].store(n, std::memory_order_relaxed);
  return n;
}

int n_vocab_tiles(int V) { return (V + kVocabTile - 1) / kVocabTile; }
int n_half_tiles(int V) { return (V + kHalfTile - 1) / kHalfTile; }

template <int NTB, int WT, bool SPLITK4, bool DUMP>
static hipError_t launch_partials_t(const LmHeadArgs& a, bool persistent, hipStream_t s) {
  const int n_vt = n_vocab_tiles(a.V);
  constexpr int BT = Tile<NTB, WT>::BT;
  const int64_t n_tt = (a.rows + BT - 1) / BT;
  const int64_t nblk = n_tt * n_vt;
  if (nblk > 0x7fffffff) return hipErrorInvalidValue;
  int64_t grid = nblk;
  if (persistent) {
    const int64_t resident = (int64_t)device_cu_count() * Shape<NTB, WT, SPLITK4>::PER_CU;
    if (resident > 0 && resident < grid) grid = resident;
  }
  hipLaunchKernelGGL((lmhead_partials<NTB, WT, SPLITK4, DUMP>), dim3((unsigned)grid), dim3(128 * WT), 0,
                     s, a, n_vt, (int)n_tt);
  return hipGetLastError();
}

// The smallest row tile, up to `rows_per_wg`, whose tiles all fit the chip at
// once (one per CU): such a call is bound by the time of a single tile, so the
// larger row tile only pays where it saves a round. With a second round the
// larger one wins (V = 151936, 200 rows: 334 us on 256-row tiles, 433 on
// 128-row ones), without one the smaller (V = 32000: 45 against 38 us).
static int fit_row_tile(int64_t rows, int V, int rows_per_wg) {
  const int64_t n_vt = n_vocab_tiles(V), cus = device_cu_count();
  for (int rt = 64; rt < rows_per_wg; rt *= 2)
    if ((rows + rt - 1) / rt * n_vt <= cus) return rt;
  return rows_per_wg;
}

hipError_t launch_partials(const LmHeadArgs& a, int rows_per_wg, bool splitk4, hipStream_t s) {
  const bool dump = a.logits != nullptr;
  const int rt = fit_row_tile(a.rows, a.V, rows_per_wg);
  if (splitk4) {
    // A second accumulator set, so waves of 128 x 32 (64 + 64 accumulators per lane). Eight of them on a 128-row
    // tile put two on each SIMD; it is bound by the LDS operand reads, 10 KB per 16 MFMAs of a wave. Per 2048 rows
    // at d = 4096, V = 151936: 2.55 ms (1.0 PFLOP/s); four waves on a 64-row tile, one per SIMD, 4.13 ms; four of
    // 128 x 64 on a 128-row tile 3.65 ms. The 64-row tile stays for calls of at most 64 rows and where its tiles
    // all fit the chip at once.
    if (dump) return launch_partials_t<1, 2, true, true>(a, false, s);
    return rt == 64 ? launch_partials_t<1, 2, true, false>(a, false, s) : launch_partials_t<1, 4, true, false>(a, true, s);
  }
  switch (rt) {
    case 64: return dump ? launch_partials_t<1, 2, false, true>(a, false, s) : launch_partials_t<1, 2, false, false>(a, false, s);
    case 128:  // 8 waves of 128 x 32, two per SIMD (four of 128 x 64 were 2-18% slower at 66..128 rows)
      return dump ? launch_partials_t<1, 4, false, true>(a, true, s) : launch_partials_t<1, 4, false, false>(a, true, s);
    default:  // 256-row tiles, 8 waves; full-size launches persistent
      return dump ? launch_partials_t<2, 4, false, true>(a, true, s) : launch_partials_t<2, 4, false, false>(a, true, s);
  }
}

// Share of the slots of the last round that hold a unit, for `units` units
// dealt to `slots` resident workgroups.
static double round_fill(int64_t units, int64_t slots) {
  const int64_t rounds = (units + slots - 1) / slots;
  return (double)units / (double)(rounds * slots);
}

bool prefer_half_tiles(int V, int64_t rows) {
  // 65..128 rows: whole tiles of this row tile run one workgroup per CU,
  // halves two (four waves each), which measured faster at every vocabulary
  // size tried
  if (rows > 64) return true;
  const int cus = device_cu_count();
  if (cus <= 0) return false;
  const int64_t whole_slots = (int64_t)cus * Shape<1, 2, false>::PER_CU;
  const int64_t half_slots = (int64_t)cus * Shape<1, 2, false, 1>::PER_CU;
  return round_fill(n_half_tiles(V), half_slots) > round_fill(n_vocab_tiles(V), whole_slots);
}

template <int NTB, int WT>
static hipError_t launch_halves_t(const LmHeadArgs& a, hipStream_t s) {
  const int n_ht = n_half_tiles(a.V);
  constexpr int BT = Tile<NTB, WT, 1>::BT;
  const int64_t n_tt = (a.rows + BT - 1) / BT;
  const int64_t nblk = n_tt * n_ht;
  if (nblk > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((lmhead_half_partials<NTB, WT>), dim3((unsigned)nblk), dim3(64 * WT), 0, s, a, n_ht, (int)n_tt);
  return hipGetLastError();
}

template <int NH, int GB, int RU>
static hipError_t launch_stream_t(const LmHeadArgs& a, hipStream_t s) {
  const int n_ht = n_half_tiles(a.V);
  hipLaunchKernelGGL((lmhead_half_stream<NH, GB, RU>), dim3((unsigned)n_ht), dim3(64), 0, s, a, n_ht);
  return hipGetLastError();
}

// Up to 64 rows: a wave per half with a ring of its own where that is the
// faster shape (stream_shape), else 64-row tiles (three workgroups of 2 waves
// of 128 x 32 per CU). 65..128 rows: 128-row tiles (two workgroups of 4 waves
// of 128 x 32 per CU: two waves per SIMD).
hipError_t launch_partials_halves(const LmHeadArgs& a, hipStream_t s) {
  const StreamShape st = stream_shape(a.rows, a.d, n_half_tiles(a.V), device_cu_count());
  switch (st.row_blocks) {
    case 1:
      return st.group == 2   ? launch_stream_t<1, 2, 12>(a, s)
             : st.group == 4 ? launch_stream_t<1, 4, 12>(a, s)
                             : launch_stream_t<1, 8, 12>(a, s);
    case 2: return st.group == 4 ? launch_stream_t<2, 4, 8>(a, s) : launch_stream_t<2, 8, 12>(a, s);
    case 4: return launch_stream_t<4, 8, 12>(a, s);
  }
  return a.rows <= 64 ? launch_halves_t<1, 2>(a, s) : launch_halves_t<1, 4>(a, s);
}

// Launches of at most this many rows merge with four waves per row.
constexpr int64_t kQuadMergeRows = 512;

template <bool HALVES>
static hipError_t launch_merge_rows(const Partial* part, const int32_t* tokens, int64_t rows, int V, float* logp,
                                    float* entropy, float* lse, hipStream_t s) {
  const int n_vt = n_vocab_tiles(V);
  const dim3 b(256);
  if (rows <= kQuadMergeRows && n_vt > 128) {
    const dim3 g((unsigned)rows);
    if (n_vt <= 256) hipLaunchKernelGGL((lmhead_merge_quad<1, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
    else if (n_vt <= 512) hipLaunchKernelGGL((lmhead_merge_quad<2, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
    else if (n_vt <= 1024) hipLaunchKernelGGL((lmhead_merge_quad<4, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
    else if (n_vt <= kMaxTiles) hipLaunchKernelGGL((lmhead_merge_quad<8, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  const dim3 g((unsigned)((rows + 3) / 4));
  if (n_vt <= 64) hipLaunchKernelGGL((lmhead_merge_tree<1, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
  else if (n_vt <= 128) hipLaunchKernelGGL((lmhead_merge_tree<2, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
  else if (n_vt <= 256) hipLaunchKernelGGL((lmhead_merge_tree<4, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
  else if (n_vt <= 512) hipLaunchKernelGGL((lmhead_merge_tree<8, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
  else if (n_vt <= 1024) hipLaunchKernelGGL((lmhead_merge_tree<16, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
  else if (n_vt <= kMaxTiles) hipLaunchKernelGGL((lmhead_merge_tree<32, HALVES>), g, b, 0, s, part, tokens, rows, n_vt, V, logp, entropy, lse);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// A grid holds fewer than 2^32 threads (a launch of more succeeds with the
// count wrapped), and the merges take 64 or 16 threads a row: 2^25 rows per launch.
constexpr int64_t kMergeRows = (int64_t)1 << 25;
template <class F>
static hipError_t merge_chunks(int64_t rows, F launch) {
  for (int64_t r = 0; r < rows; r += kMergeRows) {
    const hipError_t e = launch(r, rows - r < kMergeRows ? rows - r : kMergeRows);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool HALVES>
static hipError_t launch_merge_tree(const Partial* part, const int32_t* tokens, int64_t rows, int V, float* logp,
                                    float* entropy, float* lse, hipStream_t s) {
  const int per_row = HALVES ? n_half_tiles(V) : n_vocab_tiles(V);
  return merge_chunks(rows, [&](int64_t r, int64_t n) {
    return launch_merge_rows<HALVES>(part + r * per_row, tokens + r, n, V, logp + r, entropy ? entropy + r : nullptr,
                                     lse ? lse + r : nullptr, s);
  });
}

hipError_t launch_merge(const Partial* part, const int32_t* tokens, int64_t rows, int V,
                        bool left_fold, float* logp, float* entropy, float* lse, hipStream_t s) {
  if (left_fold) {
    const int n_vt = n_vocab_tiles(V);
    return merge_chunks(rows, [&](int64_t r, int64_t n) {
      hipLaunchKernelGGL(lmhead_merge_fold, dim3((unsigned)((n + kFoldRows - 1) / kFoldRows)), dim3(256), 0, s,
                         part + r * n_vt, tokens + r, n, n_vt, V, logp + r, entropy ? entropy + r : nullptr,
                         lse ? lse + r : nullptr);
      return hipGetLastError();
    });
  }
  return launch_merge_tree<false>(part, tokens, rows, V, logp, entropy, lse, s);
}

hipError_t launch_merge_halves(const Partial* part, const int32_t* tokens, int64_t rows, int V, float* logp,
                               float* entropy, float* lse, hipStream_t s) {
  return launch_merge_tree<true>(part, tokens, rows, V, logp, entropy, lse, s);
}

}  // namespace tim
