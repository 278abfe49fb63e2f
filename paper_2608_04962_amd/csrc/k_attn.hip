// Tree-verify attention on gfx950.
//
// Paper: App. B.1 Eq. (nodep) -- the packed verification forward must give every tree node
// the result of an ordinary autoregressive forward at prefix ++ path(u). For one attention
// layer: node u's queries see the whole cached prefix and the tree tokens on u's root path.
//
// Unit = (trajectory b, KV head g, row group): the T*G (node, head-in-group) query rows sharing KV head g, in
// groups of at most 224 (bf16) or 256 (fp32) rows, so every K/V tile staged in LDS is reused by all of them (GQA
// sharing). A unit's keys are a row of 64-key tiles, the prefix's and then the tree's (under the ancestor
// mask). All units' tiles, laid end to end, are cut into ranges of one length, one per block: every CU streams
// the same number of tiles whatever the context lengths, and a unit is cut only where a range ends. The pieces
// of a cut unit are partial results that k_attn_combine merges by log-sum-exp. Short units that fill the blocks are
// left whole (attn_plan). Every block derives the cut, or its units, from ctx_len itself, so no kernel has to plan
// it first.
// Scores are computed transposed, S^T = K Q^T on 32x32 MFMA tiles: a lane then holds 16 keys of one query row, so
// the row max needs one cross-half exchange; P stays in registers and feeds O^T = V^T P^T.
//
// The kernels:
// * k_tree_attn_dma<D> (bf16): eight waves. A row group holds at most 224 rows, so at least one wave has no query
//   rows and issues all K/V transfers straight from HBM into a four-slot LDS ring; every other wave owns 32 query
//   rows and converts a share of each V tile from bf16 to fp16 in place. Scores use v_mfma_f32_32x32x16_bf16, the
//   probability-weighted V sum v_mfma_f32_32x32x16_f16 with P and V in fp16 (bf16 P would cost ~3e-3 relative
//   error at 4k-token contexts). fp16 holds a bf16 value exactly only for magnitudes in [2^-14, 65280] (or zero);
//   the converting waves track the range of every V value they convert, and a segment that meets any other value
//   is recomputed at the end of the block with V widened to fp32 and the weighted sum on fp32 MFMA (exact for
//   every finite bf16 V).
// * k_tree_attn<D> (fp32 inputs; its segment body, with bf16 K and fp32 V, is the recomputation above): K/V staged
//   through registers into a two-slot LDS ring with V transposed, eight waves of 32 rows.
#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace sr {

constexpr int ATT_KT = 64;             // keys per LDS tile
constexpr int ATT_NW = 8;              // waves per block
constexpr int ATT_RB = 1;              // 32-row query blocks per wave
constexpr int ATT_ROWS = ATT_NW * ATT_RB * 32;  // query rows per block
constexpr int ATT_BLOCKS = 256;        // ranges (blocks) of a call: one per CU
constexpr int ATT_SEG_TILES = 1024;    // most tiles of a range: its page ids are held in LDS
constexpr int ATT_TPP = ATT_KT / 16;   // pages per tile
constexpr int ATT_WHOLE = 4;           // units of at most so many tiles are never cut (of more by attn_plan's rule)
constexpr int ATT_MIN_TILES = 2;       // least tiles of a range (bf16)
constexpr int ATT_BS = 16;             // tokens per page
constexpr int ATT_PIECES = 64;         // pieces of a unit, where a few units share the blocks (more of long ones)
constexpr int ATT_PAIRS = 2 * ATT_BLOCKS;   // most whole units that are dealt to the blocks by length
constexpr int ATT_PAIR_TILES = 26;     // and their most tiles

// Arithmetic of the register-staged kernel. QKPL / PKPL: elements a lane supplies per MFMA slot for the
// scores and for the weighted V sum.
// fp32 inputs: fp32 MFMA for both products.
struct AttnF32 {
  typedef float T;
  static constexpr int QKPL = 1, PKPL = 1;
  typedef float qfrag;
  typedef float vt;                    // V^T element in LDS
  typedef float pfrag;
  static __device__ __forceinline__ f32x16 mma_qk(qfrag a, qfrag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x16 mma_pv(pfrag a, pfrag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};
// bf16 inputs for any V: bf16 MFMA for the scores (as the DMA kernel), V widened exactly to fp32 and the
// weighted sum on fp32 MFMA with P in fp32.
struct AttnBf16Wide {
  typedef bf16_t T;
  static constexpr int QKPL = 8, PKPL = 1;
  typedef u32x4 qfrag;                 // 8 x bf16
  typedef float vt;
  typedef float pfrag;
  static __device__ __forceinline__ f32x16 mma_qk(qfrag a, qfrag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
  }
  static __device__ __forceinline__ f32x16 mma_pv(pfrag a, pfrag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};

// key (within a 32-key subtile) held by register i of a lane in half h of a 32x32 output tile
__device__ __forceinline__ int tile_row(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// LDS swizzle of V^T rows: 4-key groups of row d live at group position g ^ vswz(d), which keeps both
// the transposing writes (rows 4 apart) and the MFMA operand reads (32 consecutive rows) free of bank
// conflicts.
__device__ __forceinline__ int vswz(int d) { return (d ^ (d >> 2)) & 15; }

template <class AT, int D>
struct AttnGeom {
  static constexpr int E = sizeof(typename AT::T);       // element bytes in the cache
  static constexpr int ROWB = D * E;                     // bytes of one K row
  static constexpr int NCH = ROWB / 16;                  // 16-byte chunks per K row
  static constexpr int KTILE = ATT_KT * ROWB;            // bytes of a K tile
  static constexpr int VE = sizeof(typename AT::vt);
  static constexpr int VROWB = ATT_KT * VE;              // bytes of one V^T row (64 keys)
  static constexpr int VTILE = D * VROWB;
  static constexpr int NT = ATT_NW * 64;
  static constexpr int KVEC = KTILE / 16;                // 16-byte K vectors per tile
  static constexpr int KVPT = KVEC / NT;                 // per thread
  static constexpr int VITEMS = (ATT_KT / 4) * (D / 4);  // 4 keys x 4 dims per item
  static constexpr int VIPT = (VITEMS + NT - 1) / NT;    // per thread (the last round may be partial)
  static_assert(KVEC % NT == 0 && VITEMS % 64 == 0, "tile staging must split evenly over the block");
};

// Arguments of the attention kernels. A call's ranges have `len` tiles each (attn_len); with `whole` no unit is cut,
// and a range is the units that start in it (1), one unit, where every unit has a block (2), or one or two of at most
// ATT_PAIRS units, the longest with the shortest (3).
template <typename T>
struct AttnArgs {
  const T *q, *k_cache, *v_cache;
  const int32_t *block_table, *ctx_len;
  const T *k_tree, *v_tree;
  const int32_t* parents;
  float *out, *lse, *part_o, *part_ml;
  long long* work;                     // [0] tiles per range, [1 + b] position of trajectory b's first tile
  int B, T_, Hq, Hkv, max_blocks, num_blocks;
  float scale_log2;
  int R, row_groups, group_rows, n_ranges, min_tiles, unit_cost, whole, by_unit;
};

// 64-key tiles of each unit of a trajectory (one for an invalid ctx_len: its unit then writes NaN rows)
__device__ __forceinline__ int unit_tiles(int Lraw, int T_, int max_blocks) {
  if (Lraw < 0 || Lraw > max_blocks * ATT_BS) return 1;
  return (Lraw + ATT_KT - 1) / ATT_KT + (T_ + ATT_KT - 1) / ATT_KT;
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ long long uniform64(long long v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}

struct AttnPlanLds {
  double wsum[ATT_NW];
  long long off;
  int b;
  int tiles[ATT_PAIRS];                // units dealt by length: each trajectory's tiles, and the trajectories
  unsigned short order[ATT_PAIRS];     // from the longest to the shortest
};

// Orders the trajectories (at most ATT_PAIRS) by falling tiles, equal ones by index. Whole block.
template <typename T>
__device__ __forceinline__ void attn_sort(AttnPlanLds& p, const AttnArgs<T>& a) {
  const int tid = threadIdx.x;
  static_assert(ATT_PAIRS <= ATT_NW * 64, "one trajectory per thread");
  if (tid < a.B) p.tiles[tid] = unit_tiles(a.ctx_len[tid], a.T_, a.max_blocks);
  __syncthreads();
  if (tid < a.B) {
    const int t = p.tiles[tid];
    int rank = 0;
    for (int c = 0; c < a.B; ++c) rank += p.tiles[c] > t || (p.tiles[c] == t && c < tid) ? 1 : 0;
    p.order[rank] = (unsigned short)tid;
  }
  __syncthreads();
}

// Unit at position pos of that order (uniform): trajectory, number in it and tiles.
__device__ __forceinline__ void attn_dealt(const AttnPlanLds& p, int units, int pos, int& b, int& j, int& t) {
  const int i = pos / units;
  b = __builtin_amdgcn_readfirstlane(p.order[i]);
  j = pos - i * units;
  t = __builtin_amdgcn_readfirstlane(p.tiles[b]);
}

// Length of all units together, in tiles; a unit counts as unit_cost tiles (what starting and writing it takes)
// more than it has, before its first (whole block; sums in float64 are exact here). Where a range is one or two given
// units: the number of ranges.
template <typename T>
__device__ __forceinline__ long long attn_total(AttnPlanLds& p, const AttnArgs<T>& a) {
  if (a.whole == 3) attn_sort(p, a);
  if (a.whole >= 2) return a.n_ranges;          // ranges of length 1
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double t = 0.0;
  for (int b = tid; b < a.B; b += ATT_NW * 64) t += (double)(unit_tiles(a.ctx_len[b], a.T_, a.max_blocks) + a.unit_cost);
  t = wave_sum_f64(t);
  if (lane == 0) p.wsum[wave] = t;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < ATT_NW; ++w) s += p.wsum[w];
  __syncthreads();
  return uniform64((long long)s * a.Hkv * a.row_groups);
}

// Trajectory that position pos lies in and the position inside it (p.b, p.off); with `store` also every
// trajectory's first position into a.work[1 + b]. Whole block.
template <typename T>
__device__ __forceinline__ void attn_locate(AttnPlanLds& p, const AttnArgs<T>& a, long long pos, bool store) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long units = (long long)a.Hkv * a.row_groups;
  double base = 0.0;
  if (tid == 0) p.b = -1;
  for (int b0 = 0; b0 < a.B; b0 += ATT_NW * 64) {
    const int b = b0 + tid;
    const double t = b < a.B ? (double)(unit_tiles(a.ctx_len[b], a.T_, a.max_blocks) + a.unit_cost) : 0.0;
    const double incl = wave_incl_scan_f64(t);
    if (lane == 63) p.wsum[wave] = incl;
    __syncthreads();
    double before = base;
#pragma unroll
    for (int w = 0; w < ATT_NW; ++w) {
      before += w < wave ? p.wsum[w] : 0.0;
      base += p.wsum[w];
    }
    const long long first = (long long)(before + (incl - t)) * units;
    if (b < a.B) {
      if (store) a.work[1 + b] = first;
      if (first <= pos && pos < first + (long long)t * units) { p.b = b; p.off = pos - first; }
    }
    __syncthreads();
    if (!store && p.b >= 0) break;              // uniform
  }
}

// Where range r starts: tile ta of unit j = g row_groups + rg of trajectory b, whose units have t tiles; left: the
// range's length from there, unit costs included (<= 0: no tile). Whole block, uniform.
struct AttnStart {
  int b, j, t, ta, left;
};
template <typename T>
__device__ __forceinline__ AttnStart attn_start(AttnPlanLds& p, const AttnArgs<T>& a, long long total, long long len, int r,
                                                bool store) {
  AttnStart s = {0, 0, 1, 0, 0};
  if (a.whole == 2) {                           // range r is unit r
    const int units = a.Hkv * a.row_groups;
    s.b = r / units;
    s.j = r - s.b * units;
    s.t = __builtin_amdgcn_readfirstlane(unit_tiles(a.ctx_len[s.b], a.T_, a.max_blocks));
    s.left = 1;
    return s;
  }
  if (a.whole == 3) {                           // units r and ATT_PAIRS - 1 - r
    attn_dealt(p, a.Hkv * a.row_groups, r, s.b, s.j, s.t);
    s.left = 1 << 30;
    return s;
  }
  const long long start = (long long)r * len, end = min(total, start + len);
  if (start >= end) return s;
  attn_locate(p, a, start, store);
  s.b = __builtin_amdgcn_readfirstlane(p.b);
  const unsigned long long o = (unsigned long long)uniform64(p.off);
  const uint32_t lo = (uint32_t)o, hi = (uint32_t)(o >> 32);
  s.t = __builtin_amdgcn_readfirstlane(unit_tiles(a.ctx_len[s.b], a.T_, a.max_blocks));
  const unsigned vt = (unsigned)(s.t + a.unit_cost);
  s.j = hi ? (int)(o / vt) : (int)(lo / vt);
  const int in = hi ? (int)(o % vt) : (int)(lo % vt);
  s.left = (int)(end - start);
  s.ta = max(0, in - a.unit_cost);
  if (s.ta == 0) s.left -= a.unit_cost - in;    // the rest of the unit's own cost
  if (a.whole && in > 0) {                      // the unit belongs to an earlier range
    s.left = (int)(end - start) - (int)(vt - in);
    if (s.left > 0) s.left = max(1, s.left - a.unit_cost);
    s.ta = 0;
    ++s.j;
  } else if (a.whole) {
    s.left = max(1, s.left);
  }
  return s;
}

// Partial result of the piece that range r has of unit j of trajectory b: 2 r for a piece at the range's start, 2 r + 1
// for one that the range's end cuts off; or, with fewer units than ranges (by_unit), r + the unit's number, which
// grows from piece to piece along the line, so every piece has its own.
__device__ __forceinline__ int attn_slot(int by_unit, int units, int r, int b, int j, bool first) {
  return by_unit ? r + b * units + j : 2 * r + (first ? 0 : 1);
}

// Segments of range r, in order: f(b, j, ta, n, slot, k) for tiles [ta, ta + n) of unit j of trajectory b, the k-th of
// the range; slot = -1 for a whole unit, else the index of its partial result (attn_slot). Whole block, uniform.
template <typename T, class F>
__device__ __forceinline__ void attn_walk(AttnPlanLds& p, const AttnArgs<T>& a, long long total, long long len, int r,
                                          bool store, F f) {
  AttnStart s = attn_start(p, a, total, len, r, store);
  const int units = a.Hkv * a.row_groups;
  int k = 0;
  while (s.left > 0) {
    if (a.whole == 3 && k > 0) {
      if (k > 1 || ATT_PAIRS - 1 - r >= a.B * units) break;
      attn_dealt(p, units, ATT_PAIRS - 1 - r, s.b, s.j, s.t);
    } else if (s.j == units) {
      s.j = 0;
      if (++s.b == a.B) break;
      s.t = __builtin_amdgcn_readfirstlane(unit_tiles(a.ctx_len[s.b], a.T_, a.max_blocks));
    }
    if (k > 0) {
      s.left -= a.unit_cost;
      if (s.left <= 0 && !a.whole) break;
    }
    const int n = a.whole ? s.t : min(s.t - s.ta, s.left);
    f(s.b, s.j, s.ta, n, n == s.t ? -1 : attn_slot(a.by_unit, units, r, s.b, s.j, k == 0), k);
    ++k;
    s.left -= n;
    s.ta = 0;                                   // a cut unit's rest belongs to the next range
    ++s.j;
  }
}

// Per-block metadata of one segment: the validated id of every prefix page, the tree's parents and ancestor
// masks (segments with tree tiles) and an input-error flag.
struct AttnMeta {
  int pg[ATT_SEG_TILES * ATT_TPP];
  uint32_t anc[SR_MAX_TREE][SR_MAX_TREE / 32];
  int parent[SR_MAX_TREE];
  int bad;
};

// Fills AttnMeta for pages [page0, page1) of trajectory b and, with tree tiles, its tree; validates the block
// table entries and the parent array this block reads. Whole block; returns the error flag.
__device__ __forceinline__ bool attn_meta(AttnMeta& m, bool ctx_ok, bool tree, int page0, int page1, const int32_t* bt_b,
                                          const int32_t* par_b, int T_, int num_blocks) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (tid == 0) m.bad = ctx_ok ? 0 : 1;
  __syncthreads();
  for (int p = page0 + tid; p < page1; p += nt) {
    int blk = bt_b[p];
    if (blk < 0 || blk >= num_blocks) { atomicOr(&m.bad, 1); blk = 0; }
    m.pg[p - page0] = blk;
  }
  if (tree) {
    for (int i = tid; i < T_; i += nt) {
      int p = par_b[i];
      if ((i == 0 && p != -1) || (i > 0 && (p < 0 || p >= i))) atomicOr(&m.bad, 1);
      m.parent[i] = p;
    }
    __syncthreads();
    if (!m.bad)
      for (int i = tid; i < T_; i += nt) {
        uint32_t a[SR_MAX_TREE / 32] = {0, 0, 0, 0};
        for (int u = i; u >= 0; u = m.parent[u]) a[u >> 5] |= 1u << (u & 31);
#pragma unroll
        for (int w = 0; w < SR_MAX_TREE / 32; ++w) m.anc[i][w] = a[w];
      }
  }
  __syncthreads();
  return m.bad != 0;
}

// Key ranges of a segment: n_pre prefix tiles with keys [key0, key1) on pages [page0, page1), then tree tiles from
// tree key 64 tree0.
struct AttnSeg {
  bool ctx_ok, tree;
  int n_pre, key0, key1, page0, page1, tree0;
};
__device__ __forceinline__ AttnSeg attn_seg(int Lraw, int max_blocks, int ta, int n) {
  AttnSeg s;
  s.ctx_ok = Lraw >= 0 && Lraw <= max_blocks * ATT_BS;
  const int L = s.ctx_ok ? Lraw : 0;
  const int np = (L + ATT_KT - 1) / ATT_KT;
  s.n_pre = max(0, min(np - ta, n));
  s.tree = s.ctx_ok && s.n_pre < n;
  s.tree0 = max(0, ta - np);
  s.key0 = s.n_pre > 0 ? ta * ATT_KT : 0;
  s.key1 = s.n_pre > 0 ? min(L, (ta + s.n_pre) * ATT_KT) : 0;
  s.page0 = s.key0 / ATT_BS;
  s.page1 = (s.key1 + ATT_BS - 1) / ATT_BS;
  return s;
}

template <class AT, int D>
struct AttnSmem {
  using G = AttnGeom<AT, D>;
  __attribute__((aligned(16))) unsigned char k[2][G::KTILE];
  __attribute__((aligned(16))) unsigned char v[2][G::VTILE];
};

// registers holding one tile's K and V while the previous tile is being computed
template <class AT, int D>
struct TileRegs {
  using G = AttnGeom<AT, D>;
  u32x4 k[G::KVPT];
  uint32_t v[G::VIPT][4][G::E];  // per item: 4 keys x (4 dims x E bytes)
};

// Segment (tiles [ta, ta + n) of the unit of trajectory b, KV head g, row group rg; slot as attn_walk gives it) of
// the register-staged path, rows [rg group_rows, min(R, (rg + 1) group_rows)) with group_rows <= ATT_ROWS. Whole
// block.
template <class AT, int D>
__device__ __forceinline__ void attn_seg_regs(AttnSmem<AT, D>& sm, AttnMeta& meta,
                                              const AttnArgs<typename AT::T>& a, int b, int g, int rg, int ta, int n,
                                              int slot) {
  using T = typename AT::T;
  using G = AttnGeom<AT, D>;
  constexpr int QKPL = AT::QKPL, KSTEP = 2 * QKPL, PKPL = AT::PKPL;
  constexpr int NQF = D / KSTEP;      // Q fragments per lane and row block
  constexpr int NDT = D / 32;         // 32-wide output tiles along D
  constexpr int NT = G::NT;
  constexpr int RB = ATT_RB;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int T_ = a.T_, Hq = a.Hq, Hkv = a.Hkv, R = a.R, group_rows = a.group_rows;
  const float scale_log2 = a.scale_log2;
  const T* __restrict__ q = a.q;
  float* __restrict__ out = a.out;
  float* __restrict__ lse = a.lse;
  const int G_ = Hq / Hkv;
  const AttnSeg sg = attn_seg(a.ctx_len[b], a.max_blocks, ta, n);
  const int page0 = sg.page0, key0 = sg.key0, key1 = sg.key1, n_pre = sg.n_pre, tree0 = sg.tree0;

  // ---- stage the page ids and (tree tiles) the ancestor masks; validate what this block reads
  __syncthreads();                    // the previous segment's LDS reads are done
  const bool bad = attn_meta(meta, sg.ctx_ok, sg.tree, page0, sg.page1, a.block_table + (size_t)b * a.max_blocks,
                             a.parents + (size_t)b * T_, T_, a.num_blocks);

  // ---- this wave's query rows: row r <-> (node t = r / G, head g*G + r % G); RB blocks of 32
  const int rend = min(R, (rg + 1) * group_rows);
  const int wrow0 = rg * group_rows + wave * RB * 32;
  int my_r[RB], my_t[RB];
  bool row_ok[RB];
  typename AT::qfrag qf[RB][NQF];
  uint32_t my_anc[RB][SR_MAX_TREE / 32];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    my_r[rb] = wrow0 + rb * 32 + (lane & 31);
    row_ok[rb] = my_r[rb] < rend;
    my_t[rb] = row_ok[rb] ? my_r[rb] / G_ : 0;
    const T* qp = q + (((size_t)b * T_ + my_t[rb]) * Hq + g * G_ + (row_ok[rb] ? my_r[rb] % G_ : 0)) * D;
#pragma unroll
    for (int kq = 0; kq < NQF; ++kq) {
      const int dd = kq * KSTEP + half * QKPL;
      if constexpr (QKPL == 8) {
        u32x4 z = {0, 0, 0, 0};
        if (row_ok[rb]) z = *(const u32x4*)(qp + dd);
        qf[rb][kq] = z;
      } else {
        qf[rb][kq] = row_ok[rb] ? qp[dd] : 0.f;
      }
    }
#pragma unroll
    for (int w = 0; w < SR_MAX_TREE / 32; ++w) my_anc[rb][w] = (sg.tree && !bad && row_ok[rb]) ? meta.anc[my_t[rb]][w] : 0u;
  }

  f32x16 o[RB][NDT];
  float m_run[RB], l_run[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int i = 0; i < NDT; ++i) o[rb][i] = (f32x16){};
    m_run[rb] = -INFINITY;
    l_run[rb] = 0.f;
  }
  const bool wave_active = wrow0 < rend && !bad;

  // ---- tile schedule: the segment's prefix tiles, then its tree tiles
  const int n_tiles = bad ? 0 : n;

  // The addresses inside a tile are formed again for every tile at D = 128: kept, they are registers that spill, and a
  // reload waits for the tile in flight (256 units of 224 rows, contexts of 750 to 6000 keys: 1249 -> 1012 us; 64 of
  // 320 rows, 250 to 2000: 242 -> 208). At D = 64 they fit (128 of 40 rows, 750 to 6000: 154 against 161).
  auto fresh = [](int v) __attribute__((always_inline)) -> int {
    if constexpr (D == 128) asm volatile("" : "+v"(v));
    return v;
  };
  // global -> registers for tile i. A key past the range is loaded from the range's last key instead
  // (so nothing past ctx_len is read and every staged value is finite); its score is masked to -inf,
  // so its K row never matters and its V row is multiplied by an exact zero.
  // this KV head's part of page 0 (page strides in bytes)
  const long long page_b = (long long)Hkv * ATT_BS * G::ROWB;
  const unsigned char* kc_b = (const unsigned char*)(a.k_cache + (size_t)g * ATT_BS * D);
  const unsigned char* vc_b = (const unsigned char*)(a.v_cache + (size_t)g * ATT_BS * D);
  const unsigned char* kt_b = (const unsigned char*)(a.k_tree + ((size_t)b * T_ * Hkv + g) * D);
  const unsigned char* vt_b = (const unsigned char*)(a.v_tree + ((size_t)b * T_ * Hkv + g) * D);
  const int tree_rowb = Hkv * G::ROWB;                                  // bytes between tree nodes
  auto load_tile = [&](const unsigned char* kb, const unsigned char* vb, int t0, int lim, auto off_of,
                       TileRegs<AT, D>& r) {
    const int tid = fresh(threadIdx.x);
#pragma unroll
    for (int j = 0; j < G::KVPT; ++j) {
      const int vi = tid + j * NT;
      const int key = vi / G::NCH, ch = vi % G::NCH;
      r.k[j] = *(const u32x4*)(kb + off_of(min(t0 + key, lim - 1)) + ch * 16);
    }
#pragma unroll
    for (int it = 0; it < G::VIPT; ++it) {
      const int item = tid + it * NT;
      if (item >= G::VITEMS) break;                   // uniform per wave
      const int kg = item / (D / 4), dg = item % (D / 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned char* src = vb + off_of(min(t0 + kg * 4 + j, lim - 1)) + dg * 4 * G::E;
        if constexpr (G::E == 2) {
          const u32x2 z = *(const u32x2*)src;
          r.v[it][j][0] = z[0];
          r.v[it][j][1] = z[1];
        } else {
          const u32x4 z = *(const u32x4*)src;
#pragma unroll
          for (int w = 0; w < 4; ++w) r.v[it][j][w] = z[w];
        }
      }
    }
  };
  auto fetch = [&](int i, TileRegs<AT, D>& r) {
    if (i < n_pre) {
      load_tile(kc_b, vc_b, key0 + i * ATT_KT, key1,
                [&](int kidx) -> long long { return meta.pg[(kidx >> 4) - page0] * page_b + (kidx & 15) * G::ROWB; }, r);
    } else {
      load_tile(kt_b, vt_b, (i - n_pre + tree0) * ATT_KT, T_, [&](int kidx) -> long long { return (long long)kidx * tree_rowb; },
                r);
    }
  };
  // registers -> LDS stage (K row-major with chunk swizzle, V transposed with group swizzle; bf16 V is
  // widened to the fp32 V^T element exactly)
  auto stash = [&](int st, const TileRegs<AT, D>& r) {
    const int tid = fresh(threadIdx.x);
#pragma unroll
    for (int j = 0; j < G::KVPT; ++j) {
      const int vi = tid + j * NT;
      const int key = vi / G::NCH, ch = vi % G::NCH;
      *(u32x4*)(sm.k[st] + key * G::ROWB + ((ch ^ (key & (G::NCH - 1))) * 16)) = r.k[j];
    }
#pragma unroll
    for (int it = 0; it < G::VIPT; ++it) {
      const int item = tid + it * NT;
      if (item >= G::VITEMS) break;
      const int kg = item / (D / 4), dg = item % (D / 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d = dg * 4 + i;
        unsigned char* dst = sm.v[st] + d * G::VROWB + ((kg ^ vswz(d)) * 4 * G::VE);
        f32x4 h;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (G::E == 2) {
            const uint32_t w = r.v[it][j][i >> 1];
            h[j] = bf2f((i & 1) ? (w >> 16) : (w & 0xffffu));
          } else {
            h[j] = __uint_as_float(r.v[it][j][i]);
          }
        }
        *(f32x4*)dst = h;
      }
    }
  };
  static_assert(G::VE == 4, "V^T is staged as fp32");

  auto compute = [&](int i, int st) {
    const bool tree = i >= n_pre;
    const int t0 = tree ? (i - n_pre + tree0) * ATT_KT : key0 + i * ATT_KT;
    const unsigned char* ks_ = sm.k[st];
    const unsigned char* vs_ = sm.v[st];
    // scores S^T: each K fragment feeds every row block
    f32x16 s[RB][2];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) s[rb][0] = s[rb][1] = (f32x16){};
#pragma unroll
    for (int kq = 0; kq < NQF; ++kq) {
      const int e = kq * KSTEP + half * QKPL;           // first element this lane supplies
      const int ch = (e * G::E) / 16;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int key = kt * 32 + (lane & 31);
        const unsigned char* p = ks_ + key * G::ROWB + ((ch ^ (key & (G::NCH - 1))) * 16) + (e * G::E) % 16;
        typename AT::qfrag kf;
        if constexpr (QKPL == 8) kf = *(const u32x4*)p; else kf = *(const float*)p;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) s[rb][kt] = AT::mma_qk(kf, qf[rb][kq], s[rb][kt]);
      }
    }
    // online softmax per row block; vis holds one bit per key of each 32-key subtile, pre-shifted by
    // this lane half's row offset
    typename AT::pfrag pf[RB][2][16 / PKPL];
    const bool full = !tree && t0 + ATT_KT <= key1;      // every key of the tile is visible to every row
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      uint32_t vis[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int kb = t0 + kt * 32;
        uint32_t v;
        if (tree) {
          const int wi = kb >> 5;
          v = wi == 0 ? my_anc[rb][0] : wi == 1 ? my_anc[rb][1] : wi == 2 ? my_anc[rb][2] : my_anc[rb][3];
        } else {
          const int nv = key1 - kb;
          v = nv >= 32 ? 0xffffffffu : (nv <= 0 ? 0u : ((1u << nv) - 1u));
        }
        vis[kt] = v >> (4 * half);
      }
      if (!full) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const bool ok = (vis[kt] >> (8 * (r >> 2) + (r & 3))) & 1u;
            s[rb][kt][r] = ok ? s[rb][kt][r] : -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[rb][kt][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      // the reference max moves only when the tile max exceeds it by more than 2^8 (P in [0, 256]), so
      // the accumulator is rarely rescaled
      const float tmax = mx * scale_log2;
      const float m_new = (tmax > m_run[rb] + 8.f) ? tmax : m_run[rb];
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run[rb] - m_use);
      float psum = 0.f;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][kt][r], scale_log2, -m_use));
          psum += p;
          pf[rb][kt][r] = p;
        }
      l_run[rb] = l_run[rb] * alpha + psum;
      m_run[rb] = m_new;
      if (__ballot(alpha != 1.f) != 0) {      // rescale only when some row's running max moved
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[rb][dt] *= alpha;
      }
    }
    // O^T += V^T P^T; each V fragment feeds every row block
    const int lane = fresh(threadIdx.x & 63), half = lane >> 5;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int kq = 0; kq < 16 / PKPL; ++kq) {
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int d = dt * 32 + (lane & 31);
          const unsigned char* vrow = vs_ + d * G::VROWB;
          const int sw = vswz(d);
          const int key = kt * 32 + tile_row(kq, half);
          const float vf = *(const float*)(vrow + (((key >> 2) ^ sw) * 16) + (key & 3) * 4);
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) o[rb][dt] = AT::mma_pv(vf, pf[rb][kt][kq], o[rb][dt]);
        }
      }
  };

  // ---- software pipeline: tile i+1 is in flight (registers) while tile i is computed from LDS
  if (n_tiles > 0) {
    TileRegs<AT, D> regs;
    fetch(0, regs);
    stash(0, regs);
    __syncthreads();
    for (int i = 0; i < n_tiles; ++i) {
      const int st = i & 1;
      const bool more = i + 1 < n_tiles;
      if (more) fetch(i + 1, regs);
      if (wave_active) compute(i, st);
      if (more) stash(st ^ 1, regs);
      __syncthreads();
    }
  }

  // ---- write the normalised result (a whole unit) or a partial (m, l, O/l)
  const float qnan = __uint_as_float(0x7fc00000u);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float l_tot = l_run[rb] + __shfl_xor(l_run[rb], 32, 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (!row_ok[rb]) continue;
    if (slot < 0) {
      const int h = g * G_ + my_r[rb] % G_;
      float* op = out + (((size_t)b * T_ + my_t[rb]) * Hq + h) * D;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = bad ? qnan : o[rb][dt][i + e] * inv;
          *(f32x4*)(op + dt * 32 + tile_row(i, half)) = v;
        }
      if (lse != nullptr && half == 0)
        lse[((size_t)b * T_ + my_t[rb]) * Hq + h] = bad ? qnan : (m_run[rb] + log2f(l_tot)) * kLn2;
    } else {
      const size_t pr = (size_t)slot * group_rows + (my_r[rb] - rg * group_rows);
      float* op = a.part_o + pr * D;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = o[rb][dt][i + e] * inv;
          *(f32x4*)(op + dt * 32 + tile_row(i, half)) = v;
        }
      if (half == 0) {
        a.part_ml[pr * 2 + 0] = bad ? qnan : m_run[rb];
        a.part_ml[pr * 2 + 1] = bad ? qnan : l_tot;
      }
    }
  }
}

// The range of block blk, for its it-th round (-1: none). Ranges that hold tiles are dealt so that neighbours (the
// row groups and pieces of one KV head) run on one XCD: consecutive blocks go to the XCDs in turn.
__device__ __forceinline__ int attn_range(int blk, int it, int grid, long long total, long long len) {
  const long long n_act = (total + len - 1) / len;
  long long r;
  if (n_act <= grid) {
    const int per = (int)((n_act + 7) / 8);
    r = it > 0 || (blk >> 3) >= per ? n_act : (long long)(blk & 7) * per + (blk >> 3);
    if (grid < 8 * per) r = it > 0 ? n_act : blk;      // a grid that does not fill the XCDs evenly
  } else {
    r = (long long)it * grid + blk;
  }
  return r < n_act ? (int)r : -1;
}

// Tiles per range: one range per block, as long as a range's page ids fit the LDS table; else as many for every
// block, in rounds. The plan's number of ranges allows for contexts of the block table's width, which the call's
// contexts mostly stay far below; cut into that many (265 for 256 trajectories of up to 16384 keys), nine blocks took
// two ranges: 0.59 ms where 256 ranges take 0.40.
template <typename T>
__device__ __forceinline__ long long attn_len(const AttnArgs<T>& a, long long total) {
  if (a.whole >= 2) return 1;
  const long long grid = gridDim.x, one = (total + grid - 1) / grid;
  const long long ranges = min((long long)a.n_ranges, grid * ((one + ATT_SEG_TILES - 1) / ATT_SEG_TILES));
  return uniform64(max((long long)a.min_tiles, (total + ranges - 1) / ranges));
}

// fp32 inputs.
template <int D>
__global__ __launch_bounds__(ATT_NW * 64) void k_tree_attn(AttnArgs<float> a) {
  __shared__ AttnSmem<AttnF32, D> sm;
  __shared__ AttnMeta meta;
  __shared__ AttnPlanLds plan;
  const long long total = attn_total(plan, a);
  const long long len = attn_len(a, total);
  if (blockIdx.x == 0 && threadIdx.x == 0 && !a.whole) a.work[0] = len;
  for (int it = 0;; ++it) {
    const int r = attn_range(blockIdx.x, it, gridDim.x, total, len);
    if (r < 0) break;
    attn_walk(plan, a, total, len, r, r == 0 && !a.whole, [&](int b, int j, int ta, int n, int slot, int) {
      attn_seg_regs<AttnF32, D>(sm, meta, a, b, j / a.row_groups, j % a.row_groups, ta, n, slot);
    });
  }
}

// fp32 inputs with at most 32 query rows per KV head. The kernel above gives one wave of such a block the whole chain
// of 64-cycle MFMAs of every tile; here each of the eight waves takes every eighth 32-key half tile of the segment
// for the same rows, its K and V straight from memory into MFMA operands, and the waves' results are merged in LDS.
// Bound by the MFMA chain of a half tile (2 us at D = 64) in small calls and by latency, one half tile per wave in
// flight, in large ones. Two trajectories, 16 rows, 100 and 160 keys: 28.6 -> 15.0 us; 64 trajectories, 2 KV heads,
// 32 rows, 200 to 3000 keys, D = 128: 325 -> 106 us; 16 trajectories, 4 KV heads, 32 rows, 30000 keys, D = 64: 612 ->
// 244 us. More than 32 rows would walk the same keys once per 32 of them.
template <int D>
struct AttnFew {
  static constexpr int RS = D + 4;      // staged row stride: the 32 rows of a store on distinct bank groups
  float o[ATT_NW][32][RS];
  float ml[ATT_NW][32][2];
};
template <int D>
__device__ __forceinline__ void attn_seg_few(AttnFew<D>& sm, AttnMeta& meta, const AttnArgs<float>& a, int b, int g, int rg,
                                             int ta, int n, int slot) {
  constexpr int NDT = D / 32, NK4 = D / 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int T_ = a.T_, G_ = a.Hq / a.Hkv;
  const AttnSeg sg = attn_seg(a.ctx_len[b], a.max_blocks, ta, n);
  __syncthreads();                    // the previous segment's LDS reads are done
  const bool bad = attn_meta(meta, sg.ctx_ok, sg.tree, sg.page0, sg.page1, a.block_table + (size_t)b * a.max_blocks,
                             a.parents + (size_t)b * T_, T_, a.num_blocks);
  const int rows = min(a.R - rg * a.group_rows, 32);
  const int my_r = rg * a.group_rows + (lane & 31);
  const bool row_ok = (lane & 31) < rows;
  const int my_t = row_ok ? my_r / G_ : 0;
  // dims in MFMA order: slot `half` of step 4 j + e is dim 8 j + 4 half + e, for K and Q alike
  float qf[4 * NK4];
  {
    const float* qp = a.q + (((size_t)b * T_ + my_t) * a.Hq + g * G_ + (row_ok ? my_r % G_ : 0)) * D;
#pragma unroll
    for (int j = 0; j < NK4; ++j) {
      const f32x4 v = *(const f32x4*)(qp + 8 * j + 4 * half);
#pragma unroll
      for (int e = 0; e < 4; ++e) qf[4 * j + e] = row_ok ? v[e] : 0.f;
    }
  }
  f32x16 o[NDT];
#pragma unroll
  for (int i = 0; i < NDT; ++i) o[i] = (f32x16){};
  float m_run = -INFINITY, l_run = 0.f;
  const long long page_e = (long long)a.Hkv * ATT_BS * D;          // elements per page
  const float* kc = a.k_cache + (size_t)g * ATT_BS * D;
  const float* vc = a.v_cache + (size_t)g * ATT_BS * D;
  const float* kt_b = a.k_tree + ((size_t)b * T_ * a.Hkv + g) * D;
  const float* vt_b = a.v_tree + ((size_t)b * T_ * a.Hkv + g) * D;
  const long long tree_e = (long long)a.Hkv * D;
  for (int sub = wave; sub < 2 * n && !bad; sub += ATT_NW) {
    const int i = sub >> 1;
    const bool tree = i >= sg.n_pre;
    const int t0 = (tree ? (i - sg.n_pre + sg.tree0) * ATT_KT : sg.key0 + i * ATT_KT) + 32 * (sub & 1);
    const int lim = tree ? T_ : sg.key1;
    if (t0 >= lim) continue;                      // uniform over the wave
    // a key past the range is loaded from the range's last key instead; its score is masked
    auto off_of = [&](int key) __attribute__((always_inline)) -> long long {
      const int k = min(key, lim - 1);
      return tree ? (long long)k * tree_e : meta.pg[(k >> 4) - sg.page0] * page_e + (k & 15) * D;
    };
    f32x4 kf[NK4];
    {
      const float* kp = (tree ? kt_b : kc) + off_of(t0 + (lane & 31));
#pragma unroll
      for (int j = 0; j < NK4; ++j) kf[j] = *(const f32x4*)(kp + 8 * j + 4 * half);
    }
    float vf[16][NDT];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* vp = (tree ? vt_b : vc) + off_of(t0 + tile_row(r, half));
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) vf[r][dt] = vp[dt * 32 + (lane & 31)];
    }
    f32x16 sc = (f32x16){};
#pragma unroll
    for (int j = 0; j < NK4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][e], qf[4 * j + e], sc, 0, 0, 0);
    uint32_t vis;
    if (tree) {
      vis = row_ok ? meta.anc[my_t][t0 >> 5] : 0u;
    } else {
      const int nv = lim - t0;
      vis = nv >= 32 ? 0xffffffffu : ((1u << nv) - 1u);
    }
    vis >>= 4 * half;
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = ((vis >> (8 * (r >> 2) + (r & 3))) & 1u) ? sc[r] : -INFINITY;
      mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx * a.scale_log2);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[r], a.scale_log2, -m_use));
      psum += sc[r];
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      o[dt] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r][dt], sc[r], o[dt], 0, 0, 0);
    }
  }
  // ---- merge the waves
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; i += 4)
      *(f32x4*)&sm.o[wave][lane & 31][dt * 32 + tile_row(i, half)] = (f32x4){o[dt][i], o[dt][i + 1], o[dt][i + 2], o[dt][i + 3]};
  if (half == 0) { sm.ml[wave][lane & 31][0] = m_run; sm.ml[wave][lane & 31][1] = l_tot; }
  __syncthreads();
  constexpr int TPR = ATT_NW * 64 / 32, DPT = D / TPR;   // threads per row, dims per thread
  const int row = tid / TPR, d0 = (tid % TPR) * DPT;
  if (row >= rows) return;
  float M = -INFINITY, W = 0.f, acc[DPT];
#pragma unroll
  for (int w = 0; w < ATT_NW; ++w) M = fmaxf(M, sm.ml[w][row][0]);
  const float Mu = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int e = 0; e < DPT; ++e) acc[e] = 0.f;
#pragma unroll
  for (int w = 0; w < ATT_NW; ++w) {
    const float f = __builtin_amdgcn_exp2f(sm.ml[w][row][0] - Mu);
    W += f * sm.ml[w][row][1];
#pragma unroll
    for (int e = 0; e < DPT; ++e) acc[e] += f * sm.o[w][row][d0 + e];
  }
  const float inv = W > 0.f ? 1.f / W : 0.f, qnan = __uint_as_float(0x7fc00000u);
  const int r = rg * a.group_rows + row, t = r / G_, h = g * G_ + r % G_;
  const size_t pr = slot < 0 ? ((size_t)b * T_ + t) * a.Hq + h : (size_t)slot * a.group_rows + row;
  float* op = (slot < 0 ? a.out : a.part_o) + pr * D + d0;
#pragma unroll
  for (int e = 0; e < DPT; e += 4) {
    f32x4 v;
#pragma unroll
    for (int f = 0; f < 4; ++f) v[f] = bad ? qnan : acc[e + f] * inv;
    *(f32x4*)(op + e) = v;
  }
  if (d0 == 0) {
    if (slot >= 0) {
      a.part_ml[pr * 2] = bad ? qnan : M;
      a.part_ml[pr * 2 + 1] = bad ? qnan : W;
    } else if (a.lse != nullptr) {
      a.lse[pr] = bad ? qnan : (M + log2f(W)) * kLn2;
    }
  }
}

template <int D>
__global__ __launch_bounds__(ATT_NW * 64) void k_tree_attn_few(AttnArgs<float> a) {
  __shared__ __attribute__((aligned(16))) AttnFew<D> sm;
  __shared__ AttnMeta meta;
  __shared__ AttnPlanLds plan;
  const long long total = attn_total(plan, a);
  const long long len = attn_len(a, total);
  if (blockIdx.x == 0 && threadIdx.x == 0 && !a.whole) a.work[0] = len;
  for (int it = 0;; ++it) {
    const int r = attn_range(blockIdx.x, it, gridDim.x, total, len);
    if (r < 0) break;
    attn_walk(plan, a, total, len, r, r == 0 && !a.whole, [&](int b, int j, int ta, int n, int slot, int) {
      attn_seg_few<D>(sm, meta, a, b, j / a.row_groups, j % a.row_groups, ta, n, slot);
    });
  }
}

// ============================================================================ bf16, direct-to-LDS
// The bf16 path streams K and V tiles from HBM straight into LDS (global_load_lds_dwordx4) through a
// four-slot ring: while tile i is finished and tile i+1 prepared, tiles i+2 and i+3 are in flight. In LDS,
// 16-byte chunk c of key row k sits at chunk position c ^ (k mod NCH) for K and c ^ (4 (k mod 4) mod NCH)
// for V, chosen by the source address each lane loads, which keeps the operand reads free of bank
// conflicts. Once per tile the block converts the tile's V from bf16 to fp16 in place, and the P V
// MFMAs read their V^T fragments straight from the row-major tile with the transposing LDS read
// (ds_read_b64_tr_b16: within 16 lanes, lane i receives element i mod 4 of the 8-byte rows addressed by
// lanes i/4, 4 + i/4, 8 + i/4 and 12 + i/4, so lanes addressing four keys of four consecutive dims each
// receive four keys of one dim). Each wave computes the scores of tile i+1 in the same instruction
// stream as the exponentials of tile i, so its matrix and vector work overlap. One barrier per tile.
template <int D>
struct DmaGeom {
  static constexpr int ROWB = D * 2;                   // bytes of one K or V row
  static constexpr int NCH = ROWB / 16;                // 16-byte chunks per row
  static constexpr int KPB = 1024 / ROWB;              // keys per 1 KB DMA block
  static constexpr int TILE = ATT_KT * ROWB;           // bytes of a K (or raw V) tile
  static constexpr int BLK = TILE / 1024;              // DMA blocks per tile, each of K and V
  static constexpr int CITEMS = TILE / 16;             // 16-byte chunks of a V tile (conversion items)
  static constexpr int CPL = CITEMS / 64;                // V chunks of a tile per lane of one wave
  static_assert(CITEMS % 64 == 0 && CPL >= ATT_NW, "tile split");
  static_assert(2 * BLK <= 63, "one tile of DMA per wave must fit the vmcnt counter");
  static_assert(KPB % 4 == 0, "a DMA block holds whole 4-key groups");
};

// max of x over lanes l and l ^ 32 (v_permlane32_swap exchanges the two 32-lane halves without LDS)
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// chunk-position swizzle of V row k: the eight rows of one transposing read (k mod 4 = 0..3, twice)
// take four different 64-byte column groups
template <int NCH> __device__ __forceinline__ int vswz(int k) { return (4 * (k & 3)) & (NCH - 1); }

// Complete this wave's LDS writes and its DMA for the next tile, then meet the block. A DMA wave (PT transfers
// per tile) may leave the transfers of the tile after that in flight when `ahead`.
template <int PT>
__device__ __forceinline__ void attn_sync(bool ahead) {
  if (!ahead) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PT) : "memory");
  }
}

// Read-only device data at wave-uniform addresses, through the scalar cache: these loads are not counted with the
// DMA transfers, so waiting for one does not wait for them.
__device__ __forceinline__ int uload(const int32_t* p, long long i) {
  typedef const __attribute__((address_space(4))) int32_t* cptr;
  return *((cptr)(uintptr_t)(p + i));
}

// The kernel's arguments, read from the argument segment where they are used: held in scalar registers throughout,
// they and the two segment iterators spill, and a DMA wave's reloads wait for its transfers.
typedef const __attribute__((address_space(4))) AttnArgs<bf16_t>* AttnKernArgs;
__device__ __forceinline__ AttnKernArgs kargs(AttnKernArgs p) {
  asm volatile("" : "+s"(p));
  return p;
}

__device__ __forceinline__ AttnArgs<bf16_t> kargs_copy(AttnKernArgs p) {
  union {
    AttnArgs<bf16_t> a;
    uint32_t w[sizeof(AttnArgs<bf16_t>) / 4];
  } u;
  const auto* w = (const __attribute__((address_space(4))) uint32_t*)kargs(p);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(u.w) / 4); ++i) u.w[i] = w[i];
  return u.a;
}

// Each compute wave's own tree scratch: the parents and its 32 rows' ancestor masks.
struct AttnWaveLds {
  int parent[ATT_NW - 1][SR_MAX_TREE];
  __attribute__((aligned(16))) uint32_t anc[ATT_NW - 1][32][SR_MAX_TREE / 32];
};

// 64-chunk blocks [first, first + n) of a V tile's CPL that a wave converts: one for each of the n_act compute
// waves (the first blocks), the rest for the waves without rows, the np DMA waves (the last) at half the weight;
// two for each when that leaves a lone DMA wave some (it sets the pace with nine blocks: 385 us against 375 us for
// 128 trajectories of 224 rows with 1-8k-token contexts).
template <int CPL>
__device__ __forceinline__ void attn_conv_share(int wave, int n_act, int np, int& first, int& n) {
  if (np == 1 && CPL > 2 * n_act) {
    first = 2 * wave;
    n = wave < n_act ? 2 : CPL - 2 * n_act;
    return;
  }
  if (wave < n_act) { first = wave; n = 1; return; }
  const int rest = CPL - n_act, nh = ATT_NW - n_act - np;
  const int ch = nh > 0 ? min((2 * rest + 2 * nh + np - 1) / (2 * nh + np), (rest + nh - 1) / nh) : 0;
  const int hsum = min(rest, nh * ch);             // blocks of the helpers together
  const int h = wave - n_act;
  if (h < nh) {
    first = n_act + min(h * ch, hsum);
    n = n_act + min((h + 1) * ch, hsum) - first;
  } else {
    const int rem = rest - hsum, p = h - nh, per = (rem + np - 1) / np;
    first = n_act + hsum + min(p * per, rem);
    n = n_act + hsum + min((p + 1) * per, rem) - first;
  }
}

// The segments of a range, one after the other (all uniform; attn_walk's order). A wave steps through them on its
// own: the DMA waves are up to three tiles ahead of the others.
struct SegIter {
  int b, j, t, ta, left, k;            // trajectory, unit, its tiles, first tile, virtual tiles left, ordinal
  int n, slot, tree0, n_pre, key0, key1;
  bool ctx_ok, head;
};

// Range r: its segments' tiles as one stream through the ring, so the next segment's first tiles are in flight
// while the last one's results are written. ring: four slots of a K tile then a V tile (bf16 as loaded, fp16 once
// converted). vw[k] receives the largest V magnitude pattern of segment k. Whole block; returns the number of
// segments, with the block's DMA drained.
//
// Roles. Waves [0, n_act) own 32 query rows each. The last wave (np = 1, when n_act = 7) or the last two (np = 2:
// one for K, one for V) issue the DMA, pacing themselves on the memory system (about 60 cycles a transfer: one
// wave takes 1.9k cycles for a tile's 32). The 16-byte chunks of a V tile are converted to fp16 one per lane by
// each compute wave, which has its own work, and the rest by the waves without rows, the DMA waves taking half
// the share of the others (attn_conv_share); all on one DMA wave took it 2.0k cycles a tile.
template <int D>
__device__ __forceinline__ int attn_range_dma(unsigned char (&ring)[4][2 * DmaGeom<D>::TILE], AttnWaveLds& wl, uint32_t* vw,
                                              int* badseg, AttnPlanLds& plan, AttnKernArgs kp,
                                              long long total, long long len, int r, bool store) {
  using G = DmaGeom<D>;
  constexpr int NQF = D / 16;         // Q fragments per lane
  constexpr int NDT = D / 32;         // 32-wide output tiles along D

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const float scale_log2 = kargs(kp)->scale_log2;
  AttnStart st0;
  {
    const AttnArgs<bf16_t> a = kargs_copy(kp);
    st0 = attn_start(plan, a, total, len, r, store);
  }
  if (st0.left <= 0) return 0;

  SegIter it;
  it.b = st0.b;
  it.j = st0.j;
  it.t = st0.t;
  it.ta = st0.ta;
  it.left = st0.left;
  it.k = 0;
  it.head = true;
  // fields of the segment at (b, j, ta); false past the range's last one
  auto seg_begin = [&](SegIter& i) __attribute__((always_inline)) -> bool {
    const auto* a = kargs(kp);
    if (i.left <= 0) return false;
    if (a->whole == 3 && !i.head) {
      const int units = a->Hkv * a->row_groups;
      if (i.k > 1 || ATT_PAIRS - 1 - r >= a->B * units) return false;
      attn_dealt(plan, units, ATT_PAIRS - 1 - r, i.b, i.j, i.t);
    } else if (i.j == a->Hkv * a->row_groups) {
      i.j = 0;
      if (++i.b == a->B) return false;
      i.t = unit_tiles(uload(a->ctx_len, i.b), a->T_, a->max_blocks);
    }
    if (i.ta == 0 && !i.head) {                  // the unit's own cost comes off the range first
      i.left -= a->unit_cost;
      if (i.left <= 0 && !a->whole) return false;
    }
    i.n = a->whole ? i.t : min(i.t - i.ta, i.left);
    i.slot = i.n == i.t ? -1 : attn_slot(a->by_unit, a->Hkv * a->row_groups, r, i.b, i.j, i.head);
    const AttnSeg sg = attn_seg(uload(a->ctx_len, i.b), a->max_blocks, i.ta, i.n);
    i.ctx_ok = sg.ctx_ok;
    i.tree0 = sg.tree0;
    i.n_pre = sg.n_pre;
    i.key0 = sg.key0;
    i.key1 = sg.key1;
    return true;
  };
  auto seg_end = [&](SegIter& i) __attribute__((always_inline)) {
    i.left -= i.n;
    i.ta = 0;
    ++i.j;
    ++i.k;
    i.head = false;
  };

  // ---- V of a tile, bf16 -> fp16 in place: every converting lane takes whole 16-byte chunks (their positions
  // do not matter). The conversion is exact for magnitudes in [2^-14, 65280] and truncates smaller ones to fp16's
  // subnormal step, an absolute error below 2^-24; larger ones would overflow. Each converting lane keeps the
  // largest magnitude pattern of everything it converts (two 16-bit lanes per register).
  u16x2 vmag_hi = {0, 0};
  auto conv_chunk = [&](const u32x4& x, unsigned char* dst) __attribute__((always_inline)) {
    // two values per instruction, rounding toward zero: exact for every value in fp16's normal range,
    // within one subnormal step (2^-24) below it; segments out of that range are recomputed anyway
    u32x4 h;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      h[w] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(x[w] << 16),
                                                                     __uint_as_float(x[w] & 0xffff0000u)));
      vmag_hi = __builtin_elementwise_max(vmag_hi, __builtin_bit_cast(u16x2, x[w] & 0x7fff7fffu));
    }
    *(u32x4*)dst = h;
  };
  // the segment whose tiles were converted so far ends: its largest pattern
  auto vmag_flush = [&](int k, u16x2 v) __attribute__((always_inline)) {
    const int hi = wave_max_i32((int)max((uint32_t)v[0], (uint32_t)v[1]));
    if (lane == 0) atomicMax(&vw[k], (uint32_t)hi);
  };

  const int n_act = min(ATT_NW - 1, (min(kargs(kp)->R, kargs(kp)->group_rows) + 31) / 32);
  const int np = n_act == ATT_NW - 1 ? 1 : 2;
  int c_first, c_n;                              // 64-chunk blocks of a V tile that this wave converts
  attn_conv_share<G::CPL>(wave, n_act, np, c_first, c_n);

  if (wave >= n_act) {
    // ================================================================ waves without query rows
    const int prod = wave - (ATT_NW - np);       // >= 0: a DMA wave
    const bool doK = np == 1 || prod == 0, doV = np == 1 || prod == 1;
    SegIter is = it;                             // the segment being issued
    int il = 0;                                  // its next tile
    bool more = seg_begin(is);
    int pg[4];                                   // page ids of the next tile (prefix tiles)
    // the segment's K and V (this head's part of page 0), page list and page stride
    const unsigned char *kc_b = nullptr, *vc_b = nullptr;
    const int32_t* bt = nullptr;
    const int num_blocks = kargs(kp)->num_blocks;
    const unsigned long long page_b = (unsigned long long)kargs(kp)->Hkv * ATT_BS * G::ROWB;
    auto seg_bases = [&]() __attribute__((always_inline)) {
      const auto* a = kargs(kp);
      const int g = is.j / a->row_groups;
      kc_b = (const unsigned char*)(a->k_cache + (size_t)g * ATT_BS * D);
      vc_b = (const unsigned char*)(a->v_cache + (size_t)g * ATT_BS * D);
      bt = a->block_table + (long long)is.b * a->max_blocks;
    };
    auto load_pages = [&]() __attribute__((always_inline)) {
      if (more && il < is.n_pre) {
        const int p0 = (is.key0 >> 4) + il * ATT_TPP, pl = (is.key1 - 1) >> 4;
#pragma unroll
        for (int p = 0; p < ATT_TPP; ++p) pg[p] = uload(bt, min(p0 + p, pl));
      }
    };
    if (prod >= 0 && more) {
      seg_bases();
      load_pages();
    }
    // issue the next tile of the stream into slot. A full prefix tile is four whole pages: each page's K and V
    // bases are uniform (scalar registers) and a block's per-lane offset inside its page depends only on the
    // block's position in the page, so every transfer is a scalar base plus one of BPP lane offsets. Other tiles
    // clamp keys past the range to its last key (nothing past ctx_len is read and every staged value is finite;
    // such a key's score is masked to -inf, so its K row never matters and its V row is multiplied by an exact
    // zero).
    auto issue = [&](unsigned char* slot) __attribute__((always_inline)) {
      const bool tree = il >= is.n_pre;
      const int t0 = tree ? (il - is.n_pre + is.tree0) * ATT_KT : is.key0 + il * ATT_KT;
      int ln = lane;
      asm volatile("" : "+v"(ln));                // lane offsets are rebuilt per tile, not kept live
      const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
          (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)slot);
      bool bad = false;
      if (!tree) {
#pragma unroll
        for (int p = 0; p < ATT_TPP; ++p) {
          const bool out = pg[p] < 0 || pg[p] >= num_blocks;
          bad |= out;
          pg[p] = out ? 0 : pg[p];
        }
      }
      if (!tree && t0 + ATT_KT <= is.key1) {
        constexpr int BPP = ATT_BS / G::KPB;          // DMA blocks per page
        uint32_t ko[BPP], vo[BPP];
#pragma unroll
        for (int j = 0; j < BPP; ++j) {
          const int kr = j * G::KPB + ln / G::NCH, pos = ln % G::NCH;   // key row in the page, chunk
          ko[j] = kr * G::ROWB + ((pos ^ (kr & (G::NCH - 1))) * 16);
          vo[j] = kr * G::ROWB + ((pos ^ vswz<G::NCH>(kr)) * 16);
        }
        if (doK) {
#pragma unroll
          for (int p = 0; p < ATT_TPP; ++p) {
            const unsigned char* kb = kc_b + (unsigned long long)(uint32_t)pg[p] * page_b;
#pragma unroll
            for (int j = 0; j < BPP; ++j) lds_dma16_sv(ko[j], kb, lds0 + (p * BPP + j) * 1024);
          }
        }
        if (doV) {
#pragma unroll
          for (int p = 0; p < ATT_TPP; ++p) {
            const unsigned char* vb = vc_b + (unsigned long long)(uint32_t)pg[p] * page_b;
#pragma unroll
            for (int j = 0; j < BPP; ++j) lds_dma16_sv(vo[j], vb, lds0 + G::TILE + (p * BPP + j) * 1024);
          }
        }
      } else {
        const auto* a = kargs(kp);
        const int Hkv = a->Hkv, T_ = a->T_, g = is.j / a->row_groups;
        const long long tree_rowb = (long long)Hkv * G::ROWB;
        const unsigned char* kt_b = (const unsigned char*)(a->k_tree + ((size_t)is.b * T_ * Hkv + g) * D);
        const unsigned char* vt_b = (const unsigned char*)(a->v_tree + ((size_t)is.b * T_ * Hkv + g) * D);
        for (int blk = 0; blk < G::BLK; ++blk) {
          const int kk = blk * G::KPB + ln / G::NCH, pos = ln % G::NCH;
          long long off;
          if (tree) {
            off = (long long)min(t0 + kk, T_ - 1) * tree_rowb;
          } else {
            const int key = min(t0 + kk, is.key1 - 1), p = (key - t0) >> 4;
            const int id = p == 0 ? pg[0] : p == 1 ? pg[1] : p == 2 ? pg[2] : pg[3];
            off = (long long)((unsigned long long)(uint32_t)id * page_b) + (key & 15) * G::ROWB;
          }
          if (doK) lds_dma16_manual((tree ? kt_b : kc_b) + off + ((pos ^ (kk & (G::NCH - 1))) * 16), slot + blk * 1024);
          if (doV) lds_dma16_manual((tree ? vt_b : vc_b) + off + ((pos ^ vswz<G::NCH>(kk)) * 16), slot + G::TILE + blk * 1024);
        }
      }
      if (bad && lane == 0) badseg[is.k & 7] = is.k + 1;
      if (++il == is.n) {
        seg_end(is);
        il = 0;
        more = seg_begin(is);
        if (more) seg_bases();
      }
      load_pages();
    };
    // conversions: the reads are issued early and the converted chunks written later, so the LDS latency overlaps
    // the issue of the tile's transfers
    constexpr int CMAX = G::CPL - (ATT_NW - 1) > 5 ? G::CPL - (ATT_NW - 1) : 5;
    u32x4 cw[CMAX];
    auto conv_load = [&](const unsigned char* v) __attribute__((always_inline)) {
      int ln = lane;
      asm volatile("" : "+v"(ln));                  // addresses are not hoisted out of the tile loop
#pragma unroll
      for (int k = 0; k < CMAX; ++k)
        if (k < c_n) cw[k] = *(const u32x4*)(v + (ln + (c_first + k) * 64) * 16);
    };
    auto conv_store = [&](unsigned char* v) __attribute__((always_inline)) {
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll
      for (int k = 0; k < CMAX; ++k)
        if (k < c_n) conv_chunk(cw[k], v + (ln + (c_first + k) * 64) * 16);
    };
    // step x of the stream (one copy of the code for the two steps that only fill the ring, the one that waits for
    // tile 0, and the tiles'): wait for tile x + 1 -- tile x + 2 may be in flight -- and meet the block; refill the
    // slot of tile x - 1 with tile x + 3; convert this wave's share of tile x + 1's V
    SegIter cs = it;                             // the segment of tile x + 1 (of tile 0 at first)
    int l = 0;
    bool have = seg_begin(cs);
    bool ahead = false;                          // tile x + 2 was issued
    // Nothing that the compiler tracks may be in flight here: it does not see the transfers, and would wait for such a
    // load inside the loop, at every tile, with a vmcnt(0) that drains the tiles ahead (56 rows per KV head, 7B heads:
    // 128 contexts of 1-8k keys 309 against 258 us, 256 lognormal contexts 406 against 333).
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0) alone, and known to the compiler
    if (np == 1) __builtin_amdgcn_s_setprio(3);   // the one DMA wave shares its SIMD with a compute wave
#pragma unroll 1
    for (int x = -3; have; ++x) {
      unsigned char* vn = ring[(x + 1) & 3] + G::TILE;
      bool cv = false;
      if (x >= -1) {
        if (prod < 0) lds_barrier();             // a wave without transfers of its own waits for its LDS writes only
        else if (np == 1) attn_sync<2 * G::BLK>(ahead);
        else attn_sync<G::BLK>(ahead);
        cv = true;
        if (x >= 0 && ++l == cs.n) {             // tile x was its segment's last
          vmag_flush(cs.k, vmag_hi);
          vmag_hi = (u16x2){0, 0};
          seg_end(cs);
          l = 0;
          have = cv = seg_begin(cs);
        }
        if (cv) conv_load(vn);
      }
      ahead = more;
      if (more && prod >= 0) issue(ring[(x + 3) & 3]);
      if (cv) conv_store(vn);
    }
    return cs.k;
  }

  // ================================================================== compute waves
  // this wave's 32 query rows in a segment: row r <-> (node t = r / G, head g*G + r % G)
  u32x4 qf[NQF];
  int par0 = 0, par1 = 0;
  int my_r = 0, my_t = 0;
  bool row_ok = false;
  // issue the loads of segment i's queries and tree
  auto load_rows = [&](const SegIter& i) __attribute__((always_inline)) {
    const auto* a = kargs(kp);
    const int G_ = a->Hq / a->Hkv, T_ = a->T_, R = a->R, group_rows = a->group_rows;
    const int g = i.j / a->row_groups, rg = i.j - g * a->row_groups;
    my_r = rg * group_rows + wave * 32 + (lane & 31);
    row_ok = my_r < min(R, (rg + 1) * group_rows);
    my_t = row_ok ? my_r / G_ : 0;
    const bf16_t* qp = a->q + (((size_t)i.b * T_ + my_t) * a->Hq + g * G_ + (row_ok ? my_r % G_ : 0)) * D;
#pragma unroll
    for (int kq = 0; kq < NQF; ++kq) {
      u32x4 z = {0, 0, 0, 0};
      if (row_ok) z = *(const u32x4*)(qp + kq * 16 + half * 8);
      qf[kq] = z;
    }
    if (i.n_pre < i.n) {
      const int32_t* pb = a->parents + (size_t)i.b * T_;
      par0 = lane < T_ ? pb[lane] : 0;
      par1 = lane + 64 < T_ ? pb[lane + 64] : 64;
    }
  };
  // ancestor mask of this lane's row into the wave's own LDS; true: the parent array is malformed
  auto tree_masks = [&](const SegIter& i) __attribute__((always_inline)) -> bool {
    if (i.n_pre >= i.n) return false;
    const int T_ = kargs(kp)->T_;
    const bool b0 = lane < T_ && (lane == 0 ? par0 != -1 : par0 < 0 || par0 >= lane);
    const bool b1 = lane + 64 < T_ && (par1 < 0 || par1 >= lane + 64);
    if (__ballot(b0 || b1)) return true;
    wl.parent[wave][lane] = par0;
    wl.parent[wave][lane + 64] = par1;
    uint32_t m0 = 0, m1 = 0, m2 = 0, m3 = 0;
    for (int u = my_t; u >= 0; u = wl.parent[wave][u]) {   // terminates: parents strictly decrease
      const uint32_t bit = 1u << (u & 31);
      m0 |= u < 32 ? bit : 0u;
      m1 |= (u >> 5) == 1 ? bit : 0u;
      m2 |= (u >> 5) == 2 ? bit : 0u;
      m3 |= (u >> 5) == 3 ? bit : 0u;
    }
    *(u32x4*)wl.anc[wave][lane & 31] = (u32x4){m0, m1, m2, m3};
    return false;
  };

  f32x16 o[NDT];
  float m_run = -INFINITY, l_run = 0.f;
  const int help_off = (c_first * 64 + lane) * 16;   // this wave's chunk of a V tile
  // scores S^T = K Q^T of the tile in ks
  auto qk = [&](const unsigned char* ks, f32x16 (&s)[2]) {
    s[0] = s[1] = (f32x16){};
#pragma unroll
    for (int kq = 0; kq < NQF; ++kq) {
      const int ch = 2 * kq + half;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int key = kt * 32 + (lane & 31);
        const u32x4 kf = *(const u32x4*)(ks + key * G::ROWB + ((ch ^ (key & (G::NCH - 1))) * 16));
        s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf),
                                                        __builtin_bit_cast(bf16x8, qf[kq]), s[kt], 0, 0, 0);
      }
    }
  };
  // mask, online softmax and O^T += V^T P^T for a tile (scores s); the next tile's scores (K in nks) are
  // computed into sn in the same basic block as this tile's exponentials
  float f_muse = 0.f, f_alpha = 1.f;
  // mask of the scores of the segment's tile i (a whole prefix tile needs none)
  auto tile_full = [&](int i) -> bool { return i < it.n_pre && it.key0 + i * ATT_KT + ATT_KT <= it.key1; };
  auto mask_tile = [&](int i, f32x16 (&s)[2]) {
    const bool tree = i >= it.n_pre;
    const int t0 = tree ? (i - it.n_pre + it.tree0) * ATT_KT : it.key0 + i * ATT_KT;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const int kb = t0 + kt * 32;
      uint32_t v;
      if (tree) {
        v = row_ok ? wl.anc[wave][lane & 31][kb >> 5] : 0u;
      } else {
        const int nv = it.key1 - kb;
        v = nv >= 32 ? 0xffffffffu : (nv <= 0 ? 0u : ((1u << nv) - 1u));
      }
      v >>= 4 * half;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool ok = (v >> (8 * (r >> 2) + (r & 3))) & 1u;
        s[kt][r] = ok ? s[kt][r] : -INFINITY;
      }
    }
  };
  // from a lane's max of a tile's (masked) scores: the row max, the new reference max and the accumulator
  // rescale. The reference max moves only when the tile max exceeds it by more than 2^8, so the accumulator
  // is rarely rescaled. Run for the first tile and for a tile whose weights outgrow the reference
  // (finish_rest).
  auto commit_max = [&](float mx) {
    mx = max_halves(mx);
    const float tmax = mx * scale_log2;
    const float m_new = (tmax > m_run + 8.f) ? tmax : m_run;
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
    if (__ballot(alpha != 1.f) != 0) {      // rescale only when some row's running max moved
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) o[dt] *= alpha;
    }
    m_run = m_new;
    f_muse = m_use;
    f_alpha = alpha;
  };
  // exponentials of a tile (scores s) against the current reference max, computed in one basic block with
  // the scores of the next tile (K in nks, into sn), then O^T += V^T P^T with V of the tile (vs); then
  // the mask of the next tile's scores (partial or tree tiles; mask_next: its index in the segment, or -1)
  auto finish_rest = [&](f32x16 (&s)[2], const unsigned char* vs, const unsigned char* nks, f32x16 (&sn)[2], int mask_next) {
    float m_use = f_muse;
    // From here on one basic block, laid out by hand with scheduling fences: each step issues the
    // K fragment reads one step ahead, two score MFMAs of the next tile and 32/NQF of this tile's
    // exponentials (the matrix core works while the vector ALU exponentiates); then the P V MFMAs
    // with their V fragment reads two ahead.
    constexpr int EPQ = 32 / NQF;                 // exponentials per score step
    f16x8 pf[2][2];
    float psum = 0.f;
    // weights of scores e, e+1 of this tile into pf; the row sum takes the fp16 weights the P V product
    // uses, in fp32 (v_dot2_f32_f16)
    auto exp_pair = [&](int e) __attribute__((always_inline)) {
      const int kt = e >> 4, r = e & 15;
      const _Float16 h0 = (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][r], scale_log2, -m_use));
      const _Float16 h1 = (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][r + 1], scale_log2, -m_use));
      pf[kt][r >> 3][r & 7] = h0;
      pf[kt][r >> 3][(r & 7) + 1] = h1;
      psum = __builtin_amdgcn_fdot2((f16x2){h0, h1}, (f16x2){(_Float16)1.f, (_Float16)1.f}, psum, false);
    };
    u32x4 kf[2][2];
    auto kread = [&](int kq, u32x4 (&dst)[2]) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int key = kt * 32 + (lane & 31), ch = 2 * kq + half;
        dst[kt] = *(const u32x4*)(nks + key * G::ROWB + ((ch ^ (key & (G::NCH - 1))) * 16));
      }
    };
    sn[0] = sn[1] = (f32x16){};
    kread(0, kf[0]);
#pragma unroll
    for (int kq = 0; kq < NQF; ++kq) {
      if (kq + 1 < NQF) kread(kq + 1, kf[(kq + 1) & 1]);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        sn[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[kq & 1][kt]),
                                                         __builtin_bit_cast(bf16x8, qf[kq]), sn[kt], 0, 0, 0);
#pragma unroll
      for (int e = kq * EPQ; e < (kq + 1) * EPQ; e += 2) exp_pair(e);
      __builtin_amdgcn_sched_barrier(0);
    }
    // The reference max is lazy: no tile max is taken while every lane's weights stay small. A tile whose
    // half-row weights add up past 2^14 (or overflow) moves the reference to its own max (the row max and
    // the accumulator rescale as for the first tile) and is weighted again; weights below 2^14 are exact in
    // fp16 up to its rounding, like those below 2^8.
    if (__ballot(!(psum <= 16384.f)) != 0) {
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
      const float a0 = f_alpha;
      commit_max(mx);
      f_alpha *= a0;
      m_use = f_muse;
      psum = 0.f;
#pragma unroll
      for (int e = 0; e < 32; e += 2) exp_pair(e);
    }
    l_run = l_run * f_alpha + psum;
    f_alpha = 1.f;
    constexpr int NPV = 4 * NDT;                  // P V MFMAs per tile
    f16x8 vf[3];
    // V^T fragment (dims dt*32 + lane%32; keys of k-slot 8*half + j: 16 kq + 8 (j/4) + 4 half + j%4) as two
    // transposing reads of four keys each: lane s of a 16-lane group addresses key row kb + s/4, dims
    // d0 + 4 (s mod 4) .. + 3
    auto vread = [&](int j) __attribute__((always_inline)) -> f16x8 {
      const int kt = j / (2 * NDT), kq = (j / NDT) & 1, dt = j % NDT;
      const int s16 = lane & 15, d0 = dt * 32 + 16 * ((lane >> 4) & 1);
      const int col = d0 + 4 * (s16 & 3);             // first of the four dims this lane addresses
      f16x4 part[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int row = kt * 32 + kq * 16 + 8 * r + 4 * half + (s16 >> 2);
        const unsigned char* a = vs + row * G::ROWB + (((col >> 3) ^ vswz<G::NCH>(row)) * 16) + (col & 7) * 2;
        part[r] = __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                (__attribute__((address_space(3))) v4i16*)(a)));
      }
      return (f16x8){part[0][0], part[0][1], part[0][2], part[0][3], part[1][0], part[1][1], part[1][2], part[1][3]};
    };
    if (mask_next >= 0 && !tile_full(mask_next)) mask_tile(mask_next, sn);
    vf[0] = vread(0);
    vf[1] = vread(1);
#pragma unroll
    for (int j = 0; j < NPV; ++j) {
      if (j + 2 < NPV) vf[(j + 2) % 3] = vread(j + 2);
      const int kt = j / (2 * NDT), kq = (j / NDT) & 1, dt = j % NDT;
      o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[j % 3], pf[kt][kq], o[dt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };


  // ---- pipeline. step(gi): wait for tile gi + 1 of the stream, then finish tile gi while computing the scores of
  // tile gi + 1 (discarded when that tile belongs to the next segment or is past the last) and converting this
  // wave's chunk of its V, which is consumed after the next barrier. The DMA waves keep the same barriers: wait
  // for tile gi + 1 (tiles gi + 2, gi + 3 may stay in flight), refill the slot of tile gi - 1 with tile gi + 3.
  bool have = seg_begin(it);
  load_rows(it);
  lds_barrier();                                // tile 0 landed
  {
    unsigned char* hc = ring[0] + G::TILE + help_off;
    conv_chunk(*(const u32x4*)hc, hc);
    if (c_n == 2) conv_chunk(*(const u32x4*)(hc + 1024), hc + 1024);
  }
  int si = 0;
  f32x16 sa[2], sb[2];
  while (have) {
    const bool bad_tree = tree_masks(it);
#pragma unroll
    for (int i = 0; i < NDT; ++i) o[i] = (f32x16){};
    m_run = -INFINITY;
    l_run = 0.f;
    f_alpha = 1.f;
    qk(ring[si], sa);
    {
      if (!tile_full(0)) mask_tile(0, sa);
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sa[kt][r]);
      commit_max(mx);
    }
    SegIter nx = it;
    seg_end(nx);
    const bool have_n = seg_begin(nx);
    u16x2 vseg = {0, 0};
    auto step = [&](int i, f32x16 (&s)[2], f32x16 (&sn)[2]) __attribute__((always_inline)) {
      const int sn_ = (si + 1) & 3;
      lds_barrier();
      const bool last = i + 1 == it.n;
      const bool cvn = !last || have_n;
      unsigned char* hc = ring[sn_] + G::TILE + help_off;   // this wave's chunks of the next tile's V
      u32x4 hw, hw2;
      if (cvn) hw = *(const u32x4*)hc;
      if (cvn && c_n == 2) hw2 = *(const u32x4*)(hc + 1024);
      // after the last tile the next scores come from a slot no DMA is writing and are discarded
      finish_rest(s, ring[si] + G::TILE, ring[sn_], sn, last ? -1 : i + 1);
      vseg = vmag_hi;                           // without the next tile's chunk: the segment's, after its last tile
      vmag_hi = last ? (u16x2){0, 0} : vmag_hi;
      if (cvn) conv_chunk(hw, hc);
      if (cvn && c_n == 2) conv_chunk(hw2, hc + 1024);
      si = sn_;
    };
    for (int i = 0; i < it.n; i += 2) {
      step(i, sa, sb);
      if (i + 1 < it.n) step(i + 1, sb, sa);
    }
    vmag_flush(it.k, vseg);

    // ---- write the normalised result (a whole unit) or a partial (m, l, O/l); the next segment's queries are
    // loaded first, so that waiting for them does not wait for these stores
    const auto* a = kargs(kp);
    const int G_ = a->Hq / a->Hkv, T_ = a->T_, group_rows = a->group_rows;
    float* __restrict__ out = a->out;
    float* __restrict__ lse = a->lse;
    const int w_b = it.b, w_g = it.j / a->row_groups, w_r = my_r, w_t = my_t, w_slot = it.slot;
    const int w_rr = my_r - (it.j - w_g * a->row_groups) * group_rows;
    const bool w_ok = row_ok;
    const bool bad = bad_tree || !it.ctx_ok || badseg[it.k & 7] == it.k + 1;
    it = nx;
    have = have_n;
    if (have) load_rows(it);
    const float qnan = __uint_as_float(0x7fc00000u);
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (w_ok) {
      const int h = w_g * G_ + w_r % G_;
      const size_t pr = w_slot < 0 ? ((size_t)w_b * T_ + w_t) * a->Hq + h : (size_t)w_slot * group_rows + w_rr;
      float* op = (w_slot < 0 ? out : a->part_o) + pr * D;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = bad ? qnan : o[dt][i + e] * inv;
          *(f32x4*)(op + dt * 32 + tile_row(i, half)) = v;
        }
      if (half == 0) {
        if (w_slot >= 0) {
          a->part_ml[pr * 2 + 0] = bad ? qnan : m_run;
          a->part_ml[pr * 2 + 1] = bad ? qnan : l_tot;
        } else if (lse != nullptr) {
          lse[pr] = bad ? qnan : (m_run + log2f(l_tot)) * kLn2;
        }
      }
    }
  }
  return it.k;
}

// One block per range. Segments whose V needs fp32 (largest magnitude past 65280, pattern 0x477f, inf and NaN
// included; or, below 2^-6, 0x3c80, too small for fp16's subnormal step) are recomputed by the same block at the
// end of its range, so no launch has to look for them.
template <int D>
struct AttnWide {
  AttnSmem<AttnBf16Wide, D> kv;
  AttnMeta meta;
};
// Recomputes range r's segments whose vw asks for it. Out of line, with its arguments in LDS: inlined, its registers
// cost the kernel's tile loop 70 spilled ones.
template <int D>
__device__ __attribute__((noinline)) void attn_redo(__attribute__((address_space(3))) void* lds,
                                                    __attribute__((address_space(3))) const uint32_t* args,
                                                    __attribute__((address_space(3))) void* plan,
                                                    __attribute__((address_space(3))) const uint32_t* vw, long long total,
                                                    long long len, int r) {
  union {
    AttnArgs<bf16_t> a;
    uint32_t w[sizeof(AttnArgs<bf16_t>) / 4];
  } u;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(u.w) / 4); ++i) u.w[i] = __builtin_amdgcn_readfirstlane(args[i]);
  AttnWide<D>* wide = (AttnWide<D>*)lds;
  r = __builtin_amdgcn_readfirstlane(r);
  attn_walk(*(AttnPlanLds*)plan, u.a, total, len, r, false, [&](int b, int j, int ta, int n, int slot, int k) __attribute__((always_inline)) {
    const uint32_t hi = __builtin_amdgcn_readfirstlane(vw[k]);
    if (hi > 0x477fu || hi < 0x3c80u)
      attn_seg_regs<AttnBf16Wide, D>(wide->kv, wide->meta, u.a, b, j / u.a.row_groups, j % u.a.row_groups, ta, n, slot);
  });
}

template <int D>
__global__ __launch_bounds__(ATT_NW * 64) void k_tree_attn_dma(AttnArgs<bf16_t>) {
  const AttnKernArgs kp = (AttnKernArgs)__builtin_amdgcn_kernarg_segment_ptr();
  using Wide = AttnWide<D>;
  constexpr int RING = 4 * 2 * DmaGeom<D>::TILE;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[RING > (int)sizeof(Wide) ? RING : (int)sizeof(Wide)];
  __shared__ AttnWaveLds wl;
  __shared__ AttnPlanLds plan;
  __shared__ uint32_t vw[ATT_SEG_TILES];
  __shared__ AttnArgs<bf16_t> args;
  __shared__ int badseg[8];
  const int tid = threadIdx.x;
  long long total, len;
  {
    const AttnArgs<bf16_t> a = kargs_copy(kp);
    total = attn_total(plan, a);
    len = attn_len(a, total);
    if (blockIdx.x == 0 && tid == 0 && !a.whole) a.work[0] = len;
  }
  for (int it = 0;; ++it) {
    const int r = attn_range(blockIdx.x, it, gridDim.x, total, len);
    if (r < 0) break;
    __syncthreads();
    for (int i = tid; i < ATT_SEG_TILES; i += ATT_NW * 64) vw[i] = 0u;
    if (tid < 8) badseg[tid] = 0;
    __syncthreads();
    const bool store = r == 0 && !kargs(kp)->whole;
    const int n = attn_range_dma<D>(*(unsigned char(*)[4][2 * DmaGeom<D>::TILE])lds, wl, vw, badseg, plan, kp, total, len, r, store);
    __syncthreads();
    bool w = false;
    for (int k = tid; k < n; k += ATT_NW * 64) w |= vw[k] > 0x477fu || vw[k] < 0x3c80u;
    if (__syncthreads_or(w)) {
      if (tid == 0) args = kargs_copy(kp);
      __syncthreads();
      attn_redo<D>((__attribute__((address_space(3))) void*)lds, (__attribute__((address_space(3))) const uint32_t*)&args,
                   (__attribute__((address_space(3))) void*)&plan, (__attribute__((address_space(3))) const uint32_t*)vw, total, len, r);
    }
  }
}

// Merge the partial results of every unit that a range boundary cuts.
__device__ __forceinline__ bool total_fits_u32(long long hi, long long len) { return hi <= 0xffffffffll && len <= 0xffffffffll; }

template <int D>
__global__ __launch_bounds__(256) void k_attn_combine(const int32_t* __restrict__ ctx_len,
                                                      const long long* __restrict__ work,
                                                      const float* __restrict__ part_o,
                                                      const float* __restrict__ part_ml, float* __restrict__ out,
                                                      float* __restrict__ lse, int T_, int Hq, int Hkv,
                                                      int max_blocks, int R, int row_groups, int group_rows, int unit_cost, int by_unit) {
  constexpr int TPR = D / 4;                 // threads per row (4 floats each)
  constexpr int RPB = 256 / TPR;             // rows per block (all of one row group: groups are whole 32s)
  const int g = blockIdx.y, b = blockIdx.z;
  const long long len = work[0];
  const int t_u = unit_tiles(ctx_len[b], T_, max_blocks);
  const int rg = blockIdx.x * RPB / group_rows;
  // first tile and end of the unit
  const long long uv = work[1 + b] + (long long)(g * row_groups + rg) * (t_u + unit_cost), us = uv + unit_cost, ue = us + t_u;
  // the unit's pieces lie in ranges i0..i1
  const long long i0 = (total_fits_u32(ue, len) ? (long long)((uint32_t)us / (uint32_t)len) : us / len);
  const long long i1 = (total_fits_u32(ue, len) ? (long long)((uint32_t)(ue - 1) / (uint32_t)len) : (ue - 1) / len);
  if (i0 == i1) return;
  const int n_chunks = (int)(i1 - i0) + 1;
  const int r = blockIdx.x * RPB + threadIdx.x / TPR;
  const int d4 = (threadIdx.x % TPR) * 4;
  if (r >= R) return;
  const size_t rr = (size_t)(r - rg * group_rows);
  // pieces in groups of four: every load of a group is in flight at once, then the group is merged into
  // the running (M, W, acc) (one group, i.e. up to four pieces, is the plain max-then-sum)
  constexpr int CGRP = 4;
  float M = -INFINITY, W = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  bool nan = false;
  for (int c0 = 0; c0 < n_chunks; c0 += CGRP) {
    float2 ml[CGRP];
    f32x4 po[CGRP];
#pragma unroll
    for (int k = 0; k < CGRP; ++k) {
      const int slot = attn_slot(by_unit, Hkv * row_groups, (int)i0 + c0 + k, b, g * row_groups + rg,
                                 c0 + k > 0 || i0 * len >= uv);
      const size_t pr = (size_t)slot * group_rows + rr;
      if (c0 + k < n_chunks) {
        ml[k] = *(const float2*)(part_ml + pr * 2);
        po[k] = *(const f32x4*)(part_o + pr * D + d4);
      } else {
        ml[k] = make_float2(-INFINITY, 0.f);
        po[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
    }
    float Mn = M;
#pragma unroll
    for (int k = 0; k < CGRP; ++k) {
      nan |= isnan(ml[k].x) || isnan(ml[k].y);
      Mn = fmaxf(Mn, ml[k].x);
    }
    const float Mu = (Mn == -INFINITY) ? 0.f : Mn;
    const float sc = exp2f(M - Mu);           // 0 while nothing is merged yet (M = -inf)
    W *= sc;
    acc *= sc;
#pragma unroll
    for (int k = 0; k < CGRP; ++k) {
      const float w = ml[k].y * exp2f(ml[k].x - Mu);
      W += w;
      acc += w * po[k];
    }
    M = Mn;
  }
  const int G = Hq / Hkv;
  const int t = r / G, h = g * G + r % G;
  const float qnan = __uint_as_float(0x7fc00000u);
  const float inv = W > 0.f ? 1.f / W : 0.f;
  f32x4 v = acc * inv;
  if (nan) v = (f32x4){qnan, qnan, qnan, qnan};
  *(f32x4*)(out + (((size_t)b * T_ + t) * Hq + h) * D + d4) = v;
  if (lse != nullptr && d4 == 0) lse[((size_t)b * T_ + t) * Hq + h] = nan ? qnan : (M + log2f(W)) * kLn2;
}

AttnPlan attn_plan(const sr_attn_desc& d, size_t avail) {
  AttnPlan p;
  p.R = d.T * (d.Hq / d.Hkv);
  p.Rpad = (p.R + 31) / 32 * 32;
  // bf16: more than 224 rows split evenly into groups of at most 224, so every work item keeps a wave
  // free of query rows to issue its DMA (fp32: groups of 256). Fewer rows are one group of whole 32s: group_rows is
  // also the stride of the partial results, so their scratch follows the rows there are.
  p.group_rows = std::min(p.Rpad, ATT_ROWS);
  if (d.dtype == SR_BF16 && p.R > ATT_ROWS - 32) {
    const int ng = (p.R + (ATT_ROWS - 32) - 1) / (ATT_ROWS - 32);
    p.group_rows = ((p.R + ng - 1) / ng + 31) / 32 * 32;
  }
  p.row_groups = (p.R + p.group_rows - 1) / p.group_rows;
  // Ranges: one per CU; more, in whole rounds, only so that a range's page ids fit its LDS table at the longest
  // contexts the block table can hold. Short units are not worth cutting (a piece costs about as much to start and
  // merge as it saves): such calls keep them whole and need no partial results. With a block for every unit that is
  // so the longer the more blocks the units fill: bf16, 256 units of 224 rows, contexts of hi / 8 to hi keys: whole
  // 30, 48, 60, 87 us against cut 46, 59, 68, 86 at hi = 300, 1000, 1500, 2500; 128 of 112 rows 21, 28, 33, 41
  // against 29, 32, 34, 37 at 300, 700, 1000, 1500; 64 of 224 rows 25, 30, 35 against 31, 33, 33 at 300, 500, 700; 32 of
  // 192 rows 23, 28 against 25, 27 at 300, 500. Up to two for a block, dealt by length (cutting them costs every block a
  // third start, and the merge): 512 of 56 rows 36, 44, 54, 61, 91 against 41, 54, 64, 70, 99 at hi = 300, 700, 1200,
  // 1500, 2400; 344 of 84 rows 39, 47, 63 against 45, 54, 71 at 600, 1200, 2400; lognormal contexts of median hi / 6, whose
  // longest unit sets the time: 512 of 56 rows 50, 70 against 49, 59 at 1200, 2400. More units, ranges of whole ones: 1024
  // of 56 rows 65, 77 against 70, 78 at 300, 500. fp32, whose tiles are long: 256 units of 56 rows 84, 147 against 92,
  // 128 at 300, 700; 128 of 40 rows, D = 64, 37 against 28 at 300.
  const long long units = (long long)d.B * d.Hkv * p.row_groups;
  const int most = (d.max_blocks * ATT_BS + ATT_KT - 1) / ATT_KT + (d.T + ATT_KT - 1) / ATT_KT;   // tiles of a unit
  const bool each = units <= ATT_BLOCKS;
  const bool pairs = d.dtype == SR_BF16 && !each && units <= ATT_PAIRS && most <= ATT_PAIR_TILES;
  p.whole = pairs || most <= ATT_WHOLE + (d.dtype == SR_BF16 ? (each ? units * 5 / 64 : 3) : (each ? units / 128 : 0));
  p.min_tiles = d.dtype == SR_BF16 ? ATT_MIN_TILES : 1;
  // What starting and writing a unit counts for, fitted on lognormal and uniform contexts with 1 to 7 waves of rows
  // (1, 2, 3, 4, 6, 8, 12 tiles): 64 to 256 contexts of 56 to 112 rows, D = 128: 99, 180, 329 us with 6, 98, 181, 333
  // with 8, 113, 190, 337 with 3; 224 rows 364 with 6, 366 with 8; D = 64, whose tiles are half the bytes: 128
  // contexts of 32 rows 100 with 6, 101 with 8, 64 of 128 rows 62 with 6, 60 with 8. fp32 tiles are long: 8 contexts
  // of 320 rows 237 with 1, 253 with 2.
  p.unit_cost = d.dtype != SR_BF16 ? 1 : d.D == 64 ? 8 : 6;
  const long long tiles = units * (most + p.unit_cost);
  const long long table = (tiles + ATT_SEG_TILES - 1) / ATT_SEG_TILES;   // least ranges whose page ids fit the table
  const long long rounds = (table + ATT_BLOCKS - 1) / ATT_BLOCKS;
  // One to three units are cut into fewer pieces than there are blocks, since the merge takes a unit's pieces one after
  // the other (about a tenth of the time of a tile each): sqrt(8 tiles), at least ATT_PIECES (one unit of 64 rows,
  // D = 64, of 8000, 16000, 30000 keys: 25, 25, 28 us with 64, 25, 32, 47 with 256; 448 rows, 120000 keys: 70 with 64, 65
  // with 128 or 256).
  long long pieces = ATT_PIECES;
  while (pieces < ATT_BLOCKS && pieces * pieces < 8 * (long long)most) ++pieces;
  const long long ranges = std::min(tiles, rounds > 1 ? rounds * ATT_BLOCKS
                                                      : std::max(table, std::min<long long>(ATT_BLOCKS, pieces * units)));
  p.n_ranges = p.whole && each ? units : pairs ? ATT_BLOCKS : ranges;
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t row_bytes = (size_t)p.group_rows * (d.D + 2) * sizeof(float);   // one partial result
  const size_t work_bytes = up((size_t)(1 + d.B) * sizeof(long long));
  // Two partial results per range, or, with fewer units than ranges, one per range and one per unit.
  auto sizes = [&]() {
    p.by_unit = units < p.n_ranges;
    const size_t rows = p.whole ? 0 : (size_t)(p.n_ranges + std::min(units, p.n_ranges)) * p.group_rows;
    p.part_o_bytes = rows * d.D * sizeof(float);       // whole 256-byte lines: group_rows is a multiple of 32
    p.part_ml_bytes = rows * 2 * sizeof(float);
    p.work_bytes = p.whole ? 0 : work_bytes;
  };
  sizes();
  // The least workspace a call takes: the size of one partial result per prefix chunk of 32, 128 or 256 pages and,
  // for bf16, of two lists of the chunks. A workspace between that and the sizes above gets fewer ranges.
  const int cp = units < 64 ? 32 : units < 512 ? 128 : 256;
  const size_t nch = std::max(1, (d.max_blocks + cp - 1) / cp);
  const size_t crows = (size_t)d.B * d.Hkv * nch * p.Rpad;
  p.min_bytes = (nch > 1 ? up(crows * d.D * sizeof(float)) + up(crows * 2 * sizeof(float)) : 0) +
                (d.dtype == SR_BF16 ? up((size_t)(3 + 2 * units * (long long)nch) * sizeof(unsigned)) : 0);
  p.full_bytes = std::max(p.part_o_bytes + p.part_ml_bytes + p.work_bytes, p.min_bytes);
  if (avail < p.full_bytes && !p.whole) {
    const long long parts = avail > work_bytes ? (long long)std::min<size_t>((avail - work_bytes) / row_bytes, INT32_MAX) : 0;
    p.n_ranges = std::min(ranges, std::max(parts - units, parts / 2));
    // Units are left whole when that keeps more blocks busy than the ranges that fit, but never a unit whose page ids
    // would not fit the table. The least workspace always holds ranges that do (2 chunks of at most 64 tiles, and
    // what a unit has beside them, per range); should one not, the call is refused.
    if (p.n_ranges < table || p.n_ranges < std::min<long long>(units, ATT_BLOCKS)) {
      if (most <= ATT_SEG_TILES) {
        p.whole = true;
        p.n_ranges = each ? units : ranges;
      } else if (p.n_ranges < table) {
        p.n_ranges = table;
        p.min_bytes = p.full_bytes;
      }
    }
    sizes();
  }
  p.each = p.whole && each;
  p.pairs = p.whole && pairs;
  return p;
}

template <typename T, int D>
static sr_status launch_attn_t(const sr_attn_desc& d, const AttnPlan& p, const void* q, const void* kc,
                               const void* vc, const int32_t* bt, const int32_t* cl, const void* kt,
                               const void* vt, const int32_t* par, float* out, float* lse, float* po, float* pml,
                               long long* work, hipStream_t s) {
  if (p.n_ranges > INT32_MAX / 4) return SR_ERR_INVALID;
  const AttnArgs<T> a = {(const T*)q, (const T*)kc, (const T*)vc, bt, cl, (const T*)kt, (const T*)vt, par, out, lse, po, pml,
                         work, d.B, d.T, d.Hq, d.Hkv, d.max_blocks, d.num_blocks, d.scale * kLog2e, p.R, p.row_groups,
                         p.group_rows, (int)p.n_ranges, p.min_tiles, p.unit_cost, p.whole ? (p.each ? 2 : p.pairs ? 3 : 1) : 0, p.by_unit ? 1 : 0};
  const dim3 grid((unsigned)std::min<long long>(p.n_ranges, ATT_BLOCKS));
  if constexpr (sizeof(T) == 2) {
    SR_LAUNCH("sr_tree_attn", (k_tree_attn_dma<D>), grid, dim3(ATT_NW * 64), 0, s, a);
  } else if (p.R <= 32) {
    SR_LAUNCH("sr_tree_attn", (k_tree_attn_few<D>), grid, dim3(ATT_NW * 64), 0, s, a);
  } else {
    SR_LAUNCH("sr_tree_attn", (k_tree_attn<D>), grid, dim3(ATT_NW * 64), 0, s, a);
  }
  if (!p.whole) {
    constexpr int RPB = 256 / (D / 4);
    dim3 cgrid((p.R + RPB - 1) / RPB, d.Hkv, d.B);
    SR_LAUNCH("sr_attn_combine", (k_attn_combine<D>), cgrid, dim3(256), 0, s, cl, (const long long*)work, po, pml, out, lse,
              d.T, d.Hq, d.Hkv, d.max_blocks, p.R, p.row_groups, p.group_rows, a.unit_cost, a.by_unit);
  }
  return SR_OK;
}

sr_status launch_tree_attn(const sr_attn_desc& d, const AttnPlan& p, const void* q, const void* k_cache,
                           const void* v_cache, const int32_t* block_table, const int32_t* ctx_len,
                           const void* k_tree, const void* v_tree, const int32_t* parents, float* out,
                           float* lse, float* part_o, float* part_ml, long long* work, hipStream_t s) {
#define SR_ATTN_CASE(TT, DD)                                                                                  \
  return launch_attn_t<TT, DD>(d, p, q, k_cache, v_cache, block_table, ctx_len, k_tree, v_tree, parents, out, \
                               lse, part_o, part_ml, work, s)
  if (d.dtype == SR_BF16) {
    if (d.D == 128) SR_ATTN_CASE(bf16_t, 128);
    SR_ATTN_CASE(bf16_t, 64);
  }
  if (d.D == 128) SR_ATTN_CASE(float, 128);
  SR_ATTN_CASE(float, 64);
#undef SR_ATTN_CASE
}

}  // namespace sr
