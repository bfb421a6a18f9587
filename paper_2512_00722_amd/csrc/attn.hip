// Sparse GQA decode attention on gfx950 (SpeContext Eq. 1 over the selected
// tokens; Sec. 4.3 "Support for GQA": the G query heads of a group share one
// KV head, which is read directly -- no repeat_kv copy).
//
// Flash decode over work units (layer, sequence, KV head g, split of the
// selection).  One workgroup per CU runs one wavefront per SIMD; its
// wavefronts take units from a contiguous range on demand.  A wavefront walks
// its unit in chunks of 32 selected tokens:
//  * the unit's row indices are staged in LDS first, so no chunk waits on an
//    index load;
//  * S^T = K Q^T on the matrix cores (v_mfma_f32_16x16x32_bf16): A = 16
//    selected K rows, each lane feeding one 16-byte slice of one row straight
//    from HBM (no LDS staging, no conversion); B = Q^T with the G query heads
//    of the group as columns (columns >= G are zero).  Only G/16 of the tile
//    is useful, which does not matter: the op is HBM-bound;
//  * online softmax in log2 units (scale and log2(e) folded into one
//    multiply); the four lanes that hold one head combine with permlane swaps;
//  * O^T += V^T P^T on the matrix cores: V rows arrive as 16-byte loads (four
//    whole 256-byte rows per instruction), are staged in LDS and read back
//    transposed with ds_read_b64_tr_b16; P is split into a bf16 high part and
//    a bf16 low part (two MFMAs), which keeps it to ~2^-16 relative;
//  * K and V of chunk c+1 are requested as soon as chunk c's registers are
//    consumed and stay in flight through chunk c's softmax and MFMAs;
//  * when a wavefront has several units they are pipelined: when it starts a
//    unit it also takes its next one and requests that unit's count, row indices and queries
//    together (the indices unconditionally; the count only masks them), and
//    stages its rows in the other half of a double-buffered row area.  The
//    last chunk's refill then requests the next unit's first chunk, so a unit
//    boundary costs no round trip.
// Launches with fewer groups than that keeps busy take attn_team_kernel, whose
// workgroups share a unit between their wavefronts (see there).
// The workgroups own contiguous ranges of a permuted unit order (groups of a
// (layer, sequence, split) spread over the whole range), so that ragged
// selections even out across workgroups.  Pipelined launches over batches
// of unequal selections deal the groups to the workgroups by selection size
// instead (longest first, in a snake), which evens them out further.
// A unit that covers a whole selection normalises and writes out/lse itself;
// split selections leave (max, sum, acc) partials that a second kernel merges
// with a log-sum-exp combine.
#include <float.h>
#include <stdlib.h>
#include <string.h>

#include "device_common.h"
#include "internal.h"

namespace spec {
namespace {

#ifndef SPEC_ATTN_CHUNK
#define SPEC_ATTN_CHUNK 32
#endif
#ifndef SPEC_ATTN_NT
#define SPEC_ATTN_NT 1
#endif
#ifndef SPEC_ATTN_WPE
#define SPEC_ATTN_WPE 2  // wavefronts per SIMD the register budget is sized for
#endif
#ifndef SPEC_ATTN_WAVES
#define SPEC_ATTN_WAVES 4
#endif
constexpr int kWaves = SPEC_ATTN_WAVES;   // wavefronts per workgroup
constexpr int kChunk = SPEC_ATTN_CHUNK;   // selected tokens per inner step (32 or 64)
constexpr int kTiles = kChunk / 16;       // 16-token MFMA tiles per chunk
constexpr int kVRows = kChunk / 4;        // V rows per lane per chunk
constexpr int kD = 128;                   // head dimension
constexpr int kMaxSplit = 2048;           // longest split (tokens per work item)
#ifndef SPEC_ATTN_MIN_SPLIT
#define SPEC_ATTN_MIN_SPLIT 256
#endif

constexpr int kMinSplitTokens = SPEC_ATTN_MIN_SPLIT;
#ifndef SPEC_ATTN_SLOT_UNITS
#define SPEC_ATTN_SLOT_UNITS 1
#endif
// Work units per resident wavefront the selections are split into when there
// are fewer (layer, sequence, KV head) groups than wavefronts.
constexpr int kSlotUnits = SPEC_ATTN_SLOT_UNITS;

// K/V rows are read once per launch: stream them past the caches.
__device__ __forceinline__ uint4 ldkv(const uint16_t* p) {
#if SPEC_ATTN_NT
  return ldg16_stream(p);
#else
  return ldg16(p);
#endif
}

// How the selection of a (layer, sequence, KV head) group is covered:
//  kDirect:         one work unit per group; the wave writes out/lse.
//  kGlobalPartials: the selection is split over several units; partial
//                   results go to the workspace and a second kernel merges
//                   them.
enum AttnMode { kDirect = 0, kGlobalPartials = 1 };

// Where a unit's K/V rows come from:
//  kKvIndexed: the cache, at the selected token indices (idx);
//  kKvCompact: the compact slot buffers, slots 0 .. count-1;
//  kKvElastic: the slot buffers, except the slots an elastic update has just
//              assigned (src[b][slot] = token >= 0): those rows are read from
//              the cache and written into their slot as they stream through
//              (Sec. 5.4's loads fused into the attention's reads).
enum KvMode { kKvIndexed = 0, kKvCompact = 1, kKvElastic = 2 };

struct AttnArgs {
  const uint16_t* q;      // [n_layers][B][H_q][d]
  const uint16_t* k;      // indexed, elastic: cache; compact: [n_layers][B][k_max][H_kv][d]
  const uint16_t* v;
  const int32_t* idx;     // [B][k_max] (indexed mode)
  uint16_t* kbuf;         // elastic: slot buffers [n_layers][B][k_max][H_kv][d]
  uint16_t* vbuf;
  const int32_t* src;     // elastic: [B][k_max] token loaded into the slot, or -1
  const int32_t* fused;   // elastic: [B] or null; 0: the sequence's rows are all in the slots
  const int32_t* counts;  // [B]
  float* part_acc;        // [n_layers*B][n_split][H_q][d]
  float* part_ml;         // [n_layers*B][n_split][H_q][2]
  float* out;             // [n_layers*B][H_q][d]
  float* lse;             // [n_layers*B][H_q] or null
  int64_t stride_layer;   // elements between layers of the cache (indexed, elastic)
  int64_t stride_b;       // elements between sequences of the cache
  int B, H_q, H_kv, G, k_max, L_cap, n_split, split_tokens, n_items;
  int R;                  // column groups per KV head (1; G/16 for more than 16 query heads)
                          // G above: query heads per column group (at most 16)
  int mode;               // kDirect or kGlobalPartials
  int n_groups, perm;     // work order: group g (G_u = H_kv R consecutive units) runs as group
                          // (g perm) mod n_groups, perm coprime to n_groups
  int n_sets;             // 1: idx [B][k_max]; H_kv: idx [B][H_kv][k_max], one set per KV head
  float scale_log2;       // scale * log2(e)
  int team_heads;         // team kernel: column groups of a workgroup's wavefronts
  int sorted;             // pipelined launches: groups by selection size (see attn_split_kernel)
};

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS row pitch of a staged V tile in bf16: 288 bytes, so that the rows of
// one transpose read start 32 bytes apart and spread over the banks.
constexpr int kVPitch = kD + 16;

__device__ __forceinline__ uint32_t f2bf_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// 8 probabilities -> bf16 hi part and bf16 lo part (p - hi), packed for MFMA.
__device__ __forceinline__ void split_bf16x8(const float* p, bf16x8& hi, bf16x8& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t h0 = f2bf_rne(p[2 * j]), h1 = f2bf_rne(p[2 * j + 1]);
    const uint32_t l0 = f2bf_rne(p[2 * j] - __uint_as_float(h0 << 16));
    const uint32_t l1 = f2bf_rne(p[2 * j + 1] - __uint_as_float(h1 << 16));
    h[j] = h0 | (h1 << 16);
    l[j] = l0 | (l1 << 16);
  }
  hi = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
  lo = __builtin_bit_cast(bf16x8, make_uint4(l[0], l[1], l[2], l[3]));
}

// max / sum over the four lanes {l, l^16, l^32, l^48} (one head's lanes).
__device__ __forceinline__ float xgroup_max(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float xgroup_sum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Transposing LDS read: within each 16-lane group, lane i receives element
// (i & 3) of the 8-byte chunks read by lanes (i >> 2) + 4j, j = 0..3.
__device__ __forceinline__ bf16x4 lds_read_tr(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
      (__attribute__((address_space(3))) bf16x4*)(p));
}

// Rows staged per unit: up to kMaxSplit rows of the selection split plus one
// chunk of padding (the software pipeline reads one chunk past the end when
// no unit follows).
constexpr int kRowsCap = kMaxSplit + kChunk;
constexpr int kRowLoads = kMaxSplit / 64;  // index loads per lane for one unit
// Sequences a launch may rank by selection size (one per thread of the workgroup).
constexpr int kSortMaxB = kWaves * 64;

// One work unit: (layer, sequence, KV-head column group, split).  A group of
// more than 16 query heads is covered by R column groups of 16 (gv = g R ..
// g R + R - 1), each a unit of its own that reads KV head g; the query heads
// of column group gv are gv G .. gv G + G - 1.
struct Unit {
  int lb, b, gv, g, split, j0;
  int n_tok;  // tokens of the unit (<= 0: none), known once the count has arrived
};

__device__ __forceinline__ Unit decode_unit(const AttnArgs& a, int item) {
  Unit u;
  u.gv = item % (a.H_kv * a.R);
  u.g = u.gv / a.R;
  const int rest = item / (a.H_kv * a.R);
  u.split = rest % a.n_split;
  u.lb = rest / a.n_split;  // layer * B + b
  u.b = u.lb % a.B;
  u.j0 = u.split * a.split_tokens;
  u.n_tok = 0;
  return u;
}

// Elastic mode: the staged value of a row is the cache token to read (and
// write into the slot), or -1 - slot for a row read from its slot.  Other
// modes stage the token or slot index clamped into range.
template <int KV>
__device__ __forceinline__ int elastic_row(int v, int slot, int L_cap) {
  if (KV != kKvElastic) return clampi(v, 0, L_cap - 1);
  return v >= 0 ? min(v, L_cap - 1) : -1 - slot;
}
// The row that padding reads (cache hits): row 0, or in elastic mode the unit's
// first token (lane 0's staged value and slot), wherever that lies: its slot
// may be one that this launch has yet to fill, and whatever it holds until then
// would reach the output (0 x NaN).
template <int KV>
__device__ __forceinline__ int pad_row(int v, int slot, int L_cap) {
  return KV == kKvElastic ? elastic_row<KV>(__builtin_amdgcn_readfirstlane(v), slot, L_cap) : 0;
}
template <int KV>
__device__ __forceinline__ const uint16_t* row_ptr(const uint16_t* base, const uint16_t* buf,
                                                   int r, int64_t rs) {
  if (KV != kKvElastic) return base + (int64_t)r * rs;
  return r >= 0 ? base + (int64_t)r * rs : buf + (int64_t)(-1 - r) * rs;
}

// The rows of one chunk that came from the cache, written into their slots
// (dst: the chunk's first slot, this KV head): the data registers as loaded,
// so each slot receives the cache row bit for bit.  n: tokens of the unit
// from this chunk on.
__device__ __forceinline__ void store_k_rows(const int* rc, const uint4 (&kr)[kTiles][4],
                                             uint16_t* dst, int64_t rs, int n, int kg, int r16) {
#pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    const int j = 16 * t + r16;
    if (rc[j] >= 0 && j < n) {
      uint16_t* p = dst + (int64_t)j * rs + 8 * kg;
#pragma unroll
      for (int s = 0; s < 4; ++s) *reinterpret_cast<uint4*>(p + 32 * s) = kr[t][s];
    }
  }
}
__device__ __forceinline__ void store_v_rows(const int* rc, const uint4 (&vr)[kVRows],
                                             uint16_t* dst, int64_t rs, int n, int kg, int r16) {
#pragma unroll
  for (int r = 0; r < kVRows; ++r) {
    const int j = 4 * r + kg;
    if (rc[j] >= 0 && j < n) *reinterpret_cast<uint4*>(dst + (int64_t)j * rs + 8 * r16) = vr[r];
  }
}

// The running maximum before the first logit: below every finite one, and
// finite itself, so that logits of -inf have weight 0 from the first chunk on
// and results over nothing else (this maximum, sum 0) weigh nothing in a merge.
// A whole selection of them is 0 / 0.
constexpr float kNoMax = -FLT_MAX;

// One chunk's online softmax and O^T += V^T P^T.  sacc: its S^T tiles (lane
// holds S[head r16][token 16t + 4kg + i]), c: its first token of the n_tok, V:
// its V tile in LDS, which is no longer read on return.
__device__ __forceinline__ void softmax_pv(const floatx4 (&sacc)[kTiles], const int c,
                                           const int n_tok, const float scale_log2,
                                           const uint16_t* V, const int r16, const int kg,
                                           float& m_run, float& l_run, floatx4 (&acc)[8]) {
  float sv[kTiles][4];
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < kTiles; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool valid = c + 16 * t + 4 * kg + i < n_tok;
      sv[t][i] = valid ? sacc[t][i] * scale_log2 : -INFINITY;
      mx = fmaxf(mx, sv[t][i]);
    }
  mx = xgroup_max(mx);
  const float mn = fmaxf(m_run, mx);
  const float alpha = exp2f(m_run - mn);
  float ls = 0.f;
#pragma unroll
  for (int t = 0; t < kTiles; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sv[t][i] = exp2f(sv[t][i] - mn);
      ls += sv[t][i];
    }
  l_run = l_run * alpha + ls;
  m_run = mn;
#pragma unroll
  for (int db = 0; db < 8; ++db) acc[db] *= alpha;

  // O^T += V^T P^T on the matrix cores.  The k-slots 8kg..8kg+7 of a
  // 32-token block are tokens 4kg..4kg+3 of its first tile and of its
  // second tile: exactly the S^T entries this lane holds.
  wave_sync_lds();
#pragma unroll
  for (int kb2 = 0; kb2 < kChunk / 32; ++kb2) {
    float pv[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pv[i] = sv[2 * kb2][i];
      pv[4 + i] = sv[2 * kb2 + 1][i];
    }
    bf16x8 phi, plo;
    split_bf16x8(pv, phi, plo);
    const uint16_t* r0 = V + (32 * kb2 + 4 * kg + (r16 >> 2)) * kVPitch + 4 * (r16 & 3);
    const uint16_t* r1 = r0 + 16 * kVPitch;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const bf16x4 va = lds_read_tr(r0 + 16 * db);
      const bf16x4 vb4 = lds_read_tr(r1 + 16 * db);
      const bf16x8 vA = __builtin_shufflevector(va, vb4, 0, 1, 2, 3, 4, 5, 6, 7);
      acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vA, phi, acc[db], 0, 0, 0);
      acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vA, plo, acc[db], 0, 0, 0);
    }
  }
  wave_sync_lds();  // the V tile is rewritten by the next chunk
}

// A wavefront's tokens of one (layer, sequence, KV head) group, whose row
// values are staged in `rows`: n_tok tokens, and one chunk of padding after
// the last whole or partial chunk.  Local chunk c / kChunk holds the tokens
// (slots) slot0 + c cstride ..: consecutive chunks (cstride 1), or every
// cstride-th chunk of the selection.  Leaves the running maximum and sum of
// head r16 (the sum not yet added over the four lanes of a head) and the
// accumulators O^T[16db + 4kg + i][head r16].
template <int KV>
__device__ __forceinline__ void attend(const AttnArgs& a, const int lb, const int gv,
                                       const int slot0, const int cstride, const int n_tok,
                                       const int* rows, const bf16x8 (&qf)[4], uint16_t* V,
                                       const int lane, float& m_run, float& l_run,
                                       floatx4 (&acc)[8]) {
  const int b = lb % a.B;
  const int layer = lb / a.B;
  const int g = gv / a.R;
  const int64_t rs = (int64_t)a.H_kv * kD;  // elements per token row
  // kb/vb: the rows a staged row value r >= 0 addresses (the cache, or the
  // slot buffers in compact mode); kbf/vbf: elastic mode's slot buffers, for
  // r < 0 (slot -1 - r).
  const int64_t coff = (int64_t)layer * a.stride_layer + (int64_t)b * a.stride_b + g * kD;
  const int64_t boff = (int64_t)lb * a.k_max * rs + g * kD;
  const uint16_t* kb = a.k + (KV == kKvCompact ? boff : coff);
  const uint16_t* vb = a.v + (KV == kKvCompact ? boff : coff);
  uint16_t* kbf = a.kbuf + boff;
  uint16_t* vbf = a.vbuf + boff;
  const bool writer = KV == kKvElastic && gv % a.R == 0;  // one column group writes the slots
  const int r16 = lane & 15;  // head of this lane (MFMA column); token of a K tile row
  const int kg = lane >> 4;   // MFMA k-group; also the token phase of V loads

  // K rows in the MFMA A-operand layout: tile t, token 16t + r16, dims
  // 32s + 8kg .. +8.  V rows: load r brings token 4r + kg, dims 8 r16 .. +8,
  // i.e. four whole 256-byte rows per instruction.
  auto load_k = [&](int c, uint4 (&kr)[kTiles][4]) {
    const int* rc = rows + c;
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      const uint16_t* p = row_ptr<KV>(kb, kbf, rc[16 * t + r16], rs) + 8 * kg;
#pragma unroll
      for (int s = 0; s < 4; ++s) kr[t][s] = ldkv(p + 32 * s);
    }
  };
  auto load_v = [&](int c, uint4 (&vr)[kVRows]) {
    const int* rc = rows + c;
#pragma unroll
    for (int r = 0; r < kVRows; ++r)
      vr[r] = ldkv(row_ptr<KV>(vb, vbf, rc[4 * r + kg], rs) + 8 * r16);
  };

  m_run = kNoMax;
  l_run = 0.f;
#pragma unroll
  for (int db = 0; db < 8; ++db) acc[db] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Single register buffers, refilled as soon as they are consumed: V(c+1)
  // is requested right after V(c) is staged in LDS, K(c+1) right after the
  // Q.K^T MFMAs have read K(c); both stay in flight through the softmax and
  // the P.V MFMAs of chunk c.  Loads retire in issue order, so each wait is
  // a partial one.  The prefetch past the last chunk reads padding rows
  // (row 0, cache hits).
  uint4 kraw[kTiles][4], vraw[kVRows];
  load_v(0, vraw);
  __builtin_amdgcn_sched_barrier(0);
  load_k(0, kraw);
  __builtin_amdgcn_sched_barrier(0);
  for (int c = 0; c < n_tok; c += kChunk) {
    const int64_t slot = slot0 + (int64_t)c * cstride;  // elastic: the chunk's first slot
#pragma unroll
    for (int r = 0; r < kVRows; ++r)
      *reinterpret_cast<uint4*>(V + (4 * r + kg) * kVPitch + 8 * r16) = vraw[r];
    if (writer) store_v_rows(rows + c, vraw, vbf + slot * rs, rs, n_tok - c, kg, r16);
    load_v(c + kChunk, vraw);
    __builtin_amdgcn_sched_barrier(0);  // keep the refill here: issue order = retire order

    // S^T tiles: lane holds S[head r16][token 16t + 4kg + i].
    floatx4 sacc[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      sacc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        sacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kraw[t][s]),
                                                          qf[s], sacc[t], 0, 0, 0);
    }
    if (writer) store_k_rows(rows + c, kraw, kbf + slot * rs, rs, n_tok - c, kg, r16);
    load_k(c + kChunk, kraw);
    __builtin_amdgcn_sched_barrier(0);

    softmax_pv(sacc, c, n_tok, a.scale_log2, V, r16, kg, m_run, l_run, acc);
  }
}

// B operand of S^T = K Q^T: Q^T column r16 = query head gv*G + r16 (zero if
// >= G), dims 32s + 8kg .. +8.
__device__ __forceinline__ void load_q(const AttnArgs& a, int lb, int gv, int lane,
                                       bf16x8 (&qf)[4]) {
  const int r16 = lane & 15, kg = lane >> 4;
  const uint16_t* qp =
      a.q + ((size_t)lb * a.H_q + gv * a.G + (r16 < a.G ? r16 : 0)) * kD + 8 * kg;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint4 w = r16 < a.G ? ldg16(qp + 32 * s) : make_uint4(0, 0, 0, 0);
    qf[s] = __builtin_bit_cast(bf16x8, w);
  }
}

// One unit from a cold start (a wavefront with a single unit): count, then
// indices staged in LDS, then the first chunk.
template <int KV>
__device__ __forceinline__ void process_item(const AttnArgs& a, const int item, const int lane,
                                             uint16_t* V, int* rows) {
  // A group of more than 16 query heads is covered by R column groups of
  // 16 (gv = g R .. g R + R - 1), each a unit of its own that reads KV head
  // g; the query heads of column group gv are gv G .. gv G + G - 1.
  const int G = a.G;
  const int gv = item % (a.H_kv * a.R);
  const int g = gv / a.R;
  const int rest = item / (a.H_kv * a.R);
  const int split = rest % a.n_split;
  const int lb = rest / a.n_split;  // layer * B + b
  const int b = lb % a.B;
  const int count = __builtin_amdgcn_readfirstlane(clampi(a.counts[b], 0, a.k_max));
  const int j0 = split * a.split_tokens;
  const int r16 = lane & 15;  // head of this lane
  const int kg = lane >> 4;
  if (j0 >= count) {  // uniform per wavefront
    if (a.mode == kDirect && r16 < G) {  // no tokens: out = 0, lse = -inf
      const size_t orow = (size_t)lb * a.H_q + (size_t)gv * G + r16;
      float* dst = a.out + orow * kD + 4 * kg;
#pragma unroll
      for (int db = 0; db < 8; ++db)
        *reinterpret_cast<float4*>(dst + 16 * db) = make_float4(0.f, 0.f, 0.f, 0.f);
      if (a.lse && kg == 0) a.lse[orow] = -INFINITY;
    }
    return;
  }
  const int n_tok = min(a.split_tokens, count - j0);  // tokens of this work item

  bf16x8 qf[4];  // loaded together with the row indices
  load_q(a, lb, gv, lane, qf);

  // Stage the rows of this item's tokens in LDS (masked tokens: the padding
  // row), so that no chunk waits on an index load from memory.
  wave_sync_lds();  // the previous item's reads of rows/V are done
  {
    // All index loads are issued before any is used (one round trip), and
    // one chunk of padding follows the end: the software pipeline always
    // prefetches the next chunk, and its rows are all one (cache hits).
    const int32_t* idx_b =
        KV == kKvIndexed ? a.idx + ((size_t)b * a.n_sets + (a.n_sets > 1 ? g : 0)) * a.k_max + j0
        : KV == kKvElastic ? a.src + (size_t)b * a.k_max + j0
                           : nullptr;
    const bool fz = KV == kKvElastic && (a.fused == nullptr || a.fused[b] != 0);
    const int n_pad = (n_tok + kChunk - 1) / kChunk * kChunk + kChunk;
    constexpr int kColdRowLoads = (kMaxSplit + kChunk + 63) / 64;
    int rv[kColdRowLoads];
#pragma unroll
    for (int m = 0; m < kColdRowLoads; ++m) {
      const int j = lane + 64 * m;
      rv[m] = KV == kKvElastic ? -1 : 0;
      if (j < n_tok && (KV != kKvElastic || fz)) rv[m] = KV == kKvCompact ? j0 + j : idx_b[j];
    }
    const int pad = pad_row<KV>(rv[0], j0, a.L_cap);
#pragma unroll
    for (int m = 0; m < kColdRowLoads; ++m) {
      const int j = lane + 64 * m;
      if (j < n_pad)
        rows[j] = KV == kKvElastic && j >= n_tok ? pad : elastic_row<KV>(rv[m], j0 + j, a.L_cap);
    }
  }
  wave_sync_lds();

  float m_run, l_run;  // head r16
  floatx4 acc[8];      // O^T[16db + 4kg + i][head r16]
  attend<KV>(a, lb, gv, j0, 1, n_tok, rows, qf, V, lane, m_run, l_run, acc);

  l_run = xgroup_sum(l_run);
  if (r16 < G) {
    if (a.mode == kDirect) {  // the whole selection: normalise and write the output
      const size_t orow = (size_t)lb * a.H_q + (size_t)gv * G + r16;
      const float inv = 1.f / l_run;
      float* dst = a.out + orow * kD + 4 * kg;
#pragma unroll
      for (int db = 0; db < 8; ++db)
        *reinterpret_cast<float4*>(dst + 16 * db) =
            make_float4(acc[db][0] * inv, acc[db][1] * inv, acc[db][2] * inv, acc[db][3] * inv);
      if (a.lse && kg == 0) a.lse[orow] = (m_run + log2f(l_run)) * kLn2;
    } else {
      const size_t prow = ((size_t)lb * a.n_split + split) * a.H_q + (size_t)gv * G + r16;
      float* dst = a.part_acc + prow * kD + 4 * kg;
#pragma unroll
      for (int db = 0; db < 8; ++db)
        *reinterpret_cast<float4*>(dst + 16 * db) =
            make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
      if (kg == 0) {
        a.part_ml[prow * 2] = m_run;
        a.part_ml[prow * 2 + 1] = l_run;
      }
    }
  }
}

// Launches with too few groups to give every wavefront of the chip a unit of
// its own (team_plan): a workgroup of W wavefronts works on team_heads (layer,
// sequence, KV head) groups, or on one of n_split parts of them, P = W /
// team_heads wavefronts to each, and merges a group's wavefronts in LDS.
// Such a launch is bound by its chain of round trips and by the ~31 GB/s that
// one CU streams, so what counts is that every CU takes part, that few
// partial results are left, and that the chain is short: chunk c of the
// selection belongs to wavefront c mod (P n_split) of the group, whatever the
// selection's length, so that no index address depends on the count (the
// count, the indices and the queries arrive in one round trip) and a short
// selection divides as evenly as a long one.
constexpr int kTeamRows = 512;  // tokens per wavefront at most

template <int KV, int W>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(W > 4 ? 2 : 1)))
void attn_team_kernel(AttnArgs a) {
  __shared__ __align__(16) uint16_t vlds[W][kChunk * kVPitch];
  __shared__ int rows_lds[W][kTeamRows + kChunk];
  __shared__ float2 ml_lds[W][16];
  // a wavefront's results, once it has no more use for its V tile: 16 heads
  // of 128 floats, 132 apart
  constexpr int kMPitch = kD + 4;
  static_assert(16 * kMPitch * sizeof(float) <= kChunk * kVPitch * sizeof(uint16_t), "merge area");
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int G = a.G;
  const int hb = a.H_kv * a.R / a.team_heads;  // workgroups over the heads
  const int gv0 = blockIdx.x % hb * a.team_heads;
  const int gv = gv0 + wave % a.team_heads;
  const int g = gv / a.R;
  const int rest = blockIdx.x / hb;
  const int split = rest % a.n_split;
  const int lb = rest / a.n_split;  // layer * B + b
  const int b = lb % a.B;
  const int r16 = lane & 15;
  const int kg = lane >> 4;
  const int P = W / a.team_heads;       // wavefronts per head
  const int NW = P * a.n_split;         // wavefronts of the group
  const int gw = split * P + wave / a.team_heads;  // this one
  uint16_t* V = vlds[wave];
  int* rows = rows_lds[wave];

  // count, queries and this wavefront's indices: independent of each other.
  // Lane l of load m holds the token of local row 64 m + l.
  const int cnt_raw = a.counts[b];
  const int fz_raw = KV == kKvElastic && a.fused ? a.fused[b] : 1;
  bf16x8 qf[4];
  load_q(a, lb, gv, lane, qf);
  const int32_t* idx_b =
      KV == kKvIndexed ? a.idx + ((size_t)b * a.n_sets + (a.n_sets > 1 ? g : 0)) * a.k_max
      : KV == kKvElastic ? a.src + (size_t)b * a.k_max
                         : nullptr;
  auto token = [&](int j) { return kChunk * (gw + NW * (j / kChunk)) + j % kChunk; };
  const int most = (a.k_max + kChunk * NW - 1) / (kChunk * NW) * kChunk;  // <= kTeamRows (host)
  constexpr int kLoads = kTeamRows / 64;
  int rv[kLoads];
#pragma unroll
  for (int m = 0; m < kLoads; ++m) {
    // rows past the index row re-read its last entry (one cache line)
    const int t = token(lane + 64 * m);
    rv[m] = 0;
    if (64 * m < most) rv[m] = KV == kKvCompact ? t : idx_b[min(t, a.k_max - 1)];
  }
  const int count = __builtin_amdgcn_readfirstlane(clampi(cnt_raw, 0, a.k_max));
  const bool fz = __builtin_amdgcn_readfirstlane(fz_raw) != 0;
  // this wavefront's tokens: whole chunks, the selection's last one perhaps partial
  const int n_chunks = (count + kChunk - 1) / kChunk;
  const int mine = n_chunks > gw ? (n_chunks - gw + NW - 1) / NW : 0;
  const int n_tok = mine == 0 ? 0
                    : kChunk * mine - ((n_chunks - 1) % NW == gw ? kChunk * n_chunks - count : 0);
  const int pad = pad_row<KV>(fz ? rv[0] : -1, kChunk * gw, a.L_cap);
#pragma unroll
  for (int m = 0; m < kLoads; ++m) {
    const int j = lane + 64 * m;
    if (64 * m < most + kChunk)
      rows[j] = j < n_tok ? elastic_row<KV>(fz ? rv[m] : -1, token(j), a.L_cap) : pad;
  }
  if (lane < kChunk) rows[kTeamRows + lane] = pad;
  wave_sync_lds();

  float m_run = kNoMax, l_run = 0.f;
  floatx4 acc[8];
  if (n_tok > 0) {  // uniform per wavefront
    attend<KV>(a, lb, gv, kChunk * gw, NW, n_tok, rows, qf, V, lane, m_run, l_run, acc);
    l_run = xgroup_sum(l_run);
  } else {
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  float* dst = reinterpret_cast<float*>(V) + r16 * kMPitch + 4 * kg;
#pragma unroll
  for (int db = 0; db < 8; ++db)
    *reinterpret_cast<float4*>(dst + 16 * db) =
        make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
  if (kg == 0) ml_lds[wave][r16] = make_float2(m_run, l_run);
  __syncthreads();
  if (a.mode == kGlobalPartials && split * P >= n_chunks) return;  // no tokens: no partial

  // Merge: thread = (head, 4 dims); the wavefronts' results in order.
  for (int e = threadIdx.x; e < a.team_heads * G * (kD / 4); e += W * 64) {
    const int d4 = e % (kD / 4);
    const int hh = e / (kD / 4);  // query head among the workgroup's
    const int hs = hh / G;        // its column group: wavefronts hs, hs + team_heads, ..
    const int h = hh - hs * G;
    float M = -INFINITY;
    for (int w = hs; w < W; w += a.team_heads) M = fmaxf(M, ml_lds[w][h].x);
    float L = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int w = hs; w < W; w += a.team_heads) {
      const float2 ml = ml_lds[w][h];
      const float f = exp2f(ml.x - M);
      const float4 x =
          reinterpret_cast<const float4*>(reinterpret_cast<const float*>(vlds[w]) + h * kMPitch)[d4];
      L += ml.y * f;
      o.x += x.x * f;
      o.y += x.y * f;
      o.z += x.z * f;
      o.w += x.w * f;
    }
    if (a.mode == kDirect) {
      const size_t orow = (size_t)lb * a.H_q + (size_t)gv0 * G + hh;
      const float inv = count > 0 ? 1.f / L : 0.f;
      reinterpret_cast<float4*>(a.out + orow * kD)[d4] =
          make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
      if (a.lse && d4 == 0) a.lse[orow] = count > 0 ? (M + log2f(L)) * kLn2 : -INFINITY;
    } else {
      const size_t prow = ((size_t)lb * a.n_split + split) * a.H_q + (size_t)gv0 * G + hh;
      reinterpret_cast<float4*>(a.part_acc + prow * kD)[d4] = o;
      if (d4 == 0) reinterpret_cast<float2*>(a.part_ml)[prow] = make_float2(M, L);
    }
  }
}

// Dynamic LDS requested on top of the static arrays so that one workgroup
// takes more than half of a CU's 160 KiB: exactly one per CU.
constexpr size_t kLdsPerCU = 160 * 1024;
constexpr size_t static_lds(bool pipe) {
  return sizeof(uint16_t) * kWaves * kChunk * kVPitch + sizeof(int) * kWaves * (pipe ? 2 : 1) * kRowsCap +
         sizeof(int) * (pipe ? kSortMaxB : 1) + 16;
}
constexpr size_t lds_reserve(bool pipe) {
  return kLdsPerCU / 2 + 1024 > static_lds(pipe) ? kLdsPerCU / 2 + 1024 - static_lds(pipe) : 0;
}

// PIPE: some wavefront has more than one unit, and units are pipelined
// across their boundaries; otherwise each unit starts cold (the pipeline's
// bookkeeping made one-unit launches ~1.5 us slower).
template <int KV, bool PIPE>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(SPEC_ATTN_WPE)))
void attn_split_kernel(AttnArgs a) {
  __shared__ __align__(16) uint16_t vlds[kWaves][kChunk * kVPitch];
  __shared__ int rows_lds[kWaves][PIPE ? 2 : 1][kRowsCap];
  __shared__ int next_unit;
  __shared__ int seq_order[PIPE ? kSortMaxB : 1];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // One workgroup per CU, one wavefront per SIMD.  Two wavefronts on a SIMD
  // do not progress at equal rates (the older one wins instruction issue), and
  // they add no bandwidth over one wavefront with its loads in flight, so the
  // CU runs one per SIMD.  The workgroup owns a contiguous range of the
  // permuted unit order; its wavefronts take them on demand from an LDS
  // counter, which evens out units of unequal length within the workgroup
  // (the permutation evens them out across workgroups).
  //
  // Sorted order (pipelined launches over ragged batches): the sequences are
  // ranked by selection size, longest first, and the (layer, sequence,
  // split) groups in that order are dealt to the workgroups in a snake
  // (row r of gridDim.x groups left to right for even r, right to left for
  // odd r), so that every workgroup receives about the same number of
  // tokens.  The units of one group (its KV heads) stay consecutive.
  // Selections of one size need no sorting: the permuted order is kept.
  bool sorted = false;
  if (PIPE && a.sorted) {
    int* cnt = &rows_lds[0][0][0];  // scratch until the first unit is staged
    const int t = threadIdx.x;      // kWaves * 64 = kSortMaxB >= B threads
    const int c = t < a.B ? clampi(a.counts[t], 0, a.k_max) : -1;
    cnt[t] = c;
    __syncthreads();
    sorted = !__syncthreads_and(t >= a.B || c == cnt[0]);  // uniform for the workgroup
    if (sorted && t < a.B) {
      int r = 0;
      for (int u = 0; u < a.B; ++u) {
        const int cu = cnt[u];
        r += cu > c || (cu == c && u < t);
      }
      seq_order[r] = t;
    }
  }
  const int per_block = (a.n_items + gridDim.x - 1) / gridDim.x;
  const int u0 = sorted ? 0 : blockIdx.x * per_block;
  const int u1 = min(u0 + per_block, a.n_items);
  if (threadIdx.x == 0) next_unit = u0;
  __syncthreads();
  auto take = [&]() -> int {
    int t = 0;
    if (lane == 0) t = atomicAdd(&next_unit, 1);
    const int unit = __builtin_amdgcn_readfirstlane(t);
    const int gu = a.H_kv * a.R;  // units per group (all column groups of one (layer, sequence, split))
    if (sorted) {
      const int row = unit / gu;
      const int col = (row & 1) ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x;
      const int64_t j = (int64_t)row * gridDim.x + col;  // group in size order
      if (j >= a.n_groups) return -1;  // uniform per wave; later rows are past the end too
      const int per_seq = a.n_groups / a.B;  // layers x splits
      const int rank = (int)(j / per_seq);
      const int rem = (int)(j - (int64_t)rank * per_seq);
      const int layer = rem / a.n_split;
      const int split = rem - layer * a.n_split;
      const int lb = layer * a.B + seq_order[rank];
      return (lb * a.n_split + split) * gu + (unit - row * gu);
    }
    if (unit >= u1) return -1;  // uniform per wave
    const int grp = unit / gu;
    return (int)(((int64_t)grp * a.perm) % a.n_groups) * gu + (unit - grp * gu);
  };

  if constexpr (!PIPE) {
    for (;;) {
      const int item = take();
      if (item < 0) return;  // uniform per wave: every wave ends here
      process_item<KV>(a, item, lane, vlds[wave], rows_lds[wave][0]);
    }
  } else {
  uint16_t* V = vlds[wave];
  const int r16 = lane & 15;  // head of this lane (MFMA column); token of a K tile row
  const int kg = lane >> 4;   // MFMA k-group; also the token phase of V loads
  const int64_t rs = (int64_t)a.H_kv * kD;  // elements per token row

  // The rows a staged value r >= 0 addresses (the cache; the slot buffers in
  // compact mode), and elastic mode's slot buffers (r < 0: slot -1 - r).
  auto kv_base = [&](const Unit& u, const uint16_t* p) -> const uint16_t* {
    if (KV != kKvCompact)
      return p + (int64_t)(u.lb / a.B) * a.stride_layer + (int64_t)u.b * a.stride_b + u.g * kD;
    return p + (int64_t)u.lb * a.k_max * rs + u.g * kD;
  };
  auto buf_base = [&](const Unit& u, uint16_t* p) -> uint16_t* {
    return KV == kKvElastic ? p + (int64_t)u.lb * a.k_max * rs + u.g * kD : nullptr;
  };

  // The loads that start a unit, all independent of each other: its count,
  // its row indices (all of a split's, clamped into the index row: the count
  // only masks them later) and its queries.  B operand of S^T = K Q^T: Q^T
  // column r16 = query head gv G + r16 (zero if >= G), dims 32s + 8kg .. +8.
  int cnt_raw, fz_raw = 1;
  int rv[kRowLoads];
  uint4 qraw[4];
  auto fetch = [&](const Unit& u) {
    cnt_raw = a.counts[u.b];
    if (KV == kKvElastic && a.fused) fz_raw = a.fused[u.b];
    const int32_t* idx_b =
        KV == kKvIndexed ? a.idx + ((size_t)u.b * a.n_sets + (a.n_sets > 1 ? u.g : 0)) * a.k_max
        : KV == kKvElastic ? a.src + (size_t)u.b * a.k_max
                           : nullptr;
    // loads past the split re-read its last index (one cache line)
    const int jmax = min(u.j0 + a.split_tokens, a.k_max) - 1;
#pragma unroll
    for (int m = 0; m < kRowLoads; ++m) {
      const int j = u.j0 + lane + 64 * m;
      rv[m] = KV == kKvCompact ? j : idx_b[min(j, jmax)];
    }
    const uint16_t* qp =
        a.q + ((size_t)u.lb * a.H_q + u.gv * a.G + (r16 < a.G ? r16 : 0)) * kD + 8 * kg;
#pragma unroll
    for (int s = 0; s < 4; ++s) qraw[s] = ldg16(qp + 32 * s);
  };
  // Rows of a unit's tokens into LDS; tokens past the unit, and the padding
  // chunk, read the padding row.  Sets u.n_tok.
  auto stage = [&](Unit& u, int* rows) {
    const int count = __builtin_amdgcn_readfirstlane(clampi(cnt_raw, 0, a.k_max));
    u.n_tok = min(a.split_tokens, count - u.j0);
    const bool fz = __builtin_amdgcn_readfirstlane(fz_raw) != 0;  // elastic: rows may come from the caches
    const int pad = pad_row<KV>(fz ? rv[0] : -1, u.j0, a.L_cap);
#pragma unroll
    for (int m = 0; m < kRowLoads; ++m) {
      const int j = lane + 64 * m;
      rows[j] = j < u.n_tok ? elastic_row<KV>(fz ? rv[m] : -1, u.j0 + j, a.L_cap) : pad;
    }
    if (lane < kChunk) rows[kMaxSplit + lane] = pad;
  };

  // K rows in the MFMA A-operand layout: tile t, token 16t + r16, dims
  // 32s + 8kg .. +8.  V rows: load r brings token 4r + kg, dims 8 r16 .. +8,
  // i.e. four whole 256-byte rows per instruction.
  auto load_k = [&](const int* rc, const uint16_t* kb, const uint16_t* kbf,
                    uint4 (&kr)[kTiles][4]) {
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      const uint16_t* p = row_ptr<KV>(kb, kbf, rc[16 * t + r16], rs) + 8 * kg;
#pragma unroll
      for (int s = 0; s < 4; ++s) kr[t][s] = ldkv(p + 32 * s);
    }
  };
  auto load_v = [&](const int* rc, const uint16_t* vb, const uint16_t* vbf, uint4 (&vr)[kVRows]) {
#pragma unroll
    for (int r = 0; r < kVRows; ++r)
      vr[r] = ldkv(row_ptr<KV>(vb, vbf, rc[4 * r + kg], rs) + 8 * r16);
  };

  int buf = 0;
  int item = take();
  if (item < 0) return;
  Unit cur = decode_unit(a, item);
  fetch(cur);
  wave_sync_lds();
  stage(cur, rows_lds[wave][buf]);
  wave_sync_lds();
  uint4 kraw[kTiles][4], vraw[kVRows];
  const uint16_t* kb = kv_base(cur, a.k);
  const uint16_t* vb = kv_base(cur, a.v);
  uint16_t* kbf = buf_base(cur, a.kbuf);
  uint16_t* vbf = buf_base(cur, a.vbuf);
  bf16x8 qf[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    qf[s] = __builtin_bit_cast(bf16x8, r16 < a.G ? qraw[s] : make_uint4(0, 0, 0, 0));
  if (cur.n_tok > 0) {  // uniform per wavefront
    load_v(rows_lds[wave][buf], vb, vbf, vraw);
    __builtin_amdgcn_sched_barrier(0);
    load_k(rows_lds[wave][buf], kb, kbf, kraw);
    __builtin_amdgcn_sched_barrier(0);
  }

  for (;;) {
    // The next unit: its count, indices and queries are requested now and its
    // rows staged before this unit's chunks, so that this unit's last refill
    // can request the next unit's first chunk.
    const int nitem = take();
    Unit nxt = decode_unit(a, nitem < 0 ? 0 : nitem);
    bf16x8 qn[4];
    if (nitem >= 0) {
      fetch(nxt);
      wave_sync_lds();  // the previous unit's reads of this row buffer are done
      stage(nxt, rows_lds[wave][buf ^ 1]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
        qn[s] = __builtin_bit_cast(bf16x8, r16 < a.G ? qraw[s] : make_uint4(0, 0, 0, 0));
    }
    // the next unit's chunk 0 is requested by this unit's last refill
    const bool chain = cur.n_tok > 0 && nitem >= 0 && nxt.n_tok > 0;
    const uint16_t* kbn = kv_base(nxt, a.k);
    const uint16_t* vbn = kv_base(nxt, a.v);
    uint16_t* kbfn = buf_base(nxt, a.kbuf);
    uint16_t* vbfn = buf_base(nxt, a.vbuf);
    const bool writer = KV == kKvElastic && cur.gv % a.R == 0;  // one column group writes
    const int* rows = rows_lds[wave][buf];
    const int* rows_n = rows_lds[wave][buf ^ 1];
    wave_sync_lds();

    const int n_tok = cur.n_tok;
    float m_run = kNoMax, l_run = 0.f;  // head r16
    floatx4 acc[8];                        // O^T[16db + 4kg + i][head r16]
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Single register buffers, refilled as soon as they are consumed: V(c+1)
    // is requested right after V(c) is staged in LDS, K(c+1) right after the
    // Q.K^T MFMAs have read K(c); both stay in flight through the softmax and
    // the P.V MFMAs of chunk c.  Loads retire in issue order, so each wait is
    // a partial one.  After the last chunk the refill requests the next
    // unit's first chunk, or padding rows (cache hits) if none follows.
    for (int c = 0; c < n_tok; c += kChunk) {
      const bool last = c + kChunk >= n_tok;
      const int* rsrc = last && chain ? rows_n : rows + c + kChunk;
      const uint16_t* ksrc = last && chain ? kbn : kb;
      const uint16_t* vsrc = last && chain ? vbn : vb;
      const uint16_t* kfsrc = last && chain ? kbfn : kbf;
      const uint16_t* vfsrc = last && chain ? vbfn : vbf;
#pragma unroll
      for (int r = 0; r < kVRows; ++r)
        *reinterpret_cast<uint4*>(V + (4 * r + kg) * kVPitch + 8 * r16) = vraw[r];
      if (writer)
        store_v_rows(rows + c, vraw, vbf + (int64_t)(cur.j0 + c) * rs, rs, n_tok - c, kg, r16);
      load_v(rsrc, vsrc, vfsrc, vraw);
      __builtin_amdgcn_sched_barrier(0);  // keep the refill here: issue order = retire order

      // S^T tiles: lane holds S[head r16][token 16t + 4kg + i].
      floatx4 sacc[kTiles];
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        sacc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          sacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kraw[t][s]),
                                                            qf[s], sacc[t], 0, 0, 0);
      }
      if (writer)
        store_k_rows(rows + c, kraw, kbf + (int64_t)(cur.j0 + c) * rs, rs, n_tok - c, kg, r16);
      load_k(rsrc, ksrc, kfsrc, kraw);
      __builtin_amdgcn_sched_barrier(0);

      softmax_pv(sacc, c, n_tok, a.scale_log2, V, r16, kg, m_run, l_run, acc);
    }

    // This unit's output: normalised (the whole selection) or a partial.
    // A unit without tokens writes out = 0 and lse = -inf (direct mode); its
    // partials are skipped by the combine.
    const int G = a.G;
    l_run = xgroup_sum(l_run);
    if (r16 < G) {
      if (a.mode == kDirect) {
        const size_t orow = (size_t)cur.lb * a.H_q + (size_t)cur.gv * G + r16;
        const bool any = n_tok > 0;
        const float inv = any ? 1.f / l_run : 0.f;
        float* dst = a.out + orow * kD + 4 * kg;
#pragma unroll
        for (int db = 0; db < 8; ++db)
          *reinterpret_cast<float4*>(dst + 16 * db) =
              make_float4(acc[db][0] * inv, acc[db][1] * inv, acc[db][2] * inv, acc[db][3] * inv);
        if (a.lse && kg == 0) a.lse[orow] = any ? (m_run + log2f(l_run)) * kLn2 : -INFINITY;
      } else if (n_tok > 0) {
        const size_t prow = ((size_t)cur.lb * a.n_split + cur.split) * a.H_q + (size_t)cur.gv * G + r16;
        float* dst = a.part_acc + prow * kD + 4 * kg;
#pragma unroll
        for (int db = 0; db < 8; ++db)
          *reinterpret_cast<float4*>(dst + 16 * db) =
              make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
        if (kg == 0) {
          a.part_ml[prow * 2] = m_run;
          a.part_ml[prow * 2 + 1] = l_run;
        }
      }
    }

    if (nitem < 0) break;
    cur = nxt;
    kb = kbn;
    vb = vbn;
    kbf = kbfn;
    vbf = vbfn;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = qn[s];
    if (!chain && cur.n_tok > 0) {  // not chained (this unit had no tokens): start it cold
      load_v(rows_n, vb, vbf, vraw);
      __builtin_amdgcn_sched_barrier(0);
      load_k(rows_n, kb, kbf, kraw);
      __builtin_amdgcn_sched_barrier(0);
    }
    buf ^= 1;
  }
  }
}

struct CombineArgs {
  const float* part_acc;
  const float* part_ml;
  const int32_t* counts;
  float* out;  // [n_layers*B][H_q][d]
  float* lse;  // [n_layers*B][H_q] or null
  int B, H_q, k_max, n_split, split_tokens;
};

// One workgroup per (layer*B + b, 8 / S heads); thread = (head, part, 4 dims).
// A thread's splits (part, part + S, ..) have their (max, sum) pairs and
// accumulator slices requested eight at a time, all before any is used: one
// round trip for up to 8 S splits.  S > 1: the S results of a head are merged
// in LDS.
template <int S>
__global__ __launch_bounds__(256) void attn_combine_kernel(CombineArgs a) {
  constexpr int kBatch = 8;
  __shared__ float2 ml_lds[S > 1 ? 8 : 1];
  __shared__ float4 acc_lds[S > 1 ? 8 : 1][32];
  const int lb = blockIdx.x;
  const int slot = threadIdx.x >> 5;
  const int h = blockIdx.y * (8 / S) + slot / S;
  const int part = slot % S;
  const int d4 = threadIdx.x & 31;
  if (S == 1 && h >= a.H_q) return;
  const int b = lb % a.B;
  const int count = clampi(a.counts[b], 0, a.k_max);
  const int ns = min(a.n_split, (count + a.split_tokens - 1) / a.split_tokens);
  float4* o = reinterpret_cast<float4*>(a.out + ((size_t)lb * a.H_q + h) * kD) + d4;
  if (ns == 0) {  // uniform per workgroup
    if (h < a.H_q && part == 0) {
      *o = make_float4(0.f, 0.f, 0.f, 0.f);
      if (a.lse && d4 == 0) a.lse[(size_t)lb * a.H_q + h] = -INFINITY;
    }
    return;
  }
  const size_t base = (size_t)lb * a.n_split * a.H_q + min(h, a.H_q - 1);  // row of split 0
  const float2* ml2 = reinterpret_cast<const float2*>(a.part_ml);
  float M = -INFINITY, L = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = part; s0 < ns; s0 += kBatch * S) {
    float2 ml[kBatch];
    float4 pa[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {  // clamped: every load is issued
      const size_t row = base + (size_t)min(s0 + u * S, ns - 1) * a.H_q;
      ml[u] = ml2[row];
      pa[u] = reinterpret_cast<const float4*>(a.part_acc + row * kD)[d4];
    }
    float Mb = M;
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (s0 + u * S < ns) Mb = fmaxf(Mb, ml[u].x);
    const float r = exp2f(M - Mb);  // earlier batches onto the new maximum (0 at the first)
    L *= r;
    acc.x *= r;
    acc.y *= r;
    acc.z *= r;
    acc.w *= r;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (s0 + u * S < ns) {
        const float w = exp2f(ml[u].x - Mb);
        L += ml[u].y * w;
        acc.x += pa[u].x * w;
        acc.y += pa[u].y * w;
        acc.z += pa[u].z * w;
        acc.w += pa[u].w * w;
      }
    }
    M = Mb;
  }
  if (S > 1) {
    if (d4 == 0) ml_lds[slot] = make_float2(M, L);
    acc_lds[slot][d4] = acc;
    __syncthreads();
    if (part != 0 || h >= a.H_q) return;
    const int parts = min(S, ns);  // parts with a split
    for (int p = 1; p < parts; ++p) M = fmaxf(M, ml_lds[slot + p].x);
    const float r = exp2f(ml_lds[slot].x - M);
    L *= r;
    acc.x *= r;
    acc.y *= r;
    acc.z *= r;
    acc.w *= r;
    for (int p = 1; p < parts; ++p) {
      const float w = exp2f(ml_lds[slot + p].x - M);
      const float4 x = acc_lds[slot + p][d4];
      L += ml_lds[slot + p].y * w;
      acc.x += x.x * w;
      acc.y += x.y * w;
      acc.z += x.z * w;
      acc.w += x.w * w;
    }
  }
  const float inv = 1.f / L;
  *o = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  if (a.lse && d4 == 0) a.lse[(size_t)lb * a.H_q + h] = (M + log2f(L)) * kLn2;
}

// Resident wavefront slots the work is sized for: one per SIMD on 256 CUs.
constexpr int64_t kWaveSlots = (int64_t)kWaves * kCUs;

struct AttnPlan {
  int mode, n_split, split;
  int team;  // wavefronts of a workgroup that share a unit (attn_team_kernel), or 0
  int team_heads;  // column groups those wavefronts cover: team / team_heads of them each
};

// Work units are (layer, sequence, KV head, split of the selection).  With at
// least one (layer, sequence, KV head) group per wavefront slot there is no
// split and each unit writes its output (kDirect).  With fewer groups the
// selections are split until there is about one unit per slot, but not below
// kMinSplitTokens (each unit pays a start-up latency and a partial-result
// store) nor above kMaxSplit (the index staging area) (kGlobalPartials).
// Units are numbered KV head fastest, so that the wavefronts of a workgroup
// read the same selected tokens' rows for neighbouring heads at the same time:
// those pieces share DRAM pages.  A split is a whole number of chunks.
// Column groups of at most 16 query heads per KV head.
int attn_col_groups(const Dims& d) { return d.G > 16 ? d.G / 16 : 1; }

// Launches of at most 512 groups, which leave the chip short of units: a
// workgroup of several wavefronts per unit (attn_team_kernel).  Either a group
// is one workgroup's, which writes the output (no combine: ~3.5 us), or the
// selections are split over as many four-wavefront workgroups as CUs.  The
// choice follows a cost fitted to launches of 8 to 256 workgroups: a CU
// streams its tokens at ~0.017 us each when few CUs stream, ~0.025 us when all
// do.  Two heads per workgroup read neighbouring pieces of the same rows
// (2-4% faster on splits of at least 64 groups; 128 groups, k = 2048: 32.2 ->
// 30.0 us); fewer, larger partials are better below that, unless the two read
// the same rows (more than 16 query heads per KV head) and there are 300 tokens
// per CU: 60 groups, k = 1750 20.5 -> 19.1, 28 groups, k = 6000 25.0 -> 23.1,
// but 24 groups, k = 1000 12.1 -> 12.5.  us per launch in a
// HIP graph, one wavefront per unit -> this plan, one layer, 32 query heads, 8
// KV heads:
//   1 x k=128 8.8 -> 5.7, 1 x k=512 9.3 -> 8.4, 9 x k=321 14.6 -> 8.4,
//   1 x k=4096 (64 query heads) 15.7 -> 10.0, 8 x k=2048 17.9 -> 17.5,
//   60 x k=300 27.2 -> 18.3, 50 ragged, k=1200 50.8 -> 43.6;
//   61 ragged, k=1500, 4 KV heads 42.1 -> 34.2; 24 layers x 2 ragged, k=1000 44.1 -> 32.6.
//
// One wavefront per unit stays better
//  - with more than 512 groups, and for short selections of 256 groups or more
//    (four chunks per wavefront);
//  - where its units, of full length, just fill the wavefronts and the
//    selections are equal or per head: 256 groups, k = 4096 94.7 against 102.9
//    us, per-head sets of 160 groups, k = 1536, in a step 26.1 against 26.6.
//    (Ragged selections shared by the heads would gain: 160 groups, k = 1536
//    24.5 -> 22.1; equal ones are within 2%.  Units of which many are short do
//    not fill them: 480 to 512 groups, k = 260 to 400, are the 24 to 29 us that
//    this plan does in 15 to 23.);
//  - where it puts several units on every CU while this plan leaves CUs idle,
//    or has a selection too long for the splits that would fill them: 136
//    groups, k = 4096, direct 63.2 against 84.2 us; 144 groups, k = 1000, direct
//    22.2 against 25.7; 96 groups, k = 2048, 5 splits 22.6 against 24.1.  That
//    is decided by a second estimate, which counts what a launch takes besides
//    streaming.  Of 1800 one-layer launches (1 to 124 sequences, 2 to 8 KV heads,
//    k = 100 to 6000, equal and ragged, rows not in the caches) it leaves 29
//    more than 3% slower than with one wavefront per unit throughout (at most
//    7%: 48 to 56 groups, k = 2048, and 8 to 24 groups, k = 300 of equal length,
//    whose ragged ones gain as much), against 142 (up to 31%) without.
// wave: the plan with one wavefront per unit (wave_plan).
bool team_plan(const Dims& d, int64_t groups, const AttnPlan& wave, AttnPlan* p) {
  const int gu = d.H_kv * attn_col_groups(d);
  const int64_t units = groups * wave.n_split;
  if (units <= kWaveSlots && units >= kWaveSlots / 16 * 15 &&
      10 * (int64_t)d.k_max >= 9 * (int64_t)wave.n_split * wave.split)
    return false;
  if (groups >= kCUs && d.k_max <= 4 * kChunk) return false;
  auto cost = [](int64_t wgs, int64_t tokens) { return tokens * (0.017 + 3e-5 * wgs); };
  auto time = [](double base, int64_t wgs, int64_t tokens) {
    return base + tokens * (0.0125 + 3e-5 * wgs);
  };
  double best = 1e30, est = 0;
  // direct: one workgroup per group, or per two where they fill the CUs
  const int dh = groups <= kCUs ? 1 : 2;  // heads per workgroup
  const int64_t dw = groups / dh;
  const int W = (int64_t)d.k_max * dh >= 512 ? 8 : 4;
  if (gu % dh == 0 && dw <= kCUs && (dh == 1 || dw >= 3 * kCUs / 4) &&
      W / dh * kTeamRows >= d.k_max) {
    best = cost(dw, (int64_t)d.k_max * dh);
    est = time(dh == 1 && attn_col_groups(d) == 1 ? 7 : 6, dw, (int64_t)d.k_max * dh);
    *p = {kDirect, 1, 0, W, dh};
  }
  // split: parts of at least a chunk per wavefront
  const bool same_rows = attn_col_groups(d) > 1 && groups * d.k_max >= 300 * kCUs;
  const int sh = gu % 2 == 0 && (groups >= 64 || same_rows) ? 2 : 1;
  const int P = 4 / sh;
  const int64_t chunks = (d.k_max + kChunk - 1) / kChunk;
  int64_t ns = kCUs * sh / groups;
  if (ns > (chunks + P - 1) / P) ns = (chunks + P - 1) / P;
  if (ns >= 2 && ns * P * kTeamRows >= d.k_max) {
    const int64_t tok = ((chunks + ns * P - 1) / (ns * P)) * P * kChunk;
    const double c = 3.5 + cost(groups / sh * ns, tok * sh);
    if (c < best) {
      best = c;
      est = time(7, groups / sh * ns, tok * sh);
      *p = {kGlobalPartials, (int)ns, kChunk * P, 4, sh};
    }
  }
  // one wavefront per unit, several of them on every CU
  const int64_t per_cu = (units + kCUs - 1) / kCUs;
  if (per_cu >= 2 && wave.n_split > 1 &&
      time(units <= kWaveSlots ? 8 : 13, (units + per_cu - 1) / per_cu, per_cu * wave.split) < est)
    return false;
  return best < 1e30;
}

// One wavefront per unit.  A launch whose units of kMinSplitTokens would not
// reach one per four CUs (a single short layer) may go down to 64 tokens.
AttnPlan wave_plan(const Dims& d, int64_t groups) {
  auto round_chunk = [](int64_t t) { return (t + kChunk - 1) / kChunk * kChunk; };
  const bool small = groups * ((d.k_max + kMinSplitTokens - 1) / kMinSplitTokens) < kCUs / 4;
  const int64_t least = small ? 64 : kMinSplitTokens;
  int64_t n_split = (kWaveSlots * kSlotUnits + groups - 1) / groups;
  int64_t split = round_chunk((d.k_max + n_split - 1) / n_split);
  if (split < least) split = least;
  if (split > kMaxSplit) split = kMaxSplit;
  n_split = (d.k_max + split - 1) / split;
  if (n_split == 1) return {kDirect, 1, (int)round_chunk(d.k_max), 0, 1};
  return {kGlobalPartials, (int)n_split, (int)split, 0, 1};
}

AttnPlan attn_plan(const Dims& d) {
  const int64_t groups = (int64_t)d.n_layers * d.B * d.H_kv * attn_col_groups(d);
  const AttnPlan wave = wave_plan(d, groups);
  AttnPlan team;
  return !d.plain && team_plan(d, groups, wave, &team) ? team : wave;
}

}  // namespace

int device_cu_count() {
  static const int n = [] {
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n_cu <= 0)
      n_cu = 256;
    return n_cu;
  }();
  return n;
}

// The larger of what the plan and the plain one (one wavefront per unit) take.
size_t attn_ws_bytes(const Dims& d) {
  Dims plain = d;
  plain.plain = true;
  size_t most = 0;
  for (const Dims* e : {&d, (const Dims*)&plain}) {
    const AttnPlan p = attn_plan(*e);
    const size_t rows = (size_t)d.n_layers * d.B * p.n_split * d.H_q;
    const size_t n = p.mode == kGlobalPartials ? align_up(sizeof(float) * rows * d.d) +
                                                     align_up(sizeof(float) * rows * 2)
                                               : 0;
    if (n > most) most = n;
  }
  return most;
}

namespace {

template <int KV>
void launch_split(dim3 grid, bool pipe, const AttnArgs& a, hipStream_t s) {
  if (pipe)
    attn_split_kernel<KV, true><<<grid, kWaves * 64, lds_reserve(true), s>>>(a);
  else
    attn_split_kernel<KV, false><<<grid, kWaves * 64, lds_reserve(false), s>>>(a);
}

template <int W>
void launch_team_w(int kv, dim3 grid, const AttnArgs& a, hipStream_t s) {
  if (kv == kKvIndexed) attn_team_kernel<kKvIndexed, W><<<grid, W * 64, 0, s>>>(a);
  else if (kv == kKvCompact) attn_team_kernel<kKvCompact, W><<<grid, W * 64, 0, s>>>(a);
  else attn_team_kernel<kKvElastic, W><<<grid, W * 64, 0, s>>>(a);
}
void launch_team(int kv, int W, dim3 grid, const AttnArgs& a, hipStream_t s) {
  if (W == 4) launch_team_w<4>(kv, grid, a, s);
  else launch_team_w<8>(kv, grid, a, s);
}

// Merges the partial results of split selections (a direct launch has none).
hipError_t launch_combine(const Dims& d, const AttnPlan& pl, const float* part_acc,
                          const float* part_ml, const int32_t* counts, float* out, float* lse,
                          hipStream_t s) {
  if (pl.mode != kGlobalPartials) return hipGetLastError();
  CombineArgs c{part_acc, part_ml, counts, out, lse, d.B, d.H_q, d.k_max, pl.n_split, pl.split};
  const unsigned lb = (unsigned)(d.n_layers * d.B);
  auto heads = [&](int per) { return dim3(lb, (unsigned)((d.H_q + per - 1) / per)); };
  if (pl.n_split <= 8) attn_combine_kernel<1><<<heads(8), 256, 0, s>>>(c);
  else if (pl.n_split <= 16) attn_combine_kernel<2><<<heads(4), 256, 0, s>>>(c);
  else if (pl.n_split <= 32) attn_combine_kernel<4><<<heads(2), 256, 0, s>>>(c);
  else attn_combine_kernel<8><<<heads(1), 256, 0, s>>>(c);
  return hipGetLastError();
}

hipError_t launch_attn_mode(const Dims& d, int kv, const uint16_t* q, const uint16_t* k,
                            const uint16_t* v, const int32_t* idx, uint16_t* kbuf,
                            uint16_t* vbuf, const int32_t* src, const int32_t* fused,
                            const int32_t* counts, float* out, float* lse, void* ws,
                            hipStream_t s) {
  const AttnPlan pl = attn_plan(d);
  // the row staging area holds one split plus a chunk of padding
  if (pl.split > kMaxSplit || pl.split % kChunk != 0) return hipErrorInvalidValue;
  const size_t rows = (size_t)d.n_layers * d.B * pl.n_split * d.H_q;
  float* part_acc = static_cast<float*>(ws);
  float* part_ml = pl.mode == kGlobalPartials
                       ? reinterpret_cast<float*>(static_cast<char*>(ws) +
                                                  align_up(sizeof(float) * rows * d.d))
                       : nullptr;
  const int R = attn_col_groups(d);
  const int64_t n_groups = (int64_t)d.n_layers * d.B * d.H_kv * R;
  const int64_t n_items = n_groups * pl.n_split;
  if (n_items > INT32_MAX / 2) return hipErrorInvalidValue;
  // Work order: the ranges of consecutive units the workgroups own are spread
  // over all (layer, sequence, split) groups by a multiplicative permutation,
  // so that ragged selections even out across workgroups.
  const int n_order = (int)(n_items / (d.H_kv * R));  // (layer, sequence, split) groups
  int perm = 1;
  if (n_order > 2) {
    perm = (int)(0.618 * n_order);
    auto gcd = [](int x, int y) { while (y) { const int t = x % y; x = y; y = t; } return x; };
    while (gcd(perm, n_order) != 1) ++perm;
  }
  AttnArgs a{q, k, v, idx, kbuf, vbuf, src, fused, counts, part_acc, part_ml, out, lse,
             d.kv_stride_layer, d.kv_stride_b, d.B, d.H_q, d.H_kv, d.G / R, d.k_max, d.L_cap,
             pl.n_split, pl.split, (int)n_items, R, pl.mode, n_order, perm, d.n_sets,
             d.scale * kLog2e, pl.team_heads, 0};
  // One workgroup per CU, fewer only when there are fewer units than CUs:
  // with few units they are spread over all CUs (each CU's share of the
  // bandwidth is limited) rather than packed four to a CU.
  if (pl.team) {
    launch_team(kv, pl.team, dim3((unsigned)(n_items / pl.team_heads)), a, s);
    return launch_combine(d, pl, part_acc, part_ml, counts, out, lse, s);
  }
  const int n_cu = device_cu_count();
  const dim3 grid((unsigned)(n_items < n_cu ? n_items : n_cu));
  // SPEC_ATTN_SCHEDULE=cold runs every unit from a cold start even where a
  // wavefront takes several (the tests compare both schedules bit for bit).
  const char* sched = getenv("SPEC_ATTN_SCHEDULE");
  const bool force_cold = sched && strcmp(sched, "cold") == 0;
  // some wavefront takes several units: pipeline them
  const bool pipe = !force_cold && n_items > (int64_t)grid.x * kWaves;
  // Sorted order: pipelined, at most one sequence per thread of a workgroup
  // to rank, and at least two groups per workgroup.  SPEC_ATTN_ORDER=perm
  // keeps the permuted order (the tests compare both orders bit for bit).
  const char* order = getenv("SPEC_ATTN_ORDER");
  const bool want_sorted = !(order && strcmp(order, "perm") == 0);
  a.sorted = pipe && want_sorted && d.B <= kSortMaxB && n_order >= 2 * (int64_t)grid.x;
  if (kv == kKvIndexed)
    launch_split<kKvIndexed>(grid, pipe, a, s);
  else if (kv == kKvCompact)
    launch_split<kKvCompact>(grid, pipe, a, s);
  else
    launch_split<kKvElastic>(grid, pipe, a, s);
  return launch_combine(d, pl, part_acc, part_ml, counts, out, lse, s);
}

}  // namespace

hipError_t launch_attn(const Dims& d, const uint16_t* q, const uint16_t* k,
                       const uint16_t* v, const int32_t* idx, const int32_t* counts,
                       float* out, float* lse, void* ws, hipStream_t s) {
  return launch_attn_mode(d, idx ? kKvIndexed : kKvCompact, q, k, v, idx, nullptr, nullptr,
                          nullptr, nullptr, counts, out, lse, ws, s);
}

hipError_t launch_attn_elastic(const Dims& d, const uint16_t* q, const uint16_t* k_cache,
                               const uint16_t* v_cache, uint16_t* kbuf, uint16_t* vbuf,
                               const int32_t* slot_src, const int32_t* counts, float* out,
                               float* lse, void* ws, hipStream_t s, const int32_t* fused) {
  return launch_attn_mode(d, kKvElastic, q, k_cache, v_cache, nullptr, kbuf, vbuf, slot_src,
                          fused, counts, out, lse, ws, s);
}

}  // namespace spec
