// DMS-masked chunked prefill attention, gfx950.
//
// Query at position t of a chunk [p0, p0 + C) attends to key j iff j <= t and
// (j > t - w or key j is kept) -- the binary mask of Fig. 1b (Sec. 3.1), passed
// as the per-token decision vector and never materialised (Sec. 3.1
// "Performance Considerations"); the sparsity it creates is used to skip work
// (Sec. 3.2).  For a block of queries [t0, t1) keys come from three places:
//   1. the cache: the L0 live slots of the head before the chunk; all of them
//      are visible except flagged tokens of the last w positions, which expire
//      inside the chunk by the same rule (slot_meta holds owner position and
//      flag);
//   2. kept chunk keys before the band -- visible to every query of the
//      block; flagged ones there are hidden from all of them and skipped;
//   3. the band: the chunk tiles from the one holding max(p0, t0 - w + 1) to
//      t1, masked per element.
//
// Pass 0 (chunk_scan_kernel) lists the kept chunk tokens; pass 1 copies the chunk's keys and
// values, in chunk order and in kept order, into workspace tiles in the
// pool's tile layout (16-byte pieces in the decode MFMAs' fragment order:
// keys by (k-step, half, lane), values transposed), so the attention pass
// stages every source the same way.
//
// Attention pass: a work item is one (sequence, KV head, block of query
// positions).  Its columns are (position, query head) pairs, the g heads of a
// position consecutive, packed to the MFMA column blocks (a position's heads
// may straddle two): 32 per wave under delayed eviction, NQ blocks of 16 per
// wave under immediate eviction.  Key tiles are staged into LDS in the order
// the MFMA operand loads consume them (no bank conflicts) -- by hardware
// copies for bf16 pages under delayed eviction, through registers otherwise --
// and read by every wave with 16-byte LDS loads straight into operand
// registers.  A tile is masked per element only when some query of the block
// does not see one of its keys; the online softmax works in the exp2 domain
// with a lazy rescale.  Pass 0 also counts the kept chunk tokens before every
// 32-aligned position and the first block of pass 1 ranks the call's (sequence,
// head) rows by work; the attention launch keeps as many workgroups as fit on the
// chip, each taking (row, query block) items in that order.
#include <type_traits>

#include "dms_common.h"
#include "dms_fp8.h"

namespace dms {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kThreads = 256;
// Attention pass workgroup: eight waves for FP8 pages at d = 128 (one
// workgroup per CU, two waves per SIMD), else four.  Each of a chunk's query
// blocks stages every cached tile of its head, so more waves per workgroup
// means fewer stagings per query: with FP8 pages a staging dequantizes the
// tile; with bf16 pages it is a hardware copy, and more waves wait at every
// barrier.
template <int D, bool FP8>
constexpr int attn_threads() { return FP8 && D == 128 ? 512 : 256; }
constexpr uint32_t kNoKey = 0x7FFFFFFFu;  // key position of padding rows (never visible)
constexpr float kRescale = 8.0f;          // lazy rescale threshold, log2 units
constexpr float kMInit = -1.0e30f;        // running max before the first visible key

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// LDS tile layout.  A wave's MFMA operand load -- lane (r, G) = (lane % 16,
// lane / 16) takes 16 bytes -- is free of bank conflicts when the 64 lanes
// read one contiguous 1 KB block in lane order (measured on gfx950; rows of
// 64 bytes read column-wise are not).  The pool's tile layout is already in
// that order (dms_common.h): keys as 1 KB blocks per (32-dim slice, score
// MFMA row set), values (V^T) as 1 KB blocks per 16 dims, lane-ordered pieces
// inside each.  So staging copies a tile's 16-byte piece P to LDS slot P.

// max over the four lanes r, r + 16, r + 32, r + 48 (the key rows of one column)
__device__ inline float col_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ inline int load_status(const int32_t* status) {
  return __atomic_load_n(status, __ATOMIC_RELAXED);
}

__device__ inline f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Attention grid row: call head, first token and length of its chunk, state
// head, position and live length before the chunk, first workspace tile.
struct __attribute__((aligned(32))) PrefillRow {
  int hh, tok0, C, sh, p0, L0, tile0, pad;
};

struct PrefillArgs {
  const int32_t* status;
  const int32_t* seq_ids;
  const int32_t* cu;
  const uint16_t* q;      // [T, Hq, D]
  const uint16_t* k;      // [T, H, D]
  const uint16_t* v;      // [T, H, D]
  const uint8_t* flags;   // [T, H]
  const char* pool;
  const int32_t* page_table;
  const int32_t* slot_meta;
  const int32_t* len;
  const int32_t* pos;
  int32_t* list;          // [H][total]: chunk-local indices of kept tokens
  int32_t* list_cnt;      // [n * H]
  int32_t* kept_before;   // [H][tph]: kept chunk tokens before chunk position 32 j (tile indexing)
  PrefillRow* rows;       // [n * H]: attention grid rows, heaviest first
  int32_t* first_item;    // [n * H + 1]: first work item of each row (n * H <= kOrderMax)
  int32_t* work_ctr;      // attention work items taken so far (zeroed by pass 0)
  int nx, items;          // query blocks per grid row; rows x nx
  char* tiles;            // [2][H][tph] tiles: chunk tokens, then compacted kept tokens
  uint32_t* tmeta;        // [2][H][tph][32]: key rows of those tiles (position | flag << 31)
  char* zeros;            // values of one tile, all 0 (bf16 pages)
  float* out;             // [T, Hq, D]
  size_t page_bytes;
  int n, H, g, w, P, log2P, maxp, max_slots, max_seqs, total, max_len, PB, tph;
  int order;        // 1: the first blocks of pass 1 order the rows
  int immediate;    // eviction timing: key j is hidden by the decision of j + w
  int zero_neuron;  // element 0 of each group's first query head is read as 0
  float scale_log2;
};

// Decision that hides chunk key c (chunk-local) once it leaves the window:
// its own (delayed eviction) or that of chunk token c + w (immediate
// eviction; none yet if c + w is past the chunk).
__device__ inline bool key_flag(const PrefillArgs& a, int tok0, int C, int c, int h) {
  const int x = a.immediate ? c + a.w : c;
  return x < C && a.flags[static_cast<size_t>(tok0 + x) * a.H + h] != 0;
}

// Decisions from the borrowed query neuron (Sec. 3.2 rounding, App. C):
// flags[t][h] = (bf16 q[t][h * g][0] + bias > 0) in float32.
__global__ __launch_bounds__(kThreads) void prefill_decide_kernel(const uint16_t* q, uint8_t* flags,
                                                                  int total, int H, int g, int D,
                                                                  float bias) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(total) * H) return;
  const uint32_t bits = q[static_cast<size_t>(idx) * g * D];
  flags[idx] = (__uint_as_float(bits << 16) + bias) > 0.f;
}

__device__ inline size_t ws_tile(const PrefillArgs& a, int region, int h, int i, int k) {
  return ((static_cast<size_t>(region) * a.H + h) * a.tph + a.cu[i] / 32 + i + k);
}
// kept_before entry of chunk position 32 j of sequence i, head h
__device__ inline size_t ws_kb(const PrefillArgs& a, int h, int i, int j) {
  return static_cast<size_t>(h) * a.tph + a.cu[i] / 32 + i + j;
}

// Attention grid rows by decreasing work (rows are dispatched in order, so
// the longest heads start first and the short ones fill the tail): one
// workgroup ranks the n * H (sequence, head) rows by their live length plus
// half their kept chunk tokens (the cached keys every block of the row
// attends to, and the mean of its kept-prefix keys); ties keep row order, and
// calls of more than kOrderMax rows keep theirs.  It also writes each row's
// descriptor (which saves a work item three dependent loads) and first work
// item, so that rows of shorter chunks have no empty items.  Like pass 1 it
// needs nothing but pass 0's results, so it runs as the first blocks of that
// launch (`part`: one of every 256 unranked rows, one in all of ranked ones): a
// launch of its own took 3.4 to 6.2 us a chunk.
constexpr int kOrderMax = 512;
__device__ __forceinline__ void order_rows(const PrefillArgs& a, int part) {
  __shared__ int work[kOrderMax], blocks[kOrderMax], lds[17];
  const int NH = a.n * a.H;
  const bool ranked = NH <= kOrderMax;
  if (ranked && part > 0) return;
  if (ranked)
    for (int x = threadIdx.x; x < kOrderMax; x += kThreads) {
      work[x] = x < NH ? a.len[a.seq_ids[x / a.H] * a.H + x % a.H] + a.list_cnt[x] / 2 : 0;
      blocks[x] = 0;
    }
  __syncthreads();
  const int end = ranked ? NH : min(NH, (part + 1) * kThreads);
  for (int x = part * kThreads + threadIdx.x; x < end; x += kThreads) {
    int rank = x;
    if (ranked) {
      rank = 0;
      const int wx = work[x];
      for (int y = 0; y < NH; ++y) rank += work[y] > wx || (work[y] == wx && y < x);
    }
    const int i = x / a.H, s = a.seq_ids[i], sh = s * a.H + x % a.H, tok0 = a.cu[i];
    PrefillRow r;
    r.hh = x;
    r.tok0 = tok0;
    r.C = a.cu[i + 1] - tok0;
    r.sh = sh;
    r.p0 = a.pos[s];
    r.L0 = a.len[sh];
    r.tile0 = tok0 / 32 + i;
    r.pad = 0;
    a.rows[rank] = r;
    if (ranked) blocks[rank] = (r.C + a.PB - 1) / a.PB;
  }
  if (!ranked) return;
  // first work item of every row
  __syncthreads();
  constexpr int kPer = kOrderMax / kThreads;
  int mine = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) mine += blocks[kPer * threadIdx.x + u];
  int total;
  int at = block_exclusive_scan(mine, lds, &total);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int x = kPer * threadIdx.x + u;
    if (x < NH) a.first_item[x] = at;
    at += blocks[x];
  }
  if (threadIdx.x == 0) a.first_item[NH] = total;
}

// Pass 1 (one block per (32-token tile, sequence x head, region), after those
// that order the rows): copy the
// chunk's keys and values -- region 0: in chunk order; region 1: the kept
// tokens in list order -- into workspace tiles in the pool's tile layout
// (fragment order, values transposed); rows past the end are 0.
template <int D, bool FP8>
__global__ __launch_bounds__(kThreads) void prefill_tile_kernel(PrefillArgs a) {
  __shared__ uint16_t vrows[32][D + 2];
  if (load_status(a.status) != 0) return;
  const int k = blockIdx.x - a.order, hh = blockIdx.y, region = blockIdx.z;
  if (k < 0) {
    if (region == 0) order_rows(a, hh);
    return;
  }
  if (!FP8 && k == 0 && hh == 0 && region == 1)
    for (int x = threadIdx.x; x < D * 4; x += kThreads) reinterpret_cast<u32x4*>(a.zeros)[x] = u32x4{0u, 0u, 0u, 0u};
  const int i = hh / a.H, h = hh % a.H;
  const int tok0 = a.cu[i], C = a.cu[i + 1] - a.cu[i];
  const int cnt = region ? a.list_cnt[hh] : C;
  if (k * 32 >= cnt) return;
  const int32_t* lst = a.list + static_cast<size_t>(h) * a.total + tok0;
  const int tid = threadIdx.x;
  constexpr int kPieces = 32 * D / 8;   // 16-byte pieces of 32 rows
  if (tid < 32) {
    // the tile's key rows as the pool's slot metadata has them: position |
    // flag << 31 (kept-list rows carry no flag); rows past the end: no key
    const int idx = 32 * k + tid;
    const int p0 = a.pos[a.seq_ids[i]];
    uint32_t mt = kNoKey;
    if (idx < cnt)
      mt = region ? static_cast<uint32_t>(p0 + lst[idx])
                  : (static_cast<uint32_t>(p0 + idx) | (key_flag(a, tok0, C, idx, h) ? kFlagBit : 0u));
    a.tmeta[ws_tile(a, region, h, i, k) * 32 + tid] = mt;
  }
  if constexpr (FP8) {
    // FP8 pages: the chunk's rows are quantized exactly as the commit will
    // store them (D/8 consecutive threads per row; rows past the end get
    // zero codes)
    char* tile = a.tiles + ws_tile(a, region, h, i, k) * fp8_tile_bytes(D);
    for (int pc = tid; pc < kPieces; pc += kThreads) {
      const int j = pc / (D / 8), part = pc % (D / 8);
      const int idx = 32 * k + j;
      uint4 kx = make_uint4(0u, 0u, 0u, 0u), vx = make_uint4(0u, 0u, 0u, 0u);
      if (idx < cnt) {
        const int c = region ? lst[idx] : idx;
        const size_t row = (static_cast<size_t>(tok0 + c) * a.H + h) * D + 8 * part;
        kx = *reinterpret_cast<const uint4*>(a.k + row);
        vx = *reinterpret_cast<const uint4*>(a.v + row);
      }
      fp8_store_token(tile, j, D, part, kx, vx);
    }
    return;
  }
  char* tile = a.tiles + ws_tile(a, region, h, i, k) * (D * 128);
  for (int pc = tid; pc < kPieces; pc += kThreads) {
    const int j = pc / (D / 8), e0 = 8 * (pc % (D / 8));
    const int idx = 32 * k + j;
    u32x4 kx = {0u, 0u, 0u, 0u}, vx = {0u, 0u, 0u, 0u};
    if (idx < cnt) {
      const int c = region ? lst[idx] : idx;
      const size_t row = (static_cast<size_t>(tok0 + c) * a.H + h) * D + e0;
      kx = *reinterpret_cast<const u32x4*>(a.k + row);
      vx = *reinterpret_cast<const u32x4*>(a.v + row);
    }
    *reinterpret_cast<u32x4*>(tile + k_elem_off(j, e0)) = kx;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vrows[j][e0 + 2 * e] = static_cast<uint16_t>(vx[e] & 0xFFFFu);
      vrows[j][e0 + 2 * e + 1] = static_cast<uint16_t>(vx[e] >> 16);
    }
  }
  __syncthreads();
  // value piece q: dim q / 4, keys 8 (q % 4) .. + 7 (contiguous in the tile)
  for (int q = tid; q < kPieces; q += kThreads) {
    const int e = q >> 2, j0 = 8 * (q & 3);
    u32x4 x;
#pragma unroll
    for (int t = 0; t < 4; ++t)
      x[t] = static_cast<uint32_t>(vrows[j0 + 2 * t][e]) | (static_cast<uint32_t>(vrows[j0 + 2 * t + 1][e]) << 16);
    *reinterpret_cast<u32x4*>(tile + v_elem_off(j0, e, D)) = x;
  }
}

template <int D>
struct Frag {
  u32x4 ka[D / 32];
  u32x4 kb[D / 32];
  u32x4 vt[D / 16];
};

// Staging of one 32-key tile: each thread moves 16-byte pieces of a tile in
// the pool layout (a pool page or a workspace tile) through registers.
template <int D>
struct Stage {
  static constexpr int kPieces = (D * 128) / 16 / attn_threads<D, false>();  // 16-byte pieces per thread
  u32x4 kx[kPieces / 2];   // key pieces
  u32x4 vx[kPieces / 2];   // value pieces
  uint32_t meta;           // this thread's key row (threads 0..31): position | flag << 31
};

// FP8 staging: each thread moves 16-byte pieces of the code part (keys then
// values) and threads 0..15 one 16-byte piece of the scales.
template <int D>
struct StageF8 {
  static constexpr int kPieces = (D * 64) / 16;              // code pieces per tile
  static constexpr int kPer = (kPieces + attn_threads<D, true>() - 1) / attn_threads<D, true>();
  u32x4 cx[kPer];
  float ks[kPer];          // key scale of the token a key piece belongs to
  u32x4 sx;                // scales: [G][key scales (8) | value scales (8)]
  uint32_t meta;
};

// Online-softmax weights of one key tile for one column block: s0 / s1 are
// the scores of key rows 8 G .. 8 G + 3 and 8 G + 4 .. 8 G + 7 of the lane's
// column t.  kp / kx (read only when masked): position and expiry (first
// query that no longer sees it) of those rows; vsc (FP8): their value scales.
// Rescales o and l_run when the column's max rises past the threshold;
// returns the weights rounded to bf16 for the PV MFMAs.
template <int D, bool FP8>
__device__ __forceinline__ u32x4 col_weights(f32x4 s0, f32x4 s1, const float (&vsc)[8], bool masked,
                                             const int (&kp)[8], const int (&kx)[8], int t,
                                             f32x4 (&o)[D / 16], float& m_ref, float& l_run, float thr,
                                             float scale_log2) {
  float sc[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sc[j] = s0[j];
    sc[j + 4] = s1[j];
  }
  if (masked) {
#pragma unroll
    for (int j = 0; j < 8; ++j) sc[j] = (kp[j] <= t && t < kx[j]) ? sc[j] : -INFINITY;
  }
  float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])),
                   fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
  mx = col_max(mx);
  const bool raise = mx > m_ref + thr;   // false while the column has seen no key
  if (__builtin_amdgcn_ballot_w64(raise)) {
    const float m_new = raise ? mx : m_ref;
    const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * scale_log2);
    l_run *= alpha;
#pragma unroll
    for (int b = 0; b < D / 16; ++b) o[b] *= alpha;
    m_ref = m_new;
  }
  // p = 2^((s - m) * scale); hidden keys give exactly 0
  const float mb = m_ref * scale_log2;
  float e[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = __builtin_amdgcn_exp2f(fmaf(sc[j], scale_log2, -mb));
  // P is rounded to bf16 for the MFMA; the denominator adds the same
  // rounded values (dot with (1, 1)), so a single dominant key returns its
  // value row exactly
  u32x4 pu;
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const f32x2 pr = {e[2 * j], e[2 * j + 1]};
    const bf16x2 pb = __builtin_convertvector(pr, bf16x2);
    pu[j] = __builtin_bit_cast(uint32_t, pb);
    l_run = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, l_run, false);
    if constexpr (FP8) {
      // PV weights carry the value scale: rounding commutes with a
      // power-of-two factor, so these are the rounded weights times it
      const f32x2 pv = {e[2 * j] * vsc[2 * j], e[2 * j + 1] * vsc[2 * j + 1]};
      pu[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pv, bf16x2));
    }
  }
  return pu;
}

// Scores, online softmax and PV of one key tile for the NQ column blocks of a
// wave.
template <int D, int NQ, bool FP8>
__device__ __forceinline__ void attend_tile(const Frag<D>& f, const float (&vsc)[8], bool masked,
                                            const int (&kp)[8], const int (&kx)[8],
                                            const int (&tcol)[NQ], const u32x4 (&qf)[NQ][D / 32],
                                            f32x4 (&o)[NQ][D / 16], float (&m_ref)[NQ],
                                            float (&l_run)[NQ], float thr, float scale_log2) {
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s2 = 0; s2 < D / 32; ++s2) {
      s0 = mfma_bf16(f.ka[s2], qf[qb][s2], s0);
      s1 = mfma_bf16(f.kb[s2], qf[qb][s2], s1);
    }
    const u32x4 pu = col_weights<D, FP8>(s0, s1, vsc, masked, kp, kx, tcol[qb], o[qb], m_ref[qb], l_run[qb],
                                         thr, scale_log2);
#pragma unroll
    for (int b = 0; b < D / 16; ++b) o[qb][b] = mfma_bf16(f.vt[b], pu, o[qb][b]);
  }
}

template <int D, int NQ, bool FP8>
__global__ __launch_bounds__((attn_threads<D, FP8>()), (512 / attn_threads<D, FP8>())) void prefill_kernel(PrefillArgs a) {
  constexpr int kThreads = attn_threads<D, FP8>();
  __shared__ __attribute__((aligned(16))) char tile_lds[2][D * 128];
  __shared__ __attribute__((aligned(16))) float scale_lds[2][64];   // FP8: tile scales
  __shared__ uint32_t meta_lds[2][32];
  __shared__ int masked_lds[2];   // tile has a key hidden from some query of the block
  __shared__ int item_lds[2];
  if (load_status(a.status) != 0) return;
  // attention of work item `item` = (grid row item / nx, query block item % nx)
  auto attend = [&](int item) {
  const int row = item / a.nx;
  const int hh = a.rows[row].hh;
  const int i = hh / a.H, h = hh % a.H;
  const int tok0 = a.cu[i], C = a.cu[i + 1] - a.cu[i];
  const int pb0 = (item - row * a.nx) * a.PB;
  if (pb0 >= C) return;
  const int s = a.seq_ids[i];
  const int sh = s * a.H + h;
  const int p0 = a.pos[s];
  const int L0 = a.len[sh];
  const int t0 = p0 + pb0;
  const int t1 = p0 + min(C, pb0 + a.PB);
  // band: chunk tiles from the one holding max(p0, t0 - w + 1) up to t1
  const int band_c0 = (max(0, pb0 - a.w + 1) >> 5) << 5;   // chunk-local, < C
  // kept chunk keys strictly before the band (a prefix of the sorted list),
  // counted by pass 0
  const int32_t* lst = a.list + static_cast<size_t>(h) * a.total + tok0;
  const int n_pre = a.kept_before[ws_kb(a, h, i, band_c0 >> 5)];
  const int nc = (L0 + 31) >> 5;
  const int np = (n_pre + 31) >> 5;
  const int nb = (t1 - p0 - band_c0 + 31) >> 5;
  constexpr size_t kTB = FP8 ? static_cast<size_t>(D) * 64 + 256 : static_cast<size_t>(D) * 128;
  const char* pre_tiles = a.tiles + ws_tile(a, 1, h, i, 0) * kTB;
  const char* band_tiles = a.tiles + ws_tile(a, 0, h, i, band_c0 >> 5) * kTB;
  const int ntiles = nc + np + nb;
  const int32_t* pt = a.page_table + static_cast<size_t>(sh) * a.maxp;
  const int32_t* smeta = a.slot_meta + static_cast<size_t>(sh) * a.max_slots;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, G = lane >> 4;
  const int Hq = a.H * a.g;

  // ---- columns of this lane: column c of the workgroup's (wave, block,
  // lane r) is query head c % g at position t0 + c / g (a position's heads
  // may straddle two column blocks)
  int tcol[NQ];
  u32x4 qf[NQ][D / 32];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const int col = (wave * NQ + qb) * 16 + r;
    const int pl = col / a.g, qh = col % a.g;
    const int t = t0 + pl;
    const bool ok = (pl < a.PB) && (t < t1);
    tcol[qb] = ok ? t : -1;
    const u32x4 z = {0u, 0u, 0u, 0u};
    const char* qrow = reinterpret_cast<const char*>(
        a.q + (static_cast<size_t>(tok0 + (t - p0)) * Hq + h * a.g + qh) * D);
#pragma unroll
    for (int s2 = 0; s2 < D / 32; ++s2)
      qf[qb][s2] = ok ? *reinterpret_cast<const u32x4*>(qrow + (32 * s2 + 8 * G) * 2) : z;
    // the borrowed decision neuron takes no part in attention (App. C)
    if (a.zero_neuron && qh == 0 && G == 0) qf[qb][0][0] &= 0xFFFF0000u;
  }

  // ---- staging: global -> registers (A), registers -> LDS (B)
  using StageT = typename std::conditional<FP8, StageF8<D>, Stage<D>>::type;
  StageT stg;
  auto stage_load = [&](int k) {
    const char* tile;
    if (k < nc) {
      const int sb = k * 32;
      tile = a.pool + static_cast<size_t>(pt[sb >> a.log2P]) * a.page_bytes +
             static_cast<size_t>((sb & (a.P - 1)) >> 5) * kTB;
      if (tid < 32) {
        uint32_t mt = sb + tid < L0 ? static_cast<uint32_t>(smeta[sb + tid]) : kNoKey;
        if (mt != kNoKey) {
          // a cached key j is hidden by the decision of position j + w, which
          // (for a live key) lies in this chunk or later
          const int kp = static_cast<int>(mt & ~kFlagBit);
          const int x = kp + a.w - p0;
          mt = static_cast<uint32_t>(kp) |
               ((x >= 0 && x < C && a.flags[static_cast<size_t>(tok0 + x) * a.H + h]) ? kFlagBit : 0u);
        }
        stg.meta = mt;
      }
    } else if (k < nc + np) {
      const int kk = k - nc;
      tile = pre_tiles + static_cast<size_t>(kk) * kTB;
      if (tid < 32) {
        const int idx = kk * 32 + tid;
        stg.meta = idx < n_pre ? static_cast<uint32_t>(p0 + lst[idx]) : kNoKey;
      }
    } else {
      const int kb = k - nc - np;
      tile = band_tiles + static_cast<size_t>(kb) * kTB;
      if (tid < 32) {
        const int c = band_c0 + kb * 32 + tid;
        stg.meta = c < t1 - p0 ? (static_cast<uint32_t>(p0 + c) |
                                  (key_flag(a, tok0, C, c, h) ? kFlagBit : 0u))
                               : kNoKey;
      }
    }
    if constexpr (FP8) {
#pragma unroll
      for (int m = 0; m < StageF8<D>::kPer; ++m) {
        const int Q = tid + m * kThreads;
        if (Q < StageF8<D>::kPieces) stg.cx[m] = *reinterpret_cast<const u32x4*>(tile + Q * 16);
        if (Q < 2 * D) {
          // key piece (p, h, lane L): all 16 codes belong to slot 8 (r/4) + r%4 + 4 h
          const int r = Q & 15, j = 8 * (r >> 2) + (r & 3) + 4 * ((Q >> 6) & 1);
          stg.ks[m] = *reinterpret_cast<const float*>(tile + D * 64 + (j >> 3) * 64 + (j & 7) * 4);
        }
      }
      if (tid < 16) stg.sx = *reinterpret_cast<const u32x4*>(tile + D * 64 + tid * 16);
    } else {
      constexpr int KP = Stage<D>::kPieces / 2;
#pragma unroll
      for (int m = 0; m < KP; ++m) {
        stg.kx[m] = *reinterpret_cast<const u32x4*>(tile + (tid + m * kThreads) * 16);
        stg.vx[m] = *reinterpret_cast<const u32x4*>(tile + D * 64 + (tid + m * kThreads) * 16);
      }
    }
  };
  auto stage_store = [&](int k, int buf) {
    char* dst = tile_lds[buf];
    // pool slots past L hold stale data: their value elements are zeroed
    // (workspace tiles are zero past their last row)
    const int valid = k < nc ? min(32, L0 - k * 32) : 32;
    if constexpr (FP8) {
      // a 16-byte code piece becomes two bf16 LDS slots (exact conversion);
      // the FP8 tile order matches the LDS fragment order (dms_fp8.h)
#pragma unroll
      for (int m = 0; m < StageF8<D>::kPer; ++m) {
        const int Q = tid + m * kThreads;
        if (Q < StageF8<D>::kPieces) {
          u32x4 x = stg.cx[m];
          int P0, step;
          float scale = 1.0f;
          if (Q < 2 * D) {            // keys: piece (p, h, lane L), dequantized exactly
            P0 = 256 * (Q >> 7) + (Q & 127);
            step = 128;
            scale = stg.ks[m];
          } else {                    // values: piece (p, lane L), slots 8G .. 8G+7
            const int Qv = Q - 2 * D;
            P0 = D * 4 + 128 * (Qv >> 6) + (Qv & 63);
            step = 64;
            const int nv = valid - 8 * ((Qv >> 4) & 3);
            if (nv < 8) {
              const uint64_t keep8 = nv <= 0 ? 0ull : (~0ull >> (8 * (8 - nv)));
              const uint32_t klo = static_cast<uint32_t>(keep8), khi = static_cast<uint32_t>(keep8 >> 32);
              x[0] &= klo;
              x[1] &= khi;
              x[2] &= klo;
              x[3] &= khi;
            }
          }
          u32x4 lo, hi;
#pragma unroll
          for (int w2 = 0; w2 < 2; ++w2) {
            lo[2 * w2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[w2], scale, false));
            lo[2 * w2 + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[w2], scale, true));
            hi[2 * w2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[2 + w2], scale, false));
            hi[2 * w2 + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[2 + w2], scale, true));
          }
          *reinterpret_cast<u32x4*>(dst + P0 * 16) = lo;
          *reinterpret_cast<u32x4*>(dst + (P0 + step) * 16) = hi;
        }
      }
      if (tid < 16) {
        // scale piece tid: group G = tid / 4, key (tid % 4 < 2) or value scales of
        // slots 8 G + 4 (tid % 2) .. + 3; missing slots get 0
        u32x4 x = stg.sx;
        const int j0 = 8 * (tid >> 2) + 4 * (tid & 1);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (j0 + c >= valid) x[c] = 0u;
        *reinterpret_cast<u32x4*>(&scale_lds[buf][4 * tid]) = x;
      }
    } else {
      constexpr int KP = Stage<D>::kPieces / 2;
#pragma unroll
      for (int m = 0; m < KP; ++m) {
        const int P = tid + m * kThreads;
        *reinterpret_cast<u32x4*>(dst + P * 16) = stg.kx[m];
        u32x4 x = stg.vx[m];
        // element i of the value piece is key row 8 G + i
        const int j0 = 8 * ((P >> 4) & 3);
        if (j0 + 8 > valid) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (j0 + e >= valid) x[e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
        }
        *reinterpret_cast<u32x4*>(dst + D * 64 + P * 16) = x;
      }
    }
    if (tid < 64) {
      // a key row needs the per-element mask iff some query t in [t0, t1)
      // does not see it: padding, causal (position > t0) or flagged and
      // expiring by t1 - 1
      bool need = false;
      if (tid < 32) {
        const uint32_t mt = stg.meta;
        const int kp = static_cast<int>(mt & ~kFlagBit);
        need = mt == kNoKey || kp > t0 || ((mt & kFlagBit) && kp + a.w <= t1 - 1);
        meta_lds[buf][tid] = mt;
      }
      const uint64_t any = __builtin_amdgcn_ballot_w64(need);
      if (tid == 0) masked_lds[buf] = any != 0;
    }
  };

  // ---- accumulators
  f32x4 o[NQ][D / 16];
  float m_ref[NQ], l_run[NQ];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
#pragma unroll
    for (int b = 0; b < D / 16; ++b) o[qb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_ref[qb] = kMInit;
    l_run[qb] = 0.f;
  }
  const uint32_t lo_k = static_cast<uint32_t>(lane * 16);
  const uint32_t lo_v = static_cast<uint32_t>(D * 64 + lane * 16);
  const float thr = kRescale / a.scale_log2;   // rescale threshold in score units

  if (ntiles > 0) {
    stage_load(0);
    stage_store(0, 0);
  }
  __syncthreads();
  for (int k = 0; k < ntiles; ++k) {
    const int buf = k & 1;
    if (k + 1 < ntiles) stage_load(k + 1);
    // operands of this tile from LDS
    const char* tl = tile_lds[buf];
    Frag<D> f;
#pragma unroll
    for (int s2 = 0; s2 < D / 32; ++s2) {
      f.ka[s2] = *reinterpret_cast<const u32x4*>(tl + lo_k + s2 * 2048);
      f.kb[s2] = *reinterpret_cast<const u32x4*>(tl + lo_k + 1024 + s2 * 2048);
    }
#pragma unroll
    for (int b = 0; b < D / 16; ++b) f.vt[b] = *reinterpret_cast<const u32x4*>(tl + lo_v + b * 1024);
    float vsc[8];   // FP8: value scales of rows 8G .. 8G+7 (keys are staged dequantized)
    if constexpr (FP8) {
      const f32x4 v0 = *reinterpret_cast<const f32x4*>(&scale_lds[buf][16 * G + 8]);
      const f32x4 v1 = *reinterpret_cast<const f32x4*>(&scale_lds[buf][16 * G + 12]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        vsc[j] = v0[j];
        vsc[j + 4] = v1[j];
      }
    }
    const bool masked = __builtin_amdgcn_readfirstlane(masked_lds[buf]) != 0;
    int kp[8], kx[8];   // key position and expiry (first query that no longer sees it)
    if (masked) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t km = meta_lds[buf][8 * G + j];
        kp[j] = static_cast<int>(km & ~kFlagBit);
        kx[j] = (km & kFlagBit) ? kp[j] + a.w : 0x7FFFFFFF;
      }
    }
    attend_tile<D, NQ, FP8>(f, vsc, masked, kp, kx, tcol, qf, o, m_ref, l_run, thr, a.scale_log2);
    if (k + 1 < ntiles) stage_store(k + 1, buf ^ 1);
    __syncthreads();
  }

  // ---- outputs
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    float l = l_run[qb];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const int t = tcol[qb];
    if (t >= 0) {
      const int qh = ((wave * NQ + qb) * 16 + r) % a.g;
      const float inv = 1.0f / l;
      float* dst = a.out + (static_cast<size_t>(tok0 + (t - p0)) * Hq + h * a.g + qh) * D + 4 * G;
#pragma unroll
      for (int b = 0; b < D / 16; ++b) *reinterpret_cast<f32x4*>(dst + 16 * b) = o[qb][b] * inv;
    }
  }
};

  // items: grid position first, then the counter
  int item = blockIdx.x, buf = 0;
  if (threadIdx.x == 0) item_lds[0] = gridDim.x + atomicAdd(a.work_ctr, 1);
  while (item < a.items) {
    attend(item);
    __syncthreads();   // the fetched index is visible; every wave is done with the LDS buffers
    const int next = item_lds[buf];
    if (threadIdx.x == 0) item_lds[buf ^ 1] = gridDim.x + atomicAdd(a.work_ctr, 1);
    buf ^= 1;
    item = next;
  }
}

// ---------------------------------------------------------------------------
// Attention pass under delayed eviction, 32x32 MFMA products.  A wave holds
// 32 columns; keys go through LDS 64 at a time (two tiles, two buffers): both
// tiles' scores, one column maximum and (rare) rescale, the weights, both
// tiles' value products, one barrier.  A tile read from LDS feeds 32 columns
// with half the MFMA and LDS read instructions of 16x16 products, and the
// pool's tile order serves them with one base address per operand and
// constant offsets:
//   keys: lane l of k-step s takes dims 16 s + 8 (l / 32) .. + 7 of token
//     row_token(l % 32) (accumulator registers 8 y .. 8 y + 7 are then tokens
//     16 y + 8 (l / 32) .. + 7, the B operand of half y of the value product);
//   values: lane l of (32-dim block b, half y) takes tokens 16 y + 8 (l / 32)
//     .. + 7 of dim 32 b + l % 32.
// Both are free of bank conflicts (8-lane runs of 128 bytes).
//
// bf16 pages (four waves, two workgroups per CU): every key source is a plain
// copy -- pool tiles with their slot metadata, workspace tiles with the
// metadata pass 1 wrote -- so global -> LDS loads move a quarter of a stage
// per wave while the stage before it is attended.  FP8 pages (eight waves at
// d = 128: each of a chunk's query blocks stages every cached tile of its
// head, so more columns per workgroup means fewer dequantizations): codes go
// through registers and are dequantized into the same order.  Rows past a
// source's end are fixed up when read: pool slots past the live length hold
// stale data (values zeroed in LDS, keys hidden), kept-list rows from
// the band on are hidden.
//
// The two tiles' score chains alternate, and the second tile's weights are
// formed between the first tile's value products.  Operands are read kAhead
// products before their use, in pinned order: left to itself the compiler
// reads each just before its product and waits.  The first stage of the next
// item is copied beside the last one of the present item.  Four prompts of
// 4096 to 16384 tokens in chunks of 4096 a sequence (8 KV heads of 5, d = 128,
// window 256, 7/8 flagged) take 1628 us, every pass and commit counted, from
// 2068 us with 16x16 products and 32 keys per barrier (1856 before the operand
// order and the item overlap); two of 3001 and 11999 tokens with FP8 pages (4
// heads of 7) take 856, from 1084 us.  Bound by the softmax's exponentials
// and conversions, which the matrix core does not fully cover with two waves
// per SIMD.
//
// The LDS destination of a copy goes in M0, written by the same inline
// assembly statement as the load; nothing else in this file reads M0.  The
// compiler does not count these loads, so the kernel waits for them itself
// (vmcnt) before the barrier that publishes a stage.
// ---------------------------------------------------------------------------
#define DMS_LDS __attribute__((address_space(3)))
#define DMS_CONST __attribute__((address_space(4)))

constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

__device__ inline uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DMS_LDS const char*)p));
}

// 64 lanes x 16 bytes from g (per lane) to LDS m0 + 16 lane
__device__ inline void lds_copy16(const char* g, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(m0), "v"(g) : "memory", "m0");
}
// 64 lanes x 4 bytes from g (per lane) to LDS m0 + 4 lane
__device__ inline void lds_copy4(const char* g, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" : : "s"(m0), "v"(g) : "memory", "m0");
}

typedef __attribute__((ext_vector_type(16))) float f32x16;
__device__ inline f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// max / sum over the two lanes of one column (l and l + 32)
__device__ inline float col_max32(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ inline float col_sum32(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
// keeps the compiler from forming what follows from x ahead of a loop and holding it
__device__ inline int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ inline int row_token(int r) {
  return 16 * (r >> 4) + 8 * ((r >> 2) & 1) + 4 * ((r >> 3) & 1) + (r & 3);
}

// One work item of an attention pass: (row, query block) and the key tiles it
// attends -- nc pool tiles, np tiles of kept chunk keys, then the band.
struct Item {
  int hh, tok0, C, sh, p0, L0, t0, t1, n_pre, nc, np, ntiles, pre0, band0;
};

// Work item `item`; `first`: the rows' first items in LDS (ranked calls).
__device__ __forceinline__ Item prefill_item(const PrefillArgs& a, const int* first, int item, int lane) {
  Item it;
  const int NH = a.n * a.H;
  int row, block;
  if (NH <= kOrderMax) {
    // the last row whose first item is not past this one
    row = -1;
    for (int x = 0; x < NH; x += 64)
      row += __builtin_popcountll(__builtin_amdgcn_ballot_w64(x + lane < NH && first[min(x + lane, NH)] <= item));
    row = __builtin_amdgcn_readfirstlane(row);
    block = item - __builtin_amdgcn_readfirstlane(first[row]);
  } else {
    row = item / a.nx;
    block = item - row * a.nx;
  }
  typedef int __attribute__((ext_vector_type(8))) i32x8;
  const i32x8 rd = *((const DMS_CONST i32x8*)(a.rows + row));
  it.hh = rd[0];
  it.tok0 = rd[1];
  it.C = rd[2];
  it.sh = rd[3];
  it.p0 = rd[4];
  it.L0 = rd[5];
  const int h = it.hh % a.H, pb0 = block * a.PB;
  it.t0 = it.p0 + pb0;
  it.t1 = it.p0 + min(it.C, pb0 + a.PB);
  // band: chunk tiles from the one holding max(p0, t0 - w + 1) up to t1
  const int band_c0 = (max(0, pb0 - a.w + 1) >> 5) << 5;   // chunk-local, < C
  it.pre0 = (a.H + h) * a.tph + rd[6];
  it.band0 = h * a.tph + rd[6] + (band_c0 >> 5);
  it.nc = (it.L0 + 31) >> 5;
  if (pb0 >= it.C) {   // unranked calls only: no columns, one tile of any bits
    it.t1 = it.t0;
    it.n_pre = it.nc = it.np = 0;
    it.ntiles = 1;
    it.band0 = h * a.tph + rd[6];
    return it;
  }
  // kept chunk keys strictly before the band, counted by pass 0
  it.n_pre = ((const DMS_CONST int32_t*)a.kept_before)[it.band0];
  it.np = (it.n_pre + 31) >> 5;
  it.ntiles = it.nc + it.np + ((it.t1 - it.p0 - band_c0 + 31) >> 5);
  return it;
}
// pool page of tile k (only read for k < nc)
__device__ __forceinline__ int pool_page(const PrefillArgs& a, const Item& it, int k) {
  return k < it.nc ? ((const DMS_CONST int32_t*)(a.page_table + static_cast<size_t>(it.sh) * a.maxp))[(32 * k) >> a.log2P] : 0;
}
// stored tile k and its key rows (workspace tiles of one region and head are consecutive)
__device__ __forceinline__ void tile_source(const PrefillArgs& a, const Item& it, int k, int page, size_t tile_size,
                                            const char*& tile, const uint32_t*& mt) {
  if (k < it.nc) {
    const int sb = 32 * k;
    tile = a.pool + static_cast<size_t>(page) * a.page_bytes + static_cast<size_t>((sb & (a.P - 1)) >> 5) * tile_size;
    mt = reinterpret_cast<const uint32_t*>(a.slot_meta + static_cast<size_t>(it.sh) * a.max_slots) + sb;
  } else {
    const size_t x = k < it.nc + it.np ? it.pre0 + (k - it.nc) : it.band0 + (k - it.nc - it.np);
    tile = a.tiles + x * tile_size;
    mt = a.tmeta + x * 32;
  }
}
// rows of tile k that exist
__device__ __forceinline__ int rows_of(const Item& it, int k) {
  return k >= it.ntiles ? 0 : k < it.nc ? it.L0 - 32 * k : (k < it.nc + it.np ? it.n_pre - 32 * (k - it.nc) : 32);
}
// a key row (position | flag << 31) needs the per-element mask iff some query t in [t0, t1) does
// not see it: no key, causal (position > t0) or flagged and expiring by t1 - 1
__device__ __forceinline__ bool row_hidden(uint32_t mrow, const Item& it, int w) {
  const int kp = static_cast<int>(mrow & ~kFlagBit);
  return (mrow == kNoKey) | (kp > it.t0) | (((mrow & kFlagBit) != 0) & (kp + w <= it.t1 - 1));
}
// Scores of one tile with the keys that the column at position t does not see
// set to -inf; mp: the lane's key rows (register i: row 16 (i / 8) + i % 8 past mp).
__device__ __forceinline__ void mask_scores(f32x16& s, const uint32_t* mp, int rows, int t, int w, int lane) {
  if (rows < 32) {   // rows past the source's end hold no key
    const int j0 = 8 * (fresh(lane) >> 5);
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (j0 + 16 * (i >> 3) + (i & 7) >= rows) s[i] = -INFINITY;
  }
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const u32x4 km = *reinterpret_cast<const u32x4*>(mp + 16 * (i4 >> 1) + 4 * (i4 & 1));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // seen from its own position on, if flagged for w positions (no key: position
      // 2^31 - 1; unused column: t = -1)
      const uint32_t age = static_cast<uint32_t>(t) - (km[e] & ~kFlagBit);
      const uint32_t seen = (km[e] & kFlagBit) ? static_cast<uint32_t>(w) : 0x7FFFFFFFu;
      s[4 * i4 + e] = age < seen ? s[4 * i4 + e] : -INFINITY;
    }
  }
}
constexpr int kAhead = 4;   // MFMAs between an operand's LDS read and its use

template <int D, bool FP8>
constexpr int delayed_waves() { return attn_threads<D, FP8>() / 64; }

template <int D, bool FP8>
__global__ __launch_bounds__((64 * delayed_waves<D, FP8>()), (8 / delayed_waves<D, FP8>()))
void prefill_delayed_kernel(PrefillArgs a) {
  constexpr int NW = delayed_waves<D, FP8>();
  constexpr int kTB = D * 128;          // one staged (bf16) tile
  constexpr size_t kSB = FP8 ? static_cast<size_t>(D) * 64 + 256 : static_cast<size_t>(kTB);   // one stored tile
  constexpr int KS = D / 16, OB = D / 32;
  __shared__ __attribute__((aligned(16))) char tile_lds[2][2 * kTB];
  __shared__ __attribute__((aligned(16))) uint32_t meta_lds[2][2][64];   // [buffer][tile], rows 0..31 twice
  __shared__ __attribute__((aligned(16))) float scale_lds[FP8 ? 2 : 1][2][64];   // FP8: tile scales
  __shared__ int item_lds[2], first_lds[kOrderMax + 1];
  if (load_status(a.status) != 0) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5;
  const int Hq = a.H * a.g;
  const float thr = kRescale / a.scale_log2, sl2 = a.scale_log2;
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
  const int kt = row_token(lane & 31);
  const char* k_base = tile_lds[0] + ((kt >> 2) & 1) * 1024 + hf * 256 + (4 * (kt >> 3) + (kt & 3)) * 16;
  const char* v_base = tile_lds[0] + D * 64 + ((lane >> 4) & 1) * 1024 + hf * 256 + (lane & 15) * 16;

  // ---- work items: (row, query block), heaviest rows first.  The next item's
  // descriptor is loaded and its first stage copied beside the last stage of
  // the present one, so that a short item does not wait
  // for its chain of dependent loads (about a third of a 600-key item's time).
  const int NH = a.n * a.H;
  const bool ranked = NH <= kOrderMax;
  if (ranked)
    for (int x = tid; x <= NH; x += 64 * NW) first_lds[x] = a.first_item[x];
  __syncthreads();
  const int items = ranked ? __builtin_amdgcn_readfirstlane(first_lds[NH]) : a.items;
  // ranked: first_lds holds the rows' first items (see order_rows)
  auto load_item = [&](int item) { return prefill_item(a, first_lds, item, lane); };
  auto page_of = [&](const Item& it, int k) { return pool_page(a, it, k); };
  auto source = [&](const Item& it, int k, int page, const char*& tile, const uint32_t*& mt) {
    tile_source(a, it, k, page, kSB, tile, mt);
  };

  // ---- staging of stage st (tiles 2 st, 2 st + 1; the last one again past the end)
  constexpr int kSubs = 2;
  u32x4 cx[kSubs], sx[kSubs];      // FP8: this thread's code piece, scales (threads 0..15) of each tile
  float ks[kSubs];                 // key scale of a key piece's token
  uint32_t mt_reg[kSubs];
  const int my_sub = (wave >> 1) & 1;
  auto stage_pages = [&](const Item& it, int st, int (&pg)[kSubs]) {
    if constexpr (FP8) {
#pragma unroll
      for (int u = 0; u < kSubs; ++u) pg[u] = page_of(it, min(2 * st + u, it.ntiles - 1));
    } else {
      pg[0] = page_of(it, min(2 * st + my_sub, it.ntiles - 1));
    }
  };
  auto stage_load = [&](const Item& it, int st, int buf, const int (&pg)[kSubs]) {
    const char* tile;
    const uint32_t* mt;
    if constexpr (FP8) {
#pragma unroll
      for (int u = 0; u < kSubs; ++u) {
        source(it, min(2 * st + u, it.ntiles - 1), pg[u], tile, mt);
        cx[u] = *reinterpret_cast<const u32x4*>(tile + tid * 16);
        if (tid < 2 * D) {
          // key piece (p, h, lane L): all 16 codes belong to slot 8 (r/4) + r%4 + 4 h
          const int r = tid & 15, j = 8 * (r >> 2) + (r & 3) + 4 * ((tid >> 6) & 1);
          ks[u] = *reinterpret_cast<const float*>(tile + D * 64 + (j >> 3) * 64 + (j & 7) * 4);
        }
        if (tid < 16) sx[u] = *reinterpret_cast<const u32x4*>(tile + D * 64 + tid * 16);
        if (tid < 64) mt_reg[u] = mt[tid & 31];
      }
    } else {
      // wave w copies the keys (w even) or values of tile w / 2 of the stage
      source(it, min(2 * st + my_sub, it.ntiles - 1), pg[0], tile, mt);
      // a tile past the last (the last one again, its keys hidden) has zero values: 0 times an Inf
      // of the last one must not reach the sums
      if (wave & 1) tile = 2 * st + my_sub >= it.ntiles ? a.zeros : tile + D * 64;
      const char* src = tile + lane * 16;
      const uint32_t dst = lds_addr(tile_lds[0]) + buf * 2 * kTB + my_sub * kTB + (wave & 1) * (D * 64);
#pragma unroll
      for (int m = 0; m < D / 16; ++m) lds_copy16(src + m * 1024, dst + m * 1024);
      if (!(wave & 1)) lds_copy4(reinterpret_cast<const char*>(mt + (lane & 31)), lds_addr(meta_lds[buf][my_sub]));
    }
  };
  auto stage_store = [&](const Item& it, int st, int buf) {
    if constexpr (FP8) {
      // a 16-byte code piece becomes two bf16 LDS slots (exact conversion);
      // the FP8 tile order matches the LDS fragment order (dms_fp8.h)
#pragma unroll
      for (int u = 0; u < kSubs; ++u) {
        const int k = min(2 * st + u, it.ntiles - 1);
        // (a tile past the last: none)
        const int valid = 2 * st + u >= it.ntiles ? 0 : k < it.nc ? min(32, it.L0 - k * 32) : 32;
        char* dst = tile_lds[buf] + u * kTB;
        u32x4 x = cx[u];
        int P0, step;
        float scale = 1.0f;
        if (tid < 2 * D) {          // keys: piece (p, h, lane L), dequantized exactly
          P0 = 256 * (tid >> 7) + (tid & 127);
          step = 128;
          scale = ks[u];
        } else {                    // values: piece (p, lane L), slots 8G .. 8G+7
          const int Qv = tid - 2 * D;
          P0 = D * 4 + 128 * (Qv >> 6) + (Qv & 63);
          step = 64;
          const int nv = valid - 8 * ((Qv >> 4) & 3);
          if (nv < 8) {
            const uint64_t keep8 = nv <= 0 ? 0ull : (~0ull >> (8 * (8 - nv)));
            const uint32_t klo = static_cast<uint32_t>(keep8), khi = static_cast<uint32_t>(keep8 >> 32);
            x &= u32x4{klo, khi, klo, khi};
          }
        }
        u32x4 lo, hi;
#pragma unroll
        for (int w2 = 0; w2 < 2; ++w2) {
          lo[2 * w2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[w2], scale, false));
          lo[2 * w2 + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[w2], scale, true));
          hi[2 * w2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[2 + w2], scale, false));
          hi[2 * w2 + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x[2 + w2], scale, true));
        }
        *reinterpret_cast<u32x4*>(dst + P0 * 16) = lo;
        *reinterpret_cast<u32x4*>(dst + (P0 + step) * 16) = hi;
        if (tid < 16) {
          // scale piece tid: group G = tid / 4, key (tid % 4 < 2) or value scales of
          // slots 8 G + 4 (tid % 2) .. + 3; missing slots get 0
          const int j0 = 8 * (tid >> 2) + 4 * (tid & 1);
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (j0 + c >= valid) sx[u][c] = 0u;
          *reinterpret_cast<u32x4*>(&scale_lds[buf][u][4 * tid]) = sx[u];
        }
        if (tid < 64) meta_lds[buf][u][tid] = mt_reg[u];
      }
    }
  };

  if (static_cast<int>(blockIdx.x) >= items) return;
  Item cur = load_item(blockIdx.x);
  int pg[kSubs] = {0, 0};
  stage_pages(cur, 0, pg);
  stage_load(cur, 0, 0, pg);
  stage_pages(cur, 1, pg);
  if constexpr (FP8) stage_store(cur, 0, 0);
  int par = 0, ib = 0;   // LDS buffer of the present stage, slot of the next item's index

  // this lane's column: query head col % g at position t0 + col / g (a
  // position's g heads may straddle two waves; the last 32 NW mod g columns go
  // unused)
  const int col = wave * 32 + (lane & 31);
  const int pl = col / a.g, qh = col % a.g;
  while (true) {
    const int h = cur.hh % a.H;
    const bool ok = pl < a.PB && cur.t0 + pl < cur.t1;
    const int t = ok ? cur.t0 + pl : -1;
    const size_t orow = static_cast<size_t>(cur.tok0 + (ok ? t - cur.p0 : 0)) * Hq + h * a.g + qh;
    u32x4 qf[KS];
#pragma unroll
    for (int x = 0; x < KS; ++x)
      qf[x] = ok ? *reinterpret_cast<const u32x4*>(a.q + orow * D + 16 * x + 8 * hf) : u32x4{0u, 0u, 0u, 0u};
    // the borrowed decision neuron takes no part in attention (App. C)
    if (a.zero_neuron && qh == 0 && hf == 0) qf[0][0] &= 0xFFFF0000u;
    f32x16 o[OB];
#pragma unroll
    for (int x = 0; x < OB; ++x)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[x][i] = 0.f;
    float m_ref = kMInit, l_run = 0.f;
    if (tid == 0) item_lds[ib] = gridDim.x + atomicAdd(a.work_ctr, 1);   // read after this item's last barrier
    Item nxt = cur;
    bool have_next = false;
    auto stage = [&](int st, auto last_c) {
      constexpr bool last = decltype(last_c)::value;
      const int buf = par, tl = par * 2 * kTB;
      if constexpr (!FP8) __builtin_amdgcn_s_waitcnt(wait_vm(0));
      __syncthreads();
      if constexpr (!last) {
        stage_load(cur, st + 1, buf ^ 1, pg);
      } else {
        const int item = __builtin_amdgcn_readfirstlane(item_lds[ib]);
        have_next = item < items;
        if (have_next) {
          nxt = load_item(item);
          stage_pages(nxt, 0, pg);
          stage_load(nxt, 0, buf ^ 1, pg);
        }
      }
      const int rows0 = rows_of(cur, 2 * st), rows1 = rows_of(cur, 2 * st + 1);
      if (!FP8 && (cur.L0 & 31) && st == (cur.nc - 1) >> 1) {
        // the pool's last tile: value elements of slots past the live length are stale
        const int sub = (cur.nc - 1) & 1, valid = cur.L0 & 31;
        for (int P = tid; P < D * 4; P += 64 * NW) {
          const int nv = valid - 8 * ((P >> 4) & 3);   // elements of this piece that exist
          if (nv >= 8) continue;
          u32x4* x = reinterpret_cast<u32x4*>(tile_lds[0] + tl + sub * kTB + D * 64 + P * 16);
          u32x4 keep;
#pragma unroll
          for (int e = 0; e < 4; ++e) keep[e] = (2 * e < nv ? 0x0000FFFFu : 0u) | (2 * e + 1 < nv ? 0xFFFF0000u : 0u);
          *x &= keep;
        }
        __syncthreads();
      }
      // this lane's of the stage's 64 key rows
      uint32_t mrow = meta_lds[buf][0][64 * hf + (lane & 31)];
      if ((lane & 31) >= (hf ? rows1 : rows0)) mrow = kNoKey;
      const uint64_t hidden = __builtin_amdgcn_ballot_w64(row_hidden(mrow, cur, a.w));
      __builtin_amdgcn_sched_barrier(0);
      // Operands are read kAhead MFMAs ahead of their use in an order that is
      // pinned step by step: left alone the compiler reads each operand right
      // before its MFMA and waits out the LDS latency every time.
      f32x16 s[2];
#pragma unroll
      for (int i = 0; i < 16; ++i) s[0][i] = s[1][i] = 0.f;
      {
        u32x4 op[kAhead];
        auto read = [&](int e) {   // tile e % 2, k-step e / 2: the two chains take turns
          return *reinterpret_cast<const u32x4*>(k_base + tl + (e & 1) * kTB + (e >> 2) * 2048 + ((e >> 1) & 1) * 512);
        };
#pragma unroll
        for (int e = 0; e < kAhead; ++e) op[e] = read(e);
#pragma unroll
        for (int e = 0; e < 2 * KS; ++e) {
          __builtin_amdgcn_sched_barrier(0);
          s[e & 1] = mfma32(op[e % kAhead], qf[e >> 1], s[e & 1]);
          if (e + kAhead < 2 * KS) op[e % kAhead] = read(e + kAhead);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (hidden) {
        mask_scores(s[0], &meta_lds[buf][0][8 * hf], rows0, t, a.w, lane);
        mask_scores(s[1], &meta_lds[buf][1][8 * hf], rows1, t, a.w, lane);
      }
      float mx = fmaxf(s[0][0], s[1][0]);
  #pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(fmaxf(mx, s[0][i]), s[1][i]);
      mx = col_max32(mx);
      const bool raise = mx > m_ref + thr;   // false while the column has seen no key
      if (__builtin_amdgcn_ballot_w64(raise)) {
        const float m_new = raise ? mx : m_ref;
        const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * sl2);
        l_run *= alpha;
  #pragma unroll
        for (int x = 0; x < OB; ++x) o[x] *= alpha;
        m_ref = m_new;
      }
      const float mb = m_ref * sl2;
      // weights p = 2^((s - m) scale) rounded to bf16 for the MFMA; the
      // denominator adds the same rounded values (dot with (1, 1)), so a
      // single dominant key returns its value row exactly; hidden keys give 0
      u32x4 pu[2][2];
      auto weight_pair = [&](int u, int j) {
        const f32x2 pr = {__builtin_amdgcn_exp2f(fmaf(s[u][2 * j], sl2, -mb)),
                          __builtin_amdgcn_exp2f(fmaf(s[u][2 * j + 1], sl2, -mb))};
        const bf16x2 pb = __builtin_convertvector(pr, bf16x2);
        pu[u][j >> 2][j & 3] = __builtin_bit_cast(uint32_t, pb);
        l_run = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, l_run, false);
        if constexpr (FP8) {
          // PV weights carry the value scale: rounding commutes with a
          // power-of-two factor, so these are the rounded weights times it.
          // scales: [slot group of 8][key scales (8) | value scales (8)]
          const f32x2 vs = *reinterpret_cast<const f32x2*>(&scale_lds[buf][u][16 * (2 * (j >> 2) + hf) + 8 + 2 * (j & 3)]);
          pu[u][j >> 2][j & 3] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr * vs, bf16x2));
        }
      };
#pragma unroll
      for (int j = 0; j < 8; ++j) weight_pair(0, j);
      // value product e of the stage: tile e / (2 OB), token half (e / OB) % 2, dim block e % OB
      auto read_v = [&](int e) {
        return *reinterpret_cast<const u32x4*>(v_base + tl + e / (2 * OB) * kTB + (e % OB) * 2048 + (e / OB) % 2 * 512);
      };
      // the second tile's weights beside the first one's products
      u32x4 op[kAhead];
#pragma unroll
      for (int e = 0; e < kAhead; ++e) op[e] = read_v(e);
#pragma unroll
      for (int e = 0; e < 4 * OB; ++e) {
        __builtin_amdgcn_sched_barrier(0);
        o[e % OB] = mfma32(op[e % kAhead], pu[e / (2 * OB)][(e / OB) % 2], o[e % OB]);
        if (e + kAhead < 4 * OB) op[e % kAhead] = read_v(e + kAhead);
        if (e < 2 * OB) {
#pragma unroll
          for (int j = e * 8 / (2 * OB); j < (e + 1) * 8 / (2 * OB); ++j) weight_pair(1, j);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!last) stage_store(cur, st + 1, buf ^ 1);
      else if (have_next) stage_store(nxt, 0, buf ^ 1);
      par ^= 1;
      // after this stage's last LDS operand use: a scalar load in flight would
      // turn every LDS wait before it into a full one
      if constexpr (!last) stage_pages(cur, st + 2, pg);
      else if (have_next) stage_pages(nxt, 1, pg);
    };
    const int last_st = (cur.ntiles - 1) >> 1;
    for (int st = 0; st < last_st; ++st) stage(st, std::false_type{});
    stage(last_st, std::true_type{});

    const float l = col_sum32(l_run);
    if (ok) {
      const float inv = 1.0f / l;
      float* dst = a.out + orow * D + 4 * hf;
#pragma unroll
      for (int x = 0; x < OB; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          *reinterpret_cast<f32x4*>(dst + 32 * x + 8 * y) =
              f32x4{o[x][4 * y], o[x][4 * y + 1], o[x][4 * y + 2], o[x][4 * y + 3]} * inv;
    }
    if (!have_next) return;
    cur = nxt;
    ib ^= 1;
  }
}

constexpr int kNQ = 2;

// compute units of the current device (queried once)
int cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n = v;
    else
      return 256;
  }
  return n;
}

template <int D, bool FP8>
hipError_t launch_prefill_d(const dms_config& c, const Layout& lo, void* meta, void* ws, void* pool,
                            int layer, int n, const int32_t* seq_ids, const int32_t* cu,
                            int total_tokens, int max_len, const void* q, const void* k,
                            const void* v, const uint8_t* flags, float* out, hipStream_t st,
                            hipEvent_t ev_start, hipEvent_t ev_stop) {
  char* w = static_cast<char*>(ws);
  LayerState ls = layer_state(lo, meta, layer);
  PrefillArgs a;
  a.status = reinterpret_cast<const int32_t*>(static_cast<char*>(meta) + lo.status);
  a.seq_ids = seq_ids;
  a.cu = cu;
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.flags = flags;
  a.pool = static_cast<const char*>(pool);
  a.page_table = ls.page_table;
  a.slot_meta = ls.slot_meta;
  a.len = ls.len;
  a.pos = ls.pos;
  a.list = reinterpret_cast<int32_t*>(w + lo.ws_pf_meta);
  a.list_cnt = reinterpret_cast<int32_t*>(w + lo.ws_pf_cum);
  a.tiles = w + lo.ws_pf_tiles;
  a.tmeta = reinterpret_cast<uint32_t*>(w + lo.ws_pf_tmeta);
  a.zeros = w + lo.ws_pf_zeros;
  a.kept_before = reinterpret_cast<int32_t*>(w + lo.ws_pf_kb);
  a.rows = reinterpret_cast<PrefillRow*>(w + lo.ws_pf_order);
  a.first_item = reinterpret_cast<int32_t*>(a.rows + lo.max_heads);
  a.work_ctr = a.list_cnt + lo.max_heads;   // the word after the per-head counts
  a.nx = a.items = 0;
  a.tph = lo.pf_tiles_per_head;
  a.immediate = c.eviction == DMS_EVICT_IMMEDIATE;
  a.zero_neuron = c.decision_source == DMS_DECIDE_QUERY;
  a.out = out;
  a.page_bytes = lo.page_bytes;
  a.n = n;
  a.H = c.num_kv_heads;
  a.g = c.group_size;
  a.w = c.window;
  a.P = c.page_size;
  a.log2P = __builtin_ctz(static_cast<unsigned>(c.page_size));
  a.maxp = c.max_pages_per_head;
  a.max_slots = lo.max_slots;
  a.max_seqs = c.max_seqs;
  a.total = total_tokens;
  a.max_len = max_len;
  // positions per attention workgroup: its (position, head) columns, 32 per wave
  a.PB = attn_threads<D, FP8>() / 64 * 32 / c.group_size;
  a.scale_log2 = c.softmax_scale * 1.4426950408889634f;
  const int NH = n * c.num_kv_heads;
  // the timing events bracket every pass
  if (ev_start) (void)hipEventRecord(ev_start, st);
  hipError_t e = launch_chunk_scan(c, lo, meta, ws, layer, n, seq_ids, cu, total_tokens, max_len, flags, true, st);
  if (e != hipSuccess) return e;
  a.order = 1;
  hipLaunchKernelGGL((prefill_tile_kernel<D, FP8>), dim3(a.order + (max_len + 31) / 32, NH, 2), dim3(kThreads), 0,
                     st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 grid((max_len + a.PB - 1) / a.PB, NH);
  // as many workgroups as fit on the chip at once, each taking work items
  // until none is left
  a.nx = static_cast<int>(grid.x);
  a.items = a.nx * NH;
  const dim3 wgs(min(a.items, 512 / attn_threads<D, FP8>() * cu_count()));
  if (a.immediate)
    hipLaunchKernelGGL((prefill_kernel<D, kNQ, FP8>), wgs, dim3(attn_threads<D, FP8>()), 0, st, a);
  else
    hipLaunchKernelGGL((prefill_delayed_kernel<D, FP8>), wgs, dim3(attn_threads<D, FP8>()), 0, st, a);
  e = hipGetLastError();
  if (ev_stop) (void)hipEventRecord(ev_stop, st);
  return e;
}


// ---------------------------------------------------------------------------
// Chunked prefill over a latent-attention (MLA) cache: one KV head of
// 576-dim rows shared by the g query heads, in the absorbed form of the
// latent decode: column (position t, query head h) scores row j by q . row
// over all 576 dims and sums the rows' first 512 (latent) dims.  The mask and
// the three key sources are the standard prefill's.  Under delayed
// eviction prefill_mla_delayed_kernel attends; under immediate eviction
// prefill_mla_kernel: columns packed 16
// per MFMA block -- 16 / g positions x g heads for g <= 16, else one position
// x 16 of its heads -- and each of a workgroup's four waves takes one column
// block (its 16 x 512 float32 accumulators fill most of a wave's registers).
// Per 32-row tile staged in LDS a wave runs 36 score MFMAs, reading the rows
// in their stored fragment order, and 32 PV MFMAs whose V^T operand (8 rows
// of one latent dim per lane) comes from the LDS transpose read.
// ---------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef short v4i16 __attribute__((ext_vector_type(4)));

constexpr int kMlaThreads = 256;
constexpr int kMlaKSteps = kMlaDim / 32;                         // 18
constexpr int kMlaTileBytes = kMlaDim * 64;                      // 32 rows of 576 bf16
constexpr int kMlaPieces = kMlaTileBytes / 16 / kMlaThreads;     // staged 16-byte pieces per thread (9)
constexpr int kMlaOBlocks = kMlaLatent / 16;                     // 16-dim row blocks of O^T (32)
constexpr int kMlaScoreBatch = 3;                                // score k-steps whose operands are read together
static_assert(kMlaTileBytes % (16 * kMlaThreads) == 0, "tile staged evenly");

__device__ inline u32x2 tr_read16(const char* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                       (__attribute__((address_space(3))) v4i16*)(p)));
}

// Pass 1 for latent rows (one block per (32-token tile, sequence, region)):
// the chunk's rows in chunk order (region 0) and the kept ones in list order
// (region 1) into workspace tiles in the pool's layout; rows past the end
// are 0.
__global__ __launch_bounds__(kThreads) void prefill_tile_mla_kernel(PrefillArgs a) {
  if (load_status(a.status) != 0) return;
  const int k = blockIdx.x - a.order, i = blockIdx.y, region = blockIdx.z;
  if (k < 0) {
    if (region == 0) order_rows(a, i);
    return;
  }
  const int tok0 = a.cu[i], C = a.cu[i + 1] - a.cu[i];
  const int cnt = region ? a.list_cnt[i] : C;
  if (k * 32 >= cnt) return;
  const int32_t* lst = a.list + tok0;
  if (threadIdx.x < 32) {   // key rows, as prefill_tile_kernel writes them
    const int idx = 32 * k + threadIdx.x, p0 = a.pos[a.seq_ids[i]];
    uint32_t mt = kNoKey;
    if (idx < cnt)
      mt = region ? static_cast<uint32_t>(p0 + lst[idx])
                  : (static_cast<uint32_t>(p0 + idx) | (key_flag(a, tok0, C, idx, 0) ? kFlagBit : 0u));
    a.tmeta[ws_tile(a, region, 0, i, k) * 32 + threadIdx.x] = mt;
  }
  char* tile = a.tiles + ws_tile(a, region, 0, i, k) * kMlaTileBytes;
  constexpr int kRow = kMlaDim / 8;   // 16-byte pieces per row
  for (int pc = threadIdx.x; pc < 32 * kRow; pc += kThreads) {
    const int j = pc / kRow, e0 = 8 * (pc % kRow);
    const int idx = 32 * k + j;
    u32x4 x = {0u, 0u, 0u, 0u};
    if (idx < cnt) {
      const int c = region ? lst[idx] : idx;
      x = *reinterpret_cast<const u32x4*>(a.k + static_cast<size_t>(tok0 + c) * kMlaDim + e0);
    }
    *reinterpret_cast<u32x4*>(tile + k_elem_off(j, e0)) = x;
  }
}

__global__ __launch_bounds__(kMlaThreads, 1) void prefill_mla_kernel(PrefillArgs a) {
  __shared__ __attribute__((aligned(16))) char tile_lds[2][kMlaTileBytes];
  __shared__ uint32_t meta_lds[2][32];
  __shared__ int masked_lds[2];
  if (load_status(a.status) != 0) return;
  const int i = blockIdx.y;   // sequence of the call (one KV head)
  const int tok0 = a.cu[i], C = a.cu[i + 1] - a.cu[i];
  const int g = a.g;
  const int pcb = g <= kMaxGroup ? kMaxGroup / g : 1;     // positions per column block
  const int cgs = (g + kMaxGroup - 1) / kMaxGroup;        // column blocks per position set
  const int ncb = (C + pcb - 1) / pcb * cgs;
  const int cb0 = blockIdx.x * (kMlaThreads / 64);
  if (cb0 >= ncb) return;
  const int cb1 = min(cb0 + kMlaThreads / 64, ncb) - 1;
  const int s = a.seq_ids[i];
  const int sh = s;
  const int p0 = a.pos[s];
  const int L0 = a.len[sh];
  // the block's positions [t0, t1)
  const int t0 = p0 + (cb0 / cgs) * pcb;
  const int t1 = p0 + min(C, (cb1 / cgs + 1) * pcb);
  // band: chunk tiles from the one holding max(p0, t0 - w + 1) up to t1
  const int band_c0 = (max(0, t0 - a.w + 1 - p0) >> 5) << 5;   // chunk-local, < C
  // kept chunk keys strictly before the band (a prefix of the sorted list),
  // counted by pass 0
  const int32_t* lst = a.list + tok0;
  const int n_pre = a.kept_before[ws_kb(a, 0, i, band_c0 >> 5)];
  const int nc = (L0 + 31) >> 5;
  const int np = (n_pre + 31) >> 5;
  const int nb = (t1 - p0 - band_c0 + 31) >> 5;
  const char* pre_tiles = a.tiles + ws_tile(a, 1, 0, i, 0) * kMlaTileBytes;
  const char* band_tiles = a.tiles + ws_tile(a, 0, 0, i, band_c0 >> 5) * kMlaTileBytes;
  const int ntiles = nc + np + nb;
  const int32_t* pt = a.page_table + static_cast<size_t>(sh) * a.maxp;
  const int32_t* smeta = a.slot_meta + static_cast<size_t>(sh) * a.max_slots;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, G = lane >> 4;
  // ---- this wave's column block and this lane's column (position, head)
  const int cb = cb0 + wave;
  const bool active = cb < ncb;
  const int pbk = cb / cgs, hg = cb % cgs;
  int pl, qh;
  bool ok;
  if (g <= kMaxGroup) {
    pl = r / g;
    qh = r % g;
    ok = pl < pcb;
  } else {
    pl = 0;
    qh = kMaxGroup * hg + r;
    ok = qh < g;
  }
  const int cpos = pbk * pcb + pl;   // chunk-local position
  ok = ok && active && cpos < C;
  const int tcol = ok ? p0 + cpos : -1;
  u32x4 qf[kMlaKSteps];
  {
    const char* qrow = reinterpret_cast<const char*>(
        a.q + (static_cast<size_t>(tok0 + (ok ? cpos : 0)) * g + (ok ? qh : 0)) * kMlaDim);
#pragma unroll
    for (int s2 = 0; s2 < kMlaKSteps; ++s2)
      qf[s2] = ok ? *reinterpret_cast<const u32x4*>(qrow + (32 * s2 + 8 * G) * 2) : u32x4{0u, 0u, 0u, 0u};
  }

  // ---- staging: global -> registers, registers -> LDS (the tile as stored)
  u32x4 kx[kMlaPieces];
  uint32_t smt = kNoKey;
  auto stage_load = [&](int k) {
    const char* tile;
    if (k < nc) {
      const int sb = k * 32;
      tile = a.pool + static_cast<size_t>(pt[sb >> a.log2P]) * a.page_bytes +
             static_cast<size_t>((sb & (a.P - 1)) >> 5) * kMlaTileBytes;
      if (tid < 32) {
        uint32_t mt = sb + tid < L0 ? static_cast<uint32_t>(smeta[sb + tid]) : kNoKey;
        if (mt != kNoKey) {
          const int kp = static_cast<int>(mt & ~kFlagBit);
          const int x = kp + a.w - p0;
          mt = static_cast<uint32_t>(kp) |
               ((x >= 0 && x < C && a.flags[static_cast<size_t>(tok0 + x)]) ? kFlagBit : 0u);
        }
        smt = mt;
      }
    } else if (k < nc + np) {
      const int kk = k - nc;
      tile = pre_tiles + static_cast<size_t>(kk) * kMlaTileBytes;
      if (tid < 32) {
        const int idx = kk * 32 + tid;
        smt = idx < n_pre ? static_cast<uint32_t>(p0 + lst[idx]) : kNoKey;
      }
    } else {
      const int kb = k - nc - np;
      tile = band_tiles + static_cast<size_t>(kb) * kMlaTileBytes;
      if (tid < 32) {
        const int c = band_c0 + kb * 32 + tid;
        smt = c < t1 - p0 ? (static_cast<uint32_t>(p0 + c) | (key_flag(a, tok0, C, c, 0) ? kFlagBit : 0u))
                          : kNoKey;
      }
    }
#pragma unroll
    for (int m = 0; m < kMlaPieces; ++m) kx[m] = *reinterpret_cast<const u32x4*>(tile + (tid + m * kMlaThreads) * 16);
  };
  auto stage_store = [&](int k, int buf) {
    char* dst = tile_lds[buf];
    // pool slots past L hold stale bits (a freed page may hold NaNs): their
    // rows are zeroed, which zeroes them in the V^T operand too
    const int valid = k < nc ? min(32, L0 - k * 32) : 32;
#pragma unroll
    for (int m = 0; m < kMlaPieces; ++m) {
      const int P = tid + m * kMlaThreads;
      // piece P: 1 KB block P / 64 of half (P / 64) % 2, lane row P % 16
      const int pr = P & 15, row = 8 * (pr >> 2) + (pr & 3) + 4 * ((P >> 6) & 1);
      const u32x4 x = row < valid ? kx[m] : u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(dst + P * 16) = x;
    }
    if (tid < 64) {
      // a key row needs the per-element mask iff some query of the block does
      // not see it: padding, causal (position > t0) or flagged and expiring
      // by t1 - 1
      bool need = false;
      if (tid < 32) {
        const uint32_t mt = smt;
        const int kp = static_cast<int>(mt & ~kFlagBit);
        need = mt == kNoKey || kp > t0 || ((mt & kFlagBit) && kp + a.w <= t1 - 1);
        meta_lds[buf][tid] = mt;
      }
      const uint64_t any = __builtin_amdgcn_ballot_w64(need);
      if (tid == 0) masked_lds[buf] = any != 0;
    }
  };

  // ---- accumulators: O^T rows 16 b + 4G .. + 3 of column r
  f32x4 o[kMlaOBlocks];
#pragma unroll
  for (int b = 0; b < kMlaOBlocks; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref = kMInit, l_run = 0.f;
  const float thr = kRescale / a.scale_log2;   // rescale threshold in score units
  // transpose-read address of this lane in a tile (row block 0, rows 0-3 of
  // each 8): lane 16 G' + 4 j + q reads dims 4q .. 4q + 3 of row 8 G' + j
  const int tr_j = (lane & 15) >> 2, tr_q = lane & 3;
  const int tr_off = (tr_q >> 1) * 256 + (4 * G + tr_j) * 16 + 8 * (tr_q & 1);

  if (ntiles > 0) {
    stage_load(0);
    stage_store(0, 0);
  }
  __syncthreads();
  for (int k = 0; k < ntiles; ++k) {
    const int buf = k & 1;
    if (k + 1 < ntiles) stage_load(k + 1);
    const char* tl = tile_lds[buf];
    if (active) {
      // scores: the 36 A pieces (piece 2s + h: half h, k-step s) read in
      // batches, the next batch in flight while one is multiplied
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
      u32x4 kp2[2][2 * kMlaScoreBatch];
      const char* kl = tl + lane * 16;
#pragma unroll
      for (int e = 0; e < 2 * kMlaScoreBatch; ++e) kp2[0][e] = *reinterpret_cast<const u32x4*>(kl + e * 1024);
#pragma unroll
      for (int bt = 0; bt < kMlaKSteps / kMlaScoreBatch; ++bt) {
        if (bt + 1 < kMlaKSteps / kMlaScoreBatch) {
#pragma unroll
          for (int e = 0; e < 2 * kMlaScoreBatch; ++e)
            kp2[(bt + 1) & 1][e] = *reinterpret_cast<const u32x4*>(kl + (2 * kMlaScoreBatch * (bt + 1) + e) * 1024);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < kMlaScoreBatch; ++e) {
          s0 = mfma_bf16(kp2[bt & 1][2 * e], qf[kMlaScoreBatch * bt + e], s0);
          s1 = mfma_bf16(kp2[bt & 1][2 * e + 1], qf[kMlaScoreBatch * bt + e], s1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // lane (r, G): keys 8G .. 8G+3 (s0) and 8G+4 .. 8G+7 (s1) of column r
      float sc[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sc[j] = s0[j];
        sc[j + 4] = s1[j];
      }
      if (__builtin_amdgcn_readfirstlane(masked_lds[buf]) != 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t km = meta_lds[buf][8 * G + j];
          const int kpos = static_cast<int>(km & ~kFlagBit);
          const int kexp = (km & kFlagBit) ? kpos + a.w : 0x7FFFFFFF;
          sc[j] = (kpos <= tcol && tcol < kexp) ? sc[j] : -INFINITY;
        }
      }
      float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])),
                       fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
      mx = col_max(mx);
      const bool raise = mx > m_ref + thr;   // false while the column has seen no key
      if (__builtin_amdgcn_ballot_w64(raise)) {
        const float m_new = raise ? mx : m_ref;
        const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * a.scale_log2);
        l_run *= alpha;
#pragma unroll
        for (int b = 0; b < kMlaOBlocks; ++b) o[b] *= alpha;
        m_ref = m_new;
      }
      const float mb = m_ref * a.scale_log2;
      u32x4 pu;
      const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x2 pr = {__builtin_amdgcn_exp2f(fmaf(sc[2 * j], a.scale_log2, -mb)),
                          __builtin_amdgcn_exp2f(fmaf(sc[2 * j + 1], a.scale_log2, -mb))};
        const bf16x2 pb = __builtin_convertvector(pr, bf16x2);
        pu[j] = __builtin_bit_cast(uint32_t, pb);
        l_run = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, l_run, false);
      }
      // PV: V^T of latent row block b (dims 16 b ..), rows 8G .. 8G+7, from
      // the transpose read; four blocks' reads ahead of their products
#pragma unroll
      for (int b0 = 0; b0 < kMlaOBlocks; b0 += 4) {
        u32x4 vt[4];
#pragma unroll
        for (int i2 = 0; i2 < 4; ++i2) {
          const int b = b0 + i2;
          const char* base = tl + (b >> 1) * 2048 + (b & 1) * 512 + tr_off;
          const u32x2 lo = tr_read16(base), hi = tr_read16(base + 1024);
          vt[i2] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
        for (int i2 = 0; i2 < 4; ++i2) o[b0 + i2] = mfma_bf16(vt[i2], pu, o[b0 + i2]);
      }
    }
    if (k + 1 < ntiles) stage_store(k + 1, buf ^ 1);
    __syncthreads();
  }

  // ---- outputs
  float l = l_run;
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (tcol >= 0) {
    const float inv = 1.0f / l;
    float* dst = a.out + (static_cast<size_t>(tok0 + cpos) * g + qh) * kMlaLatent + 4 * G;
#pragma unroll
    for (int b = 0; b < kMlaOBlocks; ++b) *reinterpret_cast<f32x4*>(dst + 16 * b) = o[b] * inv;
  }
}

// Latent-attention pass under delayed eviction, 32x32 MFMA products: the work
// items, masks and copies of prefill_delayed_kernel, a wave holding 32
// (position, head) columns with their queries (144 registers) and 32 x 512
// accumulators (256), one wave per SIMD.  A 32-row tile is staged by hardware
// copies beside the attention of the tile before it and read twice: as rows
// for the scores, through the LDS transpose read for the values.  Inside each
// 1 KB block (32 dims of 16 rows) the copy permutes the 16-byte pieces, row r
// of dim group G to place r ^ 4 G, so that the four dim groups of a transpose
// read fall into different banks.  16x16 products read every operand for 16
// columns and were bound by those reads; now the matrix core is the bound,
// and, with one wave per SIMD, the softmax between its two products.  Four
// prompts of 4096 to 8192 tokens in chunks of 4096, 16 heads: 933 us with
// every pass, from 1703 us.
__global__ __launch_bounds__(kMlaThreads, 1) void prefill_mla_delayed_kernel(PrefillArgs a) {
  constexpr int NW = kMlaThreads / 64;
  constexpr int KS = kMlaDim / 16, OB = kMlaLatent / 32;
  __shared__ __attribute__((aligned(256))) char tile_lds[2][kMlaTileBytes];
  __shared__ __attribute__((aligned(16))) uint32_t meta_lds[2][64];   // rows 0..31 twice
  __shared__ int item_lds[2], first_lds[kOrderMax + 1];
  if (load_status(a.status) != 0) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5;
  const float thr = kRescale / a.scale_log2, sl2 = a.scale_log2;
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
  // operand addresses: rows of k-steps e, e even / odd, + 2048 (e / 2); columns of token half y, +
  // 2048 per 32-dim block, + 1024 for tokens 4-7 of the eight
  uint32_t k_addr[2], v_addr[2];
  {
    const int kt = row_token(lane & 31), r = 4 * (kt >> 3) + (kt & 3);
    const int G = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1), j = (lane & 15) >> 2;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int Gk = 2 * e + hf;
      k_addr[e] = lds_addr(tile_lds) + ((kt >> 2) & 1) * 1024 + Gk * 256 + (r ^ (4 * Gk)) * 16;
      v_addr[e] = lds_addr(tile_lds) + G * 256 + ((4 * (2 * e + hf) + j) ^ (4 * G)) * 16 + 8 * (lane & 1);
    }
  }
  const uint32_t piece = (lane ^ (4 * (lane >> 4))) * 16;   // source of a copy's lane in its 1 KB block

  const int NH = a.n;
  const bool ranked = NH <= kOrderMax;
  if (ranked)
    for (int x = tid; x <= NH; x += kMlaThreads) first_lds[x] = a.first_item[x];
  __syncthreads();
  const int items = ranked ? __builtin_amdgcn_readfirstlane(first_lds[NH]) : a.items;
  if (static_cast<int>(blockIdx.x) >= items) return;
  auto copy_tile = [&](const Item& it, int k, int page, int buf) {
    const char* tile;
    const uint32_t* mt;
    tile_source(a, it, k, page, kMlaTileBytes, tile, mt);
    const char* src = tile + wave * (kMlaTileBytes / NW) + piece;
    const uint32_t dst = lds_addr(tile_lds) + buf * kMlaTileBytes + wave * (kMlaTileBytes / NW);
#pragma unroll
    for (int m = 0; m < kMlaTileBytes / NW / 1024; ++m) lds_copy16(src + m * 1024, dst + m * 1024);
    if (wave == 0) lds_copy4(reinterpret_cast<const char*>(mt + (lane & 31)), lds_addr(meta_lds[buf]));
  };
  Item cur = prefill_item(a, first_lds, blockIdx.x, lane);
  copy_tile(cur, 0, pool_page(a, cur, 0), 0);
  int page = pool_page(a, cur, 1);
  int par = 0, ib = 0;   // LDS buffer of the present tile, slot of the next item's index

  const int col = wave * 32 + (lane & 31);
  const int pl = col / a.g, qh = col % a.g;
  while (true) {
    const bool ok = pl < a.PB && cur.t0 + pl < cur.t1;
    const int t = ok ? cur.t0 + pl : -1;
    const size_t orow = static_cast<size_t>(cur.tok0 + (ok ? t - cur.p0 : 0)) * a.g + qh;
    const size_t qrow = ok ? orow : 0;   // unused columns: any row (masked by t)
    u32x4 qf[KS];
#pragma unroll
    for (int x = 0; x < KS; ++x) qf[x] = *reinterpret_cast<const u32x4*>(a.q + qrow * kMlaDim + 16 * x + 8 * hf);
    f32x16 o[OB];
#pragma unroll
    for (int x = 0; x < OB; ++x)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[x][i] = 0.f;
    float m_ref = kMInit, l_run = 0.f;
    if (tid == 0) item_lds[ib] = gridDim.x + atomicAdd(a.work_ctr, 1);   // read after this item's last barrier
    Item nxt = cur;
    bool have_next = false;
    for (int k = 0; k < cur.ntiles; ++k) {
      const int buf = par;
      __builtin_amdgcn_s_waitcnt(wait_vm(0));
      __syncthreads();
      if (k + 1 < cur.ntiles) {
        copy_tile(cur, k + 1, page, buf ^ 1);
      } else {
        const int item = __builtin_amdgcn_readfirstlane(item_lds[ib]);
        have_next = item < items;
        if (have_next) {
          nxt = prefill_item(a, first_lds, item, lane);
          copy_tile(nxt, 0, pool_page(a, nxt, 0), buf ^ 1);
        }
      }
      const int rows = rows_of(cur, k);
      if (k == cur.nc - 1 && rows < 32) {
        // the pool's last tile: rows past the live length are stale (a freed page may hold NaNs)
        for (int P = tid; P < kMlaTileBytes / 16; P += kMlaThreads) {
          const int r = (P & 15) ^ (4 * ((P >> 4) & 3));
          if (8 * (r >> 2) + (r & 3) + 4 * ((P >> 6) & 1) >= rows)
            *reinterpret_cast<u32x4*>(tile_lds[buf] + P * 16) = u32x4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
      }
      uint32_t mrow = meta_lds[buf][lane & 31];
      if ((lane & 31) >= rows) mrow = kNoKey;
      const bool masked = __builtin_amdgcn_ballot_w64(row_hidden(mrow, cur, a.w)) != 0;
      const uint32_t tl = buf * kMlaTileBytes;
      const uint32_t ka[2] = {k_addr[0] + tl, k_addr[1] + tl}, va[2] = {v_addr[0] + tl, v_addr[1] + tl};
      // scores: two chains (even and odd k-steps), operands read ahead in pinned order
      f32x16 s, s1;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = s1[i] = 0.f;
      u32x4 op[kAhead];
      auto read_k = [&](int e) {
        return *reinterpret_cast<DMS_LDS const u32x4*>(ka[e & 1] + (e >> 1) * 2048);
      };
      auto read_v = [&](int e) {   // 32-dim block e % OB, token half e / OB
        const char* p = (const char*)(DMS_LDS const char*)(va[e / OB] + (e % OB) * 2048);
        const u32x2 lo = tr_read16(p), hi = tr_read16(p + 1024);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
      };
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < kAhead; ++e) op[e] = read_k(e);
#pragma unroll
      for (int e = 0; e < KS; ++e) {
        __builtin_amdgcn_sched_barrier(0);
        if (e & 1) s1 = mfma32(op[e % kAhead], qf[e], s1);
        else s = mfma32(op[e % kAhead], qf[e], s);
        if (e + kAhead < KS) op[e % kAhead] = read_k(e + kAhead);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < kAhead; ++e) op[e] = read_v(e);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] += s1[i];
      if (masked) mask_scores(s, &meta_lds[buf][8 * hf], rows, t, a.w, lane);
      float mx = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
      mx = col_max32(mx);
      const bool raise = mx > m_ref + thr;   // false while the column has seen no key
      uint64_t rescale = __builtin_amdgcn_ballot_w64(raise);
      if (rescale) {
        // not where no raised column has a sum yet, as in an item's first tile: 256 accumulators
        // through the vector registers are about 2 us (4 prompts of 4096 to 8192 tokens 959 -> 933 us)
        rescale = __builtin_amdgcn_ballot_w64(raise && col_sum32(l_run) > 0.f);
        if (!rescale) m_ref = raise ? mx : m_ref;
      }
      if (rescale) {
        const float m_new = raise ? mx : m_ref;
        const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * sl2);
        l_run *= alpha;
#pragma unroll
        for (int x = 0; x < OB; ++x)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            // in place: the compiler would move all accumulators at once and spill (the products
            // before and after are many instructions away, past every matrix core hazard)
            float v = o[x][i], u;
            asm volatile(
                "v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                : "+a"(v), "=&v"(u)
                : "v"(alpha));
            o[x][i] = v;
          }
        m_ref = m_new;
      }
      const float mb = m_ref * sl2;
      u32x4 pu[2];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const f32x2 pr = {__builtin_amdgcn_exp2f(fmaf(s[2 * j], sl2, -mb)),
                          __builtin_amdgcn_exp2f(fmaf(s[2 * j + 1], sl2, -mb))};
        const bf16x2 pb = __builtin_convertvector(pr, bf16x2);
        pu[j >> 2][j & 3] = __builtin_bit_cast(uint32_t, pb);
        l_run = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, l_run, false);
      }
#pragma unroll
      for (int e = 0; e < 2 * OB; ++e) {
        __builtin_amdgcn_sched_barrier(0);
        o[e % OB] = mfma32(op[e % kAhead], pu[e / OB], o[e % OB]);
        if (e + kAhead < 2 * OB) op[e % kAhead] = read_v(e + kAhead);
      }
      __builtin_amdgcn_sched_barrier(0);
      par ^= 1;
      if (k + 2 < cur.ntiles) page = pool_page(a, cur, k + 2);
    }
    if (have_next) page = pool_page(a, nxt, 1);

    const float l = col_sum32(l_run);
    if (ok) {
      const float inv = 1.0f / l;
      float* dst = a.out + orow * kMlaLatent + 4 * hf;
#pragma unroll
      for (int x = 0; x < OB; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          *reinterpret_cast<f32x4*>(dst + 32 * x + 8 * y) =
              f32x4{o[x][4 * y], o[x][4 * y + 1], o[x][4 * y + 2], o[x][4 * y + 3]} * inv;
    }
    if (!have_next) return;
    cur = nxt;
    ib ^= 1;
  }
}

hipError_t launch_prefill_mla(const dms_config& c, const Layout& lo, void* meta, void* ws, void* pool,
                              int layer, int n, const int32_t* seq_ids, const int32_t* cu,
                              int total_tokens, int max_len, const void* q, const void* k,
                              const uint8_t* flags, float* out, hipStream_t st, hipEvent_t ev_start,
                              hipEvent_t ev_stop) {
  char* w = static_cast<char*>(ws);
  LayerState ls = layer_state(lo, meta, layer);
  PrefillArgs a;
  a.status = reinterpret_cast<const int32_t*>(static_cast<char*>(meta) + lo.status);
  a.seq_ids = seq_ids;
  a.cu = cu;
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = nullptr;
  a.flags = flags;
  a.pool = static_cast<const char*>(pool);
  a.page_table = ls.page_table;
  a.slot_meta = ls.slot_meta;
  a.len = ls.len;
  a.pos = ls.pos;
  a.list = reinterpret_cast<int32_t*>(w + lo.ws_pf_meta);
  a.list_cnt = reinterpret_cast<int32_t*>(w + lo.ws_pf_cum);
  a.tiles = w + lo.ws_pf_tiles;
  a.tmeta = reinterpret_cast<uint32_t*>(w + lo.ws_pf_tmeta);
  a.zeros = w + lo.ws_pf_zeros;
  a.kept_before = reinterpret_cast<int32_t*>(w + lo.ws_pf_kb);
  a.rows = reinterpret_cast<PrefillRow*>(w + lo.ws_pf_order);
  a.first_item = reinterpret_cast<int32_t*>(a.rows + lo.max_heads);
  a.work_ctr = a.list_cnt + lo.max_heads;
  a.nx = a.items = 0;
  a.tph = lo.pf_tiles_per_head;
  a.immediate = c.eviction == DMS_EVICT_IMMEDIATE;
  a.zero_neuron = 0;
  a.out = out;
  a.page_bytes = lo.page_bytes;
  a.n = n;
  a.H = 1;
  a.g = c.group_size;
  a.w = c.window;
  a.P = c.page_size;
  a.log2P = __builtin_ctz(static_cast<unsigned>(c.page_size));
  a.maxp = c.max_pages_per_head;
  a.max_slots = lo.max_slots;
  a.max_seqs = c.max_seqs;
  a.total = total_tokens;
  a.max_len = max_len;
  a.PB = kMlaThreads / 64 * 32 / c.group_size;   // positions per workgroup: 32 columns per wave
  a.scale_log2 = c.softmax_scale * 1.4426950408889634f;
  // the timing events bracket every pass
  if (ev_start) (void)hipEventRecord(ev_start, st);
  hipError_t e = launch_chunk_scan(c, lo, meta, ws, layer, n, seq_ids, cu, total_tokens, max_len, flags, true, st);
  if (e != hipSuccess) return e;
  a.order = !a.immediate;
  hipLaunchKernelGGL(prefill_tile_mla_kernel, dim3(a.order + (max_len + 31) / 32, n, 2), dim3(kThreads), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!a.immediate) {
    a.nx = (max_len + a.PB - 1) / a.PB;
    a.items = a.nx * n;
    hipLaunchKernelGGL(prefill_mla_delayed_kernel, dim3(min(a.items, cu_count())), dim3(kMlaThreads), 0, st, a);
    e = hipGetLastError();
    if (ev_stop) (void)hipEventRecord(ev_stop, st);
    return e;
  }
  const int g = c.group_size;
  const int pcb = g <= kMaxGroup ? kMaxGroup / g : 1;
  const int cgs = (g + kMaxGroup - 1) / kMaxGroup;
  const int ncb = (max_len + pcb - 1) / pcb * cgs;
  const int per_block = kMlaThreads / 64;
  hipLaunchKernelGGL(prefill_mla_kernel, dim3((ncb + per_block - 1) / per_block, n), dim3(kMlaThreads), 0, st, a);
  e = hipGetLastError();
  if (ev_stop) (void)hipEventRecord(ev_stop, st);
  return e;
}

}  // namespace

hipError_t launch_prefill_decide(const dms_config& c, const void* q, int total_tokens,
                                 uint8_t* flags, hipStream_t st) {
  const int64_t n = static_cast<int64_t>(total_tokens) * c.num_kv_heads;
  const int blocks = static_cast<int>((n + kThreads - 1) / kThreads);
  hipLaunchKernelGGL(prefill_decide_kernel, dim3(blocks), dim3(kThreads), 0, st,
                     static_cast<const uint16_t*>(q), flags, total_tokens, c.num_kv_heads,
                     c.group_size, c.head_dim, c.decision_bias);
  return hipGetLastError();
}

hipError_t launch_prefill_attention(const dms_config& c, const Layout& lo, void* meta, void* ws,
                                    void* pool, int layer, int n, const int32_t* seq_ids,
                                    const int32_t* cu, int total_tokens, int max_len,
                                    const void* q, const void* k, const void* v,
                                    const uint8_t* flags, float* out, hipStream_t st,
                                    hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (c.kv_format == DMS_KV_MLA)
    return launch_prefill_mla(c, lo, meta, ws, pool, layer, n, seq_ids, cu, total_tokens, max_len, q, k, flags,
                              out, st, ev_start, ev_stop);
  const bool fp8 = c.kv_format == DMS_KV_FP8;
  if (c.head_dim == 128)
    return fp8 ? launch_prefill_d<128, true>(c, lo, meta, ws, pool, layer, n, seq_ids, cu, total_tokens,
                                             max_len, q, k, v, flags, out, st, ev_start, ev_stop)
               : launch_prefill_d<128, false>(c, lo, meta, ws, pool, layer, n, seq_ids, cu, total_tokens,
                                              max_len, q, k, v, flags, out, st, ev_start, ev_stop);
  return fp8 ? launch_prefill_d<64, true>(c, lo, meta, ws, pool, layer, n, seq_ids, cu, total_tokens,
                                          max_len, q, k, v, flags, out, st, ev_start, ev_stop)
             : launch_prefill_d<64, false>(c, lo, meta, ws, pool, layer, n, seq_ids, cu, total_tokens,
                                           max_len, q, k, v, flags, out, st, ev_start, ev_stop);
}

}  // namespace dms
