// Training-time DMS attention with continuous decisions, gfx950.
//
// Sec. 3.1 (Eq. 1, Fig. 1b): each key j of a KV head carries alpha_j in
// [0, 1]; the scaled scores of every query head reading that KV head get the
// additive mask M_alpha: -inf for j > t, 0 for the w most recent positions
// (j > t - w, delayed eviction), log(1 - alpha_j) for older keys.  The mask
// is never materialised: the key's bias travels with its tile, and tiles are
// classified per block of queries as entirely old (bias per key), entirely
// inside the window (no bias) or mixed (per-element select).
//
// Passes (all MFMA v_mfma_f32_32x32x16_bf16, fp32 accumulation):
//   bias   -- log2(1 - alpha) per key, token order per head;
//   fwd    -- query-major online softmax, as in the masked prefill: out, lse;
//   dq     -- query-major: D_t = sum_d dout * out, recompute P, dP = dO V^T,
//             dS = P (dP - D), dQ = scale dS K;
//   dkv    -- key-major: each wave keeps 32 keys' K and V operands in
//             registers and walks the query tiles of every query head of the
//             group: dV = P^T dO, dK = scale dS^T Q and
//             dalpha_j = -sum_t exp(s_tj - lse_t) (dP_tj - D_t) over t >= j + w
//             (the probability without the (1 - alpha_j) factor, so the
//             gradient stays finite where alpha_j = 1).
// What bounds them: instruction issue and operand latency beside the matrix
// core (about half busy in each).  32x32 products take half the MFMA and LDS
// read instructions per key of 16x16 ones.  One layer of 8 x 5 heads, 2 x
// 8192 tokens, w = 256, before (16x16 products on tiles re-laid in memory by a
// pass of their own) and now: forward 1836 -> 1390 us (990 TFLOP/s), dQ 4005
// -> 1800 us (1150 of its three products), dK / dV 5160 -> 2540 us (1080 of
// its four), tiling and row sums 380 us -> none; the clock drops under the
// matrix core, so that single runs lie within 4 % of these.  Operands read
// ahead in pinned order are 2 to 4 % of each pass here, 6 to 14 % with 1777
// tokens of 2 heads.
// Pairing each tile's weights with the next tile's scores and the last tile's
// value products in one scheduled stretch ran 1540 to 1700 us forward: the
// second wave of a SIMD already fills the gaps, and the tile-by-tile barriers
// cost more.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dms_common.h"
#include "dms_train.h"

namespace dms {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef short v4i16 __attribute__((ext_vector_type(4)));

#define DMS_LDS __attribute__((address_space(3)))

constexpr int kThreads = 256;
constexpr int kTrainD = kTrainHeadDim;
constexpr int kRowB = kTrainD * 2;    // bytes of one bf16 row
constexpr int kUnit = 32 * kRowB;     // one 32-token tile of one tensor in LDS (8 KB)
constexpr int kStage = 4 * kUnit;     // one staged step: two tensors x two tiles
constexpr int kKS = kTrainD / 16;     // k-steps of a product over the head dimension
constexpr int kDB = kTrainD / 32;     // 32-dim blocks of a head
constexpr float kRescale = 8.0f;      // lazy rescale threshold, log2 units
constexpr float kMInit = -1.0e30f;    // running max before the first visible key
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ inline f32x16 mfma(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ inline u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }

// max / sum over the two lanes of one column (l and l + 32)
__device__ inline float col_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ inline float col_sum(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// The dispatcher deals workgroups to the 8 XCDs round-robin by linear id, and
// each XCD has its own L2.  Map the linear id so that the workgroups one XCD
// receives, in dispatch order, are a contiguous range of logical ids
// (x fastest): the blocks of one (sequence, head) then share an L2 and start
// together.
constexpr int kXcds = 8;
__device__ inline int2 xcd_order() {
  const int nx = gridDim.x;
  const int N = nx * gridDim.y;
  const int id = blockIdx.x + nx * blockIdx.y;
  const int x = id % kXcds, k = id / kXcds;
  const int L = x * (N / kXcds) + min(x, N % kXcds) + k;
  return int2{L % nx, L / nx};
}

// 8 fp32 values -> 4 packed bf16 pairs (round to nearest even)
__device__ inline u32x4 pack_bf16(const float* e) {
  u32x4 u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const f32x2 pr = {e[2 * j], e[2 * j + 1]};
    u[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
  }
  return u;
}

// ---------------------------------------------------------------------------
// LDS tiles.  A 32-token tile of one head is staged row-major (256 bytes a
// token) straight from the [B, T, heads, D] input by global -> LDS copies,
// its 16-byte pieces permuted inside each row: piece dg of token t lies at
// t * 256 + 16 (dg ^ x(t)), x(t) = 4 (t % 4) + (t / 4) % 4.  Both operand
// reads then spread over all 64 banks:
//   rows (a product over dims): lane l of k-step s takes dims 16 s + 8 (l / 32)
//     .. + 7 of token row_token(l % 32) with one 16-byte read;
//   columns (a product over tokens): lane l of (dim block b, half s) takes
//     tokens 16 s + 8 (l / 32) .. + 7 of dim 32 b + l % 32 with two LDS
//     transpose reads (ds_read_b64_tr_b16: in a 16-lane group, lane 4 j + q
//     passes the address of dims 4 q .. of token j and lane i receives dim i).
// Measured with eight waves reading: 4.0 cycles per wave read for both (256
// bytes a cycle for rows), 7.6 or more for the transpose reads of the
// unpermuted or t % 16-permuted rows.  Against tiles re-laid in memory by a
// pass of their own (row part and transposed part) this halves the staged
// bytes of the key-major pass and saves the pass.
// row_token orders the rows of a score MFMA so that accumulator registers
// 8 s .. 8 s + 7 of a lane are tokens 16 s + 8 (l / 32) .. + 7: exactly the B
// operand of half s of the next product.
// ---------------------------------------------------------------------------
__device__ inline int row_token(int r) {
  return 16 * (r >> 4) + 8 * ((r >> 2) & 1) + 4 * ((r >> 3) & 1) + (r & 3);
}

// Per-lane byte offsets; the others follow by an exclusive or (offsets of
// rows are multiples of 256, so it stays inside a row).
struct LaneOffsets {
  uint32_t row;   // row operand of k-step 0; k-step s: ^ 32 s
  uint32_t col;   // column operand of dim block 0, tokens 0-3 of the eight; block b: ^ 64 b,
                  // tokens 4-7: ^ 16, + 1024
  uint32_t src;   // source of copy 0 (rows 0 .. 3); copy m (rows 4 m ..): ^ 16 (m % 4)
};

__device__ inline LaneOffsets lane_offsets(int lane, uint32_t row_stride) {
  LaneOffsets o;
  const int hf = lane >> 5;
  const int t = row_token(lane & 31);
  o.row = t * kRowB + 16 * (hf ^ (4 * (t & 3) + ((t >> 2) & 3)));
  const int blk = (lane >> 4) & 1, j = (lane & 15) >> 2, q = lane & 3;
  o.col = (8 * hf + j) * kRowB + 16 * ((2 * blk + (q >> 1)) ^ (4 * j + 2 * hf)) + 8 * (q & 1);
  const int tr = lane >> 4, c = lane & 15;
  o.src = tr * row_stride + 16 * (c ^ (4 * tr));
  return o;
}

__device__ inline uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DMS_LDS const char*)p));
}
// 64 lanes x 16 bytes (4 bytes) from base + off (per lane), or src (per lane), to LDS m0 + 16 (4) lane.  The LDS
// destination goes in M0, written by the same statement; nothing else in this
// file reads M0.  The compiler does not count these loads: the kernels wait
// for them (vmcnt) before the barrier that publishes a stage.
__device__ inline void lds_copy16(const void* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(m0), "v"(off), "s"(base) : "memory", "m0");
}
__device__ inline void lds_copy16(const void* src, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(m0), "v"(src) : "memory", "m0");
}
__device__ inline void lds_copy4(const void* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" : : "s"(m0), "v"(off), "s"(base) : "memory", "m0");
}
__device__ inline void wait_copies() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// keeps the compiler from forming what follows from x ahead of a loop and holding it
__device__ inline int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// One wave copies rows t0 .. t0 + 31 of one head (row t at base + t * stride
// bytes) to the LDS tile `dst`.  Rows from `end` on are copied from 16 zero
// bytes: their weights are 0, and 0 times an Inf or NaN of some token must not
// reach the sums.
__device__ inline void copy_tile(const char* base, int t0, int end, uint32_t stride, const LaneOffsets& o,
                                 int lane, uint32_t dst, const void* zeros) {
  if (t0 + 32 <= end) {
    const char* src = base + static_cast<size_t>(t0) * stride;
#pragma unroll
    for (int m = 0; m < 8; ++m) lds_copy16(src + static_cast<size_t>(4 * m) * stride, o.src ^ (16 * (m & 3)), dst + 1024 * m);
  } else {
    const int ln = fresh(lane);   // formed here, not held ahead of the loop
    const int tr = ln >> 4, c = ln & 15;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int t = t0 + 4 * m + tr;
      const char* p = base + static_cast<size_t>(t) * stride + 16 * (c ^ (4 * tr + (m & 3)));
      lds_copy16(t < end ? p : static_cast<const char*>(zeros), dst + 1024 * m);
    }
  }
}

// Operand reads of the LDS tile at byte address `t` (a multiple of 256).
__device__ inline u32x4 row_operand(uint32_t t, const LaneOffsets& o, int s) {
  return *reinterpret_cast<DMS_LDS const u32x4*>((t + o.row) ^ (32 * s));
}
__device__ inline u32x2 tr_read16(uint32_t p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<DMS_LDS v4i16*>(p)));
}
// column operand of dim block b, token half s
__device__ inline u32x4 col_operand(uint32_t t, const LaneOffsets& o, int b, int s) {
  const u32x2 lo = tr_read16(((t + o.col) ^ (64 * b)) + 16 * s * kRowB);
  const u32x2 hi = tr_read16(((t + o.col) ^ (64 * b) ^ 16) + 16 * s * kRowB + 1024);
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}
// Every operand address of a lane in the tile at LDS byte address 0: passes
// with registers to spare hold them, so that a read is one instruction with
// the tile as its immediate offset (formed per read they were a sixth of the
// forward's VALU instructions).
struct LaneAddresses {
  uint32_t row[kKS], col[kDB][2];
};
__device__ inline LaneAddresses lane_addresses(uint32_t t, const LaneOffsets& o) {
  LaneAddresses r;
#pragma unroll
  for (int s = 0; s < kKS; ++s) r.row[s] = (t + o.row) ^ (32 * s);
#pragma unroll
  for (int b = 0; b < kDB; ++b) {
    r.col[b][0] = (t + o.col) ^ (64 * b);
    r.col[b][1] = ((t + o.col) ^ (64 * b) ^ 16) + 1024;
  }
  return r;
}
__device__ inline u32x4 row_operand(int tile, const LaneAddresses& r, int s) {
  return *reinterpret_cast<DMS_LDS const u32x4*>(r.row[s] + tile);
}
__device__ inline u32x4 col_operand(int tile, const LaneAddresses& r, int b, int s) {
  const u32x2 lo = tr_read16(r.col[b][0] + tile + 16 * s * kRowB);
  const u32x2 hi = tr_read16(r.col[b][1] + tile + 16 * s * kRowB);
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}
// keeps the compiler from forming (and holding) every operand address ahead of the loop
__device__ inline void refresh(LaneOffsets& o) { asm volatile("" : "+v"(o.row), "+v"(o.col), "+v"(o.src)); }

// Operands are read kAhead MFMAs ahead of their use, in an order pinned step
// by step (sched_barrier): left alone the compiler reads most operands right
// before their MFMA and waits out the LDS latency every time.
constexpr int kAhead = 4;
// Scheduling order of a stretch of M MFMAs: P LDS reads ahead, then R reads
// beside each (bounds the operands in flight, so that the accumulators and the
// resident operands fit without spills).
template <int P, int M, int R>
__device__ __forceinline__ void paced() {
  __builtin_amdgcn_sched_group_barrier(0x100, P, 0);
#pragma unroll
  for (int i = 0; i < M; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
  }
}
// Key-major pass, whose sums and operands leave few registers: its score
// products are paced (pinned, they ran 2680 against 2437 us), its sums pinned
// with two operands ahead (2437 against 2495 us paced, and 72 against 84 where
// splits leave one wave per SIMD or fewer).
constexpr int kFew = 2;

// ---------------------------------------------------------------------------
// Shared arguments of the attention passes
// ---------------------------------------------------------------------------
struct TrainArgs {
  const uint16_t* q;       // [B, T, Hq, D]
  const uint16_t* k;       // [B, T, H, D]
  const uint16_t* v;
  const uint16_t* dout;    // [B, T, Hq, D]
  const float* alpha;      // [B, T, H]
  const float* out;        // [B, T, Hq, D]
  const float* lse;        // [B, Hq, T]
  float* bias;             // [B, H, 64 nst]: key biases in raw score units
  float* nlse;             // [B, Hq, 32 nt]: -lse / scale (raw score units), -inf past the last token
  float* nsum;             // [B, Hq, 32 nt]: -sum_d dout * out, 0 past the last token
  float* zeros;            // 16 zero bytes
  float* part;             // [sets] of (dk, dv [B, T, H, D], dalpha [B, T, H])
  float* o_out;
  float* lse_out;
  float* dq;
  float* dk;
  float* dv;
  float* dalpha;
  size_t part_stride;      // floats of one set
  int B, T, H, g, w, nt, nst, PB;
  int splits;              // shares of a key block's steps (key-major pass)
  int split0, count, sets; // of them this launch: the first, how many, and how many go to `part`
  float scale_log2;        // softmax scale * log2(e)
};

// Key bias log2(1 - alpha) / (scale * log2 e): in raw score units, so that
// adding it to q.k and scaling gives log2 of the weight (-inf at alpha = 1).
// Written per (sequence, head) in token order, 0 past the last token.
__global__ __launch_bounds__(kThreads) void train_bias_kernel(TrainArgs a, bool backward) {
  const int n = 64 * a.nst;
  const int j = blockIdx.x * kThreads + threadIdx.x;
  if (j >= n) return;
  if (blockIdx.y == 0 && j < 4) a.zeros[j] = 0.f;
  const int b = blockIdx.y / a.H, h = blockIdx.y % a.H;
  float x = 0.f;
  if (j < a.T) x = __log2f(1.0f - a.alpha[(static_cast<size_t>(b) * a.T + j) * a.H + h]) / a.scale_log2;
  a.bias[static_cast<size_t>(blockIdx.y) * n + j] = x;
  if (backward && j >= a.T && j < 32 * a.nt)   // rows past the last token weigh nothing
    for (int i = 0; i < a.g; ++i) {
      const size_t ni = (static_cast<size_t>(blockIdx.y) * a.g + i) * 32 * a.nt + j;
      a.nlse[ni] = -INFINITY;
      a.nsum[ni] = 0.f;
    }
}

// Mask class of keys [j0, j1) for queries [q0, q1): 0 = every key older
// than every query's window (bias log(1 - alpha)), 1 = every key inside every
// query's window and not after any query (no bias), 2 = per element.
__device__ inline int mask_class(int j0, int j1, int q0, int q1, int w) {
  if (j1 - 1 <= q0 - w) return 0;
  if (j0 > q1 - 1 - w && j1 - 1 <= q0) return 1;
  return 2;
}

// Scores of one 32-key tile for a wave's 32 columns: register i of a lane is
// key jt + 16 (i / 8) + 8 (lane / 32) + i % 8.  The bias of old keys starts the
// accumulation (class 0; zeros otherwise); mixed tiles (class 2) are masked
// after it, t < 0 (unused column) hiding every key.
__device__ inline f32x16 score_start(const float* bias, const float* zeros, int cls, int hf) {
  const float* c = (cls == 0 ? bias : zeros) + 8 * hf;
  f32x16 s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(c + 16 * (i >> 1) + 4 * (i & 1));
#pragma unroll
    for (int e = 0; e < 4; ++e) s[4 * i + e] = x[e];
  }
  return s;
}
__device__ inline void score_mask(f32x16& s, const float* bias, int jt, int t, int w, int hf) {
  const int d = t - jt - 8 * hf;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 bv = *reinterpret_cast<const f32x4*>(bias + 16 * (i >> 1) + 8 * hf + 4 * (i & 1));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 16 * (i >> 1) + 4 * (i & 1) + e;
      s[4 * i + e] = k > d ? -INFINITY : (k > d - w ? s[4 * i + e] : s[4 * i + e] + bv[e]);
    }
  }
}

// ---------------------------------------------------------------------------
// Forward.  Workgroup = (sequence b, KV head h, block of PB query positions);
// columns are (position, query head) pairs, the g heads of a position
// consecutive, 32 per wave (a position's heads may straddle two waves).  Key
// tiles 0 .. ceil(t1 / 32) - 1 (causal) go through LDS two at a time, the next
// two being copied while these are attended: one barrier per 64 keys.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads, 2) void train_fwd_kernel(TrainArgs a) {
  __shared__ __attribute__((aligned(256))) char tile_lds[2][kStage];   // [K tile | V tile] x 2
  __shared__ __attribute__((aligned(16))) float bias_lds[2][64], zero_lds[32];
  if (threadIdx.x < 32) zero_lds[threadIdx.x] = 0.f;
  const int2 wg = xcd_order();               // latest (longest) query blocks first
  const int bh = wg.y;
  const int b = bh / a.H, h = bh % a.H;
  const int t0 = (gridDim.x - 1 - wg.x) * a.PB;
  if (t0 >= a.T) return;
  const int t1 = min(a.T, t0 + a.PB);
  const int ntiles = (t1 + 31) >> 5;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5;
  const int Hq = a.H * a.g;

  const int col = wave * 32 + (lane & 31);
  const int pl = col / a.g, qh = col % a.g;
  const bool ok = pl < a.PB && t0 + pl < t1;
  const int t = ok ? t0 + pl : -1;
  const size_t row = (static_cast<size_t>(b) * a.T + (ok ? t : 0)) * Hq + h * a.g + qh;
  u32x4 qf[kKS];
#pragma unroll
  for (int x = 0; x < kKS; ++x)
    qf[x] = ok ? ld16(a.q + row * kTrainD + 16 * x + 8 * hf) : u32x4{0u, 0u, 0u, 0u};

  const uint32_t stride = a.H * kRowB;
  LaneOffsets lo = lane_offsets(lane, stride);
  const uint32_t tiles = lds_addr(tile_lds);
  const LaneAddresses ad = lane_addresses(tiles, lo);
  const char* kv = reinterpret_cast<const char*>((wave >> 1 ? a.v : a.k) + (static_cast<size_t>(b) * a.T * a.H + h) * kTrainD);
  const float* bias = a.bias + static_cast<size_t>(bh) * 64 * a.nst;
  const int end = min(a.T, 32 * ntiles);   // a second tile past the block's last one is not read
  auto issue = [&](int st, int buf) {
    copy_tile(kv, 64 * st + 32 * (wave & 1), end, stride, lo, lane,
              tiles + buf * kStage + 2 * kUnit * (wave & 1) + kUnit * (wave >> 1), a.zeros);
    if (wave == 0) lds_copy4(bias + 64 * st, 4 * lane, lds_addr(bias_lds[buf]));
  };

  f32x16 o[kDB];
#pragma unroll
  for (int x = 0; x < kDB; ++x)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[x][i] = 0.f;
  float m_ref = kMInit, l_run = 0.f;
  const float thr = kRescale / a.scale_log2;
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);

  issue(0, 0);
  auto attend = [&](int st, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    wait_copies();
    __syncthreads();
    if (2 * st + 2 < ntiles) issue(st + 1, buf ^ 1);
    // 64 keys at a time: both tiles' scores, one maximum and (rare) rescale, the weights, both
    // tiles' products (a second tile past the last is hidden: every key is after t)
    constexpr int tl = buf * kStage;
    const int jt = 64 * st;
    const int c0 = mask_class(jt, jt + 32, t0, t1, a.w), c1 = mask_class(jt + 32, jt + 64, t0, t1, a.w);
    f32x16 s[2] = {score_start(&bias_lds[buf][0], zero_lds, c0, hf), score_start(&bias_lds[buf][32], zero_lds, c1, hf)};
    u32x4 op[kAhead];
    // score product e: tile e % 2, k-step e / 2 (the two chains take turns)
#pragma unroll
    for (int e = 0; e < kAhead; ++e) op[e] = row_operand(tl + 2 * kUnit * (e & 1), ad, e >> 1);
#pragma unroll
    for (int e = 0; e < 2 * kKS; ++e) {
      __builtin_amdgcn_sched_barrier(0);
      s[e & 1] = mfma(op[e % kAhead], qf[e >> 1], s[e & 1]);
      if (e + kAhead < 2 * kKS) op[e % kAhead] = row_operand(tl + 2 * kUnit * (e & 1), ad, (e + kAhead) >> 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (c0 == 2) score_mask(s[0], &bias_lds[buf][0], jt, t, a.w, hf);
    if (c1 == 2) score_mask(s[1], &bias_lds[buf][32], jt + 32, t, a.w, hf);
    float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(fmaxf(mx, s[0][i]), s[1][i]);
    mx = col_max(mx);
    const bool raise = mx > m_ref + thr;
    if (__builtin_amdgcn_ballot_w64(raise)) {
      const float m_new = raise ? mx : m_ref;
      const float alpha_s = __builtin_amdgcn_exp2f((m_ref - m_new) * a.scale_log2);
      l_run *= alpha_s;
#pragma unroll
      for (int x = 0; x < kDB; ++x) o[x] *= alpha_s;
      m_ref = m_new;
    }
    const float mb = m_ref * a.scale_log2;
    // the denominator adds the bf16-rounded weights the MFMA uses (dot
    // with (1, 1) on each packed pair as it is made)
    u32x4 pu[2][2];
    auto weight_pair = [&](int u, int j) {
      const f32x2 pr = {__builtin_amdgcn_exp2f(fmaf(s[u][2 * j], a.scale_log2, -mb)),
                        __builtin_amdgcn_exp2f(fmaf(s[u][2 * j + 1], a.scale_log2, -mb))};
      const bf16x2 pb = __builtin_convertvector(pr, bf16x2);
      pu[u][j >> 2][j & 3] = __builtin_bit_cast(uint32_t, pb);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, l_run, false);
    };
#pragma unroll
    for (int j = 0; j < 8; ++j) weight_pair(0, j);
    // value product e: tile e / 8, token half (e / 4) % 2, dim block e % 4; the
    // second tile's weights are formed beside the first one's products
    auto read_v = [&](int e) {
      return col_operand(tl + 2 * kUnit * (e / (2 * kDB)) + kUnit, ad, e % kDB, (e / kDB) % 2);
    };
#pragma unroll
    for (int e = 0; e < kAhead; ++e) op[e] = read_v(e);
#pragma unroll
    for (int e = 0; e < 4 * kDB; ++e) {
      __builtin_amdgcn_sched_barrier(0);
      o[e % kDB] = mfma(op[e % kAhead], pu[e / (2 * kDB)][(e / kDB) % 2], o[e % kDB]);
      if (e + kAhead < 4 * kDB) op[e % kAhead] = read_v(e + kAhead);
      if (e < 8) weight_pair(1, e);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int st = 0; 2 * st < ntiles; st += 2) {
    attend(st, std::integral_constant<int, 0>{});
    if (2 * st + 2 < ntiles) attend(st + 1, std::integral_constant<int, 1>{});
  }

  const float l = col_sum(l_run);
  if (ok) {
    float* dst = a.o_out + row * kTrainD + 4 * hf;
    const float inv = 1.0f / l;
#pragma unroll
    for (int x = 0; x < kDB; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y)
        *reinterpret_cast<f32x4*>(dst + 32 * x + 8 * y) =
            f32x4{o[x][4 * y], o[x][4 * y + 1], o[x][4 * y + 2], o[x][4 * y + 3]} * inv;
    if (hf == 0)
      a.lse_out[(static_cast<size_t>(b) * Hq + h * a.g + qh) * a.T + t] =
          (m_ref * a.scale_log2 + __log2f(l)) * kLn2;
  }
}

// ---------------------------------------------------------------------------
// dQ pass.  Same workgroups and columns as the forward; it also forms each
// row's sum of dout * out and hands that and lse, negated and in the units
// that start the key-major pass's products, to that pass.  Per key tile:
// S^T = K Q^T and dP^T = V dO^T over rows, dQ^T += K^T dS^T over columns.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads, 2) void train_dq_kernel(TrainArgs a) {
  __shared__ __attribute__((aligned(256))) char tile_lds[2][kStage];
  __shared__ __attribute__((aligned(16))) float bias_lds[2][64], zero_lds[32];
  if (threadIdx.x < 32) zero_lds[threadIdx.x] = 0.f;
  const int2 wg = xcd_order();
  const int bh = wg.y;
  const int b = bh / a.H, h = bh % a.H;
  const int t0 = (gridDim.x - 1 - wg.x) * a.PB;
  if (t0 >= a.T) return;
  const int t1 = min(a.T, t0 + a.PB);
  const int ntiles = (t1 + 31) >> 5;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5;
  const int Hq = a.H * a.g;

  const int col = wave * 32 + (lane & 31);
  const int pl = col / a.g, qh = col % a.g;
  const bool ok = pl < a.PB && t0 + pl < t1;
  const int t = ok ? t0 + pl : -1;
  const size_t row = (static_cast<size_t>(b) * a.T + (ok ? t : 0)) * Hq + h * a.g + qh;

  const uint32_t stride = a.H * kRowB;
  LaneOffsets lo = lane_offsets(lane, stride);
  const uint32_t tiles = lds_addr(tile_lds);
  const LaneAddresses ad = lane_addresses(tiles, lo);
  const char* kv = reinterpret_cast<const char*>((wave >> 1 ? a.v : a.k) + (static_cast<size_t>(b) * a.T * a.H + h) * kTrainD);
  const float* bias = a.bias + static_cast<size_t>(bh) * 64 * a.nst;
  const int end = min(a.T, 32 * ntiles);   // a second tile past the block's last one is not read
  auto issue = [&](int st, int buf) {
    copy_tile(kv, 64 * st + 32 * (wave & 1), end, stride, lo, lane,
              tiles + buf * kStage + 2 * kUnit * (wave & 1) + kUnit * (wave >> 1), a.zeros);
    if (wave == 0) lds_copy4(bias + 64 * st, 4 * lane, lds_addr(bias_lds[buf]));
  };
  issue(0, 0);

  u32x4 qf[kKS], df[kKS];
  float dcol = 0.f;
#pragma unroll
  for (int x = 0; x < kKS; ++x) {
    qf[x] = ok ? ld16(a.q + row * kTrainD + 16 * x + 8 * hf) : u32x4{0u, 0u, 0u, 0u};
    df[x] = ok ? ld16(a.dout + row * kTrainD + 16 * x + 8 * hf) : u32x4{0u, 0u, 0u, 0u};
    if (ok) {
      const f32x4 o0 = *reinterpret_cast<const f32x4*>(a.out + row * kTrainD + 16 * x + 8 * hf);
      const f32x4 o1 = *reinterpret_cast<const f32x4*>(a.out + row * kTrainD + 16 * x + 8 * hf + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lof = __uint_as_float(df[x][i] << 16), hif = __uint_as_float(df[x][i] & 0xFFFF0000u);
        dcol += lof * (i < 2 ? o0[2 * i] : o1[2 * i - 4]) + hif * (i < 2 ? o0[2 * i + 1] : o1[2 * i - 3]);
      }
    }
  }
  dcol = col_sum(dcol);
  float lse2 = 0.f;
  if (ok) {
    const size_t li = (static_cast<size_t>(b) * Hq + h * a.g + qh) * a.T + t;
    lse2 = a.lse[li] * kLog2e;
    if (hf == 0) {
      const size_t ni = (static_cast<size_t>(b) * Hq + h * a.g + qh) * 32 * a.nt + t;
      a.nlse[ni] = -lse2 / a.scale_log2;
      a.nsum[ni] = -dcol;
    }
  }

  f32x16 dqa[kDB];
#pragma unroll
  for (int x = 0; x < kDB; ++x)
#pragma unroll
    for (int i = 0; i < 16; ++i) dqa[x][i] = 0.f;

  // -D in every row starts the dP products
  f32x16 neg_d;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_d[i] = -dcol;
  auto attend = [&](int st, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    wait_copies();
    __syncthreads();
    if (2 * st + 2 < ntiles) issue(st + 1, buf ^ 1);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {   // a second tile past the last is hidden: every key is after t
      const int jt = 64 * st + 32 * sub;
      constexpr int t_buf = buf * kStage;
      const int tl = t_buf + 2 * kUnit * sub;
      const int cls = mask_class(jt, jt + 32, t0, t1, a.w);
      f32x16 s = score_start(&bias_lds[buf][32 * sub], zero_lds, cls, hf), dp;
      u32x4 op[kAhead];
      // product e: scores (keys) and dP (values) take turns, k-step e / 2
#pragma unroll
      for (int e = 0; e < kAhead; ++e) op[e] = row_operand(tl + kUnit * (e & 1), ad, e >> 1);
#pragma unroll
      for (int e = 0; e < 2 * kKS; ++e) {
        __builtin_amdgcn_sched_barrier(0);
        if (e & 1) dp = mfma(op[e % kAhead], df[e >> 1], e == 1 ? neg_d : dp);
        else s = mfma(op[e % kAhead], qf[e >> 1], s);
        if (e + kAhead < 2 * kKS) op[e % kAhead] = row_operand(tl + kUnit * (e & 1), ad, (e + kAhead) >> 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (cls == 2) score_mask(s, &bias_lds[buf][32 * sub], jt, t, a.w, hf);
#pragma unroll
      for (int e = 0; e < kAhead; ++e) op[e] = col_operand(tl, ad, e % kDB, e / kDB);
      float ds[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) ds[i] = __builtin_amdgcn_exp2f(fmaf(s[i], a.scale_log2, -lse2)) * dp[i];
      const u32x4 du[2] = {pack_bf16(ds), pack_bf16(ds + 8)};
#pragma unroll
      for (int e = 0; e < 2 * kDB; ++e) {
        __builtin_amdgcn_sched_barrier(0);
        dqa[e % kDB] = mfma(op[e % kAhead], du[e / kDB], dqa[e % kDB]);
        if (e + kAhead < 2 * kDB) op[e % kAhead] = col_operand(tl, ad, (e + kAhead) % kDB, (e + kAhead) / kDB);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int st = 0; 2 * st < ntiles; st += 2) {
    attend(st, std::integral_constant<int, 0>{});
    if (2 * st + 2 < ntiles) attend(st + 1, std::integral_constant<int, 1>{});
  }

  const float scale = a.scale_log2 / kLog2e;
  if (ok) {
    float* dst = a.dq + row * kTrainD + 4 * hf;
#pragma unroll
    for (int x = 0; x < kDB; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y)
        *reinterpret_cast<f32x4*>(dst + 32 * x + 8 * y) =
            f32x4{dqa[x][4 * y], dqa[x][4 * y + 1], dqa[x][4 * y + 2], dqa[x][4 * y + 3]} * scale;
  }
}

// ---------------------------------------------------------------------------
// dK / dV / dalpha pass.  Workgroup = (b, KV head h, 128 keys, share of the
// steps); wave w owns keys j0 + 32 w .. + 31 as the 32 columns of its MFMAs,
// with those keys' K and V (B operands) in registers: a row or column operand
// read from LDS feeds 32 columns.  It walks every query head of the group and
// every 32-position query tile from the block's first key on, the last tile
// first (the blocks of one (sequence, head) that run together read the same
// tile at about the same time); two (tile, head) steps are staged at a time.
// Query tiles that are entirely past a key's window come first and add
// without the factor 1 - alpha, which is applied once to the sums where the
// walk leaves them; -lse and -sum dout out start the products' accumulators.
// When the call has too few blocks to fill the chip, each block's steps are
// split over `splits` workgroups whose sums train_sum_kernel adds in order:
// 1777 tokens of 2 x 6 heads, 518 us with one workgroup of 64 keys per block,
// 75 + 8 us with six of 128.  Both loops hold 256 registers without a spill
// only when a step's products and its element-wise part are kept apart and not
// unrolled over the two steps; a reload from scratch waits for every copy in
// flight (4400 us against 2600 us).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads, 2) void train_dkv_kernel(TrainArgs a) {
  __shared__ __attribute__((aligned(256))) char tile_lds[2][kStage];                 // [Q tile | dO tile] x 2
  __shared__ __attribute__((aligned(16))) float row_lds[2][2][2][32];   // [step][-lse / scale, -sum][row]
  const int2 wg = xcd_order();               // earliest (longest) key blocks first
  const int bh = wg.y;
  const int b = bh / a.H, h = bh % a.H;
  const int split = a.split0 + wg.x % a.count;
  const int j0 = wg.x / a.count * 128;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5;
  const int Hq = a.H * a.g;
  const int jw = j0 + 32 * wave;             // this wave's keys jw .. jw + 31
  const int j = jw + (lane & 31);            // this lane's key
  const bool jok = j < a.T;
  const size_t krow = (static_cast<size_t>(b) * a.T + (jok ? j : 0)) * a.H + h;

  // steps first .. last - 1 of the block's list: (query tile, query head) pairs
  const int total = a.g * (a.nt - (j0 >> 5));
  const int first = static_cast<int>(static_cast<int64_t>(total) * split / a.splits);
  const int last = static_cast<int>(static_cast<int64_t>(total) * (split + 1) / a.splits);
  const int nst = (last - first + 1) >> 1;

  const uint32_t stride = Hq * kRowB;
  LaneOffsets lo = lane_offsets(lane, stride);
  const uint32_t tiles = lds_addr(tile_lds);
  const uint16_t* src = wave >> 1 ? a.dout : a.q;
  // this wave copies tensor wave / 2 of step 2 st + wave % 2
  int ld_step = first + (wave & 1);
  int ld_qh = ld_step % a.g, ld_tile = a.nt - 1 - ld_step / a.g;
  auto issue = [&](int buf) {
    if (ld_step < last) {
      const size_t hq = h * a.g + ld_qh;
      copy_tile(reinterpret_cast<const char*>(src + (static_cast<size_t>(b) * a.T * Hq + hq) * kTrainD), 32 * ld_tile,
                a.T, stride, lo, lane, tiles + buf * kStage + 2 * kUnit * (wave & 1) + kUnit * (wave >> 1), a.zeros);
      if (wave < 2) {
        const int ln = fresh(lane);
        const uint32_t off = 4 * (32 * ld_tile + (ln & 31));
        const float* rows = a.nlse + (static_cast<size_t>(b) * Hq + hq) * 32 * a.nt;
        lds_copy4(rows, off + (ln >= 32 ? static_cast<uint32_t>(reinterpret_cast<const char*>(a.nsum) -
                                                          reinterpret_cast<const char*>(a.nlse)) : 0u),
                  lds_addr(row_lds[buf][wave & 1]));
      }
    }
    ld_step += 2;
    ld_qh += 2;
    while (ld_qh >= a.g) {
      ld_qh -= a.g;
      --ld_tile;
    }
  };
  issue(0);

  u32x4 kf[kKS], vf[kKS];
#pragma unroll
  for (int x = 0; x < kKS; ++x) {
    kf[x] = jok ? ld16(a.k + krow * kTrainD + 16 * x + 8 * hf) : u32x4{0u, 0u, 0u, 0u};
    vf[x] = jok ? ld16(a.v + krow * kTrainD + 16 * x + 8 * hf) : u32x4{0u, 0u, 0u, 0u};
  }
  const float keep = 1.0f - (jok ? a.alpha[krow] : 0.f);   // weight of the key outside the window
  f32x16 dka[kDB], dva[kDB];
#pragma unroll
  for (int x = 0; x < kDB; ++x)
#pragma unroll
    for (int i = 0; i < 16; ++i) dka[x][i] = dva[x][i] = 0.f;
  float dal = 0.f;

  // scores and dP of the step staged at `tl`, started from its rows' -lse and -sum
  auto products = [&](uint32_t tl, const float* rows, f32x16& s, f32x16& dp) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 l = *reinterpret_cast<const f32x4*>(rows + 16 * (i >> 1) + 8 * hf + 4 * (i & 1));
      const f32x4 d = *reinterpret_cast<const f32x4*>(rows + 32 + 16 * (i >> 1) + 8 * hf + 4 * (i & 1));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[4 * i + e] = l[e];
        dp[4 * i + e] = d[e];
      }
    }
#pragma unroll
    for (int x = 0; x < kKS; ++x) s = mfma(row_operand(tl, lo, x), kf[x], s);
#pragma unroll
    for (int x = 0; x < kKS; ++x) dp = mfma(row_operand(tl + kUnit, lo, x), vf[x], dp);
    paced<10, 2 * kKS, 1>();
    __builtin_amdgcn_sched_barrier(0);
  };
  // dV^T += dO^T P, dK^T += Q^T dS with P, dS rounded to bf16
  auto sums = [&](uint32_t tl, const f32x16& s, const f32x16& dp) {
    float p[16], ds[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = s[i];
      ds[i] = dp[i];
    }
    const u32x4 pu[2] = {pack_bf16(p), pack_bf16(p + 8)}, du[2] = {pack_bf16(ds), pack_bf16(ds + 8)};
    // product e: dV (dO) and dK (Q) take turns, dim block (e / 2) % 4, token half e / 8
    u32x4 op[kFew];
    auto read = [&](int e) { return col_operand(tl + kUnit * ((e & 1) ^ 1), lo, (e >> 1) % kDB, e / (2 * kDB)); };
#pragma unroll
    for (int e = 0; e < kFew; ++e) op[e] = read(e);
#pragma unroll
    for (int e = 0; e < 4 * kDB; ++e) {
      __builtin_amdgcn_sched_barrier(0);
      const int x = (e >> 1) % kDB, y = e / (2 * kDB);
      if (e & 1) dka[x] = mfma(op[e % kFew], du[y], dka[x]);
      else dva[x] = mfma(op[e % kFew], pu[y], dva[x]);
      if (e + kFew < 4 * kDB) op[e % kFew] = read(e + kFew);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto publish = [&](int st) {   // stage st is in LDS for every wave; copy the next one
    wait_copies();
    __syncthreads();
    if (st + 1 < nst) issue((st & 1) ^ 1);
  };

  int step_qh = first % a.g, tq = 32 * (a.nt - 1 - first / a.g);   // step being computed
  int st = 0;
  // ---- stages whose queries are all past the window of each of this wave's keys
  for (; st < nst && tq - (step_qh + 1 >= a.g ? 32 : 0) - a.w >= jw + 31 && first + 2 * st + 1 < last; ++st) {
    publish(st);
#pragma unroll 1
    for (int sub = 0; sub < 2; ++sub) {
      const uint32_t tl = tiles + (st & 1) * kStage + 2 * kUnit * sub;
      refresh(lo);
      f32x16 s, dp;
      products(tl, &row_lds[st & 1][sub][0][0], s, dp);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = __builtin_amdgcn_exp2f(s[i] * a.scale_log2);   // exp(s - lse), no bias
        dp[i] *= s[i];
        dal += dp[i];
      }
      sums(tl, s, dp);
      if (++step_qh == a.g) {
        step_qh = 0;
        tq -= 32;
      }
    }
  }
  // a fully evicted key (keep = 0) takes exactly nothing from them, also where its sums, formed
  // without that factor, overflowed
#pragma unroll
  for (int x = 0; x < kDB; ++x)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      dka[x][i] = keep == 0.f ? 0.f : dka[x][i] * keep;
      dva[x][i] = keep == 0.f ? 0.f : dva[x][i] * keep;
    }
  // ---- the rest, masked per element
  for (; st < nst; ++st) {
    publish(st);
#pragma unroll 1
    for (int sub = 0; sub < 2; ++sub) {
      if (first + 2 * st + sub >= last) break;
      if (tq + 31 >= jw) {                   // else every query precedes every key
        const uint32_t tl = tiles + (st & 1) * kStage + 2 * kUnit * sub;
        refresh(lo);
        f32x16 s, dp;
        products(tl, &row_lds[st & 1][sub][0][0], s, dp);
        // register i of the lane: query tq + 16 (i / 8) + 8 hf + i % 8; it sees the lane's key
        // from c = d on and is past the key's window from c = d + w on
        const int ln = fresh(lane);
        const int d = jw + (ln & 31) - tq - 8 * (ln >> 5);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int c = 16 * (i >> 3) + (i & 7);
          s[i] = d <= c ? __builtin_amdgcn_exp2f(s[i] * a.scale_log2) : 0.f;
          dp[i] *= s[i];
          const bool old = d <= c - a.w;
          dal += old ? dp[i] : 0.f;
          const float f = old ? keep : 1.0f;
          s[i] *= f;
          dp[i] *= f;
        }
        sums(tl, s, dp);
      }
      if (++step_qh == a.g) {
        step_qh = 0;
        tq -= 32;
      }
    }
  }

  dal = col_sum(dal);
  const int je = jw + (fresh(lane) & 31);
  if (je < a.T) {
    const size_t krow = (static_cast<size_t>(b) * a.T + je) * a.H + h;
    const float scale = a.scale_log2 / kLog2e;
    float *dk = a.dk, *dv = a.dv, *dal_out = a.dalpha;
    if (split) {
      const size_t kv = static_cast<size_t>(a.B) * a.T * a.H * kTrainD;
      dk = a.part + (split - max(a.split0, 1)) * a.part_stride;
      dv = dk + kv;
      dal_out = dv + kv;
    }
    dk += krow * kTrainD + 4 * hf;
    dv += krow * kTrainD + 4 * hf;
#pragma unroll
    for (int x = 0; x < kDB; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        *reinterpret_cast<f32x4*>(dk + 32 * x + 8 * y) =
            f32x4{dka[x][4 * y], dka[x][4 * y + 1], dka[x][4 * y + 2], dka[x][4 * y + 3]} * scale;
        *reinterpret_cast<f32x4*>(dv + 32 * x + 8 * y) =
            f32x4{dva[x][4 * y], dva[x][4 * y + 1], dva[x][4 * y + 2], dva[x][4 * y + 3]};
      }
    if (hf == 0) dal_out[krow] = -dal;
  }
}

// Adds the sums that a split key-major pass left in `part` to the outputs, in
// split order.
__global__ __launch_bounds__(kThreads) void train_sum_kernel(TrainArgs a) {
  const size_t rows = static_cast<size_t>(a.B) * a.T * a.H, kv = rows * kTrainD;
  const size_t i = (static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x) * 4;
  if (i >= 2 * kv + rows) return;
  auto add = [&](float* dst, int n) {
    float x[4];
    for (int e = 0; e < n; ++e) x[e] = dst[e];
    for (int sp = 0; sp < a.sets; ++sp)
      for (int e = 0; e < n; ++e) x[e] += a.part[sp * a.part_stride + i + e];
    for (int e = 0; e < n; ++e) dst[e] = x[e];
  };
  if (i < 2 * kv) {   // rows of 128 floats: four at a time never straddle the two tensors
    float* dst = i < kv ? a.dk + i : a.dv + (i - kv);
    f32x4 x = *reinterpret_cast<const f32x4*>(dst);
    for (int sp = 0; sp < a.sets; ++sp) x += *reinterpret_cast<const f32x4*>(a.part + sp * a.part_stride + i);
    *reinterpret_cast<f32x4*>(dst) = x;
  } else {
    add(a.dalpha + (i - 2 * kv), static_cast<int>(min(static_cast<size_t>(4), 2 * kv + rows - i)));
  }
}

__global__ __launch_bounds__(kThreads) void gumbel_fwd_kernel(int n, const float* x, const float* u,
                                                              float inv_tau, float* alpha) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const float uu = u[i];
  const float z = (x[i] + (__logf(uu) - __logf(1.0f - uu))) * inv_tau;
  alpha[i] = 1.0f / (1.0f + __expf(-z));
}

__global__ __launch_bounds__(kThreads) void gumbel_bwd_kernel(int n, const float* alpha, const float* da,
                                                              float inv_tau, float* dx) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const float al = alpha[i];
  dx[i] = da[i] * al * (1.0f - al) * inv_tau;
}

// Global -> LDS copies of 16 bytes a lane need their rows 16-byte aligned; an
// input that is not (a view into a larger buffer) is copied to the workspace.
__global__ __launch_bounds__(kThreads) void train_align_kernel(const uint16_t* src, uint16_t* dst, size_t n) {
  for (size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * kThreads)
    dst[i] = src[i];
}

// Workspace (2 (H + Hq) 16 KB per sequence and 32 positions, and 4 B Hq T):
// 16 zero bytes, key biases, the two per-row arrays, aligned copies of inputs that need one
// and, for a split key-major pass, the further workgroups' sums in what is left.
struct TrainLayout {
  size_t zeros, bias, nlse, nsum, part, bytes;
  size_t part_stride;   // floats of one set of sums
  int nt, nst;
};

TrainLayout train_layout(const dms_train_config& c) {
  TrainLayout l{};
  const size_t B = c.batch, T = c.seq_len, H = c.num_kv_heads, Hq = H * c.group_size;
  const size_t D = c.head_dim;
  l.nt = static_cast<int>((T + 31) / 32);
  l.nst = (l.nt + 1) / 2;
  const size_t tile = D * 128;
  l.bytes = 2 * align_up(B * H * l.nt * tile, kAlign) + 2 * align_up(B * Hq * l.nt * tile, kAlign) +
            align_up(B * Hq * T * 4, kAlign);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, kAlign); return o; };
  l.zeros = take(16);
  l.bias = take(B * H * l.nst * 64 * 4);
  l.nlse = take(B * Hq * l.nt * 32 * 4);
  l.nsum = take(B * Hq * l.nt * 32 * 4);
  l.part_stride = align_up((2 * B * T * H * D + B * T * H) * 4, kAlign) / 4;
  l.part = off;
  return l;
}

// Sets `dst` to `src`, or to an aligned copy taken from the workspace's free part.
hipError_t align_input(const uint16_t*& dst, const void* src, size_t rows, TrainLayout& l, char* ws, hipStream_t st) {
  dst = static_cast<const uint16_t*>(src);
  if (reinterpret_cast<uintptr_t>(src) % 16 == 0) return hipSuccess;
  uint16_t* copy = reinterpret_cast<uint16_t*>(ws + l.part);
  l.part = align_up(l.part + rows * kRowB, kAlign);
  hipLaunchKernelGGL(train_align_kernel, dim3(1024), dim3(kThreads), 0, st, dst, copy, rows * kTrainD);
  dst = copy;
  return hipGetLastError();
}

TrainArgs train_args(const dms_train_config& c, const TrainLayout& l, void* ws) {
  TrainArgs a{};
  char* w = static_cast<char*>(ws);
  a.zeros = reinterpret_cast<float*>(w + l.zeros);
  a.bias = reinterpret_cast<float*>(w + l.bias);
  a.nlse = reinterpret_cast<float*>(w + l.nlse);
  a.nsum = reinterpret_cast<float*>(w + l.nsum);
  a.part_stride = l.part_stride;
  a.B = c.batch;
  a.T = c.seq_len;
  a.H = c.num_kv_heads;
  a.g = c.group_size;
  a.w = c.window;
  a.nt = l.nt;
  a.nst = l.nst;
  a.PB = 4 * 32 / c.group_size;   // (position, head) columns packed across the waves' column blocks
  a.splits = 1;
  const float scale = c.softmax_scale > 0.f ? c.softmax_scale : 1.0f / sqrtf(static_cast<float>(c.head_dim));
  a.scale_log2 = scale * kLog2e;
  return a;
}

hipError_t launch_bias(const TrainArgs& a, bool backward, hipStream_t st) {
  hipLaunchKernelGGL(train_bias_kernel, dim3((64 * a.nst + kThreads - 1) / kThreads, a.B * a.H), dim3(kThreads), 0,
                     st, a, backward);
  return hipGetLastError();
}

}  // namespace

size_t train_workspace_bytes(const dms_train_config& c) { return train_layout(c).bytes; }

hipError_t launch_train_fwd(const dms_train_config& c, const void* q, const void* k, const void* v,
                            const float* alpha, float* out, float* lse, void* ws, hipStream_t st) {
  TrainLayout l = train_layout(c);
  TrainArgs a = train_args(c, l, ws);
  char* w = static_cast<char*>(ws);
  const size_t rows = static_cast<size_t>(c.batch) * c.seq_len * c.num_kv_heads;
  a.q = static_cast<const uint16_t*>(q);
  a.alpha = alpha;
  a.o_out = out;
  a.lse_out = lse;
  hipError_t e = align_input(a.k, k, rows, l, w, st);
  if (e == hipSuccess) e = align_input(a.v, v, rows, l, w, st);
  if (e == hipSuccess) e = launch_bias(a, false, st);
  if (e != hipSuccess) return e;
  dim3 grid((c.seq_len + a.PB - 1) / a.PB, c.batch * c.num_kv_heads);
  hipLaunchKernelGGL(train_fwd_kernel, grid, dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_train_bwd(const dms_train_config& c, const void* q, const void* k, const void* v,
                            const float* alpha, const float* out, const float* lse,
                            const void* dout, float* dq, float* dk, float* dv, float* dalpha,
                            void* ws, hipStream_t st) {
  TrainLayout l = train_layout(c);
  TrainArgs a = train_args(c, l, ws);
  char* w = static_cast<char*>(ws);
  const size_t rows = static_cast<size_t>(c.batch) * c.seq_len * c.num_kv_heads;
  a.alpha = alpha;
  a.out = out;
  a.lse = lse;
  a.dq = dq;
  a.dk = dk;
  a.dv = dv;
  a.dalpha = dalpha;
  hipError_t e = align_input(a.k, k, rows, l, w, st);
  if (e == hipSuccess) e = align_input(a.v, v, rows, l, w, st);
  if (e == hipSuccess) e = align_input(a.q, q, rows * c.group_size, l, w, st);
  if (e == hipSuccess) e = align_input(a.dout, dout, rows * c.group_size, l, w, st);
  if (e == hipSuccess) e = launch_bias(a, true, st);
  if (e != hipSuccess) return e;
  dim3 grid((c.seq_len + a.PB - 1) / a.PB, c.batch * c.num_kv_heads);
  hipLaunchKernelGGL(train_dq_kernel, grid, dim3(kThreads), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // Key-major pass: about two workgroups per CU.  Copies of unaligned inputs
  // can leave room for fewer sets of sums than there are splits (with aligned
  // inputs at least g sets fit, with four copies at least one for g > 1): the
  // splits then take several launches, each added before the next, so that
  // the order of the sums does not depend on the addresses.
  a.part = reinterpret_cast<float*>(w + l.part);
  const int blocks = (c.seq_len + 127) / 128;
  const int64_t wgs = static_cast<int64_t>(blocks) * c.batch * c.num_kv_heads;
  const int room = l.bytes > l.part ? static_cast<int>(std::min<size_t>(kMaxGroup, (l.bytes - l.part) / (l.part_stride * 4))) : 0;
  a.splits = room ? static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(512 / wgs, c.group_size))) : 1;
  for (int s = 0; s < a.splits; s += a.count) {
    a.split0 = s;
    a.sets = std::min(room, a.splits - std::max(s, 1));
    a.count = a.sets + (s == 0);
    hipLaunchKernelGGL(train_dkv_kernel, dim3(blocks * a.count, c.batch * c.num_kv_heads), dim3(kThreads), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.sets == 0) continue;
    const size_t n = (rows * (2 * kTrainD + 1) + 3) / 4;
    hipLaunchKernelGGL(train_sum_kernel, dim3(static_cast<unsigned>((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_gumbel_fwd(int n, const float* x, const float* u, float tau, float* alpha,
                             hipStream_t st) {
  hipLaunchKernelGGL(gumbel_fwd_kernel, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, st, n,
                     x, u, 1.0f / tau, alpha);
  return hipGetLastError();
}

hipError_t launch_gumbel_bwd(int n, const float* alpha, const float* da, float tau, float* dx,
                             hipStream_t st) {
  hipLaunchKernelGGL(gumbel_bwd_kernel, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, st, n,
                     alpha, da, 1.0f / tau, dx);
  return hipGetLastError();
}

}  // namespace dms
