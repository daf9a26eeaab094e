// One streaming pass over a sequence's KV cache for one KV head: the kernel
// behind vp_visual_mass (Eq. (2), (5), (6)) and the attention partials of
// vp_sparse_decode_attn (Sec. 4.1/4.2).
//
// Work decomposition: one 64-lane wave per work-group; grid = (parts, Hkv, B)
// (kept pass: (splits, Hkv * T, B), one row of work-groups per query). Up to
// mid-size caches kPartWaves waves share a part, each with the visual and the
// text role, and merge their partials in LDS (attend_waves_kernel).
// In the context pass part p of `nparts` takes the 32-row tiles p, p + nparts,
// p + 2 nparts, ... of the cache (a cyclic deal: every part, and so every XCD,
// sees the sequence's own mix of visual and text rows); in the kept pass a part
// is `split` consecutive entries of the kept-index list.
//
// Three roles share this kernel:
//   visual pass  visual rows only: Eq. (5)/(6) and Eq. (2) statistics and the
//                logit spill (the only large write of the step);
//   text pass    text rows only: the same statistics and/or the attention
//                partial over text K/V, with no large writes, so its reads
//                stream without write traffic mixed in;
//   kept pass    gathered kept visual rows: the attention partial.
//
// Memory path. Every K and V row of a tile is copied HBM -> LDS with
// global_load_lds_dwordx4 (non-temporal): one instruction moves whole rows (1 KB contiguous
// per instruction for 256-byte rows), the access pattern that streams at full
// HBM rate on gfx950 (the matrix-core operand layout, 16 rows x 64 B per load,
// streams about 25% slower). All of a tile's copies are issued before any of
// it is used, so no registers are held by data in flight. Inside LDS a row's
// 16-byte pieces are XOR-swizzled by the row index (slot = piece ^ row), which
// keeps the operand reads below free of bank conflicts.
//
// Per 32-row sub-tile the query rows of this KV head -- its G grouped heads for
// each of the sequence's T queries, T*G <= 16, padded to 16 -- are scored
// against the key rows on the matrix cores (with several queries per sequence
// the K/V rows are read once for all of them; query t sees the positions
// before L - T + 1 + t):
//   C'[token][head] = K_tile[token][:] . q[head][:]
// bf16: v_mfma_f32_16x16x32_bf16 (two 16-row halves x d/32 k-steps);
// fp32: v_mfma_f32_16x16x4_f32. Lane l then holds head l%16 for tokens
// 16*half + 4*(l/16) + r.
//
// Statistics, all in the log2 domain z = Z * log2(e), each over the rows of its
// pass relative to a running maximum m (lane-local in the visual pass, shared
// by the four lanes of a head in the text pass):
//   Ls = sum_j 2^((z_j - m)/tau_score)   (normaliser of the Eq. (2) attention)
//   Lm = sum_j 2^((z_j - m)/tau_mass)    (Eq. (6) denominator; over the visual
//                                         rows alone it is the Eq. (5) numerator)
// A maximum is raised only when a logit exceeds it by more than a margin that
// keeps every weight below 2^64, so rescaling is rare.
// Visual logits are spilled to the workspace for the scores, which need the
// global (m, Ls) of every head. The spill holds one plane per (sequence, KV
// group) with a row of zs_gp floats (the group's heads, padded to 8 or 16) per
// cache position; a full visual sub-tile is transposed through a small LDS
// stage so that its 32 rows leave as one contiguous 1-2 KB store (whole lines:
// partial-line writes would compete with the streaming reads for the L1's
// outstanding-request slots), and the scores read each (token, group) row with
// 16-byte loads.
//
// Attention partial (text rows of the context pass, or the gathered kept rows):
//   (m_t, l_t, acc[d]) with p_j = 2^(z_j - m_t), acc = sum_j p_j V_j.
// The value product runs on the matrix cores as out^T[dim][head] += V^T P^T:
// V is read transposed from LDS, P comes straight from the score registers, so
// the accumulator keeps lane l on head l%16 and the rescaling factor is lane-local.
#include "vp_common.h"
#include "vp_internal.h"

#include <hip/hip_ext.h>

#ifndef VP_ATTEND_WAVES
#define VP_ATTEND_WAVES 2  // bf16 passes that read V
#endif
#ifndef VP_ATTEND_WAVES_LEAN
#define VP_ATTEND_WAVES_LEAN 4  // bf16 passes that read only K
#endif

typedef __attribute__((address_space(1))) void global_void;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) unsigned char lds_byte;

// Cache policy of the K/V row copies: non-temporal (the "nt" bit). Every row is
// used once per step, and streaming it without cache allocation measured ~13%
// faster on the text pass (5.4 -> 6.1 TB/s on the 64 x 32k batch).
constexpr int kCopyPolicy = 2;

// s_waitcnt immediates (gfx9 encoding: vmcnt [3:0]+[15:14], expcnt [6:4], lgkmcnt [11:8])
constexpr int kWaitLgkm0 = 0xC07F;  // lgkmcnt(0), others unconstrained
constexpr int kWaitVm0 = 0x0F70;    // vmcnt(0), others unconstrained
// buffer resource word 3 for raw (untyped) dword access: 32-bit data format
constexpr int kRawBufferWord3 = 0x00020000;
// cache policy of the full-tile spill stores: sc1 (device scope) in the visual
// pass launched alone (64 x 32k batch: visual pass 230 -> 226 us; non-temporal
// stores: 242), the default in the one-launch context pass (sc1 there: 72B-class
// decode loop 84.0 -> 84.6 us per step)
constexpr int spill_policy(int mode) { return vp::base_mode(mode) == vp::MODE_VIS ? 16 : 0; }

namespace vp {
namespace {

// waves per SIMD the register allocation is sized for (one wave per work-group)
constexpr bool reads_v(int mode) { return (base_mode(mode) & (MODE_TEXT_ATTN | MODE_KEPT)) != 0; }
constexpr int attend_waves(int dt, int mode) {
  return dt != VP_BF16 ? 1 : (reads_v(mode) ? VP_ATTEND_WAVES : VP_ATTEND_WAVES_LEAN);
}

// LDS floor per work-group: 20 KB keeps the bf16 passes that read V at 8
// resident work-groups per CU (their 160 registers would allow 10 with 16 KB);
// measured ~8% faster on the text pass of the 64 x 32k batch.
#ifndef VP_LDS_FLOOR_TEXT
#define VP_LDS_FLOOR_TEXT 20480  // bytes; bf16 passes that read V
#endif
#ifndef VP_LDS_FLOOR_VIS
#define VP_LDS_FLOOR_VIS 0  // bytes; bf16 K-only passes
#endif
constexpr int max_i(int x, int y) { return x > y ? x : y; }
constexpr int lds_floor(int dt, int mode) {
  return dt != VP_BF16 ? 0 : (reads_v(mode) ? VP_LDS_FLOOR_TEXT : VP_LDS_FLOOR_VIS);
}

// Make a value unknown to the optimiser at this point, so that what is computed
// from it stays where it is instead of being kept in registers through a loop
// (device code only: the constraints name scalar and vector registers)
template <typename X>
__device__ __forceinline__ void unhoist_scalar(X& x) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(x));
#endif
}
template <typename X>
__device__ __forceinline__ void unhoist_vector(X& x) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+v"(x));
#endif
}

template <int DT, int D>
struct Cfg {
  static constexpr bool BF = DT == VP_BF16;
  static constexpr int ESZ = BF ? 2 : 4;
  static constexpr int ROWB = D * ESZ;                      // bytes per K/V row
  static constexpr int PIECES = ROWB / 16;                  // 16-byte pieces per row
  static constexpr int RPI = 64 / PIECES;                   // rows per 1 KB copy instruction
  static constexpr int SUB_ROWS_BYTES = 32 * ROWB;          // one 32-row block of K or V
  static constexpr int STAGE_BYTES = 16 * 32 * 4;           // logits of 16 heads x 32 rows
  static constexpr int COPIES = 32 / RPI;                   // copy instructions per block
  static constexpr int ACC_N = BF ? (D / 64) * 4 : D / 16;  // f32x4 accumulators
  // LDS byte offset of 16-byte piece p of row r inside a block
  static __device__ __forceinline__ int at(int r, int p) { return r * ROWB + 16 * (p ^ (r & (PIECES - 1))); }
};

template <int DT, int D>
struct QFrag;

template <int D>
struct QFrag<VP_BF16, D> {
  bf16x8 v[D / 32];
};
template <int D>
struct QFrag<VP_F32, D> {
  float v[D / 4];
};

// q row of head h as the B operand (k-slot (a4, i) of step s <-> dim s*32 + 8*a4 + i
// for bf16; dim (D/4)*a4 + s for fp32)
template <int DT, int D>
__device__ __forceinline__ void load_q(QFrag<DT, D>& f, const void* qrow, bool valid, int a4) {
  if constexpr (DT == VP_BF16) {
    const uint4* p = reinterpret_cast<const uint4*>(qrow);
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
      uint4 u = valid ? p[4 * s + a4] : make_uint4(0, 0, 0, 0);
      f.v[s] = __builtin_bit_cast(bf16x8, u);
    }
  } else {
    const float4* p = reinterpret_cast<const float4*>(qrow);
#pragma unroll
    for (int s4 = 0; s4 < D / 16; ++s4) {
      float4 u = valid ? p[(D / 16) * a4 + s4] : make_float4(0.f, 0.f, 0.f, 0.f);
      f.v[4 * s4 + 0] = u.x;
      f.v[4 * s4 + 1] = u.y;
      f.v[4 * s4 + 2] = u.z;
      f.v[4 * s4 + 3] = u.w;
    }
  }
}

// C'[token n16 of 16-row half hf][head] from the key block in LDS (same dim
// mapping as load_q)
template <int DT, int D>
__device__ __forceinline__ f32x4 score_half(const unsigned char* kb, int hf, const QFrag<DT, D>& q, int a4,
                                            int n16) {
  using C = Cfg<DT, D>;
  const int r = 16 * hf + n16;
  f32x4 c = {0.f, 0.f, 0.f, 0.f};
  if constexpr (DT == VP_BF16) {
    uint4 k[D / 32];
#pragma unroll
    for (int s = 0; s < D / 32; ++s) k[s] = *reinterpret_cast<const uint4*>(kb + C::at(r, 4 * s + a4));
#pragma unroll
    for (int s = 0; s < D / 32; ++s)
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[s]), q.v[s], c, 0, 0, 0);
  } else {
    float4 k[D / 16];
#pragma unroll
    for (int s4 = 0; s4 < D / 16; ++s4) k[s4] = *reinterpret_cast<const float4*>(kb + C::at(r, (D / 16) * a4 + s4));
#pragma unroll
    for (int s4 = 0; s4 < D / 16; ++s4) {
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s4].x, q.v[4 * s4 + 0], c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s4].y, q.v[4 * s4 + 1], c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s4].z, q.v[4 * s4 + 2], c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s4].w, q.v[4 * s4 + 3], c, 0, 0, 0);
    }
  }
  return c;
}

// sub-tile-relative token held by lane slot (a4, i) of the value product: the
// score registers of lane l hold tokens 4*a4 + r (half 0) and 16 + 4*a4 + r (half 1)
__device__ __forceinline__ int pv_token(int a4, int i) { return i < 4 ? 4 * a4 + i : 16 + 4 * a4 + (i - 4); }

template <int DT, int D, int N>
__device__ __forceinline__ void value_product(f32x4 (&acc)[N], const unsigned char* vb, const float (&p)[8],
                                              int a4, int n16) {
  using C = Cfg<DT, D>;
  if constexpr (DT == VP_BF16) {
    // P^T operand: slot (a4, i) <-> token pv_token(a4, i), head n16
    bf16x8 pf;
#pragma unroll
    for (int i = 0; i < 8; ++i) pf[i] = static_cast<__bf16>(p[i]);
#pragma unroll
    for (int u = 0; u < D / 64; ++u) {
      // lane n16 takes dims 64u + 4*n16 .. +3 = 8 bytes in piece 8u + n16/2
      uint2 w[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        w[i] = *reinterpret_cast<const uint2*>(vb + C::at(pv_token(a4, i), 8 * u + (n16 >> 1)) + 8 * (n16 & 1));
      // A operand of MFMA (u, e): row n16 <-> dim 64u + 4*n16 + e, slot i <-> token pv_token(a4, i)
      uint32_t lo0[4], hi0[4], lo1[4], hi1[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lo0[j] = __builtin_amdgcn_perm(w[2 * j + 1].x, w[2 * j].x, 0x05040100u);
        hi0[j] = __builtin_amdgcn_perm(w[2 * j + 1].x, w[2 * j].x, 0x07060302u);
        lo1[j] = __builtin_amdgcn_perm(w[2 * j + 1].y, w[2 * j].y, 0x05040100u);
        hi1[j] = __builtin_amdgcn_perm(w[2 * j + 1].y, w[2 * j].y, 0x07060302u);
      }
      const bf16x8 a0 = __builtin_bit_cast(bf16x8, make_uint4(lo0[0], lo0[1], lo0[2], lo0[3]));
      const bf16x8 a1 = __builtin_bit_cast(bf16x8, make_uint4(hi0[0], hi0[1], hi0[2], hi0[3]));
      const bf16x8 a2 = __builtin_bit_cast(bf16x8, make_uint4(lo1[0], lo1[1], lo1[2], lo1[3]));
      const bf16x8 a3 = __builtin_bit_cast(bf16x8, make_uint4(hi1[0], hi1[1], hi1[2], hi1[3]));
      acc[4 * u + 0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, pf, acc[4 * u + 0], 0, 0, 0);
      acc[4 * u + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, pf, acc[4 * u + 1], 0, 0, 0);
      acc[4 * u + 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, pf, acc[4 * u + 2], 0, 0, 0);
      acc[4 * u + 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a3, pf, acc[4 * u + 3], 0, 0, 0);
    }
  } else {
    // k-step s covers tokens pv_token(a4, s) (one per lane group); row n16 <-> dim 16*dt + n16
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int t = pv_token(a4, s);
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        const int dim = 16 * dt + n16;
        const float v = *reinterpret_cast<const float*>(vb + C::at(t, dim >> 2) + 4 * (dim & 3));
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, p[s], acc[dt], 0, 0, 0);
      }
    }
  }
}

// store the lane's accumulator slice (head n16) of a (D)-float partial row
template <int DT, int D, int N>
__device__ __forceinline__ void store_acc(float* dst, const f32x4 (&acc)[N], int a4) {
  if constexpr (DT == VP_BF16) {
    // acc[4u + e][r] holds dim 64u + 16*a4 + 4r + e
#pragma unroll
    for (int u = 0; u < D / 64; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float4 o = make_float4(acc[4 * u + 0][r], acc[4 * u + 1][r], acc[4 * u + 2][r], acc[4 * u + 3][r]);
        *reinterpret_cast<float4*>(dst + 64 * u + 16 * a4 + 4 * r) = o;
      }
  } else {
    // acc[dt][r] holds dim 16*dt + 4*a4 + r
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      *reinterpret_cast<float4*>(dst + 16 * dt + 4 * a4) = make_float4(acc[dt][0], acc[dt][1], acc[dt][2], acc[dt][3]);
  }
}

// A running maximum before any finite logit: the least float, not -inf, so that rows
// of logit -inf weigh 2^-inf = 0 until then (relative to -inf they would be NaN).
// Written out as -inf (an empty partial).
constexpr float kNoLogit = -3.402823466e38f;

enum TileClass : int { TILE_TEXT = 0, TILE_VIS = 1, TILE_MIXED = 2 };

// class of tile [t0, t_end) given a walker already seeked to t0
__device__ __forceinline__ int classify(const SegWalker& w, int t0, int t_end) {
  if (w.s < w.nseg && w.st < t_end) return (w.st <= t0 && w.en >= t_end) ? TILE_VIS : TILE_MIXED;
  return TILE_TEXT;
}

struct Sub {
  int t0;       // first row of the 32-row sub-tile (cache position, or index into the kept list)
  int cls;      // TileClass (context pass)
  int kp;       // kept pass: lane r < 32 holds the cache position of row t0 + r (-1 past the list)
  int blk;      // paged caches: lane r < 32 holds the physical block of row t0 + r
  SegWalker w;  // segment walker positioned at t0 (context pass)
};

// All per-wave state of one part; member functions are force-inlined.
template <int DT, int D, int MODE>
struct Pass {
  using C = Cfg<DT, D>;
  static constexpr int BASE = base_mode(MODE);
  static constexpr bool PAGED = (MODE & MODE_PAGED) != 0;        // rows through the block table
  static constexpr bool KEPT = BASE == MODE_KEPT;
  static constexpr bool ZSPILL = KEPT && (MODE & MODE_ZSPILL) != 0;  // kept logits from the spill
  static constexpr bool VIS = (BASE & MODE_VIS) != 0;            // visual rows: statistics + spill
  static constexpr bool TSTATS = (BASE & MODE_TEXT_STATS) != 0;  // text rows: statistics
  static constexpr bool ATTN = KEPT || (BASE & MODE_TEXT_ATTN) != 0;
  static constexpr bool TEXT = (BASE & MODE_TEXT_BOTH) != 0;     // text rows: statistics and/or attention

  const AttendArgs& a;
  int lane, n16, a4, L, r0, r1, step, h;  // rows [r0, r1) in tiles `step` apart; h: virtual head
  int L0, lim;  // rows from L0 on are the queries' own; this lane's query sees rows < lim
  bool hv;
  const int32_t* kept;
  const char* Kb;
  const char* Vb;
  size_t rstride;
  const int32_t* bt;  // paged caches: this sequence's block table (else null)
  size_t bstride;     // paged caches: bytes per physical block
  int bmask;          // paged caches: rows per block - 1
  float* zbase;  // spill plane of this KV group: row p holds the logits of its heads at position p
                 // (kept pass from the spill: offset to the query's first head)
  QFrag<DT, D> qf;
  // visual pass: lane-local reference and sums (merged over a head's 4 lanes at the end)
  float m_v, Ls_v, Lm_v;
  // text / kept pass: reference shared by a head's 4 lanes, sums and value partial
  float m_t, l_t, Lm_t, Ls_t;
  f32x4 acc[C::ACC_N];
  // copies after which the swizzle repeats
  static constexpr int STEPS = C::PIECES / C::RPI < C::COPIES ? max_i(C::PIECES / C::RPI, 1) : C::COPIES;
  uint32_t row_step[STEPS];  // context passes: init_row_step
  bool even;

  __device__ __forceinline__ explicit Pass(const AttendArgs& a_) : a(a_) {}

  // cache position of row r of sub-tile s (clamped to a readable row; validity is tracked separately)
  __device__ __forceinline__ int row_pos(const Sub& s, int r) const {
    if constexpr (KEPT) {
      const int p = __shfl(s.kp, r);
      return (p < 0 || p >= L) ? 0 : p;
    } else {
      const int t = s.t0 + r;
      return t < L ? t : L - 1;
    }
  }

  // does this pass have rows in sub-tile s
  __device__ __forceinline__ bool active(const Sub& s) const {
    if (s.t0 >= r1) return false;
    if constexpr (VIS && !TEXT) return s.cls != TILE_TEXT;
    if constexpr (TEXT && !VIS) return s.cls != TILE_VIS;
    return true;
  }
  __device__ __forceinline__ bool needs_v(const Sub& s) const { return ATTN && (!VIS || s.cls != TILE_VIS); }

  __device__ __forceinline__ Sub sub_at(const Sub& prev, int t0, int kp_loaded = -2) const {
    Sub n = prev;
    n.t0 = t0;
    n.cls = TILE_TEXT;
    if constexpr (KEPT) {
      // one coalesced load of the tile's kept positions (issued a tile ahead;
      // the first tile's come in as kp_loaded, requested before the budget)
      const int t = t0 + lane;
      n.kp = (lane < 32 && t < r1) ? (kp_loaded != -2 ? kp_loaded : kept[t]) : -1;
      if constexpr (PAGED) {
        if (lane < 32) n.blk = block_of((n.kp < 0 || n.kp >= L) ? 0 : n.kp);
      }
    } else {
      if (t0 < r1) {
        n.w.seek(t0);
        n.cls = classify(n.w, t0, min(t0 + 32, r1));
        if constexpr (PAGED && !(VIS && TEXT)) {
          if (active(n) && lane < 32) n.blk = block_of(min(t0 + lane, L - 1));
        }
      }
      // a wave of both roles needs the ids of every tile: no branch around the load
      // (blocks of 16 rows, 64 pairs x 9.1k tokens: 73.7 us per step with one, 72.0
      // without). Tiles past the end and empty sequences read an entry of the
      // sequence's own row, which is not used
      if constexpr (PAGED && VIS && TEXT) {
        if (lane < 32) n.blk = block_of(max(min(t0 + lane, L - 1), 0));
      }
    }
    return n;
  }

  // paged caches: the physical block of position p >= 0 (of each of a tile's rows: the
  // position that row_pos will read, clipped ones included)
  __device__ __forceinline__ int block_of(int p) const {
    return bt[p >> __builtin_ctz(static_cast<unsigned>(bmask + 1))];
  }

  // kept pass from the spill: the logits of this lane's 8 rows (head n16 of
  // the query), requested with the tile's V rows; rows past the list read
  // position 0 and are masked like their V rows, lanes without a head read
  // head 0's (no branch around a load: the compiler would wait for each)
  __device__ __forceinline__ void load_spill(const Sub& s, float (&z)[8]) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int p = __shfl(s.kp, 16 * (i >> 2) + 4 * a4 + (i & 3));
      const int pp = (p < 0 || p >= L) ? 0 : p;
      z[i] = zbase[static_cast<size_t>(pp) * a.zs_gp + (hv ? n16 : 0)];
    }
  }

  // byte offsets (from the head's base) of what lane l copies in copy j: row
  // j*RPI + l/PIECES, 16-byte piece (l%PIECES) ^ (row & (PIECES-1)) (the swizzle)
  __device__ __forceinline__ void row_offsets(const Sub& s, size_t (&off)[C::COPIES]) const {
    const int rr = lane / C::PIECES;
    const int slot = lane % C::PIECES;
#pragma unroll
    for (int j = 0; j < C::COPIES; ++j) {
      const int r = j * C::RPI + rr;
      const int piece = slot ^ (r & (C::PIECES - 1));
      const int pos = row_pos(s, r);
      if constexpr (PAGED) {
        const int blk = __shfl(s.blk, r);
        off[j] = static_cast<size_t>(blk) * bstride + static_cast<size_t>(pos & bmask) * rstride + 16 * piece;
      } else {
        off[j] = static_cast<size_t>(pos) * rstride + 16 * piece;
      }
    }
  }

  // A tile whose 32 rows are all inside the sequence (a context pass) has them
  // at equal steps from one address, in one physical block when a paged cache's
  // blocks hold 32 rows or more. Its copies take that address as a buffer and
  // lane offsets that never change (row_step), so they cost no address
  // arithmetic; `even` says that the offsets fit 32 bits.
  __device__ __forceinline__ void init_row_step() {
    const int rr = lane / C::PIECES;
    const int slot = lane % C::PIECES;
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
      const int r = j * C::RPI + rr;
      row_step[j] = static_cast<uint32_t>(r) * static_cast<uint32_t>(rstride) + 16 * (slot ^ (r & (C::PIECES - 1)));
    }
    even = rstride < (1u << 25) && (!PAGED || bmask >= 31);
  }
  __device__ __forceinline__ size_t tile_offset(const Sub& s) const {
    if constexpr (PAGED)
      return static_cast<size_t>(__builtin_amdgcn_readfirstlane(s.blk)) * bstride +
             static_cast<size_t>(s.t0 & bmask) * rstride;
    return static_cast<size_t>(s.t0) * rstride;
  }
  __device__ __forceinline__ void copy_even_rows(const char* src, lds_byte* block) const {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, 0x7fffffff, kRawBufferWord3);
#pragma unroll
    for (int j = 0; j < C::COPIES; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(block + 1024 * j), 16, row_step[j % STEPS],
                                               j / STEPS * (STEPS * C::RPI) * static_cast<int>(rstride), 0,
                                               kCopyPolicy);
  }

  // the 32 rows of a sub-tile from `src` (K or V of this head) into an LDS block
  __device__ __forceinline__ void copy_rows(const char* src, const size_t (&off)[C::COPIES],
                                            lds_byte* block) const {
#pragma unroll
    for (int j = 0; j < C::COPIES; ++j)
      __builtin_amdgcn_global_load_lds((global_void*)(src + off[j]), (lds_void*)(block + 1024 * j), 16, 0,
                                       kCopyPolicy);
  }

  // Whole tiles have code without masks of their own, and masked tiles compute
  // their addresses anew (unhoist_lane): the bf16 passes, whose registers must
  // leave room for two waves per SIMD. An fp32 wave has a SIMD's registers to
  // itself: there two copies of the tile's code and addresses computed per tile
  // cost 8 to 22% of the step (16 x 28/4 heads x 7k tokens 112.8 -> 104.0 us without them,
  // 3 x 16 heads of 64 x 2k 40.5 -> 33.7).
  static constexpr bool WHOLE = C::BF && !KEPT;

  // Lane indices that the compiler cannot prove unchanged from tile to tile:
  // what the rare tiles compute from them is computed there, instead of being
  // kept in registers through the loop.
  __device__ __forceinline__ void unhoist_lane() {
    unhoist_vector(lane);
    n16 = lane & 15;
    a4 = lane >> 4;
  }

  // FULL: 32 rows of one kind, all visible to every query (no masks)
  template <bool FULL>
  __device__ __forceinline__ void process(const Sub& tile, const unsigned char* kblk, const unsigned char* vblk,
                                         float* stage, const float (&zk)[8]) {
    const int t0 = tile.t0;
    const int cls = tile.cls;
    const int t_end = min(t0 + 32, r1);
    // ---- scores of the 32 rows against the query group ----
    float z[8];
    if constexpr (ZSPILL) {
      // the visual pass computed these logits with the same products (the
      // same operands and instructions give the same bits)
#pragma unroll
      for (int i = 0; i < 8; ++i) z[i] = zk[i];
    } else {
      const f32x4 c0 = score_half<DT, D>(kblk, 0, qf, a4, n16);
      const f32x4 c1 = score_half<DT, D>(kblk, 1, qf, a4, n16);
#pragma unroll
      for (int i = 0; i < 8; ++i) z[i] = (i < 4 ? c0[i & 3] : c1[i & 3]) * a.zscale;
    }

    // value i of this lane is row t0 + 16*(i/4) + 4*a4 + i%4; bit i of the masks
    // (`valid_rows`: before the causal mask of several queries)
    unsigned valid = 0xffu, vis = 0u;
    if constexpr (KEPT) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int p = __shfl(tile.kp, 16 * (i >> 2) + 4 * a4 + (i & 3));  // -1 past the list
        valid &= (p >= 0 && p < L) ? 0xffu : ~(1u << i);
      }
    } else if constexpr (FULL) {
      vis = cls == TILE_VIS ? 0xffu : 0u;
    } else {
      if (t_end - t0 < 32) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (t0 + 16 * (i >> 2) + 4 * a4 + (i & 3) >= t_end) valid &= ~(1u << i);
      }
      const unsigned valid_rows = valid;
      if (t_end > L0) {
        // several queries: the rows after a query's own position are hidden from it
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (t0 + 16 * (i >> 2) + 4 * a4 + (i & 3) >= lim) valid &= ~(1u << i);
      }
      if (cls == TILE_VIS) {
        vis = valid;
      } else if (cls == TILE_MIXED) {
        // the segments that meet the tile, one after another (the same for every lane)
        for (SegWalker lw = tile.w; lw.s < lw.nseg && lw.st < t_end; lw.next()) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int p = t0 + 16 * (i >> 2) + 4 * a4 + (i & 3);
            if (p >= lw.st && p < lw.en) vis |= 1u << i;
          }
        }
        vis &= valid_rows;
      }
    }

    if (VIS && (!TEXT || cls != TILE_TEXT)) {
      // ---- Eq. (5)/(6) and Eq. (2) statistics over visual rows ----
      float lmax = kNegInf;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (FULL || (vis & (1u << i))) lmax = fmaxf(lmax, z[i]);
      const bool up = lmax > m_v + a.thr_s;  // per lane; rare after the first tile
      if (__builtin_amdgcn_ballot_w64(up)) {
        Ls_v *= up ? fast_exp2((m_v - lmax) * a.inv_tau_s) : 1.f;
        Lm_v *= up ? fast_exp2((m_v - lmax) * a.inv_tau_m) : 1.f;
        m_v = up ? lmax : m_v;
      }
      float ts = 0.f, tm = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = FULL || (vis & (1u << i)) ? z[i] - m_v : kNegInf;
        ts += fast_exp2(d * a.inv_tau_s);
        tm += fast_exp2(d * a.inv_tau_m);
      }
      Ls_v += ts;
      Lm_v += tm;
      // visual logits: spill rows of zs_gp floats (this KV group's heads) by position
      if (FULL || (cls == TILE_VIS && t_end - t0 == 32)) {
        // transpose through the stage (row = token, zs_gp heads): lane (a4, n16)
        // holds head n16 for tokens 16*(i/4) + 4*a4 + i%4; then the 32 rows go
        // out as one contiguous block of 32 * zs_gp floats, 16 bytes per lane
        const int gp = a.zs_gp;
        if (n16 < gp) {
#pragma unroll
          for (int i = 0; i < 8; ++i) stage[(16 * (i >> 2) + 4 * a4 + (i & 3)) * gp + n16] = z[i];
        }
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        const u32x4* src = reinterpret_cast<const u32x4*>(stage);
        const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
            zbase + static_cast<size_t>(t0) * gp, 0, 32 * gp * 4, kRawBufferWord3);
        __builtin_amdgcn_raw_buffer_store_b128(src[lane], rows, lane * 16, 0, spill_policy(MODE));
        if (gp > 8)
          __builtin_amdgcn_raw_buffer_store_b128(src[64 + lane], rows, 1024 + lane * 16, 0, spill_policy(MODE));
      } else if (hv && vis) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (vis & (1u << i)) zbase[static_cast<size_t>(t0 + 16 * (i >> 2) + 4 * a4 + (i & 3)) * a.zs_gp + n16] = z[i];
      }
    }
    if (KEPT || (TEXT && (!VIS || cls != TILE_VIS))) {
      // ---- text rows (or kept rows): attention weights, statistics, value product ----
      const unsigned att = FULL ? 0xffu : valid & ~vis;
      float lmax = kNegInf;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (att & (1u << i)) lmax = fmaxf(lmax, z[i]);
      if (__builtin_amdgcn_ballot_w64(lmax > m_t + a.thr_t)) {
        // the four lanes of a head share the reference (their weights meet in one MFMA)
        const float tm = max_over_quads(lmax);
        const bool up = tm > m_t + a.thr_t;
        const float d = m_t - tm;
        const float al = up ? fast_exp2(d) : 1.f;
        l_t *= al;
        if constexpr (TSTATS) {
          Lm_t *= up ? fast_exp2(d * a.inv_tau_m) : 1.f;
          Ls_t *= up ? fast_exp2(d * a.inv_tau_s) : 1.f;
        }
        if constexpr (ATTN) {
#pragma unroll
          for (int i = 0; i < C::ACC_N; ++i) acc[i] *= al;
        }
        m_t = up ? tm : m_t;
      }
      float p[8];
      float ps = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        p[i] = (att & (1u << i)) ? fast_exp2(z[i] - m_t) : 0.f;
        ps += p[i];
      }
      l_t += ps;
      if constexpr (TSTATS) {
        float tm = 0.f, ts = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float d = (att & (1u << i)) ? z[i] - m_t : kNegInf;
          tm += fast_exp2(d * a.inv_tau_m);
          if (!a.tau_s_one) ts += fast_exp2(d * a.inv_tau_s);
        }
        Lm_t += tm;
        Ls_t += ts;
      }
      if constexpr (ATTN) {
        if (__builtin_amdgcn_ballot_w64(att != 0u)) value_product<DT, D, C::ACC_N>(acc, vblk, p, a4, n16);
      }
    }
  }
};

// LDS layout of one pass: per sub-tile a K block, a V block (passes that read
// V) and a logit stage (visual pass); the total also sets how many work-groups
// stay resident per CU
template <int DT, int D, int MODE, int W>
struct PassLds {
  using C = Cfg<DT, D>;
  using P = Pass<DT, D, MODE>;
  static constexpr int VB = P::ATTN ? C::SUB_ROWS_BYTES : 0;
  static constexpr int SB = P::VIS ? C::STAGE_BYTES : 0;
  static constexpr int SUB = C::SUB_ROWS_BYTES + VB + SB;
  static constexpr int BYTES = W > 1 ? SUB : max_i(SUB, lds_floor(DT, MODE));  // per wave
};

// Per-head statistics of the W waves of a work-group, gathered in LDS
// ([0..2] visual {m, Ls, Lm}, [3..6] text {m, l, Lm, Ls})
template <int W>
struct WaveStats {
  float v[W][16][8];
};

// Merges the partials of a work-group's W waves (every wave calls it, waves
// without tiles included, with m = -inf and sums of zero) and writes the part's
// statistics and attention partial. Each wave leaves its maxima, sums and
// accumulator in LDS (accumulator rows padded by four floats: consecutive heads
// start on different banks); after the one barrier wave 0 merges the visual
// statistics and the last wave the text ones (sums in double), and the block adds the W
// accumulators in wave order, each rescaled to the common maximum.
template <int DT, int D, int MODE, int W>
__device__ __forceinline__ void combine_waves(const AttendArgs& a, Pass<DT, D, MODE>& s, WaveStats<W>& ws,
                                              unsigned char* lds, int wave, int part, int g, int b, float m_v,
                                              float ls_v, float lm_v, float l_t, float lm_t, float ls_t) {
  using C = Cfg<DT, D>;
  using P = Pass<DT, D, MODE>;
  constexpr int PITCH = D + 4;
  static_assert(16 * PITCH * 4 <= PassLds<DT, D, MODE, W>::BYTES, "accumulator rows of a wave");
  if (s.a4 == 0) {
    float* o = ws.v[wave][s.n16];
    if constexpr (P::VIS) {
      o[0] = m_v;
      o[1] = ls_v;
      o[2] = lm_v;
    }
    if constexpr (P::TEXT) {
      o[3] = s.m_t;
      o[4] = l_t;
      o[5] = lm_t;
      o[6] = ls_t;
    }
  }
  if constexpr (P::ATTN)
    store_acc<DT, D, C::ACC_N>(reinterpret_cast<float*>(lds + wave * PassLds<DT, D, MODE, W>::BYTES) + s.n16 * PITCH,
                               s.acc, s.a4);
  __syncthreads();
  // the common maximum of column c of head h
  auto top = [&](int h, int c) {
    float M = kNegInf;
#pragma unroll
    for (int w = 0; w < W; ++w) M = fmaxf(M, ws.v[w][h][c]);
    return M;
  };
  // the weight of wave w's sums after its maximum (column c) is raised to M, at 1/tau
  auto weight = [&](int w, int h, int c, float M, float inv_tau) {
    const float m = ws.v[w][h][c];
    return m == kNegInf ? 0.f : fast_exp2((m - M) * inv_tau);
  };
  const size_t head0 = static_cast<size_t>(b) * a.T * a.Hq + static_cast<size_t>(g) * a.T * a.G;
  if (s.a4 == 0 && s.hv) {
    const int h = s.n16;
    float* st = a.stats + ((head0 + h) * a.nparts + part) * 8;
    if (P::VIS && wave == 0) {
      const float M = top(h, 0);
      double ls = 0.0, lm = 0.0;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        ls += static_cast<double>(weight(w, h, 0, M, a.inv_tau_s)) * ws.v[w][h][1];
        lm += static_cast<double>(weight(w, h, 0, M, a.inv_tau_m)) * ws.v[w][h][2];
      }
      *reinterpret_cast<float4*>(st) = make_float4(M, static_cast<float>(ls), static_cast<float>(lm), 0.f);
    }
    if (P::TEXT && wave == W - 1) {
      const float M = top(h, 3);
      double l = 0.0, lm = 0.0, ls = 0.0;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        l += static_cast<double>(weight(w, h, 3, M, 1.f)) * ws.v[w][h][4];
        if constexpr (P::TSTATS) {
          lm += static_cast<double>(weight(w, h, 3, M, a.inv_tau_m)) * ws.v[w][h][5];
          ls += static_cast<double>(weight(w, h, 3, M, a.inv_tau_s)) * ws.v[w][h][6];
        }
      }
      if constexpr (P::TSTATS)
        *reinterpret_cast<float4*>(st + 4) =
            make_float4(M, static_cast<float>(l), static_cast<float>(lm), static_cast<float>(ls));
      else
        *reinterpret_cast<float2*>(st + 4) = make_float2(M, static_cast<float>(l));
    }
  }
  if constexpr (P::ATTN) {
    constexpr int COLS = D / 4;
    for (int i = threadIdx.x; i < a.T * a.G * COLS; i += 64 * W) {
      const int h = i / COLS, c = i % COLS;
      const float M = top(h, 3);
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float f = weight(w, h, 3, M, 1.f);
        const float4 x = reinterpret_cast<const float4*>(
            reinterpret_cast<const float*>(lds + w * PassLds<DT, D, MODE, W>::BYTES) + h * PITCH)[c];
        t.x = fmaf(f, x.x, t.x);
        t.y = fmaf(f, x.y, t.y);
        t.z = fmaf(f, x.z, t.z);
        t.w = fmaf(f, x.w, t.w);
      }
      reinterpret_cast<float4*>(a.acc + ((head0 + h) * a.nparts + part) * D)[c] = t;
    }
  }
}

// Once per sequence in a launch with the visual role, by one wave: a new step's
// arrival counters of the sequence's T*U selection rows at zero, and the
// sequence's clipped segment table (positions and visual ranks) for the select
// kernel. It has a work-group of its own where the launch leaves slots free (the
// one-wave passes, small steps); in a launch that fills the GPU a wave of the
// sequence's last part of KV head 0 does it (there, extra work-groups push the
// launch past one resident round: 52 -> 61 us at the 8 x 10.8k batch of the 72B
// shape; in a small step, that wave is on the critical path: the fp32 step of 384
// tokens 23.4 -> 24.4 us).
template <int D>
__device__ __forceinline__ void step_setup(const AttendArgs& a, int b) {
  const int lane = threadIdx.x & 63;
  for (int i = lane; i < a.T * a.U; i += 64)
    reinterpret_cast<uint32_t*>(a.kacc)[arrival_word(b, i / a.U, i % a.U, a.Hq, a.G, a.T, a.U, a.nsplit, D)] = 0u;
  if (a.segtab) {
    const int L = vis_len(clamp_len(a.seq_len[b], a.max_seq_len), a.T);
    const int o0 = a.seg_off[b];
    load_segments(static_cast<SegTable*>(a.segtab)[b], a.seg + 2 * static_cast<long>(o0), a.seg_off[b + 1] - o0, L,
                  lane);
  }
}

// The work of one wave (part `part` of KV head g of sequence b; in the kept
// pass gy = g*T + t also names the query t whose kept list it reads). Of the W
// waves that share a part, wave w takes the tiles part + nparts*w, every
// nparts*W; the kept pass has one wave per part.
template <int DT, int D, int MODE, int W = 1>
__device__ __forceinline__ void attend_body(const AttendArgs& a, unsigned char* lds_block, int part, int gy, int b,
                                            int wave = 0, WaveStats<W>* ws = nullptr) {
  using C = Cfg<DT, D>;
  using P = Pass<DT, D, MODE>;
  using Q = PassLds<DT, D, MODE, W>;
  constexpr int VB = Q::VB;
  constexpr bool BOTH = P::VIS && P::ATTN;  // both roles
  constexpr bool PAIRS = BOTH && W > 1;     // two visual tiles per step (single-wave parts of both roles have one tile)
  unsigned char* lds = lds_block + wave * Q::BYTES;
  lds_byte* lds_dma = (lds_byte*)lds;  // the copies' view of it (converted once: a generic pointer may be null)

  P s(a);
  s.lane = threadIdx.x & 63;
  s.n16 = s.lane & 15;
  s.a4 = s.lane >> 4;
  s.L = clamp_len(a.seq_len[b], a.max_seq_len);
  s.kept = nullptr;
  const int qk = P::KEPT ? gy % a.T : 0;  // kept pass: the query
  const int g = P::KEPT ? gy / a.T : gy;   // KV head
  // lane row n16 <-> virtual head vh of this KV head: query vh / G, head g*G + vh % G
  const int vh = P::KEPT ? qk * a.G + s.n16 : s.n16;
  s.hv = s.n16 < (P::KEPT ? a.G : a.T * a.G);
  const int tq = s.hv ? vh / a.G : 0;
  s.h = g * a.T * a.G + vh;
  int kp0 = -2;  // kept pass: the first tile's kept positions, requested with the budget
  if constexpr (P::KEPT) {
    // the selection row of query qk that KV head g belongs to
    const size_t row = (static_cast<size_t>(b) * a.T + qk) * a.U + g / (a.Hkv / a.U);
    s.kept = a.vis_idx + row * a.k_cap;
    s.r0 = part * a.split;
    const int t = s.r0 + s.lane;
    kp0 = (s.lane < 32 && t < a.k_cap) ? s.kept[t] : -1;  // entries past the budget are masked below
    int kb = a.kk[row];
    kb = kb < 0 ? 0 : (kb > a.k_cap ? a.k_cap : kb);
    s.r1 = s.L == 0 ? s.r0 : min(s.r0 + a.split, kb);
    s.step = 32;
  } else {
    s.r0 = 32 * (part + a.nparts * wave);
    s.r1 = s.L;
    s.step = 32 * a.nparts * W;
  }
  // the query rows load while the length and the budget arrive
  const size_t qrow = s.hv ? (static_cast<size_t>(b) * a.T + tq) * a.Hq + g * a.G + (vh - tq * a.G) : 0;
  load_q<DT, D>(s.qf, static_cast<const char*>(a.q) + qrow * C::ROWB, s.hv, s.a4);
  if (W == 1 && s.r0 >= s.r1) {
    // no rows: an empty partial (max -inf, sum 0), so that the merge can read
    // every part's slot without first learning the length and the budget
    if constexpr (P::ATTN) {
      if (s.hv && s.a4 == 0) {
        if constexpr (P::KEPT) {
          const size_t row = (static_cast<size_t>(b) * a.T * a.Hq + s.h) * a.nsplit + part;
          *reinterpret_cast<float2*>(a.kstats + row * 2) = make_float2(kNegInf, 0.f);
        } else {
          const size_t row = (static_cast<size_t>(b) * a.T * a.Hq + s.h) * a.nparts + part;
          if constexpr (P::TSTATS)
            *reinterpret_cast<float4*>(a.stats + row * 8 + 4) = make_float4(kNegInf, 0.f, 0.f, 0.f);
          else
            *reinterpret_cast<float2*>(a.stats + row * 8 + 4) = make_float2(kNegInf, 0.f);
        }
      }
    }
    return;
  }

  s.L0 = s.L - a.T + 1;
  s.lim = s.L0 + tq;
  // contiguous caches: sequence b's rows from its base; paged caches: rows of
  // physical blocks (the block offset is added per row)
  constexpr bool paged = P::PAGED;
  const size_t seq_off = paged ? 0 : static_cast<size_t>(b) * a.sb;
  s.Kb = static_cast<const char*>(a.K) + (seq_off + static_cast<size_t>(g) * a.sh) * C::ESZ;
  s.Vb = P::ATTN ? static_cast<const char*>(a.V) + (seq_off + static_cast<size_t>(g) * a.sh) * C::ESZ : nullptr;
  s.rstride = static_cast<size_t>(a.ss) * C::ESZ;
  s.bt = paged ? a.block_table + static_cast<size_t>(b) * a.nblk : nullptr;
  s.bstride = static_cast<size_t>(a.sb) * C::ESZ;
  s.bmask = paged ? (1 << a.bs_log2) - 1 : 0;
  if constexpr (!P::KEPT) s.init_row_step();
  s.m_v = kNoLogit;
  s.Ls_v = s.Lm_v = 0.f;
  s.m_t = kNoLogit;
  s.l_t = s.Lm_t = s.Ls_t = 0.f;
#pragma unroll
  for (int i = 0; i < C::ACC_N; ++i) s.acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  s.zbase = (P::VIS || P::ZSPILL)
                ? a.zs + (static_cast<size_t>(b) * a.Hkv + g) * a.zs_rows * static_cast<size_t>(a.zs_gp) + qk * a.G
                : nullptr;

  // a wave of both roles needs its first tile's K rows whatever they are: they are
  // requested before the segments are known
  bool k_early = false;
  if constexpr (BOTH && !P::PAGED) {
    k_early = s.even && s.r0 + 32 <= s.L;
    if (k_early) s.copy_even_rows(s.Kb + static_cast<size_t>(s.r0) * s.rstride, lds_dma);
  }
  // the step setup waits for its loads in the shadow of the first tile's copies
  bool setup = P::VIS && W > 1 && static_cast<int>(gridDim.x) == a.nparts && g == 0 && part == a.nparts - 1 &&
               wave == W - 1;

  Sub cur;
  cur.t0 = s.r0;
  cur.cls = TILE_TEXT;
  if constexpr (!P::KEPT) {
    const int o0 = a.seg_off[b];
    cur.w.start(a.seg + 2 * static_cast<long>(o0), a.seg_off[b + 1] - o0, vis_len(s.L, a.T));
  }
  cur = s.sub_at(cur, s.r0, kp0);

  // All copies of a step are issued before any of it is used. A step is one tile,
  // or, with both roles, two visual tiles of the wave (the second one's K rows in
  // the block that holds a text tile's V rows), so that a wave has 16 KB in
  // flight whatever its tiles hold.
  while (cur.t0 < s.r1) {
    const Sub t0 = cur;
    const bool act = s.active(t0);
    Sub t1 = t0;
    bool pair = false;
    if constexpr (PAIRS) {
      if (t0.cls == TILE_VIS) {
        t1 = s.sub_at(t0, t0.t0 + s.step);
        pair = t1.t0 < s.r1 && t1.cls == TILE_VIS;
      }
    }
    // The work-group's waves share nothing here, so ordering needs counters, not
    // barriers (a barrier's release fence would also wait for the logit stores of
    // the previous tile). LDS reads of the previous tile must have returned before
    // the copies overwrite it:
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    float zk[8];
    if (act) {
      // the 16 copy destinations are added up per tile, not held in scalar registers
      lds_byte* dma = lds_dma;
      if constexpr (W > 1) unhoist_scalar(dma);
      if (!P::KEPT && s.even && t0.t0 + 32 <= s.L) {
        const size_t off = s.tile_offset(t0);
        if (!k_early) s.copy_even_rows(s.Kb + off, dma);
        k_early = false;
        if (s.needs_v(t0)) s.copy_even_rows(s.Vb + off, dma + C::SUB_ROWS_BYTES);
      } else {
        size_t off[C::COPIES];
        if constexpr (P::WHOLE) s.unhoist_lane();
        s.row_offsets(t0, off);
        if constexpr (!P::ZSPILL) s.copy_rows(s.Kb, off, dma);
        if (s.needs_v(t0)) s.copy_rows(s.Vb, off, dma + C::SUB_ROWS_BYTES);
      }
      if (pair) {
        if (s.even && t1.t0 + 32 <= s.L) {
          s.copy_even_rows(s.Kb + s.tile_offset(t1), dma + C::SUB_ROWS_BYTES);
        } else {
          size_t off[C::COPIES];
          if constexpr (P::WHOLE) s.unhoist_lane();
          s.row_offsets(t1, off);
          s.copy_rows(s.Kb, off, dma + C::SUB_ROWS_BYTES);
        }
      }
      if constexpr (P::ZSPILL) s.load_spill(t0, zk);
    }
    // the next step's kept positions / segment state load while these copies fly
    cur = s.sub_at(pair ? t1 : t0, (pair ? t1.t0 : t0.t0) + s.step);
    if (setup) {
      step_setup<D>(a, b);
      setup = false;
    }
    if (!act) continue;  // (nothing was copied: no wait)
    // the copies have landed in LDS once the vector-memory counter drains
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    unsigned char* kblk = lds;
    unsigned char* vblk = lds + C::SUB_ROWS_BYTES;
    float* stage = reinterpret_cast<float*>(vblk + VB);
    Sub t = t0;
#pragma unroll 1
    for (int i = 0;; ++i) {
      if (P::WHOLE && t.cls != TILE_MIXED && t.t0 + 32 <= min(s.L, s.L0)) {
        s.template process<P::WHOLE>(t, kblk, vblk, stage, zk);
      } else {
        if constexpr (P::WHOLE) s.unhoist_lane();
        s.template process<false>(t, kblk, vblk, stage, zk);
      }
      if (!PAIRS || !pair || i == 1) break;
      t = t1;
      kblk = vblk;
    }
  }

  // ---- write this part's partials ----
  float M_v = kNegInf, ls_v = 0.f, lm_v = 0.f;
  if constexpr (P::VIS) {
    // merge the four lanes' statistics onto their common maximum
    M_v = max_over_quads(s.m_v);
    const bool any = s.m_v != kNoLogit;
    const float fs = any ? fast_exp2((s.m_v - M_v) * a.inv_tau_s) : 0.f;
    const float fm = any ? fast_exp2((s.m_v - M_v) * a.inv_tau_m) : 0.f;
    ls_v = sum_over_quads(s.Ls_v * fs);
    lm_v = sum_over_quads(s.Lm_v * fm);
    M_v = M_v == kNoLogit ? kNegInf : M_v;
    if (W == 1 && s.hv && s.a4 == 0) {
      float* st = a.stats + ((static_cast<size_t>(b) * a.T * a.Hq + s.h) * a.nparts + part) * 8;
      *reinterpret_cast<float4*>(st) = make_float4(M_v, ls_v, lm_v, 0.f);
    }
  }
  s.m_t = s.m_t == kNoLogit ? kNegInf : s.m_t;
  if constexpr (W > 1) {
    if (setup) step_setup<D>(a, b);  // a wave without tiles
    const float s_lt = P::TEXT ? sum_over_quads(s.l_t) : 0.f;
    const float s_lm = P::TSTATS ? sum_over_quads(s.Lm_t) : 0.f;
    const float s_ls = P::TSTATS ? (a.tau_s_one ? s_lt : sum_over_quads(s.Ls_t)) : 0.f;
    combine_waves<DT, D, MODE, W>(a, s, *ws, lds_block, wave, part, g, b, M_v, ls_v, lm_v, s_lt, s_lm, s_ls);
  } else if constexpr (P::KEPT || P::TEXT) {
    const float s_lt = sum_over_quads(s.l_t);
    const float s_lm = P::TSTATS ? sum_over_quads(s.Lm_t) : 0.f;
    const float s_ls = P::TSTATS ? (a.tau_s_one ? s_lt : sum_over_quads(s.Ls_t)) : 0.f;
    if (s.hv) {
      if constexpr (P::KEPT) {
        const size_t row = (static_cast<size_t>(b) * a.T * a.Hq + s.h) * a.nsplit + part;
        if (s.a4 == 0) *reinterpret_cast<float2*>(a.kstats + row * 2) = make_float2(s.m_t, s_lt);
        store_acc<DT, D, C::ACC_N>(a.kacc + row * D, s.acc, s.a4);
      } else {
        const size_t row = (static_cast<size_t>(b) * a.T * a.Hq + s.h) * a.nparts + part;
        if (s.a4 == 0) {
          if constexpr (P::TSTATS)
            *reinterpret_cast<float4*>(a.stats + row * 8 + 4) = make_float4(s.m_t, s_lt, s_lm, s_ls);
          else
            *reinterpret_cast<float2*>(a.stats + row * 8 + 4) = make_float2(s.m_t, s_lt);
        }
        if constexpr (P::ATTN) store_acc<DT, D, C::ACC_N>(a.acc + row * D, s.acc, s.a4);
      }
    }
  }
}

template <int DT, int D, int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(attend_waves(DT, MODE)))) void attend_kernel(
    const AttendArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[PassLds<DT, D, MODE, 1>::BYTES];
  if ((base_mode(MODE) & MODE_VIS) != 0 && static_cast<int>(blockIdx.x) == a.nparts) {
    if (blockIdx.y == 0) step_setup<D>(a, blockIdx.z);
    return;
  }
  attend_body<DT, D, MODE>(a, lds, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The index of this thread's wave in its work-group, as a scalar
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6); }

// W waves per part: both roles of the context pass in one launch (MODE_BOTH,
// or MODE_BOTH_STATS when no V is given). Every
// wave takes whatever its tiles hold: a visual tile's K rows, a text tile's K
// and V rows (a mixed tile is read once for both).
template <int DT, int D, int MODE, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(attend_waves(DT, MODE)))) void
attend_waves_kernel(const AttendArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[W * PassLds<DT, D, MODE, W>::BYTES];
  __shared__ WaveStats<W> ws;
  static_assert((sizeof(lds) + sizeof(ws)) * (resident_groups(DT, D) / 256) <= 160 * 1024, "work-groups of a CU");
  const int wave = wave_index();
  if (static_cast<int>(blockIdx.x) == a.nparts) {
    if (wave == 0 && blockIdx.y == 0) step_setup<D>(a, blockIdx.z);
    return;
  }
  attend_body<DT, D, MODE, W>(a, lds, blockIdx.x, blockIdx.y, blockIdx.z, wave, &ws);
}

// A later layer's text attention pass and kept pass in one launch (their rows
// are disjoint and the kept list is the anchor layer's, known before the
// launch): per (KV head, sequence) the work-groups of the text parts, then those
// of T*splits kept splits, one split per wave. Each does what it does in its
// own launch, so the partials are the same bits, and the kept work-groups fill
// the text pass's tail.
template <int DT, int D, int PG, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(attend_waves(DT, MODE_TEXT_ATTN)))) void
attend_text_kept_kernel(const AttendArgs a) {
  constexpr int TEXT = MODE_TEXT_ATTN | PG;
  constexpr int KEPT = MODE_KEPT | PG;
  static_assert(PassLds<DT, D, TEXT, W>::BYTES == PassLds<DT, D, KEPT, W>::BYTES, "LDS blocks of the waves");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[W * PassLds<DT, D, TEXT, W>::BYTES];
  __shared__ WaveStats<W> ws;
  const int wave = wave_index();
  int x = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const unsigned pairs = gridDim.y * gridDim.z;
  const unsigned kept_groups = gridDim.x - a.nparts;  // of a pair
  if (W > 1 && 12 * kept_groups * pairs > resident_groups(DT, D)) {
    // the text work-groups of every pair come first: they fill the launch's first
    // round by themselves, and the short kept ones follow as slots fall free. With
    // the two interleaved, the last pairs' text work-groups waited for that round
    // (a later layer at 72 (sequence, KV head) pairs x 10k tokens 53.5 -> 44.5 us,
    // 80 x 9k 52.7 -> 43.5, 256 x 4k 64.4 -> 55.5; kept ones first: 47.3, 44.9, 59.5).
    // With few kept work-groups that wait is short, and theirs at the end is not:
    // interleaved (a launch of 512 text and 16 kept ones, 8 pairs x 8k tokens, 14.4
    // us, text first 15.7; 32 kept, 16 x 9k, 18.5 and 19.6; but 64 kept, 32 x 9k, 25.9
    // and 24.1)
    const unsigned n = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned n_text = a.nparts * pairs;
    const unsigned x0 = n < n_text ? 0 : a.nparts;
    const unsigned per_pair = n < n_text ? a.nparts : kept_groups;
    const unsigned i = n < n_text ? n : n - n_text;
    const unsigned pair = i / per_pair;
    x = static_cast<int>(x0 + i - pair * per_pair);
    b = static_cast<int>(pair / gridDim.y);
    g = static_cast<int>(pair - b * gridDim.y);
  }
  if (x < a.nparts) {
    attend_body<DT, D, TEXT, W>(a, lds, x, g, b, wave, &ws);
  } else {
    const int j = (x - a.nparts) * W + wave;
    const int t = j / a.nsplit;
    if (t < a.T)
      attend_body<DT, D, KEPT>(a, lds + wave * PassLds<DT, D, KEPT, W>::BYTES, j - t * a.nsplit, g * a.T + t, b);
  }
}

// Launches one pass. With events given, they are attached to the launch itself
// (hipExtLaunchKernel): they time the kernel's execution alone, as a profiler does.
template <typename K>
hipError_t launch_one(K kernel, dim3 grid, int threads, const AttendArgs& a, hipStream_t st, hipEvent_t ev0,
                      hipEvent_t ev1) {
  if (ev0 || ev1) {
    void* args[1] = {const_cast<AttendArgs*>(&a)};
    return hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(threads), args, 0, st, ev0, ev1, 0);
  }
  hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, a);
  return hipGetLastError();
}

// the one-wave passes of large caches, and the kept pass
template <int DT, int D, int PG>
hipError_t launch_single(const AttendArgs& a, int mode, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const bool kept = base_mode(mode) == MODE_KEPT;
  int gx = a.nparts;
  if (kept) gx = a.nsplit;
  else if ((mode & MODE_VIS) != 0) gx = a.nparts + 1;  // the step setup
  else if (mode == MODE_TEXT_KEPT) gx = a.nparts + a.T * a.nsplit;
  const dim3 grid(gx, kept ? a.Hkv * a.T : a.Hkv, a.B);
  switch (mode) {
    case MODE_TEXT_KEPT: return launch_one(attend_text_kept_kernel<DT, D, PG, 1>, grid, 64, a, st, ev0, ev1);
    case MODE_VIS: return launch_one(attend_kernel<DT, D, MODE_VIS | PG>, grid, 64, a, st, ev0, ev1);
    case MODE_TEXT_STATS: return launch_one(attend_kernel<DT, D, MODE_TEXT_STATS | PG>, grid, 64, a, st, ev0, ev1);
    case MODE_TEXT_ATTN: return launch_one(attend_kernel<DT, D, MODE_TEXT_ATTN | PG>, grid, 64, a, st, ev0, ev1);
    case MODE_TEXT_BOTH: return launch_one(attend_kernel<DT, D, MODE_TEXT_BOTH | PG>, grid, 64, a, st, ev0, ev1);
    case MODE_KEPT: return launch_one(attend_kernel<DT, D, MODE_KEPT | PG>, grid, 64, a, st, ev0, ev1);
    case MODE_KEPT | MODE_ZSPILL:
      return launch_one(attend_kernel<DT, D, MODE_KEPT | MODE_ZSPILL | PG>, grid, 64, a, st, ev0, ev1);
    case MODE_BOTH:  // (both roles in one wave per part: fp32 only, see make_plan)
      if constexpr (DT == VP_F32) return launch_one(attend_kernel<DT, D, MODE_BOTH | PG>, grid, 64, a, st, ev0, ev1);
      return hipErrorInvalidValue;
    case MODE_BOTH_STATS:
      if constexpr (DT == VP_F32)
        return launch_one(attend_kernel<DT, D, MODE_BOTH_STATS | PG>, grid, 64, a, st, ev0, ev1);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

// the passes with kPartWaves waves per part
template <int DT, int D, int PG>
hipError_t launch_waves(const AttendArgs& a, int mode, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  constexpr int W = kPartWaves;
  int gx = a.nparts;
  if ((mode & MODE_VIS) != 0 && static_cast<int64_t>(a.nparts + 1) * a.Hkv * a.B <= resident_groups(DT, D))
    gx = a.nparts + 1;  // room for the step setup's own work-groups
  else if (mode == MODE_TEXT_KEPT) gx = a.nparts + (a.T * a.nsplit + W - 1) / W;
  const dim3 grid(gx, a.Hkv, a.B);
  switch (mode) {
    case MODE_TEXT_ATTN:  // the text parts alone
    case MODE_TEXT_KEPT: return launch_one(attend_text_kept_kernel<DT, D, PG, W>, grid, 64 * W, a, st, ev0, ev1);
    case MODE_BOTH: return launch_one(attend_waves_kernel<DT, D, MODE_BOTH | PG, W>, grid, 64 * W, a, st, ev0, ev1);
    case MODE_BOTH_STATS:
      return launch_one(attend_waves_kernel<DT, D, MODE_BOTH_STATS | PG, W>, grid, 64 * W, a, st, ev0, ev1);
    default: return hipErrorInvalidValue;
  }
}

template <int DT, int D, int PG>
hipError_t launch_dd(const AttendArgs& a, int mode, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  return a.waves == 1 || base_mode(mode) == MODE_KEPT ? launch_single<DT, D, PG>(a, mode, st, ev0, ev1)
                                                      : launch_waves<DT, D, PG>(a, mode, st, ev0, ev1);
}

}  // namespace

hipError_t launch_attend(const AttendArgs& a, int mode, int dtype, int head_dim, hipStream_t st, hipEvent_t ev0,
                         hipEvent_t ev1) {
  const bool paged = a.bs_log2 >= 0;
  if (dtype == VP_BF16) {
    if (head_dim == 128)
      return paged ? launch_dd<VP_BF16, 128, MODE_PAGED>(a, mode, st, ev0, ev1) : launch_dd<VP_BF16, 128, 0>(a, mode, st, ev0, ev1);
    if (head_dim == 64)
      return paged ? launch_dd<VP_BF16, 64, MODE_PAGED>(a, mode, st, ev0, ev1) : launch_dd<VP_BF16, 64, 0>(a, mode, st, ev0, ev1);
  } else if (dtype == VP_F32) {
    if (head_dim == 128)
      return paged ? launch_dd<VP_F32, 128, MODE_PAGED>(a, mode, st, ev0, ev1) : launch_dd<VP_F32, 128, 0>(a, mode, st, ev0, ev1);
    if (head_dim == 64)
      return paged ? launch_dd<VP_F32, 64, MODE_PAGED>(a, mode, st, ev0, ev1) : launch_dd<VP_F32, 64, 0>(a, mode, st, ev0, ev1);
  }
  return hipErrorInvalidValue;
}

}  // namespace vp
