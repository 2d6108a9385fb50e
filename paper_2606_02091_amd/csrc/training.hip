// Training-side kernels of the block diffusion draft model and their C-ABI entry points:
//   * anchor attention (Sec. 3.3): the sampled blocks of a sequence are processed together;
//     the rows of block i (anchored at position a_i) attend to the context features of the
//     positions before a_i and to the B positions of their own block, never to another
//     block.  Forward (outputs, log-sum-exp) and backward (dQ, context dK/dV, block dK/dV).
//   * progressive position-weighted cross-entropy (Sec. 4.3, Eq. 5): weights
//     w_k = exp(-(k - 1) / gamma) on the k-th masked position of each block, the loss is
//     their weighted mean; forward and the gradient of the logits.
//
// Matrix products run on the bf16 matrix cores.  Scores are formed transposed (S^T = K Q^T) where
// the probabilities feed a product over keys (P V, dS K), and untransposed (S = Q K^T) where they
// feed a product over query rows (P^T dO, dS^T Q), so that the score tile a wave has just computed
// is the other product's B operand without leaving the registers.  That product's A operand is a
// transposed tile (V^T, K^T, Q^T, dO^T), read from LDS by the transposing read (ds_read_b64_tr_b16), so
// no transposed copy exists anywhere.
//
// Tiles reach LDS through registers, a tile ahead: loaded while the tile before is worked on, stored
// after the barrier that ends it.  LDS-direct loads would save these registers, but the compiler waits
// for all of them before any LDS read that follows, so that a tile's products waited for the loads
// just issued for the next (context dK, dV of 512 blocks, T = 3,072: 580 against 500 us).
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "device_common.h"
#include "dflare.h"

namespace dflare {

namespace {

constexpr int kTrT = 256;  // threads per work-group (4 waves)
constexpr int kChunkBlocks = 64;  // most blocks per partial of the context-key gradients
constexpr int kMaxBlockKeys = 16;  // block size B the training entry points accept
// (block, KV head) pairs up to which a block's key tiles are split over a work-group's waves: above
// one pair per CU the waves of further blocks occupy the chip without a merge.  Up to 256 pairs the split is ahead or
// even in every form measured (forward, whole / split, heads of 128: 256 pairs of 32 rows, T = 3,072 74 / 49 us, T = 500
// 19 / 16; of 64 rows 76 / 54 and 20 / 17; heads of 64, 32 rows 52 / 28 and 17 / 17).  Above, long contexts still favour it
// (512 pairs of 32 rows, T = 3,072: 74 / 65) and short ones do not (T = 500: 384 pairs 20 / 23, 512 20 / 25), and from
// 768 pairs neither does (73 / 86); anchors are not known to the host, so the line is where it never loses.  Blocks
// of 65 to 128 rows occupy three or four waves themselves and are not split: their merge would need
// work-groups of eight waves with twice the LDS.
constexpr long kRowsSplitMax = 256;

struct AttnShapeT {
  int n_blocks, B, T, n_q, n_kv, hd;
  int G, R, Rp;  // heads per group, rows per (block, group), the same padded to 32
};

struct AttnT {
  AttnShapeT s;
  const uint16_t *q, *kc, *vc, *kb, *vb;  // bf16 inputs
  const int32_t* anchors;
  // workspace
  uint16_t *qf, *df;                // [n_kv][n_blocks][Rp / 32][32 x hd] Q and dO (bf16) rows in fragment tiles
  float* st;                        // [n_kv][n_blocks][2][Rp] -lse / scale, -rowsum(dO O); (-inf, 0) past R
  float* part;                      // [nch][T][n_kv][hd] x2 (dK, dV)
  int* order;                       // [n_blocks] blocks by decreasing anchor (work order)
  int nch;                          // chunks of the context-key gradients: chunk z takes order[z], order[z + nch], ...
  // outputs
  float *out, *lse;
  const float* dout;
  float *dq, *dkc, *dvc, *dkb, *dvb;
  float scale;
};

__device__ __forceinline__ u32x4 ld16(const uint16_t* p) { return *reinterpret_cast<const u32x4*>(p); }
// two fp32 values -> two bf16 (round to nearest even) in one word, by the packed conversion
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_bf2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), bf16x2_t));
}
// two result tiles of a lane (4 + 4 values) as one bf16 operand (k order 0..3, then 16..19)
__device__ __forceinline__ u32x4 pack_bf8(f32x4 x, f32x4 y) {
  return u32x4{cvt_bf2(x[0], x[1]), cvt_bf2(x[2], x[3]), cvt_bf2(y[0], y[1]), cvt_bf2(y[2], y[3])};
}
// 2^x by the hardware instruction: results below 2^-126 (far below a bf16 probability's
// resolution) are not kept as denormals; 2^-inf = 0
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                 0, 0);
}
__device__ __forceinline__ f32x16 splat16(float x) {
  f32x16 v;
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = x;
  return v;
}
// registers 8 ks .. 8 ks + 7 of a 32 x 32 result tile as one bf16 operand (16 values of k)
__device__ __forceinline__ u32x4 pack_half(const f32x16& x, int ks) {
  return u32x4{cvt_bf2(x[8 * ks], x[8 * ks + 1]), cvt_bf2(x[8 * ks + 2], x[8 * ks + 3]),
               cvt_bf2(x[8 * ks + 4], x[8 * ks + 5]), cvt_bf2(x[8 * ks + 6], x[8 * ks + 7])};
}

// barrier that waits for this wave's LDS operations only: its loads into registers stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---- fragment tiles: 32 rows of HD bf16, in memory and in LDS alike.  The 16-byte piece c = 2 k + h of
// a row is an operand's piece for k-step k and lane half h: fragment k is 1 KB, piece (row, h) in slot
// 32 h + (row ^ (4 h + 8 (k mod 2))).  An untransposed operand is one fragment (contiguous for a
// wave); a transposed read covers 4 rows x 32 columns per half wave, and the xor puts these in
// 256 different bytes modulo the bank cycle. ----
template <int HD>
constexpr int kTileBytes = 32 * HD * 2;
__device__ __forceinline__ int frag_slot(int row, int h, int kodd) { return 32 * h + (row ^ (4 * h + 8 * kodd)); }
// byte offset of piece c of a row
__device__ __forceinline__ int piece_at(int row, int c) {
  return (c >> 1) * 1024 + frag_slot(row, c & 1, (c >> 1) & 1) * 16;
}
// Transposed read of 4 rows r0 .. r0 + 3 x 16 columns 16 k ..: lane i of a 16-lane group gets column
// 16 k + i of the 4 rows; its address (a byte offset here) is that of row r0 + i / 4, columns
// 16 k + 4 (i mod 4).  The group's r0 and k may differ from the other groups'.
__device__ __forceinline__ int tr_at(int r0, int k, int lane) {
  const int i = lane & 15;
  return piece_at(r0 + (i >> 2), 2 * k + ((i >> 1) & 1)) + (i & 1) * 8;
}
__device__ __forceinline__ u32x2 ld_tr(const char* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDSP s16x4*)(LDSP char*)const_cast<char*>(p)));
}
// A operand (32 x 16) of a transposed tile: output rows = columns 32 dt + (0..31), k = rows
// 16 ks + {4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3} in lane half h -- the rows whose values a 32 x 32
// result tile holds in registers 8 ks .. 8 ks + 7 of that half.
__device__ __forceinline__ u32x4 ld_tr_op(const char* tile, const int (&off)[2], int ks, int dt) {
  const u32x2 lo = ld_tr(tile + dt * 2048 + ks * 256 + off[0]);
  const u32x2 hi = ld_tr(tile + dt * 2048 + ks * 256 + off[1]);
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}
__device__ __forceinline__ void tr_offsets(int lane, int (&off)[2]) {
#pragma unroll
  for (int x = 0; x < 2; ++x) off[x] = tr_at(8 * x + 4 * (lane >> 5), (lane >> 4) & 1, lane);
}
// this lane's byte offset in fragment k of an untransposed operand: o[k mod 2] + 1024 k
__device__ __forceinline__ void frag_offsets(int lane, int (&o)[2]) {
#pragma unroll
  for (int x = 0; x < 2; ++x) o[x] = frag_slot(lane & 31, lane >> 5, x) * 16;
}
__device__ __forceinline__ u32x4 ld16b(const char* p) { return *reinterpret_cast<const u32x4*>(p); }

// Work-group n of a launch over (unit, KV head) pairs.  Work-groups go to the 8 XCDs in turn, each with an
// L2 of its own; an XCD takes every 8th unit and, one after another, all KV heads of it.  So the
// work-groups that run together on an XCD read all heads: rows of one head alone lie a whole
// row of heads apart and would meet in a few of the L2's channels.
__device__ __forceinline__ void unit_head(int n, int n_kv, int& unit, int& g) {
  const int m = n / 8;
  g = m % n_kv;
  unit = m / n_kv * 8 + n % 8;
}

// ---- backward operands and block-key gradients of (block i, KV head g), one work-group each.  Row
// r < R of the pair is block position r % B of query head g G + r / B; a row is read once (Q, dO, O: 16
// bytes of bf16 per thread and piece) and gives -lse / scale and -rowsum(dO O) (st; (-inf, 0) past R) and
// the fragment tiles of Q and dO, in LDS and copied out (qf, df).  From these every wave
// forms S and dP of all rows against the block's B keys and adds up dK and dV of its HD / 4 dims. ----
template <int HD>
__global__ __launch_bounds__(kTrT) void k_bwd_prep(AttnT a, const float* out) {
  extern __shared__ char sm[];
  constexpr int PK = HD / 8, RPS = kTrT / PK;
  const AttnShapeT& s = a.s;
  int i, g;
  unit_head(blockIdx.x, s.n_kv, i, g);
  if (i >= s.n_blocks) return;
  char* tq = sm;
  char* td = sm + s.Rp * HD * 2;
  float* snl = reinterpret_cast<float*>(sm + 2 * s.Rp * HD * 2);
  float* snd = snl + s.Rp;
  const long tile = (long)g * s.n_blocks + i;
  const float rscale = 1.f / a.scale, sl2 = a.scale * 1.4426950408889634f;
  {
    const int c = threadIdx.x % PK, rs = threadIdx.x / PK;
    for (int r = rs; r < s.Rp; r += RPS) {
      const bool rv = r < s.R;
      const long rh = rv ? (long)(i * s.B + r % s.B) * s.n_q + g * s.G + r / s.B : 0;
      f32x4 x0 = zero4(), x1 = zero4(), o0 = zero4(), o1 = zero4();
      u32x4 qv = {0u, 0u, 0u, 0u};
      if (rv) {
        const f32x4* px = reinterpret_cast<const f32x4*>(a.dout + rh * HD + 8 * c);
        const f32x4* po = reinterpret_cast<const f32x4*>(out + rh * HD + 8 * c);
        x0 = px[0];
        x1 = px[1];
        o0 = po[0];
        o1 = po[1];
        qv = ld16(a.q + rh * HD + 8 * c);
      }
      const f32x4 pr = x0 * o0 + x1 * o1;
      float acc = (pr[0] + pr[1]) + (pr[2] + pr[3]);
#pragma unroll
      for (int off = PK / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
      const u32x4 dv = {f2bf(x0[0]) | (f2bf(x0[1]) << 16), f2bf(x0[2]) | (f2bf(x0[3]) << 16),
                        f2bf(x1[0]) | (f2bf(x1[1]) << 16), f2bf(x1[2]) | (f2bf(x1[3]) << 16)};
      const int at = (r >> 5) * kTileBytes<HD> + piece_at(r & 31, c);
      *reinterpret_cast<u32x4*>(tq + at) = qv;
      *reinterpret_cast<u32x4*>(td + at) = dv;
      if (c == 0) {
        const float nl = rv ? -a.lse[rh] * rscale : -INFINITY;
        snl[r] = a.st[tile * 2 * s.Rp + r] = nl;
        snd[r] = a.st[(tile * 2 + 1) * s.Rp + r] = rv ? -acc : 0.f;
      }
    }
  }
  // B operand columns (keys) of this lane: key `col`; keys past B repeat key 0 and are not stored
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 15, q4 = lane >> 4;
  u32x4 kf[HD / 32], vf[HD / 32];
  {
    const long row = ((long)(i * s.B + (col < s.B ? col : 0)) * s.n_kv + g) * HD;
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) {
      kf[ks] = ld16(a.kb + row + ks * 32 + 8 * q4);
      vf[ks] = ld16(a.vb + row + ks * 32 + 8 * q4);
    }
  }
  __syncthreads();
  {
    const long bytes = (long)s.Rp * HD * 2;
    char* qd = reinterpret_cast<char*>(a.qf) + tile * bytes;
    char* dd = reinterpret_cast<char*>(a.df) + tile * bytes;
    for (int e = threadIdx.x * 16; e < bytes; e += kTrT * 16) {
      *reinterpret_cast<u32x4*>(qd + e) = ld16b(tq + e);
      *reinterpret_cast<u32x4*>(dd + e) = ld16b(td + e);
    }
  }
  constexpr int DT = HD / 64;  // 16-dim tiles per wave
  f32x4 dk[DT], dv[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) dk[t] = dv[t] = zero4();
  for (int r0 = 0; r0 < s.Rp; r0 += 32) {
    f32x4 P[2], dS[2];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const f32x4 nl = *reinterpret_cast<const f32x4*>(snl + r0 + 16 * y + 4 * q4);
      f32x4 sc = zero4(), dp = *reinterpret_cast<const f32x4*>(snd + r0 + 16 * y + 4 * q4);
#pragma unroll
      for (int ks = 0; ks < HD / 32; ++ks) {
        const int at = r0 * HD * 2 + piece_at(16 * y + col, ks * 4 + q4);
        sc = mfma(*reinterpret_cast<const u32x4*>(tq + at), kf[ks], sc);
        dp = mfma(*reinterpret_cast<const u32x4*>(td + at), vf[ks], dp);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        P[y][e] = ex2((sc[e] + nl[e]) * sl2);
        dS[y][e] = P[y][e] * dp[e];
      }
    }
    const u32x4 pb = pack_bf8(P[0], P[1]), sb = pack_bf8(dS[0], dS[1]);
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      const int lo = r0 * HD * 2 + tr_at(4 * q4, w * DT + t, lane), hi = r0 * HD * 2 + tr_at(16 + 4 * q4, w * DT + t, lane);
      const u32x2 d0 = ld_tr(td + lo), d1 = ld_tr(td + hi), q0 = ld_tr(tq + lo), q1 = ld_tr(tq + hi);
      dv[t] = mfma(u32x4{d0[0], d0[1], d1[0], d1[1]}, pb, dv[t]);
      dk[t] = mfma(u32x4{q0[0], q0[1], q1[0], q1[1]}, sb, dk[t]);
    }
  }
  if (col < s.B) {
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      const long at = ((long)(i * s.B + col) * s.n_kv + g) * HD + (w * DT + t) * 16 + 4 * q4;
      *reinterpret_cast<f32x4*>(a.dkb + at) = dk[t] * a.scale;
      *reinterpret_cast<f32x4*>(a.dvb + at) = dv[t];
    }
  }
}

// ---- work order of the row and context-key kernels: the blocks by decreasing anchor (ties by
// index), so that the work-groups with the longest contexts start first, the blocks of one
// work-group are of nearly equal length, and a chunk's blocks that see a key come first.  Thread
// (i, part) counts the blocks of its sixteenth that go before block i. ----
__global__ __launch_bounds__(256) void k_anchor_order(const int32_t* __restrict__ anchors, int n, int T,
                                                      int* __restrict__ order) {
  __shared__ int cnt[16][17];
  const int l = threadIdx.x & 15, part = threadIdx.x >> 4;
  const int i = blockIdx.x * 16 + l;
  const int ai = i < n ? min(max(anchors[i], 0), T) : 0;
  int rank = 0;
#pragma unroll 8
  for (int j = part; j < n; j += 16) {
    const int aj = min(max(anchors[j], 0), T);
    rank += (aj > ai || (aj == ai && j < i)) ? 1 : 0;
  }
  cnt[l][part] = rank;
  __syncthreads();
  if (part == 0 && i < n) {
    for (int p = 1; p < 16; ++p) rank += cnt[l][p];
    order[rank] = i;
  }
}

// ---- forward and dQ.  A wave takes 32 query rows of a block (its B operand, in registers) through
// 32-key tiles: the context before the anchor, then the block's own keys.  A block is WPB
// waves; the 4 waves of a work-group are NB = 4 / WPB blocks that follow each other in the work
// order (KS = 1), or one block whose key tiles go to KS wave groups in turn, merged at the end.
// The K and V tiles go through two LDS buffers of KS tiles each, one barrier per buffer.
// Bound by instruction issue: per tile and wave 16 (dQ: 24) 32 x 32 x 16 products of 32 clocks and about
// 110 vector instructions, which share the issue slots of two waves per SIMD.  512 blocks of 4 x 16
// rows, T = 3,072, 8 KV heads x 128: 330 -> 255 us forward, 440 -> 325 us dQ against 16-row waves
// on 16 x 16 x 32 products.
template <int HD, bool DQ, int WPB, int KS>
__global__ __launch_bounds__(kTrT, KS == 1 ? 2 : 1) void k_aatt_rows(AttnT a) {
  constexpr int NB = KS > 1 ? 1 : 4 / WPB;
  constexpr int NK = HD / 16, ND = HD / 32;  // k-steps and dim tiles of a head
  constexpr int TB = kTileBytes<HD>;
  constexpr int PW = NK * KS / 4;            // K (and V) fragments per wave and step
  constexpr int SB = 2 * KS * TB;            // bytes of a buffer: KS K tiles, KS V tiles
  constexpr int NOWN = (NB + 1) / 2;         // tiles of own keys: 16 rows of each of two blocks (past B key B - 1)
  __shared__ __attribute__((aligned(1024))) char lds[2 * SB];
  __shared__ __attribute__((aligned(1024))) char own[2 * NOWN * TB];  // K tiles, V tiles
  const AttnShapeT& s = a.s;
  int g, unit;
  unit_head(blockIdx.x, s.n_kv, unit, g);
  if (unit * NB >= s.n_blocks) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n32 = lane & 31, h = lane >> 5;
  const int wr = w % WPB, grp = w / WPB;
  const int ks_id = KS > 1 ? grp : 0, nb = KS > 1 ? 0 : grp;
  int blk[NB], nctx = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    blk[b] = a.order[min(unit * NB + b, s.n_blocks - 1)];
    nctx = max(nctx, (min(max(a.anchors[blk[b]], 0), s.T) + 31) / 32);
  }
  const bool active = grp < (KS > 1 ? KS : NB) && unit * NB + nb < s.n_blocks && 32 * wr < s.R;
  const int i = a.order[min(unit * NB + (active ? nb : 0), s.n_blocks - 1)];
  const int anchor = active ? min(max(a.anchors[i], 0), s.T) : 0;
  // steps of the work-group, and of this wave
  const int nstep = (nctx + KS - 1) / KS, mine = max(0, ((anchor + 31) / 32 - ks_id + KS - 1) / KS);
  const float sl2 = a.scale * 1.4426950408889634f;
  const u32x4 z4 = {0u, 0u, 0u, 0u};
  // A step's K and V tiles into registers (past the last tile the last again, rows past T repeat the
  // last one: masked), and from there into a buffer.  A wave-load is 16 rows x 4 pieces: 64-byte
  // segments from memory, and to LDS every 16 lanes write 256 different bytes modulo the bank cycle (the
  // conflict counter still shows about 8 cycles per store; the reads, which k_aatt_kvc has too, show none).
  const int lr = lane >> 2, lc = lane & 3;
  u32x4 nk[PW], nv[PW];
  auto fetch = [&](int step) {
#pragma unroll
    for (int t = 0; t < PW; ++t) {
      const int ins = w + 4 * t;
      const int row = min(step * KS + ins / NK, nctx - 1) * 32 + 16 * (ins & 1) + lr;
      const long at = ((long)min(row, s.T - 1) * s.n_kv + g) * HD + (ins % NK >> 1) * 32 + lc * 8;
      nk[t] = ld16(a.kc + at);
      nv[t] = ld16(a.vc + at);
    }
  };
  auto slot_of = [&](int ins) { return ins / NK * TB + piece_at(16 * (ins & 1) + lr, (ins % NK >> 1) * 4 + lc); };
  auto store = [&](int bi) {
#pragma unroll
    for (int t = 0; t < PW; ++t) {
      char* dst = lds + bi * SB + slot_of(w + 4 * t);
      *reinterpret_cast<u32x4*>(dst) = nk[t];
      *reinterpret_cast<u32x4*>(dst + KS * TB) = nv[t];
    }
  };
#pragma unroll
  for (int t = 0; t < NOWN * NK / 4; ++t) {
    const int ins = w + 4 * t;
    constexpr int kLast = NB - 1;
    const int b0 = blk[min(2 * (4 * t / NK), kLast)], b1 = blk[min(2 * (4 * t / NK) + 1, kLast)];
    const int row = (ins & 1 ? b1 : b0) * s.B + min(lr, s.B - 1);
    const long at = ((long)row * s.n_kv + g) * HD + (ins % NK >> 1) * 32 + lc * 8;
    *reinterpret_cast<u32x4*>(own + slot_of(ins)) = ld16(a.kb + at);
    *reinterpret_cast<u32x4*>(own + NOWN * TB + slot_of(ins)) = ld16(a.vb + at);
  }
  if (nctx > 0) {
    fetch(0);
    store(0);
    fetch(1);
  }
  int fo[2], off[2];
  frag_offsets(lane, fo);
  tr_offsets(lane, off);

  // this wave's rows: Q (and dO) operands, softmax state or row statistics, accumulators
  const int r = 32 * wr + n32;
  const bool rv = active && r < s.R;
  const long rh = rv ? (long)(i * s.B + r % s.B) * s.n_q + g * s.G + r / s.B : 0;
  u32x4 qf[NK], df[DQ ? NK : 1];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    if constexpr (DQ) {
      const long at = ((long)(g * s.n_blocks + i) * (s.Rp / 32) + (active ? wr : 0)) * TB + k * 1024 + fo[k & 1];
      qf[k] = ld16b(reinterpret_cast<const char*>(a.qf) + at);
      df[k] = ld16b(reinterpret_cast<const char*>(a.df) + at);
    } else {
      qf[k] = rv ? ld16(a.q + rh * HD + k * 16 + 8 * h) : z4;
    }
  }
  float m = -1e30f, l = 0.f;  // m finite: 2^(-inf - m) = 0 for masked keys before any visible one
  float lse2 = 0.f, nd = 0.f;
  if constexpr (DQ) {
    lse2 = rv ? a.lse[rh] * 1.4426950408889634f : 0.f;
    nd = rv ? a.st[(((long)g * s.n_blocks + i) * 2 + 1) * s.Rp + r] : 0.f;
  }
  f32x16 o[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) o[dt] = splat16(0.f);
  // a tile's scores: raw ones of this lane's row against keys 8 (e / 4) + 4 h + e mod 4 (the log2-domain
  // scale sl2 > 0 goes into each exponent as one fma), and dP for dQ
  f32x16 sc, dp;
  auto scores = [&](const char* kt, const char* vt) {
    sc = splat16(0.f);
    dp = splat16(nd);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      sc = mfma32(ld16b(kt + k * 1024 + fo[k & 1]), qf[k], sc);
      if constexpr (DQ) dp = mfma32(ld16b(vt + k * 1024 + fo[k & 1]), df[k], dp);
    }
  };
  // only the tile's keys k0 .. k1 - 1 are visible
  auto mask = [&](int k0, int k1) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int key = 8 * (e >> 2) + 4 * h + (e & 3);
      if (key < k0 || key >= k1) sc[e] = -INFINITY;
    }
  };
  // scores -> P (forward; O and l follow the running maximum) or dS
  f32x16 p;
  auto weigh = [&]() {
    if constexpr (!DQ) {
      // the running maximum moves only when the tile's maximum exceeds it by more than 8 (so
      // unnormalised probabilities stay below 2^8); the rescale of O and l then runs for the
      // whole wave, with factor 1 on rows that did not move
      float tm = sc[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) tm = fmaxf(tm, sc[e]);
      tm = fmaxf(tm, __shfl_xor(tm, 32));
      tm *= sl2;  // max of the log2-domain scores (scaling by sl2 > 0 keeps the maximum)
      const bool grow = tm > m + 8.f;
      if (__builtin_amdgcn_ballot_w64(grow) != 0) {
        const float mn = grow ? tm : m;
        const float corr = ex2(m - mn);
        l *= corr;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) o[dt] *= corr;
        m = mn;
      }
      float ps = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        p[e] = ex2(fmaf(sc[e], sl2, -m));
        ps += p[e];
      }
      l += ps;
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) p[e] = ex2(fmaf(sc[e], sl2, -lse2)) * dp[e];
    }
  };
  // O^T += V^T P^T (forward) or dQ^T += K^T dS^T, over keys 16 ks .. 16 ks + 15 of the tile
  auto gather = [&](const char* lt, int ks) {
    const u32x4 pb = pack_half(p, ks);
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) o[dt] = mfma32(ld_tr_op(lt, off, ks, dt), pb, o[dt]);
  };
  // one step; the buffer index is a compile-time constant (steps run in pairs)
  auto step = [&](int st, auto BI) {
    constexpr int bi = decltype(BI)::value;
    lds_barrier();
    store(bi ^ 1);  // step st + 1's tiles
    fetch(st + 2);
    if (st >= mine) return;  // the work-group's other waves have longer contexts
    const char* kt = lds + bi * SB + ks_id * TB;
    const char* vt = kt + KS * TB;
    scores(kt, vt);
    const int keys = anchor - (st * KS + ks_id) * 32;
    if (keys < 32) mask(0, keys);
    weigh();
    gather(DQ ? kt : vt, 0);
    gather(DQ ? kt : vt, 1);
  };
  for (int st = 0; st < nstep; st += 2) {
    step(st, std::integral_constant<int, 0>{});
    if (st + 1 < nstep) step(st + 1, std::integral_constant<int, 1>{});
  }
  if (nstep == 0) lds_barrier();
  if (active && ks_id == 0) {  // (the other block's half of the tile takes no part, whatever it holds)
    const char* kt = own + nb / 2 * TB;
    const char* vt = kt + NOWN * TB;
    const int half = nb & 1;
    scores(kt, vt);
    mask(16 * half, 16 * half + s.B);
    weigh();
    if (half == 0) gather(DQ ? kt : vt, 0);
    else gather(DQ ? kt : vt, 1);
  }
  if constexpr (KS > 1) {
    // merge the wave groups in order: 4-dim pieces of O [group - 1][WPB][piece][lane], (m, l)
    constexpr int NP = ND * 4;
    f32x4* mo = reinterpret_cast<f32x4*>(lds);
    float2* ml = reinterpret_cast<float2*>(lds + SB);
    static_assert((KS - 1) * WPB * NP * 1024 <= SB, "merge area");
    __syncthreads();
    if (grp > 0) {
#pragma unroll
      for (int x = 0; x < NP; ++x)
        mo[(((grp - 1) * WPB + wr) * NP + x) * 64 + lane] =
            f32x4{o[x / 4][4 * (x % 4)], o[x / 4][4 * (x % 4) + 1], o[x / 4][4 * (x % 4) + 2], o[x / 4][4 * (x % 4) + 3]};
      ml[((grp - 1) * WPB + wr) * 64 + lane] = make_float2(m, l);
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int y = 0; y < KS - 1; ++y) {
      float ca = 1.f, cb = 1.f;
      if constexpr (!DQ) {
        const float2 v = ml[(y * WPB + wr) * 64 + lane];
        const float mn = fmaxf(m, v.x);
        ca = ex2(m - mn);
        cb = ex2(v.x - mn);
        l = l * ca + v.y * cb;
        m = mn;
      }
#pragma unroll
      for (int x = 0; x < NP; ++x) {
        const f32x4 v = mo[((y * WPB + wr) * NP + x) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = o[x / 4][4 * (x % 4) + e];
          o[x / 4][4 * (x % 4) + e] = DQ ? t + v[e] : t * ca + v[e] * cb;
        }
      }
    }
  }
  float out_scale = a.scale;
  if constexpr (!DQ) {
    l += __shfl_xor(l, 32);
    out_scale = 1.f / l;
    if (rv && h == 0) a.lse[rh] = (m + log2f(l)) * 0.6931471805599453f;
  }
  if (!rv) return;
  float* dst = (DQ ? a.dq : a.out) + rh * HD + 4 * h;
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int x = 0; x < 4; ++x)
      *reinterpret_cast<f32x4*>(dst + 32 * dt + 8 * x) =
          f32x4{o[dt][4 * x], o[dt][4 * x + 1], o[dt][4 * x + 2], o[dt][4 * x + 3]} * out_scale;
}

// ---- context dK, dV: work-group (128-key tile kt, KV head g, chunk z); wave w owns keys 128 kt + 32 w
// + (0..31): their K and V rows are its B operands, dK^T and dV^T its accumulators, all in
// registers.  The waves walk the (block, 32-row tile) units of the chunk's blocks that see a key of
// the tile (the first nvis in the work order): per unit a wave forms S = Q K^T and dP = dO V^T (the
// row statistics are their initial values) and adds dO^T P and Q^T dS.  The units' tiles and
// statistics go through three LDS buffers, one barrier per unit.  The scores of one unit are formed
// between the gradient products of the unit before, so that the exponentials have products beside
// them; one wave per SIMD, with 512 registers.
// Writes this chunk's partial dK, dV.  512 blocks, T = 3,072: 658 -> 500 us against 16-key waves with
// transposed copies of Q and dO; with two waves per SIMD and 256 registers 650.  Work-groups start
// with the first key tiles, which the most blocks see, so that the short ones fill the end (300 blocks of
// 8 x 16 rows, T = 3,072, 8 KV heads x 64: 330 -> 284 us against chunk by chunk).
constexpr int kKvcKeys = 128;
template <int HD>
__global__ __launch_bounds__(kTrT, 1) void k_aatt_kvc(AttnT a) {
  constexpr int NK = HD / 16, ND = HD / 32;
  constexpr int TB = kTileBytes<HD>, PW = NK / 4;
  constexpr int SB = 2 * TB + 256;  // a buffer: Q tile, dO tile, the rows' 2 x 32 statistics
  __shared__ __attribute__((aligned(1024))) char lds[3 * SB];
  const AttnShapeT& s = a.s;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n32 = lane & 31, h = lane >> 5;
  const int n = blockIdx.x, g = n % s.n_kv, z = n / s.n_kv % a.nch, kt = n / (s.n_kv * a.nch);

  const float sl2 = a.scale * 1.4426950408889634f;
  const int NPr = s.Rp / 32;
  const int key0 = kt * kKvcKeys;
  // the chunk's blocks, one per lane, by decreasing anchor: those that see a key come first
  const int pos = z + a.nch * lane;
  const int myblk = pos < s.n_blocks && lane < kChunkBlocks ? a.order[pos] : 0;
  const int myanc = pos < s.n_blocks && lane < kChunkBlocks ? min(max(a.anchors[myblk], 0), s.T) : 0;
  const int nvis = __builtin_popcountll(__builtin_amdgcn_ballot_w64(myanc > key0));
  const int units = nvis * NPr;

  // (a key that no block of the chunk sees takes part as zeros: its row may hold anything, NaN too)
  const int myk = key0 + 32 * w + n32;
  const bool seen = myk < __builtin_amdgcn_readfirstlane(myanc);
  u32x4 kf[NK], vf[NK];
  {
    const u32x4 z4 = {0u, 0u, 0u, 0u};
    const long row = ((long)min(myk, s.T - 1) * s.n_kv + g) * HD;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      kf[k] = seen ? ld16(a.kc + row + k * 16 + 8 * h) : z4;
      vf[k] = seen ? ld16(a.vc + row + k * 16 + 8 * h) : z4;
    }
  }
  f32x16 dk[ND], dv[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) dk[dt] = dv[dt] = splat16(0.f);
  int fo[2], off[2];
  frag_offsets(lane, fo);
  tr_offsets(lane, off);
  // the walk over the units; past the last unit the last again
  struct Walk {
    int j = 0, p = 0;
  };
  auto next = [&](Walk& u) {
    if (u.p + 1 < NPr) ++u.p;
    else if (u.j + 1 < nvis) {
      u.p = 0;
      ++u.j;
    }
  };
  auto tile_of = [&](const Walk& u) { return ((long)g * s.n_blocks + __builtin_amdgcn_readlane(myblk, u.j)) * NPr + u.p; };
  Walk wl, wc;  // the unit to load, the unit whose scores come next
  // a unit's tiles and statistics into registers, and from there into a buffer
  u32x4 nq[PW], nd[PW];
  float ns = 0.f;
  auto fetch = [&]() {
    const long at = tile_of(wl);
    const char* bq = reinterpret_cast<const char*>(a.qf) + at * TB + lane * 16;
    const char* bd = reinterpret_cast<const char*>(a.df) + at * TB + lane * 16;
#pragma unroll
    for (int t = 0; t < PW; ++t) {
      nq[t] = ld16b(bq + (w + 4 * t) * 1024);
      nd[t] = ld16b(bd + (w + 4 * t) * 1024);
    }
    if (w == 0) ns = a.st[(at - wl.p) * 64 + h * s.Rp + 32 * wl.p + n32];
    next(wl);
  };
  auto store = [&](int bi) {
#pragma unroll
    for (int t = 0; t < PW; ++t) {
      char* dst = lds + bi * SB + (w + 4 * t) * 1024 + lane * 16;
      *reinterpret_cast<u32x4*>(dst) = nq[t];
      *reinterpret_cast<u32x4*>(dst + TB) = nd[t];
    }
    if (w == 0) *reinterpret_cast<float*>(lds + bi * SB + 2 * TB + lane * 4) = ns;
  };
  // S = Q K^T (kind 0) or dP = dO V^T (kind 1) of the unit, on top of the rows' statistics
  auto scores = [&](int bi, int kind, const u32x4* bf) {
    const char* b = lds + bi * SB;
    const f32x4* st = reinterpret_cast<const f32x4*>(b + 2 * TB + kind * 128);
    f32x16 c;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const f32x4 v = st[2 * x + h];
#pragma unroll
      for (int e = 0; e < 4; ++e) c[4 * x + e] = v[e];
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) c = mfma32(ld16b(b + kind * TB + k * 1024 + fo[k & 1]), bf[k], c);
    return c;
  };
  u32x4 pb[2], sb[2];  // P and dS of the current unit as operands
  // one unit: P and dS of the next one (buffer b1), beside the current one's gradient products (b0)
  auto unit = [&](auto B0, auto FIRST) {
    constexpr int b0 = decltype(B0)::value, b1 = (b0 + 1) % 3, b2 = (b0 + 2) % 3;
    lds_barrier();
    store(b2);
    fetch();
    const int anchor = __builtin_amdgcn_readlane(myanc, wc.j);
    next(wc);
    const float bias = myk < anchor ? 0.f : -INFINITY;
    const char* tq = lds + b0 * SB;
    const char* td = tq + TB;
    f32x16 sc = scores(b1, 0, kf);
    f32x16 dp = scores(b1, 1, vf);
    if constexpr (!decltype(FIRST)::value) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
          dv[dt] = mfma32(ld_tr_op(td, off, ks, dt), pb[ks], dv[dt]);
          dk[dt] = mfma32(ld_tr_op(tq, off, ks, dt), sb[ks], dk[dt]);
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = ex2(fmaf(sc[e], sl2, bias));
#pragma unroll
    for (int e = 0; e < 16; ++e) dp[e] *= sc[e];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      pb[ks] = pack_half(sc, ks);
      sb[ks] = pack_half(dp, ks);
    }
  };
  if (units > 0) {
    fetch();
    store(0);
    fetch();
    unit(std::integral_constant<int, 2>{}, std::true_type{});  // stores unit 1, scores of unit 0
    for (int u = 0; u < units; u += 3) {
      unit(std::integral_constant<int, 0>{}, std::false_type{});
      if (u + 1 < units) unit(std::integral_constant<int, 1>{}, std::false_type{});
      if (u + 2 < units) unit(std::integral_constant<int, 2>{}, std::false_type{});
    }
  }
  if (myk < s.T) {
    float* pk = a.part + (((long)z * s.T + myk) * s.n_kv + g) * HD + 4 * h;
    float* pv = a.part + ((((long)a.nch + z) * s.T + myk) * s.n_kv + g) * HD + 4 * h;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const f32x4 k4 = {dk[dt][4 * x], dk[dt][4 * x + 1], dk[dt][4 * x + 2], dk[dt][4 * x + 3]};
        const f32x4 v4 = {dv[dt][4 * x], dv[dt][4 * x + 1], dv[dt][4 * x + 2], dv[dt][4 * x + 3]};
        *reinterpret_cast<f32x4*>(pk + 32 * dt + 8 * x) = k4 * a.scale;
        *reinterpret_cast<f32x4*>(pv + 32 * dt + 8 * x) = v4;
      }
  }
}

// context dK, dV = the chunks' partials added in chunk order, U of each loaded at a time
template <int U>
__global__ void k_aatt_sum(const float* part, int nch, long n, float* dk, float* dv) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    float sk = 0.f, sv = 0.f;
    for (int c0 = 0; c0 < nch; c0 += U) {
      float xk[U], xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // (past the last chunk the last again)
        const long c = min(c0 + u, nch - 1);
        xk[u] = part[c * n + e];
        xv[u] = part[(nch + c) * n + e];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u < nch) {
          sk += xk[u];
          sv += xv[u];
        }
    }
    dk[e] = sk;
    dv[e] = sv;
  }
}

// ---- weighted CE (Eq. 5).  The row weights and 1 / sum w depend on labels and block positions
// only and come first; then each row's log-sum-exp, CE and gradient, a work-group per row: held in
// registers as a whole or in part (k_wce_reg), held on chip (k_wce_chip), or cut into pieces for
// several work-groups (k_wce_piece); last, the loss in row order. ----
constexpr int kCeT = 1024;       // threads of the row work-group
constexpr int kCeRows = 256;     // rows in flight (work-groups)
constexpr int kCeLaunch = 1 << 21;  // most rows of one launch of a work-group per row (it takes less than 2^32 threads)
constexpr int kCePieces = 512;   // work-groups of a last turn of rows cut into pieces
constexpr int kCeTailMax = 64;   // rows of such a turn: from there both ways cost the same (151,936 values, 90 us)

// w[r] = exp(-(b - 1) / gamma) for block position b = r mod B > 0 with a label in range, else 0;
// 1 / sum w in fp64, summed in the loss kernel's order
__global__ __launch_bounds__(256) void k_wce_weights(const int32_t* labels, int rows, int V, int B, float gamma,
                                                     float* w, float* inv_wsum) {
  __shared__ double sw[256];
  double a = 0.0;
  for (int r = threadIdx.x; r < rows; r += 256) {
    const int b = r % B, y = labels[r];
    const float wr = (b > 0 && y >= 0 && y < V) ? expf(-(float)(b - 1) / gamma) : 0.f;
    w[r] = wr;
    a += wr;
  }
  sw[threadIdx.x] = a;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sw[threadIdx.x] += sw[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) inv_wsum[0] = sw[0] > 0.0 ? (float)(1.0 / sw[0]) : 0.f;
}

// max or sum over a work-group of T threads, the same value in every thread (fixed order)
template <int T, bool MAX>
__device__ __forceinline__ float ce_reduce(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(v, off);
    v = MAX ? fmaxf(v, o) : v + o;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = red[0];
#pragma unroll
  for (int k = 1; k < T / 64; ++k) v = MAX ? fmaxf(v, red[k]) : v + red[k];
  return v;
}

// per row: lse (log2 domain: max of z log2 e, sum of 2^(z log2 e - max)), ce = lse - z[label] for
// rows that take part, and dz = (w / sum w) (softmax(z) - onehot(label)).  One work-group per row, which
// holds S 16-byte pieces per thread in registers, all their loads in flight together, so that
// rows of up to 4 S T values are read once; of longer rows (REST) the values past those are read again
// for the gradient.  The pieces start at the row's first aligned value; the up to 6 values before and
// after them go to the first threads.  Rows without a loss get zeros and are not read.
// Bound by memory and, with few rows, by the latency of one row.  Against two sweeps per row by
// 1,024 threads, with single-value accesses where 4 does not divide V (whole call): 207 rows x 32,003
// 31 -> 19 us, 4,800 x 4,000 74 -> 37, 1,600 x 98,000 317 -> 246, 528 x 100,001 284 -> 96, 1,040 x 201,088
// (with the last turn in pieces, below) 441 -> 357.
template <int T, int S, bool REST>
__global__ __launch_bounds__(T) void k_wce_reg(const float* logits, const int32_t* labels, int row0, int V, int B,
                                               const float* w, const float* inv_wsum, float* ce_out, float* dz) {
  __shared__ float red[T / 64];
  const int row = row0 + blockIdx.x, tid = threadIdx.x;
  const float L2E = 1.4426950408889634f;
  const float* z = logits + (long)row * V;
  float* d = dz + (long)row * V;
  const int y = labels[row];
  const bool on = row % B > 0 && y >= 0 && y < V;
  const int head = min(V, (int)((0u - (unsigned)(reinterpret_cast<uintptr_t>(z) >> 2)) & 3u));
  const int n4 = (V - head) / 4, tail = V - head - 4 * n4;
  const int edge = tid < head ? tid : tid < head + tail ? V - tail + tid - head : -1;
  const f32x4* z4 = reinterpret_cast<const f32x4*>(z + head);
  const f32x4 none = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  f32x4 r[S];
  float e1 = -INFINITY;
  float lse2 = 0.f;
  auto max4 = [](f32x4 x) { return fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])); };
  auto exp4 = [&](f32x4 x, float m) {
    return (ex2(fmaf(x[0], L2E, -m)) + ex2(fmaf(x[1], L2E, -m))) + (ex2(fmaf(x[2], L2E, -m)) + ex2(fmaf(x[3], L2E, -m)));
  };
  if (on) {
    if (n4 > 0) {
#pragma unroll
      for (int k = 0; k < S; ++k) r[k] = z4[min(k * T + tid, n4 - 1)];
    }
    if (edge >= 0) e1 = z[edge];
    float m = e1;
#pragma unroll
    for (int k = 0; k < S; ++k) {
      if (k * T + tid >= n4) r[k] = none;
      m = fmaxf(m, max4(r[k]));
    }
    float rest = 0.f;
    if constexpr (REST) {  // running (max, sum) of the values past the registers, four pieces at a time
      for (int v = S * T + tid; v < n4; v += 4 * T) {
        f32x4 x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = z4[min(v + k * T, n4 - 1)];
#pragma unroll
        for (int k = 1; k < 4; ++k)
          if (v + k * T >= n4) x[k] = none;
        const float mx = fmaxf(fmaxf(max4(x[0]), max4(x[1])), fmaxf(max4(x[2]), max4(x[3])));
        if (mx > m) {
          rest *= ex2((m - mx) * L2E);
          m = mx;
        }
        const float ml = fmaxf(m * L2E, -FLT_MAX);  // (finite while all values so far are masked: they add 0)
        rest += (exp4(x[0], ml) + exp4(x[1], ml)) + (exp4(x[2], ml) + exp4(x[3], ml));
      }
    }
    const float M = ce_reduce<T, true>(m, red) * L2E;
    float sum = ex2(fmaf(e1, L2E, -M));
#pragma unroll
    for (int k = 0; k < S; ++k) sum += exp4(r[k], M);
    if (REST && S * T + tid < n4) sum += rest * ex2(fmaf(m, L2E, -M));
    lse2 = M + log2f(ce_reduce<T, false>(sum, red));
  }
  if (tid == 0) ce_out[row] = on ? lse2 * 0.6931471805599453f - z[y] : 0.f;
  const float c = on ? w[row] * inv_wsum[0] : 0.f;
  const int yv = c != 0.f ? y - head : -1;  // the label's place after the first aligned value
  const bool wide = (reinterpret_cast<uintptr_t>(d + head) & 15) == 0;  // (the gradient may be aligned otherwise)
  auto grad = [&](f32x4 x, int v) {
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    if (c != 0.f) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = c * ex2(fmaf(x[e], L2E, -lse2));
        if (4 * v + e == yv) o[e] -= c;
      }
    }
    if (wide) __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(d + head) + v);
    else
#pragma unroll
      for (int e = 0; e < 4; ++e) d[head + 4 * v + e] = o[e];
  };
  if constexpr (REST) {  // first: its values were read last
#pragma unroll 4
    for (int v = S * T + tid; v < n4; v += T) grad(c != 0.f ? z4[v] : none, v);
  }
#pragma unroll
  for (int k = 0; k < S; ++k)
    if (k * T + tid < n4) grad(r[k], k * T + tid);
  if (edge >= 0) d[edge] = c == 0.f ? 0.f : c * ex2(fmaf(e1, L2E, -lse2)) - (edge == y ? c : 0.f);
}

// The same per row with the whole row held on chip: one work-group per CU (its LDS share is
// the CU's), kCeOR 16-byte pieces per thread in registers and kCeOL in LDS, so that the row is
// read from memory once; the max, sum and gradient sweeps run over the held values.  Piece v of
// the row: registers slot k of thread t for v = k kCeOT + t, else LDS slot v - kCeOR kCeOT.  For
// rows of kCeOMin .. kCeOCap values (a multiple of 4), so that every register slot is inside the
// row (no per-slot bounds masks to keep).
constexpr int kCeOT = 256;
constexpr int kCeOR = 109;
constexpr int kCeOL = 10224;
constexpr long kCeOCap = ((long)kCeOR * kCeOT + kCeOL) * 4;  // values of a row held on chip
constexpr long kCeOMin = (long)kCeOR * kCeOT * 4;

__global__ __launch_bounds__(kCeOT) void k_wce_chip(const float* logits, const int32_t* labels, int rows, int V,
                                                   int B, const float* w, const float* inv_wsum, float* ce_out,
                                                   float* dz) {
  __shared__ f32x4 lrow[kCeOL];
  __shared__ float red[kCeOT / 64], redm[kCeOT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float L2E = 1.4426950408889634f;
  const int V4 = V / 4;
  const float inv = inv_wsum[0];
  for (int row = blockIdx.x; row < rows; row += gridDim.x) {
    const f32x4* z4 = reinterpret_cast<const f32x4*>(logits + (long)row * V);
    f32x4 r[kCeOR];
#pragma unroll
    for (int k = 0; k < kCeOR; ++k) r[k] = z4[k * kCeOT + tid];
    // the rest of the row into LDS (pieces past the row re-read piece 0 and are skipped below)
    for (int m0 = wv * 64; m0 < kCeOL; m0 += kCeOT) {
      const int v = kCeOR * kCeOT + m0 + lane;
      const f32x4* src = z4 + (v < V4 ? v : 0);
      __builtin_amdgcn_global_load_lds(src, (LDSP char*)(char*)&lrow[m0], 16, 0, 0);
    }
    const int nl = min(kCeOL, max(0, V4 - kCeOR * kCeOT));  // LDS pieces of this row
    // running (max, sum) of the log2-domain values, one 16-byte piece at a time (the register
    // pieces in load order, so the sweep follows their arrival), then the LDS pieces; the maximum starts
    // at the lowest finite value, so that masked values (-inf, or scaled to it) add 0
    float m = -FLT_MAX, sum = 0.f;
    auto take4 = [&](f32x4 x) {
      const float t0 = x[0] * L2E, t1 = x[1] * L2E, t2 = x[2] * L2E, t3 = x[3] * L2E;
      const float m4 = fmaxf(fmaxf(t0, t1), fmaxf(t2, t3));
      if (m4 > m) {
        sum *= ex2(m - m4);
        m = m4;
      }
      sum += (ex2(t0 - m) + ex2(t1 - m)) + (ex2(t2 - m) + ex2(t3 - m));
    };
#pragma unroll
    for (int k = 0; k < kCeOR; ++k) take4(r[k]);
    wait_vm();
    __syncthreads();
    for (int j = tid; j < nl; j += kCeOT) take4(lrow[j]);
    // combine the threads' (max, sum) pairs
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const float om = __shfl_xor(m, off), os = __shfl_xor(sum, off);
      const float nm = fmaxf(m, om);
      sum = sum * ex2(m - nm) + os * ex2(om - nm);
      m = nm;
    }
    if (lane == 0) {
      redm[wv] = m;
      red[wv] = sum;
    }
    __syncthreads();
    float M = redm[0], S = red[0];
#pragma unroll
    for (int k = 1; k < kCeOT / 64; ++k) {
      const float nm = fmaxf(M, redm[k]);
      S = S * ex2(M - nm) + red[k] * ex2(redm[k] - nm);
      M = nm;
    }
    __syncthreads();  // red, redm are rewritten by the next row
    const float lse2 = M + log2f(S);
    const int y = labels[row];
    const bool on = row % B > 0 && y >= 0 && y < V;
    if (tid == 0) ce_out[row] = on ? lse2 * 0.6931471805599453f - logits[(long)row * V + y] : 0.f;
    const float c = w[row] * inv;
    // (rows of weight 0: c 2^(x - inf) = 0 for every value, so no branch per piece)
    const float sub = c == 0.f ? INFINITY : lse2;
    f32x4* d4 = reinterpret_cast<f32x4*>(dz + (long)row * V);
    auto grad = [&](f32x4 x, int v) {
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = c * ex2(fmaf(x[e], L2E, -sub));
      __builtin_nontemporal_store(o, d4 + v);
    };
#pragma unroll
    for (int k = 0; k < kCeOR; ++k) grad(r[k], k * kCeOT + tid);
    for (int j = tid; j < nl; j += kCeOT) grad(lrow[j], kCeOR * kCeOT + j);
    // the label's value, c p - c, rewritten by the thread that stored its piece (a thread's
    // stores to one address land in program order)
    if (on) {
      const int y4 = y >> 2, rest = y4 - kCeOR * kCeOT;
      if ((rest < 0 ? y4 % kCeOT : rest % kCeOT) == tid) {
        const float zy = logits[(long)row * V + y];
        dz[(long)row * V + y] = c * ex2(fmaf(zy, L2E, -sub)) - c;
      }
    }
    __syncthreads();  // lrow is refilled by the next row
  }
}

// The rows of a last, nearly empty turn of the kernel above, each cut into `pieces` for as many
// work-groups: pass 0 leaves each piece's (max, sum of 2^(z log2 e - max)) in part, pass 1 forms the row's
// from them in piece order and writes the gradient.  A piece of masked values alone (-inf, or so low
// that the scaling overflows) leaves the sum 0 at the lowest finite maximum.  Rows without a loss get
// zeros and are not read.
template <int PASS>
__global__ __launch_bounds__(kCeT) void k_wce_piece(const float* logits, const int32_t* labels, int row0, int pieces,
                                                    int V, int B, const float* w, const float* inv_wsum, float* part,
                                                    float* ce_out, float* dz) {
  __shared__ float red[kCeT / 64];
  const int row = row0 + blockIdx.x / pieces, pc = blockIdx.x % pieces, tid = threadIdx.x;
  const float L2E = 1.4426950408889634f;
  const int V4 = V / 4, v0 = (int)((long)V4 * pc / pieces), v1 = (int)((long)V4 * (pc + 1) / pieces);
  const f32x4* z4 = reinterpret_cast<const f32x4*>(logits + (long)row * V);
  if constexpr (PASS == 0) {
    float m = -INFINITY;
#pragma unroll 4
    for (int v = v0 + tid; v < v1; v += kCeT) {
      const f32x4 x = z4[v];
      m = fmaxf(m, fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
    }
    const float M = fmaxf(ce_reduce<kCeT, true>(m, red) * L2E, -FLT_MAX);
    float sum = 0.f;
#pragma unroll 4
    for (int v = v0 + tid; v < v1; v += kCeT) {
      const f32x4 x = z4[v];
      sum += (ex2(fmaf(x[0], L2E, -M)) + ex2(fmaf(x[1], L2E, -M))) +
             (ex2(fmaf(x[2], L2E, -M)) + ex2(fmaf(x[3], L2E, -M)));
    }
    sum = ce_reduce<kCeT, false>(sum, red);
    if (tid == 0) {
      part[2 * blockIdx.x] = M;
      part[2 * blockIdx.x + 1] = sum;
    }
  } else {
    const float* pp = part + 2 * (blockIdx.x - pc);
    float M = pp[0], S = pp[1];
    for (int k = 1; k < pieces; ++k) {
      const float nm = fmaxf(M, pp[2 * k]);
      S = S * ex2(M - nm) + pp[2 * k + 1] * ex2(pp[2 * k] - nm);
      M = nm;
    }
    const float lse2 = M + log2f(S);
    const int y = labels[row];
    const bool on = row % B > 0 && y >= 0 && y < V;
    if (tid == 0 && pc == 0) ce_out[row] = on ? lse2 * 0.6931471805599453f - logits[(long)row * V + y] : 0.f;
    const float c = w[row] * inv_wsum[0];
    f32x4* d4 = reinterpret_cast<f32x4*>(dz + (long)row * V);
#pragma unroll 4
    for (int v = v0 + tid; v < v1; v += kCeT) {
      f32x4 o = zero4();
      if (c != 0.f) {
        const f32x4 x = z4[v];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = c * ex2(fmaf(x[e], L2E, -lse2));
        if (on && v == y >> 2) o[y & 3] -= c;
      }
      __builtin_nontemporal_store(o, d4 + v);
    }
  }
}

// loss = sum w ce / sum w over the rows, in row order (one work-group)
__global__ __launch_bounds__(256) void k_wce_loss(const float* w, const float* ce, int rows, float* loss) {
  __shared__ double sw[256], sl[256];
  double a = 0.0, c = 0.0;
  for (int r = threadIdx.x; r < rows; r += 256) {
    a += w[r];
    c += (double)w[r] * ce[r];
  }
  sw[threadIdx.x] = a;
  sl[threadIdx.x] = c;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) {
      sw[threadIdx.x] += sw[threadIdx.x + k];
      sl[threadIdx.x] += sl[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    loss[0] = sw[0] > 0.0 ? (float)(sl[0] / sw[0]) : 0.f;
  }
}

}  // namespace

// ---- entry points ----------------------------------------------------------------------

static AttnShapeT att_shape(int n_blocks, int B, int T, int n_q, int n_kv, int hd) {
  AttnShapeT s{};
  s.n_blocks = n_blocks;
  s.B = B;
  s.T = T;
  s.n_q = n_q;
  s.n_kv = n_kv;
  s.hd = hd;
  s.G = n_q / n_kv;
  s.R = s.G * B;
  s.Rp = (s.R + 31) / 32 * 32;
  return s;
}

static int att_check(int n_blocks, int B, int T, int n_q, int n_kv, int hd) {
  if (n_blocks < 1 || B < 1 || B > kMaxBlockKeys || T < 0 || n_q < 1 || n_kv < 1 || n_q % n_kv) return DFLARE_ERR_INVALID_ARG;
  if (hd != 64 && hd != 128) return DFLARE_ERR_UNSUPPORTED;
  if ((n_q / n_kv) * B > 128) return DFLARE_ERR_UNSUPPORTED;
  return DFLARE_OK;
}

struct WsLayout {
  size_t st, qf, df, part, order, total;
  int nch;
};

// Chunks of the context-key gradients: at most 64 blocks each (one per lane of a wave), and enough
// of them that the (key tile, KV head, chunk) work-groups fill 256 CUs twice (kKvcGroups), down to 4 blocks.
constexpr int kKvcGroups = 512;
static int kv_chunks_least(const AttnShapeT& s) { return (s.n_blocks + kChunkBlocks - 1) / kChunkBlocks; }
static int kv_chunks_most(const AttnShapeT& s) { return (s.n_blocks + 3) / 4; }
static int kv_chunks(const AttnShapeT& s) {
  const long per = (long)((s.T + kKvcKeys - 1) / kKvcKeys) * s.n_kv;
  const int fill = per > 0 ? (int)((kKvcGroups + per - 1) / per) : 1;
  return std::max(kv_chunks_least(s), std::min(fill, kv_chunks_most(s)));
}
// Rows of the chunks' partials that the workspace holds: at least kv_chunks(s) T n_kv (the chunks that fill the
// chip are fewer than kKvcGroups / per + 1), and growing with every size, so that a workspace made for a
// program's longest sequence and most blocks serves the smaller calls.
static size_t kv_part_rows(const AttnShapeT& s) {
  const size_t keys = (size_t)s.T * s.n_kv;
  return std::max(kv_chunks_least(s) * keys, std::min(kv_chunks_most(s) * keys, (size_t)kKvcGroups * kKvcKeys + keys));
}

static WsLayout ws_layout(const AttnShapeT& s) {
  WsLayout L{};
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t o = 0;
  const size_t padded = (size_t)s.n_kv * s.n_blocks * s.Rp;
  L.nch = kv_chunks(s);
  L.st = o; o = al(o + padded * 8);
  L.qf = o; o = al(o + padded * s.hd * 2);
  L.df = o; o = al(o + padded * s.hd * 2);
  L.part = o; o = al(o + 2 * kv_part_rows(s) * s.hd * 4);
  L.order = o; o = al(o + (size_t)s.n_blocks * 4);
  L.total = o;
  return L;
}

static AttnT att_args(const AttnShapeT& s, const void* q, const void* kc, const void* vc, const void* kb,
                      const void* vb, const int32_t* anchors, void* ws) {
  const WsLayout L = ws_layout(s);
  char* w = static_cast<char*>(ws);
  AttnT a{};
  a.s = s;
  a.q = (const uint16_t*)q;
  a.kc = (const uint16_t*)kc;
  a.vc = (const uint16_t*)vc;
  a.kb = (const uint16_t*)kb;
  a.vb = (const uint16_t*)vb;
  a.anchors = anchors;
  a.st = (float*)(w + L.st);
  a.qf = (uint16_t*)(w + L.qf);
  a.df = (uint16_t*)(w + L.df);
  a.part = (float*)(w + L.part);
  a.order = (int*)(w + L.order);
  a.nch = L.nch;
  a.scale = 1.0f / sqrtf((float)s.hd);
  return a;
}

static void launch_order(hipStream_t st, const AttnT& a) {
  hipLaunchKernelGGL(k_anchor_order, dim3((a.s.n_blocks + 15) / 16), dim3(256), 0, st, a.anchors, a.s.n_blocks, a.s.T,
                     a.order);
}

template <int HD, bool DQ, int WPB, int KS>
static void launch_rows_as(hipStream_t st, const AttnT& a) {
  constexpr int NB = KS > 1 ? 1 : 4 / WPB;
  const int units = ((a.s.n_blocks + NB - 1) / NB + 7) / 8 * 8;  // whole turns of the 8 XCDs
  hipLaunchKernelGGL((k_aatt_rows<HD, DQ, WPB, KS>), dim3(units * a.s.n_kv), dim3(kTrT), 0, st, a);
}

template <typename F>
static void by_hd(int hd, F&& f) {
  if (hd == 64) f(std::integral_constant<int, 64>{});
  else f(std::integral_constant<int, 128>{});
}

// The row kernel's form.  A wave takes 32 of a block's R rows, so a block is WPB = ceil(R / 32)
// waves; the work-group's other waves take further blocks where there are enough of them to
// occupy the chip (kRowsSplitMax), else the same block's other key tiles.
template <bool DQ>
static void launch_rows(hipStream_t st, const AttnT& a) {
  const AttnShapeT& s = a.s;
  const bool split = (long)s.n_blocks * s.n_kv <= kRowsSplitMax;
  by_hd(s.hd, [&](auto h) {
    constexpr int HD = decltype(h)::value;
    switch (s.Rp / 32) {
      case 1: return split ? launch_rows_as<HD, DQ, 1, 4>(st, a) : launch_rows_as<HD, DQ, 1, 1>(st, a);
      case 2: return split ? launch_rows_as<HD, DQ, 2, 2>(st, a) : launch_rows_as<HD, DQ, 2, 1>(st, a);
      case 3: return launch_rows_as<HD, DQ, 3, 1>(st, a);
      default: return launch_rows_as<HD, DQ, 4, 1>(st, a);
    }
  });
}

}  // namespace dflare

using namespace dflare;

extern "C" {

size_t dflare_anchor_attention_workspace(int32_t n_blocks, int32_t B, int32_t T, int32_t n_q, int32_t n_kv,
                                         int32_t hd) {
  if (att_check(n_blocks, B, T, n_q, n_kv, hd) != DFLARE_OK) return 0;
  return ws_layout(att_shape(n_blocks, B, T, n_q, n_kv, hd)).total;
}

int dflare_anchor_attention_fwd(const void* q, const void* k_ctx, const void* v_ctx, const void* k_blk,
                                const void* v_blk, const int32_t* anchors, int32_t n_blocks, int32_t B, int32_t T,
                                int32_t n_q, int32_t n_kv, int32_t hd, float* out, float* lse, void* workspace,
                                size_t workspace_bytes, void* stream) {
  const int rc = att_check(n_blocks, B, T, n_q, n_kv, hd);
  if (rc != DFLARE_OK) return rc;
  if (!q || !k_blk || !v_blk || !anchors || !out || !lse || !workspace || (T > 0 && (!k_ctx || !v_ctx)))
    return DFLARE_ERR_INVALID_ARG;
  const AttnShapeT s = att_shape(n_blocks, B, T, n_q, n_kv, hd);
  if (workspace_bytes < ws_layout(s).total) return DFLARE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  AttnT a = att_args(s, q, k_ctx, v_ctx, k_blk, v_blk, anchors, workspace);
  a.out = out;
  a.lse = lse;
  launch_order(st, a);
  launch_rows<false>(st, a);
  return hipGetLastError() == hipSuccess ? DFLARE_OK : DFLARE_ERR_HIP;
}

int dflare_anchor_attention_bwd(const void* q, const void* k_ctx, const void* v_ctx, const void* k_blk,
                                const void* v_blk, const int32_t* anchors, int32_t n_blocks, int32_t B, int32_t T,
                                int32_t n_q, int32_t n_kv, int32_t hd, const float* out, const float* lse,
                                const float* dout, float* dq, float* dk_ctx, float* dv_ctx, float* dk_blk,
                                float* dv_blk, void* workspace, size_t workspace_bytes, void* stream) {
  const int rc = att_check(n_blocks, B, T, n_q, n_kv, hd);
  if (rc != DFLARE_OK) return rc;
  if (!q || !k_blk || !v_blk || !anchors || !out || !lse || !dout || !dq || !dk_blk || !dv_blk || !workspace ||
      (T > 0 && (!k_ctx || !v_ctx || !dk_ctx || !dv_ctx)))
    return DFLARE_ERR_INVALID_ARG;
  const AttnShapeT s = att_shape(n_blocks, B, T, n_q, n_kv, hd);
  if (workspace_bytes < ws_layout(s).total) return DFLARE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  AttnT a = att_args(s, q, k_ctx, v_ctx, k_blk, v_blk, anchors, workspace);
  a.out = nullptr;
  a.lse = const_cast<float*>(lse);
  a.dout = dout;
  a.dq = dq;
  a.dkc = dk_ctx;
  a.dvc = dv_ctx;
  a.dkb = dk_blk;
  a.dvb = dv_blk;
  launch_order(st, a);
  by_hd(hd, [&](auto h) {
    constexpr int HD = decltype(h)::value;
    hipLaunchKernelGGL((k_bwd_prep<HD>), dim3((n_blocks + 7) / 8 * 8 * n_kv), dim3(kTrT), (size_t)(4 * HD + 8) * s.Rp, st, a, out);
  });
  launch_rows<true>(st, a);
  if (T > 0)
    by_hd(hd, [&](auto h) {
      constexpr int HD = decltype(h)::value;
      hipLaunchKernelGGL((k_aatt_kvc<HD>), dim3((T + kKvcKeys - 1) / kKvcKeys * n_kv * a.nch), dim3(kTrT), 0, st, a);
    });
  if (T > 0) {
    // few keys and many blocks: a thread's chain of chunks is what the sum takes (256 values, 250 chunks: 54 us with
    // one load at a time, 10 with eight); with more values the waves hide it and the repeats of the last chunk
    // cost (397,824 values, 11 chunks: 6.3 us against 7.6)
    const long n = (long)T * n_kv * hd;
    hipLaunchKernelGGL(n < 65536 ? k_aatt_sum<8> : k_aatt_sum<1>, dim3((int)std::min<long>((n + 255) / 256, 4096)),
                       dim3(256), 0, st, a.part, a.nch, n, dk_ctx, dv_ctx);
  }
  return hipGetLastError() == hipSuccess ? DFLARE_OK : DFLARE_ERR_HIP;
}

size_t dflare_weighted_ce_workspace(int32_t rows) { return ((size_t)3 * rows + 64 + 2 * kCePieces) * 4; }

}  // extern "C"

namespace {

// The launches of the weighted CE; w holds at least rows + 64 + 2 kCePieces floats (the row weights,
// 1 / sum w, from rows + 64 on the partial sums of pieces), every one written by an earlier launch
// of the call than reads it.
void launch_weighted_ce(hipStream_t st, const float* logits, const int32_t* labels, int32_t rows, int32_t V,
                        int32_t B, float gamma, float* loss, float* row_ce, float* dlogits, float* w) {
  const float *wr = w, *inv = w + rows;
  float* part = w + rows + 64;
  hipLaunchKernelGGL(k_wce_weights, dim3(1), dim3(256), 0, st, labels, rows, V, B, gamma, w, w + rows);
  auto reg = [&](auto kernel, int n, int threads) {
    for (int r0 = 0; r0 < n; r0 += std::min(n - r0, kCeLaunch))
      hipLaunchKernelGGL(kernel, dim3(std::min(n - r0, kCeLaunch)), dim3(threads), 0, st, logits, labels, r0, V, B, wr,
                         inv, row_ce, dlogits);
  };
  // rows that fit the registers of a work-group: the fewest registers that hold them, and the fewest threads,
  // so that several rows share a CU.  4,096 rows with the form taken / with the next: 1,000 values 20 / 25 us, 4,000
  // 32 / 34, 8,200 55 / 66, 16,400 96 / 103, 40,000 252 / 269, 58,000 376 / 391; at the upper end of a form the two are
  // within 4% either way (24,000 152 / 148), and up to 240 rows within 1 us, except 512 threads against 1,024 at
  // 49,000 values (16 rows 13.9 / 15.5).  From 65,536 to 81,920 values the form with a rest runs with an empty
  // rest: 4 pieces a thread fewer than the form for 98,304 loads (16 rows of 65,540: 16.1 against 17.2).
  const int n4 = V / 4;
  if (n4 <= 512) reg(k_wce_reg<256, 2, false>, rows, 256);
  else if (n4 <= 2048) reg(k_wce_reg<256, 8, false>, rows, 256);
  else if (n4 <= 4096) reg(k_wce_reg<256, 16, false>, rows, 256);
  else if (n4 <= 8192) reg(k_wce_reg<512, 16, false>, rows, 512);
  else if (n4 <= 12288) reg(k_wce_reg<512, 24, false>, rows, 512);
  else if (n4 <= 16384) reg(k_wce_reg<1024, 16, false>, rows, 1024);
  else if (n4 <= 20480) reg(k_wce_reg<1024, 20, true>, rows, 1024);
  else if (n4 <= 24576) reg(k_wce_reg<1024, 24, false>, rows, 1024);
  else {
    // longer ones turn by turn of a row per CU, a nearly empty last turn cut into pieces
    const int last = rows % kCeRows, tail = V % 4 == 0 && last <= kCeTailMax ? last : 0, full = rows - tail;
    const bool chip = V % 4 == 0 && (long)V >= kCeOMin && (long)V <= kCeOCap;
    if (full > 0 && chip)
      hipLaunchKernelGGL(k_wce_chip, dim3(std::min(full, kCeRows)), dim3(kCeOT), 0, st, logits, labels, full, V, B, wr,
                         inv, row_ce, dlogits);
    else if (full > 0)
      reg(k_wce_reg<1024, 20, true>, full, 1024);
    if (tail > 0) {
      const int pieces = kCePieces / tail;
      hipLaunchKernelGGL((k_wce_piece<0>), dim3(tail * pieces), dim3(kCeT), 0, st, logits, labels, full, pieces, V, B,
                         wr, inv, part, row_ce, dlogits);
      hipLaunchKernelGGL((k_wce_piece<1>), dim3(tail * pieces), dim3(kCeT), 0, st, logits, labels, full, pieces, V, B,
                         wr, inv, part, row_ce, dlogits);
    }
  }
  hipLaunchKernelGGL(k_wce_loss, dim3(1), dim3(256), 0, st, wr, row_ce, rows, loss);
}

bool ce_args_ok(const float* logits, const int32_t* labels, int32_t rows, int32_t V, int32_t B, float gamma,
                const float* loss, const float* row_ce, const float* dlogits) {
  return logits && labels && loss && row_ce && dlogits && rows >= 1 && V >= 1 && B >= 1 && rows % B == 0 &&
         gamma > 0.f && isfinite(gamma);
}

// Scratch of the allocation-free weighted CE: the row weights, 1 / sum w and the pieces' partial
// sums of one call.
// Each GPU the library runs on holds its own copy until the process ends.  In host code the
// array's name is not a device address: kernels get the address hipGetSymbolAddress returns
// for the current device, looked up once per device.
constexpr int kCeNoAllocMaxRows = DFLARE_WEIGHTED_CE_NOALLOC_MAX_ROWS;
__device__ __align__(256) float scratch[kCeNoAllocMaxRows + 64 + 2 * kCePieces];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch[kMaxDevices];

// address of this device's scratch array (the device of `st`, which must be current)
int scratch_address(hipStream_t st, float** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return DFLARE_ERR_HIP;
  if (st) {
    int sdev = -1;
    if (hipStreamGetDevice(st, &sdev) != hipSuccess) return DFLARE_ERR_HIP;
    if (sdev != dev) return DFLARE_ERR_INVALID_ARG;
  }
  if (dev < 0 || dev >= kMaxDevices) return DFLARE_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DFLARE_ERR_HIP;
    g_scratch[dev] = static_cast<float*>(p);
  }
  *out = g_scratch[dev];
  return DFLARE_OK;
}

}  // namespace

extern "C" {

int dflare_weighted_ce(const float* logits, const int32_t* labels, int32_t rows, int32_t V, int32_t B, float gamma,
                       float* loss, float* row_ce, float* dlogits, void* workspace, size_t workspace_bytes,
                       void* stream) {
  if (!ce_args_ok(logits, labels, rows, V, B, gamma, loss, row_ce, dlogits) || !workspace)
    return DFLARE_ERR_INVALID_ARG;
  if (workspace_bytes < dflare_weighted_ce_workspace(rows)) return DFLARE_ERR_INVALID_ARG;
  launch_weighted_ce((hipStream_t)stream, logits, labels, rows, V, B, gamma, loss, row_ce, dlogits,
                     static_cast<float*>(workspace));
  return hipGetLastError() == hipSuccess ? DFLARE_OK : DFLARE_ERR_HIP;
}

int dflare_weighted_ce_noalloc(const float* logits, const int32_t* labels, int32_t rows, int32_t V, int32_t B,
                               float gamma, float* loss, float* row_ce, float* dlogits, void* stream) {
  if (!ce_args_ok(logits, labels, rows, V, B, gamma, loss, row_ce, dlogits)) return DFLARE_ERR_INVALID_ARG;
  if (rows > kCeNoAllocMaxRows) return DFLARE_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  float* w = nullptr;
  const int rc = scratch_address(st, &w);
  if (rc != DFLARE_OK) return rc;
  launch_weighted_ce(st, logits, labels, rows, V, B, gamma, loss, row_ce, dlogits, w);
  return hipGetLastError() == hipSuccess ? DFLARE_OK : DFLARE_ERR_HIP;
}

}  // extern "C"
