// Encode / cache write (Sec. 3, Eq. 2): c = (x - mu) W_down for the M new
// tokens of every sequence, both axes, written into the paged latent cache.
//
// bf16: a dense contraction on MFMA.  Per (axis, head) the output is the
// r x (B*M) matrix C^T = W_down^T X^T - (W_down^T mu) 1^T, computed with
// v_mfma_f32_32x32x16_bf16 on 32-row x 32-token tiles:
//   A operand  = 32 rows of W_down^T (row-major [r][T*d], 8 contiguous k per lane),
//   B operand  = 32 tokens of x      (each token's T*d stack is contiguous),
//   accumulator column = one token, so the 32x32 fp32 tile maps straight onto
//   the feature-major cache page (one feature row of consecutive tokens).
// The mean's product W_down^T mu is formed apart (a second accumulator fed with mu
// as a broadcast B operand; in the GEMM on the vector unit from the staged
// weights) and subtracted, so (x - mu) W_down is formed in fp32 without
// re-rounding x - mu to bf16.
// The pass reads x once (HBM-bound at the paper's ranks: about (r_k + r_v)/2
// flop per byte).
//
// fp32: the same product on the fp32 matrix instructions, 32 x 32 tiles.

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lla_device.h"
#include "lla_internal.h"
#include "../../include/lla.h"

namespace lla {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Per-axis fields selected without dynamic indexing (which would spill the
// argument struct to scratch).
template <typename T>
__device__ __forceinline__ T pick(const T (&v)[2], int axis) {
  const T v0 = v[0], v1 = v[1];  // values, so the select is not between two addresses
  return axis ? v1 : v0;
}

// Cache index of (b, h, slot pos, feature row): the paged feature-major layout,
// or (tm, the LLA-2D key cache) token-major rows of r features.
__device__ __forceinline__ size_t cache_index(int b, int h, int H, int n_max, int r, int pos,
                                              int row, bool tm = false) {
  if (tm) return ((size_t)(b * H + h) * n_max + pos) * r + row;
  return ((size_t)(b * H + h) * n_max + (size_t)(pos / kPage) * kPage) * r + (size_t)row * kPage +
         (pos % kPage);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kEncTok = 32;           // tokens per workgroup block
constexpr int kEncKC = 512;           // K elements staged per step
constexpr int kEncXS = kEncKC + 8;    // LDS row stride (elements): 1040 B, staggers banks
constexpr int kEncMaxTasks = 4;       // 16x16 output tiles per wavefront

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// One workgroup: 32 consecutive tokens (b, m flattened) x heads [h0, h1) x
// 16-row output tiles [rt0, rt1) of one axis.  x is streamed through
// double-buffered LDS one (head, 512-element K chunk) stage at a time: each
// wave-wide load reads one token's contiguous 1 KB, and the next stage's loads
// are in flight while the current stage is multiplied.  Each wavefront owns up
// to 4 (row tile, token tile) 16x16 accumulators (v_mfma_f32_16x16x32_bf16:
// A = 16 rows of W_down^T from L2, B = 16 tokens from LDS); a head's tiles
// are written to the feature-major cache pages after its last K chunk.
// grid: x = token blocks, y = head chunks, z = axis * nrc + row chunk
__global__ __launch_bounds__(256) void encode_bf16_kernel(EncodeArgs a, int heads_per_wg, int rt_per_wg,
                                                          int nrc) {
  __shared__ __attribute__((aligned(16))) bf16_t s_x[2][kEncTok * kEncXS];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int axis = blockIdx.z / nrc, rc = blockIdx.z - axis * nrc;
  const int r = pick(a.r, axis), K = a.K, H = a.H;
  const int RT = (r + 15) / 16;
  const int rt0 = rc * rt_per_wg;
  if (rt0 >= RT) return;  // uniform over the workgroup
  const int rt1 = min(RT, rt0 + rt_per_wg);
  const int ntask = (rt1 - rt0) * 2;  // x 2 token tiles of 16
  const int h0 = blockIdx.y * heads_per_wg, h1 = min(H, h0 + heads_per_wg);
  const int TT = a.B * a.M;
  const int t0 = blockIdx.x * kEncTok;
  const int nkc = (K + kEncKC - 1) / kEncKC;
  const int nstage = (h1 - h0) * nkc;
  const bf16_t* xg = static_cast<const bf16_t*>(pick(a.x, axis));
  const bf16_t* wg = static_cast<const bf16_t*>(pick(a.wdt, axis));
  const bf16_t* mug = static_cast<const bf16_t*>(pick(a.mu, axis));

  uint4 rgs[8];
  auto stage_load = [&](int st) {
    const int h = h0 + st / nkc, k0 = (st % nkc) * kEncKC;
    const int cpt = min(kEncKC, K - k0) / 8;  // 16-byte chunks per token
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = tid + i * 256;
      if (c < kEncTok * cpt) {
        const int tok = c / cpt, part = c - tok * cpt, t = t0 + tok;
        // tokens past the last one re-read it: their output columns are never stored
        rgs[i] = ld16(xg + ((size_t)min(t, TT - 1) * H + h) * K + k0 + part * 8);
      }
    }
  };
  auto stage_store = [&](int st, int buf) {
    const int k0 = (st % nkc) * kEncKC;
    const int cpt = min(kEncKC, K - k0) / 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = tid + i * 256;
      if (c < kEncTok * cpt) {
        const int tok = c / cpt, part = c - tok * cpt;
        *reinterpret_cast<uint4*>(&s_x[buf][tok * kEncXS + part * 8]) = rgs[i];
      }
    }
  };

  f32x4 acc[kEncMaxTasks], accm[kEncMaxTasks];
#pragma unroll
  for (int u = 0; u < kEncMaxTasks; ++u) acc[u] = accm[u] = f32x4{0.f};
  const int li = lane & 15, lg = lane >> 4;

  stage_load(0);
  stage_store(0, 0);
  __syncthreads();
  for (int st = 0; st < nstage; ++st) {
    const int buf = st & 1;
    if (st + 1 < nstage) stage_load(st + 1);
    const int h = h0 + st / nkc, kc = st % nkc, k0 = kc * kEncKC;
    const int ks = min(kEncKC, K - k0) / 32;  // K-steps of 32 in this chunk
#pragma unroll
    for (int u = 0; u < kEncMaxTasks; ++u) {
      const int task = wave + 4 * u;
      if (task < ntask) {
        const int rt = rt0 + task / 2, tt = task % 2;
        const int row = rt * 16 + li;
        const bool row_ok = row < r;
        const bf16_t* wrow = wg + ((size_t)h * r + (row_ok ? row : 0)) * K + k0 + 8 * lg;
        const bf16_t* xrow = &s_x[buf][(tt * 16 + li) * kEncXS + 8 * lg];
        const bf16_t* mrow = mug ? mug + (size_t)h * K + k0 + 8 * lg : nullptr;
        // eight K-steps of W_down^T fragments in flight at once (with few
        // tokens the weights are the whole traffic, and a load per step
        // would expose the load latency sixteen times per chunk)
        for (int s0 = 0; s0 < ks; s0 += 8) {
          bf16x8 av[8];
#pragma unroll
          for (int j = 0; j < 8; ++j)
            av[j] = as_bf16x8(row_ok && s0 + j < ks ? ld16(wrow + 32 * (s0 + j)) : make_uint4(0, 0, 0, 0));
          if (s0 + 8 <= ks) {
            // a whole group: no guard per product (a guard there makes each
            // MFMA a block of its own, waiting on its own operand reads)
            if (mrow) {
              uint4 mv[8];
#pragma unroll
              for (int j = 0; j < 8; ++j) mv[j] = ld16(mrow + 32 * (s0 + j));
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const bf16x8 bv = as_bf16x8(*reinterpret_cast<const uint4*>(xrow + 32 * (s0 + j)));
                acc[u] = mfma16(av[j], bv, acc[u]);
                accm[u] = mfma16(av[j], as_bf16x8(mv[j]), accm[u]);
              }
            } else {
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const bf16x8 bv = as_bf16x8(*reinterpret_cast<const uint4*>(xrow + 32 * (s0 + j)));
                acc[u] = mfma16(av[j], bv, acc[u]);
              }
            }
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              if (s0 + j < ks) {
                const bf16x8 bv = as_bf16x8(*reinterpret_cast<const uint4*>(xrow + 32 * (s0 + j)));
                acc[u] = mfma16(av[j], bv, acc[u]);
                if (mrow) accm[u] = mfma16(av[j], as_bf16x8(ld16(mrow + 32 * (s0 + j))), accm[u]);
              }
            }
          }
        }
        if (kc == nkc - 1) {  // head done: write its tile, c = x W - mu W
          const int t = t0 + tt * 16 + li;
          if (t < TT) {
            const int b = t / a.M, pos = ring_slot(a.pos0 + (t - b * a.M), a.sink, a.window);
            bf16_t* c = static_cast<bf16_t*>(pick(a.c, axis));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int rr = rt * 16 + 4 * lg + e;
              if (rr < r) c[cache_index(b, h, H, a.n_max, r, pos, rr, axis == 0 && a.k_token_major)] = f32_to_bf16(acc[u][e] - accm[u][e]);
            }
          }
          acc[u] = accm[u] = f32x4{0.f};
        }
      }
    }
    if (st + 1 < nstage) stage_store(st + 1, buf ^ 1);
    __syncthreads();
  }
}

// Many new tokens at small ranks (a prefill's cache write, r <= 64, T*d = KS*32):
// the weights stay in registers and the tokens stream past them.  Grid:
// x = token ranges, y = head, z = axis.  Wavefront w owns 16-row tile rt of
// the head's W_down^T (its A fragments for the whole T*d held in KS registers
// of 16 bytes) and one or two 16-token tiles of every 32-token block; blocks
// of x are staged through double-buffered LDS with coalesced 1 KB loads.  The
// mean term W_down^T mu is one extra product per workgroup at the start.
template <int KS>
__global__ __launch_bounds__(256) void encode_stream_kernel(EncodeArgs a, int blocks_per_wg) {
  constexpr int K = KS * 32;
  constexpr int XS = K + 8;
  __shared__ __attribute__((aligned(16))) bf16_t s_x[2][kEncTok * XS];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int axis = blockIdx.z, h = blockIdx.y, H = a.H;
  const int r = pick(a.r, axis);
  const int RT = r > 32 ? 4 : 2;           // 16-row tiles (rows >= r are zero)
  const int rt = wave % RT;
  const int ntt = RT == 4 ? 2 : 1;         // token tiles per wavefront
  const int tt0 = RT == 4 ? 0 : wave / 2;
  const int TT = a.B * a.M;
  const int nblk = (TT + kEncTok - 1) / kEncTok;
  const int b0 = blockIdx.x * blocks_per_wg, b1 = min(nblk, b0 + blocks_per_wg);
  if (b0 >= b1) return;
  const int li = lane & 15, lg = lane >> 4;
  const int row = rt * 16 + li;
  const bool row_ok = row < r;

  // resident A fragments of W_down^T rows [16 rt, 16 rt + 16)
  const bf16_t* wrow = static_cast<const bf16_t*>(pick(a.wdt, axis)) + ((size_t)h * r + (row_ok ? row : 0)) * K + 8 * lg;
  bf16x8 wf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) wf[s] = as_bf16x8(row_ok ? ld16(wrow + 32 * s) : make_uint4(0, 0, 0, 0));
  f32x4 bmu = f32x4{0.f};
  if (pick(a.mu, axis)) {
    const bf16_t* mrow = static_cast<const bf16_t*>(pick(a.mu, axis)) + (size_t)h * K + 8 * lg;
#pragma unroll
    for (int s = 0; s < KS; ++s) bmu = mfma16(wf[s], as_bf16x8(ld16(mrow + 32 * s)), bmu);
  }

  const bf16_t* xg = static_cast<const bf16_t*>(pick(a.x, axis));
  constexpr int CPT = K / 8;                               // 16-byte chunks per token
  constexpr int NCH = (kEncTok * CPT + 255) / 256;         // chunks per thread per block
  uint4 rgs[NCH];
  auto load_blk = [&](int blk) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 256;
      if (c < kEncTok * CPT) {
        const int tok = c / CPT, part = c - tok * CPT, t = blk * kEncTok + tok;
        // tokens past the last one re-read it: their output columns are never stored;
        // x is read once (non-temporal: 210 -> 192 us on the 4 x 8192-token write)
        rgs[i] = ld16_nt(xg + ((size_t)min(t, TT - 1) * H + h) * K + part * 8);
      }
    }
  };
  auto store_blk = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 256;
      if (c < kEncTok * CPT) {
        const int tok = c / CPT, part = c - tok * CPT;
        *reinterpret_cast<uint4*>(&s_x[buf][tok * XS + part * 8]) = rgs[i];
      }
    }
  };

  bf16_t* cout = static_cast<bf16_t*>(pick(a.c, axis));
  load_blk(b0);
  store_blk(0);
  __syncthreads();
  for (int blk = b0; blk < b1; ++blk) {
    const int buf = (blk - b0) & 1;
    if (blk + 1 < b1) load_blk(blk + 1);
    for (int u = 0; u < ntt; ++u) {
      const int tt = tt0 + u;
      const bf16_t* xrow = &s_x[buf][(tt * 16 + li) * XS + 8 * lg];
      f32x4 acc = f32x4{0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s)
        acc = mfma16(wf[s], as_bf16x8(*reinterpret_cast<const uint4*>(xrow + 32 * s)), acc);
      const int t = blk * kEncTok + tt * 16 + li;
      if (t < TT) {
        const int b = t / a.M, pos = ring_slot(a.pos0 + (t - b * a.M), a.sink, a.window);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int rr = rt * 16 + 4 * lg + e;
          if (rr < r) cout[cache_index(b, h, H, a.n_max, r, pos, rr, axis == 0 && a.k_token_major)] = f32_to_bf16(acc[e] - bmu[e]);
        }
      }
    }
    if (blk + 1 < b1) store_blk(buf ^ 1);
    __syncthreads();
  }
}

// Few new tokens (a decode step writes one per sequence): the weights are the
// whole traffic, so every W_down^T element is read once and nothing waits on
// more than one round of loads.  Workgroup = 32 rows of one (axis, head) x 32
// tokens; wavefront w computes the 16x16 tile (row tile w % 2, token tile
// w / 2) with both operands loaded straight from global memory, sixteen
// K-steps of A and B fragments in flight at once (no LDS, no barrier).
// With a long K (the LLA-2D stack) the K-steps are split over ksplit
// workgroups per tile so the weights spread over the whole machine; each
// writes its fp32 partial tile and encode_reduce_kernel (the next launch)
// adds them and writes the cache.
// grid: x = 32-token blocks, y = 32-row chunks of axis k then axis v,
// z = head * ksplit + K-split
__global__ __launch_bounds__(256) void encode_few_kernel(EncodeArgs a, int nrc_k) {
  constexpr int CH = 16;  // K-steps per round of loads
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int axis = blockIdx.y >= (unsigned)nrc_k ? 1 : 0;
  const int rc = blockIdx.y - axis * nrc_k;
  const int split = blockIdx.z % a.ksplit, h = blockIdx.z / a.ksplit, H = a.H, K = a.K;
  const int r = pick(a.r, axis);
  const int li = lane & 15, lg = lane >> 4;
  const int row = rc * 32 + (wave & 1) * 16 + li;
  const int TT = a.B * a.M;
  const int tcol = blockIdx.x * 32 + (wave >> 1) * 16 + li;  // token of this lane's B column
  const bool row_ok = row < r, tok_ok = tcol < TT;
  const bf16_t* wrow = static_cast<const bf16_t*>(pick(a.wdt, axis)) + ((size_t)h * r + (row_ok ? row : 0)) * K + 8 * lg;
  const bf16_t* xrow = static_cast<const bf16_t*>(pick(a.x, axis)) + ((size_t)(tok_ok ? tcol : 0) * H + h) * K + 8 * lg;
  const bf16_t* mrow = pick(a.mu, axis) ? static_cast<const bf16_t*>(pick(a.mu, axis)) + (size_t)h * K + 8 * lg : nullptr;
  const uint4 zero = make_uint4(0, 0, 0, 0);
  const int per = (K / 32 + a.ksplit - 1) / a.ksplit;  // K-steps of this split: [sb, se)
  const int sb = split * per, se = min(K / 32, sb + per);
  f32x4 acc = f32x4{0.f}, accm = f32x4{0.f};
  for (int s0 = sb; s0 < se; s0 += CH) {
    bf16x8 wf[CH], xf[CH], mf[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const bool in = s0 + j < se;
      wf[j] = as_bf16x8(row_ok && in ? ld16(wrow + 32 * (s0 + j)) : zero);
      xf[j] = as_bf16x8(tok_ok && in ? ld16(xrow + 32 * (s0 + j)) : zero);
      mf[j] = as_bf16x8(mrow && in ? ld16(mrow + 32 * (s0 + j)) : zero);
    }
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      acc = mfma16(wf[j], xf[j], acc);
      if (mrow) accm = mfma16(wf[j], mf[j], accm);
    }
  }
  acc -= accm;
  if (a.ksplit > 1) {  // partial tile; encode_reduce_kernel adds the splits
    const size_t unit = ((size_t)h * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    *reinterpret_cast<f32x4*>(a.part + (unit * a.ksplit + split) * 1024 + tid * 4) = acc;
    return;
  }
  // output tile: lane (li, lg) holds rows 4 lg .. 4 lg + 3 of token column li
  const int t = blockIdx.x * 32 + (wave >> 1) * 16 + li;
  if (t < TT) {
    const int b = t / a.M, pos = ring_slot(a.pos0 + (t - b * a.M), a.sink, a.window);
    bf16_t* c = static_cast<bf16_t*>(pick(a.c, axis));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rr = rc * 32 + (wave & 1) * 16 + 4 * lg + e;
      if (rr < r) c[cache_index(b, h, H, a.n_max, r, pos, rr, axis == 0 && a.k_token_major)] = f32_to_bf16(acc[e]);
    }
  }
}

// Writes of many tokens: 2 r flops per byte of x, a GEMM.  A workgroup of 4
// wavefronts takes 128 XT tokens x up to 96 rows of one axis, wavefront w tokens
// 32 XT w .. x all rows on v_mfma_f32_32x32x16_bf16:
//   keys   (token-major cache): D = C^T (M = row, N = token), a lane holds
//          4-row runs of one token;
//   values, per-head keys (feature-major pages): D = C (M = token, N = row).
// Weights pass through double-buffered LDS chunks of 64 values, read by every
// wavefront.  A token belongs to one wavefront: its x passes through a region
// of LDS that only this wavefront uses (a wave-wide load covers 8 tokens x 128
// bytes; straight to the operand registers each lane's 16 bytes were a cache
// line of their own, which bound the loop), with one or two further chunks in
// registers and no barrier.  5 KB of LDS reads feed 6 products, where one
// 32-token tile per wavefront took 4 KB for 3; two workgroups share a compute
// unit.
// The row blocks of one token block are dispatched back to back on one XCD
// (workgroup i runs on XCD i % 8), so its x comes from that XCD's L2 after the
// first read.  W_down^T mu is formed on the vector unit from the staged weights.
// Measured against one 8-wavefront workgroup of 256 x 96 per compute unit with
// both operands in shared LDS: 2 x 3001 tokens (192, 320) with means 216 -> 119
// us (its bytes at the copy rate take 59), 4 x 8192 (288, 480) 950 -> 686 us (601
// TFLOP/s), 300 tokens (96, 160) 35 -> 17, the LLA-2D stack (K = 8192) 4 x 8192
// tokens 615 -> 484 us (852 TFLOP/s).  Bound by latency: at 2 x 3001 the vector unit
// (epilogue, mean) is busy 33% of the time, LDS 27%, the matrix units 18%, at 2 x 4096
// of the stack 16, 43 and 32%; wavefronts wait a third of theirs.
constexpr int kGRow = 96, kGKC = 64, kGS = kGKC + 8;
constexpr int kGThreads = 256;
template <int XT>
constexpr int kGRing = XT == 2 ? 1 : 2;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

template <int XT>
struct GemmLds {
  __attribute__((aligned(16))) bf16_t x[4][32 * XT * kGS];  // each wavefront's tokens, one chunk
  __attribute__((aligned(16))) bf16_t w[2][kGRow * kGS];
  __attribute__((aligned(16))) bf16_t mu[2][kGKC];
  float wmu[kGRow];                                       // W_down^T mu of the current head
  __attribute__((aligned(16))) bf16_t tile[4][32 * 40];   // epilogue tile of each wavefront
};

// AXIS: 0 keys, 1 values.  TM: the output cache is token-major (the LLA-2D key
// cache); the products then hold rows in a lane's registers (one token per
// lane), stored as 8 bytes of 4 consecutive features.  Otherwise a lane's
// register groups hold 4 consecutive tokens of one row, and the tile reaches
// the feature-major pages through LDS as 16-byte pieces of whole page rows.
// RT: 32-row tiles.  The workgroup walks heads h0 .. h0 + nh - 1 as one stream
// of K-chunks, so a head's first loads are in flight while the previous head
// finishes.
template <int AXIS, bool TM, int RT, int XT>
__device__ __forceinline__ void encode_gemm_body(const EncodeArgs& a, int tfirst, int tlo, int thi, int row0, int h0, int nh,
                                                 GemmLds<XT>& s) {
  constexpr int NR = kGRing<XT>;  // chunks of x in registers
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 31, g = lane >> 5;
  const int r = pick(a.r, AXIS), K = a.K, H = a.H;
  const int t0 = tfirst + wave * 32 * XT;
  const bf16_t* mug = static_cast<const bf16_t*>(pick(a.mu, AXIS));
  const bool mu = mug != nullptr;  // uniform
  const int nkc = K / kGKC, total = nh * nkc;

  // x: the heads of a token are adjacent, so chunk q of the stream is at 64 q;
  // lane (token lane / 8 of 8, piece lane % 8).  Tokens outside [tlo, thi)
  // re-read one inside: their columns are never stored.
  const bf16_t* xp[4 * XT];
#pragma unroll
  for (int i = 0; i < 4 * XT; ++i)
    xp[i] = static_cast<const bf16_t*>(pick(a.x, AXIS)) +
            ((size_t)max(tlo, min(t0 + 8 * i + (lane >> 3), thi - 1)) * H + h0) * K + 8 * (lane & 7);
  uint4 x[NR][4 * XT];
  auto xload = [&](uint4 (&v)[4 * XT], int q) {
    const int o = kGKC * min(q, total - 1);
#pragma unroll
    for (int i = 0; i < 4 * XT; ++i) v[i] = ld16(xp[i] + o);
  };
  bf16_t* const xs = s.x[wave];
  auto xstore = [&](const uint4 (&v)[4 * XT]) {
#pragma unroll
    for (int i = 0; i < 4 * XT; ++i)
      *reinterpret_cast<uint4*>(&xs[(8 * i + (lane >> 3)) * kGS + 8 * (lane & 7)]) = v[i];
  };
  // W chunk: RT * 32 rows x 64, RT 16-byte pieces per thread; the mean's 64
  // values, one piece of threads 0 .. 7
  uint4 sw[RT], sm = make_uint4(0, 0, 0, 0);
  int lh = h0, lk = 0;  // head and K-chunk of the next W load
  auto wload = [&]() {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int row = min(row0 + 32 * i + (tid >> 3), r - 1);  // rows past the rank: never stored
      sw[i] = ld16(static_cast<const bf16_t*>(pick(a.wdt, AXIS)) + ((size_t)lh * r + row) * K + lk * kGKC + 8 * (tid & 7));
    }
    if (mu && tid < 8) sm = ld16(mug + (size_t)lh * K + lk * kGKC + 8 * tid);
    if (lk + 1 < nkc) {
      ++lk;
    } else if (lh + 1 < h0 + nh) {  // the last chunk is re-read, not multiplied
      lk = 0;
      ++lh;
    }
  };
  auto wstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
      *reinterpret_cast<uint4*>(&s.w[buf][(32 * i + (tid >> 3)) * kGS + 8 * (tid & 7)]) = sw[i];
    if (mu && tid < 8) *reinterpret_cast<uint4*>(&s.mu[buf][8 * tid]) = sm;
  };

  f32x16 acc[XT][RT];
#pragma unroll
  for (int u = 0; u < XT; ++u)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[u][rt] = f32x16{0.f};
  float wmu = 0.f;  // row tid / 2, half tid % 2 of every chunk

  auto chunk = [&](int buf) {
    const bf16_t* ws = &s.w[buf][col * kGS + 8 * g];
    const bf16_t* xr = &xs[col * kGS + 8 * g];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      bf16x8 wo[RT], xo[XT];
#pragma unroll
      for (int u = 0; u < XT; ++u) xo[u] = as_bf16x8(*reinterpret_cast<const uint4*>(xr + 32 * u * kGS + 16 * k));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) wo[rt] = as_bf16x8(*reinterpret_cast<const uint4*>(ws + 32 * rt * kGS + 16 * k));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int u = 0; u < XT; ++u)
          acc[u][rt] = TM ? mfma32(wo[rt], xo[u], acc[u][rt]) : mfma32(xo[u], wo[rt], acc[u][rt]);
    }
  };
  auto mean = [&](int buf) {
    if (mu && tid < 64 * RT) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float wv[8], mv[8];
        Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(&s.w[buf][(tid >> 1) * kGS + 32 * (tid & 1) + 8 * k]), wv);
        Elem<bf16_t>::unpack(*reinterpret_cast<const uint4*>(&s.mu[buf][32 * (tid & 1) + 8 * k]), mv);
#pragma unroll
        for (int e = 0; e < 8; ++e) wmu = fmaf(wv[e], mv[e], wmu);
      }
    }
  };
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // head hh done: the tile to the cache, then the accumulators cleared
  auto finish = [&](int hh_) {
    // Opaque copies: the epilogue's row and token bookkeeping is then formed
    // here, per head, instead of being hoisted out of the head loop, where it
    // would hold registers across every chunk.
    int hh = hh_, r = pick(a.r, AXIS), rw = row0, tw = t0;
    asm volatile("" : "+s"(hh), "+s"(r), "+s"(rw), "+s"(tw));
    if (mu) {
      wmu += xor_shfl(wmu, 1);
      if (tid < 64 * RT && (tid & 1) == 0) s.wmu[tid >> 1] = wmu;
      wmu = 0.f;
      __syncthreads();
    }
    bf16_t* cout = static_cast<bf16_t*>(pick(a.c, AXIS));
    if constexpr (TM) {
      // lane (token col, half g), register q of row tile rt: row 32 rt + 8(q/4) + 4g + q%4
#pragma unroll
      for (int u = 0; u < XT; ++u) {
        const int t = tw + 32 * u + col;
        if (t >= tlo && t < thi) {
          const int b = t / a.M, pos = ring_slot(a.pos0 + (t - b * a.M), a.sink, a.window);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int rl = 32 * rt + 8 * i + 4 * g, row = rw + rl;  // first of 4 consecutive rows
              bf16_t v[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = f32_to_bf16(acc[u][rt][4 * i + e] - (mu ? s.wmu[rl + e] : 0.f));
              bf16_t* dst = &cout[cache_index(b, hh, H, a.n_max, r, pos, row, true)];
              if (row + 3 < r)  // the 4 rows are contiguous, 8-byte aligned (r_k % 32 == 0)
                *reinterpret_cast<uint2*>(dst) = make_uint2(v[0] | (uint32_t(v[1]) << 16), v[2] | (uint32_t(v[3]) << 16));
              else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (row + e < r) dst[e] = v[e];
            }
        }
      }
    } else {
      // lane (row col of tile rt, half g), register q: token 8(q/4) + 4g + q%4
      // of a 32-token tile, so registers 4i .. 4i + 3 are 4 consecutive tokens
      // of one feature row.  Each wavefront turns a row tile through its own
      // LDS tile [row][token]; runs of 4 lanes then store a row's tokens 16
      // bytes each where their slots are 8 consecutive ones of one sequence from
      // a multiple of 8.  Other tokens are stored by a lane each, two rows of 32 or
      // more of fewer at a time (a wavefront's stores are then runs of consecutive
      // slots; eight tokens by one lane in turn touched 16 rows per store).
      bf16_t* tile = s.tile[wave];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float m = mu ? s.wmu[32 * rt + col] : 0.f;
#pragma unroll
        for (int u = 0; u < XT; ++u) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            uint32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = f32_to_bf16(acc[u][rt][4 * i + e] - m);
            *reinterpret_cast<uint2*>(&tile[col * 40 + 8 * i + 4 * g]) = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
          }
          wave_sync();
          const int tt = tw + 32 * u;
          // whether the 8 tokens from t are 8 consecutive slots from a multiple of 8
          auto whole = [&](int t, int& b, int& p) {
            b = t / a.M;
            const int m0 = t - b * a.M;
            p = ring_slot(a.pos0 + m0, a.sink, a.window);
            return t >= tlo && t + 7 < thi && m0 + 7 < a.M && (p & 7) == 0 &&
                   ring_slot(a.pos0 + m0 + 7, a.sink, a.window) == p + 7;
          };
          const int grp = lane & 3;
          int b, p;
          if (whole(tt + 8 * grp, b, p)) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const int rl = (lane >> 2) + 16 * k, row = rw + 32 * rt + rl;
              if (row < r)
                *reinterpret_cast<uint4*>(&cout[cache_index(b, hh, H, a.n_max, r, p, row)]) =
                    *reinterpret_cast<const uint4*>(&tile[rl * 40 + 8 * grp]);
            }
          }
          const int te = tt + col;
          const uint32_t single = (uint32_t)__builtin_amdgcn_ballot_w64(te >= tlo && te < thi &&
                                                                        !whole(tt + (col & ~7), b, p));
          if (single) {  // uniform; tokens first .. first + 2^sh - 1 over the lanes, 64 / 2^sh rows at a time
            const int first = __builtin_ctz(single), n = 32 - __builtin_clz(single) - first;
            const int sh = n > 1 ? 32 - __builtin_clz(n - 1) : 0;
            const int tk = first + (lane & ((1 << sh) - 1));
            if (tk < 32 && ((single >> tk) & 1)) {
              b = (tt + tk) / a.M;
              p = ring_slot(a.pos0 + (tt + tk - b * a.M), a.sink, a.window);
              bf16_t* dst = &cout[cache_index(b, hh, H, a.n_max, r, p, rw + 32 * rt)];
              const int rows = min(32, r - (rw + 32 * rt));
#pragma unroll 4
              for (int row = lane >> sh; row < rows; row += kWave >> sh) dst[row * kPage] = tile[row * 40 + tk];
            }
          }
          wave_sync();
        }
      }
    }
#pragma unroll
    for (int u = 0; u < XT; ++u)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[u][rt] = f32x16{0.f};
  };

  // Chunk q's weights are in LDS buffer q % 2, its x in the wavefront's region,
  // chunks q + 1 .. q + NR of x in registers (q + 1 in slot q % NR; with
  // NR = 2 a workgroup takes one head, so any number of chunks will do).  W
  // chunk q + 1 is stored to the buffer that chunk q - 1 left, after chunk q's
  // products; x chunk q + 1 after them in the wavefront's own order.
  wload();
  xload(x[NR - 1], 0);
  wstore(0);
  xstore(x[NR - 1]);
  wload();
#pragma unroll
  for (int q = 0; q < NR; ++q) xload(x[q], q + 1);
  __syncthreads();
  for (int hq = 0, q = 0; hq < nh; ++hq) {
    for (int kc = 0; kc < nkc; kc += NR, q += NR) {
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        if (kc + i < nkc) {
          const int buf = (q + i) & 1;
          chunk(buf);
          wave_sync();
          xstore(x[i]);
          xload(x[i], q + i + 1 + NR);
          mean(buf);
          wstore(buf ^ 1);
          wload();
          __syncthreads();
        }
      }
    }
    finish(h0 + hq);
  }
}

// Both axes in one launch.  XCD-aware order: the j-th workgroup of XCD x takes
// token block x + 8 (j / nrb) and row block j % nrb (the row blocks of axis k,
// then those of axis v).  An axis of n 32-row tiles is cut into ceil(n / 3)
// blocks of 3, 2 or 1 tiles (160 rows: 3 + 2; 320: 3 + 3 + 2 + 2).
template <int XT>
__global__ __launch_bounds__(kGThreads) __attribute__((amdgpu_waves_per_eu(2)))
void encode_gemm_kernel(EncodeArgs a, int nrb_k, int nrb, int ntb, int nsb, int hpw) {
  __shared__ GemmLds<XT> s;
  const int xcd = blockIdx.x % 8, j = blockIdx.x / 8;
  const int tb = xcd + 8 * (j / nrb), rb = j % nrb;
  if (tb >= ntb) return;  // padding of the grid to whole rounds of 8 token blocks
  // nsb blocks per sequence, cut at cache slots that are multiples of the block
  // (the pieces of the epilogue then start on 16 bytes whatever M and pos0
  // are), or (nsb 0) blocks of the flattened tokens
  int tfirst = tb * 128 * XT, tlo = 0, thi = a.B * a.M;
  if (nsb) {
    const int b = tb / nsb;
    tlo = b * a.M;
    thi = tlo + a.M;
    tfirst = tlo + (tb - b * nsb) * 128 * XT - (a.pos0 & 7);
  }
  const int h0 = blockIdx.y * hpw, nh = min(hpw, a.H - h0);  // a run of heads
  const int axis = rb >= nrb_k ? 1 : 0, blocks = axis ? nrb - nrb_k : nrb_k, i = rb - axis * nrb_k;
  const int nt = (pick(a.r, axis) + 31) / 32;  // tiles of the axis
  const int f0 = i * nt / blocks, rt = (i + 1) * nt / blocks - f0;
  auto run = [&](auto ax, auto tm) {
    constexpr int A = decltype(ax)::value;
    constexpr bool T = decltype(tm)::value;
    if (rt == 3)
      encode_gemm_body<A, T, 3, XT>(a, tfirst, tlo, thi, 32 * f0, h0, nh, s);
    else if (rt == 2)
      encode_gemm_body<A, T, 2, XT>(a, tfirst, tlo, thi, 32 * f0, h0, nh, s);
    else
      encode_gemm_body<A, T, 1, XT>(a, tfirst, tlo, thi, 32 * f0, h0, nh, s);
  };
  if (axis)
    run(std::integral_constant<int, 1>{}, std::false_type{});
  else if (a.k_token_major)
    run(std::integral_constant<int, 0>{}, std::true_type{});
  else
    run(std::integral_constant<int, 0>{}, std::false_type{});
}

// Second launch of a split write: tile unit (grid x, y, z as the split launch
// with z = head) adds its ksplit fp32 partials in split order and writes the
// cache exactly as the unsplit path does.
__global__ __launch_bounds__(256) void encode_reduce_kernel(EncodeArgs a, int nrc_k) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int axis = blockIdx.y >= (unsigned)nrc_k ? 1 : 0;
  const int rc = blockIdx.y - axis * nrc_k;
  const int h = blockIdx.z, H = a.H, r = pick(a.r, axis), TT = a.B * a.M;
  const int li = lane & 15, lg = lane >> 4;
  const size_t unit = ((size_t)h * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
  const float* part = a.part + unit * a.ksplit * 1024 + tid * 4;
  constexpr int kPre = 32;  // partials in flight at once
  f32x4 v[kPre];
#pragma unroll
  for (int s = 0; s < kPre; ++s)
    v[s] = s < a.ksplit ? *reinterpret_cast<const f32x4*>(part + (size_t)s * 1024) : f32x4{0.f};
  f32x4 acc = f32x4{0.f};
#pragma unroll
  for (int s = 0; s < kPre; ++s) acc += v[s];
  const int t = blockIdx.x * 32 + (wave >> 1) * 16 + li;
  if (t < TT) {
    const int b = t / a.M, pos = ring_slot(a.pos0 + (t - b * a.M), a.sink, a.window);
    bf16_t* c = static_cast<bf16_t*>(pick(a.c, axis));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rr = rc * 32 + (wave & 1) * 16 + 4 * lg + e;
      if (rr < r) c[cache_index(b, h, H, a.n_max, r, pos, rr, axis == 0 && a.k_token_major)] = f32_to_bf16(acc[e]);
    }
  }
}

// fp32, on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: products and
// sums in fp32).  Workgroup = 32 rows x 32 tokens of one (axis, head); its four
// wavefronts split K in turn, 16 values at a time, each with a 2 x 2 block of
// 16x16 tiles: a lane's 16 bytes (row or token lane % 16, values 4 (lane / 16) ..)
// are the operands of four products with both tiles of the other side,
// straight from memory.  The four partial blocks add
// through LDS in wavefront order, and a row of 32 tokens leaves as 128
// consecutive bytes.  x - mu is formed in fp32 before the product.
// grid: x = token block x row block (axis k, then v), y = head; a head's
// workgroups on one XCD, whose L2 then holds its weights.  500 tokens of 16
// heads, K = 512, (96, 160): 159 us with LDS-staged vector products (two LDS
// reads per multiply-add), 37 us here (14 us of products at the matrix rate).
constexpr int kFS = 36;  // LDS row stride of a partial block
__global__ __launch_bounds__(256) void encode_f32_kernel(EncodeArgs a, int nrc_k, int nrc) {
  __shared__ __attribute__((aligned(16))) float s_part[4][32 * kFS];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  int bx, h;
  xcd_head_order(bx, h, true);
  const int tb = (unsigned)bx / (unsigned)nrc, rc_ = bx - tb * nrc;
  const int axis = rc_ >= nrc_k ? 1 : 0, rc = rc_ - axis * nrc_k;
  const int r = pick(a.r, axis), K = a.K, H = a.H, TT = a.B * a.M;
  const int c = lane & 15, g = lane >> 4;
  const float* mu = pick(a.mu, axis) ? static_cast<const float*>(pick(a.mu, axis)) + (size_t)h * K + 4 * g : nullptr;
  const float *xp[2], *wp[2];  // rows and tokens past the last one re-read it: never stored
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    xp[u] = static_cast<const float*>(pick(a.x, axis)) + ((size_t)min(tb * 32 + 16 * u + c, TT - 1) * H + h) * K + 4 * g;
    wp[u] = static_cast<const float*>(pick(a.wdt, axis)) + ((size_t)h * r + min(rc * 32 + 16 * u + c, r - 1)) * K + 4 * g;
  }
  f32x4 acc[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u) acc[u][0] = acc[u][1] = f32x4{0.f};
#pragma unroll 2
  for (int k0 = 16 * wave; k0 < K; k0 += 64) {
    f32x4 x[2], w[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      x[u] = *reinterpret_cast<const f32x4*>(xp[u] + k0);
      w[u] = *reinterpret_cast<const f32x4*>(wp[u] + k0);
    }
    if (mu) {
      const f32x4 m = *reinterpret_cast<const f32x4*>(mu + k0);
      x[0] -= m;
      x[1] -= m;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
          acc[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][e], x[v][e], acc[u][v], 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) s_part[wave][(16 * u + 4 * g + e) * kFS + 16 * v + c] = acc[u][v][e];
  __syncthreads();
  const int t = tb * 32 + (tid & 31);
  if (t >= TT) return;
  const int b = t / a.M, pos = ring_slot(a.pos0 + (t - b * a.M), a.sink, a.window);
  float* out = static_cast<float*>(pick(a.c, axis));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = (tid >> 5) + 8 * i, row = rc * 32 + rl;
    const int e = rl * kFS + (tid & 31);
    if (row < r)
      out[cache_index(b, h, H, a.n_max, r, pos, row, axis == 0 && a.k_token_major)] =
          s_part[0][e] + s_part[1][e] + s_part[2][e] + s_part[3][e];
  }
}

// Launch of a bf16 GEMM write with 32 XT tokens per wavefront.
template <int XT>
struct GemmGrid {
  int nrb_k, nrb;  // row blocks of axis k, of both axes
  int nsb, ntb;    // token blocks per sequence (0: of the flattened tokens), in all
  int hpw;         // heads per workgroup
  double rounds;   // workgroups that a slot of the busiest XCD takes in turn (two slots per compute unit)
  explicit GemmGrid(const EncodeArgs& a) {
    const int TT = a.B * a.M, q = 128 * XT;
    nrb_k = (a.r[0] + kGRow - 1) / kGRow;
    nrb = nrb_k + (a.r[1] + kGRow - 1) / kGRow;
    // Blocks cut per sequence unless that adds more than an eighth to the rounds
    // of the 8 XCDs (3 x 600 tokens (240, 400) with means: 9 blocks for 8 took 88 us,
    // 60 in one round; 5 x 3225 of 32 heads (120, 200), K = 256: 65 for 63 299, 342
    // over the flattened tokens, whose pieces are not whole).
    nsb = (a.M + (a.pos0 & 7) + q - 1) / q;
    ntb = (TT + q - 1) / q;
    if (((int64_t)nsb * a.B + 7) / 8 <= (ntb + 7) / 8 * 9 / 8)
      ntb = nsb * a.B;
    else
      nsb = 0;
    // With 64 tokens per wavefront as many heads as keep at least 2048
    // workgroups (four rounds of the machine), so short stacks (per-head
    // writes) do not pay the pipeline fill per head; 32 are for few workgroups.
    hpw = 1;
    if (XT == 2) hpw = (int)std::min<int64_t>(a.H, std::max<int64_t>(1, (int64_t)a.H * nrb * ntb / 2048));
    // While they are few the last round takes half a round and its share (workgroups
    // alone on a unit run faster), the first a whole one; then half a round of slack.
    rounds = std::max(1.0, (double)((ntb + 7) / 8) * nrb * a.H / std::max(1, device_cu_count() / 4));
    const double whole = std::floor(rounds);
    rounds = rounds >= 3 ? rounds + 0.5 : rounds > whole ? 0.5 * (rounds + whole + 1) : rounds;
  }
};

// Whether a bf16 write of more than 64 tokens runs the GEMM rather than the
// 32-token kernel.  A GEMM workgroup takes longer and does more (the more, the
// fuller its row blocks), so it pays where the 32-token kernel's workgroups
// (tokens / 32 x heads x 32-row tiles) come in several rounds: from about 640 at K
// = 512 and row blocks of 2.5 tiles, more the shorter K is; the 32-token kernel
// multiplies a mean once more, the GEMM nearly for free.  The line was drawn over
// 3871 writes of 1 to 32 heads, K 64 to 2048, ranks 1 to 512 and 192 to 40,000
// tokens, every kernel timed on each, with repeated and with other inputs: the one chosen
// is within 4% of the best of the three in 95 of 100, within 10% in 99.  32-token
// kernel / GEMM, 16 heads, K = 512: 300 tokens (96, 160) 24.4 / 20.1 us, 651 tokens (18, 30)
// 13.1 / 8.5, 3000 tokens (36, 60) 75.7 / 26.4; 4 heads, 203 tokens (96, 160) 8.4 / 14.6;
// 2 heads, 1532 tokens (36, 60) 10.2 / 13.6.  Below 256 tokens a token block is
// largely padding (2 x 98 tokens (120, 200) 22.3 / 24.0, 197 (288, 480) 43.6 /
// 31.2).  Stacks of 2048 values and more (LLA-2D) gain from 256 tokens.
bool gemm_ok(const EncodeArgs& a) {
  const int TT = a.B * a.M, nt = (a.r[0] + 31) / 32 + (a.r[1] + 31) / 32, nrb = GemmGrid<1>(a).nrb;
  if (TT < 192 || a.K % kGKC) return false;
  if (a.K >= 2048 && TT >= 256) return true;
  if (a.K >= 4096) return false;
  const double mean = a.mu[0] || a.mu[1] ? 1.375 : 1.0;
  const double work = (double)((TT + kEncTok - 1) / kEncTok) * a.H * nt * (a.K + 576) * mean * nrb / (nrb + nt);
  return work > (TT < 256 ? 512 << 10 : 195 << 10);
}

// 64 tokens per wavefront where 32 take more than 1.63 times the rounds (a
// workgroup of 64 takes that much longer), else 32: 1800 tokens of 16 heads (240, 400)
// with means 60 us with 32, 88 with 64 in the same number of rounds.
bool gemm_wide(const EncodeArgs& a) { return 1.63 * GemmGrid<2>(a).rounds < GemmGrid<1>(a).rounds; }

// The kernel of a bf16 write.
enum Route { kFew, kStream, kTok32, kGemm1, kGemm2 };
Route bf16_route(const EncodeArgs& a) {
  const int TT = a.B * a.M, blocks = (TT + kEncTok - 1) / kEncTok, rmax = a.r[0] > a.r[1] ? a.r[0] : a.r[1];
  if (TT <= 64) return kFew;  // a decode step's writes: weights read once, one round of loads
  // prefill-sized write at small ranks: resident weights, streamed tokens
  if (blocks >= 256 && rmax <= 64 && (a.K == 512 || a.K == 256)) return kStream;
  if (gemm_ok(a)) return gemm_wide(a) ? kGemm2 : kGemm1;
  return kTok32;
}

template <int XT>
hipError_t launch_gemm(const EncodeArgs& a, hipStream_t stream) {
  const GemmGrid<XT> g(a);
  hipLaunchKernelGGL((encode_gemm_kernel<XT>), dim3(g.nrb * ((g.ntb + 7) / 8 * 8), (a.H + g.hpw - 1) / g.hpw),
                     dim3(kGThreads), 0, stream, a, g.nrb_k, g.nrb, g.ntb, g.nsb, g.hpw);
  return hipGetLastError();
}

}  // namespace

int encode_ksplit(int TT, int K) {
  if (TT > 64 || K < 2048) return 1;
  const int s = K / 512;  // 16 K-steps (one round of loads) per split
  return s > 32 ? 32 : s;
}

size_t encode_ws_bytes(int B, int M, int H, int K, int r_k, int r_v) {
  const int TT = B * M, ks = encode_ksplit(TT, K);
  if (ks == 1) return 0;
  const size_t units = (size_t)((TT + kEncTok - 1) / kEncTok) * ((r_k + 31) / 32 + (r_v + 31) / 32) * H;
  return units * ks * 1024 * sizeof(float);
}

hipError_t launch_encode(const EncodeArgs& a, hipStream_t stream) {
  const int TT = a.B * a.M;
  const int rmax = a.r[0] > a.r[1] ? a.r[0] : a.r[1];
  const int nrc_k = (a.r[0] + 31) / 32, nrc_v = (a.r[1] + 31) / 32;
  if (a.dtype == LLA_F32) {
    // A launch takes fewer than 2^32 threads along x, 2^24 - 1 workgroups: larger
    // writes go out in runs of whole sequences, or of a sequence's tokens.
    const int nrc = nrc_k + nrc_v, most = ((1 << 24) - 1) / nrc * 32;
    const int nb = a.M <= most ? std::min(a.B, most / a.M) : 1, nm = std::min(a.M, most);
    for (int b = 0; b < a.B; b += nb)
      for (int m = 0; m < a.M; m += nm) {
        EncodeArgs s = a;
        s.B = std::min(nb, a.B - b);
        s.M = std::min(nm, a.M - m);
        s.pos0 = a.pos0 + m;
        for (int i = 0; i < 2; ++i) {
          s.x[i] = static_cast<const float*>(a.x[i]) + ((size_t)b * a.M + m) * a.H * a.K;
          s.c[i] = static_cast<float*>(a.c[i]) + (size_t)b * a.H * a.n_max * a.r[i];
        }
        dim3 grid((s.B * s.M + 31) / 32 * nrc, a.H);
        hipLaunchKernelGGL(encode_f32_kernel, grid, dim3(256), 0, stream, s, nrc_k, nrc);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
    return hipSuccess;
  }
  const int blocks = (TT + kEncTok - 1) / kEncTok;
  switch (bf16_route(a)) {
    case kFew: {
      dim3 grid(blocks, nrc_k + nrc_v, a.H * a.ksplit);
      hipLaunchKernelGGL(encode_few_kernel, grid, dim3(256), 0, stream, a, nrc_k);
      if (a.ksplit > 1)
        hipLaunchKernelGGL(encode_reduce_kernel, dim3(blocks, nrc_k + nrc_v, a.H), dim3(256), 0, stream, a, nrc_k);
      return hipGetLastError();
    }
    case kStream: {  // ~2 workgroups per CU
      const int per_head = 2 * a.H;
      int wgx = (2 * device_cu_count() + per_head - 1) / per_head;
      if (wgx > blocks) wgx = blocks;
      const int bpw = (blocks + wgx - 1) / wgx;
      dim3 grid((blocks + bpw - 1) / bpw, a.H, 2);
      if (a.K == 512)
        hipLaunchKernelGGL((encode_stream_kernel<16>), grid, dim3(256), 0, stream, a, bpw);
      else
        hipLaunchKernelGGL((encode_stream_kernel<8>), grid, dim3(256), 0, stream, a, bpw);
      return hipGetLastError();
    }
    case kGemm1: return launch_gemm<1>(a, stream);
    case kGemm2: return launch_gemm<2>(a, stream);
    case kTok32: break;
  }
  // One head and two row tiles per workgroup, so that the weights spread over
  // the machine; of 8192 tokens and more (mostly K an odd multiple of 32)
  // all heads of its 32 tokens, one contiguous region of x.
  const int heads_per_wg = blocks >= 256 ? a.H : 1;
  const int rtmax = (rmax + 15) / 16;
  const int rt_per_wg = blocks >= 256 ? (rtmax < 8 ? rtmax : 8) : 2;
  const int nrc = (rtmax + rt_per_wg - 1) / rt_per_wg;
  dim3 grid(blocks, (a.H + heads_per_wg - 1) / heads_per_wg, 2 * nrc);
  hipLaunchKernelGGL(encode_bf16_kernel, grid, dim3(256), 0, stream, a, heads_per_wg, rt_per_wg, nrc);
  return hipGetLastError();
}

}  // namespace lla

// Kernel of a bf16 write (enum Route), and of a GEMM write its heads per
// workgroup and token blocks.
extern "C" int lla_internal_encode_route(int B, int M, int H, int K, int r_k, int r_v, int means, int pos0,
                                         int* heads, int* blocks) {
  lla::EncodeArgs a{};
  a.dtype = LLA_BF16;
  a.B = B;
  a.M = M;
  a.H = H;
  a.K = K;
  a.r[0] = r_k;
  a.r[1] = r_v;
  a.mu[0] = means ? &a : nullptr;
  a.pos0 = pos0;
  const lla::Route route = lla::bf16_route(a);
  *heads = *blocks = 0;
  auto fill = [&](const auto& g) {
    *heads = g.hpw;
    *blocks = g.ntb;
  };
  if (route == lla::kGemm1) fill(lla::GemmGrid<1>(a));
  if (route == lla::kGemm2) fill(lla::GemmGrid<2>(a));
  return route;
}
