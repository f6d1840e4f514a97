// LLA-2D causal prefill at loop l (Sec. 3 "The LLA-2D variant (loop x head)";
// App. J "Per-head LLA versus LLA-2D at inference": either variant may take
// the full-memory path that materialises K/V or attend over the latents).
//
// With one latent per token for all heads the ranks exceed d_head (288 / 480
// against 128 at the 21.33x operating point), so the absorbed form would cost
// 2 (r_k + r_v) flops per causal score, against 2 d_head (r_k + r_v) per key
// and head to rebuild K and V once plus 4 d_head per score to attend over them.
// For a prompt of M new tokens that is about 3x fewer flops from M ~ 128 on,
// so this path rebuilds:
//
//   recon2d_kernel:  K_h = C_k U_{k,h}^T and V_h = C_v U_{v,h}^T (Eq. 3 with the
//                    (l, h) slice of W_up) for every cached token n < p0 + M,
//                    rounded to fp16, into a caller-owned workspace;
//   flash2d_kernel:  causal attention of the M queries of every head over its
//                    rebuilt K_h, V_h (d_head = 128), online softmax over
//                    64-key pages, then out = O / l + mu_v.
//
// mu_k is not added: q . mu_k is the same for every key and cancels in the
// softmax.  mu_v is added to the normalised output (the weights sum to 1).
//
// The attention's products run on fp16 MFMAs (the same rate as bf16 on this
// chip): the bf16 query converts to fp16 exactly, and the rebuilt K and V and
// the softmax weights keep 11 significant bits instead of bf16's 8, so the
// rounding of these intermediates stays well inside the bf16 error budget even
// for peaked rows.  Values beyond fp16's range (65504) become infinite and the
// output is then not finite.
//
// Workspace layouts, chosen so that every MFMA operand of the attention is one
// 16-byte LDS read:
//   kh [B][H][nk][128]            keys token-major (a key's 128 features contiguous)
//   vt [B][H][nk/32][128][32]     values feature-major per 32-key block; inside each
//                                 16-key run the keys are stored in the order
//                                 0-3, 8-11, 4-7, 12-15 (the order in which a
//                                 32x32 accumulator hands its rows to a lane half)
// with nk = p0 + M rounded up to a page; tokens n >= p0 + M are written as 0.

#include "lla_device.h"
#include "lla_internal.h"
#include "../../include/lla.h"

namespace lla {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kD = 128;            // d_head of both kernels
constexpr int kThreads = 256;      // 4 wavefronts
constexpr int kVBlk = 32;          // keys per block of the rebuilt values
constexpr int kRTok = 128;         // tokens per rebuild workgroup (two pages)
constexpr int kQBlock = 256;       // queries per attention workgroup (32 per wavefront)
constexpr int kFThreads = 512;     // attention workgroup: 8 wavefronts
constexpr float kLazy = 8.0f;      // raise the running max only when it grows by more than this (log2)

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f16x8 as_f16x8(uint4 v) { return __builtin_bit_cast(f16x8, v); }
__device__ __forceinline__ f32x16 mfma_h(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
// two fp32 values as bf16 (output) or fp16 (rebuilt K / V), round to nearest even
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return uint32_t(f32_to_bf16(lo)) | (uint32_t(f32_to_bf16(hi)) << 16);
}
__device__ __forceinline__ uint32_t pack2h(float lo, float hi) {
  const _Float16 a = (_Float16)lo, b = (_Float16)hi;
  return uint32_t(__builtin_bit_cast(uint16_t, a)) | (uint32_t(__builtin_bit_cast(uint16_t, b)) << 16);
}
typedef short i16x4 __attribute__((ext_vector_type(4)));
// ds_read_b64_tr_b16: each 16-lane group reads a 16 x 4 block of 16-bit values
// (lane L: 4 consecutive elements at its address) and lane L receives element
// L % 4 of the lanes 4 e + L / 4, e = 0..3
__device__ __forceinline__ uint2 lds_tr16(const bf16_t* p) {
  return __builtin_bit_cast(uint2,
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p)));
}

// max over both halves of the wavefront (lane i and lane i ^ 32)
__device__ __forceinline__ float half_swap_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The running maximum m of a query once a block's largest score is m + mx, an
// fp16 value (the score product subtracts it as an operand).  A wavefront may
// meet keys far below the query's others first: m stays finite below fp16's range
// (their weights are 0 either way), and where fp16 values are 32 apart a maximum
// halfway is not rounded down, which would make its weight 2^16, infinity in fp16.
__device__ __forceinline__ float raised_max(float m, float mx) {
  const float x = m + mx;
  float r = fmaxf((float)(_Float16)x, -65504.f);
  if (x - r >= 16.f) r += 32.f;
  return r;
}

// ---------------------------------------------------------------------------
// Rebuild.  One workgroup = 128 tokens of one sequence and a run of heads (all of
// them for a long prompt): the latent tile is staged once in LDS token-major (a token's r features contiguous) and
// wavefront w computes features 32w .. 32w + 31 of every head, with that
// head's up-projection rows as the other operand (16-byte loads).
//   keys:   D = K^T (M = feature, N = token, K = latent feature j), so a lane
//           holds 4-feature runs of one token (8-byte stores);
//   values: D = V (M = token, N = feature), so a lane holds the tokens
//           16 b + 8 g .. + 7 of the permuted order of one feature (16-byte stores).
// ---------------------------------------------------------------------------
template <int N>
struct IntC {
  static constexpr int value = N;
};

// Feature-major pages (the values; the per-head caches below) are staged as
// they are, 16-byte chunks of 8 tokens of one feature, with the chunk index of
// rows 4k+2, 4k+3 XORed with 4; ds_read_b64_tr_b16 then hands each lane one
// token's 4 consecutive features, the MFMA operand layout.  Both the staging
// stores and the transposed reads are free of bank conflicts.  (The keys are
// token-major already and are staged row by row.)
template <int AXIS, int KS>  // AXIS 0: keys, 1: values; KS = r / 16
__global__ __launch_bounds__(kThreads) void recon2d_kernel(Prefill2dArgs a) {
  constexpr int R = KS * 16;
  constexpr int TOK = kRTok;           // tokens per workgroup
  constexpr bool FM = AXIS == 1;       // the latents arrive as feature-major pages
  constexpr int CS = R + 8;  // token-major LDS row stride (bf16): 16-byte reads of 16 rows hit distinct banks
  constexpr int LDS = FM ? (TOK / kPage) * R * kPage : TOK * CS;
  __shared__ __attribute__((aligned(16))) bf16_t s_c[LDS];

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 31, g = lane >> 5;
  const int b = blockIdx.y, n0 = blockIdx.x * TOK;
  const int nvalid = a.p0 + a.M;  // tokens that hold latents; the rest are rebuilt as 0
  const int H = a.H;
  constexpr int rr = R;  // the cache's rank (row pitch of its pages)

  // ---- latent tile, zero past nvalid (and past rr) ----
  if constexpr (!FM) {
    const bf16_t* src = static_cast<const bf16_t*>(a.ck) + (size_t)b * a.n_max * R;
    constexpr int C8 = R / 8;
    for (int e = tid; e < TOK * C8; e += kThreads) {
      const int n = e / C8, c8 = e - n * C8;
      const uint4 v = n0 + n < nvalid ? ld16(src + (size_t)(n0 + n) * R + 8 * c8) : make_uint4(0, 0, 0, 0);
      *reinterpret_cast<uint4*>(&s_c[n * CS + 8 * c8]) = v;
    }
  } else {
    // chunk e: page pg, feature row j, 8-token chunk c (consecutive e are
    // consecutive 16 bytes of the cache)
    const bf16_t* src = static_cast<const bf16_t*>(a.cv) + (size_t)b * a.n_max * rr;
    for (int e = tid; e < TOK / kPage * R * 8; e += kThreads) {
      const int pg = e / (R * 8), rem = e - pg * (R * 8), j = rem >> 3, c = rem & 7;
      const int nb = n0 + pg * kPage + 8 * c;  // first token of the chunk
      uint4 v = make_uint4(0, 0, 0, 0);
      if (nb < nvalid && j < rr) {
        v = ld16(src + (size_t)(n0 / kPage + pg) * kPage * rr + (size_t)j * kPage + 8 * c);
        const int nv = nvalid - nb;  // tokens of the chunk that hold latents
        if (nv < 8) {
          auto keep = [nv](int i) { return nv > 2 * i + 1 ? 0xffffffffu : nv > 2 * i ? 0x0000ffffu : 0u; };
          v.x &= keep(0);
          v.y &= keep(1);
          v.z &= keep(2);
          v.w &= keep(3);
        }
      }
      *reinterpret_cast<uint4*>(&s_c[(pg * R + j) * kPage + ((c ^ (((j >> 1) & 1) << 2)) << 3)]) = v;
    }
  }
  __syncthreads();

  // The latent operand of K-step s for 32-token tile nt: lane (col, g) gets
  // features 16 s + 8 g .. + 7 of token 32 nt + col.  Transposed reads: lane
  // (x16, th) of a 16-lane group addresses feature row 16 s + 8 g + x16 / 4
  // (+ 4 for the second read) and tokens 16 th + 4 (x16 % 4) .. + 3 of its tile.
  const int x16 = lane & 15, th = (lane >> 4) & 1, sw1 = (x16 >> 3) & 1;
  const int troff = (8 * g + (x16 >> 2)) * kPage + ((2 * th + ((x16 & 3) >> 1)) << 3) + 4 * (x16 & 1);
  auto lat_op = [&](int nt, int s) -> bf16x8 {
    if constexpr (!FM) {
      return as_bf16x8(*reinterpret_cast<const uint4*>(&s_c[(32 * nt + col) * CS + 16 * s + 8 * g]));
    } else {
      const bf16_t* p = s_c + (nt >> 1) * R * kPage + troff + ((4 * ((nt & 1) ^ sw1)) << 3) + 16 * s * kPage;
      const uint2 r0 = lds_tr16(p), r1 = lds_tr16(p + 4 * kPage);
      return as_bf16x8(make_uint4(r0.x, r0.y, r1.x, r1.y));
    }
  };

  const bf16_t* U = static_cast<const bf16_t*>(AXIS == 0 ? a.uk : a.uv);
  const int ntile = min(TOK, a.nk - n0) / 32;  // 32-token tiles of this workgroup inside nk
  // up-projection rows 32 wave + col of head h as K-step operands
  auto load_u = [&](int h, uint4 (&u)[KS]) {
    const bf16_t* row = U + ((size_t)h * kD + 32 * wave + col) * R + 8 * g;
#pragma unroll
    for (int s = 0; s < KS; ++s) u[s] = ld16(row + 16 * s);
  };
  uint4 ua[KS];
  // NT = the workgroup's token tiles, a compile-time count so the product loop
  // has no branches (a guard per product had split every MFMA into a block of
  // its own, each waiting on its own LDS read)
  auto head = [&](int h, const uint4 (&u)[KS], auto ntc) {
    constexpr int NT = decltype(ntc)::value;
    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x16{0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const bf16x8 c = lat_op(nt, s);
        acc[nt] = AXIS == 0 ? mfma(as_bf16x8(u[s]), c, acc[nt]) : mfma(c, as_bf16x8(u[s]), acc[nt]);
      }
    }
    const size_t bh = (size_t)b * H + h;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (AXIS == 0) {
        // lane (token col, half g), register r: feature 32 wave + 8 (r/4) + 4 g + r%4
        uint16_t* dst = static_cast<uint16_t*>(a.kh) + (bh * a.nk + n0 + 32 * nt + col) * kD + 32 * wave + 4 * g;
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4)
          *reinterpret_cast<uint2*>(dst + 8 * c4) =
              make_uint2(pack2h(acc[nt][4 * c4], acc[nt][4 * c4 + 1]), pack2h(acc[nt][4 * c4 + 2], acc[nt][4 * c4 + 3]));
      } else {
        // lane (feature col, half g), registers 8 blk .. 8 blk + 7: tokens at
        // permuted positions 16 blk + 8 g .. + 7 of the tile's 32
        const int tok0 = n0 + 32 * nt;
        uint16_t* dst = static_cast<uint16_t*>(a.vt) +
                      ((bh * (a.nk / kVBlk) + tok0 / kVBlk) * kD + 32 * wave + col) * kVBlk + 8 * g;
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
          const f32x16& x = acc[nt];
          const int r0 = 8 * blk;
          *reinterpret_cast<uint4*>(dst + 16 * blk) =
              make_uint4(pack2h(x[r0], x[r0 + 1]), pack2h(x[r0 + 2], x[r0 + 3]), pack2h(x[r0 + 4], x[r0 + 5]),
                         pack2h(x[r0 + 6], x[r0 + 7]));
        }
      }
    }
  };
  // every operand load of a head is issued before its first product, so the
  // products of the early K-steps overlap the later loads
  for (int h = blockIdx.z * a.hpw; h < min(H, (int)(blockIdx.z + 1) * a.hpw); ++h) {
    load_u(h, ua);
    switch (ntile) {  // uniform; 2 or 4 (the key count is a multiple of 64)
      case 4: head(h, ua, IntC<4>{}); break;
      case 2: head(h, ua, IntC<2>{}); break;
      default: break;
    }
  }
}

// ---------------------------------------------------------------------------
// Per-head rebuild over a run of pages.  One workgroup = one (b, h) and up to
// `ppw` consecutive 64-token pages: the head's up-projection rows are loaded
// into registers once, and while one page's products run from LDS the next
// page's latents are already in flight into registers.  Staging, operand
// reads (ds_read_b64_tr_b16) and outputs are those of the per-head
// recon2d_kernel above.
// ---------------------------------------------------------------------------
// KS: K-steps of 16 features; BOTH: of the larger rank, and the other axis skips
// the steps past its own rank in groups of 4.
constexpr int kBothSteps = 20;  // largest K-step count of the launch of both axes
template <int AXIS, int KS, bool BOTH>
__device__ __forceinline__ void recon_ph_body(const Prefill2dArgs& a, int ppw, bf16_t* s_c) {
  constexpr int CPT = (KS * 16 * 8 + kThreads - 1) / kThreads;  // 16-byte chunks of a page per thread

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 31, g = lane >> 5;
  const int bh = blockIdx.y, h = bh % a.H;
  const int nvalid = a.p0 + a.M;
  const int rr = AXIS == 0 ? a.rk : a.rv;
  const int R = BOTH ? min((rr + 63) / 64 * 64, KS * 16) : KS * 16;  // staged features (zero past rr)
  const int pg0 = blockIdx.x * ppw, pg1 = min(pg0 + ppw, a.nk / kPage);
  const bf16_t* src = static_cast<const bf16_t*>(AXIS == 0 ? a.ck : a.cv) + (size_t)bh * a.n_max * rr;

  // this thread's chunks of a page: chunk e = tid + 256 i is feature row e / 8,
  // tokens 8 (e % 8) .. + 7
  uint4 stg[CPT];
  auto gload = [&](int pg) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int e = tid + i * kThreads, j = e >> 3, c = e & 7;
      const int nb = pg * kPage + 8 * c;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (e < R * 8 && j < rr && nb < nvalid) {
        v = ld16(src + (size_t)pg * kPage * rr + (size_t)j * kPage + 8 * c);
        const int nv = nvalid - nb;
        if (nv < 8) {
          auto keep = [nv](int q) { return nv > 2 * q + 1 ? 0xffffffffu : nv > 2 * q ? 0x0000ffffu : 0u; };
          v.x &= keep(0);
          v.y &= keep(1);
          v.z &= keep(2);
          v.w &= keep(3);
        }
      }
      stg[i] = v;
    }
  };
  auto lstore = [&]() {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int e = tid + i * kThreads, j = e >> 3, c = e & 7;
      if (e < R * 8) *reinterpret_cast<uint4*>(&s_c[j * kPage + ((c ^ (((j >> 1) & 1) << 2)) << 3)]) = stg[i];
    }
  };
  const int x16 = lane & 15, th = (lane >> 4) & 1, sw1 = (x16 >> 3) & 1;
  const int troff = (8 * g + (x16 >> 2)) * kPage + ((2 * th + ((x16 & 3) >> 1)) << 3) + 4 * (x16 & 1);
  auto lat_op = [&](int nt, int s) -> bf16x8 {  // token tile nt (0, 1) of the staged page
    const bf16_t* p = s_c + troff + ((4 * (nt ^ sw1)) << 3) + 16 * s * kPage;
    const uint2 r0 = lds_tr16(p), r1 = lds_tr16(p + 4 * kPage);
    return as_bf16x8(make_uint4(r0.x, r0.y, r1.x, r1.y));
  };
  // up-projection rows 32 wave + col of head h (features past rr are zero)
  uint4 ua[KS];
  {
    const bf16_t* row = static_cast<const bf16_t*>(AXIS == 0 ? a.uk : a.uv) + ((size_t)h * kD + 32 * wave + col) * rr + 8 * g;
#pragma unroll
    for (int s = 0; s < KS; ++s) ua[s] = 16 * s + 8 * g < rr ? ld16(row + 16 * s) : make_uint4(0, 0, 0, 0);
  }
  if (pg0 < pg1) gload(pg0);
  for (int pg = pg0; pg < pg1; ++pg) {
    lstore();
    __syncthreads();
    if (pg + 1 < pg1) gload(pg + 1);  // in flight during this page's products
    f32x16 acc[2] = {f32x16{0.f}, f32x16{0.f}};
#pragma unroll
    for (int s0 = 0; s0 < KS; s0 += 4) {
      if (16 * s0 >= R) break;  // uniform
#pragma unroll
      for (int s = s0; s < (s0 + 4 < KS ? s0 + 4 : KS); ++s)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const bf16x8 c = lat_op(nt, s);
          acc[nt] = AXIS == 0 ? mfma(as_bf16x8(ua[s]), c, acc[nt]) : mfma(c, as_bf16x8(ua[s]), acc[nt]);
        }
    }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int tok0 = pg * kPage + 32 * nt;
      if (AXIS == 0) {
        // lane (token col, half g), register r: feature 32 wave + 8 (r/4) + 4 g + r%4
        uint16_t* dst = static_cast<uint16_t*>(a.kh) + ((size_t)bh * a.nk + tok0 + col) * kD + 32 * wave + 4 * g;
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4)
          *reinterpret_cast<uint2*>(dst + 8 * c4) =
              make_uint2(pack2h(acc[nt][4 * c4], acc[nt][4 * c4 + 1]), pack2h(acc[nt][4 * c4 + 2], acc[nt][4 * c4 + 3]));
      } else {
        // lane (feature col, half g), registers 8 blk .. + 7: tokens at permuted
        // positions 16 blk + 8 g .. + 7 of the tile
        uint16_t* dst = static_cast<uint16_t*>(a.vt) +
                        (((size_t)bh * (a.nk / kVBlk) + 2 * pg + nt) * kD + 32 * wave + col) * kVBlk + 8 * g;
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
          const f32x16& x = acc[nt];
          const int r0 = 8 * blk;
          *reinterpret_cast<uint4*>(dst + 16 * blk) =
              make_uint4(pack2h(x[r0], x[r0 + 1]), pack2h(x[r0 + 2], x[r0 + 3]), pack2h(x[r0 + 4], x[r0 + 5]),
                         pack2h(x[r0 + 6], x[r0 + 7]));
        }
      }
    }
    __syncthreads();  // the page's LDS tile is read by every wavefront before the next is stored
  }
}

// AXIS 0 or 1: one axis; 2: both in one launch (blockIdx.z).  With few pages a
// workgroup's chain of dependent steps (latents, LDS, products, stores) is longer
// than its share of the machine's work, so the axes overlap.
template <int AXIS, int KS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void recon_ph_kernel(Prefill2dArgs a, int ppw) {
  __shared__ __attribute__((aligned(16))) bf16_t s_c[KS * 16 * kPage];
  if (AXIS == 0 || (AXIS == 2 && blockIdx.z == 0))
    recon_ph_body<0, KS, AXIS == 2>(a, ppw, s_c);
  else
    recon_ph_body<1, KS, AXIS == 2>(a, ppw, s_c);
}

// ---------------------------------------------------------------------------
// Attention.  One workgroup = 8 wavefronts x 32 queries of one (b, h); keys in
// 64-token pages staged in LDS (K token-major, V feature-major) once for the 8
// wavefronts, two pages in flight in registers.  Products (v_mfma_f32_32x32x16_f16), transposed so each
// accumulator feeds the next product with no lane exchange:
//   S^T  (M = key, N = query, K = feature): A = K tile rows,  B = the query (registers)
//   O^T += (M = feature, N = query, K = key): A = V^T tile rows, B = P from S^T
// A 32x32 accumulator gives lane (q + 32 g), register r the row 8(r/4) + 4g + r%4
// of column q: registers 8u .. 8u + 7 of a key tile are the keys
// 16u + 8(e/4) + 4g + e%4, e < 8, which the permuted V^T rows hold contiguously.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kFThreads) __attribute__((amdgpu_waves_per_eu(2)))
void flash2d_kernel(Prefill2dArgs a) {
  constexpr int KS = kD / 16;       // K-steps of the score product
  constexpr int KST = kD + 8;       // K tile row stride (fp16 elements)
  constexpr int VST = kPage + 8;    // V^T tile row stride (fp16 elements)
  constexpr int KTILE = kPage * KST, VTILE = kD * VST;
  constexpr int CH = kPage * kD / 8 / kFThreads;  // 16-byte chunks per thread per page and axis (2)
  __shared__ __attribute__((aligned(16))) uint16_t s_k[2 * KTILE];  // fp16
  __shared__ __attribute__((aligned(16))) uint16_t s_v[2 * VTILE];

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 31, g = lane >> 5;
  const int bh = blockIdx.x, h = bh % a.H;
  const int M = a.M, p0 = a.p0;
  const int nqb = (M + kQBlock - 1) / kQBlock;
  const int qb = nqb - 1 - (int)blockIdx.y;  // heaviest (latest) query blocks first
  const int q0 = qb * kQBlock, qw0 = q0 + 32 * wave;
  const int myq = qw0 + col;
  const bool q_ok = myq < M, wave_live = qw0 < M;
  const int qlast_w = min(qw0 + 31, M - 1);
  const int kmax = p0 + min(q0 + kQBlock, M);  // keys [0, kmax) matter to the workgroup
  const int npages = (kmax + kPage - 1) / kPage;

  // ---- page staging: both pages are 16 KB contiguous in the workspace ----
  const uint16_t* kbase = static_cast<const uint16_t*>(a.kh) + (size_t)bh * a.nk * kD;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.vt) + (size_t)bh * a.nk * kD;
  uint4 stk[2][CH], stv[2][CH];
  auto load_page = [&](int pg, int set) {
    const uint16_t* kp = kbase + (size_t)pg * kPage * kD;
    const uint16_t* vp = vbase + (size_t)pg * kPage * kD;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      stk[set][c] = ld16(kp + 8 * (tid + c * kFThreads));
      stv[set][c] = ld16(vp + 8 * (tid + c * kFThreads));
    }
  };
  auto store_page = [&](int set, int buf) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int ch = tid + c * kFThreads;
      *reinterpret_cast<uint4*>(&s_k[buf * KTILE + (ch >> 4) * KST + 8 * (ch & 15)]) = stk[set][c];
      // value chunk ch: block ch / 512, feature (ch / 4) % 128, keys 8 (ch % 4) .. + 7 of the block
      *reinterpret_cast<uint4*>(&s_v[buf * VTILE + ((ch >> 2) & (kD - 1)) * VST + kVBlk * (ch >> 9) + 8 * (ch & 3)]) =
          stv[set][c];
    }
  };

  load_page(0, 0);
  load_page(min(1, npages - 1), 1);
  // the query as the score product's B operand: lane (q, g), K-step s = features
  // 16s + 8g .. + 7, scaled by scale * log2(e) and rounded to fp16, so the score
  // product yields base-2 logits
  const float qs = a.qscale;
  f16x8 qop[KS];
  {
    const bf16_t* qrow = static_cast<const bf16_t*>(a.q) + ((size_t)bh * M + (q_ok ? myq : 0)) * kD + 8 * g;
    uint4 raw[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = ld16(qrow + 16 * s);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float x[8];
      Elem<bf16_t>::unpack(raw[s], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) qop[s][e] = (_Float16)(x[e] * qs);
    }
  }
  // One more K-step carries the running max: A holds 1 in feature 0 for every
  // key, B holds -m in feature 0 for the lane's query, so the score products
  // yield s - m directly.  m is kept representable in fp16 (every raise rounds
  // it), which makes the shift exact and the rescale exp2(m_old - m_new) exact.
  const f16x8 a_one = {(_Float16)(g == 0 ? 1.f : 0.f), 0, 0, 0, 0, 0, 0, 0};
  store_page(0, 0);
  __syncthreads();

  f32x16 oacc[kD / 32];
#pragma unroll
  for (int t = 0; t < kD / 32; ++t) oacc[t] = f32x16{0.f};
  float m_run = 0.f, l_lane = 0.f;  // the first page always raises m
  const int qpos = p0 + myq;

  auto page = [&](int p, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    // set buf held page p (already in LDS); page p + 2 goes into it (near the
    // end the last page is re-read, so every wait is for exactly one page)
    load_page(min(p + 2, npages - 1), buf);
    const int key0 = p * kPage;
    if (wave_live && key0 <= p0 + qlast_w) {
      const bool diag = key0 + kPage - 1 > p0 + qw0;
      const uint16_t* kt_row = s_k + buf * KTILE + col * KST + 8 * g;
      const uint16_t* vt_row = s_v + buf * VTILE + col * VST + 8 * g;
      // all of the page's operand fragments are read from LDS ahead of their
      // products (scheduling fences keep them there): the 16 K fragments before
      // the score products, which then issue back to back, and the 16 V fragments
      // right after them, so the value reads overlap the score products and the
      // softmax (1.314 -> 1.281 ms per call on 4 x 8192 tokens, 16 heads)
      uint4 kop[KS][2];
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) kop[s][kt] = *reinterpret_cast<const uint4*>(kt_row + 32 * kt * KST + 16 * s);
      __builtin_amdgcn_sched_barrier(0);
      const f16x8 b_m = {(_Float16)(g == 0 ? -m_run : 0.f), 0, 0, 0, 0, 0, 0, 0};
      f32x16 sc[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) sc[kt] = mfma_h(a_one, b_m, f32x16{0.f});
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) sc[kt] = mfma_h(as_f16x8(kop[s][kt]), qop[s], sc[kt]);
      uint4 vop[2][kD / 32][2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int t = 0; t < kD / 32; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            vop[kt][t][u] = *reinterpret_cast<const uint4*>(vt_row + 32 * t * VST + 32 * kt + 16 * u);
      __builtin_amdgcn_sched_barrier(0);
      const int lim = qpos - key0 - 4 * g;
      if (__builtin_expect(diag, 0)) {
        // key 32kt + 8(r/4) + 4g + r%4 of the page is visible iff 32kt + 8(r/4) + r%4 <= lim
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (32 * kt + 8 * (r / 4) + (r % 4) > lim) sc[kt][r] = neg_inf();
      }
      // page maximum of the lane's query: four max3 chains, then the other lane half
      float m0 = fmaxf(fmaxf(sc[0][0], sc[0][1]), sc[0][2]), m1 = fmaxf(fmaxf(sc[0][8], sc[0][9]), sc[0][10]);
      float m2 = fmaxf(fmaxf(sc[1][0], sc[1][1]), sc[1][2]), m3 = fmaxf(fmaxf(sc[1][8], sc[1][9]), sc[1][10]);
#pragma unroll
      for (int r = 3; r < 7; r += 2) {
        m0 = fmaxf(fmaxf(m0, sc[0][r]), sc[0][r + 1]);
        m1 = fmaxf(fmaxf(m1, sc[0][8 + r]), sc[0][9 + r]);
        m2 = fmaxf(fmaxf(m2, sc[1][r]), sc[1][r + 1]);
        m3 = fmaxf(fmaxf(m3, sc[1][8 + r]), sc[1][9 + r]);
      }
      m0 = fmaxf(fmaxf(m0, sc[0][7]), fmaxf(m1, sc[0][15]));
      m2 = fmaxf(fmaxf(m2, sc[1][7]), fmaxf(m3, sc[1][15]));
      const float mx = half_swap_max(fmaxf(m0, m2));  // page max of s - m
      // raise the running max on the first page, then only when a score
      // exceeds it by more than 2^kLazy (the weights stay below 2^kLazy)
      const bool raise = mx > kLazy || p == 0;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
        if (raise) {
          const float m_new = raised_max(m_run, mx);
          const float delta = m_new - m_run;  // exact: both are fp16 values
          const float alpha = p == 0 ? 0.f : __builtin_amdgcn_exp2f(-delta);
#pragma unroll
          for (int t = 0; t < kD / 32; ++t) oacc[t] *= alpha;
          l_lane *= alpha;
#pragma unroll
          for (int kt = 0; kt < 2; ++kt) sc[kt] -= delta;
          m_run = m_new;
        }
      }
      // one branch-free block: the second half's exponentials can issue
      // between the first half's value products
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        f16x8 pop[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            pop[u][e] = (_Float16)__builtin_amdgcn_exp2f(sc[kt][8 * u + e]);  // exp2(-inf) = 0
        // the normaliser sums the fp16 weights the value product uses, two per
        // v_dot2_f32_f16 against (1, 1) with fp32 accumulation
        const f16x2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 8; e += 2)
            l_lane = __builtin_amdgcn_fdot2(f16x2{pop[u][e], pop[u][e + 1]}, ones, l_lane, false);
#pragma unroll
        for (int t = 0; t < kD / 32; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            oacc[t] = mfma_h(as_f16x8(vop[kt][t][u]), pop[u], oacc[t]);
      }
    }
    if (p + 1 < npages) store_page(buf ^ 1, buf ^ 1);
    __syncthreads();
  };
  for (int p = 0; p < npages; p += 2) {
    page(p, IntC<0>{});
    if (p + 1 < npages) page(p + 1, IntC<1>{});
  }

  // ---- epilogue: out = O / l + mu_v ----
  if (!wave_live) return;
  const float inv_l = 1.0f / half_swap_sum(l_lane);
  const bf16_t* muv = a.muv ? static_cast<const bf16_t*>(a.muv) + (size_t)h * kD : nullptr;
  const size_t orow = ((size_t)bh * M + myq) * kD;
  if (!q_ok) return;
#pragma unroll
  for (int t = 0; t < kD / 32; ++t) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i0 = 32 * t + 8 * c + 4 * g;
      const uint2 mw = muv ? *reinterpret_cast<const uint2*>(muv + i0) : make_uint2(0, 0);
      const float v0 = fmaf(oacc[t][4 * c + 0], inv_l, bf16_lo(mw.x));
      const float v1 = fmaf(oacc[t][4 * c + 1], inv_l, bf16_hi(mw.x));
      const float v2 = fmaf(oacc[t][4 * c + 2], inv_l, bf16_lo(mw.y));
      const float v3 = fmaf(oacc[t][4 * c + 3], inv_l, bf16_hi(mw.y));
      if (a.out_dtype == LLA_F32)
        *reinterpret_cast<float4*>(static_cast<float*>(a.out) + orow + i0) = make_float4(v0, v1, v2, v3);
      else
        *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.out) + orow + i0) = make_uint2(pack2(v0, v1), pack2(v2, v3));
    }
  }
}

// ---------------------------------------------------------------------------
// Attention for calls with few query blocks (a chunk appended to a longer
// context).  One workgroup = 32 queries of one (b, h); its 8 wavefronts split
// the keys instead of the queries: wavefront w takes the 32-key blocks w, w + 8,
// ... and their (m, l, O) are combined through LDS at the end, so a call has
// eight times the workgroups of flash2d_kernel.  No key block is shared between
// wavefronts: each stages its own (8 KB of keys, 8 KB of values, whole lines;
// operands loaded straight from memory touch 32 bytes of every row and ran 4 us
// per block) in its own LDS, with the next block in flight in registers, so the
// key loop has no barrier.  Products and the fp16 running max are
// flash2d_kernel's.
// ---------------------------------------------------------------------------
constexpr int kSQ = 32;  // queries per workgroup
constexpr int kSK = 32;  // keys per block
static_assert(kSK == kVBlk, "a block of values is contiguous");
__global__ __launch_bounds__(kFThreads) __attribute__((amdgpu_waves_per_eu(2)))
void flash2d_split_kernel(Prefill2dArgs a) {
  constexpr int KS = kD / 16;
  constexpr int NW = kFThreads / kWave;
  constexpr int BLK = kSK * kD;         // elements of a staged block and axis
  constexpr int CH = BLK / 8 / kWave;   // 16-byte chunks per lane and axis (8)
  // each wavefront's key and value block, then its accumulators [register][lane]
  __shared__ __attribute__((aligned(16))) uint16_t s_kv[NW][2 * BLK];
  __shared__ float s_m[NW][kSQ], s_l[NW][kSQ];
  static_assert(2 * BLK * sizeof(uint16_t) == kD / 2 * kWave * sizeof(float), "");

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 31, g = lane >> 5;
  const int bh = blockIdx.x, h = bh % a.H;
  const int M = a.M, p0 = a.p0;
  const int nqb = (M + kSQ - 1) / kSQ;
  const int q0 = (nqb - 1 - (int)blockIdx.y) * kSQ;  // heaviest (latest) query blocks first
  const int myq = q0 + col;
  const bool q_ok = myq < M;
  const int kmax = p0 + min(q0 + kSQ, M);  // keys [0, kmax) matter to the workgroup
  const int nblk = (kmax + kSK - 1) / kSK;

  // Block j (keys 32 j .. + 31) is 8 KB contiguous per axis.  In LDS the 16-byte
  // chunks of key row r (16 of them) are XORed with r % 16 and those of value
  // row f (4) with (f / 4) % 4: 16-byte reads of 16 rows hit distinct banks.
  const uint16_t* kbase = static_cast<const uint16_t*>(a.kh) + (size_t)bh * a.nk * kD + 8 * lane;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.vt) + (size_t)bh * a.nk * kD + 8 * lane;
  uint16_t* const sk = s_kv[wave];
  uint16_t* const sv = s_kv[wave] + BLK;
  uint4 pk[CH], pv[CH];
  auto load = [&](int j) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      pk[c] = ld16(kbase + (size_t)j * BLK + c * 8 * kWave);
      pv[c] = ld16(vbase + (size_t)j * BLK + c * 8 * kWave);
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int kr = 4 * c + (lane >> 4), vr = 16 * c + (lane >> 2);
      *reinterpret_cast<uint4*>(sk + kr * kD + (((lane & 15) ^ (kr & 15)) << 3)) = pk[c];
      *reinterpret_cast<uint4*>(sv + vr * kVBlk + (((lane & 3) ^ ((vr >> 2) & 3)) << 3)) = pv[c];
    }
  };
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  if (wave < nblk) load(wave);

  const float qs = a.qscale;
  f16x8 qop[KS];
  {
    const bf16_t* qrow = static_cast<const bf16_t*>(a.q) + ((size_t)bh * M + (q_ok ? myq : 0)) * kD + 8 * g;
    uint4 raw[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = ld16(qrow + 16 * s);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float x[8];
      Elem<bf16_t>::unpack(raw[s], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) qop[s][e] = (_Float16)(x[e] * qs);
    }
  }
  const f16x8 a_one = {(_Float16)(g == 0 ? 1.f : 0.f), 0, 0, 0, 0, 0, 0, 0};

  f32x16 oacc[kD / 32];
#pragma unroll
  for (int t = 0; t < kD / 32; ++t) oacc[t] = f32x16{0.f};
  // seen: this lane's query has attended a key of this wavefront's blocks (a
  // diagonal block may hold none); m is raised at the first one
  float m_run = 0.f, l_lane = 0.f;
  bool seen = false;
  const int qpos = p0 + myq;
  for (int j = wave; j < nblk; j += NW) {
    store();
    wave_sync();
    if (j + NW < nblk) load(j + NW);
    uint4 kop[KS], vop[kD / 32][2];
#pragma unroll
    for (int s = 0; s < KS; ++s)
      kop[s] = *reinterpret_cast<const uint4*>(sk + col * kD + (((2 * s + g) ^ (col & 15)) << 3));
    const f16x8 b_m = {(_Float16)(g == 0 ? -m_run : 0.f), 0, 0, 0, 0, 0, 0, 0};
    f32x16 sc = mfma_h(a_one, b_m, f32x16{0.f});
#pragma unroll
    for (int s = 0; s < KS; ++s) sc = mfma_h(as_f16x8(kop[s]), qop[s], sc);
#pragma unroll
    for (int t = 0; t < kD / 32; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        vop[t][u] = *reinterpret_cast<const uint4*>(sv + (32 * t + col) * kVBlk + (((2 * u + g) ^ ((col >> 2) & 3)) << 3));
    __builtin_amdgcn_sched_barrier(0);
    const int key0 = j * kSK;
    if (__builtin_expect(key0 + kSK - 1 > p0 + q0, 0)) {
      // key 8(r/4) + 4g + r%4 of the block is visible iff 8(r/4) + r%4 <= lim
      const int lim = qpos - key0 - 4 * g;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r / 4) + (r % 4) > lim) sc[r] = neg_inf();
    }
    float m0 = fmaxf(fmaxf(sc[0], sc[1]), sc[2]), m1 = fmaxf(fmaxf(sc[8], sc[9]), sc[10]);
#pragma unroll
    for (int r = 3; r < 7; r += 2) {
      m0 = fmaxf(fmaxf(m0, sc[r]), sc[r + 1]);
      m1 = fmaxf(fmaxf(m1, sc[8 + r]), sc[9 + r]);
    }
    const float mx = half_swap_max(fmaxf(fmaxf(m0, sc[7]), fmaxf(m1, sc[15])));
    const bool raise = mx > kLazy || (!seen && mx > neg_inf());
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
      if (raise) {
        const float m_new = raised_max(m_run, mx);
        const float delta = m_new - m_run;  // exact: both are fp16 values
        const float alpha = seen ? __builtin_amdgcn_exp2f(-delta) : 0.f;
#pragma unroll
        for (int t = 0; t < kD / 32; ++t) oacc[t] *= alpha;
        l_lane *= alpha;
        sc -= delta;
        m_run = m_new;
        seen = true;
      }
    }
    f16x8 pop[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) pop[u][e] = (_Float16)__builtin_amdgcn_exp2f(sc[8 * u + e]);
    const f16x2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; e += 2)
        l_lane = __builtin_amdgcn_fdot2(f16x2{pop[u][e], pop[u][e + 1]}, ones, l_lane, false);
#pragma unroll
    for (int t = 0; t < kD / 32; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u) oacc[t] = mfma_h(as_f16x8(vop[t][u]), pop[u], oacc[t]);
    wave_sync();  // the block's LDS reads are done before the next one is stored
  }

  // ---- combine the wavefronts: wavefront w finishes registers 8 w .. 8 w + 7 ----
  float* const s_o = reinterpret_cast<float*>(s_kv);  // [wave][register][lane]
#pragma unroll
  for (int t = 0; t < kD / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) s_o[(wave * (kD / 2) + 16 * t + r) * kWave + lane] = oacc[t][r];
  l_lane = half_swap_sum(l_lane);
  if (g == 0) {
    s_m[wave][col] = seen ? m_run : neg_inf();
    s_l[wave][col] = l_lane;
  }
  __syncthreads();
  float mm = neg_inf(), l = 0.f, wt[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) mm = fmaxf(mm, s_m[w][col]);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wt[w] = __builtin_amdgcn_exp2f(s_m[w][col] - mm);  // 0 for a wavefront that saw no key
    l = fmaf(wt[w], s_l[w][col], l);
  }
  if (!q_ok) return;
  const float inv_l = 1.0f / l;
  const bf16_t* muv = a.muv ? static_cast<const bf16_t*>(a.muv) + (size_t)h * kD : nullptr;
  const size_t orow = ((size_t)bh * M + myq) * kD;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int r0 = 8 * wave + 4 * c;  // tile r0 / 16, registers r0 % 16 ..: 4 consecutive features
    const int i0 = 32 * (wave >> 1) + 8 * ((r0 & 15) >> 2) + 4 * g;
    float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(wt[w], s_o[(w * (kD / 2) + r0 + e) * kWave + lane], o[e]);
    const uint2 mw = muv ? *reinterpret_cast<const uint2*>(muv + i0) : make_uint2(0, 0);
    const float v0 = fmaf(o[0], inv_l, bf16_lo(mw.x)), v1 = fmaf(o[1], inv_l, bf16_hi(mw.x));
    const float v2 = fmaf(o[2], inv_l, bf16_lo(mw.y)), v3 = fmaf(o[3], inv_l, bf16_hi(mw.y));
    if (a.out_dtype == LLA_F32)
      *reinterpret_cast<float4*>(static_cast<float*>(a.out) + orow + i0) = make_float4(v0, v1, v2, v3);
    else
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.out) + orow + i0) = make_uint2(pack2(v0, v1), pack2(v2, v3));
  }
}

// ---------------------------------------------------------------------------
// Attention between the two: 8 / S query groups of 32 by S key streams in a
// workgroup.  128 keys per round are staged for all (K rows and V blocks as
// in flash2d_split_kernel's swizzled layout, double buffered, the next
// round's loads in flight in registers); stream s takes keys 128 / S * s .. of
// every round, and the streams' (m, l, O) are combined through LDS at the end.
// ---------------------------------------------------------------------------
template <int S>
__global__ __launch_bounds__(kFThreads) __attribute__((amdgpu_waves_per_eu(2)))
void flash2d_streams_kernel(Prefill2dArgs a) {
  constexpr int KS = kD / 16;
  constexpr int NW = kFThreads / kWave, QW = NW / S;
  constexpr int RK = 128;                       // keys per round
  constexpr int NT = RK / S / 32;               // 32-key tiles of a stream's share
  constexpr int QB = 32 * QW;                   // queries per workgroup
  constexpr int CH = RK * kD / 8 / kFThreads;   // 16-byte chunks per thread and axis (4)
  constexpr int BUF = 2 * RK * kD;              // elements of one buffer: keys, then values
  __shared__ __attribute__((aligned(16))) uint16_t s_kv[2 * BUF];
  __shared__ float s_m[NW][32], s_l[NW][32];
  static_assert(2 * BUF * sizeof(uint16_t) == NW * kD / 2 * kWave * sizeof(float), "");

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int st = wave % S, qg = wave / S;
  const int col = lane & 31, g = lane >> 5;
  const int bh = blockIdx.x, h = bh % a.H;
  const int M = a.M, p0 = a.p0;
  const int nqb = (M + QB - 1) / QB;
  const int q0 = (nqb - 1 - (int)blockIdx.y) * QB;  // heaviest (latest) query blocks first
  const int qw0 = q0 + 32 * qg, myq = qw0 + col;
  const bool q_ok = myq < M, wave_live = qw0 < M;
  const int qlast_w = min(qw0 + 31, M - 1);
  const int kmax = p0 + min(q0 + QB, M);  // keys [0, kmax) matter to the workgroup
  const int rounds = (kmax + RK - 1) / RK;

  // staging: chunk ch = tid + 512 c: key row ch / 16, or value block ch / 512 and
  // feature (ch / 4) % 128.  The last round may reach past the rebuilt keys: it
  // re-reads the last row or block (masked, like every key past a query).
  const uint16_t* kbase = static_cast<const uint16_t*>(a.kh) + (size_t)bh * a.nk * kD;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.vt) + (size_t)bh * a.nk * kD;
  uint4 pk[CH], pv[CH];
  auto load = [&](int i) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int kr = min(RK * i + 32 * c + (tid >> 4), a.nk - 1);
      const int vb = min(RK / kVBlk * i + c, a.nk / kVBlk - 1);
      pk[c] = ld16(kbase + (size_t)kr * kD + 8 * (tid & 15));
      pv[c] = ld16(vbase + (size_t)vb * kVBlk * kD + 8 * tid);
    }
  };
  const int kst = (tid >> 4) * kD + (((tid & 15) ^ ((tid >> 4) & 15)) << 3);
  const int vst = (tid >> 2) * kVBlk + (((tid & 3) ^ ((tid >> 4) & 3)) << 3);
  auto store = [&](int buf) {
    uint16_t* d = s_kv + buf * BUF;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      *reinterpret_cast<uint4*>(d + 32 * c * kD + kst) = pk[c];
      *reinterpret_cast<uint4*>(d + RK * kD + c * kVBlk * kD + vst) = pv[c];
    }
  };
  load(0);

  const float qs = a.qscale;
  f16x8 qop[KS];
  {
    const bf16_t* qrow = static_cast<const bf16_t*>(a.q) + ((size_t)bh * M + (q_ok ? myq : 0)) * kD + 8 * g;
    uint4 raw[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = ld16(qrow + 16 * s);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float x[8];
      Elem<bf16_t>::unpack(raw[s], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) qop[s][e] = (_Float16)(x[e] * qs);
    }
  }

  f32x16 oacc[kD / 32];
#pragma unroll
  for (int t = 0; t < kD / 32; ++t) oacc[t] = f32x16{0.f};
  float m_run = 0.f, l_lane = 0.f;
  bool seen = false;
  const int qpos = p0 + myq;
  store(0);
  load(min(1, rounds - 1));
  __syncthreads();
  for (int i = 0; i < rounds; ++i) {
    const int buf = i & 1;
    if (i + 1 < rounds) store(buf ^ 1);
    if (i + 2 < rounds) load(i + 2);
    const int key0 = RK * i + 32 * NT * st;
    if (wave_live && key0 <= p0 + qlast_w) {
      const uint16_t* sk = s_kv + buf * BUF + (32 * NT * st + col) * kD;
      const uint16_t* sv = s_kv + buf * BUF + RK * kD + NT * st * kVBlk * kD + col * kVBlk;
      uint4 kop[KS][NT];
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
          kop[s][kt] = *reinterpret_cast<const uint4*>(sk + 32 * kt * kD + (((2 * s + g) ^ (col & 15)) << 3));
      __builtin_amdgcn_sched_barrier(0);
      int gr = g;
      asm volatile("" : "+v"(gr));  // a_one formed here, not held over the rounds (it would spill)
      const f16x8 a_one = {(_Float16)(gr == 0 ? 1.f : 0.f), 0, 0, 0, 0, 0, 0, 0};
      const f16x8 b_m = {(_Float16)(g == 0 ? -m_run : 0.f), 0, 0, 0, 0, 0, 0, 0};
      f32x16 sc[NT];
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) sc[kt] = mfma_h(a_one, b_m, f32x16{0.f});
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) sc[kt] = mfma_h(as_f16x8(kop[s][kt]), qop[s], sc[kt]);
      uint4 vop[NT][kD / 32][2];
#pragma unroll
      for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int t = 0; t < kD / 32; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            vop[kt][t][u] = *reinterpret_cast<const uint4*>(sv + (kt * kD + 32 * t) * kVBlk + (((2 * u + g) ^ ((col >> 2) & 3)) << 3));
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(key0 + 32 * NT - 1 > p0 + qw0, 0)) {
        const int lim = qpos - key0 - 4 * g;
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (32 * kt + 8 * (r / 4) + (r % 4) > lim) sc[kt][r] = neg_inf();
      }
      float mx = neg_inf();
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        float m0 = fmaxf(fmaxf(sc[kt][0], sc[kt][1]), sc[kt][2]), m1 = fmaxf(fmaxf(sc[kt][8], sc[kt][9]), sc[kt][10]);
#pragma unroll
        for (int r = 3; r < 7; r += 2) {
          m0 = fmaxf(fmaxf(m0, sc[kt][r]), sc[kt][r + 1]);
          m1 = fmaxf(fmaxf(m1, sc[kt][8 + r]), sc[kt][9 + r]);
        }
        mx = fmaxf(mx, fmaxf(fmaxf(m0, sc[kt][7]), fmaxf(m1, sc[kt][15])));
      }
      mx = half_swap_max(mx);
      const bool raise = mx > kLazy || (!seen && mx > neg_inf());
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
        if (raise) {
          const float m_new = raised_max(m_run, mx);
          const float delta = m_new - m_run;  // exact: both are fp16 values
          const float alpha = seen ? __builtin_amdgcn_exp2f(-delta) : 0.f;
#pragma unroll
          for (int t = 0; t < kD / 32; ++t) oacc[t] *= alpha;
          l_lane *= alpha;
#pragma unroll
          for (int kt = 0; kt < NT; ++kt) sc[kt] -= delta;
          m_run = m_new;
          seen = true;
        }
      }
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        f16x8 pop[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 8; ++e) pop[u][e] = (_Float16)__builtin_amdgcn_exp2f(sc[kt][8 * u + e]);
        const f16x2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 8; e += 2)
            l_lane = __builtin_amdgcn_fdot2(f16x2{pop[u][e], pop[u][e + 1]}, ones, l_lane, false);
#pragma unroll
        for (int t = 0; t < kD / 32; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u) oacc[t] = mfma_h(as_f16x8(vop[kt][t][u]), pop[u], oacc[t]);
      }
    }
    __syncthreads();
  }

  // ---- combine the streams: wavefront (qg, st) finishes registers 64 / S st .. of its queries ----
  constexpr int RPW = kD / 2 / S;
  float* const s_o = reinterpret_cast<float*>(s_kv);  // [wave][register][lane]
#pragma unroll
  for (int t = 0; t < kD / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) s_o[(wave * (kD / 2) + 16 * t + r) * kWave + lane] = oacc[t][r];
  l_lane = half_swap_sum(l_lane);
  if (g == 0) {
    s_m[wave][col] = seen ? m_run : neg_inf();
    s_l[wave][col] = l_lane;
  }
  __syncthreads();
  float mm = neg_inf(), l = 0.f, wt[S];
#pragma unroll
  for (int w = 0; w < S; ++w) mm = fmaxf(mm, s_m[qg * S + w][col]);
#pragma unroll
  for (int w = 0; w < S; ++w) {
    wt[w] = __builtin_amdgcn_exp2f(s_m[qg * S + w][col] - mm);  // 0 for a stream that saw no key
    l = fmaf(wt[w], s_l[qg * S + w][col], l);
  }
  if (!q_ok) return;
  const float inv_l = 1.0f / l;
  const bf16_t* muv = a.muv ? static_cast<const bf16_t*>(a.muv) + (size_t)h * kD : nullptr;
  const size_t orow = ((size_t)bh * M + myq) * kD;
#pragma unroll
  for (int c = 0; c < RPW / 4; ++c) {
    const int r0 = RPW * st + 4 * c;  // tile r0 / 16, registers r0 % 16 ..: 4 consecutive features
    const int i0 = 32 * (r0 >> 4) + 8 * ((r0 & 15) >> 2) + 4 * g;
    float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < S; ++w)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(wt[w], s_o[((qg * S + w) * (kD / 2) + r0 + e) * kWave + lane], o[e]);
    const uint2 mw = muv ? *reinterpret_cast<const uint2*>(muv + i0) : make_uint2(0, 0);
    const float v0 = fmaf(o[0], inv_l, bf16_lo(mw.x)), v1 = fmaf(o[1], inv_l, bf16_hi(mw.x));
    const float v2 = fmaf(o[2], inv_l, bf16_lo(mw.y)), v3 = fmaf(o[3], inv_l, bf16_hi(mw.y));
    if (a.out_dtype == LLA_F32)
      *reinterpret_cast<float4*>(static_cast<float*>(a.out) + orow + i0) = make_float4(v0, v1, v2, v3);
    else
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.out) + orow + i0) = make_uint2(pack2(v0, v1), pack2(v2, v3));
  }
}

template <int AXIS, int KS>
hipError_t launch_recon(const Prefill2dArgs& args, hipStream_t stream) {
  Prefill2dArgs a = args;
  // heads per workgroup: with fewer token blocks than compute units the heads are
  // split too, up to one workgroup per unit (a value tile fills a unit's LDS);
  // both axes and the attention per call at (288, 480), one against this many
  // groups: 300 tokens 115 -> 31 us, 1024 tokens 140 -> 47, 2 x 4096 256 -> 203
  const int nb = (a.nk + kRTok - 1) / kRTok;
  const long groups = max(1L, (long)device_cu_count() / ((long)nb * a.B));
  a.hpw = (int)((a.H + groups - 1) / groups);
  const dim3 grid(nb, a.B, (a.H + a.hpw - 1) / a.hpw);
  hipLaunchKernelGGL((recon2d_kernel<AXIS, KS>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

template <int AXIS>
hipError_t launch_recon_r(const Prefill2dArgs& a, int r, hipStream_t stream) {
  switch (r / 16) {
#define LLA_R(ks) \
  case ks: return launch_recon<AXIS, ks>(a, stream);
    LLA_R(1) LLA_R(2) LLA_R(3) LLA_R(4) LLA_R(5) LLA_R(6) LLA_R(7) LLA_R(8)
    LLA_R(9) LLA_R(10) LLA_R(11) LLA_R(12) LLA_R(13) LLA_R(14) LLA_R(15) LLA_R(16)
    LLA_R(17) LLA_R(18) LLA_R(19) LLA_R(20) LLA_R(21) LLA_R(22) LLA_R(23) LLA_R(24)
    LLA_R(25) LLA_R(26) LLA_R(27) LLA_R(28) LLA_R(29) LLA_R(30) LLA_R(31) LLA_R(32)
#undef LLA_R
    default: return hipErrorInvalidValue;
  }
}

// Key streams per workgroup of the attention: 1 (flash2d_kernel, 256 queries),
// 2, 4 (flash2d_streams_kernel, 128 and 64 queries) or 8 (flash2d_split_kernel,
// 32).  Fewer queries per workgroup put more workgroups on the machine, each
// through its keys in less time (1.3, 1.6 and 2.1 times flash2d_kernel's rate), but
// stage every key for fewer queries: a full machine runs at 0.65, 0.4 and 0.26 of
// its rate.  The estimate, in keys of flash2d_kernel's loop: the heaviest
// workgroup, or the mean load of a compute unit (and where workgroups come in
// rounds half of the lightest one, heaviest first), each workgroup with its keys
// and a fixed cost.  Numbers from all four measured on 1871 drawn calls (1 to 32
// heads, 1 to 9000 queries after up to 9000 keys, both caches; repeated and with
// other inputs between): the choice is nowhere more than 3% slower than
// flash2d_kernel and loses 0.2% to the best of the four.  Attention and
// rebuilds per call at (96, 160), 16 heads, 1 / 2 / 4 / 8 streams: 300 tokens
// after 7000 211 / 150 / 118 / 85 us; 1024 tokens 47 / 38 / 32 / 33; 2048 tokens
// 76 / 60 / 55 / 64; 2 x 3191 (104, 96) 126 / 146 / 186 / 217; 4 x 2048 138 / 160
// / 191 / 242.
int key_streams(const Prefill2dArgs& a) {
  const int cus = device_cu_count();
  const double rate[4] = {1.0, 1.3, 1.6, 2.1}, fixed[4] = {95, 130, 130, 160};
  const double bh = (double)a.B * a.H;
  int best = 1;
  double best_t = 0.0;
  for (int k = 0; k < 4; ++k) {
    const int qb = kQBlock >> k, nqb = (a.M + qb - 1) / qb;
    const double wgs = bh * nqb;
    if (k == 0 && wgs > 8.0 * cus) return 1;
    if (nqb > 65535) break;
    const double keys = bh * ((double)nqb * a.p0 + 0.5 * qb * nqb * (nqb - 1.0) + a.M);
    double t = (keys + wgs * fixed[k]) / cus;
    if (wgs > cus) t += 0.5 * (a.p0 + min(qb, a.M) + fixed[k]);
    t = fmax(t, a.p0 + a.M + fixed[k]) / rate[k];
    if (k == 0 || t < 0.97 * best_t) {
      best = 1 << k;
      best_t = t;
    }
  }
  return best;
}

hipError_t launch_attention(const Prefill2dArgs& a, hipStream_t stream) {
  const int bh = a.B * a.H, threads = kFThreads;
  switch (key_streams(a)) {
    case 1: hipLaunchKernelGGL(flash2d_kernel, dim3(bh, (a.M + 255) / 256), dim3(threads), 0, stream, a); break;
    case 2: hipLaunchKernelGGL(flash2d_streams_kernel<2>, dim3(bh, (a.M + 127) / 128), dim3(threads), 0, stream, a); break;
    case 4: hipLaunchKernelGGL(flash2d_streams_kernel<4>, dim3(bh, (a.M + 63) / 64), dim3(threads), 0, stream, a); break;
    default: hipLaunchKernelGGL(flash2d_split_kernel, dim3(bh, (a.M + 31) / 32), dim3(threads), 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace

size_t prefill_2d_ws_bytes(int B, int H, int n_keys) {
  const size_t nk = ((size_t)n_keys + kPage - 1) / kPage * kPage;
  return 2 * (size_t)B * H * nk * kD * sizeof(bf16_t);
}

hipError_t launch_prefill_2d(const Prefill2dArgs& a, hipStream_t stream) {
  hipError_t e = launch_recon_r<0>(a, a.rk, stream);
  if (e != hipSuccess) return e;
  e = launch_recon_r<1>(a, a.rv, stream);
  if (e != hipSuccess) return e;
  return launch_attention(a, stream);
}

template <int AXIS>
hipError_t launch_recon_ph(const Prefill2dArgs& a, int r, int ppw, hipStream_t stream) {
  const dim3 grid((a.nk / kPage + ppw - 1) / ppw, a.B * a.H, AXIS == 2 ? 2 : 1);
  switch ((r + 15) / 16) {
#define LLA_R(ks)                                                                                        \
  case ks:                                                                                               \
    if constexpr (AXIS < 2 || ks <= kBothSteps)                                                          \
      hipLaunchKernelGGL((recon_ph_kernel<AXIS, ks>), grid, dim3(kThreads), 0, stream, a, ppw);          \
    break;
    LLA_R(1) LLA_R(2) LLA_R(3) LLA_R(4) LLA_R(5) LLA_R(6) LLA_R(7) LLA_R(8)
    LLA_R(9) LLA_R(10) LLA_R(11) LLA_R(12) LLA_R(13) LLA_R(14) LLA_R(15) LLA_R(16)
    LLA_R(17) LLA_R(18) LLA_R(19) LLA_R(20) LLA_R(21) LLA_R(22) LLA_R(23) LLA_R(24)
    LLA_R(25) LLA_R(26) LLA_R(27) LLA_R(28) LLA_R(29) LLA_R(30) LLA_R(31) LLA_R(32)
#undef LLA_R
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prefill_rebuild(const Prefill2dArgs& a, hipStream_t stream) {
  // pages per workgroup: about 2048 workgroups over the (b, h) pages, 1 to 8 pages each
  const long total = (long)(a.nk / kPage) * a.B * a.H;
  const int ppw = (int)max(1L, min(8L, total / 2048));
  const int r = max(a.rk, a.rv);
  // Both axes in one launch below 4096 pages (one workgroup per page, two rounds
  // of the machine at most): per call, 16 heads, two launches / one, 70 tokens
  // after 100 (192, 320) 21.2 / 15.2 us, 100 tokens (96, 160) 16.9 / 14.9, 2 x 500
  // after 500 (120, 200) 34.5 / 30.2, 300 after 7000 (96, 160) 87.4 / 85.6.  With
  // more pages nothing is gained, and above 320 features the kernel of both axes
  // spills registers.
  hipError_t e;
  if (r <= 16 * kBothSteps && total < 4096) {
    e = launch_recon_ph<2>(a, r, ppw, stream);
  } else {
    e = launch_recon_ph<0>(a, a.rk, ppw, stream);
    if (e == hipSuccess) e = launch_recon_ph<1>(a, a.rv, ppw, stream);
  }
  if (e != hipSuccess) return e;
  return launch_attention(a, stream);
}

}  // namespace lla

extern "C" int lla_internal_key_streams(int B, int H, int M, int p0) {
  lla::Prefill2dArgs a{};
  a.B = B;
  a.H = H;
  a.M = M;
  a.p0 = p0;
  return lla::key_streams(a);
}
