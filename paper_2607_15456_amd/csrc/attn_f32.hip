// fp32 attention over the paged latent cache, absorbed form, on the fp32
// matrix instructions: decode (one query per (b, h)) and the causal prefill
// (query m attends positions [0, p0 + m]).
//
// One workgroup of 8 wavefronts takes a tile of 16 queries of one (b, h) and
// walks its pages in groups of 8; v_mfma_f32_16x16x4_f32 multiplies in fp32 and
// accumulates in fp32, as the vector unit would.  Both contractions read their
// operands straight from the feature-major page:
//   * scores, wavefront w on page w of the group: D[key][query] +=
//     c_k[feature][key] q~[feature][query].  Lane (c, g) = (lane % 16, lane / 16)
//     loads the 16 bytes of keys 4c .. 4c + 3 of feature 4s + g; component t is
//     the A operand of score tile t, whose row c is key 4c + t, so a wave-wide
//     load is 1 KB of consecutive bytes and feeds four products.  q~ comes from
//     LDS ([feature][16 queries]: step s reads 64 consecutive words).
//   * softmax: lane (c, g) holds query c's scores of keys 16g + 4i + t
//     (register i of tile t), so a page's maximum takes two lane exchanges; the
//     group's goes through LDS, the same in every wavefront, and so do the
//     probabilities.
//   * values, wavefront w on the 16-row feature tiles w, w + 8, .. over all
//     pages of the group: D[feature][query] += c_v[feature][key] p[key][query].
//     The product for (i, t) takes key 16g + 4i + t from lane group g, so the
//     probabilities are B operands as they were written, and A is component t
//     of the 16 bytes at keys 16g + 4i of feature row c.
// A feature tile thus has one owner, nothing is merged at the end, and the
// walk is a short loop (with a page of its own per wavefront for both products
// and three merge rounds a 500-token prompt's call took 55 us, now 38).
//
// What bounds it: at small sizes the chain of load batches (q~, K, V, U_v, about
// 1 us each from beyond L2) and 2 us of launch; a 500-token prompt of 16 heads at
// (96, 160) has 12 us of products, and two workgroups per compute unit.  Against
// the vector-unit scan, per call: that prompt 305 -> 38 us; one decode query
// over 512 tokens 26 -> 24 (39 -> 25 with other inputs between the calls).
// A page's products are summed apart from the running sum (chains of 32), q~
// and the output in four chains: the error against 64 bits stays that of the
// scan (4.2e-7 at 500 tokens) or below.
//
// The weights of keys that a query does not attend are 0, and latents past the
// tile's last key count as 0 whatever they hold.  A key between the tile's first
// and last query is attended by some of them only: an infinity or NaN there is
// left out of the product (0 times it would reach the others) and added on the
// vector unit to the queries that attend it.

#include "lla_device.h"
#include "lla_internal.h"
#include "../../include/lla.h"

namespace lla {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kThreads = kWaves * kWave;
constexpr int kTile = 16;  // queries per workgroup

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bool finite(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

// Buffer loads: one lane offset plus a uniform offset, so no address registers
// per row.  aux 0: ordinary cache policy (the tiles of a prefill share pages).
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc region(const float* base, size_t floats) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)(floats * 4), 0x00020000);
}
__device__ __forceinline__ f32x4 ld4(Rsrc r, int lane_off, int off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
}

// TPW: value tiles per wavefront (r_v <= 128 TPW).  DEEP: one workgroup per
// compute unit with more loads in flight; otherwise two (see the launch).
template <int TPW, bool DEEP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(DEEP ? 2 : 4)))
void attn_f32_kernel(DecodeArgs a) {
  constexpr int KB = DEEP ? 8 : 4;  // K steps per load batch, two batches in flight
  constexpr int NI = DEEP ? 4 : 2;  // value items in the register ring
  constexpr int QB = DEEP ? 8 : 4;  // q~: 16-column blocks of U_k^T q in flight
  static_assert(NI % TPW == 0, "a round holds whole pages");
  // q~ rows: content padded to whole batches of steps, rotary after them; in
  // the end z [feature][query], padded to 64 rows.  Padding rows are zero.
  __shared__ __attribute__((aligned(16))) float s_q[(kMaxRank + 64) * kTile];
  __shared__ __attribute__((aligned(16))) float s_p[kWaves][kPage * kTile];  // [page][4i + t][lane]
  __shared__ float s_own[kTile * kTile];  // scores of the tile's own keys n_lo .. n_hi - 1 (at most 15)
  __shared__ float s_m[kWaves][kTile], s_l[kWaves][kTile];
  __shared__ int s_last;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c = lane & 15, g = lane >> 4;
  int bx, h;
  xcd_head_order(bx, h, !(a.dr > 0 && a.Hr == 1));
  const int tiles = (a.M + kTile - 1) / kTile;
  const unsigned ubx = bx;
  const int bt = ubx / a.splits, split = ubx - bt * a.splits;
  const int b = bt / tiles, m0 = (tiles - 1 - (bt - b * tiles)) * kTile;  // longest tiles first
  const int mq = min(m0 + c, a.M - 1);  // this lane's query (columns past M repeat the last one)
  int n_lo, n_hi, N;  // keys of the tile's first and last query, of this lane's query
  if (a.causal) {
    n_lo = a.p0 + m0 + 1;
    n_hi = a.p0 + min(m0 + kTile, a.M);
    N = a.p0 + mq + 1;
  } else {
    n_lo = n_hi = N = a.ctx_len ? a.ctx_len[b] : a.n_ctx;
  }
  const bool bad = n_hi < 1 || n_hi > a.n_ctx;
  const int pages = bad ? 0 : (n_hi + kPage - 1) / kPage;
  const int per = (pages + a.splits - 1) / a.splits;
  const int pb = min(pages, split * per), pe = min(pages, pb + per);
  const size_t bh = (size_t)b * a.H + h;
  const int d = a.d, rk = a.rk, rv = a.rv;
  const int nkc = (rk + 4 * KB - 1) / (4 * KB) * KB;  // K steps of 4 content features, whole batches
  // regions of this (b, h): below 2^31 bytes, checked on the host
  const Rsrc k_src = region(static_cast<const float*>(a.ck) + bh * (size_t)a.n_max * rk, (size_t)a.n_max * rk);
  const float* const cvb = static_cast<const float*>(a.cv) + bh * (size_t)a.n_max * rv;
  const Rsrc v_src = region(cvb, (size_t)a.n_max * rv);
  const Rsrc r_src =
      a.dr ? region(static_cast<const float*>(a.rc) + ((size_t)b * a.Hr + (a.Hr == 1 ? 0 : h)) * (size_t)a.n_max * a.dr,
                    (size_t)a.n_max * a.dr)
           : k_src;

  const int nvt = (rv + 15) / 16;
  // K steps s0 .. s0 + KB - 1 of a page.  Rows past the rank read on (the next
  // page, or past the region: zero) and are replaced by zero.
  auto kload = [&](f32x4 (&r)[KB], int p, int s0) {
    const unsigned lo = lane * 16 + (unsigned)(p * rk + 4 * s0) * kPage * 4;
#pragma unroll
    for (int u = 0; u < KB; ++u) r[u] = ld4(k_src, (int)(lo + u * 1024), 0);
  };
  auto kmul = [&](f32x4 (&r)[KB], int s0, f32x4 (&s4)[4]) {
    float qv[KB];
#pragma unroll
    for (int u = 0; u < KB; ++u) qv[u] = s_q[(s0 + u) * 64 + lane];
    if (4 * (s0 + KB) > rk) {
#pragma unroll
      for (int u = 0; u < KB; ++u)
        if (4 * (s0 + u) + g >= rk) r[u] = f32x4{0.f};
    }
    // no guard per step (one makes each step wait for its own LDS read)
#pragma unroll
    for (int u = 0; u < KB; ++u)
#pragma unroll
      for (int t = 0; t < 4; ++t) s4[t] = mfma4(r[u][t], qv[u], s4[t]);
  };
  // V row c of the wavefront's tiles; rows past the rank re-read its last row
  // (not stored), tiles past the last one the last tile
  auto vload = [&](f32x4 (&r)[4], int p, int u) {
    const int row = min(16 * (wave + kWaves * u) + c, rv - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = ld4(v_src, ((p * rv + row) * kPage + 16 * g) * 4 + 16 * i, 0);
  };
  f32x4 ka[KB], kb[KB];
  if (pb + wave < pe) kload(ka, pb + wave, 0);  // in flight while q~ is formed

  // ---- q~ = U_k^T q (scale * log2(e) folded in): wavefront w takes the
  // 16-feature tiles w, w + 8, ..; both operands straight from memory ----
  {
    const float* uk = static_cast<const float*>(a.uk) + (size_t)h * d * rk;
    const float* qp = static_cast<const float*>(a.q) + (bh * a.M + mq) * (size_t)d + 4 * g;
#pragma unroll 1
    for (int t = wave; t < nkc / 4; t += kWaves) {
      const int j = 16 * t + c;
      const float* up = uk + (size_t)(4 * g) * rk + min(j, rk - 1);
      f32x4 part[4];  // four chains of products, added at the end
#pragma unroll
      for (int e = 0; e < 4; ++e) part[e] = f32x4{0.f};
#pragma unroll 1
      for (int i0 = 0; i0 < d; i0 += 16 * QB) {  // d is a multiple of 32
        f32x4 qv[QB];
        float uv[QB][4];
#pragma unroll
        for (int s = 0; s < QB; ++s) {
          const int i = i0 + 16 * s < d ? i0 + 16 * s : i0;
          qv[s] = *reinterpret_cast<const f32x4*>(qp + i);
#pragma unroll
          for (int e = 0; e < 4; ++e) uv[s][e] = up[(size_t)(i + e) * rk];
        }
#pragma unroll
        for (int s = 0; s < QB; ++s)
          if (i0 + 16 * s < d)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[e] = mfma4(uv[s][e], qv[s][e], part[e]);
      }
      const f32x4 acc = (part[0] + part[1]) + (part[2] + part[3]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 16 * t + 4 * g + e;
        s_q[row * kTile + c] = row < rk ? acc[e] * a.qscale : 0.f;
      }
    }
#pragma unroll 1
    for (int e = tid; e < a.dr * kTile; e += kThreads) {
      const int f = e / kTile, m = min(m0 + e % kTile, a.M - 1);
      s_q[4 * nkc * kTile + e] = a.qscale * static_cast<const float*>(a.qr)[(bh * a.M + m) * (size_t)a.dr + f];
    }
    __syncthreads();
  }

  // ---- the pages, in groups of 8 ----
  f32x4 z[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u) z[u] = f32x4{0.f};
  float m_run = neg_inf(), l_run = 0.f;  // of query c; l of this lane's keys only
  bool odd = false;                      // an infinity or NaN among the tile's own keys
  for (int g0 = pb; g0 < pe; g0 += kWaves) {
    const int p = g0 + wave, np = min(kWaves, pe - g0);
    f32x4 s4[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) s4[t] = f32x4{neg_inf(), neg_inf(), neg_inf(), neg_inf()};
    float mx = m_run;
    if (p < pe) {
#pragma unroll
      for (int t = 0; t < 4; ++t) s4[t] = f32x4{0.f};
      f32x4 odd4[4];  // DEEP: every second batch on its own chain
#pragma unroll
      for (int t = 0; t < 4; ++t) odd4[t] = f32x4{0.f};
      if (g0 > pb) kload(ka, p, 0);
#pragma unroll 1
      for (int s0 = 0; s0 < nkc; s0 += 2 * KB) {
        if (s0 + KB < nkc) kload(kb, p, s0 + KB);
        kmul(ka, s0, s4);
        if (s0 + 2 * KB < nkc) kload(ka, p, s0 + 2 * KB);
        if (s0 + KB < nkc) kmul(kb, s0 + KB, DEEP ? odd4 : s4);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) s4[t] += odd4[t];
#pragma unroll 2
      for (int s = 0; s < a.dr / 4; ++s) {  // rotary rows
        const f32x4 r = ld4(r_src, lane * 16 + (p * a.dr + 4 * s) * kPage * 4, 0);
        const float qv = s_q[(nkc + s) * 64 + lane];
#pragma unroll
        for (int t = 0; t < 4; ++t) s4[t] = mfma4(r[t], qv, s4[t]);
      }
      if ((p + 1) * kPage > n_lo) {
        const int key0 = p * kPage + 16 * g;  // key of (i, t): key0 + 4i + t
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = key0 + 4 * i + t;
            if (key >= n_lo && key < n_hi) s_own[(key - n_lo) * kTile + c] = s4[t][i];
            if (key >= N) s4[t][i] = neg_inf();
          }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s4[t][i]);
      mx = fmaxf(mx, xor_shfl(mx, 16));
      mx = fmaxf(mx, xor_shfl(mx, 32));
      if (g == 0) s_m[wave][c] = mx;
    }
    // items (page, tile) of the value products, NI per round, the loads of
    // NI - 1 items in flight ahead
    f32x4 v[NI][4];
    const int items = wave < nvt ? np * TPW : 0;
#pragma unroll
    for (int j = 0; j < NI - 1; ++j) vload(v[j], g0 + min(j / TPW, np - 1), j % TPW);
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < np; ++w) mx = fmaxf(mx, s_m[w][c]);
    const float ms = mx == neg_inf() ? 0.f : mx;  // no key of this query so far: weights 0
    if (__any(mx > m_run)) {
      const float alpha = exp2_fast(m_run - ms);
      l_run *= alpha;
#pragma unroll
      for (int u = 0; u < TPW; ++u) z[u] *= alpha;
      m_run = mx;
    }
    if (p < pe) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float w = exp2_fast(s4[t][i] - ms);
          l_run += w;
          s_p[wave][(4 * i + t) * kWave + lane] = w;
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int n0 = 0; n0 < items; n0 += NI) {
      float w[16];  // probabilities of the item's page
      const int pg0 = n0 / TPW;
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int pg = pg0 + j / TPW;
        constexpr int kAhead = NI - 1;
        const int u = j % TPW;
        if (pg >= np) break;
        vload(v[(j + kAhead) % NI], g0 + min(pg0 + (j + kAhead) / TPW, np - 1), (j + kAhead) % TPW);
        f32x4(&r)[4] = v[j];
        if ((g0 + pg + 1) * kPage > n_lo) {
          int key0 = (g0 + pg) * kPage + 16 * g;
          asm volatile("" : "+v"(key0));  // compared here, not held as masks over the items
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int key = key0 + 4 * i + t;
              if (key >= n_lo && (key >= n_hi || !finite(r[i][t]))) {
                odd |= key < n_hi;
                r[i][t] = 0.f;
              }
            }
        }
        if (u == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) w[e] = s_p[pg][e * kWave + lane];
        }
        f32x4 one = f32x4{0.f}, two = f32x4{0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          one = mfma4(r[i][0], w[4 * i], one);
          two = mfma4(r[i][1], w[4 * i + 1], two);
          one = mfma4(r[i][2], w[4 * i + 2], one);
          two = mfma4(r[i][3], w[4 * i + 3], two);
        }
        z[u] += one + two;
      }
    }
  }

  // ---- l of all wavefronts (m is the same in each); z to LDS ----
  l_run += xor_shfl(l_run, 16);
  l_run += xor_shfl(l_run, 32);
  if (g == 0) s_l[wave][c] = l_run;
  __syncthreads();  // also: every wavefront is done with q~
  float lg = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) lg += s_l[w][c];
  const float mgs = m_run == neg_inf() ? 0.f : m_run;
  const bool any_odd = __any(odd);
#pragma unroll
  for (int u = 0; u < TPW; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * (wave + kWaves * u) + 4 * g + e;
      if (row < kMaxRank) {
        float t = row < rv ? z[u][e] : 0.f;
        if (any_odd && row < rv)
#pragma unroll 1
          for (int k = 0; k < N - n_lo; ++k) {
            const int key = n_lo + k;
            const float x = cvb[((size_t)(key / kPage) * rv + row) * kPage + key % kPage];
            if (!finite(x)) t = fmaf(exp2_fast(s_own[k * kTile + c] - mgs), x, t);
          }
        s_q[row * kTile + c] = t;
      }
    }
  __syncthreads();

  const size_t unit = bh;  // split launches: one query per (b, h)
  if (a.splits > 1) {
    // publish this split's (m, l, z); the last arrival merges all of them
    const int stride = rv + 2;
    float* part = a.part + (unit * a.splits + split) * stride;
#pragma unroll 1
    for (int j = tid; j < rv; j += kThreads) part[2 + j] = s_q[j * kTile];
    if (tid == 0) {
      part[0] = m_run;
      part[1] = lg;
    }
    wait_stores_in_l2();
    __syncthreads();
    if (tid == 0) {
      const uint32_t prev = __hip_atomic_fetch_add(a.cnt + unit, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      s_last = (prev == (uint32_t)(a.splits - 1));
    }
    __syncthreads();
    if (!s_last) return;
    const float* P = a.part + unit * a.splits * stride;
    float ma = neg_inf();
#pragma unroll 1
    for (int s = 0; s < a.splits; ++s) ma = fmaxf(ma, P[(size_t)s * stride]);
    if (ma == neg_inf()) ma = 0.f;
    lg = 0.f;
#pragma unroll 1
    for (int s = 0; s < a.splits; ++s) lg = fmaf(exp2_fast(P[(size_t)s * stride] - ma), P[(size_t)s * stride + 1], lg);
#pragma unroll 1
    for (int j = tid; j < rv; j += kThreads) {
      float t = 0.f;
#pragma unroll 1
      for (int s = 0; s < a.splits; ++s) t = fmaf(exp2_fast(P[(size_t)s * stride] - ma), P[(size_t)s * stride + 2 + j], t);
      s_q[j * kTile] = t;
    }
    if (tid == 0) __hip_atomic_store(a.cnt + unit, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
  }

  // ---- out = U_v (z / l) + mu_v: D[i][query], wavefront w the 16-row tiles w, w + 8, .. ----
  const float* uvh = static_cast<const float*>(a.uv) + (size_t)h * d * rv;
  const float* muv = a.muv ? static_cast<const float*>(a.muv) + (size_t)h * d : nullptr;
  const bool live = m0 + c < a.M;
  const size_t obase = (bh * a.M + mq) * (size_t)d;
#pragma unroll 1
  for (int t = wave; t < d / 16; t += kWaves) {
    const float* up = uvh + (size_t)(16 * t + c) * rv;
    f32x4 part[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) part[e] = f32x4{0.f};
    if (rv % 4 == 0) {  // rows of U_v start on 16 bytes; columns past the rank count as zero
      auto uload = [&](f32x4 (&r)[4], int j0) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
          r[s] = *reinterpret_cast<const f32x4*>(up + min(j0 + 16 * s + 4 * g, rv - 4));
      };
      f32x4 cur[4], next[4];
      uload(cur, 0);
#pragma unroll 1
      for (int j0 = 0; j0 < rv; j0 += 64) {
        uload(next, j0 + 64);
        float zv[16];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int e = 0; e < 4; ++e) zv[4 * s + e] = s_q[(j0 + 16 * s + 4 * g + e) * kTile + c];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if (j0 + 16 * s + 4 * g >= rv) cur[s] = f32x4{0.f};
#pragma unroll
          for (int e = 0; e < 4; ++e) part[e] = mfma4(cur[s][e], zv[4 * s + e], part[e]);
          cur[s] = next[s];
        }
      }
    } else {
#pragma unroll 1
      for (int j0 = 4 * g; j0 < rv + 4 * g; j0 += 16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = j0 + e < rv;
          part[e] = mfma4(in ? up[j0 + e] : 0.f, in ? s_q[(j0 + e) * kTile + c] : 0.f, part[e]);
        }
      }
    }
    const f32x4 acc = (part[0] + part[1]) + (part[2] + part[3]);
    if (live) {
      f32x4 o = acc / lg;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 16 * t + 4 * g + e;
        float v = o[e];
        if (muv) v += muv[i];
        if (bad) v = __builtin_nanf("");
        if (a.out_dtype == LLA_F32)
          static_cast<float*>(a.out)[obase + i] = v;
        else
          static_cast<bf16_t*>(a.out)[obase + i] = f32_to_bf16(v);
      }
    }
  }
}

template <int TPW>
hipError_t launch_tpw(const DecodeArgs& a, hipStream_t stream) {
  const dim3 grid(a.B * ((a.M + kTile - 1) / kTile) * a.splits, a.H);
  if constexpr (TPW <= 2) {
    // More workgroups than compute units: two share one.
    if ((int64_t)grid.x * grid.y > device_cu_count()) {
      hipLaunchKernelGGL((attn_f32_kernel<TPW, false>), grid, dim3(kThreads), 0, stream, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((attn_f32_kernel<TPW, true>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const DecodeArgs& a, hipStream_t stream) {
  if (a.splits > 1 && a.M != 1) return hipErrorInvalidValue;
  if (a.rv <= 128) return launch_tpw<1>(a, stream);
  if (a.rv <= 256) return launch_tpw<2>(a, stream);
  return launch_tpw<4>(a, stream);
}

}  // namespace lla
