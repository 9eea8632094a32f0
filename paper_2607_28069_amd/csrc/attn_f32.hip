// Attention of query rows over a float32 cache with the frontier mask of App. C.1 (the query at
// logical position p sees slots [0, p]; slot index = logical position): suffix prefill, frontier
// prefill and decode on v_mfma_f32_16x16x4_f32, in float32 throughout.
//
// Per (layer, request, kv head) the M = n_q * n_rep query rows are packed as in the bf16 prefill
// (row r = token r / n_rep, head g * n_rep + r % n_rep).  A workgroup takes 16 or 32 of them and
// every key they see; its waves take the 16-key tiles in turn (wave w: tiles w, w + W, ...), each
// with its own online softmax, and merge by log-sum-exp in LDS at the end.  The key range is
// thereby split W ways without a workspace (float32 calls take none).
//
//  * S^T = K Q^T: a lane holds K row n = lane % 16 at 4 consecutive head dims per 16-byte load
//    (dims 16 j + 4 g .. + 3, g = lane / 16), and Q^T in the same order, so the 16 x 4 operands
//    need no rearrangement; the accumulator gives a lane query n and keys 4 g + i.
//  * O^T = V^T P^T: that accumulator is the B operand as it stands when step i takes keys
//    {4 g + i}; V comes as whole rows, 16 bytes per lane (dims 64 h + 4 n + e), and output
//    block e collects dims 4 row + e, which leaves a lane 4 consecutive dims to store.
//  * K and V go straight from global memory to registers (no LDS, no barrier in the loop), the
//    next tile's loads in flight while a tile is used.  Tiles that some row does not see all of,
//    or that reach the call's own tokens, are left to a second loop that addresses row by row:
//    with both kinds in one loop the register count doubled.
//  * The rate bound is the float32 matrix rate, 64 flops per cycle and SIMD (1/16 of bf16; a large
//    library product reaches 150 TFLOP/s): a 16-key tile of 16 rows at head_dim 64 is 32 products
//    of 32 cycles for 8 KB loaded.  Measured against a kernel with one row per workgroup and
//    plain vector arithmetic: 16 heads over 4 kv heads at head_dim 64, four requests of 2077 keys,
//    61 tokens 356 -> 26.0 us; four requests of 4160 keys, 32 heads over 8 at head_dim 128, 64
//    tokens 3520 -> 148 us (119 TFLOP/s); a decode step of one request at 4096 keys 293 -> 41 us.
//  * New tokens' K/V are read from k_new / v_new and stored into the cache by the workgroups of
//    their (request, kv head), each a share of the rows; no workgroup reads those slots from the
//    cache.
//  * A tile some rows see only in part has its scores masked; a probability of 0 times a value
//    that is not finite is no 0, so a tile that holds such a value takes its PV products one
//    query column at a time, with the values that column does not see cleared.
#include <algorithm>

#include "pic_bounds.h"
#include "pic_internal.h"

namespace pic {
namespace {

constexpr int kTile = 16;   // keys per wave tile
constexpr int kNumXcd = 8;

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Lanes n, n + 16, n + 32, n + 48 hold the same query column.
__device__ __forceinline__ float column_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float column_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// grid (ceil(n_units / 8) * 8, L), 64 W threads; NB blocks of 16 query rows.  Units [unit0, unit0 +
// n_units) of the m_tiles * batch * Hkv.
template <int HD, int NB, int W>
__global__ void __launch_bounds__(64 * W) attn_f32_kernel(F32AttnArgs a, int32_t m_tiles, int32_t unit0, int32_t n_units) {
  constexpr int QJ = HD / 16;         // 16-byte pieces of a Q or K row per lane
  constexpr int VH = HD / 64;         // 16-byte pieces of a V row per lane
  constexpr int ROWS = 16 * NB;
  constexpr int LROW = HD + 4;        // floats per row of the merge area (4 of padding)
  __shared__ __attribute__((aligned(16))) float o_lds[W * ROWS * LROW];
  __shared__ float m_lds[W * ROWS], l_lds[W * ROWS];

  // blocks are dealt round-robin to the 8 XCDs: a contiguous range of units for each, so that
  // the m-tiles of one (request, kv head) read its keys through one L2
  const int per_xcd = (n_units + kNumXcd - 1) / kNumXcd;
  const int at = ((int)blockIdx.x % kNumXcd) * per_xcd + (int)blockIdx.x / kNumXcd;
  if (at >= n_units) return;
  const int unit = unit0 + at;
  const AttnShape& s = a.s;
  const int mt = m_tiles - 1 - unit % m_tiles, bg = unit / m_tiles;   // later rows see more keys: first
  const int Hkv = s.n_kv_heads, Hq = s.n_q_heads, n_rep = Hq / Hkv, n_q = a.n_q;
  const int b = bg / Hkv, g = bg % Hkv, l = blockIdx.y;
  const int64_t lb = (int64_t)l * s.batch + b;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = n_q * n_rep, row0 = mt * ROWS;

  // query rows and their positions; an unused row (past M, or a token without a position) takes
  // the workgroup's furthest position and is dropped at the end
  bool row_ok[NB];
  int64_t qrow[NB];
  int qpos[NB], lo = INT32_MAX, hi = -1;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int r = row0 + 16 * nb + n;
    const int tok = r < M ? r / n_rep : n_q - 1;
    const int64_t p = a.pos(b, tok);
    row_ok[nb] = r < M && p >= 0;
    qpos[nb] = (int)p;
    qrow[nb] = (lb * n_q + tok) * Hq + g * n_rep + (r < M ? r - tok * n_rep : 0);
    if (row_ok[nb]) {
      lo = min(lo, qpos[nb]);
      hi = max(hi, qpos[nb]);
    }
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o, 64));
    hi = max(hi, __shfl_xor(hi, o, 64));
  }
  const int pos_min = __builtin_amdgcn_readfirstlane(lo), last = __builtin_amdgcn_readfirstlane(hi);
  // slots from `fresh` on are the call's own tokens (table positions: all slots are in the cache)
  const int fresh = a.k_new ? (int)a.pos(b, 0) : INT32_MAX;

  const int64_t kv0 = (lb * Hkv + g) * s.cache_cap * HD;
  const float* Kg = a.cache_k + kv0;
  const float* Vg = a.cache_v + kv0;
  const int64_t new0 = (lb * n_q * Hkv + g) * HD;
  const int64_t new_stride = (int64_t)Hkv * HD;
  if (a.k_new) {   // this workgroup's share of the new rows -> the cache, 16 bytes per thread
    constexpr int CPR = HD / 4;
    const int per = (n_q + m_tiles - 1) / m_tiles;
    const int i0 = min(mt * per, n_q), i1 = min(i0 + per, n_q);
    for (int c = tid; c < (i1 - i0) * 2 * CPR; c += 64 * W) {
      const int i = i0 + c / (2 * CPR), part = c % (2 * CPR), d = 4 * (part % CPR);
      const float* src = (part < CPR ? a.k_new : a.v_new) + new0 + i * new_stride + d;
      float* dst = (part < CPR ? a.cache_k : a.cache_v) + kv0 + (int64_t)(fresh + i) * HD + d;
      *reinterpret_cast<f32x4*>(dst) = *reinterpret_cast<const f32x4*>(src);
    }
  }
  if (last < 0) return;   // (uniform) no used row

  f32x4 q[NB][QJ];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    if (!row_ok[nb]) qpos[nb] = last;
#pragma unroll
    for (int j = 0; j < QJ; ++j)
      q[nb][j] = row_ok[nb] ? *reinterpret_cast<const f32x4*>(a.q + qrow[nb] * HD + 16 * j + 4 * g4) : f32x4{};
  }

  f32x4 o[NB][VH][4];
  float m_run[NB], m_use[NB], l_run[NB];   // reference max, the same with 0 for "no key yet", lane's row sum
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    m_run[nb] = -INFINITY;
    m_use[nb] = l_run[nb] = 0.f;
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[nb][h][e] = f32x4{};
  }

  // S^T of a tile: two accumulation chains per block of rows, added at the end
  auto scores = [&](const f32x4 (&kr)[QJ], f32x4 (&sc)[NB]) {
    f32x4 c2[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) sc[nb] = c2[nb] = f32x4{};
#pragma unroll
    for (int j = 0; j < QJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          f32x4& c = e & 1 ? c2[nb] : sc[nb];
          c = mfma(kr[j][e], q[nb][j][e], c);
        }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) sc[nb] += c2[nb];
  };
  // scores -> probabilities against the running reference (moved only when a score exceeds it by
  // 2^8: below that nothing loses relative precision)
  auto softmax = [&](f32x4 (&sc)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float mx = fmaxf(fmaxf(sc[nb][0], sc[nb][1]), fmaxf(sc[nb][2], sc[nb][3])) * s.scale_log2;
      if (__any(mx > m_run[nb] + 8.f)) {
        const float m_new = fmaxf(m_run[nb], column_max(mx));
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[nb] - m_new);
        m_run[nb] = m_new;
        m_use[nb] = m_new == -INFINITY ? 0.f : m_new;
        l_run[nb] *= alpha;
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[nb][h][e] *= alpha;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[nb][i] = __builtin_amdgcn_exp2f(fmaf(sc[nb][i], s.scale_log2, -m_use[nb]));
        l_run[nb] += sc[nb][i];
      }
    }
  };
  auto pv = [&](const f32x4 (&vr)[4][VH], const f32x4 (&p)[NB]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) o[nb][h][e] = mfma(vr[i][h][e], p[nb][i], o[nb][h][e]);
  };

  // ---- tiles of cache rows that every row sees: read from a uniform base, the next tile's loads
  // in flight while this one is used
  const int n_tiles = last / kTile + 1, n_full = min(fresh, pos_min + 1) / kTile;
  int t = wave;
  {
    const int k_lane = n * HD + 4 * g4, v_lane = 4 * g4 * HD + 4 * n;
    auto load = [&](int t, f32x4 (&kr)[QJ], f32x4 (&vr)[4][VH]) {
      const float* kp = Kg + (int64_t)t * (kTile * HD);
      const float* vp = Vg + (int64_t)t * (kTile * HD);
#pragma unroll
      for (int j = 0; j < QJ; ++j) kr[j] = *reinterpret_cast<const f32x4*>(kp + k_lane + 16 * j);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < VH; ++h) vr[i][h] = *reinterpret_cast<const f32x4*>(vp + v_lane + i * HD + 64 * h);
    };
    auto step = [&](const f32x4 (&kr)[QJ], const f32x4 (&vr)[4][VH], f32x4 (&kn)[QJ], f32x4 (&vn)[4][VH]) {
      // (past the last full tile: that tile again, dropped)
      load(t + W < n_full ? t + W : t, kn, vn);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 sc[NB];
      scores(kr, sc);
      softmax(sc);
      pv(vr, sc);
      t += W;
    };
    f32x4 ka[QJ], va[4][VH], kb[QJ], vb[4][VH];
    if (t < n_full) {
      load(t, ka, va);
      while (true) {
        step(ka, va, kb, vb);
        if (t >= n_full) break;
        step(kb, vb, ka, va);
        if (t >= n_full) break;
      }
    }
  }
  // ---- the rest: tiles that reach the call's own tokens or that some row does not see all of.
  // Rows are addressed one by one, slots past the last visible one clamped to it (their scores
  // are masked, their values cleared).
  for (; t < n_tiles; t += W) {
    const int k0 = t * kTile;
    auto row_of = [&](const float* cache, const float* fresh_rows, int key) {
      key = min(key, last);
      return key < fresh ? cache + (int64_t)key * HD : fresh_rows + new0 + (int64_t)(key - fresh) * new_stride;
    };
    f32x4 kr[QJ], vr[4][VH], p[NB];
    const float* kp = row_of(Kg, a.k_new, k0 + n) + 4 * g4;
#pragma unroll
    for (int j = 0; j < QJ; ++j) kr[j] = *reinterpret_cast<const f32x4*>(kp + 16 * j);
    bool odd = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* vp = row_of(Vg, a.v_new, k0 + 4 * g4 + i) + 4 * n;
#pragma unroll
      for (int h = 0; h < VH; ++h) vr[i][h] = *reinterpret_cast<const f32x4*>(vp + 64 * h);
    }
    scores(kr, p);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k0 + 4 * g4 + i > qpos[nb]) p[nb][i] = -INFINITY;
    softmax(p);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (k0 + 4 * g4 + i > last) vr[i][h][e] = 0.f;
          odd |= !(fabsf(vr[i][h][e]) < INFINITY);
        }
    if (!__any(odd)) {
      pv(vr, p);
    } else {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        for (int c = 0; c < 16; ++c) {   // column c's products, kept by its lanes only
          const int pc = __shfl(qpos[nb], c, 64);
#pragma unroll
          for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              f32x4 x = o[nb][h][e];
#pragma unroll
              for (int i = 0; i < 4; ++i) x = mfma(k0 + 4 * g4 + i <= pc ? vr[i][h][e] : 0.f, p[nb][i], x);
#pragma unroll
              for (int i = 0; i < 4; ++i) o[nb][h][e][i] = n == c ? x[i] : o[nb][h][e][i];
            }
        }
    }
  }

  // ---- merge the waves (log-sum-exp); a wave whose tiles held no key of a row adds nothing
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float l_tot = column_sum(l_run[nb]);
    const int r = wave * ROWS + 16 * nb + n;
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(o_lds + r * LROW + 64 * h + 16 * g4 + 4 * i) =
            f32x4{o[nb][h][0][i], o[nb][h][1][i], o[nb][h][2][i], o[nb][h][3][i]};
    if (g4 == 0) {
      m_lds[r] = m_run[nb];
      l_lds[r] = l_tot;
    }
  }
  __syncthreads();
  for (int c = tid; c < ROWS * (HD / 4); c += 64 * W) {
    const int rr = c / (HD / 4), d = 4 * (c % (HD / 4));
    const int r = row0 + rr;
    if (r >= M) continue;
    const int tok = r / n_rep;
    if (a.pos(b, tok) < 0) continue;   // a token without a position: its row is left untouched
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < W; ++w) m = fmaxf(m, m_lds[w * ROWS + rr]);
    float den = 0.f;
    f32x4 acc = {};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float mw = m_lds[w * ROWS + rr], lw = l_lds[w * ROWS + rr];
      if (mw == -INFINITY && lw == 0.f) continue;   // no key of this row (NaN sums pass on)
      const float wt = mw == m ? 1.f : __builtin_amdgcn_exp2f(mw - m);
      den += wt * lw;
      acc += wt * *reinterpret_cast<const f32x4*>(o_lds + (w * ROWS + rr) * LROW + d);
    }
    *reinterpret_cast<f32x4*>(a.out + ((lb * n_q + tok) * Hq + g * n_rep + (r - tok * n_rep)) * HD + d) = acc / den;
  }
}

template <int HD, int NB, int W>
hipError_t launch_as(const F32AttnArgs& a) {
  const int64_t M = (int64_t)a.n_q * (a.s.n_q_heads / a.s.n_kv_heads);
  const int64_t m_tiles = (M + 16 * NB - 1) / (16 * NB);
  const int64_t units = m_tiles * a.s.batch * a.s.n_kv_heads;   // at most the query rows: fits int32
  // a grid holds fewer than 2^32 threads per dimension: 2^23 workgroups of 512
  constexpr int64_t kPart = int64_t(1) << 22;
  for (int64_t u0 = 0; u0 < units; u0 += kPart) {
    const int64_t part = std::min(units - u0, kPart), grid = (part + kNumXcd - 1) / kNumXcd * kNumXcd;
    hipLaunchKernelGGL((attn_f32_kernel<HD, NB, W>), dim3((unsigned)grid, a.s.n_layers), dim3(64 * W), 0, a.stream, a,
                       (int32_t)m_tiles, (int32_t)u0, (int32_t)part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_attn_f32(const F32AttnArgs& a) {
  const int64_t M = (int64_t)a.n_q * (a.s.n_q_heads / a.s.n_kv_heads);
  const int64_t pairs = (int64_t)a.s.batch * a.s.n_kv_heads * a.s.n_layers;
  if (M == 0 || pairs == 0) return hipSuccess;
  // 32 rows halve the K/V traffic per row and feed each loaded value to two products; they are
  // taken where they still give every compute unit a workgroup.  Measured (16 rows / 32 rows): 256
  // workgroups of 32 rows 48.0 / 45.0 us at head_dim 64, 189 / 148 us at 128; half as many 26.3 /
  // 44.2 us and 94 / 146 us.  (256 decode pairs, 4 rows each, pay for the empty second block: 182 / 192.)
  // Eight waves: sixteen took 29.3 us instead of 26.3.  Head_dim 128 with 32 rows needs the
  // registers of one wave per SIMD: eight waves took 212 us instead of 148.
  const bool wide = M > 16 && (M + 31) / 32 * pairs >= 256;
  if (a.s.head_dim == 64) return wide ? launch_as<64, 2, 8>(a) : launch_as<64, 1, 8>(a);
  if (a.s.head_dim == 128) return wide ? launch_as<128, 2, 4>(a) : launch_as<128, 1, 8>(a);
  return hipErrorInvalidValue;
}

}  // namespace pic
