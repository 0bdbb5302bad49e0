// MoL scoring in float32 on gfx950 matrix cores (Eq. 1 / Eq. 2 with the
// two-layer SiLU gating MLP of Appendix A.3), any supported shape and both
// storage types: the float32 problems, bf16 problems that ask for float32
// gating, and the bf16 shapes beyond the f16 chains.
//
// A workgroup walks tiles of QB queries x TI items.  For each tile
//  1. the waves form the component dot products of the tile's queries and
//     items as 16 x 16 blocks straight from global memory (float32 rows on
//     16x16x4 f32 MFMAs, bf16 rows on 16x16x32 bf16 MFMAs: exact products,
//     float32 sums) and leave them in LDS as s[query][p][item];
//  2. each wave takes units of 16 items of one query, one or two at a time, through
//     the gating chain on 16x16x4 f32 MFMAs, 16 hidden units per round:
//       u^T[j][item] = b1[j] + sum_p W1[j][p] s[p][item]
//       l^T[p][item] += sum_j W2[p][j] SiLU(u_j)
//     then the softmax over p and phi.
// Lane (c = lane % 16, g = lane / 16) of a unit holds item c's components
// p = RUN g + mu, mu < RUN = PV / 4 (PV: P padded to 16, 32 or 64 with zero
// weights and -inf logits).  The K slot of an f32 MFMA is the lane group g,
// so register s[mu] is GEMM2's B operand of K block mu as it stands, and
// the four hidden units of an accumulator are GEMM3's B operands of four K
// blocks: nothing is exchanged between lanes.  Output row 16 pt + 4 g + i of
// GEMM3 is ordered to be p = RUN g + 4 pt + i, the lane's own component.
//
// What bounds it: the f32 matrix rate (2048 flop in 32 cycles a SIMD,
// 157 TFLOP/s): 4 P H + 2 P d flop a pair.  The weights sit in LDS as
// prepared A operands (4 H PV bytes each, read as 16-byte vectors, one read
// per four 32-cycle MFMAs of a unit), so that H up to 256 needs no more
// registers than H = 16 and four waves a SIMD stay resident.  Measured: 32 x
// 65,537 pairs of 4 x 4 float32 components, d = 64, H = 32: 0.158 ms (one
// thread a pair, scalar dot products: 29.8 ms); 16 x 32,768 pairs of 8 x 8 bf16
// components, d = 64, H = 64: 0.121 ms (7.1 ms).  A third and not quite half of
// the f32 matrix rate: the rest is the latency of each tile's item rows and the two barriers
// of a tile, which the other workgroups of the CU cover only in part.
#include "mol_tile.h"

namespace mol {

using namespace tile;

namespace {

// Waves of a workgroup: 8, or 4 where the weights are small enough that four
// workgroups fit a CU (P <= 16), whose barriers then stop a quarter of the
// CU's waves each instead of half.
template <int PV>
constexpr int f32_waves() { return PV == 16 ? 4 : 8; }
// dot products of one tile, PV * QB * TI at most: 4 KB of LDS a wave
template <int PV>
constexpr int f32_tile() { return 1024 * f32_waves<PV>(); }

__device__ __forceinline__ f32x4_t mfma_f32(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// floats of padding per LDS row of s, so that the four lane groups of a unit
// read rows RUN apart on different quarters of the 64 banks
template <int PV>
constexpr int s_pad() { return 64 / PV; }

// units a wave takes through the gating chain at once: two where registers
// leave four waves a SIMD resident (two chains of dependent MFMAs), else one
template <int PV>
constexpr int units_at_once() { return PV == 64 ? 1 : 2; }

// 16 bytes (or their zero-padded tail) of a row of `d` elements from element t
template <typename T, bool VEC>
__device__ __forceinline__ uint4 row_chunk(const T* row, int t, int d) {
  constexpr int E = 16 / sizeof(T);
  if constexpr (VEC) {
    // d is a multiple of E: a chunk is wholly inside the row or wholly past it
    const uint4 v = *reinterpret_cast<const uint4*>(row + min(t, d - E));
    return t < d ? v : make_uint4(0, 0, 0, 0);
  } else {
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const T x = row[min(t + e, d - 1)];
      uint32_t bits;
      if constexpr (sizeof(T) == 4) bits = __float_as_uint(x);
      else bits = x;
      if (t + e >= d) bits = 0;
      if constexpr (sizeof(T) == 4) w[e] = bits;
      else w[e / 2] |= bits << (16 * (e & 1));
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// one K chunk (16 bytes of each operand row) of a 16 x 16 block
template <typename T>
__device__ __forceinline__ f32x4_t mma_chunk(uint4 a, uint4 b, f32x4_t c) {
  if constexpr (sizeof(T) == 4) {
    c = mfma_f32(__uint_as_float(a.x), __uint_as_float(b.x), c);
    c = mfma_f32(__uint_as_float(a.y), __uint_as_float(b.y), c);
    c = mfma_f32(__uint_as_float(a.z), __uint_as_float(b.z), c);
    return mfma_f32(__uint_as_float(a.w), __uint_as_float(b.w), c);
  } else {
    return mfma_bf16(a, b, c);
  }
}

}  // namespace

// items: NULL (items n_begin .. n_begin + n_count - 1 for every query) or
// candidate lists [B][item_stride], item_count[b] of them (then QB is 1).
// Writes a score (phi) and/or sort keys as GenMode says; key slots past a
// query's item count are cleared.  Workgroups take equal runs of the tiles,
// ordered item tile by item tile with its nqb query blocks inside.
template <typename T, int PV, bool VEC>
__global__ __launch_bounds__(64 * f32_waves<PV>(), 4) void k_mol_f32(
    DevProb pr, int mode, const float* __restrict__ bound, int n_begin, int n_count, int QB, int ti_log2, int nqb,
    long tiles, const int32_t* __restrict__ items, const int32_t* __restrict__ item_count, long item_stride,
    float* __restrict__ phi, long phi_stride, uint64_t* __restrict__ keys, long key_stride) {
  constexpr int RUN = PV / 4, PT = PV / 16, E = 16 / sizeof(T), KCH = 4 * E;   // KCH: elements of a K chunk
  constexpr int NU = units_at_once<PV>(), CH = VEC ? 4 : 2, NW = f32_waves<PV>(), NT = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) float smf[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int P = pr.P, H = pr.H, d = pr.d, N = pr.N;
  const bool gate = mode != kGenMaxDot && mode != kGenDotKeys;
  const int JT = gate ? (H + 15) / 16 : 0;
  const int TI = 1 << ti_log2, TIP = TI + s_pad<PV>();
  // LDS: W1 and W2 operands, b1, a_q + b2 of the tile's queries, a_x of its
  // items, s, and the s row (q, pq, 0) of each of the tile's query vectors
  float4* sW1 = reinterpret_cast<float4*>(smf);
  float4* sW2 = sW1 + JT * (PV / 16) * 64;
  float* sB1 = reinterpret_cast<float*>(sW2 + JT * PT * 64);
  float* sC = sB1 + 16 * JT;
  float* sAx = sC + QB * PV;                       // [TI][PV + 4]: rows of a lane group's runs on distinct banks
  float* sS = sAx + (gate ? TI * (PV + 4) : 0);
  int* sRow = reinterpret_cast<int*>(sS + QB * PV * TIP);   // [32 ceil(QB P_q / 32)], -1 past the vectors
  const T* X = static_cast<const T*>(pr.X);
  const T* Q = static_cast<const T*>(pr.Q);

  if (gate) {
    const T* W1 = static_cast<const T*>(pr.W1);
    const T* W2 = static_cast<const T*>(pr.W2);
    // sW1[(jt * RUN / 4 + m4) * 64 + lane].e = W1[16 jt + c][RUN g + 4 m4 + e]
    // sW2[(jt * PT + pt) * 64 + lane].e = W2[p][16 jt + 4 g + e], row c of
    // tile pt being p = RUN (c / 4) + 4 pt + c % 4
    for (int i = tid; i < JT * PT * 64; i += NT) {
      const int l = i & 63, m = (i >> 6) % PT, jt = (i >> 6) / PT, lc = l & 15, lg = l >> 4;
      float a[4], b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j1 = 16 * jt + lc, p1 = RUN * lg + 4 * m + e;
        const int p2 = RUN * (lc >> 2) + 4 * m + (lc & 3), j2 = 16 * jt + 4 * lg + e;
        a[e] = j1 < H && p1 < P ? to_f32(W1[j1 * P + p1]) : 0.f;
        b[e] = j2 < H && p2 < P ? to_f32(W2[p2 * H + j2]) : 0.f;
      }
      sW1[i] = float4{a[0], a[1], a[2], a[3]};
      sW2[i] = float4{b[0], b[1], b[2], b[3]};
    }
    for (int i = tid; i < 16 * JT; i += NT) sB1[i] = i < H ? pr.b1[i] : 0.f;
  }
  // the padded components' rows of s stay zero
  for (int i = tid; i < QB * PV * TIP; i += NT) sS[i] = 0.f;
  if (gate)
    for (int i = tid; i < TI * (PV + 4); i += NT) sAx[i] = 0.f;

  for (int i = tid; i < (QB * pr.Pq + 31) / 32 * 32; i += NT)
    sRow[i] = i < QB * pr.Pq ? (i / pr.Pq * PV + i % pr.Pq * pr.Px) * TIP : -1;

  // consecutive tiles of a workgroup: the query blocks of one item tile one
  // after another, whose re-reads of the item rows hit the nearest caches
  const long t0 = tiles * blockIdx.x / gridDim.x, t1 = tiles * (blockIdx.x + 1l) / gridDim.x;
  for (long tile = t0; tile < t1; ++tile) {
    const int b0 = static_cast<int>(tile % nqb) * QB, i0 = static_cast<int>(tile / nqb) * TI;
    const int nq = min(QB, pr.B - b0);
    const int cnt = items ? min(item_count[b0], n_count) : n_count;   // valid items of the row
    const int ni = min(TI, n_count - i0);                             // slots of the tile
    auto item_of = [&](int i) -> int {                                // item of slot i (clamped to a valid one)
      const int s = min(i0 + i, max(cnt, 1) - 1);
      return items ? (cnt > 0 ? min(max(items[b0 * item_stride + s], 0), N - 1) : 0) : n_begin + s;
    };
    __syncthreads();                                                  // the previous tile's units are done
    if (gate)
      for (int i = tid; i < nq * PV; i += NT) {
        const int q = i / PV, p = i % PV;
        sC[i] = p < P ? pr.a_q[static_cast<long>(b0 + q) * P + p] + pr.b2[p] : -__builtin_inff();
      }
    // the items' gating logits, once per item tile (every tile has its own
    // items with candidate lists)
    if (gate && (items || tile == t0 || b0 == 0)) {
      for (int i = tid; i < TI * P; i += NT) {
        const int n = i / P, p = i - n * P;
        sAx[n * (PV + 4) + p] = pr.a_x[static_cast<long>(item_of(n)) * P + p];
      }
    }
    // 1. dot products: jobs of (item component, 32 items, 32 vector rows), so
    // that an item row is read once for two blocks of vectors
    const int nvec = nq * pr.Pq, nrt = (nvec + 31) / 32, nct = TI / 32;   // (TI, nct: powers of two)
    for (int job = wave; job < pr.Px * nrt * nct; job += NW) {
      const int ct = job & (nct - 1), jr = job >> (ti_log2 - 5), px = jr / nrt, rt = jr - px * nrt;
      const T* qb = Q + static_cast<long>(b0) * pr.Pq * d;
      const T* q0 = qb + min(32 * rt + c, nvec - 1) * d;
      const T* q1 = qb + min(32 * rt + 16 + c, nvec - 1) * d;
      const bool two = 32 * rt + 16 < nvec;                           // wave-uniform
      const T* Xp = X + static_cast<long>(px) * N * d;
      const T* x0 = Xp + static_cast<long>(item_of(32 * ct + c)) * d;
      const T* x1 = Xp + static_cast<long>(item_of(32 * ct + 16 + c)) * d;
      f32x4_t acc[2][2] = {};
      int k0 = 0;
      for (; k0 + CH * KCH <= d; k0 += CH * KCH) {                      // CH chunks in flight
        uint4 q[2][CH], x[2][CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          const int t = k0 + e * KCH + g * E;
          x[0][e] = row_chunk<T, VEC>(x0, t, d);
          x[1][e] = row_chunk<T, VEC>(x1, t, d);
          q[0][e] = row_chunk<T, VEC>(q0, t, d);
          q[1][e] = row_chunk<T, VEC>(q1, t, d);
        }
#pragma unroll
        for (int e = 0; e < CH; ++e) {
#pragma unroll
          for (int h = 0; h < 2; ++h) acc[0][h] = mma_chunk<T>(q[0][e], x[h][e], acc[0][h]);
          if (two) {
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[1][h] = mma_chunk<T>(q[1][e], x[h][e], acc[1][h]);
          }
        }
      }
      for (; k0 < d; k0 += KCH) {
        const int t = k0 + g * E;
        const uint4 xa = row_chunk<T, VEC>(x0, t, d), xb = row_chunk<T, VEC>(x1, t, d);
        const uint4 qa = row_chunk<T, VEC>(q0, t, d), qc = row_chunk<T, VEC>(q1, t, d);
        acc[0][0] = mma_chunk<T>(qa, xa, acc[0][0]);
        acc[0][1] = mma_chunk<T>(qa, xb, acc[0][1]);
        acc[1][0] = mma_chunk<T>(qc, xa, acc[1][0]);
        acc[1][1] = mma_chunk<T>(qc, xb, acc[1][1]);
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int v = 32 * rt + 16 * r + 4 * g;
        const int4 row = *reinterpret_cast<const int4*>(sRow + v);
        const int ro[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (v + i < nvec) {
            float* dst = sS + ro[i] + px * TIP + 32 * ct + c;
            dst[0] = acc[r][0][i];
            dst[16] = acc[r][1][i];
          }
      }
    }
    __syncthreads();

    if (mode == kGenDotKeys) {
      // per-component sort keys, rows (b, p)
      for (int r = wave; r < nq * P; r += NW) {
        const int q = r / P, p = r - q * P;
        uint64_t* dst = keys + (static_cast<long>(b0 + q) * P + p) * key_stride + i0;
        for (int i = lane; i < ni; i += 64) dst[i] = make_key(sS[(q * PV + p) * TIP + i], item_of(i));
      }
      continue;
    }

    // 2. units of 16 items of one query, NU at a time
    const int upq_log2 = ti_log2 - 4, nunits = nq << upq_log2;
    for (int u0 = NU * wave; u0 < nunits; u0 += NU * NW) {
      int q[NU], it[NU];
      float s[NU][RUN];
      float out[NU];
      bool live[NU], keep[NU], any = false;
#pragma unroll
      for (int t = 0; t < NU; ++t) {
        const int u = min(u0 + t, nunits - 1);
        q[t] = u >> upq_log2;
        it[t] = 16 * (u & ((1 << upq_log2) - 1)) + c;                            // slot within the tile
        live[t] = u0 + t < nunits && i0 + it[t] < cnt;
        keep[t] = live[t];
        const float* src = sS + (q[t] * PV + RUN * g) * TIP + it[t];
#pragma unroll
        for (int mu = 0; mu < RUN; ++mu) s[t][mu] = src[mu * TIP];
        out[t] = 0.f;
        if (mode == kGenBounded || mode == kGenMaxDot) {
          float mx = -__builtin_nanf(""), mabs = 0.f;   // (nothing but NaN: NaN, which is kept)
#pragma unroll
          for (int mu = 0; mu < RUN; ++mu)
            if (RUN * g + mu < P) {
              mx = fmaxf(mx, s[t][mu]);
              mabs = fmaxf(mabs, fabsf(s[t][mu]));
            }
          out[t] = max_groups(mx);
          if (mode == kGenBounded)   // phi <= m: items that cannot reach the bound
            keep[t] = keep[t] && !(out[t] + bound_margin(max_groups(mabs)) < bound[b0 + q[t]]);
        }
        any = any || keep[t];
      }
      if (gate && __any(any)) {
        f32x4_t l[NU][PT];
#pragma unroll
        for (int t = 0; t < NU; ++t) {
          const float* ax = sAx + it[t] * (PV + 4) + RUN * g;
#pragma unroll
          for (int pt = 0; pt < PT; ++pt) {
            const float4 cq = *reinterpret_cast<const float4*>(sC + q[t] * PV + RUN * g + 4 * pt);   // -inf past P
            const float4 a = *reinterpret_cast<const float4*>(ax + 4 * pt);
            l[t][pt] = f32x4_t{cq.x + a.x, cq.y + a.y, cq.z + a.z, cq.w + a.w};
          }
        }
        for (int jt = 0; jt < JT; ++jt) {
          const float4 bj = *reinterpret_cast<const float4*>(sB1 + 16 * jt + 4 * g);
          f32x4_t u[NU];
#pragma unroll
          for (int t = 0; t < NU; ++t) u[t] = f32x4_t{bj.x, bj.y, bj.z, bj.w};
#pragma unroll
          for (int m4 = 0; m4 < RUN / 4; ++m4) {
            const float4 w = sW1[(jt * (RUN / 4) + m4) * 64 + lane];
#pragma unroll
            for (int t = 0; t < NU; ++t) u[t] = mfma_f32(w.x, s[t][4 * m4 + 0], u[t]);
#pragma unroll
            for (int t = 0; t < NU; ++t) u[t] = mfma_f32(w.y, s[t][4 * m4 + 1], u[t]);
#pragma unroll
            for (int t = 0; t < NU; ++t) u[t] = mfma_f32(w.z, s[t][4 * m4 + 2], u[t]);
#pragma unroll
            for (int t = 0; t < NU; ++t) u[t] = mfma_f32(w.w, s[t][4 * m4 + 3], u[t]);
          }
          // SiLU: u sigma(u), sigma(u) = 1 / (1 + e^-u)
          float h[NU][4];
#pragma unroll
          for (int t = 0; t < NU; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              h[t][i] = u[t][i] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-kLog2e * u[t][i]));
#pragma unroll
          for (int pt = 0; pt < PT; ++pt) {
            const float4 w = sW2[(jt * PT + pt) * 64 + lane];
#pragma unroll
            for (int t = 0; t < NU; ++t) {
              l[t][pt] = mfma_f32(w.x, h[t][0], l[t][pt]);
              l[t][pt] = mfma_f32(w.y, h[t][1], l[t][pt]);
              l[t][pt] = mfma_f32(w.z, h[t][2], l[t][pt]);
              l[t][pt] = mfma_f32(w.w, h[t][3], l[t][pt]);
            }
          }
        }
#pragma unroll
        for (int t = 0; t < NU; ++t) {
          float mx = l[t][0][0];
#pragma unroll
          for (int pt = 0; pt < PT; ++pt)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx = fmaxf(mx, l[t][pt][i]);
          mx = max_groups(mx);
          float den = 0.f, num = 0.f;
#pragma unroll
          for (int pt = 0; pt < PT; ++pt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float w = __builtin_amdgcn_exp2f(kLog2e * (l[t][pt][i] - mx));   // 0 past P
              den += w;
              num = fmaf(w, s[t][4 * pt + i], num);
            }
          out[t] = sum_groups(num) * __builtin_amdgcn_rcpf(sum_groups(den));
        }
      }
      // one lane per item writes; slots past the count are cleared keys
#pragma unroll
      for (int t = 0; t < NU; ++t) {
        if (g != 0 || u0 + t >= nunits || it[t] >= ni) continue;
        const long b = b0 + q[t];
        const int i = i0 + it[t];
        if (!keep[t]) {
          if (phi && live[t]) phi[b * phi_stride + i] = excluded_score();
          if (keys) keys[b * key_stride + i] = 0;
        } else {
          if (phi) phi[b * phi_stride + i] = out[t];
          if (keys) keys[b * key_stride + i] = make_key(out[t], item_of(it[t]));
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Tile shape: QB queries (up to four, eight for P <= 16: whole blocks of
// vectors, and the item rows' reads serve them all) by TI items (a power of
// two, at least 32), with PV QB TI at most f32_tile, or half of that where the
// weights leave no room.
struct F32Plan {
  int QB, TI, ti_log2;
  size_t lds;
};

template <int PV>
static F32Plan f32_plan(const DevProb& pr, bool gate, bool gather) {
  const int JT = gate ? (pr.H + 15) / 16 : 0;
  const size_t weights = 2ul * JT * (PV / 16) * 1024 + 64ul * JT;
  int pairs = f32_tile<PV>() / PV;
  F32Plan f;
  for (;;) {
    f.QB = gather ? 1 : std::min({pr.B, std::max(1, pairs / 32), PV == 16 ? 8 : 4});
    f.TI = 32;
    f.ti_log2 = 5;
    while (2 * f.TI * f.QB <= pairs) {
      f.TI *= 2;
      ++f.ti_log2;
    }
    f.lds = weights + 4ul * (f.QB * PV * (1 + f.TI + s_pad<PV>()) + (gate ? f.TI * (PV + 4) : 0) +
                             (f.QB * pr.Pq + 31) / 32 * 32);
    if (f.lds <= 160 * 1024 || pairs <= 32) return f;
    pairs /= 2;
  }
}

template <typename T, int PV, bool VEC>
static hipError_t launch_f32_k(const DevProb& pr, int mode, const float* bound, int n_begin, int n_count,
                               const int32_t* items, const int32_t* item_count, long item_stride, float* phi,
                               long phi_stride, uint64_t* keys, long key_stride, hipStream_t st) {
  const F32Plan f = f32_plan<PV>(pr, mode != kGenMaxDot && mode != kGenDotKeys, items != nullptr);
  auto kern = &k_mol_f32<T, PV, VEC>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(f.lds));
  if (e != hipSuccess) return e;
  const int nqb = (pr.B + f.QB - 1) / f.QB;
  const long tiles = (static_cast<long>(n_count) + f.TI - 1) / f.TI * nqb;
  // persistent: the weights are laid out once per resident workgroup
  const long resident = 256l * std::max<long>(1, std::min<long>(16 / f32_waves<PV>(), (160 * 1024) / f.lds));
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(std::min(tiles, resident))), dim3(64 * f32_waves<PV>()), f.lds, st, pr,
                     mode, bound, n_begin, n_count, f.QB, f.ti_log2, nqb, tiles, items, item_count, item_stride, phi,
                     phi_stride, keys, key_stride);
  return hipGetLastError();
}

template <typename T, int PV>
static hipError_t launch_f32_v(const DevProb& pr, int mode, const float* bound, int n_begin, int n_count,
                               const int32_t* items, const int32_t* item_count, long item_stride, float* phi,
                               long phi_stride, uint64_t* keys, long key_stride, hipStream_t st) {
  // 16-byte row reads where every row starts on a 16-byte boundary
  const bool vec = (pr.d * sizeof(T)) % 16 == 0 &&
                   ((reinterpret_cast<uintptr_t>(pr.Q) | reinterpret_cast<uintptr_t>(pr.X)) & 15) == 0;
  return vec ? launch_f32_k<T, PV, true>(pr, mode, bound, n_begin, n_count, items, item_count, item_stride, phi,
                                         phi_stride, keys, key_stride, st)
             : launch_f32_k<T, PV, false>(pr, mode, bound, n_begin, n_count, items, item_count, item_stride, phi,
                                          phi_stride, keys, key_stride, st);
}

template <typename T>
static hipError_t launch_f32_t(const DevProb& pr, int mode, const float* bound, int n_begin, int n_count,
                               const int32_t* items, const int32_t* item_count, long item_stride, float* phi,
                               long phi_stride, uint64_t* keys, long key_stride, hipStream_t st) {
  auto f = pr.P <= 16 ? &launch_f32_v<T, 16> : pr.P <= 32 ? &launch_f32_v<T, 32> : &launch_f32_v<T, 64>;
  return f(pr, mode, bound, n_begin, n_count, items, item_count, item_stride, phi, phi_stride, keys, key_stride, st);
}

hipError_t launch_mol_f32(const DevProb& pr, int mode, const float* bound, int n_begin, int n_count,
                          const int32_t* items, const int32_t* item_count, long item_stride, float* phi,
                          long phi_stride, uint64_t* keys, long key_stride, hipStream_t st) {
  if (n_count <= 0) return hipSuccess;
  if (items && mode == kGenDotKeys) return hipErrorInvalidValue;
  auto f = pr.dtype == MOL_BF16 ? &launch_f32_t<bf16_t> : &launch_f32_t<float>;
  return f(pr, mode, bound, n_begin, n_count, items, item_count, item_stride, phi, phi_stride, keys, key_stride, st);
}

}  // namespace mol
