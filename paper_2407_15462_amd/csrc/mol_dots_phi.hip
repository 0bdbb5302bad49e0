// Dense MoL scores for P_x = 4, P <= 16 (P_q 1, 2 or 4), any d that is a
// multiple of 32 and H <= 128, bf16: the component dot products and the
// gating chain of Eq. 1 / Eq. 2 in one kernel, for the shapes the fused
// P_q = 8 kernels do not cover (question answering: 4 x 4 components of width
// 768).
//
// What bounds it: reading X once (0.67 GB at 109,739 items of 4 x 768: 0.14 ms)
// and, next to it, the gating chain's vector instructions. As two kernels the
// dot products were written and read back once more (0.22 GB each way) and
// neither kernel's memory or vector work ran under the other's: 0.20 + 0.14 ms,
// 0.006 ms for the bucket maxima that this kernel writes itself.
//
// Workgroup: a 64-item x TV-vector tile (TV = 32, 64 or 128 vectors: whole
// queries), every wave 32 items x 32 NJ vectors for all four item components
// at once (32x32x16 bf16 MFMAs: 64 NJ accumulator registers), so that a query
// vector's K chunk is read from LDS once for four items' worth of matrix work.
// K is walked 32 at a time through a three-deep ring of direct global -> LDS
// copies, two workgroups a CU: 64 KB of X in flight per CU cover HBM's latency.
// Rows of 64 bytes are XOR-swizzled by chunk so that the 16 rows a 16-lane
// group reads lie in distinct 16-byte bank slots.
//
// Then each wave passes its own accumulators through LDS, 16 items and 32
// vectors at a time, into the layout of the K = 16 gating chain (MolMlp16:
// lane (item c, g) holds p = 4 g + e, i.e. P_q component g and P_x component
// e), and scores them two queries per call.  The dot products' accumulation
// order and the chain are those of the two-kernel path: the same scores bit
// for bit.
#include "mol_tile.h"

namespace mol {

using namespace tile;

namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16_t mfma32x16(uint4 a, uint4 b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

template <int NJ, int WV>
struct DotsPhiShape {
  static constexpr int PX = 4, TI = 64, KS = 32;
  static constexpr int W = 2 * WV;                     // waves: item half x vector group
  static constexpr int TV = 32 * NJ * WV;
  static constexpr int XB = PX * TI * KS * 2, QB = TV * KS * 2, STAGE = XB + QB;
  static constexpr int RING = 3;
  static constexpr int LOADS = STAGE / 1024 / W;       // copies per wave and stage
  static constexpr int RS = 20;                        // floats per s row: 16 items + 4
  static constexpr int SWAVE = 32 * PX * RS * 4;       // bytes of a wave's s region
  static constexpr int LDS_MAIN = RING * STAGE > W * SWAVE ? RING * STAGE : W * SWAVE;
  static constexpr int LDS_AQ = TV * 4 * 4;            // a_q rows of the tile's TV / P_q queries
  static constexpr int LDS_MAX = 2 * TV * 4;           // per (item half, query) maxima
  static constexpr int LDS_TOTAL = LDS_MAIN + LDS_AQ + LDS_MAX;
  static_assert(STAGE % (1024 * W) == 0, "whole copies");
  static_assert(2 * LDS_TOTAL <= 160 * 1024, "two workgroups a CU");
};

}  // namespace

// phi [B][phi_stride], bmax NULL or [B][bmax_stride] (64-item buckets);
// BOUNDED: items that cannot reach bound[b] get excluded_score().
template <int NJ, int WV, int HV, bool BOUNDED, bool X2>
__global__ __launch_bounds__(128 * WV, 2) void k_dots_phi(DevProb pr, const float* __restrict__ bound, int ny,
                                                         float* __restrict__ phi, long phi_stride,
                                                         float* __restrict__ bmax, long bmax_stride) {
  using S = DotsPhiShape<NJ, WV>;
  using Mlp = MolMlp16<HV, X2>;
  constexpr int PX = S::PX;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* sAq = reinterpret_cast<float*>(smem + S::LDS_MAIN);            // [query][P]
  float* sMax = sAq + S::TV * 4;                                        // [item half][query]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int c = lane & 31, h = lane >> 5;
  const int tile = blockIdx.x / ny, i0 = tile * S::TI;
  const int v0 = (blockIdx.x % ny) * S::TV;
  const int Pq = pr.Pq, P = pr.P, N = pr.N, D = pr.d;
  const int nvec = pr.B * Pq;
  const int b0 = v0 / Pq, nq = min(S::TV / Pq, pr.B - b0);              // queries of the tile
  const bf16_t* X = static_cast<const bf16_t*>(pr.X);
  const bf16_t* Q = static_cast<const bf16_t*>(pr.Q);

  // copy blocks of 16 rows of 64 bytes: 4 per item component, then the
  // vectors'; lane l holds row l / 4's chunk (l % 4) ^ (row / 4) % 4
  const bf16_t* src[S::LOADS];
#pragma unroll
  for (int i = 0; i < S::LOADS; ++i) {
    const int blk = wave + S::W * i, row = lane >> 2, cc = (lane & 3) ^ ((lane >> 4) & 3);
    if (blk < 4 * PX) {
      const int item = min(i0 + 16 * (blk & 3) + row, N - 1);           // past the end: never stored
      src[i] = X + (static_cast<long>(blk >> 2) * N + item) * D + 8 * cc;
    } else {
      src[i] = Q + static_cast<long>(min(v0 + 16 * (blk - 4 * PX) + row, nvec - 1)) * D + 8 * cc;
    }
  }
  auto stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < S::LOADS; ++i) {
      copy16_to_lds(src[i], lds_addr(smem + buf * S::STAGE + (wave + S::W * i) * 1024));
      src[i] += S::KS;
    }
  };
  const int nk = D / S::KS;
  stage(0);
  if (nk > 1) stage(1);
  for (int i = tid; i < nq * P; i += 64 * S::W) sAq[i] = pr.a_q[static_cast<long>(b0) * P + i];

  // the gating operands (their conversion to float16 waits here for their reads,
  // and for the first two stages with them)
  const int ci = lane & 15, g = lane >> 4;
  Mlp mlp;
  mlp.load_padded(pr, ci, g);

  f32x16_t acc[PX][NJ];
#pragma unroll
  for (int px = 0; px < PX; ++px)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[px][j] = f32x16_t{};
  for (int t = 0, cur = 0; t < nk; ++t) {
    // stage t has landed (t + 1 may be in flight) and every wave is done with
    // stage t - 1, whose buffer takes stage t + 2
    if (t + 1 < nk) ring_barrier<S::LOADS>();
    else ring_barrier<0>();
    if (t + 2 < nk) stage(cur == 0 ? 2 : cur - 1);
    const unsigned char* xs = smem + cur * S::STAGE;
    const unsigned char* qs = xs + S::XB;
    const int n = 32 * wm + c;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      uint4 bv[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int r = 32 * (NJ * wn + j) + c;
        bv[j] = *reinterpret_cast<const uint4*>(qs + r * 64 + 16 * ((2 * kb + h) ^ ((r >> 2) & 3)));
      }
#pragma unroll
      for (int px = 0; px < PX; ++px) {
        const uint4 a =
            *reinterpret_cast<const uint4*>(xs + px * (S::TI * 64) + n * 64 + 16 * ((2 * kb + h) ^ ((n >> 2) & 3)));
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[px][j] = mfma32x16(a, bv[j], acc[px][j]);
      }
    }
    cur = cur == 2 ? 0 : cur + 1;
  }
  __syncthreads();                                      // the ring becomes the waves' s regions

  float b2v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) b2v[e] = kLog2e * pr.b2[min(4 * g + e, P - 1)];
  const int gp = min(g, Pq - 1);                        // padded components read a valid row, masked below
  const bool comp = g < Pq;
  float* sw = reinterpret_cast<float*>(smem + wave * S::SWAVE);
  const int qpb = 32 / Pq;                              // queries per block of 32 vectors (even)
#pragma unroll
  for (int rd = 0; rd < 2; ++rd) {
    const int item = i0 + 32 * wm + 16 * rd + ci;
    const bool live = item < N;
    float ax[4];                                        // (any alignment)
    __builtin_memcpy(ax, pr.a_x + static_cast<long>(min(item, N - 1)) * P + 4 * gp, sizeof ax);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      // lane (c, h) holds vector c's items 8 k + 4 h + i: those of this round
      wave_lds_sync();
#pragma unroll
      for (int px = 0; px < PX; ++px)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int e = 4 * (2 * rd + k);
          *reinterpret_cast<float4*>(sw + (c * PX + px) * S::RS + 8 * k + 4 * h) =
              float4{acc[px][j][e], acc[px][j][e + 1], acc[px][j][e + 2], acc[px][j][e + 3]};
        }
      wave_lds_sync();
      const int q0 = (NJ * wn + j) * qpb;               // first query of the block, within the tile
      // the next pair's reads go out before a pair's chain, which covers their
      // latency
      struct Pair {
        float s[2][4];
        float4 aq[2];
      };
      auto fetch = [&](int q, Pair& p) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int qs = min(q, qpb - 2) + u;
          const float* sr = sw + (qs * Pq + gp) * PX * S::RS + ci;
#pragma unroll
          for (int e = 0; e < 4; ++e) p.s[u][e] = sr[e * S::RS];
          p.aq[u] = *reinterpret_cast<const float4*>(sAq + min(q0 + qs, nq - 1) * P + 4 * gp);
        }
      };
      Pair nx;
      fetch(0, nx);
      for (int q = 0; q < qpb && q0 + q < nq; q += 2) {
        const Pair cu = nx;
        fetch(q + 2, nx);
        float s[2][4];
        f32x4_t c0[2][1];
        bool keep[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {                   // (a query past the batch: computed, never stored)
          const float aq[4] = {cu.aq[u].x, cu.aq[u].y, cu.aq[u].z, cu.aq[u].w};
          float m = -__builtin_inff(), mabs = 0.f;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s[u][e] = live && comp ? cu.s[u][e] : 0.f;
            c0[u][0][e] = comp ? fmaf(kLog2e, ax[e] + aq[e], b2v[e]) : -__builtin_inff();
            if (BOUNDED && comp) {
              m = fmaxf(m, s[u][e]);
              mabs = fmaxf(mabs, fabsf(s[u][e]));
            }
          }
          keep[u] = live;
          if (BOUNDED)
            keep[u] = live && !(max_groups(m) + bound_margin(max_groups(mabs)) < bound[b0 + min(q0 + q + u, nq - 1)]);
        }
        // out[u] is valid in rows 2 u and 2 u + 1
        float out[2] = {0.f, 0.f};
        if (!BOUNDED || __any(keep[0] || keep[1])) mlp.template phi<2>(s, c0, out);
        const int u = g >> 1, ql = q0 + q + u;
        const bool kept = u == 0 ? keep[0] : keep[1];
        const float v = kept ? (u == 0 ? out[0] : out[1]) : excluded_score();
        const bool mine = (g & 1) == 0 && ql < nq;
        if (mine && live) phi[(b0 + ql) * phi_stride + item] = v;
        if (bmax) {
          const float m = row16_max(v);
          if (mine && ci == 0) {
            float* mx = sMax + wm * S::TV + ql;
            *mx = rd == 0 ? m : fmaxf(*mx, m);
          }
        }
      }
    }
  }
  if (bmax) {
    __syncthreads();
    for (int q = tid; q < nq; q += 64 * S::W) bmax[(b0 + q) * bmax_stride + tile] = fmaxf(sMax[q], sMax[S::TV + q]);
  }
}

// ---------------------------------------------------------------------------
bool dots_phi_supported(const DevProb& pr) {
  return phi_mfma_supported(pr) && dots_mfma_supported(pr) && pr.Px == 4 &&
         (pr.Pq == 1 || pr.Pq == 2 || pr.Pq == 4);
}

template <int NJ, int WV, int HV>
static hipError_t launch_dots_phi_t(const DevProb& pr, const float* bound, float* phi, long phi_stride, float* bmax,
                                    long bmax_stride, hipStream_t st) {
  using S = DotsPhiShape<NJ, WV>;
  const bool x2 = pr.flags & MOL_FLAG_BF16X2_GATING;
  auto kern = bound ? (x2 ? &k_dots_phi<NJ, WV, HV, true, true> : &k_dots_phi<NJ, WV, HV, true, false>)
                    : (x2 ? &k_dots_phi<NJ, WV, HV, false, true> : &k_dots_phi<NJ, WV, HV, false, false>);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_TOTAL);
  if (e != hipSuccess) return e;
  // the vector tiles of an item tile are neighbours in the grid: they run
  // together and meet in the last-level cache
  const int ny = (pr.B * pr.Pq + S::TV - 1) / S::TV;
  const long tiles = (static_cast<long>(pr.N) + S::TI - 1) / S::TI;
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(tiles * ny)), dim3(64 * S::W), S::LDS_TOTAL, st, pr, bound, ny,
                     phi, phi_stride, bmax, bmax_stride);
  return hipGetLastError();
}

template <int HV>
static hipError_t launch_dots_phi_h(const DevProb& pr, const float* bound, float* phi, long phi_stride, float* bmax,
                                    long bmax_stride, hipStream_t st) {
  // the smallest tile that holds the batch's vectors, at most 128 (64 with
  // H = 128, whose operands leave no registers for two vector blocks a wave)
  const int nvec = pr.B * pr.Pq;
  if (nvec <= 32) return launch_dots_phi_t<1, 1, HV>(pr, bound, phi, phi_stride, bmax, bmax_stride, st);
  if constexpr (HV > 64) {
    return launch_dots_phi_t<1, 2, HV>(pr, bound, phi, phi_stride, bmax, bmax_stride, st);
  } else {
    if (nvec <= 64) return launch_dots_phi_t<2, 1, HV>(pr, bound, phi, phi_stride, bmax, bmax_stride, st);
    return launch_dots_phi_t<2, 2, HV>(pr, bound, phi, phi_stride, bmax, bmax_stride, st);
  }
}

hipError_t launch_dots_phi(const DevProb& pr, const float* bound, float* phi, long phi_stride, float* bmax,
                           long bmax_stride, hipStream_t st) {
  auto f = pr.H <= 32 ? &launch_dots_phi_h<32> : pr.H <= 64 ? &launch_dots_phi_h<64> : &launch_dots_phi_h<128>;
  return f(pr, bound, phi, phi_stride, bmax, bmax_stride, st);
}

}  // namespace mol
