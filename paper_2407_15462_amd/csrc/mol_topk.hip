// Top-k of dense float32 score rows (Definition 1's selection step), one
// workgroup per row, straight to the decoded outputs.
//
// Every thread takes the maximum of its own share of the row (256 or 1024
// disjoint buckets; for k beyond half of them every bucket of bmax, or score,
// counts by itself).  k buckets whose maxima reach T hold k items scoring at
// least T, so T = the k-th largest bucket maximum bounds the row's k-th score
// from below.  Of M buckets, k hold one of the best -M ln(1 - k / M) scores in
// a random order, so about that many items of the row reach T: 105 for k = 100
// of 1024 buckets, 1.65 k where the kernel's rules leave the fewest, M = 1.5 k
// (3,375 of the list's 4,096 slots at k = 2048).  Those are collected in LDS,
// ranked by counting (long lists inside bins of the score range) and written
// out.  A row whose items reaching T exceed the LDS list (massive ties, as a
// query of zeros makes them, or the best items side by side) is finished by a
// radix search over its 64-bit sort keys, 8 bits a pass: it begins at the bits in
// which they can differ, reads only the buckets that reach T while their list
// holds them, and with nothing but ties above only the columns of the first k,
// counts the lanes of one bin with one add and ends where the list holds the
// rest.  (All 64 bits, every score a pass, one add a lane -> now, and the list
// form or the chunked radix selection of keys: 32 rows of 100,000 equal scores
// 721 -> 230, 257 us; a query of zeros against 2^20 items of 8 x 8, d = 64, in
// all, 6,460 -> 284, 653; one ascending row of 2^20 2,069 -> 109, 136.)
//
// What bounds it: one read of the row at a workgroup's rate (about 100 GB/s)
// and a dozen barriers.  With per-bucket maxima from the kernel that scored
// the row (64 items a bucket) it reads those instead, a 64th of the row, and
// then only the items of the buckets that reach T, by the loads a CU can keep
// in flight to memory other CUs wrote (about 20 GB/s with 16 KB of them).
// Measured: top-100 of 32 rows of 109,739 scores 13 us plus 6 us for the
// maxima (chunked radix selection, segmented sort and decode of 64-bit keys:
// 52 us; straight from the rows 61 us), of one row of 2^20 19 us; top-2000 of
// 32 rows of 674,044 71 us.
#include <type_traits>

#include "mol_tile.h"

namespace mol {

namespace {

constexpr int kTopWhole = 128;          // rows of up to this many scores are ranked without a threshold
constexpr int kTopRankMax = 256;        // up to this many keys are ranked by counting, more are sorted
constexpr uint32_t kTopBinMax = 64;     // keys of one bin of the binned sort

// score image, 0 for NaN (which no bound on the k-th score counts)
__device__ __forceinline__ uint32_t score_image(float f) { return f == f ? float_to_ordered(f) : 0u; }

}  // namespace

// phi [rows][phi_stride] (P lists a query: list p of query b is row p * p_rows
// + b, written as row b * P + p), L scores a row (row_len: NULL or the valid count of
// each row); bmax: NULL, or [rows][bmax_stride] bucket maxima; ids: NULL (item
// = column), or the item of each column [rows][ids_stride]; rank_nan: see
// DenseRows.  Rows with fewer than k items are padded with (-inf, -1).
// NT threads a row (1024: two workgroups a CU, at most 64 registers; 8 to 16
// are spilled, in the binned sort and the radix finish).  NEG: the rows are ranked by
// -phi, and that is what is written (a runtime sign is 500 instructions more,
// 0.3 us a call).
template <int NT, bool NEG>
__global__ __launch_bounds__(NT, 8) void k_topk_dense(const float* __restrict__ phi, long phi_stride, int P,
                                                           long p_rows, int L_all,
                                                           const int32_t* __restrict__ row_len,
                                                           const float* __restrict__ bmax, long bmax_stride, int SL,
                                                           const int32_t* __restrict__ ids, long ids_stride, int k,
                                                           int rank_nan, float* __restrict__ out_score,
                                                           int32_t* __restrict__ out_idx) {
  constexpr int kTopThreads = NT;
  constexpr int kTopCap = 4 * NT;        // keys held in LDS
  constexpr int kTopCoarse = NT / 2;     // largest k ranked by the threads' maxima
  constexpr int kTopHot = 4 * NT;        // buckets collected before their items are read
  static_assert(NT >= 256 && NT >= kTopRankMax, "a thread a histogram bin, and a key ranked by counting");
  __shared__ uint64_t buf[kTopCap];
  __shared__ uint32_t hist[256];
  __shared__ int hot[kTopHot];
  __shared__ uint32_t s_hi, s_lo, s_count, s_hot, s_bin, s_above;
  const int tid = threadIdx.x, lane = tid & 63;
  const long row = blockIdx.x;
  // row r is list (b, p) = (r / P, r % P) of a [p][b] layout; P = 1: row r
  const long at = row / P + (row % P) * p_rows;
  const int L = row_len ? min(row_len[row], L_all) : L_all;
  const float* src = phi + at * phi_stride;
  const int32_t* id = ids ? ids + row * ids_stride : nullptr;
  // (a NaN keeps its payload and takes part in the sign)
  auto value = [](float f) { return NEG ? __uint_as_float(__float_as_uint(f) ^ 0x80000000u) : f; };
  // image of a score: 0 for a column that is not ranked
  auto image = [&](float f) {
    const bool ranked = f == f || (rank_nan && __float_as_uint(f) != kExcludedBits);
    return ranked ? float_to_ordered(value(f)) : 0u;
  };
  // f(index of the first, 4 values, how many are valid) over n floats: four
  // consecutive ones a thread and load, or single ones where those would leave
  // threads without a value; U loads in flight
  auto for_values = [&](const float* v0, int n, auto&& f) {
    constexpr int U = 4;
    if (n <= 4 * kTopThreads) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = v0[max(min(tid + u * kTopThreads, n - 1), 0)];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (tid + u * kTopThreads < n) f(tid + u * kTopThreads, float4{v[u], v[u], v[u], v[u]}, 1);
      return;
    }
    const bool vec = (reinterpret_cast<uintptr_t>(v0) & 15) == 0;
    for (int i0 = 4 * tid; i0 < n; i0 += U * 4 * kTopThreads) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * 4 * kTopThreads;
        if (vec && i + 4 <= n) {
          v[u] = *reinterpret_cast<const float4*>(v0 + i);
        } else {
          const int last = n - 1;
          v[u] = float4{v0[min(i, last)], v0[min(i + 1, last)], v0[min(i + 2, last)], v0[min(i + 3, last)]};
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * 4 * kTopThreads;
        if (i < n) f(i, v[u], min(4, n - i));
      }
    }
  };
  const int nb = bmax ? (L + 64 * SL - 1) / (64 * SL) * SL : L;     // values of the first pass
  const float* val = bmax ? bmax + at * bmax_stride : src;

  // the thread's maximum, in floats (values past the end repeat the last one;
  // fmaxf passes NaN over)
  float fm = __builtin_nanf("");
  for_values(val, nb, [&](int, const float4& v, int) {
    fm = fmaxf(fm, fmaxf(fmaxf(value(v.x), value(v.y)), fmaxf(value(v.z), value(v.w))));
  });
  const uint32_t mx = score_image(fm);
  // beyond kTopCoarse every value counts by itself: the thread maxima are too
  // few to hold the k-th
  const bool fine = k > kTopCoarse;
  uint32_t lo_v = mx ? mx : 0xFFFFFFFFu, n_v = mx ? 1u : 0u;   // smallest nonzero image, count
  auto for_images = [&](auto&& f) {                            // f(image) of each value, or of the maximum
    if (!fine) {
      if (mx) f(mx);
      return;
    }
    for_values(val, nb, [&](int, const float4& v4, int nv) {
      const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t im = e < nv ? score_image(value(v[e])) : 0u;
        if (im) f(im);
      }
    });
  };
  if (fine) {
    lo_v = 0xFFFFFFFFu;
    n_v = 0u;
    for_images([&](uint32_t im) {
      lo_v = min(lo_v, im);
      ++n_v;
    });
  }

  // T: the k-th largest of them, to 24 bits below the highest bit in which
  // they differ (the bits left out only lower T); 0 with fewer than k
  if (tid == 0) {
    s_hi = 0u;
    s_lo = 0xFFFFFFFFu;
    s_count = 0u;
  }
  __syncthreads();
  {
    uint32_t hi = mx, lo = lo_v, n = n_v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      hi = max(hi, static_cast<uint32_t>(__shfl_xor(static_cast<int>(hi), o)));
      lo = min(lo, static_cast<uint32_t>(__shfl_xor(static_cast<int>(lo), o)));
      n += static_cast<uint32_t>(__shfl_xor(static_cast<int>(n), o));
    }
    if (lane == 0 && n) {
      atomicMax(&s_hi, hi);
      atomicMin(&s_lo, lo);
      atomicAdd(&s_count, n);
    }
  }
  __syncthreads();
  const uint32_t diff = s_hi ^ s_lo, nonzero = s_count;
  uint32_t T = 0u;
  // rank `kk` (from the top) among the values with image >> shift + 8 equal
  // to the prefix: the bin of `hist` that holds it, found by wave 0
  auto find_bin = [&](uint32_t kk) {
    if (tid < 64) {
      uint32_t h[4], sum = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h[j] = hist[255 - 4 * lane - j];
        sum += h[j];
      }
      uint32_t incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      const uint64_t hit = __ballot(incl >= kk);
      if (hit && lane == __ffsll(static_cast<long long>(hit)) - 1) {
        uint32_t above = incl - sum;
        int bin = 255 - 4 * lane;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (above + h[j] >= kk) {
            bin = 255 - 4 * lane - j;
            break;
          }
          above += h[j];
        }
        s_bin = static_cast<uint32_t>(bin);
        s_above = above;
      }
    }
    __syncthreads();
  };
  if (nonzero >= static_cast<uint32_t>(k) && L > kTopWhole) {   // (a short row is ranked whole)
    uint32_t kk = static_cast<uint32_t>(k);
    int bits = diff ? 32 - __clz(static_cast<int>(diff)) : 0;   // low bits that may differ
    T = bits >= 32 ? 0u : s_hi >> bits << bits;
    for (int pass = 0; pass < 3 && bits > 0; ++pass) {
      const int shift = max(0, bits - 8);
      __syncthreads();
      if (tid < 256) hist[tid] = 0u;
      __syncthreads();
      for_images([&](uint32_t im) {
        if (bits >= 32 || (im >> bits) == (T >> bits))
          atomicAdd(&hist[(im >> shift) & ((1u << (bits - shift)) - 1u)], 1u);
      });
      __syncthreads();
      find_bin(kk);
      kk -= s_above;
      T |= s_bin << shift;
      bits = shift;
    }
  }
  T = max(T, 1u);                                    // image 0: no item

  // every item at or above T
  __syncthreads();
  if (tid == 0) s_count = s_hot = 0u;
  __syncthreads();
  // the float compare decides almost every value; images decide the rest
  const float Tf = T > float_to_ordered(-__builtin_inff()) ? ordered_to_float(T) : -__builtin_inff();
  // f(index, image) of the values at or above T of an array (NaN is looked at)
  auto for_hits = [&](const float* v0, int n, auto&& image_of, auto&& f) {
    for_values(v0, n, [&](int i, const float4& v4, int nv) {
      const float v[4] = {v4.x, v4.y, v4.z, v4.w};
      if (value(v[0]) < Tf && value(v[1]) < Tf && value(v[2]) < Tf && value(v[3]) < Tf) return;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t im = e < nv ? image_of(v[e]) : 0u;
        if (im >= T) f(i + e, im);
      }
    });
  };
  auto key_of = [&](uint32_t u, int col) {
    const int32_t item = id ? id[col] : col;
    return (static_cast<uint64_t>(u) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(item));
  };
  auto collect = [&](int col, uint32_t u) {
    const uint32_t pos = atomicAdd(&s_count, 1u);
    if (pos < static_cast<uint32_t>(kTopCap)) buf[pos] = key_of(u, col);
  };
  // (a bucket of nothing but NaN only where every column counts)
  const auto bucket_image = [&](float f) { return f == f ? float_to_ordered(f) : rank_nan ? 1u : 0u; };
  uint32_t hot_n = kTopHot + 1;
  if (bmax) {
    // the buckets that reach T, then their items, a wave a bucket: the loads
    // of all buckets in flight instead of one bucket's after another's
    for_hits(val, nb, bucket_image, [&](int i, uint32_t) {
      const uint32_t pos = atomicAdd(&s_hot, 1u);
      if (pos < static_cast<uint32_t>(kTopHot)) hot[pos] = i;
    });
    __syncthreads();
    hot_n = s_hot;
    // four loads of W consecutive items a thread in flight (a bucket is runs of 16)
    auto gather = [&](auto wc) {
      constexpr int W = decltype(wc)::value, PB = 64 / W, PR = 16 / W;   // loads per bucket and run
      const int nl = PB * static_cast<int>(hot_n);
      for (int t0 = tid; t0 < nl; t0 += 4 * kTopThreads) {
        float x[4][W];
        int col[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * kTopThreads;
          col[u] = L;
          if (t < nl) {                              // load t % PB of bucket hot[t / PB]
            const int bk = hot[t / PB], blk = bk / SL;
            col[u] = 16 * (4 * SL * blk + (bk - blk * SL) + SL * (t % PB / PR)) + W * (t % PR);
          }
          if (W == 4 && col[u] + W <= L) {
            const float4 q = *reinterpret_cast<const float4*>(src + col[u]);
            const float v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < W; ++e) x[u][e] = v[e];
          } else {
#pragma unroll
            for (int e = 0; e < W; ++e) x[u][e] = src[min(col[u] + e, L - 1)];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < W; ++e) {
            const uint32_t im = col[u] + e < L ? image(x[u][e]) : 0u;
            if (im >= T) collect(col[u] + e, im);
          }
      }
    };
    // 16-byte loads where single ones take more than four rounds of the
    // workgroup, each a trip to memory (about 2,700 buckets, top-2000 of 32
    // rows of 674,044: 92 -> 71 us); for about 105 buckets (k = 100) single
    // loads are 0.6 to 1.3 us faster
    if (hot_n <= static_cast<uint32_t>(kTopHot)) {
      if (hot_n > 256u && (reinterpret_cast<uintptr_t>(src) & 15) == 0)
        gather(std::integral_constant<int, 4>{});
      else
        gather(std::integral_constant<int, 1>{});
    }
  }
  // (one item at least in each of more buckets than the list has places; T > 1: a score)
  const bool over = bmax && hot_n > static_cast<uint32_t>(kTopHot) && T > 1u;
  if (!over && hot_n > static_cast<uint32_t>(kTopHot)) for_hits(src, L, image, collect);
  __syncthreads();
  uint32_t n = over ? kTopCap + 1u : s_count;
  if (__builtin_expect(n > static_cast<uint32_t>(kTopCap), 0)) {
    int cols = L;                                    // the k best lie in the first so many columns
    // f(column, image) of the items at or above T: the buckets' in `hot`, else the columns'
    auto for_items = [&](auto&& f) {
      if (hot_n > static_cast<uint32_t>(kTopHot)) {
        for_hits(src, cols, image, f);
        return;
      }
#pragma unroll 1
      for (int t = tid; t < 64 * static_cast<int>(hot_n); t += kTopThreads) {
        const int bk = hot[t >> 6], blk = bk / SL;
        const int col = 16 * (4 * SL * blk + (bk - blk * SL) + SL * (t >> 4 & 3)) + (t & 15);
        const uint32_t im = col < L ? image(src[col]) : 0u;
        if (im >= T) f(col, im);
      }
    };
    if (rank_nan) {                                  // the largest image may be a NaN's
      uint32_t top = 0u;
      for_items([&](int, uint32_t u) { top = max(top, u); });
      atomicMax(&s_hi, top);
      __syncthreads();
    }
    if (over && s_hi == T) {
      // nothing above T: the k lowest columns at T lie in the first k of those
      // buckets, and a histogram over their places ends the row behind them
      if (tid < 256) hist[tid] = 0u;
      __syncthreads();
      int sh = 0;
      while (nb >> sh >= 256) ++sh;
      for_hits(val, nb, bucket_image, [&](int i, uint32_t) { atomicAdd(&hist[255 - (i >> sh)], 1u); });
      __syncthreads();
      find_bin(static_cast<uint32_t>(k));
      const int last = min(nb, static_cast<int>(256u - s_bin) << sh) - 1;   // a bucket at or behind the k-th
      cols = min(L, 64 * SL * (last / SL + 1));
    }
    // the k-th largest key, 8 bits a pass over the items at or above T (at
    // least k of them: more than kTopCap >= k reach T), from the highest bit in
    // which they can differ until no more than kTopCap keys are left above
    const uint32_t span = s_hi ^ T;                  // images lie in [T, s_hi]
    const int ibits = id ? 32 : 32 - __clz(L);       // items: columns up to L, or any
    int bits = span ? 64 - __clz(static_cast<int>(span)) : ibits;   // low bits of the key that are open
    auto above = [&](uint64_t key) { return bits < 64 ? key >> bits : 0ull; };
    uint64_t prefix = bits < 64 ? above(static_cast<uint64_t>(T) << 32 | 0xFFFFFFFFu) << bits : 0ull;
    uint32_t kk = static_cast<uint32_t>(k);
    while (bits > 0) {
      const int shift = bits > 32 ? max(32, bits - 8) : max(0, bits - 8);
      __syncthreads();
      if (tid < 256) hist[tid] = 0u;
      __syncthreads();
      for_items([&](int col, uint32_t u) {
        const uint64_t key = key_of(u, col);
        if (above(key) != above(prefix)) return;
        // tied scores share a bin: one add for the lanes of the first one's
        const uint32_t bin = static_cast<uint32_t>(key >> shift) & ((1u << (bits - shift)) - 1u);
        const uint32_t lead = __builtin_amdgcn_readfirstlane(bin);
        const uint64_t same = __ballot(bin == lead);
        if (bin != lead) atomicAdd(&hist[bin], 1u);
        else if (lane == __ffsll(static_cast<long long>(same)) - 1) atomicAdd(&hist[bin], __popcll(same));
      });
      __syncthreads();
      find_bin(kk);
      kk -= s_above;
      prefix |= static_cast<uint64_t>(s_bin) << shift;
      bits = shift;
      if (static_cast<uint32_t>(k) - kk + hist[s_bin] <= static_cast<uint32_t>(kTopCap)) break;
      if (bits == 32 && !id) {                       // the items' bits above those of L are set
        prefix |= 0xFFFFFFFFu >> ibits << ibits;
        bits = ibits;
      }
    }
    __syncthreads();
    if (tid == 0) s_count = 0u;
    __syncthreads();
    for_items([&](int col, uint32_t u) {
      const uint64_t key = key_of(u, col);
      if (key >= prefix) {
        const uint32_t pos = atomicAdd(&s_count, 1u);
        if (pos < static_cast<uint32_t>(kTopCap)) buf[pos] = key;
      }
    });
    __syncthreads();
    n = min(s_count, static_cast<uint32_t>(kTopCap));
  }
  float* os = out_score + row * k;
  int32_t* oi = out_idx + row * k;
  const int ni = static_cast<int>(n);
  // More keys than that: a counting pass over kTopHot bins of the image range
  // [T, s_hi] (in descending order, about one key a bin), every key to its
  // bin's slots, and its rank is the bin's start plus the larger keys of the
  // bin.  A dozen barriers where the bitonic network below takes 78 at 4096
  // keys (top-2000 of 32 rows of 674,044: 124 -> 92 us); false, with buf
  // unchanged, if a bin holds more than kTopBinMax keys (ties), which the
  // network then sorts.
  auto sort_binned = [&](int ni) {
    static_assert(kTopCap == kTopHot && kTopCap == 4 * kTopThreads, "four keys and four bins a thread");
    uint32_t* cnt = reinterpret_cast<uint32_t*>(hot);
    const uint32_t span = max(s_hi, T) - T;
    constexpr int kBinBits = 31 - __builtin_clz(kTopHot);
    const int sh = max(0, 32 - kBinBits - __clz(static_cast<int>(span | 1u)));   // span >> sh < kTopHot
#pragma unroll
    for (int j = 0; j < 4; ++j) cnt[tid + j * kTopThreads] = 0u;
    if (tid == 0) s_bin = 0u;
    __syncthreads();
    uint64_t key[4];
    uint32_t b[4], r[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = tid + j * kTopThreads;
      key[j] = i < ni ? buf[i] : 0ull;
      b[j] = r[j] = 0u;
      if (i < ni) {
        const uint32_t u = static_cast<uint32_t>(key[j] >> 32);
        b[j] = kTopHot - 1u - min((u - T) >> sh, kTopHot - 1u);
        r[j] = atomicAdd(&cnt[b[j]], 1u);
      }
    }
    __syncthreads();
    // counts -> first slots
    uint32_t h[4], sum = 0u, most = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      h[j] = cnt[4 * tid + j];
      most = max(most, h[j]);
      sum += h[j];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (most > kTopBinMax) s_bin = 1u;
    if (lane == 63) hist[tid >> 6] = incl;
    __syncthreads();
    if (s_bin) return false;
    uint32_t at0 = incl - sum;
    for (int w = 0; w < (tid >> 6); ++w) at0 += hist[w];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cnt[4 * tid + j] = at0;
      at0 += h[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (tid + j * kTopThreads < ni) buf[cnt[b[j]] + r[j]] = key[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (tid + j * kTopThreads >= ni) continue;
      const int first = static_cast<int>(cnt[b[j]]);
      const int last = b[j] + 1u < static_cast<uint32_t>(kTopHot) ? static_cast<int>(cnt[b[j] + 1]) : ni;
      int rank = first;
      for (int x = first; x < last; ++x) rank += buf[x] > key[j] ? 1 : 0;
      if (rank < k) {
        os[rank] = key_score(key[j]);
        oi[rank] = key_item(key[j]);
      }
    }
    return true;
  };
  if (ni <= kTopRankMax) {
    // a key's rank is the number of larger ones (keys are distinct)
    if (tid < ni) {
      const uint64_t key = buf[tid];
      int rank = 0;
      int j = 0;
      for (; j + 8 <= ni; j += 8) {
        uint64_t o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = buf[j + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) rank += o[e] > key ? 1 : 0;
      }
      for (; j < ni; ++j) rank += buf[j] > key ? 1 : 0;
      if (rank < k) {
        os[rank] = key_score(key);
        oi[rank] = key_item(key);
      }
    }
  } else if (!sort_binned(ni)) {
    int S = 2 * kTopRankMax;
    while (S < ni) S <<= 1;
    for (int i = ni + tid; i < S; i += kTopThreads) buf[i] = 0ull;
    __syncthreads();
    for (int size = 2; size <= S; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = tid; i < S / 2; i += kTopThreads) {
          const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
          const bool desc = (lo & size) == 0;
          const uint64_t a = buf[lo], c = buf[hi];
          if ((a < c) == desc) {
            buf[lo] = c;
            buf[hi] = a;
          }
        }
        __syncthreads();
      }
    for (int i = tid; i < min(k, ni); i += kTopThreads) {
      os[i] = key_score(buf[i]);
      oi[i] = key_item(buf[i]);
    }
  }
  for (int i = ni + tid; i < k; i += kTopThreads) {
    os[i] = -__builtin_inff();
    oi[i] = -1;
  }
}

// Bucket maxima of dense rows (SL = 1: 64 consecutive columns a bucket): a
// lane reads four columns, 16 lanes a bucket.  The rows' strides keep the
// reads aligned and inside the buffer (a multiple of 4 floats).
__global__ __launch_bounds__(256) void k_bucket_max(const float* __restrict__ phi, long phi_stride, int L,
                                                    float* __restrict__ bmax, long bmax_stride) {
  const long row = blockIdx.y;
  const int col = (blockIdx.x * 256 + threadIdx.x) * 4;
  float m = __builtin_nanf("");
  if (col < L) {
    const float4 v = *reinterpret_cast<const float4*>(phi + row * phi_stride + col);
    m = v.x;
    if (col + 1 < L) m = fmaxf(m, v.y);
    if (col + 2 < L) m = fmaxf(m, v.z);
    if (col + 3 < L) m = fmaxf(m, v.w);
  }
  m = tile::row16_max(m);
  if ((threadIdx.x & 15) == 0 && col < L) bmax[row * bmax_stride + (col >> 6)] = m;
}

hipError_t launch_bucket_max(const float* phi, long phi_stride, int rows, int L, float* bmax, long bmax_stride,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_bucket_max, dim3((L + 1023) / 1024, rows), dim3(256), 0, st, phi, phi_stride, L, bmax,
                     bmax_stride);
  return hipGetLastError();
}

// Threads a row.  With more rows than the chip holds of the large workgroups
// (two a CU), the small ones (eight a CU) give every CU more rows in flight;
// rows of up to four values a thread gain by their cheaper barriers at any
// count, rows of up to 3,072 scores from more than one row a CU on.  Longer
// rows only for k <= 128, the small workgroup's coarse threshold; rows that its
// list holds whole up to k = 512, while its share of the ranking stays the
// smaller part.
// Top-10, the dots before it included, 1024 -> 256 threads: 32 rows of 1000
// 13.4 -> 12.2 us, of 2196 15.4 -> 16.4 (left large); 300 rows of 2196 27.6 ->
// 26.2, of 4096 36.1 -> 35.7 and for k = 128 38.2 -> 38.9 (left large); 600 of
// 8192 40.8 -> 32.7, 2000 of 16,000 104 -> 100, 5000 of 300 79 -> 30, 20,000 of
// 1000 314 -> 100; 1000 of 60,000 (bucket maxima) 90 -> 80.
// k of L whole rows, the same way: 3000 rows, 172 of 172 69.5 -> 36.9 us, 200 of
// 700 99.5 -> 67.6, 512 of 1000 122 -> 94; 800 rows, 512 of 1000 44.4 -> 40.5,
// 600 of 1000 48 -> 53; 300 rows, 200 of 700 20.5 -> 19.2, 512 of 1000 26.2 ->
// 30.2 (these three left large).
constexpr int kTopSmall = 256, kTopLarge = 1024;
static int topk_threads(int rows, int L, int k) {
  const bool whole = L <= 4 * kTopSmall, many = rows > 512 || (rows > 256 && L <= 3 * kTopLarge);
  if (k <= kTopSmall / 2) return whole || many ? kTopSmall : kTopLarge;
  return whole && rows > 512 && k <= 2 * kTopSmall ? kTopSmall : kTopLarge;
}

hipError_t launch_topk_dense(const DenseRows& r, int rows, int k, float* out_score, int32_t* out_idx,
                             hipStream_t st) {
  if (k > kTopkDenseMaxK) return hipErrorInvalidValue;
  const int nt = topk_threads(rows, r.L, k);
  auto kern = nt == kTopSmall ? (r.negate ? &k_topk_dense<kTopSmall, true> : &k_topk_dense<kTopSmall, false>)
                              : (r.negate ? &k_topk_dense<kTopLarge, true> : &k_topk_dense<kTopLarge, false>);
  hipLaunchKernelGGL(kern, dim3(rows), dim3(nt), 0, st, r.phi, r.phi_stride, r.P, r.p_rows, r.L, r.row_len, r.bmax,
                     r.bmax_stride, r.SL, r.ids, r.ids_stride, k, r.rank_nan ? 1 : 0, out_score, out_idx);
  return hipGetLastError();
}

}  // namespace mol
