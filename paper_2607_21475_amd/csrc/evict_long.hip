// evict_long.hip -- the Poisson sampler for long units of launches that cannot fill the chip with a
// work-group per unit (one layer of a few long-context sequences).  The same selection as
// evict_select, every pass over the scores spread over the whole chip by segments of kSegRows
// tokens:
//   evict_long_zero   clears the histograms and flags in the workspace
//   evict_long_hist   per segment, a histogram of its positive tail scores in LDS, added to the
//                     unit's.  A bin counts its scores and adds up their low mantissa bits; scores of
//                     a bin share their other bits, so counts and sums are exact integers
//                     whatever the order of the additions
//   evict_long_solve  one work-group per unit: lambda.  The bins that the two clipping thresholds
//                     1 / lambda and eps / lambda cannot touch enter g(lambda) by their exact sums;
//                     the scores of the few bins around them are picked out of the unit once
//                     and classified exactly in every Newton pass
//   evict_long_count  per segment, how many of its tokens the mask keeps
//   evict_long_write  per segment, the mask again, the retained rows' pi and positions at their
//                     final slots, and the gather of their K and V rows
// A work-group per unit spent 250 us on 32 units of 131072 tokens before the first row was gathered,
// and then gathered with 32 of the 256 CUs (513 us together).
#include "ebd.h"
#include "ebd_device.hpp"
#include "ebd_internal.hpp"
#include "evict_common.hpp"

namespace ebd {

namespace {

constexpr int kSegThreads = 256;
constexpr int kSegQuads = kSegRows / (4 * kSegThreads);  // groups of 4 tokens per thread
constexpr int kSolveThreads = 1024;
constexpr int kSolveList = 16384;  // scores around the thresholds kept in LDS
constexpr int kBinReach = 2;       // bins collected on either side of a threshold's

// Workspace of a unit: the histogram (count << 40 | sum of the low kHistShift mantissa bits per
// bin), a header, then the segments' retained counts.
constexpr int kLowBits = 40;
struct LongHeader {
  uint32_t bad;
  float lamf;
  uint32_t st;
  uint32_t pad[13];
};

struct UnitWs {
  unsigned long long *hist;
  LongHeader *hdr;
  int32_t *seg;
};

__device__ __forceinline__ UnitWs unit_ws(const EvictLaunch &L, int u) {
  char *p = L.ws + (int64_t)u * L.ws_unit;
  return {reinterpret_cast<unsigned long long *>(p),
          reinterpret_cast<LongHeader *>(p + kHistBins * sizeof(unsigned long long)),
          reinterpret_cast<int32_t *>(p + kHistBins * sizeof(unsigned long long) + sizeof(LongHeader))};
}

struct Unit {
  int64_t base, n, cbase, cap;
  bool ok;  // within what the launch was planned for
};

__device__ __forceinline__ Unit load_unit(const EvictLaunch &L, int u) {
  Unit U;
  U.base = L.seq_off[u];
  U.n = L.seq_off[u + 1] - U.base;
  U.cbase = L.cap_off[u];
  U.cap = L.cap_off[u + 1] - U.cbase;
  U.ok = U.n <= L.max_rows && U.cap <= (int64_t)L.copy_blocks * kCopyRows;
  return U;
}

// The scores of the group of 4 tokens at token i of a unit (0 past its end).
__device__ __forceinline__ float4 load4(const float *sc, int64_t i, int64_t n, bool vec) {
  if (vec && i + 3 < n) return *reinterpret_cast<const float4 *>(sc + i);
  float4 r;
  r.x = i < n ? sc[i] : 0.0f;
  r.y = i + 1 < n ? sc[i + 1] : 0.0f;
  r.z = i + 2 < n ? sc[i + 2] : 0.0f;
  r.w = i + 3 < n ? sc[i + 3] : 0.0f;
  return r;
}

// Sum of a bin's scores: they share the bits above kHistShift.
__device__ __forceinline__ double bin_sum(int b, unsigned long long v) {
  const int e = b >> (23 - kHistShift);
  const uint32_t top = ((uint32_t)b << kHistShift) & 0x7fffffu;
  const double mant = (double)(v >> kLowBits) * (double)(e ? top + 0x800000u : top) +
                      (double)(v & ((1ull << kLowBits) - 1));
  return ldexp(mant, (e ? e : 1) - 150);
}

__device__ __forceinline__ float bin_low(int b) { return __uint_as_float((uint32_t)b << kHistShift); }
__device__ __forceinline__ int bin_of(float x) { return (int)(__float_as_uint(x) >> kHistShift); }

}  // namespace

__global__ __launch_bounds__(256) void evict_long_zero_kernel(EvictLaunch L) {
  const int64_t words = (kHistBins * sizeof(unsigned long long) + sizeof(LongHeader)) / sizeof(uint4);
  const int64_t per = (words + 256 * 4 - 1) / (256 * 4);  // work-groups per unit
  const int u = (int)(blockIdx.x / per);
  uint4 *p = reinterpret_cast<uint4 *>(L.ws + (int64_t)u * L.ws_unit);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = (blockIdx.x % per) * 1024 + k * 256 + threadIdx.x;
    if (i < words) p[i] = make_uint4(0u, 0u, 0u, 0u);
  }
}

__global__ __launch_bounds__(kSegThreads) void evict_long_hist_kernel(EvictLaunch L) {
  __shared__ unsigned long long s_h[kHistBins];
  const int u = blockIdx.x / L.segs, sg = blockIdx.x % L.segs, t = threadIdx.x;
  const Unit U = load_unit(L, u);
  const int64_t i0 = (int64_t)sg * kSegRows;
  if (!U.ok || i0 >= U.n) return;
  const float *sc = L.scores + U.base;
  const bool vec = (U.base & 3) == 0;
  float4 raw[kSegQuads];
#pragma unroll
  for (int q = 0; q < kSegQuads; ++q) raw[q] = load4(sc, i0 + 4 * (q * kSegThreads + t), U.n, vec);
  for (int b = t; b < kHistBins; b += kSegThreads) s_h[b] = 0ull;
  __syncthreads();
  uint32_t bad = 0;
  const int64_t tail_lo = L.n_sink, tail_hi = U.n - (int64_t)L.n_recent;
#pragma unroll
  for (int q = 0; q < kSegQuads; ++q) {
    const float v[4] = {raw[q].x, raw[q].y, raw[q].z, raw[q].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = i0 + 4 * (q * kSegThreads + t) + j;
      const float c = clean_score(v[j], bad);  // past the end: 0, which is not bad
      if (c > 0.0f && i >= tail_lo && i < tail_hi) {
        const uint32_t w = __float_as_uint(c);
        atomicAdd(&s_h[w >> kHistShift],
                  (1ull << kLowBits) | (unsigned long long)(w & ((1u << kHistShift) - 1u)));
      }
    }
  }
  const UnitWs W = unit_ws(L, u);
  if (__any(bad != 0u) && (t & 63) == 0) atomicOr(&W.hdr->bad, 1u);
  __syncthreads();
  for (int b = t; b < kHistBins; b += kSegThreads) {
    const unsigned long long v = s_h[b];
    if (v) atomicAdd(&W.hist[b], v);
  }
}

__global__ __launch_bounds__(kSolveThreads) void evict_long_solve_kernel(EvictLaunch L) {
  constexpr int NT = kSolveThreads, NW = NT / 64, PER = kHistBins / NT;
  extern __shared__ float s_list[];  // [kSolveList]
  __shared__ double s_ps[NT + 1];    // scores below bin PER t: their sum
  __shared__ int s_pc[NT + 1];       // ... and their number
  __shared__ double s_red[2][NW][3];
  __shared__ int s_edge[2], s_best, s_n;
  const int u = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const Unit U = load_unit(L, u);
  const UnitWs W = unit_ws(L, u);
  if (!U.ok) return;
  const double f = L.budget_per_unit ? (double)L.budget_per_unit[u] : (double)L.budget_frac;
  const double m = f * (double)U.n - (double)min(U.n, (int64_t)L.n_sink + (int64_t)L.n_recent);
  const float eps = L.pi_min;
  const int64_t tail_lo = L.n_sink, tail_hi = U.n - (int64_t)L.n_recent;
  const double n_tail = (double)max(tail_hi - tail_lo, (int64_t)0);
  int rb = 0;
  // The work-group's totals of two counts (below 2^24: they share one exact double) and two sums.
  auto bsum = [&](int a, int b, double c, double d, double &A, double &B, double &C, double &D) {
    double x = wave_sum((double)a + (double)b * 16777216.0);
    c = wave_sum(c);
    d = wave_sum(d);
    if (lane == 0) {
      s_red[rb][wv][0] = x;
      s_red[rb][wv][1] = c;
      s_red[rb][wv][2] = d;
    }
    __syncthreads();
    x = C = D = 0.0;
    for (int w = 0; w < NW; ++w) {
      x += s_red[rb][w][0];
      C += s_red[rb][w][1];
      D += s_red[rb][w][2];
    }
    B = floor(x * (1.0 / 16777216.0));
    A = x - B * 16777216.0;
    rb ^= 1;
  };

  // Prefixes of (count, sum) over the bins, PER bins per thread, in a fixed order.
  if (t == 0) {
    s_edge[0] = kHistBins;
    s_edge[1] = -1;
    s_best = -1;
  }
  unsigned long long hv[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) hv[k] = W.hist[PER * t + k];
  int ct = 0;
  double st_ = 0.0;
  int first = kHistBins, last = -1;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    ct += (int)(hv[k] >> kLowBits);
    if (hv[k]) {
      st_ += bin_sum(PER * t + k, hv[k]);
      first = min(first, PER * t + k);
      last = PER * t + k;
    }
  }
  int ic = ct;
  double is = st_;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int yc = __shfl_up(ic, o);
    const double ys = __shfl_up(is, o);
    if (lane >= o) {
      ic += yc;
      is += ys;
    }
  }
  if (lane == 63) {
    s_red[1][wv][0] = (double)ic;
    s_red[1][wv][1] = is;
  }
  __syncthreads();
  {
    double pc = 0.0, ps = 0.0;
    for (int w = 0; w < wv; ++w) {
      pc += s_red[1][w][0];
      ps += s_red[1][w][1];
    }
    s_pc[t] = (int)pc + ic - ct;
    s_ps[t] = ps + (is - st_);
    if (t == NT - 1) {
      s_pc[NT] = (int)pc + ic;
      s_ps[NT] = ps + is;
    }
  }
  if (last >= 0) {
    atomicMin(&s_edge[0], first);
    atomicMax(&s_edge[1], last);
  }
  __syncthreads();
  const double n_pos = (double)s_pc[NT], s_sum = s_ps[NT];
  const double n_zero = n_tail - n_pos;
  uint32_t st = W.hdr->bad ? EBD_ST_BAD_SCORE : 0u;
  const TailStats ts{n_tail, n_pos, s_sum, 0.0f, 0.0f};
  double lam = 0.0;
  if (!lambda_boundary(ts, m, eps, L.pi_mode, st, lam)) {
    // n_pos > 0 here (an interior lambda).  The bracket from the outermost bins' edges.
    const double lo0 = (double)eps / (double)bin_low(s_edge[1] + 1);
    const double hi0 = 1.0 / fmax((double)bin_low(s_edge[0]), 1e-45);
    // Start: the highest bin edge x whose g(1 / x) still reaches m (the lower threshold's bin taken
    // to the nearest of the PER-bin prefixes), then the linear solve of the piece above it.
    auto piece = [&](int k, int pc, double ps, double &H, double &Lo, double &S) {
      const int be = bin_of(eps * bin_low(PER * t + k)) / PER;
      H = n_pos - (double)pc;
      Lo = (double)s_pc[be] + n_zero;
      S = ps - s_ps[be];
    };
    int best = -1;
    {
      int pc = s_pc[t];
      double ps = s_ps[t];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        double H, Lo, S;
        piece(k, pc, ps, H, Lo, S);
        const double x = (double)bin_low(PER * t + k);
        if (hv[k] && x > 0.0 && H + (double)eps * Lo + S / x >= m) best = PER * t + k;
        pc += (int)(hv[k] >> kLowBits);
        ps += bin_sum(PER * t + k, hv[k]);
      }
    }
    if (best >= 0) atomicMax(&s_best, best);
    __syncthreads();
    best = s_best;
    if (best >= 0 && best / PER == t) {  // its owner solves the piece with the bin in the middle
      int pc = s_pc[t];
      double ps = s_ps[t];
      for (int k = 0; k <= best % PER; ++k) {
        pc += (int)(hv[k] >> kLowBits);
        ps += bin_sum(PER * t + k, hv[k]);
      }
      double H, Lo, S;
      piece(best % PER, pc, ps, H, Lo, S);
      const double top = 1.0 / (double)bin_low(best);
      const double x = S > 0.0 ? (m - H - (double)eps * Lo) / S : top;
      s_red[0][0][0] = (x > 0.0 && x <= top) ? x : top;
    }
    __syncthreads();
    const double start = best >= 0 ? s_red[0][0][0] : m / s_sum;
    __syncthreads();

    // What the list of scores around the thresholds covers, and g's terms of everything else.  The
    // list's order follows its atomics.  The middle scores of the upper threshold's bins (from `split`
    // on) and those of the lower one's are summed apart: five bins share two exponents, so up to
    // kSolveList of their scores are summed exactly in double (40 bits), in any order, however far
    // apart eps puts the two.
    const float *sc = L.scores + U.base;
    const bool vec = (U.base & 3) == 0;
    int c1 = -1, c0 = -1;  // bins of the thresholds it was collected around
    bool listed = false;
    double bH = 0.0, bL = 0.0, bS = 0.0;
    float split = 0.0f;
    auto for_tail = [&](auto &&fn) {  // every cleaned tail score
      const int64_t nq = (U.n + 3) / 4;
      for (int64_t g0 = 0; g0 < nq; g0 += 4 * NT) {
        float4 raw[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[q] = load4(sc, 4 * (g0 + q * NT + t), U.n, vec);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float v[4] = {raw[q].x, raw[q].y, raw[q].z, raw[q].w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t i = 4 * (g0 + q * NT + t) + j;
            uint32_t b = 0;
            const float c = clean_score(v[j], b);
            if (i >= tail_lo && i < tail_hi) fn(c);
          }
        }
      }
    };
    auto collect = [&](int b1, int b0) {
      c1 = b1;
      c0 = b0;
      split = bin_low(max(b1 - kBinReach, 0));
      const int r1 = b1 - kBinReach, R1 = b1 + kBinReach, r0 = b0 - kBinReach, R0 = b0 + kBinReach;
      if (t == 0) s_n = 0;
      __syncthreads();
      for_tail([&](float c) {
        const int b = bin_of(c);
        if (c > 0.0f && ((b >= r1 && b <= R1) || (b >= r0 && b <= R0))) {
          const int k = atomicAdd(&s_n, 1);
          if (k < kSolveList) s_list[k] = c;
        }
      });
      int H = 0, Lo = 0;
      double S = 0.0, none;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int b = PER * t + k;
        if (b > R1) H += (int)(hv[k] >> kLowBits);
        else if (b < r0) Lo += (int)(hv[k] >> kLowBits);
        else if (b > R0 && b < r1) S += bin_sum(b, hv[k]);
      }
      bsum(H, Lo, S, 0.0, bH, bL, bS, none);  // its barrier also completes the list
      bL += n_zero;
      listed = s_n <= kSolveList;
    };
    auto pass = [&](float lf, double &dH, double &dL, double &dS, PieceEdges &edges) {
      edges.valid = false;
      // the thresholds' bins; a score within rounding of a threshold lies in them or beside them
      // (a threshold beyond the bins' range is met by reading every score)
      const bool far = !(1.0f / lf < 1.0e38f);
      const int b1 = far ? 0 : bin_of(1.0f / lf), b0 = far ? 0 : bin_of(eps / lf);
      if (!far && (c1 < 0 || (listed && (abs(b1 - c1) >= kBinReach || abs(b0 - c0) >= kBinReach)))) {
        __syncthreads();  // every thread is done with the list
        collect(b1, b0);
      }
      int H = 0, Lo = 0;
      double S1 = 0.0, S0 = 0.0;  // the middle at and above `split`, and below it
      auto add = [&](float s) {
        const float p = lf * s;
        const bool hb = p >= 1.0f, lb = p <= eps;
        H += hb ? 1 : 0;
        Lo += lb ? 1 : 0;
        const double mid = (hb || lb) ? 0.0 : (double)s;
        if (s >= split) S1 += mid;
        else S0 += mid;
      };
      const bool from_list = !far && listed;
      if (from_list) {
        for (int i = t; i < s_n; i += NT) add(s_list[i]);
      } else {
        for_tail(add);  // more scores around the thresholds than the list holds
      }
      bsum(H, Lo, S1, S0, dH, dL, S1, S0);
      dS = S1 + S0;
      if (from_list) {
        dH += bH;
        dL += bL;
        dS += bS;
      }
    };
    lam = newton_lambda(m, eps, lo0, hi0, fmin(fmax(start, lo0), hi0), pass);
  }
  if (t == 0) {
    W.hdr->lamf = (float)lam;
    W.hdr->st = st;
    if (L.lambda_out) L.lambda_out[u] = (float)lam;
  }
}

namespace {

// pi and the mask of a thread's tokens of a segment: groups of 4 tokens at i0 + 4 (q kSegThreads + t).
struct SegMask {
  float p[kSegQuads][4];
  uint32_t keep;  // bit 4 q + j
  __device__ __forceinline__ void draw(const EvictLaunch &L, const Unit &U, int u, int64_t i0, float lamf) {
    const int t = threadIdx.x;
    const float *sc = L.scores + U.base;
    const bool vec = (U.base & 3) == 0;
    const uint64_t sd = L.seed_per_unit ? L.seed_per_unit[u] : L.seed;
    const int64_t tail_lo = L.n_sink, tail_hi = U.n - (int64_t)L.n_recent;
    float4 raw[kSegQuads];
#pragma unroll
    for (int q = 0; q < kSegQuads; ++q) raw[q] = load4(sc, i0 + 4 * (q * kSegThreads + t), U.n, vec);
    keep = 0u;
#pragma unroll
    for (int q = 0; q < kSegQuads; ++q) {
      const int64_t i = i0 + 4 * (q * kSegThreads + t);
      const uint4 x = philox4x32_10(make_uint4((uint32_t)(i >> 2), (uint32_t)u, L.epoch, kPhiloxTag),
                                    (uint32_t)sd, (uint32_t)(sd >> 32));
      const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
      const float v[4] = {raw[q].x, raw[q].y, raw[q].z, raw[q].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t b = 0;
        const float c = clean_score(v[j], b);
        p[q][j] = token_pi(i + j >= tail_lo && i + j < tail_hi, c, lamf, L.pi_min);
        if (i + j < U.n && keep_token(xw[j], p[q][j])) keep |= 1u << (4 * q + j);
      }
    }
  }
};

}  // namespace

__global__ __launch_bounds__(kSegThreads) void evict_long_count_kernel(EvictLaunch L) {
  __shared__ int s_c[kSegThreads / 64];
  const int u = blockIdx.x / L.segs, sg = blockIdx.x % L.segs, t = threadIdx.x;
  const Unit U = load_unit(L, u);
  const int64_t i0 = (int64_t)sg * kSegRows;
  if (!U.ok || i0 >= U.n) return;
  const UnitWs W = unit_ws(L, u);
  SegMask M;
  M.draw(L, U, u, i0, W.hdr->lamf);
  const int c = wave_sum((int)__popc(M.keep));
  if ((t & 63) == 0) s_c[t >> 6] = c;
  __syncthreads();
  if (t == 0) {
    int s = 0;
    for (int w = 0; w < kSegThreads / 64; ++w) s += s_c[w];
    W.seg[sg] = s;
  }
}

__global__ __launch_bounds__(kSegThreads) void evict_long_write_kernel(EvictLaunch L) {
  constexpr int NW = kSegThreads / 64;
  __shared__ int s_idx[kSegRows];
  __shared__ float s_pi[kSegRows];
  __shared__ int s_cnt[kSegQuads][NW];
  __shared__ int s_pre[NW];
  const int u = blockIdx.x / L.segs, sg = blockIdx.x % L.segs;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const Unit U = load_unit(L, u);
  const int64_t i0 = (int64_t)sg * kSegRows;
  const UnitWs W = unit_ws(L, u);
  const int64_t nseg = (U.n + kSegRows - 1) / kSegRows;
  if (!U.ok || U.n == 0) {  // larger than the launch was planned for, or empty: nothing to write
    if (sg == 0 && t == 0) {
      L.count[u] = 0;
      L.status[u] = U.ok ? W.hdr->st : EBD_ST_BAD_LAYOUT;
      if (!U.ok && L.lambda_out) L.lambda_out[u] = 0.0f;
    }
    return;
  }
  if (sg >= nseg) return;
  // retained rows of the segments before this one (the last segment's work-group takes all)
  int pre = 0;
  for (int k = t; k < sg; k += kSegThreads) pre += W.seg[k];
  pre = wave_sum(pre);
  if (lane == 0) s_pre[wv] = pre;
  SegMask M;
  M.draw(L, U, u, i0, W.hdr->lamf);
  if (L.pi_full) {
#pragma unroll
    for (int q = 0; q < kSegQuads; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t i = i0 + 4 * (q * kSegThreads + t) + j;
        if (i < U.n) L.pi_full[U.base + i] = M.p[q][j];
      }
  }
  // ranks within the segment: positions ascend with (q, wave, lane, j)
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int before[kSegQuads];
#pragma unroll
  for (int q = 0; q < kSegQuads; ++q) {
    int b = 0, tot = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t bal = __ballot((M.keep >> (4 * q + j)) & 1u);
      b += __popcll(bal & below);
      tot += __popcll(bal);
    }
    before[q] = b;
    if (lane == 0) s_cnt[q][wv] = tot;
  }
  __syncthreads();
  int64_t first = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) first += s_pre[w];
  int total = 0;
#pragma unroll
  for (int q = 0; q < kSegQuads; ++q) {
    int r = total + before[q];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int c = s_cnt[q][w];
      r += w < wv ? c : 0;
      total += c;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if ((M.keep >> (4 * q + j)) & 1u) {
        s_idx[r] = (int)(i0 + 4 * (q * kSegThreads + t) + j);
        s_pi[r] = M.p[q][j];
        ++r;
      }
    }
  }
  __syncthreads();
  if (sg == nseg - 1 && t == 0) {
    const int64_t all = first + total;
    L.count[u] = (int32_t)all;
    L.status[u] = W.hdr->st | (all > U.cap ? EBD_ST_CAP_OVERFLOW : 0u);
  }
  // the rows that the unit's capacity holds: pi, positions, then K and V (16 lanes per 256-byte row,
  // 8 rows per thread in flight, every byte touched once)
  const int rows = (int)max(min((int64_t)total, U.cap - first), (int64_t)0);
  for (int r = t; r < rows; r += kSegThreads) {
    L.pic[U.cbase + first + r] = s_pi[r];
    L.idxc[U.cbase + first + r] = s_idx[r];
  }
  constexpr int kPass = kSegThreads / 16, kIt = 8;
  const int sub = t & 15, grow = t >> 4;
  const u32x4 *K4 = reinterpret_cast<const u32x4 *>(L.K) + U.base * (kHeadDim / 8) + sub;
  const u32x4 *V4 = reinterpret_cast<const u32x4 *>(L.V) + U.base * (kHeadDim / 8) + sub;
  u32x4 *Kc4 = reinterpret_cast<u32x4 *>(L.Kc) + (U.cbase + first) * (kHeadDim / 8) + sub;
  u32x4 *Vc4 = reinterpret_cast<u32x4 *>(L.Vc) + (U.cbase + first) * (kHeadDim / 8) + sub;
  for (int r0 = 0; r0 < rows; r0 += kPass * kIt) {
    u32x4 kv[kIt], vv[kIt];
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
      const int r = r0 + grow + k * kPass;
      const int64_t sr = (int64_t)s_idx[r < rows ? r : 0] * (kHeadDim / 8);
      kv[k] = __builtin_nontemporal_load(&K4[sr]);
      vv[k] = __builtin_nontemporal_load(&V4[sr]);
    }
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
      const int r = r0 + grow + k * kPass;
      if (r < rows) {
        __builtin_nontemporal_store(kv[k], &Kc4[(int64_t)r * (kHeadDim / 8)]);
        __builtin_nontemporal_store(vv[k], &Vc4[(int64_t)r * (kHeadDim / 8)]);
      }
    }
  }
}

size_t evict_long_unit_bytes(int64_t max_rows) {
  const size_t segs = (size_t)((max_rows + kSegRows - 1) / kSegRows);
  return kHistBins * sizeof(unsigned long long) + sizeof(LongHeader) + (4 * segs + 63) / 64 * 64;
}

hipError_t launch_evict_long_select(const EvictLaunch &L, hipStream_t s) {
  const int64_t words = (kHistBins * sizeof(unsigned long long) + sizeof(LongHeader)) / sizeof(uint4);
  const unsigned U = (unsigned)L.U, zper = (unsigned)((words + 1023) / 1024);
  hipLaunchKernelGGL(evict_long_zero_kernel, dim3(U * zper), dim3(256), 0, s, L);
  hipLaunchKernelGGL(evict_long_hist_kernel, dim3(U * (unsigned)L.segs), dim3(kSegThreads), 0, s, L);
  hipLaunchKernelGGL(evict_long_solve_kernel, dim3(U), dim3(kSolveThreads), kSolveList * sizeof(float), s, L);
  hipLaunchKernelGGL(evict_long_count_kernel, dim3(U * (unsigned)L.segs), dim3(kSegThreads), 0, s, L);
  return hipGetLastError();
}

hipError_t launch_evict_long_write(const EvictLaunch &L, hipStream_t s) {
  hipLaunchKernelGGL(evict_long_write_kernel, dim3((unsigned)L.U * (unsigned)L.segs), dim3(kSegThreads), 0,
                     s, L);
  return hipGetLastError();
}

}  // namespace ebd
