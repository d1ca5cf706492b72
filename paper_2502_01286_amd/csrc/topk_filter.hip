// Top-k of (frame, template) pairs by filter and rescoring.
//
// dense_filter gives FP32 rho of every offset with a known error bound.  The k
// best offsets by the reference arithmetic (FP32: the segment form's chains in
// their order of summation; FP64: box sums in FP64) are then among the
// candidates: the offsets whose filter value is not below the k-th largest by
// more than twice the two errors.  filter_select finds them (one workgroup per
// pair), forms their accurate values, scores those near the k-th of them again
// by the reference arithmetic and orders these, so the result is the
// reference's, bit for bit.  A pair whose candidates do not fit, or whose nearly
// uniform windows (where the FP32 bound is too wide) come near the k-th value,
// is scored at every offset: FP32 pairs by the segment form itself, whose work
// items filter_select lists for a launch that finds none on most frames, FP64
// pairs by seq_topk, which also takes those that no filter serves.  Such a call
// costs that form and the filter: 8 FP32 pairs of 1280 x 720 in us, segment form
// alone / with the filter, K 2 to 1444: uniform 790 / 980, nearly uniform 795 /
// 1080, rows of glyphs 1210 / 1050, K 571 to 4957 periodic 4080 / 4070.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device_util.hpp"

namespace sncc {

// --------------------------------------------------------- reference values
// Per-offset quantities of the FP32 segment form: the negated integer mean and
// the scale 1 / sqrt(V q_k / n), with run_item's operations.
struct Ref32 {
  int nb;
  float scale;
};

__device__ __forceinline__ uint32_t ref_box(const uint32_t *__restrict__ a0, int W, int H, int P) {
  const uint32_t *a1 = a0 + (long long)H * P;
  return (a1[W] - a1[0]) - (a0[W] - a0[0]);
}

__device__ __forceinline__ Ref32 ref32(const uint32_t *__restrict__ S,
                                       const uint32_t *__restrict__ S2, int P, int u, int v, int W,
                                       int H, int n, int sq_rows, double q_k) {
  const long long o = (long long)v * P + u;
  const uint32_t sf = ref_box(S + o, W, H, P);
  const float inv_n = 1.0f / (float)n;
  const double qnd = q_k / (double)n;
  Ref32 r;
  r.nb = -(int)__builtin_rintf((float)sf * inv_n);
  if (n <= kMaxSqBoxArea) {
    const double fs = (double)sf;
    const double Vd = __builtin_fma((double)n, (double)ref_box(S2 + o, W, H, P), -(fs * fs));
    r.scale = Vd == 0.0 ? 0.f : __builtin_amdgcn_rsqf((float)(Vd * qnd));
  } else {
    const u64 sf2 = window_sq(S2 + o, W, H, P, sq_rows);
    const u64 V = (u64)(uint32_t)n * sf2 - (u64)sf * sf;
    r.scale = V == 0 ? 0.f : __builtin_amdgcn_rsqf((float)((double)V * qnd));
  }
  return r;
}

// A compensated step of the FP32 sum; y starts the next block.
__device__ __forceinline__ void ref_step(float &acc, float &cmp, float &y) {
  const float t = acc + y;
  cmp = (t - acc) - y;
  acc = t;
  y = -cmp;
}

// Accurate rho of one offset by a whole wave, FP64: box sums less A_i b (b the
// window mean rounded to an integer) in integers, c_i times them summed over the
// lanes and then the wave, and the mean term of Eq. (12) for what b leaves.
// (Neither reference's order of summation: it only tells which candidates the
// reference is asked about.)
__device__ __forceinline__ double wave_value(const uint32_t *__restrict__ S,
                                             const uint32_t *__restrict__ S2, int P, int u, int v,
                                             int W, int H, int sq_rows, double q_k, int K,
                                             double r64, const int4 *__restrict__ geom,
                                             const double *__restrict__ c64, int lane) {
  const long long o = (long long)v * P + u;
  const int n = W * H;
  const uint32_t sf = ref_box(S + o, W, H, P);
  const u64 sf2 = window_sq(S2 + o, W, H, P, sq_rows);
  const long long V = (long long)((u64)(uint32_t)n * sf2 - (u64)sf * sf);
  const double fbar = (double)sf / (double)n;
  const int b = (int)rint(fbar);
  double acc = 0.0;
  for (int i = lane; i < K; i += 64) {
    const int4 g = geom[i];
    const uint32_t F = ref_box(S + o + (long long)g.y * P + g.x, g.z, g.w, P);
    acc = __builtin_fma((double)((int)F - g.z * g.w * b), c64[i], acc);
  }
  for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
  const double num = acc + ((double)b - fbar) * r64;
  return V == 0 ? 0.0 : num / sqrt((double)V / (double)n * q_k);
}

// ----------------------------------------------------------------- selection
constexpr int kSelThreads = 1024;
constexpr int kRefGroup = kSelThreads / 64 - 1;  // candidates scored at a time in FP32
constexpr int kRefChunk = 256;                   // records per step of them
constexpr int kSelBins = 2048;
constexpr int kSelBlocks = 2048;

// Workgroup memory of ordered_group: the candidates' terms (rows of a pitch
// that spreads 16-byte reads of one place over the banks) and their c, twice,
// and the candidates' scales.
template <int NP>
struct OrderedLds {
  alignas(16) float g[2][NP][kRefChunk / 2 + 4];
  alignas(16) float c[2][kRefChunk / 2];
  float scale[NP];
};

// FP32 reference values of the candidates c0 .. c0 + NP - 1 (those below n,
// whose sums all have the pair's records of kind `side`) by a workgroup of
// NP + 1 waves, as keys.  The terms are added in the segment
// form's order, a chain of one addition after the other: waves 0 .. NP - 1 take
// a candidate each and form its terms G_i = F_i - A_i b, a lane per record,
// kRefChunk records ahead, and the last wave adds them, a lane per candidate,
// four terms and a compensated step at a time without a branch (a branch per
// term on the step's end took 60 cycles a term: 125 us for K 5000).
template <int NP>
__device__ __forceinline__ void ordered_group(const uint32_t *__restrict__ S,
                                              const uint32_t *__restrict__ S2, int P,
                                              const FilterPair &fp,
                                              const SeqRec *__restrict__ seq, const int *cand,
                                              int c0, int n, int side, OrderedLds<NP> &sh,
                                              u64 *key, int wave, int lane) {
  const SeqRec *sr = seq + fp.seq0[side];
  const int n_seq = fp.n_seq[side], nu = fp.a.nu;
  const bool mine = wave < NP && c0 + wave < n;  // wave 0's always is
  const uint32_t *w = S;
  int nb0 = 0;
  if (mine) {
    const int idx = __builtin_amdgcn_readfirstlane(cand[c0 + wave]);
    const int v = idx / nu, u = idx - v * nu;
    const Ref32 rf = ref32(S, S2, P, u, v, fp.a.W, fp.a.H, fp.a.n, fp.a.sq_rows, fp.a.q_k);
    nb0 = rf.nb;
    w = S + (long long)v * P + u;
    if (lane == 0) sh.scale[wave] = rf.scale;
  }
  auto produce = [&](int base, int buf) {
    constexpr int Q = kRefChunk / 64;
    SeqRec e[Q];
    uint32_t D[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = base + 64 * q + lane;
      e[q] = SeqRec{0, 0, kSeqNoTerm, 0.f};
      if (i < n_seq) e[q] = sr[i];
    }
    const char *wb = reinterpret_cast<const char *>(w);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      D[q] = *reinterpret_cast<const uint32_t *>(wb + e[q].bot) -
             *reinterpret_cast<const uint32_t *>(wb + e[q].top);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t prev = (uint32_t)__shfl_up((int)D[q], 1);
      const uint32_t af = e[q].area_flags;
      const int G = (int)(D[q] - prev) + __mul24((int)(af & kSeqArea), nb0);
      if (!(af & kSeqNoTerm)) {
        const int j = (64 * q + lane) / 8 * 4 + ((af >> kSeqSlot) & 3);
        sh.g[buf][wave][j] = af & kSeqZero ? 0.f : (float)G;
        if (wave == 0) sh.c[buf][j] = e[q].c;
      }
    }
  };
  if (mine) produce(0, 0);
  float acc = 0.f, cmp = 0.f, y = -cmp;
  __syncthreads();
  for (int base = 0, buf = 0; base < n_seq; base += kRefChunk, buf ^= 1) {
    if (wave == NP) {
      const float4 *gl = reinterpret_cast<const float4 *>(sh.g[buf][min(lane, NP - 1)]);
      const float4 *cl = reinterpret_cast<const float4 *>(sh.c[buf]);
      const int m = min(kRefChunk, n_seq - base) / 8;  // blocks
#pragma unroll 4
      for (int l = 0; l < m; ++l) {
        const float4 g = gl[l], c = cl[l];
        y = __builtin_fmaf(g.x, c.x, y);
        y = __builtin_fmaf(g.y, c.y, y);
        y = __builtin_fmaf(g.z, c.z, y);
        y = __builtin_fmaf(g.w, c.w, y);
        ref_step(acc, cmp, y);
      }
    } else if (mine && base + kRefChunk < n_seq) {
      produce(base + kRefChunk, buf ^ 1);
    }
    __syncthreads();
  }
  if (wave == NP && lane < NP && c0 + lane < n)
    key[c0 + lane] = make_key((acc - cmp) * sh.scale[lane], cand[c0 + lane]);
  __syncthreads();
}

// The same for FP64: box sums times c_i added in segment order (as lane_ref64
// does), one fused multiply-add after the other.
constexpr int kRefChunk64 = 128;  // segments per step
template <int NP>
struct OrderedLds64 {
  alignas(16) uint32_t f[2][NP][kRefChunk64 + 4];
  alignas(16) double c[2][kRefChunk64];
  long long V[NP];
  uint32_t sf[NP];
};

template <int NP>
__device__ __forceinline__ void ordered_group64(const uint32_t *__restrict__ S,
                                                const uint32_t *__restrict__ S2, int P,
                                                const FilterPair &fp,
                                                const int4 *__restrict__ geom,
                                                const double *__restrict__ c64, const int *cand,
                                                int c0, int n, OrderedLds64<NP> &sh, u64 *key_hi,
                                                uint32_t *key_lo, int wave, int lane) {
  const int4 *gp = geom + fp.seg_off;
  const double *cp = c64 + fp.seg_off;
  const int K = fp.K, nu = fp.a.nu, W = fp.a.W, H = fp.a.H;
  const bool mine = wave < NP && c0 + wave < n;  // wave 0's always is
  const uint32_t *w = S;
  if (mine) {
    const int idx = __builtin_amdgcn_readfirstlane(cand[c0 + wave]);
    const int v = idx / nu, u = idx - v * nu;
    const long long o = (long long)v * P + u;
    w = S + o;
    const uint32_t sf = ref_box(w, W, H, P);
    const u64 sf2 = window_sq(S2 + o, W, H, P, fp.a.sq_rows);
    if (lane == 0) {
      sh.sf[wave] = sf;
      sh.V[wave] = (long long)((u64)(uint32_t)fp.a.n * sf2 - (u64)sf * sf);
    }
  }
  auto produce = [&](int base, int buf) {
    constexpr int Q = kRefChunk64 / 64;
    int4 g[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) g[q] = gp[min(base + 64 * q + lane, K - 1)];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      sh.f[buf][wave][64 * q + lane] =
          ref_box(w + (long long)g[q].y * P + g[q].x, g[q].z, g[q].w, P);
      if (wave == 0) sh.c[buf][64 * q + lane] = cp[min(base + 64 * q + lane, K - 1)];
    }
  };
  if (mine) produce(0, 0);
  double acc = 0.0;
  __syncthreads();
  for (int base = 0, buf = 0; base < K; base += kRefChunk64, buf ^= 1) {
    if (wave == NP) {
      const uint32_t *fl = sh.f[buf][min(lane, NP - 1)];
      const double *cl = sh.c[buf];
      const int m = min(kRefChunk64, K - base);
      int l = 0;
#pragma unroll 2
      for (; l + 4 <= m; l += 4) {
        const uint4 b = *reinterpret_cast<const uint4 *>(fl + l);
        acc = __builtin_fma((double)b.x, cl[l], acc);
        acc = __builtin_fma((double)b.y, cl[l + 1], acc);
        acc = __builtin_fma((double)b.z, cl[l + 2], acc);
        acc = __builtin_fma((double)b.w, cl[l + 3], acc);
      }
      for (; l < m; ++l) acc = __builtin_fma((double)fl[l], cl[l], acc);
    } else if (mine && base + kRefChunk64 < K) {
      produce(base + kRefChunk64, buf ^ 1);
    }
    __syncthreads();
  }
  if (wave == NP && lane < NP && c0 + lane < n) {
    key_hi[c0 + lane] = double_order(
        plain_rho(acc, sh.sf[lane], sh.V[lane], fp.a.n, fp.a.q_k, fp.r64));
    key_lo[c0 + lane] = 0xffffffffu - (uint32_t)cand[c0 + lane];
  }
  __syncthreads();
}

// From the keys of n candidates' accurate values, one wave: the candidates
// within twice the reference's error (FP32's, which is the larger) of the k-th
// largest, listed in
// `near`, those left of column u_split (m_main of them) first; returns their
// number.
__device__ __forceinline__ int near_kth(const u64 *key, int n, int k, int nu, int u_split,
                                        int *near, int *m_main, int lane) {
  u64 lk = 0;
  for (int c = 0; c < n; c += 64)
    topk_merge_sorted(lk, wave_sort_desc_u64(c + lane < n ? key[c + lane] : 0, lane), k, lane);
  const u64 kth = lane_u64(lk, k - 1);
  const float t = kth == 0 ? -__builtin_inff()
                           : float_unorder((uint32_t)(kth >> 32)) - 2.f * (3e-6f + 1e-7f);
  int m = 0;
  for (int side = 0; side < 2; ++side) {
    for (int c = 0; c < n; c += 64) {
      const u64 x = c + lane < n ? key[c + lane] : 0;
      const int idx = (int)(0xffffffffu - (uint32_t)(x & 0xffffffffu));
      const u64 keep = __ballot(x != 0 && float_unorder((uint32_t)(x >> 32)) >= t &&
                                (idx % nu >= u_split) == (side == 1));
      if ((keep >> lane) & 1) near[m + __popcll(keep & ((1ull << lane) - 1))] = idx;
      m += __popcll(keep);
    }
    if (side == 0) *m_main = m;
  }
  return m;
}

// The k best of n keys, by one wave, as a pair's matches.
__device__ __forceinline__ void write_topk32(const u64 *key, int n, int k, int nu,
                                             sncc_match *__restrict__ out, int lane) {
  u64 lh = 0;
  for (int c = 0; c < n; c += 64)
    topk_merge_sorted(lh, wave_sort_desc_u64(c + lane < n ? key[c + lane] : 0, lane), k, lane);
  if (lane < k) {
    sncc_match m;
    m.u = m.v = -1;
    m.rho = -__builtin_inff();
    if (lh != 0) {
      const int idx = (int)(0xffffffffu - (uint32_t)(lh & 0xffffffffu));
      m.v = idx / nu;
      m.u = idx - m.v * nu;
      m.rho = float_unorder((uint32_t)(lh >> 32));
    }
    out[lane] = m;
  }
}

// Largest bin b with at least k entries in bins b and above (0 when there are
// fewer in all); every thread of the workgroup gets it.
__device__ __forceinline__ int kth_bin(const int *hist, int k, int *out) {
  __syncthreads();
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    constexpr int PER = kSelBins / 64;
    int sum = 0;
    for (int i = 0; i < PER; ++i) sum += hist[lane * PER + i];
    const int incl = (int)wave_incl_scan((uint32_t)sum);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const u64 ok = __ballot(total - incl + sum >= k);  // entries in this lane's bins and above
    int b = 0;
    if (ok) {
      const int L = 63 - __builtin_clzll(ok);
      const int above = total - __builtin_amdgcn_readlane(incl, L);
      const int mine = lane < PER ? hist[L * PER + lane] : 0;
      const int in2 = (int)wave_incl_scan((uint32_t)mine);
      const int t2 = __builtin_amdgcn_readlane(in2, 63);
      const u64 ok2 = __ballot(lane < PER && above + t2 - in2 + mine >= k);
      b = L * PER + 63 - __builtin_clzll(ok2);
    }
    if (lane == 0) *out = b;
  }
  __syncthreads();
  return *out;
}

template <bool F64, bool SPREAD>
__global__ __launch_bounds__(kSelThreads) void filter_select(
    const uint32_t *__restrict__ s, const uint32_t *__restrict__ s2, long long frame_stride, int P,
    const FilterPair *__restrict__ fps, const float *__restrict__ map,
    const float2 *__restrict__ bmax, const SeqRec *__restrict__ seq,
    const int4 *__restrict__ geom, const double *__restrict__ c64, int k,
    sncc_match *__restrict__ out, int *__restrict__ direct, Undecided und,
    FilterSpread *__restrict__ spread) {
  __shared__ int hist[kSelBins];
  __shared__ int list[kSelBlocks];
  __shared__ int cand[kFilterCands];
  __shared__ u64 key_hi[SPREAD ? 1 : kFilterCands];
  __shared__ uint32_t key_lo[F64 ? kFilterCands : 1];
  __shared__ OrderedLds<F64 || SPREAD ? 1 : kRefGroup> group;
  __shared__ OrderedLds64<F64 ? kRefGroup : 1> group64;
  __shared__ int n_list, n_cand, bin, bad;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const FilterPair &fp = fps[blockIdx.x];
  const int nb = fp.n_blocks, rv = fp.a.rv, nu = fp.a.nu;
  const float2 *bm = bmax + fp.block0;
  const float *vals = map + fp.map0;
  // twice the errors of the filter (fp.error: its rounded c; the result's
  // roundings and 1 / sqrt, 3e-7; the thresholds' below, 1e-7) and of the reference (FP32: at
  // most 3e-6 for windows of energy n / 100 and above, 1e-4 for any window; FP64: K 2^-53
  // sum |c_i| F_i, so K 2^-53 times 2550 and 255 sqrt(n), 4e-8 and 2e-6 at the largest K and n)
  const float margin = 2.f * (fp.error + 4e-7f + (F64 ? 1e-7f : 3e-6f));
  const float low_margin = 2.f * (fp.error + 1e-4f);

  auto clear = [&]() {
    __syncthreads();
    for (int i = tid; i < kSelBins; i += kSelThreads) hist[i] = 0;
    if (tid == 0) n_list = 0;
    __syncthreads();
  };
  auto blocks_from = [&](float t) {  // the blocks whose largest value is at least t
    for (int i = tid; i < nb; i += kSelThreads)
      if (bm[i].x >= t) {
        const int at = atomicAdd(&n_list, 1);
        if (at < kSelBlocks) list[at] = i;
      }
    __syncthreads();
  };
  // calls f(value, row-major index) for the values of the listed blocks (until
  // there are more candidates than the pair may hold)
  auto scan = [&](auto f) {
    const int units = min(n_list, kSelBlocks) * rv;
    for (int un = wave * 4; un < units; un += kSelThreads / 64 * 4) {
      if (__hip_atomic_load(&n_cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >
          kFilterCands)
        break;
      float4 w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int x = min(un + q, units - 1);
        w[q] = reinterpret_cast<const float4 *>(vals)[((long long)list[x / rv] * rv + x % rv) * 64 +
                                                      lane];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (un + q >= units) break;
        const int blk = list[(un + q) / rv], r = (un + q) % rv;
        const int tile = blk / kDenseNW, wv = blk % kDenseNW, tv = tile / fp.a.ntu;
        const int u = (tile - tv * fp.a.ntu) * kDenseBU + 16 * (lane & 7) + 4 * (lane >> 4);
        const int v = tv * 2 * kDenseNW * rv + rv * (2 * wv + ((lane >> 3) & 1)) + r;
        const float e[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (e[c] != -__builtin_inff()) f(e[c], v * nu + u + c);
      }
    }
    __syncthreads();
  };

  // T0: at least k blocks reach it, so the k-th largest value does (the lower
  // edge of a bin of block maxima, less a rounding allowance)
  if (tid == 0) n_cand = bad = 0;
  clear();
  for (int i = tid; i < nb; i += kSelThreads) {
    const float x = bm[i].x;
    if (x != -__builtin_inff())
      atomicAdd(&hist[min(kSelBins - 1, max(0, (int)((x + 1.0f) * 1000.0f)))], 1);
  }
  const int b0 = kth_bin(hist, k, &bin);
  const float T0 = b0 == 0 ? -__builtin_inff() : (float)b0 * 1e-3f - 1.0f - 1e-5f;
  // T1: the same for the values of the blocks that reach T0, in finer bins
  clear();
  blocks_from(T0);
  const float lo = b0 == 0 ? -1.001f : T0;
  const float scale = (float)(kSelBins - 1) / (1.001f - lo);
  scan([&](float x, int) {
    if (x >= T0) {
      // lanes that all meet one bin (uniform frames) add once (8 pairs of a
      // uniform 1280 x 720: 1870 -> 980 us a call, with the candidates' end above)
      const int b = min(kSelBins - 1, max(0, (int)((x - lo) * scale)));
      const int b_first = __builtin_amdgcn_readfirstlane(b);
      const u64 active = __ballot(1);
      const bool one = __ballot(b == b_first) == active;
      if (!one || lane == __ffsll((long long)active) - 1)
        atomicAdd(&hist[b], one ? __popcll(active) : 1);
    }
  });
  const int b1 = kth_bin(hist, k, &bin);
  const float T1 = b1 == 0 ? T0 : lo + ((float)b1 - 0.01f) / scale;
  if (tid == 0 && n_list > kSelBlocks) bad = 1;
  clear();
  blocks_from(T1 - margin);
  if (tid == 0 && n_list > kSelBlocks) bad = 1;
  for (int i = tid; i < nb; i += kSelThreads)
    if (bm[i].y + low_margin >= T1) bad = 1;
  scan([&](float x, int idx) {
    if (x >= T1 - margin) {
      const int at = atomicAdd(&n_cand, 1);
      if (at < kFilterCands) cand[at] = idx;
    }
  });
  int n = n_cand;
  if (bad || n > kFilterCands) {
    if (tid == 0) direct[fp.pair] = 1;
    if (SPREAD && tid == 0) spread[blockIdx.x].n = -1;
    if constexpr (!F64) {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int m = fp.n_items[x];
        if (m == 0) continue;
        __syncthreads();
        if (tid == 0) n_list = atomicAdd(und.n[x], m);
        __syncthreads();
        int *to = und.order[x] + n_list;
        for (int i = tid; i < m; i += kSelThreads) to[i] = fp.item0[x] + i;
      }
    }
    return;
  }
  if constexpr (SPREAD) {
    FilterSpread &sp = spread[blockIdx.x];
    for (int c = tid; c < n; c += kSelThreads) sp.cand[c] = cand[c];
    if (tid == 0) {
      sp.n = n;
      direct[fp.pair] = 0;
    }
    return;
  }
  // the candidates' accurate values (FP64, a wave each, lanes over the
  // segments), then those near the k-th by the reference arithmetic
  const uint32_t *S = s + (long long)fp.frame * frame_stride;
  const uint32_t *S2 = s2 + (long long)fp.frame * frame_stride;
  if constexpr (!SPREAD) {
    // (few FP64 candidates, all of one kind of records, at once)
    if (!F64 || n > kRefGroup) {
      for (int c = wave; c < n; c += kSelThreads / 64) {
        const int idx = __builtin_amdgcn_readfirstlane(cand[c]);
        const int v = idx / nu, u = idx - v * nu;
        const double r = wave_value(S, S2, P, u, v, fp.a.W, fp.a.H, fp.a.sq_rows, fp.a.q_k, fp.K,
                                    fp.r64, geom + fp.seg_off, c64 + fp.seg_off, lane);
        if (lane == 0) key_hi[c] = make_key((float)r, idx);
      }
      __syncthreads();
      if (wave == 0) {
        int m_main = 0;
        const int m = near_kth(key_hi, n, k, nu, fp.u_split, cand, &m_main, lane);
        if (lane == 0) {
          n_cand = m;
          n_list = m_main;
        }
      }
      __syncthreads();
      n = n_cand;
    }
    if constexpr (F64) {
      for (int c0 = 0; c0 < n; c0 += kRefGroup)
        ordered_group64<kRefGroup>(S, S2, P, fp, geom, c64, cand, c0, n, group64, key_hi, key_lo,
                                   wave, lane);
    } else {
      const int n_main = n_list;
      for (int c0 = 0; c0 < n_main; c0 += kRefGroup)
        ordered_group<kRefGroup>(S, S2, P, fp, seq, cand, c0, n_main, 0, group, key_hi, wave, lane);
      for (int c0 = n_main; c0 < n; c0 += kRefGroup)
        ordered_group<kRefGroup>(S, S2, P, fp, seq, cand, c0, n, 1, group, key_hi, wave, lane);
    }
  }
  __syncthreads();
  if (wave != 0) return;
  sncc_match *o = out + (long long)fp.pair * k;
  if constexpr (F64) {
    u64 lh = 0;
    uint32_t ll = 0;
    for (int c = 0; c < n; c += 64) {
      const u64 h = c + lane < n ? key_hi[c + lane] : 0;
      const uint32_t l = c + lane < n ? key_lo[c + lane] : 0;
      u64 todo = __ballot(key96_gt(h, l, lane_u64(lh, k - 1),
                                   (uint32_t)__builtin_amdgcn_readlane((int)ll, k - 1)));
      while (todo) {
        const int q = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        const u64 kh = lane_u64(h, q);
        const uint32_t kl = (uint32_t)__builtin_amdgcn_readlane((int)l, q);
        if (key96_gt(kh, kl, lane_u64(lh, k - 1),
                     (uint32_t)__builtin_amdgcn_readlane((int)ll, k - 1)))
          topk96_insert(lh, ll, kh, kl, k, lane);
      }
    }
    if (lane < k) {
      sncc_match m;
      m.u = m.v = -1;
      m.rho = -__builtin_inff();
      if (lh != 0 || ll != 0) {
        const int idx = (int)(0xffffffffu - ll);
        m.v = idx / nu;
        m.u = idx - m.v * nu;
        m.rho = (float)double_unorder(lh);
      }
      o[lane] = m;
    }
  } else if constexpr (!SPREAD) {
    write_topk32(key_hi, n, k, nu, o, lane);
  }
  if (lane == 0) direct[fp.pair] = 0;
}

// The spread form of the FP32 candidates' scoring: accurate values, one wave
// per candidate; the near ones in order, kSpreadNP at a time per workgroup; the
// result, one wave per pair.
constexpr int kSpreadWgs = 16, kSpreadNP = 3;

__global__ __launch_bounds__(256) void filter_values(
    const uint32_t *__restrict__ s, const uint32_t *__restrict__ s2, long long frame_stride, int P,
    const FilterPair *__restrict__ fps, const int4 *__restrict__ geom,
    const double *__restrict__ c64, FilterSpread *__restrict__ spread) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int f = blockIdx.x / kSpreadWgs, part = blockIdx.x % kSpreadWgs;
  const FilterPair &fp = fps[f];
  FilterSpread &sp = spread[f];
  const uint32_t *S = s + (long long)fp.frame * frame_stride;
  const uint32_t *S2 = s2 + (long long)fp.frame * frame_stride;
  for (int c = part * 4 + wave; c < sp.n; c += 4 * kSpreadWgs) {
    const int idx = __builtin_amdgcn_readfirstlane(sp.cand[c]);
    const int v = idx / fp.a.nu, u = idx - v * fp.a.nu;
    const double r = wave_value(S, S2, P, u, v, fp.a.W, fp.a.H, fp.a.sq_rows, fp.a.q_k, fp.K, fp.r64,
                                  geom + fp.seg_off, c64 + fp.seg_off, lane);
    if (lane == 0) sp.val[c] = make_key((float)r, idx);
  }
}

__global__ __launch_bounds__(64 * (kSpreadNP + 1)) void filter_order(
    const uint32_t *__restrict__ s, const uint32_t *__restrict__ s2, long long frame_stride, int P,
    const FilterPair *__restrict__ fps, const SeqRec *__restrict__ seq, int k,
    FilterSpread *__restrict__ spread) {
  __shared__ OrderedLds<kSpreadNP> group;
  __shared__ int near[kFilterCands];
  __shared__ int n_near, n_near_main;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int f = blockIdx.x / kSpreadWgs, part = blockIdx.x % kSpreadWgs;
  const FilterPair &fp = fps[f];
  FilterSpread &sp = spread[f];
  if (sp.n < 0) return;
  if (wave == 0) {  // every workgroup of the pair lists the same ones
    int m_main = 0;
    const int m = near_kth(sp.val, sp.n, k, fp.a.nu, fp.u_split, near, &m_main, lane);
    if (lane == 0) {
      n_near = m;
      n_near_main = m_main;
      if (part == 0) sp.m = m;
    }
  }
  __syncthreads();
  const uint32_t *S = s + (long long)fp.frame * frame_stride;
  const uint32_t *S2 = s2 + (long long)fp.frame * frame_stride;
  const int n = n_near, n_main = n_near_main;
  for (int c0 = part * kSpreadNP; c0 < n_main; c0 += kSpreadWgs * kSpreadNP)
    ordered_group<kSpreadNP>(S, S2, P, fp, seq, near, c0, n_main, 0, group, sp.key, wave, lane);
  for (int c0 = n_main + part * kSpreadNP; c0 < n; c0 += kSpreadWgs * kSpreadNP)
    ordered_group<kSpreadNP>(S, S2, P, fp, seq, near, c0, n, 1, group, sp.key, wave, lane);
}

__global__ __launch_bounds__(64) void filter_result(const FilterPair *__restrict__ fps,
                                                    const FilterSpread *__restrict__ spread, int k,
                                                    sncc_match *__restrict__ out) {
  const FilterPair &fp = fps[blockIdx.x];
  const FilterSpread &sp = spread[blockIdx.x];
  if (sp.n < 0) return;
  write_topk32(sp.key, sp.m, k, fp.a.nu, out + (long long)fp.pair * k, (int)threadIdx.x);
}

int launch_filter_select(bool fp64, const uint32_t *s, const uint32_t *s2, long long frame_stride,
                         int P, const FilterPair *fps, int n_fps, const float *map,
                         const float2 *bmax, const SeqRec *seq, const int4 *geom,
                         const double *c64, int k, sncc_match *out, int *direct,
                         const Undecided &und, FilterSpread *spread, hipStream_t st) {
#define SNCC_SELECT(F64, SPREAD)                                                               \
  hipLaunchKernelGGL((filter_select<F64, SPREAD>), dim3(n_fps), dim3(kSelThreads), 0, st, s, s2, \
                     frame_stride, P, fps, map, bmax, seq, geom, c64, k, out, direct, und, \
                     spread)
  if (fp64) {
    SNCC_SELECT(true, false);
  } else if (!spread) {
    SNCC_SELECT(false, false);
  } else {
    SNCC_SELECT(false, true);
    hipLaunchKernelGGL(filter_values, dim3(n_fps * kSpreadWgs), dim3(256), 0, st, s, s2,
                       frame_stride, P, fps, geom, c64, spread);
    hipLaunchKernelGGL(filter_order, dim3(n_fps * kSpreadWgs), dim3(64 * (kSpreadNP + 1)), 0, st, s,
                       s2, frame_stride, P, fps, seq, k, spread);
    hipLaunchKernelGGL(filter_result, dim3(n_fps), dim3(64), 0, st, fps, spread, k, out);
  }
#undef SNCC_SELECT
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// --------------------------------------------------------------- direct form
// rho_plain's arithmetic: box_i c_i summed in segment order, FP64.
__device__ __forceinline__ double lane_ref64(const uint32_t *__restrict__ S,
                                             const uint32_t *__restrict__ S2, int P, int u, int v,
                                             const SeqPair &sp, const int4 *__restrict__ geom,
                                             const double *__restrict__ c64) {
  const uint32_t *a0 = S + (long long)v * P + u;
  const uint32_t sf = ref_box(a0, sp.W, sp.H, P);
  const u64 sf2 = window_sq(S2 + (long long)v * P + u, sp.W, sp.H, P, sp.sq_rows);
  const long long V = (long long)((u64)(uint32_t)sp.n * sf2 - (u64)sf * sf);
  double acc = 0.0;
  const int4 *gp = geom + sp.seg_off;
  const double *cp = c64 + sp.seg_off;
#pragma unroll 4
  for (int i = 0; i < sp.K; ++i) {
    const int4 g = gp[i];
    acc = __builtin_fma((double)ref_box(a0 + (long long)g.y * P + g.x, g.z, g.w, P), cp[i], acc);
  }
  return plain_rho(acc, sf, V, sp.n, sp.q_k, sp.r64);
}

// The k best offsets of each sp.chunk offsets of the pairs that direct[] marks;
// the chunks of all of them go round the workgroups.  A launch without such
// pairs only reads the marks.
__global__ __launch_bounds__(256) void seq_topk(
    const uint32_t *__restrict__ s, const uint32_t *__restrict__ s2, long long frame_stride, int P,
    const SeqPair *__restrict__ pairs, int n_pairs, const int *__restrict__ direct,
    const int4 *__restrict__ geom, const double *__restrict__ c64, int k,
    Key96 *__restrict__ partial) {
  __shared__ u64 bh[4 * 64];
  __shared__ uint32_t bl[4 * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int before = 0;  // chunks of the marked pairs so far, modulo the grid
  for (int p0 = 0; p0 < n_pairs; p0 += 64) {
    u64 marked = __ballot(p0 + lane < n_pairs && direct[p0 + lane] != 0);
    while (marked) {
      const int p = p0 + __ffsll((long long)marked) - 1;
      marked &= marked - 1;
      const SeqPair sp = pairs[p];
      const uint32_t *S = s + (long long)sp.frame * frame_stride;
      const uint32_t *S2 = s2 + (long long)sp.frame * frame_stride;
      const int grid = gridDim.x;
      int c = (int)blockIdx.x - before;
      if (c < 0) c += grid;
      for (; c < sp.n_chunks; c += grid) {
        const long long total = (long long)sp.nu * sp.nv;
        const long long c0 = (long long)c * sp.chunk, c1 = min(total, c0 + sp.chunk);
        u64 lh = 0;
        uint32_t ll = 0;
        for (long long e0 = c0 + wave * 64; e0 < c1; e0 += 4 * 64) {
          const long long e = min(e0 + lane, c1 - 1);
          const int v = (int)(e / sp.nu), u = (int)(e - (long long)v * sp.nu);
          const bool ok = e0 + lane < c1;
          const double r = lane_ref64(S, S2, P, u, v, sp, geom, c64);
          u64 ch = ok ? double_order(r) : 0;
          uint32_t cl = ok ? 0xffffffffu - (uint32_t)e : 0;
          for (;;) {  // best first, while they beat the k-th
            if (!key96_gt(ch, cl, lane_u64(lh, k - 1),
                          (uint32_t)__builtin_amdgcn_readlane((int)ll, k - 1)))
              ch = 0, cl = 0;
            if (__ballot(ch != 0 || cl != 0) == 0) break;
            u64 mh;
            uint32_t ml;
            wave_max96(ch, cl, mh, ml);
            topk96_insert(lh, ll, mh, ml, k, lane);
            if (ch == mh && cl == ml) ch = 0, cl = 0;
          }
        }
        if (lane < k) {
          bh[wave * k + lane] = lh;
          bl[wave * k + lane] = ll;
        }
        __syncthreads();
        if (wave == 0) {
          for (int w = 1; w < 4; ++w)
            for (int j = 0; j < k; ++j) {  // each wave's list is in descending order
              const u64 kh = bh[w * k + j];
              const uint32_t kl = bl[w * k + j];
              if (!key96_gt(kh, kl, lane_u64(lh, k - 1),
                            (uint32_t)__builtin_amdgcn_readlane((int)ll, k - 1)))
                break;
              topk96_insert(lh, ll, kh, kl, k, lane);
            }
          if (lane < k) partial[(long long)(sp.chunk0 + c) * k + lane] = Key96{lh, ll, 0};
        }
        __syncthreads();
      }
      before = (before + sp.n_chunks) % grid;
    }
  }
}

// One wave per marked pair: the k best of its chunks' lists; one load brings
// 64 / k of them.
__global__ __launch_bounds__(256) void seq_merge(const SeqPair *__restrict__ pairs, int n_pairs,
                                                 const int *__restrict__ direct,
                                                 const Key96 *__restrict__ partial, int k,
                                                 sncc_match *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (p >= n_pairs || direct[p] == 0) return;
  const SeqPair sp = pairs[p];
  u64 lh = 0;
  uint32_t ll = 0;
  const int g = 64 / k, end = sp.chunk0 + sp.n_chunks;
  for (int c = sp.chunk0; c < end; c += g) {
    u64 h = 0;
    uint32_t l = 0;
    if (lane < g * k && c + lane / k < end) {
      const Key96 e = partial[(long long)c * k + lane];
      h = e.hi;
      l = e.lo;
    }
    u64 todo = __ballot(key96_gt(h, l, lane_u64(lh, k - 1),
                                 (uint32_t)__builtin_amdgcn_readlane((int)ll, k - 1)));
    while (todo) {
      const int q = __ffsll((long long)todo) - 1;
      todo &= todo - 1;
      const u64 kh = lane_u64(h, q);
      const uint32_t kl = (uint32_t)__builtin_amdgcn_readlane((int)l, q);
      if (key96_gt(kh, kl, lane_u64(lh, k - 1),
                   (uint32_t)__builtin_amdgcn_readlane((int)ll, k - 1)))
        topk96_insert(lh, ll, kh, kl, k, lane);
    }
  }
  if (lane < k) {
    sncc_match m;
    m.u = m.v = -1;
    m.rho = -__builtin_inff();
    if (lh != 0 || ll != 0) {
      const int idx = (int)(0xffffffffu - ll);
      m.v = idx / sp.nu;
      m.u = idx - m.v * sp.nu;
      m.rho = (float)double_unorder(lh);
    }
    out[(long long)p * k + lane] = m;
  }
}

int launch_seq_topk(const uint32_t *s, const uint32_t *s2, long long frame_stride, int P,
                    const SeqPair *pairs, int n_pairs, const int *direct,
                    const int4 *geom, const double *c64, int k, Key96 *partial, int grid,
                    sncc_match *out, hipStream_t st) {
  hipLaunchKernelGGL(seq_topk, dim3(grid), dim3(256), 0, st, s, s2, frame_stride, P, pairs,
                     n_pairs, direct, geom, c64, k, partial);
  hipLaunchKernelGGL(seq_merge, dim3((n_pairs + 3) / 4), dim3(256), 0, st, pairs, n_pairs, direct,
                     partial, k, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ------------------------------------------------------ two-threshold search
// Per run of the fast pass's survivors (a wave each), those that the filter
// leaves or did not judge; runs without any are dropped.  (Scoring a few
// survivors here, segments over lanes with corners from the tables, was slower
// than the slow pass at any number of them: 490 against 502 to 760 us a call.)
__global__ __launch_bounds__(256) void live_runs(
    const FilterPair *__restrict__ fps, const int *__restrict__ fp_of_pair, int rv,
    const int *__restrict__ tile_count, const uint32_t *__restrict__ bits,
    const sncc_hit *__restrict__ cand, const int *__restrict__ cand_count, int cand_cap,
    const RunDesc *__restrict__ runs, const int *__restrict__ run_count, int run_cap,
    LiveRun *__restrict__ live, int *__restrict__ live_count) {
  constexpr int NR = 4;  // runs per wave at a time
  __shared__ int cnt[2][4], base[2];  // by turns, so that two barriers do
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_cand = min(*cand_count, cand_cap), n_runs = min(*run_count, run_cap);
  const int bv = 2 * kDenseNW * rv;
  for (int b = 4 * NR * blockIdx.x, turn = 0; b < n_runs; b += 4 * NR * gridDim.x, turn ^= 1) {
    const int r0 = b + NR * wave;
    LiveRun lr[NR];
    int2 uv[NR][2];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      lr[q].rd = runs[min(r0 + q, n_runs - 1)];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const sncc_hit &c = cand[min(lr[q].rd.start + 64 * h + lane, n_cand - 1)];
        uv[q][h] = make_int2(c.u, c.v);
      }
    }
    int left = 0;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const RunDesc &rd = lr[q].rd;
      const int n = r0 + q < n_runs ? max(0, min(rd.count, n_cand - rd.start)) : 0;
      lr[q].m[0] = n >= 64 ? ~0ull : (1ull << n) - 1ull;
      lr[q].m[1] = n >= 128 ? ~0ull : n > 64 ? (1ull << (n - 64)) - 1ull : 0ull;
      const int at = fp_of_pair[rd.pair];
      if (at >= 0) {
        const FilterPair &fp = fps[at];
        // a run lies inside one tile
        const int tu = rd.u0 / kDenseBU, tv = rd.v0 / bv;
        if (tile_survivors(fp, tile_count, tu, tv, bv) >= fp.min_count) {
          const uint32_t *w = bits + fp.map0 + (long long)(tv * fp.a.ntu + tu) * (kDenseNW * 64);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            bool keep = false;
            if (64 * h + lane < n) {
              const int x = uv[q][h].x - tu * kDenseBU, y = uv[q][h].y - tv * bv;
              const int row = y / rv, l = (x >> 4) + 8 * (row & 1) + 16 * ((x >> 2) & 3);
              keep = (w[(row >> 1) * 64 + l] >> (4 * (y - row * rv) + (x & 3))) & 1u;
            }
            lr[q].m[h] = __ballot(keep);
          }
        }
      }
      left += (lr[q].m[0] | lr[q].m[1]) != 0;
    }
    // one addition to the shared counter for the workgroup's runs: the
    // additions of many workgroups go one by one (23 thousand runs, most of
    // them left: 40 us with one per run, 24 with one per sixteen)
    if (lane == 0) cnt[turn][wave] = left;
    __syncthreads();
    if (threadIdx.x == 0) {
      const int all = cnt[turn][0] + cnt[turn][1] + cnt[turn][2] + cnt[turn][3];
      base[turn] = all ? atomicAdd(live_count, all) : 0;
    }
    __syncthreads();
    if (lane == 0) {
      LiveRun *to = live + base[turn];
      for (int w = 0; w < wave; ++w) to += cnt[turn][w];
#pragma unroll
      for (int q = 0; q < NR; ++q)
        if ((lr[q].m[0] | lr[q].m[1]) != 0) *to++ = lr[q];
    }
  }
}

int launch_live_runs(const SlowArgs &a, const FilterPair *fps, const int *fp_of_pair, int rv,
                     const int *tile_count, const uint32_t *bits, LiveRun *live, int *live_count,
                     int grid, hipStream_t st) {
  hipLaunchKernelGGL(live_runs, dim3(grid), dim3(256), 0, st, fps, fp_of_pair, rv, tile_count,
                     bits, a.cand, a.cand_count, a.cand_cap, a.runs, a.run_count, a.run_cap, live,
                     live_count);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace sncc
