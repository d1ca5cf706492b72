// Matrix-core scoring of a rho map (Eqs. (11)-(18)) for approximations with
// many segments.
//
// The numerator sum_i c_i F_i of Eq. (12) equals the correlation of the frame
// with the approximation's zero-mean image c(x, y) (c_i on segment i).  Its
// cost does not grow with the number of segments, so above some K per template
// pixel it beats the segment sums.  It is formed in integers: c is held as
// fixed-point digits, c ~ 2^-e sum_d q_d 256^d with q_d in [-128, 127], the
// frame as f - 128 in [-128, 127], and each digit's correlation is an exact
// 32-bit integer sum on the i8 matrix instructions.  Seven digits serve FP64,
// three or four FP32 (dense_digits32 in api.cpp).  The only roundings are those
// of c and of the result: rms error of an FP32 map against 64 bits 2.5e-8
// relative (the result's own rounding; 4.5e-8 to 6e-8 in the segment form), of
// an FP64 map 0 to 1e-14 (0 to 1e-13 in the plain form).
//
// What bounds it: large templates the matrix rate (3840 x 2160, 128 x 128,
// K 4465: 280 us, 3.0e15 operations/s, where a loop of these instructions alone
// reaches 3.4e15 on random data; the segment form took 6678 us; FP64 620 us,
// 3.2e15/s, against 16.0 ms in the plain form), small ones the launch, the
// staging and the epilogue's table reads (1920 x 1080, 64 x 64: 36 us, about
// half of it matrix work).
//
// Contraction: one instruction multiplies A (16 x 64) by B (64 x 16).  Column
// j of B is a block of 16 offset columns, u = u0 + 16 (j mod 8) + i, of one of
// two offset rows (j / 8); row i of A is the offset within the block.  The 64
// products are four template rows y .. y + 3 of 16 template columns 16 x - i
// .. + 15 (x = 0 .. G - 1, G = ceil((W + 15) / 16)), so that B's entries are
// aligned 16-byte pieces of frame rows, the same for every i, and A holds the
// template rows shifted by i (banded Toeplitz blocks, zero outside the
// template), prepared once per template in the instruction's register layout
// (dense_pack).  W / (16 G) of the products are
// not zero: 0.80 at W = 64, 0.89 at 128.  B of offset row v + 4 is B of offset
// row v one step (four template rows) later, so a wave with eight offset rows
// reads each B once for two uses.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device_util.hpp"

namespace sncc {

typedef int v4i __attribute__((ext_vector_type(4)));
// Operands in global memory, said so: through a generic pointer (one read from
// a descriptor) they would be flat loads, which count as LDS reads too, and
// every step would wait for all of both.
typedef const __attribute__((address_space(1))) v4i *frag_ptr;
typedef uint32_t v4u_a4 __attribute__((ext_vector_type(4), aligned(4)));  // any word address

// ------------------------------------------------------------- preparation
// c in fixed point, painted over the template: one workgroup per segment.
// Pixel i of a segment gets rint(c scale (i + 1)) - rint(c scale i), so that
// the rounding of a segment's pixels adds up to less than one unit instead of
// A_i times the rounding of c_i.
__global__ __launch_bounds__(64) void dense_paint(const int4 *__restrict__ geom,
                                                  const double *__restrict__ c64, double scale,
                                                  int W, long long *__restrict__ img) {
  const int4 g = geom[blockIdx.x];
  const double c = c64[blockIdx.x] * scale;
  const int n = g.z * g.w;
  const double whole = rint(c), part = c - whole;  // the part's multiples stay exact enough
  for (int i = threadIdx.x; i < n; i += 64) {
    const int y = i / g.z, x = i - y * g.z;
    img[(long long)(g.y + y) * W + g.x + x] =
        (long long)whole + (long long)(rint(part * (i + 1)) - rint(part * i));
  }
}

// A operands: one thread per (step, lane) writes its 16 bytes of every digit,
// leading digit first: frag[(step * D + d) * 64 + lane], steps ordered by
// column group x, then by rows.
template <int D>
__global__ __launch_bounds__(64) void dense_pack(const long long *__restrict__ img, int W, int H,
                                                 v4i *__restrict__ frag) {
  const int n4 = dense_rows4(H), step = blockIdx.x, xg = step / n4;
  const int lane = threadIdx.x, y = 4 * (step - xg * n4) + (lane >> 4);
  const int x0 = 16 * xg - (lane & 15);
  uint32_t w[D][4] = {};
#pragma unroll
  for (int b = 0; b < 16; ++b) {
    const int x = x0 + b;
    long long c = x >= 0 && x < W && y < H ? img[(long long)y * W + x] : 0;
#pragma unroll
    for (int d = D - 1; d >= 0; --d) {  // balanced digits, last one first
      const int lo = (int)(int8_t)(c & 0xff);
      w[d][b >> 2] |= (uint32_t)(lo & 0xff) << (8 * (b & 3));
      c = (c - lo) >> 8;
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d) {
    v4i o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = (int)w[d][k];
    frag[((long long)step * D + d) * 64 + lane] = o;
  }
}

int launch_dense_pack(const int4 *geom, const double *c64, int K, double scale, int W, int H,
                      int digits, long long *img, void *frag, hipStream_t st) {
  hipLaunchKernelGGL(dense_paint, dim3(K), dim3(64), 0, st, geom, c64, scale, W, img);
  const dim3 grid(dense_steps(W, H));
  v4i *o = static_cast<v4i *>(frag);
  switch (digits) {
    case 2: hipLaunchKernelGGL(dense_pack<2>, grid, dim3(64), 0, st, img, W, H, o); break;
    case 3: hipLaunchKernelGGL(dense_pack<3>, grid, dim3(64), 0, st, img, W, H, o); break;
    case 4: hipLaunchKernelGGL(dense_pack<4>, grid, dim3(64), 0, st, img, W, H, o); break;
    default: hipLaunchKernelGGL(dense_pack<7>, grid, dim3(64), 0, st, img, W, H, o); break;
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Notes in host memory that the work before it on the stream is complete.
__global__ void count_kernel(unsigned long long *p, unsigned long long n) {
  __hip_atomic_store(p, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

int launch_count(unsigned long long *p, unsigned long long n, hipStream_t st) {
  hipLaunchKernelGGL(count_kernel, dim3(1), dim3(1), 0, st, p, n);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ------------------------------------------------------------------ scoring
// Rows [y0, y0 + rows) x columns [x0, x0 + 4 n4) of the frame to LDS, each
// pixel as f - 128 in a byte, `pitch` bytes per row.  Pixels come from the sum
// table: f(x, y) is the one-pixel box sum of Eq. (11).  A thread walks down a
// stripe of rows with four columns, RB rows of table entries requested at a
// time (a stripe is 20 to 40 rows: the staging is a few memory latencies).
// Table rows past N and entries past the pitch are clamped: only offsets
// outside the valid range and zero rows of A use such pixels.
template <int NT, int RB>
__device__ __forceinline__ void dense_region(const uint32_t *__restrict__ S, int P, int N, int x0,
                                             int y0, int rows, int n4, int pitch,
                                             uint8_t *__restrict__ lds, int t) {
  const int ns = max(1, NT / n4), per = (rows + ns - 1) / ns;
  for (int unit = t; unit < n4 * ns; unit += NT) {
    const int stripe = unit / n4, c4 = unit - stripe * n4;
    const int ra = stripe * per, rb = min(rows, ra + per);
    const int c = min(x0 + 4 * c4, P - 4), e = min(x0 + 4 * c4 + 4, P - 1);
    auto row = [&](int r, uint32_t (&d)[4]) {  // horizontal differences of table row r
      const uint32_t *p = S + (long long)min(r, N) * P;
      const uint4 a = *reinterpret_cast<const uint4 *>(p + c);
      const uint32_t z = p[e];
      d[0] = a.y - a.x;
      d[1] = a.z - a.y;
      d[2] = a.w - a.z;
      d[3] = z - a.w;
    };
    uint32_t up[4];
    row(y0 + ra, up);
    for (int r = ra; r < rb; r += RB) {
      uint32_t d[RB][4];
#pragma unroll
      for (int k = 0; k < RB; ++k) row(y0 + min(r + k, rb - 1) + 1, d[k]);
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        if (r + k < rb) {
          const uint32_t px = (d[k][0] - up[0]) | (d[k][1] - up[1]) << 8 |
                              (d[k][2] - up[2]) << 16 | (d[k][3] - up[3]) << 24;
          *reinterpret_cast<uint32_t *>(lds + (r + k) * pitch + 4 * c4) = px ^ 0x80808080u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) up[q] = d[k][q];
      }
    }
  }
}

// Four consecutive entries of a table row from entry x on, all when x + 3 is
// inside the pitch, else each from the nearest entry inside it.
__device__ __forceinline__ v4u_a4 dense_row4(const uint32_t *__restrict__ p, int x, int P) {
  if (x + 3 < P) return *reinterpret_cast<const v4u_a4 *>(p + x);
  v4u_a4 o;
#pragma unroll
  for (int k = 0; k < 4; ++k) o[k] = p[min(x + k, P - 1)];
  return o;
}

// The products of one tile of 128 x (2 NW RV) offsets, by a workgroup; wave w
// takes offset rows 2 w RV .. 2 w RV + 2 RV - 1, and lane (j = lane mod 16, g =
// lane / 16) ends with the offsets u0 + 16 (j mod 8) + 4 g + 0..3 of rows
// v0 + RV (2 w + j / 8) + r.  (Against 256 x (NW RV): fewer staged bytes per
// offset and less waste at the right edge.)  Template rows are taken in passes
// of a.hb, whose frame rows are staged in LDS.  Per step a wave loads D
// operands A (from the caches: every wave of the launch reads the same ones)
// and min(RV, 4) operands B (LDS) for D RV instructions.
// `stage(first row, rows, column quads)` stages frame rows below v0.
template <int D, int RV, int NW, class Stage>
__device__ __forceinline__ void dense_products(Stage stage, const DenseArgs &a, int row0,
                                               const uint8_t *lds8, int lane,
                                               v4i (&acc)[RV][D]) {
  constexpr int BV = 2 * NW * RV;
  const frag_ptr frag = (frag_ptr)a.frag;
  const int j = lane & 7, g = lane >> 4;
#pragma unroll
  for (int r = 0; r < RV; ++r)
#pragma unroll
    for (int d = 0; d < D; ++d) acc[r][d] = v4i{0, 0, 0, 0};

  // B of offset rows row0 + t .. t + NB - 1 (t = 4 y for the step of template
  // rows 4 y .. 4 y + 3), two register sets: with eight rows per wave a step
  // uses both (rows 0-3, 4-7) and the first is the next step's second; with
  // fewer the second holds the next step's.  A set is reloaded as soon as its
  // last use is issued, A's two sets one step ahead (requested before the step
  // they are not used in, so that waiting for one leaves the other in flight).
  constexpr int NB = RV < 4 ? RV : 4;
  const int G = a.G, pitch = a.pitch, n4all = dense_rows4(a.H), hb4 = a.hb >> 2;
  for (int yp4 = 0; yp4 < n4all; yp4 += hb4) {
    const int n4 = min(hb4, n4all - yp4);
    if (yp4) __syncthreads();
    stage(4 * yp4, BV + 4 * n4 - 1, 28 + 4 * G);
    __syncthreads();
    // A of the pass's steps in order, the last one's again after it
    frag_ptr fa = frag + (long long)yp4 * (D * 64) + lane;
    int ax = 0, ay = 0;
    auto load_A = [&](v4i(&A)[D]) {
#pragma unroll
      for (int d = 0; d < D; ++d) A[d] = fa[d * 64];
      const bool wrap = ++ay == n4;
      ax += wrap;
      ay = wrap ? 0 : ay;
      fa += ax >= G ? 0 : (wrap ? n4all - n4 + 1 : 1) * (D * 64);
    };
    v4i A0[D], A1[D], b0[NB], b1[NB];
    load_A(A0);
    const uint8_t *base = lds8 + (row0 + g) * pitch + 16 * j;
    for (int x = 0; x < G; ++x, base += 16) {
      auto load_B = [&](int y, v4i(&b)[NB]) {
#pragma unroll
        for (int r = 0; r < NB; ++r)
          b[r] = *reinterpret_cast<const v4i *>(base + (4 * y + r) * pitch);
      };
      auto mul = [&](const v4i(&A)[D], const v4i(&b)[NB], int r0) {
#pragma unroll
        for (int r = 0; r < NB; ++r)
#pragma unroll
          for (int d = 0; d < D; ++d)
            acc[r0 + r][d] =
                __builtin_amdgcn_mfma_i32_16x16x64_i8(A[d], b[r], acc[r0 + r][d], 0, 0, 0);
      };
      load_B(0, b0);
      load_B(1, b1);
      for (int y = 0; y < n4; y += 2) {
        const bool more = y + 2 < n4;
        load_A(A1);
        mul(A0, b0, 0);
        if (RV > 4 || more) load_B(y + 2, b0);
        if constexpr (RV > 4) mul(A0, b1, 4);
        load_A(A0);
        mul(A1, b1, 0);
        if (more) load_B(y + 3, b1);
        if constexpr (RV > 4) mul(A1, b0, 4);
      }
    }
  }
}

// Calls f(r, sum f (Eq. (13)), V as double) for the lane's rows v0 + r, four
// consecutive offsets from column u each; V is the exact window energy (n
// times Eq. (16), an integer below 2^53 where the window is one exact box of
// squares).  Away from the table's right edge, and for such windows, all eight
// corner loads of a row are 16 bytes at any word address; with eight rows per
// wave half (two waves a SIMD in any case) the next row's are requested before
// this one's are used.
template <int RV, bool LOW, class F>
__device__ __forceinline__ void dense_windows(const uint32_t *__restrict__ S,
                                              const uint32_t *__restrict__ S2, const DenseArgs &a,
                                              int u0, int u, int v0, F f) {
  const int uc = min(u, a.nu - 1);
  const double n = (double)a.n;
  if (u0 + kDenseBU + 3 + a.W <= a.P && a.sq_rows >= a.H) {
    constexpr bool AHEAD = RV >= 8 && !LOW;
    v4u_a4 c[2][8];
    const long long down = (long long)a.H * a.P;
    auto load = [&](int r, v4u_a4(&q)[8]) {
      const long long o = (long long)min(v0 + r, a.nv - 1) * a.P + uc;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint32_t *p = (t ? S2 : S) + o;
        q[4 * t] = *reinterpret_cast<const v4u_a4 *>(p);
        q[4 * t + 1] = *reinterpret_cast<const v4u_a4 *>(p + a.W);
        q[4 * t + 2] = *reinterpret_cast<const v4u_a4 *>(p + down);
        q[4 * t + 3] = *reinterpret_cast<const v4u_a4 *>(p + down + a.W);
      }
    };
    if (AHEAD) load(0, c[0]);
#pragma unroll
    for (int r = 0; r < RV; ++r) {
      if (!AHEAD) load(r, c[r & 1]);
      if (AHEAD && r + 1 < RV) load(r + 1, c[(r + 1) & 1]);
      if (AHEAD) __builtin_amdgcn_sched_barrier(0);
      const v4u_a4(&q)[8] = c[r & 1];
      const v4u_a4 sf = (q[3] - q[2]) - (q[1] - q[0]), sf2 = (q[7] - q[6]) - (q[5] - q[4]);
      double V[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double fs = (double)sf[k];
        V[k] = __builtin_fma(n, (double)sf2[k], -(fs * fs));
      }
      f(r, sf, V);
      __builtin_amdgcn_sched_barrier(0);
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < RV; ++r) {
    const int v = min(v0 + r, a.nv - 1);
    const uint32_t *t0 = S + (long long)v * a.P, *t1 = t0 + (long long)a.H * a.P;
    const v4u_a4 sf = (dense_row4(t1, uc + a.W, a.P) - dense_row4(t1, uc, a.P)) -
                      (dense_row4(t0, uc + a.W, a.P) - dense_row4(t0, uc, a.P));
    u64 sf2[4] = {0, 0, 0, 0};
    for (int y = 0; y < a.H; y += a.sq_rows) {  // Eq. (15), in exact boxes
      const uint32_t *q0 = S2 + (long long)(v + y) * a.P;
      const uint32_t *q1 = q0 + (long long)min(a.sq_rows, a.H - y) * a.P;
      const v4u_a4 b = (dense_row4(q1, uc + a.W, a.P) - dense_row4(q1, uc, a.P)) -
                       (dense_row4(q0, uc + a.W, a.P) - dense_row4(q0, uc, a.P));
#pragma unroll
      for (int k = 0; k < 4; ++k) sf2[k] += b[k];
    }
    double V[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      V[k] = (double)(long long)((u64)(uint32_t)a.n * sf2[k] - (u64)sf[k] * sf[k]);
    f(r, sf, V);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Numerator of Eq. (12) from a lane's digit sums: their value less the digits'
// own mean term (the rounded c need not sum to zero), in FP64.
template <int D>
__device__ __forceinline__ double dense_num(const v4i (&acc)[D], int k, uint32_t sf,
                                            const DenseArgs &a) {
  double T;
  if constexpr (D == kDenseDigits) {
    const long long hi = ((long long)acc[0][k] << 16) + ((long long)acc[1][k] << 8) + acc[2][k];
    const long long lo = ((long long)acc[3][k] << 24) + ((long long)acc[4][k] << 16) +
                         ((long long)acc[5][k] << 8) + acc[6][k];
    T = __builtin_fma((double)hi, 4294967296.0, (double)lo);
  } else {
    T = (double)acc[0][k];  // below 2^55, sums of digits exact below 2^53
#pragma unroll
    for (int d = 1; d < D; ++d) T = __builtin_fma(T, 256.0, (double)acc[d][k]);
  }
  return (T - a.csum * ((double)sf * a.inv_n - 128.0)) * a.inv_scale;
}

template <int D, int RV, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void dense_kernel(
    const uint32_t *__restrict__ S, const uint32_t *__restrict__ S2, DenseArgs a) {
  extern __shared__ __align__(16) uint8_t lds8[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // tiles row by row, a contiguous range of them per XCD (workgroups go round
  // the XCDs), so that neighbouring tiles share the table rows in its L2
  const int per = (int)gridDim.x >> 3;
  const int tile = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (tile >= a.ntu * a.ntv) return;
  const int tv = tile / a.ntu, u0 = (tile - tv * a.ntu) * kDenseBU, v0 = tv * 2 * NW * RV;
  const int row0 = RV * (2 * wave + ((lane >> 3) & 1));  // the lane's first offset row
  v4i acc[RV][D];
  auto stage = [&](int y, int rows, int n4) {
    dense_region<64 * NW, (RV >= 8 && D != 2) ? 16 : 8>(S, a.P, a.N, u0, v0 + y, rows, n4, a.pitch,
                                                        lds8, threadIdx.x);
  };
  dense_products<D, RV, NW>(stage, a, row0, lds8, lane, acc);

  const int u = u0 + 16 * (lane & 7) + 4 * (lane >> 4);
  dense_windows<RV, false>(S, S2, a, u0, u, v0 + row0,
                           [&](int r, const v4u_a4 &sf, const double(&V)[4]) {
    const int v = v0 + row0 + r;
    const long long o = (long long)v * a.rho_pitch + u;
    if (v >= a.nv) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double num = dense_num<D>(acc[r], k, sf[k], a);
      double rho;
      if constexpr (D == kDenseDigits) {
        rho = num / sqrt(V[k] / (double)a.n * a.q_k);
      } else {
        // 1 / sqrt of the energy in FP64 (the FP32 estimate and one Newton
        // step), so that the result is rounded once
        const double e = V[k] * a.qnd, y = (double)__builtin_amdgcn_rsqf((float)e);
        rho = num * (y * __builtin_fma(-0.5 * e * y, y, 1.5));
      }
      if (V[k] == 0.0) rho = 0.0;
      if (u + k < a.nu) {
        if constexpr (D == kDenseDigits)
          static_cast<double *>(a.rho)[o + k] = rho;
        else
          static_cast<float *>(a.rho)[o + k] = (float)rho;
        if (a.degen) a.degen[o + k] = V[k] == 0.0 ? 1 : 0;
      }
    }
  });
}

// The filter of the top-k search (topk_filter.hip): rho of many pairs in
// one launch, from two digits of c (its values only choose which offsets are
// scored again; three digits where two would leave a bound above 2^-12),
// one workgroup per item {pair, tile} (pair -1: none).  A wave writes its
// RV x 64 x 4 values as they lie in its lanes (offsets past the valid range as
// -inf), and its block's largest rho; offsets whose window is nearly uniform
// (energy below n / 100, where the segment form's FP32 error bound grows) do
// not count there but raise a second maximum.
template <int D, int RV, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void dense_filter(
    const uint32_t *__restrict__ s, const uint32_t *__restrict__ s2, long long frame_stride,
    const FilterPair *__restrict__ fps, const int2 *__restrict__ items, float *__restrict__ map,
    float2 *__restrict__ bmax, int *__restrict__ zero, int n_zero) {
  extern __shared__ __align__(16) uint8_t lds8[];
  for (int i = blockIdx.x * (64 * NW) + threadIdx.x; i < n_zero; i += gridDim.x * (64 * NW))
    zero[i] = 0;  // counters of the launches after this one
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int2 it = items[blockIdx.x];
  if (it.x < 0) return;
  const FilterPair &fp = fps[it.x];
  const DenseArgs a = fp.a;
  const uint32_t *S = s + (long long)fp.frame * frame_stride;
  const uint32_t *S2 = s2 + (long long)fp.frame * frame_stride;
  const int tile = it.y, tv = tile / a.ntu;
  const int u0 = (tile - tv * a.ntu) * kDenseBU, v0 = tv * 2 * NW * RV;
  const int row0 = RV * (2 * wave + ((lane >> 3) & 1));
  v4i acc[RV][D];
  auto stage = [&](int y, int rows, int n4) {
    dense_region<64 * NW, (RV >= 8 && D != 2) ? 16 : 8>(S, a.P, a.N, u0, v0 + y, rows, n4, a.pitch,
                                                        lds8, threadIdx.x);
  };
  dense_products<D, RV, NW>(stage, a, row0, lds8, lane, acc);

  const int u = u0 + 16 * (lane & 7) + 4 * (lane >> 4);
  const double low = (double)a.n * (double)a.n * 0.01;
  const int block = tile * NW + wave;
  float4 *o = reinterpret_cast<float4 *>(map + fp.map0 + (long long)block * (RV * 256)) + lane;
  float top = -__builtin_inff(), top_low = -__builtin_inff();
  dense_windows<RV, D == 2>(S, S2, a, u0, u, v0 + row0,
                            [&](int r, const v4u_a4 &sf, const double(&V)[4]) {
    const bool row_ok = v0 + row0 + r < a.nv;
    float w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float num = (float)dense_num<D>(acc[r], k, sf[k], a);
      const float y = __builtin_amdgcn_rsqf((float)(V[k] * a.qnd));
      w[k] = V[k] == 0.0 ? 0.f : num * y;
      if (!row_ok || u + k >= a.nu) w[k] = -__builtin_inff();
      const bool flat = V[k] != 0.0 && V[k] < low;
      top_low = fmaxf(top_low, flat ? w[k] : -__builtin_inff());
      top = fmaxf(top, flat ? -__builtin_inff() : w[k]);
    }
    o[r * 64] = make_float4(w[0], w[1], w[2], w[3]);
  });
  const uint32_t m = wave_incl_max(float_order(top)), ml = wave_incl_max(float_order(top_low));
  if (lane == 63) bmax[fp.block0 + block] = make_float2(float_unorder(m), float_unorder(ml));
}

// The two-threshold search's filter: which offsets of the tiles that hold many
// survivors of the fast pass can reach the slow threshold, as one bit each, in
// one word per lane (bit 4 r + k: row r, column k of the lane's offsets).  Two
// digits of c and a margin of their error decide, so that the slow pass in FP64
// sees a few per cent of the survivors (2 frames 1920 x 1080 x 4 templates 64 x
// 64, 1.69 million survivors: 92 us here, the slow pass 810 -> 58 us).
template <int D, int RV, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void dense_above(
    const uint32_t *__restrict__ s, const uint32_t *__restrict__ s2, long long frame_stride,
    const FilterPair *__restrict__ fps, const int2 *__restrict__ items,
    const int *__restrict__ tile_count, uint32_t *__restrict__ bits) {
  extern __shared__ __align__(16) uint8_t lds8[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int2 it = items[blockIdx.x];
  if (it.x < 0) return;
  const FilterPair &fp = fps[it.x];
  const int tile = it.y, tv = tile / fp.a.ntu, tu = tile - tv * fp.a.ntu;
  if (tile_survivors(fp, tile_count, tu, tv, 2 * NW * RV) < fp.min_count) return;
  const DenseArgs a = fp.a;
  const uint32_t *S = s + (long long)fp.frame * frame_stride;
  const uint32_t *S2 = s2 + (long long)fp.frame * frame_stride;
  const int u0 = tu * kDenseBU, v0 = tv * 2 * NW * RV;
  const int row0 = RV * (2 * wave + ((lane >> 3) & 1));
  v4i acc[RV][D];
  auto stage = [&](int y, int rows, int n4) {
    dense_region<64 * NW, (RV >= 8 && D != 2) ? 16 : 8>(S, a.P, a.N, u0, v0 + y, rows, n4, a.pitch,
                                                        lds8, threadIdx.x);
  };
  dense_products<D, RV, NW>(stage, a, row0, lds8, lane, acc);

  const int u = u0 + 16 * (lane & 7) + 4 * (lane >> 4);
  const float above = fp.above;
  uint32_t word = 0;
  dense_windows<RV, D == 2>(S, S2, a, u0, u, v0 + row0,
                            [&](int r, const v4u_a4 &sf, const double(&V)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float num = (float)dense_num<D>(acc[r], k, sf[k], a);
      const float y = __builtin_amdgcn_rsqf((float)(V[k] * a.qnd));
      const float rho = V[k] == 0.0 ? 0.f : num * y;
      word |= (rho >= above ? 1u : 0u) << (4 * r + k);
    }
    asm volatile("" : "+v"(word));  // row by row: all rows' loads at once would spill
  });
  bits[fp.map0 + (long long)(tile * NW + wave) * 64 + lane] = word;
}

// ------------------------------------------------------- straight from a frame
// Rows [y0, y0 + rows) x columns [x0, x0 + 4 n4) of the frame to LDS as f - 128
// (rows past the frame as its last, columns past it as 0).
template <int NT>
__device__ __forceinline__ void frame_region(const uint8_t *__restrict__ f, int M, int N,
                                             int f_pitch, int x0, int y0, int rows, int n4,
                                             int pitch, uint8_t *__restrict__ lds, int t) {
  const int ns = max(1, NT / n4), per = (rows + ns - 1) / ns;
  for (int unit = t; unit < n4 * ns; unit += NT) {
    const int stripe = unit / n4, c4 = unit - stripe * n4, x = x0 + 4 * c4;
    const int ra = stripe * per, rb = min(rows, ra + per);
    typedef uint32_t u32_a1 __attribute__((aligned(1)));
    auto px4 = [&](int r) {
      const uint8_t *row = f + (size_t)min(r, N - 1) * f_pitch;
      if (x + 3 < M) return (uint32_t)*reinterpret_cast<const u32_a1 *>(row + x);
      uint32_t w = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (x + q < M) w |= (uint32_t)row[x + q] << (8 * q);
      return w;
    };
    for (int r = ra; r < rb; r += 16) {
      uint32_t w[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) w[k] = px4(y0 + min(r + k, rb - 1));
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (r + k < rb)
          *reinterpret_cast<uint32_t *>(lds + (r + k) * pitch + 4 * c4) = w[k] ^ 0x80808080u;
    }
  }
}

// A rho map from the frame itself, for templates whose region fits one pass and
// whose windows are one exact box of squares: no tables are built, which for a
// small frame are two launches more and most of the time.  The windows' sums
// come from the staged region: each column's sums of f and f^2 over H rows for
// every offset row (a thread takes four columns of some rows: the first H rows
// added up, then one row added and one taken off per step), then running sums
// along each row, in 32-bit modular arithmetic as in the tables.
// What bounds it: one workgroup's chain of staging, sums, scans and matrix
// steps where the frame is small (640 x 480, 32 x 32: 12.4 us a call, where the
// tile-local form took 17.3 at K 21 and tables and a map 21.9; 64 x 64: 19.3
// against 29.2), the matrix steps on larger ones (1920 x 1080, 64 x 64: 38.8
// against 58.2).
template <int RV, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void dense_frame(
    const uint8_t *__restrict__ f, int M, int f_pitch, DenseArgs a,
    long long *__restrict__ energy) {
  extern __shared__ __align__(16) uint8_t lds8[];
  constexpr int D = 3, BV = 2 * NW * RV, NT = 64 * NW;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tv = (int)blockIdx.x / a.ntu;
  const int u0 = ((int)blockIdx.x - tv * a.ntu) * kDenseBU, v0 = tv * BV;
  const int row0 = RV * (2 * wave + ((lane >> 3) & 1));
  const int C = 112 + 16 * a.G, sp = C + 4;  // region columns; pitch of the sums (words)
  uint32_t *const ps = reinterpret_cast<uint32_t *>(lds8 + (BV + a.hb - 1) * a.pitch);
  uint32_t *const pq = ps + BV * sp;
  v4i acc[RV][D];
  auto stage = [&](int y, int rows, int n4) {
    frame_region<NT>(f, M, a.N, f_pitch, u0, v0 + y, rows, n4, a.pitch, lds8, t);
    __syncthreads();
    // sums over H rows: column c of offset row v at [v][c + 1]
    const int nq = C / 4, ns = max(1, NT / nq), per = (BV + ns - 1) / ns;
    for (int unit = t; unit < nq * ns; unit += NT) {
      const int stripe = unit / nq, q4 = unit - stripe * nq;
      const int va = stripe * per, vb = min(BV, va + per);
      const uint8_t *col = lds8 + 4 * q4;
      uint32_t lo = 0, hi = 0, in[4] = {0, 0, 0, 0}, gone[4] = {0, 0, 0, 0};
      auto px = [&](int r) {
        return *reinterpret_cast<const uint32_t *>(col + r * a.pitch) ^ 0x80808080u;
      };
      auto squares = [&](uint32_t w, uint32_t(&s)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t m = w & (0xffu << (8 * q));
          s[q] = __builtin_amdgcn_udot4(m, m, s[q], false);
        }
      };
      auto add = [&](uint32_t w) {  // f as two 16-bit halves of a word: H <= 257 rows
        lo += w & 0x00ff00ffu;
        hi += (w >> 8) & 0x00ff00ffu;
        squares(w, in);
      };
      if (va < vb) {
#pragma unroll 8
        for (int r = 0; r < a.H; ++r) add(px(va + r));
        for (int v = va;; ++v) {
          const uint32_t s[4] = {lo & 0xffffu, hi & 0xffffu, lo >> 16, hi >> 16};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            ps[v * sp + 4 * q4 + 1 + q] = s[q];
            pq[v * sp + 4 * q4 + 1 + q] = in[q] - gone[q];
          }
          if (v + 1 >= vb) break;
          const uint32_t w = px(v);
          lo -= w & 0x00ff00ffu;
          hi -= (w >> 8) & 0x00ff00ffu;
          squares(w, gone);
          add(px(v + a.H));
        }
      }
    }
    __syncthreads();
    // running sums along the rows, in place
    for (int i = wave; i < 2 * BV; i += NW) {
      uint32_t *row = ps + i * sp;  // the rows of pq follow those of ps
      if (lane == 0) row[0] = 0;
      uint32_t carry = 0;
      for (int c0 = 0; c0 < C; c0 += 256) {
        const int c = c0 + 4 * lane;
        uint32_t p[4] = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = (q ? p[q - 1] : 0u) + (c < C ? row[1 + c + q] : 0u);
        const uint32_t incl = wave_incl_scan(p[3]), base = carry + incl - p[3];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (c < C) row[1 + c + q] = base + p[q];
        carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      }
    }
  };
  dense_products<D, RV, NW>(stage, a, row0, lds8, lane, acc);

  const int ul = 16 * (lane & 7) + 4 * (lane >> 4), u = u0 + ul;
  const double n = (double)a.n;
#pragma unroll
  for (int r = 0; r < RV; ++r) {
    const int v = v0 + row0 + r;
    const uint32_t *sr = ps + (row0 + r) * sp + ul, *qr = pq + (row0 + r) * sp + ul;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t sf = sr[a.W + k] - sr[k];   // Eq. (13)
      const uint32_t sf2 = qr[a.W + k] - qr[k];  // Eq. (15)
      const double fs = (double)sf, V = __builtin_fma(n, (double)sf2, -(fs * fs));
      const double e = V * a.qnd, y = (double)__builtin_amdgcn_rsqf((float)e);
      double rho = dense_num<D>(acc[r], k, sf, a) * (y * __builtin_fma(-0.5 * e * y, y, 1.5));
      if (V == 0.0) rho = 0.0;
      if (v < a.nv && u + k < a.nu) {
        const long long o = (long long)v * a.rho_pitch + u + k;
        static_cast<float *>(a.rho)[o] = (float)rho;
        if (a.degen) a.degen[o] = V == 0.0 ? 1 : 0;
        if (energy) energy[o] = (long long)V;
      }
    }
  }
}

template <int RV, int NW>
static int frame_go(const DenseArgs &a, const uint8_t *f, int M, int f_pitch, long long *energy,
                    hipStream_t st) {
  static bool attr = false;
  const void *fn = (const void *)dense_frame<RV, NW>;
  if (!attr) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kTileMaxLds) !=
        hipSuccess)
      return -1;
    attr = true;
  }
  const size_t lds = dense_frame_lds(a);
  hipLaunchKernelGGL((dense_frame<RV, NW>), dim3(a.ntu * a.ntv), dim3(64 * NW), lds, st, f, M,
                     f_pitch, a, energy);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_dense_frame(const DenseArgs &a, const uint8_t *f, int M, int f_pitch,
                       long long *energy, hipStream_t st) {
  if (a.digits != 3) return -1;
  switch (a.rv) {
    case 2: return frame_go<2, kDenseNW>(a, f, M, f_pitch, energy, st);
    case 4: return frame_go<4, kDenseNW>(a, f, M, f_pitch, energy, st);
    default: return -1;
  }
}

template <int D, int RV, int NW>
static int dense_go(const DenseArgs &a, hipStream_t st) {
  static bool attr = false;
  const void *fn = (const void *)dense_kernel<D, RV, NW>;
  if (!attr) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kTileMaxLds) !=
        hipSuccess)
      return -1;
    attr = true;
  }
  const int lds = (2 * NW * RV + a.hb - 1) * a.pitch;
  const int grid = (a.ntu * a.ntv + 7) / 8 * 8;
  hipLaunchKernelGGL((dense_kernel<D, RV, NW>), dim3(grid), dim3(64 * NW), lds, st, a.s, a.s2, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_dense(const DenseArgs &a, hipStream_t st) {
  switch (a.digits * 100 + a.rv) {
    case 308: return dense_go<3, 8, kDenseNW>(a, st);
    case 304: return dense_go<3, 4, kDenseNW>(a, st);
    case 302: return dense_go<3, 2, kDenseNW>(a, st);
    case 404: return dense_go<4, 4, kDenseNW>(a, st);
    case 402: return dense_go<4, 2, kDenseNW>(a, st);
    case 704: return dense_go<7, 4, kDenseNW>(a, st);
    case 702: return dense_go<7, 2, kDenseNW>(a, st);
    default: return -1;
  }
}

template <int D, int RV, int NW>
static int filter_go(const uint32_t *s, const uint32_t *s2, long long frame_stride,
                     const FilterPair *fps, const int2 *items, int n_items, int lds, float *map,
                     float2 *bmax, int *zero, int n_zero, hipStream_t st) {
  static bool attr = false;
  const void *fn = (const void *)dense_filter<D, RV, NW>;
  if (!attr) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kTileMaxLds) !=
        hipSuccess)
      return -1;
    attr = true;
  }
  hipLaunchKernelGGL((dense_filter<D, RV, NW>), dim3(n_items), dim3(64 * NW), lds, st, s, s2,
                     frame_stride, fps, items, map, bmax, zero, n_zero);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_dense_filter(int digits, int rv, const uint32_t *s, const uint32_t *s2,
                        long long frame_stride, const FilterPair *fps, const int2 *items,
                        int n_items, int lds, float *map, float2 *bmax, int *zero, int n_zero,
                        hipStream_t st) {
  switch (digits * 100 + rv) {
#define SNCC_FILTER(D, RV)                                                                       \
  case D * 100 + RV:                                                                             \
    return filter_go<D, RV, kDenseNW>(s, s2, frame_stride, fps, items, n_items, lds, map, bmax, \
                                      zero, n_zero, st)
    SNCC_FILTER(2, 8);
    SNCC_FILTER(2, 4);
    SNCC_FILTER(2, 2);
    SNCC_FILTER(3, 8);
    SNCC_FILTER(3, 4);
    SNCC_FILTER(3, 2);
#undef SNCC_FILTER
    default: return -1;
  }
}

template <int D, int RV, int NW>
static int above_go(const uint32_t *s, const uint32_t *s2, long long frame_stride,
                    const FilterPair *fps, const int2 *items, int n_items, int lds,
                    const int *tile_count, uint32_t *bits, hipStream_t st) {
  static bool attr = false;
  const void *fn = (const void *)dense_above<D, RV, NW>;
  if (!attr) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kTileMaxLds) !=
        hipSuccess)
      return -1;
    attr = true;
  }
  hipLaunchKernelGGL((dense_above<D, RV, NW>), dim3(n_items), dim3(64 * NW), lds, st, s, s2,
                     frame_stride, fps, items, tile_count, bits);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_dense_above(int digits, int rv, const uint32_t *s, const uint32_t *s2,
                       long long frame_stride, const FilterPair *fps, const int2 *items,
                       int n_items, int lds, const int *tile_count, uint32_t *bits,
                       hipStream_t st) {
  switch (digits * 100 + rv) {
#define SNCC_ABOVE(D, RV)                                                                       \
  case D * 100 + RV:                                                                            \
    return above_go<D, RV, kDenseNW>(s, s2, frame_stride, fps, items, n_items, lds, tile_count, \
                                     bits, st)
    SNCC_ABOVE(2, 8);
    SNCC_ABOVE(2, 4);
    SNCC_ABOVE(2, 2);
    SNCC_ABOVE(3, 8);
    SNCC_ABOVE(3, 4);
    SNCC_ABOVE(3, 2);
#undef SNCC_ABOVE
    default: return -1;
  }
}

}  // namespace sncc
