// Pointwise part of an LSTM cell with FP16 tensors and FP32 math (paper Sec. 3.3, "point-wise operations"; the
// recurrent layers of Sec. 4), forward and backward, for gfx950.  The matrix products around it are the GEMM entry
// points.  Gate order (i, f, g, o) along the 4H axis.  A thread owns 4 consecutive hidden units of one batch row
// (or one of the up to 3 that are left at its end), wherever the rows start (250 x 8001 forward: 19.5 us element by element, 15.9 so,
// 11.6 with a thread's loads together): every tensor is touched once, 8 bytes per lane.  HBM-bound at large B*H: 30 bytes per hidden unit forward
// (two pre-activation tensors of 4 gates, previous state in; activations, state, output out), 22 bytes backward.
#include "gemm_parts.h"

typedef _Float16 lh4 __attribute__((ext_vector_type(4), aligned(2)));    // at any address: 8-byte accesses need no more alignment than their elements

namespace {

constexpr int kT = 256;

__device__ __forceinline__ float sigmoidf_(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
// tanh to a relative error of about 1e-6 (the results are stored as FP16, whose step is 5e-4): (1 - t) / (1 + t) with
// t = exp(-2|x|); below 2^-4, where 1 - t cancels, the odd series x - x^3/3 + 2x^5/15 (next term 3e-9 relative).
// A third of the instructions of the library routine, which matters here: the kernels are within reach of HBM speed.
__device__ __forceinline__ float tanhf_(float x) {
  const float ax = fabsf(x);
  const float t = __expf(-2.0f * ax);
  const float big = (1.0f - t) * __builtin_amdgcn_rcpf(1.0f + t);
  const float x2 = ax * ax;
  const float small = ax * (1.0f + x2 * (-0.33333334f + x2 * 0.13333334f));
  return copysignf(ax < 0.0625f ? small : big, x);
}

// NT: nontemporal accesses, for tensors that outgrow the 256 MB memory-side cache (streaming them is faster there,
// slower for small tensors that the next kernel reads again).
template <int V> struct RawOf { typedef lh4 type; };
template <> struct RawOf<1> { typedef _Float16 type; };
template <int V> using Raw = typename RawOf<V>::type;
template <int V, bool NT>
__device__ __forceinline__ Raw<V> raw(const uint16_t* p) {
  const Raw<V>* q = reinterpret_cast<const Raw<V>*>(p);
  if constexpr (NT) return __builtin_nontemporal_load(q);
  else return *q;
}
template <int V>
__device__ __forceinline__ void widen(const Raw<V>& q, float (&v)[V]) {
  if constexpr (V == 1) {
    v[0] = (float)q;
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = (float)q[e];
  }
}
template <int V, bool NT = false>
__device__ __forceinline__ void ld16(const uint16_t* p, float (&v)[V]) { widen<V>(raw<V, NT>(p), v); }
template <int V, bool NT = false>
__device__ __forceinline__ void st16(uint16_t* p, const float (&v)[V]) {
  if constexpr (V == 4) {
    lh4 q;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = (_Float16)mpt_rounded_f32(v[e]);
    if constexpr (NT) __builtin_nontemporal_store(q, reinterpret_cast<lh4*>(p));
    else *reinterpret_cast<lh4*>(p) = q;
  } else {
    *reinterpret_cast<_Float16*>(p) = (_Float16)mpt_rounded_f32(v[0]);
  }
}

using mpt_gemm::FastDiv;

// Which V cells a thread of the forward kernel has.  ROWS: a workgroup lies in one row, whose addresses are then formed once per
// wavefront, a lane adding 32 bits; else threads are dealt over the rows one after the other.  The division of a 64-bit index
// per thread and the 64-bit addresses that stood here were a third of the kernel's instructions.  (The backward kernel, whose loads
// all go out at once, has them under its waits: 64 x 1023 2.5 us with them, 2.7 without.)
struct Share {
  int64_t B;
  uint32_t H, groups, per_row;     // groups of V cells; and the cells left over, one per thread
  FastDiv blocks;                  // ROWS: workgroups per row; else: threads per row
};
template <bool ROWS>
__device__ __forceinline__ bool my_cells(const Share& s, int64_t& b, uint32_t& k) {
  uint32_t q, r;
  if constexpr (ROWS) {
    s.blocks.divmod(blockIdx.x, q, r);
    k = r * kT + threadIdx.x;
    b = q;
    return k < s.per_row;
  } else {
    s.blocks.divmod(blockIdx.x * kT + threadIdx.x, q, k);
    b = q;
    return b < s.B;
  }
}

// V cells of row b from unit j on
template <int V, bool NT>
__device__ __forceinline__ void cell_fwd(int64_t b, uint32_t j, uint32_t H, const uint16_t* __restrict__ gx, int64_t ldgx,
                                         const uint16_t* __restrict__ gr, int64_t ldgr, const float* __restrict__ bias,
                                         const uint16_t* cprev, int64_t ldcp, uint16_t* __restrict__ act, int64_t ldact,
                                         uint16_t* c, int64_t ldc, uint16_t* __restrict__ h, int64_t ldh) {
  // All loads first, those of optional tensors behind one branch each: with a branch behind every load the nine of a thread went out
  // one after the other, each waited for (both changes: 250 x 8001 14.1 -> 11.6 us, 1000 x 8192 44.6 -> 39.4, 256 x 8192 12.5 -> 11.7, 64 x 1023 3.1 -> 2.6).
  float a[4][V], r[4][V], bi[4][V], cp[V];
  Raw<V> qa[4], qr[4], qc;
#pragma unroll
  for (int g = 0; g < 4; ++g) qa[g] = raw<V, NT>(gx + b * ldgx + (int64_t)g * H + j);
  qc = raw<V, NT>(cprev + b * ldcp + j);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    qr[g] = Raw<V>{};
#pragma unroll
    for (int e = 0; e < V; ++e) bi[g][e] = 0.f;
  }
  if (gr != nullptr) {
#pragma unroll
    for (int g = 0; g < 4; ++g) qr[g] = raw<V, NT>(gr + b * ldgr + (int64_t)g * H + j);
  }
  if (bias != nullptr) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < V; ++e) bi[g][e] = bias[(int64_t)g * H + j + e];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) widen<V>(qa[g], a[g]);
  if (gr != nullptr) {                            // (adding nothing would turn -0 into +0)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      widen<V>(qr[g], r[g]);
#pragma unroll
      for (int e = 0; e < V; ++e) a[g][e] = __fadd_rn(a[g][e], r[g][e]);
    }
  }
  if (bias != nullptr) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < V; ++e) a[g][e] = __fadd_rn(a[g][e], bi[g][e]);
  }
  widen<V>(qc, cp);
  float cn[V], hn[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const float i = sigmoidf_(a[0][e]), f = sigmoidf_(a[1][e]), g = tanhf_(a[2][e]), o = sigmoidf_(a[3][e]);
    a[0][e] = i; a[1][e] = f; a[2][e] = g; a[3][e] = o;
    cn[e] = __fadd_rn(__fmul_rn(f, cp[e]), __fmul_rn(i, g));
    hn[e] = __fmul_rn(o, tanhf_(cn[e]));
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) st16<V, NT>(act + b * ldact + (int64_t)g * H + j, a[g]);
  st16<V, NT>(c + b * ldc + j, cn);
  st16<V, NT>(h + b * ldh + j, hn);
}

template <int V, bool NT, bool ROWS>
__global__ __launch_bounds__(kT) void k_lstm_cell_fwd(Share s, const uint16_t* __restrict__ gx, int64_t ldgx,
                                                      const uint16_t* __restrict__ gr, int64_t ldgr, const float* __restrict__ bias,
                                                      const uint16_t* cprev, int64_t ldcp, uint16_t* __restrict__ act, int64_t ldact,
                                                      uint16_t* c, int64_t ldc, uint16_t* __restrict__ h, int64_t ldh) {
  int64_t b;
  uint32_t k;
  if (!my_cells<ROWS>(s, b, k)) return;
  if (V == 1 || k < s.groups) cell_fwd<V, NT>(b, k * V, s.H, gx, ldgx, gr, ldgr, bias, cprev, ldcp, act, ldact, c, ldc, h, ldh);
  else cell_fwd<1, false>(b, s.groups * (V - 1) + k, s.H, gx, ldgx, gr, ldgr, bias, cprev, ldcp, act, ldact, c, ldc, h, ldh);
}

template <int V, bool NT>
__device__ __forceinline__ void cell_bwd(int64_t b, int64_t j, int64_t H, const uint16_t* __restrict__ dh, int64_t lddh,
                                         const uint16_t* dcn, int64_t lddcn, const uint16_t* __restrict__ act, int64_t ldact,
                                         const uint16_t* __restrict__ c, int64_t ldc, const uint16_t* __restrict__ cprev, int64_t ldcp,
                                         uint16_t* __restrict__ da, int64_t ldda, uint16_t* dcp, int64_t lddcp) {
  float a[4][V], dhv[V], dc[V], cv[V], cp[V];
#pragma unroll
  for (int g = 0; g < 4; ++g) ld16<V, NT>(act + b * ldact + g * H + j, a[g]);
  ld16<V, NT>(dh + b * lddh + j, dhv);
  ld16<V, NT>(c + b * ldc + j, cv);
  ld16<V, NT>(cprev + b * ldcp + j, cp);
  if (dcn != nullptr) {
    ld16<V, NT>(dcn + b * lddcn + j, dc);
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e) dc[e] = 0.f;
  }
  float out[4][V], dprev[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const float i = a[0][e], f = a[1][e], g = a[2][e], o = a[3][e];
    const float tc = tanhf_(cv[e]);
    const float d = __fadd_rn(__fmul_rn(__fmul_rn(dhv[e], o), __fsub_rn(1.0f, __fmul_rn(tc, tc))), dc[e]);
    out[0][e] = __fmul_rn(__fmul_rn(d, g), __fmul_rn(i, __fsub_rn(1.0f, i)));
    out[1][e] = __fmul_rn(__fmul_rn(d, cp[e]), __fmul_rn(f, __fsub_rn(1.0f, f)));
    out[2][e] = __fmul_rn(__fmul_rn(d, i), __fsub_rn(1.0f, __fmul_rn(g, g)));
    out[3][e] = __fmul_rn(__fmul_rn(dhv[e], tc), __fmul_rn(o, __fsub_rn(1.0f, o)));
    dprev[e] = __fmul_rn(d, f);
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) st16<V, NT>(da + b * ldda + g * H + j, out[g]);
  st16<V, NT>(dcp + b * lddcp + j, dprev);
}

template <int V, bool NT>
__global__ __launch_bounds__(kT) void k_lstm_cell_bwd(int64_t B, int64_t H, const uint16_t* __restrict__ dh, int64_t lddh,
                                                      const uint16_t* dcn, int64_t lddcn, const uint16_t* __restrict__ act, int64_t ldact,
                                                      const uint16_t* __restrict__ c, int64_t ldc, const uint16_t* __restrict__ cprev, int64_t ldcp,
                                                      uint16_t* __restrict__ da, int64_t ldda, uint16_t* dcp, int64_t lddcp) {
  const int64_t groups = H / V, per_row = groups + H % V;
  const int64_t u = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (u >= B * per_row) return;
  const int64_t b = u / per_row, k = u - b * per_row;
  if (V == 1 || k < groups) cell_bwd<V, NT>(b, k * V, H, dh, lddh, dcn, lddcn, act, ldact, c, ldc, cprev, ldcp, da, ldda, dcp, lddcp);
  else cell_bwd<1, false>(b, groups * (V - 1) + k, H, dh, lddh, dcn, lddcn, act, ldact, c, ldc, cprev, ldcp, da, ldda, dcp, lddcp);
}

// Few cells: one per thread.  A launch whose threads are all on the chip at once takes as long as one of them does, and that is the
// longer the more cells it has, longer still where a wavefront holds a row's left-over cells as well (64 x 1023 forward
// 5.1 us in fours, 3.2 singly, backward 2.9 and 2.2; 512 x 1023 6.8 and 5.4, 4.5 and 4.1; 768 x 1023 8.6 and 10.7, 5.5 and 5.0).
bool one_per_thread(int64_t B, int64_t H) { return B * H <= 512 * 1024; }

// The launch over cells of V: by rows where at most a fifth of the workgroups' threads stay idle so, and where the flat index is too long for 32 bits.
struct Launch { Share s; int64_t grid; bool rows; };
Launch plan(int64_t B, int64_t H, int V) {
  const int64_t groups = H / V, per_row = groups + H % V, blocks = (per_row + kT - 1) / kT, flat = (B * per_row + kT - 1) / kT;
  const bool rows = per_row * 5 >= blocks * kT * 4 || flat * kT > 0xFFFFFFFFLL;
  return {{B, (uint32_t)H, (uint32_t)groups, (uint32_t)per_row, FastDiv((uint32_t)(rows ? blocks : per_row))}, rows ? B * blocks : flat, rows};
}

bool dims_ok(int64_t B, int64_t H) { return B >= 1 && H >= 1 && B <= (1LL << 31) && H <= (1LL << 24); }

}  // namespace

extern "C" int mpt_lstm_cell_fwd(void* stream, int64_t B, int64_t H, const uint16_t* gx, int64_t ldgx, const uint16_t* gr, int64_t ldgr,
                                 const float* bias, const uint16_t* c_prev, int64_t ldcp, uint16_t* act, int64_t ldact,
                                 uint16_t* c, int64_t ldc, uint16_t* h, int64_t ldh) {
  if (gx == nullptr || c_prev == nullptr || act == nullptr || c == nullptr || h == nullptr) return MPT_ERR_NULL;
  if (!dims_ok(B, H) || ldgx < 4 * H || (gr && ldgr < 4 * H) || ldcp < H || ldact < 4 * H || ldc < H || ldh < H) return MPT_ERR_SHAPE;
  if (!mpt_aligned(gx, 2) || !mpt_aligned(gr, 2) || !mpt_aligned(c_prev, 2) || !mpt_aligned(act, 2) || !mpt_aligned(c, 2) || !mpt_aligned(h, 2) ||
      !mpt_aligned(bias, 4))
    return MPT_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool singly = one_per_thread(B, H);
  const Launch l = plan(B, H, singly ? 1 : 4);               // 4 cells (8 bytes) per lane: measured 5.5 vs 5.3 TB/s against 8 cells
  const bool stream_it = B * H * 30 > (192LL << 20);         // bytes moved beyond the memory-side cache
  auto k = singly ? (l.rows ? k_lstm_cell_fwd<1, false, true> : k_lstm_cell_fwd<1, false, false>)
           : stream_it ? (l.rows ? k_lstm_cell_fwd<4, true, true> : k_lstm_cell_fwd<4, true, false>)
                       : (l.rows ? k_lstm_cell_fwd<4, false, true> : k_lstm_cell_fwd<4, false, false>);
  hipLaunchKernelGGL(k, dim3((unsigned)l.grid), dim3(kT), 0, st, l.s, gx, ldgx, gr, ldgr, bias, c_prev, ldcp, act, ldact, c, ldc, h, ldh);
  MPT_LAUNCH_CHECK();
  return MPT_OK;
}

extern "C" int mpt_lstm_cell_bwd(void* stream, int64_t B, int64_t H, const uint16_t* dh, int64_t lddh, const uint16_t* dc_next, int64_t lddcn,
                                 const uint16_t* act, int64_t ldact, const uint16_t* c, int64_t ldc, const uint16_t* c_prev, int64_t ldcp,
                                 uint16_t* da, int64_t ldda, uint16_t* dc_prev, int64_t lddcp) {
  if (dh == nullptr || act == nullptr || c == nullptr || c_prev == nullptr || da == nullptr || dc_prev == nullptr) return MPT_ERR_NULL;
  if (!dims_ok(B, H) || lddh < H || (dc_next && lddcn < H) || ldact < 4 * H || ldc < H || ldcp < H || ldda < 4 * H || lddcp < H) return MPT_ERR_SHAPE;
  if (!mpt_aligned(dh, 2) || !mpt_aligned(dc_next, 2) || !mpt_aligned(act, 2) || !mpt_aligned(c, 2) || !mpt_aligned(c_prev, 2) || !mpt_aligned(da, 2) ||
      !mpt_aligned(dc_prev, 2))
    return MPT_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool singly = one_per_thread(B, H);
  const int64_t units = singly ? B * H : B * (H / 4 + (H & 3));
  const unsigned grid = (unsigned)((units + kT - 1) / kT);
  const bool stream_it = B * H * 22 > (192LL << 20);
  if (singly) hipLaunchKernelGGL((k_lstm_cell_bwd<1, false>), dim3(grid), dim3(kT), 0, st, B, H, dh, lddh, dc_next, lddcn, act, ldact, c, ldc, c_prev, ldcp, da, ldda, dc_prev, lddcp);
  else if (stream_it) hipLaunchKernelGGL((k_lstm_cell_bwd<4, true>), dim3(grid), dim3(kT), 0, st, B, H, dh, lddh, dc_next, lddcn, act, ldact, c, ldc, c_prev, ldcp, da, ldda, dc_prev, lddcp);
  else hipLaunchKernelGGL((k_lstm_cell_bwd<4, false>), dim3(grid), dim3(kT), 0, st, B, H, dh, lddh, dc_next, lddcn, act, ldact, c, ldc, c_prev, ldcp, da, ldda, dc_prev, lddcp);
  MPT_LAUNCH_CHECK();
  return MPT_OK;
}
