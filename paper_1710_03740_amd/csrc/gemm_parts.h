// What the matrix-product translation units share: exact division, the description of a problem and of its store, the
// walk over output tiles, the LDS reads that are waited for by hand, and the launchers of gemm_ring.hip.
#pragma once
#include "mpt_internal.h"
#include "gemm_plan.h"

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

namespace mpt_gemm {

// ---------------------------------------------------------------- exact 32-bit division by an invariant
struct FastDiv {
  uint32_t d, m, s;               // q = (umulhi(m, n) + n') >> s  (round-up method)
  __host__ __device__ FastDiv() : d(1), m(0), s(0) {}
  explicit FastDiv(uint32_t div) : d(div) {
    if (div <= 1) { m = 0; s = 0; d = 1; return; }
    uint32_t l = 0;
    while ((1ull << l) < div) ++l;                                 // l = ceil(log2 d), 1..32
    m = (uint32_t)(((1ull << 32) * ((1ull << l) - div)) / div + 1);
    s = l - 1;
  }
  __device__ __forceinline__ uint32_t div(uint32_t n) const {
    if (d == 1) return n;
    const uint32_t t = __umulhi(m, n);
    return (t + ((n - t) >> 1)) >> s;
  }
  __device__ __forceinline__ void divmod(uint32_t n, uint32_t& q, uint32_t& r) const {
    q = div(n);
    r = n - q * d;
  }
};

// ---------------------------------------------------------------- epilogue description
struct Epilogue {
  void* out;            // uint16_t* (FP16) or float* (FP32 / split partials)
  int64_t ld;
  int mode;             // 0: FP16 store, 1: FP32 store, 2: FP32 accumulate, 3: FP32 partial [split][I][J]
  uint32_t* flag;       // nullable; OR 1 when an FP16/FP32 stored value is Inf/NaN (modes 0..2)
  int act;              // FP16 store only.  0: none; 1: ReLU, store 0 unless the value is > 0;
                        // 2: store 0 unless mask[i][j] > 0 (the ReLU of the layer below, backward)
  const uint16_t* mask; // act == 2: FP16 matrix of the output's shape
  int64_t ldmask;
};

// FP16 bit pattern of a value > 0 (Inf included, NaN not).
__device__ __forceinline__ bool half_bits_positive(uint32_t b) { return (uint16_t)((b & 0xFFFFu) - 1u) < 0x7C00u; }
// Pointwise stage of an FP16 store: 4 consecutive outputs (packed in hb); mk = their mask values when act == 2.
__device__ __forceinline__ uint2v apply_act4(uint2v hb, const Epilogue& ep, uint2v mk) {
  if (ep.act == 0) return hb;
  uint32_t keep = 0;
  const uint2v src = ep.act == 1 ? hb : mk;
#pragma unroll
  for (int e = 0; e < 4; ++e) keep |= (uint32_t)half_bits_positive(src[e >> 1] >> ((e & 1) * 16)) << e;
  hb[0] &= ((keep & 1u) ? 0x0000FFFFu : 0u) | ((keep & 2u) ? 0xFFFF0000u : 0u);
  hb[1] &= ((keep & 4u) ? 0x0000FFFFu : 0u) | ((keep & 8u) ? 0xFFFF0000u : 0u);
  return hb;
}

struct Problem {
  int I, J, R;          // output rows, output cols, reduction length
  int tiles_i, tiles_j, splits, ktiles_per_split;   // ktiles_per_split: reduction tiles of 64 per split
};

// Workgroup id -> (tile_i, tile_j, split).  Consecutive ids land on different XCDs
// (8 of them, round-robin), so ids are first regrouped per XCD and then walked in
// panels of 4 tile-rows so that one XCD's L2 sees a compact block of tiles.
__device__ __forceinline__ void tile_of(const Problem& pb, int wg, int& ti, int& tj, int& sp) {
  const int per_split = pb.tiles_i * pb.tiles_j;
  const int total = per_split * pb.splits;
  const int xcd = wg & 7, local = wg >> 3;
  const int n_per = total >> 3, rem = total & 7;
  int id = xcd * n_per + min(xcd, rem) + local;
  sp = id / per_split;
  id -= sp * per_split;
  constexpr int GM = 4;
  const int panel = id / (GM * pb.tiles_j);
  const int first_i = panel * GM;
  const int rows = min(GM, pb.tiles_i - first_i);
  const int in_panel = id - panel * GM * pb.tiles_j;
  ti = first_i + in_panel % rows;
  tj = in_panel / rows;
}

__device__ __forceinline__ bool half_bits_special(uint32_t b) { return (b & 0x7C00u) == 0x7C00u; }

// ---------------------------------------------------------------- LDS-direct loads and LDS reads waited for by hand
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(1))) void* global_void_ptr;

// XOR key of reduction row r for the 32-byte units of an outer-contiguous stage row (256 or 512 bytes per row; see gemm.hip).
__device__ __forceinline__ int oc_key(int r) { return (r & 3) | ((r >> 1) & 4); }

// LDS reads are issued through inline assembly so that their completion is tracked here, by explicit
// s_waitcnt on the in-order LGKM counter, and not by the compiler, which would otherwise put a full vmcnt(0)
// wait in front of every read that follows an LDS-direct load.
__device__ __forceinline__ uint32_t lds_offset(const char* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}
template <int IMM>
__device__ __forceinline__ uint4v lds_read_b128_imm(uint32_t addr) {
  static_assert(IMM >= 0 && IMM < 65536, "LDS immediate offset");
  uint4v v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM) : "memory");
  return v;
}
template <int IMM>
__device__ __forceinline__ uint2v lds_read_tr_b64_imm(uint32_t addr) {
  static_assert(IMM >= 0 && IMM < 65536, "LDS immediate offset");
  uint2v v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM) : "memory");
  return v;
}

// The compiler takes an inline-assembly LDS read to be complete when the statement ends.  A fragment that nothing
// consumes afterwards (the prefetch past the last stage) would leave its registers free for reuse, for instance as the
// address of the next LDS-direct load, while the data is still on its way and lands on top of the new value.  Passing
// such fragments through this statement after the final wait keeps their registers reserved until then.
__device__ __forceinline__ void keep_until_here(const half8& f) { asm volatile("" ::"v"(f)); }

// ---------------------------------------------------------------- launchers of gemm_ring.hip
// One matrix operand: element (o, r) at base[o*ld + r] (reduction-contiguous) or base[r*ld + o] (outer-contiguous).
struct RingMatSrc { const uint16_t* base; int64_t ld; int O, R; };
// C[i,j] = sum_r A(i,r) * B(r,j) over plain matrices; `whole_chunks`: both operands can be fetched in 16-byte aligned
// pieces (base and row stride 16-byte aligned, contiguous extent a multiple of 8).  ktiles_per_split > 0 and
// splits = ceil(ceil(R / 64) / ktiles_per_split); the caller reduces the partials of more than one split.  cut > 0:
// sums in pieces of so many tiles of 64, added in order.
int launch_ring_plain(hipStream_t s, bool a_rc, bool b_rc, const RingMatSrc& A, const RingMatSrc& B, bool whole_chunks, RingTile tile,
                      int ktiles_per_split, int cut, int I, int J, int R, const Epilogue& ep);
// The same in 32 x 32 tiles whose `pieces` pieces of `piece` tiles of 64 are summed side by side (pieces_side_by_side); no partials (mode 3).
int launch_pieces_plain(hipStream_t s, bool a_rc, bool b_rc, const RingMatSrc& A, const RingMatSrc& B, bool whole_chunks, int piece, int pieces, int I, int J, int R,
                        const Epilogue& ep);
// The three passes of the 3x3 convolution (op: MPT_OP_*): x[Nb,H,W,C], w[Kf,3,3,C], y / dy[Nb,H,W,Kf]; `cut` as above.
int launch_ring_conv(hipStream_t s, int op, int64_t Nb, int64_t H, int64_t W, int64_t C, int64_t Kf, const uint16_t* img, const uint16_t* other,
                     RingTile tile, int ktiles_per_split, int cut, const Epilogue& ep);

}  // namespace mpt_gemm
