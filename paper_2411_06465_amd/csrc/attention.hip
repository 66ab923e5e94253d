// Causal grouped-query attention on the gfx950 matrix cores, FlashAttention
// style: the forward keeps only the output and the per-row log-sum-exp, the
// backward recomputes the probabilities from Q, K and the log-sum-exp
// (the activation accounting of Sec. 3.2 counts QK^T and softmax as zero).
//
// Keys come as up to kMaxSeg runs with consecutive global positions: the
// rank's own context-parallel chunks and the remote chunks of the other CP
// ranks.  A key is visible to a query iff key position <= query position.
//
// gfx950 design:
//  * every K/V/Q/dO tile is copied global -> LDS with global_load_lds_dwordx4
//    (no staging registers) into a row-major tile with an XOR swizzle of its
//    16-byte chunks; two buffers alternate (forward, dQ), or a ring of four turns
//    (dK/dV), so that the next tiles stream in while the current one is used;
//  * operands that need the token index contiguous (V in P V, Q and dO in the
//    dK/dV products, K in dQ) are read transposed straight from those tiles
//    with ds_read_b64_tr_b16 (16 lanes x 4 rows -> 4 rows per lane);
//  * scores are computed transposed where that puts one query per lane
//    (forward, dQ), so the softmax statistics are per-lane scalars; the bf16
//    probabilities then feed the next MFMA from registers with the
//    contraction index permuted consistently on both operands;
//  * masks are applied only on tiles that straddle the diagonal;
//  * forward and dQ: 256 threads and at most 64 KB of LDS, two workgroups per
//    CU; dK/dV: 512 threads and 97 KB, one workgroup per CU, two waves per SIMD.
//  * dK/dV are accumulated over the query heads of a kv-head inside one
//    workgroup, or, when that leaves too few workgroups, over a slice of them
//    with an fp32 partial per slice that a small kernel sums: no atomics, the
//    result is deterministic.
#include <math.h>

#include <type_traits>

#include <algorithm>
#include <vector>

#include "kernels.h"

namespace l4d {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

#define LPTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int KT = 64;            // keys per tile (forward; dQ takes 32)
constexpr int QT = 32;            // queries per tile (dK/dV)
constexpr int kDkvStages = 4;     // dK/dV: query tiles in the copy ring (even: the handover buffer is the stage's parity)
// LDS fragment reads kept in flight ahead of the products, per kernel
constexpr int kLookFwd = 6, kLookDq = 4;

__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// Two floats to a packed bf16 pair with one conversion (round to nearest even).
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float lo16(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi16(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// Wait until at most N of this wave's copies are still in flight.
template <int N>
__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// Workgroup barrier that does not drain the copies still in flight (unlike
// __syncthreads): only this wave's LDS reads must be done before it.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Make the compiler wait for a value loaded from global memory here, before
// the tile loop: otherwise it places the wait at the value's first use inside
// the loop, on every iteration, where the hardware counter also holds the
// next tile's copies (issued as inline assembly) -- and the wait drains them.
template <class T>
__device__ __forceinline__ void settle(const T& v) {
  asm volatile("" ::"v"(v));
}

// ------------------------------------------------------------------ LDS tiles
// Row-major [rows][D] bf16 tile; 16-byte chunk c of row r sits at chunk c ^ swz(r).
// The LDS serves 256 bytes (64 banks) per cycle.  Two read patterns must be
// conflict-free: a row fragment (16 lanes, 16 consecutive rows, one chunk
// each) needs swz to be a permutation over every aligned block of 16 rows; a
// transposing column fragment (32 lanes, 4 consecutive rows x an aligned group
// of 4 chunks) needs the 4 rows to map that group to 4 different groups, i.e.
// distinct swz >> 2 across 4 consecutive rows.  At D = 64 a row is half a
// bank line, so row parity picks the half and swz only has to separate rows
// of equal parity.  Also swz(r + 8) = swz(r) ^ 4: a column fragment reads
// rows r and r + 8, and the second address is then the first address of the
// neighbouring 32-column block plus a constant, so no extra register holds it.
template <int D>
__device__ __forceinline__ int swz(int row) {
  const int b1 = (row >> 1) & 1, b2 = (row >> 2) & 1, b3 = (row >> 3) & 1;
  return D == 128 ? ((((row & 3) ^ b3) << 2) | (b2 << 1) | (row & 1)) : (((b1 ^ b3) << 2) | (b2 << 1) | b1);
}

// Direct-to-LDS copy of `size` bytes per lane from sbase + voff (uniform base,
// per-lane byte offset) into the wave's LDS chunk at lds (lane i lands at
// lds + size * i).  Inline assembly: the compiler's wait-count pass does not
// see the LDS write in flight, so it does not drain the prefetch before the
// reads of the other buffer (it cannot tell the buffers apart).  The kernels
// wait for their own copies (vmcnt) before the barrier that publishes a tile.
// The LDS address is uniform by construction; readfirstlane states it for the
// compiler, which otherwise may keep it in a vector register.
// The s_nop is the wait state that gfx9 needs between a scalar write of m0 and a
// copy into LDS that reads it; the compiler adds none inside an assembly block.
__device__ __forceinline__ uint32_t lds_addr(const void* lds) {
  return __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(LPTR(const_cast<void*>(lds)))));
}
template <int IMM>
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds) {   // LDS chunk at lds + IMM
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds), "n"(IMM)
               : "memory", "m0", "scc");
}
__device__ __forceinline__ void dma4(const void* sbase, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(voff), "s"(sbase), "s"(lds) : "memory", "m0");
}

// Copy rows [0, ROWS) of src (row stride ld, rows >= n_valid clamped to the
// last valid row) into an LDS tile; the NW waves of the block share the work.
// A copy instruction moves RPK whole rows (1 KB); lane i lands at byte 16 i of
// the instruction's LDS chunk.  The wave's copies start at rows that agree
// modulo 4 * RPK (the waves take every NW-th chunk, NW a multiple of 4), which
// fixes swz, so each lane's swizzled source column is fixed: its byte offsets are
// formed once, and a copy is two instructions on a uniform base, except on a
// ragged tail.
template <int D, int ROWS, int NW = 4>
struct TileCopy {
  static constexpr int CH = D / 8;              // 16-byte chunks per row
  static constexpr int RPK = 64 / CH;           // rows per 1 KB wave chunk
  static constexpr int NKB = ROWS / RPK;
  static_assert(NKB % NW == 0, "every wave issues the same number of copies");
  int row0, lc, ldb;            // the lane's row in the first copy, its chunk, the row stride in bytes
  uint32_t off[NKB / NW];       // byte offset of the lane's 16 bytes of each copy
  uint32_t lds0;                // the wave's chunk within a tile
  __device__ __forceinline__ TileCopy(int64_t ld, int wave, int lane) {
    row0 = wave * RPK + lane / CH;
    lc = (lane % CH) ^ swz<D>(row0);            // the same for every copy of this wave
    ldb = static_cast<int>(ld) * 2;
#pragma unroll
    for (int j = 0; j < NKB / NW; ++j) off[j] = static_cast<uint32_t>((row0 + j * NW * RPK) * ldb + lc * 16);
    lds0 = wave * 1024;
  }
  __device__ __forceinline__ void operator()(uint32_t lds, const uint16_t* src, int n_valid) const {
    if (n_valid >= ROWS) {
      each<0>(lds + lds0, src, off);
    } else {                               // ragged tail: rows past n_valid repeat the last valid row
      uint32_t o[NKB / NW];
#pragma unroll
      for (int j = 0; j < NKB / NW; ++j)
        o[j] = static_cast<uint32_t>(min(row0 + j * NW * RPK, n_valid - 1) * ldb + lc * 16);
      each<0>(lds + lds0, src, o);
    }
  }
  template <int J>
  __device__ __forceinline__ void each(uint32_t lds, const uint16_t* src, const uint32_t (&o)[NKB / NW]) const {
    if constexpr (J < NKB / NW) {
      dma16<J * NW * 1024>(src, o[J], lds);
      each<J + 1>(lds, src, o);
    }
  }
};

// Per-lane LDS byte offsets of the two fragment shapes below, at kk = 0 and
// dt = 0 of a tile's first row block.  With swz periodic in 16 rows, the
// other kk / dt are an XOR of the low byte (the 16-byte chunk within a row),
// and other row blocks a constant: one register per shape.
struct LaneAddr {
  int rows;   // row fragment: row lane%32, chunk lane/32
  int cols;   // column fragment: row 4 (lane/32) + (lane%16)/4, column 16 ((lane/16)%2) + 4 (lane%4)
};
template <int D>
__device__ __forceinline__ LaneAddr lane_addr(int lane) {
  const int h = lane >> 5, li = lane & 15;
  const int rr = lane & 31;
  const int cr = 4 * h + (li >> 2);
  const int low = 2 * ((lane >> 4) & 1) + ((li & 3) >> 1);   // chunk within the 4-chunk group
  return LaneAddr{rr * (D * 2) + ((swz<D>(rr) ^ h) << 4),
                  cr * (D * 2) + ((low ^ swz<D>(cr)) << 4) + ((li & 1) << 3)};
}
// MFMA operand with the tile's rows as its 32 rows: rows row0 + lane%32 (row0
// a multiple of 16), contraction chunk 2*kk + lane/32 (d = 16 kk + 8 (lane/32) + 0..7).
template <int D>
__device__ __forceinline__ bf16x8 frag_rows(const uint8_t* lds, int row0, int kk, LaneAddr la) {
  return *reinterpret_cast<const bf16x8*>(lds + row0 * (D * 2) + (la.rows ^ (kk << 5)));
}
// MFMA operand with the tile's columns as its rows: d = 32 dt + lane%32; its 8
// contraction slots are tile rows 16 g16 + {4h .. 4h+3, 8+4h .. 8+4h+3},
// h = lane/32 -- the same order in which a lane holds accumulator rows of a
// 32x32 MFMA (see frag_acc).  Two transposing 64-bit LDS reads; rows r + 8
// have swz(r) ^ 4, which is the XOR pattern of column block dt ^ 1.
template <int D>
__device__ __forceinline__ bf16x8 frag_cols(const uint8_t* lds, int dt, int g16, LaneAddr la) {
  const uint8_t* base = lds + g16 * 16 * (D * 2);
  const i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) i16x4*>(
      LPTR(const_cast<uint8_t*>(base) + (la.cols ^ (dt << 6)))));
  const i16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) i16x4*>(
      LPTR(const_cast<uint8_t*>(base) + 8 * (D * 2) + (la.cols ^ ((dt ^ 1) << 6)))));
  return __builtin_bit_cast(bf16x8, u32x4{__builtin_bit_cast(u32x2, a)[0], __builtin_bit_cast(u32x2, a)[1],
                                          __builtin_bit_cast(u32x2, b)[0], __builtin_bit_cast(u32x2, b)[1]});
}
// Operand from 8 accumulator registers i0..i0+7 (rows 16 (i0/8) + {4h..4h+3, 8+4h..}).
__device__ __forceinline__ bf16x8 frag_acc(const f32x16& s, int i0) {
  return __builtin_bit_cast(bf16x8, u32x4{pack2(s[i0], s[i0 + 1]), pack2(s[i0 + 2], s[i0 + 3]),
                                          pack2(s[i0 + 4], s[i0 + 5]), pack2(s[i0 + 6], s[i0 + 7])});
}
// The rounding residual of frag_acc: bf16(s - hi) for the same 8 registers,
// given hi = frag_acc(s, i0).  hi + lo carries about 16 significant bits.
__device__ __forceinline__ bf16x8 frag_acc_lo(const f32x16& s, int i0, bf16x8 hi) {
  const u32x4 h = __builtin_bit_cast(u32x4, hi);
  u32x4 r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = pack2(s[i0 + 2 * k] - lo16(h[k]), s[i0 + 2 * k + 1] - hi16(h[k]));
  return __builtin_bit_cast(bf16x8, r);
}
// Row of accumulator register i for this lane (32x32 MFMA output layout).
__device__ __forceinline__ int acc_row(int i, int lane) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

// Global position of local query row `row` (at most two chunks).  A select
// between the two scalar chunk ids, not an indexed load: a per-lane index into
// the kernel arguments would become a vector load whose wait drains every copy
// in flight.
__device__ __forceinline__ int qpos(const ChunkMap& m, int row) {
  const bool second = row >= m.chunk_len;
  return (second ? m.chunk_id[1] : m.chunk_id[0]) * m.chunk_len + (second ? row - m.chunk_len : row);
}

// Key tile `tile` (of `tsz` tokens) across the segments.
__device__ __forceinline__ bool find_tile(const AttnParams& p, int tile, int tsz, int& seg, int& t0) {
  int acc = 0;
  for (int s = 0; s < p.n_seg; ++s) {
    const int nt = (p.seg[s].n + tsz - 1) / tsz;
    if (tile < acc + nt) {
      seg = s;
      t0 = (tile - acc) * tsz;
      return true;
    }
    acc += nt;
  }
  return false;
}

// ------------------------------------------------------------------ forward
// One workgroup per (128-query tile, query head, batch element); 4 waves x 32
// queries, each lane holding one query's scores (S^T = K Q^T).  The launch is
// one-dimensional with the head index varying fastest and the query tiles in
// descending order, so the longest causal rows are dispatched first across all
// heads.  Registers stay within 256 per lane and LDS within 64 KB, so two
// workgroups share a CU and each SIMD interleaves the matrix products of one
// wave with the softmax of another.
//
// The output and the row sum are rescaled only on tiles where some row's
// maximum grew (a wave-wide vote).  The reference is the exact maximum: the
// largest probability is then exactly 1, and the row sum, whose logarithm goes
// into the log-sum-exp, at least 1.  A reference that may lag by 2^8 rescales
// less (7B forward 196 us, exact 204) but made the stored log-sum-exp 10% worse
// (rms error 3.1e-7 -> 3.4e-7 at 1000 keys, 3.7e-7 -> 4.2e-7 at 4096 with larger
// scores), since exponents of up to 8 carry their own rounding.

// The key tiles of `step` keys that a query at pos_max can see, over the
// segments in order: the first tile of a segment whose first key is visible and
// the ones after it.  Positions grow within a segment, so the rest of a segment
// is skipped once a tile starts past pos_max.  A segment's fields are loaded
// when the walk enters it: loading them for every tile put several scalar loads,
// each waited for, in front of every tile's products.
struct Tile {
  int kpos0, kvalid;           // position of its first key; keys, 0 = no tile
};
struct KeyWalk {
  const AttnParams& p;
  const int pos_max, step, bi;
  const int64_t col, stride;   // the kv head's column; bytes per step (every segment has the same row stride)
  int seg = -1, left = 0;      // segment; its keys from the next tile on (0 = none, or none visible)
  int pos = 0;                 // position of the next tile's first key
  uint64_t ka = 0, va = 0;     // addresses of the first rows of the tile last returned, at the kv head's column
  __device__ __forceinline__ KeyWalk(const AttnParams& p_, int pos_max_, int step_, int bi_, int64_t col_)
      : p(p_), pos_max(pos_max_), step(step_), bi(bi_), col(col_), stride(step_ * p_.seg[0].ld * 2) {}
  __device__ __forceinline__ const uint16_t* k() const { return reinterpret_cast<const uint16_t*>(ka); }
  __device__ __forceinline__ const uint16_t* v() const { return reinterpret_cast<const uint16_t*>(va); }
  __device__ __forceinline__ Tile next() {
    ka += stride;
    va += stride;
    while (left <= 0 || pos > pos_max) {
      if (++seg >= p.n_seg) {
        left = 0;              // stays at the end
        seg = p.n_seg;
        return Tile{0, 0};
      }
      const KvSeg& s = p.seg[seg];
      left = s.n;
      pos = s.pos0;
      ka = reinterpret_cast<uint64_t>(s.k + bi * s.bstride + col);
      va = reinterpret_cast<uint64_t>(s.v + bi * s.bstride + col);
    }
    const Tile t{pos, min(step, left)};
    pos += step;
    left -= step;
    return t;
  }
};

// ------------------------------------------------------------------ pipelined products
// Two accumulator chains over the D columns of LDS tiles, with the B operands
// in registers:  s0 += A0[r0 + (0..31)] x0^T,  s1 += A1[r1 + (0..31)] x1^T.
// The schedule keeps LA fragment reads in flight ahead of the products
// (without it the compiler reads each fragment right before its product and
// the LDS latency is exposed on every step).
template <int D, int LA>
__device__ __forceinline__ void scores2(const uint8_t* a0, int r0, const bf16x8 (&x0)[D / 16], f32x16& s0,
                                        const uint8_t* a1, int r1, const bf16x8 (&x1)[D / 16], f32x16& s1,
                                        LaneAddr la) {
  constexpr int N = D / 8;               // products (and fragment reads)
  constexpr int L = LA < N ? LA : N - 1;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    s0 = mfma(frag_rows<D>(a0, r0, kk, la), x0[kk], s0);
    s1 = mfma(frag_rows<D>(a1, r1, kk, la), x1[kk], s1);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, L, 0);      // LDS reads
#pragma unroll
  for (int i = 0; i < N - L; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, L, 0);
}

// acc[dt] += A^T x over NG groups of 16 rows: A the LDS tile read transposed
// (d rows, row-index contraction), x[g] a bf16 operand from registers (P^T,
// dS^T); two reads per fragment, LA fragments in flight.
template <int D, int NG, int LA>
__device__ __forceinline__ void accum_t(const uint8_t* lds, const bf16x8 (&x)[NG], f32x16 (&acc)[D / 32], LaneAddr la) {
  constexpr int N = NG * D / 32;
  constexpr int L = LA < N ? LA : N - 1;
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) acc[dt] = mfma(frag_cols<D>(lds, dt, g, la), x[g], acc[dt]);
  __builtin_amdgcn_sched_group_barrier(0x100, 2 * L, 0);
#pragma unroll
  for (int i = 0; i < N - L; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, L, 0);
}

// max(x, x of the other half-wave), in every lane
__device__ __forceinline__ float half_max(float x) {
  const u32x2 r = __builtin_bit_cast(
      u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) attn_fwd_kernel(AttnParams p) {
  constexpr int TB = KT * D * 2;
  __shared__ __attribute__((aligned(16))) uint8_t k0[TB], v0[TB], k1[TB], v1[TB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_qt = (p.n_q + 127) / 128;
  const int nh = p.a_t * p.b;
  const int qt = n_qt - 1 - static_cast<int>(blockIdx.x) / nh;   // heaviest tiles first
  const int hq = static_cast<int>(blockIdx.x) % nh % p.a_t, bi = static_cast<int>(blockIdx.x) % nh / p.a_t;
  const int hk = hq / (p.a_t / p.k_t);
  const int q_row0 = qt * 128;
  const int my_q = q_row0 + wave * 32 + (lane & 31);
  const bool q_ok = my_q < p.n_q;
  const int my_pos = q_ok ? qpos(p.qmap, my_q) : -1;
  const int blk_last = min(q_row0 + 127, p.n_q - 1);
  const int pos_min = qpos(p.qmap, q_row0), pos_max = qpos(p.qmap, blk_last);
  const int rbase = 4 * (lane >> 5);
  const LaneAddr la = lane_addr<D>(lane);

  bf16x8 qf[D / 16];
  {
    const uint16_t* qb = p.q + bi * p.q_bstride + static_cast<int64_t>(q_ok ? my_q : 0) * p.q_ld + hq * D;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qb + (2 * kk + (lane >> 5)) * 8);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) settle(qf[kk]);
  }
  const float c = p.scale * kLog2e;
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 o[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; ++i) o[i] = f32x16{};

  KeyWalk walk(p, pos_max, KT, bi, hk * D);
  const TileCopy<D, KT> copy(p.seg[0].ld, wave, lane);
  const uint32_t ka0 = lds_addr(k0), ka1 = lds_addr(k1), va0 = lds_addr(v0), va1 = lds_addr(v1);
  // maximum of a lane's 32 scores: a chain of three-input maxima
  const auto row_max = [](const f32x16 (&s)[2]) __attribute__((always_inline)) {
    float m = __builtin_fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) m = __builtin_fmaxf(__builtin_fmaxf(m, s[0][i]), s[0][i + 1]);
#pragma unroll
    for (int i = 0; i < 16; i += 2) m = __builtin_fmaxf(__builtin_fmaxf(m, s[1][i]), s[1][i + 1]);
    return m;
  };
  // One key tile, its scores already in s (their maximum in mx): the softmax and
  // O += V^T P, with the next tile's scores S^T = K Q^T (into sn, mxn) computed
  // under the exponentials.  After the last tile sn comes from stale LDS and is
  // never used.
  const auto step = [&](Tile t, const uint8_t* vt, const uint8_t* kt_next, f32x16 (&s)[2], float mx, f32x16 (&sn)[2],
                        float& mxn) __attribute__((always_inline)) {
    if (t.kpos0 + KT - 1 > pos_min || t.kvalid < KT) {     // tile straddles the diagonal (or is ragged)
      // last visible key row for this query, relative to the lane's first row
      const int lim = min(my_pos - t.kpos0, t.kvalid - 1) - rbase;
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (t2 * 32 + 8 * (i >> 2) + (i & 3) > lim) s[t2][i] = -INFINITY;
      mx = row_max(s);
    }
    mx = half_max(mx) * c;
    if (__builtin_amdgcn_ballot_w64(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(m_run - m_new);   // 0 while m_run is -inf
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) o[dt] *= alpha;
      l_run *= alpha;
      m_run = m_new;
    }
    const float m_use = m_run == -INFINITY ? 0.f : m_run;
    sn[0] = f32x16{};
    sn[1] = f32x16{};
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      sn[0] = mfma(frag_rows<D>(kt_next, 0, kk, la), qf[kk], sn[0]);
      sn[1] = mfma(frag_rows<D>(kt_next, 32, kk, la), qf[kk], sn[1]);
    }
    float rs[2] = {0.f, 0.f};
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float pr = fast_exp2(fmaf(s[t2][i], c, -m_use));
        s[t2][i] = pr;
        rs[i & 1] += pr;
      }
    l_run += rs[0] + rs[1];
    // P enters the P V product as bf16 hi + lo parts (two products per V
    // fragment): a plain bf16 P carries a relative error of up to 2^-9 into
    // every output, which the bf16 stores after attention then amplify.  The
    // high products of a group's column blocks go before their low products,
    // so no product waits on the one just before it; the next group's split and
    // V fragments go between them.
    bf16x8 ph[2], pl[2], f[2][D / 32];
    const auto group = [&](int g) __attribute__((always_inline)) {
      ph[g & 1] = frag_acc(s[g >> 1], 8 * (g & 1));
      pl[g & 1] = frag_acc_lo(s[g >> 1], 8 * (g & 1), ph[g & 1]);
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) f[g & 1][dt] = frag_cols<D>(vt, dt, g, la);
    };
    group(0);
    // the score products: an LDS read (kLookFwd ahead), exponentials and their sums between every two
    constexpr int NS = D / 8, NV = 2 * (D / 32);
    __builtin_amdgcn_sched_group_barrier(0x100, kLookFwd, 0);
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);            // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);            // LDS read
      __builtin_amdgcn_sched_group_barrier(0x400, 32 / NS, 0);      // exponentials
      __builtin_amdgcn_sched_group_barrier(0x002, 96 / NS, 0);      // other VALU
    }
    __builtin_amdgcn_sched_group_barrier(0x100, NV, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (g < 3) group(g + 1);
      else mxn = row_max(sn);
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) o[dt] = mfma(f[g & 1][dt], ph[g & 1], o[dt]);
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) o[dt] = mfma(f[g & 1][dt], pl[g & 1], o[dt]);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 24 / NV, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Two buffers each for K and V.  While tile j is in step, V_j and K_(j+1) are
  // in use, V_(j+1) and K_(j+2) land in the buffers that V_(j-1) and K_j held.
  Tile t = walk.next();
  if (t.kvalid) {
    copy(ka0, walk.k(), t.kvalid);
    copy(va0, walk.v(), t.kvalid);
    Tile t1 = walk.next();
    const uint16_t* v_next = walk.v();       // V of tile t1
    if (t1.kvalid) copy(ka1, walk.k(), t1.kvalid);
    wait_copies<0>();
    ring_barrier();
    f32x16 sa[2] = {f32x16{}, f32x16{}}, sb[2];
    scores2<D, kLookFwd>(k0, 0, qf, sa[0], k0, 32, qf, sa[1], la);
    float ma = row_max(sa), mb = -INFINITY;
    const auto turn = [&](const uint8_t* vt, uint32_t va_next, uint32_t ka, const uint8_t* kt_next, f32x16 (&s)[2],
                          float mx, f32x16 (&sn)[2], float& mxn) __attribute__((always_inline)) {
      const Tile t2 = walk.next();
      wait_copies<0>();
      ring_barrier();                      // every wave's copies are visible and the two old buffers are free
      if (t1.kvalid) copy(va_next, v_next, t1.kvalid);
      if (t2.kvalid) copy(ka, walk.k(), t2.kvalid);
      __builtin_amdgcn_sched_barrier(0);   // the copies go out now, not next to the wait for them
      step(t, vt, kt_next, s, mx, sn, mxn);
      t = t1;
      t1 = t2;
      v_next = walk.v();
    };
    while (true) {
      turn(v0, va1, ka0, k1, sa, ma, sb, mb);
      if (!t.kvalid) break;
      turn(v1, va0, ka1, k0, sb, mb, sa, ma);
      if (!t.kvalid) break;
    }
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (!q_ok) return;
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  uint16_t* ob = p.o + bi * p.q_bstride + static_cast<int64_t>(my_q) * p.q_ld + hq * D;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int d = dt * 32 + 8 * jj + rbase;
      *reinterpret_cast<u32x2*>(ob + d) = u32x2{pack2(o[dt][4 * jj] * inv, o[dt][4 * jj + 1] * inv),
                                                pack2(o[dt][4 * jj + 2] * inv, o[dt][4 * jj + 3] * inv)};
    }
  if (lane < 32) {
    const float m_fin = m_run == -INFINITY ? 0.f : m_run;
    p.lse[(static_cast<int64_t>(bi) * p.a_t + hq) * p.n_q + my_q] = (m_fin + __builtin_amdgcn_logf(l_tot)) * kLn2;
  }
}


// ------------------------------------------------------------------ backward: dK, dV
// Flat grid over (key block of 128 over all segments, kv head, split, b), key
// block slowest: the earliest key blocks see the most query tiles, so they are
// dispatched first (longest job first keeps the last CUs from running one long
// block alone), and with the heads varying fastest every block of a head lands
// on the same XCD (dispatch deals block ids round-robin over the 8 XCDs),
// where its query-tile stream is shared in L2.  8 waves.
// Workgroup (kb, hk, split) sums over query heads hk*g + [split*hpb, (split+1)*hpb).
//
// The block's 128 keys form four groups of 32, and each group has two waves
// with different jobs, on the same SIMD (wave w runs on SIMD w % 4):
//  * role 0 (waves 0-3) holds K, computes S^T = K Q^T, P^T = exp(S^T - lse),
//    hands P^T (fp32) to its partner through LDS and accumulates dV^T += dO^T P^T;
//  * role 1 (waves 4-7) holds V, computes dP^T = V dO^T, takes P^T and forms
//    dS^T = P^T (dP^T - delta), and accumulates dK^T += Q^T dS^T.
// Each wave then needs one operand block and one accumulator block, which fits
// 256 registers, and the two waves of a SIMD issue different instruction mixes
// (softmax on one, products on the other) that interleave.  dS^T is formed
// from the fp32 P^T and rounded to bf16 once, as in the dQ kernel.
template <int D>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) attn_bwd_dkdv_kernel(AttnParams p) {
  constexpr int TB = QT * D * 2;
  // Four stages of Q and dO tiles (64 KB at D = 128: every tile offset fits a
  // ds_read immediate), their statistics, and two P^T handovers.
  __shared__ __attribute__((aligned(16))) uint8_t qg[kDkvStages][2][TB];   // per stage: Q tile, then dO tile
  __shared__ __attribute__((aligned(16))) float st[kDkvStages][2][QT];    // lse, delta
  // P^T handover in fp32, so that dS^T = P^T (dP^T - delta) rounds once: [buffer][group][16 queries][half][lane]
  __shared__ __attribute__((aligned(16))) float4 xp[2][4][QT / 16][2][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave & 3, role = wave >> 2;
  const int group = p.a_t / p.k_t;
  const int hpb = group / p.n_split;
  const int nyz = p.k_t * p.n_split * p.b;
  const int kb_raw = static_cast<int>(blockIdx.x) / nyz, yz = static_cast<int>(blockIdx.x) % nyz;
  const int kb = p.n_order ? p.kb_order[kb_raw] : kb_raw;
  const int hk = yz % (p.k_t * p.n_split) / p.n_split, split = yz % p.n_split;
  const int bi = yz / (p.k_t * p.n_split);
  int seg, k0;
  if (!find_tile(p, kb, 128, seg, k0)) return;
  const KvSeg& S = p.seg[seg];
  const int my_key = k0 + grp * 32 + (lane & 31);
  const bool key_ok = my_key < S.n;
  const int my_kpos = S.pos0 + my_key;
  const int grp_kpos0 = S.pos0 + k0 + grp * 32;
  const int blk_kpos0 = S.pos0 + k0;
  const int rbase = 4 * (lane >> 5);
  const LaneAddr la = lane_addr<D>(lane);
  // Offsets into a stage's [Q | dO] pair: the first product reads Q (role 0)
  // or dO (role 1), the second reads dO (role 0) or Q (role 1).
  const LaneAddr la1{la.rows + role * TB, la.cols};
  const LaneAddr la2{la.rows, la.cols + (1 - role) * TB};

  bf16x8 kv[D / 16];                     // role 0: K rows, role 1: V rows of the group's keys
  {
    const uint16_t* src = role == 0 ? S.k : S.v;
    const int64_t off = bi * S.bstride + static_cast<int64_t>(key_ok ? my_key : 0) * S.ld + hk * D;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
      kv[kk] = *reinterpret_cast<const bf16x8*>(src + off + (2 * kk + (lane >> 5)) * 8);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) settle(kv[kk]);
  }
  f32x16 acc[D / 32];                    // role 0: dV^T, role 1: dK^T (d rows, the lane's key)
#pragma unroll
  for (int i = 0; i < D / 32; ++i) acc[i] = f32x16{};
  const float c = p.scale * kLog2e;
  const int n_qt = (p.n_q + QT - 1) / QT;
  const int head0 = hk * group + split * hpb;
  // The query tiles that see the block: local rows are in position order, so
  // those from qt0 on, of each of the hpb heads.
  int qt0 = 0;
  while (qt0 < n_qt && qpos(p.qmap, min(qt0 * QT + QT - 1, p.n_q - 1)) < blk_kpos0) ++qt0;
  const int per_head = n_qt - qt0;
  // waves 0-3 copy the Q tiles and their lse, waves 4-7 the dO tiles and delta
  const TileCopy<D, QT> copy(p.q_ld, grp, lane);
  const uint32_t qg_addr = lds_addr(qg) + role * TB, st_addr = lds_addr(st) + (role * QT + grp * (QT / 4)) * 4;
  // the next tile to copy: its first row, its head's statistics, its query tile, tiles left to copy after it
  // (the role's pointers by arithmetic: a select of the two members' addresses
  // would put the kernel argument on the stack)
  const auto pick = [&](const void* a, const void* b) {
    const uint64_t x = reinterpret_cast<uint64_t>(a), y = reinterpret_cast<uint64_t>(b);
    return x + ((y - x) & (0ull - static_cast<uint64_t>(role)));
  };
  uint64_t src = pick(p.q, p.dout) + (bi * p.q_bstride + static_cast<int64_t>(qt0) * QT * p.q_ld + head0 * D) * 2;
  uint64_t row = pick(p.lse, p.delta) + (static_cast<int64_t>(bi) * p.a_t + head0) * p.n_q * 4;
  const int64_t tile_step = static_cast<int64_t>(QT) * p.q_ld * 2, head_step = D * 2 - (per_head - 1) * tile_step;
  int copy_qt = qt0, copy_left = hpb * per_head - 1;
  // Copies that tile into stage b, kCopies per wave, and moves on; past the last
  // tile it repeats it, so that the waits count exactly.
  constexpr int kCopies = TileCopy<D, QT>::NKB / 4 + 1;
  auto issue = [&](int b) __attribute__((always_inline)) {
    const int q0 = copy_qt * QT;
    if (lane < QT / 4)
      dma4(reinterpret_cast<const float*>(row), static_cast<uint32_t>(min(q0 + grp * (QT / 4) + lane, p.n_q - 1)) * 4u,
           st_addr + b * (2 * QT * 4));
    copy(qg_addr + b * (2 * TB), reinterpret_cast<const uint16_t*>(src), p.n_q - q0);
    const bool more = copy_left > 0, wrap = copy_qt + 1 == n_qt;
    src += more ? (wrap ? head_step : tile_step) : 0;
    row += more && wrap ? static_cast<int64_t>(p.n_q) * 4 : 0;
    copy_qt = more ? (wrap ? qt0 : copy_qt + 1) : copy_qt;
    copy_left -= more;
  };
  f32x16 s;                  // role 0: S^T -> P^T of a tile, role 1: its dP^T
  bf16x8 x[2];               // role 0: P^T, role 1: dS^T (bf16)
  // role 0: P^T = exp(S^T - lse) of tile qt from its scores in s; bf16 into x, fp32 into handover hb
  auto probs = [&](int qt, const float4 (&ls4)[4], float4 (*hb)[2][64]) __attribute__((always_inline)) {
    const int qr0 = qt * QT;
    const int qlast = min(qr0 + QT - 1, p.n_q - 1);
    const int qp0 = qpos(p.qmap, qr0), qpl = qpos(p.qmap, qlast);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const float4 ls = ls4[jj];
      const float lsv[4] = {ls.x * kLog2e, ls.y * kLog2e, ls.z * kLog2e, ls.w * kLog2e};
#pragma unroll
      for (int u = 0; u < 4; ++u) s[4 * jj + u] = fast_exp2(fmaf(s[4 * jj + u], c, -lsv[u]));
    }
    // Every group works on every tile the block visits; on the few diagonal
    // tiles where all of a group's keys follow every query, the causal mask
    // zeroes its P^T.
    if (!(qp0 >= grp_kpos0 + 31 && qlast == qr0 + QT - 1 && qpl - qp0 == QT - 1)) {   // causal / ragged masks
      if (qpl - qp0 == qlast - qr0) {
        // visible query rows r (relative to the lane's first row): lo <= r <= hi
        const int lo = (key_ok ? my_kpos - qp0 : QT) - rbase;
        const int hi = qlast - qr0 - rbase;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int r = 8 * (i >> 2) + (i & 3);
          if (r < lo || r > hi) s[i] = 0.f;
        }
      } else {                                     // the tile spans two context-parallel chunks
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int qr = 8 * (i >> 2) + rbase + (i & 3);
          const int qp = qr0 + qr <= qlast ? qpos(p.qmap, qr0 + qr) : -1;
          if (my_kpos > qp || !key_ok) s[i] = 0.f;
        }
      }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int i0 = 8 * g;
      x[g] = frag_acc(s, i0);
      hb[g][0][lane] = make_float4(s[i0], s[i0 + 1], s[i0 + 2], s[i0 + 3]);
      hb[g][1][lane] = make_float4(s[i0 + 4], s[i0 + 5], s[i0 + 6], s[i0 + 7]);
    }
  };
  // role 1: dS^T = P^T (dP^T - delta) of the tile whose dP^T - delta is in s, into x
  auto grads = [&](const float4 (*hb)[2][64]) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const float4 p0 = hb[g][0][lane], p1 = hb[g][1][lane];
      const float pv[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
      float ds[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) ds[j] = pv[j] * s[8 * g + j];
      x[g] = __builtin_bit_cast(
          bf16x8, u32x4{pack2(ds[0], ds[1]), pack2(ds[2], ds[3]), pack2(ds[4], ds[5]), pack2(ds[6], ds[7])});
    }
  };
  auto minus = [&](const float4 (&d4)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      s[4 * jj] -= d4[jj].x;
      s[4 * jj + 1] -= d4[jj].y;
      s[4 * jj + 2] -= d4[jj].z;
      s[4 * jj + 3] -= d4[jj].w;
    }
  };
  // Both roles run one stream of products over role-selected tiles (role 0: S^T
  // from Q, dV^T from dO; role 1: dP^T from dO, dK^T from Q), so the accumulators
  // never meet at a branch join: the next tile's scores (stage bn) alternating
  // with this tile's accumulation (stage b) of x.
  auto products = [&](int b, int bn, bool accumulate) __attribute__((always_inline)) {
    s = f32x16{};
    const uint8_t* tb = qg[b][0];
    const uint8_t* tn = qg[bn][0];
    constexpr int NS = D / 16, NA = 2 * (D / 32);     // products of either kind (equal)
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      s = mfma(frag_rows<D>(tn, 0, i, la1), kv[i], s);
      if (accumulate) {
        const int g = i / (D / 32), dt = i % (D / 32);
        acc[dt] = mfma(frag_cols<D>(tb, dt, g, la2), x[g], acc[dt]);
      }
    }
    static_assert(NS == NA, "scores and accumulation alternate");
  };

  // One barrier per tile.  Interval j, after the barrier that publishes tile
  // j + 1 and the handover of P_j: role 1 forms dS_j; both roles run tile j's
  // accumulation and tile j + 1's scores; role 0 forms and hands over P_(j+1).
  // The two waves of a SIMD so have their VALU work at opposite ends of the
  // interval, under the other's products.  The copies of tile j + 3 go out
  // behind the products; past the last tile its scores are computed once more,
  // unused.
  if (qt0 < n_qt) {
    float4 stat[4];            // the lane's rows of the next tile's lse (role 0) or delta (role 1)
    const auto read_stat = [&](int b) __attribute__((always_inline)) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) stat[jj] = *reinterpret_cast<const float4*>(&st[b][role][8 * jj + rbase]);
    };
#pragma unroll
    for (int b = 0; b < kDkvStages - 1; ++b) issue(b);
    wait_copies<(kDkvStages - 2) * kCopies>();
    ring_barrier();
    read_stat(0);
    products(0, 0, false);
    if (role == 0) probs(qt0, stat, xp[0][grp]);
    else minus(stat);
    int left = hpb * per_head, qt = qt0;
    const auto interval = [&](auto stage) __attribute__((always_inline)) {
      constexpr int b = decltype(stage)::value, bn = (b + 1) % kDkvStages;
      wait_copies<(kDkvStages - 3) * kCopies>();
      ring_barrier();
      if (role == 1) grads(xp[b & 1][grp]);
      __builtin_amdgcn_sched_barrier(0);
      products(b, bn, true);
      __builtin_amdgcn_sched_group_barrier(0x100, 3 * 2, 0);
#pragma unroll
      for (int i = 0; i < D / 16; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      read_stat(bn);
      issue((b + kDkvStages - 1) % kDkvStages);     // under the last products
      if (++qt == n_qt) qt = qt0;
      if (role == 0) probs(qt, stat, xp[bn & 1][grp]);
      else minus(stat);
    };
    while (true) {
      interval(std::integral_constant<int, 0>{});
      if (--left == 0) break;
      interval(std::integral_constant<int, 1>{});
      if (--left == 0) break;
      interval(std::integral_constant<int, 2>{});
      if (--left == 0) break;
      interval(std::integral_constant<int, 3>{});
      if (--left == 0) break;
    }
    wait_copies<0>();      // no copy may land after the end
  }

  if (!key_ok) return;
  // lane owns key my_key; register i of tile dt is d = 32 dt + acc_row(i)
  if (role == 1) {
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) acc[dt] *= p.scale;
  }
  if (p.n_split > 1) {
    // fp32 partial [split][b][key (over segments)][k_t][D], dK then dV at +partial_half; summed by attn_dkv_reduce
    const int64_t key_index = static_cast<int64_t>(p.seg_key0[seg]) + my_key;
    const int64_t row = ((static_cast<int64_t>(split) * p.b + bi) * p.total_keys + key_index) * p.k_t + hk;
    float* pa = p.dkv_partial + (role == 1 ? 0 : p.partial_half) + row * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int d = dt * 32 + 8 * jj + rbase;
        *reinterpret_cast<float4*>(pa + d) = make_float4(acc[dt][4 * jj], acc[dt][4 * jj + 1], acc[dt][4 * jj + 2],
                                                         acc[dt][4 * jj + 3]);
      }
    return;
  }
  const int64_t off = bi * S.bstride + static_cast<int64_t>(my_key) * S.ld + hk * D;
  const int64_t doff = bi * S.d_bstride + static_cast<int64_t>(my_key) * S.d_ld + hk * D;
  const uint16_t* receipt = role == 1 ? S.rk : S.rv;
  if (receipt) {
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int d = dt * 32 + 8 * jj + rbase;
        const u32x2 r = *reinterpret_cast<const u32x2*>(receipt + off + d);
        acc[dt][4 * jj] += lo16(r[0]);
        acc[dt][4 * jj + 1] += hi16(r[0]);
        acc[dt][4 * jj + 2] += lo16(r[1]);
        acc[dt][4 * jj + 3] += hi16(r[1]);
      }
  }
  if (role == 1 && S.rope) {
    constexpr int HALF_T = D / 64;
    const float2* tab = p.rope + static_cast<int64_t>(S.rope_row0 + my_key) * (D / 2);
#pragma unroll
    for (int dt = 0; dt < HALF_T; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float2 cs = tab[dt * 32 + acc_row(i, lane)];
        const float a = acc[dt][i], b = acc[dt + HALF_T][i];
        acc[dt][i] = a * cs.x + b * cs.y;              // rotate by -angle
        acc[dt + HALF_T][i] = b * cs.x - a * cs.y;
      }
  }
  uint16_t* dst = (role == 1 ? S.dk : S.dv) + doff;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int d = dt * 32 + 8 * jj + rbase;
      *reinterpret_cast<u32x2*>(dst + d) =
          u32x2{pack2(acc[dt][4 * jj], acc[dt][4 * jj + 1]), pack2(acc[dt][4 * jj + 2], acc[dt][4 * jj + 3])};
    }
}

// Sum the per-slice fp32 partials, add the receipts, apply the inverse RoPE to
// local keys and store bf16.  One 64-thread block per (key, kv-head, b); thread
// j handles the RoPE pair (j, j + D/2) of dK and of dV.
template <int D>
__global__ void __launch_bounds__(64) attn_dkv_reduce_kernel(AttnParams p) {
  const int key_index = blockIdx.x, hk = blockIdx.y, bi = blockIdx.z;
  const int j = threadIdx.x;
  if (j >= D / 2) return;
  int seg = 0;
  while (seg + 1 < p.n_seg && key_index >= p.seg_key0[seg + 1]) ++seg;
  const KvSeg& S = p.seg[seg];
  const int key = key_index - p.seg_key0[seg];
  float a = 0.f, b = 0.f, va = 0.f, vb = 0.f;
  for (int sp = 0; sp < p.n_split; ++sp) {
    const int64_t row = ((static_cast<int64_t>(sp) * p.b + bi) * p.total_keys + key_index) * p.k_t + hk;
    const float* pk = p.dkv_partial + row * D;
    const float* pv = p.dkv_partial + p.partial_half + row * D;
    a += pk[j];
    b += pk[j + D / 2];
    va += pv[j];
    vb += pv[j + D / 2];
  }
  const int64_t off = bi * S.bstride + static_cast<int64_t>(key) * S.ld + hk * D;
  if (S.rk) {
    a += __uint_as_float(static_cast<uint32_t>(S.rk[off + j]) << 16);
    b += __uint_as_float(static_cast<uint32_t>(S.rk[off + j + D / 2]) << 16);
    va += __uint_as_float(static_cast<uint32_t>(S.rv[off + j]) << 16);
    vb += __uint_as_float(static_cast<uint32_t>(S.rv[off + j + D / 2]) << 16);
  }
  if (S.rope) {
    const float2 cs = p.rope[static_cast<int64_t>(S.rope_row0 + key) * (D / 2) + j];
    const float ra = a * cs.x + b * cs.y, rb = b * cs.x - a * cs.y;
    a = ra;
    b = rb;
  }
  const int64_t doff = bi * S.d_bstride + static_cast<int64_t>(key) * S.d_ld + hk * D;
  S.dk[doff + j] = f2bf(a);
  S.dk[doff + j + D / 2] = f2bf(b);
  S.dv[doff + j] = f2bf(va);
  S.dv[doff + j + D / 2] = f2bf(vb);
}

// ------------------------------------------------------------------ backward: dQ
// One workgroup per (128-query tile, query head, batch element), flat grid in
// the forward's heaviest-first order; 4 waves x 32 queries.  Key tiles of 32
// keep Q, dO, dQ and the two score tiles within 256 registers, so two
// workgroups share a CU.  Per tile: S^T = K Q^T and dP^T = V dO^T, then
// dS^T = P^T (dP^T - delta) feeds dQ^T += K^T dS^T from registers.
// delta = rowsum(dO * O) of the block's queries is formed here, from the dO
// fragments it holds anyway and the matching fragments of O, and written out
// for the dK/dV pass, which runs after this one.
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) attn_bwd_dq_kernel(AttnParams p) {
  constexpr int KQ = 32;                     // keys per tile
  constexpr int TB = KQ * D * 2;
  __shared__ __attribute__((aligned(16))) uint8_t k0[TB], v0[TB], k1[TB], v1[TB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_qt = (p.n_q + 127) / 128;
  const int nh = p.a_t * p.b;
  const int qt = n_qt - 1 - static_cast<int>(blockIdx.x) / nh;
  const int hq = static_cast<int>(blockIdx.x) % nh % p.a_t, bi = static_cast<int>(blockIdx.x) % nh / p.a_t;
  const int hk = hq / (p.a_t / p.k_t);
  const int q_row0 = qt * 128;
  const int my_q = q_row0 + wave * 32 + (lane & 31);
  const bool q_ok = my_q < p.n_q;
  const int my_pos = q_ok ? qpos(p.qmap, my_q) : -1;
  const int blk_last = min(q_row0 + 127, p.n_q - 1);
  const int pos_min = qpos(p.qmap, q_row0), pos_max = qpos(p.qmap, blk_last);
  const int rbase = 4 * (lane >> 5);
  const LaneAddr la = lane_addr<D>(lane);

  bf16x8 qf[D / 16], dof[D / 16];
  float my_delta = 0.f;
  {
    const int64_t off = bi * p.q_bstride + static_cast<int64_t>(q_ok ? my_q : 0) * p.q_ld + hq * D;
    u32x4 of[D / 16];
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const int dcol = (2 * kk + (lane >> 5)) * 8;
      qf[kk] = *reinterpret_cast<const bf16x8*>(p.q + off + dcol);
      dof[kk] = *reinterpret_cast<const bf16x8*>(p.dout + off + dcol);
      of[kk] = *reinterpret_cast<const u32x4*>(p.o + off + dcol);
    }
    // the lane's half of the row (8-column chunks of one parity), then its partner's half
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const u32x4 g = __builtin_bit_cast(u32x4, dof[kk]);
#pragma unroll
      for (int j = 0; j < 4; ++j) my_delta += lo16(g[j]) * lo16(of[kk][j]) + hi16(g[j]) * hi16(of[kk][j]);
    }
    my_delta += __shfl_xor(my_delta, 32, 64);
  }
  const int64_t sidx = (static_cast<int64_t>(bi) * p.a_t + hq) * p.n_q + (q_ok ? my_q : 0);
  const float my_lse = p.lse[sidx] * kLog2e;
  if (q_ok && lane < 32) p.delta[sidx] = my_delta;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    settle(qf[kk]);
    settle(dof[kk]);
  }
  settle(my_lse);
  settle(my_delta);
  const float c = p.scale * kLog2e;
  f32x16 dq[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; ++i) dq[i] = f32x16{};

  KeyWalk walk(p, pos_max, KQ, bi, hk * D);
  const TileCopy<D, KQ> copy(p.seg[0].ld, wave, lane);
  const uint32_t ka[2] = {lds_addr(k0), lds_addr(k1)}, va[2] = {lds_addr(v0), lds_addr(v1)};
  auto issue = [&](Tile t, int b) __attribute__((always_inline)) {
    copy(ka[b], walk.k(), t.kvalid);
    copy(va[b], walk.v(), t.kvalid);
  };
  auto compute = [&](Tile t, const uint8_t* kt, const uint8_t* vt) __attribute__((always_inline)) {
    const int kpos0 = t.kpos0, kvalid = t.kvalid;
    f32x16 sc = f32x16{}, dp = f32x16{};
    scores2<D, kLookDq>(kt, 0, qf, sc, vt, 0, dof, dp, la);
    if (kpos0 + KQ - 1 > pos_min || kvalid < KQ) {      // tile straddles the diagonal (or is ragged)
      const int lim = (q_ok ? min(my_pos - kpos0, kvalid - 1) : -1) - rbase;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + (i & 3) > lim) sc[i] = -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i] = fast_exp2(fmaf(sc[i], c, -my_lse)) * (dp[i] - my_delta);   // dS^T
    const bf16x8 sf[2] = {frag_acc(sc, 0), frag_acc(sc, 8)};
    accum_t<D, 2, kLookDq>(kt, sf, dq, la);
  };
  // Two-stage copy ring: a tile is computed from one buffer pair while the next
  // one lands in the other.
  Tile t = walk.next();
  if (t.kvalid) issue(t, 0);
  while (t.kvalid) {
    Tile t1 = walk.next();
    wait_copies<0>();
    ring_barrier();                      // every wave's copy is visible; the other buffers are free
    if (t1.kvalid) issue(t1, 1);
    __builtin_amdgcn_sched_barrier(0);   // the copies go out now, not next to the wait for them
    compute(t, k0, v0);
    if (!t1.kvalid) break;
    t = walk.next();
    wait_copies<0>();
    ring_barrier();
    if (t.kvalid) issue(t, 0);
    __builtin_amdgcn_sched_barrier(0);
    compute(t1, k1, v1);
  }

  if (!q_ok) return;
  constexpr int HALF_T = D / 64;
  const float2* tab = p.rope + static_cast<int64_t>(my_q) * (D / 2);
#pragma unroll
  for (int dt = 0; dt < HALF_T; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float2 cs = tab[dt * 32 + acc_row(i, lane)];
      const float a = dq[dt][i] * p.scale, b = dq[dt + HALF_T][i] * p.scale;
      dq[dt][i] = a * cs.x + b * cs.y;
      dq[dt + HALF_T][i] = b * cs.x - a * cs.y;
    }
  uint16_t* out = p.dq + (bi * static_cast<int64_t>(p.n_q) + my_q) * p.dq_ld + hq * D;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int d = dt * 32 + 8 * jj + rbase;
      *reinterpret_cast<u32x2*>(out + d) =
          u32x2{pack2(dq[dt][4 * jj], dq[dt][4 * jj + 1]), pack2(dq[dt][4 * jj + 2], dq[dt][4 * jj + 3])};
    }
}

int count_blocks(const AttnParams& p, int tsz) {
  int n = 0;
  for (int s = 0; s < p.n_seg; ++s) n += (p.seg[s].n + tsz - 1) / tsz;
  return n;
}

template <int D>
hipError_t fwd_impl(const AttnParams& p, hipStream_t stream) {
  const unsigned blocks = static_cast<unsigned>((p.n_q + 127) / 128) * p.a_t * p.b;
  hipLaunchKernelGGL(attn_fwd_kernel<D>, dim3(blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

// Host copy of the query-tile walk of the dK/dV kernel: the number of QT-query
// tiles a 128-key block starting at global position kpos0 visits per head.
int dkdv_tiles(const AttnParams& p, int kpos0) {
  const int n_qt = (p.n_q + QT - 1) / QT;
  int n = 0;
  for (int qt = 0; qt < n_qt; ++qt) {
    const int last = std::min(qt * QT + QT - 1, p.n_q - 1);
    const bool second = last >= p.qmap.chunk_len;
    const int pos = (second ? p.qmap.chunk_id[1] : p.qmap.chunk_id[0]) * p.qmap.chunk_len +
                    (second ? last - p.qmap.chunk_len : last);
    if (pos >= kpos0) ++n;
  }
  return n;
}

// Dispatch order of the dK/dV key blocks: most query tiles first (stable), so
// that with context parallelism the long blocks of every key segment start
// before the short ones instead of segment by segment.
void dkdv_order(AttnParams& p) {
  const int nb = count_blocks(p, 128);
  p.n_order = 0;
  if (nb > kMaxKeyBlocks) return;
  std::vector<std::pair<int, int>> w;
  w.reserve(nb);
  int kb = 0;
  for (int s = 0; s < p.n_seg; ++s)
    for (int k0 = 0; k0 < p.seg[s].n; k0 += 128, ++kb) w.push_back({-dkdv_tiles(p, p.seg[s].pos0 + k0), kb});
  std::stable_sort(w.begin(), w.end(), [](const auto& a, const auto& b) { return a.first < b.first; });
  for (int i = 0; i < nb; ++i) p.kb_order[i] = static_cast<uint16_t>(w[i].second);
  p.n_order = nb;
}

template <int D>
hipError_t bwd_impl(const AttnParams& p, int part, hipStream_t stream) {
  if (part == 1) {
    const unsigned blocks = static_cast<unsigned>(count_blocks(p, 128)) * p.k_t * p.n_split * p.b;
    AttnParams q = p;
    dkdv_order(q);
    hipLaunchKernelGGL(attn_bwd_dkdv_kernel<D>, dim3(blocks), dim3(512), 0, stream, q);
  } else if (part == 3) {
    if (p.n_split == 1) return hipSuccess;
    hipLaunchKernelGGL(attn_dkv_reduce_kernel<D>, dim3(p.total_keys, p.k_t, p.b), dim3(64), 0, stream, p);
  } else {
    const unsigned blocks = static_cast<unsigned>((p.n_q + 127) / 128) * p.a_t * p.b;
    hipLaunchKernelGGL(attn_bwd_dq_kernel<D>, dim3(blocks), dim3(256), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace

int attn_bwd_splits(const AttnParams& p) {
  // Split the query heads of a kv-head over workgroups until the dK/dV grid
  // has at least 512 workgroups or every head has its own.  One workgroup runs on
  // a CU at a time, and under the causal mask they differ in length: two per CU
  // let the short ones fill up behind the long ones.  Stopping at 256: 312 + 14 us (the
  // sum of the partials) -> 471 + 10 on the 70B TP8 shard, 301 + 20 -> 458 on 8B
  // TP2 CP2; grids that reach neither number are not touched.
  const int group = p.a_t / p.k_t;
  const int base = count_blocks(p, 128) * p.k_t * p.b;
  int n = 1;
  while (base * n < 512 && n < group && group % (2 * n) == 0) n *= 2;
  return n;
}

hipError_t attn_fwd(const AttnParams& p, hipStream_t stream) {
  if (p.n_q <= 0) return hipSuccess;
  if (p.d_h == 128) return fwd_impl<128>(p, stream);
  if (p.d_h == 64) return fwd_impl<64>(p, stream);
  return hipErrorInvalidValue;
}

hipError_t attn_bwd(const AttnParams& p, int part, hipStream_t stream) {
  if (p.n_q <= 0) return hipSuccess;
  if (p.d_h == 128) return bwd_impl<128>(p, part, stream);
  if (p.d_h == 64) return bwd_impl<64>(p, part, stream);
  return hipErrorInvalidValue;
}

}  // namespace l4d
