// bf16 GEMM on the gfx950 matrix cores: C[m][n] = sum_k A(m,k) B(n,k), fp32
// accumulation, with the layer's fused epilogues.
//
// Operand tiles move global -> LDS by global_load_lds_dwordx4 (direct-to-LDS
// DMA, one contiguous KB per wave instruction, no staging registers), in stages
// of 64 k.  Where K ends inside a stage the copies take zeros instead, so any K
// runs on the same kernels.  Two kernels:
//
//  * gemm_bk64: a workgroup of 8 waves (two per SIMD) owns a 256x256 tile of C,
//    each wave a 128x64 block of v_mfma_f32_32x32x16_bf16 tiles; two stages.  A
//    K-contiguous copy moves 8 whole 128-byte rows per instruction (one cache
//    line each); the fragments of the next 16-k sub-step are read from LDS under
//    the MFMAs of the current one, and the barrier that publishes stage kt+1
//    sits before the last sub-step of stage kt, right after which the freed
//    buffers take stage kt+2 (the A half there, the B half one sub-step later,
//    so the copies do not all reach the texture path at once).
//  * gemm_tile: 128- or 64-row tiles with a deep ring of stages, for the grids
//    that 256-row tiles would leave mostly empty (gemm_plan picks).
//
// Operand layouts: "KC" (reduction index contiguous: activations in the
// forward, the output gradient in dX) is stored row by row, the 16-byte chunks
// of a row permuted by an XOR with row bits so that the 16 rows a 16-lane
// group of a fragment read touches cover all 64 banks (256 bytes) once.  "MN" (reduction
// index strided: the weight in dX, both operands of dW) is stored as k-rows
// of the tile's columns with the 16-byte chunks XOR-swizzled by row, and read with
// two ds_read_b64_tr_b16 that hand each lane 4 consecutive k of one column --
// the transpose happens in the LDS read, not in registers.
//
// A wave's 32-column blocks come in pairs PAIR columns apart, so the columns
// n and n + PAIR land in the same lane and register: a RoPE pair (i, i + d_h/2)
// or a gate/up pair of the fused FFN weight.  The epilogue stages rows through
// LDS and hands 8-column vectors to the fused operation, with that operation's
// global inputs loaded for a whole pass first.  The fp32 accumulate (dW) of the
// 256-row kernel needs no staging: the C tile meets the accumulators in registers.
#include "kernels.h"

namespace l4d {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // the caller's fp32 arrays: float-aligned
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define LPTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int BM = 256, BN = 256, WAVES = 8;   // the 256-row kernel's tile and waves
constexpr int GROUP_M = 4;

__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// Direct-to-LDS copy: 16 bytes per lane from g into the wave's 1 KB LDS chunk
// at lds (lane i lands at byte 16 i).  Inline assembly, so that the compiler's
// wait-count pass does not see an LDS write in flight: it cannot tell one
// stage buffer from another and would wait for every copy before the first
// LDS read of the next stage, exposing the copy latency on every stage.  The
// kernels wait for their own copies (vmcnt) before the barrier that publishes
// a stage, and before the stages are reused as epilogue staging space.
// A scalar write of m0 needs one wait state before a copy into LDS reads it
// (gfx9), which the compiler adds around its own instructions but not inside an
// assembly block: the s_nop is that wait.
// TAG only changes the asm text (a comment), to keep copies in the two arms of
// a branch from being merged.
__device__ __forceinline__ uint32_t lds_addr(const uint8_t* lds) {
  return __builtin_amdgcn_readfirstlane(   // uniform by construction; stated for the compiler
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>(LPTR(const_cast<uint8_t*>(lds)))));
}
template <int TAG = 0>
__device__ __forceinline__ void dma16(const uint16_t* g, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off ; copy form %2" ::"v"(g), "s"(lds), "n"(TAG)
               : "memory", "m0");
}
template <int TAG = 0>
__device__ __forceinline__ void dma16(const uint16_t* g, const uint8_t* lds) {
  dma16<TAG>(g, lds_addr(lds));
}

__device__ __forceinline__ u32x4 pack8(const float* v) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[2 * i], v[2 * i + 1]}, bf16x2));
  return r;
}
__device__ __forceinline__ void unpack8(u32x4 u, float* v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(u[i] << 16);
    v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
  }
}

__device__ __forceinline__ int xcd_remap(int bid, int nwg) {
  const int X = 8;   // workgroups go round-robin over the 8 XCDs; give each a contiguous tile range
  int per = nwg / X, rem = nwg % X, xcd = bid % X, local = bid / X;
  return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// Sixteen zero bytes: the source of a copy whose k lies past the end of K, so
// that a ragged K ends in zeros in LDS and the products need no mask (both
// operands are zero there, so an infinity or NaN elsewhere stays where it is).
__device__ __align__(16) const uint32_t kZeros[4] = {0u, 0u, 0u, 0u};
__device__ __forceinline__ const uint16_t* zeros() { return reinterpret_cast<const uint16_t*>(kZeros); }

// ------------------------------------------------------------------ LDS layouts
// A stage holds 64 k of an operand tile of T rows (T = 256, 128 or 64).
// KC tile: row r holds its 64 k (128 bytes) at r * 128, chunk c of 16 bytes at
// slot c ^ ((r >> 1) & 7).  Two rows share a 256-byte bank line (r % 2 picks
// the half), so the 16 rows one 16-lane group of a fragment read touches cover
// all 64 banks once.
constexpr int BK2 = 64;
constexpr int TILE2 = 256 * BK2 * 2;     // 32 KB per operand per stage of a 256-row tile

__device__ __forceinline__ int kc2_off(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }
// MN tile: k-row r (0..63) of T columns, 16-byte chunk c stored at chunk
// c ^ mn_swz(r).  A transposing read (32 lanes: 4 k-rows x an aligned group of
// 4 chunks) then touches all 64 banks once: with T >= 128 a row spans whole
// bank lines and the 4 rows take 4 different chunk groups; with T = 64 a row is
// half a line, r % 2 picks the half and the swizzle separates rows r and r + 2.
// k-rows r and r + 4 share the pattern.
template <int T>
__device__ __forceinline__ int mn_swz(int row) { return T >= 128 ? (row & 3) << 2 : (row & 2) << 1; }
template <int T>
__device__ __forceinline__ int mn_off(int row, int chunk) { return row * (2 * T) + ((chunk ^ mn_swz<T>(row)) << 4); }

// MFMA operand for rows x0 + lane%32 (x0 a multiple of 32), k = 16 kk + 8 (lane/32) + 0..7.
template <Layout L, int T>
__device__ __forceinline__ bf16x8 frag(const uint8_t* lds, int x0, int kk, int lane) {
  if constexpr (L == Layout::KC) {
    return *reinterpret_cast<const bf16x8*>(lds + kc2_off(x0 + (lane & 31), 2 * kk + (lane >> 5)));
  } else {
    const int li = lane & 15;
    const int row = 16 * kk + 8 * (lane >> 5) + (li >> 2);
    const int x = x0 + 16 * ((lane >> 4) & 1) + 4 * (li & 3);
    const int off = mn_off<T>(row, x >> 3) + ((x & 7) << 1);
    const int off4 = mn_off<T>(row + 4, x >> 3) + ((x & 7) << 1);
    const i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) i16x4*>(LPTR(const_cast<uint8_t*>(lds) + off)));
    const i16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) i16x4*>(LPTR(const_cast<uint8_t*>(lds) + off4)));
    const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
    return __builtin_bit_cast(bf16x8, u32x4{ua[0], ua[1], ub[0], ub[1]});
  }
}

// -------------------------------------------------------------- epilogues

// silu(g) = g * sigmoid(g); the reciprocal is the hardware one (1 ulp), far
// below the bf16 rounding of every value it feeds.
__device__ __forceinline__ float sigmoid_f(float g) { return __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// Global inputs of one epilogue call (8 columns at `col` and the 8 PAIR
// further), loaded for a whole pass of the staged epilogue before the tile is
// staged, so that their latencies overlap instead of adding up.
template <EpiKind KIND>
struct EpiIn {};
template <>
struct EpiIn<EpiKind::ResidualSP> {
  u32x4 r[2], q[2];       // residual, receipt: low and high half
};
template <>
struct EpiIn<EpiKind::SwiGLUBwd> {
  u32x4 g[2], u[2], a[2];
};
template <>
struct EpiIn<EpiKind::QkvRope> {
  float4 cs[4];           // (cos, sin) of the 8 columns
};
template <>
struct EpiIn<EpiKind::AccF32> {
  f32x4 c[4];             // the accumulator: low and high half
};

// Output row of logical row m for ResidualSP: own rows map into own_out,
// the others into the send buffer.
__device__ __forceinline__ int64_t resid_row(const EpiParams& e, int64_t m, bool& own) {
  own = true;
  if (e.t == 1) return m;
  const int64_t bi = m / e.s_c;
  const int32_t i = static_cast<int32_t>(m - bi * e.s_c);
  const int32_t lo_row = e.r * e.s_sp;
  own = i >= lo_row && i < lo_row + e.s_sp;
  return own ? bi * e.s_sp + (i - lo_row) : bi * static_cast<int64_t>(e.t - 1) * e.s_sp + (i < lo_row ? i : i - e.s_sp);
}

// The two halves start at columns n_lo and n_lo + pair.
template <EpiKind KIND, bool STREAM = false>
__device__ __forceinline__ void epi_load(const GemmParams& p, int64_t m, int n_lo, int pair, EpiIn<KIND>& in) {
  const EpiParams& e = p.epi;
  if (m >= p.M) return;
  if constexpr (KIND == EpiKind::ResidualSP) {
    bool own;
    const int64_t orow = resid_row(e, m, own);
    if (!own) return;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = n_lo + h * pair;
      if (n >= p.N) continue;
      const int64_t off = orow * e.ldc + n;
      if (e.resid) in.r[h] = *reinterpret_cast<const u32x4*>(e.resid + off);
      if (e.receipt) in.q[h] = *reinterpret_cast<const u32x4*>(e.receipt + off);
    }
  } else if constexpr (KIND == EpiKind::SwiGLUBwd) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = n_lo + h * pair;
      if (n >= p.N) continue;
      const int64_t off = m * e.f + n;
      in.g[h] = *reinterpret_cast<const u32x4*>(e.g_in + off);
      in.u[h] = *reinterpret_cast<const u32x4*>(e.u_in + off);
      in.a[h] = *reinterpret_cast<const u32x4*>(e.act_in + off);
    }
  } else if constexpr (KIND == EpiKind::AccF32) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = n_lo + h * pair;
      if (n >= p.N) continue;
      const f32x4_a4* c = reinterpret_cast<const f32x4_a4*>(static_cast<const float*>(e.c) + m * e.ldc + n);
      if constexpr (STREAM) {
        in.c[2 * h] = __builtin_nontemporal_load(c);
        in.c[2 * h + 1] = __builtin_nontemporal_load(c + 1);
      } else {
        in.c[2 * h] = c[0];
        in.c[2 * h + 1] = c[1];
      }
    }
  } else if constexpr (KIND == EpiKind::QkvRope) {
    if (n_lo >= p.N || n_lo >= e.nq + e.nk) return;     // V columns are not rotated
    const int n = n_lo < e.nq ? n_lo : n_lo - e.nq;
    const int32_t i = static_cast<int32_t>(m % e.s_c);
    const float4* tab = reinterpret_cast<const float4*>(e.rope + static_cast<int64_t>(i) * (e.d_h / 2) + (n % e.d_h));
#pragma unroll
    for (int j = 0; j < 4; ++j) in.cs[j] = tab[j];
  }
}

// lo: 8 columns starting at column n_lo; hi: the 8 columns `pair` further.
template <EpiKind KIND, bool STREAM = false>
__device__ __forceinline__ void epilogue(const GemmParams& p, int64_t m, int n_lo, int pair, float* lo, float* hi,
                                         const EpiIn<KIND>& in) {
  const EpiParams& e = p.epi;
  if (m >= p.M) return;
  switch (KIND) {
    case EpiKind::StoreBF16: {
      uint16_t* c = static_cast<uint16_t*>(e.c) + m * e.ldc;
      if (n_lo < p.N) *reinterpret_cast<u32x4*>(c + n_lo) = pack8(lo);
      if (n_lo + pair < p.N) *reinterpret_cast<u32x4*>(c + n_lo + pair) = pack8(hi);
      break;
    }
    case EpiKind::StoreF32: {
      float* c = static_cast<float*>(e.c) + m * e.ldc;
      if (n_lo < p.N) {
        *reinterpret_cast<float4*>(c + n_lo) = make_float4(lo[0], lo[1], lo[2], lo[3]);
        *reinterpret_cast<float4*>(c + n_lo + 4) = make_float4(lo[4], lo[5], lo[6], lo[7]);
      }
      if (n_lo + pair < p.N) {
        *reinterpret_cast<float4*>(c + n_lo + pair) = make_float4(hi[0], hi[1], hi[2], hi[3]);
        *reinterpret_cast<float4*>(c + n_lo + pair + 4) = make_float4(hi[4], hi[5], hi[6], hi[7]);
      }
      break;
    }
    case EpiKind::AccF32: {   // the 256-row kernel adds in registers instead (acc_add_store_f32)
      if constexpr (KIND == EpiKind::AccF32) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int n = n_lo + h * pair;
          if (n >= p.N) continue;
          const float* src = h ? hi : lo;
          float* c = static_cast<float*>(e.c) + m * e.ldc + n;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const f32x4 v = in.c[2 * h + q] + f32x4{src[4 * q], src[4 * q + 1], src[4 * q + 2], src[4 * q + 3]};
            f32x4_a4* out = reinterpret_cast<f32x4_a4*>(c + 4 * q);
            if constexpr (STREAM) __builtin_nontemporal_store(static_cast<f32x4_a4>(v), out);
            else *out = v;
          }
        }
      }
      break;
    }
    case EpiKind::QkvRope: {
      if constexpr (KIND == EpiKind::QkvRope) {
        // n_lo lies in the first half of a head, n_lo + pair (pair = d_h/2) in the second.
        if (n_lo >= p.N) break;
        uint16_t* dst;
        int64_t ld;
        int n;
        bool rot = true;
        if (n_lo < e.nq) { dst = e.q; ld = e.nq; n = n_lo; }
        else if (n_lo < e.nq + e.nk) { dst = e.k; ld = e.nk; n = n_lo - e.nq; }
        else { dst = e.v; ld = e.nk; n = n_lo - e.nq - e.nk; rot = false; }
        if (rot) {
          float a[8], b[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float c = j & 1 ? in.cs[j >> 1].z : in.cs[j >> 1].x;
            const float sn = j & 1 ? in.cs[j >> 1].w : in.cs[j >> 1].y;
            a[j] = lo[j] * c - hi[j] * sn;
            b[j] = hi[j] * c + lo[j] * sn;
          }
          *reinterpret_cast<u32x4*>(dst + m * ld + n) = pack8(a);
          *reinterpret_cast<u32x4*>(dst + m * ld + n + pair) = pack8(b);
        } else {
          *reinterpret_cast<u32x4*>(dst + m * ld + n) = pack8(lo);
          *reinterpret_cast<u32x4*>(dst + m * ld + n + pair) = pack8(hi);
        }
      }
      break;
    }
    case EpiKind::ResidualSP: {
      if constexpr (KIND == EpiKind::ResidualSP) {
        bool own;
        const int64_t orow = resid_row(e, m, own);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int n = n_lo + h * pair;
          if (n >= p.N) continue;
          float* src = h ? hi : lo;
          const int64_t off = orow * e.ldc + n;
          if (own) {
            float r[8];
            if (e.resid) {
              unpack8(in.r[h], r);
#pragma unroll
              for (int j = 0; j < 8; ++j) src[j] += r[j];
            }
            if (e.receipt) {
              unpack8(in.q[h], r);
#pragma unroll
              for (int j = 0; j < 8; ++j) src[j] += r[j];
            }
            if (e.own_out_f32) {
              float4* o32 = reinterpret_cast<float4*>(e.own_out_f32 + off);
              o32[0] = make_float4(src[0], src[1], src[2], src[3]);
              o32[1] = make_float4(src[4], src[5], src[6], src[7]);
            } else {
              *reinterpret_cast<u32x4*>(e.own_out + off) = pack8(src);
            }
          } else {
            *reinterpret_cast<u32x4*>(e.send + off) = pack8(src);
          }
        }
      }
      break;
    }
    case EpiKind::SwiGLUFwd: {
      const int j = n_lo;                 // FFN column of this gate/up pair
      if (j >= e.f) break;
      const int64_t off = m * e.f + j;
      float g[8], u[8], a[8], pr[8];
      unpack8(pack8(lo), g);              // the stored (rounded) G and U feed act and prod
      unpack8(pack8(hi), u);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        a[q] = g[q] * sigmoid_f(g[q]);
        pr[q] = a[q] * u[q];
      }
      *reinterpret_cast<u32x4*>(e.g_out + off) = pack8(g);
      *reinterpret_cast<u32x4*>(e.u_out + off) = pack8(u);
      *reinterpret_cast<u32x4*>(e.act_out + off) = pack8(a);
      *reinterpret_cast<u32x4*>(e.prod_out + off) = pack8(pr);
      break;
    }
    case EpiKind::SwiGLUBwd: {
      if constexpr (KIND == EpiKind::SwiGLUBwd) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int n = n_lo + h * pair;
          if (n >= p.N) continue;
          const float* dp = h ? hi : lo;
          const int64_t off = m * e.f + n;
          float g[8], u[8], a[8], dg[8], du[8];
          unpack8(in.g[h], g);
          unpack8(in.u[h], u);
          unpack8(in.a[h], a);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float s = sigmoid_f(g[q]);
            dg[q] = dp[q] * u[q] * (s * (1.0f + g[q] * (1.0f - s)));
            du[q] = dp[q] * a[q];
          }
          uint16_t* out = e.dgu + m * (2 * static_cast<int64_t>(e.f));
          *reinterpret_cast<u32x4*>(out + n) = pack8(dg);
          *reinterpret_cast<u32x4*>(out + e.f + n) = pack8(du);
        }
      }
      break;
    }
  }
}

// Tile column of a wave's low 32-column block; its partner is PAIR further.
template <int PAIR>
__device__ __forceinline__ int lo_col(int wn) {
  constexpr int PW = PAIR / 32;
  return (wn / PW) * (2 * PAIR) + (wn % PW) * 32;
}

// -------------------------------------------------------------- the kernels

// Workgroup barrier between pipeline steps.  __syncthreads() would also fence
// global memory, i.e. wait for every copy still in flight -- including the
// stages being prefetched; each wave has already waited for its own copies of
// the step that is about to be read, so only the LDS reads of the previous
// step (lgkmcnt) must drain before the barrier.
__device__ __forceinline__ void stage_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Wait until at most N of the wave's copies are still in flight.
template <int N>
__device__ __forceinline__ void wait_copies() {
  static_assert(N <= 63, "the wait counter holds 6 bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// First column of tile tn: a gate/up tile holds 128 FFN columns of each half.
template <EpiKind KIND>
__device__ __forceinline__ int n_first(int tn) { return KIND == EpiKind::SwiGLUFwd ? tn * 128 : tn * BN; }

// Epilogue: each wave stages R rows x (NS*32) columns of fp32 at a time in its
// own 16 KB of LDS (column halves swapped on rows with bit 2 set, so the two
// half-waves write different banks) and hands out 8-column vectors of its low
// blocks with their PAIR partners.  Accumulator register i of a lane: row
// 8(i/4) + 4(lane/32) + i%4, column lane%32 of its 32x32 tile.  The global
// inputs of a pass are loaded before its rows are staged.
template <EpiKind KIND, int PAIR, int NS>
__device__ __forceinline__ void store_tile(const GemmParams& p, f32x16 (&acc)[4][NS], float* st, int64_t row0,
                                           int tn, const int* ncol, int lane) {
  constexpr int C = NS * 32, R = 4096 / C, PASSES = 128 / R, MS_PER = R / 32;
  constexpr int VEC = R * (NS / 2) * 4;  // 8-column vectors of the low blocks per pass
  constexpr int ITERS = VEC / 64;
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    EpiIn<KIND> in[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int idx = it * 64 + lane;
      const int rr = idx / ((NS / 2) * 4), v = idx % ((NS / 2) * 4);
      epi_load<KIND>(p, row0 + pass * R + rr, n_first<KIND>(tn) + ncol[v >> 2] + (v & 3) * 8, PAIR, in[it]);
    }
#pragma unroll
    for (int mm = 0; mm < MS_PER; ++mm)
#pragma unroll
      for (int ns = 0; ns < NS; ++ns)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int r = mm * 32 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
          const int cc = (ns * 32 + (lane & 31)) ^ (((r >> 2) & 1) << 4);
          st[r * C + cc] = acc[pass * MS_PER + mm][ns][i];
        }
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int idx = it * 64 + lane;
      const int rr = idx / ((NS / 2) * 4), v = idx % ((NS / 2) * 4);
      const int j = v >> 2, c8 = (v & 3) * 8;
      const int flip = ((rr >> 2) & 1) << 4;
      const float4* lo4 = reinterpret_cast<const float4*>(st + rr * C + ((j * 32 + c8) ^ flip));
      const float4* hi4 = reinterpret_cast<const float4*>(st + rr * C + (((j + NS / 2) * 32 + c8) ^ flip));
      const float4 l0 = lo4[0], l1 = lo4[1], h0 = hi4[0], h1 = hi4[1];
      float lo[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
      float hi[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
      epilogue<KIND>(p, row0 + pass * R + rr, n_first<KIND>(tn) + ncol[j] + c8, PAIR, lo, hi, in[it]);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
  }
}

// AccF32 (C += A B^T in fp32) of the 256-row kernel works on the accumulators
// directly: in the accumulator layout the 32 lanes of a half-wave cover 32
// consecutive columns (128 bytes) of one row, so loads and stores are
// whole-line accesses without staging.  Whole tiles load and store
// non-temporally: each C element is touched once per launch, and streaming it
// leaves L2 to the operand tiles the neighbouring workgroups share (4-5% off
// the largest weight-gradient GEMM of the Llama-2-7B layer).
template <int NS>
__device__ __forceinline__ void acc_store_f32(const f32x16 (&acc)[4][NS], const GemmParams& p, float* cbase,
                                              int64_t ldc, int64_t row0, int tn, const int* ncol, int lane) {
  const int rl = 4 * (lane >> 5);
  int32_t off[NS];
#pragma unroll
  for (int ns = 0; ns < NS; ++ns) off[ns] = static_cast<int32_t>(rl * ldc) + tn * BN + ncol[ns] + (lane & 31);
  const bool full = row0 + 128 <= p.M && (tn + 1) * BN <= p.N;
#pragma unroll
  for (int ms = 0; ms < 4; ++ms)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = ms * 32 + 8 * (i >> 2) + (i & 3);
      float* row = cbase + (row0 + r) * ldc;
#pragma unroll
      for (int ns = 0; ns < NS; ++ns) {
        const int n = tn * BN + ncol[ns] + (lane & 31);
        if (full || (row0 + r + rl < p.M && n < p.N)) __builtin_nontemporal_store(acc[ms][ns][i], &row[off[ns]]);
      }
    }
}

// acc + C -> C for a tile whose products started from zero, one accumulator
// row block (32 rows) at a time.  Whole tiles are software-pipelined: the
// loads of block ms + 1 are issued before the stores of block ms, so that
// waiting for a block's C values (the wait counter also counts stores) does
// not wait for the stores issued after them.  They go through a buffer
// descriptor of the wave's 128 rows: the row offset is a scalar, the lane
// offset one register per column block, which leaves the registers for the
// two blocks of C in flight.  Edge tiles go element by element.
constexpr int kBufNT = 2;   // cache-policy bit of a non-temporal buffer access
template <int NS>
__device__ __forceinline__ void acc_add_store_f32(const f32x16 (&acc)[4][NS], const GemmParams& p, float* cbase,
                                                  int64_t ldc, int64_t row0, int tn, const int* ncol, int lane) {
  const int rl = 4 * (lane >> 5);
  if (row0 + 128 <= p.M && (tn + 1) * BN <= p.N) {   // uniform
    const __amdgpu_buffer_rsrc_t win =
        __builtin_amdgcn_make_buffer_rsrc(cbase + row0 * ldc, 0, static_cast<int>(0x7fffffff), 0x00020000);
    int32_t voff[NS];   // lane's byte offset in its row
#pragma unroll
    for (int ns = 0; ns < NS; ++ns) voff[ns] = (static_cast<int32_t>(rl * ldc) + tn * BN + ncol[ns] + (lane & 31)) * 4;
    const int32_t ldc4 = static_cast<int32_t>(ldc * 4);
    float c[2][16][NS];   // the buffer builtins move 32-bit words: bit casts, not conversions
    auto load = [&](int ms, float (&cb)[16][NS]) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
          cb[i][ns] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                       win, voff[ns], (ms * 32 + 8 * (i >> 2) + (i & 3)) * ldc4, kBufNT));
    };
    load(0, c[0]);
#pragma unroll
    for (int ms = 0; ms < 4; ++ms) {
      if (ms + 1 < 4) load(ms + 1, c[(ms + 1) & 1]);
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, acc[ms][ns][i] + c[ms & 1][i][ns]), win,
                                                voff[ns], (ms * 32 + 8 * (i >> 2) + (i & 3)) * ldc4, kBufNT);
    }
    return;
  }
  int32_t off[NS];
#pragma unroll
  for (int ns = 0; ns < NS; ++ns) off[ns] = static_cast<int32_t>(rl * ldc) + tn * BN + ncol[ns] + (lane & 31);
#pragma unroll
  for (int ms = 0; ms < 4; ++ms)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = ms * 32 + 8 * (i >> 2) + (i & 3);
      float* row = cbase + (row0 + r) * ldc;
#pragma unroll
      for (int ns = 0; ns < NS; ++ns) {
        const int n = tn * BN + ncol[ns] + (lane & 31);
        if (row0 + r + rl < p.M && n < p.N) row[off[ns]] += acc[ms][ns][i];
      }
    }
}

struct TileCoord {
  int tm, tn;
};
// Tile `pid` in the grouped order: GROUP_M tile rows at a time, column by column.
__device__ __forceinline__ TileCoord tile_coord(const GemmParams& p, int pid) {
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tiles_n = p.B.split_rows ? (p.B.split_rows + 127) / 128 : (p.N + BN - 1) / BN;
  const int group = GROUP_M * tiles_n;
  const int first_m = (pid / group) * GROUP_M;
  const int gm = min(tiles_m - first_m, GROUP_M);
  return TileCoord{first_m + (pid % group) % gm, (pid % group) / gm};
}
__device__ __forceinline__ TileCoord tile_of(const GemmParams& p) {
  return tile_coord(p, xcd_remap(blockIdx.x, gridDim.x));
}

// ---------------------------------------------------------- 256-row tiles, BK = 64
struct Kc2Rows {
  const uint16_t* row[32 / WAVES];
  int c8;
};

// Copy q of wave w moves rows 8 kb + lane/8, kb = w + WAVES q; (row >> 1) & 7 =
// 4 (w & 1) + lane/16 is the same for every q.
__device__ __forceinline__ Kc2Rows kc2_rows(const Operand& op, int x0, int tile_idx, int wave, int lane) {
  Kc2Rows r;
  r.c8 = 8 * ((lane & 7) ^ (4 * (wave & 1) + (lane >> 4)));
#pragma unroll
  for (int q = 0; q < 32 / WAVES; ++q) {
    const int xr = 8 * (wave + WAVES * q) + (lane >> 3);
    int64_t gx;
    if (op.split_rows) {
      int i = tile_idx * 128 + (xr & 127);
      if (i >= op.split_rows) i = op.split_rows - 1;
      gx = (xr >= 128 ? op.split_off : 0) + i;
    } else {
      gx = x0 + xr;
      if (gx >= op.rows) gx = op.rows - 1;
    }
    r.row[q] = op.src.row(gx);
  }
  return r;
}

// RAGGED: K may end inside the stage (or before it); chunks past it copy zeros.
template <bool RAGGED>
__device__ __forceinline__ void copy2_kc(uint8_t* lds, const Kc2Rows& rows, int k0, int K, int wave) {
  const int k = k0 + rows.c8;
#pragma unroll
  for (int q = 0; q < 32 / WAVES; ++q)
    dma16(!RAGGED || k < K ? rows.row[q] + k : zeros(), lds + (wave + WAVES * q) * 1024);
}

// MN copies.  For an operand whose rows are one plain array (no sequence-
// parallel split) a lane's offset is fixed over K and across its copies up to
// a uniform stride: copy q reads k-row kr0 + 2 * WAVES * q, and the column
// swizzle depends on kr mod 4, which q does not change.  One offset per lane
// is kept; each stage adds one uniform row offset.  A split operand whose
// slots hold a multiple of 64 rows does the same from the mapped first row of
// the stage; any other split operand resolves every k-row through RowSrc.  The
// two arms issue textually different copies
// (dma16<1> for the split one): with identical ones the compiler sinks the copy
// below the branch and computes both addresses on every copy.
// How the k-rows of the MN operands map to memory: one plain array; runs of at
// least 64 rows per stage (plain, or gathered slots of a multiple of 64 rows:
// one scalar mapping per stage); or any slots (a mapping per lane and copy).  The
// host picks the kernel, so that a main loop holds only its own mapping.
constexpr int kPlainRows = 0, kRunRows = 1, kAnyRows = 2;

// The own or the peer pointer, picked by arithmetic on the two values: a select
// of the members' addresses would put the kernel argument on the stack.
__device__ __forceinline__ const uint16_t* pick(const RowSrc& src, bool peer) {
  const uint64_t a = reinterpret_cast<uint64_t>(src.own), b = reinterpret_cast<uint64_t>(src.peer);
  return reinterpret_cast<const uint16_t*>(a + ((b - a) & (0ull - static_cast<uint64_t>(peer))));
}
__device__ __forceinline__ const uint16_t* mapped_row(const RowSrc& src, int k) {
  if (src.t == 1) return src.own + static_cast<int64_t>(k) * src.ld;
  const uint32_t o = src.row_index(k);
  return pick(src, o >> 31) + static_cast<int64_t>(o & 0x7fffffffu) * src.ld;
}
// Rows of a stage of a split operand whose slots are no multiple of 64 rows:
// the sequence of the stage's first row is found once (a scalar division), a
// lane steps to the next sequence at most once where s_c >= 64.  Rows past the
// last sequence give addresses that the caller replaces.
struct StageRows {
  int b0, i0;
  __device__ __forceinline__ const uint16_t* row(const RowSrc& src, int kr) const {
    int bi = b0, i = i0 + kr;
    while (i >= src.s_c) {
      i -= src.s_c;
      ++bi;
    }
    const int lo = src.r * src.s_sp;
    const bool own = i >= lo && i < lo + src.s_sp;
    const int r = own ? bi * src.s_sp + (i - lo) : bi * (src.t - 1) * src.s_sp + (i < lo ? i : i - src.s_sp);
    return pick(src, !own) + static_cast<int64_t>(r) * src.ld;
  }
};
__device__ __forceinline__ StageRows stage_rows(const RowSrc& src, int k0) {
  const int b0 = k0 / src.s_c;
  return StageRows{b0, k0 - b0 * src.s_c};
}

struct Mn2Rows {
  uint32_t off0;   // element offset of the lane's 16 bytes for copy 0 at k0 = 0
};

__device__ __forceinline__ Mn2Rows mn2_rows(const Operand& op, int x0, int wave, int lane) {
  const int kr = 2 * wave + (lane >> 5);
  const int lc = (lane & 31) ^ mn_swz<256>(kr);
  int x = x0 + lc * 8;
  if (x >= op.rows) x = op.rows - 8;
  return Mn2Rows{static_cast<uint32_t>(kr * op.src.ld + x)};
}

template <bool RAGGED, int MAP>
__device__ __forceinline__ void copy2_mn(uint8_t* lds, const Operand& op, const Mn2Rows& rows, int x0, int k0, int K,
                                         int wave, int lane) {
  // A stage's 64 k-rows are consecutive in memory when the operand is one
  // plain array, and also when it is split but every sequence-parallel slot
  // holds a multiple of 64 rows (stages start at multiples of 64, so none
  // straddles a slot or a sequence): then the stage's first row is mapped
  // once (uniform, scalar) and each lane adds its fixed offset.
  if (MAP != kAnyRows || op.src.t == 1 || op.src.s_sp % BK2 == 0) {       // uniform
    const uint16_t* base0 = MAP != kPlainRows ? mapped_row(op.src, RAGGED && k0 >= K ? 0 : k0)
                                              : op.src.own + static_cast<int64_t>(k0) * op.src.ld;
#pragma unroll
    for (int q = 0; q < 32 / WAVES; ++q) {
      const uint16_t* g = base0 + static_cast<int64_t>(2 * WAVES * q) * op.src.ld + rows.off0;
      if constexpr (RAGGED) g = k0 + 2 * (wave + WAVES * q) + (lane >> 5) < K ? g : zeros();
      dma16(g, lds + (wave + WAVES * q) * 1024);
    }
    return;
  }
  const StageRows sr = stage_rows(op.src, k0);
#pragma unroll
  for (int q = 0; q < 32 / WAVES; ++q) {
    const int kb = wave + WAVES * q;
    const int kr = 2 * kb + (lane >> 5);
    const int lc = (lane & 31) ^ mn_swz<256>(kr);
    int x = x0 + lc * 8;
    if (x >= op.rows) x = op.rows - 8;
    const uint16_t* g = sr.row(op.src, kr) + x;
    if constexpr (RAGGED) g = k0 + kr < K ? g : zeros();
    dma16<1>(g, lds + kb * 1024);
  }
}

template <int NS>
struct Frags2 {
  bf16x8 a[4], b[NS];
};

// Fragments are read in the order the products consume them (A0, B0 .. B(NS-1),
// A1, A2, A3), so the first products of the next sub-step wait on the
// earliest reads.
template <Layout LA, Layout LB, int NS>
__device__ __forceinline__ void read_frags2(Frags2<NS>& f, const uint8_t* la, const uint8_t* lb, int wm,
                                            const int* ncol, int kk, int lane) {
  f.a[0] = frag<LA, 256>(la, wm * 128, kk, lane);
#pragma unroll
  for (int ns = 0; ns < NS; ++ns) f.b[ns] = frag<LB, 256>(lb, ncol[ns], kk, lane);
#pragma unroll
  for (int ms = 1; ms < 4; ++ms) f.a[ms] = frag<LA, 256>(la, wm * 128 + ms * 32, kk, lane);
}

template <int NS>
__device__ __forceinline__ void mfma_frags2(f32x16 (&acc)[4][NS], const Frags2<NS>& f) {
#pragma unroll
  for (int ms = 0; ms < 4; ++ms)
#pragma unroll
    for (int ns = 0; ns < NS; ++ns)
      acc[ms][ns] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ms], f.b[ns], acc[ms][ns], 0, 0, 0);
}

// Spread DS reads over the MFMAs of a sub-step: 8 slots of (DS share, M MFMAs).
// A K-contiguous fragment is one LDS read, a transposed one two.
template <int DS, int M, int I = 0>
__device__ __forceinline__ void interleave2_slots() {
  if constexpr (I < 8) {
    constexpr int n = (DS * (I + 1)) / 8 - (DS * I) / 8;
    if constexpr (n > 0) __builtin_amdgcn_sched_group_barrier(0x100, n, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, M, 0);
    interleave2_slots<DS, M, I + 1>();
  }
}
template <Layout LA, Layout LB, int NS>
__device__ __forceinline__ void interleave2() {
  constexpr int DS = 4 * (LA == Layout::KC ? 1 : 2) + NS * (LB == Layout::KC ? 1 : 2);
  interleave2_slots<DS, NS / 2>();
}

// The BK = 64 main loop of one tile over its stages [kb, kb + n), n even:
// products added into acc.  The four stage buffers a0 b0 a1 b1 (32 KB each)
// hold two stages.
template <Layout LA, Layout LB, int NS, bool RAGGED, int MAP>
__device__ __forceinline__ void mainloop64(const GemmParams& p, f32x16 (&acc)[4][NS], int tm, int tn,
                                           int kb, int n, uint8_t* a0, uint8_t* b0, uint8_t* a1, uint8_t* b1,
                                           int wave, int lane, int wm, const int* ncol) {
  const int m0 = tm * BM, n0 = tn * BN;
  Kc2Rows ra{}, rb{};
  Mn2Rows ma{}, mb{};
  if constexpr (LA == Layout::KC) ra = kc2_rows(p.A, m0, tm, wave, lane);
  else ma = mn2_rows(p.A, m0, wave, lane);
  if constexpr (LB == Layout::KC) rb = kc2_rows(p.B, n0, tn, wave, lane);
  else mb = mn2_rows(p.B, n0, wave, lane);
  // stage kt of the range (stages past its end repeat the last one: the wait counts stay fixed)
  auto issue_a = [&](int kt, uint8_t* la) {
    const int k0 = (kb + min(kt, n - 1)) * BK2;
    if constexpr (LA == Layout::KC) copy2_kc<RAGGED>(la, ra, k0, p.K, wave);
    else copy2_mn<RAGGED, MAP>(la, p.A, ma, m0, k0, p.K, wave, lane);
  };
  auto issue_b = [&](int kt, uint8_t* lb) {
    const int k0 = (kb + min(kt, n - 1)) * BK2;
    if constexpr (LB == Layout::KC) copy2_kc<RAGGED>(lb, rb, k0, p.K, wave);
    else copy2_mn<RAGGED, MAP>(lb, p.B, mb, n0, k0, p.K, wave, lane);
  };

  Frags2<NS> f0, f1;
  // Stage kt (buffers X, next stage in Y): sub-steps kk = 0..3 each read the
  // fragments of the next sub-step under their own MFMAs.  Before the last
  // sub-step every wave has read all of X: wait for stage kt+1, publish it
  // with the barrier, refill X's A half with stage kt+2 and read the first
  // fragments of Y under the last MFMAs.  The B half of stage kt+2 follows at
  // the start of stage kt+1 (measured a few percent faster than issuing both
  // halves at the barrier).
  auto stage = [&](int kt, uint8_t* xa, uint8_t* xb, const uint8_t* ya, uint8_t* yb) {
    if (kt > 0) {
      issue_b(kt + 1, yb);   // stage kt+1's B half (Y's B buffer was freed at kt-1's barrier)
      __builtin_amdgcn_sched_barrier(0);
    }
    read_frags2<LA, LB, NS>(f1, xa, xb, wm, ncol, 1, lane);
    mfma_frags2<NS>(acc, f0);
    interleave2<LA, LB, NS>();
    read_frags2<LA, LB, NS>(f0, xa, xb, wm, ncol, 2, lane);
    mfma_frags2<NS>(acc, f1);
    interleave2<LA, LB, NS>();
    read_frags2<LA, LB, NS>(f1, xa, xb, wm, ncol, 3, lane);
    mfma_frags2<NS>(acc, f0);
    interleave2<LA, LB, NS>();
    wait_copies<0>();
    stage_barrier();
    issue_a(kt + 2, xa);
    // Keep the copies here, right after the barrier: left alone, the scheduler
    // sinks them to the end of the next stage, next to the wait for them, and
    // no computation overlaps their latency.
    __builtin_amdgcn_sched_barrier(0);
    read_frags2<LA, LB, NS>(f0, ya, yb, wm, ncol, 0, lane);   // after the last stage: read, never used
    mfma_frags2<NS>(acc, f1);
    interleave2<LA, LB, NS>();
  };

  issue_a(0, a0);
  issue_b(0, b0);
  issue_a(1, a1);
  issue_b(1, b1);
  wait_copies<8>();      // stage 0 is there; the 4 + 4 copies of stage 1 may be in flight
  stage_barrier();
  read_frags2<LA, LB, NS>(f0, a0, b0, wm, ncol, 0, lane);
  for (int kt = 0; kt < n; kt += 2) {
    stage(kt, a0, b0, a1, b1);
    stage(kt + 1, a1, b1, a0, b0);
  }
  wait_copies<0>();      // the last (repeated) stage copy has landed
}

// Wave-private staging space of the epilogue in the stage buffers.
__device__ __forceinline__ float* stage_space(uint8_t* a0, uint8_t* b0, uint8_t* a1, uint8_t* b1, int wave) {
  const int q = wave >> 1;
  uint8_t* mine = q == 0 ? a0 : q == 1 ? b0 : q == 2 ? a1 : b1;
  mine += (wave & 1) * 16384;
  return reinterpret_cast<float*>(mine);
}

template <Layout LA, Layout LB, EpiKind KIND, int PAIR, bool RAGGED, int MAP>
__global__ void __launch_bounds__(WAVES * 64, 1) gemm_bk64(GemmParams p) {
  constexpr int NS = 2;      // 32-column blocks of a wave
  __shared__ __attribute__((aligned(16))) uint8_t a0[TILE2], b0[TILE2], a1[TILE2], b1[TILE2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform per wave: scalar code for wave-level decisions
  // AccF32 with a split K range: the grid is k_splits copies of the tile grid,
  // part-major after the XCD remap, so an XCD's neighbouring tiles share a part.
  constexpr bool kSplittable = KIND == EpiKind::AccF32 || KIND == EpiKind::StoreBF16;
  const int parts = kSplittable && p.k_splits > 1 ? p.k_splits : 1;
  const int pid_all = xcd_remap(blockIdx.x, gridDim.x);
  const int tiles = static_cast<int>(gridDim.x) / parts;
  const int part = pid_all / tiles;
  const TileCoord tc = tile_coord(p, pid_all - part * tiles);
  const int tm = tc.tm, tn = tc.tn, m0 = tm * BM;
  const int wm = wave >> 2, wn = wave & 3;
  int ncol[NS];
#pragma unroll
  for (int j = 0; j < NS / 2; ++j) {
    ncol[j] = lo_col<PAIR>(wn);
    ncol[j + NS / 2] = ncol[j] + PAIR;
  }
  // stages per part, even; past the end of K they hold zeros (only without a split)
  const int n_st = RAGGED ? (p.K + 2 * BK2 - 1) / (2 * BK2) * 2 : p.K / BK2 / parts;
  float* cbase = nullptr;
  int64_t ldc = 0;
  if constexpr (KIND == EpiKind::AccF32) {
    cbase = part == 0 ? static_cast<float*>(p.epi.c) : p.partial + static_cast<int64_t>(part - 1) * p.M * p.N;
    ldc = part == 0 ? p.epi.ldc : p.N;
  } else if constexpr (KIND == EpiKind::StoreBF16) {
    // split: every part stores its fp32 sum; the reduce pass adds them and rounds to bf16
    cbase = p.partial + static_cast<int64_t>(part) * p.M * p.N;
    ldc = p.N;
  }

  f32x16 acc[4][NS];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NS; ++j) acc[i][j] = f32x16{};
  // Unless RAGGED, K is a multiple of 2 * BK2 * parts.
  mainloop64<LA, LB, NS, RAGGED, MAP>(p, acc, tm, tn, part * n_st, n_st, a0, b0, a1, b1, wave, lane, wm, ncol);
  // The fp32 accumulate: the products start from zero and part 0 adds the C
  // tile in the epilogue, whose loads overlap its stores (loading C into the
  // accumulators before the first product measured 2-3% slower on the largest
  // weight-gradient GEMMs of the Llama-3-70B TP8 shard).
  if (KIND == EpiKind::AccF32 && part == 0) {
    acc_add_store_f32<NS>(acc, p, cbase, ldc, static_cast<int64_t>(m0) + wm * 128, tn, ncol, lane);
    return;
  }
  if (KIND == EpiKind::AccF32 || (KIND == EpiKind::StoreBF16 && parts > 1)) {
    acc_store_f32<NS>(acc, p, cbase, ldc, static_cast<int64_t>(m0) + wm * 128, tn, ncol, lane);
  } else {
    __syncthreads();   // every wave is done reading the stages
    store_tile<KIND, PAIR, NS>(p, acc, stage_space(a0, b0, a1, b1, wave), static_cast<int64_t>(m0) + wm * 128,
                               tn, ncol, lane);
  }
}

// ---------------------------------------------------------- T-row tiles, T = 128 or 64
// For grids that 256-row tiles would leave mostly empty: with one workgroup per
// CU or less, a 256-row stage costs about 1.1 us (copy latency, LDS latency and
// barrier in turn), whatever the chip does elsewhere.  A workgroup owns a
// T x T tile: W / 4 groups of 4 waves, each wave a quarter of the tile (2 x 2
// MFMA blocks at T = 128, one at T = 64) over its group's share of every
// stage's k; with W = 8 the two groups' sums meet in the epilogue.  Operands
// stream through a ring of S stages of 64 k with S - 1 of them in flight: a
// tile's time is the copy latency plus its products, where the 256-row kernel's
// two stages expose the latency when few workgroups run.  One barrier per stage;
// at a full chip the copies bound it (T = 128: 32 KB per stage in 0.6 us, 14 TB/s
// over the chip).  Layer of hidden 1024 on 1000 tokens, forward + backward: 690 ->
// 347 us; hidden 256 on 128 tokens: 317 -> 125 us (all GEMMs on 256-row tiles
// before).
// W = 8 (two waves per SIMD), S = 128 KB of stages: one workgroup per CU, for
// grids that fit the chip once.  W = 4 with 64 KB of stages: two workgroups per
// CU, for larger grids.
//
// Columns: the tile's T/2 "low" columns j = tn T/2 + (0..T/2) and their partners
// `pair` further, low column j sitting at matrix column (j / pair) 2 pair +
// j % pair.  With pair = T/2 that is T consecutive columns; with pair = d_h/2 it
// keeps RoPE pairs together and with pair = f the gate and up columns, for any T.
//
// A wave issues C = T / (8 W) copies of 1 KB per operand and stage.
template <int T, int W>
struct RowPtrs {
  const uint16_t* row[T / (8 * W)];
  int c8;
};

// Source rows of the wave's copies of a KC stage: copy q moves tile rows
// 8 (wave + W q) + lane/8.
template <int T, int W, bool PAIRED>
__device__ __forceinline__ RowPtrs<T, W> tile_rows(const Operand& op, int tile, int pair, int wave, int lane) {
  RowPtrs<T, W> r;
  r.c8 = 8 * ((lane & 7) ^ (4 * (wave & 1) + (lane >> 4)));
#pragma unroll
  for (int q = 0; q < T / (8 * W); ++q) {
    const int xr = 8 * (wave + W * q) + (lane >> 3);
    int gx = tile * T + xr;
    if constexpr (PAIRED) {
      const int j = tile * (T / 2) + (xr & (T / 2 - 1));
      gx = j / pair * 2 * pair + j % pair + (xr >= T / 2 ? pair : 0);
    }
    r.row[q] = op.src.row(min(gx, op.rows - 1));
  }
  return r;
}

// The source addresses of the wave's copies of a stage are formed ahead of the
// barrier that frees the stage's slot, under the products; the copies then go
// out between the products that follow the barrier.
template <int C>
struct StageSrc {
  const uint16_t* g[C];
};
template <int T, int W>
__device__ __forceinline__ StageSrc<T / (8 * W)> tile_src_kc(const RowPtrs<T, W>& rows, int k0, int K) {
  StageSrc<T / (8 * W)> r;
  const int k = k0 + rows.c8;
#pragma unroll
  for (int q = 0; q < T / (8 * W); ++q) r.g[q] = k < K ? rows.row[q] + k : zeros();
  return r;
}

// MN stage: an instruction moves 512 / T k-rows of T columns; a lane's offset
// in its stage is the same for every copy up to a uniform stride, as in
// copy2_mn (the swizzle depends on k-row bits that the copies do not change).
template <int T>
__device__ __forceinline__ uint32_t tile_lane_off(const Operand& op, int x0, int wave, int lane) {
  constexpr int LPR = T / 8, RPI = 64 / LPR;      // lanes per k-row, k-rows per instruction
  const int kr = RPI * wave + lane / LPR;
  return static_cast<uint32_t>(kr * op.src.ld + min(x0 + ((lane % LPR) ^ mn_swz<T>(kr)) * 8, op.rows - 8));
}
// First row of the stage at hand of a kRunRows operand: stages are taken in
// order, so it moves 64 rows on within a slot, and a slot's first row is mapped
// when the walk enters it.  The form for any slots, whose lanes map their own
// rows on every stage, spends more on that than on the products: M 768 N 4096 K
// 8192 on 128-row tiles 124 us, this walk 94; M 1024 N 512 K 4096 on 64-row tiles
// 42 and 28 (23 where no rows are gathered).
struct RunWalk {
  const uint16_t* base = nullptr;
  int left = 0;                // stages of the slot after the one at hand
  __device__ __forceinline__ void next(const RowSrc& src, int k0, int K) {
    if (--left >= 0) {
      base += static_cast<int64_t>(BK2) * src.ld;
      return;
    }
    k0 = min(k0, K - 1);       // stages past K copy zeros
    base = mapped_row(src, k0);
    left = (src.t == 1 ? K - k0 - 1 : src.s_sp - k0 % src.s_sp - 1) / BK2;
  }
};
template <int T, int W, int MAP>
__device__ __forceinline__ StageSrc<T / (8 * W)> tile_src_mn(const Operand& op, uint32_t off, RunWalk& run, int x0,
                                                             int k0, int K, int wave, int lane) {
  constexpr int LPR = T / 8, RPI = 64 / LPR, C = T / (8 * W);
  StageSrc<C> r;
  if constexpr (MAP == kRunRows) run.next(op.src, k0, K);
  if (MAP != kAnyRows || op.src.t == 1 || op.src.s_sp % BK2 == 0) {   // uniform: the stage is one run of rows (see copy2_mn)
    const uint16_t* base0 = (MAP == kRunRows   ? run.base
                             : MAP == kAnyRows ? mapped_row(op.src, min(k0, K - 1))
                                               : op.src.own + static_cast<int64_t>(k0) * op.src.ld) + off;
#pragma unroll
    for (int q = 0; q < C; ++q) {
      const uint16_t* g = base0 + static_cast<int64_t>(W * RPI * q) * op.src.ld;
      r.g[q] = k0 + RPI * (wave + W * q) + lane / LPR < K ? g : zeros();
    }
    return r;
  }
  const StageRows sr = stage_rows(op.src, k0);
#pragma unroll
  for (int q = 0; q < C; ++q) {
    const int kr = RPI * (wave + W * q) + lane / LPR;
    const int x = min(x0 + ((lane % LPR) ^ mn_swz<T>(kr)) * 8, op.rows - 8);
    r.g[q] = k0 + kr < K ? sr.row(op.src, kr) + x : zeros();
  }
  return r;
}

template <Layout LA, Layout LB, EpiKind KIND, int T, int W, int S, int MAP, bool STREAM>
__global__ void __launch_bounds__(W * 64) gemm_tile(GemmParams p) {
  constexpr int OPB = T * BK2 * 2, STB = 2 * OPB;   // bytes per operand and per stage
  constexpr int R = T / 64;                         // 32-row blocks per wave and operand
  constexpr int C = T / (8 * W), PER = 2 * C;       // copies per wave, per operand and per stage
  constexpr int KS = 2, NSUB = BK2 / 16 / (W / 4) / KS;   // a wave's share of a stage: NSUB sub-steps of KS 16-k products
  constexpr int NACC = T == 64 ? 2 : 1;             // T = 64: two chains, so that no product waits for the one before it
  constexpr bool PAIRED = KIND == EpiKind::QkvRope || KIND == EpiKind::SwiGLUFwd;
  static_assert(S * STB >= T * T * 4, "the tile is staged in the ring");
  __shared__ __attribute__((aligned(16))) uint8_t ring[S * STB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;

  const int parts = p.k_splits > 1 ? p.k_splits : 1;
  const int tiles_m = (p.M + T - 1) / T, tiles_n = (p.N + T - 1) / T, tiles = tiles_m * tiles_n;
  const int pid_all = xcd_remap(blockIdx.x, gridDim.x);
  const int part = pid_all / tiles, pid = pid_all - part * tiles;
  constexpr int GM = GROUP_M * BM / T;              // the same rows of C per group as the 256-row kernel
  const int first_m = pid / (GM * tiles_n) * GM, gm = min(tiles_m - first_m, GM);
  const int tm = first_m + pid % (GM * tiles_n) % gm, tn = pid % (GM * tiles_n) / gm;
  const int pair = PAIRED ? p.pair : T / 2;

  const int all_st = (p.K + BK2 - 1) / BK2;
  const int per_part = (all_st + parts - 1) / parts;
  const int st0 = part * per_part, n = min(per_part, all_st - st0);   // the last part may be shorter (or empty)

  RowPtrs<T, W> ra{}, rb{};
  uint32_t oa = 0, ob = 0;
  if constexpr (LA == Layout::KC) ra = tile_rows<T, W, false>(p.A, tm, pair, wave, lane);
  else oa = tile_lane_off<T>(p.A, tm * T, wave, lane);
  if constexpr (LB == Layout::KC) rb = tile_rows<T, W, PAIRED>(p.B, tn, pair, wave, lane);
  else ob = tile_lane_off<T>(p.B, tn * T, wave, lane);
  const uint32_t ring_addr = lds_addr(ring) + wave * 1024;
  StageSrc<C> ga, gb;
  RunWalk run_a, run_b;
  auto prepare = [&](int st) __attribute__((always_inline)) {
    const int k0 = (st0 + st) * BK2;
    if constexpr (LA == Layout::KC) ga = tile_src_kc<T, W>(ra, k0, p.K);
    else ga = tile_src_mn<T, W, MAP>(p.A, oa, run_a, tm * T, k0, p.K, wave, lane);
    if constexpr (LB == Layout::KC) gb = tile_src_kc<T, W>(rb, k0, p.K);
    else gb = tile_src_mn<T, W, MAP>(p.B, ob, run_b, tn * T, k0, p.K, wave, lane);
  };
  auto fire = [&](int c, int slot) __attribute__((always_inline)) {   // copy c of the prepared stage
    dma16(c < C ? ga.g[c % C] : gb.g[c % C], ring_addr + slot * STB + (c < C ? 0 : OPB) + c % C * (W * 1024));
  };

  f32x16 acc[NACC][R][R];
#pragma unroll
  for (int c = 0; c < NACC; ++c)
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j) acc[c][i][j] = f32x16{};

  struct Frags {
    bf16x8 a[KS][R], b[KS][R];
  };
  auto read = [&](Frags& f, int slot, int sub) __attribute__((always_inline)) {
    const uint8_t* la = ring + slot * STB;
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i) {
        f.a[q][i] = frag<LA, T>(la, wm * (T / 2) + 32 * i, (kg * NSUB + sub) * KS + q, lane);
        f.b[q][i] = frag<LB, T>(la + OPB, wn * (T / 2) + 32 * i, (kg * NSUB + sub) * KS + q, lane);
      }
  };
  // The products of one sub-step, the LDS reads of the next one going out between the first of them.
  auto products = [&](const Frags& f) __attribute__((always_inline)) {
    constexpr int NM = KS * R * R;
    constexpr int DS = KS * R * ((LA == Layout::KC ? 1 : 2) + (LB == Layout::KC ? 1 : 2));
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int q = m / (R * R), i = m / R % R, j = m % R;
      acc[q % NACC][i][j] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[q][i], f.b[q][j], acc[q % NACC][i][j], 0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (m < NM / 2) __builtin_amdgcn_sched_group_barrier(0x100, DS * 2 / NM, 0);
    }
  };
  // Stages past the last one are copied too (their k is past the part's end or
  // past K, and nothing uses them), so that the number in flight is fixed.
#pragma unroll
  for (int st = 0; st < S; ++st) {
    prepare(st);
#pragma unroll
    for (int c = 0; c < PER; ++c) fire(c, st);
  }
  wait_copies<(S - 1) * PER>();
  stage_barrier();
  Frags f0, f1;
  read(f0, 0, 0);
  int slot = 0;
  // Ends stage st: publishes the next stage and starts reading it into nxt, runs
  // the products of cur (the stage's last sub-step), and refills the freed slot.
  auto turn = [&](int st, const Frags& cur, Frags& nxt) __attribute__((always_inline)) {
    wait_copies<(S - 2) * PER>();
    stage_barrier();                    // stage st + 1 is visible, and every wave has read all of stage st
    const int next = slot + 1 == S ? 0 : slot + 1;
    read(nxt, next, 0);
    products(cur);
#pragma unroll
    for (int c = 0; c < PER; ++c) fire(c, slot);
    slot = next;
  };
  if constexpr (NSUB == 2) {
    for (int st = 0; st < n; ++st) {
      prepare(st + S);
      read(f1, slot, 1);
      products(f0);
      turn(st, f1, f0);
    }
  } else {
    int st = 0;
    for (; st + 2 <= n; st += 2) {
      prepare(st + S);
      turn(st, f0, f1);
      prepare(st + 1 + S);
      turn(st + 1, f1, f0);
    }
    if (st < n) {
      prepare(st + S);
      turn(st, f0, f1);
    }
  }
  wait_copies<0>();   // no copy may land in the ring once it is staging space

  // Epilogue: the tile goes through LDS (columns of rows with bit 2 set moved by
  // 32, so that the two half-waves write different banks), then every thread
  // takes 8-column vectors of the low half with their partners.
  constexpr int VPR = T / 16, ITERS = T * VPR / (W * 64) > 0 ? T * VPR / (W * 64) : 1;
  const bool has_vec = T * VPR >= W * 64 || tid < T * VPR;
  float* stg = reinterpret_cast<float*>(ring);
  constexpr bool kSplit = KIND == EpiKind::AccF32 || KIND == EpiKind::StoreBF16;
  const bool to_partial = kSplit && (KIND == EpiKind::AccF32 ? part > 0 : parts > 1);
  auto column = [&](int v) {
    const int j = tn * (T / 2) + 8 * v;
    return PAIRED ? j / pair * 2 * pair + j % pair : tn * T + 8 * v;
  };
  EpiIn<KIND> in[ITERS];
  if (!to_partial && has_vec) {
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int idx = it * (W * 64) + tid;
      epi_load<KIND, STREAM>(p, tm * T + idx / VPR, column(idx % VPR), pair, in[it]);
    }
  }
  __syncthreads();    // every wave is done reading the ring
  auto stage_acc = [&](bool add) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = wm * (T / 2) + 32 * i + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
          const int c = wn * (T / 2) + 32 * j + (lane & 31);
          float* d = stg + r * T + (c ^ (((r >> 2) & 1) << 5));
          float v = acc[0][i][j][e];
          if constexpr (NACC == 2) v += acc[1][i][j][e];
          *d = add ? *d + v : v;
        }
  };
  if (kg == 0) stage_acc(false);
  __syncthreads();
  if constexpr (W == 8) {             // the second k group adds its sums
    if (kg == 1) stage_acc(true);
    __syncthreads();
  }
  if (!has_vec) return;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int idx = it * (W * 64) + tid;
    const int r = idx / VPR, v = idx % VPR;
    const int64_t m = static_cast<int64_t>(tm) * T + r;
    const int flip = ((r >> 2) & 1) << 5;
    const float4* lo4 = reinterpret_cast<const float4*>(stg + r * T + ((8 * v) ^ flip));
    const float4* hi4 = reinterpret_cast<const float4*>(stg + r * T + ((T / 2 + 8 * v) ^ flip));
    const float4 l0 = lo4[0], l1 = lo4[1], h0 = hi4[0], h1 = hi4[1];
    if (to_partial) {
      if (m >= p.M) continue;
      float* c = p.partial + (static_cast<int64_t>(KIND == EpiKind::AccF32 ? part - 1 : part) * p.M + m) * p.N;
      const int nlo = column(v), nhi = nlo + pair;
      if (nlo < p.N) {
        reinterpret_cast<float4*>(c + nlo)[0] = l0;
        reinterpret_cast<float4*>(c + nlo)[1] = l1;
      }
      if (nhi < p.N) {
        reinterpret_cast<float4*>(c + nhi)[0] = h0;
        reinterpret_cast<float4*>(c + nhi)[1] = h1;
      }
      continue;
    }
    float lo[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
    float hi[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
    epilogue<KIND, STREAM>(p, m, column(v), pair, lo, hi, in[it]);
  }
}

template <Layout LA, Layout LB, EpiKind KIND, int T, int W, int S, int MAP>
hipError_t launch_tile(const GemmParams& p, hipStream_t stream) {
  const int parts = p.k_splits > 1 ? p.k_splits : 1;
  const dim3 grid(static_cast<unsigned>((p.M + T - 1) / T) * ((p.N + T - 1) / T) * parts);
  if (KIND == EpiKind::AccF32 && p.stream_c)
    hipLaunchKernelGGL((gemm_tile<LA, LB, KIND, T, W, S, MAP, KIND == EpiKind::AccF32>), grid, dim3(W * 64), 0, stream, p);
  else
    hipLaunchKernelGGL((gemm_tile<LA, LB, KIND, T, W, S, MAP, false>), grid, dim3(W * 64), 0, stream, p);
  return hipGetLastError();
}

// Tile size and split: see gemm_plan.
template <Layout LA, Layout LB, EpiKind KIND, int MAP>
hipError_t launch_small(const GemmParams& p, hipStream_t stream) {
  const int T = p.tile, parts = p.k_splits > 1 ? p.k_splits : 1;
  const int64_t blocks = static_cast<int64_t>((p.M + T - 1) / T) * ((p.N + T - 1) / T) * parts;
  if (T == 128)
    return blocks <= 256 ? launch_tile<LA, LB, KIND, 128, 8, 4, MAP>(p, stream)
                         : launch_tile<LA, LB, KIND, 128, 4, 2, MAP>(p, stream);
  return blocks <= 256 ? launch_tile<LA, LB, KIND, 64, 8, 8, MAP>(p, stream)
                       : launch_tile<LA, LB, KIND, 64, 4, 4, MAP>(p, stream);
}
template <Layout LA, Layout LB, EpiKind KIND, int PAIR, int MAP>
hipError_t launch256(const GemmParams& p, hipStream_t stream) {
  const int parts = p.k_splits > 1 ? p.k_splits : 1;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tiles_n = p.B.split_rows ? (p.B.split_rows + 127) / 128 : (p.N + BN - 1) / BN;
  if (parts > 1 && p.K % (2 * BK2 * parts) != 0) return hipErrorInvalidValue;
  // the fp32 accumulate's whole-tile epilogue addresses 128 rows of C with 32-bit byte offsets
  if (KIND == EpiKind::AccF32 && p.epi.ldc > (int64_t{1} << 21)) return hipErrorInvalidValue;
  const dim3 grid(tiles_m * tiles_n * parts);
  if (p.K % (2 * BK2) == 0)
    hipLaunchKernelGGL((gemm_bk64<LA, LB, KIND, PAIR, false, MAP>), grid, dim3(512), 0, stream, p);
  else
    hipLaunchKernelGGL((gemm_bk64<LA, LB, KIND, PAIR, true, MAP>), grid, dim3(512), 0, stream, p);
  return hipGetLastError();
}
template <Layout LA, Layout LB, EpiKind KIND, int PAIR>
hipError_t launch(const GemmParams& p, hipStream_t stream) {
  if (p.k_splits > 1 && ((KIND != EpiKind::AccF32 && KIND != EpiKind::StoreBF16) || !p.partial))
    return hipErrorInvalidValue;
  const RowSrc &a = p.A.src, &b = p.B.src;
  const bool plain = (LA == Layout::KC || a.t == 1) && (LB == Layout::KC || b.t == 1);
  const bool small = p.tile == 128 || p.tile == 64;
  if constexpr (LA == Layout::MN) {            // the weight gradients: gathered activations as MN operands
    const bool runs = (a.t == 1 || a.s_sp % BK2 == 0) && (b.t == 1 || b.s_sp % BK2 == 0);
    if (small)
      return plain  ? launch_small<LA, LB, KIND, kPlainRows>(p, stream)
             : runs ? launch_small<LA, LB, KIND, kRunRows>(p, stream)
                    : launch_small<LA, LB, KIND, kAnyRows>(p, stream);
    return plain  ? launch256<LA, LB, KIND, PAIR, kPlainRows>(p, stream)
           : runs ? launch256<LA, LB, KIND, PAIR, kRunRows>(p, stream)
                  : launch256<LA, LB, KIND, PAIR, kAnyRows>(p, stream);
  }
  if (!plain) return hipErrorInvalidValue;     // every other MN operand is a weight
  // kRunRows maps a plain array too; on the dX GEMMs of full chips its main loop
  // measured 1-2% faster than the shorter one of kPlainRows (7B gate|up 547 against
  // 555 us, QKV 310 / 316; 70B TP8 gate|up 756 / 771)
  return small ? launch_small<LA, LB, KIND, kPlainRows>(p, stream) : launch256<LA, LB, KIND, PAIR, kRunRows>(p, stream);
}

}  // namespace

hipError_t gemm(const GemmParams& params, Layout la, Layout lb, hipStream_t stream) {
  if (params.M <= 0 || params.N <= 0 || params.K <= 0) return hipSuccess;
  using L = Layout;
  using E = EpiKind;
  const E k = params.epi.kind;
  GemmParams p = params;
  p.pair = k == E::QkvRope ? p.epi.d_h / 2 : k == E::SwiGLUFwd ? p.epi.f : 0;
  if (la == L::KC && lb == L::KC) {
    if (k == E::QkvRope && p.epi.d_h == 128) return launch<L::KC, L::KC, E::QkvRope, 64>(p, stream);
    if (k == E::QkvRope && p.epi.d_h == 64) return launch<L::KC, L::KC, E::QkvRope, 32>(p, stream);
    if (k == E::ResidualSP) return launch<L::KC, L::KC, E::ResidualSP, 128>(p, stream);
    if (k == E::SwiGLUFwd) return launch<L::KC, L::KC, E::SwiGLUFwd, 128>(p, stream);
    if (k == E::StoreBF16) return launch<L::KC, L::KC, E::StoreBF16, 128>(p, stream);
    if (k == E::StoreF32) return launch<L::KC, L::KC, E::StoreF32, 128>(p, stream);
  } else if (la == L::KC && lb == L::MN) {
    if (k == E::SwiGLUBwd) return launch<L::KC, L::MN, E::SwiGLUBwd, 128>(p, stream);
    if (k == E::ResidualSP) return launch<L::KC, L::MN, E::ResidualSP, 128>(p, stream);
    if (k == E::StoreBF16) return launch<L::KC, L::MN, E::StoreBF16, 128>(p, stream);
  } else if (la == L::MN && lb == L::MN) {
    if (k == E::AccF32) return launch<L::MN, L::MN, E::AccF32, 128>(p, stream);
  }
  return hipErrorInvalidValue;     // a layout / epilogue pairing the layer never uses
}

namespace {
// C += partial[0] + partial[1] + ..., four floats per thread (N % 4 == 0 and
// ldc % 4 == 0 are required by the caller; C may start at any float).
__global__ void __launch_bounds__(256) split_reduce_kernel(float* __restrict__ c, int64_t ldc,
                                                          const float* __restrict__ part, int64_t M, int64_t N,
                                                          int32_t n_part) {
  const int64_t n4 = N / 4;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= M * n4) return;
  const int64_t m = i / n4, j = (i - m * n4) * 4;
  f32x4_a4* cp = reinterpret_cast<f32x4_a4*>(c + m * ldc + j);
  f32x4 v = *cp;
  for (int s = 0; s < n_part; ++s) v += *reinterpret_cast<const f32x4*>(part + static_cast<int64_t>(s) * M * N + m * N + j);
  *cp = v;
}
// C (bf16) = partial[0] + partial[1] + ..., four columns per thread.
__global__ void __launch_bounds__(256) split_store_kernel(uint16_t* __restrict__ c, int64_t ldc,
                                                         const float* __restrict__ part, int64_t M, int64_t N,
                                                         int32_t n_part) {
  const int64_t n4 = N / 4;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= M * n4) return;
  const int64_t m = i / n4, j = (i - m * n4) * 4;
  float4 v = *reinterpret_cast<const float4*>(part + m * N + j);
  for (int s = 1; s < n_part; ++s) {
    const float4 q = *reinterpret_cast<const float4*>(part + static_cast<int64_t>(s) * M * N + m * N + j);
    v.x += q.x;
    v.y += q.y;
    v.z += q.z;
    v.w += q.w;
  }
  uint16_t* o = c + m * ldc + j;
  o[0] = f2bf(v.x);
  o[1] = f2bf(v.y);
  o[2] = f2bf(v.z);
  o[3] = f2bf(v.w);
}
}  // namespace

hipError_t gemm_split_store(uint16_t* c, int64_t ldc, const float* partial, int64_t M, int64_t N, int32_t splits,
                            hipStream_t stream) {
  if (splits < 1 || M <= 0 || N <= 0) return hipSuccess;
  const int64_t n = M * (N / 4);
  hipLaunchKernelGGL(split_store_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, c, ldc,
                     partial, M, N, splits);
  return hipGetLastError();
}

int gemm_max_splits(int64_t M, int64_t N, int64_t K, bool acc_f32) {
  // Model: a wave of 256 tiles of full K takes T = 2*256*256*K / (1 PFLOP/s / 256 CUs);
  // s parts take ceil(tiles*s / 256) waves of T/s, plus writing and reading the
  // fp32 partials at about 4 TB/s (s - 1 of them when part 0 accumulates into an
  // fp32 C, all s when the result is stored as bf16).  Pick the cheapest s of 1..4.
  const int64_t tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const double t_wave = 2.0 * BM * BN * static_cast<double>(K) / (1e15 / 256.0);
  int best = 1;
  double best_t = 1e30;
  for (int s = 1; s <= 4; ++s) {
    if (K % (2 * BK2 * s) != 0 || N % 4 != 0) continue;
    const double waves = static_cast<double>((tiles * s + 255) / 256);
    const int n_part = s == 1 ? 0 : (acc_f32 ? s - 1 : s);
    const double t = waves * t_wave / s + n_part * 2.0 * 4.0 * static_cast<double>(M) * N / 4e12;
    if (t < best_t * 0.97) {       // a split has to win by a margin
      best_t = t;
      best = s;
    }
  }
  return best;
}

namespace {
// What a grid of T-row tiles costs on a kernel that keeps `slots` workgroups on
// the chip: per round of workgroups a fixed part (launch or drain, first copies),
// the tiles' C traffic at c_tbs TB/s and c0 + c1 fill us per stage of 64 k, where fill is
// the part of the slots in use (an emptier chip clocks higher and waits less for
// memory); m_edge and n_edge once per grid whose last tiles are cut in M, in N.
struct GridCost {
  int T, slots;
  double fixed, c_tbs, c0, c1, m_edge = 0.0, n_edge = 0.0;
};
double grid_us(const GridCost& g, int64_t tiles, int64_t st, double c_bytes) {
  const double c_us = static_cast<double>(g.slots) * g.T * g.T * c_bytes / (g.c_tbs * 1e6);
  const auto round = [&](double fill) { return g.fixed + fill * c_us + st * (g.c0 + g.c1 * fill); };
  const int64_t full = tiles / g.slots, rest = tiles % g.slots;
  return full * round(1.0) + (rest ? round(static_cast<double>(rest) / g.slots) : 0.0);
}
// 256-row tiles, 128 one and two workgroups per CU, 64 one and two per CU.
//
// Forward and dX (a K-contiguous operand): fits to GEMMs of 128 to 8192 rows, 256
// to 32064 columns and K 128 to 32000 timed in every form on one MI355X, within
// about 15% of the times, the traffic of C at 8 bytes an element: e.g. M 2048 N
// 2048 K 5464 K-contiguous 125 us with 64 tiles of 256 rows, 60 with 256 of 128; M
// 600 N 1280 K 8192 143 / 52 / 27 us with tiles of 256 / 128 / 64; M 4000 N 7168
// K 4096 210 / 249 / 402; M 512 N 4096 K 32000 605 in one part and 317 in two with
// 256-row tiles, 274 and 161 with 128-row ones.
constexpr GridCost kForward[5] = {{256, 256, 8.0, 4.8, 1.0, 0.65},
                                  {128, 256, 5.0, 4.8, 0.33, 0.27},
                                  {128, 512, 5.0, 4.8, 0.25, 0.85},
                                  {64, 256, 4.0, 4.8, 0.15, 0.06},
                                  {64, 512, 4.0, 4.8, 0.20, 0.32}};
// Weight gradients of a layer (both operands transposed, C read and written):
// fits to 393 of them, hidden 256 to 8192 and K 512 to 16384, each timed in 9 forms (rms error
// 7 to 16% over the forms within 1.6 times the best).  The form picked takes 0.5% more
// than the best one on average (at worst 27%: M 2752 N 4096 K 512, 46 us against
// 36); with the constants above it took 2.7%, at worst 57% (M 4096 N 2752 K 1024: 82
// us on 256-row tiles, whose cut tiles add C element by element, 52 on 128-row
// ones; M 1024 N 1024 K 16384: 87 us unsplit on 64-row tiles, 59 in 4 parts on
// 128-row ones).
constexpr GridCost kWeightGrad[5] = {{256, 256, 12.6, 8.9, 1.20, 0.40, 7.0, 23.0},
                                     {128, 256, 9.8, 7.0, 0.43, 0.18},
                                     {128, 512, 11.6, 28.0, 0.73, 0.35},
                                     {64, 256, 8.3, 1e3, 0.24, 0.06},
                                     {64, 512, 5.9, 1e3, 0.34, 0.14}};
// A layer's weight gradient of this size is streamed past the caches on small
// tiles too, as the 256-row kernel does with all of them: left there it displaces
// the operands of the kernels that follow (a layer of hidden 2048, FFN 5464 on
// 1000 tokens 677 us, streamed 630; hidden 4096, FFN 11008 on TP 4, 1024 tokens 637
// and 602), while smaller ones are found there by the next call (hidden 1024 on
// 1000 tokens 302, streamed 307).  The head's weight gradient is the last product
// of its call: whether streaming it pays depends on what the caller does next, and
// timed in a row 64 tokens of a 16032-wide shard take 121 us streamed and 86 not,
// of a 32064-wide one 268 and 327 (hidden 2048).  It stays as it was: 256-row tiles
// (streamed) or, where kForward prefers them, smaller ones (not).
constexpr int64_t kStreamBytes = 32 << 20;
}  // namespace

GemmPlan gemm_plan(int64_t M, int64_t N, int64_t K, EpiKind kind, int max_splits, bool layer) {
  const bool acc = kind == EpiKind::AccF32, layer_dw = layer && acc;
  const GridCost* cost = layer_dw ? kWeightGrad : kForward;
  const int64_t stages = (K + BK2 - 1) / BK2;
  const double mn = static_cast<double>(M) * N;
  GemmPlan best{256, 1, layer_dw && static_cast<int64_t>(4 * mn) >= kStreamBytes};
  double best_us = 1e30;
  for (int s = 1; s <= max_splits; ++s) {
    if (s > 1 && (N % 4 != 0 || stages < 4 * s)) break;
    const int n_part = s == 1 ? 0 : (acc ? s - 1 : s);
    const int64_t st = (stages + s - 1) / s;
    for (int f = 0; f < 5; ++f) {
      const GridCost& g = cost[f];
      const int64_t tiles = (M + g.T - 1) / g.T * ((N + g.T - 1) / g.T) * s;
      if (g.T == 256 && s > 1 && K % (2 * BK2 * s) != 0) continue;     // that kernel takes equal, even parts
      if (g.T != 256 && (tiles <= 256) != (g.slots == 256)) continue;  // see launch_small
      // Parts store 4 bytes an element, but for part 0 of an accumulate, which reads
      // and writes C.  The reduce pass reads the partials and writes C (an
      // accumulate reads it too), 5.7 us and 6.9 TB/s over 5 to 55 us.  The price of
      // other parts (dX on small tiles, the head's d_hidden, whose workspace would
      // grow with more of them) stands for their stores as well.
      double c_bytes = 8.0, reduce = 0.0;
      if (s > 1 && (layer_dw || (layer && g.T == 256))) {
        reduce = 5.7 + (4.0 * n_part + (acc ? 8.0 : 2.0)) * mn / 6.9e6;
        c_bytes = acc ? (8.0 + 4.0 * n_part) / s : 4.0;
      } else if (s > 1) {
        reduce = 4.0 + n_part * 8.0 * mn / 4e6;
      }
      const double us = reduce + grid_us(g, tiles, g.T == 256 ? (st + 1) / 2 * 2 : st, c_bytes) +
                        (M % g.T ? g.m_edge : 0.0) + (N % g.T ? g.n_edge : 0.0);
      if (us < 0.97 * best_us) {       // a split or a smaller tile has to win by a margin
        best.tile = g.T;
        best.splits = s;
        best_us = us;
      }
    }
  }
  return best;
}

hipError_t gemm_split_reduce(float* c, int64_t ldc, const float* partial, int64_t M, int64_t N, int32_t splits,
                             hipStream_t stream) {
  if (splits <= 1 || M <= 0 || N <= 0) return hipSuccess;
  const int64_t n = M * (N / 4);
  hipLaunchKernelGGL(split_reduce_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, c, ldc,
                     partial, M, N, splits - 1);
  return hipGetLastError();
}

}  // namespace l4d
