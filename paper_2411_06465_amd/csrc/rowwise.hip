// Memory-bound row kernels: RMSNorm forward/backward, the gain-gradient
// reduction, the RoPE angle table, the vocabulary-parallel cross-entropy (bf16
// logits, or FP32 logits kept as the softmax) and the vocabulary-parallel
// embedding lookup and its gradient.
// One wave (64 lanes) owns one row; every global access is a 16-byte vector.
#include <math.h>

#include "kernels.h"

namespace l4d {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ void unpack8(u32x4 u, float* v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(u[i] << 16);
    v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ u32x4 pack8(const float* v) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[2 * i], v[2 * i + 1]}, bf16x2));
  return r;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

constexpr int kMaxChunks = 16;   // h <= 64 lanes * 16 chunks * 8 = 8192

// ------------------------------------------------------------------ RoPE table

// Entry idx of the cos/sin table.  The table has no launch of its own: its
// entries are extra blocks of a kernel that runs ahead of the first reader anyway
// (the first norm in the forward, the second norm's gain sum in the backward).
// That saves the launch (6 to 7 us timed alone) but not all of the
// double-precision work: the first norm takes 0.8 us longer on 2000 tokens (8B TP4),
// 2.7 on 4096 of head size 128 (7B), 4.8 to 6.8 on the 8B and 70B shards.
__device__ __forceinline__ void rope_entry(const RopeTable& r, int64_t idx) {
  const int half = r.d_h / 2;
  if (idx >= static_cast<int64_t>(r.rows) * half) return;
  const int i = static_cast<int>(idx / half), j = static_cast<int>(idx % half);
  const int ci = i / r.map.chunk_len;
  const int64_t pos = static_cast<int64_t>(r.map.chunk_id[ci]) * r.map.chunk_len + (i - ci * r.map.chunk_len);
  const double ang = static_cast<double>(pos) * exp(-2.0 * j / r.d_h * r.log_base);
  double s, c;
  sincos(ang, &s, &c);
  r.tab[idx] = make_float2(static_cast<float>(c), static_cast<float>(s));
}
unsigned rope_blocks(const RopeTable* r, int threads) {
  return r ? static_cast<unsigned>((static_cast<int64_t>(r->rows) * (r->d_h / 2) + threads - 1) / threads) : 0u;
}

// ------------------------------------------------------------------ RMSNorm

// One wave per row.  All of the row's loads are issued before the first use,
// so that a wave keeps its whole row (8 KB at h = 4096) in flight: a use right
// after each load waits for it and leaves one kilobyte in flight per wave.
// CPT > 0: h = 512 CPT (every lane holds CPT chunks, no bounds); CPT = 0: any
// h that is a multiple of 8.  ROPE: the first rope_blk blocks fill the RoPE table.
template <int CPT, bool ROPE>
__global__ void __launch_bounds__(256) rmsnorm_fwd_kernel(const uint16_t* __restrict__ x,
                                                          const uint16_t* __restrict__ gain,
                                                          uint16_t* __restrict__ y, uint16_t* __restrict__ x_copy,
                                                          int64_t rows, int32_t h, float eps, RopeTable rope,
                                                          int32_t rope_blk) {
  constexpr int NC = CPT > 0 ? CPT : kMaxChunks;
  const int lane = threadIdx.x & 63;
  int64_t block = blockIdx.x;
  if constexpr (ROPE) {
    if (block < rope_blk) {
      rope_entry(rope, block * 256 + threadIdx.x);
      return;
    }
    block -= rope_blk;
  }
  const int64_t row = block * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int nch = CPT > 0 ? 64 * CPT : h / 8;
  const u32x4* xr = reinterpret_cast<const u32x4*>(x + row * h);
  const u32x4* gr = reinterpret_cast<const u32x4*>(gain);
  u32x4 v[NC], gv[NC];
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int c = lane + 64 * it;
    if (CPT > 0 || c < nch) v[it] = __builtin_nontemporal_load(&xr[c]);     // read once
  }
  // the gain too, before any store: a load issued after a store waits for it
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int c = lane + 64 * it;
    if (CPT > 0 || c < nch) gv[it] = gr[c];
  }
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int c = lane + 64 * it;
    if (CPT > 0 || c < nch) {
      float f[8];
      unpack8(v[it], f);
#pragma unroll
      for (int j = 0; j < 8; ++j) ss += f[j] * f[j];
    }
  }
  if (x_copy) {     // the input, kept for the backward
    u32x4* cr = reinterpret_cast<u32x4*>(x_copy + row * h);
#pragma unroll
    for (int it = 0; it < NC; ++it) {
      const int c = lane + 64 * it;
      if (CPT > 0 || c < nch) cr[c] = v[it];
    }
  }
  const float rstd = rsqrtf(wave_sum(ss) / h + eps);
  u32x4* yr = reinterpret_cast<u32x4*>(y + row * h);
#pragma unroll
  for (int it = 0; it < NC; ++it) {
    const int c = lane + 64 * it;
    if (CPT > 0 || c < nch) {
      float f[8], g[8];
      unpack8(v[it], f);
      unpack8(gv[it], g);
#pragma unroll
      for (int j = 0; j < 8; ++j) f[j] = f[j] * rstd * g[j];
      yr[c] = pack8(f);
    }
  }
}

// Eight consecutive values of a bf16 row (one 16-byte load) or an fp32 row (two).
template <bool F32>
struct Vec8 {
  u32x4 v;
};
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <>
struct Vec8<true> {
  f32x4 a, b;
};
template <bool F32>
__device__ __forceinline__ Vec8<F32> load8(const void* row, int c) {      // read-once rows: non-temporal
  if constexpr (F32) {
    const f32x4* p = reinterpret_cast<const f32x4*>(row) + 2 * c;
    return Vec8<true>{__builtin_nontemporal_load(p), __builtin_nontemporal_load(p + 1)};
  } else {
    return Vec8<false>{__builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row) + c)};
  }
}
template <bool F32>
__device__ __forceinline__ void unpack(const Vec8<F32>& u, float* v) {
  if constexpr (F32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = u.a[i];
      v[4 + i] = u.b[i];
    }
  } else {
    unpack8(u.v, v);
  }
}

// Grid-stride over rows, one 256-thread block per row: thread t owns the
// 8-column chunks t + 256 it (it < CPT, h <= 2048 * CPT) of every row, so it
// keeps its columns' partial sums of dy*xhat in registers and writes them to
// partial[blockIdx.x][h] at the end.  The two row sums go through LDS,
// double-buffered by row parity so one barrier per row suffices.
// DY32: the incoming gradient d(out) is fp32 (else bf16); RES: the residual
// gradient added to the result is absent (0), bf16 (1) or fp32 (2); OUT32:
// the result is also stored in fp32.
template <int CPT, bool DY32, int RES, bool OUT32>
__global__ void __launch_bounds__(256) rmsnorm_bwd_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ gain, const void* __restrict__ dy,
    const void* __restrict__ dres, uint16_t* __restrict__ dx, float* __restrict__ dx32, float* __restrict__ partial,
    int64_t rows, int32_t h, float eps) {
  constexpr bool R32 = RES == 2;
  __shared__ float sums[2][4][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nch = h / 8;
  float acc[CPT][8];
#pragma unroll
  for (int it = 0; it < CPT; ++it)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[it][j] = 0.f;
  const u32x4* gr = reinterpret_cast<const u32x4*>(gain);
  u32x4 gv[CPT];
  const int64_t dsz = DY32 ? 4 : 2, rsz = R32 ? 4 : 2;
  // row `row`'s x, d(out) and residual gradient into (a, b, r); every lane
  // loads (a lane past the row end reloads the row's last chunk, unused), so
  // the number of loads in flight is fixed and the waits for a row count exactly
  auto load_row = [&](int64_t row, u32x4 (&a)[CPT], Vec8<DY32> (&b)[CPT], Vec8<R32> (&r)[CPT])
                      __attribute__((always_inline)) {
    const u32x4* xr = reinterpret_cast<const u32x4*>(x + row * h);
    const void* dr = static_cast<const uint8_t*>(dy) + row * h * dsz;
    const void* rr = RES ? static_cast<const uint8_t*>(dres) + row * h * rsz : nullptr;
#pragma unroll
    for (int it = 0; it < CPT; ++it) {
      const int c = min(tid + 256 * it, nch - 1);
      a[it] = __builtin_nontemporal_load(&xr[c]);
      b[it] = load8<DY32>(dr, c);
      if constexpr (RES != 0) r[it] = load8<R32>(rr, c);
    }
  };
#pragma unroll
  for (int it = 0; it < CPT; ++it) gv[it] = gr[min(tid + 256 * it, nch - 1)];
  int parity = 0;
  // one row: the two row sums, then dx and the gain partials.  A lane past the
  // row end holds a copy of the last chunk (loads clamped), so it stores the
  // same values to the same place as the chunk's own lane, and no store is
  // conditional; it leaves the row sums and the gain partials alone.
  auto process = [&](int64_t row, const u32x4 (&xv)[CPT], const Vec8<DY32> (&dv)[CPT], const Vec8<R32> (&rv)[CPT])
                     __attribute__((always_inline)) {
    float ss = 0.f, dot = 0.f;
#pragma unroll
    for (int it = 0; it < CPT; ++it) {
      const int c = tid + 256 * it;
      if (c < nch) {
        float f[8], d[8], g[8];
        unpack8(xv[it], f);
        unpack<DY32>(dv[it], d);
        unpack8(gv[it], g);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          ss += f[j] * f[j];
          dot += g[j] * d[j] * f[j];
        }
      }
    }
    ss = wave_sum(ss);
    dot = wave_sum(dot);
    if (lane == 0) {
      sums[parity][wave][0] = ss;
      sums[parity][wave][1] = dot;
    }
    __syncthreads();
    ss = (sums[parity][0][0] + sums[parity][1][0]) + (sums[parity][2][0] + sums[parity][3][0]);
    dot = (sums[parity][0][1] + sums[parity][1][1]) + (sums[parity][2][1] + sums[parity][3][1]);
    parity ^= 1;
    const float rstd = rsqrtf(ss / h + eps);
    const float c_mean = dot * rstd / h;        // mean over the row of (gain*dy) * xhat
    u32x4* out = reinterpret_cast<u32x4*>(dx + row * h);
    float4* out32 = OUT32 ? reinterpret_cast<float4*>(dx32 + row * h) : nullptr;
#pragma unroll
    for (int it = 0; it < CPT; ++it) {
      const int c = min(tid + 256 * it, nch - 1);
      const float own = tid + 256 * it < nch ? 1.f : 0.f;
      float f[8], d[8], g[8], r[8];
      unpack8(xv[it], f);
      unpack<DY32>(dv[it], d);
      unpack8(gv[it], g);
      if constexpr (RES != 0) {
        unpack<R32>(rv[it], r);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) r[j] = 0.f;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float xh = f[j] * rstd;
        acc[it][j] += own * (d[j] * xh);
        r[j] += rstd * (g[j] * d[j] - xh * c_mean);
      }
      out[c] = pack8(r);
      if constexpr (OUT32) {
        out32[2 * c] = make_float4(r[0], r[1], r[2], r[3]);
        out32[2 * c + 1] = make_float4(r[4], r[5], r[6], r[7]);
      }
    }
  };
  const int64_t G = gridDim.x, last = rows - 1;
  if constexpr (CPT <= 2 && DY32 && RES == 2) {
    // The read-heaviest form (10 of its 12 bytes per element are reads) keeps
    // two rows in flight, in three register sets: rows row + G and row + 2G
    // load while row is processed (a load past the last row reloads the last
    // row, unused).  On 268 MB cache-cold tensors: 302 -> 287 us; the lighter
    // forms measured no better.
    u32x4 xa[CPT], xb[CPT], xc[CPT];
    Vec8<DY32> da[CPT], db[CPT], dc[CPT];
    Vec8<R32> ra[CPT], rb[CPT], rc[CPT];
    int64_t row = blockIdx.x;
    if (row < rows) {
      load_row(row, xa, da, ra);
      load_row(min(row + G, last), xb, db, rb);
    }
    for (; row < rows; row += 3 * G) {
      load_row(min(row + 2 * G, last), xc, dc, rc);
      process(row, xa, da, ra);
      if (row + G >= rows) break;
      load_row(min(row + 3 * G, last), xa, da, ra);
      process(row + G, xb, db, rb);
      if (row + 2 * G >= rows) break;
      load_row(min(row + 4 * G, last), xb, db, rb);
      process(row + 2 * G, xc, dc, rc);
    }
  } else {
    u32x4 xv[CPT], xn[CPT];
    Vec8<DY32> dv[CPT], dn[CPT];
    Vec8<R32> rv[CPT], rn[CPT];
    if (static_cast<int64_t>(blockIdx.x) < rows) load_row(blockIdx.x, xn, dn, rn);
    for (int64_t row = blockIdx.x; row < rows; row += G) {
#pragma unroll
      for (int it = 0; it < CPT; ++it) {
        xv[it] = xn[it];
        dv[it] = dn[it];
        if constexpr (RES != 0) rv[it] = rn[it];
      }
      // the next row's loads fly under this row's reductions and stores
      if (row + G < rows) load_row(row + G, xn, dn, rn);
      process(row, xv, dv, rv);
    }
  }
  float* pr = partial + static_cast<int64_t>(blockIdx.x) * h;
#pragma unroll
  for (int it = 0; it < CPT; ++it) {
    const int c = tid + 256 * it;
    if (c < nch) {
      reinterpret_cast<float4*>(pr + c * 8)[0] = make_float4(acc[it][0], acc[it][1], acc[it][2], acc[it][3]);
      reinterpret_cast<float4*>(pr + c * 8)[1] = make_float4(acc[it][4], acc[it][5], acc[it][6], acc[it][7]);
    }
  }
}

// out += the column sums of partial[n][h], n <= 256, in a fixed order (no
// atomics): a block of 16 waves per 64 columns, wave w taking rows w, w + 16, ..,
// all their loads in flight at once, since the kernel's time is the latency of
// its loads (128 rows of 256 columns 4.0 -> 2.0 us, 256 rows of 2048 to 8192
// columns 7 -> 4.7 us against 4 waves with 4 loads in flight each).  ROPE: the
// blocks past the columns fill the RoPE table.
constexpr int kSumWaves = 16, kSumRows = 256 / kSumWaves;
template <bool ROPE>
__global__ void __launch_bounds__(kSumWaves * 64) column_sums_kernel(const float* __restrict__ partial, int32_t n,
                                                                     int32_t h, float* __restrict__ out,
                                                                     RopeTable rope) {
  if constexpr (ROPE) {
    const int col_blk = (h + 63) / 64, blk = static_cast<int>(blockIdx.x) - col_blk;
    if (blk >= 0) {
      rope_entry(rope, static_cast<int64_t>(blk) * (kSumWaves * 64) + threadIdx.x);
      return;
    }
  }
  __shared__ float sums[kSumWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + lane;
  float v[kSumRows];
#pragma unroll
  for (int i = 0; i < kSumRows; ++i) {
    const int r = wave + kSumWaves * i;
    v[i] = r < n && col < h ? partial[static_cast<int64_t>(r) * h + col] : 0.f;
  }
#pragma unroll
  for (int d = kSumRows / 2; d > 0; d /= 2)
#pragma unroll
    for (int i = 0; i < d; ++i) v[i] += v[i + d];
  sums[wave][lane] = v[0];
  __syncthreads();
  if (wave == 0 && col < h) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kSumWaves; ++w) s += sums[w][lane];
    out[col] += s;
  }
}

// ------------------------------------------------------------------ cross-entropy
// One block per token row of logits [n][v_t].  Both passes over a row (its
// log-sum-exp; the softmax or the gradient) need all of it, so a block keeps the
// row in registers where it fits, V 16-byte vectors per thread: the row is read
// once, with all its loads in flight, and the kernel is bound by one read and
// one write of the logits.  A row read twice came from memory twice: the rows of
// the blocks in flight (32 MB per XCD at 32064 fp32 columns) are far more than
// an L2 holds.  4096 fp32 rows of 32064 columns 287 -> 177 us (5.9 TB/s), 8192
// bf16 rows 242 -> 188 us (5.6 TB/s).  Rows past 65536 columns are read twice.

// (max, sum of exponentials relative to it) of every thread -> log of the row's
// whole sum, combined with the other shards' log-sum-exp; stores the row's loss.
// z_at(i): logit i of the row.
template <int WAVES, typename Z>
__device__ __forceinline__ float xent_lse(float mx, float se, int32_t v_t, int64_t v0, int64_t row,
                                          const int64_t* __restrict__ targets, const float* __restrict__ peer_lse,
                                          const float* __restrict__ peer_z, float* __restrict__ loss, Z&& z_at) {
  __shared__ float red_m[WAVES], red_s[WAVES];
  __shared__ float bcast;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // combine (max, sum) pairs across the wave, then the waves
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float m2 = __shfl_xor(mx, o, 64), s2 = __shfl_xor(se, o, 64);
    const float m = fmaxf(mx, m2);
    se = (mx == -INFINITY ? 0.f : se * __expf(mx - m)) + (m2 == -INFINITY ? 0.f : s2 * __expf(m2 - m));
    mx = m;
  }
  if (lane == 0) {
    red_m[wave] = mx;
    red_s[wave] = se;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float m = red_m[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) m = fmaxf(m, red_m[w]);
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) sum += red_m[w] == -INFINITY ? 0.f : red_s[w] * __expf(red_m[w] - m);
    float lse = m + logf(sum);
    if (peer_lse) {
      const float p = peer_lse[row];
      const float hi = fmaxf(lse, p), lo = fminf(lse, p);
      lse = hi + log1pf(__expf(lo - hi));
    }
    const int64_t tgt = targets[row] - v0;
    const float z = tgt >= 0 && tgt < v_t ? z_at(tgt) : peer_z ? peer_z[row] : 0.f;
    loss[row] = lse - z;
    bcast = lse;
  }
  __syncthreads();
  return bcast;
}

// The running (max, sum) of a thread after eight, or four, more values.
template <int N>
__device__ __forceinline__ void xent_add(const float* f, float& mx, float& se) {
  float m = f[0];
#pragma unroll
  for (int j = 1; j < N; ++j) m = fmaxf(m, f[j]);
  if (m > mx) {
    se *= __expf(mx - m);       // 0 while mx is -inf
    mx = m;
  }
#pragma unroll
  for (int j = 0; j < N; ++j) se += __expf(f[j] - mx);
}
__device__ __forceinline__ void xent_grad8(u32x4 v, int c, int64_t tgt, float lse, float grad_scale, u32x4* out) {
  float f[8];
  unpack8(v, f);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float g = __expf(f[j] - lse);
    if (c * 8 + j == tgt) g -= 1.0f;
    f[j] = g * grad_scale;
  }
  out[c] = pack8(f);
}

// bf16 logits (v_t % 8 == 0): loss and gradient.  logits and dlogits may be the
// same buffer (the LM head overwrites the logits with their gradient in place),
// so neither is declared __restrict__.  V = 0: any row length, read twice.
template <int THREADS, int V>
__global__ void __launch_bounds__(THREADS) xent_rows_kernel(
    const uint16_t* logits, int32_t v_t, int64_t v0, const int64_t* __restrict__ targets,
    const float* __restrict__ peer_lse, const float* __restrict__ peer_z, float grad_scale,
    float* __restrict__ loss, uint16_t* dlogits) {
  const int64_t row = blockIdx.x;
  const u32x4* lr = reinterpret_cast<const u32x4*>(logits + row * v_t);
  u32x4* dr = reinterpret_cast<u32x4*>(dlogits + row * v_t);
  const int nch = v_t / 8;
  float mx = -INFINITY, se = 0.f;
  auto z_at = [&](int64_t i) { return __uint_as_float(static_cast<uint32_t>(logits[row * v_t + i]) << 16); };
  const int64_t tgt = targets[row] - v0;
  if constexpr (V > 0) {
    u32x4 v[V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int c = q * THREADS + threadIdx.x;
      v[q] = lr[min(c, nch - 1)];
    }
#pragma unroll
    for (int q = 0; q < V; ++q) {
      float f[8];
      unpack8(v[q], f);
      if (q * THREADS + static_cast<int>(threadIdx.x) < nch) xent_add<8>(f, mx, se);
    }
    const float lse = xent_lse<THREADS / 64>(mx, se, v_t, v0, row, targets, peer_lse, peer_z, loss, z_at);
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int c = q * THREADS + threadIdx.x;
      if (c < nch) xent_grad8(v[q], c, tgt, lse, grad_scale, dr);
    }
  } else {
    for (int c = threadIdx.x; c < nch; c += THREADS) {
      float f[8];
      unpack8(lr[c], f);
      xent_add<8>(f, mx, se);
    }
    const float lse = xent_lse<THREADS / 64>(mx, se, v_t, v0, row, targets, peer_lse, peer_z, loss, z_at);
    for (int c = threadIdx.x; c < nch; c += THREADS) xent_grad8(lr[c], c, tgt, lse, grad_scale, dr);
  }
}

// FP32 logits (v_t % 4 == 0): the loss, and the row overwritten with the softmax
// exp(z - LSE) over the whole vocabulary.
template <int THREADS, int V>
__global__ void __launch_bounds__(THREADS) xent_probs_kernel(
    float* __restrict__ lp, int32_t v_t, int64_t v0, const int64_t* __restrict__ targets,
    const float* __restrict__ peer_lse, const float* __restrict__ peer_z, float* __restrict__ loss) {
  const int64_t row = blockIdx.x;
  f32x4* r4 = reinterpret_cast<f32x4*>(lp + row * v_t);
  const int nch = v_t / 4;
  float mx = -INFINITY, se = 0.f;
  auto z_at = [&](int64_t i) { return lp[row * v_t + i]; };
  auto put = [&](f32x4 f, int c, float lse) {
    r4[c] = f32x4{__expf(f[0] - lse), __expf(f[1] - lse), __expf(f[2] - lse), __expf(f[3] - lse)};
  };
  auto add = [&](f32x4 v) {
    const float f[4] = {v[0], v[1], v[2], v[3]};
    xent_add<4>(f, mx, se);
  };
  if constexpr (V > 0) {
    f32x4 v[V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int c = q * THREADS + threadIdx.x;
      v[q] = r4[min(c, nch - 1)];
    }
#pragma unroll
    for (int q = 0; q < V; ++q)
      if (q * THREADS + static_cast<int>(threadIdx.x) < nch) add(v[q]);
    const float lse = xent_lse<THREADS / 64>(mx, se, v_t, v0, row, targets, peer_lse, peer_z, loss, z_at);
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int c = q * THREADS + threadIdx.x;
      if (c < nch) put(v[q], c, lse);
    }
  } else {
    for (int c = threadIdx.x; c < nch; c += THREADS) add(r4[c]);
    const float lse = xent_lse<THREADS / 64>(mx, se, v_t, v0, row, targets, peer_lse, peer_z, loss, z_at);
    for (int c = threadIdx.x; c < nch; c += THREADS) put(r4[c], c, lse);
  }
}

// dlogits = (softmax - onehot(target)) * grad_scale as bf16, 8 elements per
// thread over the flattened [n][v_t] (v_t % 8 == 0).
__global__ void __launch_bounds__(256) xent_grad_kernel(const float* __restrict__ probs, int64_t n8, int32_t v8,
                                                       int64_t v0, const int64_t* __restrict__ targets,
                                                       float grad_scale, uint16_t* __restrict__ dl) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n8) return;
  const int64_t row = i / v8;
  const int32_t col0 = static_cast<int32_t>(i - row * v8) * 8;
  const int64_t tgt = targets[row] - v0 - col0;
  const float4* p4 = reinterpret_cast<const float4*>(probs) + 2 * i;
  const float4 a = p4[0], b = p4[1];
  float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = (j == tgt ? f[j] - 1.0f : f[j]) * grad_scale;
  reinterpret_cast<u32x4*>(dl)[i] = pack8(f);
}

// ------------------------------------------------------------------ embedding
// Rows of the gathered [b][s_c] token view are split between this rank's own
// sequence-parallel rows and the peers' rows as in the layer (SpRows below).

struct SpRows {
  int32_t s_c, s_sp, r, t;
  // logical row m -> (own row index) or (peer row index) | 0x80000000
  __device__ uint32_t map(int64_t m64) const {
    const int32_t m = static_cast<int32_t>(m64);
    if (t == 1) return static_cast<uint32_t>(m);
    const int32_t bi = m / s_c, i = m - bi * s_c, lo = r * s_sp;
    if (i >= lo && i < lo + s_sp) return static_cast<uint32_t>(bi * s_sp + (i - lo));
    return static_cast<uint32_t>(bi * (t - 1) * s_sp + (i < lo ? i : i - s_sp)) | 0x80000000u;
  }
};

// One wave per gathered row: the table row when the id is in [v0, v0 + v_t),
// zeros otherwise.  Own rows: bf16(partial + receipt); peer rows: the partial.
__global__ void __launch_bounds__(256) embed_fwd_kernel(const int64_t* __restrict__ ids,
                                                       const uint16_t* __restrict__ w, int64_t v0, int32_t v_t,
                                                       int32_t h, int64_t rows, SpRows sp,
                                                       const uint16_t* __restrict__ receipt,
                                                       uint16_t* __restrict__ own, uint16_t* __restrict__ send,
                                                       int64_t* __restrict__ kept) {
  const int lane = threadIdx.x & 63;
  const int64_t m = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (m >= rows) return;
  const int64_t id = ids[m], j = id - v0;
  if (lane == 0) kept[m] = id;          // the backward's copy of the ids
  const bool hit = j >= 0 && j < v_t;
  const uint32_t o = sp.map(m);
  const bool mine = !(o & 0x80000000u);
  const int64_t orow = o & 0x7fffffffu;
  u32x4* dst = reinterpret_cast<u32x4*>((mine ? own : send) + orow * h);
  const u32x4* src = reinterpret_cast<const u32x4*>(w + (hit ? j : 0) * h);
  const u32x4* rc = (mine && receipt) ? reinterpret_cast<const u32x4*>(receipt + orow * h) : nullptr;
  for (int c = lane; c < h / 8; c += 64) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    const u32x4 v = hit ? src[c] : z;
    if (rc) {
      float a[8], b[8];
      unpack8(v, a);
      unpack8(rc[c], b);
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] += b[e];
      dst[c] = pack8(a);
    } else {
      dst[c] = v;
    }
  }
}

// dW[id - v0] += dY[row] over the gathered rows whose id is in range, in fp32.
// One atomic row per token was bound by the atomics: a few ids repeat often in
// text, so their rows were added one after another at the same addresses, and
// a lane's 8 consecutive columns spread every atomic instruction over 16 cache
// lines.  Now chunks of kEmbChunk tokens are sorted by id (embed_sort, into
// workspace: the stashed ids stay, so a captured backward can be replayed), a
// workgroup walks a window of kEmbWin sorted tokens over 1024 columns and adds
// each run of equal ids up in registers before one atomic add per column,
// consecutive lanes on consecutive columns.  8192 tokens of hidden 4096 over a
// shard of 32064 (heavy-tailed ids, a quarter of them in the shard): 627 -> 15
// (sort) + 28 us.
constexpr int kEmbChunk = 2048, kEmbWin = 16;

// Keys (id - v0) << 32 | token, out-of-range ids as all ones, sorted ascending
// per chunk: a bitonic network over LDS (66 steps, one exchange per
// thread and step).
__global__ void __launch_bounds__(kEmbChunk / 2) embed_sort_kernel(const int64_t* __restrict__ ids,
                                                                  uint64_t* __restrict__ keys, int64_t v0, int32_t v_t,
                                                                  int64_t n) {
  __shared__ uint64_t k[kEmbChunk];
  const int tid = threadIdx.x;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kEmbChunk;
#pragma unroll
  for (int i = tid; i < kEmbChunk; i += kEmbChunk / 2) {
    uint64_t key = ~0ull;
    if (base + i < n) {
      const int64_t j = ids[base + i] - v0;
      if (j >= 0 && j < v_t) key = static_cast<uint64_t>(j) << 32 | static_cast<uint32_t>(base + i);
    }
    k[i] = key;
  }
  for (int len = 2; len <= kEmbChunk; len <<= 1)
    for (int half = len >> 1; half > 0; half >>= 1) {
      __syncthreads();
      const int i = 2 * tid - (tid & (half - 1)), j = i + half;   // pairs (i, i + half)
      const uint64_t a = k[i], b = k[j];
      if ((a > b) == ((i & len) == 0)) {
        k[i] = b;
        k[j] = a;
      }
    }
  __syncthreads();
#pragma unroll
  for (int i = tid; i < kEmbChunk; i += kEmbChunk / 2)
    if (base + i < n) keys[base + i] = k[i];
}

// SORTED: ids holds embed_sort's keys, else the raw ids in token order.
template <bool SORTED>
__global__ void __launch_bounds__(256) embed_bwd_kernel(const int64_t* __restrict__ ids, RowSrc dy, int64_t v0,
                                                       int32_t v_t, int32_t h, int64_t rows, float* __restrict__ dw) {
  const int64_t p0 = static_cast<int64_t>(blockIdx.x) * kEmbWin;
  const int nw = static_cast<int>(rows - p0 < kEmbWin ? rows - p0 : kEmbWin);
  const int col = blockIdx.y * 1024 + threadIdx.x;
  // the window's ids and rows, wave-uniform values
  int64_t cur = -1;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  const auto flush = [&] {
    if (cur < 0) return;
    float* d = dw + cur * h;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (col + 256 * q < h) unsafeAtomicAdd(d + col + 256 * q, acc[q]);
  };
  for (int w0 = 0; w0 < nw; w0 += 4) {
    int64_t id[4];
    uint16_t v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {       // four rows' loads in flight
      id[u] = -1;
      if (w0 + u < nw) {
        int64_t m = p0 + w0 + u, j;
        if constexpr (SORTED) {
          const uint64_t key = static_cast<uint64_t>(ids[m]);
          j = key == ~0ull ? -1 : static_cast<int64_t>(key >> 32);
          m = static_cast<uint32_t>(key);
        } else {
          j = ids[m] - v0;
        }
        if (j >= 0 && j < v_t) {
          id[u] = j;
          const uint16_t* src = dy.row(m);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (col + 256 * q < h) v[u][q] = src[col + 256 * q];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (id[u] < 0) continue;
      if (id[u] != cur) {
        flush();
        cur = id[u];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = 0.f;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (col + 256 * q < h) acc[q] += __uint_as_float(static_cast<uint32_t>(v[u][q]) << 16);
    }
  }
  flush();
}

}  // namespace

hipError_t rmsnorm_fwd(const uint16_t* x, const uint16_t* gain, uint16_t* y, int64_t rows, int32_t h,
                       float eps, hipStream_t stream, uint16_t* x_copy, const RopeTable* rope) {
  if (rows <= 0) return hipSuccess;
  const unsigned rope_blk = rope_blocks(rope, 256);
  const dim3 grid(static_cast<unsigned>((rows + 3) / 4) + rope_blk);
  auto go = [&](auto with_rope, auto without) {
    hipLaunchKernelGGL(rope ? with_rope : without, grid, dim3(256), 0, stream, x, gain, y, x_copy, rows, h, eps,
                       rope ? *rope : RopeTable{}, static_cast<int32_t>(rope_blk));
  };
  switch (h % 512 == 0 ? h / 512 : 0) {
    case 8: go(rmsnorm_fwd_kernel<8, true>, rmsnorm_fwd_kernel<8, false>); break;
    case 16: go(rmsnorm_fwd_kernel<16, true>, rmsnorm_fwd_kernel<16, false>); break;
    default: go(rmsnorm_fwd_kernel<0, true>, rmsnorm_fwd_kernel<0, false>);
  }
  return hipGetLastError();
}

int32_t rmsnorm_bwd_partials(int64_t rows) {
  return static_cast<int32_t>(rows < 256 ? rows : 256);     // one block per row, one per CU
}

hipError_t rmsnorm_bwd(const uint16_t* x, const uint16_t* gain, const NormBwdIo& io, float* partial,
                       int32_t n_partial, int64_t rows, int32_t h, float eps, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  const int cpl = (h + 2047) / 2048;
  const bool dy32 = io.dy_f32 != nullptr;
  const int res = io.dres_f32 ? 2 : io.dres ? 1 : 0;
  const bool out32 = io.dx_f32 != nullptr;
  const void* dy = dy32 ? static_cast<const void*>(io.dy_f32) : io.dy;
  const void* dres = res == 2 ? static_cast<const void*>(io.dres_f32) : io.dres;
  // the three forms the layer and the LM-head block use
#define L4D_RMS_BWD(C, D32, R, O32)                                                                            \
  hipLaunchKernelGGL((rmsnorm_bwd_kernel<C, D32, R, O32>), dim3(n_partial), dim3(256), 0, stream, x, gain, dy, \
                     dres, io.dx, io.dx_f32, partial, rows, h, eps)
#define L4D_RMS_BWD_FORM(C)                                                      \
  if (!dy32 && res == 0 && !out32) L4D_RMS_BWD(C, false, 0, false);              \
  else if (dy32 && res == 1 && out32) L4D_RMS_BWD(C, true, 1, true);             \
  else if (dy32 && res == 2 && !out32) L4D_RMS_BWD(C, true, 2, false);           \
  else return hipErrorInvalidValue;
  if (cpl <= 1) {
    L4D_RMS_BWD_FORM(1)
  } else if (cpl <= 2) {
    L4D_RMS_BWD_FORM(2)
  } else {
    L4D_RMS_BWD_FORM(4)
  }
#undef L4D_RMS_BWD_FORM
#undef L4D_RMS_BWD
  return hipGetLastError();
}

hipError_t reduce_rows_add(const float* partial, int32_t n_partial, int32_t h, float* out, hipStream_t stream,
                           const RopeTable* rope) {
  if (n_partial > 256) return hipErrorInvalidValue;      // rmsnorm_bwd_partials gives at most 256
  if (n_partial <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((h + 63) / 64) + rope_blocks(rope, kSumWaves * 64));
  hipLaunchKernelGGL(rope ? column_sums_kernel<true> : column_sums_kernel<false>, grid, dim3(kSumWaves * 64), 0, stream,
                     partial, n_partial, h, out, rope ? *rope : RopeTable{});
  return hipGetLastError();
}

hipError_t xent_rows(const uint16_t* logits, int64_t n, int32_t v_t, int64_t v0, const int64_t* targets,
                     const float* peer_lse, const float* peer_z, float grad_scale, float* loss,
                     uint16_t* dlogits, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  // the fewest threads whose registers hold the row, up to 1024
  const dim3 grid(static_cast<unsigned>(n));
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, logits, v_t, v0, targets, peer_lse, peer_z, grad_scale,
                       loss, dlogits);
  };
  if (v_t <= 256 * 4 * 8) go(xent_rows_kernel<256, 4>, 256);
  else if (v_t <= 512 * 8 * 8) go(xent_rows_kernel<512, 8>, 512);
  else if (v_t <= 1024 * 8 * 8) go(xent_rows_kernel<1024, 8>, 1024);
  else go(xent_rows_kernel<256, 0>, 256);
  return hipGetLastError();
}

hipError_t xent_probs(float* logits, int64_t n, int32_t v_t, int64_t v0, const int64_t* targets,
                      const float* peer_lse, const float* peer_z, float* loss, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(n));
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, logits, v_t, v0, targets, peer_lse, peer_z, loss);
  };
  if (v_t <= 256 * 8 * 4) go(xent_probs_kernel<256, 8>, 256);
  else if (v_t <= 1024 * 8 * 4) go(xent_probs_kernel<1024, 8>, 1024);
  else if (v_t <= 1024 * 16 * 4) go(xent_probs_kernel<1024, 16>, 1024);
  else go(xent_probs_kernel<256, 0>, 256);
  return hipGetLastError();
}

hipError_t xent_grad(const float* probs, int64_t n, int32_t v_t, int64_t v0, const int64_t* targets,
                     float grad_scale, uint16_t* dlogits, hipStream_t stream) {
  const int64_t n8 = n * (v_t / 8);
  if (n8 <= 0) return hipSuccess;
  hipLaunchKernelGGL(xent_grad_kernel, dim3(static_cast<unsigned>((n8 + 255) / 256)), dim3(256), 0, stream, probs,
                     n8, v_t / 8, v0, targets, grad_scale, dlogits);
  return hipGetLastError();
}

hipError_t embed_fwd(const int64_t* ids, const uint16_t* w, int64_t v0, int32_t v_t, int32_t h, int64_t rows,
                     int32_t s_c, int32_t s_sp, int32_t r, int32_t t, const uint16_t* receipt, uint16_t* own,
                     uint16_t* send, int64_t* kept, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(embed_fwd_kernel, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, stream, ids, w,
                     v0, v_t, h, rows, SpRows{s_c, s_sp, r, t}, receipt, own, send, kept);
  return hipGetLastError();
}

// The sort costs a launch and a fixed 11 us or so (a chain of 66 exchange steps),
// what it saves grows with the rows that are added: about rows / t of them hit
// this rank's shard.  From 2^20 gradient elements on, the sorted form is never
// behind one atomic row per token, whatever the ids (hidden 4096 on TP 4: 1024
// tokens 32 us against 39 with uniform ids, 31 against 74 with heavy-tailed ones);
// below, token order is the faster one (hidden 512, TP 1, 1024 tokens: 16 us, sorted
// 28, one atomic row per token 22; heavy-tailed 16, 27, 48).
uint64_t embed_bwd_ws_bytes(int64_t rows, int32_t h, int32_t t) {
  return rows <= 512 || rows * h / t < (int64_t{1} << 20) ? 0 : static_cast<uint64_t>(rows) * 8;
}

hipError_t embed_bwd(const int64_t* ids, uint64_t* keys, RowSrc dy, int64_t v0, int32_t v_t, int32_t h, int64_t rows,
                     float* dw, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((rows + kEmbWin - 1) / kEmbWin), static_cast<unsigned>((h + 1023) / 1024));
  if (!keys) {
    hipLaunchKernelGGL(embed_bwd_kernel<false>, grid, dim3(256), 0, stream, ids, dy, v0, v_t, h, rows, dw);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(embed_sort_kernel, dim3(static_cast<unsigned>((rows + kEmbChunk - 1) / kEmbChunk)),
                     dim3(kEmbChunk / 2), 0, stream, ids, keys, v0, v_t, rows);
  hipLaunchKernelGGL(embed_bwd_kernel<true>, grid, dim3(256), 0, stream, reinterpret_cast<const int64_t*>(keys), dy,
                     v0, v_t, h, rows, dw);
  return hipGetLastError();
}

}  // namespace l4d
