// Device side of the scans that more than one launch runs: a row scan, a column scan and what finishes them
// (see scan_kernels.hip, which launches them on their own and in pairs, and gemm_kernels.hip, where the
// parity blocks of C-bar ride in the product's launch).
#pragma once
#include <type_traits>
#include "gecc_internal.h"

namespace gecc {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t stream_t;

template <int DT> struct Elem;
template <> struct Elem<GECC_F32> {
  using type = float;
  static constexpr int VEC = 4;
  using raw = float4;
  // (memcpy: rows may start at any element; the hardware takes a 16-byte load at any address)
  static __device__ __forceinline__ raw load_raw(const float* p) { raw x; __builtin_memcpy(&x, p, 16); return x; }
  // (16-byte aligned; marked as not to be kept in the caches)
  static __device__ __forceinline__ raw load_stream(const float* p) {
    return __builtin_bit_cast(raw, __builtin_nontemporal_load(reinterpret_cast<const stream_t*>(p)));
  }
  static __device__ __forceinline__ void widen(const raw& x, double* v) {
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  }
  static __device__ __forceinline__ double load_one(const float* p) { return (double)*p; }
};
template <> struct Elem<GECC_BF16> {
  using type = uint16_t;
  static constexpr int VEC = 8;
  using raw = uint4;
  static __device__ __forceinline__ raw load_raw(const uint16_t* p) { raw x; __builtin_memcpy(&x, p, 16); return x; }
  static __device__ __forceinline__ raw load_stream(const uint16_t* p) {
    return __builtin_bit_cast(raw, __builtin_nontemporal_load(reinterpret_cast<const stream_t*>(p)));
  }
  static __device__ __forceinline__ void widen(const raw& x, double* v) {
    uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = (double)__uint_as_float(w[i] << 16);
      v[2 * i + 1] = (double)__uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ double load_one(const uint16_t* p) {
    return (double)__uint_as_float(((uint32_t)*p) << 16);
  }
};

// the same in vectors of 8 bytes
template <int DT> struct ElemHalf;
template <> struct ElemHalf<GECC_F32> : Elem<GECC_F32> {
  static constexpr int VEC = 2;
  using raw = float2;
  static __device__ __forceinline__ raw load_raw(const float* p) { raw x; __builtin_memcpy(&x, p, 8); return x; }
  static __device__ __forceinline__ void widen(const raw& x, double* v) { v[0] = x.x; v[1] = x.y; }
};
template <> struct ElemHalf<GECC_BF16> : Elem<GECC_BF16> {
  static constexpr int VEC = 4;
  using raw = uint2;
  static __device__ __forceinline__ raw load_raw(const uint16_t* p) { raw x; __builtin_memcpy(&x, p, 8); return x; }
  static __device__ __forceinline__ void widen(const raw& x, double* v) {
    v[0] = (double)__uint_as_float(x.x << 16); v[1] = (double)__uint_as_float(x.x & 0xffff0000u);
    v[2] = (double)__uint_as_float(x.y << 16); v[3] = (double)__uint_as_float(x.y & 0xffff0000u);
  }
};

__device__ __forceinline__ bool gated_off(const int32_t* gate, int64_t stride, int b, int value) {
  if (!gate) return false;
  const int32_t g = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(gate) + stride * b);
  return g != value;
}

// wavefront-local ordering of LDS traffic: the hardware keeps a wavefront's LDS instructions in
// order; this keeps the compiler from moving them across
// (a compiler barrier only: a fence instruction would also wait for the wavefront's outstanding
// global loads and stores, which is exactly what the loop must not do)
__device__ __forceinline__ void wave_lds_fence() { asm volatile("" ::: "memory"); }

// The second stage of a column reduction adds the chunk partials of an output in one fixed order,
// whoever does it (a kernel of its own, workgroups carried by a row scan, or the last workgroup of
// the first stage): four slices, slice w over the chunks w, w + 4, ..., each with four running sums,
// combined as ((s0 + s1) + (s2 + s3)).
// One slice of G outputs at once (G independent chains of loads in flight); part[g]: chunk 0's
// partial of output g, stride: doubles between chunks.
// DEV: the partials were written by other workgroups of this launch (load_dev)
template <int G, bool DEV>
__device__ __forceinline__ void slice_sums(const double* const* part, int64_t stride, int nchunk, int w, double* s) {
  double t[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g) { t[g][0] = 0.0; t[g][1] = 0.0; t[g][2] = 0.0; t[g][3] = 0.0; }
  int ch = w;
  for (; ch + 12 < nchunk; ch += 16) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double* q = part[g] + (int64_t)(ch + 4 * u) * stride;
        t[g][u] += DEV ? load_dev(q) : *q;
      }
  }
  for (; ch < nchunk; ch += 4) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double* q = part[g] + (int64_t)ch * stride;
      t[g][0] += DEV ? load_dev(q) : *q;
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) s[g] = (t[g][0] + t[g][1]) + (t[g][2] + t[g][3]);
}

// Stage 2 of coldot as workgroups of its own: 64 outputs per workgroup of 256 threads, wavefront w
// takes slice w.  scratch, out: of batch item b; red: 256 doubles of LDS.
__device__ __forceinline__ void coldot_stage2_body(const double* scratch, double* out, int Cc, int nchunk, int blk,
                                                   double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int o = blk * 64 + lane;                   // index into [2][Cc]
  double s = 0.0;
  if (o < 2 * Cc) {
    const double* part = scratch + o;
    slice_sums<1, false>(&part, 2 * (int64_t)Cc, nchunk, wave, &s);
  }
  red[wave * 64 + lane] = s;
  __syncthreads();
  if (wave == 0 && o < 2 * Cc) out[o] = (red[lane] + red[64 + lane]) + (red[128 + lane] + red[192 + lane]);
}

// The whole of that sum by one thread, sixteen loads in flight
__device__ __forceinline__ double chunk_sum(const double* part, int64_t stride, int nchunk) {
  double t[4][4];                                  // [slice][running sum]
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int u = 0; u < 4; ++u) t[w][u] = 0.0;
#pragma unroll 1
  for (int c0 = 0; c0 < nchunk; c0 += 16) {
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = part[(int64_t)min(c0 + i, nchunk - 1) * stride];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const bool four = c0 + w + 12 < nchunk;      // (slice_sums' first loop; its second one puts what is left into the first sum)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double x = c0 + w + 4 * u < nchunk ? v[w + 4 * u] : 0.0;
        if (u == 0 || !four) t[w][0] += x;
        else t[w][u] += x;
      }
    }
  }
  double s[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) s[w] = (t[w][0] + t[w][1]) + (t[w][2] + t[w][3]);
  return (s[0] + s[1]) + (s[2] + s[3]);
}
// the same for G outputs at once and at most MAX (<= 16) chunks
template <int G, int MAX>
__device__ __forceinline__ void chunk_sums(const double* const* part, int64_t stride, int nchunk, double* s) {
  double v[G][MAX];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int i = 0; i < MAX; ++i) v[g][i] = part[g][(int64_t)min(i, nchunk - 1) * stride];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    double t[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      double first = 0.0, other[3] = {0.0, 0.0, 0.0};
      const bool four = MAX > 12 && w + 12 < nchunk;
#pragma unroll
      for (int u = 0; w + 4 * u < MAX; ++u) {
        const double x = w + 4 * u < nchunk ? v[g][w + 4 * u] : 0.0;
        if (u == 0 || !four) first += x;
        else other[u - 1] += x;
      }
      t[w] = (first + other[0]) + (other[1] + other[2]);
    }
    s[g] = (t[0] + t[1]) + (t[2] + t[3]);
  }
}
// Sum of kind t of output i (of len) of batch item b
__device__ __forceinline__ double parts_sum(const Parts& p, int b, int len, int t, int i) {
  if (p.nchunk > 0) return chunk_sum(p.chunks + (int64_t)b * p.nchunk * 2 * len + (int64_t)t * len + i, 2 * (int64_t)len, p.nchunk);
  const double* q = p.segs + ((int64_t)b * len + i) * p.nseg * 2 + t;
  double s = 0.0;
#pragma unroll 1
  for (int g0 = 0; g0 < p.nseg; g0 += 8) {
    double v[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) v[g] = q[2 * min(g0 + g, p.nseg - 1)];
#pragma unroll
    for (int g = 0; g < 8; ++g) s += g0 + g < p.nseg ? v[g] : 0.0;
  }
  return s;
}

// The same sums for the 2 * 64 * VEC outputs of one column segment, by the workgroup that finished
// the segment's last chunk.  col0: first column of the segment; red: 4 * 256 doubles of LDS.
template <int VEC>
__device__ __forceinline__ void coldot_finish_segment(const double* scratch, double* out, int Cc, int nchunk, int col0,
                                                      double* red) {
  constexpr int G = 4;                              // groups of 64 outputs a thread works on at once
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  static_assert((2 * VEC) % G == 0, "groups");
#pragma unroll 1
  for (int g0 = 0; g0 < 2 * VEC; g0 += G) {
    const double* part[G];
    int o[G];
    bool ok[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int t = (g0 + g) / VEC, col = col0 + ((g0 + g) % VEC) * 64 + lane;
      ok[g] = col < Cc;
      o[g] = t * Cc + min(col, Cc - 1);
      part[g] = scratch + o[g];
    }
    double s[G];
    slice_sums<G, true>(part, 2 * (int64_t)Cc, nchunk, wave, s);
#pragma unroll
    for (int g = 0; g < G; ++g) red[(g * 4 + wave) * 64 + lane] = s[g];
    __syncthreads();
    if (wave < G) {                                 // wavefront g writes group g
      const int g = wave;
      if (ok[g]) out[o[g]] = (red[(g * 4 + 0) * 64 + lane] + red[(g * 4 + 1) * 64 + lane]) +
                             (red[(g * 4 + 2) * 64 + lane] + red[(g * 4 + 3) * 64 + lane]);
    }
    __syncthreads();
  }
}

// Stage 2 of the row part of tile_scan (see below): the segments of a row added in order.
// part: [R][nseg][2], out: [2][R], both of batch item b.
template <bool DEV>
__device__ __forceinline__ void rowseg_sum(const double* part, double* out, int R, int nseg, int r) {
  const double* p = part + (int64_t)r * nseg * 2;
  double s0 = 0.0, s1 = 0.0;
  for (int g = 0; g < nseg; ++g) {
    s0 += DEV ? load_dev(p + 2 * g) : p[2 * g];
    s1 += DEV ? load_dev(p + 2 * g + 1) : p[2 * g + 1];
  }
  out[r] = s0;
  out[(int64_t)R + r] = s1;
}
// as workgroups of their own: 256 rows each
__device__ __forceinline__ void rowseg_stage2_body(const double* part, double* out, int R, int nseg, int blk) {
  const int r = blk * 256 + threadIdx.x;
  if (r < R) rowseg_sum<false>(part, out, R, nseg, r);
}

// a pending second stage (column chunks and / or row segments), by workgroup index
__device__ __forceinline__ void stage2_dispatch(const Stage2Job& j, int b, int blk, double* lds) {
  const int col_blocks = j.Cc > 0 ? (2 * j.Cc + 63) / 64 : 0;
  if (blk < col_blocks)
    coldot_stage2_body(j.scratch + (int64_t)b * j.nchunk * 2 * j.Cc, j.out + (int64_t)b * j.out_stride, j.Cc,
                       j.nchunk, blk, lds);
  else
    rowseg_stage2_body(j.row_scratch + (int64_t)b * j.R * j.nseg * 2, j.row_out + (int64_t)b * j.row_out_stride,
                       j.R, j.nseg, blk - col_blocks);
}

// -------------------------------------------------------------------------------------------
// rowdot: out[t][r] = sum_c w_t[c] X[r,c].   One workgroup owns RB rows and walks all columns;
// a thread keeps the weights of its VEC columns in registers and reuses them for the RB rows.
constexpr int RD_THREADS = 256;
constexpr int RD_BIG_RB = 16, RD_BIG_U = 1, RD_SMALL_RB = 4, RD_SMALL_U = 2;
constexpr int RD_BIG_RB_W = 8;   // with explicit weights (they take registers too)

// RD_RB rows per workgroup: 16 when there are rows enough to fill the chip, else 4.  RD_U column
// steps are taken together, so that a thread has RD_RB * RD_U independent 16-byte loads in
// flight before the first of them is used (the kernel is a stream over the operand: what it
// needs is memory-level parallelism, the arithmetic hides behind it).
// The rows bx * RD_RB ... of batch item b.  red: RD_RB * RD_THREADS doubles of LDS.  The sums of a row
// do not depend on RD_RB or RD_U (a thread adds its columns in ascending order either way).
template <int DT, bool IDXW, int RD_RB, int RD_U>
__device__ __forceinline__ void rowdot_body(const ScanArgs& a, int bx, int b, double* lds) {
  using E = Elem<DT>;
  using T = typename E::type;
  constexpr int VEC = E::VEC;
  constexpr int STEP = RD_THREADS * VEC;   // columns one pass of the workgroup covers
  const T* X = reinterpret_cast<const T*>(a.X) + (int64_t)b * a.xs;
  const double* w0 = IDXW ? nullptr : a.w + (int64_t)b * a.w_stride;
  const double* w1 = IDXW ? nullptr : w0 + a.Cc;
  double* out = a.out + (int64_t)b * a.out_stride;
  const int r0 = bx * RD_RB;
  const int tid = threadIdx.x;

  double acc0[RD_RB], acc1[RD_RB];
#pragma unroll
  for (int r = 0; r < RD_RB; ++r) { acc0[r] = 0.0; acc1[r] = 0.0; }

  // whole vectors for every thread: rows past the end are clamped to the last one (their sums
  // are computed and never stored), so the body has no branches
  int c0 = 0;
  for (; c0 + RD_U * STEP <= a.Cc; c0 += RD_U * STEP) {
    typename E::raw x[RD_U][RD_RB];
    double wa[RD_U][VEC], wb[RD_U][VEC];
#pragma unroll
    for (int u = 0; u < RD_U; ++u) {
      const int c = c0 + u * STEP + tid * VEC;
#pragma unroll
      for (int r = 0; r < RD_RB; ++r)
        x[u][r] = E::load_raw(X + (int64_t)min(r0 + r, a.R - 1) * a.ld + (unsigned)c);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if (IDXW) { wa[u][e] = 1.0; wb[u][e] = (double)(c + e + 1); }
        else      { wa[u][e] = w0[c + e]; wb[u][e] = w1[c + e]; }
      }
    }
#pragma unroll
    for (int u = 0; u < RD_U; ++u) {
#pragma unroll
      for (int r = 0; r < RD_RB; ++r) {
        double v[VEC];
        E::widen(x[u][r], v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          acc0[r] = IDXW ? acc0[r] + v[e] : fma(wa[u][e], v[e], acc0[r]);
          acc1[r] = fma(wb[u][e], v[e], acc1[r]);
        }
        __builtin_amdgcn_sched_barrier(0);   // widen one vector at a time (registers)
      }
    }
  }
  // the remaining columns; the thread on which the row ends in mid-vector reads the row's last vector
  // and drops the elements its neighbour has
  for (; c0 < a.Cc; c0 += STEP) {
    const int c_true = c0 + tid * VEC;
    if (c_true >= a.Cc) continue;
    if (a.Cc >= VEC) {
      const int c = min(c_true, a.Cc - VEC), drop = c_true - c;
      double wa[VEC], wb[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if (IDXW) { wa[e] = 1.0; wb[e] = (double)(c + e + 1); }
        else      { wa[e] = w0[c + e]; wb[e] = w1[c + e]; }
      }
      typename E::raw x[RD_RB];
#pragma unroll
      for (int r = 0; r < RD_RB; ++r) x[r] = E::load_raw(X + (int64_t)min(r0 + r, a.R - 1) * a.ld + c);
#pragma unroll
      for (int r = 0; r < RD_RB; ++r) {
        double v[VEC];
        E::widen(x[r], v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const double y = e < drop ? 0.0 : v[e];
          acc0[r] = IDXW ? acc0[r] + y : fma(wa[e], y, acc0[r]);
          acc1[r] = fma(wb[e], y, acc1[r]);
        }
      }
    } else {
      for (int r = 0; r < RD_RB; ++r) {
        const int row = r0 + r;
        if (row < a.R)
          for (int e = 0; e < a.Cc - c_true; ++e) {
            const double v = E::load_one(X + (int64_t)row * a.ld + c_true + e);
            acc0[r] = fma(IDXW ? 1.0 : w0[c_true + e], v, acc0[r]);
            acc1[r] = fma(IDXW ? (double)(c_true + e + 1) : w1[c_true + e], v, acc1[r]);
          }
      }
    }
  }

  // fixed-order reduction over the 256 threads, one parity kind (t) at a time
  double (*red)[RD_THREADS] = reinterpret_cast<double (*)[RD_THREADS]>(lds);
  const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (t) __syncthreads();
#pragma unroll
    for (int r = 0; r < RD_RB; ++r) red[r][tid] = t ? acc1[r] : acc0[r];
    __syncthreads();
    for (int q = wave; q < RD_RB; q += RD_THREADS / 64) {
      double s = (red[q][lane] + red[q][lane + 64]) + (red[q][lane + 128] + red[q][lane + 192]);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
      const int row = r0 + q;
      if (lane == 0 && row < a.R) out[(int64_t)t * a.R + row] = s;
    }
  }
}

// Rows per workgroup of a scan that rides in a product's launch: as many as leave the product its occupancy (of 1024^3 fp32, 160
// scan workgroups of eight rows instead of 288 of four, and before the product's instead of among them: 53.6 -> 50.7 us a
// call; bf16 has no registers for eight)
template <int DT> constexpr int side_rows() { return DT == GECC_F32 ? RD_BIG_RB_W : RD_SMALL_RB; }

// The same reduction with a wavefront per RB rows (4 RB rows per workgroup): no barrier, and no idle threads
// where a row is shorter than one pass of the workgroup.
constexpr int RW_RB = 8;
constexpr int RW_LDS_LD = 65;
constexpr int RW_LDS_DOUBLES = 4 * 2 * RW_RB * RW_LDS_LD;
template <int DT, bool IDXW>
__device__ __forceinline__ void rowdot_wave_body(const ScanArgs& a, int bx, int b, double* lds) {
  using E = Elem<DT>;
  using T = typename E::type;
  constexpr int VEC = E::VEC, STEP = 64 * VEC, RB = RW_RB;
  const T* X = reinterpret_cast<const T*>(a.X) + (int64_t)b * a.xs;
  const double* w0 = IDXW ? nullptr : a.w + (int64_t)b * a.w_stride;
  const double* w1 = IDXW ? nullptr : w0 + a.Cc;
  double* out = a.out + (int64_t)b * a.out_stride;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = (bx * 4 + wave) * RB;
  if (r0 >= a.R) return;
  double acc0[RB], acc1[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) { acc0[r] = 0.0; acc1[r] = 0.0; }
  for (int c0 = 0; c0 < a.Cc; c0 += STEP) {
    const int c_true = c0 + lane * VEC;
    if (a.Cc >= VEC) {
      // (lanes past the end read the row's last vector and drop all of it)
      const int c = min(c_true, a.Cc - VEC), drop = c_true - c;
      typename E::raw x[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) x[r] = E::load_raw(X + (int64_t)min(r0 + r, a.R - 1) * a.ld + c);
      double wa[VEC], wb[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if (IDXW) { wa[e] = 1.0; wb[e] = (double)(c + e + 1); }
        else      { wa[e] = w0[c + e]; wb[e] = w1[c + e]; }
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        double v[VEC];
        E::widen(x[r], v);
        if (c0 + STEP > a.Cc) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[e] = e < drop ? 0.0 : v[e];
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          acc0[r] = IDXW ? acc0[r] + v[e] : fma(wa[e], v[e], acc0[r]);
          acc1[r] = fma(wb[e], v[e], acc1[r]);
        }
        __builtin_amdgcn_sched_barrier(0);   // widen one vector at a time (registers)
      }
    } else if (c_true < a.Cc) {
#pragma unroll
      for (int r = 0; r < RB; ++r)
        for (int e = 0; e < a.Cc; ++e) {
          const double v = E::load_one(X + (int64_t)min(r0 + r, a.R - 1) * a.ld + e);
          acc0[r] = fma(IDXW ? 1.0 : w0[e], v, acc0[r]);
          acc1[r] = fma(IDXW ? (double)(e + 1) : w1[e], v, acc1[r]);
        }
    }
  }
  // the 64 lanes' sums, transposed through the wavefront's own LDS: four lanes per output add 16 each
  double* tr = lds + wave * (2 * RB * RW_LDS_LD);
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    tr[(2 * r) * RW_LDS_LD + lane] = acc0[r];
    tr[(2 * r + 1) * RW_LDS_LD + lane] = acc1[r];
  }
  wave_lds_fence();
  const int o = lane >> 2, q = lane & 3;
  double part[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) part[i] = tr[o * RW_LDS_LD + q * 16 + i];
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) s += part[i];
  s += __shfl_xor(s, 1, 64);
  s += __shfl_xor(s, 2, 64);
  const int row = r0 + (o >> 1);
  if (q == 0 && row < a.R) out[(int64_t)(o & 1) * a.R + row] = s;
}

// -------------------------------------------------------------------------------------------
// coldot: out[t][c] = sum_r w_t[r] X[r,c].   Stage 1: a workgroup owns 64*VEC columns and one
// chunk of SCAN_CHUNK_ROWS rows; its 4 wavefronts interleave the rows and are combined through
// LDS.  Stage 2 adds the chunks in order.
constexpr int CD_THREADS = 256;

// LDS of a coldot workgroup: the four wavefronts' sums, reused by the last workgroup of a segment
constexpr int CD_LDS_DOUBLES = 4 * 2 * 8 * 64;
constexpr int CD_FLAG_AT = 1024;     // (behind what coldot_finish_segment uses)

// Column segment bx, chunk `chunk` of batch item b.  With a.done set, the workgroup that finishes a
// segment's last chunk also adds the chunks up (no second stage to launch).
// CD_NB: rows a wavefront loads at once (its sums do not depend on it)
// WPARTS: explicit weights that may still be in parts (wp).  Every workgroup adds up those of its own rows, which costs less
// than the launch that would have to come first.  (Not in the scans' own launches, for the registers.)
// ONE: whether the one chunk of a short column (nchunk == 1) is taken for the sums themselves: never, in this launch, or where
// it turns out to be one (0.3 us of a long column's 6 to 10, for the question)
constexpr int CD_ROWS = 8;
enum : int { CD_CHUNKS = 0, CD_ONE = 1, CD_ASK = 2 };
// E: Elem, or ElemHalf for a scan of few workgroups: half the columns to each, so that twice as many share the rows out, and as many
// bytes of a wavefront's rows on their way (the sums of a column are the same)
template <class E, bool IDXW, int CD_NB, int ONE, bool WPARTS = false>
__device__ __forceinline__ void coldot_body(const ScanArgs& a, const Parts& wp, int nchunk, int nsegx, int bx, int chunk,
                                            int b, double* lds) {
  using T = typename E::type;
  constexpr int VEC = E::VEC;
  const T* X = reinterpret_cast<const T*>(a.X) + (int64_t)b * a.xs;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // first column of a lane's vector; the lane on which the row ends in mid-vector reads the row's last
  // vector (the columns it shares with its neighbour are left to that one below)
  auto first_col = [&](int l) { return min((bx * 64 + l) * VEC, max(a.Cc - VEC, 0)); };
  const int c = first_col(lane);
  const int rbeg = chunk * SCAN_CHUNK_ROWS;
  const int rend = min(a.R, rbeg + SCAN_CHUNK_ROWS);
  const bool owns = (bx * 64 + lane) * VEC < a.Cc;
  const double* w0 = IDXW ? nullptr : a.w + (int64_t)b * a.w_stride;
  const double* w1 = IDXW ? nullptr : w0 + a.R;
  // Explicit weights of the chunk's rows go to LDS first: read where they are needed, every row waits for its own (bf16 4096^2 12.1 ->
  // 8.8 us, 3001^2 10.3 -> 7.6, 4096 x 14336 25.4 -> 23.3, 16384 x 4096 30.3 -> 28.3)
  const double2* wl = reinterpret_cast<const double2*>(lds);
  auto load_weights = [&] {
    const int t = tid / SCAN_CHUNK_ROWS, row = rbeg + tid % SCAN_CHUNK_ROWS;
    static_assert(CD_THREADS == 2 * SCAN_CHUNK_ROWS, "a thread per weight");
    if (row < rend) {
      const bool parts = WPARTS && (wp.nchunk > 0 || wp.nseg > 0);
      lds[2 * (row - rbeg) + t] = parts ? parts_sum(wp, b, a.R, t, row) : (t ? w1 : w0)[row];
    }
    __syncthreads();
  };
  auto weights = [&](int row, double& wa, double& wb) {
    if (IDXW) { wa = 1.0; wb = (double)(row + 1); }
    else { const double2 w = wl[row - rbeg]; wa = w.x; wb = w.y; }
  };

  double acc0[VEC], acc1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) { acc0[e] = 0.0; acc1[e] = 0.0; }

  // Batches of CD_NB rows per wavefront, double buffered: the loads of the next batch are in
  // flight while this one is added up (a wavefront walks its rows one batch after the other,
  // so without this every batch would pay the full memory latency).
  typename E::raw xa[CD_NB], xb[CD_NB];
  const bool vec = owns && a.Cc >= VEC;
  const T* col = X + c;
  auto load = [&](typename E::raw* x, int rr) {
#pragma unroll
    for (int u = 0; u < CD_NB; ++u) x[u] = E::load_raw(col + (int64_t)(rr + 4 * u) * a.ld);
  };
  int r = rbeg + wave;
  const int cnt = r < rend ? (rend - r + 3) / 4 : 0;   // rows of this wavefront
  const int nb = cnt / CD_NB;
  if (vec && nb > 0) load(xa, r);
  if (!IDXW) load_weights();
  if (vec) {
    auto add_row = [&](const typename E::raw& x, int row) {
      double v[VEC];
      E::widen(x, v);
      double wa, wb;
      weights(row, wa, wb);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        acc0[e] = IDXW ? acc0[e] + v[e] : fma(wa, v[e], acc0[e]);
        acc1[e] = fma(wb, v[e], acc1[e]);
      }
    };
    auto add = [&](const typename E::raw* x, int rr) {
#pragma unroll
      for (int u = 0; u < CD_NB; ++u) {
        add_row(x[u], rr + 4 * u);
        if (!IDXW && u % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (weights of four rows at a time: registers)
      }
    };
    constexpr int STEP = 4 * CD_NB;
    if (nb > 0) {
      int bi = 0;
      for (; bi + 1 < nb; bi += 2) {
        load(xb, r + STEP);
        add(xa, r);
        if (bi + 2 < nb) load(xa, r + 2 * STEP);
        add(xb, r + STEP);
        r += 2 * STEP;
      }
      if (bi < nb) { add(xa, r); r += STEP; }
    }
    if (r < rend) {
      // the last few rows, loaded together as well (one after the other they took a latency each)
#pragma unroll
      for (int u = 0; u < CD_NB; ++u) xa[u] = E::load_raw(col + (int64_t)min(r + 4 * u, rend - 1) * a.ld);
#pragma unroll
      for (int u = 0; u < CD_NB; ++u)
        if (r + 4 * u < rend) add_row(xa[u], r + 4 * u);
    }
  } else if (owns) {
    for (; r < rend; r += 4) {
      double wa, wb;
      weights(r, wa, wb);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {      // (rows shorter than a vector)
        if (e >= a.Cc) continue;
        const double v = E::load_one(X + (int64_t)r * a.ld + c + e);
        acc0[e] = fma(wa, v, acc0[e]);
        acc1[e] = fma(wb, v, acc1[e]);
      }
    }
  }

  double (*red)[2][VEC][64] = reinterpret_cast<double (*)[2][VEC][64]>(lds);
  if (!IDXW) __syncthreads();      // every wavefront is done with the weights
#pragma unroll
  for (int e = 0; e < VEC; ++e) { red[wave][0][e][lane] = acc0[e]; red[wave][1][e][lane] = acc1[e]; }
  __syncthreads();
  // thread -> (t, e, lane'): 2*VEC*64 outputs, 256 threads
  const bool whole = ONE == CD_ONE || (ONE == CD_ASK && nchunk == 1);
  double* part = whole ? a.out + (int64_t)b * a.out_stride : a.scratch + ((int64_t)b * nchunk + chunk) * 2 * a.Cc;
  for (int o = tid; o < 2 * VEC * 64; o += CD_THREADS) {
    const int l = o & 63, e0 = (o >> 6) % VEC, t = o / (64 * VEC);
    const int col = (bx * 64 + l) * VEC + e0;
    if (col < a.Cc) {
      const int e = col - first_col(l);
      double s = (red[0][t][e][l] + red[1][t][e][l]) + (red[2][t][e][l] + red[3][t][e][l]);
      if (ONE != CD_CHUNKS) s += 0.0;        // (as the second stage would)
      // (written through only when another workgroup of this launch reads it: such stores cost more)
      if (a.done && !whole) store_dev(part + (int64_t)t * a.Cc + col, s);
      else part[(int64_t)t * a.Cc + col] = s;
    }
  }
  if (a.done && !whole && arrive_last(a.done + (int64_t)b * nsegx + bx, (uint32_t)nchunk, reinterpret_cast<int*>(lds + CD_FLAG_AT)))
    coldot_finish_segment<VEC>(a.scratch + (int64_t)b * nchunk * 2 * a.Cc, a.out + (int64_t)b * a.out_stride, a.Cc,
                               nchunk, bx * 64 * VEC, lds);
}

// -------------------------------------------------------------------------------------------
// tile_scan: both reductions of an operand in ONE pass over it.
//   column part  out_col[t][c] = sum_r wr_t[r] X[r,c]      (two-stage, like coldot)
//   row part     out_row[t][r] = sum_c wc_t[c] X[r,c]      (two-stage: per 64*VEC-column segment)
// Each part has either the index weights of Section III (1, index + 1) or two fp64 vectors.  With
// both parts on, encoding an operand (A_P, index weights along one axis) and its parity block of
// C-bar (P_r = A B_P, vector weights along the other) cost one read of the operand instead of two.
// A part switched off costs nothing; a part computes the same sums in the same order whether the
// other one is on or not, so the gated audit (one part) reproduces an encoding (maybe both) bit for
// bit.  All products go through fma(), never a*b+c, for the same reason.
//
// A workgroup is four wavefronts on one segment of 64*VEC columns; each walks its own quarter of
// the chunk's rows, TS_RB rows (loads) at a time; three wavefronts share a SIMD and cover each
// other's waits.  Per 16 bytes a lane spends 8 conversions and 32 fp64 operations of 4.4 cycles each, about
// 220 cycles per row and wavefront, 9.8 TB/s if nothing else were to do; its loads alone stream at 5.8 TB/s, the
// whole kernel at 4.2, and with eight rows on their way at all times (registers reloaded as they fall free) no faster.  (4.4 with
// loads that are not kept in the caches: 470 MB 107 us instead of 114, the row part alone over 117 MB of 28 KiB rows
// 22.5 instead of 27.7, for the whole step a gain only where the operands are beyond the caches anyway (stream, see
// gecc_create); more loads in flight, 8-byte lanes, rows DMA'd into an LDS ring or workgroups that read 4 KiB of
// every row change nothing).  A lane keeps the column sums of its VEC columns in registers for the whole walk.
// The row sums of a block of rows (TS_RB rows x 2 kinds, one partial per lane) are transposed through
// LDS and added by four lanes per output; only the wavefront's own LDS region is involved, so no
// workgroup barrier sits in the loop.
constexpr int TS_THREADS = 256;
constexpr int TS_RB = 8;            // rows per block of loads
constexpr int TS_LDS_LD = 65;       // doubles per output row of the transpose (64 lanes + 1: conflict-free)

constexpr int TS_FLAG_AT = 1024;   // doubles into the LDS: behind what coldot_finish_segment uses

constexpr int TS_LDS_DOUBLES = 4 * 2 * TS_RB * TS_LDS_LD;

// segment `seg` of the columns, chunk `chunk` of the rows, batch item b; ts_lds: TS_LDS_DOUBLES of LDS
template <int DT, bool COL, bool ROW, bool COL_IDX, bool ROW_IDX>
__device__ __forceinline__ void tile_scan_body(const TileScanArgs& a, int seg, int chunk, int b, double* ts_lds) {
  using E = Elem<DT>;
  using T = typename E::type;
  constexpr int VEC = E::VEC;
  constexpr int SEG = 64 * VEC;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const T* X = reinterpret_cast<const T*>(a.X) + (int64_t)b * a.xs;
  // columns of this lane (Cc is a multiple of VEC; lanes past the end read the last vector and drop it)
  const int c_true = seg * SEG + lane * VEC;
  const bool lane_ok = c_true < a.Cc;
  const int c = lane_ok ? c_true : a.Cc - VEC;
  const T* col = X + c;
  // rows of this wavefront: a quarter of the chunk (multiple of TS_RB, so only the last has a tail)
  const int rbeg = chunk * a.chunk_rows;
  const int rend = min(a.R, rbeg + a.chunk_rows);
  const int quarter = a.chunk_rows >> 2;
  const int w_beg = min(rend, rbeg + wave * quarter), w_end = min(rend, w_beg + quarter);

  const double* wr0 = (COL && !COL_IDX) ? a.wr + (int64_t)b * a.wr_stride : nullptr;
  const double* wr1 = (COL && !COL_IDX) ? wr0 + a.R : nullptr;
  double wc0[VEC], wc1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    if (ROW && !ROW_IDX) {
      const double* w = a.wc + (int64_t)b * a.wc_stride;
      wc0[e] = w[c + e]; wc1[e] = w[a.Cc + c + e];
    } else {
      wc0[e] = 1.0; wc1[e] = (double)(c + e + 1);
    }
  }
  double ca0[VEC], ca1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) { ca0[e] = 0.0; ca1[e] = 0.0; }

  double* tr = ts_lds + wave * (2 * TS_RB * TS_LDS_LD);     // this wavefront's transpose region
  double* rp_out = ROW ? a.row_part + ((int64_t)b * a.R * a.nseg + seg) * 2 : nullptr;

  // one row into the column sums; its two row partials go straight into the transpose region
  auto take = [&](const typename E::raw& x, int u, double u0, double u1) {
    double v[VEC];
    E::widen(x, v);
    if (COL) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        ca0[e] = COL_IDX ? ca0[e] + v[e] : fma(u0, v[e], ca0[e]);
        ca1[e] = fma(u1, v[e], ca1[e]);
        // (pins the update to this row: left alone, the compiler keeps the widened values of all
        // the rows of a block alive and adds them up at the end, at the cost of half the occupancy)
        asm volatile("" : "+v"(ca0[e]), "+v"(ca1[e]));
      }
    }
    if (ROW) {
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        s0 = ROW_IDX ? s0 + v[e] : fma(wc0[e], v[e], s0);
        s1 = fma(wc1[e], v[e], s1);
      }
      tr[(2 * u) * TS_LDS_LD + lane] = lane_ok ? s0 : 0.0;
      tr[(2 * u + 1) * TS_LDS_LD + lane] = lane_ok ? s1 : 0.0;
    }
  };
  // row partials of `cnt` rows starting at r0: LDS -> four lanes per output add 16 lanes' values each
  auto emit_rows = [&](int r0, int cnt) {
    wave_lds_fence();
    const int o = lane >> 2, q = lane & 3;      // output (row u = o / 2, kind t = o % 2), quarter of the lanes
    // (all sixteen reads are issued before the first is used: one wait instead of eight)
    double part[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) part[i] = tr[o * TS_LDS_LD + q * 16 + i];
    __builtin_amdgcn_sched_barrier(0);
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += part[i];
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    wave_lds_fence();
    const int u = o >> 1, t = o & 1;
    if (q == 0 && u < cnt) {
      double* dst = rp_out + (int64_t)(r0 + u) * a.nseg * 2 + t;
      if (a.done_row) store_dev(dst, s); else *dst = s;
    }
  };

  int r = w_beg;
  const int nfull = (w_end - w_beg) / TS_RB;
  if (nfull > 0) {
    typename E::raw xa[TS_RB];
    auto load = [&](typename E::raw* x, int rr, auto stream) {
#pragma unroll
      for (int u = 0; u < TS_RB; ++u) {
        const T* src = col + (int64_t)(rr + u) * a.ld;
        x[u] = stream.value ? E::load_stream(src) : E::load_raw(src);
      }
    };
    auto work = [&](const typename E::raw* x, int rr) {
      // the row weights of the whole block first (uniform loads: one wait, not one per row)
      double u0[TS_RB], u1[TS_RB];
#pragma unroll
      for (int u = 0; u < TS_RB; ++u) {
        u0[u] = (COL && !COL_IDX) ? wr0[rr + u] : 1.0;
        u1[u] = (COL && !COL_IDX) ? wr1[rr + u] : (double)(rr + u + 1);
      }
#pragma unroll
      for (int u = 0; u < TS_RB; ++u) {
        take(x[u], u, u0[u], u1[u]);
        __builtin_amdgcn_sched_barrier(0);   // one row at a time: widening all of them first costs the occupancy
      }
      if (ROW) emit_rows(rr, TS_RB);
    };
    // (a loop for either kind of load: a branch around the loads alone would keep them from starting early)
    auto walk = [&](auto stream) {
      for (int bi = 0; bi < nfull; ++bi) {
        load(xa, r, stream);
        work(xa, r);
        r += TS_RB;
      }
    };
    if (a.stream) walk(std::true_type{});
    else walk(std::false_type{});
  }
  if (r < w_end) {     // the last rows of the operand: fewer than TS_RB
    const int cnt = w_end - r;
    for (int u = 0; u < TS_RB; ++u) {
      if (u < cnt) {
        take(E::load_raw(col + (int64_t)(r + u) * a.ld), u, (COL && !COL_IDX) ? wr0[r + u] : 1.0,
             (COL && !COL_IDX) ? wr1[r + u] : (double)(r + u + 1));
      } else if (ROW) {
        tr[(2 * u) * TS_LDS_LD + lane] = 0.0;
        tr[(2 * u + 1) * TS_LDS_LD + lane] = 0.0;
      }
    }
    if (ROW) emit_rows(r, cnt);
  }

  if (COL) {
    // the four quarters of the chunk, combined in order
    __syncthreads();
    double* cb = ts_lds;                          // [4][2 * VEC][64]
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      cb[(wave * 2 * VEC + e) * 64 + lane] = ca0[e];
      cb[(wave * 2 * VEC + VEC + e) * 64 + lane] = ca1[e];
    }
    __syncthreads();
    double* part = a.col_part + ((int64_t)b * a.nchunk + chunk) * 2 * a.Cc;
    for (int o = threadIdx.x; o < 2 * VEC * 64; o += TS_THREADS) {
      const int l = o & 63, e = (o >> 6) % VEC, t = o / (64 * VEC);
      const int cc = seg * SEG + l * VEC + e;
      if (cc < a.Cc) {
        const int x = (t * VEC + e) * 64 + l;
        const double v = (cb[x] + cb[2 * VEC * 64 + x]) + (cb[2 * 2 * VEC * 64 + x] + cb[3 * 2 * VEC * 64 + x]);
        if (a.done_col) store_dev(part + (int64_t)t * a.Cc + cc, v);
        else part[(int64_t)t * a.Cc + cc] = v;
      }
    }
  }

  if ((COL && a.done_col) || (ROW && a.done_row)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's partial results have been written through
    __syncthreads();
    int* flag = reinterpret_cast<int*>(ts_lds + TS_FLAG_AT);
    if (threadIdx.x == 0) {
      flag[0] = (COL && a.done_col) ? atomicInc(a.done_col + (int64_t)b * a.nseg + seg, (uint32_t)a.nchunk - 1) == (uint32_t)a.nchunk - 1 : 0;
      flag[1] = (ROW && a.done_row) ? atomicInc(a.done_row + (int64_t)b * a.nchunk + chunk, (uint32_t)a.nseg - 1) == (uint32_t)a.nseg - 1 : 0;
    }
    __syncthreads();
    const bool last_col = flag[0] != 0, last_row = flag[1] != 0;
    if (ROW && last_row) {
      const double* part = a.row_part + (int64_t)b * a.R * a.nseg * 2;
      double* out = a.row_out + (int64_t)b * a.row_out_stride;
      for (int rr = rbeg + (int)threadIdx.x; rr < rend; rr += TS_THREADS) rowseg_sum<true>(part, out, a.R, a.nseg, rr);
    }
    if (COL && last_col)
      coldot_finish_segment<VEC>(a.col_part + (int64_t)b * a.nchunk * 2 * a.Cc, a.col_out + (int64_t)b * a.col_out_stride,
                                 a.Cc, a.nchunk, seg * SEG, ts_lds);
  }
}

// -------------------------------------------------------------------------------------------
// The two gated re-encodings of the operand audit, as jobs of one launch (the decoder's, see
// decode_kernels.hip): every column reduction in here is finished by the workgroup that comes last to its
// segment (done / done_col / done_row set).
constexpr int PAIR_LDS_DOUBLES = TS_LDS_DOUBLES > CD_LDS_DOUBLES ? TS_LDS_DOUBLES : CD_LDS_DOUBLES;

// workgroup (x, y) of batch item b
template <int DT>
__device__ __forceinline__ void pair_body(const PairJob& j, int x, int y, int b, double* lds) {
  if (j.kind == PJ_ROW) rowdot_body<DT, true, RD_SMALL_RB, RD_SMALL_U>(j.s, x, b, lds);
  else if (j.kind == PJ_ROW_BIG) rowdot_body<DT, true, RD_BIG_RB, RD_BIG_U>(j.s, x, b, lds);
  else if (j.kind == PJ_ROW_WAVE) rowdot_wave_body<DT, true>(j.s, x, b, lds);
  else if (j.kind == PJ_COL) coldot_body<Elem<DT>, true, CD_ROWS, CD_CHUNKS>(j.s, Parts{}, j.gy, j.gx, x, y, b, lds);
  else if (j.kind == PJ_COL_HALF) coldot_body<ElemHalf<DT>, true, CD_ROWS, CD_CHUNKS>(j.s, Parts{}, j.gy, j.gx, x, y, b, lds);
  else if (j.kind == PJ_TILE_COL) tile_scan_body<DT, true, false, true, true>(j.t, x, y, b, lds);
  else tile_scan_body<DT, false, true, true, true>(j.t, x, y, b, lds);
}

}  // namespace
}  // namespace gecc
