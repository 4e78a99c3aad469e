// Section V on the device: syndromes from the per-tile partial sums, threshold tests, the
// correction rule for flagged rows/columns, and the operand audit that completes it for
// errors in A and B (each column of [A; A_P] and each row of [B B_P] is a codeword with two
// parity symbols, Section III).  All scalar decoding arithmetic is fp64; everything is
// stream-ordered and gated on state kept in device memory, so no host round trip is needed.
#include <type_traits>
#include "scan_device.h"

namespace gecc {
namespace {

struct Est { int i, j; double x, u; };

__device__ __forceinline__ DecodeState* state_of(const DecodeArgs& a, int b) { return a.state + b; }
__device__ __forceinline__ double* synd_of(const DecodeArgs& a, int b) {
  return a.synd + (int64_t)b * (2 * a.p.n + 2 * a.p.m);
}
__device__ __forceinline__ double* allow_of(const DecodeArgs& a, int b) {
  return a.allow + (int64_t)b * (2 * a.p.n + 2 * a.p.m);
}
__device__ __forceinline__ double* cpar_of(const DecodeArgs& a, int b) {
  return a.C_par + (int64_t)b * (2 * a.p.n + 2 * a.p.m + 4);
}

__device__ __forceinline__ double load_elem(const void* P, int dtype, int64_t idx) {
  if (dtype == GECC_BF16)
    return (double)__uint_as_float(((uint32_t) reinterpret_cast<const uint16_t*>(P)[idx]) << 16);
  return (double)reinterpret_cast<const float*>(P)[idx];
}
// round-to-nearest-even store into the operand's storage type
__device__ __forceinline__ void store_elem(void* P, int dtype, int64_t idx, double v) {
  const float f = (float)v;
  if (dtype == GECC_BF16) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    reinterpret_cast<uint16_t*>(P)[idx] = (uint16_t)(u >> 16);
  } else {
    reinterpret_cast<float*>(P)[idx] = f;
  }
}
// item b -> its row block I (A, A_P) and column block J (B, B_P); batch items: I = J = b
__device__ __forceinline__ int item_i(const DecodeArgs& a, int b) { return a.nbj ? b / a.nbj : b; }
__device__ __forceinline__ int item_j(const DecodeArgs& a, int b) { return a.nbj ? b % a.nbj : b; }
__device__ __forceinline__ int64_t a_index(const DecodeArgs& a, int b, int i, int l) {
  const gecc_params& p = a.p;
  return (int64_t)item_i(a, b) * a.ia_stride + (p.trans_a ? (int64_t)l * p.lda + i : (int64_t)i * p.lda + l);
}
__device__ __forceinline__ int64_t b_index(const DecodeArgs& a, int b, int l, int j) {
  const gecc_params& p = a.p;
  return (int64_t)item_j(a, b) * a.jb_stride + (p.trans_b ? (int64_t)j * p.ldb + l : (int64_t)l * p.ldb + j);
}
__device__ __forceinline__ float* c_of(const DecodeArgs& a, int b) {
  return a.C + (int64_t)item_i(a, b) * a.ic_stride + (int64_t)item_j(a, b) * a.jc_stride;
}
__device__ __forceinline__ const double* apar_of(const DecodeArgs& a, int b) { return a.A_par + (int64_t)item_i(a, b) * 2 * a.p.k; }
__device__ __forceinline__ const double* bpar_of(const DecodeArgs& a, int b) { return a.B_par + (int64_t)item_j(a, b) * 2 * a.p.k; }

// Section V step 1 clears a line when |sum - parity| <= threshold holds; anything else, a NaN
// included, flags it.
__device__ __forceinline__ bool outside(double v, double tau) { return !(fabs(v) <= tau); }
__device__ __forceinline__ bool finite2(double a, double b) { return isfinite(a) && isfinite(b); }
// maximum that keeps a NaN (fmax would drop it)
__device__ __forceinline__ double max_nan(double a, double b) { return (a != a || a > b) ? a : b; }

// -------------------------------------------------------------------------------------------
// partial sums -> syndromes (sum - parity, Section V step 1) -> flags
constexpr int TH_SLICES = 4;    // wavefronts of a workgroup; each adds every 4th sub-tile of a line

// TH_MAXLOADS: loads a thread keeps in flight, chosen by the launcher to fit the number of sub-tiles along a line
// (more than there are would only read the last one again: 256 x 512^3, four sub-tiles, 26 us with 32 of
// them, 9 with 4).  The sums do not depend on it.
// PARTS: pr and pc may hold something (kernels of their own, since the others pay 0.2 to 0.4 us for the question).
template <int TH_MAXLOADS, bool PARTS>
__device__ __forceinline__ void threshold_body(const DecodeArgs& a, const Parts& pr, const Parts& pc) {
  const int b = blockIdx.y;
  DecodeState* st = state_of(a, b);
  const int n = a.p.n, m = a.p.m;
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int o = blockIdx.x * 64 + lane;          // line: rows first, then columns
  const double* cpar = cpar_of(a, b);
  double* synd = synd_of(a, b);
  const bool is_row = o < n, valid = o < n + m;
  const bool wt = a.p.weighted != 0;     // single-checksum mode: the weighted sums are not read

  // Partial sums of this line over the sub-tiles slice, slice + 4, ... (fixed order), and its parity symbols.  All loads are
  // issued before the first is used (the kernel is a chain of latencies).
  const int len_o = is_row ? n : m, i_o = is_row ? o : o - n;      // the line among its kind
  const int at_o = is_row ? o : 2 * n + i_o;                        // its first parity symbol
  // (lanes past the last line read the last line's data and drop the result; sub-tiles past
  // the last one are clamped and count as zero: no load depends on a branch)
  const int oo = min(o, n + m - 1);
  const bool rowline = oo < n;
  const int nt = rowline ? a.ntn : a.ntm, len = rowline ? a.rp_ld : a.cp_ld, tile = rowline ? a.tile_n : a.tile_m;
  const float2* pp = rowline ? reinterpret_cast<const float2*>(a.rowpart) + (int64_t)b * a.ntn * a.rp_ld + oo
                             : reinterpret_cast<const float2*>(a.colpart) + (int64_t)b * a.ntm * a.cp_ld + (oo - n);
  float2 v[TH_MAXLOADS];
  auto load = [&](int t0) {
#pragma unroll
    for (int u = 0; u < TH_MAXLOADS; ++u) v[u] = pp[(int64_t)min(t0 + u * TH_SLICES, nt - 1) * len];
  };
  load(slice);
  // What the scans have left of this line's two parity symbols.  Chunks: a wavefront's slice is the second stage's own;
  // segments: one wavefront per kind.  (A second stage in a launch of its own costs 5 us for the same loads.)
  const Parts parts = {is_row ? pr.chunks : pc.chunks, is_row ? pr.segs : pc.segs, is_row ? pr.nchunk : pc.nchunk, is_row ? pr.nseg : pc.nseg};
  const bool in_parts = PARTS && (parts.nchunk > 0 || parts.nseg > 0);
  double stored[2] = {0.0, 0.0};
  if (slice == 0 && valid && !in_parts) { stored[0] = cpar[at_o]; stored[1] = cpar[at_o + len_o]; }
  __shared__ double par[PARTS ? 2 : 1][TH_SLICES][64];
  auto add_parts = [&] {
    if (PARTS && valid && in_parts) {
      if (parts.nchunk > 0) {
        const double* p0 = parts.chunks + (int64_t)b * parts.nchunk * 2 * len_o + i_o;
        const double* p[2] = {p0, p0 + len_o};
        double s[2];
        static_assert(TH_SLICES == 4, "slices of a column scan's second stage");
        slice_sums<2, false>(p, 2 * (int64_t)len_o, parts.nchunk, slice, s);
        par[0][slice][lane] = s[0];
        par[1][slice][lane] = s[1];
      } else if (slice < 2) {
        par[slice][0][lane] = parts_sum(parts, b, len_o, slice, i_o);
      }
    }
  };
  // (32 loads of a thread fill its registers and the memory system: then one after the other, 10.4 us and not 15 at 16384 x 14336)
  if (TH_MAXLOADS < 32) add_parts();
  double S = 0.0, W = 0.0;
  for (int t0 = slice; t0 < nt; t0 += TH_SLICES * TH_MAXLOADS) {
    if (t0 != slice) load(t0);
#pragma unroll
    for (int u = 0; u < TH_MAXLOADS; ++u) {
      const int t = t0 + u * TH_SLICES;
      const double x = t < nt ? (double)v[u].x : 0.0, y = t < nt ? (double)v[u].y : 0.0;
      S += x;
      W += y + (double)(t * tile) * x;
    }
  }
  if (TH_MAXLOADS >= 32) add_parts();
  __shared__ double red[2][TH_SLICES][64];
  red[0][slice][lane] = S;
  red[1][slice][lane] = W;
  __syncthreads();
  if (slice != 0) return;
  double v1 = 0.0, v2 = 0.0;
  if (valid) {
    if (PARTS && in_parts) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        stored[t] = parts.nchunk > 0 ? (par[t][0][lane] + par[t][1][lane]) + (par[t][2][lane] + par[t][3][lane]) : par[t][0][lane];
        const_cast<double*>(cpar)[at_o + t * len_o] = stored[t];
      }
    }
    S = (red[0][0][lane] + red[0][1][lane]) + (red[0][2][lane] + red[0][3][lane]);
    W = (red[1][0][lane] + red[1][1][lane]) + (red[1][2][lane] + red[1][3][lane]);
    if (is_row) {
      const int i = o;
      v1 = S - stored[0];
      v2 = W - stored[1];
      synd[i] = v1;
      synd[n + i] = v2;
      if (outside(v1, a.p.tau_r1) || (wt && outside(v2, a.p.tau_r2))) {
        const int idx = atomicAdd(&st->s_cnt, 1);
        if (idx < GECC_MAX_ERR) st->rows[idx] = i;
      }
    } else {
      const int j = o - n;
      v1 = S - stored[0];
      v2 = W - stored[1];
      synd[2 * n + j] = v1;
      synd[2 * n + m + j] = v2;
      if (outside(v1, a.p.tau_q1) || (wt && outside(v2, a.p.tau_q2))) {
        const int idx = atomicAdd(&st->t_cnt, 1);
        if (idx < GECC_MAX_ERR) st->cols[idx] = j;
      }
    }
    if (!wt) v2 = 0.0;
    if (!finite2(v1, v2)) atomicOr(&st->nonfinite, 1);
  }
  {
    // family maxima of this workgroup (rows: [0], [1]; columns: [2], [3]); the summary reduces
    // them (atomics on one line from every workgroup would serialise in L2)
    double mr1 = (valid && is_row) ? fabs(v1) : 0.0, mr2 = (valid && is_row) ? fabs(v2) : 0.0;
    double mq1 = (valid && !is_row) ? fabs(v1) : 0.0, mq2 = (valid && !is_row) ? fabs(v2) : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      mr1 = max_nan(mr1, __shfl_down(mr1, off, 64));
      mr2 = max_nan(mr2, __shfl_down(mr2, off, 64));
      mq1 = max_nan(mq1, __shfl_down(mq1, off, 64));
      mq2 = max_nan(mq2, __shfl_down(mq2, off, 64));
    }
    if (lane == 0) {
      double* bm = a.blockmax + ((int64_t)b * gridDim.x + blockIdx.x) * 4;
      bm[0] = mr1; bm[1] = mr2; bm[2] = mq1; bm[3] = mq2;
    }
  }
}

template <int TH_MAXLOADS>
__global__ __launch_bounds__(64 * TH_SLICES) void threshold_kernel(DecodeArgs a) { threshold_body<TH_MAXLOADS, false>(a, Parts{}, Parts{}); }
template <int TH_MAXLOADS>
__global__ __launch_bounds__(64 * TH_SLICES) void threshold_parts_kernel(DecodeArgs a, Parts pr, Parts pc) { threshold_body<TH_MAXLOADS, true>(a, pr, pc); }

// first report after detection: CLEAN or DETECTED.  Called by every thread of a workgroup of 1, 2 or 4 wavefronts, which
// share the four families out; returns the status to all of them.  if_clean: nothing is written unless it is CLEAN.  (No
// barrier, and the maxima do not wait for the counters: it is all that a clean product's last but one launch does, which
// with one wait after the other took 3.8 us and takes 2.0.)
__device__ __forceinline__ int summarize(const DecodeArgs& a, int b, const DecodeState* st, gecc_report* rep, bool if_clean = false) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const double* bm = a.blockmax + (int64_t)b * a.nblk * 4;
  const int sc = st->s_cnt, tc = st->t_cnt;
  for (int f = wave; f < 4; f += nw) {
    double mx = 0.0;
    for (int i0 = lane; i0 < a.nblk; i0 += 4 * 64) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = bm[(int64_t)min(i0 + 64 * u, a.nblk - 1) * 4 + f];
#pragma unroll
      for (int u = 0; u < 4; ++u) mx = max_nan(mx, v[u]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max_nan(mx, __shfl_down(mx, off, 64));
    if (lane == 0 && (!if_clean || (sc == 0 && tc == 0))) rep->max_abs_synd[f] = mx;
  }
  const int status = (sc == 0 && tc == 0) ? GECC_CLEAN : GECC_DETECTED;
  if (threadIdx.x == 0 && (!if_clean || status == GECC_CLEAN)) {
    rep->s = sc;
    rep->t = tc;
    rep->n_err = 0;
    rep->n_total = 0;
    rep->reserved = 0;
    rep->status = status;
  }
  return status;
}
__global__ __launch_bounds__(256) void summarize_kernel(DecodeArgs a) {   // four wavefronts per item
  const int b = blockIdx.x;
  summarize(a, b, state_of(a, b), a.report + b);
}

// ---- Section V step 2 ------------------------------------------------------------------------
// The decoder's workgroup-wide routines below are written for exactly DC_THREADS threads
// (threadIdx.x < DC_THREADS; a larger workgroup lets its other wavefronts end first).
constexpr int DC_THREADS = 256;

struct Synd {
  const double *r1, *r2, *q1, *q2;
  double b_r1, b_r2, b_q1, b_q2;            // thresholds of the four families
  const double *a_r1, *a_r2, *a_q1, *a_q2;  // per-line allowances
  double rel;                               // relative rounding allowance of a syndrome value
  bool wt;                                  // false: single-checksum mode, r2 / q2 are not read
  // how far each syndrome value is trusted when an estimate is verified
  __device__ double tr1(int i) const { return b_r1 + a_r1[i] + rel * fabs(r1[i]); }
  __device__ double tr2(int i) const { return b_r2 + a_r2[i] + rel * fabs(r2[i]); }
  __device__ double tq1(int j) const { return b_q1 + a_q1[j] + rel * fabs(q1[j]); }
  __device__ double tq2(int j) const { return b_q2 + a_q2[j] + rel * fabs(q2[j]); }
};

// The syndromes of the flagged lines alone: kind 0 and 1 of a line and how far each is trusted, rows [0], columns [1], in the
// order of Er and Et
struct FlagSynd {
  double v[2][2][2];                        // [rows, columns][line][kind]
  double tr[2][2][2];
  bool wt;
};

// every syndrome of a flagged line has to be explained by the estimate, within the thresholds
// widened by the uncertainty the estimate itself carries
__device__ bool residual_ok(const Est* est, int ne, const int* Er, int s, const int* Et, int t,
                            const FlagSynd& y) {
#pragma unroll 1
  for (int x = 0; x < s + t; ++x) {
    const bool row = x < s;
    const int c = row ? x : x - s, line = row ? Er[c] : Et[c];
    double sx = 0, su = 0, wx = 0, wu = 0;
#pragma unroll 1
    for (int e = 0; e < ne; ++e)
      if ((row ? est[e].i : est[e].j) == line) {
        const double w = (double)((row ? est[e].j : est[e].i) + 1);
        sx += est[e].x; su += est[e].u;
        wx += w * est[e].x; wu += w * est[e].u;
      }
    const double *v = y.v[row ? 0 : 1][c], *tr = y.tr[row ? 0 : 1][c];
    if (fabs(v[0] - sx) > tr[0] + su) return false;
    if (y.wt && fabs(v[1] - wx) > tr[1] + wu) return false;
  }
  return true;
}

// drops insignificant parts, verifies, sorts by (i, j).  Returns the count or -1.
__device__ int accept(Est* est, int ne, const int* Er, int s, const int* Et, int t, const FlagSynd& y) {
  int k = 0;
  for (int e = 0; e < ne; ++e)
    if (fabs(est[e].x) > est[e].u) est[k++] = est[e];
  if (!residual_ok(est, k, Er, s, Et, t, y)) return -1;
  for (int x = 1; x < k; ++x) {
    const Est key = est[x];
    int z = x - 1;
    while (z >= 0 && (est[z].i > key.i || (est[z].i == key.i && est[z].j > key.j))) {
      est[z + 1] = est[z];
      --z;
    }
    est[z + 1] = key;
  }
  return k;
}

// Correction rule for 1 <= s, t <= 2 (s <= t: columns carry the information; s > t mirrored).  By one thread
// of the workgroup; Er, Et and out are in LDS like the estimates here (indexed at run time, they would put
// a quarter of a KiB of scratch under every thread of the kernel).
__device__ __noinline__ int d0_correct(Est* out, const int* Er, int s, const int* Et, int t, const FlagSynd& y) {
  __shared__ Est est[4], dg[4], an[4];
  const int few = s <= t ? s : t;
  if (few == 1) {
    // one line of one kind: each line of the other kind (columns, where there is one of each) holds one error
    const bool row = s <= t;
    const int many = row ? t : s;
    for (int c = 0; c < many; ++c)
      est[c] = Est{row ? Er[0] : Er[c], row ? Et[c] : Et[0], y.v[row ? 1 : 0][c][0], y.tr[row ? 1 : 0][c][0]};
    const int k = accept(est, many, Er, s, Et, t, y);
    for (int e = 0; e < k; ++e) out[e] = est[e];
    return k;
  }
  const int s1 = Er[0], s2 = Er[1];
  for (int c = 0; c < 2; ++c) {
    dg[c] = Est{Er[c], Et[c], y.v[1][c][0], y.tr[1][c][0]};
    an[c] = Est{Er[c], Et[1 - c], y.v[1][1 - c][0], y.tr[1][1 - c][0]};
  }
  const int kd = accept(dg, 2, Er, s, Et, t, y);
  const int ka = accept(an, 2, Er, s, Et, t, y);
  if (kd >= 0 && ka >= 0) return -1;   // cannot tell the two apart
  if (kd >= 0) { for (int e = 0; e < kd; ++e) out[e] = dg[e]; return kd; }
  if (ka >= 0) { for (int e = 0; e < ka; ++e) out[e] = an[e]; return ka; }
  const double w1 = s1 + 1.0, w2 = s2 + 1.0;
  int ne = 0;
  for (int c = 0; c < 2; ++c) {
    const int j = Et[c];
    const double q1 = y.v[1][c][0], q2 = y.v[1][c][1], t1 = y.tr[1][c][0], t2 = y.tr[1][c][1];
    const double e2 = (q2 - w1 * q1) / (w2 - w1);
    const double e1 = q1 - e2;
    const double u2 = (t2 + w1 * t1) / (w2 - w1);
    const double u1 = t1 + u2;
    est[ne++] = Est{s1, j, e1, u1};
    est[ne++] = Est{s2, j, e2, u2};
  }
  const int k = accept(est, ne, Er, s, Et, t, y);
  for (int e = 0; e < k; ++e) out[e] = est[e];
  return k;
}

// fp64 dot product of row i of A with column j of B over the terms l_beg .. l_end, by the whole workgroup
__device__ double block_dot(const DecodeArgs& a, int b, int i, int j, int l_beg, int l_end, double* red) {
  double s = 0.0;
  constexpr int U = 8;   // products per thread whose loads are issued together (one workgroup: latency-bound)
  for (int l0 = l_beg + (int)threadIdx.x; l0 < l_end; l0 += U * DC_THREADS) {
    double x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int l = min(l0 + u * DC_THREADS, l_end - 1);
      x[u] = load_elem(a.A, a.p.dtype, a_index(a, b, i, l));
      y[u] = load_elem(a.B, a.p.dtype, b_index(a, b, l, j));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (l0 + u * DC_THREADS < l_end) s = fma(x[u], y[u], s);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = DC_THREADS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// a lane's terms of that product over l_beg .. l_end, by one wavefront
__device__ double wave_dot(const DecodeArgs& a, int b, int i, int j, int l_beg, int l_end) {
  double s = 0.0;
  constexpr int U = 8;
  for (int l0 = l_beg + (int)(threadIdx.x & 63); l0 < l_end; l0 += U * 64) {
    double x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int l = min(l0 + u * 64, l_end - 1);
      x[u] = load_elem(a.A, a.p.dtype, a_index(a, b, i, l));
      y[u] = load_elem(a.B, a.p.dtype, b_index(a, b, l, j));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (l0 + u * 64 < l_end) s = fma(x[u], y[u], s);
  }
  return s;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Theorem 2 (Appendix B): min(s, t) <= 2 < max(s, t).  The at most two flagged lines of the
// short side are the known lines; every flagged line c of the other kind is decoded on its own
// from its two syndromes (one known line: e = y1_c; two: the 2x2 system of Section V), the
// estimates are verified against every flagged line like those of d0_correct, and Section V's
// subtraction is applied.  All threads of the workgroup take part: thread x owns a contiguous
// chunk of the other-kind lines.  Returns the number of corrected symbols, or -1.
struct LineEst { double x[2], u[2]; bool sig[2], flagged; };

// pool: POOL_DOUBLES of LDS
constexpr int POOL_DOUBLES = 2048 + 256;
__device__ int known_lines_correct(const DecodeArgs& a, int b, DecodeState* st, gecc_report* rep,
                                   const Synd& y, double* pool) {
  const int n = a.p.n, m = a.p.m;
  const int s = st->s_cnt, t = st->t_cnt;
  const bool rows_known = a.p.weighted ? s <= 2 : s == 1;
  const int nk = rows_known ? s : t;
  const int L = rows_known ? m : n;
  int K[2] = {0, 0};
  for (int q = 0; q < nk; ++q) K[q] = rows_known ? st->rows[q] : st->cols[q];
  if (nk == 2 && K[0] > K[1]) { const int z = K[0]; K[0] = K[1]; K[1] = z; }
  const double w1 = K[0] + 1.0, w2 = K[1] + 1.0;
  const double *y1 = rows_known ? y.q1 : y.r1, *y2 = rows_known ? y.q2 : y.r2;
  const double b1 = rows_known ? y.b_q1 : y.b_r1, b2 = rows_known ? y.b_q2 : y.b_r2;
  const double *a1 = rows_known ? y.a_q1 : y.a_r1, *a2 = rows_known ? y.a_q2 : y.a_r2;

  auto estimate = [&](int c) {
    LineEst e;
    e.flagged = fabs(y1[c]) > b1 + a1[c] || (y.wt && fabs(y2[c]) > b2 + a2[c]);
    e.sig[0] = e.sig[1] = false; e.x[0] = e.x[1] = e.u[0] = e.u[1] = 0.0;
    if (!e.flagged) return e;
    const double u1 = rows_known ? y.tq1(c) : y.tr1(c), u2 = rows_known ? y.tq2(c) : y.tr2(c);
    if (nk == 1) {
      e.x[0] = y1[c]; e.u[0] = u1;
    } else {
      e.x[1] = (y2[c] - w1 * y1[c]) / (w2 - w1);
      e.x[0] = y1[c] - e.x[1];
      e.u[1] = (u2 + w1 * u1) / (w2 - w1);
      e.u[0] = u1 + e.u[1];
    }
    for (int q = 0; q < nk; ++q) e.sig[q] = fabs(e.x[q]) > e.u[q];   // insignificant parts are dropped
    return e;
  };

  double (*t2_red)[256] = reinterpret_cast<double (*)[256]>(pool);             // [8][256]
  int (*t2_cnt)[256] = reinterpret_cast<int (*)[256]>(pool + 2048);             // [2][256]
  __shared__ int t2_bad;
  const int tid = threadIdx.x, ch = (L + DC_THREADS - 1) / DC_THREADS;
  const int c0 = min(L, tid * ch), c1 = min(L, c0 + ch);
  if (tid == 0) t2_bad = 0;
  __syncthreads();
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // per known line: sum x, sum u, weighted sum x, weighted sum u
  int cnt[2] = {0, 0};
  bool bad = false;
  for (int c = c0; c < c1; ++c) {
    const LineEst e = estimate(c);
    if (!e.flagged) continue;
    // this line's own two syndromes
    double sx = 0, su = 0, wx = 0, wu = 0;
    for (int q = 0; q < nk; ++q)
      if (e.sig[q]) {
        const double w = K[q] + 1.0;
        sx += e.x[q]; su += e.u[q]; wx += w * e.x[q]; wu += w * e.u[q];
        acc[4 * q + 0] += e.x[q]; acc[4 * q + 1] += e.u[q];
        acc[4 * q + 2] += (c + 1.0) * e.x[q]; acc[4 * q + 3] += (c + 1.0) * e.u[q];
        ++cnt[q];
      }
    const double u1 = rows_known ? y.tq1(c) : y.tr1(c), u2 = rows_known ? y.tq2(c) : y.tr2(c);
    bad = bad || fabs(y1[c] - sx) > u1 + su || (y.wt && fabs(y2[c] - wx) > u2 + wu);
  }
  for (int q = 0; q < 8; ++q) t2_red[q][tid] = acc[q];
  t2_cnt[0][tid] = cnt[0]; t2_cnt[1][tid] = cnt[1];
  if (bad) t2_bad = 1;
  __syncthreads();
  if (tid == 0) {
    // the known lines' own syndromes against everything attributed to them
    for (int q = 0; q < nk; ++q) {
      double v[4] = {0, 0, 0, 0};
      for (int x = 0; x < DC_THREADS; ++x)
        for (int f = 0; f < 4; ++f) v[f] += t2_red[4 * q + f][x];
      const int line = K[q];
      const double z1 = rows_known ? y.r1[line] : y.q1[line], z2 = rows_known ? y.r2[line] : y.q2[line];
      const double tz1 = rows_known ? y.tr1(line) : y.tq1(line), tz2 = rows_known ? y.tr2(line) : y.tq2(line);
      if (fabs(z1 - v[0]) > tz1 + v[1] || (y.wt && fabs(z2 - v[2]) > tz2 + v[3])) t2_bad = 1;
    }
  }
  __syncthreads();
  if (t2_bad) return -1;
  // position of this thread's entries in the list sorted by (row, column)
  int before[2] = {0, 0}, total[2] = {0, 0};
  for (int x = 0; x < DC_THREADS; ++x)
    for (int q = 0; q < 2; ++q) {
      if (x < tid) before[q] += t2_cnt[q][x];
      total[q] += t2_cnt[q][x];
    }
  const int ne0 = st->n_err;                  // operand errors of the audit come first
  int idx[2];
  if (rows_known) { idx[0] = before[0]; idx[1] = total[0] + before[1]; }     // row K0 first, then row K1
  else            { idx[0] = idx[1] = before[0] + before[1]; }               // row by row
  float* C = c_of(a, b);
  for (int c = c0; c < c1; ++c) {
    const LineEst e = estimate(c);
    if (!e.flagged) continue;
    for (int q = 0; q < nk; ++q)
      if (e.sig[q]) {
        const int i = rows_known ? K[q] : c, j = rows_known ? c : K[q];
        const int64_t ic = (int64_t)i * a.p.ldc + j;
        C[ic] = (float)((double)C[ic] - e.x[q]);
        const int pos = ne0 + (rows_known ? idx[q]++ : idx[0]++);
        if (pos < GECC_MAX_ERR) {
          gecc_err g;
          g.matrix = GECC_MAT_C; g.row = i; g.col = j; g.reserved = 0; g.magnitude = e.x[q];
          rep->err[pos] = g;
        }
      }
  }
  return total[0] + total[1];
}

// What Section V step 2 makes of the flagged lines: thread 0 fills fix[0 .. *nfix); *nfix = -1: the rule does
// not apply or failed.  By all threads of the workgroup (the flagged lines' syndromes are loaded side by side, past the caches:
// other workgroups of the launch may have written them), which meet at a barrier before they read fix and *nfix.
__device__ void plan_fixes(const DecodeArgs& a, int b, int s, int t, const int* rows, const int* cols, int final_pass, Est* fix, int* nfix) {
  const int n = a.p.n, m = a.p.m;
  if (!(s >= 1 && s <= 2 && t >= 1 && t <= 2 && (a.p.weighted || (s == 1 && t == 1)))) {
    if (threadIdx.x == 0) *nfix = s == 0 && t == 0 ? 0 : -1;
    return;
  }
  __shared__ int E[2][2];
  __shared__ FlagSynd y;
  if (threadIdx.x < 8) {
    const int col = threadIdx.x >> 2, at = (threadIdx.x >> 1) & 1, kind = threadIdx.x & 1;
    const int cnt = col ? t : s, *list = col ? cols : rows;
    if (at < cnt) {
      const int x0 = list[0], x1 = list[cnt - 1], line = at == 0 ? min(x0, x1) : max(x0, x1);
      const int64_t idx = (col ? 2 * (int64_t)n : 0) + (kind ? (col ? m : n) : 0) + line;
      const double v = load_dev(synd_of(a, b) + idx), al = final_pass ? load_dev(allow_of(a, b) + idx) : 0.0;
      const double tau = col ? (kind ? a.p.tau_q2 : a.p.tau_q1) : (kind ? a.p.tau_r2 : a.p.tau_r1);
      y.v[col][at][kind] = v;
      y.tr[col][at][kind] = tau + al + a.p.tau_rel * fabs(v);
      E[col][at] = line;
    }
    if (threadIdx.x == 0) y.wt = a.p.weighted != 0;
  }
  __syncthreads();
  if (threadIdx.x == 0) *nfix = d0_correct(fix, E[0], s, E[1], t, y);
}

__device__ void give_up(DecodeState* st, gecc_report* rep) {
  rep->status = GECC_UNCORRECTABLE;
  rep->n_err = 0;
  rep->n_total = 0;
  st->phase = PH_DONE;
}

// patch C: Section V's subtraction, or the symbol evaluated again (dots: what block_dot gives for every fix, or
// null: by this workgroup); then the report
__device__ void apply_fixes(const DecodeArgs& a, int b, DecodeState* st, gecc_report* rep, const Est* fix, int k, double* pool,
                            const double* dots) {
  float* C = c_of(a, b);
  for (int e = 0; e < k; ++e) {
    const int64_t idx = (int64_t)fix[e].i * a.p.ldc + fix[e].j;
    if (a.p.refine) {
      const double d = dots ? dots[e] : block_dot(a, b, fix[e].i, fix[e].j, 0, a.p.k, pool);
      if (threadIdx.x == 0) C[idx] = (float)d;
    } else if (threadIdx.x == 0) {
      C[idx] = (float)((double)load_dev(C + idx) - fix[e].x);
    }
  }
  if (threadIdx.x == 0) {
    int ne = 0;
    for (int e = 0; e < st->n_err; ++e) rep->err[ne++] = st->errs[e];   // A then B, sorted (at most 8)
    const int total = ne + k;
    for (int e = 0; e < k && ne < GECC_MAX_ERR; ++e) {
      gecc_err g;
      g.matrix = GECC_MAT_C; g.row = fix[e].i; g.col = fix[e].j; g.reserved = 0;
      g.magnitude = fix[e].x;
      rep->err[ne++] = g;
    }
    rep->n_total = total;
    rep->n_err = ne;
    rep->status = GECC_CORRECTED;
    st->phase = PH_DONE;
  }
}

// Section V step 2 for one batch item, by DC_THREADS threads.  final_pass = 0: right after
// detection; = 1: on the residual syndromes after an operand repair (per-line allowances apply,
// failure is final).  pool: POOL_DOUBLES of LDS
__device__ void decode_c_body(const DecodeArgs& a, int b, DecodeState* st, gecc_report* rep, int final_pass, double* pool) {
  __shared__ Est fix[4];
  __shared__ int nfix;
  const int n = a.p.n, m = a.p.m;
  if (st->nonfinite) {
    // a syndrome that is not a number: no estimate can be subtracted, the product is computed again
    if (threadIdx.x == 0) give_up(st, rep);
    return;
  }
  {
    const int s = st->s_cnt, t = st->t_cnt, lo = min(s, t), hi = max(s, t);
    // Theorem 2: many lines of one kind, at most two of the other.  Its errors all lie in C-bar,
    // so it runs only after the operand audit (on what the repair leaves, or on the whole pattern
    // when both operands are intact): a wrong symbol of A a few rows from a flagged row would
    // otherwise pass for a row full of small errors of C.
    // (single-checksum mode: one known line only, any number of the other kind -- Appendix A, case s = 1)
    if (final_pass && (a.p.weighted ? (lo >= 1 && lo <= 2 && hi > 2) : (lo == 1 && hi >= 2))) {
      // (the launch's other workgroups have written through what this reads, by all of its lines)
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const double* sy = synd_of(a, b);
      const double* al = allow_of(a, b);
      const Synd y{sy, sy + n, sy + 2 * n, sy + 2 * n + m, a.p.tau_r1, a.p.tau_r2, a.p.tau_q1, a.p.tau_q2,
                   al, al + n, al + 2 * n, al + 2 * n + m, a.p.tau_rel, a.p.weighted != 0};
      const int k = known_lines_correct(a, b, st, rep, y, pool);
      if (threadIdx.x == 0) {
        if (k < 0) {
          give_up(st, rep);
        } else {
          for (int e = 0; e < st->n_err; ++e) rep->err[e] = st->errs[e];
          rep->n_total = st->n_err + k;
          rep->n_err = min(rep->n_total, GECC_MAX_ERR);
          rep->status = GECC_CORRECTED;
          st->phase = PH_DONE;
        }
      }
      return;
    }
  }
  plan_fixes(a, b, st->s_cnt, st->t_cnt, st->rows, st->cols, final_pass, fix, &nfix);
  __syncthreads();
  const int k = nfix;
  if (k < 0) {
    if (threadIdx.x == 0) {
      if (final_pass) give_up(st, rep);
      else            { st->phase = PH_AUDIT; if (a.gate_word) *a.gate_word = PH_AUDIT; }
    }
    return;
  }
  apply_fixes(a, b, st, rep, fix, k, pool, nullptr);
}

// One workgroup per batch item, right after detection.  with_summary: this kernel also writes
// the first report (saves the summary launch).
__global__ __launch_bounds__(DC_THREADS) void decode_c_kernel(DecodeArgs a, int with_summary) {
  const int b = blockIdx.x;
  DecodeState* st = state_of(a, b);
  gecc_report* rep = a.report + b;
  if (with_summary) {
    if (summarize(a, b, st, rep) == GECC_CLEAN) return;
  } else {
    if (rep->status != GECC_DETECTED) return;
  }
  __shared__ double pool[DC_THREADS];     // (no Theorem 2 in this pass)
  decode_c_body(a, b, st, rep, 0, pool);
}

// ---- operand audit -----------------------------------------------------------------------------
// A single wrong symbol of a line (column l of A, row l of B) shows as (u1, u2) = (e, (pos+1) e)
// in the difference of re-formed and stored parities.
__device__ __forceinline__ AuditHit located(double u1, double u2, int l, int len, double tau) {
  AuditHit h;
  h.line = l; h.pos = -1; h.e = u1;
  if (fabs(u1) > tau && finite2(u1, u2)) {
    const double rho = u2 / u1, w = rint(rho);
    if (fabs(rho - w) < 0.25 && w >= 1.0 && w <= (double)len) h.pos = (int)w - 1;
  }
  return h;
}

__device__ void sort_hits(AuditHit* h, int cnt) {
  for (int x = 1; x < cnt; ++x) {
    const AuditHit key = h[x];
    int y = x - 1;
    while (y >= 0 && h[y].line > key.line) { h[y + 1] = h[y]; --y; }
    h[y + 1] = key;
  }
}

// Remove the rank-one footprint of every audit hit from C-bar, then patch the operands.
// Order (it absorbs the cross term when an A hit and a B hit share the index l): rows of the
// A hits first, using B as the product read it; then columns of the B hits, using the
// corrected A.
//
// Several workgroups share an item (how many: repair_wgs): each owns a slice of the columns (threads 0 .. RP_LINES - 1)
// and a slice of the rows (the others), finds the hits for itself and takes every hit's footprint out of its own lines.
// What concerns a hit's own line (its sums over all slices) and the symbols where the row of an A hit meets the column
// of a B hit is left to the workgroup that comes last; it also puts the operands right, which the others read until then.
//
// What bounds it: a column of C or of A is a line of memory per row, and one compute unit keeps a few dozen of them on
// their way.  Between event pairs, one workgroup -> sixteen at 4096^3 bf16: an error of A 28.3 -> 20.5 us, of B
// 49.4 -> 21.5, of both 53.3 -> 24.4; 256 items of 512^3 fp32 keep one workgroup each, 35.6 -> 32.0, since a load then
// waits for another and not for its turn.  What is left is that chain, and where a symbol of C is evaluated again the
// 4096 lines of a column of B by one compute unit (15 us).
constexpr int RP_LINES = 256;
constexpr int RP_THREADS = 2 * RP_LINES;
constexpr int RP_WGS = 64;         // workgroups of an item, at most
struct RepairRecord {              // what a workgroup leaves to the last one
  double sums[GECC_MAX_ERR][4];    // per hit: its footprint's squares, plain and weighted, and what the line's two sums lose
  int32_t s, t, bad, reserved;     // lines of its slices that are still flagged; some of them not finite
  int32_t rows[GECC_MAX_ERR], cols[GECC_MAX_ERR];
};

// SPLIT (blocked mode: several blocks share an operand line): this launch leaves the operands alone
// and stops before Section V's second pass; patch_operands_kernel and final_decode_kernel follow.
constexpr int RP_U = 2;            // lines a thread has in flight
template <int DT, bool SPLIT>
__global__ __launch_bounds__(RP_THREADS) void repair_kernel(DecodeArgs a, RepairRecord* records, uint32_t* done, int wgs) {
  const int b = blockIdx.x / wgs, w = blockIdx.x % wgs;
  DecodeState* st = state_of(a, b);
  if (st->phase != PH_AUDIT) return;
  gecc_report* rep = a.report + b;
  __shared__ double pool[POOL_DOUBLES];
  __shared__ int ok, cnt_a, cnt_b, flag;
  __shared__ AuditHit hit[2 * GECC_MAX_ERR];           // of A, then of B
  __shared__ double own[GECC_MAX_ERR][5];              // per hit: its line's two syndromes, the parities it meets, the wrong symbol
  __shared__ double cross[GECC_MAX_ERR * GECC_MAX_ERR / 4][3];   // where A hit x meets B hit y: C, the symbols of B and of A
  __shared__ RepairRecord mine;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.p.n, m = a.p.m, k = a.p.k;
  AuditHit *ha = hit, *hb = hit + GECC_MAX_ERR;
  if (tid == 0) { cnt_a = 0; cnt_b = 0; mine.s = 0; mine.t = 0; mine.bad = 0; }
  __syncthreads();
  {   // difference of the re-formed and the stored operand parities, line by line
    const double* cur_a = a.audit_a + (int64_t)item_i(a, b) * 2 * k;
    const double* cur_b = a.audit_b + (int64_t)item_j(a, b) * 2 * k;
    const double* ref_a = apar_of(a, b);
    const double* ref_b = bpar_of(a, b);
    const bool wt = a.p.weighted != 0;
    constexpr int U = 2;
    for (int l0 = tid; l0 < k; l0 += U * RP_THREADS) {
      double d[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int l = min(l0 + u * RP_THREADS, k - 1);
        d[u][0] = cur_a[l] - ref_a[l]; d[u][1] = cur_a[k + l] - ref_a[k + l];
        d[u][2] = cur_b[l] - ref_b[l]; d[u][3] = cur_b[k + l] - ref_b[k + l];
      }
#pragma unroll 1
      for (int x = 0; x < 2 * U; ++x) {
        const int l = l0 + (x >> 1) * RP_THREADS;
        const double u1 = x == 0 ? d[0][0] : x == 1 ? d[0][2] : x == 2 ? d[1][0] : d[1][2];
        const double u2 = x == 0 ? d[0][1] : x == 1 ? d[0][3] : x == 2 ? d[1][1] : d[1][3];
        if (l < k && (outside(u1, a.p.tau_op) || (wt && outside(u2, a.p.tau_op)))) {
          const int idx = atomicAdd(x & 1 ? &cnt_b : &cnt_a, 1);
          if (idx < GECC_MAX_ERR) hit[(x & 1) * GECC_MAX_ERR + idx] = located(u1, u2, l, x & 1 ? m : n, a.p.tau_op);
        }
      }
    }
  }
  __syncthreads();
  const int na = cnt_a, nb = cnt_b;
  if (tid == 0) {
    ok = na + nb <= GECC_MAX_ERR;       // no hit at all: the pattern lies in C-bar alone (second pass below)
    // single-checksum mode: one parity names the line of a wrong operand symbol, not its place in it
    if (!a.p.weighted && na + nb > 0) ok = 0;
    if (ok) {
      for (int x = 0; x < na; ++x) if (ha[x].pos < 0) ok = 0;
      for (int x = 0; x < nb; ++x) if (hb[x].pos < 0) ok = 0;
    }
    if (ok) { sort_hits(ha, na); sort_hits(hb, nb); }
  }
  __syncthreads();
  if (!ok) {
    // (every workgroup comes to this; the last one says so, when none is left that has not read the phase)
    const bool last = wgs == 1 || arrive_last(done + b, (uint32_t)wgs, &flag);
    if (last && tid == 0) give_up(st, rep);
    return;
  }
  float* C = c_of(a, b);
  double* cpar = cpar_of(a, b);
  // threshold allowances of the lines a repair touches (rounding noise of the corrupted terms)
  double* al_r1 = allow_of(a, b);
  const double cc = a.p.tau_rep * sqrt((double)k);
  // residual syndromes: every repair below also moves the syndromes by exactly what it changes
  // (the stored symbols' differences and the parity symbols), so that Section V can run again
  // without another pass over C
  double* sy_r1 = synd_of(a, b);
  const bool wt = a.p.weighted != 0;
  auto elem = [](const void* P, int64_t idx) { return load_elem(P, DT, idx); };
  // Section V step 1 on a residual line (threshold widened by the allowance); the first of them go on the list
  auto test = [&](bool is_row, int o, double y1, double y2, double g1, double g2) {
    if (outside(y1, (is_row ? a.p.tau_r1 : a.p.tau_q1) + g1) || (wt && outside(y2, (is_row ? a.p.tau_r2 : a.p.tau_q2) + g2))) {
      const int idx = atomicAdd(is_row ? &mine.s : &mine.t, 1);
      if (idx < GECC_MAX_ERR) (is_row ? mine.rows : mine.cols)[idx] = o;
    }
    if (!finite2(y1, wt ? y2 : 0.0)) mine.bad = 1;
  };
  // whether line o is the row of an A hit (the column of a B hit)
  auto own_line = [&](bool is_row, int o) {
    bool is = false;
    for (int x = 0; x < (is_row ? na : nb); ++x) is = is || (is_row ? ha : hb)[x].pos == o;
    return is;
  };
  auto hit_at = [&](int z) -> const AuditHit& { return z < na ? ha[z] : hb[z - na]; };
  // What only the last workgroup needs, but nobody changes before it: loaded here, where the loads of the lines are in flight as well
  double pre[5];
  const bool pre_own = tid < na + nb, pre_cross = tid >= 64 && tid < 64 + na * nb;
  if (pre_own) {
    const bool za = tid < na;
    const AuditHit h = hit_at(tid);
    const double *y = sy_r1 + (za ? 0 : 2 * (int64_t)n) + h.pos, *par = (za ? bpar_of(a, b) : apar_of(a, b)) + h.line;
    pre[0] = y[0]; pre[1] = y[za ? n : m]; pre[2] = par[0]; pre[3] = par[k];
    pre[4] = za ? elem(a.A, a_index(a, b, h.pos, h.line)) : elem(a.B, b_index(a, b, h.line, h.pos));
  }
  if (pre_cross) {
    const AuditHit x = ha[(tid - 64) / nb], y = hb[(tid - 64) % nb];
    pre[0] = (double)C[(int64_t)x.pos * a.p.ldc + y.pos];
    pre[1] = elem(a.B, b_index(a, b, x.line, y.pos));
    pre[2] = elem(a.A, a_index(a, b, x.pos, y.line));
  }
  const int rows_per = (n + wgs - 1) / wgs, cols_per = (m + wgs - 1) / wgs;
  const bool by_row = wave >= RP_LINES / 64;
  const int t0 = by_row ? tid - RP_LINES : tid;
  const int o_beg = by_row ? min(n, w * rows_per) : min(m, w * cols_per), o_end = by_row ? min(n, o_beg + rows_per) : min(m, o_beg + cols_per);
  const int nh = by_row ? nb : na;          // hits whose footprint crosses these lines
  const AuditHit* hits = by_row ? hb : ha;
  const int len = by_row ? n : m;
  double* y1p = sy_r1 + (by_row ? 0 : 2 * (int64_t)n);
  double* g1p = al_r1 + (by_row ? 0 : 2 * (int64_t)n);
  // (what another workgroup reads is written through)
  constexpr int HALF_WAVES = RP_LINES / 64;
  double* red = pool;                       // [halves][hits][4][wavefronts]
  static_assert(2 * GECC_MAX_ERR * 4 * HALF_WAVES <= POOL_DOUBLES, "sums of the hits");
  for (int x = 0; x < max(nh, 1); ++x) {    // (one round without a hit: the test and the allowances)
    const bool last = x + 1 >= nh, some = x < nh;
    const int pos = some ? hits[x].pos : 0, l = some ? hits[x].line : 0;
    const double e = some ? hits[x].e : 0.0;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int o0 = o_beg + t0; o0 < o_end; o0 += RP_U * RP_LINES) {
      double y1[RP_U], y2[RP_U], g1[RP_U], g2[RP_U], v[RP_U];
      float cold[RP_U];
#pragma unroll
      for (int u = 0; u < RP_U; ++u) {
        const int o = min(o0 + u * RP_LINES, o_end - 1);
        y1[u] = y1p[o]; y2[u] = y1p[len + o];
        g1[u] = 0.0; g2[u] = 0.0; v[u] = 0.0; cold[u] = 0.f;
        if (x > 0) { g1[u] = g1p[o]; g2[u] = g1p[len + o]; }
        if (some) {
          cold[u] = C[by_row ? (int64_t)o * a.p.ldc + pos : (int64_t)pos * a.p.ldc + o];
          v[u] = by_row ? elem(a.A, a_index(a, b, o, l)) : elem(a.B, b_index(a, b, l, o));
        }
      }
#pragma unroll
      for (int u = 0; u < RP_U; ++u) {
        const int o = o0 + u * RP_LINES;
        if (o >= o_end || own_line(by_row, o)) continue;
        if (some) {
          const double f = v[u] * e;
          const float cnew = (float)((double)cold[u] - f);
          store_dev(C + (by_row ? (int64_t)o * a.p.ldc + pos : (int64_t)pos * a.p.ldc + o), cnew);
          const double d = (double)cold[u] - (double)cnew;   // what the sums of the symbol's row and column lose
          y1[u] -= d;
          y2[u] -= (double)(pos + 1) * d;
          g1[u] += cc * fabs(f);
          g2[u] += cc * (double)(pos + 1) * fabs(f);
          sum[0] += f * f;
          sum[1] += (double)(o + 1) * (o + 1) * f * f;
          sum[2] += d;
          sum[3] += (double)(o + 1) * d;
          store_dev(y1p + o, y1[u]);
          store_dev(y1p + len + o, y2[u]);
        }
        store_dev(g1p + o, g1[u]);
        store_dev(g1p + len + o, g2[u]);
        if (last) test(by_row, o, y1[u], y2[u], g1[u], g2[u]);
      }
    }
    if (!some) break;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[q] += __shfl_down(sum[q], off, 64);
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[(((by_row ? GECC_MAX_ERR : 0) + x) * 4 + q) * HALF_WAVES + (wave % HALF_WAVES)] = sum[q];
  }
  if (pre_own)
#pragma unroll
    for (int q = 0; q < 5; ++q) own[tid][q] = pre[q];
  if (pre_cross)
#pragma unroll
    for (int q = 0; q < 3; ++q) cross[tid - 64][q] = pre[q];
  __syncthreads();
  // the sums of this workgroup: A hits first, then B hits
  if (tid < 4 * (na + nb)) {
    const int x = tid >> 2, q = tid & 3;
    const double* r = red + (((x < na ? x : GECC_MAX_ERR + x - na)) * 4 + q) * HALF_WAVES;
    static_assert(HALF_WAVES == 4, "wavefronts of a half");
    mine.sums[x][q] = (r[0] + r[1]) + (r[2] + r[3]);
  }
  __syncthreads();
  if (wgs > 1) {
    static_assert(sizeof(RepairRecord) % 8 == 0 && sizeof(RepairRecord) / 8 <= RP_THREADS, "a word per thread");
    unsigned long long* out = reinterpret_cast<unsigned long long*>(records + (int64_t)b * wgs + w);
    if (tid < (int)(sizeof(RepairRecord) / 8)) store_dev(out + tid, reinterpret_cast<const unsigned long long*>(&mine)[tid]);
    if (!arrive_last(done + b, (uint32_t)wgs, &flag)) return;
    if (tid == 0) { mine.s = 0; mine.t = 0; mine.bad = 0; }
    __syncthreads();
    const RepairRecord* all = records + (int64_t)b * wgs;
    if (tid < 4 * (na + nb)) {
      double v[RP_WGS / 4], s = 0.0;
      for (int r0 = 0; r0 < wgs; r0 += RP_WGS / 4) {
#pragma unroll
        for (int r = 0; r < RP_WGS / 4; ++r) v[r] = load_dev(&all[min(r0 + r, wgs - 1)].sums[tid >> 2][tid & 3]);
#pragma unroll
        for (int r = 0; r < RP_WGS / 4; ++r) s += r0 + r < wgs ? v[r] : 0.0;
      }
      mine.sums[tid >> 2][tid & 3] = s;
    } else if (tid >= 64 && tid < 64 + wgs) {
      const RepairRecord& r = all[tid - 64];
      const int rs = load_dev(&r.s), rt = load_dev(&r.t), rb = load_dev(&r.bad);
      if (rs > 0) { const int at = atomicAdd(&mine.s, rs); for (int z = 0; z < min(rs, GECC_MAX_ERR) && at + z < GECC_MAX_ERR; ++z) mine.rows[at + z] = load_dev(&r.rows[z]); }
      if (rt > 0) { const int at = atomicAdd(&mine.t, rt); for (int z = 0; z < min(rt, GECC_MAX_ERR) && at + z < GECC_MAX_ERR; ++z) mine.cols[at + z] = load_dev(&r.cols[z]); }
      if (rb) mine.bad = 1;
    }
    __syncthreads();
  }
  if (tid == 0) {
    // The lines of the hits.  pool[4 z ..]: residuals and allowances of the line of hit z, kept at the first hit of that line
    auto first_at = [&](int z) {
      int x = z < na ? 0 : na;
      while (hit_at(x).pos != hit_at(z).pos) ++x;
      return x;
    };
    for (int z = 0; z < na + nb; ++z) { double* X = pool + 4 * z; X[0] = own[z][0]; X[1] = own[z][1]; X[2] = 0.0; X[3] = 0.0; }
    // first the symbols where the row of an A hit meets the column of a B hit, which nobody has touched
    for (int xy = 0; xy < na * nb; ++xy) {
      const int x = xy / nb, y = na + xy % nb;
      if (first_at(x) != x || first_at(y) != y) continue;
      const int i = hit_at(x).pos, j = hit_at(y).pos;
      float v = (float)cross[xy][0];
      // (for an A hit the column is the crossed line and the row its own, for a B hit the other way round)
      for (int z = 0; z < na + nb; ++z) {
        const bool za = z < na;
        const AuditHit h = hit_at(z);
        if (first_at(z) != (za ? x : y)) continue;
        double val = za ? cross[z * nb + y - na][1] : cross[x * nb + z - na][2];
        for (int q = 0; q < na && !za; ++q)
          if (ha[q].pos == i && ha[q].line == h.line) val -= ha[q].e;         // A as corrected
        const double f = val * h.e;
        const float cnew = (float)((double)v - f);
        const double d = (double)v - (double)cnew;
        v = cnew;
        double* X = pool + 4 * (za ? y : x);
        const int at = za ? i : j, other = za ? j : i;
        X[0] -= d;
        X[1] -= (double)(at + 1) * d;
        X[2] += cc * fabs(f);
        X[3] += cc * (double)(at + 1) * fabs(f);
        double* S = mine.sums[z];
        S[0] += f * f;
        S[1] += (double)(other + 1) * (other + 1) * f * f;
        S[2] += d;
        S[3] += (double)(other + 1) * d;
      }
      store_dev(C + (int64_t)i * a.p.ldc + j, v);
    }
    for (int z = 0; z < na + nb; ++z) {
      const bool za = z < na;
      const AuditHit h = hit_at(z);
      const double p1 = own[z][2] * h.e, p2 = own[z][3] * h.e, *S = mine.sums[z];
      double* cp = cpar + (za ? 0 : 2 * (int64_t)n) + h.pos;
      cp[0] -= p1;                           // cbar_{i,m+1} (cbar_{n+1,j})
      cp[za ? n : m] -= p2;                  // cbar_{i,m+2} (cbar_{n+2,j})
      double* X = pool + 4 * first_at(z);
      X[0] += p1 - S[2];                     // sum - parity: both moved
      X[1] += p2 - S[3];
      X[2] += cc * sqrt(S[0]);
      X[3] += cc * sqrt(S[1]);
    }
    // ... Section V step 1 on them, the operands, and the located errors, sorted by (matrix, row, col)
    for (int z = 0; z < na + nb; ++z) {
      const bool za = z < na;
      const AuditHit h = hit_at(z);
      if (first_at(z) == z) {
        const double* X = pool + 4 * z;
        double *y = sy_r1 + (za ? 0 : 2 * (int64_t)n) + h.pos, *g = al_r1 + (za ? 0 : 2 * (int64_t)n) + h.pos;
        const int step = za ? n : m;
        store_dev(y, X[0]); store_dev(y + step, X[1]); store_dev(g, X[2]); store_dev(g + step, X[3]);
        test(za, h.pos, X[0], X[1], X[2], X[3]);
      }
      if (!SPLIT) {
        if (za) store_elem(a.A, DT, a_index(a, b, h.pos, h.line), own[z][4] - h.e);
        else    store_elem(a.B, DT, b_index(a, b, h.line, h.pos), own[z][4] - h.e);
      }
      // (A hits are ordered by column, B hits by row; one hit per row of B)
      gecc_err g;
      g.matrix = za ? GECC_MAT_A : GECC_MAT_B; g.row = za ? h.pos : h.line; g.col = za ? h.line : h.pos; g.reserved = 0;
      g.magnitude = h.e;
      int at = z;
      for (int q = 0; q < na && za; ++q) at += q > z && ha[q].pos < h.pos ? 1 : q < z && ha[q].pos > h.pos ? -1 : 0;
      st->errs[at] = g;
    }
    st->n_err = na + nb;
    for (int x = 0; x < min(mine.s, GECC_MAX_ERR); ++x) st->rows[x] = mine.rows[x];
    for (int x = 0; x < min(mine.t, GECC_MAX_ERR); ++x) st->cols[x] = mine.cols[x];
    st->s_cnt = mine.s; st->t_cnt = mine.t; st->nonfinite = mine.bad; st->phase = PH_REVERIFY;
  }
  // ... and Section V step 2 on what is left, by the first DC_THREADS threads (the other wavefronts end here)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (it loads some of this past the caches)
  __syncthreads();
  if (SPLIT || tid >= DC_THREADS) return;
  decode_c_body(a, b, st, rep, 1, pool);
}

// Section V step 2 and, where it fails, the two re-encodings of the operand audit in one launch: a launch that
// waits for the one before it costs 2 to 5 us of the stream and 3 of the host whatever it does, and after a clean product this
// one only has the report to write.  Workgroup v of the audits decides from the counters and syndromes of the threshold pass,
// on its own and like all others, what Section V step 2 makes of its item: nothing or patches of C, or the
// audit (done by all of them; the repair follows as a launch of its own, with more threads).  Nobody writes
// what the others decide by.
// A symbol of C that is evaluated again is a dot product whose one operand lies in memory with a stride: a
// line per term, of which one compute unit keeps a few dozen on their way (k = 4096: 25 us a symbol).
// The first workgroups of the item share it out, at least FINISH_TERMS terms each; the one that comes last
// adds the shares up, a lane each, and patches (two symbols at 16384 x 4096 x 14336, rocprofv3: by one thread and with a workgroup for
// one symbol after the other 25.2 us, now 15).
// A closed launch lasts as long as its dispatch, about 2 us per thousand workgroups (the caller keeps very
// large pairs out).  Walking the rest with a grid that fits the chip was measured and is not kept: the
// compiler then holds what every scan needs across the walk (226 registers instead of 168, and audits that
// took 28 to 55 us from one build to the next instead of 24).
static_assert(DC_THREADS <= PAIR_LDS_DOUBLES, "the decoder works in the audits' LDS");
constexpr int FINISH_SHARES = 64, FINISH_TERMS = 64;
struct FinishArgs {
  DecodeArgs a;
  PairArgs audits;
  double* shares;        // per item 2k doubles (the audits' own, unused while C alone is patched)
  uint32_t* share_done;  // per item a counter
  int with_summary;
};
struct FinishWork {
  int b, x, y, q;        // item, workgroup of the scan, number among the item's workgroups
  bool second;
};
__device__ __forceinline__ FinishWork finish_work(const PairArgs& audits, int w) {
  FinishWork o;
  o.second = w >= audits.j[0].nblk;
  const PairJob& j = o.second ? audits.j[1] : audits.j[0];
  const int v = o.second ? w - audits.j[0].nblk : w, per_item = j.gx * j.gy;
  o.b = v / per_item; o.x = (v % per_item) % j.gx; o.y = (v % per_item) / j.gx;
  o.q = v % per_item + (o.second ? audits.j[0].gx * audits.j[0].gy : 0);
  return o;
}
template <int DT>
__global__ __launch_bounds__(DC_THREADS, 3) void finish_kernel(FinishArgs);
// (it reads its argument from the start of the kernel's argument segment, so it can have no other)
static_assert(std::is_same<decltype(&finish_kernel<GECC_F32>), void (*)(FinishArgs)>::value, "FinishArgs is all of finish_kernel's arguments");
template <int DT>
__global__ __launch_bounds__(DC_THREADS, 3) void finish_kernel(FinishArgs) {
  // (the arguments where the launch left them: through the parameter, the compiler gives every thread a copy
  // in scratch to write before the first decision)
  const FinishArgs& f = *(const FinishArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const DecodeArgs& a = f.a;
  __shared__ double lds[PAIR_LDS_DOUBLES];
  __shared__ Est fix[4];
  __shared__ double dots[4];
  __shared__ int nfix, act, flag;
  enum { NOTHING, PATCH, AUDIT };
  const FinishWork o = finish_work(f.audits, blockIdx.x);
  DecodeState* st = state_of(a, o.b);
  gecc_report* rep = a.report + o.b;
  if (f.with_summary) {
    if (o.q == 0) {
      if (summarize(a, o.b, st, rep, true) == GECC_CLEAN) return;
    } else if (st->s_cnt == 0 && st->t_cnt == 0) {
      return;
    }
  } else {
    // (one thread decides for the workgroup: the item's first workgroups may be writing the report meanwhile)
    if (threadIdx.x == 0) act = rep->status == GECC_DETECTED ? AUDIT : NOTHING;
    __syncthreads();
    if (act == NOTHING) return;
  }

  // workgroups of an item that share a dot product
  const int per_item = f.audits.j[0].gx * f.audits.j[0].gy + f.audits.j[1].gx * f.audits.j[1].gy;
  const int shares = a.p.refine ? max(1, min(min(per_item, FINISH_SHARES), a.p.k / FINISH_TERMS)) : 1;
  __syncthreads();
  plan_fixes(a, o.b, st->s_cnt, st->t_cnt, st->rows, st->cols, 0, fix, &nfix);
  if (threadIdx.x == 0)
    act = !st->nonfinite && nfix < 0 ? AUDIT : o.q == 0 || (!st->nonfinite && nfix > 0 && o.q < shares) ? PATCH : NOTHING;
  __syncthreads();
  const int todo = act;
  if (todo == NOTHING) return;
  bool writes = o.q == 0;
  const bool dot = todo == PATCH && !st->nonfinite && nfix > 0 && shares > 1;
  if (dot) {
    // a wavefront per symbol; the shares are added up by its lanes, in a fixed order
    static_assert(DC_THREADS / 64 >= 4 && FINISH_SHARES == 64, "a wavefront per fix, a lane per share");
    double* mine = f.shares + (int64_t)o.b * 2 * a.p.k;
    const int per = (a.p.k + shares - 1) / shares, l0 = min(a.p.k, o.q * per), l1 = min(a.p.k, l0 + per);
    const int e = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (e < nfix) {
      const double d = wave_sum(wave_dot(a, o.b, fix[e].i, fix[e].j, l0, l1));
      if (lane == 0) store_dev(mine + e * shares + o.q, d);
    }
    writes = arrive_last(f.share_done + o.b, (uint32_t)shares, &flag);
    if (writes && e < nfix) {
      const double d = wave_sum(lane < shares ? load_dev(mine + e * shares + lane) : 0.0);
      if (lane == 0) dots[e] = d;
    }
    __syncthreads();
  }
  if (writes) {
    if (f.with_summary) { summarize(a, o.b, st, rep); __syncthreads(); }
    if (todo == AUDIT) { if (threadIdx.x == 0) st->phase = PH_AUDIT; }
    else if (!st->nonfinite) apply_fixes(a, o.b, st, rep, fix, nfix, lds, dot ? dots : nullptr);
    else if (threadIdx.x == 0) give_up(st, rep);
    __syncthreads();
  }
  if (todo == AUDIT) pair_body<DT>(o.second ? f.audits.j[1] : f.audits.j[0], o.x, o.y, o.b, lds);
}

// Blocked mode, after repair_kernel<true>: the located operand symbols are put right, once per
// operand line (workgroup x < nbi: row block x of A; otherwise column block x - nbi of B), from
// the same parity differences the blocks used -- after every block has finished reading the
// operands as the product read them.
__global__ __launch_bounds__(256) void patch_operands_kernel(DecodeArgs a, int nbi) {
  if (*a.gate_word != PH_AUDIT) return;
  const bool is_a = (int)blockIdx.x < nbi;
  const int line_blk = is_a ? blockIdx.x : blockIdx.x - nbi;
  const int b = is_a ? line_blk * a.nbj : line_blk;           // an item of that line (item_i / item_j = line_blk)
  const int k = a.p.k, len = is_a ? a.p.n : a.p.m;
  const double* cur = (is_a ? a.audit_a : a.audit_b) + (int64_t)line_blk * 2 * k;
  const double* ref = (is_a ? a.A_par : a.B_par) + (int64_t)line_blk * 2 * k;
  __shared__ int cnt;
  __shared__ AuditHit h[GECC_MAX_ERR];
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int l = threadIdx.x; l < k; l += blockDim.x) {
    const double u1 = cur[l] - ref[l], u2 = cur[k + l] - ref[k + l];
    if (outside(u1, a.p.tau_op) || outside(u2, a.p.tau_op)) {
      const int idx = atomicAdd(&cnt, 1);
      if (idx < GECC_MAX_ERR) h[idx] = located(u1, u2, l, len, a.p.tau_op);
    }
  }
  __syncthreads();
  if (threadIdx.x != 0 || cnt == 0 || cnt > GECC_MAX_ERR) return;
  for (int x = 0; x < cnt; ++x) if (h[x].pos < 0) return;      // a line no single wrong symbol explains: hands off
  for (int x = 0; x < cnt; ++x) {
    const int64_t idx = is_a ? a_index(a, b, h[x].pos, h[x].line) : b_index(a, b, h[x].line, h[x].pos);
    void* M = is_a ? a.A : a.B;
    store_elem(M, a.p.dtype, idx, load_elem(M, a.p.dtype, idx) - h[x].e);
  }
}

// Blocked mode: Section V once more on what the repairs left, block by block.
__global__ __launch_bounds__(DC_THREADS) void final_decode_kernel(DecodeArgs a) {
  const int b = blockIdx.x;
  DecodeState* st = state_of(a, b);
  if (st->phase != PH_REVERIFY) return;
  __shared__ double pool[POOL_DOUBLES];
  decode_c_body(a, b, st, a.report + b, 1, pool);
}

// Blocked mode: syndromes of every block from the partial sums of the 128 x 128 sub-tiles (a block
// is a whole number of them), one thread per line and block along it.  a.p.n, a.p.m: block sizes.
__global__ __launch_bounds__(256) void threshold_blocked_kernel(DecodeArgs a, int n_full, int m_full) {
  const int nb = a.p.n, mb = a.p.m, nbj = a.nbj, nbi = n_full / nb;
  // (n_full, m_full are multiples of 128: the 64 lines of a wavefront lie in one block, and every
  // wavefront of the grid is full)
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total_r = (int64_t)n_full * nbj, total = total_r + (int64_t)m_full * nbi;
  if (idx >= total) return;
  const bool is_row = idx < total_r;
  double S = 0.0, W = 0.0;
  int b, loc;
  if (is_row) {
    const int i = (int)(idx % n_full), J = (int)(idx / n_full);
    const float2* pp = reinterpret_cast<const float2*>(a.rowpart) + i;
    for (int t = J * (mb / 128); t < (J + 1) * (mb / 128); ++t) {
      const float2 v = pp[(int64_t)t * a.rp_ld];
      S += (double)v.x;
      W += (double)v.y + (double)(t * 128 - J * mb) * (double)v.x;
    }
    b = (i / nb) * nbj + J; loc = i % nb;
  } else {
    const int64_t o = idx - total_r;
    const int j = (int)(o % m_full), I = (int)(o / m_full);
    const float2* pp = reinterpret_cast<const float2*>(a.colpart) + j;
    for (int t = I * (nb / 128); t < (I + 1) * (nb / 128); ++t) {
      const float2 v = pp[(int64_t)t * a.cp_ld];
      S += (double)v.x;
      W += (double)v.y + (double)(t * 128 - I * nb) * (double)v.x;
    }
    b = I * nbj + j / mb; loc = j % mb;
  }
  DecodeState* st = state_of(a, b);
  const double* cpar = cpar_of(a, b);
  double* synd = synd_of(a, b);
  const int o1 = is_row ? loc : 2 * nb + loc, o2 = is_row ? nb + loc : 2 * nb + mb + loc;
  const double v1 = S - cpar[o1], v2 = W - cpar[o2];
  synd[o1] = v1;
  synd[o2] = v2;
  const double t1 = is_row ? a.p.tau_r1 : a.p.tau_q1, t2 = is_row ? a.p.tau_r2 : a.p.tau_q2;
  if (outside(v1, t1) || outside(v2, t2)) {
    const int x = atomicAdd(is_row ? &st->s_cnt : &st->t_cnt, 1);
    if (x < GECC_MAX_ERR) (is_row ? st->rows : st->cols)[x] = loc;
  }
  if (!finite2(v1, v2)) atomicOr(&st->nonfinite, 1);
  // family maxima of the block: first over the wavefront (one block, see above), then one atomic per
  // wavefront -- non-negative doubles order like their bit patterns, a NaN above all
  double m1 = fabs(v1), m2 = fabs(v2);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    m1 = max_nan(m1, __shfl_xor(m1, off, 64));
    m2 = max_nan(m2, __shfl_xor(m2, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    unsigned long long* mx = reinterpret_cast<unsigned long long*>(a.blockmax) + (int64_t)b * 4 + (is_row ? 0 : 2);
    atomicMax(mx, (unsigned long long)__double_as_longlong(m1));
    atomicMax(mx + 1, (unsigned long long)__double_as_longlong(m2));
  }
}

// Blocked mode: the parity blocks of every block of C-bar from the two side products (A times the
// parity columns of all column blocks, the parity rows of all row blocks times B), P_g in fp64,
// and the per-block resets.  One workgroup per block; short chains of loads are all it does, so a full
// workgroup (224 blocks of 1024 x 1024, k = 4096: 25 us with 256 threads).
constexpr int BP_THREADS = 1024;
__global__ __launch_bounds__(BP_THREADS) void blocked_parities_kernel(BlockedParityArgs a) {
  const int b = blockIdx.x, I = b / a.nbj, J = b % a.nbj;
  const int nb = a.nb, mb = a.mb, S = a.pieces;
  double* cpar = a.C_par + (int64_t)b * (2 * nb + 2 * mb + 4);
  for (int il = threadIdx.x; il < nb; il += BP_THREADS) {      // 2 S consecutive floats of a row of the side product
    const float* p = a.side_r + (int64_t)(I * nb + il) * a.ld_r + J * 2 * S;
    double v0 = 0.0, v1 = 0.0;
    for (int s = 0; s < S; ++s) { v0 += (double)p[s]; v1 += (double)p[S + s]; }
    cpar[il] = v0;
    cpar[nb + il] = v1;
  }
  for (int o = threadIdx.x; o < 2 * mb; o += BP_THREADS) {
    const int t = o / mb, jl = o % mb;
    const float* p = a.side_c + (int64_t)((I * 2 + t) * S) * a.ld_c + J * mb + jl;
    double v = 0.0;
    for (int s = 0; s < S; ++s) v += (double)p[(int64_t)s * a.ld_c];
    cpar[2 * nb + o] = v;
  }
  const double* ap = a.A_par + (int64_t)I * 2 * a.k;
  const double* bp = a.B_par + (int64_t)J * 2 * a.k;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int l = threadIdx.x; l < a.k; l += BP_THREADS) {
    const double a0 = ap[l], a1 = ap[a.k + l], b0 = bp[l], b1 = bp[a.k + l];
    acc[0] = fma(a0, b0, acc[0]); acc[1] = fma(a0, b1, acc[1]);
    acc[2] = fma(a1, b0, acc[2]); acc[3] = fma(a1, b1, acc[3]);
  }
  __shared__ double red[BP_THREADS / 64][4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_down(acc[q], off, 64);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) red[threadIdx.x >> 6][q] = acc[q];
  __syncthreads();
  if (threadIdx.x < 4) {
    double v = red[0][threadIdx.x];
    for (int w = 1; w < BP_THREADS / 64; ++w) v += red[w][threadIdx.x];
    cpar[2 * nb + 2 * mb + threadIdx.x] = v;
  }
  if (threadIdx.x == 0) {
    reset_state(a.state + b);
    for (int f = 0; f < 4; ++f) a.itemmax[(int64_t)b * 4 + f] = 0.0;
    if (b == 0) *a.gate_word = PH_DONE;
  }
}

// fp64 parities -> rows of an operand of the product: `pieces` values of the operand's type per
// parity whose sum (in fp32 arithmetic of the product) restores 24 bits of it
__global__ __launch_bounds__(256) void split_parities_kernel(const double* par, void* W, int dtype, int lines, int k,
                                                             int pieces, int rows_padded) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)rows_padded * k) return;
  const int row = (int)(idx / k), l = (int)(idx % k);
  const int line_t = row / pieces, s = row % pieces;     // line_t = line * 2 + t
  double x = line_t < 2 * lines ? par[(int64_t)line_t * k + l] : 0.0;
  if (dtype == GECC_F32) {
    reinterpret_cast<float*>(W)[idx] = (float)x;
    return;
  }
  float piece = 0.f;
  for (int q = 0; q <= s; ++q) {          // hi, then what is left of it, then what is left of that
    uint32_t u = __float_as_uint((float)x);
    u += 0x7fffu + ((u >> 16) & 1u);
    u &= 0xffff0000u;
    piece = __uint_as_float(u);
    x -= (double)piece;
  }
  reinterpret_cast<uint16_t*>(W)[idx] = (uint16_t)(__float_as_uint(piece) >> 16);
}

}  // namespace

hipError_t launch_threshold(const DecodeArgs& a, const Parts& pr, const Parts& pc, hipStream_t st) {
  dim3 grid((a.p.n + a.p.m + 63) / 64, a.p.batch);   // 64 lines per workgroup: spreads over all CUs
  const int nt = a.ntm > a.ntn ? a.ntm : a.ntn;
  const dim3 block(64 * TH_SLICES);
  auto launch = [&](auto loads) {
    constexpr int N = decltype(loads)::value;
    if (pr.nchunk > 0 || pr.nseg > 0 || pc.nchunk > 0 || pc.nseg > 0) hipLaunchKernelGGL(threshold_parts_kernel<N>, grid, block, 0, st, a, pr, pc);
    else hipLaunchKernelGGL(threshold_kernel<N>, grid, block, 0, st, a);
  };
  if (nt <= 4 * TH_SLICES)      launch(std::integral_constant<int, 4>{});
  else if (nt <= 8 * TH_SLICES) launch(std::integral_constant<int, 8>{});
  else                          launch(std::integral_constant<int, 32>{});
  return hipGetLastError();
}

hipError_t launch_summarize(const DecodeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(summarize_kernel, dim3(a.p.batch), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_decode_c(const DecodeArgs& a, int with_summary, hipStream_t st) {
  hipLaunchKernelGGL(decode_c_kernel, dim3(a.p.batch), dim3(DC_THREADS), 0, st, a, with_summary);
  return hipGetLastError();
}

// Workgroups of an item in the repair: one per RP_LINES rows and columns, at most 256 in all, as many as there are records and counters
// for.  More than 128 items of long lines would have one each for them: then at most 512.  Repair, us (at most 256 / 512 / 1024):
//                                     an error of A in all items    in one item
//   f32 4096 x 64 x 4096 x 129          48.4 / 39.8 / 49.0         39.4 / 26.4 / 21.7
//   f32 8192 x 32 x 1024 x 256          55.8 / 44.4 / 53.6         40.4 / 28.6 / 22.4
//   f32 2048 x 128 x 2048 x 200         37.6 / 35.6 / 45.4         26.5 / 22.0 / 19.7
//   f32 1024 x 256 x 1024 x 200         31.4 / 31.8 / 41.4         21.7 / 19.6 / 18.3
//   bf16, 128 blocks of 2048 x 512      34.2 / 35.4 / 45.0         23.8 / 25.3 / 28.0
// Where no item is repaired it lasts 6.4 between event pairs with any of them.
static int repair_wgs(const DecodeArgs& a, const RepairScratch& s) {
  const int len = a.p.n > a.p.m ? a.p.n : a.p.m;
  int wgs = (len + RP_LINES - 1) / RP_LINES;
  if (wgs > RP_WGS) wgs = RP_WGS;
  const int most = len >= 2048 && a.p.batch > 128 ? 512 : 256;
  if ((int64_t)wgs * a.p.batch > most) wgs = most / a.p.batch;
  while (wgs > 1 && (size_t)wgs * a.p.batch * sizeof(RepairRecord) > s.bytes) --wgs;
  return wgs > 1 && a.p.batch <= s.counters ? wgs : 1;
}

hipError_t launch_repair(const DecodeArgs& a, const RepairScratch& s, hipStream_t st) {
  const int wgs = repair_wgs(a, s);
  const dim3 grid((unsigned)wgs * a.p.batch);
  RepairRecord* records = static_cast<RepairRecord*>(s.records);
  if (a.p.dtype == GECC_BF16) hipLaunchKernelGGL((repair_kernel<GECC_BF16, false>), grid, dim3(RP_THREADS), 0, st, a, records, s.done, wgs);
  else                        hipLaunchKernelGGL((repair_kernel<GECC_F32, false>), grid, dim3(RP_THREADS), 0, st, a, records, s.done, wgs);
  return hipGetLastError();
}

hipError_t launch_finish(const DecodeArgs& a, const PairArgs& audits, uint32_t* share_done, int with_summary, hipStream_t st) {
  const dim3 grid(audits.j[0].nblk + audits.j[1].nblk);
  const FinishArgs f{a, audits, const_cast<double*>(a.audit_a), share_done, with_summary};
  if (a.p.dtype == GECC_BF16) hipLaunchKernelGGL(finish_kernel<GECC_BF16>, grid, dim3(DC_THREADS), 0, st, f);
  else                        hipLaunchKernelGGL(finish_kernel<GECC_F32>, grid, dim3(DC_THREADS), 0, st, f);
  return hipGetLastError();
}

hipError_t launch_repair_blocked(const DecodeArgs& a, const RepairScratch& s, int nbi, hipStream_t st) {
  const int wgs = repair_wgs(a, s);
  const dim3 grid((unsigned)wgs * a.p.batch);
  RepairRecord* records = static_cast<RepairRecord*>(s.records);
  if (a.p.dtype == GECC_BF16) hipLaunchKernelGGL((repair_kernel<GECC_BF16, true>), grid, dim3(RP_THREADS), 0, st, a, records, s.done, wgs);
  else                        hipLaunchKernelGGL((repair_kernel<GECC_F32, true>), grid, dim3(RP_THREADS), 0, st, a, records, s.done, wgs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(patch_operands_kernel, dim3(nbi + a.nbj), dim3(256), 0, st, a, nbi);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(final_decode_kernel, dim3(a.p.batch), dim3(DC_THREADS), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_threshold_blocked(const DecodeArgs& a, int n_full, int m_full, hipStream_t st) {
  const int64_t total = (int64_t)n_full * a.nbj + (int64_t)m_full * (n_full / a.p.n);
  hipLaunchKernelGGL(threshold_blocked_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, n_full, m_full);
  return hipGetLastError();
}

hipError_t launch_blocked_parities(const BlockedParityArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(blocked_parities_kernel, dim3(a.nbi * a.nbj), dim3(BP_THREADS), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_split_parities(const double* par, void* W, int dtype, int lines, int k, int pieces, int rows_padded,
                                 hipStream_t st) {
  const int64_t total = (int64_t)rows_padded * k;
  hipLaunchKernelGGL(split_parities_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, par, W, dtype, lines, k,
                     pieces, rows_padded);
  return hipGetLastError();
}


}  // namespace gecc
