// The data block of the encoded product (Section III, C = A B) on the MFMA units for fp32 operands and
// for the bf16 products that the 256 x 256-tile kernel does not take (small ones, ragged k, rows that
// are not 16-byte aligned), with the row/column sums that Section V's syndromes need taken from the
// accumulators before C leaves the compute unit, so that verification never re-reads C from HBM.
//
// Workgroup: a TILE x TILE tile of C (128 or 64), 4 wavefronts (2 x 2), MFMA 16x16x32 bf16.  Operand
// tiles go HBM -> registers -> LDS, the next k-tile's loads in flight while this one is multiplied; two
// to five workgroups share a compute unit and cover each other's barriers.  No load assumes an alignment
// beyond the element's own.
//
// fp32 operands run on the bf16 units too: x = x1 + x2 + x3, each piece the bf16 nearest to what is left
// (8 significand bits and a sign each, so the three hold all 24 bits of x exactly), and
//   a b = a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1) + terms below 2^-25 |a b|,
// six exact products per pair, accumulated in fp32.  Native fp32 MFMAs do 64 flop per cycle and SIMD,
// bf16 ones 1024: six of those are 2.7 times as fast.  Measured when this kernel replaced one of native fp32
// MFMAs: 256 x 512^3 766 -> 430 us, 1024^3 50 -> 28, 128^3 28 -> 7.7, with a result closer to the fp64 product
// (2.1e-7 -> 6.5e-8 at 128^3, 2.9e-7 -> 9e-8 at 1024^3); bf16, 1500 x 1000 x 1100 with rows that are not
// 16-byte aligned, 67 -> 20 us, the loads being vectors whatever the alignment.  As it is now: 1024^3 25.7 us,
// 128^3 7.2, the bf16 product 14.1.  What bounds it: the pieces (13 vector instructions per two staged elements)
// and the two barriers per k-tile, which the other workgroups of the compute unit cover.
// Where a piece cannot hold its part of x the tile is computed again with native fp32 MFMAs, from the
// same operands in the same launch:
//   - some accumulator is not finite (an infinite or NaN operand, |x| that rounds past the largest bf16,
//     a sum that overflows): the fp32 arithmetic decides what C holds there;
//   - an operand value of the tile is below 2^-110 and not zero: its last bit is below 2^-133, the smallest
//     subnormal bf16 (the matrix units keep subnormal operands: measured, the error of one product is the
//     same for every power of two down to 2^-110 and doubles with each one below).  One such value is enough:
//     beside ordinary ones of its row it may meet a large value of the other operand.
// k of one k-tile (32 and less) goes through fp64 MFMAs instead.  Such a sum is a few roundings of native fp32
// products; the matrix unit's own sum of 32 products and the pairs that the six leave out are more than those where
// one or two products decide it (values spread over 17 decades, distance from the fp64 product against native ones:
// k = 1 2.66e-8 against 2.63e-8, k = 8 3.64e-8 against 2.94e-8, k = 32 4.73e-8 against 4.06e-8).  Rounded once it is
// closer than either on any operands (2.5e-8 for all three; normal ones, k = 32: 2.5e-8 against 3.9e-8 through pieces).
// Bound there by the fp64 rate or by C's stores: 8192 x k x 8192 through fp64 and through pieces, k = 1 70 against
// 80 us, k = 8 87 against 89, k = 32 111 against 78.
#include <cmath>
#include <type_traits>
#include "gemm_device.h"

namespace gecc {
namespace {

template <int DT> struct GT;
template <> struct GT<GECC_BF16> {
  using T = uint16_t;
  static constexpr int PIECES = 1;
  static constexpr int BK = 64;
};
template <> struct GT<GECC_F32> {
  using T = float;
  static constexpr int PIECES = 3;
  static constexpr int BK = 32;
};

// ---- staging of one operand tile: ROWS (m- or n-index) x BK ------------------------------------
// KC: element (r, kk) lives at P[r * ld + kk]; otherwise at P[kk * ld + r].  Rows past the last one are
// clamped to it (what they accumulate is masked in the epilogue), k past the end counts as zero.
// D k-tiles are on their way at a time, each in registers of its own (d).  load() issues the same loads whatever
// k0 is, clamped into the range (so that addresses stay a base and a stride), and fix() puts the last k-tile right
// in the registers: a branch around a load makes every later wait one for all loads in flight, the next k-tile's
// included (bf16 1500 x 1000 x 1100: 0.82 us per k-tile however many were on their way).  Product alone, with the
// branches -> without, us:
//   bf16 1500 x 1000 x 1100   19.6 -> 14.6 (TN 23.2 -> 15.7, NT 15.2 -> 12.2)
//   bf16 2500^3               69.5 -> 56.0
//   bf16 96 x 16384 x 4096    69.5 -> 49.7
//   fp32 2000 x 1000 x 2000   NT 63.5 -> 57.4
template <int DT, int ROWS, bool KC, int D> struct Stager;

// k contiguous: 16-byte loads, eight lanes to a row
template <int DT, int ROWS, int D>
struct Stager<DT, ROWS, true, D> {
  using T = typename GT<DT>::T;
  static constexpr int BK = GT<DT>::BK, V = 16 / (int)sizeof(T), N = ROWS * BK / V / THREADS;
  static constexpr int PLANE = ROWS * BK * 2;
  const T* src[N];
  uint4 regs[D][N];
  Least least;      // of the values this thread has staged
  int kk, klim;
  __device__ __forceinline__ void init(const T* P, int64_t ld, int r0, int rlim, int k_end) {
    kk = (threadIdx.x & 7) * V;
    klim = k_end;
#pragma unroll
    for (int i = 0; i < N; ++i) src[i] = P + (int64_t)min(r0 + (int)(threadIdx.x >> 3) + 32 * i, rlim - 1) * ld;
  }
  // (past the end: the row's last V elements)
  __device__ __forceinline__ void load(int k0, int d) {
    const int c = min(k0 + kk, klim - V);
#pragma unroll
    for (int i = 0; i < N; ++i) __builtin_memcpy(&regs[d][i], src[i] + c, 16);
  }
  __device__ __forceinline__ void fix(int k0, int d) {
    const int drop = max(0, min(k0 + kk - (klim - V), V));      // elements that belong to a neighbour
#pragma unroll
    for (int i = 0; i < N; ++i) {
      uint4& r = regs[d][i];
      uint64_t lo = (uint64_t)r.y << 32 | r.x, hi = (uint64_t)r.w << 32 | r.z;
      int sh = drop * 8 * (int)sizeof(T);
      if (sh >= 64) { lo = hi; hi = 0; sh -= 64; }
      if (sh >= 64) { lo = 0; sh = 0; }
      if (sh > 0) { lo = lo >> sh | hi << (64 - sh); hi >>= sh; }
      r = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
  }
  // k < 16: all of the range, in the first registers
  __device__ __forceinline__ void load_short(int k0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      T x[V];
#pragma unroll
      for (int e = 0; e < V; ++e) x[e] = k0 + kk + e < klim ? src[i][k0 + kk + e] : (T)0;
      __builtin_memcpy(&regs[0][i], x, 16);
    }
  }
  __device__ __forceinline__ void store(char* S, int d) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint4 r = regs[d][i];
      const int row = (threadIdx.x >> 3) + 32 * i;
      if constexpr (DT == GECC_BF16) {
        *reinterpret_cast<uint4*>(S + lds_at<BK>(row, threadIdx.x & 7)) = r;
      } else {
        const float x[4] = {__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w)};
        uint32_t a[3], b[3];
        split2(x[0], x[1], a);
        split2(x[2], x[3], b);
        least.see(x[0], x[1]);
        least.see(x[2], x[3]);
        char* dst = S + lds_at<BK>(row, (threadIdx.x & 7) >> 1) + (threadIdx.x & 1) * 8;
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(dst + q * PLANE) = make_uint2(a[q], b[q]);
      }
    }
  }
  __device__ __forceinline__ bool tiny() const { return least.tiny(); }
  // the fp32 values as they are, rows of BK + 1 floats (native fp32 pass)
  __device__ __forceinline__ void store_plain(float* S) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint4 r = regs[0][i];
      float* d = S + ((threadIdx.x >> 3) + 32 * i) * (BK + 1) + kk;
      d[0] = __uint_as_float(r.x); d[1] = __uint_as_float(r.y);
      d[2] = __uint_as_float(r.z); d[3] = __uint_as_float(r.w);
    }
  }
};

// r contiguous: a thread's KPT consecutive k end with the last one at the latest; what it then has of its neighbours' moves out
template <class T, int KPT>
__device__ __forceinline__ void shift_out(T (&r)[KPT], int drop) {
#pragma unroll
  for (int bit = KPT; bit > 0; bit >>= 1)
    if (drop & bit) {
#pragma unroll
      for (int x = 0; x < KPT; ++x) r[x] = x + bit < KPT ? r[x + bit] : (T)0;
    }
}

// r contiguous, fp32: a thread owns one row and KPT consecutive k (a wavefront reads 256 contiguous bytes
// of a k-row per instruction), so that its stores are whole 16-byte chunks along k
template <int ROWS, int D>
struct Stager<GECC_F32, ROWS, false, D> {
  static constexpr int BK = GT<GECC_F32>::BK, KPT = ROWS * BK / THREADS;
  static constexpr int PLANE = ROWS * BK * 2;
  const float* src;
  float regs[D][KPT];
  Least least;
  int64_t ld;
  int row, kg, klim;
  __device__ __forceinline__ void init(const float* P, int64_t ld_, int r0, int rlim, int k_end) {
    row = threadIdx.x & (ROWS - 1);
    kg = __builtin_amdgcn_readfirstlane(threadIdx.x / ROWS) * KPT;     // ROWS >= 64: one k group per wavefront
    ld = ld_; klim = k_end;
    src = P + min(r0 + row, rlim - 1);
  }
  __device__ __forceinline__ void load(int k0, int d) {
#pragma unroll
    for (int x = 0; x < KPT; ++x) regs[d][x] = src[(int64_t)(min(k0 + kg, klim - KPT) + x) * ld];
  }
  __device__ __forceinline__ void fix(int k0, int d) { shift_out(regs[d], max(0, min(k0 + kg - (klim - KPT), KPT))); }
  __device__ __forceinline__ void load_short(int k0) {
#pragma unroll
    for (int x = 0; x < KPT; ++x) regs[0][x] = k0 + kg + x < klim ? src[(int64_t)(k0 + kg + x) * ld] : 0.f;
  }
  __device__ __forceinline__ void store(char* S, int d) {
#pragma unroll
    for (int c = 0; c < KPT / 8; ++c) {
      uint32_t p[4][3];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const float x0 = regs[d][c * 8 + 2 * h], x1 = regs[d][c * 8 + 2 * h + 1];
        split2(x0, x1, p[h]);
        least.see(x0, x1);
      }
      char* dst = S + lds_at<BK>(row, (kg >> 3) + c);
#pragma unroll
      for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(dst + q * PLANE) = make_uint4(p[0][q], p[1][q], p[2][q], p[3][q]);
    }
  }
  __device__ __forceinline__ bool tiny() const { return least.tiny(); }
  __device__ __forceinline__ void store_plain(float* S) const {
#pragma unroll
    for (int x = 0; x < KPT; ++x) S[row * (BK + 1) + kg + x] = regs[0][x];
  }
};

// r contiguous, bf16: a thread owns two neighbouring rows (one 4-byte load per k) and KPT consecutive k
template <int ROWS, int D>
struct Stager<GECC_BF16, ROWS, false, D> {
  static constexpr int BK = GT<GECC_BF16>::BK, KPT = ROWS * BK / THREADS / 2;
  static constexpr int PLANE = ROWS * BK * 2;
  const uint16_t* src;
  uint32_t regs[D][KPT];
  int64_t ld;
  int row, kg, klim, shift;
  bool single;
  __device__ __forceinline__ void init(const uint16_t* P, int64_t ld_, int r0, int rlim, int k_end) {
    row = 2 * (threadIdx.x & (ROWS / 2 - 1));
    kg = (threadIdx.x / (ROWS / 2)) * KPT;
    ld = ld_; klim = k_end;
    // the last row of an odd number of them is read as the second of a pair; an operand of one row has no pairs
    const int r = min(r0 + row, rlim - 1), base = max(0, min(r, rlim - 2));
    shift = r > base ? 16 : 0;
    single = rlim < 2;
    src = P + base;
  }
  __device__ __forceinline__ void load(int k0, int d) {
    const uint16_t* p = src + (int64_t)min(k0 + kg, klim - KPT) * ld;
    // (as many loads either way)
    if (!single) {
#pragma unroll
      for (int x = 0; x < KPT; ++x) __builtin_memcpy(&regs[d][x], p + x * ld, 4);
    } else {
#pragma unroll
      for (int x = 0; x < KPT; ++x) regs[d][x] = p[x * ld];
    }
  }
  __device__ __forceinline__ void fix(int k0, int d) { shift_out(regs[d], max(0, min(k0 + kg - (klim - KPT), KPT))); }
  __device__ __forceinline__ void load_short(int k0) {
#pragma unroll
    for (int x = 0; x < KPT; ++x) {
      const uint16_t* p = src + (int64_t)(k0 + kg + x) * ld;
      uint32_t v = 0;
      if (k0 + kg + x < klim) { v = p[0]; if (!single) v |= (uint32_t)p[1] << 16; }
      regs[0][x] = v;
    }
  }
  __device__ __forceinline__ void store(char* S, int d) {
#pragma unroll
    for (int c = 0; c < KPT / 8; ++c) {
      uint32_t lo[4], hi[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const uint32_t v0 = regs[d][c * 8 + 2 * h] >> shift, v1 = regs[d][c * 8 + 2 * h + 1] >> shift;
        lo[h] = (v0 & 0xffffu) | (v1 << 16);
        hi[h] = (v0 >> 16) | (v1 & 0xffff0000u);
      }
      *reinterpret_cast<uint4*>(S + lds_at<BK>(row, (kg >> 3) + c)) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
      *reinterpret_cast<uint4*>(S + lds_at<BK>(row + 1, (kg >> 3) + c)) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    }
  }
};

// k-tiles on their way, and of two halves of the LDS (then one barrier per k-tile instead of two): two for bf16 tiles of 64; those of
// 128 would lose their third workgroup on a compute unit (1536 x 4224 x 768 with two 60.5 us a call, with one 58.6), and fp32, three
// pieces per value, has neither the registers nor the LDS (1024^3 with two 42.5 us, with one 41.7).
template <int DT, int TILE> constexpr int tile_depth() { return DT == GECC_BF16 && TILE == 64 ? 2 : 1; }

// workgroup v of the scans that ride along (see GemmSide).  Fewer rows in flight than in the scans' own
// launches: more registers here would cost the product workgroups per compute unit
template <int DT>
__device__ __forceinline__ void side_job(const GemmArgs& a, const GemmSide& side, int v, double* lds) {
  if (v < side.pg_items) {
    if (side.par_out) {
      // (one workgroup and its latencies: as many outputs at once as 32 loads in flight allow)
      const int len = 2 * a.k, nchunk = side.par.nchunk;
      double* out = side.par_out + (int64_t)v * len;
      const double* from = side.par.chunks + (int64_t)v * nchunk * len;
      auto finish = [&](auto g_, auto max_) {
        constexpr int G = decltype(g_)::value, MAX = decltype(max_)::value;
        for (int o0 = threadIdx.x; o0 < len; o0 += G * THREADS) {
          const double* part[G];
          double s[G];
#pragma unroll
          for (int g = 0; g < G; ++g) part[g] = from + min(o0 + g * THREADS, len - 1);
          chunk_sums<G, MAX>(part, len, nchunk, s);
#pragma unroll
          for (int g = 0; g < G; ++g)
            if (o0 + g * THREADS < len) out[o0 + g * THREADS] = s[g];
        }
      };
      if (nchunk <= 8) finish(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
      else if (nchunk <= 16) finish(std::integral_constant<int, 2>{}, std::integral_constant<int, 16>{});
      else for (int o = threadIdx.x; o < len; o += THREADS) out[o] = chunk_sum(from + o, len, nchunk);
      __syncthreads();
    }
    form_pg(a, v, lds);
    return;
  }
  v -= side.pg_items;
  const bool second = v >= side.j[0].nblk;
  if (second) v -= side.j[0].nblk;
  const SideJob& j = second ? side.j[1] : side.j[0];
  const int per_item = j.gx * j.gy;
  const int b = v / per_item, x = (v % per_item) % j.gx, y = (v % per_item) / j.gx;
  if (j.kind == SIDE_ROW) rowdot_body<DT, false, side_rows<DT>(), 1>(j.s, x, b, lds);
  else if (j.kind == SIDE_COL) coldot_body<Elem<DT>, false, DT == GECC_F32 ? 4 : 2, CD_ASK, true>(j.s, j.w, j.gy, j.gx, x, y, b, lds);
  else if constexpr (DT == GECC_F32) rowdot_wave_body<DT, false>(j.s, x, b, lds);
}

// The tile of this workgroup; false: it was one of the scans that ride along, which is done, or has no tile.
struct Place { int tm, tn, b, split; };
template <int DT, int TILE>
__device__ __forceinline__ bool place(const GemmArgs& a, const GemmSide& side, int S, char* smem, Place& o) {
  const int ntm = (a.n + TILE - 1) / TILE, ntn = (a.m + TILE - 1) / TILE;
  int id = blockIdx.x;
  if (side.groups > 0) {
    // in whole groups of 8 workgroups (one per XCD): side.lead of P_g and, where they go first, the scans; then the
    // product's; then the scans
    const int first = side.lead * 8, own = (side.own + 7) / 8 * 8;
    if (id < first || id >= first + own) {
      const int v = id < first ? id : side.lead_blocks + id - first - own;
      if (v < (id < first ? side.lead_blocks : side.blocks)) side_job<DT>(a, side, v, reinterpret_cast<double*>(smem));
      return false;
    }
    id -= first;
    if (id >= side.own) return false;
  }
  {
    const int N = side.own, per = N / 8, rem = N - per * 8, x = id & 7;
    id = x * per + min(x, rem) + (id >> 3);
  }
  const int bs = id / (ntn * ntm);
  o.tn = id % ntn; o.tm = (id / ntn) % ntm;
  o.b = bs / S; o.split = bs - o.b * S;
  return true;
}

// Accumulators of a TILE x TILE tile, four wavefronts (2 x 2): acc[i][j][v] = C[16 i + 4 lg + v][16 j + l16] of a quarter

// rows and columns past the end count as zero
template <int TILE>
__device__ __forceinline__ void mask_edges(const GemmArgs& a, int tile_r0, int tile_c0, f32x4_t (&acc)[TILE / 32][TILE / 32]) {
  constexpr int W = TILE / 2, NI = W / 16;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = tile_r0 + (wave >> 1) * W + (lane >> 4) * 4, c0 = tile_c0 + (wave & 1) * W + (lane & 15);
  if (tile_r0 + TILE > a.n || tile_c0 + TILE > a.m) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (r0 + i * 16 + v >= a.n || c0 + j * 16 >= a.m) acc[i][j][v] = 0.f;
  }
}

// k-split: every workgroup of the tile leaves its partial sums in memory (in register order, 16 bytes a lane: whole
// lines per store), the one that arrives last adds them all up, in an order that is the same whichever that is, and
// goes on with the tile (true).  Written through and read past the caches, like store_dev and load_dev, for which
// 16 bytes are too many.  (Whole calls, with 4 bytes a lane -> with 16: 300 x 2000 x 400 bf16 in eight ranges
// 30.2 -> 28.4 us, 700^3 in four 28.6 -> 26.9, 512^3 fp32 in four 25.9 -> 25.4.)
// The order: tiles of 64, two neighbouring ranges and then the pair to the sum, which halves the chain of additions
// (fp32 256 x 512 x 256 in eight ranges, distance from the fp64 product 7.27e-8 -> 6.73e-8; time unchanged); tiles of
// 128, which have no registers for a second range on its way, one after the other.
template <int TILE>
__device__ __forceinline__ bool add_splits(const GemmArgs& a, int b, int tm, int tn, int split, int S,
                                           f32x4_t (&acc)[TILE / 32][TILE / 32], char* smem) {
  constexpr int NI = TILE / 32, DEV = 16;         // (the bit of device scope among a buffer instruction's cache bits)
  const int ntm = (a.n + TILE - 1) / TILE, ntn = (a.m + TILE - 1) / TILE;
  const int64_t tile_id = ((int64_t)b * ntm + tm) * ntn + tn;
  __amdgpu_buffer_rsrc_t part = __builtin_amdgcn_make_buffer_rsrc(a.split_part + tile_id * S * (TILE * TILE), 0, S * TILE * TILE * 4, 0x00027000);
  const int at = threadIdx.x * 16;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(stream_t, acc[i][j]), part, at + (i * NI + j) * THREADS * 16,
                                             split * TILE * TILE * 4, DEV);
  if (!arrive_last(a.split_done + tile_id, (uint32_t)S, reinterpret_cast<int*>(smem))) return false;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int q, int at_ij) {
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(part, at + at_ij * THREADS * 16, q * TILE * TILE * 4, DEV));
  };
  int q = 0;
  if constexpr (TILE == 64)
#pragma unroll 2
    for (; q + 1 < S; q += 2)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const f32x4_t x = load(q, i * NI + j), y = load(q + 1, i * NI + j);
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] += x[v] + y[v];
        }
#pragma unroll 2
  for (; q < S; ++q)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const f32x4_t x = load(q, i * NI + j);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][v] += x[v];
      }
  return true;
}

// C, and the tile's share of the syndromes
template <int TILE>
__device__ __forceinline__ void finish_tile(const GemmArgs& a, int b, int tm, int tn, f32x4_t (&acc)[TILE / 32][TILE / 32], char* smem) {
  constexpr int W = TILE / 2, NI = W / 16;
  const int tile_r0 = tm * TILE, tile_c0 = tn * TILE;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1, l16 = lane & 15, lg = lane >> 4;
  // ---- epilogue, from the accumulators -------------------------------------------------------------
  // Test faults (none in production calls): the workgroup searches the list for those that strike its
  // tile, then every wavefront adds them to its accumulators.
  if (a.n_faults > 0) {
    int* hits = reinterpret_cast<int*>(smem);
    int2* hit = reinterpret_cast<int2*>(smem + 16);
    __syncthreads();
    if (tid == 0) *hits = 0;
    __syncthreads();
    for (int f = tid; f < a.n_faults; f += THREADS) {
      const gecc_fault ft = a.faults[f];
      const int r = ft.row - tile_r0, c = ft.col - tile_c0;
      if (ft.batch == b + a.fault_bias && r >= 0 && r < min(TILE, a.n - tile_r0) && c >= 0 && c < min(TILE, a.m - tile_c0))
        hit[atomicAdd(hits, 1)] = make_int2(r * TILE + c, __float_as_int(ft.offset));
    }
    __syncthreads();
    const int nh = *hits;
    for (int f = 0; f < nh; ++f) {
      const int r = hit[f].x / TILE - wr * W, c = hit[f].x % TILE - wc * W;
      const float off = __int_as_float(hit[f].y);
      const bool mine = r >= 0 && r < W && c >= 0 && c < W && ((r >> 2) & 3) == lg && (c & 15) == l16;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (mine && i == r >> 4 && j == c >> 4 && v == (r & 3)) acc[i][j][v] += off;
    }
  }

  // C: the registers of two neighbouring 16-column blocks first trade their odd / even groups of 16 lanes
  // (v_permlane16_swap): each then holds 2 rows x 32 consecutive columns, two full lines per store
  {
    const int R0 = tile_r0 + wr * W + (lg >> 1) * 8, C0 = tile_c0 + wc * W + (lg & 1) * 16 + l16;
    float* C = a.C + (int64_t)b * a.sc + (int64_t)R0 * a.ldc + C0;
    const bool whole = tile_r0 + TILE <= a.n && tile_c0 + TILE <= a.m;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int jp = 0; jp < NI / 2; ++jp) {
          float t0 = acc[i][2 * jp][v], t1 = acc[i][2 * jp + 1][v];
          // (inline: this compiler's builtin for the swap loses its second result; the wait states are the
          // ones a swap needs after a vector instruction wrote its operands)
          asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(t0), "+v"(t1));
          float* dst = C + (int64_t)(i * 16 + v) * a.ldc + jp * 32;
          if (whole) {
            dst[0] = t0;
            dst[4 * a.ldc] = t1;
          } else if (C0 + jp * 32 < a.m) {
            if (R0 + i * 16 + v < a.n) dst[0] = t0;
            if (R0 + i * 16 + v + 4 < a.n) dst[4 * a.ldc] = t1;
          }
        }
  }
  if (!a.rowpart) return;

  // Row sums: a lane adds its columns of a row (plain, and u = sum of j x_j: the block part of the column
  // weight), the 16 lanes of a group are added across the lanes; lane l16 of a group keeps row number
  // l16 = 4 i + v of its 4 NI.  Column sums: in the lane, then across the four groups; group lg keeps block lg.
  float2* rowred = reinterpret_cast<float2*>(smem);          // [2: wc][TILE]
  float2* colred = rowred + 2 * TILE;                         // [2: wr][TILE]
  __syncthreads();
  {
    float ks = 0.f, kw = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float s = acc[i][0][v], u = 0.f;
#pragma unroll
        for (int j = 1; j < NI; ++j) { s += acc[i][j][v]; u = fmaf((float)j, acc[i][j][v], u); }
        const float w = row16_sum(fmaf((float)(l16 + 1), s, 16.f * u));
        s = row16_sum(s);
        if (l16 == i * 4 + v) { ks = s; kw = w; }
      }
    if (l16 < 4 * NI)
      rowred[wc * TILE + wr * W + (l16 >> 2) * 16 + lg * 4 + (l16 & 3)] = make_float2(ks, fmaf((float)(wc * W), ks, kw));
    float cs = 0.f, cw = 0.f;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      float s = 0.f, w = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) { s += acc[i][j][v]; w = fmaf((float)(i * 16 + v + 1), acc[i][j][v], w); }
      w = fmaf((float)(lg * 4), s, w);
      s += __shfl_xor(s, 16, 64); w += __shfl_xor(w, 16, 64);
      s += __shfl_xor(s, 32, 64); w += __shfl_xor(w, 32, 64);
      if (lg == j) { cs = s; cw = w; }
    }
    if (lg < NI) colred[wr * TILE + wc * W + lg * 16 + l16] = make_float2(cs, fmaf((float)(wr * W), cs, cw));
  }
  __syncthreads();
  if (tid < TILE) {
    if (tile_r0 + tid < a.n)
      *reinterpret_cast<float2*>(a.rowpart + (((int64_t)b * a.ntn + tn) * a.rp_ld + tile_r0 + tid) * 2) =
          make_float2(rowred[tid].x + rowred[TILE + tid].x, rowred[tid].y + rowred[TILE + tid].y);
  } else if (tid < 2 * TILE) {
    const int c = tid - TILE;
    if (tile_c0 + c < a.m)
      *reinterpret_cast<float2*>(a.colpart + (((int64_t)b * a.ntm + tm) * a.cp_ld + tile_c0 + c) * 2) =
          make_float2(colred[c].x + colred[TILE + c].x, colred[c].y + colred[TILE + c].y);
  }
}

// -------------------------------------------------------------------------------------------
// Grid: one dimension, tiles x batch x ksplit workgroups, and the scans that ride along before or behind them.
// Consecutive workgroups go to the 8 XCDs in turn, so every XCD is given a contiguous range of the (item,
// split, tile row, tile column) sequence: tiles that share operand panels share an L2.  The scans are
// HBM-bound and the product is not: in one launch they cost little more than the
// product alone, and a launch of their own 2 to 5 us of the stream and 3 of the host beside their time.
// WHAT: the operands' type, or BF16_FOLD (tiles of 64): the sums of every k_fold terms are put aside, so that the chains
// of additions are no longer than with more ranges of k (k_fold_of).
constexpr int BF16_FOLD = GECC_BF16 + 2;
template <int WHAT, bool KCA, bool KCB, int TILE>
__global__ __launch_bounds__(THREADS, TILE == 64 ? 4 : WHAT == GECC_BF16 ? 3 : 2) void gemm_tile(GemmArgs a, GemmSide side) {
  constexpr bool FOLD = WHAT == BF16_FOLD;
  constexpr int DT = FOLD ? (int)GECC_BF16 : WHAT;
  using T = typename GT<DT>::T;
  constexpr int BK = GT<DT>::BK, PIECES = GT<DT>::PIECES, W = TILE / 2, NI = W / 16;   // W x W per wavefront
  constexpr int PLANE = TILE * BK * 2, OPERAND = PIECES * PLANE;
  constexpr int PLAIN = DT == GECC_F32 ? 2 * TILE * (BK + 1) * 4 : 0;
  constexpr int FAULTS = GECC_MAX_FAULTS * 8 + 16;        // list of the faults that strike this tile
  constexpr int SCAN = 8 * (CD_LDS_DOUBLES > RW_LDS_DOUBLES ? CD_LDS_DOUBLES : RW_LDS_DOUBLES);
  constexpr int D = tile_depth<DT, TILE>();
  constexpr bool TWICE = D == 2;
  constexpr int TILES = (TWICE ? 4 : 2) * OPERAND;
  constexpr int SM0 = TILES > PLAIN ? TILES : PLAIN;
  constexpr int SM1 = FAULTS > SCAN ? FAULTS : SCAN;      // (the sums of the wavefronts, 32 TILE bytes, are less)
  __shared__ __attribute__((aligned(16))) char smem[SM0 > SM1 ? SM0 : SM1];

  const int S = a.ksplit > 1 ? a.ksplit : 1;
  Place o;
  if (!place<DT, TILE>(a, side, S, smem, o)) return;
  const int tm = o.tm, tn = o.tn, b = o.b, split = o.split;
  const int k_begin = S > 1 ? min(a.k, split * a.k_per) : 0;
  const int k_end = S > 1 ? min(a.k, k_begin + a.k_per) : a.k;
  const int tile_r0 = tm * TILE, tile_c0 = tn * TILE;
  const T* A = reinterpret_cast<const T*>(a.A) + (int64_t)b * a.sa;
  const T* B = reinterpret_cast<const T*>(a.B) + (int64_t)b * a.sb;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;

  // acc[i][j][v] = C[16 i + 4 lg + v][16 j + l16] of the wavefront's sub-tile
  f32x4_t acc[NI][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

  // Second set of accumulators.  fp32: for the five small pairs, so that the large sums are rounded once
  // per 32 terms and not six times (512^3: 1.3e-7 from the fp64 product instead of 1.6e-7, native fp32
  // MFMAs 2.1e-7).  bf16, 64 x 64: for every other 32 terms (chains half as long).
  constexpr bool TWO = PIECES > 1 || TILE == 64;
  f32x4_t low[NI][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) low[i][j][v] = 0.f;

  // 64 x 64: a third set, for shorter chains again.  fp32: the first half of the range (1024^3 in three ranges of k:
  // 1.10e-7 from the fp64 product with one chain, 8.7e-8 with two; in four ranges with one 9.8e-8).  FOLD: what has been put aside.
  constexpr bool HALVES = PIECES > 1 && TILE == 64;
  static_assert(!FOLD || (PIECES == 1 && TILE == 64), "bf16 tiles of 64");
  constexpr int NT = HALVES || FOLD ? NI : 1;
  f32x4_t third[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) third[i][j][v] = 0.f;
  const int k_mid = k_begin + ((k_end - k_begin) / (2 * BK)) * BK;

  Stager<DT, TILE, KCA, D> sa;
  Stager<DT, TILE, KCB, D> sb;
  sa.init(A, a.lda, tile_r0, a.n, k_end);
  sb.init(B, a.ldb, tile_c0, a.m, k_end);
  const bool once = DT == GECC_F32 && a.k <= BK;       // (then k is not split)
  const bool is_short = !FOLD && a.k < 16;             // (a row has no vector then, or a thread no KPT values of k)
  // fresh: whether the sums start anew with this k-tile
  auto multiply = [&](const char* As, const char* Bs, auto fresh) {
    constexpr bool NEW = decltype(fresh)::value;
    static_assert(!NEW || BK == 64, "one step of either set");
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      bf16x8_t fb[NI][PIECES];
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
          fb[j][q] = *reinterpret_cast<const bf16x8_t*>(Bs + q * PLANE + lds_at<BK>(wc * W + j * 16 + l16, ks * 4 + lg));
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        bf16x8_t fa[PIECES];
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
          fa[q] = *reinterpret_cast<const bf16x8_t*>(As + q * PLANE + lds_at<BK>(wr * W + i * 16 + l16, ks * 4 + lg));
        // pairs of pieces, the small ones first
#pragma unroll
        for (int o = PIECES - 1; o > 0; --o)
#pragma unroll
          for (int q = o; q >= 0; --q)
#pragma unroll
            for (int j = 0; j < NI; ++j)
              low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[q], fb[j][o - q], low[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          f32x4_t& sum = PIECES == 1 && TWO && (ks & 1) ? low[i][j] : acc[i][j];
          sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0], fb[j][0], NEW ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
        }
      }
    }
  };
  if (is_short) {
    // (one k-tile, element by element)
    sa.load_short(k_begin);
    sb.load_short(k_begin);
    if (!once) {
      sa.store(smem, 0);
      sb.store(smem + OPERAND, 0);
      __syncthreads();
      multiply(smem, smem + OPERAND, std::false_type{});
    }
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d) { sa.load(k_begin + d * BK, d); sb.load(k_begin + d * BK, d); }
    if (once) { sa.fix(k_begin, 0); sb.fix(k_begin, 0); }
    if constexpr (FOLD) {
      // (a k-tile, in half d of the LDS; fresh: the first of a piece)
      auto tile = [&](int k0, auto half, auto fresh) {
        constexpr int d = decltype(half)::value;
        char* As = smem + d * 2 * OPERAND;
        if (k0 + BK > k_end) { sa.fix(k0, d); sb.fix(k0, d); }
        sa.store(As, d);
        sb.store(As + OPERAND, d);
        __syncthreads();
        sa.load(k0 + D * BK, d);
        sb.load(k0 + D * BK, d);
        multiply(As, As + OPERAND, fresh);
      };
      const std::integral_constant<int, 0> even{};
      const std::integral_constant<int, 1> odd{};
      for (int k1 = k_begin; k1 < k_end; k1 += a.k_fold) {
        const int k_to = min(k_end, k1 + a.k_fold);
        tile(k1, even, std::true_type{});
        if (k1 + BK < k_to) tile(k1 + BK, odd, std::false_type{});
        for (int kt = k1 + 2 * BK; kt < k_to; kt += 2 * BK) {
          tile(kt, even, std::false_type{});
          if (kt + BK < k_to) tile(kt + BK, odd, std::false_type{});
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) third[i][j][v] += acc[i][j][v] + low[i][j][v];
      }
    } else {
    for (int kt = once ? k_end : k_begin; kt < k_end; kt += D * BK)
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k0 = kt + d * BK;
      if (d > 0 && k0 >= k_end) break;
      char* As = smem + (TWICE && (d & 1) ? 2 * OPERAND : 0);
      char* Bs = As + OPERAND;
      if (!TWICE) __syncthreads();   // previous tile fully consumed
      if (k0 + BK > k_end) { sa.fix(k0, d); sb.fix(k0, d); }
      sa.store(As, d);
      sb.store(Bs, d);
      __syncthreads();
      sa.load(k0 + D * BK, d);
      sb.load(k0 + D * BK, d);
      if constexpr (HALVES) {
        if (k0 == k_mid) {
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
              for (int v = 0; v < 4; ++v) { third[i][j][v] = acc[i][j][v]; acc[i][j][v] = 0.f; }
        }
      }
      multiply(As, Bs, std::false_type{});
    }
    }
  }

  if constexpr (TWO) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float x = third[NT > 1 ? i : 0][NT > 1 ? j : 0][v];
          acc[i][j][v] = HALVES ? (acc[i][j][v] + x) + low[i][j][v] : FOLD ? x : acc[i][j][v] + low[i][j][v];
        }
  }
  if constexpr (DT == GECC_F32) {
    if (once) {
      // The only k-tile, as it is, through fp64 MFMAs.  Their result has row 4 v + lg where the others have 4 lg + v:
      // lane l16 is given the row of A that makes up for it.
      float* Ap = reinterpret_cast<float*>(smem);
      float* Bp = Ap + TILE * (BK + 1);
      sa.store_plain(Ap);
      sb.store_plain(Bp);
      __syncthreads();
      const float* fa = Ap + (wr * W + 4 * (l16 & 3) + (l16 >> 2)) * (BK + 1) + lg;
      const float* fb = Bp + (wc * W + l16) * (BK + 1) + lg;
      constexpr int IB = 4 / NI;                     // four independent chains
#pragma unroll
      for (int i0 = 0; i0 < NI; i0 += IB) {
        f64x4_t d[IB][NI];
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) d[i][j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int ks = 0; ks < a.k; ks += 4) {
          double x[IB], y[NI];
#pragma unroll
          for (int i = 0; i < IB; ++i) x[i] = fa[(i0 + i) * 16 * (BK + 1) + ks];
#pragma unroll
          for (int j = 0; j < NI; ++j) y[j] = fb[j * 16 * (BK + 1) + ks];
#pragma unroll
          for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) d[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], y[j], d[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i0 + i][j][v] = (float)d[i][j][v];
      }
    }
  }
  // rows and columns past the end count as zero
  mask_edges<TILE>(a, tile_r0, tile_c0, acc);

  if constexpr (DT == GECC_F32) {
    float worst = 0.f;             // 0, or NaN when some accumulator is not finite
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) worst = fmaf(acc[i][j][v], 0.f, worst);
    if (__syncthreads_or(!once && (worst != 0.f || sa.tiny() || sb.tiny()))) {
      // native fp32 pass (see the head of this file)
      float* Ap = reinterpret_cast<float*>(smem);
      float* Bp = Ap + TILE * (BK + 1);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
      for (int k0 = k_begin; k0 < k_end; k0 += BK) {
        sa.load(k0, 0);
        sb.load(k0, 0);
        if (k0 + BK > k_end) { sa.fix(k0, 0); sb.fix(k0, 0); }
        __syncthreads();
        sa.store_plain(Ap);
        sb.store_plain(Bp);
        __syncthreads();
#pragma unroll 1
        for (int ks = 0; ks < BK; ks += 4) {
          float fb[NI];
#pragma unroll
          for (int j = 0; j < NI; ++j) fb[j] = Bp[(wc * W + j * 16 + l16) * (BK + 1) + ks + lg];
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            const float fa = Ap[(wr * W + i * 16 + l16) * (BK + 1) + ks + lg];
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa, fb[j], acc[i][j], 0, 0, 0);
          }
        }
      }
      mask_edges<TILE>(a, tile_r0, tile_c0, acc);
    }
  }

  if (S > 1 && !add_splits<TILE>(a, b, tm, tn, split, S, acc, smem)) return;
  finish_tile<TILE>(a, b, tm, tn, acc, smem);
}

// -------------------------------------------------------------------------------------------
// Stand-alone partial sums of a C that sits in HBM (same TILE x TILE tiling and workspace layout
// as the fused epilogues).  HBM-bound: every thread streams RPT rows x 4 columns with 16-byte
// loads (full tile rows per wavefront instruction), keeps its row and column partial sums in
// registers, and the workgroup combines them through LDS in a fixed order.
// STREAM: nothing it reads is kept in the caches -- for a C well beyond the 256 MiB of the memory-side cache
// (940 MB: 156 us = 6.0 TB/s, with ordinary loads 172 to 175; 268 MB, part of which the last writer or reader
// left there, 44 against 41).
template <int TILE, bool STREAM>
__global__ __launch_bounds__(THREADS) void partials_kernel(PartialArgs a) {
  constexpr int CG = TILE / 4, RG = THREADS / CG, RPT = TILE / RG;   // column groups of 4, row groups of RPT
  const int b = blockIdx.z;
  const int tm = blockIdx.y, tn = blockIdx.x;
  if (tm == 0 && tn == 0 && threadIdx.x == 0) reset_state(a.state + b);      // (nothing in this launch reads it)
  const int tile_r0 = tm * TILE, tile_c0 = tn * TILE;
  const float* C = a.C + (int64_t)b * a.sc;
  const int tid = threadIdx.x;
  const int cg = tid % CG, rg = tid / CG;
  const int gj = tile_c0 + cg * 4;
  const bool vec = (reinterpret_cast<uintptr_t>(C) % 16 == 0) && (a.ldc % 4 == 0) && gj + 4 <= a.m;
  __shared__ float red_row[2][TILE][CG + 1];
  __shared__ float red_col[2][RG][TILE];
  float cs[4] = {0.f, 0.f, 0.f, 0.f}, cw[4] = {0.f, 0.f, 0.f, 0.f};
  // the kernel is a stream over C: all loads of a thread are issued before the first is used
  // (rows past the end are clamped, not branched on, and count as zero below)
  f32x4_t pre[RPT];
  if (vec) {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const f32x4_t* src = reinterpret_cast<const f32x4_t*>(C + (int64_t)min(tile_r0 + rg * RPT + r, a.n - 1) * a.ldc + gj);
      pre[r] = STREAM ? __builtin_nontemporal_load(src) : *src;
    }
  }
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int rl = rg * RPT + r, gi = tile_r0 + rl;
    float x[4] = {0.f, 0.f, 0.f, 0.f};
    if (gi < a.n) {
      if (vec) {
        x[0] = pre[r].x; x[1] = pre[r].y; x[2] = pre[r].z; x[3] = pre[r].w;
      } else {
        const float* src = C + (int64_t)gi * a.ldc + gj;
        for (int e = 0; e < 4; ++e) if (gj + e < a.m) x[e] = src[e];
      }
    }
    float rs = 0.f, rw = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      cs[e] += x[e];
      cw[e] = fmaf((float)(rl + 1), x[e], cw[e]);
      rs += x[e];
      rw = fmaf((float)(cg * 4 + e + 1), x[e], rw);
    }
    red_row[0][rl][cg] = rs;
    red_row[1][rl][cg] = rw;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    red_col[0][rg][cg * 4 + e] = cs[e];
    red_col[1][rg][cg * 4 + e] = cw[e];
  }
  __syncthreads();
  if (tid < TILE) {
    float s = 0.f, w = 0.f;
#pragma unroll
    for (int c = 0; c < CG; ++c) { s += red_row[0][tid][c]; w += red_row[1][tid][c]; }
    const int gi = tile_r0 + tid;
    if (gi < a.n) {
      float2* rp = reinterpret_cast<float2*>(a.rowpart + (((int64_t)b * a.ntn + tn) * a.rp_ld + gi) * 2);
      *rp = make_float2(s, w);
    }
  } else if (tid < 2 * TILE) {
    const int c = tid - TILE;
    float s = 0.f, w = 0.f;
#pragma unroll
    for (int g = 0; g < RG; ++g) { s += red_col[0][g][c]; w += red_col[1][g][c]; }
    const int gc = tile_c0 + c;
    if (gc < a.m) {
      float2* cp = reinterpret_cast<float2*>(a.colpart + (((int64_t)b * a.ntm + tm) * a.cp_ld + gc) * 2);
      *cp = make_float2(s, w);
    }
  }
}

// The scans come first where all workgroups of the launch run at once (256 compute units with as many as their
// registers and LDS allow): nobody waits for a place, and theirs is the longer chain.  Beyond that they come behind:
// what does not fit at first is then short scans and not workgroups of the product that begin 5 us late and last 20.
// Whole calls, us, scans first -> behind:
//   beyond that number, 87 products of all layouts, 0.3 % slower to 20 % faster
//     bf16 295 x 6020 x 4321    100 -> 82         bf16 4648 x 1232 x 272 NT   52.4 -> 44.0
//     bf16 2432 x 3584 x 256    56.5 -> 50.6      fp32 1991 x 1907 x 220      49.7 -> 44.2
//   below it, 4 % slower to 7 % faster
//     bf16 192 x 3520 x 1408    39.8 -> 41.3      TT 1216 x 960 x 576         76.8 -> 80.5
// P_g, one workgroup with a long chain, goes first in either case (behind: no difference seen).  Behind, a column
// scan, whose workgroups take longer, comes before a row scan (bf16 TT 1632 x 624 x 2328 40.9 us, the other way
// round 46.7; first, where it is the other way round 34.7 -> 34.1 at 1536 x 1280 x 256).
template <int DT, int TILE> constexpr int at_once() { return 256 * (TILE == 64 ? 4 : DT == GECC_BF16 ? 3 : 2); }

// bf16 tiles of 64 in fewer ranges of k than they could have: terms after which the accumulators are added to the
// third set and start anew, for a range of k_per terms.  A chain of N additions is off by N^2 / 2 squared last bits
// (a walk that grows); B pieces with a chain of their sums by N^2 / 2B + NB / 2, least where B is about sqrt(N).
// Distance of the product from the fp64 one, in 1e-8 (normal operands):
//   terms of a piece   128   192   256   384   512   no pieces
//   range of  260      6.0   6.1   6.8   6.6   6.6    6.6
//   range of  700      7.1   7.1   7.3   8.0   8.7   10.5
//   range of 1000      7.6   7.7   7.7   8.3   9.3   12.6
//   range of 2112      9.9   9.2   9.3   9.6  10.5   19.1
//   range of 5800     13.7  12.1  11.3  11.1  11.3   32.9
// (700 terms in four ranges 7.1.)  Products alone, us, pieces of 128, 256, 384 terms / in the kernel without pieces:
//   700^3               8.9  8.7  8.6 / 8.8   (with the sums set to zero, and not begun by a product that adds
//   3976 x 456 x 176 TN 8.8  8.5  8.5 / 8.7    nothing, pieces of 128 terms 9.6)
//   2056 x 664 x 168    8.8  8.7  8.6 / 8.7
// A kernel of its own all the same: the loop twice is more code than most products need (as a branch in the one for
// all bf16 tiles of 64 it cost 1500 x 1000 x 1100 2 %).
int k_fold_of(int k_per) {
  constexpr int STEP = 128;        // (two k-tiles, one to each half of the LDS)
  const int steps = (int)(5.0 * sqrt((double)k_per) / STEP + 0.5);
  return STEP * (steps > 1 ? steps : 1);
}

template <int DT, int TILE>
hipError_t launch_tile(const GemmArgs& a0, const GemmSide* side0, hipStream_t st) {
  GemmArgs a = a0;
  const int64_t tiles = (int64_t)((a.m + TILE - 1) / TILE) * ((a.n + TILE - 1) / TILE) * a.batch;
  if (a.ksplit > 1 && a.split_part && a.split_done && tiles <= SCAN_DONE_WORDS) {
    if ((size_t)tiles * a.ksplit * TILE * TILE * sizeof(float) > a.split_bytes) return hipErrorInvalidValue;
    const int bk = GT<DT>::BK;
    a.k_per = ((a.k + a.ksplit - 1) / a.ksplit + bk - 1) / bk * bk;
  } else {
    a.ksplit = 1;
  }
  GemmSide side = side0 ? *side0 : GemmSide{};
  side.pg_items = a.pg_out ? a.batch : 0;
  side.blocks = side.pg_items + side.j[0].nblk + side.j[1].nblk;
  const int64_t own = tiles * a.ksplit;
  const bool behind = own + side.blocks > at_once<DT, TILE>();
  side.lead_blocks = behind ? side.pg_items : side.blocks;
  if (behind && side.j[0].kind != SIDE_COL && side.j[1].kind == SIDE_COL) {
    const SideJob row = side.j[0];
    side.j[0] = side.j[1];
    side.j[1] = row;
  }
  side.lead = (side.lead_blocks + 7) / 8;
  side.groups = side.lead + (side.blocks - side.lead_blocks + 7) / 8;
  const int64_t grid_all = side.groups > 0 ? ((own + 7) / 8 + side.groups) * 8 : own;
  if (grid_all > 0xffffff) return hipErrorInvalidValue;      // (2^32 threads)
  side.own = (int)own;
  const dim3 grid((unsigned)grid_all);
  // k-contiguous storage: A when not transposed, B when transposed
  const bool kca = a.trans_a == 0, kcb = a.trans_b != 0;
  auto launch = [&](auto what) {
    constexpr int WHAT = decltype(what)::value;
    if (kca && kcb)        hipLaunchKernelGGL((gemm_tile<WHAT, true, true, TILE>), grid, dim3(THREADS), 0, st, a, side);
    else if (kca && !kcb)  hipLaunchKernelGGL((gemm_tile<WHAT, true, false, TILE>), grid, dim3(THREADS), 0, st, a, side);
    else if (!kca && kcb)  hipLaunchKernelGGL((gemm_tile<WHAT, false, true, TILE>), grid, dim3(THREADS), 0, st, a, side);
    else                   hipLaunchKernelGGL((gemm_tile<WHAT, false, false, TILE>), grid, dim3(THREADS), 0, st, a, side);
  };
  if constexpr (DT == GECC_BF16 && TILE == 64) {
    if (a.fold && a.k >= 16) {
      a.k_fold = k_fold_of(a.ksplit > 1 ? a.k_per : a.k);
      launch(std::integral_constant<int, BF16_FOLD>{});
      return hipGetLastError();
    }
  }
  launch(std::integral_constant<int, DT>{});
  return hipGetLastError();
}

}  // namespace

bool gemm_takes_256(const GemmArgs& a) { return a.fast && gemm_bf16_fast_ok(a); }

hipError_t launch_gemm(const GemmArgs& a, const GemmSide* side, hipStream_t st) {
  if (a.tile_m != a.tile_n || (a.tile_m != 128 && a.tile_m != 64)) return hipErrorInvalidValue;
  if (gemm_takes_256(a)) return side ? hipErrorInvalidValue : launch_gemm_bf16_fast(a, st);
  if (a.tile_m == 64) return a.dtype == GECC_BF16 ? launch_tile<GECC_BF16, 64>(a, side, st) : launch_tile<GECC_F32, 64>(a, side, st);
  if (a.dtype == GECC_BF16) return launch_tile<GECC_BF16, 128>(a, side, st);
  return !side && gemm_f32_wide_pays(a) ? launch_gemm_f32_wide(a, st) : launch_tile<GECC_F32, 128>(a, side, st);
}

namespace {
// C += P, 16 bytes per thread where the rows allow it
__global__ __launch_bounds__(256) void accumulate_kernel(float* C, const float* P, int n, int m, int64_t ldc, int vec_ok) {
  const int64_t total4 = (int64_t)n * ((m + 3) / 4);
  for (int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x; o < total4; o += (int64_t)gridDim.x * 256) {
    const int64_t i = o / ((m + 3) / 4);
    const int j = (int)(o - i * ((m + 3) / 4)) * 4;
    float* c = C + i * ldc + j;
    const float* p = P + i * ldc + j;
    if (vec_ok && j + 4 <= m) {
      float4 x = *reinterpret_cast<const float4*>(c);
      const float4 y = *reinterpret_cast<const float4*>(p);
      x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
      *reinterpret_cast<float4*>(c) = x;
    } else {
      for (int e = 0; e < 4 && j + e < m; ++e) c[e] += p[e];
    }
  }
}
}  // namespace

hipError_t launch_accumulate(float* C, const float* P, int n, int m, int64_t ldc, hipStream_t st) {
  const int vec_ok = ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
  const int64_t total4 = (int64_t)n * ((m + 3) / 4);
  const int blocks = (int)((total4 + 255) / 256 < 16384 ? (total4 + 255) / 256 : 16384);
  hipLaunchKernelGGL(accumulate_kernel, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, st, C, P, n, m, ldc, vec_ok);
  return hipGetLastError();
}

hipError_t launch_partials(const PartialArgs& a, hipStream_t st) {
  if (a.tile_m != a.tile_n || (a.tile_m != 128 && a.tile_m != 64)) return hipErrorInvalidValue;
  dim3 grid(a.ntn, a.ntm, a.batch);
  const bool stream = (int64_t)a.n * a.m * a.batch > ((int64_t)96 << 20);    // 384 MiB
  if (a.tile_m == 64) {
    if (stream) hipLaunchKernelGGL((partials_kernel<64, true>), grid, dim3(THREADS), 0, st, a);
    else        hipLaunchKernelGGL((partials_kernel<64, false>), grid, dim3(THREADS), 0, st, a);
  } else {
    if (stream) hipLaunchKernelGGL((partials_kernel<128, true>), grid, dim3(THREADS), 0, st, a);
    else        hipLaunchKernelGGL((partials_kernel<128, false>), grid, dim3(THREADS), 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace gecc
