// Large fp32 products: tiles of 128 x 256, 8 wavefronts (2 x 4), one workgroup per compute unit, two k-tiles in LDS; the
// arithmetic of gemm_kernels.hip (three bf16 pieces per value, six products; 128 x 128 symbols whose operands the pieces
// cannot hold again with native fp32 MFMAs) in the same order, so that the results are the same to the bit.
// Beside gemm_kernels.hip and not in it: as one template, that kernel's bf16 instances took 188 registers for 157.
#include "gemm_device.h"

namespace gecc {
namespace {

constexpr int BK = 32, PIECES = 3, TILE = 128, W = TILE / 2, NI = W / 16;      // W x W per wavefront
constexpr int WC = 4, TILE_N = WC * W, NT = 64 * 2 * WC;

// buffer descriptor of everything from p on: the loads through it are in bounds by construction, as any others
__device__ __forceinline__ __amdgpu_buffer_rsrc_t whole_memory(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00027000);
}

// ---- staging of one operand tile: ROWS (m- or n-index) x BK ------------------------------------
// KC: element (r, kk) lives at P[r * ld + kk]; otherwise at P[kk * ld + r].  Rows past the last one are clamped to it (what
// they accumulate is masked in the epilogue), k past the end reads as zero.  What a thread stages comes in CHUNKS.
template <int ROWS, bool KC> struct WideStager;

// k contiguous: 16-byte loads, eight lanes to a row
template <int ROWS>
struct WideStager<ROWS, true> {
  static constexpr int N = ROWS * BK / 4 / NT, RSTEP = NT / 8, CHUNKS = N;
  static constexpr int PLANE = ROWS * BK * 2;
  __amdgpu_buffer_rsrc_t rsrc;
  const float* src;
  uint32_t off[N];
  uint4 reg[N];
  Least least;      // of the values this thread has staged
  int kk, klim;
  __device__ __forceinline__ void init(const float* P, int64_t ld, int r0, int rlim, int k_end) {
    kk = (threadIdx.x & 7) * 4;
    klim = k_end;
    src = P + (int64_t)r0 * ld;
    rsrc = whole_memory(src);
#pragma unroll
    for (int i = 0; i < N; ++i)
      off[i] = ((uint32_t)(min(r0 + (int)(threadIdx.x >> 3) + RSTEP * i, rlim - 1) - r0) * (uint32_t)ld + (uint32_t)kk) * 4u;
  }
  // (the whole k-tile lies before the end of k)
  __device__ __forceinline__ void load_chunk(int k0, int i) {
    reg[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off[i], k0 * 4, 0));
  }
  __device__ __forceinline__ void load(int k0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (k0 + BK <= klim) {
        load_chunk(k0, i);
      } else {
        const float* p = reinterpret_cast<const float*>(reinterpret_cast<const char*>(src + k0) + off[i]);
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = k0 + kk + e < klim ? p[e] : 0.f;
        __builtin_memcpy(&reg[i], x, 16);
      }
    }
  }
  __device__ __forceinline__ void store_chunk(char* S, int i) {
    const int row = (threadIdx.x >> 3) + RSTEP * i;
    const float x[4] = {__uint_as_float(reg[i].x), __uint_as_float(reg[i].y), __uint_as_float(reg[i].z), __uint_as_float(reg[i].w)};
    uint32_t a[3], b[3];
    split2(x[0], x[1], a);
    split2(x[2], x[3], b);
    least.see(x[0], x[1]);
    least.see(x[2], x[3]);
    char* dst = S + lds_at<BK>(row, (threadIdx.x & 7) >> 1) + (threadIdx.x & 1) * 8;
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(dst + q * PLANE) = make_uint2(a[q], b[q]);
  }
  __device__ __forceinline__ void store(char* S) {
#pragma unroll
    for (int i = 0; i < N; ++i) store_chunk(S, i);
  }
  __device__ __forceinline__ bool tiny() const { return least.tiny(); }
  // the loaded values, each 128 rows into a minimum of their own
  __device__ __forceinline__ void see(Least* of) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      static_assert(TILE % RSTEP == 0, "rows of one load in one half");
      of[RSTEP * i / TILE].see(__uint_as_float(reg[i].x), __uint_as_float(reg[i].y));
      of[RSTEP * i / TILE].see(__uint_as_float(reg[i].z), __uint_as_float(reg[i].w));
    }
  }
  // the fp32 values as they are, rows of BK + 1 floats (native fp32 pass)
  __device__ __forceinline__ void store_plain(float* S) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      float* d = S + ((threadIdx.x >> 3) + RSTEP * i) * (BK + 1) + kk;
      d[0] = __uint_as_float(reg[i].x); d[1] = __uint_as_float(reg[i].y);
      d[2] = __uint_as_float(reg[i].z); d[3] = __uint_as_float(reg[i].w);
    }
  }
};

// r contiguous: a thread owns one row and KPT consecutive k (a wavefront reads 256 contiguous bytes of a k-row per
// instruction), so that its stores are whole 16-byte chunks along k
template <int ROWS>
struct WideStager<ROWS, false> {
  static constexpr int KPT = ROWS * BK / NT, CHUNKS = KPT / 8;
  static constexpr int PLANE = ROWS * BK * 2;
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off;
  float reg[KPT];
  Least least;
  int64_t ld;
  int row, kg, klim;
  __device__ __forceinline__ void init(const float* P, int64_t ld_, int r0, int rlim, int k_end) {
    row = threadIdx.x & (ROWS - 1);
    kg = __builtin_amdgcn_readfirstlane(threadIdx.x / ROWS) * KPT;     // ROWS >= 64: one k group per wavefront
    ld = ld_; klim = k_end;
    rsrc = whole_memory(P + r0);
    off = (uint32_t)(min(r0 + row, rlim - 1) - r0) * 4u;
  }
  __device__ __forceinline__ float at(int k) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off, (int)((uint32_t)k * (uint32_t)ld * 4u), 0));
  }
  __device__ __forceinline__ void load_chunk(int k0, int c) {
#pragma unroll
    for (int x = c * 8; x < c * 8 + 8; ++x) reg[x] = at(k0 + kg + x);
  }
  __device__ __forceinline__ void load(int k0) {
#pragma unroll
    for (int x = 0; x < KPT; ++x) reg[x] = k0 + kg + x < klim ? at(k0 + kg + x) : 0.f;
  }
  __device__ __forceinline__ void store_chunk(char* S, int c) {
    uint32_t p[4][3];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const float x0 = reg[c * 8 + 2 * h], x1 = reg[c * 8 + 2 * h + 1];
      split2(x0, x1, p[h]);
      least.see(x0, x1);
    }
    char* dst = S + lds_at<BK>(row, (kg >> 3) + c);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(dst + q * PLANE) = make_uint4(p[0][q], p[1][q], p[2][q], p[3][q]);
  }
  __device__ __forceinline__ void store(char* S) {
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) store_chunk(S, c);
  }
  __device__ __forceinline__ bool tiny() const { return least.tiny(); }
  __device__ __forceinline__ void see(Least* of) const {
#pragma unroll
    for (int h = 0; h < ROWS / TILE; ++h)
      if (row / TILE == h) {
#pragma unroll
        for (int x = 0; x < KPT; x += 2) of[h].see(reg[x], reg[x + 1]);
      }
  }
  __device__ __forceinline__ void store_plain(float* S) const {
#pragma unroll
    for (int x = 0; x < KPT; ++x) S[row * (BK + 1) + kg + x] = reg[x];
  }
};

// -------------------------------------------------------------------------------------------
template <bool KCA, bool KCB>
__global__ __launch_bounds__(NT, 2) void gemm_f32_wide(GemmArgs a, int pg_groups, int own) {
  constexpr int PLANE = TILE * BK * 2, OPERAND = PIECES * PLANE, PLANE_B = TILE_N * BK * 2, BUFFER = OPERAND + PIECES * PLANE_B;
  static_assert(2 * BUFFER >= (TILE + TILE_N) * (BK + 1) * 4 && 2 * BUFFER >= GECC_MAX_FAULTS * 8 + 16, "what else lies in LDS");
  __shared__ __attribute__((aligned(16))) char smem[2 * BUFFER];
  const int ntm = (a.n + TILE - 1) / TILE, ntn = (a.m + TILE_N - 1) / TILE_N;
  int id = blockIdx.x;
  // P_g first, in whole groups of 8 workgroups (one per XCD), then the tiles: a contiguous range for every XCD
  if (id < pg_groups * 8) {
    if (id < a.batch) form_pg<THREADS>(a, id, reinterpret_cast<double*>(smem));     // (in the order of gemm_tile's 256 threads)
    return;
  }
  id -= pg_groups * 8;
  if (id >= own) return;
  {
    const int per = own / 8, rem = own - per * 8, x = id & 7;
    id = x * per + min(x, rem) + (id >> 3);
  }
  const int tn = id % ntn, tm = (id / ntn) % ntm, b = id / (ntn * ntm);
  const int tile_r0 = tm * TILE, tile_c0 = tn * TILE_N;
  const float* A = reinterpret_cast<const float*>(a.A) + (int64_t)b * a.sa;
  const float* B = reinterpret_cast<const float*>(a.B) + (int64_t)b * a.sb;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / WC, wc = wave % WC;
  const int l16 = lane & 15, lg = lane >> 4;

  // acc[i][j][v] = C[16 i + 4 lg + v][16 j + l16] of the wavefront's sub-tile
  f32x4_t acc[NI][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

  // second set of accumulators, for the five small pairs
  f32x4_t low[NI][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) low[i][j][v] = 0.f;

  WideStager<TILE, KCA> sa;
  WideStager<TILE_N, KCB> sb;
  sa.init(A, a.lda, tile_r0, a.n, a.k);
  sb.init(B, a.ldb, tile_c0, a.m, a.k);
  sa.load(0);
  sb.load(0);

  // Two k-tiles in LDS, one barrier per k-tile: while one is multiplied the next one's pieces are formed from registers,
  // three vector instructions behind every MFMA, and the registers are loaded again for the one after it.  With 128 x 128
  // tiles, matrix pipes (44 % of the cycles) and vector units (39 %) took turns: 256 x 512^3 434 us, here (49 and 27 %) 398.
  // What bounds it: registers (with B's fragments of all four column blocks held at once more of them spill, and a reload
  // waits for every load from memory that was issued before it: 495 us; as it is NN and TN spill none, TT two and NT six),
  // the first fragment reads behind each barrier and prologue and epilogue, which nothing else on the compute unit covers.
  // The MFMAs of one k-tile that lies in LDS; between(s): what comes with those of section s, a block of 16 rows and half of
  // the wavefront's columns.
  constexpr int NJ = NI / 2, SECTIONS = 2 * NI;
  auto multiply = [&](const char* Ap, const char* Bp, auto between) {
#pragma unroll
    for (int j0 = 0; j0 < NI; j0 += NJ) {
      bf16x8_t fb[NJ][PIECES];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
          fb[j][q] = *reinterpret_cast<const bf16x8_t*>(Bp + q * PLANE_B + lds_at<BK>(wc * W + (j0 + j) * 16 + l16, lg));
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        bf16x8_t fa[PIECES];
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
          fa[q] = *reinterpret_cast<const bf16x8_t*>(Ap + q * PLANE + lds_at<BK>(wr * W + i * 16 + l16, lg));
        between(j0 / NJ * NI + i);
        // pairs of pieces, the small ones first
#pragma unroll
        for (int o = PIECES - 1; o > 0; --o)
#pragma unroll
          for (int q = o; q >= 0; --q)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
              low[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[q], fb[j][o - q], low[i][j0 + j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0], fb[j][0], acc[i][j0 + j], 0, 0, 0);
      }
    }
  };
  auto lds_barrier = [&] {       // (__syncthreads() would also wait for the loads from memory)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  constexpr int CA = decltype(sa)::CHUNKS, CB = decltype(sb)::CHUNKS;
  sa.store(smem);
  sb.store(smem + OPERAND);
  if (BK < a.k) { sa.load(BK); sb.load(BK); }
  lds_barrier();
  int at = 0, k0 = 0;
  for (; k0 + 3 * BK <= a.k; k0 += BK) {
    char* cur = smem + at;
    char* next = smem + (BUFFER - at);
    multiply(cur, cur + OPERAND, [&](int sec) {
      // the chunks, spread over all sections but the last
#pragma unroll
      for (int c = 0; c < CA + CB; ++c)
        if (sec == c * (SECTIONS - 1) / (CA + CB)) {
          if (c < CA) { sa.store_chunk(next, c); sa.load_chunk(k0 + 2 * BK, c); }
          else { sb.store_chunk(next + OPERAND, c - CA); sb.load_chunk(k0 + 2 * BK, c - CA); }
        }
    });
#pragma unroll
    for (int x = 0; x < NI * NI * 6; ++x) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // an MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);    // and the vector instructions that fit behind it
    }
    lds_barrier();
    at = BUFFER - at;
  }
  for (; k0 < a.k; k0 += BK) {
    char* cur = smem + at;
    char* next = smem + (BUFFER - at);
    if (k0 + BK < a.k) { sa.store(next); sb.store(next + OPERAND); }
    if (k0 + 2 * BK < a.k) { sa.load(k0 + 2 * BK); sb.load(k0 + 2 * BK); }
    multiply(cur, cur + OPERAND, [](int) {});
    lds_barrier();
    at = BUFFER - at;
  }
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] += low[i][j][v];
  // rows and columns past the end count as zero
  if (tile_r0 + TILE > a.n || tile_c0 + TILE_N > a.m) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (tile_r0 + wr * W + i * 16 + lg * 4 + v >= a.n || tile_c0 + wc * W + j * 16 + l16 >= a.m) acc[i][j][v] = 0.f;
  }

  float worst = 0.f;             // 0, or NaN when some accumulator is not finite
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) worst = fmaf(acc[i][j][v], 0.f, worst);
  if (__syncthreads_or((worst != 0.f || sa.tiny() || sb.tiny()))) {
    // Native fp32 pass (see the head of gemm_kernels.hip).  Each half of 128 columns takes its sums only where that half
    // needs them and else keeps what its pieces gave, as in a tile of its own; which half a tiny value lies in is seen here
    // (a second minimum in the k loop is a register, and there is none left).
    Least least_a, least_b[TILE_N / TILE];
    float* Ap = reinterpret_cast<float*>(smem);
    float* Bp = Ap + TILE * (BK + 1);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) low[i][j][v] = 0.f;
    for (int k0 = 0; k0 < a.k; k0 += BK) {
      sa.load(k0);
      sb.load(k0);
      sa.see(&least_a);
      sb.see(least_b);
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
          for (int j = 0; j < NI; ++j) low[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa, fb[j], low[i][j], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int h = 0; h < TILE_N / TILE; ++h) {
      const bool mine = wc * W / TILE == h;
      if (__syncthreads_or((mine && worst != 0.f) || least_a.tiny() || least_b[h].tiny()) && mine) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const bool in = tile_r0 + wr * W + i * 16 + lg * 4 + v < a.n && tile_c0 + wc * W + j * 16 + l16 < a.m;
              acc[i][j][v] = in ? low[i][j][v] : 0.f;
            }
      }
    }
  }

  // ---- epilogue, from the accumulators -------------------------------------------------------------
  // Test faults (none in production calls): the workgroup searches the list for those that strike its
  // tile, then every wavefront adds them to its accumulators.
  if (a.n_faults > 0) {
    int* hits = reinterpret_cast<int*>(smem);
    int2* hit = reinterpret_cast<int2*>(smem + 16);
    __syncthreads();
    if (tid == 0) *hits = 0;
    __syncthreads();
    for (int f = tid; f < a.n_faults; f += NT) {
      const gecc_fault ft = a.faults[f];
      const int r = ft.row - tile_r0, c = ft.col - tile_c0;
      if (ft.batch == b + a.fault_bias && r >= 0 && r < min(TILE, a.n - tile_r0) && c >= 0 && c < min(TILE_N, a.m - tile_c0))
        hit[atomicAdd(hits, 1)] = make_int2(r * TILE_N + c, __float_as_int(ft.offset));
    }
    __syncthreads();
    const int nh = *hits;
    for (int f = 0; f < nh; ++f) {
      const int r = hit[f].x / TILE_N - wr * W, c = hit[f].x % TILE_N - wc * W;
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
    const bool whole = tile_r0 + TILE <= a.n && tile_c0 + TILE_N <= a.m;
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
  float2* rowred = reinterpret_cast<float2*>(smem);          // [WC: wc][TILE]
  float2* colred = rowred + WC * TILE;                        // [2: wr][TILE_N]
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
      rowred[wc * TILE + wr * W + (l16 >> 2) * 16 + lg * 4 + (l16 & 3)] = make_float2(ks, fmaf((float)((wc & 1) * W), ks, kw));
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
    if (lg < NI) colred[wr * TILE_N + wc * W + lg * 16 + l16] = make_float2(cs, fmaf((float)(wr * W), cs, cw));
  }
  __syncthreads();
  // (a tile of TILE_N columns is WC / 2 sub-tiles)
  if (tid < TILE * WC / 2) {
    const int row = tid % TILE, sub = tid / TILE;
    const float2 x = rowred[2 * sub * TILE + row], y = rowred[(2 * sub + 1) * TILE + row];
    if (tile_r0 + row < a.n && tile_c0 + sub * TILE < a.m)
      *reinterpret_cast<float2*>(a.rowpart + (((int64_t)b * a.ntn + tn * (WC / 2) + sub) * a.rp_ld + tile_r0 + row) * 2) = make_float2(x.x + y.x, x.y + y.y);
  } else if (tid < TILE * WC / 2 + TILE_N) {
    const int c = tid - TILE * WC / 2;
    if (tile_c0 + c < a.m)
      *reinterpret_cast<float2*>(a.colpart + (((int64_t)b * a.ntm + tm) * a.cp_ld + tile_c0 + c) * 2) =
          make_float2(colred[c].x + colred[TILE_N + c].x, colred[c].y + colred[TILE_N + c].y);
  }
}

}  // namespace

namespace {
constexpr int64_t MAX_GRID = 0x7fffff;      // workgroups: 2^32 threads
// the tiles and P_g's workgroups, both in whole groups of 8
int64_t grid_of(const GemmArgs& a) {
  const int64_t own = (int64_t)((a.m + TILE_N - 1) / TILE_N) * ((a.n + TILE - 1) / TILE) * a.batch;
  return (own + 7) / 8 * 8 + (a.pg_out ? ((int64_t)a.batch + 7) / 8 * 8 : 0);
}
}  // namespace

// Whether an fp32 product of 128 x 128 tiles goes in tiles of 128 x 256: a round of 256 of those, one per compute unit,
// is done in 0.92 of the time of the same symbols in 512 of 128 x 128, two per compute unit, but has to be a whole one,
// while the smaller ones fill gaps.  Product alone, us, 128 x 128 -> 128 x 256:
//   yes   256 x 512^3     434 -> 398 (TT 429 -> 380)      no   48 x 500 x 321 x 381    64 -> 68
//         16 x 1024^3     197 -> 173                           100 x 384^3             76 -> 105
//         64 x 500^3      112 -> 99                            40 x 600^3              123 -> 143
bool gemm_f32_wide_pays(const GemmArgs& a) {
  if (a.dtype != GECC_F32 || a.ksplit > 1 || a.k < 128) return false;
  // (offsets of 32 bits: 256 rows, or k of them where rows run along the other axis)
  const int64_t rows_a = a.trans_a ? a.k : 128, rows_b = a.trans_b ? 256 : a.k;
  if (rows_a * a.lda >= ((int64_t)1 << 30) || rows_b * a.ldb >= ((int64_t)1 << 30)) return false;
  const int64_t tm = (a.n + 127) / 128, narrow = tm * ((a.m + 127) / 128) * a.batch, wide = tm * ((a.m + 255) / 256) * a.batch;
  return (wide + 255) / 256 * 471 < narrow && grid_of(a) <= MAX_GRID;
}

hipError_t launch_gemm_f32_wide(const GemmArgs& a, hipStream_t st) {
  const int64_t own = (int64_t)((a.m + TILE_N - 1) / TILE_N) * ((a.n + TILE - 1) / TILE) * a.batch;
  const int pg_groups = a.pg_out ? (a.batch + 7) / 8 : 0;
  if (grid_of(a) > MAX_GRID) return hipErrorInvalidValue;
  const dim3 grid((unsigned)grid_of(a)), block(NT);
  // k-contiguous storage: A when not transposed, B when transposed
  const bool kca = a.trans_a == 0, kcb = a.trans_b != 0;
  if (kca && kcb)        hipLaunchKernelGGL((gemm_f32_wide<true, true>), grid, block, 0, st, a, pg_groups, (int)own);
  else if (kca && !kcb)  hipLaunchKernelGGL((gemm_f32_wide<true, false>), grid, block, 0, st, a, pg_groups, (int)own);
  else if (!kca && kcb)  hipLaunchKernelGGL((gemm_f32_wide<false, true>), grid, block, 0, st, a, pg_groups, (int)own);
  else                   hipLaunchKernelGGL((gemm_f32_wide<false, false>), grid, block, 0, st, a, pg_groups, (int)own);
  return hipGetLastError();
}

}  // namespace gecc
