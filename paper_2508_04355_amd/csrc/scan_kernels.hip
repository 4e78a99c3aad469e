// HBM-bound weighted reductions over an operand: parity encoding (Section III, A_P and B_P),
// the parity blocks of the encoded product (P_r = A B_P, P_c = A_P B) and the operand audit.
//
// Both kernels read the operand once with 16-byte loads that are contiguous across a
// wavefront, accumulate in fp64 and reduce in a fixed order (no floating-point atomics), so
// that re-forming a parity from an unchanged operand reproduces it bit for bit.
#include "scan_device.h"
#include <cstdlib>

namespace gecc {
namespace {

// GATED: the launch belongs to the operand audit and returns at once unless the decoder asked for
// it (a separate instantiation, so that profiles list encoding and audit launches apart).
template <int DT, bool IDXW, bool GATED>
__global__ __launch_bounds__(RD_THREADS) void rowdot_wave_kernel(ScanArgs a) {
  __shared__ double lds[RW_LDS_DOUBLES];
  const int b = blockIdx.y;
  if (GATED && gated_off(a.gate, a.gate_stride, b, a.gate_value)) return;
  const int own = (int)gridDim.x - a.carry_blocks;
  if ((int)blockIdx.x >= own) {
    stage2_dispatch(a.carry, b, (int)blockIdx.x - own, lds);
    return;
  }
  rowdot_wave_body<DT, IDXW>(a, blockIdx.x, b, lds);
}
template <int DT, bool IDXW, int RD_RB, int RD_U, bool GATED>
__global__ __launch_bounds__(RD_THREADS) void rowdot_kernel(ScanArgs a) {
  __shared__ double lds[RD_RB * RD_THREADS];
  const int b = blockIdx.y;
  if (GATED && gated_off(a.gate, a.gate_stride, b, a.gate_value)) return;
  const int own = (int)gridDim.x - a.carry_blocks;
  if ((int)blockIdx.x >= own) {   // carried second stage of an earlier column / tile scan
    stage2_dispatch(a.carry, b, (int)blockIdx.x - own, lds);
    return;
  }
  rowdot_body<DT, IDXW, RD_RB, RD_U>(a, blockIdx.x, b, lds);
}

// Column scans of few workgroups take vectors of 8 bytes and twice the rows at once (see coldot_body).  With 16 -> 8
// bytes, bf16, us: one scan, 4096^2 index weights 8.9 -> 7.9, explicit 8.8 either way, 4096 x 14336 (896 workgroups)
// 25.4 -> 23.3; two in a launch, 2048^2 7.6 -> 7.0, 3001^2 13.9 -> 11.8, 4096^2 16.4 -> 23.0.
template <int DT, bool HALF> using ColElem = std::conditional_t<HALF, ElemHalf<DT>, Elem<DT>>;
constexpr int CD_HALF_BELOW = 1024, CD_PAIR_HALF_BELOW = 512;       // workgroups of the scan (of both of a pair) in vectors of 16 bytes

template <int DT, bool IDXW, bool GATED, bool ONE, bool HALF>
__global__ __launch_bounds__(CD_THREADS) void coldot_stage1(ScanArgs a, int nchunk) {
  __shared__ double lds[CD_LDS_DOUBLES];
  const int b = blockIdx.z;
  if (GATED && gated_off(a.gate, a.gate_stride, b, a.gate_value)) return;
  coldot_body<ColElem<DT, HALF>, IDXW, HALF ? 2 * CD_ROWS : CD_ROWS, ONE ? CD_ONE : CD_CHUNKS>(a, Parts{}, nchunk, gridDim.x, blockIdx.x, blockIdx.y, b, lds);
}

__global__ __launch_bounds__(256) void coldot_stage2(Stage2Job j) {
  __shared__ double lds[256];
  const int b = blockIdx.y;
  if (gated_off(j.gate, j.gate_stride, b, j.gate_value)) return;
  stage2_dispatch(j, b, blockIdx.x, lds);
}

// Two of them, not gated (own0: workgroups of j0, those of j1 come behind).  A kernel of its own: to read which job it is
// costs 0.3 to 0.6 us of the 3 to 4 that a single one takes.
__global__ __launch_bounds__(256) void coldot_stage2_pair(Stage2Job j0, Stage2Job j1, int own0) {
  __shared__ double lds[256];
  const int b = blockIdx.y;
  if ((int)blockIdx.x < own0) stage2_dispatch(j0, b, blockIdx.x, lds);
  else stage2_dispatch(j1, b, (int)blockIdx.x - own0, lds);
}

// Two scans that do not read each other's results (both encodings, or both parity blocks): what each of them would
// leave idle at its end the other one fills, and a launch that waits for the one before it costs 2 to 5 us whatever it does.
// Two parity blocks are scans of one kind, and each kind has a kernel of its own (in one for both, registers of the
// bf16 column scan spilled).  Row scans keep three wavefronts per SIMD (with two, 3072 x 2048 x 6144 NT 150.0 -> 152.5 us
// a call); column scans have the weights of four rows in registers, which is worth more than the third wavefront
// (spilled for it, 4096^3 TN 25.6 us for 16.4).
struct ScanPair { SideJob j[2]; };
enum : int { PAIR_ANY = 0,       // (explicit weights: row scans)
             PAIR_WAVE = 1,      // one of them a row scan with a wavefront per RW_RB rows, a third more registers than the others
             PAIR_COLS = 2 };    // two column scans
template <int DT, bool IDXW, int WHAT, bool HALF>
__global__ __launch_bounds__(256, WHAT == PAIR_ANY ? 3 : 2) void scan_pair(ScanPair p) {
  constexpr bool WAVE = WHAT == PAIR_WAVE, COL = IDXW || WHAT == PAIR_COLS;
  constexpr int BIG = IDXW ? RD_BIG_RB : RD_BIG_RB_W;
  static_assert(BIG * RD_THREADS <= CD_LDS_DOUBLES, "LDS of a row scan");
  __shared__ double lds[WAVE && RW_LDS_DOUBLES > CD_LDS_DOUBLES ? RW_LDS_DOUBLES : CD_LDS_DOUBLES];
  int v = blockIdx.x;
  const bool second = v >= p.j[0].nblk;
  if (second) v -= p.j[0].nblk;
  const SideJob& j = second ? p.j[1] : p.j[0];
  const int per_item = j.gx * j.gy;
  const int b = v / per_item, x = (v % per_item) % j.gx, y = (v % per_item) / j.gx;
  if constexpr (COL) {
    if (WHAT == PAIR_COLS || j.kind == SIDE_COL) {
      coldot_body<ColElem<DT, HALF>, IDXW, HALF ? 2 * CD_ROWS : CD_ROWS, CD_ASK>(j.s, Parts{}, j.gy, j.gx, x, y, b, lds);
      return;
    }
  }
  if constexpr (WHAT != PAIR_COLS) {
    if (j.kind == SIDE_ROW) rowdot_body<DT, IDXW, RD_SMALL_RB, RD_SMALL_U>(j.s, x, b, lds);
    else if (j.kind == SIDE_ROW_BIG) rowdot_body<DT, IDXW, BIG, RD_BIG_U>(j.s, x, b, lds);
    else if constexpr (WAVE) rowdot_wave_body<DT, IDXW>(j.s, x, b, lds);
  }
}

template <int DT, bool COL, bool ROW, bool COL_IDX, bool ROW_IDX, bool GATED>
__global__ __launch_bounds__(TS_THREADS) void tile_scan(TileScanArgs a) {
  extern __shared__ double ts_lds[];
  const int b = blockIdx.z;
  if (GATED && gated_off(a.gate, a.gate_stride, b, a.gate_value)) return;
  tile_scan_body<DT, COL, ROW, COL_IDX, ROW_IDX>(a, blockIdx.x, blockIdx.y, b, ts_lds);
}

// A wavefront per RW_RB rows where that alone fills the chip (two workgroups per compute unit) and the rows
// are short: 256 x 128 rows of 128 fp32 7.0 us against 21.0, 200 x 300 of 300 16 against 37, 16384 rows of
// 1024 bf16 9.0 against 14.9; equal from rows of 4096 on; with fewer rows the workgroup per row set keeps
// more loads in flight (4096 rows of 2048 fp32 7.7 against 12.1, 1024 of 1024 3.6 against 5.3).
bool rowdot_wavewise(const ScanArgs& a) {
  return a.Cc <= 2048 && (int64_t)((a.R + 4 * RW_RB - 1) / (4 * RW_RB)) * a.batch >= 512;
}

// workgroups of a column scan in vectors of 16 bytes
int64_t coldot_blocks(const ScanArgs& a) {
  const int seg = 64 * (a.dtype == GECC_BF16 ? 8 : 4);
  return (int64_t)((a.Cc + seg - 1) / seg) * ((a.R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS) * a.batch;
}

}  // namespace

size_t coldot_scratch_doubles(int R, int Cc, int batch) {
  const size_t nchunk = (R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
  return (size_t)batch * nchunk * 2 * (size_t)Cc;
}

hipError_t launch_rowdot(const ScanArgs& a0, const Stage2Job* carry, hipStream_t st) {
  ScanArgs a = a0;
  a.carry_blocks = 0;
  if (carry && carry->valid) {
    if (carry->batch != a.batch || carry->gate != a.gate || carry->gate_stride != a.gate_stride ||
        carry->gate_value != a.gate_value)
      return hipErrorInvalidValue;
    a.carry = *carry;
    a.carry_blocks = stage2_blocks(*carry);
  }
  const int extra = a.carry_blocks;
  const bool idx = a.w == nullptr;
  const bool small = (int64_t)((a.R + RD_BIG_RB - 1) / RD_BIG_RB) * a.batch < 1024;   // fewer than 4 workgroups per CU
  const bool gated = a.gate != nullptr;   // audits only, and audits use the index weights
  const bool wavewise = rowdot_wavewise(a);
#define GECC_LAUNCH_ROWDOT(DT, IDX, G)                                                               \
  do {                                                                                              \
    constexpr int BIG = IDX ? RD_BIG_RB : RD_BIG_RB_W;                                                \
    if (wavewise) hipLaunchKernelGGL((rowdot_wave_kernel<DT, IDX, G>),                                \
                                  dim3((a.R + 4 * RW_RB - 1) / (4 * RW_RB) + extra, a.batch),         \
                                  dim3(RD_THREADS), 0, st, a);                                        \
    else if (small) hipLaunchKernelGGL((rowdot_kernel<DT, IDX, RD_SMALL_RB, RD_SMALL_U, G>),               \
                                  dim3((a.R + RD_SMALL_RB - 1) / RD_SMALL_RB + extra, a.batch),       \
                                  dim3(RD_THREADS), 0, st, a);                                        \
    else       hipLaunchKernelGGL((rowdot_kernel<DT, IDX, BIG, RD_BIG_U, G>),                         \
                                  dim3((a.R + BIG - 1) / BIG + extra, a.batch),                       \
                                  dim3(RD_THREADS), 0, st, a);                                        \
  } while (0)
  if (gated && !idx) return hipErrorInvalidValue;
  if (a.dtype == GECC_BF16) {
    if (gated) GECC_LAUNCH_ROWDOT(GECC_BF16, true, true);
    else if (idx) GECC_LAUNCH_ROWDOT(GECC_BF16, true, false);
    else GECC_LAUNCH_ROWDOT(GECC_BF16, false, false);
  } else {
    if (gated) GECC_LAUNCH_ROWDOT(GECC_F32, true, true);
    else if (idx) GECC_LAUNCH_ROWDOT(GECC_F32, true, false);
    else GECC_LAUNCH_ROWDOT(GECC_F32, false, false);
  }
#undef GECC_LAUNCH_ROWDOT
  return hipGetLastError();
}

int coldot_done_words(const ScanArgs& a) {
  const int vec = a.dtype == GECC_BF16 ? 8 : 4;
  const int nchunk = (a.R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
  if (nchunk > SCAN_FUSE_MAX_CHUNKS) return 0;
  const int64_t words = (int64_t)((a.Cc + 64 * vec - 1) / (64 * vec)) * a.batch;
  return words <= SCAN_DONE_WORDS ? (int)words : 0;
}

hipError_t launch_coldot_stage1(const ScanArgs& a0, Stage2Job* pending, hipStream_t st) {
  ScanArgs a = a0;
  a.carry_blocks = 0;
  const int vec = a.dtype == GECC_BF16 ? 8 : 4;
  const int nchunk = (a.R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
  const bool idx = a.w == nullptr, gated = a.gate != nullptr;
  const bool half = !gated && !a.done && coldot_blocks(a) < CD_HALF_BELOW;
  const int seg = 64 * (half ? vec / 2 : vec);
  dim3 grid((a.Cc + seg - 1) / seg, nchunk, a.batch);
  if (gated && !idx) return hipErrorInvalidValue;
  if (a.done && coldot_done_words(a) == 0) return hipErrorInvalidValue;
  // (gated ones leave a chunk of any length to the counters or to the second stage)
  const bool one = nchunk == 1 && !gated && !a.done;
#define GECC_LAUNCH_COLDOT(DT)                                                                                           \
  do {                                                                                                                   \
    if (gated)           hipLaunchKernelGGL((coldot_stage1<DT, true, true, false, false>), grid, dim3(CD_THREADS), 0, st, a, nchunk);   \
    else if (half)       launch(std::integral_constant<int, DT>{}, std::true_type{});                                    \
    else                 launch(std::integral_constant<int, DT>{}, std::false_type{});                                   \
  } while (0)
  auto launch = [&](auto dt, auto h) {
    constexpr int DT = decltype(dt)::value;
    constexpr bool H = decltype(h)::value;
    if (idx && one)   hipLaunchKernelGGL((coldot_stage1<DT, true, false, true, H>), grid, dim3(CD_THREADS), 0, st, a, nchunk);
    else if (idx)     hipLaunchKernelGGL((coldot_stage1<DT, true, false, false, H>), grid, dim3(CD_THREADS), 0, st, a, nchunk);
    else if (one)     hipLaunchKernelGGL((coldot_stage1<DT, false, false, true, H>), grid, dim3(CD_THREADS), 0, st, a, nchunk);
    else              hipLaunchKernelGGL((coldot_stage1<DT, false, false, false, H>), grid, dim3(CD_THREADS), 0, st, a, nchunk);
  };
  if (a.dtype == GECC_BF16) GECC_LAUNCH_COLDOT(GECC_BF16); else GECC_LAUNCH_COLDOT(GECC_F32);
#undef GECC_LAUNCH_COLDOT
  *pending = Stage2Job{};
  if (!a.done && !one) {
    pending->valid = true;
    pending->scratch = a.scratch; pending->out = a.out; pending->out_stride = a.out_stride;
    pending->Cc = a.Cc; pending->nchunk = nchunk; pending->batch = a.batch;
    pending->gate = a.gate; pending->gate_stride = a.gate_stride; pending->gate_value = a.gate_value;
  }
  return hipGetLastError();
}

// ---- tile_scan ------------------------------------------------------------------------------
bool tile_scan_ok(const TileScanJob& t) {
  const int vec = t.dtype == GECC_BF16 ? 8 : 4;
  const size_t esz = t.dtype == GECC_BF16 ? 2 : 4;
  return reinterpret_cast<uintptr_t>(t.X) % 16 == 0 && t.ld % vec == 0 && (t.xs * esz) % 16 == 0 &&
         t.Cc % vec == 0 && t.Cc >= vec && t.R >= 1;
}

int tile_scan_segments(int Cc, int dtype) {
  const int seg = 64 * (dtype == GECC_BF16 ? 8 : 4);
  return (Cc + seg - 1) / seg;
}

size_t tile_scan_row_scratch_doubles(int R, int Cc, int dtype, int batch) {
  return (size_t)batch * (size_t)R * tile_scan_segments(Cc, dtype) * 2;
}

// rows per chunk: 128 (the chunk the column scratch is sized for) or, as long as two workgroups per
// compute unit remain, 256 or 512 (fewer column partial sums to write and read back; measured at
// 16384 x 4096: 30.3 us with 256-row chunks against 32.3 with 128)
static int tile_scan_chunk_rows(int R, int nseg, int batch) {
  int ch = SCAN_CHUNK_ROWS;
  while (ch < 512 && (int64_t)nseg * ((R + 2 * ch - 1) / (2 * ch)) * batch * 4 >= 2048) ch *= 2;
  return ch;
}

// kernel arguments of a tile scan; fuse_col / fuse_row: parts that finish by themselves (t.done set:
// the column part when a segment has few enough chunks for one workgroup to add up, the row part
// always -- as far as the counters reach).  done_words: counters used.
static bool make_tile_args(const TileScanJob& t, TileScanArgs& a, bool& fuse_col, bool& fuse_row, int& done_words) {
  if (!tile_scan_ok(t) || (!t.col_on && !t.row_on)) return false;
  a = TileScanArgs{};
  a.X = t.X; a.dtype = t.dtype; a.R = t.R; a.Cc = t.Cc; a.ld = t.ld; a.xs = t.xs; a.batch = t.batch;
  a.wr = t.wr; a.wr_stride = t.wr_stride; a.col_part = t.col_scratch;
  a.wc = t.wc; a.wc_stride = t.wc_stride; a.row_part = t.row_scratch;
  a.nseg = tile_scan_segments(t.Cc, t.dtype);
  a.stream = t.stream;
  // (larger chunks only save column partial sums: a row part alone takes the smallest, for the balance)
  a.chunk_rows = t.col_on ? tile_scan_chunk_rows(t.R, a.nseg, t.batch) : SCAN_CHUNK_ROWS;
  a.nchunk = (t.R + a.chunk_rows - 1) / a.chunk_rows;
  a.gate = t.gate; a.gate_stride = t.gate_stride; a.gate_value = t.gate_value;
  fuse_col = false; fuse_row = false;
  int64_t used = 0;
  if (t.done) {
    if (t.col_on && a.nchunk <= SCAN_FUSE_MAX_CHUNKS && (int64_t)t.batch * a.nseg <= SCAN_DONE_WORDS) {
      fuse_col = true; a.done_col = t.done; used = (int64_t)t.batch * a.nseg;
    }
    if (t.row_on && used + (int64_t)t.batch * a.nchunk <= SCAN_DONE_WORDS) {
      fuse_row = true; a.done_row = t.done + used; used += (int64_t)t.batch * a.nchunk;
    }
  }
  done_words = (int)used;
  a.col_out = t.col_out; a.col_out_stride = t.col_out_stride;
  a.row_out = t.row_out; a.row_out_stride = t.row_out_stride;
  return true;
}

hipError_t launch_tile_scan(const TileScanJob& t, Stage2Job* pending, hipStream_t st) {
  TileScanArgs a;
  bool fuse_col, fuse_row;
  int words;
  if (!make_tile_args(t, a, fuse_col, fuse_row, words)) return hipErrorInvalidValue;
  const dim3 grid(a.nseg, a.nchunk, a.batch), block(TS_THREADS);
  const size_t lds = TS_LDS_DOUBLES * sizeof(double);
  const bool gated = t.gate != nullptr;
  const bool cidx = t.wr == nullptr, ridx = t.wc == nullptr;
#define GECC_TS(DT, COL, ROW, CI, RI, G) \
  hipLaunchKernelGGL((tile_scan<DT, COL, ROW, CI, RI, G>), grid, block, lds, st, a)
#define GECC_TS_DT(DT)                                                                       \
  do {                                                                                       \
    if (t.col_on && t.row_on) {                                                              \
      if (gated) return hipErrorInvalidValue;                                                \
      if (cidx && !ridx) GECC_TS(DT, true, true, true, false, false);                        \
      else if (!cidx && ridx) GECC_TS(DT, true, true, false, true, false);                   \
      else return hipErrorInvalidValue;                                                      \
    } else if (t.col_on) {                                                                   \
      if (!cidx) return hipErrorInvalidValue;                                                \
      if (gated) GECC_TS(DT, true, false, true, true, true);                                 \
      else GECC_TS(DT, true, false, true, true, false);                                      \
    } else {                                                                                 \
      if (gated && !ridx) return hipErrorInvalidValue;                                       \
      if (gated) GECC_TS(DT, false, true, true, true, true);                                 \
      else if (ridx) GECC_TS(DT, false, true, true, true, false);                            \
      else GECC_TS(DT, false, true, true, false, false);                                     \
    }                                                                                        \
  } while (0)
  if (t.dtype == GECC_BF16) GECC_TS_DT(GECC_BF16); else GECC_TS_DT(GECC_F32);
#undef GECC_TS_DT
#undef GECC_TS
  *pending = Stage2Job{};
  pending->valid = (t.col_on && !fuse_col) || (t.row_on && !fuse_row);
  pending->batch = t.batch;
  pending->gate = t.gate; pending->gate_stride = t.gate_stride; pending->gate_value = t.gate_value;
  if (t.col_on && !fuse_col) {
    pending->scratch = t.col_scratch; pending->out = t.col_out; pending->out_stride = t.col_out_stride;
    pending->Cc = t.Cc; pending->nchunk = a.nchunk;
  }
  if (t.row_on && !fuse_row) {
    pending->row_scratch = t.row_scratch; pending->row_out = t.row_out; pending->row_out_stride = t.row_out_stride;
    pending->R = t.R; pending->nseg = a.nseg;
  }
  return hipGetLastError();
}

bool make_side_job(const ScanArgs& s, const Parts& w, bool rowdot, uint32_t* done, int words_left, SideJob& j, int& words) {
  j = SideJob{};
  j.s = s;
  j.w = w;
  j.s.carry_blocks = 0;
  words = 0;
  if (s.gate || !s.w) return false;
  if (rowdot) {
    // (no wavefront-per-rows scan of bf16 rows: its registers would halve the product's occupancy)
    const bool wavewise = s.dtype == GECC_F32 && rowdot_wavewise(s);
    const int rb = wavewise ? 4 * RW_RB : s.dtype == GECC_F32 ? side_rows<GECC_F32>() : side_rows<GECC_BF16>();
    j.kind = wavewise ? SIDE_ROW_WAVE : SIDE_ROW;
    j.gx = (s.R + rb - 1) / rb; j.gy = 1;
  } else {
    if (done) {
      words = coldot_done_words(s);
      if (words == 0 || words > words_left) return false;
    }
    const int vec = s.dtype == GECC_BF16 ? 8 : 4;
    j.kind = SIDE_COL;
    j.s.done = done;
    j.gx = (s.Cc + 64 * vec - 1) / (64 * vec);
    j.gy = (s.R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
  }
  const int64_t blocks = (int64_t)j.gx * j.gy * s.batch;
  if (blocks > (1 << 28)) return false;
  j.nblk = (int)blocks;
  return true;
}

namespace {
// the two scans as jobs of one grid; returns its workgroups
int64_t plan_pair(const ScanArgs* s, const bool* rowdot, ScanPair& p, Parts* left, bool& half) {
  int64_t grid = 0;
  const int64_t cols = (rowdot[0] ? 0 : coldot_blocks(s[0])) + (rowdot[1] ? 0 : coldot_blocks(s[1]));
  half = cols > 0 && cols < CD_PAIR_HALF_BELOW;
  for (int i = 0; i < 2; ++i) {
    SideJob& j = p.j[i];
    j.s = s[i];
    j.s.carry_blocks = 0;
    j.s.done = nullptr;
    left[i] = Parts{};
    if (rowdot[i]) {
      // (rows per workgroup as in launch_rowdot)
      const bool wavewise = rowdot_wavewise(s[i]), small = (int64_t)((s[i].R + RD_BIG_RB - 1) / RD_BIG_RB) * s[i].batch < 1024;
      const int rb = wavewise ? 4 * RW_RB : small ? RD_SMALL_RB : s[i].w ? RD_BIG_RB_W : RD_BIG_RB;
      j.kind = wavewise ? SIDE_ROW_WAVE : small ? SIDE_ROW : SIDE_ROW_BIG;
      j.gx = (s[i].R + rb - 1) / rb; j.gy = 1;
    } else {
      const int seg = 64 * (s[i].dtype == GECC_BF16 ? 8 : 4) / (half ? 2 : 1);
      j.kind = SIDE_COL;
      j.gx = (s[i].Cc + seg - 1) / seg;
      j.gy = (s[i].R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
      if (j.gy > 1) { left[i].chunks = s[i].scratch; left[i].nchunk = j.gy; }
    }
    const int64_t blocks = (int64_t)j.gx * j.gy * s[i].batch;
    grid += blocks;
    j.nblk = (int)blocks;
  }
  return grid;
}
}  // namespace

bool scan_pair_fits(const ScanArgs* s, const bool* rowdot) {
  ScanPair p{};
  Parts left[2];
  bool half;
  return plan_pair(s, rowdot, p, left, half) <= 0xffffff;          // (2^32 threads)
}

hipError_t launch_scan_pair(const ScanArgs* s, const bool* rowdot, Parts* left, hipStream_t st) {
  for (int i = 0; i < 2; ++i)
    if (s[i].gate || s[i].dtype != s[0].dtype || (s[i].w == nullptr) != (s[0].w == nullptr)) return hipErrorInvalidValue;
  ScanPair p{};
  bool half;
  const int64_t grid = plan_pair(s, rowdot, p, left, half);
  if (grid > 0xffffff) return hipErrorInvalidValue;
  const dim3 g((unsigned)grid), block(256);
  const bool idx = s[0].w == nullptr, wave = p.j[0].kind == SIDE_ROW_WAVE || p.j[1].kind == SIDE_ROW_WAVE;
  if (!idx && rowdot[0] != rowdot[1]) return hipErrorInvalidValue;
#define GECC_LAUNCH_PAIR(DT)                                                                            \
  do {                                                                                                  \
    if (idx && wave && half)     hipLaunchKernelGGL((scan_pair<DT, true, PAIR_WAVE, true>), g, block, 0, st, p);   \
    else if (idx && wave)        hipLaunchKernelGGL((scan_pair<DT, true, PAIR_WAVE, false>), g, block, 0, st, p);  \
    else if (idx && half)        hipLaunchKernelGGL((scan_pair<DT, true, PAIR_ANY, true>), g, block, 0, st, p);    \
    else if (idx)                hipLaunchKernelGGL((scan_pair<DT, true, PAIR_ANY, false>), g, block, 0, st, p);   \
    else if (wave)               hipLaunchKernelGGL((scan_pair<DT, false, PAIR_WAVE, false>), g, block, 0, st, p); \
    else if (!rowdot[0] && half) hipLaunchKernelGGL((scan_pair<DT, false, PAIR_COLS, true>), g, block, 0, st, p);  \
    else if (!rowdot[0])         hipLaunchKernelGGL((scan_pair<DT, false, PAIR_COLS, false>), g, block, 0, st, p); \
    else                         hipLaunchKernelGGL((scan_pair<DT, false, PAIR_ANY, false>), g, block, 0, st, p);  \
  } while (0)
  if (s[0].dtype == GECC_BF16) GECC_LAUNCH_PAIR(GECC_BF16); else GECC_LAUNCH_PAIR(GECC_F32);
#undef GECC_LAUNCH_PAIR
  return hipGetLastError();
}

// ---- the two audits as jobs of the decoder's launch -----------------------------------------------
constexpr int AUDIT_PAIR_MAX_BLOCKS = 5120;
// A column audit of fewer workgroups than compute units goes in vectors of 8 bytes, twice the workgroups.  The decoder's
// launch with an operand error, us, 16 -> 8 bytes:
//   bf16  1500 x 1000   21.8 -> 17.2      4 x 1024^2      21.5 -> 17.8      fp32  1024^2        16.6 -> 15.0
//         2048^2        22.0 -> 18.1      8 x 500 x 700   18.4 -> 19.0            3000 x 1000   19.2 -> 17.5
//         4096 x 2048   26.1 -> 22.5      16 x 256^2      the same
// From 256 on what the audit saves is lost where C alone is patched and the others only decide that: bf16 4096^2
// 31.5 -> 29.1 and 20.7 -> 22.6.
constexpr int CD_AUDIT_HALF_BELOW = 256;
// fills j from x; returns the counters it uses, or -1 when x cannot finish by itself
static int make_pair_job(const ScanPairItem& x, uint32_t* done, PairJob& j) {
  j = PairJob{};
  if (x.kind == 2) {
    TileScanJob t = x.t;
    if (t.col_on == t.row_on || !t.gate) return -1;                       // one part, gated
    if ((t.col_on && t.wr) || (t.row_on && t.wc)) return -1;              // index weights
    t.done = done;
    bool fc, fr;
    int words;
    if (!make_tile_args(t, j.t, fc, fr, words) || !(t.col_on ? fc : fr)) return -1;
    j.kind = t.col_on ? PJ_TILE_COL : PJ_TILE_ROW;
    j.gx = j.t.nseg; j.gy = j.t.nchunk;
    if ((int64_t)j.gx * j.gy * t.batch > (1 << 29)) return -1;
    j.nblk = j.gx * j.gy * t.batch;
    return words;
  }
  j.s = x.s;
  j.s.carry_blocks = 0;
  if (!j.s.gate || j.s.w) return -1;
  if (x.kind == 0) {
    // (rows per workgroup as in launch_rowdot; the sums of a row do not depend on it)
    const bool small = (int64_t)((j.s.R + RD_BIG_RB - 1) / RD_BIG_RB) * j.s.batch < 1024;
    const bool wavewise = rowdot_wavewise(j.s);
    const int rb = wavewise ? 4 * RW_RB : small ? RD_SMALL_RB : RD_BIG_RB;
    j.kind = wavewise ? PJ_ROW_WAVE : small ? PJ_ROW : PJ_ROW_BIG;
    j.gx = (j.s.R + rb - 1) / rb; j.gy = 1;
    if ((int64_t)j.gx * j.s.batch > (1 << 29)) return -1;
    j.nblk = j.gx * j.s.batch;
    return 0;
  }
  if (coldot_done_words(j.s) == 0) return -1;
  const bool half = coldot_blocks(j.s) < CD_AUDIT_HALF_BELOW;
  const int vec = (j.s.dtype == GECC_BF16 ? 8 : 4) / (half ? 2 : 1);
  j.kind = half ? PJ_COL_HALF : PJ_COL;
  j.s.done = done;
  j.gx = (j.s.Cc + 64 * vec - 1) / (64 * vec);
  j.gy = (j.s.R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
  if ((int64_t)j.gx * j.gy * j.s.batch > (1 << 29)) return -1;
  j.nblk = j.gx * j.gy * j.s.batch;
  return j.gx * j.s.batch;
}

static int pair_dtype(const ScanPairItem& x) { return x.kind == 2 ? x.t.dtype : x.s.dtype; }

bool make_audit_pair(const ScanPairItem& x0, const ScanPairItem& x1, uint32_t* done, PairArgs& p, int& words) {
  if (pair_dtype(x0) != pair_dtype(x1)) return false;
  const int w0 = make_pair_job(x0, done, p.j[0]);
  if (w0 < 0) return false;
  const int w1 = make_pair_job(x1, done + w0, p.j[1]);
  words = w0 + w1;
  // (a closed gate still costs the dispatch of every workgroup, about 2 us per thousand: a pair of very large
  // grids is no cheaper than launches of their own)
  return w1 >= 0 && words <= SCAN_DONE_WORDS && p.j[0].nblk + p.j[1].nblk <= AUDIT_PAIR_MAX_BLOCKS;
}

namespace {
__global__ void zero_words_kernel(uint32_t* w, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) w[i] = 0u;
}
}  // namespace
hipError_t launch_zero_words(uint32_t* words, int count, hipStream_t st) {
  hipLaunchKernelGGL(zero_words_kernel, dim3((count + 255) / 256), dim3(256), 0, st, words, count);
  return hipGetLastError();
}

int stage2_blocks(const Stage2Job& j) {
  return (j.Cc > 0 ? (2 * j.Cc + 63) / 64 : 0) + (j.R > 0 ? (j.R + 255) / 256 : 0);
}

hipError_t launch_stage2(const Stage2Job& j0, const Stage2Job& j1, hipStream_t st) {
  if (j1.valid && (j0.gate || j1.gate || j0.batch != j1.batch)) return hipErrorInvalidValue;
  const int own0 = stage2_blocks(j0);
  dim3 g2(own0 + (j1.valid ? stage2_blocks(j1) : 0), j0.batch);
  if (j1.valid) hipLaunchKernelGGL(coldot_stage2_pair, g2, dim3(256), 0, st, j0, j1, own0);
  else          hipLaunchKernelGGL(coldot_stage2, g2, dim3(256), 0, st, j0);
  return hipGetLastError();
}

}  // namespace gecc
