// vd_linear.hip -- the batch-invariant linear layer of libvdattn.so (gfx950).
//
// c[m][n] = bf16_RNE( sum_k a[m][k] * b[n][k] ): the matmul contract of the
// paper's Section 5.4 (Fig. 3): the output row of a token depends only on that
// token's input row and on the weights, however many rows the call holds and
// wherever the row sits among them.
//
// Canonical arithmetic (one chain per output element, fixed by K alone):
//   acc = +0 (fp32); for k0 = 0, 32, 64, ... < K (ascending):
//     acc = v_mfma_f32_16x16x32_bf16(a[m][k0 .. k0+31], b[n][k0 .. k0+31], acc)
//   c[m][n] = bf16 round-to-nearest-even of acc.
// The result of one MFMA output cell depends only on its own row of the A
// operand, its own column of the B operand and its accumulator cell (the
// property vd_cas.hpp relies on), so neither the tiling, nor the workgroup that
// computes a row, nor the other rows of the call reach its bits; only K (the
// chain length and order) does, and there is no split over K.
//
// Launch: one workgroup per output tile, of one of the tile shapes below, the
// shape chosen from M and N alone (run).  K advances in steps of BK values
// through an LDS ring of ST stages of A and B tiles filled by direct
// global-to-LDS copies, with one barrier per step; the 16-byte chunks of each
// LDS row are XOR-swizzled by the row so that the 16 rows one operand read
// touches fall in different banks.  Tiles are taken in groups of 4 row tiles
// sweeping the column tiles, and each XCD (workgroup id mod the die count, 8 on
// a whole MI355X) takes a contiguous range of that order, so the A and B
// panels of its workgroups are shared in its L2.
//
// What bounds it: with few rows (decode), the weights from HBM (50 MB at
// 4096 -> 6144: 7.9 us at the streaming rate) and, per workgroup, the chain of
// steps -- copies, barrier, operand reads, dependent matrix instructions -- so
// the small shapes take long steps (256 values) with up to 5 of them in
// flight; with thousands of rows, the matrix cores (1.17 PFLOP/s at 4096 rows).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/vdattn.h"
#include "vd_cas.hpp"
#include "vd_hw.hpp"

using namespace vd;

namespace {

constexpr int kKStep = 64;  // K is a multiple of this
constexpr int kGroupM = 4;  // row tiles per group of the tile order

// One tile shape: WM x WN wavefronts, each computing XB x YB MFMA blocks of
// 16 x 16; K advances BK per step through an LDS ring of ST stages; EU is the
// wavefronts per SIMD the registers are budgeted for.  LATE: half of a step's
// copies are issued after the first products instead of before them (a CU
// takes 64 bytes a cycle, and the whole burst holds up the wavefront).
template <int WM_, int WN_, int XB_, int YB_, int BK_, int ST_, int EU_, bool LATE_>
struct Tile {
  static constexpr int WM = WM_, WN = WN_, XB = XB_, YB = YB_, BK = BK_, ST = ST_, EU = EU_;
  static constexpr bool LATE = LATE_;
  static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
  static constexpr int BM = WM * 16 * XB;         // rows of a (tokens) per workgroup tile
  static constexpr int BN = WN * 16 * YB;         // rows of b (output features) per tile
  static constexpr int kRowBytes = BK * 2;        // one staged row
  static constexpr int kChunks = kRowBytes / 16;  // 16-byte chunks per staged row
  static constexpr int kRowsPerCopy = 1024 / kRowBytes;
  static constexpr int kTileA = BM * kRowBytes, kTileB = BN * kRowBytes;
  static constexpr int kStage = kTileA + kTileB;
  static constexpr int kLds = ST * kStage;
  static constexpr int kCopiesA = kTileA / 1024, kCopiesB = kTileB / 1024;
  static constexpr int kCopies = (kCopiesA + kCopiesB) / kWaves;  // per wavefront and stage
  static_assert(kChunks >= 8 && kRowsPerCopy >= 1, "staged rows of 128 to 1024 bytes");
  static_assert(kCopies * kWaves == kCopiesA + kCopiesB, "copy split");
  static_assert((ST - 2) * kCopies < 64, "copies in flight within the wait counter");
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
};

// Waits until at most `later` stages of N copies each are outstanding.
template <int N, int MAX>
__device__ __forceinline__ void wait_stages(int later) {
  if constexpr (MAX == 0) {
    wait_vmcnt<0>();
  } else {
    if (later >= MAX)
      wait_vmcnt<N * MAX>();
    else
      wait_stages<N, MAX - 1>(later);
  }
}

template <class T>
__global__ __launch_bounds__(T::kThreads) __attribute__((amdgpu_waves_per_eu(T::EU, T::EU))) void linear_kernel(
    const uint16_t* a, int64_t lda, const uint16_t* b, int64_t ldb, uint16_t* c, int64_t ldc,
    int64_t M, int N, int K, int tiles_m, int tiles_n, int xcd_shift) {
  constexpr int XB = T::XB, YB = T::YB, BK = T::BK, ST = T::ST, CH = T::kChunks;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  const int wave = uni(threadIdx.x >> 6);
  const int lane = __lane_id();
  // tile order: groups of kGroupM row tiles, each sweeping the column tiles
  // (row tile fastest); XCD x takes the x-th contiguous share of the order
  const int64_t total = (int64_t)tiles_m * tiles_n;
  const int xcds = 1 << xcd_shift;
  const int64_t per_xcd = (total + xcds - 1) >> xcd_shift;
  const int64_t jx = blockIdx.x >> xcd_shift;
  if (jx >= per_xcd) return;
  const int64_t i = (int64_t)(blockIdx.x & (xcds - 1)) * per_xcd + jx;
  if (i >= total) return;
  const int64_t group = i / ((int64_t)kGroupM * tiles_n);
  const int64_t first_m = group * kGroupM;
  const int size_m = (int)((tiles_m - first_m) < kGroupM ? (tiles_m - first_m) : kGroupM);
  const int in_group = (int)(i - group * (int64_t)kGroupM * tiles_n);
  const int64_t m0 = (first_m + in_group % size_m) * T::BM;
  const int n0 = (in_group / size_m) * T::BN;

  // Copies: a stage is kCopiesA copies of the A tile, then kCopiesB of the B
  // tile, 1 KB (kRowsPerCopy rows) each; a wavefront takes kCopies of them, of
  // each tile its even share where that divides.  Lane l of a copy carries
  // row l / CH of it and 16-byte slot l % CH, i.e. source chunk slot ^ (row &
  // 7), so that the 8 consecutive rows an operand read touches at one chunk
  // lie in 8 distinct 16-byte slots of a 128-byte bank window.  Rows past M
  // (or N) repeat the last row: in bounds, and never stored.
  auto copy_of = [&](int j) {
    constexpr bool even = T::kCopiesA % T::kWaves == 0 && T::kCopiesB % T::kWaves == 0;
    constexpr int ca = T::kCopiesA / T::kWaves, cb = T::kCopiesB / T::kWaves;
    if (!even) return wave * T::kCopies + j;
    return j < ca ? wave * ca + j : T::kCopiesA + wave * cb + j - ca;
  };
  const uint16_t* src[T::kCopies];
  int ck[T::kCopies];  // first k of the lane's chunk within the step
#pragma unroll
  for (int j = 0; j < T::kCopies; ++j) {
    const int q = copy_of(j);
    const bool is_a = q < T::kCopiesA;
    const int r = (is_a ? q : q - T::kCopiesA) * T::kRowsPerCopy + lane / CH;
    ck[j] = 8 * ((lane % CH) ^ (r & 7));
    if (is_a) {
      const int64_t ra = m0 + r < M ? m0 + r : M - 1;
      src[j] = a + ra * lda;
    } else {
      const int rb = n0 + r < N ? n0 + r : N - 1;
      src[j] = b + (int64_t)rb * ldb;
    }
    src[j] += ck[j];
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const int steps = (K + BK - 1) / BK;
  // copies first .. last - 1 of this wavefront's share of a step
  auto fetch = [&](int step, int first, int last) {
    const int k0 = step * BK;
    const uint32_t st = lds0 + (step % ST) * T::kStage;
    if (BK == kKStep || k0 + BK <= K) {
#pragma unroll
      for (int j = 0; j < T::kCopies; ++j)
        if (j >= first && j < last) lds_dma16(src[j] + k0, uni((int)(st + 1024 * copy_of(j))));
    } else {
      // the ragged last step: chunks past K repeat the row's last one (never used)
#pragma unroll
      for (int j = 0; j < T::kCopies; ++j)
        if (j >= first && j < last)
          lds_dma16(src[j] - ck[j] + min(k0 + ck[j], K - 8), uni((int)(st + 1024 * copy_of(j))));
    }
  };

  // this wavefront's part: rows wm .. wm + 16 XB - 1, columns wn .. wn + 16 YB - 1
  const int wm = 16 * XB * (wave / T::WN), wn = 16 * YB * (wave % T::WN);
  const int col = lane & 15, grp = lane >> 4;
  f32x4 acc[XB][YB];
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int y = 0; y < YB; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};

  // One barrier per step: after it, step t's copies are visible to every
  // wavefront and every wavefront is done with step t - 1, whose stage the
  // copies of step t + ST - 1 then refill while step t is computed.
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < steps) fetch(t, 0, T::kCopies);
  for (int t = 0; t < steps; ++t) {
    const int later = steps - 1 - t;
    wait_stages<T::kCopies, ST - 2>(later);  // this wavefront's copies of step t have landed
    lds_barrier();
    constexpr int early = T::LATE ? T::kCopies / 2 : T::kCopies;
    const bool more = t + ST - 1 < steps;
    if (more) fetch(t + ST - 1, 0, early);
    const char* TA = reinterpret_cast<const char*>(lds) + (t % ST) * T::kStage;
    const char* TB = TA + T::kTileA;
    auto chunk = [&](int kc) {
      // operand of lane (col, grp): row col of the block, k = 32 kc + 8 grp .. + 7
      // (wm, wn and 16 x are multiples of 16, so the swizzle key is col & 7)
      const int o = ((4 * kc + grp) ^ (col & 7)) << 4;
      u16x8 af[XB], bf[YB];
#pragma unroll
      for (int x = 0; x < XB; ++x)
        af[x] = *reinterpret_cast<const u16x8*>(TA + (wm + 16 * x + col) * T::kRowBytes + o);
#pragma unroll
      for (int y = 0; y < YB; ++y)
        bf[y] = *reinterpret_cast<const u16x8*>(TB + (wn + 16 * y + col) * T::kRowBytes + o);
#pragma unroll
      for (int x = 0; x < XB; ++x)
#pragma unroll
        for (int y = 0; y < YB; ++y) acc[x][y] = mfma(af[x], bf[y], acc[x][y]);
    };
    if (BK == kKStep || (t + 1) * BK <= K) {
#pragma unroll
      for (int kc = 0; kc < BK / 32; ++kc) {
        chunk(kc);
        if (T::LATE && kc == 0 && more) fetch(t + ST - 1, early, T::kCopies);
      }
    } else {
      // (the ragged last step: no copies are left)
      for (int kc = 0; kc < (K - t * BK) / 32; ++kc) chunk(kc);
    }
  }

  // accumulator cell i of block (x, y) in lane (col, grp): row 16 x + 4 grp + i, column 16 y + col
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = m0 + wm + 16 * x + 4 * grp + i;
      if (row >= M) continue;
#pragma unroll
      for (int y = 0; y < YB; ++y) {
        const int cn = n0 + wn + 16 * y + col;
        if (cn < N) c[row * ldc + cn] = bf16_rne(acc[x][y][i]);
      }
    }
}

struct Call {
  const uint16_t *a, *b;
  uint16_t* c;
  int64_t lda, ldb, ldc, M;
  int N, K;
  hipStream_t stream;
};

// Workgroups for the output tiles of bm x bn (M, N > 0), a multiple of the dies, or
// -1 when a grid cannot hold them: the runtime counts a launch's threads in 32
// bits, and a larger grid wraps.
int64_t grid_blocks(const Call& x, int bm, int bn, int threads, int xcds) {
  const int64_t tiles_m = (x.M - 1) / bm + 1, tiles_n = (x.N - 1) / bn + 1;
  if (tiles_m > UINT32_MAX / tiles_n) return -1;
  const int64_t blocks = (tiles_m * tiles_n + xcds - 1) / xcds * xcds;
  return blocks * threads <= UINT32_MAX ? blocks : -1;
}

template <class T>
int launch(const Call& x) {
  const int64_t tiles_m = (x.M - 1) / T::BM + 1, tiles_n = (x.N - 1) / T::BN + 1;
  const Geometry geo = device_geometry();
  const int64_t blocks = grid_blocks(x, T::BM, T::BN, T::kThreads, geo.xcds);
  if (blocks < 0) return VD_ERR_INVALID_ARG;
  static std::atomic<unsigned char> lds_set[kMaxDevices];
  if (set_lds_limit(reinterpret_cast<const void*>(&linear_kernel<T>), T::kLds, lds_set) != hipSuccess)
    return VD_ERR_LAUNCH;
  hipLaunchKernelGGL(linear_kernel<T>, dim3((unsigned)blocks), dim3(T::kThreads), T::kLds, x.stream,
                     x.a, x.lda, x.b, x.ldb, x.c, x.ldc, x.M, x.N, x.K, (int)tiles_m,
                     (int)tiles_n, geo.xcd_shift);
  return hipGetLastError() == hipSuccess ? VD_OK : VD_ERR_LAUNCH;
}

// The tile shapes, smallest first, each with the time of one round of its
// tiles (a tile per CU of 256 at K = 4096, in us, kernel launches back to
// back).  A call takes about ceil(tiles / CUs) rounds, so a shape that just
// fills the chip wins over a larger one that leaves CUs idle and over a
// smaller one that needs a second round or reads its operands more often.
// Measured at K = 4096 (us; the 256 x 192 shape, used for every call before,
// in brackets): 1 x 6144 12.0 [70.9], 32 x 6144 14.1 [71.7], 48 x 6144 16.0
// [72.4], 100 x 6144 20.0 [74.4], 200 x 6144 23.3 [81.1], 300 x 6144 29.7
// [75.6], 512 x 6144 38.0 [86.6], 1024 x 6144 52.0 [86.2], 4096 x 1024 40.4
// [81.0], 2048 x 6144 (a full round) [93.4], 4096 x 6144 [177.0; 128 x 192
// 203.8, 256 x 128 187.8, 256 x 256 182.5]; on another card the 16 x 64 shape, 16
// x 16000 20.4 [67.5] (its weights are 131 MB).  A round's time has a fixed part,
// so the ratios follow K: with the table's times, at K = 1024, 1 x 6144 4.4
// [18.7], 16 x 16000 5.1 [19.6], 48 x 6144 5.7 [20.7], 200 x 6144 8.3 [22.3], 512 x
// 6144 11.5 [23.1], 1024 x 6144 16.9 [25.2], 4096 x 1024 12.4 [23.8], 4096 x 6144
// 53.6 [53.7]; at K = 8192, 20.4 [130.8], 39.0 [132.8], 29.5 [133.0], 44.2
// [136.1], 62.8 [137.3], 96.2 [141.2], 71.3 [140.0], 324 [320].  Of 283 calls over
// 18 N x K (K 64 .. 14336, M 1 .. 8192) none is slower than with that one shape by
// more than 3%.  LATE, on one card without
// and with: 64 x 32 16.8 / 16.0, 64 x 128 30.2 / 29.7, 128 x 128 38.7 / 38.0, 128 x
// 192 58.4 / 52.0; 64 x 64 20.4 / 21.1, 64 x 96 23.2 / 23.9, 256 x 192 178.7 / 185.1.
// The same blocks as 32 x 32 x 16 steps are slower in every shape (256 x 192:
// 198).
#define VD_LINEAR_SHAPES(X)              \
  X(1, 2, 1, 1, 256, 6, 1, false, 12.0f) \
  X(2, 2, 1, 1, 256, 5, 1, false, 14.0f) \
  X(1, 4, 1, 1, 256, 3, 1, false, 15.2f) \
  X(4, 2, 1, 1, 256, 3, 1, true, 16.0f)  \
  X(2, 2, 2, 2, 64, 4, 2, false, 20.0f)  \
  X(2, 2, 2, 3, 64, 4, 2, false, 23.5f)  \
  X(2, 4, 2, 2, 64, 4, 2, true, 27.5f)   \
  X(4, 4, 2, 2, 64, 4, 4, true, 37.0f)   \
  X(4, 2, 2, 6, 64, 3, 2, true, 51.0f)   \
  X(4, 2, 4, 6, 64, 2, 2, false, 88.0f)

// The launch of the shape with the least rounds x time of a round, of those whose
// grid can be launched (a small tile's cannot for 2^29 rows).  The choice
// never reaches a value (the arithmetic above).
int run(const Call& x) {
  const Geometry geo = device_geometry();
  float best = 0.0f;
  int (*fn)(const Call&) = nullptr;
  auto consider = [&](int bm, int bn, int threads, float round_us, int (*f)(const Call&)) {
    if (grid_blocks(x, bm, bn, threads, geo.xcds) < 0) return;
    const int64_t tiles = ((x.M - 1) / bm + 1) * ((x.N - 1) / bn + 1);
    const float t = (float)((tiles + geo.cus - 1) / geo.cus) * round_us;
    if (!fn || t < best) {
      best = t;
      fn = f;
    }
  };
#define VD_LINEAR_CONSIDER(wm, wn, xb, yb, bk, st, eu, late, us) \
  consider(16 * wm * xb, 16 * wn * yb, 64 * wm * wn, us, &launch<Tile<wm, wn, xb, yb, bk, st, eu, late>>);
  VD_LINEAR_SHAPES(VD_LINEAR_CONSIDER)
#undef VD_LINEAR_CONSIDER
  return fn ? fn(x) : VD_ERR_INVALID_ARG;
}

}  // namespace

extern "C" int vd_linear(const void* a, int64_t lda, const void* b, int64_t ldb, void* c,
                         int64_t ldc, int64_t M, int32_t N, int32_t K, hipStream_t stream) {
  if (M < 0 || N < 0 || K < 0) return VD_ERR_INVALID_ARG;
  if (M == 0 || N == 0) return VD_OK;
  if (!c || ldc < N || (uintptr_t)c % 2 != 0) return VD_ERR_INVALID_ARG;
  if (K % kKStep != 0) return VD_ERR_UNSUPPORTED;
  // a and b are read only when K > 0 (K = 0: every output is the empty sum, +0)
  if (K > 0) {
    if (!a || !b) return VD_ERR_INVALID_ARG;
    if (lda < K || ldb < K || lda % 8 != 0 || ldb % 8 != 0) return VD_ERR_INVALID_ARG;
    if (((uintptr_t)a | (uintptr_t)b) % 16 != 0) return VD_ERR_INVALID_ARG;
  }
  const Call x{static_cast<const uint16_t*>(a), static_cast<const uint16_t*>(b),
               static_cast<uint16_t*>(c), lda, ldb, ldc, M, N, K, stream};
  return run(x);
}
