// HIP kernels for gfx950 (CDNA4, 64-wide wavefronts) and their launchers.
//
//   k_igemm*       implicit-GEMM convolution (3x3 / 1x1, stride 1 / 2, optional nearest-2x input,
//                  optional channel concatenation) and linear layers on MFMA, with fused epilogues
//   k_attn_mfma*   fused attention (online softmax, K and V^T tiles in LDS, MFMA for QK^T and PV)
//   k_attn_generic generic attention on fp32 MFMA, keys shared out over the wavefronts (fp32 mode, odd head sizes)
//   k_attn_frames_mfma / k_attn_frames  attention over the frame axis of a video model (one wavefront per
//                  position and head; MFMA without LDS for bf16, LDS-staged generic kernel otherwise)
//   k_gn_*         GroupNorm (+SiLU): one launch where a group fits a workgroup's registers, else partial sums, then statistics + apply
//   k_layernorm    several rows per wavefront
//   k_time_*, k_linear_rows  time embedding: in one launch for narrow models, else layer by layer
//   k_sampler      guidance combination + DDIM / Euler latent update
#include "ad_device.h"
#include "ad_kernels.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <numeric>
#include <type_traits>

namespace ad {

static thread_local Profiler* g_prof = nullptr;
void set_profiler(Profiler* p) { g_prof = p; }
ProfLaunch::ProfLaunch(const char* name, double flops, double bytes, hipStream_t s, int m, int n, int k) {
  if (!g_prof || !g_prof->on) return;
  hipEvent_t a = nullptr, b = nullptr;
  if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return;
  (void)hipEventRecord(a, s);
  g_prof->recs.push_back(ProfRec{name, flops, bytes, a, b, m, n, k});
  stop_ = b;
  s_ = s;
}
ProfLaunch::~ProfLaunch() {
  if (stop_) (void)hipEventRecord(stop_, s_);
}
void ProfLaunch::fetches(const void* ahead) {
  if (stop_) g_prof->recs.back().ahead = ahead;
}

// GN: how the wavefronts of a small-tile convolution hold the samples that they normalise, see gn_stats()
struct GnLayout {
  int log_vps;                                           // log2 of a wavefront's accesses to a pixel
  int vpp, per_access;                                   // accesses that a group has to a pixel, groups in an access: one of the two is 1
  int run;                                               // accesses of a lane that make up a wavefront of k_gn_group
  int pixels, slots;                                     // pixels that begin in lane 0, accesses of a lane to them at the most (0: no layout)
  int bits;                                              // of a sample's pixels in an access
  int chained;                                           // threads of k_gn_group have several accesses
};

// =================================================================================================
// Implicit GEMM:  out[m][n] = sum_k A[m][k] * W[n][k],  m = (batch, oy, ox), k = (tap, channel).
// Block tile BM x BN, 4 wavefronts in a 2 x 2 grid, each computing (BM/2) x (BN/2) with 32x32 MFMA
// tiles.  One k-tile is 128 bytes of K per row (64 bf16 / 32 fp32), staged through LDS with a
// 16-byte row pad; the next k-tile is fetched into registers while the current one is multiplied.
// =================================================================================================
struct IgemmParams {
  const void* src0; const void* src1;
  int c0, c1, ctot;
  int hs, ws, up, hin, win;
  int hout, wout, hw_out, stride, ksize, pad;
  int M, N, Kp, tiles_n, ktiles;
  unsigned w_row, xw_row, w_kt;       // weights: bytes between the rows of a block of 32 (of w, of xw) and between k-tiles, see weight_at()
  const void* w; const float* bias; const float* rowvec; const void* residual;
  void* out; int out_mode; int ld_t; int rowvec_ld;
  unsigned bytes0, bytes1, bytes_w;   // sizes of the two sources and of the packed weights
  int kt_per_split;                   // k-tiles handled by one workgroup along grid.y (split-K), else ktiles
  float* partial;                     // split-K: fp32 partial sums [splits][M][N]; nullptr otherwise
  void* out2; void* out3;             // OUT_QKV
  FastDiv div_hw, div_w;              // by hw_out and by wout (row index -> sample, output row, output column)
  int tiles_m;                        // row tiles
  int k_prof;                         // K the profiler counts (the real one where the operand is zero-padded), else Kp
  int vec16;                          // row-major outputs and the residual can be accessed 16 bytes at a time
  int turn16;                         // OUT_QKV: so can the rows of the transposed third
  int band;                           // workgroup order: row tiles per band, see tile_of(); 0 = all of them
  FastDiv div_tiles, div_band, div_rows, div_last;      // by tiles, tiles of a band, row tiles of a band and of the last band
  const void* x0; const void* x1; const void* xw;       // XTRA (k_igemm_p3): sources and weights of the 1x1 convolution behind the taps
  int xc0, xc1, kt_main;                                // its channels; k-tiles of the taps
  unsigned xbytes0, xbytes1, xbytes_w;
  const float* ln_gain; const float* ln_offset; float ln_eps;      // LN, GN (k_igemm_small): of the channels
  int gn_groups; GnLayout gn; double gn_inv_n;            // GN: groups (0: none)
  const void* ahead; unsigned ahead_bytes, ahead_span;             // k_igemm_p3: weights of a later launch (0 bytes: none), and a wavefront's share of them
};

// Byte offset of a row of a packed operand within a k-tile (k-tile kt is kt * p.w_kt further).  Two layouts: rows of k_bytes one after the other
// (ad_pack_conv_weight), or blocks of 32 rows with the 128 bytes of a k-tile of the rows side by side, k-tile after k-tile (pack_blocks(), what a
// loaded model holds).  The workgroups of a launch walk K side by side, so at any time they ask for one k-tile of all rows: in rows these are pieces of
// 128 bytes at a pitch of k_bytes, which for K = 1280, 2560, 5120 fall on half, a quarter, an eighth of the channels of an L2 and of memory; in blocks
// they are runs of 4 KiB.  Weights from memory, us (rows -> blocks): 2048x1280x5120 46.8 -> 43.2, 2048x1280x1280 15.3 -> 14.3, 8192x640x2560 35.4 -> 33.3,
// 1152x1280x5120 33.0 -> 30.7, 720x640x2560 13.2 -> 12.3, 3x3 4608x640x11520 82.5 -> 78.5; K = 320 and 640, whose pitch falls on all channels, level.
// Blocks of all rows (one run per k-tile): as fast for long K, 2-4 % slower for K = 320 and 640.
__device__ __forceinline__ unsigned weight_at(int row, unsigned k_bytes, unsigned row_bytes) {
  return (unsigned)(row >> 5) * (32u * k_bytes) + (unsigned)(row & 31) * row_bytes;
}

// Which (row tile, column tile, split) a workgroup computes.  Workgroups go to the 8 XCDs round-robin in
// launch order (x fastest, then y); xcd_remap turns that into 8 contiguous runs of a virtual index.  The virtual index
// is laid out [split][band of row tiles][column tile][row tile of the band]: an XCD's run is a block of row and column
// tiles, and what its L2 takes in per k-tile is the rows of that block plus its columns.  Bands of one row tile: a slice
// of the activations and every weight; one band: a slice of the weights and every activation; between them (see
// best_band()) the blocks are about square.
struct TileId { int m_tile, n_tile, split; };
__device__ __forceinline__ TileId tile_of(const IgemmParams& p) {
  const int tiles = p.tiles_m * p.tiles_n;
  const int lid = blockIdx.y * gridDim.x + blockIdx.x;
  const int vid = xcd_remap(lid, gridDim.x * gridDim.y);
  const int split = (int)fast_div((unsigned)vid, p.div_tiles), t = vid - split * tiles;
  const int b = (int)fast_div((unsigned)t, p.div_band), r = t - b * p.band * p.tiles_n;
  const int rows = min(p.band, p.tiles_m - b * p.band);
  const int n_tile = (int)(rows == p.band ? fast_div((unsigned)r, p.div_rows) : fast_div((unsigned)r, p.div_last));
  return TileId{b * p.band + r - n_tile * rows, n_tile, split};
}
static void set_tiles(IgemmParams& p, int bm, int bn) {
  p.tiles_m = (p.M + bm - 1) / bm;
  p.tiles_n = (p.N + bn - 1) / bn;
  if (p.band < 1 || p.band > p.tiles_m) p.band = p.tiles_m;
  p.div_tiles = make_fastdiv((unsigned)(p.tiles_m * p.tiles_n));
  p.div_band = make_fastdiv((unsigned)(p.band * p.tiles_n));
  p.div_rows = make_fastdiv((unsigned)p.band);
  p.div_last = make_fastdiv((unsigned)(p.tiles_m % p.band ? p.tiles_m % p.band : p.band));
}

constexpr size_t kLdsLimit = 160 * 1024;
constexpr int kPitch = kRowBytes + 16;   // LDS row pitch in bytes

template <typename T> struct Mma;
template <> struct Mma<bf16> {
  static __device__ __forceinline__ void run(const bf16x8& a, const bf16x8& b, f32x16& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mma<float> {
  // a 16-byte fragment holds 4 consecutive k per half-wave; MFMA j pairs element j of both halves
  static __device__ __forceinline__ void run(const f32x4& a, const f32x4& b, f32x16& c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], c, 0, 0, 0);
  }
};

// MODE: epilogue selected at compile time (the OUT_* value, or OUT_PARTIAL for split-K partial sums)
constexpr int OUT_PARTIAL = 5;
// How a wavefront's WTM x WTN tile leaves in rows: slabs of 128 bytes of a row (the last one may be 64), 16 bytes a lane.
template <typename T, int WTM, int WTN>
struct RowSlabs {
  static constexpr int VN = Vec<T>::N, FULL = 8 * VN, COUNT = (WTN + FULL - 1) / FULL;
  static constexpr int width(int s) { return WTN - s * FULL < FULL ? WTN - s * FULL : FULL; }
  static constexpr int rows(int s) { return 64 * VN / width(s); }              // rows of one access of the wavefront
  static constexpr int accesses(int s) { return WTM / rows(s); }
  static constexpr int MAX = WTM / 8;
  static constexpr int VGPRS = COUNT * MAX * 4;                                // the whole tile, 16 bytes a lane and access
};
// Residual rows of slab s in the layout they are added in (p.vec16; rows and columns beyond the output repeat its last ones).
template <typename T, int WTM, int WTN>
__device__ __forceinline__ void load_residual(const IgemmParams& p, int s, int row0, int col0, int lane,
                                              typename Vec<T>::type (&dst)[RowSlabs<T, WTM, WTN>::MAX]) {
  typedef RowSlabs<T, WTM, WTN> RS;
  const int lpr = RS::width(s) / RS::VN;
  const int col = min(col0 + s * RS::FULL + (lane % lpr) * RS::VN, p.N - RS::VN);
#pragma unroll
  for (int it = 0; it < RS::accesses(s); ++it) {
    const int row = min(row0 + it * RS::rows(s) + lane / lpr, p.M - 1);
    dst[it] = *(const typename Vec<T>::type*)((const T*)p.residual + (size_t)row * p.N + col);
  }
}
// Bytes of LDS a wavefront stages its output in: CR rows of the tile (or all rows of 32 columns, for transposed outputs).
// The pitch puts the rows that the two halves of a wavefront write together 32 banks apart.
constexpr int stage_pitch(int columns) { return columns * 4 + 32; }
template <typename T, int WTM, int WTN>
constexpr int stage_bytes(int cr) {
  const int rows = cr * stage_pitch(RowSlabs<T, WTM, WTN>::width(0)), cols = 32 * (WTM * (int)sizeof(T) + 16);
  return rows > cols ? rows : cols;
}
// Orders a wavefront's LDS writes before the reads of other lanes that follow (the LDS unit serves a wavefront in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Epilogue shared by the GEMM kernels.  A lane holds column l32 of each 32x32 tile; accumulator register r is row
// 8*(r/4) + 4*half + r%4 of the tile.  Row-major outputs go through LDS, CR rows of a slab at a time in fp32 (so the result is
// rounded once), and leave as whole 128-byte lines, 16 bytes a lane.  What limits it is latency: the residual, the bias and the
// time projection are requested before the first store of the wavefront (loads and stores retire in order, a load behind a store
// waits for it), the residual of small tiles even before the k-loop (res, PRE).  `stage`: the wavefront's private LDS area of
// stage_bytes(CR), swap: WTM x 32 floats that the wavefronts of the same rows share (GEGLU, odd TN); the caller has synchronised the
// workgroup after its last read of the k-loop tiles.
// Measured (bf16, bias and residual, us; 64-byte pieces of lines and the residual read between the stores -> this): 65536x320x320
// 62 -> 41, 16384x640x640 37 -> 27, 18432x320x320 16.4 -> 14.1, 2048x1280x1280 18.0 -> 16.5, 3x3 18432x320x2880 45.3 -> 41.2.
template <typename T, int WTM, int WTN, int TM, int TN, int MODE, int CR, bool PRE>
__device__ __forceinline__ void igemm_epilogue(const IgemmParams& p, f32x16 (&acc)[TM][TN], int m0, int n0, int wave_m,
                                               int wave_n, int l32, int half, char* stage, int split,
                                               typename Vec<T>::type (&res)[RowSlabs<T, WTM, WTN>::COUNT][RowSlabs<T, WTM, WTN>::MAX],
                                               float* swap = nullptr) {
  typedef typename Vec4<T>::type V4;
  typedef typename Vec<T>::type V;
  typedef RowSlabs<T, WTM, WTN> RS;
  constexpr int VN = RS::VN;
  const int row_base = m0 + wave_m * WTM + 4 * half;
  const int row0 = m0 + wave_m * WTM, col0 = n0 + wave_n * WTN;      // first row and column of this wavefront
  const int col_base = col0 + l32;
  const int lane = l32 + 32 * half;
  // VN columns of one row, staged in fp32
  auto staged = [&](int row, int pitch, int col, float (&v)[VN]) {
    const float* src = (const float*)(stage + row * pitch) + col;
#pragma unroll
    for (int e = 0; e < VN; e += 4) {
      const f32x4 x = *(const f32x4*)(src + e);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[e + k] = x[k];
    }
  };
  // VN columns to dst, `left` of them inside the output
  auto store = [&](T* dst, const float (&v)[VN], int ncols, int left) {
    if (p.vec16) {
      V o;
#pragma unroll
      for (int e = 0; e < VN; ++e) o[e] = from_f<T>(v[e]);
      *(V*)dst = o;
    } else if ((ncols & 3) == 0) {
#pragma unroll
      for (int e = 0; e < VN; e += 4)
        if (e < left) *(V4*)(dst + e) = V4{from_f<T>(v[e]), from_f<T>(v[e + 1]), from_f<T>(v[e + 2]), from_f<T>(v[e + 3])};
    } else {
#pragma unroll
      for (int e = 0; e < VN; ++e)
        if (e < left) dst[e] = from_f<T>(v[e]);
    }
  };
  if constexpr (MODE == OUT_PARTIAL) {
    float* dst = p.partial + (size_t)split * p.M * p.N;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = col_base + j * 32;
      if (col >= p.N) continue;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row_base + i * 32 + 8 * (r >> 2) + (r & 3);
          if (row < p.M) dst[(size_t)row * p.N + col] = acc[i][j][r];
        }
    }
  } else if constexpr (MODE == OUT_GEGLU) {
    // packed columns: 32 value, 32 gate; N is a multiple of 64.  With an odd number of 32-column tiles per wavefront (two wavefronts
    // along N) the last value tile of the first one belongs to the first gate tile of the second, which gets it through LDS.
    constexpr int PITCH = stage_pitch(32), LPR = 32 / VN, ROWS = 64 / LPR;
    constexpr bool ODD = TN % 2 != 0;
    const int half_n = p.N >> 1;
    float bias[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bias[j] = p.bias ? p.bias[min(col_base + j * 32, p.N - 1)] : 0.f;
    auto emit = [&](int tile, auto val, auto gate) {           // tile: first packed column of the pair; val / gate: (i, r) -> value
      const int oc = (tile >> 1) + (lane % LPR) * VN;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int c = 0; c < 32 / CR; ++c) {
          wave_lds_fence();
#pragma unroll
          for (int q = 0; q < CR / 2; ++q) {
            const int r = c * (CR / 2) + q;
            *(float*)(stage + (4 * half + 8 * (q >> 2) + (q & 3)) * PITCH + l32 * 4) = val(i, r) * gelu_f(gate(i, r));
          }
          wave_lds_fence();
#pragma unroll
          for (int it = 0; it < CR / ROWS; ++it) {
            const int rl = it * ROWS + lane / LPR, row = row0 + i * 32 + c * CR + rl;
            float v[VN];
            staged(rl, PITCH, (lane % LPR) * VN, v);
            if (row < p.M && oc < half_n) store((T*)p.out + (size_t)row * half_n + oc, v, half_n, half_n - oc);
          }
        }
    };
    auto pair = [&](auto jc) {
      constexpr int J = decltype(jc)::value;
      emit(col0 + J * 32, [&](int i, int r) { return acc[i][J][r] + bias[J]; }, [&](int i, int r) { return acc[i][J + 1][r] + bias[J + 1]; });
    };
    if constexpr (!ODD) {
      pair(std::integral_constant<int, 0>{});
      static_assert(TN <= 2, "further pairs");
    } else {
      static_assert(TN == 5, "two whole pairs and a shared one");
      if (wave_n == 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) swap[(i * 16 + r) * 64 + lane] = acc[i][4][r] + bias[4];
      }
      __syncthreads();
      if (wave_n == 0) {
        pair(std::integral_constant<int, 0>{});
        pair(std::integral_constant<int, 2>{});
      } else {
        emit(col0 - 32, [&](int i, int r) { return swap[(i * 16 + r) * 64 + lane]; }, [&](int i, int r) { return acc[i][0][r] + bias[0]; });
        pair(std::integral_constant<int, 1>{});
        pair(std::integral_constant<int, 3>{});
      }
    }
  } else {
    auto sample_of = [&](int row) { return (int)fast_div((unsigned)row, p.div_hw); };
    constexpr bool VECTOR = MODE != OUT_QKV;                 // a per-sample vector may be added
    const int c3 = MODE == OUT_QKV ? p.N / 3 : p.N;          // columns of one destination
    // first column that leaves transposed (a 32-column tile never straddles two thirds: c3 is a multiple of 32)
    const int turned = (MODE == OUT_TRANSPOSED || MODE == OUT_TRANSPOSED_F32) ? 0 : (MODE == OUT_QKV && p.ld_t > 0) ? 2 * c3 : p.N;
    // what is added to a column: the bias, and the per-sample vector where the wavefront's rows belong to one sample
    const int b0 = sample_of(min(row0, p.M - 1));
    const bool mixed = VECTOR && p.rowvec && sample_of(min(row0 + WTM, p.M) - 1) != b0;
    float add[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = min(col_base + j * 32, p.N - 1);
      add[j] = p.bias ? p.bias[col] : 0.f;
      if (VECTOR && p.rowvec && !mixed) add[j] += p.rowvec[(size_t)b0 * p.rowvec_ld + col];
    }
    if (VECTOR && mixed) {                                   // rows of two samples: the vector goes into the accumulators
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = min(col_base + j * 32, p.N - 1);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = min(row_base + i * 32 + 8 * (r >> 2) + (r & 3), p.M - 1);
            acc[i][j][r] += add[j] + p.rowvec[(size_t)sample_of(row) * p.rowvec_ld + col];
          }
        add[j] = 0.f;
      }
    }
    // accumulator register r of tile (i, j), with everything added that belongs to its column
    auto value = [&](int i, int j, int r) { return acc[i][j][r] + add[j]; };
    const bool with_res = MODE == OUT_ROWMAJOR && p.residual != nullptr;
    if (MODE == OUT_ROWMAJOR && !PRE && with_res && p.vec16) load_residual<T, WTM, WTN>(p, 0, row0, col0, lane, res[0]);
    if constexpr (MODE == OUT_ROWMAJOR || MODE == OUT_QKV) {
      // distances of the other destinations (a lane's columns decide which one it writes)
      const ptrdiff_t to_k = MODE == OUT_QKV ? (const T*)p.out2 - (const T*)p.out : 0, to_v = MODE == OUT_QKV ? (const T*)p.out3 - (const T*)p.out : 0;
#pragma unroll
      for (int s = 0; s < RS::COUNT; ++s) {
        if (!PRE && s + 1 < RS::COUNT && with_res && p.vec16) load_residual<T, WTM, WTN>(p, s + 1, row0, col0, lane, res[s + 1]);
        const int width = RS::width(s), pitch = stage_pitch(width), lpr = width / VN, rows = RS::rows(s);
        const int first = col0 + s * RS::FULL;
        if (first >= turned) continue;
        const int cl = (lane % lpr) * VN, col = first + cl;
        const int which = MODE == OUT_QKV ? (col >= c3) + (col >= 2 * c3) : 0;
        T* const dst = (T*)p.out + (which == 0 ? 0 : which == 1 ? to_k : to_v) + (col - which * c3);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int c = 0; c < 32 / CR; ++c) {
            wave_lds_fence();
#pragma unroll
            for (int jj = 0; jj < width / 32; ++jj)
#pragma unroll
              for (int q = 0; q < CR / 2; ++q)
                *(float*)(stage + (4 * half + 8 * (q >> 2) + (q & 3)) * pitch + (jj * 32 + l32) * 4) =
                    value(i, s * (RS::FULL / 32) + jj, c * (CR / 2) + q);
            wave_lds_fence();
#pragma unroll
            for (int it = 0; it < CR / rows; ++it) {
              const int rl = it * rows + lane / lpr, row = row0 + i * 32 + c * CR + rl;
              float v[VN];
              staged(rl, pitch, cl, v);
              if (row >= p.M || col >= turned) continue;
              if (with_res) {
                if (p.vec16) {
#pragma unroll
                  for (int e = 0; e < VN; ++e) v[e] += to_f(res[s][(i * 32 + c * CR) / rows + it][e]);
                } else {
#pragma unroll
                  for (int e = 0; e < VN; ++e)
                    if (col + e < p.N) v[e] += to_f(((const T*)p.residual)[(size_t)row * p.N + col + e]);
                }
              }
              store(dst + (size_t)row * c3, v, c3, c3 - (col - which * c3));
            }
          }
      }
    }
    if constexpr (MODE != OUT_ROWMAJOR) {
      const int ncols = c3, third = MODE == OUT_QKV ? 2 * c3 : 0;
      void* dstp = MODE == OUT_QKV ? p.out3 : p.out;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int tile = col0 + j * 32, col = tile + l32, cc = col - third;
        if (tile < turned || tile >= p.N) continue;
        if (MODE == OUT_QKV && p.turn16) {
          // through LDS: the rows of a column leave 16 bytes a lane (eight rows never straddle two samples)
          constexpr int PITCH = WTM * (int)sizeof(T) + 16, LPC = WTM / VN, COLS = 64 / LPC;
          wave_lds_fence();
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              *(V4*)(stage + l32 * PITCH + (i * 32 + 8 * g + 4 * half) * (int)sizeof(T)) =
                  V4{from_f<T>(value(i, j, 4 * g)), from_f<T>(value(i, j, 4 * g + 1)), from_f<T>(value(i, j, 4 * g + 2)), from_f<T>(value(i, j, 4 * g + 3))};
          wave_lds_fence();
          const int row = row0 + (lane % LPC) * VN, b = sample_of(min(row, p.M - 1));
#pragma unroll
          for (int it = 0; it < 32 / COLS; ++it) {
            const int cl = it * COLS + lane / LPC;
            const V v = *(const V*)(stage + cl * PITCH + (lane % LPC) * 16);
            if (row < p.M && tile + cl < p.N) *(V*)((T*)dstp + ((size_t)b * ncols + (tile + cl - third)) * p.ld_t + (row - b * p.hw_out)) = v;
          }
          continue;
        }
        if (col >= p.N) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int row = row_base + i * 32 + 8 * g;                // 4 consecutive rows: registers 4g .. 4g+3
            if (row >= p.M) continue;
            const int b = sample_of(row);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = value(i, j, 4 * g + e);
            const size_t o = ((size_t)b * ncols + cc) * p.ld_t + (row - b * p.hw_out);
            if ((p.hw_out & 3) == 0 && (p.ld_t & 3) == 0 && row + 3 < p.M) {
              if constexpr (MODE == OUT_TRANSPOSED_F32) *(f32x4*)((float*)dstp + o) = f32x4{v[0], v[1], v[2], v[3]};
              else *(V4*)((T*)dstp + o) = V4{from_f<T>(v[0]), from_f<T>(v[1]), from_f<T>(v[2]), from_f<T>(v[3])};
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (row + e >= p.M) break;
                const int be = sample_of(row + e);
                const size_t oe = ((size_t)be * ncols + cc) * p.ld_t + (row + e - be * p.hw_out);
                if constexpr (MODE == OUT_TRANSPOSED_F32) ((float*)dstp)[oe] = v[e];
                else ((T*)dstp)[oe] = from_f<T>(v[e]);
              }
            }
          }
      }
    }
  }
}

template <typename T, int BM, int BN, int WGM, int WGN, int NSET, int MODE>
__global__ __launch_bounds__(256) void k_igemm(IgemmParams p) {
  typedef typename Vec<T>::type V;
  constexpr int BK = kRowBytes / (int)sizeof(T);
  constexpr int ES = (int)sizeof(T);
  constexpr int WTM = BM / WGM, WTN = BN / WGN;  // wavefront tile
  constexpr int TM = WTM / 32, TN = WTN / 32;    // 32x32 MFMA tiles per wavefront
  constexpr int AV = BM / 32, BV = BN / 32;      // 16-byte vectors per thread per k-tile
  constexpr int STAGE = (BM + BN) * kPitch;
  extern __shared__ __attribute__((aligned(16))) char lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int wave_m = wave / WGN, wave_n = wave % WGN;
  const TileId tid3 = tile_of(p);
  const int m0 = tid3.m_tile * BM, n0 = tid3.n_tile * BN;

  const __amdgpu_buffer_rsrc_t rs0 = make_rsrc(p.src0, p.bytes0);
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(p.src1, p.bytes1);
  const __amdgpu_buffer_rsrc_t rsw = make_rsrc(p.w, p.bytes_w);

  // per-thread rows of the A tile: row = tid/8 + 32 i, 16-byte column = tid%8
  const int vcol = tid & 7, vrow = tid >> 3;
  int a_iy0[AV], a_ix0[AV], a_b[AV];
#pragma unroll
  for (int i = 0; i < AV; ++i) {
    const int m = m0 + vrow + 32 * i;
    if (m < p.M) {
      const int b = (int)fast_div((unsigned)m, p.div_hw), r = m - b * p.hw_out;
      const int oy = (int)fast_div((unsigned)r, p.div_w), ox = r - oy * p.wout;
      a_b[i] = b * p.hs; a_iy0[i] = oy * p.stride - p.pad; a_ix0[i] = ox * p.stride - p.pad;
    } else {
      a_b[i] = -1; a_iy0[i] = 0; a_ix0[i] = 0;
    }
  }
  unsigned b_off[BV];
#pragma unroll
  for (int i = 0; i < BV; ++i) b_off[i] = weight_at(n0 + vrow + 32 * i, (unsigned)p.Kp * ES, p.w_row) + vcol * 16;

  // byte offsets of this thread's A vectors for the tap being fetched (kOob = reads zeros)
  unsigned a_off0[AV], a_off1[AV];
  auto set_tap = [&](int tap) {
    const int u = tap / p.ksize, v = tap - u * p.ksize;
#pragma unroll
    for (int i = 0; i < AV; ++i) {
      const int iy = a_iy0[i] + u, ix = a_ix0[i] + v;
      const bool ok = a_b[i] >= 0 && iy >= 0 && iy < p.hin && ix >= 0 && ix < p.win;
      const unsigned pix = (unsigned)((a_b[i] + (iy >> p.up)) * p.ws + (ix >> p.up));
      a_off0[i] = ok ? (pix * (unsigned)p.c0 + vcol * (16 / ES)) * ES : kOob;
      a_off1[i] = ok ? (pix * (unsigned)p.c1 + vcol * (16 / ES)) * ES : kOob;
    }
  };

  // NSET register sets hold the k-tiles in flight: a tile is requested NSET iterations before it is
  // multiplied, which is what hides the latency of the memory system at the low occupancy these
  // problem sizes allow.
  V areg[NSET][AV], breg[NSET][BV];
  // this workgroup's range of k-tiles (all of them unless the launch splits K along grid.y)
  const int kt_begin = tid3.split * p.kt_per_split;
  const int nkt = min(p.ktiles - kt_begin, p.kt_per_split);
  const int f_k0 = kt_begin * BK;        // position of the next k-tile to fetch
  int f_tap = f_k0 / p.ctot, f_cc = f_k0 - f_tap * p.ctot;
  unsigned f_w = kt_begin * p.w_kt;      // and of its weights
  set_tap(f_tap);
  auto fetch = [&](V (&ar)[AV], V (&br)[BV]) {
    if (f_cc < p.c0) {
#pragma unroll
      for (int i = 0; i < AV; ++i) ar[i] = buffer_load16<V>(rs0, a_off0[i], (unsigned)(f_cc * ES));
    } else {
#pragma unroll
      for (int i = 0; i < AV; ++i) ar[i] = buffer_load16<V>(rs1, a_off1[i], (unsigned)((f_cc - p.c0) * ES));
    }
#pragma unroll
    for (int i = 0; i < BV; ++i) br[i] = buffer_load16<V>(rsw, b_off[i], f_w);
    f_w += p.w_kt;
    f_cc += BK;
    if (f_cc >= p.ctot) {
      f_cc = 0;
      ++f_tap;
      if (f_tap < p.ksize * p.ksize) set_tap(f_tap);
    }
  };
  auto stash = [&](int stage, const V (&ar)[AV], const V (&br)[BV]) {
    char* As = lds + stage * STAGE;
    char* Bs = As + BM * kPitch;
#pragma unroll
    for (int i = 0; i < AV; ++i) *(V*)(As + (vrow + 32 * i) * kPitch + vcol * 16) = ar[i];
#pragma unroll
    for (int i = 0; i < BV; ++i) *(V*)(Bs + (vrow + 32 * i) * kPitch + vcol * 16) = br[i];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // tile t travels in register set t % NSET; LDS stage t & 1 is written while stage (t-1) & 1 is multiplied
  fetch(areg[0], breg[0]);
  stash(0, areg[0], breg[0]);
#pragma unroll
  for (int t = 1; t <= NSET; ++t)
    if (t < nkt) fetch(areg[t % NSET], breg[t % NSET]);
  __syncthreads();
  const int a_rd = (wave_m * WTM + l32) * kPitch + half * 16;
  const int b_rd = BM * kPitch + (wave_n * WTN + l32) * kPitch + half * 16;
  for (int kt0 = 0; kt0 < nkt; kt0 += NSET) {
#pragma unroll
    for (int u = 0; u < NSET; ++u) {
      const int kt = kt0 + u;
      if (kt >= nkt) break;
      const char* st = lds + (kt & 1) * STAGE;
      if (kt + 1 < nkt) {
        stash((kt + 1) & 1, areg[(u + 1) % NSET], breg[(u + 1) % NSET]);
        if (kt + 1 + NSET < nkt) fetch(areg[(u + 1) % NSET], breg[(u + 1) % NSET]);
      }
#pragma unroll
      for (int ks = 0; ks < kRowBytes / 32; ++ks) {
        V af[TM], bf[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = *(const V*)(st + a_rd + i * 32 * kPitch + ks * 32);
#pragma unroll
        for (int j = 0; j < TN; ++j) bf[j] = *(const V*)(st + b_rd + j * 32 * kPitch + ks * 32);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) Mma<T>::run(af[i], bf[j], acc[i][j]);
      }
      __syncthreads();
    }
  }

  // the k-loop ended with a barrier: every wavefront is done with the tiles, LDS can be reused
  typename Vec<T>::type res[RowSlabs<T, WTM, WTN>::COUNT][RowSlabs<T, WTM, WTN>::MAX];
  igemm_epilogue<T, WTM, WTN, TM, TN, MODE, 16, false>(p, acc, m0, n0, wave_m, wave_n, l32, half, lds + wave * stage_bytes<T, WTM, WTN>(16), tid3.split, res);
}

// =================================================================================================
// The same GEMM with the tiles brought into LDS by the load unit itself (buffer_load ... lds): no
// VGPR staging, no ds_write (which shares the LDS pipe with the fragment reads and is the slower of
// the two).  LDS rows are dense (128 bytes); the 16-byte column
// of a row is XOR-swizzled with the row number so that fragment reads stay conflict-free.  A
// wavefront's load covers 8 rows x 128 bytes = 1 KiB, written at m0 + lane * 16.  The loads are
// issued from inline assembly so that the k-loop can wait for exactly the tile it is about to use.
// =================================================================================================
__device__ __forceinline__ void dma_load16(u32x4 rsrc, unsigned voffset, unsigned soffset, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset) : "memory");
}
// A load whose data nobody wants: 64 pieces of 128 bytes are on their way from memory to the caches, 4 bytes of each to LDS
__device__ __forceinline__ void dma_touch(u32x4 rsrc, unsigned voffset, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_addr), "v"(voffset), "s"(rsrc) : "memory");
}
__device__ __forceinline__ u32x4 make_rsrc_words(const void* base, unsigned bytes) {
  const unsigned long long a = (unsigned long long)base;
  return u32x4{(unsigned)a, (unsigned)(a >> 32) & 0xffffu, bytes, 0x00020000u};
}
// waits until at most n of this wavefront's vector-memory operations are outstanding (n < 64)
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Swizzle of the dense 128-byte LDS rows the load unit fills: row r keeps its 16-byte chunk c at position
// c ^ lds_swizzle(r).  A ds_read_b128 serves 16 lanes (256 bytes, the width of the bank window) per cycle; the
// fragment reads take the same chunk of 16 consecutive rows, which (r >> 1) & 7 spreads over the 16 positions of
// the window (two rows share a window).  With r & 7 rows r and r + 8 collide: every read takes twice as long
// (counter SQ_LDS_BANK_CONFLICT: half of the LDS cycles).
__device__ __forceinline__ int lds_swizzle(int row) { return (row >> 1) & 7; }

// =================================================================================================
// The same GEMM with the tiles brought into LDS by the load unit itself (see above), NSTAGE - 1 k-tiles in flight.  The loads of
// tile kt + NSTAGE - 1 are spread between the MFMAs of the first three k-steps of tile kt (so the load unit's queue never backs up
// into the issuing wavefront), every fragment read is issued one k-step ahead of its use, and the workgroup barrier sits before the
// last k-step: once it is passed, tile kt + 1 has landed for everyone and everyone holds its last fragments of tile kt in registers,
// so the first fragments of tile kt + 1 are read during that last k-step and the stage of tile kt can be refilled in the next
// iteration.
// Three stages, one workgroup per CU: 256x128 (144 KiB), 128x128 (96 KiB).  Two stages: 128x128 and 128x160 with two workgroups per
// CU, which hide each other's prologue and epilogue, and 256x320 (144 KiB), whose k-tile is long enough for one tile in flight.
// WM x WN wavefronts; with two per SIMD one has MFMAs to issue while the other waits at the barrier or for its fragments.
// KG > 1: the k-tiles are shared out over KG groups of WM x WN wavefronts, each with stages of its own; the sums meet in LDS.  For launches of
// at most a 64x64 workgroup per CU, whose four wavefronts would wait for two tiles of 16 KiB at a time: 2880x320x2880 16.0 -> 12.4 us,
// 720x640x2560 14.4 -> 12.0, 180x3840x1280 11.2 -> 9.7, 288x1280x1280 8.3 -> 7.2 (two stages, four groups or 128-row tiles: slower).
// Bound by the feed from beyond the L2 and by what a launch of few rounds leaves idle, hence the choice of tiles (see kDmaTiles): with the
// MFMAs taken out 2048x1280x5120 still took 49 of the 50 us that it took in the order of rows (weights from memory; 48 in that of best_band()), with the
// loads taken out 29.  More stages do not help (four and five: 49), nor does a wavefront that asks for the lines ahead (53).
// Measured, bf16, us (best of 128x128, 256x128 and 64x64 -> the tile of this list that kDmaTiles names): GEGLU 2048x10240x1280 72 -> 58
// (256x320), 3x3 16384x640x5760 139 -> 116 (128x160), 3x3 65536x320x2880 130 -> 121 (256x320), q/k/v 65536x960x320 79 -> 64 (256x320),
// GEGLU 8192x5120x640 78 -> 66 (256x320), 2048x1280x1280 16.2 -> 13.7 (128x128 for 64x64).
// =================================================================================================
constexpr int kTouches = 2, kTouchLds = 256;      // weights ahead: loads of a wavefront, where they land
// Wavefronts per SIMD that LDS allows: what the register budget is set for.
constexpr int p3_waves_per_simd(int bm, int bn, int waves, int stages) { return (int)(kLdsLimit / (stages * (bm + bn) * kRowBytes)) * waves / 4; }
template <typename T, int BM, int BN, int MODE, int WM = 2, int WN = 2, int NSTAGE = 3, int KG = 1, bool XTRA = false>
__global__ __launch_bounds__(64 * WM * WN * KG, p3_waves_per_simd(BM, BN, WM * WN, NSTAGE)) void k_igemm_p3(IgemmParams p) {
  typedef typename Vec<T>::type V;
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int ES = (int)sizeof(T), VN = Vec<T>::N, BK = kRowBytes / ES;
  constexpr int STAGE = (BM + BN) * kRowBytes;
  constexpr int AG = BM / (8 * NW), BG = BN / (8 * NW), OPS = AG + BG;     // 8-row groups (= loads) per wavefront and k-tile
  constexpr int RND = 8 * NW;                                  // rows one round of loads (one per wavefront) covers
  constexpr int NG = TM * TN;                                  // MFMA groups per k-step; loads go out during the first three k-steps
  static_assert(OPS < 32, "vmcnt range");
  extern __shared__ __attribute__((aligned(16))) char lds_all[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave_all % NW, group = KG > 1 ? wave_all / NW : 0;
  char* const lds = lds_all + group * (NSTAGE * STAGE);
  const int l32 = lane & 31, half = lane >> 5;
  // wavefronts w and w + 4 share a SIMD: with wave_n = w / WM they hold different column halves whenever a SIMD has two,
  // so when the tile's second half lies beyond N (N = 320: 2.5 tiles of 128) every SIMD keeps one working wavefront
  const int wave_m = wave % WM, wave_n = wave / WM;
  const TileId tid3 = tile_of(p);
  const int m0 = tid3.m_tile * BM, n0 = tid3.n_tile * BN;
  // all 64 columns of this wavefront are padding: it takes part in the tile loads and the barriers and skips the rest
  const bool idle = n0 + wave_n * WTN >= p.N;
  u32x4 rs0 = make_rsrc_words(p.src0, p.bytes0), rs1 = make_rsrc_words(p.src1, p.bytes1);
  u32x4 rsw = make_rsrc_words(p.w, p.bytes_w);

  // load i of a k-tile covers rows (NW i + wave) * 8 .. + 7 of the A tile (i < AG) or of the B tile
  const int r8 = lane >> 3, scol = (lane & 7) ^ (((wave * 8 + r8) >> 1) & 7);      // see lds_swizzle(); rows (NW i + wave) * 8 + r8
  const int kt_first = tid3.split * p.kt_per_split, kt_all = min(p.ktiles - kt_first, p.kt_per_split);
  // this group's share of them (never none, see the launcher)
  const int kt_each = (kt_all + KG - 1) / KG, kt_begin = kt_first + group * kt_each, nkt = KG == 1 ? kt_all : min(kt_all - group * kt_each, kt_each);
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds;
  const unsigned grp = (unsigned)wave * 8 * kRowBytes;
  // load i of the weights is RND rows after load 0; large tiles form its offset anew each time, for want of registers
  constexpr bool TIGHT = TM * TN * 16 > 128;
  unsigned b_row0 = weight_at(n0 + wave * 8 + r8, (unsigned)p.Kp * ES, p.w_row) + scol * 16, b_step = (unsigned)(RND * p.Kp) * ES;
  unsigned b_off[TIGHT ? 1 : BG];
  if constexpr (!TIGHT) {
#pragma unroll
    for (int i = 0; i < BG; ++i) b_off[i] = b_row0 + i * b_step;
  }
  auto b_at = [&](int i) {
    if constexpr (!TIGHT) return b_off[i];
    unsigned o;
    asm volatile("v_add_u32 %0, %1, %2" : "=v"(o) : "s"(i * b_step), "v"(b_row0));
    return o;
  };
  constexpr int CR = NW * stage_bytes<T, WTM, WTN>(32) <= NSTAGE * STAGE ? 32 : 16;
  constexpr bool PRE = MODE == OUT_ROWMAJOR && RowSlabs<T, WTM, WTN>::VGPRS <= 32;
  V res[RowSlabs<T, WTM, WTN>::COUNT][RowSlabs<T, WTM, WTN>::MAX];
  // the weight tiles of the first k-tiles go out before the row arithmetic below, which they do not need
#pragma unroll
  for (int t = 0; t < NSTAGE - 1; ++t)
    if (t < nkt) {
#pragma unroll
      for (int i = 0; i < BG; ++i) {
        if (XTRA && kt_begin + t >= p.kt_main) {
          const int xk = p.xc0 + p.xc1;
          dma_load16(make_rsrc_words(p.xw, p.xbytes_w), weight_at(n0 + wave * 8 + r8 + i * RND, (unsigned)xk * ES, p.xw_row) + scol * 16,
                     (unsigned)(kt_begin + t - p.kt_main) * p.w_kt, lds_base + t * STAGE + grp + (BM + i * RND) * kRowBytes);
        } else {
          dma_load16(rsw, b_at(i), (unsigned)(kt_begin + t) * p.w_kt, lds_base + t * STAGE + grp + (BM + i * RND) * kRowBytes);
        }
      }
    }
  if (PRE && p.residual && p.vec16 && !idle && group == 0) {
#pragma unroll
    for (int t = 0; t < RowSlabs<T, WTM, WTN>::COUNT; ++t) load_residual<T, WTM, WTN>(p, t, m0 + wave_m * WTM, n0 + wave_n * WTN, lane, res[t]);
  }
  // stored pixel of tap (0, 0), a bit per tap that falls inside the image, and (bits 9, 10) its parities for a nearest-2x input
  int a_pix[AG], a_taps[AG];
#pragma unroll
  for (int i = 0; i < AG; ++i) {
    const int m = m0 + (NW * i + wave) * 8 + r8;
    a_pix[i] = 0; a_taps[i] = 0;
    if (m < p.M) {
      const int b = (int)fast_div((unsigned)m, p.div_hw), r = m - b * p.hw_out;
      const int oy = (int)fast_div((unsigned)r, p.div_w), ox = r - oy * p.wout;
      const int iy = oy * p.stride - p.pad, ix = ox * p.stride - p.pad;
      a_pix[i] = (b * p.hs + (iy >> p.up)) * p.ws + (ix >> p.up);
      if (p.ksize == 1) {
        a_taps[i] = 1;
      } else {
        int in_row = 0;
#pragma unroll
        for (int v = 0; v < 3; ++v) in_row |= (ix + v >= 0 && ix + v < p.win) ? 1 << v : 0;
#pragma unroll
        for (int u = 0; u < 3; ++u) a_taps[i] |= (iy + u >= 0 && iy + u < p.hin) ? in_row << (3 * u) : 0;
      }
      a_taps[i] |= (iy & 1) << 9 | (ix & 1) << 10;
    }
  }
  // byte offsets of this lane's rows for the tap and the source being fetched
  unsigned a_off[AG];
  auto set_tap = [&](int tap, unsigned c) {                  // c: channels of the source
    const int u = p.ksize == 3 ? tap * 11 >> 5 : 0, v = tap - 3 * u;      // tap / 3 without vector work
    const int step = u * p.ws + v;
#pragma unroll
    for (int i = 0; i < AG; ++i) {
      const int pix = a_pix[i] + (p.up ? (((a_taps[i] >> 9 & 1) + u) >> 1) * p.ws + (((a_taps[i] >> 10 & 1) + v) >> 1) : step);
      a_off[i] = (a_taps[i] >> tap & 1) ? ((unsigned)pix * c + scol * VN) * ES : kOob;
    }
  };
  const int f_k0 = kt_begin * BK;
  unsigned f_w = (unsigned)kt_begin * p.w_kt;
  int f_tap = __builtin_amdgcn_readfirstlane(f_k0 / p.ctot);    // the division is vector work; what follows from it must not be
  int f_cc = f_k0 - f_tap * p.ctot;
  unsigned c0 = (unsigned)p.c0, c1 = (unsigned)p.c1;
  int s_c0 = p.c0, s_ctot = p.ctot;                          // channels of the first source and of both
  // XTRA: behind the nine taps other sources and weights take over, k counted anew; their pixel is the one of the middle tap
  auto begin_extra = [&]() {
    rs0 = make_rsrc_words(p.x0, p.xbytes0); rs1 = make_rsrc_words(p.x1, p.xbytes1); rsw = make_rsrc_words(p.xw, p.xbytes_w);
    c0 = (unsigned)p.xc0; c1 = (unsigned)p.xc1;
    s_c0 = p.xc0; s_ctot = p.xc0 + p.xc1;
    b_row0 = weight_at(n0 + wave * 8 + r8, (unsigned)s_ctot * ES, p.xw_row) + scol * 16;
    b_step = (unsigned)(RND * s_ctot) * ES;
    if constexpr (!TIGHT) {
#pragma unroll
      for (int i = 0; i < BG; ++i) b_off[i] = b_row0 + i * b_step;
    }
  };
  auto pixel_tap = [&](int tap) { return XTRA && tap >= 9 ? 4 : tap; };
  if (XTRA && kt_begin >= p.kt_main) {
    begin_extra();
    f_cc = (kt_begin - p.kt_main) * BK;
    f_w = (unsigned)(kt_begin - p.kt_main) * p.w_kt;
    f_tap = 9;
  }
  set_tap(pixel_tap(f_tap), f_cc >= s_c0 ? c1 : c0);
  // per-tile state of the loads being issued: the source that holds the channels, and the scalar offsets
  u32x4 rsa = rs0;
  unsigned soff_a = 0, soff_b = 0;
  auto begin_tile = [&]() {
    const bool second = f_cc >= s_c0;
    rsa = second ? rs1 : rs0;
    soff_a = (unsigned)((second ? f_cc - s_c0 : f_cc) * ES);
    soff_b = f_w;
  };
  auto issue_one = [&](int stage, int i) {
    const unsigned st = lds_base + stage * STAGE + grp;
    if (i < AG) dma_load16(rsa, a_off[i], soff_a, st + i * RND * kRowBytes);
    else dma_load16(rsw, b_at(i - AG), soff_b, st + (BM + (i - AG) * RND) * kRowBytes);
  };
  auto end_tile = [&]() {
    f_w += p.w_kt;
    f_cc += BK;
    if (f_cc == s_c0 || f_cc == s_ctot) {                    // the next source (c0 and ctot are multiples of the k-tile) or the next tap
      const int wrap = f_cc == s_ctot ? 1 : 0;
      f_cc = wrap ? 0 : f_cc;
      f_tap += wrap;
      if (XTRA && wrap && f_tap == 9) { begin_extra(); f_w = 0; }
      set_tap(pixel_tap(f_tap), wrap ? c0 : c1);             // behind the last tap nothing is fetched any more
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
  for (int t = 0; t < NSTAGE - 1; ++t) {
    if (t < nkt) {
      begin_tile();
#pragma unroll
      for (int i = 0; i < AG; ++i) issue_one(t, i);      // the B part of these tiles is already on its way
      end_tile();
    }
    if (t == 0 && p.ahead_bytes) {
      // Weights of a later launch, from memory into the memory-side cache (when that pays: kAheadRows): behind tile 0, ahead of tile 1, whose wait is the
      // first that includes them.  All wavefronts take the same share: 3.3 MB by the first 25 of 240 workgroups made 2048x3840x1280 1.7 us slower, by all of
      // them 0.5.  Workgroups of their own instead, in the launches of norms and attention in between, cost those 0.5 to 3 us each, and on other CUs they
      // took from the other streams what they gave: 1024px 0.2 to 0.7 % slower than without.
      const u32x4 rsn = make_rsrc_words(p.ahead, p.ahead_bytes);
      const unsigned first = ((blockIdx.y * gridDim.x + blockIdx.x) * (NW * KG) + wave_all) * p.ahead_span;
#pragma unroll
      for (int i = 0; i < kTouches; ++i) {
        const unsigned at = lane * 128 + i * 8192;
        dma_touch(rsn, at < p.ahead_span ? first + at : kOob, (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds_all + KG * NSTAGE * STAGE);
      }
    }
  }
  // fragment reads: row * 128 + ((chunk ^ lds_swizzle(row)) * 16), chunk = 2 ks + half
  const int a_row = (wave_m * WTM + l32) * kRowBytes, b_row = (BM + wave_n * WTN + l32) * kRowBytes;
  const int x7 = lds_swizzle(l32);
  int sw[kRowBytes / 32];
#pragma unroll
  for (int ks = 0; ks < kRowBytes / 32; ++ks) sw[ks] = ((ks * 2 + half) ^ x7) << 4;
  V fr[2][TM + TN];
  auto read_frag = [&](const char* st, int ks, int r) {
    fr[ks & 1][r] = r < TM ? *(const V*)(st + a_row + r * 32 * kRowBytes + sw[ks & 3])
                           : *(const V*)(st + b_row + (r - TM) * 32 * kRowBytes + sw[ks & 3]);
  };
  int stage = 0;
  // PHASE 2: a next tile follows and tile kt + NSTAGE - 1 is fetched; 1: a next tile follows; 0: last tile
  auto k_tile = [&](auto phase, auto idle_c) {
    constexpr int PHASE = decltype(phase)::value;
    constexpr bool IDLE = decltype(idle_c)::value;
    int target = stage + NSTAGE - 1;
    if (target >= NSTAGE) target -= NSTAGE;
    int next = stage + 1;
    if (next >= NSTAGE) next -= NSTAGE;
    const char* st = lds + stage * STAGE;
    const char* sn = lds + next * STAGE;
    if (PHASE == 2) begin_tile();
    int q = 0;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks == 3 && PHASE >= 1) {
        if (PHASE == 2) wait_vmcnt<(NSTAGE - 2) * OPS>(); else wait_vmcnt<0>();
        __syncthreads();
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int g = i * TN + j;
          if constexpr (!IDLE) Mma<T>::run(fr[ks & 1][i], fr[ks & 1][TM + j], acc[i][j]);
          // fragment r of the next k-step follows MFMA group floor(r NG / (TM+TN)); the loads follow one another over the first three
          // k-steps, with two stages over the first one (they are needed before this tile ends: 256x320 tiles, K = 5760, 246 -> 236 us)
#pragma unroll
          for (int r = 0; r < TM + TN; ++r)
            if (!IDLE && r * NG / (TM + TN) == g) {
              if (ks < 3) read_frag(st, ks + 1, r);
              else if (PHASE >= 1) read_frag(sn, 4, r);
            }
          if (PHASE == 2 && ks < 3) {
#pragma unroll
            for (int l = 0; l < OPS; ++l)
              if (l * (NSTAGE == 2 ? 1 : 3) * NG / OPS == q) issue_one(target, l);
          }
          __builtin_amdgcn_sched_barrier(0);
          ++q;
        }
    }
    if (PHASE == 2) end_tile();
    stage = next;
  };
  // issue order so far: B(0), B(1), A(0), weights ahead, A(1): tile 0 is complete once only those and A(1) are outstanding
  if (nkt < NSTAGE - 1) wait_vmcnt<0>();
  else if (p.ahead_bytes) wait_vmcnt<(NSTAGE - 2) * AG + kTouches>();
  else wait_vmcnt<(NSTAGE - 2) * AG>();
  __syncthreads();
  int kt = 0;
  if (idle) {
    for (; kt + NSTAGE - 1 < nkt; ++kt) k_tile(std::integral_constant<int, 2>{}, std::true_type{});
    for (; kt + 1 < nkt; ++kt) k_tile(std::integral_constant<int, 1>{}, std::true_type{});
    k_tile(std::integral_constant<int, 0>{}, std::true_type{});
    for (int i = nkt; i < kt_each; ++i) __syncthreads();
    __syncthreads();
    if constexpr (KG > 1) __syncthreads();
    if constexpr (MODE == OUT_GEGLU && TN % 2 != 0) __syncthreads();      // the epilogue's exchange
    return;
  }
#pragma unroll
  for (int r = 0; r < TM + TN; ++r) read_frag(lds, 0, r);
  for (; kt + NSTAGE - 1 < nkt; ++kt) k_tile(std::integral_constant<int, 2>{}, std::false_type{});
  for (; kt + 1 < nkt; ++kt) k_tile(std::integral_constant<int, 1>{}, std::false_type{});
  k_tile(std::integral_constant<int, 0>{}, std::false_type{});
  for (int i = nkt; i < kt_each; ++i) __syncthreads();       // every group passes the same barriers
  __syncthreads();     // every wavefront holds its last fragments: LDS can be reused by the epilogue
  if constexpr (KG > 1) {
    // the other groups hand over their sums, a register of all lanes at a time, behind what the epilogue stages in; added in order
    float* const hand = (float*)(lds_all + NSTAGE * STAGE);
    auto at = [&](int g, int i, int j, int r) { return hand + ((((g - 1) * NW + wave) * TM + i) * TN + j) * 1024 + r * 64 + lane; };
    static_assert((KG - 1) * NW * TM * TN * 4096 <= (KG - 1) * NSTAGE * STAGE, "hand-over area");
    if (group > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) *at(group, i, j, r) = acc[i][j][r];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += *at(g, i, j, r);
  }
  igemm_epilogue<T, WTM, WTN, TM, TN, MODE, CR, PRE>(p, acc, m0, n0, wave_m, wave_n, l32, half, lds + wave * stage_bytes<T, WTM, WTN>(CR), tid3.split, res,
                                                         (float*)(lds + NW * stage_bytes<T, WTM, WTN>(CR)) + wave_m * (WTM * 32));
}

// the instances that conv_takes_shortcut() counts on: 64x64, the two-stage tiles, and 128x128 and 256x128 on eight wavefronts
constexpr bool p3_takes_shortcut(int mode, int bn, int waves, int stages) {
  return (mode == OUT_ROWMAJOR || mode == OUT_PARTIAL) && (bn == 64 || stages == 2 || waves == 8);
}
template <typename T, int BM, int BN, int MODE, int WM = 2, int WN = 2, int NSTAGE = 3, int KG = 1, bool XTRA = false>
static ad_status run_igemm_p3(const IgemmParams& p0, const char* name, hipStream_t s) {
  if constexpr (!XTRA && p3_takes_shortcut(MODE, BN, WM * WN, NSTAGE))
    if (p0.xw) return run_igemm_p3<T, BM, BN, MODE, WM, WN, NSTAGE, KG, true>(p0, name, s);
  if (!XTRA && p0.xw) AD_FAIL(AD_ERR_INVALID, "conv: this tile does not take a shortcut");
  IgemmParams p = p0;
  set_tiles(p, BM, BN);
  // what the epilogue uses ends where the loads of weights ahead land: with two stages and a single k-tile those may still be on their way
  constexpr int tile_bytes = KG * NSTAGE * (BM + BN) * kRowBytes, lds_bytes = tile_bytes + kTouchLds;
  static_assert(tile_bytes / KG >= WM * WN * stage_bytes<T, BM / WM, BN / WN>(16) && lds_bytes <= (int)kLdsLimit, "epilogue staging fits");
  static_assert(MODE != OUT_GEGLU || BN / WN / 32 % 2 == 0 || tile_bytes >= WM * WN * stage_bytes<T, BM / WM, BN / WN>(32) + BM * 128, "so does the exchange");
  static std::atomic<bool> attr_set{false};
  if (!attr_set) {
    AD_HIP(hipFuncSetAttribute((const void*)k_igemm_p3<T, BM, BN, MODE, WM, WN, NSTAGE, KG, XTRA>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
    attr_set = true;
  }
  const int xk = p.xc0 + p.xc1;
  const double in_bytes = (double)p.M * (p.ctot + xk) * sizeof(T) * (p.stride == 2 ? 4 : 1) / (p.up ? 4 : 1);
  const double out_cols = p.out_mode == OUT_GEGLU ? p.N / 2 : p.N;
  ProfLaunch pl(name, 2.0 * p.M * p.N * (p.k_prof + xk), in_bytes + (double)p.N * (p.Kp + xk) * sizeof(T) + (double)p.M * out_cols * sizeof(T), s, p.M, p.N, p.Kp + xk);
  if (p.ahead_bytes) pl.fetches(p.ahead);
  const int splits = (p.ktiles + p.kt_per_split - 1) / p.kt_per_split;
  const unsigned waves = (unsigned)(p.tiles_n * p.tiles_m * splits * WM * WN * KG);
  p.ahead_span = (p.ahead_bytes / 128 + waves - 1) / waves * 128;
  hipLaunchKernelGGL((k_igemm_p3<T, BM, BN, MODE, WM, WN, NSTAGE, KG, XTRA>), dim3(p.tiles_n * p.tiles_m, splits), dim3(64 * WM * WN * KG), lds_bytes, s, p);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// =================================================================================================
// GEMM for outputs of a few hundred small tiles (the deep levels, narrow models, single samples).
//
// Such a launch is bound by latency: its operands come from memory (weights) or the memory-side cache (activations the
// previous launch has just written), a CU takes in only about 60 GB/s of those, and with 64x64 tiles there are fewer
// workgroups than CUs, each walking the whole of K tile by tile behind a barrier.  So the tiles are small (16x16 to 32x64,
// enough of them for the chip), the wavefronts of a workgroup share K (wavefront w takes k-tiles w, w + NW, ...) and load
// their 16x16x32 MFMA fragments straight from memory into registers, two k-tiles ahead: no LDS, no barrier before the
// partial tiles are added, in wavefront order, through LDS.  The weights are the A operand, so that a lane holds four
// consecutive columns of a row.  What the epilogue adds is requested before the loop.
// Measured, bf16, weights from memory, us (64x64 tiles in three stages -> this kernel): 1152x64x64 4.1 -> 3.1, 3x3 1152x64x576
// 7.4 -> 4.4, 3x3 288x128x1152 10.8 -> 4.8, 72x256x1024 7.8 -> 4.7, 180x1280x1280 11.4 -> 7.9; 3x3 72x256x2304 with K split
// over workgroups and a second launch 11.8 -> 6.8.
//
// LN: a LayerNorm in front of the (linear) layer, without a launch and a pass through memory of its own: the fragments of the rows are normalised in
// registers on their way into the matrix cores, with the arithmetic of k_layernorm (fp32 statistics, gain and offset, the result rounded to T).  Neither
// the row's mean nor the gain goes through the product: taken off the sum over K the mean costs relative precision by its ratio to the row's spread
// (fp32, 256 channels, 100 standard deviations: 1.1e-5 instead of 3.5e-6; rows of one value 1e-2), and a gain that is rounded into bf16 weights shows where
// the products cancel (3e-2 instead of 2e-3).  The statistics are those of k_layernorm to the bit: a workgroup reads its rows, 16 bytes a thread, ahead of
// the fragments and adds them up in two passes in the order of 64 lanes a row.  (Sums and squared deviations that the launch in front leaves for every 16 or
// 32 columns save that reading, level in time, but are another order of the sums: whole bf16 runs differed by 2e-3 to 6e-3 from those with a launch.)
// Gain and offset go through LDS: in registers, two k-tiles ahead like the fragments, they take 64 of them.
// Measured inside the models, us (norm + GEMM -> GEMM): bf16 72x768x256 3.6 + 3.8 -> 5.5, 72x2048x256 3.6 + 4.5 -> 6.0, 18x2048x256 3.3 + 4.2 -> 5.9, 45x3840x1280
// 3.9 + 8.6 -> 11.0; fp32 288x384x128 3.6 + 4.0 -> 5.2, 288x1024x128 3.6 + 6.2 -> 7.6, 72x2048x256 3.6 + 6.0 -> 7.6; and the gap between two launches.  Whole runs
// against a launch for every norm, ms: narrow model 37.28 -> 36.73, fp32 17.53 -> 17.21, with stride 2 27.04 -> 25.84, 576x320 px 64.39 -> 64.13, 512px level.
// The larger tiles, whose LDS is filled by the load unit and whose fragments every column tile would normalise again, leave the norm to k_layernorm.
//
// GN: a GroupNorm (and SiLU) in front of a 3x3 convolution of a small map, likewise: the launch it saves takes 3.6 us, nearly all of it the launch itself and a
// round trip to memory, in a chain of launches that wait for one another.  Every workgroup takes in the samples that its rows belong to (9 to 256 pixels), a
// wavefront an eighth of the channels, so that the statistics of its groups need no other wavefront; the pixels that the taps read are normalised once, on
// their way into LDS, and the fragments come from there.  Statistics and norm are k_gn_group's to the bit (gn_stats()): its order of the sums, one number taken off all values
// of a group, the last sums in double.  Bound by vector instructions: two wavefronts a SIMD, 680 to 1120 each with the product's 160.
// Measured inside the models, us (norm + convolution -> convolution): bf16 18x256x2304 3.8 + 5.9 -> 9.3, 72x256x2304 3.7 + 6.3 -> 9.5, 128x256x2304 3.7 + 7.4 -> 9.6,
// 288x128x1152 3.7 + 4.8 -> 8.9; fp32 288x128x1152 3.7 + 7.9 -> 9.9, 64x64x576 3.7 + 4.8 -> 7.1, 256x32x288 3.6 + 3.9 -> 8.3: what it saves is the gap between two launches.
// Whole runs, a launch for every norm / this, ms, the same bits: tiny fp32 2.16 / 1.74, narrow 35.2 / 34.5, with stride 2 25.35 / 25.11, narrow fp32 12.93 / 12.28.  (With every
// lane's sums over its own accesses, rotated within the row and folded in fp32, a launch took 1 to 1.5 us less, but lanes took different numbers off the values of a group
// where their sums met a boundary of 12 bits (fp32 values up to 2e-2 off), and sums of squares beyond fp32 left the offset alone.)
// XTRA: the 1x1 shortcut of a ResBlock as k-tiles behind the taps, in sums of their own, which take the storage type before they are added: the bits of a launch for the
// shortcut, whose sum is the residual.  (In one sum with the taps, as in k_igemm_p3, it saves 0.1 us, but bf16 runs differed by 4e-3 to 7e-3 from those with a launch.)  fp32 too.
// us (norm + shortcut + second convolution -> one): bf16 18x256 of 2304 + 512 3.8 + 4.2 + 6.3 -> 10.3, 72x256 3.7 + 4.1 + 6.7 -> 11.7, 288x128 of 1152 + 256 3.7 + 3.8 + 4.9 ->
// 9.1; fp32 256x32 of 288 + 96 3.6 + 3.6 + 4.3 -> 7.6.  Launches of a step: tiny fp32 34 -> 29, narrow 204 -> 190, narrow fp32 223 -> 213.
// Taken back: statistics over all wavefronts through LDS, merged in double (4.3 us a launch), and 1x1 convolutions (72x256x256 3.7 + 3.9 -> 7.9).
// Four k-tiles of fragments on their way instead of two are level (18x256x2304 8.5 / 8.7 us, fp32 10.4 / 10.7, fp32 72x2048x256 8.1 / 7.9; whole runs 0.993 to 1.003): what a CU
// takes in at a time decides, not how early a wavefront asks.
// =================================================================================================
constexpr int small_ktiles(int bm, int bn) { return 200 * 1024 / ((bm + bn) * kRowBytes); }      // k-tiles that small_tile() takes at the most (bf16), and of a LayerNorm in front
// Sum over the threads of a row, TPR = 16 or 32 neighbouring lanes, as k_layernorm's lanes add up: distances 32 / TPR .. 1, where a distance within 16 lanes is a
// rotation, since the lanes that it brings together hold the same already.
template <int TPR>
__device__ __forceinline__ float ln_threads(float v) {
  if (TPR == 32) v += __shfl_xor(v, 16, 64);
  v += dpp_f<0x128>(v);                                  // row_ror 8
  v += dpp_f<0x124>(v);                                  // row_ror 4
  v += dpp_f<0x4E>(v);                                   // quad_perm 2 3 0 1
  return v + dpp_f<0xB1>(v);                             // quad_perm 1 0 3 2
}
// What k_layernorm and a linear layer with the norm inside have in common: the squared deviations of an access added to those of the lane's earlier ones
// (first: there are none), and the norm of an element, with the products fused as written here and not as the compiler would choose for either of them.
template <typename V>
__device__ __forceinline__ float ln_squares(const V& x, float mean, float q, bool first) {
  const float d0 = to_f(x[0]) - mean, d1 = to_f(x[1]) - mean;
  q = first ? fmaf(d0, d0, d1 * d1) : fmaf(d1, d1, fmaf(d0, d0, q));
#pragma unroll
  for (int e = 2; e < (int)(sizeof(V) / sizeof(x[0])); ++e) { const float d = to_f(x[e]) - mean; q = fmaf(d, d, q); }
  return q;
}
__device__ __forceinline__ float ln_value(float x, float mean, float rstd, float gain, float offset) { return fmaf((x - mean) * rstd, gain, offset); }
// Thread `sub` of a row has its accesses sub, sub + TPR, ...: those of the lanes sub, sub + TPR, ... of 64, each of which k_layernorm sums for itself.  (Where it
// gives a row fewer lanes, each has one access at the most in all launches that small_tile() takes, and the sums are the same.)
template <typename T, int TPR, int LD>
__device__ __forceinline__ void ln_load(const IgemmParams& p, int row, int sub, typename Vec<T>::type (&x)[LD]) {
  typedef typename Vec<T>::type V;
  const T* rp = (const T*)p.src0 + (size_t)min(row, p.M - 1) * p.ctot;
#pragma unroll
  for (int i = 0; i < LD; ++i)
    if ((sub + TPR * i) * Vec<T>::N < p.ctot) x[i] = *(const V*)(rp + (sub + TPR * i) * Vec<T>::N);
}
template <typename T, int TPR, int LD>
__device__ __forceinline__ void ln_stats(const IgemmParams& p, int sub, const typename Vec<T>::type (&x)[LD], float* mean_out, float* rstd_out) {
  constexpr int VN = Vec<T>::N, LANES = 64 / TPR;
  auto row_sum = [&](const float (&v)[LANES]) {
    if constexpr (LANES == 4) return ln_threads<TPR>((v[0] + v[2]) + (v[1] + v[3]));
    else return ln_threads<TPR>(v[0] + v[1]);
  };
  float s[LANES] = {}, q[LANES] = {};
#pragma unroll
  for (int i = 0; i < LD; ++i)
    if ((sub + TPR * i) * VN < p.ctot)
#pragma unroll
      for (int e = 0; e < VN; ++e) s[i % LANES] += to_f(x[i][e]);
  const float mean = row_sum(s) / p.ctot;
#pragma unroll
  for (int i = 0; i < LD; ++i)
    if ((sub + TPR * i) * VN < p.ctot) q[i % LANES] = ln_squares(x[i], mean, q[i % LANES], i < LANES);
  const float rstd = rsqrtf(row_sum(q) / p.ctot + p.ln_eps);
  if (sub == 0) { *mean_out = mean; *rstd_out = rstd; }
}

constexpr int small_sum_bytes(int bm, int bn) { return 8 * bm * (bn + 4) * 4; }      // partial sums of the wavefronts of a small tile
constexpr int gn_pitch(int row_bytes) { return row_bytes + 16; }      // of a pixel in LDS: 16 neighbouring pixels fall on different banks
constexpr int gn_act_bytes(int bm, int ws, int row_bytes) { return 256 + (bm + 2 * (ws + 1)) * gn_pitch(row_bytes); }
// What k_gn_group and a convolution with the norm inside have in common, with the products fused as written: the deviations of a group's channels in an access, FROM and
// the PER - 1 behind it, added to a thread's sums (first: there are none yet), what the sums make of a group, and the norm of an element.  sum: of the deviations
// from `about`; rest: what the mean is beyond that.
template <int FROM, int PER, typename V>
__device__ __forceinline__ void gn_add(const V& x, float about, float& s, float& q, bool first) {
  float d[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) { d[e] = to_f(x[FROM + e]) - about; s += d[e]; }
  constexpr int NEXT = PER > 1 ? 1 : 0;
  if (PER > 1 && first) q = fmaf(d[0], d[0], d[NEXT] * d[NEXT]);
  else q = fmaf(d[0], d[0], q);
#pragma unroll
  for (int e = 1; e < PER; ++e)
    if (e > 1 || !first) q = fmaf(d[e], d[e], q);
}
__device__ __forceinline__ void gn_moments(double sum, double squares, double inv_n, float eps, float& rstd, float& rest) {
  const double mean = sum * inv_n;
  double var = fma(inv_n, squares, -(mean * mean));
  var = (var < 0.0 ? 0.0 : var) + (double)eps;
  // 1 / sqrt(var): one Newton step on the fp32 value, a fifth of the instructions of the double division and root
  const double r0 = rsqrtf((float)var);
  rstd = (float)(var > 1e-30 && var < 1e30 ? fma(-0.5 * var * r0, r0, 1.5) * r0 : 1.0 / sqrt(var));
  rest = (float)mean;
}
__device__ __forceinline__ float gn_about(float sum, double inv_n) { return __uint_as_float(__float_as_uint(sum * (float)inv_n) & 0xfffff000u); }
__device__ __forceinline__ float gn_value(float x, float about, float gain, float offset) { return fmaf(x - about, gain, offset); }

// Pixel of a lane in an access: pixel bit 0 is the highest of the row's bits behind the accesses, and so on downwards, so that the pixels to be added up first lie 8
// lanes apart, the next 4, ...; then the rows of 16 lanes
__device__ __forceinline__ int gn_pixel(int lane, int log_vps) {
  const int r = (lane & 15) >> log_vps, bits = 4 - log_vps;
  return (int)(__brev((unsigned)r) >> 1 >> (31 - bits)) + (lane >> 4 << bits);
}
// Sums over the lanes of a group, in every one of them: first over its accesses to a pixel, then over pixels 1, 2, 4, ... apart, as the 64 threads of a wavefront
// of k_gn_group add up.  Both lanes of a pair add the same two numbers, so all lanes hold the same; a distance of 4 lanes is a rotation by 4 where lanes
// 8 apart hold the same already.
template <int GP, int S>
__device__ __forceinline__ void gn_lanes(const GnLayout& g, float (&sums)[GP][S]) {
  constexpr int N = GP * S;
  float v[(N + 3) / 4 * 4];
#pragma unroll
  for (int i = 0; i < (N + 3) / 4 * 4; ++i) v[i] = i < N ? sums[i < N ? i / S : 0][i % S] : 0.f;
  const int in_row = 4 - g.log_vps;                      // pixel bits within a row
  if (g.vpp >= 2)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += dpp_f<0xB1>(v[i]);                   // quad_perm 1 0 3 2
  if (g.vpp >= 4)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += dpp_f<0x4E>(v[i]);                   // quad_perm 2 3 0 1
  if (g.bits > 0 && in_row > 0)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += dpp_f<0x128>(v[i]);                  // row_ror 8
  if (g.bits > 1 && in_row > 1)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += dpp_f<0x124>(v[i]);                  // row_ror 4
  if (g.bits > 2 && in_row > 2)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += dpp_f<0x122>(v[i]);                  // row_ror 2
  if (g.bits > 3 && in_row > 3)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += dpp_f<0x121>(v[i]);                  // row_ror 1
  auto swap16 = [](float& x, float& y) {                 // odd rows of x and even rows of y change places
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(h[0]); y = __uint_as_float(h[1]);
  };
  auto swap32 = [](float& x, float& y) {                 // upper half of x and lower half of y
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(h[0]); y = __uint_as_float(h[1]);
  };
  if (g.bits > in_row + 1) {
    // four sums at a time, a row of the result each, and back to all rows
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      float a = v[i], b = v[i + 1], c = v[i + 2], d = v[i + 3];
      swap16(a, b); a += b;
      swap16(c, d); c += d;
      swap32(a, c); a += c;
      b = a;
      swap16(a, b);
      c = a; d = b;
      swap32(a, c); swap32(b, d);
      v[i] = a; v[i + 1] = b; v[i + 2] = c; v[i + 3] = d;
    }
  } else if (g.bits > in_row) {
#pragma unroll
    for (int i = 0; i < N; ++i) { float o = v[i]; swap16(v[i], o); v[i] += o; }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) sums[i / S][i % S] = v[i];
}
// Sum over the accesses of a group as k_gn_group's wavefronts add up: `run` accesses are one of them, pairwise, the wavefronts follow one another (ACC)
template <typename ACC, int S>
__device__ __forceinline__ ACC gn_waves(int run, const float (&r)[S]) {
  ACC sum = 0;
  auto add = [&](auto size) {
    constexpr int R = decltype(size)::value;
#pragma unroll
    for (int k = 0; k < S; k += R) {
      float w[R];
#pragma unroll
      for (int i = 0; i < R; ++i) w[i] = k + i < S ? r[k + i < S ? k + i : 0] : 0.f;
#pragma unroll
      for (int n = 1; n < R; n *= 2)
#pragma unroll
        for (int i = 0; i + n < R; i += 2 * n)
          if (k + i + n < S) w[i] += w[i + n];
      sum += w[0];
    }
  };
  if (run == 1) add(std::integral_constant<int, 1>{});
  else if (S <= 2 || run == 2) add(std::integral_constant<int, 2>{});
  else if (S <= 4 || run == 4) add(std::integral_constant<int, 4>{});
  else add(std::integral_constant<int, 8>{});
  return sum;
}
// A wavefront's eighth of the channels (whole groups; of those of an access the first GP, PER channels each) of the pixels that begin in its lane 0, in registers: access
// k < S of a lane is pixel px + k * step, nothing from `left` on.  `about`, gain and offset of the lane's channels, for gn_value().  The statistics are k_gn_group's to the bit: there 256 threads
// hold a group, thread t the access t % vpp of pixels t / vpp, + 256 / vpp, ...; every thread adds up its own elements, the lanes of a wavefront
// pairwise, the wavefronts in order, in double the deviations.  Here 4 * run accesses of the lanes are those threads.
template <typename T, int S, int GP, int PER, bool CHAINED, int N>
__device__ __forceinline__ void gn_stats(const IgemmParams& p, const GnLayout& gn, const u32x4 (&x)[N], int px, int left, float (&about)[Vec<T>::N], float (&gain)[Vec<T>::N],
                                         float (&offset)[Vec<T>::N]) {
  typedef typename Vec<T>::type V;
  constexpr int CN = GP * PER;
  const int step = 64 >> gn.log_vps, threads = 4 * gn.run;
  float s[GP][S], q[GP][S];
  // what thread `k` of the group adds up: access k and (CHAINED) those a multiple of `threads` behind it
  auto each = [&](int k, auto visit) {
    if (!CHAINED) return visit(k);
    if (k >= threads) return;
#pragma unroll
    for (int j = k; j < S; j += 4)
      if (j == k || ((j - k) & (threads - 1)) == 0) visit(j);
  };
  auto clear = [&](float (&v)[GP][S]) {
#pragma unroll
    for (int g = 0; g < GP; ++g)
#pragma unroll
      for (int k = 0; k < S; ++k) v[g][k] = 0.f;
  };
  static_assert(GP <= 2, "groups that all_groups() visits");
  auto all_groups = [&](auto visit) {
    visit(std::integral_constant<int, 0>{});
    if constexpr (GP > 1) visit(std::integral_constant<int, 1>{});
  };
  clear(s);
#pragma unroll
  for (int k = 0; k < S; ++k)
    each(k, [&](int j) {
      if (px + j * step < left)
#pragma unroll
        for (int e = 0; e < CN; ++e) s[e / PER][k] += to_f(__builtin_bit_cast(V, x[j])[e]);
    });
  gn_lanes(gn, s);
#pragma unroll
  for (int g = 0; g < GP; ++g) {
    const float a = gn_about(gn_waves<float>(gn.run, s[g]), p.gn_inv_n);
#pragma unroll
    for (int e = g * PER; e < (g + 1) * PER; ++e) about[e] = a;
  }
  clear(s); clear(q);
#pragma unroll
  for (int k = 0; k < S; ++k)
    each(k, [&](int j) {
      if (px + j * step < left)
        all_groups([&](auto g) { gn_add<decltype(g)::value * PER, PER>(__builtin_bit_cast(V, x[j]), about[decltype(g)::value * PER], s[decltype(g)::value][k], q[decltype(g)::value][k], j == k); });
    });
  gn_lanes(gn, s);
  gn_lanes(gn, q);
#pragma unroll
  for (int g = 0; g < GP; ++g) {
    float rstd, rest;
    gn_moments(gn_waves<double>(gn.run, s[g]), gn_waves<double>(gn.run, q[g]), p.gn_inv_n, p.ln_eps, rstd, rest);
#pragma unroll
    for (int e = g * PER; e < (g + 1) * PER; ++e) { gain[e] *= rstd; offset[e] = fmaf(-rest, gain[e], offset[e]); }
  }
}
// Normalises the samples of a tile, one after the other, and leaves the pixels that the tile reads, rows lo .. hi - 1, in LDS behind 256 zero bytes.  One barrier.
template <typename T, int N>
__device__ __forceinline__ void gn_stage(const IgemmParams& p, u32x4 (&x)[N], const float (&gain)[Vec<T>::N], const float (&offset)[Vec<T>::N],
                                         int first, int pixels, int px, int channel, int lo, int hi, char* base) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  if (threadIdx.x < 16) *(f32x4*)(base + threadIdx.x * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
  const int pitch = gn_pitch(p.ctot * (int)sizeof(T)), step = 64 >> p.gn.log_vps;
  char* const to = base + 256 + channel * (int)sizeof(T);
  for (int at = 0; at < pixels; at += p.gn.pixels) {
    GnLayout gn = p.gn;
    // not known to be the same for every sample: the compiler would make a copy of the loop for each of their values
    asm volatile("" : "+s"(gn.vpp), "+s"(gn.per_access), "+s"(gn.run), "+s"(gn.slots), "+s"(gn.bits), "+s"(gn.chained), "+s"(gn.log_vps));
    const int left = min(gn.pixels, pixels - at);
    float about[VN], ga[VN], be[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) { ga[e] = gain[e]; be[e] = offset[e]; }
    auto by_slots = [&](auto groups, auto channels) {
      constexpr int GP = decltype(groups)::value, PER = decltype(channels)::value;
      constexpr bool WHOLE = PER == VN;
      if (WHOLE && gn.chained && gn.slots == N) gn_stats<T, N, GP, PER, WHOLE>(p, gn, x, px, left, about, ga, be);
      else if (WHOLE && gn.chained) gn_stats<T, N / 2, GP, PER, WHOLE>(p, gn, x, px, left, about, ga, be);
      else if (gn.slots == N) gn_stats<T, N, GP, PER, false>(p, gn, x, px, left, about, ga, be);
      else if (gn.slots == N / 2) gn_stats<T, N / 2, GP, PER, false>(p, gn, x, px, left, about, ga, be);
      else gn_stats<T, N / 5, GP, PER, false>(p, gn, x, px, left, about, ga, be);
    };
    if (gn.per_access == 1) by_slots(std::integral_constant<int, 1>{}, std::integral_constant<int, VN>{});
    else if (VN == 8 && gn.per_access == 2) by_slots(std::integral_constant<int, 2>{}, std::integral_constant<int, VN / 2>{});
    else {
      // groups of two channels: half of an access at a time, for want of registers
      auto turn = [](float& y, float& z) { const float w = y; y = z; z = w; };
#pragma nounroll
      for (int half = 0; half < 2; ++half) {
        by_slots(std::integral_constant<int, VN / 4>{}, std::integral_constant<int, 2>{});
#pragma unroll
        for (int e = 0; e < VN / 2; ++e) { turn(about[e], about[e + VN / 2]); turn(ga[e], ga[e + VN / 2]); turn(be[e], be[e + VN / 2]); }
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = __builtin_shufflevector(x[k], x[k], 2, 3, 0, 1);
      }
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int row = first + at + px + k * step;
      if (k >= gn.slots || px + k * step >= left || row < lo || row >= hi) continue;
      V o;
#pragma unroll
      for (int e = 0; e < VN; ++e) o[e] = from_f<T>(silu_f(gn_value(to_f(__builtin_bit_cast(V, x[k])[e]), about[e], ga[e], be[e])));
      *(V*)(to + (row - lo) * pitch) = o;
    }
    // the next sample's accesses to the front
    auto shift = [&](auto by) {
#pragma unroll
      for (int k = 0; k + decltype(by)::value < N; ++k) x[k] = x[k + decltype(by)::value];
    };
    if (at + gn.pixels >= pixels) break;
    if (gn.slots == N / 2) shift(std::integral_constant<int, N / 2>{});
    else shift(std::integral_constant<int, N / 5>{});
  }
  __syncthreads();
}

enum { NORM_NONE = 0, NORM_LAYER = 1, NORM_GROUP = 2 };
constexpr int gn_hold(int vn) { return vn == 8 ? 6 : 10; }      // GN: accesses of vn elements that a thread holds at the most
template <typename T, int TM, int TN, int MODE, int NORM = NORM_NONE, bool XTRA = false>
__global__ __launch_bounds__(512) void k_igemm_small(IgemmParams p) {
  constexpr bool LN = NORM == NORM_LAYER, GN = NORM == NORM_GROUP;
  typedef typename Vec<T>::type V;
  typedef typename Vec4<T>::type V4;
  constexpr int BM = 16 * TM, BN = 16 * TN, NW = 8, PF = 2, PITCH = BN + 4;
  constexpr int ES = (int)sizeof(T), BK = kRowBytes / ES, VN = Vec<T>::N;
  constexpr bool TRANSPOSED = MODE == OUT_TRANSPOSED || MODE == OUT_TRANSPOSED_F32;
  static_assert(MODE != OUT_GEGLU || BN == 64, "32 value columns and their 32 gates");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* const part = (float*)lds;                       // [wavefront][BM][PITCH]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const TileId t3 = tile_of(p);
  const int m0 = t3.m_tile * BM, n0 = t3.n_tile * BN;

  // byte offsets of this lane's rows; the activations' at tap (0, 0) (modulo 2^32 where that tap lies before the tensor), with a bit per
  // tap that falls inside the image
  unsigned a_off0[TM], a_off1[TM], a_taps[TM], b_off[TN];
  int a_par[TM];                                         // nearest-2x input: row and column parity of tap (0, 0)
#pragma unroll
  for (int j = 0; j < TN; ++j) b_off[j] = weight_at(n0 + 16 * j + r16, (unsigned)p.Kp * ES, p.w_row) + kg * 16;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + 16 * i + r16;
    a_taps[i] = 0; a_off0[i] = 0; a_off1[i] = 0; a_par[i] = 0;
    if (m < p.M) {
      const int b = (int)fast_div((unsigned)m, p.div_hw), r = m - b * p.hw_out;
      const int oy = (int)fast_div((unsigned)r, p.div_w), ox = r - oy * p.wout;
      const int iy0 = oy * p.stride - p.pad, ix0 = ox * p.stride - p.pad;
      const unsigned pix = (unsigned)((b * p.hs + (iy0 >> p.up)) * p.ws + (ix0 >> p.up));
      a_off0[i] = (pix * (unsigned)p.c0 + kg * VN) * ES;
      a_off1[i] = (pix * (unsigned)p.c1 + kg * VN) * ES;
      a_par[i] = (iy0 & 1) + 2 * (ix0 & 1);
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v)
          if (u < p.ksize && v < p.ksize && iy0 + u >= 0 && iy0 + u < p.hin && ix0 + v >= 0 && ix0 + v < p.win) a_taps[i] |= 1u << (u * 3 + v);
    }
  }
  const __amdgpu_buffer_rsrc_t rs0 = make_rsrc(p.src0, p.bytes0);
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(p.src1, p.bytes1);
  const __amdgpu_buffer_rsrc_t rsw = make_rsrc(p.w, p.bytes_w);

  const int kt_taps = XTRA ? p.kt_main : p.ktiles, mine = (kt_taps - wave + NW - 1) / NW;      // k-tiles of this wavefront (0 when there are fewer k-tiles than wavefronts)
  int f_tap = wave * BK / p.ctot, f_cc = wave * BK - f_tap * p.ctot;
  unsigned f_w = (unsigned)wave * p.w_kt;
  V af[GN ? 1 : PF][TM][2], bf[PF][TN][2];
  // GN: a wavefront's eighth of the channels of the samples that the tile's rows belong to, asked for ahead of everything else
  constexpr int HOLD = GN ? gn_hold(VN) : 1;
  u32x4 held[HOLD];
  float g_gain[GN ? VN : 1], g_offset[GN ? VN : 1];
  int g_px = 0, g_channel = 0, g_first = 0, g_pixels = 0, g_lo = 0, g_hi = 0;
  if constexpr (GN) {
    const int m_last = min(m0 + BM, p.M) - 1, z0 = (int)fast_div((unsigned)m0, p.div_hw), reach = p.ws + 1;
    g_first = z0 * p.hw_out;
    g_pixels = ((int)fast_div((unsigned)m_last, p.div_hw) - z0 + 1) * p.hw_out;
    g_lo = max(m0 - reach, g_first); g_hi = min(m_last + reach + 1, g_first + g_pixels);
    g_px = gn_pixel(lane, p.gn.log_vps);
    g_channel = (((wave << p.gn.log_vps) + (lane & ((1 << p.gn.log_vps) - 1)))) * VN;
    const bool second = g_channel >= p.c0;
    const T* src = second ? (const T*)p.src1 + (g_channel - p.c0) : (const T*)p.src0 + g_channel;
    const int ld = second ? p.c1 : p.c0, step = 64 >> p.gn.log_vps;
    int at = 0, slot = 0;                                // the samples one after the other, each from lane 0 on
#pragma unroll
    for (int k = 0; k < HOLD; ++k) {
      const int in_sample = g_px + slot * step;
      // a lane without a pixel loads the first one: without branches all loads go out one after the other
      if (at < g_pixels) held[k] = *(const u32x4*)(src + (size_t)(g_first + (in_sample < p.gn.pixels && at + in_sample < g_pixels ? at + in_sample : 0)) * ld);
      if (++slot == p.gn.slots) { slot = 0; at += p.gn.pixels; }
    }
#pragma unroll
    for (int e = 0; e < VN; e += 4) {
      const f32x4 g = *(const f32x4*)(p.ln_gain + g_channel + e), o = *(const f32x4*)(p.ln_offset + g_channel + e);
#pragma unroll
      for (int i = 0; i < 4; ++i) { g_gain[e + i] = g[i]; g_offset[e + i] = o[i]; }
    }
  }
  auto fetch = [&](int s) {
    const int u = p.ksize == 3 ? f_tap / 3 : 0, v = p.ksize == 3 ? f_tap - 3 * u : 0;
    const unsigned bit = 1u << (u * 3 + v), sb = f_w;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) bf[s][j][h] = buffer_load16<V>(rsw, b_off[j] + h * 64, sb);
    if constexpr (GN) { f_w += NW * p.w_kt; return; }
    const bool second = f_cc >= p.c0;
    const unsigned cs = (unsigned)(second ? p.c1 : p.c0) * ES, sc = (unsigned)(second ? f_cc - p.c0 : f_cc) * ES;
    // the tap goes into the lane's offset: the range check compares that offset with the tensor's size less the scalar one, which
    // therefore has to stay below the size (it does: a channel, never a row, of the tensor)
    const unsigned tap = (unsigned)(u * p.ws + v) * cs;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      unsigned o = second ? a_off1[i] : a_off0[i];
      o += p.up ? (unsigned)((((a_par[i] & 1) + u) >> 1) * p.ws + (((a_par[i] >> 1) + v) >> 1)) * cs : tap;
      o = (a_taps[i] & bit) ? o : kOob;
#pragma unroll
      for (int h = 0; h < 2; ++h) af[s][i][h] = second ? buffer_load16<V>(rs1, o + h * 64, sc) : buffer_load16<V>(rs0, o + h * 64, sc);
    }
    f_w += NW * p.w_kt; f_cc += BK * NW;
    if constexpr (LN) return;                            // one tap, one source
    while (f_cc >= p.ctot) { f_cc -= p.ctot; ++f_tap; }
  };
  // LN: threads a row, the accesses of 16 bytes a thread has to it and to gain and offset at the most, and what is asked for ahead of the fragments
  constexpr int TPR = 64 * NW / BM, KT = LN ? small_ktiles(BM, BN) : 0, LD = LN ? (KT * (kRowBytes / 16) + TPR - 1) / TPR : 1, GL = LN ? (KT * BK / 2 + 511) / 512 : 1;
  float* const ln_rows = part + NW * BM * PITCH;         // [BM] mean, [BM] 1 / standard deviation
  float* const ln_chan = ln_rows + 2 * BM;               // [ctot] gain, [ctot] offset (in registers, two k-tiles ahead, they take 64 of them)
  V x[LD];
  f32x4 chan[GL];
  if constexpr (LN) {
    ln_load<T, TPR, LD>(p, m0 + tid / TPR, tid % TPR, x);
#pragma unroll
    for (int i = 0; i < GL; ++i) {
      const int at = 4 * (tid + 512 * i);
      if (at < 2 * p.ctot) chan[i] = *(const f32x4*)(at < p.ctot ? p.ln_gain + at : p.ln_offset + (at - p.ctot));
    }
  }
#pragma unroll
  for (int s = 0; s < PF; ++s)
    if (s < mine) fetch(s);

  // XTRA: behind the taps the k-tiles of a 1x1 convolution of other sources, taken in turn as well; a wavefront's first one, x_first, is asked for ahead of the loop
  V xa[XTRA ? TM : 1][2], xb[XTRA ? TN : 1][2];
  const int x_tiles = p.ktiles - kt_taps, x_first = (wave + NW - kt_taps % NW) % NW;
  auto fetch_extra = [&](int e) {
    const int xk = p.xc0 + p.xc1, cc = e * BK;
    const bool second = cc >= p.xc0;
    const __amdgpu_buffer_rsrc_t rx = second ? make_rsrc(p.x1, p.xbytes1) : make_rsrc(p.x0, p.xbytes0), rw = make_rsrc(p.xw, p.xbytes_w);
    const unsigned row = (unsigned)(second ? p.xc1 : p.xc0) * ES, sc = (unsigned)(second ? cc - p.xc0 : cc) * ES;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        xb[j][h] = buffer_load16<V>(rw, weight_at(n0 + 16 * j + r16, (unsigned)xk * ES, p.xw_row) + kg * 16 + h * 64, (unsigned)e * p.w_kt);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + 16 * i + r16;
      const unsigned o = m < p.M ? (unsigned)m * row + kg * 16 : kOob;
#pragma unroll
      for (int h = 0; h < 2; ++h) xa[i][h] = buffer_load16<V>(rx, o + h * 64, sc);
    }
  };
  if constexpr (XTRA && !GN)
    if (x_first < x_tiles) fetch_extra(x_first);

  // what the epilogue adds.  A thread of it finishes four consecutive columns of a row, or, for transposed outputs, four
  // consecutive rows of a column
  int which = 0, c3 = p.N;
  if constexpr (MODE == OUT_QKV) { c3 = p.N / 3; which = n0 / c3; }          // a tile never straddles two thirds
  const bool by_column = TRANSPOSED || (MODE == OUT_QKV && which == 2 && p.ld_t > 0);
  constexpr int BO = MODE == OUT_GEGLU ? BN / 2 : BN;    // output columns of the tile
  constexpr int QUADS = BM * BO / 4;
  static_assert(QUADS <= 64 * NW, "one item per thread");
  const int rl = by_column ? (tid % (BM / 4)) * 4 : tid / (BO / 4), cl = by_column ? tid / (BM / 4) : (tid % (BO / 4)) * 4;
  const int row = m0 + rl, col = n0 + cl;
  const bool live = tid < QUADS && row < p.M && (MODE == OUT_GEGLU || col < p.N);
  float add[4] = {0.f, 0.f, 0.f, 0.f}, gate[4] = {0.f, 0.f, 0.f, 0.f}, shortcut[4] = {0.f, 0.f, 0.f, 0.f};
  if (live) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = by_column ? col : col + e, r = min(by_column ? row + e : row, p.M - 1);
      if (c >= p.N) continue;
      if (p.bias) { add[e] = p.bias[c]; if constexpr (MODE == OUT_GEGLU) gate[e] = p.bias[c + 32]; }
      if constexpr (MODE == OUT_ROWMAJOR || TRANSPOSED)
        if (p.rowvec) (XTRA ? shortcut : add)[e] += p.rowvec[(size_t)fast_div((unsigned)r, p.div_hw) * p.rowvec_ld + c];
      if constexpr (MODE == OUT_ROWMAJOR)
        if (p.residual) add[e] += to_f(((const T*)p.residual)[(size_t)row * p.N + c]);
    }
  }

  float mean[TM], rstd[TM];
  if constexpr (LN) {
    ln_stats<T, TPR, LD>(p, tid % TPR, x, ln_rows + tid / TPR, ln_rows + BM + tid / TPR);
#pragma unroll
    for (int i = 0; i < GL; ++i) {
      const int at = 4 * (tid + 512 * i);
      if (at < 2 * p.ctot) *(f32x4*)(ln_chan + at) = chan[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i) { mean[i] = ln_rows[16 * i + r16]; rstd[i] = ln_rows[BM + 16 * i + r16]; }
  }
  // GN: the normalised pixels in LDS, behind the partial sums
  const int g_pitch = gn_pitch(p.ctot * ES);
  char* const act = lds + (XTRA ? 2 : 1) * NW * BM * PITCH * 4;
  unsigned g_at[TM];
  if constexpr (GN) {
    gn_stage<T, HOLD>(p, held, g_gain, g_offset, g_first, g_pixels, g_px, g_channel, g_lo, g_hi, act);
    if constexpr (XTRA)
      if (x_first < x_tiles) fetch_extra(x_first);
#pragma unroll
    for (int i = 0; i < TM; ++i) {                       // pixel of tap (0, 0), modulo 2^32 where it lies before the staged ones (the tap is masked then)
      const int m = m0 + 16 * i + r16;
      g_at[i] = 256u + (unsigned)(m - (p.ws + 1) - g_lo) * (unsigned)g_pitch + kg * 16;
    }
  }
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // fp32: every SUM_TILES k-tiles the sum goes to another one, so that no chain of additions is longer than 32 * SUM_TILES.  Error against 64 bits, 2-norm
  // (register-staged tiles with K split / one chain a wavefront / this): 18x256x2304 2.96e-7 / 3.13e-7 / 2.10e-7, 18x256x4608 3.17e-7 / 4.35e-7 / 2.12e-7,
  // 45x64x4800 3.36e-7 / 4.42e-7 / 2.12e-7; narrow fp32 runs level (11.88 ms, 11.91 without).
  constexpr bool BY_PARTS = sizeof(T) == 4;
  constexpr int SUM_TILES = 4;
  static_assert(SUM_TILES % PF == 0, "a part ends between two rounds of the loop");
  f32x4 parts[BY_PARTS ? TM : 1][BY_PARTS ? TN : 1];
  auto end_part = [&]() {
    if constexpr (BY_PARTS)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) { parts[i][j] += acc[i][j]; acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  };
  if constexpr (BY_PARTS)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) parts[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < mine; i0 += PF) {
    if (BY_PARTS && i0 % SUM_TILES == 0) end_part();
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      if (i0 + s >= mine) break;
      if constexpr (GN) {
        const int u = f_tap / 3, v = f_tap - 3 * u;
        const unsigned bit = 1u << f_tap, tap = (unsigned)(u * p.ws + v) * (unsigned)g_pitch + (unsigned)(f_cc * ES);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const unsigned o = (a_taps[i] & bit) ? g_at[i] + tap : 0u;
#pragma unroll
          for (int h = 0; h < 2; ++h) af[0][i][h] = *(const V*)(act + o + h * 64);
        }
        f_cc += BK * NW;
        while (f_cc >= p.ctot) { f_cc -= p.ctot; ++f_tap; }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          V a = af[GN ? 0 : s][i][h];
          if constexpr (LN) {
            const float* ch = ln_chan + ((i0 + s) * NW + wave) * BK + (h * 64 + kg * 16) / ES;
#pragma unroll
            for (int q = 0; q < VN; q += 4) {
              const f32x4 gain = *(const f32x4*)(ch + q), offset = *(const f32x4*)(ch + p.ctot + q);
#pragma unroll
              for (int e = 0; e < 4; ++e) a[q + e] = from_f<T>(ln_value(to_f(a[q + e]), mean[i], rstd[i], gain[e], offset[e]));
            }
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) Mma16<T>::run(bf[s][j][h], a, acc[i][j]);
        }
      if (i0 + s + PF < mine) fetch(s);
    }
  }
  // the sum of these k-tiles, to LDS as wavefront w's; lane: row r16 of row tile i, columns 4 kg .. 4 kg + 3 of column tile j
  auto hand_over = [&](float* sums, int w) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (BY_PARTS) acc[i][j] += parts[i][j];
        *(f32x4*)(sums + w * (BM * PITCH) + (16 * i + r16) * PITCH + 16 * j + 4 * kg) = acc[i][j];
      }
  };
  hand_over(part, wave);
  float* const part_x = part + NW * BM * PITCH;
  if constexpr (XTRA) {
    // the shortcut's sum by itself, as by a launch of its own: k-tiles x, x + NW, ... are wavefront x's there
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (BY_PARTS) parts[i][j] = acc[i][j];
      }
    for (int e = x_first; e < x_tiles; e += NW) {
      if (e > x_first) fetch_extra(e);
      if (BY_PARTS && (e / NW) % SUM_TILES == 0) end_part();
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) Mma16<T>::run(xb[j][h], xa[i][h], acc[i][j]);
    }
    hand_over(part_x, x_first);
  }
  __syncthreads();
  if (!live) return;
  auto total = [&](const float* sums, int r, int c) {    // four columns of a row, over the wavefronts in order
    f32x4 v = *(const f32x4*)(sums + r * PITCH + c);
#pragma unroll
    for (int w = 1; w < NW; ++w) v += *(const f32x4*)(sums + w * (BM * PITCH) + r * PITCH + c);
    return v;
  };
  if (by_column) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = part[(rl + e) * PITCH + cl];
#pragma unroll
      for (int w = 1; w < NW; ++w) v[e] += part[w * (BM * PITCH) + (rl + e) * PITCH + cl];
      v[e] += add[e];
    }
    const int ncols = MODE == OUT_QKV ? c3 : p.N, cc = MODE == OUT_QKV ? col - 2 * c3 : col;
    void* const dst = MODE == OUT_QKV ? p.out3 : p.out;
    const int b = (int)fast_div((unsigned)row, p.div_hw);
    const size_t o = ((size_t)b * ncols + cc) * p.ld_t + (row - b * p.hw_out);
    if ((p.hw_out & 3) == 0 && (p.ld_t & 3) == 0 && row + 3 < p.M) {
      if constexpr (MODE == OUT_TRANSPOSED_F32) *(f32x4*)((float*)dst + o) = f32x4{v[0], v[1], v[2], v[3]};
      else *(V4*)((T*)dst + o) = V4{from_f<T>(v[0]), from_f<T>(v[1]), from_f<T>(v[2]), from_f<T>(v[3])};
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (row + e >= p.M) break;
      const int be = (int)fast_div((unsigned)(row + e), p.div_hw);
      const size_t oe = ((size_t)be * ncols + cc) * p.ld_t + (row + e - be * p.hw_out);
      if constexpr (MODE == OUT_TRANSPOSED_F32) ((float*)dst)[oe] = v[e];
      else ((T*)dst)[oe] = from_f<T>(v[e]);
    }
    return;
  }
  f32x4 v = total(part, rl, cl);
  int ncols = p.N, c_out = col;
  T* dst = (T*)p.out;
  if constexpr (MODE == OUT_GEGLU) {
    const f32x4 g = total(part, rl, cl + 32);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (v[e] + add[e]) * gelu_f(g[e] + gate[e]);
    ncols = p.N >> 1; c_out = (n0 >> 1) + cl;
  } else {
    if constexpr (XTRA) {
      const f32x4 x = total(part_x, rl, cl);
#pragma unroll
      for (int e = 0; e < 4; ++e) add[e] += to_f(from_f<T>(x[e] + shortcut[e]));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += add[e];
  }
  if constexpr (MODE == OUT_QKV) {
    dst = (T*)(which == 0 ? p.out : which == 1 ? p.out2 : p.out3);
    ncols = c3; c_out = col - which * c3;
  }
  const size_t o = (size_t)row * ncols + c_out;
  if ((ncols & 3) == 0) {
    *(V4*)(dst + o) = V4{from_f<T>(v[0]), from_f<T>(v[1]), from_f<T>(v[2]), from_f<T>(v[3])};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c_out + e < ncols) dst[o + e] = from_f<T>(v[e]);
  }
}

// samples that the rows of a tile belong to at the most
static int gn_samples(int bm, int batch, int hw) { return std::min(batch, hw % bm == 0 ? 1 : (bm - 2) / hw + 2); }
// How a workgroup of bm rows holds them: every sample from lane 0 on, since k_gn_group adds its pixels up by their place in it, or several samples of a power of two of
// pixels in an access; slots 0 where that does not fit.  A wavefront takes an eighth of the channels: whole groups, whole accesses, powers of two.
static GnLayout gn_layout(int vn, int bm, int batch, int hw, int c, int groups) {
  GnLayout g{};
  if (groups < 8 || groups % 8 || c % (2 * groups) || c % (8 * vn)) return g;
  const int cpg = c / groups, vps = c / (8 * vn), hold = gn_hold(vn);
  if ((vps & (vps - 1)) || vps > 16 || (cpg & (cpg - 1)) || cpg > 4 * vn) return g;
  while (1 << g.log_vps < vps) ++g.log_vps;
  g.vpp = std::max(1, cpg / vn);
  g.per_access = std::max(1, vn / cpg);
  g.run = vps / g.vpp;
  if (g.run > 8) return g;
  const int step = 64 / vps, all = gn_samples(bm, batch, hw) * hw;
  g.pixels = hw < step && (hw & (hw - 1)) == 0 ? step : hw;
  while (1 << g.bits < std::min(hw, step)) ++g.bits;
  const int accesses = (g.pixels + step - 1) / step, blocks = (all + g.pixels - 1) / g.pixels;
  g.chained = accesses > 4 * g.run;
  if (g.chained && g.per_access > 1) return g;
  for (int slots : {hold / 5, hold / 2, hold})
    if (accesses <= slots && blocks * slots <= hold) { g.slots = slots; break; }
  return g;
}
template <typename T, int TM, int TN, int MODE, int NORM = NORM_NONE, bool XTRA = false>
static ad_status run_igemm_small(const IgemmParams& p0, const char* name, hipStream_t s) {
  constexpr bool LN = NORM == NORM_LAYER;
  if constexpr (!XTRA && MODE == OUT_ROWMAJOR && !LN)
    if (p0.xw) return run_igemm_small<T, TM, TN, MODE, NORM, true>(p0, name, s);
  if constexpr (NORM == NORM_NONE && (MODE == OUT_ROWMAJOR || MODE == OUT_TRANSPOSED_F32))
    if (p0.gn_groups) return run_igemm_small<T, TM, TN, MODE, NORM_GROUP, XTRA>(p0, name, s);
  if constexpr (NORM == NORM_NONE && !XTRA && (MODE == OUT_ROWMAJOR || MODE == OUT_QKV || MODE == OUT_GEGLU))
    if (p0.ln_gain && !p0.gn_groups) return run_igemm_small<T, TM, TN, MODE, NORM_LAYER>(p0, name, s);
  IgemmParams p = p0;
  set_tiles(p, 16 * TM, 16 * TN);
  constexpr int lds_sums = small_sum_bytes(16 * TM, 16 * TN) * (XTRA ? 2 : 1);
  constexpr int lds_most = NORM == NORM_GROUP ? (int)kLdsLimit : lds_sums + (LN ? 2 * 16 * TM * 4 + small_ktiles(16 * TM, 16 * TN) * kRowBytes / (int)sizeof(T) * 8 : 0);
  const int lds_bytes = lds_sums + (LN ? 2 * 16 * TM * 4 + p.ctot * 8 : NORM == NORM_GROUP ? gn_act_bytes(16 * TM, p.ws, p.ctot * (int)sizeof(T)) : 0);
  if constexpr (lds_most > 65536) {
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
      AD_HIP(hipFuncSetAttribute((const void*)k_igemm_small<T, TM, TN, MODE, NORM, XTRA>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_most));
      attr_set = true;
    }
  }
  const double in_bytes = (double)p.M * p.ctot * sizeof(T) * (p.stride == 2 ? 4 : 1) / (p.up ? 4 : 1);
  const double out_cols = p.out_mode == OUT_GEGLU ? p.N / 2 : p.N;
  const int xk = p.xc0 + p.xc1;
  ProfLaunch pl(name, 2.0 * p.M * p.N * (p.k_prof + xk), in_bytes + ((double)p.N * (p.Kp + xk) + (double)p.M * xk) * sizeof(T) + (double)p.M * out_cols * sizeof(T), s, p.M, p.N, p.Kp + xk);
  hipLaunchKernelGGL((k_igemm_small<T, TM, TN, MODE, NORM, XTRA>), dim3(p.tiles_n * p.tiles_m), dim3(512), lds_bytes, s, p);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// =================================================================================================
// 3x3 convolution (stride 1) with the input staged in LDS as a halo tile, bf16.
//
// The implicit-GEMM kernels above fetch the A tile (BM output positions x 64 channels) once per tap: nine times the
// same pixels, shifted, through the L2 -> LDS path that already limits them.  Here a workgroup stages, per chunk of
// 64 input channels, every input pixel its BM output positions touch - the BM positions themselves plus one image
// row and one pixel on either side, (BM + 2 W + 2) rows of 128 bytes - once, and runs the nine taps out of that
// tile: tap (dy, dx) of output position m reads LDS row m - m0 + (W + 1) + dy W + dx.  Positions are linear over
// the whole batch, so a tile may straddle image rows and samples; what a shifted index would pick up from the
// neighbouring row or sample (or from beyond the tensor) is replaced by zeros by pointing the lane's fragment
// address at a 128-byte zero block - one select per (lane, row block, tap), no work per element.  With a nearest-2x
// upsampled input the staged pixels are the stored (half-resolution) ones and the row is computed from
// ((y + dy) >> 1, (x + dx) >> 1).  Weights: one 128 x 64 tile per (tap, chunk) through a ring of NB stages.
// The halo tile is double-buffered; the next chunk's tile is requested in eight slices, one per tap.
// LDS traffic from L2 per k-tile: 16 KiB of weights + a ninth of the halo (about 6.4 KiB for BM = 256, W = 96)
// instead of 16 + 32 KiB.
// =================================================================================================
struct HaloParams {
  int hr;            // rows of the halo tile: BM + 2 Ws + 2 (+ slack of the upsampled mapping), rounded up to 32
  int chunk_begin_stride;   // chunks per split (split-K over channel chunks), or all of them
  FastDiv div_hw, div_w;    // output position -> (sample, y, x)
};

template <int BM, int NB, int MODE>
__global__ __launch_bounds__(256) void k_conv3_halo(IgemmParams p, HaloParams hp) {
  typedef bf16 T;
  typedef bf16x8 V;
  constexpr int BN = 128, WTM = BM / 2, WTN = BN / 2, TM = WTM / 32, TN = WTN / 32;
  constexpr int BSTAGE = BN * kRowBytes, BG = BN / 32;          // weight tile, loads per wavefront and tile
  constexpr int ASL = BM / 128;                                 // halo loads per wavefront and tap slice (8 slices cover the tile)
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wave_m = wave >> 1, wave_n = wave & 1;
  const TileId tid3 = tile_of(p);
  const int m0 = tid3.m_tile * BM, n0 = tid3.n_tile * BN;
  const u32x4 rs0 = make_rsrc_words(p.src0, p.bytes0), rs1 = make_rsrc_words(p.src1, p.bytes1);
  const u32x4 rsw = make_rsrc_words(p.w, p.bytes_w);
  // LDS: [halo 0][halo 1][weights x NB][zero block]
  const int abytes = hp.hr * kRowBytes;
  char* const bbase = lds + 2 * abytes;
  char* const zero = bbase + NB * BSTAGE;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds;
  if (tid < 8) *(V*)(zero + tid * 16) = V{};
  const int nchunks = p.ctot / 64;
  const int c_begin = tid3.split * hp.chunk_begin_stride;
  const int c_end = min(nchunks, c_begin + hp.chunk_begin_stride);
  const int nkt = (c_end - c_begin) * 9;
  const int up = p.up, Ws = p.ws, W = p.win, H = p.hin;        // stored width, logical (convolved) size

  // ---- which stored pixel heads the halo tile: the one tap (-1, -1) of the tile's first output position maps to
  //      (clamped into the sample; everything before it in the same sample is not needed), minus nothing.
  //      Stored linear index of logical (b, yy, xx): b Hs Ws + (yy >> up) Ws + (xx >> up).
  int g_base;
  {
    const int b = (int)fast_div((unsigned)m0, hp.div_hw), r = m0 - b * p.hw_out;
    const int y = (int)fast_div((unsigned)r, hp.div_w), x = r - y * W;
    // plain input: tap (-1, -1) of the first position, m0 - W - 1 (no later position reaches further back).  Upsampled input:
    // later positions of the tile may sit in the next logical row, which shares the stored row, at smaller x: start one
    // pixel before the stored row of (y - 1) >> 1 (arithmetic shift: row -1 of the sample for y = 0)
    g_base = b * p.hs * Ws + (up ? ((y - 1) >> 1) * Ws - 1 : (y - 1) * Ws + x - 1);
  }
  const int total_pix = p.M / p.hw_out * p.hs * Ws;                        // stored pixels of a source
  // ---- loads: halo row group G = wave + 4 j covers rows 8 G .. 8 G + 7; this lane's row r8, chunk position lane & 7
  const int r8 = lane >> 3;
  const int scol = (lane & 7) ^ lds_swizzle(wave * 8 + r8);
  const int na = hp.hr / 32;                                               // loads per wavefront and halo tile
  auto issue_halo = [&](int chunk, int buf, int j0, int j1) {
    const bool second = chunk * 64 >= p.c0;
    u32x4 rs = second ? rs1 : rs0;
#pragma unroll
    for (int e = 0; e < 4; ++e) rs[e] = __builtin_amdgcn_readfirstlane(rs[e]);      // workgroup-uniform by construction
    const unsigned cs = (unsigned)(second ? p.c1 : p.c0) * 2u;             // bytes per pixel of that source
    const unsigned soff = __builtin_amdgcn_readfirstlane((unsigned)((second ? chunk * 64 - p.c0 : chunk * 64) * 2));
    for (int j = j0; j < j1 && j < na; ++j) {
      const int g = g_base + (wave + 4 * j) * 8 + r8;
      const unsigned vo = (g >= 0 && g < total_pix) ? (unsigned)g * cs + (unsigned)scol * 16u : kOob;
      dma_load16(rs, vo, soff, __builtin_amdgcn_readfirstlane(lds_base + buf * abytes + (wave + 4 * j) * 1024));
    }
  };
  unsigned b_off[BG];
#pragma unroll
  for (int i = 0; i < BG; ++i) b_off[i] = weight_at(n0 + (4 * i + wave) * 8 + r8, (unsigned)p.Kp * 2, p.w_row) + scol * 16;
  auto issue_b = [&](int chunk, int tap, int stage) {
    const unsigned soff = __builtin_amdgcn_readfirstlane((unsigned)(tap * nchunks + chunk) * p.w_kt);
#pragma unroll
    for (int i = 0; i < BG; ++i)
      dma_load16(rsw, b_off[i], soff, __builtin_amdgcn_readfirstlane(lds_base + 2 * abytes + stage * BSTAGE + (4 * i + wave) * 1024));
  };

  // ---- this lane's output positions (one per 32-row block of the wavefront's tile): sample base, y, x
  int pb_[TM], py[TM], px[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wave_m * WTM + i * 32 + l32;
    if (m < p.M) {
      const int b = (int)fast_div((unsigned)m, hp.div_hw), r = m - b * p.hw_out;
      py[i] = (int)fast_div((unsigned)r, hp.div_w);
      px[i] = r - py[i] * W;
      pb_[i] = b * p.hs * Ws - g_base;
    } else {
      py[i] = -4; px[i] = -4; pb_[i] = 0;          // every tap is out of the image
    }
  }
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // prologue: the first halo tile, then the first NB - 1 weight tiles
  if (nkt > 0) issue_halo(c_begin, 0, 0, na);
#pragma unroll
  for (int t = 0; t < NB - 1; ++t)
    if (t < nkt) issue_b(c_begin + t / 9, t % 9, t);

  const int b_row = (wave_n * WTN + l32) * kRowBytes;
  const int x7 = lds_swizzle(l32);
  const char* const zero_rd = zero + half * 16;
  int kt = 0, bstage = 0;
  for (int chunk = c_begin; chunk < c_end; ++chunk) {
    const int abuf = (chunk - c_begin) & 1;
    const char* const As = lds + abuf * abytes;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap, ++kt) {
      // weight tile kt has landed once at most the NB - 2 tiles requested after it are outstanding; the halo slice
      // requested one tap ago is older than those and is waited for with it
      if (NB == 3 && kt + 1 < nkt) wait_vmcnt<BG>(); else wait_vmcnt<0>();
      __syncthreads();       // tile kt (and at tap 0 the chunk's halo) is complete for everybody; everybody is done with tile kt - 1
      if (tap < 8 && chunk + 1 < c_end) issue_halo(chunk + 1, abuf ^ 1, tap * ASL * 2, (tap + 1) * ASL * 2);
      if (kt + NB - 1 < nkt) {
        const int t2 = kt + NB - 1;
        int st = bstage + NB - 1;
        if (st >= NB) st -= NB;
        issue_b(c_begin + t2 / 9, t2 % 9, st);
      }
      // fragment addresses of this tap: halo row of (y + dy, x + dx), or the zero block
      const int dy = tap / 3 - 1, dx = tap % 3 - 1;
      const char* a_rd[TM];
      int a_sw[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int yy = py[i] + dy, xx = px[i] + dx;
        const bool ok = yy >= 0 && yy < H && xx >= 0 && xx < W;
        const int row = pb_[i] + (yy >> up) * Ws + (xx >> up);
        a_rd[i] = ok ? As + row * kRowBytes + ((half ^ (lds_swizzle(row) & 1)) << 4) : zero_rd;
        a_sw[i] = ok ? (lds_swizzle(row) & 6) : 0;
      }
      const char* const Bs = bbase + bstage * BSTAGE + b_row;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        V af[TM], bf[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = *(const V*)(a_rd[i] + (((2 * ks) ^ a_sw[i]) << 4));
#pragma unroll
        for (int j = 0; j < TN; ++j) bf[j] = *(const V*)(Bs + j * 32 * kRowBytes + (((ks * 2 + half) ^ x7) << 4));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
      }
      if (++bstage == NB) bstage = 0;
    }
  }
  wait_vmcnt<0>();
  __syncthreads();     // every wavefront is done reading the tiles: LDS can be reused by the epilogue
  typename Vec<T>::type res[RowSlabs<T, WTM, WTN>::COUNT][RowSlabs<T, WTM, WTN>::MAX];
  igemm_epilogue<T, WTM, WTN, TM, TN, MODE, 16, false>(p, acc, m0, n0, wave_m, wave_n, l32, half, lds + wave * stage_bytes<T, WTM, WTN>(16), tid3.split, res);
}

// Rows of the halo tile for a BM-position tile: the stored pixels between the one tap (-1, -1) of the first position
// maps to and the one tap (+1, +1) of the last position maps to, at most; rounded up to whole 32-row load rounds.
static int halo_rows(int bm, int ws, int up) {
  if (!up) return round_up(bm + 2 * ws + 2, 32);
  // upsampled: bm consecutive logical positions touch at most d + 1 logical rows, d = (bm + W - 2) / W, hence with the
  // taps logical rows l0 - 1 .. l0 + d + 1, whose stored rows (l >> 1) number at most (d + 3) / 2 + 1; plus the pixel before
  const int w = 2 * ws, d = (bm + w - 2) / w;
  return round_up(((d + 3) / 2 + 1) * ws + 1, 32);
}
static size_t halo_lds_bytes(int bm, int nb, int ws, int up) {
  return (size_t)2 * halo_rows(bm, ws, up) * kRowBytes + (size_t)nb * 128 * kRowBytes + 128;
}

template <int BM, int NB, int MODE>
static ad_status run_conv3_halo(const IgemmParams& p0, int splits, const char* name, hipStream_t s) {
  IgemmParams p = p0;
  set_tiles(p, BM, 128);
  HaloParams hp;
  hp.hr = halo_rows(BM, p.ws, p.up);
  const int nchunks = p.ctot / 64;
  hp.chunk_begin_stride = splits > 1 ? (nchunks + splits - 1) / splits : nchunks;
  hp.div_hw = p.div_hw; hp.div_w = p.div_w;
  const int real_splits = (nchunks + hp.chunk_begin_stride - 1) / hp.chunk_begin_stride;
  const size_t lds_bytes = std::max(halo_lds_bytes(BM, NB, p.ws, p.up), (size_t)4 * (BM / 2) * kPitch);
  if (lds_bytes > kLdsLimit || hp.hr / 32 > 16 * (BM / 128)) AD_FAIL(AD_ERR_INVALID, "conv (halo): tile does not fit");
  static std::atomic<bool> attr_set{false};
  if (!attr_set) {
    AD_HIP(hipFuncSetAttribute((const void*)k_conv3_halo<BM, NB, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit));
    attr_set = true;
  }
  const double in_bytes = (double)p.M * p.ctot * 2 / (p.up ? 4 : 1);
  ProfLaunch pl(name, 2.0 * p.M * p.N * p.k_prof, in_bytes + (double)p.N * p.Kp * 2 + (double)p.M * p.N * 2, s, p.M, p.N, p.Kp);
  hipLaunchKernelGGL((k_conv3_halo<BM, NB, MODE>), dim3(p.tiles_n * p.tiles_m, real_splits), dim3(256), lds_bytes, s, p, hp);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

template <typename T, int BM, int BN, int WGM, int WGN, int NSET, int MODE>
static ad_status run_igemm(const IgemmParams& p0, const char* name, hipStream_t s) {
  IgemmParams p = p0;
  set_tiles(p, BM, BN);
  constexpr int lds_bytes = 2 * (BM + BN) * kPitch;
  static std::atomic<bool> attr_set{false};     // LDS above 64 KiB has to be requested once per kernel
  if (!attr_set) {
    AD_HIP(hipFuncSetAttribute((const void*)k_igemm<T, BM, BN, WGM, WGN, NSET, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
    attr_set = true;
  }
  const double in_bytes = (double)p.M * p.ctot * sizeof(T) * (p.stride == 2 ? 4 : 1) / (p.up ? 4 : 1);
  const double out_cols = p.out_mode == OUT_GEGLU ? p.N / 2 : p.N;
  ProfLaunch pl(name, 2.0 * p.M * p.N * p.k_prof, in_bytes + (double)p.N * p.Kp * sizeof(T) + (double)p.M * out_cols * sizeof(T), s, p.M, p.N, p.Kp);
  const int splits = (p.ktiles + p.kt_per_split - 1) / p.kt_per_split;
  hipLaunchKernelGGL((k_igemm<T, BM, BN, WGM, WGN, NSET, MODE>), dim3(p.tiles_n * p.tiles_m, splits), dim3(256), lds_bytes, s, p);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// Split-K second pass: sums the fp32 partials in a fixed order and applies the epilogue.
template <typename T>
__global__ __launch_bounds__(256) void k_splitk_reduce(const float* __restrict__ partial, int splits, int M, int N, int hw_out, FastDiv div_n4,
                                                       FastDiv div_hw, int vec, const float* __restrict__ bias,
                                                       const float* __restrict__ rowvec, int rowvec_ld, const T* __restrict__ residual,
                                                       void* __restrict__ out, void* __restrict__ out2, void* __restrict__ out3, int out_mode, int ld_t) {
  typedef typename Vec4<T>::type V4;
  const unsigned n4 = N / 4, total = (unsigned)M * n4;
  for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int row = (int)fast_div(i, div_n4), col = (int)(i - (unsigned)row * n4) * 4, b = (int)fast_div((unsigned)row, div_hw);
    // added in order, eight loads in flight (one at a time, each split costs a round trip to memory: 6.6 us a launch); what is added
    // behind them is requested with them
    const float* src = partial + (size_t)row * N + col;
    const size_t step = (size_t)M * N;
    float add[4] = {0.f, 0.f, 0.f, 0.f}, per[4] = {0.f, 0.f, 0.f, 0.f};
    V4 res = V4{};
    const bool with_res = out_mode == OUT_ROWMAJOR && residual;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (bias) add[e] = bias[col + e];
      if (rowvec) per[e] = rowvec[(size_t)b * rowvec_ld + col + e];
    }
    if (with_res) {
      if (vec) res = *(const V4*)(residual + (size_t)row * N + col);
      else
#pragma unroll
        for (int e = 0; e < 4; ++e) res[e] = residual[(size_t)row * N + col + e];
    }
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < splits; z += 8) {
      f32x4 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (z + u < splits) t[u] = *(const f32x4*)(src + (z + u) * step);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (z + u < splits) v += t[u];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (bias) v[e] += add[e];
      if (rowvec) v[e] += per[e];
      if (with_res) v[e] += to_f(res[e]);
    }
    // four columns of a row (never of two thirds where vec is set), or one at a time
    const int c3 = out_mode == OUT_QKV ? N / 3 : N, which = out_mode == OUT_QKV ? col / c3 : 0;
    const bool turned = out_mode == OUT_TRANSPOSED || out_mode == OUT_TRANSPOSED_F32 || (which == 2 && ld_t > 0);
    if (vec && !turned) {
      T* dst = (T*)(which == 0 ? out : which == 1 ? out2 : out3);
      *(V4*)(dst + (size_t)row * c3 + col - which * c3) = V4{from_f<T>(v[0]), from_f<T>(v[1]), from_f<T>(v[2]), from_f<T>(v[3])};
      continue;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = v[e];
      if (out_mode == OUT_ROWMAJOR) {
        ((T*)out)[(size_t)row * N + col + e] = from_f<T>(x);
      } else if (out_mode == OUT_QKV) {
        const int w = (col + e) / c3, cc = col + e - w * c3;
        if (w == 0) ((T*)out)[(size_t)row * c3 + cc] = from_f<T>(x);
        else if (w == 1) ((T*)out2)[(size_t)row * c3 + cc] = from_f<T>(x);
        else if (ld_t > 0) ((T*)out3)[((size_t)b * c3 + cc) * ld_t + (row - b * hw_out)] = from_f<T>(x);
        else ((T*)out3)[(size_t)row * c3 + cc] = from_f<T>(x);
      } else {
        const size_t o = ((size_t)b * N + col + e) * ld_t + (row - b * hw_out);
        if (out_mode == OUT_TRANSPOSED) ((T*)out)[o] = from_f<T>(x);
        else ((float*)out)[o] = x;
      }
    }
  }
}

// Tile shapes.  The register-staged kernels (64x64, 128x128) serve fp32 and the transposed epilogues; bf16 GEMMs with a row-major,
// GEGLU, fused q/k/v or split-K epilogue take the LDS-DMA kernel with a tile of kDmaTiles; launches of few small tiles k_igemm_small.
enum { TILE_128x128 = 1, TILE_64x64 = 3, TILE_D2_128 = 4, TILE_P3_128 = 5, TILE_P3_256 = 6, TILE_P3_64 = 7, TILE_HALO_128 = 8, TILE_HALO_256 = 9, TILE_P3_256_W4 = 10, TILE_P3_128_W4 = 11, TILE_P3_256_W16 = 12, TILE_SMALL = 13, TILE_D2_160 = 14, TILE_D2_320 = 15, TILE_K2_64 = 16, TILE_AUTO = -1 };
static int g_tile_override = TILE_AUTO;
static int g_order_override = -1;

struct ConvPlan { int tile, splits, band; };      // band: of tile_of(), -1 = the launcher decides between one row tile and all

static bool dma_capable(int dtype, int out_mode) {
  return dtype == AD_BF16 && (out_mode == OUT_ROWMAJOR || out_mode == OUT_GEGLU || out_mode == OUT_QKV);
}

// Split-K for the register-staged kernels: GEMMs with few output tiles and a long K are cut along K so that a
// few hundred workgroups exist.
static int splits_by_tiles(long long m, int n, int ktiles, int out_mode, int bm) {
  if (out_mode == OUT_GEGLU || n % 4) return 1;
  const long long tiles = ((m + bm - 1) / bm) * ((n + bm - 1) / bm);
  if (tiles >= 400 || ktiles < 16) return 1;
  int splits = (int)((1024 + tiles - 1) / tiles);
  if (splits > ktiles / 8) splits = ktiles / 8;
  if (splits > 16) splits = 16;
  if (splits < 2) return 1;
  const int per = (ktiles + splits - 1) / splits;
  return (ktiles + per - 1) / per;
}

// The LDS-DMA kernels and what a workgroup of theirs takes, in us: `fixed` for prologue, epilogue and launch, and per k-tile with 1, 2
// or 3 of them resident on a CU (measured over the GEMM shapes of the SD-sized models, operands from beyond the L2).  Wide tiles
// take the fewest bytes per multiply-add (256x320: 28 bytes a clock and CU at full matrix rate, 128x128: 64, of the 60 or so a CU gets
// from its L2), two resident workgroups hide each other's prologue and epilogue, small tiles fill the chip when there are few rows.
struct DmaTile { int tile, bm, bn, per_cu; double fixed, per_kt[3]; };
static const DmaTile kDmaTiles[] = {
    {TILE_P3_64, 64, 64, 3, 4.0, {0.32, 0.40, 0.62}},   {TILE_K2_64, 64, 64, 1, 4.6, {0.22, 0.22, 0.22}},   {TILE_D2_128, 128, 128, 2, 5.0, {0.90, 0.98, 0.98}},
    {TILE_P3_128, 128, 128, 1, 4.0, {0.50, 0.50, 0.50}}, {TILE_D2_160, 128, 160, 2, 7.0, {1.05, 1.25, 1.25}},
    {TILE_P3_256, 256, 128, 1, 5.0, {0.80, 0.80, 0.80}}, {TILE_D2_320, 256, 320, 1, 12.0, {2.00, 2.00, 2.00}},
};
// Time of a launch, in us.  Rounds of resident workgroups; of the part of the chip that the last round leaves idle kTail is
// charged, since other streams use the rest.  GEGLU: 1.4 us of vector work per 128x128 tile, which a second resident workgroup
// covers half of.  Split-K: a second launch that reads the partial sums.
constexpr double kTail = 0.7;
static double plan_cost(long long m, int n, int ktiles, int out_mode, const DmaTile& t, int splits) {
  const long long wgs = ((m + t.bm - 1) / t.bm) * ((n + t.bn - 1) / t.bn) * splits;
  const int resident = (int)std::min<long long>(t.per_cu, (wgs + 255) / 256);
  const int per = (ktiles + splits - 1) / splits;
  const double gelu = out_mode == OUT_GEGLU ? 1.4 * t.bm * t.bn / 16384.0 : 0.0;
  const double round = t.fixed + per * t.per_kt[resident - 1] + gelu;
  const double full = (double)wgs / (256 * resident), rounds = std::ceil(full);
  double cost = round * (kTail * rounds + (1.0 - kTail) * full);
  if (splits > 1) cost += 4.0 + 2.0 * splits * (double)m * n * 4.0 / 5e6;
  return cost;
}

// Row tiles per band (tile_of): the workgroups of an XCD that run side by side, at most 32 CUs full, should take in the fewest rows
// and columns per k-tile.  Weights from memory, launches back to back, us (bands of one row tile / one band / this): 2048x1280x5120 50.0 / 49.7 / 48.3,
// 4608x5120x640 45.0 / 46.3 / 41.8, 4928x5120x1280 92.8 / 91.1 / 84.4, 720x640x2560 12.3 / 12.4 / 11.5, 8192x640x2560 30.9 / 37.6 / 30.9; slower than one of the
// two: 2048x640x2560 15.9 / 20.3 / 18.1, 880x1280x1280 9.9 / 10.0 / 10.8 (their runs straddle two bands).  Inside the models, behind a kernel that leaves its rows
// in the L2 of the XCD that owns them, those two are level (22.7 against 23.1) and bands of many rows lose: 1152x1280x1280 15.4 / 16.8 / 15.3.
// A launch of several rounds without K-splits: no bands that leave fewer than four places where the XCDs begin in them, since XCDs that walk the same
// columns at the same time wait for the same memory: 16384x5120x640 113.3 / 125.0 / 110.8 (bands of eight, all XCDs at the first column: 123.1),
// 8192x5120x640 58.8 / 66.0 / 57.4 (eight, two places: 61.1), 4096x3840x1280 45.4 / 47.9 / 42.4 (46.7), 65536x2560x320 179 / 189 / 173 (175).
static int best_band(long long m, int n, const DmaTile& t, int splits) {
  const long long tm = (m + t.bm - 1) / t.bm, tn = (n + t.bn - 1) / t.bn, wgs = tm * tn * splits;
  const long long resident = std::min<long long>(t.per_cu, (wgs + 255) / 256);
  const long long run = std::min({(wgs + 7) / 8, 32 * resident, tm * tn});
  long long best = 1, best_rows = -1;
  for (long long band = 1; band <= std::min(tm, run); ++band) {
    const long long tiles = band * tn;                       // of a band; a run is part of one or several whole ones
    if (band > 1 && splits == 1 && wgs / 8 > run && tiles / std::gcd(wgs / 8, tiles) < 4) continue;
    const long long rows = tiles >= run ? band : std::min(tm, band * ((run + tiles - 1) / tiles)), cols = tiles >= run ? (run + band - 1) / band : tn;
    const long long taken = rows * t.bm + cols * t.bn;
    if (best_rows < 0 || taken < best_rows) { best_rows = taken; best = band; }
  }
  return (int)best;
}

// Tile of k_igemm_small (16-row and 16-column units), or {0, 0} where another kernel is the better choice: the smallest tile that
// makes at most a workgroup per CU, as long as a workgroup takes in at most 200 KiB (beyond that the 60 GB/s a CU gets from memory
// decide, and K split over workgroups wins: 3x3 72x192x5760 13 us against 11).  GEGLU pairs 32 value with 32 gate columns.
// fp32: at most 600 KiB, since what is left to split K over workgroups are register-staged tiles of 64 or 128 rows on matrix cores of a sixteenth of the rate, which
// multiply mostly padding.  3x3, us (those and their second pass / this): 18x256x2304 27.1 / 11.1, 72x256x2304 27.6 / 11.7 and 18x256x4608 29.5 / 16.6 with the norm inside, 288x256x2304 28.2 / 15.6,
// 512x128x3456 30.4 / 15.4, 1152x128x3456 21.8 / 21.4; linear: 180x1280x1280 18.8 / 14.6.  1200 KiB: 288x256x4608 31.3 / 26.6, but 1152x128x3456
// in tiles of 32x32 21.8 / 27.4.
constexpr int kSmallF32 = 600 * 1024;
struct SmallTile { int tm, tn; };
static SmallTile small_tile(int dtype, long long m, int n, int ktiles, int out_mode) {
  const SmallTile plain[] = {{1, 1}, {1, 2}, {2, 2}}, geglu[] = {{1, 4}, {2, 4}};
  for (int i = 0; i < (out_mode == OUT_GEGLU ? 2 : 3); ++i) {
    const SmallTile t = out_mode == OUT_GEGLU ? geglu[i] : plain[i];
    const long long wgs = ((m + 16 * t.tm - 1) / (16 * t.tm)) * ((n + 16 * t.tn - 1) / (16 * t.tn));
    const int most = dtype == AD_F32 ? kSmallF32 / ((16 * t.tm + 16 * t.tn) * kRowBytes) : small_ktiles(16 * t.tm, 16 * t.tn);
    if (wgs <= 256 && ktiles <= most) return t;
  }
  return SmallTile{0, 0};
}

// Where the tiles whose K two groups of wavefronts share are left out: 40 k-tiles and more a workgroup in a launch of at most
// 48 workgroups, where K split over more of them is faster; 80 and more with weights of 8 MiB and more (0.25 to 0.27 us a k-tile, 0.15 to 0.2 elsewhere) or
// fewer than 200 workgroups.  Weights from memory, us (these tiles / the next best plan), left out: 128x640x2560 11.4 / 8.8, 397x320x2560 11.5 / 9.4,
// 512x1280x5120 26.4 / 21.4, 947x960x5120 25.9 / 23.2, 1026x640x5120 20.5 / 18.7; kept: 720x1280x2560 12.3 / 14.7, 995x320x2560 11.8 / 12.3, 104x960x2304
// 10.1 / 10.9, 1168x512x4608 17.7 / 20.1, 2880x320x5760 20.3 / 23.4.
static bool k2_suits(long long m, int n, int ktiles, int splits, int per) {
  const long long wgs = ((m + 63) / 64) * ((n + 63) / 64) * splits;
  if (per >= 40 && wgs <= 48) return false;
  return per < 80 || (wgs >= 200 && (long long)n * ktiles * kRowBytes < (8 << 20));
}

static ConvPlan compute_plan(int dtype, long long m, int n, int ktiles, int out_mode, int forced) {
  const bool geglu = out_mode == OUT_GEGLU;   // needs a value and a gate tile in the same wavefront
  const bool dma = dma_capable(dtype, out_mode);
  if (forced == TILE_P3_128_W4) forced = TILE_P3_128;     // variants with other wavefront counts: same tiles, same planning
  if (forced == TILE_P3_256_W4 || forced == TILE_P3_256_W16) forced = TILE_P3_256;
  if (forced == TILE_HALO_128) forced = TILE_P3_128;      // the halo kernels share the tile shapes (and the split-K planning) of these
  if (forced == TILE_HALO_256) forced = TILE_P3_256;
  if (forced == TILE_P3_128 || forced == TILE_P3_256 || forced == TILE_D2_128 || forced == TILE_P3_64 || forced == TILE_K2_64 || forced == TILE_D2_160 || forced == TILE_D2_320) {
    if (!dma || ((forced == TILE_P3_64 || forced == TILE_K2_64 || forced == TILE_D2_160) && geglu)) forced = TILE_AUTO;
  }
  else if (forced != TILE_AUTO && geglu) forced = TILE_AUTO;
  if (forced == TILE_128x128 || forced == TILE_64x64) return ConvPlan{forced, splits_by_tiles(m, n, ktiles, out_mode, forced == TILE_64x64 ? 64 : 128), -1};
  if (forced == TILE_AUTO && small_tile(dtype, m, n, ktiles, out_mode).tm) return ConvPlan{TILE_SMALL, 1, -1};
  if (!dma) {
    // measured on the GEMM shapes of the SD-sized models: 128x128 register-staged tiles pay off once there is
    // more than one of them per CU, or with very few rows and a long K (the weights are re-read less often)
    const long long tiles128 = ((m + 127) / 128) * ((n + 127) / 128);
    const int tile = (geglu || tiles128 >= 288 || (m <= 512 && ktiles >= 64)) ? TILE_128x128 : TILE_64x64;
    return ConvPlan{tile, splits_by_tiles(m, n, ktiles, out_mode, tile == TILE_64x64 ? 64 : 128), -1};
  }
  ConvPlan best{TILE_P3_128, 1, -1};
  const DmaTile* chosen = nullptr;
  double best_cost = 1e300;
  const int max_splits = (geglu || n % 4) ? 1 : 16;
  for (const DmaTile& t : kDmaTiles) {
    if (forced != TILE_AUTO && t.tile != forced) continue;
    if (geglu && (t.tile == TILE_P3_64 || t.tile == TILE_K2_64 || t.tile == TILE_D2_160)) continue;      // value and gate columns in one wavefront
    for (int sp = 1; sp <= max_splits; ++sp) {
      if (sp > 1 && ktiles / sp < 4) break;
      const int per = (ktiles + sp - 1) / sp;
      if ((ktiles + per - 1) / per != sp) continue;          // every split must own at least one k-tile
      if (t.tile == TILE_K2_64 && ktiles - (sp - 1) * per < 2) continue;         // so must both groups of wavefronts
      if (t.tile == TILE_K2_64 && forced == TILE_AUTO && !k2_suits(m, n, ktiles, sp, per)) continue;
      const double c = plan_cost(m, n, ktiles, out_mode, t, sp);
      if (c < best_cost) { best_cost = c; best = ConvPlan{t.tile, sp, -1}; chosen = &t; }
    }
  }
  if (chosen) best.band = best_band(m, n, *chosen, best.splits);
  return best;
}

// The choice is up to a hundred evaluations of the cost above (0.2 to 1.1 us of host time, which a direct launch waits for), and a model
// repeats a few dozen shapes: every host thread remembers its last ones, by value.
static ConvPlan choose_plan(int dtype, long long m, int n, int ktiles, int out_mode) {
  struct Seen { long long m; int n, ktiles, out_mode, dtype, forced; ConvPlan plan; };
  static thread_local Seen seen[256] = {};                   // (no shape has m = 0)
  const int forced = g_tile_override;
  const unsigned h = (((unsigned)m * 31u + (unsigned)n) * 31u + (unsigned)ktiles) * 31u + (unsigned)(out_mode * 2 + dtype);
  Seen& e = seen[(h ^ h >> 8 ^ h >> 16) & 255];
  if (e.m != m || e.n != n || e.ktiles != ktiles || e.out_mode != out_mode || e.dtype != dtype || e.forced != forced)
    e = Seen{m, n, ktiles, out_mode, dtype, forced, compute_plan(dtype, m, n, ktiles, out_mode, forced)};
  return e.plan;
}

size_t conv_workspace_bytes(int dtype, long long m, int n, int k, int out_mode) {
  const int ktiles = k / bk_elems(dtype);
  const int splits = choose_plan(dtype, m, n, ktiles, out_mode).splits;
  return splits > 1 ? (size_t)splits * m * n * 4 : 0;
}

// A 1x1 convolution of the block's input (the shortcut) added to the 3x3 one: as further k-tiles of the same launch on the LDS-DMA and the small-tile kernels, a
// launch of its own, whose sum goes through memory as the residual, on the others.  Saves a launch of 7 to 25 us per such block (14 of 22
// blocks of the SD-sized models) for as many k-tiles at the rate of a long launch (figures of the small tiles at k_igemm_small): whole runs at 576x320 px 67.5 -> 66.2 ms, 512px 191.4 -> 188.3,
// 768px 299.1 -> 297.5, 1024px level.
bool conv_takes_shortcut(int dtype, long long m, int n, int c, int xc) {
  if (c % bk_elems(dtype) || xc % bk_elems(dtype)) return false;
  const int tile = choose_plan(dtype, m, n, (9 * c + xc) / bk_elems(dtype), OUT_ROWMAJOR).tile;
  if (dtype != AD_BF16) return tile == TILE_SMALL;
  switch (tile) {
    case TILE_SMALL: case TILE_P3_64: case TILE_K2_64: case TILE_D2_128: case TILE_D2_160: case TILE_D2_320: return true;
    case TILE_P3_128: case TILE_P3_256: return g_tile_override == TILE_AUTO || g_tile_override == TILE_P3_128 || g_tile_override == TILE_P3_256;
    default: return false;
  }
}

// Wherever the layer is a small-tile launch: every shape measured (above the kernel, 18 to 288 rows, 128 to 1280 channels) gains 1.5 to 2.4 us.
bool conv_takes_ln(int dtype, long long m, int n, int c, int out_mode) {
  const int bk = bk_elems(dtype);
  if (c % bk || (out_mode != OUT_ROWMAJOR && out_mode != OUT_QKV && out_mode != OUT_GEGLU) || choose_plan(dtype, m, n, c / bk, out_mode).tile != TILE_SMALL) return false;
  const SmallTile t = small_tile(dtype, m, n, c / bk, out_mode);
  return c / bk <= small_ktiles(16 * t.tm, 16 * t.tn);
}

// A small-tile launch that takes in at most 40 elements a thread: what a workgroup does for the norm grows with the samples it takes in, the launch that it
// saves does not.  us (norm + convolution / one launch): 12x12 of 128 bf16 channels (36 elements) 3.7 + 4.8 / 8.9 in a chain that is one gap shorter; beyond the line, with the
// cheaper sums named above the kernel: two samples of 24x24 of 64 (72) 3.9 + 4.3 / 10.4, 16x16 of 128 (64) 3.7 + 5.0 / 8.8.  Channels that a power of two of accesses covers (not 192
// or 384), and samples that gn_layout() can arrange: 257 to 320 pixels of groups of two or four channels it cannot, nor more than six samples of 3, 5, ... pixels.
bool conv_takes_gn(int dtype, int batch, int h, int w, int c0, int c1, int n, int groups, int out_mode, int xc) {
  const int c = c0 + c1, bk = bk_elems(dtype), es = (int)esize(dtype), vn = 16 / es, hw = h * w;
  if ((out_mode != OUT_ROWMAJOR && out_mode != OUT_TRANSPOSED_F32) || c0 % bk || c1 % bk) return false;
  const long long m = (long long)batch * hw;
  if (choose_plan(dtype, m, n, (9 * c + xc) / bk, out_mode).tile != TILE_SMALL) return false;
  const SmallTile t = small_tile(dtype, m, n, (9 * c + xc) / bk, out_mode);
  const int bm = 16 * t.tm;
  return gn_layout(vn, bm, batch, hw, c, groups).slots > 0 && (long long)gn_samples(bm, batch, hw) * hw * c <= 8 * 64 * 40 &&
         small_sum_bytes(bm, 16 * t.tn) * (xc ? 2 : 1) + gn_act_bytes(bm, w, c * es) <= (int)kLdsLimit;
}

ad_status launch_conv(const ConvArgs& a, hipStream_t s) {
  if (a.dtype != AD_F32 && a.dtype != AD_BF16) AD_FAIL(AD_ERR_INVALID, "conv: bad dtype");
  const int bk = bk_elems(a.dtype);
  if (!a.src0 || !a.w || !a.out) AD_FAIL(AD_ERR_INVALID, "conv: null pointer");
  if (a.c0 < bk || a.c0 % bk || a.c1 < 0 || a.c1 % bk || (a.c1 > 0 && !a.src1))
    AD_FAIL(AD_ERR_INVALID, "conv: channels (%d,%d) must be multiples of %d", a.c0, a.c1, bk);
  if ((a.ksize != 1 && a.ksize != 3) || (a.stride != 1 && a.stride != 2) || (a.up != 0 && a.up != 1))
    AD_FAIL(AD_ERR_INVALID, "conv: unsupported ksize/stride/up");
  if (a.batch < 1 || a.hs < 1 || a.ws < 1 || a.n_out < 1) AD_FAIL(AD_ERR_INVALID, "conv: bad shape");
  IgemmParams p;
  p.src0 = a.src0; p.src1 = a.c1 ? a.src1 : a.src0;
  p.c0 = a.c0; p.c1 = a.c1; p.ctot = a.c0 + a.c1;
  p.hs = a.hs; p.ws = a.ws; p.up = a.up; p.hin = a.hs << a.up; p.win = a.ws << a.up;
  p.stride = a.stride; p.ksize = a.ksize; p.pad = a.ksize / 2;
  p.hout = (p.hin + 2 * p.pad - a.ksize) / a.stride + 1;
  p.wout = (p.win + 2 * p.pad - a.ksize) / a.stride + 1;
  p.hw_out = p.hout * p.wout;
  p.div_hw = make_fastdiv((unsigned)p.hw_out);
  p.div_w = make_fastdiv((unsigned)p.wout);
  const long long m = (long long)a.batch * p.hw_out;
  if (m > 0x7fffffffLL / 4) AD_FAIL(AD_ERR_INVALID, "conv: too many output positions");
  p.M = (int)m; p.N = a.n_out;
  p.Kp = a.ksize * a.ksize * p.ctot;      // a multiple of the k-tile because ctot is
  p.kt_main = p.Kp / bk;
  p.xw = a.xw; p.x0 = a.x0; p.x1 = a.xc1 ? a.x1 : a.x0; p.xc0 = a.xw ? a.xc0 : 0; p.xc1 = a.xw ? a.xc1 : 0;
  p.xbytes0 = p.xbytes1 = p.xbytes_w = 0;
  // whether a source of c channels shares no memory with the result: other workgroups may read all of it behind one that has written
  auto apart = [&](const void* src, int c) {
    const size_t es = esize(a.dtype), px = (size_t)a.batch * a.hs * a.ws;
    const char *o = (const char*)a.out, *s0 = (const char*)src;
    return c == 0 || s0 + px * c * es <= o || o + (size_t)m * a.n_out * (a.out_mode == OUT_TRANSPOSED_F32 ? 4 : es) <= s0;
  };
  if (a.xw) {
    if (a.ksize != 3 || a.stride != 1 || a.up || a.c1 || a.residual || a.out_mode != OUT_ROWMAJOR || !a.x0 || a.xc0 < bk || a.xc0 % bk || a.xc1 < 0 ||
        a.xc1 % bk || (a.xc1 > 0 && !a.x1) || !apart(a.x0, a.xc0) || !apart(a.x1, a.xc1) || !conv_takes_shortcut(a.dtype, m, a.n_out, a.c0, a.xc0 + a.xc1))
      AD_FAIL(AD_ERR_INVALID, "conv: bad shortcut");
    const long long pixels = (long long)a.batch * a.hs * a.ws, es = (long long)esize(a.dtype), wb = (long long)round_up(a.n_out, kNPad) * (a.xc0 + a.xc1) * es;
    if (pixels * std::max(a.xc0, a.xc1) * es >= 0x7fffffffLL || wb >= 0x7fffffffLL) AD_FAIL(AD_ERR_INVALID, "conv: operands of 2 GiB or more are not supported");
    p.xbytes0 = (unsigned)(pixels * a.xc0 * es);
    p.xbytes1 = a.xc1 ? (unsigned)(pixels * a.xc1 * es) : p.xbytes0;
    p.xbytes_w = (unsigned)wb;
  }
  p.w_row = a.w_blocks ? kRowBytes : (unsigned)p.Kp * (unsigned)esize(a.dtype);
  p.xw_row = a.w_blocks ? kRowBytes : (unsigned)(p.xc0 + p.xc1) * (unsigned)esize(a.dtype);
  p.w_kt = a.w_blocks ? kWBlock * kRowBytes : kRowBytes;
  p.ktiles = p.kt_main + (p.xc0 + p.xc1) / bk;
  p.k_prof = a.k_real > 0 ? a.k_real : p.Kp;
  p.w = a.w; p.bias = a.bias; p.rowvec = a.rowvec; p.residual = a.residual;
  p.out = a.out; p.out_mode = a.out_mode; p.ld_t = a.ld_t; p.rowvec_ld = a.rowvec_ld > 0 ? a.rowvec_ld : (a.rowvec_ld < 0 ? 0 : a.n_out);
  p.out2 = a.out2; p.out3 = a.out3;
  p.ahead = a.ahead; p.ahead_bytes = a.ahead ? (unsigned)std::min<size_t>(a.ahead_bytes, 0x7fffffff) : 0;
  p.ln_gain = a.ln_gain; p.ln_offset = a.ln_offset; p.ln_eps = a.ln_eps;
  p.gn_groups = a.gn_groups;
  if (a.gn_groups) {
    if (!a.ln_gain || !a.ln_offset || a.ksize != 3 || a.stride != 1 || a.up || !apart(a.src0, a.c0) || !apart(a.src1, a.c1) ||
        (((uintptr_t)a.ln_gain | (uintptr_t)a.ln_offset | (uintptr_t)a.src0 | (a.c1 ? (uintptr_t)a.src1 : 0)) & 15) ||
        !conv_takes_gn(a.dtype, a.batch, a.hs, a.ws, a.c0, a.c1, a.n_out, a.gn_groups, a.out_mode, p.xc0 + p.xc1))
      AD_FAIL(AD_ERR_INVALID, "conv: bad GroupNorm");
    p.gn = gn_layout(16 / (int)esize(a.dtype), 16 * small_tile(a.dtype, m, a.n_out, p.ktiles, a.out_mode).tm, a.batch, p.hw_out, p.ctot, a.gn_groups);
    p.gn_inv_n = 1.0 / ((double)p.hw_out * (p.ctot / a.gn_groups));
  }
  if (!a.gn_groups && a.ln_gain && (!a.ln_offset || a.ksize != 1 || a.stride != 1 || a.up || a.c1 || a.residual || a.rowvec || a.xw || (((uintptr_t)a.ln_gain | (uintptr_t)a.ln_offset) & 15) ||
                    !conv_takes_ln(a.dtype, m, a.n_out, a.c0, a.out_mode)))
    AD_FAIL(AD_ERR_INVALID, "conv: bad LayerNorm");
  if (a.out_mode < OUT_ROWMAJOR || a.out_mode > OUT_QKV) AD_FAIL(AD_ERR_INVALID, "conv: bad out_mode");
  if (a.out_mode == OUT_QKV && (a.n_out % 3 || !a.out2 || !a.out3 || a.residual || a.rowvec || (a.ld_t > 0 && a.ld_t < p.hw_out)))
    AD_FAIL(AD_ERR_INVALID, "conv: bad fused q/k/v use");
  if (a.out_mode == OUT_GEGLU && (a.n_out % 64 || a.residual || a.rowvec)) AD_FAIL(AD_ERR_INVALID, "conv: bad GEGLU use");
  if ((a.out_mode == OUT_TRANSPOSED || a.out_mode == OUT_TRANSPOSED_F32) && (a.ld_t < p.hw_out || a.residual))
    AD_FAIL(AD_ERR_INVALID, "conv: bad transposed output");
  const long long in_elems = (long long)a.batch * a.hs * a.ws;
  const long long w_bytes = (long long)round_up(a.n_out, kNPad) * p.Kp * (long long)esize(a.dtype);
  if (in_elems * std::max(a.c0, a.c1) * (long long)esize(a.dtype) >= 0x7fffffffLL || w_bytes >= 0x7fffffffLL)
    AD_FAIL(AD_ERR_INVALID, "conv: operands of 2 GiB or more are not supported");
  p.bytes0 = (unsigned)(in_elems * a.c0 * esize(a.dtype));
  p.bytes1 = a.c1 ? (unsigned)(in_elems * a.c1 * esize(a.dtype)) : p.bytes0;
  p.bytes_w = (unsigned)w_bytes;
  // workgroup order where the plan has none: the operand that is re-fetched by every XCD should be the smaller one.  The activations of
  // a 3x3 convolution count once per tap: a tap's rows come back only after a whole pass over the channels, long
  // after an L2 has dropped them (measured: 333 instead of 828 MB of L2 fills for the 1920 -> 640 convolution)
  const int vn = 16 / (int)esize(a.dtype), ncols = a.out_mode == OUT_GEGLU ? a.n_out / 2 : a.out_mode == OUT_QKV ? a.n_out / 3 : a.n_out;
  const bool turned = a.out_mode == OUT_QKV && a.ld_t > 0;
  const auto at16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  p.vec16 = ncols % vn == 0 && at16(a.out) && at16(a.residual) && (a.out_mode != OUT_QKV || (at16(a.out2) && (turned || at16(a.out3))));
  p.turn16 = turned && at16(a.out3) && a.ld_t % vn == 0 && p.hw_out % vn == 0;
  const ConvPlan plan = choose_plan(a.dtype, m, a.n_out, p.ktiles, a.out_mode);
  p.band = plan.band >= 0 ? plan.band : w_bytes > in_elems * (long long)(a.c0 + a.c1) * (long long)esize(a.dtype) * a.ksize * a.ksize ? 0 : 1;
  if (g_order_override >= 0) p.band = g_order_override == 1 ? 0 : 1;
  const int tile = plan.tile;
  int splits = plan.splits;
  if (splits > 1 && (!a.splitk_ws || a.splitk_bytes < (size_t)splits * m * a.n_out * 4)) splits = 1;   // no scratch: plain launch
  if (m * (a.n_out / 4) >= 1LL << 31) splits = 1;            // the second pass counts groups of four columns in 32 bits
  p.kt_per_split = splits > 1 ? (p.ktiles + splits - 1) / splits : p.ktiles;
  p.partial = splits > 1 ? (float*)a.splitk_ws : nullptr;
  const int mode = splits > 1 ? OUT_PARTIAL : a.out_mode;
  const bool big = tile == TILE_128x128;
  const bool h16 = a.dtype == AD_BF16;
  const char* name = h16 ? (big ? "igemm_bf16_128x128" : (splits > 1 ? "igemm_bf16_64x64_splitk" : "igemm_bf16_64x64"))
                         : (big ? "igemm_f32_128x128" : (splits > 1 ? "igemm_f32_64x64_splitk" : "igemm_f32_64x64"));
  ad_status st = AD_ERR_INVALID;
#define AD_RUN(TT, BM_, MODE_) st = run_igemm<TT, BM_, BM_, 2, 2, 1, MODE_>(p, name, s)
#define AD_MODES(TT, BM_)                                              \
  switch (mode) {                                                      \
    case OUT_ROWMAJOR: AD_RUN(TT, BM_, OUT_ROWMAJOR); break;           \
    case OUT_TRANSPOSED: AD_RUN(TT, BM_, OUT_TRANSPOSED); break;       \
    case OUT_TRANSPOSED_F32: AD_RUN(TT, BM_, OUT_TRANSPOSED_F32); break; \
    case OUT_QKV: AD_RUN(TT, BM_, OUT_QKV); break;                     \
    case OUT_PARTIAL: AD_RUN(TT, BM_, OUT_PARTIAL); break;             \
    default: break;                                                    \
  }
  // 3x3, stride 1: the halo-staged kernel, on request (TILE_HALO_*) and when its tiles fit into LDS.  It moves less than
  // half the bytes from L2 into LDS per k-tile, but on the convolutions of the SD-sized models it runs at 0.70-0.85 of the
  // per-tap three-stage kernel (its k-loop has neither that kernel's fragment prefetch across the barrier nor its third
  // weight stage at 256 positions): the automatic choice keeps the per-tap kernels.
  int halo_bm = 0;
  if (h16 && a.ksize == 3 && a.stride == 1 && (mode == OUT_ROWMAJOR || mode == OUT_PARTIAL) && (tile == TILE_P3_128 || tile == TILE_P3_256) &&
      (g_tile_override == TILE_HALO_128 || g_tile_override == TILE_HALO_256)) {
    const bool want256 = tile == TILE_P3_256 && g_tile_override != TILE_HALO_128;
    if (want256 && halo_lds_bytes(256, 2, a.ws, a.up) <= kLdsLimit && halo_rows(256, a.ws, a.up) / 32 <= 32) halo_bm = 256;
    else if (halo_lds_bytes(128, 3, a.ws, a.up) <= kLdsLimit && halo_rows(128, a.ws, a.up) / 32 <= 16) halo_bm = 128;
  }
  if (halo_bm) {
    const int nchunks = p.ctot / 64;
    if (splits > 1) {
      const int per = (nchunks + splits - 1) / splits;
      splits = (nchunks + per - 1) / per;              // split-K over channel chunks: never more splits than chunks
      if (splits <= 1) { splits = 1; p.partial = nullptr; }
    }
    const int hmode = splits > 1 ? OUT_PARTIAL : a.out_mode;
    if (halo_bm == 256) {
      if (hmode == OUT_ROWMAJOR) st = run_conv3_halo<256, 2, OUT_ROWMAJOR>(p, splits, "conv3_halo_bf16_256x128", s);
      else st = run_conv3_halo<256, 2, OUT_PARTIAL>(p, splits, "conv3_halo_bf16_256x128_splitk", s);
    } else {
      if (hmode == OUT_ROWMAJOR) st = run_conv3_halo<128, 3, OUT_ROWMAJOR>(p, splits, "conv3_halo_bf16_128x128", s);
      else st = run_conv3_halo<128, 3, OUT_PARTIAL>(p, splits, "conv3_halo_bf16_128x128_splitk", s);
    }
  } else if (tile == TILE_P3_128 || tile == TILE_P3_256) {
    // eight wavefronts (two per SIMD) by default: 3-20 % faster than four on the layers of the SD-sized models; the
    // four- and sixteen-wavefront variants stay selectable for measurements
    const int wm = g_tile_override == TILE_P3_256_W4 || g_tile_override == TILE_P3_128_W4 ? 2 : (g_tile_override == TILE_P3_256_W16 && tile == TILE_P3_256 ? 8 : 4);
#define AD_P3W(BM_, WM_, TAG)                                                                                                          \
  switch (mode) {                                                                                                                      \
    case OUT_ROWMAJOR: st = run_igemm_p3<bf16, BM_, 128, OUT_ROWMAJOR, WM_>(p, "igemm_bf16_" #BM_ "x128_p3" TAG, s); break;            \
    case OUT_GEGLU: st = run_igemm_p3<bf16, BM_, 128, OUT_GEGLU, WM_>(p, "igemm_bf16_" #BM_ "x128_p3" TAG, s); break;                  \
    case OUT_QKV: st = run_igemm_p3<bf16, BM_, 128, OUT_QKV, WM_>(p, "igemm_bf16_" #BM_ "x128_p3" TAG, s); break;                      \
    case OUT_PARTIAL: st = run_igemm_p3<bf16, BM_, 128, OUT_PARTIAL, WM_>(p, "igemm_bf16_" #BM_ "x128_p3" TAG "_splitk", s); break;    \
    default: break;                                                                                                                    \
  }
    if (tile == TILE_P3_256) {
      if (wm == 2) { AD_P3W(256, 2, "w4") } else if (wm == 8) { AD_P3W(256, 8, "w16") } else { AD_P3W(256, 4, "") }
    } else {
      if (wm == 2) { AD_P3W(128, 2, "w4") } else { AD_P3W(128, 4, "") }
    }
#undef AD_P3W
  } else if (tile == TILE_SMALL) {
    const SmallTile t = small_tile(a.dtype, m, a.n_out, p.ktiles, a.out_mode);
    name = h16 ? "igemm_bf16_small" : "igemm_f32_small";
#define AD_SMALL(TM_, TN_, MODE_) st = h16 ? run_igemm_small<bf16, TM_, TN_, MODE_>(p, name, s) : run_igemm_small<float, TM_, TN_, MODE_>(p, name, s)
#define AD_SMALL_MODE(MODE_)                                  \
  case MODE_:                                                 \
    if (t.tm == 2) { AD_SMALL(2, 2, MODE_); }                 \
    else if (t.tn == 2) { AD_SMALL(1, 2, MODE_); }            \
    else { AD_SMALL(1, 1, MODE_); }                           \
    break;
    switch (a.out_mode) {
      AD_SMALL_MODE(OUT_ROWMAJOR)
      AD_SMALL_MODE(OUT_QKV)
      AD_SMALL_MODE(OUT_TRANSPOSED)
      AD_SMALL_MODE(OUT_TRANSPOSED_F32)
      default: if (t.tm == 2) { AD_SMALL(2, 4, OUT_GEGLU); } else { AD_SMALL(1, 4, OUT_GEGLU); }
    }
#undef AD_SMALL_MODE
#undef AD_SMALL
  } else if (tile == TILE_P3_64) {
    switch (mode) {
      case OUT_ROWMAJOR: st = run_igemm_p3<bf16, 64, 64, OUT_ROWMAJOR>(p, "igemm_bf16_64x64_p3", s); break;
      case OUT_QKV: st = run_igemm_p3<bf16, 64, 64, OUT_QKV>(p, "igemm_bf16_64x64_p3", s); break;
      case OUT_PARTIAL: st = run_igemm_p3<bf16, 64, 64, OUT_PARTIAL>(p, "igemm_bf16_64x64_p3_splitk", s); break;
      default: break;
    }
  } else if (tile == TILE_K2_64) {
    switch (mode) {
      case OUT_ROWMAJOR: st = run_igemm_p3<bf16, 64, 64, OUT_ROWMAJOR, 2, 2, 3, 2>(p, "igemm_bf16_64x64_k2", s); break;
      case OUT_QKV: st = run_igemm_p3<bf16, 64, 64, OUT_QKV, 2, 2, 3, 2>(p, "igemm_bf16_64x64_k2", s); break;
      case OUT_PARTIAL: st = run_igemm_p3<bf16, 64, 64, OUT_PARTIAL, 2, 2, 3, 2>(p, "igemm_bf16_64x64_k2_splitk", s); break;
      default: break;
    }
  } else if (tile == TILE_D2_128) {
    switch (mode) {
      case OUT_ROWMAJOR: st = run_igemm_p3<bf16, 128, 128, OUT_ROWMAJOR, 4, 2, 2>(p, "igemm_bf16_128x128_d2", s); break;
      case OUT_GEGLU: st = run_igemm_p3<bf16, 128, 128, OUT_GEGLU, 4, 2, 2>(p, "igemm_bf16_128x128_d2", s); break;
      case OUT_QKV: st = run_igemm_p3<bf16, 128, 128, OUT_QKV, 4, 2, 2>(p, "igemm_bf16_128x128_d2", s); break;
      case OUT_PARTIAL: st = run_igemm_p3<bf16, 128, 128, OUT_PARTIAL, 4, 2, 2>(p, "igemm_bf16_128x128_d2_splitk", s); break;
      default: break;
    }
  } else if (tile == TILE_D2_160) {
    switch (mode) {
      case OUT_ROWMAJOR: st = run_igemm_p3<bf16, 128, 160, OUT_ROWMAJOR, 4, 1, 2>(p, "igemm_bf16_128x160_d2", s); break;
      case OUT_QKV: st = run_igemm_p3<bf16, 128, 160, OUT_QKV, 4, 1, 2>(p, "igemm_bf16_128x160_d2", s); break;
      case OUT_PARTIAL: st = run_igemm_p3<bf16, 128, 160, OUT_PARTIAL, 4, 1, 2>(p, "igemm_bf16_128x160_d2_splitk", s); break;
      default: break;
    }
  } else if (tile == TILE_D2_320) {
    switch (mode) {
      case OUT_ROWMAJOR: st = run_igemm_p3<bf16, 256, 320, OUT_ROWMAJOR, 4, 2, 2>(p, "igemm_bf16_256x320_d2", s); break;
      case OUT_GEGLU: st = run_igemm_p3<bf16, 256, 320, OUT_GEGLU, 4, 2, 2>(p, "igemm_bf16_256x320_d2", s); break;
      case OUT_QKV: st = run_igemm_p3<bf16, 256, 320, OUT_QKV, 4, 2, 2>(p, "igemm_bf16_256x320_d2", s); break;
      case OUT_PARTIAL: st = run_igemm_p3<bf16, 256, 320, OUT_PARTIAL, 4, 2, 2>(p, "igemm_bf16_256x320_d2_splitk", s); break;
      default: break;
    }
  } else if (mode == OUT_GEGLU) {
    if (h16) AD_RUN(bf16, 128, OUT_GEGLU); else AD_RUN(float, 128, OUT_GEGLU);
  } else if (h16) {
    if (big) { AD_MODES(bf16, 128) } else { AD_MODES(bf16, 64) }
  } else {
    if (big) { AD_MODES(float, 128) } else { AD_MODES(float, 64) }
  }
#undef AD_MODES
#undef AD_RUN
  if (st != AD_OK || splits <= 1) return st;
  const long long quads = m * (a.n_out / 4);
  const int blocks = (int)((quads + 255) / 256 < 2048 ? (quads + 255) / 256 : 2048);
  const int rowvec_ld = a.rowvec_ld > 0 ? a.rowvec_ld : (a.rowvec_ld < 0 ? 0 : a.n_out);
  const auto at4 = [&](const void* q) { return (uintptr_t)q % (4 * esize(a.dtype)) == 0; };
  const int vec4 = ncols % 4 == 0 && at4(a.out) && at4(a.residual) && (a.out_mode != OUT_QKV || (at4(a.out2) && (turned || at4(a.out3))));
  ProfLaunch pl("splitk_reduce", 0, (double)splits * m * a.n_out * 4 + (double)m * a.n_out * esize(a.dtype), s);
#define AD_REDUCE(T_)                                                                                                                  \
  hipLaunchKernelGGL(k_splitk_reduce<T_>, dim3(blocks), dim3(256), 0, s, p.partial, splits, p.M, p.N, p.hw_out, make_fastdiv((unsigned)(p.N / 4)), \
                     p.div_hw, vec4, a.bias, a.rowvec, rowvec_ld, (const T_*)a.residual, a.out, a.out2, a.out3, a.out_mode, a.ld_t)
  if (a.dtype == AD_BF16) AD_REDUCE(bf16);
  else AD_REDUCE(float);
#undef AD_REDUCE
  AD_HIP(hipGetLastError());
  return AD_OK;
}

void set_tile_override(int tile) { g_tile_override = tile; }
void set_order_override(int order) { g_order_override = order; }

// =================================================================================================
// Fused attention for bf16, head_dim 64.  A workgroup handles 128 queries of one (batch, head); each
// wavefront owns 32 queries.  Per 64-key tile: S^T = K Q^T (keys in accumulator registers, the
// query in the lane), online softmax with one cross-half exchange, O^T += V^T P^T.
// =================================================================================================
__device__ __forceinline__ float other_half(float x, bool low) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(low ? r[1] : r[0]);
}

constexpr int kAttnStage = 2 * 64 * kPitch;   // one K tile and one V^T tile (64 rows of 128 bytes + pad each)

// four wavefronts per SIMD: with 32-bit running offsets instead of pointers the score and output tiles, the query
// fragments and the tile in flight fit the 128 VGPRs of that occupancy without accumulation-register copies
// (with pointers the compiler moved the MFMA results through accumulation registers around every softmax, about a
// third of the loop's vector instructions, and three wavefronts per SIMD were the better choice)
// RAGGED (Lk not a multiple of 64) is a template parameter: left as a run-time flag, the masking of the last key
// tile is turned into unconditional compares and selects on every tile (65-100 vector instructions per tile).
template <bool RAGGED>
__global__ __attribute__((amdgpu_waves_per_eu(4, 4))) __launch_bounds__(256) void k_attn_mfma(const bf16* __restrict__ Q, const bf16* __restrict__ K,
                                                   const bf16* __restrict__ Vt, bf16* __restrict__ O, int L, int Lk,
                                                   int C, int ldq, int ldk, int ldv, int ldo, float scale_log2, int qblocks) {
  __shared__ __attribute__((aligned(16))) char lds[2 * kAttnStage];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const bool low = half == 0;
  // one-dimensional grid, renumbered so that the query blocks of a (sample, head) run on one XCD and
  // its keys and values are fetched into a single L2
  const int vid = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = vid / qblocks, heads = C / 64;
  const int b = bh / heads, h = bh - b * heads;
  const int query = (vid - bh * qblocks) * 128 + wave * 32 + l32;
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[ks][e] = (bf16)0.f;
    if (query < L) qf[ks] = *(const bf16x8*)(Q + ((size_t)b * L + query) * ldq + h * 64 + ks * 16 + half * 8);
  }
  f32x16 o[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const int srow = tid >> 3, scol = tid & 7;
  const int ntiles = (Lk + 63) / 64;
  constexpr bool ragged = RAGGED;
  // running 32-bit element offsets of this thread's two rows of the K tile (keys) and of the V^T tile (channels)
  // from bases that are uniform over the workgroup (the launcher checks that they fit)
  const bf16* kbase = K + (size_t)b * Lk * ldk + h * 64;
  const bf16* vbase = Vt + ((size_t)b * C + h * 64) * ldv;
  unsigned kp[2], vp[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    kp[i] = (unsigned)((srow + 32 * i) * ldk + scol * 8);
    vp[i] = (unsigned)((srow + 32 * i) * ldv + scol * 8);
  }
  const unsigned kstep = 64u * (unsigned)ldk;

  // the next tile travels through registers while the current one is multiplied; tiles are loaded in order.
  // Only the last tile can be ragged: every test on key indices sits behind a workgroup-uniform branch.
  bf16x8 kr[2], vr[2];
  auto load_tile = [&](int t) {
    if (!ragged || t + 1 < ntiles) {
#pragma unroll
      for (int i = 0; i < 2; ++i) kr[i] = *(const bf16x8*)(kbase + kp[i]);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e) kr[i][e] = (bf16)0.f;
        if (t * 64 + srow + 32 * i < Lk) kr[i] = *(const bf16x8*)(kbase + kp[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      vr[i] = *(const bf16x8*)(vbase + vp[i]);          // in bounds: ldv is padded to 64 keys
      kp[i] += kstep;
      vp[i] += 64;
    }
  };
  auto store_tile = [&](int t, int parity) {
    char* st = lds + parity * kAttnStage;
    if (ragged && t + 1 == ntiles) {          // keys past the end must not contribute, whatever the pad holds
      const int kb = t * 64 + scol * 8;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (kb + e >= Lk) vr[i][e] = (bf16)0.f;
    }
    // V^T rows are stored with the keys of every group of 16 in the order 0-3, 8-11, 4-7, 12-15: that is the order
    // in which the probabilities come out of the score tile (a lane holds keys 4 half + 0..3 and 8 + 4 half + 0..3
    // of a group), so that the matching V^T fragment is one 16-byte read
    const int vslot = (scol >> 1) * 32 + (scol & 1) * 8;       // byte offset of keys 8 scol .. +3; keys +4 .. +7 follow 16 bytes on
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *(bf16x8*)(st + (srow + 32 * i) * kPitch + scol * 16) = kr[i];
      char* vrow = st + 64 * kPitch + (srow + 32 * i) * kPitch + vslot;
      *(bf16x4*)vrow = bf16x4{vr[i][0], vr[i][1], vr[i][2], vr[i][3]};
      *(bf16x4*)(vrow + 16) = bf16x4{vr[i][4], vr[i][5], vr[i][6], vr[i][7]};
    }
  };
  // one key tile; PAR (the LDS stage) is a compile-time constant so that every LDS address is base + immediate
  auto step = [&](int t, auto par) {
    constexpr int PAR = decltype(par)::value;
    if (t + 1 < ntiles) {
      store_tile(t + 1, PAR ^ 1);
      if (t + 2 < ntiles) load_tile(t + 2);
    }
    const char* Ks = lds + PAR * kAttnStage;
    const char* Vs = Ks + 64 * kPitch;
    f32x16 sc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[j][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 a = *(const bf16x8*)(Ks + (j * 32 + l32) * kPitch + ks * 32 + half * 16);
        sc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], sc[j], 0, 0, 0);
      }
    }
    if (ragged && t == ntiles - 1) {     // only the last tile can hold keys past the end
      const int key0 = t * 64;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (key0 + j * 32 + 8 * (r >> 2) + 4 * half + (r & 3) >= Lk) sc[j][r] = -INFINITY;
    }
    float mx = sc[0][0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[0][r]);
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[1][r]);
    mx = fmaxf(mx, other_half(mx, low));
    const float m_new = fmaxf(m_run, mx);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {     // some row maximum moved: rescale what was accumulated
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      m_run = m_new;
    }
    const float neg = -m_run * scale_log2;
    float psum = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sc[j][r] = __builtin_amdgcn_exp2f(fmaf(sc[j][r], scale_log2, neg));
        psum += sc[j][r];
      }
    l_run += psum;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        bf16x8 pb;
#pragma unroll
        for (int e = 0; e < 8; ++e) pb[e] = (bf16)sc[j][8 * s2 + e];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const bf16x8 a = *(const bf16x8*)(Vs + (d * 32 + l32) * kPitch + (j * 32 + 16 * s2) * 2 + 16 * half);
          o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb, o[d], 0, 0, 0);
        }
      }
    __syncthreads();
  };

  load_tile(0);
  store_tile(0, 0);
  if (ntiles > 1) load_tile(1);
  __syncthreads();
  for (int t = 0; t < ntiles; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
  }
  const float l_tot = l_run + other_half(l_run, low);
  if (query < L) {
    const float inv = 1.f / l_tot;
    bf16* orow = O + ((size_t)b * L + query) * ldo + h * 64;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(o[d][4 * g + e] * inv);
        *(bf16x4*)(orow + d * 32 + 8 * g + 4 * half) = v;
      }
  }
}

// =================================================================================================
// Fused attention, second generation (bf16, head_dim 64).  What changed against k_attn_mfma and why:
//  * a wavefront owns 32 * QSETS queries (QSETS = 2: 64), so every K and V^T fragment read from LDS feeds QSETS
//    MFMAs: at 32 queries per wavefront the fragment reads alone need the LDS port's full rate at full MFMA rate;
//  * K and V^T tiles are written into LDS by the load unit (buffer_load ... lds, three stages, dense 128-byte rows
//    with the XOR swizzle of the GEMM kernels): no staging registers, no ds_write;
//  * the vector work per score is the exponential, half a conversion and half an add.  q is multiplied by
//    log2(e) / sqrt(d) once, when it is loaded.  The reference value m that is subtracted before the exponential
//    enters the score MFMA as its C operand (a 16-register block holding -m), so the scores leave the matrix pipe
//    as s - m.  m need not be the running maximum: the result is exact for any m, and fp32 / bf16 hold
//    2^(s - m) as long as s - m stays below about 100, so m is the exact maximum of the first 32 keys and is
//    raised (with the usual rescaling of what has been accumulated) only when a row sum of a 32-key block
//    reaches 2^100 - this is tested on the sum, which is needed anyway, so the steady state computes no
//    maximum at all.  m never exceeds the running maximum, hence the largest term of a row is at least 1 and
//    nothing underflows.  The row sums are taken from the bf16 probabilities, two per instruction;
//  * the keys of a tile are placed in LDS rows so that the 8 score registers a lane holds per 16-key block are 8
//    consecutive keys (LDS row 16 b + 8 a + 4 h + e holds key 16 b + 8 h + 4 a + e): the probabilities are the B
//    operand of the PV product as they stand and V^T is read in its natural order;
//  * an accumulator is used by MFMAs that follow each other directly (the result is forwarded) or are at least
//    four apart: two alternating accumulation chains run at 58 instead of 33 cycles per MFMA on this chip.
// Scores are computed transposed (S^T = K Q^T, a lane owns one query) as in the first kernel.
// =================================================================================================
constexpr int kAttn2Stage = 2 * 64 * kRowBytes;   // one K tile and one V^T tile of 64 keys: 16 KiB
constexpr float kAttnBig = 1.2676506e30f;         // 2^100: a 32-key row sum at or above it moves the reference

// NSTG: LDS stages (tiles requested two ahead from three stages on); OCC: wavefronts per SIMD the register budget is set for.
// PIPE (one query set): the software-pipelined path.  Measured on this chip: a wavefront that issues four plain vector
// instructions between two of its own MFMAs pays nothing for them (32 -> 34 cycles per MFMA), an exponential costs about
// 4.5 cycles, whereas vector work of ANOTHER wavefront of the SIMD overlaps an MFMA stream poorly (1.25-1.45x instead of 2x).
// So the vector work has to sit between the MFMAs of the same wavefront: a step issues the score MFMAs of block u + 1,
// the exponentials / conversions / row sums of block u (whose scores the previous step left in registers) and the PV MFMAs of
// block u in one straight line, with the order pinned (one MFMA, five vector instructions, ...).  The steady state has no
// branch: the reference is the exact maximum of the first 32 keys, and whether some later score left the window
// (row sum >= 2^100 or not finite) is tested once, at the end; if so - it takes a score more than 69 nats above every
// one of the first 32 - the workgroup repeats its work with the checked block-by-block loop below.  The K fragments of a
// step are fetched from LDS one step ahead, so a tile is opened (waited for, barrier) one block before its first scores:
// three tiles are in use across that barrier plus one in flight, hence four stages (64 KiB, two workgroups per CU).
//
// KS > 1: the keys are shared out over KS groups of NWQ wavefronts, each with tiles and stages of its own, and merged at the end (launch
// rule in attn_split()).
template <int QSETS, bool RAGGED, int NSTG = 3, int OCC = (QSETS == 1 ? 3 : 2), int PIPE = 0, int NWQ = 4, int KS = 1>
__global__ __attribute__((amdgpu_waves_per_eu(OCC, OCC))) __launch_bounds__(64 * NWQ * KS) void k_attn_mfma2(
    const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ Vt, bf16* __restrict__ O, int L, int Lk, int C,
    int ldq, int ldk, int ldv, int ldo, float scale_log2, int qblocks) {
  extern __shared__ __attribute__((aligned(128))) char lds_all[];
  static_assert(KS == 1 || (PIPE == 0 && QSETS == 1), "shared keys: the plain loop");
  constexpr int QW = 32 * QSETS;                  // queries per wavefront
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave_all % NWQ, group = wave_all / NWQ;
  char* const lds = lds_all + group * (NSTG * kAttn2Stage);
  const bool low = half == 0;
  const int vid = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = vid / qblocks, heads = C / 64;
  const int b = bh / heads, h = bh - b * heads;
  const int q0 = (vid - bh * qblocks) * (NWQ * QW) + wave * QW + l32;
  const int ntiles = (Lk + 63) / 64;
  // this group's tiles (never none): t_first .. t_last - 1
  const int t_each = (ntiles + KS - 1) / KS, t_first = KS == 1 ? 0 : group * t_each, t_last = KS == 1 ? ntiles : min(ntiles, t_first + t_each);

  // ---- tile loads: per 64-key tile a wavefront issues LPT 8-row groups of K and LPT of V^T
  const bf16* kbase = K + (size_t)b * Lk * ldk + h * 64;
  const bf16* vbase = Vt + ((size_t)b * C + h * 64) * ldv;
  const u32x4 rsk = make_rsrc_words(kbase, (unsigned)(((size_t)(Lk - 1) * ldk + 64) * 2));
  const u32x4 rsv = make_rsrc_words(vbase, (unsigned)((size_t)64 * ldv * 2));
  // LDS row r keeps its 16-byte chunk c at position c ^ ((r >> 1) & 7): the 16 rows that one quarter of a wavefront
  // reads in a cycle (same chunk, consecutive rows) then fall on 16 different 16-byte bank groups of the 256-byte
  // bank window (rows r and r + 8 collide with the plain r & 7 swizzle)
  // A wavefront fills the 8-row groups g = wave, wave + NWQ, ... of the K tile and of the V^T tile: they have the same swizzle
  // column, and their rows are 8 NWQ keys (rows of V^T) apart, so one lane offset serves all (the distance goes into the
  // scalar offset of the load)
  constexpr int LPT = 8 / NWQ;
  const int r8 = lane >> 3;
  const int scol = (lane & 7) ^ (((wave * 8 + r8) >> 1) & 7);                // chunk this lane fetches for its row
  const int krow = 16 * (wave >> 1) + 8 * (r8 >> 2) + 4 * (wave & 1) + (r8 & 3);   // key held by LDS row 8 wave + r8 (+ 8 NWQ: row + 8 NWQ)
  const unsigned koff = (unsigned)(krow * ldk + scol * 8) * 2;
  const unsigned voff = (unsigned)((wave * 8 + r8) * ldv + scol * 8) * 2;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds;
  const unsigned kstep = 64u * (unsigned)ldk * 2u, khalf = 8u * NWQ * (unsigned)ldk * 2u, vhalf = 8u * NWQ * (unsigned)ldv * 2u;
  auto issue = [&](int t, int stage) {
    const unsigned st = lds_base + stage * kAttn2Stage + (unsigned)wave * 1024u;
    const bool last = RAGGED && t == ntiles - 1;
    if (!last) {
#pragma unroll
      for (int i = 0; i < LPT; ++i) dma_load16(rsk, koff, (unsigned)t * kstep + i * khalf, st + i * NWQ * 1024);
#pragma unroll
      for (int i = 0; i < LPT; ++i) dma_load16(rsv, voff, (unsigned)t * 128u + i * vhalf, st + 8192 + i * NWQ * 1024);
    } else {
      // keys past the end read zeros (their scores are masked, but the pad must not hold NaNs).  The row goes into the lane's offset:
      // the range check compares that with the size less the scalar offset, and some rows on may lie beyond the size.
#pragma unroll
      for (int i = 0; i < LPT; ++i)
        dma_load16(rsk, t * 64 + krow + 8 * NWQ * i >= Lk ? kOob : koff + (unsigned)t * kstep + i * khalf, 0u, st + i * NWQ * 1024);
      // the last, partial tile of V^T goes through registers: values of keys past the end are cleared, whatever the pad holds
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        const int g = wave + NWQ * i;
        bf16x8 v = *(const bf16x8*)(vbase + (size_t)(g * 8 + r8) * ldv + t * 64 + scol * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (t * 64 + scol * 8 + e >= Lk) v[e] = (bf16)0.f;
        *(bf16x8*)(lds + stage * kAttn2Stage + 8192 + g * 1024 + lane * 16) = v;
      }
    }
  };
  issue(t_first, 0);
  if (NSTG > 2 && t_first + 1 < t_last) issue(t_first + 1, 1);

  // ---- queries: B operand of the score product, pre-multiplied by log2(e) / sqrt(d)
  bf16x8 qf[QSETS][4];
#pragma unroll
  for (int s = 0; s < QSETS; ++s)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[s][ks][e] = (bf16)0.f;
      if (q0 + 32 * s < L) {
        const bf16x8 raw = *(const bf16x8*)(Q + ((size_t)b * L + q0 + 32 * s) * ldq + h * 64 + ks * 16 + half * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[s][ks][e] = (bf16)((float)raw[e] * scale_log2);
      }
    }
  f32x16 o[QSETS][2], negm[QSETS];
  float m_ref[QSETS], l_run[QSETS];
#pragma unroll
  for (int s = 0; s < QSETS; ++s) {
    m_ref[s] = 0.f; l_run[s] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { o[s][0][r] = 0.f; o[s][1][r] = 0.f; negm[s][r] = 0.f; }
  }
  // fragment offsets inside a tile: row l32, 16-byte chunk (2 c + half) at its swizzled place; K fragment ks uses c = ks,
  // the V^T fragment of block j and 16-key half s2 uses c = 2 j + s2
  // (c and c + 2 differ in bit 6 of the offset only)
  int cofs[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) cofs[c] = l32 * kRowBytes + (((c * 2 + half) ^ lds_swizzle(l32)) << 4);
  auto cof = [&](int c) -> int { return c < 2 ? cofs[c] : (cofs[c - 2] ^ 64); };
  const bf16x2 ones = {(bf16)1.f, (bf16)1.f};
  auto mask_tail = [&](f32x16 (&sc)[QSETS], int t, int j) {
    const int key0 = t * 64 + j * 32 + 8 * half;          // register r: key key0 + 16 (r / 8) + r % 8
#pragma unroll
    for (int s = 0; s < QSETS; ++s)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key0 + 16 * (r >> 3) + (r & 7) >= Lk) sc[s][r] = -INFINITY;
  };
  // p = 2^(s - m) in bf16 for both 16-key halves of a block, and their row sums
  auto probs = [&](const f32x16 (&sc)[QSETS], bf16x8 (&dst)[QSETS][2], float (&psum)[QSETS]) {
#pragma unroll
    for (int s = 0; s < QSETS; ++s) {
      psum[s] = 0.f;
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const bf16x2 pp = {(bf16)__builtin_amdgcn_exp2f(sc[s][8 * s2 + e]), (bf16)__builtin_amdgcn_exp2f(sc[s][8 * s2 + e + 1])};
          dst[s][s2][e] = pp[0]; dst[s][s2][e + 1] = pp[1];
          psum[s] = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, psum[s], false);
        }
    }
  };
  // One 32-key block: scores, probabilities, PV.  `first`: the block that fixes the reference (exact maximum).
  auto block = [&](const char* Ks, int t, int j, bool first) {
    const char* Vs = Ks + 8192;
    bf16x8 kf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[ks] = *(const bf16x8*)(Ks + j * 32 * kRowBytes + cof(ks));
    __builtin_amdgcn_s_setprio(0);
    f32x16 sc[QSETS];
#pragma unroll
    for (int s = 0; s < QSETS; ++s) {
      sc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[s][0], negm[s], 0, 0, 0);
#pragma unroll
      for (int ks = 1; ks < 4; ++ks) sc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[s][ks], sc[s], 0, 0, 0);
    }
    // between its products a wavefront goes ahead of those that have matrix work to issue: its exponentials are what the next products wait for, theirs
    // queue up anyway.  Alone, us: 4096 tokens, 2 x 5 heads 65.9 -> 61.8, 2304, 2 x 10 40.1 -> 39.0, 2880, 5 22.0 -> 21.1, 9216, 2 x 5 227.6 -> 228.9, 4096,
    // 2 x 10 100.9 -> 102.5 (inside the models on one stream 240.1 -> 240.8 and 107.6 -> 108.3, and all attention of a step 512px 458 -> 443, 768px 1485 -> 1481,
    // 1024px 2459 -> 2428, video 2055 -> 2040); whole runs 512px 1.006, 768px 1.004, 1024px 1.004, video 1.003 (the products ahead instead: 1-2 % slower)
    __builtin_amdgcn_s_setprio(1);
    // the V^T fragments are requested before the exponentials so that they have arrived when the PV products start
    bf16x8 vf[2][2];
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        vf[d][s2] = *(const bf16x8*)(Vs + d * 32 * kRowBytes + cof(2 * j + s2));
    if (RAGGED && t == ntiles - 1) mask_tail(sc, t, j);
    bf16x8 pb[QSETS][2];
    float psum[QSETS];
    probs(sc, pb, psum);
    bool redo = first;
#pragma unroll
    for (int s = 0; s < QSETS; ++s) redo |= !(psum[s] < kAttnBig) || (KS > 1 && m_ref[s] == -INFINITY);
    // the score MFMAs keep their program order: each chain of four runs back to back
#pragma unroll
    for (int i = 0; i < 4 * QSETS; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (__builtin_amdgcn_ballot_w64(redo) != 0) {
      // rare: the reference is too far below some score of this block (or this is the first block).  Take the exact
      // maximum of the block, move the reference there, rescale what has been accumulated, and redo the block.
#pragma unroll
      for (int s = 0; s < QSETS; ++s) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[s][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const bf16x8 kk = *(const bf16x8*)(Ks + j * 32 * kRowBytes + cof(ks));
          sc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk, qf[s][ks], sc[s], 0, 0, 0);
        }
      }
      if (RAGGED && t == ntiles - 1) mask_tail(sc, t, j);
#pragma unroll
      for (int s = 0; s < QSETS; ++s) {
        float a = fmaxf(fmaxf(sc[s][0], sc[s][1]), sc[s][2]);
#pragma unroll
        for (int r = 3; r + 1 < 16; r += 2) a = fmaxf(fmaxf(a, sc[s][r]), sc[s][r + 1]);
        a = fmaxf(a, sc[s][15]);
        a = fmaxf(a, other_half(a, low));
        const float m_new = first ? a : fmaxf(m_ref[s], a);
        // a group that starts in the middle of the keys may see nothing but minus infinity at first: no reference yet, nothing to rescale
        const bool none = KS > 1 && m_ref[s] == -INFINITY;
        const float alpha = first || none ? 1.f : __builtin_amdgcn_exp2f(m_ref[s] - m_new), sub = KS > 1 && m_new == -INFINITY ? 0.f : m_new;
        m_ref[s] = m_new;
        l_run[s] *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          o[s][0][r] *= alpha; o[s][1][r] *= alpha;
          sc[s][r] -= sub;
          negm[s][r] = -sub;
        }
      }
      probs(sc, pb, psum);
    }
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int s = 0; s < QSETS; ++s) {
      l_run[s] += psum[s];
      // O^T += V^T P^T; the two MFMAs of an accumulator follow each other directly (the result is forwarded)
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) o[s][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[d][s2], pb[s][s2], o[s][d], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4 * QSETS; ++i) __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
    __builtin_amdgcn_s_setprio(1);
  };

  // Waits for tile t and lets a free stage be refilled.  Tile t has landed once at most the loads of tile t + 1 are outstanding
  // (a partial last tile waits by itself); after the barrier tile t is complete for every wavefront and everybody is done with
  // tile t - 1 (the pipelined path, which opens a tile one block early, is then done with tile t - 2: hence its fourth stage).
  auto open_tile = [&](int t, int stage) {
    if (NSTG > 2 && t + 1 < t_last && !(RAGGED && t + 2 == ntiles)) wait_vmcnt<2 * LPT>(); else wait_vmcnt<0>();
    __syncthreads();
    constexpr int AHEAD = NSTG > 2 ? 2 : 1;      // tiles requested ahead (a fourth stage is slack for the pipelined path)
    if (t + AHEAD < t_last) {
      int target = stage + AHEAD;
      if (target >= NSTG) target -= NSTG;
      issue(t + AHEAD, target);
    }
  };
  if constexpr (PIPE != 0) {
    static_assert(QSETS == 1 && NSTG == 4, "the pipelined path is written for one query set and four stages");
    __shared__ int s_redo;
    const int nfull = RAGGED ? ntiles - 1 : ntiles;     // tiles without a ragged tail
    auto stage_of = [&](int t) { return lds + (t % NSTG) * kAttn2Stage; };
    open_tile(0, 0);
    block(lds, 0, 0, true);                              // fixes the reference: exact maximum of the first 32 keys
    if (nfull == 0) {
      block(lds, 0, 1, false);
    } else {
      auto k_frags = [&](const char* Ks, int j, bf16x8 (&kf)[4]) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) kf[ks] = *(const bf16x8*)(Ks + j * 32 * kRowBytes + cof(ks));
      };
      auto v_frags = [&](const char* Ks, int j, bf16x8 (&vf)[2][2]) {
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
            vf[d][s2] = *(const bf16x8*)(Ks + 8192 + d * 32 * kRowBytes + cof(2 * j + s2));
      };
      auto score_chain = [&](const bf16x8 (&kf)[4]) {
        f32x16 sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0][0], negm[0], 0, 0, 0);
#pragma unroll
        for (int ks = 1; ks < 4; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[0][ks], sc, 0, 0, 0);
        return sc;
      };
      // exponentials, conversion and row sum of a block whose (s - m) are in sc, then its PV products
      auto finish_block = [&](const f32x16& sc, const bf16x8 (&vf)[2][2]) {
        bf16x8 pb[2];
        float psum = 0.f;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const bf16x2 pp = {(bf16)__builtin_amdgcn_exp2f(sc[8 * s2 + e]), (bf16)__builtin_amdgcn_exp2f(sc[8 * s2 + e + 1])};
            pb[s2][e] = pp[0]; pb[s2][e + 1] = pp[1];
            psum = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, psum, false);
          }
        l_run[0] += psum;
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2) o[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[d][s2], pb[s2], o[0][d], 0, 0, 0);
      };
      // One step: the scores of the next block from the K fragments the previous step fetched (kf_c), the exponentials,
      // row sum and PV products of the current block (scores in sc_c), and the fetch of the K fragments for the step after
      // (kf_n, from block (Kf, jf); Kf == nullptr: none).  open >= 0: that block opens tile `open`, which is waited for first.
      auto pipe_step = [&](const f32x16& sc_c, f32x16& sc_n, const bf16x8 (&kf_c)[4], bf16x8 (&kf_n)[4], const char* Kc, int jc,
                           const char* Kf, int jf, int open) {
        bf16x8 vf[2][2];
        v_frags(Kc, jc, vf);
        if (open >= 0) open_tile(open, open & (NSTG - 1));
        if (Kf) k_frags(Kf, jf, kf_n);
        sc_n = score_chain(kf_c);
        finish_block(sc_c, vf);
        // order: score MFMAs with the exponentials of the current block between them, then the PV MFMAs with what is left of the
        // conversions and row sums (transcendentals form a scheduling class of their own)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 4, 0);
          if (i > 0) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        }
      };
      f32x16 sc_a, sc_b;
      bf16x8 kf_a[4], kf_b[4];
      k_frags(lds, 1, kf_b);
      if (ntiles > 1) open_tile(1, 1);
      if (nfull > 1) k_frags(stage_of(1), 0, kf_a);
      sc_a = score_chain(kf_b);
      for (int t = 1; t < nfull; ++t) {
        // (t - 1, 1) is finished while (t, 0) is scored; then (t, 0) is finished while (t, 1) is scored and tile t + 1 opened
        pipe_step(sc_a, sc_b, kf_a, kf_b, stage_of(t - 1), 1, stage_of(t), 1, -1);
        const bool more = t + 1 < nfull;
        pipe_step(sc_b, sc_a, kf_b, kf_a, stage_of(t), 0, more ? stage_of(t + 1) : nullptr, 0, t + 1 < ntiles ? t + 1 : -1);
      }
      {   // the last full block has no successor to compute scores for
        bf16x8 vf[2][2];
        v_frags(stage_of(nfull - 1), 1, vf);
        finish_block(sc_a, vf);
      }
      if (RAGGED) {
        block(stage_of(ntiles - 1), ntiles - 1, 0, false);
        block(stage_of(ntiles - 1), ntiles - 1, 1, false);
      }
    }
    // did some score leave the window above the reference?  Then every wavefront of the workgroup starts over, checked.
    const float l_chk = l_run[0] + other_half(l_run[0], low);
    wait_vmcnt<0>();
    __syncthreads();
    if (tid == 0) s_redo = 0;
    __syncthreads();
    if (__builtin_amdgcn_ballot_w64(!(l_chk < kAttnBig)) != 0 && lane == 0) s_redo = 1;
    __syncthreads();
    if (s_redo != 0) {
      m_ref[0] = 0.f; l_run[0] = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) { o[0][0][r] = 0.f; o[0][1][r] = 0.f; negm[0][r] = 0.f; }
      issue(0, 0);
      if (ntiles > 1) issue(1, 1);
    }
    if (s_redo == 0) goto finished;
  }
  {
  int stage = 0;
  for (int t = t_first; t < t_first + t_each; ++t) {         // every group passes the same barriers
    open_tile(t, stage);
    if (KS == 1 || t < t_last) {
      const char* Ks = lds + stage * kAttn2Stage;
      block(Ks, t, 0, t == t_first);
      block(Ks, t, 1, false);
    }
    if (++stage == NSTG) stage = 0;
  }
  }
finished:
  if constexpr (KS > 1) {
    // the other groups hand their sums, references and denominators to the first one, a register of all lanes at a time
    __syncthreads();
    float* const hand = (float*)lds_all;
    auto at = [&](int g, int r) { return hand + (((g - 1) * NWQ + wave) * 34 + r) * 64 + lane; };
    if (group > 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { *at(group, r) = o[0][0][r]; *at(group, 16 + r) = o[0][1][r]; }
      *at(group, 32) = m_ref[0];
      *at(group, 33) = l_run[0];
    }
    __syncthreads();
    if (group > 0) return;
    float top = m_ref[0];
#pragma unroll
    for (int g = 1; g < KS; ++g) top = fmaxf(top, *at(g, 32));
    const float f0 = __builtin_amdgcn_exp2f(m_ref[0] - top);
    l_run[0] *= f0;
#pragma unroll
    for (int r = 0; r < 16; ++r) { o[0][0][r] *= f0; o[0][1][r] *= f0; }
#pragma unroll
    for (int g = 1; g < KS; ++g) {
      const float f = __builtin_amdgcn_exp2f(*at(g, 32) - top);
      l_run[0] += f * *at(g, 33);
#pragma unroll
      for (int r = 0; r < 16; ++r) { o[0][0][r] += f * *at(g, r); o[0][1][r] += f * *at(g, 16 + r); }
    }
  }
#pragma unroll
  for (int s = 0; s < QSETS; ++s) {
    const float l_tot = l_run[s] + other_half(l_run[s], low);
    const int query = q0 + 32 * s;
    if (query < L) {
      const float inv = 1.f / l_tot;
      bf16* orow = O + ((size_t)b * L + query) * ldo + h * 64;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (bf16)(o[s][d][4 * g + e] * inv);
          *(bf16x4*)(orow + d * 32 + 8 * g + 4 * half) = v;
        }
    }
  }
}

// Generic attention (fp32, other head widths, v in its own layout): fp32 arithmetic on the 16x16x4 MFMA whatever the storage type.
// A workgroup owns 16 queries of one (sample, head); its eight wavefronts take every eighth block of 16 keys with an online softmax
// of their own (these sequences are short, so the keys have to be shared out for the chip to see enough wavefronts) and are
// merged through LDS at the end.  Scores are computed transposed, S^T = K Q^T: a lane holds four keys (4 g + r) of query
// lane & 15, which is the B operand of O^T += V^T P^T as it stands.  No LDS before the merge.  DT: head width in units of 16;
// VEC: four consecutive elements of a row can be loaded at once.  Bound by the latency of the loads of a key block and its
// dependent softmax.
// fp32, two samples, heads of 64: 576 x 576, one head, 14.7 us; 144 x 144, two heads, 7.6 us; 4096 x 4096, one head, 156 us = 55 TFLOP/s
// (124, 31 and 1660 us with one wavefront per query, one key per lane).
template <typename T, int DT, bool VEC>
__global__ __launch_bounds__(512) void k_attn_generic(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, int v_t,
                                                      T* __restrict__ O, int L, int Lk, int C, int d, int ldq, int ldk, int ldv, int ldo,
                                                      float scale_log2) {
  constexpr int NW = 8, PITCH = 16 * DT + 4;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* const part = (float*)lds;                       // [wavefront][query][PITCH]: O, then m and l behind the head width
  typedef T V4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q16 = lane & 15, g = lane >> 4;
  const int b = blockIdx.z, h = blockIdx.y, q0 = blockIdx.x * 16;
  // elements 4 i .. 4 i + 3 of a row of the head, zero beyond the head width
  auto load4 = [&](const T* row, int i) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
      if (4 * i < d) {
        const V4 t = *(const V4*)(row + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = to_f(t[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * i + e < d) v[e] = to_f(row[4 * i + e]);
    }
    return v;
  };
  f32x4 qf[DT], o[DT];
  {
    const T* row = Q + ((size_t)b * L + min(q0 + q16, L - 1)) * ldq + h * d;
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      qf[t] = load4(row, 4 * t + g) * scale_log2;
      o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  float m = -INFINITY, l = 0.f;
  for (int key0 = wave * 16; key0 < Lk; key0 += NW * 16) {
    const T* krow = K + ((size_t)b * Lk + min(key0 + q16, Lk - 1)) * ldk + h * d;
    f32x4 kf[DT], vf[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) kf[t] = load4(krow, 4 * t + g);
    // V^T rows (channels 16 t + q16) at keys 4 g + r; the probability of a key past the end is zero, its value is never read
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      const int c = 16 * t + q16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = key0 + 4 * g + r;
        vf[t][r] = c < d && key < Lk ? to_f(v_t ? V[((size_t)b * C + h * d + c) * ldv + key] : V[((size_t)b * Lk + key) * ldv + h * d + c]) : 0.f;
      }
    }
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][e], qf[t][e], s, 0, 0, 0);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (key0 + 4 * g + r >= Lk) s[r] = -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // (as long as every score has been minus infinity there is no maximum to subtract: all terms are zero)
    const float m_new = fmaxf(m, mx), ref = m_new == -INFINITY ? 0.f : m_new, alpha = __builtin_amdgcn_exp2f(m - ref);
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) { s[r] = __builtin_amdgcn_exp2f(s[r] - ref); sum += s[r]; }
    l = l * alpha + sum;                                 // of this lane's keys; the four groups are added at the end
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      o[t] *= alpha;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][r], s[r], o[t], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  float* mine = part + (wave * 16 + q16) * PITCH;
#pragma unroll
  for (int t = 0; t < DT; ++t) *(f32x4*)(mine + 16 * t + 4 * g) = o[t];          // channels 16 t + 4 g + r of query q16
  if (g == 0) { mine[16 * DT] = m; mine[16 * DT + 1] = l; }
  __syncthreads();
  for (int i = tid; i < 16 * d; i += 64 * NW) {
    const int q = i / d, c = i - q * d;
    if (q0 + q >= L) break;
    float top = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) top = fmaxf(top, part[(w * 16 + q) * PITCH + 16 * DT]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* p = part + (w * 16 + q) * PITCH;
      const float f = __builtin_amdgcn_exp2f(p[16 * DT] - top);
      num += f * p[c];
      den += f * p[16 * DT + 1];
    }
    O[((size_t)b * L + q0 + q) * ldo + h * d + c] = from_f<T>(num / den);
  }
}

template <typename T>
static ad_status run_attn_generic(const void* q, const void* k, const void* v, int v_t, int batch, int l, int lk, int c, int d, int ldq,
                                  int ldk, int ldv, int ldo, void* out, float scale_log2, hipStream_t s) {
  const bool vec = d % 4 == 0 && (ldq | ldk) % 4 == 0 && (((uintptr_t)q | (uintptr_t)k) % (4 * sizeof(T))) == 0;
  const dim3 grid((l + 15) / 16, c / d, batch);
#define AD_ATTNG(DT_, VEC_)                                                                                                              \
  do {                                                                                                                                   \
    constexpr int lds_bytes = 8 * 16 * (16 * DT_ + 4) * 4;                                                                               \
    static std::atomic<bool> attr_set{false};                                                                                            \
    if (lds_bytes > 65536 && !attr_set) {                                                                                                \
      AD_HIP(hipFuncSetAttribute((const void*)k_attn_generic<T, DT_, VEC_>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));     \
      attr_set = true;                                                                                                                   \
    }                                                                                                                                    \
    hipLaunchKernelGGL((k_attn_generic<T, DT_, VEC_>), grid, dim3(512), lds_bytes, s, (const T*)q, (const T*)k, (const T*)v, v_t,        \
                       (T*)out, l, lk, c, d, ldq, ldk, ldv, ldo, scale_log2);                                                            \
  } while (0)
#define AD_ATTNG_D(VEC_)                 \
  if (d <= 16) AD_ATTNG(1, VEC_);        \
  else if (d <= 32) AD_ATTNG(2, VEC_);   \
  else if (d <= 64) AD_ATTNG(4, VEC_);   \
  else AD_ATTNG(8, VEC_)
  if (vec) { AD_ATTNG_D(true); } else { AD_ATTNG_D(false); }
#undef AD_ATTNG_D
#undef AD_ATTNG
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// which MFMA attention kernel: 0 = first generation (32 queries per wavefront, register-staged tiles), 1 / 2 = second
// generation with 32 / 64 queries per wavefront; -1 = automatic
static int g_attn_variant = -1;
void set_attn_variant(int v) { g_attn_variant = v; }
static int attn_auto_variant(int bh, int l, int lk) {
  // measured on the self-attention shapes of the SD-sized models: the second-generation kernel with 32 queries per
  // wavefront is 8-20 % faster from a few hundred keys on; with one or two key tiles (cross-attention to the text,
  // the deepest level) its longer prologue loses, and 64 queries per wavefront (two wavefronts per SIMD) never won.
  // The pipelined variant (3) is 4-10 % faster launched alone and 1 % slower inside the concurrent schedule (its 64 KiB of
  // LDS and two wavefronts per SIMD leave less room for the other streams' workgroups), so it stays a selectable variant.
  // Up to 512 workgroups, where no CU gets a third one anyway, it is 6-12 % faster alone (two samples, 4096 tokens, 5 heads 70.6 -> 62.8 us,
  // 2304, 10 heads 45.3 -> 41.3) and whole runs of two and four components are level.
  (void)bh; (void)l;
  return lk > 256 ? 1 : 0;
}

// Where 64-query workgroups fit the chip once, the plain launch (128 queries) leaves half of it idle: 64 queries and two key halves a
// workgroup instead, which halves the chain of key tiles as well.  One sample, us (128 queries -> this): 2880 x 2880, 5 heads, 36.6 -> 25.0;
// 1536, 10 heads, 21.6 -> 14.4; 720, 10 heads, 14.2 -> 10.0; 640, 20 heads, 11.2 -> 8.2.  Up to 400 workgroups, where some CUs get two, it is still faster
// alone, by less: 1024, 20 heads 15.2 / 14.1, 2304, 10 heads 29.0 / 25.9, 5120, 5 heads 59.2 / 51.4, 576, 2 x 20 heads 10.4 / 10.2; but whole runs with the
// line there are level (512px 0.3 % faster, 768px and 576x320 px 0.0, 768px wrapped 0.6 faster with runs of one side 0.8 apart), so it stays where no CU holds
// more than one.  Far beyond it falls behind (9216, 2 x 5 heads: 230 / 268, keys and values are fetched twice as often).  Four key shares with 128 KiB of LDS
// gain another tenth from 1500 keys on, but leave the other streams' workgroups no room.
static bool attn_split(int bh, int l) { return (long long)bh * ((l + 63) / 64) <= 256; }

ad_status launch_attention(int dtype, const void* q, const void* k, const void* v, int v_t, int batch, int l, int lk, int c,
                           int head_dim, int ldq, int ldk, int ldv, int ldo, void* out, hipStream_t s) {
  if (!q || !k || !v || !out) AD_FAIL(AD_ERR_INVALID, "attention: null pointer");
  if (batch < 1 || l < 1 || lk < 1 || head_dim < 1 || head_dim > 128 || c % head_dim) AD_FAIL(AD_ERR_INVALID, "attention: bad shape");
  if (ldq < c || ldk < c || ldo < c || (v_t ? ldv < lk : ldv < c)) AD_FAIL(AD_ERR_INVALID, "attention: bad leading dimension");
  const int heads = c / head_dim;
  if (heads > 65535 || batch > 65535) AD_FAIL(AD_ERR_INVALID, "attention: too many heads/batches");
  const float scale = 1.f / sqrtf((float)head_dim);
  if (dtype == AD_BF16 && head_dim == 64 && v_t) {
    if (ldv < round_up(lk, 64) || (ldq | ldk | ldv | ldo) % 8) AD_FAIL(AD_ERR_INVALID, "attention: MFMA path needs padded, 8-aligned strides");
    // the kernel walks K and V^T with 32-bit element offsets from the (sample, head) base
    if ((long long)(lk + 64) * ldk >= (1LL << 32) || 64LL * ldv + lk >= (1LL << 32)) AD_FAIL(AD_ERR_INVALID, "attention: key tensor too large");
    int variant = g_attn_variant;
    if (variant < 0) variant = attn_auto_variant(batch * heads, l, lk);
    // the two kernel generations are separate classes for the per-launch timing, as they are separate kernels in a trace
    ProfLaunch pl(variant > 0 ? "attn_mfma2_bf16" : "attn_mfma_bf16", 4.0 * batch * l * lk * c, 2.0 * batch * c * (2.0 * l + 2.0 * lk), s,
                  batch * l, lk, c);
    if (variant > 0) {
      // the tile loads address K and V^T through 32-bit byte offsets from the (sample, head) base
      if (((long long)(lk + 64) * ldk + 64) * 2 >= (1LL << 31) || (64LL * ldv + lk + 64) * 2 >= (1LL << 31))
        AD_FAIL(AD_ERR_INVALID, "attention: key tensor too large");
      if ((((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) & 15) != 0) AD_FAIL(AD_ERR_INVALID, "attention: pointers must be 16-byte aligned");
      const float sl2 = scale * 1.44269504088896341f;
      auto run = [&](auto kern, int queries, int waves, int stages) {
        static_assert(4 * kAttn2Stage <= 65536, "what a launch gets without asking");
        const int qb = (l + queries - 1) / queries;
        hipLaunchKernelGGL(kern, dim3(qb * heads * batch), dim3(64 * waves), stages * kAttn2Stage, s, (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)out, l, lk, c,
                           ldq, ldk, ldv, ldo, sl2, qb);
      };
      const bool ragged = (lk & 63) != 0;
      if (variant == 3) ragged ? run(k_attn_mfma2<1, true, 4, 2, 1>, 128, 4, 4) : run(k_attn_mfma2<1, false, 4, 2, 1>, 128, 4, 4);
      else if (variant == 2) ragged ? run(k_attn_mfma2<2, true>, 256, 4, 3) : run(k_attn_mfma2<2, false>, 256, 4, 3);
      else if (g_attn_variant < 0 && attn_split(batch * heads, l)) ragged ? run(k_attn_mfma2<1, true, 2, 2, 0, 2, 2>, 64, 4, 4) : run(k_attn_mfma2<1, false, 2, 2, 0, 2, 2>, 64, 4, 4);
      else ragged ? run(k_attn_mfma2<1, true>, 128, 4, 3) : run(k_attn_mfma2<1, false>, 128, 4, 3);
      AD_HIP(hipGetLastError());
      return AD_OK;
    }
    const int qblocks = (l + 127) / 128;
    if (lk & 63)
      hipLaunchKernelGGL(k_attn_mfma<true>, dim3(qblocks * heads * batch), dim3(256), 0, s, (const bf16*)q, (const bf16*)k,
                         (const bf16*)v, (bf16*)out, l, lk, c, ldq, ldk, ldv, ldo, scale * 1.44269504088896341f, qblocks);
    else
      hipLaunchKernelGGL(k_attn_mfma<false>, dim3(qblocks * heads * batch), dim3(256), 0, s, (const bf16*)q, (const bf16*)k,
                         (const bf16*)v, (bf16*)out, l, lk, c, ldq, ldk, ldv, ldo, scale * 1.44269504088896341f, qblocks);
  } else if (dtype == AD_BF16) {
    ProfLaunch pl("attn_generic_bf16", 4.0 * batch * l * lk * c, 2.0 * batch * c * (2.0 * l + 2.0 * lk), s);
    return run_attn_generic<bf16>(q, k, v, v_t, batch, l, lk, c, head_dim, ldq, ldk, ldv, ldo, out, scale * 1.44269504088896341f, s);
  } else if (dtype == AD_F32) {
    ProfLaunch pl("attn_generic_f32", 4.0 * batch * l * lk * c, 4.0 * batch * c * (2.0 * l + 2.0 * lk), s);
    return run_attn_generic<float>(q, k, v, v_t, batch, l, lk, c, head_dim, ldq, ldk, ldv, ldo, out, scale * 1.44269504088896341f, s);
  } else {
    AD_FAIL(AD_ERR_INVALID, "attention: bad dtype");
  }
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// Attention over the frame axis of a video model: the tokens of one sequence are the `frames` rows (f, p),
// f = 0..frames-1, of one spatial position p; row (f, p) of q / k / v / out is f * positions + p.  One wavefront
// per (position, head): q, k and v of its `frames` x d slice are staged in LDS with coalesced reads (row stride
// padded to an odd number of 32-bit words), lane 4 f + part owns the channels t = part (mod 4) of frame f,
// partial scores are folded over the four parts with two lane exchanges, the softmax lives in registers.
constexpr int kMaxFrames = 16;

template <typename T>
__global__ __launch_bounds__(256) void k_attn_frames(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                                                     T* __restrict__ O, int frames, int positions, int heads, int d, int ds,
                                                     int ldq, int ldk, int ldv, int ldo, float scale) {
  extern __shared__ __align__(16) char frames_lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const long long item = (long long)blockIdx.x * waves + wave;
  const bool active = item < (long long)positions * heads;
  const int p = active ? (int)(item / heads) : 0, h = active ? (int)(item % heads) : 0;
  T* qs = (T*)frames_lds + (size_t)wave * 3 * kMaxFrames * ds;
  T* ks = qs + kMaxFrames * ds;
  T* vs = ks + kMaxFrames * ds;
  if (active) {
    for (int idx = lane; idx < frames * d; idx += 64) {
      const int f = idx / d, t = idx - f * d;
      const size_t row = (size_t)f * positions + p;
      qs[f * ds + t] = Q[row * ldq + h * d + t];
      ks[f * ds + t] = K[row * ldk + h * d + t];
      vs[f * ds + t] = V[row * ldv + h * d + t];
    }
  }
  __syncthreads();
  if (!active) return;
  const int f = lane >> 2, part = lane & 3;
  const bool mine = f < frames;
  float sc[kMaxFrames];
#pragma unroll
  for (int j = 0; j < kMaxFrames; ++j) sc[j] = 0.f;
  if (mine)
    for (int t = part; t < d; t += 4) {
      const float qv = to_f(qs[f * ds + t]);
#pragma unroll
      for (int j = 0; j < kMaxFrames; ++j)
        if (j < frames) sc[j] += qv * to_f(ks[j * ds + t]);
    }
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < kMaxFrames; ++j) {
    sc[j] += __shfl_xor(sc[j], 1);
    sc[j] += __shfl_xor(sc[j], 2);
    sc[j] *= scale;
    if (j < frames) m = fmaxf(m, sc[j]);
  }
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < kMaxFrames; ++j) {
    sc[j] = j < frames ? __expf(sc[j] - m) : 0.f;
    sum += sc[j];
  }
  if (!mine) return;
  const float inv = 1.f / sum;
  T* orow = O + ((size_t)f * positions + p) * ldo + h * d;
  for (int t = part; t < d; t += 4) {
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < kMaxFrames; ++j)
      if (j < frames) acc += sc[j] * to_f(vs[j * ds + t]);
    orow[t] = from_f<T>(acc * inv);
  }
}

// The same for bf16 on the matrix cores, without LDS: one wavefront per (position, head).  Scores are computed
// transposed, S^T = K Q^T, with 16x16x32 MFMAs whose operands are 16-byte row segments straight from global
// memory (lane = frame + 16 * segment); lane (f, g) then holds S^T[4g..4g+3][f], which is exactly the A-operand
// layout of the 16x16x16 MFMA that multiplies the probabilities with V (B operand: four 2-byte loads per lane and
// 16-channel step).  Frames beyond `frames` are zero rows with -inf scores.  Needs d % 8 == 0, 16-byte aligned rows.
typedef short s16x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_attn_frames_mfma(const bf16* __restrict__ Q, const bf16* __restrict__ K,
                                                          const bf16* __restrict__ V, bf16* __restrict__ O, int frames,
                                                          int positions, int heads, int d, int ldq, int ldk, int ldv, int ldo,
                                                          float scale_log2e) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long item = (long long)blockIdx.x * 4 + wave;
  if (item >= (long long)positions * heads) return;          // the kernel has no barrier: a wavefront may leave
  const int p = (int)(item / heads), h = (int)(item % heads);
  const int r = lane & 15, g = lane >> 4;
  const bool row_ok = r < frames;
  const size_t row = (size_t)(row_ok ? r : 0) * positions + p;
  const bf16* qrow = Q + row * ldq + h * d;
  const bf16* krow = K + row * ldk + h * d;
  f32x4 st = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < d; k0 += 32) {
    const int kk = k0 + 8 * g;
    bf16x8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) { a[e] = (bf16)0.f; b[e] = (bf16)0.f; }
    if (row_ok && kk < d) {
      a = *(const bf16x8*)(krow + kk);
      b = *(const bf16x8*)(qrow + kk);
    }
    st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, st, 0, 0, 0);
  }
  // st[i] = q_f . k_j for key j = 4g + i and query f = r
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    st[i] = (4 * g + i) < frames ? st[i] * scale_log2e : -INFINITY;
    m = fmaxf(m, st[i]);
  }
  m = fmaxf(m, __shfl_xor(m, 16));
  m = fmaxf(m, __shfl_xor(m, 32));
  float sum = 0.f;
  bf16x4 pb;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float e = exp2f(st[i] - m);
    sum += e;
    pb[i] = (bf16)e;
  }
  sum += __shfl_xor(sum, 16);
  sum += __shfl_xor(sum, 32);
  const float inv = 1.f / sum;                                // of query r; the output rows of this lane are 4g..4g+3
  float inv_f[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) inv_f[i] = __shfl(inv, 4 * g + i);
  const s16x4 pa = __builtin_bit_cast(s16x4, pb);
  for (int t0 = 0; t0 < d; t0 += 16) {
    const int t = t0 + r;
    bf16x4 vb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = 4 * g + i;
      vb[i] = (t < d && j < frames) ? V[((size_t)j * positions + p) * ldv + h * d + t] : (bf16)0.f;
    }
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    o = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, __builtin_bit_cast(s16x4, vb), o, 0, 0, 0);
    if (t < d) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int f = 4 * g + i;
        if (f < frames) O[((size_t)f * positions + p) * ldo + h * d + t] = (bf16)(o[i] * inv_f[i]);
      }
    }
  }
}

ad_status launch_attention_frames(int dtype, const void* q, const void* k, const void* v, int frames, int positions, int c,
                                  int heads, int ldq, int ldk, int ldv, int ldo, void* out, hipStream_t s) {
  if (!q || !k || !v || !out) AD_FAIL(AD_ERR_INVALID, "frame attention: null pointer");
  if (dtype != AD_BF16 && dtype != AD_F32) AD_FAIL(AD_ERR_INVALID, "frame attention: bad dtype");
  if (frames < 1 || frames > kMaxFrames) AD_FAIL(AD_ERR_INVALID, "frame attention: 1..%d frames", kMaxFrames);
  if (positions < 1 || heads < 1 || c < 1 || c % heads) AD_FAIL(AD_ERR_INVALID, "frame attention: bad shape");
  if (ldq < c || ldk < c || ldv < c || ldo < c) AD_FAIL(AD_ERR_INVALID, "frame attention: bad leading dimension");
  const int d = c / heads;
  const size_t es = esize(dtype);
  const long long items = (long long)positions * heads;
  if ((items + 3) / 4 > 0x7fffffffLL) AD_FAIL(AD_ERR_INVALID, "frame attention: too many positions");
  const float scale = 1.f / sqrtf((float)d);
  const bool aligned16 = (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) & 15) == 0;
  if (dtype == AD_BF16 && d % 8 == 0 && (ldq | ldk | ldv | ldo) % 8 == 0 && aligned16) {
    ProfLaunch pl("attn_frames_bf16", 4.0 * positions * frames * frames * c, 4.0 * es * positions * frames * c, s,
                  positions * frames, frames, c);
    hipLaunchKernelGGL(k_attn_frames_mfma, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, (const bf16*)q, (const bf16*)k,
                       (const bf16*)v, (bf16*)out, frames, positions, heads, d, ldq, ldk, ldv, ldo, scale * 1.44269504088896341f);
    AD_HIP(hipGetLastError());
    return AD_OK;
  }
  int ds = d;                                             // LDS row stride: a whole, odd number of 32-bit words
  while ((ds * es) % 4 || ((ds * es) / 4) % 2 == 0) ++ds;
  const size_t per_wave = (size_t)3 * kMaxFrames * ds * es;
  if (per_wave > 65536) AD_FAIL(AD_ERR_INVALID, "frame attention: head width %d too large", d);
  const int waves = (int)std::min<size_t>(4, 65536 / per_wave);
  const long long blocks = (items + waves - 1) / waves;
  ProfLaunch pl(dtype == AD_BF16 ? "attn_frames_generic_bf16" : "attn_frames_f32", 4.0 * positions * frames * frames * c,
                4.0 * es * positions * frames * c, s, positions * frames, frames, c);
  if (dtype == AD_BF16)
    hipLaunchKernelGGL(k_attn_frames<bf16>, dim3((unsigned)blocks), dim3(64 * waves), waves * per_wave, s, (const bf16*)q, (const bf16*)k,
                       (const bf16*)v, (bf16*)out, frames, positions, heads, d, ds, ldq, ldk, ldv, ldo, scale);
  else
    hipLaunchKernelGGL(k_attn_frames<float>, dim3((unsigned)blocks), dim3(64 * waves), waves * per_wave, s, (const float*)q, (const float*)k,
                       (const float*)v, (float*)out, frames, positions, heads, d, ds, ldq, ldk, ldv, ldo, scale);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// =================================================================================================
// GroupNorm (+SiLU), NHWC.  Maps whose groups fit a workgroup's registers take one launch (k_gn_group below), larger ones two.
// Pass 1: every workgroup reduces a run of pixels of one source to per-channel (sum, sum of squares) with fully
// coalesced row reads, eight rows in flight per thread, and folds the channels of each group in a fixed order: one
// (sum, sumsq) pair per (source, sample, pixel chunk, group); both sources of a concatenation in one launch.  Pass 2:
// every workgroup first folds those pairs of its sample in double precision (a few KiB, L2-resident) into mean and 1/std
// per group, then applies y = silu(x * scale + shift) to its run of pixels.  No atomics, no fences: the result does not
// depend on scheduling.  Both passes are bound by the latency of a launch (3.5 us for any map) and of the memory system
// rather than by bandwidth at these sizes: 96x96x320, two samples, 15.3 us for 35 MB (19.4 with 64 chunks, four rows in
// flight and a serial fold of the channels); 96x96x(320+320) 19.5 us (34.5 with a launch per source).
// =================================================================================================
constexpr int kGnMaxGroups = 256;

// pixel chunks of the statistics pass: 64, or 128 (a workgroup on every CU with two samples) where the partial sums of both sources
// still fit the library's own 512 KiB array and the caller's scratch (64 chunks of as many groups as there are channels, so two
// channels a group)
constexpr int kGnScratchChunks = 64;
constexpr size_t kStaticGnBytes = 512 * 1024;
static int gn_chunks(int batch, int hw, int groups, int c) {
  const int most = c >= 2 * groups && (size_t)2 * batch * 2 * kGnScratchChunks * groups * 2 * sizeof(float) <= kStaticGnBytes ? 2 * kGnScratchChunks : kGnScratchChunks;
  const int n = hw / 8;
  return n < 1 ? 1 : (n > most ? most : n);
}

// gpart layout: [source 0/1][sample][chunk][group][2]; blockIdx.z = source
template <typename T>
__global__ __launch_bounds__(256) void k_gn_partial(const T* __restrict__ src0, const T* __restrict__ src1, int c0, int c1, int hw,
                                                    int nchunk, int groups, int cpg, size_t src_stride, float* __restrict__ gpart) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  __shared__ float2 red[256 * VN];
  __shared__ float2 fold[256];
  const int chunk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const T* src = blockIdx.z ? src1 : src0;
  const int cs = blockIdx.z ? c1 : c0, coff = blockIdx.z ? c0 : 0;
  const int p0 = (int)((long long)hw * chunk / nchunk), p1 = (int)((long long)hw * (chunk + 1) / nchunk);
  const int nv = cs / VN;
  const int cvb = nv < 256 ? nv : 256;      // column vectors handled per pass
  const int pl = 256 / cvb;                 // pixel lanes
  const int cv = tid % cvb, lanep = tid / cvb;
  // channels -> groups: thread (group, part) adds every parts-th channel of its group, over the pixel lanes in order; a group may
  // extend into the other source, which adds its own pair
  const int parts = 256 / groups, g = tid / parts, part = tid - g * parts;
  const int lo = max(g * cpg, coff) - coff, hi = g < groups ? min((g + 1) * cpg, coff + cs) - coff : 0;
  float gs = 0.f, gq = 0.f;
  for (int cb = 0; cb < nv; cb += cvb) {
    float s[VN], q[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) { s[e] = 0.f; q[e] = 0.f; }
    const bool on = lanep < pl && cb + cv < nv;
    if (on) {
      constexpr int UN = 8;                     // rows in flight per thread; summed in row order
      const T* sp = src + (size_t)b * hw * cs + (size_t)(cb + cv) * VN;
      for (int p = p0 + lanep; p < p1; p += pl * UN) {
        V v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u)
          if (p + u * pl < p1) v[u] = *(const V*)(sp + (size_t)(p + u * pl) * cs);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          if (p + u * pl >= p1) break;
#pragma unroll
          for (int e = 0; e < VN; ++e) { const float f = to_f(v[u][e]); s[e] += f; q[e] += f * f; }
        }
      }
    }
    if (cb > 0) __syncthreads();                // the previous block of channels has been folded
#pragma unroll
    for (int e = 0; e < VN; ++e) red[e * 256 + tid] = make_float2(s[e], q[e]);
    __syncthreads();
    const int c_end = min(hi, min(nv, cb + cvb) * VN);
    for (int j = 0; j < pl; ++j)
      for (int c = max(lo, cb * VN) + part; c < c_end; c += parts) {
        const float2 v = red[(c % VN) * 256 + j * cvb + c / VN - cb];
        gs += v.x; gq += v.y;
      }
  }
  fold[tid] = make_float2(gs, gq);
  __syncthreads();
  if (part == 0 && lo < hi) {
    for (int j = 1; j < parts; ++j) { gs += fold[tid + j].x; gq += fold[tid + j].y; }
    *(float2*)(gpart + blockIdx.z * src_stride + (((size_t)b * nchunk + chunk) * groups + g) * 2) = make_float2(gs, gq);
  }
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_gn_apply(const T* __restrict__ src0, const T* __restrict__ src1, int c0, int c1, int hw,
                                                  int rows_per_block, int nchunk, int groups, const float* __restrict__ gpart,
                                                  size_t src_stride, FastDiv div_cpg, const float* __restrict__ gamma,
                                                  const float* __restrict__ beta, float eps, int silu, T* __restrict__ out) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  __shared__ double2 dred[NT];
  __shared__ float smean[kGnMaxGroups], srstd[kGnMaxGroups];
  const int tid = threadIdx.x, b = blockIdx.y;
  const int ctot = c0 + c1, cpg = ctot / groups;
  const int nv = ctot / VN;
  const int cvb = nv < NT ? nv : NT, pl = NT / cvb;
  const int cv = tid % cvb, lanep = tid / cvb;
  const int r0 = blockIdx.x * rows_per_block, r1 = min(hw, r0 + rows_per_block);
  // a thread's channels, their gain and offset, and its rows: UN in flight, requested one step ahead (the first before the statistics)
  constexpr int UN = 4;
  V v[UN];
  float ga[VN], be[VN];
  int c = 0;
  size_t ld = 0;
  const T* sp = nullptr;
  auto rows_from = [&](int p) {
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (p + u * pl < r1) v[u] = *(const V*)(sp + ((size_t)b * hw + p + u * pl) * ld);
  };
  auto request = [&](int cb) {
    if (lanep >= pl || cb + cv >= nv) return false;
    c = (cb + cv) * VN;
    sp = c < c0 ? src0 + c : src1 + (c - c0);
    ld = c < c0 ? c0 : c1;
    rows_from(r0 + lanep);
#pragma unroll
    for (int e = 0; e < VN; ++e) { ga[e] = gamma[c + e]; be[e] = beta[c + e]; }
    return true;
  };
  bool on = request(0);
  // statistics of this sample: thread (part, group) sums every parts-th chunk; the parts are folded in order, in two steps
  const int gw = groups < NT ? groups : NT, parts = NT / gw, quarter = (parts + 3) / 4;
  for (int g0 = 0; g0 < groups; g0 += NT) {
    const int g = g0 + tid % gw, part = tid / gw;
    double s = 0.0, q = 0.0;
    if (g < groups && part < parts) {
      // (both sources only where the group straddles them)
      for (int z = g * cpg < c0 ? 0 : 1; z <= ((g + 1) * cpg > c0 ? 1 : 0); ++z) {
        const float2* gp = (const float2*)(gpart + z * src_stride) + (size_t)b * nchunk * groups + g;
        constexpr int UN = 4;
        for (int ch = part; ch < nchunk; ch += parts * UN) {
          float2 t[UN];
#pragma unroll
          for (int u = 0; u < UN; ++u) t[u] = ch + u * parts < nchunk ? gp[(size_t)(ch + u * parts) * groups] : make_float2(0.f, 0.f);
#pragma unroll
          for (int u = 0; u < UN; ++u) { s += t[u].x; q += t[u].y; }
        }
      }
    }
    dred[tid] = make_double2(s, q);
    __syncthreads();
    if (part < 4) {
      for (int j = max(1, part * quarter); j < min(parts, (part + 1) * quarter); ++j) {
        const double2 d = dred[j * gw + tid % gw];
        if (j == part * quarter) { s = d.x; q = d.y; } else { s += d.x; q += d.y; }
      }
    }
    __syncthreads();
    if (part < 4) dred[tid] = make_double2(s, q);
    __syncthreads();
    if (part == 0 && g < groups) {
      for (int j = 1; j < 4 && j * quarter < parts; ++j) { s += dred[j * gw + tid].x; q += dred[j * gw + tid].y; }
      const double n = (double)hw * cpg;
      const double mean = s / n;
      double var = q / n - mean * mean;
      if (var < 0) var = 0;
      smean[g] = (float)mean;
      srstd[g] = (float)(1.0 / sqrt(var + (double)eps));
    }
    __syncthreads();
  }
  for (int cb = 0; cb < nv; cb += cvb) {
    if (cb > 0) on = request(cb);
    if (!on) continue;
#pragma unroll
    for (int e = 0; e < VN; ++e) {
      const int g = (int)fast_div((unsigned)(c + e), div_cpg);
      ga[e] *= srstd[g];
      be[e] -= smean[g] * ga[e];
    }
    for (int p = r0 + lanep; p < r1; p += pl * UN) {
      V x[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) x[u] = v[u];
      rows_from(p + pl * UN);
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        if (p + u * pl >= r1) break;
        V o;
#pragma unroll
        for (int e = 0; e < VN; ++e) {
          float y = to_f(x[u][e]) * ga[e] + be[e];
          if (silu) y = silu_f(y);
          o[e] = from_f<T>(y);
        }
        *(V*)(out + ((size_t)b * hw + p + u * pl) * ctot + c) = o;
      }
    }
  }
}

// GroupNorm in one launch: a workgroup keeps the (C/G) x HW elements of one (sample, group) in registers, reduces them and writes the
// normalised result, so nothing goes through scratch memory.  2^log_parts workgroups take in the same group (see launch_gn_group()), each
// writes every 2^log_parts-th of a thread's accesses: with log_parts > 0 out must not overlap a source, which another one may still read.  G: channels per
// access (the widest that divides the channels of a group), NV: accesses a thread can hold; thread (pixel lane, access of the pixel)
// walks the pixels in steps of `pl`, so its channels stay the same.
// Neighbouring groups share cache lines: xcd_remap puts them on one XCD.  Bound by one round trip to memory and the launch.
template <typename T, int G, int NT, int NV>
__global__ __launch_bounds__(NT) void k_gn_group(const T* __restrict__ src0, const T* __restrict__ src1, int c0, int c1, int hw,
                                                 int groups, int pl, int log_parts, double inv_n, const float* __restrict__ gamma,
                                                 const float* __restrict__ beta, float eps, int silu, T* __restrict__ out) {
  typedef T V __attribute__((ext_vector_type(G)));
  __shared__ float red[3][NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wg = xcd_remap(blockIdx.x, gridDim.x), vid = wg >> log_parts, mask = (1 << log_parts) - 1, part = wg & mask;
  const int b = vid / groups, g = vid - b * groups;
  const int ctot = c0 + c1, cpg = ctot / groups, vpp = cpg / G;
  const int lanep = tid / vpp, c = g * cpg + (tid - lanep * vpp) * G;
  const bool second = c >= c0;                           // an access never straddles the sources: both widths are multiples of G
  const int ld = second ? c1 : c0;
  const T* src = (second ? src1 + (c - c0) : src0 + c) + (size_t)b * hw * ld;
  const int p_end = lanep < pl ? hw : 0;
  V x[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int p = lanep + k * pl;
    if (p < p_end) x[k] = *(const V*)(src + (size_t)p * ld);
  }
  float ga[G], be[G];
#pragma unroll
  for (int e = 0; e < G; ++e) { ga[e] = p_end ? gamma[c + e] : 0.f; be[e] = p_end ? beta[c + e] : 0.f; }
  // The mean first, to the 12 leading bits (x less it is then exact but for a few elements), then the sums of the deviations from it and of
  // their squares: nothing cancels whatever the offset and the outliers.  The wavefronts' sums are folded in double, as in the two
  // launches.  gn_stats() keeps to this order of the sums.
  float s = 0.f, q = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k)
    if (lanep + k * pl < p_end)
#pragma unroll
      for (int e = 0; e < G; ++e) s += to_f(x[k][e]);
  s = wave_sum_rows(s);
  if (lane == 0) red[0][wave] = s;
  __syncthreads();
  s = 0.f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) s += red[0][w];
  float about = gn_about(s, inv_n);
  s = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k)
    if (lanep + k * pl < p_end) gn_add<0, G>(x[k], about, s, q, k == 0);
  s = wave_sum_rows(s); q = wave_sum_rows(q);
  if (lane == 0) { red[1][wave] = s; red[2][wave] = q; }
  __syncthreads();
  double ds = 0.0, dq = 0.0;
#pragma unroll 4
  for (int w = 0; w < NT / 64; ++w) { ds += red[1][w]; dq += red[2][w]; }
  float rstd, rest;
  gn_moments(ds, dq, inv_n, eps, rstd, rest);
#pragma unroll
  for (int e = 0; e < G; ++e) { ga[e] *= rstd; be[e] = fmaf(-rest, ga[e], be[e]); }
  asm volatile("" : "+v"(about));                        // x - about is formed anew: kept from the sums on, 48 elements would not fit
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int p = lanep + k * pl;
    if ((k & mask) == part && p < p_end) {
      V o;
#pragma unroll
      for (int e = 0; e < G; ++e) {
        float y = gn_value(to_f(x[k][e]), about, ga[e], be[e]);
        if (silu) y = silu_f(y);
        o[e] = from_f<T>(y);
      }
      *(V*)(out + ((size_t)b * hw + p) * ctot + c) = o;
    }
  }
}

}  // namespace ad

extern "C" size_t ad_groupnorm_scratch_bytes(int batch, int hw, int c) {
  (void)hw;
  // two sources x (sum, sum of squares) per chunk and group: 64 chunks of up to c groups, or 128 of up to c / 2 (gn_chunks)
  return (size_t)batch * ad::kGnScratchChunks * c * 4 * sizeof(float);
}

namespace ad {

constexpr long long kGnPartElements = 2048;
template <typename T, int NT, int REGS>
static ad_status launch_gn_group(const void* src0, const void* src1, int c0, int c1, int batch, int hw, int groups, int ga,
                                 const float* gamma, const float* beta, float eps, int silu, void* out, hipStream_t s) {
  const int ctot = c0 + c1, pl = NT / (ctot / groups / ga);
  constexpr int VN = Vec<T>::N;
  ProfLaunch prof("gn_group", 0, 2.0 * batch * hw * ctot * sizeof(T), s, batch * hw, ctot, 0);
  // The groups of a single sample are 32 workgroups that spend half their time on the result, 14 vector instructions an element against 6 of the
  // sums: up to four take all of a group in and write a part of it each, as long as that is a few thousand elements.  One sample, us: 2880 pixels
  // of 320 channels 15.7 -> 12.6, 720 of 640 6.2 -> 5.6, 720 of 1280 10.8 -> 9.2; the 576x320 px run 66.1 -> 64.9 ms.  Two samples' groups gain
  // 5-10 % alone as well (2304 of 640 13.8 -> 12.7), but take the CUs that other streams use: 768px runs 0.7 % slower.  One sample beside other
  // streams, whole runs (one workgroup a group / this): 576x320 px on two streams 62.5 / 61.4 ms, on four 52.5 / 52.6, 320px 45.4 / 44.8, 512px 60.4 / 60.0,
  // 768px 99.8 / 100.1.  In place, a group belongs to one workgroup.
  const long long elements = (long long)hw * (ctot / groups), rows = (long long)batch * hw;
  auto apart = [&](const void* src, int c) {
    const char *a = (const char*)src, *o = (const char*)out;
    return c == 0 || a + rows * c * sizeof(T) <= o || o + rows * ctot * sizeof(T) <= a;
  };
  const bool shared = groups * batch <= 32 && apart(src0, c0) && apart(src1, c1);
  int log_parts = 0;
  while (shared && log_parts < 2 && elements >> (log_parts + 1) >= kGnPartElements) ++log_parts;
  const dim3 grid((groups * batch) << log_parts);
  const double inv_n = 1.0 / ((double)hw * (ctot / groups));
#define AD_GN(G_) hipLaunchKernelGGL((k_gn_group<T, G_, NT, REGS * 4 / (G_ * (int)sizeof(T))>), grid, dim3(NT), 0, s, (const T*)src0, (const T*)src1, \
                                     c0, c1, hw, groups, pl, log_parts, inv_n, gamma, beta, eps, silu, (T*)out)
  if (ga == VN) AD_GN(VN);
  else if (ga == VN / 2) AD_GN(VN / 2);
  else AD_GN(VN / 4);
#undef AD_GN
  AD_HIP(hipGetLastError());
  return AD_OK;
}

template <typename T>
static ad_status run_groupnorm(const void* src0, const void* src1, int c0, int c1, int batch, int hw, int groups,
                               const float* gamma, const float* beta, float eps, int silu, void* out, void* scratch,
                               hipStream_t s) {
  const int ctot = c0 + c1, nchunk = gn_chunks(batch, hw, groups, ctot);
  const int cpg = ctot / groups;
  // One launch where a workgroup can hold a group of a sample in registers and has few enough accesses and elements to get through; two
  // launches spread a large group over more CUs.  Up to 96 workgroups most CUs have nothing to do, up to 256 one launch keeps the chip
  // busy as well, beyond that its workgroups wait for or share a CU.  More groups than the two launches take always go this way.
  // Measured on both sides of the line (32 groups, launches back to back, us, one launch / two): two samples, bf16: 24x24x1280 8.8 / 10.6,
  // 48x48x320 9.9 / 11.3, 48x48x640 12.2 / 11.9, 72x40x320 (14400 accesses) 11.8 / 11.4, 64x64x320 (20480) 17.7 / 11.7, 32x32x1920 (61440
  // elements) 14.3 / 12.7, 48x48x1280 21.1 / 14.9, narrow models 5.5 / 12; fp32: 32x32x1280 12.2 / 13.7, 48x48x640 14.7 / 13.5; eight samples:
  // 48x48x640 16.0 / 19.9, 64x64x320 21.3 / 19.2; sixteen: 32x32x640 15.2 / 18.8, 48x48x320 21.3 / 19.8, 64x64x128 21.5 / 17.6.
  // Up to 96 workgroups the line lies where two launches are a seventh faster, not where both are even: they take every CU, one launch
  // leaves the rest to the other streams (with 40960 elements and 12288 accesses whole 768px runs of four components lost 1 %).
  int ga = Vec<T>::N;                                        // channels per access: the widest that divides a group
  while (ga > 1 && cpg % ga) ga >>= 1;
  const int wgs = batch * groups;
  const long long accesses = (long long)hw * (cpg / ga), elements = (long long)hw * cpg;
  const bool few = wgs <= 256 ? hw <= 4096 && accesses <= 16384 && elements <= (wgs <= 96 ? 49152 : 65536)
                              : hw <= 3072 && accesses <= 10240 && elements <= 40960;
  if (ga * (int)sizeof(T) >= 4 && (few || groups > kGnMaxGroups)) {
    const int words = ga * (int)sizeof(T) / 4, vpp = cpg / ga;     // 32-bit registers an access takes; accesses per pixel
    auto fits = [&](int nt, int regs) { return vpp <= nt && (long long)(nt / vpp) * (regs / words) >= hw; };
#define AD_GN_ONE(NT_, REGS_) if (fits(NT_, REGS_)) return launch_gn_group<T, NT_, REGS_>(src0, src1, c0, c1, batch, hw, groups, ga, gamma, beta, eps, silu, out, s)
    AD_GN_ONE(256, 16);
    AD_GN_ONE(512, 16);
    AD_GN_ONE(1024, 16);
    AD_GN_ONE(1024, 48);
#undef AD_GN_ONE
  }
  if (groups > kGnMaxGroups) AD_FAIL(AD_ERR_INVALID, "groupnorm: at most %d groups", kGnMaxGroups);
  float* gpart = (float*)scratch;
  const size_t src_stride = (size_t)batch * nchunk * groups * 2;
  const long long rows = (long long)batch * hw;
  {
    ProfLaunch pl("gn_partial", 0, (double)rows * ctot * sizeof(T), s, (int)rows, ctot, 0);
    hipLaunchKernelGGL(k_gn_partial<T>, dim3(nchunk, batch, c1 ? 2 : 1), dim3(256), 0, s, (const T*)src0, (const T*)src1, c0, c1, hw, nchunk, groups,
                       cpg, src_stride, gpart);
  }
  // a workgroup of 1024 threads per CU: each folds the statistics of its sample once (32 KiB, four loads a thread) and then streams its
  // rows.  Two samples of 96x96x320 15.2 us for both launches, 96x96x(640+320) 23.5, 48x48x(1280+640) 17.8; with three times as many
  // workgroups of 256 threads, each folding the same 32 KiB in two dependent steps, 18.0, 28.3 and 23.0.
  constexpr int NT = 1024;
  const int nv = ctot / Vec<T>::N, pl = NT / std::min(nv, NT);
  const int per_sample = std::max(1, 256 / batch);            // a 257th workgroup would wait for a CU
  const int rows_per_block = std::max(pl, (hw + per_sample - 1) / per_sample);
  const int row_blocks = (hw + rows_per_block - 1) / rows_per_block;
  ProfLaunch pl_("gn_apply", 0, 2.0 * rows * ctot * sizeof(T), s, (int)rows, ctot, 0);
  hipLaunchKernelGGL((k_gn_apply<T, NT>), dim3(row_blocks, batch), dim3(NT), 0, s, (const T*)src0, (const T*)src1, c0, c1, hw, rows_per_block, nchunk,
                     groups, gpart, src_stride, make_fastdiv((unsigned)cpg), gamma, beta, eps, silu, (T*)out);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// bytes of partial sums the two-pass path writes: [2 sources][batch][chunks][groups][sum, sum of squares]
static size_t gn_partial_bytes(int batch, int hw, int groups, int c) {
  return (size_t)2 * batch * gn_chunks(batch, hw, groups, c) * groups * 2 * sizeof(float);
}

ad_status launch_groupnorm(int dtype, const void* src0, const void* src1, int c0, int c1, int batch, int hw, int groups,
                           const float* gamma, const float* beta, float eps, int silu, void* out, void* scratch,
                           size_t scratch_bytes, hipStream_t s) {
  if (!src0 || !gamma || !beta || !out || !scratch || (c1 > 0 && !src1)) AD_FAIL(AD_ERR_INVALID, "groupnorm: null pointer");
  const int vn = dtype == AD_BF16 ? 8 : 4;
  if (batch < 1 || hw < 1 || c0 < vn || c0 % vn || c1 < 0 || c1 % vn || groups < 1 || (c0 + c1) % groups)
    AD_FAIL(AD_ERR_INVALID, "groupnorm: bad shape");
  if (scratch_bytes < gn_partial_bytes(batch, hw, groups, c0 + c1)) AD_FAIL(AD_ERR_NOMEM, "groupnorm: scratch too small");
  if (dtype == AD_BF16) return run_groupnorm<bf16>(src0, src1, c0, c1, batch, hw, groups, gamma, beta, eps, silu, out, scratch, s);
  if (dtype == AD_F32) return run_groupnorm<float>(src0, src1, c0, c1, batch, hw, groups, gamma, beta, eps, silu, out, scratch, s);
  AD_FAIL(AD_ERR_INVALID, "groupnorm: bad dtype");
}

// -------------------------------------------------------------------------------------------------
// GroupNorm for callers that cannot allocate: the partial sums live in a fixed device array of this library
// instead of a caller-supplied scratch buffer.  Host code never uses the array's name as an address: the device
// address is looked up once per device (hipGetSymbolAddress, with that device current) and kept.
// -------------------------------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticGnBytes];
static void* g_scratch_ptr[kMaxDevices] = {nullptr};
static std::mutex g_scratch_mutex;

static ad_status static_scratch(void** out) {
  int dev = -1;
  AD_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) AD_FAIL(AD_ERR_INVALID, "groupnorm (static scratch): device %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    AD_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) AD_FAIL(AD_ERR_HIP, "groupnorm (static scratch): no device address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return AD_OK;
}

ad_status launch_groupnorm_static(int dtype, const void* src0, const void* src1, int c0, int c1, int batch, int hw, int groups,
                                  const float* gamma, const float* beta, float eps, int silu, void* out, hipStream_t s) {
  if (batch < 1 || hw < 1 || groups < 1) AD_FAIL(AD_ERR_INVALID, "groupnorm: bad shape");
  const size_t need = gn_partial_bytes(batch, hw, groups, c0 + c1);
  if (need > kStaticGnBytes)
    AD_FAIL(AD_ERR_NOMEM, "groupnorm (static scratch): batch %d x %d chunks x %d groups needs %zu bytes, the fixed buffer holds %zu",
            batch, gn_chunks(batch, hw, groups, c0 + c1), groups, need, kStaticGnBytes);
  void* ptr = nullptr;
  ad_status st = static_scratch(&ptr);
  if (st != AD_OK) return st;
  // every partial sum the second pass reads is written by the first pass of the same call: nothing to clear
  return launch_groupnorm(dtype, src0, src1, c0, c1, batch, hw, groups, gamma, beta, eps, silu, out, ptr, kStaticGnBytes, s);
}

// LayerNorm: `lanes` lanes per row (64 / lanes rows per wavefront), K accesses of 16 bytes each; the rows stay in registers between
// the two statistics passes.  Bound by the round trip to memory, so a wavefront has several rows in flight, every lane has work (a
// row of 320 channels is 40 accesses) and gain and offset are requested with the rows.  FULL: lanes * K accesses are the whole row.
// Measured, bf16, us (one row per wavefront, gain and offset read behind the statistics -> this): 65536x320 33.6 -> 14.6 (5.7 TB/s),
// 16384x640 14.4 -> 9.0, 18432x320 12.3 -> 6.9, 8192x640 8.6 -> 6.0, 2048x1280 4.9 -> 4.3.  An instance per number of accesses up to five:
// two and four in those of three and five cost a fifth (1152x2048 5.6 us against 4.5).
template <typename T, int K, bool FULL>
__global__ __launch_bounds__(256) void k_layernorm(const T* __restrict__ src, int rows, int c, int log_lanes, const float* __restrict__ gamma,
                                                   const float* __restrict__ beta, float eps, T* __restrict__ out) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  const int lane = threadIdx.x & 63, nv = c / VN, lanes = 1 << log_lanes;
  const int row = (int)((blockIdx.x * 256 + threadIdx.x) >> log_lanes), l = lane & (lanes - 1);
  const T* rp = src + (size_t)min(row, rows - 1) * c;
  V x[K];
  float ga[K][VN], be[K][VN];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int v = l + lanes * i;
    if (FULL || v < nv) x[i] = *(const V*)(rp + v * VN);
  }
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int v = FULL ? l + lanes * i : min(l + lanes * i, nv - 1);
#pragma unroll
    for (int e = 0; e < VN; ++e) { ga[i][e] = gamma[v * VN + e]; be[i][e] = beta[v * VN + e]; }
  }
  auto row_sum = [&](float v) {
    for (int o = lanes >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
  float s = 0.f, q = 0.f;
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (FULL || l + lanes * i < nv)
#pragma unroll
      for (int e = 0; e < VN; ++e) s += to_f(x[i][e]);
  const float mean = row_sum(s) / c;
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (FULL || l + lanes * i < nv) q = ln_squares(x[i], mean, q, i == 0);
  const float rstd = rsqrtf(row_sum(q) / c + eps);
  if (row >= rows) return;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int v = l + lanes * i;
    if (FULL || v < nv) {
      V t;
#pragma unroll
      for (int e = 0; e < VN; ++e) t[e] = from_f<T>(ln_value(to_f(x[i][e]), mean, rstd, ga[i][e], be[i][e]));
      *(V*)(out + (size_t)row * c + v * VN) = t;
    }
  }
}

// Lanes per row: the fewest that leave a lane at most five accesses (8 for 320 bf16 channels, 32 for 1280), doubled while that gives
// fewer than four wavefronts per CU (few rows: a shorter chain per row counts for more).
template <typename T>
static void run_layernorm(const void* src, int rows, int c, const float* gamma, const float* beta, float eps, void* out, hipStream_t s) {
  const int nv = c / Vec<T>::N;
  int lg = 0;
  while (lg < 6 && 5 << lg < nv) ++lg;
  while (lg < 6 && 1 << lg < nv && (long long)rows << lg < 64 * 1024) ++lg;
  const int lanes = 1 << lg, k = (nv + lanes - 1) / lanes, per_block = 256 / lanes;
  const dim3 grid((rows + per_block - 1) / per_block);
#define AD_LN(K_)                                                                                                                      \
  if (k <= K_) {                                                                                                                       \
    if (lanes * K_ == nv) hipLaunchKernelGGL((k_layernorm<T, K_, true>), grid, dim3(256), 0, s, (const T*)src, rows, c, lg, gamma, beta, eps, (T*)out); \
    else hipLaunchKernelGGL((k_layernorm<T, K_, false>), grid, dim3(256), 0, s, (const T*)src, rows, c, lg, gamma, beta, eps, (T*)out); \
    return;                                                                                                                            \
  }
  AD_LN(1)
  AD_LN(2)
  AD_LN(3)
  AD_LN(4)
  AD_LN(5)
  AD_LN(8)
#undef AD_LN
}

ad_status launch_layernorm(int dtype, const void* src, int rows, int c, const float* gamma, const float* beta, float eps,
                           void* out, hipStream_t s) {
  if (!src || !gamma || !beta || !out) AD_FAIL(AD_ERR_INVALID, "layernorm: null pointer");
  const int vn = dtype == AD_BF16 ? 8 : 4;
  if (rows < 1 || c < vn || c % vn || c > 64 * 8 * vn) AD_FAIL(AD_ERR_INVALID, "layernorm: unsupported width %d", c);
  ProfLaunch pl("layernorm", 0, 2.0 * rows * c * (dtype == AD_BF16 ? 2 : 4), s, rows, c, 0);
  if (dtype == AD_BF16)
    run_layernorm<bf16>(src, rows, c, gamma, beta, eps, out, s);
  else if (dtype == AD_F32)
    run_layernorm<float>(src, rows, c, gamma, beta, eps, out, s);
  else AD_FAIL(AD_ERR_INVALID, "layernorm: bad dtype");
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// Skinny linear layer of the time-embedding path: one wavefront per output feature, all rows at once.
template <typename T>
__global__ __launch_bounds__(256) void k_linear_rows(const float* __restrict__ in, int in_ld, int rows, int k, const T* __restrict__ w,
                                                     const float* __restrict__ bias, int n, int silu_in, int silu_out,
                                                     int accumulate, float* __restrict__ out) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  constexpr int MAXR = 16;
  const int lane = threadIdx.x & 63;
  const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= n) return;
  float acc[MAXR];
#pragma unroll
  for (int r = 0; r < MAXR; ++r) acc[r] = 0.f;
  for (int v = lane; v < k / VN; v += 64) {
    const V wv = *(const V*)(w + (size_t)col * k + v * VN);
#pragma unroll
    for (int r = 0; r < MAXR; ++r)
      if (r < rows)
#pragma unroll
        for (int e = 0; e < VN; ++e) {
          float x = in[(size_t)r * in_ld + v * VN + e];
          if (silu_in) x = silu_f(x);
          acc[r] += x * to_f(wv[e]);
        }
  }
#pragma unroll
  for (int r = 0; r < MAXR; ++r)
    if (r < rows) {
      float t = wave_sum(acc[r]) + (bias ? bias[col] : 0.f);
      if (silu_out) t = silu_f(t);
      if (lane == 0) out[(size_t)r * n + col] = accumulate ? out[(size_t)r * n + col] + t : t;
    }
}

ad_status launch_linear_rows(int dtype, const float* in, int in_ld, int rows, int k, const void* w, const float* bias, int n,
                             int silu_in, int silu_out, int accumulate, float* out, hipStream_t s) {
  if (!in || !w || !out) AD_FAIL(AD_ERR_INVALID, "linear_rows: null pointer");
  const int vn = dtype == AD_BF16 ? 8 : 4;
  if (rows < 1 || rows > 16 || k < vn || k % vn || n < 1) AD_FAIL(AD_ERR_INVALID, "linear_rows: bad shape");
  ProfLaunch pl("linear_rows", 2.0 * rows * n * k, (double)n * k * (dtype == AD_BF16 ? 2 : 4), s);
  if (dtype == AD_BF16)
    hipLaunchKernelGGL(k_linear_rows<bf16>, dim3((n + 3) / 4), dim3(256), 0, s, in, in_ld, rows, k, (const bf16*)w, bias, n, silu_in, silu_out, accumulate, out);
  else if (dtype == AD_F32)
    hipLaunchKernelGGL(k_linear_rows<float>, dim3((n + 3) / 4), dim3(256), 0, s, in, in_ld, rows, k, (const float*)w, bias, n, silu_in, silu_out, accumulate, out);
  else AD_FAIL(AD_ERR_INVALID, "linear_rows: bad dtype");
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// Sinusoidal timestep embedding [cos | sin], evaluated in double because tau * f reaches ~1e3 rad; by the threads of a workgroup.  Frequencies
// from .. from + count - 1 of dim / 2: out is the cosines, then the sines.
__device__ __forceinline__ void sinusoid(float tau, int dim, int from, int count, float* out) {
  const int half = dim / 2;
  for (int k = threadIdx.x; k < count; k += blockDim.x) {
    const double a = (double)tau * exp(-9.210340371976184 * (double)(from + k) / (double)half);   // ln(10^4)
    double s, c;
    sincos(a, &s, &c);
    out[k] = (float)c;
    out[count + k] = (float)s;
  }
}

// First layer of the time embedding: out[n] = SiLU(bias[n] + w[n] . sinusoid), one wavefront per feature; every workgroup evaluates the
// sinusoid for itself (1.5 us more than the layer alone; a launch for it 3.4), kTimePiece frequencies at a time.
constexpr int kTimePiece = 512;
template <typename T>
__global__ __launch_bounds__(256) void k_time_first(float tau, StepRef ref, int dim, const T* __restrict__ w, const float* __restrict__ bias, int n,
                                                    float* __restrict__ out) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  __shared__ __attribute__((aligned(16))) float s[2 * kTimePiece];
  const int lane = threadIdx.x & 63, col = blockIdx.x * 4 + (threadIdx.x >> 6), half = dim / 2;
  if (ref.table) tau = ref.table[*ref.counter + ref.offset].tau;
  const T* const row = w + (size_t)min(col, n - 1) * dim;
  float acc = 0.f;
  for (int from = 0; from < half; from += kTimePiece) {
    const int count = min(kTimePiece, half - from);
    if (from > 0) __syncthreads();                           // the last piece has been read
    sinusoid(tau, dim, from, count, s);
    __syncthreads();
    for (int i = lane * VN; i < 2 * count; i += 64 * VN) {   // (VN divides count: no access spans cosines and sines)
      const V wv = *(const V*)(row + from + (i < count ? i : half - count + i));
#pragma unroll
      for (int e = 0; e < VN; ++e) acc += s[i + e] * to_f(wv[e]);
    }
  }
  if (col >= n) return;
  const float t = wave_sum_rows(acc) + bias[col];
  if (lane == 0) out[col] = silu_f(t);
}

// The whole time embedding of a component in one launch: sinusoid, two layers, pooled branch, projections of its ResBlocks.  Every workgroup
// computes the embedding for itself and a share of the projections: it takes in the weights of all layers, those of the pooled branch once a
// sample (see time_fused_fits()); a launch of the four or six it replaces takes 3.7 us inside a replayed graph.  Two threads a feature in the
// layers, eight in the projections; rows of weights are read 16 bytes at a time, four loads of a thread in flight.  Bound by that chain.
constexpr int kTimeFusedLayer = 256 * 1024, kTimeRows = 64;
struct TimeParams {
  const void *w1, *w2, *w3, *w4, *wp; const float *b1, *b2, *b3, *b4, *bp;
  const float* pooled;                  // [batch][pooled_dim], or null
  int c0, td, batch, pooled_dim, rows;
  float tau; StepRef ref; float* out;   // out [batch][rows]
};
template <typename T>
__global__ __launch_bounds__(512) void k_time_fused(TimeParams p) {
  typedef typename Vec<T>::type V;
  constexpr int VN = Vec<T>::N;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* const s = (float*)lds;                              // [c0], later [batch][td] of the embedding
  float* const t1 = s + max(p.c0, p.batch * p.td);           // [td]
  float* const p1 = t1 + p.td;                               // [batch][td], pooled branch
  const int tid = threadIdx.x;
  // sum over `parts` threads of one feature of w[row] . x (part: which of them), complete in all of them
  auto dot = [&](const void* w, int row, int k, const float* x, int part, int parts) {
    float acc = 0.f;
    const T* const r = (const T*)w + (size_t)row * k;
#pragma unroll 4
    for (int v = part; v < k / VN; v += parts) {
      const V wv = *(const V*)(r + v * VN);
#pragma unroll
      for (int e = 0; e < VN; ++e) acc += x[v * VN + e] * to_f(wv[e]);
    }
    for (int o = 1; o < parts; o <<= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
  };
  float tau = p.tau;
  if (p.ref.table) tau = p.ref.table[*p.ref.counter + p.ref.offset].tau;
  sinusoid(tau, p.c0, 0, p.c0 / 2, s);
  __syncthreads();
  const int part = tid & 1;
  for (int n = tid >> 1; n < p.td; n += 256) {
    const float t = silu_f(dot(p.w1, n, p.c0, s, part, 2) + p.b1[n]);
    if (part == 0) t1[n] = t;
  }
  if (p.pooled)
    for (int i = tid >> 1; i < p.batch * p.td; i += 256) {
      const int b = i / p.td, n = i - b * p.td;
      const float t = silu_f(dot(p.w3, n, p.pooled_dim, p.pooled + (size_t)b * p.pooled_dim, part, 2) + p.b3[n]);
      if (part == 0) p1[i] = t;
    }
  __syncthreads();
  for (int n = tid >> 1; n < p.td; n += 256) {
    const float t = dot(p.w2, n, p.td, t1, part, 2) + p.b2[n];
    for (int b = 0; b < p.batch; ++b) {
      float u = t;
      if (p.pooled) u += dot(p.w4, n, p.td, p1 + b * p.td, part, 2) + p.b4[n];
      if (part == 0) s[b * p.td + n] = silu_f(u);
    }
  }
  __syncthreads();
  const int n = blockIdx.x * kTimeRows + (tid >> 3);
  if (n >= p.rows) return;
  for (int b = 0; b < p.batch; ++b) {
    const float t = dot(p.wp, n, p.td, s + b * p.td, tid & 7, 8) + p.bp[n];
    if ((tid & 7) == 0) p.out[(size_t)b * p.rows + n] = t;
  }
}

// (other: a second counter, or null)
__global__ void k_advance(int* counter, int* other, int by) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    *counter += by;
    if (other) *other += by;
  }
}

ad_status launch_advance(int* counter, int by, hipStream_t s, int* other) {
  if (!counter) AD_FAIL(AD_ERR_INVALID, "advance: null counter");
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, counter, other, by);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

ad_status launch_time_first(int dtype, float tau, StepRef ref, int dim, const void* w, const float* bias, int n, float* out, hipStream_t s) {
  const int vn = dtype == AD_BF16 ? 8 : 4;
  if (!w || !bias || !out || dim < 2 || dim % (2 * vn) || n < 1) AD_FAIL(AD_ERR_INVALID, "time_first: bad argument");
  ProfLaunch pl("linear_rows", 2.0 * n * dim, (double)n * dim * (dtype == AD_BF16 ? 2 : 4), s);
  if (dtype == AD_BF16) hipLaunchKernelGGL(k_time_first<bf16>, dim3((n + 3) / 4), dim3(256), 0, s, tau, ref, dim, (const bf16*)w, bias, n, out);
  else if (dtype == AD_F32) hipLaunchKernelGGL(k_time_first<float>, dim3((n + 3) / 4), dim3(256), 0, s, tau, ref, dim, (const float*)w, bias, n, out);
  else AD_FAIL(AD_ERR_INVALID, "time_first: bad dtype");
  AD_HIP(hipGetLastError());
  return AD_OK;
}

static size_t time_fused_lds(const TimeArgs& a) {
  return ((size_t)std::max(a.c0, a.batch * a.td) + a.td + (a.pooled ? (size_t)a.batch * a.td : 0)) * 4;
}
// One launch as long as the second layer (td x td) is at most kTimeFusedLayer and what a workgroup takes in costs less than the launches.  A
// ResBlock of 4x4 positions behind it, us, layer by layer / one launch: bf16, no pooled branch (160 KiB) 21.9 / 19.8, with it, one sample 352 KiB
// 27.5 / 23.9, 480 KiB 27.4 / 27.4, 640 KiB 28.1 / 31.8, 1.2 MiB 28.5 / 39.7, two samples 544 KiB 31.0 / 29.1, 640 KiB 30.9 / 30.5, 672 KiB 30.8 / 32.5,
// 3.2 MiB 34.7 / 101; fp32, half the arithmetic a byte: 320 KiB 23.8 / 23.7, one sample 584 KiB 29.6 / 27.8, 704 KiB 29.8 / 30.5, two samples 464 KiB
// 30.3 / 25.9, 720 KiB 30.9 / 31.3, 1088 KiB 32.6 / 37.9.
bool time_fused_fits(const TimeArgs& a) {
  const size_t es = esize(a.dtype), td = (size_t)a.td, pooled = a.pooled ? (size_t)a.batch * (a.pooled_dim + td) : 0;
  const size_t limit = (320 + 160 * (size_t)a.batch) * (a.dtype == AD_F32 ? 1280 : 1024);
  return td * td * es <= (size_t)kTimeFusedLayer && td * (a.c0 + td + pooled) * es <= limit && a.rows > 0 && time_fused_lds(a) <= 64 * 1024;
}

ad_status launch_time_fused(const TimeArgs& a, hipStream_t s) {
  const int vn = a.dtype == AD_BF16 ? 8 : 4;
  if (a.dtype != AD_BF16 && a.dtype != AD_F32) AD_FAIL(AD_ERR_INVALID, "time_fused: bad dtype");
  if (!a.w1 || !a.w2 || !a.wp || !a.out || !time_fused_fits(a) || a.c0 % vn || a.td % vn || (a.pooled && (!a.w3 || !a.w4 || a.pooled_dim % vn)))
    AD_FAIL(AD_ERR_INVALID, "time_fused: bad argument");
  const TimeParams p{a.w1, a.w2, a.w3, a.w4, a.wp, a.b1, a.b2, a.b3, a.b4, a.bp, a.pooled, a.c0, a.td, a.batch, a.pooled_dim, a.rows, a.tau, a.ref, a.out};
  const dim3 grid((a.rows + kTimeRows - 1) / kTimeRows);
  ProfLaunch pl("time_fused", 2.0 * a.td * (a.c0 + a.td + (double)a.batch * a.rows), (double)a.td * (a.c0 + a.td + a.rows) * esize(a.dtype), s);
  if (a.dtype == AD_BF16) hipLaunchKernelGGL(k_time_fused<bf16>, grid, dim3(512), time_fused_lds(a), s, p);
  else hipLaunchKernelGGL(k_time_fused<float>, grid, dim3(512), time_fused_lds(a), s, p);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// im2col of the latent for the first convolution: row (b, y, x), column tap * cl + c, zero padded to kConvInK.
template <typename T>
__global__ __launch_bounds__(256) void k_pack_latent(const float* __restrict__ latent, size_t sample_stride, float scale, StepRef ref,
                                                     int cl, int h, int w, int batch, T* __restrict__ out) {
  if (ref.table) scale = ref.table[*ref.counter + ref.offset].in_scale;
  const long long total = (long long)batch * h * w * kConvInK;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const int kk = (int)(i % kConvInK);
    const long long m = i / kConvInK;
    const int pix = (int)(m % (h * w));
    const int y = pix / w, x = pix - y * w;
    float v = 0.f;
    if (kk < 9 * cl) {
      const int tap = kk / cl, c = kk - tap * cl;
      const int iy = y + tap / 3 - 1, ix = x + tap % 3 - 1;
      if (iy >= 0 && iy < h && ix >= 0 && ix < w) v = latent[(size_t)(m / (h * w)) * sample_stride + ((size_t)c * h + iy) * w + ix] * scale;
    }
    out[i] = from_f<T>(v);
  }
}

ad_status launch_pack_latent(int dtype, const float* latent, int per_sample, float scale, StepRef ref, int cl, int h, int w, int batch,
                             void* out, hipStream_t s) {
  const size_t sample_stride = per_sample ? (size_t)cl * h * w : 0;
  if (!latent || !out || cl < 1 || 9 * cl > kConvInK || h < 1 || w < 1 || batch < 1) AD_FAIL(AD_ERR_INVALID, "pack_latent: bad argument");
  const long long total = (long long)batch * h * w * kConvInK;
  const int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
  ProfLaunch pl("pack_latent", 0, (double)total * (dtype == AD_BF16 ? 2 : 4), s);
  if (dtype == AD_BF16) hipLaunchKernelGGL(k_pack_latent<bf16>, dim3(blocks), dim3(256), 0, s, latent, sample_stride, scale, ref, cl, h, w, batch, (bf16*)out);
  else hipLaunchKernelGGL(k_pack_latent<float>, dim3(blocks), dim3(256), 0, s, latent, sample_stride, scale, ref, cl, h, w, batch, (float*)out);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

// Sampler: x <- cx * x + ce * eps, eps = eps_u + g (eps_c - eps_u) when batch == 2 (row 0 conditional).
__global__ __launch_bounds__(256) void k_sampler(float* __restrict__ x, const float* __restrict__ eps, size_t n, int batch,
                                                 float cx, float ce, StepRef ref, float g) {
  if (ref.table) {
    const StepRec r = ref.table[*ref.counter + ref.offset];
    cx = r.cx; ce = r.ce;
  }
  const size_t n4 = n / 4;
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    f32x4 xv = ((const f32x4*)x)[i];
    f32x4 e = ((const f32x4*)eps)[i];
    if (batch == 2) {
      const f32x4 eu = ((const f32x4*)(eps + n))[i];
      e = eu + g * (e - eu);
    }
    ((f32x4*)x)[i] = cx * xv + ce * e;
  }
  for (size_t i = n4 * 4 + (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    float e = eps[i];
    if (batch == 2) { const float eu = eps[n + i]; e = eu + g * (e - eu); }
    x[i] = cx * x[i] + ce * e;
  }
}

ad_status launch_sampler(float* x, const float* eps, size_t n, int batch, float cx, float ce, StepRef ref, float g, hipStream_t s) {
  if (!x || !eps || n == 0) AD_FAIL(AD_ERR_INVALID, "sampler: bad argument");
  if (batch != 1 && batch != 2) AD_FAIL(AD_ERR_INVALID, "sampler: batch must be 1 (no guidance) or 2 (guidance)");
  if (((uintptr_t)x | (uintptr_t)eps) & 15 || (batch == 2 && (n % 4))) {
    // unaligned layouts are not produced by this library; keep the vector path exact
    AD_FAIL(AD_ERR_INVALID, "sampler: pointers must be 16-byte aligned and n a multiple of 4 with guidance");
  }
  size_t blocks = (n / 4 + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 2048) blocks = 2048;
  ProfLaunch pl("sampler", 0, (double)n * 4 * (2 + batch), s);
  hipLaunchKernelGGL(k_sampler, dim3((unsigned)blocks), dim3(256), 0, s, x, eps, n, batch, cx, ce, ref, g);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

}  // namespace ad

// -------------------------------------------------------------------------------------------------
// C ABI wrappers of the single kernels.
// -------------------------------------------------------------------------------------------------
using namespace ad;

extern "C" {

ad_status ad_conv_forward(int dtype, const void* src0, const void* src1, int c0, int c1, int batch, int hs, int ws,
                          int up, int ksize, int stride, const void* w_packed, int n_out, const float* bias,
                          const float* rowvec, const void* residual, void* out, void* out2, void* out3, int out_mode, int ld_t,
                          void* splitk_ws, size_t splitk_bytes, ad_stream stream) {
  ConvArgs a{dtype, src0, src1, c0, c1, batch, hs, ws, up, ksize, stride, w_packed, n_out, bias, rowvec, n_out, residual, out, out_mode, ld_t, splitk_ws, splitk_bytes, out2, out3};
  return launch_conv(a, (hipStream_t)stream);
}

ad_status ad_groupnorm_forward(int dtype, const void* src0, const void* src1, int c0, int c1, int batch, int hw,
                               int groups, const float* gamma, const float* beta, float eps, int silu, void* out,
                               void* scratch, ad_stream stream) {
  return launch_groupnorm(dtype, src0, src1, c0, c1, batch, hw, groups, gamma, beta, eps, silu, out, scratch,
                          ad_groupnorm_scratch_bytes(batch, hw, c0 + c1), (hipStream_t)stream);
}

ad_status ad_groupnorm_forward_static(int dtype, const void* src0, const void* src1, int c0, int c1, int batch, int hw,
                                      int groups, const float* gamma, const float* beta, float eps, int silu, void* out,
                                      ad_stream stream) {
  return launch_groupnorm_static(dtype, src0, src1, c0, c1, batch, hw, groups, gamma, beta, eps, silu, out, (hipStream_t)stream);
}

ad_status ad_layernorm_forward(int dtype, const void* src, int rows, int c, const float* gamma, const float* beta,
                               float eps, void* out, ad_stream stream) {
  return launch_layernorm(dtype, src, rows, c, gamma, beta, eps, out, (hipStream_t)stream);
}

ad_status ad_attention_forward(int dtype, const void* q, const void* k, const void* v, int v_is_transposed, int batch,
                               int l, int lk, int c, int head_dim, int ldq, int ldk, int ldv, int ldo, void* out,
                               ad_stream stream) {
  return launch_attention(dtype, q, k, v, v_is_transposed, batch, l, lk, c, head_dim, ldq, ldk, ldv, ldo, out, (hipStream_t)stream);
}

ad_status ad_attention_frames_forward(int dtype, const void* q, const void* k, const void* v, int frames, int positions, int c,
                                      int heads, int ldq, int ldk, int ldv, int ldo, void* out, ad_stream stream) {
  return launch_attention_frames(dtype, q, k, v, frames, positions, c, heads, ldq, ldk, ldv, ldo, out, (hipStream_t)stream);
}

size_t ad_conv_workspace_bytes(int dtype, int batch, int h_out, int w_out, int n_out, int c_in_total, int ksize, int out_mode) {
  return conv_workspace_bytes(dtype, (long long)batch * h_out * w_out, n_out, ksize * ksize * c_in_total, out_mode);
}

ad_status ad_tune_conv_tile(int tile) {
  if (tile != -1 && tile != 1 && (tile < 3 || tile > 16 || tile == 13)) AD_FAIL(AD_ERR_INVALID, "tile must be -1, 1, 3..12 or 14..16");
  set_tile_override(tile);
  return AD_OK;
}

ad_status ad_tune_attention(int variant) {
  if (variant < -1 || variant > 3) AD_FAIL(AD_ERR_INVALID, "variant must be -1 .. 3");
  set_attn_variant(variant);
  return AD_OK;
}

ad_status ad_tune_conv_order(int order) {
  if (order < -1 || order > 1) AD_FAIL(AD_ERR_INVALID, "order must be -1, 0 or 1");
  set_order_override(order);
  return AD_OK;
}

ad_status ad_sampler_update_raw(void* x, const void* eps, size_t n, int batch, float c_x, float c_eps, float cfg_scale,
                                ad_stream stream) {
  return launch_sampler((float*)x, (const float*)eps, n, batch, c_x, c_eps, StepRef{}, cfg_scale, (hipStream_t)stream);
}

}  // extern "C"
