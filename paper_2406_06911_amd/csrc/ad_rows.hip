// The row-local part of a transformer block in one launch (narrow models).
#include "ad_device.h"
#include "ad_kernels.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

namespace ad {

// =================================================================================================
// Between two attentions over the image everything a transformer block does is local to a token: output projection, LayerNorm, query
// projection, attention to the text (whose keys and values are there already), its output projection, LayerNorm, GEGLU, second
// feed-forward layer, and then either the next layer's LayerNorm and q/k/v or the block's output projection; the same goes for the
// block's input projection with the first LayerNorm and q/k/v.  In a narrow model each of these is a launch of 3 to 5 us that works for a
// fraction of a microsecond, so a workgroup takes 16 TM tokens of a sample through all of them, with every intermediate in LDS and
// rounded to the storage type where the separate launches round it.
//
// The launch is a short list of GEMMs (RowOp) with what goes before (LayerNorm) and behind them (attention to the text, rows out): one
// copy of the code of every step, whatever the list, since straight-line code that runs once is paid for in instruction fetches.  The
// eight wavefronts share the columns of a GEMM in tiles of 16, two at a time (or two halves of K of one tile, where there are no more
// tiles than wavefronts): weights in fragment order (pack_fragments) straight from memory into registers, up to RING items ahead of the
// MFMAs, the first ones before the barrier, activations from LDS.  Weights are the A operand, so a lane ends up with four consecutive
// columns of a row.  Biases, gains and offsets of the whole list come in with the rows.
// Bound by the chain of dependent steps (about 1.1 us a GEMM, 2.5 us the text) and by the weights a workgroup takes in (15 C^2 of them at the
// 64 bytes a clock of a CU's vector cache).
// Measured, bf16, us (the separate launches at 3.7 each inside a replayed graph -> this): behind an attention 1152 tokens of 64 channels
// 33 -> 13.1, 288 of 128 33 -> 18.1; input projection, LayerNorm and q/k/v 11 -> 7.2 and 8.4.  Weights in rows instead of fragment order (16
// rows of 64 bytes an access, half the rate from beyond the L2): 19 and 23.  At 256 channels the weights decide: 34.5 and 12.8, and whole runs
// with it are 1 % slower than with the separate launches, which use the whole chip; hence kRowsMaxBytes.
// =================================================================================================
enum { ROW_SYNC = 1, ROW_GEGLU = 2, ROW_HALVES = 4, ROW_SHORT = 8, ROW_TEXT = 16, ROW_PUT = 32, ROW_PUT_QKV = 64, ROW_NORM = 128 };
constexpr int kRowsMaxBytes = 256;      // of a row of C channels
constexpr int kRowOps = 9, kRowVecs = 24, kRowWaves = 8, kRowRing = 4;
struct RowOp {
  const void* w;
  unsigned wbytes;
  unsigned short tiles, kt;             // 16-column tiles (GEGLU: value tiles), 128-byte pieces of K
  int src, dst, res, norm;              // LDS byte offsets: activations, results, rows that are added (< 0: none), rows that are normalised into src first
  unsigned short src_pitch, dst_pitch;
  unsigned short bias, gain, offset, flags;      // places in the vector area (floats); bias kNoVec: none
};
static_assert(sizeof(RowOp) == 48, "twelve scalar registers");
constexpr unsigned short kNoVec = 0xffff;
struct RowParams {
  RowOp ops[kRowOps];                   // n_ops of them and an empty one (tiles = 0)
  const float* vecs[kRowVecs];          // C floats each
  int n_ops, n_vecs;
  FastDiv div_tiles, div_per;           // by tiles, by 16-byte pieces of a row
  int L, C, tiles;                      // tokens a sample, channels, row tiles a sample
  int lds_in, lds_h, lds_x, lds_part, lds_vec, pitch;
  const void *in, *h, *x;               // rows that are loaded: to lds_in, lds_h, lds_x (the last two may be null)
  void* put;                            // destination of ROW_PUT
  void *q, *k, *v; int ld_t;            // ROW_PUT_QKV: v rows, or transposed [sample][C][ld_t]
  const void *tk, *tv; int Lk, ldv, text_shared;
  int splits, split_keys;               // ROW_TEXT: the keys of a head are shared out over `splits` wavefronts
  float scale_log2, eps;
};

// waits for every load and store of this wavefront
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

template <typename T, int TM, int DT>
__global__ __launch_bounds__(64 * kRowWaves, 4) void k_tfm_rows(RowParams p) {
  typedef typename Vec<T>::type V;
  typedef typename Vec4<T>::type V4;
  constexpr int R = 16 * TM, ES = (int)sizeof(T), VN = Vec<T>::N, NW = kRowWaves, NT = 64 * NW, RING = kRowRing;
  constexpr int FRAG = 16 * kRowBytes;                       // bytes of a weight item: 16 rows, 128 bytes of K
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = (int)fast_div(blockIdx.x, p.div_tiles), l0 = ((int)blockIdx.x - b * p.tiles) * R;
  const int C = p.C, rows = min(R, p.L - l0);
  const size_t row0 = (size_t)b * p.L + l0;
  const float* const vec = (const float*)(lds + p.lds_vec);
  const int text_b = p.text_shared ? 0 : b;

  // the rows (those beyond the sample repeat its last one and are never stored) and the vectors: requested first (an access of a lane each)
  const int per = C / VN;
  const T* const src[3] = {(const T*)p.in, (const T*)(p.h ? p.h : p.in), (const T*)(p.x ? p.x : p.in)};   // (no branch around a load)
  V rv[TM][3];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int at = min(tid + i * NT, R * per - 1), r = (int)fast_div((unsigned)at, p.div_per), cv = at - r * per;
    const size_t o = (row0 + min(r, rows - 1)) * C + cv * VN;
#pragma unroll
    for (int j = 0; j < 3; ++j) rv[i][j] = *(const V*)(src[j] + o);
  }
  f32x4 vr[kRowVecs / NW];
#pragma unroll
  for (int i = 0; i < kRowVecs / NW; ++i) vr[i] = *(const f32x4*)(p.vecs[min(wave + NW * i, p.n_vecs - 1)] + min(lane * 4, C - 4));

  // The ring of weight fragments: items of this wavefront, in order.  A GEMM of at most RING items requests them all at once; in a longer
  // one every item is followed by a request, from beyond the range check where there is no item left (which reads zeros without touching
  // memory): with a branch around it the compiler could not tell how many are in flight and would wait for all of them every time.
  u32x4 wf[RING][2][2];
  int f_ct = 0, f_kt = 0;
  auto items_a_round = [&](const RowOp& op) { return op.flags & ROW_HALVES ? op.kt / 2 : (int)op.kt; };
  auto step_of = [&](const RowOp& op) { return op.flags & ROW_GEGLU || op.tiles <= NW ? NW : 2 * NW; };
  auto rounds_of = [&](const RowOp& op) { return (op.tiles - wave + step_of(op) - 1) >> (step_of(op) == NW ? 3 : 4); };      // 0 where there is no tile left
  static_assert(NW == 8, "rounds_of");
  // first and second half of an item: tile ct and the one NW further on; GEGLU (packed columns: 32 value, 32 gate): value tile ct and its
  // gate; or the two halves of K
  auto first_at = [&](const RowOp& op, int ct, int kt) { return (unsigned)(((op.flags & ROW_GEGLU ? 4 * (ct >> 1) + (ct & 1) : ct) * op.kt + kt) * FRAG); };
  auto second_by = [&](const RowOp& op) {
    return (unsigned)((op.flags & ROW_GEGLU ? 2 * op.kt : op.flags & ROW_HALVES ? op.kt / 2 : NW * op.kt) * FRAG);
  };
  auto second = [&](const RowOp& op, int ct) { return op.flags & (ROW_GEGLU | ROW_HALVES) || ct + NW < op.tiles; };
  auto load = [&](const RowOp& op, u32x4 (&dst)[2], unsigned at) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(op.w, op.wbytes);
#pragma unroll
    for (int h = 0; h < 2; ++h) dst[h] = buffer_load16<u32x4>(rs, at + (unsigned)lane * 16 + h * 1024, 0);
  };
  auto fetch = [&](const RowOp& op, int s) {
    const unsigned at = first_at(op, f_ct, f_kt);
    load(op, wf[s][0], f_ct < op.tiles ? at : kOob);
    load(op, wf[s][1], f_ct < op.tiles && second(op, f_ct) ? at + second_by(op) : kOob);
    if (++f_kt == items_a_round(op)) { f_kt = 0; f_ct += step_of(op); }
  };
  auto prime = [&](const RowOp& op) {
    f_ct = wave; f_kt = 0;
    // (nothing in the ring is wanted any more: says so, or the parts that are not loaded below would be kept through everything before)
#pragma unroll
    for (int s = 0; s < RING; ++s)
#pragma unroll
      for (int h = 0; h < 4; ++h) asm volatile("" : "=v"(wf[s][h >> 1][h & 1]));
    if (op.flags & ROW_SHORT) {
      const int n = rounds_of(op) * items_a_round(op);
#pragma unroll
      for (int s = 0; s < RING; ++s)
        if (s < n) {
          const unsigned at = first_at(op, f_ct, f_kt);
          load(op, wf[s][0], at);
          if (second(op, f_ct)) load(op, wf[s][1], at + second_by(op));
          if (++f_kt == items_a_round(op)) { f_kt = 0; f_ct += step_of(op); }
        }
    } else {
#pragma unroll
      for (int s = 0; s < RING; ++s) {
        fetch(op, s);
        __builtin_amdgcn_sched_barrier(0);                   // in order
      }
    }
  };
  // an operation's description in scalar registers, read as a whole and ahead of its use
  auto read_op = [&](int o) {
    RowOp op = p.ops[o];
    unsigned (&d)[12] = *(unsigned (*)[12])&op;
#pragma unroll
    for (int i = 0; i < 12; ++i) asm volatile("" : "+s"(d[i]));
    return op;
  };
  RowOp op = read_op(0);
  __builtin_amdgcn_s_barrier();                              // every wavefront has asked for its rows before the first asks for weights
  prime(op);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int at = tid + i * NT, r = (int)fast_div((unsigned)at, p.div_per), cv = at - r * per;
    if (at < R * per) {
      char* const dst = lds + r * p.pitch + cv * 16;
      *(V*)(dst + p.lds_in) = rv[i][0];
      if (p.h) *(V*)(dst + p.lds_h) = rv[i][1];
      if (p.x) *(V*)(dst + p.lds_x) = rv[i][2];
    }
  }
#pragma unroll
  for (int i = 0; i < kRowVecs / NW; ++i)
    if (lane * 4 < C && wave + NW * i < p.n_vecs) *(f32x4*)(lds + p.lds_vec + ((wave + NW * i) * C + lane * 4) * 4) = vr[i];

  f32x4 acc[2][TM];
  auto clear = [&]() {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
#pragma unroll 1
  for (int o = 0; o < p.n_ops; ++o) {
    const RowOp next = read_op(o + 1);
    if (op.flags & ROW_SYNC) __syncthreads();
    if (op.flags & ROW_NORM) {
      // 32 lanes a row, four channels an access; the row stays in registers between the two passes over it
      const int l = lane & 31, nv = C / 4;
      static_assert(kRowsMaxBytes / ES <= 128, "one access a lane");
      auto row_sum = [&](float v) {
        v += dpp_f<0xB1>(v);
        v += dpp_f<0x4E>(v);
        v += dpp_f<0x141>(v);
        v += dpp_f<0x140>(v);
        return v + __shfl_xor(v, 16, 64);
      };
#pragma unroll 1
      for (int r = 2 * wave + (lane >> 5); r < R; r += 2 * NW) {
        f32x4 x = {0.f, 0.f, 0.f, 0.f}, ga = x, be = x;
        if (l < nv) {
          const V4 t = *(const V4*)(lds + op.norm + r * p.pitch + l * 4 * ES);
          ga = *(const f32x4*)(vec + op.gain + l * 4);
          be = *(const f32x4*)(vec + op.offset + l * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = to_f(t[e]);
        }
        const float mean = row_sum((x[0] + x[1]) + (x[2] + x[3])) / C;
        if (l < nv) x -= mean;
        const float rstd = rsqrtf(row_sum((x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3])) / C + p.eps);
        if (l < nv) {
          V4 t;
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = from_f<T>(x[e] * rstd * ga[e] + be[e]);
          *(V4*)(lds + op.src + r * op.src_pitch + l * 4 * ES) = t;
        }
      }
      __syncthreads();
    }
    {
      const int round = items_a_round(op), n = rounds_of(op) * round, step = step_of(op);
      const char* const act = lds + op.src + r16 * op.src_pitch + kg * 16;
      const int half_k = op.flags & ROW_HALVES ? round * kRowBytes : 0;
      int ct = wave, kt = 0;
      // four columns of every row: result tile `tile`
      auto emit = [&](int tile, const f32x4 (&sum)[TM]) {
        const int col = 16 * tile + 4 * kg;
        const f32x4 add = op.bias != kNoVec ? *(const f32x4*)(vec + op.bias + col) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int at = (16 * i + r16) * op.dst_pitch + col * ES;
          f32x4 v = sum[i] + add;
          if (op.res >= 0) {
            const V4 t = *(const V4*)(lds + op.res + at);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += to_f(t[e]);
          }
          *(V4*)(lds + op.dst + at) = V4{from_f<T>(v[0]), from_f<T>(v[1]), from_f<T>(v[2]), from_f<T>(v[3])};
        }
      };
      auto consume = [&](int s) {
        // (where there is no second half, its sums are of whatever the registers hold and go nowhere)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const char* const at = act + i * 16 * op.src_pitch + kt * kRowBytes + h * 64;
            Mma16<T>::run(__builtin_bit_cast(V, wf[s][0][h]), *(const V*)at, acc[0][i]);
            Mma16<T>::run(__builtin_bit_cast(V, wf[s][1][h]), *(const V*)(at + half_k), acc[1][i]);
          }
        if (++kt < round) return;
        kt = 0;
        if (op.flags & ROW_GEGLU) {
          const int packed = 64 * (ct >> 1) + 16 * (ct & 1) + 4 * kg;
          const f32x4 bv = *(const f32x4*)(vec + op.bias + packed), bg = *(const f32x4*)(vec + op.bias + packed + 32);
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            V4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = from_f<T>((acc[0][i][e] + bv[e]) * gelu_f(acc[1][i][e] + bg[e]));
            *(V4*)(lds + op.dst + (16 * i + r16) * op.dst_pitch + (16 * ct + 4 * kg) * ES) = t;
          }
        } else {
          if (op.flags & ROW_HALVES)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[0][i] += acc[1][i];
          emit(ct, acc[0]);
          if (!(op.flags & ROW_HALVES) && ct + NW < op.tiles) emit(ct + NW, acc[1]);
        }
        ct += step;
        clear();
      };
      clear();
      int it = 0;
      if (!(op.flags & ROW_SHORT)) {
        wait_vmem();                                         // what is in flight here came from either branch of prime(): start counting afresh
#pragma unroll 1
        for (; it + RING < n; it += RING)
#pragma unroll
          for (int s = 0; s < RING; ++s) {
            consume(s);
            fetch(op, s);
          }
      }
#pragma unroll
      for (int s = 0; s < RING; ++s)
        if (it + s < n) consume(s);
    }
    if (op.flags & ROW_TEXT) {
      // Attention to the text: a wavefront takes 16 queries of a head and a share of the keys at a time, scores transposed (S^T = K Q^T: a
      // lane holds keys of query r16), online softmax over blocks of keys, the next block requested ahead; the shares are merged through
      // LDS.  Probabilities leave the score tile in the order in which the second product takes them.
      __syncthreads();
      constexpr int d = 16 * DT, PP = d + 4;                 // a query's partial result: d sums, maximum, denominator
      const int heads = C / d, S = p.splits;
      float* const part = (float*)(lds + p.lds_part);
      // (a text sample is less than 2 GiB, see tfm_rows_fits)
      const __amdgpu_buffer_rsrc_t rsk = make_rsrc((const T*)p.tk + (size_t)text_b * p.Lk * C, (unsigned)(p.Lk * C) * ES);
      const __amdgpu_buffer_rsrc_t rsv = make_rsrc((const T*)p.tv + (size_t)text_b * (ES == 2 ? p.ldv : p.Lk) * C, (unsigned)((ES == 2 ? p.ldv : p.Lk) * C) * ES);
#pragma unroll 1
      for (int u = wave; u < heads * TM * S; u += NW) {
        const int sp = u % S, hi = u / S, h = hi / TM, i = hi - h * TM;
        const int first = sp * p.split_keys, last = min(p.Lk, first + p.split_keys);       // not empty
        const char* const qrow = lds + op.dst + (16 * i + r16) * op.dst_pitch + h * d * ES;
        float m = -INFINITY, l = 0.f;
        f32x4 o[DT];
#pragma unroll
        for (int t = 0; t < DT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        // adds a block's scores (base-2 logarithms, minus infinity beyond the last key) to the running maximum; e[] becomes the terms
        auto softmax = [&](auto& e, auto count) {
          constexpr int N = decltype(count)::value;
          float mx = -INFINITY;
#pragma unroll
          for (int r = 0; r < N; ++r) mx = fmaxf(mx, e[r >> 2][r & 3]);
          mx = fmaxf(mx, __shfl_xor(mx, 16));
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          const float m_new = fmaxf(m, mx), ref = m_new == -INFINITY ? 0.f : m_new, alpha = __builtin_amdgcn_exp2f(m - ref);
          m = m_new;
          float sum = 0.f;
#pragma unroll
          for (int r = 0; r < N; ++r) {
            e[r >> 2][r & 3] = __builtin_amdgcn_exp2f(e[r >> 2][r & 3] - ref);
            sum += e[r >> 2][r & 3];
          }
          l = l * alpha + sum;
#pragma unroll
          for (int t = 0; t < DT; ++t) o[t] *= alpha;
        };
        if constexpr (ES == 2) {
          // head width 64, values transposed; blocks of 32 keys: row r16 of key tile t is key 8 (r16 / 4) + 4 t + r16 % 4
          static_assert(DT == 4, "bf16: head width 64");
          const unsigned kcol = (unsigned)(h * 64 + kg * 8) * ES, krow = 8 * (r16 >> 2) + (r16 & 3);
          const unsigned vat = (unsigned)((h * 64 + r16) * p.ldv + kg * 8) * ES;
          V qf[2], kf[2][2], vf[4];
          auto fetch_k = [&](int key0) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int ks = 0; ks < 2; ++ks)
                kf[t][ks] = buffer_load16<V>(rsk, (unsigned)(min(key0 + (int)krow + 4 * t, p.Lk - 1) * C) * ES + kcol + ks * 64, 0);
          };
          auto fetch_v = [&](int key0) {                     // ldv is padded to 64 keys
#pragma unroll
            for (int t = 0; t < 4; ++t) vf[t] = buffer_load16<V>(rsv, vat + (unsigned)(16 * t * p.ldv * ES), (unsigned)(key0 * ES));
          };
          fetch_k(first);
          fetch_v(first);
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) qf[ks] = *(const V*)(qrow + ks * 64 + kg * 16);
#pragma unroll 1
          for (int key0 = first; key0 < last; key0 += 32) {
            f32x4 s[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int ks = 0; ks < 2; ++ks) Mma16<T>::run(kf[t][ks], qf[ks], s[t]);
              s[t] *= p.scale_log2;
            }
            if (key0 + 32 < last) fetch_k(key0 + 32);
            if (key0 + 32 > p.Lk) {                          // what the pad behind the last key holds must not count
#pragma unroll
              for (int e = 0; e < 8; ++e)
                if (key0 + 8 * kg + e >= p.Lk) {
                  s[e >> 2][e & 3] = -INFINITY;
#pragma unroll
                  for (int t = 0; t < 4; ++t) vf[t][e] = from_f<T>(0.f);
                }
            }
            softmax(s, std::integral_constant<int, 8>{});
            V pb;
#pragma unroll
            for (int e = 0; e < 8; ++e) pb[e] = from_f<T>(s[e >> 2][e & 3]);
#pragma unroll
            for (int t = 0; t < 4; ++t) Mma16<T>::run(vf[t], pb, o[t]);
            if (key0 + 32 < last) fetch_v(key0 + 32);
          }
        } else {
          // fp32, values in rows; blocks of 16 keys, head width 16 DT
          f32x4 qf[DT], kf[DT], vf[DT];
          auto fetch_k = [&](int key0) {
            const unsigned at = (unsigned)(min(key0 + r16, p.Lk - 1) * C + h * d + 4 * kg) * ES;
#pragma unroll
            for (int t = 0; t < DT; ++t) kf[t] = buffer_load16<f32x4>(rsk, at + t * 64, 0);
          };
          auto fetch_v = [&](int key0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const unsigned at = (unsigned)(min(key0 + 4 * kg + r, p.Lk - 1) * C + h * d + r16) * ES;
#pragma unroll
              for (int t = 0; t < DT; ++t) vf[t][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsv, (int)(at + t * 64), 0, 0));
            }
          };
          fetch_k(first);
          fetch_v(first);
#pragma unroll
          for (int t = 0; t < DT; ++t) qf[t] = *(const f32x4*)(qrow + (16 * t + 4 * kg) * ES) * p.scale_log2;
#pragma unroll 1
          for (int key0 = first; key0 < last; key0 += 16) {
            f32x4 s[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int t = 0; t < DT; ++t) Mma16<float>::run(kf[t], qf[t], s[0]);
            if (key0 + 16 < last) fetch_k(key0 + 16);
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (key0 + 4 * kg + r >= p.Lk) s[0][r] = -INFINITY;
            softmax(s, std::integral_constant<int, 4>{});
#pragma unroll
            for (int t = 0; t < DT; ++t) Mma16<float>::run(vf[t], s[0], o[t]);
            if (key0 + 16 < last) fetch_v(key0 + 16);
          }
        }
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        float* const mine = part + (u * 16 + r16) * PP;
#pragma unroll
        for (int t = 0; t < DT; ++t) *(f32x4*)(mine + 16 * t + 4 * kg) = o[t];
        if (kg == 0) { mine[d] = m; mine[d + 1] = l; }
      }
      __syncthreads();
      for (int at = tid; at < R * C / 4; at += NT) {
        const int r = at / (C / 4), c = (at - r * (C / 4)) * 4, h = c / d;
        const float* const from = part + (((h * TM + (r >> 4)) * S) * 16 + (r & 15)) * PP;
        float top = -INFINITY;
        for (int sp = 0; sp < S; ++sp) top = fmaxf(top, from[sp * 16 * PP + d]);
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
        for (int sp = 0; sp < S; ++sp) {
          const float f = __builtin_amdgcn_exp2f(from[sp * 16 * PP + d] - top);
          num += f * *(const f32x4*)(from + sp * 16 * PP + (c - h * d));
          den += f * from[sp * 16 * PP + d + 1];
        }
        V4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = from_f<T>(num[e] / den);
        *(V4*)(lds + p.lds_in + r * p.pitch + c * ES) = x;
      }
    }
    prime(next);                                             // (behind the attention, whose own registers it would crowd out)
    if (op.flags & (ROW_PUT | ROW_PUT_QKV)) {
      __syncthreads();
      if (op.flags & ROW_PUT) {
        for (int i = tid; i < rows * per; i += NT) {
          const int r = i / per, cv = i - r * per;
          *(V*)((T*)p.put + (row0 + r) * C + cv * VN) = *(const V*)(lds + op.dst + r * op.dst_pitch + cv * 16);
        }
      } else {
        const int which = p.ld_t > 0 ? 2 : 3;
        for (int i = tid; i < rows * which * per; i += NT) {
          const int r = i / (which * per), c = i - r * (which * per), w = c / per, cv = c - w * per;
          T* const dst = (T*)(w == 0 ? p.q : w == 1 ? p.k : p.v);
          *(V*)(dst + (row0 + r) * C + cv * VN) = *(const V*)(lds + op.dst + r * op.dst_pitch + (w * C + cv * VN) * ES);
        }
        if (p.ld_t > 0) {
          const int groups = (rows + VN - 1) / VN;             // VN tokens of a column are 16 bytes of its row (l0 and ld_t are multiples of VN)
          for (int i = tid; i < groups * C; i += NT) {
            const int g = i / C, c = i - g * C;
            T* const dst = (T*)p.v + ((size_t)b * C + c) * p.ld_t + l0 + g * VN;
            const char* const src = lds + op.dst + g * VN * op.dst_pitch + (2 * C + c) * ES;
            V t;
#pragma unroll
            for (int e = 0; e < VN; ++e) t[e] = *(const T*)(src + e * op.dst_pitch);
            if (g * VN + VN <= rows) *(V*)dst = t;
            else
#pragma unroll
              for (int e = 0; e < VN; ++e)
                if (g * VN + e < rows) dst[e] = t[e];
          }
        }
      }
    }
    op = next;
  }
}

// Buffers in LDS: A, H, X of C channels a row and G of 4 C (the feed-forward's inner rows; q of the attention to the text; q, k, v), the
// attention's partial results and the vectors.  Keys are shared out so that there is work for eight wavefronts.
struct RowPlan { int tm, splits, split_keys, part, bytes; };
static RowPlan plan_rows(int dtype, int c, int head_dim, int batch, int l, int lk) {
  const int es = (int)esize(dtype), block = dtype == AD_BF16 ? 32 : 16;
  auto plan = [&](int tm) {
    RowPlan r{tm};
    const int heads = c / head_dim, blocks = (lk + block - 1) / block, want = std::max(1, kRowWaves / (heads * tm));
    r.split_keys = (blocks + want - 1) / want * block;
    r.splits = (lk + r.split_keys - 1) / r.split_keys;
    r.part = 16 * tm * (3 * (c * es + 16) + (4 * c * es + 16));
    r.bytes = r.part + heads * tm * r.splits * 16 * (head_dim + 4) * 4 + kRowVecs * c * 4;
    return r;
  };
  // tiles of 16 tokens, or of 32 once those fill the chip twice over, as LDS allows
  if ((long long)batch * ((l + 15) / 16) > 512) {
    const RowPlan r = plan(2);
    if (r.bytes <= 160 * 1024) return r;
  }
  return plan(1);
}

// Up to kRowsMaxBytes a row, and beyond kRowsManyTokens only where C x C weights are at most 16 KiB: with that many tokens the separate launches
// fill the chip, and a workgroup that takes in 15 C^2 weights for its 32 tokens falls behind.  Whole block, us (separate launches -> this): bf16, 128
// channels 4608 tokens 106 -> 64, 10368 158 -> 148, 16384 (16 frames) 143 -> 123, but 18432 254 -> 267, 20480 (frames, as the next) 209 -> 220, 25600
// 184 -> 208, 36864 245 -> 278, 65536 415 -> 485; 64 channels 18432 191 -> 177, 36864 180 -> 157, 65536 247 -> 242; fp32, 64 channels 36864 657 -> 579,
// 65536 1448 -> 1406.
constexpr long long kRowsManyTokens = 16384;
bool tfm_rows_fits(int dtype, int c, int head_dim, int lk, long long tokens) {
  if (dtype != AD_BF16 && dtype != AD_F32) return false;
  if ((long long)(lk + 64) * c * (int)esize(dtype) >= 1LL << 31) return false;       // 32-bit offsets into a text sample
  if (c * (int)esize(dtype) > kRowsMaxBytes || c % bk_elems(dtype) || c % head_dim) return false;
  if (tokens > kRowsManyTokens && c * c * (int)esize(dtype) > 16384) return false;
  return dtype == AD_BF16 ? head_dim == 64 : (head_dim == 16 || head_dim == 32 || head_dim == 64);
}

template <typename T, int TM, int DT>
static ad_status run_tfm_rows(const RowParams& p, int grid, int lds_bytes, hipStream_t s) {
  static std::atomic<bool> attr_set{false};
  if (!attr_set) {
    AD_HIP(hipFuncSetAttribute((const void*)k_tfm_rows<T, TM, DT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    attr_set = true;
  }
  hipLaunchKernelGGL((k_tfm_rows<T, TM, DT>), dim3(grid), dim3(64 * kRowWaves), lds_bytes, s, p);
  AD_HIP(hipGetLastError());
  return AD_OK;
}

ad_status launch_tfm_rows(const TfmRows& a, hipStream_t s) {
  if (a.batch < 1 || a.l < 1 || !a.in || !tfm_rows_fits(a.dtype, a.c, a.head_dim, a.lk, (long long)a.batch * a.l)) AD_FAIL(AD_ERR_INVALID, "tfm_rows: unsupported shape");
  if ((a.w_in != nullptr) == (a.w_o != nullptr)) AD_FAIL(AD_ERR_INVALID, "tfm_rows: either the input projection or the layer behind an attention");
  const int c = a.c, es = (int)esize(a.dtype);
  const RowPlan plan = plan_rows(a.dtype, c, a.head_dim, a.batch, a.l, a.w_o ? a.lk : 1);
  const int r = 16 * plan.tm, pitch = c * es + 16, gpitch = 4 * c * es + 16;
  const int lds_a = 0, lds_h = r * pitch, lds_x = 2 * r * pitch, lds_g = 3 * r * pitch;
  RowParams p = {};
  p.lds_part = plan.part;
  p.lds_vec = plan.bytes - kRowVecs * c * 4;
  p.splits = plan.splits; p.split_keys = plan.split_keys;
  p.L = a.l; p.C = c; p.tiles = (a.l + r - 1) / r;
  p.lds_in = lds_a; p.lds_h = lds_h; p.lds_x = lds_x; p.pitch = pitch;
  p.in = a.in;
  p.eps = a.eps;
  p.scale_log2 = 1.f / sqrtf((float)a.head_dim) * 1.44269504088896341f;
  double flops = 0;
  auto vecs = [&](const float* v, int count) {               // count * C floats; place in the vector area
    const int at = p.n_vecs * c;
    for (int i = 0; i < count && p.n_vecs < kRowVecs; ++i) p.vecs[p.n_vecs++] = v + (size_t)i * c;
    return (unsigned short)at;
  };
  auto gemm = [&](int src, const void* w, const float* bias, int n, int k, int dst, int res, int flags = 0) -> RowOp& {
    RowOp& op = p.ops[p.n_ops++];
    op.w = w; op.wbytes = (unsigned)((size_t)round_up(n, kNPad) * k * es);
    op.tiles = (unsigned short)(flags & ROW_GEGLU ? n / 32 : n / 16); op.kt = (unsigned short)(k * es / kRowBytes);
    op.src = src; op.src_pitch = (unsigned short)(src == lds_g ? gpitch : pitch);
    op.dst = dst; op.dst_pitch = (unsigned short)(dst == lds_g ? gpitch : pitch);
    op.res = res; op.bias = bias ? vecs(bias, n / c) : kNoVec;
    op.flags = (unsigned short)(flags | ROW_SYNC);
    if (!(flags & ROW_GEGLU) && op.tiles <= kRowWaves && op.kt % 2 == 0) op.flags |= ROW_HALVES;
    const int step = flags & ROW_GEGLU || op.tiles <= kRowWaves ? kRowWaves : 2 * kRowWaves;
    const int items = (op.tiles + step - 1) / step * (op.flags & ROW_HALVES ? op.kt / 2 : op.kt);
    if (items <= kRowRing) op.flags |= ROW_SHORT;
    flops += 2.0 * a.batch * a.l * n * k;
    return op;
  };
  auto with_norm = [&](RowOp& op, int rows_at, const float* gain, const float* offset) {
    op.norm = rows_at; op.gain = vecs(gain, 1); op.offset = vecs(offset, 1);
    op.flags |= ROW_NORM;
  };
  int cur = lds_h;                                           // the rows as they are so far
  if (a.w_in) {
    gemm(lds_a, a.w_in, a.b_in, c, c, lds_h, -1);
  } else {
    if (!a.h || !a.text_k || !a.text_v || a.lk < 1) AD_FAIL(AD_ERR_INVALID, "tfm_rows: null pointer");
    p.h = a.h;
    p.tk = a.text_k; p.tv = a.text_v; p.Lk = a.lk; p.ldv = a.text_ldv; p.text_shared = a.text_shared;
    gemm(lds_a, a.w_o, a.b_o, c, c, lds_h, lds_h);
    RowOp& q = gemm(lds_a, a.w_q2, nullptr, c, c, lds_g, -1);
    with_norm(q, lds_h, a.ln2_g, a.ln2_b);
    q.flags |= ROW_TEXT;
    flops += 4.0 * a.batch * a.l * a.lk * c;
    gemm(lds_a, a.w_o2, a.b_o2, c, c, lds_h, lds_h);
    with_norm(gemm(lds_a, a.w_ff1, a.b_ff1, 8 * c, c, lds_g, -1, ROW_GEGLU), lds_h, a.ln3_g, a.ln3_b);
    gemm(lds_g, a.w_ff2, a.b_ff2, c, 4 * c, lds_h, lds_h);
  }
  if (a.w_out) {
    if (!a.x || !a.z) AD_FAIL(AD_ERR_INVALID, "tfm_rows: null pointer");
    p.x = a.x;
    gemm(lds_h, a.w_out, a.b_out, c, c, lds_a, lds_x);
    cur = lds_a;
  }
  p.put = a.w_out ? a.z : a.h;
  if (!p.put) AD_FAIL(AD_ERR_INVALID, "tfm_rows: null pointer");
  p.ops[p.n_ops - 1].flags |= ROW_PUT;
  if (a.w_qkv) {
    if (!a.q || !a.k || !a.v || (a.ld_t > 0 && a.ld_t < round_up(a.l, 8))) AD_FAIL(AD_ERR_INVALID, "tfm_rows: bad q/k/v");
    RowOp& op = gemm(cur == lds_h ? lds_a : lds_h, a.w_qkv, nullptr, 3 * c, c, lds_g, -1);
    with_norm(op, cur, a.ln_g, a.ln_b);
    op.flags &= (unsigned short)~ROW_SYNC;                   // the rows went out behind a barrier
    op.flags |= ROW_PUT_QKV;
    p.q = a.q; p.k = a.k; p.v = a.v; p.ld_t = a.ld_t;
  }
  p.ops[p.n_ops].flags = ROW_SHORT;                          // the empty operation
  p.div_tiles = make_fastdiv((unsigned)p.tiles);
  p.div_per = make_fastdiv((unsigned)(c * es / 16));
  const int lds_bytes = plan.bytes, grid = a.batch * p.tiles;
  if (p.n_ops >= kRowOps || p.n_vecs >= kRowVecs || lds_bytes > 160 * 1024) AD_FAIL(AD_ERR_INVALID, "tfm_rows: does not fit");
  ProfLaunch pl(a.dtype == AD_BF16 ? "tfm_rows_bf16" : "tfm_rows_f32", flops, 0, s, a.batch * a.l, c, a.w_o ? 15 * c : 4 * c);
#define AD_ROWS(T_, DT_) return plan.tm == 2 ? run_tfm_rows<T_, 2, DT_>(p, grid, lds_bytes, s) : run_tfm_rows<T_, 1, DT_>(p, grid, lds_bytes, s)
  if (a.dtype == AD_BF16) AD_ROWS(bf16, 4);
  if (a.head_dim == 16) AD_ROWS(float, 1);
  if (a.head_dim == 32) AD_ROWS(float, 2);
  AD_ROWS(float, 4);
#undef AD_ROWS
}

}  // namespace ad
