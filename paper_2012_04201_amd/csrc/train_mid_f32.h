// Register-resident training / scoring kernel for fp32 models with one hidden layer whose input or output side is too
// wide for train_small_f32.h (the digits shape: up to 127 inputs, hidden width up to 256, up to 16 outputs), on that
// kernel's row pipeline with an output layer on MFMA.  Wave w owns the unit tiles w, w + W, .. with their hidden
// parameters, moments and gradients in registers; the output layer's rows of those units in registers too, in the
// layout its gradient comes out in (lane: output li, units 4q..4q+3), their moments in LDS.
//
//   forward   D[row][unit] = xs[row][k] . w1[unit][k] on MFMA (16x16x4 fp32), ReLU in the accumulators.  Each
//             activation tile is turned over in an LDS patch of the wave's own (no workgroup barrier) to become the A
//             operand of z[row][out] += a[row][unit] . w2[unit][out]; the wave's partial outputs go to LDS.
//   outputs   rows are dealt to the waves in groups of four (lane: output li, row q): the sum of the waves' partials,
//             softmax / loss / delta with reductions over the 16 lanes of a row; the delta goes to LDS.
//   backward  hidden delta = delta . w2^T (w2 turned over in the patch), masked by the activations; it is the B operand
//             of the hidden layer's weight gradient, the activations are the A operand of the output layer's.
//   update    Adam / SGD on registers.
//
// Two workgroup barriers per chunk of 64 rows.  What bounds it: at 64 inputs, 10 outputs and 128 units the fp32 MFMA
// pipes are busy a third of the time, the rest is the chain of a chunk (LDS reads in front of the products, the output
// layer's reductions, the barriers) with two waves per SIMD to cover it.  Its predecessor kept the weights in LDS and the
// moments in L2, one model of 8 waves per CU, four barriers per chunk: 1000 models of 64-128-10 on 1797 rows, 3 epochs,
// took 5.5 ms and take 3.2 ms (64 units: 4.2 and 2.5 ms; 200 units: 8.7 and 5.1 ms).  With the row pipeline's leaner schedule
// and the input layer's products in split bfloat16 (md_splittable()) 512 suggestions of the digits shape took 14.0 ms instead
// of 15.5, 13.2 with the row tiles of a chunk together and moments in units of their own, and take 12.9 with rare code apart.
#pragma once
#include "common.h"
#include "train_small_f32.h"  // the row pipeline

namespace {

constexpr int MD_RS = 20;  // row stride of 16-wide LDS blocks: conflict-free both ways

// Reductions over the 16 lanes of a DPP row (the lanes that share lane / 16); every lane gets the result.
// Rotations by 8 and 4 within the row, then the two quad permutations: four cross-lane moves, no LDS traffic.
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
template <class Op>
__device__ __forceinline__ float r16_reduce(float v, Op op) {
  v = op(v, __builtin_bit_cast(float, dpp_mov<0x128>(__builtin_bit_cast(int, v))));
  v = op(v, __builtin_bit_cast(float, dpp_mov<0x124>(__builtin_bit_cast(int, v))));
  v = op(v, __builtin_bit_cast(float, dpp_mov<0x4E>(__builtin_bit_cast(int, v))));
  v = op(v, __builtin_bit_cast(float, dpp_mov<0xB1>(__builtin_bit_cast(int, v))));
  return v;
}
__device__ __forceinline__ float r16_sum(float v) {
  return r16_reduce(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float r16_max(float v) {
  return r16_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ int r16_min(int v) {
  v = min(v, dpp_mov<0x128>(v));
  v = min(v, dpp_mov<0x124>(v));
  v = min(v, dpp_mov<0x4E>(v));
  v = min(v, dpp_mov<0xB1>(v));
  return v;
}

struct MLay {
  PipeLay p;
  int32_t h, c, nut;
  int32_t cw[2], cb[2];
  uint32_t lds_total, slot_floats;
};
struct MItem {
  ItemDesc d;
  MLay y;
};

// Input-layer products in split bfloat16 (see SmPlanes)?  With eight waves and two to five input tiles (six and more leave no
// LDS for two buffers of planes).  With two unit tiles a wave the weights' planes push the moments out of the registers and an
// update takes 8000 cycles instead of 4500, which pays past a chunk of 64 rows a step, with three input tiles (three quarters
// of the products' columns) past a chunk and a half.  us a call with fp32 products and split, 10 classes, 3 epochs: 900 rows, 200
// suggestions, 64 inputs, 100 units at 32 and 160 rows a step 1930 and 1750, 1458 and 1219; 64 inputs, 200 units at 48, 65, 80,
// 96 and 128 rows 2659 and 2935, 3085 and 3207, 2508 and 2581, 2408 and 2356, 2293 and 2148; 1797 rows, 8 suggestions at 48, 65,
// 80 and 96 rows 1310 and 1332, 1500 and 1465, 1228 and 1197, 1173 and 1080: past a chunk what few models gain is what many
// lose, up to 96 rows.  45 inputs, 200 units at 65, 80 and 96 rows: 200 suggestions 2664 and 2736, 2160 and 2210, 2061 and 2032, 8
// suggestions 1299 and 1330, 1065 and 1086, 1009 and 984.  30 inputs: 1.01 of its time at most from 65 rows on.  (Four waves:
// 64 inputs, 64 units, 32 rows 1555 and 1566.)
__host__ __device__ constexpr bool md_splittable(int kt, int nt, int waves) {
  return waves == 8 && kt >= 2 && kt <= 5 && kt * nt <= 8;
}
// How a model is cut, by shape and batch size alone (a suggestion's scores may not depend on its companions); waves == 0: not a shape
// of this kernel.  One tile a wave while eight waves reach (more models a CU with four), else two: one tile leaves the
// registers for everything, and eight waves of one tile beat four of two by a quarter even with the chip full (64-100-10,
// 1000 models: 3.2 ms against 3.9).  Beyond kt * nt = 12 the weights and gradients alone overflow the registers; close to
// it they crowd others out: by the compiler's report <3,2,8> and <4,2,8> spill 10 vector registers, <5,2,8> 50, <6,2,8> 110,
// the split forms of <3,2,8> and <4,2,8> 24 and 45, the others 2 at most.  (<6,2,8> against its form before the leaner schedule, 90 inputs, 200 and
// 250 units: 0.95 at 32 rows a step, 1.02 to 1.04 at 65 to 128.)
__host__ inline SmallCut mid_cut(const int32_t* dims, int L, int32_t batch_size) {
  SmallCut m = {0, 0, 0, 0};
  if (L != 2 || dims[0] > 127 || dims[1] > 256 || dims[2] > 16) return m;
  const int nut = rup(dims[1], 16) / 16, waves = nut <= 4 ? 4 : 8;
  m.kt = rup(dims[0], 16) / 16;
  m.nt = (nut + waves - 1) / waves;
  m.waves = m.kt * m.nt <= 12 ? waves : 0;
  // (co: split products)
  m.co = md_splittable(m.kt, m.nt, waves) && (m.nt == 1 || batch_size <= 0 || batch_size > (m.kt == 3 ? 3 * SM_RC / 2 - 1 : SM_RC)) ? 1 : 0;
  return m;
}
__host__ __device__ constexpr int md_regs(int kt, int nt) { return nt * (4 * kt + 1 + 4) + 1; }
// Tiles of a wave whose hidden moments live in registers; the others' stay in global memory (the slot) and are read and
// written once per step, when the activations' registers are free.
__host__ __device__ constexpr int md_near(int kt, int nt, bool split) {
  return nt == 1 ? (kt <= 6 ? 1 : 0) : (split ? (kt <= 2 ? 2 : (kt == 3 ? 1 : 0)) : (kt <= 3 ? 2 : (kt == 4 ? 1 : 0)));
}
__host__ __device__ constexpr uint32_t md_fixed_lds(int kt, int nt, int waves, bool split) {
  // partial outputs, deltas, and per wave: the moments of w2, the bias moments
  return pipe_lds(kt, 2, split) + (waves * SM_RC * MD_RS + SM_RC * MD_RS + waves * (nt * 2 * 256 + (nt + 1) * 32)) * 4;
}
__host__ inline void make_mlay(MLay& y, const int32_t* dims, int64_t n, const SmallCut& m) {
  const int d = dims[0];
  y.h = dims[1];
  y.c = dims[2];
  y.nut = rup(dims[1], 16) / 16;
  y.cw[0] = 0;
  y.cb[0] = d * y.h;
  y.cw[1] = y.cb[0] + y.h;
  y.cb[1] = y.cw[1] + y.h * y.c;
  make_pipelay(y.p, d, y.cb[1] + y.c, n, md_fixed_lds(m.kt, m.nt, m.waves, m.co));
  y.slot_floats = (uint32_t)(m.waves * (md_regs(m.kt, m.nt) + (m.nt - md_near(m.kt, m.nt, m.co)) * 8 * m.kt) * 64);
  y.lds_total = y.p.total;
}
// workgroups a CU holds: registers are budgeted for two waves per SIMD
__host__ inline int md_per_cu(const SmallCut& m, uint32_t lds_bytes) {
  const int by_regs = 8 / m.waves, by_lds = (int)(160u * 1024u / (lds_bytes + 512));
  const int n = by_regs < by_lds ? by_regs : by_lds;
  return n < 1 ? 1 : n;
}

template <int KT, int NT, int W, bool SPLIT>
struct Mid : RowPipe<Mid<KT, NT, W, SPLIT>, MLay, KT, W, 2, SPLIT> {
  typedef RowPipe<Mid<KT, NT, W, SPLIT>, MLay, KT, W, 2, SPLIT> Base;
  using Base::Base;
  using Base::f;
  using Base::init_value;
  using Base::it;
  using Base::n_classes;
  using Base::red;
  using Base::slot;
  using Base::tid;
  using Base::wave;
  using Base::xs;
  using Base::y;
  using Base::ys;
  static constexpr int LDW = Base::LDW;
  int nut = 0, c = 0;
  __device__ __forceinline__ void pin_own() {
    nut = pin(y.nut);
    c = pin(y.c);
  }
  __device__ __forceinline__ double total(double v) const { return block_sum(v, red); }

  static constexpr int NEAR = md_near(KT, NT, SPLIT), NREGM = NEAR ? NEAR : 1;
  static constexpr int KB = sm_blocks(KT);
  static constexpr bool LOAD_AHEAD = false;  // (see Small)
  // (us a call without and with, 24 rows a step: 40 models 900 x 48, ten classes, 150 units 2050 and 2028; 500 of 900 x 90, 250 units
  // 4909 and 5258)
  static constexpr bool RARE_APART = !(NT == 2 && KT >= 5);
  // The forward pass takes the row tiles of a chunk together, except where their operands do not fit the registers: us a call one
  // by one and together, 200 suggestions: 64 inputs, 10 classes, 150 units, 128 rows a step, split 2377 and 2493; 80 inputs, 190
  // units, 24 rows 5809 and 6233; but fp32 products, 64 inputs, 150 units, 64 rows 2663 and 2576; 64 units, 128 rows 1473 and 1412;
  // 80 inputs, 50 units, 128 rows 1256 and 1188.
  static constexpr bool CROWDED = NT == 2 && KT >= (SPLIT ? 4 : 5);
  static constexpr int GROUP = NT == 1 ? 2 : 1;  // row tiles whose hidden products take turns
  struct State {
    HiddenWeights<KT, NT, SPLIT> w;
    f32x4 m[NREGM][KT], v[NREGM][KT], g[NT][KT];       // hidden layer: lane (unit li, columns 16 kk + 4q + e)
    float bw[NT], bg[NT];                              // its bias
    f32x4 w2[NT], g2[NT];                              // output layer: lane (output li, units 4q + e of the tile)
    float ow, og;                                      // output bias: output li, alike in every q and wave
  };
  struct Acts {
    f32x4 a[NT][4];  // lane (unit li, rows 16 r + 4q..+3)
  };
  static constexpr int O_ZP = Base::O_OWN, O_D3 = O_ZP + W * SM_RC * MD_RS, O_M2 = O_D3 + SM_RC * MD_RS, O_MOM = O_M2 + W * NT * 512, O_TOP = O_MOM + W * (NT + 1) * 32;
  static_assert(O_TOP * 4 == md_fixed_lds(KT, NT, W, SPLIT), "LDS layout");
  __device__ __forceinline__ bool has(int i, int w) const { return i + 1 < NT || w + i * W < nut; }
  // A 16 x 16 block of four values a lane (lane: column li, rows 4q..4q+3) turned over: lane li gets row li, columns
  // 4q..4q+3.  The patch is where the wave's partial outputs of row tile r go once it is done: the wave's LDS accesses
  // stay in order, and nobody else reads them between the outputs of a chunk and the first barrier of the next.
  __device__ __forceinline__ void turn_put(const f32x4& v, int r) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    float* p = f(O_ZP) + (wave() * SM_RC + r * 16 + 4 * q) * MD_RS + li;
#pragma unroll
    for (int e = 0; e < 4; e++) p[e * MD_RS] = v[e];
  }
  __device__ __forceinline__ f32x4 turn_get(int r) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    return *(const f32x4*)(f(O_ZP) + (wave() * SM_RC + r * 16 + li) * MD_RS + 4 * q);
  }
  __device__ __forceinline__ f32x4 turn(const f32x4& v, int r) const {
    turn_put(v, r);
    __builtin_amdgcn_wave_barrier();
    const f32x4 t = turn_get(r);
    __builtin_amdgcn_wave_barrier();
    return t;
  }
  __device__ __forceinline__ f32x4* mom2(int i, int which) const {
    return (f32x4*)(f(O_M2) + ((wave() * NT + i) * 2 + which) * 256) + (threadIdx.x & 63);
  }
  // moments of the biases: k < NT the tile's units, k == NT the outputs; alike in the four q
  __device__ __forceinline__ float* mom(int k, int which) const {
    return f(O_MOM) + ((wave() * (NT + 1) + k) * 2 + which) * 16 + (threadIdx.x & 15);
  }

  // ---- parameters ----------------------------------------------------------
  static constexpr int NREG = md_regs(KT, NT), PER = 4 * KT + 1 + 4;
  __device__ __forceinline__ float* park() const { return slot + wave() * (NREG * 64) + (threadIdx.x & 63); }
  __device__ __forceinline__ void unpack(const float* st, float unit = 1.f) const {
    const int lane = threadIdx.x & 63, w_ = wave(), li = lane & 15, q = lane >> 4;
    const int d = y.p.d, h = y.h;
    float* b = park();
#pragma unroll 1
    for (int n = 0; n < NREG; n++) {
      const int i = n / PER, r = n - i * PER, j = (w_ + i * W) * 16 + li;
      int l = 0, ci = -1, e = 0;
      bool isb = false;
      if (i == NT) {  // output bias
        l = 1;
        isb = true;
        e = li;
        if (li < c) ci = y.cb[1] + li;
      } else if (r < 4 * KT) {
        const int k = (r >> 2) * 16 + 4 * q + (r & 3);
        e = k * h + j;
        if (j < h && k < d) ci = y.cw[0] + e;
      } else if (r == 4 * KT) {
        isb = true;
        e = j;
        if (j < h) ci = y.cb[0] + j;
      } else {
        l = 1;
        const int u = (w_ + i * W) * 16 + 4 * q + (r - 4 * KT - 1);
        e = u * c + li;
        if (u < h && li < c) ci = y.cw[1] + e;
      }
      float val = 0.f;
      if (ci >= 0) val = st ? st[ci] * unit : init_value(l, e, isb);
      b[64 * n] = val;
    }
  }
  // moments of tile i >= NEAR: [which][kk], four values a lane
  typedef __attribute__((address_space(1))) f32x4 GlobalF32x4;
  __device__ __forceinline__ GlobalF32x4* far(int i, int which, int kk) const {
    return (GlobalF32x4*)(slot + W * (NREG * 64) + (((wave() * (NT - NEAR) + i - NEAR) * 2 + which) * KT + kk) * 256) +
           (threadIdx.x & 63);
  }
  // fn(index, reference) for the hidden weights or one of their moments
  template <class F>
  __device__ __forceinline__ static void each_hidden(HiddenWeights<KT, NT, SPLIT>& w, F fn) {
#pragma unroll
    for (int i = 0; i < NT; i++)
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        f32x4 x = w.get(i, kk);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float y_ = x[e];
          fn(i * PER + 4 * kk + e, y_);
          x[e] = y_;
        }
        w.put(i, kk, x);
      }
  }
  template <int N, class F>
  __device__ __forceinline__ static void each_hidden(f32x4 (&w)[N][KT], F fn) {
#pragma unroll
    for (int i = 0; i < N; i++)
#pragma unroll
      for (int kk = 0; kk < KT; kk++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float x = w[i][kk][e];
          fn(i * PER + 4 * kk + e, x);
          w[i][kk][e] = x;
        }
  }
  __device__ __forceinline__ void load(State& R, const float* st, float um, float uv) const {
    const float* b = park();
    auto take = [&](int n, float& x) { x = b[64 * n]; };
    auto zero = [&](int, float& x) { x = 0.f; };
#pragma unroll
    for (int which = 0; which < 2; which++) {
      if (st) unpack(st + (1 + which) * y.p.P, which ? uv : um);
      if constexpr (NEAR > 0) {
        if (st)
          each_hidden(which ? R.v : R.m, take);
        else
          each_hidden(which ? R.v : R.m, zero);
      }
#pragma unroll
      for (int i = NEAR; i < NT; i++)
#pragma unroll
        for (int kk = 0; kk < KT; kk++) {
          f32x4 x = f32x4{0.f, 0.f, 0.f, 0.f};
          if (st) {
#pragma unroll
            for (int e = 0; e < 4; e++) x[e] = b[64 * (i * PER + 4 * kk + e)];
          }
          *far(i, which, kk) = x;
        }
#pragma unroll
      for (int i = 0; i < NT; i++) {
        f32x4 x = f32x4{0.f, 0.f, 0.f, 0.f};
        if (st) {
#pragma unroll
          for (int e = 0; e < 4; e++) x[e] = b[64 * (i * PER + 4 * KT + 1 + e)];
        }
        *mom2(i, which) = x;
        *mom(i, which) = st ? b[64 * (i * PER + 4 * KT)] : 0.f;
      }
      *mom(NT, which) = st ? b[64 * (NT * PER)] : 0.f;
    }
    unpack(st);
    restore_best(R);
  }
  __device__ __forceinline__ void keep_best(State& R) const {
    float* b = park();
    each_hidden(R.w, [&](int n, float& x) { b[64 * n] = x; });
#pragma unroll
    for (int i = 0; i < NT; i++) {
      b[64 * (i * PER + 4 * KT)] = R.bw[i];
#pragma unroll
      for (int e = 0; e < 4; e++) b[64 * (i * PER + 4 * KT + 1 + e)] = R.w2[i][e];
    }
    b[64 * (NT * PER)] = R.ow;
  }
  __device__ __forceinline__ void restore_best(State& R) const {
    const float* b = park();
    each_hidden(R.w, [&](int n, float& x) { x = b[64 * n]; });
#pragma unroll
    for (int i = 0; i < NT; i++) {
      R.bw[i] = b[64 * (i * PER + 4 * KT)];
#pragma unroll
      for (int e = 0; e < 4; e++) R.w2[i][e] = b[64 * (i * PER + 4 * KT + 1 + e)];
    }
    R.ow = b[64 * (NT * PER)];
    __builtin_amdgcn_s_waitcnt(0);  // see k_train_small
  }
  __device__ __forceinline__ static void zero_grad(State& R) {
#pragma unroll
    for (int i = 0; i < NT; i++) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++) R.g[i][kk] = f32x4{0.f, 0.f, 0.f, 0.f};
      R.bg[i] = 0.f;
      R.g2[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    R.og = 0.f;
  }

  // ---- forward ---------------------------------------------------------------
  // The wave's hidden tiles of N row tiles from R0 on and then their shares of the outputs, each step of it for all of them
  // before the next: they wait for LDS and for each other's products together.
  template <bool ALL, int R0, int N>
  __device__ __forceinline__ void forward_rows(const State& R, int b, f32x4 (&acc)[NT][4]) const {
    constexpr int TILES = NT - (ALL ? 0 : 1);
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < TILES; i++) {
      float x = R.bw[i];
      // (as in the small kernel: keeps the small parameters out of scratch memory, where the registers have room for them)
      if (!(SPLIT && KT == 4)) asm("" : "+v"(x));
#pragma unroll
      for (int r = R0; r < R0 + N; r++) acc[i][r] = f32x4{x, x, x, x};
    }
    if constexpr (TILES > 0) {
#pragma unroll
      for (int r = R0; r < R0 + N; r += GROUP) {
        if constexpr (SPLIT) {
#pragma unroll
          for (int kb = 0; kb < KB; kb++) {
            SmPlanes a[GROUP];
#pragma unroll
            for (int g = 0; g < GROUP; g++)
              if (r + g < R0 + N) a[g] = Base::by_row(Base::planes(b), r + g, kb);
            hidden_products<TILES, R0 + N>(a, R.w.p[kb], r, acc);
          }
        } else {
#pragma unroll
          for (int g = 0; g < GROUP; g++) {
            if (r + g >= R0 + N) continue;
            const float* a_ = xs(b) + ((r + g) * 16 + li) * LDW + 4 * q;
            f32x4 a[KT];
#pragma unroll
            for (int kk = 0; kk < KT; kk++) a[kk] = *(const f32x4*)(a_ + kk * 16);
#pragma unroll
            for (int kk = 0; kk < KT; kk++)
#pragma unroll
              for (int e = 0; e < 4; e++)
#pragma unroll
                for (int i = 0; i < TILES; i++)
                  acc[i][r + g] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk][e], R.w.w[i][kk][e], acc[i][r + g], 0, 0, 0);
          }
        }
      }
    }
    f32x4 z[N];
#pragma unroll
    for (int n = 0; n < N; n++) z[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < TILES; i++) {
      f32x4 ar[N];  // row li, units 4q..4q+3
#pragma unroll
      for (int n = 0; n < N; n++) {
#pragma unroll
        for (int e = 0; e < 4; e++) acc[i][R0 + n][e] = relu(acc[i][R0 + n][e]);
        turn_put(acc[i][R0 + n], R0 + n);
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int n = 0; n < N; n++) ar[n] = turn_get(R0 + n);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int n = 0; n < N; n++) z[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[n][e], R.w2[i][e], z[n], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < N; n++) {
      float* zp = f(O_ZP) + (wave() * SM_RC + (R0 + n) * 16 + 4 * q) * MD_RS + li;
#pragma unroll
      for (int e = 0; e < 4; e++) zp[e * MD_RS] = z[n][e];
    }
  }
  // one of the six split products of the group's row tiles from r on after the other
  template <int TILES, int END, int S = 0>
  __device__ __forceinline__ static void hidden_products(const SmPlanes (&a)[GROUP], const SmPlanes (&w)[NT], int r, f32x4 (&acc)[NT][4]) {
#pragma unroll
    for (int g = 0; g < GROUP; g++)
#pragma unroll
      for (int i = 0; i < TILES; i++)
        if (r + g < END) acc[i][r + g] = sm_product<S>(a[g], w[i], acc[i][r + g]);
    if constexpr (S < 5) hidden_products<TILES, END, S + 1>(a, w, r, acc);
  }
  template <bool ALL>
  __device__ __forceinline__ void forward_chunk(const State& R, int b, int nrt, f32x4 (&acc)[NT][4]) const {
    if constexpr (CROWDED) {  // row tile by row tile
      forward_rows<ALL, 0, 1>(R, b, acc);
      if (nrt > 1) forward_rows<ALL, 1, 1>(R, b, acc);
      if (nrt > 2) forward_rows<ALL, 2, 1>(R, b, acc);
      if (nrt > 3) forward_rows<ALL, 3, 1>(R, b, acc);
    } else if (nrt == 4) {
      forward_rows<ALL, 0, 4>(R, b, acc);
    } else if (nrt == 3) {
      forward_rows<ALL, 0, 3>(R, b, acc);
    } else if (nrt == 2) {
      forward_rows<ALL, 0, 2>(R, b, acc);
    } else {
      forward_rows<ALL, 0, 1>(R, b, acc);
    }
  }
  __device__ __forceinline__ void forward(const State& R, int b, int, int nrt, Acts& A) const {
    if (has(NT - 1, wave()))
      forward_chunk<true>(R, b, nrt, A.a);
    else
      forward_chunk<false>(R, b, nrt, A.a);
  }

  // ---- outputs: group g of four rows belongs to wave g mod W; lane (output li, row 4g + q) ----
  __device__ __forceinline__ void outputs(State& R, int b, int, int rows, bool train, bool loss, float inv_mb, double& lsum, double& hits) const {
    const int lane = tid() & 63, w_ = wave(), li = lane & 15, q = lane >> 4, groups = (rows + 3) / 4;
    float* d3 = f(O_D3);
#pragma unroll
    for (int g0 = 0; g0 < SM_RC / 4; g0 += W) {
      if (g0 >= groups) {  // rows nobody has: their deltas are still read with their row tile
        if (train && g0 < (groups + 3) / 4 * 4) d3[(4 * (g0 + w_) + q) * MD_RS + li] = 0.f;
        continue;
      }
      const int row = 4 * (g0 + w_) + q;
      const float* zp = f(O_ZP) + row * MD_RS + li;
      float z = R.ow;
#pragma unroll
      for (int ww = 0; ww < W; ww++) z += zp[ww * (SM_RC * MD_RS)];
      const bool valid = row < rows;
      const float yv = ys(b)[row];
      float dl = 0.f;
      if (n_classes >= 2) {
        const int yr = __float_as_int(yv);
        const float zz = li < c ? z : -INFINITY;
        const float mx = r16_max(zz);
        const float ex = li < c ? expf(zz - mx) : 0.f, se = r16_sum(ex);
        if (loss) {
          if (valid && li == 0) lsum += (double)(mx + logf(se));
          if (valid && li == yr && li < c) lsum -= (double)zz;  // (a label outside [0, c) matches no class)
        }
        if (!train) {
          const int best = r16_min(zz == mx ? li : 99);
          if (valid && li == 0) hits += best == yr ? 1.0 : 0.0;
        }
        if (valid && li < c) dl = (ex * (1.f / se) - (li == yr ? 1.f : 0.f)) * inv_mb;
      } else if (n_classes == 1) {
        // one logit, labels 0/1: log(1 + e^z) - y z, delta (sigmoid(z) - y)/m
        const int yr = __float_as_int(yv);
        if (valid && li == 0) {
          if (loss) {
            lsum += (double)(fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - (yr ? z : 0.f));
            hits += (z > 0.f) == (yr != 0) ? 1.0 : 0.0;
          }
          dl = (1.f / (1.f + expf(-z)) - (float)yr) * inv_mb;
        }
      } else {
        const float e0 = z - yv;
        if (valid && li == 0) {
          if (loss) {
            lsum += train ? 0.5 * (double)e0 * (double)e0 : (double)e0 * (double)e0;
            hits += (double)fabsf(e0);  // the absolute error
          }
          dl = e0 * inv_mb;
        }
      }
      if (train) d3[row * MD_RS + li] = dl;
    }
  }

  // ---- backward ----------------------------------------------------------------
  // the hidden deltas of a row tile, and its share of the output layer's gradient
  template <bool ALL>
  __device__ __forceinline__ void deltas(State& R, int r, const f32x4 (&acc)[NT][4], const f32x4 (&wt)[NT], f32x4 (&dh)[NT]) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    const float* d3 = f(O_D3);
    const f32x4 da = *(const f32x4*)(d3 + (r * 16 + li) * MD_RS + 4 * q);  // A: row li, outputs 4q..4q+3
    float db[4];
#pragma unroll
    for (int e = 0; e < 4; e++) db[e] = d3[(r * 16 + 4 * q + e) * MD_RS + li];  // B: row 4q + e, output li
#pragma unroll
    for (int i = 0; i < NT; i++) dh[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; e++) {
      R.og += db[e];
#pragma unroll
      for (int i = 0; i < NT; i++)
        if (i + 1 < NT || ALL) {
          dh[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(da[e], wt[i][e], dh[i], 0, 0, 0);
          R.g2[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(acc[i][r][e], db[e], R.g2[i], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < NT; i++)
      if (i + 1 < NT || ALL) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float x = acc[i][r][e] > 0.f ? dh[i][e] : 0.f;
          dh[i][e] = x;
          R.bg[i] += x;
        }
      }
  }
  // the hidden weights' gradient of a row tile ...
  template <bool ALL>
  __device__ __forceinline__ void backward_tile(State& R, const float* s, int r, const f32x4 (&acc)[NT][4], const f32x4 (&wt)[NT]) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    float a[KT][4];
    const float* a_ = s + (r * 16 + 4 * q) * LDW + li;
#pragma unroll
    for (int kk = 0; kk < KT; kk++)
#pragma unroll
      for (int e = 0; e < 4; e++) a[kk][e] = a_[e * LDW + kk * 16];
    f32x4 dh[NT];
    deltas<ALL>(R, r, acc, wt, dh);
#pragma unroll
    for (int kk = 0; kk < KT; kk++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
#pragma unroll
        for (int i = 0; i < NT; i++)
          if (i + 1 < NT || ALL) R.g[i][kk] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk][e], dh[i][e], R.g[i][kk], 0, 0, 0);
      }
  }
  // ... or of two, r and r + 1 (BOTH), which fill the 32 contracted rows of a split product
  template <bool ALL, bool BOTH>
  __device__ __forceinline__ void backward_pair(State& R, const char* x, int r, const f32x4 (&acc)[NT][4], const f32x4 (&wt)[NT]) const {
    constexpr int TILES = NT - (ALL ? 0 : 1);
    SmPlanes dp[NT];
#pragma unroll
    for (int t = 0; t < 2; t++) {
      f32x4 dh[NT];
      if (t == 0 || BOTH) deltas<ALL>(R, r + t, acc, wt, dh);
#pragma unroll
      for (int i = 0; i < TILES; i++)
#pragma unroll
        for (int e = 0; e < 2; e++) {
          uint32_t h = 0u, m = 0u, l = 0u;
          if (t == 0 || BOTH) sm_split2(dh[i][2 * e], dh[i][2 * e + 1], h, m, l);
          dp[i].h[2 * t + e] = h;
          dp[i].m[2 * t + e] = m;
          dp[i].l[2 * t + e] = l;
        }
    }
    if constexpr (TILES > 0) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        f32x4 c[NT];
#pragma unroll
        for (int i = 0; i < TILES; i++) c[i] = R.g[i][kk];
        sm_products<TILES>(Base::template by_column<BOTH>(x, r, kk), dp, c);
#pragma unroll
        for (int i = 0; i < TILES; i++) R.g[i][kk] = c[i];
      }
    }
  }
  template <bool ALL>
  __device__ __forceinline__ void backward_chunk(State& R, int b, int nrt, const f32x4 (&acc)[NT][4]) const {
    f32x4 wt[NT];  // unit li, outputs 4q..4q+3
#pragma unroll
    for (int i = 0; i < NT; i++) wt[i] = turn(R.w2[i], 0);
    if constexpr (SPLIT) {
      const char* x = Base::planes(b);
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        if (r >= nrt) break;
        if (r + 1 < nrt)
          backward_pair<ALL, true>(R, x, r, acc, wt);
        else
          backward_pair<ALL, false>(R, x, r, acc, wt);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; r++) {
        if (r >= nrt) break;
        backward_tile<ALL>(R, xs(b), r, acc, wt);
      }
    }
  }
  __device__ __forceinline__ void backward(State& R, int b, int nrt, const Acts& A) const {
    if (has(NT - 1, wave()))
      backward_chunk<true>(R, b, nrt, A.a);
    else
      backward_chunk<false>(R, b, nrt, A.a);
  }

  // ---- optimizer step (pads: see k_train_small) ----------------------------------
  template <bool ADAM>
  __device__ __forceinline__ void update(State& R, const OptC& oc) const {
    const int w_ = wave();
    OptC o = oc;
    o.adam = ADAM;
    f32x4 mf[NT - NEAR + 1][KT], vf[NT - NEAR + 1][KT];  // moments from the slot, all requested at once
#pragma unroll
    for (int i = NEAR; i < NT; i++)
      if (has(i, w_)) {
#pragma unroll
        for (int kk = 0; kk < KT; kk++) {
          mf[i - NEAR][kk] = *far(i, 0, kk);
          if (ADAM) vf[i - NEAR][kk] = *far(i, 1, kk);
        }
      }
    f32x4 m2[NT], v2[NT];
    float gb[NT + 1], mb[NT + 1], vb[NT + 1];
#pragma unroll
    for (int i = 0; i < NT; i++) {
      m2[i] = *mom2(i, 0);
      v2[i] = ADAM ? *mom2(i, 1) : f32x4{0.f, 0.f, 0.f, 0.f};
      gb[i] = R.bg[i];
    }
    gb[NT] = R.og;
#pragma unroll
    for (int k = 0; k <= NT; k++) {
      mb[k] = *mom(k, 0);
      vb[k] = ADAM ? *mom(k, 1) : 0.f;
    }
#pragma unroll
    for (int k = 0; k <= NT; k++) gb[k] += __shfl_xor(gb[k], 16);
#pragma unroll
    for (int k = 0; k <= NT; k++) gb[k] += __shfl_xor(gb[k], 32);
#pragma unroll
    for (int i = 0; i < NT; i++)
      if (has(i, w_)) {
#pragma unroll
        for (int kk = 0; kk < KT; kk++) {
          f32x4& mm = i < NEAR ? R.m[i < NEAR ? i : 0][kk] : mf[i < NEAR ? 0 : i - NEAR][kk];
          f32x4& vv = i < NEAR ? R.v[i < NEAR ? i : 0][kk] : vf[i < NEAR ? 0 : i - NEAR][kk];
          f32x4 x = R.w.get(i, kk);
#pragma unroll
          for (int e = 0; e < 4; e++) {
            float wr = x[e], mr = mm[e], vr = vv[e];
            opt_step(o, R.g[i][kk][e] + o.am * wr, wr, mr, vr);
            x[e] = wr;
            mm[e] = mr;
            vv[e] = vr;
          }
          R.w.put(i, kk, x);
        }
        if (i >= NEAR) {
#pragma unroll
          for (int kk = 0; kk < KT; kk++) {
            *far(i, 0, kk) = mf[i < NEAR ? 0 : i - NEAR][kk];
            if (ADAM) *far(i, 1, kk) = vf[i < NEAR ? 0 : i - NEAR][kk];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float wr = R.w2[i][e], mr = m2[i][e], vr = v2[i][e];
          opt_step(o, R.g2[i][e] + o.am * wr, wr, mr, vr);
          R.w2[i][e] = wr;
          m2[i][e] = mr;
          v2[i][e] = vr;
        }
        *mom2(i, 0) = m2[i];
        if (ADAM) *mom2(i, 1) = v2[i];
      }
#pragma unroll
    for (int k = 0; k <= NT; k++) {
      opt_step(o, gb[k], k < NT ? R.bw[k < NT ? k : 0] : R.ow, mb[k], vb[k]);
      *mom(k, 0) = mb[k];
      if (ADAM) *mom(k, 1) = vb[k];
    }
  }
  template <bool GRAD>
  __device__ __forceinline__ void record(const State& R, float am, float* out) const {
    const int t_ = tid(), lane = t_ & 63, w_ = wave(), li = lane & 15, q = lane >> 4;
    const int d = y.p.d, h = y.h;
#pragma unroll
    for (int i = 0; i < NT; i++) {
      const int t0 = (w_ + i * W) * 16, j = t0 + li;
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        const f32x4 x = R.w.get(i, kk);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int k = kk * 16 + 4 * q + e;
          if (j < h && k < d) out[y.cw[0] + k * h + j] = GRAD ? R.g[i][kk][e] + am * x[e] : x[e];
        }
      }
      const float b = GRAD ? sm_rowsum(R.bg[i]) : R.bw[i];
      if (j < h && q == 0) out[y.cb[0] + j] = b;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int u = t0 + 4 * q + e;
        if (u < h && li < c) out[y.cw[1] + u * c + li] = GRAD ? R.g2[i][e] + am * R.w2[i][e] : R.w2[i][e];
      }
    }
    const float o = GRAD ? sm_rowsum(R.og) : R.ow;
    if (t_ < c) out[y.cb[1] + t_] = o;
  }
  __device__ __forceinline__ double penalty_sum(const State& R) const {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NT; i++) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        const f32x4 x = R.w.get(i, kk);
#pragma unroll
        for (int e = 0; e < 4; e++) s += (double)x[e] * (double)x[e];
      }
#pragma unroll
      for (int e = 0; e < 4; e++) s += (double)R.w2[i][e] * (double)R.w2[i][e];
    }
    return block_sum(s, red);
  }
};

template <int KT, int NT, int W, bool SPLIT>
__device__ __forceinline__ void mid_models(const TrainParams& P) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_item;
  __shared__ double red[W], trace_stash[2];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    if (item >= P.n_items) break;
    const __attribute__((address_space(4))) MItem* mi = (const __attribute__((address_space(4))) MItem*)P.items + item / P.n_folds;
    Mid<KT, NT, W, SPLIT> T(P, mi->d, mi->y, smem, (float*)(P.slots + (uint64_t)blockIdx.x * P.slot_bytes), red, trace_stash,
                            item % P.n_folds);
    T.run();
  }
}
// the products as they are with one unit tile a wave, and up to 64 or 95 rows a step with two ...
template <int KT, int NT, int W>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * W, 64 * W), amdgpu_waves_per_eu(2, 2)))
void k_train_mid(const TrainParams P) {
  mid_models<KT, NT, W, NT == 1 && md_splittable(KT, NT, W)>(P);
}
// ... and split with two
template <int KT>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void k_train_mid2_split(const TrainParams P) {
  mid_models<KT, 2, 8, true>(P);
}

}  // namespace
