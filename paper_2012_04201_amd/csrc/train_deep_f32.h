// Training / scoring kernel for fp32 models with two or three hidden layers (up to 64 inputs, hidden widths up to 128, up
// to 16 outputs) on the row pipeline of train_small_f32.h.
//
// One workgroup trains one model.  Wave w owns unit tile w (16 units) of every level: its gradients, and its weights where
// they fit (dp_stream()), stay in registers for the whole run, as blocks of four values a lane in the layout the MFMA
// (16x16x4 fp32) both takes them in and leaves their gradient in (lane: unit li, columns 4q..4q+3 of a k tile).  The levels of a chunk of 64 rows
// lie in LDS, row-major, because every wave needs all of them; a level's deltas are written over its activations.
//
//   forward   level l+1 [row][unit] = level l . W: operand rows from LDS, weights from registers, ReLU, back to LDS
//   outputs   wave r takes row tile r: z = last level . W_out (its blocks gathered in LDS), softmax / loss / delta with
//             reductions over the 16 lanes of a row
//   backward  the data gradient contracts over a level's units, which are spread over the waves: their weights are in global
//             memory too (they stay in L2), in an order that can be read along either side of a tile, and are fetched
//             once per chunk; the weight gradient takes a level's activations from LDS and the wave's own deltas from registers
//   update    Adam / SGD; the moments in registers where they fit, else in global memory, touched once per step
//
// Four waves up to 64 units (two models a CU), eight up to 128.  Barriers per chunk: 6 with two hidden layers, 9 with
// three; per step one more where the second hidden layer has more than 64 units.  What bounds it: two waves per SIMD in step
// with each other, the waves past a narrow level's tiles idle, and the chain of a chunk's phases; the kernel for any shape,
// which these models ran on before, kept every operand in global
// memory.  256 suggestions x 5 folds on 569 x 30, one to three layers of 16..128 units, 10 epochs: 25.4 -> 9.4 ms a call, and
// 8.0 with the moments' branches gone, the weights of the widest cuts in global memory alone and operands read a tile ahead.
#pragma once
#include <type_traits>

#include "common.h"
#include "train_mid_f32.h"  // reductions over 16 lanes; the row pipeline

namespace {

struct DLay {
  PipeLay p;
  int32_t U[5], T[5];  // units and 16-wide tiles per level: inputs, hidden.., outputs
  int32_t cw[4], cb[4];
  uint32_t lds_total, slot_floats;
  int32_t per_wave, region;  // blocks of a wave, its biases apart; 16-byte vectors of a set of blocks in the slot
};
struct DItem {
  ItemDesc d;
  DLay y;
};

// How a model is cut, by shape alone; nt: hidden layers; waves == 0: not a shape of this kernel.
__host__ inline SmallCut deep_cut(const int32_t* dims, int L) {
  SmallCut m = {0, 0, 0, 0};
  if (L < 3 || L > 4 || dims[0] > 64 || dims[L] > 16) return m;
  int widest = 0;
  for (int l = 1; l < L; l++) widest = dims[l] > widest ? dims[l] : widest;
  if (widest > 128) return m;
  m.kt = rup(dims[0], 16) / 16;
  m.nt = L - 1;
  m.waves = widest <= 64 ? 4 : 8;
  return m;
}
// Blocks of four values a lane holds: input layer, hidden layers, output layer, biases.
__host__ __device__ constexpr int dp_blocks(int kt, int h, int waves) { return kt + (h - 1) * waves + 2; }
// The moments live in registers up to here (with weights and gradients four times the blocks, of 256 registers).  Without
// them three layers on eight waves still overflow: dp_stream().
__host__ __device__ constexpr bool dp_near(int kt, int h, int waves) { return dp_blocks(kt, h, waves) <= 8; }
// The weights of the hidden layers past the first are in global memory alone (one copy serves the forward products, the
// data gradient and the update) where weights and gradients would take 152 registers and more: held, they made these cuts
// spill 59, 117, 151 and 172 vector registers at one to four input tiles; now 0, 0, 2 and 4.  [128, 40, 100] on 50 inputs,
// batch 24: 500 models a call 4.70 -> 3.29 ms, 20 models 1.73 -> 1.37.  The price is the bandwidth of a full chip where
// little was spilled: [128, 128, 128] on 20 inputs 5.37 -> 5.77 ms at batch 24 and 2.43 -> 2.31 at 160.
__host__ __device__ constexpr bool dp_stream(int h, int waves) { return h == 3 && waves == 8; }
__host__ __device__ constexpr uint32_t dp_fixed_lds(int kt, int h, int waves) {
  // levels, the output layer's blocks, output deltas
  return pipe_lds(kt, 1, false) + (h * SM_RC * (16 * waves + 4) + waves * 256 + SM_RC * MD_RS) * 4;
}
__host__ inline void make_dlay(DLay& y, const int32_t* dims, int L, int64_t n, const SmallCut& m) {
  int c = 0;
  for (int l = 0; l <= L; l++) {
    y.U[l] = dims[l];
    y.T[l] = rup(dims[l], 16) / 16;
  }
  for (int l = 0; l < L; l++) {
    y.cw[l] = c;
    c += dims[l] * dims[l + 1];
    y.cb[l] = c;
    c += dims[l + 1];
  }
  make_pipelay(y.p, dims[0], c, n, dp_fixed_lds(m.kt, m.nt, m.waves));
  // the slot: parameters as they are drawn, later the best epoch's; moments; transposed hidden weights.  Only the tiles
  // there are take room: a narrow model's slot is no larger than one of the kernel for any shape.
  int owners = 0, turned = 0;
  y.per_wave = m.kt + 1;
  for (int l = 1; l < L; l++) {
    owners = y.T[l] > owners ? y.T[l] : owners;
    if (l + 1 < L) {
      y.per_wave += y.T[l];
      turned += y.T[l] * y.T[l + 1];
    }
  }
  y.region = (owners * y.per_wave + m.waves) * 64;
  y.slot_floats = (uint32_t)(4 * y.region * (dp_near(m.kt, m.nt, m.waves) ? 1 : 3) + turned * 256);
  y.lds_total = y.p.total;
}
// workgroups a CU holds: registers are budgeted for two waves per SIMD
__host__ inline int deep_per_cu(const SmallCut& m, uint32_t lds_bytes) {
  const int by_regs = 8 / m.waves, by_lds = (int)(160u * 1024u / (lds_bytes + 512));
  const int n = by_regs < by_lds ? by_regs : by_lds;
  return n < 1 ? 1 : n;
}

// H: hidden layers.  W: waves, and the most 16-unit tiles a hidden level has.
template <int KT, int H, int W>
struct Deep : RowPipe<Deep<KT, H, W>, DLay, KT, W, 3, false> {
  typedef RowPipe<Deep<KT, H, W>, DLay, KT, W, 3, false> Base;
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
  static constexpr int LDW = Base::LDW, LDH = 16 * W + 4;
  static constexpr int NB = dp_blocks(KT, H, W), B_OUT = NB - 2, B_BIAS = NB - 1;
  static constexpr bool LOAD_AHEAD = false;  // (see Small)
  // us a call of 500 models without and with: 569 x 40, 120-60-60, 17 rows a step 7265 and 5960; 100-70, 24 rows 3284 and 3155; 569 x 30,
  // 128-100-60 5880 and 5229; but 569 x 50, 60-60-60, 17 rows 3845 and 4572.
  // (These kernels are larger than an instruction cache, and where one lies counts for as much: the same code of <3,3,4> and
  // <2,3,8> took 1.00 to 1.14 and 1.01 to 1.17 of its time at twelve places that other kernels' sizes gave it.)
  static constexpr bool RARE_APART = !(H == 3 && W == 4 && KT >= 3);
  static constexpr bool NEAR = dp_near(KT, H, W), STREAM = dp_stream(H, W);
  static constexpr int NM = NEAR ? NB : 1;
  static constexpr int O_LEV = Base::O_OWN, O_WO = O_LEV + H * SM_RC * LDH, O_D3 = O_WO + W * 256, O_TOP = O_D3 + SM_RC * MD_RS;
  static_assert(O_TOP * 4 == dp_fixed_lds(KT, H, W), "LDS layout");
  typedef __attribute__((address_space(1))) f32x4 GlobalF32x4;

  int T[H + 1] = {}, c = 0, per_wave = 0, region = 0;  // T: tiles of the hidden levels 1..H
  __device__ __forceinline__ void pin_own() {
#pragma unroll
    for (int l = 1; l <= H; l++) T[l] = pin(y.T[l]);
    c = pin(y.U[H + 1]);
    per_wave = pin(y.per_wave);
    region = pin(y.region);
  }
  __device__ __forceinline__ double total(double v) const { return block_sum(v, red); }

  // Blocks: 0..KT-1 the input layer (lane: unit li of the wave's tile, inputs 16 kk + 4q + e), then W for each further
  // hidden layer (inputs: units of the level below), the output layer (lane: output li, units 4q + e of the wave's
  // tile), the biases (e < H: hidden layer e, unit li; e == H: output li; alike in the four q).
  struct State {
    f32x4 w[STREAM ? KT + 2 : NB], g[NB], m[NM], v[NM];
  };
  __device__ __forceinline__ static constexpr bool hidden(int n) { return n >= KT && n < B_OUT; }
  // the register block of the weights of block n, which is not streamed
  __device__ __forceinline__ static constexpr int reg(int n) { return STREAM && n >= KT ? n - B_OUT + KT : n; }
  __device__ __forceinline__ static constexpr int layer(int n) { return n < KT ? 0 : (n >= B_OUT ? H : 1 + (n - KT) / W); }
  struct Acts {
    uint32_t bits[H];  // ReLU patterns of the wave's units: bit 4 r + e of row 16 r + 4q + e
  };
  __device__ __forceinline__ static constexpr int blk(int l, int kk) { return l == 0 ? kk : KT + (l - 1) * W + kk; }
  __device__ __forceinline__ float* lev(int l) const { return f(O_LEV + (l - 1) * (SM_RC * LDH)); }
  // What the addresses in the slot depend on, as values of each phase's own: kept for the whole run, the addresses of all
  // blocks would crowd the scalar registers out into vector registers.
  struct Places {
    int own, biases, region, turned, t1, t2, t3;
  };
  __device__ __forceinline__ Places places() const {
    return Places{pin(wave() * per_wave * 64), pin(region - (W - wave()) * 64), pin(region), pin(region * (NEAR ? 1 : 3)),
                  pin(T[1]), pin(T[2]), pin(T[H])};
  }
  // block n in a set of the slot, in 16-byte vectors
  __device__ __forceinline__ static int place(const Places& z, int n) {
    int at = z.biases;
    if (n < B_BIAS) {
      const int l = n < KT ? 0 : 1 + (n - KT) / W;
      at = n < KT ? n : (n - KT) % W + KT + (l == 2 ? z.t1 : 0);
      if (n == B_OUT) at = KT + z.t1 + (H == 3 ? z.t2 : 0);
      at = z.own + at * 64;
    }
    return at;
  }
  // block n: set 0 the parameters, 1 and 2 the moments
  __device__ __forceinline__ GlobalF32x4* kept(const Places& z, int set, int n) const {
    return (GlobalF32x4*)slot + set * z.region + place(z, n) + (tid() & 63);
  }
  // Weights of layer l (1..H-1) from in tile i to out tile o, 256 floats: element e of lane n of the wave that owns them at
  // 64 e + n, which is a row of 16 out units for each in unit, the rows in the order 0 4 8 12 1 5 ..
  __device__ __forceinline__ static int turned(const Places& z, int l, int i, int o) {  // in 16-byte vectors
    return z.turned + ((l == 2 ? z.t1 * z.t2 : 0) + i * (l == 1 ? z.t2 : z.t3) + o) * 64;
  }
  __device__ __forceinline__ GlobalF32* wt(const Places& z, int l, int i, int o) const {
    return (GlobalF32*)((GlobalF32x4*)slot + turned(z, l, i, o)) + (tid() & 63);
  }
  // transposed: units 4q.. of the out tile for unit li of the in tile
  __device__ __forceinline__ f32x4 across(const Places& z, int l, int i, int o) const {
    const int li = tid() & 15, q = (tid() & 63) >> 4;
    return ((GlobalF32x4*)slot + turned(z, l, i, o))[((li & 3) * 4 + (li >> 2)) * 4 + q];
  }
  __device__ __forceinline__ f32x4 along(const Places& z, int l, int i, int o) const {
    const GlobalF32* p = wt(z, l, i, o);
    return f32x4{p[0], p[64], p[128], p[192]};
  }
  __device__ __forceinline__ void put(const Places& z, int l, int i, int o, const f32x4& x) const {
    GlobalF32* p = wt(z, l, i, o);
#pragma unroll
    for (int e = 0; e < 4; e++) p[e * 64] = x[e];
  }
  // the weights of block n, wherever they are
  __device__ __forceinline__ f32x4 weights(const State& R, const Places& z, int n) const {
    if constexpr (STREAM)
      if (hidden(n)) return used(n) ? along(z, layer(n), (n - KT) % W, wave()) : f32x4{0.f, 0.f, 0.f, 0.f};
    return R.w[reg(hidden(n) && STREAM ? 0 : n)];
  }
  __device__ __forceinline__ bool used(int n) const {  // block n holds parameters of this wave
    const int w_ = wave();
    if (n < KT) return w_ < T[1];
    if (n < B_OUT) {
      const int l = 1 + (n - KT) / W, kk = (n - KT) % W;
      return w_ < T[l + 1] && kk < T[l];
    }
    return n == B_BIAS || w_ < T[H];
  }
  // Where element e of the lane's block n stands in the packed parameters; -1: a pad.
  __device__ __forceinline__ int packed(int n, int e, int& l, int& i, bool& isb) const {
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4, j = wave() * 16 + li;
    isb = n == B_BIAS;
    if (isb) {
      l = e;
      i = e < H ? j : li;
      return e <= H && i < y.U[min(l, H) + 1] ? y.cb[min(l, H)] + i : -1;
    }
    int k, o;
    if (n == B_OUT) {
      l = H;
      k = wave() * 16 + 4 * q + e;
      o = li;
    } else {
      l = n < KT ? 0 : 1 + (n - KT) / W;
      k = (n < KT ? n : (n - KT) % W) * 16 + 4 * q + e;
      o = j;
    }
    i = k * y.U[l + 1] + o;
    return k < y.U[l] && o < y.U[l + 1] ? y.cw[l] + i : -1;
  }

  // ---- parameters ----------------------------------------------------------
  // packed parameters (or moments), or the initial draw, -> the blocks of a set
  __device__ __forceinline__ void unpack(const float* st, int set, float unit = 1.f) const {
    const Places z = places();
#pragma unroll 1
    for (int n = 0; n < NB; n++) {
      const int w_ = wave();
      if (n < B_BIAS) {
        const int l = n < KT ? 0 : (n == B_OUT ? H : 1 + (n - KT) / W);
        if (w_ >= y.T[l == H ? H : l + 1] || (l > 0 && l < H && (n - KT) % W >= y.T[l])) continue;
      }
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        int l, i;
        bool isb;
        const int ci = packed(n, e, l, i, isb);
        x[e] = ci < 0 ? 0.f : (st ? st[ci] * unit : init_value(l, i, isb));
      }
      *kept(z, set, n) = x;
    }
  }
  template <class To>
  __device__ __forceinline__ void take(int set, To& to) const {
    const Places z = places();
#pragma unroll
    for (int n = 0; n < NB; n++) {
      if (STREAM && hidden(n)) {
        if (used(n)) put(z, layer(n), (n - KT) % W, wave(), (f32x4)*kept(z, set, n));
        continue;
      }
      to[reg(n)] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (used(n)) to[reg(n)] = *kept(z, set, n);
    }
  }
  __device__ __forceinline__ void load(State& R, const float* st, float um, float uv) const {
    const Places z = places();
#pragma unroll
    for (int which = 0; which < 2; which++) {
      if (st) {
        unpack(st + (1 + which) * y.p.P, NEAR ? 0 : 1 + which, which ? uv : um);
        if constexpr (NEAR) take(0, which ? R.v : R.m);
      } else {
#pragma unroll
        for (int n = 0; n < NB; n++) {
          if constexpr (NEAR)
            (which ? R.v[n] : R.m[n]) = f32x4{0.f, 0.f, 0.f, 0.f};
          else if (used(n))
            *kept(z, 1 + which, n) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
    unpack(st, 0);
    restore_best(R);
  }
  __device__ __forceinline__ void keep_best(State& R) const {
    const Places z = places();
#pragma unroll
    for (int n = 0; n < NB; n++)
      if (used(n)) *kept(z, 0, n) = weights(R, z, n);
  }
  __device__ __forceinline__ void restore_best(State& R) const {
    take(0, R.w);
    __builtin_amdgcn_s_waitcnt(0);  // see k_train_small
    publish(R);
  }
  __device__ __forceinline__ static void zero_grad(State& R) {
#pragma unroll
    for (int n = 0; n < NB; n++) R.g[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // The wave's output blocks into LDS and its hidden blocks into global memory: row by row of 16 units, so
  // that no turning is needed on the way (through an LDS patch each block waited for the one before: [60, 60, 60] on 50 inputs
  // 2.07 -> 1.95 ms, [128, 100] 1.29 -> 1.33 at batch 160).
  __device__ __forceinline__ void publish(const State& R) const {
    const int w_ = wave();
    const Places z = places();
#pragma unroll
    for (int l = 1; l < H; l++)
      if (w_ < T[l + 1]) {
#pragma unroll
        for (int kk = 0; kk < W; kk++)
          if (kk < T[l]) put(z, l, kk, w_, weights(R, z, blk(l, kk)));
      }
    publish_outputs(R);
  }
  __device__ __forceinline__ void publish_outputs(const State& R) const {
    *((f32x4*)(f(O_WO) + wave() * 256) + (tid() & 63)) = R.w[reg(B_OUT)];
  }

  // ---- products over the rows R0..R0+N-1 (16 rows each) ------------------------
  // Operand tiles requested before the products of the tile at hand (past the last: read, not used).  Up to two row tiles the
  // products of a tile are too short to hide the next one's reads: [60, 60, 60] at batch 24 796 -> 764 us, [128, 128,
  // 128] 1913 -> 1851.  Four row tiles need no look-ahead, and 14 blocks of weights and gradients leave no room for it
  // (48 vector registers spilled: [128, 100] on 50 inputs 2.60 -> 3.35 ms).
  __device__ __forceinline__ static constexpr int ahead(int n) { return n <= 2 && (STREAM || NB <= 13) ? 1 : 0; }
  // acc[r] += rows of s . b, over nk k tiles
  template <int R0, int N, int K>
  __device__ __forceinline__ static void rows_times(const float* s, int ld, const f32x4* b, int nk, f32x4* acc) {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    const float* a_ = s + (R0 * 16 + li) * ld + 4 * q;
    constexpr int AHEAD = ahead(N);
    f32x4 a[2][N];
    if (AHEAD) {
#pragma unroll
      for (int r = 0; r < N; r++) a[0][r] = *(const f32x4*)(a_ + r * 16 * ld);
    }
#pragma unroll
    for (int kk = 0; kk < K; kk++)
      if (kk < nk) {
        if (kk + AHEAD < K) {
#pragma unroll
          for (int r = 0; r < N; r++) a[(kk + AHEAD) & 1][r] = *(const f32x4*)(a_ + r * 16 * ld + (kk + AHEAD) * 16);
          if (AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
          for (int r = 0; r < N; r++)
            acc[R0 + r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk & 1][r][e], b[kk][e], acc[R0 + r], 0, 0, 0);
      }
  }
  // g[kk] += columns of s^T . d
  template <int R0, int N, int K>
  __device__ __forceinline__ static void gradient(const float* s, int ld, const f32x4* d, int nk, f32x4* g) {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    const float* a_ = s + (R0 * 16 + 4 * q) * ld + li;
    constexpr int AHEAD = ahead(N);
    float a[2][N][4];
    auto read = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < N; r++)
#pragma unroll
        for (int e = 0; e < 4; e++) a[kk & 1][r][e] = a_[(r * 16 + e) * ld + kk * 16];
    };
    if (AHEAD) read(0);
#pragma unroll
    for (int kk = 0; kk < K; kk++)
      if (kk < nk) {
        if (kk + AHEAD < K) {
          read(kk + AHEAD);
          if (AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < N; r++)
#pragma unroll
          for (int e = 0; e < 4; e++)
            g[kk] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk & 1][r][e], d[R0 + r][e], g[kk], 0, 0, 0);
      }
  }
  // fn(first row tile, number of them), compile-time, for the row tiles of a chunk
  template <class F>
  __device__ __forceinline__ static void each_rows(int nrt, F fn) {
    if (nrt == 4) {
      fn(std::integral_constant<int, 0>(), std::integral_constant<int, 4>());
    } else {
      if (nrt >= 2)
        fn(std::integral_constant<int, 0>(), std::integral_constant<int, 2>());
      else
        fn(std::integral_constant<int, 0>(), std::integral_constant<int, 1>());
      if (nrt == 3) fn(std::integral_constant<int, 2>(), std::integral_constant<int, 1>());
    }
  }

  // ---- forward ---------------------------------------------------------------
  __device__ __forceinline__ void forward(const State& R, int, int, int nrt, Acts& A) const {
    const int w_ = wave();
    const Places z = places();
    f32x4 ws[STREAM ? W : 1];  // a hidden layer's blocks, requested while the level below is computed
    auto request = [&](int l) __attribute__((always_inline)) {
      if constexpr (STREAM)
        if (w_ < T[l + 1]) {
#pragma unroll
          for (int kk = 0; kk < W; kk++)
            if (kk < T[l]) ws[STREAM ? kk : 0] = along(z, l, kk, w_);
        }
    };
    request(1);
    __syncthreads();  // the chunk's inputs
#pragma unroll
    for (int l = 0; l < H; l++) {
      A.bits[l] = 0;
      if (w_ < T[l + 1]) {
        const float bias = R.w[reg(B_BIAS)][l];
        const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
        float* o = lev(l + 1) + 4 * q * LDH + w_ * 16 + li;
        uint32_t bits = 0;
        each_rows(nrt, [&](auto r0, auto cnt) __attribute__((always_inline)) {
          constexpr int R0 = decltype(r0)::value, N = decltype(cnt)::value;
          f32x4 acc[4];
#pragma unroll
          for (int r = 0; r < N; r++) acc[R0 + r] = f32x4{bias, bias, bias, bias};
          if (l == 0)
            rows_times<R0, N, KT>(xs(0), LDW, &R.w[0], KT, acc);
          else
            rows_times<R0, N, W>(lev(l ? l : 1), LDH, STREAM ? ws : &R.w[STREAM ? 0 : blk(l ? l : 1, 0)], T[l], acc);
#pragma unroll
          for (int r = R0; r < R0 + N; r++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
              const float x = relu(acc[r][e]);
              o[(r * 16 + e) * LDH] = x;
              bits |= (x > 0.f ? 1u : 0u) << (4 * r + e);
            }
        });
        A.bits[l] = bits;
      }
      if (l + 1 < H) {
        if (l > 0) request(l + 1);
        __syncthreads();
      }
    }
  }

  // ---- outputs: wave r takes row tile r; lane (output li, rows 4q + e) -----------
  __device__ __forceinline__ void outputs(State& R, int, int, int rows, bool train, bool loss, float inv_mb, double& lsum, double& hits) const {
    const int lane = tid() & 63, r = wave(), li = lane & 15, q = lane >> 4;
    if (r * 16 >= rows) return;
    const float* a_ = lev(H) + (r * 16 + li) * LDH + 4 * q;
    const f32x4* b_ = (const f32x4*)f(O_WO) + lane;
    f32x4 z0 = f32x4{0.f, 0.f, 0.f, 0.f}, z1 = z0;
    // operands a tile ahead: few waves are at work here, so nothing else hides the reads
    f32x4 as[2] = {*(const f32x4*)a_, f32x4{0.f, 0.f, 0.f, 0.f}}, bs[2] = {b_[0], f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kk = 0; kk < W; kk++)
      if (kk < T[H]) {
        if (kk + 1 < W) {
          as[(kk + 1) & 1] = *(const f32x4*)(a_ + (kk + 1) * 16);
          bs[(kk + 1) & 1] = b_[(kk + 1) * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
        const f32x4 a = as[kk & 1], b = bs[kk & 1];
        z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], z0, 0, 0, 0);
        z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], z1, 0, 0, 0);
        z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], z0, 0, 0, 0);
        z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], z1, 0, 0, 0);
      }
    const f32x4 yv4 = *(const f32x4*)(ys(0) + r * 16 + 4 * q);
    float* d3 = f(O_D3) + (r * 16 + 4 * q) * MD_RS + li;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float z = z0[e] + z1[e] + R.w[reg(B_BIAS)][H], yv = yv4[e];
      const bool valid = r * 16 + 4 * q + e < rows;
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
      if (train) d3[e * MD_RS] = dl;
    }
  }

  // ---- backward ----------------------------------------------------------------
  __device__ __forceinline__ void backward(State& R, int, int nrt, const Acts& A) const {
    const int w_ = wave();
    f32x4 d[4];  // the wave's deltas of the level being worked on
    const Places z = places();
    f32x4 tr[4];  // four transposed blocks at a time
    auto fetch_tr = [&](int l, int o0) __attribute__((always_inline)) {
      if (w_ < T[l]) {
#pragma unroll
        for (int o = 0; o < 4; o++)
          if (o0 + o < T[l + 1]) tr[o] = across(z, l, w_, o0 + o);
      }
    };
    fetch_tr(H - 1, 0);
    {
      const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
      const float* d3 = f(O_D3);
      const bool own = w_ < T[H];
      const float* p = f(O_WO) + w_ * 256 + ((li >> 2) * 16 + 4 * q) * 4 + (li & 3);
      float wo[4];  // unit li, outputs 4q..4q+3
#pragma unroll
      for (int e = 0; e < 4; e++) wo[e] = p[e * 4];
      float* o = lev(H) + 4 * q * LDH + w_ * 16 + li;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        if (r >= nrt) break;
        float db[4];  // row 4q + e, output li
#pragma unroll
        for (int e = 0; e < 4; e++) {
          db[e] = d3[(r * 16 + 4 * q + e) * MD_RS + li];
          R.g[B_BIAS][H] += db[e];
        }
        if (own) {
          const f32x4 da = *(const f32x4*)(d3 + (r * 16 + li) * MD_RS + 4 * q);  // row li, outputs 4q..4q+3
          f32x4 a, x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 4; e++) a[e] = o[(r * 16 + e) * LDH];
#pragma unroll
          for (int e = 0; e < 4; e++) {
            x = __builtin_amdgcn_mfma_f32_16x16x4f32(da[e], wo[e], x, 0, 0, 0);
            R.g[B_OUT] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], db[e], R.g[B_OUT], 0, 0, 0);
          }
#pragma unroll
          for (int e = 0; e < 4; e++) {
            x[e] = a[e] > 0.f ? x[e] : 0.f;
            R.g[B_BIAS][H - 1] += x[e];
            o[(r * 16 + e) * LDH] = x[e];
          }
          d[r] = x;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int l = H - 1; l >= 1; l--) {  // from level l+1 to level l, through layer l
      f32x4 dn[4];
#pragma unroll
      for (int r = 0; r < 4; r++) dn[r] = f32x4{0.f, 0.f, 0.f, 0.f};
      auto times_tr = [&](int o0) __attribute__((always_inline)) {
        if (w_ < T[l] && o0 < T[l + 1])
          each_rows(nrt, [&](auto r0, auto cnt) __attribute__((always_inline)) {
            rows_times<decltype(r0)::value, decltype(cnt)::value, 4>(lev(l + 1) + o0 * 16, LDH, tr, T[l + 1] - o0, dn);
          });
      };
      times_tr(0);
      // in flight during the weight gradient: the second half if there is one, else the level below's first
      if (W > 4 && T[l + 1] > 4)
        fetch_tr(l, 4);
      else if (l > 1)
        fetch_tr(l - 1, 0);
      if (w_ < T[l + 1])
        each_rows(nrt, [&](auto r0, auto cnt) __attribute__((always_inline)) {
          gradient<decltype(r0)::value, decltype(cnt)::value, W>(lev(l), LDH, d, T[l], &R.g[blk(l, 0)]);
        });
      if (W > 4 && T[l + 1] > 4) {
        times_tr(4);
        if (l > 1) fetch_tr(l - 1, 0);
      }
      if (w_ < T[l]) {
#pragma unroll
        for (int r = 0; r < 4; r++)
#pragma unroll
          for (int e = 0; e < 4; e++) {
            dn[r][e] = (A.bits[l - 1] >> (4 * r + e)) & 1u ? dn[r][e] : 0.f;
            R.g[B_BIAS][l - 1] += dn[r][e];
          }
      }
      if (l > 1) {
        __syncthreads();  // nobody reads this level's activations any more
        if (w_ < T[l]) {
          const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
          float* o = lev(l) + 4 * q * LDH + w_ * 16 + li;
#pragma unroll
          for (int r = 0; r < 4; r++)
            if (r < nrt) {
#pragma unroll
              for (int e = 0; e < 4; e++) o[(r * 16 + e) * LDH] = dn[r][e];
            }
        }
        __syncthreads();
      }
#pragma unroll
      for (int r = 0; r < 4; r++) d[r] = dn[r];
    }
    if (w_ < T[1])
      each_rows(nrt, [&](auto r0, auto cnt) __attribute__((always_inline)) {
        gradient<decltype(r0)::value, decltype(cnt)::value, KT>(xs(0), LDW, d, KT, &R.g[0]);
      });
  }

  // Ahead of the first store to layer 1's weights in global memory: behind the last barrier of the backward pass the waves of
  // the first level still fetch the second half of that layer's out tiles, those of waves 4 and up.  (Every other fetch of
  // another wave's weights lies ahead of that barrier.)  The condition is the fetch's own, the same in every wave.
  __device__ __forceinline__ void before_weights() const {
    if (W > 4 && T[2] > 4) __syncthreads();
  }
  // Blocks in the order of their update.  Where it stores the weights itself, layer 1's come last and the barrier in front of
  // them finds the waves past most of their work: 256 suggestions of one to three layers 7.99 ms a call as without it, 8.09
  // with the barrier ahead of all hidden blocks, 8.43 with one ahead of the whole update in place of the chunk's last.
  __device__ __forceinline__ static constexpr int turn_of(int k) {
    if (!STREAM || k < KT) return k;
    return k < NB - W ? k + W : k - (NB - W) + KT;
  }

  // ---- optimizer step (pads: see k_train_small) ----------------------------------
  template <bool ADAM>
  __device__ __forceinline__ void update(State& R, const OptC& oc) const {
    OptC o = oc;
    o.adam = ADAM;
    // Pads need no mask (see k_train_small).  In two cuts the least eps clears them all the same: no value
    // changes, but the branch parts the blocks for the register allocation.  Three layers on four waves: 500 models of 569 x 50,
    // 60-60-60, 24 rows a step, 3 epochs 1957 us a call without it, 1755 with it; elsewhere it costs (128-40-100 3252 and 3491,
    // 128-128-128 5245 and 6026).  Two layers on eight waves and three input tiles spill 28 registers without it and 8 with it: 500
    // models of 569 x 40, 128-100, 5 epochs, 24, 64 and 128 rows a step 3946 and 3765, 2314 and 2146, 1953 and 1925, 100-70
    // 3231 and 3269; with one, two and four tiles it costs 1 to 4 %.
    const bool pads = ADAM && ((H == 3 && W == 4) || (H == 2 && W == 8 && KT == 3)) && least_eps(o);
    const Places z = places();
    // Moments in the slot are fetched AHEAD blocks early.  A block that the wave does not have is sent out of the
    // descriptor's range (zeros come back, nothing is written) instead of branched around: with the same memory operations
    // on every path the waits are for the block that is needed, not for all that is in flight.
    f32x4 mf[NEAR ? 1 : NB], vf[NEAR ? 1 : NB], wf[STREAM ? NB : 1];
    const __amdgpu_buffer_rsrc_t mem = __builtin_amdgcn_make_buffer_rsrc(slot, 0, y.slot_floats * 4u, 0x00020000);
    const uint32_t lane16 = (tid() & 63) * 16;
    auto where = [&](int n) __attribute__((always_inline)) { return used(n) ? lane16 : 0x80000000u; };
    auto fetch = [&](int n) __attribute__((always_inline)) {
      if constexpr (!NEAR)
        if (n < NB) {
          const uint32_t vo = where(n);
          const int at = place(z, n) * 16;
          mf[n] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(mem, vo, at + z.region * 16, 0));
          if (ADAM) vf[n] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(mem, vo, at + z.region * 32, 0));
          if (STREAM && hidden(n)) {
            const int block = turned(z, layer(n), (n - KT) % W, wave()) * 16;
            const uint32_t from = used(n) ? lane16 / 4 : 0x80000000u;
#pragma unroll
            for (int e = 0; e < 4; e++)
              wf[STREAM ? n : 0][e] =
                  __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mem, from + e * 256, block, 0));
          }
        }
    };
    // The whole offset in the vector register: with a scalar register in the instruction the compiler leaves no wait state
    // between a 16-byte store and an instruction that overwrites its data, and the last lanes then stored what came next.
    auto store = [&](const f32x4& x, uint32_t at) __attribute__((always_inline)) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), mem, at, 0, 0);
    };
    // blocks of moments in flight (256 suggestions of one to three layers: 7.98 ms a call, with three 8.01, with six 8.02)
    constexpr int AHEAD = 4;
#pragma unroll
    for (int k = 0; k < AHEAD; k++) fetch(turn_of(k));
#pragma unroll
    for (int e = 0; e <= H; e++) R.g[B_BIAS][e] = sm_rowsum(R.g[B_BIAS][e]);
#pragma unroll
    for (int k = 0; k < NB; k++) {
      const int n = turn_of(k);
      if (STREAM && k == NB - W) before_weights();
      if (k + AHEAD < NB) fetch(turn_of(k + AHEAD));
      f32x4& mm = NEAR ? R.m[NEAR ? n : 0] : mf[NEAR ? 0 : n];
      f32x4& vv = NEAR ? R.v[NEAR ? n : 0] : vf[NEAR ? 0 : n];
      f32x4& ww = STREAM && hidden(n) ? wf[STREAM ? n : 0] : R.w[reg(STREAM && hidden(n) ? 0 : n)];
      if (used(n)) {
        const float am = n == B_BIAS ? 0.f : o.am;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          if (n == B_BIAS && e > H) continue;
          float wr = ww[e], mr = mm[e], vr = vv[e];
          opt_step(o, n == B_BIAS ? R.g[n][e] : R.g[n][e] + am * wr, wr, mr, vr);
          ww[e] = wr;
          mm[e] = mr;
          vv[e] = vr;
        }
        if (pads) {
#pragma unroll
          for (int e = 0; e < 4; e++) {
            int l, i;
            bool isb;
            if (packed(n, e, l, i, isb) < 0) ww[e] = mm[e] = vv[e] = 0.f;
          }
        }
      }
      if constexpr (!NEAR) {
        const uint32_t vo = where(n);
        const int at = place(z, n) * 16;
        store(mm, vo + (uint32_t)(at + z.region * 16));
        if (ADAM) store(vv, vo + (uint32_t)(at + z.region * 32));
        if constexpr (STREAM)
          if (hidden(n)) {
            const int block = turned(z, layer(n), (n - KT) % W, wave()) * 16;
            const uint32_t to = used(n) ? lane16 / 4 : 0x80000000u;
#pragma unroll
            for (int e = 0; e < 4; e++)
              __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)ww[e]), mem, to + e * 256, block, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (STREAM) {
      publish_outputs(R);
    } else {
      before_weights();
      publish(R);
    }
    asm volatile("" ::: "memory");  // (what comes next reads through pointers what was written through the descriptor)
  }
  template <bool GRAD>
  __device__ __forceinline__ void record(const State& R, float am, float* out) const {
    const bool first = (threadIdx.x & 63) < 16;
    const Places z = places();
#pragma unroll
    for (int n = 0; n < NB; n++) {
      const f32x4 ww = weights(R, z, n);
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if (n == B_BIAS && e > H) continue;
        int l, i;
        bool isb;
        const int ci = packed(n, e, l, i, isb);
        float x = ww[e];
        if (GRAD) x = n == B_BIAS ? sm_rowsum(R.g[n][e]) : R.g[n][e] + am * x;
        if (ci >= 0 && (n != B_BIAS || (first && (e < H || wave() == 0)))) out[ci] = x;
      }
    }
  }
  __device__ __forceinline__ double penalty_sum(const State& R) const {
    double s = 0.0;
#pragma unroll
    for (int n = 0; n < B_BIAS; n++) {
      const f32x4 ww = weights(R, places(), n);
#pragma unroll
      for (int e = 0; e < 4; e++) s += (double)ww[e] * (double)ww[e];
    }
    return block_sum(s, red);
  }
};

template <int KT, int H, int W>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * W, 64 * W), amdgpu_waves_per_eu(2, 2)))
void k_train_deep(const TrainParams P) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_item;
  __shared__ double red[W], trace_stash[2];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    if (item >= P.n_items) break;
    const __attribute__((address_space(4))) DItem* di = (const __attribute__((address_space(4))) DItem*)P.items + item / P.n_folds;
    Deep<KT, H, W> T(P, di->d, di->y, smem, (float*)(P.slots + (uint64_t)blockIdx.x * P.slot_bytes), red, trace_stash,
                     item % P.n_folds);
    T.run();
  }
}

}  // namespace
