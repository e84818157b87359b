// Training / scoring kernel for small fp32 models with one hidden layer that take all their rows in every step (full-batch
// training of a tiny data set): up to 31 inputs, 64 units, 4 outputs, data set in LDS.
//
// An epoch is one step over the same rows, so nothing is fetched or permuted while it runs: a workgroup gathers the rows of
// its model into LDS once (those it is fitted on, those set aside for early stopping and the held fold's, each part
// padded to whole tiles of 16 rows) and its W waves (four up to 80 rows, eight beyond) share the row tiles of a step.  Where train_small_f32.h gives the
// waves units, and walks the rows chunk by chunk, every wave here computes all of the model for its rows:
//
//   forward   D[row][unit] = xs[row][k] . w1[unit][k] on MFMA (16x16x4 fp32); the bias is column d of the inputs, a 1.
//             ReLU; the outputs are sums over the 16 unit lanes, alike in the four quads: no exchange between waves.
//   outputs   lane (row 4q + li % 4): softmax / logistic / squared loss, output delta (two classes: one column)
//   backward  hidden deltas in the accumulators, products xs^T . delta in registers over the wave's row tiles
//   reduce    the waves' gradients meet in LDS, a slot of 64 values per register; slot r belongs to wave r mod W
//   update    Adam / SGD of the wave's slots, a parameter a lane, moments in registers; the weights go back to LDS
//
// Two barriers a step.  What bounds it: the chain of a step, about 5500 cycles at 120 rows and 20 units, of which the
// products are a sixth (a matrix instruction takes 32 cycles and no vector instruction of the SIMD runs beside it).  5
// models of 20 units on 150 x 4, three classes, 20 epochs: 160 us a call on the chunks of 64 rows of train_small_f32.h, 64
// here.  That kernel keeps the larger models: there a step is more than its chain.
#pragma once
#include "common.h"
#include "train_small_f32.h"  // folding sums, outputs

namespace {

struct FLay {
  int32_t d, h, P;
  int32_t cw[2], cb[2];
};
struct FItem {
  ItemDesc d;
  FLay y;
};

// parameters per lane: input layer with its bias, output layer and bias (four of those share a register)
__host__ __device__ constexpr int fu_slots(int kt, int nt, int co) { return nt * kt * 4 + (nt * co + co + 3) / 4; }
__host__ __device__ constexpr uint32_t fu_lds(int kt, int nt, int co, int waves, int64_t n) {
  return (uint32_t)(fu_slots(kt, nt, co) * (1 + waves) * 64 + (n + 48) * (sm_ldw(kt) + 1)) * 4;
}
// Waves per SIMD the registers of a variant are budgeted for.  27 of the 44 variants do not fit altogether: by the compiler's
// report <2,2,3..4,4> spill 54 and 66 vector registers, <1,3,3..4,4> 53 and 52, <2,2,3..4,8> 20 and 34, <1,3,3..4,8> 18 and 30,
// <1,4,1..2,8> 21 and 19, the others 19 at most.
__host__ __device__ constexpr int fu_occupancy(int kt, int nt, int co) { return nt == 4 && co > 2 ? 2 : 4; }
// By shape, rows and batch size alone; waves == 0: not a case of this kernel.  Four unit tiles are the edge: us a call here over
// train_small_f32.h as it was before this kernel, 14 inputs, 64 units, 15 epochs, 4, 200 and 1000 suggestions: two classes,
// 100 rows 0.63, 0.84, 0.94; three classes, 256 rows 0.50, 0.84, 1.00, and 600 rows 0.43, 0.73, 0.82; four classes (4 inputs), 256
// rows 0.54, 0.93, 1.11, and 300 rows 0.53, 0.87, 1.03.
__host__ inline SmallCut full_cut(const int32_t* dims, int L, int64_t n, int32_t batch_size) {
  SmallCut m = {0, 0, 0, 0};
  if (L != 2 || dims[0] > 31 || dims[1] > 64 || dims[2] > 4 || n < 1 || (batch_size > 0 && batch_size < n)) return m;
  m.kt = rup(dims[0] + 1, 16) / 16;
  m.nt = rup(dims[1], 16) / 16;
  m.co = dims[2];
  m.waves = n <= 80 ? 4 : 8;
  if (m.nt == 4 && n < (m.co > 2 ? 256 : 100)) return SmallCut{0, 0, 0, 0};
  if (m.kt * m.nt > 4 || n > 4096 || fu_lds(m.kt, m.nt, m.co, m.waves, n) > SM_LDS_LIMIT) m.waves = 0;
  return m;
}
// workgroups a CU holds
__host__ inline int full_per_cu(const SmallCut& m, uint32_t lds_bytes) {
  const int by_regs = 4 * fu_occupancy(m.kt, m.nt, m.co) / m.waves, by_lds = (int)(160u * 1024u / (lds_bytes + 512));
  const int n = by_regs < by_lds ? by_regs : by_lds;
  return n < 1 ? 1 : n;
}
__host__ inline void make_flay(FLay& y, const int32_t* dims) {
  y.d = dims[0];
  y.h = dims[1];
  y.cw[0] = 0;
  y.cb[0] = y.d * y.h;
  y.cw[1] = y.cb[0] + y.h;
  y.cb[1] = y.cw[1] + y.h * dims[2];
  y.P = y.cb[1] + dims[2];
}
// the slot in the workspace: the best epoch's parameters
__host__ inline uint64_t fu_slot_bytes(const SmallCut& m) {
  return (uint64_t)rup(fu_slots(m.kt, m.nt, m.co), m.waves) * 256;
}

template <int KT, int NT, int CO, int W>
struct Full {
  static constexpr int NTHR = 64 * W, K0 = 16 * KT, LDW = sm_ldw(KT), ZO = sm_columns(CO);
  static constexpr int NSMALL = NT * CO + CO, NG = (NSMALL + 3) / 4, NH = NT * KT * 4, NS = NH + NG, RS = (NS + W - 1) / W;
  static_assert(NS == fu_slots(KT, NT, CO), "slots");
  typedef const __attribute__((address_space(4))) FLay ConstLay;
  // LDS, in floats: weights as the products read them, the waves' gradients, inputs, labels
  static constexpr int O_W = 0, O_PART = NS * 64, O_X = O_PART + NS * W * 64;
  const TrainParams& P;
  const ConstItemDesc& it;
  ConstLay& y;
  float* lds;
  float* slot;
  double* red;
  int fl;  // which row list
  int d, n_classes, rows_cap;

  struct Weights {
    f32x4 w[NT][KT];
    float w2[NT][ZO], ow[ZO];
  };
  struct Grads {
    f32x4 g[NT][KT];
    float g2[NT][ZO], og[ZO];
  };
  __device__ __forceinline__ float* ys() const { return lds + O_X + rows_cap * LDW; }
  __device__ __forceinline__ static int wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

  // ---- parameters: slot r of a wave holds a parameter a lane ----------------------
  // Where the lane's parameter of slot r stands in the packed parameters; -1: a pad.
  __device__ __forceinline__ int packed(int r) const {
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
    if (r < NH) {
      const int i = (r >> 2) / KT, k = (r >> 2) % KT * 16 + 4 * q + (r & 3), j = i * 16 + li;
      return j >= y.h || k > d ? -1 : (k < d ? y.cw[0] + k * y.h + j : y.cb[0] + j);
    }
    const int k = 4 * (r - NH) + q, j = k / CO * 16 + li, cc = k % CO;
    if (k >= NSMALL) return -1;
    return k >= NT * CO ? y.cb[1] + cc : (j < y.h ? y.cw[1] + j * CO + cc : -1);
  }
  __device__ __forceinline__ bool penalised(int ci) const { return (ci >= 0 && ci < y.cb[0]) || (ci >= y.cw[1] && ci < y.cb[1]); }
  __device__ __forceinline__ float draw(int ci) const {
    const int l = ci >= y.cw[1] ? 1 : 0;
    const bool isb = ci >= y.cb[l];
    const int e = ci - (isb ? y.cb[l] : y.cw[l]);
    const uint64_t kt = key_fold(key_model(it.seed, fl + P.fold_base), 16 + 2 * l + (isb ? 1 : 0));
    const uint32_t k24 = (uint32_t)(key_fold(kt, (uint64_t)e) >> 40);
    return it.bound[l] * ((float)((int32_t)k24 - 8388608) * 0x1p-23f);
  }
  __device__ __forceinline__ void publish(const float (&p)[RS]) const {
    const int lane = threadIdx.x & 63, w_ = wave();
#pragma unroll
    for (int s = 0; s < RS; s++) {
      const int r = s * W + w_;
      if (r < NH)
        lds[O_W + (r >> 2) * 256 + lane * 4 + (r & 3)] = p[s];
      else if (r < NS)
        lds[O_W + r * 64 + lane] = p[s];
    }
  }
  __device__ __forceinline__ void weights(Weights& R) const {
    const int lane = threadIdx.x & 63, li = lane & 15;
    const float* s = lds + O_W + NH * 64 + li;
#pragma unroll
    for (int i = 0; i < NT; i++) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++) R.w[i][kk] = *(const f32x4*)(lds + O_W + (i * KT + kk) * 256 + lane * 4);
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) R.w2[i][cc] = CO == 2 ? s[(i * CO + 1) * 16] - s[i * CO * 16] : s[(i * CO + cc) * 16];
    }
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) R.ow[cc] = CO == 2 ? s[(NT * CO + 1) * 16] - s[NT * CO * 16] : s[(NT * CO + cc) * 16];
  }

  // ---- rows -> LDS ------------------------------------------------------------------
  template <class RowAt>
  __device__ __forceinline__ void gather(int base, int count, RowAt row_at) const {
    float *xs = lds + O_X, *yl = ys();
    const float *X = (const float*)P.X, *Y = (const float*)P.y;
#pragma unroll 4
    for (int i = threadIdx.x; i < rup(count, 16) * K0; i += NTHR) {
      const int r = i / K0, k = i % K0;
      float x = 0.f;
      if (r < count) {
        const int row = row_at(r);
        x = k < d ? X[(uint32_t)(row * d + k)] : (k == d ? 1.f : 0.f);
        if (k == 0) yl[base + r] = Y[row];  // (class ids as they are)
      } else if (k == 0) {
        yl[base + r] = 0.f;
      }
      xs[(base + r) * LDW + k] = x;
    }
  }

  // A value that is rounded before it is used: where a product meets a sum the compiler would be free to contract the two
  // in one variant and not in another, but a model has the same bits in all that hold it.
  __device__ __forceinline__ static float rounded(float x) {
    asm("" : "+v"(x));
    return x;
  }
  // ---- one tile of 16 rows, its first at `base + 16 t` --------------------------------
  template <bool TRAIN>
  __device__ __forceinline__ void tile(const Weights& R, Grads& G, int base, int t, int count, bool loss, float inv_mb,
                                       double& lsum, double& hits) const {
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
    const float* s = lds + O_X + (base + t * 16) * LDW;
    f32x4 a[KT], acc[NT];
    float xt[KT][4];
#pragma unroll
    for (int kk = 0; kk < KT; kk++) a[kk] = *(const f32x4*)(s + li * LDW + kk * 16 + 4 * q);
    const int row = t * 16 + 4 * q + (li & 3);
    float yv = ys()[base + row];
    if (TRAIN) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++)
#pragma unroll
        for (int e = 0; e < 4; e++) xt[kk][e] = s[(4 * q + e) * LDW + kk * 16 + li];
    }
#pragma unroll
    for (int i = 0; i < NT; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KT; kk++)
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int i = 0; i < NT; i++) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk][e], R.w[i][kk][e], acc[i], 0, 0, 0);
    asm volatile("" : "+v"(yv));  // (requested here, not where the outputs begin)
    float z[ZO], dl[ZO];
#pragma unroll
    for (int i = 0; i < NT; i++)
#pragma unroll
      for (int e = 0; e < 4; e++) acc[i][e] = relu(acc[i][e]);
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) {
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        p[e] = rounded(acc[0][e] * R.w2[0][cc]);
#pragma unroll
        for (int i = 1; i < NT; i++) p[e] = fmaf(acc[i][e], R.w2[i][cc], p[e]);
      }
      float x = sm_fold_quad(p, li & 1, li & 2);  // lane e of each quad: row 4q + e
      x += sm_dpp<0x128>(x);                      // the other quads: rotations by 8 and by 4
      z[cc] = R.ow[cc] + x + sm_dpp<0x124>(x);
    }
    double l1 = 0.0, h1 = 0.0;
    sm_outputs<CO>(z, yv, row < count, CO, n_classes, TRAIN, loss, inv_mb, dl, l1, h1);
    if (loss && li < 4) {  // (the quads are alike)
      lsum += l1;
      hits += h1;
    }
    if constexpr (TRAIN) {
      float dv[ZO][4];
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) {  // of row 4q + e, from lane e of the quad
        dl[cc] = rounded(dl[cc]);
        G.og[cc] += dl[cc];
        dv[cc][0] = sm_dpp<0x00>(dl[cc]);
        dv[cc][1] = sm_dpp<0x55>(dl[cc]);
        dv[cc][2] = sm_dpp<0xAA>(dl[cc]);
        dv[cc][3] = sm_dpp<0xFF>(dl[cc]);
      }
#pragma unroll
      for (int i = 0; i < NT; i++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float av = acc[i][e];
          float sum = dv[0][e] * R.w2[i][0];
          G.g2[i][0] = fmaf(av, dv[0][e], G.g2[i][0]);
#pragma unroll
          for (int cc = 1; cc < ZO; cc++) {
            sum = fmaf(dv[cc][e], R.w2[i][cc], sum);
            G.g2[i][cc] = fmaf(av, dv[cc][e], G.g2[i][cc]);
          }
          acc[i][e] = av > 0.f ? sum : 0.f;
        }
#pragma unroll
      for (int kk = 0; kk < KT; kk++)
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
          for (int i = 0; i < NT; i++) G.g[i][kk] = __builtin_amdgcn_mfma_f32_16x16x4f32(xt[kk][e], acc[i][e], G.g[i][kk], 0, 0, 0);
    }
  }
  // the wave's gradients -> its part of every slot
  __device__ __forceinline__ void hand_over(const Grads& G) const {
    const int lane = threadIdx.x & 63;
    float* b = lds + O_PART + wave() * 64 + lane;
    float x[4 * NG];
#pragma unroll
    for (int k = 0; k < 4 * NG; k++) {
      const int i = k / CO, cc = k % CO;
      x[k] = 0.f;
      if (k >= NSMALL) continue;
      float v = i < NT ? G.g2[i < NT ? i : 0][CO == 2 ? 0 : cc] : G.og[CO == 2 ? 0 : cc];
      if (i >= NT) {  // over the four rows of the quad
        v += sm_dpp<0xB1>(v);
        v += sm_dpp<0x4E>(v);
      }
      x[k] = CO == 2 && cc == 0 ? -v : v;
    }
#pragma unroll
    for (int i = 0; i < NT; i++)
#pragma unroll
      for (int kk = 0; kk < KT; kk++)
#pragma unroll
        for (int e = 0; e < 4; e++) b[((i * KT + kk) * 4 + e) * (W * 64)] = G.g[i][kk][e];
#pragma unroll
    for (int g = 0; g < NG; g++)
      b[(NH + g) * (W * 64)] = sm_fold32(sm_fold16(x[4 * g], x[4 * g + 1]), sm_fold16(x[4 * g + 2], x[4 * g + 3]));
  }
  // loss and second score, summed per lane, of the `count` rows from `base` on
  __device__ __forceinline__ void score_rows(int base, int count, double& lsum, double& hits) const {
    Weights R;
    Grads none;
    weights(R);
    for (int t = wave(); t * 16 < count; t += W) tile<false>(R, none, base, t, count, true, 0.f, lsum, hits);
  }

  __device__ __forceinline__ void run() {
    const int n_tr = uniform(P.counts[2 * fl]), n_va = uniform(P.counts[2 * fl + 1]);
    const uint64_t km = key_model(it.seed, fl + P.fold_base);
    const RowSplit sp = row_split(km, it.patience, it.val_frac, n_tr);
    const int n_fit = uniform(sp.n_fit), n_hold = uniform(sp.n_hold), lane = threadIdx.x & 63, w_ = wave();
    const int b_hold = rup(n_fit, 16), b_va = b_hold + rup(n_hold, 16);  // where the parts begin
    const int32_t *tr = P.train_idx + (int64_t)fl * P.n, *va = P.val_idx + (int64_t)fl * P.n;
    gather(0, n_fit, [&](int p) { return tr[n_hold ? (int)perm_index(sp.ksplit, (uint32_t)n_tr, (uint32_t)p) : p]; });
    if (n_hold) gather(b_hold, n_hold, [&](int p) { return tr[held_index(sp, (uint32_t)p)]; });
    gather(b_va, n_va, [&](int p) { return va[p]; });

    const bool traced = P.trace_item == it.b * P.n_folds + fl, resume = traced && P.state_in && n_fit > 0;
    const bool watch = it.patience > 0 && n_fit > 0 && !resume;
    const bool want_loss = traced || (watch && !n_hold);
    const int epochs = n_fit > 0 ? it.epochs : 0;
    float p[RS], m[RS], v[RS];
    int ci[RS];
    uint32_t pen = 0;  // bit s: the penalty applies to the lane's parameter of the wave's slot s
#pragma unroll
    for (int s = 0; s < RS; s++) {
      const int r = s * W + w_;
      ci[s] = r < NS ? packed(r) : -1;
      p[s] = m[s] = v[s] = 0.f;
      if (ci[s] >= 0) {
        p[s] = resume ? P.state_in[ci[s]] : draw(ci[s]);
        if (resume) {
          m[s] = P.state_in[y.P + ci[s]];
          v[s] = P.state_in[2 * y.P + ci[s]];
        }
        if (penalised(ci[s])) pen |= 1u << s;
      }
    }
    publish(p);

    OptC oc;
    oc.adam = it.solver == BBO_ADAM;
    oc.nest = it.nesterov != 0;
    oc.b1 = it.beta1;
    oc.b2 = it.beta2;
    oc.omb1 = 1.f - it.beta1;
    oc.omb2 = 1.f - it.beta2;
    oc.eps = it.eps;
    oc.mu = it.momentum;
    oc.lr = it.lr;
    oc.lr_t = it.lr;
    const float mb = (float)n_fit, inv_mb = 1.f / mb;
    oc.am = it.alpha / mb;
    float lr_tab = 0.f;  // Adam: the step sizes of 64 steps, one per lane
    int lr_at = 64;      // ... the next of them
    Plateau plateau;
    bool have_best = false;
    float* best = slot + w_ * 64 + lane;
    __syncthreads();  // rows and weights
    for (int e = resume ? (int)P.step_begin : 0; e < epochs; e++) {  // an epoch is a step
      Weights R;
      Grads G;
      weights(R);
#pragma unroll
      for (int i = 0; i < NT; i++) {
#pragma unroll
        for (int kk = 0; kk < KT; kk++) G.g[i][kk] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc = 0; cc < ZO; cc++) G.g2[i][cc] = 0.f;
      }
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) G.og[cc] = 0.f;
      double lsum = 0.0, hits = 0.0;
      for (int t = w_; t * 16 < n_fit; t += W) tile<true>(R, G, 0, t, n_fit, want_loss, inv_mb, lsum, hits);
      hand_over(G);
      if (oc.adam) {
        if (lr_at == 64) {
          // beta^t of the next 64 steps, a step per lane, by repeated squaring in double
          lr_at = 0;
          double q1 = (double)it.beta1, q2 = (double)it.beta2, b1t = 1.0, b2t = 1.0;
#pragma unroll 1
          for (uint32_t t = (uint32_t)(e + 1 + lane); __any(t != 0); t >>= 1) {
            b1t *= t & 1 ? q1 : 1.0;
            b2t *= t & 1 ? q2 : 1.0;
            q1 *= q1;
            q2 *= q2;
          }
          lr_tab = (float)((double)it.lr * sqrt(1.0 - b2t) / (1.0 - b1t));
        }
        oc.lr_t = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lr_tab), lr_at));
        lr_at++;
      } else {
        oc.lr = epoch_lr(it.lr, it.power_t, e, n_fit);
      }
      __syncthreads();  // the gradients
      float g[RS];
#pragma unroll
      for (int s = 0; s < RS; s++) {
        const int r = s * W + w_;
        const float* b = lds + O_PART + r * (W * 64) + lane;
        g[s] = 0.f;
        if (r < NS) {
#pragma unroll
          for (int ww = 0; ww < W; ww++) g[s] += b[ww * 64];
        }
        g[s] = fmaf((pen >> s) & 1u ? oc.am : 0.f, p[s], g[s]);
      }
      float* rec = nullptr;
      if (traced && e >= P.step_begin && e < P.step_end) {
        rec = P.trace_out + (e - P.step_begin) * (1 + 2 * (int64_t)y.P);
        double sq = 0.0;
#pragma unroll
        for (int s = 0; s < RS; s++) sq += (pen >> s) & 1u ? (double)p[s] * (double)p[s] : 0.0;
        const double data = block_sum(lsum, red), pn = block_sum(sq, red);
        if (threadIdx.x == 0) rec[0] = (float)((data + 0.5 * (double)it.alpha * pn) / (double)mb);
      }
#pragma unroll
      for (int s = 0; s < RS; s++) {
        if (rec && ci[s] >= 0) rec[1 + ci[s]] = g[s];
        opt_update(oc, g[s], p[s], m[s], v[s]);
        if (ci[s] < 0) p[s] = m[s] = v[s] = 0.f;  // (an infinite input makes its gradient NaN)
        if (rec && ci[s] >= 0) rec[1 + y.P + ci[s]] = p[s];
      }
      publish(p);
      __syncthreads();  // the weights
      if (watch) {
        float watched;
        if (n_hold) {
          double hl = 0.0, hh = 0.0;
          score_rows(b_hold, n_hold, hl, hh);
          watched = (float)(block_sum(hl, red) / (double)n_hold);
        } else {
          watched = (float)(block_sum(lsum, red) / (double)n_fit);
        }
        const bool stop = plateau.stop_after(watched, it.tol, it.patience);
        if (n_hold && plateau.improved) {
#pragma unroll
          for (int s = 0; s < RS; s++) best[s * (W * 64)] = p[s];
          have_best = true;
        }
        if (stop) break;
      }
    }
    if (have_best) {  // the best epoch's model is the one scored
#pragma unroll
      for (int s = 0; s < RS; s++) p[s] = best[s * (W * 64)];
      __syncthreads();
      publish(p);
      __syncthreads();
    }
    double lsum = 0.0, hits = 0.0;
    score_rows(b_va, n_va, lsum, hits);
    lsum = block_sum(lsum, red);
    hits = block_sum(hits, red);
    if (threadIdx.x == 0) {
      float* out = P.item_out + 2 * ((int64_t)it.b * P.n_folds + fl);
      out[0] = n_va > 0 ? (float)(lsum / (double)n_va) : __builtin_nanf("");
      out[1] = n_va > 0 ? (float)(hits / (double)n_va) : __builtin_nanf("");  // accuracy | mean absolute error
    }
  }
};

template <int KT, int NT, int CO, int W>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * W, 64 * W), amdgpu_waves_per_eu(fu_occupancy(KT, NT, CO), fu_occupancy(KT, NT, CO))))
void k_train_full(const TrainParams P) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_item;
  __shared__ double red[W];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    if (item >= P.n_items) break;
    const __attribute__((address_space(4))) FItem* fi = (const __attribute__((address_space(4))) FItem*)P.items + item / P.n_folds;
    Full<KT, NT, CO, W> T{P, fi->d, fi->y, (float*)smem, (float*)(P.slots + (uint64_t)blockIdx.x * P.slot_bytes), red,
                       item % P.n_folds, fi->y.d, P.n_classes, (int)P.n + 48};
    T.run();
  }
}

}  // namespace
