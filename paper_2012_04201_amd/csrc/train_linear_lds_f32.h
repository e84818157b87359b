// Training / scoring kernel for fp32 models without a hidden layer and with one or two outputs (linear and logistic
// regression, two-class softmax) on data sets that fit into a CU's LDS: the case of thousands of them in one call.
// train_linear_f32.h takes every other linear model.
//
// As there, a wavefront trains one model and there is no workgroup barrier in the training loop; several wavefronts form
// a workgroup only to share the inputs: the workgroup copies the whole data set into LDS once (row stride D + 4, a 1 in
// column d for the bias, labels behind it) and each of its wavefronts then works through models from the queue.
//
//   forward   lane = row: the row is read from LDS into registers (16 bytes a read; stride / 4 is odd, so that scattered
//             rows spread over the banks), the weights are broadcast reads of the wave's own copy.
//   outputs   loss and output delta in the lane.
//   gradient  the lane keeps D sums x[k] * delta of its own rows in registers over the chunks of the step; at the step's
//             end they are folded over the 64 lanes, a halving at a time, which leaves lane t with the sum of column t.
//   update    in the owning lane, which refreshes the wave's copy of the weights.
//
// Two classes are worked on as one column.  Their softmax, its loss and both deltas depend on z[1] - z[0] alone, and the
// deltas are p and -p, p the probability of the class that is not the row's: the products run over the differences of the
// weights, one sum per column serves both gradients, and the weights themselves, their moments and their updates stay two
// (the classes of a column in lanes t and t + 32, or in one lane where there are more columns than 32).
//
// What bounds it: vector instructions, about 2 D + 40 per 64 rows for products and deltas, 2.5 D per step for the folds, and
// the row order's walk; four fifths of the time are theirs.  The order's lanes take positions from one counter: with fixed
// positions a lane, the slowest went through the network 27 times an epoch of 455 rows, and goes 16 times.  The first chunk of a
// step starts the sums, which nothing has to clear.  10,240 models of 569 x 30, two classes, 20 epochs, took 1.67 ms a call
// with a column per class and folds through the LDS crossbar, 1.11 ms before the last three, and take 0.98 ms.  (Weights in
// scalar registers instead of broadcast reads: 1.09 ms, by the 32 lane reads a step.  Gathering each chunk's rows from global
// memory, as train_linear_f32.h does: 4.9 ms.)
#pragma once
#include "common.h"
#include "train_small_f32.h"  // folding sums

namespace {

constexpr uint32_t LL_LDS_LIMIT = 160 * 1024 - 64;

// Wavefronts per SIMD the registers of a variant are budgeted for: the lane's row, its sums and about 64 more (weights on
// their way, the optimizer's and the folds' temporaries).
__host__ __device__ constexpr int ll_occupancy(int dd) { return 2 * dd + 64 <= 128 ? 4 : (2 * dd + 64 <= 168 ? 3 : 2); }
struct LinLds {
  int32_t dd, waves;           // columns (inputs and bias padded to a multiple of 8); wavefronts per workgroup, 0: not a case for it
  int32_t far;                 // groups of four columns, from the first on, that stay in global memory
  uint32_t shared, wave_bytes; // LDS of the data set and of each wavefront
};
// LDS of a wavefront: weights, the training list in the order of the early-stopping cut, the epoch's row order, the round
// function of the permutation
__host__ __device__ inline uint32_t ll_wave_bytes(int dd, int64_t n) {
  int hb = 1;
  while ((1 << (2 * hb)) < n) hb++;
  return (uint32_t)((dd * 4 + 2 * ((2 * n + 15) & ~15) + ((4 << hb) * 2)) + 15) & ~15u;
}
__host__ __device__ inline int ll_stride(int dd, int far) { return far > 0 ? dd - 4 * far : dd + 4; }
// By the size of the data set and the model alone: at least a wavefront per SIMD must fit beside the data set.  Where it
// does not, the first columns stay in global memory, as few as leave room for two wavefronts per SIMD (an odd number of
// groups: the row stride of the others must be an odd number of 16 bytes), or for one.  A lane reads its row's first columns
// itself, 16 bytes of a line of its own at a time, which the vector cache serves at a line per cycle and CU: 64 cycles a group and
// chunk.  train_linear_f32.h, which took these sets before, brings a chunk into LDS element by element.  us a call of it and
// of this: 735 x 52, 8715 models, 17 epochs 10253 and 2121; 5000 models, 10 epochs on 827 x 39 (one far group) 2893 and 904, on
// 900 x 60 (9) 4970 and 1154, on 1500 x 60 (13) 8550 and 1958; 2000 models on 4096 x 60 (15) 13381 and 3953, 40 models 6888 and 2649.
// (Room for one wavefront per SIMD only, with fewer far columns: 1500 x 60 2694 instead of 1941, 5000 models 2000 x 30 1851 and 1496.)
__host__ __device__ inline LinLds ll_plan(int64_t n, int d, int c) {
  LinLds l = {0, 0, 0, 0, 0};
  if (c > 2 || d > 63 || n < 1 || n > 4096) return l;
  l.dd = rup(d + 1, 8);
  l.wave_bytes = ll_wave_bytes(l.dd, n);
  const int most = 4 * ll_occupancy(l.dd);
  for (int least = 4; least <= 8; least += 4) {
    LinLds t = l;
    for (t.far = least == 4 ? 0 : 1; 4 * t.far <= d; t.far += t.far ? 2 : 1) {
      t.shared = (uint32_t)((n * ll_stride(l.dd, t.far) * 4 + n * 4 + 15) & ~15);
      const int fit = t.shared < LL_LDS_LIMIT ? (int)((LL_LDS_LIMIT - t.shared) / l.wave_bytes) : 0;
      t.waves = fit < most ? fit : most;
      if (t.waves >= least) break;
      t.waves = 0;
    }
    if (t.waves) l = t;
    if (l.waves && !l.far) break;
  }
  return l;
}

template <int D, int CO, bool FAR>
struct LinearLds {
  static constexpr int NQ = D / 4;
  static constexpr bool SPLIT = CO == 2 && D <= 32;  // the classes of a column in lanes t and t + 32
  static constexpr int NB = CO == 2 && !SPLIT ? 2 : 1;  // parameters of a lane
  const TrainParams& P;
  const float *xs, *ys;
  float* ws;
  uint16_t *sl, *ep, *ft;
  int lane, d, n_classes, Pn, far;

  __device__ __forceinline__ void load_row(int row, f32x4 (&x)[NQ]) const {
    if constexpr (FAR) {
      // The compiler joins the two kinds of load in one generic load of a chosen address.  Kept apart by a branch a group they are
      // slower (735 x 52 2409 us a call instead of 2121), by straight code for each number of far groups no faster in all (735 x 52
      // 2179, 900 x 60 1102 and 1154, 4096 x 60 3684 and 3953, 2300 x 56 2473 and 2253).
      typedef f32x4 __attribute__((aligned(4))) Unaligned;
      const float* away = (const float*)P.X + row * d;
      const int at = row * ll_stride(D, far) - 4 * far;
#pragma unroll
      for (int q = 0; q < NQ; q++) x[q] = q < far ? *(const Unaligned*)(away + 4 * q) : *(const f32x4*)(xs + (at + 4 * q));
    } else {
      const float* p = xs + row * (D + 4);
#pragma unroll
      for (int q = 0; q < NQ; q++) x[q] = *(const f32x4*)(p + 4 * q);
    }
  }
  // the output, or with two classes z[1] - z[0]
  __device__ __forceinline__ float forward(const f32x4 (&x)[NQ]) const {
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < NQ; i++) {
      const f32x4 w = *(const f32x4*)(ws + 4 * i);
#pragma unroll
      for (int u = 0; u < 4; u++) z += x[i][u] * w[u];
    }
    return z;
  }
  // output delta (TRAIN; with two classes that of class 1) and, if `loss`, the loss and second score of the lane's row
  template <bool TRAIN>
  __device__ __forceinline__ float outputs(float z, bool valid, float y, float inv_mb, bool loss, double& lsum, double& hits) const {
    float dl = 0.f;
    if constexpr (CO == 2) {
      const bool one = __float_as_int(y) == 1;
      if (loss && valid) {
        lsum += (double)sm_two_class_loss(z, one);
        hits += (z > 0.f) == one ? 1.0 : 0.0;
      }
      if (TRAIN) dl = sm_two_class_delta(z, one) * inv_mb;
    } else if (n_classes == 1) {
      const int yr = __float_as_int(y);
      if (loss && valid) {
        lsum += (double)(fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - (yr ? z : 0.f));
        hits += (z > 0.f) == (yr != 0) ? 1.0 : 0.0;
      }
      if (TRAIN) dl = (1.f / (1.f + expf(-z)) - (float)yr) * inv_mb;
    } else {
      const float e0 = z - y;
      if (loss && valid) {
        lsum += TRAIN ? 0.5 * (double)e0 * (double)e0 : (double)e0 * (double)e0;
        hits += (double)fabsf(e0);  // the absolute error
      }
      if (TRAIN) dl = e0 * inv_mb;
    }
    return valid ? dl : 0.f;  // (a row that is not there must not put an infinity of another row into the sums)
  }
  // Sum over the 64 lanes of g[t] for column t = lane, or lane mod 32 where there are no more than 32.  The halvings over the
  // 16-lane rows come first, while there are the most columns: two instructions each, where one within a row takes three.
  __device__ __forceinline__ float fold(const float (&g)[D]) const {
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
    constexpr int H = D < 16 ? D : 16;
    auto upper = [&](int t) { return sm_fold32(g[t], t + 32 < D ? g[t + 32 < D ? t + 32 : 0] : 0.f); };
    float v[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int c = 4 * t + e;
        p[e] = 0.f;
        if (c < H) {
          if constexpr (D > 32)
            p[e] = sm_fold16(upper(c < H ? c : 0), upper(c < H ? c + 16 : 0));
          else if constexpr (D > 16)
            p[e] = sm_fold16(g[c < H ? c : 0], c + 16 < D ? g[c + 16 < D ? c + 16 : 0] : 0.f);
          else
            p[e] = g[c < H ? c : 0];
        }
      }
      v[t] = 4 * t < H ? sm_fold_quad(p, b0, b1) : 0.f;
    }
    float r = sm_fold_row(v, b2, b3);
    if constexpr (D <= 16) r = sm_fold16(r, r);
    if constexpr (D <= 32) r = sm_fold32(r, r);
    return r;
  }
  // the epoch's rows in visiting order (see train_linear_f32.h)
  __device__ __forceinline__ void epoch_order(uint64_t ke, int n_fit) const {
    if (n_fit <= 1) {
      if (lane < n_fit) ep[lane] = sl[0];
    } else {
      const PermDomain dm = perm_domain((uint32_t)n_fit);
      for (int i = lane; i < (4 << dm.hb); i += 64)
        ft[i] = (uint16_t)((uint32_t)key_fold(ke, ((uint64_t)(i >> dm.hb) << 32) | ((uint32_t)i & dm.mask)) & dm.mask);
      __builtin_amdgcn_wave_barrier();
      // a lane that has its position's row takes the next position that no lane has: positions differ in how often they
      // go through the network
      int p = lane, next = 64;
      uint32_t x = (uint32_t)p;
      while (p < n_fit) {
        uint32_t Lh = x >> dm.hb, Rh = x & dm.mask;
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const uint32_t t = Lh ^ ft[(r << dm.hb) + Rh];
          Lh = Rh;
          Rh = t;
        }
        x = (Lh << dm.hb) | Rh;
        const bool found = x < (uint32_t)n_fit;
        const uint64_t all = __ballot(found);
        if (found) {
          ep[p] = sl[x];
          p = next + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0));
          x = (uint32_t)p;
        }
        next += __popcll(all);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // The lane's column and its b-th parameter: class, place in the packed order W[in][out], b[out] (from Pn on: none).
  __device__ __forceinline__ int column() const { return SPLIT ? lane & 31 : lane; }
  __device__ __forceinline__ int cls(int b) const { return SPLIT ? lane >> 5 : b; }
  __device__ __forceinline__ int packed(int b) const { return column() * CO + cls(b); }
  __device__ __forceinline__ void put_weights(const float (&w)[NB]) const {
    float x = w[NB - 1];
    if constexpr (SPLIT) x = __shfl_xor(x, 32) - x;  // (class 0 of a column is in the lower lane)
    if constexpr (NB == 2) x -= w[0];
    if (lane < D) ws[lane] = x;
    __builtin_amdgcn_wave_barrier();
  }
  // loss and second score, summed per lane, of `count` rows
  template <class RowAt>
  __device__ __forceinline__ void score_rows(int count, RowAt row_at, double& lsum, double& hits) const {
    for (int off = 0; off < count; off += 64) {
      const bool valid = off + lane < count;
      const int row = row_at(valid ? off + lane : count - 1);
      f32x4 x[NQ];
      load_row(row, x);
      outputs<false>(forward(x), valid, ys[row], 0.f, true, lsum, hits);
    }
  }

  __device__ __forceinline__ void run(const ConstItemDesc& it, int fl) const {  // fl: which row list
    const int n_tr = uniform(P.counts[2 * fl]), n_va = uniform(P.counts[2 * fl + 1]);
    const int32_t* tr = P.train_idx + (int64_t)fl * P.n;
    const int32_t* va = P.val_idx + (int64_t)fl * P.n;
    const uint64_t km = key_model(it.seed, fl + P.fold_base);
    const RowSplit sp = row_split(km, it.patience, it.val_frac, n_tr);
    const int n_fit = sp.n_fit, n_hold = sp.n_hold;
    const int bs = eff_batch(it.batch_size, n_fit);
    const int steps = n_fit > 0 ? (n_fit + bs - 1) / bs : 0;
    const float alpha = it.alpha;
    // of a step of all `bs` rows and of an epoch's last (divisions take a dozen instructions each)
    const float mb_full = (float)bs, mb_rest = (float)(n_fit - (steps - 1) * bs);
    const float inv_full = uniform(1.f / mb_full), inv_rest = uniform(1.f / mb_rest);
    const float am_full = uniform(alpha / mb_full), am_rest = uniform(alpha / mb_rest);
    const bool traced = P.trace_item == it.b * P.n_folds + fl;
    const bool resume = traced && P.state_in && steps > 0;

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
    oc.am = 0.f;

    for (int p = lane; p < n_tr; p += 64) sl[p] = (uint16_t)tr[n_hold ? (int)perm_index(sp.ksplit, (uint32_t)n_tr, (uint32_t)p) : p];
    float w[NB], m[NB], v[NB], wb[NB];
    const int n_w = d * CO;  // weights in front, biases behind
#pragma unroll
    for (int b = 0; b < NB; b++) {
      const int i = packed(b);
      w[b] = m[b] = v[b] = wb[b] = 0.f;
      if (i < Pn) {
        if (resume) {
          w[b] = P.state_in[i];
          m[b] = P.state_in[Pn + i];
          v[b] = P.state_in[2 * Pn + i];
        } else {
          const uint32_t k24 = (uint32_t)(key_fold(key_fold(km, i < n_w ? 16 : 17), (uint64_t)(i < n_w ? i : i - n_w)) >> 40);
          w[b] = it.bound[0] * ((float)((int32_t)k24 - 8388608) * 0x1p-23f);
        }
      }
    }
    put_weights(w);

    int64_t gstep = resume ? P.step_begin : 0;
    const int e0 = resume ? (int)(gstep / steps) : 0, st0 = resume ? (int)(gstep % steps) : 0;
    float lr_tab = 0.f;  // Adam: the step sizes of 64 steps, one per lane
    int lr_at = 64;      // ... the next of them
    Plateau plateau;
    bool have_best = false;
    const bool watch = it.patience > 0 && steps > 0 && !resume;
    const bool loss = traced || (watch && !n_hold);
    for (int e = e0; e < it.epochs && steps > 0; e++) {
      epoch_order(key_epoch(km, e), n_fit);
      if (!oc.adam) oc.lr = epoch_lr(it.lr, it.power_t, e, n_fit);
      double esum = 0.0, unused = 0.0;  // the lane's share of the epoch's summed data loss
      for (int st = e == e0 ? st0 : 0; st < steps; st++, gstep++) {
        const int lo = st * bs, hi = min(lo + bs, n_fit);
        const float mb = (float)(hi - lo), inv_mb = hi - lo == bs ? inv_full : inv_rest;
        float g[D];
        double lstep = 0.0;
        auto chunk = [&](int at, auto first) {
          asm volatile("" ::: "memory");  // the weights are read again for every chunk, not kept in registers
          const int row = ep[min(at + lane, hi - 1)];
          f32x4 x[NQ];
          load_row(row, x);
          const float dl = outputs<true>(forward(x), at + lane < hi, ys[row], inv_mb, loss, lstep, unused);
#pragma unroll
          for (int i = 0; i < D; i++) g[i] = first ? x[i / 4][i % 4] * dl : fmaf(x[i / 4][i % 4], dl, g[i]);
        };
        chunk(lo, std::true_type{});
        for (int at = lo + 64; at < hi; at += 64) chunk(at, std::false_type{});
        const float gs = fold(g);
        esum += lstep;
        oc.am = hi - lo == bs ? am_full : am_rest;
        if (oc.adam) {
          if (lr_at == 64) {
            // beta^t of the next 64 steps, a step per lane, by repeated squaring in double
            lr_at = 0;
            double q1 = (double)it.beta1, q2 = (double)it.beta2, b1t = 1.0, b2t = 1.0;
#pragma unroll 1
            for (uint64_t t = (uint64_t)(gstep + 1) + lane; __any(t != 0); t >>= 1) {
              b1t *= t & 1 ? q1 : 1.0;
              b2t *= t & 1 ? q2 : 1.0;
              q1 *= q1;
              q2 *= q2;
            }
            lr_tab = (float)((double)it.lr * sqrt(1.0 - b2t) / (1.0 - b1t));
          }
          oc.lr_t = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lr_tab), lr_at));
          lr_at++;
        }
        float* rec = nullptr;
        if (traced && gstep >= P.step_begin && gstep < P.step_end) {
          rec = P.trace_out + (gstep - P.step_begin) * (1 + 2 * (int64_t)Pn);
          double pen = 0.0;
#pragma unroll
          for (int b = 0; b < NB; b++)
            if (packed(b) < n_w) pen += (double)w[b] * (double)w[b];
          const double data = sm_wavesum_d(lstep) / (double)mb;
          pen = sm_wavesum_d(pen);
          if (lane == 0) rec[0] = (float)(data + 0.5 * (double)alpha * pen / (double)mb);
        }
#pragma unroll
        for (int b = 0; b < NB; b++) {
          const int i = packed(b);
          if (i < Pn) {
            const float gg = (CO == 2 && cls(b) == 0 ? -gs : gs) + (i < n_w ? oc.am * w[b] : 0.f);
            opt_update(oc, gg, w[b], m[b], v[b]);
            if (rec) {
              rec[1 + i] = gg;
              rec[1 + Pn + i] = w[b];
            }
          }
        }
        put_weights(w);
      }
      if (watch) {
        float watched = (float)(sm_wavesum_d(esum) / (double)n_fit);
        if (n_hold) {  // the loss of the rows set aside for early stopping, under the weights the epoch ends with
          double hl = 0.0, hh = 0.0;
          score_rows(n_hold, [&](int p) { return (int)sl[n_fit + p]; }, hl, hh);
          watched = (float)(sm_wavesum_d(hl) / (double)n_hold);
        }
        const bool stop = plateau.stop_after(watched, it.tol, it.patience);
        if (n_hold && plateau.improved) {
#pragma unroll
          for (int b = 0; b < NB; b++) wb[b] = w[b];
          have_best = true;
        }
        if (stop) break;
      }
    }
    if (have_best) put_weights(wb);  // early stopping on held-out rows scores the best epoch's model

    double lsum = 0.0, hits = 0.0;
    score_rows(n_va, [&](int p) { return va[p]; }, lsum, hits);
    lsum = sm_wavesum_d(lsum);
    hits = sm_wavesum_d(hits);
    if (lane == 0) {
      float* out = P.item_out + 2 * ((int64_t)it.b * P.n_folds + fl);
      out[0] = n_va > 0 ? (float)(lsum / (double)n_va) : __builtin_nanf("");
      out[1] = n_va > 0 ? (float)(hits / (double)n_va) : __builtin_nanf("");  // accuracy | mean absolute error
    }
  }
};

// The launch gives a workgroup the LDS of the data set and ll_wave_bytes() for each of its wavefronts.
template <int D, int CO, bool FAR>
__global__ __attribute__((amdgpu_flat_work_group_size(64, 256 * ll_occupancy(D)),
                          amdgpu_waves_per_eu(ll_occupancy(D), ll_occupancy(D))))
void k_train_linear_lds(const TrainParams P) {
  extern __shared__ __align__(16) char ll_lds[];
  typedef LinearLds<D, CO, FAR> T;
  const int n = (int)P.n, d = P.d;
  const int far = FAR ? uniform(ll_plan(n, d, CO).far) : 0, S = ll_stride(D, far);
  float *xs = (float*)ll_lds, *ys = xs + n * S;
#pragma unroll 8
  for (int i = threadIdx.x; i < n * S; i += blockDim.x) {
    const int r = i / S, k = 4 * far + i - r * S;
    xs[i] = k < d ? ((const float*)P.X)[r * d + k] : (k == d ? 1.f : 0.f);
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) ys[i] = ((const float*)P.y)[i];  // (class ids as they are)
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  char* own = ll_lds + (((uint32_t)(n * S + n) * 4 + 15) & ~15u) + wave * ll_wave_bytes(D, n);
  const uint32_t list = (2 * n + 15) & ~15u;
  T t{P, xs, ys, (float*)own, (uint16_t*)(own + D * 4), (uint16_t*)(own + D * 4 + list),
      (uint16_t*)(own + D * 4 + 2 * list), lane, d, P.n_classes, (d + 1) * CO, far};
  for (;;) {
    // every lane takes part in the pop (see k_train_linear)
    __builtin_amdgcn_wave_barrier();
    const int item = __builtin_amdgcn_readfirstlane(atomicAdd(P.queue, lane == 0 ? 1 : 0));
    if (item >= P.n_items) break;
    t.run(((ConstItemDesc*)P.items)[item / P.n_folds], item % P.n_folds);
  }
}

}  // namespace
