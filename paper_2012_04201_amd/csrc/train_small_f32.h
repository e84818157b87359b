// Register-resident training / scoring kernel for small fp32 models with one hidden layer (the "many concurrent
// studies" shape: up to 63 inputs, hidden width up to 224, up to 4 outputs).  Two classes are one output column, the
// difference of the logits (see sm_two_class_delta()).
//
// One workgroup of W waves trains one model.  Wave w owns the hidden-unit tiles (16 units) w, w + W, .. for the
// whole run, and everything that belongs to them stays in its registers (as far as these reach: sm_occupancy()) from the
// first draw to the score: the
// hidden layer's weights, both moments and the step's gradient, and the units' rows of the output layer with
// theirs.  That works because the MFMA (16x16x4 fp32) wants a weight in the same lane as operand of the forward
// product as it leaves its gradient in: lane (unit li, columns 4q..4q+3 of a k tile).  The output bias is kept by
// every wave, and every wave computes the loss and the output delta of all rows of a chunk (lane = row), so the
// waves exchange nothing but their partial outputs: ONE barrier per chunk of 64 rows.
//
//   forward   D[row][unit] = xs[row][k] . w1[unit][k], accumulators started at the unit's bias; ReLU; the wave's
//             share of the outputs is summed over the 16 unit lanes by a folding tree that leaves the total of row
//             (rt, 4q + e) in lane (q, li = 4 rt + e): one value per lane and output, parked in LDS
//   outputs   sum of the waves' shares, softmax / logistic / squared loss, output delta (lane = row)
//   backward  hidden deltas in the accumulators, which feed the MFMA again as the B operand of the weight gradient
//             D[k][unit] += xs[row][k] . delta[row][unit]
//   update    Adam / SGD, registers only
//
// Inputs are fetched two chunks ahead: requested into registers right after a chunk's barrier, put into LDS before
// the next one (three input tiles in rotation, so that neither needs a barrier of its own).  The rows of an epoch
// are tabled in LDS (16-bit row ids; one table, written anew when the epoch's first chunk is about to be requested); the
// rows set aside for early stopping are scored by the same loop as chunks of their own between two epochs, and so are
// the held fold's rows at the end.  A set of more than 65,535 rows, or whose tables do not fit, is permuted chunk by chunk.
//
// What bounds it: with the chip full, the matrix pipe shares its SIMD with the vector work around it (ReLU, output
// layer, softmax, update), and two to four waves per SIMD have to cover each other's latencies; with few models,
// the chain of a step's dependent phases.  The optimizer's work on the small parameters (biases, output layer: alike in the
// four lane groups q) is done four parameters at a time, one per q; the loss of a training chunk is computed only where the
// stopping rule or a trace reads it.  With the output columns of two classes merged, these took 10,240 models 569 x 30 from
// 30.7 to 27.4 ms and 40 models of 10,000 x 45 from 4.02 to 3.59; products in split bfloat16 (sm_split()) and the leaner
// schedule then to 24.2 and 3.56, hidden deltas without the output weight, small parameters in registers and moments in units of
// their own to 19.0 and 3.46, rare code apart to 18.9 and 3.42.  The form before this one kept the weights in LDS and the moments in L2, at
// two workgroups per CU whatever the width and two barriers per chunk.  Before and after, per call: 10,240 models
// 569 x 30, 50..200 units, 20 epochs 45.3 -> 32.4 ms; 40 models 506 x 13, SGD, 30 epochs 3.41 -> 1.74 ms; 40 models of
// 10,000 x 45 rows, 3 epochs 10.9 -> 4.45 ms; 40 models 150 x 4, 20 epochs 0.39 -> 0.25 ms.
//
// LDS: xs[3][64][16 KT + 4] inputs (the stride spreads the 16 rows of an operand over all banks and the four row
// groups of a gradient operand over its quarters), zp[2][W][CO][64], d2[CO][64], ys[3][64], row lists.
#pragma once
#include "common.h"

namespace {

constexpr int SM_RC = 64;                   // rows per chunk
constexpr int SM_MAX_WAVES = 8;
constexpr uint32_t SM_LDS_LIMIT = 156 * 1024;  // of a workgroup, row tables included
constexpr int SM_NET = 4096;                 // rows up to which an epoch's permutation network is tabled whole

// How a model is cut: waves per workgroup and unit tiles per wave.
struct SmallCut {
  int kt, nt, co, waves;
};

// Row pipeline part of a model's LDS layout: where the row tables lie (what precedes them is fixed by the variant).
struct PipeLay {
  int32_t d, P;    // inputs; parameters of the model
  int32_t netted;  // the permutation network is tabled whole
  int32_t tabled;  // the epoch's rows are tabled in LDS; otherwise they are permuted chunk by chunk
  uint32_t o_ft, o_net, o_sl, o_ep, total;
};

struct SLay {
  PipeLay p;
  int32_t h, c, nut;
  int32_t cw[2], cb[2];
  uint32_t lds_total, slot_floats;  // slot: the wave's parameters as they are drawn, and the best epoch's
};

struct SItem {
  ItemDesc d;
  SLay y;
};

__host__ __device__ inline bool small_eligible(const int32_t* dims, int L) {
  return L == 2 && dims[0] <= 63 && dims[1] <= 224 && dims[2] <= 4;
}
__host__ __device__ constexpr int sm_ldw(int kt) { return 16 * kt + 4; }
// registers a wave needs to park its share of the parameters
__host__ __device__ constexpr int sm_regs(int kt, int nt, int co) { return nt * (4 * kt + 1 + co) + co; }

// The cut depends on the shape alone, never on the call: the order in which the waves' partial outputs are added
// is part of a suggestion's result, and that must not depend on its companions.
constexpr SmallCut sm_cut(int kt, int nut, int co) {  // nut: unit tiles
  const int ntmax = kt == 4 ? 1 : (kt == 3 || co == 4 ? 2 : 3);
  int waves = kt == 1 && nut <= 2 ? 2 : 4;  // two waves could not hold the inputs of a wider chunk in flight
  if (nut > waves * ntmax) waves = 8;
  return SmallCut{kt, (nut + waves - 1) / waves, co, waves};
}
__host__ inline SmallCut small_cut(const int32_t* dims) {
  return sm_cut(rup(dims[0], 16) / 16, rup(dims[1], 16) / 16, dims[2] <= 2 ? dims[2] : 4);
}
// is there a model with this cut?
constexpr bool sm_occurs(int kt, int nt, int co, int waves) {
  for (int nut = 1; nut <= 224 / 16; nut++) {
    const SmallCut s = sm_cut(kt, nut, co);
    if (s.nt == nt && s.waves == waves) return true;
  }
  return false;
}

// Inputs in three bfloat16 planes (see SmPlanes): blocks of 32 columns, elements of a row (the pad spreads the rows over
// the banks), bytes of a tile of 64 rows.
__host__ __device__ constexpr int sm_blocks(int kt) { return (kt + 1) / 2; }
__host__ __device__ constexpr int sm_ldb(int kt) { return 32 * sm_blocks(kt) + 8; }
__host__ __device__ constexpr uint32_t sm_tile_bytes(int kt, bool planes) {
  return planes ? 3 * SM_RC * sm_ldb(kt) * 2 : SM_RC * sm_ldw(kt) * 4;
}
// LDS of the row pipeline: input tiles, labels, row lists
__host__ __device__ constexpr uint32_t pipe_lds(int kt, int buffers, bool planes) {
  return buffers * sm_tile_bytes(kt, planes) + (buffers * SM_RC + 2 * SM_RC) * 4;
}
// LDS of a variant of k_train_small ahead of the row tables
__host__ __device__ constexpr int sm_columns(int co) { return co == 2 ? 1 : co; }
// Products in split bfloat16 (see SmPlanes)?  With two input tiles, and with four where they fill the wave's registers least:
// one tile is half of such a product, three are three quarters of two.  569 x 30 and 569 x 60, two classes, 400 suggestions,
// us a call with fp32 products and split: 200 units, 30 inputs, 128 rows a step 1483 and 1175, 32 rows 2018 and 1917; 64
// units, 60 inputs 813 and 643, 1122 and 984.  What does not fit spills and loses: one unit tile and two input tiles (four
// waves a SIMD) 430 and 287 the other way, 128 units and 45 inputs 1648 and 1299.
__host__ __device__ constexpr bool sm_split(int kt, int nt, int co) { return (kt == 2 && nt >= 2) || (kt == 4 && nt == 1 && co <= 2); }
// With four input tiles three buffers of planes would leave room for one workgroup a CU: two, and a second barrier.
__host__ __device__ constexpr int sm_barriers(int kt, int nt, int co) { return kt == 4 && sm_split(kt, nt, co) ? 2 : 1; }
// Hidden deltas without the output weight (see Small::FACTORED): the rows' deltas lie in LDS as planes too.
__host__ __device__ constexpr bool sm_factored(int kt, int nt, int co) { return sm_columns(co) == 1 && (kt > 1 || sm_split(kt, nt, co)); }
__host__ __device__ constexpr uint32_t sm_delta_planes(int kt, int nt, int co) {
  return sm_factored(kt, nt, co) && sm_split(kt, nt, co) ? 3 * SM_RC * 2 : 0;
}
__host__ __device__ constexpr uint32_t sm_fixed_lds(int kt, int nt, int co, int waves) {
  return pipe_lds(kt, 4 - sm_barriers(kt, nt, co), sm_split(kt, nt, co)) + (2 * waves + 1) * sm_columns(co) * SM_RC * 4 +
         sm_delta_planes(kt, nt, co);
}

// ... and the row tables behind `fixed` bytes of everything else
__host__ inline void make_pipelay(PipeLay& y, int d, int P, int64_t n, uint32_t fixed) {
  y.d = d;
  y.P = P;
  uint32_t o = 0;
  auto take = [&](uint32_t bytes) {
    uint32_t r = o;
    o += (bytes + 15) & ~15u;
    return r;
  };
  take(fixed);
  // 16-bit tables: the fold's row list in the order of the early-stopping cut, the epoch's row order, the round
  // function of the permutation network and, up to SM_NET rows, the whole network
  int hb = 1;
  while ((1 << (2 * hb)) < n) hb++;
  const uint32_t ft = (uint32_t)((4 << hb) * 2), net = n <= SM_NET ? 2u << (2 * hb) : 0u;
  const uint32_t tab = (uint32_t)(2 * (n + SM_RC));  // (a chunk may read its row ids past the end: spare entries)
  const uint32_t need = o + ft + 2 * tab + 64;         // (rounded up to 16 bytes each)
  y.tabled = n >= 1 && n <= 0xffff && need <= SM_LDS_LIMIT;
  y.netted = net > 0 && need + net <= SM_LDS_LIMIT;  // (sized for n rows; the fold's own network is never wider)
  y.o_ft = y.o_net = y.o_sl = y.o_ep = o;
  if (y.tabled) {
    y.o_ft = take(ft);
    y.o_net = take(y.netted ? net : 0u);
    y.o_sl = take(tab);
    y.o_ep = take(tab);
  }
  y.total = o;
}

__host__ inline void make_slay(SLay& y, const int32_t* dims, int64_t n, const SmallCut& s) {
  const int d = dims[0];
  y.h = dims[1];
  y.c = dims[2];
  y.nut = rup(dims[1], 16) / 16;
  y.cw[0] = 0;
  y.cb[0] = d * y.h;
  y.cw[1] = y.cb[0] + y.h;
  y.cb[1] = y.cw[1] + y.h * y.c;
  make_pipelay(y.p, d, y.cb[1] + y.c, n, sm_fixed_lds(s.kt, s.nt, s.co, s.waves));
  y.slot_floats = (uint32_t)(s.waves * sm_regs(s.kt, s.nt, s.co) * 64);
  y.lds_total = y.p.total;
}

// Waves per SIMD the registers of a variant are budgeted for (512 registers per lane and SIMD).  The largest variants of a
// budget do not fit it altogether: by the compiler's report <2,3,1,4> and <2,3,2,4> (129 to 192 units, 17 to 32 inputs)
// spill 102 and 118 vector registers, <3,2,4,4> and <3,2,4,8> 103 and 75, <4,2,.,8> (129 units and more, 49 inputs and more)
// 109, 105 and 222 at one, two and four output slots; the others 21 at most.  (<3,2,4,.> at first spilled 82 and 62 with the moments of the
// small parameters in LDS.  45 inputs, four classes, 200 suggestions, us a call then and now: 100 units, 24, 64 and 128 rows a step
// 1202 and 1185, 727 and 720, 649 and 669; 130 units 1165 and 1081 at 64 rows.  These moments in LDS again, four a lane: 60 and
// 42 spilled, 100 units 671 at 128 rows, 130 units 1100 at 64.)  Four output slots need more than the 128
// registers of four waves even at one tile: at three, 569 x 30, three classes, 16 units, 32 rows a step, 400 suggestions take
// 622 us a call instead of 857.
__host__ __device__ constexpr int sm_occupancy(int kt, int nt, int co) {
  return nt == 1 && kt <= 2 ? (co == 4 ? 3 : 4) : 2;
}
// workgroups a CU holds
__host__ inline int small_per_cu(const SmallCut& s, uint32_t lds_bytes) {
  const int by_regs = 4 * sm_occupancy(s.kt, s.nt, s.co) / s.waves, by_lds = (int)(160u * 1024u / (lds_bytes + 512));
  const int n = by_regs < by_lds ? by_regs : by_lds;
  return n < 1 ? 1 : n;
}

template <int CTRL>
__device__ __forceinline__ float sm_dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// Halvings over the four 16-lane rows of a wave.  sm_fold16: rows 0, 1 get the sums of a over rows 0 and 1 and of b over
// rows 0 and 1, rows 2, 3 the same of rows 2 and 3; sm_fold32: the lower half gets the sum of a over both halves, the upper
// half that of b.  (The swaps return a pair; an element of it must be read as the integer it is: a bit cast of the
// element itself takes the first one.)
__device__ __forceinline__ float sm_fold16(float a, float b) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const uint32_t x = s[0], y = s[1];
  return __uint_as_float(x) + __uint_as_float(y);
}
__device__ __forceinline__ float sm_fold32(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const uint32_t x = s[0], y = s[1];
  return __uint_as_float(x) + __uint_as_float(y);
}
// Sum over the four 16-lane rows of a wave, the same bits in every lane.
__device__ __forceinline__ float sm_rowsum(float v) {
  v = sm_fold16(v, v);
  return sm_fold32(v, v);
}
// Sum over the 16 lanes of a row, the same bits in every lane.
__device__ __forceinline__ float sm_row16sum(float v) {
  v += sm_dpp<0x128>(v);  // row rotation by 8
  v += sm_dpp<0x141>(v);  // mirror within 8 lanes
  v += sm_dpp<0x4E>(v);   // quad permutations
  return v + sm_dpp<0xB1>(v);
}
__device__ __forceinline__ double sm_wavesum_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
// Folding sums over the 16 lanes of a row.  sm_fold_quad: four values p[e]; lane e of each quad is left with the
// quad's sum of p[e].  sm_fold_row: four values v[rt]; quad rt of each row is left with the sum over the four
// quads of v[rt], lane by lane.  A lane hands on the half it does not keep: three instructions per halving.
__device__ __forceinline__ float sm_fold_quad(const float (&p)[4], bool b0, bool b1) {
  const float A = (b0 ? p[1] : p[0]) + sm_dpp<0xB1>(b0 ? p[0] : p[1]);
  const float B = (b0 ? p[3] : p[2]) + sm_dpp<0xB1>(b0 ? p[2] : p[3]);
  return (b1 ? B : A) + sm_dpp<0x4E>(b1 ? A : B);
}
__device__ __forceinline__ float sm_fold_row(const float (&v)[4], bool b2, bool b3) {
  const float A = (b3 ? v[2] : v[0]) + sm_dpp<0x128>(b3 ? v[0] : v[2]);
  const float B = (b3 ? v[3] : v[1]) + sm_dpp<0x128>(b3 ? v[1] : v[3]);
  const float x = sm_dpp<0x141>(b2 ? A : B);       // lane i gets 7 - i of its eight,
  return (b2 ? B : A) + sm_dpp<0x1B>(x);           // and the reversal of the quad makes that i ^ 4
}

// Two classes by the difference of their logits, z = z[1] - z[0], of a row of class `one`.  The delta of class 1 (before
// the division by the step's rows; class 0 has its negative): the probability of the other class, which does not cancel
// as p - 1 does.  An infinite difference is a NaN in both, as it is with the logits apart.
__device__ __forceinline__ float sm_two_class_delta(float z, bool one) {
  const float p = fmaf(z, 0.f, 1.f / (1.f + expf(one ? z : -z)));
  return one ? -p : p;
}
__device__ __forceinline__ float sm_two_class_loss(float z, bool one) {
  const float s = one ? -z : z;  // of the other class over the row's own
  return fmaf(z, 0.f, fmaxf(s, 0.f) + log1pf(expf(-fabsf(s))));
}

// Output deltas of a lane's row from its outputs (two classes: their difference) and, if `loss`, its loss and second score.
template <int CO>
__device__ __forceinline__ void sm_outputs(const float (&z)[sm_columns(CO)], float yv, bool valid, int c, int n_classes, bool train,
                                           bool loss, float inv_mb, float (&dl)[sm_columns(CO)], double& lsum, double& hits) {
  constexpr int ZO = sm_columns(CO);
  const int yr = __float_as_int(yv);
#pragma unroll
  for (int cc = 0; cc < ZO; cc++) dl[cc] = 0.f;
  if (!valid) return;
  if constexpr (CO == 2) {
    const bool one = yr == 1;
    if (loss) {
      lsum += (double)sm_two_class_loss(z[0], one);
      hits += (z[0] > 0.f) == one ? 1.0 : 0.0;
    }
    dl[0] = sm_two_class_delta(z[0], one) * inv_mb;
  } else if constexpr (CO > 2) {
    float mx = z[0], zy = z[0];
    int best = 0;
#pragma unroll
    for (int cc = 1; cc < ZO; cc++)
      if (cc < c) {
        if (z[cc] > mx) {
          mx = z[cc];
          best = cc;
        }
        zy = cc == yr ? z[cc] : zy;
      }
    float ex[ZO], se = 0.f;
#pragma unroll
    for (int cc = 0; cc < ZO; cc++)
      if (cc < c) {
        ex[cc] = expf(z[cc] - mx);
        se += ex[cc];
      }
    if (loss) {
      lsum += (double)(mx + logf(se) - zy);
      hits += best == yr ? 1.0 : 0.0;
    }
    const float inv = 1.f / se;
#pragma unroll
    for (int cc = 0; cc < ZO; cc++)
      if (cc < c) dl[cc] = (ex[cc] * inv - (cc == yr ? 1.f : 0.f)) * inv_mb;
  } else if (n_classes == 1) {
    // one logit, labels 0/1: log(1 + e^z) - y z, delta (sigmoid(z) - y)/m
    const float zz = z[0];
    if (loss) {
      lsum += (double)(fmaxf(zz, 0.f) + log1pf(expf(-fabsf(zz))) - (yr ? zz : 0.f));
      hits += (zz > 0.f) == (yr != 0) ? 1.0 : 0.0;
    }
    dl[0] = (1.f / (1.f + expf(-zz)) - (float)yr) * inv_mb;
  } else {
    const float e0 = z[0] - yv;
    if (loss) {
      lsum += train ? 0.5 * (double)e0 * (double)e0 : (double)e0 * (double)e0;
      hits += (double)fabsf(e0);  // the absolute error
    }
    dl[0] = e0 * inv_mb;
  }
}

// A float in three bfloat16 parts, x = h + m + l: each the rest rounded to nearest, so that the sum is exact (8 + 8 + 8 bits
// of 24).  A product of two such numbers is summed over six of the nine pairs, smallest first; the three left out are below
// 2^-24 of it.  Per 32 contracted elements that is six matrix instructions of 16 cycles instead of eight of 32, and the
// result is closer to the exact one: over 64 normal pairs 9.4e-8 relative rms against 1.45e-7 of the fp32 instructions.
// (Infinities come out as NaN.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
struct SmPlanes {  // eight elements a lane, as operands
  u32x4 h, m, l;
};
__device__ __forceinline__ uint32_t sm_pack(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 x = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}
__device__ __forceinline__ float sm_low(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float sm_high(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ void sm_split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = sm_pack(a, b);
  a -= sm_low(h);
  b -= sm_high(h);
  m = sm_pack(a, b);
  l = sm_pack(a - sm_low(m), b - sm_high(m));
}
__device__ __forceinline__ f32x4 sm_mfma(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// An activation's derivative, 1 or 0 (0 for a NaN), and two of them as a mask of two bfloat16 values.
__device__ __forceinline__ float sm_active(float a) { return __builtin_amdgcn_fmed3f(__builtin_ldexpf(a, 200), 0.f, 1.f); }
__device__ __forceinline__ uint32_t sm_mask(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pknorm_u16(a, b)); }
// The s-th of the six products, smallest first.
template <int S>
__device__ __forceinline__ f32x4 sm_product(const SmPlanes& a, const SmPlanes& b, const f32x4& c) {
  if constexpr (S == 0) return sm_mfma(a.l, b.h, c);
  if constexpr (S == 1) return sm_mfma(a.h, b.l, c);
  if constexpr (S == 2) return sm_mfma(a.m, b.m, c);
  if constexpr (S == 3) return sm_mfma(a.m, b.h, c);
  if constexpr (S == 4) return sm_mfma(a.h, b.m, c);
  return sm_mfma(a.h, b.h, c);
}
// N independent sums, c[i] += a . b[i], one product of each in turn
template <int N, int S = 0>
__device__ __forceinline__ void sm_products(const SmPlanes& a, const SmPlanes* b, f32x4* c) {
#pragma unroll
  for (int i = 0; i < N; i++) c[i] = sm_product<S>(a, b[i], c[i]);
  if constexpr (S < 5) sm_products<N, S + 1>(a, b, c);
}
// Transposing LDS read of 16-bit elements: of the 16 x 4 elements that a row of 16 lanes addresses (lane t: four columns of
// row t / 4 from column 4 (t mod 4) on) lane t gets column t of the four rows.
__device__ __forceinline__ u32x2 sm_read_tr(const char* p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p));
}

// What the phases of a chunk need to know about it, packed into one scalar (two chunks are in the pipeline behind
// the position that is being advanced): its rows (0..64), what it is, and flags, one bit for each question that the loop
// asks of a chunk.  Scalar work is slow for the few waves of a SIMD (8 cycles an instruction, 26 a taken branch, 32 for a
// value fetched back from a spill), and all of it lies on the chain of a step.
enum {
  SC_ROWS = 0x7f,
  SC_TRAIN = 1 << 7,     // rows of an epoch's step
  SC_HELD = 1 << 8,      // rows set aside
  SC_PLAIN = 1 << 9,     // the held fold
  SC_LIVE = 7 << 7,      // any of these: the pipeline is neither filling nor running dry
  SC_END = 1 << 10,      // past the last chunk
  SC_FIRST = 1 << 11,    // first chunk of a step, or of a scoring pass
  SC_LAST = 1 << 12,     // last chunk of a step
  SC_RAGGED = 1 << 13,   // the epoch's last step
  SC_EPOCH = 1 << 14,    // the epoch's first step
  SC_DECIDE = 1 << 15,   // the stopping rule is applied after it
  SC_SLOW = 1 << 16,     // first chunk of a step that opens with more than the next learning rate
  SC_PARK = 1 << 17,     // its rows are looked up chunk by chunk
  SC_TABLE = 1 << 18,    // its epoch's rows are to be tabled
};

// A condition of RowPipe::run() that few steps meet: its code goes behind the step's, and what spills, spills there.  Not
// the row lookups, which are every chunk's where rows are not tabled (70,000 x 13 1.01 to 1.02 of its time with them).  A macro: the
// compiler takes the hint at a branch, before it inlines anything.
#define SM_RARE(x) (Self::RARE_APART ? __builtin_expect(!!(x), 0) : !!(x))

// The row pipeline of a training run, shared by the kernels that take their inputs through LDS in chunks of 64 rows:
// the schedule, the rows of an epoch, the inputs two chunks ahead, the stopping rules, tracing and the scores.  `Self`
// has the model: its state (State, what stays in registers for the run; Acts, what a chunk's forward pass leaves for
// its backward pass), forward(), outputs(), backward(), update(), record(), penalty_sum(), load(), keep_best(),
// restore_best(), zero_grad() and total() (a sum over the block of what outputs() accumulates per thread).
//   KT        16-wide k tiles of the input layer
//   W         waves
//   BARRIERS  1: a chunk has one barrier, between forward() and outputs(); its inputs were put into LDS before the
//             barrier of the chunk before, so three input tiles rotate.  2: one more between outputs() and
//             backward(), and two input tiles are enough.  3: forward() begins with a barrier of its own, the chunk ends
//             with one, and the next chunk's inputs take the place of the last one's: one input tile.
//   PLANES    the inputs lie in LDS as three bfloat16 planes, [plane][row][block of 32 columns], a block in the order in which
//             a lane reads eight elements at a time: column 16 t + 4q + e of the block's tile t at 8q + 4t + e
template <class Self, class Lay, int KT, int W, int BARRIERS, bool PLANES>
struct RowPipe {
  static constexpr int K0 = 16 * KT, LDW = sm_ldw(KT), LDB = sm_ldb(KT), NB = 4 - BARRIERS, PC = PLANES ? 2 : 1;
  static constexpr int KL = K0 / PC;  // lanes per row when inputs are fetched, PC columns each
  static constexpr int KS = KL <= 16 ? 16 : (KL <= 32 ? 32 : (KL <= 64 ? 64 : 128));
  static constexpr int NTHR = 64 * W, RSTEP = NTHR / KS, NP = SM_RC / RSTEP, NX = NP * PC;  // rows per pass, passes, values
  static constexpr uint32_t TILE = sm_tile_bytes(KT, PLANES), PLANE = SM_RC * LDB * 2;
  typedef const __attribute__((address_space(4))) Lay ConstLay;
  const TrainParams& P;
  const ConstItemDesc& it;
  ConstLay& y;
  char* lds;
  float* slot;
  double* red;
  double* trace_stash;  // thread 0's own
  int fl;               // which row list
  // What every chunk needs of the item and the call, held in scalar registers: left to itself the compiler reloads
  // each field where it is used, a few hundred cycles every time.
  const GlobalF32* X = nullptr;
  const GlobalI32* Y = nullptr;
  int d = 0, n_fit = 0, n_classes = 0, o_sl = 0, o_ep = 0, tabled = 0;

  __device__ __forceinline__ RowPipe(const TrainParams& P_, const ConstItemDesc& it_, ConstLay& y_, char* lds_, float* slot_,
                                     double* red_, double* stash_, int fl_)
      : P(P_), it(it_), y(y_), lds(lds_), slot(slot_), red(red_), trace_stash(stash_), fl(fl_) {}

  // offsets in floats; what the model keeps in LDS starts at O_OWN
  static constexpr int O_YS = NB * (int)(TILE / 4), O_ROWS = O_YS + NB * SM_RC, O_OWN = O_ROWS + 2 * SM_RC;
  static_assert(O_OWN * 4 == pipe_lds(KT, NB, PLANES), "LDS layout");
  __device__ __forceinline__ float* f(int off) const { return (float*)lds + off; }
  __device__ __forceinline__ float* xs(int b) const { return f(b * (int)(TILE / 4)); }
  __device__ __forceinline__ const char* planes(int b) const { return lds + b * TILE; }
  // Operands of a row tile's block of 32 columns: lane (row li, eight columns of the lane's q) ...
  __device__ __forceinline__ static SmPlanes by_row(const char* x, int r, int kb) {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    const char* a = x + ((r * 16 + li) * LDB + kb * 32 + 8 * q) * 2;
    return SmPlanes{*(const u32x4*)a, *(const u32x4*)(a + PLANE), *(const u32x4*)(a + 2 * PLANE)};
  }
  // ... and of two row tiles r, r + 1 (without `both` zeros in place of the second) of a tile of 16 columns turned over:
  // lane (column li, rows 4q..+3 of each)
  template <bool BOTH>
  __device__ __forceinline__ static SmPlanes by_column(const char* x, int r, int kk) {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    const char* a = x + ((r * 16 + 4 * q + (li >> 2)) * LDB + (kk >> 1) * 32 + 8 * (li & 3) + 4 * (kk & 1)) * 2;
    u32x4 p[3];
#pragma unroll
    for (int i = 0; i < 3; i++) {
      const u32x2 lo = sm_read_tr(a + i * PLANE);
      u32x2 hi = u32x2{0u, 0u};
      if (BOTH) hi = sm_read_tr(a + i * PLANE + 16 * LDB * 2);
      p[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
    return SmPlanes{p[0], p[1], p[2]};
  }
  __device__ __forceinline__ float* ys(int b) const { return f(O_YS + b * SM_RC); }
  __device__ __forceinline__ int32_t* rowlist(int par) const { return (int32_t*)lds + O_ROWS + par * SM_RC; }
  __device__ __forceinline__ uint16_t* u16(uint32_t off) const { return (uint16_t*)(lds + off); }
  // The thread index as a value the compiler cannot see through: lane coordinates and the addresses derived
  // from them are recomputed in each phase instead of being kept in registers for the whole run.
  __device__ __forceinline__ static int tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  }
  __device__ __forceinline__ static int wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
  __device__ __forceinline__ float init_value(int l, int e, bool isb) const {
    const uint64_t kt = key_fold(key_model(it.seed, fl + P.fold_base), 16 + 2 * l + (isb ? 1 : 0));
    const uint32_t k24 = (uint32_t)(key_fold(kt, (uint64_t)e) >> 40);
    return it.bound[l] * ((float)((int32_t)k24 - 8388608) * 0x1p-23f);
  }

  // The epoch's rows in visiting order -> ep.  The permutation network's round function sees the round and one half
  // of the position only, so its 4 x 2^hb values are tabled first: a network evaluation is four LDS reads instead of twelve
  // 64-bit multiplies.  Small data sets table the whole network from it, so that the walk back into the list is one read
  // per hop; a lane whose position has landed starts its next one, and several positions of a lane walk side by side,
  // because each hop waits for LDS.
  __device__ __forceinline__ void build_epoch(uint64_t ke) const {
    const int t_ = tid();
    uint16_t* ep = u16(o_ep);
    const uint16_t* sl = u16(o_sl);
    if (n_fit <= 1) {
      __syncthreads();
      if (t_ < SM_RC) ep[t_] = sl[0];
      return;
    }
    const PermDomain dm = perm_domain((uint32_t)n_fit);
    const int half = 1 << dm.hb;
    uint16_t* ft = u16(y.p.o_ft);
    for (int i = t_; i < 4 * half; i += NTHR)
      ft[i] = (uint16_t)((uint32_t)key_fold(ke, ((uint64_t)(i >> dm.hb) << 32) | ((uint32_t)i & dm.mask)) & dm.mask);
    __syncthreads();  // nobody reads the last epoch's order, or the network, any more
    if (t_ < SM_RC) ep[n_fit + t_] = sl[0];  // the spare entries
    auto network = [&](uint32_t x) {
      uint32_t Lh = x >> dm.hb, Rh = x & dm.mask;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const uint32_t t = Lh ^ ft[(r << dm.hb) + Rh];
        Lh = Rh;
        Rh = t;
      }
      return (Lh << dm.hb) | Rh;
    };
    if (y.p.netted) {
      int p = t_;
      uint16_t* net = u16(y.p.o_net);
      for (int x = t_; x < half * half; x += 4 * NTHR) {  // four evaluations in flight
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; u++) v[u] = network((uint32_t)(x + u * NTHR) & (uint32_t)(half * half - 1));
#pragma unroll
        for (int u = 0; u < 4; u++)
          if (x + u * NTHR < half * half) net[x + u * NTHR] = (uint16_t)v[u];
      }
      __syncthreads();
      // two positions of a lane walk side by side
      for (; p < n_fit; p += 2 * NTHR) {
        const int p2 = p + NTHR < n_fit ? p + NTHR : p;
        uint32_t x = net[p], z = net[p2];
        while (x >= (uint32_t)n_fit || z >= (uint32_t)n_fit) {
          const uint32_t nx = net[x], nz = net[z];
          x = x >= (uint32_t)n_fit ? nx : x;
          z = z >= (uint32_t)n_fit ? nz : z;
        }
        const uint16_t rx = sl[x], rz = sl[z];
        ep[p] = rx;
        ep[p2] = rz;
      }
    } else {
      constexpr int U = 4;
      int pos[U];
      uint32_t x[U];
#pragma unroll
      for (int u = 0; u < U; u++) {
        pos[u] = t_ + u * NTHR;
        x[u] = (uint32_t)pos[u];
      }
      // (n_fit > SM_NET / 2: every lane has several positions, and the first of them is the last to run out)
      while (pos[0] < n_fit || pos[1] < n_fit || pos[2] < n_fit || pos[3] < n_fit) {
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = network(pos[u] < n_fit ? x[u] : 0u);
#pragma unroll
        for (int u = 0; u < U; u++)
          if (pos[u] < n_fit && x[u] < (uint32_t)n_fit) {
            ep[pos[u]] = sl[x[u]];
            pos[u] += U * NTHR;
            x[u] = (uint32_t)pos[u];
          }
      }
    }
  }
  // What only the rare paths need is derived there, from pointers the compiler cannot see through: kept for the whole
  // run it would crowd the scalar registers.
  struct Lists {
    const int32_t *tr, *va;
    RowSplit sp;
    uint64_t km;
  };
  __device__ __forceinline__ static const ConstParams& params() { return *launder((const ConstParams*)__builtin_amdgcn_kernarg_segment_ptr()); }
  __device__ __forceinline__ const ConstItemDesc& item() const { return *launder(&it); }
  __device__ __forceinline__ Lists lists() const {
    const ConstParams& p = params();
    const ConstItemDesc& i = item();
    Lists l;
    l.tr = p.train_idx + (int64_t)fl * p.n;
    l.va = p.val_idx + (int64_t)fl * p.n;
    l.km = key_model(i.seed, fl + p.fold_base);
    l.sp = row_split(l.km, i.patience, i.val_frac, uniform(p.counts[2 * fl]));
    return l;
  }
  // Row ids of a chunk that is not tabled, into rowlist(par) by the first 64 threads.
  __device__ __forceinline__ void park_rows(int chunk, int at, int e, int par) const {
    const int r = threadIdx.x;
    const Lists l = lists();
    if (r >= SM_RC) return;
    const int p = at + min(r, (chunk & SC_ROWS) - 1);  // past the chunk's rows: its last one again
    rowlist(par)[r] = chunk & SC_PLAIN ? l.va[p]
                                       : l.tr[row_index(l.sp, chunk & SC_HELD ? ROWS_HELD : ROWS_EPOCH, key_epoch(l.km, e), (uint32_t)p)];
  }
  // The chunk's input values (and label) requested into registers; `at`: its first row's position in the epoch's
  // order, or in the list being scored.  Past the chunk's last row the entries that follow in the list are fetched
  // (rows the model trains on, or any when it only scores): nothing masks rows, because a row that is not the chunk's
  // has no loss and a zero delta.  Columns past the inputs stay zero in the registers.
  __device__ __forceinline__ void fetch(int chunk, int at, int par, float (&xr)[NX], float& yv) const {
    const int t_ = tid(), k = t_ % KS * PC, r0 = t_ / KS;
    uint32_t row[NP], yrow;
    if (!(chunk & SC_PARK)) {
      const uint16_t* t16 = (chunk & SC_TRAIN ? u16(o_ep) : u16(o_sl) + n_fit) + at;
#pragma unroll
      for (int i = 0; i < NP; i++) row[i] = t16[r0 + i * RSTEP];
      yrow = t16[t_ & 63];
    } else {
      const int32_t* t32 = rowlist(par);
#pragma unroll
      for (int i = 0; i < NP; i++) row[i] = (uint32_t)t32[r0 + i * RSTEP];
      yrow = (uint32_t)t32[t_ & 63];
    }
    // 32-bit byte offsets: the host sends matrices of 4 GiB and more elsewhere
    if (k < d) {
#pragma unroll
      for (int i = 0; i < NP; i++) xr[i * PC] = *(const GlobalF32*)((const GlobalChar*)X + (row[i] * (uint32_t)d + (uint32_t)k) * 4u);
    }
    if (PLANES && k + 1 < d) {
#pragma unroll
      for (int i = 0; i < NP; i++)
        xr[i * PC + PC - 1] = *(const GlobalF32*)((const GlobalChar*)X + (row[i] * (uint32_t)d + (uint32_t)k) * 4u + 4u);
    }
    yv = __int_as_float(*(const GlobalI32*)((const GlobalChar*)Y + yrow * 4u));  // class id or target: 32 bits either way
  }
  // registers -> input tile and labels of buffer b (columns past the inputs: fetch() leaves zeros in them)
  __device__ __forceinline__ void commit(int b, const float (&xr)[NX], float yv) const {
    const int t_ = tid(), k = t_ % KS * PC, r0 = t_ / KS;
    if (KS == KL || k < K0) {
      if constexpr (PLANES) {
        char* s = lds + b * TILE + (r0 * LDB + (k >> 5) * 32 + ((k >> 2) & 3) * 8 + ((k >> 4) & 1) * 4 + (k & 3)) * 2;
#pragma unroll
        for (int i = 0; i < NP; i++) {
          uint32_t h, m, l;
          sm_split2(xr[2 * i], xr[2 * i + 1], h, m, l);
          char* o = s + i * RSTEP * LDB * 2;
          *(uint32_t*)o = h;
          *(uint32_t*)(o + PLANE) = m;
          *(uint32_t*)(o + 2 * PLANE) = l;
        }
      } else {
        float* s = xs(b);
#pragma unroll
        for (int i = 0; i < NX; i++) s[(r0 + i * RSTEP) * LDW + k] = xr[i];
      }
    }
    if (t_ < SM_RC) ys(b)[t_] = yv;
  }
  // Zeros into the input tiles (an absent tile's half of a block is never written) and into the row list's spare entries.
  __device__ __forceinline__ void clear_tiles(int n_tr) const {
    for (int i = threadIdx.x; i < NB * (int)(TILE / 4); i += NTHR) f(0)[i] = 0.f;
    if (tabled && threadIdx.x < SM_RC) u16(o_sl)[n_tr + threadIdx.x] = 0;
  }

  // Traced gradients of `steps` steps as the caller wants them (see AdamUnits).
  __device__ __forceinline__ void out_of_units(int64_t steps) const {
    const float unit = AdamUnits(item().beta1, item().beta2, item().eps).grad;
    float* rec = params().trace_out + 1;
    __syncthreads();
#pragma unroll 1
    for (; steps > 0; steps--, rec += 1 + 2 * (int64_t)y.p.P) {
#pragma unroll 1
      for (int k = tid(); k < y.p.P; k += NTHR) rec[k] /= unit;
    }
  }

  __device__ __forceinline__ void run() {
    Self& self = *static_cast<Self*>(this);
    const int n_tr = uniform(P.counts[2 * fl]), n_va = uniform(P.counts[2 * fl + 1]);
    const RowSplit sp = row_split(key_model(it.seed, fl + P.fold_base), it.patience, it.val_frac, n_tr);
    X = pin((const GlobalF32*)P.X);
    Y = pin((const GlobalI32*)P.y);
    d = pin(y.p.d);
    n_fit = pin(uniform(sp.n_fit));
    n_classes = pin(P.n_classes);
    o_sl = pin((int)y.p.o_sl);
    o_ep = pin((int)y.p.o_ep);
    tabled = pin(y.p.tabled);
    self.pin_own();
    const int bs = pin(uniform(eff_batch(it.batch_size, n_fit)));
    const int steps = pin(uniform(n_fit > 0 ? (n_fit + bs - 1) / bs : 0));
    const int epochs = pin(it.epochs);
    const int traced = pin(uniform(P.trace_item == it.b * P.n_folds + fl ? 1 : 0));
    const bool resume = traced && P.state_in && steps > 0;
    const bool watch = it.patience > 0 && steps > 0 && !resume;
    const int n_hold = pin(uniform(watch ? sp.n_hold : 0));
    const float mb_last = (float)(n_fit - (steps - 1) * bs);
    const float unit = it.solver == BBO_ADAM ? AdamUnits(it.beta1, it.beta2, it.eps).grad : 1.f;  // of the gradients
    const float inv_full = uniform(unit / (float)bs), inv_last = uniform(unit / mb_last);
    const float am_full = uniform(unit * (it.alpha / (float)bs)), am_last = uniform(unit * (it.alpha / mb_last));

    // ---- the schedule: training chunks, after each epoch the rows set aside, at the end the held fold ----
    // Position of the chunk whose inputs are requested next: first row `at` in its order, step st of epoch e, `left`
    // rows of that step from this chunk on.
    const int last_rows = pin(uniform(n_fit - (steps - 1) * bs)), decide = pin(uniform(watch && !n_hold ? (int)SC_DECIDE : 0));
    const int train_loss = traced | decide;  // somebody reads the loss of training chunks
    const int untabled = tabled ? 0 : (int)SC_PARK;
    int e = 0, at = 0, left = 0;
    int step_flags = 0;  // SC_RAGGED and SC_EPOCH of the step at this position
    int opened = 0;      // an epoch's rows have been asked for
    auto training = [&](int flags) {  // the chunk at this position
      return min(SM_RC, left) | SC_TRAIN | flags | step_flags |
             (left <= SM_RC ? SC_LAST | (step_flags & SC_RAGGED ? decide : 0) : 0) | untabled;
    };
    auto list_chunk = [&](int what, int count) {
      int ch = what | min(SM_RC, count - at);
      if (at == 0) ch |= SC_FIRST;
      if (what & SC_HELD) {
        ch |= untabled;
        if (count - at <= SM_RC) ch |= SC_DECIDE;
      } else {
        ch |= SC_PARK;
      }
      return ch;
    };
    auto score_start = [&]() -> int {
      at = 0;
      return n_va > 0 ? list_chunk(SC_PLAIN, n_va) : (int)SC_END;
    };
    auto epoch_start = [&](int st) -> int {  // at step st of epoch e
      if (steps == 0 || e >= epochs) return score_start();
      at = st * bs;
      left = st + 1 == steps ? last_rows : bs;
      step_flags = (st == 0 ? SC_EPOCH : 0) | (st + 1 == steps ? SC_RAGGED : 0);
      // (an epoch of one step takes all rows at once: their order says nothing, and the first epoch's serves all)
      const int table = !untabled && (steps > 1 || !opened) ? (int)SC_TABLE : 0;
      opened = 1;
      return training(SC_FIRST | SC_SLOW | table);
    };
    auto next = [&](int ch) -> int {
      at += ch & SC_ROWS;
      if (ch & SC_TRAIN) {
        left -= ch & SC_ROWS;
        if (left > 0) return training(0);
        if (at < n_fit) {  // the epoch goes on
          left = min(bs, n_fit - at);
          step_flags = at + left == n_fit ? SC_RAGGED : 0;
          return training(SC_FIRST | (traced | step_flags ? (int)SC_SLOW : 0));
        }
        if (n_hold) {
          at = 0;
          return list_chunk(SC_HELD, n_hold);
        }
        e++;
        return epoch_start(0);
      }
      if (ch & SC_HELD) {
        if (at < n_hold) return list_chunk(SC_HELD, n_hold);
        e++;
        return epoch_start(0);
      }
      return ch & SC_PLAIN && at < n_va ? list_chunk(SC_PLAIN, n_va) : (int)SC_END;
    };

    typename Self::State R;
    int64_t gstep = 0;
    int st0 = 0;
    if (resume) {
      gstep = P.step_begin;
      e = (int)(gstep / steps);
      st0 = (int)(gstep % steps);
    }
    int e_lr = st0 > 0 ? e : e - 1;  // epoch of the step being worked on (set when one opens)
    int c2 = epoch_start(st0);       // the chunk at the position above
    if constexpr (Self::LOAD_AHEAD) {
      if (resume) {
        const AdamUnits units(it.beta1, it.beta2, it.eps);
        self.load(R, P.state_in, it.solver == BBO_ADAM ? units.m : 1.f, it.solver == BBO_ADAM ? units.v : 1.f);
      } else {
        self.load(R, nullptr, 1.f, 1.f);
      }
    }
    OptC oc;
    const int solver = pin(it.solver);
    oc.adam = solver == BBO_ADAM;
    if constexpr (!Self::LOAD_AHEAD)
      self.load(R, resume ? P.state_in : nullptr, oc.adam ? AdamUnits(it.beta1, it.beta2, it.eps).m : 1.f,
                oc.adam ? AdamUnits(it.beta1, it.beta2, it.eps).v : 1.f);
    oc.nest = it.nesterov != 0;
    oc.b1 = pin(it.beta1);
    oc.b2 = pin(it.beta2);
    oc.omb1 = oc.omb2 = 0.f;  // (not in these units)
    oc.eps = uniform(AdamUnits(it.beta1, it.beta2, it.eps).eps);
    oc.mu = pin(it.momentum);
    oc.lr = it.lr;
    oc.lr_t = it.lr;
    oc.am = 0.f;
    float lr_tab = 0.f;  // Adam: the step sizes of 64 steps, one per lane
    int lr_at = 64;      // ... the next of them

    clear_tiles(n_tr);
    if (tabled) {  // rows of the training list in the order of the early-stopping cut
      uint16_t* sl = u16(o_sl);
      const int32_t* tr = P.train_idx + (int64_t)fl * P.n;
      for (int p = threadIdx.x; p < n_tr; p += blockDim.x)
        sl[p] = (uint16_t)tr[sp.n_hold ? (int)perm_index(sp.ksplit, (uint32_t)n_tr, (uint32_t)p) : p];
    }
    __syncthreads();
    float xr[NX], yv = 0.f;
#pragma unroll
    for (int i = 0; i < NX; i++) xr[i] = 0.f;
    int b = 0, par = 0;  // input buffer and exchange parity of the current chunk
    int c0 = 0, c1 = 0;  // the chunk being worked on; the one whose inputs are on their way in registers
    double lsum = 0.0, hits = 0.0;  // the lane's share of the summed data loss: of the epoch, or of a scoring pass
    Plateau plateau;
    int recording = 0, have_best = 0;
    float inv_mb = inv_full;
    if (!oc.adam) oc.lr = uniform(epoch_lr(it.lr, it.power_t, e_lr, n_fit));
    for (int phase = 0; phase < 2; phase++) {  // training with its stopping rule; the score
      if (phase == 1 && have_best) self.restore_best(R);  // the best epoch's model is the one scored
      const int stop_at = phase == 0 ? SC_PLAIN | SC_END : (int)SC_END;
      while (!(c0 & stop_at)) {
        const int bn = b == NB - 1 ? 0 : b + 1, rows = c0 & SC_ROWS, nrt = (rows + 15) / 16;
        if (BARRIERS == 1 && (c1 & SC_LIVE)) commit(bn, xr, yv);
        // the rows of the chunk whose inputs are requested next: its epoch's table if it opens one, or a row list
        if (c2 & (SC_PARK | SC_TABLE)) {
          if (c2 & SC_PARK)
            park_rows(c2, at, e, par);
          else
            build_epoch(key_epoch(key_model(item().seed, fl + params().fold_base), steps > 1 ? e : 0));
        }
        if (c0 & SC_FIRST) {
          if (c0 & SC_TRAIN) {  // first chunk of a step
            if (c0 & SC_SLOW) {
              const bool last = c0 & SC_RAGGED;
              oc.am = last ? am_last : am_full;
              inv_mb = last ? inv_last : inv_full;
              if (c0 & SC_EPOCH) {
                e_lr++;
                lsum = 0.0;
                if (!oc.adam) oc.lr = uniform(epoch_lr(item().lr, item().power_t, e_lr, n_fit));
              }
              if (SM_RARE(traced)) {
                recording = gstep >= params().step_begin && gstep < params().step_end ? 1 : 0;
                if (SM_RARE(recording)) {
                  const double pen = self.penalty_sum(R);
                  // the step's loss is the difference this step makes to the epoch's sum; both wait in LDS
                  const double before = self.total(lsum);
                  if (threadIdx.x == 0) {
                    trace_stash[0] = pen;
                    trace_stash[1] = before;
                  }
                }
              }
            }
            if (oc.adam) {
              if (SM_RARE(lr_at == 64)) {
                // beta^t of the next 64 steps, a step per lane, by repeated squaring in double
                lr_at = 0;
                double q1 = (double)item().beta1, q2 = (double)item().beta2, b1t = 1.0, b2t = 1.0;
#pragma unroll 1
                for (uint64_t t = (uint64_t)(gstep + 1) + (threadIdx.x & 63); __any(t != 0); t >>= 1) {
                  b1t *= t & 1 ? q1 : 1.0;
                  b2t *= t & 1 ? q2 : 1.0;
                  q1 *= q1;
                  q2 *= q2;
                }
                const double rest = AdamUnits(item().beta1, item().beta2, item().eps).lr;
                lr_tab = (float)((double)item().lr * sqrt(1.0 - b2t) / (1.0 - b1t) * rest);
              }
              oc.lr_t = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lr_tab), lr_at));
              lr_at++;
            }
            self.zero_grad(R);
          } else {
            lsum = hits = 0.0;
          }
        }
        typename Self::Acts acc;
        const bool live = c0 & SC_LIVE;
        if (live) self.forward(R, b, par, nrt, acc);
        __syncthreads();  // the outputs' shares, the next chunk's inputs and the rows of the one after it
        if (BARRIERS == 2 && (c1 & SC_LIVE)) commit(bn, xr, yv);
        if (BARRIERS < 3 && (c2 & SC_LIVE)) fetch(c2, at, par, xr, yv);  // in flight until the next chunk is under way
        if (live) {
          const bool train = c0 & SC_TRAIN;
          self.outputs(R, b, par, rows, train, !train || train_loss, inv_mb, lsum, hits);
        }
        if (BARRIERS >= 2) __syncthreads();  // the output deltas
        if (c0 & SC_TRAIN) {
          self.backward(R, b, nrt, acc);
          if (c0 & SC_LAST) {  // last chunk of the step
            float* rec = nullptr;
            if (SM_RARE(recording)) {
              rec = params().trace_out + (gstep - params().step_begin) * (1 + 2 * (int64_t)y.p.P);
              self.template record<true>(R, oc.am, rec + 1);
            }
            if (oc.adam)
              self.template update<true>(R, oc);
            else
              self.template update<false>(R, oc);
            if (SM_RARE(recording)) {
              self.template record<false>(R, oc.am, rec + 1 + y.p.P);
              const double after = self.total(lsum);
              const float mb = c0 & SC_RAGGED ? (float)last_rows : (float)bs;
              if (threadIdx.x == 0)
                rec[0] = (float)((after - trace_stash[1] + 0.5 * (double)item().alpha * trace_stash[0]) / (double)mb);
            }
            gstep++;
          }
        }
        if (BARRIERS == 3) {
          __syncthreads();  // the chunk's inputs have been read for the last time
          if (c1 & SC_LIVE) commit(bn, xr, yv);
          if (c2 & SC_LIVE) fetch(c2, at, par, xr, yv);
        }
        const int done = c0;
        c0 = c1;
        c1 = c2;
        c2 = next(c2);
        b = bn;
        par ^= 1;
        // the end of an epoch (with the rows set aside, if any): the stopping rule, decided alike in every wave
        if (SM_RARE(done & SC_DECIDE)) {
          const float watched = (float)(self.total(lsum) / (double)(n_hold ? n_hold : n_fit));
          const int stop = uniform(plateau.stop_after(watched, item().tol, item().patience) ? 1 : 0);
          if (n_hold && uniform(plateau.improved ? 1 : 0)) {
            self.keep_best(R);
            have_best = 1;
          }
          if (stop && (c0 & SC_TRAIN)) {  // what is already on its way is dropped, and the pipeline starts over
            __syncthreads();
            c2 = score_start();
            c0 = c1 = 0;
          }
        }
      }
    }
    if (SM_RARE(traced && oc.adam)) out_of_units(min(gstep, params().step_end) - params().step_begin);
    lsum = self.total(lsum);
    hits = self.total(hits);
    if (threadIdx.x == 0) {
      float* out = P.item_out + 2 * ((int64_t)it.b * P.n_folds + fl);
      out[0] = n_va > 0 ? (float)(lsum / (double)n_va) : __builtin_nanf("");
      out[1] = n_va > 0 ? (float)(hits / (double)n_va) : __builtin_nanf("");  // accuracy | mean absolute error
    }
  }
};

// The weights of a wave's hidden units: lane (unit li, columns 16 kk + 4q + e), as floats or as the three planes of two
// tiles of columns, which hold the same numbers.
template <int KT, int NT, bool SPLIT>
struct HiddenWeights {
  f32x4 w[NT][KT];
  __device__ __forceinline__ f32x4 get(int i, int kk) const { return w[i][kk]; }
  __device__ __forceinline__ void put(int i, int kk, const f32x4& x) { w[i][kk] = x; }
};
template <int KT, int NT>
struct HiddenWeights<KT, NT, true> {
  SmPlanes p[sm_blocks(KT)][NT];
  static constexpr bool MASTER = KT * NT <= 4;
  f32x4 w[MASTER ? NT : 1][MASTER ? KT : 1];
  __device__ __forceinline__ f32x4 get(int i, int kk) const {
    if constexpr (MASTER) return w[i][kk];
    const SmPlanes& s = p[kk >> 1][i];
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 2; e++) {
      const int j = 2 * (kk & 1) + e;
      x[2 * e] = (sm_low(s.h[j]) + sm_low(s.m[j])) + sm_low(s.l[j]);
      x[2 * e + 1] = (sm_high(s.h[j]) + sm_high(s.m[j])) + sm_high(s.l[j]);
    }
    return x;
  }
  __device__ __forceinline__ void put(int i, int kk, const f32x4& x) {
    if constexpr (MASTER) w[i][kk] = x;
    SmPlanes& s = p[kk >> 1][i];
#pragma unroll
    for (int e = 0; e < 2; e++) {
      uint32_t h, m, l;
      sm_split2(x[2 * e], x[2 * e + 1], h, m, l);
      s.h[2 * (kk & 1) + e] = h;
      s.m[2 * (kk & 1) + e] = m;
      s.l[2 * (kk & 1) + e] = l;
    }
    if (KT % 2 && kk == KT - 1) s.h[2] = s.h[3] = s.m[2] = s.m[3] = s.l[2] = s.l[3] = 0u;
  }
};

// KT: 16-wide k tiles of the input layer.  NT: unit tiles per wave (every wave has NT, or NT - 1, of them).
// CO: output slots in use (1 and 2 are exact output counts, 4 serves 3 or 4 outputs).  W: waves.
template <int KT, int NT, int CO, int W>
struct Small : RowPipe<Small<KT, NT, CO, W>, SLay, KT, W, sm_barriers(KT, NT, CO), sm_split(KT, NT, CO)> {
  typedef RowPipe<Small<KT, NT, CO, W>, SLay, KT, W, sm_barriers(KT, NT, CO), sm_split(KT, NT, CO)> Base;
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
  int nut = 0;
  __device__ __forceinline__ void pin_own() { nut = pin(y.nut); }
  __device__ __forceinline__ static double total(double v) { return sm_wavesum_d(v); }  // every wave has the whole sum

  // Output columns the products run over: two classes are one, the difference z[1] - z[0], on which their softmax, loss
  // and deltas (p and -p) depend alone.
  static constexpr int ZO = sm_columns(CO);
  // The small parameters: the bias and the row of the output layer of each tile's unit li, then the output bias.  The
  // optimizer works on four at a time: parameter k in the lanes of row q = k % 4, group k / 4.
  static constexpr int NSMALL = NT * (1 + CO) + CO, NG = (NSMALL + 3) / 4;
  static constexpr bool SPLIT = sm_split(KT, NT, CO);
  static constexpr int KB = sm_blocks(KT);
  // One output column: a unit's hidden deltas are its output weight times the rows' deltas where it is active, and the
  // weight is the same for a whole step.  So the step's sums leave it out, and its gradients take it in at the end: with split
  // products the deltas are then split once a row and not once a row and unit.  2000 models 569 x 30, us a call before and
  // after: 128 units, 24 and 128 rows a step 2026 and 1959, 1057 and 1003; 190 units 3764 and 3145, 1656 and 1388.  fp32 products
  // save a multiplication of each value for one of each parameter and step: 2 % at 45 inputs, a loss at 13.
  static constexpr bool FACTORED = sm_factored(KT, NT, CO);
  // With one input tile the model is loaded ahead of the optimizer's constants, and its moments' units are made only where there
  // are moments.  40 models 506 x 13 of 50 units, 24 and 64 rows a step: SGD 1049 -> 1024 and 608 -> 593 us a call, Adam 1093 -> 1067
  // and 627 -> 608; 1000 models at 64 rows 490 -> 481 and 496 -> 481.  Wider inputs keep their registers the other way round
  // (<2,3,1,4> spills 102 against 128).
  static constexpr bool LOAD_AHEAD = KT == 1;
  // us a call without and with, 24 rows a step: 40 models 569 x 60, four classes, 180 units 5686 and 5477, 569 x 45, 100 units 3375 and 3197;
  // but three unit tiles a wave, 569 x 30, two classes, 180 units 2538 and 2837, by five more registers spilled.
  static constexpr bool RARE_APART = NT < 3;
  struct State {
    HiddenWeights<KT, NT, SPLIT> w;
    f32x4 m[NT][KT], v[NT][KT], g[NT][KT];  // hidden layer: lane (unit li, columns 16 kk + 4q + e)
    float pw[NG], pm[NG], pv[NG];                      // the small parameters and their moments
    float bw[NT], w2[NT][ZO], ow[ZO];                  // the same as the products want them: alike in the four q
    float bg[NT], g2[NT][ZO], og[ZO];                  // the lane's share of their gradients
    __device__ __forceinline__ float factor(int i) const { return FACTORED ? w2[i][0] : 1.f; }  // (of g and bg)
  };

  struct Acts {
    f32x4 a[NT][4];  // activations of the wave's tiles: lane (unit li, rows 16 r + 4q..+3)
  };
  // offsets in floats
  static constexpr int O_ZP = Base::O_OWN, O_D2 = O_ZP + 2 * W * ZO * SM_RC, O_DP = O_D2 + ZO * SM_RC,
                       O_TOP = O_DP + (int)sm_delta_planes(KT, NT, CO) / 4;
  static_assert(O_TOP * 4 == sm_fixed_lds(KT, NT, CO, W), "LDS layout");
  // does the wave's i-th tile exist?  Only the last one can be missing.
  __device__ __forceinline__ bool has(int i, int w) const { return i + 1 < NT || w + i * W < nut; }

  // ---- parameters ----------------------------------------------------------
  // The wave's share of the parameters as it lies in its part of the slot: [register][lane], the registers in the
  // order each_param() visits them.
  static constexpr int NREG = sm_regs(KT, NT, CO), PER = 4 * KT + 1 + CO;
  __device__ __forceinline__ float* park() const { return slot + wave() * (NREG * 64) + (threadIdx.x & 63); }
  // fn(index, reference) for the hidden weights or one of their moments
  template <class F>
  __device__ __forceinline__ static void each_hidden(f32x4 (&w)[NT][KT], F fn) {
#pragma unroll
    for (int i = 0; i < NT; i++)
#pragma unroll
      for (int kk = 0; kk < KT; kk++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float x = w[i][kk][e];
          fn(i * PER + 4 * kk + e, x);
          w[i][kk][e] = x;
        }
  }
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
  // small parameter k: of tile k / (1 + CO), 0 its bias, else an output; from NT (1 + CO) on the output bias
  __device__ __forceinline__ static int small_register(int k) {
    return k >= NT * (1 + CO) ? NT * PER + k - NT * (1 + CO) : k / (1 + CO) * PER + 4 * KT + k % (1 + CO);
  }
  __device__ __forceinline__ static constexpr bool small_weight(int k) { return k < NT * (1 + CO) && k % (1 + CO) != 0; }
  // fn(reference, place in the slot) for the lane's small parameters
  template <class F>
  __device__ __forceinline__ void each_small(float (&p)[NG], F fn) const {
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
    float* b = slot + wave() * (NREG * 64) + li;
#pragma unroll
    for (int g = 0; g < NG; g++) {
      p[g] = 4 * g + q < NSMALL ? p[g] : 0.f;
      if (4 * g + q < NSMALL) fn(p[g], b + 64 * small_register(4 * g + q));
    }
  }
  // pw -> bw, w2, ow
  __device__ __forceinline__ static void spread(State& R) {
    float x[4 * NG];
#pragma unroll
    for (int g = 0; g < NG; g++) {
      const uint32_t p = __float_as_uint(R.pw[g]);
      const auto h = __builtin_amdgcn_permlane32_swap(p, p, false, false);
      const uint32_t lo = h[0], hi = h[1];
      const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
      const uint32_t x0 = a[0], x1 = a[1], x2 = b[0], x3 = b[1];
      x[4 * g] = __uint_as_float(x0);
      x[4 * g + 1] = __uint_as_float(x1);
      x[4 * g + 2] = __uint_as_float(x2);
      x[4 * g + 3] = __uint_as_float(x3);
    }
#pragma unroll
    for (int i = 0; i < NT; i++) {
      const int o = i * (1 + CO);
      R.bw[i] = x[o];
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) R.w2[i][cc] = CO == 2 ? x[o + 2] - x[o + 1] : x[o + 1 + cc];
    }
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) R.ow[cc] = CO == 2 ? x[NT * (1 + CO) + 1] - x[NT * (1 + CO)] : x[NT * (1 + CO) + cc];
  }
  // the gradients of the lane's small parameters, summed over the wave
  __device__ __forceinline__ static void small_grads(const State& R, float (&gp)[NG]) {
    float x[4 * NG];
#pragma unroll
    for (int i = 0; i < NT; i++) {
      x[i * (1 + CO)] = R.bg[i] * R.factor(i);
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) {
        x[i * (1 + CO) + CO - ZO + 1 + cc] = R.g2[i][cc];
        if (CO == 2) x[i * (1 + CO) + 1] = -R.g2[i][cc];
      }
    }
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) {
      const float o = sm_row16sum(R.og[cc]);
      x[NT * (1 + CO) + CO - ZO + cc] = o;
      if (CO == 2) x[NT * (1 + CO)] = -o;
    }
#pragma unroll
    for (int k = NSMALL; k < 4 * NG; k++) x[k] = 0.f;
#pragma unroll
    for (int g = 0; g < NG; g++) gp[g] = sm_fold32(sm_fold16(x[4 * g], x[4 * g + 1]), sm_fold16(x[4 * g + 2], x[4 * g + 3]));
  }
  // the penalty's factor for the lane's parameter of group g: none on the biases
  __device__ __forceinline__ static float small_penalty(int g, int q, float am) {
    const int weights = (small_weight(4 * g) ? 1 : 0) | (small_weight(4 * g + 1) ? 2 : 0) | (small_weight(4 * g + 2) ? 4 : 0) |
                        (small_weight(4 * g + 3) ? 8 : 0);
    return (weights >> q) & 1 ? am : 0.f;
  }
  // Packed parameters (or one of their moments) `st`, or the initial draw where st is null, into the wave's part of
  // the slot.  A rolled loop: the registers are filled from the slot afterwards.
  __device__ __forceinline__ void unpack(const float* st, float unit = 1.f) const {
    const int lane = threadIdx.x & 63, w_ = wave(), li = lane & 15, q = lane >> 4;
    const int d = y.p.d, h = y.h, c = y.c;
    float* b = park();
#pragma unroll 1
    for (int n = 0; n < NREG; n++) {
      const int i = n / PER, r = n - i * PER, j = (w_ + i * W) * 16 + li;
      int l = 0, ci = -1, e = 0;
      bool isb = false;
      if (i == NT) {  // output bias
        l = 1;
        isb = true;
        e = n - NT * PER;
        if (e < c) ci = y.cb[1] + e;
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
        const int cc = r - 4 * KT - 1;
        e = j * c + cc;
        if (j < h && cc < c) ci = y.cw[1] + e;
      }
      float val = 0.f;
      if (ci >= 0) val = st ? st[ci] * unit : init_value(l, e, isb);
      b[64 * n] = val;
    }
  }
  __device__ __forceinline__ void load(State& R, const float* st, float um, float uv) const {
    const float* b = park();
    auto take = [&](int n, float& x) { x = b[64 * n]; };
    auto take_small = [](float& x, const float* at) { x = *at; };
    auto zero = [](int, float& x) { x = 0.f; };
    auto zero_small = [](float& x, const float*) { x = 0.f; };
    if (st) {
      unpack(st + y.p.P, um);
      each_hidden(R.m, take);
      each_small(R.pm, take_small);
      unpack(st + 2 * y.p.P, uv);
      each_hidden(R.v, take);
      each_small(R.pv, take_small);
    } else {
      each_hidden(R.m, zero);
      each_small(R.pm, zero_small);
      each_hidden(R.v, zero);
      each_small(R.pv, zero_small);
    }
    unpack(st);
    restore_best(R);
  }
  // Keep the current parameters aside / take the kept ones back: every wave its own, no barrier.
  __device__ __forceinline__ void keep_best(State& R) const {
    float* b = park();
    each_hidden(R.w, [&](int n, float& x) { b[64 * n] = x; });
    each_small(R.pw, [](float& x, float* at) { *at = x; });
  }
  __device__ __forceinline__ void restore_best(State& R) const {
    const float* b = park();
    each_hidden(R.w, [&](int n, float& x) { x = b[64 * n]; });
    each_small(R.pw, [](float& x, const float* at) { x = *at; });
    spread(R);
    // waited for here: the loop's own waits would otherwise have to allow for these loads, at the price of the input
    // values that are meant to stay in flight
    __builtin_amdgcn_s_waitcnt(0);
  }
  __device__ __forceinline__ static void zero_grad(State& R) {
#pragma unroll
    for (int i = 0; i < NT; i++) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++) R.g[i][kk] = f32x4{0.f, 0.f, 0.f, 0.f};
      R.bg[i] = 0.f;
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) R.g2[i][cc] = 0.f;
    }
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) R.og[cc] = 0.f;
  }

  // ---- rows and inputs ------------------------------------------------------
  // ---- hidden layer forward; the wave's share of the outputs -> zp ----------------
  // One row tile: products of all the wave's tiles in turn (independent accumulators), ReLU, output-layer share.
  // ALL: the wave's last tile exists.
  template <bool ALL>
  __device__ __forceinline__ void forward_tile(const State& R, int b, int r, f32x4 (&acc)[NT][4], float (&v)[ZO][4]) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    f32x4 c[NT];
#pragma unroll
    for (int i = 0; i < NT; i++) {
      // A vector made of the register straight away became a wide load of its neighbours before the compiler had given
      // them registers, and kept the small parameters and their gradients in scratch memory, where each wait is one for
      // the inputs in flight too.  2000 models 569 x 30, 128 units, 24 rows a step: 2372 us a call then, 1961 now.
      float x = R.bw[i];
      if (NT > 1 || KT > 1) asm("" : "+v"(x));
      c[i] = f32x4{x, x, x, x};
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int kb = 0; kb < KB; kb++) sm_products<NT - (ALL ? 0 : 1)>(Base::by_row(Base::planes(b), r, kb), R.w.p[kb], c);
    } else {
      const float* a_ = xs(b) + (r * 16 + li) * LDW + 4 * q;
      f32x4 a[KT];
#pragma unroll
      for (int kk = 0; kk < KT; kk++) a[kk] = *(const f32x4*)(a_ + kk * 16);
#pragma unroll
      for (int kk = 0; kk < KT; kk++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
#pragma unroll
          for (int i = 0; i < NT; i++)
            if (i + 1 < NT || ALL) c[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk][e], R.w.w[i][kk][e], c[i], 0, 0, 0);
        }
    }
    float p[ZO][4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
#pragma unroll
      for (int i = 0; i < NT; i++) {
        const float av = relu(c[i][e]);
        acc[i][r][e] = av;
#pragma unroll
        for (int cc = 0; cc < ZO; cc++) p[cc][e] = i == 0 ? av * R.w2[0][cc] : p[cc][e] + av * R.w2[i][cc];
      }
    }
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) v[cc][r] = sm_fold_quad(p[cc], li & 1, li & 2);
  }
  template <bool ALL, int N>
  __device__ __forceinline__ void forward_tiles(const State& R, int b, f32x4 (&acc)[NT][4], float (&v)[ZO][4]) const {
#pragma unroll
    for (int r = 0; r < 4; r++) {
      if (r < N) {
        forward_tile<ALL>(R, b, r, acc, v);
      } else {
#pragma unroll
        for (int cc = 0; cc < ZO; cc++) v[cc][r] = 0.f;
      }
    }
  }
  template <bool ALL>
  __device__ __forceinline__ void forward_chunk(const State& R, int b, int nrt, f32x4 (&acc)[NT][4], float (&v)[ZO][4]) const {
    if (nrt == 4)
      forward_tiles<ALL, 4>(R, b, acc, v);
    else if (nrt == 3)
      forward_tiles<ALL, 3>(R, b, acc, v);
    else if (nrt == 2)
      forward_tiles<ALL, 2>(R, b, acc, v);
    else
      forward_tiles<ALL, 1>(R, b, acc, v);
  }
  __device__ __forceinline__ void forward(const State& R, int b, int par, int nrt, Acts& A) const {
    f32x4 (&acc)[NT][4] = A.a;
    const int w_ = wave();
    float v[ZO][4];
    if (has(NT - 1, w_))
      forward_chunk<true>(R, b, nrt, acc, v);
    else
      forward_chunk<false>(R, b, nrt, acc, v);
    const int lane = tid() & 63, li = lane & 15;
    float* zp = f(O_ZP) + (par * W + w_) * (ZO * SM_RC) + lane;
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) zp[cc * SM_RC] = sm_fold_row(v[cc], li & 4, li & 8);
  }

  // ---- outputs, loss and output delta of the chunk's rows; the same in every wave ----
  // (train: the delta is wanted; loss: the loss is, and when scoring the hits)
  __device__ __forceinline__ void outputs(State& R, int b, int par, int rows, bool train, bool loss, float inv_mb, double& lsum, double& hits) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4, c = CO <= 2 ? CO : y.c;
    const int row = (li >> 2) * 16 + 4 * q + (li & 3);  // the row the folding tree left in this lane
    const float* zp = f(O_ZP) + par * W * (ZO * SM_RC) + lane;
    float z[ZO];
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) z[cc] = R.ow[cc];
#pragma unroll
    for (int ww = 0; ww < W; ww++) {
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) z[cc] += zp[(ww * ZO + cc) * SM_RC];
    }
    const float yv = ys(b)[row];
    float dl[ZO];
    sm_outputs<CO>(z, yv, row < rows, c, n_classes, train, loss, inv_mb, dl, lsum, hits);
    if (train) {
      float* d2 = f(O_D2) + lane;  // every wave writes the same values, and reads back only what it wrote itself
#pragma unroll
      for (int cc = 0; cc < ZO; cc++) {
        d2[cc * SM_RC] = dl[cc];
        R.og[cc] += dl[cc];
      }
      if constexpr (FACTORED && SPLIT) {
        uint16_t* dp = (uint16_t*)f(O_DP) + lane;
        uint32_t h, m, l;
        sm_split2(dl[0], 0.f, h, m, l);
        dp[0] = (uint16_t)h;
        dp[SM_RC] = (uint16_t)m;
        dp[2 * SM_RC] = (uint16_t)l;
      }
      __builtin_amdgcn_wave_barrier();
    }
  }

  // ---- backward: hidden deltas, output-layer gradient, hidden weight gradient -------
  // the hidden deltas of a row tile, and its shares of the small parameters' gradients
  template <bool ALL>
  __device__ __forceinline__ void deltas(State& R, int r, const f32x4 (&acc)[NT][4], f32x4 (&dh)[NT]) const {
    const float* d2 = f(O_D2) + ((tid() & 63) >> 4) * 16 + r * 4;
    f32x4 dv[ZO];
#pragma unroll
    for (int cc = 0; cc < ZO; cc++) dv[cc] = *(const f32x4*)(d2 + cc * SM_RC);
#pragma unroll
    for (int i = 0; i < NT; i++)
      if (i + 1 < NT || ALL) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float av = acc[i][r][e];
          float sum = FACTORED ? dv[0][e] : dv[0][e] * R.w2[i][0];
          R.g2[i][0] += av * dv[0][e];
#pragma unroll
          for (int cc = 1; cc < ZO; cc++) {
            sum += dv[cc][e] * R.w2[i][cc];
            R.g2[i][cc] += av * dv[cc][e];
          }
          const float x = av > 0.f ? sum : 0.f;
          dh[i][e] = x;
          R.bg[i] += x;
        }
      }
  }
  template <bool ALL>
  __device__ __forceinline__ void backward_tile(State& R, const float* s, int r, const f32x4 (&acc)[NT][4]) const {
    const int lane = tid() & 63, li = lane & 15, q = lane >> 4;
    const float* a_ = s + (r * 16 + 4 * q) * LDW + li;
    float a[KT][4];
#pragma unroll
    for (int kk = 0; kk < KT; kk++)
#pragma unroll
      for (int e = 0; e < 4; e++) a[kk][e] = a_[e * LDW + kk * 16];
    f32x4 dh[NT];
    deltas<ALL>(R, r, acc, dh);
#pragma unroll
    for (int kk = 0; kk < KT; kk++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
#pragma unroll
        for (int i = 0; i < NT; i++)
          if (i + 1 < NT || ALL) R.g[i][kk] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk][e], dh[i][e], R.g[i][kk], 0, 0, 0);
      }
  }
  // The hidden deltas of row tiles r and r + 1 (BOTH) as planes, and their shares of the small parameters' gradients.
  template <bool ALL, int TILES, bool BOTH>
  __device__ __forceinline__ void split_planes(State& R, int r, const f32x4 (&acc)[NT][4], SmPlanes (&dp)[TILES]) const {
#pragma unroll
    for (int t = 0; t < 2; t++) {
      f32x4 dh[NT];
      if (t == 0 || BOTH) deltas<ALL>(R, r + t, acc, dh);
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
  }
  // The same without the unit's output weight: the rows' deltas, which outputs() has split once for all units, masked by
  // the unit's activations.  Five vector instructions a value instead of eleven.
  template <int TILES, bool BOTH>
  __device__ __forceinline__ void masked_planes(State& R, int r, const f32x4 (&acc)[NT][4], SmPlanes (&dp)[TILES]) const {
    const int o = ((tid() & 63) >> 4) * 16 + r * 4;
    const uint16_t* s = (const uint16_t*)f(O_DP) + o;
    u32x4 row[3];
#pragma unroll
    for (int j = 0; j < 3; j++) {
      if (BOTH) {
        row[j] = *(const u32x4*)(s + j * SM_RC);
      } else {
        const u32x2 x = *(const u32x2*)(s + j * SM_RC);
        row[j] = u32x4{x[0], x[1], 0u, 0u};
      }
    }
#pragma unroll
    for (int t = 0; t < 2; t++) {
      f32x4 dv;
      if (t == 0 || BOTH) dv = *(const f32x4*)(f(O_D2) + o + 4 * t);
#pragma unroll
      for (int i = 0; i < TILES; i++)
#pragma unroll
        for (int e = 0; e < 2; e++) {
          uint32_t on = 0u;
          if (t == 0 || BOTH) {
            float a[2];
#pragma unroll
            for (int j = 0; j < 2; j++) {
              const float av = acc[i][r + t][2 * e + j], d = dv[2 * e + j];
              a[j] = sm_active(av);
              R.g2[i][0] = fmaf(av, d, R.g2[i][0]);
              R.bg[i] = fmaf(a[j], d, R.bg[i]);
            }
            on = sm_mask(a[0], a[1]);
          }
          dp[i].h[2 * t + e] = row[0][2 * t + e] & on;
          dp[i].m[2 * t + e] = row[1][2 * t + e] & on;
          dp[i].l[2 * t + e] = row[2][2 * t + e] & on;
        }
    }
  }
  // row tiles r and r + 1 (BOTH), which fill the 32 contracted rows of a product
  template <bool ALL, bool BOTH>
  __device__ __forceinline__ void backward_pair(State& R, const char* x, int r, const f32x4 (&acc)[NT][4]) const {
    constexpr int TILES = NT - (ALL ? 0 : 1);
    if constexpr (TILES > 0) {
      SmPlanes dp[TILES];
      if constexpr (FACTORED)
        masked_planes<TILES, BOTH>(R, r, acc, dp);
      else
        split_planes<ALL, TILES, BOTH>(R, r, acc, dp);
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        f32x4 c[TILES];
#pragma unroll
        for (int i = 0; i < TILES; i++) c[i] = R.g[i][kk];
        sm_products<TILES>(Base::template by_column<BOTH>(x, r, kk), dp, c);
#pragma unroll
        for (int i = 0; i < TILES; i++) R.g[i][kk] = c[i];
      }
    }
  }
  template <bool ALL, int N>
  __device__ __forceinline__ void backward_tiles(State& R, int b, const f32x4 (&acc)[NT][4]) const {
    if constexpr (SPLIT) {
#pragma unroll
      for (int r = 0; r + 1 < N; r += 2) backward_pair<ALL, true>(R, Base::planes(b), r, acc);
      if constexpr (N % 2) backward_pair<ALL, false>(R, Base::planes(b), N - 1, acc);
    } else {
#pragma unroll
      for (int r = 0; r < N; r++) backward_tile<ALL>(R, xs(b), r, acc);
    }
  }
  template <bool ALL>
  __device__ __forceinline__ void backward_chunk(State& R, int b, int nrt, const f32x4 (&acc)[NT][4]) const {
    if (nrt == 4)
      backward_tiles<ALL, 4>(R, b, acc);
    else if (nrt == 3)
      backward_tiles<ALL, 3>(R, b, acc);
    else if (nrt == 2)
      backward_tiles<ALL, 2>(R, b, acc);
    else
      backward_tiles<ALL, 1>(R, b, acc);
  }
  __device__ __forceinline__ void backward(State& R, int b, int nrt, const Acts& A) const {
    const f32x4 (&acc)[NT][4] = A.a;
    if (has(NT - 1, wave()))
      backward_chunk<true>(R, b, nrt, acc);
    else
      backward_chunk<false>(R, b, nrt, acc);
  }

  // ---- optimizer step -------------------------------------------------------------
  // Pad elements need no mask: their inputs, deltas and weights are zero, and so is their step (0 / eps).
  template <bool ADAM>
  __device__ __forceinline__ void update(State& R, const OptC& oc) const {
    const int w_ = wave();
    OptC o = oc;
    o.adam = ADAM;
#pragma unroll
    for (int i = 0; i < NT; i++)
      if (has(i, w_)) {
#pragma unroll
        for (int kk = 0; kk < KT; kk++) {
          f32x4 x = R.w.get(i, kk);
#pragma unroll
          for (int e = 0; e < 4; e++) {
            float wr = x[e], mr = R.m[i][kk][e], vr = R.v[i][kk][e];
            opt_step(o, fmaf(o.am, wr, R.g[i][kk][e] * R.factor(i)), wr, mr, vr);
            x[e] = wr;
            R.m[i][kk][e] = mr;
            R.v[i][kk][e] = vr;
          }
          R.w.put(i, kk, x);
        }
      }
    const int q = (tid() & 63) >> 4;
    float gp[NG];
    small_grads(R, gp);
#pragma unroll
    for (int g = 0; g < NG; g++) opt_step(o, gp[g] + small_penalty(g, q, o.am) * R.pw[g], R.pw[g], R.pm[g], R.pv[g]);
    spread(R);
  }
  // A traced step's gradient (before the update: GRAD) or new parameters into out[P].
  template <bool GRAD>
  __device__ __forceinline__ void record(const State& R, float am, float* out) const {
    const int t_ = tid(), lane = t_ & 63, w_ = wave(), li = lane & 15, q = lane >> 4;
    const int d = y.p.d, h = y.h;
#pragma unroll
    for (int i = 0; i < NT; i++) {
      const int j = (w_ + i * W) * 16 + li;
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        const f32x4 x = R.w.get(i, kk);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int k = kk * 16 + 4 * q + e;
          if (j < h && k < d) out[y.cw[0] + k * h + j] = GRAD ? fmaf(am, x[e], R.g[i][kk][e] * R.factor(i)) : x[e];
        }
      }
    }
    float gp[NG];
    if (GRAD) small_grads(R, gp);
#pragma unroll
    for (int g = 0; g < NG; g++) {
      const int ci = small_packed(4 * g + q);
      const float x = GRAD ? gp[g] + small_penalty(g, q, am) * R.pw[g] : R.pw[g];
      if (ci >= 0 && (4 * g + q < NT * (1 + CO) || t_ - 16 * q == 0)) out[ci] = x;  // (the output bias once)
    }
  }
  // where the lane's small parameter k stands in the packed parameters; -1: a pad
  __device__ __forceinline__ int small_packed(int k) const {
    const int j = (wave() + k / (1 + CO) * W) * 16 + (threadIdx.x & 15), r = k % (1 + CO), c = CO <= 2 ? CO : y.c;
    if (k >= NSMALL) return -1;
    if (k >= NT * (1 + CO)) return k - NT * (1 + CO) < c ? y.cb[1] + k - NT * (1 + CO) : -1;
    return j >= y.h || r > c ? -1 : (r == 0 ? y.cb[0] + j : y.cw[1] + j * c + r - 1);
  }
  // squared weights, for a traced step's loss
  __device__ __forceinline__ double penalty_sum(const State& R) const {
    const int q = (threadIdx.x & 63) >> 4;
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NT; i++) {
#pragma unroll
      for (int kk = 0; kk < KT; kk++) {
        const f32x4 x = R.w.get(i, kk);
#pragma unroll
        for (int e = 0; e < 4; e++) s += (double)x[e] * (double)x[e];
      }
    }
#pragma unroll
    for (int g = 0; g < NG; g++) s += (double)small_penalty(g, q, 1.f) * (double)R.pw[g] * (double)R.pw[g];
    return block_sum(s, red);
  }

};

template <int KT, int NT, int CO, int W>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * W, 64 * W), amdgpu_waves_per_eu(sm_occupancy(KT, NT, CO), sm_occupancy(KT, NT, CO))))
void k_train_small(const TrainParams P) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_item;
  __shared__ double red[W], trace_stash[2];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    if (item >= P.n_items) break;
    const __attribute__((address_space(4))) SItem* si = (const __attribute__((address_space(4))) SItem*)P.items + item / P.n_folds;
    Small<KT, NT, CO, W> T(P, si->d, si->y, smem, (float*)(P.slots + (uint64_t)blockIdx.x * P.slot_bytes), red, trace_stash,
                           item % P.n_folds);
    T.run();
  }
}

}  // namespace
