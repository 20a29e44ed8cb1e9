// The forward pass (product, activation, M3 forward) in one kernel, the
// workgroup's waves split over the samples.
//
// This file is compiled once per padded batch size (PMLP_FWD_BP), each time
// with the instances of that batch.

#include "device_common.h"

#include <algorithm>

#ifndef PMLP_FWD_BP
#error "compile with -DPMLP_FWD_BP=16|32|64|128|256"
#endif

namespace pmlpk {

namespace {

// ---------------------------------------------------------------------------
// Z = X W1^T on the three-piece products of k_fwd_x3, with the activation and
// the M3 forward (Section 3, steps 1-4): the logits alone, for forward passes,
// so that Z is neither written nor read.
//
// In k_fwd_x3m (the epilogue in the layout that sums over units in the lane)
// every wave multiplies its own units by all the samples: the batch comes
// from LDS for every 16 units and the epilogue keeps a running sum per
// 16-sample block.  Here a workgroup of NW waves takes BP = 16 NW NI samples,
// wave w the 16 NI from 16 NI w on, and holds the pieces of those samples in
// registers for the whole launch.  The units go by in tiles of 16, ST of them
// a stage: every stage the waves whose turn it is load and split the W1 strip
// of one tile each into LDS (operand order, double buffered, the loads one of
// their turns ahead), and all waves multiply all tiles of the stage by their
// own samples: 9 KB of LDS reads per tile and wave for 36 products at two
// blocks, against 144 KB for 288 in k_fwd_x3m.  Lane (li, lk) ends with Z of
// unit li for the samples 16 ib + 4 lk + r and adds act(Z) W2 to its running
// sums; the sum over a model's units is one reduction over the 16 li lanes at
// the model's end.  A model's samples belong to one wave each, so no sum
// crosses a wave and there are no atomics.
//
// Workgroups take groups of whole models (the handle's plans), wide ones first,
// forwards and backwards in turn, which leaves their loads within a group of
// each other.
//
// At 100 features the matrix products (36 of 8.7 ns per tile and block pair)
// and the vector work (activation, sums, splitting) are about half of the time
// each: with two waves per SIMD they overlap in part only.  In packs below
// some 50,000 units the launch is one workgroup's chain: X from memory and its
// pieces 8 us, then 0.1 us per unit.  Measured, us a call, batch copy, product
// and M3 forward / this kernel: 60 models x 1 sample, 10 features, 15 / 7; 50,500
// units x 10,000 samples, 50 features, 1948 / 628; 505,000 x 256, 100 features,
// 341 / 227; 5,005,000 x 256, widths up to 1,000, 2748 / 1953.
//
// The six products hold an fp32 product as long as no piece and no partial sum
// leaves the range of fp32.  An infinite operand has NaN for its second piece,
// one above the largest bf16 (3.39e38) an infinite first one, and where a sum
// overflows, the lower products, added first, may do so with the other sign
// (1300 x 3e38 is inf - inf).  All of these end in NaN, which every activation
// here passes on, so the logits say where it happened: a wave that wrote a NaN
// computes those models again at its end with fp32 products, whose result
// (finite, infinite or NaN, as fp32 sums are) replaces the NaN.  A test of each
// tile's operands instead made the launch 3 to 6 % longer; this, a comparison per
// logit, 0 to 2 %.
// For finite operands the pieces lose nothing: norm of the error of the logits
// over their norm against 64 bits, fp32 MFMAs / this kernel: 16 features 1.2e-7 /
// 0.9e-7, 100 features and 16 or 64 samples 1.9e-7 / 1.5e-7 (120 models of 1 to
// 100 units).  (A piece of an operand below 1e-33 is subnormal.)
//
// Training steps stay on the unit-split kernels, by choice: with Z stored as well
// this kernel took 2410 us of the last of these (5.1 GB of stores) and made an
// epoch of 1,000 models a fifth shorter, at the same error against 64 bits, but
// an epoch's parameters would then carry another rounding of every step (samples
// that end up on the other side of ReLU's kink moved single weights of narrow
// models by up to 4.7e-4 of the weights' rms), and trained pools stay the same
// bits as long as no error is at stake.
// ---------------------------------------------------------------------------

constexpr int kBp = PMLP_FWD_BP;
constexpr int kNI = kBp == 16 ? 1 : 2;       // 16-sample blocks per wave
constexpr int kNW = kBp / 16 / kNI;          // waves per workgroup
constexpr int kST = kNW;                     // tiles per stage, one from each wave

// NC 32-wide k chunks on the three-piece products and, for odd TQ, up to
// three fp32 steps of four columns: F4 = 32 NC + 4 rem.  Even TQ covers
// F4 = 16 TQ - 16 + {0, 4, 8, 12, 16} with zero columns past F4.
template <int TQ>
struct FwdShape {
  static constexpr int NC = TQ / 2;
  static constexpr int RM = TQ & 1 ? 3 : 0;
};

constexpr int kTileOne = 256, kTileEnd = 512;  // bits of a tile's word
constexpr int kUnitLast = 256;                 // bit of a unit's uinfo
constexpr int kRowPad = 512;                  // of a tile's row past its group

__host__ __device__ constexpr int fwd_tile_bytes(int NC, int rem, int OM) {
  return NC * 3072 + rem * 256 + 64 * (1 + OM) + 16;
}

template <class T>
__device__ __forceinline__ T opaque_v(T v) {
  asm volatile("" : "+v"(v));
  return v;
}

template <class T>
__device__ __forceinline__ T opaque_s(T v) {
  asm volatile("" : "+s"(v));
  return v;
}

// The batch X [B][F] of one workgroup's samples as rows of F4 floats in LDS,
// with the constant input and the zero padding: the waves take their pieces
// from it.  All of a thread's loads are in flight at once (a round
// trip takes 2 us while the other workgroups stream).
template <int TQ, int BP, int NW>
__device__ __forceinline__ void stage_x(float* xs, const float* X, int F, int F4, int bcol,
                                             int B, int tid) {
  constexpr int NT = 64 * NW, NX = 16 * TQ * BP / NT;
  const int db = NT / F4, df = NT - db * F4;
  int b = tid / F4, f = tid - b * F4;
  float v[NX];
  const int b1 = b, f1 = f;
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int bc = b < B ? b : B - 1, fc = f < F ? f : F - 1;
    v[i] = X[(uint32_t)(bc * F + fc)];
    f += df;
    b += db;
    if (f >= F4) {
      f -= F4;
      ++b;
    }
  }
  b = opaque_v(b1);  // (the comparisons again, rather than kept in scalar registers)
  f = opaque_v(f1);
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const float w = b < B ? (f < F ? v[i] : (f == bcol ? 1.f : 0.f)) : 0.f;
    if (b < BP) xs[tid + i * NT] = w;
    f += df;
    b += db;
    if (f >= F4) {
      f -= F4;
      ++b;
    }
  }
}

// One of the pair of lanes whose low four index bits differ in the bit
// `step` selects (8, 4, 2, 1): xor 8, xor 7 (row_half_mirror), xor 2, xor 1.
// For a sum over 16 lanes in that order each lane meets every other once.
template <int STEP>
__device__ __forceinline__ float row_partner(float v) {
  constexpr int ctrl = STEP == 8 ? 0x128 : STEP == 4 ? 0x141 : STEP == 2 ? 0x4E : 0xB1;
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true));
}

// Sum of V values over the 16 lanes of a row, scattered: with V >= 16 the
// lane li ends with the sums of values li V/16 .. + V/16 - 1 in v[0 ..];
// with V = 8 lanes 2i and 2i + 1 both end with that of value i.
template <int V, int STEP>
__device__ __forceinline__ void row_reduce(float* v, int li) {
  constexpr bool halve = V > 1;
  const bool up = (li & STEP) != 0;
  if constexpr (halve) {
#pragma unroll
    for (int q = 0; q < V / 2; ++q) {
      const float keep = up ? v[q + V / 2] : v[q];
      const float send = up ? v[q] : v[q + V / 2];
      v[q] = keep + row_partner<STEP>(send);
    }
  } else {
    v[0] += row_partner<STEP>(v[0]);
  }
  if constexpr (STEP > 1) row_reduce<(halve ? V / 2 : 1), STEP / 2>(v, li);
}

// Activation id `act` (uniform over the wave below 255, else each lane's own
// arow) of NV values, in place.  Rows of several activations take the same
// code once per activation.
#define PMLP_ACTS                                                                      \
  PMLP_ACT(0) PMLP_ACT(1) PMLP_ACT(2) PMLP_ACT(3) PMLP_ACT(4) PMLP_ACT(5) PMLP_ACT(6)       \
  PMLP_ACT(7) PMLP_ACT(8) PMLP_ACT(9) PMLP_ACT(10) PMLP_ACT(11) PMLP_ACT(12)

// act_fwd, with KEEP NaN for NaN also where its choice of a branch drops it.
template <bool KEEP>
__device__ __forceinline__ float tile_act_fwd(int a, float z) {
  if (KEEP && a == 1) return z <= 0.f ? 0.f : z;
  if (KEEP && a == 11) return fabsf(z) <= 0.5f ? 0.f : z;
  return act_fwd(a, z);
}

template <bool KEEP, int NV>
__device__ __forceinline__ void tile_act(int act, int arow, float (&z)[NV]) {
  const bool one = act < 255;
  int A = one ? act : __builtin_amdgcn_readfirstlane(arow);
  bool done = false;
#pragma unroll 1
  while (true) {
    float v[NV];
    // (opaque, or every activation's terms would be hoisted out of the loop)
#pragma unroll
    for (int j = 0; j < NV; ++j) z[j] = opaque_v(z[j]);
    switch (A) {
#define PMLP_ACT(AA)                                                         \
  case AA: {                                                                 \
    _Pragma("unroll") for (int j = 0; j < NV; ++j) v[j] = tile_act_fwd<KEEP>(AA, z[j]); \
    break;                                                                   \
  }
      PMLP_ACTS
#undef PMLP_ACT
    }
    if (one) {
#pragma unroll
      for (int j = 0; j < NV; ++j) z[j] = v[j];
      return;
    }
    const bool mine = !done && arow == A;
#pragma unroll
    for (int j = 0; j < NV; ++j) z[j] = mine ? v[j] : z[j];
    done |= mine;
    const uint64_t left = __ballot(!done);
    if (!left) return;
    A = __builtin_amdgcn_readlane(arow, __builtin_ctzll(left));
  }
}

// The logits of model m for the samples b0 .. b0+15 again, where one of them is
// NaN: the products as fp32 MFMAs, 16 columns a step (4 lk .. 4 lk + 3 of them
// each lane's).
constexpr int kRedo = 4;  // steps whose loads are in flight
template <int OM>
__device__ __forceinline__ void model_fp32(const FwdSArgs& a, int m, int b0, int li, int lk) {
  // value `idx` of a lane's 4 OM sums after the reduction over the 16 li
  const int idx = OM == 2 ? li >> 1 : li, o1 = idx % OM, b1 = b0 + 4 * lk + idx / OM;
  float* const dst = a.out + (int64_t)m * a.sm + (int64_t)b1 * a.sb + o1;
  const bool mine = b1 < a.B && o1 < a.O;
  const float old = mine ? *dst : 0.f;
  if (!__any(old != old)) return;
  const int b = b0 + li, bc = b < a.B ? b : a.B - 1;
  const float* const xr = a.X + (int64_t)bc * a.F;
  const int64_t u1 = a.seg_off[m + 1];
  const int act = a.uinfo[a.seg_off[m]] & 255;
  float S[4 * OM];
#pragma unroll
  for (int q = 0; q < 4 * OM; ++q) S[q] = 0.f;
#pragma unroll 1
  for (int64_t u0 = a.seg_off[m]; u0 < u1; u0 += 16) {
    const bool in = u0 + li < u1;
    const int64_t u = in ? u0 + li : u1 - 1;
    const float* const wr = a.W1 + u * a.F4;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int k0 = 4 * lk; k0 - 4 * lk < a.F4; k0 += 16 * kRedo) {
      f32x4 wv[kRedo], xv[kRedo];
#pragma unroll
      for (int j = 0; j < kRedo; ++j) {
        const int k = k0 + 16 * j;
        wv[j] = *(const f32x4*)(wr + (k < a.F4 ? k : 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) xv[j][e] = xr[k + e < a.F ? k + e : 0];
      }
#pragma unroll
      for (int j = 0; j < kRedo; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = k0 + 16 * j + e;
          const float x = k < a.F ? xv[j][e] : (k == a.bcol ? 1.f : 0.f);
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, k < a.F4 ? wv[j][e] : 0.f, acc, 0, 0, 0);
        }
    }
    float h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = in ? acc[r] : 0.f;
    tile_act<false>(act, 0, h);
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = in ? h[r] : 0.f;
#pragma unroll
    for (int o = 0; o < OM; ++o) {
      const float w2 = a.W2[(int64_t)(o < a.O ? o : 0) * a.ldw + u];
#pragma unroll
      for (int r = 0; r < 4; ++r) S[r * OM + o] = fmaf(h[r], in ? w2 : 0.f, S[r * OM + o]);
    }
  }
  row_reduce<4 * OM, 8>(S, li);
  if (mine && !(OM == 2 && (li & 1))) *dst = S[0] + (a.b2 ? a.b2[(int64_t)m * a.O + o1] : 0.f);
}

template <int TQ, int OM>
__global__ __launch_bounds__(64 * kNW) __attribute__((amdgpu_waves_per_eu(2)))
void k_fwd_s(FwdSArgs a) {
  constexpr int NW = kNW, NI = kNI, BP = kBp, ST = kST;
  constexpr int NC = FwdShape<TQ>::NC, RM = FwdShape<TQ>::RM;
  constexpr int V = 4 * NI;  // samples per lane
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int F4 = a.F4;
  const int rem = RM ? (F4 - 32 * NC) >> 2 : 0;
  const int TB = fwd_tile_bytes(NC, rem, OM);
  const int W = a.wpc;

  // W workgroups per chunk of BP samples, one launched for each: with a loop
  // over chunks around it the compiler moved address arithmetic out of the
  // stages and spilled 137 registers
  const int chunk = blockIdx.x / W, w = blockIdx.x - chunk * W;
  const int B = a.B - chunk * BP < BP ? a.B - chunk * BP : BP;
  // ---- this wave's samples: X pieces, and the remainder columns in fp32 ----
  bf16x8 x0[NI][NC > 0 ? NC : 1], x1[NI][NC > 0 ? NC : 1], x2[NI][NC > 0 ? NC : 1];
  float xt[NI][RM > 0 ? RM : 1];
  float* const xs = (float*)lds;
  stage_x<TQ, BP, NW>(xs, a.X + (int64_t)chunk * BP * a.F, a.F, F4, a.bcol, B, threadIdx.x);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const float* xr = xs + (16 * (wave * NI + i) + li) * F4;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      f32x4 q[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int k = 32 * c + 8 * lk + 4 * e;
        if (RM || c < NC - 1) {
          q[e] = *(const f32x4*)(xr + k);
        } else {  // the last chunk may pass F4
          q[e] = *(const f32x4*)(xr + (k < F4 ? k : F4 - 4));
          if (k >= F4) q[e] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      split3(q[0], q[1], x0[i][c], x1[i][c], x2[i][c]);
    }
#pragma unroll
    for (int q = 0; q < RM; ++q) xt[i][q] = q < rem ? xr[32 * NC + 4 * q + lk] : 0.f;
  }
  __syncthreads();

  // ---- the stages, over the ends of groups ----------------------------------
  struct Pos {  // stage s of the workgroup's k-th group; len 0 past the last
    int64_t n0;
    int32_t len, m0, k, s;
  };
  auto group = [&](Pos& p, int k) {
    const int g = k * W + (k & 1 ? W - 1 - w : w);
    p.k = k;
    p.s = 0;
    p.len = 0;
    p.m0 = 0;
    p.n0 = 0;
    if (g < a.ngroups) {
      const FwdGroup q = a.groups[g];
      p.n0 = q.n0;
      p.len = q.len;
      p.m0 = q.m0;
    }
  };
  auto next = [&](const Pos& p) {
    Pos q = p;
    if ((p.s + 1) * (16 * ST) < p.len) ++q.s;
    else if (p.len > 0) group(q, p.k + 1);
    return q;
  };
  struct Raw {  // W1 strip of one tile and its units' data, as loaded
    f32x4 c[NC > 0 ? 2 * NC : 1];
    float t[RM > 0 ? RM : 1];
    int info;  // uinfo, + the model's place in the group << 10
    float w2[OM];
  };
  // row li of this wave's tile of the stage (tiles and rows past the group
  // repeat its last unit with zero output weights and no end mark; put() makes
  // their strip zero, or a last unit that overflows would add 0 inf)
  auto fetch = [&](Raw& r, const Pos& p) {
    const int last = (p.len - 1) >> 4;
    const int t = p.s * ST + wave < last ? p.s * ST + wave : last;
    const int64_t p0 = p.n0 + t * 16;
    const int left = p.len - t * 16;
    const bool in = li < left;
    const uint32_t row = in ? li : left - 1;
    const float* wt = a.W1 + p0 * F4;
    const uint32_t wo = row * (uint32_t)F4;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int k = 32 * c + 8 * lk + 4 * e;
        if (RM || c < NC - 1) {
          r.c[2 * c + e] = *(const f32x4*)(wt + (wo + (uint32_t)k));
        } else {  // the last chunk may pass F4
          const f32x4 q = *(const f32x4*)(wt + (wo + (uint32_t)(k < F4 ? k : F4 - 4)));
          r.c[2 * c + e] = k < F4 ? q : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
#pragma unroll
    for (int q = 0; q < RM; ++q)
      r.t[q] = wt[wo + (uint32_t)(32 * NC + 4 * (q < rem ? q : 0) + lk)];
    const int info = (a.uinfo + p0)[row];
    r.info = (in ? info : (info & 255) | kRowPad) | (((a.mid + p0)[row] - p.m0) << 10);
#pragma unroll
    for (int o = 0; o < OM; ++o)
      r.w2[o] = in && o < a.O ? (a.W2 + ((int64_t)o * a.ldw + p0))[row] : 0.f;
  };
  auto put = [&](Raw& r, int buf) {
    char* base = lds + (buf * ST + wave) * TB;
    if (__any(r.info & kRowPad)) {
      const bool pad = r.info & kRowPad;
#pragma unroll
      for (int c = 0; c < 2 * NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) r.c[c][e] = pad ? 0.f : r.c[c][e];
#pragma unroll
      for (int q = 0; q < RM; ++q) r.t[q] = pad ? 0.f : r.t[q];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      bf16x8 p0, p1, p2;
      split3(r.c[2 * c], r.c[2 * c + 1], p0, p1, p2);
      bf16x8* d = (bf16x8*)(base + c * 3072) + lane;
      d[0] = p0;
      d[64] = p1;
      d[128] = p2;
    }
#pragma unroll
    for (int q = 0; q < RM; ++q)
      if (q < rem) ((float*)(base + NC * 3072))[q * 64 + lane] = r.t[q];
    const int i0 = __builtin_amdgcn_readfirstlane(r.info);
    // one activation (else 255), one model, a model's last unit
    const int word = (__all(((r.info ^ i0) & 255) == 0) ? i0 & 255 : 255) |
                     (__all((r.info >> 10) == (i0 >> 10)) ? kTileOne : 0) |
                     (__any(r.info & kUnitLast) ? kTileEnd : 0);
    if (lk == 0) {
      int* mt = (int*)(base + NC * 3072 + rem * 256) + li;
      mt[0] = r.info;
#pragma unroll
      for (int o = 0; o < OM; ++o) mt[16 + 16 * o] = __float_as_int(r.w2[o]);
      if (li == 0) mt[16 + 16 * OM] = word;
    }
  };
  float S[V * OM];  // running sums of the open model
#pragma unroll
  for (int q = 0; q < V * OM; ++q) S[q] = 0.f;
  uint64_t bad = 0;  // bit m % 64: a logit of model m is NaN
  // the open model ends: its logits, and the sums start again
  auto emit = [&](int mm) {
    row_reduce<V * OM, 8>(S, li);
    constexpr int PER = V * OM >= 16 ? V * OM / 16 : 1;  // values per lane
    const int idx0 = V * OM >= 16 ? li * PER : li >> 1;
    float* const dst = a.out + (int64_t)chunk * BP * a.sb + (int64_t)mm * a.sm;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int idx = idx0 + e, o = idx % OM, q = idx / OM;
      const int b = 16 * (wave * NI + (q >> 2)) + 4 * lk + (q & 3);
      float s = S[e];
      if (a.b2 && o < a.O) s += a.b2[(int64_t)mm * a.O + o];
      if (NC) bad |= (uint64_t)(__any(s != s) ? 1 : 0) << (mm & 63);
      if (V * OM < 16 && (li & 1)) continue;
      if (b < B && o < a.O) dst[b * a.sb + o] = s;
    }
#pragma unroll
    for (int q = 0; q < V * OM; ++q) S[q] = 0.f;
  };

  // the stage at work, the one whose tiles are in registers or LDS already and
  // the one to be loaded
  Pos p0, p1, p2;
  group(p0, 0);
  p1 = next(p0);
  p2 = next(p1);
  if (p0.len == 0) return;
  Raw raw;
  fetch(raw, p0);
  put(raw, 0);
  if (p1.len) fetch(raw, p1);
  __syncthreads();
#pragma unroll 1
  for (int it = 0; p0.len; ++it) {
    const int t0 = p0.s * ST, nt = (p0.len + 15) >> 4;
    const int cnt = nt - t0 < ST ? nt - t0 : ST;
#pragma unroll 1
    for (int j = 0; j < ST; ++j) {
      if (j < cnt) {
        const char* const base = lds + ((it & 1) * ST + j) * TB;
        f32x4 acc[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          bf16x8 wc[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) wc[q] = ((const bf16x8*)(base + c * 3072))[64 * q + lane];
          // the piece products smallest first, the sample blocks in turn
#define PMLP_PIECE(XP, Q)                                 \
_Pragma("unroll") for (int i = 0; i < NI; ++i) acc[i] = \
    __builtin_amdgcn_mfma_f32_16x16x32_bf16(XP[i][c], wc[Q], acc[i], 0, 0, 0)
          PMLP_PIECE(x2, 0);
          PMLP_PIECE(x1, 1);
          PMLP_PIECE(x0, 2);
          PMLP_PIECE(x1, 0);
          PMLP_PIECE(x0, 1);
          PMLP_PIECE(x0, 0);
#undef PMLP_PIECE
        }
#pragma unroll
        for (int q = 0; q < RM; ++q)
          if (q < rem) {
            const float wt = ((const float*)(base + NC * 3072))[q * 64 + lane];
#pragma unroll
            for (int i = 0; i < NI; ++i)
              acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xt[i][q], wt, acc[i], 0, 0, 0);
          }
        const int* mt = (const int*)(base + NC * 3072 + rem * 256);
        const int word = __builtin_amdgcn_readfirstlane(mt[16 + 16 * OM]);
        float w2[OM];
#pragma unroll
        for (int o = 0; o < OM; ++o) w2[o] = __int_as_float(mt[16 + 16 * o + li]);
        float h[V];
#pragma unroll
        for (int q = 0; q < V; ++q) h[q] = acc[q >> 2][q & 3];
        tile_act<NC != 0>(word & 255, (word & 255) == 255 ? mt[li] & 255 : 0, h);
        if (word & kTileOne) {
#pragma unroll
          for (int q = 0; q < V; ++q)
#pragma unroll
            for (int o = 0; o < OM; ++o) S[q * OM + o] = fmaf(h[q], w2[o], S[q * OM + o]);
          if (word & kTileEnd)
            emit(p0.m0 + __builtin_amdgcn_readfirstlane(mt[0] >> 10));
        } else {
          // a model at a time, the other models' rows out of the sums
          const int mrow = mt[li] >> 10;
          const bool last = mt[li] & kUnitLast;
          const int m0 = __builtin_amdgcn_readfirstlane(mrow);
          const int ml = __builtin_amdgcn_readlane(mrow, 15);
          for (int mm = m0; mm <= ml; ++mm) {
            const bool mine = mrow == mm;
#pragma unroll
            for (int q = 0; q < V; ++q) {
              const float hv = mine ? h[q] : 0.f;
#pragma unroll
              for (int o = 0; o < OM; ++o)
                S[q * OM + o] = fmaf(hv, mine ? w2[o] : 0.f, S[q * OM + o]);
            }
            if (__any(mine && last)) emit(p0.m0 + mm);
          }
        }
      }
      // the next stage, each wave at a tile of its own
      if (j == wave && p1.len) {
        put(raw, (it + 1) & 1);
        if (p2.len) fetch(raw, p2);
      }
    }
    p0 = p1;
    p1 = p2;
    p2 = next(p2);
    __syncthreads();
  }
  if (NC && bad) {
    __threadfence_block();  // (a logit is read by another lane than wrote it)
    // (arguments and indices afresh: held over the stages they would cost
    // registers there)
    const FwdSArgs& r = *(const FwdSArgs*)opaque_s(__builtin_amdgcn_kernarg_segment_ptr());
    const int t = opaque_v((int)threadIdx.x), bid = opaque_s((int)blockIdx.x);
    const int c = bid / r.wpc, first = bid - c * r.wpc;
    const int b0 = c * BP + 16 * NI * __builtin_amdgcn_readfirstlane(t >> 6);
#pragma unroll 1
    for (int k = 0;; ++k) {
      const int g = k * r.wpc + (k & 1 ? r.wpc - 1 - first : first);
      if (g >= r.ngroups) break;
      const FwdGroup q = r.groups[g];
#pragma unroll 1
      for (int m = q.m0; m < q.m0 + q.nm; ++m)
        if (bad >> (m & 63) & 1)
#pragma unroll 1
          for (int i = 0; i < NI; ++i)
            model_fp32<OM>(r, m, b0 + 16 * i, t & 15, (t & 63) >> 4);
    }
  }
}

size_t fwd_s_lds(int32_t F4, int OM) {
  const int tq = (F4 + 15) / 16;
  const int odd = tq & 1 && F4 % 32 != 16;
  const int NC = odd ? tq / 2 : (tq + 1) / 2;
  const int rem = odd ? (F4 - 32 * NC) / 4 : 0;
  const size_t tiles = (size_t)2 * kST * fwd_tile_bytes(NC, rem, OM);
  return (std::max(tiles, (size_t)kBp * F4 * 4) + 15) / 16 * 16;
}

typedef void (*FwdSFn)(FwdSArgs);

template <int OM>
FwdSFn fwd_s_fn(int32_t F4) {
  // TQ odd for F4 = 32 NC + {4, 8, 12}, even above
  const int tq = (F4 + 15) / 16;
  switch (tq & 1 && F4 % 32 == 16 ? tq + 1 : tq) {
    case 1: return k_fwd_s<1, OM>;
    case 2: return k_fwd_s<2, OM>;
    case 3: return k_fwd_s<3, OM>;
    case 4: return k_fwd_s<4, OM>;
    case 5: return k_fwd_s<5, OM>;
    case 6: return k_fwd_s<6, OM>;
    case 7: return k_fwd_s<7, OM>;
    default: return nullptr;
  }
}

FwdSFn fwd_s_pick(int32_t F4, int32_t O) {
  if (F4 < 4 || F4 > 108) return nullptr;
  return O <= 2 ? fwd_s_fn<2>(F4) : O <= 4 ? fwd_s_fn<4>(F4) : nullptr;
}

}  // namespace

#define PMLP_CAT_(a, b) a##b
#define PMLP_CAT(a, b) PMLP_CAT_(a, b)

// Workgroups of this batch size the device holds at once, or 0 where the
// shape has no instance or does not fit in LDS.
int PMLP_CAT(fwd_s_slots_, PMLP_FWD_BP)(int32_t F4, int32_t O) {
  FwdSFn fn = fwd_s_pick(F4, O);
  return fn ? resident_blocks((const void*)fn, 64 * kNW, fwd_s_lds(F4, fwd_om(O))) : 0;
}

hipError_t PMLP_CAT(launch_fwd_s_, PMLP_FWD_BP)(const FwdSArgs& a, hipStream_t s) {
  FwdSFn fn = fwd_s_pick(a.F4, a.O);
  if (!fn || a.ngroups <= 0 || a.wpc <= 0 || a.nchunk <= 0 ||
      (int64_t)a.nchunk * a.wpc > 0x7fffffff)
    return hipErrorInvalidValue;
  fn<<<(unsigned)(a.nchunk * a.wpc), 64 * kNW, fwd_s_lds(a.F4, fwd_om(a.O)), s>>>(a);
  return hipGetLastError();
}

}  // namespace pmlpk
