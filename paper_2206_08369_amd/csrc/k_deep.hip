// Kernels of packs whose models have two hidden layers (Section 7, Figure 3:
// the packed network extended by a second hidden layer in which a unit only
// ever sums the first-layer units of its own model).
//
// The hidden-to-hidden weights are block diagonal: model m's block W12_m
// [h2_m, h1_m] is stored row-major at offset koff[m] of one packed vector.
// With Zt1 [N1pad][Bp] and Zt2 [N2pad][Bp] batch-minor as everywhere else,
// the products of this layer are, per model,
//   forward   Z2_m  = W12_m act(Z1_m)                 [h2_m, Bp]
//   gradient  dW12_m = dZ2_m act(Z1_m)^T               [h2_m, h1_m]
//   backward  dZ1_m = (W12_m^T dZ2_m) * act'(Z1_m)     [h1_m, Bp]
// The first layer's product, the M3 forward / backward of the output layer,
// the loss and the dW1 product are the one-hidden-layer kernels.

#include "device_common.h"

#include <type_traits>

namespace pmlpk {

// W12[k] = uniform(tag 5, idx k) * bound12[model of k]; the model is found
// by binary search over koff [M+1].
__global__ __launch_bounds__(kBlock) void k_init_w12(float* __restrict__ W12, int64_t K,
                                                     const int64_t* __restrict__ koff, int M,
                                                     const float* __restrict__ bound12,
                                                     uint64_t key) {
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < K;
       k += (int64_t)gridDim.x * kBlock) {
    int lo = 0, hi = M - 1;  // last m with koff[m] <= k
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (koff[mid] <= k) lo = mid;
      else hi = mid - 1;
    }
    W12[k] = uniform_weight(key, 5, (uint64_t)k, bound12[lo]);
  }
}

hipError_t launch_init_w12(float* W12, int64_t K, const int64_t* koff, int32_t M,
                           const float* bound12, uint64_t key, hipStream_t s) {
  if (K <= 0) return hipSuccess;
  k_init_w12<<<grid_for(K), kBlock, 0, s>>>(W12, K, koff, M, bound12, key);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The three products of this layer on the fp32 matrix cores
// (v_mfma_f32_16x16x4f32: A 16 x 4, lane (li, lk) holds row li of column lk;
// B 4 x 16 likewise; lane (li, lk) ends with rows 4 lk + r of column li).
// They are small (at 1,000 models of 1..100 and 100..1 units and 128 samples
// 0.44 GFLOP each over 78 MB that stay in the caches), so what counts is the
// number of waves and of loads each has in flight: the wave that walked a
// model's units one dependent load at a time, eight scalar weights to each,
// took 60 to 76 us per product; these take 25 to 30 with their launch.  A wave
// has 16 rows of one layer and up to 64 samples, and kSegStep steps of four
// units are loaded, a pass ahead of their use, before the first is multiplied.
// ---------------------------------------------------------------------------

constexpr int kSegStep = 4;

// f(integral_constant<int, A>) for the uniform activation id.
template <class F>
__device__ __forceinline__ void seg_act_switch(int act, F&& f) {
  switch (act) {
    case 0: f(std::integral_constant<int, 0>{}); break;
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 11: f(std::integral_constant<int, 11>{}); break;
    default: f(std::integral_constant<int, 12>{}); break;
  }
}

// acc[i] += f(src)[.. n units ..]^T W for one wave: A[b][k] = f(src[k][b]) for
// the samples b0 + NBB li + i, B[k][li] = w[k wk + ...] (the lane's column).
// src: the lane's samples of the first unit; units past the last are zero in
// both operands, and a lane whose column does not exist has col = false.
template <int NBB, class F>
__device__ __forceinline__ void seg_product(f32x4 (&acc)[NBB], const float* __restrict__ src,
                                            int Bp, const float* __restrict__ w, int64_t wk,
                                            bool col, int n, int lk, F f) {
  struct Pass {
    float z[kSegStep][NBB];
    float w[kSegStep];
  };
  auto fetch = [&](Pass& p, int k0) {
#pragma unroll
    for (int u = 0; u < kSegStep; ++u) {
      int k = k0 + 4 * u + lk;
      if (k > n - 1) k = n - 1;
      const float* z = src + (int64_t)k * Bp;
      if constexpr (NBB == 4) {
        const f32x4 v = *(const f32x4*)z;
#pragma unroll
        for (int i = 0; i < 4; ++i) p.z[u][i] = v[i];
      } else if constexpr (NBB == 2) {
        const f32x2 v = *(const f32x2*)z;
        p.z[u][0] = v[0];
        p.z[u][1] = v[1];
      } else {
        p.z[u][0] = *z;
      }
      p.w[u] = w[k * wk];
    }
  };
  auto use = [&](const Pass& p, int k0) {
#pragma unroll
    for (int u = 0; u < kSegStep; ++u) {
      if (k0 + 4 * u >= n) break;  // wave-uniform
      const bool in = k0 + 4 * u + lk < n;
      const float wv = in && col ? p.w[u] : 0.f;
#pragma unroll
      for (int i = 0; i < NBB; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? f(p.z[u][i]) : 0.f, wv, acc[i], 0, 0, 0);
    }
  };
  constexpr int STEP = 4 * kSegStep;
  Pass p0, p1;
  fetch(p0, 0);
  for (int k0 = 0; k0 < n; k0 += 2 * STEP) {
    if (k0 + STEP < n) fetch(p1, k0 + STEP);
    use(p0, k0);
    if (k0 + STEP >= n) break;
    if (k0 + 2 * STEP < n) fetch(p0, k0 + 2 * STEP);
    use(p1, k0 + STEP);
  }
}

// ---------------------------------------------------------------------------
// Forward: one wave per (unit: model m, rows r0 .. r0+15 of its second layer)
// and 16 NBB samples; contraction over the model's first-layer units.
// ---------------------------------------------------------------------------

template <int NBB>
__global__ __launch_bounds__(64) void k_seg_fwd(const float* __restrict__ Zt1,
                                                float* __restrict__ Zt2, int Bp,
                                                const DeepArgs a,
                                                const SegUnit* __restrict__ units) {
  const SegUnit u = units[blockIdx.x];
  const int m = u.m, h1 = a.h1[m], h2 = a.h2[m];
  const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4;
  const int b0 = blockIdx.y * 16 * NBB;
  int bl = b0 + NBB * li;
  if (bl > Bp - NBB) bl = Bp - NBB;  // samples past the batch are not stored
  const int row = u.r0 + li;
  const bool ok = row < h2;
  const float* w = a.W12 + a.koff[m] + (int64_t)(ok ? row : h2 - 1) * h1;
  const float* z1 = Zt1 + a.off1[m] * Bp + bl;
  f32x4 acc[NBB];
#pragma unroll
  for (int i = 0; i < NBB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  seg_act_switch(a.act[m], [&](auto ac) {
    seg_product<NBB>(acc, z1, Bp, w, 1, ok, h1, lk,
                     [](float z) { return act_fwd(decltype(ac)::value, z); });
  });
  if (!ok) return;
  float* z2 = Zt2 + (a.off2[m] + row) * Bp;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int b = b0 + NBB * (4 * lk + r);
    if (b >= Bp) break;
#pragma unroll
    for (int i = 0; i < NBB; ++i) z2[b + i] = acc[i][r];
  }
}

// ---------------------------------------------------------------------------
// Backward into the first layer: one wave per (unit: model m, rows r0 ..
// r0+15 of its first layer) and 16 NBB samples; contraction over the model's
// second-layer units, then act'(Z1) and dZ1 over Z1 in place (each element is
// read and written by the same lane).  W12 is read before its update.
// ---------------------------------------------------------------------------

template <int NBB>
__global__ __launch_bounds__(64) void k_seg_back(float* __restrict__ Zt1,
                                                 const float* __restrict__ dZ2, int Bp,
                                                 const DeepArgs a,
                                                 const SegUnit* __restrict__ units) {
  const SegUnit u = units[blockIdx.x];
  const int m = u.m, h1 = a.h1[m], h2 = a.h2[m];
  const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4;
  const int b0 = blockIdx.y * 16 * NBB;
  int bl = b0 + NBB * li;
  if (bl > Bp - NBB) bl = Bp - NBB;
  const int row = u.r0 + li;
  const bool ok = row < h1;
  const float* w = a.W12 + a.koff[m] + (ok ? row : h1 - 1);  // w[i h1] = W12_m[i][row]
  const float* d2 = dZ2 + a.off2[m] * Bp + bl;
  f32x4 acc[NBB];
#pragma unroll
  for (int i = 0; i < NBB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  seg_product<NBB>(acc, d2, Bp, w, h1, ok, h2, lk, [](float d) { return d; });
  if (!ok) return;
  float* z1 = Zt1 + (a.off1[m] + row) * Bp;
  seg_act_switch(a.act[m], [&](auto ac) {
    float z[4][NBB];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int b = b0 + NBB * (4 * lk + r);
#pragma unroll
      for (int i = 0; i < NBB; ++i) z[r][i] = z1[(b < Bp ? b : 0) + i];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int b = b0 + NBB * (4 * lk + r);
      if (b >= Bp) break;
#pragma unroll
      for (int i = 0; i < NBB; ++i) {
        float der;
        (void)act_fwd_bwd(decltype(ac)::value, z[r][i], &der);
        z1[b + i] = acc[i][r] * der;
      }
    }
  });
}

// Up to four 16-sample blocks per wave; a batch class below 64 (16 or 32)
// takes fewer.
template <class K1, class K2, class K4, class... Args>
static void seg_launch(K1 k1, K2 k2, K4 k4, int32_t Bp, int32_t nunits, hipStream_t s, Args... args) {
  const int nbb = Bp <= 16 ? 1 : Bp <= 32 ? 2 : 4;
  const dim3 grid((unsigned)nunits, (unsigned)ceil_div_i(Bp, 16 * nbb));
  if (nbb == 1) k1<<<grid, 64, 0, s>>>(args...);
  else if (nbb == 2) k2<<<grid, 64, 0, s>>>(args...);
  else k4<<<grid, 64, 0, s>>>(args...);
}

hipError_t launch_seg_fwd(const float* Zt1, float* Zt2, int32_t Bp, const DeepArgs& a,
                          const SegUnit* units, int32_t nunits, hipStream_t s) {
  note_variant("k_seg_fwd", kArithFp32);
  if (nunits <= 0) return hipSuccess;
  seg_launch(k_seg_fwd<1>, k_seg_fwd<2>, k_seg_fwd<4>, Bp, nunits, s, Zt1, Zt2, (int)Bp, a, units);
  return hipGetLastError();
}

hipError_t launch_seg_back(float* Zt1, const float* dZ2, int32_t Bp, const DeepArgs& a,
                           const SegUnit* units, int32_t nunits, hipStream_t s) {
  note_variant("k_seg_back", kArithFp32);
  if (nunits <= 0) return hipSuccess;
  seg_launch(k_seg_back<1>, k_seg_back<2>, k_seg_back<4>, Bp, nunits, s, Zt1, dZ2, (int)Bp, a, units);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Weight gradient: one workgroup per tile of 16 rows x 64 columns of a
// model's block, a wave per 16 columns; contraction over the samples.  Lane
// (li, lk) loads four consecutive samples 16 s + 4 lk of its row of dZ2 and
// of its column's Z1, which are one k of four steps each (the same samples in
// both operands), so nothing is staged and a wave has 2 kSegStep vector loads
// in flight, a pass ahead.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_seg_grad(const float* __restrict__ Zt1,
                                                  const float* __restrict__ dZ2, int Bp,
                                                  const DeepArgs a,
                                                  const SegTile* __restrict__ tiles,
                                                  float* __restrict__ G12) {
  const SegTile t = tiles[blockIdx.x];
  const int m = t.m, h1 = a.h1[m], h2 = a.h2[m];
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int j0 = t.j0 + 16 * __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (j0 >= h1) return;
  const int i = t.i0 + li, j = j0 + li;
  const bool iok = i < h2, jok = j < h1;
  const float* d2 = dZ2 + (a.off2[m] + (iok ? i : h2 - 1)) * Bp + 4 * lk;
  const float* z1 = Zt1 + (a.off1[m] + (jok ? j : h1 - 1)) * Bp + 4 * lk;
  const int ns = Bp >> 4;  // 16-sample steps
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  seg_act_switch(a.act[m], [&](auto ac) {
    struct Pass {
      f32x4 d[kSegStep], z[kSegStep];
    };
    auto fetch = [&](Pass& p, int s0) {
#pragma unroll
      for (int u = 0; u < kSegStep; ++u) {
        const int s = s0 + u < ns ? s0 + u : ns - 1;
        p.d[u] = *(const f32x4*)(d2 + 16 * s);
        p.z[u] = *(const f32x4*)(z1 + 16 * s);
      }
    };
    auto use = [&](const Pass& p, int s0) {
#pragma unroll
      for (int u = 0; u < kSegStep; ++u) {
        if (s0 + u >= ns) break;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(
              iok ? p.d[u][e] : 0.f, jok ? act_fwd(decltype(ac)::value, p.z[u][e]) : 0.f, acc, 0, 0, 0);
      }
    };
    Pass p0, p1;
    fetch(p0, 0);
    for (int s = 0; s < ns; s += 2 * kSegStep) {
      if (s + kSegStep < ns) fetch(p1, s + kSegStep);
      use(p0, s);
      if (s + kSegStep >= ns) break;
      if (s + 2 * kSegStep < ns) fetch(p0, s + 2 * kSegStep);
      use(p1, s + kSegStep);
    }
  });
  if (!jok) return;
  float* out = G12 + a.koff[m];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = t.i0 + 4 * lk + r;
    if (row < h2) out[(int64_t)row * h1 + j] = acc[r];
  }
}

hipError_t launch_seg_grad(const float* Zt1, const float* dZ2, int32_t Bp, const DeepArgs& a,
                           const SegTile* tiles, int32_t ntiles, float* G12, hipStream_t s) {
  note_variant("k_seg_grad", kArithFp32);
  if (ntiles <= 0) return hipSuccess;
  k_seg_grad<<<(unsigned)ntiles, 256, 0, s>>>(Zt1, dZ2, Bp, a, tiles, G12);
  return hipGetLastError();
}

// W -= lr G over n entries (the hidden-to-hidden SGD update, after the
// backward has read the old weights).
__global__ __launch_bounds__(kBlock) void k_sgd(float* __restrict__ W,
                                                const float* __restrict__ G, int64_t n,
                                                float lr) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock)
    W[i] -= lr * G[i];
}

hipError_t launch_sgd(float* W, const float* G, int64_t n, float lr, hipStream_t s) {
  note_variant("k_sgd", kArithNone);
  if (n <= 0) return hipSuccess;
  k_sgd<<<grid_for(n), kBlock, 0, s>>>(W, G, n, lr);
  return hipGetLastError();
}

}  // namespace pmlpk
