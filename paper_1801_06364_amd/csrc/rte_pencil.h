// Pencil passes of FP32 grids with the FFT stages that touch HBM kept in
// registers: the z derivative at 32^3 and 64^3 (orders the streaming pass
// does not hold) and 256^3, the y passes of 256^3 grids.
//
// A workgroup owns TZ kx columns of one pencil (all n points along the
// pencil axis, z for the z derivative, y for the y passes of 256^3 grids).
// At 256, thread (kx, j) loads the 16 points j + 16 r of its
// column straight from HBM (one row segment of TZ complex values per wavefront
// load) and applies the first radix-16 Stockham stage in registers; one
// exchange through LDS (row pitch TZ: the 16 lanes of one LDS cycle touch 16
// consecutive columns of a row) feeds the last stage, whose outputs are in
// natural order. For the z derivative the product with
// i k_z / n and the first stage of the inverse transform follow in registers
// on exactly those outputs, then one more exchange and the inverse's last
// stage, written straight to HBM. At 64 and 32 four threads share a
// column, each loading the n/4 points j + 4 r. Plans (verified against a
// direct DFT): 256 = 16 x 16, 64 = 16 x 4 and 32 = 8 x 4 both ways. Twiddles between the stages come
// from an LDS copy of the table exp(-2 pi i t / n).
#pragma once

namespace rte {
namespace pen {

#ifndef RTE_PEN_TZ256
#define RTE_PEN_TZ256 16
#endif

// TZ columns per workgroup; J = n / 16 threads per column, one per radix-16
// butterfly of the first stage; LDS holds the whole n x TZ tile. TZ = 8 and
// 32 measured no faster than 16.
template <int NN> struct Shape;
template <> struct Shape<256> {
  static constexpr int TZ = RTE_PEN_TZ256, NTILE = 128 / TZ, J = 16, THREADS = J * TZ;
};
// 64 and 32: J = 4 threads per column (radix-16 / 8 first stage), TZ = 16 kx
// columns per workgroup (one wavefront)
template <> struct Shape<64> {
  static constexpr int TZ = 16, NTILE = 32 / TZ, J = 4, THREADS = J * TZ;
};
template <> struct Shape<32> {
  static constexpr int TZ = 16, NTILE = 16 / TZ, J = 4, THREADS = J * TZ;
};

// FP32 pencils of these grids and modes run here; the others (FP64, the
// full 3D transforms of the exact propagation) in k_pencil.
template <typename T, int NN, int MODE> constexpr bool use_reg() {
  return std::is_same<T, float>::value && (NN == 32 || NN == 64 || NN == 256) &&
         (MODE == PENCIL_ZDERIV || (NN == 256 && (MODE == PENCIL_YFWD || MODE == PENCIL_YINV)));
}

template <int DIR> __device__ __forceinline__ float2 tw_dir(float2 w) {
  if constexpr (DIR > 0) w.y = -w.y;
  return w;
}

// x <- x * (i k / n)
__device__ __forceinline__ float2 times_ik(float2 x, float k) { return cmk<float2>(-k * x.y, k * x.x); }

template <int NN, int MODE>
__global__ void __launch_bounds__(Shape<NN>::THREADS)
k_pencil_reg(const float2* src, float2* dst,   // may alias (in place)
             const float2* __restrict__ twg, const float* __restrict__ kv, const Ctl* __restrict__ ctl,
             long long bs) {
  constexpr int n = NN, TZ = Shape<NN>::TZ, NTILE = Shape<NN>::NTILE;
  using Spec = SpecLayout<float, NN>;
  // offset of point i along the pencil axis
  auto axis = [](int i) { return pencil_z(MODE) ? size_t(i) * Spec::ZS : Spec::row(i); };
  constexpr int DIR = pencil_inverse(MODE) ? +1 : -1;
  src = slot_ptr(src, bs);
  dst = slot_ptr(dst, bs);
  twg = slot_ptr(twg, bs);
  kv = slot_ptr(kv, bs);
  ctl = slot_ptr(ctl, bs);
  if (ctl->stop) return;
  // 64 / 32: the four row blocks of the tile sit PAD entries apart, so
  // that the four row groups of one wavefront access fall in different banks
  constexpr int PAD = NN < 256 ? 16 : 0;
  __shared__ float2 tw[n];
  __shared__ float2 col[n * TZ + 4 * PAD];
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int bw = tile / NTILE;
  const int kx0 = (tile - bw * NTILE) * TZ;
  const int b = bw / n, w = bw - b * n;
  const size_t base = size_t(b) * Spec::MS + (pencil_z(MODE) ? Spec::row(w) : size_t(w) * Spec::ZS) + kx0;
  const int tid = threadIdx.x, kx = tid % TZ, j = tid / TZ;
  for (int i = tid; i < n; i += Shape<NN>::THREADS) tw[i] = twg[i];
  const float2* s = src + base + kx;
  float2* d = dst + base + kx;
  constexpr float inv_n = 1.0f / float(n);
  if constexpr (NN < 256) {
    static_assert(MODE == PENCIL_ZDERIV, "64- and 32-point register pencils do the z derivative only");
    // R = n / 4. Thread j < 4: stage 1 radix R over rows j + 4 r -> Y_j[k1];
    // stage 2 radix 4 over j for k1 = j + 4 t (t < R / 4) -> X[k1 + R k2],
    // with the twiddles exp(-2 pi i j k1 / n) applied after the exchange
    constexpr int R = NN / 4, NT = R / 4;
    auto at = [&](int blk, int row) { return (R * blk + row) * TZ + blk * PAD + kx; };
    float2 x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = s[axis(j + 4 * r)];
    Bfly<float2, R, -1>::run(x);
#pragma unroll
    for (int k1 = 0; k1 < R; ++k1) col[at(j, k1)] = x[k1];
    __syncthreads();
    float2 y[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int k1 = j + 4 * t;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) y[t][jj] = col[at(jj, k1)];
#pragma unroll
      for (int jj = 1; jj < 4; ++jj) y[t][jj] = cmul(y[t][jj], tw_dir<-1>(tw[jj * k1]));
      Bfly<float2, 4, -1>::run(y[t]);   // element k1 + R k2
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) y[t][k2] = times_ik(y[t][k2], kv[k1 + R * k2] * inv_n);
      // inverse: radix 4 over k2 -> Z[k1][p], times exp(2 pi i k1 p / n)
      Bfly<float2, 4, +1>::run(y[t]);
#pragma unroll
      for (int p = 1; p < 4; ++p) y[t][p] = cmul(y[t][p], tw_dir<+1>(tw[k1 * p]));
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int p = 0; p < 4; ++p) col[at(p, j + 4 * t)] = y[t][p];
    __syncthreads();
    // thread p = j: radix R over k1 -> output rows p + 4 s
#pragma unroll
    for (int k1 = 0; k1 < R; ++k1) x[k1] = col[at(j, k1)];
    Bfly<float2, R, +1>::run(x);
#pragma unroll
    for (int q = 0; q < R; ++q) d[axis(j + 4 * q)] = x[q];
  } else {
    // j < 16: stage 1 radix 16 over rows j + 16 r, stage 2 radix 16 (butterfly j)
    float2 x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = s[axis(j + 16 * r)];
    Bfly<float2, 16, DIR>::run(x);
#pragma unroll
    for (int q = 0; q < 16; ++q) col[(16 * j + q) * TZ + kx] = x[q];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = col[(j + 16 * r) * TZ + kx];
#pragma unroll
    for (int r = 1; r < 16; ++r) x[r] = cmul(x[r], tw_dir<DIR>(tw[r * j]));
    Bfly<float2, 16, DIR>::run(x);   // element j + 16 q
    if constexpr (MODE == PENCIL_ZDERIV) {
#pragma unroll
      for (int q = 0; q < 16; ++q) x[q] = times_ik(x[q], kv[j + 16 * q] * inv_n);
      Bfly<float2, 16, +1>::run(x);  // inverse stage 1 on the same elements: outputs 16 j + q
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 16; ++q) col[(16 * j + q) * TZ + kx] = x[q];
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = col[(j + 16 * r) * TZ + kx];
#pragma unroll
      for (int r = 1; r < 16; ++r) x[r] = cmul(x[r], tw_dir<+1>(tw[r * j]));
      Bfly<float2, 16, +1>::run(x);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) d[axis(j + 16 * q)] = x[q];
  }
}

}  // namespace pen
}  // namespace rte
