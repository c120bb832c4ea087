// Streaming pass: z derivative and moment coupling in one sweep over the
// spectrum (orders up to kDenseOrder).
//
// Per spectral point the streaming term of eq. (10) in the real basis is
//   W_a = -i (kx Bx + ky By)[a,b] S_b  -  Bz[a,b] dS_b/dz,
// S the moments' xy spectra [b][z][ky][kx]. The stage's scale is left to the
// epilogue of the inverse pass, which multiplies and adds in one rounding. Folded
// into k here, the rounding of every product would enter all steps alike and add
// up over a solve: geometric mean of the errors of 41 FP32 solves against 64 bits
// 1.577e-7, 1.505e-7 with the scale left out (1.562e-7 with the two passes). (W
// carries 2^-2 ceil(log2 n) instead, which rounds nothing and keeps the range of a
// scaled one.) Every B_j moves degree l to
// l +- 1 (eq. 6), so the rows of even degree read the odd degrees only and
// the other way round: the operator splits into two halves that share no
// input and no output. A workgroup owns one half Q (inputs of degree parity
// Q, outputs of the other one), one ky and TZ kx columns at every z. Its
// waves take the inputs one moment (tile of n x TZ points) each: load it
// into registers, transform it along z (Stockham stages exchanged through a
// wave-private LDS buffer), multiply by i k_z, transform back and publish the
// derivative there; then all threads add the moments of this round, at their
// own points, to the accumulators of every output, which stay in registers
// for the whole sweep. S itself is published in LDS too, or, where that would
// halve the workgroups per CU and the spectra sit in the Infinity Cache, read
// a second time from the caches. Each input is read from HBM once and each
// output written once (2F per stage, F = M n^3 elements, instead of 5F for a
// derivative pass and a coupling pass).
//
// Bound: HBM at 128^3 P_7 (without transforms and sums the same sweep takes
// 230 us); transforms and LDS on the other grids. Against the two passes it
// replaces: FP32 128^3 P_7 490 -> 285 us, FP64 1003 -> 516, 256^3 P_5 2345 ->
// 1635, 64^3 P_7 55 -> 30, 64^3 P_5 32 -> 19, 96^3 P_3 47 -> 33, 48^3 P_4 FP64
// 47 -> 15 (inside a time step, whose field passes take the caches in turn; in a
// loop of its own 275, 1590, 28 and 31 of these).
// The transforms of the outputs instead of the inputs (all three terms summed
// in kz space, one tile per wave) run 2 us faster at 96^3 P_3 and 10% at 256^3,
// but pass the x and y terms through the z transforms' rounding: the error of
// whole solves against 64 bits grows by 1.3 (1.5 to 2 on the radix-3 grids).
// Loading the next round's tiles before this round's transforms (instead of
// after them) measured slower on every grid (64^3 P_7 37 against 28), so the
// loads are not waited for long.
#pragma once

namespace rte {
namespace strm {

// ---------------------------------------------------------- moment sets ---
// degree parity of moment a, and the moments of one parity in order
__host__ __device__ constexpr int l_parity(int a) { return isqrt_c(a) & 1; }
__host__ __device__ constexpr int set_size(int N, int Q) {
  int c = 0;
  for (int l = Q; l <= N; l += 2) c += 2 * l + 1;
  return c;
}
__host__ __device__ constexpr int set_at(int N, int Q, int i) {
  for (int l = Q; l <= N; l += 2) {
    if (i < 2 * l + 1) return l * l + i;
    i -= 2 * l + 1;
  }
  return -1;
}
// position of moment a within its set
__host__ __device__ constexpr int set_pos(int a) {
  const int l = isqrt_c(a);
  int c = a - l * l;
  for (int k = l & 1; k < l; k += 2) c += 2 * k + 1;
  return c;
}

// ----------------------------------------------------------------- plans ---
// TZ columns per tile, L lanes per column with P = n / L points each, the
// radices of the forward transform (the inverse takes them in reverse, so
// that its first stage starts on the registers the forward ends in).
// A row of a tile is 64 bytes (TZ = 8 FP32, 4 FP64) or 128.
struct Plan {
  int TZ, L, R[3], stages;
};
template <typename T> __host__ __device__ constexpr Plan plan_of(int n) {
  const bool f = sizeof(T) == 4;
  switch (n) {
    case 16: return {8, 4, {4, 4, 1}, 2};
    case 32: return {8, 4, {8, 4, 1}, 2};
    case 48: return {f ? 8 : 4, 4, {12, 4, 1}, 2};
    case 64: return {8, 8, {8, 8, 1}, 2};
    case 96: return f ? Plan{8, 8, {12, 2, 4}, 3} : Plan{4, 8, {12, 2, 4}, 3};
    case 128: return f ? Plan{8, 8, {16, 8, 1}, 2} : Plan{4, 16, {8, 4, 4}, 3};
    default: return f ? Plan{8, 16, {16, 16, 1}, 2} : Plan{4, 32, {8, 8, 4}, 3};
  }
}

template <typename T, int NN, int N> struct Cfg {
  using V = typename cplx_of<T>::type;
  using Lay = SpecLayout<T, NN>;
  static constexpr Plan pl = plan_of<T>(NN);
  static constexpr int n = NN, H = NN / 2, TZ = pl.TZ, L = pl.L, P = NN / L;
  static constexpr int G = L * TZ;                       // lanes per moment tile
  static constexpr int WPM = G > 64 ? G / 64 : 1;        // waves per moment
  static constexpr int MPW = G < 64 ? 64 / G : 1;        // moments per wave
  static constexpr int OUT = set_size(N, 0) > set_size(N, 1) ? set_size(N, 0) : set_size(N, 1);
  // registers of the accumulators per thread of a workgroup of w waves
  static constexpr int acc_regs(int w) { return OUT * (n * TZ / (64 * w)) * 2 * int(sizeof(T) / 4); }
  // Waves that sum. The largest halves (P_7, 36 moments) run at one point
  // per thread as far as 12 waves go (96^3 141 us against 161 with two points;
  // at 128^3 the tiles of 16 waves exceed the LDS: 286 against 275 with
  // eight). Otherwise the fewest waves, a divisor of the tile's points, whose
  // accumulators fit 168 of 256 registers, from four on large grids (96^3 FP32, 64^3
  // FP64 and above: more workgroups per CU: 128^3 P_5 156 us with 4, 197 with 8;
  // 64^3 P_5 FP64 30 with 4, 35 with 8) and eight on small ones (more inputs
  // per round: 64^3 P_5 18.9 with 8, 19.6 with 4; 48^3 P_3 7.0 with 6, 7.5 with
  // 3, 9.5 with 2).
  static constexpr int waves() {
    const int full = n * TZ / 64;                        // waves at one point per thread
    if (OUT > 28) return full <= 12 ? full : full / 2;
    const int lo = n * int(sizeof(T)) >= 384 ? 4 : 8;
    for (int w = 1; w <= 16; ++w)
      if (full % w == 0 && w % WPM == 0 && (w >= lo || w == full) && acc_regs(w) <= 168) return w;
    return full;
  }
  static constexpr int NW = waves(), ST = 64 * NW;
  // Waves of the workgroup. A round is a chain of loads, transforms and barriers,
  // so a half should not need many: as long as it takes more than eight, waves
  // that transform only are added to those that sum too. 16^3 P_7 (36 moments,
  // two to a wave): five rounds instead of nine, step 60 us FP32 and 70 FP64 instead
  // of 76 and 86 (73 and 85 with a derivative and a coupling pass), of eight solves
  // together 99 and 121 instead of 111 and 136 (253 and 295).
  static constexpr int all_waves() {
    int w = NW;
    while (w * MPW * 8 < OUT * WPM && w + NW <= 8) w += NW;
    return w;
  }
  static constexpr int TW = all_waves(), BT = 64 * TW;
  static constexpr int PTS = n * TZ;
  static constexpr int VW = (PTS / ST) % 2 == 0 && sizeof(T) == 4 ? 2 : 1;   // points per 16-byte access
  static constexpr int PPT = PTS / ST;
  static constexpr int RK = pl.R[pl.stages - 1];         // last radix of the forward
  static constexpr int PADROWS = n / pl.R[0] > n / RK ? n / pl.R[0] : n / RK;
  static constexpr int DROWS = n + PADROWS;              // exchange buffer
  // S read again from the caches instead of published in LDS: fields below
  // 120 MB, which leaves LDS for more workgroups per CU (96^3 P_3 31 us against 39,
  // P_4 47 against 51, P_5 with 127 MB 76 against 73; 96^3 P_3 FP64 54 against 74,
  // 48^3 P_4 FP64 15 against 24). Not at 64^3, where two workgroups of eight
  // wavefronts fit with S in LDS too (FP64 P_6, P_7: one): reading again costs steps
  // of P_2 to P_7 0 to 5.5%, FP32 and FP64, and those of eight solves together 0 to 9%.
  // The size is one solve's, also where a batch's slots exceed the caches, since
  // a slot computes what a solve alone does: eight slots gain 3 to 17% from it in
  // FP64 (32^3 to 128^3) and at 48^3 P_3, P_4, and lose 2 to 5% in FP32 at 32^3 P_4 and
  // up, 48^3 P_5 and up, 96^3 P_3, P_4 and 128^3 P_1, P_2.
  static constexpr bool SG =
      n != 64 && size_t(N + 1) * (N + 1) * n * n * n * sizeof(T) < size_t(120) * 1000 * 1000;
  static constexpr int SLOT = ((SG ? 0 : n) + DROWS) * TZ;   // LDS of one moment: S (if published), derivative
  static constexpr size_t lds_of(int moments) {
    return (size_t(moments) * SLOT + n) * sizeof(V) + size_t(n) * sizeof(T);
  }
  // moments per round: one tile for each wave (or part of one), no more than
  // a half has, within 160 KB
  static constexpr int moments() {
    int m = TW * MPW / WPM;
    while (m > MPW && (m - MPW >= OUT || lds_of(m) > 160 * 1024)) m -= MPW;
    return m;
  }
  static constexpr int MPR = moments();
  // moments whose S loads from the caches are in flight together (32 registers)
  static constexpr int sb() {
    const int b = 32 / (PPT * 2 * int(sizeof(T) / 4));
    return b < 1 ? 1 : (b > MPR ? MPR : b);
  }
  static constexpr int SB = sb();
  static constexpr size_t lds() { return lds_of(MPR); }
  // waves per SIMD asked of the compiler: what accumulators, points and about
  // 44 other registers leave, two at least
  static constexpr int min_waves() {
    const int r = acc_regs(NW) + 2 * P * int(sizeof(T) / 4) + 44;
    const int w = 512 / r;
    return w < 2 ? 2 : (w > 4 ? 4 : w);
  }
  static_assert(PTS % ST == 0 && ST % TZ == 0 && 64 % TZ == 0, "a thread keeps its kx over its points");
};

// Configurations that run this pass: the accumulators, one column's points
// and the addresses fit the registers (256 per thread up to eight waves, 168
// beyond), a round's tiles fit 160 KB of LDS, and where several waves share a
// tile all of them take part in its barriers (N = 0 has no round). Left out:
// 256^3 above P_5.
template <typename T, int NN, int N> constexpr bool use_stream() {
  using C = Cfg<T, NN, N>;
  return N <= kDenseOrder && C::TW <= 12 && C::acc_regs(C::NW) <= (C::TW > 8 ? 88 : 168) &&
         C::lds() <= 160 * 1024 && (C::WPM == 1 || C::MPR * C::WPM == C::TW || N == 0);
}

// ------------------------------------------------------------ transforms ---
// Orders LDS accesses among the lanes that share a tile (one wave: they
// execute in order; more: a workgroup barrier).
template <int WPM> __device__ __forceinline__ void tile_sync() {
  if constexpr (WPM == 1) wave_sync();
  else __syncthreads();
}

// Stages ST.. of a transform in direction DIR (radices in reverse order for
// the inverse), S the product of the radices done. x: inputs of stage ST,
// [t][r] = row j + r n / R of butterfly j = l + L t; on return the outputs of
// the last stage, [t][q] = row j + q n / R of the same butterflies.
// The rows that a first stage writes (R j + q) are stored one row further
// per R rows, so that the two columns groups of one LDS cycle fall in
// different banks.
template <class C, int DIR, int ST = 0, int S = 1>
__device__ __forceinline__ void stages(typename C::V* x, typename C::V* buf, int l, int kx, const typename C::V* tw) {
  using V = typename C::V;
  constexpr int n = C::n, L = C::L, P = C::P, NS = C::pl.stages;
  constexpr int R = DIR < 0 ? C::pl.R[ST] : C::pl.R[NS - 1 - ST];
  constexpr int NB = P / R, SPAN = n / (S * R);
  static_assert(P % R == 0, "whole butterflies per lane");
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    if constexpr (S > 1) {
      const int k = (l + L * t) % S;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        V w = tw[r * k * SPAN];
        if constexpr (DIR > 0) w.y = -w.y;
        x[t * R + r] = cmul(x[t * R + r], w);
      }
    }
    Bfly<V, R, DIR>::run(x + t * R);
  }
  if constexpr (ST + 1 < NS) {
    constexpr int R2 = DIR < 0 ? C::pl.R[ST + 1] : C::pl.R[NS - 2 - ST];
    constexpr int PADR = S == 1 ? R : 0;
    static_assert(PADR == 0 || (n / R2) % (PADR ? PADR : 1) == 0, "padding splits over the rows read");
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int j = l + L * t;
      const int o = S == 1 ? j * (R + 1) : (j / S) * S * R + j % S;
#pragma unroll
      for (int q = 0; q < R; ++q) buf[(o + q * S) * C::TZ + kx] = x[t * R + q];
    }
    tile_sync<C::WPM>();
#pragma unroll
    for (int t = 0; t < P / R2; ++t) {
      const int j = l + L * t;
      const int o = PADR ? j + j / (PADR ? PADR : 1) : j;
      constexpr int st = n / R2 + (PADR ? n / R2 / (PADR ? PADR : 1) : 0);
#pragma unroll
      for (int r = 0; r < R2; ++r) x[t * R2 + r] = buf[(o + r * st) * C::TZ + kx];
    }
    tile_sync<C::WPM>();
    stages<C, DIR, ST + 1, S * R>(x, buf, l, kx, tw);
  }
}

// -------------------------------------------------------------- coupling ---
// acc[pos(a)] += B[a, b] (X | Y | Z)_b for every output a that reads input b.
template <class C, typename T, int N, int B, int S>
struct Scatter {
  static __device__ __forceinline__ void run(typename C::V (*acc)[C::VW], const typename C::V* X,
                                             const typename C::V* Y, const typename C::V* Z) {
    constexpr int l = isqrt_c(B);
    constexpr SlotList sl = slots_of(N, l, B - l * l - l);
    if constexpr (S < sl.count) {
      constexpr int a = sl.b[S];
      constexpr double c0 = ct::real_coef(N, 0, a, B), c1 = ct::real_coef(N, 1, a, B), c2 = ct::real_coef(N, 2, a, B);
      constexpr int p = set_pos(a);
#pragma unroll
      for (int v = 0; v < C::VW; ++v) {
        if constexpr (c0 != 0.0) {
          acc[p][v].x += T(c0) * X[v].x;
          acc[p][v].y += T(c0) * X[v].y;
        }
        if constexpr (c1 != 0.0) {
          acc[p][v].x += T(c1) * Y[v].x;
          acc[p][v].y += T(c1) * Y[v].y;
        }
        if constexpr (c2 != 0.0) {
          acc[p][v].x += T(c2) * Z[v].x;
          acc[p][v].y += T(c2) * Z[v].y;
        }
      }
      Scatter<C, T, N, B, S + 1>::run(acc, X, Y, Z);
    }
  }
};

// X = -i kx S_b (S: VW points), Y the same with ky, Z = -dS_b/dz from LDS.
template <class C, typename T, int N, int B>
__device__ __forceinline__ void add_moment(typename C::V (*acc)[C::VW], const typename C::V* S, const typename C::V* d,
                                           const T* kxs, T kys) {
  using V = typename C::V;
  V X[C::VW], Y[C::VW], Z[C::VW];
  if constexpr (C::VW == 2) {
    const float4 dv = *reinterpret_cast<const float4*>(d);
    Z[0] = cmk<V>(dv.x, dv.y);
    Z[1] = cmk<V>(dv.z, dv.w);
  } else {
    Z[0] = *d;
  }
#pragma unroll
  for (int v = 0; v < C::VW; ++v) {
    const V s = cmk<V>(S[v].y, -S[v].x);
    Y[v] = cscale(s, kys);
    X[v] = cscale(s, kxs[v]);
  }
  Scatter<C, T, N, B, 0>::run(acc, X, Y, Z);
}
// VW points of a field, one 16-byte access where there are two
template <class C> __device__ __forceinline__ void load_points(typename C::V* x, const typename C::V* p) {
  if constexpr (C::VW == 2) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    x[0] = cmk<typename C::V>(v.x, v.y);
    x[1] = cmk<typename C::V>(v.z, v.w);
  } else {
    x[0] = *p;
  }
}

// Moments I0 .. I0 + NM - 1 of round RD: S at every item of the thread.
template <class C, int N, int Q, int RD, int I0, int NM, int I = 0>
__device__ __forceinline__ void load_s(typename C::V (*sv)[C::PPT / C::VW][C::VW], const typename C::V* __restrict__ src,
                                       unsigned lo) {
  constexpr int i = RD * C::MPR + I0 + I;
  if constexpr (I < NM && I0 + I < C::MPR && i < set_size(N, Q)) {
#pragma unroll
    for (int k = 0; k < C::PPT / C::VW; ++k)
      load_points<C>(sv[I][k], src + (size_t(set_at(N, Q, i)) * C::Lay::MS +
                                      size_t(k * C::ST * C::VW / C::TZ) * C::Lay::ZS) + lo);
    load_s<C, N, Q, RD, I0, NM, I + 1>(sv, src, lo);
  }
}
template <class C, typename T, int N, int Q, int RD, int I0, int NM, int I = 0>
__device__ __forceinline__ void add_s(typename C::V (*acc)[set_size(N, 1 - Q)][C::VW],
                                      const typename C::V (*sv)[C::PPT / C::VW][C::VW], const typename C::V* pub, int e,
                                      const T* kxs, T kys) {
  constexpr int i = RD * C::MPR + I0 + I;
  if constexpr (I < NM && I0 + I < C::MPR && i < set_size(N, Q)) {
#pragma unroll
    for (int k = 0; k < C::PPT / C::VW; ++k)
      add_moment<C, T, N, set_at(N, Q, i)>(acc[k], sv[I][k], pub + (I0 + I) * C::SLOT + e + k * C::ST * C::VW, kxs, kys);
    // (else the LDS reads of the whole round are hoisted above the sums)
    if constexpr (I % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    add_s<C, T, N, Q, RD, I0, NM, I + 1>(acc, sv, pub, e, kxs, kys);
  }
}
// Batches I0.. of a round after the first
template <class C, typename T, int N, int Q, int RD, int I0>
__device__ __forceinline__ void add_batches(typename C::V (*acc)[set_size(N, 1 - Q)][C::VW],
                                            typename C::V (*sv)[C::PPT / C::VW][C::VW],
                                            const typename C::V* __restrict__ src, const typename C::V* pub, int e,
                                            unsigned lo, const T* kxs, T kys) {
  if constexpr (I0 < C::MPR && RD * C::MPR + I0 < set_size(N, Q)) {
    if constexpr (C::SG) {
      if constexpr (I0 > 0) load_s<C, N, Q, RD, I0, C::SB>(sv, src, lo);
      add_s<C, T, N, Q, RD, I0, C::SB>(acc, sv, pub, e, kxs, kys);
      __builtin_amdgcn_sched_barrier(0);
      add_batches<C, T, N, Q, RD, I0 + C::SB>(acc, sv, src, pub, e, lo, kxs, kys);
    } else {
      typename C::V s1[1][C::PPT / C::VW][C::VW];
#pragma unroll
      for (int k = 0; k < C::PPT / C::VW; ++k)
        load_points<C>(s1[0][k], pub + I0 * C::SLOT + C::DROWS * C::TZ + e + k * C::ST * C::VW);
      add_s<C, T, N, Q, RD, I0, 1>(acc, s1, pub, e, kxs, kys);
      if constexpr (I0 % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      add_batches<C, T, N, Q, RD, I0 + 1>(acc, sv, src, pub, e, lo, kxs, kys);
    }
  }
}

// Workgroup barrier that orders LDS only: loads of the next round stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Offset of moment i of the set of degree parity Q (degrees Q, Q + 2, ...).
template <class C> __device__ __forceinline__ size_t set_offset(int Q, int i) {
  int l = Q;
  while (i >= 2 * l + 1) {
    i -= 2 * l + 1;
    l += 2;
  }
  return size_t(l * l + i) * C::Lay::MS;
}

// Loads the tile of input g of round RD (rows l + L t + n / R0 r, column kx).
template <class C, int N, int Q, int RD>
__device__ __forceinline__ void load_tile(typename C::V* x, const typename C::V* __restrict__ src, int g, int gl) {
  constexpr int n = C::n, R0 = C::pl.R[0];
  constexpr size_t AX = C::Lay::ZS;
  const int i = RD * C::MPR + g;
  if (g < C::MPR && i < set_size(N, Q)) {
    const typename C::V* s = src + set_offset<C>(Q, i);
    asm volatile("" : "+v"(gl));   // (offsets formed anew in every round, see `rounds`)
    const unsigned lo = unsigned(gl / C::TZ) * unsigned(AX) + gl % C::TZ;
#pragma unroll
    for (int t = 0; t < C::P / R0; ++t)
#pragma unroll
      for (int r = 0; r < R0; ++r) x[t * R0 + r] = (s + (size_t(C::L) * t + size_t(n / R0) * r) * AX)[lo];
  }
}

// Rounds RD.. : differentiate, publish, add.
template <class C, typename T, int N, int Q, int RD>
__device__ __forceinline__ void rounds(typename C::V (*acc)[set_size(N, 1 - Q)][C::VW], typename C::V* x,
                                       const typename C::V* __restrict__ src, typename C::V* pub,
                                       const typename C::V* tw, const T* kz, const T* kxs, T kys, int g, int gl) {
  using V = typename C::V;
  constexpr int IN = set_size(N, Q);
  if constexpr (RD * C::MPR < IN) {
    constexpr int n = C::n, TZ = C::TZ, L = C::L, P = C::P, R0 = C::pl.R[0], RK = C::RK;
    if ((g < C::MPR && RD * C::MPR + g < IN) || C::WPM > 1) {
      // opaque copy: the index arithmetic of the stages is redone in every
      // round instead of being held in registers across the rounds
      int o = gl;
      asm volatile("" : "+v"(o));
      const int kx = o % TZ, l = (o / TZ) % L;
      V* ex = pub + g * C::SLOT;
      if constexpr (!C::SG) {
#pragma unroll
        for (int t = 0; t < P / R0; ++t)
#pragma unroll
          for (int r = 0; r < R0; ++r) ex[(C::DROWS + l + L * t + n / R0 * r) * TZ + kx] = x[t * R0 + r];
      }
      stages<C, -1>(x, ex, l, kx, tw);
#pragma unroll
      for (int t = 0; t < P / RK; ++t)
#pragma unroll
        for (int r = 0; r < RK; ++r) {
          const T k = kz[l + L * t + n / RK * r];
          x[t * RK + r] = cmk<V>(-k * x[t * RK + r].y, k * x[t * RK + r].x);
        }
      stages<C, +1>(x, ex, l, kx, tw);
#pragma unroll
      for (int t = 0; t < P / R0; ++t)
#pragma unroll
        for (int r = 0; r < R0; ++r) ex[(l + L * t + n / R0 * r) * TZ + kx] = x[t * R0 + r];
    }
    int e = int(threadIdx.x) * C::VW;
    asm volatile("" : "+v"(e));
    // (k moves a whole number of rows: uniform base, one lane offset)
    const unsigned lo = unsigned(e / TZ) * unsigned(C::Lay::ZS) + e % TZ;
    V sv[C::SB][C::PPT / C::VW][C::VW];
    const bool sums = C::TW == C::NW || int(threadIdx.x) < C::ST;   // uniform per wavefront
    if constexpr (C::SG) {
      if (sums) load_s<C, N, Q, RD, 0, C::SB>(sv, src, lo);
    }
    load_tile<C, N, Q, RD + 1>(x, src, g, gl);
    lds_barrier();
    if (sums) add_batches<C, T, N, Q, RD, 0>(acc, sv, src, pub, e, lo, kxs, kys);
    // the sums are formed here (the compiler would sink them to the stores
    // and hold the published values of every round instead)
#pragma unroll
    for (int k = 0; k < C::PPT / C::VW; ++k)
#pragma unroll
      for (int a = 0; a < set_size(N, 1 - Q); ++a)
#pragma unroll
        for (int v = 0; v < C::VW; ++v) asm volatile("" : "+v"(acc[k][a][v].x), "+v"(acc[k][a][v].y));
    lds_barrier();
    rounds<C, T, N, Q, RD + 1>(acc, x, src, pub, tw, kz, kxs, kys, g, gl);
  }
}

template <class C, typename T, int N, int Q>
__device__ __forceinline__ void sweep(const typename C::V* __restrict__ src, typename C::V* __restrict__ dst,
                                      typename C::V* pub, const typename C::V* tw, const T* kz, const T* kxs, T kys) {
  using V = typename C::V;
  constexpr int OUTQ = set_size(N, 1 - Q);
  if constexpr (OUTQ > 0) {
    constexpr int NI = C::PPT / C::VW;
    const int tid = threadIdx.x;
    const int g = C::MPW == 1 ? __builtin_amdgcn_readfirstlane(tid / C::G) : tid / C::G;   // moment slot of this lane
    V acc[NI][OUTQ][C::VW];
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
      for (int a = 0; a < OUTQ; ++a)
#pragma unroll
        for (int v = 0; v < C::VW; ++v) acc[k][a][v] = cmk<V>(T(0), T(0));
    V x[C::P];
    load_tile<C, N, Q, 0>(x, src, g, tid % C::G);
    rounds<C, T, N, Q, 0>(acc, x, src, pub, tw, kz, kxs, kys, g, tid % C::G);
    if (C::TW > C::NW && tid >= C::ST) return;
    const int e = tid * C::VW;
    const unsigned lo = unsigned(e / C::TZ) * unsigned(C::Lay::ZS) + e % C::TZ;
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
      for (int a = 0; a < OUTQ; ++a) {
        V* o = dst + (size_t(set_at(N, 1 - Q, a)) * C::Lay::MS + size_t(k * C::ST * C::VW / C::TZ) * C::Lay::ZS) + lo;
        if constexpr (C::VW == 2)
          *reinterpret_cast<float4*>(o) = make_float4(acc[k][a][0].x, acc[k][a][0].y, acc[k][a][1].x, acc[k][a][1].y);
        else *o = acc[k][a][0];
      }
  }
}

// W's power-of-two scale, about 1 / n^2
template <int NN> constexpr double w_scale() {
  double s = 1.0;
  for (int m = 1; m < NN; m *= 2) s *= 0.25;
  return s;
}

// Grid: (ky, kx tile, Q), neighbouring tiles on one XCD.
template <typename T, int NN, int N>
__global__ void __launch_bounds__((Cfg<T, NN, N>::BT), (Cfg<T, NN, N>::min_waves()))
k_stream(const typename cplx_of<T>::type* __restrict__ spec, typename cplx_of<T>::type* __restrict__ wspec,
         const typename cplx_of<T>::type* __restrict__ twg, const T* __restrict__ kv,
         const Ctl* __restrict__ ctl, long long bs) {
  using C = Cfg<T, NN, N>;
  using V = typename C::V;
  constexpr int n = NN, TZ = C::TZ, NT = C::H / TZ;
  constexpr T ws = T(w_scale<NN>());
  spec = slot_ptr(spec, bs);
  wspec = slot_ptr(wspec, bs);
  twg = slot_ptr(twg, bs);
  kv = slot_ptr(kv, bs);
  ctl = slot_ptr(ctl, bs);
  if (ctl->stop) return;
  extern __shared__ __align__(16) unsigned char smem[];
  V* pub = reinterpret_cast<V*>(smem);
  V* tw = pub + C::MPR * C::SLOT;
  T* kz = reinterpret_cast<T*>(tw + n);
  const int lt = xcd_tile(blockIdx.x, gridDim.x);
  const int Q = lt & 1, tile = lt >> 1;
  const int ky = tile / NT, kx0 = (tile - ky * NT) * TZ;
  for (int i = threadIdx.x; i < n; i += C::BT) {
    tw[i] = twg[i];
    kz[i] = -ws * (kv[i] / T(n));
  }
  T kxs[C::VW];
#pragma unroll
  for (int v = 0; v < C::VW; ++v) kxs[v] = ws * kv[kx0 + (int(threadIdx.x) * C::VW) % TZ + v];
  const T kys = ws * kv[ky];
  const size_t off = C::Lay::row(ky) + kx0;
  lds_barrier();
  if (Q == 0) sweep<C, T, N, 0>(spec + off, wspec + off, pub, tw, kz, kxs, kys);
  else sweep<C, T, N, 1>(spec + off, wspec + off, pub, tw, kz, kxs, kys);
}

}  // namespace strm
}  // namespace rte
