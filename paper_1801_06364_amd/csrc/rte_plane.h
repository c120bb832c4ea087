// Plane passes of grids up to 128 points per axis.
//
// Inverse pass, per (moment, z-plane): inverse y FFT of the xy spectrum,
// complex-to-real merge, inverse x FFT, the pointwise epilogue (loss,
// in-scatter, boundary layer, source, RK combine; eqs. (9), (11), (12)) and,
// fused, the forward transform of the output plane (the next stage's
// spectrum). The transform stages that touch HBM stay in registers:
//
//   columns (n points, y): L lanes per column, P = n / L points each, lanes
//     along kx; the first stage reads its inputs straight from HBM and the
//     forward's last stage writes straight to HBM;
//   rows (H = n / 2 packed points, x): RL lanes of one wavefront per row,
//     H = Ra Rb, Ra = RL NB; stage one (radix Ra) reads X_k and X_{H-k} and
//     merges them on the way in; the real-to-complex split of the forward is
//     done by the column stage that reads the rows' results (its twiddle
//     depends on the lane's kx only), so neither costs a pass over the plane;
//   epilogue: a wavefront owns RW = 64 / RL consecutive rows, one contiguous
//     piece of every field, and works them off in memory order from LDS, 1 KB
//     per access. The row transform's own lane order would touch 16 to 32
//     bytes of 16 to 32 rows at a time: 96^3 P_7 FP32 317 -> 237 us, 96^3 P_5
//     FP64 415 -> 277, 128^3 P_7 FP64 1257 -> 1145, 64^3 P_7 FP32 69 -> 59,
//     48^3 P_3 FP32 (eight solves) 57 -> 47 per fused middle pass.
//
// The plane sits in LDS with an odd row pitch: the 16 lanes of one LDS cycle
// touch 16 consecutive columns of a row or one column of 16 rows. The epilogue's
// items are two consecutive elements per lane (FP32), so its lanes lie two elements
// apart: 0.62 conflict cycles per LDS instruction of the pass at 128^3 P_7, beside
// the loads from HBM that it waits for.
//
// Bound: HBM (5F + maps per fused middle pass, F = M n^3 elements), 4.6-5.0
// TB/s where the fields exceed the Infinity Cache and 5.3-6.0 where they do
// not; skipping every butterfly changes that by 3%. Fused middle pass against
// the pass with one LDS round trip per Stockham stage that it replaces:
// 64^3 P_7 FP32 83 -> 60 us (Euler), 48^3 P_3 (eight solves) 111 -> 47, 96^3 P_3
// 91 -> 53, 48^3 P_4 FP64 47 -> 27, 128^3 P_7 FP64 1363 -> 1145; 128^3 P_7 FP32
// (a 128-point schedule of its own before) 582 -> 578.
#pragma once

namespace rte {
namespace pln {

// Lanes per column and column radices (forward order; the inverse takes them
// in reverse), lanes per row, row radices, planes per workgroup. 8 to 16
// points per lane where they give whole butterflies on both axes; fewer lanes
// with more points (16 at 64, 24 at 96) measured 10% slower or the same, and at
// 32^3 FP64, where few wavefronts run, four points beat eight (5.1 against 7.4
// us for four moments).
struct Plan {
  int L, C[3], nc, RL, Ra, Rb, PPW;
};
template <typename T> __host__ __device__ constexpr Plan plan_of(int n) {
  const bool f = sizeof(T) == 4;
  switch (n) {
    case 16: return {4, {4, 4, 1}, 2, 2, 4, 2, 2};
    case 32: return f ? Plan{4, {8, 4, 1}, 2, 2, 4, 4, 1} : Plan{8, {4, 4, 2}, 3, 4, 4, 4, 1};
    case 48: return {4, {12, 4, 1}, 2, 2, 4, 6, 2};
    case 64: return {8, {8, 8, 1}, 2, 4, 8, 4, 1};
    case 96: return {8, {12, 2, 4}, 3, 4, 12, 4, 1};
    default: return {8, {16, 8, 1}, 2, 4, 8, 8, 1};
  }
}


template <typename T, int NN> struct Cfg {
  using V = typename cplx_of<T>::type;
  using Spec = SpecLayout<T, NN>;
  static constexpr Plan pl = plan_of<T>(NN);
  static constexpr int n = NN, H = NN / 2, L = pl.L, P = n / L, PITCH = H + 1;
  static constexpr int RL = pl.RL, Ra = pl.Ra, Rb = pl.Rb, PR = H / RL, NB = PR / Rb;
  static constexpr int PT = L * H;                 // threads per plane
  static constexpr int PPW = pl.PPW, BT = PT * PPW;
  static constexpr int RW = 64 / RL;               // rows per wavefront
  static constexpr int CW = 8 / int(sizeof(T));    // packed elements per 16-byte epilogue access
  static constexpr int ITEMS = PR / CW;            // epilogue accesses per lane and field
  // items whose loads are in flight together: all of up to four, else two in
  // FP32 (four measured 8% slower at 96^3) and four in FP64 (3% faster)
  static constexpr int BATCH = ITEMS <= 4 ? ITEMS : (sizeof(T) == 4 ? 2 : 4);
  static constexpr int PSIZE = n * PITCH;          // plane in LDS
  static constexpr size_t lds() {
    const size_t b = size_t(PSIZE * PPW + n) * sizeof(V);
    return b < size_t(2 * BT * 8) ? size_t(2 * BT * 8) : b;
  }
  static_assert(PR * RL == H && Ra * Rb == H && Ra == RL * NB && PT == RL * n, "rows and columns of one thread count");
  static_assert(BT % 64 == 0 && PR % Ra == 0, "whole wavefronts, whole butterflies");
  static_assert(ITEMS % BATCH == 0 && H % CW == 0, "whole batches, rows of whole accesses");
  // waves per SIMD that the LDS planes allow (at most four: 128 registers)
  static constexpr int waves() {
    const int w = int(160 * 1024 / lds()) * (BT / 64) / 4;
    return w < 1 ? 1 : (w > 4 ? 4 : w);
  }
};

template <int DIR, typename V> __device__ __forceinline__ V twd(V w) {
  if constexpr (DIR > 0) w.y = -w.y;
  return w;
}

// Column stages ST.. (S: product of the radices done). x: inputs of stage ST,
// [t][r] = row j + r n / R of butterfly j = l + L t; on return the last
// stage's outputs [t][q] = row j + q n / R. col: the lane's column in LDS.
// FRESH: nobody reads the plane any more when the first write comes.
template <class C, int DIR, bool FRESH, int ST = 0, int S = 1>
__device__ __forceinline__ void columns(typename C::V* x, typename C::V* col, int l, const typename C::V* tw) {
  using V = typename C::V;
  constexpr int n = C::n, L = C::L, P = C::P, NS = C::pl.nc;
  constexpr int R = DIR < 0 ? C::pl.C[ST] : C::pl.C[NS - 1 - ST];
  constexpr int SPAN = n / (S * R);
#pragma unroll
  for (int t = 0; t < P / R; ++t) {
    if constexpr (S > 1) {
      const int k = (l + L * t) % S;
#pragma unroll
      for (int r = 1; r < R; ++r) x[t * R + r] = cmul(x[t * R + r], twd<DIR>(tw[r * k * SPAN]));
    }
    Bfly<V, R, DIR>::run(x + t * R);
  }
  if constexpr (ST + 1 < NS) {
    constexpr int R2 = DIR < 0 ? C::pl.C[ST + 1] : C::pl.C[NS - 2 - ST];
    if constexpr (!FRESH) __syncthreads();
#pragma unroll
    for (int t = 0; t < P / R; ++t) {
      const int j = l + L * t;
      V* o = col + ((j / S) * S * R + j % S) * C::PITCH;
#pragma unroll
      for (int q = 0; q < R; ++q) o[q * S * C::PITCH] = x[t * R + q];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < P / R2; ++t)
#pragma unroll
      for (int r = 0; r < R2; ++r) x[t * R2 + r] = col[(l + L * t + r * (n / R2)) * C::PITCH];
    columns<C, DIR, false, ST + 1, S * R>(x, col, l, tw);
  }
}

// Complex-to-real merge of X_k with its partner X_{H-k}:
// (P + conj Q) + i conj(w) (P - conj Q), w = exp(-2 pi i k / n).
template <typename V> __device__ __forceinline__ V merge_inv(V p, V q, V w) {
  const auto dx = p.x - q.x, dy = p.y + q.y;
  const auto ex = w.x * dx + w.y * dy, ey = w.x * dy - w.y * dx;
  return cmk<V>(p.x + q.x - ey, p.y - q.y + ex);
}
// Real-to-complex split: (P + conj Q)/2 - i w (P - conj Q)/2.
template <typename V> __device__ __forceinline__ V split_fwd(V p, V q, V w) {
  using T = decltype(V::x);
  const T ex = T(0.5) * (p.x + q.x), ey = T(0.5) * (p.y - q.y);
  const T ox = T(0.5) * (p.y + q.y), oy = T(-0.5) * (p.x - q.x);
  return cmk<V>(ex + w.x * ox - w.y * oy, ey + w.x * oy + w.y * ox);
}

// Forward transform of the plane whose packed rows the lanes hold:
// c[i Rb + r] = element (t NB + i) + Ra r of row `row` (in LDS, no lane reads
// the plane any more), to the spectrum fd.
template <class C>
__device__ __forceinline__ void forward(typename C::V* c, typename C::V* plane, typename C::V* row, int t, int kx,
                                        int l, const typename C::V* tw, typename C::V* fd) {
  using V = typename C::V;
  using Spec = typename C::Spec;
  constexpr int n = C::n, H = C::H, L = C::L, P = C::P, Ra = C::Ra, Rb = C::Rb, NB = C::NB, RL = C::RL;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    Bfly<V, Rb, -1>::run(c + i * Rb);
#pragma unroll
    for (int q = 0; q < Rb; ++q) row[(t * NB + i) * Rb + q] = c[i * Rb + q];
  }
  wave_sync();
  {
    constexpr int NA = C::PR / Ra;
    V v[NA * Ra];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int r = 0; r < Ra; ++r) v[i * Ra + r] = row[t + RL * i + Rb * r];
    wave_sync();
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int j = t + RL * i;
#pragma unroll
      for (int r = 1; r < Ra; ++r) v[i * Ra + r] = cmul(v[i * Ra + r], tw[2 * r * j]);
      Bfly<V, Ra, -1>::run(v + i * Ra);
#pragma unroll
      for (int q = 0; q < Ra; ++q) row[j + Rb * q] = v[i * Ra + q];
    }
  }
  __syncthreads();
  // columns: the split on the way in
  constexpr int R0 = C::pl.C[0], RK = C::pl.C[C::pl.nc - 1];
  V x[P];
  const V wk = tw[kx];
  const V* a = plane + kx;
  const V* b = plane + (kx ? H - kx : 0);
#pragma unroll
  for (int s = 0; s < P / R0; ++s)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const int o = (l + L * s + r * (n / R0)) * C::PITCH;
      const V p = a[o], q = b[o];
      const V y = split_fwd(p, q, wk);
      x[s * R0 + r] = kx ? y : cmk<V>(p.x + p.y, p.x - p.y);   // kx = 0 packs (X_0, X_{n/2})
    }
  columns<C, -1, false>(x, plane + kx, l, tw);
  V* d = fd + Spec::row(l) + kx;
#pragma unroll
  for (int s = 0; s < P / RK; ++s)
#pragma unroll
    for (int q = 0; q < RK; ++q) d[Spec::row(L * s + q * (n / RK))] = x[s * RK + q];
}

// CW packed elements: 16 bytes
template <typename C, typename T> struct alignas(2 * C::CW * sizeof(T)) Item { T v[2 * C::CW]; };

// Standalone forward transform of real planes, plane index b n + z.
template <typename T, int NN>
__global__ void __launch_bounds__((Cfg<T, NN>::BT), (Cfg<T, NN>::waves()))
k_fwd(const T* __restrict__ src, typename cplx_of<T>::type* __restrict__ spec,
      const typename cplx_of<T>::type* __restrict__ twg, const Ctl* __restrict__ ctl) {
  using C = Cfg<T, NN>;
  using V = typename C::V;
  using Spec = typename C::Spec;
  constexpr int n = NN, H = C::H;
  if (ctl->stop) return;
  extern __shared__ __align__(16) unsigned char smem[];
  V* tw = reinterpret_cast<V*>(smem);
  V* pls = tw + n;
  const int tid = threadIdx.x;
  for (int i = tid; i < n; i += C::BT) tw[i] = twg[i];
  const int ln = tid & 63, y0 = (tid >> 6) * C::RW, yy = y0 + ln % C::RW, t = ln / C::RW;   // row lane
  const int pr = yy / n, y = yy - pr * n;
  V* row = pls + pr * C::PSIZE + y * C::PITCH;
  // the wavefront's rows in memory order (its planes lie back to back)
  using I = Item<C, T>;
  const I* s = reinterpret_cast<const I*>(src + (size_t(blockIdx.x) * C::PPW * n + y0) * n);
  I x[C::ITEMS];
#pragma unroll
  for (int k = 0; k < C::ITEMS; ++k) x[k] = s[k * 64 + ln];
#pragma unroll
  for (int k = 0; k < C::ITEMS; ++k) {
    const int idx = k * 64 + ln, r = y0 + idx / (H / C::CW), p = r / n;
    V* lp = pls + p * C::PSIZE + (r - p * n) * C::PITCH + idx % (H / C::CW) * C::CW;
#pragma unroll
    for (int w = 0; w < C::CW; ++w) lp[w] = cmk<V>(x[k].v[2 * w], x[k].v[2 * w + 1]);
  }
  wave_sync();
  V c[C::PR];
#pragma unroll
  for (int i = 0; i < C::NB; ++i)
#pragma unroll
    for (int q = 0; q < C::Rb; ++q) c[i * C::Rb + q] = row[t * C::NB + i + C::Ra * q];
  __syncthreads();   // (the twiddles too)
  const int pc = tid / C::PT, ct = tid - pc * C::PT, kx = ct % H, l = ct / H;   // column lane
  const size_t cp = size_t(blockIdx.x) * C::PPW + pc;
  forward<C>(c, pls + pc * C::PSIZE, row, t, kx, l, tw, spec + cp / n * Spec::MS + cp % n * Spec::ZS);
}

template <typename T, int NN, int MODE, bool FUSE>
__global__ void __launch_bounds__((Cfg<T, NN>::BT), (Cfg<T, NN>::waves()))
k_plane(const typename cplx_of<T>::type* spec, const T* vin, T* u, T* dst, const T* __restrict__ sig,
        const T* __restrict__ q, const int* __restrict__ qflag, double* __restrict__ phi_int,
        double* __restrict__ partial, const typename cplx_of<T>::type* __restrict__ twg, int M, T h, T ws, double dt,
        const Ctl* __restrict__ ctl, int stage, long long step1, typename cplx_of<T>::type* fspec, long long bs) {
  using C = Cfg<T, NN>;
  using V = typename C::V;
  using Spec = typename C::Spec;
  constexpr int n = NN, H = C::H, L = C::L, P = C::P, Ra = C::Ra, Rb = C::Rb, NB = C::NB, RL = C::RL, CW = C::CW;
  spec = slot_ptr(spec, bs);
  vin = slot_ptr(vin, bs);
  u = slot_ptr(u, bs);
  dst = slot_ptr(dst, bs);
  sig = slot_ptr(sig, bs);
  q = slot_ptr(q, bs);
  qflag = slot_ptr(qflag, bs);
  phi_int = slot_ptr(phi_int, bs);
  partial = slot_ptr(partial, bs);
  twg = slot_ptr(twg, bs);
  ctl = slot_ptr(ctl, bs);
  fspec = slot_ptr(fspec, bs);
  if (ctl->stop) {
    if constexpr (MODE == EPI_LAST || MODE == EPI_EULER) hold_state<C::BT, C::PPW * n * n>(u, dst);
    return;
  }
  extern __shared__ __align__(16) unsigned char smem[];
  V* tw = reinterpret_cast<V*>(smem);
  V* pls = tw + n;
  const int tid = threadIdx.x;
  for (int i = tid; i < n; i += C::BT) tw[i] = twg[i];
  // logical order z-major, moment-minor: moments of one z-plane (which share
  // the loss maps) run back to back on one XCD, ZG planes side by side
  const int lt0 = xcd_tile(blockIdx.x, gridDim.x) * C::PPW;
  auto plane_of = [&](int p, int& b, int& z) {
    const int lt = lt0 + p, zg = lt / (M * Spec::ZG), rem = lt - zg * (M * Spec::ZG);
    b = rem / Spec::ZG;
    z = zg * Spec::ZG + rem % Spec::ZG;
  };
  // column lane: plane pc, column kx, butterflies l + L t
  const int pc = C::PPW == 1 ? 0 : tid / C::PT, ct = tid - pc * C::PT, kx = ct % H, l = ct / H;
  int cb, cz;
  plane_of(pc, cb, cz);
  const size_t soff = size_t(cb) * Spec::MS + size_t(cz) * Spec::ZS;
  V* plane = pls + pc * C::PSIZE;
  {
    constexpr int R0 = C::pl.C[C::pl.nc - 1], RK = C::pl.C[0];
    const V* sp = spec + soff + Spec::row(l) + kx;
    V x[P];
#pragma unroll
    for (int s = 0; s < P / R0; ++s)
#pragma unroll
      for (int r = 0; r < R0; ++r) x[s * R0 + r] = sp[Spec::row(L * s + r * (n / R0))];
    __syncthreads();   // the twiddles
    columns<C, +1, true>(x, plane + kx, l, tw);
#pragma unroll
    for (int s = 0; s < P / RK; ++s)
#pragma unroll
      for (int r = 0; r < RK; ++r) plane[kx + (l + L * s + r * (n / RK)) * C::PITCH] = x[s * RK + r];
  }
  __syncthreads();

  // row lane: plane pr, row y, lane t of RL
  const int ln = tid & 63, y0 = (tid >> 6) * C::RW, yy = y0 + ln % C::RW, t = ln / C::RW;
  const int pr = C::PPW == 1 ? 0 : yy / n, y = yy - pr * n;
  V* row = pls + pr * C::PSIZE + y * C::PITCH;
  constexpr bool kLast = (MODE == EPI_LAST || MODE == EPI_EULER);
  constexpr bool kAdj = (MODE == EPI_ADJ || MODE == EPI_ADJL);
  constexpr bool kSrc = kLast || MODE == EPI_FIRST || MODE == EPI_MID;
  V c[C::PR];
  {
    constexpr int NA = C::PR / Ra;
    V v[NA * Ra];
    // inverse x, stage 1 (radix Ra): butterflies t + RL i, merged on the way in
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int r = 0; r < Ra; ++r) {
        const int e = t + RL * i + Rb * r;
        const V p = row[e], o = row[e ? H - e : 0];
        const V m = merge_inv(p, o, tw[e]);
        v[i * Ra + r] = (i == 0 && r == 0 && t == 0) ? cmk<V>(p.x + p.y, p.x - p.y) : m;
      }
    wave_sync();
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      Bfly<V, Ra, +1>::run(v + i * Ra);
#pragma unroll
      for (int k = 0; k < Ra; ++k) row[(t + RL * i) * Ra + k] = v[i * Ra + k];
    }
  }
  wave_sync();
  // stage 2 (radix Rb): butterflies t NB + i
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int j = t * NB + i;
#pragma unroll
    for (int r = 0; r < Rb; ++r) c[i * Rb + r] = row[j + Ra * r];
#pragma unroll
    for (int r = 1; r < Rb; ++r) c[i * Rb + r] = cmul(c[i * Rb + r], twd<+1>(tw[2 * r * j]));
    Bfly<V, Rb, +1>::run(c + i * Rb);
  }
  wave_sync();

  // epilogue: one 16-byte access per item and field, BATCH items in flight.
  // The wavefront's RW rows go back to LDS and are worked off in memory order
  // (lane ln: item 64 k + ln), so that every access covers 1 KB of HBM
  double acc_d[C::PPW], acc_o[C::PPW];
  int pb[C::PPW], pz[C::PPW], psig[C::PPW];   // the planes: moment, z, loss map offset
  T pq[C::PPW];                               // source weight
  bool phq[C::PPW];                           // source present
#pragma unroll
  for (int p = 0; p < C::PPW; ++p) {
    acc_d[p] = acc_o[p] = 0.0;
    plane_of(p, pb[p], pz[p]);
    psig[p] = isqrt_c(pb[p]) * n * n * n;
    phq[p] = kSrc && (q != nullptr) && qflag[pb[p] * n + pz[p]];
    pq[p] = phq[p] ? T(source_weight(ctl, stage, step1)) : T(0);
  }
  auto of = [](const auto* v, int p) { return C::PPW == 1 || p == 0 ? v[0] : v[C::PPW - 1]; };
  static_assert(C::PPW <= 2, "two planes are told apart");
  {
    constexpr int IR = H / CW;   // items per row
    using I = Item<C, T>;
    wave_sync();
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int q = 0; q < Rb; ++q) row[t * NB + i + Ra * q] = c[i * Rb + q];
    wave_sync();
#pragma unroll
    for (int k0 = 0; k0 < C::ITEMS; k0 += C::BATCH) {
      if (k0 > 0) asm volatile("" ::: "memory");
      I uu[C::BATCH], vv[C::BATCH], ss[C::BATCH], qq[C::BATCH];
      size_t po[C::BATCH];
      int vo[C::BATCH], lo[C::BATCH], pp[C::BATCH];
#pragma unroll
      for (int k = 0; k < C::BATCH; ++k) {
        const int idx = (k0 + k) * 64 + ln, r = y0 + idx / IR, e = idx % IR;   // row of the workgroup, item in it
        const int p = C::PPW == 1 ? 0 : r / n, yr = r - p * n;
        pp[k] = p;
        lo[k] = p * C::PSIZE + yr * C::PITCH + e * CW;
        vo[k] = (of(pz, p) * n + yr) * n + e * 2 * CW;
        po[k] = size_t(of(pb, p)) * (n * n * n) + vo[k];
        if constexpr (MODE != EPI_SET) {
          if constexpr (MODE != EPI_APPLY) uu[k] = *reinterpret_cast<const I*>(u + po[k]);
          if constexpr (MODE == EPI_FIRST || MODE == EPI_EULER) vv[k] = uu[k];
          else vv[k] = *reinterpret_cast<const I*>(vin + po[k]);
          ss[k] = *reinterpret_cast<const I*>(sig + of(psig, p) + vo[k]);
          if (of(phq, p)) {
            qq[k] = *reinterpret_cast<const I*>(q + po[k]);
          } else {
#pragma unroll
            for (int w = 0; w < 2 * CW; ++w) qq[k].v[w] = T(0);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < C::BATCH; ++k) {
        V* lp = pls + lo[k];
        I o;
#pragma unroll
        for (int w = 0; w < 2 * CW; ++w) {
          const T x = (w & 1) ? lp[w / 2].y : lp[w / 2].x;
          if constexpr (MODE == EPI_SET) {
            o.v[w] = x;
          } else {
            T s = -ss[k].v[w] * vv[k].v[w];
            if constexpr (!kAdj) s += of(pq, pp[k]) * qq[k].v[w];
            if constexpr (MODE == EPI_APPLY) o.v[w] = ss[k].v[w] * vv[k].v[w] - ws * x;
            else if constexpr (kAdj) o.v[w] = ws * x + h * s;
            else o.v[w] = uu[k].v[w] + ws * x + h * s;
          }
        }
        if constexpr (MODE != EPI_ADJL) *reinterpret_cast<I*>(dst + po[k]) = o;
        if constexpr (kAdj) {
          I a;
#pragma unroll
          for (int w = 0; w < 2 * CW; ++w) a.v[w] = uu[k].v[w] + o.v[w];
          *reinterpret_cast<I*>(u + po[k]) = a;
        }
        if constexpr (kLast) {
          if (of(pb, pp[k]) == 0) {
            double d2 = 0.0, o2 = 0.0;
#pragma unroll
            for (int w = 0; w < 2 * CW; ++w) {
              phi_int[vo[k] + w] += dt * double(o.v[w]);
              const double d = double(o.v[w]) - double(uu[k].v[w]);
              d2 += d * d;
              o2 += double(o.v[w]) * double(o.v[w]);
            }
#pragma unroll
            for (int p = 0; p < C::PPW; ++p) {
              acc_d[p] += pp[k] == p ? d2 : 0.0;
              acc_o[p] += pp[k] == p ? o2 : 0.0;
            }
          }
        }
        if constexpr (FUSE) {
#pragma unroll
          for (int w = 0; w < CW; ++w) lp[w] = cmk<V>(o.v[2 * w], o.v[2 * w + 1]);
        }
      }
    }
    if constexpr (FUSE) {
      wave_sync();
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int q = 0; q < Rb; ++q) c[i * Rb + q] = row[t * NB + i + Ra * q];
      wave_sync();
    }
  }
  if constexpr (FUSE) forward<C>(c, plane, row, t, kx, l, tw, fspec + soff);
  // fluence-change partial sums of the planes of moment 0 (block_sum2 reuses
  // the LDS: it synchronises first)
  if constexpr (kLast) {
#pragma unroll
    for (int p = 0; p < C::PPW; ++p) {
      if (pb[p] == 0) {
        block_sum2<C::BT>(smem, acc_d[p], acc_o[p], partial + 2 * pz[p]);
        if (C::PPW > 1) __syncthreads();
      }
    }
  }
}

}  // namespace pln
}  // namespace rte
