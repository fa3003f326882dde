// The scaled grids of the modified methods (Sect. 7, Appendix B) plane by
// plane: passes X, YZ, IX of plane.hip for a level's N cells of the finer
// spacing on a period of C NP points and N outputs of level l's spacing, each
// the mean of S fine ones per axis.
//
// The N inputs and the S N cells they act on are (S + 1) N / 2 apart at most
// either way, so (S + 1) N points do: C = 3 classes for a doubled grid (S = 2),
// 5 for a quadrupled one (S = 4), of NP >= N points each - 0.42 and 0.24 of the
// points of the power-of-two periods 4N and 8N.  The means are taken in the
// spectrum (fold_pair), which keeps the classes apart: the points folded onto
// one another, P / S apart, are of one class, NP / S apart in it.  A class is
// then inverted on NP / S points, and its part of output p is w_Q^(-B p), Q =
// P / S, times the value at p mod NP / S: S outputs NP / S apart share one
// factor, up to turns by C-ths.
//
// 64^3 x 5: modified FP64 251 -> 160 us, three-level FP32 672 -> 220 us a
// solve against five passes at the periods 256 and 512.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "plane_device.hpp"

namespace nmc {

// One axis of a scaled grid: inputs at points ilo .. ilo + n - 1 (ilo = 0, or 2
// where S = 4 and N / 4 is odd, so that a mean starts at a multiple of S),
// outputs at points olo .. olo + n - 1 of the period Q.
template <int NP, int S>
struct ScaledAxis {
  using P = ClassPlan<NP>;
  static constexpr int N = NP, CL = S + 1, PER = CL * NP, H = PER / 2 + 1;
  static constexpr int NPC = NP / S, EF = P::E / S, Q = PER / S;
  static constexpr int QXI = S == 4 ? (2 + P::TL - 1) / P::TL : 0;
  static constexpr int RS = NP + P::R2, TPP = NP * P::TL, LINE = CL * RS + 1;
  static constexpr int NT = TPP < 64 ? 64 : TPP, PPW = NT / TPP;  // YZ: threads and planes per workgroup
};
__host__ __device__ constexpr int scaled_ilo(int N, int S) { return S == 4 && N % 8 ? 2 : 0; }
__host__ __device__ constexpr int scaled_olo(int N, int S) { return -((S - 1) * N / 2 - scaled_ilo(N, S)) / S; }

// One line's inverse transform of NPC points, EF per thread, exchanged within
// its own storage by lanes of one wavefront.
template <class R>
struct FlatView {
  cplx<R>* a;
  int SN;
  __device__ __forceinline__ void put(int n, cplx<R> v) const { a[n * SN] = v; }
  __device__ __forceinline__ cplx<R> get(int n) const { return a[n * SN]; }
};
template <class R, int NPC, int EF>
__device__ __forceinline__ void small_inv(cplx<R>* u, int t, const FlatView<R>& lv, const cplx<R>* tws) {
  using LV = FlatView<R>;
  auto go = [&]<int... RAD>(std::integer_sequence<int, RAD...>) {
    fft_stages<R, NPC, EF, +1, 1, true, false, false, true, LV, RAD...>(u, t, lv, tws);
  };
  if constexpr (EF == 8) go(std::integer_sequence<int, 8, NPC / 8>{});
  else if constexpr (EF == 4 && NPC == 4) go(std::integer_sequence<int, 4>{});
  else if constexpr (EF == 4 && NPC == 8) go(std::integer_sequence<int, 4, 2>{});
  else if constexpr (EF == 4 && NPC == 16) go(std::integer_sequence<int, 4, 4>{});
  else if constexpr (EF == 4 && NPC == 32) go(std::integer_sequence<int, 4, 4, 2>{});
  else if constexpr (EF == 2 && NPC == 2) go(std::integer_sequence<int, 2>{});
  else if constexpr (EF == 2 && NPC == 4) go(std::integer_sequence<int, 2, 2>{});
  else if constexpr (EF == 2 && NPC == 8) go(std::integer_sequence<int, 2, 2, 2>{});
  else {
    static_assert(EF == 2 && NPC == 16, "plan");
    go(std::integer_sequence<int, 2, 2, 2, 2>{});
  }
}

// Class b of a line's spectrum, w[q] = X[C (t + TL q) + b], to its part of the
// line's outputs: folded S times shorter, inverted, and u[q] the part of output
// rn = (t + TL q - olo) mod NPC, point p = rn + olo, ph[q] = S b p mod PER; that
// of output rn + s NPC is w_C^(-s b) times it.
template <class R, class AX, int S>
__device__ __forceinline__ void scaled_part(const cplx<R>* w, int b, int t, const FlatView<R>& lv,
                                            const cplx<R>* tw, const cplx<R>* tws, const int* ph, cplx<R>* u) {
  using T = cplx<R>;
  constexpr int EF = AX::EF, TL = AX::P::TL;
#pragma unroll
  for (int q = 0; q < EF; ++q) {
    const int k = AX::CL * (t + TL * q) + b;
    if constexpr (S == 2) {
      u[q] = fold_pair<R>(w[q], w[q + EF], tw[k], (R)0.5);
    } else {
      const T lo = fold_pair<R>(w[q], w[q + 2 * EF], tw[k], (R)0.5);
      const T hi = fold_pair<R>(w[q + EF], w[q + 3 * EF], tw[k + AX::Q], (R)0.5);
      u[q] = fold_pair<R>(lo, hi, tw[2 * k], (R)0.5);
    }
  }
  small_inv<R, AX::NPC, EF>(u, t, lv, tws);
  if (b) {
#pragma unroll
    for (int q = 0; q < EF; ++q) u[q] = c_mul_tw<+1>(u[q], tw[ph[q]]);
  }
}
// v exp(2 pi i s b / C), b of a wavefront.
template <class AX, class T>
__device__ __forceinline__ T turned(T v, int s, int b, const T* tw) {
  return s == 0 || b == 0 ? v : c_mul_tw<+1>(v, tw[s * b % AX::CL * AX::N]);
}

// Output index of slot s EF + q, and S p mod PER.
template <class AX, int S>
__device__ __forceinline__ int scaled_out_index(int t, int i, int olo) {
  const int s = i / AX::EF, q = i % AX::EF;
  return ((t + AX::P::TL * q - olo) & (AX::NPC - 1)) + s * AX::NPC;
}
template <class AX, int S>
__device__ __forceinline__ int scaled_phase(int r, int olo) {
  const int e = S * (r + olo);
  return e < 0 ? e + AX::PER : e >= AX::PER ? e - AX::PER : e;
}

// X: as for a level.
template <class R, int NP, int S>
__global__ void __launch_bounds__((x_threads<NP, S + 1>())) k_scaled_x(FieldTable ft, PlaneGeom g, PlaneTables<R> tb) {
  using AX = ScaledAxis<NP, S>;
  constexpr int NT = x_threads<NP, S + 1>();
  constexpr int LL = NT / AX::P::TL * AX::LINE;
  __shared__ cplx<R> lds[LL + AX::PER];
  x_body<R, AX, false, NT>(ft.f[blockIdx.y], g.N, g.N, scaled_ilo(g.N, S), lds, lds + LL, tb.tw);
}

// YZ: as for a level (one class a of ky per workgroup), the z spectrum folded
// and inverted class by class, then the y spectrum.
template <class R, int NP, int S>
__global__ void __launch_bounds__((ScaledAxis<NP, S>::NT), (sizeof(R) == 4 ? 4 : 2))
k_scaled_yz(FieldTable ft, PlaneGeom g, PlaneTables<R> tb) {
  using T = cplx<R>;
  using AX = ScaledAxis<NP, S>;
  using P = ClassPlan<NP>;
  constexpr int C = AX::CL, TL = P::TL, E = P::E, EF = AX::EF, RS = AX::RS, H = AX::H, NT = AX::NT;
  constexpr int WZ = 64 / TL < NP ? 64 / TL : NP;  // columns per wavefront
  __shared__ T lds[AX::PPW * NP * RS + AX::PER + AX::NPC];
  T* const tw = lds + AX::PPW * NP * RS;
  T* const tws = tw + AX::PER;  // exp(-2 pi i j / NPC)
  const int b = blockIdx.x, s8 = b / 8, f = s8 / C % g.nfull, group = s8 / (C * g.nfull) * 8 + b % 8, a = s8 % C;
  if (group * AX::PPW >= H) return;  // uniform
  const FieldDesc& F = ft.f[f];
  const int n = g.N, ilo = scaled_ilo(n, S), olo = scaled_olo(n, S);
  const int pi = threadIdx.x / AX::TPP, lt = threadIdx.x % AX::TPP;
  const int kx0 = group * AX::PPW + pi;
  const bool active = kx0 < H;
  const int kx = active ? kx0 : 0;
  const bool dc = kx == 0, ny = kx == AX::PER / 2;  // stored plane 0 holds both (plane.hip)
  const int ks = ny ? 0 : kx;
  T* const plane = lds + pi * (NP * RS);
  const T* const A = static_cast<const T*>(F.A) + (size_t)ks * n * n;
  T* const O = static_cast<T*>(F.B) + ((size_t)a * (AX::PER / 2) + ks) * n * n;
  const int ty = lt % TL, r = lt / TL;                                  // rows: lanes along y
  const int cz = (lt / (WZ * TL)) * WZ + lt % WZ, tz = (lt / WZ) % TL;  // columns: lanes along ky, then z
  const R sc = (R)F.scale;
  T v[E + AX::QXI];
  {
    const TableStage<R, AX::PER, NT> tws0(tb.tw);
    const T* const src = A + (size_t)(r < n ? r : 0) * n;
#pragma unroll
    for (int q = 0; q < E + AX::QXI; ++q) {
      const int i = ty + TL * (q < E ? q : q - E) + (q < E ? 0 : NP) - ilo;
      const bool in = r < n && (unsigned)i < (unsigned)n;
      const T x = src[in ? i : 0];
      v[q] = in ? x : T{0, 0};
    }
    if (dc || ny) {
#pragma unroll
      for (int q = 0; q < E + AX::QXI; ++q) v[q] = T{dc ? v[q].x : v[q].y, 0};
    }
    tws0.put(tw);
    for (int j = threadIdx.x; j < AX::NPC; j += NT) tws[j] = tb.tw[C * S * j];
  }
  __syncthreads();
  const LineStore<R, P::R1, true> row{plane + r * RS, 1};
  static_for(std::make_integer_sequence<int, C>{}, [&](auto B) {
    if (a != B) return;
#pragma unroll
    for (int q = 0; q < AX::QXI; ++q) v[q] = c_add(v[q], c_turn<-1, B, C>(v[E + q]));
    class_fwd<R, NP, C, B, true>(v, ty, row, tw);
  });
#pragma unroll
  for (int q = 0; q < E; ++q) *row.at(ty + TL * q) = v[q];  // zero in rows n and above, which were loaded as zeros
  const unsigned gy = (unsigned)(kx * H * H + class_pos<NP, C>(a, cz));
  auto spectrum = [&](int c, R* gv) {  // plane.hip
    const unsigned glo = gy + class_pos<NP, C>(c, 0) * H + tz * H;
    const unsigned ghi = gy + class_pos<NP, C>(c, NP / 2) * H - tz * H;
#pragma unroll
    for (int q = 0; q < E; ++q) gv[q] = tb.gp[q < E / 2 ? glo + q * (TL * H) : ghi - (q - E / 2) * (TL * H)];
  };
  R gv[E];
  spectrum(0, gv);
  __syncthreads();
  {  // columns
    T* const col = plane + cz + cz / P::R1;
    T x[E + AX::QXI], acc[E];
#pragma unroll
    for (int q = 0; q < E + AX::QXI; ++q) {
      const int i = tz + TL * (q < E ? q : q - E) + (q < E ? 0 : NP) - ilo;
      const bool in = AX::QXI == 0 || (unsigned)i < (unsigned)n;
      const T u = col[(in ? i : 0) * RS];
      x[q] = in ? u : T{0, 0};
    }
    int e[EF], ph[EF];
#pragma unroll
    for (int i = 0; i < EF; ++i) {
      e[i] = scaled_phase<AX, S>(scaled_out_index<AX, S>(tz, i, olo), olo);
      ph[i] = 0;
    }
    const LineStore<R, P::R1, false> st{col, RS};
    static_for(std::make_integer_sequence<int, C>{}, [&](auto B) {
      if (B > 0) spectrum(B, gv);
      T w[E], u[EF];
#pragma unroll
      for (int q = 0; q < E; ++q) w[q] = q < AX::QXI ? c_add(x[q], c_turn<-1, B, C>(x[E + q])) : x[q];
      class_fwd<R, NP, C, B, false>(w, tz, st, tw);
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const R s = sc * gv[q];
        w[q] = T{w[q].x * s, w[q].y * s};
      }
      scaled_part<R, AX, S>(w, B, tz, FlatView<R>{col, RS}, tw, tws, ph, u);
      static_for(std::make_integer_sequence<int, S>{}, [&](auto s) {
#pragma unroll
        for (int q = 0; q < EF; ++q) {
          const T v = c_turn<+1, (int)B * (int)s % C, C>(u[q]);
          acc[s * EF + q] = B == 0 ? v : c_add(acc[s * EF + q], v);
        }
      });
#pragma unroll
      for (int q = 0; q < EF; ++q) {
        ph[q] += e[q];
        if (ph[q] >= AX::PER) ph[q] -= AX::PER;
      }
    });
    wave_order();
#pragma unroll
    for (int i = 0; i < E; ++i) col[scaled_out_index<AX, S>(tz, i, olo) * RS] = acc[i];  // rows n and above: unread
  }
  __syncthreads();
  {  // rows back to y
    T w[E], u[EF];
    int ph[EF];
#pragma unroll
    for (int q = 0; q < E; ++q) w[q] = *row.at(ty + TL * q);
#pragma unroll
    for (int i = 0; i < EF; ++i)
      ph[i] = scaled_phase<AX, S>(scaled_out_index<AX, S>(ty, i, olo), olo) * a % AX::PER;
    wave_order();
    scaled_part<R, AX, S>(w, a, ty, FlatView<R>{plane + r * RS, 1}, tw, tws, ph, u);
    if (active && r < n) {
      T* const dst = O + (size_t)r * n;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int y = scaled_out_index<AX, S>(ty, i, olo);
        if (y >= n) continue;
        const T v = turned<AX>(u[i % EF], i / EF, a, tw);
        if (dc) dst[y].x = v.x;
        else if (ny) dst[y].y = v.x;
        else dst[y] = v;
      }
    }
  }
}

// IX: two rows per complex line (plane.hip), folded and inverted, each class by
// its own wavefronts; the means, with the carry S when set, are added to out.
// One class after the other in a wavefront took 42 us on one grid of 24^3 (S = 4,
// FP64), 7.3 us this way, and 30 us on four of 64^3 (S = 2), 21 this way: LDS,
// which holds all classes of a workgroup's rows, bounds the workgroups in
// flight, and this is C times the wavefronts.
template <class R, int NP, int S, bool TRI>
__global__ void __launch_bounds__((S + 1) * (x_threads<NP, S + 1>())) k_scaled_ix(FieldTable ft, PlaneGeom g, PlaneTables<R> tb) {
  using T = cplx<R>;
  using AX = ScaledAxis<NP, S>;
  using P = ClassPlan<NP>;
  constexpr int C = AX::CL, TL = P::TL, E = P::E, EF = AX::EF, NT1 = x_threads<NP, C>(), NT = C * NT1, UW = NT1 / TL;
  __shared__ T lds[UW * AX::LINE + AX::PER + AX::NPC];
  T* const tw = lds + UW * AX::LINE;
  T* const tws = tw + AX::PER;
  const FieldDesc& F = ft.f[blockIdx.y];
  const int N = g.N, olo = scaled_olo(N, S), units = N * N / 2, u0 = blockIdx.x * UW;
  const size_t pl = (size_t)N * N;
  {
    const int ul = threadIdx.x % UW, k0 = threadIdx.x / UW;
    T* const ls = lds + ul * AX::LINE;
    const T* const src = static_cast<const T*>(F.B) + k0 * pl + (u0 + ul < units ? 2 * (size_t)(u0 + ul) : 0);
    constexpr int K = E / 2;  // stored planes 0 .. PER/2 - 1 in steps of C TL
    T va[K], vb[K];
    const TableStage<R, AX::PER, NT> tws0(tb.tw);
#pragma unroll
    for (int p = 0; p < C; ++p) {  // the classes' parts
      const T* const sp = src + p * (AX::PER / 2) * pl;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const T a = sp[C * TL * i * pl], b = sp[C * TL * i * pl + 1];
        va[i] = p == 0 ? a : c_add(va[i], a);
        vb[i] = p == 0 ? b : c_add(vb[i], b);
      }
    }
    tws0.put(tw);
    for (int j = threadIdx.x; j < AX::NPC; j += NT) tws[j] = tb.tw[C * S * j];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int k = k0 + C * TL * i;
      const T a = va[i], b = vb[i];
      const int ca = k % C, j = k / C;
      int ma, mj;
      class_mirror<NP, C>(ca, j, ma, mj);
      const int mi = k == 0 ? NP / 2 + NP / 2 / P::R1 : ma * AX::RS + mj + mj / P::R1;
      ls[mi] = k == 0 ? T{a.y, b.y} : T{a.x + b.y, b.x - a.y};
      ls[ca * AX::RS + j + j / P::R1] = k == 0 ? T{a.x, b.x} : T{a.x - b.y, a.y + b.x};
    }
  }
  __syncthreads();
  {
    const int b = __builtin_amdgcn_readfirstlane(threadIdx.x / NT1);
    const int t1 = threadIdx.x % NT1, u = t1 / TL, t = t1 % TL;
    T* const line = lds + u * AX::LINE + b * AX::RS;
    const LineStore<R, P::R1, true> st{line, 1};
    T w[E], v[EF];
    int ph[EF];
#pragma unroll
    for (int q = 0; q < E; ++q) w[q] = *st.at(t + TL * q);
#pragma unroll
    for (int i = 0; i < EF; ++i)
      ph[i] = scaled_phase<AX, S>(scaled_out_index<AX, S>(t, i, olo), olo) * b % AX::PER;
    wave_order();
    scaled_part<R, AX, S>(w, b, t, FlatView<R>{line, 1}, tw, tws, ph, v);
    wave_order();
#pragma unroll
    for (int i = 0; i < E; ++i)  // outputs N and above: unread
      line[scaled_out_index<AX, S>(t, i, olo)] = turned<AX>(v[i % EF], i / EF, b, tw);
  }
  __syncthreads();
  constexpr bool CARRY = S == 2;  // quadrupled grids add none
  const float inv = 1.0f / N;
  const int NS = N / 2 + 2;
  const R* const Sc = CARRY ? static_cast<const R*>(F.S) : nullptr;
  const R* const Sl = CARRY ? static_cast<const R*>(F.Slo) : nullptr;
  R* const out = static_cast<R*>(F.out);
  constexpr int K = (E + C - 1) / C;  // items (an x of a row pair) per thread at N = NP
  bool on[K];
  int at[K], lx[K], xx[K];
  CarryRows cr[K];
  R base[2][K], s1[2][K], l[2][K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = threadIdx.x + k * NT, u = small_div(i, N, inv), x = i - u * N;
    on[k] = u < UW && u0 + u < units;
    const int rw = on[k] ? 2 * (u0 + u) : 0, z = small_div(rw, N, inv), y = rw - z * N;
    at[k] = rw * N + x;
    lx[k] = (on[k] ? u : 0) * AX::LINE + x;
    xx[k] = x;
    cr[k] = carry_rows(z, y, NS);
    base[0][k] = out[at[k]];
    base[1][k] = out[at[k] + N];
    s1[0][k] = s1[1][k] = l[0][k] = l[1][k] = 0;
  }
  if (CARRY && Sc) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        CarryRows c = cr[k];  // of row y + 1: the same parent, the neighbour behind it
        if (h) c.jj += 2 * NS, c.dyn += 2 * NS;
        carried<R, TRI>(F.comp, Sc, Sl, c, xx[k], s1[h][k], l[h][k]);
      }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    T m = lds[lx[k]];
#pragma unroll
    for (int b = 1; b < C; ++b) m = c_add(m, lds[lx[k] + b * AX::RS]);
    if (on[k]) {
      out[at[k]] = scaled_sum<R>(F.comp, Sc != nullptr, base[0][k], m.x, s1[0][k], l[0][k]);
      out[at[k] + N] = scaled_sum<R>(F.comp, Sc != nullptr, base[1][k], m.y, s1[1][k], l[1][k]);
    }
  }
}

// ---------------------------------------------------------------------------
template <class R, class F>
static hipError_t dispatch_scaled(int N, int S, F&& f) {
  auto both = [&](auto np) {
    if (S == 2) f(np, std::integral_constant<int, 2>{});
    else f(np, std::integral_constant<int, 4>{});
  };
  switch (scaled_points<R>(N)) {
    case 8: both(std::integral_constant<int, 8>{}); break;
    case 16: both(std::integral_constant<int, 16>{}); break;
    case 32: both(std::integral_constant<int, 32>{}); break;
    case 64: both(std::integral_constant<int, 64>{}); break;
    case 128:
      if constexpr (sizeof(R) == 4) {
        both(std::integral_constant<int, 128>{});
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class R>
hipError_t launch_scaled_x(const FieldTable& ft, PlaneGeom g, int S, PlaneTables<R> tb, hipStream_t s) {
  return dispatch_scaled<R>(g.N, S, [&](auto np, auto sc) {
    constexpr int NP = decltype(np)::value, SS = decltype(sc)::value;
    constexpr int NT = x_threads<NP, SS + 1>(), UW = NT / ClassPlan<NP>::TL;
    launch(k_scaled_x<R, NP, SS>, dim3((g.N * g.N / 2 + UW - 1) / UW, g.nfull), dim3(NT), 0, s, ft, g, tb);
  });
}
template <class R>
hipError_t launch_scaled_yz(const FieldTable& ft, PlaneGeom g, int S, PlaneTables<R> tb, hipStream_t s) {
  return dispatch_scaled<R>(g.N, S, [&](auto np, auto sc) {
    constexpr int NP = decltype(np)::value, SS = decltype(sc)::value;
    using AX = ScaledAxis<NP, SS>;
    launch(k_scaled_yz<R, NP, SS>, dim3(plane_blocks(AX::H, AX::PPW, SS + 1, g.nfull)), dim3(AX::NT), 0, s, ft, g, tb);
  });
}
template <class R>
hipError_t launch_scaled_ix(const FieldTable& ft, PlaneGeom g, int S, PlaneTables<R> tb, hipStream_t s) {
  return dispatch_scaled<R>(g.N, S, [&](auto np, auto sc) {
    constexpr int NP = decltype(np)::value, SS = decltype(sc)::value;
    constexpr int NT = x_threads<NP, SS + 1>(), UW = NT / ClassPlan<NP>::TL;
    const dim3 grid((g.N * g.N / 2 + UW - 1) / UW, g.nfull);
    constexpr int C = SS + 1;
    if (SS == 2 && ft.f[0].tri) launch(k_scaled_ix<R, NP, 2, true>, grid, dim3(C * NT), 0, s, ft, g, tb);
    else launch(k_scaled_ix<R, NP, SS, false>, grid, dim3(C * NT), 0, s, ft, g, tb);  // quadrupled grids add no carry
  });
}

#define NMC_INSTANTIATE(R)                                                                                \
  template hipError_t launch_scaled_x<R>(const FieldTable&, PlaneGeom, int, PlaneTables<R>, hipStream_t); \
  template hipError_t launch_scaled_yz<R>(const FieldTable&, PlaneGeom, int, PlaneTables<R>, hipStream_t); \
  template hipError_t launch_scaled_ix<R>(const FieldTable&, PlaneGeom, int, PlaneTables<R>, hipStream_t);

NMC_INSTANTIATE(double)
NMC_INSTANTIATE(float)

}  // namespace nmc
