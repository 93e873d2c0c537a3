// FFT of one line spread over a few threads, its values in registers between the stages.
//
// A line of length M = R_1 R_2 (R_3) is transformed by TPL threads with one Stockham stage per
// radix (decimation in time): stage s reads its butterfly inputs jb + r M/R_s, applies the
// twiddles and a radix-R_s DFT in registers, and its outputs go to (jb / Ns) Ns R_s + k + r Ns,
// k = jb mod Ns, Ns the product of the earlier radices.  Radices of up to 16 leave one or two
// passes through LDS per transform: the first stage's inputs come straight from global memory
// and the last stage's outputs (jb + r Ns) go straight back.  The last stage holds exactly the
// inputs that the inverse transform with the radices in reverse order starts from, so a
// convolution multiplies in registers and turns around without LDS.
//
// Every index of a stage is a compile-time product or a shift; a line length known only at run
// time would cost an integer division per butterfly, which with four times the LDS passes made
// the runtime-length engine (fft_lds) take 37 us for the z convolution of a 64^3 grid.
#pragma once
#include <cmath>

#include "internal.hpp"

namespace pic {

template <typename T>
struct Cx {
  T x, y;
};

template <typename T>
struct TwT;
template <>
struct TwT<double> {
  using type = double2;
};
template <>
struct TwT<float> {
  using type = float2;
};

// complex load through the native vector type (a struct copy of a conditional load otherwise
// goes through scratch memory)
template <typename T>
__device__ __forceinline__ Cx<T> ld(const Cx<T>* p) {
  const typename TwT<T>::type t = *reinterpret_cast<const typename TwT<T>::type*>(p);
  return Cx<T>{t.x, t.y};
}

template <typename T>
__device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__host__ __device__ __forceinline__ Cx<T> cadd(Cx<T> a, Cx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__host__ __device__ __forceinline__ Cx<T> csub(Cx<T> a, Cx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ Cx<T> cconj(Cx<T> a) { return {a.x, -a.y}; }

// cos(2 pi t / 144), t = 0..143 (144 = lcm of the composite radices 6, 8, 9, 12, 16), from
// 40-digit mpmath; sin(2 pi t / 144) is entry t - 36
__host__ __device__ constexpr double cos144(int t) {
  constexpr double tab[144] = {
    1.0, 0.999048221581857762404, 0.996194698091745532295,
    0.991444861373810411145, 0.984807753012208059367, 0.976296007119933365971,
    0.96592582628906828675, 0.953716950748226921144, 0.939692620785908384054,
    0.923879532511286756128, 0.906307787036649963243, 0.887010833178221701055,
    0.866025403784438646764, 0.843391445812885701273, 0.819152044288991789684,
    0.79335334029123516458, 0.766044443118978035202, 0.737277336810124041384,
    0.707106781186547524401, 0.675590207615660244348, 0.642787609686539326323,
    0.608761429008720639416, 0.573576436351046096108, 0.537299608346823831841,
    0.5, 0.461748613235033930563, 0.422618261740699436187,
    0.382683432365089771728, 0.342020143325668733044, 0.300705799504273121623,
    0.258819045102520762349, 0.21643961393810287976, 0.173648177666930348852,
    0.130526192220051591548, 0.0871557427476581735581, 0.0436193873653359997818,
    0.0, -0.0436193873653359997818, -0.0871557427476581735581,
    -0.130526192220051591548, -0.173648177666930348852, -0.21643961393810287976,
    -0.258819045102520762349, -0.300705799504273121623, -0.342020143325668733044,
    -0.382683432365089771728, -0.422618261740699436187, -0.461748613235033930563,
    -0.5, -0.537299608346823831841, -0.573576436351046096108,
    -0.608761429008720639416, -0.642787609686539326323, -0.675590207615660244348,
    -0.707106781186547524401, -0.737277336810124041384, -0.766044443118978035202,
    -0.79335334029123516458, -0.819152044288991789684, -0.843391445812885701273,
    -0.866025403784438646764, -0.887010833178221701055, -0.906307787036649963243,
    -0.923879532511286756128, -0.939692620785908384054, -0.953716950748226921144,
    -0.96592582628906828675, -0.976296007119933365971, -0.984807753012208059367,
    -0.991444861373810411145, -0.996194698091745532295, -0.999048221581857762404,
    -1.0, -0.999048221581857762404, -0.996194698091745532295,
    -0.991444861373810411145, -0.984807753012208059367, -0.976296007119933365971,
    -0.96592582628906828675, -0.953716950748226921144, -0.939692620785908384054,
    -0.923879532511286756128, -0.906307787036649963243, -0.887010833178221701055,
    -0.866025403784438646764, -0.843391445812885701273, -0.819152044288991789684,
    -0.79335334029123516458, -0.766044443118978035202, -0.737277336810124041384,
    -0.707106781186547524401, -0.675590207615660244348, -0.642787609686539326323,
    -0.608761429008720639416, -0.573576436351046096108, -0.537299608346823831841,
    -0.5, -0.461748613235033930563, -0.422618261740699436187,
    -0.382683432365089771728, -0.342020143325668733044, -0.300705799504273121623,
    -0.258819045102520762349, -0.21643961393810287976, -0.173648177666930348852,
    -0.130526192220051591548, -0.0871557427476581735581, -0.0436193873653359997818,
    0.0, 0.0436193873653359997818, 0.0871557427476581735581,
    0.130526192220051591548, 0.173648177666930348852, 0.21643961393810287976,
    0.258819045102520762349, 0.300705799504273121623, 0.342020143325668733044,
    0.382683432365089771728, 0.422618261740699436187, 0.461748613235033930563,
    0.5, 0.537299608346823831841, 0.573576436351046096108,
    0.608761429008720639416, 0.642787609686539326323, 0.675590207615660244348,
    0.707106781186547524401, 0.737277336810124041384, 0.766044443118978035202,
    0.79335334029123516458, 0.819152044288991789684, 0.843391445812885701273,
    0.866025403784438646764, 0.887010833178221701055, 0.906307787036649963243,
    0.923879532511286756128, 0.939692620785908384054, 0.953716950748226921144,
    0.96592582628906828675, 0.976296007119933365971, 0.984807753012208059367,
    0.991444861373810411145, 0.996194698091745532295, 0.999048221581857762404,
  };
  return tab[t];
}

// a exp(DIR 2 pi i t / N) for t known at compile time (after unrolling), 0 <= t < N.
// In float32 the constants, here and in the radix-3 DFT, carry their rounding's rest: they are a
// few, met in every line of every pass, and their roundings alone left the direct field 1e-7 too
// weak (the mean of E against the float64 grid's at 128^3: -1.1e-7, -1.4e-8 so) and the moments
// after 20 steps 1.26 times as far from the float64 grid's as radices of up to 4 had them (0.80
// times so; geometric means over 60 grids).  At no measurable cost (a float32 step of 1e8 particles
// on 128^3: 5.32 and 5.31 ms).
template <typename T, int DIR, int N>
__host__ __device__ __forceinline__ Cx<T> cmul_root(Cx<T> a, int t) {
  if (t == 0) return a;
  if (2 * t == N) return {-a.x, -a.y};
  if (4 * t == N) return DIR < 0 ? Cx<T>{a.y, -a.x} : Cx<T>{-a.y, a.x};
  if (4 * t == 3 * N) return DIR < 0 ? Cx<T>{-a.y, a.x} : Cx<T>{a.y, -a.x};
  const int q = t * (144 / N);
  const double cd = cos144(q), sd = DIR * cos144((q + 108) % 144);
  const T c = (T)cd, s = (T)sd;
  if constexpr (sizeof(T) == 4) {
    const T cl = (T)(cd - (double)c), sl = (T)(sd - (double)s);
    // the rests go in beside the product of a rounded factor: beside that of an exact one (1/2),
    // which lies on the grid of the values, they would be rounded away
    if (sl == 0)
      return {std::fma(-a.y, s, std::fma(a.x, c, a.x * cl)),
              std::fma(a.x, s, std::fma(a.y, c, a.y * cl))};
    return {std::fma(a.x, c, std::fma(-a.y, s, a.x * cl - a.y * sl)),
            std::fma(a.y, c, std::fma(a.x, s, a.x * sl + a.y * cl))};
  }
  return {a.x * c - a.y * s, a.x * s + a.y * c};
}

// Radix-R DFT in registers; DIR = -1 forward, +1 inverse (no scaling).  R is a template
// parameter so that the butterfly values stay in registers.  Composite radices R = A B: B DFTs of
// length A over the inputs n2, n2 + B, ..., the roots exp(DIR 2 pi i n2 k1 / R), A DFTs of
// length B.
template <typename T, int DIR, int R>
__host__ __device__ __forceinline__ void dft(Cx<T>* v) {
  if constexpr (R == 1) {
    return;
  } else if constexpr (R == 2) {
    Cx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    Cx<T> t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    Cx<T> t2 = cadd(v[1], v[3]), t3 = csub(v[1], v[3]);
    Cx<T> jt3 = DIR < 0 ? Cx<T>{t3.y, -t3.x} : Cx<T>{-t3.y, t3.x};  // -i t3 or +i t3
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, jt3);
    v[3] = csub(t1, jt3);
  } else if constexpr (R == 3) {
    const T s3 = (T)(DIR < 0 ? -0.86602540378443864676 : 0.86602540378443864676);
    Cx<T> a0 = v[0], a1 = v[1], a2 = v[2];
    Cx<T> sum = cadd(a1, a2), dif = csub(a1, a2);
    Cx<T> m = {a0.x - (T)0.5 * sum.x, a0.y - (T)0.5 * sum.y};
    Cx<T> jd = {-s3 * dif.y, s3 * dif.x};  // i s3 (a1 - a2)
    if constexpr (sizeof(T) == 4) {  // with the rest of s3, see cmul_root
      const T s3l = (T)((DIR < 0 ? -0.86602540378443864676 : 0.86602540378443864676) - (double)s3);
      jd = {std::fma(-s3, dif.y, -s3l * dif.y), std::fma(s3, dif.x, s3l * dif.x)};
    }
    v[0] = cadd(a0, sum);
    v[1] = cadd(m, jd);
    v[2] = csub(m, jd);
  } else {
    constexpr int A = R % 4 == 0 && R != 12 ? (R == 8 ? 2 : 4) : (R == 6 ? 2 : 3);
    constexpr int B = R / A;  // 6 = 2 3, 8 = 2 4, 9 = 3 3, 12 = 3 4, 16 = 4 4
    static_assert(B <= 4 && 144 % R == 0, "unsupported radix");
    Cx<T> y[B][A];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) y[n2][n1] = v[B * n1 + n2];
      dft<T, DIR, A>(y[n2]);
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) y[n2][k1] = cmul_root<T, DIR, R>(y[n2][k1], n2 * k1);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      Cx<T> u[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) u[n2] = y[n2][k1];
      dft<T, DIR, B>(u);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = u[k2];
    }
  }
}

// the radices of a line length, in the order of the forward transform
template <int... R>
struct Radices {};
template <int M>
struct RadicesOf;
#define PIC_RADICES(M, ...)              \
  template <>                            \
  struct RadicesOf<M> {                  \
    using fwd = Radices<__VA_ARGS__>;    \
  };
PIC_RADICES(16, 4, 4)
PIC_RADICES(18, 6, 3)
PIC_RADICES(24, 6, 4)
PIC_RADICES(27, 9, 3)
PIC_RADICES(32, 8, 4)
PIC_RADICES(36, 6, 6)
PIC_RADICES(48, 8, 6)
PIC_RADICES(54, 9, 6)
PIC_RADICES(64, 8, 8)
PIC_RADICES(72, 9, 8)
PIC_RADICES(81, 9, 9)
PIC_RADICES(96, 12, 8)
PIC_RADICES(108, 12, 9)
PIC_RADICES(128, 16, 8)
PIC_RADICES(144, 12, 12)
PIC_RADICES(162, 9, 6, 3)
PIC_RADICES(192, 16, 12)
PIC_RADICES(216, 9, 6, 4)
PIC_RADICES(256, 16, 16)
#undef PIC_RADICES

template <typename S, int... D>
struct ReverseRadices;
template <int... D>
struct ReverseRadices<Radices<>, D...> {
  using type = Radices<D...>;
};
template <int R, int... Rest, int... D>
struct ReverseRadices<Radices<R, Rest...>, D...> {
  using type = typename ReverseRadices<Radices<Rest...>, R, D...>::type;
};

constexpr int pow2_ceil(int v) {
  int p = 1;
  while (p < v) p *= 2;
  return p;
}
template <int R0, int... R>
constexpr int first_radix(Radices<R0, R...>) {
  return R0;  // the largest: the tables above start with it
}
// threads per line: a power of two, one butterfly of the largest radix each
template <int M>
constexpr int line_threads() {
  return pow2_ceil(M / first_radix(typename RadicesOf<M>::fwd{}));
}
// rounds of butterflies a thread takes in a stage of radix R
template <int M, int R>
constexpr int line_rounds() {
  return (M / R + line_threads<M>() - 1) / line_threads<M>();
}

constexpr int kFftThreads = 128;  // threads per workgroup of the register transforms
template <int M>
constexpr int line_count() {  // lines per workgroup
  return kFftThreads / line_threads<M>();
}

// Where element p of line l lies in LDS.  Lines that are consecutive in memory (y and z): the
// line runs fastest, as in global memory, so a wave's accesses are consecutive.  Lines along x:
// the element runs fastest, with one element of padding in eight against bank conflicts.
template <int M, bool LFAST>
__device__ __forceinline__ int lds_at(int l, int p) {
  if constexpr (LFAST) return p * line_count<M>() + l;
  return l * (M + M / 8 + 1) + p + p / 8;
}
template <int M, bool LFAST>
constexpr int lds_elems() {
  return LFAST ? M * line_count<M>() : line_count<M>() * (M + M / 8 + 1);
}

// a thread's line within the workgroup and its place among the line's threads
template <int M, bool LFAST>
__device__ __forceinline__ void line_pos(int* l, int* j) {
  constexpr int LB = line_count<M>(), TPL = line_threads<M>();
  if constexpr (LFAST) {
    *l = (int)threadIdx.x % LB;
    *j = (int)threadIdx.x / LB;
  } else {
    *l = (int)threadIdx.x / TPL;
    *j = (int)threadIdx.x % TPL;
  }
}

// The stages R, Rest... of a transform whose earlier stages have product NS, on the butterfly
// inputs v; `last` receives the outputs of the final stage, v[q][r] at jb + r NS' for
// jb = j + q TPL < M / R'.  FIRST: LDS has not been read yet in this workgroup.  Twiddle
// exp(-2 pi i t / M) is tw[t TWS].
template <typename T, int DIR, int M, bool LFAST, int TWS, int NS, bool FIRST, typename S>
struct Stages;
template <typename T, int DIR, int M, bool LFAST, int TWS, int NS, bool FIRST, int R, int... Rest>
struct Stages<T, DIR, M, LFAST, TWS, NS, FIRST, Radices<R, Rest...>> {
  static constexpr int TPL = line_threads<M>();
  static constexpr int Q = line_rounds<M, R>();
  template <typename Last>
  static __device__ __forceinline__ void run(Cx<T> (&v)[Q][R], Cx<T>* lds, int l, int j,
                                             const typename TwT<T>::type* __restrict__ tw,
                                             Last&& last) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int jb = j + q * TPL;
      if constexpr (NS > 1) {
        const int k = jb % NS;
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const auto w = tw[r * k * (M / (NS * R)) * TWS];
          v[q][r] = cmul(v[q][r], Cx<T>{(T)w.x, DIR < 0 ? (T)w.y : (T)-w.y});
        }
      }
      dft<T, DIR, R>(v[q]);
    }
    if constexpr (sizeof...(Rest) == 0) {
      last(v);
    } else {
      if constexpr (!FIRST) __syncthreads();
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int jb = j + q * TPL;
        const int o = (jb / NS) * (NS * R) + jb % NS;
        if (jb < M / R) {
#pragma unroll
          for (int r = 0; r < R; ++r) lds[lds_at<M, LFAST>(l, o + r * NS)] = v[q][r];
        }
      }
      __syncthreads();
      next(lds, l, j, tw, last, Radices<Rest...>{});
    }
  }
  template <typename Last, int R2, int... Rest2>
  static __device__ __forceinline__ void next(Cx<T>* lds, int l, int j,
                                              const typename TwT<T>::type* __restrict__ tw,
                                              Last&& last, Radices<R2, Rest2...>) {
    constexpr int Q2 = line_rounds<M, R2>();
    Cx<T> w[Q2][R2];
#pragma unroll
    for (int q = 0; q < Q2; ++q) {
      const int jb = j + q * TPL;
      const int at = jb < M / R2 ? jb : 0;
#pragma unroll
      for (int r = 0; r < R2; ++r) w[q][r] = lds[lds_at<M, LFAST>(l, at + r * (M / R2))];
    }
    Stages<T, DIR, M, LFAST, TWS, NS * R, false, Radices<R2, Rest2...>>::run(w, lds, l, j, tw,
                                                                            last);
  }
};

// A whole transform: load(p) gives input p of the thread's line, last(v) takes the outputs as in
// Stages.  SEQ: the radices in order.
template <typename T, int DIR, int M, bool LFAST, int TWS, typename SEQ, typename Load,
          typename Last, int R, int... Rest>
__device__ __forceinline__ void line_fft_seq(Cx<T>* lds, int l, int j,
                                             const typename TwT<T>::type* __restrict__ tw,
                                             Load&& load, Last&& last, Radices<R, Rest...>) {
  constexpr int Q = line_rounds<M, R>(), TPL = line_threads<M>();
  Cx<T> v[Q][R];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int jb = j + q * TPL;
    const int at = jb < M / R ? jb : 0;
#pragma unroll
    for (int r = 0; r < R; ++r) v[q][r] = load(at + r * (M / R));
  }
  Stages<T, DIR, M, LFAST, TWS, 1, true, SEQ>::run(v, lds, l, j, tw, last);
}
template <typename T, int DIR, int M, bool LFAST, int TWS, typename Load, typename Last>
__device__ __forceinline__ void line_fft(Cx<T>* lds, int l, int j,
                                         const typename TwT<T>::type* __restrict__ tw,
                                         Load&& load, Last&& last) {
  using SEQ = typename RadicesOf<M>::fwd;
  line_fft_seq<T, DIR, M, LFAST, TWS, SEQ>(lds, l, j, tw, load, last, SEQ{});
}

// f(r) over a final stage's outputs: out(position, value) for every value the thread holds
template <typename T, int M, int Q, int R, typename Out>
__device__ __forceinline__ void each_output(Cx<T> (&v)[Q][R], int j, Out&& out) {
  constexpr int TPL = line_threads<M>(), NS = M / R;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int jb = j + q * TPL;
    if (jb < NS) {
#pragma unroll
      for (int r = 0; r < R; ++r) out(jb + r * NS, v[q][r]);
    }
  }
}

template <int M>
struct LineLength {
  static constexpr int value = M;
};
// f(LineLength<M>{}) for a length that has register transforms, else false
template <typename F>
__host__ __device__ __forceinline__ bool with_line_length(int M, F&& f) {
  switch (M) {
#define PIC_LEN(V) \
  case V:          \
    f(LineLength<V>{}); \
    return true;
    PIC_LEN(16) PIC_LEN(18) PIC_LEN(24) PIC_LEN(27) PIC_LEN(32) PIC_LEN(36) PIC_LEN(48)
    PIC_LEN(54) PIC_LEN(64) PIC_LEN(72) PIC_LEN(81) PIC_LEN(96) PIC_LEN(108) PIC_LEN(128)
    PIC_LEN(144) PIC_LEN(162) PIC_LEN(192) PIC_LEN(216) PIC_LEN(256)
#undef PIC_LEN
  }
  return false;
}

}  // namespace pic
