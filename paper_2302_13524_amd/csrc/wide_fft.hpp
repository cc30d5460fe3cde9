// 2-D FFT plan of the workload grids (32 x 32 to 128 x 64), mixed-axis passes.
//
// A pass transforms a digit of one axis or one digit of each, up to 16 values
// in a thread's registers. 1024 to 4096 points take three passes and two LDS
// exchanges, 8192 points three such passes and one more bit that two registers
// swap across the wave's halves (v_permlane32_swap) instead of a third
// exchange. A row is T = N / 16 threads with one LDS copy (68.6 KB at 8192
// points) and at most 128 registers a thread, so two workgroups of 128 x 64
// share a CU and one's exchanges and loads run beside the other's arithmetic.
//
// Every element index is a set of bits (axis 2 low, axis 1 above); a pass
// assigns four of them to the register number and the others to the thread.
// Inside a digit the radix-2 decimation-in-time stages with a factor w other
// than a quarter turn take six operations per butterfly (bfly). The twiddles
// between digits stay separate products: taken along in the stages a launch is
// 3 to 8 % shorter, but its error against 64 bits was larger than the one-axis
// plans' (a residual 2.1e-6 off instead of 1.7e-6).
#pragma once
#include "fft_core.hpp"

#include <type_traits>

namespace tmk {

__device__ __forceinline__ int hidden_zero() {
  int z;
  asm volatile("s_mov_b32 %0, 0" : "=s"(z));
  return z;
}

constexpr int WIDE_LE = 4;
constexpr int WIDE_E = 1 << WIDE_LE;
constexpr int WIDE_LT = 9;  // most thread bits

struct WidePass {
  int reg[WIDE_LE];  // element bits of the register number, low to high
  int thr[WIDE_LT];  // element bits of the thread number, low to high
  int a_lo, a_n;     // axis-1 digit of this pass: bits [a_lo, a_lo + a_n) of i1
  int b_lo, b_n;     // axis-2 digit
  int swap;          // register bit swapped with lane bit 5 on the way from the last pass; -1: LDS exchange
};

struct WideDesc {
  int np;
  WidePass p[4];
};

// The lanes of the first pass run along axis 2 (rows and masks are read and
// written in 256- or 512-byte runs). At 64 x 64 and 128 x 64 the inverse
// transform's twiddles are the same in all lanes of a wave; those that differ
// between lanes are kept in LDS.
constexpr WideDesc wide_desc(int L1, int L2) {
  WideDesc d{};
  const int A = L2;  // element bit of a0
  if (L1 == 5 && L2 == 5) {
    d.np = 3;
    d.p[0] = {{A + 1, A + 2, A + 3, A + 4}, {0, 1, 2, 3, 4, A}, 1, 4, 0, 0, -1};
    d.p[1] = {{1, 2, 3, 4}, {A, A + 1, A + 2, A + 3, A + 4, 0}, 0, 0, 1, 4, -1};
    d.p[2] = {{A, 0, A + 1, A + 2}, {1, 2, 3, 4, A + 3, A + 4}, 0, 1, 0, 1, -1};
  } else if (L1 == 6 && L2 == 5) {
    d.np = 3;
    d.p[0] = {{A + 2, A + 3, A + 4, A + 5}, {0, 1, 2, 3, 4, A, A + 1}, 2, 4, 0, 0, -1};
    d.p[1] = {{1, 2, 3, 4}, {A, A + 1, A + 2, A + 3, A + 4, A + 5, 0}, 0, 0, 1, 4, -1};
    d.p[2] = {{A, A + 1, 0, A + 2}, {1, 2, 3, 4, A + 3, A + 4, A + 5}, 0, 2, 0, 1, -1};
  } else if (L1 == 6 && L2 == 6) {
    d.np = 3;
    d.p[0] = {{A + 2, A + 3, A + 4, A + 5}, {0, 1, 2, 3, 4, 5, A, A + 1}, 2, 4, 0, 0, -1};
    d.p[1] = {{2, 3, 4, 5}, {A, A + 1, A + 2, A + 3, A + 4, A + 5, 0, 1}, 0, 0, 2, 4, -1};
    d.p[2] = {{A, A + 1, 0, 1}, {2, 3, 4, 5, A + 2, A + 3, A + 4, A + 5}, 0, 2, 0, 2, -1};
  } else if (L1 == 7 && L2 == 6) {
    d.np = 4;
    d.p[0] = {{A + 3, A + 4, A + 5, A + 6}, {0, 1, 2, 3, 4, 5, A, A + 1, A + 2}, 3, 4, 0, 0, -1};
    d.p[1] = {{2, 3, 4, 5}, {A, A + 1, A + 2, A + 3, A + 4, A + 5, 0, 1, A + 6}, 0, 0, 2, 4, -1};
    d.p[2] = {{A, A + 1, A + 2, 1}, {2, 3, 4, 5, A + 3, 0, A + 4, A + 5, A + 6}, 0, 3, 0, 0, -1};
    d.p[3] = {{A, A + 1, 0, 1}, {2, 3, 4, 5, A + 3, A + 2, A + 4, A + 5, A + 6}, 0, 0, 0, 2, 2};
  }
  return d;
}

constexpr bool wide_compiled(int L1, int L2) { return wide_desc(L1, L2).np > 0; }

template <int L1_, int L2_>
struct WidePlan {
  static constexpr bool WIDE = true;
  static constexpr int L1 = L1_, L2 = L2_, LN = L1 + L2;
  static constexpr int N1 = 1 << L1, N2 = 1 << L2, N = 1 << LN;
  static constexpr int LE = WIDE_LE, E = 1 << LE;
  static constexpr int LT = LN - LE, T = 1 << LT;
  static constexpr WideDesc D = wide_desc(L1, L2);
  static_assert(D.np > 0, "grid without a wide plan");
  static constexpr int NP = D.np;
  // LDS slot of (i1, i2): i1 S + i2 + i2 / 16. The odd row stride keeps lanes along
  // axis 1 on distinct banks, the extra slots lanes along bits 2 to 5 of i2.
  static constexpr int S = (N2 + N2 / 16 - 1) | 1;
  static_assert(S % 2 == 1 && S >= N2 + N2 / 16 - 1, "odd stride that holds a row");
  static constexpr int LDS_ROW = N1 * S;
  // waves per SIMD: the radix-16 twiddles that differ between lanes take registers (at four
  // waves the N2 = 32 grids spill 6 to 20)
  static constexpr int WAVES = L2 == 5 ? 3 : 4;
  // twiddles that differ between lanes (WideFft::lane_off)
  static constexpr int LDS_TW = (L1 == 5 ? 32 : L2 == 5 ? 19 : L1 == 6 ? 6 : 10) * 16;

  // Maps of element bits that are linear over the bits: element, LDS slot, frequency.
  enum Map { ELEM, LDS, FREQ };
  static constexpr int lds_bit(int e) { return e >= L2 ? (1 << (e - L2)) * S : (1 << e) + ((1 << e) >> 4); }
  // digit of pass p of axis 1 (ax1) or 2
  static constexpr int lo_of(int p, bool ax1) { return ax1 ? D.p[p].a_lo : D.p[p].b_lo; }
  static constexpr int n_of(int p, bool ax1) { return ax1 ? D.p[p].a_n : D.p[p].b_n; }
  // Frequency weight within its axis of slot bit e, over the digits of passes < np: the digit
  // transformed first holds the low frequency bits.
  static constexpr int axis_freq_bit(int e, int np) {
    const bool ax1 = e >= L2;
    const int q = ax1 ? e - L2 : e;
    int done = 0;
    for (int p = 0; p < np; ++p) {
      const int lo = lo_of(p, ax1), n = n_of(p, ax1);
      if (n > 0 && q >= lo && q < lo + n) return 1 << (done + q - lo);
      done += n;
    }
    return 0;
  }
  static constexpr int freq_bit(int e) { return axis_freq_bit(e, NP) << (e >= L2 ? L2 : 0); }
  template <int M>
  static constexpr int bitval(int e) {
    return M == ELEM ? 1 << e : M == LDS ? lds_bit(e) : freq_bit(e);
  }
  template <int P, int M>
  static constexpr int reg_off(int r) {
    int s = 0;
    for (int i = 0; i < LE; ++i)
      if ((r >> i) & 1) s += bitval<M>(D.p[P].reg[i]);
    return s;
  }
  template <int P, int M>
  static __device__ __forceinline__ int thr_base(int t) {
    int s = 0;
#pragma unroll
    for (int i = 0; i < LT; ++i) s += ((t >> i) & 1) * bitval<M>(D.p[P].thr[i]);
    return s;
  }

  // ---- twiddles of axis AX's digit in pass P, forward (INV = false): base W_M^K with K the
  // frequency of the axis's digits done before and M the points done after it; inverse: base
  // conj W_B^l with l the position below the digit and B = 2^(lo + n)
  template <int P, int AX, bool INV>
  static constexpr int tw_bit(int e) {
    if ((e >= L2) != (AX == 1)) return 0;
    if (!INV) return axis_freq_bit(e, P);
    const int q = (AX == 1) ? e - L2 : e;
    return q < lo_of(P, AX == 1) ? 1 << q : 0;
  }
  template <int P, int AX, bool INV>
  static constexpr int tw_log() {  // log2 of M or B
    if (INV) return lo_of(P, AX == 1) + n_of(P, AX == 1);
    int s = 0;
    for (int i = 0; i <= P; ++i) s += n_of(i, AX == 1);
    return s;
  }
  template <int P, int AX, bool INV>
  static constexpr bool twiddled() {
    return n_of(P, AX == 1) > 0 && tw_log<P, AX, INV>() > n_of(P, AX == 1);
  }
  template <int P, int AX, bool INV>
  static constexpr int tw_reg(int r) {
    int s = 0;
    for (int i = 0; i < LE; ++i)
      if ((r >> i) & 1) s += tw_bit<P, AX, INV>(D.p[P].reg[i]);
    return s;
  }
  template <int P, int AX, bool INV>
  static constexpr int tw_lanes() {  // part of K (l) that differs between the lanes of a wave
    int s = 0;
    for (int i = 0; i < LT && i < 6; ++i) s += tw_bit<P, AX, INV>(D.p[P].thr[i]);
    return s;
  }
  template <int P, int AX, bool INV>
  static __device__ __forceinline__ int tw_thr(int t) {
    int s = 0;
#pragma unroll
    for (int i = 0; i < LT; ++i) s += ((t >> i) & 1) * tw_bit<P, AX, INV>(D.p[P].thr[i]);
    return s;
  }
  // register position (shift) of a digit: its bits are consecutive register bits
  template <int P, int AX>
  static constexpr int digit_shift() {
    const int e0 = (AX == 1) ? L2 + D.p[P].a_lo : D.p[P].b_lo;
    for (int i = 0; i < LE; ++i)
      if (D.p[P].reg[i] == e0) return i;
    return 0;
  }
};

// --------------------------------------------------------------- butterflies
// a, b <- a + w b, a - w b with w = W_16^K = exp(-2 pi j K / 16), K = 1 .. 3 (INV: conj w),
// times -j (INV: +j) when ROT. w b = s u with s = sin(pi / 8), or sqrt(1/2) for K = 2, and
// u = b's components with the cotangent cot(pi / 8), or 1, between them: two operations for u
// and one fused multiply-add per result and component, each of which rounds its own value
// once (Linzer and Feig's form for fused multiply-add machines; the difference as
// 2 a - (a + w b), of the same length, takes over the sum's rounding). Error of a transform
// against 64 bits, rms, forward / inverse, 1e-7: 128 x 64 1.164 / 1.170, one axis per pass
// 1.235 / 1.234, differences from the sums 1.268 / 1.267; 32 x 32 1.016 / 1.019, 1.064 / 1.060,
// 1.103 / 1.105.
//
// Rounded constants also change a transform's gain, which moves a residual more than its
// random rounding does. sin and cot(pi / 8) come out too large together (w by 1.7e-8; cos and
// tan too small by 2.9e-8), sqrt(1/2) too small by 1.7e-8: with the nearest values the gain is
// -2.2e-8. A radix-16 digit's last stage takes the next sqrt(1/2) up in one component (UP):
// -1.2e-8 (one axis per pass -4.0e-8). In every stage it would be -0.1e-8, but the errors of
// that value, 6.7e-8, would add 2 to 3 % to the random part.
template <int K, bool INV, bool ROT, bool UP, typename T>
__device__ __forceinline__ void bfly(cx<T>& a, cx<T>& b) {
  constexpr T r = T(0.70710678118654752440), r_up = sizeof(T) == 4 ? T(0.70710682868957519531) : r;
  constexpr T cot = T(2.41421356237309504880), sx = K == 2 ? r : T(0.38268343236508977173), sy = UP && K == 2 ? r_up : sx;
  T ux, uy;
  if constexpr (K == 1) {
    ux = fmadd(cot, b.x, INV ? -b.y : b.y);
    uy = fmadd(cot, b.y, INV ? b.x : -b.x);
  } else if constexpr (K == 2) {
    ux = INV ? b.x - b.y : b.x + b.y;
    uy = INV ? b.y + b.x : b.y - b.x;
  } else {
    ux = fmadd(INV ? -cot : cot, b.y, b.x);
    uy = fmadd(INV ? cot : -cot, b.x, b.y);
  }
  const T vx = !ROT ? ux : INV ? -uy : uy, vy = !ROT ? uy : INV ? ux : -ux;
  b = cx<T>{fmadd(-sx, vx, a.x), fmadd(-sy, vy, a.y)};
  a = cx<T>{fmadd(sx, vx, a.x), fmadd(sy, vy, a.y)};
}
// the same for w = 1
template <bool INV, bool ROT, typename T>
__device__ __forceinline__ void bfly1(cx<T>& a, cx<T>& b) {
  cx<T> t = b;
  if constexpr (ROT) t = mulmj<T, INV>(t);
  b = a - t;
  a = a + t;
}

// Twiddles of a digit of size R = 2^LR: value h takes base^h, h = 1 .. R - 1. Where
// the base differs between lanes they are read from LDS, for each h one row of 16
// values of K. In registers they would take 20 of the 128 at 128 x 64.
template <typename T>
struct LaneTw {
  typedef T Pair __attribute__((ext_vector_type(2)));
  const cx<T>* w;  // this thread's column
  __device__ __forceinline__ cx<T> operator()(int h) const {
    const Pair v = *(const Pair*)(w + (h - 1) * 16);
    return cx<T>{v.x, v.y};
  }
};

template <int R, int lm, bool INV, typename T>
__device__ __forceinline__ void dit_stage(cx<T>* u) {
  constexpr int m = 1 << lm, h = m / 2, q = m >= 4 ? m / 4 : 1;
#pragma unroll
  for (int k = 0; k < q; ++k) {
#pragma unroll
    for (int g = 0; g < R / m; ++g) {
      cx<T>* v = u + g * m;
      if (k == 0) {
        bfly1<INV, false, T>(v[0], v[h]);
        if constexpr (m >= 4) bfly1<INV, true, T>(v[q], v[q + h]);
      } else {
        auto turn = [&](auto n) {
          bfly<decltype(n)::value, INV, false, m == 16, T>(v[k], v[k + h]);
          bfly<decltype(n)::value, INV, true, m == 16, T>(v[k + q], v[k + q + h]);
        };
        switch (k * (16 / m)) {  // a constant of the unrolled loop
          case 1: turn(std::integral_constant<int, 1>{}); break;
          case 2: turn(std::integral_constant<int, 2>{}); break;
          default: turn(std::integral_constant<int, 3>{}); break;
        }
      }
    }
  }
  if constexpr (m < R) dit_stage<R, lm + 1, INV, T>(u);
}

// DFT of size R = 2^LR over register bits [SH, SH + LR) at the registers whose other bits are `rest`
template <int LR, int SH, bool INV, typename T>
__device__ __forceinline__ void dft_regs(cx<T>* x, int rest) {
  constexpr int R = 1 << LR;
  cx<T> u[R];
#pragma unroll
  for (int h = 0; h < R; ++h) {
    int rev = 0;
    for (int b = 0; b < LR; ++b) rev |= ((h >> b) & 1) << (LR - 1 - b);
    u[rev] = x[rest | (h << SH)];
  }
  dit_stage<R, 1, INV, T>(u);
#pragma unroll
  for (int h = 0; h < R; ++h) x[rest | (h << SH)] = u[h];
}
// Register numbers with the bits [SH, SH + LR) zero, by index
template <int LR, int SH>
constexpr int rest_of(int i) { return (i & ((1 << SH) - 1)) | ((i >> SH) << (SH + LR)); }

// Swap of register bit RB with lane bit 5: the upper half of the registers with the bit
// clear changes places with the lower half of those with it set.
template <int RB>
__device__ __forceinline__ void half_wave_swap(cx<float>* x) {
#pragma unroll
  for (int r = 0; r < WIDE_E; ++r) {
    if ((r >> RB) & 1) continue;
    cx<float>& p = x[r];
    cx<float>& q = x[r | (1 << RB)];
    const auto sx = __builtin_amdgcn_permlane32_swap(__float_as_uint(p.x), __float_as_uint(q.x), false, false);
    const auto sy = __builtin_amdgcn_permlane32_swap(__float_as_uint(p.y), __float_as_uint(q.y), false, false);
    p = cx<float>{__uint_as_float(sx[0]), __uint_as_float(sy[0])};
    q = cx<float>{__uint_as_float(sx[1]), __uint_as_float(sy[1])};
  }
}

// ------------------------------------------------------------ the transform
// One row group's transforms. The exchanges write each pass's values at the
// slots which the same thread read them from, so one barrier per exchange
// orders everything while forward and inverse transforms alternate; a transform
// that does not start in the layout the last one ended in needs fence() first.
template <class PL, typename T>
struct WideFft {
  // one vector access per value (as a struct its parts were also read on their own)
  typedef T Pair __attribute__((ext_vector_type(2)));
  static constexpr int NP = PL::NP;
  static constexpr WideDesc D = PL::D;

  // Twiddles that differ between lanes, in LDS behind the rows, 16 columns of K (l): those of
  // the forward, then the inverse digits, pass by pass
  template <int P, int AX, bool INV>
  static constexpr int lane_count() {
    if constexpr (P >= NP) return 0;
    else return PL::template twiddled<P, AX, INV>() && PL::template tw_lanes<P, AX, INV>() != 0
                    ? (1 << PL::n_of(P, AX == 1)) - 1 : 0;
  }
  template <int P, int AX, bool INV>
  static constexpr int lane_off() {
    if constexpr (INV) return lane_off<P, AX, false>() + lane_count<P, AX, false>();
    else if constexpr (AX == 2) return lane_off<P, 1, true>() + lane_count<P, 1, true>();
    else if constexpr (P == 0) return 0;
    else return lane_off<P - 1, 2, true>() + lane_count<P - 1, 2, true>();
  }
  static_assert(lane_off<NP, 1, false>() * 16 <= PL::LDS_TW, "LDS for the lane twiddles");

  cx<T>* lds;
  cx<T>* tws;
  int base[NP];
  const cx<T>* t1;
  const cx<T>* t2;
  int ku[NP][2][2];  // K or l: [pass][axis - 1][inverse]

  template <int P, int AX, bool INV>
  __device__ __forceinline__ void setup(int ltid, const cx<T>* tab) {
    if constexpr (PL::template twiddled<P, AX, INV>()) {
      constexpr int LR = PL::n_of(P, AX == 1), LM = PL::template tw_log<P, AX, INV>(), LA = AX == 1 ? PL::L1 : PL::L2;
      const int K = PL::template tw_thr<P, AX, INV>(ltid);  // thread's part; the register's is a constant
      if constexpr (lane_count<P, AX, INV>() > 0) {
        static_assert(LM - LR <= 4, "at most 16 values of K");
        ku[P][AX - 1][INV] = K;
        if (ltid < (1 << (LM - LR))) {  // the first exchange's barrier orders these writes before their use
#pragma unroll
          for (int h = 1; h < (1 << LR); ++h)
            tws[(lane_off<P, AX, INV>() + h - 1) * 16 + ltid] = tab[(ltid * h) << (LA - LM)];
        }
      } else {
        ku[P][AX - 1][INV] = __builtin_amdgcn_readfirstlane(K);
      }
    }
  }
  template <int P>
  __device__ __forceinline__ void setup_all(int ltid) {
    if constexpr (P < NP) {
      base[P] = PL::template thr_base<P, PL::LDS>(ltid);
      setup<P, 1, false>(ltid, t1);
      setup<P, 2, false>(ltid, t2);
      setup<P, 1, true>(ltid, t1);
      setup<P, 2, true>(ltid, t2);
      setup_all<P + 1>(ltid);
    }
  }
  // ltw: the workgroup's LDS_TW slots (its rows write the same values there)
  __device__ __forceinline__ WideFft(cx<T>* l, cx<T>* ltw, int ltid, const cx<T>* tw1, const cx<T>* tw2)
      : lds(l), tws(ltw), t1(wave_uniform(tw1)), t2(wave_uniform(tw2)) {
    setup_all<0>(ltid);
  }

  template <int P>
  __device__ __forceinline__ void store(const cx<T>* x) const {
    Pair* p = (Pair*)(lds + base[P]);
#pragma unroll
    for (int r = 0; r < PL::E; ++r) p[PL::template reg_off<P, PL::LDS>(r)] = Pair{x[r].x, x[r].y};
  }
  template <int P>
  __device__ __forceinline__ void load(cx<T>* x) const {
    const Pair* p = (const Pair*)(lds + base[P]);
#pragma unroll
    for (int r = 0; r < PL::E; ++r) {
      const Pair v = p[PL::template reg_off<P, PL::LDS>(r)];
      x[r] = cx<T>{v.x, v.y};
    }
  }
  // from the layout of pass PW to that of the neighbouring pass PR
  template <int PW, int PR>
  __device__ __forceinline__ void exchange(cx<T>* x) const {
    constexpr int hi = PW > PR ? PW : PR;
    if constexpr (D.p[hi].swap >= 0) {
      half_wave_swap<D.p[hi].swap>(x);
    } else {
      store<PW>(x);
      __syncthreads();
      load<PR>(x);
    }
  }
  __device__ __forceinline__ void fence() const { __syncthreads(); }

  // The uniform twiddles of a radix-16 digit, read ahead of the exchange before it so that
  // their scalar loads do not hold up the pass (Lanczos step at 2286 x 8192: 315 us when read
  // in it with 64-bit addresses, 287 here). Behind a zero that the compiler cannot see: taken out of the mask loop they
  // overflow the scalar registers.
  struct Ahead {
    cx<T> w[WIDE_E - 1];
    __device__ __forceinline__ cx<T> operator()(int h) const { return w[h - 1]; }
  };
  template <int P, int AX, bool INV>
  static constexpr bool uniform_tw() {
    return PL::template twiddled<P, AX, INV>() && lane_count<P, AX, INV>() == 0;
  }
  template <int P, bool INV>
  __device__ __forceinline__ Ahead ahead() const {
    Ahead a{};
    constexpr bool u1 = uniform_tw<P, 1, INV>(), u2 = uniform_tw<P, 2, INV>();
    static_assert(!(u1 && u2), "one uniform digit in a pass");
    if constexpr (u1 || u2) {
      constexpr int AX = u1 ? 1 : 2, LA = AX == 1 ? PL::L1 : PL::L2, LR = PL::n_of(P, AX == 1);
      static_assert(LR == WIDE_LE, "one butterfly");
      const int K = __builtin_amdgcn_readfirstlane(ku[P][AX - 1][INV]) + hidden_zero();
      const __attribute__((address_space(4))) char* c = (const __attribute__((address_space(4))) char*)(AX == 1 ? t1 : t2);
      const unsigned step = (unsigned)K << (LA - PL::template tw_log<P, AX, INV>());
      unsigned at = 0;  // W_LA^(h step): a 32-bit offset, the loads' own addressing
#pragma unroll
      for (int h = 1; h < WIDE_E; ++h) {
        at += step * (unsigned)sizeof(cx<T>);
        const __attribute__((address_space(4))) T* w = (const __attribute__((address_space(4))) T*)(c + at);
        a.w[h - 1] = cx<T>{w[0], w[1]};
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    return a;
  }

  // axis AX's digit of pass P
  template <int P, int AX, bool INV>
  __device__ __forceinline__ void digit(cx<T>* x, const Ahead& uni) const {
    constexpr int LR = PL::n_of(P, AX == 1);
    if constexpr (LR > 0) {
      constexpr int SH = PL::template digit_shift<P, AX>();
      if constexpr (PL::template twiddled<P, AX, INV>()) {
        // value h of every butterfly before the next h: its twiddle is live for that long only
#pragma unroll
        for (int h = 1; h < (1 << LR); ++h) {
#pragma unroll
          for (int i = 0; i < (PL::E >> LR); ++i) {
            const int rest = rest_of<LR, SH>(i);
            cx<T>& v = x[rest | (h << SH)];
            cx<T> w;
            if constexpr (lane_count<P, AX, INV>() > 0) {
              const int reg = PL::template tw_reg<P, AX, INV>(rest);
              w = LaneTw<T>{tws + lane_off<P, AX, INV>() * 16 + ku[P][AX - 1][INV] + reg}(h);
            } else {
              w = uni(h);
            }
            v = INV ? cmulc(v, w) : cmul(v, w);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < (PL::E >> LR); ++i) dft_regs<LR, SH, INV, T>(x, rest_of<LR, SH>(i));
    }
  }

  template <int P = 0>
  __device__ __forceinline__ void forward(cx<T>* x) const {
    if constexpr (P < NP) {
      const Ahead uni = ahead<P, false>();
      if constexpr (P > 0) exchange<P - 1, P>(x);
      digit<P, 1, false>(x, uni);
      digit<P, 2, false>(x, uni);
      forward<P + 1>(x);
    }
  }
  template <int P, class H>
  __device__ __forceinline__ void inverse_from(cx<T>* x, const H& before_last) const {
    if constexpr (P >= 0) {
      const Ahead uni = ahead<P, true>();
      if constexpr (P < NP - 1) exchange<P + 1, P>(x);
      if constexpr (P == 0) before_last();
      digit<P, 2, true>(x, uni);
      digit<P, 1, true>(x, uni);
      inverse_from<P - 1>(x, before_last);
    }
  }
  template <class H = NoHook>
  __device__ __forceinline__ void inverse(cx<T>* x, const H& before_last = H{}) const {
    inverse_from<NP - 1, H>(x, before_last);
  }
};

}  // namespace tmk
