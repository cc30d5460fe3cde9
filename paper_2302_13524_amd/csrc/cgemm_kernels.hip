// Complex FP32 GEMM on the FP32 matrix cores (v_mfma_f32_32x32x2_f32):
//   C[m][n] = sum_k A[m][k] op(B)[k][n]   (complex64, row-major)
// A is [M][K] (k contiguous); B is [N][K] (k contiguous, trans_b) or [K][N]
// (n contiguous). Used by the foci (patterns times the true TM, Sec. 3) and
// the dense-probing comparator (a random-phase Q in place of the FFTs).
//
// Short sums run on the FP32 matrix cores, others split into BF16 parts (further
// down). Real embedding of the complex product: for one complex k the MFMA's two
// real k are (real part, imaginary part), so that
//   C_r += [a_r a_i] . [b_r, -b_i],   C_i += [a_r a_i] . [b_i, b_r]:
// one 32x32x2 MFMA each, lanes 0-31 carrying the real parts of A (and of the
// first B operand), lanes 32-63 the imaginary parts. 128 x 128 output tiles,
// 256 threads (four waves of 64 x 64), K in steps of 16 complex values staged
// in LDS k-major ([k][row]: the 32 lanes of a half-wave read 32 consecutive
// rows), double-buffered through registers: the next step's tiles load while
// the MFMAs run on the current one.
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tmk {

namespace {

// Complex k from which the split product is taken: it wins there at every size, while its
// second, nearly empty launch (k_cgemm_redo, 2-3 us) makes it lose with few k. FP32 against
// split, us: 1024 x 1024 x 16 10.1 / 12.3, x 64 25.5 / 15.0; 128 x 128 x 16 9.9 / 12.2;
// 300 x 300 x 48 19.2 / 11.8, 2048 x 2048 x 64 28.6 / 22.5, 4096 x 4096 x 64 95 / 74,
// 2286 x 2286 x 8192 4361 / 2690.
// (At 32 the split would win by less, 1024 x 1024 15.3 / 12.0.)
constexpr int SPLIT_K = 64;

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int TM = 128, TK = 16;    // tile rows, complex k per step
constexpr int VPT = TK * TM / 256;  // complex values of a 128-row tile per thread

struct CgemmArgs {
  int M, N, K;
  const float2* A;
  int64_t lda;
  const float2* B;
  int64_t ldb;
  int trans_b;  // B stored [N][K]
  float2* C;
  int64_t ldc;
  int conj_c;   // store conj(C)
  int veca, vecb;  // 16-byte loads of two complex values allowed
  int range;       // largest sum of the (biased) exponents of A's and B's staged magnitudes
};

// The (16 VPT) x TK complex values of an operand's tile in registers, VPT per thread.
// k-contiguous source (A, or B with trans_b): row r0 + t VPT / TK, VPT consecutive k;
// n-contiguous source (B): k k0 + t / 16, VPT consecutive n.
template <int V>
struct Stage {
  float2 v[V];
};

template <int VPT, bool kcontig>
__device__ __forceinline__ void fetch(Stage<VPT>& s, const float2* __restrict__ p, int64_t ld, bool vec, int r0,
                                      int k0, int R, int K) {
  const int t = threadIdx.x;
  constexpr int NK = TK / VPT, NT = 16;  // threads along a row (k contiguous), along a k (n contiguous)
  const int a = kcontig ? r0 + t / NK : k0 + t / NT;                       // fixed index (row, or k)
  const int b = kcontig ? k0 + VPT * (t % NK) : r0 + VPT * (t % NT);       // first of VPT consecutive
  const int alim = kcontig ? R : K, blim = kcontig ? K : R;
  const float2* q = p + (int64_t)a * ld + b;
  if (vec && a < alim && b + VPT <= blim) {
#pragma unroll
    for (int i = 0; i < VPT / 2; ++i) {
      const float4 u = ((const float4*)q)[i];
      s.v[2 * i] = make_float2(u.x, u.y);
      s.v[2 * i + 1] = make_float2(u.z, u.w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < VPT; ++i) s.v[i] = (a < alim && b + i < blim) ? q[i] : make_float2(0.f, 0.f);
  }
}

// into LDS as [k][row] (row stride 16 VPT complex values)
template <int VPT, bool kcontig>
__device__ __forceinline__ void stage_store(float2* lds, const Stage<VPT>& s) {
  const int t = threadIdx.x;
  constexpr int R = 16 * VPT, NK = TK / VPT;
  if (kcontig) {
    const int r = t / NK, kb = VPT * (t % NK);
#pragma unroll
    for (int i = 0; i < VPT; ++i) lds[(kb + i) * R + r] = s.v[i];
  } else {
    const int k = t / 16, nb = VPT * (t % 16);
    float4* d = (float4*)&lds[k * R + nb];
#pragma unroll
    for (int i = 0; i < VPT / 2; ++i) d[i] = make_float4(s.v[2 * i].x, s.v[2 * i].y, s.v[2 * i + 1].x, s.v[2 * i + 1].y);
  }
}

// C tile out: lane holds column n = lane % 32 of each 32 x 32 block, rows
// 8 q + 4 (lane / 32) + r for element 4 q + r
template <int NJ>
__device__ __forceinline__ void store_tile(const CgemmArgs& g, const f32x16 (&cr)[2][NJ], const f32x16 (&ci)[2][NJ], int m0,
                                           int n0, float scale = 1.f) {
  const int lane = threadIdx.x & 63;
  const float sgn = g.conj_c ? -scale : scale;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + 32 * i + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        const int n = n0 + 32 * j + (lane & 31);
        const float x = cr[i][j][e], y = ci[i][j][e];
        if (m < g.M && n < g.N) g.C[(int64_t)m * g.ldc + n] = make_float2(scale * x, sgn * y);
      }
}

// One 128 x (64 NJ) tile on the FP32 matrix cores; four waves of 64 x (32 NJ).
// LDS: two buffers of TK (128 + 64 NJ) complex values.
template <int NJ, bool BK>
__device__ __forceinline__ void tile_f32(const CgemmArgs& g, int m0, int n0, float2* lds) {
  constexpr int TN = 64 * NJ;
  float2* const sA[2] = {lds, lds + TK * (TM + TN)};
  float2* const sB[2] = {lds + TK * TM, lds + TK * (TM + TN) + TK * TM};
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 32 * NJ;
  const bool hi = lane >= 32;
  f32x16 cr[2][NJ], ci[2][NJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) cr[i][j][e] = ci[i][j][e] = 0.f;

  Stage<VPT> ra;
  Stage<4 * NJ> rb;
  fetch<VPT, true>(ra, g.A, g.lda, g.veca != 0, m0, 0, g.M, g.K);
  fetch<4 * NJ, BK>(rb, g.B, g.ldb, g.vecb != 0, n0, 0, g.N, g.K);
  const int nk = (g.K + TK - 1) / TK;
  for (int ks = 0; ks < nk; ++ks) {
    float2* a_s = sA[ks & 1];
    float2* b_s = sB[ks & 1];
    // this buffer's last readers (step ks - 2) passed the barrier of step ks - 1
    stage_store<VPT, true>(a_s, ra);
    stage_store<4 * NJ, BK>(b_s, rb);
    __syncthreads();
    if (ks + 1 < nk) {
      fetch<VPT, true>(ra, g.A, g.lda, g.veca != 0, m0, (ks + 1) * TK, g.M, g.K);
      fetch<4 * NJ, BK>(rb, g.B, g.ldb, g.vecb != 0, n0, (ks + 1) * TK, g.N, g.K);
    }
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      float av[2], br[NJ], bi[NJ];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float2 a = a_s[kk * TM + wm + 32 * i + (lane & 31)];
        av[i] = hi ? a.y : a.x;
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const float2 b = b_s[kk * TN + wn + 32 * j + (lane & 31)];
        br[j] = hi ? -b.y : b.x;
        bi[j] = hi ? b.x : b.y;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          cr[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], br[j], cr[i][j], 0, 0, 0);
          ci[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bi[j], ci[i][j], 0, 0, 0);
        }
    }
  }
  store_tile<NJ>(g, cr, ci, m0 + wm, n0 + wn);
}

template <bool BK>
__global__ void __launch_bounds__(256, 2) k_cgemm_mfma(CgemmArgs g) {
  __shared__ float2 lds[2 * TK * (TM + 128)];
  tile_f32<2, BK>(g, blockIdx.y * TM, blockIdx.x * 128, lds);
}

// ---------------------------------------------------------------- split products
// The same product on the BF16 matrix cores (16 times the FP32 rate), after Henry, Tang
// and Heinecke ("Leveraging the bfloat16 artificial intelligence datatype for
// higher-precision computations", 2019). Every FP32 value is the exact sum of three BF16
// values, each the nearest to what the ones before it leave,
//   x = x1 + x2 + x3,  |x2| <= 2^-8 |x|,  |x3| <= 2^-17 |x|,
// and a b = a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1) + (a2 b3 + a3 b2): eight
// products that the FP32 sums take in exactly; a3 b3, at most 2^-34 of a b, is left
// out. The BF16 cores cut off what falls below the accumulator's last place, so that a
// long chain of one sign comes out short (by 1.6e-6 over 8192 k): of 16 complex k the
// products a1 b1 are summed by themselves, the others by themselves, and the rounded sum
// of the two is added to the total. A sum of one product then comes out as FP32 rounds
// it: largest error 5.9e-8 of the product, rms 2.5e-8, as on the FP32 cores (with a1 b1
// in the others' chain and without the last two products 1.3e-7 and 3.5e-8). Longer
// sums, largest error over sum |a||b| (FP32 cores): 8192 k of normal values 3.8e-8
// (2.3e-7), 64 of one sign 1.7e-7 (5.7e-7), unit phases times their conjugates 3.0e-8
// (1.8e-7).
//
// Real embedding as above over k = (re, im) pairs; the operand for C_r flips
// the imaginary parts' signs, the one for C_i swaps each pair.
//
// The operands are scaled by 2^24 each, so that every part of every FP32 value,
// subnormal ones too, is a normal number; a product that all the same falls below the
// normal range is then below 2^-174 of the result's scale, where FP32 itself ends at
// 2^-149. At the other end the largest magnitudes of a tile's rows and columns may have a
// product up to 2^76 / K (2^63 at 8192 k), so that no sum overflows. Above it, and with
// infinities, the tile stops as soon as it has staged such a value and is left to
// k_cgemm_redo (a NaN gives NaN in its row or column either way). With a range per value
// in place of the scaling, [2^-48, 2^48], one sine of pi in a row of phases sent its tiles
// there: 2286 x 2286 x 8192 with phases of 0 and pi took 4390 us, now 2400 to 2520.
//
// 128 x 64 tiles and three workgroups per CU (168 VGPRs, 48 KB of LDS): 2286 x 2286
// has 648 of them for 768 places, where 128 x 128 tiles at two per CU would leave a
// third of the chip idle. The operands are split while they are staged, so nothing
// is read twice and no workspace is kept; B is stored once for C_r and once for C_i.
// 2590 to 2690 us at 2286 x 2286 x 8192 (FP32 cores 4361): 1020 to 1060 TFLOP/s of BF16
// products, with the splitting (VALU) beside them.
constexpr int SN = 64;                                        // tile columns
constexpr int S_PLANE_A = TM * TK, S_PLANE_B = SN * TK;  // words (two BF16) of a plane

typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8_t;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// 16-byte chunk c (8 k) of a row in LDS: rows of 64 bytes, chunks permuted so that the
// lanes of a fragment read (consecutive rows) cover all banks
__device__ __forceinline__ int chunk_at(int row, int c) { return row * 4 + (c ^ ((row >> 1) & 3)); }

// the three planes of two values, packed (low half: a)
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const bf16x2_t r = __builtin_convertvector(f32x2{a, b}, bf16x2_t);  // to nearest
  unsigned w;
  __builtin_memcpy(&w, &r, sizeof w);
  return w;
}

__device__ __forceinline__ void split2(float a, float b, unsigned& p1, unsigned& p2, unsigned& p3) {
  p1 = pack_bf16(a, b);
  const float a2 = a - __uint_as_float(p1 << 16), b2 = b - __uint_as_float(p1 & 0xffff0000u);
  p2 = pack_bf16(a2, b2);
  const float a3 = a2 - __uint_as_float(p2 << 16), b3 = b2 - __uint_as_float(p2 & 0xffff0000u);
  p3 = pack_bf16(a3, b3);
}

constexpr float UP = 0x1p24f, DOWN = 0x1p-48f;  // on the operands while they are staged, on the result
constexpr float SEEN = 0x1p44f;                 // (staged) magnitudes below it are not published
constexpr int SEEN_BITS = (127 + 44) << 23;

// the tile's largest magnitude of an operand, as a bit pattern in LDS
__device__ __forceinline__ void publish(int& most, float seen) {
  if (seen > SEEN && __float_as_int(seen) > most) atomicMax(&most, __float_as_int(seen));
}

// One unit: four complex k of one row (a 16-byte chunk of each plane). A thread
// stages two units of A and one of B per step. Rows past the end repeat the last
// row (their results are not stored), k past the end are zeroed in the last step;
// the buffer's range keeps every load inside the operand.
struct Unit {
  float2 v[4];
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const float2* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000);
}

// 32 bytes at byte offset `at`, or four values ld bytes apart
template <bool wide>
__device__ __forceinline__ void unit_load(Unit& u, __amdgpu_buffer_rsrc_t r, int at, int ld) {
  if (wide) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, at + 16 * i, 0, 0);
      u.v[2 * i] = make_float2(__uint_as_float(w[0]), __uint_as_float(w[1]));
      u.v[2 * i + 1] = make_float2(__uint_as_float(w[2]), __uint_as_float(w[3]));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, at + i * ld, 0, 0);
      u.v[i] = make_float2(__uint_as_float(w[0]), __uint_as_float(w[1]));
    }
  }
}

// the unit's first `left` values are inside K
__device__ __forceinline__ void unit_tail(Unit& u, int left) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i >= left) u.v[i] = make_float2(0.f, 0.f);
}

// A unit into its three LDS planes (chunk index of the unit, words of a plane); B's
// for C_r and, three planes on, for C_i
template <bool isB>
__device__ __forceinline__ void split_store(unsigned* lds, int plane, int chunk, const Unit& u, float& seen) {
  u32x4 w[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    unsigned x, y, z;
    const float re = UP * u.v[i].x, im = UP * u.v[i].y;
    seen = fmaxf(fmaxf(seen, fabsf(re)), fabsf(im));
    split2(re, im, x, y, z);
    w[0][i] = x, w[1][i] = y, w[2][i] = z;
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    unsigned* const at = lds + p * plane + 4 * chunk;
    if (!isB) {
      *(u32x4*)at = w[p];
    } else {
      u32x4 r, q;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r[e] = w[p][e] ^ 0x80000000u;                           // (re, -im)
        q[e] = __builtin_amdgcn_alignbit(w[p][e], w[p][e], 16);  // (im, re)
      }
      *(u32x4*)at = r;
      *(u32x4*)(at + 3 * plane) = q;
    }
  }
}

__device__ __forceinline__ bf16x8_t as_bf16(u32x4 v) {
  bf16x8_t r;
  __builtin_memcpy(&r, &v, sizeof r);
  return r;
}

// what a stopped tile leaves in its first element: a NaN that no sum gives (one in
// the inputs only costs the tile a second, equal computation)
constexpr unsigned REDO = 0x7fc5a5a5u;

template <bool BK>
__global__ void __launch_bounds__(256, 3) k_cgemm_split(CgemmArgs g) {
  __shared__ __attribute__((aligned(16))) unsigned lds[3 * (S_PLANE_A + 2 * S_PLANE_B)];
  __shared__ int most[2];  // of A, of B
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 32;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * SN;
  unsigned* const sA = lds;
  unsigned* const sB = lds + 3 * S_PLANE_A;
  if (tid < 2) most[tid] = SEEN_BITS;
  f32x16 cr[2][1], ci[2][1];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) cr[i][0][e] = ci[i][0][e] = 0.f;

  // staging: A rows tid / 4 and + 64, k unit tid % 4; B the same or, n-contiguous,
  // column tid % 64 and k unit tid / 64
  const int rows = min(TM, g.M - m0) - 1, cols = min(SN, g.N - n0) - 1;
  const int kuA = tid & 3, kuB = BK ? tid & 3 : wave;
  const int rB = BK ? tid >> 2 : lane;
  const int atA0 = (min(tid >> 2, rows) * (int)g.lda + 4 * kuA) * 8;
  const int atA1 = (min((tid >> 2) + 64, rows) * (int)g.lda + 4 * kuA) * 8;
  const int ldB = (int)g.ldb * 8;
  const int atB = BK ? min(rB, cols) * ldB + 32 * kuB : 4 * kuB * ldB + min(rB, cols) * 8;
  const float2* const pA = g.A + (int64_t)m0 * g.lda;
  const float2* const pB = g.B + (BK ? (int64_t)n0 * g.ldb : n0);
  Unit ra0, ra1, rb;
  float seenA = 0.f, seenB = 0.f;
  auto load = [&](int k0) {
    const auto A = buffer_of(pA + k0, ((int64_t)rows * g.lda + g.K - k0) * 8);
    const auto B = BK ? buffer_of(pB + k0, ((int64_t)cols * g.ldb + g.K - k0) * 8)
                      : buffer_of(pB + (int64_t)k0 * g.ldb, ((int64_t)(g.K - k0 - 1) * g.ldb + cols + 1) * 8);
    if (k0 + TK <= g.K) {
      unit_load<true>(ra0, A, atA0, 0);
      unit_load<true>(ra1, A, atA1, 0);
      unit_load<BK>(rb, B, atB, ldB);
    } else {  // no load straddles the end of the range
      unit_load<false>(ra0, A, atA0, 8);
      unit_load<false>(ra1, A, atA1, 8);
      unit_load<false>(rb, B, atB, BK ? 8 : ldB);
    }
  };
  load(0);
  for (int k0 = 0; k0 < g.K; k0 += TK) {
    __syncthreads();  // the last step's reads are done
    if (k0 + TK > g.K) {
      unit_tail(ra0, g.K - k0 - 4 * kuA);
      unit_tail(ra1, g.K - k0 - 4 * kuA);
      unit_tail(rb, g.K - k0 - 4 * kuB);
    }
    split_store<false>(sA, S_PLANE_A, chunk_at(tid >> 2, kuA), ra0, seenA);
    split_store<false>(sA, S_PLANE_A, chunk_at((tid >> 2) + 64, kuA), ra1, seenA);
    split_store<true>(sB, S_PLANE_B, chunk_at(rB, kuB), rb, seenB);
    publish(most[0], seenA);
    publish(most[1], seenB);
    __syncthreads();
    // (next written behind the next barrier)
    if (__builtin_amdgcn_readfirstlane((most[0] >> 23) + (most[1] >> 23)) > g.range) {
      if (tid == 0) g.C[(int64_t)m0 * g.ldc + n0].x = __uint_as_float(REDO);
      return;
    }
    if (k0 + TK < g.K) load(k0 + TK);
    // one 32 x 32 block and part after the other, so that its two sums are the only ones beside
    // the total's (168 VGPRs): two blocks at a time spill, 2.9 ms against 2.6
    auto fragA = [&](int p, int i, int k16) {
      const int at = chunk_at(wm + 32 * i + (lane & 31), 2 * k16 + (lane >> 5));
      return as_bf16(*(const u32x4*)(sA + p * S_PLANE_A + 4 * at));
    };
    auto fragB = [&](int part, int p, int k16) {
      const int at = chunk_at(wn + (lane & 31), 2 * k16 + (lane >> 5));
      return as_bf16(*(const u32x4*)(sB + (3 * part + p) * S_PLANE_B + 4 * at));
    };
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f32x16 low = {}, high = {};
#pragma unroll
        for (int k16 = 0; k16 < 2; ++k16) {
          bf16x8_t a[3], b[3];
#pragma unroll
          for (int p = 0; p < 3; ++p) a[p] = fragA(p, i, k16), b[p] = fragB(part, p, k16);
#pragma unroll
          for (int lev = 3; lev >= 1; --lev)
#pragma unroll
            for (int p = min(lev, 2); p >= max(lev - 2, 0); --p)
              low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[lev - p], b[p], low, 0, 0, 0);
          high = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], high, 0, 0, 0);
        }
        f32x16& to = part ? ci[i][0] : cr[i][0];
#pragma unroll
        for (int e = 0; e < 16; ++e) to[e] += high[e] + low[e];
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  store_tile<1>(g, cr, ci, m0 + wm, n0 + wn, DOWN);
}

// the tiles that the split could not take
template <bool BK>
__global__ void __launch_bounds__(256, 2) k_cgemm_redo(CgemmArgs g) {
  __shared__ float2 lds[2 * TK * (TM + SN)];
  __shared__ bool redo;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * SN;
  if (threadIdx.x == 0) redo = __float_as_uint(g.C[(int64_t)m0 * g.ldc + n0].x) == REDO;
  __syncthreads();
  if (redo) tile_f32<1, BK>(g, m0, n0, lds);
}

}  // namespace

int launch_cgemm(int M, int N, int K, const void* A, int64_t lda, const void* B, int64_t ldb, int trans_b, void* C,
                 int64_t ldc, int conj_c, void* stream) {
  if (M <= 0 || N <= 0) return 0;
  if (K <= 0 || !A || !B || !C || lda < K || (trans_b ? ldb < K : ldb < N) || ldc < N)
    return (int)hipErrorInvalidValue;
  if ((int64_t)(M + TM - 1) / TM > 65535) return (int)hipErrorInvalidValue;
  CgemmArgs g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.A = (const float2*)A;
  g.lda = lda;
  g.B = (const float2*)B;
  g.ldb = ldb;
  g.trans_b = trans_b;
  g.C = (float2*)C;
  g.ldc = ldc;
  g.conj_c = conj_c;
  g.veca = lda % 2 == 0 && (uintptr_t)A % 16 == 0;
  g.vecb = ldb % 2 == 0 && (uintptr_t)B % 16 == 0;
  // sums of 2 K products of values up to 2^(e + 1) stay below 2^127
  int lg = 0;
  while ((1ll << lg) < K) ++lg;
  g.range = 127 - 3 - lg + 2 * 127;
  // 32-bit offsets inside a tile's rows
  if (K >= SPLIT_K && lda < (1 << 20) && ldb < (1 << 20)) {
    const dim3 grid((N + SN - 1) / SN, (M + TM - 1) / TM);
    (trans_b ? k_cgemm_split<true> : k_cgemm_split<false>)<<<grid, 256, 0, (hipStream_t)stream>>>(g);
    (trans_b ? k_cgemm_redo<true> : k_cgemm_redo<false>)<<<grid, 256, 0, (hipStream_t)stream>>>(g);
  } else {
    const dim3 grid((N + 127) / 128, (M + TM - 1) / TM);
    (trans_b ? k_cgemm_mfma<true> : k_cgemm_mfma<false>)<<<grid, 256, 0, (hipStream_t)stream>>>(g);
  }
  return (int)hipGetLastError();
}

}  // namespace tmk
