// Preprocessing of the camera image stack (Sec. 2.2, the paragraph after
// Algorithm 1). The kept pixels of an H x W image are its 1-based odd rows and
// columns (0-based even), a (H/2) x (W/2) grid indexed q = y (W/2) + x.
//  * energy: per kept pixel, the intensity summed over all images (FP64),
//    in image chunks (partials) and a fixed-order final sum;
//  * mask: the smallest brightest-first set of kept pixels whose summed
//    intensity first reaches frac of the total (ties by raster index), as
//    ascending raster indices: ranks by counting over the whole chip, then one
//    workgroup adds up the sorted energies and compacts the kept pixels;
//  * gather: the per-pixel rows out[p][i] (i = image = measurement index),
//    a transpose through LDS tiles of 64 images x 256 pixels so that both the
//    image reads and the row writes are contiguous.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "pre.hpp"

namespace tmk {

namespace {

__device__ __forceinline__ float pix_val(const void* s, int u16, size_t idx) {
  return u16 ? (float)((const uint16_t*)s)[idx] : ((const float*)s)[idx];
}

__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Scalar form: grid (ceil(npix / 256), nchunks), thread = kept pixel, loop
// over the chunk's images.
__global__ void __launch_bounds__(256) k_energy_part(const void* stack, int u16, int64_t n_img, int H, int W,
                                                     int64_t chunk, double* partial) {
  const int npix = (H / 2) * (W / 2);
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= npix) return;
  const int y = q / (W / 2), x = q - y * (W / 2);
  const size_t off = (size_t)(2 * y) * W + 2 * x;
  const int64_t i0 = (int64_t)blockIdx.y * chunk;
  const int64_t i1 = (i0 + chunk < n_img) ? i0 + chunk : n_img;
  double s = 0.0;
  for (int64_t i = i0; i < i1; ++i) s += (double)pix_val(stack, u16, (size_t)i * H * W + off);
  partial[(size_t)blockIdx.y * npix + q] = s;
}

// Vector form (16-byte rows segments): a thread owns one 16-byte segment of an
// even row, i.e. KP kept pixels (4 for uint16, 2 for float), and loops over
// the chunk's images with one 16-byte load each. grid (ceil(nseg / 256),
// nchunks), nseg = (H/2) * (W * sizeof / 16).
template <bool U16>
__global__ void __launch_bounds__(256) k_energy_vec(const void* stack, int64_t n_img, int H, int W, int64_t chunk,
                                                    double* partial) {
  constexpr int EPS = U16 ? 8 : 4;  // elements per segment
  constexpr int KP = EPS / 2;       // kept pixels per segment
  const int segs = W / EPS, npix = (H / 2) * (W / 2);
  const int sgi = blockIdx.x * 256 + threadIdx.x;
  if (sgi >= (H / 2) * segs) return;
  const int y = sgi / segs, sx = sgi - y * segs;
  const size_t off = (size_t)(2 * y) * W + (size_t)sx * EPS;
  const size_t plane = (size_t)H * W;
  const int64_t i0 = (int64_t)blockIdx.y * chunk;
  const int64_t i1 = (i0 + chunk < n_img) ? i0 + chunk : n_img;
  double acc[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) acc[k] = 0.0;
#pragma unroll 4
  for (int64_t i = i0; i < i1; ++i) {
    const uint4 v = *(const uint4*)((const char*)stack + (i * plane + off) * (U16 ? 2 : 4));
    if (U16) {
      acc[0] += (double)(v.x & 0xffffu);
      acc[1] += (double)(v.y & 0xffffu);
      acc[2] += (double)(v.z & 0xffffu);
      acc[3] += (double)(v.w & 0xffffu);
    } else {
      acc[0] += (double)__uint_as_float(v.x);
      acc[1] += (double)__uint_as_float(v.z);
    }
  }
  const int q = y * (W / 2) + sx * KP;
#pragma unroll
  for (int k = 0; k < KP; ++k) partial[(size_t)blockIdx.y * npix + q + k] = acc[k];
}

__global__ void __launch_bounds__(256) k_energy_final(const double* partial, int nchunks, int npix, double* energy) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= npix) return;
  double s = 0.0;
#pragma unroll 8
  for (int c = 0; c < nchunks; ++c) s += partial[(size_t)c * npix + q];
  energy[q] = s;
}

// The brightest-first order by counting: the rank of a pixel is the number of
// pixels before it (brighter; equal and of smaller raster index; a NaN comes after
// every number). A workgroup holds 16 pixels and reads all of them once, so that
// npix squared compares (16.8 M at 64 x 64) spread over the chip; one workgroup's
// bitonic sort of them took most of 141 us, this 10.5.
constexpr int RANK_P = 16;

// ascending in brightest-first order
__device__ __forceinline__ uint64_t dim_key(double e) {
  const int64_t u = __double_as_longlong(e + 0.0);  // -0 as 0
  return e != e ? ~1ull : (uint64_t)(u < 0 ? u : ~u ^ (1ll << 63));
}

__global__ void __launch_bounds__(256) k_rank(const double* __restrict__ energy, int npix, double* __restrict__ sorted,
                                             int32_t* __restrict__ rank) {
  __shared__ int part[4][RANK_P];
  const int q0 = blockIdx.x * RANK_P, tid = threadIdx.x;
  uint64_t k[RANK_P];
  int n[RANK_P];
#pragma unroll
  for (int i = 0; i < RANK_P; ++i) {
    k[i] = dim_key(energy[min(q0 + i, npix - 1)]);
    n[i] = 0;
  }
#pragma unroll 4
  for (int t = tid; t < npix; t += 256) {
    const uint64_t x = dim_key(energy[t]);
#pragma unroll
    for (int i = 0; i < RANK_P; ++i) n[i] += x < k[i] + (t < q0 + i ? 1 : 0) ? 1 : 0;
  }
#pragma unroll
  for (int i = 0; i < RANK_P; ++i) {
    for (int off = 32; off >= 1; off >>= 1) n[i] += __shfl_xor(n[i], off, 64);
    if ((tid & 63) == 0) part[tid >> 6][i] = n[i];
  }
  __syncthreads();
  if (tid < RANK_P && q0 + tid < npix) {
    const int r = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid];
    sorted[r] = energy[q0 + tid];
    rank[q0 + tid] = r;
  }
}

constexpr int MWG = 1024, MPT = PRE_MASK_MAX / MWG;

// Up to two waves' pixels k_mask counts the ranks itself (energy given, sorted and rank
// unused): the launch costs more than the count (64 pixels, with the count read back: 45 us in
// two launches, 42.4 by the bitonic sort before, 39.6 in one).
constexpr int MASK_ONE = 128;

// One workgroup; thread t holds the sorted positions t + 1024 c. Running sums in the
// Hillis-Steele order: partners less than 1024 apart through LDS (two buffers, one
// barrier a step), the others in the same thread; bound by the chain of those steps:
// 12.7 us at 64 x 64.
__global__ void __launch_bounds__(MWG) k_mask(const double* __restrict__ energy, const double* __restrict__ sorted,
                                             const int32_t* __restrict__ rank, int npix, double frac, int32_t* pix,
                                             int32_t* count_dev) {
  __shared__ double buf[2][PRE_MASK_MAX];
  __shared__ double red[MWG / 64];
  __shared__ int kept[MPT * (MWG / 64)];
  __shared__ int first;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double v[MPT];
  double tot = 0.0;
  int own = 0;  // rank of pixel tid, counted here
  const bool one = npix <= MASK_ONE;
  if (one) {
    const double e = energy[min(tid, npix - 1)];
    const uint64_t k = dim_key(e);
    uint64_t* keys = (uint64_t*)buf[0];
    if (tid < npix) keys[tid] = k;
    __syncthreads();
    if (tid < npix) {
#pragma unroll 8
      for (int t = 0; t < npix; ++t) own += keys[t] < k + (t < tid ? 1 : 0) ? 1 : 0;
      buf[1][own] = e;
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < MPT; ++c) {
    const int t = tid + c * MWG;
    v[c] = (t < npix) ? (one ? buf[1][t] : sorted[t]) : 0.0;
    if (t < npix) tot += v[c];
  }
  for (int off = 32; off >= 1; off >>= 1) tot += __shfl_xor(tot, off, 64);
  if (lane == 0) red[wave] = tot;
  if (tid == 0) first = npix;
  int cur = 0;
  for (int d = 1; d < MWG && d < npix; d <<= 1, cur ^= 1) {
#pragma unroll
    for (int c = 0; c < MPT; ++c)
      if (c * MWG < npix) buf[cur][tid + c * MWG] = v[c];
    __syncthreads();  // the step before last read this buffer, before the last step's barrier
#pragma unroll
    for (int c = 0; c < MPT; ++c)
      if (c * MWG < npix && tid + c * MWG >= d) v[c] += buf[cur][tid + c * MWG - d];
  }
#pragma unroll
  for (int m = 1; m < MPT; m <<= 1) {
#pragma unroll
    for (int c = MPT - 1; c >= m; --c)
      if (m * MWG < npix) v[c] += v[c - m];
  }
  __syncthreads();
  double total = 0.0;
  for (int w = 0; w < MWG / 64; ++w) total += red[w];
  // count = (first position whose running sum reaches frac * total) + 1
  const double thr = frac * total;
  int f = npix;
#pragma unroll
  for (int c = MPT - 1; c >= 0; --c)
    if (tid + c * MWG < npix && v[c] >= thr) f = tid + c * MWG;
  for (int off = 32; off >= 1; off >>= 1) f = min(f, __shfl_xor(f, off, 64));
  if (lane == 0) atomicMin(&first, f);
  __syncthreads();
  const int count = (total > 0.0) ? ((first < npix) ? first + 1 : npix) : 0;
  // kept pixels in raster order: places within the wave from the ballot, then the waves'
  unsigned long long keep[MPT];
#pragma unroll
  for (int c = 0; c < MPT; ++c) {
    const int t = tid + c * MWG;
    keep[c] = __ballot(t < npix && (one ? own : rank[t]) < count);
    if (lane == 0) kept[c * (MWG / 64) + wave] = __popcll(keep[c]);
  }
  __syncthreads();
  // running sums of the waves' counts, entry c (MWG / 64) + wave, two per lane
  static_assert(MPT * (MWG / 64) == 128, "two counts per lane");
  int lo = kept[lane], hi = kept[64 + lane];
  for (int d = 1; d < 64; d <<= 1) {
    const int a = __shfl_up(lo, d, 64), b = __shfl_up(hi, d, 64);
    if (lane >= d) lo += a, hi += b;
  }
  hi += __shfl(lo, 63, 64);
#pragma unroll
  for (int c = 0; c < MPT; ++c) {
    const int e = c * (MWG / 64) + wave - 1;  // the entry before this wave's
    const int base = e < 0 ? 0 : __shfl(e < 64 ? lo : hi, e & 63, 64);
    if (keep[c] >> lane & 1) pix[base + __popcll(keep[c] & ((1ull << lane) - 1))] = tid + c * MWG;
  }
  if (tid == 0) *count_dev = count;
}

constexpr int GT_I = 64, GT_P = 256;

// grid (ceil(P / 256), ceil(n_img / 64)), 256 threads. Bound by the memory: 64 images
// give each pixel row 256 bytes (128 in bfloat16) in one piece, and 32 loads of a
// thread are in flight at a time. The tile keeps the source's type. 32768 uint16 images
// of 128 x 128, 2206 kept pixels: 131 us, 5.3 TB/s (237 with 32 images and 8 loads).
template <typename T>
__global__ void __launch_bounds__(256) k_gather(const T* __restrict__ stack, int64_t n_img, int H, int W,
                                               const int32_t* __restrict__ pix, int P, void* out, int out_bf16) {
  __shared__ T tile[GT_I][GT_P + (sizeof(T) == 2 ? 2 : 1)];
  const int p0 = blockIdx.x * GT_P;
  const int64_t i0 = (int64_t)blockIdx.y * GT_I;
  const int p = p0 + threadIdx.x;
  const size_t plane = (size_t)H * W;
  if (p < P) {
    const int q = pix[p];
    const int y = q / (W / 2), x = q - y * (W / 2);
    const T* src = stack + (size_t)i0 * plane + (size_t)(2 * y) * W + 2 * x;
    const int left = (int)(n_img - i0 < GT_I ? n_img - i0 : GT_I);
    if (left == GT_I) {
#pragma unroll
      for (int h = 0; h < GT_I; h += 32) {
        T v[32];
#pragma unroll
        for (int r = 0; r < 32; ++r) v[r] = src[(h + r) * plane];
#pragma unroll
        for (int r = 0; r < 32; ++r) tile[h + r][threadIdx.x] = v[r];
      }
    } else {
      for (int r = 0; r < left; ++r) tile[r][threadIdx.x] = src[r * plane];
    }
  }
  __syncthreads();
  // 4 consecutive images per thread, 16 threads per pixel, 16 pixels per pass
  const int r4 = (threadIdx.x & 15) * 4;
  const int64_t i = i0 + r4;
  const bool whole = i + 3 < n_img && ((uintptr_t)out % 16) == 0;
#pragma unroll 4
  for (int pp = threadIdx.x >> 4; pp < GT_P; pp += 16) {
    const int pg = p0 + pp;
    if (pg >= P) break;
    const size_t o = (size_t)pg * n_img + i;
    const float v0 = (float)tile[r4][pp], v1 = (float)tile[r4 + 1][pp], v2 = (float)tile[r4 + 2][pp],
                v3 = (float)tile[r4 + 3][pp];
    if (whole && (o & 3) == 0) {
      if (out_bf16) {
        uint2 w;
        w.x = (uint32_t)to_bf16(v0) | ((uint32_t)to_bf16(v1) << 16);
        w.y = (uint32_t)to_bf16(v2) | ((uint32_t)to_bf16(v3) << 16);
        *(uint2*)((uint16_t*)out + o) = w;
      } else {
        *(float4*)((float*)out + o) = make_float4(v0, v1, v2, v3);
      }
    } else {
      const float v[4] = {v0, v1, v2, v3};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (i + k < n_img) {
          if (out_bf16) ((uint16_t*)out)[o + k] = to_bf16(v[k]);
          else ((float*)out)[o + k] = v[k];
        }
      }
    }
  }
}

}  // namespace

// The vector form needs whole 16-byte segments per row and a 16-byte aligned stack.
static bool energy_vec(const void* stack, int u16, int W) {
  return (W % (u16 ? 8 : 4)) == 0 && ((uintptr_t)stack % 16) == 0;
}

static int energy_threads(const void* stack, int u16, int H, int W) {
  return energy_vec(stack, u16, W) ? (H / 2) * (W / (u16 ? 8 : 4)) : (H / 2) * (W / 2);
}

int pre_energy_chunks(const void* stack, int u16, int64_t n_img, int H, int W) {
  // about 1024 workgroups, at least 32 images per chunk, at most 128 chunks (the
  // final pass adds the chunks of each pixel in order)
  const int blocks_x = (energy_threads(stack, u16, H, W) + 255) / 256;
  int64_t c = (1024 + blocks_x - 1) / blocks_x;
  const int64_t maxc = (n_img + 31) / 32;
  if (c > maxc) c = maxc;
  if (c > 128) c = 128;
  return (int)(c < 1 ? 1 : c);
}

int launch_pre_energy(const void* stack, int u16, int64_t n_img, int H, int W, double* partial, int nchunks,
                      double* energy, void* stream) {
  const int npix = (H / 2) * (W / 2);
  const int64_t chunk = (n_img + nchunks - 1) / nchunks;
  hipStream_t s = (hipStream_t)stream;
  dim3 g((energy_threads(stack, u16, H, W) + 255) / 256, nchunks);
  if (!energy_vec(stack, u16, W)) k_energy_part<<<g, 256, 0, s>>>(stack, u16, n_img, H, W, chunk, partial);
  else if (u16) k_energy_vec<true><<<g, 256, 0, s>>>(stack, n_img, H, W, chunk, partial);
  else k_energy_vec<false><<<g, 256, 0, s>>>(stack, n_img, H, W, chunk, partial);
  k_energy_final<<<(npix + 255) / 256, 256, 0, s>>>(partial, nchunks, npix, energy);
  return (int)hipGetLastError();
}

size_t pre_mask_scratch(int npix) { return (size_t)npix * (sizeof(double) + sizeof(int32_t)) + sizeof(int32_t); }

int launch_pre_mask(const double* energy, int npix, double frac, int32_t* pix, void* scratch, int32_t** count_dev,
                    void* stream) {
  double* sorted = (double*)scratch;
  int32_t* rank = (int32_t*)(sorted + npix);
  *count_dev = rank + npix;
  if (npix > MASK_ONE) k_rank<<<(npix + RANK_P - 1) / RANK_P, 256, 0, (hipStream_t)stream>>>(energy, npix, sorted, rank);
  k_mask<<<1, MWG, 0, (hipStream_t)stream>>>(energy, sorted, rank, npix, frac, pix, *count_dev);
  return (int)hipGetLastError();
}

int launch_pre_gather(const void* stack, int u16, int64_t n_img, int H, int W, const int32_t* pix, int P, void* out,
                      int out_bf16, void* stream) {
  if (P <= 0 || n_img <= 0) return 0;
  dim3 g((P + GT_P - 1) / GT_P, (unsigned)((n_img + GT_I - 1) / GT_I));
  hipStream_t s = (hipStream_t)stream;
  if (u16) k_gather<<<g, 256, 0, s>>>((const uint16_t*)stack, n_img, H, W, pix, P, out, out_bf16);
  else k_gather<<<g, 256, 0, s>>>((const float*)stack, n_img, H, W, pix, P, out, out_bf16);
  return (int)hipGetLastError();
}

}  // namespace tmk
