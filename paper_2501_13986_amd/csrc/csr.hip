// Integer graph preparation on the device: COO -> CSR by receiver plus the transpose
// permutation (paper Sec. 3.5: the fused kernels need row-sorted edges, and the backward pass
// a permutation that transposes the adjacency), and two small helpers of the conv path.
// Statically compiled (nothing here depends on the irreps).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <mutex>

#include <rocprim/rocprim.hpp>

#include "csr.hpp"

namespace cgtp {
namespace {

constexpr int kBlock = 256;

template <class K>
__global__ void k_make_keys(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t E, int64_t V,
                            K* __restrict__ keys, int64_t* __restrict__ idx, int* __restrict__ bad) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  int64_t r = recv[e], s = send[e];
  if (r < 0 || r >= V || s < 0 || s >= V) {
    *bad = 1;  // plain store of the same value from any thread
    r = 0;
    s = 0;
  }
  keys[e] = (K)((uint64_t)r * (uint64_t)V + (uint64_t)s);
  idx[e] = e;
}

// first position whose key is >= target, for targets j*stride, j = 0..V
template <class K>
__global__ void k_lower_bounds(const K* __restrict__ keys, int64_t E, int64_t V, uint64_t stride,
                               int64_t* __restrict__ ptr) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j > V) return;
  uint64_t target = (uint64_t)j * stride;
  int64_t lo = 0, hi = E;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    if ((uint64_t)keys[mid] < target) lo = mid + 1; else hi = mid;
  }
  ptr[j] = lo;
}

template <class K>
__global__ void k_col_from_perm(const int64_t* __restrict__ send, const int64_t* __restrict__ perm, int64_t E,
                                int64_t* __restrict__ col, K* __restrict__ colkey, int64_t* __restrict__ pos) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  int64_t c = send[perm[e]];
  col[e] = c;
  colkey[e] = (K)c;
  pos[e] = e;
}

// receiver (CSR row) of the edge at every position of the transposed order
__global__ void k_recv_of_tperm(const int64_t* __restrict__ row_ptr, const int64_t* __restrict__ t_perm, int64_t V,
                                int64_t E, int64_t* __restrict__ t_recv) {
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= E) return;
  int64_t e = t_perm[q];
  int64_t lo = 0, hi = V;  // row_ptr[lo] <= e < row_ptr[hi]
  while (hi - lo > 1) {
    int64_t mid = (lo + hi) >> 1;
    if (row_ptr[mid] <= e) lo = mid; else hi = mid;
  }
  t_recv[q] = lo;
}

__global__ void k_fill_zero(uint32_t* __restrict__ p, int64_t n_words) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (; i < n_words; i += step) p[i] = 0u;
}

template <typename T>
__global__ void k_add_inplace(T* __restrict__ a, const T* __restrict__ b, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += step) a[i] += b[i];
}

// ---- bucket path: graphs of up to about 2.6 million edges ---------------------------------------------------------------
// A general radix sort costs a launch or two per digit or merge round (ten rounds for 800 000 keys, twice), each a few
// microseconds long whatever it does.  Here the edges are cut once into at most 1 024 buckets of consecutive rows, and
// one workgroup finishes a bucket in LDS: rows are placed by counting, and the order inside a row comes from counting
// the smaller records of that row (unique records: row, other end, original position packed into 64 bits, so the order
// of arrival does not matter and the result is the stable one).  The kernel that finishes the receivers hands its edges
// on to the buckets of the senders.  Five launches for any size, one if the graph fits a single workgroup.
// What is left is the latency of dependent passes.  Synchronous call, sorts -> buckets: 27 nodes of degree 9 72 -> 28 us,
// 300 nodes of degree 20 118 -> 45, 3 001 nodes of degree 32 176 -> 53, 20 000 nodes of degree 40 416 -> 81 us (kernels
// 2 + 9 + 14 + 21 + 14); conv_forward_perm + conv_backward_perm with the preparation, 3 001 nodes of 32 channels 343 -> 243 us.
constexpr int kThreads = 1024;     // of every kernel of this path; one thread per bucket in the scans
constexpr int kBuckets = 1024;
constexpr int kPer = 4;            // records of a thread
constexpr int kCap = kThreads * kPer;
constexpr int kRows = 4096;        // rows of a bucket
constexpr int kTilePer = 8;        // edges of a thread in the counting and distributing passes
constexpr int kTile = kThreads * kTilePer;

struct BucketPlan {
  int shift, nb, eb, vb;   // bucket of a row = row >> shift; number of buckets; bits of an edge index and of a node index
};

struct BucketWs {          // in the caller's workspace
  int *total1, *total2, *base1, *base2, *cursor2, *before;   // zeroed: total1, total2
  uint64_t *rec1, *rec2;
};

struct SortLds {
  uint64_t rec[kCap];
  int off[kRows + 1];
  int wave[kThreads / 64];
};

// exclusive sum over the 1 024 threads of the workgroup
__device__ __forceinline__ int block_scan(int v, int* wave) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int s = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(s, o, 64);
    s += lane >= o ? t : 0;
  }
  if (lane == 63) wave[w] = s;
  __syncthreads();
  int before = 0;
  for (int i = 0; i < kThreads / 64; ++i) before += i < w ? wave[i] : 0;
  __syncthreads();
  return before + s - v;
}

// rec[j] (valid for threadIdx.x + j * 1024 < n, row = rec >> row_bits < rows): on return rec[j] is some record of the same
// set and pos[j] its place in ascending order; S.off[r] = first place of row r, S.off[rows] = n.
__device__ __forceinline__ void sort_in_lds(SortLds& S, uint64_t (&rec)[kPer], int (&pos)[kPer], int n, int rows, int row_bits) {
  const int t = threadIdx.x;
  for (int r = t; r <= rows; r += kThreads) S.off[r] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) pos[j] = atomicAdd(&S.off[(int)(rec[j] >> row_bits)], 1);
  __syncthreads();
  constexpr int kRowsPer = kRows / kThreads;
  int c[kRowsPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kRowsPer; ++q) {
    const int r = t * kRowsPer + q;
    c[q] = r < rows ? S.off[r] : 0;
    sum += c[q];
  }
  int at = block_scan(sum, S.wave);
#pragma unroll
  for (int q = 0; q < kRowsPer; ++q) {
    const int r = t * kRowsPer + q;
    if (r < rows) S.off[r] = at;
    at += c[q];
  }
  if (t == 0) S.off[rows] = n;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) S.rec[S.off[(int)(rec[j] >> row_bits)] + pos[j]] = rec[j];
  __syncthreads();
  // neighbouring lanes now hold records of the same row: their reads of the row are broadcasts
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) {
      const uint64_t k = S.rec[t + j * kThreads];
      const int r = (int)(k >> row_bits), beg = S.off[r], end = S.off[r + 1];
      int less = beg;
#pragma unroll 4
      for (int q = beg; q < end; ++q) less += S.rec[q] < k ? 1 : 0;
      rec[j] = k;
      pos[j] = less;
    }
}

__device__ __forceinline__ bool load_edge(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t e, int64_t V,
                                          uint64_t& r, uint64_t& s) {
  r = (uint64_t)recv[e];
  s = (uint64_t)send[e];
  const bool ok = r < (uint64_t)V && s < (uint64_t)V;   // also refuses negative values
  if (!ok) r = s = 0;
  return ok;
}

// E <= 4 096 and V <= 4 096: everything in one workgroup
__global__ void __launch_bounds__(kThreads) k_csr_small(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int E, int V,
                                                        int eb, int vb, int64_t* __restrict__ row_ptr, int64_t* __restrict__ col,
                                                        int64_t* __restrict__ perm, int64_t* __restrict__ t_row_ptr,
                                                        int64_t* __restrict__ t_perm, int* __restrict__ bad_flag) {
  __shared__ SortLds S;
  const int t = threadIdx.x;
  const uint64_t emask = ((uint64_t)1 << eb) - 1, vmask = ((uint64_t)1 << vb) - 1;
  uint64_t rec[kPer];
  int pos[kPer], bad = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int e = t + j * kThreads;
    rec[j] = 0;
    pos[j] = 0;
    if (e < E) {
      uint64_t r, s;
      if (!load_edge(recv, send, e, V, r, s)) bad = 1;
      rec[j] = (r << (eb + vb)) | (s << eb) | (uint64_t)e;
    }
  }
  bad = __syncthreads_or(bad);
  if (t == 0 && bad_flag) *bad_flag = bad ? 1 : 0;
  sort_in_lds(S, rec, pos, E, V, eb + vb);
  for (int r = t; r <= V; r += kThreads) row_ptr[r] = S.off[r];
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < E) {
      const uint64_t s = (rec[j] >> eb) & vmask;
      perm[pos[j]] = (int64_t)(rec[j] & emask);
      col[pos[j]] = (int64_t)s;
      rec[j] = (s << eb) | (uint64_t)pos[j];
    }
  if (!t_row_ptr) return;
  __syncthreads();
  sort_in_lds(S, rec, pos, E, V, eb);
  for (int r = t; r <= V; r += kThreads) t_row_ptr[r] = S.off[r];
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < E) t_perm[pos[j]] = (int64_t)(rec[j] & emask);
}

__global__ void k_csr_clear(int* __restrict__ totals, int n, int* __restrict__ bad) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) totals[i] = 0;
  if (i == 0) *bad = 0;
}

// edges per bucket of receivers and of senders; before[block][bucket]: edges of that bucket that other workgroups placed
// ahead of this one's
__global__ void __launch_bounds__(kThreads) k_csr_count(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t E,
                                                        int64_t V, BucketPlan B, BucketWs w, int transpose) {
  __shared__ int h1[kBuckets], h2[kBuckets];
  const int t = threadIdx.x;
  h1[t] = 0;
  h2[t] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kTilePer; ++j) {
    const int64_t e = (int64_t)blockIdx.x * kTile + j * kThreads + t;
    if (e < E) {
      uint64_t r, s;
      (void)load_edge(recv, send, e, V, r, s);
      atomicAdd(&h1[(int)(r >> B.shift)], 1);
      if (transpose) atomicAdd(&h2[(int)(s >> B.shift)], 1);
    }
  }
  __syncthreads();
  if (t < B.nb) {
    const int c1 = h1[t], c2 = h2[t];
    w.before[(int64_t)blockIdx.x * B.nb + t] = c1 ? atomicAdd(&w.total1[t], c1) : 0;
    if (transpose && c2) atomicAdd(&w.total2[t], c2);
  }
}

// records into the buckets of receivers; the last workgroup (if there is a transpose) lays out the buckets of senders
__global__ void __launch_bounds__(kThreads) k_csr_distribute(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t E,
                                                             int64_t V, BucketPlan B, BucketWs w, int tiles, int* __restrict__ bad) {
  __shared__ int dst[kBuckets];
  __shared__ int wave[kThreads / 64];
  const int t = threadIdx.x;
  const bool second = (int)blockIdx.x == tiles;
  const int start = block_scan(t < B.nb ? (second ? w.total2[t] : w.total1[t]) : 0, wave);
  if (second) {
    if (t < B.nb) {
      w.base2[t] = start;
      w.cursor2[t] = start;
    }
    if (t == 0) w.base2[B.nb] = (int)E;
    return;
  }
  if (blockIdx.x == 0) {
    if (t < B.nb) w.base1[t] = start;
    if (t == 0) w.base1[B.nb] = (int)E;
  }
  if (t < B.nb) dst[t] = start + w.before[(int64_t)blockIdx.x * B.nb + t];
  __syncthreads();
  const uint64_t in_bucket = ((uint64_t)1 << B.shift) - 1;
#pragma unroll
  for (int j = 0; j < kTilePer; ++j) {
    const int64_t e = (int64_t)blockIdx.x * kTile + j * kThreads + t;
    if (e < E) {
      uint64_t r, s;
      if (!load_edge(recv, send, e, V, r, s)) *bad = 1;
      const int q = atomicAdd(&dst[(int)(r >> B.shift)], 1);
      w.rec1[q] = ((r & in_bucket) << (B.eb + B.vb)) | (s << B.eb) | (uint64_t)e;
    }
  }
}

// A bucket of more than 4 096 records (a few receivers or senders with very many edges): one workgroup sorts it in global
// memory, 8 bits at a time, between the records and the output array of the bucket's range.  An even number of passes
// leaves the result where it began.  Slow (about 4 us per pass and 1 000 records), but such graphs are not what this
// path is for and the result is the same.
__device__ void sort_in_memory(uint64_t* a, uint64_t* b, int n, int bits, SortLds& S) {
  int* count = S.off;                       // [16 waves][256 digits]
  int* next = (int*)S.rec;                  // [256]
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int passes = ((bits + 7) / 8 + 1) & ~1;
  for (int p = 0; p < passes; ++p) {
    const int sh = p * 8 < 56 ? p * 8 : 56;
    const bool empty = p * 8 >= bits;       // padding pass: keeps the order
    __syncthreads();
    if (t < 256) next[t] = 0;
    __syncthreads();
    for (int i = t; i < n; i += kThreads) atomicAdd(&next[empty ? 0 : (int)((a[i] >> sh) & 255)], 1);
    __syncthreads();
    const int c = t < 256 ? next[t] : 0;
    const int first = block_scan(c, S.wave);
    if (t < 256) next[t] = first;
    for (int i0 = 0; i0 < n; i0 += kThreads) {
      for (int q = t; q < 16 * 256; q += kThreads) count[q] = 0;
      __syncthreads();
      const int i = i0 + t;
      const bool in = i < n;
      const uint64_t k = in ? a[i] : 0;
      const int d = empty ? 0 : (int)((k >> sh) & 255);
      // lanes of this wave with the same digit
      uint64_t same = __ballot(in);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const uint64_t m = __ballot((d >> bit) & 1);
        same &= ((d >> bit) & 1) ? m : ~m;
      }
      const int rank = __popcll(same & (((uint64_t)1 << lane) - 1));
      if (in && rank == 0) count[wv * 256 + d] = __popcll(same);
      __syncthreads();
      if (t < 256) {                        // places of each wave's digit groups, and where the next tile continues
        int at = next[t];
        for (int q = 0; q < 16; ++q) {
          const int v = count[q * 256 + t];
          count[q * 256 + t] = at;
          at += v;
        }
        next[t] = at;
      }
      __syncthreads();
      if (in) b[count[wv * 256 + d] + rank] = k;
      __syncthreads();
    }
    uint64_t* x = a;
    a = b;
    b = x;
  }
  __syncthreads();
}

// One bucket: kSecond false: the rows of its receivers (row_ptr, col, perm), and its edges on to the buckets of senders;
// true: the rows of its senders (t_row_ptr, t_perm).
template <bool kSecond>
__global__ void __launch_bounds__(kThreads) k_csr_rows(BucketPlan B, BucketWs w, int64_t V, int64_t E, int64_t* __restrict__ ptr,
                                                       int64_t* idx, int64_t* __restrict__ col, int transpose) {
  __shared__ SortLds S;
  __shared__ int h2[kSecond ? 1 : kBuckets];
  const int t = threadIdx.x, bucket = blockIdx.x;
  const int base = (kSecond ? w.base2 : w.base1)[bucket], n = (kSecond ? w.base2 : w.base1)[bucket + 1] - base;
  uint64_t* const in = (kSecond ? w.rec2 : w.rec1) + base;
  const int row_bits = B.eb + (kSecond ? 0 : B.vb);
  const int64_t row0 = (int64_t)bucket << B.shift;
  const int rows = (int)(V - row0 < ((int64_t)1 << B.shift) ? V - row0 : (int64_t)1 << B.shift);
  const uint64_t emask = ((uint64_t)1 << B.eb) - 1, vmask = ((uint64_t)1 << B.vb) - 1;
  const uint64_t in_bucket = ((uint64_t)1 << B.shift) - 1;
  if (bucket == B.nb - 1 && t == 0) ptr[V] = E;
  if (n > kCap) {
    sort_in_memory(in, (uint64_t*)(idx + base), n, row_bits + B.shift, S);
    for (int i = t; i < n; i += kThreads) {
      const uint64_t k = in[i];
      const int r = (int)(k >> row_bits);
      for (int q = i > 0 ? (int)(in[i - 1] >> row_bits) + 1 : 0; q <= r; ++q) ptr[row0 + q] = base + i;
      if (i == n - 1)
        for (int q = r + 1; q < rows; ++q) ptr[row0 + q] = base + n;
      idx[base + i] = (int64_t)(k & emask);
      if (!kSecond) {
        const uint64_t s = (k >> B.eb) & vmask;
        col[base + i] = (int64_t)s;
        if (transpose) w.rec2[atomicAdd(&w.cursor2[(int)(s >> B.shift)], 1)] = ((s & in_bucket) << B.eb) | (uint64_t)(base + i);
      }
    }
    return;
  }
  uint64_t rec[kPer];
  int pos[kPer];
  if (!kSecond) h2[t] = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = t + j * kThreads;
    rec[j] = i < n ? in[i] : 0;
    pos[j] = 0;
  }
  sort_in_lds(S, rec, pos, n, rows, row_bits);
  for (int r = t; r < rows; r += kThreads) ptr[row0 + r] = base + S.off[r];
  int rank[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    rank[j] = 0;
    if (t + j * kThreads < n) {
      idx[base + pos[j]] = (int64_t)(rec[j] & emask);
      if (!kSecond) {
        const uint64_t s = (rec[j] >> B.eb) & vmask;
        col[base + pos[j]] = (int64_t)s;
        if (transpose) rank[j] = atomicAdd(&h2[(int)(s >> B.shift)], 1);
      }
    }
  }
  if (kSecond || !transpose) return;
  __syncthreads();
  if (t < B.nb) {
    const int c = h2[t];
    if (c) h2[t] = atomicAdd(&w.cursor2[t], c);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) {
      const uint64_t s = (rec[j] >> B.eb) & vmask;
      w.rec2[h2[(int)(s >> B.shift)] + rank[j]] = ((s & in_bucket) << B.eb) | (uint64_t)(base + pos[j]);
    }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Scratch for the entry point that allocates nothing (conv_forward_static): device memory that exists from the
// moment the library's code is loaded on a GPU until the process ends.  Every GPU holds its own copy at its own
// address; in host code the name below is only a handle for hipGetSymbolAddress, never a device address.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// keeps the array in the code object although no statically compiled kernel of the library reads it: the
// kernels that use it are compiled at run time and get its address as an argument
__attribute__((used)) __attribute__((used)) __global__ void k_touch_static_scratch(int v) {
  if (v == 0x7fffffff) scratch[0] = 0;
}

}  // namespace

hipError_t static_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* per_device[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {   // first call on this device, which is the current one
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

hipError_t launch_recv_of_tperm(const int64_t* row_ptr, const int64_t* t_perm, int64_t V, int64_t E, int64_t* t_recv,
                                hipStream_t st) {
  if (E == 0) return hipSuccess;
  hipLaunchKernelGGL(k_recv_of_tperm, dim3(blocks_for(E)), dim3(kBlock), 0, st, row_ptr, t_perm, V, E, t_recv);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  int64_t words = (int64_t)(bytes / 4);
  unsigned nb = (unsigned)std::min<int64_t>((words + kBlock - 1) / kBlock, 65536);
  hipLaunchKernelGGL(k_fill_zero, dim3(nb), dim3(kBlock), 0, st, (uint32_t*)p, words);
  return hipGetLastError();
}

hipError_t launch_add_inplace(void* a, const void* b, int64_t n, bool f64, hipStream_t st) {
  if (n == 0) return hipSuccess;
  unsigned nb = (unsigned)std::min<int64_t>((n + kBlock - 1) / kBlock, 65536);
  if (f64) hipLaunchKernelGGL(k_add_inplace<double>, dim3(nb), dim3(kBlock), 0, st, (double*)a, (const double*)b, n);
  else hipLaunchKernelGGL(k_add_inplace<float>, dim3(nb), dim3(kBlock), 0, st, (float*)a, (const float*)b, n);
  return hipGetLastError();
}

#define CSR_TRY(expr)                \
  do {                               \
    hipError_t e_ = (expr);          \
    if (e_ != hipSuccess) return e_; \
  } while (0)

namespace {

// only the bits a key can have take part in the sorts: recv * V + send < V * V, sender < V
unsigned bits_for(uint64_t max_value) {
  unsigned b = 1;
  while (b < 64 && (max_value >> b) != 0) ++b;
  return b;
}

struct CsrLayout {
  size_t arr = 0, tmp = 0, total = 0;   // one E-sized array (rounded), sort scratch, everything
};

// keys are 32 bits wide whenever recv * V + send fits (V <= 65 536): half the key traffic of every sort pass
bool narrow_keys(int64_t V) { return (uint64_t)V * (uint64_t)V <= ((uint64_t)1 << 32); }

template <class K>
hipError_t sort_scratch_bytes(int64_t E, unsigned bits_rs, unsigned bits_s, size_t& bytes) {
  K *keys_in = nullptr, *keys_out = nullptr;
  int64_t *vals_in = nullptr, *vals_out = nullptr;
  size_t tmp1 = 0, tmp2 = 0;
  CSR_TRY(rocprim::radix_sort_pairs(nullptr, tmp1, keys_in, keys_out, vals_in, vals_out, (size_t)E, 0, bits_rs, (hipStream_t)0));
  CSR_TRY(rocprim::radix_sort_pairs(nullptr, tmp2, keys_in, keys_out, vals_in, vals_out, (size_t)E, 0, bits_s, (hipStream_t)0));
  bytes = std::max(tmp1, tmp2);
  return hipSuccess;
}

hipError_t csr_layout(int64_t E, int64_t V, CsrLayout& L) {
  const unsigned bits_rs = bits_for((uint64_t)V * (uint64_t)V - 1), bits_s = bits_for((uint64_t)(V > 1 ? V - 1 : 1));
  size_t tmp = 0;
  if (narrow_keys(V)) CSR_TRY(sort_scratch_bytes<uint32_t>(E, bits_rs, bits_s, tmp));
  else CSR_TRY(sort_scratch_bytes<uint64_t>(E, bits_rs, bits_s, tmp));
  L.arr = ((size_t)E * 8 + 255) / 256 * 256;
  L.tmp = (tmp + 255) / 256 * 256;
  L.total = 3 * L.arr + 256 + L.tmp;
  return hipSuccess;
}

// the sorts and searches of csr_from_coo_async for one key width
template <class K>
hipError_t csr_build(const int64_t* recv, const int64_t* send, int64_t E, int64_t V, int64_t* row_ptr, int64_t* col, int64_t* perm,
                     int64_t* t_row_ptr, int64_t* t_perm, char* block, const CsrLayout& L, int* bad, hipStream_t st) {
  const bool transpose = t_row_ptr != nullptr;
  const unsigned bits_rs = bits_for((uint64_t)V * (uint64_t)V - 1), bits_s = bits_for((uint64_t)(V > 1 ? V - 1 : 1));
  K* keys_in = (K*)block;   // keys in / out, values in, range-check flag, sort scratch
  K* keys_out = (K*)(block + L.arr);
  int64_t* vals_in = (int64_t*)(block + 2 * L.arr);
  void* tmp = block + 3 * L.arr + 256;
  size_t tmp_bytes = L.tmp;
  hipLaunchKernelGGL(k_make_keys<K>, dim3(blocks_for(E)), dim3(kBlock), 0, st, recv, send, E, V, keys_in, vals_in, bad);
  CSR_TRY(hipGetLastError());
  // stable LSD radix sort: equal (receiver, sender) keep their original order
  CSR_TRY(rocprim::radix_sort_pairs(tmp, tmp_bytes, keys_in, keys_out, vals_in, perm, (size_t)E, 0, bits_rs, st));
  hipLaunchKernelGGL(k_lower_bounds<K>, dim3(blocks_for(V + 1)), dim3(kBlock), 0, st, (const K*)keys_out, E, V, (uint64_t)V, row_ptr);
  CSR_TRY(hipGetLastError());
  // col, and the keys of the transpose: CSR positions stably sorted by sender
  hipLaunchKernelGGL(k_col_from_perm<K>, dim3(blocks_for(E)), dim3(kBlock), 0, st, send, (const int64_t*)perm, E, col, keys_in, vals_in);
  CSR_TRY(hipGetLastError());
  if (transpose) {
    tmp_bytes = L.tmp;
    CSR_TRY(rocprim::radix_sort_pairs(tmp, tmp_bytes, keys_in, keys_out, vals_in, t_perm, (size_t)E, 0, bits_s, st));
    hipLaunchKernelGGL(k_lower_bounds<K>, dim3(blocks_for(V + 1)), dim3(kBlock), 0, st, (const K*)keys_out, E, V, (uint64_t)1, t_row_ptr);
    CSR_TRY(hipGetLastError());
  }
  return hipSuccess;
}

enum class CsrPath { kSmall, kBuckets, kSort };

// One workgroup where rows and edges fit its LDS; buckets up to 2 560 edges a bucket on average (4 096 fit, so rows may
// be uneven): as many buckets as leave each 512 edges (5 000 nodes of degree 32: 56 us a call, with 256 edges 69, with
// 1 300 57), but no more than the chip holds at once, two workgroups a CU (20 000 nodes of degree 40: 313 buckets 81 us,
// 625 buckets 87).  Everything else takes the sorts: above 2.6 million edges, and at most 4 096 edges on more than
// 4 096 nodes, where the buckets' tables would need more workspace than the sort.
CsrPath csr_path(int64_t E, int64_t V, BucketPlan& B) {
  B.eb = (int)bits_for((uint64_t)(E > 1 ? E - 1 : 1));
  B.vb = (int)bits_for((uint64_t)(V > 1 ? V - 1 : 1));
  if (E <= kCap) return V <= kRows ? CsrPath::kSmall : CsrPath::kSort;
  const int64_t least = 512, most = 2560, at_once = 512;
  for (int sh = 0; ((int64_t)1 << sh) <= kRows; ++sh) {
    const int64_t nb = (V + ((int64_t)1 << sh) - 1) >> sh;
    if (nb > kBuckets) continue;
    if (E > most * nb) break;
    const int64_t half = (V + ((int64_t)2 << sh) - 1) >> (sh + 1);   // buckets of twice the rows
    if (half < nb && ((int64_t)2 << sh) <= kRows && E <= most * half && (E < least * nb || nb > at_once)) continue;
    B.shift = sh;
    B.nb = (int)nb;
    return CsrPath::kBuckets;
  }
  return CsrPath::kSort;
}

size_t up256(size_t v) { return (v + 255) / 256 * 256; }

size_t bucket_layout(const BucketPlan& B, int64_t E, char* at, BucketWs& w) {
  const size_t table = up256((kBuckets + 1) * sizeof(int)), recs = up256((size_t)E * 8);
  const int64_t tiles = (E + kTile - 1) / kTile;
  size_t o = 0;
  auto take = [&](size_t bytes) { char* p = at + o; o += bytes; return p; };
  w.total1 = (int*)take(table);
  w.total2 = (int*)take(table);
  w.base1 = (int*)take(table);
  w.base2 = (int*)take(table);
  w.cursor2 = (int*)take(table);
  w.before = (int*)take(up256((size_t)tiles * B.nb * sizeof(int)));
  w.rec1 = (uint64_t*)take(recs);
  w.rec2 = (uint64_t*)take(recs);
  return o + 256;   // the range-check flag of a caller that gives none
}

hipError_t csr_buckets(const int64_t* recv, const int64_t* send, int64_t E, int64_t V, int64_t* row_ptr, int64_t* col, int64_t* perm,
                       int64_t* t_row_ptr, int64_t* t_perm, char* block, const BucketPlan& B, int* bad_flag, hipStream_t st) {
  BucketWs w;
  const size_t total = bucket_layout(B, E, block, w);
  int* bad = bad_flag ? bad_flag : (int*)(block + total - 256);
  const int transpose = t_row_ptr != nullptr, tiles = (int)((E + kTile - 1) / kTile);
  const int tables = (int)(w.base1 - w.total1);   // both totals
  hipLaunchKernelGGL(k_csr_clear, dim3((tables + kBlock - 1) / kBlock), dim3(kBlock), 0, st, w.total1, tables, bad);
  hipLaunchKernelGGL(k_csr_count, dim3(tiles), dim3(kThreads), 0, st, recv, send, E, V, B, w, transpose);
  hipLaunchKernelGGL(k_csr_distribute, dim3(tiles + transpose), dim3(kThreads), 0, st, recv, send, E, V, B, w, tiles, bad);
  hipLaunchKernelGGL(k_csr_rows<false>, dim3(B.nb), dim3(kThreads), 0, st, B, w, V, E, row_ptr, perm, col, transpose);
  if (transpose) hipLaunchKernelGGL(k_csr_rows<true>, dim3(B.nb), dim3(kThreads), 0, st, B, w, V, E, t_row_ptr, t_perm, (int64_t*)nullptr, 0);
  return hipGetLastError();
}

}  // namespace

hipError_t csr_workspace_bytes(int64_t E, int64_t V, size_t* bytes) {
  *bytes = 256;
  if (E <= 0) return hipSuccess;
  BucketPlan B;
  BucketWs w;
  switch (csr_path(E, V, B)) {
    case CsrPath::kSmall: return hipSuccess;   // no scratch
    case CsrPath::kBuckets: *bytes = bucket_layout(B, E, nullptr, w); return hipSuccess;
    case CsrPath::kSort: break;
  }
  CsrLayout L;
  CSR_TRY(csr_layout(E, V, L));
  *bytes = L.total;
  return hipSuccess;
}

// Enqueues everything on `st` and returns: no allocation, no synchronisation.  *bad_flag (device, may be null)
// receives 1 if an index lies outside [0, V), else 0.  t_row_ptr == t_perm == nullptr skips the transpose.
hipError_t csr_from_coo_async(const int64_t* recv, const int64_t* send, int64_t E, int64_t V, int64_t* row_ptr, int64_t* col,
                              int64_t* perm, int64_t* t_row_ptr, int64_t* t_perm, void* workspace, size_t workspace_bytes,
                              int* bad_flag, hipStream_t st) {
  const bool transpose = t_row_ptr != nullptr;
  if (E == 0) {
    CSR_TRY(launch_fill_zero(row_ptr, (size_t)(V + 1) * 8, st));
    if (transpose) CSR_TRY(launch_fill_zero(t_row_ptr, (size_t)(V + 1) * 8, st));
    if (bad_flag) CSR_TRY(launch_fill_zero(bad_flag, 4, st));
    return hipSuccess;
  }
  BucketPlan B;
  const CsrPath path = csr_path(E, V, B);
  if (path == CsrPath::kSmall) {
    hipLaunchKernelGGL(k_csr_small, dim3(1), dim3(kThreads), 0, st, recv, send, (int)E, (int)V, B.eb, B.vb, row_ptr, col, perm, t_row_ptr,
                       t_perm, bad_flag);
    return hipGetLastError();
  }
  if (path == CsrPath::kBuckets) {
    BucketWs w;
    if (!workspace || workspace_bytes < bucket_layout(B, E, nullptr, w)) return hipErrorInvalidValue;
    return csr_buckets(recv, send, E, V, row_ptr, col, perm, t_row_ptr, t_perm, (char*)workspace, B, bad_flag, st);
  }
  CsrLayout L;
  CSR_TRY(csr_layout(E, V, L));
  if (!workspace || workspace_bytes < L.total) return hipErrorInvalidValue;
  char* block = (char*)workspace;
  int* bad = bad_flag ? bad_flag : (int*)(block + 3 * L.arr);
  CSR_TRY(launch_fill_zero(bad, 4, st));
  if (narrow_keys(V)) return csr_build<uint32_t>(recv, send, E, V, row_ptr, col, perm, t_row_ptr, t_perm, block, L, bad, st);
  return csr_build<uint64_t>(recv, send, E, V, row_ptr, col, perm, t_row_ptr, t_perm, block, L, bad, st);
}

}  // namespace cgtp
