// Integer graph preparation on the device: COO -> CSR by receiver plus the transpose
// permutation (paper Sec. 3.5: the fused kernels need row-sorted edges, and the backward pass
// a permutation that transposes the adjacency), and two small helpers of the conv path.
// Statically compiled (nothing here depends on the irreps).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
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

// senders from the sorted keys recv * V + send (not from the list: an out-of-range edge is (0, 0))
template <class K>
__global__ void k_col_from_keys(const K* __restrict__ keys, int64_t E, int64_t V, int64_t* __restrict__ col, K* __restrict__ colkey,
                                int64_t* __restrict__ pos) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  int64_t c = (int64_t)((uint64_t)keys[e] % (uint64_t)V);
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

// The compiler moves a load down into the branch that uses it; where that would put one memory latency behind another
// (a scalar load and its wait cost about half a microsecond, of kernels of 5 to 20), the value is named before the branch.
template <class T>
__device__ __forceinline__ void here_scalar(T v) { asm volatile("" ::"s"(v)); }

// ---- bucket path: graphs of up to about 2.6 million edges ---------------------------------------------------------------
// A general radix sort costs a launch or two per digit or merge round (ten rounds for 800 000 keys, twice), each a few
// microseconds long whatever it does.  Here the edges are cut once into at most 1 024 buckets of consecutive rows, and
// one workgroup finishes a bucket in LDS: rows are placed by counting, and the order inside a row comes from counting
// the smaller records of that row (unique records: row, other end, original position packed into 64 bits, so the order
// of arrival does not matter and the result is the stable one).  The kernel that finishes the receivers hands its edges
// on to the buckets of the senders.  Five launches, one if the graph fits a single workgroup.
// Rows of very many edges (a node connected to all others, the padding of a neighbour list of fixed capacity) would leave
// one workgroup with most of the graph: a sample of the edges finds the buckets that do not fit, and these are cut
// further at keys of the sample, so that every workgroup has about the same to do whatever the degrees are.
// What is left is the latency of dependent passes.  Synchronous call, sorts -> buckets: 27 nodes of degree 9 80 -> 28 us,
// 300 nodes of degree 20 120 -> 45, 3 001 nodes of degree 32 178 -> 50, 20 000 nodes of degree 40 425 -> 80 us (kernels
// 4 + 10 + 9 + 21 + 14); conv_forward_perm + conv_backward_perm with the preparation, 3 001 nodes of 32 channels 343 -> 221 us.
// With a node connected to all others, sorts -> without cuts -> with them: 3 002 nodes 181 -> 542 -> 90 to 102 us, 20 001
// nodes 422 -> 618 -> 154; 100 000 equal edges at the end of 900 000 417 -> 3 322 -> 164; half of 800 000 edges in one row 404 ->
// 9 093 -> 170, all of a million 396 -> 22 775 -> 207; degrees of a power law 411 -> 4 573 -> 229.
constexpr int kThreads = 1024;     // of every kernel of this path; one thread per bucket of rows in the scans
constexpr int kBuckets = 1024;     // of consecutive rows
constexpr int kPer = 4;            // records of a thread
constexpr int kCap = kThreads * kPer;
constexpr int kRows = 4096;        // rows of a bucket
// Edges of a thread in the counting and distributing passes, up to a million edges: 800 000 edges 8 + 13 us with eight, 10 + 9
// with four, 15 + 9 with two.  Above it twice as many (kBigTiles), because the tables grow with the tiles: a call with
// 2 600 000 edges 142 us with eight and 161 with four.
constexpr int kTilePer = 4;
constexpr int kTile = kThreads * kTilePer;
constexpr int64_t kBigTiles = (int64_t)1 << 20;
constexpr int kSamples = kCap;     // edges that are looked at for buckets that do not fit
constexpr int kCutsPer = 3;        // buckets after the cuts, per thread
constexpr int kCuts = kThreads * kCutsPer;   // kBuckets + kSamples / 2: a cut keeps at least two samples
constexpr int kLongRow = 64;       // rows above this many records count towards kLongWork
// Sum of the squares of the long rows from which a radix sort is the faster order.  Counting costs a row of 4 096 records 220 us
// and a row of 290 4 us, the radix sort 20 us whatever the rows are: 3 770 edges with a row of 290 45 us a call with counting, 67
// with the radix sort; 4 096 in one row 476 and 64; 1 000 nodes of degree 500 133 and 112.
constexpr int kLongWork = 1 << 19;

struct BucketPlan {
  int shift, nb, eb, vb;   // bucket of a row = row >> shift; number of buckets; bits of an edge index and of a node index
  int tile;                // edges of a workgroup in the counting and distributing passes
  int samples, heavy, cut;   // edges in the sample; samples of a bucket that is cut; samples per piece
};

// The caller's workspace.  Every address follows from its start and E: the kernels' arguments come from host memory, a
// cache line at a time, and a pointer to each table was two lines more (1 to 2 us of every kernel).
constexpr size_t apart(size_t bytes) { return (bytes + 511) / 256 * 256; }   // at least 256 bytes between two tables

// One side of the graph (receivers or senders).  A bucket that is cut has several pieces, and everything after the sample
// is done by piece; without a cut the pieces are the buckets.
struct BucketSide {
  static constexpr size_t kFirst = 0, kOwner = kFirst + apart((kBuckets + 1) * 4), kLow = kOwner + apart(kCuts * 4),
                          kTotal = kLow + apart(kCuts * 8), kBase = kTotal + apart(kCuts * 4), kBytes = kBase + apart((kCuts + 1) * 4);
  char* at;
  // the first three hold anything where no bucket of the side is cut
  __host__ __device__ int* first() const { return (int*)(at + kFirst); }         // [nb + 1] first piece of a bucket
  __host__ __device__ int* owner() const { return (int*)(at + kOwner); }         // [pieces] bucket of a piece
  __host__ __device__ uint64_t* low() const { return (uint64_t*)(at + kLow); }   // [pieces] smallest key (row in the bucket, other end, edge)
  __host__ __device__ int* total() const { return (int*)(at + kTotal); }      // [pieces] records
  __host__ __device__ int* base() const { return (int*)(at + kBase); }        // [pieces + 1] first place
};

struct alignas(16) BucketInfo {   // read by every kernel as its first load
  struct { int pieces, cut; } side[2];   // number of pieces (senders: 0 without a transpose), whether any bucket is cut
};

struct BucketWs {
  static constexpr size_t kSides = 512, kCursor = kSides + 2 * BucketSide::kBytes, kBefore = kCursor + apart(kCuts * 4);
  char* at;
  __host__ __device__ BucketInfo* info() const { return (BucketInfo*)at; }
  __host__ __device__ BucketSide side(int i) const { return {at + kSides + i * BucketSide::kBytes}; }   // 0 receivers, 1 senders
  __host__ __device__ int* cursor2() const { return (int*)(at + kCursor); }
  __host__ __device__ int* before() const { return (int*)(at + kBefore); }    // [tiles][kCuts], laid out for the small tiles
  __host__ __device__ static size_t rec1_at(int64_t E) { return kBefore + (size_t)((E + kTile - 1) / kTile) * (kCuts * 4); }
  __host__ __device__ static size_t rec2_at(int64_t E) { return rec1_at(E) + apart((size_t)E * 8); }
  __host__ __device__ uint64_t* rec1(int64_t E) const { return (uint64_t*)(at + rec1_at(E)); }
  __host__ __device__ uint64_t* rec2(int64_t E) const { return (uint64_t*)(at + rec2_at(E)); }
  __host__ __device__ static size_t bytes(int64_t E) { return rec2_at(E) + apart((size_t)E * 8); }   // the last 256: range-check flag of a caller that gives none
};

struct SortLds {
  uint64_t rec[kCap];
  int off[kRows + 1];      // also [16 waves][256 digits]
  int wave[kThreads / 64];
  int any;                 // zeroed, raised by some threads and read with barriers between
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

// One step of a radix sort over up to 4 096 records, of which this thread has those at wave * 256 + j * 64 + lane, j < 4:
// digit_of(j) = 0..255, or -1 without a record.  Returns in 16 bits each how many records of the same digit stand before
// record j in its wave; afterwards count[wave][digit] = records of smaller digits, and of the same digit in waves before.
// `next` (LDS, [256], or null): where the digits begin, moved on by this step's records; else they begin at 0.
// (Rolled loops: this is the rare path of kernels that would lose a workgroup a CU to its registers.)
template <class DigitOf>
__device__ __forceinline__ uint64_t digit_places(DigitOf digit_of, int* count, int* next, int* wave) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
#pragma unroll 1
  for (int q = t; q < 16 * 256; q += kThreads) count[q] = 0;
  __syncthreads();
  uint64_t slots = 0;
#pragma unroll 1
  for (int j = 0; j < kPer; ++j) {
    const int digit = digit_of(j);
    const bool in = digit >= 0;
    uint64_t same = __ballot(in);           // lanes of this wave with the same digit
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool one = (digit >> bit) & 1;
      const uint64_t m = __ballot(one);
      same &= one ? m : ~m;
    }
    const int rank = __popcll(same & (((uint64_t)1 << lane) - 1));
    int had = 0;
    if (in && rank == 0) had = atomicAdd(&count[wv * 256 + digit], __popcll(same));
    slots |= (uint64_t)(rank + __shfl(had, in ? __ffsll((unsigned long long)same) - 1 : lane, 64)) << (16 * j);
  }
  __syncthreads();
  int sum = 0;
  if (t < 256)
#pragma unroll 4
    for (int q = 0; q < 16; ++q) sum += count[q * 256 + t];
  int at = next ? 0 : block_scan(sum, wave);
  if (t < 256) {
    if (next) {
      at = next[t];
      next[t] = at + sum;
    }
#pragma unroll 4
    for (int q = 0; q < 16; ++q) {
      const int v = count[q * 256 + t];
      count[q * 256 + t] = at;
      at += v;
    }
  }
  __syncthreads();
  return slots;
}

// S.rec[0..n) in ascending order of its lowest `bits` bits; S.off is overwritten
__device__ __forceinline__ void radix_in_lds(SortLds& S, int n, int bits) {
  const int mine = (threadIdx.x >> 6) * 256 + (threadIdx.x & 63);   // + 64 j: this thread's records
  int* const count = S.off + (threadIdx.x >> 6) * 256;
#pragma unroll 1
  for (int sh = 0; sh < bits; sh += 8) {
    const uint64_t slots = digit_places([&](int j) { return mine + 64 * j < n ? (int)((S.rec[mine + 64 * j] >> sh) & 255) : -1; }, S.off, nullptr, S.wave);
    uint64_t k[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) k[j] = mine + 64 * j < n ? S.rec[mine + 64 * j] : 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (mine + 64 * j < n) S.rec[count[(int)((k[j] >> sh) & 255)] + (int)((slots >> (16 * j)) & 0xffff)] = k[j];
    __syncthreads();
  }
}

// rec[j] (valid for threadIdx.x + j * 1024 < n, row = rec >> row_bits < rows, no bit from `bits` on): on return rec[j] is
// S.rec[threadIdx.x + j * 1024] and pos[j] its place in ascending order; S.off[r] = first place of row r, S.off[rows] = n.
__device__ __forceinline__ void sort_in_lds(SortLds& S, uint64_t (&rec)[kPer], int (&pos)[kPer], int n, int rows, int row_bits, int bits) {
  const int t = threadIdx.x;
  for (int r = t; r <= rows; r += kThreads) S.off[r] = 0;
  if (t == 0) S.any = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) pos[j] = atomicAdd(&S.off[(int)(rec[j] >> row_bits)], 1);
  __syncthreads();
  constexpr int kRowsPer = kRows / kThreads;
  int c[kRowsPer], sum = 0, work = 0;
#pragma unroll
  for (int q = 0; q < kRowsPer; ++q) {
    const int r = t * kRowsPer + q;
    c[q] = r < rows ? S.off[r] : 0;
    sum += c[q];
    if (c[q] > kLongRow) work += c[q] * c[q];
  }
  const int first = block_scan(sum, S.wave);
  auto write_offsets = [&] {
    int at = first;
#pragma unroll
    for (int q = 0; q < kRowsPer; ++q) {
      const int r = t * kRowsPer + q;
      if (r < rows) S.off[r] = at;
      at += c[q];
    }
    if (t == 0) S.off[rows] = n;
  };
  write_offsets();
  if (work) atomicAdd(&S.any, work);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) S.rec[S.off[(int)(rec[j] >> row_bits)] + pos[j]] = rec[j];
  __syncthreads();
  if (__builtin_expect(S.any > kLongWork, 0)) {
    radix_in_lds(S, n, bits);
    write_offsets();
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (t + j * kThreads < n) {
        rec[j] = S.rec[t + j * kThreads];
        pos[j] = t + j * kThreads;
      }
    return;
  }
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
  sort_in_lds(S, rec, pos, E, V, eb + vb, eb + 2 * vb);
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
  sort_in_lds(S, rec, pos, E, V, eb, eb + vb);
  for (int r = t; r <= V; r += kThreads) t_row_ptr[r] = S.off[r];
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < E) t_perm[pos[j]] = (int64_t)(rec[j] & emask);
}

__device__ __forceinline__ uint64_t edge_key(const BucketPlan& B, uint64_t row, uint64_t other, uint64_t e) {
  return ((row & (((uint64_t)1 << B.shift) - 1)) << (B.eb + B.vb)) | (other << B.eb) | e;
}

struct EdgeRun {
  int64_t end[kPer];
};

// Workgroup 0: receivers, 1: senders.  Clears the side's totals, counts the buckets of a sample of the edges (four
// neighbours from each of 1 024 equal parts) and cuts the buckets with too many at samples of theirs.
__global__ void __launch_bounds__(kThreads) k_csr_cut(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t E,
                                                      int64_t V, BucketPlan B, BucketWs w, int* __restrict__ bad) {
  __shared__ SortLds S;
  __shared__ int hist[kBuckets];
  const int t = threadIdx.x;
  const bool senders = blockIdx.x == 1;
  const BucketSide side = w.side(senders ? 1 : 0);
  const int64_t* __restrict__ own = senders ? send : recv;
  const int64_t* __restrict__ other = senders ? recv : send;
  for (int i = t; i < kCuts; i += kThreads) side.total()[i] = 0;
  if (t == 0 && !senders) *bad = 0;
  if (t == 0 && gridDim.x == 1) w.info()->side[1] = {0, 0};
  hist[t] = 0;
  if (t == 0) S.any = 0;
  __syncthreads();
  // this thread's sample: kPer edges in a row (4 096 single edges made this kernel 6.6 us on 800 000 edges, runs of four 4.0).
  // Somewhere in the first half of the run's part of the list: in a list in the order of the keys the pieces between two runs
  // are then at most one and a half parts long, and fit.
  auto place = [&](int i) -> int64_t {   // the edge that is sample i: ascending
    if (E <= kSamples) return i;
    const int run = i / kPer;
    const int64_t lo = run * E / kThreads, room = ((run + 1) * E / kThreads - lo - kPer) / 2 + 1;
    return lo + (int64_t)((((uint64_t)((unsigned)run * 2654435761u)) * (uint64_t)room) >> 32) + i % kPer;
  };
  const int64_t at = place(t * kPer);
  uint64_t row[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) row[j] = 0;
  if (E > kSamples) {
    const EdgeRun four = *(const EdgeRun*)(own + at);
#pragma unroll
    for (int j = 0; j < kPer; ++j) row[j] = (uint64_t)four.end[j];
  } else {
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (at + j < E) row[j] = (uint64_t)own[at + j];
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (row[j] >= (uint64_t)V) row[j] = 0;
    if (at + j < E) atomicAdd(&hist[(int)(row[j] >> B.shift)], 1);
  }
  __syncthreads();
  const int c = t < B.nb ? hist[t] : 0;
  if (c >= B.heavy) S.any = 1;
  __syncthreads();
  if (__builtin_expect(!S.any, 1)) {
    if (t == 0) w.info()->side[senders] = {B.nb, 0};
    return;
  }
  const int pieces = t >= B.nb ? 0 : c >= B.heavy ? (c + B.cut - 1) / B.cut : 1;
  const int first = block_scan(pieces, S.wave);
  __syncthreads();
  hist[t] = first;
  if (t < B.nb) {
    side.first()[t] = first;
    if (c < B.heavy) {
      side.owner()[first] = t;
      side.low()[first] = 0;
    }
    if (t == B.nb - 1) {
      side.first()[B.nb] = first + pieces;
      w.info()->side[senders] = {first + pieces, 1};
    }
  }
  // Keys with the sample's number in place of the edge's index, in the same order: equal edges still differ.
  // Bucket (10 bits), row in it (<= 12), other end (<= 22), sample (12).
  uint64_t key[kPer];
  int pos[kPer];
  constexpr int kIndexBits = 12;
  static_assert(kSamples == 1 << kIndexBits, "a sample's number");
  const int row_at = kIndexBits + B.vb, bucket_at = row_at + B.shift;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    uint64_t o = at + j < E ? (uint64_t)other[at + j] : 0;
    if (o >= (uint64_t)V) o = 0;
    key[j] = (row[j] << row_at) | (o << kIndexBits) | (uint64_t)(t * kPer + j);   // a row is its bucket and its place there
    pos[j] = 0;
  }
  __syncthreads();
  // sort_in_lds takes records in any order, but in its own places: the first B.samples of them
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (at + j < E) S.rec[t * kPer + j] = key[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < B.samples) key[j] = S.rec[t + j * kThreads];
  __syncthreads();
  sort_in_lds(S, key, pos, B.samples, B.nb, bucket_at, row_at + B.vb);
  const uint64_t vmask = ((uint64_t)1 << B.vb) - 1;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < B.samples) {
      const int b = (int)(key[j] >> bucket_at), beg = S.off[b], have = S.off[b + 1] - beg, i = pos[j] - beg;
      if (have < B.heavy || i % B.cut) continue;
      const int piece = hist[b] + i / B.cut;
      side.owner()[piece] = b;
      side.low()[piece] = i ? edge_key(B, key[j] >> row_at, (key[j] >> kIndexBits) & vmask, (uint64_t)place((int)(key[j] & (kSamples - 1)))) : 0;
    }
}

// piece of a record of bucket b with this key (row in the bucket, other end, edge), where any bucket is cut
__device__ __forceinline__ int piece_of(const BucketSide& side, int b, uint64_t key) {
  int lo = side.first()[b], hi = side.first()[b + 1] - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (side.low()[mid] <= key) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// edges per piece of the receivers and of the senders; before[block][piece]: edges of that piece that other workgroups
// placed ahead of this one's
__global__ void __launch_bounds__(kThreads) k_csr_count(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t E,
                                                        int64_t V, BucketPlan B, BucketWs w, int transpose) {
  __shared__ int h1[kCuts], h2[kCuts];
  const int t = threadIdx.x;
  const BucketInfo info = *w.info();
  const int n1 = info.side[0].pieces, n2 = info.side[1].pieces, cut1 = info.side[0].cut, cut2 = info.side[1].cut;
#pragma unroll
  for (int i = t; i < kCuts; i += kThreads) h1[i] = h2[i] = 0;
  __syncthreads();
  const int64_t e0 = (int64_t)blockIdx.x * B.tile + t, e_end = e0 - t + B.tile < E ? e0 - t + B.tile : E;
  if (__builtin_expect(!cut1 && !cut2, 1)) {
#pragma unroll
    for (int j = 0; j < 2 * kTilePer; ++j)
      if (e0 + j * kThreads < e_end) {
        uint64_t r, s;
        (void)load_edge(recv, send, e0 + j * kThreads, V, r, s);
        atomicAdd(&h1[(int)(r >> B.shift)], 1);
        if (transpose) atomicAdd(&h2[(int)(s >> B.shift)], 1);
      }
  } else {
#pragma unroll 1
    for (int64_t e = e0; e < e_end; e += kThreads) {
      uint64_t r1, s1;
      (void)load_edge(recv, send, e, V, r1, s1);
      const int b1 = (int)(r1 >> B.shift), b2 = (int)(s1 >> B.shift);
      atomicAdd(&h1[cut1 ? piece_of(w.side(0), b1, edge_key(B, r1, s1, (uint64_t)e)) : b1], 1);
      if (transpose) atomicAdd(&h2[cut2 ? piece_of(w.side(1), b2, edge_key(B, s1, r1, (uint64_t)e)) : b2], 1);
    }
  }
  __syncthreads();
  for (int i = t; i < n1; i += kThreads) {
    const int c1 = h1[i];
    w.before()[(int64_t)blockIdx.x * kCuts + i] = c1 ? atomicAdd(&w.side(0).total()[i], c1) : 0;
  }
  for (int i = t; i < n2; i += kThreads) {
    const int c2 = h2[i];
    if (c2) atomicAdd(&w.side(1).total()[i], c2);
  }
}

// records into the pieces of the receivers; the last workgroup (if there is a transpose) lays out the pieces of the senders
__global__ void __launch_bounds__(kThreads) k_csr_distribute(const int64_t* __restrict__ recv, const int64_t* __restrict__ send, int64_t E,
                                                             int64_t V, BucketPlan B, BucketWs w, int tiles, int* __restrict__ bad) {
  __shared__ int dst[kCuts];
  __shared__ int wave[kThreads / 64];
  const int t = threadIdx.x;
  const bool second = (int)blockIdx.x == tiles;
  const BucketInfo info = *w.info();
  const BucketSide side = w.side(second ? 1 : 0);
  const int n = second ? info.side[1].pieces : info.side[0].pieces, cut = second ? info.side[1].cut : info.side[0].cut;
  const int per = cut ? kCutsPer : 1;      // pieces of this thread: t * per + q
  int have[kCutsPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kCutsPer; ++q) {
    have[q] = q < per && t * per + q < n ? side.total()[t * per + q] : 0;
    sum += have[q];
  }
  int start = block_scan(sum, wave);
#pragma unroll
  for (int q = 0; q < kCutsPer; ++q) {
    const int i = t * per + q;
    if (q < per && i < n) {
      if (second) w.cursor2()[i] = start;
      else dst[i] = start + w.before()[(int64_t)blockIdx.x * kCuts + i];
      if (second || blockIdx.x == 0) side.base()[i] = start;
    }
    start += have[q];
  }
  if (t == 0 && (second || blockIdx.x == 0)) side.base()[n] = (int)E;
  if (second) return;
  __syncthreads();
  const int64_t e0 = (int64_t)blockIdx.x * B.tile + t, e_end = e0 - t + B.tile < E ? e0 - t + B.tile : E;
  if (__builtin_expect(!cut, 1)) {
#pragma unroll
    for (int j = 0; j < 2 * kTilePer; ++j) {
      const int64_t e = e0 + j * kThreads;
      uint64_t r, s;
      if (e < e_end) {
        if (!load_edge(recv, send, e, V, r, s)) *bad = 1;
        w.rec1(E)[atomicAdd(&dst[(int)(r >> B.shift)], 1)] = edge_key(B, r, s, (uint64_t)e);
      }
    }
  } else {
#pragma unroll 1
    for (int64_t e = e0; e < e_end; e += kThreads) {
      uint64_t r1, s1;
      if (!load_edge(recv, send, e, V, r1, s1)) *bad = 1;
      const uint64_t key = edge_key(B, r1, s1, (uint64_t)e);
      w.rec1(E)[atomicAdd(&dst[piece_of(side, (int)(r1 >> B.shift), key)], 1)] = key;
    }
  }
}

// A piece of more than 4 096 records (the sample missed it, or records crowd between two cuts): one workgroup sorts it in global
// memory, 8 bits at a time, between the records and the output array of the piece's range.  An even number of passes leaves
// the result where it began.
__device__ void sort_in_memory(uint64_t* a, uint64_t* b, int n, int bits, SortLds& S) {
  int* next = (int*)S.rec;                  // [256]
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int passes = ((bits + 7) / 8 + 1) & ~1;
#pragma unroll 1
  for (int p = 0; p < passes; ++p) {
    const int sh = p * 8 < 56 ? p * 8 : 56;
    const bool empty = p * 8 >= bits;       // padding pass: keeps the order
    __syncthreads();
    if (t < 256) next[t] = 0;
    __syncthreads();
#pragma unroll 1
    for (int i = t; i < n; i += kThreads) atomicAdd(&next[empty ? 0 : (int)((a[i] >> sh) & 255)], 1);
    __syncthreads();
    const int c = t < 256 ? next[t] : 0;
    const int first = block_scan(c, S.wave);
    if (t < 256) next[t] = first;
#pragma unroll 1
    for (int i0 = 0; i0 < n; i0 += kCap) {
      const int i = i0 + wv * 256 + lane;
      auto digit = [&](int j) { return empty ? 0 : (int)((a[i + 64 * j] >> sh) & 255); };
      const uint64_t slots = digit_places([&](int j) { return i + 64 * j < n ? digit(j) : -1; }, S.off, next, S.wave);
#pragma unroll 1
      for (int j = 0; j < kPer; ++j)
        if (i + 64 * j < n) b[S.off[wv * 256 + digit(j)] + (int)((slots >> (16 * j)) & 0xffff)] = a[i + 64 * j];
      __syncthreads();
    }
    uint64_t* x = a;
    a = b;
    b = x;
  }
  __syncthreads();
}

// One piece: kSecond false: the rows of its receivers (row_ptr, col, perm), and its edges on to the pieces of the senders;
// true: the rows of its senders (t_row_ptr, t_perm).  A row belongs to the piece whose range of keys holds the row's first
// possible key, whether it has edges there or not.  (8 waves per SIMD: two workgroups a CU.)
template <bool kSecond>
__global__ void __launch_bounds__(kThreads, 8) k_csr_rows(BucketPlan B, BucketWs w, int64_t V, int64_t E, int64_t* __restrict__ ptr,
                                                       int64_t* idx, int64_t* __restrict__ col, int transpose) {
  __shared__ SortLds S;
  __shared__ int h2[kSecond ? 1 : kCuts];
  const int t = threadIdx.x, piece = blockIdx.x;
  const BucketSide side = w.side(kSecond ? 1 : 0), to = w.side(1);
  // requested together: what is not in use holds anything
  const BucketInfo info = *w.info();
  const int base = side.base()[piece], end = side.base()[piece + 1], owner = side.owner()[piece];
  const int pieces = info.side[kSecond].pieces, cut = info.side[kSecond].cut, n2 = kSecond ? 0 : info.side[1].pieces;
  const bool cut2 = !kSecond && info.side[1].cut;
  here_scalar(base);
  here_scalar(end);
  here_scalar(owner);
  here_scalar(cut);
  here_scalar(n2);
  here_scalar(ptr);
  here_scalar(col);
  const int row_bits = B.eb + (kSecond ? 0 : B.vb), key_bits = B.eb + B.vb;
  const uint64_t emask = ((uint64_t)1 << B.eb) - 1, vmask = ((uint64_t)1 << B.vb) - 1;
  const uint64_t in_bucket = ((uint64_t)1 << B.shift) - 1;
  if (piece >= pieces) return;   // the grid is as large as any cut can make it
  const int bucket = cut ? owner : piece, n = end - base;
  uint64_t* const in = (kSecond ? w.rec2(E) : w.rec1(E)) + base;
  const int64_t row0 = (int64_t)bucket << B.shift;
  const int rows = (int)(V - row0 < ((int64_t)1 << B.shift) ? V - row0 : (int64_t)1 << B.shift);
  int row_lo = 0, row_hi = rows;          // rows of this piece
  if (__builtin_expect(cut, 0)) {
    const uint64_t one = ((uint64_t)1 << key_bits) - 1;
    row_lo = (int)((side.low()[piece] + one) >> key_bits);
    if (piece + 1 < pieces && side.owner()[piece + 1] == bucket) row_hi = (int)((side.low()[piece + 1] + one) >> key_bits);
  }
  if (piece == pieces - 1 && t == 0) ptr[V] = E;
  // the senders' piece of an edge
  auto senders_piece = [&](uint64_t rec) {
    const uint64_t s = (rec >> B.eb) & vmask;
    const int b = (int)(s >> B.shift);
    return cut2 ? piece_of(to, b, edge_key(B, s, (uint64_t)row0 + (rec >> row_bits), rec & emask)) : b;
  };
  if (n > kCap) {
    sort_in_memory(in, (uint64_t*)(idx + base), n, row_bits + B.shift, S);
    for (int i = t; i < n; i += kThreads) {
      const uint64_t k = in[i];
      const int r = (int)(k >> row_bits), q0 = i > 0 ? (int)(in[i - 1] >> row_bits) + 1 : 0;
      for (int q = q0 > row_lo ? q0 : row_lo; q <= r && q < row_hi; ++q) ptr[row0 + q] = base + i;
      if (i == n - 1)
        for (int q = r + 1 > row_lo ? r + 1 : row_lo; q < row_hi; ++q) ptr[row0 + q] = base + n;
      idx[base + i] = (int64_t)(k & emask);
      if (!kSecond) {
        const uint64_t s = (k >> B.eb) & vmask;
        col[base + i] = (int64_t)s;
        if (transpose) w.rec2(E)[atomicAdd(&w.cursor2()[senders_piece(k)], 1)] = ((s & in_bucket) << B.eb) | (uint64_t)(base + i);
      }
    }
    return;
  }
  uint64_t rec[kPer];
  int pos[kPer];
  if (!kSecond)
#pragma unroll
    for (int i = t; i < kCuts; i += kThreads) h2[i] = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = t + j * kThreads;
    rec[j] = i < n ? in[i] : 0;
    pos[j] = 0;
  }
  sort_in_lds(S, rec, pos, n, rows, row_bits, row_bits + B.shift);
  for (int r = row_lo + t; r < row_hi; r += kThreads) ptr[row0 + r] = base + S.off[r];
  int rank[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    rank[j] = 0;
    if (t + j * kThreads < n) {
      idx[base + pos[j]] = (int64_t)(rec[j] & emask);
      if (!kSecond) {
        const uint64_t s = (rec[j] >> B.eb) & vmask;
        col[base + pos[j]] = (int64_t)s;
        if (transpose && !cut2) rank[j] = atomicAdd(&h2[(int)(s >> B.shift)], 1);
      }
    }
  }
  __syncthreads();
  if (kSecond || !transpose) return;
  if (__builtin_expect(cut2, 0)) {   // rolled; this thread's place in S.rec, which held its record, takes the piece and the rank in it
#pragma unroll 1
    for (int i = t; i < n; i += kThreads) {
      const int p = senders_piece(S.rec[i]);
      S.rec[i] = (uint64_t)p << 32 | (uint64_t)atomicAdd(&h2[p], 1);
    }
    __syncthreads();
  }
  for (int i = t; i < n2; i += kThreads) {
    const int c = h2[i];
    if (c) h2[i] = atomicAdd(&w.cursor2()[i], c);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (t + j * kThreads < n) {
      const uint64_t s = (rec[j] >> B.eb) & vmask, mine = cut2 ? S.rec[t + j * kThreads] : 0;
      const int p = cut2 ? (int)(mine >> 32) : (int)(s >> B.shift), at = cut2 ? (int)(uint32_t)mine : rank[j];
      w.rec2(E)[h2[p] + at] = ((s & in_bucket) << B.eb) | (uint64_t)(base + pos[j]);
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
  hipLaunchKernelGGL(k_col_from_keys<K>, dim3(blocks_for(E)), dim3(kBlock), 0, st, (const K*)keys_out, E, V, col, keys_in, vals_in);
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

// One workgroup where rows and edges fit its LDS; buckets up to 2 560 edges for each of 1 024 (4 096 fit, so rows may
// be uneven): as many buckets as leave each 512 edges (5 000 nodes of degree 32: 56 us a call, with 256 edges 69, with
// 1 300 57), but no more than the chip holds at once, two workgroups a CU (20 000 nodes of degree 40: 313 buckets 81 us,
// 625 buckets 87).  With fewer rows than that most buckets are cut; up to two million edges this is faster than the sorts (300
// nodes, a million edges 200 us against 415; 20 000 nodes, 1.7 million 192 against 291), at 2.6 million it is not (1 000 nodes 407
// against 332).  Larger graphs take the sorts.
constexpr int64_t kMostEdges = (int64_t)2560 * kBuckets, kMostNodes = (int64_t)kBuckets * kRows, kMostCrowded = (int64_t)1 << 21;

CsrPath csr_path(int64_t E, int64_t V, BucketPlan& B) {
  B.eb = (int)bits_for((uint64_t)(E > 1 ? E - 1 : 1));
  B.vb = (int)bits_for((uint64_t)(V > 1 ? V - 1 : 1));
  if (E <= kCap && V <= kRows) return CsrPath::kSmall;
  if (E > kMostEdges || V > kMostNodes) return CsrPath::kSort;
  const int64_t least = 512, most = 2560, at_once = 512;
  B.samples = (int)std::min<int64_t>(E, kSamples);
  B.tile = E > kBigTiles ? 2 * kTile : kTile;
  B.shift = 0;
  auto buckets = [&](int shift) { return (V + ((int64_t)1 << shift) - 1) >> shift; };
  while (buckets(B.shift) > kBuckets) ++B.shift;
  for (; ((int64_t)2 << B.shift) <= kRows; ++B.shift) {
    const int64_t nb = buckets(B.shift), half = buckets(B.shift + 1);   // half: with buckets of twice the rows
    if (half == nb || E > most * half || (E >= least * nb && nb <= at_once)) break;
  }
  B.nb = (int)buckets(B.shift);
  if (E > kMostCrowded && E > most * B.nb) return CsrPath::kSort;
  // A bucket is cut if its samples speak for more than fits: 3 500 records, or `most` and five standard deviations of the
  // sample's count, whichever is more (buckets of `most` would be cut for nothing otherwise).  Where few rows leave more than
  // `most` to the average bucket, every one of about 1 024 is cut.  Pieces of about 1 536 records, but not of a single sample.
  const double share = (double)B.samples / (double)E;
  B.heavy = E > most * B.nb ? std::max(2, (int)(1024 * share))
                            : (int)std::ceil(std::max(3500 * share, most * share + 5 * std::sqrt(most * share)));
  B.cut = std::max(2, (int)(1536 * share));
  return CsrPath::kBuckets;
}

hipError_t csr_buckets(const int64_t* recv, const int64_t* send, int64_t E, int64_t V, int64_t* row_ptr, int64_t* col, int64_t* perm,
                       int64_t* t_row_ptr, int64_t* t_perm, char* block, const BucketPlan& B, int* bad_flag, hipStream_t st) {
  const BucketWs w{block};
  int* bad = bad_flag ? bad_flag : (int*)(block + BucketWs::bytes(E) - 256);
  const int transpose = t_row_ptr != nullptr, tiles = (int)((E + B.tile - 1) / B.tile);
  const int groups = B.nb + B.samples / B.cut;   // a bucket with c samples has at most 1 + c / cut pieces
  hipLaunchKernelGGL(k_csr_cut, dim3(1 + transpose), dim3(kThreads), 0, st, recv, send, E, V, B, w, bad);
  hipLaunchKernelGGL(k_csr_count, dim3(tiles), dim3(kThreads), 0, st, recv, send, E, V, B, w, transpose);
  hipLaunchKernelGGL(k_csr_distribute, dim3(tiles + transpose), dim3(kThreads), 0, st, recv, send, E, V, B, w, tiles, bad);
  hipLaunchKernelGGL(k_csr_rows<false>, dim3(groups), dim3(kThreads), 0, st, B, w, V, E, row_ptr, perm, col, transpose);
  if (transpose) hipLaunchKernelGGL(k_csr_rows<true>, dim3(groups), dim3(kThreads), 0, st, B, w, V, E, t_row_ptr, t_perm, (int64_t*)nullptr, 0);
  return hipGetLastError();
}

}  // namespace

// Grows with E and with V, so that one buffer serves every smaller graph: nothing where one workgroup does it, what E makes of
// the buckets' tables as long as they take any number of rows, and beyond that at least as much as the sorts need too.
hipError_t csr_workspace_bytes(int64_t E, int64_t V, size_t* bytes) {
  *bytes = 256;
  if (E <= 0) return hipSuccess;
  BucketPlan B;
  if (csr_path(E, V, B) == CsrPath::kSmall) return hipSuccess;
  *bytes = BucketWs::bytes(std::min(E, kMostEdges));
  if (E <= kMostCrowded && V <= kMostNodes) return hipSuccess;
  CsrLayout L;
  CSR_TRY(csr_layout(E, V, L));
  *bytes = std::max(*bytes, L.total);
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
    if (!workspace || workspace_bytes < BucketWs::bytes(E)) return hipErrorInvalidValue;
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
