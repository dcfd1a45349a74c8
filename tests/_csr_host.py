"""Runs the bucket path of the CSR preparation on the host: the kernels' own source between two marks of csr.hip, compiled
with g++ (and its address sanitizer: every array is exactly as large as the path says) behind a small model of a
workgroup - 1 024 fibers that change at barriers and wave operations.  The result is compared with a sort.  Test
infrastructure: nothing in the product imports this."""
import os
import subprocess
import tempfile

CSR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2501_13986_amd", "csrc", "csr.hip")

_PRE = r'''
#include <ucontext.h>
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <random>
#include <vector>
#include <sanitizer/asan_interface.h>
#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)
struct Dim { unsigned x; };
static Dim blockIdx, gridDim, blockDim;
static const int kGroup = 1024;
static ucontext_t g_main, g_fiber[kGroup];
static std::vector<char> g_stack[kGroup];
static int g_me, g_left;
static bool g_done[kGroup];
static std::function<void()> g_body;
#define threadIdx (Dim{(unsigned)g_me})
static void g_yield() {            // to the next live fiber, round robin
  const int from = g_me;
  do g_me = (g_me + 1) % kGroup; while (g_done[g_me]);
  if (g_me != from) swapcontext(&g_fiber[from], &g_fiber[g_me]);
}
static void g_entry() {
  g_body();
  g_done[g_me] = true;
  if (--g_left == 0) setcontext(&g_main);
  const int from = g_me;
  do g_me = (g_me + 1) % kGroup; while (g_done[g_me]);
  (void)from;
  setcontext(&g_fiber[g_me]);
}
// a barrier of n fibers in group g (groups: 0..15 waves, 16 the workgroup)
static int g_in[17], g_gen[17];
static void g_wait(int g, int n) {
  const int gen = g_gen[g];
  if (++g_in[g] == n) { g_in[g] = 0; ++g_gen[g]; }
  else while (g_gen[g] == gen) g_yield();
}
static int g_or, g_or_out;
static void __syncthreads() { g_wait(16, kGroup); }
static int __syncthreads_or(int v) {
  if (v) g_or = 1;
  g_wait(16, kGroup);
  g_or_out = g_or;
  g_wait(16, kGroup);
  g_or = 0;
  return g_or_out;
}
static int64_t g_x[kGroup];
static int g_exchange(int v, int from) {     // from: lane of this wave
  const int w = g_me / 64;
  g_x[g_me] = v;
  g_wait(w, 64);
  const int r = (int)g_x[w * 64 + from];
  g_wait(w, 64);
  return r;
}
static int __shfl(int v, int lane, int) { if (lane < 0 || lane > 63) { std::printf("lane %d\n", lane); std::exit(3); } return g_exchange(v, lane); }
static int __shfl_up(int v, int d, int) { const int l = g_me % 64; return g_exchange(v, l >= d ? l - d : l); }
static uint64_t __ballot(bool p) {
  const int w = g_me / 64;
  g_x[g_me] = p;
  g_wait(w, 64);
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) m |= (uint64_t)(g_x[w * 64 + l] != 0) << l;
  g_wait(w, 64);
  return m;
}
static int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
static int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
static int atomicAdd(int* p, int v) { const int o = *p; *p = o + v; return o; }
template <class F> static void run_grid(int grid, F f) {
  gridDim.x = grid;
  for (int b = 0; b < grid; ++b) {
    blockIdx.x = b;
    g_body = f;
    g_left = kGroup;
    for (int i = 0; i < kGroup; ++i) {
      g_done[i] = false;
      if (g_stack[i].empty()) g_stack[i].resize(1 << 15);
      getcontext(&g_fiber[i]);
      g_fiber[i].uc_stack.ss_sp = g_stack[i].data();
      g_fiber[i].uc_stack.ss_size = g_stack[i].size();
      g_fiber[i].uc_link = nullptr;
      makecontext(&g_fiber[i], (void (*)())g_entry, 0);
    }
    g_me = 0;
    swapcontext(&g_main, &g_fiber[0]);
  }
}
static unsigned bits_for(uint64_t max_value) { unsigned b = 1; while (b < 64 && (max_value >> b) != 0) ++b; return b; }
template <class T> static void here_scalar(T) {}
enum class CsrPath { kSmall, kBuckets, kSort };
'''

_POST = r'''
// prints: path, pieces of receivers and senders, records of the largest piece; exit status 1 if the result is wrong
int main(int argc, char** argv) {
  const int64_t V = atoll(argv[1]), E = atoll(argv[2]);
  const char *rh = argv[3], *sh = argv[4];
  std::mt19937_64 g(V * 131 + E);
  std::vector<int64_t> recv(E), send(E);
  auto fill = [&](std::vector<int64_t>& a, const char* how) {
    for (int64_t e = 0; e < E; ++e) {
      a[e] = (int64_t)(g() % (uint64_t)V);
      if (!strcmp(how, "hub") && g() % 2) a[e] = V / 3;
      if (!strcmp(how, "one")) a[e] = V - 1;
      if (!strcmp(how, "pad") && e >= E / 3) a[e] = V - 1;       // equal edges at the end of the list
      if (!strcmp(how, "tail") && e >= E - E / 9) a[e] = V - 1;  // fewer of them
      if (!strcmp(how, "two") && e % 2) a[e] = e % 4 == 1 ? 0 : V - 1;
      if (!strcmp(how, "missed")) {                              // a row that no sampled edge enters
        int64_t t = e * 1024 / E;
        while (t + 1 < 1024 && (t + 1) * E / 1024 <= e) ++t;
        while (t * E / 1024 > e) --t;
        const int64_t lo = t * E / 1024, room = ((t + 1) * E / 1024 - lo - 4) / 2 + 1;
        const int64_t hit = lo + (int64_t)((((uint64_t)((unsigned)t * 2654435761u)) * (uint64_t)room) >> 32);
        if ((e < hit || e > hit + 3) && e % 3) a[e] = V / 2;
      }
      if (!strcmp(how, "bad") && e % 97 == 5) a[e] = e % 2 ? -1 : V;
    }
    if (!strcmp(how, "sorted")) std::sort(a.begin(), a.end());
  };
  fill(recv, rh);
  fill(send, sh);
  BucketPlan B;
  const CsrPath path = csr_path(E, V, B);
  std::vector<int64_t> rp(V + 1, -7), col(E, -7), perm(E, -7), trp(V + 1, -7), tp(E, -7);
  int bad = 9, n1 = 0, n2 = 0, largest = 0;
  if (path == CsrPath::kSmall) {
    run_grid(1, [&] { k_csr_small(recv.data(), send.data(), (int)E, (int)V, B.eb, B.vb, rp.data(), col.data(), perm.data(), trp.data(), tp.data(), &bad); });
  } else if (path == CsrPath::kBuckets) {
    // one block as large as the path says, with the space between its tables poisoned
    const int64_t tiles = (E + B.tile - 1) / B.tile, rows = (E + kTile - 1) / kTile;
    const size_t bytes = BucketWs::bytes(E);
    char* const block = (char*)aligned_alloc(256, (bytes + 255) / 256 * 256);
    memset(block, 0x5a, bytes);
    const BucketWs w{block};
    std::vector<std::pair<char*, size_t>> tables = {{block, sizeof(BucketInfo)}, {(char*)w.cursor2(), kCuts * 4}, {(char*)w.before(), rows * kCuts * 4}, {(char*)w.rec1(E), E * 8}, {(char*)w.rec2(E), E * 8}};
    for (int s = 0; s < 2; ++s) {
      const BucketSide d = w.side(s);
      for (auto t : std::vector<std::pair<char*, size_t>>{{(char*)d.first(), (kBuckets + 1) * 4}, {(char*)d.owner(), kCuts * 4},
                                                          {(char*)d.low(), kCuts * 8}, {(char*)d.total(), kCuts * 4}, {(char*)d.base(), (kCuts + 1) * 4}})
        tables.push_back(t);
    }
    std::sort(tables.begin(), tables.end());
    __asan_poison_memory_region(block, bytes);
    for (size_t i = 0; i < tables.size(); ++i) {
      __asan_unpoison_memory_region(tables[i].first, tables[i].second);
      const size_t end = tables[i].first - block + tables[i].second;
      if (end > (i + 1 < tables.size() ? (size_t)(tables[i + 1].first - block) : bytes)) { std::printf("tables overlap\n"); return 1; }
    }
    const int groups = B.nb + B.samples / B.cut;
    run_grid(2, [&] { k_csr_cut(recv.data(), send.data(), E, V, B, w, &bad); });
    run_grid((int)tiles, [&] { k_csr_count(recv.data(), send.data(), E, V, B, w, 1); });
    run_grid((int)tiles + 1, [&] { k_csr_distribute(recv.data(), send.data(), E, V, B, w, (int)tiles, &bad); });
    run_grid(groups, [&] { k_csr_rows<false>(B, w, V, E, rp.data(), perm.data(), col.data(), 1); });
    run_grid(groups, [&] { k_csr_rows<true>(B, w, V, E, trp.data(), tp.data(), nullptr, 0); });
    n1 = w.info()->side[0].pieces; n2 = w.info()->side[1].pieces;
    for (int s = 0; s < 2; ++s)
      for (int p = 0; p < w.info()->side[s].pieces; ++p) largest = std::max(largest, w.side(s).base()[p + 1] - w.side(s).base()[p]);
  }
  std::printf("path %d pieces %d %d largest %d buckets %d\n", (int)path, n1, n2, largest, path == CsrPath::kBuckets ? B.nb : 0);
  if (path == CsrPath::kSort) return 0;
  int want_bad = 0;
  for (int64_t e = 0; e < E; ++e)
    if (recv[e] < 0 || recv[e] >= V || send[e] < 0 || send[e] >= V) { recv[e] = send[e] = 0; want_bad = 1; }
  std::vector<int64_t> o(E), q(E), c1(V + 1, 0), c2(V + 1, 0);
  for (int64_t e = 0; e < E; ++e) { o[e] = q[e] = e; ++c1[recv[e] + 1]; ++c2[send[e] + 1]; }
  for (int64_t v = 0; v < V; ++v) { c1[v + 1] += c1[v]; c2[v + 1] += c2[v]; }
  std::stable_sort(o.begin(), o.end(), [&](int64_t a, int64_t b) { return recv[a] != recv[b] ? recv[a] < recv[b] : send[a] < send[b]; });
  std::stable_sort(q.begin(), q.end(), [&](int64_t a, int64_t b) { return send[o[a]] < send[o[b]]; });
  for (int64_t e = 0; e < E; ++e)
    if (perm[e] != o[e] || col[e] != send[o[e]] || tp[e] != q[e]) { std::printf("WRONG at %lld\n", (long long)e); return 1; }
  if (rp != c1 || trp != c2 || bad != want_bad) { std::printf("WRONG row pointers or flag\n"); return 1; }
  return 0;
}
'''


def build():
    """Path of the compiled program (in a directory of its own)."""
    s = open(CSR).read()
    kernels = s[s.index("// ---- bucket path"):s.index("inline unsigned blocks_for(int64_t n)")]
    host = s[s.index("constexpr int64_t kMostEdges"):s.index("hipError_t csr_buckets(")]
    d = tempfile.mkdtemp(prefix="csr_host_")
    src = os.path.join(d, "csr_host.cpp")
    with open(src, "w") as f:
        f.write(_PRE + kernels + host + _POST)
    exe = os.path.join(d, "csr_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address", "-Wno-unknown-pragmas", "-w", src, "-o", exe], check=True)
    return exe


def run(exe, V, E, receivers, senders):
    """(exit status, numbers of the program's line): pieces of receivers and senders, records of the largest, buckets."""
    p = subprocess.run([exe, str(V), str(E), receivers, senders], capture_output=True, text=True, timeout=600,
                       env={**os.environ, "ASAN_OPTIONS": "detect_stack_use_after_return=0:detect_leaks=0"})
    text = p.stdout + p.stderr[-1500:]
    t = p.stdout.split()
    seen = {"path": int(t[1]), "pieces": (int(t[3]), int(t[4])), "largest": int(t[6]), "buckets": int(t[8])} if len(t) >= 9 else {}
    return p.returncode, text, seen
