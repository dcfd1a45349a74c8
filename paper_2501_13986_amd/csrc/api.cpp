// The C ABI of include/cgtp.h: planning (static analysis of the irreps, paper Sec. 3.1),
// kernel generation and the launches.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <stdexcept>
#include <string>
#include <tuple>

#include "conv_split.hpp"
#include "csr.hpp"
#include "plan.hpp"

struct cgtp_plan {
  cgtp::Plan P;
};

namespace {

thread_local std::string g_err;

cgtp_status fail(cgtp_status s, const std::string& msg) {
  g_err = msg;
  return s;
}

#define HIP_TRY(expr)                                                                                   \
  do {                                                                                                  \
    hipError_t e_ = (expr);                                                                             \
    if (e_ != hipSuccess) return fail(CGTP_ERUNTIME, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

using cgtp::Irrep;
using cgtp::Kernel;
using cgtp::LaneMap;
using cgtp::PathInfo;
using cgtp::Plan;

bool allowed(const Irrep& a, const Irrep& b, const Irrep& c) {
  return std::abs(a.l - b.l) <= c.l && c.l <= a.l + b.l && c.p == a.p * b.p;
}

std::vector<int64_t> prefix(const std::vector<Irrep>& v) {
  std::vector<int64_t> o{0};
  for (auto& ir : v) o.push_back(o.back() + ir.dim());
  return o;
}

int pow2ceil(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

// Channel -> lane assignment.  Adjacent channels share a lane (`cpl` of them) so that a lane's
// words are contiguous; a wave is filled with several samples when the multiplicity is small.
// step: 0 the convolution's wide map, 1 the narrow one, 2 one channel per lane (other kernels: the same map for all).
LaneMap pick_map(const Plan& P, int kind, int step) {
  static const char* const kTag[9] = {"TP_FWD",          "TP_BWD",     "CONV_FWD",     "CONV_BWD",    "CONV_FWD_ATOMIC",
                                      "CONV_BWD_ATOMIC", "TP_DBL_BWD", "CONV_DBL_FWD", "CONV_DBL_BWD"};
  const bool conv = kind == CGTP_K_CONV_FWD || kind == CGTP_K_CONV_BWD || kind == CGTP_K_CONV_FWD_ATOMIC ||
                    kind == CGTP_K_CONV_DBL_FWD || kind == CGTP_K_CONV_DBL_BWD;
  const bool atomic = kind == CGTP_K_CONV_FWD_ATOMIC || kind == CGTP_K_CONV_BWD_ATOMIC;
  int M = 1;
  bool even = true;
  for (auto& q : P.paths) {
    M = std::max(M, q.mul_x);
    even = even && (q.mul_x % 2 == 0);
  }
  LaneMap m;
  // tuning overrides: CGTP_CPL / CGTP_OCC for all kernels, CGTP_CPL_<KIND> / CGTP_OCC_<KIND> for one
  int cpl = cgtp::env_int((std::string("CGTP_CPL_") + kTag[kind]).c_str(), cgtp::env_int("CGTP_CPL", 0));
  if (cpl <= 0) {
    cpl = (even && M >= 128) ? 2 : 1;
    // measured on the 128-channel MACE shape: the fp32 batched backward is faster with one channel per
    // lane and two passes (more waves in flight), everything else with two adjacent channels per lane
    if (kind == CGTP_K_TP_BWD && P.dtype == CGTP_F32) cpl = 1;
    // float atomics are carried out at the memory side in 32-byte requests: one channel per lane makes the
    // 64 lanes of an atomic instruction cover contiguous words (8 requests in fp32 instead of 16 with pairs)
    if (atomic) cpl = 1;
    // twice the operands of the first-order kernels per channel
    if (kind == CGTP_K_TP_DBL_BWD || (kind == CGTP_K_CONV_DBL_FWD && step > 0)) cpl = 1;
    // A convolution kernel that needs a second pass walks its whole edge range again (y, the graph arrays and the
    // gathers' latency once more, and a sender walk reads back its gy words), so the lane takes as many adjacent
    // channels (up to `most`) as bring it to one pass.
    // us on 3 000 nodes of degree 30 (* 1 500), fp32, with two passes -> one: 96 channels fwd 92 -> 83, bwd 160 -> 141,
    // second order 365 -> 338; 192 channels 228 -> 199, 402 -> 356, 990 -> 882; 256 channels, l <= 3 (*) backward
    // 378 -> 357, second order 1013 -> 883 (and the forward would be 222 -> 190).  fp64 with 96 channels 163 -> 129, 310 -> 241, 732 -> 573, but three or four channels are
    // too many registers there: bwd 192 channels 740 -> 822, 256 channels 774 -> 855.  The forward
    // walk stops at three: with four, a 256-channel plan would have half the edge ranges, and conv_forward_static, which refuses
    // by their number, would take what it refuses.  The receiver walk of the
    // second-order pass up to 128 fp32 channels stays at one channel and two passes (128 channels 645, in one pass 667).
    if (conv && step == 2) cpl = 1;
    if (conv && !atomic && step == 0) {
      int most = P.dtype == CGTP_F32 ? (kind == CGTP_K_CONV_FWD ? 3 : 4) : 2;
      if (kind == CGTP_K_CONV_DBL_FWD && P.dtype == CGTP_F32 && M <= 128) most = 1;
      for (int c = 1; c <= most; ++c) {
        bool divides = true;
        for (auto& q : P.paths) divides = divides && q.mul_x % c == 0;
        if (divides && M <= 64 * c) {
          cpl = c;
          break;
        }
      }
      if (most == 1) cpl = 1;
    }
  }
  for (auto& q : P.paths)
    if (q.mul_x % cpl) cpl = 1;
  m.cpl = cpl;
  m.occ = cgtp::env_int((std::string("CGTP_OCC_") + kTag[kind]).c_str(), cgtp::env_int("CGTP_OCC", 0));
  if (m.occ == 0 && kind == CGTP_K_TP_FWD && P.dtype == CGTP_F64 && cpl == 2) m.occ = 2;  // measured: 0.45 vs 0.49 ms
  int lanes = (M + cpl - 1) / cpl;
  // a multiplicity that fills only part of a wave: several samples (batched kernels) or several independent
  // edge-range workers (convolution kernels) share the wave
  m.G = (conv && cgtp::env_int("CGTP_CONV_SPLIT_WAVE", 1) == 0) ? 64 : std::min(64, pow2ceil(lanes));
  m.spw = 64 / m.G;
  m.npass = (M + m.G * cpl - 1) / (m.G * cpl);
  return m;
}

// Schedules to try for a kernel, most aggressive first (all loads of a row in flight, software pipelining)
// down to the most economical in registers (products v*y[j] local to each path, accumulators brought up to
// date after every path, loads where they are used, x segments in phases).
std::vector<cgtp::Schedule> schedule_candidates(int kind, bool small) {
  using S = cgtp::Schedule;
  auto mk = [](int w_upfront, int upfront, int prefetch, int pin, int fresh_y, int phases) {
    S s;
    s.w_upfront = w_upfront;
    s.upfront = upfront;
    s.prefetch = prefetch;
    s.pin = pin;
    s.fresh_y = fresh_y;
    s.phases = phases;
    return s;
  };
  switch (kind) {
    case CGTP_K_TP_FWD:
      // many paths: per-path y products first (measured 0.32 vs 0.40 ms on a 68-path plan, fewer registers)
      if (!small) return {mk(-1, -1, -1, -1, 1, 1), mk(0, -1, -1, -1, 1, 1), S()};
      return {S(), mk(-1, -1, -1, -1, 1, 1), mk(0, -1, -1, -1, 1, 1)};
    case CGTP_K_CONV_FWD:
    case CGTP_K_CONV_FWD_ATOMIC:
      return {S(), mk(-1, -1, 0, -1, -1, 1), mk(-1, -1, 0, -1, 1, 1), mk(0, -1, 0, -1, 1, 1),
              mk(0, -1, 0, -1, 1, 2), mk(0, -1, 0, -1, 1, 3)};   // last: phases over output segments
    case CGTP_K_TP_BWD:
      return {S(), mk(-1, -1, -1, 2, 1, 1), mk(-1, 0, -1, 2, 1, 1), mk(-1, 0, -1, 2, 1, 3)};
    case CGTP_K_CONV_BWD:
      return {S(), mk(-1, -1, -1, 2, 1, 1), mk(-1, 0, -1, 2, 1, 1), mk(-1, 0, -1, 2, 1, 2), mk(-1, 0, -1, 2, 1, 3)};  // last: x phases
    case CGTP_K_CONV_BWD_ATOMIC:
      return {S(), mk(-1, -1, -1, 2, 1, 1), mk(-1, 0, -1, 2, 1, 1)};
    case CGTP_K_CONV_DBL_FWD:
      return {mk(-1, -1, -1, 1, 1, 1), mk(0, -1, -1, 1, 1, 1)};
    case CGTP_K_CONV_DBL_BWD:
      return {mk(-1, -1, -1, 2, 1, 1), mk(-1, 0, -1, 2, 1, 1)};
    case CGTP_K_TP_DBL_BWD: {
      // last: the economical schedule held to two waves per SIMD; a light spill at that occupancy measured
      // faster than no spill at one wave per SIMD (0.83 vs 1.05 ms on a 68-path plan)
      S two = mk(-1, -1, -1, 2, 1, 1);
      two.occ = 2;
      return {mk(-1, -1, -1, 1, 1, 1), mk(-1, -1, -1, 2, 1, 1), two, mk(-1, -1, -1, 2, 1, 2), mk(-1, -1, -1, 2, 1, 3),
              mk(-1, -1, -1, 2, 1, 5)};
    }
  }
  return {S()};
}

// Emits and compiles the candidates of one kernel in turn and keeps the first that is free of private-memory
// spills and (for plans with many paths) fits 256 registers, i.e. two waves per SIMD.  If none does, candidates
// are ranked: within 256 registers with a light spill (<= 256 B), then spill-free with more registers, then by
// the amount of spill.  Small plans keep their first spill-free schedule: those defaults were tuned by
// measurement and some of them are fastest with more than 256 registers.  Without compilation (device == -1)
// the first candidate is taken.
struct CompileError {
  std::string msg;
};

// Plans with more paths than this are tuned for registers, not by their first schedule.
constexpr size_t kFewPaths = 24;

// What a kernel's registers cost, best first: 0 no private memory and (many paths) within 256 registers, i.e. two waves per
// SIMD; 1 within 256 with a light spill (many paths); 2 no private memory, one wave per SIMD; above: the spill.
long register_class(const Kernel& k, bool few) {
  if (k.scratch == 0) return few || k.vgprs <= 256 ? 0 : 2;
  if (!few && k.scratch <= 256 && k.vgprs <= 256) return 1;
  return 2 + k.scratch;
}

template <class Emit>
void build_kernel(cgtp::Plan& P, int kind, Emit emit, int device) {
  Kernel& K = P.k[kind];
  const bool small = P.paths.size() <= kFewPaths;
  std::vector<cgtp::Schedule> cands = schedule_candidates(kind, small);
  if (cgtp::env_int("CGTP_NO_SCHEDULE_SEARCH", 0)) cands.resize(1);
  Kernel best;
  long best_key = -1;
  std::string refused;
  for (size_t c = 0; c < cands.size(); ++c) {
    // phases cost re-reads (measured slower than a single phase at one wave per SIMD): they are tried only while
    // every schedule so far needs more than a light spill
    if (cands[c].phases > 1 && best_key >= 0 && best_key < 1000000L) continue;
    Kernel cur;
    cur.sched = cands[c];
    emit(cur);
    if (device == -1) {
      K = std::move(cur);
      return;
    }
    bool dup = false;   // environment overrides can make candidates identical
    if (best_key >= 0 && cur.source == best.source) dup = true;
    if (dup) continue;
    try {
      cgtp::jit_compile(cur, -2);
    } catch (const cgtp::RefusedCode& e) {   // this schedule's code failed the mask check: next candidate
      refused = e.what();
      continue;
    } catch (const std::exception& e) {
      throw CompileError{e.what()};
    }
    const bool fits = register_class(cur, small) == 0;
    // ranking of the candidates that do not fit (many-path plans): within 256 registers with at most 256 B of
    // private memory, then spill-free with more registers (one wave per SIMD), then by the amount of spill
    long key;
    if (cur.scratch == 0) key = cur.vgprs <= 256 ? cur.vgprs : 20000L + cur.vgprs;
    else if (!small && cur.scratch <= 256 && cur.vgprs <= 256) key = 10000L + cur.scratch;
    else key = 1000000L + cur.scratch;
    if (best_key < 0 || key < best_key) {
      best = cur;
      best_key = key;
    }
    if (fits) {
      best = std::move(cur);
      break;
    }
  }
  if (best_key < 0 && !refused.empty()) throw CompileError{refused};
  K = std::move(best);
}

// For kernels that a plan can do without.  false: the code did not compile, failed its check or needs private memory
bool compiles_without_scratch(Kernel& k, int device) {
  try {
    cgtp::jit_compile(k, device == -1 ? -1 : -2);
  } catch (const std::exception&) {
    return false;
  }
  return k.scratch == 0;
}

std::vector<Kernel*> row_kernels(Plan& P) {
  return {&P.k_row[0][0], &P.k_row[0][1], &P.k_row[1][0], &P.k_row[1][1], &P.k_dbl_row[0], &P.k_dbl_row[1], &P.k_dbl_row[2], &P.k_row_sums};
}

// The kernels that walk row by row: with the schedule of the range kernels, or the one that needs the fewest registers; not
// where that too needs private memory or fails the check of the compiled code, and not for plans of many paths.
void build_rows(Plan& P, int device) {
  if (P.paths.size() > kFewPaths || !cgtp::env_int("CGTP_CONV_ROWS", 1)) return;
  for (int back = 0; back < 2; ++back) {
    const LaneMap& m = P.map[back ? CGTP_K_CONV_BWD : CGTP_K_CONV_FWD];
    cgtp::Schedule frugal;
    frugal.w_upfront = frugal.upfront = 0;
    frugal.pin = 2;
    frugal.fresh_y = 1;
    cgtp::Schedule first = P.k[back ? CGTP_K_CONV_BWD : CGTP_K_CONV_FWD].sched;
    if (back) first.upfront = 1;
    auto compiled = [&](Kernel& k, bool nt, int waves) { return cgtp::emit_uvu_conv_row(P, back != 0, nt, waves, k) && compiles_without_scratch(k, device); };
    // Workers of a row (us per call, 128 channels unless given): eight, on eight waves; four waves where the registers leave
    // room for one workgroup of eight (forward fp64, 5 000 nodes of degree 32, 617 -> 594).  For long streams fewer, so that
    // more rows are in flight: four workers where they share waves (32 channels, 20 000 nodes of degree 9, forward 116 -> 102),
    // three or four waves in the backward (96 channels, 20 000 of degree 32, 895 on eight, 841 on four and on three; of degree 9
    // 337, 275, 268), half of that for kernels of more than 128 registers whose workers share waves (32 channels fp64, 20 000 of
    // degree 32, 1444 -> 1329).
    for (const cgtp::Schedule& s : {first, frugal}) {
      Kernel plain, nt;
      const int full = std::max(1, 8 / m.spw), many = back ? 168 : 128;
      auto attempt = [&](Kernel& k, bool stream, int waves) {
        k = Kernel();
        k.sched = s;
        return compiled(k, stream, waves);
      };
      bool ok = attempt(plain, false, full);
      if (full > 4 && (!ok || plain.vgprs > many)) ok = attempt(plain, false, 4);
      // a backward with more registers is no faster than the ranges (128 channels fp64, 100 nodes of degree 32: 44 -> 55)
      if (!ok || (back && plain.vgprs > 200)) continue;
      int waves = plain.wg / 64;
      if (m.spw > 1) waves = std::max(1, 4 / m.spw);
      else if (back) waves = std::min(waves, plain.vgprs > 128 ? 4 : 3);
      if (back && m.spw > 1 && plain.vgprs > 128) waves = std::max(1, waves / 2);
      if (!attempt(nt, true, waves)) continue;
      P.k_row[back][0] = std::move(plain);
      P.k_row[back][1] = std::move(nt);
      break;
    }
  }
}

// The second-order pass in one walk: eight waves a row where there are few rows (32 channels, 300 nodes of degree 32, 66 us on
// two waves and 38 on eight), four workers where there are many (2 000 nodes of degree 9, 56 and 68).
void build_double_rows(Plan& P, int device) {
  if (P.paths.size() > kFewPaths || !cgtp::env_int("CGTP_CONV_ROWS", 1)) return;
  const int spw = P.map[CGTP_K_CONV_DBL_BWD].spw, many = std::max(1, 4 / spw), few = spw >= 16 ? 2 : 8;
  Kernel k[3], sums;
  for (int t = 0; t < 3; ++t) {
    k[t].sched = P.k[CGTP_K_CONV_DBL_BWD].sched;
    if (!cgtp::emit_uvu_conv_double_row(P, t == 2, t == 0 ? few : many, k[t]) || !compiles_without_scratch(k[t], device)) return;
  }
  if (!cgtp::emit_row_sums(P, sums) || !compiles_without_scratch(sums, device)) return;
  for (int t = 0; t < 3; ++t) P.k_dbl_row[t] = std::move(k[t]);
  P.k_row_sums = std::move(sums);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

cgtp_status launch(const Kernel& k, unsigned grid, void** args, hipStream_t st) {
  if (!k.fn) return fail(CGTP_EUNSUPPORTED, "kernel " + k.name + " is not loaded (plan created without a device?)");
  HIP_TRY(hipModuleLaunchKernel(k.fn, grid, 1, 1, (unsigned)k.wg, 1, 1, 0, st, args, nullptr));
  return CGTP_OK;
}

cgtp_status ensure_ws(Plan& P, size_t bytes) {
  if (bytes <= P.ws_bytes) return CGTP_OK;
  if (P.ws) {
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipFree(P.ws));
    P.ws = nullptr;
    P.ws_bytes = 0;
  }
  hipError_t e = hipMalloc(&P.ws, bytes);
  if (e != hipSuccess) return fail(CGTP_ENOMEM, "workspace allocation of " + std::to_string(bytes) + " bytes failed");
  P.ws_bytes = bytes;
  return CGTP_OK;
}

// The merge kernel of the convolution's split rows: one wave per edge range and slice of a row (emit_fixup).
cgtp_status launch_fixup(const Plan& P, const void* out, const void* part, const int64_t* ptr, int64_t V, int64_t E, int64_t nchunk,
                         int64_t row, hipStream_t st) {
  const int64_t words = 64 * (P.dtype == CGTP_F64 ? 2 : 4), slices = (row + words - 1) / words, wpw = P.k_fix.wg / 64;
  int dim = (int)row;
  void* args[] = {(void*)&out, (void*)&part, (void*)&ptr, (void*)&V, (void*)&E, (void*)&nchunk, (void*)&dim};
  return launch(P.k_fix, (unsigned)((nchunk * slices + wpw - 1) / wpw), args, st);
}

int64_t resident_waves(const Plan& P, const Kernel& k) { return (int64_t)k.blocks_per_cu * P.num_cu * (k.wg / 64); }

int64_t most_ranges(const Plan& P, const Kernel& k, int spw) { return resident_waves(P, k) * spw * cgtp::env_int("CGTP_CONV_CHUNK_MULT", 1); }

int64_t conv_ranges(const Plan& P, const Kernel& k, int spw, int64_t E) { return cgtp::conv_ranges(most_ranges(P, k, spw), spw, E); }

// Workers of a row in a kernel that walks row by row; 0 if the plan has none.
int64_t row_workers(const Kernel& k, int spw) { return k.fn ? (int64_t)(k.wg / 64) * spw : 0; }

int row_lg(const Kernel& k, int spw, int64_t E, int64_t row_bytes) { return cgtp::row_lg(row_workers(k, spw), E, row_bytes); }

// Bytes of the pieces of split rows in the workspace of conv_forward or conv_backward: the same whichever kernel walks the graph.
size_t piece_bytes(const Plan& P, bool backward, int64_t E) {
  const int kind = backward ? CGTP_K_CONV_BWD : CGTP_K_CONV_FWD, spw = P.map[kind].spw;
  const int64_t row = (backward ? P.dim_x() : P.dim_z()) * (int64_t)P.elt();
  const Kernel* rows = P.k_row[backward];
  return (size_t)(cgtp::most_pieces(most_ranges(P, P.k[kind], spw), spw, {row_workers(rows[0], spw), row_workers(rows[1], spw)}, E, row) * row);
}

// A launch holds fewer than 2^32 work-items.
bool rows_launch(const Kernel& k, int64_t V) { return k.fn && V < ((int64_t)1 << 32) / k.wg - cgtp::kRowWindows; }

int64_t resident_groups(const Plan& P, const Kernel& k) { return (int64_t)k.blocks_per_cu * P.num_cu; }

// The kernel that walks a graph row by row, or NULL if the edge ranges do.  Non-temporal streams where the weights do not
// fit the Infinity Cache (128 channels, 300 nodes of degree 32, forward 25 us without the hint and 27 with it; 5 000 nodes 308
// and 300).
const Kernel* conv_by_rows(const Plan& P, bool backward, int64_t V, int64_t E) {
  const LaneMap& m = P.map[backward ? CGTP_K_CONV_BWD : CGTP_K_CONV_FWD];
  const int64_t stream = E * P.n_w * (int64_t)P.elt();
  const Kernel &plain = P.k_row[backward][0], &nt = P.k_row[backward][1];
  if (!rows_launch(plain, V) || !rows_launch(nt, V)) return nullptr;
  const bool few_channels = m.G * m.cpl * (int64_t)P.elt() < 128;
  if (!backward) return !few_channels && !cgtp::forward_by_rows(V, E) ? nullptr : stream > (int64_t)256 << 20 ? &nt : &plain;
  const cgtp::BackwardRows k{few_channels, P.dtype == CGTP_F64, m.cpl, m.spw, plain.vgprs > 128, resident_groups(P, plain), resident_groups(P, nt)};
  const int form = cgtp::backward_by_rows(k, V, E, stream);
  return form == 0 ? nullptr : form == 2 ? &nt : &plain;
}

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// The second-order pass of the convolution.  One walk over the receiver rows with a row of dL/dx per edge in memory, if the plan
// has the kernels and those rows are no more than four gigabytes (about half of one of the weight streams): 128 channels, 16 000
// nodes of degree 40, 2.9 GB, two walks 6043 us, one 5229.  Non-temporal where the three streams of weights do not fit the
// Infinity Cache (32 channels, 1 000 nodes of degree 32, 94 us without the hint and 103 with it; 2 000 nodes 178 and 173).
// The rows stand in the plan's workspace where the pieces and receivers of the two walks take as much anyway, else in memory
// that the caller hands over; without it the pass goes in two walks.  All of it follows from the plan, V and E, so that a call
// gives the same bits whatever was called before and whether it is captured or not.
struct DoubleWalk {
  int64_t nf = 0, nb = 0;                         // edge ranges of the two walks
  size_t part_b = 0, ws = 0;                      // their workspace, which never falls with E
  const Kernel* rows = nullptr;                   // one walk (NULL: none for this plan and graph)
  int lg = 0, lg2 = 0;
  size_t row_bytes = 0, one = 0;                  // bytes of the edges' rows, and with the pieces of cut rows
};

DoubleWalk double_walk(const Plan& P, int64_t V, int64_t E) {
  const int spwf = P.map[CGTP_K_CONV_DBL_FWD].spw, spwb = P.map[CGTP_K_CONV_DBL_BWD].spw;
  const size_t el = P.elt();
  DoubleWalk d;
  d.nf = conv_ranges(P, P.k[CGTP_K_CONV_DBL_FWD], spwf, E);
  d.nb = conv_ranges(P, P.k[CGTP_K_CONV_DBL_BWD], spwb, E);
  // the two walks run one after the other on the stream and share the side buffer; the receivers of somewhat more edges fit, as
  // neighbour lists breathe
  size_t receivers = 1024;
  while (receivers < (size_t)E) receivers *= 2;
  d.part_b = round_up((size_t)d.nb * 2 * P.dim_x() * el, 256);
  d.ws = std::max((size_t)d.nf * 2 * P.dim_z() * el, d.part_b + receivers * 8);
  const LaneMap& m = P.map[CGTP_K_CONV_DBL_BWD];
  const bool few_channels = m.G * m.cpl * (int64_t)el < 128;
  if (!few_channels && !cgtp::double_by_rows(V, E, resident_groups(P, P.k_dbl_row[1]), m.spw)) return d;
  if (!rows_launch(P.k_dbl_row[0], V) || !rows_launch(P.k_row_sums, V) || (size_t)E > ((size_t)4 << 30) / (P.dim_x() * el)) return d;
  d.row_bytes = round_up((size_t)E * P.dim_x() * el, 256);
  d.rows = &P.k_dbl_row[V <= 768 ? 0 : 3 * E * P.n_w * (int64_t)el > (int64_t)256 << 20 ? 2 : 1];
  d.lg = row_lg(*d.rows, spwb, E, P.dim_z() * (int64_t)el);
  d.lg2 = row_lg(P.k_row_sums, 1, E, P.dim_x() * (int64_t)el);
  const int64_t w = cgtp::row_windows(d.lg, E), w2 = cgtp::row_windows(d.lg2, E);   // one window: no row is cut
  d.one = d.row_bytes + 2 * el * (size_t)std::max(w > 1 ? w * P.dim_z() : 0, w2 > 1 ? w2 * P.dim_x() : 0);
  return d;
}

// 64 words of pinned host memory, one per cache line, handed out to concurrent calls; allocated on first use and kept
// until the process ends.  take() answers -1 if none is free or the allocation failed.
struct HostFlags {
  int32_t* flags = nullptr;
  std::atomic<uint64_t> used{0};
  HostFlags() {
    if (hipHostMalloc((void**)&flags, 64 * 64, hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      flags = nullptr;
    }
  }
  int take() {
    if (!flags) return -1;
    uint64_t u = used.load();
    while (~u) {
      const int slot = __builtin_ctzll(~u);
      if (used.compare_exchange_weak(u, u | ((uint64_t)1 << slot))) return slot;
    }
    return -1;
  }
  void give(int slot) { used.fetch_and(~((uint64_t)1 << slot)); }
};
HostFlags& host_flags() {
  static HostFlags* h = new HostFlags();   // not destroyed: calls may still run while the process ends
  return *h;
}


}  // namespace

extern "C" {

const char* cgtp_last_error(void) { return g_err.c_str(); }

cgtp_status cgtp_check_code_object(const char* path, char* found, size_t capacity) {
  if (!path || !found || capacity == 0) return fail(CGTP_EINVAL, "NULL argument");
  try {
    const std::string t = cgtp::jit_check_code_object(path);
    std::snprintf(found, capacity, "%s", t.c_str());
  } catch (const std::exception& e) {
    return fail(CGTP_EINVAL, e.what());
  }
  return CGTP_OK;
}

cgtp_status cgtp_plan_create(const char* irreps_x, const char* irreps_y, const char* irreps_z, const cgtp_path* paths,
                             int32_t n_paths, int32_t default_mode, int32_t shared_weights, int32_t dtype,
                             int32_t device, uint32_t flags, cgtp_plan** out) {
  return cgtp_plan_create_ex(irreps_x, irreps_y, irreps_z, paths, n_paths, default_mode, shared_weights, dtype, device,
                             flags, nullptr, out);
}

cgtp_status cgtp_plan_create_ex(const char* irreps_x, const char* irreps_y, const char* irreps_z, const cgtp_path* paths,
                                int32_t n_paths, int32_t default_mode, int32_t shared_weights, int32_t dtype,
                                int32_t device, uint32_t flags, const cgtp_options* options, cgtp_plan** out) {
  if (!out) return fail(CGTP_EINVAL, "out is NULL");
  *out = nullptr;
  if (flags & ~(uint32_t)CGTP_IR_MUL) return fail(CGTP_EINVAL, "unknown bit in flags");
  bool kahan = false;
  if (options) {
    if (options->struct_size < (int32_t)sizeof(int32_t)) return fail(CGTP_EINVAL, "cgtp_options.struct_size is not set");
    if (options->struct_size >= (int32_t)(2 * sizeof(int32_t))) kahan = options->kahan_conv != 0;
  }
  if (!irreps_x || !irreps_y || !irreps_z) return fail(CGTP_EINVAL, "irreps string is NULL");
  if (dtype != CGTP_F32 && dtype != CGTP_F64) return fail(CGTP_EINVAL, "dtype must be CGTP_F32 or CGTP_F64");
  if (n_paths < 0 || (n_paths > 0 && !paths)) return fail(CGTP_EINVAL, "bad path list");
  if (default_mode != CGTP_UVU && default_mode != CGTP_UVW) return fail(CGTP_EINVAL, "bad default_mode");
  std::unique_ptr<cgtp_plan> H(new (std::nothrow) cgtp_plan());
  if (!H) return fail(CGTP_ENOMEM, "out of host memory");
  Plan& P = H->P;
  P.kahan_conv = kahan;
  try {
    P.irx = cgtp::parse_irreps(irreps_x);
    P.iry = cgtp::parse_irreps(irreps_y);
    P.irz = cgtp::parse_irreps(irreps_z);
  } catch (const std::invalid_argument& e) {
    return fail(CGTP_EINVAL, e.what());
  }
  for (auto* v : {&P.irx, &P.iry, &P.irz})
    for (auto& ir : *v)
      if (ir.l > cgtp::kMaxL) return fail(CGTP_EUNSUPPORTED, "degree l > 8 is not supported");
  P.offx = prefix(P.irx);
  P.offy = prefix(P.iry);
  P.offz = prefix(P.irz);
  P.dtype = dtype;
  P.shared_w = shared_weights != 0;
  P.device = device;
  P.ir_mul = (flags & CGTP_IR_MUL) != 0;

  std::vector<cgtp_path> list;
  if (n_paths == 0) {
    for (int a = 0; a < (int)P.irx.size(); ++a)
      for (int b = 0; b < (int)P.iry.size(); ++b)
        for (int c = 0; c < (int)P.irz.size(); ++c)
          if (allowed(P.irx[a], P.iry[b], P.irz[c])) list.push_back(cgtp_path{a, b, c, default_mode, 1.0});
  } else {
    list.assign(paths, paths + n_paths);
  }
  if (list.empty()) return fail(CGTP_EINVAL, "no path: nothing to compute");
  std::stable_sort(list.begin(), list.end(), [](const cgtp_path& a, const cgtp_path& b) {
    return std::tie(a.ix, a.iy, a.iz) < std::tie(b.ix, b.iy, b.iz);
  });
  P.mode = list[0].mode;
  int64_t woff = 0;
  for (auto& q : list) {
    if (q.ix < 0 || q.ix >= (int)P.irx.size() || q.iy < 0 || q.iy >= (int)P.iry.size() || q.iz < 0 ||
        q.iz >= (int)P.irz.size())
      return fail(CGTP_EINVAL, "path segment index out of range");
    if (q.mode != CGTP_UVU && q.mode != CGTP_UVW) return fail(CGTP_EINVAL, "bad path mode");
    const Irrep &a = P.irx[q.ix], &b = P.iry[q.iy], &c = P.irz[q.iz];
    if (!allowed(a, b, c)) return fail(CGTP_EINVAL, "path violates the triangle or parity rule");
    if (!std::isfinite(q.coeff)) return fail(CGTP_EINVAL, "path coefficient is not finite");
    if (b.mul != 1) return fail(CGTP_EUNSUPPORTED, "y multiplicity must be 1");
    if (q.mode != P.mode) return fail(CGTP_EUNSUPPORTED, "mixing uvu and uvw paths in one plan is not supported");
    if (q.mode == CGTP_UVU && a.mul != c.mul) return fail(CGTP_EINVAL, "uvu path needs mul_x == mul_z");
    PathInfo pi;
    pi.ix = q.ix; pi.iy = q.iy; pi.iz = q.iz; pi.mode = q.mode; pi.coeff = q.coeff;
    pi.l1 = a.l; pi.l2 = b.l; pi.l3 = c.l;
    pi.mul_x = a.mul; pi.mul_z = c.mul;
    pi.w_off = woff;
    try {
      pi.nz = cgtp::cg_nonzeros(a.l, b.l, c.l);
    } catch (const std::exception& e) {
      return fail(CGTP_ERUNTIME, e.what());
    }
    woff += (int64_t)a.mul * (q.mode == CGTP_UVU ? 1 : c.mul);
    P.paths.push_back(std::move(pi));
  }
  for (size_t t = 1; t < P.paths.size(); ++t)
    if (P.paths[t].ix == P.paths[t - 1].ix && P.paths[t].iy == P.paths[t - 1].iy && P.paths[t].iz == P.paths[t - 1].iz)
      return fail(CGTP_EINVAL, "duplicate path");
  P.n_w = woff;
  if (P.shared_w && P.mode == CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "shared weights are supported for uvw plans only");
  if (P.ir_mul && P.mode != CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "the IR_MUL layout is implemented for uvu plans only");

  for (int k = 0; k < 9; ++k) P.map[k] = pick_map(P, k, 0);
  try {
    if (P.mode == CGTP_UVU) {
      // A convolution kernel whose wave holds several edge-range workers is lane-divergent by design.  If every
      // schedule of it is refused (see jit_compile: divergence together with register relocation), the kernel is
      // generated again with one worker per wave, which has no lane-conditional code.
      auto build_worker = [&](int kind, auto emit) {
        try {
          build_kernel(P, kind, emit, device);
        } catch (const CompileError&) {
          if (P.map[kind].spw <= 1) throw;
          LaneMap& m = P.map[kind];
          int M = 1;
          for (auto& q : P.paths) M = std::max(M, q.mul_x);
          m.G = 64;
          m.spw = 1;
          m.npass = (M + m.G * m.cpl - 1) / (m.G * m.cpl);
          build_kernel(P, kind, emit, device);
        }
      };
      // The wide lane map is chosen from the multiplicities alone; what it costs in registers depends on the paths.  Where its
      // kernel needs private memory or (many paths, second-order pass) leaves one wave per SIMD, the narrow map's is
      // compiled as well, then one channel per lane's, and the first of the best class (register_class) is kept.  The
      // receiver walks of a plan with many paths take the narrow map at once: they are bound by their instructions (in fp64
      // the second-order one is not where both maps leave one wave per SIMD).
      // us per kernel, 1 000 nodes of degree 30, both parities, y of l <= 3, wide -> this: second-order sender walk fp32
      // 96 channels l <= 3 1260 -> 723, 144 6377 -> 1894, 192 5893 -> 1740, 256 9028 -> 2351, 160 channels l <= 2 1377 -> 547;
      // fp64 96 channels l <= 3 8243 -> 3567, 192 channels l <= 2 5758 -> 1395; second-order receiver walk 160 channels l <= 2
      // 1137 -> 323, 192 466 -> 358; forward fp32 96 channels l <= 3 289 -> 226 (but 144 l <= 2 173 -> 223), fp64 989 -> 697.
      // The sender walk of the backward gains from the wide map with any number of paths: 96 channels l <= 3 577 -> 450.
      auto build_conv = [&](int kind, auto emit) {
        const bool receiver = kind == CGTP_K_CONV_FWD || (kind == CGTP_K_CONV_DBL_FWD && dtype == CGTP_F32), many = P.paths.size() > kFewPaths;
        std::vector<LaneMap> maps;
        auto add = [&](const LaneMap& m) {
          for (auto& have : maps)
            if (have.cpl == m.cpl) return;
          maps.push_back(m);
        };
        if (!(receiver && many)) add(pick_map(P, kind, 0));
        add(pick_map(P, kind, 1));
        if (kind == CGTP_K_CONV_BWD || kind == CGTP_K_CONV_DBL_BWD) add(pick_map(P, kind, 2));
        Kernel best;
        LaneMap best_map;
        long best_class = -1;
        for (size_t t = 0; t < maps.size(); ++t) {
          P.map[kind] = maps[t];
          P.k[kind] = Kernel();
          try {
            build_worker(kind, emit);
          } catch (const CompileError&) {
            if (best_class < 0 && t + 1 == maps.size()) throw;
            continue;
          }
          const long c = register_class(P.k[kind], !many || kind == CGTP_K_CONV_BWD);
          if (best_class < 0 || c < best_class) {
            best = std::move(P.k[kind]);
            best_map = P.map[kind];
            best_class = c;
          }
          if (device == -1 || best_class == 0) break;
        }
        P.k[kind] = std::move(best);
        P.map[kind] = best_map;
      };
      build_kernel(P, CGTP_K_TP_FWD, [&](Kernel& k) { cgtp::emit_uvu_forward(P, false, k); }, device);
      build_kernel(P, CGTP_K_TP_BWD, [&](Kernel& k) { cgtp::emit_uvu_backward(P, false, k); }, device);
      build_conv(CGTP_K_CONV_FWD, [&](Kernel& k) { cgtp::emit_uvu_forward(P, true, k); });
      build_conv(CGTP_K_CONV_BWD, [&](Kernel& k) { cgtp::emit_uvu_backward(P, true, k); });
      build_conv(CGTP_K_CONV_FWD_ATOMIC, [&](Kernel& k) { cgtp::emit_uvu_atomic(P, false, k); });
      build_kernel(P, CGTP_K_CONV_BWD_ATOMIC, [&](Kernel& k) { cgtp::emit_uvu_atomic(P, true, k); }, device);
      build_kernel(P, CGTP_K_TP_DBL_BWD, [&](Kernel& k) { cgtp::emit_uvu_double_backward(P, k); }, device);
      build_conv(CGTP_K_CONV_DBL_FWD, [&](Kernel& k) { cgtp::emit_uvu_conv_double(P, false, k); });
      build_conv(CGTP_K_CONV_DBL_BWD, [&](Kernel& k) { cgtp::emit_uvu_conv_double(P, true, k); });
      cgtp::emit_fixup(P, P.k_fix);
      build_rows(P, device);
      build_double_rows(P, device);
    } else if (!P.shared_w) {
      cgtp::emit_uvw_ps_forward(P, P.k[CGTP_K_TP_FWD]);
      cgtp::emit_uvw_ps_backward(P, P.k[CGTP_K_TP_BWD]);
      // second-order pass: a forward-like kernel (dL/dgz; kept in the slot of the convolution's forward-like kernel,
      // which a uvw plan does not use) and a backward-like kernel (dL/dx, dL/dy, dL/dW)
      // CGTP_UVWPS_DBL_ONE=1 (default): the backward-like kernel computes dL/dgz as well, from the weight tiles it
      // holds in registers anyway (W and LC are then read once per call instead of twice); 0: two kernels
      const int one = cgtp::env_int("CGTP_UVWPS_DBL_ONE", 1) ? 1 : 0;
      if (!one) cgtp::emit_uvw_ps_double_forward(P, P.k[CGTP_K_CONV_DBL_FWD]);
      {
        // the backward-like kernel lands just above 256 registers for some plans (258 in fp64 on the DiffDock-shaped
        // benchmark): two waves per SIMD are asked of the compiler, and kept only if that costs at most 64 bytes of private memory
        Kernel& kd = P.k[CGTP_K_TP_DBL_BWD];
        kd.sched.occ = device == -1 ? 0 : 2;
        kd.sched.one_kernel = one;
        cgtp::emit_uvw_ps_double_backward(P, kd);
        if (device != -1) {
          cgtp::jit_compile(kd, -2);
          if (kd.scratch > 64) {   // a few spilled words are cheaper than one wave per SIMD
            kd = Kernel();
            kd.sched.occ = 0;
            kd.sched.one_kernel = one;
            cgtp::emit_uvw_ps_double_backward(P, kd);
          }
        }
      }
    } else {
      // forward: the scalars' paths over x, or all over z' if the former needs more private memory (degree 3, 16 -> 16 channels:
      // 1 092 bytes against 600)
      Kernel& kf = P.k[CGTP_K_TP_FWD];
      cgtp::emit_uvw_forward(P, kf);
      if (device != -1) {
        auto compile = [](Kernel& k) {
          try {
            cgtp::jit_compile(k, -2);
          } catch (const std::exception& e) {
            throw CompileError{e.what()};
          }
        };
        compile(kf);
        if (kf.scratch > 0) {
          Kernel other;
          other.sched.x_form = 0;
          cgtp::emit_uvw_forward(P, other);
          compile(other);
          if (other.scratch < kf.scratch) kf = std::move(other);
        }
      }
      try {
        cgtp::emit_uvw_backward(P, P.k[CGTP_K_TP_BWD], P.k_fix);
      } catch (const cgtp::ShapeNotCovered&) {  // multiplicities the backward does not cover: forward-only plan
        P.k[CGTP_K_TP_BWD] = Kernel();          // (any other error of the emitter is a bug and is reported)
        P.k_fix = Kernel();
      }
    }
  } catch (const CompileError& e) {
    return fail(CGTP_ECOMPILE, e.msg);
  } catch (const std::exception& e) {
    return fail(CGTP_EUNSUPPORTED, e.what());
  }
  if (device >= 0) {
    HIP_TRY(hipSetDevice(device));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, device));
    P.num_cu = prop.multiProcessorCount;
    if (std::string(prop.gcnArchName).rfind("gfx950", 0) != 0)
      return fail(CGTP_EUNSUPPORTED, std::string("this library targets gfx950, device is ") + prop.gcnArchName);
  }
  try {
    for (auto& k : P.k) cgtp::jit_compile(k, device);
    cgtp::jit_compile(P.k_fix, device);
  } catch (const std::exception& e) {
    for (auto& k : P.k) cgtp::jit_unload(k);
    cgtp::jit_unload(P.k_fix);
    return fail(CGTP_ECOMPILE, e.what());
  }
  try {
    for (Kernel* k : row_kernels(P)) cgtp::jit_compile(*k, device);
  } catch (const std::exception&) {   // the walks by ranges take their place
    for (Kernel* k : row_kernels(P)) cgtp::jit_unload(*k);
    (void)hipGetLastError();
  }
  if (P.k_row[0][0].fn || P.k_row[1][0].fn || P.k_dbl_row[0].fn) {
    const size_t n = cgtp::kRowWindows * sizeof(*P.row_cnt);
    hipError_t e = hipMalloc((void**)&P.row_cnt, n);
    if (e == hipSuccess) e = hipMemset(P.row_cnt, cgtp::env_int("CGTP_ROW_CNT_FILL", 0), n);   // (tests: counts left behind)
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
      cgtp_plan_destroy(H.release());
      return fail(CGTP_ENOMEM, std::string("counters of the row kernels: ") + hipGetErrorString(e));
    }
  }
  *out = H.release();
  return CGTP_OK;
}

cgtp_status cgtp_plan_destroy(cgtp_plan* plan) {
  if (!plan) return CGTP_OK;
  for (auto& k : plan->P.k) cgtp::jit_unload(k);
  cgtp::jit_unload(plan->P.k_fix);
  for (Kernel* k : row_kernels(plan->P)) cgtp::jit_unload(*k);
  if (plan->P.row_cnt) (void)hipFree(plan->P.row_cnt);
  if (plan->P.ws) (void)hipFree(plan->P.ws);
  delete plan;
  return CGTP_OK;
}

int64_t cgtp_plan_dim(const cgtp_plan* plan, int32_t which) {
  if (!plan) return -1;
  switch (which) {
    case 0: return plan->P.dim_x();
    case 1: return plan->P.dim_y();
    case 2: return plan->P.dim_z();
    case 3: return plan->P.n_w;
    default: return -1;
  }
}

int32_t cgtp_plan_num_paths(const cgtp_plan* plan) { return plan ? (int32_t)plan->P.paths.size() : -1; }

cgtp_status cgtp_plan_get_path(const cgtp_plan* plan, int32_t p, cgtp_path* path, int32_t* l1l2l3, int32_t* nnz,
                               int64_t* w_offset) {
  if (!plan || p < 0 || p >= (int32_t)plan->P.paths.size()) return fail(CGTP_EINVAL, "bad plan or path index");
  const PathInfo& q = plan->P.paths[p];
  if (path) *path = cgtp_path{q.ix, q.iy, q.iz, q.mode, q.coeff};
  if (l1l2l3) {
    l1l2l3[0] = q.l1; l1l2l3[1] = q.l2; l1l2l3[2] = q.l3;
  }
  if (nnz) *nnz = (int32_t)q.nz.size();
  if (w_offset) *w_offset = q.w_off;
  return CGTP_OK;
}

int32_t cgtp_plan_path_nonzeros(const cgtp_plan* plan, int32_t p, int32_t cap, int32_t* i, int32_t* j, int32_t* k,
                                double* v) {
  if (!plan || p < 0 || p >= (int32_t)plan->P.paths.size()) return -1;
  const auto& nz = plan->P.paths[p].nz;
  for (int32_t t = 0; t < (int32_t)nz.size() && t < cap; ++t) {
    if (i) i[t] = nz[t].i;
    if (j) j[t] = nz[t].j;
    if (k) k[t] = nz[t].k;
    if (v) v[t] = nz[t].v;
  }
  return (int32_t)nz.size();
}

int64_t cgtp_plan_flops(const cgtp_plan* plan, int32_t which) {
  if (!plan) return -1;
  int64_t cg = 0, w = 0;
  for (auto& q : plan->P.paths) {
    cg += 2LL * (int64_t)q.nz.size() * q.mul_x;
    w += 2LL * (2 * q.l3 + 1) * (q.mode == CGTP_UVU ? (int64_t)q.mul_x : (int64_t)q.mul_x * q.mul_z);
  }
  if (which == 0) return cg + w;
  // backward: 3x the contraction; the weight part is 1.5x for uvu (g' = w*gz, gW += z'*gz) and 2x for uvw (two GEMMs)
  if (which == 1) return 3 * cg + (plan->P.mode == CGTP_UVU ? (3 * w) / 2 : 2 * w);
  // fused second-order pass.  uvu: 8 FMAs per nonzero and channel.  uvw (per-sample weights), one kernel: z' three times
  // (S = z'(La, y) + z'(x, Lb) and Z = z'(x, y)), dL/dx and dL/dy with two terms each -> 7x the contraction; five dense
  // products (W S, LC Z, S (x) gz, W gz, LC gz) -> 5x the weight part.  The two-kernel variant forms S twice more: 9x.
  if (which == 2) return plan->P.mode == CGTP_UVU ? 8 * cg + 3 * w : (plan->P.k[CGTP_K_TP_DBL_BWD].sched.one_kernel > 0 ? 7 : 9) * cg + 5 * w;
  return -1;
}

const char* cgtp_plan_source(const cgtp_plan* plan, int32_t kernel) {
  if (!plan || kernel < 0 || kernel > 8) return nullptr;
  const std::string& s = plan->P.k[kernel].source;
  return s.empty() ? nullptr : s.c_str();
}

cgtp_status cgtp_plan_kernel_info(const cgtp_plan* plan, int32_t kernel, int32_t info[6]) {
  if (!plan || kernel < 0 || kernel > 8 || !info) return fail(CGTP_EINVAL, "bad argument");
  const Kernel& k = plan->P.k[kernel];
  if (!k.fn && k.vgprs == 0) return fail(CGTP_EUNSUPPORTED, "kernel is neither compiled nor loaded");
  info[0] = k.vgprs; info[1] = k.sgprs; info[2] = k.lds; info[3] = k.scratch; info[4] = k.wg; info[5] = k.blocks_per_cu;
  return CGTP_OK;
}

cgtp_status tp_forward(cgtp_plan* plan, const void* x, const void* y, const void* W, void* z, int64_t B,
                       void* hip_stream) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (B < 0) return fail(CGTP_EINVAL, "negative batch size");
  if (B == 0) return CGTP_OK;
  if (!x || !y || !W || !z) return fail(CGTP_EINVAL, "NULL data pointer");
  if (!aligned16(x) || !aligned16(y) || !aligned16(W) || !aligned16(z)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  Plan& P = plan->P;
  const Kernel& k = P.k[CGTP_K_TP_FWD];
  hipStream_t st = (hipStream_t)hip_stream;
  if (P.mode == CGTP_UVU) {
    const int wpw = k.wg / 64;
    int64_t need = (B + (int64_t)P.map[CGTP_K_TP_FWD].spw * wpw - 1) / ((int64_t)P.map[CGTP_K_TP_FWD].spw * wpw);
    int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT", 8));
    unsigned grid = (unsigned)std::min(need, cap);
    void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&z, (void*)&B};
    return launch(k, grid, args, st);
  }
  if (!P.shared_w) {   // per-sample weights: one wave per sample, grid-stride
    const int wpw = k.wg / 64;
    int64_t need = (B + wpw - 1) / wpw;
    int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT", 8));
    unsigned grid = (unsigned)std::min(need, cap);
    void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&z, (void*)&B};
    return launch(k, grid, args, st);
  }
  // uvw: one workgroup per tile of samples (geometry fixed by the emitter: k.wg threads, tile in k.lds slot)
  // persistent workgroups: the weights are copied to LDS once per workgroup
  // at most one workgroup per 16-sample tile: the tiles of the last, incomplete round of the waves are worked on by
  // a whole workgroup each (for a small batch that is every tile)
  int64_t need = (B + 15) / 16;
  int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu);
  unsigned grid = (unsigned)std::min(need, cap);
  void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&z, (void*)&B};
  return launch(k, grid, args, st);
}

cgtp_status tp_backward(cgtp_plan* plan, const void* x, const void* y, const void* W, const void* gz, void* gx,
                        void* gy, void* gW, int64_t B, void* hip_stream) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (B < 0) return fail(CGTP_EINVAL, "negative batch size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU && P.k[CGTP_K_TP_BWD].source.empty())
    return fail(CGTP_EUNSUPPORTED, "backward of this uvw plan is not supported (needs mul_x, mul_z multiples of 16)");
  if (B == 0 && (P.mode == CGTP_UVU || !P.shared_w)) return CGTP_OK;
  if (B == 0) {   // shared weights: gW is the empty sum; no other buffer is touched
    if (!gW || !aligned16(gW)) return fail(CGTP_EINVAL, "gW must be a 16-byte aligned device pointer");
    HIP_TRY(cgtp::launch_fill_zero(gW, (size_t)P.n_w * P.elt(), (hipStream_t)hip_stream));
    return CGTP_OK;
  }
  if (!x || !y || !W || !gz || !gx || !gy || !gW) return fail(CGTP_EINVAL, "NULL data pointer");
  for (const void* p : {x, y, W, gz, (const void*)gx, (const void*)gy, (const void*)gW})
    if (!aligned16(p)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  const Kernel& k = P.k[CGTP_K_TP_BWD];
  const int wpw = k.wg / 64;
  if (P.mode == CGTP_UVW && !P.shared_w) {   // per-sample weights: gW [B, n_w], one wave per sample
    int64_t need = (B + wpw - 1) / wpw;
    int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT", 8));
    unsigned grid = (unsigned)std::min(need, cap);
    void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&gz, (void*)&gx, (void*)&gy, (void*)&gW, (void*)&B};
    return launch(k, grid, args, (hipStream_t)hip_stream);
  }
  if (P.mode == CGTP_UVW) {
    // shared weights: gW [n_w] is the sum over the batch; per-wave partial sums go through the workspace
    hipStream_t st = (hipStream_t)hip_stream;
    int64_t tile = cgtp::uvw_tile_samples(P);
    unsigned grid = (unsigned)std::min<int64_t>((B + tile - 1) / tile, std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu));
    int64_t nparts = grid;   // one partial gW per workgroup
    cgtp_status s = ensure_ws(P, (size_t)nparts * P.n_w * P.elt());
    if (s != CGTP_OK) return s;
    void* part = P.ws;
    void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&gz, (void*)&gx, (void*)&gy, (void*)&part, (void*)&B};
    s = launch(k, grid, args, st);
    if (s != CGTP_OK) return s;
    int64_t n = P.n_w;
    void* rargs[] = {(void*)&part, (void*)&gW, (void*)&nparts, (void*)&n};
    return launch(P.k_fix, (unsigned)(n / 256), rargs, st);   // one workgroup per 16x16 block (mul_x and mul_z are multiples of 16)
  }
  int64_t need = (B + (int64_t)P.map[CGTP_K_TP_BWD].spw * wpw - 1) / ((int64_t)P.map[CGTP_K_TP_BWD].spw * wpw);
  int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT", 8));
  unsigned grid = (unsigned)std::min(need, cap);
  void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&gz, (void*)&gx, (void*)&gy, (void*)&gW, (void*)&B};
  return launch(k, grid, args, (hipStream_t)hip_stream);
}

cgtp_status tp_double_backward(cgtp_plan* plan, const void* x, const void* y, const void* W, const void* gz,
                               const void* La, const void* Lb, const void* LC, void* Lx, void* Ly, void* LW,
                               void* Lgz, int64_t B, void* hip_stream) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (B < 0) return fail(CGTP_EINVAL, "negative batch size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU && P.shared_w) return fail(CGTP_EUNSUPPORTED, "double backward is not implemented for uvw plans with shared weights");
  if (B == 0) return CGTP_OK;
  if (P.mode != CGTP_UVU) {
    // uvw with per-sample weights: one kernel for all four results (W and LC streamed once), or, for plans created
    // with CGTP_UVWPS_DBL_ONE=0, the split of paper Sec. 3.4 into a forward-like and a backward-like kernel (each
    // streams W and LC); one wave per sample, no workspace
    for (const void* p : {x, y, W, gz, La, Lb, LC, (const void*)Lx, (const void*)Ly, (const void*)LW, (const void*)Lgz}) {
      if (!p) return fail(CGTP_EINVAL, "NULL data pointer");
      if (!aligned16(p)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
    }
    hipStream_t st = (hipStream_t)hip_stream;
    // CGTP_UVWPS_DBL_FUSED=0 (environment) selects the unfused route instead of the fused kernel(s): a second
    // way to the same result, kept for verification
    if (cgtp::env_int("CGTP_UVWPS_DBL_FUSED", 1) == 0) {
      // the seven dispatches of paper Sec. 3.4 as they stand (three forward, four backward calls on
      // permuted operands), sums formed in place; temporaries [B, dim_x + dim_y + dim_z + n_w] in the plan's
      // workspace (the per-sample kernels themselves use none)
      const size_t el = P.elt();
      const size_t nx = round_up((size_t)B * P.dim_x() * el, 256), ny = round_up((size_t)B * P.dim_y() * el, 256),
                   nz = round_up((size_t)B * P.dim_z() * el, 256), nw = round_up((size_t)B * P.n_w * el, 256);
      cgtp_status s = ensure_ws(P, nx + ny + nz + nw);
      if (s != CGTP_OK) return s;
      char* base = (char*)P.ws;
      void *tx = base, *ty = base + nx, *tz = base + nx + ny, *tw = base + nx + ny + nz;
      const bool f64 = P.dtype == CGTP_F64;
      auto add = [&](void* a, const void* b_, int64_t n) -> cgtp_status {
        HIP_TRY(cgtp::launch_add_inplace(a, b_, n, f64, st));
        return CGTP_OK;
      };
#define DBL_TRY(e) do { cgtp_status s_ = (e); if (s_ != CGTP_OK) return s_; } while (0)
      DBL_TRY(tp_backward(plan, La, Lb, W, gz, Lx, Ly, tw, B, hip_stream));     // op1 -> dL/dx, dL/dy
      DBL_TRY(tp_backward(plan, x, y, LC, gz, tx, ty, tw, B, hip_stream));      // op2
      DBL_TRY(add(Lx, tx, B * P.dim_x()));
      DBL_TRY(add(Ly, ty, B * P.dim_y()));
      DBL_TRY(tp_forward(plan, La, y, W, Lgz, B, hip_stream));                  // op3 -> dL/dgz
      DBL_TRY(tp_forward(plan, x, Lb, W, tz, B, hip_stream));                   // op6
      DBL_TRY(add(Lgz, tz, B * P.dim_z()));
      DBL_TRY(tp_forward(plan, x, y, LC, tz, B, hip_stream));                   // op7
      DBL_TRY(add(Lgz, tz, B * P.dim_z()));
      DBL_TRY(tp_backward(plan, La, y, W, gz, tx, ty, LW, B, hip_stream));      // op4 -> dL/dW
      DBL_TRY(tp_backward(plan, x, Lb, W, gz, tx, ty, tw, B, hip_stream));      // op5
      DBL_TRY(add(LW, tw, B * P.n_w));
#undef DBL_TRY
      return CGTP_OK;
    }
    const bool one = P.k[CGTP_K_TP_DBL_BWD].sched.one_kernel > 0;
    for (int which = one ? 1 : 0; which < 2; ++which) {
      const Kernel& kk = P.k[which == 0 ? CGTP_K_CONV_DBL_FWD : CGTP_K_TP_DBL_BWD];
      const int wpw_ = kk.wg / 64;
      int64_t need = (B + wpw_ - 1) / wpw_;
      int64_t cap = std::max<int64_t>(1, (int64_t)kk.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT", 8));
      unsigned grid = (unsigned)std::min(need, cap);
      cgtp_status s_;
      if (which == 0) {
        void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&La, (void*)&Lb, (void*)&LC, (void*)&Lgz, (void*)&B};
        s_ = launch(kk, grid, args, st);
      } else {
        void* args[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&gz, (void*)&La, (void*)&Lb, (void*)&LC, (void*)&Lx, (void*)&Ly, (void*)&LW, (void*)&B};
        void* args1[] = {(void*)&x, (void*)&y, (void*)&W, (void*)&gz, (void*)&La, (void*)&Lb, (void*)&LC, (void*)&Lx, (void*)&Ly, (void*)&LW, (void*)&Lgz, (void*)&B};
        s_ = launch(kk, grid, one ? args1 : args, st);
      }
      if (s_ != CGTP_OK) return s_;
    }
    return CGTP_OK;
  }
  for (const void* p : {x, y, W, gz, La, Lb, LC, (const void*)Lx, (const void*)Ly, (const void*)LW, (const void*)Lgz}) {
    if (!p) return fail(CGTP_EINVAL, "NULL data pointer");
    if (!aligned16(p)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  }
  const Kernel& k = P.k[CGTP_K_TP_DBL_BWD];
  const int wpw = k.wg / 64;
  const int64_t per_wg = (int64_t)P.map[CGTP_K_TP_DBL_BWD].spw * wpw;
  int64_t need = (B + per_wg - 1) / per_wg;
  int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT_DBL", 2));
  unsigned grid = (unsigned)std::min(need, cap);
  void* args[] = {(void*)&x,  (void*)&y,  (void*)&W,  (void*)&gz,  (void*)&La,  (void*)&Lb,
                  (void*)&LC, (void*)&Lx, (void*)&Ly, (void*)&LW, (void*)&Lgz, (void*)&B};
  return launch(k, grid, args, (hipStream_t)hip_stream);
}

cgtp_status conv_forward(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges, void* z_nodes,
                         int64_t V, int64_t E, const int64_t* row_ptr, const int64_t* col, void* hip_stream) {
  return conv_forward_perm(plan, x_nodes, y_edges, W_edges, z_nodes, V, E, row_ptr, col, nullptr, hip_stream);
}

}  // extern "C"

namespace {
// conv_forward / conv_forward_perm / conv_forward_static.  use_static: the side buffer of split rows is the library's
// static device array instead of the plan's workspace (nothing is allocated).
cgtp_status conv_forward_impl(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                              void* z_nodes, int64_t V, int64_t E, const int64_t* row_ptr, const int64_t* col,
                              const int64_t* edge_perm, void* hip_stream, bool use_static) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (V < 0 || E < 0) return fail(CGTP_EINVAL, "negative size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "convolution is implemented for uvu plans only");
  if (V == 0) return E == 0 ? CGTP_OK : fail(CGTP_EINVAL, "edges without nodes");
  if (!z_nodes || !row_ptr) return fail(CGTP_EINVAL, "NULL data pointer");
  hipStream_t st = (hipStream_t)hip_stream;
  if (!aligned16(z_nodes)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  if (E == 0) {
    HIP_TRY(cgtp::launch_fill_zero(z_nodes, (size_t)V * P.dim_z() * P.elt(), st));
    return CGTP_OK;
  }
  if (!x_nodes || !y_edges || !W_edges || !col) return fail(CGTP_EINVAL, "NULL data pointer");
  if (!aligned16(x_nodes) || !aligned16(y_edges) || !aligned16(W_edges)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  const Kernel& k = P.k[CGTP_K_CONV_FWD];
  if (!k.fn) return fail(CGTP_EUNSUPPORTED, "kernel is not loaded (plan created without a device?)");
  const int spw = P.map[CGTP_K_CONV_FWD].spw;   // edge-range workers per wave
  const Kernel* rows = conv_by_rows(P, false, V, E);
  const int lg = rows ? row_lg(*rows, spw, E, P.dim_z() * (int64_t)P.elt()) : 0;
  int64_t nchunk = rows ? cgtp::row_windows(lg, E) : conv_ranges(P, k, spw, E);
  void* part = nullptr;
  cgtp_status s = CGTP_OK;
  if (use_static) {
    int cur = -1;
    HIP_TRY(hipGetDevice(&cur));
    if (cur != P.device) return fail(CGTP_EINVAL, "the plan's device is not the current device");
    size_t cap = 0;
    hipError_t e = cgtp::static_scratch(&part, &cap);
    if (e != hipSuccess) return fail(CGTP_ERUNTIME, std::string("static scratch: ") + hipGetErrorString(e));
    // the limit of this entry point is a rule on the plan and E, whatever number of ranges suits a small graph
    const int64_t ranges = std::min(E, most_ranges(P, k, spw));
    const size_t need = (size_t)ranges * 2 * P.dim_z() * P.elt();
    if (need > cap || (size_t)nchunk * 2 * P.dim_z() * P.elt() > cap)
      return fail(CGTP_EINVAL, "conv_forward_static: this problem needs " + std::to_string(need) + " bytes of scratch for " +
                                   std::to_string(ranges) + " edge ranges, the static buffer holds " + std::to_string(cap) +
                                   "; use conv_forward");
  } else {
    s = ensure_ws(P, piece_bytes(P, false, E));
    if (s != CGTP_OK) return s;
    part = P.ws;
  }
  if (rows) {
    ++P.row_call;
    void* args[] = {(void*)&x_nodes, (void*)&y_edges, (void*)&W_edges,   (void*)&z_nodes, (void*)&row_ptr, (void*)&col,
                    (void*)&V,       (void*)&part,    (void*)&P.row_cnt, (void*)&P.row_call, (void*)&lg, (void*)&edge_perm};
    return launch(*rows, (unsigned)(V + nchunk - 1), args, st);
  }
  const int wpw = k.wg / 64;
  unsigned grid = (unsigned)((nchunk + (int64_t)wpw * spw - 1) / ((int64_t)wpw * spw));
  void* args[] = {(void*)&x_nodes, (void*)&y_edges, (void*)&W_edges, (void*)&z_nodes, (void*)&row_ptr,  (void*)&col,
                  (void*)&V,       (void*)&E,       (void*)&part,    (void*)&nchunk,  (void*)&edge_perm};
  s = launch(k, grid, args, st);
  if (s != CGTP_OK) return s;
  return launch_fixup(P, z_nodes, part, row_ptr, V, E, nchunk, P.dim_z(), st);
}
}  // namespace

extern "C" {

cgtp_status conv_forward_perm(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                              void* z_nodes, int64_t V, int64_t E, const int64_t* row_ptr, const int64_t* col,
                              const int64_t* edge_perm, void* hip_stream) {
  return conv_forward_impl(plan, x_nodes, y_edges, W_edges, z_nodes, V, E, row_ptr, col, edge_perm, hip_stream, false);
}

cgtp_status conv_forward_static(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                                void* z_nodes, int64_t V, int64_t E, const int64_t* row_ptr, const int64_t* col,
                                void* hip_stream) {
  return conv_forward_impl(plan, x_nodes, y_edges, W_edges, z_nodes, V, E, row_ptr, col, nullptr, hip_stream, true);
}

cgtp_status conv_backward(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                          const void* gz_nodes, void* gx_nodes, void* gy_edges, void* gW_edges, int64_t V, int64_t E,
                          const int64_t* row_ptr, const int64_t* col, const int64_t* t_row_ptr, const int64_t* t_perm,
                          void* hip_stream) {
  return conv_backward_perm(plan, x_nodes, y_edges, W_edges, gz_nodes, gx_nodes, gy_edges, gW_edges, V, E, row_ptr, col,
                            t_row_ptr, t_perm, nullptr, hip_stream);
}

cgtp_status conv_backward_perm(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                               const void* gz_nodes, void* gx_nodes, void* gy_edges, void* gW_edges, int64_t V,
                               int64_t E, const int64_t* row_ptr, const int64_t* col, const int64_t* t_row_ptr,
                               const int64_t* t_perm, const int64_t* edge_perm, void* hip_stream) {
  (void)col;
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (V < 0 || E < 0) return fail(CGTP_EINVAL, "negative size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "convolution is implemented for uvu plans only");
  if (V == 0) return E == 0 ? CGTP_OK : fail(CGTP_EINVAL, "edges without nodes");
  if (!gx_nodes) return fail(CGTP_EINVAL, "NULL data pointer");
  hipStream_t st = (hipStream_t)hip_stream;
  if (E == 0) {
    HIP_TRY(cgtp::launch_fill_zero(gx_nodes, (size_t)V * P.dim_x() * P.elt(), st));
    return CGTP_OK;
  }
  if (!x_nodes || !y_edges || !W_edges || !gz_nodes || !gy_edges || !gW_edges || !row_ptr || !t_row_ptr || !t_perm)
    return fail(CGTP_EINVAL, "NULL data pointer");
  for (const void* p : {x_nodes, y_edges, W_edges, gz_nodes, (const void*)gx_nodes, (const void*)gy_edges, (const void*)gW_edges})
    if (!aligned16(p)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  const Kernel& k = P.k[CGTP_K_CONV_BWD];
  if (!k.fn) return fail(CGTP_EUNSUPPORTED, "kernel is not loaded (plan created without a device?)");
  const int spw = P.map[CGTP_K_CONV_BWD].spw;   // edge-range workers per wave
  // the same workspace whichever kernel walks the graph
  const size_t part_bytes = round_up(piece_bytes(P, true, E), 256), recv_bytes = round_up((size_t)E * 8, 256);
  // one scratch row for the gy / gW words of the pipelined kernel's phantom edge (odd edge ranges)
  const size_t dummy_bytes = (round_up((size_t)P.dim_y(), 64) + (size_t)P.n_w) * P.elt();
  cgtp_status s = ensure_ws(P, part_bytes + recv_bytes + dummy_bytes);
  if (s != CGTP_OK) return s;
  void* part = P.ws;
  int64_t* t_recv = (int64_t*)((char*)P.ws + part_bytes);
  void* dummy = (char*)P.ws + part_bytes + recv_bytes;
  if (const Kernel* rows = conv_by_rows(P, true, V, E)) {
    const int lg = row_lg(*rows, spw, E, P.dim_x() * (int64_t)P.elt());
    if (V > cgtp::kConvRowLookup || E > INT32_MAX) HIP_TRY(cgtp::launch_recv_of_tperm(row_ptr, t_perm, V, E, t_recv, st));
    else t_recv = nullptr;   // the kernel looks them up (2 000 nodes: 30 us either way)
    ++P.row_call;
    void* args[] = {(void*)&x_nodes,  (void*)&y_edges,   (void*)&W_edges, (void*)&gz_nodes,  (void*)&gx_nodes, (void*)&gy_edges,
                    (void*)&gW_edges, (void*)&t_row_ptr, (void*)&t_perm,  (void*)&row_ptr,   (void*)&t_recv,   (void*)&V,
                    (void*)&part,     (void*)&P.row_cnt, (void*)&P.row_call, (void*)&lg,     (void*)&edge_perm};
    return launch(*rows, (unsigned)(V + cgtp::row_windows(lg, E) - 1), args, st);
  }
  int64_t nchunk = conv_ranges(P, k, spw, E);
  HIP_TRY(cgtp::launch_recv_of_tperm(row_ptr, t_perm, V, E, t_recv, st));
  const int wpw = k.wg / 64;
  unsigned grid = (unsigned)((nchunk + (int64_t)wpw * spw - 1) / ((int64_t)wpw * spw));
  void* args[] = {(void*)&x_nodes,  (void*)&y_edges,  (void*)&W_edges, (void*)&gz_nodes, (void*)&gx_nodes,
                  (void*)&gy_edges, (void*)&gW_edges, (void*)&t_row_ptr, (void*)&t_perm, (void*)&t_recv,
                  (void*)&V,        (void*)&E,        (void*)&part,    (void*)&nchunk,   (void*)&edge_perm,
                  (void*)&dummy};
  s = launch(k, grid, args, st);
  if (s != CGTP_OK) return s;
  return launch_fixup(P, gx_nodes, part, t_row_ptr, V, E, nchunk, P.dim_x(), st);
}

cgtp_status conv_double_backward_ws(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                                    const void* gz_nodes, const void* La_nodes, const void* Lb_edges,
                                    const void* LC_edges, void* Lx_nodes, void* Ly_edges, void* LW_edges,
                                    void* Lgz_nodes, int64_t V, int64_t E, const int64_t* row_ptr, const int64_t* col,
                                    const int64_t* t_row_ptr, const int64_t* t_perm, void* scratch, size_t scratch_bytes,
                                    void* hip_stream) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (V < 0 || E < 0) return fail(CGTP_EINVAL, "negative size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "convolution is implemented for uvu plans only");
  if (scratch && ((uintptr_t)scratch & 255)) return fail(CGTP_EINVAL, "scratch must be 256-byte aligned");
  if (V == 0) return E == 0 ? CGTP_OK : fail(CGTP_EINVAL, "edges without nodes");
  if (!Lx_nodes || !Lgz_nodes) return fail(CGTP_EINVAL, "NULL data pointer");
  hipStream_t st = (hipStream_t)hip_stream;
  if (E == 0) {
    HIP_TRY(cgtp::launch_fill_zero(Lx_nodes, (size_t)V * P.dim_x() * P.elt(), st));
    HIP_TRY(cgtp::launch_fill_zero(Lgz_nodes, (size_t)V * P.dim_z() * P.elt(), st));
    return CGTP_OK;
  }
  for (const void* p : {x_nodes, y_edges, W_edges, gz_nodes, La_nodes, Lb_edges, LC_edges, (const void*)Lx_nodes,
                        (const void*)Ly_edges, (const void*)LW_edges, (const void*)Lgz_nodes}) {
    if (!p) return fail(CGTP_EINVAL, "NULL data pointer");
    if (!aligned16(p)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  }
  if (!row_ptr || !col || !t_row_ptr || !t_perm) return fail(CGTP_EINVAL, "NULL graph pointer");
  const Kernel& kf = P.k[CGTP_K_CONV_DBL_FWD];
  const Kernel& kb = P.k[CGTP_K_CONV_DBL_BWD];
  if (!kf.fn || !kb.fn) return fail(CGTP_EUNSUPPORTED, "kernel is not loaded (plan created without a device?)");
  const DoubleWalk d = double_walk(P, V, E);
  cgtp_status s = ensure_ws(P, d.ws);
  if (s != CGTP_OK) return s;
  const bool fits = d.rows && d.one <= d.ws;
  if (scratch && d.rows && !fits && scratch_bytes < d.one)
    return fail(CGTP_EINVAL, "scratch of " + std::to_string(scratch_bytes) + " bytes, " + std::to_string(d.one) + " needed");
  if (fits || (scratch && d.rows)) {
    ++P.row_call;
    void *edge_rows = fits ? P.ws : scratch, *pieces = (char*)edge_rows + d.row_bytes;
    void* args[] = {(void*)&x_nodes,   (void*)&y_edges,  (void*)&W_edges, (void*)&gz_nodes,  (void*)&La_nodes,  (void*)&Lb_edges,
                    (void*)&LC_edges,  (void*)&edge_rows, (void*)&Ly_edges, (void*)&LW_edges, (void*)&Lgz_nodes, (void*)&row_ptr,
                    (void*)&col,       (void*)&V,        (void*)&pieces,  (void*)&P.row_cnt, (void*)&P.row_call, (void*)&d.lg};
    s = launch(*d.rows, (unsigned)(V + cgtp::row_windows(d.lg, E) - 1), args, st);
    if (s != CGTP_OK) return s;
    ++P.row_call;
    void* sum_args[] = {(void*)&edge_rows, (void*)&Lx_nodes, (void*)&t_row_ptr, (void*)&t_perm,
                        (void*)&V,         (void*)&pieces,   (void*)&P.row_cnt, (void*)&P.row_call, (void*)&d.lg2};
    return launch(P.k_row_sums, (unsigned)(V + cgtp::row_windows(d.lg2, E) - 1), sum_args, st);
  }
  const int spwf = P.map[CGTP_K_CONV_DBL_FWD].spw, spwb = P.map[CGTP_K_CONV_DBL_BWD].spw;
  const int64_t nf = d.nf, nb = d.nb;
  void* part = P.ws;
  {
    const int wpw = kf.wg / 64;
    unsigned grid = (unsigned)((nf + (int64_t)wpw * spwf - 1) / ((int64_t)wpw * spwf));
    void* args[] = {(void*)&x_nodes,   (void*)&y_edges, (void*)&W_edges, (void*)&La_nodes, (void*)&Lb_edges, (void*)&LC_edges,
                    (void*)&Lgz_nodes, (void*)&row_ptr, (void*)&col,     (void*)&V,        (void*)&E,        (void*)&part,
                    (void*)&nf};
    s = launch(kf, grid, args, st);
    if (s != CGTP_OK) return s;
    s = launch_fixup(P, Lgz_nodes, part, row_ptr, V, E, nf, P.dim_z(), st);
    if (s != CGTP_OK) return s;
  }
  int64_t* t_recv = (int64_t*)((char*)P.ws + d.part_b);
  HIP_TRY(cgtp::launch_recv_of_tperm(row_ptr, t_perm, V, E, t_recv, st));
  {
    const int wpw = kb.wg / 64;
    unsigned grid = (unsigned)((nb + (int64_t)wpw * spwb - 1) / ((int64_t)wpw * spwb));
    void* args[] = {(void*)&x_nodes,  (void*)&y_edges,  (void*)&W_edges,  (void*)&gz_nodes, (void*)&La_nodes, (void*)&Lb_edges,
                    (void*)&LC_edges, (void*)&Lx_nodes, (void*)&Ly_edges, (void*)&LW_edges, (void*)&t_row_ptr, (void*)&t_perm,
                    (void*)&t_recv,   (void*)&V,        (void*)&E,        (void*)&part,     (void*)&nb};
    s = launch(kb, grid, args, st);
    if (s != CGTP_OK) return s;
    return launch_fixup(P, Lx_nodes, part, t_row_ptr, V, E, nb, P.dim_x(), st);
  }
}

cgtp_status conv_double_backward(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                                 const void* gz_nodes, const void* La_nodes, const void* Lb_edges,
                                 const void* LC_edges, void* Lx_nodes, void* Ly_edges, void* LW_edges,
                                 void* Lgz_nodes, int64_t V, int64_t E, const int64_t* row_ptr, const int64_t* col,
                                 const int64_t* t_row_ptr, const int64_t* t_perm, void* hip_stream) {
  return conv_double_backward_ws(plan, x_nodes, y_edges, W_edges, gz_nodes, La_nodes, Lb_edges, LC_edges, Lx_nodes, Ly_edges, LW_edges,
                                 Lgz_nodes, V, E, row_ptr, col, t_row_ptr, t_perm, nullptr, 0, hip_stream);
}

const char* cgtp_plan_conv_kernel(const cgtp_plan* plan, int32_t kernel, int64_t V, int64_t E) {
  if (!plan || plan->P.mode != CGTP_UVU || V <= 0 || E <= 0) return nullptr;
  if (kernel != CGTP_K_CONV_FWD && kernel != CGTP_K_CONV_BWD && kernel != CGTP_K_CONV_DBL_BWD) return nullptr;
  const Plan& P = plan->P;
  if (!P.k[kernel].fn) return nullptr;
  const Kernel* rows = kernel == CGTP_K_CONV_DBL_BWD ? double_walk(P, V, E).rows : conv_by_rows(P, kernel == CGTP_K_CONV_BWD, V, E);
  return rows ? rows->name.c_str() : P.k[kernel].name.c_str();
}

size_t cgtp_conv_double_workspace_bytes(const cgtp_plan* plan, int64_t V, int64_t E) {
  if (!plan || plan->P.mode != CGTP_UVU || V <= 0 || E <= 0 || !plan->P.k[CGTP_K_CONV_DBL_BWD].fn) return 0;
  const DoubleWalk d = double_walk(plan->P, V, E);
  return d.rows && d.one > d.ws ? d.one : 0;
}

cgtp_status conv_forward_atomic(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                                void* z_nodes, int64_t V, int64_t E, const int64_t* recv, const int64_t* send,
                                void* hip_stream) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (V < 0 || E < 0) return fail(CGTP_EINVAL, "negative size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "convolution is implemented for uvu plans only");
  if (V == 0) return E == 0 ? CGTP_OK : fail(CGTP_EINVAL, "edges without nodes");
  if (!z_nodes || !aligned16(z_nodes)) return fail(CGTP_EINVAL, "z_nodes must be a 16-byte aligned device pointer");
  hipStream_t st = (hipStream_t)hip_stream;
  HIP_TRY(cgtp::launch_fill_zero(z_nodes, (size_t)V * P.dim_z() * P.elt(), st));
  if (E == 0) return CGTP_OK;
  if (!x_nodes || !y_edges || !W_edges || !recv || !send) return fail(CGTP_EINVAL, "NULL data pointer");
  if (!aligned16(x_nodes) || !aligned16(y_edges) || !aligned16(W_edges)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  const Kernel& k = P.k[CGTP_K_CONV_FWD_ATOMIC];
  const int wpw = k.wg / 64;
  const int spw = P.map[CGTP_K_CONV_FWD_ATOMIC].spw;   // edge-range workers per wave
  int64_t nchunk = conv_ranges(P, k, spw, E);
  unsigned grid = (unsigned)((nchunk + (int64_t)wpw * spw - 1) / ((int64_t)wpw * spw));
  const int64_t* no_perm = nullptr;
  void* args[] = {(void*)&x_nodes, (void*)&y_edges, (void*)&W_edges, (void*)&z_nodes, (void*)&recv,
                  (void*)&send,    (void*)&E,       (void*)&nchunk,  (void*)&no_perm};
  return launch(k, grid, args, st);
}

cgtp_status conv_backward_atomic(cgtp_plan* plan, const void* x_nodes, const void* y_edges, const void* W_edges,
                                 const void* gz_nodes, void* gx_nodes, void* gy_edges, void* gW_edges, int64_t V,
                                 int64_t E, const int64_t* recv, const int64_t* send, void* hip_stream) {
  if (!plan) return fail(CGTP_EINVAL, "plan is NULL");
  if (V < 0 || E < 0) return fail(CGTP_EINVAL, "negative size");
  Plan& P = plan->P;
  if (P.mode != CGTP_UVU) return fail(CGTP_EUNSUPPORTED, "convolution is implemented for uvu plans only");
  if (V == 0) return E == 0 ? CGTP_OK : fail(CGTP_EINVAL, "edges without nodes");
  if (!gx_nodes || !aligned16(gx_nodes)) return fail(CGTP_EINVAL, "gx_nodes must be a 16-byte aligned device pointer");
  hipStream_t st = (hipStream_t)hip_stream;
  HIP_TRY(cgtp::launch_fill_zero(gx_nodes, (size_t)V * P.dim_x() * P.elt(), st));
  if (E == 0) return CGTP_OK;
  if (!x_nodes || !y_edges || !W_edges || !gz_nodes || !gy_edges || !gW_edges || !recv || !send)
    return fail(CGTP_EINVAL, "NULL data pointer");
  for (const void* p : {x_nodes, y_edges, W_edges, gz_nodes, (const void*)gy_edges, (const void*)gW_edges})
    if (!aligned16(p)) return fail(CGTP_EINVAL, "data pointers must be 16-byte aligned");
  const Kernel& k = P.k[CGTP_K_CONV_BWD_ATOMIC];
  const int wpw = k.wg / 64;
  const int spw = P.map[CGTP_K_CONV_BWD_ATOMIC].spw;
  int64_t need = (E + (int64_t)spw * wpw - 1) / ((int64_t)spw * wpw);
  int64_t cap = std::max<int64_t>(1, (int64_t)k.blocks_per_cu * P.num_cu * cgtp::env_int("CGTP_GRID_MULT", 8));
  void* args[] = {(void*)&x_nodes,  (void*)&y_edges,  (void*)&W_edges, (void*)&gz_nodes, (void*)&gx_nodes,
                  (void*)&gy_edges, (void*)&gW_edges, (void*)&recv,    (void*)&send,     (void*)&E};
  return launch(k, (unsigned)std::min(need, cap), args, st);
}

size_t cgtp_csr_workspace_bytes(int64_t E, int64_t V) {
  size_t bytes = 0;
  if (E < 0 || V < 0 || cgtp::csr_workspace_bytes(E, V, &bytes) != hipSuccess) return 0;
  return bytes;
}

cgtp_status cgtp_csr_from_coo_async(const int64_t* recv, const int64_t* send, int64_t E, int64_t V, int64_t* row_ptr,
                                    int64_t* col, int64_t* perm, int64_t* t_row_ptr, int64_t* t_perm, void* workspace,
                                    size_t workspace_bytes, int32_t* bad_flag, void* hip_stream) {
  if (E < 0 || V < 0) return fail(CGTP_EINVAL, "negative size");
  if (!row_ptr) return fail(CGTP_EINVAL, "NULL output pointer");
  if ((t_row_ptr == nullptr) != (t_perm == nullptr) && E > 0) return fail(CGTP_EINVAL, "t_row_ptr and t_perm must both be given or both be NULL");
  if (E > 0 && (!recv || !send || !col || !perm)) return fail(CGTP_EINVAL, "NULL pointer");
  if (E > 0 && V == 0) return fail(CGTP_EINVAL, "edges without nodes");
  if (E > 0) {
    const size_t need = cgtp_csr_workspace_bytes(E, V);
    if (!workspace || workspace_bytes < need)
      return fail(CGTP_EINVAL, "workspace too small: " + std::to_string(need) + " bytes needed (cgtp_csr_workspace_bytes)");
  }
  hipError_t e = cgtp::csr_from_coo_async(recv, send, E, V, row_ptr, col, perm, t_row_ptr, t_perm, workspace, workspace_bytes,
                                          (int*)bad_flag, (hipStream_t)hip_stream);
  if (e != hipSuccess) return fail(CGTP_ERUNTIME, std::string("csr_from_coo: ") + hipGetErrorString(e));
  return CGTP_OK;
}

cgtp_status cgtp_csr_from_coo(const int64_t* recv, const int64_t* send, int64_t E, int64_t V, int64_t* row_ptr,
                              int64_t* col, int64_t* perm, int64_t* t_row_ptr, int64_t* t_perm, void* hip_stream) {
  if (E < 0 || V < 0) return fail(CGTP_EINVAL, "negative size");
  if (!row_ptr || !t_row_ptr) return fail(CGTP_EINVAL, "NULL output pointer");
  if (E > 0 && (!recv || !send || !col || !perm || !t_perm)) return fail(CGTP_EINVAL, "NULL pointer");
  if (E > 0 && V == 0) return fail(CGTP_EINVAL, "edges without nodes");
  // scratch owned by the library, one buffer per (device, stream), grown on demand and kept until the process ends:
  // a call allocates only when a larger graph than any before arrives on that stream
  struct Scratch {
    void* p = nullptr;
    size_t bytes = 0;
  };
  static std::mutex mu;
  static std::map<std::pair<int, void*>, Scratch> pool;
  int device = 0;
  HIP_TRY(hipGetDevice(&device));
  const size_t need = cgtp_csr_workspace_bytes(E, V) + 256;   // + the range-check flag
  void* ws = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    Scratch& sc = pool[{device, hip_stream}];
    if (sc.bytes < need) {
      if (sc.p) {
        HIP_TRY(hipStreamSynchronize((hipStream_t)hip_stream));
        HIP_TRY(hipFree(sc.p));
        sc = Scratch();
      }
      if (hipMalloc(&sc.p, need) != hipSuccess) {
        sc = Scratch();
        return fail(CGTP_ENOMEM, "scratch allocation of " + std::to_string(need) + " bytes failed");
      }
      sc.bytes = need;
    }
    ws = sc.p;
  }
  // the one synchronisation of this call: the range check is part of its return value.  The kernels write it into a
  // page of pinned host memory (a copy of four bytes from the device costs 8 us of the call); callers beyond the
  // page's slots copy it.
  HostFlags& hf = host_flags();
  const int slot = hf.take();
  int32_t* flag = slot >= 0 ? hf.flags + slot * 16 : (int32_t*)ws;
  if (slot >= 0) __atomic_store_n(flag, 0, __ATOMIC_RELEASE);
  cgtp_status s = cgtp_csr_from_coo_async(recv, send, E, V, row_ptr, col, perm, t_row_ptr, t_perm, (char*)ws + 256, need - 256,
                                          flag, hip_stream);
  int bad = 0;
  hipError_t e = hipSuccess;
  if (s == CGTP_OK && slot < 0) e = hipMemcpyAsync(&bad, flag, sizeof(int), hipMemcpyDeviceToHost, (hipStream_t)hip_stream);
  const hipError_t waited = hipStreamSynchronize((hipStream_t)hip_stream);   // also after a failed launch: earlier ones may still write the slot
  if (slot >= 0) {
    bad = __atomic_load_n(flag, __ATOMIC_ACQUIRE);
    if (waited == hipSuccess) hf.give(slot);
  }
  if (s != CGTP_OK) return s;
  HIP_TRY(e);
  HIP_TRY(waited);
  if (bad) return fail(CGTP_EINVAL, "edge index outside [0, V)");
  return CGTP_OK;
}

}  // extern "C"
