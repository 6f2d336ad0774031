// tre.hip - MI355X (gfx950) replay of Token Service Share (TSS) evaluation and
// TSS-guided receiver/donor rebalancing, behind the C ABI of include/tre.h.
//
// Paper: "Cross-Model Autoscaling for Shared LLM Serving" (TRE): Eq. (1) TSS,
// smoothing, Eq. (2) normalisation and the three regions (Section "Smoothing,
// Normalization, and Calibration"), dual-speed control and Eq. (3) (Section
// "Dual-Speed Control"), bounded pairwise transfer (Section "Bounded Pairwise
// Transfer").
//
// Kernels
//   tss_stream  one workgroup (4 waves) per trace, one barrier per tile of
//               rows. Every thread loads (per-trace buffer resources, the
//               next tile in flight while the current one is tallied) and
//               tallies its rows into an LDS ring of (window, model) cells
//               with one packed 64-bit LDS atomic per row (two for an
//               ADMIT row); completed
//               windows are then evaluated one cell per thread (carry scan,
//               in-window integrals, Eq. (1) in fp64) and one wave per step
//               runs the smoothing chain over the previous chunk.
//   seg_net, tss_seg, chain_smooth
//               the same with few traces: the windows of a trace in segments,
//               a workgroup each, then one chain per trace.
//   rebalance_ordered
//               one workgroup per scenario: three waves prepare the order in
//               which each tick tries receivers and donors, one decides.
//   rebalance   with many scenarios, one wave per scenario, lane = model: Eq. (2), regions,
//               cadence and the greedy receiver/donor moves, with ballots
//               as candidate sets and DPP wave folds for argmin / argmax
//               (lowest index on ties), so every decision is a scalar.
//   validate    checks the event columns once, at load time.
#include <hip/hip_runtime.h>

#include <limits.h>
#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "tre.h"
#include "tre_internal.h"

#pragma clang fp contract(off)

using tre_internal::check_device;
using tre_internal::fail;
using tre_internal::LaunchTimer;

// ------------------------------------------------------------------ errors
static thread_local std::string g_err;

int tre_internal::fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

extern "C" const char* tre_last_error(void) { return g_err.c_str(); }

// ------------------------------------------------------------------ handle

// ------------------------------------------------------------ constants
constexpr int kStreamWaves = 4;            // tss_stream workgroup (waves) with many traces
constexpr int kEvalThreads = 256;          // threads that evaluate a step's cells (one cell each)
constexpr int kStreamEPT = 4;              // rows per lane per tile
constexpr int kRingBytes = 17 * 1024;      // LDS budget of the tally ring
constexpr uint32_t kNoDefer = 0xFFFFFFFFu;

typedef long long v2i64 __attribute__((ext_vector_type(2)));
typedef unsigned int v4u32 __attribute__((ext_vector_type(4)));
typedef unsigned int v2u32 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------- tss_stream
struct StreamParams {
  const int64_t* ts;
  const uint8_t* model;
  const uint8_t* type;
  const uint16_t* tokens;
  const int64_t* off;
  int64_t n_rows;
  const tre_profile* prof;
  int64_t window_ms;
  uint32_t magic;   // floor(2^32 / window_ms), 2^32-1 for a 1 ms window
  int32_t n_windows;
  int32_t M;
  uint32_t wcap;    // ring windows, power of two
  double inv2_window;  // 1 / (2 window_ms), rounded to nearest
  int32_t chunk;    // windows evaluated per step (cells <= threads)
  int32_t fast_w;   // fast period in windows
  int32_t slow_w;   // slow period in windows
  uint32_t magic_fast;  // floor(2^32 / fast_w), 2^32 - 1 for 1
  uint32_t magic_slow;
  int32_t n_ticks;
  uint32_t* prefill;
  uint32_t* decode;
  int64_t* a_int;
  int64_t* w_int;
  double* tss64;
  float* tss32;
  uint8_t* flags;
  double* snap;     // [trace][tick][M]: S, or +inf when idle / not initialised
  // the kStage instantiation: stage-aware shares per cell (tre_eval_stage)
  double* stage64;  // [trace][w][M][2]: prefill, decode
  float* stage32;
  uint8_t* sflags;  // TRE_STAGE_*
  // the control replay streamed with its trace (tre_sweep without the
  // actuation model, for traces that carry exactly one scenario)
  const tre_scenario* sc;
  const uint32_t* sc_count;  // [trace] scenarios on the trace, or NULL
  const uint32_t* sc_first;  // [trace] the scenario when the count is 1
  int32_t ctl_one;           // one trace with one scenario: replayed without the map above
  int32_t budget;
  tre_move* moves;
  uint32_t move_cap;
  uint32_t* n_moves;
  int32_t* r_final;
  int64_t* r_windows;
  // the segmented path (few traces): a workgroup per (trace, segment of
  // seg_w windows), raw ratios to memory for chain_smooth
  int32_t nseg, seg_w;
  const int32_t* seg_row;              // [trace][nseg + 1] first row of each segment, from the trace's first
  const unsigned long long* seg_net;   // [trace][nseg][M] net changes (pack_net)
  double* raw;                         // [trace][column][window], -1 marks an idle window
  uint32_t* first;                     // [trace][column] first window that is not idle
};

// quotient and remainder of rel / window_ms for any 32-bit rel: the
// multiply-high by floor(2^32/window) undershoots by at most one
__device__ __forceinline__ void div_window(uint32_t rel, uint32_t magic, uint32_t win, uint32_t& q,
                                           uint32_t& r) {
  q = __umulhi(rel, magic);
  r = rel - q * win;
  if (r >= win) {
    q += 1;
    r -= win;
  }
}

// One producer lane's share of a tile: kEPT consecutive rows.
template <int kEPT>
struct Slice {
  long long ts[kEPT];
  uint32_t mw[kEPT / 4];  // model bytes, 4 per word
  uint32_t tw[kEPT / 4];  // type bytes
  uint32_t kw[kEPT / 2];  // tokens, 2 per word
};

// Buffer resources over one trace's rows of each column, from its first
// kEPT-aligned row; a load past the range reads zeros (no fault), so tile
// loads need no bounds branches and never touch another trace's rows
// beyond the 16-byte rounding of the range.
struct TraceRsrc {
  __amdgpu_buffer_rsrc_t ts, model, type, tokens;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, long long bytes) {
  const long long n = (bytes + 15) & ~15ll;  // columns are readable 16 bytes past the last row
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)n, 0x00020000);
}

template <int kEPT>
__device__ __forceinline__ void load_slice(Slice<kEPT>& s, const TraceRsrc& rs, int r0) {
  // r0: first row of the lane's slice, relative to the resources' base row
#pragma unroll
  for (int j = 0; j < kEPT / 2; ++j) {
    const v4u32 v = __builtin_bit_cast(
        v4u32, __builtin_amdgcn_raw_buffer_load_b128(rs.ts, r0 * 8 + 16 * j, 0, 0));
    s.ts[2 * j] = (long long)(((unsigned long long)v.y << 32) | v.x);
    s.ts[2 * j + 1] = (long long)(((unsigned long long)v.w << 32) | v.z);
  }
  if constexpr (kEPT == 4) {
    s.mw[0] = __builtin_amdgcn_raw_buffer_load_b32(rs.model, r0, 0, 0);
    s.tw[0] = __builtin_amdgcn_raw_buffer_load_b32(rs.type, r0, 0, 0);
    const v2u32 k = __builtin_bit_cast(v2u32, __builtin_amdgcn_raw_buffer_load_b64(rs.tokens, r0 * 2, 0, 0));
    s.kw[0] = k.x; s.kw[1] = k.y;
  } else if constexpr (kEPT == 8) {
    const v2u32 m = __builtin_bit_cast(v2u32, __builtin_amdgcn_raw_buffer_load_b64(rs.model, r0, 0, 0));
    const v2u32 t = __builtin_bit_cast(v2u32, __builtin_amdgcn_raw_buffer_load_b64(rs.type, r0, 0, 0));
    const v4u32 k = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rs.tokens, r0 * 2, 0, 0));
    s.mw[0] = m.x; s.mw[1] = m.y;
    s.tw[0] = t.x; s.tw[1] = t.y;
    s.kw[0] = k.x; s.kw[1] = k.y; s.kw[2] = k.z; s.kw[3] = k.w;
  } else {
    static_assert(kEPT % 16 == 0, "kEPT is 4, 8 or a multiple of 16");
#pragma unroll
    for (int j = 0; j < kEPT / 16; ++j) {
      const v4u32 m = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rs.model, r0 + 16 * j, 0, 0));
      const v4u32 t = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rs.type, r0 + 16 * j, 0, 0));
      s.mw[4 * j] = m.x; s.mw[4 * j + 1] = m.y; s.mw[4 * j + 2] = m.z; s.mw[4 * j + 3] = m.w;
      s.tw[4 * j] = t.x; s.tw[4 * j + 1] = t.y; s.tw[4 * j + 2] = t.z; s.tw[4 * j + 3] = t.w;
    }
#pragma unroll
    for (int j = 0; j < kEPT / 8; ++j) {
      const v4u32 k = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rs.tokens, r0 * 2 + 16 * j, 0, 0));
      s.kw[4 * j] = k.x; s.kw[4 * j + 1] = k.y; s.kw[4 * j + 2] = k.z; s.kw[4 * j + 3] = k.w;
    }
  }
}

// Ring layout: window slot s, model m owns the four 64-bit words at
// s * (4M + 1) + 4m (the odd slot stride puts one model's cells of
// neighbouring windows on different LDS banks):
//   +0 tokens    P (low 32 bits) | D (high 32 bits)
//   +1 arrivals  (count << 32) + sum of te over the window's ARRIVE rows
//   +2 admits    (count << 32) + sum of te over its PREFILL|ADMIT rows
//   +3 finishes  (count << 32) + sum of te over its FINISH rows
// with te = t_end - ts in [1, window_ms]. The te sums stay below 2^31
// (events per window * window_ms < 2^31), so no low half carries into its
// count. From them, per window: dA = admits - finishes, dW = arrivals -
// admits, and the in-window integral terms sum(dA * te) and sum(dW * te)
// are the same differences of the te sums.
//
// A row adds one 64-bit word: PREFILL and DECODE rows their tokens to P or
// D, ARRIVE / ADMIT / FINISH rows (1 << 32) + te to their kind's word; an
// ADMIT row also adds its prompt tokens to P. The word and the kind come
// from a table indexed by code = kind | ADMIT >> 5 (4 bits per code:
// word index, bit 2 "high half", bit 3 "lifecycle word"):
//   0 ARRIVE -> word 1, lifecycle; 1 PREFILL -> P; 2 DECODE -> D;
//   3 FINISH -> word 3, lifecycle; 5 PREFILL|ADMIT -> word 2, lifecycle
//   (+ P); 4, 6, 7 (undefined bits, unvalidated input only) -> P.
constexpr uint32_t kRowTable = 0x00A0B409u;

// cb: byte offset of the row's cell (its word 0) in the ring
__device__ __forceinline__ void tally_row(unsigned long long* ring, uint32_t cb, uint32_t ty,
                                          uint32_t tok, uint32_t te) {
  const uint32_t code = (ty & 3u) | ((ty >> 5) & 4u);
  const uint32_t nib = __builtin_amdgcn_ubfe(kRowTable, code << 2, 4);
  // token rows (word 0): the tokens shifted into their half by 32 * "high
  // half" (nib * 8 is that for them); lifecycle rows: (1 << 32) + te
  const unsigned long long tv = (unsigned long long)tok << ((nib << 3) & 63u);
  const bool life = nib >= 8u;
  const uint32_t lo = life ? te : (uint32_t)tv, hi = life ? 1u : (uint32_t)(tv >> 32);
  unsigned char* const cell = (unsigned char*)ring + cb;
  atomicAdd((unsigned long long*)(cell + ((nib & 3u) << 3)), ((unsigned long long)hi << 32) | lo);
  if (code == 5u) atomicAdd((uint32_t*)cell, tok);  // the admitted request's first prompt chunk
}

// General tally of the lane's rows in [e0, e_end) whose window fits the
// ring [cbase, cbase + wcap), with per-row checks (first and last tiles of a
// trace, and tiles that reach past the ring). The first row that does not
// fit stops the lane and is published in *defer (relative to a0) with its
// window in *wdef; the lane holding row t_last (the tile's last) stores
// that row's window in *wlast. Offsets are 32-bit: timestamps are below
// 2^32 ms; a row whose high timestamp word is set (unvalidated input only)
// is skipped.
template <int kEPT>
__device__ __forceinline__ void tally_slice(const Slice<kEPT>& s, int c0, int a0, int e0, int e_end,
                                            int t_last, int cbase, uint32_t base_lo, uint32_t cap,
                                            uint32_t magic, uint32_t win32, uint32_t wmask,
                                            uint32_t sstride, uint32_t mlast,
                                            unsigned long long* ring, unsigned* defer, int* wdef,
                                            int* wlast) {
  const int lo0 = e0 - c0, hi0 = e_end - c0;
  const int lo = lo0 < 0 ? 0 : (lo0 > kEPT ? kEPT : lo0);
  const int hi = hi0 < 0 ? 0 : (hi0 > kEPT ? kEPT : hi0);
  int jdef = kEPT, wdf = INT_MAX;
  bool go = true;  // rows are sorted: the lane stops at its first row past the ring
#pragma unroll
  for (int j = 0; j < kEPT; ++j) {
    const long long ts = s.ts[j];
    if (go && j >= lo && j < hi && ((unsigned long long)ts >> 32) == 0) {
      const uint32_t d = (uint32_t)ts - base_lo;
      uint32_t q, r;
      div_window(d, magic, win32, q, r);
      const int w = cbase + (int)q;
      if (d >= cap) {
        jdef = j;
        wdf = w < cbase ? INT_MAX : w;  // before the ring: unsorted input only; the windows still complete
        go = false;
      } else {
        if (c0 + j == t_last) *wlast = w;
        uint32_t mdl = (s.mw[j >> 2] >> (8 * (j & 3))) & 0xFFu;
        mdl = mdl < mlast ? mdl : mlast;
        const uint32_t ty = (s.tw[j >> 2] >> (8 * (j & 3))) & 0xFFu;
        const uint32_t tok = (s.kw[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
        tally_row(ring, (((uint32_t)w & wmask) * sstride + 4u * mdl) << 3, ty, tok, win32 - r);
      }
    }
  }
  if (__ballot(jdef < kEPT)) {  // some row of this wave waits for a later tile
    if (jdef < kEPT) {
      atomicMin(defer, (unsigned)(c0 + jdef - a0));
      atomicMin(wdef, wdf);
    }
  }
}

// Tally of a lane whose rows all lie in the trace with the last one inside
// the ring (rows are sorted, so every row fits): no per-row checks. Here
// d = ts - base < 2^31 and the quotient q = floor(d / window) < 2^8 is
// trunc((2d + 1) * fl(1 / (2 window))) in fp64: (2d + 1) / (2 window) lies
// at least 1/(2 window) >= 2^-24 away from every integer, far above the
// product's rounding error (below 2^-43). te = (q + 1) * window - d.
// Model bytes are clamped to M - 1, so unvalidated input cannot leave the
// ring.
template <int kEPT>
__device__ __forceinline__ void tally_fast(const Slice<kEPT>& s, uint32_t base_lo, double inv2_win,
                                           uint32_t win32, uint32_t cbm, uint32_t wmask,
                                           uint32_t sstride, uint32_t mlast, bool last, int cbase,
                                           unsigned long long* ring, int* wlast) {
  // (ts << 1) + odd = 2d + 1 (one shift-add: the compiler is not shown how
  // odd derives from base_lo); q * window + wb - ts = te
  uint32_t odd = 1u - 2u * base_lo;
  __asm__("" : "+s"(odd));
  const uint32_t wb = win32 + base_lo;
  const uint32_t sstride8 = sstride << 3;  // ring bytes per window slot
  uint32_t ql = 0;
#pragma unroll
  for (int j = 0; j < kEPT; ++j) {
    const uint32_t t = (uint32_t)s.ts[j];
    const uint32_t q = (uint32_t)((double)((t << 1) + odd) * inv2_win);
    const uint32_t te = __umul24(q, win32) + wb - t;
    ql = q;
    uint32_t mdl = (s.mw[j >> 2] >> (8 * (j & 3))) & 0xFFu;
    mdl = mdl < mlast ? mdl : mlast;
    const uint32_t ty = (s.tw[j >> 2] >> (8 * (j & 3))) & 0xFFu;
    const uint32_t tok = (s.kw[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
    tally_row(ring, __umul24((q + cbm) & wmask, sstride8) + (mdl << 5), ty, tok, te);
  }
  if (last) *wlast = cbase + (int)ql;
}

// A segment's net changes of one model's active and waiting counts as one
// 64-bit sum of (dA << 32) + dW over its rows, dW of either sign; the halves
// come apart again because |dA|, |dW| < 2^27.
__device__ __forceinline__ int net_w(unsigned long long v) { return (int)(uint32_t)v; }
__device__ __forceinline__ int net_a(unsigned long long v) {
  return (int)(uint32_t)((v - (unsigned long long)(long long)net_w(v)) >> 32);
}

// x / d likewise
__device__ __forceinline__ uint32_t div_magic(uint32_t x, uint32_t d, uint32_t magic) {
  const uint32_t q = __umulhi(x, magic);
  return q + (x - q * d >= d ? 1u : 0u);
}

// x mod d for x < 2^32, with magic = floor(2^32 / d) (2^32 - 1 for d = 1):
// the multiply-high undershoots the quotient by at most one
__device__ __forceinline__ uint32_t mod_magic(uint32_t x, uint32_t d, uint32_t magic) {
  const uint32_t r = x - __umulhi(x, magic) * d;
  return r >= d ? r - d : r;
}

// ------------------------------------------------------- control rules
__device__ __forceinline__ unsigned long long dbits(double x) {
  return (unsigned long long)__double_as_longlong(x);
}

// Wave-wide min / max of a 32-bit value, broadcast as a scalar: butterfly
// within quads and rows (DPP quad_perm, half-row and row mirrors), then
// rows folded through row broadcasts; lane 63 ends with the result.
template <bool kMax>
__device__ __forceinline__ uint32_t wave_fold(uint32_t x) {
  // lanes a step does not reach read the identity, so each step is one
  // DPP-sourced min / max
  constexpr int id = kMax ? 0 : -1;
  auto op = [](uint32_t a, uint32_t b) { return kMax ? (a > b ? a : b) : (a < b ? a : b); };
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x140, 0xF, 0xF, false));  // row_mirror
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x142, 0xA, 0xF, false));  // row_bcast:15
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)x, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// Lowest lane among the candidates (bit per lane in cand) holding the
// minimum (kMax: maximum) of Z, or -1. Z >= 0 and never NaN, so its bit
// pattern orders like its value: the high words decide, and the low words
// only where several candidates share the highest / lowest high word
// (for +inf the low word is zero).
template <bool kMax>
__device__ __forceinline__ int wave_arg(unsigned long long cand, double Z, int lane) {
  if (cand == 0ull) return -1;
  const bool c = (cand >> lane) & 1ull;
  const unsigned long long key = dbits(Z);
  const uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key;
  const uint32_t h = wave_fold<kMax>(c ? hi : (kMax ? 0u : 0xFFFFFFFFu));
  unsigned long long tie = __ballot(c && hi == h);
  if (__popcll(tie) > 1 && h != 0x7FF00000u) {
    const bool c2 = (tie >> lane) & 1ull;
    const uint32_t l = wave_fold<kMax>(c2 ? lo : (kMax ? 0u : 0xFFFFFFFFu));
    tie = __ballot(c2 && lo == l);
  }
  return __ffsll((long long)tie) - 1;
}

__device__ __forceinline__ double read_lane_f64(double x, int l) {
  const unsigned long long b = dbits(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

constexpr int kTickBlock = 8;  // ticks loaded and normalised per block

// Replica state of one scenario in the control replay, lane m = model m;
// pool and nm hold the same value in every lane.
struct CtlState {
  int R;          // routable replicas of the lane's model
  long long rw;   // replica-window sum over the windows before `since`
  int since;
  int pool;       // idle replicas (GPUs under the actuation model)
  uint32_t nm;    // moves decided so far
  int g;          // GPUs per replica (1 without the actuation model)
  // actuation: transition in flight (0 none, 1 wake, 2 sleep), the window at
  // whose end it completes, GPUs a sleep returns to the idle pool
  int tkind, tuntil, tret;
};

// Per-scenario constants of the replay, lane m = model m.
struct CtlConst {
  double tau_c, tau_s;
  int r_min;
  uint32_t K;                    // moves allowed per tick
  bool act;                      // the lane holds a model
  unsigned long long live_lanes;
  int32_t wake_w, sleep_w;       // actuation delays in windows
  tre_move* moves;               // the scenario's move log
  uint32_t move_cap;
};

// Transitions that completed before window w (actuation model only): a
// finished wake closes the lane's replica-window sum and raises R; finished
// sleeps return GPUs to the idle pool.
template <bool kAct>
__device__ __forceinline__ void ctl_complete(CtlState& st, int w) {
  if constexpr (kAct) {
    const bool done = st.tkind != 0 && st.tuntil < w;
    if (done && st.tkind == 1) {
      st.rw += (long long)st.R * (st.tuntil + 1 - st.since);
      st.since = st.tuntil + 1;
      st.R += 1;
    }
    unsigned long long back = __ballot(done && st.tkind == 2 && st.tret > 0);
    while (back) {
      const int l = __ffsll((long long)back) - 1;
      st.pool += __builtin_amdgcn_readlane(st.tret, l);
      back &= back - 1ull;
    }
    if (done) st.tkind = 0;
  }
}

// One tick of the control rules at the end of window w (tws: w in bits
// 0-29, kind in bits 30-31: bit 0 fast, bit 1 slow; wave-uniform), with the
// lane's normalised state Z (Eq. (2); +inf when idle or not initialised):
// the regions, the cadence rule, then up to K greedy moves with Eq. (3) for
// the receiver and the donor order of the bounded transfer. Every decision
// is wave-uniform (ballots are the candidate sets, receiver and donor are
// scalars). kAct adds the actuation model: the budget counts GPUs
// (footprint g per replica); a woken replica becomes routable wake_w
// windows after its wake starts; a donor's replica stops being routable at
// once and its GPUs reach the receiver after sleep_w windows, when the
// receiver's wake starts (any shortfall g_r - g_d comes from the idle GPUs
// at the move, any excess returns to them after the sleep); a model with a
// transition in flight is neither receiver nor donor; vetoed models do not
// release. A transition completing at the end of window u counts from
// window u + 1.
template <bool kAct>
__device__ __forceinline__ void ctl_tick(CtlState& st, const CtlConst& c, int lane, uint32_t tws, double Z,
                                         unsigned long long vetoed) {
  const int w = (int)(tws & 0x3FFFFFFFu);
  const uint32_t kind = tws >> 30;
  ctl_complete<kAct>(st, w);
  const unsigned long long crit = __ballot(c.act && Z < c.tau_c);
  unsigned long long ok;
  int path;
  if (crit) {
    if (!(kind & 1u)) return;  // rescue pending: rebalancing defers
    path = TRE_PATH_RESCUE;
    ok = crit;
  } else if (kind & 2u) {
    path = TRE_PATH_REBALANCE;
    ok = __ballot(c.act && Z < 1.0);
  } else {
    return;
  }
  const unsigned long long sur = __ballot(c.act && Z > c.tau_s);
  // models already in a transition: earlier in this tick, or in flight
  unsigned long long used = kAct ? __ballot(st.tkind != 0) : 0ull;
  // both halves widened as unsigned (a set bit 31 must not sign-extend)
  const unsigned long long veto_mask =
      kAct ? ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)vetoed) |
              ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(vetoed >> 32)) << 32))
           : 0ull;
  for (uint32_t k = 0; k < c.K; ++k) {
    const int r = wave_arg<false>(ok & ~used, Z, lane);  // Eq. (3)
    if (r < 0) break;
    const int g_r = kAct ? __builtin_amdgcn_readlane(st.g, r) : 1;
    int d;
    if (st.pool >= g_r) {
      st.pool -= g_r;
      d = TRE_DONOR_POOL;
      if (kAct && lane == r) {
        st.tkind = 1;
        st.tuntil = w + c.wake_w;
      }
    } else {
      const double Zr = read_lane_f64(Z, r);
      const unsigned long long cd =
          __ballot(c.act && st.R > c.r_min && Z > Zr && (!kAct || st.pool >= g_r - st.g)) & ~crit & ~used &
          ~(1ull << r) & c.live_lanes & ~veto_mask;
      d = wave_arg<true>(cd & sur, Z, lane);
      if (d < 0) d = wave_arg<true>(cd & ~sur, Z, lane);
      if (d < 0) break;
      used |= 1ull << d;
      if constexpr (kAct) {
        const int short_by = g_r - __builtin_amdgcn_readlane(st.g, d);
        if (short_by > 0) st.pool -= short_by;
        if (lane == d) {
          st.tkind = 2;
          st.tuntil = w + c.sleep_w;
          st.tret = short_by < 0 ? -short_by : 0;
        }
        if (lane == r) {
          st.tkind = 1;
          st.tuntil = w + c.sleep_w + c.wake_w;
        }
      }
    }
    used |= 1ull << r;
    // routable changes: the donor's at once (from w+1), the receiver's here
    // only without the actuation model (else when its wake completes)
    if (lane == d || (!kAct && lane == r)) {
      st.rw += (long long)st.R * (w + 1 - st.since);
      st.since = w + 1;
      st.R += lane == d ? -1 : 1;
    }
    if (lane == 0 && st.nm < c.move_cap) {
      tre_move mv;
      mv.window = (uint32_t)w;
      mv.path = (uint8_t)path;
      mv.receiver = (uint8_t)r;
      mv.donor = (uint8_t)d;
      mv.pad = 0;
      c.moves[st.nm] = mv;
    }
    ++st.nm;
  }
}

// Initial replica state of a scenario (lane m = model m): R = r_init, idle
// = budget - sum of g * r_init over the models.
__device__ __forceinline__ void ctl_init(CtlState& st, int r_init, int g, bool act, int budget) {
  st.R = act ? r_init : 0;
  st.g = g;
  int rsum = st.R * g;
  rsum += __shfl_xor(rsum, 1);
  rsum += __shfl_xor(rsum, 2);
  rsum += __shfl_xor(rsum, 4);
  rsum += __shfl_xor(rsum, 8);
  rsum += __shfl_xor(rsum, 16);
  rsum += __shfl_xor(rsum, 32);
  st.pool = budget - __builtin_amdgcn_readfirstlane(rsum);
  st.rw = 0;
  st.since = 0;
  st.nm = 0;
  st.tkind = 0;
  st.tuntil = 0;
  st.tret = 0;
}

// ---- a tick's decisions prepared ahead of the replay
// What a tick decides depends on the replica state only through who may
// give and how much is idle; the order in which receivers and donors are
// tried does not. So waves other than the replay's put both orders of each
// tick into LDS (tick_order), several ticks at a time, and the replay's
// serial part per move is bit scans on wave masks and one compare
// (ctl_batch) instead of two or three wave-wide folds of 64-bit values:
// 1024 replays of 720 ticks over 8 models, one wave each, took 0.53 ms with
// the folds.
//   recv[i]  the i-th receiver: models of the tick's path (critical, or Z <
//            1), lowest Z first, lowest index on ties: model | rank << 8
//   don[i]   the i-th donor: models not critical, surplus before the rest,
//            highest Z first, lowest index on ties: model | rank << 8 |
//            position among the receivers << 16 (64: not one)
// with rank the number of models with a smaller Z (equal Z, equal rank), and
// kNoModel past the last; head: window | path << 30, path 0 when no move can
// follow.
constexpr uint32_t kNoModel = 0xFFFFFFFFu;

// Lanes in groups of G = 2^lg (the least power of two that holds M models),
// one group per tick, sub-lane = model: Z of the lane's tick and model
// (unused lanes of a tick, and lanes whose `in` is false, take no part).
// recv, don, head: the lane's tick. zs: 64 words of LDS for this wave alone.
__device__ __forceinline__ void tick_order(uint32_t* recv, uint32_t* don, uint32_t* head, unsigned long long* zs, int lane, int lg, int M,
                                           bool in, double Z, double tau_c, double tau_s, uint32_t w, uint32_t kind) {
  const int sub = lane & ((1 << lg) - 1), base = lane - sub;
  const unsigned long long gm = (lg == 6 ? 0ull : 1ull << (1 << lg)) - 1ull;
  auto group = [&](bool b) { return (__ballot(b) >> base) & gm; };
  const bool act = in && sub < M;
  const bool cr = act && Z < tau_c;
  const bool crit = group(cr) != 0ull;
  const bool ok = crit ? cr : (act && Z < 1.0);
  const bool give = act && !cr, sur = Z > tau_s;
  const unsigned long long okm = group(ok), givem = group(give), surm = group(give && sur);
  uint32_t path = crit ? ((kind & 1u) ? TRE_PATH_RESCUE : 0u)  // rescue pending: rebalancing defers
                       : ((kind & 2u) ? TRE_PATH_REBALANCE : 0u);
  if (okm == 0ull) path = 0u;
  if (in && sub == 0) *head = w | (path << 30);
  if (!__ballot(in && path != 0u)) return;
  uint32_t rank = 0, p = 0, q = 0;  // models with a smaller Z; receivers and donors before this lane's model
  // Z >= 0 or NaN. The bit patterns order like the values; a NaN, which is no
  // receiver, takes the lowest, so that its rank lies above no receiver's and it
  // never gives. zs holds the wave's own words (its LDS operations stay in order)
  const unsigned long long zm = Z == Z ? dbits(Z) : 0ull;
  const uint32_t nsur = sur ? 0u : 1u;
  zs[lane] = zm;
  __builtin_amdgcn_wave_barrier();
  auto count = [&](uint32_t okw, uint32_t givew, uint32_t surw, int j0, int n) {  // models j0 .. j0 + n - 1 (at most 32)
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const unsigned long long zj = zs[base + j0 + j];
      const uint32_t less = zj < zm ? 1u : 0u, first = (j0 + j < sub ? zj <= zm : zj < zm) ? 1u : 0u;
      const uint32_t above = (j0 + j < sub ? zj >= zm : zj > zm) ? 1u : 0u;
      const uint32_t sj = __builtin_amdgcn_ubfe(surw, (uint32_t)j, 1);
      rank += less;
      p += __builtin_amdgcn_ubfe(okw, (uint32_t)j, 1) & first;
      // a surplus model goes before every other, then the higher Z
      q += __builtin_amdgcn_ubfe(givew, (uint32_t)j, 1) & ((sj & nsur) | ((sj ^ nsur) & above));
    }
  };
  count((uint32_t)okm, (uint32_t)givem, (uint32_t)surm, 0, M < 32 ? M : 32);
  if (M > 32) count((uint32_t)(okm >> 32), (uint32_t)(givem >> 32), (uint32_t)(surm >> 32), 32, M - 32);
  if (act && path != 0u) {
    const uint32_t word = (uint32_t)sub | (rank << 8);
    if (ok) recv[p] = word;
    if (sub >= __popcll(okm)) recv[sub] = kNoModel;
    if (give) don[q] = word | ((ok ? p : 64u) << 16);
    if (sub >= __popcll(givem)) don[sub] = kNoModel;
  }
}

// Replica state of a replay of prepared ticks: lane m = model m; pool and nm
// are the same in every lane.
struct OrdState {
  int R;         // routable replicas of the lane's model
  long long rw;  // sum over all windows of R as it stands: a change at window w adds it times the windows after w
  int pool;      // idle replicas (GPUs under the actuation model)
  uint32_t nm;   // moves decided so far
  int g;
  int tkind, tuntil, tret;  // as CtlState
};

struct OrdConst {
  int r_min;
  uint32_t K;
  bool act;
  int32_t n_windows, wake_w, sleep_w;
  tre_move* moves;
  uint32_t move_cap;
};

template <bool kAct>
__device__ __forceinline__ void ord_complete(OrdState& st, const OrdConst& c, int w) {
  if constexpr (kAct) {
    const bool done = st.tkind != 0 && st.tuntil < w;
    if (done && st.tkind == 1) {
      st.rw += c.n_windows - 1 - st.tuntil;
      st.R += 1;
    }
    unsigned long long back = __ballot(done && st.tkind == 2 && st.tret > 0);
    while (back) {
      const int l = __ffsll((long long)back) - 1;
      st.pool += __builtin_amdgcn_readlane(st.tret, l);
      back &= back - 1ull;
    }
    if (done) st.tkind = 0;
  }
}

// The prepared ticks [0, n) of a batch, in order (recv and don M entries a
// tick), with the rules and results of ctl_tick. Ticks that can move nothing
// are passed over 64 at a time, and a tick's entries are read while the one
// before it is decided. Receivers are taken in ascending Z, so one is never
// a donor of the same tick (a donor's Z lies above the receiver's); a donor
// leaves the receivers by its position among them. gm: the models'
// footprints in LDS (kAct); veto(i): the tick's mask.
template <bool kAct, class Veto>
__device__ __forceinline__ void ctl_batch(OrdState& st, const OrdConst& c, int lane, int M, int n,
                                          const uint32_t* recv, const uint32_t* don, const uint32_t* head,
                                          const int* gm, Veto veto) {
  for (int i0 = 0; i0 < n; i0 += 64) {
    const uint32_t h = i0 + lane < n ? head[i0 + lane] : 0u;
    unsigned long long todo = __ballot((h >> 30) != 0u);
    if (!todo) continue;
    const int ml = lane < M ? lane : 0;
    int i = __ffsll((long long)todo) - 1;
    uint32_t rw = recv[(i0 + i) * M + ml], dw = don[(i0 + i) * M + ml];
    while (todo) {
      todo &= todo - 1ull;
      const int nx = todo ? __ffsll((long long)todo) - 1 : i;
      const uint32_t rn = recv[(i0 + nx) * M + ml], dn = don[(i0 + nx) * M + ml];
      const uint32_t hd = (uint32_t)__builtin_amdgcn_readlane((int)h, i);
      const int w = (int)(hd & 0x3FFFFFFFu);
      ord_complete<kAct>(st, c, w);
      // the candidates, in order, as wave masks
      const unsigned long long busy = kAct ? __ballot(st.tkind != 0) : 0ull;
      const unsigned long long can =
          __ballot(c.act && st.R > c.r_min) & (kAct ? ~(busy | veto(i0 + i)) : ~0ull);
      unsigned long long rc = __ballot(c.act && rw != kNoModel && !(kAct && ((busy >> (rw & 63u)) & 1ull)));
      unsigned long long dc = __ballot(c.act && dw != kNoModel && ((can >> (dw & 63u)) & 1ull));
      const uint32_t drank = (dw >> 8) & 0xFFu;
      int gd = 1;
      if constexpr (kAct) gd = gm[dw & 63u];
      unsigned long long gain = 0ull, lose = 0ull, slept = 0ull;  // models: a replica more, one less; receivers of a slept one
      uint32_t k = 0, mv = 0;  // moves of this tick (at most one per receiver), lane i: the i-th
      while (k < c.K && rc) {
        const uint32_t rr = (uint32_t)__builtin_amdgcn_readlane((int)rw, __ffsll((long long)rc) - 1);  // Eq. (3)
        const uint32_t r = rr & 63u;
        const int g_r = kAct ? __builtin_amdgcn_readlane(st.g, (int)r) : 1;
        const bool pool = st.pool >= g_r;
        const unsigned long long cd = dc & __ballot(drank > (rr >> 8) && (!kAct || st.pool >= g_r - gd));
        if (!pool && !cd) break;
        const int at = (__ffsll((long long)cd) - 1) & 63;
        const uint32_t dd = pool ? (64u << 16) | TRE_DONOR_POOL : (uint32_t)__builtin_amdgcn_readlane((int)dw, at);
        const uint32_t rp = dd >> 16;
        const unsigned long long dbit = pool ? 0ull : 1ull << (dd & 63u);
        dc &= ~(pool ? 0ull : 1ull << at);
        rc &= rc - 1ull;
        rc &= ~(rp < 64u ? 1ull << (rp & 63u) : 0ull);
        lose |= dbit;
        gain |= 1ull << r;
        if constexpr (kAct) {
          slept |= pool ? 0ull : 1ull << r;
          const int short_by = pool ? g_r : g_r - __builtin_amdgcn_readlane(st.g, (int)(dd & 63u));
          if ((dbit >> lane) & 1ull) st.tret = short_by < 0 ? -short_by : 0;
          st.pool -= short_by > 0 ? short_by : 0;
        } else {
          st.pool -= pool ? 1 : 0;
        }
        mv = (uint32_t)lane == k ? (hd >> 30) | (r << 8) | ((dd & 0xFFu) << 16) : mv;
        ++k;
      }
      if ((uint32_t)lane < k && st.nm + (uint32_t)lane < c.move_cap) {
        tre_move m;
        m.window = (uint32_t)w;
        m.path = (uint8_t)mv;
        m.receiver = (uint8_t)(mv >> 8);
        m.donor = (uint8_t)(mv >> 16);
        m.pad = 0;
        c.moves[st.nm + (uint32_t)lane] = m;
      }
      st.nm += k;
      // the routable changes: the donors' at once (from w + 1), the receivers'
      // here only without the actuation model (else when their wakes complete)
      const bool lost = (lose >> lane) & 1ull, got = (gain >> lane) & 1ull;
      const int dR = (!kAct && got ? 1 : 0) - (lost ? 1 : 0);
      st.R += dR;
      st.rw += (long long)dR * (c.n_windows - 1 - w);
      if constexpr (kAct) {
        if (got) {
          st.tkind = 1;
          st.tuntil = w + c.wake_w + (((slept >> lane) & 1ull) ? c.sleep_w : 0);
        }
        if (lost) {
          st.tkind = 2;
          st.tuntil = w + c.sleep_w;
        }
      }
      i = nx;
      rw = rn;
      dw = dn;
    }
  }
}

// the state before the first window, and the outputs after the last
__device__ __forceinline__ void ord_init(OrdState& st, const OrdConst& c, int r_init, int g, int budget) {
  CtlState s0;
  ctl_init(s0, r_init, g, c.act, budget);
  st.R = s0.R;
  st.rw = (long long)s0.R * c.n_windows;
  st.pool = s0.pool;
  st.nm = 0;
  st.g = g;
  st.tkind = st.tuntil = st.tret = 0;
}

template <bool kAct>
__device__ __forceinline__ void ord_finish(OrdState& st, const OrdConst& c, int lane, int32_t* r_final,
                                           int64_t* r_windows, uint32_t* n_moves) {
  ord_complete<kAct>(st, c, c.n_windows);  // transitions completing at the end of the last window count as done
  if (c.act) {
    r_final[lane] = st.R;
    r_windows[lane] = st.rw;
  }
  if (lane == 0) *n_moves = st.nm;
}

// One model's replay constants and state in LDS, for a replay that moves
// between waves from step to step.
struct CtlModel {
  double theta;     // theta * theta_scale
  double tau_c, tau_s;
  long long rw;
  int R, since, r_min, pad;
};

// One workgroup per trace; every thread tallies and evaluates, one barrier
// per step. Step k, with [cA, cB) the chunk evaluated in step k-1 and
// [cB, cC), cC = min(wl, cB + C), the windows completed by earlier tiles
// (wl: the window of the last row tallied so far, or of the first row
// deferred):
//   - wave k % kWaves runs the smoothing chain over [cA, cB) from the
//     staging buffer of step k-1 (state in LDS, so the chain can move
//     between waves), its tick windows from one ballot; first, so that its
//     LDS reads find the queue the barrier just drained;
//   - read and clear the ring cells of [cB, cC): complete windows;
//   - issue the loads of tile k+1 and tally tile k into the ring: rows
//     whose window reaches cB + wcap wait for a later tile. Rows of tile k
//     come after every row of a complete window, so they land in windows
//     >= cC, on slots disjoint from the chunk's;
//   - evaluate [cB, cC), one (window, model) cell per thread: carry prefix
//     over the chunk, window integrals, Eq. (1) -> raw ratio, staged in LDS
//     (two staging buffers, by step parity);
//   -- barrier -- the tile's rows are in; windows < wl are complete.
//
// kSeg: the workgroup takes one segment of a trace's windows, [w_lo, w_hi),
// and that segment's rows; its carries start from the net changes of the
// segments before it, the raw ratios go to memory and chain_smooth smooths
// them, so there is no chain, control replay or staging here.
template <int kWaves, int kEPT, bool kCells, bool kStage, bool kSeg = false>
__device__ __forceinline__ void stream_body(const StreamParams& p) {
  constexpr int kThreads = kWaves * 64;
  constexpr long long kTile = (long long)kThreads * kEPT;
  extern __shared__ unsigned long long ring[];
  __shared__ int s_carry[2][2][TRE_MAX_MODELS];  // [parity][active, waiting][model], |count| < 2^27
  __shared__ double s_S[TRE_MAX_MODELS];               // smoothed TSS per model
  __shared__ double s_alpha[TRE_MAX_MODELS];
  __shared__ uint8_t s_init[TRE_MAX_MODELS];
  __shared__ int s_tick[3];                            // fast / slow counters, tick ordinal
  __shared__ unsigned s_defer[3];
  __shared__ int s_wdef[3];
  __shared__ int s_wlast[3];  // window of the tile's last row
  __shared__ uint32_t s_first[kSeg ? 2 * TRE_MAX_MODELS : 1];  // kSeg: per column, the first window not idle

  const int trace = kSeg ? (int)(blockIdx.x / (unsigned)p.nseg) : (int)blockIdx.x;
  const int seg = kSeg ? (int)(blockIdx.x % (unsigned)p.nseg) : 0;
  const int tid = threadIdx.x;
  const int M = p.M;
  const uint32_t wcap = p.wcap;
  const int C = p.chunk;
  const uint32_t sstride = 4u * (uint32_t)M + 1u;  // ring words per window slot
  const int nring = (int)(wcap * sstride);
  // [nbuf][C][M] staged raw ratios (>= 0), -1 marks an idle window. Step k's
  // evaluation writes buffer k % nbuf and the smoothing chain of step k + 1
  // reads it; with the control replay in the stream the chain writes the
  // smoothed values of its tick windows back into it, and the replay reads
  // them in step k + 2 (hence three buffers)
  constexpr int nbuf = kStage ? 2 : 3;
  double* st_raw = (double*)(ring + nring);
  // kStage (no scalar TSS is written): the staged prefill ratios in the
  // scalar ratios' place and the decode ratios after them ([2][C][M] each,
  // -1 idle), then each model's smoothed shares and init flags
  double* const st_p = st_raw;
  double* const st_d = st_raw + 2 * C * M;
  double* const s_Sp = st_d + 2 * C * M;
  double* const s_Sd = s_Sp + M;
  uint8_t* const s_ip = (uint8_t*)(s_Sd + M);
  uint8_t* const s_id = s_ip + M;
  // the control replay (not kStage): one record per model, then idle
  // replicas, moves, and per staging buffer the fast- and slow-tick masks of
  // its chunk and the chunk's first window
  CtlModel* const s_cm = (CtlModel*)(st_raw + 3 * C * M);
  uint32_t* const s_cmeta = (uint32_t*)(s_cm + M);  // [0] idle, [1] moves, [2+b] fast, [5+b] slow, [8+b] window
  long long e_begin = p.off[trace];
  long long e_end = p.off[trace + 1];
  if constexpr (kSeg) {
    const int32_t* const sr = p.seg_row + (int64_t)trace * (p.nseg + 1) + seg;
    const int r0 = sr[0], r1 = sr[1];  // within the trace's rows; r0 <= r1 when they are sorted
    e_end = e_begin + (r1 > r0 ? r1 : r0);
    e_begin += r0;
  }
  const long long win = p.window_ms;
  const uint32_t win32 = (uint32_t)win;
  const double dwin = (double)win;
  const int nWt = p.n_windows;  // windows of the trace
  const int w_lo = kSeg ? seg * p.seg_w : 0;
  const int nW = kSeg ? (w_lo + p.seg_w < nWt ? w_lo + p.seg_w : nWt) : nWt;  // one past this workgroup's last
  constexpr bool cells = kCells;

  for (int i = tid; i < nring; i += kThreads) ring[i] = 0ull;
  for (int i = tid; i < 2 * 2 * TRE_MAX_MODELS; i += kThreads) (&s_carry[0][0][0])[i] = 0;
  if (tid < 3) {
    s_defer[tid] = kNoDefer;
    s_wdef[tid] = INT_MAX;
    s_wlast[tid] = -1;
  }

  // the cell this thread evaluates: model rm, window offset rj in the chunk
  // (C is a power of two and C * M <= kEvalThreads <= threads; the rest have no cell)
  const int rm = tid / C, rj = tid & (C - 1);
  const bool r_thread = rm < M;
  // bit sh set where the lane 2^sh below lies in the same group of C lanes
  // (rj >= 2^sh, so never for 2^sh >= C); opaque to the compiler so that it
  // stays one per-lane register, not four lane masks held in SGPRs
  uint32_t r_take = 0;
#pragma unroll
  for (int sh = 0; sh < 4; ++sh) r_take |= rj >= (1 << sh) ? 1u << sh : 0u;
  __asm__("" : "+v"(r_take));
  double w_p = 0.0, w_q = 0.0;
  if (r_thread) {
    const tre_profile pr = p.prof[(int64_t)trace * M + rm];
    w_p = pr.w_p;
    w_q = pr.w_q;
  }
  // smoothing chain: one wave per step (rotating), lane m owns model m; its
  // state lives in LDS between steps
  if (!kSeg && tid < M) {
    s_alpha[tid] = p.prof[(int64_t)trace * M + tid].alpha;
    s_S[tid] = 0.0;
    s_init[tid] = 0;
    if constexpr (kStage) {
      s_Sp[tid] = 0.0;
      s_Sd[tid] = 0.0;
      s_ip[tid] = 0;
      s_id[tid] = 0;
    }
  }
  if (tid < 3) s_tick[tid] = 0;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;

  // the trace's one scenario, replayed here (else -1: the tick snapshot is
  // written for a separate replay)
  int ctl_s = -1;
  uint32_t ctl_K = 0;
  if constexpr (!kStage && !kSeg) {
    if (p.ctl_one) ctl_s = 0;
    else if (p.sc_count && p.sc_count[trace] == 1u) ctl_s = (int)p.sc_first[trace];
  }
  ctl_s = __builtin_amdgcn_readfirstlane(ctl_s);
  if (ctl_s >= 0) {
    const tre_scenario sc = p.sc[ctl_s];
    ctl_K = sc.max_moves;
    if (wave == 0) {
      const bool act = lane < M;
      const tre_profile pr = p.prof[(int64_t)trace * M + (act ? lane : 0)];
      CtlState st;
      ctl_init(st, pr.r_init, 1, act, p.budget);
      if (act) {
        CtlModel cm;
        cm.theta = pr.theta * sc.theta_scale;
        cm.tau_c = sc.tau_crit_override >= 0.0 ? sc.tau_crit_override : pr.tau_crit;
        cm.tau_s = pr.tau_surplus;
        cm.rw = 0;
        cm.R = st.R;
        cm.since = 0;
        cm.r_min = pr.r_min;
        cm.pad = 0;
        s_cm[lane] = cm;
      }
      if (lane < 11) s_cmeta[lane] = lane == 0 ? (uint32_t)st.pool : 0u;
    }
  }
  // the replay of the ticks the chain recorded in staging buffer b: state
  // from LDS, ctl_tick per tick in window order, state back to LDS; the
  // buffer's ticks are then consumed
  auto ctl_run = [&](int b) {
    const uint32_t tmf = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cmeta[2 + b]);
    const uint32_t tms = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cmeta[5 + b]);
    uint32_t tm = tmf | tms;
    if (!tm) return;
    const int w0 = __builtin_amdgcn_readfirstlane((int)s_cmeta[8 + b]);
    const bool act = lane < M;
    const int m = act ? lane : 0;
    CtlModel* const cm = s_cm + m;
    CtlState st;
    st.R = cm->R;
    st.rw = cm->rw;
    st.since = cm->since;
    st.pool = __builtin_amdgcn_readfirstlane((int)s_cmeta[0]);
    st.nm = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cmeta[1]);
    st.g = 1;
    st.tkind = 0;
    st.tuntil = 0;
    st.tret = 0;
    CtlConst c;
    c.tau_c = cm->tau_c;
    c.tau_s = cm->tau_s;
    c.r_min = cm->r_min;
    c.K = ctl_K;
    c.act = act;
    c.live_lanes = __ballot(act);
    c.wake_w = 0;
    c.sleep_w = 0;
    c.moves = p.moves + (int64_t)ctl_s * p.move_cap;
    c.move_cap = p.move_cap;
    const double th = cm->theta;
    const double* sb = st_raw + b * C * M + m;
    while (tm) {
      const int u = __ffs(tm) - 1;
      tm &= tm - 1u;
      const double Z = act ? sb[u * M] / th : INFINITY;  // Eq. (2); the buffer holds +inf when idle / not initialised
      const uint32_t kind = ((tmf >> u) & 1u) | (((tms >> u) & 1u) << 1);
      ctl_tick<false>(st, c, lane, (uint32_t)(w0 + u) | (kind << 30), Z, 0ull);
    }
    if (act) {
      cm->R = st.R;
      cm->rw = st.rw;
      cm->since = st.since;
    }
    if (lane == 0) {
      s_cmeta[0] = (uint32_t)st.pool;
      s_cmeta[1] = st.nm;
      s_cmeta[2 + b] = 0u;
      s_cmeta[5 + b] = 0u;
    }
  };

  // rows are counted from the trace's first kEPT-aligned row (below 2^27)
  const long long brow = e_begin & ~(long long)(kEPT - 1);
  const int rend = (int)(e_end - brow);  // one past the trace's last row
  int e0 = (int)(e_begin - brow);        // first row not yet tallied
  int cA = w_lo, cB = w_lo, wl = w_lo;
  TraceRsrc rs;
  rs.ts = rsrc(p.ts + brow, (long long)rend * 8);
  rs.model = rsrc(p.model + brow, rend);
  rs.type = rsrc(p.type + brow, rend);
  rs.tokens = rsrc(p.tokens + brow, (long long)rend * 2);
  Slice<kEPT> buf0, buf1;
  int held = 0;  // tile base held by the current buffer
  load_slice<kEPT>(buf0, rs, tid * kEPT);
  __syncthreads();
  if constexpr (kSeg) {
    for (int i = tid; i < (kStage ? 2 : 1) * M; i += kThreads) s_first[i] = kNoDefer;
    // the carries: the net changes of the segments before this one
    const unsigned long long* const net = p.seg_net + (int64_t)trace * p.nseg * M;
    for (int i = tid; i < seg * M; i += kThreads) {
      const unsigned long long v = net[i];
      const int m = i % M;
      if (v) {
        atomicAdd(&s_carry[0][0][m], net_a(v));
        atomicAdd(&s_carry[0][1][m], net_w(v));
      }
    }
    __syncthreads();
  }

  // one step; returns true when every window has been smoothed
  auto step = [&](Slice<kEPT>& cur, Slice<kEPT>& nxt, int k) -> bool {
    if ((kSeg ? cB : cA) >= nW) return true;
    const int b3 = k % 3;
    // ---- issue the loads of tile k+1 first (and of tile k again when the
    // prefetch missed it): with both buffers live from here on, nothing
    // below reuses a register a load is still filling
    const int a0 = e0 & ~(kEPT - 1);
    if (held != a0) load_slice<kEPT>(cur, rs, a0 + tid * kEPT);  // prefetch missed
    const int pref = a0 + (int)kTile;
    load_slice<kEPT>(nxt, rs, pref + tid * kEPT);  // zeros past the trace
    // ---- smooth [cA, cB) (staged last step); wave k mod kWaves, lanes < M
    if (!kSeg && wave == k % kWaves && cB > cA) {
      // the whole workgroup waits for this wave at the step's barrier: let its
      // dependent chain issue ahead of the other waves on its SIMD
      __builtin_amdgcn_s_setprio(3);
      const bool own = lane < M;
      const int m = own ? lane : 0;
      const int bc = (k + nbuf - 1) % nbuf;  // staged in step k - 1
      double* const pr = st_raw + bc * C * M + m;
      const double alpha = s_alpha[m];
      const double oma = 1.0 - alpha;
      double S = s_S[m];
      bool init = s_init[m] != 0;
      double Sp = 0.0, Sd = 0.0;
      bool ip = false, id = false;
      if constexpr (kStage) {
        Sp = s_Sp[m];
        Sd = s_Sd[m];
        ip = s_ip[m] != 0;
        id = s_id[m] != 0;
      }
      // windows since the last fast / slow tick before cA, ticks so far
      const uint32_t fctr = (uint32_t)__builtin_amdgcn_readfirstlane(s_tick[0]);
      const uint32_t sctr = (uint32_t)__builtin_amdgcn_readfirstlane(s_tick[1]);
      int tick = __builtin_amdgcn_readfirstlane(s_tick[2]);
      const int nw = cB - cA;
      // tick windows of the chunk: bit u for window cA + u (u < nw), fast
      // and slow cadences apart (scalar loops over the period ends)
      uint32_t tmf = 0u, tms = 0u;
      for (uint32_t u = (uint32_t)p.fast_w - 1u - fctr; u < (uint32_t)nw; u += (uint32_t)p.fast_w) tmf |= 1u << u;
      for (uint32_t u = (uint32_t)p.slow_w - 1u - sctr; u < (uint32_t)nw; u += (uint32_t)p.slow_w) tms |= 1u << u;
      const uint32_t tm = tmf | tms;
      for (int u0 = 0; u0 < nw; u0 += 4) {
        double rv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) rv[u] = pr[((u0 + u) & (C - 1)) * M];  // past nw: unused
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (u0 + u < nw) {
            const int w = cA + u0 + u;
            const double raw = rv[u];
            const bool idle = raw < 0.0;
            if constexpr (!kStage) {
              const double t1 = alpha * raw;
              const double t2 = oma * S;
              const double Sn = t1 + t2;
              S = idle ? S : (init ? Sn : raw);
              init = init || !idle;
            }
            if (cells && own) {
              const int64_t c = ((int64_t)trace * nW + w) * M + m;
              if (p.tss64) p.tss64[c] = S;
              if (p.tss32) p.tss32[c] = (float)S;
              if (p.flags) p.flags[c] = (uint8_t)((idle ? TRE_FLAG_IDLE : 0) | (init ? TRE_FLAG_INIT : 0));
            }
            if constexpr (kStage) {  // the stage shares: the same smoothing per stage
              const int j = ((u0 + u) & (C - 1)) * M + bc * C * M + m;
              const double rp = raw, rd = st_d[j];  // st_p is st_raw
              const bool pi = rp < 0.0, di = rd < 0.0;
              const double p1 = alpha * rp;
              const double p2 = oma * Sp;
              const double pn = p1 + p2;
              Sp = pi ? Sp : (ip ? pn : rp);
              ip = ip || !pi;
              const double d1 = alpha * rd;
              const double d2 = oma * Sd;
              const double dn = d1 + d2;
              Sd = di ? Sd : (id ? dn : rd);
              id = id || !di;
              if (own) {
                const int64_t c = ((int64_t)trace * nW + w) * M + m;
                if (p.stage64) *(double2*)(p.stage64 + 2 * c) = make_double2(Sp, Sd);
                if (p.stage32) *(float2*)(p.stage32 + 2 * c) = make_float2((float)Sp, (float)Sd);
                if (p.sflags)
                  p.sflags[c] = (uint8_t)((pi ? TRE_STAGE_P_IDLE : 0) | (ip ? TRE_STAGE_P_INIT : 0) |
                                          (di ? TRE_STAGE_D_IDLE : 0) | (id ? TRE_STAGE_D_INIT : 0));
              }
            }
            if ((tm >> (u0 + u)) & 1u) {
              const double zs = (idle || !init) ? INFINITY : S;
              if (ctl_s >= 0) {  // for the replay two steps on (the raw ratio is read already)
                if (own) pr[((u0 + u) & (C - 1)) * M] = zs;
              } else if (own && p.snap && tick < p.n_ticks) {
                p.snap[((int64_t)trace * p.n_ticks + tick) * M + m] = zs;
              }
              ++tick;
            }
          }
        }
      }
      if (own) {
        s_S[m] = S;
        s_init[m] = init ? 1 : 0;
        if constexpr (kStage) {
          s_Sp[m] = Sp;
          s_Sd[m] = Sd;
          s_ip[m] = ip ? 1 : 0;
          s_id[m] = id ? 1 : 0;
        }
      }
      if (lane == 0) {
        s_tick[0] = (int)mod_magic(fctr + (uint32_t)nw, (uint32_t)p.fast_w, p.magic_fast);
        s_tick[1] = (int)mod_magic(sctr + (uint32_t)nw, (uint32_t)p.slow_w, p.magic_slow);
        s_tick[2] = tick;
        if (ctl_s >= 0) {
          s_cmeta[2 + bc] = tmf;
          s_cmeta[5 + bc] = tms;
          s_cmeta[8 + bc] = (uint32_t)cA;
        }
      }
      __builtin_amdgcn_s_setprio(0);
    }
    // ---- read and clear the cells of [cB, cC), one cell per thread (groups
    // of C lanes per model): complete windows that no row of this tile
    // reaches. LDS operations of a wave retire in order, so these reads go
    // ahead of the tally's atomics.
    const int cC = wl < cB + C ? wl : cB + C;
    const int n = cC - cB;
    const bool valid = r_thread && rj < n;
    unsigned long long pd = 0, w_arr = 0, w_adm = 0, w_fin = 0;
    if (valid) {
      const uint32_t c = ((uint32_t)(cB + rj) & (wcap - 1)) * sstride + 4u * (uint32_t)rm;
      pd = ring[c];
      w_arr = ring[c + 1];
      w_adm = ring[c + 2];
      w_fin = ring[c + 3];
      ring[c] = 0ull;
      ring[c + 1] = 0ull;
      ring[c + 2] = 0ull;
      ring[c + 3] = 0ull;
    }
    // ---- tally tile k (tile k+1 loading meanwhile), capacity [cB, cB + wcap)
    const int t_last = (pref < rend ? pref : rend) - 1;
    {
      const int c0 = a0 + tid * kEPT;
      const uint32_t base_lo = (uint32_t)((long long)cB * win);
      const uint32_t cap = wcap * win32;
      const bool lane_fast = c0 >= e0 && c0 + kEPT <= rend && (uint32_t)cur.ts[kEPT - 1] - base_lo < cap;
      if (__ballot(!lane_fast) == 0ull)  // wave-uniform
        tally_fast<kEPT>(cur, base_lo, p.inv2_window, win32, (uint32_t)cB & (wcap - 1), wcap - 1, sstride,
                         (uint32_t)M - 1u, c0 + kEPT - 1 == t_last, cB, ring, &s_wlast[b3]);
      else
        tally_slice<kEPT>(cur, c0, a0, e0, rend, t_last, cB, base_lo, cap, p.magic, win32, wcap - 1,
                          sstride, (uint32_t)M - 1u, ring, &s_defer[b3], &s_wdef[b3], &s_wlast[b3]);
    }
    // ---- evaluate [cB, cC): carry prefix, window integrals, Eq. (1)
    const int* cin = s_carry[k & 1][0];
    int* cout = s_carry[(k + 1) & 1][0];
    double* sr = st_raw + (k % nbuf) * C * M;
    if (r_thread) {  // uniform over each group of C lanes
      // net active / waiting changes and their in-window integral terms
      const int ca = (int)((uint32_t)(w_adm >> 32) - (uint32_t)(w_fin >> 32));
      const int cw = (int)((uint32_t)(w_arr >> 32) - (uint32_t)(w_adm >> 32));
      const int la32 = (int)((uint32_t)w_adm - (uint32_t)w_fin);
      const int lw32 = (int)((uint32_t)w_arr - (uint32_t)w_adm);
      int ia = ca, iw = cw;  // inclusive prefix over the chunk's windows
      if (C <= 16) {
        uint32_t rt = r_take;  // re-read each step: the masks are not kept live across steps
        __asm__ volatile("" : "+v"(rt));
        // row shifts by 1, 2, 4, 8 lanes (groups are aligned inside a row),
        // each taken where the neighbour lies in the lane's own group; the
        // masks are per-lane integers, so no lane mask stays live in SGPRs
#define TRE_ROW_SHR_STAGE(sh)                                                   \
  {                                                                             \
    const int ya = __builtin_amdgcn_mov_dpp(ia, 0x110 | (1 << (sh)), 0xF, 0xF, true); \
    const int yw = __builtin_amdgcn_mov_dpp(iw, 0x110 | (1 << (sh)), 0xF, 0xF, true); \
    const int mk = __builtin_amdgcn_sbfe((int)rt, (sh), 1); /* -1 or 0 */       \
    ia += ya & mk;                                                              \
    iw += yw & mk;                                                              \
  }
        TRE_ROW_SHR_STAGE(0)
        TRE_ROW_SHR_STAGE(1)
        TRE_ROW_SHR_STAGE(2)
        TRE_ROW_SHR_STAGE(3)
#undef TRE_ROW_SHR_STAGE
      } else {
        for (int dd = 1; dd < C; dd <<= 1) {
          const int ya = __shfl_up(ia, dd, C);
          const int yw = __shfl_up(iw, dd, C);
          if (rj >= dd) {
            ia += ya;
            iw += yw;
          }
        }
      }
      if (valid) {
        const int w = cB + rj;
        const int A0 = cin[rm] + (ia - ca), W0 = cin[TRE_MAX_MODELS + rm] + (iw - cw);
        // the window integrals in fp64, exactly: a trace has fewer than 2^27
        // rows, so |A0|, |W0| < 2^27, A0 * window < 2^50 and the sum with the
        // in-window term (below 2^31) stays below 2^53
        const double A_f = __builtin_fma((double)A0, dwin, (double)la32);
        const double W_f = __builtin_fma((double)W0, dwin, (double)lw32);
        const uint32_t P = (uint32_t)pd, Dt = (uint32_t)(pd >> 32);
        const bool idle = pd == 0ull && A_f == 0.0 && W_f == 0.0;
        double raw = 0.0;
        if (!kStage && !idle) {
          // Eq. (1), evaluated in the documented order
          double num = w_p * (double)P;
          num = num + (double)Dt;
          num = num * 1000.0;
          const double q = w_q * W_f;
          double den = A_f + q;
          if (den < dwin) den = dwin;
          raw = num / den;
        }
        if constexpr (!kStage && !kSeg) sr[rj * M + rm] = idle ? -1.0 : raw;
        if constexpr (!kStage && kSeg) {
          p.raw[((int64_t)trace * M + rm) * nWt + w] = idle ? -1.0 : raw;
          if (!idle && (uint32_t)w < s_first[rm]) atomicMin(&s_first[rm], (uint32_t)w);
        }
        if constexpr (kStage) {
          // the two parts of Eq. (1), each with its one-request floor; a
          // stage is idle when its tokens and its demand integral are zero
          double rp = -1.0, rd = -1.0;
          if (P != 0u || W_f != 0.0) {
            double num = w_p * (double)P;
            num = num * 1000.0;
            double den = w_q * W_f;
            if (den < dwin) den = dwin;
            rp = num / den;
          }
          if (Dt != 0u || A_f != 0.0) {
            const double num = (double)Dt * 1000.0;
            double den = A_f;
            if (den < dwin) den = dwin;
            rd = num / den;
          }
          if constexpr (kSeg) {
            double* const rw = p.raw + ((int64_t)trace * M + rm) * 2 * nWt + w;
            rw[0] = rp;
            rw[nWt] = rd;
            // not idle: also a NaN (infinite tokens over infinite demand)
            if (!(rp < 0.0) && (uint32_t)w < s_first[2 * rm]) atomicMin(&s_first[2 * rm], (uint32_t)w);
            if (!(rd < 0.0) && (uint32_t)w < s_first[2 * rm + 1]) atomicMin(&s_first[2 * rm + 1], (uint32_t)w);
          } else {
            st_p[(k % nbuf) * C * M + rj * M + rm] = rp;
            st_d[(k % nbuf) * C * M + rj * M + rm] = rd;
          }
        }
        if (cells) {
          const int64_t o = ((int64_t)trace * nWt + w) * M + rm;
          if (p.prefill) p.prefill[o] = P;
          if (p.decode) p.decode[o] = Dt;
          if (p.a_int) p.a_int[o] = (long long)A0 * win + la32;
          if (p.w_int) p.w_int[o] = (long long)W0 * win + lw32;
        }
        if (rj == n - 1) {
          cout[rm] = cin[rm] + ia;
          cout[TRE_MAX_MODELS + rm] = cin[TRE_MAX_MODELS + rm] + iw;
        }
      }
    }
    if (n == 0 && tid < M) {
      cout[tid] = cin[tid];
      cout[TRE_MAX_MODELS + tid] = cin[TRE_MAX_MODELS + tid];
    }
    // ---- the control replay of the ticks the chain smoothed in step k - 1,
    // on another wave than this step's chain, after its tally (the tile it
    // tallied no longer holds registers)
    if (ctl_s >= 0 && wave == (k + kWaves / 2) % kWaves) {
      __builtin_amdgcn_s_setprio(3);
      ctl_run((k + 1) % 3);
      __builtin_amdgcn_s_setprio(0);
    }
    // entries rotate over three steps: step k writes entry k % 3, every wave
    // reads it right after the barrier that ends step k, and it is reset
    // here in step k + 2 (a barrier after those reads, a barrier before its
    // next use in step k + 3)
    if (tid == 0) {
      const int r = (k + 1) % 3;
      s_defer[r] = kNoDefer;
      s_wdef[r] = INT_MAX;
      s_wlast[r] = -1;
    }
    __syncthreads();
    // ---- the next tile and the completeness bound (same on every thread;
    // shared scalars are read into scalar registers)
    const unsigned dfr = (unsigned)__builtin_amdgcn_readfirstlane((int)s_defer[b3]);
    int en = a0 + (int)kTile;
    if (en > rend) en = rend;
    if (en < e0) en = e0;
    int wn;
    if (dfr != kNoDefer) {
      en = a0 + dfr;
      wn = __builtin_amdgcn_readfirstlane(s_wdef[b3]);
    } else if (en >= rend) {
      wn = nW;
    } else {
      wn = __builtin_amdgcn_readfirstlane(s_wlast[b3]);
    }
    wn = wn > nW ? nW : wn;
    e0 = en;
    wl = wn < wl ? wl : wn;
    held = pref;
    cA = cB;
    cB = cC;
    return false;
  };
  int k_end = 0;
  for (int k = 0;; k += 2) {
    if (step(buf0, buf1, k)) {
      k_end = k;
      break;
    }
    if (step(buf1, buf0, k + 1)) {
      k_end = k + 1;
      break;
    }
  }
  if constexpr (kSeg) {  // the last step's barrier made every s_first visible
    const int K = (kStage ? 2 : 1) * M;
    for (int i = tid; i < K; i += kThreads)
      if (s_first[i] != kNoDefer) atomicMin(&p.first[(int64_t)trace * K + i], s_first[i]);
  }
  // the ticks of the last chunk, then the replay's outputs (the last step's
  // barrier made the chain's values visible)
  if (ctl_s >= 0 && wave == 0) {
    ctl_run((k_end + 1) % 3);
    if (lane < M) {
      const CtlModel cm = s_cm[lane];
      p.r_final[(int64_t)ctl_s * M + lane] = cm.R;
      p.r_windows[(int64_t)ctl_s * M + lane] = cm.rw + (long long)cm.R * (nW - cm.since);
    }
    if (lane == 0) p.n_moves[ctl_s] = s_cmeta[1];
  }
}

template <int kWaves, int kEPT, bool kCells>
__global__ __launch_bounds__(kWaves * 64) void tss_stream(StreamParams p) {
  stream_body<kWaves, kEPT, kCells, false>(p);
}

// ------------------------------------------------------- segmented path
// With few traces one workgroup per trace leaves most of the chip idle and
// pays the smoothing chain, the evaluation and the tally in turn at every
// step. There the windows of each trace are cut into segments:
//   seg_net       per (trace, segment): its rows by binary search in the
//                 sorted timestamps, and its net changes of the active and
//                 waiting counts per model;
//   tss_seg       per (trace, segment): stream_body with kSeg;
//   chain_smooth  per trace: the smoothing chain over the raw ratios, the
//                 per-cell outputs, the tick snapshot and, for a trace with
//                 one scenario, the control replay.
struct SegNetParams {
  const int64_t* ts;
  const uint8_t* model;
  const uint8_t* type;
  const int64_t* off;
  int64_t window_ms;
  int32_t M, nseg, seg_w;
  int32_t* seg_row;             // [trace][nseg + 1]
  unsigned long long* seg_net;  // [trace][nseg][M]
  uint32_t* first;              // [trace][K], set to "none" here
  int32_t K;
};

// first row in [0, n) whose timestamp is at or above t (n if none): the whole
// wave probes 64 rows a round, so a trace of 2^21 rows takes four rounds of
// one load latency instead of 21. Unsorted input gives some row of [0, n].
__device__ __forceinline__ int wave_lower_bound(const int64_t* ts, int n, int64_t t, int lane) {
  int lo = 0, len = n;  // the answer lies in [lo, lo + len]
  while (len > 0) {
    const int stp = (len + 64) / 65;  // probes lo + stp * (lane + 1) - 1, at most 64 of them inside
    const int at = lo + stp * (lane + 1) - 1;
    const bool below = at < lo + len && ts[at] < t;
    const int c = __popcll(__ballot(below));  // probes below t (a prefix when sorted)
    const int nlo = lo + stp * c;
    const int end = lo + stp * (c + 1) - 1;  // the first probe not below, or past the range
    const int nend = c < 64 && end < lo + len ? end : lo + len;
    len = nend > nlo ? nend - nlo : 0;
    lo = nlo;
  }
  return lo < n ? lo : n;
}

constexpr int kNetThreads = 256;

// bound by latency (the search's dependent probes) on short segments, by the
// 2 bytes per row on long ones; a row costs one LDS add only if it changes a
// count (about three in eleven)
__global__ __launch_bounds__(kNetThreads) void seg_net(SegNetParams p) {
  __shared__ unsigned long long s_net[4][TRE_MAX_MODELS];  // one copy per wave: fewer adds meet on one word
  __shared__ int s_row[2];
  const int trace = (int)(blockIdx.x / (unsigned)p.nseg), seg = (int)(blockIdx.x % (unsigned)p.nseg);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = p.off[trace], e = p.off[trace + 1];
  const int n = (int)(e - b);
  for (int i = tid; i < 4 * TRE_MAX_MODELS; i += kNetThreads) (&s_net[0][0])[i] = 0ull;
  if (wave < 2) {  // wave 0: the first row, wave 1: the end
    const int sg = seg + wave;
    int r = sg == 0 ? 0 : n;
    if (sg > 0 && sg < p.nseg) r = wave_lower_bound(p.ts + b, n, (int64_t)sg * p.seg_w * p.window_ms, lane);
    if (lane == 0) s_row[wave] = r;
  }
  if (seg == 0)
    for (int i = tid; i < p.K; i += kNetThreads) p.first[(int64_t)trace * p.K + i] = kNoDefer;
  __syncthreads();
  const int r0 = s_row[0], r1 = s_row[1] > r0 ? s_row[1] : r0;
  if (tid == 0) {
    // unsorted input may put a segment's first row after the next one's; each
    // workgroup then reads rows [own first, next first) or none
    int32_t* const sr = p.seg_row + (int64_t)trace * (p.nseg + 1);
    sr[seg] = r0;
    if (seg == p.nseg - 1) sr[p.nseg] = n;
  }
  // 16 rows per lane: 16-byte loads of the model and type bytes from the
  // first 4-aligned row (buffer loads: past the range they read zeros)
  const int64_t brow = (b + r0) & ~(int64_t)3;
  const int skip = (int)(b + r0 - brow), rend = skip + (r1 - r0);
  const __amdgpu_buffer_rsrc_t rm = rsrc(p.model + brow, rend), rt = rsrc(p.type + brow, rend);
  unsigned long long* const net = s_net[wave];
  const uint32_t mlast = (uint32_t)p.M - 1u;
  v4u32 m4, t4, mn, tn;
  m4 = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rm, tid * 16, 0, 0));
  t4 = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rt, tid * 16, 0, 0));
  for (int i0 = 0; i0 < rend; i0 += kNetThreads * 16) {
    const int i = i0 + tid * 16;
    mn = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rm, i + kNetThreads * 16, 0, 0));
    tn = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(rt, i + kNetThreads * 16, 0, 0));
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const uint32_t ty = (t4[j >> 2] >> (8 * (j & 3))) & 0xFFu;
      const uint32_t code = (ty & 3u) | ((ty >> 5) & 4u);  // as tally_row: 0 ARRIVE, 3 FINISH, 5 ADMIT
      if (((1u << code) & 0x29u) && i + j >= skip && i + j < rend) {
        uint32_t mdl = (m4[j >> 2] >> (8 * (j & 3))) & 0xFFu;
        mdl = mdl < mlast ? mdl : mlast;
        // ARRIVE: dW + 1; ADMIT: dA + 1, dW - 1; FINISH: dA - 1
        const unsigned long long d = code == 0u ? 1ull : code == 5u ? (1ull << 32) - 1ull : 0xFFFFFFFF00000000ull;
        atomicAdd(&net[mdl], d);
      }
    }
    m4 = mn;
    t4 = tn;
  }
  __syncthreads();
  if (tid < p.M)
    p.seg_net[((int64_t)trace * p.nseg + seg) * p.M + tid] = s_net[0][tid] + s_net[1][tid] + s_net[2][tid] + s_net[3][tid];
}

template <int kWaves, int kEPT, bool kStage>
__global__ __launch_bounds__(kWaves * 64) void tss_seg(StreamParams p) {
  stream_body<kWaves, kEPT, !kStage, kStage, true>(p);
}

struct ChainParams {
  const double* raw;       // [trace][column][window], -1 idle
  const uint32_t* first;   // [trace][column]
  const tre_profile* prof;
  int32_t n_windows, M;
  int32_t chunk_log2;      // windows per step: 2^chunk_log2, at least 8, chunk * columns <= kChainCells
  int32_t stride;          // LDS words of 8 bytes per window: 9, 17, 33, 65 or 129
  int32_t fast_w, slow_w, n_ticks;
  uint32_t magic_fast, magic_slow, magic_both;  // floor(2^32 / d), 2^32 - 1 for 1
  int32_t both_w;          // least common multiple of the two periods, or past the last window
  uint32_t magic_k;        // floor(2^20 / columns) + 1: cell / columns for cells below 2^10
  double* tss64;           // kStage: stage64
  float* tss32;            // kStage: stage32
  uint8_t* flags;
  double* snap;
  const uint32_t* tick_window;
  const uint8_t* tick_kind;
  // the control replay of a trace with one scenario
  const tre_scenario* sc;
  const uint32_t* sc_count;
  const uint32_t* sc_first;
  int32_t ctl_one;
  int32_t budget;
  tre_move* moves;
  uint32_t move_cap;
  uint32_t* n_moves;
  int32_t* r_final;
  int64_t* r_windows;
};

constexpr int kChainCells = 1024;       // cells per step
constexpr int kChainWindows = 128;      // windows per step at most
constexpr int kChainIO = 256;           // loading threads, and as many storing
constexpr int kChainPer = kChainCells / kChainIO;
constexpr int kChainRows = 16;          // columns up to which the chain runs in rows of 16 lanes
// chain waves: four of four columns each, or a lane per column
constexpr int chain_waves(bool rows) { return rows ? kChainRows / 4 : 2; }
constexpr int chain_threads(bool rows) { return 64 * (chain_waves(rows) + 1) + 2 * kChainIO; }

// S over C windows (a multiple of 8) of one column: S' = t1 + o * S with t1
// and o of window u at t[u * kStr] and t[plane + u * kStr]; S' is written over
// o. Two groups of windows in registers: the LDS reads of one (about 170
// cycles) are in flight while the other's dependent multiplies and adds (12.4
// cycles a window) run, and the stride is a constant, so that two windows
// share one LDS instruction.
template <int kStr>
__device__ __forceinline__ double chain_run(double* t, int plane, int C, double S) {
  constexpr int kG = 8;
  double qt[kG], qo[kG], rt[kG], ro[kG];
  double* o = t + plane;
  auto read = [&](double (&x)[kG], double (&y)[kG], int at) {
#pragma unroll
    for (int u = 0; u < kG; ++u) x[u] = t[at + u * kStr];
#pragma unroll
    for (int u = 0; u < kG; ++u) y[u] = o[at + u * kStr];
  };
  auto run = [&](const double (&x)[kG], const double (&y)[kG]) {
#pragma unroll
    for (int u = 0; u < kG; ++u) {
      const double t2 = y[u] * S;
      S = x[u] + t2;
      o[u * kStr] = S;
    }
    t += kG * kStr;
    o += kG * kStr;
  };
  read(qt, qo, 0);
  int u0 = 0;
  for (; u0 + 2 * kG <= C; u0 += 2 * kG) {
    read(rt, ro, kG * kStr);
    run(qt, qo);
    read(qt, qo, u0 + 2 * kG < C ? kG * kStr : 0);  // past the chunk: read, not used
    run(rt, ro);
  }
  if (u0 < C) run(qt, qo);
  return S;
}

// The same for up to four columns a wave, one row of 16 lanes each, lane u of
// a row at window u0 + u of its column's plane: S moves one lane to the right
// per window (DPP row_shr; lane 0 keeps the S of the row's last lane from the
// block before). Every lane recomputes its own S at every step, and from step
// u on lane u's is right. One LDS read of t1 and of o and one write of S per
// 16 windows instead of 16 half-empty ones, whose cost does not fall with the
// lanes in use: in a loop of their own 25.9 cycles a window against 45 with a
// lane per column; 33 in the kernel, beside its other waves (7200 windows of 8
// models 101 us).
__device__ __forceinline__ double chain_rows(double* t, int plane, int str, int C, double S) {
  double t1 = t[0], o = t[plane];
  for (int u0 = 0; u0 < C; u0 += 16) {
    const int nx = u0 + 16 < C ? 16 * str : 0;
    const double tn = t[nx], on = t[plane + nx];
    auto lo = [](double x) { return (int)(uint32_t)dbits(x); };
    auto hi = [](double x) { return (int)(uint32_t)(dbits(x) >> 32); };
    auto of = [](int l, int h) { return __longlong_as_double((long long)(((unsigned long long)(uint32_t)h << 32) | (uint32_t)l)); };
    int pl = __builtin_amdgcn_update_dpp(0, lo(S), 0x121, 0xF, 0xF, false);  // row_ror:1
    int ph = __builtin_amdgcn_update_dpp(0, hi(S), 0x121, 0xF, 0xF, false);
    double t2 = o * of(pl, ph);
    S = t1 + t2;
#pragma unroll
    for (int u = 1; u < 16; ++u) {
      pl = __builtin_amdgcn_update_dpp(pl, lo(S), 0x111, 0xF, 0xF, false);  // row_shr:1
      ph = __builtin_amdgcn_update_dpp(ph, hi(S), 0x111, 0xF, 0xF, false);
      t2 = o * of(pl, ph);
      S = t1 + t2;
    }
    t[plane] = S;
    t += nx;
    t1 = tn;
    o = on;
  }
  return S;
}

// t1 of an idle window: -0.0, which no other window has (alpha * raw of a raw
// ratio >= 0 is +0.0 or more, or a NaN of either sign); the high word tells
__device__ __forceinline__ bool idle_t1(double t1) { return (uint32_t)(dbits(t1) >> 32) == 0x80000000u; }

// One workgroup per trace, waves of four kinds that meet at one barrier per
// step of `chunk` windows. A column is a model (kStage: a model's prefill or
// decode share). In step k
//   the loading waves put chunk k + 1 into LDS: per cell the t1 of S' = t1 +
//     o * S, the smoothing of its window, and o: alpha * raw and 1 - alpha;
//     raw at the column's first busy window, where S is still 0; -0.0 and 1
//     at an idle one: the same binary64 operations on the same values as the
//     documented order, and S itself where it is held. Their global loads run
//     two chunks further ahead;
//   the chain waves (kRows: a row of lanes per column, else a lane) run S over chunk k, one multiply and one
//     add per window, writing S over o;
//   the storing waves write the per-cell outputs of chunk k - 1, and prepare
//     its ticks for the replay (or store them for a separate one);
//   the control wave replays the ticks of chunk k - 2.
// Bound by the dependent multiply-add of each window: everything else a
// window needs is on other waves.
template <bool kStage, bool kRows>
__global__ __launch_bounds__(chain_threads(kRows), kRows ? 7 : 5) void chain_smooth(ChainParams p) {
  constexpr int kChainWaves = chain_waves(kRows), kChainThreads = chain_threads(kRows);
  extern __shared__ __align__(16) double cbuf[];  // [3][t1, then o and S][windows][stride]
  __shared__ uint32_t s_first[2 * TRE_MAX_MODELS];
  // the prepared ticks of a chunk (at most its windows), by step parity
  __shared__ uint32_t s_recv[2][kStage ? 1 : kChainCells], s_don[2][kStage ? 1 : kChainCells];
  __shared__ uint32_t s_head[2][kStage ? 1 : kChainWindows];
  __shared__ unsigned long long s_z[kStage ? 1 : kChainIO / 64][64];
  const int trace = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = p.M, K = kStage ? 2 * M : M, nW = p.n_windows;
  const int lg = p.chunk_log2, C = 1 << lg;
  const int str = p.stride;  // odd, so that a column's windows spread over the banks
  const int plane = C * str, bufn = 2 * plane;
  const int steps = (nW + C - 1) >> lg;
  for (int i = tid; i < K; i += kChainThreads) s_first[i] = p.first[(int64_t)trace * K + i];
  // the trace's one scenario, replayed here (else -1)
  int ctl_s = -1;
  if (!kStage) {
    if (p.ctl_one) ctl_s = 0;
    else if (p.sc_count && p.sc_count[trace] == 1u) ctl_s = (int)p.sc_first[trace];
  }
  ctl_s = __builtin_amdgcn_readfirstlane(ctl_s);
  // ticks among the windows before w
  auto ticks_before = [&](int w) {
    return (int)(div_magic((uint32_t)w, (uint32_t)p.fast_w, p.magic_fast) +
                 div_magic((uint32_t)w, (uint32_t)p.slow_w, p.magic_slow) -
                 div_magic((uint32_t)w, (uint32_t)p.both_w, p.magic_both));
  };
  const bool act = lane < M;
  const int m = act ? lane : 0;
  __syncthreads();

  if (wave >= kChainWaves + 1 && wave < kChainWaves + 1 + kChainIO / 64) {
    // ---- loading waves
    const int l = tid - 64 * (kChainWaves + 1);
    double al[kChainPer], om[kChainPer];
    int fst[kChainPer], dst[kChainPer], win[kChainPer];
    const double* src[kChainPer];
#pragma unroll
    for (int j = 0; j < kChainPer; ++j) {
      const int i = l + kChainIO * j, col = i >> lg, u = i & (C - 1);
      const bool in = col < K;
      al[j] = in ? p.prof[(int64_t)trace * M + (kStage ? col >> 1 : col)].alpha : 0.0;
      om[j] = 1.0 - al[j];
      fst[j] = in ? (int)s_first[col] - u : 0;  // the chunk's first window with which u is the first busy one
      dst[j] = in ? u * str + col : -1;
      win[j] = u;
      src[j] = p.raw + ((int64_t)trace * K + (in ? col : 0)) * nW;
    }
    // no branch around a load, so that a wait covers only the older chunk's
    auto load = [&](double (&v)[kChainPer], int k) {
#pragma unroll
      for (int j = 0; j < kChainPer; ++j) {
        const int w = (k << lg) + win[j];
        v[j] = src[j][w < nW ? w : nW - 1];
      }
    };
    auto put = [&](const double (&v)[kChainPer], int k) {
      double* const b = cbuf + (k % 3) * bufn;
      const int w0 = k << lg;
#pragma unroll
      for (int j = 0; j < kChainPer; ++j) {
        const bool idle = v[j] < 0.0;
        const double a = al[j] * v[j];
        if (dst[j] >= 0) {
          b[dst[j]] = idle ? -0.0 : (w0 == fst[j] ? v[j] : a);
          b[plane + dst[j]] = idle ? 1.0 : om[j];
        }
      }
    };
    double va[kChainPer], vb[kChainPer];
    load(va, 0);
    load(vb, 1);
    put(va, 0);
    load(va, 2);
    __syncthreads();
    for (int k = 0; k <= steps + 1; k += 2) {  // vb holds chunk k + 1, va chunk k + 2
      if (k + 1 < steps) put(vb, k + 1);
      load(vb, k + 3);
      __syncthreads();
      if (k > steps) break;
      if (k + 2 < steps) put(va, k + 2);
      load(va, k + 4);
      __syncthreads();
    }
  } else if (wave < kChainWaves) {
    // ---- chain waves
    const int col = kRows ? wave * 4 + (lane >> 4) : tid;
    const bool own = col < K;
    double S = 0.0;
    __builtin_amdgcn_s_setprio(3);
    __syncthreads();
    for (int k = 0; k <= steps + 1; ++k) {
      double* const b = cbuf + (k % 3) * bufn + col;
      if constexpr (kRows) {
        if (k < steps && wave * 4 < K && own) S = chain_rows(b + (lane & 15) * str, plane, str, C, S);
      } else if (k < steps && own) {
        if (str == 33) S = chain_run<33>(b, plane, C, S);
        else if (str == 65) S = chain_run<65>(b, plane, C, S);
        else S = chain_run<129>(b, plane, C, S);
      }
      __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
  } else if (wave == kChainWaves) {
    // ---- control wave: the prepared ticks of chunk k - 2
    OrdState st{};
    OrdConst c{};
    c.n_windows = nW;
    c.act = act;
    if (ctl_s >= 0) {
      const tre_profile pr = p.prof[(int64_t)trace * M + m];
      c.r_min = pr.r_min;
      c.K = (uint32_t)__builtin_amdgcn_readfirstlane((int)p.sc[ctl_s].max_moves);
      c.moves = p.moves + (int64_t)ctl_s * p.move_cap;
      c.move_cap = p.move_cap;
      ord_init(st, c, pr.r_init, 1, p.budget);
    }
    __builtin_amdgcn_s_setprio(2);
    __syncthreads();
    for (int k = 0; k <= steps + 1; ++k) {
      if (!kStage && k > 1 && ctl_s >= 0) {
        const int w0 = (k - 2) << lg, we = w0 + C < nW ? w0 + C : nW;
        ctl_batch<false>(st, c, lane, M, ticks_before(we) - ticks_before(w0), s_recv[k & 1], s_don[k & 1],
                         s_head[k & 1], nullptr, [](int) { return 0ull; });
      }
      __syncthreads();
    }
    if (!kStage && ctl_s >= 0)
      ord_finish<false>(st, c, lane, p.r_final + (int64_t)ctl_s * M, p.r_windows + (int64_t)ctl_s * M,
                        p.n_moves + ctl_s);
  } else {
    // ---- storing waves: cells in output order, so that stores are contiguous
    const int l = tid - 64 * (kChainWaves + 1) - kChainIO;
    const bool vals = p.tss64 || p.tss32;
    const int wv = wave - (kChainWaves + 1) - kChainIO / 64;  // storing wave
    // ticks: lanes in groups of 2^lt, one group per tick, sub-lane = model
    int lt = 0;
    while ((1 << lt) < M) ++lt;
    const int per = 64 >> lt, sub = lane & ((1 << lt) - 1);  // ticks a wave takes at once
    const int ms = sub < M ? sub : 0;
    const int fst = (int)s_first[kStage ? 0 : ms];
    const bool ticks = !kStage && (ctl_s >= 0 || p.snap);
    double th = 1.0, tau_c = 0.0, tau_s = 0.0;
    if (!kStage && ctl_s >= 0) {
      const tre_scenario sc = p.sc[ctl_s];
      const tre_profile pr = p.prof[(int64_t)trace * M + ms];
      th = pr.theta * sc.theta_scale;
      tau_c = sc.tau_crit_override >= 0.0 ? sc.tau_crit_override : pr.tau_crit;
      tau_s = pr.tau_surplus;
    }
    // the window and kind of tick `t`, clamped (read a step ahead)
    auto tick_at = [&](int t) {
      t = t < p.n_ticks ? t : p.n_ticks - 1;
      return p.n_ticks > 0 ? p.tick_window[t] | ((uint32_t)p.tick_kind[t] << 30) : 0u;
    };
    const int mine = wv * per + (lane >> lt);  // this lane's tick among a round's
    int t0 = 0;                                // ticks before the chunk
    uint32_t twn = ticks ? tick_at(mine) : 0u;
    __syncthreads();
    for (int k = 0; k <= steps + 1; ++k) {
      const int w0 = (k - 1) << lg;
      const int n = w0 + C < nW ? C : nW - w0;
      const double* const b = cbuf + ((k + 2) % 3) * bufn;  // chunk k - 1
      if (ticks && k > 0 && k <= steps) {
        const int nt = ticks_before(w0 + n) - t0;
        uint32_t tw = twn;
        twn = tick_at(t0 + nt + mine);
        for (int i0 = 0; i0 < nt; i0 += 4 * per) {
          const int i = i0 + mine;
          if (i0) tw = tick_at(t0 + i);
          const bool in = i < nt;
          const int w = (int)(tw & 0x3FFFFFFFu);
          const int u = in ? w - w0 : 0;
          const double t1 = b[u * str + ms], Sw = b[plane + u * str + ms];
          const bool dead = idle_t1(t1) || w < fst || fst < 0;  // idle, or not initialised
          if (ctl_s >= 0) {
            const double Z = in && sub < M && !dead ? Sw / th : INFINITY;  // Eq. (2)
            const int e = in ? i : 0;
            tick_order(&s_recv[(k + 1) & 1][e * M], &s_don[(k + 1) & 1][e * M], &s_head[(k + 1) & 1][e], s_z[wv], lane, lt, M,
                       in, Z, tau_c, tau_s, (uint32_t)w, tw >> 30);
          } else if (in && sub < M) {
            p.snap[((int64_t)trace * p.n_ticks + t0 + i) * M + sub] = dead ? INFINITY : Sw;
          }
        }
        t0 += nt;
      }
      if (k > 0 && k <= steps && (vals || p.flags)) {
        const int64_t o = ((int64_t)trace * nW + w0) * K;
        for (int i = l; i < n * K; i += kChainIO) {
          const int u = (int)(((uint32_t)i * p.magic_k) >> 20), col = i - u * K;
          const double t1 = b[u * str + col], Sw = b[plane + u * str + col];
          if (p.tss64) p.tss64[o + i] = Sw;
          if (p.tss32) p.tss32[o + i] = (float)Sw;
          if (!kStage && p.flags) {
            const bool idle = idle_t1(t1), init = (uint32_t)(w0 + u) >= s_first[col];
            p.flags[o + i] = (uint8_t)((idle ? TRE_FLAG_IDLE : 0) | (init ? TRE_FLAG_INIT : 0));
          }
        }
        if (kStage && p.flags) {
          const int64_t of = ((int64_t)trace * nW + w0) * M;
          for (int i = l; i < n * M; i += kChainIO) {
            const int u = (int)(((uint32_t)(2 * i) * p.magic_k) >> 20), col = 2 * (i - u * M);
            const bool pi = idle_t1(b[u * str + col]), di = idle_t1(b[u * str + col + 1]);
            const uint32_t w = (uint32_t)(w0 + u);
            p.flags[of + i] = (uint8_t)((pi ? TRE_STAGE_P_IDLE : 0) |
                                        (w >= s_first[col] ? TRE_STAGE_P_INIT : 0) |
                                        (di ? TRE_STAGE_D_IDLE : 0) |
                                        (w >= s_first[col + 1] ? TRE_STAGE_D_INIT : 0));
          }
        }
      }
      __syncthreads();
    }
  }
}

// the stage-share instantiation, held to 80 VGPRs so that six workgroups
// fit on a CU (its LDS allows six)
template <int kWaves, int kEPT>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(6))) void tss_stream_stage(
    StreamParams p) {
  stream_body<kWaves, kEPT, false, true>(p);
}

// --------------------------------------------------------------- rebalance
struct CtlParams {
  const tre_profile* prof;
  const tre_scenario* sc;
  uint32_t n_sc;
  const double* vals;     // snapshot [trace][tick][M] (flags NULL) or S [trace][w][M]
  const uint8_t* flags;   // per-cell flags, or NULL
  const uint32_t* tick_window;
  const uint8_t* tick_kind;  // bit 0 fast, bit 1 slow
  int32_t n_ticks;
  int32_t n_windows;
  int32_t M;
  int32_t budget;
  uint32_t n_traces;
  tre_move* moves;
  uint32_t move_cap;
  uint32_t* n_moves;
  int32_t* r_final;
  int64_t* r_windows;
  // actuation model (the kAct instantiation)
  int32_t wake_w;            // windows from a wake's start until routable
  int32_t sleep_w;           // windows a released replica hides, drains and sleeps
  const int32_t* footprint;  // [trace][M] GPUs per replica, or NULL (1)
  const uint64_t* veto;      // [trace][tick] donor releases refused, or NULL
  const uint32_t* sc_count;  // [trace] scenarios per trace of a sweep, or NULL
};

// One wave per scenario, lane m = model m: per tick Z = S / (theta * scale)
// (Eq. (2)), then ctl_tick. Scenarios whose trace streamed its own replay
// (sc_count[trace] == 1 in a sweep) are skipped.
template <bool kAct>
__global__ __launch_bounds__(256) void rebalance(CtlParams p) {
  const int lane = threadIdx.x & 63;
  const uint32_t s = (uint32_t)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (s >= p.n_sc) return;  // whole wave
  const int M = p.M;
  const bool act = lane < M;
  const int mc = act ? lane : 0;
  const tre_scenario sc = p.sc[s];
  const uint32_t trace = sc.trace < p.n_traces ? sc.trace : 0;
  if (p.sc_count && p.sc_count[trace] == 1u) return;  // replayed in the stream
  const tre_profile pr = p.prof[(int64_t)trace * M + mc];
  const double theta_eff = pr.theta * sc.theta_scale;
  CtlConst c;
  c.tau_c = sc.tau_crit_override >= 0.0 ? sc.tau_crit_override : pr.tau_crit;
  c.tau_s = pr.tau_surplus;
  c.r_min = pr.r_min;
  c.K = sc.max_moves;
  c.act = act;
  c.live_lanes = __ballot(act);
  c.wake_w = p.wake_w;
  c.sleep_w = p.sleep_w;
  c.moves = p.moves + (int64_t)s * p.move_cap;
  c.move_cap = p.move_cap;
  int g = 1;
  if (kAct && p.footprint && act) g = p.footprint[(int64_t)trace * M + lane];
  CtlState st;
  ctl_init(st, pr.r_init, g, act, p.budget);

  const int nt = p.n_ticks;
  const int64_t tbase = (int64_t)trace * (p.flags ? p.n_windows : nt);
  // normalised values of ticks [t0, t0 + kTickBlock): unconditional loads
  // from clamped indices, then the divisions, independent of each other
  // (the tick's window, kind and vetoes ride along: loads that other
  // threads' stores might alias stay vector loads, so they are issued a
  // block ahead)
  auto load_block = [&](int t0, double (&v)[kTickBlock], uint32_t (&f)[kTickBlock],
                        uint32_t (&tw)[kTickBlock], unsigned long long (&vt)[kTickBlock]) {
#pragma unroll
    for (int u = 0; u < kTickBlock; ++u) {
      const int t = t0 + u < nt ? t0 + u : nt - 1;
      tw[u] = p.tick_window[t] | ((uint32_t)p.tick_kind[t] << 30);
      vt[u] = (kAct && p.veto) ? p.veto[(int64_t)trace * nt + t] : 0ull;
      if (p.flags) {
        const int64_t cc = (tbase + p.tick_window[t]) * M + mc;
        v[u] = p.vals[cc];
        f[u] = p.flags[cc];
      } else {
        v[u] = p.vals[(tbase + t) * M + mc];
        f[u] = TRE_FLAG_INIT;
      }
    }
  };
  auto normalise = [&](double (&v)[kTickBlock], const uint32_t (&f)[kTickBlock]) {
#pragma unroll
    for (int u = 0; u < kTickBlock; ++u) {
      const bool live = act && !(f[u] & TRE_FLAG_IDLE) && (f[u] & TRE_FLAG_INIT);
      v[u] = live ? v[u] / theta_eff : INFINITY;  // Eq. (2); +inf when idle or not initialised
    }
  };
  auto decide = [&](uint32_t twk, double Z, unsigned long long vetoed) {
    ctl_tick<kAct>(st, c, lane, (uint32_t)__builtin_amdgcn_readfirstlane((int)twk), Z, vetoed);
  };
  if (nt > 0) {
    double va[kTickBlock], vb[kTickBlock];
    uint32_t fa[kTickBlock], fb[kTickBlock], wa[kTickBlock], wb[kTickBlock];
    unsigned long long xa[kTickBlock], xb[kTickBlock];
    load_block(0, va, fa, wa, xa);
    for (int t0 = 0; t0 < nt; t0 += 2 * kTickBlock) {
      load_block(t0 + kTickBlock, vb, fb, wb, xb);
      normalise(va, fa);
#pragma unroll
      for (int u = 0; u < kTickBlock; ++u)
        if (t0 + u < nt) decide(wa[u], va[u], xa[u]);
      load_block(t0 + 2 * kTickBlock, va, fa, wa, xa);
      normalise(vb, fb);
#pragma unroll
      for (int u = 0; u < kTickBlock; ++u)
        if (t0 + kTickBlock + u < nt) decide(wb[u], vb[u], xb[u]);
    }
  }
  ctl_complete<kAct>(st, p.n_windows);  // transitions completing at the end of the last window count as done
  st.rw += (long long)st.R * (p.n_windows - st.since);
  if (act) {
    p.r_final[(int64_t)s * M + lane] = st.R;
    p.r_windows[(int64_t)s * M + lane] = st.rw;
  }
  if (lane == 0) p.n_moves[s] = st.nm;
}

// The same replay with one workgroup per scenario: kOrdWaves waves prepare the
// ticks of the next batch (tick_order), eight each, while one more decides those
// of the batch before it.
template <bool kAct, int kOrdWaves>
__global__ __launch_bounds__(64 * (kOrdWaves + 1)) void rebalance_ordered(CtlParams p) {
  constexpr int kOrdBatch = 8 * kOrdWaves;  // at most 64: a lane per tick holds its vetoes
  __shared__ uint32_t s_recv[2][kOrdBatch * TRE_MAX_MODELS], s_don[2][kOrdBatch * TRE_MAX_MODELS];
  __shared__ uint32_t s_head[2][kOrdBatch];
  __shared__ unsigned long long s_z[kOrdWaves][64];
  __shared__ int s_g[TRE_MAX_MODELS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const uint32_t s = blockIdx.x;
  const int M = p.M;
  const tre_scenario sc = p.sc[s];
  const uint32_t trace = sc.trace < p.n_traces ? sc.trace : 0;
  if (p.sc_count && p.sc_count[trace] == 1u) return;  // replayed in the stream (whole workgroup)
  const int nt = p.n_ticks;
  const int nb = (nt + kOrdBatch - 1) / kOrdBatch;
  if (wave == 0) {
    const tre_profile pr = p.prof[(int64_t)trace * M + (lane < M ? lane : 0)];
    OrdConst c;
    c.r_min = pr.r_min;
    c.K = (uint32_t)__builtin_amdgcn_readfirstlane((int)sc.max_moves);
    c.act = lane < M;
    c.n_windows = p.n_windows;
    c.wake_w = p.wake_w;
    c.sleep_w = p.sleep_w;
    c.moves = p.moves + (int64_t)s * p.move_cap;
    c.move_cap = p.move_cap;
    int g = 1;
    if (kAct && p.footprint && c.act) g = p.footprint[(int64_t)trace * M + lane];
    s_g[lane] = g;  // read by this wave only
    OrdState st;
    ord_init(st, c, pr.r_init, g, p.budget);
    // lane i: the vetoes of tick i of a batch, read a batch ahead
    auto vetoes = [&](int b) {
      const int t = b * kOrdBatch + lane;
      return (kAct && p.veto && lane < kOrdBatch && t < nt) ? p.veto[(int64_t)trace * nt + t] : 0ull;
    };
    unsigned long long vt = 0, vn = vetoes(0);
    __builtin_amdgcn_s_setprio(3);  // the workgroup waits for this wave
    for (int b = 0; b <= nb; ++b) {
      if (b > 0) {
        const int t0 = (b - 1) * kOrdBatch;
        ctl_batch<kAct>(st, c, lane, M, nt - t0 < kOrdBatch ? nt - t0 : kOrdBatch, s_recv[(b + 1) & 1],
                        s_don[(b + 1) & 1], s_head[(b + 1) & 1], s_g, [&](int i) {
                          if (!kAct) return 0ull;
                          return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)vt, i) |
                                 ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(vt >> 32), i) << 32);
                        });
      }
      vt = vn;
      vn = vetoes(b + 1);
      __syncthreads();
    }
    ord_finish<kAct>(st, c, lane, p.r_final + (int64_t)s * M, p.r_windows + (int64_t)s * M, p.n_moves + s);
  } else {
    int lg = 0;
    while ((1 << lg) < M) ++lg;
    const int per = (64 >> lg) < 8 ? 64 >> lg : 8;  // ticks a wave takes at once, of its 8 per batch
    const int sub = lane & ((1 << lg) - 1), tk = lane >> lg;
    const int mc = sub < M ? sub : 0;
    const tre_profile pr = p.prof[(int64_t)trace * M + mc];
    const double theta_eff = pr.theta * sc.theta_scale;
    const double tau_c = sc.tau_crit_override >= 0.0 ? sc.tau_crit_override : pr.tau_crit;
    const int64_t tbase = (int64_t)trace * (p.flags ? p.n_windows : nt);
    // round r of the wave: ticks at(r) + [0, per), one per lane group
    const int rounds = 8 / per;
    auto at = [&](int r) { return (r / rounds) * kOrdBatch + (wave - 1) * 8 + (r % rounds) * per + tk; };
    // unconditional loads from clamped indices, a round (the tick's place in
    // the log: two) ahead of their use
    auto place = [&](int r) {
      int t = at(r);
      t = t < nt ? t : nt - 1;
      return p.tick_window[t] | ((uint32_t)p.tick_kind[t] << 30);
    };
    auto value = [&](int r, uint32_t tw, uint32_t& f) {
      int t = at(r);
      t = t < nt ? t : nt - 1;
      f = TRE_FLAG_INIT;
      if (!p.flags) return p.vals[(tbase + t) * M + mc];
      const int64_t cc = (tbase + (tw & 0x3FFFFFFFu)) * M + mc;
      f = p.flags[cc];
      return p.vals[cc];
    };
    uint32_t tw = 0, tn = 0, f = 0;
    double v = 0.0;
    if (nb > 0) {
      tw = place(0);
      tn = place(1);
      v = value(0, tw, f);
    }
    for (int b = 0; b <= nb; ++b) {
      if (b < nb) {
        for (int r = b * rounds; r < (b + 1) * rounds; ++r) {
          uint32_t fn;
          const double vn = value(r + 1, tn, fn);
          const uint32_t t2 = place(r + 2);
          const bool live = sub < M && !(f & TRE_FLAG_IDLE) && (f & TRE_FLAG_INIT);
          const double Z = live ? v / theta_eff : INFINITY;  // Eq. (2); +inf when idle or not initialised
          const int t = at(r);
          const bool in = t < nt && tk < per;
          const int e = in ? t - b * kOrdBatch : 0;
          tick_order(&s_recv[b & 1][e * M], &s_don[b & 1][e * M], &s_head[b & 1][e], s_z[wave - 1], lane, lg, M, in, Z,
                     tau_c, pr.tau_surplus, tw & 0x3FFFFFFFu, tw >> 30);
          v = vn;
          f = fn;
          tw = tn;
          tn = t2;
        }
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------- validate
// Error kinds of the load-time checks, one bit and one lowest-row slot each.
enum { kValOrder = 0, kValSchema = 1, kValRange = 2, kValState = 3, kValKinds = 4 };

struct ValParams {
  const int64_t* ts;
  const uint8_t* model;
  const uint32_t* req;  // or NULL
  const uint8_t* type;
  const int64_t* off;
  const uint64_t* sub_off;   // [n_traces + 1] pieces of the traces before each
  int64_t sub_rows;          // rows of a piece
  uint32_t n_traces;
  int64_t duration_ms;
  int64_t window_ms;
  int32_t M;
  int64_t max_per_window;
  unsigned* err;             // bit k: an error of kind k
  unsigned long long* first; // [kValKinds] lowest failing row of each kind
  unsigned long long* net;   // per trace [M][pieces]: net changes of the counts in each piece
  uint2* sub_max;            // [all pieces] largest id of an admission, of an ARRIVE or FINISH row
};

// A trace's rows in pieces of kSubRows, one wave each: few traces then still
// fill the chip (4 traces of 1.9 M rows are 3760 waves). Pieces double until
// at most kMaxSubs (and one per trace) are left, which bounds the memory of
// their counts (8 bytes a model each) and still fills every SIMD.
constexpr int kSubRows = 2048;
constexpr uint64_t kMaxSubs = 16384;

// One pass over the rows: order, schema and per-window range of each row, the
// net change of each model's active and waiting counts over each piece (for
// validate_state), and the largest ids (they size the id tables). Bound by
// the 14 bytes a row; the windows of a row and of the one max_per_window
// later are divided out only when less than a window apart (two 64-bit
// divisions a row cost 30 of 85 us on 7.7 M rows).
__global__ __launch_bounds__(256) void validate(ValParams p) {
  __shared__ unsigned long long s_net[4][TRE_MAX_MODELS];
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
  for (uint32_t t = blockIdx.y; t < p.n_traces; t += gridDim.y) {
    const int64_t b = p.off[t], e = p.off[t + 1];
    const int64_t c0 = b + ((int64_t)blockIdx.x * 4 + wv) * p.sub_rows;
    if (c0 >= e) continue;  // whole wave; the waves share no barrier
    const int64_t c1 = c0 + p.sub_rows < e ? c0 + p.sub_rows : e;
    unsigned long long* const net = s_net[wv];
    net[lane] = 0ull;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint32_t mxa = 0, mxl = 0;
    constexpr int kU = 4;  // rows a lane loads before it uses any
    for (int64_t i0 = c0 + lane; i0 < c1; i0 += 64 * kU) {
      int64_t tv[kU], tp[kU], tj[kU];
      uint32_t ty[kU], md[kU], id[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t i = i0 + 64 * u < c1 ? i0 + 64 * u : c1 - 1;  // past the piece, its last row again
        tv[u] = p.ts[i];
        tp[u] = p.ts[i > b ? i - 1 : b];
        tj[u] = p.ts[i + p.max_per_window < e ? i + p.max_per_window : e - 1];
        ty[u] = p.type[i];
        md[u] = p.model[i];
        id[u] = p.req ? p.req[i] : 0u;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t i = i0 + 64 * u;
        if (i >= c1) break;
        const int64_t t_i = tv[u];
        unsigned bad = 0;
        if (t_i < 0 || t_i >= p.duration_ms || t_i < tp[u]) bad |= 1u << kValOrder;
        if (md[u] >= (uint32_t)p.M || (ty[u] & 0x7Cu) || ((ty[u] & TRE_ADMIT) && (ty[u] & 3u) != TRE_PREFILL))
          bad |= 1u << kValSchema;
        if (!(bad & (1u << kValOrder)) && i + p.max_per_window < e && tj[u] < t_i + p.window_ms &&
            tj[u] / p.window_ms == t_i / p.window_ms)
          bad |= 1u << kValRange;
        if (bad) {
          atomicOr(p.err, bad);
          for (int k = 0; k < kValState; ++k)
            if (bad & (1u << k)) atomicMin(&p.first[k], (unsigned long long)i);
        }
        const uint32_t kind = ty[u] & 3u;
        const bool admit = ty[u] == (TRE_PREFILL | TRE_ADMIT);
        if (admit) mxa = id[u] > mxa ? id[u] : mxa;
        if (kind == TRE_ARRIVE || kind == TRE_FINISH) mxl = id[u] > mxl ? id[u] : mxl;
        // counts as validate_state reads them: waiting in the low word, active in the high one
        const bool arrive = ty[u] == TRE_ARRIVE, finish = ty[u] == TRE_FINISH;
        if (arrive || admit || finish)
          atomicAdd(&net[md[u] & 63u],
                    arrive ? 1ull : admit ? (1ull << 32) - 1ull : 0xFFFFFFFF00000000ull);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t so = p.sub_off[t], n_sub = p.sub_off[t + 1] - so, sub = (uint64_t)blockIdx.x * 4 + wv;
    if (lane < p.M) p.net[so * p.M + (uint64_t)lane * n_sub + sub] = net[lane];
    if (p.req) {
      for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t oa = (uint32_t)__shfl_xor((int)mxa, d), ol = (uint32_t)__shfl_xor((int)mxl, d);
        mxa = oa > mxa ? oa : mxa;
        mxl = ol > mxl ? ol : mxl;
      }
      if (lane == 0) p.sub_max[so + sub] = make_uint2(mxa, mxl);
    }
  }
}

// the pieces' net changes of each (trace, model) into the counts before each
// piece, in place: one wave per model at a time, 64 pieces a step; one more
// wave's turn takes the largest ids of the trace (an atomicMax of every piece
// on the trace's words held `validate` back: 7.7 M rows 154 us against 27)
__global__ __launch_bounds__(256) void net_scan(unsigned long long* net, const uint64_t* sub_off, uint32_t n_traces,
                                                int M, const uint2* sub_max, uint32_t* max_admit, uint32_t* max_life) {
  const int wv = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  for (uint32_t t = blockIdx.x; t < n_traces; t += gridDim.x) {
    const uint64_t so = sub_off[t], n = sub_off[t + 1] - so;
    for (int m = (int)blockIdx.y * 4 + wv; m < M + (sub_max ? 1 : 0); m += 4 * (int)gridDim.y) {
      if (m == M) {
        uint32_t a = 0, l = 0;
        for (uint64_t k = lane; k < n; k += 64) {
          const uint2 v = sub_max[so + k];
          a = v.x > a ? v.x : a;
          l = v.y > l ? v.y : l;
        }
        for (int d = 32; d >= 1; d >>= 1) {
          const uint32_t oa = (uint32_t)__shfl_xor((int)a, d), ol = (uint32_t)__shfl_xor((int)l, d);
          a = oa > a ? oa : a;
          l = ol > l ? ol : l;
        }
        if (lane == 0) {
          max_admit[t] = a;
          max_life[t] = l;
        }
        break;
      }
      unsigned long long* const x = net + so * M + (uint64_t)m * n;
      unsigned long long carry = 0ull;
      for (uint64_t k0 = 0; k0 < n; k0 += 64) {
        const bool in = k0 + lane < n;
        const unsigned long long v = in ? x[k0 + lane] : 0ull;
        unsigned long long incl = v;
        for (int o = 1; o < 64; o <<= 1) {
          const unsigned long long u = __shfl_up(incl, o);
          if (lane >= o) incl += u;
        }
        if (in) x[k0 + lane] = carry + incl - v;
        carry += __shfl(incl, 63);
      }
    }
  }
}

// A_m(t) and W_m(t) of Eq. (1) count active and waiting requests, so a
// stream whose transitions take either below zero at some instant is
// invalid. They are right-continuous step functions: the value at t counts
// every row with ts <= t, so only the counts after the last row of an
// instant are checked (rows of one instant may come in any order). For
// model m that is the count after its last row with that timestamp.
//
// One wave per piece of a trace, 64 rows per step, one per lane, from the
// counts before the piece (net_scan); it does nothing where rows failed the other
// checks (an instant could then be a whole trace, and every piece would read on
// to its end). Rows of the same model are found with ballots over the
// model's bits; a lane's count is its model's carry plus the signed
// transitions of the same-model lanes up to it. A row whose next same-model
// row in the step has a later timestamp is the last of its instant and is
// checked at once; the model's last row of a step is checked when the
// model's next row (in a later step) has a later timestamp, or at the end of
// the piece, unless the rows after the piece go on with the model at the same
// instant. Per-model state (carries, the timestamp and row of the last row
// seen) lives in the wave's LDS slice. A step is a chain of ballots and LDS
// round trips (about 0.8 us alone), so it is the waves in flight that count:
// one wave per trace took 24.0 ms on 4 traces of 1.9 M rows.
struct StateParams {
  const int64_t* ts;
  const uint8_t* model;
  const uint8_t* type;
  const int64_t* off;
  const uint64_t* sub_off;
  int64_t sub_rows;
  const unsigned long long* net;
  uint32_t n_traces;
  int32_t M;
  unsigned* err;
  unsigned long long* first;
};

__global__ __launch_bounds__(256) void validate_state(StateParams p) {
  __shared__ int s_a[4][TRE_MAX_MODELS], s_w[4][TRE_MAX_MODELS];  // counts after the rows seen
  __shared__ uint32_t s_t[4][TRE_MAX_MODELS];                      // timestamp of the model's last row
  __shared__ int s_r[4][TRE_MAX_MODELS];                           // that row (from the trace's first), -1 none
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
  int* const ca = s_a[wv];
  int* const cw = s_w[wv];
  uint32_t* const lt = s_t[wv];
  int* const lr = s_r[wv];
  if (*p.err & ((1u << kValState) - 1u)) return;  // the whole grid: those bits are set before this kernel
  const int nbits = p.M > 1 ? 32 - __clz(p.M - 1) : 0;
  const unsigned long long le = (2ull << lane) - 1ull;  // lanes <= this one
  auto fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for (uint32_t t = blockIdx.y; t < p.n_traces; t += gridDim.y) {
    const int64_t b = p.off[t];
    const int n = (int)(p.off[t + 1] - b);  // below 2^27
    const int sub = (int)blockIdx.x * 4 + wv;
    if (sub * p.sub_rows >= n) continue;  // whole wave; the waves share no barrier
    const int r_begin = (int)(sub * p.sub_rows), r_end = r_begin + p.sub_rows < n ? (int)(r_begin + p.sub_rows) : n;
    const uint64_t so = p.sub_off[t], n_sub = p.sub_off[t + 1] - so;
    const unsigned long long before = lane < p.M ? p.net[so * p.M + (uint64_t)lane * n_sub + (uint64_t)sub] : 0ull;
    ca[lane] = net_a(before);
    cw[lane] = net_w(before);
    lt[lane] = 0u;
    lr[lane] = -1;
    fence();
    int bad = INT_MAX;
    const int64_t* const ts_ = p.ts + b;
    const uint8_t* const mo_ = p.model + b;
    const uint8_t* const ty_ = p.type + b;
    // rows of the next step are loaded before the current one is processed
    auto load = [&](int i, uint32_t& ts, uint32_t& m, uint32_t& ty) {
      const bool v = i < r_end;
      const int k = v ? i : r_end - 1;
      ts = (uint32_t)ts_[k];  // timestamps lie in [0, duration) below 2^32
      m = (uint32_t)mo_[k] & 63u;
      ty = v ? (uint32_t)ty_[k] : 0xFFu;
    };
    uint32_t tsn, mn, tyn;
    load(r_begin + lane, tsn, mn, tyn);
    for (int r0 = r_begin; r0 < r_end; r0 += 64) {
      const int i = r0 + lane;
      const bool v = i < r_end;
      const uint32_t ts = tsn, m = mn, ty = tyn;
      load(i + 64, tsn, mn, tyn);
      const int dA = (ty == (TRE_PREFILL | TRE_ADMIT) ? 1 : 0) - (ty == TRE_FINISH ? 1 : 0);
      const int dW = (ty == TRE_ARRIVE ? 1 : 0) - (ty == (TRE_PREFILL | TRE_ADMIT) ? 1 : 0);
      unsigned long long same = __ballot(v);
      for (int k = 0; k < nbits; ++k) {
        const unsigned long long bk = __ballot((m >> k) & 1u);
        same &= ((m >> k) & 1u) ? bk : ~bk;
      }
      const unsigned long long pa = __ballot(dA > 0), na = __ballot(dA < 0);
      const unsigned long long pw = __ballot(dW > 0), nw = __ballot(dW < 0);
      const unsigned long long upto = same & le;
      const int ca0 = ca[m], cw0 = cw[m];
      const int va = ca0 + __popcll(pa & upto) - __popcll(na & upto);
      const int vw = cw0 + __popcll(pw & upto) - __popcll(nw & upto);
      const unsigned long long after = same & ~le;
      const int nl = after ? __ffsll((long long)after) - 1 : lane;
      const uint32_t tnext = (uint32_t)__shfl((int)ts, nl);
      // the last row of its instant inside this step
      if (v && after && tnext != ts && (va < 0 || vw < 0)) bad = bad < i ? bad : i;
      // the model's first row in this step settles its last row of an earlier step
      if (v && (upto & ~(1ull << lane)) == 0ull && (ca0 < 0 || cw0 < 0)) {
        const int rp = lr[m];
        if (rp >= 0 && lt[m] != ts) bad = bad < rp ? bad : rp;
      }
      fence();
      if (v && !after) {  // the model's last row in this step
        ca[m] = va;
        cw[m] = vw;
        lt[m] = ts;
        lr[m] = i;
      }
      fence();
    }
    // each model's last row is the last of its instant unless a later piece
    // goes on with it: rows after this piece at the timestamp of its last row,
    // read until every such model has been seen again (an instant has at most
    // 65535 rows, the limit of its window)
    const bool neg = lane < p.M && lr[lane] >= 0 && (ca[lane] < 0 || cw[lane] < 0);
    bool on = false;
    const uint32_t tl = (uint32_t)ts_[r_end - 1];
    if (__ballot(neg && lt[lane] == tl)) {
      for (int r0 = r_end; r0 < n; r0 += 64) {
        const int i = r0 + lane < n ? r0 + lane : n - 1;
        const bool at = r0 + lane < n && (uint32_t)ts_[i] == tl;
        unsigned long long rows = __ballot(at);
        const bool more = rows == ~0ull;
        const int m = (int)mo_[i] & 63;
        while (rows) {
          const int l = __ffsll((long long)rows) - 1;
          on = on || __builtin_amdgcn_readlane(m, l) == lane;
          rows &= rows - 1ull;
        }
        if (!more || !__ballot(neg && lt[lane] == tl && !on)) break;
      }
    }
    if (neg && !(lt[lane] == tl && on)) bad = bad < lr[lane] ? bad : lr[lane];
    if (bad != INT_MAX) {
      atomicOr(p.err, 1u << kValState);
      atomicMin(p.first, (unsigned long long)(b + bad));
    }
    fence();  // the next trace's state goes to the same slice
  }
}

// With request ids given, each id follows one lifecycle: a request is
// admitted once (its first prefill chunk carries the ADMIT bit), arrives
// once, finishes once, and neither arrives nor decodes after it finished
// (rows of its FINISH instant in any order). The id_scan that marks sets one bit per
// admitted and per arrived id in per-trace bitmaps and stores each id's
// FINISH timestamp, and records the smallest (trace, id) whose mark was
// already set; the id_scan that checks compares every ARRIVE and DECODE row with the FINISH
// timestamp of its id. Bound by the atomics of the marks (three in eleven
// rows). A bitmap of 2^k words holds id i in word i mod 2^k: ids count up
// with time, and 32 neighbours in one word meet there (7.7 M rows 96 us
// against 78).
struct IdParams {
  const int64_t* ts;
  const uint32_t* req;
  const uint8_t* type;
  const int64_t* off;
  uint32_t t0, n_traces;        // traces [t0, t0 + n_traces) of this launch
  const uint64_t* word_off;     // [all traces + 1] first bitmap word of each trace's admitted ids
  const uint64_t* arr_off;      // [all traces + 1] the same of its arrived ids
  const uint64_t* slot_off;     // [all traces + 1] first slot of each trace's ARRIVE and FINISH ids
  uint64_t word_base, arr_base, slot_base;  // those of trace t0
  uint32_t* bits;               // admitted ids of this launch's traces
  uint32_t* arr;                // arrived ids
  uint32_t* fin;                // FINISH timestamp per slot, 0xFFFFFFFF when none
  unsigned long long* dup;      // smallest (trace << 32 | id) admitted twice
  unsigned long long* bad;      // smallest (trace << 32 | id) off its lifecycle
};

template <bool kCheck>
__global__ __launch_bounds__(256) void id_scan(IdParams p) {
  const uint32_t t = p.t0 + blockIdx.y;
  const int64_t b = p.off[t], e = p.off[t + 1];
  const int64_t c0 = b + (int64_t)blockIdx.x * kSubRows;
  if (c0 >= e) return;
  const int64_t c1 = c0 + kSubRows < e ? c0 + kSubRows : e;
  const uint64_t n_words = p.word_off[t + 1] - p.word_off[t], w0 = p.word_off[t] - p.word_base;
  const uint64_t n_arr = p.arr_off[t + 1] - p.arr_off[t], a0 = p.arr_off[t] - p.arr_base;
  const uint64_t n_slots = p.slot_off[t + 1] - p.slot_off[t], s0 = p.slot_off[t] - p.slot_base;
  const int kw = 63 - __clzll((long long)n_words), ka = 63 - __clzll((long long)n_arr);  // powers of two
  constexpr int kU = 4;
  for (int64_t i0 = c0 + threadIdx.x; i0 < c1; i0 += 256 * kU) {
    uint32_t tyv[kU], idv[kU], tv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t i = i0 + 256 * u < c1 ? i0 + 256 * u : c1 - 1;
      tyv[u] = i0 + 256 * u < c1 ? (uint32_t)p.type[i] : (uint32_t)TRE_PREFILL;  // a plain PREFILL row marks nothing
      idv[u] = p.req[i];
      tv[u] = (uint32_t)p.ts[i];  // timestamps lie in [0, duration) below 2^32
    }
    // every mark (or FINISH read) issued before any result is used
    uint32_t old[kU], bit[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t kind = tyv[u] & 3u, id = idv[u];
      const bool slot = (uint64_t)id < n_slots;  // always, for ARRIVE and FINISH
      const uint64_t sl = s0 + id;
      if constexpr (!kCheck) {
        const bool admit = tyv[u] == (TRE_PREFILL | TRE_ADMIT);
        old[u] = 0u;
        bit[u] = 0u;
        const uint32_t b = id >> (admit ? kw : ka);
        if ((admit || (kind == TRE_ARRIVE && slot)) && b < 32u) {  // always below, for ids up to the largest
          uint32_t* const w = admit ? &p.bits[w0 + (id & (n_words - 1))] : &p.arr[a0 + (id & (n_arr - 1))];
          bit[u] = 1u << b;
          old[u] = atomicOr(w, bit[u]);
        } else if (kind == TRE_FINISH && slot) {
          old[u] = ~atomicCAS(&p.fin[sl], 0xFFFFFFFFu, tv[u]);
          bit[u] = 0xFFFFFFFFu;  // set before when the word was not all ones
        }
      } else {
        old[u] = 0xFFFFFFFFu;
        if ((kind == TRE_ARRIVE || kind == TRE_DECODE) && slot) old[u] = p.fin[sl];
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const unsigned long long key = ((unsigned long long)t << 32) | idv[u];
      if constexpr (!kCheck) {
        if (old[u] & bit[u]) atomicMin((tyv[u] & 3u) == TRE_PREFILL ? p.dup : p.bad, key);
      } else {
        if (old[u] != 0xFFFFFFFFu && tv[u] > old[u]) atomicMin(p.bad, key);
      }
    }
  }
}

// ------------------------------------------------ scratch of one call
// The segmented path's scratch and the load checks' memory come from blocks that
// the library keeps per device. A block serves one call at a time, from the
// constructor to the destructor on the host and from there to the block's event
// on the device: another call takes it once the event has completed, or on the
// same stream behind it. So calls on several streams and threads never share
// one. (A HIP memory pool gives its memory back at every hipMalloc and hipFree of
// the process, whatever its release threshold: the first call on new traces
// mapped its scratch anew, 350 to 500 us.)
//
// The blocks of a device hold at most kPoolKeep in all, and no call takes more.
// When the device's last handle is freed one block of once to twice what the
// largest call since the last such time needed is kept for the next handle's
// calls, and the others are given back; all of them after a load that is refused.
// A stream that is being captured gets none (the caller then takes the path that
// needs no scratch).
constexpr uint64_t kPoolKeep = 1ull << 30;
constexpr int kPoolBlocks = 16;

namespace {
constexpr int kMaxDevices = 256;
struct Block {
  void* ptr;
  uint64_t bytes;
  hipEvent_t done;  // recorded behind the last call's work
  hipStream_t st;   // its stream
  bool busy;        // a call holds it
};
struct Pool {
  int handles;
  uint64_t need;   // largest call since the device last had no handle
  uint64_t bytes;  // of all blocks
  Block b[kPoolBlocks];
};
std::mutex g_pool_mu;
Pool g_pool[kMaxDevices];

bool block_done(const Block& b) {
  const hipError_t e = hipEventQuery(b.done);
  if (e != hipSuccess) (void)hipGetLastError();
  return e == hipSuccess;
}

void block_free(Pool& p, Block& b) {
  (void)hipEventSynchronize(b.done);
  (void)hipEventDestroy(b.done);
  (void)hipFree(b.ptr);
  p.bytes -= b.bytes;
  b = Block{};
}

// A block of at least `bytes` for work on `st`, marked busy, or NULL. The smallest
// that fits among those free to use, else a new one, for which blocks free to
// use are given back (waiting for the device) while all of them would hold more
// than kPoolKeep.
Block* block_take(int dev, uint64_t bytes, hipStream_t st) {
  if (dev < 0 || dev >= kMaxDevices || bytes > kPoolKeep) return nullptr;
  std::lock_guard<std::mutex> lk(g_pool_mu);
  Pool& p = g_pool[dev];
  p.need = std::max(p.need, bytes);
  Block *fit = nullptr, *slot = nullptr;
  for (Block& b : p.b) {
    if (!b.ptr) slot = &b;
    else if (!b.busy && b.bytes >= bytes && (!fit || b.bytes < fit->bytes) && (b.st == st || block_done(b))) fit = &b;
  }
  if (fit) {
    // (the stream that had this handle may be gone and its work still under way)
    if (fit->st == st && hipStreamWaitEvent(st, fit->done, 0) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    fit->busy = true;
    return fit;
  }
  // nothing below is part of a capture that goes on elsewhere
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  for (Block& b : p.b) {
    if (slot && p.bytes + bytes <= kPoolKeep) break;
    if (b.ptr && !b.busy && block_done(b)) {
      block_free(p, b);
      slot = &b;
    }
  }
  Block nb{};
  nb.bytes = bytes;
  nb.busy = true;
  const bool room = slot && p.bytes + bytes <= kPoolKeep;
  if (room && hipMalloc(&nb.ptr, bytes) != hipSuccess) nb.ptr = nullptr;
  if (nb.ptr && hipEventCreateWithFlags(&nb.done, hipEventDisableTiming) != hipSuccess) {
    (void)hipFree(nb.ptr);
    nb.ptr = nullptr;
  }
  if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (!nb.ptr) {
    if (room) (void)hipGetLastError();
    return nullptr;
  }
  p.bytes += bytes;
  *slot = nb;
  return slot;
}

// the call's work is enqueued on `st`
void block_return(Block* b, hipStream_t st) {
  std::lock_guard<std::mutex> lk(g_pool_mu);
  if (hipEventRecord(b->done, st) != hipSuccess) {  // then the event's last record stands: wait instead
    (void)hipGetLastError();
    (void)hipStreamSynchronize(st);
  }
  b->st = st;
  b->busy = false;
}

void count_handle(int dev, int d, bool refused = false) {
  if (dev < 0 || dev >= kMaxDevices) return;
  std::lock_guard<std::mutex> lk(g_pool_mu);
  Pool& p = g_pool[dev];
  p.handles += d;
  if (p.handles > 0) return;
  Block* keep = nullptr;
  if (!refused)
    for (Block& b : p.b)
      if (b.ptr && b.bytes >= p.need && b.bytes <= 2 * p.need && (!keep || b.bytes < keep->bytes)) keep = &b;
  for (Block& b : p.b)
    if (b.ptr && !b.busy && &b != keep) block_free(p, b);
  p.need = 0;
}

// `bytes` of scratch for work enqueued on `st` until the destructor, or NULL
class Scratch {
 public:
  Scratch(int dev, size_t bytes, hipStream_t st) : st_(st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return;
    }
    b_ = block_take(dev, (bytes + kRound - 1) & ~(kRound - 1), st);
  }
  ~Scratch() {
    if (b_) block_return(b_, st_);
  }
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  char* get() const { return b_ ? (char*)b_->ptr : nullptr; }

 private:
  static constexpr uint64_t kRound = 1ull << 20;  // calls of nearly one size share a block
  Block* b_ = nullptr;
  hipStream_t st_;
};

}  // namespace

// ------------------------------------------------------------------ timing
namespace {
struct Pending {
  const char* name;
  hipEvent_t start, stop;
};
std::mutex g_tmu;
bool g_timing = false;
std::vector<Pending> g_pending;

}  // namespace

static thread_local int g_no_timing = 0;

tre_internal::NoTimingScope::NoTimingScope() { ++g_no_timing; }
tre_internal::NoTimingScope::~NoTimingScope() { --g_no_timing; }

tre_internal::LaunchTimer::LaunchTimer(const char* name, hipStream_t s) : st_(s) {
  if (g_no_timing) return;
  std::lock_guard<std::mutex> lk(g_tmu);
  if (!g_timing) return;
  name_ = name;
  if (hipEventCreate(&start_) != hipSuccess) return;
  if (hipEventCreate(&stop_) != hipSuccess) {
    (void)hipEventDestroy(start_);
    return;
  }
  on_ = hipEventRecord(start_, st_) == hipSuccess;
}

void tre_internal::LaunchTimer::done() {
  if (!on_) return;
  (void)hipEventRecord(stop_, st_);
  std::lock_guard<std::mutex> lk(g_tmu);
  g_pending.push_back(Pending{name_, start_, stop_});
  on_ = false;
}


extern "C" int tre_set_timing(int enable) {
  std::lock_guard<std::mutex> lk(g_tmu);
  g_timing = enable != 0;
  return TRE_OK;
}

extern "C" int tre_kernel_time(const char* kernel, double* total_ms, uint64_t* launches) {
  if (!kernel || !total_ms || !launches) return fail(TRE_EINVAL, "tre_kernel_time: NULL argument");
  std::vector<Pending> mine;
  {
    std::lock_guard<std::mutex> lk(g_tmu);
    std::vector<Pending> rest;
    for (auto& pe : g_pending) (strcmp(pe.name, kernel) == 0 ? mine : rest).push_back(pe);
    g_pending.swap(rest);
  }
  double tot = 0.0;
  int rc = TRE_OK;
  for (auto& pe : mine) {
    float ms = 0.f;
    if (hipEventSynchronize(pe.stop) != hipSuccess ||
        hipEventElapsedTime(&ms, pe.start, pe.stop) != hipSuccess)
      rc = fail(TRE_EHIP, "tre_kernel_time: event query failed");
    tot += ms;
    (void)hipEventDestroy(pe.start);
    (void)hipEventDestroy(pe.stop);
  }
  *total_ms = tot;
  *launches = mine.size();
  return rc;
}

// --------------------------------------------------------------- host ABI
int tre_internal::check_device(const tre_events* ev) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev != ev->device)
    return fail(TRE_EINVAL, "handle belongs to device %d, current device is %d", ev->device, dev);
  return TRE_OK;
}

// events one window of one trace may hold: the packed per-window sums stay
// inside their 32-bit halves
static int64_t max_events_per_window(int64_t window_ms) {
  const int64_t by_integral = 2147483647ll / window_ms;
  return by_integral < TRE_MAX_EVENTS_PER_WINDOW ? by_integral : TRE_MAX_EVENTS_PER_WINDOW;
}

static uint32_t ring_windows(int M) {
  uint32_t w = 256;
  while (w > 2 && (size_t)w * (4 * (size_t)M + 1) * 8 > (size_t)kRingBytes) w >>= 1;
  return w;
}

// windows evaluated per step: a power of two, one cell per thread of the
// first kEvalThreads, at most half the ring (the same for every workgroup
// size, so the LDS layout does not depend on it)
static int chunk_windows(int M, uint32_t wcap) {
  int c = 32;
  while (c > 1 && (c * M > kEvalThreads || c > (int)wcap / 2)) c >>= 1;
  return c;
}

// Waves per tss_stream workgroup. One workgroup streams one trace; with 4
// waves (about 75 VGPRs) six fit on a CU, so 1536 traces fill the chip.
// With fewer traces the resident workgroups alone cannot keep enough loads
// in flight, so each trace gets a larger workgroup: 16 waves (one per CU,
// four per SIMD) up to 384 traces, 8 waves up to 768.
static int stream_waves(uint32_t n_traces) {
  return n_traces <= 384 ? 16 : (n_traces <= 768 ? 8 : kStreamWaves);
}

// The segmented path: about kSegGrid workgroups in all, at most kSegMax
// segments a trace (every workgroup adds up the net changes of the segments
// before its own), each a whole number of evaluation chunks; workgroups of 16
// waves while they are at most kSegWide. It costs three launches, 2 bytes a row
// and 16 bytes a cell more than one workgroup per trace (seg_pays).
constexpr int64_t kSegGrid = 2048, kSegMax = 256, kSegWide = 512;

static size_t stream_lds(const tre_events* ev, bool stage = false) {
  const size_t M = (size_t)ev->cfg.n_models, C = (size_t)chunk_windows(ev->cfg.n_models, ev->wcap);
  const size_t ring = ev->wcap * (4 * M + 1) * 8;
  // stage: two staging buffers of prefill ratios (in the scalar ratios'
  // place) and two of decode ratios, two shares and two flags per model
  if (stage) return ring + 4 * C * M * 8 + 2 * M * 8 + ((2 * M + 7) & ~(size_t)7);
  // three staging buffers, then the control replay's per-model records and
  // 11 words
  return ring + 3 * C * M * 8 + M * sizeof(CtlModel) + ((11 * 4 + 7) & ~(size_t)7);
}

// Device memory of one call: a kept block, or its own when there is none to be had
class CallMemory {
 public:
  CallMemory(int dev, size_t bytes, hipStream_t st) : pooled_(dev, bytes, st) {
    if (!pooled_.get() && hipMalloc(&own_, bytes) != hipSuccess) {
      own_ = nullptr;
      (void)hipGetLastError();
    }
  }
  ~CallMemory() {
    if (own_) (void)hipFree(own_);
  }
  CallMemory(const CallMemory&) = delete;
  CallMemory& operator=(const CallMemory&) = delete;
  char* get() const { return own_ ? (char*)own_ : pooled_.get(); }

 private:
  Scratch pooled_;
  void* own_ = nullptr;
};

// The load-time checks (synchronous): order, schema and per-window range
// of every row; on rows that pass, counts never negative; then, with
// request ids, one lifecycle per id. The error reported is the kind of the
// lowest failing row among the first three kinds (order before schema
// before range on one row), else a negative count (its lowest row), else a
// duplicate admission (the smallest trace, then id), else an id off its
// lifecycle. Two waits in all: after the checks without ids, whose results
// size the id tables, and at the end.
static int validate_events(const tre_events* ev, hipStream_t st) {
  const uint32_t n_traces = ev->n_traces;
  const tre_trace_cfg& c = ev->cfg;
  const size_t nt = n_traces;
  int64_t maxlen = 0;
  // one block, copied both ways at once: the results, the largest ids of each
  // trace, the traces' first pieces
  struct Slots {
    unsigned err, pad;
    unsigned long long first[kValKinds];
    unsigned long long dup, life;
  };
  static_assert(sizeof(Slots) % 8 == 0, "");
  const size_t max_at = sizeof(Slots), sub_at = max_at + 8 * nt, net_at = sub_at + 8 * (nt + 1);
  std::vector<uint64_t> host(net_at / 8);
  Slots& h = *(Slots*)host.data();
  uint32_t* const h_admit = (uint32_t*)((char*)host.data() + max_at);
  uint32_t* const h_life = h_admit + nt;
  uint64_t* const h_sub = (uint64_t*)((char*)host.data() + sub_at);
  memset(&h, 0xFF, sizeof h);
  h.err = 0;
  h.pad = 0;
  h_sub[0] = 0;
  int64_t sub_rows = kSubRows;
  while ((uint64_t)(ev->n_events / sub_rows) > kMaxSubs) sub_rows *= 2;
  for (uint32_t i = 0; i < n_traces; ++i) {
    const int64_t len = ev->h_off[i + 1] - ev->h_off[i];
    maxlen = std::max(maxlen, len);
    h_sub[i + 1] = h_sub[i] + (uint64_t)((len + sub_rows - 1) / sub_rows);
  }
  if (maxlen == 0) return TRE_OK;
  const uint64_t net_bytes = h_sub[nt] * (uint64_t)c.n_models * 8;
  CallMemory mem(ev->device, net_at + net_bytes + (ev->req ? h_sub[nt] * sizeof(uint2) : 0), st);
  if (!mem.get()) return fail(TRE_EHIP, "hipMalloc failed");
  Slots* const d = (Slots*)mem.get();
  uint32_t* const d_admit = (uint32_t*)(mem.get() + max_at);
  const uint64_t* const d_sub = (const uint64_t*)(mem.get() + sub_at);
  unsigned long long* const d_net = (unsigned long long*)(mem.get() + net_at);
  uint2* const d_smax = ev->req ? (uint2*)(mem.get() + net_at + net_bytes) : nullptr;
  auto readback = [&](size_t bytes) {
    return hipMemcpyAsync(host.data(), d, bytes, hipMemcpyDeviceToHost, st) == hipSuccess &&
           hipStreamSynchronize(st) == hipSuccess;
  };
  bool ok = hipMemcpyAsync(d, host.data(), net_at, hipMemcpyHostToDevice, st) == hipSuccess;
  const dim3 grid((unsigned)((maxlen + 4 * sub_rows - 1) / (4 * sub_rows)), std::min<uint32_t>(n_traces, 65535u));
  if (ok) {
    ValParams vp{ev->ts, ev->model, ev->req, ev->type, ev->d_off, d_sub, sub_rows, n_traces, c.duration_ms, c.window_ms,
                 c.n_models, max_events_per_window(c.window_ms), &d->err, d->first, d_net, d_smax};
    LaunchTimer lt("validate", st);
    hipLaunchKernelGGL(validate, grid, dim3(256), 0, st, vp);
    ok = hipGetLastError() == hipSuccess;
    lt.done();
  }
  if (ok) {
    hipLaunchKernelGGL(net_scan, dim3(std::min<uint32_t>(n_traces, 65535u), (unsigned)(c.n_models / 4 + 1)), dim3(256), 0, st, d_net, d_sub, n_traces,
                       c.n_models, d_smax, d_admit, d_admit + nt);
    StateParams sp{ev->ts, ev->model, ev->type, ev->d_off, d_sub, sub_rows, d_net, n_traces, c.n_models, &d->err,
                   &d->first[kValState]};
    hipLaunchKernelGGL(validate_state, grid, dim3(256), 0, st, sp);
    ok = hipGetLastError() == hipSuccess;
  }
  if (!ok || !readback(sub_at)) return fail(TRE_EHIP, "validation launch failed");
  if (h.err) {
    int kind = -1;
    for (int k = 0; k < kValState; ++k)
      if ((h.err >> k & 1u) && (kind < 0 || h.first[k] < h.first[kind])) kind = k;
    if (kind < 0)
      return fail(TRE_ESTATE, "row %llu: an active or waiting count below zero after this instant",
                  h.first[kValState]);
    const unsigned long long row = h.first[kind];
    if (kind == kValOrder) return fail(TRE_EORDER, "row %llu: timestamp unsorted or outside [0, duration)", row);
    if (kind == kValSchema) return fail(TRE_ESCHEMA, "row %llu: model index or type byte invalid", row);
    return fail(TRE_ERANGE, "row %llu: more than %lld events in one window", row,
                (long long)max_events_per_window(c.window_ms));
  }
  if (!ev->req) return TRE_OK;
  // the id tables, in batches of traces of at most 2^26 bitmap words (256
  // MiB) and 2^26 slots (256 MiB of FINISH timestamps), or one trace's if larger
  std::vector<uint64_t> offs(3 * (nt + 1));
  uint64_t* const woff = offs.data();
  uint64_t* const aoff = woff + nt + 1;
  uint64_t* const soff = aoff + nt + 1;
  uint64_t most_w = 0, most_s = 0;
  woff[0] = aoff[0] = soff[0] = 0;
  auto words = [](uint32_t max_id) {  // a power of two whose bits hold ids 0 .. max_id
    uint64_t w = 1;
    while (32 * w <= max_id) w <<= 1;
    return w;
  };
  for (uint32_t t = 0; t < n_traces; ++t) {
    const uint64_t w = words(h_admit[t]), n = (uint64_t)h_life[t] + 1u;
    woff[t + 1] = woff[t] + w;
    aoff[t + 1] = aoff[t] + words(h_life[t]);
    soff[t + 1] = soff[t] + n;
    most_w = std::max(most_w, w);
    most_s = std::max(most_s, n);
  }
  const uint64_t cap_w = std::max<uint64_t>(most_w, std::min<uint64_t>(woff[nt], 1ull << 26));
  const uint64_t cap_s = std::max<uint64_t>(most_s, std::min<uint64_t>(soff[nt], 1ull << 26));
  // a trace's words are at most 2 + a sixteenth of its slots
  const uint64_t cap_a = cap_s / 16 + 2 * std::min<uint64_t>(nt, 65535u);
  const size_t offs_bytes = offs.size() * 8;
  CallMemory tab(ev->device, offs_bytes + 4 * (cap_a + cap_w + cap_s), st);
  if (!tab.get()) return fail(TRE_EHIP, "hipMalloc failed");
  ok = hipMemcpyAsync(tab.get(), woff, offs_bytes, hipMemcpyHostToDevice, st) == hipSuccess;
  IdParams ip{};
  ip.ts = ev->ts;
  ip.req = ev->req;
  ip.type = ev->type;
  ip.off = ev->d_off;
  ip.word_off = (const uint64_t*)tab.get();
  ip.arr_off = ip.word_off + nt + 1;
  ip.slot_off = ip.arr_off + nt + 1;
  ip.arr = (uint32_t*)(tab.get() + offs_bytes);
  ip.bits = ip.arr + cap_a;
  ip.fin = ip.bits + cap_w;
  ip.dup = &d->dup;
  ip.bad = &d->life;
  for (uint32_t t0 = 0; ok && t0 < n_traces;) {
    uint32_t t1 = t0 + 1;
    while (t1 < n_traces && t1 - t0 < 65535u && woff[t1 + 1] - woff[t0] <= cap_w && soff[t1 + 1] - soff[t0] <= cap_s)
      ++t1;
    int64_t len = 0;
    for (uint32_t t = t0; t < t1; ++t) len = std::max<int64_t>(len, ev->h_off[t + 1] - ev->h_off[t]);
    ip.t0 = t0;
    ip.n_traces = t1 - t0;
    ip.word_base = woff[t0];
    ip.arr_base = aoff[t0];
    ip.slot_base = soff[t0];
    // the two bitmaps lie side by side
    ok = hipMemsetAsync(ip.arr, 0, 4 * (cap_a + woff[t1] - woff[t0]), st) == hipSuccess &&
         hipMemsetAsync(ip.fin, 0xFF, 4 * (soff[t1] - soff[t0]), st) == hipSuccess;
    if (ok && len > 0) {
      const dim3 g((unsigned)((len + kSubRows - 1) / kSubRows), t1 - t0);
      hipLaunchKernelGGL(id_scan<false>, g, dim3(256), 0, st, ip);
      hipLaunchKernelGGL(id_scan<true>, g, dim3(256), 0, st, ip);
      ok = hipGetLastError() == hipSuccess;
    }
    t0 = t1;
  }
  if (!ok || !readback(sizeof(Slots))) return fail(TRE_EHIP, "validation launch failed");
  if (h.dup != ~0ull)
    return fail(TRE_ESTATE, "trace %u: request id %u admitted more than once", (unsigned)(h.dup >> 32),
                (unsigned)h.dup);
  if (h.life != ~0ull)
    return fail(TRE_ESTATE, "trace %u: request id %u arrives or finishes twice, or arrives or decodes after its FINISH",
                (unsigned)(h.life >> 32), (unsigned)h.life);
  return TRE_OK;
}

static void free_events(tre_events* ev, bool refused) {
  if (ev->d_off) (void)hipFree(ev->d_off);  // with the tick tables
  if (ev->counted) count_handle(ev->device, -1, refused);
  delete ev;
}

extern "C" int tre_load_events(const int64_t* ts, const uint8_t* model, const uint32_t* req,
                               const uint8_t* type, const uint16_t* tokens,
                               const int64_t* trace_off, uint32_t n_traces,
                               const tre_trace_cfg* cfg, uint32_t flags, void* stream,
                               tre_events** out) {
  if (!out) return fail(TRE_EINVAL, "tre_load_events: out is NULL");
  *out = nullptr;
  if (!ts || !model || !type || !tokens || !trace_off || !cfg)
    return fail(TRE_EINVAL, "tre_load_events: NULL column, offsets or cfg");
  if (n_traces == 0) return fail(TRE_EINVAL, "tre_load_events: no traces");
  if (((uintptr_t)ts & 15) || ((uintptr_t)tokens & 15) || ((uintptr_t)model & 7) ||
      ((uintptr_t)type & 7))
    return fail(TRE_EINVAL, "tre_load_events: misaligned column (ts/tokens need 16, model/type 8)");
  const tre_trace_cfg c = *cfg;
  if (c.window_ms < 1 || c.window_ms > (1 << 23))
    return fail(TRE_EINVAL, "window_ms %lld outside [1, 2^23]", (long long)c.window_ms);
  if (c.duration_ms <= 0 || c.duration_ms % c.window_ms)
    return fail(TRE_EINVAL, "duration_ms must be a positive multiple of window_ms");
  if (c.duration_ms >= (1ll << 32)) return fail(TRE_EINVAL, "duration_ms must be below 2^32");
  if (c.duration_ms / c.window_ms > (1ll << 30)) return fail(TRE_EINVAL, "too many windows");
  if (c.fast_period_ms <= 0 || c.slow_period_ms <= 0 || c.fast_period_ms % c.window_ms ||
      c.slow_period_ms % c.window_ms)
    return fail(TRE_EINVAL, "periods must be positive multiples of window_ms");
  if (c.n_models < 1 || c.n_models > TRE_MAX_MODELS)
    return fail(TRE_EINVAL, "n_models %d outside [1, %d]", c.n_models, TRE_MAX_MODELS);
  if (c.budget < 0) return fail(TRE_EINVAL, "negative budget");
  if (trace_off[0] < 0) return fail(TRE_EINVAL, "trace_off[0] < 0");
  for (uint32_t i = 0; i < n_traces; ++i) {
    if (trace_off[i + 1] < trace_off[i]) return fail(TRE_EINVAL, "trace_off decreases at %u", i);
    if (trace_off[i + 1] - trace_off[i] >= (1ll << 27))
      return fail(TRE_ERANGE, "trace %u has 2^27 or more events", i);
  }
  tre_events* ev = new (std::nothrow) tre_events();
  if (!ev) return fail(TRE_EINVAL, "out of host memory");
  ev->ts = ts;
  ev->model = model;
  ev->req = req;
  ev->type = type;
  ev->tokens = tokens;
  ev->n_traces = n_traces;
  ev->cfg = c;
  ev->n_windows = c.duration_ms / c.window_ms;
  ev->h_off.assign(trace_off, trace_off + n_traces + 1);
  ev->n_events = trace_off[n_traces] - trace_off[0];
  ev->n_rows = trace_off[n_traces];
  ev->wcap = ring_windows(c.n_models);
  const int64_t fw = c.fast_period_ms / c.window_ms, sw = c.slow_period_ms / c.window_ms;
  std::vector<uint32_t> tw;
  std::vector<uint8_t> tk;
  // the windows that end on a multiple of either period, in order
  for (int64_t f = fw, s = sw; f <= ev->n_windows || s <= ev->n_windows;) {
    const int64_t x = std::min(f, s);
    tw.push_back((uint32_t)(x - 1));
    tk.push_back((uint8_t)((x == f ? 1 : 0) | (x == s ? 2 : 0)));
    if (x == f) f += fw;
    if (x == s) s += sw;
  }
  ev->n_ticks = (int64_t)tw.size();
  hipStream_t st = (hipStream_t)stream;
  int rc = TRE_OK;
  auto cleanup = [&](int code) {
    free_events(ev, true);
    return code;
  };
  if (hipGetDevice(&ev->device) != hipSuccess) return cleanup(fail(TRE_EHIP, "hipGetDevice failed"));
  count_handle(ev->device, 1);
  ev->counted = true;
  // the handle's tables in one allocation and one copy: offsets, tick windows, tick kinds
  const size_t off_bytes = sizeof(int64_t) * ((size_t)n_traces + 1), tw_bytes = sizeof(uint32_t) * (tw.size() + 1);
  std::vector<char> tables(off_bytes + tw_bytes + tk.size() + 1);
  memcpy(tables.data(), trace_off, off_bytes);
  if (!tw.empty()) memcpy(tables.data() + off_bytes, tw.data(), sizeof(uint32_t) * tw.size());
  if (!tk.empty()) memcpy(tables.data() + off_bytes + tw_bytes, tk.data(), tk.size());
  if (hipMalloc(&ev->d_off, tables.size()) != hipSuccess)
    return cleanup(fail(TRE_EHIP, "hipMalloc of handle tables failed"));
  ev->d_tick_window = (uint32_t*)((char*)ev->d_off + off_bytes);
  ev->d_tick_kind = (uint8_t*)((char*)ev->d_off + off_bytes + tw_bytes);
  if (hipMemcpyAsync(ev->d_off, tables.data(), tables.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return cleanup(fail(TRE_EHIP, "copy of handle tables failed"));

  if (flags & TRE_VALIDATE) {
    rc = validate_events(ev, st);
    if (rc != TRE_OK) return cleanup(rc);
  }
  *out = ev;
  return TRE_OK;
}

extern "C" void tre_free_events(tre_events* ev) {
  if (ev) free_events(ev, false);
}

extern "C" int tre_events_info(const tre_events* ev, tre_info* info) {
  if (!ev || !info) return fail(TRE_EINVAL, "tre_events_info: NULL argument");
  info->n_traces = ev->n_traces;
  info->n_models = (uint32_t)ev->cfg.n_models;
  info->n_events = ev->n_events;
  info->n_windows = ev->n_windows;
  info->n_ticks = ev->n_ticks;
  return TRE_OK;
}

// tre_sweep's workspace: the per-tick smoothed TSS of every trace (read by
// the separate replay of traces with several scenarios), then per trace
// its scenario count and one of its scenarios
static size_t snapshot_bytes(const tre_events* ev) {
  return ((size_t)ev->n_traces * (size_t)ev->n_ticks * (size_t)ev->cfg.n_models * sizeof(double) + 255) &
         ~(size_t)255;
}

extern "C" int tre_workspace_size(const tre_events* ev, uint32_t n_scenarios, size_t* bytes) {
  if (!ev || !bytes) return fail(TRE_EINVAL, "tre_workspace_size: NULL argument");
  (void)n_scenarios;
  *bytes = snapshot_bytes(ev) + 2 * sizeof(uint32_t) * (size_t)ev->n_traces;
  return TRE_OK;
}

extern "C" int tre_check_params(const tre_events* ev, const tre_profile* prof,
                                const tre_scenario* sc, uint32_t n_scenarios) {
  if (!ev || !prof) return fail(TRE_EINVAL, "tre_check_params: NULL handle or profiles");
  if (n_scenarios && !sc) return fail(TRE_EINVAL, "tre_check_params: NULL scenarios");
  int rc = check_device(ev);
  if (rc) return rc;
  const size_t M = (size_t)ev->cfg.n_models;
  std::vector<tre_profile> hp((size_t)ev->n_traces * M);
  std::vector<tre_scenario> hs(n_scenarios);
  HIP_TRY(hipMemcpy(hp.data(), prof, hp.size() * sizeof(tre_profile), hipMemcpyDeviceToHost));
  if (n_scenarios)
    HIP_TRY(hipMemcpy(hs.data(), sc, hs.size() * sizeof(tre_scenario), hipMemcpyDeviceToHost));
  for (uint32_t t = 0; t < ev->n_traces; ++t) {
    long long rsum = 0;
    for (size_t m = 0; m < M; ++m) {
      const tre_profile& q = hp[t * M + m];
      if (!(q.w_p >= 0.0 && q.w_q >= 0.0 && q.alpha > 0.0 && q.alpha <= 1.0 && q.theta > 0.0 &&
            isfinite(q.w_p) && isfinite(q.w_q) && isfinite(q.theta) && q.tau_crit >= 0.0 &&
            q.tau_crit < q.tau_surplus && q.r_min >= 0 && q.r_init >= 0))
        return fail(TRE_EINVAL, "profile of trace %u model %zu out of range", t, m);
      rsum += q.r_init;
    }
    if (rsum > ev->cfg.budget)
      return fail(TRE_EINVAL, "trace %u: initial replicas %lld exceed the budget %d", t, rsum,
                  ev->cfg.budget);
  }
  for (uint32_t s = 0; s < n_scenarios; ++s) {
    const tre_scenario& q = hs[s];
    if (q.trace >= ev->n_traces) return fail(TRE_EINVAL, "scenario %u: trace out of range", s);
    if (!(q.theta_scale > 0.0 && isfinite(q.theta_scale)))
      return fail(TRE_EINVAL, "scenario %u: theta_scale must be positive", s);
    if (q.tau_crit_override >= 0.0) {
      for (size_t m = 0; m < M; ++m)
        if (!(q.tau_crit_override < hp[q.trace * M + m].tau_surplus))
          return fail(TRE_EINVAL, "scenario %u: tau_crit_override >= tau_surplus", s);
    }
  }
  return TRE_OK;
}

static StreamParams stream_params(const tre_events* ev, const tre_profile* prof) {
  StreamParams p{};
  p.ts = ev->ts;
  p.model = ev->model;
  p.type = ev->type;
  p.tokens = ev->tokens;
  p.off = ev->d_off;
  p.n_rows = ev->n_rows;
  p.prof = prof;
  p.window_ms = ev->cfg.window_ms;
  p.magic = ev->cfg.window_ms == 1 ? 0xFFFFFFFFu
                                   : (uint32_t)((1ull << 32) / (uint64_t)ev->cfg.window_ms);
  p.inv2_window = 0.5 / (double)ev->cfg.window_ms;
  p.n_windows = (int32_t)ev->n_windows;
  p.M = ev->cfg.n_models;
  p.wcap = ev->wcap;
  p.chunk = chunk_windows(ev->cfg.n_models, ev->wcap);
  // a period longer than the trace never ticks
  p.fast_w = (int32_t)std::min<int64_t>(ev->cfg.fast_period_ms / ev->cfg.window_ms, ev->n_windows + 1);
  p.slow_w = (int32_t)std::min<int64_t>(ev->cfg.slow_period_ms / ev->cfg.window_ms, ev->n_windows + 1);
  p.magic_fast = p.fast_w == 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / (uint64_t)p.fast_w);
  p.magic_slow = p.slow_w == 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / (uint64_t)p.slow_w);
  p.n_ticks = (int32_t)ev->n_ticks;
  return p;
}

// Scenarios per trace of a sweep: count[t] and, for a trace with exactly
// one, that scenario in first[t] (count is zeroed first)
__global__ __launch_bounds__(256) void zero_u32(uint32_t* q, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) q[i] = 0u;
}

__global__ __launch_bounds__(256) void sweep_map(const tre_scenario* sc, uint32_t n_sc, uint32_t n_traces,
                                                 uint32_t* count, uint32_t* first) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_sc) return;
  const uint32_t t = sc[s].trace;
  if (t >= n_traces) return;
  if (atomicAdd(&count[t], 1u) == 0u) first[t] = s;
}

namespace {
// the segmented path's shape and scratch for one call
struct SegPlan {
  int32_t nseg = 0, seg_w = 0, K = 0, chunk_log2 = 0, waves = 0;
  size_t raw = 0, net = 0, row = 0, first = 0, bytes = 0;  // offsets of the scratch arrays, total
};

// Whether segments beat one workgroup per trace. They do where those leave the
// chip idle and the trace has steps enough to pay for three launches instead of
// one. `cells`: per-cell outputs, which one workgroup per trace writes from its
// serial chain. C: windows of a chunk, the step's evaluation. Measured, one
// workgroup per trace / segments in us, 550 shapes (5 of them are slower by 4 to
// 17% with this rule):
// - below four chunks (three for the stage shares) or 40 windows the launches
//   cost more: 1 model x 40 windows 38 / 48, 32 x 10 windows 39 / 59 (160
//   traces), x 20 windows 35 / 45; 1 model x 160 windows 60 / 43;
// - few traces: up to 160 segments win at up to 16 models (160 traces x 8 models x
//   500 ms 999 / 639; 128 x 8 x 1 s 1434 / 968); above, the chain is a lane per
//   column and the line lies lower (64 x 64 models x 1 s 121 / 103; 160 x 64
//   108 / 118, 160 x 32 46 / 56). The stage shares have no workgroups above 4
//   waves: up to 384 (384 x 64 models 584 / 526);
// - more traces: one workgroup per trace is bound by its chunks of windows while
//   rows are few, and by the rows' tallies, which segments do not make cheaper,
//   when they are many. What counts is the rows of one chunk over all traces.
//   Up to 256 traces (one 16-wave workgroup a CU): 1.5 M with per-cell outputs
//   (1.56 M 606 / 578, 1.71 M 665 / 689), 1.1 M without (1.02 M 614 / 581, 1.12 M
//   624 / 633); above 16 models 0.85 M (0.72 M 1245 / 644, 0.89 M 634 / 701, 1.08 M
//   521 / 615), 1.0 M up to 160 traces (0.93 M 460 / 352, 1.06 M 64 / 77). To 384
//   traces, whose workgroups take two rounds: 2.0 M (1.68 M 1123 / 922, 2.57 M 221
//   / 237), above 16 models 1.5 M (0.82 M 2079 / 656, 1.60 M 587 / 719), 1.75 M with
//   outputs (1.69 M 512 / 416, 2.05 M 530 / 603). To 768
//   (8-wave workgroups): 1.0 M (0.97 M 960 / 714, 0.96 M 805 / 650, 1.14 M 547 / 688,
//   1.7 M 418 / 568), 1.2 M in long calls with per-cell outputs (1.14 M 423 / 339,
//   1.05 M under actuation 1712 / 1421, without outputs 1121 / 1390).
//   Stage shares: 1.5 tiles a chunk and trace.
bool seg_pays(const tre_events* ev, bool stage, bool cells) {
  constexpr int64_t kFew = 160, kFewWide = 96, kFewStage = 384, kMost = 768;
  const int64_t T = ev->n_traces, M = ev->cfg.n_models, nW = ev->n_windows, C = chunk_windows((int)M, ev->wcap);
  const bool wide = M > kChainRows;
  if ((nW + C - 1) / C < (stage ? 3 : 4) || (!stage && nW < 40)) return false;
  if (T <= (stage ? kFewStage : wide ? kFewWide : kFew)) return true;
  if (T > kMost) return false;
  const double chunk_rows = (double)C * (double)ev->n_events / (double)nW;
  if (stage) return chunk_rows <= 1.5 * (kStreamWaves * 64 * kStreamEPT) * (double)T;
  if (T <= 256) return chunk_rows <= (wide ? (T <= kFew ? 1.0e6 : 0.85e6) : cells ? 1.5e6 : 1.1e6);
  if (T <= 384) return chunk_rows <= (wide ? (cells ? 1.75e6 : 1.5e6) : 2.0e6);
  return chunk_rows <= (cells && nW >= 1000 ? 1.2e6 : 1.0e6);
}

SegPlan seg_plan(const tre_events* ev, bool stage, bool cells) {
  SegPlan g;
  const int64_t T = ev->n_traces, M = ev->cfg.n_models, nW = ev->n_windows;
  const int64_t C = chunk_windows((int)M, ev->wcap);
  if (!seg_pays(ev, stage, cells)) return g;
  const int64_t most = std::min<int64_t>({(int64_t)kSegMax, (kSegGrid + T - 1) / T, (nW + C - 1) / C});
  if (most < 2) return g;
  const int64_t per = (nW + most - 1) / most;
  g.seg_w = (int32_t)((per + C - 1) / C * C);
  const int64_t nseg = (nW + g.seg_w - 1) / g.seg_w;
  if (nseg < 2) return g;
  g.K = (int32_t)(stage ? 2 * M : M);
  while ((2 << g.chunk_log2) <= kChainWindows && (g.K << (g.chunk_log2 + 1)) <= kChainCells) ++g.chunk_log2;
  g.waves = T * nseg <= kSegWide ? 16 : kStreamWaves;
  auto take = [&](size_t n) {
    const size_t at = g.bytes;
    g.bytes += (n + 255) & ~(size_t)255;
    return at;
  };
  g.raw = take((size_t)T * g.K * nW * sizeof(double));
  g.net = take((size_t)T * nseg * M * sizeof(unsigned long long));
  g.row = take((size_t)T * (nseg + 1) * sizeof(int32_t));
  g.first = take((size_t)T * g.K * sizeof(uint32_t));
  if (g.bytes > kPoolKeep) return g;
  g.nseg = (int32_t)nseg;  // > 0: the path applies
  return g;
}
}  // namespace

static int launch_segments(const tre_events* ev, const SegPlan& g, StreamParams p, bool stage, char* ws,
                           hipStream_t st) {
  LaunchTimer lt("tss_stream", st);
  const int M = ev->cfg.n_models;
  const unsigned T = ev->n_traces, blocks = T * (unsigned)g.nseg;
  SegNetParams np{};
  np.ts = p.ts;
  np.model = p.model;
  np.type = p.type;
  np.off = p.off;
  np.window_ms = p.window_ms;
  np.M = M;
  np.nseg = g.nseg;
  np.seg_w = g.seg_w;
  np.seg_row = (int32_t*)(ws + g.row);
  np.seg_net = (unsigned long long*)(ws + g.net);
  np.first = (uint32_t*)(ws + g.first);
  np.K = g.K;
  hipLaunchKernelGGL(seg_net, dim3(blocks), dim3(kNetThreads), 0, st, np);
  p.nseg = g.nseg;
  p.seg_w = g.seg_w;
  p.seg_row = np.seg_row;
  p.seg_net = np.seg_net;
  p.raw = (double*)(ws + g.raw);
  p.first = np.first;
  const size_t ring = ev->wcap * (4 * (size_t)M + 1) * 8;
  if (stage && g.waves == 16)
    hipLaunchKernelGGL((tss_seg<16, kStreamEPT, true>), dim3(blocks), dim3(16 * 64), ring, st, p);
  else if (stage)
    hipLaunchKernelGGL((tss_seg<kStreamWaves, kStreamEPT, true>), dim3(blocks), dim3(kStreamWaves * 64), ring, st, p);
  else if (g.waves == 16)
    hipLaunchKernelGGL((tss_seg<16, kStreamEPT, false>), dim3(blocks), dim3(16 * 64), ring, st, p);
  else
    hipLaunchKernelGGL((tss_seg<kStreamWaves, kStreamEPT, false>), dim3(blocks), dim3(kStreamWaves * 64), ring, st, p);
  ChainParams c{};
  c.raw = p.raw;
  c.first = p.first;
  c.prof = p.prof;
  c.n_windows = p.n_windows;
  c.M = M;
  c.chunk_log2 = g.chunk_log2;
  c.fast_w = p.fast_w;
  c.slow_w = p.slow_w;
  c.n_ticks = p.n_ticks;
  {
    int64_t a = p.fast_w, b = p.slow_w;
    while (b) {
      const int64_t r = a % b;
      a = b;
      b = r;
    }
    c.both_w = (int32_t)std::min<int64_t>((int64_t)p.fast_w / a * p.slow_w, INT_MAX);
    c.magic_fast = p.magic_fast;
    c.magic_slow = p.magic_slow;
    c.magic_both = c.both_w == 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / (uint64_t)c.both_w);
  }
  c.magic_k = (1u << 20) / (uint32_t)g.K + 1u;
  c.tss64 = stage ? p.stage64 : p.tss64;
  c.tss32 = stage ? p.stage32 : p.tss32;
  c.flags = stage ? p.sflags : p.flags;
  c.snap = p.snap;
  c.tick_window = ev->d_tick_window;
  c.tick_kind = ev->d_tick_kind;
  c.sc = p.sc;
  c.sc_count = p.sc_count;
  c.sc_first = p.sc_first;
  c.ctl_one = p.ctl_one;
  c.budget = p.budget;
  c.moves = p.moves;
  c.move_cap = p.move_cap;
  c.n_moves = p.n_moves;
  c.r_final = p.r_final;
  c.r_windows = p.r_windows;
  c.stride = 9;
  while (c.stride < g.K) c.stride = 2 * c.stride - 1;
  if (g.K > kChainRows && c.stride < 33) c.stride = 33;
  const size_t lds = (6 * sizeof(double) * (size_t)c.stride) << g.chunk_log2;
  const bool rows = g.K <= kChainRows;
  const dim3 block(chain_threads(rows));
  if (stage && rows) hipLaunchKernelGGL((chain_smooth<true, true>), dim3(T), block, lds, st, c);
  else if (stage) hipLaunchKernelGGL((chain_smooth<true, false>), dim3(T), block, lds, st, c);
  else if (!(c.tss64 || c.tss32 || c.flags || c.snap)) {}  // tallies only
  else if (rows) hipLaunchKernelGGL((chain_smooth<false, true>), dim3(T), block, lds, st, c);
  else hipLaunchKernelGGL((chain_smooth<false, false>), dim3(T), block, lds, st, c);
  const hipError_t e = hipGetLastError();
  lt.done();
  if (e != hipSuccess) return fail(TRE_EHIP, "tss_stream launch: %s", hipGetErrorString(e));
  return TRE_OK;
}

// ws, ws_bytes: scratch the caller holds for the segmented path; without it
// the call takes a kept block
static int launch_stream(const tre_events* ev, const StreamParams& p, hipStream_t st, char* ws = nullptr,
                         size_t ws_bytes = 0) {
  const bool stage = p.stage64 || p.stage32 || p.sflags;
  const bool cells = p.prefill || p.decode || p.a_int || p.w_int || p.tss64 || p.tss32 || p.flags;
  const SegPlan g = seg_plan(ev, stage, cells);
  if (g.nseg && ws) {
    if (g.bytes <= ws_bytes) return launch_segments(ev, g, p, stage, ws, st);
  } else if (g.nseg) {
    const Scratch sx(ev->device, g.bytes, st);
    if (sx.get()) return launch_segments(ev, g, p, stage, sx.get(), st);
  }
  const size_t lds = stream_lds(ev, stage);
  LaunchTimer lt("tss_stream", st);
  const int waves = stream_waves(ev->n_traces);
  if (stage)
    hipLaunchKernelGGL((tss_stream_stage<kStreamWaves, kStreamEPT>), dim3(ev->n_traces),
                       dim3(kStreamWaves * 64), lds, st, p);
  else if (waves == 16 && cells)
    hipLaunchKernelGGL((tss_stream<16, kStreamEPT, true>), dim3(ev->n_traces), dim3(16 * 64), lds, st, p);
  else if (waves == 16)
    hipLaunchKernelGGL((tss_stream<16, kStreamEPT, false>), dim3(ev->n_traces), dim3(16 * 64), lds, st, p);
  else if (waves == 8 && cells)
    hipLaunchKernelGGL((tss_stream<8, kStreamEPT, true>), dim3(ev->n_traces), dim3(8 * 64), lds, st, p);
  else if (waves == 8)
    hipLaunchKernelGGL((tss_stream<8, kStreamEPT, false>), dim3(ev->n_traces), dim3(8 * 64), lds, st, p);
  else if (cells)
    hipLaunchKernelGGL((tss_stream<kStreamWaves, kStreamEPT, true>), dim3(ev->n_traces),
                       dim3(kStreamWaves * 64), lds, st, p);
  else
    hipLaunchKernelGGL((tss_stream<kStreamWaves, kStreamEPT, false>), dim3(ev->n_traces),
                       dim3(kStreamWaves * 64), lds, st, p);
  const hipError_t e = hipGetLastError();
  lt.done();
  if (e != hipSuccess) return fail(TRE_EHIP, "tss_stream launch: %s", hipGetErrorString(e));
  return TRE_OK;
}

// the actuation model in whole windows (delays rounded up)
struct ActWindows {
  int32_t wake_w, sleep_w;
  const int32_t* footprint;
  const uint64_t* veto;
};

static int act_windows(const tre_events* ev, const tre_actuation* act, ActWindows* aw) {
  if (!act) return fail(TRE_EINVAL, "NULL actuation model");
  if (act->wake_ms < 0 || act->sleep_ms < 0)
    return fail(TRE_EINVAL, "actuation delays must be >= 0");
  const int64_t win = ev->cfg.window_ms;
  // whole windows, rounded up; a transition completing after the last window
  // never counts, so the delays are capped just past the trace
  const int64_t cap = ev->n_windows + 1;
  auto to_windows = [&](int64_t ms) { return ms > cap * win ? cap : (ms + win - 1) / win; };
  aw->wake_w = (int32_t)to_windows(act->wake_ms);
  aw->sleep_w = (int32_t)to_windows(act->sleep_ms);
  aw->footprint = act->footprint;
  aw->veto = act->veto;
  return TRE_OK;
}

// Scenarios up to which each gets a workgroup (rebalance_ordered): of four waves
// up to 32 models, six of them a CU by LDS and registers; above of eight, since
// ordering a tick costs an instruction stream per model. The folds' cost hardly
// grows with the models, so the line falls with them. Measured, one wave a
// scenario / this, us for 360 ticks (240 where marked *, with many moves, as the
// generator's workloads have them): 8 models: 1024 scenarios 312 / 143, 1536 341 /
// 169, 2048 341 / 276; under actuation 1536 413 / 255, 2048 414 / 429; 16 models:
// 2048 368 / 317; 24 models: 1024 374 / 307, 1536 407 / 416; 32 models: 768 398 /
// 317 (seldom moving 337 / 302, *589 / 267), 1024 seldom moving 336 / 361; 33
// models: 512 402 / 368 (*591 / 325), 768 401 / 542; 48 models: 256 444 / 303
// (*553 / 261), 512 443 / 489; 64 models: 256 442 / 369 (seldom moving 371 / 368,
// *576 / 286), 1 365 / 354 (seldom moving 323 / 350), 512 444 / 627.
static uint32_t ord_scenarios(int M, bool act) {
  return M <= 16 ? (act ? 1536 : 2048) : M <= 24 ? 1024 : M <= 32 ? 768 : M <= 40 ? 512 : 256;
}

static int launch_rebalance(const tre_events* ev, const tre_profile* prof, const double* vals,
                            const uint8_t* flags, const tre_scenario* sc, uint32_t n_sc,
                            const tre_ctl_out* out, const ActWindows* aw, hipStream_t st,
                            const uint32_t* sc_count = nullptr) {
  CtlParams c{};
  c.sc_count = sc_count;
  c.prof = prof;
  c.sc = sc;
  c.n_sc = n_sc;
  c.vals = vals;
  c.flags = flags;
  c.tick_window = ev->d_tick_window;
  c.tick_kind = ev->d_tick_kind;
  c.n_ticks = (int32_t)ev->n_ticks;
  c.n_windows = (int32_t)ev->n_windows;
  c.M = ev->cfg.n_models;
  c.budget = ev->cfg.budget;
  c.n_traces = ev->n_traces;
  c.moves = out->moves;
  c.move_cap = out->move_cap;
  c.n_moves = out->n_moves;
  c.r_final = out->r_final;
  c.r_windows = out->r_windows;
  if (aw) {
    c.wake_w = aw->wake_w;
    c.sleep_w = aw->sleep_w;
    c.footprint = aw->footprint;
    c.veto = aw->veto;
  }
  // one wave per scenario, four per workgroup
  const dim3 grid((unsigned)(((uint64_t)n_sc + 3) / 4)), block(256);
  LaunchTimer lt("rebalance", st);
  const bool ordered = n_sc <= ord_scenarios(c.M, aw != nullptr);
  if (ordered && c.M > 32 && aw)
    hipLaunchKernelGGL((rebalance_ordered<true, 7>), dim3(n_sc), dim3(64 * 8), 0, st, c);
  else if (ordered && c.M > 32)
    hipLaunchKernelGGL((rebalance_ordered<false, 7>), dim3(n_sc), dim3(64 * 8), 0, st, c);
  else if (ordered && aw)
    hipLaunchKernelGGL((rebalance_ordered<true, 3>), dim3(n_sc), dim3(64 * 4), 0, st, c);
  else if (ordered)
    hipLaunchKernelGGL((rebalance_ordered<false, 3>), dim3(n_sc), dim3(64 * 4), 0, st, c);
  else if (aw)
    hipLaunchKernelGGL(rebalance<true>, grid, block, 0, st, c);
  else
    hipLaunchKernelGGL(rebalance<false>, grid, block, 0, st, c);
  const hipError_t e = hipGetLastError();
  lt.done();
  if (e != hipSuccess) return fail(TRE_EHIP, "rebalance launch: %s", hipGetErrorString(e));
  return TRE_OK;
}

static int check_ctl_out(const tre_ctl_out* out, uint32_t n_sc) {
  if (!out) return fail(TRE_EINVAL, "NULL control outputs");
  if (n_sc && (!out->n_moves || !out->r_final || !out->r_windows || (out->move_cap && !out->moves)))
    return fail(TRE_EINVAL, "NULL control output array");
  return TRE_OK;
}

extern "C" int tre_eval_tss(const tre_events* ev, const tre_profile* prof, const tre_tss_out* out,
                            void* stream) {
  if (!ev || !prof || !out) return fail(TRE_EINVAL, "tre_eval_tss: NULL argument");
  int rc = check_device(ev);
  if (rc) return rc;
  StreamParams p = stream_params(ev, prof);
  p.prefill = out->prefill;
  p.decode = out->decode;
  p.a_int = out->a_int;
  p.w_int = out->w_int;
  p.tss64 = out->tss64;
  p.tss32 = out->tss32;
  p.flags = out->flags;
  return launch_stream(ev, p, (hipStream_t)stream);
}

extern "C" int tre_eval_stage(const tre_events* ev, const tre_profile* prof, double* stage64, float* stage32,
                              uint8_t* flags, void* stream) {
  if (!ev || !prof) return fail(TRE_EINVAL, "tre_eval_stage: NULL handle or profiles");
  if (!stage64 && !stage32 && !flags) return fail(TRE_EINVAL, "tre_eval_stage: no output");
  if (((uintptr_t)stage64 & 15) || ((uintptr_t)stage32 & 7))
    return fail(TRE_EINVAL, "tre_eval_stage: stage64 needs 16-byte, stage32 8-byte alignment");
  int rc = check_device(ev);
  if (rc) return rc;
  StreamParams p = stream_params(ev, prof);
  p.stage64 = stage64;
  p.stage32 = stage32;
  p.sflags = flags;
  return launch_stream(ev, p, (hipStream_t)stream);
}

static int rebalance_impl(const tre_events* ev, const tre_profile* prof, const double* tss64,
                          const uint8_t* flags, const tre_scenario* sc, uint32_t n_scenarios,
                          const tre_actuation* act, const tre_ctl_out* out, void* stream,
                          const char* who) {
  if (!ev || !prof || !tss64 || !flags) return fail(TRE_EINVAL, "%s: NULL argument", who);
  if (n_scenarios && !sc) return fail(TRE_EINVAL, "%s: NULL scenarios", who);
  int rc = check_ctl_out(out, n_scenarios);
  if (rc) return rc;
  rc = check_device(ev);
  if (rc) return rc;
  ActWindows aw;
  if (act && (rc = act_windows(ev, act, &aw))) return rc;
  if (n_scenarios == 0) return TRE_OK;
  return launch_rebalance(ev, prof, tss64, flags, sc, n_scenarios, out, act ? &aw : nullptr,
                          (hipStream_t)stream);
}

static int sweep_impl(const tre_events* ev, const tre_profile* prof, const tre_scenario* sc,
                      uint32_t n_scenarios, const tre_actuation* act, const tre_ctl_out* out,
                      float* tss32, void* ws, size_t ws_bytes, void* stream, const char* who,
                      bool own_scratch = false) {
  if (!ev || !prof) return fail(TRE_EINVAL, "%s: NULL argument", who);
  if (n_scenarios && !sc) return fail(TRE_EINVAL, "%s: NULL scenarios", who);
  int rc = check_ctl_out(out, n_scenarios);
  if (rc) return rc;
  rc = check_device(ev);
  if (rc) return rc;
  ActWindows aw;
  if (act && (rc = act_windows(ev, act, &aw))) return rc;
  size_t need = 0;
  tre_workspace_size(ev, n_scenarios, &need);
  if (!ws || ws_bytes < need)
    return fail(TRE_ENOMEM, "workspace of %zu bytes is smaller than the %zu needed", ws_bytes, need);
  if ((uintptr_t)ws & 7) return fail(TRE_EINVAL, "workspace must be 8-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  StreamParams p = stream_params(ev, prof);
  p.tss32 = tss32;
  p.snap = (double*)ws;
  // without the actuation model, a trace with exactly one scenario replays
  // it in the stream (rebalance skips it)
  uint32_t* count = nullptr;
  if (n_scenarios && !act) {
    p.sc = sc;
    p.budget = ev->cfg.budget;
    p.moves = out->moves;
    p.move_cap = out->move_cap;
    p.n_moves = out->n_moves;
    p.r_final = out->r_final;
    p.r_windows = out->r_windows;
  }
  // (with one trace the host knows: no map)
  if (n_scenarios == 1 && !act && ev->n_traces == 1) {
    p.ctl_one = 1;
  } else if (n_scenarios && !act && ev->n_traces > 1) {
    count = (uint32_t*)((char*)ws + snapshot_bytes(ev));
    uint32_t* first = count + ev->n_traces;
    hipLaunchKernelGGL(zero_u32, dim3((ev->n_traces + 255) / 256), dim3(256), 0, st, count, ev->n_traces);
    hipLaunchKernelGGL(sweep_map, dim3((n_scenarios + 255) / 256), dim3(256), 0, st, sc, n_scenarios,
                       ev->n_traces, count, (uint32_t*)first);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TRE_EHIP, "sweep_map launch: %s", hipGetErrorString(e));
    p.sc_count = count;
    p.sc_first = first;
  }
  // own_scratch: what lies past the sweep's own part of ws serves the segments
  const size_t used = (need + 255) & ~(size_t)255;
  if (own_scratch)
    rc = launch_stream(ev, p, st, (char*)ws + used, ws_bytes > used ? ws_bytes - used : 0);
  else
    rc = launch_stream(ev, p, st);
  if (rc || n_scenarios == 0 || p.ctl_one) return rc;
  return launch_rebalance(ev, prof, (const double*)ws, nullptr, sc, n_scenarios, out,
                          act ? &aw : nullptr, st, count);
}

extern "C" int tre_rebalance(const tre_events* ev, const tre_profile* prof, const double* tss64,
                             const uint8_t* flags, const tre_scenario* sc, uint32_t n_scenarios,
                             const tre_ctl_out* out, void* stream) {
  return rebalance_impl(ev, prof, tss64, flags, sc, n_scenarios, nullptr, out, stream, "tre_rebalance");
}

extern "C" int tre_sweep(const tre_events* ev, const tre_profile* prof, const tre_scenario* sc,
                         uint32_t n_scenarios, const tre_ctl_out* out, float* tss32, void* ws,
                         size_t ws_bytes, void* stream) {
  return sweep_impl(ev, prof, sc, n_scenarios, nullptr, out, tss32, ws, ws_bytes, stream, "tre_sweep");
}

// ------------------------------------------------ sweep without allocation
// The sweep's scratch (the per-tick smoothed TSS snapshot) in a static
// device array for callers that cannot allocate. Each GPU the library runs
// on holds its own copy until the process ends; its device address is
// looked up once per device, with that device current, at the entry
// point's first call there, and only that address is used afterwards.
static __device__ __align__(256) unsigned char scratch[TRE_NOALLOC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[256];  // per device ordinal, NULL until looked up
}  // namespace

static int scratch_for(int dev, void** out) {
  if (dev < 0 || dev >= 256) return fail(TRE_EINVAL, "device ordinal %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(TRE_EHIP, "hipGetSymbolAddress of the static scratch: %s", hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return TRE_OK;
}

extern "C" int tre_sweep_noalloc(const tre_events* ev, const tre_profile* prof, const tre_scenario* sc,
                                 uint32_t n_scenarios, const tre_ctl_out* out, float* tss32, void* stream) {
  if (!ev) return fail(TRE_EINVAL, "tre_sweep_noalloc: NULL handle");
  int rc = check_device(ev);  // the handle's device is the current one
  if (rc) return rc;
  size_t need = 0;
  tre_workspace_size(ev, n_scenarios, &need);
  if (need > (size_t)TRE_NOALLOC_SCRATCH_BYTES)
    return fail(TRE_ENOMEM, "tre_sweep_noalloc: the sweep needs %zu bytes of scratch, above the static %zu",
                need, (size_t)TRE_NOALLOC_SCRATCH_BYTES);
  void* ws = nullptr;
  if ((rc = scratch_for(ev->device, &ws))) return rc;
  tre_internal::NoTimingScope quiet;  // no event objects are created for this call
  return sweep_impl(ev, prof, sc, n_scenarios, nullptr, out, tss32, ws, (size_t)TRE_NOALLOC_SCRATCH_BYTES, stream,
                    "tre_sweep_noalloc", true);
}

extern "C" int tre_rebalance_act(const tre_events* ev, const tre_profile* prof, const double* tss64,
                                 const uint8_t* flags, const tre_scenario* sc, uint32_t n_scenarios,
                                 const tre_actuation* act, const tre_ctl_out* out, void* stream) {
  if (!act) return fail(TRE_EINVAL, "tre_rebalance_act: NULL actuation model");
  return rebalance_impl(ev, prof, tss64, flags, sc, n_scenarios, act, out, stream, "tre_rebalance_act");
}

extern "C" int tre_sweep_act(const tre_events* ev, const tre_profile* prof, const tre_scenario* sc,
                             uint32_t n_scenarios, const tre_actuation* act, const tre_ctl_out* out,
                             float* tss32, void* ws, size_t ws_bytes, void* stream) {
  if (!act) return fail(TRE_EINVAL, "tre_sweep_act: NULL actuation model");
  return sweep_impl(ev, prof, sc, n_scenarios, act, out, tss32, ws, ws_bytes, stream, "tre_sweep_act");
}

extern "C" int tre_check_actuation(const tre_events* ev, const tre_profile* prof,
                                   const tre_actuation* act) {
  if (!ev || !prof || !act) return fail(TRE_EINVAL, "tre_check_actuation: NULL argument");
  int rc = check_device(ev);
  if (rc) return rc;
  ActWindows aw;
  if ((rc = act_windows(ev, act, &aw))) return rc;
  const size_t M = (size_t)ev->cfg.n_models;
  std::vector<tre_profile> hp((size_t)ev->n_traces * M);
  HIP_TRY(hipMemcpy(hp.data(), prof, hp.size() * sizeof(tre_profile), hipMemcpyDeviceToHost));
  std::vector<int32_t> g(hp.size(), 1);
  if (act->footprint)
    HIP_TRY(hipMemcpy(g.data(), act->footprint, g.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
  for (uint32_t t = 0; t < ev->n_traces; ++t) {
    long long gsum = 0;
    for (size_t m = 0; m < M; ++m) {
      const int32_t gm = g[t * M + m];
      if (gm < 1 || gm > ev->cfg.budget)
        return fail(TRE_EINVAL, "trace %u model %zu: footprint %d outside 1 .. budget", t, m, gm);
      gsum += (long long)gm * hp[t * M + m].r_init;
    }
    if (gsum > ev->cfg.budget)
      return fail(TRE_EINVAL, "trace %u: initial replicas hold %lld GPUs, above the budget %d", t,
                  gsum, ev->cfg.budget);
  }
  return TRE_OK;
}
