// Persistent per-frame kernel of pROST (Sec. 3.3, Steps 1-3, plus the 3x3
// median of Sec. 3.4) for one video stream.
//
// One launch processes one frame (or, in the sequence form, several frames
// with the tile kept in registers between them and U stored after the last
// one).  The m x k subspace U is split into workgroup tiles of `tpw` pixels
// (all colour entries of a pixel stay in one tile); each thread keeps NR rows
// of U in registers for the whole frame (K floats per row, or K bfloat16
// pairs per two rows with bfloat16 storage), so U is read from HBM once and
// written once per frame (per launch in the sequence form).
// The frame's sequence of dependent reductions runs as gang-wide reductions
// between all workgroups of the launch (cooperative launch, so all of them
// are resident):
//   for each CG step j:  A: g = -U^T(w phi'(r)), f = sum w phi(r)
//                        B: d^T H d = sum w c(r) (u.d)^2
//   eta pass:            a = U^T eta, ||eta||^2, f at the final y
// The 3x3 median of a frame's labels runs in the next frame, in the wavefronts
// that do not wait in its first single-value exchange (at its start where the
// weights come from it; in mask_kernel when the mask is asked for first), which
// saves the exchange that would otherwise separate the label writes from it.
// Every workgroup reduces the published partials in the same fixed order, so
// all of them hold bit-identical k-vectors without a broadcast step.  Waiting
// workgroups spin on epoch-tagged float64 slots (each thread on its own
// values, no barrier inside the wait, bounded by one wall-clock time-out per
// exchange).
#pragma once

#include <utility>

#include "prost_device.hpp"
#include "../../include/prost.h"

namespace prost {
inline namespace PROST_BLOCK_NS {

// A pointer that was itself loaded from memory (frame tables, the descriptors of
// a batch), in the global address space: the compiler knows that only of kernel
// arguments, and reaches through other pointers with flat instructions, which
// wait for the LDS and the memory counters both.
template <typename T>
__device__ __forceinline__ T* global_ptr(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p;
}

struct FrameArgs {
  void* U;               // K planes of ldU entries (storage type)
  const void* x;         // frame, m entries (storage type); used when xtab is NULL
  const void* const* xtab;  // ring of `ring` frame pointers, frame n at xtab[n % ring]
  int ring;
  uint8_t* lab;          // raw labels, P bytes (read: previous frame, write: this frame)
  uint8_t* mask;         // median-filtered mask, P bytes
  double* y;             // k coefficients (float64 state)
  long long* nframe;     // frame counter
  pros_stats* stats;     // statistics of the frame
  double* part;          // (2 * G + kExtraSlots) * kSlot doubles of workgroup partials
  unsigned* sync;        // [0] arrival counter, [1] counter base, [2] error bits, [3] epoch base,
                         // [4] 1: the mask already is the median of the labels (mask_kernel),
                         // [5] rejected frames since the epochs last went back (frame_epochs)
  long long ldU;
  int m, P, C, W, H, k;
  int G, tpw;
  CostParams cp;
  float delta, omega;
  double t_init, t_min, tau;
  int J;
  int labels_after_update;
  int weights_from_filtered;
  long long timeout;     // wall-clock ticks a barrier may wait
  long long* trace;      // optional per-tile timestamps (diagnostics), 64 per tile
  int pair_aligned;      // bfloat16: row pairs are aligned 32-bit words (U planes and frame)
  float* pre_mean;       // pre-processing (Sec. 3.4): running average (m), NULL when off
  float* pre_m2;         // per-entry sum of squared deviations (m)
  double* pre_stat;      // [0] entry sum of pre_m2, [1] initialization frames accumulated
  int i_init;            // length of the initialization phase
  float* score;          // optional: |r'| of every entry after Step 3 (m floats), or NULL
  int ysolve;            // 0: CG with the PR+ direction, 1: gradient descent
  int sync_mode;         // 0: counter barrier + all-read, 1: tagged gather/broadcast,
                         // 2: two-level tagged gather (groups of tiles with equal t % 8),
                         // 3: every workgroup reads all tagged partials
  int curv;              // curvature schedule of a CG step: 0 = d^T H d in a second pass
                         // and exchange, 1 = H reduced with the gradient (one wide exchange)
  const void* const* seq;  // frames 1 .. nseq - 1 of a sequence launch (frame 0 is x), device array;
                           // with xtab (batched form) the ring is read instead
  int nseq;                // frames processed by this launch (1: one frame)
};

constexpr int kReplicas = 8;      // copies of a gathered result (spread the pollers)
constexpr int kGroups = 8;        // groups of the two-hop exchange
// slots beyond 2 G: two alternating sets of the kGroups group sums in kReplicas copies
constexpr int kExtraSlots = 2 * kGroups * kReplicas;

// Shared k-space state of one workgroup (all float64 unless noted).
constexpr int kMaxNR = 32;   // register rows per thread (bfloat16 pairs at small k)
template <int K>
struct KSpace {
  double y[K];
  double d[K];
  double gp[K];     // previous gradient
  double dp[K];     // previous direction
  double a[K];      // U^T eta
  double red[kSlot];
  double gd;        // g . d of the current step
  double gg;        // g . g of the latest gradient
  double t;         // step size of this frame (Sec. 3.4)
  float df[K];      // direction (float) for the row passes
  float vf[K];      // v = y/||y||
  float af[K];      // a (float)
  float yf[K];
  float scal[8];    // row-pass scalars
  int flag[4];      // [0] stop CG, [1] bad frame, [2] do update
  double pre_sum;   // pre-processing: entry sum of the deviation sums after this frame
  float pre_inv_s;  // 1 / scale applied to this frame
  float pre_inv_n;  // 1 / (frames accumulated including this one)
  int pre_upd;      // this frame joins the running average
};

// Workgroup-shared scratch of one frame tile (sized for the largest k / NR).
// Wide exchange (IRLS step, one-exchange curvature schedule): g, f and the upper triangle of H
// (K + 1 + K (K + 1) / 2 <= 153 values) in vectors of kWideMax float64.
constexpr int kWideChunks = 5;
constexpr int kWideMax = kWideChunks * kSlot;
constexpr int kWideIn = kWideMax + kSlot;   // room for the last zero-padded chunk

struct FrameSmem {
  KSpace<kMaxK> ks;
  double red[kWaves][kSlot];   // wavefront partials of a vector exchange
  double red1[kWaves];         // ... of a single-value exchange
  double got[kWaves][kSlot];   // gathered sums, one row per wavefront
  double one;                  // total of a single-value exchange
  double wg[kSlot];
  double big[kBlock];          // one float64 per thread (gathers)
  int ctl[4];                  // [2] the gang gave up waiting (checked after the barrier that follows an exchange)
  uint8_t flag[kBlock * kMaxNR];
  double wide_in[kWideIn];     // wide exchange: this workgroup's partials
  double wide_out[kWideMax];   // wide exchange: gang totals
  double hs[kMaxK][kMaxK + 1]; // IRLS: augmented [H | -g] for the k-space solve
};


// Diagnostics: wall-clock timestamp `idx` (< 64) of a tile, by thread 0.
__device__ __forceinline__ void trace_point(const FrameArgs& a, int tile, int idx) {
  if (a.trace && thread_index() == 0 && (unsigned)idx < 64u) a.trace[(size_t)tile * 64 + idx] = wall_clock64();
}

// Waits for component `comp` of the tagged slots q = row0, row0 + rs, ...
// (q < n, slot q at base + q * qstride) to carry epoch ep and returns their
// sum in slot order.  Each thread spins on its own values with no barrier
// inside the wait (a barrier per poll round made every round cost a memory
// round trip plus two workgroup barriers); `bad` is set on time-out or when
// another workgroup has raised the time-out bit.
__device__ __forceinline__ double spin_sum(const double* base, int n, int rs, size_t qstride, int comp, int row0,
                                           unsigned ep, const FrameArgs& a, int& bad) {
  double v = 0.0;
  const long long t0 = now_ticks();
  for (int q = row0; q < n; q += rs) {
    const double* p = base + (size_t)q * qstride + comp;
    double x = ld_tagged(p);
    unsigned spins = 0;
    while (tag_of(x) != ep) {
      x = ld_tagged(p);
      if ((++spins & 63u) == 0 &&
          (now_ticks() - t0 > a.timeout ||
           (__hip_atomic_load(&a.sync[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrTimeout))) {
        bad = 1;
        return v;
      }
    }
    v += untag(x);
  }
  return v;
}

// Uniform end of a spin wait: false in every thread (and the gang's
// time-out bit raised) if any thread gave up.  The barrier also publishes
// the threads' s_big entries.
__device__ __forceinline__ bool spin_end(int bad, const FrameArgs& a) {
  if (__syncthreads_or(bad)) {
    if (thread_index() == 0) __hip_atomic_fetch_or(&a.sync[2], kErrTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  return true;
}

// Workgroup + gang reduction of L float partials held by every thread.
// Result (float64, identical in every workgroup) lands in s_out[0..L).
// Tagged gather/broadcast: every workgroup publishes its tagged partial
// vector; the gang's tile 0 polls all of them, sums them in tile order and
// publishes the tagged totals in kReplicas copies that the other workgroups
// poll.  No shared counter, so no serialised atomics on one address.
// `fenced` adds release/acquire fences around the exchange so that plain
// global writes made before it (labels) are visible after it.
template <int L>
__device__ __forceinline__ bool gang_reduce_tagged(const double* wg_sum, const FrameArgs& a, const int tile,
                                                   int& nbar, unsigned ebase, double* s_big,
                                                   double* s_out, int* s_ctl, bool fenced) {
  const int tid = thread_index();
  const int lane = tid & 63;
  const int wv = tid >> 6;
  ++nbar;
  const unsigned ep = (ebase + (unsigned)nbar) & 0xFFu;
  double* slots = a.part;                                 // G slots
  double* rep = a.part + (size_t)2 * a.G * kSlot;         // kReplicas slots
  if (fenced) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  if (tid < L) st_tagged(&slots[(size_t)tile * kSlot + tid], tag_value(wg_sum[tid], ep));
  if (tile == 0) {
    constexpr int kRows = kBlock / 32;
    const int comp = tid & 31, row0 = tid >> 5;
    int bad = 0;
    const double v = (comp < L) ? spin_sum(slots, a.G, kRows, kSlot, comp, row0, ep, a, bad) : 0.0;
    s_big[tid] = v;
    if (!spin_end(bad, a)) return false;
    if (tid < L) {
      double tot = 0.0;
#pragma unroll
      for (int r = 0; r < kRows; ++r) tot += s_big[r * 32 + tid];
      s_out[tid] = untag(tag_value(tot, ep));   // what every other workgroup will read
    }
    if (fenced) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
    __syncthreads();
    for (int q = tid; q < kReplicas * L; q += kBlock) {
      const int r = q / L, i = q - r * L;
      st_tagged(&rep[(size_t)r * kSlot + i], tag_value(s_out[i], ep));
    }
    __syncthreads();
    return true;
  }
  // other workgroups: poll their replica
  if (tid == 0) s_ctl[1] = 0;
  __syncthreads();
  if (tid < L) {
    const double* src = &rep[(size_t)(tile % kReplicas) * kSlot + tid];
    const long long t0 = now_ticks();
    unsigned spins = 0;
    while (true) {
      const double x = ld_tagged(src);
      if (tag_of(x) == ep) {
        s_out[tid] = untag(x);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      if ((++spins & 63u) == 0) {
        if ((__hip_atomic_load(&a.sync[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrTimeout) ||
            now_ticks() - t0 > a.timeout) {
          __hip_atomic_fetch_or(&a.sync[2], kErrTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          s_ctl[1] = 1;
          break;
        }
      }
    }
  }
  if (fenced) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __syncthreads();
  return s_ctl[1] == 0;
}

// Compiler and LDS order within one wavefront (its LDS accesses execute in
// order; nothing is waited for).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The waits of an exchange: one clock for all of its gathers, slots and
// components, read where the exchange begins: its latency is behind the
// workgroup's own sums there.  A frame takes 0.5 us more with it than with a
// clock for every value (160x120x3 to 640x480x3), 0.6 with the read next to the
// gather, 1.2 with one that the first missing value starts.
struct GangWait {
  long long t0;
  int bad;   // gave up
};

// Waits for *p to carry epoch ep, x being what a load of it returned; the
// value without its tag, or 0 with w.bad set after the time-out (what is still
// missing then costs 64 polls each).
__device__ __forceinline__ double wait_tagged(const double* p, double x, unsigned ep, const FrameArgs& a,
                                              GangWait& w) {
  unsigned spins = 0;
  while (tag_of(x) != ep) {
    x = ld_tagged(p);
    if ((++spins & 63u) == 0 &&
        (now_ticks() - w.t0 > a.timeout ||
         (__hip_atomic_load(&a.sync[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrTimeout))) {
      w.bad = 1;
      return 0.0;
    }
  }
  return untag(x);
}

// Two of the tagged slots q0 and q1 = q0 + dq (where they are below n), their
// loads both in flight before either is waited for: component comp (< L) into
// v, and component 16 + comp, if there is one, into vx.
template <int L>
__device__ __forceinline__ void poll_pair(const double* base, int n, size_t qstride, int q0, int dq, int comp,
                                          unsigned ep, const FrameArgs& a, double& v, double& vx, GangWait& w) {
  const double* p0 = base + (size_t)q0 * qstride + comp;
  const double* p1 = p0 + (size_t)dq * qstride;
  const bool on0 = comp < L && q0 < n, on1 = comp < L && q0 + dq < n;
  const bool ex0 = 16 + comp < L && q0 < n, ex1 = 16 + comp < L && q0 + dq < n;
  double x0 = 0.0, x1 = 0.0, e0 = 0.0, e1 = 0.0;
  if (on0) x0 = ld_tagged(p0);
  if (on1) x1 = ld_tagged(p1);
  if (L > 16 && ex0) e0 = ld_tagged(p0 + 16);
  if (L > 16 && ex1) e1 = ld_tagged(p1 + 16);
  if (on0) v += wait_tagged(p0, x0, ep, a, w);
  if (on1) v += wait_tagged(p1, x1, ep, a, w);
  if (L > 16 && ex0) vx += wait_tagged(p0 + 16, e0, ep, a, w);
  if (L > 16 && ex1) vx += wait_tagged(p1 + 16, e1, ep, a, w);
}

// Sum of the slots q0, q0 + dq, q0 + 2 dq, ... below n, two at a time.
template <int L>
__device__ __forceinline__ void poll_slots(const double* base, int n, size_t qstride, int q0, int dq, int comp,
                                           unsigned ep, const FrameArgs& a, double& v, double& vx, GangWait& w) {
  for (int q = q0; q < n; q += 2 * dq) poll_pair<L>(base, n, qstride, q, dq, comp, ep, a, v, vx, w);
}

// Raises the gang's time-out bit and the workgroup's flag if a lane of this
// wavefront gave up.
__device__ __forceinline__ void wave_give_up(const GangWait& w, const FrameArgs& a, FrameSmem& sm) {
  if (__any(w.bad) && (thread_index() & 63) == 0) {
    sm.ctl[2] = 1;
    __hip_atomic_fetch_or(&a.sync[2], kErrTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Gather by the whole workgroup: the sum of n tagged slots, one row of sums per
// wavefront into sm.got.  Lane l of wavefront w takes component l % 16 of slots
// 4 w + l / 16, then those 4 kWaves further on: the slots' lines spread over all
// wavefronts (measured: one wavefront that polls 32 lines of 16 values takes
// longer than eight that poll four each), two in flight per lane.  Ends with a
// barrier; after a time-out sm.ctl[2] is set (a plain barrier and a flag: the
// barrier that also reduces a predicate takes 0.2 us more).
template <int L>
__device__ __forceinline__ void gather_slots(const double* base, int n, size_t qstride, unsigned ep,
                                             const FrameArgs& a, FrameSmem& sm, long long t0) {
  const int lane = thread_index() & 63, wv = thread_index() >> 6;
  const int comp = lane & 15;
  constexpr int kRows = 4 * kWaves;
  double v = 0.0, vx = 0.0;
  GangWait w{t0, 0};
  poll_slots<L>(base, n, qstride, 4 * wv + (lane >> 4), kRows, comp, ep, a, v, vx, w);
  v = swap_sum<16>(swap_sum<32>(v));
  if (L > 16) vx = swap_sum<16>(swap_sum<32>(vx));
  if (lane < 16) {
    sm.got[wv][comp] = v;
    if (16 + comp < L) sm.got[wv][16 + comp] = vx;
  }
  wave_give_up(w, a, sm);
  __syncthreads();
}

// The slot set of an exchange: it alternates with the epoch, so a workgroup
// that is one exchange ahead never writes what another still reads.  Frames
// whose CG steps go through the wide exchange have one regular exchange per
// launch and keep to set 0, which every frame then rewrites.
__device__ __forceinline__ int slot_set(const FrameArgs& a, unsigned ep) {
  return (a.ysolve == 2 || a.curv == 1) ? 0 : (int)(ep & 1);
}

// Gang-wide sum of L float partials per thread in the tagged exchanges 2 and 3.
// The first wavefront publishes the workgroup's sums and, on return, holds the
// totals in s_out[0..L - LATE) (LDS, written by itself): the k-space step that
// follows runs in that wavefront, and the barrier at its end is the one that the
// other wavefronts wait at, so an exchange costs two barriers (three in a
// workgroup that gathers) instead of five.  After that barrier the caller checks
// sm.ctl[2].
//   3: every workgroup gathers all G slots (two alternating sets).
//   2: the tiles t = x mod 8 form group x, whose first tile gathers them and
//      writes the group sum into eight copies, one for each residue of the
//      readers (two alternating sets); every first wavefront sums the groups.
// The last LATE values (those that would take a second line of every slot) only
// tile 0 needs, after the next barrier: its second wavefront sums them from the
// slots meanwhile.  (As a 17th value of the exchange the final cost made the eta
// exchange of k = 15 take 1.1 us longer than the gradient's.)
// Per exchange with nothing in between (us): 226 workgroups 2.9 -> 2.6, 57:
// 2.5 -> 2.3, 29 (exchange 3): 2.4 -> 1.9; with the exchanges below, a frame
// with its mask read takes 89 us instead of 106 at 640x480x3, k = 15, float32,
// 46 instead of 64 at 320x240x3, k = 10 (ordinary dispatch), 59 instead of 67
// at 160x120x3, k = 15.
template <int L, int LATE>
__device__ __forceinline__ void gang_reduce_wave0(float (&acc)[L], const FrameArgs& a, const int tile, int& nbar,
                                                  unsigned ebase, FrameSmem& sm, double* s_out) {
  constexpr int LM = L - LATE;
  const int tid = thread_index(), lane = tid & 63, wv = tid >> 6;
  const long long t0 = now_ticks();
  {
    int comp;
    const float v = wave_reduce_scatter<L>(acc, comp);
    if (wave_rs_owner<L>(lane) && comp < L) sm.red[wv][comp] = (double)v;
  }
  ++nbar;
  const unsigned ep = (ebase + (unsigned)nbar) & 0xFFu;
  const int set = slot_set(a, ep);
  __syncthreads();
  double* slots = a.part + (size_t)(a.sync_mode == 3 && set ? a.G : 0) * kSlot;
  if (tid < L) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v += sm.red[q][tid];
    if (a.G == 1)
      s_out[tid] = v;   // a gang of one workgroup: its sums are the totals
    else
      st_tagged(&slots[(size_t)tile * kSlot + tid], tag_value(v, ep));
  }
  if (a.G == 1) {
    wave_order();
    return;
  }
  trace_point(a, tile, 24 + 3 * nbar);
  const int comp = lane & 15;
  if (a.sync_mode == 3) {
    gather_slots<LM>(slots, a.G, kSlot, ep, a, sm, t0);
    if (tid < LM) {
      double v = 0.0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) v += sm.got[q][tid];
      s_out[tid] = v;
    }
    wave_order();
  } else {
    double* gs = a.part + (size_t)(2 * a.G + set * kGroups * kReplicas) * kSlot;   // [copy][group]
    if (tile < kGroups) {   // group leader: members tile, tile + 8, ...
      const int n = (a.G - tile + kGroups - 1) / kGroups;
      gather_slots<LM>(slots + (size_t)tile * kSlot, n, (size_t)kGroups * kSlot, ep, a, sm, t0);
      if (wv == 0 && sm.ctl[2] == 0) {
        double v = 0.0, vx = 0.0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
          v += sm.got[q][comp];
          if (16 + comp < LM) vx += sm.got[q][16 + comp];
        }
        for (int c = lane >> 4; c < kReplicas; c += 4) {
          double* p = gs + (size_t)(c * kGroups + tile) * kSlot;
          if (comp < LM) st_tagged(p + comp, tag_value(v, ep));
          if (16 + comp < LM) st_tagged(p + 16 + comp, tag_value(vx, ep));
        }
      }
      trace_point(a, tile, 25 + 3 * (nbar - 1));
    }
    if (wv == 0) {
      double v = 0.0, vx = 0.0;
      GangWait w{t0, 0};
      poll_pair<LM>(gs + (size_t)(tile & (kReplicas - 1)) * kGroups * kSlot, min(kGroups, a.G), kSlot, lane >> 4, 4,
                    comp, ep, a, v, vx, w);
      v = swap_sum<16>(swap_sum<32>(v));
      if (LM > 16) vx = swap_sum<16>(swap_sum<32>(vx));
      if (lane < 16) {
        if (comp < LM) s_out[comp] = v;
        if (16 + comp < LM) s_out[16 + comp] = vx;
      }
      wave_give_up(w, a, sm);
      wave_order();
    }
  }
  if (LATE > 0 && tile == 0 && wv == 1) {
    GangWait w{t0, 0};
#pragma unroll
    for (int c = LM; c < L; ++c) {
      double v = 0.0, none = 0.0;
      poll_slots<1>(slots + c, a.G, kSlot, lane, 64, 0, ep, a, v, none, w);
      v = wave_sum(v);
      if (lane == 0) s_out[c] = v;
    }
    wave_give_up(w, a, sm);
  }
}

// Gang-wide sum of one float per thread in the tagged exchanges 2 and 3, in
// `total` of every thread.  Only the first wavefront waits for the gang (one
// slot per lane: with a single value per workgroup the lines need no spreading;
// 226 workgroups 2.9 -> 2.2 us, 57: 2.5 -> 1.7, 29: 2.4 -> 1.6 with nothing in
// between); the others run idle() meanwhile.  False when the gang gave up.
template <typename IDLE>
__device__ __forceinline__ bool gang_reduce_one(float acc, const FrameArgs& a, const int tile, int& nbar,
                                                unsigned ebase, FrameSmem& sm, double& total, IDLE idle) {
  const int tid = thread_index(), lane = tid & 63;
  const long long t0 = now_ticks();
  {
    float v[1] = {acc};
    int comp;
    const float w = wave_reduce_scatter<1>(v, comp);
    if (lane == 0) sm.red1[tid >> 6] = (double)w;
  }
  ++nbar;
  const unsigned ep = (ebase + (unsigned)nbar) & 0xFFu;
  __syncthreads();
  double v = 0.0;
  if (a.G == 1 || tid < 64) {
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v += sm.red1[q];
  }
  if (a.G == 1) {
    total = v;
    return true;
  }
  trace_point(a, tile, 24 + 3 * nbar);
  if (tid < 64) {
    const int set = slot_set(a, ep);
    double* slots = a.part + (size_t)(a.sync_mode == 3 && set ? a.G : 0) * kSlot;
    GangWait w{t0, 0};
    if (lane == 0) st_tagged(slots + (size_t)tile * kSlot, tag_value(v, ep));
    v = 0.0;
    double none = 0.0;
    if (a.sync_mode == 3) {
      poll_slots<1>(slots, a.G, kSlot, lane, 64, 0, ep, a, v, none, w);
    } else {
      double* gs = a.part + (size_t)(2 * a.G + set * kGroups * kReplicas) * kSlot;
      if (tile < kGroups) {
        const int n = (a.G - tile + kGroups - 1) / kGroups;
        poll_slots<1>(slots + (size_t)tile * kSlot, n, (size_t)kGroups * kSlot, lane, 64, 0, ep, a, v, none, w);
        v = wave_sum(v);
        if (!__any(w.bad) && lane < kReplicas) st_tagged(gs + (size_t)(lane * kGroups + tile) * kSlot, tag_value(v, ep));
        trace_point(a, tile, 25 + 3 * (nbar - 1));
        v = 0.0;
      }
      if (!__any(w.bad) && lane < min(kGroups, a.G)) {
        const double* p = gs + (size_t)((tile & (kReplicas - 1)) * kGroups + lane) * kSlot;
        v = wait_tagged(p, ld_tagged(p), ep, a, w);
      }
    }
    v = wave_sum(v);
    if (lane == 0) sm.one = v;
    wave_give_up(w, a, sm);
  } else {
    idle();
  }
  __syncthreads();
  total = sm.one;
  return sm.ctl[2] == 0;
}

// Poll n tagged vectors of LT values (vector q at base + q * qstride) until
// every value carries epoch ep; out[v] = sum over q in order.  Threads:
// value tid % kWideMax, vectors tid / kWideMax + 3 i.  Uniform exit.
__device__ __forceinline__ bool poll_sum_wide(const double* base, int n, int qstride, int LT, unsigned ep,
                                              const FrameArgs& a, double* s_big, double* out) {
  const int tid = thread_index();
  constexpr int kRowsW = kBlock / kWideMax;
  const int v = tid % kWideMax, row = tid / kWideMax;
  const bool act = row < kRowsW && v < LT;
  int bad = 0;
  const double acc = act ? spin_sum(base, n, kRowsW, (size_t)qstride, v, row, ep, a, bad) : 0.0;
  s_big[tid] = acc;
  if (!spin_end(bad, a)) return false;
  if (tid < LT) {
    double t = 0.0;
#pragma unroll
    for (int r = 0; r < kRowsW; ++r) t += s_big[r * kWideMax + tid];
    out[tid] = t;
  }
  __syncthreads();
  return true;
}

// Gang sum of LT (<= kWideMax) float64 values per workgroup, in the
// two-hop form of sync mode 2 (groups of tiles t = x mod 8), in its own
// region of the exchange buffer after the regular slots.  Every workgroup
// ends with bit-identical totals in out.
__device__ __forceinline__ bool gang_reduce_wide(const double* in, int LT, const FrameArgs& a, const int tile,
                                                 int& nbar, unsigned ebase, double* s_big, double* out) {
  const int tid = thread_index();
  ++nbar;
  if (a.G == 1) {   // a gang of one workgroup: its sums are the totals
    for (int q = tid; q < LT; q += kBlock) out[q] = in[q];
    __syncthreads();
    return true;
  }
  const unsigned ep = (ebase + (unsigned)nbar) & 0xFFu;
  const int x = tile & 7;
  const int ngrp = min(8, a.G);
  double* slots = a.part + (size_t)(2 * a.G + kExtraSlots) * kSlot;           // G vectors
  double* gs = slots + (size_t)a.G * kWideMax + (size_t)(nbar & 1) * 8 * kWideMax;   // 2 x 8 group sums
  for (int q = tid; q < LT; q += kBlock) st_tagged(&slots[(size_t)tile * kWideMax + q], tag_value(in[q], ep));
  if (tile < 8) {   // group leader: members x, x + 8, ...
    const int n = (a.G - x + 7) >> 3;
    if (!poll_sum_wide(slots + (size_t)x * kWideMax, n, 8 * kWideMax, LT, ep, a, s_big, out)) return false;
    for (int q = tid; q < LT; q += kBlock) st_tagged(&gs[(size_t)x * kWideMax + q], tag_value(out[q], ep));
  }
  return poll_sum_wide(gs, ngrp, kWideMax, LT, ep, a, s_big, out);
}

// Workgroup sum of L float partials (one value per thread each), float64
// result in wg_sum[0..L) (shared).
template <int L>
__device__ __forceinline__ void wg_reduce(float (&acc)[L], double (*s_red)[kSlot], double* wg_sum) {
  const int lane = thread_index() & 63;
  const int wv = thread_index() >> 6;
  int comp;
  const float v = wave_reduce_scatter<L>(acc, comp);
  if (wave_rs_owner<L>(lane) && comp < L) s_red[wv][comp] = (double)v;
  __syncthreads();
  if (thread_index() < L) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v += s_red[q][thread_index()];
    wg_sum[thread_index()] = v;
  }
  __syncthreads();
}

template <int L>
__device__ __forceinline__ bool gang_reduce_counter(float (&acc)[L], const FrameArgs& a, const int tile, int& nbar,
                                                    unsigned base, double (*s_red)[kSlot], double* s_big,
                                                    double* s_out, int* s_ctl) {
  const int lane = thread_index() & 63;
  const int wv = thread_index() >> 6;
  // 1. per wave
  {
    int comp;
    const float v = wave_reduce_scatter<L>(acc, comp);
    if (wave_rs_owner<L>(lane) && comp < L) s_red[wv][comp] = (double)v;
  }
  __syncthreads();
  double* slot = a.part + ((size_t)(nbar & 1) * a.G + tile) * kSlot;
  if (thread_index() < L) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v += s_red[q][thread_index()];
    __hip_atomic_store(&slot[thread_index()], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // 2. gang barrier
  ++nbar;
  if (!gang_barrier(a.sync, base + (unsigned)a.G * (unsigned)nbar, a.timeout, s_ctl)) return false;
  // 3. every workgroup sums all partials in the same order: thread t adds
  // component t % 32 of slots t / 32, t / 32 + kRows, ... (contiguous loads),
  // then the kRows partial sums of each component are added in order.
  // Plain (cached) loads: the barrier's acquire fence invalidated stale lines,
  // so the first workgroup of each XCD pulls the partials into its L2.
  const double* buf = a.part + (size_t)((nbar - 1) & 1) * a.G * kSlot;
  constexpr int kRows = kBlock / 32;
  const int comp = thread_index() & 31, row0 = thread_index() >> 5;
  double v = 0.0;
  if (comp < L)
    for (int w = row0; w < a.G; w += kRows) v += buf[(size_t)w * kSlot + comp];
  s_big[thread_index()] = v;
  __syncthreads();
  if (thread_index() < L) {
    double tot = 0.0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) tot += s_big[r * 32 + thread_index()];
    s_out[thread_index()] = tot;
  }
  __syncthreads();
  return true;
}

// The exchange runs in the first wavefront (gang_reduce_wave0 / _one): the
// tagged exchanges 2 and 3, and gangs of one workgroup.
__device__ __forceinline__ bool wave0_exchange(const FrameArgs& a) { return a.G == 1 || a.sync_mode >= 2; }

// Gang-wide sum of L float partials: the same float64 totals in every workgroup
// of the gang, in s_out[0..L) for the first wavefront.  The caller's next
// barrier makes them visible to the others; sm.ctl[2] is checked after it.  The
// last LATE of them reach tile 0 alone, and only with that barrier.
template <int L, int LATE = 0>
__device__ __forceinline__ bool gang_reduce(float (&acc)[L], const FrameArgs& a, const int tile, int& nbar,
                                            unsigned base, unsigned ebase, FrameSmem& sm, double* s_out) {
  trace_point(a, tile, 2 + 2 * nbar);
  bool ok = true;
  if (wave0_exchange(a)) {
    gang_reduce_wave0<L, LATE>(acc, a, tile, nbar, ebase, sm, s_out);
  } else if (a.sync_mode == 1) {
    wg_reduce<L>(acc, sm.red, sm.wg);
    ok = gang_reduce_tagged<L>(sm.wg, a, tile, nbar, ebase, sm.big, s_out, sm.ctl, false);
  } else {
    ok = gang_reduce_counter<L>(acc, a, tile, nbar, base, sm.red, sm.big, s_out, sm.ctl);
  }
  trace_point(a, tile, 1 + 2 * nbar);
  return ok;
}

// Gang-wide sum of one float, in `total` of every thread; idle() runs in the
// wavefronts that do not wait for the gang (not at all where all of them do:
// wave0_exchange() false or a gang of one).
template <typename IDLE>
__device__ __forceinline__ bool gang_reduce1(float acc, const FrameArgs& a, const int tile, int& nbar, unsigned base,
                                             unsigned ebase, FrameSmem& sm, double& total, IDLE idle) {
  trace_point(a, tile, 2 + 2 * nbar);
  bool ok;
  if (wave0_exchange(a)) {
    ok = gang_reduce_one(acc, a, tile, nbar, ebase, sm, total, idle);
  } else {
    float v[1] = {acc};
    if (a.sync_mode == 1) {
      wg_reduce<1>(v, sm.red, sm.wg);
      ok = gang_reduce_tagged<1>(sm.wg, a, tile, nbar, ebase, sm.big, sm.ks.red, sm.ctl, false);
    } else {
      ok = gang_reduce_counter<1>(v, a, tile, nbar, base, sm.red, sm.big, sm.ks.red, sm.ctl);
    }
    total = sm.ks.red[0];
  }
  trace_point(a, tile, 1 + 2 * nbar);
  return ok;
}

// 3x3 median of binary labels (>= 5 of the 9 neighbours, edges replicated,
// Sec. 3.4) for pixels [p0, p0 + npx) of a W x H image.
// COH: the labels were written in this launch by other workgroups, with
// device-coherent stores; read them with device-coherent loads.  Thread t0 of
// the nt that share the work.
template <bool COH = false>
__device__ __forceinline__ void median3x3_range(const uint8_t* __restrict__ lab, uint8_t* __restrict__ mask, int W,
                                                int H, int p0, int npx, int t0, int nt) {
  // kMedBatch pixels per thread at a time: their 9 kMedBatch loads are all
  // issued before the first is used (an entry past the tile loads the
  // tile's last pixel again and is not stored), so a tile costs one memory
  // latency per batch instead of one per pixel
  constexpr int kMedBatch = 3;
  for (int pl0 = t0; pl0 < npx; pl0 += kMedBatch * nt) {
    int rb[kMedBatch][3], cb[kMedBatch][3];   // clamped neighbour rows (times W) and columns
#pragma unroll
    for (int b = 0; b < kMedBatch; ++b) {
      const int pix = p0 + min(pl0 + b * nt, npx - 1);
      const int row = pix / W, col = pix - row * W;
      rb[b][0] = max(row - 1, 0) * W;
      rb[b][1] = row * W;
      rb[b][2] = min(row + 1, H - 1) * W;
      cb[b][0] = max(col - 1, 0);
      cb[b][1] = col;
      cb[b][2] = min(col + 1, W - 1);
    }
    uint8_t v[kMedBatch][9];
#pragma unroll
    for (int b = 0; b < kMedBatch; ++b)
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const uint8_t* p = lab + rb[b][i] + cb[b][j];
          v[b][3 * i + j] = COH ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
        }
#pragma unroll
    for (int b = 0; b < kMedBatch; ++b) {
      int cnt = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) cnt += v[b][t];
      const int pl = pl0 + b * nt;
      if (pl < npx) mask[p0 + pl] = (cnt >= 5) ? 1 : 0;
    }
  }
}

// ---------------------------------------------------------------------------
// Pieces shared by the two register layouts of a tile
// ---------------------------------------------------------------------------

// Per-tile constants.
struct TileCtx {
  int p0, npx, nq;        // first pixel, pixels, register rows (npx * C)
  unsigned base, ebase;   // exchange counter / epoch bases of this launch
  long long n;            // frame index
  bool lead;              // tile 0 writes the stream's statistics and y
  int rejected;           // rejected frames since the epochs last went back
  int median;             // the previous frame's median of this tile is still to be formed:
                          // 1 from labels of an earlier launch, 2 of this launch
};

// Reads y and the frame index.  The median of the previous frame's labels is
// left for a wait later in the frame (between_frames) unless this frame's weights
// come from it.  A mask that has been read already is the median of these
// labels, and nothing is left to do.
template <int K>
__device__ __forceinline__ TileCtx tile_begin(const FrameArgs& a, const int tile, KSpace<kMaxK>& ks) {
  TileCtx t;
  const int tid = thread_index();
  t.p0 = tile * a.tpw;
  t.npx = min(a.tpw, a.P - t.p0);
  t.nq = t.npx * a.C;
  t.base = __hip_atomic_load(&a.sync[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  t.ebase = __hip_atomic_load(&a.sync[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  t.rejected = __builtin_amdgcn_readfirstlane(
      (int)__hip_atomic_load(&a.sync[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  t.n = *a.nframe;
  t.lead = (tile == 0);
  if (tid < K) {
    const double yv = (tid < a.k) ? a.y[tid] : 0.0;
    ks.y[tid] = yv;
    ks.yf[tid] = (float)yv;
  }
  if (tid < 4) ks.flag[tid] = 0;
  if (tid == 0) {
    float inv_s = 1.f, inv_n = 1.f;
    int upd = 0;
    if (a.pre_mean) {
      const double cnt = a.pre_stat[1];
      const double var = cnt >= 2.0 ? a.pre_stat[0] / ((double)a.m * (cnt - 1.0)) : 0.0;
      inv_s = var > 0.0 ? (float)(1.0 / sqrt(var)) : 1.f;
      upd = (t.n < (long long)a.i_init) ? 1 : 0;
      inv_n = (float)(1.0 / (cnt + 1.0));
    }
    ks.pre_inv_s = inv_s;
    ks.pre_inv_n = inv_n;
    ks.pre_upd = upd;
    ks.pre_sum = 0.0;
  }
  __syncthreads();
  trace_point(a, tile, 0);
  t.median = __hip_atomic_load(&a.sync[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 0 : 1;
  if (a.weights_from_filtered && t.median) {
    median3x3_range(a.lab, a.mask, a.W, a.H, t.p0, t.npx, tid, kBlock);
    t.median = 0;
  }
  __syncthreads();
  trace_point(a, tile, 1);
  return t;
}

// Colour plane of tile entry q = c * npx + pixel (at most 4 planes): compares
// instead of an integer division per row and pass.
__device__ __forceinline__ int plane_of(int q, int npx) {
  return (q >= npx ? 1 : 0) + (q >= 2 * npx ? 1 : 0) + (q >= 3 * npx ? 1 : 0);
}
__device__ __forceinline__ float ld_f32(const float* base, unsigned boff) {
  return *(const float*)((const char*)base + boff);
}

// Pre-processing of one frame entry (Sec. 3.4): with upd the entry joins the
// running average (Welford update of mean and deviation sum; the new
// deviation sum is added to m2_sum), then the frame value minus the average
// is scaled by inv_s.  Returns the pre-processed value.
__device__ __forceinline__ float pre_entry(const FrameArgs& a, long long e, float x, bool upd, float inv_n,
                                           float inv_s, float& m2_sum) {
  float mean = a.pre_mean[e];
  if (upd) {
    const float d = x - mean;
    mean = fmaf(d, inv_n, mean);
    m2_sum += fmaf(d, x - mean, a.pre_m2[e]);
  }
  return (x - mean) * inv_s;
}

// Store the running average and deviation sum of one entry after an
// accepted initialization frame (same arithmetic as pre_entry).
__device__ __forceinline__ void pre_store(const FrameArgs& a, long long e, float x, float inv_n) {
  const float mean = a.pre_mean[e];
  const float d = x - mean;
  const float mn = fmaf(d, inv_n, mean);
  a.pre_m2[e] = fmaf(d, x - mn, a.pre_m2[e]);
  a.pre_mean[e] = mn;
}

// Step size t = max(exp(-tau n) t_init, t_min) of frame n (Sec. 3.4).  Out of
// line like geodesic_scalars.  It needs nothing but the frame index: a thread of
// the second wavefront forms it while the first takes the frame's first
// direction (0.4 us in the one lane that forms the angle otherwise).
__device__ __attribute__((noinline)) double step_size(double tau_n, double t_init, double t_min) {
  return fmax(exp(-tau_n) * t_init, t_min);
}

// PR+ conjugate direction from the reduced gradient and cost in ks.red
// (Sec. 3.3, Step 1): wave 0, lane j owns component j.  Sets ks.d / df / gp,
// ks.gd and the stop flag ks.flag[0]; a non-finite first cost marks the frame
// bad (ks.flag[1]).
template <int K>
__device__ __forceinline__ void cg_direction(const FrameArgs& a, KSpace<kMaxK>& ks, long long n, int it, bool lead,
                                             int& restarts) {
  const int tid = thread_index(), lane = tid & 63;
  if (tid == 64 && it == 0) ks.t = step_size(a.tau * (double)n, a.t_init, a.t_min);
  if (tid < 64) {
    const double g = (lane < K) ? -ks.red[lane] : 0.0;
    const double f = ks.red[K];
    const double gg = row16_sum(g * g);
    int stop = 0;
    if (it == 0 && !(isfinite(f) && isfinite(gg))) {
      stop = 1;
      if (lane == 0) ks.flag[1] = 1;
    }
    if (gg == 0.0) stop = 1;
    if (lead && lane == 0) a.stats->f[it] = f;
    // g . d of a direction -g is -(g . g), term by term, and the gp . gp of
    // the PR+ coefficient is the previous step's g . g
    double beta = 0.0, dj = -g, gd = -gg;
    if (!stop && it > 0 && a.ysolve == 0) {
      const double gp = (lane < K) ? ks.gp[lane] : 0.0;
      const double num = row16_sum(g * (g - gp));
      beta = fmax(0.0, num / ks.gg);
      const double dpv = (lane < K) ? ks.dp[lane] : 0.0;
      const double dv = -g + beta * dpv;
      const double gdv = row16_sum(g * dv);
      if (gdv >= 0.0) {
        if (lane == 0) ++restarts;
      } else {
        dj = dv;
        gd = gdv;
      }
    }
    if (lane < K) {
      ks.d[lane] = dj;
      ks.df[lane] = (float)dj;
      ks.gp[lane] = g;
    }
    if (lane == 0) {
      ks.gd = gd;
      ks.gg = gg;
      ks.flag[0] = stop;
      if (lead) a.stats->beta[it] = beta;
    }
  }
  __syncthreads();
}

// ---- steps with H reduced alongside the gradient (one wide exchange per step) ----

// Upper-triangle pair p -> (row, column) of a K x K matrix, row-major.
__host__ __device__ constexpr int tri_row(int p, int K) {
  int i = 0;
  while (p >= K - i) { p -= K - i; ++i; }
  return i;
}
__host__ __device__ constexpr int tri_col(int p, int K) {
  int i = 0;
  while (p >= K - i) { p -= K - i; ++i; }
  return i + p;
}

template <int K, int P>
struct TriPair {   // compile-time (row, column) of upper-triangle pair P
  static constexpr int i = tri_row(P, K);
  static constexpr int j = tri_col(P, K);
};

// One register row's contribution to chunk C (pairs C*32 .. C*32+31) of H.
template <int K, int C, typename UF, int... Q>
__device__ __forceinline__ void irls_h_row(float (&h)[kSlot], float wci, int row, UF uval,
                                           std::integer_sequence<int, Q...>) {
  constexpr int NP = K * (K + 1) / 2;
  ((C * kSlot + Q < NP
        ? (void)(h[Q] = fmaf(wci * uval(row, TriPair<K, (C * kSlot + Q < NP ? C * kSlot + Q : 0)>::i),
                             uval(row, TriPair<K, (C * kSlot + Q < NP ? C * kSlot + Q : 0)>::j), h[Q]))
        : (void)0),
   ...);
}

template <int K, int ROWS, int C, typename UF, typename PF>
__device__ __forceinline__ void irls_h_chunk(const float (&wc)[ROWS], UF uval, PF pin, FrameSmem& sm) {
  float h[kSlot];
#pragma unroll
  for (int q = 0; q < kSlot; ++q) h[q] = 0.f;
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    pin();
    irls_h_row<K, C>(h, wc[i], i, uval, std::make_integer_sequence<int, kSlot>{});
  }
  wg_reduce<kSlot>(h, sm.red, sm.wide_in + K + 1 + C * kSlot);
}

template <int K, int ROWS, typename UF, typename PF, int... C>
__device__ __forceinline__ void irls_h_chunks(const float (&wc)[ROWS], UF uval, PF pin, FrameSmem& sm,
                                              std::integer_sequence<int, C...>) {
  (irls_h_chunk<K, ROWS, C>(wc, uval, pin, sm), ...);
}

// This workgroup's partial sums of H = U^T diag(w c) U (upper triangle),
// 32 entries at a time, into sm.wide_in[K + 1 ...].  uval(i, j): entry j of
// the thread's register row i (j a compile-time constant); wc[i] = w c(r)
// of that row; pin() is called before each row (keeps widened copies of a
// packed tile from being held across rows).
template <int K, int ROWS, typename UF, typename PF>
__device__ __forceinline__ void irls_h_partials(const float (&wc)[ROWS], UF uval, PF pin, FrameSmem& sm) {
  constexpr int NP = K * (K + 1) / 2;
  irls_h_chunks<K, ROWS>(wc, uval, pin, sm, std::make_integer_sequence<int, (NP + kSlot - 1) / kSlot>{});
}

// Solve H d = -g from the gang totals (g, f, H in sm.wide_out) by Gaussian
// elimination without pivoting (H is symmetric positive definite for a
// non-degenerate frame) on the augmented matrix in LDS, all threads, fixed
// order.  Sets ks.d / df, ks.gd, the stop flag (zero gradient or H not
// positive definite) and, in the first step, the bad-frame flag.
template <int K>
__device__ __forceinline__ void irls_direction(const FrameArgs& a, FrameSmem& sm, long long n, int it, bool lead) {
  KSpace<kMaxK>& ks = sm.ks;
  const double* tot = sm.wide_out;
  const int tid = thread_index(), lane = tid & 63;
  for (int q = tid; q < K * (K + 1); q += kBlock) {
    const int i = q / (K + 1), j = q - i * (K + 1);
    double v;
    if (j == K) {
      v = tot[i];                     // -g = U^T (w phi'(r))
    } else {
      const int lo = min(i, j), hi = max(i, j);
      v = tot[K + 1 + lo * K - lo * (lo - 1) / 2 + (hi - lo)];
    }
    sm.hs[i][j] = v;
  }
  if (tid == 0) ks.flag[3] = 0;
  if (tid == 64 && it == 0) ks.t = step_size(a.tau * (double)n, a.t_init, a.t_min);
  __syncthreads();
  if (tid < 64) {
    const double g = (lane < K) ? -tot[lane] : 0.0;
    const double gg = row16_sum(g * g);
    const double f = tot[K];
    int stop = (gg == 0.0) ? 1 : 0;
    if (it == 0 && !(isfinite(f) && isfinite(gg))) {
      stop = 1;
      if (lane == 0) ks.flag[1] = 1;
    }
    if (lead && lane == 0) {
      a.stats->f[it] = f;
      a.stats->beta[it] = 0.0;
    }
    if (lane == 0) ks.flag[3] = stop;
  }
  __syncthreads();
  for (int k = 0; k < K; ++k) {          // elimination, rows below k
    const double piv = sm.hs[k][k];
    if (!(piv > 0.0) || !isfinite(piv)) {
      if (tid == 0) ks.flag[3] = 1;      // not positive definite: no step
      break;                             // uniform: every thread reads the same pivot
    }
    const double inv = 1.0 / piv;
    const int w = K - k - 1;
    for (int q = tid; q < w * (w + 1); q += kBlock) {
      const int i = k + 1 + q / (w + 1), j = k + 1 + q % (w + 1);
      sm.hs[i][j] -= sm.hs[i][k] * inv * sm.hs[k][j];
    }
    __syncthreads();
  }
  __syncthreads();
  const bool ok = ks.flag[3] == 0;
  if (ok)
    for (int k = K - 1; k >= 0; --k) {   // back substitution, d_k in place of the right-hand side
      if (tid == 0) sm.hs[k][K] = sm.hs[k][K] / sm.hs[k][k];
      __syncthreads();
      const double dk = sm.hs[k][K];
      for (int i = tid; i < k; i += kBlock) sm.hs[i][K] -= sm.hs[i][k] * dk;
      __syncthreads();
    }
  if (tid < 64) {
    const double g = (lane < K) ? -tot[lane] : 0.0;
    const double dj = (ok && lane < K) ? sm.hs[lane][K] : 0.0;
    const double gd = row16_sum(g * dj);
    if (lane < K) {
      ks.d[lane] = dj;
      ks.df[lane] = (float)dj;
    }
    if (lane == 0) {
      ks.gd = gd;
      ks.flag[0] = ok ? 0 : 1;
    }
  }
  __syncthreads();
}

// y += d (unit step of the IRLS iteration).
template <int K>
__device__ __forceinline__ void irls_advance(const FrameArgs& a, KSpace<kMaxK>& ks, int it, bool lead) {
  const int tid = thread_index();
  if (tid < K) {
    ks.y[tid] += ks.d[tid];
    ks.dp[tid] = ks.d[tid];
  }
  if (lead && tid == 0) a.stats->alpha[it] = 1.0;
}

// CG step of the one-exchange curvature schedule: g and f come from the wide
// totals in sm.wide_out (with the upper triangle of H = U^T diag(w c) U);
// the direction is the one cg_direction forms, and d^T H d is summed from
// the reduced H in a fixed order (lane i: row i of H times d, then the
// 16-lane sum), into ks.red[K + 1].  Same value, up to rounding, as the
// second pass sum_e w c (u_e . d)^2.
template <int K>
__device__ __forceinline__ void wide_cg_direction(const FrameArgs& a, FrameSmem& sm, long long n, int it, bool lead,
                                                  int& restarts) {
  KSpace<kMaxK>& ks = sm.ks;
  const double* tot = sm.wide_out;
  const int tid = thread_index(), lane = tid & 63;
  if (tid <= K) ks.red[tid] = tot[tid];
  __syncthreads();
  cg_direction<K>(a, ks, n, it, lead, restarts);
  if (tid < 64) {
    double t = 0.0;
    if (lane < K) {
      for (int j = 0; j < K; ++j) {
        const int lo = min(lane, j), hi = max(lane, j);
        t = fma(tot[K + 1 + lo * K - lo * (lo - 1) / 2 + (hi - lo)], ks.d[j], t);
      }
      t *= ks.d[lane];
    }
    const double dhd = row16_sum(t);
    if (lane == 0) ks.red[K + 1] = dhd;
  }
  __syncthreads();
}

// Majoriser step along d: alpha = -g.d / d^T H d, y += alpha d.  Returns
// alpha as float for the residual update.
template <int K>
__device__ __forceinline__ float cg_advance(const FrameArgs& a, KSpace<kMaxK>& ks, double dHd, int it, bool lead) {
  const int tid = thread_index();
  const double alpha = -ks.gd / dHd;
  // y, d and dp are the first wavefront's own until the next barrier
  if (tid < K) {
    ks.y[tid] += alpha * ks.d[tid];
    ks.dp[tid] = ks.d[tid];
  }
  if (lead && tid == 0) a.stats->alpha[it] = alpha;
  return (float)alpha;
}

// Angle of the geodesic step and the trigonometric scalars of the row pass:
// theta = sigma t, cos(theta) - 1 = -2 sin^2(theta / 2),
// sin(theta) / zeta = 2 sin(theta / 2) cos(theta / 2) / zeta.
// Out of line on purpose: inlined into the persistent kernels, the float64
// polynomial constants of exp and sin were hoisted out of the tile loop and
// held in registers (and spilled) for the whole launch.
struct GeoScalars {
  double theta, cm1, sz;
};
__device__ __attribute__((noinline)) GeoScalars geodesic_scalars(double t, double sigma, double zeta) {
  GeoScalars g;
  g.theta = sigma * t;
  double sh, ch;   // sin and cos of theta / 2 from one range reduction; sin(theta) = 2 sh ch
  sincos(0.5 * g.theta, &sh, &ch);
  g.cm1 = -2.0 * sh * sh;
  g.sz = zeta > 0.0 ? 2.0 * sh * ch / zeta : 0.0;
  return g;
}

// Scalars of the rank-one geodesic step (Sec. 3.3, Step 2) from the reduced
// a = U^T eta, ||eta||^2 and the final cost in ks.red: zeta = ||pi(eta)||,
// nu = ||y||, sigma = zeta nu, theta = sigma t_n; row-pass coefficients in
// ks.scal / vf / af.
template <int K>
__device__ __forceinline__ void geodesic_setup(const FrameArgs& a, KSpace<kMaxK>& ks, int steps, bool lead) {
  const int tid = thread_index(), lane = tid & 63;
  if (tid < 64) {
    const double av = (lane < K) ? ks.red[lane] : 0.0;
    const double yv = (lane < K) ? ks.y[lane] : 0.0;
    const double aa = row16_sum(av * av);
    const double yy = row16_sum(yv * yv);
    const double ee = ks.red[K];
    const double zeta = sqrt(fmax(ee - aa, 0.0));
    const double nu = sqrt(yy);
    const double sigma = zeta * nu;
    const int upd = (zeta > 0.0 && nu > 0.0) ? 1 : 0;
    if (lane < K) {
      ks.af[lane] = (float)av;
      ks.vf[lane] = upd ? (float)(yv / nu) : 0.f;
      ks.yf[lane] = (float)yv;
    }
    if (lane == 0) {
      const GeoScalars g = geodesic_scalars(ks.t, sigma, zeta);
      ks.scal[0] = upd ? (float)g.cm1 : 0.f;   // cos(theta) - 1
      ks.scal[1] = upd ? (float)g.sz : 0.f;    // sin(theta) / zeta
      ks.scal[2] = (float)nu;
      ks.flag[2] = upd;
      if (lead) {
        a.stats->t = ks.t;
        a.stats->sigma = sigma;
        a.stats->theta = g.theta;
        a.stats->zeta = zeta;
        a.stats->nu = nu;
        a.stats->updated = upd;
      }
    }
  }
  __syncthreads();
}

// Start of frame i > 0 of a sequence launch: y and the frame index carry
// over in the workgroup (identical in every workgroup of the gang).  The
// finished frame's labels went out with device-coherent stores; every thread
// waits for its stores to complete before any partial of the next frame is
// published, so that the mask of the finished frame (its 3x3 median reads
// neighbouring tiles' labels) can be formed after the next frame's first
// exchange (between_frames), which no workgroup completes before all have
// published.  (A device-scope release / acquire fence pair would also
// write back and invalidate the L2: measured 3x slower.)
__device__ __forceinline__ void next_frame_begin(KSpace<kMaxK>& ks, TileCtx& t, bool bad) {
  if (!bad) ++t.n;
  t.median = 2;
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this thread's stores have completed
  __syncthreads();   // everyone is past the previous frame's use of ks.flag and s_flag
  if (thread_index() < 4) ks.flag[thread_index()] = 0;
  __syncthreads();
}

// The deferred median of the previous frame's labels, by thread t0 of nt.  The
// labels of the whole gang are complete once this frame's first exchange is,
// and no workgroup writes this frame's labels before the last exchange, so the
// wavefronts that do not wait for the gang form it during its first
// single-value exchange, where it costs no time of its own (1.8 us of a
// 640x480x3 float32 frame, 2.5 in bfloat16).
template <bool SEQ>
__device__ __forceinline__ void between_frames(const FrameArgs& a, const TileCtx& t, int t0, int nt) {
  if (SEQ && t.median == 2)
    median3x3_range<true>(a.lab, a.mask, a.W, a.H, t.p0, t.npx, t0, nt);
  else if (t.median)
    median3x3_range(a.lab, a.mask, a.W, a.H, t.p0, t.npx, t0, nt);
}

// Label of tile pixel pl from the per-entry flags of the last labelled frame.
__device__ __forceinline__ bool pixel_label(const uint8_t* s_flag, int C, int npx, int pl) {
  uint8_t f = 0;
  for (int c = 0; c < C; ++c) f |= s_flag[c * npx + pl];
  return f != 0;
}

// Pixel labels (Sec. 3.3, Step 3): foreground when any colour entry was
// flagged in s_flag (entry q = c * npx + pixel).  COH: device-coherent
// stores (read by other workgroups in the same launch).
template <bool COH = false>
__device__ __forceinline__ void write_labels(const FrameArgs& a, const uint8_t* s_flag, int p0, int npx) {
  // four pixels per thread at a time, their flags read together: the LDS
  // latency is paid once per four pixels
  constexpr int kLabBatch = 4;
  __syncthreads();
  for (int pl0 = thread_index(); pl0 < npx; pl0 += kLabBatch * kBlock) {
    uint8_t f[kLabBatch] = {0, 0, 0, 0};
    for (int c = 0; c < a.C; ++c) {
#pragma unroll
      for (int b = 0; b < kLabBatch; ++b) f[b] |= s_flag[c * npx + min(pl0 + b * kBlock, npx - 1)];
    }
#pragma unroll
    for (int b = 0; b < kLabBatch; ++b) {
      const int pl = pl0 + b * kBlock;
      if (pl >= npx) break;
      if (COH)
        __hip_atomic_store(&a.lab[p0 + pl], f[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        a.lab[p0 + pl] = f[b];
    }
  }
}

// The exchange count at the end of a frame.  A rejected frame takes one exchange,
// and the values that only a whole frame exchanges keep the tags of the last one.
// Tags repeat after 256 exchanges, so a run of rejected frames goes round in four
// epochs: the slots of its exchanges then never hold the tag that comes next (a
// set is written every second exchange), and the others' tags stay recent.  The
// same in every workgroup.
constexpr int kRejectedEpochs = 4;
__device__ __forceinline__ void frame_epochs(const FrameArgs& a, TileCtx& t, bool bad, int& nbar) {
  t.rejected = __builtin_amdgcn_readfirstlane(bad) ? t.rejected + 1 : 0;   // scalar, as the count is
  if (t.rejected == kRejectedEpochs && a.sync_mode != 0) {   // the counter has no tags, and only counts up
    nbar -= kRejectedEpochs;
    t.rejected = 0;
  }
}

// Statistics, frame counter, y and the exchange bases for the next launch.
__device__ __forceinline__ void tile_end(const FrameArgs& a, const int tile, KSpace<kMaxK>& ks, const TileCtx& t,
                                         int steps, int restarts, bool bad, int nbar) {
  const int tid = thread_index();
  trace_point(a, tile, 63);
  if (t.lead && tid == 0) {
    a.stats->frame = t.n;
    a.stats->cg_steps = steps;
    a.stats->restarts = restarts;
    a.stats->bad_frame = bad ? 1 : 0;
    // every tile read the flag before its first partial went out
    __hip_atomic_store(&a.sync[4], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (bad) {
      __hip_atomic_fetch_or(&a.sync[2], kErrBadFrame, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      *a.nframe = t.n + 1;
      if (ks.pre_upd) {
        a.pre_stat[0] = ks.pre_sum;
        a.pre_stat[1] = a.pre_stat[1] + 1.0;
      }
    }
    if (a.G == 1) {
      // a one-workgroup gang used no slots or counters: the bases stay
    } else if (a.sync_mode != 0) {
      __hip_atomic_store(&a.sync[3], t.ebase + (unsigned)nbar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.sync[5], (unsigned)t.rejected, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else
      __hip_atomic_store(&a.sync[1], t.base + (unsigned)a.G * (unsigned)nbar, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
  if (t.lead && !bad && tid < a.k) a.y[tid] = ks.y[tid];
  __syncthreads();   // shared scratch may be reused by the next tile
}

// One column of U as a buffer: a store at kNowhere lies past its end and is
// dropped, so a tile is stored without a branch and a lane mask per entry (the
// masks and the K base addresses did not fit the scalar registers: 1433 lane
// reads for them in the k = 15 bfloat16 update).  640x480x3, k = 15, update pass:
// 16 bfloat16 rows per thread 9.9 -> 5.7 us, 8 rows 6.5 -> 3.8, one frame's kernel
// 55.6 -> 51.5; float32 160x120x3 2.8 -> 1.9.
constexpr unsigned kNowhere = 0xFFFFFFF0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t column_rows(void* col, int m, int entry_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(col, 0, (unsigned)m * entry_bytes, 0x00027000);
}

// ---------------------------------------------------------------------------
// float32 storage: row q = tid + s * kBlock of the tile, K floats per row
// ---------------------------------------------------------------------------
template <int K, int NR, bool EXT, bool WIDE, bool SEQ>
__device__ __forceinline__ bool frame_tile(const FrameArgs& a, const int tile, FrameSmem& sm) {
  KSpace<kMaxK>& ks = sm.ks;
  uint8_t* s_flag = sm.flag;
  int tid = thread_index();
  if (tid == 0) sm.ctl[2] = 0;
  TileCtx ctx = tile_begin<K>(a, tile, ks);
  int nbar = 0;

  // ---- load the register tile: U rows, residual r = x - U y, weights ----
  const float* __restrict__ Ug = (const float*)a.U;
  const float* __restrict__ xg = (const float*)(a.xtab ? global_ptr(a.xtab[ctx.n % a.ring]) : a.x);
  const uint8_t* __restrict__ wsrc = a.weights_from_filtered ? a.mask : a.lab;
  float u[NR][K];
  float r[NR], wt[NR], cw[NR];
  int eix[NR];
  // Rows past the tile's end: a tile of 16 rows per thread is chosen for whatever
  // 8 do not hold, so its upper half is worked in pairs, up to the last one in use
  // (80x60x1: 10 rows of 16, a frame with its mask 36 -> 32 us); a scalar compare
  // and one exit per pair of rows.
  auto past = [&](int s) { return NR == 16 && s >= 8 && (s & ~1) * kBlock >= ctx.nq; };
  bool u_pending = false;   // sequence: the registers hold an update not yet stored
  auto store_tile = [&]() {  // sequence: the register tile to the U planes
#pragma unroll
    for (int j = 0; j < K; ++j) {   // a plane at a time: one base address held
      if (j >= a.k) continue;
      const __amdgpu_buffer_rsrc_t col = column_rows((float*)a.U + (long long)j * a.ldU, a.m, 4);
#pragma unroll
      for (int s = 0; s < NR; ++s) {
        if (past(s)) continue;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(u[s][j]), col,
                                              eix[s] >= 0 ? 4u * (unsigned)eix[s] : kNowhere, 0, 0);
      }
    }
  };
  const bool pre = EXT && a.pre_mean != nullptr;   // compiled out without EXT
  const bool pupd = EXT && ks.pre_upd != 0;
  const float pinv_n = ks.pre_inv_n, pinv_s = ks.pre_inv_s;
  float m2sum = 0.f;
  // Every load of the tile is asked for before any is used (a thread's rows one
  // after the other cost a memory latency each: to the first exchange 640x480x3,
  // k = 15 10.5 -> 7.8 us, 160x120x3 4.4 -> 3.0, 80x60x1, k = 5 4.4 -> 3.7).  A row
  // past the tile's end takes the first entry's values; its weight is 0 and it is
  // never written.  32-bit byte offsets from uniform plane bases: a resident
  // frame's planes are far below 4 GB.
  uint8_t fgl[NR];
  unsigned ub[NR];
#pragma unroll
  for (int s = 0; s < NR; ++s) {   // rows that the passes leave out
    eix[s] = -1;
    r[s] = wt[s] = cw[s] = 0.f;
    fgl[s] = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) u[s][j] = 0.f;
  }
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    if (past(s)) break;
    const int q = tid + s * kBlock;
    const bool in = q < ctx.nq;
    const int c = plane_of(q, ctx.npx);
    const int pl = in ? q - c * ctx.npx : 0;
    const int e = in ? c * a.P + ctx.p0 + pl : ctx.p0;
    eix[s] = in ? e : -1;
    fgl[s] = wsrc[ctx.p0 + pl];
    ub[s] = 4u * (unsigned)e;
    r[s] = ld_f32(xg, ub[s]);
  }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    if (j >= a.k) continue;   // columns >= k are 0
    const float* col = Ug + (long long)j * a.ldU;
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (past(s)) continue;
      u[s][j] = ld_f32(col, ub[s]);
    }
  }
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    if (past(s)) break;
    const bool in = eix[s] >= 0;
    wt[s] = in ? (fgl[s] ? a.omega : 1.0f) : 0.f;
    float acc = r[s];
    if (pre && in) acc = pre_entry(a, eix[s], acc, pupd, pinv_n, pinv_s, m2sum);
#pragma unroll
    for (int j = 0; j < K; ++j) acc = fmaf(-u[s][j], ks.yf[j], acc);
    r[s] = in ? acc : 0.f;
  }

  for (int fi = 0;;) {   // frames of this launch; U stays in the registers between them
  if constexpr (SEQ) {
    // Per-row indices re-enter opaquely each frame: otherwise every address
    // derived from them is hoisted out of the frame loop and held in registers.
    tid = thread_index();
#pragma unroll
    for (int s = 0; s < NR; ++s) asm volatile("" : "+v"(eix[s]));
  }
  // ---- Step 1: CG on y ----
  int steps = 0, restarts = 0;
  bool between = true;   // the previous frame's median is still to be formed
  for (int it = 0; it < a.J; ++it) {
    // phase A: gradient and cost at the current y
    float acc[K + 1];   // g, f
#pragma unroll
    for (int j = 0; j <= K; ++j) acc[j] = 0.f;
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (past(s)) break;
      float phi, c;
      cost_eval(r[s], a.cp, phi, c);
      const float wc = wt[s] * c;
      cw[s] = wc;
      const float wd = wc * r[s];          // w phi'(r)
      acc[K] = fmaf(wt[s], phi, acc[K]);
#pragma unroll
      for (int j = 0; j < K; ++j) acc[j] = fmaf(wd, u[s][j], acc[j]);
    }
    if (WIDE && (a.ysolve == 2 || a.curv == 1)) {   // g, f and H in one (wide) exchange
      wg_reduce<K + 1>(acc, sm.red, sm.wide_in);
      irls_h_partials<K, NR>(cw, [&](int i, int j) { return u[i][j]; }, [] {}, sm);
      if (!gang_reduce_wide(sm.wide_in, K + 1 + K * (K + 1) / 2, a, tile, nbar, ctx.ebase, sm.big, sm.wide_out))
        return false;
      float af = 1.0f;
      if (a.ysolve == 2) {   // IRLS: unit step along -H^{-1} g
        irls_direction<K>(a, sm, ctx.n, it, ctx.lead);
        if (ks.flag[0]) break;
        irls_advance<K>(a, ks, it, ctx.lead);
      } else {               // CG / gradient descent with d^T H d from the reduced H
        wide_cg_direction<K>(a, sm, ctx.n, it, ctx.lead, restarts);
        if (ks.flag[0]) break;
        const double dHd = ks.red[K + 1];
        if (!(dHd > 0.0)) break;
        af = cg_advance<K>(a, ks, dHd, it, ctx.lead);
      }
#pragma unroll
      for (int s = 0; s < NR; ++s) {
        if (past(s)) break;
        float t = 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j) t = fmaf(u[s][j], ks.df[j], t);
        r[s] = fmaf(-af, t, r[s]);
      }
      ++steps;
      __syncthreads();
      continue;
    }
    if (!gang_reduce<K + 1>(acc, a, tile, nbar, ctx.base, ctx.ebase, sm, ks.red)) return false;
    cg_direction<K>(a, ks, ctx.n, it, ctx.lead, restarts);
    if (sm.ctl[2]) return false;
    if (ks.flag[0]) break;
    // phase B: curvature of the majoriser along d; cw then holds u.d
    float accb[1] = {0.f};
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (past(s)) break;
      float t = 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j) t = fmaf(u[s][j], ks.df[j], t);
      accb[0] = fmaf(cw[s] * t, t, accb[0]);
      cw[s] = t;
    }
    double dHd;
    if (!gang_reduce1(accb[0], a, tile, nbar, ctx.base, ctx.ebase, sm, dHd, [&] {
          if (between) between_frames<SEQ>(a, ctx, thread_index() - 64, kBlock - 64);
        }))
      return false;
    if (wave0_exchange(a) && a.G > 1) between = false;
    if (!(dHd > 0.0)) break;   // same decision in every workgroup
    const float af = cg_advance<K>(a, ks, dHd, it, ctx.lead);
#pragma unroll
    for (int s = 0; s < NR; ++s) r[s] = fmaf(-af, cw[s], r[s]);
    ++steps;
  }
  const bool bad = ks.flag[1] != 0;
  if (between) between_frames<SEQ>(a, ctx, thread_index(), kBlock);

  if (!bad) {
    // ---- Step 2: eta pass (a = U^T eta, ||eta||^2, final cost) ----
    constexpr int LE = K + 2 + (EXT ? 1 : 0);   // a, ||eta||^2, f (+ pre-processing deviation sum)
    float acce[LE];
#pragma unroll
    for (int j = 0; j < LE; ++j) acce[j] = 0.f;
    if constexpr (EXT) acce[LE - 1] = pupd ? m2sum : 0.f;
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (past(s)) break;
      float phi, c;
      cost_eval(r[s], a.cp, phi, c);
      const float eta = -wt[s] * c * r[s];
      cw[s] = eta;
      acce[K] = fmaf(eta, eta, acce[K]);
      acce[K + 1] = fmaf(wt[s], phi, acce[K + 1]);
#pragma unroll
      for (int j = 0; j < K; ++j) acce[j] = fmaf(eta, u[s][j], acce[j]);
    }
    // the final cost and the deviation sum serve the statistics alone
    constexpr int kLate = LE - (K + 1 > 16 ? K + 1 : LE < 16 ? LE : 16);
    if (!gang_reduce<LE, kLate>(acce, a, tile, nbar, ctx.base, ctx.ebase, sm, ks.red)) return false;
    geodesic_setup<K>(a, ks, steps, ctx.lead);
    if (sm.ctl[2]) return false;
    if (ctx.lead && tid == 0) {
      a.stats->f[steps] = ks.red[K + 1];
      if (EXT && pupd) ks.pre_sum = ks.red[K + 2];
    }
    trace_point(a, tile, 60);

    // ---- Step 2 update + Step 3 labels, one pass over the register tile ----
    const float cm1 = ks.scal[0], sz = ks.scal[1], nu_f = ks.scal[2];
    const bool upd = ks.flag[2] != 0;
    // a sequence keeps U in the registers (the next frame starts from them)
    // and stores it after its last frame only, in a loop of its own, so the
    // update of the other frames carries no per-entry store decisions
    const bool store_u = !SEQ || fi + 1 >= a.nseq;
    if (SEQ && upd) u_pending = !store_u;
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (past(s)) break;
      const int q = tid + s * kBlock;
      if (eix[s] >= 0) {
        float rl = r[s];
        if (upd) {
          float uv = 0.f, ua = 0.f;
#pragma unroll
          for (int j = 0; j < K; ++j) {
            uv = fmaf(u[s][j], ks.vf[j], uv);
            ua = fmaf(u[s][j], ks.af[j], ua);
          }
          const float coef = fmaf(cm1, uv, -sz * (cw[s] - ua));
#pragma unroll
          for (int j = 0; j < K; ++j) u[s][j] = fmaf(coef, ks.vf[j], u[s][j]);   // columns >= k stay 0 (v_j = 0)
          if (a.labels_after_update) rl = fmaf(-coef, nu_f, rl);
        }
        if (pre && pupd) pre_store(a, eix[s], xg[eix[s]], pinv_n);
        if (EXT && a.score) a.score[eix[s]] = fabsf(rl);
        s_flag[q] = (fabsf(rl) >= a.delta) ? 1 : 0;
      }
    }
    if (upd && store_u) store_tile();
    trace_point(a, tile, 61);
    write_labels<SEQ>(a, s_flag, ctx.p0, ctx.npx);
    trace_point(a, tile, 62);
  }
  frame_epochs(a, ctx, bad, nbar);
  tile_end(a, tile, ks, ctx, steps, restarts, bad, nbar);
  if (!SEQ || ++fi >= a.nseq) break;

  // ---- next frame of a sequence: weights from this frame's labels (still in
  // s_flag; unchanged after a rejected frame), residuals of the next frame ----
  next_frame_begin(ks, ctx, bad);
  xg = (const float*)(global_ptr(a.xtab ? a.xtab[ctx.n % a.ring] : a.seq[fi]));
#pragma unroll
  for (int s = 0; s < NR; ++s) r[s] = ld_f32(xg, 4u * (unsigned)(eix[s] >= 0 ? eix[s] : ctx.p0));
  if (!bad) {
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (past(s)) break;
      const int q = tid + s * kBlock;
      const int pl = eix[s] >= 0 ? q - plane_of(q, ctx.npx) * ctx.npx : 0;
      const float wn = pixel_label(s_flag, a.C, ctx.npx, pl) ? a.omega : 1.0f;
      wt[s] = eix[s] >= 0 ? wn : 0.f;
    }
  }
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    if (past(s)) break;
    float acc = r[s];
#pragma unroll
    for (int j = 0; j < K; ++j) acc = fmaf(-u[s][j], ks.yf[j], acc);
    r[s] = eix[s] >= 0 ? acc : 0.f;
  }
  }
  // the last frame stored nothing (rejected, or no step): store the updated tile
  if (SEQ && u_pending) store_tile();
  return true;
}

// ---------------------------------------------------------------------------
// bfloat16 storage: the register tile keeps U in bfloat16, two rows per
// 32-bit register (row 2i in the low half, row 2i + 1 in the high half), so a
// tile holds twice the rows of the float32 layout in the same registers.
// Values are widened to float32 (exact) where they are used; the update is
// computed in float32 and rounded to nearest-even once, as it is stored.
// Row pair s of thread tid covers rows q0 = 2 (tid + s kBlock) and q0 + 1.
// When a.pair_aligned is set (even P, even tpw, 4-byte aligned frame) a pair
// is one aligned 32-bit word in the U planes and in the frame; otherwise the
// two halves are accessed separately and may lie in two colour planes.
// NL > 0 (batched form): pairs NP .. NP + NL - 1 of every thread are held in
// LDS instead (lt[((s - NP) K + j) kBlock + tid], their residuals after the
// NL K kBlock words, each thread its own words: no barriers), processed by a
// loop that is not unrolled; results are identical.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ float bf_half(uint32_t w, int h) { return h ? bf_hi(w) : bf_lo(w); }

// Two float32 values rounded to nearest-even bfloat16 and packed (lo, hi):
// one v_cvt_pk_bf16_f32 on gfx950.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Marks the packed tile as redefined at the start of every row pass, so the
// compiler cannot hoist widened float32 copies of U out of the CG loop
// (which would double the registers the tile needs).  No instructions.
template <int NP, int K>
__device__ __forceinline__ void pin_tile(uint32_t (&u)[NP][K]) {
#pragma unroll
  for (int s = 0; s < NP; ++s)
#pragma unroll
    for (int j = 0; j < K; ++j) asm volatile("" : "+v"(u[s][j]));
}

// 32- and 16-bit accesses at a byte offset (32-bit) from a base pointer.
__device__ __forceinline__ uint32_t ld_u32(const uint16_t* base, unsigned boff) {
  return *(const uint32_t*)((const char*)base + boff);
}
__device__ __forceinline__ uint32_t ld_u16(const uint16_t* base, unsigned boff) {
  return *(const uint16_t*)((const char*)base + boff);
}
__device__ __forceinline__ void st_u32(uint16_t* base, unsigned boff, uint32_t v) {
  *(uint32_t*)((char*)base + boff) = v;
}
__device__ __forceinline__ void st_u16(uint16_t* base, unsigned boff, uint16_t v) {
  *(uint16_t*)((char*)base + boff) = v;
}

template <int K, int NP, bool EXT, int NL = 0, bool SEQ = false>
__device__ __forceinline__ bool frame_tile_packed(const FrameArgs& a, const int tile, FrameSmem& sm,
                                                  uint32_t* __restrict__ lt = nullptr) {
  constexpr int NT = NP + NL;   // row pairs per thread: NP in registers, NL in LDS
  static_assert(2 * NT <= kMaxNR && NT <= 16, "row bit masks hold 32 rows");
  static_assert(NL == 0 || !EXT, "the LDS pairs serve the default features only");
  KSpace<kMaxK>& ks = sm.ks;
  uint8_t* s_flag = sm.flag;
  int tid = thread_index();
  if (tid == 0) sm.ctl[2] = 0;
  TileCtx ctx = tile_begin<K>(a, tile, ks);
  int nbar = 0;
  const bool al = a.pair_aligned != 0;

  // ---- load the register tile ----
  const uint16_t* __restrict__ Ug = (const uint16_t*)a.U;
  const uint16_t* __restrict__ xg = (const uint16_t*)(a.xtab ? global_ptr(a.xtab[ctx.n % a.ring]) : a.x);
  const uint8_t* __restrict__ wsrc = a.weights_from_filtered ? a.mask : a.lab;
  uint32_t u[NP][K];
  // cw: w c in phase A, u.d in phase B, eta in the update (register rows);
  // the LDS rows keep r in LDS and recompute these where needed (the same
  // operations on the same values, so the same results)
  float r[2 * NP], cw[2 * NP];
  float* __restrict__ lr = NL > 0 ? (float*)(lt + NL * K * kBlock) : nullptr;   // r of the LDS rows
  uint32_t vbits = 0;         // bit i: row i exists
  uint32_t fbits = 0;         // bit i: row i's pixel was foreground (weight omega)
  uint32_t sbits = 0;         // bit s: pair s continues in the next colour plane
  const bool pre = EXT && a.pre_mean != nullptr;   // compiled out without EXT
  const bool pupd = EXT && ks.pre_upd != 0;
  const float pinv_n = ks.pre_inv_n, pinv_s = ks.pre_inv_s;
  float m2sum = 0.f;
  // Loads first, as in the float32 tile (640x480x3, k = 15, 16 rows per thread:
  // 14.3 -> 7.0 us to the first exchange; 8 rows 8.0 -> 4.6).  A pair past the
  // tile's end takes the first entry's values.  The pairs held in LDS go before the
  // register pairs, while the registers are free.
  // byte offsets in 32 bits from uniform plane bases: the addresses are a
  // scalar base plus one vector offset, not 64-bit vector arithmetic
  auto offsets = [&](int s, unsigned& b0, unsigned& b1) -> int {   // returns the pair's pixel in the tile
    const int q0 = 2 * (tid + s * kBlock);
    const bool in = q0 < ctx.nq, has1 = q0 + 1 < ctx.nq;
    const int c = plane_of(q0, ctx.npx);
    const int pl = in ? q0 - c * ctx.npx : 0;
    const int e = in ? c * a.P + ctx.p0 + pl : ctx.p0;
    const bool split = in && pl + 1 == ctx.npx;
    b0 = 2u * (unsigned)e;
    b1 = 2u * (unsigned)(!has1 ? e : split ? e + 1 + (a.P - ctx.npx) : e + 1);
    if (in) vbits |= (has1 ? 3u : 1u) << (2 * s);
    if (split) sbits |= 1u << s;
    return pl;
  };
  auto labels = [&](int s, int pl, uint8_t& f0, uint8_t& f1) {
    const bool one = (vbits >> (2 * s + 1)) & 1u;
    f0 = wsrc[ctx.p0 + pl];
    f1 = wsrc[ctx.p0 + (((sbits >> s) & 1u) || !one ? 0 : pl + 1)];
  };
  auto set_fbits = [&](int s, uint8_t f0, uint8_t f1) {
    fbits |= (((f0 ? 1u : 0u) | (f1 ? 2u : 0u)) << (2 * s)) & vbits;
  };
  // The loads of NN pairs from pair s0 on.  The two forms of a pair (one word, or
  // two halves to be put together) are told apart once for all of them: with the
  // choice inside, every load of halves was waited for before the next.
  auto load_pairs = [&](auto first, uint32_t* xw, uint32_t (*w)[K], uint8_t* f0, uint8_t* f1, auto count) {
    constexpr int s0 = decltype(first)::value, nn = decltype(count)::value;
    unsigned b0[nn], b1[nn];
#pragma unroll
    for (int i = 0; i < nn; ++i) {
      const int pl = offsets(s0 + i, b0[i], b1[i]);
      labels(s0 + i, pl, f0[i], f1[i]);
    }
    if (al) {
#pragma unroll
      for (int i = 0; i < nn; ++i) xw[i] = ld_u32(xg, b0[i]);
    } else {
#pragma unroll
      for (int i = 0; i < nn; ++i) xw[i] = ld_u16(xg, b0[i]) | (ld_u16(xg, b1[i]) << 16);
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const uint16_t* col = Ug + (long long)j * a.ldU;
      if (j >= a.k) {   // columns >= k are 0
#pragma unroll
        for (int i = 0; i < nn; ++i) w[i][j] = 0u;
      } else if (al) {
#pragma unroll
        for (int i = 0; i < nn; ++i) w[i][j] = ld_u32(col, b0[i]);
      } else {
#pragma unroll
        for (int i = 0; i < nn; ++i) w[i][j] = ld_u16(col, b0[i]) | (ld_u16(col, b1[i]) << 16);
      }
    }
  };
  if constexpr (NL > 0) {
    uint32_t v[NL][K], xw[NL];
    uint8_t f0[NL], f1[NL];
    load_pairs(std::integral_constant<int, NP>(), xw, v, f0, f1, std::integral_constant<int, NL>());
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int s = NP + i;
      set_fbits(s, f0[i], f1[i]);
      uint32_t* lts = lt + i * K * kBlock + tid;
      float* rls = lr + i * 2 * kBlock + tid;
      float acc0 = bf_lo(xw[i]), acc1 = bf_hi(xw[i]);
#pragma unroll
      for (int j = 0; j < K; ++j) {
        lts[j * kBlock] = v[i][j];
        acc0 = fmaf(-bf_lo(v[i][j]), ks.yf[j], acc0);
        acc1 = fmaf(-bf_hi(v[i][j]), ks.yf[j], acc1);
      }
      rls[0] = ((vbits >> (2 * s)) & 1u) ? acc0 : 0.f;
      rls[kBlock] = ((vbits >> (2 * s + 1)) & 1u) ? acc1 : 0.f;
    }
  }
  {
    uint32_t xw[NP];
    uint8_t f0[NP], f1[NP];
    load_pairs(std::integral_constant<int, 0>(), xw, u, f0, f1, std::integral_constant<int, NP>());
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      set_fbits(s, f0[s], f1[s]);
      const bool in = (vbits >> (2 * s)) & 1u, has1 = (vbits >> (2 * s + 1)) & 1u;
      float acc0 = bf_lo(xw[s]), acc1 = bf_hi(xw[s]);
      if (pre && in) {
        const int q0 = 2 * (tid + s * kBlock);
        const int c = plane_of(q0, ctx.npx);
        const int e = c * a.P + ctx.p0 + (q0 - c * ctx.npx);
        acc0 = pre_entry(a, e, acc0, pupd, pinv_n, pinv_s, m2sum);
        if (has1)
          acc1 = pre_entry(a, ((sbits >> s) & 1u) ? e + 1 + (a.P - ctx.npx) : e + 1, acc1, pupd, pinv_n, pinv_s, m2sum);
      }
#pragma unroll
      for (int j = 0; j < K; ++j) {
        acc0 = fmaf(-bf_lo(u[s][j]), ks.yf[j], acc0);
        acc1 = fmaf(-bf_hi(u[s][j]), ks.yf[j], acc1);
      }
      r[2 * s] = in ? acc0 : 0.f;
      r[2 * s + 1] = has1 ? acc1 : 0.f;
    }
  }
  const float om = a.omega;
  auto weight = [&](int i) -> float {
    return ((vbits >> i) & 1u) ? (((fbits >> i) & 1u) ? om : 1.0f) : 0.f;
  };
  static_assert(!(SEQ && NL > 0), "sequences keep register tiles only");
  bool u_pending = false;   // sequence: the registers hold an update not yet stored
  auto store_tile = [&]() {  // sequence: the register tile to the U planes
    unsigned b0[NP], b1[NP];
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const int q0 = 2 * (tid + s * kBlock);
      const int c = plane_of(q0, ctx.npx);
      const unsigned b = 2u * (unsigned)(c * a.P + ctx.p0 + (q0 - c * ctx.npx));
      const unsigned next = b + 2u + (((sbits >> s) & 1u) ? 2u * (unsigned)(a.P - ctx.npx) : 0u);
      b0[s] = ((vbits >> (2 * s)) & 1u) ? b : kNowhere;
      b1[s] = ((vbits >> (2 * s + 1)) & 1u) ? next : kNowhere;
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {   // a plane at a time: one base address held
      if (j >= a.k) continue;
      const __amdgpu_buffer_rsrc_t col = column_rows((uint16_t*)a.U + (long long)j * a.ldU, a.m, 2);
      if (al) {
#pragma unroll
        for (int s = 0; s < NP; ++s) __builtin_amdgcn_raw_buffer_store_b32(u[s][j], col, b0[s], 0, 0);
      } else {
#pragma unroll
        for (int s = 0; s < NP; ++s) {
          __builtin_amdgcn_raw_buffer_store_b16((uint16_t)u[s][j], col, b0[s], 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(u[s][j] >> 16), col, b1[s], 0, 0);
        }
      }
    }
  };

  for (int fi = 0;;) {   // frames of this launch; U stays in the registers between them
  if constexpr (SEQ) tid = thread_index();   // re-enters opaquely each frame (see the float32 tile)
  // ---- Step 1: CG on y ----
  int steps = 0, restarts = 0;
  bool between = true;   // the previous frame's median is still to be formed
  for (int it = 0; it < a.J; ++it) {
    float acc[K + 1];   // g, f
#pragma unroll
    for (int j = 0; j <= K; ++j) acc[j] = 0.f;
    pin_tile(u);
#pragma unroll
    for (int s = 0; s < NP; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = 2 * s + h;
        const float wt = weight(i);
        float phi, c;
        cost_eval(r[i], a.cp, phi, c);
        const float wc = wt * c;
        cw[i] = wc;
        const float wd = wc * r[i];
        acc[K] = fmaf(wt, phi, acc[K]);
#pragma unroll
        for (int j = 0; j < K; ++j) acc[j] = fmaf(wd, bf_half(u[s][j], h), acc[j]);
      }
#pragma unroll 1
    for (int s = NP; s < NT; ++s) {   // LDS pairs: each word read once for both rows
      const uint32_t* lts = lt + (s - NP) * K * kBlock + tid;
      float* rls = lr + (s - NP) * 2 * kBlock + tid;
      float wd[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float ri = rls[h * kBlock];
        const float wt = weight(2 * s + h);
        float phi, c;
        cost_eval(ri, a.cp, phi, c);
        wd[h] = wt * c * ri;
        acc[K] = fmaf(wt, phi, acc[K]);
      }
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const uint32_t v = lts[j * kBlock];
        acc[j] = fmaf(wd[0], bf_lo(v), acc[j]);
        acc[j] = fmaf(wd[1], bf_hi(v), acc[j]);
      }
    }
    if (!gang_reduce<K + 1>(acc, a, tile, nbar, ctx.base, ctx.ebase, sm, ks.red)) return false;
    cg_direction<K>(a, ks, ctx.n, it, ctx.lead, restarts);
    if (sm.ctl[2]) return false;
    if (ks.flag[0]) break;
    float accb[1] = {0.f};
    pin_tile(u);
#pragma unroll
    for (int s = 0; s < NP; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = 2 * s + h;
        float t = 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j) t = fmaf(bf_half(u[s][j], h), ks.df[j], t);
        accb[0] = fmaf(cw[i] * t, t, accb[0]);
        cw[i] = t;
      }
#pragma unroll 1
    for (int s = NP; s < NT; ++s) {
      const uint32_t* lts = lt + (s - NP) * K * kBlock + tid;
      float* rls = lr + (s - NP) * 2 * kBlock + tid;
      float t0 = 0.f, t1 = 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const uint32_t v = lts[j * kBlock];
        t0 = fmaf(bf_lo(v), ks.df[j], t0);
        t1 = fmaf(bf_hi(v), ks.df[j], t1);
      }
      float wc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float phi, c;
        cost_eval(rls[h * kBlock], a.cp, phi, c);
        wc[h] = weight(2 * s + h) * c;
      }
      accb[0] = fmaf(wc[0] * t0, t0, accb[0]);
      accb[0] = fmaf(wc[1] * t1, t1, accb[0]);
    }
    double dHd;
    if (!gang_reduce1(accb[0], a, tile, nbar, ctx.base, ctx.ebase, sm, dHd, [&] {
          if (between) between_frames<SEQ>(a, ctx, thread_index() - 64, kBlock - 64);
        }))
      return false;
    if (wave0_exchange(a) && a.G > 1) between = false;
    if (!(dHd > 0.0)) break;
    const float af = cg_advance<K>(a, ks, dHd, it, ctx.lead);
#pragma unroll
    for (int i = 0; i < 2 * NP; ++i) r[i] = fmaf(-af, cw[i], r[i]);
#pragma unroll 1
    for (int s = NP; s < NT; ++s) {   // u.d of the LDS rows again, as in phase B
      const uint32_t* lts = lt + (s - NP) * K * kBlock + tid;
      float* rls = lr + (s - NP) * 2 * kBlock + tid;
      float t0 = 0.f, t1 = 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const uint32_t v = lts[j * kBlock];
        t0 = fmaf(bf_lo(v), ks.df[j], t0);
        t1 = fmaf(bf_hi(v), ks.df[j], t1);
      }
      rls[0] = fmaf(-af, t0, rls[0]);
      rls[kBlock] = fmaf(-af, t1, rls[kBlock]);
    }
    ++steps;
  }
  const bool bad = ks.flag[1] != 0;
  if (between) between_frames<SEQ>(a, ctx, thread_index(), kBlock);

  if (!bad) {
    constexpr int LE = K + 2 + (EXT ? 1 : 0);   // a, ||eta||^2, f (+ pre-processing deviation sum)
    float acce[LE];
#pragma unroll
    for (int j = 0; j < LE; ++j) acce[j] = 0.f;
    if constexpr (EXT) acce[LE - 1] = pupd ? m2sum : 0.f;
    pin_tile(u);
#pragma unroll
    for (int s = 0; s < NP; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = 2 * s + h;
        const float wt = weight(i);
        float phi, c;
        cost_eval(r[i], a.cp, phi, c);
        const float eta = -wt * c * r[i];
        cw[i] = eta;
        acce[K] = fmaf(eta, eta, acce[K]);
        acce[K + 1] = fmaf(wt, phi, acce[K + 1]);
#pragma unroll
        for (int j = 0; j < K; ++j) acce[j] = fmaf(eta, bf_half(u[s][j], h), acce[j]);
      }
#pragma unroll 1
    for (int s = NP; s < NT; ++s) {
      const uint32_t* lts = lt + (s - NP) * K * kBlock + tid;
      float* rls = lr + (s - NP) * 2 * kBlock + tid;
      float et[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float ri = rls[h * kBlock];
        const float wt = weight(2 * s + h);
        float phi, c;
        cost_eval(ri, a.cp, phi, c);
        const float eta = -wt * c * ri;
        et[h] = eta;
        acce[K] = fmaf(eta, eta, acce[K]);
        acce[K + 1] = fmaf(wt, phi, acce[K + 1]);
      }
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const uint32_t v = lts[j * kBlock];
        acce[j] = fmaf(et[0], bf_lo(v), acce[j]);
        acce[j] = fmaf(et[1], bf_hi(v), acce[j]);
      }
    }
    // the final cost and the deviation sum serve the statistics alone
    constexpr int kLate = LE - (K + 1 > 16 ? K + 1 : LE < 16 ? LE : 16);
    if (!gang_reduce<LE, kLate>(acce, a, tile, nbar, ctx.base, ctx.ebase, sm, ks.red)) return false;
    geodesic_setup<K>(a, ks, steps, ctx.lead);
    if (sm.ctl[2]) return false;
    if (ctx.lead && tid == 0) {
      a.stats->f[steps] = ks.red[K + 1];
      if (EXT && pupd) ks.pre_sum = ks.red[K + 2];
    }
    trace_point(a, tile, 60);

    uint16_t* __restrict__ Uw = (uint16_t*)a.U;
    const float cm1 = ks.scal[0], sz = ks.scal[1], nu_f = ks.scal[2];
    const bool upd = ks.flag[2] != 0;
    // a sequence keeps U in the registers (the next frame starts from them)
    // and stores it after its last frame only, in a loop of its own, so the
    // update of the other frames carries no per-entry store decisions
    const bool store_u = !SEQ || fi + 1 >= a.nseq;
    if (SEQ && upd) u_pending = !store_u;
    pin_tile(u);
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const int q0 = 2 * (tid + s * kBlock);
      if (q0 >= ctx.nq) continue;
      const bool has1 = (vbits >> (2 * s + 1)) & 1u;
      const int c = plane_of(q0, ctx.npx);
      const int e = c * a.P + ctx.p0 + (q0 - c * ctx.npx);
      const int e1 = ((sbits >> s) & 1u) ? e + 1 + (a.P - ctx.npx) : e + 1;
      float rl0 = r[2 * s], rl1 = r[2 * s + 1];
      if (upd) {
        float uv0 = 0.f, ua0 = 0.f, uv1 = 0.f, ua1 = 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const float a0 = bf_lo(u[s][j]), a1 = bf_hi(u[s][j]);
          uv0 = fmaf(a0, ks.vf[j], uv0);
          ua0 = fmaf(a0, ks.af[j], ua0);
          uv1 = fmaf(a1, ks.vf[j], uv1);
          ua1 = fmaf(a1, ks.af[j], ua1);
        }
        const float coef0 = fmaf(cm1, uv0, -sz * (cw[2 * s] - ua0));
        const float coef1 = fmaf(cm1, uv1, -sz * (cw[2 * s + 1] - ua1));
#pragma unroll
        for (int j = 0; j < K; ++j) {
          // columns >= k stay 0 (v_j = 0)
          u[s][j] = pack_bf16_rne(fmaf(coef0, ks.vf[j], bf_lo(u[s][j])), fmaf(coef1, ks.vf[j], bf_hi(u[s][j])));
        }
        if (a.labels_after_update) {
          rl0 = fmaf(-coef0, nu_f, rl0);
          rl1 = fmaf(-coef1, nu_f, rl1);
        }
      }
      if (pre && pupd) {   // the frame joined the running average: store it
        pre_store(a, e, bf_lo(ld_u16(xg, 2u * (unsigned)e)), pinv_n);
        if (has1) pre_store(a, e1, bf_lo(ld_u16(xg, 2u * (unsigned)e1)), pinv_n);
      }
      if (EXT && a.score) {
        a.score[e] = fabsf(rl0);
        if (has1) a.score[e1] = fabsf(rl1);
      }
      s_flag[q0] = (fabsf(rl0) >= a.delta) ? 1 : 0;
      if (has1) s_flag[q0 + 1] = (fabsf(rl1) >= a.delta) ? 1 : 0;
    }
    if (upd && store_u) store_tile();
#pragma unroll 1
    for (int s = NP; s < NT; ++s) {   // LDS pairs (no optional features)
      const int q0 = 2 * (tid + s * kBlock);
      if (q0 >= ctx.nq) continue;
      const uint32_t* lts = lt + (s - NP) * K * kBlock + tid;
      float* rls = lr + (s - NP) * 2 * kBlock + tid;
      const bool has1 = (vbits >> (2 * s + 1)) & 1u;
      const int c = plane_of(q0, ctx.npx);
      const int e = c * a.P + ctx.p0 + (q0 - c * ctx.npx);
      const int e1 = ((sbits >> s) & 1u) ? e + 1 + (a.P - ctx.npx) : e + 1;
      float rl0 = rls[0], rl1 = rls[kBlock];
      if (upd) {
        float uv0 = 0.f, ua0 = 0.f, uv1 = 0.f, ua1 = 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const uint32_t v = lts[j * kBlock];
          const float a0 = bf_lo(v), a1 = bf_hi(v);
          uv0 = fmaf(a0, ks.vf[j], uv0);
          ua0 = fmaf(a0, ks.af[j], ua0);
          uv1 = fmaf(a1, ks.vf[j], uv1);
          ua1 = fmaf(a1, ks.af[j], ua1);
        }
        float et[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          float phi, c;
          const float ri = rls[h * kBlock];
          cost_eval(ri, a.cp, phi, c);
          et[h] = -weight(2 * s + h) * c * ri;
        }
        const float coef0 = fmaf(cm1, uv0, -sz * (et[0] - ua0));
        const float coef1 = fmaf(cm1, uv1, -sz * (et[1] - ua1));
#pragma unroll
        for (int j = 0; j < K; ++j)
          if (j < a.k) {
            const uint32_t v = lts[j * kBlock];
            const uint32_t nw = pack_bf16_rne(fmaf(coef0, ks.vf[j], bf_lo(v)), fmaf(coef1, ks.vf[j], bf_hi(v)));
            uint16_t* col = Uw + (long long)j * a.ldU;
            if (al) {
              st_u32(col, 2u * (unsigned)e, nw);
            } else {
              st_u16(col, 2u * (unsigned)e, (uint16_t)(nw & 0xFFFFu));
              if (has1) st_u16(col, 2u * (unsigned)e1, (uint16_t)(nw >> 16));
            }
          }
        if (a.labels_after_update) {
          rl0 = fmaf(-coef0, nu_f, rl0);
          rl1 = fmaf(-coef1, nu_f, rl1);
        }
      }
      s_flag[q0] = (fabsf(rl0) >= a.delta) ? 1 : 0;
      if (has1) s_flag[q0 + 1] = (fabsf(rl1) >= a.delta) ? 1 : 0;
    }
    trace_point(a, tile, 61);
    write_labels<SEQ>(a, s_flag, ctx.p0, ctx.npx);
    trace_point(a, tile, 62);
  }
  frame_epochs(a, ctx, bad, nbar);
  tile_end(a, tile, ks, ctx, steps, restarts, bad, nbar);
  if (!SEQ || NL > 0 || ++fi >= a.nseq) break;   // sequences: register tiles only

  // ---- next frame of a sequence (as in the float32 tile) ----
  next_frame_begin(ks, ctx, bad);
  xg = (const uint16_t*)(global_ptr(a.xtab ? a.xtab[ctx.n % a.ring] : a.seq[fi]));
#pragma unroll
  for (int s = 0; s < NP; ++s) {   // both entries of a pair into the first's register
    const int q0 = 2 * (tid + s * kBlock);
    const bool in = q0 < ctx.nq, has1 = q0 + 1 < ctx.nq;
    const int c = plane_of(q0, ctx.npx);
    const int e = in ? c * a.P + ctx.p0 + (q0 - c * ctx.npx) : ctx.p0;
    const int e1 = !has1 ? e : ((sbits >> s) & 1u) ? e + 1 + (a.P - ctx.npx) : e + 1;
    const unsigned b0 = 2u * (unsigned)e, b1 = 2u * (unsigned)e1;
    r[2 * s] = __uint_as_float(al ? ld_u32(xg, b0) : (ld_u16(xg, b0) | (ld_u16(xg, b1) << 16)));
  }
  if (!bad) {
    fbits = 0;
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const int q0 = 2 * (tid + s * kBlock);
      const bool in = q0 < ctx.nq, has1 = q0 + 1 < ctx.nq, split = (sbits >> s) & 1u;
      const int pl = in ? q0 - plane_of(q0, ctx.npx) * ctx.npx : 0;
      if (in && pixel_label(s_flag, a.C, ctx.npx, pl)) fbits |= 1u << (2 * s);
      if (has1 && pixel_label(s_flag, a.C, ctx.npx, split || !has1 ? 0 : pl + 1)) fbits |= 2u << (2 * s);
    }
  }
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int q0 = 2 * (tid + s * kBlock);
    const uint32_t xw = __float_as_uint(r[2 * s]);
    float acc0 = bf_lo(xw), acc1 = bf_hi(xw);
#pragma unroll
    for (int j = 0; j < K; ++j) {
      acc0 = fmaf(-bf_lo(u[s][j]), ks.yf[j], acc0);
      acc1 = fmaf(-bf_hi(u[s][j]), ks.yf[j], acc1);
    }
    r[2 * s] = q0 < ctx.nq ? acc0 : 0.f;
    r[2 * s + 1] = q0 + 1 < ctx.nq ? acc1 : 0.f;
  }
  }
  // the last frame stored nothing (rejected, or no step): store the updated tile
  if (SEQ && u_pending) store_tile();
  return true;
}

// One workgroup's share of one frame in the storage type's register layout.
// Returns false when the gang aborted.
// EXT: the optional features are compiled in (pre-processing when the
// stream has its statistics, per-entry label scores when a score buffer is
// given); without it the hot path carries none of their code.  WIDE: the
// steps that reduce H with the gradient in one wide exchange (the IRLS
// variant and the one-exchange curvature schedule of CG) are compiled in as
// well: float32 tiles of the single-stream kernel only, as the H partials
// would spill the packed tile and the batch kernel's registers.
// SEQ: the sequence form (a.nseq frames per launch, the tile kept in
// registers between frames), a separate instantiation so that the one-frame
// kernels carry none of its loop.
template <int K, int NR, typename TS, bool EXT, bool WIDE = false, int NL = 0, bool SEQ = false>
__device__ __forceinline__ bool run_tile(const FrameArgs& a, const int tile, FrameSmem& sm,
                                         uint32_t* __restrict__ lt = nullptr) {
  if constexpr (sizeof(TS) == 2) {
    static_assert(NR % 2 == 0, "bfloat16 tiles hold row pairs");
    return frame_tile_packed<K, NR / 2, EXT, NL, SEQ>(a, tile, sm, lt);
  } else {
    static_assert(NL == 0, "LDS row pairs: bfloat16 tiles only");
    return frame_tile<K, NR, EXT, WIDE, SEQ>(a, tile, sm);
  }
}

// Workgroups of a frame kernel that a compute unit holds: 4, 3 and 2 up to the
// given k, else 1.
struct PerUnit {
  int four, three, two;
};
constexpr int per_unit(const PerUnit& u, int K) { return K <= u.four ? 4 : K <= u.three ? 3 : K <= u.two ? 2 : 1; }
// Without a register limit: all loads of a tile are in flight before any is used.
template <int NR, typename TS, bool EXT>
constexpr PerUnit wide_per_unit() {
  if constexpr (sizeof(TS) == 4) {
    if constexpr (EXT)
      return NR == 1 ? PerUnit{0, 0, 16} : NR == 2 ? PerUnit{0, 0, 11} : NR == 4 ? PerUnit{0, 0, 7}
           : NR == 8 ? PerUnit{0, 0, 1} : PerUnit{0, 0, 0};
    else
      return NR == 1 ? PerUnit{0, 16, 16} : NR == 2 ? PerUnit{0, 6, 16} : NR == 4 ? PerUnit{0, 1, 14}
           : NR == 8 ? PerUnit{0, 0, 6} : PerUnit{0, 0, 1};
  } else {
    if constexpr (EXT)
      return NR == 2 ? PerUnit{0, 4, 16} : NR == 4 ? PerUnit{0, 0, 16} : NR == 8 ? PerUnit{0, 0, 6} : PerUnit{0, 0, 0};
    else
      return NR == 2 ? PerUnit{0, 9, 16} : NR == 4 ? PerUnit{0, 1, 16} : NR == 8 ? PerUnit{0, 0, 8} : PerUnit{0, 0, 0};
  }
}
// With one.  A gang must be resident as a whole, so these times the compute units
// are the largest gangs that pros_set_launch accepts.  The limit costs up to 4 %
// of a frame (160x120x3, k = 15, float32 33.4 and 34.9 us; 640x480x3, k = 9,
// bfloat16 48.4 and 49.9), so a kernel of its own has it, for the gangs that need it.
template <int NR, typename TS, bool EXT>
constexpr PerUnit dense_per_unit() {
  if constexpr (sizeof(TS) == 4) {
    if constexpr (EXT)
      return NR == 1 ? PerUnit{3, 7, 16} : NR == 2 ? PerUnit{0, 5, 16} : NR == 4 ? PerUnit{0, 2, 8}
           : NR == 8 ? PerUnit{0, 0, 3} : PerUnit{0, 0, 0};
    else
      return NR == 1 ? PerUnit{10, 16, 16} : NR == 2 ? PerUnit{4, 11, 16} : NR == 4 ? PerUnit{0, 4, 15}
           : NR == 8 ? PerUnit{0, 0, 6} : PerUnit{0, 0, 1};
  } else {
    if constexpr (EXT)
      return NR == 2 ? PerUnit{5, 15, 16} : NR == 4 ? PerUnit{0, 8, 16} : NR == 8 ? PerUnit{0, 2, 11}
           : NR == 16 ? PerUnit{0, 0, 3} : PerUnit{0, 0, 0};
    else
      return NR == 2 ? PerUnit{10, 15, 16} : NR == 4 ? PerUnit{2, 9, 16} : NR == 8 ? PerUnit{0, 2, 12}
           : NR == 16 ? PerUnit{0, 0, 3} : PerUnit{0, 0, 0};
  }
}

// WGS: workgroups of a compute unit that the registers are limited for (1: no limit).
template <int K, int NR, typename TS, bool EXT, bool SEQ = false, int WGS = 1>
__global__ __launch_bounds__(kBlock, WGS * kWaves / 4) void frame_kernel(FrameArgs a) {
  __shared__ FrameSmem sm;
  run_tile<K, NR, TS, EXT, EXT, 0, SEQ>(a, blockIdx.x, sm);
}

}  // inline namespace PROST_BLOCK_NS
}  // namespace prost
