// ct_kernels.hip -- HIP kernels of the CT library for gfx950 (CDNA4).
//
// Work is exact bitwise integer arithmetic on uint64 words; nothing here is
// a dense contraction, so there is no MFMA: the kernels are built around
// coalesced 512-byte granule loads (one word per lane of a wave64), wave
// ballots and LDS.
//
// propagate_kernel runs a job either in solo mode -- one workgroup, the whole
// of Alg. 1-3 with no hand-off between workgroups (small tables, negative
// tables) -- or, for one synchronous call of a table whose update one
// workgroup takes, in split mode, as items of one launch:
//   prep   (calls that pop, and pure push/pop calls)  backtrack restore, pushes
//   update updateTable (Alg. 2) with the Delta / s_val / s_sup prologue of
//          Alg. 1 in LDS; records the call's pushes, partitions the sparse
//          index and decides FAIL (Alg. 1's failure test)
//   filter filterDomains (Alg. 3), one domain word per wave, residue word
//          first, then a scan of active granules
// An item only waits for earlier items (the update for the prep when the call
// pops, the filters for the update), and all of them are resident.  Waits are
// bounded: on expiry the kernel records a device error and the remaining work
// of the launch is skipped.  Larger tables and batches run staged
// (ct_staged.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ct_device.h"

namespace ctk {

constexpr int NGW = 2;                 // granules per wave per update step (split mode)
constexpr int NGS = 4;                 // default granules per wave per step (solo mode)
constexpr int LANE_SCAN = 16;          // words each missing lane checks before the wave scan
constexpr int FULL_SCAN_GRAN = 4;      // at most this many active granules: misses test every active word
constexpr int FULL_SCAN_VALS = 8;      //   for this many values per round trip
constexpr int ROW_UNROLL = 8;          // support rows loaded per batch
constexpr int ROWS_CHUNK = 8192;       // row-list entries staged in LDS at a time
constexpr uint32_t SPIN_LIMIT = 1u << 22;
constexpr int32_t STAR_CELL = (int32_t)0x80000000;  // a short table's cell: every value of its column

__device__ __forceinline__ int lane_id() { return threadIdx.x & (WAVE - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x / WAVE; }

__device__ __forceinline__ void st_release(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_relaxed(int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A word of the slot's previous domains (JF_COHLAST: read at device scope,
// around this XCD's L2)
__device__ __forceinline__ uint64_t ld_last(const CT_G uint64_t* p, bool coh) {
  return coh ? __hip_atomic_load(const_cast<CT_G uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

// The slot's array addresses (they never change), loaded together: an item
// that reads them early has them when its first loads from the arrays go.
struct SlotPtrs {
  CT_G uint64_t* ct;
  CT_G int32_t* idx[2];
  CT_G int32_t* stamp;
  CT_G uint64_t* trailWords;
  CT_G TrailHdr* trailHdr;
  int64_t trailCap;
};

struct Shared {
  int32_t item, ok, isLast, status, noop, nseg, nrows, limit, serial, depth, bad_stray, bad_sub;
  int64_t trailTop;
  int32_t size[MAX_ARITY];
  int32_t dcnt[MAX_ARITY];
  int32_t segOf[MAX_ARITY];   // var -> segment, -1 if not in s_val
  int32_t segEnd[MAX_ARITY];  // exclusive end of segment rows
  int32_t segInc[MAX_ARITY];
  int32_t wsum[WAVES];
  int32_t trailCount;          // trail entries of a job run by one workgroup
  uint64_t din[MAX_D];         // the job's first MAX_D domain words (the rest are read from memory)
  uint64_t dout[MAX_D];        // negative tables: the filtered domains, published if no domain empties
  uint32_t rows[ROWS_CHUNK];   // entries [k0, k0 + ROWS_CHUNK) of the job's row list
  uint8_t nz[MAX_GRAN];        // granule non-zero flags of a job run by one workgroup
  uint16_t gidx[MAX_GRAN];     // granule list of a job run by one workgroup
  unsigned long long fcnt[3];  // a filter item's counters (residue checks, misses, scans)
  int32_t cur;                 // the slot's index buffer in use at the job's start (prologue)
  SlotPtrs sp;                 // the slot's array addresses (prologue)
  int32_t seOp, seNPop, seNPush, seSerial, seDepth;  // resident split schedule: the call's header
};

__device__ __forceinline__ SlotPtrs slot_ptrs(const SlotDesc* s) {
  SlotPtrs p;
  p.ct = s->ct;
  p.idx[0] = s->idx[0];
  p.idx[1] = s->idx[1];
  p.stamp = s->stamp;
  p.trailWords = s->trailWords;
  p.trailHdr = s->trailHdr;
  p.trailCap = s->trailCap;
  return p;
}

// Record a device error: the host sees it through hostErr (pinned) and the
// other workgroups of the launch stop waiting.
__device__ void raise_error(const KArgs& a, int code) {
  atomicExch(&a.queue[3], code);
  if (a.hostErr) {
    __hip_atomic_store(a.hostErr, code, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Thread 0 spins until *flag == want; the result is broadcast to the block.
// The spin reads the flag relaxed and takes one acquire fence once it holds:
// an acquire load per poll would invalidate the L2 on every iteration (an
// agent-scope acquire does on this chip), under the feet of the workgroup
// being waited for.
__device__ bool block_wait(const KArgs& a, int32_t* flag, int32_t want, Shared& sh) {
  if (threadIdx.x == 0) {
    int ok = 1;
    for (uint32_t it = 0;; ++it) {
      if (ld_relaxed(flag) == want) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        break;
      }
      if (ld_relaxed(&a.queue[3])) { ok = 0; break; }
      if (it > SPIN_LIMIT) { raise_error(a, 1); ok = 0; break; }
      __builtin_amdgcn_s_sleep(1);
    }
    sh.ok = ok;
  }
  __syncthreads();
  const int ok = sh.ok;
  __syncthreads();
  return ok != 0;
}

// Workgroup barrier that orders LDS only: global stores still in flight
// need not complete here (__syncthreads waits for them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Inclusive prefix sum over the 64 lanes (every lane active), with DPP
// moves (VALU, no LDS round trips): shifts within rows of 16 lanes, then
// the row broadcasts of lanes 15 and 31.
__device__ __forceinline__ int wave_scan_incl(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_scan_incl(v), WAVE - 1); }

// Exclusive prefix sum over the block; *total receives the sum.
// (LDS_ONLY: its barriers order LDS only, so global stores still in flight
// need not complete there)
template <bool LDS_ONLY = false>
__device__ int block_scan_excl(int v, int* total, Shared& sh) {
  const int lane = lane_id(), w = wave_id();
  const int x = wave_scan_incl(v);
  if (lane == WAVE - 1) sh.wsum[w] = x;
  if (LDS_ONLY) lds_barrier();
  else __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const int s = sh.wsum[k];
    if (k < w) off += s;
    tot += s;
  }
  if (LDS_ONLY) lds_barrier();
  else __syncthreads();
  *total = tot;
  return off + x - v;
}

// The job descriptor by value: from the batch array (global memory) or from
// the kernel arguments; a reference chosen between the two would be a flat
// pointer and turn every field access into a flat load.
__device__ __forceinline__ DevJob job_of(const KArgs& a, int j) {
  DevJob J;
  if (a.jobs) J = a.jobs[j];
  else J = a.job;
  return J;
}

__device__ __forceinline__ uint64_t job_din(const KArgs& a, const DevJob& J, int k) {
  return (J.flags & JF_INLINE_DOM) ? a.inl[k] : J.dom_in[k];
}

// Domain word q of the job's input: the prologue's LDS copy for the first
// MAX_D words, memory beyond (inline inputs have at most INLINE_WORDS words,
// all in the copy).
__device__ __forceinline__ uint64_t din_at(const DevJob& J, const Shared& sh, int q) {
  return q < MAX_D ? sh.din[q] : J.dom_in[q];
}

// Word w of the set of all tuples (the starting currTable of a root state
// recomputed from scratch): ones up to the last tuple, zero past it.
__device__ __forceinline__ uint64_t all_tuples_word(const TabDesc* T, int64_t w) {
  if (w >= T->W) return 0ull;
  if (w < T->W - 1 || T->tailBits >= 64) return ~0ull;
  return (1ull << T->tailBits) - 1ull;
}

// Job status for the caller.  Outputs in host memory are published with a
// system-scope release after a system-scope fence, so a host that sees the
// status also sees the domain words written before it.
__device__ __forceinline__ void ll_put(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ void publish_status(const DevJob& J, int st) {
  if (J.flags & JF_LL) {  // a flagged slot: no fence (see JF_LL)
    ll_put(J.ll, eng_slot((uint32_t)st, (uint32_t)J.seq));
    return;
  }
  if (!J.status_out) return;
  if (J.flags & JF_HOST_OUT) {
    __threadfence_system();
    __hip_atomic_store(J.status_out, st, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  } else {
    *J.status_out = st;
  }
}

__device__ __forceinline__ void item_fence(const DevJob& J) {
  if (J.flags & JF_HOST_OUT) __threadfence_system();
  else __threadfence();
}

// Before a job's status is published or its last item is counted: the host
// reads a synchronous call's outputs (pinned memory, JF_HOST_OUT) as soon as
// the status changes, so they must be visible first; a batch's statuses and
// outputs are read after the launch has ended, which makes them visible.  A
// device-scope fence here costs an L2 write-back and invalidate per job (per
// search node: thousands per batch), so batch jobs take none.
__device__ __forceinline__ void status_fence(const DevJob& J) {
  if (J.flags & JF_HOST_OUT) __threadfence_system();
}

// Push nPush levels recording (trailTop, limit, failed, serial, domains);
// the k-th new level continues with serial serialBase + k.  Whole block.
__device__ void push_levels(const DevJob& J, SlotDesc* s, int depth0, int64_t trailTop, int limit,
                            int failed, int serial0, int D) {
  for (int k = 0; k < J.nPush; ++k) {
    const int d = depth0 + k;
    for (int q = threadIdx.x; q < D; q += BLOCK)
      s->levelDom[(int64_t)d * D + q] = ld_last(&s->lastDom[q], J.flags & JF_COHLAST);
    if (threadIdx.x == 0) {
      Level L;
      L.trailTop = trailTop;
      L.limit = limit;
      L.failed = failed;
      L.serial = k == 0 ? serial0 : J.serialBase + k - 1;
      L.pad = 0;
      s->levels[d] = L;
    }
  }
}

// ---------------------------------------------------------------------------
// prep: pops then pushes (whole block), for jobs that pop or only push/pop
// ---------------------------------------------------------------------------
__device__ void apply_pops_pushes(const DevJob& J, Shared& sh) {
  SlotDesc* s = J.slot;
  const int D = J.tab->D;
  for (int p = 0; p < J.nPop; ++p) {
    if (threadIdx.x == 0) {
      sh.depth = s->depth - 1;
      sh.trailTop = s->trailTop;
    }
    __syncthreads();
    const int d = sh.depth;
    const Level L = s->levels[d];
    const int64_t top = sh.trailTop;
    // entries of one level name distinct granules: restore 4 per wave at once
    for (int64_t e0 = L.trailTop + 4 * wave_id(); e0 < top; e0 += 4 * WAVES) {
      TrailHdr h[4];
      uint64_t w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t e = e0 + j;
        if (e < top) {
          h[j] = s->trailHdr[e];
          w[j] = s->trailWords[e * GW + lane_id()];
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (e0 + j < top) {
          s->ct[(int64_t)h[j].gran * GW + lane_id()] = w[j];
          if (lane_id() == 0) s->stamp[h[j].gran] = h[j].oldStamp;
        }
      }
    }
    for (int q = threadIdx.x; q < D; q += BLOCK) s->lastDom[q] = s->levelDom[(int64_t)d * D + q];
    __syncthreads();
    if (threadIdx.x == 0) {
      s->trailTop = L.trailTop;
      s->limit = L.limit;
      s->failed = L.failed;
      s->serial = L.serial;
      s->depth = d;
    }
    __syncthreads();
  }
  if (J.nPush > 0) {
    if (threadIdx.x == 0) {
      sh.depth = s->depth;
      sh.trailTop = s->trailTop;
      sh.limit = s->limit;
      sh.status = s->failed;
      sh.serial = s->serial;
    }
    __syncthreads();
    push_levels(J, s, sh.depth, sh.trailTop, sh.limit, sh.status, sh.serial, D);
    __syncthreads();
    if (threadIdx.x == 0) {
      s->depth = sh.depth + J.nPush;
      s->serial = J.serialBase + J.nPush - 1;
    }
    __syncthreads();
  }
}

__device__ __forceinline__ void do_prep(const KArgs& a, const DevJob& J, Shared& sh) {
  apply_pops_pushes(J, sh);
  if (threadIdx.x == 0) {
    // (the barrier at the end of apply_pops_pushes orders the block's
    // writes before thread 0's release)
    if (!(J.flags & JF_PROPAGATE)) publish_status(J, ST_OK);
    else st_release(&J.slot->prepDone, 1);  // consumed (and reset) by the job's last update item
  }
}

__device__ void stage_rows(const DevJob& J, Shared& sh, int k0, const CT_G uint64_t* lastArr = nullptr,
                           const CT_G WordDesc* wordsArr = nullptr);

// ---------------------------------------------------------------------------
// prologue of Alg. 1 for one job, in LDS.  Its barriers order LDS only: what
// it stores to memory (pushed levels) is read by later calls.  The job's
// granule list goes into sh.gidx as well, loaded with the domain words.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void prologue(const KArgs& a, const DevJob& J, Shared& sh, bool pushHere) {
  const TabDesc* T = J.tab;
  SlotDesc* s = J.slot;
  const bool fromRoot = J.flags & JF_FROM_ROOT;
  const bool root = J.flags & JF_ROOT;
  const bool scratch = J.flags & JF_SCRATCH;
  const int n = T->n, D = T->D;
  // read before the first barrier (a load after one waits its round trip):
  // the table's and slot's addresses, this thread's first domain word with
  // its record and previous word, and its entry of both index buffers (the
  // one in use is known after the barrier); addresses are clamped, values
  // selected afterwards
  const int policy = T->policy;
  const int nGran = T->nGran;
  const CT_G WordDesc* words = T->words;
  const CT_G uint64_t* last = fromRoot ? T->dom0 : s->lastDom;
  const int q0 = min((int)threadIdx.x, D - 1);
  const uint64_t din0 = job_din(a, J, q0);
  const WordDesc wd0 = words[q0];
  const bool coh = J.flags & JF_COHLAST;
  const uint64_t ld0 = ld_last(last + q0, coh);
  const int p0 = min((int)threadIdx.x, nGran - 1);
  int ga = 0, gb = 0;
  if (!scratch) {
    ga = (fromRoot ? T->idx0 : s->idx[0])[p0];
    gb = fromRoot ? ga : s->idx[1][p0];
  }
  if (threadIdx.x == 0) {
    sh.bad_stray = 0;
    sh.bad_sub = 0;
    if (scratch) {  // every tuple, every granule
      sh.limit = T->nGran;
      sh.status = ST_OK;
    } else if (fromRoot) {
      sh.limit = T->limit0;
      sh.status = T->rootFailed ? ST_STATE : ST_OK;
    } else {
      sh.limit = s->limit;
      sh.status = s->failed ? ST_STATE : ST_OK;
    }
    sh.trailTop = s->trailTop;
    sh.cur = s->cur;
    sh.sp = slot_ptrs(s);
    sh.serial = J.nPush > 0 ? J.serialBase + J.nPush - 1 : s->serial;
    if (pushHere) {
      // this job's pushes record the state before it (levels of push_levels)
      const int d0 = s->depth;
      const int failed = s->failed;
      for (int k = 0; k < J.nPush; ++k) {
        Level L;
        L.trailTop = sh.trailTop;
        L.limit = sh.limit;
        L.failed = failed;
        L.serial = k == 0 ? s->serial : J.serialBase + k - 1;
        L.pad = 0;
        s->levels[d0 + k] = L;
      }
      sh.depth = d0;
      s->depth = d0 + J.nPush;
      s->serial = J.serialBase + J.nPush - 1;
    }
  }
  for (int i = threadIdx.x; i < n; i += BLOCK) {
    sh.size[i] = 0;
    sh.dcnt[i] = 0;
  }
  lds_barrier();
  // one domain word per thread and pass: validation, Delta, |dom| per
  // variable; the first pass takes the words loaded above, and wider tables
  // load PRE_PASSES passes at once (one round trip, not one per pass: the
  // input may be in host memory)
  constexpr int PRE_PASSES = 4;
  uint64_t dinK = 0, dlK = 0;  // this thread's word and Delta word (D <= BLOCK)
  for (int qg = threadIdx.x; qg < D; qg += PRE_PASSES * BLOCK) {
    uint64_t dv[PRE_PASSES], lv[PRE_PASSES];
    WordDesc wv[PRE_PASSES];
#pragma unroll
    for (int g = 0; g < PRE_PASSES; ++g) {
      const int q = min(qg + g * BLOCK, D - 1);
      const bool first = g == 0 && qg == (int)threadIdx.x;
      if (g > 0 && D <= BLOCK) break;  // (one pass: nothing more to load)
      dv[g] = first ? din0 : job_din(a, J, q);
      wv[g] = first ? wd0 : words[q];
      lv[g] = first ? ld0 : ld_last(last + q, coh);
    }
#pragma unroll
    for (int g = 0; g < PRE_PASSES; ++g) {
      const int q = qg + g * BLOCK;
      if (q >= D) break;
      const uint64_t din = dv[g];
      const int i = wv[g].var;
      const VarDesc v = wv[g].v;
      const int used = v.dsize - 64 * (q - v.domOff);
      if (used < 64 && (din >> used) != 0) sh.bad_stray = 1;
      uint64_t dl = 0;
      if (!root) {
        const uint64_t ld = lv[g];
        if (din & ~ld) sh.bad_sub = 1;
        dl = ld & ~din;
        if (pushHere)
          for (int k = 0; k < J.nPush; ++k) s->levelDom[(int64_t)(sh.depth + k) * D + q] = ld;
      }
      if (q < MAX_D) sh.din[q] = din;
      if (q == (int)threadIdx.x) {
        dinK = din;
        dlK = dl;
      }
      atomicAdd(&sh.size[i], __popcll(din));
      atomicAdd(&sh.dcnt[i], __popcll(dl));
    }
  }
  if ((int)threadIdx.x < nGran) sh.gidx[threadIdx.x] = (uint16_t)(scratch ? (int)threadIdx.x : sh.cur ? gb : ga);
  const CT_G int32_t* gsrc = fromRoot ? T->idx0 : sh.sp.idx[sh.cur];
  for (int p = threadIdx.x + BLOCK; p < nGran; p += BLOCK) sh.gidx[p] = (uint16_t)(scratch ? p : gsrc[p]);
  lds_barrier();
  if (threadIdx.x < WAVE) {
    // wave 0: the segments of s_val in variable order (prefix sums over the
    // variables, 64 at a time)
    const int lane = threadIdx.x;
    int nseg = 0, nrows = 0;
    for (int i0 = 0; i0 < n; i0 += WAVE) {
      const int i = i0 + lane;
      bool inSval = false;
      int inc = 0, cnt = 0;
      if (i < n) {
        inSval = root || sh.dcnt[i] > 0;  // |dom| changed since the last call
        if (inSval) {
          inc = root ? 0 : (policy == 2 ? 1 : policy == 1 ? 0 : (sh.dcnt[i] < sh.size[i] ? 1 : 0));
          cnt = inc ? sh.dcnt[i] : sh.size[i];
        }
      }
      const int segIncl = wave_scan_incl(inSval ? 1 : 0);
      const int rowsIncl = wave_scan_incl(cnt);
      if (i < n) {
        if (inSval) {
          const int sg = nseg + segIncl - 1;
          sh.segOf[i] = sg;
          sh.segInc[sg] = inc;
          sh.segEnd[sg] = nrows + rowsIncl;
        } else {
          sh.segOf[i] = -1;
        }
      }
      nseg += __builtin_amdgcn_readlane(segIncl, WAVE - 1);
      nrows += __builtin_amdgcn_readlane(rowsIncl, WAVE - 1);
    }
    if (lane == 0) {
      if (sh.status == ST_OK) {
        if (sh.bad_stray) sh.status = ST_INVALID;
        else if (sh.bad_sub) sh.status = ST_NOT_SUBSET;
      }
      sh.nseg = nseg;
      sh.nrows = nrows;
      sh.noop = (nseg == 0) && !fromRoot;
    }
  }
  lds_barrier();
  if (sh.status != ST_OK || sh.noop) return;
  if (D <= BLOCK && sh.nrows <= ROWS_CHUNK) {
    // the row list from the words in registers: segments follow variable
    // order and a variable's words are consecutive, so a word's first entry
    // is the exclusive prefix sum of the selected bits of the words before it
    const int q = threadIdx.x;
    const int sg = q < D ? sh.segOf[wd0.var] : -1;
    const bool inc = sg >= 0 && sh.segInc[sg];
    uint64_t bits = sg < 0 ? 0ull : inc ? dlK : dinK;
    int tot = 0;
    int off = block_scan_excl<true>(__popcll(bits), &tot, sh);
    const int base = wd0.v.rowStart + (q - wd0.v.domOff) * 64;
    while (bits) {
      const int b = __ffsll((unsigned long long)bits) - 1;
      bits &= bits - 1;
      sh.rows[off++] = (uint32_t)(base + b);
    }
  } else {
    stage_rows(J, sh, 0, last, words);
  }
  lds_barrier();
}

// Entries [k0, k0 + ROWS_CHUNK) of the job's row list into sh.rows: the
// selected rows of every segment, in segment order; word q of variable i
// contributes the set bits of its Delta word (incremental) or domain word
// (reset) in ascending order.  Whole block; a barrier must follow.
// (lastArr, wordsArr: the previous domains and the word records as the
// caller read their addresses, else read here)
__device__ void stage_rows(const DevJob& J, Shared& sh, int k0, const CT_G uint64_t* lastArr,
                           const CT_G WordDesc* wordsArr) {
  const TabDesc* T = J.tab;
  const CT_G uint64_t* last = lastArr ? lastArr : (J.flags & JF_FROM_ROOT) ? T->dom0 : J.slot->lastDom;
  const bool coh = J.flags & JF_COHLAST;
  const CT_G WordDesc* words = wordsArr ? wordsArr : T->words;
  const int k1 = k0 + ROWS_CHUNK;
  for (int q = threadIdx.x; q < T->D; q += BLOCK) {
    const WordDesc wd = words[q];
    const int sg = sh.segOf[wd.var];
    if (sg < 0) continue;
    const VarDesc v = wd.v;
    const int inc = sh.segInc[sg];
    int off = sg == 0 ? 0 : sh.segEnd[sg - 1];
    for (int k = v.domOff; k < q && off < k1; ++k) {
      const uint64_t dk = din_at(J, sh, k);
      off += __popcll(inc ? (ld_last(last + k, coh) & ~dk) : dk);
    }
    const uint64_t dq = din_at(J, sh, q);
    uint64_t bits = inc ? (ld_last(last + q, coh) & ~dq) : dq;
    if (off >= k1 || off + __popcll(bits) <= k0) continue;
    const int base = v.rowStart + (q - v.domOff) * 64;
    while (bits && off < k1) {
      const int b = __ffsll((unsigned long long)bits) - 1;
      bits &= bits - 1;
      if (off >= k0) sh.rows[off - k0] = (uint32_t)(base + b);
      ++off;
    }
  }
}

// ---------------------------------------------------------------------------
// updateTable (Alg. 2) for NG granules per wave starting at position p0,
// RU support rows in flight per granule.  Granule flags go to LDS.
// ---------------------------------------------------------------------------
template <int NG, int RU = ROW_UNROLL>
__device__ __forceinline__ void update_granules(const KArgs& a, const DevJob& J, Shared& sh, int p0,
                                int* trailCounter, const SlotPtrs* sp = nullptr) {
  const TabDesc* T = J.tab;
  SlotDesc* s = J.slot;
  const bool fromRoot = J.flags & JF_FROM_ROOT;
  const bool root = J.flags & JF_ROOT;
  // levels exist only above depth 0: nothing is saved at depth 0
  const bool trailOn = !fromRoot && !root && J.depthAfter > 0;
  const int nGran = T->nGran;
  const int64_t stride = T->stride;
  const int64_t W = T->W;
  const int limit = sh.limit;
  const int status = sh.status;
  const int noop = sh.noop;
  const int nseg = sh.nseg, nrows = sh.nrows;
  const int serial = sh.serial;
  const int lane = lane_id();
  const bool scratch = J.flags & JF_SCRATCH;
  // the slot's arrays as the prologue read them (sp, in LDS), or from the
  // descriptor
  const CT_G uint64_t* srcCt = fromRoot ? T->ct0 : sp ? sp->ct : s->ct;
  const CT_G int32_t* stampArr = sp ? sp->stamp : s->stamp;
  const int64_t trailTop = sh.trailTop;

  // Loads below are unconditional, from clamped (always valid) addresses, and
  // their results are selected afterwards: a load under a branch is followed
  // by a wait for it, which would serialize the round trips to memory.
  unsigned long long nAct = 0;
  int pos[NG], g[NG], gs[NG], stv[NG];
  bool act[NG];
  uint64_t old[NG], m[NG], acc[NG];
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    pos[u] = p0 + u;
    const int pc = min(pos[u], nGran - 1);
    g[u] = scratch ? pc : (int)sh.gidx[pc];
    if (pos[u] >= nGran) g[u] = -1;
    act[u] = pos[u] < limit && status == ST_OK;
    gs[u] = act[u] ? g[u] : 0;
    const uint64_t o = scratch ? all_tuples_word(T, (int64_t)gs[u] * GW + lane) : srcCt[(int64_t)gs[u] * GW + lane];
    const int sv = stampArr[gs[u]];
    old[u] = act[u] ? o : 0ull;
    stv[u] = (act[u] && trailOn && !noop) ? sv : serial;
    m[u] = ~0ull;
    acc[u] = 0ull;
    nAct += act[u] ? 1 : 0;
  }
  // a row list longer than the LDS chunk is staged chunk by chunk, with the
  // whole block (every wave runs this loop the same number of times)
  const bool work = status == ST_OK && !noop;
  const bool chunked = nrows > ROWS_CHUNK;
  int seg = 0;
  int segEnd = nseg > 0 ? sh.segEnd[0] : 0;
  for (int c0 = 0; work && c0 < nrows; c0 += ROWS_CHUNK) {
    if (chunked) {
      __syncthreads();
      stage_rows(J, sh, c0);
      __syncthreads();
    }
    if (nAct == 0) continue;
    const int c1 = min(nrows, c0 + ROWS_CHUNK);
    for (int k0 = c0; k0 < c1; k0 += RU) {
      uint64_t v[RU][NG];
#pragma unroll
      for (int j = 0; j < RU; ++j) {
        const int k = k0 + j;
        const int r = k < c1 ? (int)sh.rows[k - c0] : 0;  // rows past the end are never used
#pragma unroll
        for (int u = 0; u < NG; ++u) v[j][u] = T->S[(int64_t)r * stride + (int64_t)gs[u] * GW + lane];
      }
#pragma unroll
      for (int j = 0; j < RU; ++j) {
        const int k = k0 + j;
        if (k >= c1) break;
        while (k >= segEnd) {
          const int inc = sh.segInc[seg];
#pragma unroll
          for (int u = 0; u < NG; ++u) {
            m[u] &= inc ? ~acc[u] : acc[u];
            acc[u] = 0ull;
          }
          ++seg;
          segEnd = sh.segEnd[seg];
        }
#pragma unroll
        for (int u = 0; u < NG; ++u) acc[u] |= v[j][u];
      }
    }
  }
  if (work && nAct > 0) {
    while (seg < nseg) {  // remaining segments (an empty reset segment gives 0)
      const int inc = sh.segInc[seg];
#pragma unroll
      for (int u = 0; u < NG; ++u) {
        m[u] &= inc ? ~acc[u] : acc[u];
        acc[u] = 0ull;
      }
      ++seg;
    }
  }
  // new words, and which granules need saving on the trail (first change in
  // this level); one trail allocation per wave
  uint64_t nw[NG];
  bool need[NG], wr[NG];
  int nNeed = 0;
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    nw[u] = noop ? old[u] : (old[u] & m[u]);
    const bool changed = act[u] && (__ballot(nw[u] != old[u]) != 0ull);
    need[u] = changed && trailOn && stv[u] != serial;
    nNeed += need[u] ? 1 : 0;
    wr[u] = act[u] && (changed || fromRoot || root);
  }
  int tbase = 0;
  // the slot's arrays, read once: the stores below could otherwise force a
  // reload (and a wait) of the descriptor before each of them
  const SlotPtrs P = sp ? *sp : slot_ptrs(s);
  const int64_t trailCap = P.trailCap;
  CT_G uint64_t* const sCt = P.ct;
  CT_G uint64_t* const sTrailWords = P.trailWords;
  CT_G TrailHdr* const sTrailHdr = P.trailHdr;
  CT_G int32_t* const sStamp = P.stamp;
  CT_G uint64_t* const ctOut = J.ct_out;
  if (nNeed) {
    if (lane == 0) tbase = atomicAdd(trailCounter, nNeed);
    tbase = __shfl(tbase, 0);
  }
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    if (pos[u] >= nGran || status != ST_OK) continue;
    const int64_t w = (int64_t)g[u] * GW + lane;
    if (pos[u] >= limit) {
      // inactive granule (all zero by invariant)
      if (fromRoot) sCt[w] = 0ull;
      if (ctOut && w < W) ctOut[w] = 0ull;
      continue;
    }
    if (need[u]) {
      const int64_t tp = trailTop + tbase++;
      if (tp < trailCap) {
        sTrailWords[tp * GW + lane] = old[u];
        if (lane == 0) {
          TrailHdr h;
          h.gran = g[u];
          h.oldStamp = stv[u];
          sTrailHdr[tp] = h;
          sStamp[g[u]] = serial;
        }
      } else if (lane == 0) {
        raise_error(a, 2);  // capacity is sized so that this cannot happen
      }
    }
    if (wr[u]) sCt[w] = nw[u];
    if (ctOut && w < W) ctOut[w] = nw[u];
    const bool nz = __ballot(nw[u] != 0ull) != 0ull;
    if (lane == 0) sh.nz[pos[u]] = nz ? 1 : 0;
  }
  if (lane == 0 && status == ST_OK) {
    if (nAct && !noop) atomicAdd(&s->stats[S_GRAN_ROWS], nAct * (unsigned long long)nrows);
    if (nNeed) atomicAdd(&s->stats[S_TRAIL], (unsigned long long)nNeed);
  }
}

// ---------------------------------------------------------------------------
// A job that resets its slot to the root (depth 0) and then rejects its input
// still performs the reset: the slot becomes a copy of the table's root state
// (threads tid of nthr, a workgroup or a wave; a rare path, so the whole
// currTable is copied).
// ---------------------------------------------------------------------------
__device__ void slot_reset_root(const TabDesc* T, SlotDesc* s, int serial, int tid, int nthr) {
  for (int64_t w = tid; w < T->stride; w += nthr) s->ct[w] = T->ct0[w];
  for (int p = tid; p < T->nGran; p += nthr) s->idx[0][p] = T->idx0[p];
  for (int q = tid; q < T->D; q += nthr) s->lastDom[q] = T->dom0[q];
  if (tid == 0) {
    s->cur = 0;
    s->limit = T->limit0;
    s->failed = T->rootFailed;
    s->depth = 0;
    s->trailTop = 0;
    s->serial = serial;
  }
}

// ---------------------------------------------------------------------------
// End of updateTable for a job (one workgroup): stable partition of the
// active granule list (survivors first), new limit, trail top, FAIL when no
// granule survives (Alg. 1's failure test).  Returns the job status.
// ---------------------------------------------------------------------------
__device__ int finalize_update(const DevJob& J, Shared& sh, int jobTrail, bool count = true) {
  const TabDesc* T = J.tab;
  // a negative table's currTable holds forbidden tuples: empty means no
  // combination is forbidden, not a failure
  const bool negative = T->kind != 0;
  SlotDesc* s = J.slot;
  const bool fromRoot = J.flags & JF_FROM_ROOT;
  const int limit = sh.limit;
  const int nGran = T->nGran;
  int st = sh.status;
  if (st == ST_OK && !sh.noop) {
    const bool scratch = J.flags & JF_SCRATCH;  // index = identity
    // the index buffers as the prologue read them (sh.sp, sh.cur)
    const int dstBuf = fromRoot ? 0 : 1 - sh.cur;
    CT_G int32_t* dst = sh.sp.idx[dstBuf];
    const int per = (limit + BLOCK - 1) / BLOCK;
    const int b = min((int)threadIdx.x * per, limit);
    const int e = min(b + per, limit);
    int cnt = 0;
    for (int p = b; p < e; ++p) cnt += sh.nz[p];
    int nSurv = 0;
    int sv = block_scan_excl<true>(cnt, &nSurv, sh);
    int zr = nSurv + (b - sv);
    for (int p = b; p < e; ++p) {
      const int gid = scratch ? p : (int)sh.gidx[p];
      const int f = sh.nz[p];
      if (f) dst[sv++] = gid; else dst[zr++] = gid;
    }
    for (int p = limit + threadIdx.x; p < nGran; p += BLOCK)
      dst[p] = scratch ? p : (int)sh.gidx[p];
    if (nSurv == 0 && !negative) st = ST_FAIL;
    if (threadIdx.x == 0) {
      s->cur = dstBuf;
      sh.cur = dstBuf;  // a second pass over the job (negative tables) reads it
      s->limit = nSurv;
      if (fromRoot) {
        s->depth = 0;
        s->trailTop = 0;
        s->serial = J.serialBase;
        s->failed = 0;
      } else {
        s->trailTop = sh.trailTop + jobTrail;
      }
      if (nSurv == 0 && !negative) s->failed = 1;
    }
  } else if (fromRoot && st != ST_OK) {
    slot_reset_root(T, s, J.serialBase, threadIdx.x, blockDim.x);
  }
  if (threadIdx.x == 0) {
    s->status = st;
    s->noop = sh.noop;
    if (count && (st == ST_OK || st == ST_FAIL)) {
      atomicAdd(&s->stats[S_JOBS], 1ull);
      atomicAdd(&s->stats[S_GRAN_IN], (unsigned long long)limit);
      atomicAdd(&s->stats[S_ROWS], (unsigned long long)(sh.noop ? 0 : sh.nrows));
    }
  }
  __syncthreads();
  return st;
}

// ---------------------------------------------------------------------------
// filterDomains (Alg. 3) for domain word q, by one wave: residue word first,
// then the active granules in index order until a support is found.
// ---------------------------------------------------------------------------
// What filterDomains reads for domain word q before currTable is final: the
// word, its variable's size, and per value (lane) the residue and the support
// word at the residue (supports and residues do not change during the
// update), so a filter that waits for the update has them loaded meanwhile.
struct FilterPre {
  uint64_t din, sres;
  VarDesc v;
  int size, rl, rw0;
};

// (din: the input word q, size: the size of its variable's input domain)
__device__ __forceinline__ FilterPre filter_pre_of(const DevJob& J, int q, const VarDesc& v, uint64_t din,
                                                   int size) {
  const TabDesc* T = J.tab;
  const int lane = lane_id();
  FilterPre f;
  f.v = v;
  f.din = din;
  f.size = size;
  const int rowBase = f.v.rowStart + (q - f.v.domOff) * 64;
  // these loads run before the job's input is validated: a lane past the
  // variable's last value (a stray bit) takes the word's first row, and the
  // residue is clamped to the row, so every address is inside the table
  const int used = f.v.dsize - 64 * (q - f.v.domOff);
  const bool present = lane < used && ((f.din >> lane) & 1ull);
  // unconditional loads from valid addresses (row of the word's first value
  // for absent lanes), results selected afterwards
  f.rl = present ? rowBase + lane : rowBase;
  f.rw0 = min(max(J.slot->res[f.rl], 0), (int)T->stride - 1);
  f.sres = T->S[(int64_t)f.rl * T->stride + f.rw0];
  return f;
}

__device__ __forceinline__ FilterPre filter_pre(const KArgs& a, const DevJob& J, int q) {
  const VarDesc v = J.tab->words[q].v;
  int size = 0;
  for (int k = v.domOff; k < v.domOff + v.domWords; ++k) size += __popcll(job_din(a, J, k));
  return filter_pre_of(J, q, v, job_din(a, J, q), size);
}

__device__ __forceinline__ void filter_word(const KArgs& a, const DevJob& J, int q, int noop, int lim,
                                            const CT_G int32_t* idx, unsigned long long* cnt, const FilterPre& f,
                            bool haveCtRes = false, uint64_t ctRes = 0ull, CT_G uint64_t* ctArr = nullptr,
                            CT_G int32_t* resArr = nullptr, const int* idxHead = nullptr,
                            const uint64_t* ctHead = nullptr, bool phys = false) {
  const TabDesc* T = J.tab;
  SlotDesc* slot = J.slot;
  // the slot's arrays, read once (see update_granules), or as the caller
  // read them
  struct {
    CT_G uint64_t* ct;
    CT_G int32_t* res;
  } sv{ctArr ? ctArr : slot->ct, resArr ? resArr : slot->res}, *s = &sv;
  const int lane = lane_id();
  const VarDesc v = f.v;
  const uint64_t din = f.din;
  const int size = f.size;
  uint64_t dout = din;
  if (!noop && size > 1) {  // s_sup: non-singleton variables
    const int64_t stride = T->stride;
    const int rowBase = v.rowStart + (q - v.domOff) * 64;
    const bool present = (din >> lane) & 1ull;
    const int rl = f.rl;
    const int rw0 = f.rw0;
    // the currTable word at the residue (loaded by the caller with those of
    // other words, or here)
    const uint64_t cr = haveCtRes ? ctRes : s->ct[rw0];
    const bool hit = present && (cr & f.sres) != 0ull;
    unsigned long long miss = __ballot(present && !hit);
    cnt[0] += __popcll(__ballot(present));
    cnt[1] += __popcll(miss);
    uint64_t unsup = 0;
    // phys: the caller loaded every granule of a table of at most
    // FULL_SCAN_GRAN granules into ctHead (physical order; inactive ones are
    // all zero)
    if (miss && lim > 0 && (phys || lim <= FULL_SCAN_GRAN)) {
      // few active granules: each missing value tests every active word at
      // once (FULL_SCAN_VALS values per round trip, one word per lane and
      // granule); a value with no supported word among them has no support
      int gg[FULL_SCAN_GRAN];
      uint64_t c[FULL_SCAN_GRAN];
      const int nG = T->nGran;
#pragma unroll
      for (int j = 0; j < FULL_SCAN_GRAN; ++j) {
        if (phys) {
          gg[j] = j < nG ? j : -1;
          c[j] = j < nG ? ctHead[j] : 0ull;
          continue;
        }
        // the first FULL_SCAN_GRAN entries of the index as the caller read
        // them, or from memory
        const int gv = idxHead ? idxHead[j] : idx[min(j, lim - 1)];
        gg[j] = j < lim ? gv : -1;
        const uint64_t cv = s->ct[(int64_t)gv * GW + lane];
        c[j] = j < lim ? cv : 0ull;
      }
      uint64_t todo = miss;
      while (todo) {
        int ls[FULL_SCAN_VALS];
#pragma unroll
        for (int v = 0; v < FULL_SCAN_VALS; ++v) {
          ls[v] = todo ? __ffsll((unsigned long long)todo) - 1 : -1;
          todo &= todo - 1;
        }
        uint64_t x[FULL_SCAN_VALS][FULL_SCAN_GRAN];
#pragma unroll
        for (int v = 0; v < FULL_SCAN_VALS; ++v) {
          const CT_G uint64_t* row = T->S + (int64_t)(rowBase + max(ls[v], 0)) * stride;
#pragma unroll
          for (int j = 0; j < FULL_SCAN_GRAN; ++j) x[v][j] = row[(int64_t)max(gg[j], 0) * GW + lane] & c[j];
        }
#pragma unroll
        for (int v = 0; v < FULL_SCAN_VALS; ++v) {
          if (ls[v] < 0) continue;
          cnt[2] += (unsigned long long)lim;
          bool found = false;
#pragma unroll
          for (int j = 0; j < FULL_SCAN_GRAN; ++j) {
            const unsigned long long bm = __ballot(x[v][j] != 0ull);
            if (bm) {
              if (lane == 0) s->res[rowBase + ls[v]] = gg[j] * GW + (__ffsll(bm) - 1);
              found = true;
              break;
            }
          }
          if (!found) unsup |= 1ull << ls[v];
        }
      }
    } else {
      if (miss) {
        // every missing lane first walks the words after its old residue
        // (wrapping at the end of the table): a value's supports are spread
        // over the whole table, so a nearby word usually still holds one
        const bool mine = (miss >> lane) & 1ull;
        const int r = rl;
        const int64_t words = (int64_t)T->nGran * GW;
        int64_t w = mine ? (int64_t)rw0 : 0;
        bool found = false;
  #pragma unroll 1
        for (int step = 0; step < LANE_SCAN; step += 8) {
          uint64_t x[8];
          int64_t ww[8];
  #pragma unroll
          for (int j = 0; j < 8; ++j) {
            ww[j] = w + 1 + step + j;
            if (ww[j] >= words) ww[j] -= words;
            const uint64_t y = s->ct[ww[j]] & T->S[(int64_t)r * stride + ww[j]];
            x[j] = (mine && !found) ? y : 0ull;
          }
  #pragma unroll
          for (int j = 0; j < 8; ++j) {
            if (!found && x[j]) {
              found = true;
              s->res[r] = (int)ww[j];
            }
          }
          if (!__ballot(mine && !found)) break;
        }
        cnt[2] += __popcll(__ballot(mine));
        miss = __ballot(mine && !found);
      }
      // the values still without a support scan the active granules in index
      // order together: each step loads 4 currTable granules once and tests
      // them against the rows of up to 3 values at a time; a value leaves the
      // scan at its first supported word (its new residue)
      uint64_t todo = miss;
      for (int p = 0; p < lim && todo; p += 4) {
        int gg[4];
        uint64_t c[4];
  #pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int gv = idx[min(p + j, lim - 1)];
          gg[j] = (p + j < lim) ? gv : -1;
          const uint64_t cv = s->ct[(int64_t)gv * GW + lane];
          c[j] = gg[j] >= 0 ? cv : 0ull;
        }
        cnt[2] += (unsigned long long)min(4, lim - p) * (unsigned long long)__popcll(todo);
        uint64_t t = todo;
        while (t) {
          int ls[3];
  #pragma unroll
          for (int v = 0; v < 3; ++v) {
            ls[v] = t ? __ffsll((unsigned long long)t) - 1 : -1;
            t &= t - 1;
          }
          uint64_t x[3][4];
  #pragma unroll
          for (int v = 0; v < 3; ++v) {
            const CT_G uint64_t* row = T->S + (int64_t)(rowBase + max(ls[v], 0)) * stride;
  #pragma unroll
            for (int j = 0; j < 4; ++j) {
              const uint64_t y = c[j] & row[(int64_t)max(gg[j], 0) * GW + lane];
              x[v][j] = (ls[v] >= 0 && gg[j] >= 0) ? y : 0ull;
            }
          }
  #pragma unroll
          for (int v = 0; v < 3; ++v) {
            if (ls[v] < 0) continue;
  #pragma unroll
            for (int j = 0; j < 4; ++j) {
              const unsigned long long bm = __ballot(x[v][j] != 0ull);
              if (bm) {
                if (lane == 0) s->res[rowBase + ls[v]] = gg[j] * GW + (__ffsll(bm) - 1);
                todo &= ~(1ull << ls[v]);
                break;
              }
            }
          }
        }
      }
      unsup = todo;
    }
    dout = din & ~unsup;
  }
  if (J.flags & JF_LL) {
    if (lane < 2) ll_put(J.ll + 2 + 2 * q + lane, eng_slot((uint32_t)(lane ? dout >> 32 : dout), (uint32_t)J.seq));
  } else if (lane == 0) {
    J.dom_out[q] = dout;
  }
  if (lane == 0) slot->lastDom[q] = dout;
}

__device__ __forceinline__ void filter_word(const KArgs& a, const DevJob& J, int q, int noop, int lim,
                                            const CT_G int32_t* idx, unsigned long long* cnt) {
  filter_word(a, J, q, noop, lim, idx, cnt, filter_pre(a, J, q));
}

__device__ void add_filter_stats(SlotDesc* s, const unsigned long long* cnt) {
  if (lane_id() == 0 && (cnt[0] | cnt[1] | cnt[2])) {
    atomicAdd(&s->stats[S_RES_CHECK], cnt[0]);
    atomicAdd(&s->stats[S_RES_MISS], cnt[1]);
    atomicAdd(&s->stats[S_SCAN], cnt[2]);
  }
}

// ---------------------------------------------------------------------------
// split mode: a job's update item (tables of at most WAVES x NGW granules:
// larger ones run staged)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void do_update(const KArgs& a, const DevJob& J, Shared& sh) {
  SlotDesc* s = J.slot;
  if (J.nPop > 0) {
    if (!block_wait(a, &s->prepDone, 1, sh)) return;
  }
  // the whole update runs in this workgroup, as in solo mode: pushes in the
  // prologue (unless the prep item made them), granule list, flags and trail
  // count in LDS, no global round trip between the update and the partition
  // (one call site each of the prologue and the update: a second would take
  // the kernel arguments' address)
  if (threadIdx.x == 0) sh.trailCount = 0;
  prologue(a, J, sh, J.nPop == 0 && J.nPush > 0);
  if (J.tab->nGran <= WAVES) {
    // at most one granule per wave: twice the rows in flight instead
    update_granules<1, 2 * ROW_UNROLL>(a, J, sh, wave_id(), &sh.trailCount, &sh.sp);
  } else {
    update_granules<NGW>(a, J, sh, wave_id() * NGW, &sh.trailCount, &sh.sp);
  }
  lds_barrier();
  if (J.nPop > 0 && threadIdx.x == 0) s->prepDone = 0;  // the prep item also did the pushes
  const int st = finalize_update(J, sh, sh.trailCount);
  if (threadIdx.x == 0) {
    if (st != ST_OK) publish_status(J, st);
    // finalize_update ends with a full barrier: the block's writes are
    // ordered before this release; a currTable copy in host memory is
    // made visible before the filter publishes the status
    if (J.ct_out) status_fence(J);
    // consumed (and reset) by the job's last filter item, or a flagged
    // job's number
    st_release(&s->updDone, (J.flags & JF_LL) ? ll_gen(J.seq) : 1);
  }
}

// split mode: one filter item (one domain word per wave)
__device__ __forceinline__ void do_filter(const KArgs& a, const DevJob& J, int chunk, Shared& sh) {
  SlotDesc* s = J.slot;
  const int q = chunk * WAVES + wave_id();
  const int qc = min(q, J.tab->D - 1);
  // in flight while the update runs: what filterDomains needs of the input
  // (filter_pre) and the slot's array addresses, which never change
  CT_G uint64_t* const sct = s->ct;
  CT_G int32_t* const sres = s->res;
  CT_G int32_t* const idx0 = s->idx[0];
  CT_G int32_t* const idx1 = s->idx[1];
  const FilterPre pre = filter_pre(a, J, qc);
  if (threadIdx.x < 3) sh.fcnt[threadIdx.x] = 0ull;
  const bool ll = J.flags & JF_LL;
  if (!block_wait(a, &s->updDone, ll ? ll_gen(J.seq) : 1, sh)) return;
  // one round trip: the job's state after the update, per value the
  // currTable word at its residue, and the head of both index buffers (the
  // one in use is known with the state)
  const int jobStatus = s->status, noop = s->noop, lim = s->limit, cur = s->cur;
  const uint64_t cr = sct[pre.rw0];
  const int nG = J.tab->nGran;
  int h0[FULL_SCAN_GRAN], h1[FULL_SCAN_GRAN], head[FULL_SCAN_GRAN];
#pragma unroll
  for (int j = 0; j < FULL_SCAN_GRAN; ++j) {
    h0[j] = idx0[min(j, nG - 1)];
    h1[j] = idx1[min(j, nG - 1)];
  }
#pragma unroll
  for (int j = 0; j < FULL_SCAN_GRAN; ++j) head[j] = cur ? h1[j] : h0[j];
  // a table of at most FULL_SCAN_GRAN granules: all of currTable, in the
  // same round trip
  uint64_t cth[FULL_SCAN_GRAN];
#pragma unroll
  for (int j = 0; j < FULL_SCAN_GRAN; ++j) cth[j] = sct[(int64_t)min(j, nG - 1) * GW + lane_id()];
  unsigned long long cnt[3] = {0, 0, 0};
  if (q < J.tab->D && jobStatus == ST_OK)
    filter_word(a, J, q, noop, lim, cur ? idx1 : idx0, cnt, pre, true, cr, sct, sres, head, cth,
                nG <= FULL_SCAN_GRAN);
  // the item's counts, summed in LDS: one set of counter atomics per item
  if (lane_id() == 0 && (cnt[0] | cnt[1] | cnt[2]))
    for (int k = 0; k < 3; ++k) atomicAdd(&sh.fcnt[k], cnt[k]);
  // the last filter item of the job reports OK
  __syncthreads();
  if (threadIdx.x == 0) add_filter_stats(s, sh.fcnt);
  if (ll) return;  // the host counts the domain words itself
  if (threadIdx.x == 0) {
    status_fence(J);  // no other item reads this one's outputs
    const int prev = atomicAdd(&s->filtCount, 1);
    if (prev == J.nFilt - 1) {
      s->filtCount = 0;
      s->updDone = 0;
      if (jobStatus == ST_OK) publish_status(J, ST_OK);
    }
  }
}

// ---------------------------------------------------------------------------
// filterDomains of a negative table (whole job in one workgroup).  currTable
// holds the forbidden tuples whose values are all in the input domains; value
// a of x_i has an allowed tuple iff fewer than prod_{k != i} |dom(x_k)|
// (sh.dcnt[i], capped above the tuple count) of them have x_i = a.
// sh.rows[0 .. total) lists the values to count (domain word << 6 | bit); a
// wave counts NEG_VALS of them, a granule's words of each in one coalesced
// load, and clears those without an allowed tuple from sh.dout.  Many values
// over few granules take neg_count_word instead (neg_by_lane).
// ---------------------------------------------------------------------------
constexpr int NEG_VALS = 4, NEG_GRAN = 4;  // values per wave, granules in flight
__device__ void neg_count(const DevJob& J, int total, int lim, const CT_G int32_t* idx, Shared& sh) {
  const TabDesc* T = J.tab;
  const CT_G uint64_t* ct = J.slot->ct;
  const CT_G uint64_t* S = T->S;
  const int64_t stride = T->stride;
  const int lane = lane_id();
  for (int k0 = wave_id() * NEG_VALS; k0 < total; k0 += WAVES * NEG_VALS) {
    uint32_t val[NEG_VALS];
    int row[NEG_VALS], var[NEG_VALS], cnt[NEG_VALS];
#pragma unroll
    for (int k = 0; k < NEG_VALS; ++k) {
      val[k] = __builtin_amdgcn_readfirstlane(sh.rows[min(k0 + k, total - 1)]);
      const int q = (int)(val[k] >> 6);
      var[k] = T->wordVar[q];
      const VarDesc v = T->vars[var[k]];
      row[k] = v.rowStart + (q - v.domOff) * 64 + (int)(val[k] & 63u);
      cnt[k] = 0;
    }
    for (int p0 = 0; p0 < lim; p0 += NEG_GRAN) {
      uint64_t c[NEG_GRAN], x[NEG_VALS][NEG_GRAN];
#pragma unroll
      for (int j = 0; j < NEG_GRAN; ++j) {
        const int64_t w = (int64_t)idx[min(p0 + j, lim - 1)] * GW + lane;
        const uint64_t y = ct[w];
        c[j] = p0 + j < lim ? y : 0ull;
#pragma unroll
        for (int k = 0; k < NEG_VALS; ++k) x[k][j] = S[(int64_t)row[k] * stride + w];
      }
#pragma unroll
      for (int k = 0; k < NEG_VALS; ++k)
#pragma unroll
        for (int j = 0; j < NEG_GRAN; ++j) cnt[k] += __popcll(c[j] & x[k][j]);
    }
#pragma unroll
    for (int k = 0; k < NEG_VALS; ++k) {
      const int sum = wave_sum(cnt[k]);
      if (lane == 0 && k0 + k < total && sum == sh.dcnt[var[k]])
        atomicAnd((unsigned long long*)&sh.dout[val[k] >> 6], ~(1ull << (val[k] & 63u)));
    }
  }
}

// The same for the values of domain word q, one to a lane, which walks its row
// (64 rows a load: slow per granule, but a wave has 64 values in hand).
__device__ void neg_count_word(const DevJob& J, int q, int lim, const CT_G int32_t* idx, Shared& sh) {
  const TabDesc* T = J.tab;
  const CT_G uint64_t* ct = J.slot->ct;
  const int i = T->wordVar[q];
  const VarDesc v = T->vars[i];
  const uint64_t din = sh.din[q];
  const int prod = sh.dcnt[i];
  if (din == 0ull || prod > (int64_t)lim * GW * 64) return;
  const int lane = lane_id();
  const bool present = (din >> lane) & 1ull;
  const int row = v.rowStart + (q - v.domOff) * 64 + (present ? lane : 0);
  const CT_G uint64_t* srow = T->S + (int64_t)row * T->stride;
  int cnt = 0;
  for (int p = 0; p < lim; ++p) {
    const int64_t base = (int64_t)idx[p] * GW;
#pragma unroll 8
    for (int k = 0; k < GW; ++k) cnt += __popcll(ct[base + k] & srow[base + k]);
  }
  const uint64_t gone = __ballot(present && cnt == prod);
  if (lane == 0) sh.dout[q] = din & ~gone;
}

// Which of the two counts `values` values in `words` domain words over `lim`
// granules: by their round trips, those of a lane's walk counted four times
// (us a call, by lane / by wave: 305 values, 1 granule 20 / 27; 120, 1: 21 / 25;
// 200, 2: 26 / 28; 4,005, 5: 49 / 66; 90, 5: 25 / 23; 45, 3: 27 / 22; 400, 8:
// 54 / 42; 100, 49: 217 / 76).
__device__ __forceinline__ bool neg_by_lane(int values, int words, int lim) {
  const int byWave = (values + WAVES * NEG_VALS - 1) / (WAVES * NEG_VALS) * ((lim + NEG_GRAN - 1) / NEG_GRAN);
  return byWave >= 4 * ((words + WAVES - 1) / WAVES) * lim;
}

// A negative table's filterDomains in one workgroup, after updateTable and
// its partition (st: the job status so far): per-variable products,
// every variable filtered into sh.dout, failure iff a domain empties.  On
// success the removed values' rows are listed as one incremental segment
// (in word order) for a second update pass that takes their tuples out of
// currTable.  Returns the status; *rows2 receives the listed rows.
__device__ int neg_filter(const DevJob& J, Shared& sh, int st, int* rows2) {
  SlotDesc* s = J.slot;
  const TabDesc* T = J.tab;
  const int n = T->n, D = T->D;
  *rows2 = 0;
  if (st != ST_OK) return st;
  const int64_t cap = (int64_t)T->nGran * GW * 64 + 1;
  for (int i = threadIdx.x; i < n; i += BLOCK) {
    int64_t prod = 1;
    for (int k = 0; k < n; ++k) {
      if (k == i) continue;
      prod = min(prod * (int64_t)sh.size[k], cap);
    }
    sh.dcnt[i] = (int32_t)prod;
  }
  if (threadIdx.x == 0) sh.bad_sub = 0;
  __syncthreads();
  const int per = (D + BLOCK - 1) / BLOCK;
  const int b = min((int)threadIdx.x * per, D), e = min(b + per, D);
  {
    // the values whose count can reach their product
    const int lim = s->limit;
    const int64_t most = (int64_t)lim * GW * 64;
    int cnt = 0;
    for (int q = b; q < e; ++q) {
      const uint64_t din = sh.din[q];
      sh.dout[q] = din;
      if (!sh.noop && sh.dcnt[T->wordVar[q]] <= most) cnt += (din ? 1 << 16 : 0) + __popcll(din);
    }
    // (words << 16 | values: at most 1,024 and 8,192)
    int total = 0;
    int off = block_scan_excl(cnt, &total, sh) & 0xffff;
    const int words = total >> 16, values = total & 0xffff;
    if (neg_by_lane(values, words, lim)) {
      if (values)
        for (int q = wave_id(); q < D; q += WAVES) neg_count_word(J, q, lim, s->idx[s->cur], sh);
    } else {
      for (int q = b; q < e; ++q) {
        uint64_t bits = sh.noop || sh.dcnt[T->wordVar[q]] > most ? 0ull : sh.din[q];
        while (bits) {
          const int k = __ffsll((unsigned long long)bits) - 1;
          bits &= bits - 1;
          sh.rows[off++] = (uint32_t)(q << 6 | k);
        }
      }
      __syncthreads();
      neg_count(J, values, lim, s->idx[s->cur], sh);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += BLOCK) {
    const VarDesc v = T->vars[i];
    uint64_t any = 0ull;
    for (int k = 0; k < v.domWords; ++k) any |= sh.dout[v.domOff + k];
    if (!any) sh.bad_sub = 1;
  }
  __syncthreads();
  if (sh.bad_sub) {
    if (threadIdx.x == 0) {
      s->failed = 1;
      s->status = ST_FAIL;
    }
    return ST_FAIL;
  }
  if (sh.noop) return ST_OK;
  int cnt = 0;
  for (int q = b; q < e; ++q) cnt += __popcll(sh.din[q] & ~sh.dout[q]);
  int total = 0;
  int off = block_scan_excl(cnt, &total, sh);
  for (int q = b; q < e; ++q) {
    const VarDesc v = T->vars[T->wordVar[q]];
    const int base = v.rowStart + (q - v.domOff) * 64;
    uint64_t bits = sh.din[q] & ~sh.dout[q];
    while (bits) {
      const int k = __ffsll((unsigned long long)bits) - 1;
      bits &= bits - 1;
      sh.rows[off++] = (uint32_t)(base + k);
    }
  }
  if (total > 0) {
    // the second pass reads the slot's own (updated) currTable and granule
    // list; its trail entries follow the first pass's
    if (threadIdx.x == 0) {
      sh.nseg = 1;
      sh.segEnd[0] = total;
      sh.segInc[0] = 1;
      sh.nrows = total;
      sh.status = ST_OK;
      sh.limit = s->limit;
      sh.trailTop = s->trailTop;
      sh.trailCount = 0;
    }
    __syncthreads();
    const CT_G int32_t* idx = s->idx[s->cur];
    // (all of it: the partition copies the inactive part too)
    for (int p = threadIdx.x; p < T->nGran; p += BLOCK) sh.gidx[p] = (uint16_t)idx[p];
    __syncthreads();
  }
  *rows2 = total;
  return ST_OK;
}

// ---------------------------------------------------------------------------
// solo mode: the whole job in one workgroup -- pops/pushes, prologue, all
// granules, partition, filter -- with no hand-off between workgroups.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void do_solo(const KArgs& a, const DevJob& J0, Shared& sh) {
  // a negative table filters before its update is complete (its second
  // pass takes the removed values' tuples out) and writes currTable out at
  // the end of the call
  const bool negative = J0.tab->kind != 0;
  DevJob J = J0;
  if (negative) J.ct_out = nullptr;
  SlotDesc* s = J.slot;
  const bool pushHere = J.nPop == 0 && J.nPush > 0;
  if (!pushHere) apply_pops_pushes(J, sh);
  // (the job's granule list is read once, in the prologue: each update step
  // is then a single round of independent loads)
  prologue(a, J, sh, pushHere);
  if (threadIdx.x == 0) sh.trailCount = 0;
  const int nGran = J.tab->nGran;
  int span = sh.status == ST_OK ? nGran : 0;
  __syncthreads();
  int st = ST_OK;
  for (int pass = 0;; ++pass) {
    for (int c = 0; c < span; c += WAVES * NGS) {
      update_granules<NGS>(a, J, sh, c + wave_id() * NGS, &sh.trailCount);
    }
    __syncthreads();
    st = finalize_update(J, sh, sh.trailCount, pass == 0);
    if (!negative || pass == 1) break;
    int rows2 = 0;
    st = neg_filter(J, sh, st, &rows2);
    if (rows2 == 0) break;
    span = sh.limit;
    J.flags &= ~(JF_FROM_ROOT | JF_ROOT | JF_SCRATCH);
  }
  if (negative) {
    __syncthreads();
    const TabDesc* T = J.tab;
    if (st == ST_OK) {
      for (int q = threadIdx.x; q < T->D; q += BLOCK) {
        const uint64_t dout = sh.dout[q];
        if (J0.flags & JF_LL) {
          ll_put(J0.ll + 2 + 2 * q, eng_slot((uint32_t)dout, (uint32_t)J0.seq));
          ll_put(J0.ll + 3 + 2 * q, eng_slot((uint32_t)(dout >> 32), (uint32_t)J0.seq));
        } else {
          J0.dom_out[q] = dout;
        }
        s->lastDom[q] = dout;
      }
    }
    if (J0.ct_out && (st == ST_OK || st == ST_FAIL))
      for (int64_t w = threadIdx.x; w < T->W; w += BLOCK) J0.ct_out[w] = st == ST_OK ? s->ct[w] : 0ull;
  } else if (st == ST_OK) {
    unsigned long long cnt[3] = {0, 0, 0};
    const int lim = s->limit;
    const CT_G int32_t* idx = s->idx[s->cur];
    const int noop = sh.noop;
    for (int q = wave_id(); q < J.tab->D; q += WAVES) filter_word(a, J, q, noop, lim, idx, cnt);
    add_filter_stats(s, cnt);
  }
  __syncthreads();
  // (a flagged call's success is its domain words)
  if (threadIdx.x == 0 && !(st == ST_OK && (J.flags & JF_LL))) {
    if (!(J.flags & JF_LL)) status_fence(J);
    publish_status(J, st);
  }
}

// Device-clock duration of a launch: first workgroup start to last end.
__device__ void clock_begin(const KArgs& a) {
  if (a.clock && threadIdx.x == 0) atomicMin(&a.clock[0], wall_clock64());
}

__device__ void clock_end(const KArgs& a) {
  if (!a.clock || threadIdx.x != 0) return;
  const unsigned long long now = wall_clock64();
  atomicMax(&a.clock[1], now);
  __threadfence();
  const unsigned long long prev = atomicAdd(&a.clock[2], 1ull);
  if (prev == gridDim.x - 1) {
    const unsigned long long t0 = atomicOr(&a.clock[0], 0ull);
    const unsigned long long t1 = atomicOr(&a.clock[1], 0ull);
    atomicAdd(&a.clock[3], t1 > t0 ? t1 - t0 : 0ull);
    atomicAdd(&a.clock[4], 1ull);
    a.clock[0] = ~0ull;
    a.clock[1] = 0ull;
    a.clock[2] = 0ull;
    __threadfence();
  }
}

// Either one job (the kernel argument): a workgroup per item -- prep, update
// or solo, filters -- all resident at once, so every wait between them ends;
// or an array of jobs that each run in one workgroup.
__global__ void __launch_bounds__(BLOCK) propagate_kernel(KArgs a) {
  __shared__ Shared sh;
  clock_begin(a);
  if (a.jobs || (a.job.flags & JF_SOLO)) {
    for (int j = blockIdx.x; j < a.nJobs; j += gridDim.x) {
      const DevJob J = job_of(a, j);
      if (J.active && !*J.active) continue;  // a clean job of a model round
      do_solo(a, J, sh);
      __syncthreads();
    }
  } else {
    const int item = blockIdx.x;
    const DevJob J = job_of(a, 0);
    if (item < a.nPrep) do_prep(a, J, sh);
    else if (item < a.nPrep + a.nUpd) do_update(a, J, sh);
    else do_filter(a, J, item - a.nPrep - a.nUpd, sh);
  }
  __syncthreads();
  clock_end(a);
}

// ---------------------------------------------------------------------------
// Resident split schedule of slot 0, for synchronous calls on tables whose
// update is one item: the split schedule's update item and filter items as
// one persistent launch that takes calls from the resident engine's mailbox
// (pinned host memory), so a call pays no kernel launch.  Workgroup 0 polls
// the mailbox, rings the doorbell ctl[SE_CALL] once a whole call is there,
// runs the call's pops, pushes, prologue, updateTable and partition, writes
// the status slot and hands over to the filters with the call's generation in
// updDone.  Filter workgroup c (filter item c) waits for the doorbell, reads
// its domain words from the mailbox itself, so its residue loads are in
// flight during the update; after the hand-over it filters and answers with
// flagged domain slots, then counts the call in ctl[SE_DONE] behind a
// release: workgroup 0 waits for that count before the next call reads the
// slot's domains.  The other workgroups of XCD 0 stay empty and workgroup 0
// takes no acquire between calls (JF_COHLAST), so its L2 keeps the table
// and the slot.  Workgroup 0 alone stops (a stop command, or no call for
// idleTicks) and sets ctl[SE_STOP], the word every wait of the launch
// watches, so the filters end too.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t mb_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Workgroup 0's wave 0: waits for call `want` in the mailbox, copies its
// input words into ka.inl and its header into sh.se*; sh.seOp is 0 when no
// call came within idleTicks.  It polls the op slot alone (written last by
// the host: the lines the host is still writing are not read meanwhile),
// two loads in flight, then reads the whole command, U chunks of 64 slots
// per round trip.  Every lane loads (lanes past the command re-read its
// last slot): a load under a lane condition would be waited for before the
// test after it.
__device__ __forceinline__ void se_take_call(const EngDesc& E, KArgs& ka, Shared& sh, uint32_t want, int D) {
  constexpr int U = 8;
  const int l = lane_id();
  const uint64_t* slots = E.cmd->slot;
  const int nS = EC_DOM + 2 * D;
  uint32_t* in32 = (uint32_t*)ka.inl;
  const unsigned long long t0 = wall_clock64();
  bool seen = false;
  {
    uint64_t p0 = mb_load(slots + EC_OP);
    for (;;) {
      const uint64_t p1 = mb_load(slots + EC_OP);
      if (__builtin_amdgcn_readfirstlane((uint32_t)p0) == want) {
        seen = true;
        break;
      }
      p0 = mb_load(slots + EC_OP);
      if (__builtin_amdgcn_readfirstlane((uint32_t)p1) == want) {
        seen = true;
        break;
      }
      if ((long long)(wall_clock64() - t0) > E.idleTicks) break;
    }
  }
  uint32_t hv = 0;
  for (int c0 = 0; seen && c0 < nS; c0 += U * WAVE) {
    for (;;) {  // written before the op slot: normally present at once
      uint64_t w[U];
      bool ok = true;
#pragma unroll
      for (int u = 0; u < U; ++u) w[u] = mb_load(slots + min(c0 + u * WAVE + l, nS - 1));
#pragma unroll
      for (int u = 0; u < U; ++u) ok = ok && (uint32_t)w[u] == want;
      if (__all(ok)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = c0 + u * WAVE + l;
          if (i >= EC_DOM && i < nS) in32[i - EC_DOM] = (uint32_t)(w[u] >> 32);
        }
        if (c0 == 0) hv = (uint32_t)(w[0] >> 32);
        break;
      }
      if ((long long)(wall_clock64() - t0) > E.idleTicks) {
        seen = false;
        break;
      }
    }
  }
  const int h0 = __shfl((int)hv, EC_OP), h1 = __shfl((int)hv, EC_NPOP), h2 = __shfl((int)hv, EC_NPUSH);
  const int h3 = __shfl((int)hv, EC_SERIAL), h4 = __shfl((int)hv, EC_DEPTH);
  if (l == 0) {
    sh.seOp = seen ? h0 : 0;
    sh.seNPop = h1;
    sh.seNPush = h2;
    sh.seSerial = h3;
    sh.seDepth = h4;
    // the filters' doorbell: the whole call is in the mailbox (a release: a
    // relaxed store can wait in this XCD's L2 until the next release, and
    // polls of one word at system scope from every filter workgroup queue
    // up at the memory)
    if (seen && h0 == ENG_OP_PROPAGATE) st_release(&E.ctl[SE_CALL], (int32_t)want);
  }
}

// A filter workgroup's input of call `want`.  Wave 0 waits for the doorbell
// (device memory: the host's lines are read by workgroup 0 alone) while the
// others wait at the barrier; then each wave reads the input slots of its
// variable's words (at most SE_MAX_VAR_WORDS, one slot per lane; the lanes
// past them re-read the last one, so a wave reads one or two lines of host
// memory) from the mailbox.  Returns false once the launch stops; else the
// word q and the size of its variable's input.
__device__ __forceinline__ bool se_filter_input(const EngDesc& E, Shared& sh, const VarDesc& v, int q,
                                                uint32_t want, uint64_t* din, int* size) {
  const int l = lane_id();
  const unsigned long long t0 = wall_clock64();
  if (wave_id() == 0) {
    int go = 0;
    for (;;) {
      if ((uint32_t)ld_relaxed(&E.ctl[SE_CALL]) == want) {
        go = 1;
        break;
      }
      // the launch has stopped, or (a bound that is never reached while
      // workgroup 0 runs) nothing has come for far longer than it waits
      if (ld_relaxed(&E.ctl[SE_STOP]) != 0 || (long long)(wall_clock64() - t0) > 8 * E.idleTicks) break;
      __builtin_amdgcn_s_sleep(1);
    }
    if (l == 0) sh.ok = go;
  }
  lds_barrier();
  if (!sh.ok) return false;
  const int nW = 2 * v.domWords;
  const uint64_t* mine = E.cmd->slot + EC_DOM + 2 * v.domOff + min(l, nW - 1);
  uint64_t x;
  for (;;) {  // all there once workgroup 0 rang
    x = mb_load(mine);
    if (__all((uint32_t)x == want)) break;
    if (ld_relaxed(&E.ctl[SE_STOP]) != 0 || (long long)(wall_clock64() - t0) > 8 * E.idleTicks) return false;
  }
  const uint32_t p = (uint32_t)(x >> 32);
  *size = __builtin_amdgcn_readlane(wave_scan_incl(l < nW ? __popc(p) : 0), WAVE - 1);
  const int k = 2 * (q - v.domOff);
  const uint32_t lo = (uint32_t)__shfl((int)p, k), hi = (uint32_t)__shfl((int)p, k + 1);
  *din = ((uint64_t)hi << 32) | lo;
  return true;
}

// Workgroup 0 waits until the filters have counted `want` calls (bounded:
// false on a device error or when the wait runs out).
__device__ __forceinline__ bool se_wait_done(const EngDesc& E, int want, Shared& sh) {
  if (threadIdx.x == 0) {
    int ok = 1;
    for (uint32_t it = 0;; ++it) {
      if (ld_relaxed(&E.ctl[SE_DONE]) == want) break;
      if (ld_relaxed(&E.ctl[SE_STOP]) > 0) { ok = 0; break; }
      if (it > SPIN_LIMIT) {
        atomicExch(&E.ctl[SE_STOP], 1);
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    sh.ok = ok;
  }
  lds_barrier();
  const int ok = sh.ok;
  lds_barrier();
  return ok != 0;
}

// One call's update on workgroup 0: pops and pushes, prologue, updateTable
// and partition, then the hand-over to the filters.  Returns the status.
__device__ __forceinline__ int se_update(const KArgs& a, const DevJob& J, Shared& sh) {
  SlotDesc* s = J.slot;
  if (J.nPop > 0) apply_pops_pushes(J, sh);  // the pops, then the pushes
  if (threadIdx.x == 0) sh.trailCount = 0;
  prologue(a, J, sh, J.nPop == 0 && J.nPush > 0);
  if (J.tab->nGran <= WAVES)  // at most one granule per wave: twice the rows in flight
    update_granules<1, 2 * ROW_UNROLL>(a, J, sh, wave_id(), &sh.trailCount, &sh.sp);
  else
    update_granules<NGW>(a, J, sh, wave_id() * NGW, &sh.trailCount, &sh.sp);
  lds_barrier();
  const int st = finalize_update(J, sh, sh.trailCount);
  // finalize_update ends with a full barrier: the block's writes are ordered
  // before this release
  if (threadIdx.x == 0) st_release(&s->updDone, ll_gen(J.seq));
  return st;
}

__global__ void __launch_bounds__(BLOCK) split_engine_kernel(EngDesc E) {
  __shared__ Shared sh;
  __shared__ KArgs ka;  // the calls' view of the launched schedule's arguments
  const CT_G TabDesc* T = E.tab;
  CT_G SlotDesc* s = E.slot;
  const int D = T->D;
  if (threadIdx.x == 0) {
    ka.jobs = nullptr;
    ka.nJobs = 1;
    ka.queue = E.ctl;  // queue[3] = ctl[SE_STOP]: raise_error and block_wait use it
    ka.hostErr = nullptr;
    ka.clock = nullptr;
  }
  __syncthreads();
  DevJob J = {};
  J.tab = T;
  J.slot = s;
  J.flags = JF_PROPAGATE | JF_LL | JF_INLINE_DOM | JF_COHLAST;
  J.nUpd = 1;
  J.nFilt = E.nFilt;
  J.ll = E.res->slot + ER_DOM - 2;  // domain word q in slots ER_DOM + 2q, + 1
  uint32_t last = (uint32_t)E.startSeq;
  if (blockIdx.x == 0) {
    const unsigned long long tLife = wall_clock64();
    for (int served = 0;; ++served) {
      const uint32_t want = last + 1;
      if (threadIdx.x < WAVE) se_take_call(E, ka, sh, want, D);
      lds_barrier();
      if (sh.seOp != ENG_OP_PROPAGATE) break;
      // the filters' writes of the previous call (the slot's domains) first;
      // no acquire (it would invalidate this XCD's L2, which holds the table
      // and the slot between calls): those domains are read at device scope
      if (served > 0 && !se_wait_done(E, served * E.nFilt, sh)) {
        if (threadIdx.x == 0) ll_put(&E.res->slot[ER_STATUS], eng_slot((uint32_t)ST_DEVICE, want));
        last = want;
        break;
      }
      const unsigned long long tStart = wall_clock64();
      J.nPop = sh.seNPop;
      J.nPush = sh.seNPush;
      J.serialBase = sh.seSerial;
      J.depthAfter = sh.seDepth;
      J.seq = (int32_t)want;
      int st = se_update(ka, J, sh);
      if (threadIdx.x == 0) {
        if (ld_relaxed(&E.ctl[SE_STOP]) > 0) st = ST_DEVICE;
        const unsigned long long ticks = wall_clock64() - tStart;
        ll_put(&E.res->slot[ER_TICKS], eng_slot((uint32_t)min(ticks, 0xffffffffull), want));
        ll_put(&E.res->slot[ER_STATUS], eng_slot((uint32_t)st, want));
      }
      last = want;
      lds_barrier();
    }
    if (threadIdx.x == 0) {
      atomicCAS(&E.ctl[SE_STOP], 0, -1);
      E.res->exitSeq = (int32_t)last;
      E.res->lifeTicks = wall_clock64() - tLife;
      __threadfence_system();
      __hip_atomic_store(&E.res->alive, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  // filter workgroup c: the workgroups of XCD 0 (every eighth, in the
  // dispatch order's round robin) are left to workgroup 0 and end here, so
  // the filters' acquires never invalidate its L2
  if (blockIdx.x % 8 == 0) return;
  const int c = (int)blockIdx.x - 1 - (int)blockIdx.x / 8;
  if (c >= E.nFilt) return;
  const int q = c * WAVES + wave_id();
  const int qc = min(q, D - 1);
  const VarDesc v = T->words[qc].v;
  CT_G uint64_t* const sct = s->ct;
  CT_G int32_t* const sres = s->res;
  CT_G int32_t* const idx0 = s->idx[0];
  CT_G int32_t* const idx1 = s->idx[1];
  const int nG = T->nGran;
  for (;;) {
    const uint32_t want = last + 1;
    uint64_t din = 0;
    int size = 0;
    const bool go = se_filter_input(E, sh, v, qc, want, &din, &size);
    if (lane_id() == 0) sh.wsum[wave_id()] = go ? 1 : 0;
    if (threadIdx.x < 3) sh.fcnt[threadIdx.x] = 0ull;
    lds_barrier();
    bool all = true;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) all = all && sh.wsum[w] != 0;
    if (!all) break;
    J.seq = (int32_t)want;
    const FilterPre pre = filter_pre_of(J, qc, v, din, size);
    if (!block_wait(ka, &s->updDone, ll_gen(J.seq), sh)) break;
    // as do_filter: the state after the update, the currTable word at each
    // value's residue and the head of both index buffers in one round trip
    const int jobStatus = s->status, noop = s->noop, lim = s->limit, cur = s->cur;
    const uint64_t cr = sct[pre.rw0];
    int h0[FULL_SCAN_GRAN], h1[FULL_SCAN_GRAN], head[FULL_SCAN_GRAN];
#pragma unroll
    for (int j = 0; j < FULL_SCAN_GRAN; ++j) {
      h0[j] = idx0[min(j, nG - 1)];
      h1[j] = idx1[min(j, nG - 1)];
    }
#pragma unroll
    for (int j = 0; j < FULL_SCAN_GRAN; ++j) head[j] = cur ? h1[j] : h0[j];
    uint64_t cth[FULL_SCAN_GRAN];
#pragma unroll
    for (int j = 0; j < FULL_SCAN_GRAN; ++j) cth[j] = sct[(int64_t)min(j, nG - 1) * GW + lane_id()];
    unsigned long long cnt[3] = {0, 0, 0};
    if (q < D && jobStatus == ST_OK)
      filter_word(ka, J, q, noop, lim, cur ? idx1 : idx0, cnt, pre, true, cr, sct, sres, head, cth,
                  nG <= FULL_SCAN_GRAN);
    if (lane_id() == 0 && (cnt[0] | cnt[1] | cnt[2]))
      for (int k = 0; k < 3; ++k) atomicAdd(&sh.fcnt[k], cnt[k]);
    // every wave's stores of the slot's domains complete at the barrier; the
    // release makes them visible to workgroup 0 before the call is counted
    __syncthreads();
    if (threadIdx.x == 0) {
      add_filter_stats(s, sh.fcnt);
      __threadfence();
      atomicAdd(&E.ctl[SE_DONE], 1);
    }
    last = want;
  }
}

// ---------------------------------------------------------------------------
// support bitset builder: one wave per 64 tuples (one word column); for each
// column of the table every distinct row among the wave's lanes is written
// once with the ballot of the lanes holding that value (no atomics, each
// (row, word) has exactly one writer).  S must be zeroed beforehand.  A tuple
// all of whose values are in dom0 is valid at the root: the ballot of those is
// the root's currTable word.
// The cells come from pinned host memory: a wave reads its 64 tuples in
// coalesced 16-byte loads, once, into LDS (BUILD_COLS columns at a time), and
// takes the columns from there.
// ---------------------------------------------------------------------------
constexpr int BUILD_COLS = 64;
__global__ void __launch_bounds__(BLOCK) build_supports_kernel(BuildArgs B) {
  extern __shared__ int32_t cells[];
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(wave_id());
  const int64_t w = B.w0 + (int64_t)blockIdx.x * (blockDim.x / WAVE) + wv;
  if (w >= B.w0 + B.nw) return;
  const int n = B.n;
  const CT_G int32_t* src = (const CT_G int32_t*)B.tuples + (w - B.w0) * 64 * n;
  const int cnt = (int)min((int64_t)64, B.t - w * 64);
  const int cols = min(n, BUILD_COLS), pitch = cols | 1;
  int32_t* my = cells + wv * 64 * pitch;
  bool valid = lane < cnt && !B.empty, starred = false;
  for (int c0 = 0; c0 < n; c0 += BUILD_COLS) {
    const int tc = min(n - c0, BUILD_COLS);
    if (tc == n) {
      // (16-byte loads: the word's cells begin at a multiple of 256 bytes, and
      // the buffer is longer than the last one reads)
      const int total = cnt * n;
      constexpr int BU = 4;  // loads in flight
      for (int b0 = 0; b0 < total; b0 += BU * WAVE * 4) {
        int4 x[BU];
#pragma unroll
        for (int u = 0; u < BU; ++u) {
          const int e0 = b0 + u * WAVE * 4 + lane * 4;
          x[u] = *(const CT_G int4*)(src + (e0 < total ? e0 : 0));
        }
#pragma unroll
        for (int u = 0; u < BU; ++u) {
          const int v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t e = (uint32_t)(b0 + u * WAVE * 4 + lane * 4 + k), j = e / (uint32_t)n;
            if ((int)e < total) my[j * pitch + (e - j * n)] = v[k];
          }
        }
      }
    } else {
#pragma unroll 8
      for (int j = 0; j < cnt; ++j)
        if (lane < tc) my[j * pitch + lane] = src[j * n + c0 + lane];
    }
    // the wave's own LDS traffic is in order: nothing but the compiler to stop
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int i = 0; i < tc; ++i) {
      const VarDesc v = B.vars[c0 + i];
      int r = -1;
      bool star = false;
      if (lane < cnt) {
        const int32_t raw = my[lane * pitch + i];
        star = raw == STAR_CELL;
        const int64_t val = (int64_t)raw - B.lo[c0 + i];
        if (!star) {
          const bool in = val >= 0 && val < v.dsize;
          if (in) r = v.rowStart + (int)val;
          const int a = in ? (int)val : 0;
          valid = valid && in && ((B.dom0[v.domOff + (a >> 6)] >> (a & 63)) & 1ull);
        }
      }
      // a star cell (short table) is in every row of its column: each row
      // word is the ballot of its lanes or'ed with the star lanes, written once
      const unsigned long long starMask = __ballot(star);
      if (starMask) {
        starred = true;
        for (int k = 0; k < v.dsize; ++k) {
          const unsigned long long m = __ballot(r == v.rowStart + k) | starMask;
          if (lane == 0) B.S[(int64_t)(v.rowStart + k) * B.stride + w] = m;
        }
        continue;
      }
      bool pending = r >= 0;
      for (;;) {
        const unsigned long long act = __ballot(pending);
        if (!act) break;
        const int leader = __ffsll(act) - 1;
        const int rl = __shfl(r, leader);
        const unsigned long long mask = __ballot(pending && r == rl);
        if (lane == leader) B.S[(int64_t)rl * B.stride + w] = mask;
        if (r == rl) pending = false;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  const unsigned long long m = __ballot(valid);
  if (lane == 0) {
    if (starred) *B.star = 1;
    if (B.ct) {
      B.ct[w] = m;
      if (m) B.nz[w / GW] = 1;
    }
  }
}

// The root slot before its propagation: no tuple (a negative table: all of
// them), every granule active, the domains dom0.
__global__ void __launch_bounds__(BLOCK) init_root_kernel(TabDesc* T, SlotDesc* root, const uint64_t* dom0) {
  const int64_t at = (int64_t)blockIdx.x * BLOCK + threadIdx.x, step = (int64_t)gridDim.x * BLOCK;
  for (int64_t w = at; w < T->stride; w += step) root->ct[w] = T->kind ? all_tuples_word(T, w) : 0ull;
  for (int64_t p = at; p < T->nGran; p += step) {
    root->idx[0][p] = (int32_t)p;
    root->idx[1][p] = (int32_t)p;
    root->stamp[p] = 0;
    root->nzFlag[p] = 0;
  }
  for (int64_t q = at; q < T->D; q += step) root->lastDom[q] = dom0[q];
  for (int64_t r = at; r < T->rows; r += step) root->res[r] = 0;
}

// a slot's state at the root, but its arrays
__device__ void slot_fresh(SlotDesc* s, int limit, int failed) {
  s->trailTop = 0;
  s->cur = 0;
  s->limit = limit;
  s->failed = failed;
  s->depth = 0;
  s->serial = 0;
  s->filtCount = 0;
  s->prepDone = 0;
  s->updDone = 0;
  s->status = 0;
  s->noop = 0;
  for (int x = 0; x < 8; ++x) s->stats[x] = 0;
}

// After the root propagation: the table's first slot takes the root state, and
// the table's descriptor what was not known before.  A failed root keeps dom0
// as its domains and no valid tuple.  out (host memory): status, star.
__global__ void __launch_bounds__(BLOCK) init_first_kernel(TabDesc* T, SlotDesc* s, SlotDesc* root, const uint64_t* dom0,
                                                           const int32_t* star, int32_t* out) {
  const bool failed = root->status == ST_FAIL;
  const CT_G int32_t* idx = root->idx[root->cur];
  const int limit = failed ? 0 : root->limit;
  const int64_t at = (int64_t)blockIdx.x * BLOCK + threadIdx.x, step = (int64_t)gridDim.x * BLOCK;
  for (int64_t w = at; w < T->stride; w += step) {
    const uint64_t x = failed ? 0ull : root->ct[w];
    if (failed) root->ct[w] = 0ull;
    s->ct[w] = x;
  }
  for (int64_t p = at; p < T->nGran; p += step) {
    const int g = idx[p];
    s->idx[0][p] = g;
    s->idx[1][p] = g;
    s->stamp[p] = 0;
    s->nzFlag[p] = 0;
  }
  for (int64_t q = at; q < T->D; q += step) {
    const uint64_t x = failed ? dom0[q] : root->lastDom[q];
    if (failed) root->lastDom[q] = x;
    s->lastDom[q] = x;
  }
  for (int64_t r = at; r < T->rows; r += step) s->res[r] = root->res[r];
  if (at == 0) {
    slot_fresh(s, limit, failed);
    T->idx0 = idx;
    T->limit0 = limit;
    T->rootFailed = failed;
    if (*star) T->policy = 1;  // a short table: reset
    out[0] = root->status;
    out[1] = *star;
  }
}

// copy the root state into n fresh slots (one workgroup per slot)
__global__ void __launch_bounds__(BLOCK) init_slots_kernel(const TabDesc* T, SlotDesc* slots,
                                                           int n, const int32_t* rootRes) {
  const int k = blockIdx.x;
  if (k >= n) return;
  SlotDesc* s = slots + k;
  const int64_t words = T->stride;
  for (int64_t w = threadIdx.x; w < words; w += BLOCK) s->ct[w] = T->ct0[w];
  for (int p = threadIdx.x; p < T->nGran; p += BLOCK) {
    s->idx[0][p] = T->idx0[p];
    s->idx[1][p] = T->idx0[p];
    s->stamp[p] = 0;
    s->nzFlag[p] = 0;
  }
  for (int q = threadIdx.x; q < T->D; q += BLOCK) s->lastDom[q] = T->dom0[q];
  for (int r = threadIdx.x; r < T->rows; r += BLOCK) s->res[r] = rootRes[r];
  if (threadIdx.x == 0) {
    slot_fresh(s, T->limit0, T->rootFailed);
  }
}

}  // namespace ctk

// ---------------------------------------------------------------------------
// launch wrappers used by the host runtime
// ---------------------------------------------------------------------------
namespace ctk {

// update items of a split job: WAVES x NGW granules each
int propagate_items_per_job_update(int nGran) { return (nGran + WAVES * NGW - 1) / (WAVES * NGW); }
int propagate_items_per_job_filter(int D) { return (D + WAVES - 1) / WAVES; }

// Workgroups of the propagate kernel that are resident at once on the whole
// device: the grid never exceeds it, so every workgroup that holds an item
// is running and every wait in the kernel can end.
int propagate_max_grid() {
  static int cached = 0;
  if (cached) return cached;
  int dev = 0, cus = 0, perCu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&perCu, propagate_kernel, BLOCK, 0) != hipSuccess ||
      perCu < 1)
    perCu = 1;
  cached = cus * perCu;
  return cached;
}

hipError_t launch_split_engine(const EngDesc& E, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(split_engine_kernel, dim3(grid), dim3(BLOCK), 0, stream, E);
  return hipGetLastError();
}

hipError_t launch_propagate(const KArgs& a, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(propagate_kernel, dim3(grid), dim3(BLOCK), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_build_supports(const BuildArgs& B, hipStream_t stream) {
  if (B.nw <= 0) return hipSuccess;
  // as many waves of a workgroup as 32 KB of cells take
  const int perWave = 64 * (std::min(B.n, BUILD_COLS) | 1) * (int)sizeof(int32_t);
  const int waves = std::max(1, std::min(WAVES, 32768 / perWave));
  hipLaunchKernelGGL(build_supports_kernel, dim3((unsigned)((B.nw + waves - 1) / waves)), dim3(waves * WAVE),
                     (size_t)waves * perWave, stream, B);
  return hipGetLastError();
}

// workgroups of a table's initialization kernels
static int init_grid(int64_t words) { return (int)std::max<int64_t>(1, std::min<int64_t>(256, words / BLOCK)); }

hipError_t launch_init_root(TabDesc* T, SlotDesc* root, const uint64_t* dom0, int64_t words, hipStream_t stream) {
  hipLaunchKernelGGL(init_root_kernel, dim3(init_grid(words)), dim3(BLOCK), 0, stream, T, root, dom0);
  return hipGetLastError();
}

hipError_t launch_init_first(TabDesc* T, SlotDesc* slot, SlotDesc* root, const uint64_t* dom0, const int32_t* star,
                             int32_t* out, int64_t words, hipStream_t stream) {
  hipLaunchKernelGGL(init_first_kernel, dim3(init_grid(words)), dim3(BLOCK), 0, stream, T, slot, root, dom0, star, out);
  return hipGetLastError();
}

hipError_t launch_init_slots(const TabDesc* T, SlotDesc* slots, int n, const int32_t* rootRes,
                             hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(init_slots_kernel, dim3(n), dim3(BLOCK), 0, stream, T, slots, n, rootRes);
  return hipGetLastError();
}

}  // namespace ctk
