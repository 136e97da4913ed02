// ct_staged.hip -- staged schedule of propagation jobs: the steps of
// enforceGAC (Alg. 1) of all jobs of a launch as three kernels,
//
//   prep    pops and pushes, Alg. 1's checks, Delta and s_val, the list of
//           support rows that updateTable ORs (one workgroup per job)
//   update  updateTable (Alg. 2), one wave per active granule of any job
//   finish  the sparse bitset's partition and FAIL (Alg. 1), filterDomains
//           (Alg. 3), one wave per domain word of any job
//
// The launch boundaries order the steps, so no workgroup waits for another
// and nothing is fenced inside a launch (an agent-scope release writes this
// chip's L2 back, an acquire invalidates it), and each kernel has the
// registers and LDS of its own step only: the update runs at eight waves per
// SIMD, the finish at six.  The jobs that run are known on the device after the
// prep (a model's clean tables, rejected inputs): it appends the later
// kernels' items to lists that their workgroups walk.
//
// Against the same steps as one launch whose workgroups wait for each other
// (agent-scope releases and acquires, 198 VGPRs and 79 KB of LDS a workgroup
// for every step, items from one queue): a call of 2,000,000 tuples 26 us
// against 64, of 2,422 domain words and 15,000 tuples 62 against 104, a batch
// of 128 searches over tables of 1,000 to 2,000,000 tuples 36 against 132, of
// 1,000 searches over tables of 16,000 38 against 71.
//
// A model's round is the same three launches: the prep takes each table's
// input from the pool and skips the tables none of whose variables changed,
// the finish ANDs the results into the next pool.  6 search steps on 400
// tables of up to 500,000 tuples: 730 us, against 1,240 with separate kernels
// for gather, merge, change and mark, captured 1, 1, then 8 rounds at a time.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ct_device.h"

namespace ctk {

hipError_t launch_propagate(const KArgs& a, int grid, hipStream_t stream);
int propagate_max_grid();

namespace {

// Prep workgroup: 1,024 threads for a launch of few jobs or with wide tables,
// else as many as let the jobs' workgroups all run at once: 512 (three on a
// CU), or 256 (six) beyond that many jobs (1,500 jobs: 16 us against 30).
constexpr int PMAX = 1024, PBLOCK_MANY = 512, PBLOCK_MOST = 256;
constexpr int SBLOCK = 256;              // update workgroup
constexpr int SWAVES = SBLOCK / WAVE;

// A finish workgroup filters FIN_WORDS domain words (or partitions): 256
// threads, or 1,024 whose waves share the scans of the missing values, for
// tables of more than FIN_WIDE_GRAN granules, which a value without a support
// reads in full.  The residue checks of a word gather 64 lines each, which one
// CU takes in turn, so a workgroup has few words: a call of 590 words and
// 15,000 tuples 31 us, with 16 words in a workgroup of 1,024 threads 39; of
// 1,744 words 50 against 56; of 2,541 the same.
constexpr int FIN_WORDS = 4, FIN_WIDE_GRAN = 64;
constexpr int PREP_WIDE_D = 512;  // domain words that want the large prep workgroup

// Waves that share a granule's row list in a batch of roots, which select most
// rows of their tables, too small to stream (stage_stream_roots): one wave's
// chain of round trips over 600 rows takes as long as the whole batch's
// traffic (300 tables of up to 500,000 tuples: 92 us a batch, streamed 96;
// 100 tables 50 against 79).
constexpr int SPLIT_ROWS = 96;
__host__ __device__ inline int stage_parts(int nrows) {
  return nrows >= 2 * SPLIT_ROWS ? 4 : nrows >= SPLIT_ROWS ? 2 : 1;
}

constexpr int ROW_U = 16;                // support rows in flight per wave; the list is padded to it
constexpr uint32_t SEG_FIRST = 1u << 31; // list entry: first row of its segment
constexpr uint32_t SEG_INC = 1u << 30;   //   of an incremental segment

__device__ __forceinline__ int s_lane() { return threadIdx.x & (WAVE - 1); }
__device__ __forceinline__ int s_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE); }

// The same pointer for every lane, known as such.
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t x = (uint64_t)p;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
  return (T*)((uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ int s_scan(int v) {  // inclusive prefix sum over the wave
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

__device__ __forceinline__ void s_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void put_slot(uint64_t* p, uint32_t payload, int32_t seq) {
  __hip_atomic_store(p, eng_slot(payload, (uint32_t)seq), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A status for the caller: a flagged slot (JF_LL) or a plain word read after
// the launch.
__device__ __forceinline__ void put_status(uint32_t flags, uint64_t* ll, int32_t seq, CT_G int32_t* out, int st) {
  if (flags & JF_LL) put_slot(ll, (uint32_t)st, seq);
  else if (out) *out = st;
}

__device__ __forceinline__ uint64_t all_tuples(const TabDesc* T, int64_t w) {
  if (w >= T->W) return 0ull;
  if (w < T->W - 1 || T->tailBits >= 64) return ~0ull;
  return (1ull << T->tailBits) - 1ull;
}

// ---------------------------------------------------------------------------
// Update: a wave takes one granule position of a job.  The record and the row
// list are the same for every lane: scalar loads, ROW_U rows in flight.
// Bound: the support rows (HBM, MALL or L2), or the round trips of one wave
// (position -> granule -> rows) when a job has few rows.
// ---------------------------------------------------------------------------
// A job's record (the same for every lane: scalar loads of the fields used).
__device__ __forceinline__ StageRec load_rec(const StageArgs& A, int job) {
  StageRec V;
  const CT_K uint32_t* from = (const CT_K uint32_t*)(A.rec + job);
  uint32_t* to = (uint32_t*)&V;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(StageRec) / sizeof(uint32_t)); ++i) to[i] = from[i];
  return V;
}

__device__ __forceinline__ void seg_close(uint64_t& m, uint64_t& acc, bool inc) {
  m &= inc ? ~acc : acc;
  acc = 0ull;
}

// A granule whose row list is split over `parts` waves of its workgroup: what
// each leaves for the first (segments cross the parts' borders).
struct SplitShared {
  uint64_t mask[SWAVES][WAVE];   // the segments that end in the part
  uint64_t first[SWAVES][WAVE];  // the OR up to the part's first segment start
  uint64_t open[SWAVES][WAVE];   // the OR of the segment that its end leaves open
  int32_t has[SWAVES], inc[SWAVES];  // a segment starts in the part; the open one's kind
};

__device__ __forceinline__ void stage_granule(const StageArgs& A, const StageRec& V, CT_G int32_t* trailCount,
                                              int pos, int part, int parts, SplitShared& sh) {
  const StageRec* R = &V;
  const int limit = R->limit, nGran = R->nGran, mode = R->mode;
  const uint32_t flags = R->flags;
  const bool fromRoot = flags & JF_FROM_ROOT, scratch = flags & JF_SCRATCH;
  const int lane = s_lane();
  CT_G uint64_t* const ctOut = R->ct_out;
  const bool active = pos < limit;
  if (parts > 1 && !active && part > 0) pos = nGran;  // (one wave writes an inactive granule)
  if (pos >= nGran || (!active && !fromRoot && !ctOut)) {
    if (parts > 1) s_lds_barrier();
    return;
  }
  const int g = scratch ? pos : ((const CT_K int32_t*)R->idxSrc)[pos];
  const int64_t w = (int64_t)g * GW + lane;
  if (!active) {  // inactive granule (all zero by invariant)
    if (fromRoot) R->ct[w] = 0ull;
    if (ctOut && w < R->W) {
      ctOut[w] = 0ull;
      if (flags & JF_HOST_OUT) __threadfence_system();
    }
    if (parts > 1) s_lds_barrier();
    return;
  }
  const uint64_t old = scratch ? all_tuples((const TabDesc*)R->tab, w) : R->ctSrc[w];
  const int serial = R->serial;
  const int trail = R->trailOn;
  const int stv = trail != STAGE_TRAIL_OFF ? R->stamp[g] : serial;
  const int64_t stride = R->stride;
  const CT_G uint64_t* S = R->S + w;
  uint64_t m = ~0ull, acc = 0ull;
  if (mode == STAGE_LIST) {
    bool inc = true;  // nothing before the first segment: ~0 leaves m alone
    const int nrows = R->nrows;
    const CT_K uint32_t* list = (const CT_K uint32_t*)R->rows;
    // this wave's part of the list, in whole groups
    const int groups = (nrows + ROW_U - 1) / ROW_U, per = (groups + parts - 1) / parts;
    const int kEnd = parts > 1 ? min(nrows, (part + 1) * per * ROW_U) : nrows;
    uint64_t first = 0ull;
    bool has = part == 0;
    for (int k0 = part * per * ROW_U; k0 < kEnd; k0 += ROW_U) {
      uint32_t e[ROW_U];
      uint64_t v[ROW_U];
#pragma unroll
      for (int j = 0; j < ROW_U; ++j) e[j] = list[k0 + j];
      if (scratch) {  // (a root: most rows, each read once, pass the caches by)
#pragma unroll
        for (int j = 0; j < ROW_U; ++j) v[j] = __builtin_nontemporal_load(S + (int64_t)(e[j] & 0x3fffffffu) * stride);
      } else {
#pragma unroll
        for (int j = 0; j < ROW_U; ++j) v[j] = S[(int64_t)(e[j] & 0x3fffffffu) * stride];
      }
#pragma unroll
      for (int j = 0; j < ROW_U; ++j) {
        if (e[j] & SEG_FIRST) {
          if (has) {
            seg_close(m, acc, inc);
          } else {
            first = acc;
            acc = 0ull;
            has = true;
          }
          inc = e[j] & SEG_INC;
        }
        acc |= v[j];
      }
    }
    if (parts > 1) {
      if (part > 0) {
        sh.mask[s_wave()][lane] = m;
        sh.first[s_wave()][lane] = has ? first : acc;
        sh.open[s_wave()][lane] = acc;
        if (lane == 0) {
          sh.has[s_wave()] = has;
          sh.inc[s_wave()] = inc;
        }
      }
      s_lds_barrier();
      if (part > 0) return;
      for (int p = s_wave() + 1; p < s_wave() + parts; ++p) {
        acc |= sh.first[p][lane];
        if (__builtin_amdgcn_readfirstlane(sh.has[p])) {
          seg_close(m, acc, inc);
          m &= sh.mask[p][lane];
          acc = sh.open[p][lane];
          inc = __builtin_amdgcn_readfirstlane(sh.inc[p]);
        }
      }
    }
    if (nrows) seg_close(m, acc, inc);
  } else if (mode == STAGE_BITS) {
    const CT_K uint64_t* sel = (const CT_K uint64_t*)R->rows;
    const CT_K int32_t* size = (const CT_K int32_t*)R->size;
    const CT_K WordDesc* words = (const CT_K WordDesc*)R->words;
    const int D = R->D;
    bool inc = false, in = false;
    for (int q = 0; q < D; ++q) {
      const int domOff = words[q].v.domOff;
      if (q == domOff) {
        if (in) seg_close(m, acc, inc);
        const int sz = size[q];
        in = !(sz & (1 << 29));
        inc = sz & (1 << 30);
      }
      uint64_t bits = in ? sel[q] : 0ull;
      const CT_G uint64_t* Sq = S + (int64_t)(words[q].v.rowStart + 64 * (q - domOff)) * stride;
      int b = 0;
      while (bits) {
        uint64_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (bits) {  // past the last value: the previous row again
            b = __ffsll((unsigned long long)bits) - 1;
            bits &= bits - 1;
          }
          v[u] = Sq[(int64_t)b * stride];
        }
        acc |= (v[0] | v[1]) | (v[2] | v[3]);
      }
    }
    if (in) seg_close(m, acc, inc);
  } else if (mode == STAGE_ZERO) {
    m = 0ull;
  }
  const uint64_t nw = old & m;
  const bool changed = __ballot(nw != old) != 0ull;
  if (trail == STAGE_TRAIL_ALL || (trail == STAGE_TRAIL_FIRST && changed && stv != serial)) {
    // a level pushed by this job saves every active granule at its position's
    // entry: counting entries would take an atomic on one word per granule
    // (about 20 ns each).  Later jobs of the level save the first change of a
    // granule not saved yet.
    int t = pos;
    if (trail == STAGE_TRAIL_FIRST) {
      if (lane == 0) t = atomicAdd((int32_t*)trailCount, 1);
      t = __builtin_amdgcn_readfirstlane(t);
    }
    const int64_t tp = R->trailTop + t;
    if (tp < R->trailCap) {
      R->trailWords[tp * GW + lane] = old;
      if (lane == 0) {
        TrailHdr h;
        h.gran = g;
        h.oldStamp = stv;
        R->trailHdr[tp] = h;
        R->stamp[g] = serial;
      }
    } else if (lane == 0) {  // capacity is sized so that this cannot happen
      atomicExch(&A.queue[3], 2);
      if (A.hostErr) __hip_atomic_store(A.hostErr, 2, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  if (changed || fromRoot || (flags & JF_ROOT)) R->ct[w] = nw;
  if (ctOut && w < R->W) {
    ctOut[w] = nw;
    // a synchronous call's copy is in host memory: there before the finish's
    // result slots
    if (flags & JF_HOST_OUT) __threadfence_system();
  }
  const bool nz = __ballot(nw != 0ull) != 0ull;
  if (lane == 0) R->nz[pos] = (nz ? 1 : 0) | (changed ? 2 : 0);
}

// ---------------------------------------------------------------------------
// Finish, item 0 of a job: the stable partition of the active granule list
// (survivors first) into the other index buffer, the new limit, FAIL when no
// granule survives (Alg. 1's failure test), the slot's state and counters.
// One workgroup.
// ---------------------------------------------------------------------------
template <int FBLOCK>
struct FinShared {
  static constexpr int FWAVES = FBLOCK / WAVE;
  int32_t wsum[FWAVES], wsum2[FWAVES];
  unsigned long long unsup[FWAVES];  // per word: values without a support
  int32_t nMiss, nLeft, scans;
  uint16_t miss[FWAVES * 64];        // word << 6 | bit
  int32_t res[FWAVES * 64];          // the residue that missed
  uint8_t found[FWAVES * 64];
  uint16_t gran[MAX_GRAN];           // surviving granules
};

// Prefix sum over the workgroup (before this thread); *total the sum.
template <int FWAVES>
__device__ __forceinline__ int fin_scan(int v, int* total, int32_t (&wsum)[FWAVES]) {
  const int x = s_scan(v);
  if (s_lane() == WAVE - 1) wsum[s_wave()] = x;
  s_lds_barrier();
  int off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < FWAVES; ++k) {
    const int w = wsum[k];
    off += k < s_wave() ? w : 0;
    tot += w;
  }
  s_lds_barrier();
  *total = tot;
  return off + x - v;
}

template <int FBLOCK>
__device__ __forceinline__ void stage_partition(const StageRec& V, FinShared<FBLOCK>& sh) {
  const StageRec* R = &V;
  CT_G SlotDesc* s = R->slot;
  const int limit = R->limit, nGran = R->nGran, tid = threadIdx.x;
  const bool fromRoot = R->flags & JF_FROM_ROOT, scratch = R->flags & JF_SCRATCH;
  const bool noop = R->mode == STAGE_NOOP;
  const CT_G int32_t* src = R->idxSrc;
  CT_G int32_t* dst = R->idxDst;
  const CT_G int32_t* nz = R->nz;
  int nSurv = limit, nChanged = 0;
  if (!noop) {
    // survivors and changed granules in all, then the survivors' places; the
    // first pass's flags and granules stay in registers
    int f0 = 0, g0 = 0, c = 0, ch = 0;
    for (int p = tid; p < limit; p += FBLOCK) {
      const int f = nz[p];
      if (p == tid) {
        f0 = f;
        g0 = scratch ? p : src[p];
      }
      c += f & 1;
      ch += f >> 1;
    }
    fin_scan(ch, &nChanged, sh.wsum2);
    fin_scan(c, &nSurv, sh.wsum);
    int sv = 0, zr = nSurv;
    for (int p0 = 0; p0 < limit; p0 += FBLOCK) {
      const int p = p0 + tid;
      const bool in = p < limit;
      const int f = in ? (p0 == 0 ? f0 : nz[p]) & 1 : 0;
      const int g = in ? (p0 == 0 ? g0 : scratch ? p : src[p]) : 0;
      int tot = 0;
      const int before = fin_scan(f, &tot, sh.wsum);  // survivors before this position in the pass
      if (in) dst[f ? sv + before : zr + (tid - before)] = g;
      sv += tot;
      zr += min(FBLOCK, limit - p0) - tot;
    }
    for (int p = limit + tid; p < nGran; p += FBLOCK) dst[p] = scratch ? p : src[p];
  }
  if (tid == 0) {
    const int st = noop || nSurv ? ST_OK : ST_FAIL;
    const int trail = R->trailOn;
    // entries written, and the granules among them that changed (the counter)
    const int entries = trail == STAGE_TRAIL_ALL ? limit : trail == STAGE_TRAIL_FIRST ? R->trailCount : 0;
    const int saved = trail == STAGE_TRAIL_ALL ? nChanged : entries;
    if (!noop) {
      s->cur = R->curNew;
      s->limit = nSurv;
      if (fromRoot) {
        s->depth = 0;
        s->trailTop = 0;
        s->serial = R->serialBase;
        s->failed = 0;
      } else {
        s->trailTop = R->trailTop + entries;
      }
      if (!nSurv) s->failed = 1;
    }
    s->status = st;
    s->noop = noop;
    const unsigned long long nrows = (unsigned long long)R->nrows, lim = (unsigned long long)limit;
    atomicAdd(&s->stats[S_JOBS], 1ull);
    atomicAdd(&s->stats[S_GRAN_IN], lim);
    atomicAdd(&s->stats[S_ROWS], nrows);
    if (nrows && lim) atomicAdd(&s->stats[S_GRAN_ROWS], lim * nrows);
    if (saved) atomicAdd(&s->stats[S_TRAIL], (unsigned long long)saved);
    // a flagged call reports success by its domain words
    if (st != ST_OK || !(R->flags & JF_LL)) put_status(R->flags, R->ll, R->seq, R->status_out, st);
    if (R->poolMap && st != ST_OK) R->model->fail = (R->round + 1) << 2 | 1;
  }
}

// What a table of a model round removed leaves the pool: domain word q, one lane.
__device__ __forceinline__ void stage_merge(const StageRec& R, int q, uint64_t dout) {
  const int pw = R.poolMap[q];
  if (R.poolCur[pw] & ~dout) {
    atomicAnd((unsigned long long*)(R.poolNext + pw), dout);
    R.model->lastChanged = R.round + 1;
  }
}

// ---------------------------------------------------------------------------
// Finish, other items: filterDomains of FIN_WORDS domain words by one workgroup.
//   A. one wave per word: the support word at every value's residue against
//      currTable; the values that miss go to a list;
//   B. (more than FULL_GRAN surviving granules) one thread per missing value
//      walks the words after its residue;
//   C. the values left scan the surviving granules: a wave takes tasks of
//      (FULL_VALS values, FULL_GRAN granules), so a word with many missing
//      values, or a value that has no support left (all granules read), does
//      not wait for one wave.
// Bound: the chain of round trips (record -> residues -> words -> scans).
// ---------------------------------------------------------------------------
constexpr int FULL_GRAN = 4, FULL_VALS = 4;
constexpr int WALK = 8, WALKS = 2;

template <int FBLOCK>
__device__ __forceinline__ void stage_filter(const StageRec& V, int q0, int nWords, FinShared<FBLOCK>& sh) {
  constexpr int FWAVES = FBLOCK / WAVE;
  const StageRec* R = &V;
  const int lane = s_lane(), wv = s_wave(), tid = threadIdx.x;
  const int D = R->D, q = q0 + wv;
  const bool word = wv < nWords && q < D;
  const int qc = word ? q : q0;
  const CT_K WordDesc* wds = (const CT_K WordDesc*)R->words;
  const int rowStart = wds[qc].v.rowStart, domOff = wds[qc].v.domOff, dsize = wds[qc].v.dsize;
  const uint64_t din = ((const CT_K uint64_t*)R->din)[qc];
  const int size = ((const CT_K int32_t*)R->size)[qc] & 0x1fffffff;
  const int64_t stride = R->stride;
  const CT_G uint64_t* ct = R->ct;
  const CT_G int32_t* nz = R->nz;
  const CT_G int32_t* idx = R->idxSrc;
  CT_G int32_t* res = R->res;
  const int limit = R->limit;
  const bool noop = R->mode == STAGE_NOOP, scratch = R->flags & JF_SCRATCH;
  const bool filter = word && !noop && size > 1;  // s_sup: variables with two or more values
  int nSurv = 0;
  uint64_t unsup = 0ull;
  if (!noop) {
    // A, and the surviving granules into LDS meanwhile
    const int cBase = rowStart + (qc - domOff) * 64;
    const int row = cBase + (filter ? min(lane, dsize - 64 * (qc - domOff) - 1) : 0);
    const int r = min(max(res[row], 0), (int)stride - 1);
    // (at most 64 active positions: every wave has them all)
    const bool small = limit <= WAVE;
    const int at = small ? lane : tid;
    const int pc = max(min(at, limit - 1), 0);
    const int f0 = at < limit ? nz[pc] & 1 : 0;
    const int g0 = scratch ? pc : idx[pc];
    if (tid == 0) {
      sh.nMiss = 0;
      sh.nLeft = 0;
      sh.scans = 0;
    }
    const uint64_t sw = R->S[(int64_t)row * stride + r], cw = ct[r];
    if (small) {
      const uint64_t act = __ballot(f0);
      nSurv = __popcll(act);
      if (wv == 0 && f0) sh.gran[__popcll(act & ((1ull << lane) - 1ull))] = (uint16_t)g0;
      s_lds_barrier();  // (the counters are zero)
    } else {
      for (int p0 = 0; p0 < limit; p0 += FBLOCK) {
        const int p = p0 + tid;
        const int f = p0 == 0 ? f0 : p < limit ? nz[p] & 1 : 0;
        int tot = 0;
        const int before = fin_scan(f, &tot, sh.wsum);
        if (f) sh.gran[nSurv + before] = (uint16_t)(p0 == 0 ? g0 : scratch ? p : idx[p]);
        nSurv += tot;
      }
    }
    if (nSurv == 0) return;  // FAIL leaves the domains alone (the same for the whole workgroup)
    const bool present = filter && ((din >> lane) & 1ull);  // (validated: no stray bits)
    const bool lost = present && (sw & cw) == 0ull;
    const uint64_t miss = __ballot(lost);
    if (miss) {
      int k = 0;
      if (lane == 0) k = atomicAdd(&sh.nMiss, __popcll(miss));
      k = __builtin_amdgcn_readfirstlane(k) + __popcll(miss & ((1ull << lane) - 1ull));
      if (lost) {
        sh.miss[k] = (uint16_t)(wv << 6 | lane);
        sh.res[k] = r;
        sh.found[k] = 0;
      }
    }
    if (lane == 0) {
      sh.unsup[wv] = miss;
      sh.wsum[wv] = filter ? __popcll(din) : 0;
    }
    s_lds_barrier();
    const int nMiss = sh.nMiss;
    if (nMiss) {
      const bool walk = nSurv > FULL_GRAN;
      int nLeft = nMiss;
      if (walk) {
        const int words = (int)stride;
        if (tid < nMiss) {
          const int m = sh.miss[tid], qm = q0 + (m >> 6);
          const CT_G WordDesc* w = R->words + qm;
          const int rm = w->v.rowStart + (qm - w->v.domOff) * 64 + (m & 63), r0 = sh.res[tid];
          const CT_G uint64_t* row = R->S + (int64_t)rm * stride;
          int found = -1;
          for (int k = 0; k < WALKS && found < 0; ++k) {
            uint64_t y[WALK];
#pragma unroll
            for (int t = 0; t < WALK; ++t) {
              int x = r0 + 1 + k * WALK + t;
              if (x >= words) x -= words;
              y[t] = row[x] & ct[x];
            }
#pragma unroll
            for (int t = WALK - 1; t >= 0; --t) {
              int x = r0 + 1 + k * WALK + t;
              if (x >= words) x -= words;
              if (y[t]) found = x;
            }
          }
          if (found >= 0) {
            res[rm] = found;
            atomicAnd(&sh.unsup[m >> 6], ~(1ull << (m & 63)));
            sh.found[tid] = 1;
          }
        }
        s_lds_barrier();
        // the values left, compacted in place (every thread has read its own)
        const int m = tid < nMiss ? sh.miss[tid] : 0;
        const int keep = tid < nMiss && !sh.found[tid];
        s_lds_barrier();
        const int at = fin_scan(keep, &nLeft, sh.wsum2);
        if (keep) {
          sh.miss[at] = (uint16_t)m;
          sh.found[at] = 0;
        }
        s_lds_barrier();
      }
      // C: task t = value group t % nGrp, granules FULL_GRAN (t / nGrp) ..:
      // every group's first granules come first
      const int nGrp = (nLeft + FULL_VALS - 1) / FULL_VALS;
      const int nTasks = nGrp * ((nSurv + FULL_GRAN - 1) / FULL_GRAN);
      int scans = 0;
      for (int t = wv; t < nTasks; t += FWAVES) {
        const int k0 = (t % nGrp) * FULL_VALS, p0 = (t / nGrp) * FULL_GRAN;
        int rm[FULL_VALS];
        bool live[FULL_VALS], any = false;
#pragma unroll
        for (int k = 0; k < FULL_VALS; ++k) {
          const int i = min(k0 + k, nLeft - 1);
          live[k] = __builtin_amdgcn_readfirstlane(k0 + k < nLeft && !sh.found[i]);
          any = any || live[k];
          const int m = __builtin_amdgcn_readfirstlane(sh.miss[i]), qm = q0 + (m >> 6);
          rm[k] = wds[qm].v.rowStart + (qm - wds[qm].v.domOff) * 64 + (m & 63);
        }
        if (!any) continue;
        int gg[FULL_GRAN];
        uint64_t c[FULL_GRAN], x[FULL_VALS][FULL_GRAN];
#pragma unroll
        for (int j = 0; j < FULL_GRAN; ++j) {
          gg[j] = __builtin_amdgcn_readfirstlane(sh.gran[min(p0 + j, nSurv - 1)]);
          c[j] = ct[(int64_t)gg[j] * GW + lane];
        }
#pragma unroll
        for (int k = 0; k < FULL_VALS; ++k)
#pragma unroll
          for (int j = 0; j < FULL_GRAN; ++j) x[k][j] = R->S[(int64_t)rm[k] * stride + (int64_t)gg[j] * GW + lane];
#pragma unroll
        for (int k = 0; k < FULL_VALS; ++k) {
          if (!live[k]) continue;
          scans += min(FULL_GRAN, nSurv - p0);
          int at = -1;
#pragma unroll
          for (int j = FULL_GRAN - 1; j >= 0; --j) {
            const uint64_t bm = __ballot((x[k][j] & c[j]) != 0ull);
            if (bm) at = gg[j] * GW + __ffsll((unsigned long long)bm) - 1;
          }
          if (at >= 0 && lane == 0) {
            const int m = sh.miss[k0 + k];
            res[rm[k]] = at;
            sh.found[k0 + k] = 1;
            atomicAnd(&sh.unsup[m >> 6], ~(1ull << (m & 63)));
          }
        }
      }
      if (lane == 0 && scans) atomicAdd(&sh.scans, scans);
      s_lds_barrier();
    }
    unsup = sh.unsup[wv];
    if (tid == 0) {
      int chk = 0;
#pragma unroll
      for (int k = 0; k < FWAVES; ++k) chk += sh.wsum[k];
      if (chk) {
        CT_G SlotDesc* s = R->slot;
        atomicAdd(&s->stats[S_RES_CHECK], (unsigned long long)chk);
        if (nMiss) atomicAdd(&s->stats[S_RES_MISS], (unsigned long long)nMiss);
        if (sh.scans) atomicAdd(&s->stats[S_SCAN], (unsigned long long)sh.scans);
      }
    }
  }
  if (!word) return;
  const uint64_t dout = din & ~unsup;
  if (R->poolMap) {
    if (lane == 0) stage_merge(*R, q, dout);
  } else if (R->flags & JF_LL) {
    if (lane < 2) put_slot(R->ll + 2 + 2 * q + lane, (uint32_t)(lane ? dout >> 32 : dout), R->seq);
  } else if (lane == 0) {
    R->dom_out[q] = dout;
  }
  if (lane == 0) R->lastDom[q] = dout;
}

template <int FBLOCK>
__device__ __forceinline__ void stage_finish_item(const StageArgs& A, int job, int chunk, FinShared<FBLOCK>& sh) {
  const StageRec R = load_rec(A, job);
  if (!R.run) return;
  if (chunk == 0) stage_partition(R, sh);
  else stage_filter(R, (chunk - 1) * FIN_WORDS, FIN_WORDS, sh);
}

struct PrepShared {
  int32_t size[MAX_ARITY], dcnt[MAX_ARITY];
  int32_t seg[MAX_ARITY];  // first list entry of the variable's segment; -1: not in s_val
  int32_t inc[MAX_ARITY];
  int32_t wsum[PMAX / WAVE];
  uint32_t job[sizeof(DevJob) / sizeof(uint32_t)];
  int32_t stray, notSub, dirty, status, noop, zero, nrows;
  // the job's places in the item lists: fields of their own, because a wave
  // may still be reading the others when thread 0 writes these (a job without
  // a row list passes no barrier between the two)
  int32_t u0, f0, nU, nF;
};

// Exclusive prefix sum over the workgroup; *total receives the sum.
template <int PWAVES>
__device__ int prep_scan(int v, int* total, PrepShared& sh) {
  const int x = s_scan(v);
  if (s_lane() == WAVE - 1) sh.wsum[s_wave()] = x;
  s_lds_barrier();
  int off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < PWAVES; ++k) {
    const int w = sh.wsum[k];
    off += k < s_wave() ? w : 0;
    tot += w;
  }
  s_lds_barrier();
  *total = tot;
  return off + x - v;
}

// A model round's first workgroups: next starts as a copy of cur; the host
// hears how the round before ended, and gets the pool when it was the last.
__device__ __forceinline__ int model_code(const ModelRound& M) {
  const int fail = M.state->fail, last = M.state->lastChanged;
  if (M.round == 0) return 0;
  if (fail && (fail >> 2) <= M.round) return fail & 3;
  return last < M.round ? MODEL_DONE : 0;
}

// A failed round was the last (after a round without a change no table is
// dirty).  Jobs of this round may set fail meanwhile: theirs does not count.
__device__ __forceinline__ bool model_over(const ModelRound& M) {
  const int fail = M.state->fail;
  return fail && (fail >> 2) <= M.round;
}

template <int PBLOCK>
__device__ __forceinline__ void model_head(const ModelRound& M) {
  const int code = model_code(M);
  CT_G uint64_t* dst = code ? M.poolOut : M.next;
  for (int w = blockIdx.x * PBLOCK + threadIdx.x; w < M.poolWords; w += M.nHead * PBLOCK) dst[w] = M.cur[w];
  if (blockIdx.x == 0 && threadIdx.x < WAVE && M.round > 0) {
    const int p = s_scan(s_lane() < MODEL_PROPS ? M.state->props[s_lane() * 16] : 0);
    if (s_lane() == WAVE - 1) {
      __hip_atomic_store(&M.host[1], (uint64_t)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(&M.host[0], (uint64_t)(uint32_t)M.call << 32 | (uint32_t)(M.round << 8 | code),
                         __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// The pool a fixpoint starts from: the input ANDed with the domains that every
// table returned last (an earlier pruning holds under a smaller pool).  8 lanes
// per pool word, src[off[w] .. off[w + 1]) its words in the tables.
__global__ void __launch_bounds__(SBLOCK) model_start_kernel(const uint64_t* poolIn, uint64_t* pool, const int32_t* off,
                                                             const uint64_t* const* src, int poolWords,
                                                             ModelState* state) {
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < (int)(sizeof(ModelState) / sizeof(int32_t)); k += SBLOCK) ((int32_t*)state)[k] = 0;
  const int w = (int)(blockIdx.x * SBLOCK + threadIdx.x) / 8, l = threadIdx.x & 7;
  const int wc = min(w, poolWords - 1);
  uint64_t x = ((const CT_G uint64_t*)poolIn)[wc];
  const int end = off[wc + 1];
#pragma unroll 4
  for (int k = off[wc] + l; k < end; k += 8) x &= *(const CT_G uint64_t*)src[k];
  for (int d = 1; d < 8; d <<= 1) x &= __shfl_xor((unsigned long long)x, d);
  if (l == 0 && w < poolWords) pool[w] = x;
}

// Negative tables of a model round (they run in the propagate kernel): which
// run and on what; then what they remove leaves the pool.  One workgroup per
// job; map: the pool word of each domain word.
__global__ void __launch_bounds__(SBLOCK) model_neg_gather_kernel(const DevJob* jobs, const int32_t* const* maps,
                                                                  int32_t* dirty, ModelRound M) {
  __shared__ int32_t any;
  const DevJob J = jobs[blockIdx.x];
  const CT_G int32_t* map = (const CT_G int32_t*)maps[blockIdx.x];
  if (threadIdx.x == 0) any = 0;
  __syncthreads();
  const int D = J.tab->D;
  const CT_G uint64_t* last = J.slot->lastDom;
  CT_G uint64_t* in = (CT_G uint64_t*)J.dom_in;
  const bool over = model_over(M);
  for (int q = threadIdx.x; q < D; q += SBLOCK) {
    const int pw = map[q];
    const uint64_t x = M.cur[pw], ld = last[q];
    if (!over && (M.round ? x != M.prev[pw] : (ld & ~x) != 0)) any = 1;
    in[q] = x & ld;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    dirty[blockIdx.x] = any;
    if (any) atomicAdd((int32_t*)&M.state->props[((int)blockIdx.x % MODEL_PROPS) * 16], 1);
  }
}

__global__ void __launch_bounds__(SBLOCK) model_neg_merge_kernel(const DevJob* jobs, const int32_t* const* maps,
                                                                 const int32_t* dirty, ModelRound M) {
  if (!dirty[blockIdx.x]) return;
  const DevJob J = jobs[blockIdx.x];
  const CT_G int32_t* map = (const CT_G int32_t*)maps[blockIdx.x];
  const int st = *J.status_out;
  if (st != ST_OK) {
    if (threadIdx.x == 0) M.state->fail = (M.round + 1) << 2 | (st == ST_FAIL ? 1 : 2);
    return;
  }
  for (int q = threadIdx.x; q < J.tab->D; q += SBLOCK) {
    const int pw = map[q];
    const uint64_t x = J.dom_out[q];
    if (M.cur[pw] & ~x) {
      atomicAnd((unsigned long long*)(M.next + pw), x);
      M.state->lastChanged = M.round + 1;
    }
  }
}

// ---------------------------------------------------------------------------
// Prep: one workgroup per job.  Dynamic LDS: an int per granule of the
// largest popping table of the launch.
// Bound: its chain of memory round trips (job -> slot -> domains -> list).
// ---------------------------------------------------------------------------
template <int PBLOCK, bool MODEL>
__global__ void __launch_bounds__(PBLOCK, 4) stage_prep_kernel(KArgs a, StageArgs A, ModelRound M) {
  constexpr int PWAVES = PBLOCK / WAVE;
  __shared__ PrepShared sh;
  extern __shared__ int32_t first[];
  if (a.clock && threadIdx.x == 0) atomicMin(&a.clock[0], wall_clock64());
  const int tid = threadIdx.x, lane = s_lane();
  if (MODEL && (int)blockIdx.x < M.nHead) {
    model_head<PBLOCK>(M);
    return;
  }
  const int job = MODEL ? (int)blockIdx.x - M.nHead : (int)blockIdx.x;
  // the descriptor may be in host memory: read once per workgroup, into LDS
  constexpr int JW = sizeof(DevJob) / sizeof(uint32_t);
  const CT_G uint32_t* from = (const CT_G uint32_t*)(a.jobs + job);
  if (tid < JW) sh.job[tid] = a.jobs ? from[tid] : ((const uint32_t*)&a.job)[tid];
  if (MODEL && model_over(M)) return;
  s_lds_barrier();
  DevJob J;
  __builtin_memcpy(&J, sh.job, sizeof(J));
  J.tab = uniform_ptr(J.tab);
  J.slot = uniform_ptr(J.slot);
  J.dom_in = uniform_ptr(J.dom_in);
  J.flags = a.uniform ? 0 : __builtin_amdgcn_readfirstlane((int)J.flags);
  J.nPop = a.uniform ? a.job.nPop : __builtin_amdgcn_readfirstlane(J.nPop);
  J.nPush = a.uniform ? a.job.nPush : __builtin_amdgcn_readfirstlane(J.nPush);
  J.serialBase = a.uniform ? a.job.serialBase : J.serialBase;
  CT_G StageRec* rec = A.rec + job;
  const CT_G TabDesc* T = J.tab;
  CT_G SlotDesc* s = J.slot;
  const int n = T->n, D = T->D, nGran = T->nGran;
  const bool fromRoot = J.flags & JF_FROM_ROOT, root = J.flags & JF_ROOT, scratch = J.flags & JF_SCRATCH;
  if (A.roots)  // (also of a job that is rejected: the update looks at the record)
    for (int k = tid; k < (nGran + SWAVES - 1) / SWAVES; k += PBLOCK) A.items[J.seq + k] = StageItem{job, k};
  // the slot's state before the job
  int depth = s->depth, limit = s->limit, failed = s->failed, serial = s->serial;
  const int cur = s->cur;
  int64_t trailTop = s->trailTop;
  const CT_G uint64_t* last = s->lastDom;
  if (J.nPop > 0) {
    // every popped level at once: the level popped to holds its state; a
    // granule saved on the trail after it gets the words of its first entry
    // there (the oldest save holds the words of that level)
    depth -= J.nPop;
    const Level Lv = s->levels[depth];
    const int64_t lo = Lv.trailTop;
    const CT_G TrailHdr* hdr = s->trailHdr;
    const CT_G uint64_t* words = s->trailWords;
    for (int g = tid; g < nGran; g += PBLOCK) first[g] = 0x7fffffff;
    s_lds_barrier();
    for (int64_t e = lo + tid; e < trailTop; e += PBLOCK) atomicMin(&first[hdr[e].gran], (int)(e - lo));
    s_lds_barrier();
    constexpr int U = 8;  // granules per wave and round trip
    CT_G uint64_t* ct = s->ct;
    CT_G int32_t* stamp = s->stamp;
    for (int g0 = s_wave() * U; g0 < nGran; g0 += PWAVES * U) {
      int f[U], st[U];
      uint64_t w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f[u] = g0 + u < nGran ? __builtin_amdgcn_readfirstlane(first[g0 + u]) : 0x7fffffff;
        if (f[u] != 0x7fffffff) {
          st[u] = hdr[lo + f[u]].oldStamp;
          w[u] = words[(lo + f[u]) * GW + lane];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (f[u] != 0x7fffffff) {
          ct[(int64_t)(g0 + u) * GW + lane] = w[u];
          if (lane == 0) stamp[g0 + u] = st[u];
        }
    }
    last = s->levelDom + (int64_t)depth * D;
    for (int q = tid; q < D; q += PBLOCK) s->lastDom[q] = last[q];
    limit = Lv.limit;
    failed = Lv.failed;
    serial = Lv.serial;
    trailTop = lo;
  }
  // pushes record the state here
  if (tid < J.nPush) {
    Level Lv;
    Lv.trailTop = trailTop;
    Lv.limit = limit;
    Lv.failed = failed;
    Lv.serial = tid == 0 ? serial : J.serialBase + tid - 1;
    Lv.pad = 0;
    s->levels[depth + tid] = Lv;
  }
  for (int k = PBLOCK + tid; k < J.nPush; k += PBLOCK) {
    Level Lv;
    Lv.trailTop = trailTop;
    Lv.limit = limit;
    Lv.failed = failed;
    Lv.serial = J.serialBase + k - 1;
    Lv.pad = 0;
    s->levels[depth + k] = Lv;
  }
  if (J.nPush > 0) serial = J.serialBase + J.nPush - 1;
  if (J.nPop > 0 || J.nPush > 0) {
    __syncthreads();  // every wave has the slot's state
    if (tid == 0) {
      s->trailTop = trailTop;
      s->limit = limit;
      s->failed = failed;
      s->serial = serial;
      s->depth = depth + J.nPush;
    }
  }
  if (!(J.flags & JF_PROPAGATE)) {
    for (int k = 0; k < J.nPush; ++k)
      for (int q = tid; q < D; q += PBLOCK) s->levelDom[(int64_t)(depth + k) * D + q] = last[q];
    if (tid == 0) {
      if (!A.items) rec->run = 0;  // (with lists: no items)
      put_status(J.flags, J.ll, J.seq, J.status_out, ST_OK);
    }
    return;
  }
  if (fromRoot) {
    last = T->dom0;
    limit = scratch ? nGran : T->limit0;
    failed = scratch ? 0 : T->rootFailed;
  }
  // Alg. 1: checks, |dom| and |Delta| per variable
  for (int i = tid; i < n; i += PBLOCK) {
    sh.size[i] = 0;
    sh.dcnt[i] = 0;
  }
  if (tid == 0) {
    sh.stray = 0;
    sh.notSub = 0;
    sh.dirty = 0;
  }
  s_lds_barrier();
  CT_G uint64_t* dinW = (CT_G uint64_t*)(A.jobMem + (int64_t)J.stageOff * 256);  // D: the input
  CT_G int32_t* sizeW = (CT_G int32_t*)(dinW + D);   // D: |dom| of the word's variable
  CT_G uint32_t* rows = (CT_G uint32_t*)(sizeW + ((D + 1) & ~1));
  const CT_G WordDesc* words = T->words;
  // PU words per thread and round trip (the input may be in host memory); a
  // domain of at most PU x PBLOCK words stays in registers for the row list
  constexpr int PU = 3;
  const bool kept = D <= PU * PBLOCK;
  CT_G uint64_t* levelDom = s->levelDom;
  uint64_t din[PU], ld[PU];
  WordDesc wd[PU];
  for (int q0 = tid; q0 < D; q0 += PU * PBLOCK) {
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int q = min(q0 + u * PBLOCK, D - 1);
      if (u == 0 || D > u * PBLOCK) {
        if (!MODEL) din[u] = (J.flags & JF_INLINE_DOM) ? a.inl[q] : J.dom_in[q];
        wd[u] = words[q];
        ld[u] = last[q];
      }
    }
    if (MODEL) {
      // the table runs if the round before removed a value of one of its
      // variables (first round: if the pool lacks a value of its domains)
      int pw[PU];
      uint64_t pv[PU];
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (u == 0 || D > u * PBLOCK) pw[u] = ((const CT_G int32_t*)J.dom_in)[min(q0 + u * PBLOCK, D - 1)];
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (u == 0 || D > u * PBLOCK) {
          din[u] = M.cur[pw[u]];
          pv[u] = M.prev[pw[u]];
        }
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (u == 0 || D > u * PBLOCK) {
          if (M.round ? din[u] != pv[u] : (ld[u] & ~din[u]) != 0) sh.dirty = 1;
          din[u] &= ld[u];
        }
    }
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int q = q0 + u * PBLOCK;
      if (q < D) {
        const int used = wd[u].v.dsize - 64 * (q - wd[u].v.domOff);
        if (used < 64 && (din[u] >> used) != 0) sh.stray = 1;
        if (!root && (din[u] & ~ld[u])) sh.notSub = 1;
        dinW[q] = din[u];
        for (int k = 0; k < J.nPush; ++k) levelDom[(int64_t)(depth + k) * D + q] = ld[u];
        atomicAdd(&sh.size[wd[u].var], __popcll(din[u]));
        if (!root) atomicAdd(&sh.dcnt[wd[u].var], __popcll(ld[u] & ~din[u]));
      }
    }
  }
  s_lds_barrier();
  if (MODEL) {
    if (!sh.dirty) return;
    if (tid == 0) atomicAdd((int32_t*)&M.state->props[(job % MODEL_PROPS) * 16], 1);
  }
  if (tid < WAVE) {
    const int policy = T->policy;
    int nrows = 0, nseg = 0;
    bool zero = false;
    for (int i0 = 0; i0 < n; i0 += WAVE) {
      const int i = i0 + lane;
      int cnt = 0, inc = 0;
      bool in = false;
      if (i < n) {
        const int sz = sh.size[i], dc = sh.dcnt[i];
        in = root || dc > 0;  // |dom| changed since the last call: in s_val
        inc = root ? 0 : policy == 2 ? 1 : policy == 1 ? 0 : (dc < sz ? 1 : 0);
        cnt = in ? (inc ? dc : sz) : 0;
        if (in && !inc && sz == 0) zero = true;  // the OR over an empty domain
      }
      const int sc = s_scan(cnt);
      if (i < n) {
        sh.seg[i] = in ? nrows + sc - cnt : -1;
        sh.inc[i] = inc;
      }
      nrows += __builtin_amdgcn_readlane(sc, WAVE - 1);
      nseg += __popcll(__ballot(in));
    }
    const bool anyZero = __ballot(zero) != 0ull;
    if (lane == 0) {
      sh.status = failed ? ST_STATE : sh.stray ? ST_INVALID : sh.notSub ? ST_NOT_SUBSET : ST_OK;
      sh.noop = nseg == 0 && !fromRoot;
      sh.zero = anyZero;
      sh.nrows = nrows;
    }
  }
  s_lds_barrier();
  const int status = sh.status, noop = sh.noop, nrows = sh.nrows;
  if (status != ST_OK) {
    // rejected: nothing changes, but a job that resets its slot to the root
    // still does
    if (fromRoot) {
      for (int64_t w = tid; w < T->stride; w += PBLOCK) s->ct[w] = T->ct0[w];
      for (int p = tid; p < nGran; p += PBLOCK) s->idx[0][p] = T->idx0[p];
      for (int q = tid; q < D; q += PBLOCK) s->lastDom[q] = T->dom0[q];
    }
    if (tid == 0) {
      if (fromRoot) {
        s->cur = 0;
        s->limit = T->limit0;
        s->failed = T->rootFailed;
        s->depth = 0;
        s->trailTop = 0;
        s->serial = J.serialBase;
      }
      rec->run = 0;
      put_status(J.flags, J.ll, J.seq, J.status_out, status);
      if (MODEL) M.state->fail = (M.round + 1) << 2 | 2;
    }
    return;
  }
  // the row list: segments in variable order, a variable's words in order, so
  // a word's first entry is the prefix sum of the selected bits before it;
  // longer lists than the job's room are not written (the update then walks
  // the selected bits)
  const bool list = nrows <= J.listCap;
  int base = 0;
  // PBLOCK words from q - tid: x the input, y the previous word
  auto put_words = [&](int q, uint64_t x, uint64_t y, int var, int rowStart, int domOff) {
    uint64_t bits = 0;
    int seg = -1, inc = 0;
    if (q < D) {
      seg = sh.seg[var];
      inc = sh.inc[var];
      if (seg >= 0) bits = inc ? (y & ~x) : x;
      // bits mode: 1 << 29 a variable not in s_val, 1 << 30 an incremental one
      sizeW[q] = sh.size[var] | (seg < 0 ? 1 << 29 : inc && q == domOff ? 1 << 30 : 0);
    }
    if (noop || nrows == 0) return;
    if (!list) {
      if (q < D) ((CT_G uint64_t*)rows)[q] = bits;  // (the list's room holds at least D words)
      return;
    }
    int tot = 0;
    int off = base + prep_scan<PWAVES>(__popcll(bits), &tot, sh);
    base += tot;
    const int row0 = rowStart + (q - domOff) * 64;
    while (bits) {
      const int b = __ffsll((unsigned long long)bits) - 1;
      bits &= bits - 1;
      rows[off] = (uint32_t)(row0 + b) | (off == seg ? SEG_FIRST | (inc ? SEG_INC : 0u) : 0u);
      // padding: the last row again (OR-ing it twice changes nothing)
      if (off == nrows - 1)
        for (int k = nrows; k & (ROW_U - 1); ++k) rows[k] = (uint32_t)(row0 + b);
      ++off;
    }
  };
  if (kept) {
#pragma unroll
    for (int u = 0; u < PU; ++u)
      if (u * PBLOCK < D)
        put_words(u * PBLOCK + tid, din[u], ld[u], wd[u].var, wd[u].v.rowStart, wd[u].v.domOff);
  } else {
    for (int q0 = 0; q0 < D; q0 += PBLOCK) {
      const int q = min(q0 + tid, D - 1);  // (dinW: this thread's own store, or not used)
      put_words(q0 + tid, dinW[q], last[q], words[q].var, words[q].v.rowStart, words[q].v.domOff);
    }
  }
  StageRec R = {};
  R.run = 1;
  R.flags = J.flags;
  R.mode = noop ? STAGE_NOOP : sh.zero ? STAGE_ZERO : list ? STAGE_LIST : STAGE_BITS;
  R.nrows = noop ? 0 : nrows;
  R.limit = limit;
  R.serial = serial;
  // levels exist only above depth 0: nothing is saved at depth 0
  // (only a root's list is long enough, and only those items are counted so)
  R.parts = (J.flags & (JF_ROOT | JF_FROM_ROOT)) == (JF_ROOT | JF_FROM_ROOT) && R.mode == STAGE_LIST
                ? stage_parts(nrows) : 1;
  R.trailOn = fromRoot || root || J.depthAfter <= 0 || noop ? STAGE_TRAIL_OFF
              : J.nPush > 0 ? STAGE_TRAIL_ALL : STAGE_TRAIL_FIRST;
  R.D = D;
  R.nGran = nGran;
  R.curNew = fromRoot ? 0 : 1 - cur;
  R.serialBase = J.serialBase;
  R.seq = J.seq;
  R.tab = T;
  R.slot = s;
  R.S = T->S;
  R.stride = T->stride;
  R.W = T->W;
  R.words = words;
  R.ctSrc = fromRoot ? T->ct0 : s->ct;
  R.idxSrc = fromRoot ? T->idx0 : s->idx[cur];
  R.idxDst = s->idx[R.curNew];
  R.ct = s->ct;
  R.stamp = s->stamp;
  R.nz = s->nzFlag;
  R.trailHdr = s->trailHdr;
  R.trailWords = s->trailWords;
  R.trailTop = trailTop;
  R.trailCap = s->trailCap;
  R.res = s->res;
  R.lastDom = s->lastDom;
  R.din = dinW;
  R.size = sizeW;
  R.rows = rows;
  R.dom_out = J.dom_out;
  R.ct_out = J.ct_out;
  R.status_out = J.status_out;
  R.ll = J.ll;
  if (MODEL) {
    R.poolMap = (const CT_G int32_t*)J.dom_in;
    R.poolCur = M.cur;
    R.poolNext = M.next;
    R.model = M.state;
    R.round = M.round;
  }
  if (tid == 0) {
    *rec = R;
    if (A.items) {
      // update items: SWAVES granule positions each (all of them when the
      // inactive ones are written too); finish items: the partition, then
      // FIN_WORDS domain words each
      const int pos = fromRoot || J.ct_out ? nGran : limit;
      const int nU = A.roots ? 0 : (pos * R.parts + SWAVES - 1) / SWAVES, nF = 1 + (D + FIN_WORDS - 1) / FIN_WORDS;
      const int l = job % STAGE_LISTS;
      const unsigned long long at = atomicAdd((unsigned long long*)&A.count->n[l * STAGE_LINE],
                                              (unsigned long long)(uint32_t)nF << 32 | (uint32_t)nU);
      sh.u0 = l * A.uCap + (int)(uint32_t)at;
      sh.f0 = l * A.fCap + (int)(at >> 32);
      sh.nU = nU;
      sh.nF = nF;
    }
  }
  if (!A.items) return;
  s_lds_barrier();
  const int u0 = sh.u0, f0 = sh.f0, nU = sh.nU, nF = sh.nF;
  for (int k = tid; k < nU; k += PBLOCK) A.items[u0 + k] = StageItem{job, k};
  for (int k = tid; k < nF; k += PBLOCK) A.fItems[f0 + k] = StageItem{job, k};
}

// The lists' items as one sequence: lane l < STAGE_LISTS has the items before
// list l.
struct ItemLists {
  int before, total;
};

__device__ __forceinline__ ItemLists item_lists(int n) {
  ItemLists L;
  const int c = s_lane() < STAGE_LISTS ? n : 0;
  const int x = s_scan(c);
  L.before = x - c;
  L.total = __builtin_amdgcn_readlane(x, WAVE - 1);
  return L;
}

// Item i of the sequence: its place in the item array.
__device__ __forceinline__ int item_at(const ItemLists& L, int i, int cap) {
  const int l = __popcll(__ballot(s_lane() < STAGE_LISTS && L.before <= i)) - 1;
  return l * cap + i - __builtin_amdgcn_readlane(L.before, l);
}

__device__ __forceinline__ void stage_update_item(const StageArgs& A, int job, int chunk, SplitShared& sh) {
  const StageRec R = load_rec(A, job);
  if (!R.run) return;
  const int at = chunk * SWAVES + s_wave(), parts = R.parts;
  stage_granule(A, R, &A.rec[job].trailCount, at / parts, at % parts, parts, sh);
}

__global__ void __launch_bounds__(SBLOCK, 8) stage_update_kernel(StageArgs A) {
  __shared__ SplitShared sh;
  if (!A.items) {
    stage_update_item(A, 0, blockIdx.x, sh);
    return;
  }
  const ItemLists L = item_lists((int)(uint32_t)A.count->n[min(s_lane(), STAGE_LISTS - 1) * STAGE_LINE]);
  if (blockIdx.x == 0 && threadIdx.x < STAGE_LISTS)  // (the finish empties the counts)
    A.count->fin[threadIdx.x] = (int32_t)(A.count->n[threadIdx.x * STAGE_LINE] >> 32);
  for (int i = blockIdx.x; i < L.total; i += gridDim.x) {
    const CT_K StageItem* it = (const CT_K StageItem*)A.items + item_at(L, i, A.uCap);
    stage_update_item(A, it->job, it->chunk, sh);
    s_lds_barrier();  // (the parts' words are read)
  }
}

// ---------------------------------------------------------------------------
// Update of a large launch of root jobs (stage_stream_roots): a wave per granule
// streams the rows of the input's values, ROOT_U in flight, reading nothing
// else (no row list, no old words).  A workgroup's four waves take adjacent
// granules, 2 KB of every row.  The items lie in the order of the jobs, which
// the host sorts by support rows, so the longest waves start first and a
// table's granules spread over the XCDs.
// Bound: HBM.  2,000 tables of up to 500,000 tuples, 1.8 GB: 315 us, 5.7 TB/s;
// with row lists shared by a granule's waves 350; in the order in which the
// preps end 342.
// ---------------------------------------------------------------------------
constexpr int ROOT_U = 4;

__global__ void __launch_bounds__(SBLOCK, 8) stage_root_kernel(StageArgs A) {
  if (blockIdx.x == 0 && threadIdx.x < STAGE_LISTS)  // (the finish empties the counts)
    A.count->fin[threadIdx.x] = (int32_t)(A.count->n[threadIdx.x * STAGE_LINE] >> 32);
  const CT_K StageItem* it = (const CT_K StageItem*)A.items + blockIdx.x;
  const CT_K StageRec* R = (const CT_K StageRec*)(A.rec + it->job);
  const int g = it->chunk * SWAVES + s_wave();
  if (!R->run || g >= R->nGran) return;
  const unsigned lane = (unsigned)s_lane();
  const TabDesc* T = (const TabDesc*)R->tab;
  const CT_K VarDesc* vars = (const CT_K VarDesc*)T->vars;
  const CT_K uint64_t* din = (const CT_K uint64_t*)R->din;
  const int n = T->n;
  const int64_t stride = R->stride, w0 = (int64_t)g * GW;
  uint64_t m = all_tuples(T, w0 + lane);
  for (int i = 0; i < n; ++i) {
    const VarDesc v = vars[i];
    uint64_t acc = 0ull;
    for (int k = 0; k < v.domWords; ++k) {
      uint64_t bits = din[v.domOff + k];
      const CT_G uint64_t* rows = R->S + (int64_t)(v.rowStart + 64 * k) * stride + w0;
      int b = 0;
      while (bits) {
        uint64_t x[ROOT_U];
#pragma unroll
        for (int u = 0; u < ROOT_U; ++u) {
          if (bits) {  // past the last value: the previous row again
            b = __ffsll((unsigned long long)bits) - 1;
            bits &= bits - 1;
          }
          x[u] = __builtin_nontemporal_load(rows + (int64_t)b * stride + lane);
        }
#pragma unroll
        for (int u = 0; u < ROOT_U; ++u) acc |= x[u];
      }
    }
    m &= acc;
    if (__ballot(m != 0ull) == 0ull) break;
  }
  R->ct[w0 + lane] = m;
  if (R->ct_out && w0 + lane < R->W) R->ct_out[w0 + lane] = m;
  const bool nz = __ballot(m != 0ull) != 0ull;
  if (lane == 0) R->nz[g] = nz ? 1 : 0;
}

// Device-clock duration of the three launches: first prep workgroup's start
// to the last finish workgroup's end.
__device__ void stage_clock_end(unsigned long long* clock) {
  atomicMax(&clock[1], wall_clock64());
  __threadfence();
  if (atomicAdd(&clock[2], 1ull) == gridDim.x - 1) {
    const unsigned long long t0 = atomicOr(&clock[0], 0ull), t1 = atomicOr(&clock[1], 0ull);
    atomicAdd(&clock[3], t1 > t0 ? t1 - t0 : 0ull);
    atomicAdd(&clock[4], 1ull);
    clock[0] = ~0ull;
    clock[1] = 0ull;
    clock[2] = 0ull;
    __threadfence();
  }
}

template <int FBLOCK>
__global__ void __launch_bounds__(FBLOCK) stage_finish_kernel(StageArgs A) {
  __shared__ FinShared<FBLOCK> sh;
  if (!A.items) {
    stage_finish_item(A, 0, blockIdx.x, sh);
    if (A.clock) {
      __syncthreads();
      if (threadIdx.x == 0) stage_clock_end(A.clock);
    }
    return;
  }
  const ItemLists L = item_lists(A.count->fin[min(s_lane(), STAGE_LISTS - 1)]);
  if (blockIdx.x == 0 && threadIdx.x < STAGE_LISTS) A.count->n[threadIdx.x * STAGE_LINE] = 0ull;
  for (int i = blockIdx.x; i < L.total; i += gridDim.x) {
    const CT_K StageItem* it = (const CT_K StageItem*)A.fItems + item_at(L, i, A.fCap);
    stage_finish_item(A, it->job, it->chunk, sh);
    s_lds_barrier();
  }
}

int stage_grid() {
  static int cached = 0;
  if (cached) return cached;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 256;
  cached = 8 * cus;
  return cached;
}

}  // namespace

int stage_row_pad() { return ROW_U; }
// (rows: at most as many are selected; 0 for a job that is no root)
int stage_update_items(int nGran, int rows) { return (nGran * stage_parts(rows) + SWAVES - 1) / SWAVES; }
// A launch with more finish items than CUs keeps the small workgroups: 1,024 threads for four words leave one workgroup on a
// CU (roots of 400 tables: the finish 20 us against 12; 128 searches 9 against
// 11).
bool stage_wide_launch(bool wide, int nF) { return wide && nF <= stage_grid() / 8; }
// A launch of roots streams from half as many granules as waves run at once
// (mixes of tables of up to 500,000 tuples, a tenth of the values removed:
// 4,891 granules 123 us against 128, 10,102 195 against 222, 8,033 of large
// tables 150 against 176; 3,643 96 against 92, 1,039 79 against 50).
bool stage_stream_roots(int64_t granules) { return granules >= (int64_t)stage_grid() * SWAVES / 2; }
bool stage_wide_dom(int D) { return D > PREP_WIDE_D; }
bool stage_wide(int nGran) { return nGran > FIN_WIDE_GRAN; }
int stage_finish_items(int D) { return 1 + (D + FIN_WORDS - 1) / FIN_WORDS; }

namespace {

// The prep of a.nJobs jobs (a.jobs, or the one of the arguments; MODEL: of a
// model's round); popGran: granules of the largest table that pops.
template <bool MODEL>
void launch_prep(const KArgs& a, const StageArgs& A, const ModelRound& M, int popGran, hipStream_t stream) {
  const size_t lds = sizeof(int32_t) * (size_t)popGran;
  const int np = a.nJobs + (MODEL ? M.nHead : 0);
  const int cus = stage_grid() / 8;
  if (a.nJobs > 3 * cus && !A.wideDom)
    hipLaunchKernelGGL((stage_prep_kernel<PBLOCK_MOST, MODEL>), dim3(np), dim3(PBLOCK_MOST), lds, stream, a, A, M);
  else if (a.nJobs > cus && !A.wideDom)
    hipLaunchKernelGGL((stage_prep_kernel<PBLOCK_MANY, MODEL>), dim3(np), dim3(PBLOCK_MANY), lds, stream, a, A, M);
  else
    hipLaunchKernelGGL((stage_prep_kernel<PMAX, MODEL>), dim3(np), dim3(PMAX), lds, stream, a, A, M);
}

// The update and the finish; nU / nF: at most this many items.  sparse: most of
// a launch's items are not there (a model's clean tables), so its workgroups
// are those that run at once and walk the lists; otherwise a workgroup each
// (1,500 roots, 1.28 GB: the update 246 us against 258).
void launch_items(const StageArgs& A, int nU, int nF, bool sparse, hipStream_t stream) {
  if (nF <= 0) return;
  const int gu = A.items ? std::min(std::max(nU, 1), sparse ? stage_grid() : 1 << 20) : nU;
  if (A.roots) hipLaunchKernelGGL(stage_root_kernel, dim3(gu), dim3(SBLOCK), 0, stream, A);
  else hipLaunchKernelGGL(stage_update_kernel, dim3(gu), dim3(SBLOCK), 0, stream, A);
  if (A.wide) {
    const int gf = A.items ? std::min(nF, stage_grid() / 4) : nF;
    hipLaunchKernelGGL(stage_finish_kernel<1024>, dim3(gf), dim3(1024), 0, stream, A);
  } else {
    const int gf = A.items ? std::min(nF, sparse ? stage_grid() : 1 << 20) : nF;
    hipLaunchKernelGGL(stage_finish_kernel<256>, dim3(gf), dim3(256), 0, stream, A);
  }
}

}  // namespace

hipError_t launch_staged(const KArgs& a, const StageArgs& A, int nU, int nF, int popGran, hipStream_t stream) {
  launch_prep<false>(a, A, ModelRound{}, popGran, stream);
  launch_items(A, nU, nF, false, stream);
  return hipGetLastError();
}

// The finish of one job whose record A.rec holds.
hipError_t launch_staged_finish(const StageArgs& A, int nF, hipStream_t stream) {
  if (A.wide) hipLaunchKernelGGL(stage_finish_kernel<1024>, dim3(nF), dim3(1024), 0, stream, A);
  else hipLaunchKernelGGL(stage_finish_kernel<256>, dim3(nF), dim3(256), 0, stream, A);
  return hipGetLastError();
}

hipError_t launch_model_start(const ModelRound& M, const uint64_t* poolIn, const int32_t* off,
                              const uint64_t* const* src, hipStream_t stream) {
  hipLaunchKernelGGL(model_start_kernel, dim3((8 * M.poolWords + SBLOCK - 1) / SBLOCK), dim3(SBLOCK), 0, stream, poolIn,
                     (uint64_t*)M.cur, off, src, M.poolWords, (ModelState*)M.state);
  return hipGetLastError();
}

// A round's prep, and what follows it.
hipError_t launch_model_prep(const KArgs& a, const StageArgs& A, const ModelRound& M, hipStream_t stream) {
  launch_prep<true>(a, A, M, 0, stream);
  return hipGetLastError();
}

hipError_t launch_model_items(const StageArgs& A, const ModelRound& M, int nU, int nF, const ModelNeg& neg,
                              hipStream_t stream) {
  if (neg.a.nJobs > 0) {
    const DevJob* jobs = (const DevJob*)neg.a.jobs;
    hipLaunchKernelGGL(model_neg_gather_kernel, dim3(neg.a.nJobs), dim3(SBLOCK), 0, stream, jobs, neg.maps, neg.dirty, M);
    const hipError_t e = launch_propagate(neg.a, std::min(neg.a.nJobs, propagate_max_grid()), stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(model_neg_merge_kernel, dim3(neg.a.nJobs), dim3(SBLOCK), 0, stream, jobs, neg.maps, neg.dirty, M);
  }
  launch_items(A, nU, nF, true, stream);
  return hipGetLastError();
}

}  // namespace ctk
