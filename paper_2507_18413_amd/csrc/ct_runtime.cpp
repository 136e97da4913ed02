// ct_runtime.cpp -- host runtime and C ABI of the CT library (include/ct.h).
//
// Owns device memory, streams and the host-side mirror of each slot's depth.
// Every step of propagation runs in the HIP kernels of ct_kernels.hip; the
// host only validates arguments, lays out job descriptors and moves the
// domain bitmaps across the boundary.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "ct.h"
#include "ct_device.h"

using namespace ctk;

namespace ctk {
int propagate_items_per_job_update(int nGran);
int propagate_items_per_job_filter(int D);
int propagate_max_grid();
hipError_t launch_propagate(const KArgs& a, int grid, hipStream_t stream);
size_t engine_lds_bytes(int n, int D, int nGran, int rows);
hipError_t launch_engine(const EngDesc& D, size_t lds, hipStream_t stream);
hipError_t launch_split_engine(const EngDesc& E, int grid, hipStream_t stream);
int stage_row_pad();
int stage_update_items(int nGran, int rows);
bool stage_wide(int nGran);
bool stage_wide_dom(int D);
bool stage_wide_launch(bool wide, int nF);
bool stage_stream_roots(int64_t granules);
int stage_finish_items(int D);
hipError_t launch_staged(const KArgs& a, const StageArgs& A, int nU, int nF, int popGran, hipStream_t stream);
int nodes_max_vec_rows(size_t lds);
size_t nodes_scratch_bytes(int vecRows, int nJobs, int nGran);
size_t nodes_ids_bytes(int n, int64_t stride);
hipError_t launch_nodes_ids(const TabDesc* T, int nGran, uint16_t* ids, hipStream_t stream);
hipError_t launch_nodes(NodesDesc N, char* scratch, hipStream_t stream);
hipError_t noalloc_scratch(char** ptr, size_t* bytes);
int slots_alloc(ct_table* T, int32_t n, int32_t max_depth, bool search, int32_t* first_slot);
hipError_t launch_build_supports(const BuildArgs& B, hipStream_t stream);
hipError_t launch_init_root(TabDesc* T, SlotDesc* root, const uint64_t* dom0, int64_t words, hipStream_t stream);
hipError_t launch_init_first(TabDesc* T, SlotDesc* slot, SlotDesc* root, const uint64_t* dom0, const int32_t* star,
                             int32_t* out, int64_t words, hipStream_t stream);
hipError_t launch_staged_finish(const StageArgs& A, int nF, hipStream_t stream);
hipError_t launch_init_slots(const TabDesc* T, SlotDesc* slots, int n, const int32_t* rootRes,
                             hipStream_t stream);
}  // namespace ctk

namespace {

// the calling thread's last error message, in a fixed buffer: reporting an
// error allocates nothing
thread_local char g_err[512];

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define HIPCHK(expr)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return fail(CT_E_DEVICE, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_),       \
                  __FILE__, __LINE__);                                                      \
  } while (0)

constexpr int32_t kStatusPending = 0x7fff0001;

// device-side errors of ct_propagate_batch_noalloc calls on `stream`
int noalloc_status(hipStream_t stream);

// Injected allocation failure (a test hook): the g_failAlloc-th allocation
// from now fails.
std::atomic<int32_t> g_failAlloc{0};

bool alloc_injected() {
  int32_t n = g_failAlloc.load();
  while (n > 0)
    if (g_failAlloc.compare_exchange_weak(n, n - 1)) return n == 1;
  return false;
}

// A device or pinned host allocation: CT_E_NOMEM when it fails (or when
// the injected failure fires on it).
#define ALLOCCHK(expr)                                                                      \
  do {                                                                                      \
    if (alloc_injected()) return fail(CT_E_NOMEM, "injected allocation failure: %s", #expr); \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) {                                                                 \
      (void)hipGetLastError();                                                              \
      return fail(CT_E_NOMEM, "%s failed: %s", #expr, hipGetErrorString(e_));              \
    }                                                                                       \
  } while (0)

// failed flag as known on the host: 0 no, 1 yes, 2 unknown (after batches)
struct SlotHost {
  SlotDesc* dev = nullptr;
  int maxDepth = 0;
  int capDepth = 0;        // levels the slot's device trail was sized for
  bool freed = false;      // released by ct_slots_free (reused by ct_slots_alloc)
  int depth = 0;           // depth including pending operations
  int pendPop = 0, pendPush = 0;
  int8_t failed = 0;
  std::vector<int8_t> failedAt;  // failed flag recorded by each push
  uint64_t batchMark = 0;        // last batch that named this slot
};

struct DevBlock {
  void* ptr = nullptr;
};

// What a table's own launches need (a model walks its tables several times a
// step: nothing else in here).
struct TableQueue {
  int32_t* queue = nullptr;   // on the device: [3] error word
  int32_t* hostErr = nullptr; // pinned
  // staged schedule scratch (see StageNeed)
  char* dStaged = nullptr;
  size_t capStaged = 0;
};

// Device queue + staging for one stream.
struct QueueCtx : TableQueue {
  // batch staging: job descriptors, in two pinned buffers in turn.  Batches
  // fill a buffer one after the other; its event, recorded when it is full,
  // says that their descriptors have been read.  (An event behind every batch
  // costs the stream 4.6 us: a push and a pop batch of one job 32 us with it,
  // 23 without.)
  char* dStage = nullptr;
  char* pStage[2] = {nullptr, nullptr};
  char* pStageDev[2] = {nullptr, nullptr};  // their device addresses
  hipEvent_t staged[2] = {nullptr, nullptr};
  size_t capStage = 0, usedStage = 0;       // bytes of a buffer; used of the one in turn
  int turn = 0;
  // host scratch of a batch, kept between batches (no allocation per call)
  std::vector<DevJob> hJobs;
  std::vector<int32_t> chunks;
  std::vector<uint64_t> order;
  // search-node schedule scratch (node records | row vectors | non-zero words)
  void* dNodes = nullptr;
  size_t capNodes = 0;
};

int queue_init(QueueCtx& q) {
  ALLOCCHK(hipMalloc(&q.queue, 4 * sizeof(int32_t)));
  HIPCHK(hipMemset(q.queue, 0, 4 * sizeof(int32_t)));
  ALLOCCHK(hipHostMalloc((void**)&q.hostErr, sizeof(int32_t), hipHostMallocMapped | hipHostMallocCoherent));
  *q.hostErr = 0;
  for (int k = 0; k < 2; ++k) HIPCHK(hipEventCreateWithFlags(&q.staged[k], hipEventDisableTiming));
  return CT_OK;
}

void queue_free(QueueCtx& q) {
  if (q.queue) (void)hipFree(q.queue);
  if (q.hostErr) (void)hipHostFree(q.hostErr);
  if (q.dStage) (void)hipFree(q.dStage);
  for (int k = 0; k < 2; ++k) {
    if (q.pStage[k]) (void)hipHostFree(q.pStage[k]);
    if (q.staged[k]) (void)hipEventDestroy(q.staged[k]);
  }
  if (q.dNodes) (void)hipFree(q.dNodes);
  if (q.dStaged) (void)hipFree(q.dStaged);
  q = QueueCtx();
}

std::mutex g_qmu;
std::map<hipStream_t, QueueCtx*> g_queues;

}  // namespace

// A table's share of a staged launch.
struct StageShape {
  int nU = 0, nURoot = 0, nF = 0;  // (nURoot: a batch's root job)
  bool wide = false, wideDom = false;
  size_t bytes = 0;
};

struct ct_table {
  // the fields every call reads first, together (a batch of thousands of
  // jobs touches them for every table)
  int n = 0;
  int64_t t = 0, W = 0, stride = 0;
  int rows = 0, D = 0, nGran = 0;
  ct_config cfg{};
  TabDesc* dTab = nullptr;
  std::vector<SlotHost> slots;
  int32_t serialCounter = 1;
  StageShape stage;
  bool poisoned = false;
  bool tailPending = false;  // a synchronous call returned before its kernel ended
  bool engEligible = false, engOn = false;
  int kind = CT_KIND_POSITIVE;  // CT_KIND_POSITIVE or CT_KIND_NEGATIVE
  bool shortTab = false;        // a positive table with star cells
  int rootFailed = 0;
  hipStream_t stream = nullptr;
  uint64_t batchMark = 0;    // last batch that named this table
  hipStream_t pendStream = nullptr;  // a model's stream holding queued work on slot 0
  std::vector<int32_t> lo, dsz, domOff;
  std::vector<VarDesc> vars;
  std::vector<int32_t> wordVar;
  // device
  uint64_t* dS = nullptr;
  VarDesc* dVars = nullptr;
  int32_t* dWordVar = nullptr;
  WordDesc* dWords = nullptr;
  int32_t* dLo = nullptr;
  TabDesc hTab{};
  SlotDesc* dRoot = nullptr;
  SlotDesc hRoot{};
  // search-node schedule: row vectors of a batch (0: the table does not take
  // it) and the row numbers of every tuple's values (see nodes_ids_ensure)
  int nodesVecRows = 0;
  uint16_t* dIds = nullptr;
  std::vector<void*> blocks;  // device allocations to free
  TableQueue q;               // (queue, hostErr: parts of other blocks)
  // pinned staging of the synchronous calls, parts of one block
  char* pBlock = nullptr;
  uint64_t* pDomOut = nullptr;  // D words
  uint64_t* pLL = nullptr;      // result slots of flagged synchronous jobs (2 + 2D)
  uint64_t* pDomIn = nullptr;   // D words (used when D > INLINE_WORDS)
  uint64_t* pCt = nullptr;      // W words (lazily)
  int32_t* pStatus = nullptr;
  // optional kernel timing of synchronous launches, on the device clock
  // (no host events: they would add dispatch packets to every call)
  unsigned long long* dClock = nullptr;  // 5 words, see KArgs::clock
  bool timing = false;
  // resident engine of slot 0 (see ct_engine.hip; engEligible, engOn above)
  size_t engLds = 0;
  hipStream_t engStream = nullptr;
  EngCmd* pCmd = nullptr;   // coherent pinned mailbox
  EngRes* pRes = nullptr;
  int32_t engSeq = 0;  // call numbers of the mailbox and of flagged launched calls (one sequence)
  bool engSplit = false;    // the running engine is the resident split schedule
  int32_t* dCtl = nullptr;  // its control words (SE_CTL_WORDS)
  int seVarWords = -1;      // largest domain words of one variable (computed once)
  std::vector<uint64_t> engDom;        // the last call's output domains (D words)
  unsigned long long engStats[8] = {};  // the slot's counters after the last call
  bool engStatsFresh = false;  // engStats is from the last call
  unsigned long long engTicks = 0, engCalls = 0;  // timing of engine calls
  // lifetimes of the engine launches started while timing was on
  bool engTimed = false;
  unsigned long long engLifeTicks = 0, engLaunches = 0;
};

namespace {

int dev_alloc(ct_table* T, void** p, size_t bytes) {
  if (bytes == 0) bytes = 8;
  if (alloc_injected()) return fail(CT_E_NOMEM, "injected allocation failure: hipMalloc(%zu)", bytes);
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(CT_E_NOMEM, "hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
  }
  T->blocks.push_back(*p);
  return CT_OK;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Allocate n slot descriptors and their arrays in one device block.
int alloc_slots(ct_table* T, int n, int maxDepth, SlotDesc** dSlots, std::vector<SlotDesc>& h) {
  const size_t ctB = align256(sizeof(uint64_t) * T->stride);
  const size_t idxB = align256(sizeof(int32_t) * T->nGran);
  const size_t domB = align256(sizeof(uint64_t) * T->D);
  const size_t resB = align256(sizeof(int32_t) * T->rows);
  const int64_t trailCap = (int64_t)maxDepth * T->nGran;
  const size_t thB = align256(sizeof(TrailHdr) * std::max<int64_t>(trailCap, 1));
  const size_t twB = align256(sizeof(uint64_t) * GW * std::max<int64_t>(trailCap, 1));
  const size_t lvB = align256(sizeof(Level) * std::max(maxDepth, 1));
  const size_t ldB = align256(sizeof(uint64_t) * T->D * std::max(maxDepth, 1));
  const size_t per = ctB + 4 * idxB + domB + resB + thB + twB + lvB + ldB;
  const size_t descB = align256(sizeof(SlotDesc) * n);
  char* base = nullptr;
  int rc = dev_alloc(T, (void**)&base, descB + per * (size_t)n);
  if (rc != CT_OK) return rc;
  *dSlots = (SlotDesc*)base;
  h.assign(n, SlotDesc{});
  char* p = base + descB;
  for (int k = 0; k < n; ++k) {
    SlotDesc& s = h[k];
    s.ct = (uint64_t*)p; p += ctB;
    s.idx[0] = (int32_t*)p; p += idxB;
    s.idx[1] = (int32_t*)p; p += idxB;
    s.stamp = (int32_t*)p; p += idxB;
    s.nzFlag = (int32_t*)p; p += idxB;
    s.lastDom = (uint64_t*)p; p += domB;
    s.res = (int32_t*)p; p += resB;
    s.trailHdr = (TrailHdr*)p; p += thB;
    s.trailWords = (uint64_t*)p; p += twB;
    s.levels = (Level*)p; p += lvB;
    s.levelDom = (uint64_t*)p; p += ldB;
    s.trailCap = trailCap;
    s.maxDepth = maxDepth;
  }
  HIPCHK(hipMemcpyAsync(base, h.data(), sizeof(SlotDesc) * n, hipMemcpyHostToDevice, T->stream));
  return CT_OK;
}

int check_poison(const ct_table* T) {
  if (!T) return fail(CT_E_INVALID, "null table");
  if (T->poisoned) return fail(CT_E_DEVICE, "table handle poisoned by an earlier device error");
  return CT_OK;
}

constexpr int SOLO_MAX_GRAN = 4;      // tables up to 16,384 tuples run in one workgroup ...
constexpr int SOLO_MAX_D = 16;        // ... unless their filterDomains has more words than that takes at once
constexpr int NODES_MIN_BATCH = 64;   // AUTO: batches of root resets this large run granule-major

bool use_solo(const ct_table* T) {
  // a negative table's call filters and then removes the pruned values'
  // tuples, in one workgroup
  if (T->kind == CT_KIND_NEGATIVE || T->cfg.schedule == CT_SCHED_SOLO) return true;
  if (T->cfg.schedule == CT_SCHED_SPLIT) return false;
  return T->nGran <= SOLO_MAX_GRAN && T->D <= SOLO_MAX_D;
}

// Largest LDS of one workgroup on the current device (0 if unknown).
int device_lds() {
  int dev = 0, lds = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    return 0;
  return lds;
}

// Whether the search-node schedule pays for a batch of n jobs (AUTO).  It takes
// 5 us more than the staged launches and 0.6 us for each variable (a tuple's
// row numbers are read in turn), whatever the jobs remove; the staged update
// takes, for each granule of each job, 0.7 ns and 0.06 ns a support row it
// ORs, a fifth of the table's being what search nodes have removed at most
// (half a variable's values, on average of none to a few tenths).  Measured,
// search nodes / staged us: 100 variables of 20 values, 100,000 tuples, 64
// jobs 88 / 25; 6 of 20, 60,000, 256 jobs 37 / 24-29, 1,024 jobs 43 / 45-60,
// 400,000, 256 jobs 38 / 38-62; 16 of 60, 400,000, 64 jobs 37-70 / 25-184; 200
// of 3, 60,000, 1,024 jobs 195 / 150-225; 100 of 20, 400,000, 256 jobs 107 /
// 51-1,323.
bool nodes_pays(const ct_table* T, int n) {
  return (double)T->nGran * n * (7e-4 + 1.2e-5 * T->rows) >= 5 + 0.6 * T->n;
}

// The search-node schedule reads, per tuple, the row numbers of its values
// (2 bytes each).  They are made once per table, when its slots reach a batch
// for which the schedule pays (or at the first such batch): a table never
// searched that way does not pay for them.  Without memory for them the
// batches take the other schedules.
bool nodes_ids_ensure(ct_table* T) {
  if (T->dIds) return true;
  if (T->nodesVecRows == 0 || alloc_injected()) return false;
  void* p = nullptr;
  if (hipMalloc(&p, nodes_ids_bytes(T->n, T->stride)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (launch_nodes_ids(T->dTab, T->nGran, (uint16_t*)p, T->stream) != hipSuccess ||
      hipStreamSynchronize(T->stream) != hipSuccess) {
    (void)hipFree(p);
    return false;
  }
  T->blocks.push_back(p);
  T->dIds = (uint16_t*)p;
  return true;
}

// Batches whose jobs all recompute a root from scratch (their descriptors
// count the tasks of NA_ROOT_GRAN granules in a no-allocation batch's limit).
bool use_roots(const ct_job* jobs, int n) {
  for (int j = 0; j < n; ++j)
    if (jobs[j].flags != (CT_JOB_PROPAGATE | CT_JOB_ROOT) || jobs[j].table->cfg.schedule != CT_SCHED_AUTO ||
        jobs[j].table->kind != CT_KIND_POSITIVE)
      return false;
  return true;
}

// The search-node schedule can take a batch whose jobs all reset slots of one
// table to the root and propagate (the slots are distinct: checked before).
bool nodes_form(const ct_job* jobs, int n) {
  const ct_table* T = jobs[0].table;
  if (T->cfg.schedule != CT_SCHED_NODES && (T->cfg.schedule != CT_SCHED_AUTO || n < NODES_MIN_BATCH))
    return false;
  if (T->nodesVecRows == 0) return false;
  for (int j = 0; j < n; ++j)
    if (jobs[j].table != T || jobs[j].flags != (CT_JOB_PROPAGATE | CT_JOB_FROM_ROOT)) return false;
  return true;
}

bool nodes_batch(const ct_job* jobs, int n) {
  return nodes_form(jobs, n) && (jobs[0].table->cfg.schedule == CT_SCHED_NODES || nodes_pays(jobs[0].table, n));
}

// Staged schedule: what a job needs of a launch's scratch.  A launch's
// scratch holds the records of its jobs, the update items, the finish items,
// then each job's input words, |dom| words and row list.
constexpr int STAGE_LIST_CAP = 65536;  // row-list entries of a job (more: the update walks the selected bits)
constexpr size_t STAGE_BUFFER = (size_t)64 << 10;   // the least of a staging buffer: some ten batches of 60 jobs
constexpr size_t STAGE_SCRATCH = (size_t)64 << 20;  // a batch beyond it runs as several launches

int stage_list_cap(const ct_table* T) { return std::min(T->rows, STAGE_LIST_CAP); }

size_t stage_job_bytes(const ct_table* T) {
  const size_t list = sizeof(uint32_t) * ((size_t)stage_list_cap(T) + stage_row_pad());
  return align256(sizeof(uint64_t) * T->D + sizeof(int32_t) * ((T->D + 1) & ~1) +
                  std::max(list, sizeof(uint64_t) * (size_t)T->D));
}

// A table's share of a launch, computed once (batches of a thousand jobs add
// it up per call).
StageShape stage_shape(const ct_table* T) {
  StageShape S;
  S.nU = stage_update_items(T->nGran, 0);
  S.nURoot = stage_update_items(T->nGran, T->rows);
  S.nF = stage_finish_items(T->D);
  S.wide = stage_wide(T->nGran);
  S.wideDom = stage_wide_dom(T->D);
  S.bytes = stage_job_bytes(T);
  return S;
}

struct StageNeed {
  int nJobs = 0, nU = 0, nF = 0, popGran = 0;
  int u[STAGE_LISTS] = {}, f[STAGE_LISTS] = {};  // items per list
  int uCap = 0, fCap = 0;                        // the most of a list
  size_t jobBytes = 0;
  bool wide = false, wideDom = false;
  void add(const ct_table* T, bool propagate, bool pops, bool root = false) {
    if (pops) popGran = std::max(popGran, T->nGran);
    if (!propagate) {
      ++nJobs;
      return;
    }
    const StageShape& S = T->stage;
    jobBytes += S.bytes;
    wide = wide || S.wide;
    wideDom = wideDom || S.wideDom;
    add_items(root ? S.nURoot : S.nU, S.nF);
  }
  void add_items(int du, int df) {
    const int l = nJobs++ % STAGE_LISTS;
    nU += du;
    nF += df;
    uCap = std::max(uCap, u[l] += du);
    fCap = std::max(fCap, f[l] += df);
  }
  static size_t total(size_t jobs, size_t uc, size_t fc, size_t jb) {
    return align256(sizeof(StageCounts)) + align256(sizeof(StageRec) * jobs) +
           align256(sizeof(StageItem) * STAGE_LISTS * uc) + align256(sizeof(StageItem) * STAGE_LISTS * fc) + jb;
  }
  size_t bytes() const { return total(nJobs, uCap, fCap, jobBytes); }
  // the bytes with one more propagation of T
  size_t bytes_with(const ct_table* T, bool root = false) const {
    const StageShape& S = T->stage;
    const int l = nJobs % STAGE_LISTS;
    return total(nJobs + 1, std::max(uCap, u[l] + (root ? S.nURoot : S.nU)), std::max(fCap, f[l] + S.nF), jobBytes + S.bytes);
  }
};

// The launch's view of its scratch (count: the item counts are elsewhere).
StageArgs stage_args(const StageNeed& n, char* scratch, int32_t* queue, int32_t* hostErr,
                     StageCounts* count = nullptr) {
  StageArgs A{};
  A.count = count ? count : (StageCounts*)scratch;
  scratch += align256(sizeof(StageCounts));
  A.rec = (StageRec*)scratch;
  scratch += align256(sizeof(StageRec) * (size_t)n.nJobs);
  A.items = (StageItem*)scratch;
  scratch += align256(sizeof(StageItem) * STAGE_LISTS * (size_t)n.uCap);
  A.fItems = (StageItem*)scratch;
  scratch += align256(sizeof(StageItem) * STAGE_LISTS * (size_t)n.fCap);
  A.uCap = n.uCap;
  A.fCap = n.fCap;
  A.wide = stage_wide_launch(n.wide, n.nF);
  A.wideDom = n.wideDom;
  A.queue = queue;
  A.hostErr = hostErr;
  A.jobMem = scratch;
  return A;
}

int stage_reserve(TableQueue& q, size_t bytes, hipStream_t stream) {
  if (q.capStaged >= bytes) return CT_OK;
  HIPCHK(hipStreamSynchronize(stream));
  if (q.dStaged) (void)hipFree(q.dStaged);
  q.dStaged = nullptr;
  q.capStaged = 0;
  ALLOCCHK(hipMalloc((void**)&q.dStaged, bytes));
  HIPCHK(hipMemsetAsync(q.dStaged, 0, sizeof(StageCounts), stream));
  q.capStaged = bytes;
  return CT_OK;
}

// Run one job synchronously on the table's stream.
int quiesce(ct_table* T, hipStream_t same = nullptr);

uint64_t* pinned_dev64(ct_table* T, uint64_t* host);

// A synchronous call of a table whose update is one item of 8 granules and
// whose input fits the kernel arguments runs as one launch with hand-offs
// (measured 20-21 us a call against 21-22 us staged at 12,000 and 30,000 tuples);
// the others run staged (200,000 tuples: 22 against 27 us; 2,000,000: 26
// against 64; 307 domain words: 28 against 33; 1,105: 39 against 55).
bool stage_single(const ct_table* T) {
  return propagate_items_per_job_update(T->nGran) > 1 || T->D > INLINE_WORDS;
}

int run_single(ct_table* T, DevJob& J, const uint64_t* dom_in_host) {
  int qrc = quiesce(T);
  if (qrc) return qrc;
  KArgs a{};
  a.jobs = nullptr;
  a.nJobs = 1;
  const bool prop = J.flags & JF_PROPAGATE;
  if (prop && use_solo(T)) J.flags |= JF_SOLO;
  const bool solo = J.flags & JF_SOLO;
  const bool staged = prop && !solo && stage_single(T);
  J.nUpd = prop ? 1 : 0;
  J.nFilt = prop && !solo ? propagate_items_per_job_filter(T->D) : 0;
  a.nPrep = !prop || (!solo && J.nPop > 0) ? 1 : 0;
  J.flags |= JF_HOST_OUT;
  StageNeed need;
  StageArgs A{};
  if (staged) {
    need.add(T, true, J.nPop > 0);  // (the scratch is there: call_reserve)
    A = stage_args(need, T->q.dStaged, T->q.queue, T->q.hostErr);
    A.items = nullptr;  // one job: its items by workgroup
    J.listCap = stage_list_cap(T);
  }
  // a propagation answers through flagged slots; not with a currTable copy
  // that is not staged (that one keeps the fenced status), nor a negative
  // table of many domain words, whose one workgroup writes all the slots (7
  // words 26 us a call against 27 fenced, 18 words the same, 65 words 71
  // against 66, 200 words 60 against 30)
  constexpr int NEG_LL_D = 16;
  const bool ll = (J.flags & JF_PROPAGATE) && (staged || !J.ct_out) && T->pLL &&
                  (T->kind != CT_KIND_NEGATIVE || T->D <= NEG_LL_D);
  uint32_t sq = 0;
  if (ll) {
    J.flags |= JF_LL;
    J.seq = ++T->engSeq;
    if (J.seq == 0) J.seq = ++T->engSeq;  // (0 is the slots' initial flag)
    sq = (uint32_t)J.seq;
    if (!(J.ll = pinned_dev64(T, T->pLL))) return fail(CT_E_DEVICE, "no device address for the result slots");
  }
  a.nUpd = J.nUpd;
  a.nFilt = J.nFilt;
  a.queue = T->q.queue;
  a.hostErr = T->q.hostErr;
  if (dom_in_host) {
    if (T->D <= INLINE_WORDS) {
      memcpy(a.inl, dom_in_host, sizeof(uint64_t) * T->D);
      J.flags |= JF_INLINE_DOM;
    } else {
      memcpy(T->pDomIn, dom_in_host, sizeof(uint64_t) * T->D);
      uint64_t* dp = nullptr;
      HIPCHK(hipHostGetDevicePointer((void**)&dp, T->pDomIn, 0));
      J.dom_in = dp;
    }
  }
  a.job = J;
  const int total = a.nPrep + a.nUpd + a.nFilt;
  if (total == 0) return CT_OK;
  volatile int32_t* status = T->pStatus;
  *status = kStatusPending;
  a.clock = T->timing ? T->dClock : nullptr;
  if (staged) {
    A.clock = a.clock;
    HIPCHK(launch_staged(a, A, need.nU, need.nF, need.popGran, T->stream));
  } else {
    HIPCHK(launch_propagate(a, std::min(total, propagate_max_grid()), T->stream));
  }
  T->tailPending = true;
  if (ll) {
    // the status slot (a job that does not succeed) or every domain word
    const uint64_t* sl = T->pLL;
    const int nS = 2 * T->D;
    int got = 0;
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t spin = 0;; ++spin) {
      const uint64_t v = __atomic_load_n(&sl[0], __ATOMIC_ACQUIRE);
      if ((uint32_t)v == sq) {
        *status = (int32_t)(uint32_t)(v >> 32);
        break;
      }
      // (a wide table's slots are many lines the device has just written:
      // fetched ahead, they do not miss one after the other)
      while (got < nS && (uint32_t)__atomic_load_n(&sl[2 + got], __ATOMIC_ACQUIRE) == sq) {
        if ((got & 7) == 0) __builtin_prefetch(&sl[2 + std::min(got + 128, nS - 1)]);
        ++got;
      }
      if (got == nS) {
        for (int q = 0; q < T->D; ++q)
          T->pDomOut[q] = ((uint64_t)(uint32_t)(sl[3 + 2 * q] >> 32) << 32) | (uint32_t)(sl[2 + 2 * q] >> 32);
        *status = CT_OK;
        break;
      }
      if ((spin & 1023) == 1023 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) {
        hipError_t e = hipStreamSynchronize(T->stream);
        if (e != hipSuccess) {
          T->poisoned = true;
          return fail(CT_E_DEVICE, "kernel failed: %s", hipGetErrorString(e));
        }
        T->poisoned = true;
        return fail(CT_E_DEVICE, "kernel finished without a result (device error %d)", *T->q.hostErr);
      }
    }
    if (*T->q.hostErr) {
      T->poisoned = true;
      return fail(CT_E_DEVICE, "device-side error %d (wait timeout or trail overflow)", *T->q.hostErr);
    }
    return CT_OK;
  }
  // The job publishes its status (and its outputs before it) to coherent
  // host memory with a system-scope release: wait for that word instead of
  // the whole kernel.  The kernel's tail finishes on the stream, which
  // orders it before the next launch.
  const auto t0 = std::chrono::steady_clock::now();
  for (uint32_t spin = 0; *status == kStatusPending; ++spin) {
    if ((spin & 1023) == 1023 &&
        std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) {
      hipError_t e = hipStreamSynchronize(T->stream);
      if (e != hipSuccess) {
        T->poisoned = true;
        return fail(CT_E_DEVICE, "kernel failed: %s", hipGetErrorString(e));
      }
      if (*status == kStatusPending) {
        T->poisoned = true;
        return fail(CT_E_DEVICE, "kernel finished without a status (device error %d)", *T->q.hostErr);
      }
    }
  }
  if (*T->q.hostErr) {
    T->poisoned = true;
    return fail(CT_E_DEVICE, "device-side error %d (wait timeout or trail overflow)", *T->q.hostErr);
  }
  return CT_OK;
}

int ensure_pinned_ct(ct_table* T);

// ---------------------------------------------------------------------------
// resident engine of a table's slot 0 (one engine alive per process: each
// holds a hardware queue while it waits for calls)
// ---------------------------------------------------------------------------
std::mutex g_engMu;
ct_table* g_engOwner = nullptr;
std::set<ct_table*> g_tables;  // live tables (for ct_quiesce)
constexpr double kEngineIdleMs = 2.0;  // an engine without calls for this long exits

int64_t engine_idle_ticks() {
  int dev = 0, khz = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
    khz = 100000;
  return (int64_t)(kEngineIdleMs * khz);
}

// Waits for the engine of T to end (it has exited or was told to) and
// marks it stopped; its state is then back in the slot's device arrays.
int engine_join(ct_table* T) {
  const auto t0 = std::chrono::steady_clock::now();
  while (__atomic_load_n(&T->pRes->alive, __ATOMIC_ACQUIRE) != 0) {
    if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) break;
  }
  hipError_t e = hipStreamSynchronize(T->engStream);
  T->engOn = false;
  if (g_engOwner == T) g_engOwner = nullptr;
  if (e == hipSuccess && T->engTimed && T->timing) {
    T->engLifeTicks += T->pRes->lifeTicks;
    T->engLaunches += 1;
  }
  if (e != hipSuccess) {
    T->poisoned = true;
    return fail(CT_E_DEVICE, "engine failed: %s", hipGetErrorString(e));
  }
  return CT_OK;
}

// Writes a call into the mailbox: every command slot, flagged with the
// call's sequence number, the domain words first and the op last (the
// engine takes the call once all of them carry the number).
void engine_post(ct_table* T, int32_t seq, int32_t op, const DevJob* J, const uint64_t* dom_in, bool wantCt,
                 bool wantStats) {
  uint64_t* s = T->pCmd->slot;
  const uint32_t sq = (uint32_t)seq;
  for (int i = 0; i < 2 * T->D; ++i) {
    const uint32_t half = dom_in ? (uint32_t)(dom_in[i >> 1] >> (i & 1 ? 32 : 0)) : 0u;
    __atomic_store_n(&s[EC_DOM + i], eng_slot(half, sq), __ATOMIC_RELAXED);
  }
  const uint32_t hdr[EC_DOM] = {(uint32_t)op,
                                J ? (uint32_t)J->nPop : 0u,
                                J ? (uint32_t)J->nPush : 0u,
                                J ? (uint32_t)J->serialBase : 0u,
                                J ? (uint32_t)J->depthAfter : 0u,
                                wantCt ? 1u : 0u,
                                wantStats ? 1u : 0u,
                                0u};
  for (int i = EC_DOM - 1; i > 0; --i) __atomic_store_n(&s[i], eng_slot(hdr[i], sq), __ATOMIC_RELAXED);
  __atomic_store_n(&s[EC_OP], eng_slot(hdr[EC_OP], sq), __ATOMIC_RELEASE);
}

int engine_stop(ct_table* T) {
  if (!T || !T->engOn) return CT_OK;
  if (__atomic_load_n(&T->pRes->alive, __ATOMIC_ACQUIRE) != 0) engine_post(T, ++T->engSeq, ENG_OP_STOP, nullptr,
                                                                           nullptr, false, false);
  return engine_join(T);
}

bool engine_wanted(const ct_table* T);
bool split_engine_wanted(ct_table* T);

// What an engine of T needs, made once, before the first call that it serves
// takes the slot's pending operations (call_reserve).
int engine_reserve(ct_table* T) {
  if (!T->pCmd) {
    ALLOCCHK(hipHostMalloc((void**)&T->pCmd, sizeof(EngCmd), hipHostMallocMapped | hipHostMallocCoherent));
    memset((void*)T->pCmd, 0, sizeof(EngCmd));
  }
  if (!T->pRes) {
    ALLOCCHK(hipHostMalloc((void**)&T->pRes, sizeof(EngRes), hipHostMallocMapped | hipHostMallocCoherent));
    memset((void*)T->pRes, 0, sizeof(EngRes));
  }
  int rc = ensure_pinned_ct(T);
  if (rc) return rc;
  if (!T->dCtl && !engine_wanted(T)) {
    void* p = nullptr;
    ALLOCCHK(hipMalloc(&p, sizeof(int32_t) * SE_CTL_WORDS));
    T->blocks.push_back(p);
    T->dCtl = (int32_t*)p;
  }
  return CT_OK;
}

int engine_start(ct_table* T) {
  if (g_engOwner && g_engOwner != T) {
    int rc = engine_stop(g_engOwner);
    if (rc) return rc;
  }
  if (T->tailPending) {  // earlier launches on the slot end first
    HIPCHK(hipStreamSynchronize(T->stream));
    T->tailPending = false;
  }
  if (!T->engStream) HIPCHK(hipStreamCreateWithFlags(&T->engStream, hipStreamNonBlocking));
  EngDesc D{};
  D.tab = T->dTab;
  D.slot = T->slots[0].dev;
  HIPCHK(hipHostGetDevicePointer((void**)&D.cmd, T->pCmd, 0));
  HIPCHK(hipHostGetDevicePointer((void**)&D.res, T->pRes, 0));
  HIPCHK(hipHostGetDevicePointer((void**)&D.ctOut, T->pCt, 0));
  D.idleTicks = engine_idle_ticks();
  D.startSeq = T->engSeq;
  T->engTimed = T->timing;
  T->engSplit = !engine_wanted(T) && split_engine_wanted(T);
  if (T->engSplit) {
    // (stream-ordered before the launch; never inside a captured graph)
    HIPCHK(hipMemsetAsync(T->dCtl, 0, sizeof(int32_t) * SE_CTL_WORDS, T->engStream));
    D.ctl = T->dCtl;
    D.nFilt = propagate_items_per_job_filter(T->D);
  }
  __atomic_store_n(&T->pRes->alive, 1, __ATOMIC_RELEASE);
  if (T->engSplit) {
    // workgroup 0, then the filter workgroups with every eighth workgroup
    // (XCD 0 in the dispatch round robin) left empty
    int grid = 1;
    for (int f = 0; f < D.nFilt; ++grid)
      if (grid % 8 != 0) ++f;
    HIPCHK(launch_split_engine(D, grid, T->engStream));
  }
  else HIPCHK(launch_engine(D, T->engLds, T->engStream));
  T->engOn = true;
  g_engOwner = T;
  return CT_OK;
}

// Waits for a result slot of call `sq` (written at most a few microseconds
// after its status) and returns its payload; false after two seconds.
bool engine_slot(const ct_table* T, int i, uint32_t sq, uint32_t* payload) {
  const uint64_t* p = &T->pRes->slot[i];
  const auto t0 = std::chrono::steady_clock::now();
  for (uint32_t spin = 0;; ++spin) {
    const uint64_t v = __atomic_load_n(p, __ATOMIC_ACQUIRE);
    if ((uint32_t)v == sq) {
      *payload = (uint32_t)(v >> 32);
      return true;
    }
    if ((spin & 1023) == 1023 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) return false;
  }
}

// One call through the engine; *status receives the call's status and the
// outputs are in T->engDom, T->engStats (wantStats) and T->pCt (wantCt).
int engine_call(ct_table* T, const DevJob& J, const uint64_t* dom_in, bool wantCt, bool wantStats, int* status) {
  std::lock_guard<std::mutex> lk(g_engMu);
  int rc;
  if (T->engOn && __atomic_load_n(&T->pRes->alive, __ATOMIC_ACQUIRE) == 0 && (rc = engine_join(T))) return rc;
  if (!T->engOn && (rc = engine_start(T))) return rc;
  const int32_t seq = ++T->engSeq;
  const uint32_t sq = (uint32_t)seq;
  engine_post(T, seq, ENG_OP_PROPAGATE, &J, dom_in, wantCt, wantStats);
  const uint64_t* stSlot = &T->pRes->slot[ER_STATUS];
  const auto t0 = std::chrono::steady_clock::now();
  uint64_t sv = 0;
  for (uint32_t spin = 0;; ++spin) {
    if ((uint32_t)(sv = __atomic_load_n(stSlot, __ATOMIC_ACQUIRE)) == sq) break;
    if (__atomic_load_n(&T->pRes->alive, __ATOMIC_ACQUIRE) == 0) {
      if ((uint32_t)(sv = __atomic_load_n(stSlot, __ATOMIC_ACQUIRE)) == sq) break;
      // the engine went idle before it saw this call: start a new one (the
      // command stays in the mailbox)
      if ((rc = engine_join(T))) return rc;
      T->engSeq = seq - 1;
      if ((rc = engine_start(T))) return rc;
      T->engSeq = seq;
      continue;
    }
    if ((spin & 1023) == 1023 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) {
      T->poisoned = true;
      return fail(CT_E_DEVICE, "engine did not answer");
    }
  }
  *status = (int32_t)(uint32_t)(sv >> 32);
  bool whole = true;
  if (*status == CT_OK) {
    // every domain slot carries the number (in order of arrival: one clock
    // read per poll round, not per slot)
    const uint64_t* sl = &T->pRes->slot[ER_DOM];
    const int nS = 2 * T->D;
    int got = 0;
    const auto t1 = std::chrono::steady_clock::now();
    for (uint32_t spin = 0;; ++spin) {
      while (got < nS && (uint32_t)__atomic_load_n(&sl[got], __ATOMIC_ACQUIRE) == sq) ++got;
      if (got == nS) break;
      if ((spin & 1023) == 1023 && std::chrono::steady_clock::now() - t1 > std::chrono::seconds(2)) {
        whole = false;
        break;
      }
    }
    T->engDom.resize(T->D);
    for (int q = 0; q < T->D && whole; ++q)
      T->engDom[q] = ((uint64_t)(uint32_t)(sl[2 * q + 1] >> 32) << 32) | (uint32_t)(sl[2 * q] >> 32);
  }
  if (wantStats) {
    for (int k = 0; k < 8 && whole; ++k) {
      uint32_t lo = 0, hi = 0;
      whole = engine_slot(T, ER_STATS + 2 * k, sq, &lo) && engine_slot(T, ER_STATS + 2 * k + 1, sq, &hi);
      T->engStats[k] = ((unsigned long long)hi << 32) | lo;
    }
  }
  uint32_t ticks = 0;
  if (whole && T->timing) whole = engine_slot(T, ER_TICKS, sq, &ticks);
  if (!whole) {
    T->poisoned = true;
    return fail(CT_E_DEVICE, "engine answer incomplete");
  }
  T->engStatsFresh = wantStats;
  if (T->timing) {
    T->engTicks += ticks;
    T->engCalls += 1;
  }
  return CT_OK;
}

// AUTO takes the engine for tables of at most ENG_AUTO_D domain words: on
// wider tables one workgroup's filterDomains (a gather of one word per
// checked value) is slower than the launched schedules, which spread it over
// many workgroups; RESIDENT takes it up to ENG_MAX_D words.
constexpr int ENG_AUTO_D = 64;
bool engine_wanted(const ct_table* T) {
  return T->engEligible &&
         ((T->cfg.schedule == CT_SCHED_AUTO && T->D <= ENG_AUTO_D) || T->cfg.schedule == CT_SCHED_RESIDENT);
}

// AUTO takes the resident split schedule (split_engine_kernel) for the other
// positive tables whose split update is one item (at most 8 granules) and
// whose input fits the kernel-argument view (D <= INLINE_WORDS, so at most
// 64 filter workgroups, all resident at once), with variables of at most
// SE_MAX_VAR_WORDS domain words: plain synchronous calls on slot 0 then pay
// no kernel launch.  Calls that want currTable or counters, and the other
// slots, take the launched schedules.
bool split_engine_wanted(ct_table* T) {
  if (T->seVarWords < 0) {
    int m = 0;
    for (const VarDesc& v : T->vars) m = std::max(m, (int)v.domWords);
    T->seVarWords = m;
  }
  return T->cfg.schedule == CT_SCHED_AUTO && T->kind == CT_KIND_POSITIVE && !engine_wanted(T) &&
         !use_solo(T) && propagate_items_per_job_update(T->nGran) == 1 && T->D <= INLINE_WORDS &&
         T->D <= ENG_MAX_D && T->seVarWords <= SE_MAX_VAR_WORDS &&
         2 + (8 * propagate_items_per_job_filter(T->D)) / 7 <= propagate_max_grid();
}

// Before any other use of a table's device state (from `same`, nullable):
// work a model queued on slot 0 from another stream has ended, and the
// table's engine is stopped.
int quiesce(ct_table* T, hipStream_t same) {
  if (!T) return CT_OK;
  if (T->pendStream && T->pendStream != same) {
    HIPCHK(hipStreamSynchronize(T->pendStream));
    T->pendStream = nullptr;
  }
  if (!T->engOn) return CT_OK;
  std::lock_guard<std::mutex> lk(g_engMu);
  return engine_stop(T);
}

int32_t* pinned_dev(ct_table* T, int32_t* host) {
  int32_t* d = nullptr;
  if (hipHostGetDevicePointer((void**)&d, host, 0) != hipSuccess) return nullptr;
  return d;
}
uint64_t* pinned_dev64(ct_table* T, uint64_t* host) {
  uint64_t* d = nullptr;
  if (hipHostGetDevicePointer((void**)&d, host, 0) != hipSuccess) return nullptr;
  return d;
}

// What a synchronous propagation may have to allocate, before it takes the
// slot's pending operations: a refused allocation leaves the slot as it was
// (pending pops and pushes that were lost would leave the device's level
// behind the host's).
int call_reserve(ct_table* T, bool engine, bool wantCt) {
  if (engine) return engine_reserve(T);
  int rc = wantCt ? ensure_pinned_ct(T) : CT_OK;
  if (rc || use_solo(T) || !stage_single(T)) return rc;
  StageNeed need;
  need.add(T, true, false);
  return stage_reserve(T->q, need.bytes(), T->stream);
}

// Apply pending pushes/pops of a slot (device work) without propagating.
int flush_slot(ct_table* T, int slot) {
  SlotHost& S = T->slots[slot];
  if (S.pendPop == 0 && S.pendPush == 0) return CT_OK;
  DevJob J{};
  J.tab = T->dTab;
  J.slot = S.dev;
  J.flags = 0;
  J.nPop = S.pendPop;
  J.nPush = S.pendPush;
  J.serialBase = T->serialCounter;
  T->serialCounter += S.pendPush;
  J.depthAfter = S.depth;
  J.status_out = pinned_dev(T, T->pStatus);
  S.pendPop = S.pendPush = 0;
  const int rc = run_single(T, J, nullptr);
  if (rc) T->poisoned = true;  // (a device error: the pending operations are gone)
  return rc;
}

int ensure_pinned_ct(ct_table* T) {
  if (T->pCt) return CT_OK;
  ALLOCCHK(hipHostMalloc((void**)&T->pCt, sizeof(uint64_t) * std::max<int64_t>(T->W, 1),
                       hipHostMallocMapped | hipHostMallocCoherent));
  return CT_OK;
}

int check_slot(const ct_table* T, int slot) {
  if (slot < 0 || slot >= (int)T->slots.size())
    return fail(CT_E_INVALID, "slot %d out of range (%zu slots)", slot, T->slots.size());
  if (T->slots[slot].freed) return fail(CT_E_INVALID, "slot %d was freed", slot);
  return CT_OK;
}

// ---------------------------------------------------------------------------
// batch staging shared by ct_propagate_batch and ct_propagate_batch_static
// ---------------------------------------------------------------------------
// Validates every job (no state is touched before all pass; the marks that
// find a slot named twice carry no state), then waits for what the tables
// may still have in flight elsewhere (a model's queued work, the resident
// engine, the tail of a synchronous call).
int batch_validate_quiesce(const ct_job* jobs, int n_jobs, hipStream_t stream) {
  static std::atomic<uint64_t> batchCounter{0};
  const uint64_t mark = ++batchCounter;
  for (int j = 0; j < n_jobs; ++j) {
    const ct_job& cj = jobs[j];
    ct_table* T = cj.table;
    int rc = check_poison(T);
    if (rc) return rc;
    if ((rc = check_slot(T, cj.slot))) return rc;
    if (T->slots[cj.slot].batchMark == mark)
      return fail(CT_E_INVALID, "job %d: slot %d appears twice in the batch", j, cj.slot);
    T->slots[cj.slot].batchMark = mark;
    if (cj.flags & ~(CT_JOB_PROPAGATE | CT_JOB_FROM_ROOT | CT_JOB_ROOT))
      return fail(CT_E_INVALID, "job %d: unknown flags", j);
    if ((cj.flags & CT_JOB_ROOT) && (cj.flags & CT_JOB_FROM_ROOT))
      return fail(CT_E_INVALID, "job %d: ROOT and FROM_ROOT together", j);
    if ((cj.flags & CT_JOB_ROOT) && (cj.n_pop || cj.n_push || !(cj.flags & CT_JOB_PROPAGATE)))
      return fail(CT_E_INVALID, "job %d: ROOT needs PROPAGATE and no pops/pushes", j);
    if (cj.n_pop < 0 || cj.n_push < 0) return fail(CT_E_INVALID, "job %d: negative pops/pushes", j);
    const SlotHost& S = T->slots[cj.slot];
    if (cj.flags & CT_JOB_FROM_ROOT) {
      if (cj.n_pop || cj.n_push) return fail(CT_E_INVALID, "job %d: FROM_ROOT with pops/pushes", j);
      if (!(cj.flags & CT_JOB_PROPAGATE)) return fail(CT_E_INVALID, "job %d: FROM_ROOT needs PROPAGATE", j);
    } else {
      if (cj.n_pop > S.depth) return fail(CT_E_INVALID, "job %d: pop below depth 0", j);
      if (S.depth - cj.n_pop + cj.n_push > S.maxDepth)
        return fail(CT_E_NOMEM, "job %d: depth beyond max_depth", j);
    }
    if ((cj.flags & CT_JOB_PROPAGATE) && (!cj.dom_in || !cj.dom_out))
      return fail(CT_E_INVALID, "job %d: dom_in / dom_out is NULL", j);
  }
  // the synchronous calls of these tables may still be finishing their tail
  for (int j = 0; j < n_jobs; ++j) {
    ct_table* T = jobs[j].table;
    if (T->batchMark == mark) continue;
    T->batchMark = mark;
    int rc = quiesce(T, stream);
    if (rc) return rc;
    if (T->tailPending) {
      HIPCHK(hipStreamSynchronize(T->stream));
      T->tailPending = false;
    }
  }
  return CT_OK;
}

// How a batch's jobs are laid out: the staged ones first (in launches of at
// most the scratch's size: chunks[k] is the first job of launch k), then
// those that run in one workgroup of the propagate kernel (negative tables).
struct BatchShape {
  int nStaged = 0, nChunks = 0, popGran = 0;
  bool wide = false, wideDom = false;
};

// Negative tables run in one workgroup of the propagate kernel.
bool batch_staged(const ct_table* T, bool propagate) { return !propagate || T->kind != CT_KIND_NEGATIVE; }

// A single job's scratch is within every launch's: the records and item lists
// of a table of MAX_GRAN granules and MAX_TABLE_D domain words, four waves to
// a granule's list, and the job's own words.
constexpr size_t STAGE_JOB_MAX = 4096 + sizeof(StageRec) +
                                 sizeof(StageItem) * STAGE_LISTS * ((size_t)MAX_GRAN + MAX_TABLE_D / 4 + 2) +
                                 (sizeof(uint64_t) + sizeof(int32_t)) * (size_t)MAX_TABLE_D +
                                 std::max(sizeof(uint64_t) * (size_t)MAX_TABLE_D, sizeof(uint32_t) * (size_t)(STAGE_LIST_CAP + 64));
static_assert(STAGE_JOB_MAX <= (size_t)14 << 20, "a job fits the no-allocation scratch");

// Device descriptors of a validated batch, written into out[n_jobs] (other:
// the search-node schedule takes them in the batch's order).
// Applies the jobs' pops and pushes to the host mirror of each slot.
BatchShape batch_build(const ct_job* jobs, int n_jobs, int32_t* status_dev, bool other, bool streamRoots,
                       size_t scratchCap, DevJob* out, int32_t* chunks, uint64_t* order) {
  BatchShape B;
  StageNeed need;
  int at = 0;
  if (streamRoots) {
    // the tables with the most support rows first: their waves take longest
    for (int j = 0; j < n_jobs; ++j) order[j] = (uint64_t)~(uint32_t)jobs[j].table->rows << 32 | (uint32_t)j;
    std::sort(order, order + n_jobs);
  }
  for (int pass = 0; pass < 2 && at < n_jobs; ++pass)
    for (int k = 0; k < n_jobs; ++k) {
      const int j = streamRoots ? (int)(uint32_t)order[k] : k;
      const ct_job& cj = jobs[j];
      ct_table* T = cj.table;
      const bool propagate = cj.flags & CT_JOB_PROPAGATE;
      const bool root = (cj.flags & CT_JOB_ROOT) && !streamRoots;  // (row lists shared by waves)
      const bool staged = !other && batch_staged(T, propagate);
      if (!other && staged != (pass == 0)) continue;
      SlotHost& S = T->slots[cj.slot];
      DevJob& J = out[at++];
      J = DevJob{};
      J.tab = T->dTab;
      J.slot = S.dev;
      J.dom_in = cj.dom_in;
      J.dom_out = cj.dom_out;
      J.ct_out = cj.ct_out;
      J.status_out = status_dev + j;
      J.flags = (propagate ? JF_PROPAGATE : 0u) | ((cj.flags & CT_JOB_FROM_ROOT) ? JF_FROM_ROOT : 0u) |
                ((cj.flags & CT_JOB_ROOT) ? (JF_ROOT | JF_FROM_ROOT | JF_SCRATCH) : 0u);
      if (cj.flags & (CT_JOB_FROM_ROOT | CT_JOB_ROOT)) {
        S.pendPop = S.pendPush = 0;
        S.depth = 0;
        S.failedAt.clear();
        J.serialBase = T->serialCounter++;
        J.depthAfter = 0;
      } else {
        // pending single-call operations (pops P then pushes Q) come first
        int P = S.pendPop, Q = S.pendPush;
        if (cj.n_pop <= Q) {
          Q = Q - cj.n_pop + cj.n_push;
        } else {
          P += cj.n_pop - Q;
          Q = cj.n_push;
        }
        S.pendPop = S.pendPush = 0;
        J.nPop = P;
        J.nPush = Q;
        J.serialBase = T->serialCounter;
        T->serialCounter += Q;
        for (int k = 0; k < cj.n_pop; ++k) S.failedAt.pop_back();
        for (int k = 0; k < cj.n_push; ++k) S.failedAt.push_back(2);
        S.depth = S.depth - cj.n_pop + cj.n_push;
        J.depthAfter = S.depth;
      }
      S.failed = 2;
      if (other) continue;
      if (!staged) {
        J.flags |= JF_SOLO;
        continue;
      }
      if (B.nStaged == 0 || need.bytes_with(T, root) > scratchCap) {
        chunks[B.nChunks++] = B.nStaged;
        need = StageNeed();
      }
      J.stageOff = (int32_t)(need.jobBytes / 256);
      J.listCap = streamRoots ? 0 : stage_list_cap(T);
      if (streamRoots) J.seq = need.nU;
      J.nUpd = !propagate ? 0 : root ? T->stage.nURoot : T->stage.nU;
      J.nFilt = propagate ? T->stage.nF : 0;
      need.add(T, propagate, J.nPop > 0, root);
      B.popGran = std::max(B.popGran, need.popGran);
      B.wide = B.wide || need.wide;
      B.wideDom = B.wideDom || need.wideDom;
      ++B.nStaged;
    }
  return B;
}

// Host mirrors of n fresh slots in the root state.
void slots_add(ct_table* T, SlotDesc* d, int n, int max_depth) {
  for (int k = 0; k < n; ++k) {
    SlotHost s;
    s.dev = d + k;
    s.maxDepth = max_depth;
    s.capDepth = max_depth;
    s.failed = T->rootFailed ? 1 : 0;
    // a push never grows this vector past its capacity (no allocation per push)
    s.failedAt.reserve(max_depth);
    T->slots.push_back(s);
  }
}

// ---------------------------------------------------------------------------
// Upload of a table's tuples.  The caller's array is pageable: up to UP_WORKERS
// threads copy it, a chunk each, into a window of pinned memory, which the
// support build reads where it is (each tuple once) while they fill the other
// window: copies and builds overlap and no device copy of the tuples exists.
// Creating a table of 1,000,000 tuples of 6 columns (24 MB): 1.2 ms, of which
// the builds take 0.7 at 37 GB/s of the bus, against 3.65 ms with a pass over
// the cells (1.2), a copy and transfer by one thread (1.25), a device copy to
// allocate and free (0.4) and 24 small copies (0.8).  Chunks of 1/4 MiB 1.5 ms.
// ---------------------------------------------------------------------------
constexpr size_t UP_CHUNK = (size_t)1 << 20;       // bytes of a worker's part of a window
constexpr int UP_WORKERS = 4, UP_KEEP = 2;
constexpr size_t UP_PER_WORKER = (size_t)2 << 20;  // tuples' bytes for each further worker

// Two windows in one pinned block.
struct UploadBuf {
  int dev = 0;
  size_t window = 0;  // bytes of a window (its reads may pass its end by 16)
  char* p = nullptr;
  hipEvent_t ev[2] = {nullptr, nullptr};
};

// Free blocks, at most UP_KEEP, the first to come back; given back with the last
// table.  (Keeping the largest instead: creations of many sizes allocate and
// free less, but a wait for the whole device in a program of 800 tables then
// takes 28 us against 24, and 400 tables' search steps 5 % longer: freeing
// pinned memory leaves the runtime's streams in a state that is cheaper to
// wait for.)
std::mutex g_upMu;
UploadBuf* g_upFree[UP_KEEP] = {};

void upload_free(UploadBuf* b) {
  if (b->p) (void)hipHostFree(b->p);
  for (hipEvent_t e : b->ev)
    if (e) (void)hipEventDestroy(e);
  delete b;
}

void upload_drain() {
  std::lock_guard<std::mutex> lk(g_upMu);
  for (UploadBuf*& b : g_upFree) {
    if (b) upload_free(b);
    b = nullptr;
  }
}

void upload_give(UploadBuf* b) {
  if (!b) return;
  {
    std::lock_guard<std::mutex> lk(g_upMu);
    for (UploadBuf*& f : g_upFree)
      if (!f) std::swap(f, b);
  }
  if (b) upload_free(b);
}

int upload_take(int dev, size_t window, UploadBuf** out) {
  {
    // the smallest that is large enough
    std::lock_guard<std::mutex> lk(g_upMu);
    UploadBuf** at = nullptr;
    for (UploadBuf*& f : g_upFree)
      if (f && f->dev == dev && f->window >= window && (!at || f->window < (*at)->window)) at = &f;
    if (at) {
      *out = *at;
      *at = nullptr;
      return CT_OK;
    }
  }
  if (alloc_injected()) return fail(CT_E_NOMEM, "injected allocation failure: upload block");
  UploadBuf* b = new (std::nothrow) UploadBuf();
  if (!b) return fail(CT_E_NOMEM, "host allocation failed");
  b->dev = dev;
  b->window = (window + 255) & ~(size_t)255;
  hipError_t e = hipHostMalloc((void**)&b->p, 2 * b->window + 256, hipHostMallocDefault);
  for (int k = 0; k < 2 && e == hipSuccess; ++k) e = hipEventCreateWithFlags(&b->ev[k], hipEventDisableTiming);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    upload_free(b);
    return fail(CT_E_NOMEM, "upload block: %s", hipGetErrorString(e));
  }
  *out = b;
  return CT_OK;
}

// Words of 64 tuples in a worker's chunk, and the workers for a table.
int64_t upload_chunk_words(int n) { return std::max<int64_t>(1, (int64_t)(UP_CHUNK / (sizeof(int32_t) * 64 * (size_t)n))); }
int upload_workers(int64_t W, int n) {
  const size_t bytes = sizeof(int32_t) * 64 * (size_t)n * (size_t)W;
  return (int)std::min<size_t>(UP_WORKERS, 1 + bytes / UP_PER_WORKER);
}
size_t upload_window(int64_t W, int n) {
  const int64_t words = std::min(W, upload_chunk_words(n) * upload_workers(W, n));
  return sizeof(int32_t) * 64 * (size_t)n * (size_t)words;
}

// Queues the support build of all tuples on the stream (B: the kernel's
// arguments but the window).  b must stay until the stream has ended.
hipError_t upload_run(const int32_t* tuples, BuildArgs B, hipStream_t stream, const UploadBuf* b) {
  const int64_t chunk = upload_chunk_words(B.n);
  const int nW = upload_workers(B.W, B.n);
  const int64_t per = chunk * nW, windows = (B.W + per - 1) / per;
  std::atomic<int64_t> released{2};              // windows that may be filled
  std::atomic<int> arrived[2] = {{0}, {0}};      // workers done with a window
  std::atomic<bool> stop{false};
  auto copy = [&](int id, int64_t win) {         // worker id's part of a window
    const int64_t w0 = win * per + id * chunk, j0 = w0 * 64;
    const int64_t j1 = std::min(B.t, std::min(w0 + chunk, (win + 1) * per) * 64);
    if (j0 < j1)
      memcpy(b->p + (win & 1) * b->window + sizeof(int32_t) * (size_t)(id * chunk * 64) * B.n, tuples + j0 * B.n,
             sizeof(int32_t) * (size_t)(j1 - j0) * B.n);
  };
  auto work = [&](int id) {
    for (int64_t win = 0; win < windows; ++win) {
      while (released.load(std::memory_order_acquire) <= win) {
        if (stop.load()) return;
        std::this_thread::yield();
      }
      copy(id, win);
      arrived[win & 1].fetch_add(1, std::memory_order_release);
    }
  };
  std::thread th[UP_WORKERS];
  int started = 1;
  try {
    for (; started < nW; ++started) th[started] = std::thread(work, started);
  } catch (...) {
    // fewer threads (none to be had, or no memory): their parts are copied here
  }
  char* dp = nullptr;
  hipError_t e = hipHostGetDevicePointer((void**)&dp, b->p, 0);
  for (int64_t win = 0; win < windows && e == hipSuccess; ++win) {
    const int k = (int)(win & 1);
    if (win >= 2) {
      e = hipEventSynchronize(b->ev[k]);
      if (e != hipSuccess) break;
      released.store(win + 1, std::memory_order_release);
    }
    copy(0, win);
    for (int id = started; id < nW; ++id) copy(id, win);
    while (arrived[k].load(std::memory_order_acquire) < started - 1) std::this_thread::yield();
    arrived[k].store(0, std::memory_order_relaxed);
    B.tuples = (const int32_t*)(dp + k * b->window);
    B.w0 = win * per;
    B.nw = std::min(per, B.W - B.w0);
    e = launch_build_supports(B, stream);
    // (only where a later window waits for it: an event left behind on every
    // table's stream costs each later wait for the device, 1,000 tables 40 us)
    if (e == hipSuccess && win + 2 < windows) e = hipEventRecord(b->ev[k], stream);
  }
  stop.store(true);
  for (int id = 1; id < started; ++id) th[id].join();
  return e;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* ct_last_error(void) { return g_err; }

int ct_debug_fail_alloc(int32_t nth) { return g_failAlloc.exchange(nth > 0 ? nth : 0); }

int ct_quiesce(void) {
  std::lock_guard<std::mutex> lk(g_engMu);
  return g_engOwner ? engine_stop(g_engOwner) : CT_OK;
}

void ct_destroy(ct_table* T) {
  if (!T) return;
  (void)quiesce(T);
  bool last = false;
  {
    std::lock_guard<std::mutex> lk(g_engMu);
    g_tables.erase(T);
    last = g_tables.empty();
  }
  if (last) upload_drain();
  if (T->pCmd) (void)hipHostFree(T->pCmd);
  if (T->pRes) (void)hipHostFree(T->pRes);
  if (T->engStream) (void)hipStreamDestroy(T->engStream);
  if (T->stream) (void)hipStreamSynchronize(T->stream);
  for (void* p : T->blocks) (void)hipFree(p);
  if (T->q.dStaged) (void)hipFree(T->q.dStaged);
  if (T->pBlock) (void)hipHostFree(T->pBlock);
  if (T->pCt) (void)hipHostFree(T->pCt);
  if (T->stream) (void)hipStreamDestroy(T->stream);
  delete T;
}

// 1 if two tuples of the table are equal (hash of each row, then the rows
// with equal hashes compared)
bool has_duplicate_rows(const int32_t* tuples, int64_t t, int n) {
  std::vector<std::pair<uint64_t, int64_t>> h((size_t)t);
  for (int64_t j = 0; j < t; ++j) {
    uint64_t x = 1469598103934665603ull;
    for (int i = 0; i < n; ++i) x = (x ^ (uint32_t)tuples[j * n + i]) * 1099511628211ull;
    h[(size_t)j] = {x, j};
  }
  std::sort(h.begin(), h.end());
  for (size_t k = 1; k < h.size(); ++k)
    if (h[k].first == h[k - 1].first &&
        std::equal(tuples + h[k].second * n, tuples + h[k].second * n + n, tuples + h[k - 1].second * n))
      return true;
  return false;
}

static int create_impl(ct_table* T, const int32_t* tuples, int64_t t, int32_t n,
                       const int32_t* lo, const int32_t* dsz, const uint64_t* init_dom) {
  const bool negative = T->kind == CT_KIND_NEGATIVE;
  if (negative) {
    for (int64_t k = 0; k < t * n; ++k)
      if (tuples[k] == CT_STAR) return fail(CT_E_INVALID, "a negative table has no star cell");
    if (has_duplicate_rows(tuples, t, n)) return fail(CT_E_INVALID, "a negative table lists distinct tuples");
  }
  T->n = n;
  T->t = t;
  T->W = (t + 63) / 64;
  T->nGran = (int)std::max<int64_t>(1, (T->W + GW - 1) / GW);
  T->stride = (int64_t)T->nGran * GW;
  T->lo.assign(lo, lo + n);
  T->dsz.assign(dsz, dsz + n);
  int rows = 0, D = 0;
  for (int i = 0; i < n; ++i) {
    VarDesc v;
    v.rowStart = rows;
    v.dsize = dsz[i];
    v.domOff = D;
    v.domWords = (dsz[i] + 63) / 64;
    T->vars.push_back(v);
    T->domOff.push_back(D);
    for (int k = 0; k < v.domWords; ++k) T->wordVar.push_back(i);
    rows += dsz[i];
    D += v.domWords;
  }
  T->rows = rows;
  T->D = D;
  T->stage = stage_shape(T);
  if (rows > MAX_TABLE_ROWS) return fail(CT_E_INVALID, "%d support rows exceed the limit %d", rows, MAX_TABLE_ROWS);
  if (D > MAX_TABLE_D) return fail(CT_E_INVALID, "%d domain words exceed the limit %d", D, MAX_TABLE_D);
  if (T->kind == CT_KIND_NEGATIVE && (rows > NEG_MAX_ROWS || D > MAX_D))
    return fail(CT_E_INVALID, "a negative table has at most %d support rows and %d domain words", NEG_MAX_ROWS,
                MAX_D);
  if (T->nGran > MAX_GRAN)
    return fail(CT_E_INVALID, "%lld tuples exceed the limit %lld", (long long)t,
                (long long)MAX_GRAN * GW * 64);
  // initial domains (validated on the host, before any device work)
  std::vector<uint64_t> dom0(D, 0);
  for (int i = 0; i < n; ++i) {
    const VarDesc& v = T->vars[i];
    for (int k = 0; k < v.domWords; ++k) {
      const int used = std::min(64, v.dsize - 64 * k);
      const uint64_t full = used == 64 ? ~0ull : ((1ull << used) - 1);
      if (init_dom) {
        if (init_dom[v.domOff + k] & ~full)
          return fail(CT_E_INVALID, "init_dom has stray bits in variable %d", i);
        dom0[v.domOff + k] = init_dom[v.domOff + k];
      } else {
        dom0[v.domOff + k] = full;
      }
    }
  }
  HIPCHK(hipStreamCreateWithFlags(&T->stream, hipStreamNonBlocking));
  // coherent (fine-grained) pinned buffers: the kernel's writes reach host
  // memory without waiting for the end of the kernel
  const auto line = [](size_t x) { return (x + 127) & ~(size_t)127; };
  const size_t domB = line(sizeof(uint64_t) * D), llB = line(sizeof(uint64_t) * (2 + 2 * (size_t)D));
  ALLOCCHK(hipHostMalloc((void**)&T->pBlock, 256 + 2 * domB + llB, hipHostMallocMapped | hipHostMallocCoherent));
  T->pStatus = (int32_t*)T->pBlock;
  T->q.hostErr = (int32_t*)(T->pBlock + 128);
  T->pDomOut = (uint64_t*)(T->pBlock + 256);
  T->pDomIn = (uint64_t*)(T->pBlock + 256 + domB);
  T->pLL = (uint64_t*)(T->pBlock + 256 + 2 * domB);
  *T->q.hostErr = 0;
  memset(T->pLL, 0, sizeof(uint64_t) * (2 + 2 * (size_t)D));

  // the supports; the static data and the root slot's descriptor, one image
  // sent in one copy; the root slot's arrays
  int rc;
  if ((rc = dev_alloc(T, (void**)&T->dS, sizeof(uint64_t) * (size_t)rows * T->stride))) return rc;
  size_t imgB = 0;
  const auto part = [&imgB](size_t bytes) {
    const size_t at = imgB;
    imgB += align256(bytes);
    return at;
  };
  const size_t oVars = part(sizeof(VarDesc) * n), oWordVar = part(sizeof(int32_t) * D), oWords = part(sizeof(WordDesc) * D),
               oLo = part(sizeof(int32_t) * n), oTab = part(sizeof(TabDesc)), oQueue = part(sizeof(int32_t) * 8),
               oDom = part(sizeof(uint64_t) * D), oSize = part(sizeof(int32_t) * D), oRec = part(sizeof(StageRec)),
               oRoot = part(sizeof(SlotDesc));
  size_t arrB = imgB;
  const auto array = [&arrB](size_t bytes) {
    const size_t at = arrB;
    arrB += align256(bytes);
    return at;
  };
  const size_t oCt = array(sizeof(uint64_t) * T->stride), oIdx0 = array(sizeof(int32_t) * T->nGran),
               oIdx1 = array(sizeof(int32_t) * T->nGran), oStamp = array(sizeof(int32_t) * T->nGran),
               oNz = array(sizeof(int32_t) * T->nGran), oLast = array(sizeof(uint64_t) * D),
               oRes = array(sizeof(int32_t) * rows);
  char* base = nullptr;
  if ((rc = dev_alloc(T, (void**)&base, arrB))) return rc;
  std::vector<char> img(imgB, 0);
  T->dVars = (VarDesc*)(base + oVars);
  T->dWordVar = (int32_t*)(base + oWordVar);
  T->dWords = (WordDesc*)(base + oWords);
  T->dLo = (int32_t*)(base + oLo);
  T->dTab = (TabDesc*)(base + oTab);
  T->q.queue = (int32_t*)(base + oQueue);  // [3] error word; [4] a star cell was seen
  T->dRoot = (SlotDesc*)(base + oRoot);
  memcpy(img.data() + oVars, T->vars.data(), sizeof(VarDesc) * n);
  memcpy(img.data() + oWordVar, T->wordVar.data(), sizeof(int32_t) * D);
  memcpy(img.data() + oLo, lo, sizeof(int32_t) * n);
  memcpy(img.data() + oDom, dom0.data(), sizeof(uint64_t) * D);
  WordDesc* words = (WordDesc*)(img.data() + oWords);
  int32_t* size = (int32_t*)(img.data() + oSize);  // |dom| of the word's variable
  bool empty = false;
  int64_t selected = 0;
  for (int i = 0; i < n; ++i) {
    const VarDesc& v = T->vars[i];
    int sz = 0;
    for (int k = 0; k < v.domWords; ++k) sz += __builtin_popcountll(dom0[v.domOff + k]);
    for (int k = 0; k < v.domWords; ++k) {
      words[v.domOff + k].v = v;
      words[v.domOff + k].var = i;
      size[v.domOff + k] = sz;
    }
    empty = empty || sz == 0;
    selected += sz;
  }
  // root slot: every granule active, domains dom0
  SlotDesc& r = T->hRoot;
  r = SlotDesc{};
  r.ct = (uint64_t*)(base + oCt);
  r.idx[0] = (int32_t*)(base + oIdx0);
  r.idx[1] = (int32_t*)(base + oIdx1);
  r.stamp = (int32_t*)(base + oStamp);
  r.nzFlag = (int32_t*)(base + oNz);
  r.lastDom = (uint64_t*)(base + oLast);
  r.res = (int32_t*)(base + oRes);
  r.limit = T->nGran;
  memcpy(img.data() + oRoot, &r, sizeof(SlotDesc));
  // (its index buffer, limit and failed flag are filled in after the root
  // propagation)
  TabDesc& tb = T->hTab;
  tb.n = n;
  tb.rows = rows;
  tb.D = D;
  tb.nGran = T->nGran;
  tb.W = T->W;
  tb.stride = T->stride;
  tb.S = T->dS;
  tb.vars = T->dVars;
  tb.wordVar = T->dWordVar;
  tb.words = T->dWords;
  tb.ct0 = r.ct;
  tb.dom0 = r.lastDom;
  tb.policy = T->cfg.branch_policy;
  tb.tailBits = T->W > 0 ? (int32_t)(t - 64 * (T->W - 1)) : 0;
  tb.kind = T->kind;
  memcpy(img.data() + oTab, &tb, sizeof(TabDesc));
  // The root of a positive table: a tuple is valid iff each of its values is
  // in dom0 (or is a star), which the support build sees as it passes: no
  // support row is read for the root's currTable.  The partition and
  // filterDomains are the staged finish's.
  StageRec& rec = *(StageRec*)(img.data() + oRec);
  rec.run = 1;
  rec.flags = JF_PROPAGATE | JF_ROOT;
  rec.mode = STAGE_LIST;
  rec.nrows = (int32_t)selected;
  rec.limit = T->nGran;
  rec.D = D;
  rec.nGran = T->nGran;
  rec.curNew = 1;
  rec.tab = T->dTab;
  rec.slot = T->dRoot;
  rec.S = T->dS;
  rec.stride = T->stride;
  rec.W = T->W;
  rec.words = T->dWords;
  rec.idxSrc = r.idx[0];
  rec.idxDst = r.idx[1];
  rec.ct = r.ct;
  rec.nz = r.nzFlag;
  rec.res = r.res;
  rec.lastDom = r.lastDom;
  rec.din = (uint64_t*)(base + oDom);
  rec.size = (int32_t*)(base + oSize);
  rec.dom_out = r.lastDom;
  // slot 0
  SlotDesc* d0 = nullptr;
  std::vector<SlotDesc> h0;
  if ((rc = alloc_slots(T, 1, T->cfg.max_depth, &d0, h0))) return rc;
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  UploadBuf* up = nullptr;
  if (t > 0 && (rc = upload_take(dev, upload_window(T->W, n), &up))) {
    (void)hipStreamSynchronize(T->stream);
    return rc;
  }
  hipError_t e = hipMemsetAsync(T->dS, 0, sizeof(uint64_t) * (size_t)rows * T->stride, T->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(base, img.data(), imgB, hipMemcpyHostToDevice, T->stream);
  if (e == hipSuccess) e = launch_init_root(T->dTab, T->dRoot, (uint64_t*)(base + oDom),
                                           std::max<int64_t>(T->stride, rows), T->stream);
  if (e == hipSuccess && t > 0) {
    BuildArgs B{};
    B.t = t;
    B.W = T->W;
    B.n = n;
    B.empty = empty;
    B.vars = T->dVars;
    B.lo = T->dLo;
    B.dom0 = (uint64_t*)(base + oDom);
    B.S = T->dS;
    B.stride = T->stride;
    B.ct = negative ? nullptr : r.ct;
    B.nz = r.nzFlag;
    B.star = T->q.queue + 4;
    e = upload_run(tuples, B, T->stream, up);
  }
  if (e == hipSuccess && !negative) {
    StageArgs A{};
    A.rec = (StageRec*)(base + oRec);
    A.wide = stage_wide_launch(T->stage.wide, T->stage.nF);
    e = launch_staged_finish(A, T->stage.nF, T->stream);
  }
  rc = CT_OK;
  if (e == hipSuccess && negative) {
    // every variable takes the reset branch over dom0
    DevJob J{};
    J.tab = T->dTab;
    J.slot = T->dRoot;
    J.flags = JF_PROPAGATE | JF_ROOT;
    J.dom_out = pinned_dev64(T, T->pDomOut);
    J.status_out = pinned_dev(T, T->pStatus);
    J.depthAfter = 0;
    rc = run_single(T, J, dom0.data());
  }
  if (e == hipSuccess && rc == CT_OK)
    e = launch_init_first(T->dTab, d0, T->dRoot, (uint64_t*)(base + oDom), T->q.queue + 4, pinned_dev(T, T->pStatus),
                          std::max<int64_t>(T->stride, rows), T->stream);
  const hipError_t e2 = hipStreamSynchronize(T->stream);
  upload_give(up);
  if (rc) return rc;
  if (e != hipSuccess || e2 != hipSuccess)
    return fail(CT_E_DEVICE, "support build failed: %s", hipGetErrorString(e != hipSuccess ? e : e2));
  T->tailPending = false;
  const int st = T->pStatus[0];
  if (st != CT_OK && st != CT_FAIL) return fail(CT_E_DEVICE, "root propagation returned %d", st);
  T->rootFailed = st == CT_FAIL;
  if (T->pStatus[1]) {
    // a star cell supports every value of its column: the update takes the
    // reset branch (OR over the remaining values), which needs no other rows
    // (the table's descriptor has it already)
    if (T->cfg.branch_policy == CT_BRANCH_INCREMENTAL)
      return fail(CT_E_INVALID, "a short table's update takes the reset branch");
    T->cfg.branch_policy = CT_BRANCH_RESET;
    T->shortTab = true;
  }
  // search-node schedule: the row vectors of a batch's smallest group fit LDS
  if (T->kind == CT_KIND_POSITIVE) {
    const int vecRows = rows + 2 + (T->shortTab ? n : 0);
    if (vecRows <= nodes_max_vec_rows((size_t)device_lds())) T->nodesVecRows = vecRows;
  }
  if (T->cfg.schedule == CT_SCHED_NODES) (void)nodes_ids_ensure(T);
  slots_add(T, d0, 1, T->cfg.max_depth);
  // the resident engine holds the slot's state in one workgroup's LDS
  T->engLds = engine_lds_bytes(T->n, T->D, T->nGran, T->rows);
  int lds = 0;
  HIPCHK(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  // (the engine lists rows with 16-bit ids)
  T->engEligible = T->D <= ENG_MAX_D && T->W > 0 && T->engLds <= (size_t)lds && T->kind == CT_KIND_POSITIVE &&
                   T->rows <= 65535;
  std::lock_guard<std::mutex> lk(g_engMu);
  g_tables.insert(T);
  return CT_OK;
}

int ct_create(const int32_t* tuples, int64_t n_tuples, int32_t arity, const int32_t* dom_lo,
              const int32_t* dom_size, const uint64_t* init_dom, const ct_config* cfg,
              ct_table** out) {
  return ct_create_table(tuples, n_tuples, arity, dom_lo, dom_size, init_dom, cfg, CT_KIND_POSITIVE, out);
}

int ct_create_table(const int32_t* tuples, int64_t n_tuples, int32_t arity, const int32_t* dom_lo,
                    const int32_t* dom_size, const uint64_t* init_dom, const ct_config* cfg, int32_t kind,
                    ct_table** out) {
  if (!out) return fail(CT_E_INVALID, "out is NULL");
  *out = nullptr;
  if (kind != CT_KIND_POSITIVE && kind != CT_KIND_NEGATIVE) return fail(CT_E_INVALID, "kind %d", kind);
  if (arity < 1 || arity > MAX_ARITY) return fail(CT_E_INVALID, "arity %d not in [1, %d]", arity, MAX_ARITY);
  if (n_tuples < 0) return fail(CT_E_INVALID, "n_tuples < 0");
  if (n_tuples > 0 && !tuples) return fail(CT_E_INVALID, "tuples is NULL");
  if (!dom_lo || !dom_size) return fail(CT_E_INVALID, "dom_lo / dom_size is NULL");
  for (int i = 0; i < arity; ++i)
    if (dom_size[i] < 1) return fail(CT_E_INVALID, "dom_size[%d] < 1", i);
  ct_table* T = new (std::nothrow) ct_table();
  if (!T) return fail(CT_E_NOMEM, "host allocation failed");
  T->cfg.branch_policy = CT_BRANCH_AUTO;
  T->cfg.max_depth = 256;
  T->cfg.schedule = CT_SCHED_AUTO;
  T->kind = kind;
  if (cfg) {
    if (cfg->schedule < 0 || cfg->schedule > 4) {
      delete T;
      return fail(CT_E_INVALID, "schedule %d", cfg->schedule);
    }
    T->cfg.schedule = cfg->schedule;
    if (cfg->branch_policy < 0 || cfg->branch_policy > 2) {
      delete T;
      return fail(CT_E_INVALID, "branch_policy %d", cfg->branch_policy);
    }
    T->cfg.branch_policy = cfg->branch_policy;
    if (cfg->max_depth < 0) {
      delete T;
      return fail(CT_E_INVALID, "max_depth < 0");
    }
    T->cfg.max_depth = cfg->max_depth;
  }
  int rc;
  try {
    rc = create_impl(T, tuples, n_tuples, arity, dom_lo, dom_size, init_dom);
  } catch (const std::bad_alloc&) {
    rc = fail(CT_E_NOMEM, "host allocation failed");
  }
  if (rc != CT_OK) {
    char msg[sizeof(g_err)];
    memcpy(msg, g_err, sizeof(g_err));
    ct_destroy(T);
    memcpy(g_err, msg, sizeof(g_err));
    return rc;
  }
  *out = T;
  return T->rootFailed ? CT_FAIL : CT_OK;
}

int ct_layout(const ct_table* T, ct_layout_info* info, int32_t* dom_off) {
  if (!T) return fail(CT_E_INVALID, "null table");
  if (info) {
    info->n_vars = T->n;
    info->D = T->D;
    info->W = T->W;
    info->n_tuples = T->t;
    info->rows = T->rows;
    info->n_slots = (int32_t)T->slots.size();
    info->granules = T->nGran;
    info->root_failed = T->rootFailed;
    info->resident = engine_wanted(T) ? 1 : split_engine_wanted(const_cast<ct_table*>(T)) ? 2 : 0;
    info->kind = T->kind == CT_KIND_NEGATIVE ? CT_KIND_NEGATIVE : T->shortTab ? CT_KIND_SHORT : CT_KIND_POSITIVE;
  }
  if (dom_off) memcpy(dom_off, T->domOff.data(), sizeof(int32_t) * T->n);
  return CT_OK;
}

int ct_get_supports(ct_table* T, int32_t row_begin, int32_t n_rows, uint64_t* out) {
  int rc = check_poison(T);
  if (rc) return rc;
  if (row_begin < 0 || n_rows < 0 || row_begin + n_rows > T->rows || (!out && n_rows))
    return fail(CT_E_INVALID, "rows [%d, %d) out of range", row_begin, row_begin + n_rows);
  if (T->W == 0) return CT_OK;
  HIPCHK(hipMemcpy2D(out, sizeof(uint64_t) * T->W, T->dS + (size_t)row_begin * T->stride,
                     sizeof(uint64_t) * T->stride, sizeof(uint64_t) * T->W, n_rows,
                     hipMemcpyDeviceToHost));
  return CT_OK;
}

}  // extern "C"

// ct_slots_alloc; search: the slots may serve search-node batches.
int ctk::slots_alloc(ct_table* T, int32_t n, int32_t max_depth, bool search, int32_t* first_slot) {
  int rc = check_poison(T);
  if (rc) return rc;
  if (n < 1) return fail(CT_E_INVALID, "n < 1");
  if ((rc = quiesce(T))) return rc;
  if (max_depth < 0) max_depth = T->cfg.max_depth;
  const int all = (int)T->slots.size() + n;
  if (search && (T->cfg.schedule == CT_SCHED_NODES ||
                 (T->cfg.schedule == CT_SCHED_AUTO && all >= NODES_MIN_BATCH && nodes_pays(T, all))))
    (void)nodes_ids_ensure(T);
  // reuse: the first run of n consecutive freed slots whose trails hold
  // max_depth levels; each is reset to the root state
  int run = 0, first = -1;
  for (int k = 0; k < (int)T->slots.size() && first < 0; ++k) {
    const SlotHost& S = T->slots[k];
    run = (S.freed && S.capDepth >= max_depth) ? run + 1 : 0;
    if (run == n) first = k - n + 1;
  }
  if (first >= 0) {
    for (int k = first; k < first + n; ++k)
      HIPCHK(launch_init_slots(T->dTab, T->slots[k].dev, 1, T->hRoot.res, T->stream));
    HIPCHK(hipStreamSynchronize(T->stream));
    for (int k = first; k < first + n; ++k) {
      SlotHost& S = T->slots[k];
      const int cap = S.capDepth;
      SlotDesc* dev = S.dev;
      S = SlotHost();
      S.dev = dev;
      S.capDepth = cap;
      S.maxDepth = max_depth;
      S.failed = T->rootFailed ? 1 : 0;
      S.failedAt.reserve(max_depth);
    }
    if (first_slot) *first_slot = first;
    return CT_OK;
  }
  SlotDesc* d = nullptr;
  std::vector<SlotDesc> h;
  if ((rc = alloc_slots(T, n, max_depth, &d, h))) return rc;
  HIPCHK(launch_init_slots(T->dTab, d, n, T->hRoot.res, T->stream));
  HIPCHK(hipStreamSynchronize(T->stream));
  if (first_slot) *first_slot = (int32_t)T->slots.size();
  slots_add(T, d, n, max_depth);
  return CT_OK;
}

extern "C" {

int ct_slots_alloc(ct_table* T, int32_t n, int32_t max_depth, int32_t* first_slot) {
  return slots_alloc(T, n, max_depth, true, first_slot);
}

int ct_slots_free(ct_table* T, int32_t first, int32_t n) {
  int rc = check_poison(T);
  if (rc) return rc;
  if (n < 1 || first < 1 || first > (int)T->slots.size() - n)
    return fail(CT_E_INVALID, "slots [%d, %d) cannot be freed (%zu slots; slot 0 stays)", first, first + n,
                T->slots.size());
  for (int k = first; k < first + n; ++k)
    if (T->slots[k].freed) return fail(CT_E_INVALID, "slot %d is already free", k);
  // batches queued on other streams may still use the slots: the caller
  // frees a slot only after its last batch has completed
  if ((rc = quiesce(T))) return rc;
  for (int k = first; k < first + n; ++k) {
    SlotHost& S = T->slots[k];
    S.freed = true;
    S.depth = 0;
    S.pendPop = S.pendPush = 0;
    S.failedAt.clear();
  }
  return CT_OK;
}

int ct_push_slot(ct_table* T, int32_t slot) {
  int rc = check_poison(T);
  if (rc) return rc;
  if ((rc = check_slot(T, slot))) return rc;
  SlotHost& S = T->slots[slot];
  if (S.failed == 1) return fail(CT_E_STATE, "push on a failed slot");
  if (S.depth >= S.maxDepth) return fail(CT_E_NOMEM, "depth %d reaches max_depth", S.depth);
  S.failedAt.push_back(S.failed);
  S.depth++;
  S.pendPush++;
  return CT_OK;
}

int ct_pop_slot(ct_table* T, int32_t slot) {
  int rc = check_poison(T);
  if (rc) return rc;
  if ((rc = check_slot(T, slot))) return rc;
  SlotHost& S = T->slots[slot];
  if (S.depth == 0) return fail(CT_E_STATE, "pop at depth 0");
  S.depth--;
  S.failed = S.failedAt.back();
  S.failedAt.pop_back();
  if (S.pendPush > 0) S.pendPush--;
  else S.pendPop++;
  return CT_OK;
}

int ct_push(ct_table* T) { return ct_push_slot(T, 0); }
int ct_pop(ct_table* T) { return ct_pop_slot(T, 0); }

int ct_propagate_slot(ct_table* T, int32_t slot, const uint64_t* dom_in, uint64_t* dom_out,
                      uint64_t* ct_out, ct_stats* st) {
  int rc = check_poison(T);
  if (rc) return rc;
  if ((rc = check_slot(T, slot))) return rc;
  if (!dom_in || !dom_out) return fail(CT_E_INVALID, "dom_in / dom_out is NULL");
  const bool engine = slot == 0 && (engine_wanted(T) || (!ct_out && !st && split_engine_wanted(T)));
  if ((rc = call_reserve(T, engine, ct_out != nullptr))) return rc;
  SlotHost& S = T->slots[slot];
  DevJob J{};
  J.tab = T->dTab;
  J.slot = S.dev;
  J.flags = JF_PROPAGATE;
  J.nPop = S.pendPop;
  J.nPush = S.pendPush;
  J.serialBase = T->serialCounter;
  T->serialCounter += S.pendPush;
  J.depthAfter = S.depth;
  J.dom_out = pinned_dev64(T, T->pDomOut);
  J.status_out = pinned_dev(T, T->pStatus);
  if (ct_out) J.ct_out = pinned_dev64(T, T->pCt);
  S.pendPop = S.pendPush = 0;
  int status = CT_OK;
  const uint64_t* domRes = T->pDomOut;
  rc = engine ? engine_call(T, J, dom_in, ct_out != nullptr, st != nullptr, &status) : run_single(T, J, dom_in);
  if (rc) {  // (a device error: the pending operations are gone)
    T->poisoned = true;
    return rc;
  }
  if (engine) domRes = T->engDom.data();
  else status = *T->pStatus;
  if (status == CT_OK) {
    memcpy(dom_out, domRes, sizeof(uint64_t) * T->D);
    if (ct_out) memcpy(ct_out, T->pCt, sizeof(uint64_t) * T->W);
  } else if (status == CT_FAIL) {
    S.failed = 1;
    if (ct_out) memset(ct_out, 0, sizeof(uint64_t) * T->W);
  }
  if (st) {
    if ((rc = ct_slot_stats(T, slot, st))) return rc;
  }
  switch (status) {
    case CT_OK:
    case CT_FAIL:
      return status;
    case CT_E_NOT_SUBSET:
      return fail(status, "dom_in is not a subset of the slot's domains");
    case CT_E_INVALID:
      return fail(status, "dom_in has stray bits");
    case CT_E_STATE:
      return fail(status, "slot is failed; only pop is allowed");
    default:
      T->poisoned = true;
      return fail(CT_E_DEVICE, "unexpected device status %d", status);
  }
}

int ct_propagate(ct_table* T, const uint64_t* dom_in, uint64_t* dom_out, uint64_t* ct_out,
                 ct_stats* st) {
  return ct_propagate_slot(T, 0, dom_in, dom_out, ct_out, st);
}

int ct_get_state(ct_table* T, int32_t slot, uint64_t* dom_out, uint64_t* ct_out) {
  int rc = check_poison(T);
  if (rc) return rc;
  if ((rc = check_slot(T, slot))) return rc;
  if ((rc = quiesce(T))) return rc;
  if ((rc = flush_slot(T, slot))) return rc;
  HIPCHK(hipStreamSynchronize(T->stream));
  SlotDesc s{};
  HIPCHK(hipMemcpy(&s, T->slots[slot].dev, sizeof(SlotDesc), hipMemcpyDeviceToHost));
  if (dom_out) HIPCHK(hipMemcpy(dom_out, s.lastDom, sizeof(uint64_t) * T->D, hipMemcpyDeviceToHost));
  if (ct_out && T->W > 0) {
    if (s.failed) {
      memset(ct_out, 0, sizeof(uint64_t) * T->W);
    } else {
      HIPCHK(hipMemcpy(ct_out, s.ct, sizeof(uint64_t) * T->W, hipMemcpyDeviceToHost));
    }
  }
  return CT_OK;
}

int ct_slot_stats(ct_table* T, int32_t slot, ct_stats* st) {
  int rc = check_poison(T);
  if (rc) return rc;
  if ((rc = check_slot(T, slot))) return rc;
  if (!st) return fail(CT_E_INVALID, "st is NULL");
  SlotDesc s{};
  if (slot == 0 && T->engOn && T->engStatsFresh && __atomic_load_n(&T->pRes->alive, __ATOMIC_ACQUIRE) != 0) {
    // the engine holds the counters: its snapshot after the last call
    for (int k = 0; k < 8; ++k) s.stats[k] = T->engStats[k];
  } else {
    if ((rc = quiesce(T))) return rc;
    HIPCHK(hipStreamSynchronize(T->stream));
    HIPCHK(hipMemcpy(&s, T->slots[slot].dev, sizeof(SlotDesc), hipMemcpyDeviceToHost));
  }
  st->jobs = (int64_t)s.stats[S_JOBS];
  st->granules_in = (int64_t)s.stats[S_GRAN_IN];
  st->rows_or = (int64_t)s.stats[S_ROWS];
  st->granule_rows = (int64_t)s.stats[S_GRAN_ROWS];
  st->trail_granules = (int64_t)s.stats[S_TRAIL];
  st->residue_checks = (int64_t)s.stats[S_RES_CHECK];
  st->residue_misses = (int64_t)s.stats[S_RES_MISS];
  st->scan_granules = (int64_t)s.stats[S_SCAN];
  return CT_OK;
}

int ct_batch_status(void* stream_v) {
  hipStream_t stream = (hipStream_t)stream_v;
  int rc = noalloc_status(stream);
  if (rc) return rc;
  QueueCtx* q = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_qmu);
    auto it = g_queues.find(stream);
    if (it == g_queues.end()) return CT_OK;
    q = it->second;
  }
  HIPCHK(hipStreamSynchronize(stream));
  const int32_t err = *(volatile int32_t*)q->hostErr;
  if (!err) return CT_OK;
  *q->hostErr = 0;
  HIPCHK(hipMemsetAsync(q->queue + 3, 0, sizeof(int32_t), stream));
  HIPCHK(hipStreamSynchronize(stream));
  return fail(CT_E_DEVICE, "device-side error %d in a batch on this stream (wait timeout or trail "
              "overflow); the slots of that batch are undefined", err);
}

static const unsigned long long kClockInit[5] = {~0ull, 0ull, 0ull, 0ull, 0ull};

int ct_set_timing(ct_table* T, int32_t on) {
  int rc = check_poison(T);
  if (rc) return rc;
  HIPCHK(hipStreamSynchronize(T->stream));
  if (on && !T->dClock) {
    if ((rc = dev_alloc(T, (void**)&T->dClock, sizeof(kClockInit)))) return rc;
  }
  if (T->dClock) HIPCHK(hipMemcpy(T->dClock, kClockInit, sizeof(kClockInit), hipMemcpyHostToDevice));
  T->timing = on != 0;
  T->engTicks = 0;
  T->engCalls = 0;
  T->engLifeTicks = 0;
  T->engLaunches = 0;
  return CT_OK;
}

int ct_get_dispatch_timing(ct_table* T, double* dispatch_ms, int64_t* dispatches) {
  if (!T) return fail(CT_E_INVALID, "null table");
  unsigned long long c[5] = {0, 0, 0, 0, 0};
  if (T->dClock) {
    int rc = quiesce(T);  // also ends a running engine: its lifetime is then known
    if (rc) return rc;
    HIPCHK(hipStreamSynchronize(T->stream));
    HIPCHK(hipMemcpy(c, T->dClock, sizeof(c), hipMemcpyDeviceToHost));
  }
  int dev = 0, khz = 0;
  HIPCHK(hipGetDevice(&dev));
  HIPCHK(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
  if (dispatch_ms) *dispatch_ms = khz > 0 ? (double)(c[3] + T->engLifeTicks) / (double)khz : 0.0;
  if (dispatches) *dispatches = (int64_t)(c[4] + T->engLaunches);
  return CT_OK;
}

int ct_get_timing(ct_table* T, double* kernel_ms, int64_t* launches) {
  if (!T) return fail(CT_E_INVALID, "null table");
  unsigned long long c[5] = {0, 0, 0, 0, 0};
  if (T->dClock) {
    int rc = quiesce(T);  // launched calls on the table's stream have ended
    if (rc) return rc;
    HIPCHK(hipStreamSynchronize(T->stream));
    HIPCHK(hipMemcpy(c, T->dClock, sizeof(c), hipMemcpyDeviceToHost));
  }
  int dev = 0, khz = 0;
  HIPCHK(hipGetDevice(&dev));
  HIPCHK(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
  // launched calls, plus calls served by the resident engine (device time of
  // each call inside the engine)
  if (kernel_ms) *kernel_ms = khz > 0 ? (double)(c[3] + T->engTicks) / (double)khz : 0.0;
  if (launches) *launches = (int64_t)(c[4] + T->engCalls);
  return CT_OK;
}

}  // extern "C"

namespace {

// What a validated batch needs, before any slot's host state changes.
struct BatchPlan {
  bool nodes = false;
  size_t stagedBytes = 0;  // staged scratch of all jobs at once
  bool streamRoots = false;  // all jobs are roots, with enough granules for the streaming update
  size_t nodesBytes = 0;   // search-node records, row vectors and non-zero words
  size_t descBytes = 0;    // job descriptors
  // what a no-allocation batch is held to: the descriptors, three ints a job
  // and, for a batch of roots, two ints for every WAVES granules
  size_t rootInts = 0, limitBytes = 0;
};

// nodes: the batch runs on the search-node schedule if it is one
BatchPlan batch_plan(const ct_job* jobs, int n_jobs, bool nodes) {
  BatchPlan p;
  p.nodes = nodes;
  if (p.nodes) {
    const ct_table* T = jobs[0].table;
    p.nodesBytes = nodes_scratch_bytes(T->nodesVecRows, n_jobs, T->nGran);
  } else {
    if (use_roots(jobs, n_jobs))
      for (int j = 0; j < n_jobs; ++j) p.rootInts += 2 * ((size_t)(jobs[j].table->nGran + WAVES - 1) / WAVES);
    StageNeed need;
    bool roots = true;
    int64_t granules = 0;
    for (int j = 0; j < n_jobs; ++j) {
      const ct_table* T = jobs[j].table;
      const bool propagate = jobs[j].flags & CT_JOB_PROPAGATE, root = jobs[j].flags & CT_JOB_ROOT;
      roots = roots && root && T->kind != CT_KIND_NEGATIVE;
      granules += T->nGran;
      if (batch_staged(T, propagate)) need.add(T, propagate, false, root);
    }
    p.stagedBytes = need.bytes();
    p.streamRoots = roots && stage_stream_roots(granules);
  }
  p.descBytes = align256(sizeof(DevJob) * (size_t)n_jobs);
  p.limitBytes = p.descBytes + sizeof(int32_t) * (2 * (size_t)(n_jobs + 1) + (size_t)n_jobs + 2 + p.rootInts);
  return p;
}

// Where a batch's scratch lives: device counters, staging and search-node
// scratch, and the host arrays the descriptors are built in.  Capacities
// must cover the batch's plan.
struct BatchRes {
  int32_t* queue = nullptr;     // device: [3] error word
  int32_t* hostErr = nullptr;   // pinned, nullable
  char* dStage = nullptr;       // device staging
  char* hStage = nullptr;       // host staging (the source of the one copy)
  char* hStageDev = nullptr;    // its device address (pinned), or null
  void* dNodes = nullptr;
  DevJob* hJobs = nullptr;      // n_jobs
  int32_t* chunks = nullptr;    // n_jobs
  uint64_t* order = nullptr;    // n_jobs
  char* dStaged = nullptr;      // staged scratch
  size_t capStaged = 0;
  size_t countBytes = 0;        // not 0: the copy's first bytes are the staged schedule's item counts
};

// Builds the descriptors of a validated batch (applying its pops and pushes
// to the slots' host mirrors), stages them and launches it.
int batch_launch(const ct_job* jobs, int n_jobs, hipStream_t stream, int32_t* status_dev, const BatchPlan& p,
                 const BatchRes& r) {
  const BatchShape B = batch_build(jobs, n_jobs, status_dev, p.nodes, p.streamRoots, r.capStaged, r.hJobs, r.chunks, r.order);
  memset(r.hStage, 0, r.countBytes);
  memcpy(r.hStage + r.countBytes, r.hJobs, sizeof(DevJob) * n_jobs);
  // A staged batch's descriptors are read once, by the prep, straight from the
  // pinned buffer (each workgroup's read takes about 2 us; a copy between the
  // launches 12-20 us a batch)
  const bool direct = r.hStageDev && !p.nodes && B.nStaged == n_jobs;
  DevJob* dJobs = (DevJob*)((direct ? r.hStageDev : r.dStage) + r.countBytes);
  if (!direct)
    HIPCHK(hipMemcpyAsync(r.dStage, r.hStage, r.countBytes + sizeof(DevJob) * (size_t)n_jobs, hipMemcpyHostToDevice,
                          stream));
  KArgs a{};
  a.jobs = dJobs;
  a.nJobs = n_jobs;
  a.queue = r.queue;
  a.hostErr = r.hostErr;
  if (p.nodes) {
    const ct_table* T = jobs[0].table;
    NodesDesc N{};
    N.tab = T->dTab;
    N.jobs = dJobs;
    N.S = T->hTab.S;
    N.ids = T->dIds;
    N.stride = T->stride;
    N.W = T->W;
    N.nJobs = n_jobs;
    N.D = T->D;
    N.nGran = T->nGran;
    N.n2 = (T->n + 1) & ~1;
    N.vecRows = T->nodesVecRows;
    for (int j = 0; j < n_jobs && !N.anyOut; ++j) N.anyOut = jobs[j].ct_out != nullptr;
    HIPCHK(launch_nodes(N, (char*)r.dNodes, stream));
    return CT_OK;
  }
  for (int k = 0; k < B.nChunks; ++k) {
    const int j0 = r.chunks[k], j1 = k + 1 < B.nChunks ? r.chunks[k + 1] : B.nStaged;
    StageNeed need;
    need.wide = B.wide;
    need.wideDom = B.wideDom;
    for (int j = j0; j < j1; ++j) need.add_items(r.hJobs[j].nUpd, r.hJobs[j].nFilt);
    StageArgs A = stage_args(need, r.dStaged, r.queue, r.hostErr, r.countBytes ? (StageCounts*)r.dStage : nullptr);
    A.roots = p.streamRoots;
    a.jobs = dJobs + j0;
    a.nJobs = need.nJobs;
    HIPCHK(launch_staged(a, A, need.nU, need.nF, B.popGran, stream));
  }
  if (B.nStaged < n_jobs) {
    a.jobs = dJobs + B.nStaged;
    a.nJobs = n_jobs - B.nStaged;
    HIPCHK(launch_propagate(a, std::min(a.nJobs, propagate_max_grid()), stream));
  }
  return CT_OK;
}

// ct_propagate_batch_noalloc: fixed limits of the static scratch (device
// array in ct_noalloc.hip) and of the host arrays the descriptors are built in
constexpr int NA_MAX_JOBS = 8192;
constexpr size_t NA_QUEUE_BYTES = 256;
constexpr size_t NA_STAGE_BYTES = (size_t)2 << 20;
constexpr size_t NA_MAX_TASK_INTS = (NA_STAGE_BYTES - (size_t)NA_MAX_JOBS * 128) / sizeof(int32_t);
static_assert(sizeof(StageCounts) + 256 + NA_MAX_JOBS * sizeof(DevJob) <= NA_STAGE_BYTES, "the largest batch's copy");

// The documented limit of a no-allocation search-node batch (tables of at
// most NA_NODES_ROWS support rows): per node a row list and a flag byte per
// granule.
constexpr int NA_NODES_ROWS = 256;
size_t na_nodes_bytes(const ct_table* T, int n_jobs) {
  const size_t nodeWords = 4 + (size_t)(((T->rows + 3 * T->n + 3) & ~3) / 4);
  return align256(sizeof(uint64_t) * (size_t)n_jobs * nodeWords) + align256((size_t)n_jobs * T->nGran);
}

struct NoAllocHost {
  std::mutex mu;  // the host arrays are shared by every caller
  bool used = false;
  hipStream_t lastStream = nullptr;  // the stream of the last call (ct_batch_status)
  DevJob jobs[NA_MAX_JOBS];
  int32_t chunks[NA_MAX_JOBS];
  uint64_t order[NA_MAX_JOBS];
  alignas(256) char stage[NA_STAGE_BYTES];
};
NoAllocHost g_na;

int noalloc_status(hipStream_t stream) {
  std::lock_guard<std::mutex> lk(g_na.mu);
  if (!g_na.used || g_na.lastStream != stream) return CT_OK;
  char* scratch = nullptr;
  size_t bytes = 0;
  HIPCHK(noalloc_scratch(&scratch, &bytes));
  HIPCHK(hipStreamSynchronize(stream));
  int32_t err = 0;  // of a call since the last look
  HIPCHK(hipMemcpy(&err, scratch + 3 * sizeof(int32_t), sizeof(err), hipMemcpyDeviceToHost));
  if (!err) return CT_OK;
  const int32_t zero = 0;
  HIPCHK(hipMemcpy(scratch + 3 * sizeof(int32_t), &zero, sizeof(zero), hipMemcpyHostToDevice));
  return fail(CT_E_DEVICE, "device-side error %d in a ct_propagate_batch_noalloc call on this stream (wait "
              "timeout or trail overflow); the slots of that batch are undefined", err);
}

int batch_queue(const ct_job* jobs, int n_jobs, hipStream_t stream, int32_t* status_dev) {
  int rc = batch_validate_quiesce(jobs, n_jobs, stream);
  if (rc) return rc;
  QueueCtx* q = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_qmu);
    auto it = g_queues.find(stream);
    if (it == g_queues.end()) {
      q = new QueueCtx();
      int rc = queue_init(*q);
      if (rc) {
        queue_free(*q);
        delete q;
        return rc;
      }
      g_queues[stream] = q;
    } else {
      q = it->second;
    }
  }
  const BatchPlan p = batch_plan(jobs, n_jobs, nodes_batch(jobs, n_jobs) && nodes_ids_ensure(jobs[0].table));
  // device and pinned scratch, grown before any slot's host state changes:
  // a failed allocation leaves the slots as they were
  if (p.nodes && q->capNodes < p.nodesBytes) {
    HIPCHK(hipStreamSynchronize(stream));
    if (q->dNodes) (void)hipFree(q->dNodes);
    q->dNodes = nullptr;
    q->capNodes = 0;
    ALLOCCHK(hipMalloc(&q->dNodes, p.nodesBytes));
    q->capNodes = p.nodesBytes;
  }
  if (p.stagedBytes) {
    rc = stage_reserve(*q, std::min(p.stagedBytes, STAGE_SCRATCH), stream);
    if (rc) return rc;
  }
  if (q->capStage < p.descBytes) {
    HIPCHK(hipStreamSynchronize(stream));
    if (q->dStage) (void)hipFree(q->dStage);
    for (int k = 0; k < 2; ++k)
      if (q->pStage[k]) (void)hipHostFree(q->pStage[k]);
    const size_t cap = std::max({2 * p.descBytes, 2 * q->capStage, STAGE_BUFFER});
    q->dStage = nullptr;
    q->pStage[0] = q->pStage[1] = nullptr;
    q->capStage = q->usedStage = 0;
    ALLOCCHK(hipMalloc(&q->dStage, cap));
    for (int k = 0; k < 2; ++k) {
      ALLOCCHK(hipHostMalloc((void**)&q->pStage[k], cap, hipHostMallocDefault));
      HIPCHK(hipHostGetDevicePointer((void**)&q->pStageDev[k], q->pStage[k], 0));
    }
    q->capStage = cap;
  }
  q->hJobs.resize(n_jobs);
  q->chunks.resize(n_jobs);
  q->order.resize(n_jobs);
  // the next buffer when this one is full: its batches of last time have ended
  if (q->usedStage + p.descBytes > q->capStage) {
    HIPCHK(hipEventRecord(q->staged[q->turn], stream));
    q->turn ^= 1;
    q->usedStage = 0;
    HIPCHK(hipEventSynchronize(q->staged[q->turn]));
  }
  BatchRes r;
  r.queue = q->queue;
  r.hostErr = q->hostErr;
  r.dStage = q->dStage;
  r.hStage = q->pStage[q->turn] + q->usedStage;
  r.hStageDev = q->pStageDev[q->turn] + q->usedStage;
  q->usedStage += p.descBytes;
  r.dNodes = q->dNodes;
  r.hJobs = q->hJobs.data();
  r.chunks = q->chunks.data();
  r.order = q->order.data();
  r.dStaged = q->dStaged;
  r.capStaged = q->capStaged;
  rc = batch_launch(jobs, n_jobs, stream, status_dev, p, r);
  // (a launch that failed may have left item counts: the scratch is made anew)
  if (rc) q->capStaged = 0;
  return rc;
}

}  // namespace

extern "C" {

int ct_propagate_batch(const ct_job* jobs, int32_t n_jobs, void* stream_v, int32_t* status_dev) {
  if (n_jobs < 0 || (n_jobs > 0 && (!jobs || !status_dev)))
    return fail(CT_E_INVALID, "bad batch arguments");
  if (n_jobs == 0) return CT_OK;
  try {
    return batch_queue(jobs, n_jobs, (hipStream_t)stream_v, status_dev);
  } catch (const std::bad_alloc&) {  // (before any slot's host state changes: its lists are reserved)
    return fail(CT_E_NOMEM, "host allocation failed");
  }
}

int ct_propagate_batch_noalloc(const ct_job* jobs, int32_t n_jobs, void* stream_v, int32_t* status_dev) {
  if (n_jobs < 0 || (n_jobs > 0 && (!jobs || !status_dev)))
    return fail(CT_E_INVALID, "bad batch arguments");
  if (n_jobs == 0) return CT_OK;
  if (n_jobs > NA_MAX_JOBS)
    return fail(CT_E_INVALID, "ct_propagate_batch_noalloc: %d jobs, at most %d", n_jobs, NA_MAX_JOBS);
  for (int j = 0; j < n_jobs; ++j)
    if (!jobs[j].table) return fail(CT_E_INVALID, "job %d: table is NULL", j);
  char* scratch = nullptr;
  size_t scratchBytes = 0;
  HIPCHK(noalloc_scratch(&scratch, &scratchBytes));
  const size_t nodesCap = scratchBytes - NA_QUEUE_BYTES - NA_STAGE_BYTES;
  // (the row numbers of the search-node schedule are made by ct_slots_alloc)
  const bool nodes = nodes_batch(jobs, n_jobs);
  if (nodes_form(jobs, n_jobs) && jobs[0].table->rows <= NA_NODES_ROWS &&
      na_nodes_bytes(jobs[0].table, n_jobs) > nodesCap)
    return fail(CT_E_INVALID, "ct_propagate_batch_noalloc: the search-node schedule needs %zu scratch bytes, "
                "at most %zu", na_nodes_bytes(jobs[0].table, n_jobs), nodesCap);
  BatchPlan p = batch_plan(jobs, n_jobs, nodes && jobs[0].table->dIds);
  if (p.nodesBytes > nodesCap) p = batch_plan(jobs, n_jobs, false);
  if (p.limitBytes > NA_STAGE_BYTES || p.rootInts > NA_MAX_TASK_INTS)
    return fail(CT_E_INVALID, "ct_propagate_batch_noalloc: the batch needs %zu staging bytes, at most %zu",
                p.limitBytes, NA_STAGE_BYTES);
  hipStream_t stream = (hipStream_t)stream_v;
  std::lock_guard<std::mutex> lk(g_na.mu);
  int rc = batch_validate_quiesce(jobs, n_jobs, stream);
  if (rc) return rc;
  BatchRes r;
  r.queue = (int32_t*)scratch;
  r.dStage = scratch + NA_QUEUE_BYTES;
  r.hStage = g_na.stage;
  r.dNodes = scratch + NA_QUEUE_BYTES + NA_STAGE_BYTES;
  r.hJobs = g_na.jobs;
  r.chunks = g_na.chunks;
  r.order = g_na.order;
  r.dStaged = (char*)r.dNodes;
  r.capStaged = nodesCap;
  // the item counts start at zero, whatever an earlier call left: they come
  // with the descriptors' copy (a kernel that cleared them took the stream 5 us)
  r.countBytes = align256(sizeof(StageCounts));
  g_na.used = true;
  g_na.lastStream = stream;
  return batch_launch(jobs, n_jobs, stream, status_dev, p, r);
}


}  // extern "C"

// internal accessors used by the serving loop (ct_server.cpp)
namespace ctk {
int64_t slot_footprint(const ct_table* T, int maxDepth) {
  const int64_t trailCap = (int64_t)maxDepth * T->nGran;
  return (int64_t)(align256(sizeof(uint64_t) * T->stride) + 4 * align256(sizeof(int32_t) * T->nGran) +
                   align256(sizeof(uint64_t) * T->D) + align256(sizeof(int32_t) * T->rows) +
                   align256(sizeof(TrailHdr) * std::max<int64_t>(trailCap, 1)) +
                   align256(sizeof(uint64_t) * GW * std::max<int64_t>(trailCap, 1)) +
                   align256(sizeof(Level) * std::max(maxDepth, 1)) +
                   align256(sizeof(uint64_t) * T->D * std::max(maxDepth, 1)) + sizeof(SlotDesc));
}

int root_domains(ct_table* T, uint64_t* out) {
  HIPCHK(hipMemcpy(out, T->hRoot.lastDom, sizeof(uint64_t) * T->D, hipMemcpyDeviceToHost));
  return CT_OK;
}

void set_error(const char* msg) { snprintf(g_err, sizeof(g_err), "%s", msg); }

// Read-only view of a table for the split propagators (ct_split.cpp): the
// supports, the layout and the root state never change after ct_create.
int table_view(const ct_table* T, TableView* v) {
  int rc = check_poison(T);
  if (rc) return rc;
  v->S = T->dS;
  v->stride = T->stride;
  v->W = T->W;
  v->n = T->n;
  v->D = T->D;
  v->rows = T->rows;
  v->rootFailed = T->rootFailed;
  v->branchPolicy = T->cfg.branch_policy;
  v->kind = T->kind;
  v->vars = T->vars.data();
  v->rootCt = T->hRoot.ct;
  v->rootDom = T->hRoot.lastDom;
  return CT_OK;
}
}  // namespace ctk

// ===========================================================================
// Multi-table model: propagation rounds, launched ahead of the host
// ===========================================================================
namespace ctk {
hipError_t launch_model_start(const ModelRound& M, const uint64_t* poolIn, const int32_t* off,
                              const uint64_t* const* src, hipStream_t stream);
hipError_t launch_model_prep(const KArgs& a, const StageArgs& A, const ModelRound& M, hipStream_t stream);
hipError_t launch_model_items(const StageArgs& A, const ModelRound& M, int nU, int nF, const ModelNeg& neg,
                              hipStream_t stream);
}

struct ct_model {
  int nPool = 0, poolWords = 0;
  std::vector<int32_t> lo, dsz, poolOff, poolNW;
  std::vector<ct_table*> tabs;
  std::vector<std::vector<int32_t>> scopes;
  hipStream_t stream = nullptr;
  QueueCtx q;
  int soloMax = 4;
  // (solo, tile) per class of tables (granule bucket, rows bucket), set by the
  // autotuner; classes without an entry follow soloMax.  Reported only: rounds
  // run staged whichever it is.
  std::map<std::pair<int, int>, std::pair<int, int>> choice;
  // device state, rebuilt when the table set or the schedule changes
  bool built = false;
  std::vector<void*> blocks;
  uint64_t* pool[3] = {nullptr, nullptr, nullptr};  // cur, next, prev in turn
  ModelState* state = nullptr;
  int32_t* startOff = nullptr;         // per pool word, its words in the tables' last domains:
  const uint64_t** startSrc = nullptr; //   startSrc[startOff[w] .. startOff[w + 1])
  KArgs a{};
  StageArgs A{};
  int nU = 0, nF = 0;
  ModelNeg neg{};
  DevJob* dJobs = nullptr;
  std::vector<DevJob> hJobs;       // the staged jobs, then those of the propagate kernel
  std::vector<int32_t> jobOf;      // table -> its job
  uint64_t* pHost = nullptr;   // pinned: how the last finished round ended (ModelRound::host)
  uint32_t call = 0;           // fixpoints run: marks their words
  int32_t* dStatus = nullptr;  // statuses of push/pop batches
};

namespace {

int model_alloc(ct_model* m, void** p, size_t bytes) {
  if (alloc_injected()) return fail(CT_E_NOMEM, "injected allocation failure: hipMalloc(%zu)", bytes);
  hipError_t e = hipMalloc(p, bytes ? bytes : 8);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(CT_E_NOMEM, "hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
  }
  m->blocks.push_back(*p);
  return CT_OK;
}

void model_free_device(ct_model* m) {
  if (m->stream) (void)hipStreamSynchronize(m->stream);
  for (void* p : m->blocks) (void)hipFree(p);
  m->blocks.clear();
  m->dStatus = nullptr;
  m->dJobs = nullptr;
  m->built = false;
}

template <class T>
int model_upload(ct_model* m, T** dst, const std::vector<T>& src) {
  int rc = model_alloc(m, (void**)dst, sizeof(T) * std::max<size_t>(src.size(), 1));
  if (rc) return rc;
  if (!src.empty()) HIPCHK(hipMemcpy(*dst, src.data(), sizeof(T) * src.size(), hipMemcpyHostToDevice));
  return CT_OK;
}

// Class of a table for the autotuner: floor(log4) of its granule count and
// of its support-row count.
int log4_bucket(int64_t x) {
  int b = 0;
  while (x >= 4) {
    x /= 4;
    ++b;
  }
  return b;
}

std::pair<int, int> table_class(const ct_table* T) { return {log4_bucket(T->nGran), log4_bucket(T->rows)}; }

// (solo, tile) of a table
std::pair<int, int> model_choice(const ct_model* m, const ct_table* T) {
  auto it = m->choice.find(table_class(T));
  if (it != m->choice.end()) return it->second;
  return {T->nGran <= m->soloMax ? 1 : 0, 0};
}

// Device arrays and one propagate job per table.
int model_build(ct_model* m) {
  model_free_device(m);
  const int nT = (int)m->tabs.size();
  int rc;
  for (int k = 0; k < 3; ++k)
    if ((rc = model_alloc(m, (void**)&m->pool[k], sizeof(uint64_t) * m->poolWords))) return rc;
  if ((rc = model_alloc(m, (void**)&m->state, sizeof(ModelState)))) return rc;
  if ((rc = model_alloc(m, (void**)&m->dStatus, sizeof(int32_t) * std::max(nT, 1)))) return rc;
  // per table the pool word of each of its domain words; per pool word the
  // addresses of its words in the tables' last domains
  std::vector<int32_t> map;
  std::vector<size_t> mapOff(nT);
  std::vector<int32_t> startOff(m->poolWords + 1, 0);
  std::vector<const uint64_t*> last(nT);
  size_t negWords = 0;
  for (int c = 0; c < nT; ++c) {
    ct_table* T = m->tabs[c];
    SlotDesc sd{};
    HIPCHK(hipMemcpy(&sd, T->slots[0].dev, sizeof(SlotDesc), hipMemcpyDeviceToHost));
    last[c] = (const uint64_t*)sd.lastDom;
    mapOff[c] = map.size();
    map.resize(map.size() + T->D);
    for (int k = 0; k < T->n; ++k) {
      const int v = m->scopes[c][k];
      for (int q = 0; q < m->poolNW[v]; ++q) {
        map[mapOff[c] + T->domOff[k] + q] = m->poolOff[v] + q;
        ++startOff[m->poolOff[v] + q + 1];
      }
    }
    if (T->kind == CT_KIND_NEGATIVE) negWords += T->D;
  }
  for (int w = 0; w < m->poolWords; ++w) startOff[w + 1] += startOff[w];
  std::vector<const uint64_t*> startSrc(map.size());
  {
    std::vector<int32_t> at(startOff.begin(), startOff.end() - 1);
    for (int c = 0; c < nT; ++c)
      for (int q = 0; q < m->tabs[c]->D; ++q) startSrc[at[map[mapOff[c] + q]]++] = last[c] + q;
  }
  int32_t* dMap = nullptr;
  if ((rc = model_upload(m, &dMap, map))) return rc;
  if ((rc = model_upload(m, &m->startOff, startOff))) return rc;
  if ((rc = model_upload(m, &m->startSrc, startSrc))) return rc;
  // jobs: the staged ones, then the negative tables', on buffers of their own
  m->hJobs.assign(nT, DevJob{});
  m->jobOf.assign(nT, 0);
  uint64_t *negIn = nullptr, *negOut = nullptr;
  int32_t *negStatus = nullptr, *negDirty = nullptr;
  std::vector<const int32_t*> negMaps;
  if (negWords) {
    if ((rc = model_alloc(m, (void**)&negIn, sizeof(uint64_t) * negWords))) return rc;
    if ((rc = model_alloc(m, (void**)&negOut, sizeof(uint64_t) * negWords))) return rc;
    if ((rc = model_alloc(m, (void**)&negStatus, sizeof(int32_t) * nT))) return rc;
    if ((rc = model_alloc(m, (void**)&negDirty, sizeof(int32_t) * nT))) return rc;
  }
  StageNeed need;
  int at = 0;
  for (int pass = 0; pass < 2; ++pass)
    for (int c = 0; c < nT; ++c) {
      ct_table* T = m->tabs[c];
      const bool negative = T->kind == CT_KIND_NEGATIVE;
      if (negative != (pass == 1)) continue;
      m->jobOf[c] = at;
      DevJob& J = m->hJobs[at++];
      J.tab = T->dTab;
      J.slot = T->slots[0].dev;
      J.flags = JF_PROPAGATE | (negative ? JF_SOLO : JF_MODEL);
      J.depthAfter = T->slots[0].depth;
      if (negative) {
        J.dom_in = negIn;
        J.dom_out = negOut;
        negIn += T->D;
        negOut += T->D;
        J.status_out = negStatus + negMaps.size();
        J.active = negDirty + negMaps.size();
        negMaps.push_back(dMap + mapOff[c]);
        continue;
      }
      J.dom_in = (const uint64_t*)(dMap + mapOff[c]);
      J.stageOff = (int32_t)(need.jobBytes / 256);
      J.listCap = stage_list_cap(T);
      need.add(T, true, false);
    }
  if ((rc = model_upload(m, &m->dJobs, m->hJobs))) return rc;
  char* scratch = nullptr;
  if ((rc = model_alloc(m, (void**)&scratch, need.bytes()))) return rc;
  HIPCHK(hipMemsetAsync(scratch, 0, sizeof(StageCounts), m->stream));
  m->a = KArgs{};
  m->a.jobs = m->dJobs;
  m->a.nJobs = need.nJobs;
  m->a.queue = m->q.queue;
  m->a.hostErr = m->q.hostErr;
  m->neg = ModelNeg{};
  m->neg.a = m->a;
  m->neg.a.jobs = m->dJobs + need.nJobs;
  m->neg.a.nJobs = nT - need.nJobs;
  const int32_t** dMaps = nullptr;
  if ((rc = model_upload(m, &dMaps, negMaps))) return rc;
  m->neg.maps = dMaps;
  m->neg.dirty = negDirty;
  m->A = stage_args(need, scratch, m->q.queue, m->q.hostErr);
  m->nU = need.nU;
  m->nF = need.nF;
  m->built = true;
  return CT_OK;
}

// Bring every table's slot 0 up to date (pending pushes/pops) and refresh the
// depth each job trails at.
int model_sync_tables(ct_model* m) {
  bool changed = false;
  for (size_t c = 0; c < m->tabs.size(); ++c) {
    ct_table* T = m->tabs[c];
    int rc = check_poison(T);
    if (rc) return rc;
    if ((rc = flush_slot(T, 0))) return rc;
    if ((rc = quiesce(T, m->stream))) return rc;
    // only a synchronous call's unfinished tail can still be on the table's
    // stream (everything else on it is waited for where it is queued)
    if (T->tailPending) {
      HIPCHK(hipStreamSynchronize(T->stream));
      T->tailPending = false;
    }
    // a round's job only asks whether levels exist (depth > 0: trail the
    // words it changes), so the job array is sent again only when that flips
    if (m->built && (m->hJobs[m->jobOf[c]].depthAfter > 0) != (T->slots[0].depth > 0)) {
      m->hJobs[m->jobOf[c]].depthAfter = T->slots[0].depth;
      changed = true;
    }
  }
  if (changed)
    HIPCHK(hipMemcpy(m->dJobs, m->hJobs.data(), sizeof(DevJob) * m->hJobs.size(), hipMemcpyHostToDevice));
  return CT_OK;
}

int model_push_pop(ct_model* m, bool push) {
  const int nT = (int)m->tabs.size();
  if (nT == 0) return CT_OK;
  if (!m->dStatus) {
    int rc = model_alloc(m, (void**)&m->dStatus, sizeof(int32_t) * nT);
    if (rc) return rc;
  }
  // a built model has its tables' descriptors on the device: one launch with
  // the same pop or push for each
  bool direct = m->built;
  int popGran = 0;
  int32_t serial = 0;
  for (int c = 0; c < nT && direct; ++c) {
    const ct_table* T = m->tabs[c];
    const SlotHost& S = T->slots[0];
    direct = !T->poisoned && !S.freed && S.pendPop == 0 && S.pendPush == 0 && (push ? S.depth < S.maxDepth : S.depth > 0);
    popGran = std::max(popGran, T->nGran);
    serial = std::max(serial, T->serialCounter);
  }
  for (int c = 0; c < nT && direct; ++c) {
    ct_table* T = m->tabs[c];
    int rc = quiesce(T, m->stream);
    if (rc) return rc;
    if (T->tailPending) {
      HIPCHK(hipStreamSynchronize(T->stream));
      T->tailPending = false;
    }
  }
  if (direct) {
    for (ct_table* T : m->tabs) {
      SlotHost& S = T->slots[0];
      if (push) S.failedAt.push_back(2);
      else S.failedAt.pop_back();
      S.depth += push ? 1 : -1;
      S.failed = 2;
      if (push) T->serialCounter = serial + 1;
      T->pendStream = m->stream;
    }
    KArgs a = m->a;
    a.nJobs = nT;
    a.uniform = 1;
    a.job.nPop = push ? 0 : 1;
    a.job.nPush = push ? 1 : 0;
    a.job.serialBase = serial;
    HIPCHK(launch_staged(a, m->A, 0, 0, push ? 0 : popGran, m->stream));
    return CT_OK;
  }
  std::vector<ct_job> jobs(nT);
  for (int c = 0; c < nT; ++c) {
    jobs[c] = ct_job{};
    jobs[c].table = m->tabs[c];
    jobs[c].slot = 0;
    jobs[c].flags = 0;
    jobs[c].n_pop = push ? 0 : 1;
    jobs[c].n_push = push ? 1 : 0;
  }
  // queued on the model's stream, ahead of the next fixpoint's rounds; a
  // device-side error of this batch is reported by that fixpoint, and any
  // other use of a table waits for it (quiesce)
  int rc = ct_propagate_batch(jobs.data(), nT, m->stream, m->dStatus);
  if (rc) return rc;
  for (ct_table* T : m->tabs) T->pendStream = m->stream;
  return CT_OK;
}

}  // namespace

extern "C" {

int ct_model_create(int32_t n_vars, const int32_t* dom_lo, const int32_t* dom_size, ct_model** out) {
  if (!out) return fail(CT_E_INVALID, "out is NULL");
  *out = nullptr;
  if (n_vars < 1 || !dom_lo || !dom_size) return fail(CT_E_INVALID, "bad model arguments");
  ct_model* m = new (std::nothrow) ct_model();
  if (!m) return fail(CT_E_NOMEM, "host allocation failed");
  m->nPool = n_vars;
  int w = 0;
  for (int i = 0; i < n_vars; ++i) {
    if (dom_size[i] < 1) {
      delete m;
      return fail(CT_E_INVALID, "dom_size[%d] < 1", i);
    }
    m->lo.push_back(dom_lo[i]);
    m->dsz.push_back(dom_size[i]);
    m->poolOff.push_back(w);
    m->poolNW.push_back((dom_size[i] + 63) / 64);
    w += (dom_size[i] + 63) / 64;
  }
  m->poolWords = w;
  hipError_t e = hipStreamCreateWithFlags(&m->stream, hipStreamNonBlocking);
  if (e != hipSuccess) {
    delete m;
    return fail(CT_E_DEVICE, "hipStreamCreate failed: %s", hipGetErrorString(e));
  }
  int rc = queue_init(m->q);
  if (rc == CT_OK) {
    e = hipHostMalloc((void**)&m->pHost, sizeof(uint64_t) * 2, hipHostMallocMapped | hipHostMallocCoherent);
    if (e == hipSuccess) memset(m->pHost, 0, sizeof(uint64_t) * 2);
    if (e != hipSuccess) rc = fail(CT_E_NOMEM, "pinned allocation failed");
  }
  if (rc) {
    ct_model_destroy(m);
    return rc;
  }
  *out = m;
  return CT_OK;
}

void ct_model_destroy(ct_model* m) {
  if (!m) return;
  model_free_device(m);  // waits for the model's stream
  {
    // the live tables no longer wait for this stream
    std::lock_guard<std::mutex> lk(g_engMu);
    for (ct_table* T : m->tabs)
      if (g_tables.count(T) && T->pendStream == m->stream) T->pendStream = nullptr;
  }
  queue_free(m->q);
  if (m->pHost) (void)hipHostFree(m->pHost);
  if (m->stream) (void)hipStreamDestroy(m->stream);
  delete m;
}

int ct_model_add(ct_model* m, ct_table* T, const int32_t* scope, int32_t* index) {
  if (!m || !scope) return fail(CT_E_INVALID, "bad arguments");
  int rc = check_poison(T);
  if (rc) return rc;
  std::vector<int32_t> sc(scope, scope + T->n);
  std::set<int32_t> seen;
  for (int k = 0; k < T->n; ++k) {
    const int v = sc[k];
    if (v < 0 || v >= m->nPool) return fail(CT_E_INVALID, "scope[%d] = %d out of range", k, v);
    if (!seen.insert(v).second) return fail(CT_E_INVALID, "variable %d twice in a scope", v);
    if (m->lo[v] != T->lo[k] || m->dsz[v] != T->dsz[k])
      return fail(CT_E_INVALID, "column %d does not match pool variable %d", k, v);
  }
  for (ct_table* u : m->tabs)
    if (u == T) return fail(CT_E_INVALID, "table already in the model");
  if (index) *index = (int32_t)m->tabs.size();
  m->tabs.push_back(T);
  m->scopes.push_back(sc);
  model_free_device(m);
  return CT_OK;
}

int ct_model_layout(const ct_model* m, int32_t* pool_off, int32_t* pool_words) {
  if (!m) return fail(CT_E_INVALID, "null model");
  if (pool_off) memcpy(pool_off, m->poolOff.data(), sizeof(int32_t) * m->nPool);
  if (pool_words) *pool_words = m->poolWords;
  return CT_OK;
}

int ct_model_set_schedule(ct_model* m, int32_t solo_max_granules, int32_t rounds_per_graph) {
  if (!m || solo_max_granules < 0 || rounds_per_graph < 1 || rounds_per_graph > 256)
    return fail(CT_E_INVALID, "bad schedule");
  m->soloMax = solo_max_granules;
  return CT_OK;
}

int ct_model_fixpoint(ct_model* m, const uint64_t* pool_in, uint64_t* pool_out, void* stream_v,
                      int64_t* n_props, int64_t* n_rounds) {
  if (!m || !pool_in || !pool_out) return fail(CT_E_INVALID, "bad arguments");
  hipStream_t user = (hipStream_t)stream_v;
  if (user) HIPCHK(hipStreamSynchronize(user));
  int rc = model_sync_tables(m);
  if (rc) return rc;
  if (!m->built && (rc = model_build(m))) return rc;
  ModelRound M{};
  M.poolOut = pool_out;
  M.state = m->state;
  M.poolWords = m->poolWords;
  M.nHead = std::min(32, (m->poolWords + 511) / 512);
  M.call = (int32_t)++m->call;
  HIPCHK(hipHostGetDevicePointer((void**)&M.host, m->pHost, 0));
  auto set_round = [&](int r) {
    M.round = r;
    M.cur = m->pool[r % 3];
    M.next = m->pool[(r + 1) % 3];
    M.prev = m->pool[(r + 2) % 3];
  };
  set_round(0);
  HIPCHK(launch_model_start(M, pool_in, m->startOff, m->startSrc, m->stream));
  HIPCHK(launch_model_prep(m->a, m->A, M, m->stream));
  // A round's prep tells the host, as it starts, how the round before ended:
  // when that was the last one the prep copies the pool out, and nothing else
  // of its round is launched; otherwise the rest of it is queued by the time
  // the prep ends, and the next prep behind it.
  int launched = 1, code = 0;
  for (bool lost = false; !code && !lost;) {
    if (launched > 1000000) return fail(CT_E_DEVICE, "fixpoint did not converge");
    HIPCHK(launch_model_items(m->A, M, m->nU, m->nF, m->neg, m->stream));
    set_round(launched);
    HIPCHK(launch_model_prep(m->a, m->A, M, m->stream));
    const uint64_t want = (uint64_t)m->call << 32 | (uint32_t)launched++ << 8;
    bool ended = false;  // the stream was empty: then the word is there
    for (uint32_t spin = 1;; ++spin) {
      const uint64_t v = __atomic_load_n(&m->pHost[0], __ATOMIC_ACQUIRE);
      if ((v & ~(uint64_t)0xff) == want) {
        code = (int)(v & 0xff);
        break;
      }
      if ((lost = ended)) break;
      if ((spin & 0xffff) == 0) ended = hipStreamQuery(m->stream) != hipErrorNotReady;
    }
  }
  const int64_t props = (int64_t)__atomic_load_n(&m->pHost[1], __ATOMIC_ACQUIRE);
  hipError_t e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess || !code) {
    for (ct_table* T : m->tabs) T->poisoned = true;
    return fail(CT_E_DEVICE, "model round failed: %s", hipGetErrorString(e));
  }
  if (*(volatile int32_t*)m->q.hostErr) {
    for (ct_table* T : m->tabs) T->poisoned = true;
    return fail(CT_E_DEVICE, "device-side error %d in a model round", *m->q.hostErr);
  }
  // the push / pop batches queued on the model's stream before these rounds
  // have ended with them
  for (ct_table* T : m->tabs)
    if (T->pendStream == m->stream) T->pendStream = nullptr;
  if ((rc = ct_batch_status(m->stream))) {
    for (ct_table* T : m->tabs) T->poisoned = true;
    return rc;
  }
  for (ct_table* T : m->tabs) T->slots[0].failed = 2;
  if (n_props) *n_props = props;
  if (n_rounds) *n_rounds = launched - 1;
  if (code == 2)
    return fail(CT_E_STATE, "a table of the model is in the failed state (pop it first)");
  if (code == 1) return CT_FAIL;
  return CT_OK;
}

int ct_model_push(ct_model* m) {
  if (!m) return fail(CT_E_INVALID, "null model");
  return model_push_pop(m, true);
}

int ct_model_pop(ct_model* m) {
  if (!m) return fail(CT_E_INVALID, "null model");
  for (ct_table* T : m->tabs)
    if (T->slots[0].depth == 0) return fail(CT_E_STATE, "pop at depth 0");
  return model_push_pop(m, false);
}

int ct_model_get_choice(const ct_model* m, int32_t table, int32_t* solo, int32_t* tile) {
  if (!m || table < 0 || table >= (int)m->tabs.size()) return fail(CT_E_INVALID, "bad table index");
  const auto ch = model_choice(m, m->tabs[table]);
  if (solo) *solo = ch.first;
  if (tile) *tile = ch.first ? 4 : (ch.second == 0 ? 2 : ch.second);
  return CT_OK;
}

}  // extern "C"

namespace {

std::string device_arch() {
  int dev = 0;
  hipDeviceProp_t prop{};
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return "unknown";
  std::string a = prop.gcnArchName;
  const size_t c = a.find(':');
  return c == std::string::npos ? a : a.substr(0, c);
}

std::string class_key(const std::string& arch, std::pair<int, int> c) {
  return arch + " g" + std::to_string(c.first) + " r" + std::to_string(c.second);
}

// The tuning cache: a JSON object, one entry per line,
//   "gfx950 g2 r3": [solo, tile],
// keyed by architecture, granule bucket and rows bucket.
std::map<std::string, std::pair<int, int>> cache_read(const char* path) {
  std::map<std::string, std::pair<int, int>> out;
  FILE* f = path ? fopen(path, "r") : nullptr;
  if (!f) return out;
  char line[256], key[128];
  int solo = 0, tile = 0;
  while (fgets(line, sizeof(line), f))
    if (sscanf(line, " \"%127[^\"]\": [%d, %d]", key, &solo, &tile) == 3) out[key] = {solo, tile};
  fclose(f);
  return out;
}

bool cache_write(const char* path, const std::map<std::string, std::pair<int, int>>& entries) {
  const std::string tmp = std::string(path) + ".tmp";
  FILE* f = fopen(tmp.c_str(), "w");
  if (!f) return false;
  fprintf(f, "{\n");
  size_t k = 0;
  for (const auto& e : entries)
    fprintf(f, "\"%s\": [%d, %d]%s\n", e.first.c_str(), e.second.first, e.second.second,
            ++k < entries.size() ? "," : "");
  fprintf(f, "}\n");
  fclose(f);
  return rename(tmp.c_str(), path) == 0;
}

}  // namespace

extern "C" {

int ct_model_autotune(ct_model* m, const uint64_t* pool_in, const char* cache_path, int32_t* from_cache,
                      int32_t* timed) {
  if (!m || !pool_in) return fail(CT_E_INVALID, "bad arguments");
  if (from_cache) *from_cache = 0;
  if (timed) *timed = 0;
  // classes present, the largest total granule count first
  std::map<std::pair<int, int>, int64_t> work;
  for (ct_table* T : m->tabs) work[table_class(T)] += T->nGran;
  std::vector<std::pair<int64_t, std::pair<int, int>>> order;
  for (const auto& w : work) order.push_back({-w.second, w.first});
  std::sort(order.begin(), order.end());
  const std::string arch = device_arch();
  auto cache = cache_read(cache_path);
  bool all = !order.empty();
  for (const auto& o : order) all = all && cache.count(class_key(arch, o.second));
  if (cache_path && all) {
    for (const auto& o : order) m->choice[o.second] = cache[class_key(arch, o.second)];
    if (from_cache) *from_cache = 1;
    return CT_OK;
  }
  uint64_t* scratch = nullptr;
  ALLOCCHK(hipMalloc(&scratch, sizeof(uint64_t) * m->poolWords));
  std::vector<uint64_t> ref(m->poolWords), got(m->poolWords);
  int refSt = -100, rc = CT_OK, nTimed = 0;
  // one candidate: 3 fixpoints from pool_in, each between a push and a pop;
  // every candidate must reach the same fixpoint
  auto measure = [&]() -> int {
    for (int rep = 0; rep < 3; ++rep) {
      int r;
      if ((r = ct_model_push(m))) return r;
      const int st = ct_model_fixpoint(m, pool_in, scratch, nullptr, nullptr, nullptr);
      if (st != CT_OK && st != CT_FAIL) return st;
      if (st == CT_OK && hipMemcpy(got.data(), scratch, sizeof(uint64_t) * m->poolWords,
                                   hipMemcpyDeviceToHost) != hipSuccess)
        return fail(CT_E_DEVICE, "copy failed");
      if (refSt == -100) {
        refSt = st;
        ref = got;
      } else if (st != refSt || (st == CT_OK && got != ref)) {
        return fail(CT_E_DEVICE, "schedules disagree on the fixpoint");
      }
      if ((r = ct_model_pop(m))) return r;
    }
    ++nTimed;
    return CT_OK;
  };
  // both choices of every class: they run the same launches, so a class takes
  // the threshold's, whatever the clock says
  const std::pair<int, int> opts[] = {{1, 0}, {0, 2}};
  for (const auto& o : order) {
    const auto cls = o.second;
    bool solo = true;
    for (ct_table* T : m->tabs) solo = solo && (table_class(T) != cls || T->nGran <= m->soloMax);
    for (const auto& opt : opts) {
      m->choice[cls] = opt;
      if ((rc = measure())) break;
    }
    if (rc) break;
    m->choice[cls] = cache[class_key(arch, cls)] = opts[solo ? 0 : 1];
  }
  (void)hipFree(scratch);
  if (timed) *timed = nTimed;
  if (rc) return rc;
  if (cache_path && !cache_write(cache_path, cache))
    return fail(CT_E_INVALID, "cannot write the tuning cache %s", cache_path);
  return CT_OK;
}

}  // extern "C"
