// ct_nodes.hip -- search-node schedule: batches of jobs that all propagate one
// table from its root state (include/ct.h, CT_SCHED_NODES).
//
// The nodes of a batch share the table, so updateTable (Alg. 2) is turned
// round: instead of OR-ing, per node, the support rows of its removed or kept
// values (one bit per row, tuple and node), the batch is evaluated per
// *tuple*, 64 nodes to a word.  For every support row (x_i, a) one bit vector
// over the nodes says which of them keep a in dom(x_i); a tuple is valid in
// exactly the nodes of the AND of its n values' vectors (Sec. 2's definition
// of a valid tuple), so a (tuple, node) pair costs n bits read whatever the
// nodes removed, where the row form costs the removed values' rows (about 33
// bits at 6 variables of 20 values with 0-60 % removed).  The resulting
// (tuples x nodes) bit blocks are transposed in registers into the nodes'
// currTable words.
//
//   nodes_ids     (once per table)  row numbers of every tuple's values
//   nodes_prep    Alg. 1's checks and counts per node; the row vectors
//   nodes_update  the AND per tuple, the transpose, currTable writes
//   nodes_finish  partition, FAIL (Alg. 1), filterDomains (Alg. 3), status
//
// The launch boundaries order the steps; nothing waits inside a launch.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ct_device.h"

namespace ctk {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int NBLOCK = 256;
constexpr int NWAVES = NBLOCK / WAVE;

// update kernel: a wave takes a word of 64 nodes
constexpr int UBLOCK = 512;
constexpr int L = UBLOCK / WAVE;   // words of 64 nodes per group
constexpr int STEPS = 2;           // tiles (half granules) per granule

__device__ __forceinline__ int n_lane() { return threadIdx.x & (WAVE - 1); }
__device__ __forceinline__ int n_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE); }

// LDS accesses of one wave complete in issue order; only the compiler has to
// be kept from moving them.
__device__ __forceinline__ void n_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void n_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// Row numbers of the tuples' values, from the support bitsets.  One workgroup
// per granule (64 words, 4,096 tuples); support rows are staged in LDS 64 at a
// time (coalesced 512-byte loads), and a wave looks for its words' tuples in
// them, one tuple per lane.  A value outside its initial domain is in no row:
// its tuple takes the all-zero vector.  A star cell of a short table is in
// every row of its column: it takes the vector "the column is not empty".
// ids: a tile is 64 runs of 32 tuples (half a granule), and the update's lane
// is a run; per tile, variable (n2 of them: n rounded up to even with the
// all-one vector) and eighth tuple, the 64 runs' 16-byte groups of 8 numbers
// follow each other.  A number is stored as an LDS byte offset (row x 8).
// ---------------------------------------------------------------------------
constexpr int IDS_ROWS = 64;

__device__ __forceinline__ int64_t ids_at(int64_t tup, int n2, int i) {
  const int64_t tile = tup >> 11;
  const int run = (int)(tup >> 5) & 63, t = (int)tup & 31;
  return (((tile * n2 + i) * 4 + (t >> 3)) * 64 + run) * 8 + (t & 7);
}

__global__ void __launch_bounds__(1024) nodes_ids_kernel(const TabDesc* Tp, uint16_t* idsOut) {
  __shared__ uint64_t rowsL[IDS_ROWS][GW];
  const CT_G TabDesc* T = (const CT_G TabDesc*)Tp;
  CT_G uint16_t* ids = (CT_G uint16_t*)idsOut;
  const int n = T->n, n2 = (n + 1) & ~1;
  const uint16_t zero = (uint16_t)(8 * T->rows), one = (uint16_t)(8 * (T->rows + 1));
  const int64_t stride = T->stride;
  const int64_t w0 = (int64_t)blockIdx.x * GW;
  const int lane = n_lane(), wv = n_wave();
  for (int i = 0; i < n2; ++i) {
    if (i >= n) {
      for (int k = wv; k < GW; k += 16) {
        const int64_t tup = (w0 + k) * 64 + lane;
        ids[ids_at(tup, n2, i)] = one;
      }
      continue;
    }
    const VarDesc v = T->vars[i];
    int cnt[4] = {0, 0, 0, 0};
    uint16_t id[4] = {zero, zero, zero, zero};
    for (int r0 = 0; r0 < v.dsize; r0 += IDS_ROWS) {
      const int nr = min(IDS_ROWS, v.dsize - r0);
      __syncthreads();
      for (int x = threadIdx.x; x < nr * GW; x += 1024)
        rowsL[x / GW][x % GW] = T->S[(int64_t)(v.rowStart + r0 + x / GW) * stride + w0 + x % GW];
      __syncthreads();
      for (int r = 0; r < nr; ++r) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if ((rowsL[r][wv + 16 * k] >> lane) & 1ull) {
            id[k] = (uint16_t)(8 * (v.rowStart + r0 + r));
            ++cnt[k];
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t tup = (w0 + wv + 16 * k) * 64 + lane;
      ids[ids_at(tup, n2, i)] = cnt[k] > 1 ? (uint16_t)(8 * (T->rows + 2 + i)) : id[k];
    }
  }
}

// ---------------------------------------------------------------------------
// Prep.  The first workgroups take one node per wave: Alg. 1's checks and the
// row count of the node (|Delta| or |dom| per changed variable, on the branch
// Alg. 2 would take: the work counters).  The others take one (word of 64
// nodes, domain word) per wave, a node per lane: bit b's vector is the ballot
// of bit b over the lanes.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(NBLOCK) nodes_prep_kernel(NodesDesc N) {
  __shared__ int32_t shSize[NWAVES][MAX_ARITY];
  __shared__ int32_t shDcnt[NWAVES][MAX_ARITY];
  const int wv = n_wave(), lane = n_lane();
  const CT_G TabDesc* T = N.tab;
  const int n = T->n, D = T->D;
  const int infoBlocks = (N.nJobs + NWAVES - 1) / NWAVES;
  if ((int)blockIdx.x >= infoBlocks) {
    // vectors: lane = node
    const int x = ((int)blockIdx.x - infoBlocks) * NWAVES + wv;
    const int nw = x / (D + 1), q = x % (D + 1);
    if (nw >= N.groups * L) return;
    CT_G uint64_t* out = N.vec + (int64_t)(nw / L) * N.vecRows * L + nw % L;  // row r at r * L
    const int node = nw * 64 + lane;
    const bool in = node < N.nJobs;
    if (q == D) {
      if (lane < 2) out[(int64_t)(T->rows + lane) * L] = lane ? ~0ull : 0ull;
      if (!in) N.ct[node] = N.out[node] = 0ull;  // the lists' padding to whole groups
      return;
    }
    const CT_G uint64_t* dom = N.jobs[in ? node : 0].dom_in;
    const WordDesc wd = T->words[q];
    const uint64_t din = in ? dom[q] : 0ull;
    const int k = q - wd.v.domOff;
    const int used = min(64, wd.v.dsize - 64 * k);
    uint64_t mine = 0;
    for (int b = 0; b < used; ++b) {
      const uint64_t m = __ballot((din >> b) & 1ull);
      if (lane == b) mine = m;
    }
    if (lane < used) out[(int64_t)(wd.v.rowStart + 64 * k + lane) * L] = mine;
    if (k == 0 && N.vecRows > T->rows + 2) {  // short table: the column is not empty
      uint64_t any = din;
      for (int j = 1; j < wd.v.domWords; ++j) any |= in ? dom[q + j] : 0ull;
      const uint64_t m = __ballot(any != 0ull);
      if (lane == 0) out[(int64_t)(T->rows + 2 + wd.var) * L] = m;
    }
    return;
  }
  const int j = (int)blockIdx.x * NWAVES + wv;
  if (j >= N.nJobs) return;  // no workgroup barrier below
  const DevJob J = N.jobs[j];
  int32_t* size = shSize[wv];
  int32_t* dcnt = shDcnt[wv];
  for (int i = lane; i < n; i += WAVE) {
    size[i] = 0;
    dcnt[i] = 0;
  }
  n_wave_sync();
  bool stray = false, notSub = false;
  for (int q = lane; q < D; q += WAVE) {
    const uint64_t din = J.dom_in[q];
    const uint64_t ld = T->dom0[q];
    const WordDesc wd = T->words[q];
    const int used = wd.v.dsize - 64 * (q - wd.v.domOff);
    if (used < 64 && (din >> used) != 0) stray = true;
    if (din & ~ld) notSub = true;
    atomicAdd(&size[wd.var], __popcll(din));
    atomicAdd(&dcnt[wd.var], __popcll(ld & ~din));
  }
  const int st = T->rootFailed ? ST_STATE
                 : __ballot(stray) ? ST_INVALID
                 : __ballot(notSub) ? ST_NOT_SUBSET : ST_OK;
  n_wave_sync();
  const int policy = T->policy;
  int rows = 0;
  for (int i = lane; i < n; i += WAVE) {
    const int sz = size[i], dc = dcnt[i];
    if (dc == 0) continue;  // |dom| is the root's: not in s_val
    const bool inc = policy == 2 ? true : policy == 1 ? false : dc < sz;
    rows += inc ? dc : sz;
  }
  for (int o = 1; o < WAVE; o <<= 1) rows += __shfl_xor(rows, o);
  if (lane == 0) {
    const CT_G SlotDesc* s = J.slot;
    NodeInfo I;
    I.status = st;
    I.nrows = st == ST_OK ? rows : 0;
    I.ct = s->ct;
    I.res = s->res;
    I.idx = s->idx[0];
    I.lastDom = s->lastDom;
    I.dom_in = J.dom_in;
    I.dom_out = J.dom_out;
    N.info[j] = I;
    N.ct[j] = st == ST_OK ? (uint64_t)s->ct : 0ull;
    N.out[j] = st == ST_OK ? (uint64_t)J.ct_out : 0ull;
  }
}

// ---------------------------------------------------------------------------
// updateTable of all nodes.  A group is 512 nodes, one word of 64 per wave;
// its row vectors stay in LDS (word-major).  An item is a granule or half of
// one; persistent workgroups walk a contiguous range of the items.  Per step
// (half a granule, 2,048 tuples) a wave's lane takes a run of 32 tuples: it
// ANDs, per tuple, its word of the vectors of the tuple's n values (two
// variables at a time: one three-input AND per half word), which leaves a
// 32 x 64 bit block of tuples x nodes in 64 registers.  Two 32 x 32 transposes
// turn it into a dword of each of the 64 nodes' currTable, and the lanes'
// dwords of a node are 256 contiguous bytes: one store per node, with no pass
// through LDS.  The stores bypass the caches (non-temporal): a batch writes
// every node's whole currTable once, far more than the L2s hold.
// Lanes read different rows of one word column: the rows of a variable of up
// to 32 values lie in different LDS banks.
// Bound: the currTable writes.  4,096 nodes x 1,000,000 tuples x 6 variables
// of 20 values: 118-125 us for 514 MB; the same 256-byte store pattern alone
// takes 110 us, the AND and transpose work without stores 90 us (VALU, about
// 1,090 operations per 32 tuples and 64 words).  The row form it replaces (the
// removed values' support rows from LDS, per node) took 300 us at 70 % of the
// LDS rate.  500 nodes x 300,000 tuples x 8 variables of 8-128 values, with
// currTable copies: 21 us; one workgroup per node (rows from the L2s and the
// MALL) took 250 us.  Passing the dwords through LDS for longer stores (64 to
// 512 bytes per node, groups of 4,096 to 512 nodes): 137-240 us.
// ---------------------------------------------------------------------------
// Rows k and k + H of a 32 x 32 bit block exchange their off-diagonal H-bit
// squares, for every pair of rows whose numbers differ in bit H.
template <int H>
__device__ __forceinline__ void swap_squares(uint32_t (&x)[32]) {
  constexpr uint32_t m = H == 4 ? 0x0f0f0f0fu : H == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int k = (p / H) * 2 * H + p % H;
    const uint32_t lo = x[k], hi = x[k + H];
    if (H == 16) {
      x[k] = __builtin_amdgcn_perm(hi, lo, 0x05040100);
      x[k + H] = __builtin_amdgcn_perm(hi, lo, 0x07060302);
    } else if (H == 8) {
      x[k] = __builtin_amdgcn_perm(hi, lo, 0x06020400);
      x[k + H] = __builtin_amdgcn_perm(hi, lo, 0x07030501);
    } else {
      x[k] = (lo & m) | ((hi << H) & ~m);
      x[k + H] = ((lo >> H) & m) | (hi & ~m);
    }
  }
}

// x[b] bit t <- x[t] bit b
__device__ __forceinline__ void transpose32(uint32_t (&x)[32]) {
  swap_squares<16>(x);
  swap_squares<8>(x);
  swap_squares<4>(x);
  swap_squares<2>(x);
  swap_squares<1>(x);
}

// Tuples 8 C .. 8 C + 7 of the thread's run: AND of the vectors of their
// values of two variables; A, B hold the 8 tuples' LDS byte offsets.
template <int C>
__device__ __forceinline__ void and_rows(const char* vec, const u32x4 A, const u32x4 B, uint32_t (&lo)[32],
                                         uint32_t (&hi)[32]) {
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const uint32_t oa = (t & 1) ? A[t / 2] >> 16 : A[t / 2] & 0xFFFFu;
    const uint32_t ob = (t & 1) ? B[t / 2] >> 16 : B[t / 2] & 0xFFFFu;
    const u32x2 a = *(const u32x2*)(vec + oa), b = *(const u32x2*)(vec + ob);
    lo[8 * C + t] = __builtin_amdgcn_bitop3_b32(lo[8 * C + t], a.x, b.x, 0x80);  // AND
    hi[8 * C + t] = __builtin_amdgcn_bitop3_b32(hi[8 * C + t], a.y, b.y, 0x80);
  }
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) v |= __shfl_xor(v, o);
  return v;
}

// Dword `lane` of a tile of every node's currTable: x[b] belongs to node b of
// ct / out, the nodes' addresses (the same for every lane, written by the
// launch before: scalar loads, 8 at a time).
typedef uint64_t u64x8 __attribute__((ext_vector_type(8)));
typedef const __attribute__((address_space(4))) u64x8* AddrList;

template <bool COPY>
__device__ __forceinline__ void put_nodes(const uint32_t (&x)[32], AddrList ct, AddrList out, uint32_t off,
                                          bool inOut) {
#pragma unroll
  for (int b8 = 0; b8 < 4; ++b8) {
    const u64x8 c = ct[b8];
#pragma unroll
    for (int b = 0; b < 8; ++b)
      if (c[b]) __builtin_nontemporal_store(x[8 * b8 + b], (CT_G uint32_t*)((CT_G char*)c[b] + off));
    if (COPY) {
      const u64x8 o = out[b8];
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (o[b] && inOut) *(CT_G uint32_t*)((CT_G char*)o[b] + off) = x[8 * b8 + b];
    }
  }
}

template <bool COPY>  // some job wants a currTable copy
__global__ void __launch_bounds__(UBLOCK, 4) nodes_update_kernel(NodesDesc N) {
  extern __shared__ uint64_t lds[];
  const int VS = N.vecRows | 1;  // words between a row's words
  const int tid = threadIdx.x, lane = n_lane(), l = n_wave();
  const int steps = STEPS / N.parts;          // per item
  const int itemsG = N.nGran * N.parts;       // per group
  const int items = itemsG * N.groups;
  const int i1 = (int)((int64_t)items * (blockIdx.x + 1) / gridDim.x);
  const char* vecL = (const char*)(lds + l * VS);
  int curGroup = -1;
  for (int it = (int)((int64_t)items * blockIdx.x / gridDim.x); it < i1; ++it) {
    const int grp = it / itemsG;
    const int x = it % itemsG;
    const int g = x / N.parts, part = x % N.parts;
    if (grp != curGroup) {
      curGroup = grp;
      __syncthreads();
      const CT_G uint64_t* src = N.vec + (int64_t)grp * N.vecRows * L;
      for (int k = tid; k < N.vecRows * L; k += UBLOCK) lds[(k % L) * VS + k / L] = src[k];
      __syncthreads();
    }
    uint32_t nz0 = 0, nz1 = 0;
    for (int st = 0; st < steps; ++st) {
      const int tile = g * STEPS + part * steps + st;
      const CT_G u32x4* ids = (const CT_G u32x4*)N.ids + (int64_t)tile * N.n2 * 256 + lane;
      uint32_t lo[32], hi[32];
#pragma unroll
      for (int t = 0; t < 32; ++t) lo[t] = hi[t] = ~0u;
      u32x4 A0 = ids[0], B0 = ids[256];
      for (int i = 0; i < N.n2; i += 2) {
        const u32x4 A1 = ids[64], A2 = ids[128], A3 = ids[192];
        const u32x4 B1 = ids[320], B2 = ids[384], B3 = ids[448];
        and_rows<0>(vecL, A0, B0, lo, hi);
        and_rows<1>(vecL, A1, B1, lo, hi);
        and_rows<2>(vecL, A2, B2, lo, hi);
        // the next pair's first row numbers are on their way meanwhile (the
        // last pair reads its own again)
        if (i + 2 < N.n2) ids += 512;
        A0 = ids[0];
        B0 = ids[256];
        asm volatile("" ::: "memory");
        and_rows<3>(vecL, A3, B3, lo, hi);
      }
#pragma unroll
      for (int t = 0; t < 32; ++t) {
        nz0 |= lo[t];
        nz1 |= hi[t];
      }
      transpose32(lo);
      transpose32(hi);
      const uint32_t off = (uint32_t)tile * 256u + (uint32_t)lane * 4u;  // bytes; a currTable has at most 4 MiB
      const bool inOut = COPY && (int64_t)off < 8 * N.W;
      const int w8 = (grp * L + l) * 8;  // the wave's 64 nodes, in lists of 8
      const AddrList ct = (AddrList)N.ct + w8, out = (AddrList)N.out + w8;
      put_nodes<COPY>(lo, ct, out, off, inOut);
      put_nodes<COPY>(hi, ct + 4, out + 4, off, inOut);
    }
    nz0 = wave_or(nz0);
    nz1 = wave_or(nz1);
    if (lane == 0)
      N.nz[((int64_t)part * N.groups * L + grp * L + l) * N.nGran + g] = ((uint64_t)nz1 << 32) | nz0;
  }
}

// ---------------------------------------------------------------------------
// Finish.  A wave takes one task of a node: task 0 the stable partition of
// the root's granule list by the non-zero bits (survivors first), FAIL and
// the slot's state; task k > 0 filterDomains over FIN_W of its domain words.
// Every task reads the node's non-zero bits itself (the filter's scans take
// the active granules from them, not from the partition's list), so tasks
// do not wait for each other.
// Bound: the latency of a task's chain (record -> residues -> support words
// and currTable words -> rare walks), hidden by the waves in flight.
// ---------------------------------------------------------------------------
constexpr int FIN_W = 4;      // domain words per filter task
constexpr int FIN_WALK = 8;   // words a missing value checks after its residue, per round trip
constexpr int FIN_WALKS = 2;

__device__ __forceinline__ uint64_t node_nz(const NodesDesc& N, int node, int g) {
  const int nw = node / 64;
  uint64_t m = 0;
  for (int p = 0; p < N.parts; ++p)
    m |= N.nz[((int64_t)p * N.groups * L + nw) * N.nGran + min(g, N.nGran - 1)];
  return g < N.nGran ? (m >> (node % 64)) & 1ull : 0ull;
}

__device__ void finish_partition(const NodesDesc& N, int j, const CT_G NodeInfo* info, int st0) {
  const int lane = n_lane();
  const CT_G TabDesc* T = N.tab;
  const DevJob J = N.jobs[j];
  CT_G SlotDesc* s = J.slot;
  int st = st0;
  if (st0 == ST_OK) {
    const int limit0 = T->limit0, nGran = T->nGran;
    const CT_G int32_t* src = T->idx0;
    CT_G int32_t* dst = info->idx;
    const uint64_t below = (1ull << lane) - 1ull;
    int nSurv = 0;
    for (int g0 = 0; g0 < nGran; g0 += WAVE) nSurv += __popcll(__ballot(node_nz(N, j, g0 + lane)));
    int sv = 0, zr = nSurv;
    for (int p0 = 0; p0 < limit0; p0 += 4 * WAVE) {
      int gid[4];
      bool f[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int p = p0 + u * WAVE + lane;
        gid[u] = p < limit0 ? src[p] : -1;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) f[u] = gid[u] >= 0 && node_nz(N, j, gid[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t bs = __ballot(f[u]), bz = __ballot(gid[u] >= 0 && !f[u]);
        if (f[u]) dst[sv + __popcll(bs & below)] = gid[u];
        else if (gid[u] >= 0) dst[zr + __popcll(bz & below)] = gid[u];
        sv += __popcll(bs);
        zr += __popcll(bz);
      }
    }
    for (int p = limit0 + lane; p < nGran; p += WAVE) dst[p] = src[p];
    if (!nSurv) st = ST_FAIL;
    if (lane == 0) {
      const unsigned long long nrows = (unsigned long long)info->nrows;
      s->cur = 0;
      s->limit = nSurv;
      s->depth = 0;
      s->trailTop = 0;
      s->serial = J.serialBase;
      s->failed = nSurv ? 0 : 1;
      atomicAdd(&s->stats[S_JOBS], 1ull);
      atomicAdd(&s->stats[S_GRAN_IN], (unsigned long long)limit0);
      atomicAdd(&s->stats[S_ROWS], nrows);
      if (nrows) atomicAdd(&s->stats[S_GRAN_ROWS], (unsigned long long)limit0 * nrows);
    }
  } else {
    // a rejected node's slot still becomes the table's root state (a rare
    // path: the whole currTable is copied)
    for (int64_t w = lane; w < T->stride; w += WAVE) s->ct[w] = T->ct0[w];
    for (int p = lane; p < T->nGran; p += WAVE) s->idx[0][p] = T->idx0[p];
    for (int q = lane; q < T->D; q += WAVE) s->lastDom[q] = T->dom0[q];
    if (lane == 0) {
      s->cur = 0;
      s->limit = T->limit0;
      s->failed = T->rootFailed;
      s->depth = 0;
      s->trailTop = 0;
      s->serial = J.serialBase;
    }
  }
  if (lane == 0) {
    s->status = st;
    s->noop = 0;
    if (J.status_out) *J.status_out = st;  // read after the launch: no fence
  }
}

__global__ void __launch_bounds__(NBLOCK) nodes_finish_kernel(NodesDesc N) {
  const int fTasks = (N.D + FIN_W - 1) / FIN_W;
  const int x = (int)blockIdx.x * NWAVES + n_wave();
  const int j = x / (1 + fTasks), task = x % (1 + fTasks);
  if (j >= N.nJobs) return;
  const CT_G NodeInfo* info = N.info + j;
  const int st0 = info->status;
  if (task == 0) {
    finish_partition(N, j, info, st0);
    return;
  }
  if (st0 != ST_OK) return;
  const int lane = n_lane();
  const CT_G TabDesc* T = N.tab;
  const int D = N.D, nGran = N.nGran;
  const int64_t stride = N.stride;
  const CT_G uint64_t* din = info->dom_in;
  const CT_G uint64_t* S = N.S;
  const CT_G uint64_t* ct = info->ct;
  CT_G int32_t* res = info->res;
  const int q0 = (task - 1) * FIN_W;
  // the task's words, each value's residue and support word (addresses are
  // clamped into the table)
  uint64_t dw[FIN_W], sw[FIN_W], cw[FIN_W];
  int row[FIN_W], rw[FIN_W], size[FIN_W];
  WordDesc wd[FIN_W];
#pragma unroll
  for (int u = 0; u < FIN_W; ++u) {
    const int q = min(q0 + u, D - 1);
    wd[u] = T->words[q];
    dw[u] = din[q];
  }
#pragma unroll
  for (int u = 0; u < FIN_W; ++u) {
    const int q = min(q0 + u, D - 1);
    size[u] = __popcll(dw[u]);
    if (wd[u].v.domWords > 1) {
      size[u] = 0;
      for (int k = 0; k < wd[u].v.domWords; ++k) size[u] += __popcll(din[wd[u].v.domOff + k]);
    }
    const int base = wd[u].v.rowStart + (q - wd[u].v.domOff) * 64;
    row[u] = ((dw[u] >> lane) & 1ull) ? base + lane : base;  // (validated: no stray bits)
    rw[u] = min(max(res[row[u]], 0), (int)stride - 1);
  }
#pragma unroll
  for (int u = 0; u < FIN_W; ++u) {
    sw[u] = S[(int64_t)row[u] * stride + rw[u]];
    cw[u] = ct[rw[u]];
  }
  // FAIL leaves the domains alone
  bool live = false;
  for (int g0 = 0; g0 < nGran && !live; g0 += WAVE) live = __ballot(node_nz(N, j, g0 + lane)) != 0ull;
  if (!live) return;
  unsigned long long nChk = 0, nMiss = 0, nScan = 0;
  uint64_t miss[FIN_W];
#pragma unroll
  for (int u = 0; u < FIN_W; ++u) {
    const bool on = q0 + u < D && size[u] > 1;  // s_sup: variables with two or more values
    const bool present = on && ((dw[u] >> lane) & 1ull);
    miss[u] = __ballot(present && (cw[u] & sw[u]) == 0ull);
    nChk += __popcll(__ballot(present));
    nMiss += __popcll(miss[u]);
  }
  const int words = nGran * GW;
  for (int u = 0; u < FIN_W; ++u) {
    const int q = q0 + u;
    if (q >= D) break;
    uint64_t todo = miss[u];
    if (todo) {
      // every missing lane first walks the words after its old residue
      // (wrapping at the end of the table)
      const bool mine = (todo >> lane) & 1ull;
      const CT_G uint64_t* R = S + (int64_t)row[u] * stride;
      int found = -1;
      for (int k = 0; k < FIN_WALKS; ++k) {
        uint64_t y[FIN_WALK];
#pragma unroll
        for (int t = 0; t < FIN_WALK; ++t) {
          int w = rw[u] + 1 + k * FIN_WALK + t;
          if (w >= words) w -= words;
          y[t] = R[w] & ct[w];
        }
#pragma unroll
        for (int t = 0; t < FIN_WALK; ++t) {
          int w = rw[u] + 1 + k * FIN_WALK + t;
          if (w >= words) w -= words;
          if (mine && found < 0 && y[t]) found = w;
        }
        if (!__ballot(mine && found < 0)) break;
      }
      nScan += __popcll(todo);
      if (found >= 0) res[row[u]] = found;
      todo = __ballot(mine && found < 0);
      // the rest scan the active granules together, two values by two
      // granules per round trip, until each finds a support
      for (int g0 = 0; g0 < nGran && todo; g0 += WAVE) {
        uint64_t act = __ballot(node_nz(N, j, g0 + lane));
        while (act && todo) {
          const int ga = g0 + __ffsll((unsigned long long)act) - 1;
          act &= act - 1;
          const int gb = act ? g0 + __ffsll((unsigned long long)act) - 1 : ga;
          act &= act - 1;
          const uint64_t ca = ct[(int64_t)ga * GW + lane], cb = ct[(int64_t)gb * GW + lane];
          const int base = wd[u].v.rowStart + (q - wd[u].v.domOff) * 64;
          for (uint64_t t = todo; t;) {
            const int va = __ffsll((unsigned long long)t) - 1;
            t &= t - 1;
            const int vb = t ? __ffsll((unsigned long long)t) - 1 : va;
            t &= t - 1;
            const CT_G uint64_t* Ra = S + (int64_t)(base + va) * stride + lane;
            const CT_G uint64_t* Rb = S + (int64_t)(base + vb) * stride + lane;
            const uint64_t x0 = Ra[(int64_t)ga * GW] & ca, x1 = Ra[(int64_t)gb * GW] & cb;
            const uint64_t y0 = Rb[(int64_t)ga * GW] & ca, y1 = Rb[(int64_t)gb * GW] & cb;
            const uint64_t m0 = __ballot(x0 != 0ull), m1 = __ballot(x1 != 0ull);
            const uint64_t n0 = __ballot(y0 != 0ull), n1 = __ballot(y1 != 0ull);
            nScan += 4;
            if (m0 | m1) {
              todo &= ~(1ull << va);
              if (lane == 0)
                res[base + va] = m0 ? ga * GW + __ffsll((unsigned long long)m0) - 1
                                    : gb * GW + __ffsll((unsigned long long)m1) - 1;
            }
            if (n0 | n1) {
              todo &= ~(1ull << vb);
              if (lane == 0)
                res[base + vb] = n0 ? ga * GW + __ffsll((unsigned long long)n0) - 1
                                    : gb * GW + __ffsll((unsigned long long)n1) - 1;
            }
          }
        }
      }
    }
    if (lane == 0) {
      const uint64_t dout = dw[u] & ~todo;
      info->dom_out[q] = dout;
      info->lastDom[q] = dout;
    }
  }
  if (lane == 0 && nChk) {
    CT_G SlotDesc* s = N.jobs[j].slot;
    atomicAdd(&s->stats[S_RES_CHECK], nChk);
    if (nMiss) atomicAdd(&s->stats[S_RES_MISS], nMiss);
    if (nScan) atomicAdd(&s->stats[S_SCAN], nScan);
  }
}

size_t update_lds(int vecRows) {
  return sizeof(uint64_t) * (size_t)(vecRows | 1) * L;
}

int device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 256;
  return cus;
}

}  // namespace

// Largest row-vector count whose group fits a workgroup's LDS (and whose LDS
// byte offsets fit 16 bits).
int nodes_max_vec_rows(size_t lds) {
  const size_t most = lds / (L * sizeof(uint64_t));
  return most > 1 ? (int)std::min<size_t>(most - 1, 8191) : 0;
}

static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Bytes of a batch's records, row vectors and non-zero words.
size_t nodes_scratch_bytes(int vecRows, int nJobs, int nGran) {
  const size_t groups = (size_t)((nJobs + 64 * L - 1) / (64 * L));
  return up256(sizeof(NodeInfo) * (size_t)nJobs) + 2 * up256(sizeof(uint64_t) * groups * 64 * L) + up256(sizeof(uint64_t) * groups * vecRows * L) +
         up256(sizeof(uint64_t) * STEPS * groups * L * nGran);
}

size_t nodes_ids_bytes(int n, int64_t stride) { return (size_t)stride * 64 * ((n + 1) & ~1) * sizeof(uint16_t); }

hipError_t launch_nodes_ids(const TabDesc* T, int nGran, uint16_t* ids, hipStream_t stream) {
  hipLaunchKernelGGL(nodes_ids_kernel, dim3(nGran), dim3(1024), 0, stream, T, ids);
  return hipGetLastError();
}

// N: the table's and the batch's fields; the groups, the parts and the
// scratch's arrays are set here.
hipError_t launch_nodes(NodesDesc N, char* scratch, hipStream_t stream) {
  N.groups = (N.nJobs + 64 * L - 1) / (64 * L);
  N.info = (CT_G NodeInfo*)scratch;
  scratch += up256(sizeof(NodeInfo) * (size_t)N.nJobs);
  const size_t listB = up256(sizeof(uint64_t) * (size_t)N.groups * 64 * L);
  N.ct = (CT_G uint64_t*)scratch;
  scratch += listB;
  N.out = (CT_G uint64_t*)scratch;
  scratch += listB;
  N.vec = (CT_G uint64_t*)scratch;
  scratch += up256(sizeof(uint64_t) * (size_t)N.groups * N.vecRows * L);
  N.nz = (CT_G uint64_t*)scratch;
  const int infoBlocks = (N.nJobs + NWAVES - 1) / NWAVES;
  const int vecBlocks = (N.groups * L * (N.D + 1) + NWAVES - 1) / NWAVES;
  hipLaunchKernelGGL(nodes_prep_kernel, dim3(infoBlocks + vecBlocks), dim3(NBLOCK), 0, stream, N);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // two workgroups per CU (registers); a granule is cut in two while that
  // leaves fewer than two items to a workgroup
  const size_t lds = update_lds(N.vecRows);
  const int slots = 2 * device_cus();
  const int whole = N.nGran * N.groups;
  N.parts = whole < 2 * slots ? STEPS : 1;
  const int grid = std::min(whole * N.parts, slots);
  if (N.anyOut)
    hipLaunchKernelGGL(nodes_update_kernel<true>, dim3(grid), dim3(UBLOCK), lds, stream, N);
  else
    hipLaunchKernelGGL(nodes_update_kernel<false>, dim3(grid), dim3(UBLOCK), lds, stream, N);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t tasks = (int64_t)N.nJobs * (1 + (N.D + FIN_W - 1) / FIN_W);
  hipLaunchKernelGGL(nodes_finish_kernel, dim3((unsigned)((tasks + NWAVES - 1) / NWAVES)), dim3(NBLOCK), 0, stream, N);
  return hipGetLastError();
}

}  // namespace ctk
