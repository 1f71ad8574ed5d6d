// Batched RSST: many independent 2D boxes of uneven size, xi and
// background, advanced by one persistent kernel per run, captured in a HIP
// graph and replayed.
//
// Work items are (stage q, box b, row block p), q = 2 n + stage - 1 for
// step n.  A row block is `rows` rows (y, the marched axis) of a box: a few
// chunks of the strip rows, whose strips of x the four waves of a 256-thread
// workgroup march.  The boxes are dealt to queues; tickets of a queue are
// handed out in q-major order by one atomic counter, and an item only waits on
// items of its own box, which hold smaller tickets of the same queue:
//   * the row blocks of its box at q-1 that hold a row within two cells
//     of its own rows (through the boundary rule: a periodic y wraps the
//     first block onto the last ones), or whose rows are within two cells
//     of its own; this orders every read of a row by the previous stage
//     before the in-place stage-2 write of U, and every stage-2 read of U1
//     before the next stage-1 write of it;
//   * for stage 1 of step n > 0, every stage-2 block of step n-1 of its
//     box, whose per-box maximum of c_tot gives the box's CFL dt.
// Every waiting item holds a ticket larger than the ones it waits for, and
// those were taken by running workgroups, so the queue cannot deadlock.
//
// Queues and XCDs.  Data written by one XCD of the MI355X is seen by another
// only after the writer's whole L2 was written back and the reader's
// invalidated.  With one queue for the chip every item did both, several
// times, and these set the pace: 512 FP32 boxes of 64..256 cells a side ran
// 20 steps in 62.8 ms with 16-row strips (4.6 Gcell-updates/s).  So there
// are eight queues, and a queue is worked on by the workgroups of one XCD
// only (the first whose workgroup comes to it; the hardware register XCC_ID
// tells a workgroup its XCD): every wait is between CUs that share an L2,
// which a store reaches before it is counted complete and which agent-scope
// loads read past the CU's own cache.  The same run then takes 14.0 ms (20.6
// Gcell-updates/s; 32-row strips 13.3 ms, against 21.7 ms for the best strips
// before), bound by FP64 issue: 0.8 of the rate at which a SIMD can issue the
// ~390 instructions of a row (rsst_stage2.h).  Where the boxes are too few or too
// uneven to keep eight queues level, one queue serves the chip, with one
// write-back per item and one invalidation per wait.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "rsst.h"
#include "rsst_stage2.h"

#pragma clang fp contract(off)

namespace rsstk {

constexpr int kBatchThreads = 256;  // four waves, each marching strips of its own rows
// Persistent workgroups per CU.  A workgroup is one wave per SIMD, so this is
// also the waves per SIMD the kernel is compiled for (its register budget).
// 512 FP32 boxes, 20 steps, 16-row strips: 14.4 ms with three, 15.8 ms with
// four (128 VGPRs, which spill).
constexpr int kBatchPerCU = 3;
constexpr int kXcds = 8;            // XCDs of an MI355X, each with its own L2
constexpr int kLdAgent = 16;        // load cache policy sc1: agent scope, past the CU's cache

struct BoxDev {
  StageArgs s1, s2;  // stage views of the box (pointers into U_all / U1_all)
  double cfl_h;      // cfl * h of the box
  int nblk;          // row blocks
  int rbase;         // index of the box's first item in a stage
  int rows;          // rows of a block
};

// A work item: row block `blk` of box `box`, and the blocks of the same
// box whose rows its stencil reads or whose stencil reads its rows (the
// order it needs against the previous stage).
constexpr int kMaxDeps = 8;
static_assert(5 + kMaxDeps == RSST_BATCH_PLAN_COLS, "plan table layout");
struct Item {
  int box, blk, ndep;
  int dep[kMaxDeps];
};

struct BatchState {
  unsigned* ticket;              // [kXcds] next ticket of each queue
  int* owner;                    // [kXcds] XCD working on each queue, -1 none yet
  unsigned long long* maxbits;   // [nbox][max_steps + 1] max c_tot of the input of each step
  unsigned* cnt2;                // [nbox][max_steps] stage-2 blocks done per step
  unsigned* done;                // [2 max_steps][nitem] item done flags
  double* tacc;                  // [nbox] time reached
  unsigned* flags;               // non-physical flags
  int nbox, nitem, nsteps, max_steps;
  int local;                     // one queue per XCD (else queue 0 serves the chip)
  int qbase[kXcds + 1];          // first item of each queue (its items are consecutive)
  unsigned long long wait_ticks; // longest dependency wait, in wall-clock ticks (100 MHz)
};

template <typename T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The XCD this wave runs on.
__device__ __forceinline__ int xcc_id() {
  return (int)(__builtin_amdgcn_s_getreg(20 /* HW_REG_XCC_ID */ | (0 << 6) | ((4 - 1) << 11)) & (kXcds - 1));
}

// Every store and atomic of the wave so far has reached its L2.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Flag bit of a run whose queue gave up on a dependency wait (reported by
// rsst_batch_poll as RSST_E_DEVICE): a wait past its deadline means a
// dependency that will not arrive, so instead of spinning for ever the item
// is skipped (marked done, nothing stored) and every workgroup drains.
constexpr unsigned kQueueTimeout = 8u;

// Clears the per-run counters (graph-safe: a kernel, not a memset node).
__global__ void __launch_bounds__(256) batch_reset_kernel(BatchState S) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long stride = (long long)gridDim.x * blockDim.x;
  if (tid < kXcds) {
    S.ticket[tid] = 0u;
    S.owner[tid] = -1;
  }
  for (long long q = tid; q < (long long)S.nbox * (S.max_steps + 1); q += stride) S.maxbits[q] = 0ull;
  for (long long q = tid; q < (long long)S.nbox * S.max_steps; q += stride) S.cnt2[q] = 0u;
  for (long long q = tid; q < 2ll * S.max_steps * S.nitem; q += stride) S.done[q] = 0u;
}

// Per-box maximum of c_tot of the initial state -> maxbits[b][0].
template <typename ST>
__global__ void __launch_bounds__(256) batch_prime_kernel(const BoxDev* __restrict__ boxes, BatchState S,
                                                         int blocks_per_box) {
  constexpr int NV = 4;
  const int b = blockIdx.x / blocks_per_box, part = blockIdx.x % blocks_per_box;
  const StageArgs& A = boxes[b].s1;
  const Consts K{A.gamma, A.gm1, A.inv_gm1, A.inv_xi, A.f};
  const ST* u = (const ST*)A.uin;
  __shared__ double red[4];
  double cm = 0.0;
  for (long long c = (long long)part * blockDim.x + threadIdx.x; c < A.ncell;
       c += (long long)blocks_per_box * blockDim.x) {
    double q[NV];
    const int y = (int)(c / A.geo.nx);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      q[v] = (double)u[v * A.ncell + c];
      if constexpr (sizeof(ST) == 4) q[v] += A.bg[v * A.nbg + (A.bg_axis == 1 ? y : 0)];
    }
    cm = fmax(cm, cell_ctot<2>(q, K));
  }
  const double wm = wave_max(cm);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = wm;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    atomicMax(S.maxbits + (long long)b * (S.max_steps + 1), (unsigned long long)__double_as_longlong(m));
  }
}

// Completion of an item, by thread 0 after every wave's stores are complete:
// its per-box c_tot maximum (stage 2), the box time, then the done flag and
// the per-step stage-2 count.
struct Pending {
  int b, p, n;
  unsigned q, r;
  bool st2;
  double dt;
};

__device__ __forceinline__ void signal_done(const BatchState& S, const Pending& d, const double* red) {
  if (d.st2) {
    double m = 0.0;
    for (int w = 0; w < kBatchThreads / 64; ++w) m = fmax(m, red[w]);
    __hip_atomic_fetch_max(S.maxbits + (long long)d.b * (S.max_steps + 1) + d.n + 1,
                           (unsigned long long)__double_as_longlong(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (d.p == 0)
      __hip_atomic_store(S.tacc + d.b, ld_agent(S.tacc + d.b) + d.dt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  wait_stores();
  if (!S.local) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __hip_atomic_store(S.done + (long long)d.q * S.nitem + d.r, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (d.st2)
    __hip_atomic_fetch_add(S.cnt2 + (long long)d.b * S.max_steps + d.n, 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// The next ticket for a workgroup working on queue cur (of XCD x): the queue
// and the ticket, or ticket ~0 when no queue is left for this XCD.  tried:
// queues looked at so far, starting with the XCD's own.
__device__ __forceinline__ unsigned take_ticket(const BatchState& S, int x, int& tried, int& cur) {
  for (;;) {
    if (cur >= 0) {
      const unsigned total = 2u * (unsigned)S.nsteps * (unsigned)(S.qbase[cur + 1] - S.qbase[cur]);
      const unsigned t = __hip_atomic_fetch_add(S.ticket + cur, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t < total) return t;
      cur = -1;
      if (!S.local) return ~0u;
    }
    if (tried == kXcds) return ~0u;
    const int q = S.local ? (x + tried) & (kXcds - 1) : 0;
    ++tried;
    if (S.local) {
      int o = -1;
      const bool mine = __hip_atomic_compare_exchange_strong(S.owner + q, &o, x, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
      if (mine || o == x) cur = q;
    } else {
      cur = q;
    }
  }
}

// One stage of an item's rows: each of the four waves takes a quarter of them
// and marches it strip by strip across the row, so any row width keeps all
// four busy and no barrier falls inside the item.
template <int STAGE, typename ST, int FORM>
__device__ __forceinline__ double item_rows(const StageArgs& A, double* lds, int r0, int rows, double dt,
                                            unsigned& bad) {
  const Geometry& G = A.geo;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r1 = min(r0 + rows, G.nm);
  const int per = (r1 - r0 + kWaves2 - 1) / kWaves2;
  const int k0 = r0 + w * per, k1 = min(k0 + per, r1);
  double cmax = 0.0;
  if (k0 < k1) {
    const Tile2 none{nullptr, 0, 0};
    for (int c = 0; c < G.cols.ncol; ++c)
      cmax = fmax(cmax, march2<kSplit, STAGE, ST, FORM, kLdAgent>(A, lane_of(G.cols, G.nx, A.bc_lo[0] == 0, c),
                                                                  lds + w * kLds2, none, k0, k1, k0, k1, true,
                                                                  [&]() { return dt; }, bad));
  }
  return cmax;
}

// Thread 0 acts for the workgroup in exactly one region per iteration: it
// signals the item just finished and takes the next ticket.  Both sit
// between barriers, so no single-thread region ends one iteration and another
// begins the next; the compiler could otherwise join the two across the back
// edge into a loop that thread 0 leaves while the rest of its wave goes round
// without it.  The dependency wait is the whole first wave's, one lane per
// flag, in a loop that is uniform over the wave.
template <typename ST, int FORM>
__global__ void __launch_bounds__(kBatchThreads) __attribute__((amdgpu_waves_per_eu(kBatchPerCU))) batch_kernel(
    const BoxDev* __restrict__ boxes, const Item* __restrict__ items, BatchState S) {
  extern __shared__ double lds[];
  __shared__ unsigned tshare, skip;
  __shared__ int qshare, tried;  // queue worked on, queues looked at so far
  __shared__ Pending prev;       // the item being worked on
  __shared__ double red[kBatchThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x = xcc_id();
  if (tid == 0) {
    qshare = -1;
    tried = 0;
    prev.b = -1;
  }
  __syncthreads();
  for (;;) {
    if (tid == 0) {
      if (prev.b >= 0) signal_done(S, prev, red);
      tshare = take_ticket(S, x, tried, qshare);
    }
    __syncthreads();
    const unsigned t = __builtin_amdgcn_readfirstlane(tshare);  // uniform: SGPR box fields
    const int qu = __builtin_amdgcn_readfirstlane(qshare);
    __syncthreads();
    if (t == ~0u) break;
    const int i0 = S.qbase[qu], ni = S.qbase[qu + 1] - i0;
    const int q = (int)(t / (unsigned)ni), r = i0 + (int)(t % (unsigned)ni);
    // box and block are workgroup-uniform: said explicitly, every field of
    // the box's stage views stays in scalar registers (otherwise the compiler
    // wraps each buffer access built from them in a per-lane waterfall loop)
    const int b = __builtin_amdgcn_readfirstlane(items[r].box), p = __builtin_amdgcn_readfirstlane(items[r].blk);
    const int n = q >> 1;
    const bool st2 = (q & 1) != 0;
    const BoxDev& B = boxes[b];
    if (w == 0) {
      // lane d < ndep: neighbour block d of the previous stage; the next
      // lane: for stage 1, the box's stage-2 count of the previous step
      const int ndep = q > 0 ? items[r].ndep : 0;
      const unsigned* p0 = nullptr;
      unsigned need = 1u;
      if (lane < ndep) {
        p0 = S.done + (long long)(q - 1) * S.nitem + B.rbase + items[r].dep[lane];
      } else if (lane == ndep && !st2 && n > 0) {
        p0 = S.cnt2 + (long long)b * S.max_steps + (n - 1);
        need = (unsigned)B.nblk;
      }
      const unsigned long long deadline = wall_clock64() + S.wait_ticks;
      bool ok = true;
      for (;;) {
        const bool here = !p0 || ld_agent(p0) >= need;
        if (__all(here)) break;
        if (wall_clock64() > deadline) {
          ok = false;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
      if (!S.local) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (lane == 0) {
        if (!ok) atomicOr(S.flags, kQueueTimeout);
        skip = ok ? 0u : 1u;
      }
    }
    __syncthreads();
    const bool skip_item = __builtin_amdgcn_readfirstlane(skip) != 0u;
    const unsigned long long mb = ld_agent(S.maxbits + (long long)b * (S.max_steps + 1) + n);
    const double dt = B.cfl_h / __longlong_as_double((long long)mb);
    unsigned bad = 0;
    double cmax = 0.0;
    if (skip_item) {
      // nothing computed or stored; the item is still signalled done below
    } else if (!st2) {
      cmax = item_rows<1, ST, FORM>(B.s1, lds, p * B.rows, B.rows, dt, bad);
    } else {
      cmax = item_rows<2, ST, FORM>(B.s2, lds, p * B.rows, B.rows, dt, bad);
    }
    if (bad) atomicOr(S.flags, bad);
    if (st2) {
      const double wm = wave_max(cmax);
      if (lane == 0) red[w] = wm;
    }
    // every wave's stores have reached L2 before the signal
    wait_stores();
    if (tid == 0) prev = Pending{b, p, n, (unsigned)q, (unsigned)r, st2, dt};
    __syncthreads();
  }
}

template <typename ST>
static void* batch_kernel_ptr(int form) {
  switch (form) {
    case kEuler: return (void*)batch_kernel<ST, kEuler>;
    case kPVS: return (void*)batch_kernel<ST, kPVS>;
    case kPMS: return (void*)batch_kernel<ST, kPMS>;
    case kDVS: return (void*)batch_kernel<ST, kDVS>;
    case kDMS: return (void*)batch_kernel<ST, kDMS>;
    default: return (void*)batch_kernel<ST, kPD>;
  }
}

}  // namespace rsstk

using namespace rsstk;

struct rsst_batch_s {
  int nbox, prec, form, max_steps;
  std::vector<rsst_config> cfg;
  std::vector<long long> off;     // element offsets of the boxes in U_all
  long long total_elems;          // size of U_all (elements)
  int strip[4];                   // strip rows per width class (1..4 waves per row)
  // per-build host tables
  std::vector<BoxDev> boxes;
  std::vector<Item> items;
  int nitem;
  int local;                      // one queue per XCD
  int qbase[kXcds + 1];           // first item of each queue
  size_t lds_bytes;
  // device memory
  void* u1;
  BoxDev* d_boxes;
  Item* d_items;
  int d_items_cap;
  unsigned* d_ticket;
  int* d_owner;
  unsigned long long* d_maxbits;
  unsigned* d_cnt2;
  unsigned* d_done;
  long long d_done_cap;
  double* d_tacc;
  unsigned* d_flags;
  // graph of the last run
  hipStream_t cap_stream;
  hipGraphExec_t exec;
  void* cap_U;
  int cap_steps;
  bool dirty;
  int grid;
  unsigned long long wait_ticks;  // dependency-wait limit of the queue (100 MHz ticks)
};

static int batch_validate(const rsst_config* c, int nbox, const int64_t* off) {
  if (!c || nbox < 1 || !off) return RSST_E_ARG;
  for (int b = 0; b < nbox; ++b) {
    const rsst_config& k = c[b];
    if (k.ndim != 2) return RSST_E_UNSUPPORTED;
    if (k.n[0] < 4 || k.n[1] < 4 || k.n[2] != 1) return RSST_E_ARG;
    if (k.n[0] > 256) return RSST_E_UNSUPPORTED;
    if (!(k.dx[0] > 0) || !(k.dx[1] > 0)) return RSST_E_ARG;
    for (int d = 0; d < 2; ++d) {
      if (k.bc_lo[d] < RSST_PERIODIC || k.bc_lo[d] > RSST_REFLECT_HYDRO) return RSST_E_ARG;
      if (k.bc_hi[d] < RSST_PERIODIC || k.bc_hi[d] > RSST_REFLECT_HYDRO) return RSST_E_ARG;
      if ((k.bc_lo[d] == RSST_PERIODIC) != (k.bc_hi[d] == RSST_PERIODIC)) return RSST_E_ARG;
    }
    if (!(k.gamma > 1.0) || !(k.xi >= 1.0) || !(k.cfl > 0.0 && k.cfl <= 1.0)) return RSST_E_ARG;
    if (k.form != c[0].form || k.prec != c[0].prec) return RSST_E_UNSUPPORTED;
    if (k.form < RSST_EULER || k.form > RSST_PD) return RSST_E_ARG;
    if (k.prec == RSST_FP32_PERT && (!k.bg || (k.bg_axis != -1 && k.bg_axis != 1))) return RSST_E_ARG;
    if (k.t_end != 0.0 || k.cmax != 0.0 || k.flags != 0 || k.eos != RSST_EOS_IDEAL) return RSST_E_UNSUPPORTED;
    for (int d = 0; d < 2; ++d)
      if (k.bc_lo[d] == RSST_REFLECT_HYDRO || k.bc_hi[d] == RSST_REFLECT_HYDRO) return RSST_E_UNSUPPORTED;
    if (off[b] < 0) return RSST_E_ARG;
    const long long bytes = 4ll * k.n[0] * k.n[1] * (k.prec == RSST_FP32_PERT ? 4 : 8);
    if (bytes >= (1ll << 31)) return RSST_E_UNSUPPORTED;
  }
  return RSST_OK;
}

// Row index after the boundary rule of the marched axis (the host copy of
// the device rule: reflecting sides mirror, periodic sides wrap).
static int host_map_row(int q, int n, int refl_lo, int refl_hi) {
  if (q < 0) return refl_lo ? -1 - q : q + n;
  if (q >= n) return refl_hi ? 2 * n - 1 - q : q - n;
  return q;
}

// Chunks of strip rows in a row block: as many as rows of the box's waves fill
// the four of a workgroup.  Rows of 61 to 64 cells between walls are one wave
// wide but two strips, so a wave marches two chunks of a block of four: in small
// batches (`halve`) such a block is two chunks, one march per wave.  us per
// step with four and two, 64 x 64 FP64: 1 box 77 and 44, 20 boxes 76 and 43, 384
// boxes 123 and 108; 64 x 200: 200 boxes (800 blocks of four) 186 and 168, 384
// boxes (1536) 320 and 326, 768 boxes 636 and 666.
static int chunks_of(const rsst_config& c, bool halve) {
  const int nwx = (c.n[0] + 63) / 64;
  return halve && nwx == 1 && plan_cols2(c.n[0], c.bc_lo[0] == RSST_PERIODIC, 2).ncol == 2 ? 2 : 4 / nwx;
}

// A small batch: fewer row blocks than 4/3 of the workgroups that run at once.
static bool small_batch(const rsst_config* c, int nbox, const int strip[4]) {
  long long blocks = 0;
  for (int b = 0; b < nbox; ++b) {
    const int nwx = (c[b].n[0] + 63) / 64, rows = chunks_of(c[b], false) * std::min(strip[nwx - 1], c[b].n[1]);
    blocks += (c[b].n[1] + rows - 1) / rows;
  }
  return blocks < 4 * 256 * kBatchPerCU / 3;
}

// Row blocks of one box and their dependency lists, appended to `items`.  A
// block is `groups` chunks of `km` rows, marched along y.
static int plan_box(const rsst_config& c, const int strip[4], bool halve, int b, std::vector<Item>& items, int& km,
                    int& groups, int& nblk) {
  const int nx = c.n[0], nm = c.n[1];
  const int nwx = (nx + 63) / 64;
  groups = chunks_of(c, halve);
  km = strip[nwx - 1] < nm ? strip[nwx - 1] : nm;
  const int nchunk = (nm + km - 1) / km;
  nblk = (nchunk + groups - 1) / groups;
  // rows [k0, k1) of each block; blocks reading each other's rows
  const int rows = groups * km;
  const int rlo = c.bc_lo[1] == RSST_REFLECT, rhi = c.bc_hi[1] == RSST_REFLECT;
  std::vector<std::vector<char>> rel(nblk, std::vector<char>(nblk, 0));
  for (int p = 0; p < nblk; ++p) {
    const int k0 = p * rows, k1 = std::min(k0 + rows, nm);
    for (int k = k0 - 2; k < k1 + 2; ++k) {
      const int o = host_map_row(k, nm, rlo, rhi) / rows;
      rel[p][o] = rel[o][p] = 1;
    }
  }
  for (int p = 0; p < nblk; ++p) {
    Item it{};
    it.box = b;
    it.blk = p;
    for (int o = 0; o < nblk; ++o)
      if (rel[p][o]) {
        if (it.ndep == kMaxDeps) return RSST_E_UNSUPPORTED;
        it.dep[it.ndep++] = o;
      }
    items.push_back(it);
  }
  return RSST_OK;
}

// Deals the boxes to the queues: order lists them queue by queue (in the
// caller's order within a queue), qfirst[q] is where queue q starts.  Each
// box goes to the queue with the least work so far, largest box first (work:
// wave-rows, rows times strips).  Returns 1 for a queue per XCD.  Where the
// fullest queue holds more than 1.25 of the mean (few boxes, or a few large
// ones), all go to queue 0 for the whole chip and 0 is returned: the chip then
// waits for one XCD longer than the write-backs between XCDs would cost.  us
// per step with one queue and with one per XCD, by the fullest queue's share of
// the mean: FP64, 1: 8 boxes of 256 x 256 76 and 66; 1.2: 20 of 256 x 1024 368
// and 298; 1.28: 25 of 256 x 512 182 and 182; 1.33: 12 of 256 x 1024 188 and 178;
// 1.41: 17 of them 297 and 286; 1.6 and 1.78: 10 and 9 of them 171 and 176, 160
// and 173.  FP32, in the same order: 89 and 71, 262 and 277, 174 and 185, 185 and
// 190, 232 and 266, 174 and 191, 165 and 187.  Boxes of 64 and 128 rows a side
// gain a little at any share (25 of 64 x 64 46 and 42, 19 of 128 x 128 72 and 63),
// those of 256 lose (10 of 256 x 256 82 and 85).  1.25 is about where large
// boxes turn in FP64; in FP32 they turn a little below it, small boxes above.
static int deal_boxes(const std::vector<rsst_config>& cfg, std::vector<int>& order, int qfirst[kXcds + 1]) {
  const int nbox = (int)cfg.size();
  std::vector<long long> work(nbox);
  long long sum = 0;
  for (int b = 0; b < nbox; ++b) {
    work[b] = (long long)plan_cols2(cfg[b].n[0], cfg[b].bc_lo[0] == RSST_PERIODIC, 2).ncol * cfg[b].n[1];
    sum += work[b];
  }
  std::vector<int> by(nbox);
  for (int b = 0; b < nbox; ++b) by[b] = b;
  std::stable_sort(by.begin(), by.end(), [&](int p, int q) { return work[p] > work[q]; });
  long long load[kXcds] = {0};
  std::vector<int> queue(nbox, 0);
  for (int b : by) {
    const int q = (int)(std::min_element(load, load + kXcds) - load);
    queue[b] = q;
    load[q] += work[b];
  }
  const long long top = *std::max_element(load, load + kXcds);
  const int local = top * kXcds * 4 <= sum * 5;
  order.clear();
  for (int q = 0; q < kXcds; ++q) {
    qfirst[q] = (int)order.size();
    for (int b = 0; b < nbox; ++b)
      if ((local ? queue[b] : 0) == q) order.push_back(b);
  }
  qfirst[kXcds] = nbox;
  return local;
}

// Stage views, row blocks and the item table for the current strip rows.
static int batch_build(rsst_batch_s* h, void* U) {
  h->boxes.assign(h->nbox, BoxDev{});
  h->items.clear();
  size_t lds = 0;
  std::vector<int> order;
  int qfirst[kXcds + 1];
  h->local = deal_boxes(h->cfg, order, qfirst);
  const bool halve = small_batch(h->cfg.data(), h->nbox, h->strip);
  int qu = 0;
  for (int o = 0; o < h->nbox; ++o) {
    const int b = order[o];
    while (qu < kXcds && qfirst[qu] <= o) h->qbase[qu++] = (int)h->items.size();
    const rsst_config& c = h->cfg[b];
    BoxDev& B = h->boxes[b];
    B.rbase = (int)h->items.size();
    int km = 0, groups = 0, nblk = 0;
    const int ps = plan_box(c, h->strip, halve, b, h->items, km, groups, nblk);
    if (ps != RSST_OK) return ps;
    StageArgs a;
    std::memset(&a, 0, sizeof(a));
    Geometry& G = a.geo;
    G.ndim = 2;
    G.nx = c.n[0];
    G.ns = 1;
    G.nm = c.n[1];
    G.nwx = (G.nx + 63) / 64;
    G.ts = 1;
    G.km = km;
    G.cols = plan_cols2(G.nx, c.bc_lo[0] == RSST_PERIODIC, 2);
    G.ntile_s = 1;
    G.nchunk = (G.nm + G.km - 1) / G.km;
    G.threads = kBatchThreads;
    G.lds_bytes = (size_t)kRed2 * sizeof(double);
    if (G.lds_bytes > lds) lds = G.lds_bytes;
    a.ncell = (long long)G.nx * G.nm;
    for (int d = 0; d < 3; ++d) {
      a.bc_lo[d] = c.bc_lo[d];
      a.bc_hi[d] = c.bc_hi[d];
      a.inv_dx[d] = d < 2 ? 1.0 / c.dx[d] : 0.0;
      a.g[d] = d < 2 ? c.g[d] : 0.0;
    }
    a.gamma = c.gamma;
    a.gm1 = c.gamma - 1.0;
    a.inv_gm1 = 1.0 / (c.gamma - 1.0);
    a.inv_xi = 1.0 / c.xi;
    a.f = 1.0 - 1.0 / (c.xi * c.xi);
    a.form = c.form;
    a.prec = c.prec;
    a.bg = c.bg;
    a.bg_axis = c.prec == RSST_FP32_PERT ? c.bg_axis : -1;
    a.nbg = a.bg_axis >= 0 ? c.n[a.bg_axis] : 1;
    a.bg_uniform = (a.bg_axis == -1 || a.bg_axis == 1) ? 1 : 0;
    const size_t es = c.prec == RSST_FP32_PERT ? 4 : 8;
    char* u = (char*)U + h->off[b] * es;
    char* u1 = (char*)h->u1 + h->off[b] * es;
    B.s1 = a;
    B.s1.uin = u;
    B.s1.un = nullptr;
    B.s1.uout = u1;
    B.s2 = a;
    B.s2.uin = u1;
    B.s2.un = u;
    B.s2.uout = u;
    double hl;
    if (c.dt_rule == 1) hl = std::fmin(c.dx[0], c.dx[1]);
    else hl = 1.0 / (1.0 / c.dx[0] + 1.0 / c.dx[1]);
    B.cfl_h = c.cfl * hl;
    B.rows = groups * km;
    B.nblk = nblk;
  }
  h->nitem = (int)h->items.size();
  while (qu <= kXcds) h->qbase[qu++] = h->nitem;
  h->lds_bytes = lds;
  return RSST_OK;
}

template <typename ST>
static hipError_t batch_launch_all(rsst_batch_s* h, hipStream_t s, int nsteps) {
  BatchState S;
  S.ticket = h->d_ticket;
  S.owner = h->d_owner;
  S.maxbits = h->d_maxbits;
  S.cnt2 = h->d_cnt2;
  S.done = h->d_done;
  S.tacc = h->d_tacc;
  S.flags = h->d_flags;
  S.nbox = h->nbox;
  S.nitem = h->nitem;
  S.nsteps = nsteps;
  S.max_steps = h->max_steps;
  S.local = h->local;
  for (int q = 0; q <= kXcds; ++q) S.qbase[q] = h->qbase[q];
  S.wait_ticks = h->wait_ticks;
  hipLaunchKernelGGL(batch_reset_kernel, dim3(256), dim3(256), 0, s, S);
  const int bpb = 8;
  hipLaunchKernelGGL(batch_prime_kernel<ST>, dim3(h->nbox * bpb), dim3(256), 0, s, h->d_boxes, S, bpb);
  void* kern = batch_kernel_ptr<ST>(h->form);
  void* args[] = {(void*)&h->d_boxes, (void*)&h->d_items, (void*)&S};
  hipError_t e = hipLaunchKernel(kern, dim3(h->grid), dim3(kBatchThreads), args, h->lds_bytes, s);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

static int batch_prepare(rsst_batch_s* h, void* U, int nsteps) {
  const int bs = batch_build(h, U);
  if (bs != RSST_OK) return bs;
  if (h->nitem > h->d_items_cap || 2ll * h->max_steps * h->nitem > h->d_done_cap)
    return RSST_E_UNSUPPORTED;  // strip rows below those sized at init
  if (hipMemcpy(h->d_boxes, h->boxes.data(), sizeof(BoxDev) * h->nbox, hipMemcpyHostToDevice) != hipSuccess)
    return RSST_E_DEVICE;
  if (hipMemcpy(h->d_items, h->items.data(), sizeof(Item) * h->nitem, hipMemcpyHostToDevice) != hipSuccess)
    return RSST_E_DEVICE;
  void* kern = h->prec ? batch_kernel_ptr<float>(h->form) : batch_kernel_ptr<double>(h->form);
  if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)h->lds_bytes) != hipSuccess)
    return RSST_E_DEVICE;
  int per_cu = 0, dev = 0, ncu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kBatchThreads, h->lds_bytes) != hipSuccess)
    return RSST_E_DEVICE;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return RSST_E_DEVICE;
  // at most kBatchPerCU workgroups per CU
  if (per_cu > kBatchPerCU) per_cu = kBatchPerCU;
  h->grid = (per_cu > 0 ? per_cu : 1) * ncu;
  // capture reset + prime + persistent kernel in one graph
  if (h->exec) {
    (void)hipGraphExecDestroy(h->exec);
    h->exec = nullptr;
  }
  hipGraph_t graph = nullptr;
  if (hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal) != hipSuccess) return RSST_E_DEVICE;
  hipError_t e = h->prec ? batch_launch_all<float>(h, h->cap_stream, nsteps)
                         : batch_launch_all<double>(h, h->cap_stream, nsteps);
  hipError_t e2 = hipStreamEndCapture(h->cap_stream, &graph);
  if (e != hipSuccess || e2 != hipSuccess || !graph) {
    if (graph) (void)hipGraphDestroy(graph);
    return RSST_E_DEVICE;
  }
  e = hipGraphInstantiate(&h->exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) return RSST_E_DEVICE;
  h->cap_U = U;
  h->cap_steps = nsteps;
  h->dirty = false;
  return RSST_OK;
}

extern "C" {

int rsst_batch_init(const rsst_config* boxes, int nbox, const int64_t* offsets, int max_steps,
                    void* stream, rsst_batch* out) {
  if (!out) return RSST_E_ARG;
  *out = nullptr;
  if (max_steps < 1) return RSST_E_ARG;
  int st = batch_validate(boxes, nbox, offsets);
  if (st != RSST_OK) return st;
  rsst_batch_s* h = new (std::nothrow) rsst_batch_s();
  if (!h) return RSST_E_NOMEM;
  h->nbox = nbox;
  h->prec = boxes[0].prec;
  h->form = boxes[0].form;
  h->max_steps = max_steps;
  h->cfg.assign(boxes, boxes + nbox);
  h->off.resize(nbox);
  h->total_elems = 0;
  for (int b = 0; b < nbox; ++b) {
    h->off[b] = offsets[b];
    const long long end = offsets[b] + 4ll * boxes[b].n[0] * boxes[b].n[1];
    if (end > h->total_elems) h->total_elems = end;
  }
  h->strip[0] = h->strip[1] = h->strip[2] = h->strip[3] = 16;
  h->wait_ticks = 1000000000ull;  // 10 s
  // size item tables for the shortest strips the tile setter accepts (8 rows)
  long long cap_items = 0;
  for (int b = 0; b < nbox; ++b) {
    const int groups = chunks_of(boxes[b], true);
    cap_items += ((boxes[b].n[1] + 7) / 8 + groups - 1) / groups;
  }
  const size_t es = h->prec == RSST_FP32_PERT ? 4 : 8;
  h->d_items_cap = (int)cap_items;
  h->d_done_cap = 2ll * max_steps * cap_items;
  bool ok = hipMalloc(&h->u1, (size_t)h->total_elems * es) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_boxes, sizeof(BoxDev) * nbox) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_items, sizeof(Item) * (size_t)cap_items) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_ticket, sizeof(unsigned) * kXcds) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_owner, sizeof(int) * kXcds) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_maxbits, sizeof(unsigned long long) * (size_t)nbox * (max_steps + 1)) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_cnt2, sizeof(unsigned) * (size_t)nbox * max_steps) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_done, sizeof(unsigned) * (size_t)h->d_done_cap) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_tacc, sizeof(double) * nbox) == hipSuccess;
  ok = ok && hipMalloc((void**)&h->d_flags, sizeof(unsigned)) == hipSuccess;
  ok = ok && hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking) == hipSuccess;
  if (!ok) {
    rsst_batch_destroy(h);
    return RSST_E_NOMEM;
  }
  hipStream_t s = (hipStream_t)stream;
  if (hipMemsetAsync(h->d_tacc, 0, sizeof(double) * nbox, s) != hipSuccess ||
      hipMemsetAsync(h->d_flags, 0, sizeof(unsigned), s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    rsst_batch_destroy(h);
    return RSST_E_DEVICE;
  }
  h->dirty = true;
  *out = h;
  return RSST_OK;
}

int rsst_batch_plan(const rsst_config* boxes, int nbox, const int strip_rows[4], int* table, int cap,
                    int* nitem) {
  if (!boxes || nbox < 1 || !strip_rows || !nitem || cap < 0 || (cap > 0 && !table)) return RSST_E_ARG;
  std::vector<int64_t> off(nbox, 0);
  const int st = batch_validate(boxes, nbox, off.data());
  if (st != RSST_OK) return st;
  for (int c = 0; c < 4; ++c)
    if (strip_rows[c] < 8 || strip_rows[c] > 256) return RSST_E_ARG;
  std::vector<Item> items;
  const bool halve = small_batch(boxes, nbox, strip_rows);
  for (int b = 0; b < nbox; ++b) {
    int km = 0, groups = 0, nblk = 0;
    const int ps = plan_box(boxes[b], strip_rows, halve, b, items, km, groups, nblk);
    if (ps != RSST_OK) return ps;
    for (size_t i = items.size() - nblk; i < items.size(); ++i) {
      const Item& it = items[i];
      if ((long long)i >= cap) continue;
      int* row = table + i * RSST_BATCH_PLAN_COLS;
      const int rows = groups * km;
      row[0] = it.box;
      row[1] = it.blk;
      row[2] = it.blk * rows;
      row[3] = std::min((it.blk + 1) * rows, boxes[b].n[1]);
      row[4] = it.ndep;
      for (int d = 0; d < kMaxDeps; ++d) row[5 + d] = d < it.ndep ? it.dep[d] : -1;
    }
  }
  *nitem = (int)items.size();
  return RSST_OK;
}

int rsst_batch_queues(const rsst_config* boxes, int nbox, int* nqueue) {
  if (!boxes || nbox < 1 || !nqueue) return RSST_E_ARG;
  const std::vector<int64_t> off(nbox, 0);
  const int st = batch_validate(boxes, nbox, off.data());
  if (st != RSST_OK) return st;
  std::vector<int> order;
  int qfirst[kXcds + 1];
  *nqueue = deal_boxes(std::vector<rsst_config>(boxes, boxes + nbox), order, qfirst) ? kXcds : 1;
  return RSST_OK;
}

int rsst_batch_set_tiles(rsst_batch h, const int strip_rows[4]) {
  if (!h || !strip_rows) return RSST_E_ARG;
  for (int c = 0; c < 4; ++c)
    if (strip_rows[c] < 8 || strip_rows[c] > 256) return RSST_E_ARG;
  for (int c = 0; c < 4; ++c) h->strip[c] = strip_rows[c];
  h->dirty = true;
  return RSST_OK;
}

int rsst_batch_get_tiles(rsst_batch h, int strip_rows[4]) {
  if (!h || !strip_rows) return RSST_E_ARG;
  for (int c = 0; c < 4; ++c) strip_rows[c] = h->strip[c];
  return RSST_OK;
}

int rsst_batch_run(rsst_batch h, void* U_all, int nsteps, void* stream) {
  if (!h || !U_all || nsteps < 1 || nsteps > h->max_steps) return RSST_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  if (h->dirty || U_all != h->cap_U || nsteps != h->cap_steps) {
    // rebuilding the tables copies from the host: order after earlier work
    if (hipStreamSynchronize(s) != hipSuccess) return RSST_E_DEVICE;
    int st = batch_prepare(h, U_all, nsteps);
    if (st != RSST_OK) return st;
  }
  return hipGraphLaunch(h->exec, s) == hipSuccess ? RSST_OK : RSST_E_DEVICE;
}

int rsst_batch_times(rsst_batch h, double* t, void* stream) {
  if (!h || !t) return RSST_E_ARG;
  if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return RSST_E_DEVICE;
  return hipMemcpy(t, h->d_tacc, sizeof(double) * h->nbox, hipMemcpyDeviceToHost) == hipSuccess
             ? RSST_OK
             : RSST_E_DEVICE;
}

int rsst_batch_set_wait_limit(rsst_batch h, double seconds) {
  if (!h || !(seconds >= 0.0) || !(seconds <= 3600.0)) return RSST_E_ARG;
  h->wait_ticks = (unsigned long long)(seconds * 1e8);
  h->dirty = true;
  return RSST_OK;
}

int rsst_batch_set_times(rsst_batch h, const double* t, uint32_t flags, void* stream) {
  if (!h || !t) return RSST_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  if (hipStreamSynchronize(s) != hipSuccess) return RSST_E_DEVICE;
  if (hipMemcpy(h->d_tacc, t, sizeof(double) * h->nbox, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(h->d_flags, &flags, sizeof(flags), hipMemcpyHostToDevice) != hipSuccess)
    return RSST_E_DEVICE;
  return RSST_OK;
}

int rsst_batch_poll(rsst_batch h, uint32_t* flags) {
  if (!h) return RSST_E_ARG;
  if (hipDeviceSynchronize() != hipSuccess) return RSST_E_DEVICE;
  uint32_t f = 0;
  if (hipMemcpy(&f, h->d_flags, sizeof(f), hipMemcpyDeviceToHost) != hipSuccess) return RSST_E_DEVICE;
  if (f) {
    uint32_t z = 0;
    if (hipMemcpy(h->d_flags, &z, sizeof(z), hipMemcpyHostToDevice) != hipSuccess) return RSST_E_DEVICE;
  }
  if (flags) *flags = f;
  if (f & kQueueTimeout) return RSST_E_DEVICE;
  return f ? RSST_E_NONPHYSICAL : RSST_OK;
}

int rsst_batch_destroy(rsst_batch h) {
  if (!h) return RSST_E_ARG;
  (void)hipDeviceSynchronize();
  if (h->exec) (void)hipGraphExecDestroy(h->exec);
  if (h->cap_stream) (void)hipStreamDestroy(h->cap_stream);
  (void)hipFree(h->u1);
  (void)hipFree(h->d_boxes);
  (void)hipFree(h->d_items);
  (void)hipFree(h->d_ticket);
  (void)hipFree(h->d_owner);
  (void)hipFree(h->d_maxbits);
  (void)hipFree(h->d_cnt2);
  (void)hipFree(h->d_done);
  (void)hipFree(h->d_tacc);
  (void)hipFree(h->d_flags);
  delete h;
  return RSST_OK;
}

}  // extern "C"
