// C ABI and host runtime of the MI355X nonlocal-exchange library.
//
// Computes V^x_{nn'}(k) = - sum_q w_q sum_{n''} A^H v(q) A (the vector-matrix-
// vector form of Sec. III.C) on one gfx950 GPU. See include/exchange.h for the
// contract of every entry point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <map>
#include <vector>

#include "../../include/exchange.h"
#include "aux.hpp"
#include "chol.hpp"
#include "configs.hpp"
#include "tile.hpp"
#include "gamma.hpp"
#include "backx.hpp"
#include "plain.hpp"

using namespace exc;

namespace {

constexpr uint32_t kAlive = 0x45584331u;   // "EXC1"

// Scratch of the no-allocation entry point (exchange_matrix_noalloc): the partial slots and
// the block-sparse workspace of one k. One copy per GPU, held until the process ends; every
// call on a GPU shares it. Host code takes its device address from hipGetSymbolAddress
// (once per device, at exchange_init) and never uses the array's name as an address.
constexpr size_t kScratchBytes = (size_t)64 << 20;
constexpr int kScratchDevices = 64;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};

// Device buffers that replace the context's own for one call, of the no-allocation entry point or with shared FP64 slots
// (see ScratchView users: ws_base, tile_args, sparse_args, fused_args, cfg_sparse, cfg_reduce).
struct ScratchView {
  void* ws;          // workspace of the call's k, shifted by the k's first element
  double* dsp;       // FP64 |Y_s|^2 sums, shifted by the k's first pair
  void* gpart;       // Gram partial slots, shifted by the k's first slot
  double* dpart;     // FP64 diagonal partials, shifted likewise
};
thread_local std::string g_init_err;

struct KernelCfg {
  int mode, form, BM, KC, NCT, NB8M, NWR, NWC, NBUF;
  void (*fn)(TileArgs);
  size_t lds;
  int id;
  int gchain, grs, grd;             // binary32 Gram chains: kind, rows per chunk (sparse, dense)
  int NW() const { return NWR * NWC; }
};

#define CFG(MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF, ID)                                    \
  KernelCfg{MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF,                                         \
            tile_kernel<MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF>,                            \
            TileCfg<MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF>::LDS_B, ID,                     \
            TileCfg<MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF>::GCHAIN,                        \
            TileCfg<MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF>::GCH_RS,                        \
            TileCfg<MODE, FORM, BM, KC, NCT, NB8M, NWR, NWC, NBUF>::GCH_RD}

// Tile shapes: BM rows of the factor per step, split over NWR wavefronts; NCT
// 8-column band tiles per pass (n_b rounded to 8, times the n'' chunk), split
// over NWC wavefronts; KC complex k per LDS stage; NB8M the largest band-tile
// count per n'' value the instance contracts; NBUF K-loop buffers. The GEMM
// form stages two FP64 operands per row block and therefore stops at n_b <= 64.
const KernelCfg kCfgs[] = {
    CFG(M_F64, 0, 64, 16, 6, 3, 4, 1, 2, 0),       CFG(M_F64, 0, 64, 16, 8, 8, 4, 1, 2, 1),
    CFG(M_F32, 1, 128, 16, 12, 3, 4, 2, 2, 20),    CFG(M_F32, 1, 128, 16, 8, 8, 4, 2, 2, 21),
    CFG(M_F32, 1, 64, 16, 13, 13, 4, 1, 2, 23),   CFG(M_F32, 1, 128, 16, 16, 16, 4, 2, 2, 22),
    CFG(M_BF16X3, 1, 128, 32, 12, 3, 4, 2, 2, 30), CFG(M_BF16X3, 1, 128, 32, 8, 8, 4, 2, 2, 31),
    CFG(M_BF16X3, 1, 64, 32, 13, 13, 4, 1, 2, 33), CFG(M_BF16X3, 1, 64, 32, 16, 16, 4, 1, 2, 32),
    CFG(M_BF16X6, 1, 64, 32, 12, 3, 2, 2, 2, 40),  CFG(M_BF16X6, 1, 64, 32, 8, 8, 2, 2, 2, 41),
    CFG(M_BF16X6, 1, 64, 32, 13, 13, 4, 1, 1, 43), CFG(M_BF16X6, 1, 64, 32, 16, 16, 4, 1, 1, 42),
};

// Every fused and wide instance, in order of preference among equal band-tile capacity.
const std::vector<FusedKCfg>& all_fused() {
  static const std::vector<FusedKCfg> t = [] {
    std::vector<FusedKCfg> v(kFusedCfgs, kFusedCfgs + kNumFused);
    v.insert(v.end(), kWideCfgs, kWideCfgs + kNumWide);
    return v;
  }();
  return t;
}

struct Plan {
  std::vector<WorkItem> items;      // generation order: pair-major, slot = index
  std::vector<int> pair_item;       // [n_pairs + 1] item range per pair
  std::vector<int> k_item;          // [n_k + 1] item range per k
  std::vector<int> slot_begin;      // [n_k + 1]
  std::vector<double> slot_w;
  WorkItem* d_items = nullptr;      // generation order
  WorkItem* d_items_lpt = nullptr;  // longest-processing-time order
  WorkItem* d_items_xq = nullptr;   // per-XCD queues, each in LPT order (fused path)
  int32_t* d_qbeg = nullptr;        // [nq + 1]
  int nq = 1;
  int32_t* d_slot_begin = nullptr;
  double* d_slot_w = nullptr;
  int n_slots = 0;
  const Herk64K* h64 = nullptr;     // FP64 HERK: the kernel of this plan
  WorkItem* d_order = nullptr;      //  its items in launch order (padding items: pair -1)
  std::vector<int> order_begin;     //  [launches + 1]: every k at once, or one launch per k or pair
};

// One k of few pairs in a fused instance that streams its Gram tiles: items per n'' chunk and row part, every chunk of
// 64 rows in a slot of its own, a batch of pairs at a time.
struct ChunkPlan {
  struct Batch { int item0, items, pair0, pairs; };
  std::vector<Batch> batches;       // (none: one item per pair)
  WorkItem* d_items = nullptr;
  int32_t* d_base = nullptr;        // [pairs of k] first chunk slot in the batch
  int npass = 0;
  size_t slots = 0;                 // of the largest batch
};

// The last use of buffers that one call at a time may use (turn_begin).
struct Turn {
  hipEvent_t ev = nullptr;            // its end (created once a second stream uses them)
  hipStream_t st = nullptr;
  bool used = false;
};

}  // namespace

struct NnState;        // learned extrapolator (nn_abi.hpp)
struct LearnScratch;

struct exc_ctx {
  uint32_t magic = kAlive;
  std::string err;
  int n_k = 0, n_q = 0, n_occ = 0, n_ch = 0, precision = 0, form = 0, batched = 0, device = 0;
  // n_occ: columns n'' of M per band n (the kernels' view). With inversion symmetry two real
  // occupied bands share one complex column, so n_occ_v (occupied bands of V, for the
  // energy and the Gamma-point shift) is 2 n_occ or 2 n_occ - 1; otherwise n_occ_v = n_occ.
  int n_occ_v = 0;
  bool real_v = false;                // inversion symmetry: V = Re of the packed product
  std::vector<int> nb, npw, nrad, nd, nmb;
  std::vector<double> wq;
  std::vector<double> wkq;            // [n_k * n_q] weight of pair (k, q); 0: pair not computed
  bool has_wkq = false;               // the caller gave per-pair weights
  int n_s = 0, nb_max = 0, nbt_max = 0, ns_pad = 0;
  std::vector<int> ch_off, ch_len;
  std::vector<int64_t> ch_coef;
  int64_t coef_total = 0;
  int nqc = 1;                        // copies of the channel blocks (n_q when they depend on q)
  // device-resident Coulomb data
  double2* d_coef = nullptr;
  double2* d_cvec = nullptr;
  double* d_schur = nullptr;
  void* d_U = nullptr;
  std::vector<int64_t> u_off;
  std::vector<int> ldu;
  int32_t *d_row_chan = nullptr, *d_ch_off = nullptr, *d_ch_len = nullptr;
  int4* d_rowinfo = nullptr;          // fused kernel: per multipole-free row (see FusedArgs)
  double2* d_runs = nullptr;          // HERK sparse_kernel: coefficient runs by row (see SparseArgs)
  int run_max = 0, runs_ld = 0;       //  longest run, rows per run entry (n_s rounded up to 8)
  double2* d_coefpad = nullptr;       // fused kernel: padded coefficient runs (see FusedArgs)
  int4* d_schunk = nullptr;           // fused kernel: chunks of whole channels (see FusedArgs)
  uint2* d_sgroup = nullptr;          // fused kernel: row groups of each chunk (see FusedArgs)
  RowUnits row_units{};               // fused kernels: the block-sparse rows in operand order (rows.hpp)
  RowUnit* d_units = nullptr;
  int32_t* d_ucount = nullptr;
  int2* d_uowner = nullptr;
  d2_t* d_uw = nullptr;
  std::vector<int4> h_schunk;
  int n_schunk = 0;
  int64_t* d_ch_coef = nullptr;
  // pairs, plans, buffers
  std::vector<PairInfo> pairs;
  PairInfo* d_pairs = nullptr;
  std::vector<int> k_pair;            // [n_k + 1]
  std::vector<int64_t> m_len;         // [n_k] elements of M(k) (the blocks of its pairs)
  std::vector<double> pair_w;
  double* d_pair_w = nullptr;
  int32_t* d_pair_begin = nullptr;
  Plan plain, bat, perk;              // perk: FP64 HERK, one launch per k (bat when there is one k)
  Plan capt;                          // FP64 HERK with part_shared: of captured calls, slots from part_slots on
  bool part_shared = false;           // every k of perk has the first part_slots slots, in turn
  size_t part_slots = 0;
  hipEvent_t ev_part = nullptr;       //  their last use
  bool h64 = false;                   // FP64 Cholesky/HERK through herk64_kernel
  Chunk64* d_chunk64 = nullptr;          // its chunks of block-sparse rows (complex128 M); none: sparse_kernel first
  int n_chunk64 = 0;
  const KernelCfg* cfg = nullptr;
  const FusedKCfg* fcfg = nullptr;    // non-null: reduced-precision HERK through the fused kernel
  bool fused = false;
  bool fused_ok = false;              // the fused kernel can serve this context
  int sncw = 1;                       // sparse_kernel (HERK form): columns per wavefront
  bool direct = true;                 // batched path: kernels enqueued one by one (EXC_GRAPH=1: a graph)
  bool t_sparse = false;              // (direct launches) the timed replays include a sparse kernel
  int fsplit = 0;                     // fused items: 1 = one per n'' chunk, 2 = one per n'' chunk and row
                                      // part (more, smaller items)
  int tuned = 0;                      // 0 default choice, 1 timed by the autotuner, 2 from the tune cache
  bool tune_done = false;
  size_t ws_bytes = 0;                // block-sparse workspace of all pairs (the batched graph)
  size_t ws_elem = 16;                // bytes per workspace element
  std::vector<int64_t> k_ws_start;    // [n_k + 1] first workspace element of each k's pairs
  size_t ws_k_bytes = 0;              // the largest workspace of one k (per-k calls)
  size_t ws_cap = 0;                  // bytes allocated at d_ws (grown on demand)
  void* d_ws = nullptr;
  double* d_dsp = nullptr;
  void* d_gpart = nullptr;
  double* d_dpart = nullptr;
  const ScratchView* sv = nullptr;    // set only during a call on other buffers than the context's
  int gstride = 0, dstride = 0;
  double2* d_vres = nullptr;
  std::vector<int64_t> v_off;
  int64_t* d_voff = nullptr;
  int32_t* d_knb = nullptr;
  std::vector<char> v_valid;
  // pointer tables (device) and their host mirrors
  void** d_mtab = nullptr;
  void** d_vtab = nullptr;
  std::vector<void*> h_mtab, h_vtab;  // what the tables hold, or will once ev_tab has passed
  hipEvent_t ev_tab = nullptr;
  std::map<int, ChunkPlan> chunk_plans;    // by k, made at its first call
  float* d_gchunk = nullptr;
  double* d_dchunk = nullptr;
  size_t chunk_cap = 0;               // slots
  size_t chunk_fail = SIZE_MAX;       // fewest slots that there was no room for
  int chunk_fails = 0;                // allocations that failed
  size_t chunk_bytes = (size_t)256 << 20;  // of the slots of a batch (EXC_CHUNK_BYTES)
  int chunk_batches = 0;              // batches of the last exchange_matrix call (0: one item per pair)
  hipEvent_t ev_chunk = nullptr;      // the last use of the chunk slots
  bool tab_pending = false;
  int32_t* d_counter = nullptr;
  int persist_grid = 0;
  // graph of the batched path
  hipGraphExec_t gexec = nullptr;
  hipStream_t own = nullptr;          // capturable stream of the batched path
  hipEvent_t ev_in = nullptr, ev_out = nullptr;
  hipEvent_t ev_en = nullptr;         // end of the last energy call (its buffers are shared)
  bool ev_en_set = false;
  Turn turn_ws, turn_bt;              // the workspace or the unbatched GEMM form's buffers; the back-transform's
  hipEvent_t ev_learn = nullptr;      // end of the last learned call (its buffers are shared)
  bool learn_set = false;             // (it was asynchronous)
  int g_dtype = -1;
  // live kernel timing of the batched path: event-record nodes around the
  // sparse and tile kernels; one pool entry (3 events) per graph replay
  hipGraph_t graph = nullptr;
  hipGraphNode_t tnode[3] = {nullptr, nullptr, nullptr};
  std::vector<hipEvent_t> tpool;      // 3 per slot
  int t_slots = 0, t_next = 0, t_count = 0;
  // staging for host-pointer calls
  void* d_mstage = nullptr;
  size_t mstage_bytes = 0;
  double* d_eout = nullptr;
  double* d_ewk = nullptr;            // [n_k] weights of exchange_energy_device
  void** d_erho = nullptr;            // [n_k] rho pointers of exchange_energy_device
  double* d_gamma = nullptr;          // [4] Gamma-point term: C, lattice sum, terms, diagonal shift
  double* d_gpartial = nullptr;       // [2 * kGammaGrid] per-workgroup partials of the lattice sum
  hipEvent_t ev_g[2] = {nullptr, nullptr};
  float gamma_ms = 0.f;               // lattice-sum kernel of the last exchange_gamma_term
  double gamma_terms = 0.0;           // its number of terms
  double2* d_bt = nullptr;            // back-transform workspace T = Z V (grown on demand)
  uint64_t* d_tmask = nullptr;        // [n_k][3] band-tile pairs (I, J) to compute, bit J(J+1)/2 + I
  size_t bt_cap = 0;
  hipEvent_t ev_bt[2] = {nullptr, nullptr};
  bool bt_timed = false;
  hipStream_t last_stream = nullptr;
  // plain GEMM form (unbatched): one pair at a time through sparse_kernel<0> and zgemm_kernel
  bool plain_gemm = false;
  PairInfo* d_ppairs = nullptr;       // the pairs with the column pitch of W = v A (N_MB, offset 0)
  double2* d_pw = nullptr;            // W of one pair, laid out as M
  double2* d_pg = nullptr;            // split partials of A^H W of one pair
  double2* d_pvacc = nullptr;         // the upper triangle of V(k) being accumulated
  std::vector<int> p_split;           // [pairs] splits of the MPB index in A^H W
  // accounting
  double flops_nominal = 0, flops_exec = 0, bytes_alg = 0;
  // learned extrapolator
  NnState* nn = nullptr;
  LearnScratch* ls = nullptr;
};

namespace {

exc_status fail(exc_ctx* c, exc_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) c->err = buf; else g_init_err = buf;
  return st;
}

#define HIPCHK(ctx, call)                                                                       \
  do {                                                                                          \
    hipError_t e_ = (call);                                                                     \
    if (e_ != hipSuccess)                                                                       \
      return fail(ctx, EXC_EHIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, \
                  __LINE__);                                                                    \
  } while (0)

template <class T>
exc_status dalloc(exc_ctx* c, T** p, size_t n) {
  *p = nullptr;
  if (n == 0) n = 1;
  if (hipMalloc((void**)p, n * sizeof(T)) != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();          // a failed allocation must not surface at a later launch check
    return fail(c, EXC_ENOMEM, "device allocation of %zu bytes failed", n * sizeof(T));
  }
  return EXC_OK;
}
#define TRY(x)                      \
  do {                              \
    exc_status s_ = (x);            \
    if (s_ != EXC_OK) return s_;    \
  } while (0)

template <class T>
exc_status upload(exc_ctx* c, T** d, const std::vector<T>& h) {
  TRY(dalloc(c, d, h.size()));
  if (!h.empty()) HIPCHK(c, hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice));
  return EXC_OK;
}

// The block-sparse workspace holds `bytes` (the pairs of one k, or of every k for the
// batched graph). Growing it waits for the device: earlier launches may still use it.
exc_status ensure_ws(exc_ctx* c, size_t bytes) {
  if (c->d_ws && c->ws_cap >= bytes) return EXC_OK;
  if (c->d_ws) {
    HIPCHK(c, hipDeviceSynchronize());
    hipFree(c->d_ws);
    c->d_ws = nullptr;
    c->ws_cap = 0;
  }
  TRY(dalloc(c, (char**)&c->d_ws, bytes));
  c->ws_cap = bytes;
  return EXC_OK;
}

bool capturing(hipStream_t st) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return false;
}

// Buffers that one call at a time may use: the block-sparse workspace (a per-k call keeps its rows at its start, whatever
// the k), those of the unbatched GEMM form, the back-transform's T. A call on another stream than the last one comes after
// it; a context that stays on one stream records no event (3 us a call). A captured call cannot wait for an event from
// outside: its replays must not run beside other calls of the context.
exc_status turn_begin(exc_ctx* c, Turn& t, hipStream_t st) {
  if (capturing(st)) return EXC_OK;
  if (t.used && !t.ev && st != t.st && !capturing(t.st)) {
    HIPCHK(c, hipEventCreateWithFlags(&t.ev, hipEventDisableTiming));
    if (hipEventRecord(t.ev, t.st) != hipSuccess) {    // (that stream is gone)
      (void)hipGetLastError();
      HIPCHK(c, hipDeviceSynchronize());
    }
  }
  if (t.ev) HIPCHK(c, hipStreamWaitEvent(st, t.ev, 0));
  return EXC_OK;
}

exc_status turn_end(exc_ctx* c, Turn& t, hipStream_t st) {
  if (capturing(st)) return EXC_OK;
  t.used = true;
  t.st = st;
  if (t.ev) HIPCHK(c, hipEventRecord(t.ev, st));
  return EXC_OK;
}

// Workspace base for the pairs of k (k < 0: every pair). Pair offsets are global; a
// per-k call keeps only its own pairs' rows, so the base is shifted back by the
// first offset of k (an address the kernels never form below the allocation).
void* ws_base(const exc_ctx* c, int k) {
  if (c->sv) return c->sv->ws;
  if (!c->d_ws) return nullptr;
  if (k < 0) return c->d_ws;
  return (void*)((uintptr_t)c->d_ws - (uintptr_t)c->k_ws_start[k] * c->ws_elem);
}

size_t lds_elem_size(int mode) { return mode == M_F64 ? 8 : (mode == M_F32 ? 4 : 2); }
int npieces(int mode) { return mode == M_BF16X3 ? 2 : (mode == M_BF16X6 ? 3 : 1); }

void free_plan(Plan& p) {
  hipFree(p.d_items); hipFree(p.d_items_lpt); hipFree(p.d_slot_begin); hipFree(p.d_slot_w);
  hipFree(p.d_items_xq); hipFree(p.d_qbeg);
  hipFree(p.d_order);
  p.d_items = p.d_items_lpt = p.d_items_xq = p.d_order = nullptr; p.d_slot_begin = nullptr; p.d_slot_w = nullptr;
  p.d_qbeg = nullptr;
  p.n_slots = 0;
}

void free_chunk_plans(exc_ctx* c) {
  for (auto& kv : c->chunk_plans) { hipFree(kv.second.d_items); hipFree(kv.second.d_base); }
  c->chunk_plans.clear();
  hipFree(c->d_gchunk);
  hipFree(c->d_dchunk);
  c->d_gchunk = nullptr;
  c->d_dchunk = nullptr;
  c->chunk_cap = 0;
  c->chunk_fail = SIZE_MAX;
}

// The contexts' own streams, kept for the next context of the device instead of destroyed: after graph launches (the
// autotuner's, a training run's) the runtime counts their completions off in the stream object for milliseconds after the
// stream, and the device, are idle, and a destroyed stream's memory is then somebody else's. (A counter eight bytes wide,
// stepping down by some tens, in blocks allocated after a context's end; none where the stream lived on or took plain
// launches only.) Never more streams than contexts were alive at once; not freed at exit, where contexts may still end.
struct OwnStreams {
  std::mutex mu;
  std::vector<std::pair<int, hipStream_t>> idle;   // (device, stream)
};
OwnStreams& own_streams() {
  static OwnStreams* s = new OwnStreams;
  return *s;
}

hipError_t take_own(exc_ctx* c) {
  OwnStreams& s = own_streams();
  {
    std::lock_guard<std::mutex> lock(s.mu);
    for (size_t i = s.idle.size(); i-- > 0;) {
      if (s.idle[i].first != c->device) continue;
      hipStream_t st = s.idle[i].second;
      s.idle.erase(s.idle.begin() + i);
      const hipError_t e = hipStreamQuery(st);
      if (e == hipSuccess || e == hipErrorNotReady) {
        c->own = st;
        return hipSuccess;
      }
      (void)hipGetLastError();                     // (the device was reset: its streams are gone)
    }
  }
  return hipStreamCreateWithFlags(&c->own, hipStreamNonBlocking);
}

void give_own(exc_ctx* c) {
  if (!c->own) return;
  OwnStreams& s = own_streams();
  std::lock_guard<std::mutex> lock(s.mu);
  try {
    s.idle.push_back({c->device, c->own});
  } catch (const std::bad_alloc&) {}               // (no room to note it: left as it is)
  c->own = nullptr;
}

void release_timing(exc_ctx* c) {
  for (hipEvent_t e : c->tpool) hipEventDestroy(e);
  c->tpool.clear();
  c->t_slots = c->t_next = c->t_count = 0;
}

void release_learned(exc_ctx* c);

void release(exc_ctx* c) {
  release_learned(c);
  if (c->gexec) hipGraphExecDestroy(c->gexec);
  c->gexec = nullptr;
  if (c->graph) hipGraphDestroy(c->graph);
  c->graph = nullptr;
  release_timing(c);
  if (c->ev_in) hipEventDestroy(c->ev_in);
  if (c->ev_tab) hipEventDestroy(c->ev_tab);
  if (c->ev_chunk) hipEventDestroy(c->ev_chunk);
  if (c->ev_part) hipEventDestroy(c->ev_part);
  free_chunk_plans(c);
  if (c->ev_en) hipEventDestroy(c->ev_en);
  if (c->ev_learn) hipEventDestroy(c->ev_learn);
  for (Turn* t : {&c->turn_ws, &c->turn_bt}) if (t->ev) hipEventDestroy(t->ev);
  c->ev_en = c->ev_learn = c->turn_ws.ev = c->turn_bt.ev = nullptr;
  if (c->ev_out) hipEventDestroy(c->ev_out);
  give_own(c);
  for (hipEvent_t& e : c->ev_g) if (e) hipEventDestroy(e);
  c->ev_g[0] = c->ev_g[1] = nullptr;
  for (hipEvent_t& e : c->ev_bt) if (e) hipEventDestroy(e);
  c->ev_bt[0] = c->ev_bt[1] = nullptr;
  c->ev_in = c->ev_out = c->ev_tab = c->ev_chunk = c->ev_part = nullptr;
  void* ptrs[] = {c->d_coef, c->d_cvec, c->d_schur, c->d_U, c->d_row_chan, c->d_ch_off,
                  c->d_ch_len, c->d_ch_coef, c->d_rowinfo, c->d_runs, c->d_coefpad, c->d_schunk, c->d_sgroup, c->d_units, c->d_ucount, c->d_uowner, c->d_uw, c->d_chunk64, c->d_pairs, c->d_pair_w, c->d_pair_begin,
                  c->d_ws, c->d_dsp, c->d_gpart, c->d_dpart, c->d_vres, c->d_voff, c->d_knb,
                  c->d_mtab, c->d_vtab, c->d_counter, c->d_mstage, c->d_eout, c->d_ewk, c->d_erho,
                  c->d_gamma, c->d_gpartial, c->d_bt, c->d_tmask, c->d_ppairs, c->d_pw, c->d_pg,
                  c->d_pvacc};
  for (void* p : ptrs) if (p) hipFree(p);
  free_plan(c->plain);
  free_plan(c->bat);
  free_plan(c->perk);
  free_plan(c->capt);
}

// Dense rows per row block of a fused or wide instance (its row parts when items are
// split by rows).
int fused_bm(const FusedKCfg& k) { return k.nt == 512 ? 128 * k.RTW : 64 * k.RTW; }

// Fused row parts of a pair: part 0 = the block-sparse rows, part 1 + j = dense row
// block j. An item runs parts [rb0, rb1).
int fused_parts(const exc_ctx* c, const PairInfo& p) {
  const int bm = fused_bm(*c->fcfg);
  return 1 + (p.nd + bm - 1) / bm;
}
// Relative cost of the fused kernel's work on ncols columns of a pair's row part: the
// block-sparse rows and their contraction, or a dense row block's triangular product and
// contraction.
double fused_part_cost(const exc_ctx* c, const PairInfo& p, int ncols, int part) {
  const double nb2 = (double)p.nb8 * p.nb8;
  if (part == 0) return (double)c->n_s * nb2 + 4.0 * c->n_s * ncols;
  const int bm = fused_bm(*c->fcfg), r0 = (part - 1) * bm, rows = std::min(bm, p.nd - r0);
  return (double)rows * nb2 + (double)rows * (p.nd - r0) * ncols;
}

// The fused kernel's chunks of multipole-free rows: whole channels, at most kChunkRows
// rows, multipole rows (n_s + channel) within kChunkMP consecutive rows; {first row, rows,
// longest run, first multipole row}. False if a channel does not fit one chunk or there
// are more than kMaxChunks chunks.
bool sparse_chunks(const exc_ctx* c, const std::vector<int>& row_chan, std::vector<int4>& out) {
  out.clear();
  int r = 0;
  while (r < c->n_s) {
    const int r0 = r, ch0 = row_chan[r];
    int longest = 0;
    while (r < c->n_s) {
      const int ch = row_chan[r], b = c->ch_len[ch];      // r is the first row of channel ch
      if (r - r0 + b > kChunkRows || ch - ch0 >= kChunkMP) break;
      longest = std::max(longest, b);
      r += b;
    }
    if (r == r0) return false;                            // a channel longer than a chunk
    out.push_back(make_int4(r0, r - r0, longest, c->n_s + ch0));
  }
  return (int)out.size() <= kMaxChunks;
}

// herk64_kernel's chunks of multipole-free rows: whole channels within the kernel's limits (rows, multipole
// rows). Empty if a channel alone exceeds them (sparse_kernel then forms the rows).
std::vector<Chunk64> chunks64(const exc_ctx* c, const std::vector<int>& row_chan) {
  std::vector<Chunk64> out;
  int r = 0;
  while (r < c->n_s) {
    const int r0 = r, ch0 = row_chan[r];
    while (r < c->n_s) {
      const int ch = row_chan[r], b = c->ch_len[ch];      // r is the first row of channel ch
      if (r - r0 + b > kH64Rows || ch - ch0 >= kH64MP) break;
      r += b;
    }
    if (r == r0) return {};
    out.push_back(Chunk64{r0, r - r0, c->n_s + ch0, 0});
  }
  // (a chunk costs its 16 rows: with chunks less than half full sparse_kernel's separate pass is the cheaper one)
  if ((int)out.size() * kH64Rows > 2 * c->n_s + 2 * kH64Rows) return {};
  return out;
}

// Relative cost of one row block (for balancing and LPT order).
double block_cost(const exc_ctx* c, const PairInfo& p, int rb, int ncols) {
  const int BM = c->cfg->BM;
  const double contract = (double)BM * p.nb8 * p.nb8;      // Gram tiles
  if (rb < p.nsb) return contract + (double)BM * ncols;
  const int d0 = (rb - p.nsb) * BM;
  const double k = c->form == EXC_FORM_CHOL_HERK ? (double)(p.nd - d0) + c->cfg->KC : (double)p.nd;
  return contract + 2.0 * BM * ncols * k;
}

// Build work items. split_rows: 0 = one item covers all row blocks of the pair
// (n'' chunks looped inside), 1 = one item per (n'' chunk, row block).
exc_status build_plan(exc_ctx* c, Plan& P, int split_rows) {
  P.items.clear();
  P.pair_item.assign(1, 0);
  P.k_item.assign(1, 0);
  P.slot_begin.assign(1, 0);
  P.slot_w.clear();
  const int nct = c->fused ? c->fcfg->NCT : c->cfg->NCT;
  std::vector<double> cost;
  for (int k = 0; k < c->n_k; ++k) {
    for (int pidx = c->k_pair[k]; pidx < c->k_pair[k + 1]; ++pidx) {
      const PairInfo& p = c->pairs[pidx];
      const int nbt = p.nb8 / 8;
      // n'' values per K-loop pass: as many as the column tiles allow, balanced
      // so that the passes of a pair are equally full
      const int ngmax = std::max(1, std::min(c->n_occ, nct / nbt));
      const int npass = (c->n_occ + ngmax - 1) / ngmax;
      const int ngc = (c->n_occ + npass - 1) / npass;
      const int nrb = p.nsb + p.ndb;
      auto push = [&](int g0, int g1, int rb0, int rb1) {
        WorkItem w{};
        w.pair = pidx; w.g0 = g0; w.g1 = g1; w.ngc = ngc; w.rb0 = rb0; w.rb1 = rb1;
        w.slot = (int)P.items.size();
        double cs = 0;
        for (int g = g0; g < g1; g += ngc) {
          if (c->fused) {
            for (int rb = rb0; rb < rb1; ++rb) cs += fused_part_cost(c, p, std::min(ngc, g1 - g) * p.nb8, rb);
            continue;
          }
          for (int rb = rb0; rb < rb1; ++rb) cs += block_cost(c, p, rb, std::min(ngc, g1 - g) * p.nb8);
        }
        P.items.push_back(w);
        P.slot_w.push_back(c->pair_w[pidx]);     // the pair's weight (w_kq, else w_q)
        cost.push_back(cs);
      };
      if (c->fused) {
        // fused items: every row part of the pair (fsplit 0), of one n'' chunk (1), or one
        // row part of one n'' chunk (2: the block-sparse rows, or one dense row block)
        // (one launch per k: items per n'' chunk at least)
        const int nparts = fused_parts(c, p), fs = std::max(c->fsplit, split_rows);
        if (fs == 0) {
          push(0, c->n_occ, 0, nparts);
        } else {
          for (int g = 0; g < c->n_occ; g += ngc) {
            const int g1 = std::min(c->n_occ, g + ngc);
            if (fs == 1) {
              push(g, g1, 0, nparts);
              continue;
            }
            for (int part = c->n_s > 0 ? 0 : 1; part < nparts; ++part) push(g, g1, part, part + 1);
          }
        }
      } else if (!split_rows) {
        push(0, c->n_occ, 0, nrb);
      } else {
        for (int g = 0; g < c->n_occ; g += ngc)
          for (int rb = 0; rb < nrb; ++rb) push(g, std::min(c->n_occ, g + ngc), rb, rb + 1);
      }
      P.pair_item.push_back((int)P.items.size());
    }
    P.k_item.push_back((int)P.items.size());
    P.slot_begin.push_back((int)P.items.size());
  }
  P.n_slots = (int)P.items.size();
  std::vector<WorkItem> lpt(P.items);
  std::vector<int> order(P.items.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
  for (size_t i = 0; i < order.size(); ++i) lpt[i] = P.items[order[i]];
  TRY(upload(c, &P.d_items, P.items));
  TRY(upload(c, &P.d_items_lpt, lpt));
  // XCD queues: the q of the Coulomb factor decides the queue (all k of one q
  // share one factor, kept in that XCD's L2); q are dealt to the queues by
  // decreasing total cost onto the least loaded queue; LPT order inside a queue
  {
    const int nq = NQ_MAX;
    std::vector<double> qcost(c->n_q, 0.0);
    for (size_t i = 0; i < P.items.size(); ++i) qcost[c->pairs[P.items[i].pair].q] += cost[i];
    std::vector<int> qord(c->n_q);
    std::iota(qord.begin(), qord.end(), 0);
    std::stable_sort(qord.begin(), qord.end(), [&](int x, int y) { return qcost[x] > qcost[y]; });
    std::vector<int> qof(c->n_q, 0);
    std::vector<double> load(nq, 0.0);
    for (int q : qord) {
      const int b = (int)(std::min_element(load.begin(), load.end()) - load.begin());
      qof[q] = b;
      load[b] += qcost[q];
    }
    std::vector<WorkItem> xq;
    std::vector<int32_t> qbeg(1, 0);
    for (int b = 0; b < nq; ++b) {
      for (int i : order)
        if (qof[c->pairs[P.items[i].pair].q] == b) xq.push_back(P.items[i]);
      qbeg.push_back((int32_t)xq.size());
    }
    TRY(upload(c, &P.d_items_xq, xq));
    TRY(upload(c, &P.d_qbeg, qbeg));
    P.nq = nq;
  }
  std::vector<int32_t> sb(P.slot_begin.begin(), P.slot_begin.end());
  TRY(upload(c, &P.d_slot_begin, sb));
  TRY(upload(c, &P.d_slot_w, P.slot_w));
  return EXC_OK;
}

// Launch order: the hardware deals workgroup b to XCD b mod 8. Items of one q share its factor, so q are
// dealt to eight lists by decreasing cost, each list in order of decreasing cost, the lists interleaved (and
// padded); where few q leave the lists uneven, one list over all items instead.
void order64(const exc_ctx* c, const std::vector<WorkItem>& it, const std::vector<double>& cost, int i0, int i1,
             std::vector<WorkItem>& out) {
  struct Item { double cost; int i, q; };
  std::vector<Item> ord;
  ord.reserve(i1 - i0);
  for (int i = i0; i < i1; ++i) ord.push_back({cost[i], i, c->pairs[it[i].pair].q});
  auto more = [](const Item& a, const Item& b) { return a.cost > b.cost; };
  if (!std::is_sorted(ord.begin(), ord.end(), more)) std::stable_sort(ord.begin(), ord.end(), more);
  std::vector<double> qc(c->n_q, 0.0), load(8, 0.0);
  for (const Item& x : ord) qc[x.q] += x.cost;
  std::vector<int> qo(c->n_q), qof(c->n_q, 0);
  std::iota(qo.begin(), qo.end(), 0);
  std::stable_sort(qo.begin(), qo.end(), [&](int a, int b) { return qc[a] > qc[b]; });
  double tot = 0.0;
  for (int q : qo) {
    const int b = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    qof[q] = b;
    load[b] += qc[q];
    tot += qc[q];
  }
  if (*std::max_element(load.begin(), load.end()) > 1.06 * tot / 8) {
    for (const Item& x : ord) out.push_back(it[x.i]);
    return;
  }
  size_t len[8] = {}, at[8], n = 0;
  for (const Item& x : ord) n = std::max(n, ++len[qof[x.q]]);
  WorkItem none{};
  none.pair = -1;
  for (int b = 0; b < 8; ++b) at[b] = out.size() + b;
  out.resize(out.size() + 8 * n, none);
  for (const Item& x : ord) {
    size_t& p = at[qof[x.q]];
    out[p] = it[x.i];
    p += 8;
  }
}

// FP64 plan: `per` = 0 every pair in one launch, 1 one launch per k, 2 one launch per pair. At most max_slots items a
// launch and total_slots in all (see pick_split64).
exc_status build_plan64(exc_ctx* c, Plan& P, int per, size_t max_slots, size_t total_slots) {
  int n_cu = 256;
  (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, c->device);
  P.items.clear();
  P.pair_item.assign(1, 0);
  P.k_item.assign(1, 0);
  P.slot_begin.assign(1, 0);
  P.slot_w.clear();
  P.order_begin.assign(1, 0);
  // the split is chosen for all pairs, the k with the most pairs, or the largest pair
  std::vector<std::vector<int>> nd;
  int at = 0;
  if (per == 0) nd.resize(1);
  for (int k = 0; k < c->n_k; ++k) {
    if (per == 1) nd.push_back({});
    for (int i = c->k_pair[k]; i < c->k_pair[k + 1]; ++i) {
      if (per == 2) nd.push_back({});
      nd.back().push_back(c->pairs[i].nd);
      if (per == 2 && nd.back()[0] > nd[at][0]) at = i;
    }
    if (per == 1 && nd.back().size() > nd[at].size()) at = k;
  }
  const System64 sys{c->n_occ, c->n_s, c->n_chunk64, n_cu, (size_t)c->gstride * 8};
  std::vector<Shape64> shapes;
  for (const Herk64K& k : kHerk64) shapes.push_back(k.shape);
  Split64 sp;
  if (const char* ev = getenv("EXC_HERK64")) {           // a fixed instance and split (tests): id,passes,groups
    int id = 0, passes = 1, groups = 1;
    if (sscanf(ev, "%d,%d,%d", &id, &passes, &groups) == 3 && passes >= 0 && groups >= 0)
      for (int i = 0; i < kNumHerk64; ++i)
        if (kHerk64[i].id() == id && kHerk64[i].shape.nbt == c->nbt_max) sp = Split64{i, passes, groups};
  }
  if (sp.inst < 0) sp = pick_split64(sys, shapes, c->nbt_max, nd, at, max_slots, total_slots);
  if (sp.inst < 0) return fail(c, EXC_EUNSUPPORTED, "no FP64 kernel for n_b = %d", c->nb_max);
  P.h64 = &kHerk64[sp.inst];
  const Shape64& sh = P.h64->shape;
  const int npass = (c->n_occ + sh.ng - 1) / sh.ng, step = sp.passes ? sp.passes : npass;
  struct Run { int part0, part1; double cost; };
  std::vector<Run> runs;
  std::vector<double> cost;
  std::vector<WorkItem> order;
  const size_t most = c->pairs.size() * ((npass + step - 1) / step) *
                      (sp.groups ? sp.groups : 1 + (*std::max_element(c->nd.begin(), c->nd.end()) + 63) / 64);
  P.items.reserve(most);
  P.slot_w.reserve(most);
  cost.reserve(most);
  order.reserve(most);
  for (int k = 0; k < c->n_k; ++k) {
    for (int i = c->k_pair[k]; i < c->k_pair[k + 1]; ++i) {
      runs.clear();
      runs64(sys, sh, sp.groups, c->pairs[i].nd, [&](int r0, int r1, double cs) { runs.push_back({r0, r1, cs}); });
      for (int g = 0; g < npass; g += step)
        for (const Run& r : runs) {
          const int n = std::min(step, npass - g);
          WorkItem w{};
          w.pair = i; w.g0 = g * sh.ng; w.g1 = std::min(c->n_occ, (g + n) * sh.ng); w.ngc = sh.ng; w.rb0 = r.part0; w.rb1 = r.part1;
          w.slot = (int)P.items.size();
          P.items.push_back(w);
          P.slot_w.push_back(c->pair_w[i]);
          cost.push_back(r.cost * n);
        }
      P.pair_item.push_back((int)P.items.size());
      if (per == 2) {
        for (int j = P.pair_item[i]; j < P.pair_item[i + 1]; ++j) order.push_back(P.items[j]);
        P.order_begin.push_back((int)order.size());
      }
    }
    P.k_item.push_back((int)P.items.size());
    P.slot_begin.push_back((int)P.items.size());
    if (per == 1) {
      // (as a rule every k has the same q: the order of the k before it)
      const int p0 = c->k_pair[k], np = c->k_pair[k + 1] - p0, ni = P.k_item[k + 1] - P.k_item[k];
      bool same = k > 0 && p0 - c->k_pair[k - 1] == np;
      for (int i = p0; same && i < p0 + np; ++i) same = c->pairs[i].q == c->pairs[i - np].q;
      if (same) {
        for (int j = P.order_begin[k - 1]; j < P.order_begin[k]; ++j) {
          WorkItem w = order[j];
          if (w.pair >= 0) { w.pair += np; w.slot += ni; }
          order.push_back(w);
        }
      } else {
        order64(c, P.items, cost, P.k_item[k], P.k_item[k + 1], order);
      }
      P.order_begin.push_back((int)order.size());
    }
  }
  if (per == 0) {
    order64(c, P.items, cost, 0, (int)P.items.size(), order);
    P.order_begin.push_back((int)order.size());
  }
  P.n_slots = (int)P.items.size();
  TRY(upload(c, &P.d_order, order));
  TRY(upload(c, &P.d_slot_begin, std::vector<int32_t>(P.slot_begin.begin(), P.slot_begin.end())));
  TRY(upload(c, &P.d_slot_w, P.slot_w));
  return EXC_OK;
}

// Real-factor instances serve only contexts with a real factor; there they are
// preferred over the general ones of the same capacity. dtype: the element type of M
// (-1: not known yet -- instances that read complex64 only are left out).
bool fused_fits(const FusedKCfg& k, int mode, int nbt_max, bool real, int dtype) {
  return k.mode == mode && k.NB8M >= nbt_max && k.NCT >= nbt_max && (real || !k.realf) &&
         (!k.c64only || (dtype == EXC_C64 && !real));
}

const FusedKCfg* pick_fused(int mode, int nbt_max, bool real, int dtype = -1) {
  const FusedKCfg* best = nullptr;
  if (const char* ev = getenv("EXC_FUSED_CFG")) {      // a fixed configuration id (tuning runs)
    const int id = atoi(ev);
    for (const auto& k : all_fused())
      if (k.id == id && fused_fits(k, mode, nbt_max, real, k.c64only && dtype < 0 ? EXC_C64 : dtype))
        return &k;                                      // (at set-up the M type is not known yet)
  }
  for (const auto& k : all_fused()) {
    if (!fused_fits(k, mode, nbt_max, real, dtype) || k.c64only) continue;
    if (!best || k.NB8M < best->NB8M || (k.NB8M == best->NB8M && k.realf && !best->realf)) best = &k;
  }
  return best;
}

const KernelCfg* pick_cfg(int mode, int form, int nbt_max) {
  const KernelCfg* best = nullptr;
  for (const auto& k : kCfgs) {
    if (k.mode != mode || k.form != form || k.NB8M < nbt_max || k.NCT < nbt_max) continue;
    if (!best || k.NB8M < best->NB8M) best = &k;
  }
  return best;
}

// Writes n pointers to one or two device tables, in the order of st.
exc_status put_pointers(exc_ctx* c, int n, void** dst0, const void* const* src0, void** dst1, const void* const* src1,
                        hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += kPtrTab) {
    PtrTab t{};
    t.n = std::min(kPtrTab, n - i0);
    t.dst[0] = dst0 + i0;
    t.dst[1] = dst1 ? dst1 + i0 : nullptr;
    for (int i = 0; i < t.n; ++i) {
      t.p[0][i] = const_cast<void*>(src0[i0 + i]);
      t.p[1][i] = dst1 ? const_cast<void*>(src1[i0 + i]) : nullptr;
    }
    hipLaunchKernelGGL(put_pointers_kernel, dim3(1), dim3(2 * kPtrTab), 0, st, t);
  }
  HIPCHK(c, hipGetLastError());
  return EXC_OK;
}

exc_status set_tables(exc_ctx* c, int k0, int nk, const void* const* M, void* const* V,
                      hipStream_t st) {
  bool changed = false;
  for (int i = 0; i < nk; ++i)
    if (c->h_mtab[k0 + i] != M[i] || c->h_vtab[k0 + i] != V[i]) changed = true;
  const bool cap = (changed || c->tab_pending) && capturing(st);
  // the tables may have been written on another stream: after that (a call finds the pointers that it passes
  // there, whichever call wrote them)
  if (c->tab_pending && !cap) {
    if (hipEventQuery(c->ev_tab) == hipSuccess) c->tab_pending = false;
    else {
      (void)hipGetLastError();                       // (not ready is not an error)
      HIPCHK(c, hipStreamWaitEvent(st, c->ev_tab, 0));
    }
  } else if (c->tab_pending) {                       // (an event from outside cannot be part of a capture)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    HIPCHK(c, hipThreadExchangeStreamCaptureMode(&mode));
    const hipError_t e = hipEventSynchronize(c->ev_tab);
    HIPCHK(c, hipThreadExchangeStreamCaptureMode(&mode));
    HIPCHK(c, e);
    c->tab_pending = false;
  }
  if (!changed) return EXC_OK;
  // (a captured call would write the tables at replay only: refused, by the wait below)
  if (cap) HIPCHK(c, hipStreamSynchronize(st));
  for (int i = 0; i < nk; ++i) {
    c->h_mtab[k0 + i] = const_cast<void*>(M[i]);
    c->h_vtab[k0 + i] = V[i];
  }
  TRY(put_pointers(c, nk, c->d_mtab + k0, M, c->d_vtab + k0, (const void* const*)V, st));
  HIPCHK(c, hipEventRecord(c->ev_tab, st));
  c->tab_pending = true;
  return EXC_OK;
}

TileArgs tile_args(exc_ctx* c, int dtype, int k) {
  TileArgs a{};
  a.pairs = c->d_pairs;
  a.mtab = (const void* const*)c->d_mtab;
  a.m_c64 = dtype == EXC_C64;
  a.n_s = c->n_s;
  a.n_ch = c->n_ch;
  a.ns_pad = c->ns_pad;
  a.U = c->d_U;
  a.ws = ws_base(c, k);
  a.dsp = c->sv ? c->sv->dsp : c->d_dsp;
  a.dsp_stride = c->n_occ * c->nb_max;
  a.gpart = c->sv ? c->sv->gpart : c->d_gpart;
  a.dpart = c->sv ? c->sv->dpart : c->d_dpart;
  a.gstride = c->gstride;
  a.tmask = c->d_tmask;
  a.dstride = c->dstride;
  return a;
}

SparseArgs sparse_args(exc_ctx* c, int dtype, int k) {
  SparseArgs s{};
  s.pairs = c->d_pairs;
  s.mtab = (const void* const*)c->d_mtab;
  s.m_c64 = dtype == EXC_C64;
  s.n_s = c->n_s; s.n_ch = c->n_ch; s.n_occ = c->n_occ; s.nb_max = c->nb_max; s.ns_pad = c->ns_pad;
  s.row_chan = c->d_row_chan; s.ch_off = c->d_ch_off; s.ch_len = c->d_ch_len;
  s.ch_coef = c->d_ch_coef; s.coef = c->d_coef; s.cvec = c->d_cvec; s.rowinfo = c->d_rowinfo;
  s.runs = c->d_runs; s.run_max = c->run_max; s.runs_ld = c->runs_ld;
  s.runs_qs = c->nqc > 1 ? (int64_t)c->run_max * c->runs_ld : 0;
  s.coef_qs = c->nqc > 1 ? c->coef_total : 0;
  s.cvec_qs = c->nqc > 1 ? c->n_s : 0;
  s.ws = ws_base(c, k); s.dsp = c->sv ? c->sv->dsp : c->d_dsp;
  return s;
}

FusedArgs fused_args(exc_ctx* c, int dtype) {
  FusedArgs f{};
  f.pairs = c->d_pairs;
  f.mtab = (const void* const*)c->d_mtab;
  f.m_c64 = dtype == EXC_C64;
  f.n_s = c->n_s; f.n_ch = c->n_ch; f.n_occ = c->n_occ;
  f.U = c->d_U;
  f.row_chan = c->d_row_chan; f.ch_off = c->d_ch_off; f.ch_len = c->d_ch_len; f.ch_coef = c->d_ch_coef;
  f.coef = c->d_coef; f.cvec = c->d_cvec; f.rowinfo = c->d_rowinfo; f.coefpad = c->d_coefpad;
  f.schunk = c->d_schunk; f.n_schunk = c->n_schunk; f.sgroup = c->d_sgroup;
  f.rows = c->row_units;
  f.coef_qs = c->nqc > 1 ? c->coef_total : 0;
  f.cvec_qs = c->nqc > 1 ? c->n_s : 0;
  f.pad_qs = c->nqc > 1 ? (int64_t)std::max(1, c->n_schunk) * kChunkRows * kRunPad : 0;
  f.gpart = c->sv ? c->sv->gpart : c->d_gpart;
  f.dpart = c->sv ? c->sv->dpart : c->d_dpart;
  f.gstride = c->gstride; f.dstride = c->dstride;
  f.tmask = c->d_tmask;
  return f;
}

// Argument storage of the main kernel launch (tile or fused kernel).
struct MainArgs {
  TileArgs t;
  FusedArgs f;
  Herk64Args h;
};

// A configured kernel launch: enqueued directly or added to a graph as a node.
struct KLaunch {
  const void* fn = nullptr;
  dim3 grid, block{256, 1, 1};
  size_t shmem = 0;
  void* arg = nullptr;          // points at the single by-value argument struct
};

hipError_t enqueue(const KLaunch& L, hipStream_t st) {
  void* args[1] = {L.arg};
  return hipLaunchKernel(L.fn, L.grid, L.block, args, L.shmem, st);
}

hipError_t add_node(hipGraph_t g, const KLaunch& L, hipGraphNode_t* dep, hipGraphNode_t* out) {
  void* args[1] = {L.arg};
  hipKernelNodeParams p{};
  p.func = const_cast<void*>(L.fn);
  p.gridDim = L.grid;
  p.blockDim = L.block;
  p.kernelParams = args;
  p.sharedMemBytes = (unsigned)L.shmem;
  p.extra = nullptr;
  return hipGraphAddKernelNode(out, g, dep, dep ? 1 : 0, &p);
}

// sparse_kernel: HERK form, one wavefront per workgroup taking c->sncw columns (set once by
// pick_sparse_ncw); GEMM form, four wavefronts of one column each.
bool sparse_herk(const exc_ctx* c) { return c->form == EXC_FORM_CHOL_HERK; }
int sparse_ncw(const exc_ctx* c) { return sparse_herk(c) ? c->sncw : 1; }
// As many columns (1, 2 or 4) as keep the workgroup's LDS within 24 KiB: at least six
// workgroups per CU. EXC_SPARSE_NCW=1|2|4 fixes the count (fixed-configuration runs).
int pick_sparse_ncw(const exc_ctx* c) {
  const size_t col = (size_t)((c->n_s + c->n_ch + 63) / 64 * 64) * sizeof(double2);
  if (const char* ev = getenv("EXC_SPARSE_NCW")) {
    const int n = atoi(ev);
    if ((n == 1 || n == 2 || n == 4) && n * col <= 160 * 1024) return n;
  }
  return 4 * col <= 24576 ? 4 : (2 * col <= 24576 ? 2 : 1);
}
size_t sparse_lds_bytes(const exc_ctx* c) {
  if (!sparse_herk(c)) return (size_t)4 * (c->n_s + c->n_ch) * sizeof(double2);
  return (size_t)sparse_ncw(c) * ((c->n_s + c->n_ch + 63) / 64 * 64) * sizeof(double2);
}

template <int MODE>
const void* sparse_herk_fn(int ncw) {
  return ncw == 4 ? (const void*)sparse_kernel<1, MODE, 4>
                  : (ncw == 2 ? (const void*)sparse_kernel<1, MODE, 2> : (const void*)sparse_kernel<1, MODE, 1>);
}
const void* sparse_fn(const exc_ctx* c) {
  if (c->form != EXC_FORM_CHOL_HERK) return (const void*)sparse_kernel<0, M_F64>;
  const int ncw = sparse_ncw(c);
  switch (c->precision) {
    case EXC_FP64: return sparse_herk_fn<M_F64>(ncw);
    case EXC_FP32: return sparse_herk_fn<M_F32>(ncw);
    case EXC_BF16X3: return sparse_herk_fn<M_BF16X3>(ncw);
    default: return sparse_herk_fn<M_BF16X6>(ncw);
  }
}

// herk64_kernel forms the block-sparse rows itself.
bool fused64(const exc_ctx* c) { return c->h64 && c->n_chunk64 > 0; }
// The call needs the block-sparse workspace.
bool needs_ws(const exc_ctx* c) { return !c->fused && !fused64(c); }

// The call uses turn_ws's buffers.
bool shares(const exc_ctx* c) {
  if (c->plain_gemm) return true;
  const bool packs = c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64;   // (as in cfg_sparse)
  return needs_ws(c) && (packs || c->n_s > 0 || (c->form != EXC_FORM_CHOL_HERK && c->n_ch > 0));
}

// Block-sparse rows of pairs [pair0, pair0 + npairs), all of k (k < 0: every pair). Returns
// false when there is nothing to do.
bool cfg_sparse(exc_ctx* c, int dtype, int k, int pair0, int npairs, SparseArgs& s, KLaunch& L) {
  if (c->fused || fused64(c)) return false;   // the main kernel does the block-sparse rows itself
  const bool packs = c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64;   // packs the dense rows too
  if (!packs && c->n_s == 0 && (c->form == EXC_FORM_CHOL_HERK || c->n_ch == 0)) return false;
  s = sparse_args(c, dtype, k);
  s.pairs = c->d_pairs + pair0;
  // dsp is indexed by blockIdx.y: offset it to the first pair
  s.dsp = s.dsp ? s.dsp + (long)pair0 * c->n_occ * c->nb_max : nullptr;
  const int ncol = c->n_occ * c->nb_max;
  const int ncw = sparse_ncw(c);
  L.grid = sparse_herk(c) ? dim3((ncol + ncw - 1) / ncw, npairs) : dim3((ncol + 3) / 4, npairs);
  L.block = dim3(sparse_herk(c) ? 64 : 256);
  L.shmem = sparse_lds_bytes(c);
  L.fn = sparse_fn(c);
  L.arg = &s;
  return true;
}

void cfg_reduce(exc_ctx* c, const Plan& P, int k0, int nk, ReduceArgs& r, KLaunch& L) {
  r = ReduceArgs{};
  r.k_nb = c->d_knb + k0;
  r.slot_begin = P.d_slot_begin + k0;
  r.slot_w = P.d_slot_w;
  r.gpart = c->sv ? c->sv->gpart : c->d_gpart;
  r.gstride = c->gstride;
  r.acc64 = c->precision == EXC_FP64;
  r.dpart = c->sv ? c->sv->dpart : c->d_dpart;
  r.dstride = c->dstride;
  r.use_d64 = c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64;
  r.vres = c->d_vres;
  r.v_off = c->d_voff + k0;
  r.vout = c->d_vtab + k0;
  r.gshift = c->d_gamma + 3;
  r.n_occ = c->n_occ_v;
  r.real_v = c->real_v ? 1 : 0;
  L.grid = dim3(c->nbt_max * (c->nbt_max + 1) / 2, nk);
  L.block = dim3(64 * RED_SG);
  L.shmem = 0;
  L.fn = r.acc64 ? (const void*)reduce_kernel<1> : (const void*)reduce_kernel<0>;
  if (c->h64) {                                  // (no work counters to clear: one workgroup per item)
    L.grid.x *= 4;
    L.block = dim3(1024);
    L.fn = (const void*)reduce64_kernel;
  }
  L.arg = &r;
}

// Launch i of an FP64 plan: its part of the launch order.
void launch64(exc_ctx* c, const Plan& P, int i, int dtype, int k, Herk64Args& a, KLaunch& L) {
  a = Herk64Args{};
  a.pairs = c->d_pairs;
  a.items = P.d_order + P.order_begin[i];
  a.n_items = P.order_begin[i + 1] - P.order_begin[i];
  a.mtab = (const void* const*)c->d_mtab;
  a.n_s = c->n_s;
  a.n_occ = c->n_occ;
  a.U = (const double*)c->d_U;
  if (fused64(c)) {
    a.chunks = c->d_chunk64;
    a.n_chunk = c->n_chunk64;
    a.rowinfo = c->d_rowinfo;
    a.coef = c->d_coef;
    a.cvec = c->d_cvec;
    a.coef_qs = c->nqc > 1 ? c->coef_total : 0;
    a.cvec_qs = c->nqc > 1 ? c->n_s : 0;
  } else {
    a.ws = (const double2*)ws_base(c, k);
  }
  a.gpart = c->sv ? (double*)c->sv->gpart : (double*)c->d_gpart;
  a.gstride = c->gstride;
  a.tmask = c->d_tmask;
  L.grid = dim3(a.n_items);
  L.block = dim3(64 * P.h64->shape.nw);
  L.shmem = 0;
  L.fn = dtype == EXC_C64 ? (const void*)P.h64->fn64 : (const void*)P.h64->fn;
  L.arg = &a;
}

// The plan of one launch per k, and k's launch in it.
const Plan& k_plan(const exc_ctx* c) { return c->h64 && c->n_k > 1 ? c->perk : c->bat; }

void cfg_tile(exc_ctx* c, int dtype, int k, const WorkItem* items, int n, bool persistent, MainArgs& m,
              KLaunch& L) {
  if (c->h64) return launch64(c, c->bat, 0, dtype, k, m.h, L);    // (every pair at once)
  L.grid = dim3(persistent ? std::min(n, c->persist_grid) : n);
  L.shmem = 0;
  if (c->fused) {
    FusedArgs& f = m.f;
    f = fused_args(c, dtype);
    f.items = persistent ? c->bat.d_items_xq : items;
    f.n_items = n;
    f.counter = persistent ? c->d_counter : nullptr;
    f.qbeg = c->bat.d_qbeg;
    f.nq = c->bat.nq;
    L.block = dim3(c->fcfg->nt);
    L.fn = (const void*)c->fcfg->fn;
    L.arg = &f;
    return;
  }
  TileArgs& a = m.t;
  a = tile_args(c, dtype, k);
  a.items = items;
  a.n_items = n;
  a.counter = persistent ? c->d_counter : nullptr;
  L.block = dim3(64 * c->cfg->NW());
  L.fn = (const void*)c->cfg->fn;
  L.arg = &a;
}

void launch_sparse(exc_ctx* c, int dtype, int k, int pair0, int npairs, hipStream_t st) {
  SparseArgs s;
  KLaunch L;
  if (cfg_sparse(c, dtype, k, pair0, npairs, s, L)) (void)enqueue(L, st);
}

void launch_reduce(exc_ctx* c, const Plan& P, int k0, int nk, hipStream_t st) {
  ReduceArgs r;
  KLaunch L;
  cfg_reduce(c, P, k0, nk, r, L);
  (void)enqueue(L, st);
}

void launch_tile(exc_ctx* c, int dtype, int k, const WorkItem* items, int n, hipStream_t st) {
  if (n <= 0) return;
  MainArgs a;
  KLaunch L;
  cfg_tile(c, dtype, k, items, n, false, a, L);
  (void)enqueue(L, st);
}

// The main kernel of one k on plan P (k_plan).
void launch_k(exc_ctx* c, const Plan& P, int dtype, int k, hipStream_t st) {
  if (!c->h64) return launch_tile(c, dtype, k, P.d_items + P.k_item[k], P.k_item[k + 1] - P.k_item[k], st);
  Herk64Args a;
  KLaunch L;
  launch64(c, P, k, dtype, k, a, L);
  (void)enqueue(L, st);
}

// One item per pair leaves workgroup slots of the GPU empty when a k has few pairs, and a fused instance that streams
// its Gram tiles (its binary32 chain runs through the whole pair) cannot be given less than a pair per item without
// other roundings. Items per n'' chunk and row part that keep every chunk of 64 rows in a slot of its own, added up in
// the chain's order afterwards, give the same bits from a full GPU: the first V(k) of the ZnO-like workload (144 pairs
// of 18 n'', bf16x3) 13.4 -> 4.1 ms. The slots are written and read once (12 MB a pair there); batches of pairs keep
// them within chunk_bytes, about the size of the memory-side cache. A plan without batches: not for this k.
exc_status chunk_plan(exc_ctx* c, int k, ChunkPlan** out) {
  *out = nullptr;
  const FusedKCfg* f = c->fcfg;
  if (!c->fused || f->gchain != 1 || f->c64only || c->fsplit != 0) return EXC_OK;
  const int p0 = c->k_pair[k], p1 = c->k_pair[k + 1];
  auto found = c->chunk_plans.find(k);
  if (found == c->chunk_plans.end()) {
    int n_cu = 256;
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, c->device);
    ChunkPlan P;
    std::vector<WorkItem> items;
    std::vector<int32_t> base;
    // two workgroups of an instance within half the LDS share a CU
    const bool few = p1 - p0 < n_cu * (f->lds <= 81920 ? 2 : 1);
    const int n_sc = c->n_s > 0 ? c->n_schunk : 0;
    const size_t slot_b = (size_t)c->gstride * 4 + (size_t)64 * f->NCT * 8;
    size_t slots = 0;                                  // of the batch so far
    int pb = p0;
    std::vector<std::pair<double, WorkItem>> bi;       // its items, with their costs
    auto flush = [&](int pe) {
      if (pe == pb) return;
      std::stable_sort(bi.begin(), bi.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
      P.batches.push_back({(int)items.size(), (int)bi.size(), pb, pe - pb});
      for (const auto& x : bi) items.push_back(x.second);
      P.slots = std::max(P.slots, slots);
      bi.clear();
      slots = 0;
      pb = pe;
    };
    for (int i = p0; i < p1 && few; ++i) {
      const PairInfo& p = c->pairs[i];
      const int nbt = p.nb8 / 8, ngmax = std::max(1, std::min(c->n_occ, f->NCT / nbt));
      P.npass = (c->n_occ + ngmax - 1) / ngmax;
      const int ngc = (c->n_occ + P.npass - 1) / P.npass, cpp = n_sc + (p.nd + 63) / 64;
      const size_t need = (size_t)P.npass * cpp;
      if (need * slot_b > c->chunk_bytes) { P = ChunkPlan{}; items.clear(); break; }
      if ((slots + need) * slot_b > c->chunk_bytes) flush(i);
      base.push_back((int32_t)slots);
      const int nparts = fused_parts(c, p);
      for (int g = 0; g < P.npass; ++g) {
        const int g0 = g * ngc, g1 = std::min(c->n_occ, g0 + ngc);
        for (int part = n_sc ? 0 : 1; part < nparts; ++part) {
          WorkItem w{};
          w.pair = i; w.g0 = g0; w.g1 = g1; w.ngc = ngc; w.rb0 = part; w.rb1 = part + 1;
          w.slot = (int)(slots + (size_t)g * cpp + (part ? n_sc + (part - 1) * f->RTW : 0));
          bi.push_back({fused_part_cost(c, p, (g1 - g0) * p.nb8, part), w});
        }
      }
      slots += need;
      if (i + 1 == p1) flush(p1);
    }
    // (nothing to split: the merge would only come on top, one pair of 20 rows and 64 bands in bf16x3 22.7 -> 24.6 us)
    if (items.size() == (size_t)(p1 - p0)) P = ChunkPlan{};
    if (!P.batches.empty()) {
      exc_status s = upload(c, &P.d_items, items);
      if (s == EXC_OK) s = upload(c, &P.d_base, base);
      if (s != EXC_OK) {
        hipFree(P.d_items);
        hipFree(P.d_base);
        if (s != EXC_ENOMEM) return s;
        ++c->chunk_fails;
        c->err.clear();
        P = ChunkPlan{};
      }
    }
    found = c->chunk_plans.emplace(k, P).first;
  }
  ChunkPlan& P = found->second;
  if (P.batches.empty()) return EXC_OK;
  if (P.slots >= c->chunk_fail) return EXC_OK;         // (there was no room: not asked for again)
  if (P.slots > c->chunk_cap) {
    float* g = nullptr;
    double* d = nullptr;
    exc_status s = dalloc(c, &g, P.slots * c->gstride);
    if (s == EXC_OK) s = dalloc(c, &d, P.slots * (size_t)64 * f->NCT);
    if (s != EXC_OK) {
      hipFree(g);
      if (s != EXC_ENOMEM) return s;
      ++c->chunk_fails;
      c->chunk_fail = P.slots;
      c->err.clear();
      return EXC_OK;
    }
    if (c->chunk_cap) HIPCHK(c, hipDeviceSynchronize());   // earlier calls still use the smaller ones
    hipFree(c->d_gchunk);
    hipFree(c->d_dchunk);
    c->d_gchunk = g;
    c->d_dchunk = d;
    c->chunk_cap = P.slots;
  }
  if (!c->ev_chunk) HIPCHK(c, hipEventCreateWithFlags(&c->ev_chunk, hipEventDisableTiming));
  *out = &P;
  return EXC_OK;
}

// The partial slots of k's pairs (those of plan `plan`) through their chunks; the slots of the chunks are shared by
// every call of the context, whatever its stream.
exc_status launch_chunks(exc_ctx* c, const ChunkPlan& P, const Plan& plan, int dtype, int k, hipStream_t st) {
  HIPCHK(c, hipStreamWaitEvent(st, c->ev_chunk, 0));
  for (const ChunkPlan::Batch& b : P.batches) {
    MainArgs a;
    KLaunch L;
    cfg_tile(c, dtype, k, P.d_items + b.item0, b.items, false, a, L);
    a.f.gpart = c->d_gchunk;
    a.f.dpart = c->d_dchunk;
    a.f.dstride = 64 * c->fcfg->NCT;
    a.f.by_chunk = 1;
    (void)enqueue(L, st);
    const int slot = plan.slot_begin[k] + b.pair0 - c->k_pair[k];
    MergeArgs m{};
    m.pairs = c->d_pairs + b.pair0;
    m.base = P.d_base + (b.pair0 - c->k_pair[k]);
    m.chunk = c->d_gchunk;
    m.dchunk = c->d_dchunk;
    m.gstride = c->gstride; m.dstride = c->dstride; m.ncc = 8 * c->fcfg->NCT;
    m.npass = P.npass;
    m.n_sc = c->n_s > 0 ? c->n_schunk : 0;
    m.gpart = (float*)c->d_gpart + (long)slot * c->gstride;
    m.dpart = c->d_dpart + (long)slot * c->dstride;
    m.tmask = c->d_tmask;
    hipLaunchKernelGGL(merge_chunks_kernel, dim3(c->nbt_max * (c->nbt_max + 1) / 2 + 1, b.pairs), dim3(256), 0, st, m);
  }
  HIPCHK(c, hipEventRecord(c->ev_chunk, st));
  return EXC_OK;
}

// One k, batched over its q: sparse rows of all pairs of k, one tile launch, reduce.
exc_status run_k_batched(exc_ctx* c, int k, int dtype, hipStream_t st) {
  if (needs_ws(c)) TRY(ensure_ws(c, c->ws_k_bytes));
  const int p0 = c->k_pair[k], p1 = c->k_pair[k + 1];
  if (c->part_shared) {                              // (FP64) this call's slots
    const bool cap = capturing(st);
    const Plan& P = cap ? c->capt : c->perk;
    const size_t slot_b = (size_t)c->gstride * 8;
    ScratchView v{};
    v.ws = ws_base(c, k);
    v.gpart = (void*)((uintptr_t)c->d_gpart + (cap ? c->part_slots * slot_b : -(uintptr_t)P.slot_begin[k] * slot_b));
    v.dpart = c->d_dpart;
    if (!cap) HIPCHK(c, hipStreamWaitEvent(st, c->ev_part, 0));
    c->sv = &v;
    launch_sparse(c, dtype, k, p0, p1 - p0, st);
    launch_k(c, P, dtype, k, st);
    launch_reduce(c, P, k, 1, st);
    c->sv = nullptr;
    if (!cap) HIPCHK(c, hipEventRecord(c->ev_part, st));
    return EXC_OK;
  }
  launch_sparse(c, dtype, k, p0, p1 - p0, st);
  const Plan& P = k_plan(c);
  ChunkPlan* cp = nullptr;
  c->chunk_batches = 0;
  // (no room for the chunks: one item per pair; a captured call keeps to that too, as its replays may run beside
  // other calls of the context)
  if (c->fused && !capturing(st)) {
    try {
      TRY(chunk_plan(c, k, &cp));
    } catch (const std::bad_alloc&) {              // (host memory for the plan: no exception leaves the library)
      cp = nullptr;
    }
  }
  if (cp) c->chunk_batches = (int)cp->batches.size();
  if (cp) TRY(launch_chunks(c, *cp, P, dtype, k, st));
  else launch_k(c, P, dtype, k, st);
  launch_reduce(c, P, k, 1, st);
  return EXC_OK;
}

// One k, plain form: one launch of each kernel per (k, q) pair.
exc_status run_k_plain(exc_ctx* c, int k, int dtype, hipStream_t st) {
  if (needs_ws(c)) TRY(ensure_ws(c, c->ws_k_bytes));
  const Plan& P = c->plain;
  for (int p = c->k_pair[k]; p < c->k_pair[k + 1]; ++p) {
    launch_sparse(c, dtype, k, p, 1, st);
    if (c->h64) {
      Herk64Args a;
      KLaunch L;
      launch64(c, P, p, dtype, k, a, L);
      (void)enqueue(L, st);
      continue;
    }
    launch_tile(c, dtype, k, P.d_items + P.pair_item[p], P.pair_item[p + 1] - P.pair_item[p], st);
  }
  launch_reduce(c, P, k, 1, st);
  return EXC_OK;
}

// Plain GEMM form, one k: per (k, q) pair the block-sparse rows of W = v A
// (sparse_kernel<0>), the dense rows W_d = E A_d + X (zgemm_kernel), the band
// contraction G_b = A_b^H W_b split over the MPB index (zgemm_kernel) and its FP64
// accumulation into V(k); then V(k) with its mirror. One launch of each kernel per pair.
constexpr int PG_BM = 64, PG_BNC = 64, PG_KC = 16;
exc_status run_k_plain_gemm(exc_ctx* c, int k, int dtype, hipStream_t st) {
  const bool c64 = dtype == EXC_C64;
  const size_t esz = c64 ? 8 : 16;
  const char* Mk = (const char*)c->h_mtab[k];
  for (int p = c->k_pair[k]; p < c->k_pair[k + 1]; ++p) {
    const PairInfo& pi = c->pairs[p];
    const int ncol = c->n_occ * pi.nb;
    // block-sparse rows of W and X = C_c^H A_c into the multipole rows
    if (c->n_s > 0 || c->n_ch > 0) {
      SparseArgs sa = sparse_args(c, dtype, -1);
      sa.pairs = c->d_ppairs + p;
      sa.ws = c->d_pw;
      sa.dsp = nullptr;
      hipLaunchKernelGGL((sparse_kernel<0, M_F64>), dim3((ncol + 3) / 4, 1), dim3(256), sparse_lds_bytes(c), st, sa);
    }
    if (pi.nd > 0) {
      ZgemmArgs z{};
      z.a = (const double*)c->d_U + pi.u_off;
      z.lda = pi.ldu; z.a_plane = (int64_t)pi.ldu * pi.ldu; z.a_kind = 0; z.a_rows_alloc = pi.ldu;
      z.b = Mk + (pi.m_off + c->n_s) * esz; z.ldb = pi.nmb; z.b_c64 = c64;
      z.c = c->d_pw + c->n_s; z.ldc = pi.nmb;
      z.M = pi.nd; z.N = ncol; z.K = pi.nd; z.kchunk = (pi.nd + PG_KC - 1) / PG_KC * PG_KC;
      z.add_rows = c->n_ch;
      const int tiles = ((pi.nd + PG_BM - 1) / PG_BM) * ((ncol + PG_BNC - 1) / PG_BNC);
      hipLaunchKernelGGL((zgemm_kernel<PG_BM, PG_BNC, PG_KC, 2>), dim3(tiles, 1, 1), dim3(256), 0, st, z);
    }
    {
      ZgemmArgs z{};
      z.a = Mk + pi.m_off * esz; z.lda = pi.nmb; z.a_bstride = (int64_t)pi.nb * pi.nmb; z.a_kind = 1;
      z.a_c64 = c64; z.a_conj = 1;
      z.b = c->d_pw; z.ldb = pi.nmb; z.b_bstride = (int64_t)pi.nb * pi.nmb;
      z.c = c->d_pg; z.ldc = pi.nb; z.c_bstride = (int64_t)pi.nb * pi.nb;
      z.c_sstride = (int64_t)c->n_occ * pi.nb * pi.nb;
      z.M = z.N = pi.nb; z.K = pi.nmb; z.upper = 1;
      const int ns = c->p_split[p];
      z.kchunk = ((pi.nmb + ns - 1) / ns + PG_KC - 1) / PG_KC * PG_KC;
      const int nt = (pi.nb + PG_BM - 1) / PG_BM;
      hipLaunchKernelGGL((zgemm_kernel<PG_BM, PG_BNC, PG_KC, 2>), dim3(nt * nt, c->n_occ, ns), dim3(256), 0, st, z);
      hipLaunchKernelGGL(pair_accumulate_kernel, dim3((pi.nb * pi.nb + 255) / 256), dim3(256), 0, st,
                         (const double2*)c->d_pg, ns, c->n_occ, pi.nb, c->pair_w[p], (int)(p == c->k_pair[k]),
                         c->d_pvacc);
    }
  }
  const int nb = c->nb[k];
  hipLaunchKernelGGL(pair_finish_kernel, dim3((nb * nb + 255) / 256), dim3(256), 0, st, (const double2*)c->d_pvacc,
                     nb, c->n_occ_v, (const double*)(c->d_gamma + 3), (int)c->real_v,
                     (const uint64_t*)(c->d_tmask + 3 * k), c->d_vres + c->v_off[k], (double2*)c->h_vtab[k]);
  return EXC_OK;
}

// The kernels of the batched path launched one by one on st, in the graph's order, with the
// timing events recorded on st (the default: the graph's launch leaves a longer gap before
// its first kernel, 6-8 us more per step on the Si-like workload; EXC_GRAPH=1 uses the graph).
exc_status launch_batched_direct(exc_ctx* c, int dtype, hipStream_t st) {
  if (needs_ws(c)) TRY(ensure_ws(c, c->ws_bytes));
  const bool timed = c->t_slots > 0;
  const int s = c->t_next;
  SparseArgs sa;
  KLaunch L;
  c->t_sparse = false;
  if (cfg_sparse(c, dtype, -1, 0, (int)c->pairs.size(), sa, L)) {
    if (timed) HIPCHK(c, hipEventRecord(c->tpool[3 * s], st));
    HIPCHK(c, enqueue(L, st));
    c->t_sparse = true;
  }
  if (timed) HIPCHK(c, hipEventRecord(c->tpool[3 * s + 1], st));
  MainArgs ta;
  cfg_tile(c, dtype, -1, c->bat.d_items_lpt, c->bat.n_slots, true, ta, L);
  HIPCHK(c, enqueue(L, st));
  if (timed) HIPCHK(c, hipEventRecord(c->tpool[3 * s + 2], st));
  ReduceArgs ra;
  cfg_reduce(c, c->bat, 0, c->n_k, ra, L);
  ra.counter = c->d_counter;
  ra.n_counter = NQ_MAX;
  HIPCHK(c, enqueue(L, st));
  if (timed) {
    c->t_next = (s + 1) % c->t_slots;
    c->t_count = std::min(c->t_count + 1, c->t_slots);
  }
  return EXC_OK;
}

// The batched path as an explicit graph:
//   [ev0] -> block-sparse rows -> [ev1] -> persistent tile (or fused) kernel ->
//   [ev2] -> FP64 reduction, which also clears the persistent kernel's work
//   counters for the next replay (they start at zero from init).
// The event-record nodes exist only while kernel timing is on; their events are
// swapped per replay (hipGraphExecEventRecordNodeSetEvent).
exc_status build_batched_graph(exc_ctx* c, int dtype) {
  if (needs_ws(c)) TRY(ensure_ws(c, c->ws_bytes));   // every pair's block-sparse rows at once
  hipGraph_t g = nullptr;
  HIPCHK(c, hipGraphCreate(&g, 0));
  const bool timed = c->t_slots > 0;
  for (auto& t : c->tnode) t = nullptr;
  hipGraphNode_t last = nullptr, node = nullptr;
  hipError_t e = hipSuccess;
  auto add_ev = [&](int i) -> hipError_t {
    if (!timed || e != hipSuccess) return e;
    hipGraphNode_t n2 = nullptr;
    hipError_t r = hipGraphAddEventRecordNode(&n2, g, last ? &last : nullptr, last ? 1 : 0, c->tpool[i]);
    if (r == hipSuccess) { c->tnode[i] = n2; last = n2; }
    return r;
  };
  SparseArgs sa;
  KLaunch L;
  if (e == hipSuccess && cfg_sparse(c, dtype, -1, 0, (int)c->pairs.size(), sa, L)) {
    e = add_ev(0);                      // (the fused path has no block-sparse kernel to time)
    if (e == hipSuccess) e = add_node(g, L, last ? &last : nullptr, &node);
    last = node;
  }
  e = add_ev(1);
  MainArgs ta;
  if (e == hipSuccess) {
    cfg_tile(c, dtype, -1, c->bat.d_items_lpt, c->bat.n_slots, true, ta, L);
    e = add_node(g, L, last ? &last : nullptr, &node);
    last = node;
  }
  e = add_ev(2);
  ReduceArgs ra;
  if (e == hipSuccess) {
    cfg_reduce(c, c->bat, 0, c->n_k, ra, L);
    ra.counter = c->d_counter;
    ra.n_counter = NQ_MAX;
    e = add_node(g, L, &last, &node);
  }
  const char* where = e == hipSuccess ? "instantiate" : "add node";
  if (e == hipSuccess) e = hipGraphInstantiate(&c->gexec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    hipGraphDestroy(g);
    c->gexec = nullptr;
    return fail(c, EXC_EHIP, "building the batched graph failed (%s): %s", where, hipGetErrorString(e));
  }
  if (c->graph) hipGraphDestroy(c->graph);
  c->graph = g;
  c->g_dtype = dtype;
  return EXC_OK;
}

// FP64: the most partial slots per k with which every k that the no-allocation call's scratch could hold
// with one slot per pair still fits it (0: no such k, no limit).
size_t noalloc_slots(const exc_ctx* c) {
  size_t most = 0;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  for (int k = 0; k < c->n_k; ++k) {
    const size_t np = c->k_pair[k + 1] - c->k_pair[k];
    const size_t ws = up((size_t)(c->k_ws_start[k + 1] - c->k_ws_start[k]) * c->ws_elem);
    const size_t slot = ((size_t)c->gstride + c->dstride) * 8;
    if (ws + np * slot + 512 > kScratchBytes) continue;
    const size_t n = std::max(np, (kScratchBytes - ws - 512) / slot);
    most = most ? std::min(most, n) : n;
  }
  return most;
}

// FP64 HERK: the plans of the context's path; `coarse`: one item per pair.
//
// A launch of one k is split finely enough to fill the GPU by itself. With slots of its own for every k, calls on
// different streams do not meet, but over many k the slots add up: 20 k of 216 SrTiO3-like pairs to 16 GB where one item
// per pair takes 0.8 GB. Past kPartialBytes all k use the same slots and their calls follow each other; captured calls,
// whose replays nothing orders, then keep to one item per pair in slots of their own. (Coarser items for every k instead:
// 64 k of the ZnO-like system within 4 GiB 11.8 ms a k, with shared slots 6.5.) One launch per pair: past kPartialBytes no
// more slots than items of one 64-row block and up to 12 (8) band tiles of n'' take.
constexpr size_t kPartialBytes = (size_t)2 << 30;
exc_status build_plans64(exc_ctx* c, bool coarse) {
  free_plan(c->plain);
  free_plan(c->bat);
  free_plan(c->perk);
  free_plan(c->capt);
  c->part_shared = false;
  if (!c->batched) {
    const int nbt = c->nbt_max, ng = std::max(1, nbt <= 3 ? 12 / nbt : 8 / nbt);
    size_t total = 0, room = kPartialBytes / ((size_t)c->gstride * 8);
    for (const PairInfo& p : c->pairs) total += (size_t)((c->n_occ + ng - 1) / ng) * (p.nsb + p.ndb);
    return build_plan64(c, c->plain, 2, coarse ? 1 : 0, std::max(total, room));
  }
  const size_t lim = coarse ? 1 : noalloc_slots(c);
  TRY(build_plan64(c, c->bat, 0, c->n_k == 1 || coarse ? lim : 0, 0));
  if (c->n_k == 1) return EXC_OK;
  TRY(build_plan64(c, c->perk, 1, lim, 0));
  if (coarse || (size_t)c->perk.n_slots * c->gstride * 8 <= kPartialBytes) return EXC_OK;
  c->part_shared = true;
  c->part_slots = 0;
  for (int k = 0; k < c->n_k; ++k)
    c->part_slots = std::max(c->part_slots, (size_t)(c->perk.slot_begin[k + 1] - c->perk.slot_begin[k]));
  if (!c->ev_part) HIPCHK(c, hipEventCreateWithFlags(&c->ev_part, hipEventDisableTiming));
  return build_plan64(c, c->capt, 1, 1, 0);
}

// The partial slots of the context's plans.
exc_status alloc_partials(exc_ctx* c) {
  const size_t perk = c->part_shared ? c->part_slots + c->capt.n_slots : c->perk.n_slots;
  const size_t nslot = std::max({(size_t)c->plain.n_slots, (size_t)c->bat.n_slots, perk});
  const size_t asz = c->precision == EXC_FP64 ? 8 : 4;
  hipFree(c->d_gpart);
  hipFree(c->d_dpart);
  c->d_gpart = nullptr;
  c->d_dpart = nullptr;
  TRY(dalloc(c, (char**)&c->d_gpart, nslot * c->gstride * asz));
  TRY(dalloc(c, &c->d_dpart, nslot * (size_t)c->dstride));
  HIPCHK(c, hipMemset(c->d_gpart, 0, nslot * c->gstride * asz));
  HIPCHK(c, hipMemset(c->d_dpart, 0, nslot * (size_t)c->dstride * 8));
  return EXC_OK;
}

// Switch the context to a main-kernel configuration: a fused instance, or
// (f == nullptr) the block-sparse + tile kernels. Rebuilds the plans, sizes
// the partial slots and the persistent grid, allocates or releases the
// block-sparse workspace, and drops the captured graph.
exc_status configure(exc_ctx* c, const FusedKCfg* f, hipStream_t st) {
  const bool mixed_herk = c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64;
  c->fcfg = f;
  c->fused = f != nullptr;
  if (c->gexec) { hipGraphExecDestroy(c->gexec); c->gexec = nullptr; }
  HIPCHK(c, hipStreamSynchronize(st));
  if (c->own) HIPCHK(c, hipStreamSynchronize(c->own));
  // the block-sparse workspace itself is sized at first use: the pairs of one k for
  // per-k calls, every pair for the batched graph
  const bool need_ws = !c->fused;
  if (!need_ws && c->d_ws) { hipFree(c->d_ws); c->d_ws = nullptr; c->ws_cap = 0; }
  if (need_ws && mixed_herk && !c->d_dsp) {
    const size_t n = c->pairs.size() * (size_t)c->n_occ * c->nb_max;
    TRY(dalloc(c, &c->d_dsp, n));
    HIPCHK(c, hipMemset(c->d_dsp, 0, n * sizeof(double)));
  }
  if (!need_ws && c->d_dsp) { hipFree(c->d_dsp); c->d_dsp = nullptr; }
  // only the plan of the context's path: one item per pair (or n'' chunk) for the batched
  // path, one per (n'' chunk, row block) for one launch per pair
  free_chunk_plans(c);
  if (c->h64) {                                   // (one workgroup per item: no persistent grid)
    TRY(build_plans64(c, false));
    const exc_status s = alloc_partials(c);
    if (s != EXC_ENOMEM) return s;
    c->err.clear();                               // (no room for the finer items' partials)
    TRY(build_plans64(c, true));
    return alloc_partials(c);
  }
  free_plan(c->plain);
  free_plan(c->bat);
  if (c->batched) TRY(build_plan(c, c->bat, 0));
  else TRY(build_plan(c, c->plain, 1));
  TRY(alloc_partials(c));
  const void* main_fn = c->fused ? (const void*)c->fcfg->fn : (const void*)c->cfg->fn;
  const int main_threads = c->fused ? c->fcfg->nt : 64 * c->cfg->NW();
  hipFuncAttributes fa{};
  HIPCHK(c, hipFuncGetAttributes(&fa, main_fn));
  if (fa.maxThreadsPerBlock < main_threads)
    return fail(c, EXC_EUNSUPPORTED, "kernel %d allows %d threads per block, needs %d",
                c->fused ? c->fcfg->id : c->cfg->id, fa.maxThreadsPerBlock, main_threads);
  int n_cu = 0, occ = 0;
  HIPCHK(c, hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, c->device));
  HIPCHK(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, main_fn, main_threads, 0));
  c->persist_grid = std::max(1, n_cu * std::max(1, occ));
  return EXC_OK;
}

// ---------------------------------------------------------------------------
// Autotuner of the batched path: on the first batched call of a reduced-
// precision HERK context, every main-kernel configuration that can serve it
// (the fused instances with enough band tiles, and the block-sparse + tile
// kernels) runs the caller's own inputs once untimed and five times timed on
// the context's stream; the fastest is kept (a candidate later in the order of
// preference must beat the earlier best by more than 3 %, so that timing noise
// between equal configurations does not flip the choice). With EXC_TUNE_CACHE=<file> the
// choice is looked up / recorded under a key of the problem's size bucket.
// EXC_TUNE=0 keeps the default configuration.
// ---------------------------------------------------------------------------
std::string tune_key(const exc_ctx* c, int dtype) {
  long nmb = 0, nbs = 0;
  for (int q = 0; q < c->n_q; ++q) nmb += c->nmb[q];
  for (int k = 0; k < c->n_k; ++k) nbs += c->nb[k];
  char buf[256];
  snprintf(buf, sizeof buf, "v1 prec=%d form=%d dtype=%d nk=%d nq=%d nocc=%d nbt=%d nmb_avg=%ld nb_avg=%ld ns=%d pairs=%d%s",
           c->precision, c->form, dtype, c->n_k, c->n_q, c->n_occ, c->nbt_max, nmb / std::max(1, c->n_q),
           nbs / std::max(1, c->n_k), c->n_s, (int)c->pairs.size(), c->real_v ? " real" : "");
  return buf;
}

int cfg_id(const exc_ctx* c) { return c->fused ? c->fcfg->id : c->cfg->id; }

exc_status autotune(exc_ctx* c, int dtype, hipStream_t st) {
  c->tuned = 0;
  // candidates: (fused instance, one work item per n'' chunk instead of per pair), in
  // order of preference; the split items come last: they pay when few pairs leave the
  // CUs short of work
  std::vector<std::pair<const FusedKCfg*, int>> cands;
  if (c->fused_ok)
    for (const auto& k : all_fused())
      if (fused_fits(k, c->precision, c->nbt_max, c->real_v, dtype)) cands.push_back({&k, 0});
  cands.push_back({nullptr, 0});                 // block-sparse + tile kernels
  // items per n'' chunk only where the pairs alone leave the CUs short of work
  int n_cu = 256;
  (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, c->device);
  if (c->fused_ok && c->n_occ > 1 && (int)c->pairs.size() < 8 * n_cu)
    for (const auto& k : all_fused())
      if (fused_fits(k, c->precision, c->nbt_max, c->real_v, dtype) &&
          std::min(c->n_occ, k.NCT / c->nbt_max) < c->n_occ) cands.push_back({&k, 1});
  // items per n'' chunk and row part where even those leave the CUs short of work
  if (c->fused_ok && (long)c->pairs.size() * c->n_occ < 4L * n_cu)
    for (const auto& k : all_fused())
      if (fused_fits(k, c->precision, c->nbt_max, c->real_v, dtype)) cands.push_back({&k, 2});
  const std::string key = tune_key(c, dtype);
  const char* cache = getenv("EXC_TUNE_CACHE");
  if (cache) {
    if (FILE* fp = fopen(cache, "r")) {
      char line[512];
      int found = -1;
      while (fgets(line, sizeof line, fp)) {
        char* tab = strchr(line, '\t');
        if (!tab) continue;
        *tab = 0;
        if (key == line) found = atoi(tab + 1);
      }
      fclose(fp);
      for (const auto& cd : cands) {
        const int id = (cd.first ? cd.first->id : c->cfg->id) + 10000 * cd.second;
        if (id == found) {
          c->fsplit = cd.second;
          TRY(configure(c, cd.first, st));
          c->tuned = 2;
          return EXC_OK;
        }
      }
    }
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIPCHK(c, hipEventCreate(&e0));
  HIPCHK(c, hipEventCreate(&e1));
  const FusedKCfg* best = c->fcfg;
  int best_split = 0;
  float best_ms = 1e30f;
  bool any = false;
  for (const auto& cd : cands) {
    const FusedKCfg* f = cd.first;
    c->fsplit = cd.second;
    exc_status s2 = configure(c, f, st);
    if (s2 == EXC_ENOMEM) { c->err.clear(); continue; }   // e.g. no room for the block-sparse workspace
    if (s2 != EXC_OK) { hipEventDestroy(e0); hipEventDestroy(e1); return s2; }
    if ((s2 = build_batched_graph(c, dtype)) == EXC_ENOMEM) { c->err.clear(); continue; }   // workspace too large
    if (s2 != EXC_OK) { hipEventDestroy(e0); hipEventDestroy(e1); return s2; }
    // one untimed run, then one timed: a candidate more than twice as slow as the best so
    // far is dropped there; the others are timed over five more runs
    HIPCHK(c, hipGraphLaunch(c->gexec, c->own));
    HIPCHK(c, hipEventRecord(e0, c->own));
    HIPCHK(c, hipGraphLaunch(c->gexec, c->own));
    HIPCHK(c, hipEventRecord(e1, c->own));
    HIPCHK(c, hipEventSynchronize(e1));
    float ms = 0.f;
    HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
    if (any && ms > 2.0f * best_ms) continue;
    HIPCHK(c, hipEventRecord(e0, c->own));
    for (int r = 0; r < 5; ++r) HIPCHK(c, hipGraphLaunch(c->gexec, c->own));
    HIPCHK(c, hipEventRecord(e1, c->own));
    HIPCHK(c, hipEventSynchronize(e1));
    HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
    ms /= 5.0f;
    // candidates come in order of preference: a later one must be clearly faster
    if (!any || ms < 0.97f * best_ms) { best_ms = ms; best = f; best_split = cd.second; any = true; }
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  if (!any) return fail(c, EXC_ENOMEM, "no main-kernel configuration fits in device memory");
  c->fsplit = best_split;
  TRY(configure(c, best, st));
  c->tuned = 1;
  if (cache) {
    if (FILE* fp = fopen(cache, "a")) {
      fprintf(fp, "%s\t%d\n", key.c_str(), cfg_id(c) + 10000 * c->fsplit);
      fclose(fp);
    }
  }
  return EXC_OK;
}

// The wide kernel reads complex64 M only: a call with complex128 M switches the context
// to the best instance for it (which drops the captured graph).
exc_status fit_dtype(exc_ctx* c, int dtype, hipStream_t st) {
  if (!c->fused || !c->fcfg->c64only || dtype == EXC_C64) return EXC_OK;
  c->fsplit = 0;
  return configure(c, pick_fused(c->precision, c->nbt_max, c->real_v, dtype), st);
}

// The device address of this GPU's scratch array (once per device, with it current).
exc_status scratch_setup(exc_ctx* c) {
  if (c->device < 0 || c->device >= kScratchDevices)
    return fail(c, EXC_EUNSUPPORTED, "device %d beyond the %d the library keeps scratch for", c->device,
                kScratchDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[c->device]) return EXC_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p)
    return fail(c, EXC_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
  g_scratch_ptr[c->device] = p;
  return EXC_OK;
}

exc_status check_ctx(const exc_ctx* c) {
  if (!c) return EXC_EINVAL;
  if (c->magic != kAlive) return EXC_ESTATE;
  return EXC_OK;
}

}  // namespace

// ============================================================================
// C ABI
// ============================================================================
extern "C" {

exc_status exchange_init(const exc_desc* d, const exc_coulomb* cv, void* stream, exc_ctx** out) {
  if (!out) return fail(nullptr, EXC_EINVAL, "out is NULL");
  *out = nullptr;
  if (!d || !cv) return fail(nullptr, EXC_EINVAL, "desc or coulomb is NULL");
  if (d->n_k < 1 || d->n_q < 1 || d->n_occ < 1 || d->n_channels < 0)
    return fail(nullptr, EXC_EINVAL, "n_k, n_q, n_occ must be >= 1 and n_channels >= 0");
  if (!d->n_bands || !d->n_pw || (d->n_channels > 0 && !d->ch_nrad))
    return fail(nullptr, EXC_EINVAL, "n_bands, n_pw or ch_nrad is NULL");
  if (d->precision < EXC_FP64 || d->precision > EXC_BF16X6)
    return fail(nullptr, EXC_EINVAL, "bad precision %d", d->precision);
  if (d->form != EXC_FORM_GEMM && d->form != EXC_FORM_CHOL_HERK)
    return fail(nullptr, EXC_EINVAL, "bad form %d", d->form);
  if (d->form == EXC_FORM_GEMM && d->precision != EXC_FP64)
    return fail(nullptr, EXC_EUNSUPPORTED, "the GEMM form runs in FP64 only");
  if (d->inversion != 0 && d->inversion != 1) return fail(nullptr, EXC_EINVAL, "inversion must be 0 or 1");
  if (!cv->E) return fail(nullptr, EXC_EINVAL, "coulomb.E is NULL");
  for (int k = 0; k < d->n_k; ++k)
    if (d->n_bands[k] < 1 || d->n_bands[k] > 128)
      return fail(nullptr, d->n_bands[k] < 1 ? EXC_EINVAL : EXC_EUNSUPPORTED,
                  "n_bands[%d] = %d outside [1, 128]", k, d->n_bands[k]);
  for (int q = 0; q < d->n_q; ++q) {
    if (d->n_pw[q] < 0) return fail(nullptr, EXC_EINVAL, "n_pw[%d] < 0", q);
    if (d->n_channels + d->n_pw[q] < 1)          // no basis function at q: nothing to contract
      return fail(nullptr, EXC_EINVAL, "the mixed basis of q = %d is empty (no channels, no plane waves)", q);
  }
  for (int c = 0; c < d->n_channels; ++c)
    if (d->ch_nrad[c] < 1) return fail(nullptr, EXC_EINVAL, "ch_nrad[%d] < 1", c);
  if (d->w_q)
    for (int q = 0; q < d->n_q; ++q)
      if (!std::isfinite(d->w_q[q])) return fail(nullptr, EXC_EINVAL, "w_q[%d] not finite", q);
  if (d->w_kq)
    for (long i = 0; i < (long)d->n_k * d->n_q; ++i)
      if (!std::isfinite(d->w_kq[i])) return fail(nullptr, EXC_EINVAL, "w_kq[%ld] not finite", i);

  exc_ctx* c = new (std::nothrow) exc_ctx();
  if (!c) return fail(nullptr, EXC_ENOMEM, "host allocation failed");
  auto bail = [&](exc_status st) {
    g_init_err = c->err;
    release(c);
    c->magic = 0;
    delete c;
    return st;
  };
#define ITRY(x)                       \
  do {                                \
    exc_status s_ = (x);              \
    if (s_ != EXC_OK) return bail(s_); \
  } while (0)
#define IHIP(call)                                                                          \
  do {                                                                                      \
    hipError_t e_ = (call);                                                                 \
    if (e_ != hipSuccess) {                                                                 \
      fail(c, EXC_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));                     \
      return bail(EXC_EHIP);                                                                \
    }                                                                                       \
  } while (0)

  c->n_k = d->n_k; c->n_q = d->n_q; c->n_occ = d->n_occ; c->n_ch = d->n_channels;
  c->n_occ_v = d->n_occ;
  c->real_v = d->inversion != 0;
  if (c->real_v) c->n_occ = (d->n_occ + 1) / 2;
  c->precision = d->precision; c->form = d->form; c->batched = d->batched; c->device = d->device;
  c->nb.assign(d->n_bands, d->n_bands + d->n_k);
  c->npw.assign(d->n_pw, d->n_pw + d->n_q);
  if (c->n_ch) c->nrad.assign(d->ch_nrad, d->ch_nrad + c->n_ch);
  c->wq.resize(c->n_q);
  for (int q = 0; q < c->n_q; ++q) c->wq[q] = d->w_q ? d->w_q[q] : 1.0 / c->n_q;
  c->has_wkq = d->w_kq != nullptr;
  c->wkq.resize((size_t)c->n_k * c->n_q);
  for (int k = 0; k < c->n_k; ++k)
    for (int q = 0; q < c->n_q; ++q)
      c->wkq[(size_t)k * c->n_q + q] = d->w_kq ? d->w_kq[(size_t)k * c->n_q + q] : c->wq[q];

  IHIP(hipSetDevice(c->device));
  ITRY(scratch_setup(c));
  hipStream_t st = (hipStream_t)stream;
  c->last_stream = st;

  // ---- channel layout (sparse rows) ----
  c->ch_off.resize(c->n_ch); c->ch_len.resize(c->n_ch); c->ch_coef.resize(c->n_ch);
  std::vector<int32_t> row_chan;
  for (int ch = 0; ch < c->n_ch; ++ch) {
    c->ch_off[ch] = c->n_s;
    c->ch_len[ch] = c->nrad[ch] - 1;
    c->ch_coef[ch] = c->coef_total;
    c->coef_total += (int64_t)c->ch_len[ch] * c->ch_len[ch];
    for (int i = 0; i < c->ch_len[ch]; ++i) row_chan.push_back(ch);
    c->n_s += c->ch_len[ch];
  }
  c->nb_max = *std::max_element(c->nb.begin(), c->nb.end());
  c->nbt_max = (c->nb_max + 7) / 8;
  // the unbatched GEMM form runs one pair at a time through its own kernels (any band count)
  c->plain_gemm = c->form == EXC_FORM_GEMM && !c->batched;
  c->h64 = c->precision == EXC_FP64 && c->form == EXC_FORM_CHOL_HERK;
  c->cfg = c->h64 ? nullptr : pick_cfg(c->precision, c->form, c->nbt_max);
  if (!c->cfg && !c->plain_gemm && !c->h64) {
    fail(c, EXC_EUNSUPPORTED, "no tile configuration for n_b = %d%s", c->nb_max,
         c->form == EXC_FORM_GEMM ? " (the batched GEMM form takes at most 64 bands)" : "");
    return bail(EXC_EUNSUPPORTED);
  }
  if (c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64) {
    const char* ev = getenv("EXC_FUSED");
    c->fcfg = pick_fused(c->precision, c->nbt_max, c->real_v);
    c->fused_ok = c->fcfg && sparse_chunks(c, row_chan, c->h_schunk);
    if (!c->fused_ok) c->h_schunk.clear();
    c->fused = c->fused_ok && !(ev && ev[0] == '0');
    if (!c->fused) c->fcfg = nullptr;
  }
  const int BM = c->cfg ? c->cfg->BM : 64;

  c->nd.resize(c->n_q); c->nmb.resize(c->n_q); c->ldu.resize(c->n_q); c->u_off.resize(c->n_q);
  const int npl = 2 * npieces(c->precision);
  int64_t u_total = 0;
  for (int q = 0; q < c->n_q; ++q) {
    c->nd[q] = c->n_ch + c->npw[q];
    c->nmb[q] = c->n_s + c->nd[q];
    c->ldu[q] = std::max(128, (c->nd[q] + 127) / 128 * 128);
    c->u_off[q] = u_total;
    u_total += (int64_t)npl * c->ldu[q] * c->ldu[q];
  }

  // ---- Coulomb blocks to the device ----
  {
    const hipMemcpyKind kind = cv->on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    // channel blocks: one copy when every q points at the same D and C, else one per q
    if (c->n_s) {
      if (!cv->D || !cv->C) { fail(c, EXC_EINVAL, "coulomb.D or coulomb.C is NULL"); return bail(EXC_EINVAL); }
      bool alias = true;
      for (int q = 0; q < c->n_q; ++q) {
        if (!cv->D[q] || !cv->C[q]) { fail(c, EXC_EINVAL, "coulomb.D[%d] or coulomb.C[%d] is NULL", q, q); return bail(EXC_EINVAL); }
        alias = alias && cv->D[q] == cv->D[0] && cv->C[q] == cv->C[0];
      }
      c->nqc = alias ? 1 : c->n_q;
    }
    ITRY(dalloc(c, &c->d_coef, (size_t)c->coef_total * c->nqc));
    ITRY(dalloc(c, &c->d_cvec, (size_t)c->n_s * c->nqc));
    for (int i = 0; i < c->nqc && c->n_s; ++i) {
      if (c->coef_total) IHIP(hipMemcpy(c->d_coef + (size_t)i * c->coef_total, cv->D[i], c->coef_total * 16, kind));
      IHIP(hipMemcpy(c->d_cvec + (size_t)i * c->n_s, cv->C[i], (size_t)c->n_s * 16, kind));
    }
    if (c->real_v) {                  // only the real parts of v are read
      if (c->coef_total) IHIP(hipMemset2D((char*)c->d_coef + 8, 16, 0, 8, (size_t)c->coef_total * c->nqc));
      if (c->n_s) IHIP(hipMemset2D((char*)c->d_cvec + 8, 16, 0, 8, (size_t)c->n_s * c->nqc));
    }
    ITRY(upload(c, &c->d_row_chan, row_chan));
    {
      // per multipole-free row r (entry i of channel ch, b = ch_len): the coefficient
      // run L_c[i..b-1][i] starts at column-major index i*b + i of the channel's block
      std::vector<int4> ri(std::max(1, c->n_s));
      for (int r = 0; r < c->n_s; ++r) {
        const int ch = row_chan[r], i = r - c->ch_off[ch], b = c->ch_len[ch];
        ri[r] = make_int4((int)(c->ch_coef[ch] + (int64_t)i * b + i), b - i, c->n_s + ch, 0);
      }
      ITRY(upload(c, &c->d_rowinfo, ri));
      // (EXC_FUSED=0: the block-sparse rows in a kernel of their own, as in the other modes)
      const char* ev = getenv("EXC_FUSED");
      if (c->h64 && c->n_s > 0 && !(ev && ev[0] == '0')) {
        const std::vector<Chunk64> ck64 = chunks64(c, row_chan);
        c->n_chunk64 = (int)ck64.size();
        if (c->n_chunk64) ITRY(upload(c, &c->d_chunk64, ck64));
      }
      if (c->form == EXC_FORM_CHOL_HERK && c->n_s > 0) {
        c->run_max = *std::max_element(c->ch_len.begin(), c->ch_len.end());
        c->runs_ld = (c->n_s + 7) / 8 * 8;
        ITRY(dalloc(c, &c->d_runs, (size_t)c->run_max * c->runs_ld * c->nqc));
      }
      std::vector<int4> ck = c->h_schunk;
      c->n_schunk = (int)ck.size();
      if (c->n_schunk) {
        // each chunk's groups of 16 rows: units of eight rows of M from the group's first row to the end of its last
        // channel, then of its channels' multipole rows
        std::vector<RowUnit> units;
        std::vector<int2> owner;
        std::vector<int32_t> count;
        RowUnits& R = c->row_units;
        for (int t = 0; t < 4; ++t) {
          R.begin[t] = (int)units.size();
          for (const int4& x : ck) {
            const size_t at = units.size();
            const int r0 = x.x + 16 * t, n = std::min(16, x.y - 16 * t);
            auto add = [&](int row, int end) {
              for (; row < end; row += 8) {
                units.push_back({row, std::min(8, end - row)});
                owner.push_back(make_int2(r0, n));
              }
            };
            if (n > 0) {
              const int ch0 = row_chan[r0], ch1 = row_chan[r0 + n - 1];
              add(r0, (int)c->ch_off[ch1] + (int)c->ch_len[ch1]);
              add(c->n_s + ch0, c->n_s + ch1 + 1);
              while ((units.size() - at) % kUnitRing) {
                units.push_back({0, 0});
                owner.push_back(make_int2(r0, n));
              }
            }
            count.push_back((int)(units.size() - at));
          }
        }
        ITRY(upload(c, &c->d_units, units));
        ITRY(upload(c, &c->d_uowner, owner));
        ITRY(upload(c, &c->d_ucount, count));
        ITRY(dalloc(c, &c->d_uw, units.size() * 128 * c->nqc));
        R.units = c->d_units;
        R.count = c->d_ucount;
        R.n_chunk = c->n_schunk;
        R.n_units = (int)units.size();
        R.w = c->d_uw;
        R.w_qs = c->nqc > 1 ? (int64_t)units.size() * 128 : 0;
      }
      if (ck.empty()) ck.push_back(make_int4(0, 0, 0, 0));
      ITRY(upload(c, &c->d_schunk, ck));
      // row groups of each chunk: its kChunkRows rows (those past the chunk with run length 0)
      // by decreasing run length, four at a time, {rows (one byte each), longest run}
      std::vector<uint2> grp((size_t)ck.size() * (kChunkRows / 4));
      for (size_t k = 0; k < ck.size(); ++k) {
        std::vector<int> rows(kChunkRows), len(kChunkRows, 0);
        for (int r = 0; r < kChunkRows; ++r) {
          rows[r] = r;
          if (r < ck[k].y) len[r] = ri[ck[k].x + r].y;
        }
        std::stable_sort(rows.begin(), rows.end(), [&](int x, int y) { return len[x] > len[y]; });
        for (int g = 0; g < kChunkRows / 4; ++g) {
          uint32_t packed = 0;
          for (int e = 0; e < 4; ++e) packed |= (uint32_t)rows[4 * g + e] << (8 * e);
          grp[k * (kChunkRows / 4) + g] = make_uint2(packed, (uint32_t)len[rows[4 * g]]);
        }
      }
      ITRY(upload(c, &c->d_sgroup, grp));
      ITRY(dalloc(c, &c->d_coefpad, (size_t)ck.size() * kChunkRows * kRunPad * c->nqc));
    }
    ITRY(upload(c, &c->d_ch_off, std::vector<int32_t>(c->ch_off.begin(), c->ch_off.end())));
    ITRY(upload(c, &c->d_ch_len, std::vector<int32_t>(c->ch_len.begin(), c->ch_len.end())));
    ITRY(upload(c, &c->d_ch_coef, c->ch_coef));
    ITRY(dalloc(c, &c->d_schur, (size_t)std::max(1, c->n_ch) * c->nqc));

    // dense blocks: a column-major workspace per q (factored in place for HERK)
    std::vector<int64_t> e_off(c->n_q);
    std::vector<int32_t> e_ld(c->n_q), nd32(c->nd.begin(), c->nd.end()), ldu32(c->ldu.begin(), c->ldu.end());
    int64_t e_total = 0;
    for (int q = 0; q < c->n_q; ++q) { e_off[q] = e_total; e_ld[q] = std::max(1, c->nd[q]); e_total += (int64_t)c->nd[q] * c->nd[q]; }
    double2* d_E = nullptr;
    int64_t *d_eoff = nullptr, *d_uoff = nullptr;
    int32_t *d_nd = nullptr, *d_eld = nullptr, *d_ldu = nullptr;
    int* d_info = nullptr;
    auto cleanup = [&]() { hipFree(d_E); hipFree(d_eoff); hipFree(d_uoff); hipFree(d_nd); hipFree(d_eld); hipFree(d_ldu); hipFree(d_info); };
    exc_status s = dalloc(c, &d_E, (size_t)e_total);
    if (s != EXC_OK) { cleanup(); return bail(s); }
    for (int q = 0; q < c->n_q; ++q) {
      if (!cv->E[q] && c->nd[q] > 0) { cleanup(); fail(c, EXC_EINVAL, "coulomb.E[%d] is NULL", q); return bail(EXC_EINVAL); }
      if (c->nd[q] > 0) {
        hipError_t e = hipMemcpy(d_E + e_off[q], cv->E[q], (size_t)c->nd[q] * c->nd[q] * 16, kind);
        if (e == hipSuccess && c->real_v)
          e = hipMemset2D((char*)(d_E + e_off[q]) + 8, 16, 0, 8, (size_t)c->nd[q] * c->nd[q]);
        if (e != hipSuccess) { cleanup(); fail(c, EXC_EHIP, "copy of E[%d]: %s", q, hipGetErrorString(e)); return bail(EXC_EHIP); }
      }
    }
    // device-to-device copies need not have finished when hipMemcpy returns: the kernels
    // below run on `stream`
    if (cv->on_device) {
      const hipError_t e = hipDeviceSynchronize();
      if (e != hipSuccess) { cleanup(); fail(c, EXC_EHIP, "copy of the blocks: %s", hipGetErrorString(e)); return bail(EXC_EHIP); }
    }
    if ((s = upload(c, &d_eoff, e_off)) != EXC_OK || (s = upload(c, &d_uoff, c->u_off)) != EXC_OK ||
        (s = upload(c, &d_nd, nd32)) != EXC_OK || (s = upload(c, &d_eld, e_ld)) != EXC_OK ||
        (s = upload(c, &d_ldu, ldu32)) != EXC_OK || (s = dalloc(c, &d_info, (size_t)c->n_q + 1)) != EXC_OK) {
      cleanup(); return bail(s);
    }
    hipMemsetAsync(d_info, 0, (c->n_q + 1) * sizeof(int), st);
    const size_t usz = lds_elem_size(c->precision);
    s = dalloc(c, (char**)&c->d_U, (size_t)u_total * usz);
    if (s != EXC_OK) { cleanup(); return bail(s); }
    if (c->form == EXC_FORM_CHOL_HERK) {
      if (c->n_ch)
        hipLaunchKernelGGL(chan_chol_kernel, dim3((c->n_ch + 63) / 64, c->nqc), dim3(64), 0, st, c->n_ch,
                           c->d_ch_off, c->d_ch_len, c->d_ch_coef, c->d_coef, c->d_cvec,
                           c->d_schur, d_info + c->n_q, c->nqc > 1 ? c->coef_total : (int64_t)0,
                           c->nqc > 1 ? (int64_t)c->n_s : (int64_t)0);
      CholArgs ca{d_E, d_eoff, d_nd, d_eld, c->n_ch, c->n_ch ? c->d_schur : nullptr,
                  c->nqc > 1 ? c->n_ch : 0, d_info, 0};
      const int nblk = (*std::max_element(c->nd.begin(), c->nd.end()) + kCholBlock - 1) / kCholBlock;
      for (; ca.jb < nblk; ++ca.jb) {
        hipLaunchKernelGGL(chol_update_kernel, dim3(c->n_q, nblk - ca.jb), dim3(256), 0, st, ca);
        if (ca.jb + 1 < nblk)
          hipLaunchKernelGGL(chol_solve_kernel, dim3(c->n_q, nblk - ca.jb - 1), dim3(256), 0, st, ca);
      }
    }
    dim3 pg(64, c->n_q);
    const int f = c->form;
    switch (c->precision) {
      case EXC_FP64:
        if (f == 1) hipLaunchKernelGGL((prep_factor_kernel<M_F64, 1>), pg, dim3(256), 0, st, d_E, d_eoff, d_nd, d_eld, c->d_U, d_uoff, d_ldu);
        else hipLaunchKernelGGL((prep_factor_kernel<M_F64, 0>), pg, dim3(256), 0, st, d_E, d_eoff, d_nd, d_eld, c->d_U, d_uoff, d_ldu);
        break;
      case EXC_FP32:
        hipLaunchKernelGGL((prep_factor_kernel<M_F32, 1>), pg, dim3(256), 0, st, d_E, d_eoff, d_nd, d_eld, c->d_U, d_uoff, d_ldu);
        break;
      case EXC_BF16X3:
        hipLaunchKernelGGL((prep_factor_kernel<M_BF16X3, 1>), pg, dim3(256), 0, st, d_E, d_eoff, d_nd, d_eld, c->d_U, d_uoff, d_ldu);
        break;
      default:
        hipLaunchKernelGGL((prep_factor_kernel<M_BF16X6, 1>), pg, dim3(256), 0, st, d_E, d_eoff, d_nd, d_eld, c->d_U, d_uoff, d_ldu);
        break;
    }
    std::vector<int> info(c->n_q + 1, 0);
    hipError_t e1 = hipGetLastError();
    hipError_t e2 = hipStreamSynchronize(st);
    hipError_t e3 = hipMemcpy(info.data(), d_info, info.size() * sizeof(int), hipMemcpyDeviceToHost);
    cleanup();
    if (e1 != hipSuccess || e2 != hipSuccess || e3 != hipSuccess) {
      fail(c, EXC_EHIP, "factor preparation failed: %s", hipGetErrorString(e1 != hipSuccess ? e1 : (e2 != hipSuccess ? e2 : e3)));
      return bail(EXC_EHIP);
    }
    if (info[c->n_q]) { fail(c, EXC_ENOTPD, "a multipole-free channel block D_c is not positive definite"); return bail(EXC_ENOTPD); }
    if (c->n_s > 0) {
      // the fused kernel's padded runs of the (now factored) channel coefficients
      const long ne = (long)std::max(1, c->n_schunk) * kChunkRows * kRunPad;
      hipLaunchKernelGGL(pad_runs_kernel, dim3((unsigned)((ne + 255) / 256), c->nqc), dim3(256), 0, st, c->d_coef,
                         c->d_rowinfo, c->d_schunk, c->n_schunk, kRunPad, kChunkRows, c->d_coefpad,
                         c->nqc > 1 ? c->coef_total : (int64_t)0);
      // the fused kernels' operands of the block-sparse rows, from the (now factored) channel coefficients
      if (c->n_schunk)
        hipLaunchKernelGGL(pack_units_kernel, dim3(c->row_units.n_units, c->nqc), dim3(128), 0, st, c->row_units,
                           c->d_uowner, c->d_coef, c->d_cvec, c->d_rowinfo, c->n_s,
                           c->nqc > 1 ? c->coef_total : (int64_t)0, c->nqc > 1 ? (int64_t)c->n_s : (int64_t)0, c->d_uw);
      if (c->d_runs) {
        // sparse_kernel's runs of the factored channel coefficients, row by row
        const long nr = (long)c->run_max * c->runs_ld;
        hipLaunchKernelGGL(runs_by_row_kernel, dim3((unsigned)((nr + 255) / 256), c->nqc), dim3(256), 0, st,
                           c->d_coef, c->d_rowinfo, c->n_s, c->run_max, c->runs_ld, c->d_runs,
                           c->nqc > 1 ? c->coef_total : (int64_t)0);
      }
      IHIP(hipGetLastError());
      IHIP(hipStreamSynchronize(st));
    }
    for (int q = 0; q < c->n_q; ++q)
      if (info[q]) { fail(c, EXC_ENOTPD, "v(q) is not positive definite at q = %d (pivot %d)", q, info[q]); return bail(EXC_ENOTPD); }
  }

  // ---- pairs (k-major), workspace, plans ----
  // sparse-row workspace: FP64 -> double2 rows (pitch n_s, or n_s + n_ch with the
  // GEMM form's multipole corrections); reduced precision -> split planes
  // [plane][row] per column with the row pitch padded to 8 (elements of lds_t)
  // FP64: double2 sparse rows (pitch n_s, or n_s + n_ch with the GEMM form's
  // multipole corrections). Reduced precision: each column packed into split
  // planes [plane][row], rows = sparse rows padded to 8 then dense rows padded
  // to 32 (elements of the mode's storage type).
  const bool split_ws = c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64;
  c->ns_pad = (c->n_s + 7) / 8 * 8;
  const int ws_cols = split_ws ? 2 * npieces(c->precision) : 1;   // planes per column
  int64_t ws_total = 0, m_max = 0;
  c->k_pair.assign(1, 0);
  c->k_ws_start.assign(1, 0);
  int64_t ws_kmax = 0;
  for (int k = 0; k < c->n_k; ++k) {
    int64_t moff = 0;
    for (int q = 0; q < c->n_q; ++q) {
      const double wpair = c->wkq[(size_t)k * c->n_q + q];
      if (wpair == 0.0) continue;       // not computed; its block is absent from M
      PairInfo p{};
      p.k = k; p.q = q; p.nb = c->nb[k]; p.nmb = c->nmb[q]; p.nd = c->nd[q];
      p.nsb = (c->n_s + BM - 1) / BM; p.ndb = (c->nd[q] + BM - 1) / BM;
      p.nb8 = (p.nb + 7) / 8 * 8;
      const int ldw = split_ws ? c->ns_pad + (c->nd[q] + 31) / 32 * 32
                               : (c->form == EXC_FORM_CHOL_HERK ? c->n_s : c->n_s + c->n_ch);
      p.m_off = moff; p.ws_off = ws_total; p.u_off = c->u_off[q]; p.ldu = c->ldu[q]; p.ldw = std::max(1, ldw);
      moff += (int64_t)c->n_occ * p.nb * p.nmb;
      ws_total += (int64_t)c->n_occ * p.nb * ldw * ws_cols;
      c->pairs.push_back(p);
      c->pair_w.push_back(wpair);
      // accounting (nominal: sparse-aware method, Hermitian upper triangle)
      const double R = (double)c->n_occ * p.nb;
      double sp = 0;
      for (int ch = 0; ch < c->n_ch; ++ch) sp += 8.0 * c->ch_len[ch] * c->ch_len[ch] * R;
      c->flops_nominal += 8.0 * p.nd * (double)p.nd * R + sp + 16.0 * c->n_s * R +
                          4.0 * p.nb * (p.nb + 1.0) * p.nmb * c->n_occ;
      if (c->form == EXC_FORM_CHOL_HERK)
        c->flops_exec += 4.0 * p.nd * (double)p.nd * R + 4.0 * p.nb * (p.nb + 1.0) * p.nmb * c->n_occ;
      else
        c->flops_exec += 8.0 * p.nd * (double)p.nd * R + 4.0 * p.nb * (p.nb + 1.0) * p.nmb * c->n_occ;
    }
    m_max = std::max(m_max, moff);
    c->m_len.push_back(moff);
    ws_kmax = std::max(ws_kmax, ws_total - c->k_ws_start.back());
    c->k_ws_start.push_back(ws_total);
    c->k_pair.push_back((int)c->pairs.size());
  }
  for (int k = 0; k < c->n_k; ++k)
    if (c->k_pair[k + 1] == c->k_pair[k]) {
      fail(c, EXC_EINVAL, "w_kq leaves no q for k = %d", k);
      return bail(EXC_EINVAL);
    }
  // with inversion symmetry the method works in real arithmetic (2 flops per multiply-add
  // instead of 8) on n_occ_v real bands
  if (c->real_v) c->flops_nominal *= (double)c->n_occ_v / c->n_occ / 4.0;
  {
    double mb = 0, vb = 0, ub = 0;
    for (int k = 0; k < c->n_k; ++k) {
      int64_t e = 0;
      for (int q = 0; q < c->n_q; ++q)
        if (c->wkq[(size_t)k * c->n_q + q] != 0.0) e += (int64_t)c->n_occ * c->nb[k] * c->nmb[q];
      mb += (double)e;
      vb += (double)c->nb[k] * c->nb[k] * 16.0;
    }
    for (int q = 0; q < c->n_q; ++q) {                // v(q) dense block once, if some k uses q
      bool used = false;
      for (int k = 0; k < c->n_k; ++k) used = used || c->wkq[(size_t)k * c->n_q + q] != 0.0;
      if (used) ub += (double)c->nd[q] * c->nd[q] * 16.0;
    }
    c->bytes_alg = mb * 16.0 + ub + vb;   // per complex128 M; the binding rescales for complex64
  }
  c->mstage_bytes = (size_t)m_max * 16;
  ITRY(upload(c, &c->d_pairs, c->pairs));
  ITRY(upload(c, &c->d_pair_w, c->pair_w));
  ITRY(upload(c, &c->d_pair_begin, std::vector<int32_t>(c->k_pair.begin(), c->k_pair.end())));
  const size_t wsz = split_ws ? lds_elem_size(c->precision) : 16;
  c->ws_elem = wsz;
  c->ws_bytes = (size_t)std::max<int64_t>(1, ws_total) * wsz;
  c->ws_k_bytes = (size_t)std::max<int64_t>(1, ws_kmax) * wsz;
  const int nbt = c->nbt_max;
  c->gstride = nbt * (nbt + 1) / 2 * 256;
  c->dstride = nbt * 8;

  int64_t vtot = 0;
  for (int k = 0; k < c->n_k; ++k) { c->v_off.push_back(vtot); vtot += (int64_t)c->nb[k] * c->nb[k]; }
  ITRY(dalloc(c, &c->d_vres, (size_t)vtot));
  ITRY(upload(c, &c->d_voff, c->v_off));
  ITRY(upload(c, &c->d_knb, std::vector<int32_t>(c->nb.begin(), c->nb.end())));
  c->v_valid.assign(c->n_k, 0);
  ITRY(dalloc(c, &c->d_mtab, (size_t)c->n_k));
  ITRY(dalloc(c, &c->d_vtab, (size_t)c->n_k));
  c->h_mtab.assign(c->n_k, nullptr);
  c->h_vtab.assign(c->n_k, nullptr);
  IHIP(hipMemset(c->d_mtab, 0, c->n_k * sizeof(void*)));
  IHIP(hipMemset(c->d_vtab, 0, c->n_k * sizeof(void*)));
  ITRY(dalloc(c, &c->d_counter, (size_t)NQ_MAX));
  IHIP(hipMemset(c->d_counter, 0, NQ_MAX * sizeof(int32_t)));   // each q-sum clears them again
  ITRY(dalloc(c, &c->d_eout, (size_t)c->n_k));
  ITRY(dalloc(c, &c->d_ewk, (size_t)c->n_k));
  ITRY(dalloc(c, &c->d_erho, (size_t)c->n_k));
  ITRY(dalloc(c, &c->d_gamma, (size_t)4));
  ITRY(dalloc(c, &c->d_tmask, (size_t)3 * c->n_k));
  IHIP(hipMemset(c->d_tmask, 0xFF, (size_t)3 * c->n_k * sizeof(uint64_t)));   // every tile pair
  IHIP(hipMemset(c->d_gamma, 0, 4 * sizeof(double)));   // no Gamma-point shift until requested

  c->sncw = pick_sparse_ncw(c);
  if (const char* ev = getenv("EXC_GRAPH")) c->direct = ev[0] != '1';
  if (sparse_lds_bytes(c) > 65536)
    IHIP(hipFuncSetAttribute(sparse_fn(c), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sparse_lds_bytes(c)));
  if (const char* ev = getenv("EXC_CHUNK_BYTES")) c->chunk_bytes = strtoull(ev, nullptr, 10);
  if (const char* ev = getenv("EXC_FUSED_SPLIT")) c->fsplit = std::min(2, std::max(0, atoi(ev)));   // (fixed-configuration runs)
  if (c->plain_gemm) {
    // W of the largest pair (laid out as M), the split partials of A^H W, the V(k) accumulator
    std::vector<PairInfo> pp(c->pairs);
    size_t w_max = 1, g_max = 1;
    c->p_split.resize(c->pairs.size());
    for (size_t i = 0; i < pp.size(); ++i) {
      pp[i].ws_off = 0;
      pp[i].ldw = pp[i].nmb;
      w_max = std::max(w_max, (size_t)pp[i].nmb * c->n_occ * pp[i].nb);
      // split the MPB index so that the band contraction has about 512 workgroups
      const int nt = (pp[i].nb + PG_BM - 1) / PG_BM, tiles = nt * (nt + 1) / 2 * c->n_occ;
      int ns = std::max(1, std::min((512 + tiles - 1) / tiles, (pp[i].nmb + 63) / 64));
      const int kch = ((pp[i].nmb + ns - 1) / ns + PG_KC - 1) / PG_KC * PG_KC;
      ns = (pp[i].nmb + kch - 1) / kch;
      c->p_split[i] = ns;
      g_max = std::max(g_max, (size_t)ns * c->n_occ * pp[i].nb * pp[i].nb);
    }
    ITRY(upload(c, &c->d_ppairs, pp));
    ITRY(dalloc(c, &c->d_pw, w_max));
    ITRY(dalloc(c, &c->d_pg, g_max));
    ITRY(dalloc(c, &c->d_pvacc, (size_t)c->nb_max * c->nb_max));
  } else {
    ITRY(configure(c, c->fused ? c->fcfg : nullptr, st));
  }
  IHIP(take_own(c));
  IHIP(hipEventCreateWithFlags(&c->ev_in, hipEventDisableTiming));
  IHIP(hipEventCreateWithFlags(&c->ev_tab, hipEventDisableTiming));
  IHIP(hipEventCreateWithFlags(&c->ev_out, hipEventDisableTiming));
  IHIP(hipEventCreateWithFlags(&c->ev_en, hipEventDisableTiming));
  IHIP(hipStreamSynchronize(st));
#undef ITRY
#undef IHIP
  *out = c;
  return EXC_OK;
}

static exc_status ensure_stage(exc_ctx* c) {
  if (!c->d_mstage) TRY(dalloc(c, (char**)&c->d_mstage, c->mstage_bytes));
  return EXC_OK;
}

exc_status exchange_matrix(exc_ctx* c, int32_t k, const void* M, int32_t dtype, int32_t on_device,
                           void* Vx, void* stream) {
  TRY(check_ctx(c));
  if (k < 0 || k >= c->n_k) return fail(c, EXC_EINVAL, "k = %d outside [0, %d)", k, c->n_k);
  if (!M || !Vx) return fail(c, EXC_EINVAL, "M or Vx is NULL");
  if (dtype != EXC_C128 && dtype != EXC_C64) return fail(c, EXC_EINVAL, "bad dtype %d", dtype);
  hipStream_t st = (hipStream_t)stream;
  c->last_stream = st;
  HIPCHK(c, hipSetDevice(c->device));
  const size_t esz = dtype == EXC_C64 ? 8 : 16;
  const size_t mbytes = (size_t)c->m_len[k] * esz;
  const void* Md = M;
  void* Vd = Vx;
  if (!on_device) {
    TRY(ensure_stage(c));
    if (mbytes) HIPCHK(c, hipMemcpyAsync(c->d_mstage, M, mbytes, hipMemcpyHostToDevice, st));
    Md = c->d_mstage;
    Vd = nullptr;
  }
  const void* mp[1] = {Md};
  void* vp[1] = {Vd};
  TRY(fit_dtype(c, dtype, st));
  TRY(set_tables(c, k, 1, mp, vp, st));
  const bool shared = shares(c);
  if (shared) TRY(turn_begin(c, c->turn_ws, st));
  if (c->plain_gemm) TRY(run_k_plain_gemm(c, k, dtype, st));
  else if (c->batched) TRY(run_k_batched(c, k, dtype, st));
  else TRY(run_k_plain(c, k, dtype, st));
  HIPCHK(c, hipGetLastError());
  if (shared) TRY(turn_end(c, c->turn_ws, st));
  if (!on_device) {
    HIPCHK(c, hipMemcpyAsync(Vx, c->d_vres + c->v_off[k], (size_t)c->nb[k] * c->nb[k] * 16,
                             hipMemcpyDeviceToHost, st));
    HIPCHK(c, hipStreamSynchronize(st));
  }
  c->v_valid[k] = 1;
  return EXC_OK;
}

exc_status exchange_matrix_noalloc(exc_ctx* c, int32_t k, const void* M, int32_t dtype, void* Vx,
                                   void* stream) {
  TRY(check_ctx(c));
  if (k < 0 || k >= c->n_k) return fail(c, EXC_EINVAL, "k = %d outside [0, %d)", k, c->n_k);
  if (!M || !Vx) return fail(c, EXC_EINVAL, "M or Vx is NULL");
  if (dtype != EXC_C128 && dtype != EXC_C64) return fail(c, EXC_EINVAL, "bad dtype %d", dtype);
  if (!c->batched || c->plain_gemm)
    return fail(c, EXC_EUNSUPPORTED, "the no-allocation call serves batched contexts only");
  if (c->fused && c->fcfg->c64only && dtype != EXC_C64)
    return fail(c, EXC_EUNSUPPORTED, "this context's kernel reads complex64 M (exchange_matrix switches kernels)");
  void* base = c->device >= 0 && c->device < kScratchDevices ? g_scratch_ptr[c->device] : nullptr;
  if (!base) return fail(c, EXC_ESTATE, "no scratch address for device %d", c->device);
  // this k's share of the buffers, each region 256-byte aligned
  const Plan& P = k_plan(c);
  const int s0 = P.slot_begin[k], ns = P.slot_begin[k + 1] - s0;
  const int p0 = c->k_pair[k], np = c->k_pair[k + 1] - p0;
  const size_t asz = c->precision == EXC_FP64 ? 8 : 4;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t g_b = up((size_t)ns * c->gstride * asz), d_b = up((size_t)ns * c->dstride * 8);
  const bool tile_path = !c->fused;
  const size_t w_b = tile_path ? up((size_t)(c->k_ws_start[k + 1] - c->k_ws_start[k]) * c->ws_elem) : 0;
  const size_t s_b = tile_path && c->d_dsp ? up((size_t)np * c->n_occ * c->nb_max * 8) : 0;
  const size_t need = g_b + d_b + w_b + s_b;
  if (need > kScratchBytes)
    return fail(c, EXC_EINVAL, "k = %d needs %zu bytes of scratch; the no-allocation call holds %zu "
                "(exchange_matrix has no such limit)", k, need, kScratchBytes);
  const uintptr_t b = (uintptr_t)base;
  ScratchView v{};
  v.gpart = (void*)(b - (uintptr_t)s0 * c->gstride * asz);
  v.dpart = (double*)(b + g_b - (uintptr_t)s0 * c->dstride * 8);
  v.ws = tile_path ? (void*)(b + g_b + d_b - (uintptr_t)c->k_ws_start[k] * c->ws_elem) : nullptr;
  v.dsp = s_b ? (double*)(b + g_b + d_b + w_b - (uintptr_t)p0 * c->n_occ * c->nb_max * 8) : nullptr;
  hipStream_t st = (hipStream_t)stream;
  c->last_stream = st;
  HIPCHK(c, hipSetDevice(c->device));
  const void* mp[1] = {M};
  void* vp[1] = {Vx};
  TRY(set_tables(c, k, 1, mp, vp, st));
  // the launches of run_k_batched, on the scratch (every slot, workspace row and |Y_s|^2 sum
  // the reduction reads is written first by this call's kernels: nothing needs clearing)
  c->sv = &v;
  launch_sparse(c, dtype, k, p0, np, st);
  launch_k(c, P, dtype, k, st);
  launch_reduce(c, P, k, 1, st);
  c->sv = nullptr;
  HIPCHK(c, hipGetLastError());
  c->v_valid[k] = 1;
  return EXC_OK;
}

exc_status exchange_matrix_all(exc_ctx* c, const void* const* M_k, int32_t dtype, int32_t on_device,
                               void* const* Vx_k, void* stream) {
  TRY(check_ctx(c));
  if (!M_k || !Vx_k) return fail(c, EXC_EINVAL, "M_k or Vx_k is NULL");
  for (int k = 0; k < c->n_k; ++k)
    if (!M_k[k] || !Vx_k[k]) return fail(c, EXC_EINVAL, "M_k[%d] or Vx_k[%d] is NULL", k, k);
  if (dtype != EXC_C128 && dtype != EXC_C64) return fail(c, EXC_EINVAL, "bad dtype %d", dtype);
  if (!on_device) {
    for (int k = 0; k < c->n_k; ++k) TRY(exchange_matrix(c, k, M_k[k], dtype, 0, Vx_k[k], stream));
    return EXC_OK;
  }
  hipStream_t st = (hipStream_t)stream;
  c->last_stream = st;
  HIPCHK(c, hipSetDevice(c->device));
  if (!c->batched) {
    TRY(fit_dtype(c, dtype, st));
    TRY(set_tables(c, 0, c->n_k, M_k, Vx_k, st));
    const bool shared = shares(c);
    if (shared) TRY(turn_begin(c, c->turn_ws, st));
    for (int k = 0; k < c->n_k; ++k)
      TRY(c->plain_gemm ? run_k_plain_gemm(c, k, dtype, st) : run_k_plain(c, k, dtype, st));
    HIPCHK(c, hipGetLastError());
    if (shared) TRY(turn_end(c, c->turn_ws, st));
  } else {
    if (!c->tune_done) {
      const char* ev = getenv("EXC_TUNE");
      const char* fixed = getenv("EXC_FUSED_CFG");      // an explicit configuration is not tuned
      const char* off = getenv("EXC_FUSED");
      const bool mixed_herk = c->form == EXC_FORM_CHOL_HERK && c->precision != EXC_FP64 && !fixed &&
                              !(off && off[0] == '0');
      TRY(set_tables(c, 0, c->n_k, M_k, Vx_k, st));
      if (mixed_herk && !(ev && ev[0] == '0')) {
        HIPCHK(c, hipEventRecord(c->ev_in, st));          // the inputs are ready on the caller's stream
        HIPCHK(c, hipStreamWaitEvent(c->own, c->ev_in, 0));
        TRY(autotune(c, dtype, st));
      }
      c->tune_done = true;
    }
    TRY(fit_dtype(c, dtype, st));                  // (a fixed or earlier choice may read complex64 only)
    const bool shared = shares(c);
    if (shared) TRY(turn_begin(c, c->turn_ws, st));
    if (c->direct) {
      TRY(set_tables(c, 0, c->n_k, M_k, Vx_k, st));
      TRY(launch_batched_direct(c, dtype, st));
      if (shared) TRY(turn_end(c, c->turn_ws, st));
      for (int k = 0; k < c->n_k; ++k) c->v_valid[k] = 1;
      return EXC_OK;
    }
    bool same = c->gexec && c->g_dtype == dtype;
    for (int k = 0; k < c->n_k && same; ++k)
      if (c->h_mtab[k] != M_k[k] || c->h_vtab[k] != Vx_k[k]) same = false;
    TRY(set_tables(c, 0, c->n_k, M_k, Vx_k, st));
    if (!same) {
      if (c->gexec) { hipGraphExecDestroy(c->gexec); c->gexec = nullptr; }
      TRY(build_batched_graph(c, dtype));
    }
    if (c->t_slots > 0 && c->tnode[1] && c->tnode[2]) {
      // rotate the event triple of this replay
      const int s = c->t_next;
      for (int i = 0; i < 3; ++i)
        if (c->tnode[i]) HIPCHK(c, hipGraphExecEventRecordNodeSetEvent(c->gexec, c->tnode[i], c->tpool[3 * s + i]));
      c->t_next = (c->t_next + 1) % c->t_slots;
      c->t_count = std::min(c->t_count + 1, c->t_slots);
    }
    HIPCHK(c, hipGraphLaunch(c->gexec, st));     // in order with the caller's work on st
    if (shared) TRY(turn_end(c, c->turn_ws, st));
  }
  for (int k = 0; k < c->n_k; ++k) c->v_valid[k] = 1;
  return EXC_OK;
}

exc_status exchange_energy(exc_ctx* c, const double* w_k, const void* const* rho_k, double* E_out) {
  TRY(check_ctx(c));
  if (!E_out) return fail(c, EXC_EINVAL, "E_out is NULL");
  for (int k = 0; k < c->n_k; ++k)
    if (!c->v_valid[k]) return fail(c, EXC_ESTATE, "V(k=%d) has not been computed", k);
  hipStream_t st = c->last_stream;
  // the energy buffers are shared by every energy call: after the previous one, on any stream
  if (c->ev_en_set) HIPCHK(c, hipStreamWaitEvent(st, c->ev_en, 0));
  void** d_rho = nullptr;
  if (rho_k) {
    TRY(dalloc(c, &d_rho, (size_t)c->n_k));
    if (hipMemcpy(d_rho, rho_k, c->n_k * sizeof(void*), hipMemcpyHostToDevice) != hipSuccess) {
      hipFree(d_rho);
      return fail(c, EXC_EHIP, "copy of rho pointers failed");
    }
  }
  hipLaunchKernelGGL(energy_kernel, dim3(c->n_k), dim3(256), 0, st, c->d_vres, c->d_voff, c->d_knb,
                     (const void* const*)d_rho, c->n_occ_v, c->d_eout);
  std::vector<double> e(c->n_k);
  hipError_t e1 = hipGetLastError();
  if (e1 == hipSuccess) e1 = hipEventRecord(c->ev_en, st);
  c->ev_en_set = e1 == hipSuccess;
  hipError_t e2 = hipStreamSynchronize(st);
  hipError_t e3 = hipMemcpy(e.data(), c->d_eout, c->n_k * sizeof(double), hipMemcpyDeviceToHost);
  if (d_rho) hipFree(d_rho);
  if (e1 != hipSuccess || e2 != hipSuccess || e3 != hipSuccess) return fail(c, EXC_EHIP, "energy kernel failed");
  double s = 0.0;
  for (int k = 0; k < c->n_k; ++k) s += (w_k ? w_k[k] : 1.0 / c->n_k) * e[k];
  *E_out = 0.5 * s;
  return EXC_OK;
}

exc_status exchange_energy_device(exc_ctx* c, const double* w_k, const void* const* rho_k, double* E_dev,
                                  void* stream) {
  TRY(check_ctx(c));
  if (!E_dev) return fail(c, EXC_EINVAL, "E_dev is NULL");
  for (int k = 0; k < c->n_k; ++k)
    if (!c->v_valid[k]) return fail(c, EXC_ESTATE, "V(k=%d) has not been computed", k);
  hipStream_t st = stream ? (hipStream_t)stream : c->last_stream;
  if (st != c->last_stream) {                     // after the last V(k) on its stream
    HIPCHK(c, hipEventRecord(c->ev_out, c->last_stream));
    HIPCHK(c, hipStreamWaitEvent(st, c->ev_out, 0));
  }
  // the staging buffers (weights, rho pointers, per-k energies) are shared by every energy
  // call: after the previous one, whatever its stream
  if (c->ev_en_set) HIPCHK(c, hipStreamWaitEvent(st, c->ev_en, 0));
  // the host arrays are copied before this call returns (pageable source)
  if (w_k) HIPCHK(c, hipMemcpyAsync(c->d_ewk, w_k, c->n_k * sizeof(double), hipMemcpyHostToDevice, st));
  if (rho_k) HIPCHK(c, hipMemcpyAsync(c->d_erho, rho_k, c->n_k * sizeof(void*), hipMemcpyHostToDevice, st));
  if (rho_k) {
    hipLaunchKernelGGL(energy_kernel, dim3(c->n_k), dim3(256), 0, st, c->d_vres, c->d_voff, c->d_knb,
                       (const void* const*)c->d_erho, c->n_occ_v, c->d_eout);
    hipLaunchKernelGGL(energy_sum_kernel, dim3(1), dim3(256), 0, st, c->d_eout, w_k ? c->d_ewk : nullptr,
                       c->n_k, E_dev);
  } else {                                         // rho = 2 P_occ: one launch
    hipLaunchKernelGGL(energy_diag_kernel, dim3(1), dim3(256), 0, st, c->d_vres, c->d_voff, c->d_knb,
                       c->n_k, c->n_occ_v, w_k ? c->d_ewk : nullptr, E_dev);
  }
  HIPCHK(c, hipGetLastError());
  HIPCHK(c, hipEventRecord(c->ev_en, st));
  c->ev_en_set = true;
  return EXC_OK;
}

exc_status exchange_gamma_term(exc_ctx* c, const double* recip, const int32_t* mesh, double beta,
                               int32_t apply, double* C_out, void* stream) {
  TRY(check_ctx(c));
  if (!recip || !mesh) return fail(c, EXC_EINVAL, "recip and mesh must not be NULL");
  if (!(beta > 0.0 && beta < 1.0)) return fail(c, EXC_EINVAL, "beta = %g is outside (0, 1)", beta);
  for (int i = 0; i < 3; ++i)
    if (mesh[i] < 1) return fail(c, EXC_EINVAL, "mesh[%d] = %d < 1", i, mesh[i]);
  for (int i = 0; i < 9; ++i)
    if (!std::isfinite(recip[i])) return fail(c, EXC_EINVAL, "recip[%d] is not finite", i);
  if (apply && c->has_wkq)
    return fail(c, EXC_EUNSUPPORTED, "the Gamma-point shift enters the full q sum once; with per-pair weights "
                "(w_kq) add -C to the occupied diagonal after the rotation over the little group of k");
  // cofactor rows of B: a_i = 2 pi cof_i / det B are the real-space vectors
  const double(*B)[3] = (const double(*)[3])recip;
  double cof[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      const int i1 = (i + 1) % 3, i2 = (i + 2) % 3, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
      cof[i][j] = B[i1][j1] * B[i2][j2] - B[i1][j2] * B[i2][j1];
    }
  const double det = B[0][0] * cof[0][0] + B[0][1] * cof[0][1] + B[0][2] * cof[0][2];
  double bmax = 0.0;
  for (int i = 0; i < 9; ++i) bmax = std::max(bmax, std::fabs(recip[i]));
  if (!(std::fabs(det) > 1e-12 * bmax * bmax * bmax))
    return fail(c, EXC_EINVAL, "the reciprocal lattice vectors are linearly dependent");
  const double q0 = std::sqrt(-std::log(beta) / beta);   // exp(-beta q0^2) = beta
  GammaArgs ga{};
  double boxes = 1.0;
  for (int i = 0; i < 3; ++i) {
    const double an = std::sqrt(cof[i][0] * cof[i][0] + cof[i][1] * cof[i][1] + cof[i][2] * cof[i][2]);
    // |j_i| = mesh_i |p . a_i| / (2 pi) <= mesh_i q0 |a_i| / (2 pi); one more for rounding
    const double jm = std::floor(mesh[i] * q0 * an / std::fabs(det)) + 1.0;
    if (jm > 1e9) return fail(c, EXC_EINVAL, "the lattice sum is too large (beta too small for this mesh)");
    ga.J[i] = (int32_t)jm;
    boxes *= 2.0 * jm + 1.0;
    for (int d = 0; d < 3; ++d) ga.g[i][d] = recip[3 * i + d] / mesh[i];
  }
  if (boxes > 1099511627776.0)   // 2^40 candidate points
    return fail(c, EXC_EINVAL, "the lattice sum is too large (%.3g candidate points)", boxes);
  ga.beta = beta;
  ga.q0sq = q0 * q0;
  if (!c->d_gpartial) TRY(dalloc(c, &c->d_gpartial, (size_t)2 * kGammaGrid));
  ga.part = c->d_gpartial;
  if (!c->ev_g[0]) {
    HIPCHK(c, hipEventCreate(&c->ev_g[0]));
    HIPCHK(c, hipEventCreate(&c->ev_g[1]));
  }
  const double pi = 3.14159265358979323846;
  const double omega = 8.0 * pi * pi * pi / std::fabs(det);
  const double pref = 4.0 * pi / ((double)mesh[0] * mesh[1] * mesh[2] * omega);
  hipStream_t st = (hipStream_t)stream;
  if (c->last_stream && st != c->last_stream) {   // the shift changes after earlier q-sums
    HIPCHK(c, hipEventRecord(c->ev_out, c->last_stream));
    HIPCHK(c, hipStreamWaitEvent(st, c->ev_out, 0));
  }
  HIPCHK(c, hipEventRecord(c->ev_g[0], st));
  hipLaunchKernelGGL(gamma_sum_kernel, dim3(kGammaGrid), dim3(kGammaBlock), 0, st, ga);
  HIPCHK(c, hipEventRecord(c->ev_g[1], st));
  hipLaunchKernelGGL(gamma_finish_kernel, dim3(1), dim3(kGammaBlock), 0, st, (const double*)c->d_gpartial,
                     kGammaGrid, beta, q0, pref, (int)(apply != 0), c->d_gamma);
  HIPCHK(c, hipGetLastError());
  double h[4];
  HIPCHK(c, hipMemcpyAsync(h, c->d_gamma, sizeof(h), hipMemcpyDeviceToHost, st));
  HIPCHK(c, hipStreamSynchronize(st));
  HIPCHK(c, hipEventElapsedTime(&c->gamma_ms, c->ev_g[0], c->ev_g[1]));
  c->gamma_terms = h[2];
  if (C_out) *C_out = h[0];
  return EXC_OK;
}

exc_status exchange_back_transform(exc_ctx* c, int32_t k, const void* Z, int32_t n_G, void* VGG, void* stream) {
  TRY(check_ctx(c));
  if (k < 0 || k >= c->n_k) return fail(c, EXC_EINVAL, "k = %d outside [0, %d)", k, c->n_k);
  if (!Z || !VGG) return fail(c, EXC_EINVAL, "Z or VGG is NULL");
  if (n_G < 1 || n_G > (1 << 20)) return fail(c, EXC_EINVAL, "n_G = %d outside [1, 2^20]", n_G);
  if (!c->v_valid[k]) return fail(c, EXC_ESTATE, "V(k=%d) has not been computed", k);
  HIPCHK(c, hipSetDevice(c->device));
  const int nb = c->nb[k];
  const size_t need = (size_t)n_G * nb;
  if (need > c->bt_cap) {                         // earlier back-transforms may still read the old one
    if (c->d_bt) {
      HIPCHK(c, hipDeviceSynchronize());
      hipFree(c->d_bt);
      c->d_bt = nullptr;
      c->bt_cap = 0;
    }
    TRY(dalloc(c, &c->d_bt, need));
    c->bt_cap = need;
  }
  if (!c->ev_bt[0]) {
    HIPCHK(c, hipEventCreate(&c->ev_bt[0]));
    HIPCHK(c, hipEventCreate(&c->ev_bt[1]));
  }
  hipStream_t st = (hipStream_t)stream;
  if (c->last_stream && st != c->last_stream) {   // after the work that wrote V(k)
    HIPCHK(c, hipEventRecord(c->ev_out, c->last_stream));
    HIPCHK(c, hipStreamWaitEvent(st, c->ev_out, 0));
  }
  TRY(turn_begin(c, c->turn_bt, st));
  const double2* V = c->d_vres + c->v_off[k];
  hipLaunchKernelGGL(bt_left_kernel, dim3((unsigned)((n_G + 15) / 16), (unsigned)((nb + 15) / 16)), dim3(256), 0, st,
                     (const double2*)Z, V, n_G, nb, c->d_bt);
  const long nt = (n_G + 15) / 16;
  const unsigned ngrid = (unsigned)std::min<long>(nt * (nt + 1) / 2, 1 << 20);
  HIPCHK(c, hipEventRecord(c->ev_bt[0], st));
  hipLaunchKernelGGL(bt_gram_kernel, dim3(ngrid), dim3(64), 0, st, (const double2*)c->d_bt,
                     (const double2*)Z, n_G, nb, (double2*)VGG);
  HIPCHK(c, hipEventRecord(c->ev_bt[1], st));
  HIPCHK(c, hipGetLastError());
  c->bt_timed = true;
  return turn_end(c, c->turn_bt, st);
}

exc_status exchange_band_mask(exc_ctx* c, int32_t k, const uint8_t* keep) {
  TRY(check_ctx(c));
  if (k < 0 || k >= c->n_k) return fail(c, EXC_EINVAL, "k = %d outside [0, %d)", k, c->n_k);
  const int nb = c->nb[k], nbt = (nb + 7) / 8;
  uint64_t bits[3] = {~0ull, ~0ull, ~0ull};
  if (keep) {
    bits[0] = bits[1] = bits[2] = 0;
    for (int J = 0; J < nbt; ++J)
      for (int I = 0; I <= J; ++I) {
        bool any = I == J;                        // diagonal tiles carry V_nn: always computed
        for (int n = 8 * I; n < std::min(nb, 8 * I + 8) && !any; ++n)
          for (int m = 8 * J; m < std::min(nb, 8 * J + 8) && !any; ++m)
            any = keep[(size_t)n * nb + m] || keep[(size_t)m * nb + n];
        const int tp = J * (J + 1) / 2 + I;
        if (any) bits[tp >> 6] |= 1ull << (tp & 63);
      }
  }
  HIPCHK(c, hipSetDevice(c->device));
  HIPCHK(c, hipDeviceSynchronize());              // no launch in flight reads the old mask
  HIPCHK(c, hipMemcpy(c->d_tmask + 3 * k, bits, sizeof(bits), hipMemcpyHostToDevice));
  return EXC_OK;
}

const char* exchange_last_error(const exc_ctx* c) {
  if (!c) return g_init_err.c_str();
  if (c->magic != kAlive) return "context is not alive";
  return c->err.c_str();
}

void exchange_destroy(exc_ctx* c) {
  if (!c || c->magic != kAlive) return;
  hipSetDevice(c->device);
  hipDeviceSynchronize();
  release(c);
  c->magic = 0;
  delete c;
}

exc_status exchange_query(const exc_ctx* c, int32_t what, double* value) {
  TRY(check_ctx(c));
  if (!value) return EXC_EINVAL;
  switch (what) {
    case 0: *value = c->bat.n_slots; return EXC_OK;
    case 1: *value = c->flops_nominal; return EXC_OK;
    case 2: *value = c->flops_exec; return EXC_OK;
    case 3:
      if (c->h64) *value = (c->batched ? c->bat : c->plain).h64->id();
      else *value = c->plain_gemm ? 900 : (c->fused ? c->fcfg->id : (c->cfg ? c->cfg->id : -1));
      return EXC_OK;
    case 4: *value = c->bytes_alg; return EXC_OK;
    case 5:
    case 7: {
      // mean duration (ms) of the tile (5) or sparse (7) kernel over the timed replays
      if (c->t_count == 0 || (what == 7 && !(c->direct ? c->t_sparse : c->tnode[0] != nullptr))) {
        *value = 0.0;
        return EXC_OK;
      }
      double sum = 0.0;
      for (int s = 0; s < c->t_count; ++s) {
        hipEvent_t* e = const_cast<hipEvent_t*>(&c->tpool[3 * s]);
        if (hipEventSynchronize(e[2]) != hipSuccess) return EXC_EHIP;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, what == 5 ? e[1] : e[0], what == 5 ? e[2] : e[1]) != hipSuccess) return EXC_EHIP;
        sum += ms;
      }
      *value = sum / c->t_count;
      return EXC_OK;
    }
    case 6: *value = c->t_count; return EXC_OK;
    case 8: *value = c->tuned; return EXC_OK;
    case 9: *value = (double)c->ws_bytes; return EXC_OK;
    case 10: *value = c->fused ? 1.0 : 0.0; return EXC_OK;
    case 11: *value = c->gamma_ms; return EXC_OK;
    case 12: *value = c->gamma_terms; return EXC_OK;
    case 14: *value = c->fused && !c->batched ? std::max(c->fsplit, 1) : c->fsplit; return EXC_OK;
    case 20: *value = c->chunk_batches; return EXC_OK;
    case 21: *value = c->chunk_fails; return EXC_OK;
    case 19: *value = c->fused ? fused_bm(*c->fcfg) : -1; return EXC_OK;
    case 15:
    case 16:
    case 17:
    case 18: {
      // the binary32 Gram accumulation of the reduced-precision main kernel (error models):
      // band tiles per pass, chain kind, rows per chunk in the block-sparse / dense rows
      if (c->precision == EXC_FP64 || c->plain_gemm || (!c->fused && !c->cfg)) { *value = -1; return EXC_OK; }
      const int v[4] = {c->fused ? c->fcfg->NCT : c->cfg->NCT,
                        c->fused ? c->fcfg->gchain : (c->batched ? c->cfg->gchain : 3),
                        c->fused ? c->fcfg->grs : c->cfg->grs, c->fused ? c->fcfg->grd : c->cfg->grd};
      *value = v[what - 15];
      return EXC_OK;
    }
    case 13: {                                    // the last back-transform's product kernel
      if (!c->bt_timed) { *value = 0.0; return EXC_OK; }
      if (hipEventSynchronize(c->ev_bt[1]) != hipSuccess) return EXC_EHIP;
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, c->ev_bt[0], c->ev_bt[1]) != hipSuccess) return EXC_EHIP;
      *value = ms;
      return EXC_OK;
    }
    default: return EXC_EINVAL;
  }
}

exc_status exchange_timing(exc_ctx* c, int32_t n_slots) {
  TRY(check_ctx(c));
  if (n_slots < 0) return fail(c, EXC_EINVAL, "n_slots < 0");
  HIPCHK(c, hipSetDevice(c->device));
  HIPCHK(c, hipDeviceSynchronize());
  release_timing(c);
  if (c->gexec) { hipGraphExecDestroy(c->gexec); c->gexec = nullptr; }   // re-capture with / without event nodes
  if (n_slots == 0) return EXC_OK;
  c->tpool.resize(3 * (size_t)n_slots, nullptr);
  for (auto& e : c->tpool) HIPCHK(c, hipEventCreate(&e));
  c->t_slots = n_slots;
  return EXC_OK;
}

}  // extern "C"

#include "nn_abi.hpp"
