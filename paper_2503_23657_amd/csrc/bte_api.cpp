// C ABI of the sweep library: problem set-up, device state, the iteration loop
// (replayed as a hipGraph), the adjoint, batching and the kernel-shape tuner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/bte.h"
#include "bte_device.h"
#include "bte_launch.h"
#include "bte_setup.h"

using namespace bte;

namespace {

thread_local std::string g_err;

void set_err(const char* f, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, f);
  vsnprintf(buf, sizeof(buf), f, ap);
  va_end(ap);
  g_err = buf;
}

#define HIPCHK(x)                                                                       \
  do {                                                                                  \
    hipError_t e_ = (x);                                                                \
    if (e_ != hipSuccess) {                                                             \
      set_err("HIP error '%s' at %s:%d", hipGetErrorString(e_), __FILE__, __LINE__);   \
      return BTE_ERR_HIP;                                                               \
    }                                                                                   \
  } while (0)

const double kPi = 3.14159265358979323846;

// Every ABI call leaves the HIP runtime's last-error state clear on exit: the
// runtime is shared with the caller (torch), whose next call would otherwise
// report an error this library already handled or returned.
struct ErrClear {
  ~ErrClear() { (void)hipGetLastError(); }
};

// Device memory of a handle. Three modes:
//   OWNED  every array is a hipMalloc of its own, freed with the pool;
//   ARENA  arrays are carved from a caller-provided workspace (256-byte
//          aligned offsets); nothing is allocated or freed;
//   COUNT  nothing is allocated or copied: the pool only adds up the bytes
//          an ARENA would need (the pointers it returns are never used).
constexpr size_t kWsAlign = 256;
struct DevPool {
  enum Mode { OWNED, ARENA, COUNT };
  Mode mode = OWNED;
  char* base = nullptr;  // ARENA
  size_t cap = 0;        // ARENA capacity (bytes)
  size_t used = 0;       // bytes requested so far (aligned)
  std::vector<void*> ptrs;
  DevPool() = default;
  explicit DevPool(Mode m, char* b = nullptr, size_t c = 0) : mode(m), base(b), cap(c) {}
  DevPool(const DevPool&) = delete;
  DevPool& operator=(const DevPool&) = delete;
  ~DevPool() {
    for (void* p : ptrs) (void)hipFree(p);
  }
  template <typename T>
  hipError_t alloc(T** out, size_t count) {
    const size_t bytes = (std::max<size_t>(count * sizeof(T), 16) + kWsAlign - 1) / kWsAlign * kWsAlign;
    if (mode == OWNED) {
      void* p = nullptr;
      hipError_t e = hipMalloc(&p, bytes);
      if (e != hipSuccess) return e;
      ptrs.push_back(p);
      *out = reinterpret_cast<T*>(p);
    } else if (mode == ARENA) {
      if (used + bytes > cap) return hipErrorOutOfMemory;  // sizes are checked before carving
      *out = reinterpret_cast<T*>(base + used);
    } else {
      *out = reinterpret_cast<T*>(kWsAlign + used);  // placeholder, never dereferenced
    }
    used += bytes;
    return hipSuccess;
  }
  template <typename T>
  hipError_t upload(T** out, const std::vector<T>& v) {
    hipError_t e = alloc(out, v.size());
    if (e != hipSuccess) return e;
    if (mode != COUNT && !v.empty()) e = hipMemcpy(*out, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
    return e;
  }
  hipError_t memset(void* p, int val, size_t bytes) { return mode == COUNT ? hipSuccess : hipMemset(p, val, bytes); }
};

struct Inst {
  HostInst hi;
  Schedule sch;
  int grp0 = 0;   // global index of the first group
  int job0 = 0;   // global index of the first job
  int n_grp = 0, n_jobs = 0;
  int n_fblocks = 0;
  // plan-independent device data
  unsigned char* d_active = nullptr;
  double* d_X[2] = {nullptr, nullptr};
  double* d_Xa[2] = {nullptr, nullptr};
  double* d_qmag = nullptr;
  double* d_qbuf = nullptr;     // internal heat-flux output
  double* d_dqbuf = nullptr;    // internal dJ/dQ output
  double* d_blockpart = nullptr;
  int* d_bf_bc = nullptr;
  int* d_bf_cell = nullptr;
  int* d_bc_kind = nullptr;
  double* d_bc_T = nullptr;
  int* d_dface = nullptr;
  double* d_inv_half = nullptr;
  int* d_sface = nullptr;       // specular faces: slot and face direction
  int* d_sface_dir = nullptr;
  int* d_dface_axis = nullptr;  // grid axis of each diffuse face
  double* d_Qs = nullptr;       // heat source of the stored forward state
  double dJds = 0.0;            // dJ/ds of the last adjoint (s: common factor on the cell sizes)
  bool have_dJds = false;
  double* d_adj_scale = nullptr;  // [B][3] wall-value factor of the transposed sweeps
  void* d_ubf = nullptr;        // forward inflow table [B][rows][n_bface]
  void* d_ubf0 = nullptr;       // zeros (adjoint)
  // plan-dependent device data (owned by the plan pool)
  int2* d_sched = nullptr;
  int* d_pos = nullptr;
  int* d_in_slot = nullptr;
  int* d_in_chunk = nullptr;
  int* d_in_tab = nullptr;
  int* d_chunk_fl = nullptr;
  int* d_out_base = nullptr;
  int* d_pre_slot = nullptr;
  int* d_ofk = nullptr;
  int* d_ent_df = nullptr;        // [n_oct][n_out_stride] diffuse face of each out-stream entry, or -1
  double* d_wsum = nullptr;       // [n_oct][B][n_dface] per-octant sums of the diffuse-wall update
  int2* d_grp_ob = nullptr;
  void* d_xq[2] = {nullptr, nullptr};
  void* d_xqa[2] = {nullptr, nullptr};
  void* d_outv = nullptr;
  void* d_part = nullptr;
  int n_part = 0;   // indices of a partial-sum plane (cells, and the padding of its blocks)
  int* d_cell_of = nullptr;  // [n_part] cell of each plane index (NULL: itself)
  int part_bs = 0, part_cs = 0;  // plane-index steps of a block of kC2 columns and of a column
  int2* d_per_base = nullptr;    // 3D rows layout: see period_bases
  int per_stride = 0;
  int part_ld = 0;  // cells per job in a partial-sum plane (n_part padded to cell blocks)
  int part_jg = 0;  // log2 of the jobs per group of a plane
  void* d_store = nullptr;
  double* d_tgrad = nullptr;
  void* d_corr = nullptr;         // second-order faces: [n_grp][pos_per_oct] correction
  double* d_corr_coef = nullptr;  // [n_grp][3]
  int* d_stencil = nullptr;       // [n_oct][pos_per_oct][3*dim] Green-Gauss stencil codes (gather kernel)
  unsigned* d_ccode = nullptr;    // marching kernel: boundary codes, isothermal walls, units, block links
  int* d_cwslot = nullptr;
  int2* d_cunit = nullptr;
  int2* d_clink = nullptr;
  CorrTables ctab;                // host tables of the marching kernel, and whether they hold for the schedule
  bool ctab_made = false, ctab_ok = false;
  int* d_xpre = nullptr;          // 3D rows-per-lane: step-axis wall faces of the first column
  int* d_gpre = nullptr;          // 3D rows-per-lane: lane 0's lane-axis wall faces
  int* d_out_tab = nullptr;       // 3D rows-per-lane: outflow entries per chunk
  int* d_out_chunk = nullptr;     // 3D rows-per-lane: stream offset per chunk
  std::vector<int> grp_band;    // instance-local group -> band
  bool stored = false;
  int fwd_parity = 0;           // parity of the converged forward state
  double T_ref_default = 300.0; // mean temperature of the isothermal walls
  double T_ref = 300.0;         // reference temperature of the current solve
};

}  // namespace

struct bte_ctx {
  int precision = BTE_PREC_FP64;
  int dim = 0, B = 0;
  std::vector<double> v, tau, C;
  std::vector<Ordinate> ords;
  double t0 = 1e-12;
  Plan plan;
  bool plan_set = false;
  bool auto_plan = false;              // the plan is default_plan's (none was set, tuned or read from a cache)
  Plan base_plan;                      // what a plan given in part is completed from while it is
  std::vector<Inst> inst;
  bool has_diffuse = false;
  bool has_specular = false;
  int ubf_rows = 1;                    // inflow-table rows per band: 1, or the ordinate count (specular)
  int2* d_spec_src = nullptr;          // [6][M] mirror of each incoming ordinate (octant, member), or -1
  int2* d_spec_src_a = nullptr;        // [6][M] mirror of each outgoing ordinate (transposed sweeps)
  double* d_spec_iwq = nullptr;        // [6][M] 1 / (w_a' |s_a'.n|) of the mirror a'
  int n_cu = 256;
  std::unique_ptr<DevPool> spool;      // plan-independent arrays
  std::unique_ptr<DevPool> ppool;      // plan-dependent arrays
  // device memory: COUNT until the first call that needs the device (then
  // OWNED) or until a workspace is bound (ARENA)
  DevPool::Mode pool_mode = DevPool::COUNT;
  char* ws_base = nullptr;             // bound workspace
  size_t ws_cap = 0;
  bool ws_store = false;               // the bound workspace holds the adjoint's angular field
  bool ws_lost = false;                // a workspace was bound, but its arrays could not be rebuilt
  size_t need_static = 0, need_plan = 0, need_store = 0;  // workspace bytes of the current plan
  size_t base_need[2] = {0, 0}, base_store[2] = {0, 0};   // those of the base plan, by face order (0: not counted)
  bool part_blocks = true;             // the build at hand orders the cells of its partial-sum planes in
                                       // blocks of columns (see plane_order), else in grid order
  std::map<std::array<int, 6>, bool> part_choice;  // that choice of every plan built so far (see plan_key)
  long long part_extra = 0, store_extra = 0;  // bytes that order adds to need_plan and need_store
  GroupSet gs;                         // ordinate groups of the current plan
  Plan sched_plan;                     // plan the host schedules were built for
  int sched_nr = 0;                    // its NR as asked for
  bool sched_valid = false;
  int order = 1;                       // face reconstruction: 1 first order, 2 second order (deferred correction)
  bool l3r = false;                    // 3D problem swept by the rows-per-lane kernel (else the pencil-block one)
  char dev_name[96] = {0};             // device architecture and CU count (autotune-cache key)
  // shared device arrays (plan-dependent)
  InstDev* d_inst_f = nullptr;
  InstDev* d_inst_a = nullptr;
  JobDev* d_jobs_f = nullptr;
  JobDev* d_jobs_a = nullptr;
  int n_jobs = 0;
  int4* d_gi_f = nullptr;
  int4* d_gi_a = nullptr;
  void* d_gt_f = nullptr;
  void* d_gt_a = nullptr;
  void* d_zg = nullptr;
  long long zg_stride = 0;
  int* d_counters = nullptr;
  FilmInst* d_film = nullptr;          // 1D films swept in one launch per chunk (NULL: not these)
  int film_cells = 0;                  // longest of them
  bool film_reflects = false;          // some end is a diffuse or specular wall
  FinInst* d_fin_f = nullptr;
  FinInst* d_fin_a = nullptr;
  int2* d_fblocks = nullptr;
  int* d_nblocks = nullptr;
  int n_fblocks = 0;
  StatusDev* d_st_f = nullptr;
  StatusDev* d_st_a = nullptr;
  StatusDev* h_st = nullptr;           // pinned
  SweepArgs sa{};
  size_t lds = 0;
  int block = 64, grid = 1;
  int nacc_max = 1;
  size_t lds_stage_plane = 0;
  hipStream_t cap_stream = nullptr;
  // captured iteration chunks, keyed by (adjoint, iterations, tol_T bits, tol_q bits):
  // the tolerances are kernel arguments recorded in the graph
  std::map<std::tuple<int, int, uint64_t, uint64_t>, hipGraphExec_t> graphs;
  std::map<std::tuple<int, int, uint64_t, uint64_t>, hipGraph_t> graph_src;
  std::vector<FinInst> fin_f, fin_a;   // host copies
  ~bte_ctx();
};

namespace {

size_t elem(int prec) { return prec == BTE_PREC_FP32 ? 4 : 8; }

void clear_graphs(bte_ctx* h) {
  for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
  for (auto& kv : h->graph_src) (void)hipGraphDestroy(kv.second);
  h->graphs.clear();
  h->graph_src.clear();
}

}  // namespace

bte_ctx::~bte_ctx() {
  clear_graphs(this);
  if (cap_stream) (void)hipStreamDestroy(cap_stream);
  if (h_st) (void)hipHostFree(h_st);
}

namespace {

std::vector<char> to_prec(const std::vector<double>& x, int prec) {
  std::vector<char> out(x.size() * elem(prec));
  if (prec == BTE_PREC_FP32) {
    float* f = reinterpret_cast<float*>(out.data());
    for (size_t i = 0; i < x.size(); ++i) f[i] = (float)x[i];
  } else {
    memcpy(out.data(), x.data(), x.size() * 8);
  }
  return out;
}

double total_D(const bte_ctx* h) {
  double D = 0.0;
  for (int b = 0; b < h->B; ++b) D += h->C[b] / h->tau[b];
  return D;
}

DevPool* new_pool(bte_ctx* h, size_t offset) {
  if (h->pool_mode == DevPool::ARENA)
    return new DevPool(DevPool::ARENA, h->ws_base + offset, h->ws_cap > offset ? h->ws_cap - offset : 0);
  return new DevPool(h->pool_mode);
}

bte_status finish_plan(bte_ctx* h, const Plan& pl, DevPool& pp);

// Second-order faces: per group (one ordinate a of band b, G = 1) and grid
// axis d, -t0 w0 v_b s_{a,d} / 2, the factor of the Green-Gauss gradient
// difference in the deferred correction (in the sweep's weighted variable:
// w0 is the group's weight in the temperature sum, t0 the time unit).
std::vector<double> corr_coefficients(const bte_ctx* h, const HostInst& hi) {
  const GroupSet& gs = h->gs;
  const int ng = (int)gs.band.size();
  std::vector<double> out((size_t)ng * 3, 0.0);
  double D = 0.0;
  for (int b = 0; b < h->B; ++b) D += h->C[b] / h->tau[b];
  for (int g = 0; g < ng; ++g) {
    const int a = gs.ords[(size_t)g * gs.G];
    if (a < 0) continue;
    const int b = gs.band[g];
    const Ordinate& o = h->ords[a];
    double den = h->t0 / h->tau[b];
    for (int d = 0; d < hi.dim; ++d) den += h->t0 * h->v[b] * std::fabs(o.s[d]) / hi.h[d];
    const double w0 = o.w * h->C[b] / (4.0 * kPi * h->tau[b] * D) / den;
    for (int d = 0; d < hi.dim; ++d) out[(size_t)g * 3 + d] = -h->t0 * w0 * h->v[b] * o.s[d] / 2.0;
  }
  return out;
}

// Order of the cells in a rows-per-lane layout's partial-sum planes: blocks of
// kC2 columns of the step axis (padded to whole blocks), in a block plane after
// plane and row after row, a row's kC2 columns side by side. A wave writes a
// chunk's kC2 columns of 64 lanes at a time, so the 128-byte lines of a plane
// fill within two chunks; in grid order a line waited for the next block of
// columns (3D: a whole block of planes later) and left the L2 in 32-byte
// pieces once the open lines of every workgroup outgrew it (flux sweep of the
// 96x96x120 FinFET-like domain: 8.8 GB written for 4.2 GB of sums; of the 256^2
// square: 515 MB for 189 MB). 24 iterations of the FinFET-like domain went from
// 113.1 to 93.3 ms with it, the square's solve from 9.33 to 9.05 ms. In 1D/2D
// the rows are padded to whole lanes, so a lane's rows past the grid need no
// mask.
PlaneOrder plane_order(const HostInst& hi, const Schedule& S) {
  const bool d3 = hi.dim == 3;
  const int ax[3] = {d3 ? S.ax[0] : 0, d3 ? S.ax[1] : 1, d3 ? S.ax[2] : 2};
  const int st[3] = {1, hi.n[0], hi.n[0] * hi.n[1]};
  PlaneOrder po;
  for (int e = 0; e < 3; ++e) {
    po.n[e] = hi.n[ax[e]];
    po.st[e] = st[ax[e]];
  }
  po.nr = d3 ? po.n[1] : (po.n[1] + S.NR - 1) / S.NR * S.NR;
  po.n_part = (po.n[0] + kC2 - 1) / kC2 * kC2 * po.n[2] * po.nr;
  return po;
}

// 3D: the part of a plane index that a plane period fixes (its block of kC2
// columns, bs apart, and its plane, ps apart; an octant that runs an axis
// backwards counts from its end, with the columns of the last block inside the
// grid as its first) and the columns of its block, 0 for no period. Entry i of
// an octant is period i - kPerPad; the sweep reads up to T / kC2.
std::vector<int2> period_bases(const Schedule& S, const PlaneOrder& po, int bs, int ps, int& stride) {
  const int n_per = S.n_per;
  stride = S.T / kC2 + kPerPad + 1;
  std::vector<int2> pb((size_t)S.n_oct * stride, make_int2(0, 0));
  for (int o = 0; o < S.n_oct; ++o)
    for (int q = 0; q < n_per; ++q) {
      const int b = S.per_b[(size_t)o * n_per + q];
      if (b < 0) continue;
      int pl = S.gpre[(size_t)o * (S.T + n_per) + S.T + q] - 1;
      if ((o >> S.ax[2]) & 1) pl = po.n[2] - 1 - pl;
      pb[(size_t)o * stride + q + kPerPad] =
          make_int2(((o >> S.ax[0]) & 1 ? -b : b) * bs + pl * ps, std::min(kC2, po.n[0] - b * kC2));
    }
  return pb;
}

// Planes a rows-per-lane sweep stages: with one ordinate per lane one plane,
// double-buffered, whatever the sums it writes (they are multiples of it); else
// every sum's, at least two (a single one is double-buffered).
int staged_planes(int G, int nacc) { return G == 1 ? 2 : std::max(2, nacc); }

// (Re)build everything that depends on the plan: schedules, group tables and
// the plan-dependent arrays.
bte_status build_plan_arrays(bte_ctx* h, const Plan& pl_in) {
  Plan pl = pl_in;
  const bool L3 = h->dim == 3;
  // 3D: NR >= 1 asks for the rows-per-lane layout, NR = 0 for the pencil blocks
  const bool R3 = L3 && pl.NR >= 1;
  if (h->order == 2 && (pl.G != 1 || (L3 && !R3))) {
    // the correction array and the stored field hold one ordinate per group,
    // in a rows-per-lane layout
    set_err("second-order faces need plans with G = 1 (in 3D, the rows-per-lane layout)");
    return BTE_ERR_INVALID;
  }
  if (h->has_specular && pl.G != 1) {
    // a specular inflow belongs to one ordinate, and the out-stream entry of a
    // group must hold one ordinate's value
    set_err("specular walls need plans with G = 1");
    return BTE_ERR_INVALID;
  }
  if (R3) {
    pl.R = 1;
    pl.C = kC2;
    if (pl.G != 1) {
      set_err("the 3D rows-per-lane layout takes G = 1 (NR = 0 selects the pencil-block layout)");
      return BTE_ERR_INVALID;
    }
    if (pl.P != 1 && pl.P != 2 && pl.P != 4 && pl.P != 8) {
      set_err("plan P must be 1, 2, 4 or 8 in the 3D rows-per-lane layout");
      return BTE_ERR_INVALID;
    }
  } else if (L3) {
    pl.R = 1;
    pl.NR = 0;
    if (pl.G != 1 && pl.G != 2 && pl.G != 4) {
      set_err("plan G must be 1, 2 or 4");
      return BTE_ERR_INVALID;
    }
    if (pl.C < 8 || pl.C > 64 || pl.C % 8 || pl.C % pl.P) {
      set_err("plan C must be a multiple of 8 in 8..64 and of P");
      return BTE_ERR_INVALID;
    }
  } else {
    // the 1D/2D kernel works in chunks of kC2 steps
    pl.C = kC2;
    if (pl.G != 1 && pl.G != 2) {
      set_err("plan G must be 1 or 2 in 1D/2D");
      return BTE_ERR_INVALID;
    }
    if (pl.NR != 1 && pl.NR != 2 && pl.NR != 4) {
      set_err("plan NR must be 1, 2 or 4");
      return BTE_ERR_INVALID;
    }
    if (pl.P != 1 && pl.P != 2 && pl.P != 4) {
      set_err("plan P must be 1, 2 or 4 in 1D/2D");
      return BTE_ERR_INVALID;
    }
    if (pl.R * pl.P > 4) {
      // the 1D/2D kernel is built for workgroups of at most 256 threads (one
      // wave per SIMD, with the accumulation registers free for its state)
      set_err("plan needs R*P <= 4 in 1D/2D");
      return BTE_ERR_INVALID;
    }
  }
  if (pl.R < 1 || pl.P < 1 || pl.R * pl.P > 8) {
    set_err("plan needs R >= 1, P >= 1, R*P <= 8");
    return BTE_ERR_INVALID;
  }
  clear_graphs(h);
  h->ppool.reset();
  h->ppool.reset(new_pool(h, h->need_static));
  DevPool& pp = *h->ppool;
  const int prec = h->precision;
  const size_t es = elem(prec);
  // (a schedule knows nothing of the groups; in the 3D rows layout the NR asked
  // for may have been raised)
  const bool reuse_groups = h->sched_valid && h->sched_plan.G == pl.G && h->sched_plan.P == pl.P;
  const bool reuse_sched = h->sched_valid && h->l3r == R3 && h->sched_plan.R == pl.R && h->sched_plan.C == pl.C &&
                           (h->sched_plan.NR == pl.NR || (R3 && h->sched_nr == pl.NR));
  h->sched_valid = false;
  if (!reuse_groups) h->gs = build_groups(h->ords, h->B, h->dim, pl.G, pl.P);
  const GroupSet& gs = h->gs;
  if (!reuse_sched) h->sched_nr = pl.NR;
  else if (R3) pl.NR = h->sched_plan.NR;
  if (R3 && !reuse_sched) {
    // rows-per-lane schedules of every instance, with one NR for all (the
    // kernel's shape): the largest any instance needs
    int nr = std::min(std::max(pl.NR, 1), 2);
    for (int pass = 0; pass < 2; ++pass) {
      Plan p3 = pl;
      p3.NR = nr;
      int nrmax = 1;
      for (auto& I : h->inst) {
        std::string err;
        if (!build_schedule_3r(I.hi, p3, I.sch, err)) {
          set_err("%s", err.c_str());
          return BTE_ERR_INVALID;
        }
        nrmax = std::max(nrmax, I.sch.NR);
      }
      if (nrmax == nr) break;
      nr = nrmax;
    }
    pl.NR = nr;
  }
  h->l3r = R3;
  const int n_grp_inst = (int)gs.band.size();
  const int n_bund = (int)gs.bundle_first.size();
  const int n_oct = 1 << h->dim;
  std::vector<InstDev> idf(h->inst.size()), ida(h->inst.size());
  std::vector<JobDev> jf, ja;
  std::vector<int4> gif, gia;
  std::vector<double> gtf, gta;
  int W_max = 1, e_max = 1, o_max = 1;
  int grp_tot = 0;
  // accumulator planes: the temperature, and the heat flux or dJ/dQ.
  // Second-order sweeps carry three planes on flux iterations in 1D too (the
  // y-flux plane then holds zeros): one compiled variant per shape
  h->nacc_max = std::max(1 + h->dim, h->order == 2 ? 3 : 2);
  const bool rows = !L3 || R3;
  h->part_extra = h->store_extra = 0;
  auto al256 = [](size_t x) { return (long long)((x + kWsAlign - 1) / kWsAlign * kWsAlign); };
  std::vector<int2> fb;   // finalize blocks
  std::vector<int> nbi;
  for (size_t k = 0; k < h->inst.size(); ++k) {
    Inst& I = h->inst[k];
    std::string err;
    if (!reuse_sched && !R3 && !build_schedule(I.hi, pl, I.sch, err)) {
      set_err("%s", err.c_str());
      return BTE_ERR_INVALID;
    }
    const Schedule& S = I.sch;
    if (!reuse_sched || !reuse_groups) I.ctab_made = false;
    if (h->has_specular) {
      // every mirror ordinate must find its outflow entry at each specular face
      const int nbf = (int)I.hi.bf_cell.size();
      for (int sf : I.hi.sface) {
        const int fd = I.hi.bf_face[sf], d = fd / 2;
        for (const auto& oa : h->ords) {
          // forward: the outgoing ordinates' octants; transposed sweeps: the
          // flipped octants of the incoming ones
          const double sn = (fd & 1) ? oa.s[d] : -oa.s[d];
          if (sn == 0.0) continue;
          const int os = sn > 0.0 ? oa.oct : oa.oct ^ (n_oct - 1);
          if (S.ofk[(size_t)os * nbf + sf] < 0) {
            set_err("internal: specular face %d has no outflow entry in octant %d", sf, os);
            return BTE_ERR_INVALID;
          }
        }
      }
    }
    W_max = std::max(W_max, S.W);
    e_max = std::max(e_max, S.e_max);
    o_max = std::max(o_max, S.o_max);
    I.grp0 = grp_tot;
    I.n_grp = n_grp_inst;
    I.n_jobs = n_bund;
    I.grp_band = gs.band;
    grp_tot += n_grp_inst;
    // group tables
    std::vector<double> cf, ca;
    group_coefficients(gs, h->ords, I.hi, h->v, h->tau, h->C, h->t0, false, cf);
    group_coefficients(gs, h->ords, I.hi, h->v, h->tau, h->C, h->t0, true, ca);
    gtf.insert(gtf.end(), cf.begin(), cf.end());
    gta.insert(gta.end(), ca.begin(), ca.end());
    for (int g = 0; g < n_grp_inst; ++g) {
      // forward inflow-table row: the band, or (band, ordinate) with specular
      // walls (G = 1; padding groups read ordinate 0's row, their weights are 0)
      int row = gs.band[g];
      if (h->has_specular) row = gs.band[g] * h->ubf_rows + std::max(0, gs.ords[(size_t)g * pl.G]);
      gif.push_back(make_int4(gs.band[g], gs.oct[g], g, row));
      // the adjoint has its own table (zero on isothermal faces), same rows
      gia.push_back(make_int4(gs.band[g], gs.oct[g] ^ (n_oct - 1), g, row));
    }
    // device arrays of the schedule
    I.n_part = I.hi.ncell;
    I.d_cell_of = nullptr;
    int row_step = L3 ? 0 : I.hi.n[0];
    if (L3) row_step = std::vector<int>{1, I.hi.n[0], I.hi.n[0] * I.hi.n[1]}[S.ax[1]];
    HIPCHK(pp.upload(&I.d_sched, S.sched));
    PlaneOrder po;
    if (rows) po = plane_order(I.hi, S);
    const bool blocks = rows && h->part_blocks && po.n_part < (1 << 26);  // (a record holds the index << 5)
    if (blocks) {
      I.n_part = po.n_part;
      row_step = kC2;
      // (the tables in this order are made on the device, below)
      HIPCHK(pp.alloc(&I.d_pos, (size_t)S.n_oct * I.n_part));
      HIPCHK(pp.alloc(&I.d_cell_of, I.n_part));
      h->part_extra += al256((size_t)S.n_oct * I.n_part * 4) - al256(S.pos.size() * 4) + al256((size_t)I.n_part * 4);
    } else {
      HIPCHK(pp.upload(&I.d_pos, S.pos));
    }
    // the sweep's own form of the plane index: column blocks and columns, and
    // in 3D the part of every plane period's block and plane
    I.part_bs = blocks ? po.nr * po.n[2] * kC2 : kC2 * (L3 ? po.st[0] : 1);
    I.part_cs = blocks || !L3 ? 1 : po.st[0];
    I.d_per_base = nullptr;
    I.per_stride = 0;
    if (rows && L3) {
      const std::vector<int2> pb = period_bases(S, po, I.part_bs, blocks ? po.nr * kC2 : po.st[2], I.per_stride);
      HIPCHK(pp.upload(&I.d_per_base, pb));
      h->part_extra += al256(pb.size() * sizeof(int2));
    }
    if (!rows) {
      HIPCHK(pp.upload(&I.d_in_slot, S.in_slot));
      HIPCHK(pp.upload(&I.d_in_chunk, S.in_chunk));
    }
    I.n_fblocks = (I.n_part + kFinCells - 1) / kFinCells;
    HIPCHK(pp.alloc(&I.d_blockpart, (size_t)I.n_fblocks * 4));
    for (int b = 0; b < I.n_fblocks; ++b) fb.push_back(make_int2((int)k, b));
    nbi.push_back(I.n_fblocks);
    h->fin_f[k].blockpart = h->fin_a[k].blockpart = I.d_blockpart;
    HIPCHK(pp.upload(&I.d_in_tab, S.in_tab));
    std::vector<int> cfl(S.chunk_fl);
    if (rows) {
      const int nch = S.T / kC2;
      for (size_t s1 = 0; s1 < cfl.size() / (nch + 1); ++s1)
        for (int c = 0; c < nch; ++c)
          cfl[s1 * (nch + 1) + c] |=
              (S.in_chunk[s1 * (nch + 1) + c + 1] - S.in_chunk[s1 * (nch + 1) + c] + 63) / 64 << 8;
    }
    HIPCHK(pp.upload(&I.d_chunk_fl, cfl));
    HIPCHK(pp.upload(&I.d_out_base, S.out_base));
    HIPCHK(pp.upload(&I.d_pre_slot, S.pre_slot));
    HIPCHK(pp.upload(&I.d_ofk, S.ofk));
    // diffuse-wall update: the diffuse face of each out-stream entry of each
    // octant (-1: another face), and the per-octant band sums of those faces
    I.d_ent_df = nullptr;
    I.d_wsum = nullptr;
    if (!I.hi.dface.empty()) {
      const int nbf = (int)I.hi.bf_cell.size();
      std::vector<int> df_of(nbf, -1);
      for (size_t i = 0; i < I.hi.dface.size(); ++i) df_of[I.hi.dface[i]] = (int)i;
      std::vector<int> ent((size_t)n_oct * S.n_out_stride, -1);
      for (int oo = 0; oo < n_oct; ++oo)
        for (int f = 0; f < nbf; ++f) {
          const int e = S.ofk[(size_t)oo * nbf + f];
          if (e >= 0 && df_of[f] >= 0) ent[(size_t)oo * S.n_out_stride + e] = df_of[f];
        }
      HIPCHK(pp.upload(&I.d_ent_df, ent));
      HIPCHK(pp.alloc(&I.d_wsum, (size_t)n_oct * h->B * I.hi.dface.size()));
    }
    I.d_xpre = nullptr;
    I.d_gpre = nullptr;
    I.d_out_tab = nullptr;
    I.d_out_chunk = nullptr;
    if (S.l3r) {
      HIPCHK(pp.upload(&I.d_xpre, S.xpre));
      HIPCHK(pp.upload(&I.d_gpre, S.gpre));
      // the entries by their place in the kernel's staging
      std::vector<int> otab(S.out_tab);
      for (int& e : otab)
        if (e > 0) {
          const int idx = (e - 1) >> 2, row = 64 * S.NR;
          e = (idx / row * stage_row(S.NR, (int)es) + idx % row) << 3 | ((e - 1) & 3) << 1 | 1;
        }
      HIPCHK(pp.upload(&I.d_out_tab, otab));
      HIPCHK(pp.upload(&I.d_out_chunk, S.out_chunk));
    }
    std::vector<int2> gob(n_oct * h->B);
    for (int i = 0; i < n_oct * h->B; ++i) gob[i] = make_int2(gs.ob_first[i], gs.ob_count[i]);
    HIPCHK(pp.upload(&I.d_grp_ob, gob));
    const size_t nposb = (size_t)S.pos_per_oct * S.n_oct * 2 * es;
    for (int b = 0; b < 2; ++b) {
      char* p1;
      char* p2;
      HIPCHK(pp.alloc(&p1, nposb));
      HIPCHK(pp.alloc(&p2, nposb));
      HIPCHK(pp.memset(p1, 0, nposb));
      HIPCHK(pp.memset(p2, 0, nposb));
      I.d_xq[b] = p1;
      I.d_xqa[b] = p2;
    }
    char* ov;
    HIPCHK(pp.alloc(&ov, (size_t)n_grp_inst * S.n_out_stride * es));
    I.d_outv = ov;
    char* pt;
    I.part_ld = (I.n_part + kPartBlk - 1) / kPartBlk * kPartBlk;
    // job groups: 1D/2D planes, and 3D ones up to 256 MiB, keep one job per
    // group (each job's cells contiguous); larger 3D ones group as many jobs
    // as keep a group's part of a plane within the 32-bit offsets of a buffer
    // view (no more than the jobs there are), so that a finalize block reads
    // long contiguous runs
    I.part_jg = 0;
    if (h->dim == 3 && (size_t)I.part_ld * n_bund * es > (256ull << 20))
      while ((1 << I.part_jg) < n_bund && ((size_t)I.part_ld << (I.part_jg + 1)) * es < (1ull << 31)) ++I.part_jg;
    // (in blocks of columns the planes also hold the grid-order positions for a
    // moment, one per octant and cell: more than the sums where few octants have
    // ordinates, as with directions along the axes only)
    const size_t part_bytes = std::max<size_t>((size_t)h->nacc_max * part_plane_len(n_bund, I.part_jg, I.part_ld) * es,
                                               blocks ? S.pos.size() * 4 : 0);
    HIPCHK(pp.alloc(&pt, part_bytes));
    I.d_part = pt;
    if (blocks && pp.mode != DevPool::COUNT) {
      // the null stream orders the kernel before the copies that follow
      HIPCHK(hipMemcpy(I.d_part, S.pos.data(), S.pos.size() * 4, hipMemcpyHostToDevice));
      HIPCHK(launch_plane_tables(po, I.hi.ncell, S.n_oct, reinterpret_cast<const int*>(I.d_part), I.d_pos, I.d_cell_of,
                                 I.d_sched, (long long)S.sched.size(), nullptr));
    }
    const int ld0 = (I.hi.ncell + kPartBlk - 1) / kPartBlk * kPartBlk;
    h->part_extra += al256(part_bytes) - al256((size_t)h->nacc_max * part_plane_len(n_bund, I.part_jg, ld0) * es);
    h->store_extra += al256((size_t)n_grp_inst * I.n_part * pl.G * es) -
                      al256((size_t)n_grp_inst * I.hi.ncell * pl.G * es);
    I.d_store = nullptr;
    I.stored = false;
    I.have_dJds = false;
    HIPCHK(pp.alloc(&I.d_tgrad, (size_t)n_grp_inst * 2));
    I.d_corr = nullptr;
    if (h->order == 2) {
      char* pc;
      const size_t nc = (size_t)n_grp_inst * S.pos_per_oct * es;
      HIPCHK(pp.alloc(&pc, nc));
      HIPCHK(pp.memset(pc, 0, nc));  // positions of no cell stay 0
      I.d_corr = pc;
      char* ps;  // the field, in the same layout
      HIPCHK(pp.alloc(&ps, nc));
      I.d_store = ps;
      HIPCHK(pp.upload(&I.d_corr_coef, corr_coefficients(h, I.hi)));
      // one strip: the marching kernel's tables; else (or should a neighbour
      // not sit where that kernel looks for it) the gather kernel's stencil
      const CorrTables& ct = I.ctab;
      if (!I.ctab_made) I.ctab_ok = corr_tables(I.hi, S, n_grp_inst, I.ctab);
      I.ctab_made = true;
      I.d_stencil = nullptr;
      I.d_ccode = nullptr;
      if (I.ctab_ok) {
        HIPCHK(pp.upload(&I.d_ccode, ct.code));
        HIPCHK(pp.upload(&I.d_cwslot, ct.wslot));
        HIPCHK(pp.upload(&I.d_cunit, ct.unit));
        HIPCHK(pp.upload(&I.d_clink, ct.link));
      } else {
        HIPCHK(pp.upload(&I.d_stencil, corr_stencil(I.hi, S)));
      }
    }
    // descriptors
    for (int adj = 0; adj < 2; ++adj) {
      InstDev& d = adj ? ida[k] : idf[k];
      memset(&d, 0, sizeof(d));
      d.dim = I.hi.dim;
      d.nx = I.hi.n[0];
      d.ny = I.hi.n[1];
      d.nz = I.hi.n[2];
      d.ncell = I.hi.ncell;
      d.n_bface = (int)I.hi.bf_cell.size();
      d.n_jobs = n_bund;
      d.n_grp = n_grp_inst;
      d.T = S.T;
      d.n_oct = S.n_oct;
      d.W = S.W;
      d.e_max = S.e_max;
      d.o_max = S.o_max;
      d.pos_per_oct = S.pos_per_oct;
      d.sched = I.d_sched;
      d.pos = I.d_pos;
      d.in_slot = I.d_in_slot;
      d.in_chunk = I.d_in_chunk;
      d.out_base = I.d_out_base;
      d.pre_slot = I.d_pre_slot;
      d.xq[0] = adj ? I.d_xqa[0] : I.d_xq[0];
      d.xq[1] = adj ? I.d_xqa[1] : I.d_xq[1];
      d.xf = I.d_xq[0];
      d.ubf = adj ? I.d_ubf0 : I.d_ubf;
      d.outv = I.d_outv;
      d.part = I.d_part;
      d.n_part = I.n_part;
      d.part_bs = I.part_bs;
      d.part_cs = I.part_cs;
      d.per_base = I.d_per_base;
      d.per_stride = I.per_stride;
      d.cell_of = I.d_cell_of;
      d.part_ld = I.part_ld;
      d.part_jg = I.part_jg;
      d.store_u = (!adj && h->order == 2) ? I.d_store : nullptr;
      d.corr = adj ? nullptr : I.d_corr;
      d.tgrad = I.d_tgrad;
      d.status = reinterpret_cast<int*>((adj ? h->d_st_a : h->d_st_f) + k);
      d.lag = S.lag;
      d.ring = S.ring;
      d.n_out_stride = S.n_out_stride;
      d.nr = S.NR;
      d.du = S.du;
      d.n_strip = S.nS;
      d.in_E = S.in_E;
      d.in_tab = I.d_in_tab;
      d.chunk_fl = I.d_chunk_fl;
      for (int e = 0; e < 3; ++e) d.ax[e] = S.ax[e];
      for (int oo = 0; oo < 8; ++oo) {
        // the groups of the transposed sweeps run the flipped octant's schedule,
        // and the kernel indexes with its job's (schedule) octant
        d.dyo[oo] = ((oo >> (L3 ? S.ax[1] : 1)) & 1 ? -1 : 1) * row_step;
      }
      d.n_pl = S.n_pl;
      d.n_per = S.n_per;
      d.xpre = I.d_xpre;
      d.gpre = I.d_gpre;
      d.out_tab = I.d_out_tab;
      d.out_chunk = I.d_out_chunk;
      d.out_E = S.out_E;
    }
    for (int b = 0; b < n_bund; ++b) {
      const int o = gs.bundle_oct[b];
      jf.push_back(JobDev{(int)k, I.grp0 + gs.bundle_first[b], b, o});
      ja.push_back(JobDev{(int)k, I.grp0 + gs.bundle_first[b], b, o ^ (n_oct - 1)});
    }
  }
  // (schedules and groups hold whatever becomes of the rest: a plan refused for
  // its LDS leaves them to the one that follows)
  h->sched_plan = pl;
  h->sched_valid = true;
  // larger instances first (the queue hands out jobs in order)
  auto work = [&](const JobDev& j) { return (long long)h->inst[j.inst].sch.T * h->inst[j.inst].sch.R; };
  std::stable_sort(jf.begin(), jf.end(), [&](const JobDev& a, const JobDev& b) { return work(a) > work(b); });
  std::stable_sort(ja.begin(), ja.end(), [&](const JobDev& a, const JobDev& b) { return work(a) > work(b); });
  h->n_jobs = (int)jf.size();
  h->n_fblocks = (int)fb.size();
  HIPCHK(pp.upload(&h->d_fblocks, fb));
  HIPCHK(pp.upload(&h->d_nblocks, nbi));
  if (pp.mode != DevPool::COUNT) {
    HIPCHK(hipMemcpy(h->d_fin_f, h->fin_f.data(), h->fin_f.size() * sizeof(FinInst), hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(h->d_fin_a, h->fin_a.data(), h->fin_a.size() * sizeof(FinInst), hipMemcpyHostToDevice));
  }
  HIPCHK(pp.upload(&h->d_inst_f, idf));
  HIPCHK(pp.upload(&h->d_inst_a, ida));
  HIPCHK(pp.upload(&h->d_jobs_f, jf));
  HIPCHK(pp.upload(&h->d_jobs_a, ja));
  HIPCHK(pp.upload(&h->d_gi_f, gif));
  HIPCHK(pp.upload(&h->d_gi_a, gia));
  {
    std::vector<char> a = to_prec(gtf, prec), b = to_prec(gta, prec);
    char* pa;
    char* pb;
    HIPCHK(pp.upload(&pa, a));
    HIPCHK(pp.upload(&pb, b));
    h->d_gt_f = pa;
    h->d_gt_a = pb;
  }
  // 1D films in one launch per chunk (bte_film.hip): unmasked, first-order
  // faces, one ordinate per group, within the kernel's registers and LDS.
  // Iterations in us, the general kernels' and this one's: 120 cells, 96 groups
  // FP32 30.6 and 8.0, FP64 33.0 and 7.9; 960 groups FP32 39.4 and 39.7, FP64
  // 53.6 and 38.7; 1000 cells, 96 groups FP32 140 and 18.7, 960 groups 148 and
  // 96.7. One workgroup sweeps a whole film, so its time goes with the groups,
  // and in double whatever the precision: a single film in FP32 of up to 256
  // cells with more than four groups per CU takes the general kernels where the
  // lines fitted to such times put them first (1600 groups: 4 cells 35.4 and
  // 56.1, 128 cells 46.9 and 61.4, 250 cells 65.1 and 71.9; 180 cells, 1050
  // groups 50.8 and 49.0)
  h->d_film = nullptr;
  h->film_cells = 0;
  h->film_reflects = false;
  if (h->dim == 1 && pl.G == 1 && h->order == 1) {
    bool ok = true;
    std::vector<FilmInst> film;
    for (const auto& I : h->inst) {
      const int n = I.hi.ncell;
      ok = ok && I.hi.n_active == n && n <= kFilmCells;
      h->film_cells = std::max(h->film_cells, n);
      FilmInst f{};
      for (int e = 0; e < 2 && ok; ++e) {
        f.slot[e] = I.hi.bslot[(size_t)(e ? n - 1 : 0) * 6 + e];
        f.kind[e] = I.hi.bc_kind[I.hi.bf_bc[f.slot[e]]];
        f.inv_half[e] = 1.0 / half_range(h->ords, 0);
        if (f.kind[e] != BTE_BC_ISOTHERMAL) h->film_reflects = true;
      }
      film.push_back(f);
    }
    const int cpl = film_cpl(h->film_cells);
    ok = ok && film_lds_bytes(cpl, n_grp_inst) <= kFilmLds;
    if (prec == BTE_PREC_FP32 && h->inst.size() == 1 && n_grp_inst > 4 * h->n_cu && cpl <= 4) {
      const double per_grp = cpl == 1 ? 0.034 : cpl == 2 ? 0.038 : 0.0445;
      ok = ok && 3.0 + per_grp * n_grp_inst <= 13.0 + 0.13 * h->film_cells + 0.0125 * n_grp_inst;
    }
    if (ok) HIPCHK(pp.upload(&h->d_film, film));
  }
  // LDS carve-up
  const int R = L3 ? 1 : pl.R, P = pl.P, G = pl.G, Cc = pl.C;
  auto al = [](size_t x) { return (x + 15) / 16 * 16; };
  size_t off = 0;
  SweepArgs& sa = h->sa;
  memset(&sa, 0, sizeof(sa));
  if (!L3 || R3) {
    // 1D/2D: ring [P][R][W_max + 1][G], cell ids [2][R][kC2][72], inflow
    // [P*R][2][E], outflow [P*R][o_max], staging [planes][P*R][kC2][64*NR + 8
    // dwords] (staged_planes)
    int E = 64;
    for (auto& I : h->inst) E = std::max(E, I.sch.in_E);
    // (the 3D rows layout has no strip ring, forms its plane indices from the
    // period table and emits its outflows from the staging: none takes LDS)
    sa.lds_zring = (int)off;
    off += R3 ? 0 : al((size_t)P * R * (W_max + 1) * G * es);
    sa.lds_cid = (int)off;
    off += R3 ? 0 : al((size_t)2 * R * kC2 * (64 + 8) * 4);  // records, rows padded to 72 ints
    sa.lds_in = (int)off;
    off += al((size_t)P * R * 2 * E * es);
    sa.lds_out = (int)off;
    off += R3 ? 0 : al((size_t)P * R * o_max * es);
    sa.lds_stage = (int)off;
    h->lds_stage_plane = al((size_t)P * R * kC2 * stage_row(pl.NR, (int)es) * es);
    off += (size_t)staged_planes(G, h->nacc_max) * h->lds_stage_plane;
    sa.lds_total = (int)off;
    if (R3 && es == 8 && pl.NR == 2 && P == 8) {
      // never offered: the planes of every sum did not fit. With one plane
      // staged small boundary tables leave it the LDS, and though its 256
      // registers spill it is the faster at first order (100x100x30, 1920
      // groups 3076 -> 2215 us an iteration, 20x70x20 441 -> 435; second order
      // 1364 -> 1429); what was refused stays refused
      set_err("eight waves with two FP64 rows per lane need %zu bytes of LDS and spill registers: P is at most 4", off);
      return BTE_ERR_INVALID;
    }
    if (off > 160 * 1024 - 64) {
      set_err("plan needs %zu bytes of LDS (limit 160 KiB): reduce P, R, NR or G", off);
      return BTE_ERR_INVALID;
    }
    h->lds = off;
    sa.inst = h->d_inst_f;
    sa.jobs = h->d_jobs_f;
    sa.n_jobs = h->n_jobs;
    sa.counters = h->d_counters;
    sa.grp_i = h->d_gi_f;
    sa.grp_t = h->d_gt_f;
    sa.B = h->B;
    sa.R = R;
    sa.P = P;
    sa.C = kC2;
    sa.zring_len = W_max;
    sa.W_max = W_max;
    sa.e_max = E;
    sa.o_max = o_max;
    h->block = R * P * 64;
    int bpc = R3 ? sweep3r_blocks_per_cu(prec, pl.NR, P, 1, SWEEP_PLAIN, h->block,
                                         sa.lds_stage + 2 * h->lds_stage_plane)
                 : sweep2d_blocks_per_cu(prec, G, pl.NR, P, 1, SWEEP_PLAIN, h->block,
                                         sa.lds_stage + 2 * h->lds_stage_plane);
    if (bpc < 1) bpc = 1;
    h->grid = std::max(1, std::min(h->n_jobs, bpc * h->n_cu));
    if (R3) {
      // the step-axis buffers: one value per plane, lane and row, per
      // (workgroup, wave p)
      int npl = 1;
      for (auto& I : h->inst) npl = std::max(npl, I.sch.n_pl);
      h->zg_stride = (long long)npl * 64 * pl.NR;
      char* zg;
      const size_t zb = (size_t)h->grid * P * h->zg_stride * es;
      HIPCHK(pp.alloc(&zg, zb));
      HIPCHK(pp.memset(zg, 0, zb));
      h->d_zg = zg;
      sa.zg = zg;
      sa.zg_stride = h->zg_stride;
    }
    return finish_plan(h, pl, pp);
  }
  sa.lds_zring = (int)off;
  off += al(L3 ? 0 : (size_t)P * R * W_max * G * es);
  sa.lds_yring = (int)off;
  off += al(L3 ? (size_t)P * (8 * W_max + 64) * G * es : 0);  // + one dummy entry per lane
  sa.lds_xb = (int)off;
  off += al(L3 ? (size_t)P * 72 * G * es : 0);
  sa.lds_cid = (int)off;
  off += al((size_t)R * Cc * 65 * 4);
  sa.lds_in = (int)off;
  off += al((size_t)P * R * 2 * e_max * es);
  sa.lds_out = (int)off;
  off += al((size_t)P * R * (o_max + 64) * es);
  // the partial-sum staging goes last: its size depends on the number of
  // accumulator planes of the launched variant
  sa.lds_stage = (int)off;
  h->lds_stage_plane = al((size_t)P * R * Cc * 65 * es);
  off += (size_t)h->nacc_max * h->lds_stage_plane;
  sa.lds_total = (int)off;
  if (off > 160 * 1024 - 64) {
    set_err("plan needs %zu bytes of LDS (limit 160 KiB): reduce P, R, C or G", off);
    return BTE_ERR_INVALID;
  }
  h->lds = off;
  sa.inst = h->d_inst_f;
  sa.jobs = h->d_jobs_f;
  sa.n_jobs = h->n_jobs;
  sa.counters = h->d_counters;
  sa.grp_i = h->d_gi_f;
  sa.grp_t = h->d_gt_f;
  sa.B = h->B;
  sa.R = R;
  sa.P = P;
  sa.C = Cc;
  sa.zring_len = W_max;
  sa.W_max = W_max;
  sa.e_max = e_max;
  sa.o_max = o_max;
  h->block = R * P * 64;
  int bpc = sweep_blocks_per_cu(prec, L3, G, 1, SWEEP_PLAIN, h->block, sa.lds_stage + h->lds_stage_plane);
  if (bpc < 1) bpc = 1;
  h->grid = std::max(1, std::min(h->n_jobs, bpc * h->n_cu));
  if (L3) {
    int ring = 1;
    for (auto& I : h->inst) ring = std::max(ring, I.sch.ring);
    h->zg_stride = (long long)ring * 8 * G;
    char* zg;
    const size_t zb = (size_t)h->grid * P * h->zg_stride * es;
    HIPCHK(pp.alloc(&zg, zb));
    HIPCHK(pp.memset(zg, 0, zb));
    h->d_zg = zg;
    sa.zg = zg;
    sa.zg_stride = h->zg_stride;
  }
  return finish_plan(h, pl, pp);
}

// Plan-dependent arrays whose carving is sized in build_plan: records the
// plan and its workspace bytes.
bte_status finish_plan(bte_ctx* h, const Plan& pl, DevPool& pp) {
  h->plan = pl;
  h->need_plan = pp.used;
  // the angular field kept for the adjoint: part of a bound workspace when it
  // was sized for it, else allocated by the first solve that stores it
  const size_t es = elem(h->precision);
  size_t st = 0;
  for (auto& I : h->inst)
    st += ((size_t)I.n_grp * I.n_part * pl.G * es + kWsAlign - 1) / kWsAlign * kWsAlign;
  h->need_store = st;
  if (h->pool_mode == DevPool::ARENA && h->ws_store && h->order == 1) {
    for (auto& I : h->inst) {
      char* p;
      HIPCHK(pp.alloc(&p, (size_t)I.n_grp * I.n_part * pl.G * es));
      I.d_store = p;
    }
  }
  return BTE_OK;
}

// Device workspace of bte_solve_noalloc (below): the largest need it accepts.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;

// What the choice of the planes' order depends on, beside the problem.
std::array<int, 6> plan_key(const bte_ctx* h, const Plan& pl) { return {h->order, pl.G, pl.R, pl.P, pl.C, pl.NR}; }

// The plan's arrays with the partial-sum planes in blocks of columns, or in
// grid order where the blocks' padding alone would push the need past the
// allocation-free solve's fixed array (with or without the angular field).
bte_status build_plan_impl(bte_ctx* h, const Plan& pl) {
  // (a plan's choice holds whenever the plan is built again, when it was only
  // counted before or returned to after another was rejected: a workspace was
  // sized for it)
  const auto key = plan_key(h, pl);
  const auto known = h->part_choice.find(key);
  h->part_blocks = known == h->part_choice.end() || known->second;
  bte_status s = build_plan_arrays(h, pl);
  if (s != BTE_OK || known != h->part_choice.end()) return s;
  const long long lim = (long long)kStaticScratchBytes, need = (long long)(h->need_static + h->need_plan);
  const long long with = need + (long long)h->need_store;
  if ((need > lim && need - h->part_extra <= lim) ||
      (with > lim && with - h->part_extra - h->store_extra <= lim)) {
    h->part_blocks = false;
    s = build_plan_arrays(h, pl);
    if (s != BTE_OK) return s;
  }
  h->part_choice.emplace(key, h->part_blocks);
  h->part_choice.emplace(plan_key(h, h->plan), h->part_blocks);  // (as it was completed)
  return s;
}

// The plan a new handle had before its shape is looked at: in 3D the
// rows-per-lane layout, P waves of one octant per workgroup; in 1D/2D one strip
// of 64*NR rows, which covers ny <= 256.
Plan basic_plan(const bte_ctx* h) {
  Plan pl;
  pl.G = 1;
  pl.R = 1;
  pl.C = kC2;
  if (h->dim == 3) {
    pl.P = h->precision == BTE_PREC_FP32 ? 8 : 4;
    pl.NR = 1;
  } else {
    int ny = 1;
    for (auto& I : h->inst) ny = std::max(ny, I.hi.n[1]);
    pl.NR = ny <= 64 ? 1 : ny <= 128 ? 2 : 4;
    pl.P = h->precision == BTE_PREC_FP32 ? 4 : 2;
  }
  return pl;
}

// The plan of a handle that none was given to, by the groups (bands times
// ordinates, of all instances) against the 256 CUs. Times of one iteration in
// us, the basic plan's and this one's:
//   2D, ny <= 128, FP64: four waves share a plane instead of two. 64^2, 160
//     groups 40.8 -> 39.4, 960 groups 66.0 -> 53.2; 128^2, 960 groups
//     88.3 -> 73.4; a masked 60x100, 480 groups 86.0 -> 80.6; second-order
//     128^2, 960 groups 277 -> 230 (64^2, 160 groups 59.6 -> 60.2). Not below
//     0.6 groups per CU (109x63 with specular walls, 80 groups 73.7 -> 76.6,
//     144 groups 77.8 -> 78.8).
//   2D, 128 < ny <= 256, first order (second-order sweeps march along single
//     strips of four rows per lane):
//     walls inside or reflecting ones: most chunks then have boundary entries,
//       whose work is per row of a lane, and a step of two slots of two rows
//       takes 0.72 of the time of one of four while each workgroup of four
//       waves has a CU (up to 512 groups); narrow sections have too many more
//       steps that way (52x246: 89 -> 93). Masked 193x131, 480 groups: FP64 178 -> 158, FP32
//       162 -> 143; 240x250: 241 -> 220, 202 -> 178; a rectangle of 240x250 with
//       diffuse walls, 160 groups: 196 -> 175, 179 -> 158; at 960 groups it is
//       slower (FP64 326 -> 389, FP32 192 -> 204).
//     FP64 else, more than two groups per CU: two rows per lane in one slot,
//       four waves to a plane. 256^2, 960 groups 302 -> 190 (four rows and four
//       waves: 182); at fewer it wins or loses with the size (256^2, 480 groups
//       161 -> 153, but the solve and adjoint of 183^2, 448 groups 23.0 -> 25.1 ms).
//   2D, first order, more than four groups per CU (batches): with several
//     workgroups to a CU a step's time goes with its rows, so the rows per lane
//     are those with the least steps times the measured cost of one (FP32 0.37 :
//     0.53 : 1 for 1, 2 and 4 rows, FP64 0.28 : 0.52 : 1; four waves to a plane).
//     FP64 takes one or two: four rows have LDS for one such workgroup on a CU
//     only (256^2, 3840 groups 743 with two rows, 711 with four; 200x300, 1920
//     groups 378 with one, 481 with two, 493 with four). Batches of squares of
//     33 to 159 rows and columns: 64 in FP32 1406 -> 981, 8 in FP32 183 -> 131,
//     24 in FP64 1082 -> 619.
//   3D: FP32 with no more groups than CUs: 4 waves share a plane instead of 8.
//     37x29x23, 160 groups 181 -> 176, 60x60x50, 256 groups 639 -> 628; 46x45x35,
//     512 groups 552 -> 561. FP64 with more than four groups per CU: 8 instead
//     of 4. 46x45x35, 1920 groups 1197 -> 1018; 23x23x18, 960 groups 211 -> 225.
//     (Two rows per lane in FP64 are not offered with 8 and stay with 4.)
Plan default_plan(const bte_ctx* h, int order) {
  Plan pl = basic_plan(h);
  const long long n = (long long)h->B * (long long)h->ords.size() * (long long)h->inst.size(), cu = h->n_cu;
  const bool f64 = h->precision != BTE_PREC_FP32;
  if (h->dim == 3) {
    if (!f64 && n <= cu) pl.P = 4;
    if (f64 && n > 4 * cu) pl.P = 8;
  } else if (h->dim == 2) {
    int lo = 1 << 30, hi = 0;
    bool walls = h->has_diffuse || h->has_specular;
    for (auto& I : h->inst) {
      lo = std::min(lo, I.hi.n[1]);
      hi = std::max(hi, I.hi.n[1]);
      walls = walls || I.hi.n_active < I.hi.ncell;
    }
    if (order == 1 && n > 4 * cu) {
      const double cost[2][3] = {{0.37, 0.53, 1.0}, {0.28, 0.52, 1.0}};  // of a step, by NR
      double best = 0.0;
      for (int i = 0; i < (f64 ? 2 : 3); ++i) {
        double t = 0.0;
        for (auto& I : h->inst) t += cost[f64][i] * schedule_steps_2d(I.hi.n[0], I.hi.n[1], 1 << i, 1);
        if (i == 0 || t < best) {
          best = t;
          pl.NR = 1 << i;
        }
      }
      pl.P = 4;
    } else if (hi <= 128) {
      if (5 * n > 3 * cu) pl.P = 4;
    } else if (order == 1 && lo > 128 && hi <= 256) {
      double t1 = 0.0, t2 = 0.0;  // steps of one slot of four rows and of two slots of two
      for (auto& I : h->inst) {
        t1 += schedule_steps_2d(I.hi.n[0], I.hi.n[1], 4, 1);
        t2 += schedule_steps_2d(I.hi.n[0], I.hi.n[1], 2, 2);
      }
      if (walls && n <= 2 * cu && 0.72 * t2 < t1) {
        pl.NR = 2;
        pl.R = 2;
        pl.P = 2;
      } else if (f64 && n > 2 * cu) {
        pl.NR = 2;
        pl.P = 4;
      }
    }
  }
  return pl;
}

// (Re)build the plan-dependent state. With a bound workspace the plan's bytes
// are counted first, and a plan that does not fit is rejected before any array
// of the current plan is overwritten.
bte_status build_plan(bte_ctx* h, const Plan& pl) {
  if (h->pool_mode == DevPool::ARENA) {
    h->pool_mode = DevPool::COUNT;
    bte_status s = build_plan_impl(h, pl);
    h->pool_mode = DevPool::ARENA;
    if (s != BTE_OK) return s;
    const size_t need = h->need_static + h->need_plan + (h->ws_store ? h->need_store : 0);
    if (need > h->ws_cap) {
      set_err("plan needs %zu bytes of workspace, %zu bound", need, h->ws_cap);
      return BTE_ERR_WORKSPACE;
    }
    HIPCHK(hipDeviceSynchronize());  // kernels in flight may still read the current plan's arrays
    return build_plan_impl(h, Plan(h->plan));
  }
  return build_plan_impl(h, pl);
}

bte_status build_static(bte_ctx* h);

// Back to the plan (and face order) in force before one that was rejected.
// Only memory of the handle's own that is gone meanwhile or a HIP error can
// keep it from being built again: the handle then holds no device arrays, and
// its next call makes them or returns the error; one bound to a workspace
// refuses calls until a workspace is bound again. The message stays that of
// the rejection.
void restore_plan(bte_ctx* h, const Plan& old, int order) {
  const std::string msg = g_err;
  h->order = order;
  if (build_plan(h, old) != BTE_OK) {
    h->ws_lost = h->pool_mode == DevPool::ARENA;
    h->ppool.reset();
    h->spool.reset();
    h->ws_base = nullptr;
    h->ws_cap = 0;
    h->ws_store = false;
    h->pool_mode = DevPool::COUNT;
    h->plan = old;
    h->sched_valid = false;
    if (build_static(h) == BTE_OK) (void)build_plan_impl(h, old);
  }
  g_err = msg;
}

// The default plan of the handle's order, or the base plan where only that one
// stays within the allocation-free solve's fixed array.
bte_status build_default_plan(bte_ctx* h) {
  const Plan base = h->base_plan, pl = default_plan(h, h->order);
  bte_status s = build_plan(h, pl);
  if (s != BTE_OK || (pl.R == base.R && pl.P == base.P && pl.NR == base.NR)) return s;
  const size_t need = h->need_static + h->need_plan, with = need + h->need_store;
  if (with <= kStaticScratchBytes) return s;
  // (the base plan's planes and field alone tell for most, before it is built)
  size_t planes = 0, field = 0;
  const size_t es = h->precision == BTE_PREC_FP32 ? 4 : 8, n_grp = (size_t)h->B * h->ords.size();
  for (auto& I : h->inst) {
    planes += h->nacc_max * (n_grp / base.P) * I.hi.ncell * es;
    field += n_grp * I.hi.ncell * es;
  }
  const size_t least = h->need_static + planes;
  if ((need <= kStaticScratchBytes || least > kStaticScratchBytes) && least + field > kStaticScratchBytes) return s;
  s = build_plan(h, base);
  const size_t need0 = h->need_static + h->need_plan, with0 = need0 + h->need_store;
  if (s == BTE_OK && ((need > kStaticScratchBytes && need0 <= kStaticScratchBytes) || with0 <= kStaticScratchBytes)) return s;
  return build_plan(h, pl);
}

// Plan-independent per-instance device data.
bte_status build_static(bte_ctx* h) {
  clear_graphs(h);
  h->ppool.reset();
  h->spool.reset();
  h->spool.reset(new_pool(h, 0));
  DevPool& pp = *h->spool;
  const int prec = h->precision;
  const size_t es = elem(prec);
  const int n = (int)h->inst.size();
  HIPCHK(pp.alloc(&h->d_st_f, n));
  HIPCHK(pp.alloc(&h->d_st_a, n));
  HIPCHK(pp.memset(h->d_st_f, 0, n * sizeof(StatusDev)));
  HIPCHK(pp.memset(h->d_st_a, 0, n * sizeof(StatusDev)));
  HIPCHK(pp.alloc(&h->d_counters, 4));
  HIPCHK(pp.memset(h->d_counters, 0, 16));
  h->fin_f.resize(n);
  h->fin_a.resize(n);
  // specular walls (Eq. 7): the inflow of an ordinate is its mirror's outflow,
  // so the inflow table gets one row per (band, ordinate)
  h->has_specular = false;
  for (const auto& I : h->inst)
    if (!I.hi.sface.empty()) h->has_specular = true;
  const int M = (int)h->ords.size();
  h->ubf_rows = h->has_specular ? M : 1;
  if (h->has_specular) {
    std::vector<int> member(M, 0);
    {
      std::vector<int> cnt(8, 0);
      for (int a = 0; a < M; ++a) member[a] = cnt[h->ords[a].oct]++;
    }
    std::vector<int2> src((size_t)6 * M, make_int2(-1, -1)), src_a((size_t)6 * M, make_int2(-1, -1));
    std::vector<double> iwq((size_t)6 * M, 0.0);
    for (int fd = 0; fd < 2 * h->dim; ++fd) {
      const int d = fd / 2;
      for (int a = 0; a < M; ++a) {
        const double sn = (fd & 1) ? h->ords[a].s[d] : -h->ords[a].s[d];
        if (sn == 0.0) continue;
        int m = -1;
        for (int c = 0; c < M && m < 0; ++c) {
          bool same = true;
          for (int e = 0; e < h->dim; ++e) {
            const double want = e == d ? -h->ords[a].s[e] : h->ords[a].s[e];
            same = same && std::fabs(h->ords[c].s[e] - want) < 1e-12;
          }
          if (same) m = c;
        }
        if (m < 0) {
          set_err("quadrature not closed under reflection of axis %d", d);
          return BTE_ERR_INVALID;
        }
        // incoming ordinates read their mirror in the forward iteration,
        // outgoing ones in the transposed iteration
        (sn < 0.0 ? src : src_a)[(size_t)fd * M + a] = make_int2(h->ords[m].oct, member[m]);
        iwq[(size_t)fd * M + a] = 1.0 / (h->ords[m].w * std::fabs(h->ords[m].s[d]));
      }
    }
    HIPCHK(pp.upload(&h->d_spec_src, src));
    HIPCHK(pp.upload(&h->d_spec_src_a, src_a));
    HIPCHK(pp.upload(&h->d_spec_iwq, iwq));
  }
  for (int k = 0; k < n; ++k) {
    Inst& I = h->inst[k];
    const HostInst& hi = I.hi;
    HIPCHK(pp.upload(&I.d_active, std::vector<unsigned char>(hi.active.begin(), hi.active.end())));
    for (int b = 0; b < 2; ++b) {
      HIPCHK(pp.alloc(&I.d_X[b], hi.ncell));
      HIPCHK(pp.alloc(&I.d_Xa[b], hi.ncell));
    }
    HIPCHK(pp.alloc(&I.d_qmag, hi.ncell));
    HIPCHK(pp.alloc(&I.d_qbuf, (size_t)hi.ncell * hi.dim));
    HIPCHK(pp.alloc(&I.d_dqbuf, hi.ncell));
    HIPCHK(pp.upload(&I.d_bf_bc, hi.bf_bc));
    HIPCHK(pp.upload(&I.d_bf_cell, hi.bf_cell));
    HIPCHK(pp.upload(&I.d_bc_kind, hi.bc_kind));
    HIPCHK(pp.upload(&I.d_bc_T, hi.bc_T));
    HIPCHK(pp.upload(&I.d_dface, hi.dface));
    std::vector<double> ih(hi.dface.size());
    for (size_t i = 0; i < hi.dface.size(); ++i) {
      const int f = hi.bf_face[hi.dface[i]];
      ih[i] = 1.0 / half_range(h->ords, f / 2);
    }
    HIPCHK(pp.upload(&I.d_inv_half, ih));
    std::vector<int> sdir(hi.sface.size());
    for (size_t i = 0; i < hi.sface.size(); ++i) sdir[i] = hi.bf_face[hi.sface[i]];
    HIPCHK(pp.upload(&I.d_sface, hi.sface));
    HIPCHK(pp.upload(&I.d_sface_dir, sdir));
    std::vector<int> dax(hi.dface.size());
    for (size_t i = 0; i < hi.dface.size(); ++i) dax[i] = hi.bf_face[hi.dface[i]] / 2;
    HIPCHK(pp.upload(&I.d_dface_axis, dax));
    HIPCHK(pp.alloc(&I.d_Qs, hi.ncell));
    HIPCHK(pp.alloc(&I.d_adj_scale, (size_t)h->B * 3));
    const size_t nu = (size_t)h->B * h->ubf_rows * std::max<size_t>(hi.bf_cell.size(), 1);
    char* u1;
    char* u0;
    HIPCHK(pp.alloc(&u1, nu * es));
    HIPCHK(pp.alloc(&u0, nu * es));
    HIPCHK(pp.memset(u1, 0, nu * es));
    HIPCHK(pp.memset(u0, 0, nu * es));
    I.d_ubf = u1;
    I.d_ubf0 = u0;
    if (!hi.dface.empty()) h->has_diffuse = true;
    FinInst& ff = h->fin_f[k];
    ff.X[0] = I.d_X[0];
    ff.X[1] = I.d_X[1];
    ff.g = nullptr;
    ff.q = I.d_qbuf;
    ff.qmag_prev = I.d_qmag;
    ff.active = I.d_active;
    FinInst& fa = h->fin_a[k];
    fa = ff;
    fa.X[0] = I.d_Xa[0];
    fa.X[1] = I.d_Xa[1];
    fa.q = I.d_dqbuf;
  }
  HIPCHK(pp.alloc(&h->d_fin_f, n));  // filled with the plan's arrays
  HIPCHK(pp.alloc(&h->d_fin_a, n));
  h->need_static = pp.used;
  for (auto& I : h->inst) {
    I.stored = false;
    I.have_dJds = false;
  }
  return BTE_OK;
}

// Workspace bytes of a handle: those of its plan, and while that is the default
// one at least those of the base plan too. A plan given in part is completed
// from the base plan, and plan caches hold it; neither may stop to fit because
// the default plan needs less (FP64 sections up to 128 rows: half the planes).
// The base plan is counted on a handle of its own: the arrays of this one stay.
bte_status workspace_need(bte_ctx* h, bool with_adjoint, size_t* bytes) {
  size_t need = h->need_static + h->need_plan, store = h->need_store;
  const Plan &a = h->plan, &b = h->base_plan;
  if (h->auto_plan && !(a.G == b.G && a.R == b.R && a.P == b.P && a.C == b.C && a.NR == b.NR)) {
    size_t &bn = h->base_need[h->order - 1], &bs = h->base_store[h->order - 1];
    if (bn == 0) {
      bte_ctx c;
      c.precision = h->precision;
      c.dim = h->dim;
      c.B = h->B;
      c.v = h->v;
      c.tau = h->tau;
      c.C = h->C;
      c.ords = h->ords;
      c.t0 = h->t0;
      c.n_cu = h->n_cu;
      c.order = h->order;
      c.inst.resize(h->inst.size());
      for (size_t k = 0; k < c.inst.size(); ++k) c.inst[k].hi = h->inst[k].hi;
      const std::string msg = g_err;
      const bool ok = build_static(&c) == BTE_OK && build_plan_impl(&c, b) == BTE_OK;
      g_err = msg;
      bn = ok ? c.need_static + c.need_plan : need;  // (pencil blocks have no second order)
      bs = ok ? c.need_store : store;
    }
    store = std::max(need + store, bn + bs);
    need = std::max(need, bn);
    store -= need;
  }
  *bytes = need + (with_adjoint ? store : 0);
  return BTE_OK;
}

// Build the device state of a handle whose arrays have only been counted so
// far, in memory of its own (no workspace bound).
bte_status ensure_device(bte_ctx* h) {
  if (h->pool_mode != DevPool::COUNT) return BTE_OK;
  if (h->ws_lost) {
    set_err("the handle's arrays in its bound workspace were lost in a failed plan change: bind a workspace again");
    return BTE_ERR_WORKSPACE;
  }
  h->pool_mode = DevPool::OWNED;
  bte_status s = build_static(h);
  if (s == BTE_OK) s = build_plan_impl(h, h->plan);
  if (s != BTE_OK) {
    h->spool.reset();
    h->ppool.reset();
    h->pool_mode = DevPool::COUNT;
  }
  return s;
}

bte_status create_common(int n_inst, const bte_geometry* geoms, const bte_bands* bands,
                         const bte_quadrature* quad, int precision, bte_handle* out) {
  if (!out) {
    set_err("null output handle");
    return BTE_ERR_INVALID;
  }
  *out = nullptr;
  if (precision != BTE_PREC_FP32 && precision != BTE_PREC_FP64) {
    set_err("precision must be BTE_PREC_FP32 or BTE_PREC_FP64");
    return BTE_ERR_INVALID;
  }
  if (n_inst < 1 || !geoms) {
    set_err("need at least one geometry");
    return BTE_ERR_INVALID;
  }
  for (int k = 0; k < n_inst; ++k) {
    const std::string e = validate_problem(&geoms[k], bands, quad);
    if (!e.empty()) {
      set_err("instance %d: %s", k, e.c_str());
      return BTE_ERR_INVALID;
    }
    if (geoms[k].dim != geoms[0].dim) {
      set_err("all instances of a batch must have the same dimension");
      return BTE_ERR_INVALID;
    }
  }
  std::unique_ptr<bte_ctx> h(new bte_ctx());
  h->precision = precision;
  h->dim = geoms[0].dim;
  h->B = bands->n_bands;
  h->v.assign(bands->h_v, bands->h_v + h->B);
  h->tau.assign(bands->h_tau, bands->h_tau + h->B);
  h->C.assign(bands->h_C, bands->h_C + h->B);
  h->t0 = *std::min_element(h->tau.begin(), h->tau.end());
  h->ords = fold_ordinates(quad, h->dim);
  h->inst.resize(n_inst);
  for (int k = 0; k < n_inst; ++k) {
    Inst& I = h->inst[k];
    build_instance(&geoms[k], I.hi);
    // default reference temperature: the mean over the isothermal boundary faces
    double sum = 0.0;
    long cnt = 0;
    for (size_t f = 0; f < I.hi.bf_bc.size(); ++f)
      if (I.hi.bc_kind[I.hi.bf_bc[f]] == BTE_BC_ISOTHERMAL) {
        sum += I.hi.bc_T[I.hi.bf_bc[f]];
        ++cnt;
      }
    I.T_ref_default = cnt ? sum / cnt : 300.0;
    I.T_ref = I.T_ref_default;
  }
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  hipDeviceProp_t prop;
  HIPCHK(hipGetDeviceProperties(&prop, dev));
  h->n_cu = std::max(1, prop.multiProcessorCount);
  snprintf(h->dev_name, sizeof(h->dev_name), "%s:%d", prop.gcnArchName, h->n_cu);
  HIPCHK(hipHostMalloc(reinterpret_cast<void**>(&h->h_st), sizeof(StatusDev) * 2 * n_inst, hipHostMallocDefault));
  HIPCHK(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
  // device arrays are only counted here; they are built by the first call that
  // needs them, or in a workspace the caller binds before that
  h->pool_mode = DevPool::COUNT;
  bte_status s = build_static(h.get());
  if (s != BTE_OK) return s;
  Plan pl = basic_plan(h.get());
  h->base_plan = pl;
  s = build_default_plan(h.get());
  const bool by_rule = s == BTE_OK;
  if (!by_rule) s = build_plan(h.get(), pl);
  while (s != BTE_OK && h->dim == 3 && pl.NR >= 1 && pl.P > 1) {
    pl.P /= 2;
    s = build_plan(h.get(), pl);
  }
  if (s != BTE_OK && h->dim == 3 && pl.NR >= 1) {
    // pencil blocks: one ordinate per lane, eight waves of one octant per workgroup
    pl.P = 8;
    pl.NR = 0;
    pl.C = 8;
    s = build_plan(h.get(), pl);
  }
  while (s != BTE_OK && h->dim == 3 && pl.P > 1) {
    pl.P /= 2;
    s = build_plan(h.get(), pl);
  }
  if (s != BTE_OK && h->dim < 3 && pl.P > 1) {
    pl.P = 1;
    s = build_plan(h.get(), pl);
  }
  if (s != BTE_OK) return s;
  if (!by_rule) h->base_plan = h->plan;
  h->auto_plan = true;
  *out = h.release();
  return BTE_OK;
}

// ---------------------------------------------------------------- the loop
struct LoopCfg {
  bool adj;
  int nacc_q;  // accumulator planes in flux iterations
};

bte_status enqueue_sweep(bte_ctx* h, bool adj, int nacc, int mode, int force, hipStream_t st) {
  SweepArgs a = h->sa;
  a.inst = adj ? h->d_inst_a : h->d_inst_f;
  a.jobs = adj ? h->d_jobs_a : h->d_jobs_f;
  a.grp_i = adj ? h->d_gi_a : h->d_gi_f;
  a.grp_t = adj ? h->d_gt_a : h->d_gt_f;
  a.force = force;
  if (h->dim < 3 || h->l3r) {
    const size_t lds = (size_t)a.lds_stage + (size_t)staged_planes(h->plan.G, nacc) * h->lds_stage_plane;
    if (h->l3r)
      HIPCHK(launch_sweep3r(h->precision, h->plan.NR, h->plan.P, nacc, mode, a, h->grid, h->block, lds, st));
    else
      HIPCHK(launch_sweep2d(h->precision, h->plan.G, h->plan.NR, h->plan.P, nacc, mode, a, h->grid, h->block, lds,
                            st));
    return BTE_OK;
  }
  const size_t lds = (size_t)a.lds_stage + (size_t)nacc * h->lds_stage_plane;
  HIPCHK(launch_sweep(h->precision, true, h->plan.G, nacc, mode, a, h->grid, h->block, lds, st));
  return BTE_OK;
}

bte_status enqueue_finalize(bte_ctx* h, bool adj, int flags, const bte_opts& o, hipStream_t st) {
  FinArgs f;
  f.inst = adj ? h->d_inst_a : h->d_inst_f;
  f.blocks = h->d_fblocks;
  f.n_blocks_total = h->n_fblocks;
  f.n_blocks_inst = h->d_nblocks;
  f.flags = flags | (adj ? FIN_ADJ : 0);
  f.tol_T = o.tol_T;
  f.tol_q = adj ? 1.0 : o.tol_q;
  HIPCHK(launch_finalize(h->precision, f, adj ? h->d_fin_a : h->d_fin_f, st));
  return BTE_OK;
}

bte_status enqueue_walls(bte_ctx* h, bool adj, hipStream_t st) {
  for (size_t k = 0; k < h->inst.size(); ++k) {
    Inst& I = h->inst[k];
    if (I.hi.dface.empty()) continue;
    WallArgs w;
    w.inst = adj ? h->d_inst_a : h->d_inst_f;
    w.inst_id = (int)k;
    w.n_dface = (int)I.hi.dface.size();
    w.dface_slot = I.d_dface;
    w.inv_half = I.d_inv_half;
    w.ofk = I.d_ofk;
    w.grp_ob = I.d_grp_ob;
    w.B = h->B;
    w.rows = h->ubf_rows;
    w.dface_axis = I.d_dface_axis;
    w.ent_df = I.d_ent_df;
    w.wsum = I.d_wsum;
    w.n_out = I.sch.n_out_stride;
    w.oct_xor = adj ? (1 << h->dim) - 1 : 0;
    w.scale = adj ? I.d_adj_scale : nullptr;
    HIPCHK(launch_wall_update(h->precision, w, 1 << h->dim, st));
  }
  return BTE_OK;
}

bte_status enqueue_specular(bte_ctx* h, bool adj, hipStream_t st) {
  for (size_t k = 0; k < h->inst.size(); ++k) {
    Inst& I = h->inst[k];
    if (I.hi.sface.empty()) continue;
    SpecArgs a;
    a.inst = adj ? h->d_inst_a : h->d_inst_f;
    a.inst_id = (int)k;
    a.n_sface = (int)I.hi.sface.size();
    a.sface_slot = I.d_sface;
    a.sface_dir = I.d_sface_dir;
    a.src = adj ? h->d_spec_src_a : h->d_spec_src;
    a.inv_wq = h->d_spec_iwq;
    a.ofk = I.d_ofk;
    a.grp_ob = I.d_grp_ob;
    a.B = h->B;
    a.M = h->ubf_rows;
    a.oct_xor = adj ? (1 << h->dim) - 1 : 0;
    a.scale = adj ? I.d_adj_scale : nullptr;
    HIPCHK(launch_spec_update(h->precision, a, st));
  }
  return BTE_OK;
}

CorrArgs corr_args(const bte_ctx* h, size_t k) {
  const Inst& I = h->inst[k];
  CorrArgs a{};
  a.inst = h->d_inst_f;
  a.inst_id = (int)k;
  a.n_grp = I.n_grp;
  a.grp = h->d_gi_f + I.grp0;
  a.coef = I.d_corr_coef;
  a.stencil = I.d_stencil;
  a.code = I.d_ccode;
  a.wslot = I.d_cwslot;
  a.n_slot = h->dim == 3 ? 1 : I.sch.R;
  a.n_unit = I.ctab.n_unit;
  a.seg = I.ctab.seg;
  a.tail = I.ctab.tail;
  a.unit = I.d_cunit;
  a.link = I.d_clink;
  for (int d = 0; d < 3; ++d) a.h[d] = I.hi.h[d];
  a.X0 = nullptr;
  return a;
}

// Second-order faces: the next sweep's correction from the stored field.
bte_status enqueue_corr(bte_ctx* h, hipStream_t st) {
  for (size_t k = 0; k < h->inst.size(); ++k) {
    Inst& I = h->inst[k];
    CorrArgs a = corr_args(h, k);
    HIPCHK(launch_corr(h->precision, a, I.sch.pos_per_oct, I.sch.NR, h->dim == 3, st));
  }
  return BTE_OK;
}

// n iterations of 1D films, as enqueue_chunk, in one launch.
bte_status enqueue_film(bte_ctx* h, bool adj, int n, const bte_opts& o, hipStream_t st, int flags = 0) {
  FilmArgs a;
  a.inst = adj ? h->d_inst_a : h->d_inst_f;
  a.fin = adj ? h->d_fin_a : h->d_fin_f;
  a.walls = h->d_film;
  a.grp_i = adj ? h->d_gi_a : h->d_gi_f;
  a.grp_t = adj ? h->d_gt_a : h->d_gt_f;
  a.n_grp = (int)h->gs.band.size();
  a.g_split = (int)(std::find(h->gs.oct.begin(), h->gs.oct.end(), 1) - h->gs.oct.begin());
  a.n_iter = n;
  a.flags = flags | (adj ? FIN_ADJ : 0);
  a.tol_T = o.tol_T;
  a.tol_q = adj ? 1.0 : o.tol_q;
  a.B = h->B;
  a.rows = h->ubf_rows;
  a.src = h->d_spec_src;
  a.inv_wq = h->d_spec_iwq;
  a.grp_ob = h->inst[0].d_grp_ob;
  HIPCHK(launch_film_chunk(h->precision, a, (int)h->inst.size(), film_cpl(h->film_cells), st));
  return BTE_OK;
}

// n iterations; the last one checks convergence, the last two carry the flux.
bte_status enqueue_chunk(bte_ctx* h, bool adj, int n, const bte_opts& o, hipStream_t st) {
  if (h->d_film && !(adj && h->film_reflects)) return enqueue_film(h, adj, n, o, st);
  const bool second = !adj && h->order == 2;
  const int nq = second ? std::max(3, 1 + h->dim) : 1 + h->dim;
  for (int k = 0; k < n; ++k) {
    const bool last = k == n - 1, second_last = k == n - 2;
    const bool qit = !adj && (last || second_last);
    bte_status s = enqueue_sweep(h, adj, qit ? nq : 1, second ? SWEEP_SECOND : SWEEP_PLAIN, 0, st);
    if (s != BTE_OK) return s;
    int fl = 0;
    if (qit) fl |= FIN_Q;
    if (last) fl |= FIN_CHECK | FIN_QPREV;
    s = enqueue_finalize(h, adj, fl, o, st);
    if (s != BTE_OK) return s;
    if (h->has_diffuse) {
      s = enqueue_walls(h, adj, st);
      if (s != BTE_OK) return s;
    }
    if (h->has_specular) {
      s = enqueue_specular(h, adj, st);
      if (s != BTE_OK) return s;
    }
    if (second) {
      s = enqueue_corr(h, st);
      if (s != BTE_OK) return s;
    }
  }
  return BTE_OK;
}

bte_status launch_chunk(bte_ctx* h, bool adj, int n, const bte_opts& o, hipStream_t st) {
  if (!o.use_graph) return enqueue_chunk(h, adj, n, o, st);
  uint64_t bT, bq;
  memcpy(&bT, &o.tol_T, 8);
  memcpy(&bq, &o.tol_q, 8);
  const auto key2 = std::make_tuple((int)adj, n, bT, bq);
  auto it = h->graphs.find(key2);
  if (it == h->graphs.end()) {
    HIPCHK(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal));
    bte_status s = enqueue_chunk(h, adj, n, o, h->cap_stream);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(h->cap_stream, &g);
    if (s != BTE_OK) {
      if (g) (void)hipGraphDestroy(g);
      return s;
    }
    HIPCHK(e);
    hipGraphExec_t ex = nullptr;
    HIPCHK(hipGraphInstantiate(&ex, g, nullptr, nullptr, 0));
    h->graphs[key2] = ex;
    h->graph_src[key2] = g;
    it = h->graphs.find(key2);
  }
  HIPCHK(hipGraphLaunch(it->second, st));
  return BTE_OK;
}

bte_status read_status(bte_ctx* h, bool adj, hipStream_t st) {
  const size_t n = h->inst.size();
  HIPCHK(hipMemcpyAsync(h->h_st, adj ? h->d_st_a : h->d_st_f, n * sizeof(StatusDev),
                        hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  return BTE_OK;
}

// Iterate until every instance is done or max_iters iterations ran.
bte_status run_loop(bte_ctx* h, bool adj, const bte_opts& o, hipStream_t st, double* secs) {
  const int K = o.check_every > 0 ? o.check_every : 8;
  const auto t0 = std::chrono::steady_clock::now();
  int it = 0;
  while (it < o.max_iters) {
    const int n = std::min(K, o.max_iters - it);
    bte_status s = launch_chunk(h, adj, n, o, st);
    if (s != BTE_OK) return s;
    it += n;
    s = read_status(h, adj, st);
    if (s != BTE_OK) return s;
    bool all_done = true;
    for (size_t k = 0; k < h->inst.size(); ++k) all_done = all_done && h->h_st[k].done;
    if (all_done) break;
  }
  *secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return BTE_OK;
}

bte_status check_opts(const bte_opts* o) {
  if (!o) {
    set_err("null options");
    return BTE_ERR_INVALID;
  }
  if (o->max_iters < 1) {
    set_err("max_iters must be >= 1");
    return BTE_ERR_INVALID;
  }
  if (o->check_every < 0) {
    set_err("check_every must be >= 0");
    return BTE_ERR_INVALID;
  }
  if (!std::isfinite(o->T_ref)) {
    set_err("T_ref must be finite");
    return BTE_ERR_INVALID;
  }
  return BTE_OK;
}

bte_status fill_report(bte_ctx* h, size_t k, double secs, bte_report* rep, bool adj, const bte_opts& o) {
  const StatusDev& s = h->h_st[k];
  bte_status st = BTE_OK;
  if (s.nonfinite) {
    st = BTE_ERR_NONFINITE;
    set_err("a non-finite value appeared (iteration %d)", s.iter);
  } else if (!s.done) {
    st = BTE_ERR_NOT_CONVERGED;
    set_err("not converged after %d iterations (eps_T %.3g, eps_q %.3g)", s.iter, s.eps_T, s.eps_q);
  }
  (void)o;
  (void)adj;
  if (rep) {
    rep->iters = s.iter;
    rep->eps_T = s.eps_T;
    rep->eps_q = s.eps_q;
    rep->seconds = secs;
    rep->status = st;
  }
  return st;
}

bte_status init_forward(bte_ctx* h, size_t k, const double* d_Q, const double* d_T_init, hipStream_t st) {
  Inst& I = h->inst[k];
  InitArgs a;
  a.inst = h->d_inst_f;
  a.inst_id = (int)k;
  a.X0 = d_T_init;
  a.T_ref = I.T_ref;
  a.Q = d_Q;
  a.active = I.d_active;
  a.X[0] = I.d_X[0];
  a.X[1] = I.d_X[1];
  a.adjoint = 0;
  HIPCHK(launch_init_state(h->precision, a, I.n_part, st));
  HIPCHK(launch_zero(I.d_qmag, (size_t)I.hi.ncell * 8, st));
  UbfInitArgs u;
  u.ubf = I.d_ubf;
  u.n_bface = (int)I.hi.bf_cell.size();
  u.B = h->B * h->ubf_rows;
  u.bf_bc = I.d_bf_bc;
  u.bf_cell = I.d_bf_cell;
  u.bc_kind = I.d_bc_kind;
  u.bc_T = I.d_bc_T;
  u.T_init = d_T_init;
  u.T_ref = I.T_ref;
  u.zero = 0;
  HIPCHK(launch_ubf_init(h->precision, u, st));
  HIPCHK(launch_status_reset(h->d_st_f + k, (double)I.hi.n_active, st));
  I.stored = false;
  I.have_dJds = false;
  if (h->order == 2) {
    // the first sweep's correction: the initial field is the equilibrium at
    // the initial temperature, the same for every ordinate
    CorrArgs a = corr_args(h, k);
    a.X0 = I.d_X[0];
    HIPCHK(launch_corr(h->precision, a, I.sch.pos_per_oct, I.sch.NR, h->dim == 3, st));
  }
  return BTE_OK;
}

bte_status store_state(bte_ctx* h, hipStream_t st) {
  if (h->order == 2) {
    set_err("the adjoint (and the angular field it keeps) is built for first-order faces");
    return BTE_ERR_STATE;
  }
  // one more forward sweep from the converged state that writes u per ordinate
  const size_t es = elem(h->precision);
  std::vector<InstDev> idf(h->inst.size());
  HIPCHK(hipMemcpy(idf.data(), h->d_inst_f, idf.size() * sizeof(InstDev), hipMemcpyDeviceToHost));
  for (size_t k = 0; k < h->inst.size(); ++k) {
    Inst& I = h->inst[k];
    if (!I.d_store) {
      if (h->pool_mode == DevPool::ARENA) {
        set_err("the bound workspace has no room for the angular field: bind bte_workspace_bytes(h, 1) bytes");
        return BTE_ERR_WORKSPACE;
      }
      char* p;
      HIPCHK(h->ppool->alloc(&p, (size_t)I.n_grp * I.n_part * h->plan.G * es));
      I.d_store = p;
    }
    idf[k].store_u = I.d_store;
  }
  HIPCHK(hipMemcpyAsync(h->d_inst_f, idf.data(), idf.size() * sizeof(InstDev), hipMemcpyHostToDevice, st));
  bte_status s = enqueue_sweep(h, false, 1, SWEEP_STORE, 1, st);
  if (s != BTE_OK) return s;
  for (size_t k = 0; k < h->inst.size(); ++k) {
    h->inst[k].stored = true;
    h->inst[k].fwd_parity = h->h_st[k].iter & 1;
  }
  return BTE_OK;
}

bte_status default_opts(const bte_opts* o, bte_opts& out) {
  bte_status s = check_opts(o);
  if (s != BTE_OK) return s;
  out = *o;
  if (out.check_every == 0) out.check_every = 8;
  return BTE_OK;
}

// Group coefficient tables for the current tau (uploaded when the device
// state exists; otherwise they are built with it).
bte_status upload_coefficients(bte_ctx* h) {
  if (h->pool_mode == DevPool::COUNT) return BTE_OK;
  std::vector<double> gtf, gta;
  for (auto& I : h->inst) {
    std::vector<double> cf, ca;
    group_coefficients(h->gs, h->ords, I.hi, h->v, h->tau, h->C, h->t0, false, cf);
    group_coefficients(h->gs, h->ords, I.hi, h->v, h->tau, h->C, h->t0, true, ca);
    gtf.insert(gtf.end(), cf.begin(), cf.end());
    gta.insert(gta.end(), ca.begin(), ca.end());
  }
  const std::vector<char> a = to_prec(gtf, h->precision), b = to_prec(gta, h->precision);
  HIPCHK(hipDeviceSynchronize());  // a sweep in flight may still read the tables
  HIPCHK(hipMemcpy(h->d_gt_f, a.data(), a.size(), hipMemcpyHostToDevice));
  HIPCHK(hipMemcpy(h->d_gt_a, b.data(), b.size(), hipMemcpyHostToDevice));
  if (h->order == 2)
    for (auto& I : h->inst) {
      const std::vector<double> cc = corr_coefficients(h, I.hi);
      HIPCHK(hipMemcpy(I.d_corr_coef, cc.data(), cc.size() * sizeof(double), hipMemcpyHostToDevice));
    }
  return BTE_OK;
}

// New relaxation times: validated, then the coefficient tables follow. A state
// stored for the adjoint belongs to the old ones and is dropped.
bte_status apply_tau(bte_ctx* h, const double* h_tau) {
  for (int b = 0; b < h->B; ++b)
    if (!(h_tau[b] > 0 && std::isfinite(h_tau[b]))) {
      set_err("tau[%d] must be finite and > 0", b);
      return BTE_ERR_INVALID;
    }
  if (std::equal(h->tau.begin(), h->tau.end(), h_tau)) return BTE_OK;
  h->tau.assign(h_tau, h_tau + h->B);
  for (auto& I : h->inst) {
    I.stored = false;
    I.have_dJds = false;
  }
  return upload_coefficients(h);
}

// 64-bit FNV-1a, for the geometry part of an autotune-cache key.
uint64_t fnv1a(uint64_t hsh, const void* p, size_t n) {
  const unsigned char* c = static_cast<const unsigned char*>(p);
  for (size_t i = 0; i < n; ++i) {
    hsh ^= c[i];
    hsh *= 1099511628211ull;
  }
  return hsh;
}

// Autotune-cache key: what the sweep's cost depends on (dimension, precision,
// bands, swept ordinates, every instance's grid, mask and wall kinds) and the
// device.
std::string tune_key(const bte_ctx* h) {
  uint64_t g = 1469598103934665603ull;
  for (const auto& I : h->inst) {
    g = fnv1a(g, I.hi.n, sizeof(I.hi.n));
    g = fnv1a(g, I.hi.active.data(), I.hi.active.size());
    for (size_t f = 0; f < I.hi.bf_bc.size(); ++f) {
      const int kind = I.hi.bc_kind[I.hi.bf_bc[f]];
      g = fnv1a(g, &kind, sizeof(kind));
    }
  }
  char buf[256];
  snprintf(buf, sizeof(buf), "dim=%d prec=%d B=%d M=%zu inst=%zu geo=%016llx dev=%s", h->dim, h->precision, h->B,
           h->ords.size(), h->inst.size(), (unsigned long long)g, h->dev_name);
  return buf;
}

bte_status autotune_impl(bte_ctx* h, const double* d_Q, int n_iters, hipStream_t st, Plan* best);

// Autotune cache (opts->autotune_cache): use the plan stored for this
// problem's key, or tune (30 whole iterations per candidate, on d_Q) and
// append the result. Lines read "<key> plan G R P C NR"; the last match wins.
bte_status apply_tune_cache(bte_ctx* h, const char* path, const double* d_Q, hipStream_t st) {
  if (!path) return BTE_OK;
  const std::string key = tune_key(h);
  bool found = false;
  Plan pl;
  if (FILE* f = fopen(path, "r")) {
    char line[512];
    while (fgets(line, sizeof(line), f)) {
      const size_t kl = key.size();
      if (strncmp(line, key.c_str(), kl) != 0 || strncmp(line + kl, " plan ", 6) != 0) continue;
      Plan p;
      if (sscanf(line + kl + 6, "%d %d %d %d %d", &p.G, &p.R, &p.P, &p.C, &p.NR) == 5) {
        pl = p;
        found = true;
      }
    }
    fclose(f);
  }
  if (found) {
    const Plan& c = h->plan;
    const bool was_auto = h->auto_plan;
    h->auto_plan = false;
    if (pl.G == c.G && pl.R == c.R && pl.P == c.P && pl.C == c.C && pl.NR == c.NR) return BTE_OK;
    const Plan old = h->plan;
    bte_status s = build_plan(h, pl);
    if (s != BTE_OK) {
      restore_plan(h, old, h->order);
      h->auto_plan = was_auto;
      const std::string e = g_err;
      set_err("autotune cache %s: stored plan rejected: %s", path, e.c_str());
    }
    return s;
  }
  Plan best;
  bte_status s = autotune_impl(h, d_Q, 30, st, &best);
  if (s != BTE_OK) return s;
  FILE* f = fopen(path, "a");
  if (!f) {
    set_err("autotune cache %s cannot be opened for writing", path);
    return BTE_ERR_INVALID;
  }
  fprintf(f, "%s plan %d %d %d %d %d\n", key.c_str(), best.G, best.R, best.P, best.C, best.NR);
  fclose(f);
  return BTE_OK;
}

// Carve every device array of h from [d_ws, d_ws + bytes), or unbind (d_ws
// NULL); need, with: the bytes it takes without and with the angular field.
bte_status bind_impl(bte_ctx* h, void* d_ws, size_t bytes, size_t need, size_t with) {
  if (d_ws && reinterpret_cast<uintptr_t>(d_ws) % kWsAlign) {
    set_err("workspace must be %zu-byte aligned", kWsAlign);
    return BTE_ERR_INVALID;
  }
  if (d_ws && bytes < need) {
    set_err("workspace of %zu bytes is smaller than the %zu the handle needs", bytes, need);
    return BTE_ERR_WORKSPACE;
  }
  if (h->pool_mode != DevPool::COUNT) HIPCHK(hipDeviceSynchronize());
  clear_graphs(h);
  h->ppool.reset();
  h->spool.reset();
  h->ws_base = static_cast<char*>(d_ws);
  h->ws_cap = d_ws ? bytes : 0;
  h->ws_lost = false;
  h->ws_store = d_ws && bytes >= with;
  if (!d_ws) {
    // unbound: the handle's own memory is made by the next call that needs it
    h->pool_mode = DevPool::COUNT;
    return BTE_OK;
  }
  h->pool_mode = DevPool::ARENA;
  bte_status s = build_static(h);
  if (s == BTE_OK) s = build_plan_impl(h, h->plan);
  if (s != BTE_OK) {
    h->spool.reset();
    h->ppool.reset();
    h->ws_base = nullptr;
    h->ws_cap = 0;
    h->ws_store = false;
    h->pool_mode = DevPool::COUNT;
  }
  return s;
}


// The solve of a single-instance handle whose device state exists (options
// already defaulted).
bte_status solve_impl(bte_ctx* h, const double* h_tau, const double* d_Q, const double* d_T_init, double* d_T,
                      double* d_q, const bte_opts& o, hipStream_t st, bte_report* h_rep) {
  bte_status s = BTE_OK;
  if (h_tau) {
    s = apply_tau(h, h_tau);
    if (s != BTE_OK) return s;
  }
  s = apply_tune_cache(h, o.autotune_cache, d_Q, st);
  if (s != BTE_OK) return s;
  Inst& I = h->inst[0];
  I.T_ref = o.T_ref > 0 ? o.T_ref : I.T_ref_default;
  h->fin_f[0].q = d_q ? d_q : I.d_qbuf;
  HIPCHK(hipMemcpyAsync(h->d_fin_f, h->fin_f.data(), sizeof(FinInst), hipMemcpyHostToDevice, st));
  s = init_forward(h, 0, d_Q, d_T_init, st);
  if (s != BTE_OK) return s;
  double secs = 0.0;
  s = run_loop(h, false, o, st, &secs);
  if (s != BTE_OK) return s;
  if (o.store_angular) {
    s = store_state(h, st);
    if (s != BTE_OK) return s;
    if (d_Q) HIPCHK(hipMemcpyAsync(I.d_Qs, d_Q, (size_t)I.hi.ncell * 8, hipMemcpyDeviceToDevice, st));
    else HIPCHK(launch_zero(I.d_Qs, (size_t)I.hi.ncell * 8, st));
  }
  HIPCHK(launch_output(I.d_X[h->h_st[0].iter & 1], I.d_active, I.hi.ncell, I.T_ref, 1.0, d_T, st));
  HIPCHK(hipStreamSynchronize(st));
  return fill_report(h, 0, secs, h_rep, false, o);
}

// ---------------------------------------------- the allocation-free solve
// Device workspace of bte_solve_noalloc: one array per device, part of the
// library's code object (allocated when the module is loaded on a device,
// held until the process ends). Host code never uses the array's name as an
// address: the device address comes from hipGetSymbolAddress, once per
// device, and is kept per device.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};       // device address of `scratch` per device
bte_ctx* g_scratch_owner[kMaxDevices] = {};  // handle whose arrays the array holds

// Drop h's claim on the static scratch of its device (it keeps its arrays
// until it binds something else).
void release_static_scratch(bte_ctx* h) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  for (int d = 0; d < kMaxDevices; ++d)
    if (g_scratch_owner[d] == h) g_scratch_owner[d] = nullptr;
}

// Bind h to the static scratch of the current device unless it holds it
// already. Another handle holding it loses its arrays (it returns to the
// unbound state and makes or binds memory again at its next call). No
// allocation and no free: a handle with arrays of its own is refused.
bte_status bind_static_scratch(bte_ctx* h) {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    set_err("device %d out of range", dev);
    return BTE_ERR_INVALID;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = p;
  }
  char* ws = static_cast<char*>(g_scratch_ptr[dev]);
  if (g_scratch_owner[dev] == h && h->pool_mode == DevPool::ARENA && h->ws_base == ws) return BTE_OK;
  if (h->pool_mode == DevPool::OWNED) {
    set_err("bte_solve_noalloc: the handle holds device memory of its own (a previous bte_solve made it); "
            "use a fresh handle, or one bound to a workspace");
    return BTE_ERR_STATE;
  }
  const size_t need = h->need_static + h->need_plan;
  if (need > kStaticScratchBytes) {
    set_err("bte_solve_noalloc: the problem needs %zu bytes of workspace; the static workspace holds %zu", need,
            kStaticScratchBytes);
    return BTE_ERR_WORKSPACE;
  }
  bte_ctx* old = g_scratch_owner[dev];
  if (old && old != h) {
    HIPCHK(hipDeviceSynchronize());
    clear_graphs(old);
    old->ppool.reset();
    old->spool.reset();
    old->ws_base = nullptr;
    old->ws_cap = 0;
    old->ws_store = false;
    old->pool_mode = DevPool::COUNT;
    for (auto& I : old->inst) {
      I.stored = false;
      I.have_dJds = false;
    }
  }
  g_scratch_owner[dev] = nullptr;
  bte_status s = bind_impl(h, ws, kStaticScratchBytes, need, need + h->need_store);
  if (s == BTE_OK) g_scratch_owner[dev] = h;
  return s;
}

}  // namespace

// ============================================================================
extern "C" {

const char* bte_version(void) { return "bte-mi355x 0.1"; }

const char* bte_last_error(void) { return g_err.c_str(); }

bte_status bte_validate(const bte_geometry* geom, const bte_bands* bands, const bte_quadrature* quad) {
  const std::string e = validate_problem(geom, bands, quad);
  if (!e.empty()) {
    set_err("%s", e.c_str());
    return BTE_ERR_INVALID;
  }
  return BTE_OK;
}

// Gauss-Legendre nodes and weights on [-1, 1] by Newton iteration on the
// Legendre three-term recurrence.
static void gauss_legendre(int n, std::vector<double>& x, std::vector<double>& w) {
  x.assign(n, 0.0);
  w.assign(n, 0.0);
  for (int i = 0; i < (n + 1) / 2; ++i) {
    double z = std::cos(kPi * (i + 0.75) / (n + 0.5));
    double dp = 0.0;
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= n; ++k) {
        const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      if (n == 1) {
        p1 = z;
        p0 = 1.0;
      }
      dp = n * (z * p1 - p0) / (z * z - 1.0);
      const double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    double p0 = 1.0, p1 = z;
    for (int k = 2; k <= n; ++k) {
      const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    dp = n * (z * p1 - p0) / (z * z - 1.0);
    x[i] = -z;
    x[n - 1 - i] = z;
    w[i] = w[n - 1 - i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
  if (n == 1) {
    x[0] = 0.0;
    w[0] = 2.0;
  }
}

bte_status bte_quadrature_gl_mu(int n_mu, double* h_s, double* h_w) {
  if (n_mu < 1 || !h_s || !h_w) {
    set_err("n_mu >= 1 and output arrays required");
    return BTE_ERR_INVALID;
  }
  std::vector<double> x, w;
  gauss_legendre(n_mu, x, w);
  for (int a = 0; a < n_mu; ++a) {
    h_s[3 * a] = x[a];
    h_s[3 * a + 1] = std::sqrt(std::max(0.0, 1.0 - x[a] * x[a]));
    h_s[3 * a + 2] = 0.0;
    h_w[a] = 2.0 * kPi * w[a];
  }
  return BTE_OK;
}

bte_status bte_quadrature_octant_gl(int n_theta, int n_phi, int polar_axis, double* h_s, double* h_w) {
  if (n_theta < 1 || n_phi < 1 || polar_axis < 0 || polar_axis > 2 || !h_s || !h_w) {
    set_err("n_theta, n_phi >= 1, polar_axis in 0..2 and output arrays required");
    return BTE_ERR_INVALID;
  }
  std::vector<double> xt, gt, xp, gp;
  gauss_legendre(n_theta, xt, gt);
  gauss_legendre(n_phi, xp, gp);
  int a = 0;
  double tot = 0.0;
  for (int sx = 0; sx < 2; ++sx)
    for (int sy = 0; sy < 2; ++sy)
      for (int sz = 0; sz < 2; ++sz)
        for (int it = 0; it < n_theta; ++it)
          for (int ip = 0; ip < n_phi; ++ip) {
            const double t = (xt[it] + 1.0) * kPi / 4.0, p = (xp[ip] + 1.0) * kPi / 4.0;
            const double c = std::cos(t), sc = std::sin(t) * std::cos(p), ss = std::sin(t) * std::sin(p);
            double v[3];
            if (polar_axis == 0) { v[0] = c; v[1] = sc; v[2] = ss; }
            else if (polar_axis == 2) { v[0] = sc; v[1] = ss; v[2] = c; }
            else { v[0] = ss; v[1] = c; v[2] = sc; }
            v[0] *= sx ? -1.0 : 1.0;
            v[1] *= sy ? -1.0 : 1.0;
            v[2] *= sz ? -1.0 : 1.0;
            const double nn = std::sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
            for (int d = 0; d < 3; ++d) h_s[3 * a + d] = v[d] / nn;
            h_w[a] = gt[it] * kPi / 4.0 * gp[ip] * kPi / 4.0 * std::sin(t);
            tot += h_w[a];
            ++a;
          }
  for (int k = 0; k < a; ++k) h_w[k] *= 4.0 * kPi / tot;
  return BTE_OK;
}

bte_status bte_create(const bte_geometry* geom, const bte_bands* bands, const bte_quadrature* quad,
                      int precision, bte_handle* out) {
  ErrClear clear_on_exit;
  return create_common(1, geom, bands, quad, precision, out);
}

bte_status bte_batch_create(int n_inst, const bte_geometry* geoms, const bte_bands* bands,
                            const bte_quadrature* quad, int precision, bte_handle* out) {
  ErrClear clear_on_exit;
  return create_common(n_inst, geoms, bands, quad, precision, out);
}

bte_status bte_workspace_bytes(bte_handle h, int with_adjoint, size_t* bytes) {
  ErrClear clear_on_exit;
  if (!h || !bytes) {
    set_err("null handle or output");
    return BTE_ERR_INVALID;
  }
  return workspace_need(h, with_adjoint != 0, bytes);
}

bte_status bte_bind_workspace(bte_handle h, void* d_ws, size_t bytes) {
  ErrClear clear_on_exit;
  if (!h) {
    set_err("null handle");
    return BTE_ERR_INVALID;
  }
  size_t need = 0, with = 0;
  bte_status s = d_ws ? workspace_need(h, false, &need) : BTE_OK;
  if (s == BTE_OK && d_ws) s = workspace_need(h, true, &with);
  if (s != BTE_OK) return s;
  release_static_scratch(h);
  return bind_impl(h, d_ws, bytes, need, with);
}

bte_status bte_set_tau(bte_handle h, const double* h_tau) {
  ErrClear clear_on_exit;
  if (!h || !h_tau) {
    set_err("null handle or tau");
    return BTE_ERR_INVALID;
  }
  return apply_tau(h, h_tau);
}

bte_status bte_set_order(bte_handle h, int order) {
  ErrClear clear_on_exit;
  if (!h || (order != 1 && order != 2)) {
    set_err("null handle or order not 1 or 2");
    return BTE_ERR_INVALID;
  }
  if (order == h->order) return BTE_OK;
  const int old_order = h->order;
  const Plan old = h->plan;
  if (h->auto_plan && h->plan.NR >= 1) {
    h->order = order;
    if (build_default_plan(h) == BTE_OK) return BTE_OK;
    h->order = old_order;
  }
  Plan p = h->auto_plan ? h->base_plan : h->plan;
  if (order == 2) {
    p.G = 1;
    if (h->dim == 3 && p.NR < 1) {
      // the 3D pencil blocks have no second-order sweep: the rows layout
      p.NR = 1;
      p.C = kC2;
    }
  }
  h->order = order;
  bte_status s = build_plan(h, p);
  if (s != BTE_OK) restore_plan(h, old, old_order);
  return s;
}

bte_status bte_set_plan(bte_handle h, const bte_plan* plan) {
  ErrClear clear_on_exit;
  if (!h || !plan) {
    set_err("null handle or plan");
    return BTE_ERR_INVALID;
  }
  Plan p = h->auto_plan ? h->base_plan : h->plan;
  if (plan->G) p.G = plan->G;
  if (plan->R) p.R = plan->R;
  if (plan->P) p.P = plan->P;
  if (plan->C) p.C = plan->C;
  if (plan->NR) p.NR = plan->NR < 0 ? 0 : plan->NR;  // 3D: NR < 0 selects the pencil-block layout
  const Plan old = h->plan;
  bte_status s = build_plan(h, p);
  if (s != BTE_OK) restore_plan(h, old, h->order);
  else h->auto_plan = false;
  return s;
}

bte_status bte_get_plan(bte_handle h, bte_plan* plan) {
  if (!h || !plan) {
    set_err("null handle or plan");
    return BTE_ERR_INVALID;
  }
  plan->G = h->plan.G;
  plan->R = h->plan.R;
  plan->P = h->plan.P;
  plan->C = h->plan.C;
  plan->NR = h->plan.NR;
  return BTE_OK;
}

bte_status bte_solve(bte_handle h, const double* h_tau, const double* d_Q, const double* d_T_init, double* d_T,
                     double* d_q, const bte_opts* opts, void* hip_stream, bte_report* h_rep) {
  ErrClear clear_on_exit;
  if (!h || !d_T) {
    set_err("null handle or output");
    return BTE_ERR_INVALID;
  }
  if (h->inst.size() != 1) {
    set_err("bte_solve needs a single-instance handle (use bte_batch_solve)");
    return BTE_ERR_STATE;
  }
  bte_opts o;
  bte_status s = default_opts(opts, o);
  if (s != BTE_OK) return s;
  s = ensure_device(h);
  if (s != BTE_OK) return s;
  return solve_impl(h, h_tau, d_Q, d_T_init, d_T, d_q, o, reinterpret_cast<hipStream_t>(hip_stream), h_rep);
}

bte_status bte_solve_noalloc(bte_handle h, const double* h_tau, const double* d_Q, const double* d_T_init,
                             double* d_T, double* d_q, const bte_opts* opts, void* hip_stream, bte_report* h_rep) {
  ErrClear clear_on_exit;
  if (!h || !d_T) {
    set_err("null handle or output");
    return BTE_ERR_INVALID;
  }
  if (h->inst.size() != 1) {
    set_err("bte_solve_noalloc needs a single-instance handle");
    return BTE_ERR_STATE;
  }
  bte_opts o;
  bte_status s = default_opts(opts, o);
  if (s != BTE_OK) return s;
  s = bind_static_scratch(h);
  if (s != BTE_OK) return s;
  // a graph's instantiation and the tuner's events may allocate: neither here
  o.use_graph = 0;
  o.autotune_cache = nullptr;
  return solve_impl(h, h_tau, d_Q, d_T_init, d_T, d_q, o, reinterpret_cast<hipStream_t>(hip_stream), h_rep);
}

bte_status bte_batch_solve(bte_handle h, const double* const* d_Q, double* const* d_T, double* const* d_q,
                           const bte_opts* opts, void* hip_stream, bte_report* h_reps) {
  ErrClear clear_on_exit;
  if (!h || !d_T || !d_Q) {
    set_err("null handle or arrays");
    return BTE_ERR_INVALID;
  }
  bte_opts o;
  bte_status s = default_opts(opts, o);
  if (s != BTE_OK) return s;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  s = ensure_device(h);
  if (s != BTE_OK) return s;
  s = apply_tune_cache(h, o.autotune_cache, nullptr, st);
  if (s != BTE_OK) return s;
  for (size_t k = 0; k < h->inst.size(); ++k) {
    h->inst[k].T_ref = o.T_ref > 0 ? o.T_ref : h->inst[k].T_ref_default;
    if (!d_T[k]) {
      set_err("null output of instance %zu", k);
      return BTE_ERR_INVALID;
    }
    h->fin_f[k].q = (d_q && d_q[k]) ? d_q[k] : h->inst[k].d_qbuf;
  }
  HIPCHK(hipMemcpyAsync(h->d_fin_f, h->fin_f.data(), h->fin_f.size() * sizeof(FinInst),
                        hipMemcpyHostToDevice, st));
  for (size_t k = 0; k < h->inst.size(); ++k) {
    s = init_forward(h, k, d_Q[k], nullptr, st);
    if (s != BTE_OK) return s;
  }
  double secs = 0.0;
  s = run_loop(h, false, o, st, &secs);
  if (s != BTE_OK) return s;
  if (o.store_angular) {
    s = store_state(h, st);
    if (s != BTE_OK) return s;
    for (size_t k = 0; k < h->inst.size(); ++k) {
      Inst& I = h->inst[k];
      if (d_Q[k]) HIPCHK(hipMemcpyAsync(I.d_Qs, d_Q[k], (size_t)I.hi.ncell * 8, hipMemcpyDeviceToDevice, st));
      else HIPCHK(launch_zero(I.d_Qs, (size_t)I.hi.ncell * 8, st));
    }
  }
  bte_status worst = BTE_OK;
  for (size_t k = 0; k < h->inst.size(); ++k) {
    Inst& I = h->inst[k];
    HIPCHK(launch_output(I.d_X[h->h_st[k].iter & 1], I.d_active, I.hi.ncell, I.T_ref, 1.0, d_T[k], st));
  }
  HIPCHK(hipStreamSynchronize(st));
  for (size_t k = 0; k < h->inst.size(); ++k) {
    const bte_status r = fill_report(h, k, secs, h_reps ? h_reps + k : nullptr, false, o);
    if (r != BTE_OK && (worst == BTE_OK || r == BTE_ERR_NONFINITE)) worst = r;
  }
  return worst;
}

static bte_status adjoint_common(bte_handle h, const double* const* d_dJdT, double* h_dJdtau,
                                 double* const* d_dJdQ, const bte_opts* opts, void* hip_stream,
                                 bte_report* h_reps) {
  if (!h || !d_dJdT) {
    set_err("null handle or dJ/dT");
    return BTE_ERR_INVALID;
  }
  for (auto& I : h->inst)
    if (!I.stored) {
      set_err("bte_adjoint needs a previous solve with store_angular = 1 and the same tau");
      return BTE_ERR_STATE;
    }
  bte_opts o;
  bte_status s = default_opts(opts, o);
  if (s != BTE_OK) return s;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  const size_t n = h->inst.size();
  // adjoint descriptors: forward state and stored field for the tau pass
  std::vector<InstDev> ida(n);
  HIPCHK(hipMemcpy(ida.data(), h->d_inst_a, n * sizeof(InstDev), hipMemcpyDeviceToHost));
  for (size_t k = 0; k < n; ++k) {
    Inst& I = h->inst[k];
    ida[k].xf = I.d_xq[I.fwd_parity];
    ida[k].store_u = I.d_store;
    h->fin_a[k].g = d_dJdT[k];
    h->fin_a[k].q = (d_dJdQ && d_dJdQ[k]) ? d_dJdQ[k] : I.d_dqbuf;
  }
  HIPCHK(hipMemcpyAsync(h->d_inst_a, ida.data(), n * sizeof(InstDev), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(h->d_fin_a, h->fin_a.data(), n * sizeof(FinInst), hipMemcpyHostToDevice, st));
  // reflecting walls: the wall-value adjoint mu (the transpose of the lagged
  // reflection) starts at zero; the transposed sweeps take mu back as inflow
  // through the factor 4 pi tau_b D h_d / (C_b t0 v_b) per band and face axis
  const double Dtot = total_D(h);
  std::vector<std::vector<double>> adj_scale(n);
  for (size_t k = 0; k < n; ++k) {
    Inst& I = h->inst[k];
    if (I.hi.dface.empty() && I.hi.sface.empty()) continue;
    adj_scale[k].assign((size_t)h->B * 3, 0.0);
    for (int b = 0; b < h->B; ++b)
      for (int d = 0; d < I.hi.dim; ++d)
        adj_scale[k][(size_t)b * 3 + d] =
            4.0 * kPi * h->tau[b] * Dtot * I.hi.h[d] / (h->C[b] * h->t0 * h->v[b]);
    HIPCHK(hipMemcpyAsync(I.d_adj_scale, adj_scale[k].data(), adj_scale[k].size() * sizeof(double),
                          hipMemcpyHostToDevice, st));
    const size_t nu = (size_t)h->B * h->ubf_rows * std::max<size_t>(I.hi.bf_cell.size(), 1);
    HIPCHK(launch_zero(I.d_ubf0, nu * elem(h->precision), st));
  }
  for (size_t k = 0; k < n; ++k) {
    Inst& I = h->inst[k];
    InitArgs a;
    a.inst = h->d_inst_a;
    a.inst_id = (int)k;
    a.X0 = d_dJdT[k];
    a.T_ref = 0.0;
    a.Q = nullptr;
    a.active = I.d_active;
    a.X[0] = I.d_Xa[0];
    a.X[1] = I.d_Xa[1];
    a.adjoint = 1;
    HIPCHK(launch_init_state(h->precision, a, I.n_part, st));
    HIPCHK(launch_status_reset(h->d_st_a + k, (double)I.hi.n_active, st));
    HIPCHK(launch_zero(I.d_tgrad, (size_t)I.n_grp * 2 * 8, st));
  }
  double secs = 0.0;
  s = run_loop(h, true, o, st, &secs);
  if (s != BTE_OK) return s;
  std::vector<int> conv(n);
  for (size_t k = 0; k < n; ++k) conv[k] = h->h_st[k].done;
  // final pass: reopen every instance, sweep with the tau sums and dJ/dQ
  for (size_t k = 0; k < n; ++k) HIPCHK(launch_zero(&h->d_st_a[k].done, 4, st));
  s = enqueue_sweep(h, true, 2, SWEEP_TAUGRAD, 0, st);
  if (s != BTE_OK) return s;
  s = enqueue_finalize(h, true, FIN_Q, o, st);
  if (s != BTE_OK) return s;
  HIPCHK(hipStreamSynchronize(st));
  std::vector<StatusDev> sa(n);
  HIPCHK(hipMemcpy(sa.data(), h->d_st_a, n * sizeof(StatusDev), hipMemcpyDeviceToHost));
  const double D = total_D(h);
  bte_status worst = BTE_OK;
  for (size_t k = 0; k < n; ++k) {
    Inst& I = h->inst[k];
    const int nc = I.hi.ncell;
    // lambda used by the final pass (before its own update) and the forward Delta T
    std::vector<double> lam(nc), dT(nc), tg((size_t)I.n_grp * 2);
    const int lp = (sa[k].iter - 1) & 1;
    HIPCHK(hipMemcpy(lam.data(), I.d_Xa[lp], nc * 8, hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(dT.data(), I.d_X[I.fwd_parity], nc * 8, hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(tg.data(), I.d_tgrad, tg.size() * 8, hipMemcpyDeviceToHost));
    double L = 0.0;
    for (int c = 0; c < nc; ++c)
      if (I.hi.active[c]) L += lam[c] * dT[c];
    std::vector<double> T1(h->B, 0.0), T2(h->B, 0.0);
    for (int g = 0; g < I.n_grp; ++g) {
      T1[I.grp_band[g]] += tg[2 * g];
      T2[I.grp_band[g]] += tg[2 * g + 1];
    }
    if (h_dJdtau) {
      for (int b = 0; b < h->B; ++b) {
        const double tb = h->tau[b];
        h_dJdtau[k * h->B + b] = (1.0 / tb) * ((h->t0 / tb) * T1[b] - T2[b] + h->C[b] / (tb * D) * L);
      }
    }
    // dJ/ds for a common factor s on every cell size: every beta_d scales as
    // 1/s, and by the forward equation sum_d beta_d (u - u_up) equals
    // rho' (dT - u) + gamma' Q, so dJ/ds = -sum_b rho'_b T1_b + sum_c Q_c dJ/dQ_c
    {
      std::vector<double> dq(nc), Qs(nc);
      HIPCHK(hipMemcpy(dq.data(), h->fin_a[k].q, nc * 8, hipMemcpyDeviceToHost));
      HIPCHK(hipMemcpy(Qs.data(), I.d_Qs, nc * 8, hipMemcpyDeviceToHost));
      double ds = 0.0;
      for (int c = 0; c < nc; ++c)
        if (I.hi.active[c]) ds += Qs[c] * dq[c];
      for (int b = 0; b < h->B; ++b) ds -= (h->t0 / h->tau[b]) * T1[b];
      I.dJds = ds;
      I.have_dJds = true;
    }
    h->h_st[k] = sa[k];
    h->h_st[k].done = conv[k];
    const bte_status r = fill_report(h, k, secs, h_reps ? h_reps + k : nullptr, true, o);
    if (r != BTE_OK && (worst == BTE_OK || r == BTE_ERR_NONFINITE)) worst = r;
  }
  return worst;
}

bte_status bte_adjoint(bte_handle h, const double* d_dJdT, double* h_dJdtau, double* d_dJdQ,
                       const bte_opts* opts, void* hip_stream, bte_report* h_rep) {
  ErrClear clear_on_exit;
  if (h && h->inst.size() != 1) {
    set_err("bte_adjoint needs a single-instance handle (use bte_batch_adjoint)");
    return BTE_ERR_STATE;
  }
  double* dq[1] = {d_dJdQ};
  const double* g[1] = {d_dJdT};
  return adjoint_common(h, d_dJdT ? g : nullptr, h_dJdtau, dq, opts, hip_stream, h_rep);
}

bte_status bte_batch_adjoint(bte_handle h, const double* const* d_dJdT, double* h_dJdtau,
                             double* const* d_dJdQ, const bte_opts* opts, void* hip_stream,
                             bte_report* h_reps) {
  ErrClear clear_on_exit;
  return adjoint_common(h, d_dJdT, h_dJdtau, d_dJdQ, opts, hip_stream, h_reps);
}

bte_status bte_adjoint_dscale(bte_handle h, double* h_dJds) {
  ErrClear clear_on_exit;
  if (!h || !h_dJds) {
    set_err("null handle or output");
    return BTE_ERR_INVALID;
  }
  for (auto& I : h->inst)
    if (!I.have_dJds) {
      set_err("bte_adjoint_dscale needs a previous bte_adjoint or bte_batch_adjoint");
      return BTE_ERR_STATE;
    }
  for (size_t k = 0; k < h->inst.size(); ++k) h_dJds[k] = h->inst[k].dJds;
  return BTE_OK;
}

bte_status bte_get_paths(bte_handle h, unsigned* paths) {
  if (!h || !paths) {
    set_err("null handle or output");
    return BTE_ERR_INVALID;
  }
  unsigned p = h->d_film ? BTE_PATH_FILM : 0u;
  const auto all = [&](auto f) { return std::all_of(h->inst.begin(), h->inst.end(), f); };
  if (all([](const Inst& I) { return I.d_cell_of != nullptr; })) p |= BTE_PATH_PLANE_BLOCKS;
  if (h->order == 2 && all([](const Inst& I) { return I.ctab_ok; })) p |= BTE_PATH_CORR_MARCH;
  *paths = p;
  return BTE_OK;
}

bte_status bte_time_sweep(bte_handle h, int n_launches, void* hip_stream, double* h_ms, double* h_updates) {
  ErrClear clear_on_exit;
  if (!h || n_launches < 1 || !h_ms) {
    set_err("null handle/output or n_launches < 1");
    return BTE_ERR_INVALID;
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  if (h->pool_mode == DevPool::COUNT) {
    set_err("bte_time_sweep needs a previous solve");
    return BTE_ERR_STATE;
  }
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  const int mode = h->order == 2 ? SWEEP_SECOND : SWEEP_PLAIN;
  // films that one launch iterates: n_launches iterations of it
  const bte_opts film_opts{};
  auto run = [&](int n) {
    if (h->d_film) return enqueue_film(h, false, n, film_opts, st, FILM_TIMING);
    bte_status r = BTE_OK;
    for (int i = 0; i < n && r == BTE_OK; ++i) r = enqueue_sweep(h, false, 1, mode, 1, st);
    return r;
  };
  bte_status s = run(1);  // warm-up
  if (s != BTE_OK) return s;
  HIPCHK(hipEventRecord(e0, st));
  s = run(n_launches);
  HIPCHK(hipEventRecord(e1, st));
  HIPCHK(hipEventSynchronize(e1));
  float ms = 0.f;
  HIPCHK(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (s != BTE_OK) return s;
  *h_ms = ms / n_launches;
  if (h_updates) {
    double u = 0.0;
    for (auto& I : h->inst) u += (double)I.hi.n_active * h->ords.size() * h->B;
    *h_updates = u;
  }
  return BTE_OK;
}

bte_status bte_autotune(bte_handle h, const double* d_Q, int n_iters, void* hip_stream, bte_plan* best) {
  ErrClear clear_on_exit;
  if (!h || n_iters < 1) {
    set_err("null handle or n_iters < 1");
    return BTE_ERR_INVALID;
  }
  if (d_Q && h->inst.size() > 1) {
    // one source array cannot serve instances of different sizes
    set_err("bte_autotune on a batch handle takes d_Q = NULL (the timing runs use a zero source)");
    return BTE_ERR_STATE;
  }
  bte_status s = ensure_device(h);
  if (s != BTE_OK) return s;
  Plan bp;
  s = autotune_impl(h, d_Q, n_iters, reinterpret_cast<hipStream_t>(hip_stream), &bp);
  if (s != BTE_OK) return s;
  if (best) {
    best->G = bp.G;
    best->R = bp.R;
    best->P = bp.P;
    best->C = bp.C;
    best->NR = bp.NR;
  }
  return BTE_OK;
}

}  // extern "C"

namespace {

bte_status autotune_impl(bte_ctx* h, const double* d_Q, int n_iters, hipStream_t st, Plan* best) {
  // the timing runs write their flux into the handle's own buffers, never into
  // an output array of an earlier call
  for (size_t k = 0; k < h->inst.size(); ++k) h->fin_f[k].q = h->inst[k].d_qbuf;
  HIPCHK(hipMemcpyAsync(h->d_fin_f, h->fin_f.data(), h->fin_f.size() * sizeof(FinInst), hipMemcpyHostToDevice,
                        st));
  std::vector<Plan> cand;
  if (h->dim == 3) {
    for (int P : {1, 2, 4, 8}) cand.push_back(Plan{1, 1, P, kC2, 1});
    for (int G : {1, 2, 4})
      for (int P : {1, 2, 4, 8})
        for (int C : {8, 16, 32}) cand.push_back(Plan{G, 1, P, C, 0});
  } else {
    int ny = 1;
    for (auto& I : h->inst) ny = std::max(ny, I.hi.n[1]);
    for (int NR : {1, 2, 4}) {
      if (NR > 1 && 32 * NR >= ny) continue;  // mostly idle rows
      const int nS = (ny + 64 * NR - 1) / (64 * NR);
      for (int G : {1, 2})
        for (int R = 1; R <= std::min(4, nS); R *= 2)
          for (int P : {1, 2, 4})
            if (R * P <= 4) cand.push_back(Plan{G, R, P, kC2, NR});
    }
  }
  // the current plan is timed first and kept unless another is at least 3%
  // faster, so that timing noise does not flip between near-equal shapes
  const Plan keep = h->plan;
  cand.insert(cand.begin(), keep);
  double best_ms = 1e300;
  Plan bestp = keep;
  // each candidate is timed on whole iterations (sweep, finalize, wall update)
  // from a fresh state, the way the solve loop runs them
  bte_opts to{};
  to.tol_T = 0.0;
  to.tol_q = 0.0;
  to.max_iters = n_iters;
  to.check_every = n_iters;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  for (size_t ci = 0; ci < cand.size(); ++ci) {
    const Plan& p = cand[ci];
    if (build_plan(h, p) != BTE_OK) continue;
    bool ok = true;
    for (size_t k = 0; k < h->inst.size() && ok; ++k)
      ok = init_forward(h, k, d_Q, nullptr, st) == BTE_OK;
    if (ok) ok = enqueue_chunk(h, false, 1, to, st) == BTE_OK;  // warm-up
    for (size_t k = 0; k < h->inst.size() && ok; ++k)
      ok = init_forward(h, k, d_Q, nullptr, st) == BTE_OK;
    double ms = 0.0;
    if (ok) ok = hipEventRecord(e0, st) == hipSuccess && enqueue_chunk(h, false, n_iters, to, st) == BTE_OK &&
                 hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
    if (ok) {
      float f = 0.f;
      ok = hipEventElapsedTime(&f, e0, e1) == hipSuccess;
      ms = f;
    }
    if (ok && (ci == 0 ? ms < best_ms : ms < 0.97 * best_ms)) {
      best_ms = ms;
      bestp = h->plan;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  bte_status s = build_plan(h, bestp);
  if (s != BTE_OK) {
    restore_plan(h, keep, h->order);
    return s;
  }
  h->auto_plan = false;
  if (best) *best = bestp;
  return BTE_OK;
}

}  // namespace

extern "C" {

bte_status bte_destroy(bte_handle h) {
  ErrClear clear_on_exit;
  if (h) release_static_scratch(h);
  delete h;
  return BTE_OK;
}

}  // extern "C"
