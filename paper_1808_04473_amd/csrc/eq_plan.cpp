// Ragged-batch plans: host-side descriptor table, cost-ordered work items
// (rounds of whole systems, row pieces of large systems, rounds of clusters),
// the autotuner (with a JSON cache keyed by device, mode, precision and tile
// class) and hipGraph capture of the launch.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <string>
#include <vector>

#include "eq_ragged.h"

using namespace dbpeq;

namespace {
constexpr int kClasses = EQ_PLAN_CLASSES;  // tile classes: padded users 16, 32
constexpr int kDefaultRows = 256;
constexpr int kDefaultWpc = 8;
inline int cls_of(int ut) { return ut == 16 ? 0 : 1; }
constexpr int kHeads = kQueues * kQueueStride;  // scratch words of the queue heads
constexpr int kList = kHeads + 64;              // first word of the FP64 list
}  // namespace

struct eq_plan {
  int fd = 0, prec = 0;
  float es = 1.f;
  int nsys = 0, ncl = 0;
  std::vector<RSys> sys;
  std::vector<int32_t> offs;
  std::vector<int32_t> cl_sys;  // system of each global cluster
  // launch shape: workgroups per CU of the persistent grid, and per tile class
  // the row count above which a PD system is cut into pieces (0 = never)
  int wpc = kDefaultWpc;
  int piece_rows[kClasses] = {kDefaultRows, kDefaultRows};
  bool tuned_launch = false;
  bool tuned_rows[kClasses] = {false, false};
  int built_rows[kClasses] = {-1, -1};  // piece_rows the device tables were built for
  std::string cache_path;
  int cus = 0;
  // per class: systems, items, pieces (PD) or clusters (FD)
  int n_sys[kClasses] = {0, 0}, n_items[kClasses] = {0, 0}, n_pieces[kClasses] = {0, 0};
  int ntasks = 0;
  size_t cap_slots = 0;
  // device memory owned by the plan
  RSys *d_sys = nullptr;
  int32_t *d_offs = nullptr;
  int32_t *d_clsys = nullptr;
  RTask *d_tasks = nullptr;
  int32_t *d_order = nullptr;
  int32_t *d_scratch = nullptr;  // [0, kHeads) queue heads, [kHeads] FP64 count, [kHeads + 1] FP64 blocks done,
                                 // [kList, kList + nsys) FP64 list, [kList + nsys, kList + 2 nsys) arrivals
  float *d_part = nullptr;       // PD partial slots
  float *d_fpart = nullptr;      // FD fusion terms
  int32_t *d_fcode = nullptr;    // FD failure codes
  // captured graph and the arguments it was captured with
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  const void *gargs[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  hipStream_t cap = nullptr;
  // recorded after every graph launch: the executable graph is destroyed
  // (re-capture, plan destruction) only once its last launch has finished
  hipEvent_t done = nullptr;
};

namespace {

bool refining(const eq_plan &p) { return p.prec == EQ_BF16_REFINE || p.prec == EQ_BF16X3_REFINE; }

// Rows per row block of the streaming layout (the unit of a piece).
int rows_per_block(int ut) { return 8 * (64 / ut); }

double gram_cost(int rows, int ut) { return (double)rows * ut * ut; }
double solve_cost(int ut) { return 4.0 * ut * ut * ut; }

// Builds the work items for the given piece rows (PD) and uploads them with
// the updated descriptor table; the items are sorted by cost, largest first.
eq_status build_items(eq_plan *p, const int (&rows)[kClasses]) {
  bool same = p->d_tasks != nullptr;
  for (int c = 0; c < kClasses; ++c) same = same && p->built_rows[c] == rows[c];
  if (same) return EQ_OK;
  std::vector<RTask> tasks;
  std::vector<double> cost;
  std::vector<int32_t> order;
  for (int c = 0; c < kClasses; ++c) p->n_sys[c] = p->n_items[c] = p->n_pieces[c] = 0;
  for (const RSys &d : p->sys) ++p->n_sys[cls_of(d.ut)];
  size_t nslots = 0;
  if (!p->fd) {
    std::vector<int32_t> whole;
    for (int k = 0; k < p->nsys; ++k) {
      RSys &d = p->sys[k];
      const int cl = cls_of(d.ut);
      const int R = refining(*p) ? 0 : rows[cl];
      const int rpb = rows_per_block(d.ut);
      d.npieces = 1;
      d.slot0 = 0;
      if (R > 0 && d.B > R) {
        const int nb = (d.B + rpb - 1) / rpb;
        const int per = std::max(1, R / rpb);
        const int np = (nb + per - 1) / per;
        d.npieces = np;
        d.slot0 = (int32_t)nslots;
        nslots += np;
        for (int q = 0; q < np; ++q) {
          const int r0 = std::min(d.B, (int)((long long)nb * q / np) * rpb);
          const int r1 = std::min(d.B, (int)((long long)nb * (q + 1) / np) * rpb);
          tasks.push_back(RTask{kItemPiece, d.ut, d.U, k, 0, r0, r1, q});
          cost.push_back(gram_cost(r1 - r0, d.ut) + (q == np - 1 ? solve_cost(d.ut) : 0.0));
          ++p->n_items[cl];
          ++p->n_pieces[cl];
        }
      } else {
        whole.push_back(k);
      }
    }
    // rounds of up to 64/UT whole systems of equal U, largest first within a
    // U; with pieces on, a round holds at most the class's piece rows (or its
    // first system), so that no round streams much more than a piece
    std::stable_sort(whole.begin(), whole.end(), [&](int a, int b) {
      if (p->sys[a].U != p->sys[b].U) return p->sys[a].U < p->sys[b].U;
      return p->sys[a].B > p->sys[b].B;
    });
    size_t k = 0;
    while (k < whole.size()) {
      const RSys &d = p->sys[whole[k]];
      const int per = 64 / d.ut;
      const int R = refining(*p) ? 0 : rows[cls_of(d.ut)];
      int m = 0, nrows = 0;
      double cst = solve_cost(d.ut);
      while (m < per && k + m < whole.size() && p->sys[whole[k + m]].U == d.U &&
             (m == 0 || R == 0 || nrows + p->sys[whole[k + m]].B <= R)) {
        nrows += p->sys[whole[k + m]].B;
        cst += gram_cost(p->sys[whole[k + m]].B, d.ut);
        ++m;
      }
      tasks.push_back(RTask{kItemGroup, d.ut, d.U, (int32_t)order.size(), m, 0, 0, 0});
      cost.push_back(cst);
      ++p->n_items[cls_of(d.ut)];
      for (int j = 0; j < m; ++j) order.push_back(whole[k + j]);
      k += m;
    }
  } else {
    // rounds of up to 64/UT clusters of equal U: the clusters of each U in
    // system order (largest systems first), so that a system's clusters share
    // few rounds
    std::vector<int32_t> ks(p->nsys);
    for (int k = 0; k < p->nsys; ++k) ks[k] = k;
    std::stable_sort(ks.begin(), ks.end(), [&](int a, int b) {
      if (p->sys[a].U != p->sys[b].U) return p->sys[a].U < p->sys[b].U;
      return p->sys[a].B > p->sys[b].B;
    });
    size_t k = 0;
    while (k < ks.size()) {
      const int U = p->sys[ks[k]].U, ut = p->sys[ks[k]].ut;
      std::vector<int32_t> cls;
      for (; k < ks.size() && p->sys[ks[k]].U == U; ++k) {
        const RSys &d = p->sys[ks[k]];
        for (int c = 0; c < d.C; ++c) cls.push_back(d.cl0 + c);
      }
      p->n_pieces[cls_of(ut)] += (int)cls.size();
      const int per = 64 / ut;
      for (size_t j = 0; j < cls.size(); j += per) {
        const int m = (int)std::min<size_t>(per, cls.size() - j);
        double cst = solve_cost(ut);
        for (int q = 0; q < m; ++q) {
          const int gc = cls[j + q];
          const RSys &d = p->sys[p->cl_sys[gc]];
          const int c = gc - d.cl0;
          cst += gram_cost(p->offs[d.off_first + c + 1] - p->offs[d.off_first + c], ut);
        }
        tasks.push_back(RTask{kItemRound, ut, U, (int32_t)(order.size() + j), m, 0, 0, 0});
        cost.push_back(cst);
        ++p->n_items[cls_of(ut)];
      }
      order.insert(order.end(), cls.begin(), cls.end());
    }
  }
  std::vector<int> ti(tasks.size());
  for (size_t t = 0; t < ti.size(); ++t) ti[t] = (int)t;
  std::stable_sort(ti.begin(), ti.end(), [&](int a, int b) { return cost[a] > cost[b]; });
  std::vector<RTask> sorted;
  sorted.reserve(tasks.size());
  for (int t : ti) sorted.push_back(tasks[t]);
  p->ntasks = (int)sorted.size();
  // the previous tables: a failed free leaves nothing this call could repair
  if (p->d_tasks) (void)hipFree(p->d_tasks);
  p->d_tasks = nullptr;
  if (p->d_order) (void)hipFree(p->d_order);
  p->d_order = nullptr;
  if (hipMalloc(&p->d_tasks, sizeof(RTask) * std::max<size_t>(1, sorted.size())) != hipSuccess ||
      hipMalloc(&p->d_order, sizeof(int32_t) * std::max<size_t>(1, order.size())) != hipSuccess)
    return EQ_ENOMEM;
  if (nslots > p->cap_slots) {
    if (p->d_part) (void)hipFree(p->d_part);
    p->d_part = nullptr;
    p->cap_slots = 0;
    if (hipMalloc(&p->d_part, sizeof(float) * kPartStride * nslots) != hipSuccess) return EQ_ENOMEM;
    p->cap_slots = nslots;
  }
  if ((!sorted.empty() &&
       hipMemcpy(p->d_tasks, sorted.data(), sizeof(RTask) * sorted.size(), hipMemcpyHostToDevice) != hipSuccess) ||
      (!order.empty() &&
       hipMemcpy(p->d_order, order.data(), sizeof(int32_t) * order.size(), hipMemcpyHostToDevice) != hipSuccess) ||
      hipMemcpy(p->d_sys, p->sys.data(), sizeof(RSys) * p->nsys, hipMemcpyHostToDevice) != hipSuccess)
    return EQ_EHIP;
  for (int c = 0; c < kClasses; ++c) p->built_rows[c] = rows[c];
  return EQ_OK;
}

eq_status build_current(eq_plan *p) { return build_items(p, p->piece_rows); }

// Tuning cache keys: device, mode, precision and, for the piece rows, the
// tile class, so that any batch drawn from the same distribution finds them.
std::string key_launch(const eq_plan &p) {
  char buf[64];
  snprintf(buf, sizeof(buf), "gfx950/%s/p%d/launch", p.fd ? "fd" : "pd", p.prec);
  return buf;
}
std::string key_rows(const eq_plan &p, int cls) {
  char buf[64];
  snprintf(buf, sizeof(buf), "gfx950/%s/p%d/ut%d", p.fd ? "fd" : "pd", p.prec, cls == 0 ? 16 : 32);
  return buf;
}

bool is_launch_key(const std::string &k) { return k.size() >= 7 && k.compare(k.size() - 7, 7, "/launch") == 0; }
bool is_fd_key(const std::string &k) { return k.find("/fd/") != std::string::npos; }

// The cache is a JSON object with one entry per line:
//   "<mode key>/launch": {"wpc": W},   "<mode key>/utNN": {"piece_rows": R},
// FD launches also hold the waves of the workgroups that were timed, and are
// tuned again where those were others: {"wpc": W, "waves": N}.
std::map<std::string, int> read_cache(const std::string &path) {
  std::map<std::string, int> m;
  if (path.empty()) return m;
  FILE *f = fopen(path.c_str(), "r");
  if (!f) return m;
  char line[512];
  while (fgets(line, sizeof(line), f)) {
    char key[256];
    int v = 0, waves = 1;
    if (sscanf(line, " \"%255[^\"]\": {\"wpc\": %d, \"waves\": %d}", key, &v, &waves) >= 2) {
      if (v >= 1 && v <= 64 && (!is_fd_key(key) || waves == kRaggedWaves)) m[key] = v;
    } else if (sscanf(line, " \"%255[^\"]\": {\"piece_rows\": %d}", key, &v) == 2) {
      if (v == 0 || (v >= 16 && v <= EQ_MAX_B)) m[key] = v;
    }
  }
  fclose(f);
  return m;
}

void write_cache(const std::string &path, const std::map<std::string, int> &m) {
  if (path.empty()) return;
  const std::string tmp = path + ".tmp";
  FILE *f = fopen(tmp.c_str(), "w");
  if (!f) return;
  fprintf(f, "{\n");
  size_t n = 0;
  for (const auto &kv : m) {
    ++n;
    const bool launch = is_launch_key(kv.first);
    fprintf(f, "  \"%s\": {\"%s\": %d", kv.first.c_str(), launch ? "wpc" : "piece_rows", kv.second);
    if (launch && is_fd_key(kv.first)) fprintf(f, ", \"waves\": %d", kRaggedWaves);
    fprintf(f, "}%s\n", n < m.size() ? "," : "");
  }
  fprintf(f, "}\n");
  fclose(f);
  rename(tmp.c_str(), path.c_str());
}

RaggedArgs make_args(const eq_plan *p, const eq_c32 *H, const eq_c32 *y, eq_c32 *z, float *s2, int32_t *info) {
  RaggedArgs a;
  memset(&a, 0, sizeof(a));
  a.Hpool = reinterpret_cast<const float2 *>(H);
  a.ypool = reinterpret_cast<const float2 *>(y);
  a.zpool = reinterpret_cast<float2 *>(z);
  a.s2pool = s2;
  a.info = info;
  a.sys = p->d_sys;
  a.offs = p->d_offs;
  a.tasks = p->d_tasks;
  a.order = p->d_order;
  a.cl_sys = p->d_clsys;
  a.counter = p->d_scratch;
  a.fb_count = p->d_scratch + kHeads;
  a.fb_done = p->d_scratch + kHeads + 1;
  a.fb_list = p->d_scratch + kList;
  a.arrive = p->d_scratch + kList + p->nsys;
  a.part = p->d_part;
  a.fpart = p->d_fpart;
  a.fcode = p->d_fcode;
  a.nsys = p->nsys;
  a.ntasks = p->ntasks;
  a.es = p->es;
  return a;
}

// Persistent workgroups: CUs x workgroups per CU, at most one per item, and at
// least one per queue that holds items (queue q holds the items t with t % kQueues == q).
int grid_of(const eq_plan *p, int wpc) {
  const int g = std::min(p->cus * wpc, p->ntasks);
  return std::max(1, std::max(g, std::min(kQueues, p->ntasks)));
}

// Queue heads, FP64 count and arrival counters to zero.
hipError_t clear_scratch(const eq_plan *p, hipStream_t s) {
  return launch_zero_i32(p->d_scratch, kList + 2 * p->nsys, s);
}

// Runs the persistent launch, then (fp64) the FP64 re-solve of the systems it
// queued.  With fp64 the scratch is left at zero for the next execution
// (finishers reset their arrival counters, the FP64 launch the queue heads
// and its count); without it (autotuning) the scratch is cleared first, and
// clear_scratch must run once more before the next fp64 execution.
hipError_t enqueue(const eq_plan *p, int wpc, bool fp64, const eq_c32 *H, const eq_c32 *y, eq_c32 *z,
                   float *s2, int32_t *info, hipStream_t s) {
  hipError_t e;
  if (!fp64 && (e = clear_scratch(p, s)) != hipSuccess) return e;
  const RaggedArgs a = make_args(p, H, y, z, s2, info);
  if ((e = launch_ragged(a, p->fd != 0, p->prec, grid_of(p, wpc), s)) != hipSuccess) return e;
  return fp64 ? launch_fp64_ragged(a, p->fd != 0, s) : hipSuccess;
}

// Capture stream and launch event (created once per plan).
hipError_t make_streams(eq_plan *p) {
  hipError_t e = hipSuccess;
  if (!p->cap && (e = hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking)) != hipSuccess) return e;
  if (!p->done && (e = hipEventCreateWithFlags(&p->done, hipEventDisableTiming)) != hipSuccess) return e;
  return hipSuccess;
}

// Times the launch on the real pools for each candidate of whatever the
// cache did not hold: first the workgroups per CU (with the current piece rows),
// then, for PD outside the refining forms, the piece rows of each tile class
// that has systems.  Keeps the fastest of each.
eq_status autotune(eq_plan *p, const eq_c32 *H, const eq_c32 *y, eq_c32 *z, float *s2, int32_t *info,
                   hipStream_t s) {
  struct Events {
    hipEvent_t e[2] = {nullptr, nullptr};
    ~Events() {
      for (hipEvent_t x : e)
        if (x) (void)hipEventDestroy(x);
    }
  } ev;
  if (hipEventCreate(&ev.e[0]) != hipSuccess || hipEventCreate(&ev.e[1]) != hipSuccess) return EQ_EHIP;
  eq_status st = EQ_OK;
  auto time = [&](const int (&rows)[kClasses], int wpc, float &best) -> eq_status {
    eq_status bst = build_items(p, rows);
    if (bst != EQ_OK) return bst;
    best = 1e30f;
    for (int rep = 0; rep < 3; ++rep) {
      if (hipEventRecord(ev.e[0], s) != hipSuccess || enqueue(p, wpc, false, H, y, z, s2, info, s) != hipSuccess ||
          hipEventRecord(ev.e[1], s) != hipSuccess || hipEventSynchronize(ev.e[1]) != hipSuccess)
        return EQ_EHIP;
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, ev.e[0], ev.e[1]) != hipSuccess) return EQ_EHIP;
      best = std::min(best, ms);
    }
    return EQ_OK;
  };
  auto m = read_cache(p->cache_path);
  if (!p->tuned_launch) {
    // one-wave workgroups: the kernels' registers (2 to 3 waves per SIMD) and
    // LDS (13.3 KB a wave) hold 8 to 11 on a CU; FD workgroups of two waves
    // (launch_ragged): 6.  Larger grids only queue workgroups that find the
    // queues empty.
    const int wpcs[] = {4, 6, 8};
    float tbest = 1e30f;
    for (int w : wpcs) {
      float t = 0.f;
      if ((st = time(p->piece_rows, w, t)) != EQ_OK) return st;
      if (t < tbest) {
        tbest = t;
        p->wpc = w;
      }
    }
    p->tuned_launch = true;
    m[key_launch(*p)] = p->wpc;
  }
  for (int c = 0; c < kClasses; ++c) {
    if (p->tuned_rows[c] || p->fd || refining(*p) || p->n_sys[c] == 0) continue;
    const int cand[] = {0, 256, 384, 512, 768};
    float tbest = 1e30f;
    int best = p->piece_rows[c];
    for (int r : cand) {
      int rows[kClasses] = {p->piece_rows[0], p->piece_rows[1]};
      rows[c] = r;
      float t = 0.f;
      if ((st = time(rows, p->wpc, t)) != EQ_OK) return st;
      if (t < tbest) {
        tbest = t;
        best = r;
      }
    }
    p->piece_rows[c] = best;
    p->tuned_rows[c] = true;
    m[key_rows(*p, c)] = best;
  }
  write_cache(p->cache_path, m);
  // the timed launches ran without the FP64 launch that clears the scratch
  if (clear_scratch(p, s) != hipSuccess) return EQ_EHIP;
  return build_current(p);
}

void drop_graph(eq_plan *p) {
  // a launch still in flight uses the executable graph's kernel arguments; a
  // failed wait leaves nothing better than destroying it
  if (p->exec && p->done) (void)hipEventSynchronize(p->done);
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  p->exec = nullptr;
  p->graph = nullptr;
}

// Whether every tuned quantity the plan uses is known.
bool all_tuned(const eq_plan *p) {
  if (!p->tuned_launch) return false;
  if (p->fd || refining(*p)) return true;
  for (int c = 0; c < kClasses; ++c)
    if (!p->tuned_rows[c] && p->n_sys[c] > 0) return false;
  return true;
}

}  // namespace

extern "C" {

eq_status eq_plan_create(eq_plan **out, const eq_sys *desc, int32_t nsys, const int32_t *sizes,
                         int32_t nsizes, int32_t fd, int32_t precision, float es,
                         const char *tune_cache_path) {
  if (!out) return EQ_EINVAL;
  *out = nullptr;
  if (nsys < 1 || !desc || !sizes || nsizes < 1) return EQ_EINVAL;
  if (fd != 0 && fd != 1) return EQ_EINVAL;
  if (precision < EQ_FP32 || precision > EQ_BF16X3) return EQ_EINVAL;
  // FD fuses with weights from diag(A_c^{-1}), which the refinement step does
  // not correct: the single-BF16 Gram leaves them about 1e-3 off
  if (fd && precision == EQ_BF16_REFINE) return EQ_ENOTSUP;
  if (!isfinite(es) || !(es > 0.f)) return EQ_EINVAL;
  eq_plan *p = new eq_plan();
  p->fd = fd;
  p->prec = precision;
  p->es = es;
  p->nsys = nsys;
  p->sys.resize(nsys);
  for (int k = 0; k < nsys; ++k) {
    const eq_sys &d = desc[k];
    const bool ok = d.B >= 1 && d.B <= EQ_MAX_B && d.U >= 1 && d.C >= 1 && d.C <= d.B &&
                    d.C <= EQ_MAX_C && d.h_off >= 0 && d.y_off >= 0 && d.z_off >= 0 &&
                    d.clus_first >= 0 && (int64_t)d.clus_first + d.C <= nsizes && isfinite(d.n0) &&
                    d.n0 > 0.f && isfinite(d.n0 / es) && d.n0 / es > 0.f;
    if (!ok) {
      delete p;
      return d.U > EQ_MAX_U || d.B > EQ_MAX_B ? EQ_ENOTSUP : EQ_EINVAL;
    }
    if (d.U > EQ_MAX_U) {
      delete p;
      return EQ_ENOTSUP;
    }
    RSys &r = p->sys[k];
    r.h_off = d.h_off;
    r.y_off = d.y_off;
    r.z_off = d.z_off;
    r.B = d.B;
    r.U = d.U;
    r.C = d.C;
    r.n0 = d.n0;
    r.rho = d.n0 / es;
    r.ut = ut_for(d.U);
    r.npieces = 1;
    r.slot0 = 0;
    r.cl0 = (int32_t)p->cl_sys.size();
    r.off_first = (int32_t)p->offs.size();
    int acc = 0;
    p->offs.push_back(0);
    for (int c = 0; c < d.C; ++c) {
      const int sz = sizes[d.clus_first + c];
      if (sz < 1) {
        delete p;
        return EQ_EINVAL;
      }
      acc += sz;
      p->offs.push_back(acc);
      p->cl_sys.push_back(k);
    }
    if (acc != d.B) {
      delete p;
      return EQ_EINVAL;
    }
  }
  p->ncl = (int)p->cl_sys.size();
  p->cache_path = tune_cache_path ? tune_cache_path : (getenv("DBPEQ_TUNE_CACHE") ? getenv("DBPEQ_TUNE_CACHE") : "");
  {
    auto m = read_cache(p->cache_path);
    auto it = m.find(key_launch(*p));
    if (it != m.end()) {
      p->wpc = it->second;
      p->tuned_launch = true;
    }
    for (int c = 0; c < kClasses; ++c) {
      auto jt = m.find(key_rows(*p, c));
      if (jt != m.end()) {
        p->piece_rows[c] = jt->second;
        p->tuned_rows[c] = true;
      }
    }
  }
  {
    int dev = 0;
    hipDeviceProp_t prop;
    p->cus = hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess &&
                     prop.multiProcessorCount > 0
                 ? prop.multiProcessorCount
                 : 256;
  }
  bool ok = hipMalloc(&p->d_sys, sizeof(RSys) * nsys) == hipSuccess &&
            hipMalloc(&p->d_offs, sizeof(int32_t) * p->offs.size()) == hipSuccess &&
            hipMalloc(&p->d_scratch, sizeof(int32_t) * (kList + 2 * (size_t)nsys)) == hipSuccess;
  if (ok && fd)
    ok = hipMalloc(&p->d_clsys, sizeof(int32_t) * p->ncl) == hipSuccess &&
         hipMalloc(&p->d_fpart, sizeof(float) * 4 * kFusionStride * (size_t)p->ncl) == hipSuccess &&
         hipMalloc(&p->d_fcode, sizeof(int32_t) * 2 * (size_t)p->ncl) == hipSuccess;
  if (!ok) {
    eq_plan_destroy(p);
    return EQ_ENOMEM;
  }
  // executions start from zeroed scratch and leave it so (enqueue); the wait
  // covers callers whose stream does not wait on the null stream
  if (hipMemset(p->d_scratch, 0, sizeof(int32_t) * (kList + 2 * (size_t)nsys)) != hipSuccess ||
      hipStreamSynchronize(nullptr) != hipSuccess ||
      hipMemcpy(p->d_offs, p->offs.data(), sizeof(int32_t) * p->offs.size(), hipMemcpyHostToDevice) != hipSuccess ||
      (fd && hipMemcpy(p->d_clsys, p->cl_sys.data(), sizeof(int32_t) * p->ncl, hipMemcpyHostToDevice) != hipSuccess)) {
    eq_plan_destroy(p);
    return EQ_EHIP;
  }
  eq_status st = build_current(p);
  if (st != EQ_OK) {
    eq_plan_destroy(p);
    return st;
  }
  *out = p;
  return EQ_OK;
}

eq_status eq_plan_execute(eq_plan *p, const eq_c32 *H, const eq_c32 *y, eq_c32 *z, float *s2, int32_t *info,
                          void *stream) {
  if (!p || !H || !y || !z) return EQ_EINVAL;
  if (((uintptr_t)H % 8) || ((uintptr_t)y % 8) || ((uintptr_t)z % 8) || ((uintptr_t)s2 % 4) ||
      ((uintptr_t)info % 4))
    return EQ_EINVAL;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (!all_tuned(p)) {
    drop_graph(p);
    eq_status st = autotune(p, H, y, z, s2, info, s);
    if (st != EQ_OK) return st;
  }
  eq_status st = build_current(p);
  if (st != EQ_OK) return st;
  const void *args[5] = {H, y, z, s2, info};
  bool same = p->exec != nullptr;
  for (int k = 0; k < 5 && same; ++k) same = args[k] == p->gargs[k];
  if (!same) {
    drop_graph(p);
    if (make_streams(p) != hipSuccess) return EQ_EHIP;
    if (hipStreamBeginCapture(p->cap, hipStreamCaptureModeRelaxed) != hipSuccess) return EQ_EHIP;
    hipError_t e = enqueue(p, p->wpc, true, H, y, z, s2, info, p->cap);
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(p->cap, &g);
    if (e != hipSuccess || e2 != hipSuccess || !g) {
      if (g) (void)hipGraphDestroy(g);
      return EQ_EHIP;
    }
    p->graph = g;
    if (hipGraphInstantiate(&p->exec, g, nullptr, nullptr, 0) != hipSuccess) {
      drop_graph(p);
      return EQ_EHIP;
    }
    for (int k = 0; k < 5; ++k) p->gargs[k] = args[k];
  }
  if (hipGraphLaunch(p->exec, s) != hipSuccess || hipEventRecord(p->done, s) != hipSuccess) return EQ_EHIP;
  return EQ_OK;
}

eq_status eq_plan_describe(const eq_plan *p, int32_t *out_shape, int32_t *out_tasks) {
  if (!p) return EQ_EINVAL;
  if (out_shape) {
    for (int c = 0; c < kClasses; ++c) {
      int32_t *o = out_shape + 5 * c;
      o[0] = p->n_sys[c];
      o[1] = p->n_items[c];
      o[2] = p->n_pieces[c];
      o[3] = p->fd || refining(*p) ? 0 : p->piece_rows[c];
      o[4] = grid_of(p, p->wpc);
    }
  }
  if (out_tasks) *out_tasks = p->ntasks;
  return EQ_OK;
}

eq_status eq_plan_destroy(eq_plan *p) {
  if (!p) return EQ_OK;
  drop_graph(p);
  // release everything, then report whether any release failed
  bool ok = true;
  if (p->cap) ok &= hipStreamDestroy(p->cap) == hipSuccess;
  if (p->done) ok &= hipEventDestroy(p->done) == hipSuccess;
  for (void *d : {(void *)p->d_sys, (void *)p->d_offs, (void *)p->d_clsys, (void *)p->d_tasks, (void *)p->d_order,
                  (void *)p->d_scratch, (void *)p->d_part, (void *)p->d_fpart, (void *)p->d_fcode})
    if (d) ok &= hipFree(d) == hipSuccess;
  delete p;
  return ok ? EQ_OK : EQ_EHIP;
}

}  // extern "C"
