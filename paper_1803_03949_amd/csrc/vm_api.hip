// C-ABI of the voxmesh library: argument checks, workspace layout, pose
// inversion and the kernel sequence of each call.  No device allocation:
// every byte lives in the caller's buffer.
#include <math.h>
#include <stddef.h>
#include <string.h>

#include <hip/hip_ext.h>

#include <mutex>
#include <new>
#include <tuple>
#include <utility>
#include <vector>

#include "voxmesh.h"
#include "vm_internal.h"

namespace vm {
void build_mc_tables(uint8_t* tri, uint8_t* uses);
}

using namespace vm;

struct vm_volume {
  struct ProfRec {
    int kid;
    hipEvent_t a, b;
  };
  // A captured phase of vm_extract_batch with what it was captured for,
  // and the host-side state the captured forward left.
  struct BatchGraph {
    hipGraphExec_t exec = nullptr;
    vm_batch_io io;
    vm_launch launch;
    const float* d;
    const float* w;
    uint32_t frame, epoch, pass, xcount, vcount, xsel, vsel, dev_frame;
  };
  vm_config cfg;
  char* mem;
  size_t bytes;
  VolDev dev;
  float* own_d;     // the workspace's TSDF and weight arrays (d, w when unbound)
  float* own_w;
  uint32_t frame;   // last frame number handed to the device
  uint32_t epoch;   // extraction epoch (pending-list stamps)
  uint32_t pass;    // dirty / vertex-list stamps
  uint32_t xcount;  // extractions so far (parity selects the dirty-list length)
  int64_t dl_nv;    // vertices of the last download (-1: none since the mesh changed)
  uint64_t mesh = 0;      // number of the mesh held now (see vm_mesh_state)
  uint64_t dl_mesh = 0;   // number of the mesh last downloaded, 0: none since a reset
  int64_t dl_rows = 0;    // its vertices
  bool settled = false;   // the mesh is the plain extraction of the whole TSDF: another
                          // plain extraction leaves it as it is
  uint32_t vcount;  // extractions and refinements so far (vertex-list length)
  FrameParams last_fp;
  bool have_fp;
  bool last_refine = false;  // the last extraction-side call was a refinement
  int cus;          // compute units of the device
  vm_launch launch; // workgroup mapping (see vm_set_launch)
  int grid_blocks;  // workgroups of per-block kernels
  int grid_items;   // workgroups of per-item kernels
  int grid_waves;   // workgroups of wave-per-block kernels
  uint32_t prof;    // bit k: bracket launches of kernel k with events
  std::vector<hipEvent_t> ev_free;
  std::vector<ProfRec> recs;
  Report* rep = nullptr;      // the volume's record in pinned host memory (none: it is copied)
  Report* rep_dev = nullptr;  // the same for the device
  int rep_slot = -1;
  int scratch_dev = -1;  // device whose static workspace holds the volume, -1 if the caller's
  BatchGraph bgraph[2];  // vm_extract_batch: forward, backward
};

namespace {

uint8_t g_tri[256 * 16];
uint8_t g_uses[256 * 12];
std::once_flag g_tables_once;

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

bool config_ok(const vm_config* c) {
  return c && c->voxel_m > 0.f && isfinite(c->voxel_m) && c->trunc_vox > 0.f &&
         isfinite(c->trunc_vox) && c->refine_eps_vox >= 0.f && c->hash_log2 >= 10 &&
         c->hash_log2 <= 28 && c->max_blocks >= 1 && c->max_blocks <= kMaxBlocks &&
         c->max_vertices >= 1 && c->max_vertices <= (1 << 30) &&
         (c->hash_mode == 0 || c->hash_mode == 1) &&
         c->batch_volumes >= 0 && c->batch_volumes <= kMaxSlots;
}

bool launch_ok(const vm_launch* l) {
  return l && (l->wave_group_size == 2 || l->wave_group_size == 4 || l->wave_group_size == 8) &&
         l->wave_groups_per_cu >= 1 && l->wave_groups_per_cu <= 32 &&
         l->block_groups_per_cu >= 1 && l->block_groups_per_cu <= 16 &&
         l->item_groups_per_cu >= 1 && l->item_groups_per_cu <= 32 &&
         l->block_order >= 0 && l->block_order <= 3;
}

void apply_launch(vm_volume* vol, const vm_launch& l) {
  vol->launch = l;
  vol->grid_blocks = vol->cus * l.block_groups_per_cu;
  vol->grid_items = vol->cus * l.item_groups_per_cu;
  vol->grid_waves = vol->cus * l.wave_groups_per_cu;
  vol->dev.order = (uint32_t)l.block_order;
}

// Carve the workspace; with base == nullptr only the size is computed.
size_t carve(const vm_config& c, char* base, VolDev* v) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    void* p = base ? (void*)(base + off) : nullptr;
    off = align_up(off + bytes);
    return p;
  };
  const size_t H = (size_t)1 << c.hash_log2, B = (size_t)c.max_blocks,
               V = (size_t)c.max_vertices, C = B * kVox;
  // a download's vertex chunks (at most V / kDlSlots + nseg + 1), or three
  // counts per import part
  const size_t scan = (V > C ? V : C) / 1024 + 2 + 3 * (B / kImportRows + 1);
  v->cnt = (Counters*)take(sizeof(Counters));
  v->vseg = (Seg*)take(sizeof(Seg) * kSegs);
  v->cseg = (Seg*)take(sizeof(Seg) * kSegs);
  v->tri_table = (const uint8_t*)take(256 * 16);
  v->edge_uses = (const uint8_t*)take(256 * 12);
  v->slots = (HashSlot*)take(sizeof(HashSlot) * H);
  v->block_key = (uint64_t*)take(8 * B);
  v->nbr = (int32_t*)take(4 * 27 * B);
  v->d = (float*)take(4 * kVox * B);
  v->w = (float*)take(4 * kVox * B);
  v->tprev = (uint64_t*)take(kVox * B);
  v->tcur = (uint64_t*)take(kVox * B);
  v->evtx = (int32_t*)take(4 * 3 * kVox * B);
  v->et = (float*)take(4 * 3 * kVox * B);
  v->emask = (uint32_t*)take(4 * 64 * B);
  v->wmask = (uint64_t*)take(8 * 8 * B);
  v->smask = (uint64_t*)take(8 * 8 * B);
  v->nmask = (uint64_t*)take(8 * 8 * B);
  v->st_pending = (uint32_t*)take(4 * B);
  v->st_dirty = (uint32_t*)take(4 * B);
  v->st_vtx = (uint32_t*)take(4 * B);
  v->st_frame = (uint32_t*)take(4 * B);
  v->frame_list = (uint32_t*)take(4 * B);
  v->frame_key = (uint64_t*)take(8 * B);
  v->pending = (uint32_t*)take(4 * B);
  v->dirty = (uint32_t*)take(4 * B);
  v->btri = (uint32_t*)take(4 * B);
  v->vcand = (uint32_t*)take(4 * 8 * B);
  v->row_slot = v->vcand;
  v->frame_src = v->vcand ? v->vcand + B : nullptr;
  v->vblocks = (uint32_t*)take(4 * B);
  v->vowner = (uint32_t*)take(4 * V);
  v->vring = (uint32_t*)take(4 * V);
  v->vdl = (int32_t*)take(4 * V);
  v->vbirth = (uint32_t*)take(4 * V);
  v->scan = (uint32_t*)take(4 * scan);
  v->blank = (uint32_t*)take(4 * B);
  v->scan_cap = (uint32_t)scan;
  v->max_blocks = (uint32_t)B;
  v->max_vertices = (uint32_t)V;
  // one segment per 256 blocks of capacity, at most kSegs
  const size_t nseg = B / 256 < 1 ? 1 : (B / 256 > (size_t)kSegs ? (size_t)kSegs : B / 256);
  v->nseg = (uint32_t)nseg;
  v->vseg_cap = (uint32_t)((V + nseg - 1) / nseg);
  v->hash_mask = (uint32_t)(H - 1);
  v->hash_mode = c.hash_mode;
  return off;
}

int hip_status(hipError_t e) { return e == hipSuccess ? VM_OK : VM_ERR_HIP; }

int launched() { return hip_status(hipGetLastError()); }

int error_code(uint32_t bits) {
  for (int k = 0; k < 16; ++k)
    if (bits & (1u << k)) return -(k + 2);
  return VM_OK;
}

// Two events for timing a launch of kernel kid while it is profiled (not
// on a stream under capture: such launches run untimed).
bool prof_pair(vm_volume* vol, int kid, hipStream_t s, hipEvent_t* a, hipEvent_t* b) {
  if (!((vol->prof >> kid) & 1u)) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (s != nullptr && (hipStreamIsCapturing(s, &cs) != hipSuccess ||
                       cs != hipStreamCaptureStatusNone))
    return false;
  hipEvent_t e[2] = {nullptr, nullptr};
  for (hipEvent_t& x : e) {
    if (!vol->ev_free.empty()) {
      x = vol->ev_free.back();
      vol->ev_free.pop_back();
    } else if (hipEventCreate(&x) != hipSuccess) {
      x = nullptr;
    }
  }
  if (!e[0] || !e[1]) {
    for (hipEvent_t x : e)
      if (x) vol->ev_free.push_back(x);
    return false;
  }
  *a = e[0], *b = e[1];
  return true;
}

// A launch whose start and end the launch itself records in two events
// (hipExtLaunchKernel): no marker packets between kernels, and the time is
// the kernel's own.  The arguments are converted to the kernel's parameter
// types first.
template <typename... P, typename... A, size_t... I>
hipError_t launch_timed_at(void (*k)(P...), dim3 g, dim3 b, hipStream_t s, hipEvent_t e0,
                           hipEvent_t e1, std::index_sequence<I...>, A&&... a) {
  std::tuple<P...> t(std::forward<A>(a)...);
  void* args[] = {(void*)&std::get<I>(t)...};
  return hipExtLaunchKernel((const void*)k, g, b, args, 0, s, e0, e1, 0);
}
template <typename... P, typename... A>
hipError_t launch_timed(void (*k)(P...), dim3 g, dim3 b, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1, A&&... a) {
  return launch_timed_at(k, g, b, s, e0, e1, std::index_sequence_for<P...>{},
                         std::forward<A>(a)...);
}

// Launch a kernel; while it is profiled, the launch records its start and
// end (a timed launch that fails is made again untimed, so that timing
// never drops a kernel).
#define VM_LAUNCH(vol, kid, kernel, grid, block, stream, ...)                                \
  do {                                                                                     \
    hipEvent_t vm_a_ = nullptr, vm_b_ = nullptr;                                           \
    bool vm_done_ = false;                                                                 \
    if (prof_pair((vol), (kid), (stream), &vm_a_, &vm_b_)) {                               \
      if (launch_timed(kernel, grid, block, stream, vm_a_, vm_b_, __VA_ARGS__) == hipSuccess) { \
        (vol)->recs.push_back({(kid), vm_a_, vm_b_});                                      \
        vm_done_ = true;                                                                   \
      } else {                                                                             \
        (vol)->ev_free.push_back(vm_a_), (vol)->ev_free.push_back(vm_b_);                  \
        (void)hipGetLastError();                                                           \
      }                                                                                    \
    }                                                                                      \
    if (!vm_done_) hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);        \
  } while (0)

// Launch a wave-per-block kernel instantiated for the volume's group size.
#define VM_LAUNCH_W(vol, kid, kernel, stream, ...)                                          \
  do {                                                                                  \
    const dim3 vm_g_((vol)->grid_waves);                                                \
    switch ((vol)->launch.wave_group_size) {                                            \
      case 2: VM_LAUNCH(vol, kid, kernel<2>, vm_g_, dim3(128), stream, __VA_ARGS__); break; \
      case 8: VM_LAUNCH(vol, kid, kernel<8>, vm_g_, dim3(512), stream, __VA_ARGS__); break; \
      default: VM_LAUNCH(vol, kid, kernel<4>, vm_g_, dim3(256), stream, __VA_ARGS__); break; \
    }                                                                                   \
  } while (0)

// The same for kernels with a second, compile-time mode argument.
#define VM_LAUNCH_WM(vol, kid, kernel, mode, stream, ...)                                     \
  do {                                                                                      \
    const dim3 vm_g_((vol)->grid_waves);                                                    \
    switch ((vol)->launch.wave_group_size) {                                                \
      case 2: VM_LAUNCH(vol, kid, (kernel<2, mode>), vm_g_, dim3(128), stream, __VA_ARGS__); break; \
      case 8: VM_LAUNCH(vol, kid, (kernel<8, mode>), vm_g_, dim3(512), stream, __VA_ARGS__); break; \
      default: VM_LAUNCH(vol, kid, (kernel<4, mode>), vm_g_, dim3(256), stream, __VA_ARGS__); break; \
    }                                                                                       \
  } while (0)

void close_pool(vm_volume* vol, hipStream_t s) {
  VM_LAUNCH(vol, VM_K_COUNTERS, k_close, dim3(1), dim3(64), s, vol->dev);
}

// The mesh, or the TSDF it was extracted from, may differ from here on.
void mesh_changes(vm_volume* vol) {
  vol->dl_nv = -1;
  ++vol->mesh;
  vol->settled = false;
}

// The volume was emptied, and what the last download handed over with it.
void mesh_empty(vm_volume* vol) {
  mesh_changes(vol);
  vol->dl_mesh = 0;
  vol->dl_rows = 0;
}

// Workgroups of k_reset: the first does the bookkeeping.
unsigned reset_grid(const vm_volume* vol) {
  // four 16-byte stores per lane, at most eight workgroups per CU
  const VolDev& v = vol->dev;
  const uint64_t n16 = (uint64_t)v.hash_mask + 1 + v.max_blocks;
  const uint64_t g = (n16 + 1023) / 1024, most = (uint64_t)vol->cus * 8;
  return 1u + (unsigned)(g < 1 ? 1 : (g > most ? most : g));
}

// Empty the volume.  full = true (creation) also clears the running totals
// and uploads the marching-cubes tables.
int clear_state(vm_volume* vol, hipStream_t stream, bool full) {
  const VolDev& v = vol->dev;
  VM_LAUNCH(vol, VM_K_COUNTERS, k_reset, dim3(reset_grid(vol)), dim3(256), stream, v,
            full ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (full) {
    if (e == hipSuccess)
      e = hipMemcpyAsync((void*)v.tri_table, g_tri, sizeof(g_tri), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess)
      e = hipMemcpyAsync((void*)v.edge_uses, g_uses, sizeof(g_uses), hipMemcpyHostToDevice, stream);
    // no pool entry has a download row
    if (e == hipSuccess) e = hipMemsetAsync(v.vdl, 0xFF, 4 * (size_t)v.max_vertices, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
  }
  vol->frame = 0;
  vol->epoch = 1;
  vol->pass = 0;
  vol->last_refine = false;
  vol->have_fp = false;
  mesh_empty(vol);
  return hip_status(e);
}

// Records in pinned host memory: one allocation of kReports of them, made for
// the first volume that wants one and held until the process ends; a volume
// takes one and gives it back when it is destroyed.  A volume without one
// (all taken, no pinned memory, or a noalloc volume) copies instead.
constexpr int kReports = 256;
std::mutex g_reports_mutex;
Report* g_reports;
bool g_reports_tried;
bool g_report_used[kReports];

void take_report(vm_volume* vol) {
  std::lock_guard<std::mutex> lock(g_reports_mutex);
  if (!g_reports_tried) {
    g_reports_tried = true;
    void* p = nullptr;
    if (hipHostMalloc(&p, sizeof(Report) * kReports, hipHostMallocPortable | hipHostMallocMapped) ==
        hipSuccess)
      g_reports = (Report*)p;
    else
      (void)hipGetLastError();
  }
  for (int k = 0; g_reports && k < kReports; ++k) {
    if (g_report_used[k]) continue;
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, g_reports + k, 0) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    g_report_used[k] = true;
    vol->rep = g_reports + k, vol->rep_dev = (Report*)d, vol->rep_slot = k;
    return;
  }
}

void give_report(vm_volume* vol) {
  if (vol->rep_slot < 0) return;
  std::lock_guard<std::mutex> lock(g_reports_mutex);
  g_report_used[vol->rep_slot] = false;
  vol->rep = vol->rep_dev = nullptr, vol->rep_slot = -1;
}

// Host copy of the counters and both segment tables, which lie one after the
// other at the start of the workspace.
struct Snapshot {
  Counters c;
  Seg vseg[kSegs], cseg[kSegs];
};
static_assert(sizeof(Snapshot) == sizeof(Counters) + 2 * sizeof(Seg) * kSegs, "no gaps");

// The report of a volume without a pinned record (k_report otherwise).
Report host_report(const VolDev& v, const Snapshot& sn) {
  Report r{};
  const Counters& c = sn.c;
  r.error = c.error, r.n_blocks = c.n_blocks;
  for (int k = 0; k < 2; ++k) {
    r.n_frame[k] = c.n_frame[k], r.n_pending[k] = c.n_pending[k];
    r.n_dirty[k] = c.n_dirty[k], r.n_vblocks[k] = c.n_vblocks[k];
  }
  r.base_new = c.base_new, r.base_upd = c.base_upd, r.base_freed = c.base_freed;
  r.base_chg = c.base_chg, r.base_ref = c.base_ref;
  r.dl_nv = c.dl_nv, r.dl_nt = c.dl_nt;
  for (int k = 0; k < VM_TOTAL_COUNT; ++k) r.acc[k] = c.acc[k];
  for (int k = 0; k < kSegs; ++k) {
    Seg g = sn.vseg[k];
    const Seg& q = sn.cseg[k];
    finalise_seg(g, seg_size((uint32_t)k, v.vseg_cap, v.max_vertices));
    r.st_new += g.st_new, r.st_upd += g.st_upd, r.st_mov += g.st_mov, r.st_freed += g.st_freed;
    r.st_chg += q.st_chg, r.st_ref += q.st_ref, r.st_fnew += q.st_fnew, r.st_fold += q.st_fold;
    r.st_cnew += q.st_cnew, r.st_cold += q.st_cold, r.hwm += g.hwm, r.free_slots += g.count;
    const unsigned long long live = g.hwm - (g.hwm < g.count ? g.hwm : g.count);
    r.seg_live = live > r.seg_live ? live : r.seg_live;
  }
  return r;
}

// The counters and segment sums as of everything enqueued on the stream,
// which this waits for.  Nothing of the volume is written: the segments are
// closed in the copy alone.
int read_report(vm_volume* vol, Report* r, hipStream_t stream) {
  if (vol->rep) {
    VM_LAUNCH(vol, VM_K_COUNTERS, k_report, dim3(1), dim3(256), stream, vol->dev, vol->rep_dev);
    int e = launched();
    if (e == VM_OK) e = hip_status(hipStreamSynchronize(stream));
    *r = *vol->rep;
    return e;
  }
  Snapshot sn;
  hipError_t e = hipMemcpyAsync(&sn, vol->dev.cnt, sizeof(sn), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e == hipSuccess) *r = host_report(vol->dev, sn);
  return hip_status(e);
}

int read_counters(vm_volume* vol, Counters* c, hipStream_t stream) {
  hipError_t e = hipMemcpyAsync(c, vol->dev.cnt, sizeof(Counters), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  return hip_status(e);
}

// One phase of vm_extract_batch as plain launches (0 forward, 1 backward).
int batch_enqueue(vm_volume* vol, const vm_batch_io& io, int ph, hipStream_t s) {
  if (ph == 1)
    return vm_extract_backward_slots(vol, io.dL_dpos, io.rows, io.n, io.dL_dtsdf, s);
  int r = vm_reset_volume(vol, s);
  if (r == VM_OK)
    r = vm_import_batch(vol, io.slots, io.coords, io.tsdf, io.weight, io.n, io.rows, s);
  if (r == VM_OK) r = vm_extract_mesh(vol, VM_SCOPE_ALL, s);
  if (r == VM_OK) r = vm_export_positions(vol, io.pos, io.slot_of, io.pos_cap, s);
  return r;
}

// Host-side state of a volume that its calls advance.
void save_host_state(const vm_volume* vol, vm_volume::BatchGraph& g) {
  g.frame = vol->frame, g.epoch = vol->epoch, g.pass = vol->pass;
  g.xcount = vol->xcount, g.vcount = vol->vcount;
  g.xsel = vol->dev.xsel, g.vsel = vol->dev.vsel, g.dev_frame = vol->dev.frame;
}

void load_host_state(vm_volume* vol, const vm_volume::BatchGraph& g) {
  vol->frame = g.frame, vol->epoch = g.epoch, vol->pass = g.pass;
  vol->xcount = g.xcount, vol->vcount = g.vcount;
  vol->dev.xsel = g.xsel, vol->dev.vsel = g.vsel, vol->dev.frame = g.dev_frame;
  vol->have_fp = false;
  mesh_empty(vol);
}

// One phase of vm_extract_batch: replay its graph, capturing it first when
// there is none for these arguments; plain launches where a graph cannot
// be captured (a stream under capture already, the legacy default stream)
// or would hold profiling events.
int batch_phase(vm_volume* vol, const vm_batch_io& io, int ph, hipStream_t s) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (s != nullptr && hipStreamIsCapturing(s, &cs) != hipSuccess) return VM_ERR_HIP;
  if (s == nullptr || cs != hipStreamCaptureStatusNone || vol->prof != 0)
    return batch_enqueue(vol, io, ph, s);
  vm_volume::BatchGraph& g = vol->bgraph[ph];
  const bool same = g.exec && memcmp(&g.io, &io, sizeof(io)) == 0 &&
                    memcmp(&g.launch, &vol->launch, sizeof(vm_launch)) == 0 &&
                    g.d == vol->dev.d && g.w == vol->dev.w;
  if (!same) {
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    g.exec = nullptr;
    hipGraph_t graph = nullptr;
    if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) != hipSuccess) return VM_ERR_HIP;
    const int r = batch_enqueue(vol, io, ph, s);
    const hipError_t e = hipStreamEndCapture(s, &graph);
    if (r != VM_OK || e != hipSuccess) {
      if (graph) (void)hipGraphDestroy(graph);
      return r != VM_OK ? r : VM_ERR_HIP;
    }
    const hipError_t ei = hipGraphInstantiateWithFlags(&g.exec, graph, 0);
    (void)hipGraphDestroy(graph);
    if (ei != hipSuccess) {
      g.exec = nullptr;
      return VM_ERR_HIP;
    }
    g.io = io;
    g.launch = vol->launch;
    g.d = vol->dev.d;
    g.w = vol->dev.w;
    save_host_state(vol, g);
  }
  const hipError_t e = hipGraphLaunch(g.exec, s);
  if (e != hipSuccess) return VM_ERR_HIP;
  if (ph == 0) load_host_state(vol, g);
  return VM_OK;
}

// Set up a volume handle over the workspace mem (bytes long, already
// checked against the configuration) and clear the workspace on `stream`.
int init_volume(vm_volume* vol, const vm_config* cfg, char* mem, size_t bytes,
                hipStream_t stream) {
  std::call_once(g_tables_once, [] {
    build_mc_tables(g_tri, g_uses);
  });
  vol->cfg = *cfg;
  vol->mem = mem;
  vol->bytes = bytes;
  VolDev& v = vol->dev;
  carve(*cfg, vol->mem, &v);
  v.s = cfg->voxel_m;
  v.inv_s = (float)(1.0 / (double)cfg->voxel_m);
  v.inv_block = (float)(1.0 / (8.0 * (double)cfg->voxel_m));
  v.mu_m = (float)((double)cfg->trunc_vox * (double)cfg->voxel_m);
  v.mu_v = cfg->trunc_vox;
  v.eps = cfg->refine_eps_vox;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    return VM_ERR_HIP;
  v.batch = (uint32_t)cfg->batch_volumes;
  v.bound = 0;
  vol->own_d = v.d;
  vol->own_w = v.w;
  vol->cus = cus;
  apply_launch(vol, vm_launch{4, 16, 8, 8, 0});
  vol->prof = 0;
  return clear_state(vol, stream, true);
}

// Workspace of vm_create_volume_noalloc: one per device, held until the
// process ends.  Host code never passes the array's name to a kernel or a
// copy: it takes the device address from hipGetSymbolAddress, once per
// device, and uses that.
constexpr size_t kScratchBytes = (size_t)VM_NOALLOC_MAX_BYTES;
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kScratchDevices];
bool g_scratch_used[kScratchDevices];
alignas(vm_volume) unsigned char g_scratch_vol_mem[kScratchDevices][sizeof(vm_volume)];
vm_volume* const g_scratch_vol = reinterpret_cast<vm_volume*>(g_scratch_vol_mem);

}  // namespace

static __device__ __align__(256) unsigned char scratch[VM_NOALLOC_MAX_BYTES];

extern "C" {

int vm_volume_bytes(const vm_config* cfg, size_t* bytes) {
  if (!config_ok(cfg) || !bytes) return VM_ERR_ARG;
  VolDev v;
  *bytes = carve(*cfg, nullptr, &v);
  return VM_OK;
}

int vm_create_volume(const vm_config* cfg, void* dev_mem, size_t bytes, hipStream_t stream,
                     vm_volume** out) {
  if (!config_ok(cfg) || !dev_mem || !out || ((uintptr_t)dev_mem & 255)) return VM_ERR_ARG;
  VolDev probe;
  if (bytes < carve(*cfg, nullptr, &probe)) return VM_ERR_ARG;
  vm_volume* vol = new (std::nothrow) vm_volume();
  if (!vol) return VM_ERR_ARG;
  const int r = init_volume(vol, cfg, (char*)dev_mem, bytes, stream);
  if (r != VM_OK) {
    delete vol;
    return r;
  }
  take_report(vol);
  *out = vol;
  return VM_OK;
}

int vm_create_volume_noalloc(const vm_config* cfg, hipStream_t stream, vm_volume** out) {
  if (!config_ok(cfg) || !out) return VM_ERR_ARG;
  VolDev probe;
  const size_t need = carve(*cfg, nullptr, &probe);
  if (need > kScratchBytes) return VM_ERR_CAPACITY;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return VM_ERR_HIP;
  if (dev < 0 || dev >= kScratchDevices) return VM_ERR_ARG;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    // the array's device address on this device (the name itself is only
    // a host-side stand-in)
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return VM_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  if (g_scratch_used[dev]) return VM_ERR_ARG;  // one volume per device at a time
  vm_volume* vol = new (&g_scratch_vol[dev]) vm_volume();
  const int r = init_volume(vol, cfg, (char*)g_scratch_ptr[dev], kScratchBytes, stream);
  if (r != VM_OK) {
    vol->~vm_volume();
    return r;
  }
  vol->scratch_dev = dev;
  g_scratch_used[dev] = true;
  *out = vol;
  return VM_OK;
}

int vm_destroy_volume(vm_volume* vol) {
  if (!vol) return VM_ERR_ARG;
  for (auto& g : vol->bgraph)
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
  for (auto& r : vol->recs) vol->ev_free.push_back(r.a), vol->ev_free.push_back(r.b);
  for (hipEvent_t e : vol->ev_free) (void)hipEventDestroy(e);
  give_report(vol);
  const int sdev = vol->scratch_dev;
  if (sdev < 0) {
    delete vol;
    return VM_OK;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  vol->~vm_volume();
  g_scratch_used[sdev] = false;
  return VM_OK;
}

int vm_reset_volume(vm_volume* vol, hipStream_t stream) {
  if (!vol) return VM_ERR_ARG;
  return clear_state(vol, stream, false);
}

int vm_integrate_depth(vm_volume* vol, const float* depth, const vm_intrinsics* K,
                       const float cam_to_world[16], hipStream_t stream) {
  if (!vol || !depth || !K || !cam_to_world || K->width <= 0 || K->height <= 0 ||
      (int64_t)K->width * K->height > (1 << 28) || !(K->fx != 0.f) || !(K->fy != 0.f) ||
      vol->dev.batch)
    return VM_ERR_ARG;
  FrameParams fp;
  const float* T = cam_to_world;
  for (int i = 0; i < 3; ++i) {
    for (int j = 0; j < 3; ++j) {
      fp.Rcw[3 * i + j] = T[4 * i + j];
      fp.Rwc[3 * j + i] = T[4 * i + j];
    }
    fp.tcw[i] = T[4 * i + 3];
  }
  // world -> sensor translation: -R^T t in FP64, rounded once
  for (int i = 0; i < 3; ++i) {
    double acc = (double)fp.Rcw[0 * 3 + i] * (double)fp.tcw[0];
    acc = acc + (double)fp.Rcw[1 * 3 + i] * (double)fp.tcw[1];
    acc = acc + (double)fp.Rcw[2 * 3 + i] * (double)fp.tcw[2];
    fp.twc[i] = (float)(-acc);
  }
  fp.fx = K->fx, fp.fy = K->fy, fp.cx = K->cx, fp.cy = K->cy;
  fp.dmin = K->min_depth_m, fp.dmax = K->max_depth_m;
  fp.W = K->width, fp.H = K->height;
  fp.frame = ++vol->frame;
  mesh_changes(vol);
  const VolDev& v = vol->dev;
  // one workgroup per tile of pixels, and two pixels per lane where one would
  // make more workgroups than there are compute units (k_collect has both
  // sides' times)
  auto tiles = [&](int px) {
    return (unsigned)((K->width + kTileW - 1) / kTileW) *
           (unsigned)((K->height + kTileH * px - 1) / (kTileH * px));
  };
  if (tiles(1) > (unsigned)vol->cus)
    VM_LAUNCH(vol, VM_K_COLLECT, k_collect<2>, dim3(tiles(2)), dim3(512), stream, v, fp, depth,
              vol->epoch);
  else
    VM_LAUNCH(vol, VM_K_COLLECT, k_collect<1>, dim3(tiles(1)), dim3(512), stream, v, fp, depth,
              vol->epoch);
  VM_LAUNCH_W(vol, VM_K_FUSE, k_fuse, stream, v, fp, depth, vol->epoch);
  vol->last_fp = fp;
  vol->have_fp = true;
  return launched();
}

int vm_import_blocks(vm_volume* vol, const int32_t* coords, const float* tsdf,
                     const float* weight, int64_t n, hipStream_t stream) {
  if (!vol || vol->dev.batch) return VM_ERR_ARG;
  return vm_import_batch(vol, nullptr, coords, tsdf, weight, n, nullptr, stream);
}

int vm_import_batch(vm_volume* vol, const int32_t* slots, const int32_t* coords,
                    const float* tsdf, const float* weight, int64_t n, int32_t* rows,
                    hipStream_t stream) {
  if (!vol || n < 0 || n > (int64_t)vol->dev.max_blocks ||
      (n > 0 && (!coords || !tsdf || !weight)) || (vol->dev.batch != 0) != (slots != nullptr) ||
      (vol->dev.bound && n > 0 && (tsdf != vol->dev.d || weight != vol->dev.w)))
    return VM_ERR_ARG;
  if (n == 0) return VM_OK;
  const VolDev& v = vol->dev;
  const uint32_t frame = ++vol->frame;
  mesh_changes(vol);
  // blocks are listed, and new ones numbered, in row order: a caller's
  // spatially ordered rows give a spatially ordered pool
  const uint32_t nparts = (uint32_t)((n + kImportRows - 1) / kImportRows);
  VM_LAUNCH(vol, VM_K_IMPORT, k_import_insert, dim3(nparts), dim3(kImportRows), stream, v, slots,
            coords, (uint32_t)n, frame, vol->epoch);
  VM_LAUNCH(vol, VM_K_ASSIGN, k_import_assign, dim3(nparts), dim3(kImportRows), stream, v,
            (uint32_t)n, frame, vol->epoch);
  VM_LAUNCH_W(vol, VM_K_IMPORT, k_import_copy, stream, v, tsdf, weight, frame, rows);
  vol->have_fp = false;
  return launched();
}

int vm_bind_tsdf(vm_volume* vol, float* tsdf, float* weight) {
  if (!vol || (tsdf == nullptr) != (weight == nullptr) || ((uintptr_t)tsdf & 3) ||
      ((uintptr_t)weight & 3))
    return VM_ERR_ARG;
  VolDev& v = vol->dev;
  float* const d = tsdf ? tsdf : vol->own_d;
  float* const w = weight ? weight : vol->own_w;
  if (d != v.d || w != v.w) {
    ++vol->mesh;
    vol->settled = false;
  }
  v.d = d;
  v.w = w;
  v.bound = tsdf ? 1u : 0u;
  return VM_OK;
}

int vm_extract_mesh(vm_volume* vol, int scope, hipStream_t stream) {
  const bool refine = (scope & VM_EXTRACT_REFINE) != 0;
  scope &= ~VM_EXTRACT_REFINE;
  if (!vol || (scope != VM_SCOPE_DIRTY && scope != VM_SCOPE_ALL)) return VM_ERR_ARG;
  const uint32_t pass = ++vol->pass;
  if (refine || !vol->settled) mesh_changes(vol);
  vol->dl_nv = -1;
  // (the caller may write bound storage between two extractions)
  if (scope == VM_SCOPE_ALL) vol->settled = !refine && !vol->dev.bound;
  // the first kernel starts the call (segments, statistics, list lengths)
  vol->dev.xsel = ++vol->xcount & 1u;
  vol->dev.frame = vol->frame;
  vol->dev.vsel = ++vol->vcount & 1u;
  const VolDev& v = vol->dev;
  // the vertex pass re-places the vertices whose end points' blocks were
  // fused or imported since the last extraction (every block for ALL)
  const uint32_t moved = scope == VM_SCOPE_ALL ? kMovedAll : vol->epoch;
  if (scope == VM_SCOPE_ALL)
    VM_LAUNCH(vol, VM_K_DIRTY, k_dirty_all, dim3(vol->grid_items), dim3(256), stream, v, pass);
  else
    VM_LAUNCH(vol, VM_K_DIRTY, k_dirty, dim3(vol->grid_items), dim3(256), stream, v, pass,
              vol->epoch);
  ++vol->epoch;
  if (refine)
    VM_LAUNCH_WM(vol, VM_K_CLASSIFY, k_classify, kExtractRefined, stream, v, pass);
  else
    VM_LAUNCH_WM(vol, VM_K_CLASSIFY, k_classify, kExtract, stream, v, pass);
  VM_LAUNCH_W(vol, VM_K_VERTICES, k_vertices, stream, v, moved, 1);
  vol->last_refine = false;
  return launched();
}

int vm_refine_mesh(vm_volume* vol, hipStream_t stream) {
  if (!vol) return VM_ERR_ARG;
  const uint32_t pass = ++vol->pass;
  mesh_changes(vol);
  vol->dev.vsel = ++vol->vcount & 1u;
  vol->dev.frame = vol->frame;
  const VolDev& v = vol->dev;
  VM_LAUNCH_WM(vol, VM_K_REFINE, k_classify, kRefine, stream, v, pass);
  VM_LAUNCH(vol, VM_K_DIRTY, k_vblock_compact, dim3(vol->grid_items), dim3(256), stream, v);
  // refinement changes types only: the end points that moved are those in
  // blocks fused or imported since the last extraction (normally none)
  VM_LAUNCH_W(vol, VM_K_VERTICES, k_vertices, stream, v, vol->epoch, 0);
  vol->last_refine = true;
  return launched();
}

int vm_gc(vm_volume* vol, hipStream_t stream) {
  if (!vol) return VM_ERR_ARG;
  // nothing to launch: the vertex pass already freed every vertex whose
  // count dropped to zero (its edge forgot it, its slot went to the
  // segment's recycle ring), and the next extraction or refinement closes
  // the rings before it allocates
  (void)stream;
  return VM_OK;
}

int vm_download_mesh(vm_volume* vol, float* verts, uint64_t* edge_keys, int32_t* tris,
                     int64_t vcap, int64_t tcap, int64_t* nv, int64_t* nt, hipStream_t stream) {
  if (!vol || !nv || !nt || vcap < 0 || tcap < 0 || (vcap > 0 && !verts) || (tcap > 0 && !tris))
    return VM_ERR_ARG;
  const VolDev& v = vol->dev;
  Counters c;
  const uint32_t vc = (uint32_t)(vcap > 0xFFFFFFFFll ? 0xFFFFFFFFll : vcap);
  const uint32_t tc = (uint32_t)(tcap > 0xFFFFFFFFll ? 0xFFFFFFFFll : tcap);
  // grids: what the capacities can need, at most what the device holds
  const unsigned cus = (unsigned)vol->cus, chunks = v.nseg * dl_chunks(v.vseg_cap);
  auto most = [](unsigned n, unsigned m) { return n < m ? n : m; };
  const unsigned tri_chunks = (v.max_blocks + kDlBlocks - 1) / kDlBlocks;
  const unsigned gt = most(tri_chunks, cus), gv = most((chunks + 15) / 16, 2 * cus);
  const unsigned groups = most(chunks, 8 * cus);
  const int counted = dl_counts(v.vseg_cap, v.max_blocks) ? 1 : 0;
  if (counted)
    VM_LAUNCH(vol, VM_K_DOWNLOAD, k_dl_count, dim3(gt + gv), dim3(1024), stream, v, gt);
  VM_LAUNCH(vol, VM_K_DOWNLOAD, k_dl_vertices, dim3(groups + (counted ? 1u : tri_chunks)), dim3(256),
            stream, v, verts, edge_keys, vc, groups, counted);
  VM_LAUNCH(vol, VM_K_DOWNLOAD, k_dl_triangles, dim3(most((v.max_blocks + 3) / 4, 8 * cus)),
            dim3(256), stream, v, tris, tc, counted, vol->rep_dev);
  int r = launched();
  if (r != VM_OK) return r;
  if (vol->rep) {
    r = hip_status(hipStreamSynchronize(stream));
    c.dl_nv = vol->rep->dl_nv, c.dl_nt = vol->rep->dl_nt;
    c.error = vol->rep->error;
  } else {
    r = read_counters(vol, &c, stream);
  }
  if (r != VM_OK) return r;
  *nv = c.dl_nv;
  *nt = c.dl_nt;
  vol->dl_nv = vol->dl_rows = c.dl_nv;
  vol->dl_mesh = vol->mesh;
  if (c.error) return error_code(c.error);
  if ((int64_t)c.dl_nv > vcap || (int64_t)c.dl_nt > tcap) return VM_ERR_CAPACITY;
  return VM_OK;
}

int vm_mesh_state(vm_volume* vol, uint64_t* current, uint64_t* downloaded, int64_t* rows) {
  if (!vol) return VM_ERR_ARG;
  if (current) *current = vol->mesh;
  if (downloaded) *downloaded = vol->dl_mesh;
  if (rows) *rows = vol->dl_rows;
  return VM_OK;
}

int vm_download_normals(vm_volume* vol, float* normals, int64_t cap, hipStream_t stream) {
  if (!vol || (cap > 0 && !normals) || cap < 0) return VM_ERR_ARG;
  if (vol->dl_nv < 0) return VM_ERR_ARG;
  if (cap < vol->dl_nv) return VM_ERR_CAPACITY;
  VM_LAUNCH(vol, VM_K_DOWNLOAD, k_dl_normals, dim3(vol->grid_items), dim3(256), stream, vol->dev,
            normals);
  return launched();
}

int vm_download_births(vm_volume* vol, uint32_t* births, int64_t cap, hipStream_t stream) {
  if (!vol || (cap > 0 && !births) || cap < 0) return VM_ERR_ARG;
  if (vol->dl_nv < 0) return VM_ERR_ARG;
  if (cap < vol->dl_nv) return VM_ERR_CAPACITY;
  VM_LAUNCH(vol, VM_K_DOWNLOAD, k_dl_births, dim3(vol->grid_items), dim3(256), stream, vol->dev,
            births);
  return launched();
}

int vm_sharing_ablation(vm_volume* vol, int scheme, int32_t* edge_slot, float* edge_t,
                        uint32_t* counter, hipStream_t stream) {
  if (!vol || !edge_slot || !edge_t || !counter || (scheme != 0 && scheme != 1))
    return VM_ERR_ARG;
  const dim3 g(vol->grid_items), b(256);
  if (scheme == 0) {
    VM_LAUNCH(vol, VM_K_ABLATION, k_share_lock, g, b, stream, vol->dev, edge_slot, edge_t,
              counter);
  } else {
    for (int group = 0; group < 4; ++group)
      VM_LAUNCH(vol, VM_K_ABLATION, k_share_free, g, b, stream, vol->dev, group, edge_slot,
                edge_t, counter);
  }
  return launched();
}

int vm_extract_backward(vm_volume* vol, const float* dL_dverts, float* dL_dtsdf,
                        hipStream_t stream) {
  if (!vol || !dL_dtsdf || (vol->dl_rows > 0 && !dL_dverts)) return VM_ERR_ARG;
  VM_LAUNCH_W(vol, VM_K_BACKWARD, k_bwd_tsdf, stream, vol->dev, dL_dverts, 0, nullptr, 0u,
              dL_dtsdf);
  return launched();
}

int vm_extract_backward_rows(vm_volume* vol, const float* dL_dverts, const int32_t* rows,
                             int64_t n_rows, float* dL_dtsdf, hipStream_t stream) {
  if (!vol || !rows || n_rows < 0 || n_rows > (int64_t)kMaxBlocks || (n_rows > 0 && !dL_dtsdf) ||
      vol->dl_nv < 0 || (vol->dl_nv > 0 && !dL_dverts))
    return VM_ERR_ARG;
  if (n_rows == 0) return VM_OK;
  VM_LAUNCH_W(vol, VM_K_BACKWARD, k_bwd_tsdf, stream, vol->dev, dL_dverts, 0, rows,
              (uint32_t)n_rows, dL_dtsdf);
  return launched();
}

int vm_extract_backward_slots(vm_volume* vol, const float* dL_dpos, const int32_t* rows,
                              int64_t n_rows, float* dL_dtsdf, hipStream_t stream) {
  if (!vol || !dL_dpos || !dL_dtsdf || (rows && (n_rows < 0 || n_rows > (int64_t)kMaxBlocks)))
    return VM_ERR_ARG;
  VM_LAUNCH_W(vol, VM_K_BACKWARD, k_bwd_tsdf, stream, vol->dev, dL_dpos, 1, rows,
              (uint32_t)(rows ? n_rows : 0), dL_dtsdf);
  return launched();
}

int vm_export_positions(vm_volume* vol, float* pos, int32_t* slot_of, int64_t cap,
                        hipStream_t stream) {
  if (!vol || !pos) return VM_ERR_ARG;
  if (cap < (int64_t)vol->dev.max_vertices) return VM_ERR_CAPACITY;
  close_pool(vol, stream);
  VM_LAUNCH(vol, VM_K_POSITIONS, k_positions, dim3(vol->grid_items), dim3(256), stream, vol->dev,
            pos, slot_of);
  return launched();
}

int vm_sphere_loss_grad(const float* pos, const int32_t* slot, const float* centers,
                        const float* radii, int32_t rows, int64_t n, float* out,
                        hipStream_t stream) {
  if (rows < 1 || n < 0 || !centers || !radii || (n > 0 && (!pos || !slot || !out)))
    return VM_ERR_ARG;
  if (n == 0) return VM_OK;
  const int64_t g = (n + 255) / 256;
  hipLaunchKernelGGL(k_sphere_loss, dim3((unsigned)(g < 16384 ? g : 16384)), dim3(256), 0, stream, pos,
                     slot, centers, radii, rows, (uint64_t)n, out);
  return launched();
}

int vm_set_launch(vm_volume* vol, const vm_launch* launch) {
  if (!vol || !launch_ok(launch)) return VM_ERR_ARG;
  apply_launch(vol, *launch);
  return VM_OK;
}

int vm_get_launch(vm_volume* vol, vm_launch* launch) {
  if (!vol || !launch) return VM_ERR_ARG;
  *launch = vol->launch;
  return VM_OK;
}

int vm_integrate_backward(vm_volume* vol, const float* depth, const float* dL_dtsdf1,
                          float* dL_dtsdf0, float* dL_ddepth, hipStream_t stream) {
  if (!vol || !depth || !dL_dtsdf1 || !dL_dtsdf0 || !dL_ddepth || !vol->have_fp) return VM_ERR_ARG;
  const FrameParams& fp = vol->last_fp;
  VM_LAUNCH(vol, VM_K_BACKWARD, k_zero_f32, dim3(256), dim3(256), stream, dL_ddepth,
            (uint64_t)fp.W * (uint64_t)fp.H);
  VM_LAUNCH(vol, VM_K_BACKWARD, k_bwd_fusion, dim3(vol->grid_blocks), dim3(512), stream, vol->dev,
            fp, depth, dL_dtsdf1, dL_dtsdf0, dL_ddepth);
  return launched();
}

int vm_get_status(vm_volume* vol, vm_status* out, hipStream_t stream) {
  if (!vol || !out) return VM_ERR_ARG;
  Report c;
  const int r = read_report(vol, &c, stream);
  if (r != VM_OK) return r;
  const uint32_t B = vol->dev.max_blocks;
  memset(out, 0, sizeof(*out));
  out->error = error_code(c.error);
  out->error_bits = c.error;
  out->blocks = c.n_blocks < B ? c.n_blocks : B;
  const uint32_t nf = c.n_frame[vol->frame & 1];
  out->frame_blocks = nf < B ? nf : B;
  out->pending_blocks = c.n_pending[vol->epoch & 1];
  out->dirty_blocks = c.n_dirty[vol->dev.xsel];
  out->vertex_blocks = c.n_vblocks[vol->dev.vsel] + (vol->last_refine ? 0u : c.n_dirty[vol->dev.xsel]);
  out->changed_cubes = (uint32_t)c.st_chg - c.base_chg;
  out->vertex_slots = (int64_t)c.hwm;
  out->free_vertex_slots = (int64_t)c.free_slots;
  out->triangles = (int64_t)(c.st_fnew - c.st_fold);
  out->tri_cubes = (int64_t)(c.st_cnew - c.st_cold);
  out->new_vertices = (uint32_t)c.st_new - c.base_new;
  out->updated_vertices = (uint32_t)c.st_upd - c.base_upd;
  out->freed_vertices = (uint32_t)c.st_freed - c.base_freed;
  out->refined_cubes = (uint32_t)c.st_ref - c.base_ref;
  out->vertex_segments = vol->dev.nseg;
  out->segment_capacity = vol->dev.vseg_cap;
  out->max_segment_live = (int64_t)c.seg_live;
  return out->error;
}

int vm_export_blocks(vm_volume* vol, int32_t* coords, float* tsdf, float* weight,
                     uint8_t* type_prev, uint8_t* type_cur, int64_t cap, int64_t* n,
                     hipStream_t stream) {
  if (!vol || !n || cap < 0 || (cap > 0 && !coords)) return VM_ERR_ARG;
  Counters c;
  int r = read_counters(vol, &c, stream);
  if (r != VM_OK) return r;
  const VolDev& v = vol->dev;
  const size_t nb = c.n_blocks < v.max_blocks ? c.n_blocks : v.max_blocks;
  *n = (int64_t)nb;
  const size_t m = (size_t)cap < nb ? (size_t)cap : nb;
  if (m == 0) return VM_OK;
  std::vector<uint64_t> keys(m);
  hipError_t e = hipMemcpyAsync(keys.data(), v.block_key, 8 * m, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess && tsdf)
    e = hipMemcpyAsync(tsdf, v.d, 4 * kVox * m, hipMemcpyDeviceToDevice, stream);
  if (e == hipSuccess && weight)
    e = hipMemcpyAsync(weight, v.w, 4 * kVox * m, hipMemcpyDeviceToDevice, stream);
  if (type_prev)
    hipLaunchKernelGGL(k_export_types, dim3(vol->grid_items), dim3(256), 0, stream, v.tprev,
                       v.blank, type_prev, (uint64_t)kVox * m);
  if (type_cur)
    hipLaunchKernelGGL(k_export_types, dim3(vol->grid_items), dim3(256), 0, stream, v.tcur,
                       nullptr, type_cur, (uint64_t)kVox * m);
  if (e == hipSuccess) e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return VM_ERR_HIP;
  for (size_t i = 0; i < m; ++i) unpack_key(keys[i], coords[3 * i], coords[3 * i + 1], coords[3 * i + 2]);
  return VM_OK;
}

int vm_export_vertices(vm_volume* vol, uint64_t* edge_keys, float* t, int32_t* refcount,
                       int64_t cap, int64_t* n, hipStream_t stream) {
  if (!vol || !n || cap < 0 || (cap > 0 && (!edge_keys || !t || !refcount))) return VM_ERR_ARG;
  close_pool(vol, stream);
  int r = launched();
  if (r != VM_OK) return r;
  *n = vol->dev.max_vertices;
  const uint32_t m = (uint32_t)((int64_t)vol->dev.max_vertices < cap ? vol->dev.max_vertices : cap);
  if (m == 0) return hip_status(hipStreamSynchronize(stream));
  hipLaunchKernelGGL(k_export_vertices, dim3((m + 255) / 256), dim3(256), 0, stream, vol->dev,
                     edge_keys, t, refcount, m);
  r = launched();
  if (r != VM_OK) return r;
  return hip_status(hipStreamSynchronize(stream));
}

int vm_export_block_list(vm_volume* vol, int which, int32_t* coords, int64_t cap, int64_t* n,
                         hipStream_t stream) {
  if (!vol || !n || which < 0 || which > 2 || cap < 0 || (cap > 0 && !coords)) return VM_ERR_ARG;
  Counters c;
  int r = read_counters(vol, &c, stream);
  if (r != VM_OK) return r;
  const VolDev& v = vol->dev;
  const uint32_t len = which == 0 ? c.n_frame[vol->frame & 1] : which == 1 ? c.n_dirty[vol->dev.xsel] : c.n_pending[vol->epoch & 1];
  const size_t cnt = len < v.max_blocks ? len : v.max_blocks;
  *n = (int64_t)cnt;
  const size_t m = (size_t)cap < cnt ? (size_t)cap : cnt;
  if (m == 0) return VM_OK;
  const uint32_t* list = which == 0 ? v.frame_list : which == 1 ? v.dirty : v.pending;
  const size_t nb = c.n_blocks < v.max_blocks ? c.n_blocks : v.max_blocks;
  std::vector<uint32_t> idx(m);
  std::vector<uint64_t> keys(nb);
  hipError_t e = hipMemcpyAsync(idx.data(), list, 4 * m, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess && nb)
    e = hipMemcpyAsync(keys.data(), v.block_key, 8 * nb, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return VM_ERR_HIP;
  size_t k = 0;
  for (size_t i = 0; i < m; ++i) {
    if (idx[i] == kNone) continue;
    const uint32_t b = idx[i] & ~kNewFlag;
    if (b >= nb) continue;
    unpack_key(keys[b], coords[3 * k], coords[3 * k + 1], coords[3 * k + 2]);
    ++k;
  }
  *n = (int64_t)k;
  return VM_OK;
}

int vm_lookup_blocks(vm_volume* vol, const int32_t* coords, int32_t* idx, int64_t n,
                     hipStream_t stream) {
  if (!vol || n < 0 || n > 0x7FFFFFFF || (n > 0 && (!coords || !idx))) return VM_ERR_ARG;
  if (n == 0) return VM_OK;
  const uint32_t m = (uint32_t)n;
  hipLaunchKernelGGL(k_lookup, dim3((m + 255) / 256 < 65535 ? (m + 255) / 256 : 65535), dim3(256), 0,
                     stream, vol->dev, coords, idx, m);
  return launched();
}

int vm_get_totals(vm_volume* vol, int64_t* out, int n, hipStream_t stream) {
  if (!vol || !out || n < 0 || n > VM_TOTAL_COUNT) return VM_ERR_ARG;
  Report c;
  const int r = read_report(vol, &c, stream);
  if (r != VM_OK) return r;
  unsigned long long t[VM_TOTAL_COUNT];
  for (int i = 0; i < VM_TOTAL_COUNT; ++i) t[i] = c.acc[i];
  t[VM_TOTAL_NEW_VERTICES] += c.st_new;
  t[VM_TOTAL_UPDATED_VERTICES] += c.st_upd;
  t[VM_TOTAL_MOVED_VERTICES] += c.st_mov;
  t[VM_TOTAL_FREED_VERTICES] += c.st_freed;
  t[VM_TOTAL_CHANGED_CUBES] += c.st_chg;
  t[VM_TOTAL_REFINED_CUBES] += c.st_ref;
  t[VM_TOTAL_NEW_TRIANGLES] += c.st_fnew;
  t[VM_TOTAL_DROPPED_TRIANGLES] += c.st_fold;
  for (int i = 0; i < n; ++i) out[i] = (int64_t)t[i];
  return VM_OK;
}

int vm_extract_batch(vm_volume* vol, const vm_batch_io* io, int phase, hipStream_t stream) {
  if (!vol || !io || (phase != VM_BATCH_FORWARD && phase != VM_BATCH_BACKWARD) || io->n < 1 ||
      io->n > (int64_t)vol->dev.max_blocks || !io->coords || !io->tsdf || !io->weight ||
      !io->rows || (vol->dev.batch != 0) != (io->slots != nullptr))
    return VM_ERR_ARG;
  if (phase == VM_BATCH_FORWARD && !io->pos) return VM_ERR_ARG;
  if (phase == VM_BATCH_BACKWARD && (!io->dL_dpos || !io->dL_dtsdf)) return VM_ERR_ARG;
  if (io->pos_cap < (int64_t)vol->dev.max_vertices) return VM_ERR_CAPACITY;
  return batch_phase(vol, *io, phase == VM_BATCH_FORWARD ? 0 : 1, stream);
}

int vm_profile_mask(vm_volume* vol, uint32_t mask) {
  if (!vol || (mask >> VM_K_COUNT)) return VM_ERR_ARG;
  if (mask) {
    for (auto& r : vol->recs) vol->ev_free.push_back(r.a), vol->ev_free.push_back(r.b);
    vol->recs.clear();
  }
  vol->prof = mask;
  return VM_OK;
}

int vm_profile(vm_volume* vol, int enable) {
  return vm_profile_mask(vol, enable ? (1u << VM_K_COUNT) - 1u : 0u);
}

int vm_profile_read(vm_volume* vol, int64_t* launches, double* ms) {
  if (!vol || !launches || !ms) return VM_ERR_ARG;
  for (int k = 0; k < VM_K_COUNT; ++k) launches[k] = 0, ms[k] = 0.0;
  if (!vol->recs.empty() && hipEventSynchronize(vol->recs.back().b) != hipSuccess) return VM_ERR_HIP;
  for (auto& r : vol->recs) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) return VM_ERR_HIP;
    launches[r.kid] += 1;
    ms[r.kid] += (double)t;
  }
  return VM_OK;
}

}  // extern "C"
