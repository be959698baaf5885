// Host side of the C ABI declared in include/lbm.h: workspace layout, validation, state transfer,
// launch sequencing (eager or hipGraph replay), observables and the stage-export test hook.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "../../include/lbm.h"
#include "lbm_adjoint.h"
#include "lbm_internal.h"

using namespace lbm;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

// A named host range on profiler timelines (rocprofv3 --marker-trace); a plain call when no tool is attached.
struct Range {
  explicit Range(const char* name) { roctxRangePushA(name); }
  ~Range() { roctxRangePop(); }
  Range(const Range&) = delete;
  Range& operator=(const Range&) = delete;
};

#define HIPCHK(call)                                                                          \
  do {                                                                                        \
    hipError_t e_ = (call);                                                                   \
    if (e_ != hipSuccess) return fail(LBM_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

constexpr size_t ALIGN = 256;
// lbm_debug_stage exports planes only for instances up to this many nodes (its scratch is sized by it).
constexpr int64_t DEBUG_MAX_NODES = 512 * 512;
size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// D2Q9 directions in the public order rest, E, N, W, S, NE, NW, SW, SE.
constexpr int EX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int EY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
constexpr int OPP[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};  // e_OPP[k] = -e_k
constexpr double WGT[9] = {4.0 / 9.0,  1.0 / 9.0,  1.0 / 9.0,  1.0 / 9.0, 1.0 / 9.0,
                           1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};

// Workspace layout of a batch: one typed pool for all fields, then bookkeeping arrays.
struct Layout {
  int prec = 0;
  size_t elem = 8;
  std::vector<InstDev> inst;
  std::vector<TileDev> tiles;  // split-kernel tiles in launch order (XCD-aware), padded with inst = -1
  std::vector<TileDev> segs;   // fused-kernel strips in launch order
  std::vector<TileDev> ttiles;  // tiles of the tiled fused step in launch order (none if it does not apply)
  int tshape = -1, nttiles = 0;  // shape of the tiles (TILE_SHAPES)
  int64_t tpart_elems = 0;  // one of its two buffers of sums
  int ntiles = 0, nsegs = 0, ndrop_total = 0, max_nd = 0, obs_stride = 0;
  int max_segs = 0, max_seg_launch = 0, seg_rows = 0, strip_w = FUSED_TX;
  int64_t max_nodes = 0;
  size_t off_pool = 0, off_inst = 0, off_tiles = 0, off_segs = 0, off_drops = 0, off_part = 0, off_mask = 0,
         off_step = 0, off_obs = 0, off_dbg = 0, off_ttiles = 0, off_tcen = 0, off_tpart = 0, off_tmask = 0, total = 0;
};

int validate(int32_t ninst, const lbm_config* cfgs, const int32_t* ndrop) {
  if (ninst <= 0 || !cfgs || !ndrop) return fail(LBM_E_INVAL, "ninst must be > 0 with configs and droplet counts");
  for (int i = 0; i < ninst; ++i) {
    const lbm_config& c = cfgs[i];
    char where[64];
    snprintf(where, sizeof where, "instance %d: ", i);
    if (c.nx < 3 || c.ny < 3) return fail(LBM_E_INVAL, std::string(where) + "nx and ny must be >= 3");
    if ((int64_t)c.nx * c.ny > (int64_t)1 << 30) return fail(LBM_E_INVAL, std::string(where) + "lattice too large");
    if (c.precision != LBM_FP64 && c.precision != LBM_FP32 && c.precision != LBM_FP16)
      return fail(LBM_E_INVAL, std::string(where) + "precision must be LBM_FP64, LBM_FP32 or LBM_FP16");
    if (c.precision != cfgs[0].precision) return fail(LBM_E_INVAL, "all instances of a batch need the same precision");
    if (c.advection != LBM_ADV_PAPER && c.advection != LBM_ADV_FLUX)
      return fail(LBM_E_INVAL, std::string(where) + "unknown advection scheme");
    if (c.walls != LBM_WALLS_NONE && c.walls != LBM_WALLS_Y)
      return fail(LBM_E_INVAL, std::string(where) + "walls must be LBM_WALLS_NONE or LBM_WALLS_Y");
    if (!(c.tau > 0.5)) return fail(LBM_E_INVAL, std::string(where) + "tau must exceed 1/2");
    if (!(c.b > 0.0)) return fail(LBM_E_INVAL, std::string(where) + "b must be positive");
    if (!(c.n0 > 0.0)) return fail(LBM_E_INVAL, std::string(where) + "n0 must be positive");
    const double vals[] = {c.a, c.B0, c.B1, c.D, c.Gamma, c.gamma, c.A0, c.t_star, c.c0};
    for (double v : vals)
      if (!std::isfinite(v)) return fail(LBM_E_INVAL, std::string(where) + "parameters must be finite");
    if (ndrop[i] < 0 || ndrop[i] > LBM_MAXDROP)
      return fail(LBM_E_INVAL, std::string(where) + "droplet count out of range [0, LBM_MAXDROP]");
  }
  return LBM_OK;
}

// Model parameters of an instance, derived in double precision (advection form, walls, Eqs. 1-19).
void set_model(const lbm_config& c, InstDev& d) {
  d.advection = c.advection;
  d.walls = c.walls;
  d.yper = c.walls ? std::numeric_limits<double>::infinity() : (double)c.ny;
  d.a = c.a;
  d.b = c.b;
  d.B0 = c.B0;
  d.B1 = c.B1;
  d.halfB1 = 0.5 * c.B1;
  d.D = c.D;
  d.Gamma = c.Gamma;
  d.gamma = c.gamma;
  d.c0 = c.c0;
  d.omega = 1.0 / c.tau;
  d.coef = 1.0 - 1.0 / (2.0 * c.tau);
  d.A0 = c.A0;
  d.t_star = c.t_star;
  d.wn[0] = WGT[0] * c.n0;
  d.wn[1] = WGT[1] * c.n0;
  d.wn[2] = WGT[5] * c.n0;
  d.n0 = c.n0;
}

// The tile shape of the tiled fused step for these lattices (see TILE_SHAPES), -1 where it does not apply.
int tile_shape(const std::vector<InstDev>& inst) {
  for (int k = 0; k < TILE_NSHAPES; ++k) {
    const TileShape& s = TILE_SHAPES[k];
    int64_t tiles = 0;
    for (const InstDev& d : inst) {
      if (d.ndrop > TILE_DROPS || d.nx < s.ox + TILE_RINGS || d.ny < s.oy + TILE_RINGS) return -1;
      tiles += (int64_t)((d.nx + s.ox - 1) / s.ox) * ((d.ny + s.oy - 1) / s.oy);
    }
    if (tiles <= s.most) return k;
  }
  return -1;
}

int strip_count(int nx, int ny, int w, int rows) { return ((nx + w - 1) / w) * ((ny + rows - 1) / rows); }
int strip_bound(int nx, int ny) {
  return std::max(strip_count(nx, ny, STRIP_W_MIN, SEG_ROWS_MIN), strip_count(nx, ny, FUSED_TX, SHORT_ROWS[0]));
}

void make_layout(int32_t ninst, const lbm_config* cfgs, const int32_t* ndrop, Layout& L) {
  L.prec = cfgs[0].precision;
  L.elem = L.prec == LBM_FP64 ? 8 : 4;
  const size_t row_align = ALIGN / L.elem;
  int64_t pool_elems = 0;
  int tile_base = 0, seg_base = 0, drop_base = 0;
  int64_t part_elems = 0, part_elems1 = 0;
  L.inst.resize(ninst);
  for (int i = 0; i < ninst; ++i) {
    const lbm_config& c = cfgs[i];
    InstDev& d = L.inst[i];
    memset(&d, 0, sizeof d);
    d.nx = c.nx;
    d.ny = c.ny;
    d.pitch = (int32_t)align_up((size_t)c.nx, row_align);
    d.ndrop = ndrop[i];
    d.tiles_x[TILING_SPLIT] = (c.nx + TILE_X - 1) / TILE_X;
    d.tiles_y[TILING_SPLIT] = (c.ny + TILE_Y - 1) / TILE_Y;
    d.tile_base[TILING_SPLIT] = tile_base;
    // an upper bound of the strips (the narrowest and shortest that a caller may set, or the widest of SHORT_ROWS); see
    // set_segments
    d.tiles_x[TILING_FUSED] = strip_bound(c.nx, c.ny);
    d.tiles_y[TILING_FUSED] = 1;
    d.tile_base[TILING_FUSED] = seg_base;
    d.drop_base = drop_base;
    const int64_t plane = (int64_t)c.ny * d.pitch;
    d.pstride = plane;
    // a population buffer holds 9 planes of the storage type (FP16 deviations take half a field plane)
    const int64_t fbuf = L.prec == LBM_FP16 ? (int64_t)align_up((size_t)(9 * plane / 2), row_align) : 9 * plane;
    int64_t o = pool_elems;
    d.off_f[0] = o;  o += fbuf;
    d.off_f[1] = o;  o += fbuf;
    d.off_phi[0] = o; o += plane;
    d.off_phi[1] = o; o += plane;
    d.off_c[0] = o;  o += plane;
    d.off_c[1] = o;  o += plane;
    d.off_ux = o;    o += plane;
    d.off_uy = o;    o += plane;
    d.off_n = o;     o += plane;
    pool_elems = o;
    d.part_base[TILING_SPLIT] = part_elems;
    part_elems += (int64_t)d.tiles_x[TILING_SPLIT] * d.tiles_y[TILING_SPLIT] * d.ndrop * 3;
    d.part_base[TILING_FUSED] = part_elems1;
    part_elems1 += (int64_t)d.tiles_x[TILING_FUSED] * d.tiles_y[TILING_FUSED] * d.ndrop * 3;
    set_model(c, d);
    tile_base += d.tiles_x[TILING_SPLIT] * d.tiles_y[TILING_SPLIT];
    seg_base += d.tiles_x[TILING_FUSED] * d.tiles_y[TILING_FUSED];
    drop_base += d.ndrop;
    L.max_nd = std::max(L.max_nd, (int)d.ndrop);
    L.max_nodes = std::max(L.max_nodes, (int64_t)c.nx * c.ny);
  }
  L.tshape = tile_shape(L.inst);
  if (L.tshape >= 0)
    for (InstDev& d : L.inst) {
      const TileShape& t = TILE_SHAPES[L.tshape];
      d.tiles_x[TILING_TILE] = (d.nx + t.ox - 1) / t.ox;
      d.tiles_y[TILING_TILE] = (d.ny + t.oy - 1) / t.oy;
      d.tile_base[TILING_TILE] = L.nttiles;
      d.part_base[TILING_TILE] = L.tpart_elems;
      L.nttiles += d.tiles_x[TILING_TILE] * d.tiles_y[TILING_TILE];
      L.tpart_elems += (int64_t)d.tiles_x[TILING_TILE] * d.tiles_y[TILING_TILE] * d.ndrop * 6;
    }
  L.ntiles = tile_base;
  L.nsegs = seg_base;
  L.ndrop_total = drop_base;
  L.obs_stride = OBS_STRIDE(L.max_nd);
  // Work lists in launch order: workgroup b runs on XCD (b mod 8); give each XCD a contiguous run of
  // tiles (raster order within an instance) so that neighbouring tiles share that XCD's L2.
  auto build_list = [&](int tiling, int tw, int th, int count, std::vector<TileDev>& out) {
    std::vector<TileDev> natural;
    natural.reserve(count);
    for (int i = 0; i < ninst; ++i) {
      const InstDev& d = L.inst[i];
      for (int ty = 0; ty < d.tiles_y[tiling]; ++ty)
        for (int tx = 0; tx < d.tiles_x[tiling]; ++tx)
          natural.push_back(TileDev{i, tx * tw, ty * th, (int32_t)natural.size()});
    }
    const int nxcd = 8;
    const int chunk = (count + nxcd - 1) / nxcd;
    out.assign((size_t)chunk * nxcd, TileDev{-1, 0, 0, -1});
    for (int t = 0; t < count; ++t) out[(size_t)(t % chunk) * nxcd + t / chunk] = natural[t];
  };
  build_list(TILING_SPLIT, TILE_X, TILE_Y, L.ntiles, L.tiles);
  if (L.tshape >= 0) build_list(TILING_TILE, TILE_SHAPES[L.tshape].ox, TILE_SHAPES[L.tshape].oy, L.nttiles, L.ttiles);
  L.max_segs = L.nsegs;  // strips of the narrowest width and smallest height: sizes the strip list and partials
  L.max_seg_launch = ((L.nsegs + 7) / 8) * 8;
  size_t off = 0;
  L.off_pool = off;  off = align_up(off + (size_t)pool_elems * L.elem, ALIGN);
  L.off_inst = off;  off = align_up(off + sizeof(InstDev) * ninst, ALIGN);
  L.off_tiles = off; off = align_up(off + sizeof(TileDev) * L.tiles.size(), ALIGN);
  L.off_segs = off;  off = align_up(off + sizeof(TileDev) * (size_t)L.max_seg_launch, ALIGN);
  L.off_drops = off; off = align_up(off + sizeof(DropDev) * std::max(1, L.ndrop_total), ALIGN);
  // the two tilings share the partials and masks (one of them is in use at a time)
  L.off_part = off;
  off = align_up(off + sizeof(double) * std::max<int64_t>(1, std::max(part_elems, part_elems1)), ALIGN);
  L.off_mask = off;
  off = align_up(off + sizeof(uint64_t) * MASK_WORDS * (size_t)std::max(L.ntiles, L.nsegs), ALIGN);
  L.off_step = off;  off = align_up(off + sizeof(int64_t), ALIGN);
  L.off_obs = off;   off = align_up(off + sizeof(double) * (size_t)L.obs_stride * L.ntiles, ALIGN);
  L.off_dbg = off;
  off = align_up(off + sizeof(double) * (size_t)LBM_NSTAGE * std::min(L.max_nodes, DEBUG_MAX_NODES), ALIGN);
  L.off_ttiles = off; off = align_up(off + sizeof(TileDev) * L.ttiles.size(), ALIGN);
  L.off_tcen = off;   off = align_up(off + sizeof(double) * 4 * (size_t)(L.tshape >= 0 ? L.ndrop_total : 0), ALIGN);
  L.off_tpart = off;  off = align_up(off + sizeof(double) * 2 * (size_t)L.tpart_elems, ALIGN);
  L.off_tmask = off;  off = align_up(off + sizeof(uint32_t) * 2 * (size_t)L.nttiles, ALIGN);
  L.total = off;
}

// Whether the owned box [x0, x1] x [y0, y1] of a strip segment of instance d comes within R + 2 (minimum
// image) of a droplet centre, i.e. may hold the droplet's phi >= 0 nodes or its production disk.  Such
// segments take longer (centre-of-mass sums, disk test) and are dispatched first.
bool segment_holds_droplet(const InstDev& d, const std::vector<DropDev>& drops, int inst, int x0, int x1, int y0,
                           int y1) {
  const double xm = 0.5 * (x0 + x1), ym = 0.5 * (y0 + y1), hx = 0.5 * (x1 - x0), hy = 0.5 * (y1 - y0);
  for (const DropDev& q : drops) {
    if (q.inst != inst) continue;
    double dx = std::fabs(xm - q.x), dy = std::fabs(ym - q.y);
    if (dx > 0.5 * d.nx) dx = d.nx - dx;
    if (!d.walls && dy > 0.5 * d.ny) dy = d.ny - dy;
    dx = std::max(0.0, dx - hx);
    dy = std::max(0.0, dy - hy);
    const double r = q.R + 2.0;
    if (dx * dx + dy * dy <= r * r) return true;
  }
  return false;
}

// Sweeping-kernel strips for a strip width and segment height: per-instance counts, natural indices,
// partial offsets and the launch list.  The list is XCD-aware: workgroup b runs on XCD (b mod 8), and each
// XCD gets a contiguous run of strips in natural order (neighbouring strips share that XCD's L2); within
// its run, the strips that hold droplets (as of `drops`) are dispatched first, so that the longer-running
// ones do not end the launch.  The launch order does not change any result (partials are stored by natural
// index).  The caller sees to it that the strips of every instance are at most strip_bound(), which the regions are
// sized for.
void set_segments(Layout& L, int seg_rows, int strip_w, const std::vector<DropDev>& drops) {
  int base = 0;
  int64_t part = 0;
  for (auto& d : L.inst) {
    d.seg_rows = seg_rows;
    d.strip_w = strip_w;
    d.tiles_x[TILING_FUSED] = (d.nx + strip_w - 1) / strip_w;
    d.tiles_y[TILING_FUSED] = (d.ny + seg_rows - 1) / seg_rows;
    d.tile_base[TILING_FUSED] = base;
    d.part_base[TILING_FUSED] = part;
    base += d.tiles_x[TILING_FUSED] * d.tiles_y[TILING_FUSED];
    part += (int64_t)d.tiles_x[TILING_FUSED] * d.tiles_y[TILING_FUSED] * d.ndrop * 3;
  }
  L.nsegs = base;
  L.seg_rows = seg_rows;
  L.strip_w = strip_w;
  std::vector<TileDev> natural;
  natural.reserve(base);
  for (size_t i = 0; i < L.inst.size(); ++i) {
    const InstDev& d = L.inst[i];
    for (int ty = 0; ty < d.tiles_y[TILING_FUSED]; ++ty)
      for (int tx = 0; tx < d.tiles_x[TILING_FUSED]; ++tx)
        natural.push_back(TileDev{(int32_t)i, tx * strip_w, ty * seg_rows, (int32_t)natural.size()});
  }
  const int nxcd = 8;
  const int chunk = (base + nxcd - 1) / nxcd;
  L.segs.assign((size_t)chunk * nxcd, TileDev{-1, 0, 0, -1});
  std::vector<TileDev> run;
  for (int j = 0; j < nxcd; ++j) {
    run.clear();
    const int t0 = j * chunk, t1 = std::min(base, (j + 1) * chunk);
    for (int pass = 0; pass < 2; ++pass)
      for (int t = t0; t < t1; ++t) {
        const TileDev& s = natural[t];
        const InstDev& d = L.inst[s.inst];
        const bool heavy = segment_holds_droplet(d, drops, s.inst, s.x0, std::min(s.x0 + strip_w, d.nx) - 1, s.y0,
                                                 std::min(s.y0 + seg_rows, d.ny) - 1);
        if (heavy == (pass == 0)) run.push_back(s);
      }
    for (size_t k = 0; k < run.size(); ++k) L.segs[k * nxcd + j] = run[k];
  }
}


// Page-locked host memory for read-backs, in blocks of two sizes: a droplet table or observables, and two chunks of
// fields.  A call takes a block of its own and gives it back, so that calls from several threads do not meet in it.
// The blocks are the process's: a context's own would be locked by its first read-back and freed with it, which a
// program that reads each context once never earns back (64 x 64, first lbm_droplets, lbm_fields and lbm_destroy of a
// new context, us: 16, 62 and 1 with the process's blocks, 44, 350 and 260 with the context's).  Up to READ_KEPT blocks
// of a size wait for the next calls, and one of each once no context is left.
// Read-backs of more than READ_CHUNK bytes go in chunks, through the two halves of a block: the host copies one chunk
// out while the kernel fills the other half.
constexpr size_t READ_CHUNK = 512u << 10;
constexpr size_t READ_HEAD = 64;  // bytes before a chunk's values: its flag of non-finite ones
constexpr int READ_SIZES = 2, READ_KEPT = 4;
constexpr size_t READ_BLOCK[READ_SIZES] = {16u << 10, 2 * (READ_CHUNK + ALIGN)};
static_assert(sizeof(DropDev) * MAXDROP <= READ_BLOCK[0] && sizeof(double) * (6 + 5 * MAXDROP) <= READ_BLOCK[0] &&
              READ_HEAD <= ALIGN, "what the blocks hold");

class ReadBlocks {
 public:
  static ReadBlocks& get() {
    static ReadBlocks* const all = new ReadBlocks;  // never destroyed: the runtime may be gone by then
    return *all;
  }
  void add_context() {
    std::lock_guard<std::mutex> lock(mu_);
    ++contexts_;
  }
  void drop_context() {
    char* spare[READ_SIZES * READ_KEPT];
    int n = 0;
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (--contexts_ > 0) return;
      for (int s = 0; s < READ_SIZES; ++s)
        while (n_[s] > 1) spare[n++] = kept_[s][--n_[s]];
    }
    while (n > 0) (void)hipHostFree(spare[--n]);
  }
  hipError_t take(int size, char** out) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (n_[size] > 0) {
        *out = kept_[size][--n_[size]];
        return hipSuccess;
      }
    }
    void* p = nullptr;
    const hipError_t e = hipHostMalloc(&p, READ_BLOCK[size], hipHostMallocCoherent | hipHostMallocPortable);
    *out = static_cast<char*>(p);
    return e;
  }
  void give(int size, char* p) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (n_[size] < (contexts_ > 0 ? READ_KEPT : 1)) {
        kept_[size][n_[size]++] = p;
        return;
      }
    }
    (void)hipHostFree(p);
  }

 private:
  std::mutex mu_;
  char* kept_[READ_SIZES][READ_KEPT] = {};
  int n_[READ_SIZES] = {};
  int64_t contexts_ = 0;
};

}  // namespace

struct lbm_ctx {
  Layout L;
  std::vector<lbm_config> cfg;
  char* ws = nullptr;
  hipStream_t stream = nullptr;
  int parity = 0;
  int64_t step = 0;
  bool lost = false;  // a failed launch left fields and droplet table of different steps
  int graph_steps = 0;
  int path = LBM_PATH_FUSED;
  bool tile = false;  // the fused path takes its tiled kernel
  // graphs of graph_steps steps, by starting parity, and (2 and 3) of LONG_GRAPH times as many for tiled steps: the
  // last launch of a sequence and the start of the next graph take 8 us, as long as a step.  The long ones are captured
  // by the second call that could use them, so that a single call does not pay for them; a caller who sets the size of
  // the graphs gets graphs of that size alone, captured then.
  hipGraphExec_t exec[4] = {nullptr, nullptr, nullptr, nullptr};
  hipGraph_t graph[4] = {nullptr, nullptr, nullptr, nullptr};
  bool long_graphs = true, long_asked = false;
  // the last recorded forward pass of lbm_adjoint_forward (see lbm_adjoint_backward)
  struct {
    bool valid = false;
    int64_t n0 = 0, nsteps = 0;
    int every = 0, drop = 0;
  } adj;

  void* pool() const { return ws + L.off_pool; }
  InstDev* d_inst() const { return reinterpret_cast<InstDev*>(ws + L.off_inst); }
  TileDev* d_tiles() const { return reinterpret_cast<TileDev*>(ws + L.off_tiles); }
  TileDev* d_ttiles() const { return reinterpret_cast<TileDev*>(ws + L.off_ttiles); }
  TileDev* d_segs() const { return reinterpret_cast<TileDev*>(ws + L.off_segs); }
  DropDev* d_drops() const { return reinterpret_cast<DropDev*>(ws + L.off_drops); }
  double* d_part() const { return reinterpret_cast<double*>(ws + L.off_part); }
  uint64_t* d_mask() const { return reinterpret_cast<uint64_t*>(ws + L.off_mask); }
  int64_t* d_step() const { return reinterpret_cast<int64_t*>(ws + L.off_step); }
  double* d_obs() const { return reinterpret_cast<double*>(ws + L.off_obs); }
  double* d_dbg() const { return reinterpret_cast<double*>(ws + L.off_dbg); }
  bool tiled() const { return path == LBM_PATH_FUSED && tile; }
  // The buffers of step number `ahead` of a sequence of tiled steps.
  TileSeq tile_seq(int64_t ahead) const {
    double* const cen = reinterpret_cast<double*>(ws + L.off_tcen);
    double* const tpart = reinterpret_cast<double*>(ws + L.off_tpart);
    uint32_t* const tmask = reinterpret_cast<uint32_t*>(ws + L.off_tmask);
    const int out = (int)(ahead & 1), in = out ^ 1;
    TileSeq q;
    q.cen_in = ahead == 0 ? nullptr : cen + (size_t)in * 2 * L.ndrop_total;
    q.part_in = tpart + (size_t)in * L.tpart_elems;
    q.mask_in = tmask + (size_t)in * L.nttiles;
    q.cen_out = cen + (size_t)out * 2 * L.ndrop_total;
    q.part_out = tpart + (size_t)out * L.tpart_elems;
    q.mask_out = tmask + (size_t)out * L.nttiles;
    q.ahead = (int32_t)ahead;
    return q;
  }
  int nlaunch() const { return (int)L.tiles.size(); }
  int nseglaunch() const { return (int)L.segs.size(); }
};

namespace {

// Calls f(T{}, P{}) with the arithmetic type T and the population storage type P of a precision code.
template <class F>
decltype(auto) with_types(int prec, F&& f) {
  if (prec == LBM_FP64) return f(double{}, double{});
  if (prec == LBM_FP32) return f(float{}, float{});
  return f(float{}, _Float16{});
}

// Host side of the population storage (the kernels' lb_moments / lb_collide).  FP64 stores the population.
// FP32 stores the deviation from the rest population, fp32(f - fp32(w_i n0)), read back as that deviation plus
// fp32(w_i n0).  FP16 storage keeps fp16(fp32(f) - fp32(w_i n0)), widened back as fp32(stored) + fp32(w_i n0).
template <typename T, typename P>
P host_pop_store(double f, double wn) {
  if constexpr (sizeof(T) == 8) {
    (void)wn;
    return (T)f;
  } else if constexpr (std::is_same<T, P>::value) {
    return (P)(f - (double)(float)wn);
  } else {
    return (P)((float)f - (float)wn);
  }
}
// Whether every instance is periodic in y with the printed advection (the wave kernel's specialised case).
bool all_plain(const std::vector<InstDev>& inst) {
  for (const InstDev& d : inst)
    if (d.walls != LBM_WALLS_NONE || d.advection != LBM_ADV_PAPER) return false;
  return true;
}

// The single kernel of a step on the fused or wave path: over the strip list, or the tiled one with the buffers q of its
// sequence.  insts (the device's) and one (a lattice alone) describe the lattices, drops is their droplet table.
template <typename T, typename P>
hipError_t launch_sweep_on(lbm_ctx* c, int parity, const InstDev* insts, const InstDev* one, const DropDev* drops,
                           const TileSeq& q, double* dbg, int dbg_inst) {
  T* buf = reinterpret_cast<T*>(c->pool());
  if (c->tiled())
    return launch_tile<T, P>(c->stream, parity, c->L.tshape, one ? c->L.nttiles : (int)c->L.ttiles.size(), one,
                             c->d_ttiles(), insts, buf, drops, q, c->d_step(), dbg, dbg_inst);
  if (c->path == LBM_PATH_WAVE)
    return launch_wave<T, P>(c->stream, parity, c->nseglaunch(), c->d_segs(), insts, buf, drops, c->d_part(),
                             c->d_mask(), c->d_step(), dbg, dbg_inst, all_plain(c->L.inst));
  return launch_step<T, P>(c->stream, parity, c->nseglaunch(), c->d_segs(), insts, buf, drops, c->d_part(), c->d_mask(),
                           c->d_step(), dbg, dbg_inst);
}

// The same on the context's own state, as step number `ahead` of its sequence.
template <typename T, typename P>
hipError_t launch_sweep(lbm_ctx* c, int parity, double* dbg, int dbg_inst, int64_t ahead = 0) {
  return launch_sweep_on<T, P>(c, parity, c->d_inst(), c->L.inst.size() == 1 ? c->L.inst.data() : nullptr, c->d_drops(),
                               c->tile_seq(ahead), dbg, dbg_inst);
}

// The two tile kernels of the split path.
template <typename T, typename P>
hipError_t launch_split(lbm_ctx* c, int parity) {
  T* buf = reinterpret_cast<T*>(c->pool());
  hipError_t e = launch_lb<T, P>(c->stream, 0, parity, c->nlaunch(), c->d_tiles(), c->d_inst(), buf, nullptr, -1);
  if (e != hipSuccess) return e;
  return launch_fd<T>(c->stream, 0, parity, c->nlaunch(), c->d_tiles(), c->d_inst(), buf, c->d_drops(), c->d_part(),
                      c->d_mask(), c->d_step(), nullptr, -1);
}

// The centre-of-mass reduction and step counter after the kernels of one step of a path, or with tiled steps after
// the last one of a sequence of n.  write = false: the sums alone (timing).
hipError_t enqueue_reduce(lbm_ctx* c, int64_t n, bool write = true) {
  if (c->tiled())
    return launch_tile_final(c->stream, c->L.ndrop_total, c->d_inst(), c->d_drops(), c->tile_seq(n), c->d_step(),
                             write ? n : 0);
  return launch_reduce(c->stream, c->path == LBM_PATH_SPLIT ? TILING_SPLIT : TILING_FUSED, c->L.ndrop_total, c->d_inst(),
                       c->d_drops(), nullptr, c->d_part(), c->d_mask(), c->d_step(), write ? 1 : -1);
}

// n steps from the given parity.  If a launch fails, `done` tells how many steps were enqueued whole: they stand, with
// the table and the counter, and the state before the failed one is intact.
template <typename T, typename P>
hipError_t enqueue_steps(lbm_ctx* c, int parity, int64_t n, int64_t& done) {
  hipError_t e = hipSuccess;
  for (done = 0; done < n; ++done, parity ^= 1) {
    e = c->path == LBM_PATH_SPLIT ? launch_split<T, P>(c, parity) : launch_sweep<T, P>(c, parity, nullptr, -1, done);
    if (e == hipSuccess && !c->tiled()) e = enqueue_reduce(c, 1);
    if (e != hipSuccess) break;
  }
  if (!c->tiled() || done == 0) return e;
  const hipError_t f = enqueue_reduce(c, done);
  if (f == hipSuccess) return e;
  // without it the table and the counter belong to the sequence's start, whose fields the second step overwrote
  c->lost = c->lost || done > 1;
  done = 0;
  return e == hipSuccess ? f : e;
}

hipError_t enqueue_steps_any(lbm_ctx* c, int parity, int64_t n, int64_t& done) {
  return with_types(c->L.prec,
                    [&](auto t, auto p) { return enqueue_steps<decltype(t), decltype(p)>(c, parity, n, done); });
}

constexpr int LONG_GRAPH = 5;
// Steps launched one by one go in sequences of at most so many: a tiled step knows its number in the sequence in 32 bits.
constexpr int64_t SEQUENCE_MOST = 1 << 20;

void destroy_graphs(lbm_ctx* c) {
  for (int p = 0; p < 4; ++p) {
    if (c->exec[p]) (void)hipGraphExecDestroy(c->exec[p]);
    if (c->graph[p]) (void)hipGraphDestroy(c->graph[p]);
    c->exec[p] = nullptr;
    c->graph[p] = nullptr;
  }
}

int build_graph(lbm_ctx* c, int which) {
  HIPCHK(hipStreamBeginCapture(c->stream, hipStreamCaptureModeRelaxed));
  int64_t done;  // nothing runs yet: a failure here leaves the state as it is
  const bool lost = c->lost;
  const hipError_t err = enqueue_steps_any(c, which & 1, (int64_t)c->graph_steps * (which < 2 ? 1 : LONG_GRAPH), done);
  c->lost = lost;
  hipGraph_t g = nullptr;
  hipError_t e2 = hipStreamEndCapture(c->stream, &g);
  if (err != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return fail(LBM_E_HIP, std::string("kernel launch during capture: ") + hipGetErrorString(err));
  }
  if (e2 != hipSuccess) return fail(LBM_E_HIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e2));
  c->graph[which] = g;
  HIPCHK(hipGraphInstantiate(&c->exec[which], g, nullptr, nullptr, 0));
  return LBM_OK;
}

template <typename T>
void to_device_layout(const double* src, T* dst, int nx, int ny, int pitch) {
  for (int y = 0; y < ny; ++y)
    for (int x = 0; x < pitch; ++x) dst[(size_t)y * pitch + x] = x < nx ? (T)src[(size_t)y * nx + x] : T(0);
}

template <typename T, typename P>
int upload_instance(lbm_ctx* c, int i, const double* phi0, const double* c0, const double* f_pre) {
  const InstDev& d = c->L.inst[i];
  const int nx = d.nx, ny = d.ny, pitch = d.pitch;
  const size_t plane = (size_t)d.pstride;
  std::vector<T> h(plane);
  std::vector<P> hf(plane * 9);
  T* base = reinterpret_cast<T*>(c->pool());
  to_device_layout(phi0, h.data(), nx, ny, pitch);
  HIPCHK(hipMemcpyAsync(base + d.off_phi[0], h.data(), plane * sizeof(T), hipMemcpyHostToDevice, c->stream));
  HIPCHK(hipStreamSynchronize(c->stream));
  to_device_layout(c0, h.data(), nx, ny, pitch);
  HIPCHK(hipMemcpyAsync(base + d.off_c[0], h.data(), plane * sizeof(T), hipMemcpyHostToDevice, c->stream));
  HIPCHK(hipStreamSynchronize(c->stream));
  // Stored populations are post-collision values at the emitting node: f*_i(r) = f_i(r + e_i); with walls,
  // a population streamed into a plate comes back to r reversed: f*_i(r) = f_OPP[i](r).
  P* fbase = reinterpret_cast<P*>(base + d.off_f[0]);
  const bool walls = c->cfg[i].walls != 0;
  for (int k = 0; k < 9; ++k)
    for (int y = 0; y < ny; ++y)
      for (int x = 0; x < nx; ++x) {
        double v;
        if (f_pre) {
          const int yt = y + EY[k];
          if (walls && (yt < 0 || yt >= ny)) {
            v = f_pre[(size_t)OPP[k] * nx * ny + (size_t)y * nx + x];
          } else {
            const int xs = (x + EX[k] + nx) % nx, ys = (yt + ny) % ny;
            v = f_pre[(size_t)k * nx * ny + (size_t)ys * nx + xs];
          }
        } else {
          v = WGT[k] * c->cfg[i].n0;
        }
        hf[(size_t)k * plane + (size_t)y * pitch + x] = host_pop_store<T, P>(v, WGT[k] * c->cfg[i].n0);
      }
  HIPCHK(hipMemcpyAsync(fbase, hf.data(), 9 * plane * sizeof(P), hipMemcpyHostToDevice, c->stream));
  HIPCHK(hipStreamSynchronize(c->stream));
  // velocity / density planes start at zero; the second buffers are fully rewritten by the first step
  HIPCHK(hipMemsetAsync(base + d.off_ux, 0, 3 * plane * sizeof(T), c->stream));
  HIPCHK(hipMemsetAsync(base + d.off_f[1], 0, 9 * plane * sizeof(P), c->stream));
  HIPCHK(hipMemsetAsync(base + d.off_phi[1], 0, plane * sizeof(T), c->stream));
  HIPCHK(hipMemsetAsync(base + d.off_c[1], 0, plane * sizeof(T), c->stream));
  return LBM_OK;
}

int fail_lost() { return fail(LBM_E_STATE, "a failed launch left the context's state incomplete"); }

int check_inst(lbm_ctx* c, int32_t inst) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (inst < 0 || inst >= (int)c->L.inst.size()) return fail(LBM_E_INVAL, "instance index out of range");
  return c->lost ? fail_lost() : LBM_OK;
}

// n, u planes of an instance from the current state (Eq. 11 with the force of Eq. 14).
int run_diag(lbm_ctx* c, int inst) {
  const hipError_t e = with_types(c->L.prec, [&](auto t, auto p) {
    using T = decltype(t);
    return launch_lb<T, decltype(p)>(c->stream, 2, c->parity, c->nlaunch(), c->d_tiles(), c->d_inst(),
                                     reinterpret_cast<T*>(c->pool()), nullptr, inst);
  });
  if (e != hipSuccess) return fail(LBM_E_HIP, std::string("diagnostic launch: ") + hipGetErrorString(e));
  return LBM_OK;
}

// A call's block of page-locked memory, on the context's stream.
class ReadBuf {
 public:
  explicit ReadBuf(lbm_ctx* c) : c_(c) {}
  ReadBuf(const ReadBuf&) = delete;
  ReadBuf& operator=(const ReadBuf&) = delete;
  // A call that ends early leaves work on the stream that writes to the block: it is waited for.  If that fails, the
  // block is not used again.
  ~ReadBuf() {
    if (!mem_ || (pending_ && hipStreamSynchronize(c_->stream) != hipSuccess)) return;
    ReadBlocks::get().give(size_, mem_);
  }
  int take(size_t bytes) {
    size_ = bytes <= READ_BLOCK[0] ? 0 : 1;
    HIPCHK(ReadBlocks::get().take(size_, &mem_));
    return LBM_OK;
  }
  // The block, for work that is about to be enqueued.
  char* fill() {
    pending_ = true;
    return mem_;
  }
  // Waits for all of it: for the stream, or for an event recorded behind it (35 us less where a call has recorded one).
  int wait(hipEvent_t last = nullptr) {
    HIPCHK(last ? hipEventSynchronize(last) : hipStreamSynchronize(c_->stream));
    pending_ = false;
    return LBM_OK;
  }
  const char* data() const { return mem_; }

 private:
  lbm_ctx* c_;
  char* mem_ = nullptr;
  int size_ = 0;
  bool pending_ = false;
};

// One event for each half of a block: the host waits for a chunk while the kernel of the next one is already on its
// way (waiting for the stream between chunks takes 12 us more for each: 512 x 256 FP64, all fields).
struct ReadEvents {
  hipEvent_t e[2] = {nullptr, nullptr};
  hipError_t create() {
    hipError_t rc = hipSuccess;
    for (hipEvent_t& v : e)
      if (rc == hipSuccess) rc = hipEventCreateWithFlags(&v, hipEventDisableTiming);
    return rc;
  }
  ~ReadEvents() {
    for (hipEvent_t v : e)
      if (v) (void)hipEventDestroy(v);
  }
};

// Nodes of a chunk of a read-back of np planes, and the bytes of one with its head.
int64_t read_chunk(int64_t nodes, int np) {
  const size_t node_bytes = sizeof(double) * np;
  return (size_t)nodes * node_bytes <= READ_CHUNK ? nodes : (int64_t)(READ_CHUNK / node_bytes);
}
size_t read_half(int64_t nodes, int np) {
  return align_up(READ_HEAD + (size_t)read_chunk(nodes, np) * sizeof(double) * np, ALIGN);
}

// np planes of `nodes` doubles to the caller's arrays dst, by launch(first, count, values, flag): it fills the planes'
// nodes [first, first + count), one plane after another, and sets the flag where a value is not finite.
template <class F>
int read_planes(lbm_ctx* c, int64_t nodes, int np, double* const* dst, bool& finite, F launch) {
  const int64_t per = read_chunk(nodes, np), chunks = (nodes + per - 1) / per;
  const size_t half = read_half(nodes, np);
  ReadBuf buf(c);
  ReadEvents ev;
  int rc = buf.take((chunks > 1 ? 2 : 1) * half);
  if (rc != LBM_OK) return rc;
  if (chunks > 1) HIPCHK(ev.create());
  finite = true;
  for (int64_t k = 0; k <= chunks; ++k) {
    if (k < chunks) {
      char* const h = buf.fill() + (k & 1) * half;
      const int64_t first = k * per;
      *reinterpret_cast<uint32_t*>(h) = 0u;
      HIPCHK(launch(first, std::min(per, nodes - first), reinterpret_cast<double*>(h + READ_HEAD),
                    reinterpret_cast<uint32_t*>(h)));
      if (chunks > 1) HIPCHK(hipEventRecord(ev.e[k & 1], c->stream));
    }
    if (k == 0) continue;
    if (k < chunks)
      HIPCHK(hipEventSynchronize(ev.e[(k - 1) & 1]));
    else if ((rc = buf.wait(chunks > 1 ? ev.e[(k - 1) & 1] : nullptr)) != LBM_OK)
      return rc;
    const char* const h = buf.data() + ((k - 1) & 1) * half;
    const int64_t first = (k - 1) * per, count = std::min(per, nodes - first);
    const double* v = reinterpret_cast<const double*>(h + READ_HEAD);
    for (int j = 0; j < np; ++j, v += count) memcpy(dst[j] + first, v, sizeof(double) * (size_t)count);
    if (*reinterpret_cast<const uint32_t*>(h)) finite = false;
  }
  return LBM_OK;
}

// The requested fields of an instance (null: not requested) as the caller's arrays hold them; `finite` tells whether
// all their values are.
template <typename T, typename P>
int fields_impl(lbm_ctx* c, int inst, double* f_pre, double* phi, double* cc, double* n, double* ux, double* uy,
                bool& finite) {
  const InstDev& d = c->L.inst[inst];
  const int64_t nodes = (int64_t)d.nx * d.ny;
  double* dst[14];
  int np = 0, rc;
  for (int k = 0; f_pre && k < 9; ++k) dst[np++] = f_pre + k * nodes;
  for (double* o : {phi, cc, n, ux, uy})
    if (o) dst[np++] = o;
  if (np == 0) {
    HIPCHK(hipStreamSynchronize(c->stream));
    return LBM_OK;
  }
  const int want = (f_pre ? FIELD_F : 0) | (phi ? FIELD_PHI : 0) | (cc ? FIELD_C : 0) | (n ? FIELD_N : 0) |
                   (ux ? FIELD_UX : 0) | (uy ? FIELD_UY : 0);
  if ((n || ux || uy) && (rc = run_diag(c, inst)) != LBM_OK) return rc;
  return read_planes(c, nodes, np, dst, finite, [&](int64_t first, int64_t count, double* v, uint32_t* bad) {
    return launch_fields<T, P>(c->stream, d, c->parity, reinterpret_cast<const T*>(c->pool()), first, count, want, v,
                               bad);
  });
}

// Stage planes of the next step of instance `inst` from the kernels of the current path.
template <typename T, typename P>
hipError_t launch_split_export(lbm_ctx* c, int parity, const InstDev* insts, const DropDev* drops, double* dbg,
                               int dbg_inst) {
  T* buf = reinterpret_cast<T*>(c->pool());
  hipError_t e = launch_lb<T, P>(c->stream, 1, parity, c->nlaunch(), c->d_tiles(), insts, buf, dbg, dbg_inst);
  if (e != hipSuccess) return e;
  return launch_fd<T>(c->stream, 1, parity, c->nlaunch(), c->d_tiles(), insts, buf, drops, c->d_part(), c->d_mask(),
                      c->d_step(), dbg, dbg_inst);
}
template <typename T, typename P>
hipError_t debug_launch(lbm_ctx* c, int inst, double* dbg) {
  const int di = export_planes(inst, true);
  if (c->path != LBM_PATH_SPLIT) return launch_sweep<T, P>(c, c->parity, dbg, di);
  return launch_split_export<T, P>(c, c->parity, c->d_inst(), c->d_drops(), dbg, di);
}

// One eager step with hipEvents between its kernels: ev[0..nk] bracket nk launches.
template <typename T, typename P>
hipError_t timed_step(lbm_ctx* c, hipEvent_t* ev, int* nk) {
  T* buf = reinterpret_cast<T*>(c->pool());
  const int p = c->parity;
  hipError_t e;
  (void)hipEventRecord(ev[0], c->stream);
  if (c->path != LBM_PATH_SPLIT) {
    e = launch_sweep<T, P>(c, p, nullptr, -1);
    (void)hipEventRecord(ev[1], c->stream);
    if (e == hipSuccess) e = enqueue_reduce(c, 1);
    (void)hipEventRecord(ev[2], c->stream);
    *nk = 2;
  } else {
    e = launch_lb<T, P>(c->stream, 0, p, c->nlaunch(), c->d_tiles(), c->d_inst(), buf, nullptr, -1);
    (void)hipEventRecord(ev[1], c->stream);
    if (e == hipSuccess)
      e = launch_fd<T>(c->stream, 0, p, c->nlaunch(), c->d_tiles(), c->d_inst(), buf, c->d_drops(), c->d_part(),
                       c->d_mask(), c->d_step(), nullptr, -1);
    (void)hipEventRecord(ev[2], c->stream);
    if (e == hipSuccess) e = enqueue_reduce(c, 1);
    (void)hipEventRecord(ev[3], c->stream);
    *nk = 3;
  }
  c->parity ^= 1;
  c->step += 1;
  return e;
}

int read_drops(lbm_ctx* c, int inst, std::vector<DropDev>& out) {
  const InstDev& d = c->L.inst[inst];
  out.resize(d.ndrop);
  if (d.ndrop == 0) return LBM_OK;
  const size_t bytes = sizeof(DropDev) * d.ndrop;
  ReadBuf buf(c);
  int rc = buf.take(bytes);
  if (rc != LBM_OK) return rc;
  HIPCHK(hipMemcpyAsync(buf.fill(), c->d_drops() + d.drop_base, bytes, hipMemcpyDeviceToHost, c->stream));
  if ((rc = buf.wait()) != LBM_OK) return rc;
  memcpy(out.data(), buf.data(), bytes);
  return LBM_OK;
}

// The droplet table of every instance (device copy).
int read_all_drops(lbm_ctx* c, std::vector<DropDev>& out) {
  out.resize(c->L.ndrop_total);
  if (c->L.ndrop_total == 0) return LBM_OK;
  HIPCHK(hipMemcpyAsync(out.data(), c->d_drops(), sizeof(DropDev) * out.size(), hipMemcpyDeviceToHost, c->stream));
  HIPCHK(hipStreamSynchronize(c->stream));
  return LBM_OK;
}

// Rebuild the strip list for a segment height and strip width (launch order from the current droplet
// centres) and upload it.  shorter: the strips' height where it is not the height the caller sees, one of SHORT_ROWS.
int apply_segments(lbm_ctx* c, int rows, int width, int shorter = 0) {
  const int h = shorter ? shorter : rows;
  for (const InstDev& d : c->L.inst)
    if (strip_count(d.nx, d.ny, width, h) > strip_bound(d.nx, d.ny))
      return fail(LBM_E_INVAL, "more strips than the workspace is sized for");
  HIPCHK(hipStreamSynchronize(c->stream));
  destroy_graphs(c);
  std::vector<DropDev> drops;
  int rc = read_all_drops(c, drops);
  if (rc != LBM_OK) return rc;
  set_segments(c->L, h, width, drops);
  c->L.seg_rows = rows;
  HIPCHK(hipMemcpyAsync(c->d_inst(), c->L.inst.data(), sizeof(InstDev) * c->L.inst.size(), hipMemcpyHostToDevice,
                        c->stream));
  HIPCHK(hipMemcpyAsync(c->d_segs(), c->L.segs.data(), sizeof(TileDev) * c->L.segs.size(), hipMemcpyHostToDevice,
                        c->stream));
  HIPCHK(hipStreamSynchronize(c->stream));
  return LBM_OK;
}

// ---- Scratch of the entry point that allocates nothing (lbm_step_noalloc) ---------------------------------
// The instance description, the strip list, the step counter, the droplet table, the centre-of-mass partials
// and the presence masks of lbm_step_noalloc live in this device array: each GPU the library runs on holds its
// own copy until the process ends.  In host code `scratch` names the symbol, not a device address; host code
// uses only the address hipGetSymbolAddress returned on the current device (g_scratch_ptr).
static __device__ __align__(256) unsigned char scratch[LBM_NOALLOC_SCRATCH_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
constexpr int NOALLOC_ROWS_MIN = 4, NOALLOC_ROWS_MAX = 128;
constexpr int NOALLOC_ROWS_FIT = 40;  // the height that decides whether a lattice fits the scratch array
constexpr int SIMDS = 1024;           // 256 compute units

int noalloc_segments(int nx, int ny, int rows) { return ((nx + FUSED_TX - 1) / FUSED_TX) * ((ny + rows - 1) / rows); }

// Wavefronts per SIMD that k_wave's segments are planned for.
int noalloc_waves(int prec) { return prec == LBM_FP64 ? 2 : 3; }

// Strip height of lbm_step_noalloc, which has no autotuner.  A segment sweeps its rows and ten more, one iteration
// each, and an iteration takes as long as its SIMD's wavefronts make it: the height with the least
// iterations x time, for the wavefronts per SIMD that its segments make (an extra one up to the most that are
// planned for, a further round of them beyond).  Times of an iteration with 1, 2 and 3 wavefronts per SIMD, in us,
// from launches on 700^2 to 2048^2 lattices.  FP64 leaves a tenth of the slots free: 2048^2 takes 193 us with 1786
// wavefronts (44 rows), 200 with 1976 (40 rows).  FP16 storage is bound by arithmetic, and its rounds count throughout:
// 4096^2 315, 291 and, in two rounds of 54 rows, 287.  Lattices of MANY_ROUNDS in 16-row strips are bound by memory.  In
// FP32 the shortest strips are the best there: their neighbours read the shared halo rows soon after one another.  In
// FP64 they gain only in a long row of launches (4096^2 759, 780 and 801 us at 16, 40 and 80 rows) and lose in short calls
// (10 steps with 8 droplets, first call on a new state / repeated: 8900 / 7900 at 16 rows, 8350 / 7830 at 40), so it stays
// at 40.  The line lies where the two sides meet; us a step in calls of 10, repeated, the model's height / the fixed one:
// FP32 3200^2 (3.9 rounds) 269 / 278, 3600^2 (4.9) 334 / 337, 3800^2 (5.5) 374 / 381, 4096^2 (6.3) 458 / 441;
// FP64 2700^2 (4.6) 348 / 362, 2900^2 (5.3) 400 / 399, 3200^2 (6.5) 498 / 491.
// The centres' sums are rounded by strip, so the height decides their last bits.  Lattices below 256 x 256 nodes keep 40
// rows for that alone: a program that compares them with lbm_step's at that height finds the same bits as ever.  It costs
// them a good deal (250 x 250 FP64 105 us a step, 28 at the 4 rows that 256 x 256 takes; FP32 86 and 24).
int noalloc_rows(int nx, int ny, int prec) {
  if ((int64_t)nx * ny < 256 * 256) return NOALLOC_ROWS_FIT;
  static constexpr double ITER[3][3] = {{2.1, 3.4, 3.4}, {1.6, 1.65, 1.97}, {1.5, 1.6, 1.97}};
  const int most = noalloc_waves(prec);
  const double per_round = (prec == LBM_FP64 ? 0.9 : 1.0) * SIMDS;
  constexpr int SHORT = 16;
  constexpr double MANY_ROUNDS = 5.5;
  if (prec != LBM_FP16 && noalloc_segments(nx, ny, SHORT) >= MANY_ROUNDS * most * per_round)
    return prec == LBM_FP32 ? SHORT : NOALLOC_ROWS_FIT;
  int best = NOALLOC_ROWS_FIT;
  double best_cost = 1e300;
  for (int h = NOALLOC_ROWS_MIN; h <= NOALLOC_ROWS_MAX; ++h) {
    const int waves = std::max(1, (int)std::ceil(noalloc_segments(nx, ny, h) / per_round));
    const int rounds = (waves + most - 1) / most;
    const double cost = rounds * (h + 10) * ITER[prec][std::min(waves, most) - 1];
    if (cost < best_cost) {
      best_cost = cost;
      best = h;
    }
  }
  return best;
}
std::mutex g_scratch_mu;
void* g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

// Address of `scratch` on the current device, looked up once per device (with that device current).
int scratch_on_current_device(void** out) {
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return fail(LBM_E_HIP, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(LBM_E_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return LBM_OK;
}

// Byte offsets of the regions of the scratch array for one lattice.
struct NoallocLayout {
  size_t inst, step, drops, segs, mask, part, total;
};

NoallocLayout noalloc_layout(int nsegs, int nslots, int ndrop) {
  NoallocLayout L;
  size_t off = 0;
  L.inst = off;  off = align_up(off + sizeof(InstDev), ALIGN);
  L.step = off;  off = align_up(off + sizeof(int64_t), ALIGN);
  L.drops = off; off = align_up(off + sizeof(DropDev) * (size_t)std::max(1, ndrop), ALIGN);
  L.segs = off;  off = align_up(off + sizeof(TileDev) * (size_t)nslots, ALIGN);
  L.mask = off;  off = align_up(off + sizeof(uint64_t) * MASK_WORDS * (size_t)nsegs, ALIGN);
  L.part = off;  off = align_up(off + sizeof(double) * 3 * (size_t)nsegs * (size_t)std::max(1, ndrop), ALIGN);
  L.total = off;
  return L;
}

NoallocLayout noalloc_layout(const lbm_config& c, int32_t ndrop, int rows) {
  const int n = noalloc_segments(c.nx, c.ny, rows);
  return noalloc_layout(n, (n + 7) / 8 * 8, ndrop);
}

// The height that a lattice gets: the rule's, or a taller one where only that fits the scratch array.
int noalloc_height(const lbm_config& c, int32_t ndrop, int& rows) {
  const size_t need = noalloc_layout(c, ndrop, NOALLOC_ROWS_FIT).total;
  if (need > LBM_NOALLOC_SCRATCH_BYTES)
    return fail(LBM_E_NOMEM, "this lattice and droplet count need " + std::to_string(need) +
                                 " bytes of scratch, more than LBM_NOALLOC_SCRATCH_BYTES (" +
                                 std::to_string((size_t)LBM_NOALLOC_SCRATCH_BYTES) + ")");
  rows = noalloc_rows(c.nx, c.ny, c.precision);
  if (noalloc_layout(c, ndrop, rows).total > LBM_NOALLOC_SCRATCH_BYTES) rows = std::max(rows, NOALLOC_ROWS_FIT);
  return LBM_OK;
}

// Fills the scratch regions: instance description, step counter, droplet table (from the caller's), the presence
// masks cleared, and the strip list in the XCD-aware order of set_segments: block j < 8 lists the run of natural
// strips [j * chunk, (j + 1) * chunk) in the slots j, j + 8, ..., those near a droplet first if `order` is set (as
// set_segments does: the longer-running strips do not end the launch).  Any table gives a permutation of the strips.
// The order needs each strip's distance to the droplets once, in FP32, by all threads of a block.  With the distances
// taken in both passes, in FP64 and by one thread a strip the kernel took 18.6 us with 64 droplets and 86.3 us with 256
// (2048x2048 FP32, 3002 and 1976 strips); 8.3 and 12.4 us now.  An FP32 distance may put a strip on the other side of
// the line: only the order of the blocks changes, never a result.
constexpr int SETUP_THREADS = 1024;
constexpr int SETUP_STRIPS = SETUP_THREADS / 2;  // of a run that is ordered, at most
__global__ __launch_bounds__(SETUP_THREADS) void k_noalloc_setup(InstDev inst, int64_t step, NoallocLayout L, int nsegs,
                                                                 int chunk, int ndrop, int order,
                                                                 const lbm_droplet* __restrict__ drops,
                                                                 char* __restrict__ s) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int gid = blockIdx.x * SETUP_THREADS + tid;
  const int stride = gridDim.x * SETUP_THREADS;
  if (gid == 0) {
    *reinterpret_cast<InstDev*>(s + L.inst) = inst;
    *reinterpret_cast<int64_t*>(s + L.step) = step;
  }
  uint64_t* mask = reinterpret_cast<uint64_t*>(s + L.mask);
  for (int m = gid; m < nsegs * MASK_WORDS; m += stride) mask[m] = 0ull;
  DropDev* dd = reinterpret_cast<DropDev*>(s + L.drops);
  for (int k = gid; k < ndrop; k += stride) {
    const lbm_droplet q = drops[k];
    dd[k] = DropDev{q.x, q.y, q.R, q.Rs, q.ex, q.ey, q.active ? 1 : 0, 0};
  }
  if (blockIdx.x >= 8) return;
  constexpr int NW = SETUP_THREADS / 64;
  __shared__ float s_drop[MAXDROP][3];  // centre and reach
  __shared__ bool s_near[SETUP_STRIPS];
  __shared__ int s_count[NW], s_done;
  const int tx = inst.tiles_x[TILING_FUSED];
  const int t0 = blockIdx.x * chunk, t1 = min(nsegs, t0 + chunk);
  TileDev* const run = reinterpret_cast<TileDev*>(s + L.segs) + blockIdx.x;  // every eighth slot
  auto strip = [&](int t) { return TileDev{0, (t % tx) * inst.strip_w, (t / tx) * inst.seg_rows, t}; };
  if (tid == 0) s_done = 0;
  if (order) {
    for (int k = tid; k < ndrop; k += SETUP_THREADS) {
      s_drop[k][0] = (float)drops[k].x;
      s_drop[k][1] = (float)drops[k].y;
      s_drop[k][2] = (float)drops[k].R + 2.0f;
    }
    __syncthreads();
    // each strip by as many neighbouring lanes as there are threads for
    int lanes = 64;
    while (lanes * chunk > SETUP_THREADS) lanes >>= 1;
    const int t = t0 + tid / lanes;
    bool near = false;
    if (t < t1) {
      const TileDev e = strip(t);
      const int x1 = min(e.x0 + inst.strip_w, inst.nx) - 1, y1 = min(e.y0 + inst.seg_rows, inst.ny) - 1;
      const float xm = 0.5f * (e.x0 + x1), ym = 0.5f * (e.y0 + y1), hx = 0.5f * (x1 - e.x0), hy = 0.5f * (y1 - e.y0);
      for (int k = tid % lanes; k < ndrop && !near; k += lanes) {
        float dx = fabsf(xm - s_drop[k][0]), dy = fabsf(ym - s_drop[k][1]);
        if (dx > 0.5f * inst.nx) dx = inst.nx - dx;
        if (!inst.walls && dy > 0.5f * inst.ny) dy = inst.ny - dy;
        dx = fmaxf(0.0f, dx - hx);
        dy = fmaxf(0.0f, dy - hy);
        near = dx * dx + dy * dy <= s_drop[k][2] * s_drop[k][2];
      }
    }
    const unsigned long long group = (lanes == 64 ? ~0ull : (1ull << lanes) - 1ull) << (lane / lanes * lanes);
    near = (__ballot(near) & group) != 0ull;
    if (t < t1 && tid % lanes == 0) s_near[t - t0] = near;
  }
  __syncthreads();
  for (int pass = order ? 0 : 1; pass < 2; ++pass) {
    for (int base = t0; base < t1; base += SETUP_THREADS) {
      const int t = base + tid;
      const bool mine = t < t1 && (!order || s_near[t - t0] == (pass == 0));
      const unsigned long long b = __ballot(mine);
      if (lane == 0) s_count[wv] = __popcll(b);
      __syncthreads();
      int at = s_done + __popcll(b & ((1ull << lane) - 1ull)), all = 0;
      for (int w = 0; w < NW; ++w) {
        at += w < wv ? s_count[w] : 0;
        all += s_count[w];
      }
      if (mine) run[(size_t)at * 8] = strip(t);
      __syncthreads();
      if (tid == 0) s_done += all;
      __syncthreads();
    }
  }
  for (int k = max(t1 - t0, 0) + tid; k < chunk; k += SETUP_THREADS) run[(size_t)k * 8] = TileDev{-1, 0, 0, -1};
}

// The new centres back into the caller's droplet table.
__global__ __launch_bounds__(NTHREADS) void k_noalloc_centres(const DropDev* __restrict__ dd, int ndrop,
                                                              lbm_droplet* __restrict__ drops) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < ndrop) {
    drops[k].x = dd[k].x;
    drops[k].y = dd[k].y;
  }
}

}  // namespace

extern "C" {

int32_t lbm_noalloc_rows(const lbm_config* cfg, int32_t ndrop) {
  if (!cfg) return fail(LBM_E_INVAL, "cfg must not be NULL");
  int rows = 0;
  int rc = validate(1, cfg, &ndrop);
  if (rc == LBM_OK) rc = noalloc_height(*cfg, ndrop, rows);
  return rc == LBM_OK ? rows : rc;
}

int lbm_step_noalloc(const lbm_config* cfg, void* stream, void* const f[2], void* const phi[2], void* const c[2],
                     int32_t ndrop, lbm_droplet* drops, int64_t step, int64_t nsteps) {
  if (!cfg) return fail(LBM_E_INVAL, "cfg must not be NULL");
  int rc = validate(1, cfg, &ndrop);
  if (rc != LBM_OK) return rc;
  if (!f || !phi || !c) return fail(LBM_E_INVAL, "f, phi and c must not be NULL");
  void* const bufs[6] = {f[0], f[1], phi[0], phi[1], c[0], c[1]};
  for (void* b : bufs)
    if (!b || reinterpret_cast<uintptr_t>(b) % ALIGN)
      return fail(LBM_E_INVAL, "state buffers must be non-NULL and 256-byte aligned");
  if (ndrop > 0 && !drops) return fail(LBM_E_INVAL, "drops must not be NULL when ndrop > 0");
  if (step < 0 || nsteps < 0) return fail(LBM_E_INVAL, "step and nsteps must be >= 0");
  const lbm_config& cf = *cfg;
  const size_t elem = cf.precision == LBM_FP64 ? 8 : 4;
  InstDev d;
  memset(&d, 0, sizeof d);
  d.nx = cf.nx;
  d.ny = cf.ny;
  d.pitch = cf.nx;
  d.pstride = (int64_t)cf.nx * cf.ny;
  d.ndrop = ndrop;
  d.strip_w = FUSED_TX;
  if ((rc = noalloc_height(cf, ndrop, d.seg_rows)) != LBM_OK) return rc;
  d.tiles_x[TILING_FUSED] = (cf.nx + FUSED_TX - 1) / FUSED_TX;
  d.tiles_y[TILING_FUSED] = (cf.ny + d.seg_rows - 1) / d.seg_rows;
  // element offsets of the caller's buffers from f[0] (the pool base of the kernels); 256-byte alignment makes
  // every difference a whole number of elements
  const char* base = static_cast<const char*>(f[0]);
  auto off = [&](void* b) { return (int64_t)(static_cast<const char*>(b) - base) / (int64_t)elem; };
  d.off_f[0] = off(f[0]);
  d.off_f[1] = off(f[1]);
  d.off_phi[0] = off(phi[0]);
  d.off_phi[1] = off(phi[1]);
  d.off_c[0] = off(c[0]);
  d.off_c[1] = off(c[1]);
  set_model(cf, d);
  const int nsegs = d.tiles_x[TILING_FUSED] * d.tiles_y[TILING_FUSED];
  const int nslots = (nsegs + 7) / 8 * 8;
  const NoallocLayout L = noalloc_layout(nsegs, nslots, ndrop);
  void* sp = nullptr;
  if ((rc = scratch_on_current_device(&sp)) != LBM_OK) return rc;
  char* s = static_cast<char*>(sp);
  hipStream_t st = static_cast<hipStream_t>(stream);
  // with strips for a second round and more, the order within a run no longer decides how the launch ends
  const bool order = ndrop > 0 && nslots / 8 <= SETUP_STRIPS;
  static_assert(8 * SETUP_STRIPS == 4 * SIMDS, "four wavefronts per SIMD");
  const int blocks = std::max(8, (nsegs * MASK_WORDS + SETUP_THREADS - 1) / SETUP_THREADS);
  hipLaunchKernelGGL(k_noalloc_setup, dim3(blocks), dim3(SETUP_THREADS), 0, st, d, step, L, nsegs, nslots / 8, ndrop,
                     order ? 1 : 0, drops, s);
  HIPCHK(hipGetLastError());
  const InstDev* di = reinterpret_cast<const InstDev*>(s + L.inst);
  const TileDev* segs = reinterpret_cast<const TileDev*>(s + L.segs);
  DropDev* dd = reinterpret_cast<DropDev*>(s + L.drops);
  double* part = reinterpret_cast<double*>(s + L.part);
  uint64_t* mask = reinterpret_cast<uint64_t*>(s + L.mask);
  int64_t* dstep = reinterpret_cast<int64_t*>(s + L.step);
  for (int64_t k = 0; k < nsteps; ++k) {
    const int parity = (int)(k & 1);
    hipError_t e = with_types(cf.precision, [&](auto t, auto p) {
      using T = decltype(t);
      return launch_wave<T, decltype(p)>(st, parity, nslots, segs, di, reinterpret_cast<T*>(const_cast<char*>(base)), dd,
                                         part, mask, dstep, nullptr, -1,
                                         cf.walls == LBM_WALLS_NONE && cf.advection == LBM_ADV_PAPER);
    });
    if (e == hipSuccess) e = launch_reduce(st, TILING_FUSED, ndrop, di, dd, nullptr, part, mask, dstep, 1);
    if (e != hipSuccess) return fail(LBM_E_HIP, std::string("timestep launch: ") + hipGetErrorString(e));
  }
  if (ndrop > 0) {
    hipLaunchKernelGGL(k_noalloc_centres, dim3((ndrop + NTHREADS - 1) / NTHREADS), dim3(NTHREADS), 0, st, dd, ndrop,
                       drops);
    HIPCHK(hipGetLastError());
  }
  return LBM_OK;
}

int lbm_workspace_bytes(int32_t ninst, const lbm_config* cfgs, const int32_t* ndrop, size_t* bytes) {
  if (!bytes) return fail(LBM_E_INVAL, "bytes must not be NULL");
  int rc = validate(ninst, cfgs, ndrop);
  if (rc != LBM_OK) return rc;
  Layout L;
  make_layout(ninst, cfgs, ndrop, L);
  *bytes = L.total;
  return LBM_OK;
}

int lbm_init_batch(int32_t ninst, const lbm_config* cfgs, void* workspace, size_t workspace_bytes, void* stream,
                   const double* phi0, const double* c0, const double* f_pre, const int32_t* ndrop,
                   const lbm_droplet* drops, int64_t step, lbm_ctx** out) {
  if (!out) return fail(LBM_E_INVAL, "out must not be NULL");
  *out = nullptr;
  int rc = validate(ninst, cfgs, ndrop);
  if (rc != LBM_OK) return rc;
  if (!workspace) return fail(LBM_E_INVAL, "workspace must not be NULL");
  if (reinterpret_cast<uintptr_t>(workspace) % ALIGN) return fail(LBM_E_INVAL, "workspace must be 256-byte aligned");
  if (!phi0 || !c0) return fail(LBM_E_INVAL, "phi0 and c0 must not be NULL");
  if (step < 0) return fail(LBM_E_INVAL, "step must be >= 0");
  int nd_total = 0;
  for (int i = 0; i < ninst; ++i) nd_total += ndrop[i];
  if (nd_total > 0 && !drops) return fail(LBM_E_INVAL, "drops must not be NULL when droplets are requested");
  for (int k = 0; k < nd_total; ++k) {
    const lbm_droplet& d = drops[k];
    if (!std::isfinite(d.x) || !std::isfinite(d.y) || !std::isfinite(d.ex) || !std::isfinite(d.ey) ||
        !(d.R >= 0.0) || !(d.Rs >= 0.0))
      return fail(LBM_E_INVAL, "droplet table entries must be finite with R, Rs >= 0");
  }
  std::vector<DropDev> dd(std::max(1, nd_total));
  {
    int k = 0;
    for (int i = 0; i < ninst; ++i)
      for (int j = 0; j < ndrop[i]; ++j, ++k) {
        const lbm_droplet& s = drops[k];
        dd[k] = DropDev{s.x, s.y, s.R, s.Rs, s.ex, s.ey, s.active ? 1 : 0, i};
      }
  }
  lbm_ctx* c = new lbm_ctx();
  make_layout(ninst, cfgs, ndrop, c->L);
  set_segments(c->L, SEG_ROWS_DEFAULT, FUSED_TX, std::vector<DropDev>(dd.begin(), dd.begin() + nd_total));
  if (workspace_bytes < c->L.total) {
    delete c;
    return fail(LBM_E_NOMEM, "workspace smaller than lbm_workspace_bytes()");
  }
  c->cfg.assign(cfgs, cfgs + ninst);
  c->ws = static_cast<char*>(workspace);
  c->stream = static_cast<hipStream_t>(stream);
  c->step = step;
  c->tile = c->L.tshape >= 0;
  c->graph_steps = stream ? 20 : 0;

  auto bail = [&](int code) {
    destroy_graphs(c);
    delete c;
    return code;
  };
  size_t off_field = 0;
  for (int i = 0; i < ninst; ++i) {
    const size_t n = (size_t)cfgs[i].nx * cfgs[i].ny;
    rc = with_types(c->L.prec, [&](auto t, auto p) {
      return upload_instance<decltype(t), decltype(p)>(c, i, phi0 + off_field, c0 + off_field,
                                                       f_pre ? f_pre + 9 * off_field : nullptr);
    });
    if (rc != LBM_OK) return bail(rc);
    off_field += n;
  }
  hipError_t e;
#define INIT_CHK(call)                                                                               \
  do {                                                                                               \
    e = (call);                                                                                      \
    if (e != hipSuccess) return bail(fail(LBM_E_HIP, std::string(#call) + ": " + hipGetErrorString(e))); \
  } while (0)
  INIT_CHK(hipMemcpyAsync(c->d_inst(), c->L.inst.data(), sizeof(InstDev) * ninst, hipMemcpyHostToDevice, c->stream));
  INIT_CHK(hipMemcpyAsync(c->d_tiles(), c->L.tiles.data(), sizeof(TileDev) * c->L.tiles.size(), hipMemcpyHostToDevice,
                          c->stream));
  INIT_CHK(hipMemcpyAsync(c->d_segs(), c->L.segs.data(), sizeof(TileDev) * c->L.segs.size(), hipMemcpyHostToDevice,
                          c->stream));
  if (!c->L.ttiles.empty())
    INIT_CHK(hipMemcpyAsync(c->d_ttiles(), c->L.ttiles.data(), sizeof(TileDev) * c->L.ttiles.size(),
                            hipMemcpyHostToDevice, c->stream));
  INIT_CHK(hipMemcpyAsync(c->d_drops(), dd.data(), sizeof(DropDev) * dd.size(), hipMemcpyHostToDevice, c->stream));
  INIT_CHK(hipMemcpyAsync(c->d_step(), &c->step, sizeof(int64_t), hipMemcpyHostToDevice, c->stream));
  INIT_CHK(hipMemsetAsync(c->d_mask(), 0, sizeof(uint64_t) * MASK_WORDS * std::max(c->L.ntiles, c->L.max_segs),
                          c->stream));
  // first centre-of-mass pass on phi0, started from the given centres
  INIT_CHK(with_types(c->L.prec, [&](auto t, auto) {
    using T = decltype(t);
    return launch_cm_partials<T>(c->stream, 0, c->nlaunch(), c->d_tiles(), c->d_inst(), reinterpret_cast<T*>(c->pool()),
                                 c->d_drops(), c->d_part(), c->d_mask());
  }));
  INIT_CHK(launch_reduce(c->stream, TILING_SPLIT, c->L.ndrop_total, c->d_inst(), c->d_drops(), nullptr,
                         c->d_part(), c->d_mask(), c->d_step(), 0));
  INIT_CHK(hipStreamSynchronize(c->stream));
#undef INIT_CHK
  ReadBlocks::get().add_context();
  *out = c;
  g_err.clear();
  return LBM_OK;
}

int lbm_init(const lbm_config* cfg, void* workspace, size_t workspace_bytes, void* stream, const double* phi0,
             const double* c0, const double* f_pre, int32_t ndrop, const lbm_droplet* drops, int64_t step,
             lbm_ctx** out) {
  return lbm_init_batch(1, cfg, workspace, workspace_bytes, stream, phi0, c0, f_pre, &ndrop, drops, step, out);
}

int lbm_set_graph(lbm_ctx* c, int32_t steps_per_graph) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (steps_per_graph < 0 || (steps_per_graph > 0 && (steps_per_graph % 2 != 0 || steps_per_graph < 2)))
    return fail(LBM_E_INVAL, "steps_per_graph must be 0 or an even number >= 2");
  if (steps_per_graph > 0 && !c->stream) return fail(LBM_E_STATE, "graph replay needs a non-default stream");
  destroy_graphs(c);
  c->graph_steps = steps_per_graph;
  // capture the graphs now (one per starting parity), so that no later lbm_step pays for a capture
  c->long_graphs = false;
  for (int p = 0; p < 2 && steps_per_graph > 0; ++p) {
    const int rc = build_graph(c, p);
    if (rc != LBM_OK) return rc;
  }
  return LBM_OK;
}

int lbm_step(lbm_ctx* c, int64_t n) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (n < 0) return fail(LBM_E_INVAL, "n must be >= 0");
  if (c->lost) return fail_lost();
  Range range("lbm_step");
  int64_t left = n;
  if (c->graph_steps > 0) {
    const int64_t longer = (int64_t)c->graph_steps * LONG_GRAPH;
    const bool could = c->tiled() && c->long_graphs && left >= longer, use_long = could && c->long_asked;
    c->long_asked = c->long_asked || could;
    while (left >= c->graph_steps) {
      Range replay("lbm_step graph replay");
      const bool lg = use_long && left >= longer;
      const int which = c->parity + (lg ? 2 : 0);
      if (!c->exec[which]) {
        int rc = build_graph(c, which);
        if (rc != LBM_OK) return rc;
      }
      HIPCHK(hipGraphLaunch(c->exec[which], c->stream));
      left -= lg ? longer : c->graph_steps;
      c->step += lg ? longer : c->graph_steps;
    }
  }
  while (left > 0) {
    const int64_t n_now = std::min(left, SEQUENCE_MOST);
    int64_t done;
    const hipError_t e = enqueue_steps_any(c, c->parity, n_now, done);
    c->parity ^= (int)(done & 1);
    c->step += done;
    left -= n_now;
    if (e != hipSuccess) return fail(LBM_E_HIP, std::string("timestep launch: ") + hipGetErrorString(e));
  }
  return LBM_OK;
}

int lbm_sync(lbm_ctx* c) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  HIPCHK(hipStreamSynchronize(c->stream));
  return LBM_OK;
}

int64_t lbm_get_step(const lbm_ctx* c) { return c ? c->step : -1; }

int lbm_fields(lbm_ctx* c, int32_t inst, double* f_pre, double* phi, double* cc, double* n, double* ux, double* uy) {
  Range range("lbm_fields");
  int rc = check_inst(c, inst);
  if (rc != LBM_OK) return rc;
  bool finite = true;
  rc = with_types(c->L.prec, [&](auto t, auto p) {
    return fields_impl<decltype(t), decltype(p)>(c, inst, f_pre, phi, cc, n, ux, uy, finite);
  });
  if (rc != LBM_OK) return rc;
  // a non-finite state surfaces here as well as in lbm_observables (the arrays are filled regardless)
  return finite ? LBM_OK : fail(LBM_E_UNSTABLE, "non-finite values in the state");
}

int lbm_droplets(lbm_ctx* c, int32_t inst, lbm_droplet* out) {
  int rc = check_inst(c, inst);
  if (rc != LBM_OK) return rc;
  if (!out && c->L.inst[inst].ndrop > 0) return fail(LBM_E_INVAL, "out must not be NULL");
  std::vector<DropDev> dd;
  if ((rc = read_drops(c, inst, dd)) != LBM_OK) return rc;
  for (size_t k = 0; k < dd.size(); ++k)
    out[k] = lbm_droplet{dd[k].x, dd[k].y, dd[k].R, dd[k].Rs, dd[k].ex, dd[k].ey, dd[k].active, 0};
  return LBM_OK;
}

int lbm_observables(lbm_ctx* c, int32_t inst, lbm_obs* obs, double* drop_out) {
  Range range("lbm_observables");
  int rc = check_inst(c, inst);
  if (rc != LBM_OK) return rc;
  if (!obs) return fail(LBM_E_INVAL, "obs must not be NULL");
  const int nd = c->L.inst[inst].ndrop;
  ReadBuf buf(c);
  if ((rc = buf.take(sizeof(double) * (6 + 5 * (size_t)nd))) != LBM_OK) return rc;
  hipError_t e = with_types(c->L.prec, [&](auto t, auto p) {
    using T = decltype(t);
    return launch_obs<T, decltype(p)>(c->stream, c->parity, c->nlaunch(), c->d_tiles(), c->d_inst(),
                                      reinterpret_cast<const T*>(c->pool()), c->d_drops(), inst, c->d_obs(),
                                      c->L.obs_stride);
  });
  if (e == hipSuccess)
    e = launch_obs_final(c->stream, c->d_inst(), inst, nd, c->d_drops(), c->d_obs(), c->L.obs_stride,
                         reinterpret_cast<double*>(buf.fill()));
  if (e != hipSuccess) return fail(LBM_E_HIP, std::string("observables launch: ") + hipGetErrorString(e));
  if ((rc = buf.wait()) != LBM_OK) return rc;
  const double* const r = reinterpret_cast<const double*>(buf.data());
  obs->step = c->step;
  obs->mass = r[0];
  obs->sum_phi = r[1];
  obs->sum_c = r[2];
  obs->min_B = r[3];
  obs->max_u = r[4];
  obs->nonfinite = (r[5] != 0.0 || !std::isfinite(r[0]) || !std::isfinite(r[1]) || !std::isfinite(r[2])) ? 1 : 0;
  obs->ndrop = nd;
  if (drop_out) {
    for (int k = 0; k < nd; ++k) {
      const double* const d = r + 6 + 5 * k;  // x, y, sum phi, sum phi ux, sum phi uy
      drop_out[5 * k + 0] = d[0];
      drop_out[5 * k + 1] = d[1];
      drop_out[5 * k + 2] = d[2] > 0.0 ? d[3] / d[2] : 0.0;
      drop_out[5 * k + 3] = d[2] > 0.0 ? d[4] / d[2] : 0.0;
      drop_out[5 * k + 4] = d[2];
    }
  }
  if (obs->nonfinite) return fail(LBM_E_UNSTABLE, "non-finite values in the state");
  if (!(obs->min_B > 0.0)) return fail(LBM_E_UNSTABLE, "B(c) = B0 + B1 c <= 0 somewhere (interfaces unstable)");
  return LBM_OK;
}

int lbm_debug_stage(lbm_ctx* c, int32_t inst, double* out) {
  int rc = check_inst(c, inst);
  if (rc != LBM_OK) return rc;
  if (!out) return fail(LBM_E_INVAL, "out must not be NULL");
  const InstDev& d = c->L.inst[inst];
  if ((int64_t)d.nx * d.ny > DEBUG_MAX_NODES) return fail(LBM_E_INVAL, "stage export is limited to 512 x 512 nodes");
  hipError_t e = with_types(c->L.prec,
                            [&](auto t, auto p) { return debug_launch<decltype(t), decltype(p)>(c, inst, c->d_dbg()); });
  if (e != hipSuccess) return fail(LBM_E_HIP, std::string("stage launch: ") + hipGetErrorString(e));
  const size_t n = (size_t)d.nx * d.ny;
  HIPCHK(hipMemcpyAsync(out, c->d_dbg(), sizeof(double) * LBM_NSTAGE * n, hipMemcpyDeviceToHost, c->stream));
  HIPCHK(hipStreamSynchronize(c->stream));
  std::swap_ranges(out + PLANE_XH * n, out + (PLANE_XH + 1) * n, out + PLANE_M * n);
  return LBM_OK;
}

int lbm_time_kernels(lbm_ctx* c, int64_t n, double* ms_out) {
  Range range("lbm_time_kernels");
  if (!c || !ms_out) return fail(LBM_E_INVAL, "null argument");
  if (n <= 0) return fail(LBM_E_INVAL, "n must be > 0");
  std::vector<hipEvent_t> ev((size_t)n * 4);
  for (auto& x : ev) HIPCHK(hipEventCreate(&x));
  hipError_t e = hipSuccess;
  int nk = 0;
  for (int64_t s = 0; s < n && e == hipSuccess; ++s)
    e = with_types(c->L.prec,
                   [&](auto t, auto p) { return timed_step<decltype(t), decltype(p)>(c, &ev[(size_t)s * 4], &nk); });
  hipError_t es = hipStreamSynchronize(c->stream);
  double acc[3] = {0, 0, 0};
  if (e == hipSuccess && es == hipSuccess) {
    for (int64_t s = 0; s < n; ++s)
      for (int j = 0; j < nk; ++j) {
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, ev[(size_t)s * 4 + j], ev[(size_t)s * 4 + j + 1]);
        acc[j] += ms;
      }
  }
  for (auto& x : ev) (void)hipEventDestroy(x);
  if (e != hipSuccess) return fail(LBM_E_HIP, std::string("timed launch: ") + hipGetErrorString(e));
  if (es != hipSuccess) return fail(LBM_E_HIP, std::string("timed sync: ") + hipGetErrorString(es));
  for (int j = 0; j < 3; ++j) ms_out[j] = acc[j] / (double)n;
  return LBM_OK;
}

int lbm_time_launches(lbm_ctx* c, int32_t launches, double* ms_out) {
  Range range("lbm_time_launches");
  if (!c || !ms_out) return fail(LBM_E_INVAL, "null argument");
  if (launches <= 0) return fail(LBM_E_INVAL, "launches must be > 0");
  if (!c->stream) return fail(LBM_E_STATE, "timing launches in a graph needs a non-default stream");
  ms_out[0] = ms_out[1] = ms_out[2] = 0.0;
  const bool split = c->path == LBM_PATH_SPLIT;
  // kernel k of the path over the current state, writing scratch only; the last one is the centre-of-mass
  // reduction in its mode that writes nothing
  const int nk = split ? 3 : 2;
  auto one = [&](int k) -> hipError_t {
    if (k == nk - 1) return enqueue_reduce(c, 1, false);
    return with_types(c->L.prec, [&](auto t, auto p) -> hipError_t {
      using T = decltype(t);
      using P = decltype(p);
      T* buf = reinterpret_cast<T*>(c->pool());
      if (!split) return launch_sweep<T, P>(c, c->parity, nullptr, -1);
      if (k == 0) return launch_lb<T, P>(c->stream, 0, c->parity, c->nlaunch(), c->d_tiles(), c->d_inst(), buf, nullptr, -1);
      return launch_fd<T>(c->stream, 0, c->parity, c->nlaunch(), c->d_tiles(), c->d_inst(), buf, c->d_drops(),
                          c->d_part(), c->d_mask(), c->d_step(), nullptr, -1);
    });
  };
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  int rc = LBM_OK;
  for (int k = 0; k < nk && rc == LBM_OK; ++k) {
    // the launches are replayed from a graph, as lbm_step replays the timestep, so that no host launch gap
    // separates them
    hipGraph_t g = nullptr;
    hipGraphExec_t x = nullptr;
    hipError_t e = hipStreamBeginCapture(c->stream, hipStreamCaptureModeRelaxed);
    for (int r = 0; r < launches && e == hipSuccess; ++r) e = one(k);
    const hipError_t ec = hipStreamEndCapture(c->stream, &g);
    if (e == hipSuccess) e = ec;
    if (e == hipSuccess) e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
    if (e == hipSuccess) e = hipGraphLaunch(x, c->stream);  // warm-up replay
    if (e == hipSuccess) e = hipEventRecord(e0, c->stream);
    if (e == hipSuccess) e = hipGraphLaunch(x, c->stream);
    if (e == hipSuccess) e = hipEventRecord(e1, c->stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e != hipSuccess) rc = fail(LBM_E_HIP, std::string("timed launches: ") + hipGetErrorString(e));
    ms_out[k] = (double)ms / launches;
    if (x) (void)hipGraphExecDestroy(x);
    if (g) (void)hipGraphDestroy(g);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return rc;
}

int lbm_set_seg_rows(lbm_ctx* c, int32_t rows) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (rows < SEG_ROWS_MIN || rows > SEG_ROWS_MAX)
    return fail(LBM_E_INVAL, "segment height must lie in [" + std::to_string(SEG_ROWS_MIN) + ", " +
                                 std::to_string(SEG_ROWS_MAX) + "]");
  const int rc = apply_segments(c, rows, c->L.strip_w);
  if (rc == LBM_OK) c->tile = false;  // the caller asks for strips
  return rc;
}

int32_t lbm_get_seg_rows(const lbm_ctx* c) { return c ? c->L.seg_rows : -1; }

int lbm_set_strip_width(lbm_ctx* c, int32_t width) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (width < STRIP_W_MIN || width > FUSED_TX)
    return fail(LBM_E_INVAL, "strip width must lie in [" + std::to_string(STRIP_W_MIN) + ", " +
                                 std::to_string(FUSED_TX) + "]");
  const int rc = apply_segments(c, c->L.seg_rows, width);
  if (rc == LBM_OK) c->tile = false;
  return rc;
}

int lbm_debug_strips(lbm_ctx* c, int32_t rows) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (rows < SHORT_ROWS[0] || rows > SEG_ROWS_MAX)
    return fail(LBM_E_INVAL, "strips of " + std::to_string(SHORT_ROWS[0]) + " to " + std::to_string(SEG_ROWS_MAX) + " rows");
  const int rc = apply_segments(c, c->L.seg_rows, FUSED_TX, rows);
  if (rc == LBM_OK) c->tile = false;
  return rc;
}

int32_t lbm_get_strip_width(const lbm_ctx* c) { return c ? c->L.strip_w : -1; }

const int32_t* lbm_tune_widths(void) { return TUNE_WIDTHS; }

const int32_t* lbm_tune_rows(void) { return TUNE_ROWS; }

int lbm_autotune(lbm_ctx* c, int32_t launches, int32_t both_paths, int32_t* rows_out, int32_t* path_out,
                 double* ms_out) {
  Range range("lbm_autotune");
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (launches <= 0) return fail(LBM_E_INVAL, "launches must be > 0");
  constexpr int NR = LBM_TUNE_NROWS, NW = LBM_TUNE_NWIDTHS;
  if (ms_out)
    for (int k = 0; k < 2 * NW * NR + 1; ++k) ms_out[k] = -1.0;
  if (c->path == LBM_PATH_SPLIT && !both_paths) {
    if (rows_out) *rows_out = c->L.seg_rows;
    if (path_out) *path_out = c->path;
    return LBM_OK;
  }
  const int paths[2] = {LBM_PATH_FUSED, LBM_PATH_WAVE};
  const int start_path = c->path;
  const bool start_tile = c->tile;
  c->tile = false;  // the strips first; the tiled kernel is tried after them
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  int best_rows = c->L.seg_rows, best_path = c->path, best_w = c->L.strip_w;
  double best_ms = 1e300;
  int rc = LBM_OK;
  std::vector<double> cand_ms(2 * NW * NR, 1e300);
  // Heights that give the same number of strip segments as an earlier candidate are skipped.
  std::vector<bool> skip(NR, false);
  std::vector<int64_t> seen;
  auto tried = [&](int rows) {
    int64_t nseg = 0;
    for (const auto& d : c->L.inst) nseg += (d.ny + rows - 1) / rows;
    if (std::find(seen.begin(), seen.end(), nseg) != seen.end()) return true;
    seen.push_back(nseg);
    return false;
  };
  for (int k = 0; k < NR; ++k) skip[k] = tried(TUNE_ROWS[k]);
  // Trial launches read the current state and write only the inactive half of every ping-pong buffer
  // and the partials; the parity, the droplet table and the step counter are untouched.  Launches of
  // one candidate run back to back; two passes over the candidates (the first also warms clocks and
  // caches), keeping each candidate's faster pass.  The second leaves out those that took more than 1.5 times the
  // first pass's best, a third to two thirds of them: the first pass was at most 8 % slower than the second for any
  // candidate (1024 x 1024 FP64 and FP32, 32 lattices in FP32).  Whole call, ms, both passes of all / without those:
  // 106 / 72, 89 / 57, 88 / 67.
  auto trial = [&](int n) -> hipError_t {
    hipError_t e = hipSuccess;
    for (int rep = 0; rep < n && e == hipSuccess; ++rep)
      e = with_types(c->L.prec,
                     [&](auto t, auto p) { return launch_sweep<decltype(t), decltype(p)>(c, c->parity, nullptr, -1); });
    return e;
  };
  for (int pass = 0; pass < 2 && rc == LBM_OK; ++pass) {
    const double limit = 1.5 * *std::min_element(cand_ms.begin(), cand_ms.end());
    for (int pi = 0; pi < 2 && rc == LBM_OK; ++pi) {
      if (!both_paths && paths[pi] != start_path) continue;
      c->path = paths[pi];
      for (int wi = 0; wi < NW && rc == LBM_OK; ++wi)
        for (int k = 0; k < NR; ++k) {
          if (skip[k]) continue;
          if (cand_ms[(pi * NW + wi) * NR + k] > limit && pass > 0) continue;
          if ((rc = apply_segments(c, TUNE_ROWS[k], TUNE_WIDTHS[wi])) != LBM_OK) break;
          hipError_t e = trial(1);
          (void)hipEventRecord(e0, c->stream);
          if (e == hipSuccess) e = trial(launches);
          (void)hipEventRecord(e1, c->stream);
          if (e == hipSuccess) e = hipEventSynchronize(e1);
          if (e != hipSuccess) {
            rc = fail(LBM_E_HIP, std::string("autotune launch: ") + hipGetErrorString(e));
            break;
          }
          float ms = 0.f;
          (void)hipEventElapsedTime(&ms, e0, e1);
          double& m = cand_ms[(pi * NW + wi) * NR + k];
          m = std::min(m, (double)ms / launches);
        }
    }
  }
  for (int pi = 0; pi < 2; ++pi)
    for (int wi = 0; wi < NW; ++wi)
      for (int k = 0; k < NR; ++k) {
        const double m = cand_ms[(pi * NW + wi) * NR + k];
        if (ms_out && m < 1e299) ms_out[(pi * NW + wi) * NR + k] = m;
        if (m < best_ms) {
          best_ms = m;
          best_rows = TUNE_ROWS[k];
          best_w = TUNE_WIDTHS[wi];
          best_path = paths[pi];
        }
      }
  // shorter strips, the split path (two tile kernels) and the tiled fused step, which have no entry among the heights,
  // compete with the best strips, each in a second pass too unless the first was as far behind as above
  auto compete = [&](auto one, double& ms_best) -> int {
    for (int pass = 0; pass < 2; ++pass) {
      if (pass > 0 && ms_best > 1.5 * best_ms) break;
      hipError_t e = one();
      (void)hipEventRecord(e0, c->stream);
      for (int rep = 0; rep < launches && e == hipSuccess; ++rep) e = one();
      (void)hipEventRecord(e1, c->stream);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      if (e != hipSuccess) return fail(LBM_E_HIP, std::string("autotune launch: ") + hipGetErrorString(e));
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      ms_best = std::min(ms_best, (double)ms / launches);
    }
    return LBM_OK;
  };
  int best_short = 0;
  int64_t strips = 0;
  for (const InstDev& d : c->L.inst) strips += strip_count(d.nx, d.ny, FUSED_TX, SEG_ROWS_MIN);
  std::vector<int> heights;  // 16 x 16: whole call 1.1 ms without the short ones, 3.6 with all of them, 1.4 with the one new
  for (int h : SHORT_ROWS)
    if (strips <= SHORT_MOST && c->L.tshape < 0 && !tried(h)) heights.push_back(h);
  for (int pi = 0; pi < 2; ++pi) {
    if (!both_paths && paths[pi] != start_path) continue;
    c->path = paths[pi];
    for (int h : heights) {
      double ms = 1e300;
      if (rc == LBM_OK) rc = apply_segments(c, best_rows, FUSED_TX, h);
      if (rc == LBM_OK) rc = compete([&] { return trial(1); }, ms);
      if (ms < best_ms) {
        best_ms = ms;
        best_short = h;
        best_w = FUSED_TX;
        best_path = paths[pi];
      }
    }
  }
  bool best_tile = false;
  if (both_paths && rc == LBM_OK) {
    c->path = LBM_PATH_SPLIT;
    double split_ms = 1e300;
    rc = compete(
        [&] {
          return with_types(c->L.prec,
                            [&](auto t, auto p) { return launch_split<decltype(t), decltype(p)>(c, c->parity); });
        },
        split_ms);
    if (ms_out && split_ms < 1e299) ms_out[2 * NW * NR] = split_ms;
    if (split_ms < best_ms) {
      best_ms = split_ms;
      best_path = LBM_PATH_SPLIT;
    }
  }
  if (c->L.tshape >= 0 && (both_paths || start_path == LBM_PATH_FUSED) && rc == LBM_OK) {
    c->path = LBM_PATH_FUSED;
    c->tile = true;
    double tile_ms = 1e300;
    rc = compete([&] { return trial(1); }, tile_ms);
    if (tile_ms < best_ms) {
      best_ms = tile_ms;
      best_path = LBM_PATH_FUSED;
      best_tile = true;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  c->path = start_path;
  c->tile = start_tile;
  if (rc != LBM_OK) return rc;
  if ((rc = lbm_set_path(c, best_path)) != LBM_OK) return rc;
  if (best_path == LBM_PATH_FUSED) c->tile = best_tile;
  if ((rc = apply_segments(c, best_rows, best_w, best_path == LBM_PATH_SPLIT || best_tile ? 0 : best_short)) != LBM_OK)
    return rc;
  if (rows_out) *rows_out = best_rows;
  if (path_out) *path_out = best_path;
  return LBM_OK;
}

const char* lbm_kernel_name(int32_t path, int32_t which) {
  static const char* fused[3] = {"k_step", "k_reduce", ""};
  static const char* split[3] = {"k_lb", "k_fd", "k_reduce"};
  static const char* wave[3] = {"k_wave", "k_reduce", ""};
  if (which < 0 || which > 2) return "";
  return path == LBM_PATH_SPLIT ? split[which] : path == LBM_PATH_WAVE ? wave[which] : fused[which];
}

int lbm_set_path(lbm_ctx* c, int32_t path) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (path != LBM_PATH_FUSED && path != LBM_PATH_SPLIT && path != LBM_PATH_WAVE)
    return fail(LBM_E_INVAL, "unknown path");
  if (path != c->path) destroy_graphs(c);
  c->path = path;
  return LBM_OK;
}

int32_t lbm_get_path(const lbm_ctx* c) { return c ? c->path : -1; }

void lbm_destroy(lbm_ctx* c) {
  if (!c) return;
  destroy_graphs(c);
  delete c;
  ReadBlocks::get().drop_context();
}

const char* lbm_running_kernel(const lbm_ctx* c, int32_t which) {
  if (!c) return "";
  if (c->tiled()) return which == 0 ? "k_tile" : which == 1 ? "k_tile_final" : "";
  return lbm_kernel_name(c->path, which);
}

int32_t lbm_running_rows(const lbm_ctx* c) {
  return !c ? -1 : c->path == LBM_PATH_SPLIT || c->tiled() ? 0 : c->L.inst[0].seg_rows;
}

const char* lbm_last_error(void) { return g_err.c_str(); }

}  // extern "C"

// ------------------------------------------------------------------------------------------------
// Reverse mode: checkpointed forward pass and backward sweep of the adjoint kernels.
namespace {

struct AdjLayout {
  size_t pop = 0, field = 0, dropb = 0;  // bytes of the parts of a saved state
  size_t slot = 0;   // a whole state: populations, phi, c, droplet table, step counter
  size_t sslot = 0;  // what the adjoint step reads of a recomputed state: phi, c, droplet table, tiled steps' centres
  int64_t ncp = 0, nodes = 0;
  int every = 0, nparts = 0;  // nparts: running totals of dA0
  size_t off_cp = 0, off_seg = 0, off_final = 0, off_fwd = 0, off_adj = 0, off_part = 0, off_inst = 0, total = 0;
};

constexpr int ADJ_TMP_PLANES = 4;  // intermediate adjoints of one backward step
// The adjoint step reads ADJ_FWD_PLANES stage planes of the forward step, and the recompute exports only those: the
// record of an interval holds ADJ_FWD_PLANES planes per step.
constexpr int ADJ_FWD_PLANES = ADJ_EXPORT_PLANES;

// Up to five byte ranges (multiples of 8 bytes) copied by one launch.
struct CopyList {
  const uint64_t* src[5];
  uint64_t* dst[5];
  int64_t n[5];  // 8-byte words
  int nseg;
};

__global__ void __launch_bounds__(256) k_copy_list(CopyList L) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int s = 0; s < L.nseg; ++s)
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < L.n[s]; i += stride)
      L.dst[s][i] = L.src[s][i];
}

struct CopyBuilder {
  CopyList L{};
  int64_t most = 0;
  void add(const void* src, void* dst, size_t bytes) {
    L.src[L.nseg] = static_cast<const uint64_t*>(src);
    L.dst[L.nseg] = static_cast<uint64_t*>(dst);
    L.n[L.nseg] = (int64_t)(bytes / 8);
    most = std::max(most, L.n[L.nseg]);
    ++L.nseg;
  }
  hipError_t launch(hipStream_t s) const {
    const int blocks = (int)std::min<int64_t>(std::max<int64_t>((most + 255) / 256, 1), 2048);
    hipLaunchKernelGGL(k_copy_list, dim3(blocks), dim3(256), 0, s, L);
    return hipGetLastError();
  }
};

int adj_check(const lbm_ctx* c, int32_t drop, int64_t nsteps, int32_t every) {
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (c->L.inst.size() != 1) return fail(LBM_E_INVAL, "the adjoint takes a context of one lattice");
  const lbm_config& g = c->cfg[0];
  if (g.precision != LBM_FP64 && g.precision != LBM_FP32)
    return fail(LBM_E_INVAL, "the adjoint runs in LBM_FP64 or LBM_FP32");
  if (g.advection != LBM_ADV_PAPER) return fail(LBM_E_INVAL, "the adjoint is implemented for LBM_ADV_PAPER");
  if (drop < 0 || drop >= c->L.inst[0].ndrop) return fail(LBM_E_INVAL, "droplet index out of range");
  if (nsteps < 1 || every < 1) return fail(LBM_E_INVAL, "nsteps and checkpoint interval must be >= 1");
  return LBM_OK;
}

AdjLayout adj_layout(const lbm_ctx* c, int64_t nsteps, int every) {
  AdjLayout A;
  const InstDev& d = c->L.inst[0];
  A.nodes = (int64_t)d.nx * d.ny;
  A.nparts = adj_parts(d.nx, d.ny);
  A.every = every;
  A.ncp = (nsteps + every - 1) / every;
  A.pop = (size_t)9 * d.pstride * c->L.elem;
  A.field = (size_t)d.pstride * c->L.elem;
  A.dropb = sizeof(DropDev) * (size_t)std::max(1, (int)d.ndrop);
  A.slot = align_up(A.pop + 2 * A.field + A.dropb + sizeof(int64_t), ALIGN);
  A.sslot = align_up(2 * A.field + A.dropb + sizeof(double) * 2 * (size_t)d.ndrop, ALIGN);
  size_t off = 0;
  A.off_cp = off;    off += A.slot * (size_t)A.ncp;
  A.off_seg = off;   off += A.sslot * ((size_t)every + 1);
  A.off_final = off; off += A.slot;
  A.off_fwd = off;
  off = align_up(off + sizeof(double) * ADJ_FWD_PLANES * (size_t)every * (size_t)A.nodes, ALIGN);
  A.off_adj = off;   off = align_up(off + c->L.elem * (size_t)(22 + ADJ_TMP_PLANES) * A.nodes, ALIGN);
  A.off_part = off;
  off = align_up(off + sizeof(double) * (1 + (size_t)std::max(A.nparts, adj_blocks(d.nx, d.ny))), ALIGN);
  A.off_inst = off;  off = align_up(off + sizeof(InstDev) * (size_t)every, ALIGN);
  A.total = off + ALIGN;  // the caller's pointer need not be aligned, see adj_base
  return A;
}

// The first aligned byte of a workspace.  The recompute's descriptions count its planes in elements from the context's
// pool, which needs a whole number of them between the two.
char* adj_base(void* ws) {
  return reinterpret_cast<char*>(align_up(reinterpret_cast<uintptr_t>(ws), ALIGN));
}

// Copy the state of the single lattice (current buffers, droplet table, step counter) to or from a whole
// slot, in one launch.
int adj_save(lbm_ctx* c, const AdjLayout& A, char* slot) {
  const InstDev& d = c->L.inst[0];
  char* pool = static_cast<char*>(c->pool());
  const size_t e = c->L.elem;
  CopyBuilder b;
  b.add(pool + d.off_f[c->parity] * e, slot, A.pop);
  b.add(pool + d.off_phi[c->parity] * e, slot + A.pop, A.field);
  b.add(pool + d.off_c[c->parity] * e, slot + A.pop + A.field, A.field);
  b.add(c->d_drops(), slot + A.pop + 2 * A.field, sizeof(DropDev) * d.ndrop);
  b.add(c->d_step(), slot + A.pop + 2 * A.field + A.dropb, sizeof(int64_t));
  HIPCHK(b.launch(c->stream));
  return LBM_OK;
}

// A whole slot back into the current buffers, or (sslot not null) its phi and c into a segment slot and only the
// populations into the current buffers.  The droplet table goes to the context, or to the segment slot.
int adj_load(lbm_ctx* c, const AdjLayout& A, const char* slot, int64_t step, char* sslot) {
  const InstDev& d = c->L.inst[0];
  char* pool = static_cast<char*>(c->pool());
  const size_t e = c->L.elem;
  CopyBuilder b;
  b.add(slot, pool + d.off_f[c->parity] * e, A.pop);
  b.add(slot + A.pop, sslot ? sslot : pool + d.off_phi[c->parity] * e, A.field);
  b.add(slot + A.pop + A.field, sslot ? sslot + A.field : pool + d.off_c[c->parity] * e, A.field);
  b.add(slot + A.pop + 2 * A.field, sslot ? sslot + 2 * A.field : reinterpret_cast<char*>(c->d_drops()),
        sizeof(DropDev) * d.ndrop);
  b.add(slot + A.pop + 2 * A.field + A.dropb, c->d_step(), sizeof(int64_t));
  HIPCHK(b.launch(c->stream));
  c->step = step;
  return LBM_OK;
}

DropDev* adj_seg_drops(const AdjLayout& A, char* sslot) { return reinterpret_cast<DropDev*>(sslot + 2 * A.field); }
double* adj_seg_centres(const AdjLayout& A, char* sslot) {
  return reinterpret_cast<double*>(sslot + 2 * A.field + A.dropb);
}

// Description of the lattice for recomputed step j of an interval (of parity j & 1): phi and c are read from segment
// slot j and written to slot j + 1, so that the record of an interval needs no copies.  The populations alternate
// between the context's own buffers.
InstDev adj_inst(const InstDev& d, int64_t seg, int64_t sslot, int64_t field, int64_t j) {
  InstDev v = d;
  const int in = (int)(j & 1);
  v.off_phi[in] = seg + j * sslot;
  v.off_phi[in ^ 1] = seg + (j + 1) * sslot;
  v.off_c[in] = seg + j * sslot + field;
  v.off_c[in ^ 1] = seg + (j + 1) * sslot + field;
  return v;
}

template <typename T>
int adj_backward(lbm_ctx* c, const AdjLayout& A, char* w, double* dA0, double* dc0) {
  const InstDev& d = c->L.inst[0];
  const lbm_config& g = c->cfg[0];
  const int64_t n0 = c->adj.n0, N = c->adj.nsteps, M = A.nodes;
  const int every = c->adj.every, drop = c->adj.drop, nd = d.ndrop;
  int rc;
  ReadBuf buf(c);  // the seed's sum of phi, dA0
  if ((rc = buf.take(2 * sizeof(double))) != LBM_OK) return rc;
  if ((rc = adj_save(c, A, w + A.off_final)) != LBM_OK) return rc;
  const int parity = c->parity;  // of the final state, which comes back at the end
  char* const segs = w + A.off_seg;
  // the descriptions of an interval's steps, in elements from the pool
  const int64_t e = (int64_t)c->L.elem;
  const int64_t seg0 = (segs - static_cast<char*>(c->pool())) / e, sslot = (int64_t)A.sslot / e;
  const int64_t field = (int64_t)A.field / e;
  InstDev* const d_insts = reinterpret_cast<InstDev*>(w + A.off_inst);
  if (!c->tiled()) {
    std::vector<InstDev> h((size_t)every);
    for (int j = 0; j < every; ++j) h[j] = adj_inst(d, seg0, sslot, field, j);
    HIPCHK(hipMemcpyAsync(d_insts, h.data(), sizeof(InstDev) * h.size(), hipMemcpyHostToDevice, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
  }
  // stage planes of step k0 + j of the current interval start ADJ_FWD_PLANES * j planes into the record
  double* fwd = reinterpret_cast<double*>(w + A.off_fwd);
  auto fwd_rec = [&](int64_t j) { return fwd + (size_t)ADJ_FWD_PLANES * (size_t)j * (size_t)M; };
  auto fwd_at = [&](int64_t j) {
    const double* f = fwd_rec(j);
    return AdjFwd{f + 0 * M, f + 1 * M, f + 2 * M, f + 3 * M, f + 4 * M,
                  f + 5 * M, f + 6 * M, f + 7 * M, f + 8 * M, f + 9 * M};
  };
  T* adj = reinterpret_cast<T*>(w + A.off_adj);
  T* lam[2] = {adj, adj + 11 * M};  // adjoint state (f 9 planes, phi, c) at n and at n + 1
  T* tmp = adj + 22 * M;
  double* const sw = reinterpret_cast<double*>(w + A.off_part);  // the seed's sum of phi
  double* const part = sw + 1;                                   // its partial sums, then per-block dA0 totals
  AdjModel m;
  m.nx = d.nx;
  m.ny = d.ny;
  m.a = g.a;
  m.b = g.b;
  m.B0 = g.B0;
  m.B1 = g.B1;
  m.D = g.D;
  m.Gamma = g.Gamma;
  m.gamma = g.gamma;
  m.omega = d.omega;
  m.coef = d.coef;
  m.yper = d.yper;
  m.walls = d.walls;
  m.ramp = 0.0;
  auto planes = [&](const char* sslot, T* in, T* out) {
    AdjPlanes<T> p;
    p.phi = reinterpret_cast<const T*>(sslot);
    p.c = reinterpret_cast<const T*>(sslot + A.field);
    p.pitch = d.pitch;
    p.fb1 = in;
    p.pb1 = in + 9 * M;
    p.cb1 = in + 10 * M;
    p.fb = out;
    p.pb = out + 9 * M;
    p.cb = out + 10 * M;
    T** t[] = {&p.phb, &p.chb, &p.Fxb, &p.Fyb};
    static_assert(sizeof(t) / sizeof(t[0]) == ADJ_TMP_PLANES, "temporary planes");
    for (int i = 0; i < ADJ_TMP_PLANES; ++i) *t[i] = tmp + (size_t)i * M;
    return p;
  };
  auto slot_of = [&](int64_t j) { return segs + (size_t)j * A.sslot; };
  // the droplets at step j of the interval: tiled steps leave the centres alone, the others a table
  static_assert(sizeof(DropDev) % sizeof(double) == 0, "centres of a table as an array of doubles");
  auto drops_at = [&](int64_t j) {
    if (c->tiled()) return AdjDrops{adj_seg_drops(A, segs), adj_seg_centres(A, slot_of(j)), 2, nd};
    DropDev* const t = adj_seg_drops(A, slot_of(j));
    return AdjDrops{t, &t->x, (int)(sizeof(DropDev) / sizeof(double)), nd};
  };
  const int dbg_inst = export_planes(0, false);
  int cur = 1;  // lam[cur] holds the adjoint of the latest state
  for (int64_t s = A.ncp - 1; s >= 0; --s) {
    const int64_t k0 = s * every, k1 = std::min<int64_t>(N, k0 + every);
    // recompute the interval from its checkpoint: phi, c, the droplets and the stage planes of every step stay in the
    // interval's record.  The export launch is a whole step but for the centres.
    c->parity = 0;
    if ((rc = adj_load(c, A, w + A.off_cp + (size_t)s * A.slot, n0 + k0, segs)) != LBM_OK) return rc;
    for (int64_t j = 0; j < k1 - k0; ++j) {
      DropDev* const table = adj_seg_drops(A, slot_of(j));
      const int par = (int)(j & 1);
      if (c->tiled()) {
        TileSeq q = c->tile_seq(j);
        if (j > 0) q.cen_in = adj_seg_centres(A, slot_of(j - 1));
        q.cen_out = adj_seg_centres(A, slot_of(j));
        const InstDev one = adj_inst(d, seg0, sslot, field, j);
        HIPCHK((launch_sweep_on<T, T>(c, par, nullptr, &one, adj_seg_drops(A, segs), q, fwd_rec(j), dbg_inst)));
        continue;
      }
      if (c->path == LBM_PATH_SPLIT)
        HIPCHK((launch_split_export<T, T>(c, par, d_insts + j, table, fwd_rec(j), dbg_inst)));
      else
        HIPCHK((launch_sweep_on<T, T>(c, par, d_insts + j, nullptr, table, TileSeq{}, fwd_rec(j), dbg_inst)));
      HIPCHK(launch_reduce(c->stream, c->path == LBM_PATH_SPLIT ? TILING_SPLIT : TILING_FUSED, nd, d_insts + j, table,
                           adj_seg_drops(A, slot_of(j + 1)), c->d_part(), c->d_mask(), c->d_step(), 1));
    }
    // loss x_CM^N - x_CM^{n0}: seed d/d phi^N over the droplet's nodes (centres of step N - 1)
    if (s == A.ncp - 1)
      HIPCHK(launch_adjoint_seed<T>(c->stream, m, reinterpret_cast<const T*>(slot_of(k1 - k0)), d.pitch,
                                    drops_at(k1 - k0 - 1),
                                    reinterpret_cast<const DropDev*>(w + A.off_final + A.pop + 2 * A.field), drop,
                                    lam[cur], lam[cur] + 9 * M, lam[cur] + 10 * M, part, sw));
    // backward through the segment, latest step first
    for (int64_t k = k1 - 1; k >= k0; --k) {
      const double tn = (double)(n0 + k);
      m.ramp = tn < g.t_star ? tn : g.t_star;
      const AdjPlanes<T> p = planes(slot_of(k - k0), lam[cur], lam[cur ^ 1]);
      HIPCHK(launch_adjoint_step<T>(c->stream, m, fwd_at(k - k0), p, drops_at(k - k0), part));
      cur ^= 1;
    }
  }
  double* const result = reinterpret_cast<double*>(buf.fill());
  HIPCHK(hipMemcpyAsync(result, sw, sizeof(double), hipMemcpyDeviceToHost, c->stream));
  HIPCHK(launch_adjoint_total(c->stream, part, A.nparts, result + 1));
  // back to the state at the end of the forward pass
  c->parity = parity;
  if ((rc = adj_load(c, A, w + A.off_final, n0 + N, nullptr)) != LBM_OK) return rc;
  if ((rc = buf.wait()) != LBM_OK) return rc;
  if (!(result[0] > 0.0)) return fail(LBM_E_STATE, "the droplet has no nodes with phi >= 0 at the end of the run");
  if (dA0) *dA0 = result[1];
  if (!dc0) return LBM_OK;
  bool finite;
  const T* const cb = lam[cur] + 10 * M;
  return read_planes(c, M, 1, &dc0, finite, [&](int64_t first, int64_t count, double* v, uint32_t*) {
    return launch_widen<T>(c->stream, cb + first, count, v);
  });
}

}  // namespace

extern "C" {

int lbm_adjoint_bytes(const lbm_ctx* c, int64_t nsteps, int32_t every, size_t* bytes) {
  if (!c || !bytes) return fail(LBM_E_INVAL, "null argument");
  if (nsteps < 1 || every < 1) return fail(LBM_E_INVAL, "nsteps and checkpoint interval must be >= 1");
  if (c->L.inst.size() != 1) return fail(LBM_E_INVAL, "the adjoint takes a context of one lattice");
  *bytes = adj_layout(c, nsteps, every).total;
  return LBM_OK;
}

int lbm_adjoint_forward(lbm_ctx* c, void* ws, size_t bytes, int32_t drop, int64_t nsteps, int32_t every,
                        double* J) {
  Range range("lbm_adjoint_forward");
  int rc = adj_check(c, drop, nsteps, every);
  if (rc != LBM_OK) return rc;
  if (!ws) return fail(LBM_E_INVAL, "adjoint workspace must not be NULL");
  const AdjLayout A = adj_layout(c, nsteps, every);
  if (bytes < A.total) return fail(LBM_E_NOMEM, "adjoint workspace too small (see lbm_adjoint_bytes)");
  char* w = adj_base(ws);
  const InstDev& d = c->L.inst[0];
  ReadBuf buf(c);  // x of the droplet before and after
  if ((rc = buf.take(2 * sizeof(double))) != LBM_OK) return rc;
  auto read_x = [&](int i) {
    return hipMemcpyAsync(buf.fill() + i * sizeof(double), &(c->d_drops() + drop)->x, sizeof(double),
                          hipMemcpyDeviceToHost, c->stream);
  };
  HIPCHK(read_x(0));
  c->adj.valid = false;
  c->adj.n0 = c->step;
  c->adj.nsteps = nsteps;
  c->adj.every = every;
  c->adj.drop = drop;
  for (int64_t k = 0; k < nsteps; k += every) {
    if ((rc = adj_save(c, A, w + A.off_cp + (size_t)(k / every) * A.slot)) != LBM_OK) return rc;
    if ((rc = lbm_step(c, std::min<int64_t>(every, nsteps - k))) != LBM_OK) return rc;
  }
  HIPCHK(read_x(1));
  if ((rc = buf.wait()) != LBM_OK) return rc;
  const double* const at = reinterpret_cast<const double*>(buf.data());
  double dx = at[1] - at[0];
  if (dx >= 0.5 * d.nx) dx -= d.nx;
  if (dx < -0.5 * d.nx) dx += d.nx;
  if (J) *J = dx;
  c->adj.valid = true;
  return LBM_OK;
}

int lbm_adjoint_backward(lbm_ctx* c, void* ws, size_t bytes, double* dJ_dA0, double* dJ_dc0) {
  Range range("lbm_adjoint_backward");
  if (!c) return fail(LBM_E_INVAL, "null context");
  if (!c->adj.valid) return fail(LBM_E_STATE, "no forward pass recorded (lbm_adjoint_forward)");
  if (c->step != c->adj.n0 + c->adj.nsteps)
    return fail(LBM_E_STATE, "the context has moved since the recorded forward pass");
  if (!ws) return fail(LBM_E_INVAL, "adjoint workspace must not be NULL");
  const AdjLayout A = adj_layout(c, c->adj.nsteps, c->adj.every);
  if (bytes < A.total) return fail(LBM_E_NOMEM, "adjoint workspace too small (see lbm_adjoint_bytes)");
  char* w = adj_base(ws);
  return c->L.prec == LBM_FP64 ? adj_backward<double>(c, A, w, dJ_dA0, dJ_dc0)
                               : adj_backward<float>(c, A, w, dJ_dA0, dJ_dc0);
}

}  // extern "C"
