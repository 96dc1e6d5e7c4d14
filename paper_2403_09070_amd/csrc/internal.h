// Internal declarations shared by the HIP sources of libplace3d (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/place3d.h"

namespace p3d {

constexpr int kWave = 64;
constexpr int kMaxNz = 16;
constexpr int kNumXcd = 8;              // accelerator dies; workgroups go to them round-robin
constexpr int kWaBlock = 256;           // threads per wirelength block
constexpr int kPinsPerLane = 4;         // net pins a wirelength lane keeps in registers
constexpr int kNumGroups = 7;           // nets by lane group: 1, 2, 4, ..., 64 lanes
constexpr int kNumClasses = kNumGroups + 1;   // the groups, then two-pin nets (one lane each)
constexpr int kChunkGroup = 16;         // chunks of a tile whose density sums one workgroup adds

// Splits of heavy tiles: a tile of more (cell, tile) entries than `from` and than most = max(min,
// entries / count) is split into chunks of at most `most`, which leaves at most count chunks beside
// the tiles' first ones.  The gathers' chunks are independent, so that they are split as far as a
// workgroup's staging of the maps allows (min of 16384, 2048, 1024: adjoint of 320k cells on 64 tiles
// 62, 34, 23 us; gather of 200k cells on 256 tiles 28.6, 19.8, 16.1; 1.2M cells on four tiles with
// count of 256, 512, 1024: 72, 51, 46); the field gather takes a tile's chunks as one again where that
// costs it more than it gives (gather_chunks).  The density chunks' sums have to meet, 0.1 us of fence each
// beside their bytes: tiles that would make two chunks are faster whole (64 of 5500 entries 25 us,
// in two 27, in four 30), full ones in many (1.2M cells on four tiles: 165 us in 80 chunks, 86 in 160,
// 72 in 256, 83 in 512).
enum SplitKind { kSplitDensity = 0, kSplitGather = 1, kSplits = 2 };
struct SplitBound { int from, min, count; };
constexpr SplitBound kSplit[kSplits] = {{8192, 4096, 256}, {1024, 1024, 1024}};

// Reduction slots (float64, device) inside the workspace.
enum RedSlot {
  R_WA_BI = 0, R_WA_Z, R_HPWL, R_HPWL3D, R_NCUT, R_NORM_X, R_NORM_Y, R_NORM_FDA,
  R_DV2, R_DG2, R_Q_BOT, R_Q_TOP, R_EXCESS_BOT, R_EXCESS_TOP, R_ENERGY,
  R_L1_WL, R_L1_DEN, R_GMAX, R_NONFINITE, R_A_PREV,
  R_COUNT = 32
};


struct ClassTab {       // net schedule in layout order: position i < kNumGroups holds groups of
                        // 2^(kNumGroups-1-i) lanes, the last position the two-pin nets
  int32_t net_begin[kNumClasses + 1];
  int32_t block_begin[kNumClasses + 1];
};

// instance classes for the density path
constexpr uint8_t kClsCell = 0;    // movable cell bucketed by tile
constexpr uint8_t kClsLarge = 1;   // movable macro or oversized cell: swept bin-parallel
constexpr uint8_t kClsFixed = 2;   // fixed: part of the constant map

struct TileGeom {       // map tiles owned by one workgroup each, and the bucketing partition
  int T, lgT, ntx, nty, ntiles;   // T = 2^lgT bins per tile side
  int cpb, nblk;        // cells per bucket block, bucket blocks
};

struct Geom {
  int n, nx, ny, nz;
  float dx, dy, dz, wb, hb, db, inv_wb, inv_hb, inv_db, half_dz, vol_bin;
  double wbd, hbd;      // bin sizes in float64: bin origins b * size are formed in float64, so
                        // that a size that float32 cannot hold does not shift far bins' edges
};

struct DctBases {
  // float32 [N][N] row-major, see spectral.hip for the definition of each matrix
  float *Fx, *Gx, *Hx;      // x: forward (sample, freq), inverse cos (freq, sample), inverse sin*omega
  float *FyT, *Gy, *Hy;     // y: forward^T (freq, sample), inverse cos (sample, freq), inverse sin*omega
  // bfloat16 hi/lo splits, k contiguous: x bases transposed to [N][K], y bases as stored
  uint16_t *Fx_h, *Fx_l, *Gx_h, *Gx_l, *Hx_h, *Hx_l;
  uint16_t *FyT_h, *FyT_l, *Gy_h, *Gy_l, *Hy_h, *Hy_l;
  float* zmat;              // small z matrices, see spectral.hip
  int fold = 0;             // even x and y: folded contractions, spectra in even-first order
  float* inv_w2;            // [Nz][Ny][Nx] 1/|omega|^2 with the (0,0,0) entry 0
};

// hi / lo bfloat16 planes of one split operand
struct HL { uint16_t* h = nullptr; uint16_t* l = nullptr; };

// Split-bfloat16 chain of the folded solve (even x and y, Nz of 2 or 4): every contraction
// operand lives in HBM as hi / lo planes whose rows are k-contiguous, padded with zeros to a
// multiple of 32, so that the contractions stream both operands straight into LDS.  hx, hy are
// the axis halves, rx, ry their padded widths.
struct SplitChain {
  int on = 0;
  int hx = 0, hy = 0, rx = 0, ry = 0;
  HL fx[2];              // forward x, even / odd frequencies: [hx][rx], row = frequency, k = x
  HL fy[2];              // forward y: [hy][ry], row = frequency, k = y
  HL gy, hy_s;           // inverse y (cosine, sine): [hy][2 ry], row = y, k = even then odd frequencies
  HL gx, hx_s;           // inverse x: [hx][2 rx], row = x, k = even then odd frequencies
  HL xs[2];              // x-folded map (sum, difference): [Nz Ny][rx]
  HL ys[2];              // y-folded x spectra (sum, difference): [Nz Nx][ry], row = (z, x frequency)
  HL bb;                 // potential coefficients: [Nx Nz][2 ry], row = x frequency * Nz + z frequency
  HL vg, vh;             // inverse-y results (cosine, sine basis): [Nz Ny][2 rx], row = (z frequency, y)
};

// Fast transforms of the solve (fft_grid in context.cpp): tables per axis, the stages'
// twiddles (at most kFftTable N entries) and e^{-i pi k / 2N} (k <= N / 2), and the means of the rows in
// hand ([nz][ny / 2], a call's scratch).  The dense bases and the split chain are then built only where a
// step takes them (step_dense).
constexpr int kFftTable = 2;
struct FftChain {
  int on = 0;
  float2 *tx = nullptr, *wx = nullptr, *ty = nullptr, *wy = nullptr;
  float* mean = nullptr;
};

}  // namespace p3d

namespace p3d {
struct ProfRec { int stage; hipEvent_t a, b; int launches; };
}

struct place3d_ctx {
  place3d_problem prob;
  // optional per-stage event profiler
  uint32_t prof_mask = 0;              // stages whose launches are bracketed by events
  std::vector<p3d::ProfRec> prof_pending;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_free;
  double prof_ms[PLACE3D_NSTAGES] = {0};
  long long prof_count[PLACE3D_NSTAGES] = {0};
  // side stream (default priority) on which the wirelength sweep of a step runs concurrently with
  // the density / spectral chain, and the events that fork it from and join it to the caller's stream
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  ~place3d_ctx();
  p3d::Geom g;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  std::string err;
  // spectral
  p3d::DctBases dct;
  p3d::SplitChain sc;
  p3d::FftChain fft;
  bool split = false;                  // dense contractions in split bf16
  bool step_dense = false;             // steps keep the dense contractions beside the fast transforms
  float *map_t = nullptr, *map_a = nullptr, *map_vg = nullptr, *map_vh = nullptr;
  float *map_pc = nullptr, *map_ps = nullptr, *map_qc = nullptr;
  // step scratch maps (rho, phi, ex, ey, ez)
  float *rho = nullptr, *phi = nullptr, *ex = nullptr, *ey = nullptr, *ez = nullptr;
  float* fixed_map = nullptr;
  // instances
  uint8_t* cls = nullptr;              // [n] kClsCell / kClsLarge / kClsFixed
  int32_t* large_list = nullptr;       // movable macros and oversized cells
  int32_t n_large = 0;
  float4* large_rec = nullptr;         // [4 * n_large] per-call footprint records of large instances
  float4* lpart = nullptr;             // [2 * lpart_cap] per (large instance, tile) partial sums
  long long lpart_cap = 0;
  int32_t* fixed_list = nullptr;       // fixed instances (their map is built once)
  int32_t n_fixed = 0;
  int32_t n_fillers = 0;               // instances of kind FILLER (bucketed cells)
  // tiles and per-call buckets
  p3d::TileGeom tg = {};
  int32_t* bk_counts = nullptr;        // [nblk][ntiles] counts, then exclusive offsets
  int32_t* bk_totals = nullptr;        // [ntiles]
  int32_t* bk_tile_start = nullptr;    // [ntiles + 1]
  float4* bk_entries = nullptr;        // [2 * 4n] (cell, tile) entries
  // tiles holding more entries than the plan's bound are split into equal chunks: chunk 0 is
  // taken by the tile's own workgroup, the extra chunks by the workgroups past the tile count;
  // in the density pass each stores its fixed-point sums, and the last one of a tile adds them
  int32_t max_extra[p3d::kSplits] = {};  // bounds: 4n / min (+1), at most count
  // chunk plans, one array each (the tile kernels take one pointer): [0] extra chunks and [1] entries
  // that a chunk may hold in the current buckets, then per tile its first extra chunk (-1: none),
  // per extra chunk its tile and its index within the tile, and from a tile's first extra chunk on
  // the chunks of its groups that are finished and, in a second array, its finished groups (zero
  // between calls)
  int32_t* bk_plan[p3d::kSplits] = {};   // [2 + ntiles + 4 max_extra]
  unsigned long long* chunk_sums = nullptr;  // [2 max_extra][2][T * T * nz]
  int32_t* cell_entry = nullptr;       // [n] packed tile range of each bucketed cell, -1 if none
  float4* entry_out = nullptr;         // [4][n] per-(cell, tile) gather / adjoint results, cell-major
  // two-stage reductions: part[slot * part_stride + block]
  double* part = nullptr;
  int32_t part_stride = 0;
  float* npins = nullptr;              // |E_i| as float [n]
  // wirelength schedule (nets ordered by lane-group class)
  int32_t* s_net_start = nullptr;      // [n_sched_nets + 1] slot ranges
  int32_t* s_pin_node = nullptr;       // [n_pins] owner per slot
  float4* s_off = nullptr;             // [n_pins] (ox_bot, oy_bot, ox_top, oy_top) per slot
  float4* pin_out = nullptr;           // [n_pins] (gx, gy, gz_wa, fda) in node order
  int32_t* node_slot_start = nullptr;  // [n+1] node -> range of pin_out
  int32_t* slot_pos = nullptr;         // [n_pins] slot -> position in node order
  int32_t* shared_nets = nullptr;      // [n_shared_nets] schedule nets holding an instance on
  int32_t n_shared_nets = 0;           // more than one pin (their FDA is redone per instance)
  int32_t* heavy_list = nullptr;       // instances with more than 32 pins (summed per wavefront)
  int32_t n_heavy = 0;
  p3d::ClassTab classes = {};
  int field_xfold = 0;                 // the last spectral_field left its field maps x-folded
  float cell_scale = 0.f;              // factor of the per-(cell, tile) gradient shares of the last gather
  int32_t* wa_block_order = nullptr;   // [n_wa_blocks] schedule blocks in order of their first net
  int32_t n_wa_blocks = 0;
  // per-instance scratch
  float4* xyzp = nullptr;              // [n] (x, y, z, 0) per instance, the net kernel's gather source
  float* wl_gzwa = nullptr;            // [n] alpha d p^(z)/dz per instance
  float* wl_fda = nullptr;             // [n] FDA z-gradient before normalisation
  float* gw = nullptr;                 // [3][n] wirelength gradient inside the GP step
  float* den_grad = nullptr;           // [3][n] density-penalty gradient inside the GP step
  double* red = nullptr;               // [R_COUNT] reductions
  double* red2 = nullptr;              // [R_COUNT] second set (init)
};

namespace p3d {

inline int set_err(place3d_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}
int hip_fail(place3d_ctx* c, hipError_t e, const char* where);

#define P3D_HIP(ctx, call)                                                     \
  do {                                                                         \
    hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess) return p3d::hip_fail((ctx), e_, #call);              \
  } while (0)

#define P3D_LAUNCH(ctx, what)                                                  \
  do {                                                                         \
    hipError_t e_ = hipGetLastError();                                         \
    if (e_ != hipSuccess) return p3d::hip_fail((ctx), e_, what);               \
  } while (0)

// large instances go through the density tiles when their per-tile partials fit the workspace
inline bool large_in_tiles(const place3d_ctx* c) {
  return (long long)c->n_large * c->tg.ntiles <= c->lpart_cap;
}

inline unsigned blocks_for(long long n, int threads) {
  long long b = (n + threads - 1) / threads;
  return (unsigned)(b < 1 ? 1 : b);
}

// Workgroup b of a launch of nb runs on die b % kNumXcd.  This bijection hands die x the
// contiguous work range [x q + min(x, r), ...) (q = nb / kNumXcd, r = nb % kNumXcd), so that
// neighbouring work items, which read neighbouring data, share one die's L2.
__host__ __device__ inline int xcd_swizzle(int b, int nb) {
  const int q = nb / kNumXcd, r = nb % kNumXcd, x = b % kNumXcd, i = b / kNumXcd;
  return x * q + (x < r ? x : r) + i;
}

// Profiler brackets (no-ops unless profiling is on).  prof_end records on the same stream.
int prof_begin(place3d_ctx* c, int stage, hipStream_t s);
int prof_end(place3d_ctx* c, hipStream_t s, int launches);

// One event pair per scope; `launches` is how many kernel launches the scope holds (a scope
// around several consecutive launches of one stage perturbs the stream less than one per launch)
struct ProfScope {
  place3d_ctx* c;
  hipStream_t s;
  bool on;
  int launches = 1;
  ProfScope(place3d_ctx* c_, int stage, hipStream_t s_) : c(c_), s(s_), on((c_->prof_mask >> stage) & 1u) {
    if (on) prof_begin(c, stage, s);
  }
  ~ProfScope() { if (on) prof_end(c, s, launches); }
};

// Sums (or maxima) of NQ rows of nparts float64 partials by a workgroup of 256 threads, in the fixed
// order of every final reduction here; all threads get the results.  The rows' loads are in flight
// together, four per thread and row.
template <int NQ>
__device__ __forceinline__ void row_sums(const double* const (&row)[NQ], int nparts, bool is_max, double (&sh)[NQ][256],
                                         double (&out)[NQ]) {
  double a[NQ][4] = {};
  int b = threadIdx.x;
  for (; b + 768 < nparts; b += 1024) {
    double v[NQ][4];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int u = 0; u < 4; ++u) v[q][u] = row[q][b + 256 * u];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int u = 0; u < 4; ++u) a[q][u] = is_max ? fmax(a[q][u], v[q][u]) : a[q][u] + v[q][u];
  }
  for (; b < nparts; b += 256)
#pragma unroll
    for (int q = 0; q < NQ; ++q) a[q][0] = is_max ? fmax(a[q][0], row[q][b]) : a[q][0] + row[q][b];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    sh[q][threadIdx.x] = is_max ? fmax(fmax(a[q][0], a[q][1]), fmax(a[q][2], a[q][3])) : (a[q][0] + a[q][1]) + (a[q][2] + a[q][3]);
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        sh[q][threadIdx.x] = is_max ? fmax(sh[q][threadIdx.x], sh[q][threadIdx.x + o]) : sh[q][threadIdx.x] + sh[q][threadIdx.x + o];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) out[q] = sh[q][0];
}

// Pins from which an evaluation runs its wirelength sweep on a side stream beside the density chain.
// The four event operations cost the host 45 to 60 us a call (2k instances: issued in 43 us on one
// stream, 88 on two), the overlap saves less the smaller the sweep is: step of 2k instances, 8k pins,
// 65 us on one stream, 72 to 88 on two; 60k instances, 235k pins, 98 and 94 to 98; 100k, 392k pins, 108
// and 103; 200k, 760k pins, 134 and 121; 1.2M, 4.5M pins, 361 and 346.
constexpr int kForkPins = 1 << 18;

// Partials up to which the move sums a step's norms itself, every workgroup the same two rows, instead
// of reading what a reduction launched before it left: it saves a launch (2k instances 88 -> 84 us a
// step, the host's time) and costs a round of loads per 1024 partials (200k instances, 785 partials:
// 125.5 -> 126.3 us).
constexpr int kOwnSumParts = 512;

// scale of the FDA z-gradient (Eq. fda-normalize) from the evaluation's norms
__device__ __forceinline__ double fda_scale(const double* red) {
  const double nf = red[R_NORM_FDA];
  return nf > 0.0 ? (red[R_NORM_X] + red[R_NORM_Y]) / (2.0 * nf) : 0.0;
}

// Cell density gradients held as per-(cell, tile) shares (entry != nullptr, cell-major [q][n], q < the
// cell's entry count read from its packed tile range), summed in the order the separate combine pass
// uses.
struct CellShares {
  const uint8_t* cls;
  const int32_t* cell_entry;
  const float4* entry;
  float scale;
};

// cls and packed: the instance's density class and packed tile range (loaded by the caller with
// its other operands); a cell's up to four shares are loaded together and summed in q order
__device__ __forceinline__ void density_grad_of(const CellShares& cs, const float* __restrict__ gd, int n, int i,
                                                uint8_t cls, int packed, float (&d)[3]) {
  if (!cs.entry || cls == kClsLarge) {
    for (int a = 0; a < 3; ++a) d[a] = gd[a * n + i];
    return;
  }
  float sx = 0.f, sy = 0.f, sz = 0.f;
  if (cls == kClsCell) {
    // the cell's entry count from its packed tile range; its shares are cell-major [q][n]
    // (a bucketed cell has 1, 2 or 4 entries: its tile range is 1 or 2 tiles per axis)
    const int cnt = packed < 0 ? 0 : (1 + ((packed >> 24) & 1)) * (1 + ((packed >> 25) & 1));
    // All four loads are issued together: an absent share's load re-reads share 0 (the same
    // cache line) and counts as zero, which leaves the sum in q order unchanged.
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
    const size_t i1 = cnt > 1 ? (size_t)n + i : (size_t)i;
    const size_t i2 = cnt > 2 ? 2 * (size_t)n + i : (size_t)i, i3 = cnt > 2 ? 3 * (size_t)n + i : (size_t)i;
    const float4 r0 = cs.entry[i], r1 = cs.entry[i1], r2 = cs.entry[i2], r3 = cs.entry[i3];
    const float4 v0 = r0, v1 = cnt > 1 ? r1 : z4, v2 = cnt > 2 ? r2 : z4, v3 = cnt > 2 ? r3 : z4;
    if (cnt > 0) {
      sx = ((v0.x + v1.x) + v2.x) + v3.x;
      sy = ((v0.y + v1.y) + v2.y) + v3.y;
      sz = ((v0.z + v1.z) + v2.z) + v3.z;
    }
    sx *= cs.scale; sy *= cs.scale; sz *= cs.scale;
  }
  d[0] = sx; d[1] = sy; d[2] = sz;
}

// place3d_workspace_size and place3d_create; steps: place3d_step and place3d_gp_init will be called on
// the context (a multi-die problem's contexts take neither, and hold nothing for them)
int workspace_size(const place3d_problem* prob, bool steps, size_t* bytes);
int create(const place3d_problem* prob, bool steps, void* d_workspace, size_t bytes, void* stream, place3d_ctx** out);

// ---- launchers implemented in the .hip sources (all enqueue only) ----
int launch_zero_f64(place3d_ctx* c, double* p, int n, hipStream_t s);
int launch_fill_f32(place3d_ctx* c, float* p, long long n, float v, hipStream_t s);

int build_dct_bases(place3d_ctx* c, hipStream_t s);
// x_folded_out: with folded contractions, leave ex / ey / ez as even and odd x halves (columns
// [0, nx/2) and [nx/2, nx)) for a consumer that unfolds them on load; ctx->field_xfold says
// whether that happened
int spectral_field(place3d_ctx* c, const float* rho, float* phi, float* ex, float* ey, float* ez,
                   double* energy, hipStream_t s, bool x_folded_out = false, bool in_step = false);
// the split chain's bases (at creation) and its contractions; outputs in natural x order
int build_split_chain(place3d_ctx* c, hipStream_t s);
int field_split(place3d_ctx* c, const float* rho, float* phi, float* ex, float* ey, float* ez, hipStream_t s);

// the fast transforms' tables (at creation) and their solve; outputs in natural x order
int build_fft(place3d_ctx* c, hipStream_t s);
int field_fft(place3d_ctx* c, const float* rho, float* phi, float* ex, float* ey, float* ez, hipStream_t s);

// out[0..nq) = sums (max if is_max) of partial slots slot0.. over nparts blocks, fixed order
int reduce_final(place3d_ctx* c, int slot0, int nq, int nparts, bool is_max, double* out, hipStream_t s);
// the same over the partials in `part` (stride per slot) instead of the workspace's
int reduce_final_in(place3d_ctx* c, const double* part, int stride, int slot0, int nq, int nparts, bool is_max,
                    double* out, hipStream_t s);
// two sum reductions in one launch: slots slot0.. (nq0 of them, nparts0 partials) into out0[] and
// slots slot1.. (nq1, nparts1) into out1[]
int reduce_final2(place3d_ctx* c, const double* part, int stride, int slot0, int nq0, int nparts0, double* out0, int slot1, int nq1, int nparts1,
                  double* out1, hipStream_t s);

int build_fixed_map(place3d_ctx* c, hipStream_t s);
// The same launch over up to kMaxMany contexts (blockIdx.y picks one), for the layers of a multi-die
// problem: their grids and options are the same, their instances are not.
constexpr int kMaxMany = 3;
template <class A, int B>
struct Many {
  A v[B];
  __device__ __forceinline__ const A& mine() const { return v[B == 1 ? 0 : blockIdx.y]; }
};
int bucket_cells_many(place3d_ctx* const* c, const float* const* xyz, int nb, hipStream_t s);
int density_tiles_many(place3d_ctx* const* c, const float* const* xyz, float* const* rho, double* const* red, int nb,
                       hipStream_t s, bool reduce);
int gather_bucketed_many(place3d_ctx* const* c, const float* const* xyz, const float* const* ex, const float* const* ey,
                         const float* const* ez, float scale, float* const* grad, int accumulate, int nb, hipStream_t s,
                         bool cells, bool xfold);
int field_fft_many(place3d_ctx* const* c, const float* const* rho, float* const* phi, float* const* ex, float* const* ey,
                   float* const* ez, int nb, hipStream_t s);
int bucket_cells(place3d_ctx* c, const float* xyz, hipStream_t s);
// reduce: finish the overflow reduction here (else the caller reduces the R_EXCESS slots later)
int density_tiles(place3d_ctx* c, const float* xyz, float* rho, double* red, hipStream_t s, bool reduce = true);
int gather_bucketed(place3d_ctx* c, const float* xyz, const float* ex, const float* ey, const float* ez, float scale,
                    float* grad, int accumulate, hipStream_t s, bool cells = true,
                    bool xfold = false);
// dscale: a device float64 factor multiplying scale (NULL: 1)
int adjoint_bucketed(place3d_ctx* c, const float* xyz, const float* gmap, float scale, float* grad, int accumulate,
                     hipStream_t s, bool cells = true, const double* dscale = nullptr);
int density_forward(place3d_ctx* c, const float* xyz, float* rho, hipStream_t s);
int density_field_gather(place3d_ctx* c, const float* xyz, const float* ex, const float* ey,
                         const float* ez, float scale, float* grad, int accumulate, hipStream_t s);
int density_adjoint(place3d_ctx* c, const float* xyz, const float* gmap, float scale, float* grad,
                    int accumulate, hipStream_t s, const double* dscale = nullptr);

// packed: c->xyzp already holds xyz (the bucket pass of the same positions wrote it); dscale: a
// device float64 factor of the gradient (NULL: 1); with_fda: the z-gradient carries the normalised
// FDA term, else only the derivative of alpha p^(z)
// red: receives the totals and norms (null without with_fda: none are made).  finish_z: write the
// z gradient and the metrics (else the caller's kernel takes wl_gzwa, wl_fda and the norms).
int wirelength_eval(place3d_ctx* c, const float* xyz, float* grad, int accumulate, double* red,
                    double* metrics, hipStream_t s, bool packed = false, const double* dscale = nullptr,
                    bool with_fda = true, bool finish_z = true);
// the model's net totals only (no gradient, nothing per pin) into metrics[PLACE3D_NMETRICS]; the
// packed positions and the per-workgroup partials go to xyzp / part (stride per slot) when given,
// else to the workspace's
int wirelength_value(place3d_ctx* c, const float* xyz, double* metrics, hipStream_t s, float4* xyzp = nullptr,
                     double* part = nullptr, int stride = 0);
// the same with the scratch in the library's static device array (place3d_wl_value_static)
constexpr int kStaticMaxInst = 1 << 21;      // instances whose positions the static scratch holds
constexpr int kStaticMaxBlocks = 1 << 18;    // wirelength workgroups whose partials it holds
int wirelength_value_static(place3d_ctx* c, const float* xyz, double* metrics, hipStream_t s);
// device address of the static scratch on the current device, looked up once per device
int static_scratch_setup(place3d_ctx* c, void** out);

}  // namespace p3d
