// nsplat_forward / the first half of nsplat_backward: per-tile alpha
// compositing (Sec. 3.4, Eq. 8-9) and its adjoint.
//
// The forward's unit of work is one wavefront per (tile, quadrant), or, for
// the long lists of small launches, one block (fwd_serial, fwd_block).
// Centres become exact tile-local FP32 coordinates when an
// entry is loaded (FP64 centre minus the tile origin, rounded once).  The
// forward stops a pixel once T < eps_T and a wavefront once all its pixels
// have stopped, and stores each pixel's state at every chunk boundary (a
// chunk is 2^ck_lg list positions, chosen per launch) it passes.  The
// adjoint runs one wavefront per (tile, quadrant, chunk), back to front from
// the state stored at the chunk's back boundary, parks each Gaussian's
// per-lane gradient values in LDS and sums a dozen or more such rows at a time,
// with one atomic per value and wavefront.
#include "nsplat_internal.h"

namespace nsp {

namespace {

// Work decomposition: one wavefront per (tile, quadrant) item.  A quadrant is
// 8x8 pixels, one per lane, whatever the tile side: 8x8 tiles are one, 16x16
// tiles have four and 32x32 tiles sixteen.  (Four quadrants of 16x16 with 2x2
// pixels per lane at 32x32 tiles kept four times the entries and put four times
// the work of each on one wavefront: forward and adjoint of 16 mixed scenes at
// 768^2 0.695 and 1.246 -> 0.565 and 1.185 ms, of 8 at 768^2 0.463 and 0.907 ->
// 0.267 and 0.636, of 4 at 512^2 0.498 and 0.324 -> 0.203 and 0.312, of 100 fill
// paths at 512^2 0.235 and 0.105 -> 0.070 and 0.082.)  A wavefront walks the
// tile's list in steps of up to 64 entries (64 E in the adjoint): every lane
// loads one (E; the next step's loads are issued before the current step is
// processed), entries whose support disc misses the quadrant are dropped, the rest are
// compacted in order into the wavefront's own LDS arrays and then composited
// one after another.  Wavefronts work on their own, except for a block's on a long
// list (fwd_block), and where a forward with a work queue takes its next items,
// one per wavefront of the block, when all of the last are done.
template <int TILE>
struct TileCfg {
  static constexpr int SUB = 8, COLS = TILE / 8, QUADS = COLS * COLS;
  static_assert(QUADS == adj_blocks(TILE), "the binning's items");
};
constexpr int WPB = 4;                  // wavefronts per block
// Kernel forms (template KIND): with the tangent-aligned kind, with the
// fill-run walk (see FillRun), and (the adjoint) with the sums of very long
// curves (LONG_TAUS).
constexpr int KIND_ANI = 1, KIND_FILL = 2, KIND_LONG = 4;
constexpr int BLOCK = 64 * WPB;

template <int TILE>
__device__ inline void pixel_of(int blk, int lane, int* lx, int* ly) {
  *lx = (blk % TileCfg<TILE>::COLS) * 8 + (lane & 7);
  *ly = (blk / TileCfg<TILE>::COLS) * 8 + (lane >> 3);
}

// Next work item of this wavefront: the static assignment, or the next `pop`
// entries of the device work queue (persistent form).
__device__ inline int next_item(int it, int persistent, int32_t* queue, int pop) {
  if (!persistent)
    return __builtin_amdgcn_readfirstlane(it == 0 ? (int)(blockIdx.x * WPB + (threadIdx.x >> 6)) : 0x7fffffff);
  int v = 0;
  if (__lane_id() == 0) v = atomicAdd(queue, pop);
  return __builtin_amdgcn_readfirstlane(v);
}

// One list entry as loaded by a lane, in the words that the loads return: a word
// converted where it is loaded makes a load ahead wait for its round trip on the
// spot (with the kind as an integer: forward of 200 mixed curves at 777 x 1003
// 0.172 ms, 0.161 without, of 16 mixed scenes at 768^2 0.541, 0.512, of 256 fill
// paths at 512^2 and h = 4 0.084, 0.079, before the lists' blocks 0.083).
struct Entry {
  Gauss r;
  float4 cf;  // the curve's colour, and the Gaussian's kind
  int g;
  __device__ int kind() const { return (int)cf.w; }  // 0 isotropic stroke, 1 fill, 2 tangent-aligned stroke
};

__device__ inline float first_lane(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

// Record and colour of Gaussian g.
__device__ inline void load_rec(const Gauss* __restrict__ gs, const float4* __restrict__ gcol, int g, Entry* e) {
  e->g = g;
  e->r = gs[g];
  e->cf = gcol[g];
}

// The entry's record and its curve's colour / fill tag (both by Gaussian
// index, so the two loads go out together once the index has arrived).
__device__ inline void load_entry(const int32_t* __restrict__ idx, const Gauss* __restrict__ gs,
                                  const float4* __restrict__ gcol, int pos, bool ok, Entry* e) {
  if (!ok) return;
  e->g = idx[pos];
  load_rec(gs, gcol, e->g, e);
}

// Rectangle of tile-local pixel centres: x in [x0, x1], y in [y0, y1].
struct Box {
  float x0, y0, x1, y1;
};

// The pixel centres held by the lanes with a set bit in `live` (lane l owns
// the pixel at column l & 7, row l >> 3 of the quadrant): rows from
// the lowest and highest set bits, columns from the eight row bytes folded
// together.  Scalar work on a wavefront-uniform mask; `live` != 0.
__device__ inline Box live_box_of(int qx, int qy, uint64_t live) {
  const int r0 = __builtin_ctzll(live) >> 3, r1 = (63 - __builtin_clzll(live)) >> 3;
  uint64_t f = live | (live >> 32);
  f |= f >> 16;
  f |= f >> 8;
  const uint32_t cols = (uint32_t)f & 0xffu;
  const int c0 = __builtin_ctz(cols), c1 = 31 - __builtin_clz(cols);
  Box b;
  b.x0 = (float)(qx + c0);
  b.x1 = (float)(qx + c1);
  b.y0 = (float)(qy + r0);
  b.y1 = (float)(qy + r1);
  return b;
}

// All pixel centres of the quadrant.
template <int TILE>
__device__ inline Box quad_box(int quad) {
  using Cfg = TileCfg<TILE>;
  Box b;
  b.x0 = (float)((quad % Cfg::COLS) * Cfg::SUB);
  b.y0 = (float)((quad / Cfg::COLS) * Cfg::SUB);
  b.x1 = b.x0 + (float)(Cfg::SUB - 1);
  b.y1 = b.y0 + (float)(Cfg::SUB - 1);
  return b;
}

// Tile-local centre (relative to the tile's first pixel centre), and whether
// the support disc reaches the rectangle `bx` of pixel centres (the quadrant's
// pixels that can still take part), with the radius enlarged by a relative
// 1e-4 so that the test is conservative under FP32 rounding.
__device__ inline bool entry_geometry(const Gauss& r, double ox, double oy, float ks, const Box& bx, float4* geo) {
  geo->x = (float)(r.mx - ox);
  geo->y = (float)(r.my - oy);
  const float rc = ks * r.sigma * 1.0001f + 1e-4f;
  const float dx = fmaxf(fmaxf(bx.x0 - geo->x, geo->x - bx.x1), 0.0f);
  const float dy = fmaxf(fmaxf(bx.y0 - geo->y, geo->y - bx.y1), 0.0f);
  return dx * dx + dy * dy <= rc * rc;
}

// The rest of a kept entry's geometry: squared support radius and exp2
// coefficient -log2(e) / (2 sigma^2), whose division in FP64 is most of an
// entry's staging and is left out in the steps that keep none.
__device__ inline void entry_support(const Gauss& r, float ks, float4* geo) {
  const double sg = (double)r.sigma;
  const float rr = ks * r.sigma;
  geo->z = rr * rr;
  geo->w = (float)(-0.5 * LOG2E / (sg * sg));
}

// A tangent-aligned Gaussian (axis sigma along t, sp across it, sigma >= sp)
// is evaluated as exp2(-(a^2 + b^2)) with a = d . u and b = r (d x u), d the
// offset from the centre: u = t sqrt(ck) / sigma, r = sigma / sp, and
// ck = log2(e) / 2, so that a^2 + b^2 = ck (d_t^2 / sigma^2 + d_n^2 / sp^2).
// The support is a^2 + b^2 <= ck k_sigma^2, inside the disc of radius
// k_sigma sigma that binning and culling use.  Entries are staged like the
// others (exp2 coefficient -ck / sigma^2); after staging a step that holds
// such entries, the wavefront converts them, reading (t, sp, r) by Gaussian
// index, so that the other kinds carry no extra loads.  Where the two axes
// agree r is exactly 1 and the theta partial exactly 0.
constexpr float ANI_CK = (float)(0.5 * LOG2E);
constexpr float ANI_SQRT_CK = 0.8493218002880191f;  // sqrt(log2(e) / 2)
__device__ inline void aniso_axes(const float4& aux, float coef, float* ux, float* uy, float* r) {
  const float k = __builtin_sqrtf(-coef);  // sqrt(ck) / sigma
  *ux = aux.x * k;
  *uy = aux.y * k;
  *r = aux.w;  // sigma / sp, rounded once from FP64 (exactly 1 where the axes agree)
}

__device__ inline uint64_t lanes_below() {
  const int lane = __lane_id();
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// ---------------------------------------------------------------------------
// Fill runs.  A fill curve's Gaussians sit on the lattice ((i + 1/2) h,
// (j + 1/2) h) of its window and are emitted row by row (Sec. 3.3), all with
// one sigma.  Binning's test (tile_axis) is separable and monotone along each
// lattice axis, so the curve's points on a tile form a rectangle
// [i0, i1] x [j0, j1] of the window, and since a tile's list is in Gaussian
// order they occupy one run of consecutive positions, row by row.  At h = 1
// the lattice is the pixel grid: a pixel's in-support Gaussians of the run are
// its lattice neighbours at integer offsets (dx, dy) with dx^2 + dy^2 <=
// (k_sigma sigma)^2, so each lane walks those offsets (in list order) and
// gathers the opacities from LDS instead of visiting every entry of the run.
// ---------------------------------------------------------------------------
struct FillRun {
  int c, ix0, iy0, nx, goff;  // curve, window origin, window columns, first Gaussian
  int i0, i1, j0, j1, w;      // the run's rectangle (window-relative) and its width
  int p_lo, p_hi;             // its list positions
  int g_top;                  // the Gaussian at the run's entry point
  float sigma;                // the curve's fill sigma
};

// Window-relative lattice indices [k0, k1] (below n) whose binning interval
// covers tile t along one axis: each lane tests one candidate (the same
// arithmetic as binning).  False when the interval does not fit the 64
// candidates.
__device__ inline bool fill_axis(int org, int n, double h, float r, float inv, int n_tiles, int t, int tile, int* k0,
                                 int* k1) {
  const int base = (int)floor(((double)t * tile - (double)r - 2.0) / h - 0.5) - org - 1;
  const int k = base + (int)__lane_id();
  bool ok = false;
  if (k >= 0 && k < n) {
    const float m = (float)(((double)(org + k) + 0.5) * h);
    float f0, f1;
    ok = tile_axis(m, r, inv, n_tiles, &f0, &f1) && f0 <= (float)t && (float)t <= f1;
  }
  const uint64_t b = __ballot(ok);
  if (b == 0ull) return false;
  const int lo = __builtin_ctzll(b), hi = 63 - __builtin_clzll(b);
  if (__popcll(b) != hi - lo + 1) return false;           // not an interval
  if ((lo == 0 && base + lo > 0) || (hi == 63 && base + hi < n - 1)) return false;  // may extend past the candidates
  *k0 = base + lo;
  *k1 = base + hi;
  return true;
}

// A fill curve's plan row, one word per lane, so that the next run's can be
// loaded while a run is walked (the forward).
struct PlanRow {
  int c = -1, held = 0;
  __device__ void load(const int32_t* __restrict__ plan, int curve) {
    c = curve;
    held = plan[(int64_t)P_STRIDE * curve + min((int)__lane_id(), P_STRIDE - 1)];
  }
  __device__ int word(int k) const { return __builtin_amdgcn_readlane(held, k); }
};

// The same by scalar loads where the run begins: the adjoint, which the row's
// registers cost more than its loads (256 fill paths at 512^2, held by the lanes
// and so: 0.136 and 0.132 ms in 8 x 8 tiles, 0.1345 and 0.1335 in 16 x 16).
struct PlanRowScalar {
  const __attribute__((address_space(4))) int32_t* row;
  __device__ PlanRowScalar(const int32_t* plan, int curve)
      : row((const __attribute__((address_space(4))) int32_t*)(plan + (int64_t)P_STRIDE * curve)) {}
  __device__ int word(int k) const { return row[k]; }
};

// The run of fill curve c (its plan row: `row`) that holds list position `at`
// (whose Gaussian has window index `local`): its rectangle and list positions,
// if they fit the list.  Wavefront-uniform.  Whether the list holds the whole
// rectangle there is for fill_corners_ok to say.
template <class Row>
__device__ inline bool fill_run_at(const Row& row, int c, int g, int local, float sigma, int at, int start, int end,
                                   double h, float ks, float inv, const SceneTab& st, int lt, int tile, FillRun* fr) {
  fr->c = c;
  fr->ix0 = row.word(P_IX0);
  fr->iy0 = row.word(P_IY0);
  fr->nx = row.word(P_NX);
  fr->goff = row.word(P_GOFF);
  const int ny = row.word(P_NY);
  fr->g_top = g;
  fr->sigma = sigma;
  if (fr->nx <= 0 || ny <= 0) return false;
  const float r = ks * sigma;
  const int tcol = lt % st.tiles_x, trow = lt / st.tiles_x;
  if (!fill_axis(fr->ix0, fr->nx, h, r, inv, st.tiles_x, tcol, tile, &fr->i0, &fr->i1)) return false;
  if (!fill_axis(fr->iy0, ny, h, r, inv, st.tiles_y, trow, tile, &fr->j0, &fr->j1)) return false;
  const int jt = local / fr->nx, it = local - jt * fr->nx;
  if (it < fr->i0 || it > fr->i1 || jt < fr->j0 || jt > fr->j1) return false;
  fr->w = fr->i1 - fr->i0 + 1;
  const int64_t n = (int64_t)fr->w * (fr->j1 - fr->j0 + 1);
  fr->p_lo = at - ((jt - fr->j0) * fr->w + (it - fr->i0));
  const int64_t p_hi = (int64_t)fr->p_lo + n - 1;
  if (fr->p_lo < start || p_hi >= end) return false;
  fr->p_hi = (int)p_hi;
  return true;
}

// The run's two corner entries are those of the rectangle: otherwise (a run
// cut short by a capacity overflow) it is left to the entry-by-entry path.
__device__ inline bool fill_corners_ok(const int32_t* __restrict__ idx, const FillRun& fr) {
  const int g_lo = __builtin_amdgcn_readfirstlane(idx[fr.p_lo]);
  const int g_hi = __builtin_amdgcn_readfirstlane(idx[fr.p_hi]);
  return g_lo == fr.goff + fr.j0 * fr.nx + fr.i0 && g_hi == fr.goff + fr.j1 * fr.nx + fr.i1;
}

// Opacities of the quadrant's lattice neighbourhood (NB x NB cells, window
// index (ib, jb) at cell 0; lane l gathers cells it * 64 + l): those of the
// run's Gaussians at list positions p0 .. p1, `none` elsewhere, read from the
// packed fill opacities (gop, the records' values).  Reads below the record
// capacity only, so that a rectangle still to be checked is safe.
template <int NB, int NIT>
__device__ inline void fill_gather(const float* __restrict__ gop, int64_t gcap, const FillRun& fr, int ib, int jb,
                                   int p0, int p1, float none, float (&og)[NIT]) {
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int sl = it * 64 + (int)__lane_id();
    const int j = jb + sl / NB, i = ib + sl % NB;
    float o = none;
    if (sl < NB * NB && i >= fr.i0 && i <= fr.i1 && j >= fr.j0 && j <= fr.j1) {
      const int pos = fr.p_lo + (j - fr.j0) * fr.w + (i - fr.i0);
      const int64_t g = (int64_t)fr.goff + (int64_t)j * fr.nx + i;
      if (pos >= p0 && pos <= p1 && g < gcap) o = gop[g];
    }
    og[it] = o;
  }
}

// Offsets (dx, dy) of a pixel's lattice neighbours inside the 6 sigma disc at
// h = 1 (sigma = eta / rho, so k_sigma sigma = 4.5 with the paper's
// constants): dx^2 + dy^2 <= R2, walked front to back (descending list
// position: rows from the bottom, each from the right).
constexpr int FR_R = 4;   // the largest |dx| the walk visits
constexpr int FR_R2 = 20;  // dx^2 + dy^2 bound for k_sigma sigma = 4.5
// LDS row stride of the adjoint's lattice cells: 24 floats puts the four
// lane rows of a half-wavefront in four different bank octets
constexpr int FR_NS = 24;

// A forward entry: what every composited pixel reads, in one 32-byte record
// (one LDS address per entry), and the colour, read where a run begins.
struct FwdRec {
  float4 geo;      // tile-local centre, squared support radius, exp2 coefficient
                   // (tangent-aligned: centre, scaled axis u)
  float op;           // opacity
  int pos, curve, g;  // list position, curve, Gaussian (tangent-aligned, once
                      // converted: the bits of the axis ratio r)
};
constexpr int FWD_ENTRY_BYTES = sizeof(FwdRec) + 16;
// An adjoint entry: geometry (centre, squared support radius, exp2
// coefficient), (g, or ~g for fills, list position, opacity bits, 1/sigma^3
// bits), and the colour with the curve's bits.
constexpr int BWD_ENTRY_BYTES = 48;
// The adjoint parks the per-lane gradient values it still has to sum over
// the wavefront in LDS rows of 64 floats and sums 16 rows at a time
// (flush_moments, flush_rows): one row for a stroke or fill entry, three for one
// of a very long curve (LONG_TAUS), five
// for a tangent-aligned one.  Rows are padded
// to 68 floats so that the 16-byte reads of 8 rows fall into different banks.
constexpr int RB = 16;      // parked rows
constexpr int RB_ROW = 68;  // floats per parked row
// wavefronts per SIMD the adjoint is built for: five without the fill-run
// walk at one entry per lane (their LDS slices, 7.6 KB each, fill the CU), four
// with it, one at several entries per lane
__host__ __device__ constexpr int bwd_waves(int E, int kind) {
  return E == 1 ? (kind & KIND_FILL ? 4 : 5) : 1;
}
__host__ __device__ constexpr size_t bwd_wave_bytes(int E) {
  return (size_t)64 * E * BWD_ENTRY_BYTES + (size_t)RB * (RB_ROW * 4 + 8);
}
// Stroke curves of more knot intervals than this keep the per-pixel FP32 terms
// and the order of their sums (three parked rows per entry, flush_rows) that all
// strokes had before the moments of flush_moments.  Not for their precision: the
// moments are the nearer form.  A knot interval's gradient is a suffix sum over
// all samples behind it that nearly cancels, and against 64-bit values the
// intervals' gradients of one curve at 1024^2 are off by (relative, 2-norm; the
// mean of three curves, three rows and moments, in 1e-6) 8.3 and 4.7 at 2,000
// intervals, 13.5 and 6.8 at 4,000, 14.9 and 7.7 at 10,240, 21.4 and 6.1 at
// 16,000.  But the two forms also differ from each other by that much, growing
// with the count (the largest of 24 curves: 0.7e-5 at 2,000, 1.4e-5 at 4,000,
// 1.6e-5 at 6,000, 1.9e-5 at 8,000, 2.5e-5 at 10,240), and a curve's results are
// held to 2e-5 of what they were.  The switch stands where that is met with a
// margin; the price is an adjoint of 0.354 ms instead of 0.263 at 10,240.
constexpr int LONG_TAUS = 6000;
// the flush's basis table (one per block): four functions of the 64 lanes
constexpr int BASIS_BYTES = 4 * RB_ROW * 4;

// Lower end of the step that starts at list position h (walking down from
// the list end): at most `depth` entries, not below `start`, and not across
// the boundary of h's chunk.
__device__ inline int step_floor(int h, int start, int depth, int end, int ck_lg) {
  const int k = (end - h) >> ck_lg;
  return max(max(start, h - depth), end - ((k + 1) << ck_lg));
}

// A (tile, quadrant) of the forward.
struct FwdItem {
  SceneTab st;
  int s, tile, quad, lt, x0, y0, start, end;
};

// A staged tangent-aligned entry takes its axis u and ratio r.
__device__ inline void convert_aniso(const float4* __restrict__ gaux, FwdRec& rec) {
  const float4 ax = gaux[rec.g];
  float ux, uy, rq;
  aniso_axes(ax, rec.geo.w, &ux, &uy, &rq);
  rec.geo.z = ux;
  rec.geo.w = uy;
  rec.g = __float_as_int(rq);
}

// One (tile, quadrant) on one wavefront, with its own LDS slice (64 entries).
// Bound by vector instructions, a dozen per entry and pixel: where the GPU is
// full, at 4.5 cycles each per SIMD; the longest list alone, at 38 to 47 ns an
// entry (fwd_block is for those).  A pixel's stopping position is taken from
// its last composited entry at the end of a step rather than selected at every
// entry, one compare and one LDS word less: 16 x 2000 key points at 1024^2
// 0.322 -> 0.305 ms, 200 mixed curves at 777 x 1003 0.190 -> 0.182, 16 mixed
// scenes in 32 x 32 tiles 0.763 -> 0.704.  Steps are never longer than 64
// (params.batch above 64 is the adjoint's): two or four entries per lane only
// took registers and LDS from other wavefronts.
template <int C, int TILE, int KIND>
__device__ __forceinline__ void fwd_serial(const nsplat_params& pr, const Work& w, const FwdItem& im,
                                           const Gauss* __restrict__ gs, const int32_t* __restrict__ idx,
                                           const float* __restrict__ bg, float* __restrict__ image,
                                           float* __restrict__ Tfin, int32_t* __restrict__ nlast,
                                           const int32_t* __restrict__ plan, int64_t gcap, int ck_lg,
                                           bool fill_lattice, char* mine_lds) {
  using Cfg = TileCfg<TILE>;
  constexpr bool ANI = (KIND & KIND_ANI) != 0;
  const float amax = pr.alpha_max, eps = pr.eps_T, ks = pr.k_sigma;
  const float inv_tile = 1.0f / (float)TILE;
  const int depth = min(pr.batch, 64);  // entries per step
  const int lane = __lane_id();
  const uint64_t below = lanes_below();
  FwdRec* wrec = (FwdRec*)mine_lds;
  float4* wcol = (float4*)(wrec + 64);  // colour
  const int s = im.s, tile = im.tile, quad = im.quad, lt = im.lt, x0 = im.x0, y0 = im.y0, start = im.start,
            end = im.end;
  const SceneTab st = im.st;
  // The colour is accumulated per run of entries of one curve (one
  // colour): over a run, sum alpha_j T_j = T at its start - T now
  // (alpha_j T_j = T_j - T_{j+1}), so each pixel keeps Tst, its T where the
  // run began, and adds col (Tst - T) where the run ends.  Runs end where
  // the curve changes between consecutive composited entries, at chunk
  // boundaries and at the end, all fixed by the list, so the result does not
  // depend on the batch depth.  The image's sums (tot, runs from Trun) are kept
  // apart from the chunks' and don't end at their boundaries, so that an image
  // does not depend on the chunk length either, which a small launch takes
  // shorter.
  int run_curve = -1, run_kind = 0;
  float rc0 = 0.0f, rc1 = 0.0f, rc2 = 0.0f;  // the run's colour
  int lx, ly;
  pixel_of<TILE>(quad, lane, &lx, &ly);
  const float px = (float)lx, py = (float)ly;
  // a pixel is live while T >= eps_T (0 <= eps_T <= 1): T only falls,
  // and it falls below eps_T exactly at the entry where the pixel stops;
  // pixels outside the image start at T = 0
  float T = (x0 + lx < st.W && y0 + ly < st.H) ? 1.0f : 0.0f;
  float Tst = T, Trun = T, acc[3] = {0.0f, 0.0f, 0.0f}, tot[3] = {0.0f, 0.0f, 0.0f};
  int stop = start;
  // the pixel's share of the chunk's colour from the current run so far
  auto close_chunk = [&]() {
    const float a = Tst - T;
    acc[0] = __builtin_fmaf(rc0, a, acc[0]);
    if (C == 3) {
      acc[1] = __builtin_fmaf(rc1, a, acc[1]);
      acc[2] = __builtin_fmaf(rc2, a, acc[2]);
    }
    Tst = T;
  };
  // the end of a run
  auto close_run = [&]() {
    close_chunk();
    const float a = Trun - T;
    tot[0] = __builtin_fmaf(rc0, a, tot[0]);
    if (C == 3) {
      tot[1] = __builtin_fmaf(rc1, a, tot[1]);
      tot[2] = __builtin_fmaf(rc2, a, tot[2]);
    }
    Trun = T;
  };
  const double ox = (double)x0 + 0.5, oy = (double)y0 + 0.5;
  const Box qbox = quad_box<TILE>(quad);
  // front to back: list positions end-1 down to start, at most `depth` per
  // step and never across a chunk boundary, where the state is stored
  const int ck0 = w.ck_off[tile];
  int n_ck = 0;  // chunk boundaries passed (state stored)
  // loads run two steps ahead for the list indices and one step ahead for
  // the records, so a step waits for one round trip, issued a step earlier
  Entry e;
  int gnext;  // Gaussian indices of the next step
  int hi = end, lo_s = step_floor(hi, start, depth, end, ck_lg);
  int nhi = lo_s, nlo = step_floor(nhi, start, depth, end, ck_lg);
  load_entry(idx, gs, w.gcol, hi - 1 - lane, lane < hi - lo_s, &e);
  gnext = lane < nhi - nlo ? idx[nhi - 1 - lane] : 0;
  // One fill run's positions fr.p_lo .. top at h = 1, front to back for each
  // pixel: the colour run, the chunk boundaries and the per-pixel
  // arithmetic are those of the entry-by-entry path, entry for entry.
  constexpr int FNB = Cfg::SUB + 2 * FR_R;  // lattice neighbourhood of the quadrant, per axis
  constexpr int FNIT = (FNB * FNB + 63) / 64;
  PlanRow prow;
  // (by the middle of a walk the next step's first entry is there)
  auto next_row = [&]() {
    if (hi > start && __builtin_amdgcn_readfirstlane(e.kind()) == 1)
      prow.load(plan, __builtin_amdgcn_readfirstlane(e.r.curve));
  };
  auto fill_run_fwd = [&](const FillRun& fr, float col0, float col1, float col2, int top, const float (&og)[FNIT]) {
    constexpr int NB = FNB;
    float* ol = (float*)mine_lds;            // [NB][NB] opacities (0: no Gaussian of the run waits there)
    if (run_curve != fr.c) {                 // a run of this curve already open goes on
      close_run();
      rc0 = col0;
      rc1 = col1;
      rc2 = col2;
      run_curve = fr.c;
    }
    const int qx = (quad % Cfg::COLS) * Cfg::SUB, qy = (quad / Cfg::COLS) * Cfg::SUB;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int it = 0; it < FNIT; ++it)
      if (it * 64 + lane < NB * NB) ol[it * 64 + lane] = og[it];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const double sgd = (double)fr.sigma;
    const float coef = (float)(-0.5 * LOG2E / (sgd * sgd));  // as entry_geometry
    // lane k holds G at squared lattice distance k, as the entry path forms it
    const int gtab = __float_as_int(__builtin_amdgcn_exp2f(coef * (float)lane));
    bool neg = false;
#pragma unroll
    for (int it = 0; it < FNIT; ++it) neg = neg || !(og[it] >= 0.0f);
    const bool nonneg = __ballot(neg) == 0ull;  // no negative (or NaN) opacity in the run
    int nb = end - ((n_ck + 1) << ck_lg);  // the next chunk boundary still to store
    // the pixel's LDS cell and the list position of its own lattice point
    const int cell0 = (ly - qy + FR_R) * NB + (lx - qx + FR_R);
    const int pb0 = fr.p_lo + (y0 + ly - fr.iy0 - fr.j0) * fr.w + (x0 + lx - fr.ix0 - fr.i0);
    // the state at chunk boundary nb (all positions >= it done)
    auto store_boundary = [&]() {
      close_chunk();
      float* ckp = w.ckbuf + (int64_t)(ck0 + ((end - nb) >> ck_lg) - 1) * (4 * TILE * TILE);
      const int slot = quad * 64 + lane;
      ckp[slot] = T;
#pragma unroll
      for (int ch = 0; ch < C; ++ch) {
        ckp[(1 + ch) * TILE * TILE + slot] = acc[ch];
        acc[ch] = 0.0f;
      }
      nb -= 1 << ck_lg;
    };
    // A run that holds no chunk boundary, no negative opacity and none that
    // alpha_max could cut at a distance of 1 or more (all but the pixel's own
    // lattice point, the only one at G = 1): rows by their number alone, the
    // same arithmetic with nothing to look up or test per row but the stops.
    // 256 fill paths at 512^2 0.091 -> 0.074 ms, and to 0.070 with the next run's
    // plan row loaded meanwhile.
    const float G1 = __int_as_float(__builtin_amdgcn_readlane(gtab, 1));
    bool cut = false;
#pragma unroll
    for (int it = 0; it < FNIT; ++it) cut = cut || !(og[it] * G1 <= amax);
    if (nonneg && fr.p_lo >= nb && __ballot(cut) == 0ull) {
      const int Y = y0 + qy - fr.iy0;  // the quadrant's first window row
      const int d_lo = max(-FR_R, fr.j0 - (Y + Cfg::SUB - 1)), d_hi = min(FR_R, fr.j1 - Y);
      auto row = [&](auto row_tag) {
        constexpr int dy = decltype(row_tag)::value;
        constexpr int dxm = dy * dy <= 4 ? 4 : (dy * dy == 9 ? 3 : 2);  // dx^2 + dy^2 <= FR_R2
        if (dy < d_lo || dy > d_hi) return;
        const int roff = cell0 + dy * NB;
        float f[2 * FR_R + 1], Tr = T;
#pragma unroll
        for (int dx = -dxm; dx <= dxm; ++dx) f[dx + FR_R] = ol[roff + dx];
#pragma unroll
        for (int dx = dxm; dx >= -dxm; --dx) {
          const float oG = f[dx + FR_R] * __int_as_float(__builtin_amdgcn_readlane(gtab, dx * dx + dy * dy));
          f[dx + FR_R] = 1.0f - (dx == 0 && dy == 0 ? fminf(amax, oG) : oG);
          Tr = Tr * f[dx + FR_R];
        }
        const bool live = T >= eps;
        if (__ballot(live && !(Tr >= eps)) == 0ull) {
          T = live ? Tr : T;
          return;
        }
        // some pixel stops inside the row: cell by cell
        const int rpos = pb0 + dy * fr.w;
#pragma unroll
        for (int dx = dxm; dx >= -dxm; --dx) {
          const float Tn = T * f[dx + FR_R];
          const bool lv = T >= eps;
          stop = (lv && Tn < eps) ? rpos + dx : stop;
          T = lv ? Tn : T;
        }
      };
      row(std::integral_constant<int, 4>{});
      row(std::integral_constant<int, 3>{});
      row(std::integral_constant<int, 2>{});
      row(std::integral_constant<int, 1>{});
      row(std::integral_constant<int, 0>{});
      next_row();
      row(std::integral_constant<int, -1>{});
      row(std::integral_constant<int, -2>{});
      row(std::integral_constant<int, -3>{});
      row(std::integral_constant<int, -4>{});
      static_assert(FR_R == 4, "nine rows");
    } else {
#pragma unroll 1
      for (int dy = FR_R; dy >= -FR_R; --dy) {
        const int dxm = dy * dy <= 4 ? 4 : (dy * dy == 9 ? 3 : 2);  // dx^2 + dy^2 <= FR_R2
        const int roff = cell0 + dy * NB;
        const int rpos = pb0 + dy * fr.w;
        {
          // a row with no Gaussian still to composite for any live pixel
          // changes nothing (chunk boundaries it crosses are stored with
          // the unchanged state at the end)
          const int jr = y0 + ly + dy - fr.iy0, ir = x0 + lx - fr.ix0;
          const bool any = T >= eps && jr >= fr.j0 && jr <= fr.j1 && ir + dxm >= fr.i0 && ir - dxm <= fr.i1 &&
                           rpos - dxm <= top;
          if (__ballot(any) == 0ull) continue;
        }
        // the row's opacities first, one LDS wait per row, and its five
        // Gaussian factors (|dx| = 0 .. 4) from the table
        float orow[2 * FR_R + 1], Gr[FR_R + 1];
#pragma unroll
        for (int dx = -FR_R; dx <= FR_R; ++dx) orow[dx + FR_R] = ol[roff + dx];
#pragma unroll
        for (int a = 0; a <= FR_R; ++a) Gr[a] = __int_as_float(__builtin_amdgcn_readlane(gtab, a * a + dy * dy));
        auto cell = [&](int dx, bool check) {
          const float G = Gr[dx < 0 ? -dx : dx];
          const float o = orow[dx + FR_R];
          const int pos = rpos + dx;
          if (check && o != 0.0f)
            while (pos < nb) store_boundary();
          const float Tn = T * (1.0f - fminf(amax, o * G));
          const bool live = T >= eps;
          stop = (live && Tn < eps) ? pos : stop;
          T = live ? Tn : T;
        };
        // a chunk boundary falls in the row of some lane only now and then
        if (__ballot(rpos - dxm < nb) == 0ull) {
          // With no negative opacity in the run T does not grow along the
          // row, so a pixel live at its start whose T ends it at or above
          // eps_T was live at every cell: the row's product, with no stop
          // test, is then the cell-by-cell result.  Only where some pixel
          // stops inside the row is the row taken cell by cell.
          float Tr = T;
#pragma unroll
          for (int dx = FR_R; dx >= -FR_R; --dx)
            if (dx <= dxm && dx >= -dxm) Tr = Tr * (1.0f - fminf(amax, orow[dx + FR_R] * Gr[dx < 0 ? -dx : dx]));
          const bool live = T >= eps;
          if (nonneg && __ballot(live && !(Tr >= eps)) == 0ull) {
            T = live ? Tr : T;
          } else {
#pragma unroll
            for (int dx = FR_R; dx >= -FR_R; --dx)
              if (dx <= dxm && dx >= -dxm) cell(dx, false);
          }
        } else {
#pragma unroll
          for (int dx = FR_R; dx >= -FR_R; --dx)
            if (dx <= dxm && dx >= -dxm) cell(dx, true);
        }
      }
    }
    // boundaries at or above the run's bottom (none at or below start)
    const int bl = max(fr.p_lo, start + 1);
    while (nb >= bl) store_boundary();
    n_ck = (end - bl) >> ck_lg;
  };
  while (hi > start) {
    if (fill_lattice && __builtin_amdgcn_readfirstlane(e.kind()) == 1) {
      // the next entry (position hi - 1, lane 0's first) is a fill
      // Gaussian: take its run's remaining positions pixel by pixel
      FillRun fr;
      const int c = __builtin_amdgcn_readfirstlane(e.r.curve);
      const float sg = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, e.r.sigma)));
      const float rr = ks * sg;
      float og[FNIT];
      bool take = false;
      if (rr * rr >= (float)FR_R2 && rr * rr < (float)(FR_R2 + 5)) {
        if (prow.c != c) prow.load(plan, c);
        if (fill_run_at(prow, c, __builtin_amdgcn_readfirstlane(e.g), __builtin_amdgcn_readfirstlane(e.r.local), sg,
                        hi - 1, start, end, 1.0, ks, inv_tile, st, lt, TILE, &fr)) {
          // the opacities and the corner check in flight together
          const int ib = x0 + (quad % Cfg::COLS) * Cfg::SUB - fr.ix0 - FR_R,
                    jb = y0 + (quad / Cfg::COLS) * Cfg::SUB - fr.iy0 - FR_R;
          fill_gather<FNB, FNIT>(w.gop, gcap, fr, ib, jb, fr.p_lo, hi - 1, 0.0f, og);
          take = fill_corners_ok(idx, fr);
        }
      }
      if (take) {
        const int top = hi - 1;
        const float col0 = first_lane(e.cf.x), col1 = first_lane(e.cf.y), col2 = first_lane(e.cf.z);
        hi = fr.p_lo;
        // the next step's loads (as at the start of the list), in flight
        // during the walk
        lo_s = step_floor(hi, start, depth, end, ck_lg);
        nhi = lo_s;
        nlo = step_floor(nhi, start, depth, end, ck_lg);
        load_entry(idx, gs, w.gcol, hi - 1 - lane, lane < hi - lo_s, &e);
        gnext = lane < nhi - nlo ? idx[nhi - 1 - lane] : 0;
        fill_run_fwd(fr, col0, col1, col2, top, og);
        if (__ballot(T >= eps) == 0ull) break;  // every pixel of the quadrant has stopped
        continue;
      }
    }
    float4 geo;
    const bool keep = lane < hi - lo_s && entry_geometry(e.r, ox, oy, ks, qbox, &geo);
    const uint64_t m = __ballot(keep);
    const int cnt = __popcll(m);
    const bool step_aniso = ANI && __ballot(keep && e.kind() == 2) != 0ull;
    if (keep) {
      entry_support(e.r, ks, &geo);
      const int dst = __popcll(m & below);
      FwdRec rec;
      rec.geo = geo;
      rec.op = e.r.opacity;
      rec.pos = hi - 1 - lane;
      rec.curve = e.r.curve;
      rec.g = e.g;
      wrec[dst] = rec;
      wcol[dst] = make_float4(e.cf.x, e.cf.y, e.cf.z, ANI ? (float)e.kind() : 0.0f);
    }
    // next step's records (their indices arrived during this step's
    // predecessor) and the indices of the step after, in flight while
    // this step is composited
    const int n2hi = nlo, n2lo = step_floor(n2hi, start, depth, end, ck_lg);
    if (lane < nhi - nlo) load_rec(gs, w.gcol, gnext, &e);
    gnext = lane < n2hi - n2lo ? idx[n2hi - 1 - lane] : 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (ANI && step_aniso) {
      // tangent-aligned entries of the step take their axis u and ratio r
      if (lane < cnt && wcol[lane].w == 2.0f) convert_aniso(w.gaux, wrec[lane]);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // composited entries that begin a run (their curve differs from the
    // entry before, the first one compared with the previous step's run)
    const int prev = lane == 0 ? run_curve : wrec[lane > 0 ? lane - 1 : 0].curve;
    const uint64_t rs = __ballot(lane < cnt && wrec[lane].curve != prev);
    int last = 0;                // the pixel's last composited entry of the step
    const bool was = T >= eps;  // live in front of the step
    for (int j = 0; j < cnt;) {
      // this segment: j up to the next run start (or the step's end)
      const uint64_t after = j < 63 ? rs & (~0ull << (j + 1)) : 0ull;
      const int jend = after ? __builtin_ctzll(after) : cnt;
      if ((rs >> j) & 1ull) {  // a new run: close the previous one
        close_run();
        const float4 pc = wcol[j];
        rc0 = pc.x;
        rc1 = pc.y;
        rc2 = pc.z;
        run_curve = wrec[j].curve;
        if (ANI) run_kind = __builtin_amdgcn_readfirstlane((int)pc.w);
      }
      if (ANI && run_kind == 2) {
        // tangent-aligned strokes (elliptical Eq. 9)
        const float lim = ANI_CK * ks * ks;
        for (; j < jend; ++j) {
          const float4 gm = wrec[j].geo;
          const float op = wrec[j].op, rq = __int_as_float(wrec[j].g);
          const float dx = px - gm.x, dy = py - gm.y;
          const float a = __builtin_fmaf(dx, gm.z, dy * gm.w);
          const float b = rq * __builtin_fmaf(dy, gm.z, -(dx * gm.w));
          const float m = __builtin_fmaf(a, a, b * b);
          const float G = __builtin_amdgcn_exp2f(-m);
          const bool in = (m <= lim) && (T >= eps);
          const float Tn = T * (1.0f - fminf(amax, op * G));
          last = in ? j : last;
          T = in ? Tn : T;
        }
      }
#pragma unroll 8
      for (; j < jend; ++j) {
        const float4 gm = wrec[j].geo;
        const float op = wrec[j].op;
        const float dx = px - gm.x, dy = py - gm.y;
        const float d2 = __builtin_fmaf(dx, dx, dy * dy);
        const float G = __builtin_amdgcn_exp2f(gm.w * d2);
        const bool in = (d2 <= gm.z) && (T >= eps);
        const float Tn = T * (1.0f - fminf(amax, op * G));
        last = in ? j : last;
        T = in ? Tn : T;
      }
    }
    // a pixel that stopped in this step did so at the last entry it took
    if (was && T < eps) stop = wrec[last].pos;
    hi = nhi;
    lo_s = nlo;
    nhi = n2hi;
    nlo = n2lo;
    if (hi > start && ((end - hi) & ((1 << ck_lg) - 1)) == 0) {
      // at the front of chunk k = (end - hi) / CK: T, and the colour the
      // chunk just finished contributed (the current run closed at the
      // boundary; the sum restarts for the next chunk)
      float* ckp = w.ckbuf + (int64_t)(ck0 + ((end - hi) >> ck_lg) - 1) * (4 * TILE * TILE);
      close_chunk();
      const int slot = quad * 64 + lane;
      ckp[slot] = T;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        ckp[(1 + c) * TILE * TILE + slot] = acc[c];
        acc[c] = 0.0f;
      }
      ++n_ck;
    }
    __builtin_amdgcn_wave_barrier();
    if (__ballot(T >= eps) == 0ull) break;  // every pixel of the quadrant has stopped
  }
  close_run();
  // Suffix sums over the chunks, back to front: each boundary's slot
  // receives the colour of everything behind it (the chunks after it; the
  // background is added by the adjoint), a sum of the chunks' own
  // contributions with no cancellation, and the total is the pixel's
  // colour (to the rounding of tot).  Each lane rereads only the slots it wrote itself.
  const int64_t ck_first = (int64_t)ck0 * (4 * TILE * TILE);
  for (int k = n_ck; k >= 1; --k) {
    float* ckp = w.ckbuf + ck_first + (int64_t)(k - 1) * (4 * TILE * TILE);
    const int slot = quad * 64 + lane;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float ch = ckp[(1 + c) * TILE * TILE + slot];
      ckp[(1 + c) * TILE * TILE + slot] = acc[c];
      acc[c] += ch;
    }
  }
  const int x = x0 + lx, y = y0 + ly;
  if (x < st.W && y < st.H) {
    const int64_t pix = (int64_t)st.pix_off + (int64_t)y * st.W + x;
    const int64_t plane = (int64_t)st.H * st.W;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int64_t o = (int64_t)st.pix_off * C + c * plane + (int64_t)y * st.W + x;
      image[o] = __builtin_fmaf(T, bg[s * C + c], tot[c]);
    }
    Tfin[pix] = T;
    nlast[pix] = stop;
  }
}

// Totals over the 64 lanes of a wavefront of N per-lane values at once, with
// DPP row shifts and row broadcasts (no LDS traffic): inclusive sums inside
// each row of 16 lanes, then row 0 into row 1, row 2 into row 3, and rows 0-1
// into row 3, so that lane 63 ends with the total.  The N chains are
// interleaved so that each fills the others' data-hazard slots.  Lane i < N
// of the result holds the total of value i (0 elsewhere), ready for one
// N-lane atomic.
template <int N>
__device__ inline float wave_totals_to_lanes(const float (&v)[N]) {
  int x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = __float_as_int(v[i]);
#define NSP_DPP_STEP(ctrl, rmask, bc)                                                                          \
  _Pragma("unroll") for (int i = 0; i < N; ++i) x[i] = __float_as_int(                                        \
      __int_as_float(x[i]) + __int_as_float(__builtin_amdgcn_update_dpp(0, x[i], ctrl, rmask, 0xf, bc)));
  NSP_DPP_STEP(0x111, 0xf, true)
  NSP_DPP_STEP(0x112, 0xf, true)
  NSP_DPP_STEP(0x114, 0xf, true)
  NSP_DPP_STEP(0x118, 0xf, true)
  NSP_DPP_STEP(0x142, 0xa, false)
  NSP_DPP_STEP(0x143, 0xc, false)
#undef NSP_DPP_STEP
  const int lane = __lane_id();
  float out = 0.0f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float t = __int_as_float(__builtin_amdgcn_readlane(x[i], 63));
    out = lane == i ? t : out;
  }
  return out;
}

// Inclusive products over the lanes: lane l gets x_0 x_1 ... x_l.
__device__ inline float wave_scan_product(float x) {
#define NSP_DPP_MUL(ctrl, rmask)                                                                            \
  x *= __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(1.0f), __float_as_int(x), ctrl, rmask, 0xf, \
                                                  false));
  NSP_DPP_MUL(0x111, 0xf)
  NSP_DPP_MUL(0x112, 0xf)
  NSP_DPP_MUL(0x114, 0xf)
  NSP_DPP_MUL(0x118, 0xf)
  NSP_DPP_MUL(0x142, 0xa)
  NSP_DPP_MUL(0x143, 0xc)
#undef NSP_DPP_MUL
  return x;
}

// ---------------------------------------------------------------------------
// A long list on the eight wavefronts of a block.  The list is taken from its
// end in windows of 512 positions: every wavefront culls and stages 64 of them,
// the kept entries are compacted into one array, and each wavefront composites
// a share, half of what two wavefronts kept, on its own: per pixel the product
// of the factors 1 - alpha, starting from T = 1, and the colours on that
// scale.  The products go through LDS, every wavefront multiplies them up in
// list order, and T at the front of its share scales its colours.  Where a
// pixel goes below eps_T inside a share, that share's wavefront finds the entry
// with one scan over the lanes, an entry each, or, for many pixels at once, by
// compositing the share again entry by entry.  In a window with a negative (or
// NaN) opacity, where T may grow, the shares are composited one after another.
//
// On one wavefront (fwd_serial) an entry takes 38 ns, a dozen vector
// instructions at the 11 cycles between two of a single wavefront, so that
// launches with a few long lists waited for the longest one.  With eight, a
// window takes about 17,000 cycles, 6,000 of them in the composited shares,
// 900 per pixel that stops and 5,000 in staging, exchange and the chunk's
// state: 12 quintic strokes at 512^2 (longest list 9,736) 0.376 -> 0.240 ms,
// 16 closed ones at 512^2 (1,667) 0.067 -> 0.047, 32 strokes at 256^2 (1,537)
// 0.057 -> 0.036, 32 tangent-aligned ones (265) 0.031 -> 0.023.  Shares of all
// eight wavefronts' entries together were more even (0.228, 0.040, 0.028,
// 0.022 ms), but then a chunk could not end inside a window, which the adjoint
// gains more from (small_chunk_log2).  Built for six wavefronts per SIMD, so
// that three blocks share a CU: at four (two blocks) it was a quarter slower.
// ---------------------------------------------------------------------------
constexpr int FW = 8;  // wavefronts per block of the forward
constexpr int FWD_BLOCK = 64 * FW;
constexpr int FWD_WINDOW = 64 * FW;
static_assert(CK_SMALL >= 64 && FWD_WINDOW % CK_SMALL == 0 && FWD_WINDOW <= CK_MIN,
              "a window lies inside one chunk or holds whole ones");
constexpr int STOP_SCANS = 12;  // more stopping pixels than this: composite the share again

struct FwdLds {
  FwdRec rec[FWD_WINDOW];  // the window's entries (colour sums when exchanged; fwd_serial: 64 per wavefront)
  float4 col[FWD_WINDOW];
  float prod[FW][64];      // the shares' products
  float stopT[64];         // T and list position where a pixel stopped
  int stopP[64];
  int cnt[FW], neg[FW];  // entries kept per wavefront, and whether one has a negative opacity
  int next;
};

template <int C, int TILE, int KIND>
__device__ __forceinline__ void fwd_block(const nsplat_params& pr, const Work& w, const FwdItem& im,
                                          const Gauss* __restrict__ gs, const int32_t* __restrict__ idx,
                                          const float* __restrict__ bg, float* __restrict__ image,
                                          float* __restrict__ Tfin, int32_t* __restrict__ nlast, int ck_lg,
                                          FwdLds& L) {
  constexpr bool ANI = (KIND & KIND_ANI) != 0;
  static_assert(sizeof(L.rec) + sizeof(L.col) >= sizeof(float) * FW * 64 * C, "colour sums fit");
  const float amax = pr.alpha_max, eps = pr.eps_T, ks = pr.k_sigma;
  const float lim = ANI_CK * ks * ks;  // (tangent-aligned entries)
  const int lane = __lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t below = lanes_below();
  const int quad = im.quad, x0 = im.x0, y0 = im.y0, start = im.start, end = im.end;
  // T: the pixels' transmittance in front of the window, in every wavefront.
  // A pixel is live while T >= eps_T (0 <= eps_T <= 1); -1 stands for a
  // stopped one (stopT, stopP) and for pixels outside the image.
  int lx, ly;
  pixel_of<TILE>(quad, lane, &lx, &ly);
  const float px = (float)lx, py = (float)ly;
  float T = (x0 + lx < im.st.W && y0 + ly < im.st.H) ? 1.0f : -1.0f;
  const double ox = (double)x0 + 0.5, oy = (double)y0 + 0.5;
  const Box qbox = quad_box<TILE>(quad);
  // A share is taken from a group's positions, those of two wavefronts: a
  // chunk holds whole groups whatever its length, so that the image does not
  // depend on it.
  constexpr int group = CK_SMALL / 64;
  const int ck0 = w.ck_off[im.tile];
  int n_ck = 0;  // chunk boundaries passed (state stored)
  const int slot = quad * 64 + lane;
  // T at the front of share k of the window at whi, if a chunk ends there
  // (chunk number (end - lo) / CK counts from 1)
  auto boundary = [&](int lo) { return lo > start && ((end - lo) & ((1 << ck_lg) - 1)) == 0; };
  auto ck_at = [&](int lo) {
    return w.ckbuf + (int64_t)(ck0 + ((end - lo) >> ck_lg) - 1) * (4 * TILE * TILE) + slot;
  };
  auto put_T = [&](int whi, int k, float t) {
    const int lo = whi - 64 * (k + 1);
    if (wv == FW - 1 && boundary(lo)) *ck_at(lo) = t;
  };
  float tail = 0.0f, tot = 0.0f;  // channel wv's colour since the last boundary, and the image's
  float* sums = (float*)L.rec;  // [FW][C][64], at the end of a window
  // list indices are loaded two windows ahead and records one window ahead
  Entry e;
  int gnext = 0;
  e.cf.w = 0.0f;
  {
    const int p = end - 1 - 64 * wv - lane;
    load_entry(idx, gs, w.gcol, p, p >= start, &e);
    if (p - FWD_WINDOW >= start) gnext = idx[p - FWD_WINDOW];
  }
  for (int whi = end; whi > start; whi -= FWD_WINDOW) {
    const int pos = whi - 1 - 64 * wv - lane;
    float4 geo;
    const bool keep = pos >= start && entry_geometry(e.r, ox, oy, ks, qbox, &geo);
    const uint64_t m = __ballot(keep);
    const bool neg = __ballot(keep && !(e.r.opacity >= 0.0f)) != 0ull;
    if (lane == 0) {
      L.cnt[wv] = __popcll(m);
      L.neg[wv] = neg;
    }
    __syncthreads();
    int base = 0, g0 = 0, K = 0;
    bool any_neg = false;
#pragma unroll
    for (int k = 0; k < FW; ++k) {
      const int n = L.cnt[k];
      base += k < wv ? n : 0;
      g0 += k < (wv & -group) ? n : 0;
      K += (k & -group) == (wv & -group) ? n : 0;
      any_neg = any_neg || L.neg[k] != 0;
    }
    if (keep) {
      entry_support(e.r, ks, &geo);
      const int dst = base + __popcll(m & below);
      FwdRec rec;
      rec.geo = geo;
      rec.op = e.r.opacity;
      rec.pos = pos;
      rec.curve = e.r.curve;
      rec.g = e.g;
      if (ANI && e.kind() == 2) convert_aniso(w.gaux, rec);
      L.rec[dst] = rec;
      L.col[dst] = make_float4(e.cf.x, e.cf.y, e.cf.z, (float)e.kind());
    }
    // the next window's records, and the indices of the one after, in flight
    // during this window
    if (pos - FWD_WINDOW >= start) {
      load_rec(gs, w.gcol, gnext, &e);
      if (pos - 2 * FWD_WINDOW >= start) gnext = idx[pos - 2 * FWD_WINDOW];
    }
    __syncthreads();
    // this wavefront's share: n (at most 64) of the K entries of its group's
    // positions, from entry g0 on
    K = __builtin_amdgcn_readfirstlane(K);
    g0 = __builtin_amdgcn_readfirstlane(g0);
    const int in = wv & (group - 1), ja = g0 + K * in / group, n = g0 + K * (in + 1) / group - ja;
    const FwdRec* rec = L.rec + ja;
    const float4* col = L.col + ja;
    // entries whose curve differs from the entry before
    const uint64_t rs = __ballot(lane < n && (lane == 0 || rec[lane].curve != rec[lane > 0 ? lane - 1 : 0].curve));
    // Composites the share into t (from the given start) and ca, the colour
    // per run of entries of one curve as in fwd_serial.  STOP: pixels with
    // t >= eps stop where t falls below it, at position sp; lp is the last
    // position that they composited.
    float t, ca[3], con[3] = {0.0f, 0.0f, 0.0f};  // con: the share's colours at the pixels' own T
    int sp = -1, lp = start;
    auto composite = [&](auto stop_tag) {
      constexpr bool STOP = decltype(stop_tag)::value;
      float tst = t, rc0 = 0.0f, rc1 = 0.0f, rc2 = 0.0f;
#pragma unroll
      for (int c = 0; c < 3; ++c) ca[c] = 0.0f;
      auto close_run = [&]() {
        const float a = tst - t;
        ca[0] = __builtin_fmaf(rc0, a, ca[0]);
        if (C == 3) {
          ca[1] = __builtin_fmaf(rc1, a, ca[1]);
          ca[2] = __builtin_fmaf(rc2, a, ca[2]);
        }
        tst = t;
      };
      auto take = [&](bool in, float f, int at) {
        const float tn = t * f;
        if (STOP) {
          in = in && t >= eps;
          sp = (in && tn < eps) ? at : sp;
          lp = in ? at : lp;
        }
        t = in ? tn : t;
      };
      auto disc = [&](const FwdRec& r) {
        const float4 gm = r.geo;
        const float op = r.op;
        const int at = STOP ? r.pos : 0;
        const float dx = px - gm.x, dy = py - gm.y;
        const float d2 = __builtin_fmaf(dx, dx, dy * dy);
        const float G = __builtin_amdgcn_exp2f(gm.w * d2);
        take(d2 <= gm.z, 1.0f - fminf(amax, op * G), at);
      };
      for (int j = 0; j < n;) {
        const uint64_t after = j < 63 ? rs & (~0ull << (j + 1)) : 0ull;
        const int jend = after ? __builtin_ctzll(after) : n;  // up to the next run
        close_run();
        const float4 pc = col[j];
        rc0 = pc.x;
        rc1 = pc.y;
        rc2 = pc.z;
        if (ANI && __builtin_amdgcn_readfirstlane((int)pc.w) == 2) {
          // tangent-aligned strokes (elliptical Eq. 9)
          for (; j < jend; ++j) {
            const float4 gm = rec[j].geo;
            const float op = rec[j].op, rq = __int_as_float(rec[j].g);
            const int at = STOP ? rec[j].pos : 0;
            const float dx = px - gm.x, dy = py - gm.y;
            const float a = __builtin_fmaf(dx, gm.z, dy * gm.w);
            const float b = rq * __builtin_fmaf(dy, gm.z, -(dx * gm.w));
            const float mm = __builtin_fmaf(a, a, b * b);
            const float G = __builtin_amdgcn_exp2f(-mm);
            take(mm <= lim, 1.0f - fminf(amax, op * G), at);
          }
        }
        if constexpr (STOP) {
#pragma unroll 2
          for (; j < jend; ++j) disc(rec[j]);
        } else {
#pragma unroll 8
          for (; j < jend; ++j) disc(rec[j]);
        }
      }
      close_run();
    };
    if (!any_neg) {
      t = 1.0f;
      composite(std::false_type{});
      L.prod[wv][lane] = t;
      __syncthreads();
      // T through the window, and at the front of this share
      float Tw = T;
      bool flag = false;
#pragma unroll
      for (int k = 0; k < FW; ++k) {
        const float Tn = T * L.prod[k][lane];
        const bool live = T >= eps, goes = live && !(Tn >= eps);
        if (k == wv) {
          Tw = T;
          flag = goes;
        }
        T = goes ? -1.0f : (live ? Tn : T);
        put_T(whi, k, T);
      }
      uint64_t left = __ballot(flag);
      if (Tw >= eps && !flag) {
#pragma unroll
        for (int c = 0; c < C; ++c) con[c] = Tw * ca[c];
      }
      // where the products say that a pixel stops in this share but its
      // factors one by one do not, it stops at its last entry of the share
      const float under = __int_as_float(__float_as_int(eps) - 1);
      if (__popcll(left) > STOP_SCANS) {
        t = flag ? Tw : -1.0f;
        composite(std::true_type{});
        if (flag) {
          L.stopT[lane] = fminf(t, under);
          L.stopP[lane] = sp >= 0 ? sp : lp;
#pragma unroll
          for (int c = 0; c < C; ++c) con[c] = ca[c];
        }
      } else if (left) {
        const FwdRec r = rec[lane < n ? lane : 0];
        const float4 pc = col[lane < n ? lane : 0];
        while (left) {
          // the pixel of lane l: an entry per lane
          const int l = __builtin_ctzll(left);
          left &= left - 1;
          const float dx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(px), l)) - r.geo.x;
          const float dy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(py), l)) - r.geo.y;
          const float T0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Tw), l));
          float d2 = __builtin_fmaf(dx, dx, dy * dy), x = r.geo.w * d2, l2 = r.geo.z;
          if (ANI && pc.w == 2.0f) {
            const float a = __builtin_fmaf(dx, r.geo.z, dy * r.geo.w);
            const float b = __int_as_float(r.g) * __builtin_fmaf(dy, r.geo.z, -(dx * r.geo.w));
            d2 = __builtin_fmaf(a, a, b * b);
            x = -d2;
            l2 = lim;
          }
          const bool in = lane < n && d2 <= l2;
          const float f = 1.0f - fminf(amax, r.op * __builtin_amdgcn_exp2f(x));
          const float Tn = T0 * wave_scan_product(in ? f : 1.0f);
          const uint64_t dead = __ballot(in && Tn < eps), some = __ballot(in);
          const int at = dead ? __builtin_ctzll(dead) : (some ? 63 - __builtin_clzll(some) : 0);
          const float Tp =
              __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(T0), __float_as_int(Tn), 0x138, 0xf, 0xf, false));
          const float d = lane <= at ? Tp - Tn : 0.0f;
          float tot;
          if constexpr (C == 3) {
            const float v[3] = {pc.x * d, pc.y * d, pc.z * d};
            tot = wave_totals_to_lanes<3>(v);
          } else {
            const float v[1] = {pc.x * d};
            tot = wave_totals_to_lanes<1>(v);
          }
          if (lane == at) {
            L.stopT[l] = fminf(Tn, under);
            L.stopP[l] = r.pos;
          }
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tot), c));
            con[c] = lane == l ? a : con[c];
          }
        }
      }
    } else {
      // one share after another
      for (int k = 0; k < FW; ++k) {
        if (k == wv) {
          t = T;
          composite(std::true_type{});
#pragma unroll
          for (int c = 0; c < C; ++c) con[c] = ca[c];
          if (sp >= 0) {
            L.stopT[lane] = t;
            L.stopP[lane] = sp;
          }
          L.prod[0][lane] = sp >= 0 ? -1.0f : t;
        }
        __syncthreads();
        T = L.prod[0][lane];
        put_T(whi, k, T);
        __syncthreads();
      }
    }
    // the colours: wavefront c sums channel c over the shares, group by group,
    // and stores what each chunk that ends here contributed
    __syncthreads();  // every wavefront is done with the window's entries
#pragma unroll
    for (int c = 0; c < C; ++c) sums[(wv * C + c) * 64 + lane] = con[c];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < FW; k += group) {
      if (wv < C) {
        float a = 0.0f;
#pragma unroll
        for (int u = k; u < k + group; ++u) a += sums[(u * C + wv) * 64 + lane];
        tail += a;
        tot += a;
      }
      const int lo = whi - 64 * (k + group);
      if (!boundary(lo)) continue;
      if (wv < C) ck_at(lo)[(1 + wv) * TILE * TILE] = tail;
      tail = 0.0f;
      ++n_ck;
    }
    if (__ballot(T >= eps) == 0ull) break;  // every pixel of the quadrant has stopped
  }
  // Suffix sums over the chunks, back to front, as in fwd_serial.  Wavefront c
  // takes channel c and rereads only the slots that it wrote; the last one
  // writes T and the positions.
  __syncthreads();
  const int64_t plane = (int64_t)im.st.H * im.st.W;
  const int x = x0 + lx, y = y0 + ly;
  const bool inside = x < im.st.W && y < im.st.H;
  const int64_t at = (int64_t)y * im.st.W + x;
  float Tq = T;
  int stop = start;
  if (inside && !(Tq >= eps)) {
    Tq = L.stopT[lane];
    stop = L.stopP[lane];
  }
  if (wv < C) {
    float a = tail;
    for (int k = n_ck; k >= 1; --k) {
      float* ckp = w.ckbuf + (int64_t)(ck0 + k - 1) * (4 * TILE * TILE) + (1 + wv) * TILE * TILE;
      const float ch = ckp[slot];
      ckp[slot] = a;
      a += ch;
    }
    if (inside) image[(int64_t)im.st.pix_off * C + wv * plane + at] = __builtin_fmaf(Tq, bg[im.s * C + wv], tot);
  }
  if (wv == FW - 1 && inside) {
    Tfin[(int64_t)im.st.pix_off + at] = Tq;
    nlast[(int64_t)im.st.pix_off + at] = stop;
  }
}

struct FwdSerialLds {
  FwdRec rec[WPB * 64 * FWD_ENTRY_BYTES / sizeof(FwdRec)];
  int next;
};

// SPLIT: the first n_long tiles of the blend order (the binning's choice) take a
// block per quadrant, the others a wavefront per quadrant, eight to a block.
// Otherwise every quadrant takes a wavefront, four to a block, in a form of its
// own: fwd_serial alone waits for the longest list, where registers for eight
// entries in flight count and a fifth wavefront per SIMD does not.  With a given
// chunk, in the split form's registers (79), held to five wavefronts (72) and to
// four (107): 12 quintic strokes at 512^2 0.470, 0.428, 0.378 ms, 16 closed ones
// 0.077, 0.072, 0.065; 16 x 2000 key points at 1024^2, which fill the GPU, 0.298,
// 0.274, 0.295.
template <int C, int TILE, int KIND, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? FWD_BLOCK : BLOCK, SPLIT && !(KIND & KIND_FILL) ? 6 : 4) void k_blend_fwd(
    nsplat_params pr, Work w, int n_scenes, int n_tiles, const Gauss* __restrict__ gs,
    const int32_t* __restrict__ ranges, const int32_t* __restrict__ idx, const float* __restrict__ bg,
    float* __restrict__ image, float* __restrict__ Tfin, int32_t* __restrict__ nlast, const int32_t* __restrict__ plan,
    int64_t gcap, int persistent, int ck_arg) {
  using Cfg = TileCfg<TILE>;
  __shared__ __align__(16) std::conditional_t<SPLIT, FwdLds, FwdSerialLds> L;
  typedef const __attribute__((address_space(4))) int32_t* const_i32;
  // the chunk length: the caller's, or the one the binning chose
  const int ck_lg = ck_arg >= 0 ? ck_arg : ((const_i32)w.queue)[Q_CKLG];
  // fill runs at h = 1 walk each pixel's lattice neighbours (see FillRun);
  // the support radius must be the 4.5 the offsets are laid out for
  const bool fill_lattice = (KIND & KIND_FILL) != 0 && read_h(pr) == 1.0f;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_items = n_tiles * Cfg::QUADS;
  constexpr int wpb = SPLIT ? FW : WPB;
  const int n_long = !SPLIT || fill_lattice ? 0 : min(max(((const_i32)w.queue)[Q_NLONG], 0), n_tiles) * Cfg::QUADS;
  for (int it = 0;; ++it) {
    int b = blockIdx.x;
    if (persistent) {
      __syncthreads();
      if (threadIdx.x == 0) L.next = atomicAdd(w.queue, 1);
      __syncthreads();
      b = __builtin_amdgcn_readfirstlane(L.next);
    } else if (it > 0) {
      break;
    }
    const bool whole = b < n_long;
    if (!whole && n_long + (int64_t)(b - n_long) * wpb >= n_items) break;
    const int item = whole ? b : n_long + (b - n_long) * wpb + wv;
    if (item >= n_items) continue;
    FwdItem im;
    const int tq = item / Cfg::QUADS;
    im.quad = item - tq * Cfg::QUADS;
    im.tile = w.order[tq];
    im.s = scene_of_tile(w.scenes, n_scenes, im.tile);
    im.st = w.scenes[im.s];
    im.lt = im.tile - im.st.tile_off;
    im.x0 = (im.lt % im.st.tiles_x) * TILE;
    im.y0 = (im.lt / im.st.tiles_x) * TILE;
    im.start = ranges[2 * im.tile];
    im.end = ranges[2 * im.tile + 1];
    if constexpr (SPLIT) {
      if (whole) {
        fwd_block<C, TILE, KIND>(pr, w, im, gs, idx, bg, image, Tfin, nlast, ck_lg, L);
        continue;
      }
    }
    fwd_serial<C, TILE, KIND>(pr, w, im, gs, idx, bg, image, Tfin, nlast, plan, gcap, ck_lg, fill_lattice,
                              (char*)L.rec + wv * (64 * FWD_ENTRY_BYTES));
  }
}

// Minimum over the wavefront: running minima inside each row of 16 lanes by
// DPP row shifts (a lane with no source keeps its own value), then the four
// rows' last lanes.  Needs no per-lane shuffle addresses.
__device__ inline int wave_min(int v) {
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));  // row_shr:1
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));  // row_shr:2
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));  // row_shr:4
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));  // row_shr:8
  return min(min(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31)),
             min(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63)));
}

// Folds one wavefront's running FP32 per-curve sums into `tot`, whose lane 0
// keeps the FP64 opacity gradient of a stroke curve and lane 1 + ch the colour
// gradient of channel ch, dL/dI_c sum(alpha T) (aT: the pixel's sum
// of alpha T over the run, reset here).  `tot` goes to the curve's
// accumulators once, where the wavefront's run of the curve ends
// (flush_curve): with an atomic every FLUSH stroke entries a launch of few
// curves queued up on their few addresses (one curve of 10,240 key points at
// 1024^2, 2.0M pairs: adjoint 1.30 ms, now 0.39 ms).
template <int C>
__device__ inline void fold_curve(bool fill, const float (&gI)[3], float& aT, float& accO, double& tot) {
  float v[C + 1];
  v[0] = fill ? 0.0f : accO;
#pragma unroll
  for (int ch = 0; ch < C; ++ch) v[1 + ch] = gI[ch] * aT;
  aT = 0.0f;
  accO = 0.0f;
  tot += (double)wave_totals_to_lanes<C + 1>(v);
}

template <int C>
__device__ inline void flush_curve(double* gcurve, int c, double& tot) {
  const int lane = __lane_id();
  if (lane <= C && tot != 0.0) unsafeAtomicAdd(gcurve + 4 * (int64_t)c + lane, tot);
  tot = 0.0;
}

// Sums the first n (<= RB) parked rows over the 64 lanes and adds each total
// to its target ggrad[g * GG + value] (tgt[row] = (g, value)).  Lane (r, part)
// = (lane / 4, lane % 4) adds up floats part, part + 4, ..., part + 60 of row
// r; two DPP row shifts finish the sum in the quad's last lane, which issues
// the atomic.  Every lane of the wavefront must call it.
__device__ inline void flush_rows(const float* park, const int2* tgt, int n, float* __restrict__ ggrad) {
  static_assert(RB <= 16, "four lanes per parked row");
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int lane = __lane_id(), r = lane >> 2, part = lane & 3;
  const float* row = park + r * RB_ROW + part;
  float t = 0.0f;
#pragma unroll
  for (int j = 0; j < 16; ++j) t += row[4 * j];
  t += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0x111, 0xf, 0xf, true));  // row_shr:1
  t += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0x112, 0xf, 0xf, true));  // row_shr:2
  if (part == 3 && r < n && t != 0.0f) {
    const int2 tg = tgt[r];
    unsafeAtomicAdd(ggrad + (int64_t)tg.x * GG + tg.y, t);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Basis table of flush_moments: function f of lane p at table[f * RB_ROW + p]:
// 1, x, y, x^2 + y^2 with (x, y) = (p & 7, p >> 3) - 3.5, the lane's pixel
// relative to the middle of its 8 x 8 block.  One thread per entry.
__device__ inline void basis_table(float* table) {
  static_assert(BLOCK == 256, "one thread per basis value");
  const int f = threadIdx.x >> 6, p = threadIdx.x & 63;
  const float x = (float)(p & 7) - 3.5f, y = (float)(p >> 3) - 3.5f;
  table[f * RB_ROW + p] = f == 0 ? 1.0f : (f == 1 ? x : (f == 2 ? y : x * x + y * y));
}

// Lane 4 (l / 4) + Q's value of v (quad_perm broadcast).
template <int Q>
__device__ inline double quad_bcast(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  constexpr int ctrl = Q * 0x55;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, ctrl, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), ctrl, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Per-Gaussian gradients of up to RB entries (e0 .. e0 + n - 1 of the
// wavefront's LDS arrays) of a block with one pixel per lane, from their
// parked rows: row i holds, per lane, entry e0 + i's v = dL/dalpha G.  Every
// gradient of an isotropic Gaussian is a fixed combination of four sums over
// the pixels, sum v {1, x, y, x^2 + y^2} (x, y relative to the block's middle
// (mx, my)):
//   dL/dmu    = -2 ln2 a o  sum v (x - mu),     a the exp2 coefficient
//   dL/dsigma = o / sigma^3 sum v |x - mu|^2
//   dL/do_j   = sum v (fills)
// so the rows contract with the 64 x 4 basis, 16 rows at a time, on the matrix
// cores: v_mfma_f64_4x4x4, whose four blocks take four rows each.  Lane l holds
// row l & 15 in A and function l & 3 in B at pixels 16 (l >> 4) + t for step t,
// and receives function l & 3 of row 4 ((l >> 2) & 3) + (l >> 4); quad
// broadcasts give it all four sums of that row, of which it forms gradient
// value l & 3, and one atomic instruction adds them all.  An entry's lanes only form v and store it, where they formed and
// stored dL/dmu and dL/dsigma each before (adjoint of 16 closed strokes at
// 512^2 0.132 -> 0.076 ms, of 16 x 2000 key points at 1024^2 0.940 -> 0.705 ms).
// In FP64, because moving the sums to the Gaussian's centre cancels: in FP32
// (0.076, 0.726 ms, v_mfma_f32_16x16x4) the knot-interval gradients of long splines, themselves
// sums that cancel, were ten times further from the exact ones.
// A disc of a radius below a half (gm.z < 0.2, with a margin for the rounding of
// the pixels' own tests) reaches one pixel at most: there sum v |x - mu|^2 is
// |sum v (x - mu)|^2 / sum v, while the moved sum keeps 1e-15 px^2, which may be
// more than sigma^2; and with no pixel nothing is added, also where the factors
// (1 / sigma^3 from sigma = 1.4e-13 down) are infinite.  Every lane of the
// wavefront must call it.
__device__ inline void flush_moments(const float* park, const float* basis, const float4* geo, const int4* meta,
                                     int e0, int n, float mx, float my, float* __restrict__ ggrad) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int lane = __lane_id();
  const f4* ap = (const f4*)(park + (lane & 15) * RB_ROW + 16 * (lane >> 4));
  const f4* bp = (const f4*)(basis + (lane & 3) * RB_ROW + 16 * (lane >> 4));
  double m = 0.0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const f4 a = ap[s], b = bp[s];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      m = __builtin_amdgcn_mfma_f64_4x4x4f64((double)a[t], (double)b[t], m, 0, 0, 0);
  }
  const int e = 4 * ((lane >> 2) & 3) + (lane >> 4), val = lane & 3;
  const bool ok = e < n;
  const float4 gm = geo[e0 + (ok ? e : 0)];
  const int4 mt = meta[e0 + (ok ? e : 0)];
  const double M0 = quad_bcast<0>(m), Mx = quad_bcast<1>(m), My = quad_bcast<2>(m), Mr = quad_bcast<3>(m);
  const double cx = (double)gm.x - (double)mx, cy = (double)gm.y - (double)my;
  const double Ax = __builtin_fma(-cx, M0, Mx), Ay = __builtin_fma(-cy, M0, My);
  const double Ar = __builtin_fma(-cy, My + Ay, __builtin_fma(-cx, Mx + Ax, Mr));
  const float op = __int_as_float(mt.z);
  const float k1 = -2.0f * (float)LN2 * gm.w * op, k2 = op * __int_as_float(mt.w);
  const double A = val == 0 ? Ax : (val == 1 ? Ay : Ar);
  float v = mt.x < 0 ? (float)M0 : (val == 2 ? k2 : k1) * (float)A;
  const bool thin = gm.z < 0.2f && mt.x >= 0;
  if (__ballot(thin) != 0ull) {
    if (thin && val == 2) v = k2 * (float)(__builtin_fma(Ax, Ax, Ay * Ay) * __builtin_amdgcn_rcp(M0));
    if (thin && M0 == 0.0) v = 0.0f;
  }
  // strokes take values 0..2, fills value 3
  if (ok && ((val == 3) == (mt.x < 0)) && v != 0.0f)
    unsafeAtomicAdd(ggrad + (int64_t)(mt.x < 0 ? ~mt.x : mt.x) * GG + val, v);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adjoint of the forward blend, one work item per (tile, quadrant, chunk).
// Inside its chunk an item walks back to front, starting from the state the
// forward stored at the chunk's back end (T there, and the colour of
// everything behind it), or from T_final for a pixel that stopped inside the
// chunk.  With K = sum_c dL/dI_c col_c of an entry and B the loss-weighted
// colour behind it, Eq. 8 gives
//   dL/dalpha = T K - B / (1 - alpha),   T the transmittance in front of it.
// Walking back to front, B grows by K alpha T = K (T - T') from each entry
// (T' = T (1 - alpha), the transmittance behind it), and T is recovered as
// T = T' / (1 - alpha).  Over a run of one curve's entries K is fixed, so
// W = B - K T' does not change, and dL/dalpha = -W / (1 - alpha); W is
// re-expressed where K changes.  B is built from the back, a sum of the terms
// behind the entry, so its rounding stays relative to the colour actually
// behind (a front-to-back form B = R - U loses it where T is small).  Per
// Gaussian it accumulates dL/dmu and dL/dsigma for stroke Gaussians and
// dL/do_j for fill Gaussians (whose own opacity carries the SDF); colour
// gradients (and a stroke curve's opacity gradient, its o_j all being o)
// belong to the curve, so each lane keeps running per-curve sums that are
// flushed when the curve changes along the list (and for strokes folded into
// FP64 every FLUSH entries).  The entries of a step are cut into runs of one curve with one
// ballot, and each run is composited by a loop for its kind, with no
// per-entry curve test.  Occupancy: bwd_waves.
template <int C, int TILE, int E, int KIND>
__global__ __launch_bounds__(BLOCK, bwd_waves(E, KIND)) void k_blend_bwd(
    nsplat_curves cv, nsplat_params pr, Work w, int n_scenes, int n_tiles, const Gauss* __restrict__ gs,
    const int32_t* __restrict__ ranges, const int32_t* __restrict__ idx, const float* __restrict__ bg,
    const float* __restrict__ dL, const float* __restrict__ Tfin, const int32_t* __restrict__ nlast,
    const int32_t* __restrict__ plan, int64_t gcap, int persistent, int pop_from, int ck_arg) {
  constexpr int FLUSH = 32;
  extern __shared__ __align__(16) char smem[];
  typedef const __attribute__((address_space(4))) int32_t* const_i32;
  const int ck_lg = ck_arg >= 0 ? ck_arg : ((const_i32)w.queue)[Q_CKLG];
  const int depth = min(pr.batch, 64 * E);
  const float amax = pr.alpha_max, ks = pr.k_sigma;
  const float ln2 = (float)LN2;
  constexpr bool ANI = (KIND & KIND_ANI) != 0, LONG = (KIND & KIND_LONG) != 0;
  // fill runs pixel by pixel (see FillRun)
  const bool fill_lattice = (KIND & KIND_FILL) != 0 && read_h(pr) == 1.0f;
  const float inv_tile = 1.0f / (float)TILE;
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  float* basis = (float*)smem;  // (shared by the block's wavefronts)
  basis_table(basis);
  __syncthreads();
  char* mine_lds = smem + BASIS_BYTES + (size_t)wv * bwd_wave_bytes(E);
  float4* wgeo = (float4*)mine_lds;
  int4* wmeta = (int4*)(wgeo + 64 * E);  // (g, or ~g for fills), list position, opacity bits, 1/sigma^3 bits
  float4* wpc = (float4*)(wmeta + 64 * E);  // colour, curve bits
  float* park = (float*)(wpc + 64 * E);  // [RB][RB_ROW] parked gradient values
  int2* ptgt = (int2*)(park + RB * RB_ROW);  // [RB] targets of flush_rows
  const uint64_t below = lanes_below();
  float* __restrict__ ggrad = w.ggrad;
  const const_i32 taus = (const_i32)cv.tau_off;
  const const_i32 item_off = (const_i32)w.item_off;  // not written during the kernel: scalar loads
  const int n_items = item_off[n_tiles];
  // All wavefronts take their items from one address, which gives one every 12 ns:
  // with 24 items or more per wavefront slot (16 slots per compute unit: pop_from)
  // that is what the launch waits for, and they take four at a time (with fewer,
  // four long ones in one wavefront would be waited for).  16 mixed scenes at 768^2
  // in 32 x 32 tiles, one by one and by fours: chunks of 512 (196,000 items) 2.40 and
  // 1.22 ms (1.76 in the quadrants of 16 x 16 pixels, a quarter of the items), of
  // 1024 (113,000) 1.49 and 1.20, of 2048 (75,000) 1.17 and 1.18, of 4096 (58,000)
  // 1.09 and 1.30; 16 x 2000 key points at 1024^2 (120,000) 1.54 and 0.79.
  const int pop = persistent && n_items >= pop_from ? 4 : 1;
  int item = 0, left = 0;  // items of the last pop still to take
  for (int it = 0;; ++it) {
    if (left > 0) {
      ++item;
      --left;
    } else {
      item = next_item(it, persistent, w.queue, pop);
      left = pop - 1;
    }
    if (item >= n_items) break;
    // blend-order position of the item's tile: the last i with item_off[i] <= item
    int tq = 0;
    {
      int lo_t = 0, hi_t = n_tiles - 1;
      while (lo_t < hi_t) {
        const int mid = (lo_t + hi_t + 1) >> 1;
        if (item_off[mid] <= item) lo_t = mid;
        else hi_t = mid - 1;
      }
      tq = lo_t;
    }
    const int r_it = item - item_off[tq];
    const int tile = w.order[tq];
    const int s = scene_of_tile(w.scenes, n_scenes, tile);
    const SceneTab st = w.scenes[s];
    using Cfg = TileCfg<TILE>;
    const int quad = r_it % Cfg::QUADS, kc = r_it / Cfg::QUADS;
    const int qx = (quad % Cfg::COLS) * Cfg::SUB, qy = (quad / Cfg::COLS) * Cfg::SUB;  // the block's first pixel
    const int lt = tile - st.tile_off;
    const int x0 = (lt % st.tiles_x) * TILE, y0 = (lt / st.tiles_x) * TILE;
    const int start = ranges[2 * tile], end = ranges[2 * tile + 1];
    const int c_hi = end - (kc << ck_lg), c_lo = max(start, end - ((kc + 1) << ck_lg));  // the chunk's positions
    const int64_t plane = (int64_t)st.H * st.W;
    // the forward's state at the chunk's back end (the front of chunk kc + 1),
    // stored when a chunk follows
    const float* ckn = c_lo > start ? w.ckbuf + (int64_t)(w.ck_off[tile] + kc) * (4 * TILE * TILE) : nullptr;
    int lx, ly;
    pixel_of<TILE>(quad, lane, &lx, &ly);
    const float px = (float)lx, py = (float)ly;
    float T = 1.0f, Wc = 0.0f, gI[3] = {0.0f, 0.0f, 0.0f};
    int stop = end;  // invalid pixels never take part
    if (x0 + lx < st.W && y0 + ly < st.H) {
      const int64_t pix = (int64_t)st.pix_off + (int64_t)(y0 + ly) * st.W + (x0 + lx);
      const float tf = Tfin[pix];
      stop = nlast[pix];
      // a pixel still live behind this chunk starts from the stored state,
      // one that stopped inside it from T_final with only the background
      // behind it (no chunk is stored after a pixel's stop is passed)
      const int slot = quad * 64 + lane;
      float behind[3] = {0.0f, 0.0f, 0.0f};
      T = tf;
      if (stop < c_lo) {  // then c_lo > start, so a chunk follows and ckn is set
        T = ckn[slot];
#pragma unroll
        for (int c = 0; c < C; ++c) behind[c] = ckn[(1 + c) * TILE * TILE + slot];
      }
      float B = 0.0f;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int64_t o = (int64_t)st.pix_off * C + c * plane + (int64_t)(y0 + ly) * st.W + (x0 + lx);
        gI[c] = dL[o];
        B = __builtin_fmaf(gI[c], __builtin_fmaf(tf, bg[s * C + c], behind[c]), B);
      }
      Wc = B;  // W = B - K T' with no curve yet (K = 0)
    }
    // positions below every pixel's stopping position take no part
    const int lo = max(wave_min(stop), c_lo);
    if (c_hi <= lo) continue;
    int cur = -1, since = 0;
    bool cur_fill = false, cur_aniso = false, cur_long = false;
    // per pixel: K of the current curve, W (fixed over a run of one curve),
    // and the run's sum of alpha T (the curve's colour gradient is dL/dI_c
    // times it)
    float Kc = 0.0f, aT = 0.0f, accO = 0.0f;
    double ctot = 0.0;  // the open run's curve sums (fold_curve)
    // the end of the run of curve `cur`
    auto close_curve = [&]() {
      if (cur < 0) return;
      fold_curve<C>(cur_fill, gI, aT, accO, ctot);
      flush_curve<C>(w.gcurve, cur, ctot);
    };
    // the parked rows of the n entries before entry j
    auto flush_pending = [&](int j, int n) {
      flush_moments(park, basis, wgeo, wmeta, j - n, n, (float)qx + 3.5f, (float)qy + 3.5f, ggrad);
    };
    const double ox = (double)x0 + 0.5, oy = (double)y0 + 0.5;
    // back to front over the chunk's positions lo up to c_hi - 1, in steps
    // of `depth` (each lane loads one entry per 64 of a step)
    Entry e[E];
    int s_lo = lo, s_hi = min(c_hi, lo + depth);
#pragma unroll
    for (int u = 0; u < E; ++u) {
      const int k = u * 64 + lane;
      load_entry(idx, gs, w.gcol, s_lo + k, k < s_hi - s_lo, &e[u]);
    }
    // One fill run's positions p0 .. p1 at h = 1, back to front for each
    // pixel over its in-disc lattice neighbours (the reverse of the forward's
    // walk), with the per-pixel arithmetic of the entry-by-entry path; each
    // Gaussian's dL/do_j is summed over the lanes in LDS and added with one
    // atomic.
    constexpr int BNB = Cfg::SUB + 2 * FR_R;  // lattice neighbourhood of the pixel block, per axis
    constexpr int BNIT = (BNB * BNB + 63) / 64;
    auto fill_run_bwd = [&](const FillRun& fr, const float (&col)[3], int p0, int p1, const float (&og)[BNIT]) {
      constexpr int NB = BNB;                  // 16 cells per axis
      constexpr int NS = FR_NS;                // LDS row stride (conflict-free rows)
      float* ol = (float*)mine_lds;  // [NB][NS] opacities (0: no Gaussian at p0 .. p1 there)
      float* gl = park;              // [NB][NS] dL/do_j
      if (cur != fr.c) {  // a new curve: close the previous one, W for the new K
        close_curve();
        float K = 0.0f;
#pragma unroll
        for (int ch = 0; ch < C; ++ch) K = __builtin_fmaf(gI[ch], col[ch], K);
        Wc = __builtin_fmaf(-K, T, __builtin_fmaf(Kc, T, Wc));
        Kc = K;
        cur = fr.c;
        cur_fill = true;
        cur_aniso = false;
        since = 0;
      }
      const int ib = x0 + qx - fr.ix0 - FR_R, jb = y0 + qy - fr.iy0 - FR_R;  // window index of cell (0, 0)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // an absent cell composites as a zero opacity (alpha 0, T unchanged);
      // its dL/do_j sum is dropped by the presence bits
      int pm = 0;
#pragma unroll
      for (int it = 0; it < BNIT; ++it) {
        const int sl = it * 64 + lane;
        if (sl < NB * NB) {
          const bool pres = og[it] == og[it];
          ol[(sl / NB) * NS + sl % NB] = pres ? og[it] : 0.0f;
          gl[(sl / NB) * NS + sl % NB] = 0.0f;
          pm |= (int)pres << it;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const double sgd = (double)fr.sigma;
      const float coef = (float)(-0.5 * LOG2E / (sgd * sgd));  // as entry_geometry
      // lane k holds G at squared lattice distance k, as the entry path forms it
      const int gtab = __float_as_int(__builtin_amdgcn_exp2f(coef * (float)lane));
      const float nW = -Wc;  // dL/dalpha (1 - alpha) over the run
      const int lx = lane & 7, ly = lane >> 3;
      const bool col0 = lx == 0, col7 = lx == 7;
      const int pb0 = fr.p_lo + (y0 + qy + ly - fr.iy0 - fr.j0) * fr.w + (x0 + qx + lx - fr.ix0 - fr.i0);
#pragma unroll 1
      for (int dy = -FR_R; dy <= FR_R; ++dy) {
        const int dxm = dy * dy <= 4 ? 4 : (dy * dy == 9 ? 3 : 2);  // dx^2 + dy^2 <= FR_R2
        const int roff = (ly + dy + FR_R) * NS + lx + FR_R;         // this pixel's cell in row dy
        const int rpos = pb0 + dy * fr.w;
        {
          // a row with no Gaussian of p0 .. p1 at or in front of any pixel's
          // stop adds nothing
          const int jr = y0 + qy + ly + dy - fr.iy0, ir = x0 + qx + lx - fr.ix0;
          const bool any = jr >= fr.j0 && jr <= fr.j1 && ir + dxm >= fr.i0 && ir - dxm <= fr.i1 &&
                           rpos + dxm >= max(p0, stop) && rpos - dxm <= p1;
          if (__ballot(any) == 0ull) continue;
        }
        // the row's opacities first, one LDS wait per row (each becomes the
        // cell's dL/do_j in place), and its five Gaussian factors
        float v[2 * FR_R + 1], Gr[FR_R + 1];
#pragma unroll
        for (int dx = -FR_R; dx <= FR_R; ++dx) v[dx + FR_R] = ol[roff + dx];
#pragma unroll
        for (int a = 0; a <= FR_R; ++a) Gr[a] = __int_as_float(__builtin_amdgcn_readlane(gtab, a * a + dy * dy));
        const int sd = stop - rpos;  // cells at dx >= sd lie at or behind the pixel's stop
#pragma unroll
        for (int dx = -FR_R; dx <= FR_R; ++dx) {
          const float o = v[dx + FR_R];
          v[dx + FR_R] = 0.0f;
          if (dx > dxm || dx < -dxm) continue;
          // a cell in front of the stop takes part with G = 0: alpha 0, T
          // and alpha T unchanged, no gradient
          const float G = dx >= sd ? Gr[dx < 0 ? -dx : dx] : 0.0f;
          const float oG = o * G;
          const bool lt = oG < amax;
          const float alpha = fminf(oG, amax);  // lt ? oG : amax, also for a NaN oG
          const float r = __builtin_amdgcn_rcpf(1.0f - alpha);
          T *= r;
          aT = __builtin_fmaf(alpha, T, aT);
          v[dx + FR_R] = lt ? nW * r * G : 0.0f;  // dL/do_j of the cell at dx
        }
        // the row's cells get their sums over the pixels of each lane row
        // by two sliding sums along the row (DPP shifts by one lane, 8-lane
        // groups kept apart): P ends with cell lx - 4, Q with cell lx + 4
        float P = v[2 * FR_R], Q = v[0];
#pragma unroll
        for (int k = 1; k <= 2 * FR_R; ++k) {
          const float ps = col7 ? 0.0f : P, qs = col0 ? 0.0f : Q;
          P = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(ps), 0x111, 0xf, 0xf, true)) +
              v[2 * FR_R - k];  // row_shr:1
          Q = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(qs), 0x101, 0xf, 0xf, true)) +
              v[k];  // row_shl:1
        }
        const int crow = (ly + dy + FR_R) * NS;  // cell row of this lane row
        gl[crow + lx] += P;                      // cell column lx - 4
        gl[crow + lx + 2 * FR_R] += Q;           // cell column lx + 4
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int it = 0; it < (NB * NB + 63) / 64; ++it) {
        const int sl = it * 64 + lane;
        if (sl >= NB * NB) continue;
        const float val = gl[(sl / NB) * NS + sl % NB];
        if (((pm >> it) & 1) && val != 0.0f) {
          const int j = jb + sl / NB, i = ib + sl % NB;
          unsafeAtomicAdd(ggrad + ((int64_t)fr.goff + (int64_t)j * fr.nx + i) * GG + 3, val);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    while (s_lo < c_hi) {
      if (fill_lattice && __builtin_amdgcn_readfirstlane(e[0].kind()) == 1) {
        // the next entry (position s_lo, lane 0's first) is a fill Gaussian:
        // take its run's positions in this chunk pixel by pixel
        FillRun fr;
        const int c = __builtin_amdgcn_readfirstlane(e[0].r.curve);
        const float sg = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, e[0].r.sigma)));
        const float rr = ks * sg;
        float og[BNIT];
        bool take = false;
        const int p0 = s_lo;
        int p1 = 0;
        if (rr * rr >= (float)FR_R2 && rr * rr < (float)(FR_R2 + 5) &&
            fill_run_at(PlanRowScalar(plan, c), c, __builtin_amdgcn_readfirstlane(e[0].g),
                        __builtin_amdgcn_readfirstlane(e[0].r.local), sg, s_lo, start, end, 1.0, ks, inv_tile, st, lt,
                        TILE, &fr)) {
          // the opacities and the corner check in flight together
          p1 = min(fr.p_hi, c_hi - 1);
          const int ib = x0 + qx - fr.ix0 - FR_R, jb = y0 + qy - fr.iy0 - FR_R;
          fill_gather<BNB, BNIT>(w.gop, gcap, fr, ib, jb, s_lo, p1, __builtin_nanf(""), og);
          take = fill_corners_ok(idx, fr);
        }
        if (take) {
          const float col[3] = {first_lane(e[0].cf.x), first_lane(e[0].cf.y), first_lane(e[0].cf.z)};
          // the next step's loads in flight during the walk
          s_lo = p1 + 1;
          s_hi = min(c_hi, s_lo + depth);
#pragma unroll
          for (int u = 0; u < E; ++u) {
            const int k = u * 64 + lane;
            load_entry(idx, gs, w.gcol, s_lo + k, k < s_hi - s_lo, &e[u]);
          }
          fill_run_bwd(fr, col, p0, p1, og);
          continue;
        }
      }
      int cnt = 0;
      // pixels that take part somewhere in this step (their stop lies below
      // its top); walking back to front the set only grows.  Entries that
      // reach none of them are dropped.
      bool step_aniso = false;
      const Box box = live_box_of(qx, qy, __ballot(stop < s_hi));
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const int k = u * 64 + lane;
        const int mypos = s_lo + k;
        const bool ok = k < s_hi - s_lo;
        float4 geo;
        const bool keep = ok && entry_geometry(e[u].r, ox, oy, ks, box, &geo);
        const uint64_t m = __ballot(keep);
        if (ANI) step_aniso = step_aniso || __ballot(keep && e[u].kind() == 2) != 0ull;
        if (keep) {
          entry_support(e[u].r, ks, &geo);
          const int dst = cnt + __popcll(m & below);
          const double sg = (double)e[u].r.sigma;
          // tangent-aligned entries: -1 (negative: the kind) in place of 1 / sigma^3
          const float wbits = (ANI && e[u].kind() == 2) ? -1.0f : (float)(1.0 / (sg * sg * sg));
          wgeo[dst] = geo;
          wmeta[dst] = make_int4(e[u].kind() == 1 ? ~e[u].g : e[u].g, mypos, __float_as_int(e[u].r.opacity),
                                 __float_as_int(wbits));
          wpc[dst] = make_float4(e[u].cf.x, e[u].cf.y, e[u].cf.z, __int_as_float(e[u].r.curve));
        }
        cnt += __popcll(m);
      }
      const int n_lo = s_hi, n_hi = min(c_hi, s_hi + depth);
#pragma unroll
      for (int u = 0; u < E; ++u) {  // next step, in flight while this one is processed
        const int k = u * 64 + lane;
        load_entry(idx, gs, w.gcol, n_lo + k, k < n_hi - n_lo, &e[u]);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (ANI && step_aniso) {
        // tangent-aligned entries of the step take their axis u (in place of
        // the support radius and coefficient) and -r (in place of the kind)
        for (int i = lane; i < cnt; i += 64) {
          const int4 mt = wmeta[i];
          if (mt.x < 0 || mt.w >= 0) continue;
          const float4 ax = w.gaux[mt.x];
          float ux, uy, rq;
          aniso_axes(ax, wgeo[i].w, &ux, &uy, &rq);
          wgeo[i].z = ux;
          wgeo[i].w = uy;
          wmeta[i].w = __float_as_int(-rq);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      // entries that begin a run (their curve differs from the entry processed
      // before them, the first one compared with the previous step's curve)
      uint64_t rs[E];
#pragma unroll
      for (int g = 0; g < E; ++g) {
        const int i = 64 * g + lane;
        const int prev = i == 0 ? cur : __float_as_int(wpc[i > 0 ? i - 1 : 0].w);
        rs[g] = __ballot(i < cnt && __float_as_int(wpc[i < cnt ? i : 0].w) != prev);
      }
      int n_ent = 0;  // entries with parked rows: the n_ent before j (wavefront-uniform)
      for (int j = 0; j < cnt;) {
        // this segment: j up to the next run start (or the step's end)
        int jend = cnt;
#pragma unroll
        for (int g = E - 1; g >= 0; --g) {
          const int b = j + 1 - 64 * g;  // first bit of group g after j
          const uint64_t m = b <= 0 ? rs[g] : (b < 64 ? rs[g] & (~0ull << b) : 0ull);
          if (m) jend = 64 * g + __builtin_ctzll(m);
        }
        if ((rs[j >> 6] >> (j & 63)) & 1ull) {  // a new curve: close the previous one
          close_curve();
          const int4 mt = wmeta[j];
          const float4 pc = wpc[j];
          const float col[3] = {pc.x, pc.y, pc.z};
          float K = 0.0f;
#pragma unroll
          for (int c = 0; c < C; ++c) K = __builtin_fmaf(gI[c], col[c], K);
          // B = W + K_old T' is unchanged; W re-expressed with the new K
          Wc = __builtin_fmaf(-K, T, __builtin_fmaf(Kc, T, Wc));
          Kc = K;
          cur = __builtin_amdgcn_readfirstlane(__float_as_int(pc.w));
          cur_fill = __builtin_amdgcn_readfirstlane(mt.x) < 0;
          cur_aniso = ANI && !cur_fill && __builtin_amdgcn_readfirstlane(mt.w) < 0;
          cur_long = LONG && !cur_fill && taus[cur + 1] - taus[cur] > LONG_TAUS;
          since = 0;
        }
        if (ANI && cur_aniso) {
          // tangent-aligned stroke Gaussians: dL/dmu (2), dL/dsigma, dL/dsp
          // and dL/dtheta (t = (cos theta, sin theta)) parked in five rows.
          // With h = dL/dG G / ck: dG/dmu = (a u - b r u^perp) 2 ln 2 G, and so
          // on (the partials of exp(-(d_t^2 / sigma^2 + d_n^2 / sp^2) / 2)
          // rewritten in a, b).
          const float lim = ANI_CK * ks * ks;
          const float two_ln2 = 2.0f * ln2;
          if (n_ent > 0) flush_pending(j, n_ent);  // the rows are shared
          n_ent = 0;
          int n_rows = 0;
          for (; j < jend; ++j) {
            if (since >= FLUSH) {
              fold_curve<C>(false, gI, aT, accO, ctot);
              since = 0;
            }
            ++since;
            const float4 gm = wgeo[j];
            const int4 mt = wmeta[j];
            const float op = __int_as_float(mt.z);
            const float rq = -__int_as_float(mt.w);
            const float isg = __builtin_sqrtf(__builtin_fmaf(gm.z, gm.z, gm.w * gm.w)) * (1.0f / ANI_SQRT_CK);
            const float isp = isg * rq;           // 1 / sp
            const float rr = rq - 1.0f / rq;      // sigma / sp - sp / sigma
            const float rux = rq * gm.z, ruy = rq * gm.w;
            const float dx = px - gm.x, dy = py - gm.y;
            const float a = __builtin_fmaf(dx, gm.z, dy * gm.w);
            const float b = rq * __builtin_fmaf(dy, gm.z, -(dx * gm.w));
            const float m = __builtin_fmaf(a, a, b * b);
            const bool in = (mt.y >= stop) && (m <= lim);
            const float G = __builtin_amdgcn_exp2f(-m);
            const float oG = op * G;
            const bool lt = oG < amax;
            const float alpha = in ? fminf(oG, amax) : 0.0f;  // = lt ? oG : amax
            const float r = __builtin_amdgcn_rcpf(1.0f - alpha);
            const float dLda = (in && lt) ? -Wc * r : 0.0f;
            T = in ? T * r : T;
            aT = __builtin_fmaf(alpha, T, aT);
            const float h = dLda * op * G * two_ln2;
            const float v[5] = {h * __builtin_fmaf(a, gm.z, -(b * ruy)), h * __builtin_fmaf(a, gm.w, b * rux),
                                (h * a) * (a * isg), (h * b) * (b * isp), (h * a) * (b * rr)};
            if (__ballot(in) == 0ull) continue;
            if (n_rows + 5 > RB) {
              flush_rows(park, ptgt, n_rows, ggrad);
              n_rows = 0;
            }
            accO += dLda * G;  // dL/do_j
#pragma unroll
            for (int i = 0; i < 5; ++i) park[(n_rows + i) * RB_ROW + lane] = v[i];
            if (lane < 5) ptgt[n_rows + lane] = make_int2(mt.x, lane);
            n_rows = __builtin_amdgcn_readfirstlane(n_rows + 5);
          }
          if (n_rows > 0) flush_rows(park, ptgt, n_rows, ggrad);
        } else if (LONG && cur_long) {
          // stroke Gaussians of very long curves (LONG_TAUS): dL/dmu (2) and
          // dL/dsigma formed per pixel and parked in three rows
          if (n_ent > 0) flush_pending(j, n_ent);  // the rows are shared
          n_ent = 0;
          int n_rows = 0;
          for (; j < jend; ++j) {
            if (since >= FLUSH) {
              fold_curve<C>(false, gI, aT, accO, ctot);
              since = 0;
            }
            ++since;
            const float4 gm = wgeo[j];
            const int4 mt = wmeta[j];
            const float op = __int_as_float(mt.z);
            const float is3 = __int_as_float(mt.w);
            const float dx = px - gm.x, dy = py - gm.y;
            const float d2 = __builtin_fmaf(dx, dx, dy * dy);
            const bool in = (mt.y >= stop) && (d2 <= gm.z);
            const float G = __builtin_amdgcn_exp2f(gm.w * d2);
            const float oG = op * G;
            const bool lt = oG < amax;
            const float alpha = in ? fminf(oG, amax) : 0.0f;  // = lt ? oG : amax
            const float r = __builtin_amdgcn_rcpf(1.0f - alpha);
            const float dLda = (in && lt) ? -Wc * r : 0.0f;
            T *= r;
            aT = __builtin_fmaf(alpha, T, aT);
            const float dG = dLda * op;
            const float dd2 = dG * G * gm.w * ln2;  // d exp2(a d2) / d d2 = G a ln 2
            const float v[3] = {-2.0f * dx * dd2, -2.0f * dy * dd2, dG * G * (d2 * is3)};
            if (__ballot(in) == 0ull) continue;
            if (__builtin_expect(n_rows + 3 > RB, 0)) {
              flush_rows(park, ptgt, n_rows, ggrad);
              n_rows = 0;
            }
            accO += dLda * G;  // dL/do_j
#pragma unroll
            for (int i = 0; i < 3; ++i) park[(n_rows + i) * RB_ROW + lane] = v[i];
            if (lane < 3) ptgt[n_rows + lane] = make_int2(mt.x, lane);
            n_rows = __builtin_amdgcn_readfirstlane(n_rows + 3);
          }
          if (n_rows > 0) flush_rows(park, ptgt, n_rows, ggrad);
        } else {
          // stroke and fill Gaussians: v = dL/dalpha G per pixel, parked (a
          // stroke's also summed per lane into the curve's opacity gradient,
          // which is folded into FP64 every FLUSH entries to keep that FP32
          // sum short).  An entry that does not reach a pixel, or lies in
          // front of its stop, composites there with G = 0: alpha 0, r exactly
          // 1, T unchanged.
          auto eval = [&](int jj, int ent) {
            const float4 gm = wgeo[jj];
            const int4 mt = wmeta[jj];
            const float op = __int_as_float(mt.z);
            const float dx = px - gm.x, dy = py - gm.y;
            const float d2 = __builtin_fmaf(dx, dx, dy * dy);
            const bool in = (mt.y >= stop) && (d2 <= gm.z);
            const float G = in ? __builtin_amdgcn_exp2f(gm.w * d2) : 0.0f;
            const float oG = op * G;
            const bool lt = oG < amax;
            const float alpha = fminf(oG, amax);  // lt ? oG : amax, also for a NaN oG
            const float r = __builtin_amdgcn_rcpf(1.0f - alpha);
            T *= r;  // the transmittance in front of the entry
            aT = __builtin_fmaf(alpha, T, aT);
            // dL/dalpha = (T' K - B) / (1 - alpha) = -W / (1 - alpha)
            const float v = (in && lt) ? -Wc * r * G : 0.0f;
            accO += v;
            park[ent * RB_ROW + lane] = v;
          };
          while (j < jend) {
            const int m = min(jend - j, RB - n_ent);
            if (!cur_fill && since + m > FLUSH) {
              fold_curve<C>(false, gI, aT, accO, ctot);
              since = 0;
            }
            since += m;
#pragma unroll 4
            for (int i = 0; i < m; ++i) eval(j + i, n_ent + i);
            j += m;
            n_ent += m;
            if (n_ent == RB) {
              flush_pending(j, n_ent);
              n_ent = 0;
            }
          }
        }
      }
      if (n_ent > 0) flush_pending(cnt, n_ent);
      __builtin_amdgcn_wave_barrier();
      s_lo = n_lo;
      s_hi = n_hi;
    }
    close_curve();
  }
}

__global__ void k_reset_queue(int32_t* q) {
  if (threadIdx.x < 4 && blockIdx.x == 0) q[threadIdx.x] = 0;
}

template <class K>
int resident_grid(K kernel, int n_blocks, int n_cu, size_t lds, int block = BLOCK) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, lds) != hipSuccess || per_cu < 1)
    per_cu = 1;
  const int g = per_cu * n_cu;
  return g < n_blocks ? g : n_blocks;
}

inline int depth_factor(int batch) { return batch <= 64 ? 1 : (batch <= 128 ? 2 : 4); }

template <int C, int TILE, int KIND, bool SPLIT>
hipError_t fwd_s(const Launch& L, float* image, float* T_final, int32_t* n_last, int persistent) {
  constexpr int QUADS = TileCfg<TILE>::QUADS;
  const int64_t n_items = L.n_tiles * QUADS;
  if (n_items <= 0) return hipSuccess;
  // blocks: one per item of a long list (at least LONG_LEAST positions each;
  // their number is on the device), one per wpb others
  constexpr int wpb = SPLIT ? FW : WPB;
  const int64_t n_long = SPLIT ? std::min(L.n_tiles, (int64_t)L.bf->caps.pairs / LONG_LEAST) * QUADS : 0;
  int64_t blocks = std::min(n_items, n_long + (n_items + wpb - 1) / wpb);
  // (a launch counts its threads in 32 bits)
  if (persistent || blocks * 64 * wpb > 0x7fffffffLL) {
    persistent = 1;
    blocks = resident_grid(k_blend_fwd<C, TILE, KIND, SPLIT>, (int)std::min<int64_t>(blocks, 0x7fffffff), L.n_cu, 0, 64 * wpb);
    hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, L.stream, L.w.queue);
  }
  Phase ph(L, NSPLAT_T_BLEND_FWD);
  hipLaunchKernelGGL((k_blend_fwd<C, TILE, KIND, SPLIT>), dim3((int)blocks), dim3(64 * wpb), 0, L.stream, *L.pr, L.w,
                     L.sc->n_scenes, (int)L.n_tiles, (const Gauss*)L.bf->gauss, L.bf->ranges, L.bf->idx, L.sc->bg,
                     image, T_final, n_last, L.bf->plan, (int64_t)L.bf->caps.gauss, persistent, L.ck_lg);
  return hipGetLastError();
}

// Long lists on blocks (SPLIT) where the chunk length is left to choose, and not
// at a grid step of 1 known here, where fill runs are walked whole.
template <int C, int TILE, int KIND>
hipError_t fwd_t(const Launch& L, float* image, float* T_final, int32_t* n_last, int persistent) {
  if (split_long(*L.pr) && !((KIND & KIND_FILL) && !L.pr->h_dev && L.pr->h == 1.0f))
    return fwd_s<C, TILE, KIND, true>(L, image, T_final, n_last, persistent);
  return fwd_s<C, TILE, KIND, false>(L, image, T_final, n_last, persistent);
}

template <int C, int TILE, int E, int KIND>
hipError_t bwd_t(const Launch& L, const float* dL, const float* T_final, const int32_t* n_last, int persistent) {
  if (L.n_tiles <= 0) return hipSuccess;
  // the item count lives on the device; the grid covers its bound
  // sum over tiles of QUADS * ceil(len / CK) <= QUADS * (pairs / CK + tiles);
  // where the binning chose a chunk below CK_MIN, QUADS * pairs / CK is at
  // most twice its target (small_chunk_log2)
  const int64_t blocks = adj_blocks(TILE), pairs = L.bf->caps.pairs;
  int64_t max_items = blocks * (pairs >> (L.ck_lg >= 0 ? L.ck_lg : 9));
  if (L.ck_lg < 0 && TILE <= 16)
    max_items = std::max(max_items, std::min(blocks * (pairs / CK_SMALL), (int64_t)2 * SMALL_ITEMS * L.n_cu));
  max_items += blocks * L.n_tiles;
  const size_t lds = (size_t)WPB * bwd_wave_bytes(E) + BASIS_BYTES;
  int64_t grid = (max_items + WPB - 1) / WPB;
  // (a launch counts its threads in 32 bits and drops what is above: a grid for
  // 2^31 pairs in 32 x 32 tiles left out most of the items, with no error)
  if (persistent || grid * BLOCK > 0x7fffffffLL) {
    persistent = 1;
    grid = resident_grid(k_blend_bwd<C, TILE, E, KIND>, (int)std::min<int64_t>(grid, 0x7fffffff), L.n_cu, lds);
    hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, L.stream, L.w.queue);
  }
  Phase ph(L, NSPLAT_T_BLEND_BWD);
  hipLaunchKernelGGL((k_blend_bwd<C, TILE, E, KIND>), dim3((int)grid), dim3(BLOCK), lds, L.stream, *L.cv, *L.pr, L.w,
                     L.sc->n_scenes, (int)L.n_tiles, (const Gauss*)L.bf->gauss, L.bf->ranges, L.bf->idx, L.sc->bg,
                     dL, T_final, n_last, L.bf->plan, (int64_t)L.bf->caps.gauss, persistent, 24 * 16 * L.n_cu, L.ck_lg);
  return hipGetLastError();
}

// The tangent-aligned kind and the fill-run walk are compiled in only for
// batches that declare such curves (nsplat_curves.any_flags), so that the
// other batches run without their branches and registers.
inline int kinds_of(const Launch& L) {
  return ((L.cv->any_flags & NSPLAT_ANISO) ? KIND_ANI : 0) | ((L.cv->any_flags & NSPLAT_FILLED) ? KIND_FILL : 0);
}

template <int C, int TILE>
hipError_t fwd_d(const Launch& L, float* image, float* T_final, int32_t* n_last, int persistent) {
  switch (kinds_of(L)) {
    case 0: return fwd_t<C, TILE, 0>(L, image, T_final, n_last, persistent);
    case KIND_ANI: return fwd_t<C, TILE, KIND_ANI>(L, image, T_final, n_last, persistent);
    case KIND_FILL: return fwd_t<C, TILE, KIND_FILL>(L, image, T_final, n_last, persistent);
    default: return fwd_t<C, TILE, KIND_ANI | KIND_FILL>(L, image, T_final, n_last, persistent);
  }
}

// (KIND_LONG only where the batch has intervals enough for a curve of more than
// LONG_TAUS: its registers cost the other launches 1 to 2 %, 256 fill paths at
// 512^2 0.1335 -> 0.1325 ms without, 12 quintic strokes 0.293 -> 0.289)
template <int C, int TILE, int E>
hipError_t bwd_k(const Launch& L, const float* dL, const float* T_final, const int32_t* n_last, int persistent) {
  switch (kinds_of(L) | (L.cv->n_taus > LONG_TAUS ? KIND_LONG : 0)) {
    case 0: return bwd_t<C, TILE, E, 0>(L, dL, T_final, n_last, persistent);
    case KIND_ANI: return bwd_t<C, TILE, E, KIND_ANI>(L, dL, T_final, n_last, persistent);
    case KIND_FILL: return bwd_t<C, TILE, E, KIND_FILL>(L, dL, T_final, n_last, persistent);
    case KIND_ANI | KIND_FILL: return bwd_t<C, TILE, E, KIND_ANI | KIND_FILL>(L, dL, T_final, n_last, persistent);
    case KIND_LONG: return bwd_t<C, TILE, E, KIND_LONG>(L, dL, T_final, n_last, persistent);
    case KIND_FILL | KIND_LONG: return bwd_t<C, TILE, E, KIND_FILL | KIND_LONG>(L, dL, T_final, n_last, persistent);
    default: return bwd_t<C, TILE, E, KIND_ANI | KIND_FILL | KIND_LONG>(L, dL, T_final, n_last, persistent);
  }
}

template <int C, int TILE>
hipError_t bwd_d(const Launch& L, const float* dL, const float* T_final, const int32_t* n_last, int persistent) {
  switch (depth_factor(L.pr->batch)) {
    case 1: return bwd_k<C, TILE, 1>(L, dL, T_final, n_last, persistent);
    case 2: return bwd_k<C, TILE, 2>(L, dL, T_final, n_last, persistent);
    default: return bwd_k<C, TILE, 4>(L, dL, T_final, n_last, persistent);
  }
}

}  // namespace

hipError_t launch_blend_fwd(const Launch& L, float* image, float* T_final, int32_t* n_last, int persistent) {
  const int C = L.cv->channels, t = L.pr->tile;
  if (C == 1) {
    if (t == 8) return fwd_d<1, 8>(L, image, T_final, n_last, persistent);
    if (t == 16) return fwd_d<1, 16>(L, image, T_final, n_last, persistent);
    return fwd_d<1, 32>(L, image, T_final, n_last, persistent);
  }
  if (t == 8) return fwd_d<3, 8>(L, image, T_final, n_last, persistent);
  if (t == 16) return fwd_d<3, 16>(L, image, T_final, n_last, persistent);
  return fwd_d<3, 32>(L, image, T_final, n_last, persistent);
}

hipError_t launch_blend_bwd(const Launch& L, const float* dL, const float* T_final, const int32_t* n_last,
                            int persistent) {
  const int C = L.cv->channels, t = L.pr->tile;
  if (C == 1) {
    if (t == 8) return bwd_d<1, 8>(L, dL, T_final, n_last, persistent);
    if (t == 16) return bwd_d<1, 16>(L, dL, T_final, n_last, persistent);
    return bwd_d<1, 32>(L, dL, T_final, n_last, persistent);
  }
  if (t == 8) return bwd_d<3, 8>(L, dL, T_final, n_last, persistent);
  if (t == 16) return bwd_d<3, 16>(L, dL, T_final, n_last, persistent);
  return bwd_d<3, 32>(L, dL, T_final, n_last, persistent);
}

}  // namespace nsp
