// Second half of nsplat_backward: per-Gaussian adjoints -> curve parameters.
//
//   k_adj_stroke    one lane per stroke Gaussian: dL/d(mu, sigma) ->
//                   dL/d(x, y, s) of C(u_j) (sigma = s / rho, Eq. 5) -> reverse
//                   mode through the rational point (Eq. 1) and the Cox-de Boor
//                   triangle: control points, weights, widths, the 2p knots of
//                   the span, and dL/du_j -> the domain ends u_p, u_{m-p}
//                   (u_j is uniform in the domain).
//   k_adj_aniso     one lane per tangent-aligned stroke Gaussian: the same,
//                   plus dL/d(sp, theta) and the spacing term of sigma through
//                   the first derivative C'(u_j) and the domain ends.
//   k_adj_fill      one lane per fill Gaussian: dL/do_j -> curve opacity and,
//                   through the sigmoid and the SDF (Eq. 7, S1-S3, sign
//                   detached, nearest segment), the two end points of the
//                   nearest boundary segment.
//   (Colour gradients, and the opacity gradient of stroke curves, are
//   accumulated per curve by the compositing adjoint.)
//   k_adj_boundary  one lane per boundary point: the same point adjoint.
//   Both sum within the wavefront by (curve, span) run before the FP64 global
//   atomics (accumulate_points).
//   k_reg_stroke,   the geometric regularisers of Sec. 3.5 at stroke samples
//   k_reg_boundary  and fill boundary points: bounding-box penalty (Eq. 12)
//                   into the centre / boundary-point adjoints, derivative
//                   loss (Eq. 11) by reverse mode straight to the curve.
//   k_fold          one block per curve: control points -> key points
//                   (the closed wrap), knots -> intervals (suffix sums of the
//                   cumulative sum) -> tau, FP32 outputs.
#include "nsplat_internal.h"

namespace nsp {

namespace {

// The point and derivative adjoints below hold basis functions and control
// points in register arrays sized for degree PD, the batch's degree bound (3,
// or NSPLAT_MAX_DEGREE): smaller arrays for the usual quadratic and cubic
// curves keep more wavefronts resident.
constexpr int tri_n(int d) { return (d + 1) * (d + 2) / 2; }

template <int PD>
struct PtAdj {
  double cp[PD + 1][4];  // (x, y, w, s) of control points span-p..span
  double knot[2 * PD];   // slot k <-> knot index span - PD + 1 + k
  double ubar;
};

// Reciprocals of the Cox-de Boor denominators: inv[d (d - 1) / 2 + r] =
// 1 / (U[span + r + 1] - U[span - d + r + 1]), r < d (each stands in two terms
// of the triangle and in four of its reverse, as a division each time before:
// point adjoints of 1.8M samples 0.248 -> 0.098 ms with the sums below).
constexpr int inv_n(int d) { return d * (d + 1) / 2; }

// Basis triangle at u on `span`: left[k] = u - U[span + 1 - k], right[k] =
// U[span + k] - u, the reciprocals, and level d's functions at tri[d (d + 1) / 2].
template <int P>
__device__ inline void basis_triangle(const double* U, int span, double u, double (&left)[P + 1],
                                      double (&right)[P + 1], double (&inv)[inv_n(P)], double (&tri)[tri_n(P)]) {
  tri[0] = 1.0;
#pragma unroll
  for (int d = 1; d <= P; ++d) {
    const double lo = U[span + 1 - d], hi = U[span + d];
    left[d] = u - lo;
    right[d] = hi - u;
    double saved = 0.0;
#pragma unroll
    for (int r = 0; r < d; ++r) {
      inv[d * (d - 1) / 2 + r] = 1.0 / (right[r + 1] + left[d - r]);
      const double temp = tri[(d - 1) * d / 2 + r] * inv[d * (d - 1) / 2 + r];
      tri[d * (d + 1) / 2 + r] = saved + right[r + 1] * temp;
      saved = left[d - r] * temp;
    }
    tri[d * (d + 1) / 2 + d] = saved;
  }
}

// Reverse of the triangle: given the adjoints Nb of the degree-d functions,
// through N_{i,d} = (u - U_i) / (U_{i+d} - U_i) N_{i,d-1}
//                 + (U_{i+d+1} - u) / (U_{i+d+1} - U_{i+1}) N_{i+1,d-1},
// adds the adjoints of u and of the knots (slot k <-> knot index
// span - PD + 1 + k) and leaves those of the degree d - 1 functions in Nb.
template <int PD, int P>
__device__ inline void triangle_reverse(int d, const double (&left)[P + 1], const double (&right)[P + 1],
                                        const double (&inv)[inv_n(P)], const double (&tri)[tri_n(P)],
                                        double (&Nb)[P + 1], double& ub, double (&knot)[2 * PD]) {
  double Np[P + 1];
#pragma unroll
  for (int r = 0; r <= P; ++r) Np[r] = 0.0;
#pragma unroll
  for (int r = 0; r <= d; ++r) {
    const double nb = Nb[r];
    if (r >= 1) {
      const double iv = inv[d * (d - 1) / 2 + r - 1], al = left[d + 1 - r] * iv;
      Np[r - 1] += nb * al;
      const double g = nb * tri[(d - 1) * d / 2 + r - 1] * iv;
      ub += g;
      knot[PD - 1 - d + r] -= g * (right[r] * iv);
      knot[PD - 1 + r] -= g * al;
    }
    if (r <= d - 1) {
      const double iv = inv[d * (d - 1) / 2 + r], be = right[r + 1] * iv;
      Np[r] += nb * be;
      const double g = nb * tri[(d - 1) * d / 2 + r] * iv;
      ub -= g;
      knot[PD + r] += g * (left[d - r] * iv);
      knot[PD - d + r] += g * be;
    }
  }
#pragma unroll
  for (int r = 0; r <= P; ++r) Nb[r] = Np[r];
}

// Reverse-mode adjoint of the rational point (x, y, s) at u on `span` for the
// upstream gradient ab[3], for a curve of degree P <= PD.
template <int PD, int P>
__device__ inline void point_adjoint_deg(const nsplat_curves& cv, const CurveView& v, double u, int span,
                                         const double (&ab)[3], PtAdj<PD>& out) {
  double tri[tri_n(P)], left[P + 1], right[P + 1], inv[inv_n(P)];
  basis_triangle<P>(v.U, span, u, left, right, inv, tri);
  constexpr int TP = P * (P + 1) / 2;  // the degree-P functions
  // C = S / W over the span's control points
  double Q[P + 1][3], wt[P + 1];
  double S[3] = {0.0, 0.0, 0.0}, W = 0.0;
#pragma unroll
  for (int r = 0; r <= P; ++r) {
    const int k = v.k0 + v.key_of_cp(span - P + r);
    wt[r] = (double)cv.key_w[k];
    Q[r][0] = (double)cv.key_xy[2 * k];
    Q[r][1] = (double)cv.key_xy[2 * k + 1];
    Q[r][2] = (double)cv.key_s[k];
    const double nw = tri[TP + r] * wt[r];
    W += nw;
#pragma unroll
    for (int q = 0; q < 3; ++q) S[q] += nw * Q[r][q];
  }
  const double invW = 1.0 / W;
  const double Cp[3] = {S[0] * invW, S[1] * invW, S[2] * invW};
  double Nb[P + 1];
#pragma unroll
  for (int r = 0; r <= PD; ++r) {
#pragma unroll
    for (int q = 0; q < 4; ++q) out.cp[r][q] = 0.0;
    if (r > P) continue;
    const double gdot = ab[0] * (Q[r][0] - Cp[0]) + ab[1] * (Q[r][1] - Cp[1]) + ab[2] * (Q[r][2] - Cp[2]);
    const double nwW = tri[TP + r] * wt[r] * invW;
    out.cp[r][0] = ab[0] * nwW;                // dC/dP = N w / W
    out.cp[r][1] = ab[1] * nwW;
    out.cp[r][2] = tri[TP + r] * gdot * invW;  // dC/dw = N (P - C) / W
    out.cp[r][3] = ab[2] * nwW;
    Nb[r] = wt[r] * gdot * invW;               // dC/dN = w (P - C) / W
  }
  double ub = 0.0;
#pragma unroll
  for (int k = 0; k < 2 * PD; ++k) out.knot[k] = 0.0;
#pragma unroll
  for (int d = P; d >= 1; --d) triangle_reverse<PD, P>(d, left, right, inv, tri, Nb, ub, out.knot);
  out.ubar = ub;
}

// The adjoints for the degree of the lane's curve: bodies with the degree
// fixed need no tests of it and fewer registers.
template <int PD>
__device__ inline void point_adjoint(const nsplat_curves& cv, const CurveView& v, double u, int span,
                                     const double (&ab)[3], PtAdj<PD>& out) {
  if constexpr (PD >= 5) {
    if (v.p == 5) return point_adjoint_deg<PD, 5>(cv, v, u, span, ab, out);
    if (v.p == 4) return point_adjoint_deg<PD, 4>(cv, v, u, span, ab, out);
  }
  if (v.p == 3) return point_adjoint_deg<PD, 3>(cv, v, u, span, ab, out);
  if (v.p == 2) return point_adjoint_deg<PD, 2>(cv, v, u, span, ab, out);
  point_adjoint_deg<PD, 1>(cv, v, u, span, ab, out);
}

// Segmented suffix sum across the wavefront.  A run is a maximal group of
// adjacent lanes with equal keys (two runs may share a key); afterwards the
// first lane of each run holds the run total.  Each lane carries a flag that
// says whether its partial interval already reaches the end of its run.
template <int NV>
__device__ inline void seg_reduce(int64_t key, double (&v)[NV]) {
  const int lane = __lane_id();
  const int64_t next = __shfl_down(key, 1);
  bool f = (lane == 63) || (next != key);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const bool fo = __shfl_down((int)f, off) != 0;
    const bool take = !f && (lane + off < 64);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const double o = __shfl_down(v[i], off);
      if (take) v[i] += o;
    }
    if (take) f = fo;
  }
}

__device__ inline bool seg_head(int64_t key) {
  const int lane = __lane_id();
  const int64_t prev = __shfl_up(key, 1);
  return key >= 0 && (lane == 0 || prev != key);
}

// Sums of point adjoints over the wavefront into the FP64 control-point and
// knot buffers.  The lanes' values go through LDS, one row of 64 samples per
// value; lane (i, part) = (l & 31, l >> 5) then adds up value i over half of
// the samples, 32 at most, and sends the sum of each run of samples with one
// (curve, span) out with one atomic (a run that crosses the middle is joined
// there).  Shuffling every value through six rounds of a segmented scan took
// 264 LDS permutes and as many selects per wavefront before, this 22 writes and
// 32 reads (adjoint of 1.8M samples: 0.248 -> 0.098 ms with the reciprocals
// above; 16 closed strokes at 512^2 0.022 -> 0.012).  At degree 4 or 5 the values go in two rounds.
template <int PD>
struct PointSums {
  static constexpr int NCP = 4 * (PD + 1), NV = NCP + 2 * PD, ROUNDS = NV > 32 ? 2 : 1, NR = NV / ROUNDS;
  static_assert(NR * ROUNDS == NV && NR <= 32, "values per round");
  double v[NR][65];     // padded rows
  int64_t cp[64], kn[64];  // by a run's first sample: its first control-point and knot element
};

template <int PD>
__device__ inline void accumulate_points(const Work& w, PointSums<PD>* st, bool act, int64_t key, int c,
                                         const CurveView& v, int span, PtAdj<PD>& pa) {
  using S = PointSums<PD>;
  const uint64_t am = __ballot(act);
  if (am == 0ull) return;
  const int lane = __lane_id();
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  // a run begins at an active lane whose key differs from the active lane's
  // before it; inactive lanes (values 0) go on with the run
  const int pl = (am & below) ? 63 - __builtin_clzll(am & below) : -1;
  const int64_t pk = __shfl(key, pl < 0 ? 0 : pl);
  const bool head = act && (pl < 0 || pk != key);
  const uint64_t hm = __ballot(head);
  const int i = lane & 31, part = lane >> 5;
  const uint32_t mine = (uint32_t)(part ? hm >> 32 : hm);
#pragma unroll
  for (int rd = 0; rd < S::ROUNDS; ++rd) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k = 0; k < S::NR; ++k) {
      const int q = rd * S::NR + k;
      st->v[k][lane] = q < S::NCP ? pa.cp[q / 4][q & 3] : pa.knot[q - S::NCP < 2 * PD ? q - S::NCP : 0];
    }
    if (head && rd == 0) {
      st->cp[lane] = 4 * ((int64_t)v.k0 + (int64_t)c * CP_PAD + span - v.p);
      st->kn[lane] = (int64_t)v.t0 + (int64_t)c * KNOT_PAD + span - PD + 1;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int q = rd * S::NR + i;
    const bool valid = i < S::NR;
    auto emit = [&](int at, double x) {  // the run that begins at sample `at`
      if (!valid || x == 0.0) return;
      double* o = q < S::NCP ? w.gcp + st->cp[at] + q : w.gknot + st->kn[at] + (q - S::NCP);
      unsafeAtomicAdd(o, x);
    };
    const double* row = st->v[valid ? i : 0] + 32 * part;
    double sum = 0.0, first = 0.0;  // first: the upper half's samples before its first run
    int at = -1;                    // where the open run begins (-1: none in this half yet)
#pragma unroll 8
    for (int k = 0; k < 32; ++k) {
      const double x = row[k];
      if ((mine >> k) & 1u) {
        if (at >= 0) emit(at, sum);
        else first = sum;
        at = 32 * part + k;
        sum = 0.0;
      }
      sum += x;
    }
    if (at < 0) {
      first = sum;
      sum = 0.0;
    }
    // the lower half's last run goes on with the upper half's first samples (with
    // no run in the lower half, the upper half's first active sample begins one)
    const double up = __shfl(first, i + 32);
    if (at >= 0) emit(at, part == 0 ? sum + up : sum);
  }
}

// Curve-level sums dL/du_p, dL/du_{m-p} (the samples' dependence on the domain
// ends), kept per lane over consecutive groups of samples of one curve and
// sent out where the curve changes: all samples of a curve add to the same two
// addresses, where an atomic per wavefront queues up.
struct DomainSums {
  int c = -1;            // the curve of a and b (wavefront-uniform)
  int64_t ia = 0, ib = 0;
  double a = 0.0, b = 0.0;
  __device__ void flush(const Work& w) {
    if (c < 0) return;
    double x = a, y = b;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      x += __shfl_xor(x, off);
      y += __shfl_xor(y, off);
    }
    if (__lane_id() == 0) {
      if (x != 0.0) unsafeAtomicAdd(w.gknot + ia, x);
      if (y != 0.0) unsafeAtomicAdd(w.gknot + ib, y);
    }
    c = -1;
    a = b = 0.0;
  }
  // every lane of the wavefront calls it; act lanes add (xa, xb) to curve cc
  __device__ void add(const Work& w, bool act, int cc, const CurveView& v, double xa, double xb) {
    const uint64_t am = __ballot(act);
    if (am == 0ull) return;
    const int l0 = __builtin_ctzll(am);
    const int cu = __builtin_amdgcn_readlane(cc, l0);
    const int64_t base = (int64_t)v.t0 + (int64_t)cc * KNOT_PAD, pa = base + v.p, pb = base + v.m - v.p;
    if (__ballot(act && cc != cu) == 0ull) {
      if (cu != c) {
        flush(w);
        c = cu;
        ia = __shfl(pa, l0);
        ib = __shfl(pb, l0);
      }
      a += act ? xa : 0.0;
      b += act ? xb : 0.0;
      return;
    }
    double x[2] = {act ? xa : 0.0, act ? xb : 0.0};
    const int64_t key = act ? (int64_t)cc : -1 - (int64_t)__lane_id();
    seg_reduce(key, x);
    if (seg_head(key)) {
      if (x[0] != 0.0) unsafeAtomicAdd(w.gknot + pa, x[0]);
      if (x[1] != 0.0) unsafeAtomicAdd(w.gknot + pb, x[1]);
    }
  }
};

// First group of 64 samples of this wavefront and its stride over the groups
// (in samples): wavefronts take `run` consecutive groups at a time.
struct GroupWalk {
  int64_t base, jump;
  int run, k = 0;
  __device__ GroupWalk(int run_) : run(run_) {
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    base = wave * run * 64;
    jump = (((int64_t)gridDim.x * blockDim.x) >> 6) * run * 64 - (int64_t)(run - 1) * 64;
  }
  __device__ void next() {
    if (++k < run) base += 64;
    else {
      k = 0;
      base += jump;
    }
  }
};

// Stroke Gaussians: dL/d(mu, sigma) -> the curve point adjoint at u_j.  Held to
// three wavefronts per SIMD at degree 3 (168 VGPRs, 8 spilled): with 170 and two
// wavefronts 1.8M samples took 0.118 ms, with three 0.098.
template <int PD>
__global__ __launch_bounds__(256, PD <= 3 ? 3 : 2) void k_adj_stroke(nsplat_curves cv, nsplat_params pr, Work w,
                                                    const int32_t* plan, const int32_t* counters,
                                                    const Gauss* __restrict__ gs, int run) {
  __shared__ PointSums<PD> sums[4];
  if (w.queue[Q_NSTROKE] == 0) return;  // no Gaussians of this kind
  const int64_t G = counters[NSPLAT_CNT_GAUSS];
  const int lane = __lane_id();
  DomainSums dom;
  for (GroupWalk gw(run); gw.base < G; gw.next()) {
    const int64_t g = gw.base + lane;
    int64_t kspan = 0;
    double da = 0.0, db = 0.0;
    PtAdj<PD> pa;
    int c = 0, span = 0;
    CurveView v;
    v.p = 0;
    bool stroke = false;
    if (g < G) {
      // curve and sample index from the emission offsets, as in k_adj_fill
      typedef const __attribute__((address_space(4))) Gauss* const_gauss;
      const int64_t g0 = first_lane_i64(g);
      c = curve_walk(w.goff, cv.n_curves, g, g0, ((const_gauss)gs)[g0].curve);
      if (!(cv.flags[c] & (NSPLAT_FILLED | NSPLAT_ANISO))) {
        stroke = true;
        const int local = (int)(g - w.goff[c]);
        v = curve_view(cv, w.knots, c);
        const float* gg = w.ggrad + g * GG;
        const double ab[3] = {(double)gg[0], (double)gg[1], (double)gg[2] / (double)pr.rho};  // sigma = s / rho
        const int32_t* row = plan + (int64_t)P_STRIDE * c;
        const int M = row[P_NSAMP];
        int j = v.closed() ? local : local - pr.kappa;
        j = j < 0 ? 0 : (j > M - 1 ? M - 1 : j);
        double dt;
        const double u = sample_u(v.U[v.p], v.U[v.m - v.p], j, M, v.closed(), &dt);
        span = find_span(v.U, v.p, v.m, u);
        point_adjoint(cv, v, u, span, ab, pa);
        da = pa.ubar * (1.0 - dt);  // u_j = u_p + t_j (u_{m-p} - u_p)
        db = pa.ubar * dt;
        kspan = (int64_t)v.t0 + (int64_t)c * KNOT_PAD + span;
      }
    }
    if (!stroke) {
#pragma unroll
      for (int r = 0; r <= PD; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) pa.cp[r][q] = 0.0;
#pragma unroll
      for (int k = 0; k < 2 * PD; ++k) pa.knot[k] = 0.0;
    }
    accumulate_points(w, &sums[threadIdx.x >> 6], stroke, kspan, c, v, span, pa);
    dom.add(w, stroke, c, v, da, db);
  }
  dom.flush(w);
}

// Fill Gaussians: o_j = o sigmoid(z), z = gamma / h * sgn * d(q) with the
// nearest segment and the sign recorded at emission.  dL/do_j -> curve
// opacity, and dL/dd -> the segment's end points (d(d)/da = -(1 - t) n,
// d(d)/db = -t n at the projection, n the unit vector from it to q).
__global__ __launch_bounds__(256) void k_adj_fill(nsplat_curves cv, nsplat_params pr, Work w, const int32_t* plan,
                                                  const int32_t* counters, const Gauss* __restrict__ gs) {
  if (w.queue[Q_NFILL] == 0) return;  // no Gaussians of this kind
  const int64_t G = counters[NSPLAT_CNT_GAUSS];
  const int lane = __lane_id();
  const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) - lane;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const double h = (double)read_h(pr);
  const double gh = (double)pr.gamma / h;
  for (int64_t base = wave0; base < G; base += stride) {
    const int64_t g = base + lane;
    int64_t kcur = -1 - lane;
    double dop[1] = {0.0};  // dL/d(curve opacity): the only curve-level sum of a fill Gaussian
    int64_t skey = -1 - lane, sj = 0;  // boundary segment (start, end point) this lane's SDF gradient goes to
    double sv[4] = {0.0, 0.0, 0.0, 0.0};
    int c = 0;
    bool fill = false;
    if (g < G) {
      // the curve and lattice index of Gaussian g from the emission offsets
      // (the record holds the same two values), starting from the curve in
      // the record of the wavefront's first Gaussian (one scalar load)
      typedef const __attribute__((address_space(4))) Gauss* const_gauss;
      const int64_t g0 = first_lane_i64(g);
      c = curve_walk(w.goff, cv.n_curves, g, g0, ((const_gauss)gs)[g0].curve);
      if (cv.flags[c] & NSPLAT_FILLED) {
        fill = true;
        kcur = c;
        const int local = (int)(g - w.goff[c]);
        const double dO = (double)w.ggrad[g * GG + 3];
        const int32_t* row = plan + (int64_t)P_STRIDE * c;
        const int nx = row[P_NX];
        const int iy = local / nx, ix = local - iy * nx;
        const double qx = ((double)(row[P_IX0] + ix) + 0.5) * h;
        const double qy = ((double)(row[P_IY0] + iy) + 0.5) * h;
        const int nb = row[P_NSAMP];
        const int32_t xa = w.aux[g];
        const int ib = xa & 0x7fffffff;
        const double sgn = xa < 0 ? -1.0 : 1.0;
        // the nearest segment's record, with the arithmetic of the emission
        const double* sr = w.segs + SEG_WORDS * (seg_base(row[P_BOFF], c) + ib);
        const int jb = ib + 1 < nb ? ib + 1 : 0;
        const double ax = sr[0], ay = sr[1], ex = sr[2], ey = sr[3], inv = sr[4];
        const double rx = qx - ax, ry = qy - ay;
        double t = __builtin_fma(rx, ex, ry * ey) * inv;
        t = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
        const double px = __builtin_fma(t, ex, -rx), py = __builtin_fma(t, ey, -ry);
        const double d = sqrt(__builtin_fma(px, px, py * py));
        const double z = gh * (sgn * d);
        const double sz = 1.0 / (1.0 + exp(-z));
        dop[0] = dO * sz;
        const double ds = sz * (1.0 - sz);
        if (d > 0.0 && dO != 0.0 && ds > 1e-18) {
          const double dd = dO * (double)cv.opacity[c] * ds * gh * sgn;  // dL/dd
          const double nxv = -px / d, nyv = -py / d;
          skey = (int64_t)row[P_BOFF] + ib;
          sj = (int64_t)row[P_BOFF] + jb;
          sv[0] = -dd * (1.0 - t) * nxv;
          sv[1] = -dd * (1.0 - t) * nyv;
          sv[2] = -dd * t * nxv;
          sv[3] = -dd * t * nyv;
        }
      }
    }
    // lanes on the same boundary segment (neighbouring lattice points) are
    // summed in the wavefront before the FP64 atomics
    if (__ballot(skey >= 0) != 0ull) {
      seg_reduce(skey, sv);
      if (seg_head(skey)) {
        unsafeAtomicAdd(&w.gb[skey].x, sv[0]);
        unsafeAtomicAdd(&w.gb[skey].y, sv[1]);
        unsafeAtomicAdd(&w.gb[sj].x, sv[2]);
        unsafeAtomicAdd(&w.gb[sj].y, sv[3]);
      }
    }
    if (__ballot(fill) != 0ull) {
      const int64_t k0 = __builtin_amdgcn_readfirstlane((int)kcur);
      if (__ballot(kcur != k0) == 0ull) {  // one curve across the wavefront: a plain sum
        double s = dop[0];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0 && s != 0.0) unsafeAtomicAdd(w.gcurve + 4 * k0, s);
      } else {
        seg_reduce(kcur, dop);
        if (seg_head(kcur) && dop[0] != 0.0) unsafeAtomicAdd(w.gcurve + 4 * (int64_t)c, dop[0]);
      }
    }
  }
}

template <int PD>
__global__ __launch_bounds__(256, PD <= 3 ? 3 : 2) void k_adj_boundary(nsplat_curves cv, Work w, const int32_t* plan,
                                                      const int32_t* counters) {
  __shared__ PointSums<PD> sums[4];
  const int64_t NB = counters[NSPLAT_CNT_BOUND];
  const int lane = __lane_id();
  const int n = cv.n_curves;
  DomainSums dom;
  for (GroupWalk gw(1); gw.base < NB; gw.next()) {
    const int64_t b = gw.base + lane;
    bool act = false;
    int64_t kspan = 0;
    PtAdj<PD> pa;
#pragma unroll
    for (int r = 0; r <= PD; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) pa.cp[r][q] = 0.0;
#pragma unroll
    for (int k = 0; k < 2 * PD; ++k) pa.knot[k] = 0.0;
    pa.ubar = 0.0;
    double da = 0.0, db = 0.0;
    int c = 0, span = 0;
    CurveView v;
    v.p = 0;
    if (b < NB) {
      c = last_le_wave<P_STRIDE, P_BOFF>(plan, n, b);  // curve: the last c with boff <= b
      v = curve_view(cv, w.knots, c);
      const int32_t* row = plan + (int64_t)P_STRIDE * c;
      const int nb = row[P_NSAMP];
      const int j = (int)(b - row[P_BOFF]);
      const double2 adj = w.gb[b];
      if ((v.flags & NSPLAT_FILLED) && j >= 0 && j < nb && curve_valid(v) && (adj.x != 0.0 || adj.y != 0.0)) {
        act = true;
        const double ab[3] = {adj.x, adj.y, 0.0};
        double dt;
        const double u = sample_u(v.U[v.p], v.U[v.m - v.p], j, nb, true, &dt);
        span = find_span(v.U, v.p, v.m, u);
        point_adjoint(cv, v, u, span, ab, pa);
        da = pa.ubar * (1.0 - dt);
        db = pa.ubar * dt;
        kspan = (int64_t)v.t0 + (int64_t)c * KNOT_PAD + span;
      }
    }
    accumulate_points(w, &sums[threadIdx.x >> 6], act, kspan, c, v, span, pa);
    dom.add(w, act, c, v, da, db);
  }
  dom.flush(w);
}

// One block per curve: colour / opacity sums to FP32, control-point adjoints
// folded back onto key points (the closed wrap sends several control points
// to one key point), and the knot adjoints turned into interval adjoints:
// U_k = sum_{l<k} delta_l gives dL/d delta_l = sum_{k>l} dL/dU_k, a suffix sum:
// each thread sums a contiguous share of the knots, a block scan joins the
// shares.  A wavefront per curve serves short curves (a block of 1024 costs
// them more in launch than it saves); curves of hundreds of knots wait on
// that wavefront's loads, round after round (one curve of 10,240 key points:
// fold and zeroing 0.193 ms with one wavefront, 0.031 ms with sixteen; 16 of
// 2,000: 0.049 -> 0.015 ms).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_fold(nsplat_curves cv, Work w, nsplat_grads gr) {
  __shared__ double wtot[THREADS / 64];
  const int c = blockIdx.x;
  const int tid = threadIdx.x, lane = __lane_id(), wid = tid >> 6;
  const CurveView v = curve_view(cv, w.knots, c);
  const int C = cv.channels;
  const double* gc = w.gcurve + 4 * (int64_t)c;
  // a NULL output leaves that gradient group out
  if (tid == 0 && gr.opacity) gr.opacity[c] = (float)gc[0];
  if (tid < C && gr.color) gr.color[(int64_t)c * C + tid] = (float)gc[1 + tid];
  const bool ok = curve_valid(v);
  const double* gcp = w.gcp + 4 * ((int64_t)v.k0 + (int64_t)c * CP_PAD);
  for (int k = tid; k < v.nk; k += THREADS) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (ok) {
      if (!v.closed()) {
        for (int q = 0; q < 4; ++q) acc[q] = gcp[4 * k + q];
      } else {
        // control points j with key_of_cp(j) == k: j = (k + ceil(p/2)) mod n_k, and that + n_k
        const int j0 = (k + (v.p + 1) / 2) % v.nk;
        for (int j = j0; j < v.ncp; j += v.nk)
          for (int q = 0; q < 4; ++q) acc[q] += gcp[4 * j + q];
      }
    }
    const int64_t kk = v.k0 + k;
    if (gr.key_xy) {
      gr.key_xy[2 * kk] = (float)acc[0];
      gr.key_xy[2 * kk + 1] = (float)acc[1];
    }
    if (gr.key_w) gr.key_w[kk] = (float)acc[2];
    if (gr.key_s) gr.key_s[kk] = (float)acc[3];
  }
  if (!gr.tau) return;
  float* gt = gr.tau + v.t0;
  if (!ok) {
    for (int t = tid; t < v.nt; t += THREADS) gt[t] = 0.0f;
    return;
  }
  double* gk = w.gknot + (int64_t)v.t0 + (int64_t)c * KNOT_PAD;
  // knots 0 .. m, `per` of them per thread
  const int per = (v.m + THREADS) / THREADS, l0 = min(v.m + 1, tid * per), l1 = min(v.m + 1, l0 + per);
  double sum = 0.0;
  for (int l = l0; l < l1; ++l) sum += gk[l];
  double incl = sum;  // the shares of this lane and those above it in the wavefront
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_down(incl, off);
    if (lane + off < 64) incl += o;
  }
  double above = __shfl_down(incl, 1);  // the lanes above only
  if (lane == 63) above = 0.0;
  if (lane == 0) wtot[wid] = incl;
  __syncthreads();
  for (int i = THREADS / 64 - 1; i > wid; --i) above += wtot[i];
  for (int l = l1 - 1; l >= l0; --l) {  // gk[l] becomes the sum over k > l
    const double x = gk[l];
    if (l < v.m) gk[l] = above;
    above += x;
  }
  __syncthreads();
  if (!v.closed()) {
    for (int t = tid; t < v.nt; t += THREADS) gt[t] = (float)gk[v.p + t];
  } else {
    for (int t = tid; t < v.nt; t += THREADS) {
      double acc = 0.0;
      for (int l = t + v.p - v.nt; l < v.m; l += v.nt)
        if (l >= 0) acc += gk[l];
      gt[t] = (float)acc;
    }
  }
}

// Zeroes up to four FP64 arrays in one launch (index space n0 + n1 + n2 + n3).
struct ZeroSet {
  double* p[4];
  int64_t n[4];
};

// Clears the per-Gaussian adjoints (min(*count, cap) * mult floats at p) and
// the FP64 arrays of z, in one launch.
__global__ void k_zero_grads(float* p, const int32_t* count, int64_t mult, int64_t cap, ZeroSet z) {
  int64_t n = (int64_t)*count;
  n = (n < cap ? n : cap) * mult;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < n; i += stride) p[i] = 0.0f;
  const int64_t total = z.n[0] + z.n[1] + z.n[2] + z.n[3];
  for (int64_t i = i0; i < total; i += stride) {
    int64_t j = i;
    int a = 0;
    while (a < 3 && j >= z.n[a]) j -= z.n[a++];
    z.p[a][j] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Geometric regularisers (Sec. 3.5): derivative loss (Eq. 11) and
// bounding-box loss (Eq. 12), at the parameters of each curve's own samples.
// ---------------------------------------------------------------------------

constexpr int MAXR = 3;  // highest derivative order of the derivative loss

// Value scale * ||C^(r)(u)||^2 of the planar curve at u on `span` and its
// reverse-mode adjoint.  Forward: the span's homogeneous control points
// H_j = (w x, w y, w); derivative control points
//   PK_k[j] = (p - k + 1) (PK_{k-1}[j+1] - PK_{k-1}[j]) / (U[span+j+1] - U[span-p+j+k])
// (every denominator spans the non-empty span, so none vanishes);
// S^(k)(u) = sum_j N_{span-p+k+j, p-k}(u) PK_k[j], the homogeneous k-th
// derivative; and the rational Leibniz rule
//   C^(k) = (A^(k) - sum_{i=1..k} binom(k, i) W^(i) C^(k-i)) / W, (A, W) = S.
// Reverse: the same steps backwards, with the adjoint of the degree p - k
// basis functions entering the Cox-de Boor triangle at its level p - k.  With
// `up` set, the reverse pass starts from the given adjoint up[0..1] of
// C^(r)(u) instead of that of the value (whose scale is then unused).
template <int PD, int P>
__device__ inline double deriv_adjoint_deg(const nsplat_curves& cv, const CurveView& v, double u, int span, int r,
                                           double scale, PtAdj<PD>& out, const double* up) {
  constexpr int RM = MAXR < P ? MAXR : P;  // derivatives above the degree vanish
  double tri[tri_n(P)], left[P + 1], right[P + 1], inv[inv_n(P)];
  basis_triangle<P>(v.U, span, u, left, right, inv, tri);
  // PK_k[j]'s denominator U[span + j + 1] - U[span - P + j + k] is entry j of
  // level P - k + 1 of the triangle
  constexpr auto lvl = [](int k) { return (P - k + 1) * (P - k) / 2; };
  double X[P + 1], Y[P + 1], Wt[P + 1];
  double PK[RM + 1][P + 1][3];
#pragma unroll
  for (int j = 0; j <= P; ++j) {
    const int k = v.k0 + v.key_of_cp(span - P + j);
    Wt[j] = (double)cv.key_w[k];
    X[j] = (double)cv.key_xy[2 * k];
    Y[j] = (double)cv.key_xy[2 * k + 1];
    PK[0][j][0] = Wt[j] * X[j];
    PK[0][j][1] = Wt[j] * Y[j];
    PK[0][j][2] = Wt[j];
  }
#pragma unroll
  for (int k = 1; k <= RM; ++k)
#pragma unroll
    for (int j = 0; j <= P - k; ++j) {
      const double c = (double)(P - k + 1) * inv[lvl(k) + j];
#pragma unroll
      for (int q = 0; q < 3; ++q) PK[k][j][q] = c * (PK[k - 1][j + 1][q] - PK[k - 1][j][q]);
    }
  double S[MAXR + 1][3];
#pragma unroll
  for (int k = 0; k <= MAXR; ++k) {
    S[k][0] = S[k][1] = S[k][2] = 0.0;
    if (k > RM) continue;
#pragma unroll
    for (int j = 0; j <= P - k; ++j) {
      const double n = tri[(P - k) * (P - k + 1) / 2 + j];
#pragma unroll
      for (int q = 0; q < 3; ++q) S[k][q] += n * PK[k][j][q];
    }
  }
  const double binom[MAXR + 1][MAXR + 1] = {{1, 0, 0, 0}, {1, 1, 0, 0}, {1, 2, 1, 0}, {1, 3, 3, 1}};
  const double iW0 = 1.0 / S[0][2];
  double Cx[MAXR + 1], Cy[MAXR + 1];
#pragma unroll
  for (int k = 0; k <= MAXR; ++k) {
    Cx[k] = Cy[k] = 0.0;
    if (k > r) continue;
    double ax = S[k][0], ay = S[k][1];  // zero above the degree
#pragma unroll
    for (int i = 1; i <= MAXR; ++i) {
      if (i > k) break;
      ax -= binom[k][i] * S[i][2] * Cx[k - i];
      ay -= binom[k][i] * S[i][2] * Cy[k - i];
    }
    Cx[k] = ax * iW0;
    Cy[k] = ay * iW0;
  }
  // (register arrays are indexed with compile-time indices only)
  double crx = Cx[0], cry = Cy[0];
#pragma unroll
  for (int k = 1; k <= MAXR; ++k) {
    crx = k == r ? Cx[k] : crx;
    cry = k == r ? Cy[k] : cry;
  }
  const double value = scale * (crx * crx + cry * cry);
  // reverse: Leibniz rule
  double dCx[MAXR + 1], dCy[MAXR + 1], dS[MAXR + 1][3];
#pragma unroll
  for (int k = 0; k <= MAXR; ++k) {
    dCx[k] = k == r ? (up ? up[0] : 2.0 * scale * crx) : 0.0;
    dCy[k] = k == r ? (up ? up[1] : 2.0 * scale * cry) : 0.0;
    dS[k][0] = dS[k][1] = dS[k][2] = 0.0;
  }
#pragma unroll
  for (int k = MAXR; k >= 0; --k) {
    if (k > r) continue;
    const double gx = dCx[k] * iW0, gy = dCy[k] * iW0;
    dS[k][0] += gx;
    dS[k][1] += gy;
#pragma unroll
    for (int i = 1; i <= MAXR; ++i) {
      if (i > k) break;
      dS[i][2] -= binom[k][i] * (gx * Cx[k - i] + gy * Cy[k - i]);
      dCx[k - i] -= binom[k][i] * S[i][2] * gx;
      dCy[k - i] -= binom[k][i] * S[i][2] * gy;
    }
    dS[0][2] -= gx * Cx[k] + gy * Cy[k];
  }
  // reverse, level by level from the highest derivative: S^(k) =
  // sum_j N_{P-k}[j] PK_k[j] gives the adjoint of PK_k (A, joined by what the
  // level above sends down) and of the degree P - k functions (dN); knot slot
  // s <-> knot index span - PD + 1 + s
#pragma unroll
  for (int k = 0; k < 2 * PD; ++k) out.knot[k] = 0.0;
  double A[P + 1][3], dN[RM + 1][P + 1];
#pragma unroll
  for (int k = RM; k >= 0; --k) {
    double B[P + 1][3];
#pragma unroll
    for (int j = 0; j <= P - k; ++j) {
      const double n = tri[(P - k) * (P - k + 1) / 2 + j];
#pragma unroll
      for (int q = 0; q < 3; ++q) B[j][q] = n * dS[k][q];
      dN[k][j] = dS[k][0] * PK[k][j][0] + dS[k][1] * PK[k][j][1] + dS[k][2] * PK[k][j][2];
    }
    if (k < RM) {
#pragma unroll
      for (int j = 0; j <= P - k - 1; ++j) {
        const double iD = inv[lvl(k + 1) + j], c = (double)(P - k) * iD;
        double dD = 0.0;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          B[j + 1][q] += c * A[j][q];
          B[j][q] -= c * A[j][q];
          dD -= A[j][q] * PK[k + 1][j][q];
        }
        dD *= iD;
        out.knot[j + PD] += dD;              // knot span + j + 1
        out.knot[j + k + PD - P] -= dD;      // knot span - P + j + k + 1
      }
    }
#pragma unroll
    for (int j = 0; j <= P - k; ++j)
#pragma unroll
      for (int q = 0; q < 3; ++q) A[j][q] = B[j][q];
  }
  // homogeneous control points -> (x, y, w); the width does not enter
#pragma unroll
  for (int j = 0; j <= PD; ++j) {
    out.cp[j][0] = out.cp[j][1] = out.cp[j][2] = out.cp[j][3] = 0.0;
    if (j > P) continue;
    out.cp[j][0] = Wt[j] * A[j][0];
    out.cp[j][1] = Wt[j] * A[j][1];
    out.cp[j][2] = X[j] * A[j][0] + Y[j] * A[j][1] + A[j][2];
  }
  // reverse through the Cox-de Boor triangle, the degree P - k adjoint dN[k]
  // joining at level P - k (zero above min(r, P))
  double Nb[P + 1];
#pragma unroll
  for (int q = 0; q <= P; ++q) Nb[q] = dN[0][q];
  double ub = 0.0;
#pragma unroll
  for (int d = P; d >= 1; --d) {
    if (P - d >= 1 && P - d <= RM) {
#pragma unroll
      for (int q = 0; q <= d; ++q) Nb[q] += dN[P - d][q];
    }
    triangle_reverse<PD, P>(d, left, right, inv, tri, Nb, ub, out.knot);
  }
  out.ubar = ub;
  return value;
}

template <int PD>
__device__ inline double deriv_adjoint(const nsplat_curves& cv, const CurveView& v, double u, int span, int r,
                                       double scale, PtAdj<PD>& out, const double* up = nullptr) {
  if constexpr (PD >= 5) {
    if (v.p == 5) return deriv_adjoint_deg<PD, 5>(cv, v, u, span, r, scale, out, up);
    if (v.p == 4) return deriv_adjoint_deg<PD, 4>(cv, v, u, span, r, scale, out, up);
  }
  if (v.p == 3) return deriv_adjoint_deg<PD, 3>(cv, v, u, span, r, scale, out, up);
  if (v.p == 2) return deriv_adjoint_deg<PD, 2>(cv, v, u, span, r, scale, out, up);
  return deriv_adjoint_deg<PD, 1>(cv, v, u, span, r, scale, out, up);
}

// Penalty of Eq. 12 and its derivative: ReLU (kind 0) or softplus (kind 1).
__device__ inline double penalty(double x, int kind, double* d) {
  if (kind == 0) {
    *d = x > 0.0 ? 1.0 : 0.0;
    return x > 0.0 ? x : 0.0;
  }
  *d = 1.0 / (1.0 + exp(-x));
  return x > 0.0 ? x + log1p(exp(-x)) : log1p(exp(x));
}

struct RegArgs {
  double bbox_weight, deriv_weight;
  int bbox_kind, deriv_order;
  const float* bbox;
  float* loss;
};

// The scene's box: the given one, or the canvas [0, W] x [0, H].
__device__ inline void scene_box(const RegArgs& ra, const SceneTab* scenes, int s, double (&b)[4]) {
  if (ra.bbox) {
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (double)ra.bbox[4 * s + i];
  } else {
    b[0] = 0.0;
    b[1] = 0.0;
    b[2] = (double)scenes[s].W;
    b[3] = (double)scenes[s].H;
  }
}

// Bounding-box penalty of one point and its gradient.
__device__ inline double box_penalty(const RegArgs& ra, const double (&b)[4], double x, double y, double* gx,
                                     double* gy) {
  double d0, d1, d2, d3;
  const double v = penalty(b[0] - x, ra.bbox_kind, &d0) + penalty(x - b[2], ra.bbox_kind, &d1) +
                   penalty(b[1] - y, ra.bbox_kind, &d2) + penalty(y - b[3], ra.bbox_kind, &d3);
  *gx = ra.bbox_weight * (d1 - d0);
  *gy = ra.bbox_weight * (d3 - d2);
  return ra.bbox_weight * v;
}

// Number of curves of scene s (curves are grouped by scene in ascending order).
__device__ inline int curves_in_scene(const nsplat_curves& cv, int s) {
  int lo = 0, hi = cv.n_curves;  // first curve with scene >= s
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (cv.scene[mid] < s) lo = mid + 1;
    else hi = mid;
  }
  int a = lo;
  hi = cv.n_curves;  // first curve with scene > s
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (cv.scene[mid] <= s) lo = mid + 1;
    else hi = mid;
  }
  return lo - a;
}

// Trapezoid (open) or rectangle (closed) weight of sample j of `count`.
__device__ inline double quad_weight(int j, int count, bool closed) {
  if (closed) return 1.0 / (double)count;
  return (j == 0 || j == count - 1) ? 0.5 / (double)(count - 1) : 1.0 / (double)(count - 1);
}

// Block sum of two values into loss[0], loss[1] (one atomic each per block).
__device__ inline void block_loss(double a, double b, float* loss) {
  __shared__ double red[2][4];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
  }
  if (__lane_id() == 0) {
    red[0][threadIdx.x >> 6] = a;
    red[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0 && loss) {
    const double ta = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    const double tb = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    if (ta != 0.0) unsafeAtomicAdd(loss, (float)ta);
    if (tb != 0.0) unsafeAtomicAdd(loss + 1, (float)tb);
  }
}

// Registers for one wavefront per SIMD: held to two (256 VGPRs) the derivative
// adjoint spills about 110 to scratch (1.8M samples: 0.261 ms against 0.254;
// 0.375 before the fixed degrees, the reciprocals and the LDS sums).
// Stroke samples (one lane per stroke Gaussian; endpoint copies skipped): the
// box gradient joins the Gaussian's centre adjoint, the derivative loss goes
// straight to the control points, knots and domain ends.
template <int PD>
__global__ __launch_bounds__(256, 1) void k_reg_stroke(nsplat_curves cv, Work w, RegArgs ra, const int32_t* plan,
                                                    const int32_t* counters, const Gauss* __restrict__ gs,
                                                    int kappa, int run) {
  __shared__ PointSums<PD> sums[4];
  if (w.queue[Q_NSTROKE] == 0) return;  // no Gaussians of this kind
  const int64_t G = counters[NSPLAT_CNT_GAUSS];
  const int lane = __lane_id();
  double lb = 0.0, ld = 0.0;
  DomainSums dom;
  for (GroupWalk gw(run); gw.base < G; gw.next()) {
    const int64_t g = gw.base + lane;
    int64_t kspan = 0;
    double da = 0.0, db = 0.0;
    PtAdj<PD> pa;
    int c = 0, span = 0;
    CurveView v;
    v.p = 0;
    bool act = false;
    if (g < G) {
      const Gauss rec = gs[g];
      c = rec.curve;
      v = curve_view(cv, w.knots, c);
      const int32_t* row = plan + (int64_t)P_STRIDE * c;
      const int M = row[P_NSAMP];
      const int j = v.closed() ? rec.local : rec.local - kappa;
      if (!v.filled() && curve_valid(v) && j >= 0 && j < M) {
        if (ra.bbox_weight != 0.0) {
          double b[4], gx, gy;
          scene_box(ra, w.scenes, cv.scene[c], b);
          lb += box_penalty(ra, b, rec.mx, rec.my, &gx, &gy);
          float* gg = w.ggrad + g * GG;
          gg[0] += (float)gx;
          gg[1] += (float)gy;
        }
        if (ra.deriv_weight != 0.0) {
          act = true;
          double dt;
          const double u = sample_u(v.U[v.p], v.U[v.m - v.p], j, M, v.closed(), &dt);
          span = find_span(v.U, v.p, v.m, u);
          const double sc = ra.deriv_weight / (double)curves_in_scene(cv, cv.scene[c]) *
                            quad_weight(j, M, v.closed());
          ld += deriv_adjoint(cv, v, u, span, ra.deriv_order, sc, pa);
          da = pa.ubar * (1.0 - dt);
          db = pa.ubar * dt;
          kspan = (int64_t)v.t0 + (int64_t)c * KNOT_PAD + span;
        }
      }
    }
    if (!act) {
#pragma unroll
      for (int q = 0; q <= PD; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) pa.cp[q][k] = 0.0;
#pragma unroll
      for (int k = 0; k < 2 * PD; ++k) pa.knot[k] = 0.0;
    }
    accumulate_points(w, &sums[threadIdx.x >> 6], act, kspan, c, v, span, pa);
    dom.add(w, act, c, v, da, db);
  }
  dom.flush(w);
  block_loss(lb, ld, ra.loss);
}

// Fill boundary samples (one lane per boundary point): the box gradient joins
// the boundary-point adjoint, the derivative loss goes straight to the curve.
template <int PD>
__global__ __launch_bounds__(256, 1) void k_reg_boundary(nsplat_curves cv, Work w, RegArgs ra, const int32_t* plan,
                                                      const int32_t* counters) {
  __shared__ PointSums<PD> sums[4];
  const int64_t NB = counters[NSPLAT_CNT_BOUND];
  const int lane = __lane_id();
  const int n = cv.n_curves;
  double lb = 0.0, ld = 0.0;
  DomainSums dom;
  for (GroupWalk gw(1); gw.base < NB; gw.next()) {
    const int64_t bi = gw.base + lane;
    int64_t kspan = 0;
    double da = 0.0, db = 0.0;
    PtAdj<PD> pa;
    int c = 0, span = 0;
    CurveView v;
    v.p = 0;
    bool act = false;
    if (bi < NB) {
      c = last_le_wave<P_STRIDE, P_BOFF>(plan, n, bi);  // the last c with boff <= bi
      v = curve_view(cv, w.knots, c);
      const int32_t* row = plan + (int64_t)P_STRIDE * c;
      const int nb = row[P_NSAMP];
      const int j = (int)(bi - row[P_BOFF]);
      if (v.filled() && curve_valid(v) && j >= 0 && j < nb) {
        if (ra.bbox_weight != 0.0) {
          double b[4], gx, gy;
          scene_box(ra, w.scenes, cv.scene[c], b);
          const double2 q = w.bpts[bi];
          lb += box_penalty(ra, b, q.x, q.y, &gx, &gy);
          w.gb[bi].x += gx;
          w.gb[bi].y += gy;
        }
        if (ra.deriv_weight != 0.0) {
          act = true;
          double dt;
          const double u = sample_u(v.U[v.p], v.U[v.m - v.p], j, nb, true, &dt);
          span = find_span(v.U, v.p, v.m, u);
          const double sc = ra.deriv_weight / (double)curves_in_scene(cv, cv.scene[c]) * quad_weight(j, nb, true);
          ld += deriv_adjoint(cv, v, u, span, ra.deriv_order, sc, pa);
          da = pa.ubar * (1.0 - dt);
          db = pa.ubar * dt;
          kspan = (int64_t)v.t0 + (int64_t)c * KNOT_PAD + span;
        }
      }
    }
    if (!act) {
#pragma unroll
      for (int q = 0; q <= PD; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) pa.cp[q][k] = 0.0;
#pragma unroll
      for (int k = 0; k < 2 * PD; ++k) pa.knot[k] = 0.0;
    }
    accumulate_points(w, &sums[threadIdx.x >> 6], act, kspan, c, v, span, pa);
    dom.add(w, act, c, v, da, db);
  }
  dom.flush(w);
  block_loss(lb, ld, ra.loss);
}

// Tangent-aligned stroke Gaussians: centre mu = C(u_j), sp = s(u_j) / rho
// across the curve, sigma = max(sp, |C'(u_j)| du / rho) along
// t = C'(u_j) / |C'(u_j)| = (cos theta, sin theta), du the sample spacing.
// dL/d(mu, sp) and, where sigma = sp, dL/dsigma go to the point adjoint;
// dL/dtheta (d theta / d C' = n / |C'|, n = (-t_y, t_x)) and, where the
// spacing term is the larger, dL/dsigma (d sigma / d C' = t du / rho) go to
// the adjoint of the first derivative C'(u_j), whose reverse pass is that of
// the derivative loss; dL/d du = dL/dsigma |C'| / rho goes to the domain
// ends (du = (u_{m-p} - u_p) / (M - 1), or / M closed).
template <int PD>
__global__ __launch_bounds__(256, 1) void k_adj_aniso(nsplat_curves cv, nsplat_params pr, Work w,
                                                   const int32_t* plan, const int32_t* counters,
                                                   const Gauss* __restrict__ gs) {
  __shared__ PointSums<PD> sums[4];
  if (w.queue[Q_NANISO] == 0) return;  // no Gaussians of this kind
  const int64_t G = counters[NSPLAT_CNT_GAUSS];
  const int lane = __lane_id();
  const double rho = (double)pr.rho;
  DomainSums dom;
  for (GroupWalk gw(1); gw.base < G; gw.next()) {
    const int64_t g = gw.base + lane;
    int64_t kspan = 0;
    double da = 0.0, db = 0.0;
    PtAdj<PD> pa;
    int c = 0, span = 0;
    CurveView v;
    v.p = 0;
    bool act = false;
    if (g < G) {
      const Gauss r = gs[g];
      c = r.curve;
      if ((cv.flags[c] & (NSPLAT_FILLED | NSPLAT_ANISO)) == NSPLAT_ANISO) {
        act = true;
        v = curve_view(cv, w.knots, c);
        const float* gg = w.ggrad + g * GG;
        const int32_t* row = plan + (int64_t)P_STRIDE * c;
        const int M = row[P_NSAMP];
        int j = v.closed() ? r.local : r.local - pr.kappa;
        j = j < 0 ? 0 : (j > M - 1 ? M - 1 : j);
        double dt;
        const double u = sample_u(v.U[v.p], v.U[v.m - v.p], j, M, v.closed(), &dt);
        span = find_span(v.U, v.p, v.m, u);
        double pt[3], d[3];
        curve_point(cv, v, u, span, pt, d);
        const double len = sqrt(d[0] * d[0] + d[1] * d[1]);
        const double den = (double)(v.closed() ? M : M - 1);
        const double du = (v.U[v.m - v.p] - v.U[v.p]) / den;
        const double sp = pt[2] / rho;
        const bool wide = len > 0.0 && len * du / rho > sp;  // the spacing term sets sigma
        const double gsig = (double)gg[2], gsp = (double)gg[3], gth = (double)gg[4];
        const double ab[3] = {(double)gg[0], (double)gg[1], (gsp + (wide ? 0.0 : gsig)) / rho};
        point_adjoint(cv, v, u, span, ab, pa);
        double ddu = 0.0;
        if (len > 0.0) {
          const double tx = d[0] / len, ty = d[1] / len;
          double up[2] = {-ty * gth / len, tx * gth / len};
          if (wide) {
            up[0] += gsig * tx * du / rho;
            up[1] += gsig * ty * du / rho;
            ddu = gsig * len / rho;
          }
          PtAdj<PD> pd;
          deriv_adjoint(cv, v, u, span, 1, 0.0, pd, up);
#pragma unroll
          for (int q = 0; q <= PD; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) pa.cp[q][k] += pd.cp[q][k];
#pragma unroll
          for (int k = 0; k < 2 * PD; ++k) pa.knot[k] += pd.knot[k];
          pa.ubar += pd.ubar;
        }
        da = pa.ubar * (1.0 - dt) - ddu / den;  // u_j = u_p + t_j (u_{m-p} - u_p)
        db = pa.ubar * dt + ddu / den;
        kspan = (int64_t)v.t0 + (int64_t)c * KNOT_PAD + span;
      }
    }
    if (!act) {
#pragma unroll
      for (int q = 0; q <= PD; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) pa.cp[q][k] = 0.0;
#pragma unroll
      for (int k = 0; k < 2 * PD; ++k) pa.knot[k] = 0.0;
    }
    accumulate_points(w, &sums[threadIdx.x >> 6], act, kspan, c, v, span, pa);
    dom.add(w, act, c, v, da, db);
  }
  dom.flush(w);
}

}  // namespace

hipError_t launch_zero_grads(const Launch& L) {
  Phase ph(L, NSPLAT_T_FOLD);
  const nsplat_curves& cv = *L.cv;
  const int64_t ncp = (int64_t)cv.n_keys + (int64_t)cv.n_curves * CP_PAD;
  const int64_t nkn = (int64_t)cv.n_taus + (int64_t)cv.n_curves * KNOT_PAD;
  ZeroSet z;
  z.p[0] = L.w.gcp;
  z.n[0] = 4 * ncp;
  z.p[1] = L.w.gknot;
  z.n[1] = nkn;
  z.p[2] = L.w.gcurve;
  z.n[2] = (int64_t)4 * cv.n_curves;
  z.p[3] = (double*)L.w.gb;
  z.n[3] = L.bf->caps.boundary > 0 ? 2 * L.bf->caps.boundary : 0;
  const int64_t total = z.n[0] + z.n[1] + z.n[2] + z.n[3];
  const int64_t most = std::max<int64_t>(L.bf->caps.gauss * GG, total);
  hipLaunchKernelGGL(k_zero_grads, dim3(grid_for(most, 256, 8192)), dim3(256), 0, L.stream, L.w.ggrad,
                     L.bf->counters + NSPLAT_CNT_GAUSS, (int64_t)GG, (int64_t)L.bf->caps.gauss, z);
  return hipGetLastError();
}

// Array bound of the point and derivative adjoints: 3 when the batch declares
// no degree above 3 (curve_valid rejects any curve above the bound).
inline bool low_degree(const Launch& L) { return L.cv->max_degree >= 1 && L.cv->max_degree <= 3; }

// Groups of 64 samples that a wavefront of the stroke adjoints takes in a row
// (see DomainSums): four where that still leaves two wavefronts per SIMD, one
// below, where the launch would lose wavefronts it needs.
inline int sample_run(const Launch& L) { return L.bf->caps.gauss >= (int64_t)4 * 64 * 8 * L.n_cu ? 4 : 1; }

template <int PD>
void launch_reg_d(const Launch& L, const RegArgs& ra) {
  hipLaunchKernelGGL(k_reg_stroke<PD>, dim3(grid_for(L.bf->caps.gauss, 256 * sample_run(L), 4096)), dim3(256), 0, L.stream, *L.cv,
                     L.w, ra, L.bf->plan, L.bf->counters, (const Gauss*)L.bf->gauss, L.pr->kappa, sample_run(L));
  if (L.bf->caps.boundary > 0)
    hipLaunchKernelGGL(k_reg_boundary<PD>, dim3(grid_for(L.bf->caps.boundary, 256, 4096)), dim3(256), 0, L.stream,
                       *L.cv, L.w, ra, L.bf->plan, L.bf->counters);
}

template <int PD>
void launch_adj_stroke_d(const Launch& L) {
  hipLaunchKernelGGL(k_adj_stroke<PD>, dim3(grid_for(L.bf->caps.gauss, 256 * sample_run(L), 8192)), dim3(256), 0, L.stream, *L.cv,
                     *L.pr, L.w, L.bf->plan, L.bf->counters, (const Gauss*)L.bf->gauss, sample_run(L));
}

template <int PD>
void launch_adj_aniso_d(const Launch& L) {
  hipLaunchKernelGGL(k_adj_aniso<PD>, dim3(grid_for(L.bf->caps.gauss, 256, 4096)), dim3(256), 0, L.stream, *L.cv,
                     *L.pr, L.w, L.bf->plan, L.bf->counters, (const Gauss*)L.bf->gauss);
}

template <int PD>
void launch_adj_boundary_d(const Launch& L) {
  hipLaunchKernelGGL(k_adj_boundary<PD>, dim3(grid_for(L.bf->caps.boundary, 256, 4096)), dim3(256), 0, L.stream,
                     *L.cv, L.w, L.bf->plan, L.bf->counters);
}

hipError_t launch_reg(const Launch& L, const nsplat_reg* reg) {
  Phase ph(L, NSPLAT_T_REG);
  RegArgs ra;
  ra.bbox_weight = (double)reg->bbox_weight;
  ra.deriv_weight = (double)reg->deriv_weight;
  ra.bbox_kind = reg->bbox_kind;
  ra.deriv_order = reg->deriv_order;
  ra.bbox = reg->bbox;
  ra.loss = reg->loss;
  if (low_degree(L)) launch_reg_d<3>(L, ra);
  else launch_reg_d<MAXP>(L, ra);
  return hipGetLastError();
}

hipError_t launch_adjoint(const Launch& L, const nsplat_grads* g) {
  {
    Phase ph(L, NSPLAT_T_ADJ_GAUSS);
    // kinds the batch declares none of are not launched (any_flags, all_flags)
    const bool ani = (L.cv->any_flags & NSPLAT_ANISO) != 0;
    const bool strokes = (L.cv->all_flags & NSPLAT_FILLED) == 0;
    const bool fills = (L.cv->any_flags & NSPLAT_FILLED) != 0;
    if (low_degree(L)) {
      if (strokes) launch_adj_stroke_d<3>(L);
      if (ani) launch_adj_aniso_d<3>(L);
    } else {
      if (strokes) launch_adj_stroke_d<MAXP>(L);
      if (ani) launch_adj_aniso_d<MAXP>(L);
    }
    if (fills)
      hipLaunchKernelGGL(k_adj_fill, dim3(grid_for(L.bf->caps.gauss, 256, 8192)), dim3(256), 0, L.stream, *L.cv,
                         *L.pr, L.w, L.bf->plan, L.bf->counters, (const Gauss*)L.bf->gauss);
  }
  if (L.bf->caps.boundary > 0 && (L.cv->any_flags & NSPLAT_FILLED)) {
    Phase ph(L, NSPLAT_T_ADJ_BOUND);
    if (low_degree(L)) launch_adj_boundary_d<3>(L);
    else launch_adj_boundary_d<MAXP>(L);
  }
  Phase ph(L, NSPLAT_T_FOLD);
  if (L.cv->n_curves > 0) {
    // long curves on average (a launch counts its threads in 32 bits)
    if ((int64_t)L.cv->n_taus > 128 * (int64_t)L.cv->n_curves && L.cv->n_curves < (1 << 21))
      hipLaunchKernelGGL(k_fold<1024>, dim3(L.cv->n_curves), dim3(1024), 0, L.stream, *L.cv, L.w, *g);
    else
      hipLaunchKernelGGL(k_fold<64>, dim3(L.cv->n_curves), dim3(64), 0, L.stream, *L.cv, L.w, *g);
  }
  return hipGetLastError();
}

}  // namespace nsp
