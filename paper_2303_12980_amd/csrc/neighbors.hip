// Neighbour build: lattice wrap, cell-list binning, per-centre count, fill
// and canonical sort, reverse-pair index.
//
// The cutoff is inferred from the overlap threshold (the paper's "Examples"
// section): a pair (j, n) belongs to centre i when its squared distance q is
// at most the largest rc(sigma)^2.  Image shifts n range over every lattice
// translation on periodic axes, so atoms (and the centre itself) appear as
// often as they fit inside the cutoff sphere.
//
// Floating point: reciprocal rows, fractional coordinates, wrap, image
// shifts, displacements and q are FP64 in a fixed operation order with no
// contraction (the file is built with -ffp-contract=off), so every kernel that
// recomputes q gets the same bits and (j,i,-n) has exactly the q of (i,j,n).
//
// Cell list: fractional space of each structure is cut into nb_k bins per
// periodic axis (edge ~ rc_max / bin_divisor); a centre visits the "virtual"
// bins V_k in [floor((f_k - reach_k) nb_k), floor((f_k + reach_k) nb_k)],
// each of which is real bin V mod nb with image shift floor(V / nb).  Atoms
// are stored bin-sorted in SoA arrays so a bin is read with coalesced loads.
#include "gmp_internal.h"
#include "pair_key.h"

namespace gmp {
namespace {

__device__ inline void cross3(const double *a, const double *b, double *c) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ inline double dot3(const double *a, const double *b) { return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2]; }

__device__ inline int floordiv(int a, int b) { int q = a / b; return (a % b != 0 && ((a < 0) != (b < 0))) ? q - 1 : q; }
__device__ inline int pmod(int a, int b) { int r = a % b; return r < 0 ? r + b : r; }

// Structure s: reciprocal rows, reach, bins.  Faults of the lattice are kept in
// it (err) and reported by the next step, so that it can run beside the
// clearing of the status word.
__device__ inline void struct_setup(const BatchDev &bt, StructInfo *info, int s, double rcmax, int bin_div) {
  StructInfo I;
  I.err = 0;
  const int pbc = bt.pbc[s] & 7;
  const int64_t n_s = bt.atom_offsets[s + 1] - bt.atom_offsets[s];
  I.pbc = pbc;
  I.bin_base = bt.atom_offsets[s] + s;
#pragma unroll
  for (int k = 0; k < 9; ++k) I.b[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) { I.nb[k] = 1; I.reach[k] = 0.0; }
  I.lam_lo = 0.0;
  if (pbc) {
    const double *a = bt.cell + 9 * (int64_t)s;
    double c23[3], c31[3], c12[3];
    cross3(a + 3, a + 6, c23);
    cross3(a + 6, a, c31);
    cross3(a, a + 3, c12);
    double V = dot3(a, c23);
    bool ok = isfinite(V) && V != 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) ok = ok && isfinite(a[k]);
    if (!ok) {
      I.err |= ST_CELL;
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k) { I.b[k] = c23[k] / V; I.b[3 + k] = c31[k] / V; I.b[6 + k] = c12[k] / V; }
      const double ell = rcmax / (double)bin_div;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (!(pbc & (1 << k))) continue;
        double inv_h = sqrt(dot3(I.b + 3 * k, I.b + 3 * k));
        double h = 1.0 / inv_h;
        double nbk = ell > 0.0 ? floor(h / ell) : 1.0;
        if (!(nbk >= 1.0)) nbk = 1.0;
        if (nbk > 1024.0) nbk = 1024.0;
        I.nb[k] = (int)nbk;
        I.reach[k] = rcmax * inv_h * (1.0 + 1e-12) + 1e-12;
        // image shifts must fit a signed byte
        if (I.reach[k] + 2.0 > 126.0) I.err |= ST_SHIFT_RANGE;
      }
      // smallest eigenvalue of the metric G = A A^T (rows of A are the lattice vectors), for a lower
      // bound |n.A|^2 >= lambda_min |n|^2 that lets the cell list skip bin images outside the cutoff
      {
        double Gm[3][3];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) Gm[r][c] = dot3(a + 3 * r, a + 3 * c);
        const double p1 = Gm[0][1] * Gm[0][1] + Gm[0][2] * Gm[0][2] + Gm[1][2] * Gm[1][2];
        const double qq = (Gm[0][0] + Gm[1][1] + Gm[2][2]) / 3.0;
        const double d0 = Gm[0][0] - qq, d1 = Gm[1][1] - qq, d2 = Gm[2][2] - qq;
        const double p2 = d0 * d0 + d1 * d1 + d2 * d2 + 2.0 * p1;
        double lmin;
        if (p2 <= 0.0) {
          lmin = qq;
        } else {
          const double pp = sqrt(p2 / 6.0);
          const double b00 = d0 / pp, b11 = d1 / pp, b22 = d2 / pp;
          const double b01 = Gm[0][1] / pp, b02 = Gm[0][2] / pp, b12 = Gm[1][2] / pp;
          double r = 0.5 * (b00 * (b11 * b22 - b12 * b12) - b01 * (b01 * b22 - b12 * b02) + b02 * (b01 * b12 - b11 * b02));
          r = r < -1.0 ? -1.0 : (r > 1.0 ? 1.0 : r);
          const double phi = acos(r) / 3.0;
          lmin = qq + 2.0 * pp * cos(phi + 2.0943951023931957);
        }
        I.lam_lo = (isfinite(lmin) && lmin > 0.0) ? 0.99 * lmin : 0.0;
      }
      // never more bins than atoms (bin slots per structure are n_s + 1)
      int64_t cap = n_s > 1 ? n_s : 1;
      // (constant indices only: an array indexed at run time would live in scratch memory)
      int n0 = I.nb[0], n1 = I.nb[1], n2 = I.nb[2];
      while ((int64_t)n0 * n1 * n2 > cap) {
        const int m01 = n1 > n0 ? n1 : n0;
        if (n2 > m01) n2 = n2 > 1 ? (n2 + 1) / 2 : 1;
        else if (n1 > n0) n1 = n1 > 1 ? (n1 + 1) / 2 : 1;
        else n0 = n0 > 1 ? (n0 + 1) / 2 : 1;
      }
      I.nb[0] = n0; I.nb[1] = n1; I.nb[2] = n2;
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) I.inv_nb[k] = 1.0 / (double)I.nb[k];
  info[s] = I;
}

// Clears the status words, the forward's word for diverged positions and the bin
// counters, and sets up the structures.
__global__ __launch_bounds__(256) void k_setup(BatchDev bt, StructInfo *info, double rcmax, int bin_div,
                                               uint32_t *status, unsigned long long *counter, int32_t *bin_count, int32_t *bin_fill,
                                               int64_t n_bins) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 64) status[i] = 0u;
  if (i == 0) counter[1] = 0ull;
  if (i < n_bins) { bin_count[i] = 0; bin_fill[i] = 0; }
  if (i < bt.n_structs) struct_setup(bt, info, (int)i, rcmax, bin_div);
}

// Range of atom indices (of P.sub equal ones over the structure) that an atom
// falls into: monotone in the index, so the ranges of a bucket are in order.
struct SubRange {
  int64_t first;
  float scale;
  int last;
  __device__ SubRange(const PlanDev &P, const BatchDev &bt, int s) {
    first = bt.atom_offsets[s];
    const int64_t n = bt.atom_offsets[s + 1] - first;
    scale = n > 0 ? (float)P.sub / (float)n : 0.f;
    last = P.sub - 1;
  }
  __device__ int of(int32_t j) const {
    const int r = (int)((float)(int32_t)(j - first) * scale);
    return r < last ? r : last;
  }
};

// One thread per index g: atoms (wrapped, binned) and reference points
// (wrapped only; they are centres, never neighbours).  rw, wrap and fw are
// over the n_total indices.
__device__ inline void wrap_index(const BatchDev &bt, const StructInfo *info, const NbrDev &nb, double *fw,
                                  int32_t *bin_of, int32_t *bin_count, int32_t *astruct, int32_t *range_col,
                                  const PlanDev &P, uint32_t *status, int64_t i) {
  const int64_t N = n_total(bt);
  if (i < bt.n_structs && info[i].err) atomicOr(status, info[i].err);
  if (i >= N) return;
  const bool atom = i < bt.n_atoms;
  if (atom) {
    const int sp = bt.species[i];
    if (sp < 0 || sp >= P.E) atomicOr(status, ST_SPECIES);
  }
  const int s = struct_of_index(bt, i);
  if (atom) {
    const int sp = bt.species[i];
    range_col[i] = (sp < 0 ? 0 : (sp >= P.E ? P.E - 1 : sp)) * P.sub + SubRange(P, bt, s).of((int32_t)i);
  }
  astruct[i] = s;
  const StructInfo &I = info[s];
  const int64_t k = atom ? i : i - bt.n_atoms;
  // (pointers as values, each with its index: a choice between the members'
  // addresses would put the batch descriptor in scratch memory)
  const double *X = bt.x + i, *Y = bt.y + i, *Z = bt.z + i;
  asm volatile("" : "+v"(X), "+v"(Y), "+v"(Z));
  if (!atom) { X = bt.px + k; Y = bt.py + k; Z = bt.pz + k; }
  const double R[3] = {*X, *Y, *Z};
  if (!(isfinite(R[0]) && isfinite(R[1]) && isfinite(R[2]))) atomicOr(status, ST_NONFINITE);
  if (atom && bt.occ && !isfinite(bt.occ[i])) atomicOr(status, ST_NONFINITE);
  int m[3] = {0, 0, 0};
  int b[3] = {0, 0, 0};
  double f3[3] = {0.0, 0.0, 0.0};
  double rwv[3] = {R[0], R[1], R[2]};
  if (I.pbc) {
    const double *a = bt.cell + 9 * (int64_t)s;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (!(I.pbc & (1 << k))) continue;
      double f = dot3(R, I.b + 3 * k);
      if (!(fabs(f) < 1.0e9)) { atomicOr(status, ST_NONFINITE); f = 0.0; }
      double fl = floor(f);
      m[k] = (int)fl;
      double w = f - fl;  // exact, in [0, 1)
      f3[k] = w;
      int bk = (int)(w * (double)I.nb[k]);
      if (bk > I.nb[k] - 1) bk = I.nb[k] - 1;
      if (bk < 0) bk = 0;
      b[k] = bk;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double t = (double)m[0] * a[c] + (double)m[1] * a[3 + c];
      t = t + (double)m[2] * a[6 + c];
      rwv[c] = R[c] - t;
    }
  }
  nb.rw[i] = rwv[0];
  nb.rw[N + i] = rwv[1];
  nb.rw[2 * N + i] = rwv[2];
  nb.wrap[3 * i] = m[0];
  nb.wrap[3 * i + 1] = m[1];
  nb.wrap[3 * i + 2] = m[2];
  fw[i] = f3[0];
  fw[N + i] = f3[1];
  fw[2 * N + i] = f3[2];
  if (!atom) {  // reference points keep their own list order
    nb.order[k] = (int32_t)k;
    nb.slot[k] = (int32_t)k;
    return;
  }
  int64_t bin = I.bin_base + ((int64_t)b[0] * I.nb[1] + b[1]) * I.nb[2] + b[2];
  bin_of[i] = (int32_t)bin;
  atomicAdd(&bin_count[bin], 1);
}

__global__ void k_wrap(BatchDev bt, const StructInfo *info, NbrDev nb, double *fw, int32_t *bin_of,
                       int32_t *bin_count, int32_t *astruct, int32_t *range_col, PlanDev P, uint32_t *status) {
  wrap_index(bt, info, nb, fw, bin_of, bin_count, astruct, range_col, P, status,
             (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Atoms into their bins, in arrival order (the slot within a bin comes
// from an atomic counter); bin_order then orders every bin by atom index.
__device__ inline void scatter_atom(const BatchDev &bt, const int32_t *bin_of, const int64_t *bin_start,
                                    int32_t *bin_fill, int32_t *sid_tmp, int64_t i) {
  if (i >= bt.n_atoms) return;
  int32_t b = bin_of[i];
  int64_t p = bin_start[b] + atomicAdd(&bin_fill[b], 1);
  sid_tmp[p] = (int32_t)i;
}

// Deterministic cell-list order: the atom at arrival slot p of bin b goes to
// position bin_start[b] + (number of atoms of b with a smaller index); the
// bin-sorted SoA copies (wrapped positions, atom index, species) are written
// there, and with atoms as centres the list-slot order follows it.  One
// thread per arrival slot; the threads of one bin read the same members.
__device__ inline void bin_order(const BatchDev &bt, const NbrDev &nb, const int32_t *bin_of, const int64_t *bin_start,
                                 const int32_t *sid_tmp, double *sx, double *sy, double *sz, int32_t *sid,
                                 int32_t *ssp, int n_elements, int64_t p) {
  if (p >= bt.n_atoms) return;
  const int64_t N = n_total(bt);  // stride of rw
  const int32_t i = sid_tmp[p];
  const int32_t b = bin_of[i];
  const int64_t lo = bin_start[b], hi = bin_start[b + 1];
  int64_t r = 0;
  for (int64_t q = lo; q < hi; ++q) r += sid_tmp[q] < i ? 1 : 0;
  const int64_t k = lo + r;
  sx[k] = nb.rw[i];
  sy[k] = nb.rw[N + i];
  sz[k] = nb.rw[2 * N + i];
  sid[k] = i;
  const int sp = bt.species[i];
  ssp[k] = sp < 0 ? 0 : (sp >= n_elements ? n_elements - 1 : sp);  // out-of-range species are flagged in k_wrap
  if (!point_mode(bt)) {
    nb.order[k] = i;
    nb.slot[i] = (int32_t)k;
  }
}

__global__ void k_scatter(BatchDev bt, const int32_t *bin_of, const int64_t *bin_start, int32_t *bin_fill,
                          int32_t *sid_tmp) {
  scatter_atom(bt, bin_of, bin_start, bin_fill, sid_tmp, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}
__global__ void k_bin_order(BatchDev bt, NbrDev nb, const int32_t *bin_of, const int64_t *bin_start,
                            const int32_t *sid_tmp, double *sx, double *sy, double *sz, int32_t *sid, int32_t *ssp,
                            int n_elements) {
  bin_order(bt, nb, bin_of, bin_start, sid_tmp, sx, sy, sz, sid, ssp, n_elements,
            (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// The whole cell list of a small batch by one workgroup: the steps of k_setup,
// k_wrap, the bin scan, k_scatter and k_bin_order between barriers, one launch
// in place of five (their launches, not their work, are the time of a call on
// tens or hundreds of atoms; with 4096 atoms one CU takes longer than the five).
constexpr int kSmallAtoms = 1024;
__global__ __launch_bounds__(kScanThreads) void k_small_cells(PlanDev P, BatchDev bt, NbrDev nb, StructInfo *info,
                                                              double rcmax, int bin_div, uint32_t *status,
                                                              unsigned long long *counter, int32_t *bin_count, int64_t *bin_start,
                                                              int32_t *bin_fill, double *fw, int32_t *bin_of,
                                                              int32_t *astruct, int32_t *range_col, int32_t *sid_tmp,
                                                              double *sx, double *sy, double *sz, int32_t *sid,
                                                              int32_t *ssp) {
  __shared__ int64_t words[kScanWords];
  const int t = threadIdx.x;  // at least as many threads as structures, atoms and points, and half the bins
  const int64_t n_bins = bt.n_atoms + bt.n_structs;
  if (t < 64) status[t] = 0u;
  if (t == 0) counter[1] = 0ull;
  for (int64_t i = t; i < n_bins; i += kScanThreads) { bin_count[i] = 0; bin_fill[i] = 0; }
  if (t < bt.n_structs) struct_setup(bt, info, t, rcmax, bin_div);
  __syncthreads();
  wrap_index(bt, info, nb, fw, bin_of, bin_count, astruct, range_col, P, status, t);
  __syncthreads();
  block_scan([&](int64_t i) { return (int64_t)bin_count[i]; }, bin_start, n_bins, words);
  __syncthreads();
  scatter_atom(bt, bin_of, bin_start, bin_fill, sid_tmp, t);
  __syncthreads();
  bin_order(bt, nb, bin_of, bin_start, sid_tmp, sx, sy, sz, sid, ssp, P.E, t);
}

// Range of virtual bins along axis k for a centre at fractional f.
__device__ inline void vrange(const StructInfo &I, int k, double f, int &lo, int &hi) {
  if (!(I.pbc & (1 << k))) { lo = hi = 0; return; }
  double nbk = (double)I.nb[k];
  lo = (int)floor((f - I.reach[k]) * nbk - 1e-6);
  hi = (int)floor((f + I.reach[k]) * nbk + 1e-6);
}

struct Cand {
  const StructInfo *I;
  const double *cell;
  double f[3];
  int lo[3], hi[3], nv[3];
  double inv_nv[3];
  int total;
};

__device__ inline void cand_setup(Cand &C, const StructInfo *info, const BatchDev &bt, int s,
                                  const double *fw, int64_t i) {
  const int64_t N = n_total(bt);  // stride of fw
  C.I = info + s;
  C.cell = bt.cell + 9 * (int64_t)s;
  C.f[0] = fw[i]; C.f[1] = fw[N + i]; C.f[2] = fw[2 * N + i];
  C.total = 1;
  for (int k = 0; k < 3; ++k) {
    vrange(*C.I, k, C.f[k], C.lo[k], C.hi[k]);
    C.nv[k] = C.hi[k] - C.lo[k] + 1;
    C.inv_nv[k] = 1.0 / (double)C.nv[k];
    C.total *= C.nv[k];
  }
}

// Virtual bin v (linear index) -> real bin slot and image shift; returns -1
// when the whole bin image lies outside the cutoff sphere (fractional gaps
// g_k to the centre satisfy lam_lo * |g|^2 > rc_max^2).
__device__ inline int64_t cand_bin(const Cand &C, int v, int n[3], double rcmax2) {
  // small non-negative / signed integer quotients through FP64 reciprocals:
  // (x + 1/2) / d keeps its fractional part at least 1/(2d) from an integer,
  // far above the rounding of the product
  int r[3];
  int t = v;
  int q = (int)floor(((double)t + 0.5) * C.inv_nv[2]);
  r[2] = t - q * C.nv[2]; t = q;
  q = (int)floor(((double)t + 0.5) * C.inv_nv[1]);
  r[1] = t - q * C.nv[1]; t = q;
  r[0] = t;
  int b[3];
  double g2 = 0.0;
  for (int k = 0; k < 3; ++k) {
    const int V = C.lo[k] + r[k];
    const int nbk = C.I->nb[k];
    n[k] = (int)floor(((double)V + 0.5) * C.I->inv_nb[k]);
    b[k] = V - n[k] * nbk;
    if (C.I->pbc & (1 << k)) {
      // bin-image bounds in fractional coordinates; a product with the
      // reciprocal is within 2 ulp of the quotient, far inside the 1e-9
      // slack that keeps the culling conservative
      const double x0 = (double)V * C.I->inv_nb[k], x1 = (double)(V + 1) * C.I->inv_nb[k];
      double g = x0 - C.f[k];
      const double g1 = C.f[k] - x1;
      g = g > g1 ? g : g1;
      g -= 1e-9;
      if (g > 0.0) g2 += g * g;
    }
  }
  if (C.I->lam_lo * g2 > rcmax2) return -1;
  return C.I->bin_base + ((int64_t)b[0] * C.I->nb[1] + b[1]) * C.I->nb[2] + b[2];
}

// Per-wavefront LDS scratch of the candidate enumeration.
struct CandLds {
  int delta[kWave];  // bin start minus the bin's first flattened position
  int npk[kWave];
  double sh[3][kWave];
};

// Calls f(t, n, shx, shy, shz) for every candidate atom t (index into the
// bin-sorted arrays) of every bin image that is not culled.  Bin images are
// taken 64 at a time (one per lane); their atoms are then flattened so that
// consecutive lanes read consecutive atoms.  With several wavefronts on one
// centre (wave w of nw), each wavefront takes every nw-th block of 64
// flattened candidates of every chunk.  The bin of flattened position c is
// the last lane whose exclusive prefix pre is <= c: the prefixes grow with the
// lane, so for a block starting at c0 it is the count of lanes with pre <= c0
// less one, moved on past every non-empty bin that starts inside the block
// (one or two for bins of tens of atoms).
template <typename F>
__device__ inline void for_each_candidate(const Cand &C, const int64_t *bin_start, double rcmax2, int w, int nw,
                                          CandLds &L, F &&f) {
  const int lane = lane_id();
  for (int v0 = 0; v0 < C.total; v0 += kWave) {
    const int v = v0 + lane;
    int cnt = 0, start = 0, npk = 0;
    double shx = 0.0, shy = 0.0, shz = 0.0;
    if (v < C.total) {
      int n[3];
      const int64_t bin = cand_bin(C, v, n, rcmax2);
      if (bin >= 0) {
        start = (int)bin_start[bin];
        cnt = (int)(bin_start[bin + 1] - start);
        npk = (n[0] & 0xff) | ((n[1] & 0xff) << 8) | ((n[2] & 0xff) << 16);
        if (C.I->pbc) image_shift(C.cell, n[0], n[1], n[2], shx, shy, shz);
      }
    }
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    const int tot = __shfl(incl, kWave - 1, kWave);
    const int pre = incl - cnt;  // lanes past the last bin image: pre = tot
    L.delta[lane] = start - pre;
    L.npk[lane] = npk;
    L.sh[0][lane] = shx;
    L.sh[1][lane] = shy;
    L.sh[2][lane] = shz;
    wave_lds_sync();
    for (int c0 = w * kWave; c0 < tot; c0 += nw * kWave) {
      const int c = c0 + lane;
      int own = __popcll(__ballot(pre <= c0)) - 1;
      for (uint64_t starts = __ballot(cnt > 0 && pre > c0 && pre - c0 < kWave); starts; starts &= starts - 1) {
        const int l = __builtin_ctzll(starts);
        if (c >= __builtin_amdgcn_readlane(pre, l)) own = l;
      }
      if (c < tot) {
        const int t = c + L.delta[own];
        const int pk = L.npk[own];
        const int n[3] = {(int)(int8_t)(pk & 0xff), (int)(int8_t)((pk >> 8) & 0xff), (int)(int8_t)((pk >> 16) & 0xff)};
        f(t, n, L.sh[0][own], L.sh[1][own], L.sh[2][own]);
      }
    }
    wave_lds_sync();
  }
}

// Shell of a squared distance q: the number of cutoffs rc2[s] < q.  The
// cutoffs sit in registers, padded to SM (8, 12 or 16) with +infinity, so
// the count is a fixed run of compares against uniform operands.
template <int SM>
struct Shells {
  double r[SM];
  __device__ explicit Shells(const PlanDev &P) {
#pragma unroll
    for (int s = 0; s < SM; ++s) r[s] = s < P.S ? P.rc2[s] : __builtin_huge_val();
  }
  __device__ int of(double q) const {
    int sh = 0;
#pragma unroll
    for (int s = 0; s < SM; ++s) sh += r[s] < q ? 1 : 0;
    return sh;
  }
};

// One workgroup per centre (centres in cell-list order): count neighbours
// per (shell, species) bucket and range of atom indices; the wavefronts share
// the centre's candidates.
template <int SM>
__global__ __launch_bounds__(256) void k_count(PlanDev P, BatchDev bt, NbrDev nb, const StructInfo *info,
                                               const double *fw, const int64_t *bin_start,
                                               const double *sx, const double *sy, const double *sz,
                                               const int32_t *sid, const int32_t *ssp, const int32_t *astruct,
                                               int32_t *cnt, int64_t *ptotal, int32_t *bmax, uint32_t *status) {
  extern __shared__ int32_t lds_cnt[];
  __shared__ CandLds lds_cand[4];
  __shared__ int64_t lds_tot[4];
  __shared__ int32_t lds_max[4];
  const int w = threadIdx.x / kWave, nw = blockDim.x / kWave, lane = lane_id();
  const int nbk = P.E * P.S * P.sub;
  int32_t *c = lds_cnt;
  const int64_t N = n_total(bt);  // stride of rw
  // list slot k (atoms: cell-list order, each XCD one contiguous range), centre i, index g
  const int64_t k = xcd_contiguous(blockIdx.x, gridDim.x);
  const int64_t i = point_mode(bt) ? k : sid[k];
  const int64_t g = centre_base(bt) + i;
  for (int t = threadIdx.x; t < nbk; t += blockDim.x) c[t] = 0;
  __syncthreads();
  const int s = astruct[g];
  Cand C;
  cand_setup(C, info, bt, s, fw, g);
  const Shells<SM> shells(P);
  const SubRange range(P, bt, s);
  const double rix = nb.rw[g], riy = nb.rw[N + g], riz = nb.rw[2 * N + g];
  for_each_candidate(C, bin_start, P.rcmax2, w, nw, lds_cand[w],
                     [&](int t, const int *n, double shx, double shy, double shz) {
                       const double dx = (sx[t] - rix) + shx;
                       const double dy = (sy[t] - riy) + shy;
                       const double dz = (sz[t] - riz) + shz;
                       const double q = (dx * dx + dy * dy) + dz * dz;
                       if (q <= P.rcmax2)
                         atomicAdd(&c[(shells.of(q) * P.E + ssp[t]) * P.sub + range.of(sid[t])], 1);
                     });
  __syncthreads();
  int64_t tot = 0;
  int32_t longest = 0;
  for (int t = threadIdx.x; t < nbk; t += blockDim.x) cnt[k * nbk + t] = c[t];
  for (int b = threadIdx.x; b < P.E * P.S; b += blockDim.x) {
    int32_t n = 0;
    for (int r = 0; r < P.sub; ++r) n += c[b * P.sub + r];
    tot += n;
    longest = n > longest ? n : longest;
  }
  for (int o = 32; o >= 1; o >>= 1) {
    tot += __shfl_xor(tot, o, kWave);
    const int32_t y = __shfl_xor(longest, o, kWave);
    longest = y > longest ? y : longest;
  }
  if (lane == 0) { lds_tot[w] = tot; lds_max[w] = longest; }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t all = 0;
    int32_t m = 0;
    for (int u = 0; u < nw; ++u) { all += lds_tot[u]; m = lds_max[u] > m ? lds_max[u] : m; }
    ptotal[k] = all;
    bmax[k] = m;
  }
}

// Longest list (status word 4) and longest (shell, species) bucket (word 5)
// of the counted lists, for the synchronous build's sort sizes: a grid-stride
// maximum over the centres with one atomic per workgroup and word.
__device__ inline void list_stats(const int64_t *ptotal, const int32_t *bucket_max, int64_t n_centres,
                                  uint32_t *status, int64_t block, int64_t n_blocks, int64_t (*lds_m)[16]) {
  const int w = threadIdx.x / kWave, lane = lane_id();
  const int64_t stride = n_blocks * blockDim.x;
  int64_t lmax = 0, bmax = 0;
  for (int64_t t = block * blockDim.x + threadIdx.x; t < n_centres; t += stride) {
    lmax = ptotal[t] > lmax ? ptotal[t] : lmax;
    bmax = bucket_max[t] > bmax ? bucket_max[t] : bmax;
  }
  for (int o = 32; o >= 1; o >>= 1) {
    const int64_t a = __shfl_xor(lmax, o, kWave), b = __shfl_xor(bmax, o, kWave);
    lmax = a > lmax ? a : lmax;
    bmax = b > bmax ? b : bmax;
  }
  if (lane == 0) { lds_m[0][w] = lmax; lds_m[1][w] = bmax; }
  __syncthreads();
  if (threadIdx.x < 2) {
    int64_t m = 0;
    for (int k = 0; k < (int)(blockDim.x / kWave); ++k) m = lds_m[threadIdx.x][k] > m ? lds_m[threadIdx.x][k] : m;
    if (m > 0) atomicMax(status + 4 + threadIdx.x, (uint32_t)(m > 0x7fffffff ? 0x7fffffff : m));
  }
}

__global__ __launch_bounds__(256) void k_list_stats(const int64_t *ptotal, const int32_t *bucket_max,
                                                    int64_t n_centres, uint32_t *status) {
  __shared__ int64_t lds_m[2][16];
  list_stats(ptotal, bucket_max, n_centres, status, blockIdx.x, gridDim.x, lds_m);
}

// The list offsets (first workgroup) and the list statistics (the others) of a
// synchronous build, which do not depend on each other, in one launch.
__global__ __launch_bounds__(kScanThreads) void k_offsets_stats(const int64_t *ptotal, const int32_t *bucket_max,
                                                                int64_t *offsets, int64_t n_centres,
                                                                uint32_t *status) {
  __shared__ int64_t words[kScanWords], lds_m[2][16];
  if (blockIdx.x == 0) block_scan([&](int64_t i) { return ptotal[i]; }, offsets, n_centres, words);
  else list_stats(ptotal, bucket_max, n_centres, status, blockIdx.x - 1, gridDim.x - 1, lds_m);
}

__device__ inline void cmpswap(uint64_t *a, int i, int l) {
  uint64_t x = a[i], y = a[l];
  if (x > y) { a[i] = y; a[l] = x; }
}

// Four elements e0 < e1 < e2 < e3 through two comparator stages in
// registers: mirror = true compares (e0, e3), (e1, e2) and then (e0, e1),
// (e2, e3); otherwise (e0, e2), (e1, e3) and then (e0, e1), (e2, e3).
// Positions >= n read as +infinity and are not written.
__device__ inline void group4(uint64_t *a, int n, int e0, int e1, int e2, int e3, bool mirror) {
  uint64_t x0 = e0 < n ? a[e0] : ~0ull, x1 = e1 < n ? a[e1] : ~0ull;
  uint64_t x2 = e2 < n ? a[e2] : ~0ull, x3 = e3 < n ? a[e3] : ~0ull;
  uint64_t u;
  if (mirror) {
    if (x0 > x3) { u = x0; x0 = x3; x3 = u; }
    if (x1 > x2) { u = x1; x1 = x2; x2 = u; }
  } else {
    if (x0 > x2) { u = x0; x0 = x2; x2 = u; }
    if (x1 > x3) { u = x1; x1 = x3; x3 = u; }
  }
  if (x0 > x1) { u = x0; x0 = x1; x1 = u; }
  if (x2 > x3) { u = x2; x2 = x3; x3 = u; }
  if (e0 < n) a[e0] = x0;
  if (e1 < n) a[e1] = x1;
  if (e2 < n) a[e2] = x2;
  if (e3 < n) a[e3] = x3;
}

// Sort a[0..n) of distinct keys ascending by one wavefront: bitonic network
// whose first merge stage compares mirror pairs, so every comparator is
// ascending and indices >= n act as +infinity without being touched.
__device__ void wave_sort(uint64_t *a, int n) {
  const int lane = lane_id();
  if (n <= 1) return;
  int lp2 = 1;
  while ((1 << lp2) < n) ++lp2;
  const int half = 1 << (lp2 - 1);
  // Comparators in groups of four that are closed under two consecutive
  // stages: each pass reads a lane's group once, compares in registers and
  // writes it once (indices >= n stay +infinity, never written); block
  // sizes are powers of two, so block and offset are shifts and masks.
  const int quarter = half >> 1;
  for (int lk = 1; lk <= lp2; ++lk) {
    const int k = 1 << lk;
    int lj;
    if (lk == 1) {  // blocks of two: the mirror stage alone
      for (int t = lane; t < half; t += kWave) {
        const int i = t << 1;
        if (i + 1 < n) cmpswap(a, i, i + 1);
      }
      wave_lds_sync();
      lj = -1;
    } else {  // mirror stage and the stage of distance k/4
      const int lq = lk - 2, Q = 1 << lq;
      for (int t = lane; t < quarter; t += kWave) {
        const int base = (t >> lq) << lk, off = t & (Q - 1);
        group4(a, n, base + off, base + off + Q, base + k - 1 - off - Q, base + k - 1 - off, true);
      }
      wave_lds_sync();
      lj = lk - 3;
    }
    for (; lj >= 1; lj -= 2) {  // the stages of distance j and j/2
      const int J = 1 << lj, H = J >> 1;
      for (int t = lane; t < quarter; t += kWave) {
        const int b = ((t >> (lj - 1)) << (lj + 1)) + (t & (H - 1));
        group4(a, n, b, b + H, b + J, b + J + H, false);
      }
      wave_lds_sync();
    }
    if (lj == 0) {  // a last stage of distance 1
      for (int t = lane; t < half; t += kWave) {
        const int i = t << 1;
        if (i + 1 < n) cmpswap(a, i, i + 1);
      }
      wave_lds_sync();
    }
  }
}

// Ranges of up to this many keys are ordered by counting, longer ones by the
// network of wave_sort (3000 atoms 0.077 ms, 0.072 at 64 and 256; 64 atoms,
// whose ranges hold 64 to 128 keys, 0.026 ms, 0.035 at 64).
constexpr int kRankMax = 128;
// Entries after the keys that read as larger than any key (the counting reads
// four keys at a time).
constexpr int kKeyPad = 4;

// Fill of one centre's list by one workgroup: its buckets (shell h,
// species e), in bucket order h * E + e, in LDS; every bucket sorted by
// (j, n); j / shift, the bucket starts and the sigma-prefix ends written.
// The sort: the keys are placed by bucket and range of atom indices as they
// are found; then every thread takes keys of the list in turn and counts those
// of its range that are smaller, which gives the entry's place in memory
// (ranges of different lengths side by side in a wavefront, no barrier and
// no LDS write; reading past a range's end meets only larger keys).  Long
// ranges are sorted in place first.  Bound by the enumeration's and the
// counting's instructions; against a sort of each whole bucket by one
// wavefront: 4096 atoms, 6.9e6 pairs 0.156 -> 0.096 ms; 60,000 atoms, 1.3e8
// pairs 2.93 -> 1.93 ms; 512 structures, 3.3e7 pairs 0.745 -> 0.52 ms (the
// count, which counts by range too, 5% slower: 0.054 -> 0.055 ms).
// The in-LDS sort holds lds_keys entries.  RANGED = false (the short-list
// kernel) takes lists that fit in one candidate pass and hands longer ones
// to the long-list queue; RANGED = true fills range by range of consecutive
// buckets that fit, enumerating the candidates once per range; a single
// bucket longer than the sort leaves placeholders and is reported.
template <bool RANGED, int SM>
__device__ inline void fill_centre(const PlanDev &P, const BatchDev &bt, const NbrDev &nb, const StructInfo *info,
                                   const double *fw, const int64_t *bin_start, const double *sx, const double *sy,
                                   const double *sz, const int32_t *sid, const int32_t *ssp, const int32_t *astruct,
                                   const int32_t *cnt, int lds_keys, uint64_t *pair_key, int32_t *pair_centre,
                                   int32_t *range_start, uint32_t *status, int32_t *long_q,
                                   int64_t k, int64_t i, uint64_t *keys, CandLds *lds_cand, int32_t &lds_bmax, int32_t &lds_rmax) {
  const int nbk = P.E * P.S;
  const int sub = P.sub, ns = nbk * sub;
  int32_t *sstart = (int32_t *)(keys + lds_keys + kKeyPad);  // [ns+1] starts of the ranges of every bucket
  int32_t *cursor = sstart + ns + 1;                         // [ns]
  auto bstart = [&](int b) { return sstart[b * sub]; };
  const int64_t g = centre_base(bt) + i;
  const int64_t N = n_total(bt);  // stride of rw
  const int tid = threadIdx.x, w = tid / kWave, nw = blockDim.x / kWave, lane = lane_id();
  const int64_t base = nb.offsets[k];
  const int64_t total = nb.offsets[k + 1] - base;
  const bool overflow = nb.offsets[k + 1] > nb.capacity;
  for (int t = tid; t < ns; t += blockDim.x) sstart[t] = cnt[k * ns + t];
  __syncthreads();
  if (w == 0) {  // starts: exclusive scan of the centre's counts, whole buckets per lane
    const int per = (nbk + kWave - 1) / kWave;
    int32_t sum = 0, vmax = 0, rmax = 0;
    for (int b = lane * per; b < (lane + 1) * per && b < nbk; ++b) {
      int32_t n = 0;
      for (int r = 0; r < sub; ++r) {
        const int32_t v = sstart[b * sub + r];
        n += v;
        rmax = v > rmax ? v : rmax;
      }
      sum += n;
      vmax = n > vmax ? n : vmax;
    }
    int32_t incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int32_t y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    int32_t at = incl - sum;
    for (int t = lane * per * sub; t < (lane + 1) * per * sub && t < ns; ++t) {
      const int32_t v = sstart[t];
      sstart[t] = at;
      at += v;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const int32_t y = __shfl_xor(vmax, o, kWave), z = __shfl_xor(rmax, o, kWave);
      vmax = y > vmax ? y : vmax;
      rmax = z > rmax ? z : rmax;
    }
    const int32_t all = __shfl(incl, kWave - 1, kWave);
    if (lane == 0) {
      sstart[ns] = all;
      lds_bmax = vmax;
      lds_rmax = rmax;
      if (overflow) atomicOr(status, ST_OVERFLOW);
      if (RANGED && vmax > lds_keys) atomicOr(status, ST_SORT_SIZE);
      if ((int64_t)all != total) atomicOr(status, ST_INTERNAL);
      // a list the short-list kernel cannot sort in one pass goes to the queue
      if (!RANGED && !overflow && total > lds_keys) long_q[atomicAdd(status + 6, 1u)] = (int32_t)k;
    }
  }
  __syncthreads();
  if (!RANGED && !overflow && total > lds_keys) return;  // the long-list kernel writes this centre
  for (int b = tid; b <= nbk; b += blockDim.x) {
    nb.bucket_start[k * (nbk + 1) + b] = bstart(b);
  }
  if (pair_key)  // rows by atom; pair indices are below 2^31 where there is a reverse index
    for (int t = tid; t <= ns; t += blockDim.x) range_start[i * (ns + 1) + t] = (int32_t)(base + sstart[t]);
  for (int s = tid; s < P.S; s += blockDim.x) nb.sigma_end[k * P.S + s] = bstart((P.rank_lt[s] + 1) * P.E);
  if (overflow) return;  // consumers skip centres whose list ends past the capacity
  if (RANGED && lds_bmax > lds_keys) {
    // a bucket does not fit the in-LDS sort: leave in-range placeholder
    // entries (the centre itself, or atom 0 for a reference point; no shift)
    // so no consumer reads outside its arrays; the status word reports it
    const int64_t jp = point_mode(bt) ? 0 : i;
    int ei = bt.species[jp];
    ei = ei < 0 ? 0 : (ei >= P.E ? P.E - 1 : ei);
    for (int64_t t = tid; t < total; t += blockDim.x) {
      nb.j[base + t] = (int32_t)jp;
      nb.shift[base + t] = (int32_t)((uint32_t)ei << 24);
      if (pair_key) {
        const uint64_t k = make_key(i, 0, 0, 0);
        pair_key[base + t] = k;
        pair_centre[base + t] = (int32_t)i;
        nb.reverse[base + t] = -1;
      }
    }
    return;
  }
  const int s = astruct[g];
  Cand C;
  cand_setup(C, info, bt, s, fw, g);
  const Shells<SM> shells(P);
  const SubRange range(P, bt, s);
  const double rix = nb.rw[g], riy = nb.rw[N + g], riz = nb.rw[2 * N + g];
  const int species_mask = bt.n_atoms <= kKeySpeciesAtoms ? kMaxElements - 1 : 0;
  // buckets [b_lo, b_hi) whose entries fit the sort together (all of them
  // in the short-list kernel)
  for (int b_lo = 0; b_lo < nbk;) {
    int b_hi = nbk;
    if (RANGED) {
      b_hi = b_lo + 1;
      while (b_hi < nbk && bstart(b_hi + 1) - bstart(b_lo) <= lds_keys) ++b_hi;
      b_hi = __builtin_amdgcn_readfirstlane(b_hi);  // the same for every thread
    }
    const int key0 = RANGED ? __builtin_amdgcn_readfirstlane(bstart(b_lo)) : 0;
    const int n_keys = bstart(b_hi) - key0;
    for (int t = b_lo * sub + tid; t < b_hi * sub; t += blockDim.x) cursor[t] = sstart[t] - key0;
    if (tid < kKeyPad) keys[n_keys + tid] = ~0ull;
    __syncthreads();
    for_each_candidate(C, bin_start, P.rcmax2, w, nw, lds_cand[w],
                       [&](int t, const int *n, double shx, double shy, double shz) {
                         const double dx = (sx[t] - rix) + shx;
                         const double dy = (sy[t] - riy) + shy;
                         const double dz = (sz[t] - riz) + shz;
                         const double q = (dx * dx + dy * dy) + dz * dz;
                         if (q <= P.rcmax2) {
                           const int sh = shells.of(q);
                           const int bk = sh * P.E + ssp[t];
                           if (!RANGED || (bk >= b_lo && bk < b_hi)) {
                             const int sk = bk * sub + range.of(sid[t]);
                             const int pos = atomicAdd(&cursor[sk], 1);
                             if (pos < sstart[sk + 1] - key0)
                               keys[pos] = make_key(sid[t], n[0], n[1], n[2], sh) |
                                           (uint64_t)(ssp[t] & species_mask) << kKeySpecies;
                             else atomicOr(status, ST_INTERNAL);
                           }
                         }
                       });
    __syncthreads();
    if (lds_rmax > kRankMax) {
      for (int t = b_lo * sub + w; t < b_hi * sub; t += nw) {
        const int s0 = sstart[t], n = sstart[t + 1] - s0;
        if (n > kRankMax) wave_sort(keys + (s0 - key0), n);
      }
      __syncthreads();
    }
    auto place = [&](int t, auto species) {
      constexpr bool SPECIES = decltype(species)::value;
      const uint64_t key = keys[t];
      int32_t j;
      int e;
      if constexpr (SPECIES) {
        j = (int32_t)key_atom_below_species(key);
        e = key_species(key);
      } else {
        j = (int32_t)key_atom(key);
        e = bt.species[j < bt.n_atoms ? j : 0];
        e = e < 0 ? 0 : (e >= P.E ? P.E - 1 : e);
      }
      const int b = key_shell(key) * P.E + e;
      if (b >= b_hi) { atomicOr(status, ST_INTERNAL); return; }  // never for lists that were counted alike
      const int sk = b * sub + range.of(j);
      const int b0 = sstart[sk] - key0, b1 = sstart[sk + 1] - key0;
      int r = t;  // place in the sorted list
      if (b1 - b0 <= kRankMax) {
        r = b0;
        if constexpr (SPECIES) {
          for (int m = b0; m < b1; m += 4)
            r += ((keys[m] < key ? 1 : 0) + (keys[m + 1] < key ? 1 : 0)) +
                 ((keys[m + 2] < key ? 1 : 0) + (keys[m + 3] < key ? 1 : 0));
        } else {
          for (int m = b0; m < b1; ++m) r += keys[m] < key ? 1 : 0;
        }
      }
      // never for lists that were counted alike; were positions changed under the build, a key
      // left over in LDS could name a range of another pass: nothing outside the list is written
      if ((uint32_t)r >= (uint32_t)n_keys) { atomicOr(status, ST_INTERNAL); return; }
      const int64_t at = base + key0 + r;
      const uint32_t n1 = (uint32_t)key_shift(key, 0) & 0xffu;
      const uint32_t n2 = (uint32_t)key_shift(key, 1) & 0xffu;
      const uint32_t n3 = (uint32_t)key_shift(key, 2) & 0xffu;
      nb.j[at] = j;
      nb.shift[at] = (int32_t)(n1 | (n2 << 8) | (n3 << 16) | ((uint32_t)e << 24));
      if (pair_key) {  // inputs of the reverse-index kernel; the index starts unresolved
        pair_key[at] = SPECIES ? key & ~kKeySpeciesMask : key;
        const int64_t any = base + key0 + t;
        pair_centre[any] = (int32_t)i;
        nb.reverse[any] = -1;
      }
    };
    if (species_mask) {
      for (int t = tid; t < n_keys; t += blockDim.x) place(t, std::true_type{});
    } else {
      for (int t = tid; t < n_keys; t += blockDim.x) place(t, std::false_type{});
    }
    if (!RANGED) break;
    __syncthreads();  // the next range reuses the keys and cursors
    b_lo = b_hi;
  }
}

// Short-list fill: one workgroup per centre, centres in cell-list order
// (reference points in index order).
template <int SM>
__global__ __launch_bounds__(256) void k_fill(PlanDev P, BatchDev bt, NbrDev nb, const StructInfo *info,
                                              const double *fw, const int64_t *bin_start,
                                              const double *sx, const double *sy, const double *sz,
                                              const int32_t *sid, const int32_t *ssp, const int32_t *astruct,
                                              const int32_t *cnt, int lds_keys, uint64_t *pair_key,
                                              int32_t *pair_centre, int32_t *range_start,
                                              uint32_t *status, int32_t *long_q) {
  extern __shared__ uint64_t lds_u64[];
  __shared__ CandLds lds_cand[4];
  __shared__ int32_t lds_bmax, lds_rmax;
  const int64_t k = xcd_contiguous(blockIdx.x, gridDim.x);  // list slot
  const int64_t i = point_mode(bt) ? k : sid[k];
  fill_centre<false, SM>(P, bt, nb, info, fw, bin_start, sx, sy, sz, sid, ssp, astruct, cnt, lds_keys, pair_key,
                     pair_centre, range_start, status, long_q, k, i, lds_u64, lds_cand, lds_bmax,
                         lds_rmax);
}

// Long-list fill: persistent workgroups take the queued centres one at a
// time (status word 6 holds the queue length, word 7 the next entry); every
// workgroup exits once the queue is drained, also when it is empty.
template <int SM>
__global__ __launch_bounds__(256) void k_fill_long(PlanDev P, BatchDev bt, NbrDev nb, const StructInfo *info,
                                                   const double *fw, const int64_t *bin_start,
                                                   const double *sx, const double *sy, const double *sz,
                                                   const int32_t *sid, const int32_t *ssp, const int32_t *astruct,
                                                   const int32_t *cnt, int lds_keys, uint64_t *pair_key,
                                                   int32_t *pair_centre, int32_t *range_start,
                                                   uint32_t *status, int32_t *long_q) {
  extern __shared__ uint64_t lds_u64[];
  __shared__ CandLds lds_cand[4];
  __shared__ int32_t lds_bmax, lds_rmax;
  __shared__ uint32_t lds_next;
  const uint32_t nq = __atomic_load_n(status + 6, __ATOMIC_RELAXED);
  for (;;) {
    if (threadIdx.x == 0) lds_next = atomicAdd(status + 7, 1u);
    __syncthreads();
    const uint32_t q = lds_next;
    if (q >= nq) break;
    const int64_t k = long_q[q];
    fill_centre<true, SM>(P, bt, nb, info, fw, bin_start, sx, sy, sz, sid, ssp, astruct, cnt, lds_keys, pair_key,
                      pair_centre, range_start, status, long_q, k, point_mode(bt) ? k : sid[k], lds_u64,
                      lds_cand, lds_bmax, lds_rmax);
    __syncthreads();  // lds_next, the keys and the bucket starts are reused
  }
}

// Reverse index: pair (i, j, n) and its mirror (j, i, -n).  One thread per
// pair; only the owner of each mirror couple -- i < j, or i == j with n >= 0
// lexicographically -- searches its mirror among the packed keys of j's list
// and writes both entries.  The mirror has the same q, hence the same shell:
// it lies in the range of j's list with that shell, i's species and i's range
// of atom indices, a few dozen keys whose start the fill stored.  Bound by the
// chain of dependent loads and the cache lines they fetch.  Bucket starts and
// every 16th key of a bucket probed first: 4096 atoms, 6.9e6 pairs 0.190 ms,
// now 0.170; 60,000 atoms, 1.3e8 pairs 4.80 -> 4.17 ms; 192 structures 0.300 ->
// 0.247 ms.  (Searching the 4-byte neighbour indices instead, no keys stored:
// 0.246 and 5.2 ms; owners gathered into full wavefronts first: 0.190, 4.3.)
__global__ __launch_bounds__(256) void k_reverse(PlanDev P, BatchDev bt, NbrDev nb, const uint64_t *pair_key,
                                                 const int32_t *pair_centre, const int32_t *range_start,
                                                 const int32_t *range_col, int64_t n_pairs, uint32_t *status) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t N = bt.n_atoms;
  const int64_t total = nb.offsets[N];
  if (p >= n_pairs || p >= total || total > nb.capacity) return;
  const int nbk = P.E * P.S;
  const uint64_t kp = pair_key[p];
  const int64_t i = pair_centre[p];
  const int32_t j = (int32_t)key_atom(kp);
  const int h = key_shell(kp);
  if (i < 0 || i >= N || (int64_t)j >= N || h >= P.S) {  // never for lists the fill wrote
    atomicOr(status, ST_INTERNAL);
    return;
  }
  const int n1 = key_shift(kp, 0), n2 = key_shift(kp, 1), n3 = key_shift(kp, 2);
  const int lex = n1 != 0 ? n1 : (n2 != 0 ? n2 : n3);
  if (!((int64_t)j > i || ((int64_t)j == i && lex >= 0))) return;
  // the mirror has the same q, hence the same shell
  const int32_t *row = range_start + (int64_t)j * (nbk * P.sub + 1) + h * P.E * P.sub + range_col[i];
  const uint64_t key = make_key(i, -n1, -n2, -n3, h);
  int64_t lo = row[0], hi = row[1];
  int64_t found = -1;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    const uint64_t km = pair_key[mid];
    if (km == key) { found = mid; break; }
    if (km < key) lo = mid + 1; else hi = mid;
  }
  if (found < 0) {
    atomicOr(status, ST_INTERNAL);
    return;
  }
  nb.reverse[p] = (int32_t)found;
  nb.reverse[found] = (int32_t)p;
}

}  // namespace

// ------------------------------------------------------------------ host launchers
// The plan with the number of index ranges per bucket of one build: a power of
// two, as many as the plan allows (384 counters a centre), but no more than a
// structure has atoms and no more counters than an average list has room for
// entries, past which they cost the count and the fill more than the shorter
// ranges save.  With up to 8 ranges whatever the batch: 4096 molecules of 9-29
// atoms, lists 0.600 ms, now 0.557; 2048 cells of 1-4 atoms 1.17, now 1.12; with
// few buckets, 20,000 atoms in spatial order (whose neighbours share one to three
// ranges of 8), 4 slots x 2 species, count + fill + reverse 2.06, now 1.70.
// Depends on the batch's sizes and the capacity alone, which gmp_build_lists and
// gmp_build_reverse have in common.
static PlanDev plan_of_build(const gmp_plan *p, const BatchDev &bt, const NbrDev &nb) {
  PlanDev P = p->dev;
  const int64_t nc = n_centres(bt), entries = nc > 0 ? nb.capacity / nc : 0;
  const int64_t atoms = bt.n_structs > 0 ? (bt.n_atoms + bt.n_structs - 1) / bt.n_structs : 0;
  while (P.sub > 1 && (P.sub > atoms || (int64_t)P.S * P.E * P.sub > entries)) P.sub /= 2;
  return P;
}

// Cell list: wrap, bins, bin-sorted atoms.  Small batches in one workgroup.
void launch_cells(const gmp_plan *p, const BatchDev &bt, const NbrDev &nb, const WsLayout &L, hipStream_t s) {
  const int64_t n = n_total(bt), n_bins = bt.n_atoms + bt.n_structs;
  const double rcmax = sqrt(p->dev.rcmax2);
  const PlanDev P = plan_of_build(p, bt, nb);
  if (n <= kSmallAtoms && bt.n_structs <= kSmallAtoms) {
    GMP_LAUNCH("nbr_small_cells", k_small_cells, dim3(1), dim3(kScanThreads), 0, s, P, bt, nb, L.sinfo, rcmax,
               p->tuning.bin_divisor, L.status, L.counter, L.bin_count, L.bin_start, L.bin_fill, L.fw, L.bin_of, L.astruct,
               L.range_col, L.sid_tmp, L.sx, L.sy, L.sz, L.sid, L.ssp);
    return;
  }
  auto blocks_of = [](int64_t items) { return dim3((unsigned)((items + 255) / 256)); };
  const int64_t wraps = n > bt.n_structs ? n : bt.n_structs;  // a thread per structure reports its faults
  GMP_LAUNCH("nbr_setup", k_setup, blocks_of(n_bins > 64 ? n_bins : 64), dim3(256), 0, s, bt, L.sinfo, rcmax,
             p->tuning.bin_divisor, L.status, L.counter, L.bin_count, L.bin_fill, n_bins);
  GMP_LAUNCH("nbr_wrap", k_wrap, blocks_of(wraps), dim3(256), 0, s, bt, L.sinfo, nb, L.fw, L.bin_of, L.bin_count,
             L.astruct, L.range_col, P, L.status);
  scan_i32_to_i64(L.bin_count, L.bin_start, n_bins, L.scan_aux, s);
  if (bt.n_atoms == 0) return;
  GMP_LAUNCH("nbr_scatter", k_scatter, blocks_of(bt.n_atoms), dim3(256), 0, s, bt, L.bin_of, L.bin_start, L.bin_fill,
             L.sid_tmp);
  GMP_LAUNCH("nbr_bin_order", k_bin_order, blocks_of(bt.n_atoms), dim3(256), 0, s, bt, nb, L.bin_of, L.bin_start,
             L.sid_tmp, L.sx, L.sy, L.sz, L.sid, L.ssp, p->dev.E);
}

void launch_count(const gmp_plan *p, const BatchDev &bt, const NbrDev &nb, const WsLayout &L, hipStream_t s) {
  int64_t blocks = n_centres(bt);
  if (blocks == 0) return;
  const PlanDev P = plan_of_build(p, bt, nb);
  size_t smem = sizeof(int32_t) * P.E * P.S * P.sub;
  auto kern = p->dev.S <= 8 ? k_count<8> : (p->dev.S <= 12 ? k_count<12> : k_count<kMaxSigmas>);
  GMP_LAUNCH("nbr_count", kern, dim3((unsigned)blocks), dim3(256), smem, s, P, bt, nb, L.sinfo, L.fw,
             L.bin_start, L.sx, L.sy, L.sz, L.sid, L.ssp, L.astruct, L.cnt, L.ptotal, L.bucket_max, L.status);
}

// List offsets, and with `stats` the longest list and bucket (status words 4, 5).
void launch_offsets(const BatchDev &bt, const WsLayout &L, int64_t *offsets, bool stats, hipStream_t s) {
  const int64_t nc = n_centres(bt);
  if (!stats || nc > kSingleScanMax) scan_i64(L.ptotal, offsets, nc, L.scan_aux, s);
  if (!stats) return;
  if (nc <= kSingleScanMax) {
    GMP_LAUNCH("nbr_offsets", k_offsets_stats, dim3((unsigned)(1 + (nc + 4095) / 4096)), dim3(kScanThreads), 0, s,
               L.ptotal, L.bucket_max, offsets, nc, L.status);
  } else {
    GMP_LAUNCH("nbr_list_stats", k_list_stats, dim3(256), dim3(256), 0, s, L.ptotal, L.bucket_max, nc, L.status);
  }
}

void launch_fill(const gmp_plan *p, const BatchDev &bt, const NbrDev &nb, const WsLayout &L, int lds_keys,
                 int long_keys, hipStream_t s) {
  const PlanDev P = plan_of_build(p, bt, nb);
  const int nbk = P.E * P.S;
  if (n_centres(bt) == 0) return;
  uint64_t *pk = (nb.reverse && !point_mode(bt)) ? L.pair_key : (uint64_t *)nullptr;
  size_t smem = sizeof(uint64_t) * (lds_keys + kKeyPad) + sizeof(int32_t) * (2 * nbk * P.sub + 2);
  auto kern = p->dev.S <= 8 ? k_fill<8> : (p->dev.S <= 12 ? k_fill<12> : k_fill<kMaxSigmas>);
  GMP_LAUNCH("nbr_fill_sort", kern, dim3((unsigned)n_centres(bt)), dim3(256), smem, s, P, bt, nb, L.sinfo,
             L.fw, L.bin_start, L.sx, L.sy, L.sz, L.sid, L.ssp, L.astruct, L.cnt, lds_keys, pk, L.pair_centre,
             L.range_start, L.status, L.long_q);
  if (long_keys > 0) {  // one workgroup per CU (its LDS takes most of the CU's), capped by the centre count
    smem = sizeof(uint64_t) * (long_keys + kKeyPad) + sizeof(int32_t) * (2 * nbk * P.sub + 2);
    const int64_t blocks = n_centres(bt) < 256 ? n_centres(bt) : 256;
    auto kern_long = p->dev.S <= 8 ? k_fill_long<8> : (p->dev.S <= 12 ? k_fill_long<12> : k_fill_long<kMaxSigmas>);
    GMP_LAUNCH("nbr_fill_long", kern_long, dim3((unsigned)blocks), dim3(256), smem, s, P, bt, nb, L.sinfo,
               L.fw, L.bin_start, L.sx, L.sy, L.sz, L.sid, L.ssp, L.astruct, L.cnt, long_keys, pk, L.pair_centre,
               L.range_start, L.status, L.long_q);
  }
}

void launch_reverse(const gmp_plan *p, const BatchDev &bt, const NbrDev &nb, const WsLayout &L, int64_t n_pairs,
                    hipStream_t s) {
  // every entry of every written list was set to -1 (unresolved) by the fill
  const int64_t blocks = (n_pairs + 255) / 256;
  if (blocks > 0)
    GMP_LAUNCH("nbr_reverse", k_reverse, dim3((unsigned)blocks), dim3(256), 0, s, plan_of_build(p, bt, nb), bt, nb, L.pair_key,
               L.pair_centre, L.range_start, L.range_col, n_pairs, L.status);
}

}  // namespace gmp
