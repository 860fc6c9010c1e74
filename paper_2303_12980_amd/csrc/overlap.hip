// Overlap kernel (multipole moments) and norm kernel.
//
// Closed form of one pair's contribution (derived from the Gaussian product
// theorem and the mean-value property of harmonic polynomials; the paper
// defines the probe as an MCSH angular probe times a Gaussian radial probe
// and the density as per-element Gaussian primitives):
//   mu_{i,l,s,abc} += c_{l,s,e_j}(q) P_abc(d),
//   c_{l,s,e}(q) = sum_k A_{l,s,e,k} exp(-gamma_{s,e,k} q).
// P_abc is a harmonic polynomial of degree l, so the kernel accumulates the
// moments  M_{i,s,k} = sum_j c_{deg k,s,e_j}(q_j) Y_k(d_j)  of a basis of 2l+1
// solid harmonics per degree (or, below, of every monomial of each degree),
// and the norm kernel maps moments to components with the plan's exact integer
// matrices (FP64).  Each pair term is scaled by the neighbour's occupancy
// (disordered structures), which rides in the fourth component of its packed
// wrapped position.
//
// Work decomposition: persistent wavefronts pull work items (a chunk of one
// centre's list) from a global counter; lanes take consecutive pairs.  The
// list is ordered by cutoff shell first, so the pairs a slot uses form a
// prefix.  Lanes read the coefficient row of their own neighbour's species
// from the LDS copy of the plan table.  The local density of order -1 is one
// more cutoff slot, of whose moments only the degree-0 one
// rho = sum_j sum_k B exp(-beta q) is read back.
//
// Arithmetic (template MODE):
//   ACC_F64:   everything FP64 (exp in FP64), harmonics.
//   ACC_WIDE:  FP32 exponentials and radial sums; FP64 harmonics and
//              accumulation (one FP64 fma per term, which issues at the
//              non-packed FP32 rate on gfx950).  FP32-wide plans, and
//              FP32-compensated ones where only the FP32 features are asked for.
//   ACC_TERMS: FP32 pair terms throughout (displacement, monomials,
//              exponentials, radial sums, products); per-lane accumulation as
//              FP32 (hi, lo) error-free sums.  FP32-compensated plans where
//              the FP64 components are asked for.
// Cross-lane reduction, moment -> component map and norm are FP64 throughout.
#include <map>
#include <mutex>
#include <type_traits>

#include "gmp_internal.h"

namespace gmp {
namespace {

constexpr MonoTable kMT = make_mono_table();

enum AccMode { ACC_F64 = 0, ACC_WIDE = 1, ACC_TERMS = 2 };
// accumulated moments per slot
__host__ __device__ constexpr int n_moments(int mode, int lmax) { return mode == ACC_TERMS ? nmono(lmax) : nharm(lmax); }

__device__ inline float exp_scaled(float a, float q) { return __builtin_amdgcn_exp2f(a * q); }
__device__ inline double exp_scaled(double a, double q) { return exp(a * q); }

// Per list slot: the number of chunks of its list (fixed-size pieces of kc
// pairs, kc = 0: whole list, so the decomposition of a centre depends on its
// own list only and a batched launch sums in the same order as a launch over
// one structure), its structure, and its wrapped position as an AoS double4
// (one 32-byte gather per neighbour).  The first thread also clears the
// work-item counter.  The word after the counter tells the overlap kernel of a
// position, occupancy or lattice that has diverged since the lists were built.  The neighbour
// build clears it, and the norm kernel behind the overlap; a stale one costs time
// only.
// Indices g < n_total get their structure and packed position; centres
// c < n_centres their chunk count.
__device__ inline int64_t list_chunks(const NbrDev &nb, int kc, int64_t k) {
  const int64_t end = nb.offsets[k + 1], cnt = end - nb.offsets[k];
  // a list that ends past the capacity was not written (overflowed no-sync
  // build, reported in the status word): no work items, zero moments
  return end > nb.capacity ? 0 : (kc > 0 && cnt > kc ? (cnt + kc - 1) / kc : 1);
}
// Positions, occupancies and lattice vectors (times up to 126 cells) below these
// keep every monomial of degree 3 times the occupancy far from overflow in FP32.
constexpr double kFar = 1e10, kFarOcc = 1e6, kFarCell = 1e7;
__device__ inline bool diverged(const BatchDev &bt, const double4 &r, int st) {
  bool ok = __builtin_fabs(r.x) < kFar && __builtin_fabs(r.y) < kFar && __builtin_fabs(r.z) < kFar &&
            __builtin_fabs(r.w) < kFarOcc;
  if (bt.pbc[st] & 7) {
    const double *a = bt.cell + 9 * (int64_t)st;
#pragma unroll
    for (int k = 0; k < 9; ++k) ok = ok && __builtin_fabs(a[k]) < kFarCell;
  }
  return !ok;
}
__device__ inline void prep_index(const BatchDev &bt, const NbrDev &nb, double4 *rw4, int32_t *astruct,
                                  unsigned long long *counter, int64_t i) {
  if (i >= n_total(bt)) return;
  const int st = struct_of_index(bt, i);
  astruct[i] = st;
  const double4 r = wrapped_position(bt, nb, i, st);
  rw4[i] = r;
  if (diverged(bt, r, st)) atomicOr(counter + 1, 1ull);
}
__global__ void k_overlap_prep(BatchDev bt, NbrDev nb, int kc, int64_t *nch, double4 *rw4, int32_t *astruct,
                               unsigned long long *counter) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *counter = 0ull;
  if (i < n_centres(bt)) nch[i] = list_chunks(nb, kc, i);
  prep_index(bt, nb, rw4, astruct, counter, i);
}
// The same with the scan of the chunk counts, which needs nothing of the rest,
// in the first workgroup: one launch where one workgroup can scan them.
__global__ __launch_bounds__(kScanThreads) void k_overlap_prep_scan(BatchDev bt, NbrDev nb, int kc,
                                                                    int64_t *chunk_off, double4 *rw4,
                                                                    int32_t *astruct, unsigned long long *counter) {
  __shared__ int64_t words[kScanWords];
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) *counter = 0ull;
    block_scan([&](int64_t k) { return list_chunks(nb, kc, k); }, chunk_off, n_centres(bt), words);
  } else {
    prep_index(bt, nb, rw4, astruct, counter, (int64_t)(blockIdx.x - 1) * kScanThreads + threadIdx.x);
  }
}

// List slot of chunk q.  Chunk q belongs to slot q itself where every list
// before it is one chunk (the common case: one round trip in place of the
// bisection's dozen dependent ones); otherwise to an earlier slot, or a later
// one where lists before it were not written.
__device__ inline int64_t centre_of_chunk(const int64_t *chunk_off, int64_t N, int64_t q) {
  if (q < N) {
    const int64_t a = uniform64(chunk_off[q]), b = uniform64(chunk_off[q + 1]);
    if (a == q && b == q + 1) return q;
  }
  int64_t lo = 0, hi = N;  // chunk_off[lo] <= q < chunk_off[lo+1]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (chunk_off[mid] <= q) lo = mid; else hi = mid;
  }
  return lo;
}

// Per-lane accumulators of one slot's moments.
template <int MODE, int NM> struct Acc {
  double v[NM];
  __device__ void zero() {
#pragma unroll
    for (int m = 0; m < NM; ++m) v[m] = 0.0;
  }
  __device__ double value(int m) const { return v[m]; }
};
// FP32 (hi, lo) pairs updated with an error-free sum: Dekker's Fast2Sum
// on the two addends ordered by magnitude (exact when the first is the
// larger).  It yields the same exact rounding error, hence the same (hi,
// lo), as Knuth's branch-free two-sum, in as many operations (a compare on
// magnitudes, two selects, three additions), but reads the old sum only
// before the new one is formed, so the new sum takes its register without a
// copy back.
template <int NM> struct Acc<ACC_TERMS, NM> {
  float hi[NM], lo[NM];
  __device__ void zero() {
#pragma unroll
    for (int m = 0; m < NM; ++m) { hi[m] = 0.f; lo[m] = 0.f; }
  }
  __device__ void add(int m, float p) {
    const bool ge = __builtin_fabsf(hi[m]) >= __builtin_fabsf(p);
    const float big = ge ? hi[m] : p, small = ge ? p : hi[m];
    const float s = big + small;
    lo[m] += small - (s - big);
    hi[m] = s;
  }
  __device__ double value(int m) const { return (double)hi[m] + (double)lo[m]; }
};

// Slots of one pass: several cutoff slots, consecutive in cutoff order, share
// a walk over the list, and with it the displacement, the harmonics (or
// monomials) and the loads of every pair.  Their accumulators bound how many
// fit.  Harmonics, l = 4: two slots' 2 x 25 doubles leave two wavefronts per
// SIMD (held to three they spill: 0.25 instead of 0.23 ms on 4096 atoms).
// FP32 terms: two slots at l = 3 (1200 atoms, 1728 points: 0.187 -> 0.134 ms);
// at l = 4 one slot and three wavefronts (60,000 atoms 6.82 ms, two slots
// 7.16 ms), the 35 error-free sums being two thirds of the instructions.
__host__ __device__ constexpr int pass_slots(int mode, int lmax) {
  return lmax >= 4 ? (mode == ACC_TERMS ? 1 : 2) : (lmax == 3 ? (mode == ACC_TERMS ? 2 : 3) : 4);
}

// f(0), .., f(NS - 1) with the index a compile-time constant (register arrays
// indexed by it stay in registers).
template <int NS, typename F>
__device__ inline void for_slots(F &&f) {
  f(std::integral_constant<int, 0>{});
  if constexpr (NS > 1) f(std::integral_constant<int, 1>{});
  if constexpr (NS > 2) f(std::integral_constant<int, 2>{});
  if constexpr (NS > 3) f(std::integral_constant<int, 3>{});
}

// Sum over the two halves of the wavefront of a in lanes 0-31 and of b in
// lanes 32-63 (one lane swap per 32-bit word).
__device__ inline double fold32(double a, double b) {
  const uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
  return __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) + __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
}
// Sum over the two 16-lane rows of each half: of a in the even row, of b in the odd one.
__device__ inline double fold16(double a, double b) {
  const uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
  return __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) + __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
}

// Fixed-order cross-lane sum of NV per-lane doubles, written to dst[0..NV):
// two folds leave four columns per register (16 partials each), which go
// through LDS so that one lane sums one column.  A column's 16 partials are
// 144 bytes apart from the next column's: lanes read from different banks.
constexpr int kRedStride = 18;
__host__ __device__ constexpr int red_doubles(int nv) { return ((nv + 3) / 4) * 4 * kRedStride; }
template <int NV>
__device__ inline void wave_reduce_store(const double (&v)[NV], double *dst, double *lds) {
  constexpr int N1 = (NV + 1) / 2, N2 = (N1 + 1) / 2;
  const int lane = lane_id();
  double h[N1];
#pragma unroll
  for (int r = 0; r < N1; ++r) h[r] = fold32(v[2 * r], 2 * r + 1 < NV ? v[2 * r + 1] : 0.0);
#pragma unroll
  for (int r = 0; r < N2; ++r)
    lds[(4 * r + (lane >> 4)) * kRedStride + (lane & 15)] = fold16(h[2 * r], 2 * r + 1 < N1 ? h[2 * r + 1] : 0.0);
  wave_lds_sync();
  if (lane < 4 * N2) {  // register r, row w holds column 4r + 2 (w & 1) + (w >> 1)
    const double *x = lds + lane * kRedStride;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 16; ++t) s[t & 3] += x[t];
    const int col = (lane & ~3) + 2 * (lane & 1) + ((lane >> 1) & 1);
    if (col < NV) dst[col] = (s[0] + s[1]) + (s[2] + s[3]);
  }
  wave_lds_sync();
}

// Radial factors c_0..c_L of slot s and element e at squared distance q from
// the plan's table: cubic in t = r/h - k on interval k of r = sqrt(q).
template <int L>
__device__ inline void radial_from_table(const PlanDev &P, int s, int e, float q, float (&cl)[L + 1]) {
  const float x = __builtin_sqrtf(q) * P.tab_inv_h[s];
  int k = (int)x;
  k = k < P.tab_n - 1 ? k : P.tab_n - 1;
  const float t = x - (float)k;
  const float4 *c = P.rtab + (((size_t)s * P.E + e) * P.tab_n + k) * 5;
#pragma unroll
  for (int l = 0; l <= L; ++l) {
    const float4 a = c[l];
    cl[l] = fmaf(fmaf(fmaf(a.w, t, a.z), t, a.y), t, a.x);
  }
}

// Radial sums c_l += sum_k A_{l,k} exp(-gamma_k q) of NU slots together (NU
// independent chains per lane).  Table rows past an element's own primitive
// count are zero (they add exact zeros), so every lane runs the plan's
// largest count with wavefront-uniform control flow, and the rows k+1 are read
// before the rows k are used (the empty asm statement keeps the compiler from
// sinking the reads).
template <int LMAX, int KB, int NU>
__device__ inline void radial_sums(const float *const (&row)[NU], float q, int kmax,
                                   float (&cl)[NU][LMAX + 1]) {
  float4 ra[NU];
  float2 rb[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) { ra[u] = *(const float4 *)row[u]; rb[u] = *(const float2 *)(row[u] + 4); }
  auto row_step = [&](int k) {
    float4 na[NU];
    float2 nb[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (k + 1 < KB) {
        na[u] = *(const float4 *)(row[u] + (k + 1) * kCoefStride);
        nb[u] = *(const float2 *)(row[u] + (k + 1) * kCoefStride + 4);
      }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const float ek = exp_scaled(ra[u].x, q);
      const float av[5] = {ra[u].y, ra[u].z, ra[u].w, rb[u].x, rb[u].y};
#pragma unroll
      for (int l = 0; l <= LMAX; ++l) cl[u][l] = fma_(av[l], ek, cl[u][l]);
      if (k + 1 < KB) { ra[u] = na[u]; rb[u] = nb[u]; }
    }
  };
  if constexpr (KB <= 8) {  // full unroll with an early exit (trip count bound <= 8)
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (k >= kmax) break;
      row_step(k);
    }
  } else {  // 16-row tables: a wavefront-uniform guard keeps the trip count constant
#pragma unroll
    for (int k = 0; k < KB; ++k)
      if (k < kmax) row_step(k);
  }
}
template <int LMAX, int KB, int NU>
__device__ inline void radial_sums(const double *const (&row)[NU], double q, int kmax, double (&cl)[NU][LMAX + 1]) {
  for (int k = 0; k < kmax; ++k) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const double *o = row[u] + k * kCoefStride;
      const double ek = exp_scaled(o[0], q);
#pragma unroll
      for (int l = 0; l <= LMAX; ++l) cl[u][l] = fma_(o[1 + l], ek, cl[u][l]);
    }
  }
}

// Overlap kernel, persistent: every wavefront pulls work items (a chunk of
// one centre's list, for one group of passes) from a global counter until
// none are left.  A pass takes NS cutoff slots, consecutive in cutoff order,
// over the longest of their prefixes of the chunk; a slot's part of a step is
// skipped past its own prefix, for the lanes past it inside the step that
// straddles it.  The loads of pair data (j, shift) run two steps ahead and
// the gathers of the neighbours' wrapped positions one step ahead,
// continuously across the passes.  Moments of orders that were not requested
// are accumulated and not read back.
//
// Bound by VALU issue: 267 instructions per 64 pairs and two slots with
// harmonics (446 per slot with the error-free FP32 sums of 35 monomials, whose
// time is that of one pass per slot).  Harmonics against one monomial pass per
// slot: 512 structures, 3.3e7 pairs, 8 slots, FP32 features alone 1.79 -> 0.95
// ms; FP32-wide, 192 structures, 0.53 -> 0.39 ms; FP64, 1500 atoms, 0.26 ->
// 0.17 ms.  Slots of small batches as items of their own: 97 atoms 0.094 ->
// 0.036 ms.
//
// The coefficient table [slot][element][KB][8] (exponent scale, A_0..A_4, ..)
// is copied into LDS once per workgroup when it fits, with a 16-byte gap
// after every (slot, element) block: lanes of different species read their
// rows from different banks.
template <int LMAX, int KB, int MODE, bool LDS, bool SCREEN, bool OCC, bool TAB, bool STEP_K, int NS, typename TR>
__device__ __forceinline__ void overlap_items(const PlanDev &P, const BatchDev &bt, const NbrDev &nb,
                                              const double4 *rw4, const int32_t *astruct, double *partial,
                                              const int64_t *chunk_off, int kc, int ng, int nbatch,
                                              unsigned long long *counter, const TR *__restrict__ tabg,
                                              const TR *tabl, const int *lds_k, double *red) {
  constexpr int NH = n_moments(MODE, LMAX);
  constexpr int BLK = KB * kCoefStride, BLKL = BLK + 16 / (int)sizeof(TR);
  const int S = P.S, E = P.E;
  const int lane = lane_id();
  const int64_t N = n_centres(bt), cb = centre_base(bt);
  const int64_t n_items = chunk_off[N] * ng;
  const int NP = (S + NS - 1) / NS;
  auto table_row = [&](int s, int e) -> const TR * {
    return LDS ? tabl + s * E * BLKL + __umul24(e, BLKL) : tabg + (size_t)(s * E + e) * BLK;
  };
  for (int64_t item = 0, left = 0;; ++item, --left) {
    if (left == 0) {
      item = next_item(counter) * nbatch;
      left = nbatch;
    }
    if (item >= n_items) break;
    // item = (chunk qc, group g of its passes: [t0, t1)); every item writes
    // the moments of its own slots, so the rows are the same for any ng
    const int64_t qc = item / ng;
    const int g = (int)(item - qc * ng);
    const int t0 = g * NP / ng, t1 = (g + 1) * NP / ng;
    const int64_t k = centre_of_chunk(chunk_off, N, qc);  // list slot
    const int64_t i = nb.order[k];                         // its centre
    const int c = (int)(qc - chunk_off[k]);
    const int st = astruct[cb + i];
    const Cell9 cell = load_cell(bt.cell + 9 * (int64_t)st);
    const int pbc = bt.pbc[st] & 7;
    const double4 ri4 = rw4[cb + i];
    const double rix = ri4.x, riy = ri4.y, riz = ri4.z;
    const int64_t base = uniform64(nb.offsets[k]);
    const int cnt = (int)(uniform64(nb.offsets[k + 1]) - base);
    const int clo = kc > 0 ? c * kc : 0;
    const int chi = kc > 0 ? (clo + kc < cnt ? clo + kc : cnt) : cnt;
    // prefix ends inside the chunk and slots by cutoff order, one per lane
    int end_lane = clo, so_lane = 0;
    if (lane < S) {
      so_lane = P.sig_order[lane];
      const int en = nb.sigma_end[k * S + so_lane];
      end_lane = en < clo ? clo : (en < chi ? en : chi);
    }
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto slot_end = [&](int t) { return __builtin_amdgcn_readlane(end_lane, t); };
    auto pass_end = [&](int t) { return slot_end(t * NS + NS - 1 < S ? t * NS + NS - 1 : S - 1); };
    double *dst_item = partial + (size_t)qc * S * NH;
    // passes whose prefixes miss this chunk contribute zero moments (pass
    // ends are non-decreasing: they come first)
    int tb = t0, pb = clo;
    while (tb < t1 && pass_end(tb) <= clo) ++tb;
    for (int t = t0 * NS; t < tb * NS && t < S; ++t)
      for (int m = lane; m < NH; m += kWave) dst_item[(size_t)__builtin_amdgcn_readlane(so_lane, t) * NH + m] = 0.0;
    if (tb >= t1) continue;
    int tc = tb, pc = pb;
    auto advance = [&](int &t, int &p) {
      p += kWave;
      if (p >= pass_end(t)) {
        ++t;
        p = clo;
      }
      t = uni(t);
      p = uni(p);
    };
    advance(tc, pc);
    const int32_t ii = (int32_t)(cb + i);  // idle lanes read the centre's own packed position
    // stage b: positions gathered; stage c: (j, shift) loaded
    int32_t wb = 0, jc = ii, wc = 0;
    double4 rb;
    {
      int32_t jb = ii;
      const int p = pb + lane;
      if (p < pass_end(tb)) { jb = nb.j[base + p]; wb = nb.shift[base + p]; }
      if (tc < t1 && pc + lane < pass_end(tc)) { jc = nb.j[base + pc + lane]; wc = nb.shift[base + pc + lane]; }
      rb = rw4[jb];
    }
    Acc<MODE, NH> acc[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) acc[u].zero();
    while (tb < t1) {
      const int ta = tb, pa = pb;
      // the current step's pair, from what the pipeline holds
      const int p = pa + lane;
      double shx = 0.0, shy = 0.0, shz = 0.0;
      if (pbc) image_shift(cell, shift_n(wb, 0), shift_n(wb, 1), shift_n(wb, 2), shx, shy, shz);
      double dx = (rb.x - rix) + shx;
      double dy = (rb.y - riy) + shy;
      double dz = (rb.z - riz) + shz;
      double occj = rb.w;
      int e = shift_species(wb);
      // advance the pipeline.  The asm statements pin these values here, ahead
      // of the new loads, which then go into the registers they came from:
      // loaded into others, they would be waited for and copied at the end of
      // this same step.
      asm volatile("" : "+v"(dx), "+v"(dy), "+v"(dz), "+v"(e));
      if constexpr (OCC || MODE == ACC_TERMS) asm volatile("" : "+v"(occj));
      tb = tc; pb = pc; wb = wc;
      int32_t jn = jc;
      asm volatile("" : "+v"(wb), "+v"(jn));
      rb = rw4[jn];
      jc = ii; wc = 0;
      if (tc < t1) {
        advance(tc, pc);
        if (tc < t1 && pc + lane < pass_end(tc)) { jc = nb.j[base + pc + lane]; wc = nb.shift[base + pc + lane]; }
      }
      const double q = (dx * dx + dy * dy) + dz * dz;
      const TR qv = (TR)q;
      auto step = [&] {
        // radial factors of the pass's slots; zero past a slot's own prefix
        TR cl[NS][LMAX + 1];
        const int tl = ta * NS;
        const int K = STEP_K ? step_primitives(P.kmax, lds_k, e, p < pass_end(ta)) : P.kmax;
        if (NS > 1 && !SCREEN && !TAB && tl + NS <= S && pa < slot_end(tl)) {  // every slot takes pairs of this step
          const TR *row[NS];
#pragma unroll
          for (int u = 0; u < NS; ++u) {
            row[u] = table_row(__builtin_amdgcn_readlane(so_lane, tl + u), e);
#pragma unroll
            for (int l = 0; l <= LMAX; ++l) cl[u][l] = (TR)0;
          }
          radial_sums<LMAX, KB, NS>(row, qv, K, cl);
          // nothing from the lanes past a slot's prefix: a step in which any
          // prefix of the pass ends is one in which the shortest does
          if (slot_end(tl) - pa < kWave) {
#pragma unroll
            for (int u = 0; u < NS; ++u) {
              const bool in = p < slot_end(tl + u);
#pragma unroll
              for (int l = 0; l <= LMAX; ++l) cl[u][l] = in ? cl[u][l] : (TR)0;
            }
          }
        } else {
          auto slot_radial = [&](auto uc) {
            constexpr int u = decltype(uc)::value;
#pragma unroll
            for (int l = 0; l <= LMAX; ++l) cl[u][l] = (TR)0;
            const int t = tl + u;
            if (NS > 1 && (t >= S || p >= slot_end(t))) return;
            const int sgm = __builtin_amdgcn_readlane(so_lane, t);
            if constexpr (TAB) {
              radial_from_table<LMAX>(P, sgm, e, qv, cl[u]);
            } else {
              const TR *row[1] = {table_row(sgm, e)};
              if constexpr (SCREEN) {
                // the primitive's own radius; skipped by the wavefront when no lane needs it
#pragma unroll
                for (int k = 0; k < KB; ++k) {
                  if (k < K) {
                    const TR *o = row[0] + k * kCoefStride;
                    const bool use = (float)q <= (float)o[7];
                    if (__ballot(use) == 0) continue;
                    const TR ek = use ? exp_scaled(o[0], qv) : (TR)0;
#pragma unroll
                    for (int l = 0; l <= LMAX; ++l) cl[u][l] = fma_(o[1 + l], ek, cl[u][l]);
                  }
                }
              } else {
                TR c1[1][LMAX + 1];
#pragma unroll
                for (int l = 0; l <= LMAX; ++l) c1[0][l] = (TR)0;
                radial_sums<LMAX, KB, 1>(row, qv, K, c1);
#pragma unroll
                for (int l = 0; l <= LMAX; ++l) cl[u][l] = c1[0][l];
              }
            }
          };
          for_slots<NS>(slot_radial);
        }
        // harmonics (monomials), each accumulated for every slot of the pass as it is formed
        auto is_density = [&](int u) {
          return tl + u < S && __builtin_amdgcn_readlane(so_lane, tl + u < S ? tl + u : 0) == P.dens_slot;
        };
        if constexpr (MODE == ACC_TERMS) {
          float mono[NH];
          const float xv = (float)dx, yv = (float)dy, zv = (float)dz;
          mono[0] = (float)occj;  // the occupancy scales every monomial of the pair
#pragma unroll
          for (int u = 0; u < NS; ++u) acc[u].add(0, cl[u][0] * mono[0]);
          if (NS > 1 || !is_density(0)) {
#pragma unroll
            for (int m = 1; m < NH; ++m) {
              mono[m] = (kMT.var[m] == 0 ? xv : (kMT.var[m] == 1 ? yv : zv)) * mono[kMT.parent[m]];
#pragma unroll
              for (int u = 0; u < NS; ++u) acc[u].add(m, cl[u][kMT.deg[m]] * mono[m]);
            }
          }
        } else {
          if constexpr (OCC && MODE == ACC_WIDE) {  // the density is scaled in FP32, as its FP32 sum is
#pragma unroll
            for (int u = 0; u < NS; ++u) cl[u][0] *= is_density(u) ? (float)occj : 1.f;
          }
          for_harmonics<LMAX, true>(dx, dy, dz, [&](auto mc, double Y) {
            constexpr int m = decltype(mc)::value;
#pragma unroll
            for (int u = 0; u < NS; ++u) {
              double c = (double)cl[u][hdeg(m)];
              if constexpr (OCC) c *= MODE == ACC_WIDE && m == 0 && is_density(u) ? 1.0 : occj;
              acc[u].v[m] = m == 0 ? acc[u].v[m] + c : fma(c, Y, acc[u].v[m]);
            }
          });
        }
      };
      // one slot: lanes past its prefix sit out; several: they take zeros
      if (NS > 1 || p < slot_end(ta * NS)) step();
      if (tb != ta) {  // the pass is complete: cross-lane reductions, store, restart
        auto slot_store = [&](auto uc) {
          constexpr int u = decltype(uc)::value;
          const int t = ta * NS + u;
          if (t < S) {
            double v[NH];
#pragma unroll
            for (int m = 0; m < NH; ++m) v[m] = acc[u].value(m);
            wave_reduce_store<NH>(v, dst_item + (size_t)__builtin_amdgcn_readlane(so_lane, t) * NH, red);
          }
          acc[u].zero();
        };
        for_slots<NS>(slot_store);
      }
    }
  }
}

template <int LMAX, int KB, int MODE, bool LDS, bool SCREEN, bool OCC, bool TAB = false, bool STEP_K = false>
__global__ __launch_bounds__(256, pass_slots(MODE, LMAX) == 1 ? 3 : 2) void k_overlap(PlanDev P, BatchDev bt, NbrDev nb, const double4 *rw4,
                                                    const int32_t *astruct, double *partial,
                                                    const int64_t *chunk_off, int kc, int ng,
                                                    int nbatch, unsigned long long *counter, const void *tab_global) {
  using TR = typename std::conditional<MODE == ACC_F64, double, float>::type;  // radial arithmetic
  constexpr int NH = n_moments(MODE, LMAX), NS = pass_slots(MODE, LMAX);
  constexpr int BLK = KB * kCoefStride, BLKL = BLK + 16 / (int)sizeof(TR);
  extern __shared__ __align__(16) double lds_dyn[];
  __shared__ __align__(16) double lds_red[4][red_doubles(NH)];
  const int S = P.S, E = P.E;
  const TR *__restrict__ tabg = (const TR *)tab_global;
  TR *tabl = (TR *)lds_dyn;
  if (LDS) {
    const int n = S * E * BLK;
    for (int idx = threadIdx.x; idx < n; idx += blockDim.x) tabl[(idx / BLK) * BLKL + idx % BLK] = tabg[idx];
  }
  __shared__ int lds_k[STEP_K ? kMaxElements : 1];
  if (STEP_K)
    for (int e = threadIdx.x; e < E; e += blockDim.x) lds_k[e] = P.kcount[e];
  __syncthreads();
  const int *counts = lds_k;
  double *red = lds_red[threadIdx.x / kWave];
  // A lane outside a slot's prefix adds zero times its harmonics to that slot,
  // which is zero unless they overflow: where a position has diverged since the
  // lists were built, every slot walks alone, without such lanes.  (A test in
  // every step instead, of the distance or of the same word: 512 structures 0.94
  // -> 0.98 ms.)
  if (NS > 1 && __builtin_amdgcn_readfirstlane((int)counter[1]) != 0)
    overlap_items<LMAX, KB, MODE, LDS, SCREEN, OCC, TAB, STEP_K, 1, TR>(P, bt, nb, rw4, astruct, partial, chunk_off, kc,
                                                                     ng, nbatch, counter, tabg, tabl, counts, red);
  else
    overlap_items<LMAX, KB, MODE, LDS, SCREEN, OCC, TAB, STEP_K, NS, TR>(P, bt, nb, rw4, astruct, partial, chunk_off, kc,
                                                                      ng, nbatch, counter, tabg, tabl, counts, red);
}

// One wavefront per centre: sum chunk partials in order, map moments to
// components with the exact integer matrices, then the weighted norm
// F_{l,s} = sqrt(sum_abc l!/(a!b!c!) mu_abc^2).  Order -1 takes the degree-0
// moment of the density slot as its component rho and |rho| as its feature.
// Where every component and feature comes from (order, slot, position) is
// decoded once per workgroup into LDS tables, so the per-centre loops are
// table reads and dot products; the partials of a centre with one work item
// (the common case) are read directly.
template <int LMAX, bool F64OUT, bool MONO>
__global__ __launch_bounds__(256) void k_finish(PlanDev P, int64_t N, const double *partial,
                                                const int64_t *chunk_off, const int32_t *order, void *features,
                                                double *components, unsigned long long *counter) {
  extern __shared__ double lds_f[];
  if (blockIdx.x == 0 && threadIdx.x == 0) counter[1] = 0ull;
  // moment -> component maps of all orders and the multinomial weights,
  // staged in LDS once per workgroup (read with lane-varying indices)
  constexpr int NT = MONO ? kTmat : kHmat;
  __shared__ double lds_T[NT];
  __shared__ double lds_w[nmono(kMaxL)];
  constexpr int NM = MONO ? nmono(LMAX) : nharm(LMAX);  // compile-time: the index splits below are not divisions
  const int S = P.S, NC = P.ncomp_total, NF = P.nf;
  // decode tables after the four wavefronts' moment and component buffers:
  // component t: T row offset | moment offset << 10 | length << 22 (bit 31:
  // the density component, moment offset only); feature t: component offset |
  // weight offset << 12 | length << 20 (bit 31: the density feature)
  int32_t *cdec = (int32_t *)(lds_f + (size_t)4 * (S * NM + NC));
  int32_t *fdec = cdec + NC;
  for (int t = threadIdx.x; t < NT; t += blockDim.x) lds_T[t] = MONO ? P.T[t] : P.H[t];
  for (int t = threadIdx.x; t < nmono(kMaxL); t += blockDim.x) lds_w[t] = P.weight[t];
  for (int t = threadIdx.x; t < NC; t += blockDim.x) {
    int o = 0;
    while (o + 1 < P.n_orders && P.comp_off[o + 1] <= t) ++o;
    const int l = P.orders[o];
    if (l < 0) {
      cdec[t] = (int32_t)(0x80000000u | (uint32_t)((P.dens_slot * NM) << 10));
    } else {
      const int nc = ncomp(l), r = t - P.comp_off[o];
      const int sl = r / nc, cc = r - sl * nc;
      const int nm = MONO ? nc : 2 * l + 1;  // moments of degree l
      cdec[t] = ((MONO ? P.toff[l] : P.hoff[l]) + cc * nm) | ((sl * NM + (MONO ? doff(l) : l * l)) << 10) | (nm << 22);
    }
  }
  for (int t = threadIdx.x; t < NF; t += blockDim.x) {
    int o = 0;
    while (o + 1 < P.n_orders && P.feat_off[o + 1] <= t) ++o;
    const int l = P.orders[o];
    if (l < 0) {
      fdec[t] = (int32_t)(0x80000000u | (uint32_t)P.comp_off[o]);
    } else {
      const int nc = ncomp(l);
      fdec[t] = (P.comp_off[o] + (t - P.feat_off[o]) * nc) | (doff(l) << 12) | (nc << 20);
    }
  }
  __syncthreads();
  const int w = threadIdx.x / kWave, lane = lane_id();
  const int64_t i = (int64_t)blockIdx.x * (blockDim.x / kWave) + w;  // list slot
  double *mom = lds_f + (size_t)w * (S * NM + NC);
  double *mu = mom + S * NM;
  const bool live = i < N;
  const int64_t row = live ? order[i] : 0;  // the slot's centre: its row of the outputs
  if (live) {
    const int64_t q0 = chunk_off[i], q1 = chunk_off[i + 1];
    for (int t = lane; t < S * NM; t += kWave) {
      double a = 0.0;
      if (q1 - q0 == 1) {
        a = partial[(size_t)q0 * S * NM + t];
      } else {
        for (int64_t q = q0; q < q1; ++q) a += partial[(size_t)q * S * NM + t];
      }
      mom[t] = a;
    }
  }
  wave_lds_sync();
  if (live) {
    for (int t = lane; t < NC; t += kWave) {
      const int32_t d = cdec[t];
      double v = 0.0;
      if (d < 0) {
        v = mom[(d >> 10) & 0xfff];
      } else {
        const int nc = (d >> 22) & 0xf;
        const double *Tl = lds_T + (d & 0x3ff);
        const double *ms = mom + ((d >> 10) & 0xfff);
        for (int mm = 0; mm < nc; ++mm) v += Tl[mm] * ms[mm];
      }
      mu[t] = v;
      if (components) components[(size_t)row * NC + t] = v;
    }
  }
  wave_lds_sync();
  if (live) {
    for (int t = lane; t < NF; t += kWave) {
      const int32_t d = fdec[t];
      double F;
      if (d < 0) {
        F = fabs(mu[d & 0xfff]);
      } else {
        const int nc = (d >> 20) & 0xf;
        const double *mv = mu + (d & 0xfff);
        const double *wl = lds_w + ((d >> 12) & 0xff);
        double a = 0.0;
        for (int cc = 0; cc < nc; ++cc) a += wl[cc] * mv[cc] * mv[cc];
        F = sqrt(a);
      }
      if (F64OUT) ((double *)features)[(size_t)row * NF + t] = F;
      else ((float *)features)[(size_t)row * NF + t] = (float)F;
    }
  }
}

using OverlapFn = void (*)(PlanDev, BatchDev, NbrDev, const double4 *, const int32_t *, double *, const int64_t *,
                           int, int, int, unsigned long long *, const void *);

// SCREEN: per-primitive screening; OCC: the neighbours' occupancies scale the
// terms (without occupancies they are 1, so the variants that are not on the
// common path always multiply); STEP_K: a step's primitive loops end with the
// largest count among its own elements, where an exponential is dear (FP64) and
// the counts differ.  With one count for all elements the plan's is as good, and
// the test alone costs (l <= 2, 1500 atoms: 0.14 -> 0.16 ms); the screened kernels
// test every row anyway.
template <int L, int MODE, bool LDS, bool SCREEN, bool OCC, bool STEP_K> OverlapFn pick_k(int kb) {
  if (kb <= 4) return k_overlap<L, 4, MODE, LDS, SCREEN, OCC, false, STEP_K>;
  if (kb <= 8) return k_overlap<L, 8, MODE, LDS, SCREEN, OCC, false, STEP_K>;
  return k_overlap<L, 16, MODE, LDS, SCREEN, OCC, false, STEP_K>;
}
template <int MODE, bool LDS, bool SCREEN, bool OCC, bool STEP_K> OverlapFn pick_l(int lmax, int kb) {
  switch (lmax) {
    case 0: return pick_k<0, MODE, LDS, SCREEN, OCC, STEP_K>(kb);
    case 1: return pick_k<1, MODE, LDS, SCREEN, OCC, STEP_K>(kb);
    case 2: return pick_k<2, MODE, LDS, SCREEN, OCC, STEP_K>(kb);
    case 3: return pick_k<3, MODE, LDS, SCREEN, OCC, STEP_K>(kb);
    default: return pick_k<4, MODE, LDS, SCREEN, OCC, STEP_K>(kb);
  }
}
template <int MODE> OverlapFn pick_overlap(const PlanDev &P, bool lds, bool occ) {
  const int lmax = P.lmax, kb = P.kb;
  if (P.screen)
    return lds ? pick_l<MODE, true, true, true, false>(lmax, kb) : pick_l<MODE, false, true, true, false>(lmax, kb);
  if constexpr (MODE == ACC_F64)
    if (P.kmin < P.kmax)
      return lds ? pick_l<MODE, true, false, true, true>(lmax, kb) : pick_l<MODE, false, false, true, true>(lmax, kb);
  if (!lds) return pick_l<MODE, false, false, true, false>(lmax, kb);
  if constexpr (MODE == ACC_TERMS) return pick_l<MODE, true, false, true, false>(lmax, kb);
  else return occ ? pick_l<MODE, true, false, true, false>(lmax, kb) : pick_l<MODE, true, false, false, false>(lmax, kb);
}

// tabulated radial factors (FP32 modes): no coefficient table, no primitive loop
template <int MODE> OverlapFn pick_tab(int lmax) {
  switch (lmax) {
    case 0: return k_overlap<0, 4, MODE, false, false, true, true>;
    case 1: return k_overlap<1, 4, MODE, false, false, true, true>;
    case 2: return k_overlap<2, 4, MODE, false, false, true, true>;
    case 3: return k_overlap<3, 4, MODE, false, false, true, true>;
    default: return k_overlap<4, 4, MODE, false, false, true, true>;
  }
}

int acc_mode(const gmp_plan *p, bool components) {
  if (p->prec == GMP_FP64) return ACC_F64;
  return p->prec == GMP_FP32_COMPENSATED && components ? ACC_TERMS : ACC_WIDE;
}

}  // namespace

// Scratch memory of gmp_features_noalloc: a fixed array in device memory
// (each GPU the library runs on holds its own copy until the process ends).
// Host code never passes the array's name to a kernel: it takes the device
// address from hipGetSymbolAddress once per device and passes that.
constexpr size_t kNoallocScratchBytes = (size_t)GMP_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

// Device address of this GPU's scratch array (looked up on the first call on
// each device, with that device current), or null with *err set.
void *noalloc_scratch(size_t *bytes, hipError_t *err) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static void *addr[kMaxDev] = {};
  int dev = 0;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= kMaxDev) { *err = hipErrorInvalidDevice; return nullptr; }
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[dev]) {
    void *ptr = nullptr;
    *err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (*err != hipSuccess) return nullptr;
    addr[dev] = ptr;
  }
  *bytes = kNoallocScratchBytes;
  return addr[dev];
}

int chunk_size(const gmp_plan *p) { return p->tuning.chunk_pairs > 0 ? p->tuning.chunk_pairs : 0; }

// groups of cutoff slots per chunk that the tuning asks for
static int slot_groups(const gmp_plan *p) {
  const int g = p->tuning.sigma_groups > 0 ? p->tuning.sigma_groups : 1;
  return g < p->dev.S ? g : (p->dev.S > 0 ? p->dev.S : 1);
}

// Upper bound on the number of chunks of a batch with at most `pairs` pairs: the
// rows of partial moments it is given room for (groups of passes share a row, each
// writing its own slots).
int64_t max_chunks(const gmp_plan *p, int64_t n_atoms, int64_t pairs) {
  const int kc = chunk_size(p);
  return n_atoms + (kc > 0 ? pairs / kc + 1 : 0);
}

// Groups of passes per chunk (each a work item of its own): what the tuning
// asks for, and more where the centres alone leave wavefronts idle: towards
// 8,192 items, some four for each wavefront of the chip at two per SIMD (FP64,
// 1500 atoms: 0.187 ms aiming at 4,096, 0.173 at 8,192); 4,096 with the longer
// items of FP32 terms (4096 atoms: 0.396 ms, 0.420 aiming at 8,192).
static int item_groups(const gmp_plan *p, int64_t n_centres, int mode, int passes) {
  int64_t g = slot_groups(p);
  const int64_t aim = mode == ACC_TERMS ? 4096 : 8192;
  const int64_t want = (aim + n_centres - 1) / n_centres;
  if (g < want) g = want;
  return (int)(g < passes ? g : passes);
}

static int cus_cached() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, c = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
    cus = c > 0 ? c : 256;
  }
  return cus;
}

int persistent_blocks(const void *fn, size_t smem, int blocks_per_cu) {
  static std::mutex mu;
  static std::map<std::pair<const void *, size_t>, int> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto key = std::make_pair(fn, smem);
  auto itc = cache.find(key);
  if (itc != cache.end()) {
    const int per_c = itc->second / (cus_cached() > 0 ? cus_cached() : 1);
    return blocks_per_cu > 0 && blocks_per_cu < per_c ? cus_cached() * blocks_per_cu : itc->second;
  }
  int dev = 0, cus = 256, per = 2;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, 256, smem) != hipSuccess || per < 1) per = 1;
  cache[key] = cus * per;
  return blocks_per_cu > 0 && blocks_per_cu < per ? cus * blocks_per_cu : cus * per;
}

void launch_overlap(const gmp_plan *p, const BatchDev &bt, const NbrDev &nb, double *partial, int64_t *nch,
                    int64_t *chunk_off, int64_t *scan_aux, unsigned long long *counter, double4 *rw4,
                    int32_t *astruct, int64_t pairs_bound, bool components, hipStream_t s) {
  const int64_t N = n_centres(bt), NT = n_total(bt);  // NT >= N
  const int kc = chunk_size(p);
  if (N <= kSingleScanMax) {
    GMP_LAUNCH("overlap_prep", k_overlap_prep_scan, dim3((unsigned)(1 + (NT + kScanThreads - 1) / kScanThreads)),
               dim3(kScanThreads), 0, s, bt, nb, kc, chunk_off, rw4, astruct, counter);
  } else {
    GMP_LAUNCH("overlap_prep", k_overlap_prep, dim3((unsigned)((NT + 255) / 256)), dim3(256), 0, s, bt, nb, kc, nch,
               rw4, astruct, counter);
    scan_i64(nch, chunk_off, N, scan_aux, s);
  }
  const int lmax = p->dev.lmax, mode = acc_mode(p, components), slots = pass_slots(mode, lmax);
  const int passes = (p->dev.S + slots - 1) / slots, ng = item_groups(p, N, mode, passes);
  const bool f64 = mode == ACC_F64;
  const size_t tab_bytes = (size_t)p->dev.S * p->dev.E * p->dev.kb * kCoefStride * (f64 ? 8 : 4);
  const bool tabulated = p->dev.tab_n > 0 && !f64;
  const bool use_lds = tab_bytes <= 48 * 1024 && !tabulated;
  const size_t smem = use_lds ? tab_bytes + (size_t)p->dev.S * p->dev.E * 16 : 0;  // with its gaps
  const void *tab = f64 ? (const void *)p->dev.coef64 : (const void *)p->dev.coef32;
  const bool occ = bt.occ != nullptr;
  OverlapFn fn = tabulated           ? (mode == ACC_TERMS ? pick_tab<ACC_TERMS>(lmax) : pick_tab<ACC_WIDE>(lmax))
                 : f64               ? pick_overlap<ACC_F64>(p->dev, use_lds, occ)
                 : mode == ACC_TERMS ? pick_overlap<ACC_TERMS>(p->dev, use_lds, occ)
                                     : pick_overlap<ACC_WIDE>(p->dev, use_lds, occ);
  int64_t blocks = persistent_blocks((const void *)fn, smem, p->tuning.blocks_per_cu);
  // no more wavefronts than items: with some idle, those with an item would sit unevenly on the SIMDs
  const int64_t whole = kc > 0 ? pairs_bound / kc : 0;
  const int64_t need = ((N > whole ? N : whole) * ng + 3) / 4;
  if (blocks > need) blocks = need;
  if (blocks < 1) blocks = 1;
  // Items per request to the counter: requests from all wavefronts to one
  // address are served one after another, some 12 ns each (146,000 items of
  // the 512-structure batch took 1.83 ms one by one, 0.95 ms as 36,600), so
  // where a wavefront gets many items it takes several at a time, few enough
  // that the launch's end stays balanced.
  int64_t nbatch = N * ng / (blocks * 4 * 16);
  nbatch = nbatch < 1 ? 1 : (nbatch > 8 ? 8 : nbatch);
  GMP_LAUNCH("overlap", fn, dim3((unsigned)blocks), dim3(256), smem, s, p->dev, bt, nb, (const double4 *)rw4,
             (const int32_t *)astruct, partial, chunk_off, kc, ng, (int)nbatch, counter, tab);
}

void launch_finish(const gmp_plan *p, int64_t N, const double *partial, const int64_t *chunk_off,
                   const int32_t *order, void *features, double *components, unsigned long long *counter,
                   hipStream_t s) {
  if (N == 0) return;
  const int mode = acc_mode(p, components != nullptr), NM = n_moments(mode, p->dev.lmax);
  size_t smem = sizeof(double) * 4 * (size_t)(p->dev.S * NM + p->dev.ncomp_total) +
                sizeof(int32_t) * (size_t)(p->dev.ncomp_total + p->dev.nf);  // + the decode tables
  int64_t blocks = (N + 3) / 4;
  using FinishFn = void (*)(PlanDev, int64_t, const double *, const int64_t *, const int32_t *, void *, double *,
                            unsigned long long *);
  static const FinishFn fns[3][kMaxL + 1] = {
      {k_finish<0, true, false>, k_finish<1, true, false>, k_finish<2, true, false>, k_finish<3, true, false>,
       k_finish<4, true, false>},
      {k_finish<0, false, false>, k_finish<1, false, false>, k_finish<2, false, false>, k_finish<3, false, false>,
       k_finish<4, false, false>},
      {k_finish<0, false, true>, k_finish<1, false, true>, k_finish<2, false, true>, k_finish<3, false, true>,
       k_finish<4, false, true>}};
  const int lm = p->dev.lmax < 0 ? 0 : (p->dev.lmax > kMaxL ? kMaxL : p->dev.lmax);
  GMP_LAUNCH("norm", fns[mode][lm], dim3((unsigned)blocks), dim3(256), smem, s, p->dev, N,
             partial, chunk_off, order, features, components, counter);
}

}  // namespace gmp
