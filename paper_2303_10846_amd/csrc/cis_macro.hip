// gfx950 kernels of the macroscopic systems' coloured PR-SGS sweeps (Eq. 43 and its transpose) as one launch.
//
// A sweep pair over m colours is 2(m - 1) dependent relaxations of a few thousand six-component cells: bound by
// the latency of one step, not by arithmetic or bytes.  With one launch per relaxation a step costs a launch and
// its drain (4 to 5.3 us), 161 times for 40 pairs of 3 colours, whatever the mesh.  Here every cell keeps its
// operands in the registers of the lanes that own it (one lane per face slot) for all sweeps, and a step is an
// exchange through LDS and a barrier.  A mesh of up to 16 wavefronts runs in one workgroup.  A larger one is cut
// into one block a compute unit, of spatially close cells; a block relaxes, besides its own cells, those of its
// neighbours that its own depend on within the next h steps, so that increments go through memory once in h steps
// instead of after each (a word's way from a store to a load on another XCD takes 0.5 us, a whole exchange 1.5).
//
// Measured: a step costs 0.47 us in one workgroup (48 tetrahedra), most of it the relaxation's chain of FP64
// instructions; in blocks 0.85 us with windows of 4 steps (1 296 and 4 608 tetrahedra), 1.0 with windows of 3
// (3 072 cells of 6 slots) and 2.8 with an exchange every step (50 400 tetrahedra, 197 a block).  Against the
// launch per colour and its separate preparation the stage went from 400-450 to 76 us (48 tetrahedra), from
// 530-640 to 135 us (1 296), from 560-680 to 145 us (4 608) and from 945 to 450 us (50 400).  With the increments
// exchanged after every step (one wavefront a workgroup, each cell waiting for its neighbours' versions) it took
// 250 us on 1 296 and 274 us on 4 608 tetrahedra; half as many blocks cost up to a third more where the cells are
// many (4 608), since the wavefronts of a colour then share a SIMD, and nothing where they are few.
//
// Exchange: the six doubles of an increment travel as twelve 64-bit words, each holding 32 bits of payload and
// the 32-bit tag of its window, written and read with relaxed 64-bit atomics of agent scope (one word is always
// consistent, so a reader that finds the awaited tag has the value: one memory round trip and no fence).
//
// Progress: a block waits only for what the others publish before they wait in the same window (increments, and
// that they entered it), so the one furthest behind can go on, provided that all are resident and get to issue.
// Resident: the launch is cooperative (the runtime refuses a grid that does not fit and runs no two of them at
// once).  Issue: a SIMD serves its oldest wavefront first, and polling ones of other workgroups kept a younger one
// of the same SIMD from ever publishing (seen with three workgroups a SIMD), so a block has its compute unit to
// itself (kBlockLds), and its wavefronts poll only once all of them have published.  Every wait is bounded
// besides (kSweepPolls): a kernel of another stream or process may keep a block off the device for as long as it runs.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "cis_adjoint_math.h"
#include "cis_device.h"
#include "cis_internal.h"
#include "cis_macro.h"

namespace cis {

namespace {

// Lanes per cell: the face slots rounded up to 4 or 8 (lanes past NF carry zero terms).
template <int NF> struct SlotLanes { static constexpr int n = NF <= 4 ? 4 : 8; };

// The value of slot q's lane, in the lanes of a cell's first quad (4 lanes: a quad permutation; 8 lanes: slots
// 4 and 5 come from the second quad by a mirror of the eight).
template <int NF, int Q> __device__ inline double slot_value(double x) {
  if constexpr (Q < 4) return dpp_move<Q * 0x55>(x);
  else return dpp_move<0x141>(dpp_move<(Q - 4) * 0x55>(x));
}
// acc + x_0 y_0 + x_1 y_1 .. (fused) over the slots, in slot order
template <int NF, int Q = 0> __device__ inline void slot_fma(double& acc, double x, double y) {
  if constexpr (Q < NF) {
    acc = __builtin_fma(slot_value<NF, Q>(x), slot_value<NF, Q>(y), acc);
    slot_fma<NF, Q + 1>(acc, x, y);
  }
}
// x of a cell's first quad in all of its lanes
template <int NF> __device__ inline double of_first_quad(double x, int a) {
  if constexpr (SlotLanes<NF>::n == 4) return x;
  const double y = dpp_move<0x141>(x);
  return a < 4 ? x : y;
}

// The macro system's arithmetic with its roundings spelled out (no implicit fusing): the same bits as the
// per-colour launches, which keep the intermediate states in memory, whatever surrounds it here.  In the mixed
// mode a last-bit change of the prediction moves FP32 roundings of the equilibrium and, over iterations, W in the
// ninth digit.
#pragma clang fp contract(off)
__device__ inline double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline double dot3(double ax, double ay, double az, double bx, double by, double bz) {
  return fma_(az, bz, fma_(ax, bx, ay * by));
}
// Eqs. 1-5 as prim_of
__device__ inline Prim macro_prim(const double* W, double R) {
  Prim p;
  p.rho = W[0];
  const double ir = 1.0 / W[0];
  p.U[0] = W[1] * ir;
  p.U[1] = W[2] * ir;
  p.U[2] = W[3] * ir;
  const double eint = fma_(-0.5 * W[0], dot3(p.U[0], p.U[1], p.U[2], p.U[0], p.U[1], p.U[2]), W[4]);
  const double irR = ir / R;
  p.T = 0.4 * eint * irR;
  p.Trot = W[5] * irR;
  p.Ttr = (2.0 / 3.0) * (eint - W[5]) * irR;
  return p;
}
__device__ inline double macro_tau(const Prim& p, const GasC& g) { return visc(p.Ttr, g) / (p.rho * g.R * p.Ttr); }
// Spectral radius of the face between states a and b (Eq. 41, face state: the arithmetic mean)
__device__ inline double macro_radius(const Prim& a, const Prim& b, double nx, double ny, double nz, double dl,
                                      const GasC& g) {
  const double rho = 0.5 * (a.rho + b.rho), T = 0.5 * (a.T + b.T), Ttr = 0.5 * (a.Ttr + b.Ttr);
  const double Un = dot3(0.5 * (a.U[0] + b.U[0]), 0.5 * (a.U[1] + b.U[1]), 0.5 * (a.U[2] + b.U[2]), nx, ny, nz);
  return fabs(Un) + sqrt(g.gamma * g.R * T) + 2.0 * visc(Ttr, g) / (rho * dl);
}
// Euler flux with the rotational-energy row (Eq. 40), and its increment over G0
struct FluxState {
  double Un, p, H;  // normal velocity, pressure, rho E + p
};
__device__ inline FluxState flux_state(const double* W, double nx, double ny, double nz) {
  const double ir = 1.0 / W[0];
  const double Ux = W[1] * ir, Uy = W[2] * ir, Uz = W[3] * ir;
  const double e = fma_(-0.5 * W[0], dot3(Ux, Uy, Uz, Ux, Uy, Uz), W[4]);
  return FluxState{dot3(Ux, Uy, Uz, nx, ny, nz), 0.4 * e, fma_(0.4, e, W[4])};
}
__device__ inline void macro_flux(const double* W, double nx, double ny, double nz, double* G) {
  const FluxState f = flux_state(W, nx, ny, nz);
  G[0] = W[0] * f.Un;
  G[1] = fma_(W[1], f.Un, nx * f.p);
  G[2] = fma_(W[2], f.Un, ny * f.p);
  G[3] = fma_(nz, f.p, f.Un * W[3]);
  G[4] = f.H * f.Un;
  G[5] = W[5] * f.Un;
}
__device__ inline void macro_flux_increment(const double* W, double nx, double ny, double nz, const double* G0,
                                            double* dG) {
  const FluxState f = flux_state(W, nx, ny, nz);
  dG[0] = fma_(W[0], f.Un, -G0[0]);
  dG[1] = fma_(f.p, nx, W[1] * f.Un) - G0[1];
  dG[2] = fma_(f.p, ny, W[2] * f.Un) - G0[2];
  dG[3] = fma_(f.p, nz, W[3] * f.Un) - G0[3];
  dG[4] = fma_(f.H, f.Un, -G0[4]);
  dG[5] = fma_(W[5], f.Un, -G0[5]);
}

// Positions of the sequence 0, 1, .., m-1, m-2, .., 0, 1, .. for so many pairs
__host__ __device__ inline int sequence_length(int m, int pairs) {
  return pairs == 0 ? 0 : m == 1 ? 1 : pairs * 2 * (m - 1) + 1;
}

// A lane's cell and neighbour
template <int NF> struct SlotLane {
  static constexpr int NL = SlotLanes<NF>::n, CW = 64 / NL;
  int64_t i = 0, nb = kNoFace;  // cell, neighbour through this lane's slot (< 0: none)
  int a = 0, color = -1;
  bool valid = false, own = false;  // own: this launch's result of the cell comes from this lane
  int vi = 0, vn = -1;              // places of the cell's and the neighbour's increments in LDS

  // color = -1 where the wavefront owns no cells
  __device__ void find(const Dev& d, const SweepPlan& pl, int wave) {
    const int lane = threadIdx.x & 63, m = pl.m;
    a = lane % NL;
    if (wave >= pl.wave0[m]) return;
    color = 0;
    while (color + 1 < m && wave >= pl.wave0[color + 1]) ++color;
    const int64_t local = (int64_t)(wave - pl.wave0[color]) * CW + lane / NL;
    valid = local < pl.n[color];
    i = pl.off[color] + (valid ? local : 0);
    if (a < NF) nb = d.cell_nb[NF * i + a];
    if (!valid) nb = kNoFace;
    own = valid;
    vi = (int)i;
    vn = (int)nb;
  }
  __device__ void find(const Dev& d, const BlockRecord& r) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    a = lane % NL;
    color = __builtin_amdgcn_readfirstlane(r.color[wave]);
    if (color < 0) return;
    vi = wave * CW + lane / NL;
    valid = r.cell[vi] >= 0;
    i = valid ? r.cell[vi] : r.cell[wave * CW];
    if (!valid) return;
    own = r.own[vi] != 0;
    if (a < NF) {
      nb = d.cell_nb[NF * i + a];
      vn = r.nb[vi][a];
    }
  }
};

// A cell's six components over its lanes: lane a of four keeps components a and a + 4, lane a of eight component a
// (a < 6).  The lanes compute all six terms of one face each and swap them through LDS: 14 LDS accesses and one or two
// sums a lane, where every lane adding all six out of the others' registers took 72 to 120 instructions (the stage
// on 1 296 tetrahedra 152 -> 135 us, on 3 072 cells of 6 slots 282 -> 240 us).
template <int NF> struct Comps {
  static constexpr int n = NF <= 4 ? 2 : 1;
  double v[n];
  // put(component, value) for the lane's components
  template <class Put> __device__ void each(int a, Put&& put) const {
    if (n == 1 && a >= 6) return;
    put(a, v[0]);
    if (n == 2 && a < 2) put(a + 4, v[n - 1]);
  }
  __device__ void select(int a, const double* x) {
    double y[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      y[q] = x[q];
      asm("" : "+v"(y[q]));  // in registers: the selects below would otherwise become an indexed load from scratch
    }
    v[0] = a == 0 ? y[0] : a == 1 ? y[1] : a == 2 ? y[2] : a == 3 ? y[3] : a == 4 ? y[4] : y[5];
    if (n == 2) v[n - 1] = a == 0 ? y[4] : y[5];
  }
};
constexpr int kSwapRow = 65;  // doubles per component of a wavefront's swap space (64 lanes; 65: no bank conflicts)
// v -= the terms of the cell's slots, in slot order
template <int NF> __device__ inline void subtract_terms(Comps<NF>& v, const double* term, int a, double* swap) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < 6; ++q) swap[q * kSwapRow + lane] = term[q];
  asm volatile("" ::: "memory");  // a wavefront's LDS accesses keep their order
  const double* from = swap + (NF > 4 && a >= 6 ? 0 : a) * kSwapRow + (lane - a);
#pragma unroll
  for (int q = 0; q < NF; ++q) v.v[0] -= from[q];
  if constexpr (Comps<NF>::n == 2) {
    const double* high = swap + (a < 2 ? a + 4 : 4) * kSwapRow + (lane - a);
#pragma unroll
    for (int q = 0; q < NF; ++q) v.v[1] -= high[q];
  }
  asm volatile("" ::: "memory");
}

// The position after colour c of the sequence 0, 1, .., m-1, m-2, .., 0, 1, ..
__host__ __device__ inline void next_color(int& c, int& up, int m) {
  if (m < 2) return;
  if (c == m - 1) up = -1;
  if (c == 0) up = 1;
  c += up;
}

// The sweeps in one workgroup.  inc: the cells' increments in LDS, [nc][6], at the end those of the last sweep.
// relax(xj, x): one relaxation from the neighbour's increment xj to the lane's components x of the cell's.
template <int NF, class Relax>
__device__ inline void sweeps_in_lds(const SlotLane<NF>& L, int64_t nc, int m, int steps, double* inc, Relax&& relax) {
  for (int64_t k = threadIdx.x; k < 6 * nc; k += blockDim.x) inc[k] = 0.0;
  __syncthreads();
  int c = 0, up = 1;
  for (int p = 0; p < steps; ++p) {
    if (c == L.color) {
      double xj[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) xj[q] = L.vn >= 0 ? inc[6 * L.vn + q] : 0.0;
      Comps<NF> x;
      relax(xj, x);
      if (L.valid) x.each(L.a, [&](int q, double v) { inc[6 * L.vi + q] = v; });
    }
    __syncthreads();
    next_color(c, up, m);
  }
}

// LDS of a workgroup of the sweeps in blocks: more than half a compute unit's, so that no two share one (the waits of
// one would keep the other's older wavefronts from issuing).
constexpr int kBlockLds = 96 * 1024;


// The sweeps in blocks (BlockPlan).  Within a window of h steps: LDS and a barrier a step, as in one workgroup.
// After it a workgroup has published its increments of the window's colours, tagged with the window, and waits for
// those that it reads.  A slot of another block may be relaxed here from values that are not up to date; such a
// result is needed by nothing in the window and is read from its owner after it, as its colour is one of the window's.
// Two buffers in turn: window w overwrites window w - 2, so a workgroup ends window w - 1 only when every block that
// reads from it has entered that window, that is has read window w - 2 (what a block reads follows the order of the
// colours and is not mutual, so this takes a word of its own).
// false: a wait ran out.
template <int NF, int Waves, class Relax>
__device__ inline bool sweeps_in_blocks(const SlotLane<NF>& L, const BlockRecord& r, int64_t nc, int m,
                                        int steps, int h, uint64_t* words, uint32_t tag0, uint32_t polls, double* inc,
                                        Relax&& relax) {
  constexpr int NT = 64 * Waves, K = 12 * kBlockReads / NT;
  static_assert(12 * kBlockReads % NT == 0 && kBlockMax <= NT, "polls of a thread");
  __shared__ int stuck;
  const int tid = (int)threadIdx.x;
  // this thread's words of the increments that it reads: 64-bit places in the buffer, 32-bit places in LDS
  uint32_t src[K], dst[K], colors = 0;
  const int reads = 12 * __builtin_amdgcn_readfirstlane(r.reads);
  const int acks = __builtin_amdgcn_readfirstlane(r.acks);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int t = tid + NT * k, v = t < reads ? r.read[t / 12] : 0, q = t % 12;
    src[k] = (uint32_t)(kSweepWords * r.cell[v] + q);
    dst[k] = (uint32_t)(12 * v + q);
    if (t < reads) colors |= (uint32_t)r.read_color[t / 12] << (4 * k);
  }
  uint64_t* const entered = words + 2 * kSweepWords * nc;  // [2][kBlockMax][8]
  const int ack = tid < acks ? r.ack[tid] : 0;
  for (int k = tid; k < 6 * kBlockVals; k += NT) inc[k] = 0.0;
  if (tid == 0) stuck = 0;
  __syncthreads();
  int c = 0, up = 1;
  uint32_t window = 0;
  for (int p0 = 0; p0 < steps; p0 += h, ++window) {
    const int n = steps - p0 < h ? steps - p0 : h;
    const bool more = p0 + h < steps;
    uint64_t* const buf = words + (window & 1u) * (uint64_t)(kSweepWords * nc);
    uint64_t* const in = entered + (window & 1u) * (uint64_t)(8 * kBlockMax);
    const uint32_t tag = tag0 + 1u + window;
    if (tid == NT - 1)
      __hip_atomic_store(in + 8 * blockIdx.x, (uint64_t)tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int last = -1;  // last step of the window that relaxes this wavefront's colour
    uint32_t relaxed = 0;
    for (int s = 0, cc = c, uu = up; s < n; ++s, next_color(cc, uu, m)) {
      if (cc == L.color) last = s;
      relaxed |= 1u << cc;
    }
    for (int s = 0; s < n; ++s) {
      if (c == L.color) {
        double xj[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) xj[q] = L.vn >= 0 ? inc[6 * L.vn + q] : 0.0;
        Comps<NF> x;
        relax(xj, x);
        if (L.valid) x.each(L.a, [&](int q, double v) { inc[6 * L.vi + q] = v; });
        if (more && s == last && L.own)
          x.each(L.a, [&](int q, double v) {
            const uint64_t t = (uint64_t)tag << 32, u = __builtin_bit_cast(uint64_t, v);
            uint64_t* to = buf + kSweepWords * L.i + 2 * q;
            __hip_atomic_store(to, t | (uint32_t)u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(to + 1, t | (u >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          });
      }
      __syncthreads();
      next_color(c, up, m);
    }
    if (!more) break;
    uint32_t wanted = tid < acks ? 1u << K : 0u;
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (tid + NT * k < reads && ((relaxed >> ((colors >> (4 * k)) & 15u)) & 1u)) wanted |= 1u << k;
    for (uint32_t spins = 0; wanted != 0; ++spins) {
      if (spins >= polls) {
        stuck = 1;
        break;
      }
      uint64_t got[K], hers = 0;
#pragma unroll
      for (int k = 0; k < K; ++k)
        if ((wanted >> k) & 1u) got[k] = __hip_atomic_load(buf + src[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((wanted >> K) & 1u) hers = __hip_atomic_load(in + 8 * ack, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (((wanted >> k) & 1u) && (uint32_t)(got[k] >> 32) == tag) {
          reinterpret_cast<uint32_t*>(inc)[dst[k]] = (uint32_t)got[k];
          wanted &= ~(1u << k);
        }
      // the reader entered this window (or by now the next but one, whose tag replaces this one's)
      if (((wanted >> K) & 1u) && (uint32_t)hers >= tag) wanted &= ~(1u << K);
    }
    __syncthreads();
    if (stuck) return false;
  }
  return true;
}

// The forms of both kernels: the whole mesh in one workgroup of up to kLocalThreads threads, or blocks of 8 or 16
// wavefronts.
enum Form { kLocal, kBlocks, kWideBlocks };
constexpr int threads_of(Form f) {
  return f == kLocal ? kLocalThreads : 64 * (f == kBlocks ? kBlockWaves : kWideBlockWaves);
}
#define CIS_SWEEP_KERNEL __global__ __launch_bounds__(threads_of(F)) \
    __attribute__((amdgpu_waves_per_eu(threads_of(F) / 256, threads_of(F) / 256)))
template <int NF, Form F> __device__ inline SlotLane<NF> lane_of(const Dev& d, const SweepPlan& pl, const BlockPlan& bp) {
  SlotLane<NF> L;
  if constexpr (F == kLocal) L.find(d, pl, __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)));
  else L.find(d, bp.rec[blockIdx.x]);
  return L;
}
// LDS: the increments, then the swap space of every wavefront.
__host__ __device__ constexpr int64_t increments_of(Form f, int64_t nc) { return 6 * (f == kLocal ? nc : kBlockVals); }
template <Form F> __device__ inline double* swap_space(double* lds, int64_t nc) {
  return lds + increments_of(F, nc) + 6 * kSwapRow * __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}
// x: the cell's increments after the sweeps
template <Form F, int NF, class Relax>
__device__ inline bool sweeps(const SlotLane<NF>& L, const SweepPlan& pl, const BlockPlan& bp, int64_t nc, int steps,
                              uint64_t* words, double* inc, uint32_t tag0, uint32_t polls, double* x, Relax&& relax) {
  if constexpr (F == kLocal)
    sweeps_in_lds<NF>(L, nc, pl.m, steps, inc, relax);
  else if (!sweeps_in_blocks<NF, threads_of(F) / 64>(L, bp.rec[blockIdx.x], nc, pl.m, steps, bp.h, words, tag0, polls,
                                                     inc, relax))
    return false;
  if (L.valid)
    for (int q = 0; q < 6; ++q) x[q] = inc[6 * L.vi + q];
  return true;
}

// Step 4 (Eqs. 38-43): macro flux per cell (Eq. 37), spectral radii r_ij (Eq. 41), diagonal and right-hand side
// of Eq. 43, the sweeps (matrix-free increment G(W_j + dW_j) - G(W_j)) and the predicted state with its
// equilibrium coefficients (q~ = q^n).
template <int NF, Form F>
CIS_SWEEP_KERNEL void k_macro_sweeps(Dev d, const double* W, const double* q, Work w, SweepPlan pl, BlockPlan bp,
                                  uint64_t* words, uint32_t tag0, uint32_t polls, int steps) {
  extern __shared__ __align__(16) double sweep_lds[];
  const bool lost = F != kLocal && (w.flag[0] & kSweepStuck);  // an earlier launch of the call gave up
  const SlotLane<NF> L = lane_of<NF, F>(d, pl, bp);
  const int64_t i = L.i;
  const GasC& g = d.gas;
  const double* geo = d.cell_geo + Lay<NF>::CG * i;
  const double iV = geo[1];
  double Wi[6], Wj[6];
  const double* Wn = W + 6 * (L.nb >= 0 ? L.nb : i);
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    Wi[m] = W[6 * i + m];
    Wj[m] = Wn[m];
  }
  const Prim pa = macro_prim(Wi, g.R), pb = macro_prim(Wj, g.R);
  const double tau = macro_tau(pa, g);
  double nx = 0, ny = 0, nz = 0, hav = 0, r = 0, fsum[6] = {0, 0, 0, 0, 0, 0}, G0[6] = {0, 0, 0, 0, 0, 0};
  const int32_t f = L.a < NF ? d.cell_face[NF * i + L.a] : -1;
  if (f >= 0) {
    const double* s = geo + CG_FACE + CG_SLOT * L.a;
    nx = s[2];
    ny = s[3];
    nz = s[4];
    hav = 0.5 * s[1];
    r = macro_radius(pa, pb, nx, ny, nz, d.face_geo[FGW * (int64_t)f + 5], g);
    const double* fm = w.face_mac + 6 * (int64_t)f;
#pragma unroll
    for (int m = 0; m < 6; ++m) fsum[m] = s[0] * fm[m];
    // G_n(W_j^n) along the outward normal, constant during the sweeps
    if (L.nb >= 0) macro_flux(Wj, nx, ny, nz, G0);
  }
  double D = 0.0, res[6];
  slot_fma<NF>(D, hav, r);
  const double inv_dt = inv_dt_cell(d, geo[2]);
  D += inv_dt;
  D = of_first_quad<NF>(D, L.a);
  const double iD = 1.0 / D, D5 = D + 1.0 / (g.Z * tau);
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    double Fm = 0.0;
    slot_fma<NF>(Fm, fsum[m], iV);
    if (L.own && L.a == 0) w.Fmac[6 * i + m] = Fm;
    res[m] = -Fm;
  }
  res[5] += fma_(pa.rho * g.R, pa.T, -Wi[5]) / (g.Z * tau);
  // the gas's constants wait for the end of the sweeps in vector registers: the sweeps in blocks need the scalar ones
  GasC gas = g;
  if constexpr (F == kBlocks)
    for (double* c : {&gas.R, &gas.gamma, &gas.Z, &gas.delta, &gas.omega0, &gas.omega1, &gas.mu_ref, &gas.omega_v,
                      &gas.T_ref, &gas.C_s})
      asm("" : "+v"(*c));
  double dW[6] = {0, 0, 0, 0, 0, 0};
  Comps<NF> mine;
#pragma unroll
  for (int m = 0; m < 6; ++m) res[m] = of_first_quad<NF>(res[m], L.a);
  mine.select(L.a, res);
  double* const swap = swap_space<F>(sweep_lds, d.nc);
  auto relax = [&](const double* dWj, Comps<NF>& x) {
    double term[6] = {0, 0, 0, 0, 0, 0};
    if (L.nb >= 0) {
      double Wp[6], dG[6];
#pragma unroll
      for (int m = 0; m < 6; ++m) Wp[m] = Wj[m] + dWj[m];
      macro_flux_increment(Wp, nx, ny, nz, G0, dG);
#pragma unroll
      for (int m = 0; m < 6; ++m) term[m] = hav * fma_(-r, dWj[m], dG[m]);
    }
    x = mine;
    subtract_terms<NF>(x, term, L.a, swap);
    constexpr int top = Comps<NF>::n - 1;
    const double quotient = x.v[top] / D5;
    if (top == 1) x.v[0] *= iD;
    x.v[top] = L.a == (top == 1 ? 1 : 5) ? quotient : x.v[top] * iD;
  };
  if (lost || !sweeps<F>(L, pl, bp, d.nc, steps, words, sweep_lds, tag0, polls, dW, relax)) {
    atomicOr(&w.flag[0], kSweepStuck);
    return;
  }
  if (!L.own || L.a != 0) return;
  // W~ = W^n + dW~; predicted equilibrium coefficients with q~ = q^n
  double Wt[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    w.dW[6 * i + m] = dW[m];
    Wt[m] = Wi[m] + dW[m];
    w.Wt[6 * i + m] = Wt[m];
  }
  const Prim p = macro_prim(Wt, gas.R);
  if (!(p.rho > 0.0) || !(p.T > 0.0) || !(p.Ttr > 0.0) || !(p.Trot > 0.0)) atomicOr(&w.flag[0], 1);
  double* e = w.eq + ER * i;
  eq_coeffs(p, q + 6 * i, gas, e);
  const double taut = macro_tau(p, gas);
  e[7] = taut;
  w.mbase[i] = inv_dt + 1.0 / taut;
}

// Mac^T u = t: row i couples the neighbours j through Mac_ji^T = -(A_f/V_j)(dG_n/dW (W_i)^T + r_f I)/2 with n out
// of cell i (the flux Jacobian is odd in n and r_f is the same from both sides); Mac is the steady macro system,
// D_i = sum_f (A_f/V_i) r_f / 2 (+ 1/(Z tau_i) for rho E_rot).
template <int NF, Form F>
CIS_SWEEP_KERNEL void k_adj_macro_sweeps(Dev d, const double* W, const double* t, double* u, int32_t* flag, SweepPlan pl,
                                      BlockPlan bp, uint64_t* words, uint32_t tag0, uint32_t polls, int steps) {
  extern __shared__ __align__(16) double sweep_lds[];
  const bool lost = F != kLocal && (flag[0] & kSweepStuck);
  const SlotLane<NF> L = lane_of<NF, F>(d, pl, bp);
  const int64_t i = L.i;
  const GasC& g = d.gas;
  const double* geo = d.cell_geo + Lay<NF>::CG * i;
  double Wi[6], Wj[6];
  const double* Wn = W + 6 * (L.nb >= 0 ? L.nb : i);
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    Wi[m] = W[6 * i + m];
    Wj[m] = Wn[m];
  }
  const Prim pa = macro_prim(Wi, g.R), pb = macro_prim(Wj, g.R);
  double nx = 0, ny = 0, nz = 0, hav = 0, half_av = 0, r = 0;
  const int32_t f = L.a < NF ? d.cell_face[NF * i + L.a] : -1;
  if (f >= 0) {
    const double* s = geo + CG_FACE + CG_SLOT * L.a;
    nx = s[2];
    ny = s[3];
    nz = s[4];
    hav = 0.5 * s[1];
    if (L.nb >= 0) half_av = 0.5 * s[1] * geo[0] * d.cell_geo[Lay<NF>::CG * L.nb + 1];
    r = macro_radius(pa, pb, nx, ny, nz, d.face_geo[FGW * (int64_t)f + 5], g);
  }
  const double tau = macro_tau(pa, g);
  double D = 0.0;
  slot_fma<NF>(D, hav, r);
  D = of_first_quad<NF>(D, L.a);
  const double iD = 1.0 / D, iD5 = 1.0 / (D + 1.0 / (g.Z * tau));
  double ti[6], x[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int m = 0; m < 6; ++m) ti[m] = t[6 * i + m];
  Comps<NF> mine, scale;
  mine.select(L.a, ti);
  for (int k = 0; k < Comps<NF>::n; ++k) scale.v[k] = k == Comps<NF>::n - 1 && L.a == (k == 1 ? 1 : 5) ? iD5 : iD;
  double* const swap = swap_space<F>(sweep_lds, d.nc);
  auto relax = [&](const double* uj, Comps<NF>& ui) {
    double term[6] = {0, 0, 0, 0, 0, 0};
    if (L.nb >= 0) {
      double gj[6];
      euler_flux_vjp(Wi, nx, ny, nz, uj, gj);
#pragma unroll
      for (int m = 0; m < 6; ++m) term[m] = -(half_av * (gj[m] + r * uj[m]));
    }
    ui = mine;
    subtract_terms<NF>(ui, term, L.a, swap);
    for (int k = 0; k < Comps<NF>::n; ++k) ui.v[k] *= scale.v[k];
  };
  if (lost || !sweeps<F>(L, pl, bp, d.nc, steps, words, sweep_lds, tag0, polls, x, relax)) {
    atomicOr(flag, kSweepStuck);
    return;
  }
  if (!L.own || L.a != 0) return;
#pragma unroll
  for (int m = 0; m < 6; ++m) u[6 * i + m] = x[m];
}

// The readers of each block, from the links that the plans of all blocks set.  all_colors: every window relaxes
// every colour, so that a reader which this block reads from is known to have entered a window by its increments.
__global__ __launch_bounds__(kBlockMax) void k_block_acks(BlockPlan bp, int blocks, int all_colors) {
  const int me = (int)threadIdx.x;
  if (me >= blocks) return;
  BlockRecord& r = bp.rec[me];
  int n = 0;
  for (int w = 0; w < kBlockMax / 32; ++w)
    for (uint32_t bits = bp.link[me * (kBlockMax / 32) + w]; bits != 0; bits &= bits - 1u) {
      const int b = 32 * w + __ffs((int)bits) - 1;
      const bool mutual = (bp.link[b * (kBlockMax / 32) + me / 32] >> (me % 32)) & 1u;
      if (!all_colors || !mutual) r.ack[n++] = (int16_t)b;
    }
  r.acks = n;
}

// The plan of block blockIdx.x for windows of cand.h[blockIdx.y] steps (write: into its record and the
// links; else the owners and the most wavefronts of a block, into bp.most[blockIdx.y], kTooMany where something else does
// not fit).
// What a window's own values depend on, by walking its steps backwards: `need` holds the cells whose value is needed
// after the step; those of the step's colour are relaxed in it and pass the need on to their neighbours.
constexpr int kPlanThreads = 1024, kTooMany = 1 << 20;
struct BlockCands {
  int n = 0, h[kBlockCands];
};
__global__ __launch_bounds__(kPlanThreads) void k_block_plan(Dev d, SweepPlan pl, BlockPlan bp, BlockCands cand, int cw,
                                                             int write) {
  enum : uint8_t { kNeed = 1, kValue = 2, kSlot = 4, kOwn = 8, kRelax = 16, kRead = 32 };
  extern __shared__ int16_t plan_lds[];
  int16_t* const loc = plan_lds;  // [nc] place of a cell's increment
  uint8_t* const st = reinterpret_cast<uint8_t*>(plan_lds + d.nc);  // [nc]
  __shared__ int part[kSweepColors + 2][kPlanThreads / 64];
  const int nc = (int)d.nc, m = pl.m, tid = (int)threadIdx.x, h = cand.h[blockIdx.y];
  const int period = m > 1 ? 2 * (m - 1) : 1, phases = h < period ? period / h : 1;
  for (int i = tid; i < nc; i += kPlanThreads) st[i] = 0;
  __syncthreads();
  const int j0 = (int)((int64_t)nc * blockIdx.x / gridDim.x), j1 = (int)((int64_t)nc * (blockIdx.x + 1) / gridDim.x);
  for (int j = j0 + tid; j < j1; j += kPlanThreads) {
    const int i = d.spatial[j];
    st[i] = kOwn | kValue | kSlot;
    if (!write && blockIdx.y == 0) bp.owner[i] = (int32_t)blockIdx.x;
  }
  __syncthreads();
  // full windows of every phase, then windows cut short after a whole number of periods and one step
  for (int w = 0; w < phases + (h > period ? h / period : 1); ++w) {
    const bool full = w < phases;
    const int n = full ? h : (w - phases) * period + 1;
    for (int i = tid; i < nc; i += kPlanThreads) st[i] = (uint8_t)((st[i] & ~kNeed) | (st[i] & kOwn ? kNeed : 0));
    __syncthreads();
    for (int s = n - 1; s >= 0; --s) {
      const int at = ((full ? w * h : 0) + s) % period, c = at < m ? at : period - at;
      for (int i = pl.off[c] + tid; i < pl.off[c] + pl.n[c]; i += kPlanThreads)
        if (st[i] & kNeed) st[i] = (uint8_t)((st[i] & ~kNeed) | kSlot | kValue | kRelax);
      __syncthreads();
      for (int i = pl.off[c] + tid; i < pl.off[c] + pl.n[c]; i += kPlanThreads)
        if (st[i] & kRelax) {
          st[i] = (uint8_t)(st[i] & ~kRelax);
          for (int a = 0; a < d.mf; ++a) {
            const int32_t nb = d.cell_nb[(int64_t)d.mf * i + a];
            if (nb >= 0) st[nb] = (uint8_t)(st[nb] | kNeed | kValue);
          }
        }
      __syncthreads();
    }
    for (int i = tid; i < nc; i += kPlanThreads)
      if ((st[i] & kNeed) && !(st[i] & kOwn)) st[i] |= kRead;
    __syncthreads();
  }
  // Counts, then places in cell order: wavefront wv takes the wv-th part of a colour's cells, or of all cells, so that
  // its places follow those of lower wavefronts.  Rows of `part`: the slots of each colour, other values, values read.
  constexpr int kWaves = kPlanThreads / 64;
  const int lane = tid & 63, wv = tid >> 6;
  const auto cells = [&](int row, uint8_t with, uint8_t without, auto&& put) {
    const int first = row < m ? pl.off[row] : 0, n = row < m ? pl.n[row] : nc;
    const int j1 = first + (int)((int64_t)n * (wv + 1) / kWaves);
    int found = 0;
    for (int j0 = first + (int)((int64_t)n * wv / kWaves); j0 < j1; j0 += 64) {
      const int i = j0 + lane;
      const bool set = i < j1 && (st[i] & with) && !(st[i] & without);
      const uint64_t mask = __ballot(set);
      if (set) put(i, found + __popcll(mask & ((1ull << lane) - 1ull)));
      found += __popcll(mask);
    }
    return found;
  };
  for (int c = 0; c < m + 2; ++c) {
    const int found = cells(c, c < m ? kSlot : c == m ? kValue : kRead, c == m ? kSlot : 0, [](int, int) {});
    if (lane == 0) part[c][wv] = found;
  }
  __syncthreads();
  const auto sum = [&](int row, int waves) {
    int n = 0;
    for (int k = 0; k < waves; ++k) n += part[row][k];
    return n;
  };
  int waves = 0;
  for (int c = 0; c < m; ++c) waves += (sum(c, kWaves) + cw - 1) / cw;
  const int slots = waves * cw, others = sum(m, kWaves), reads = sum(m + 1, kWaves);
  if (!write) {
    const bool fits = slots + others <= kBlockVals && reads <= kBlockReads;
    if (tid == 0) atomicMax(&bp.most[blockIdx.y], fits ? waves : kTooMany);
    return;
  }
  BlockRecord* const r = bp.rec + blockIdx.x;
  if (tid < kWideBlockWaves) {  // the colour of each wavefront of slots
    int c = 0, end = 0;
    for (; c < m; ++c) {
      end += (sum(c, kWaves) + cw - 1) / cw;
      if (tid < end) break;
    }
    r->color[tid] = c < m ? c : -1;
  }
  for (int c = 0, base = 0; c < m + 1; ++c) {
    const int before = base + sum(c, wv);
    (void)cells(c, c < m ? kSlot : kValue, c < m ? 0 : kSlot,
                [&](int i, int at) { loc[i] = (int16_t)min(before + at, 32767); });
    base += c < m ? (sum(c, kWaves) + cw - 1) / cw * cw : 0;
  }
  __syncthreads();
  const int read0 = sum(m + 1, wv);
  (void)cells(m + 1, kRead, 0, [&](int i, int at) {
    at = min(read0 + at, kBlockReads - 1);
    int c = 0;
    while (c + 1 < m && i >= pl.off[c + 1]) ++c;
    r->read[at] = loc[i];
    r->read_color[at] = (uint8_t)c;
    atomicOr(&bp.link[bp.owner[i] * (kBlockMax / 32) + blockIdx.x / 32], 1u << (blockIdx.x % 32));
  });
  for (int v = tid; v < kBlockVals; v += kPlanThreads) r->cell[v] = -1;
  __syncthreads();
  if (tid == 0) r->reads = reads;
  for (int i = tid; i < nc; i += kPlanThreads) {
    const uint8_t f = st[i];
    if (!(f & kValue)) continue;
    const int v = loc[i];
    r->cell[v] = i;
    if (!(f & kSlot)) continue;
    r->own[v] = f & kOwn ? 1 : 0;
    for (int a = 0; a < d.mf; ++a) {
      const int32_t nb = d.cell_nb[(int64_t)d.mf * i + a];
      r->nb[v][a] = nb >= 0 && (st[nb] & kValue) ? loc[nb] : (int16_t)-1;
    }
  }
}

template <int NF, Form F> const void* kernel_of(bool adjoint) {
  return adjoint ? (const void*)k_adj_macro_sweeps<NF, F> : (const void*)k_macro_sweeps<NF, F>;
}
template <Form F> const void* kernel_of(bool adjoint, const Dev& d) {
  return d.mf == 4 ? kernel_of<4, F>(adjoint) : kernel_of<kMaxFaces, F>(adjoint);
}

static_assert(sizeof(double) * (6 * kBlockVals + 6 * kSwapRow * kWideBlockWaves) <= kBlockLds, "LDS of a block");

hipError_t enqueue(const Dev& d, bool adjoint, const MacroSweeps& s, void** args, hipStream_t st) {
  // as many wavefronts as own cells: idle ones cost every barrier (a pass of 48 tetrahedra 166.6 -> 162.6 us)
  if (s.plan.local) {
    const int waves = s.plan.wave0[s.plan.m];
    return hipLaunchKernel(kernel_of<kLocal>(adjoint, d), dim3(1), dim3(64u * (unsigned)waves), args,
                           sizeof(double) * (size_t)(increments_of(kLocal, d.nc) + 6 * kSwapRow * waves), st);
  }
  const void* k = s.block.wide ? kernel_of<kWideBlocks>(adjoint, d) : kernel_of<kBlocks>(adjoint, d);
  return hipLaunchCooperativeKernel(k, dim3((unsigned)s.block.blocks),
                                    dim3(threads_of(s.block.wide ? kWideBlocks : kBlocks)), args, (unsigned)kBlockLds, st);
}
// false: not launched.  An error that was there before stays for the caller's check; a refusal of this launch (a grid
// that the device cannot hold at once) keeps the state at a launch per colour from here on.
bool run(const Dev& d, bool adjoint, MacroSweeps& s, void** args, hipStream_t st) {
  if (hipPeekAtLastError() != hipSuccess) return false;
  if (enqueue(d, adjoint, s, args, st) == hipSuccess) return true;
  (void)hipGetLastError();
  s.plan.m = 0;
  return false;
}

// Zeros in the exchange words, and in what the layout of the blocks accumulates
__global__ __launch_bounds__(256) void k_clear_words(uint64_t* words, int64_t n, BlockPlan bp) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k < n) words[k] = 0;
  if (k < kBlockLink) bp.link[k] = 0;
  if (k < kBlockCands) bp.most[k] = 0;
}

// The tags of one launch follow the last launch's, so no word left behind by an earlier one carries an awaited tag and
// a later window has the larger one.  Before they would pass kSweepTagMax (13 million launches of 161 steps) the words
// are cleared and the tags start again; 0 is the tag of no window.
uint32_t take_tags(const Dev& d, MacroSweeps& f, int steps, hipStream_t st) {
  const uint32_t n = (uint32_t)steps + 1u;
  if (f.block.blocks && f.tag > kSweepTagMax - n) {
    clear_sweep_words(f, d.nc, st);
    f.tag = 0;
  }
  const uint32_t t0 = f.tag;
  f.tag += n;
  return t0;
}
uint32_t take_polls(MacroSweeps& f) { return f.polls_from > 0 ? (--f.polls_from, kSweepPolls) : f.polls; }

}  // namespace

void clear_sweep_words(const MacroSweeps& f, int64_t nc, hipStream_t st) {
  const int64_t n = sweep_words(nc);
  static_assert(2 * 8 * kBlockMax >= kBlockLink && kBlockLink >= kBlockCands, "words cover the links");
  hipLaunchKernelGGL(k_clear_words, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, f.words, n, f.block);
}

SweepPlan sweep_plan(const Dev& d, const int64_t* color_off, int64_t n_colors) {
  SweepPlan pl;
  const int cw = 64 / (d.mf == 4 ? SlotLanes<4>::n : SlotLanes<kMaxFaces>::n);
  int m = 0, waves = 0;
  for (int64_t c = 0; c < n_colors; ++c) {
    const int64_t n = color_off[c + 1] - color_off[c];
    if (n <= 0) continue;
    if (m == kSweepColors || n > (int64_t)1 << 24) return SweepPlan();
    pl.off[m] = (int32_t)color_off[c];
    pl.n[m] = (int32_t)n;
    pl.wave0[m] = waves;
    waves += (int)((n + cw - 1) / cw);
    pl.wave0[++m] = waves;
  }
  if (m == 0) return SweepPlan();
  pl.local = waves <= kLocalThreads / 64;
  pl.m = m;
  return pl;
}

int block_count(const SweepPlan& pl, const Dev& d, int64_t nc) {
  if (pl.m == 0 || pl.local || nc > kBlockCells) return 0;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return (int)std::min<int64_t>(std::min(cus, kBlockMax), nc);
}

// Windows tried, the longest first (the fewest exchanges; on 1 296 tetrahedra 144 us with 4 steps, 192 with 2):
// a period and its divisors (and two periods of two colours, whose cells all
// depend on each other only through the other colour).
static BlockCands block_windows(int m) {
  const int period = m > 1 ? 2 * (m - 1) : 1;
  BlockCands c;
  if (period == 2) c.h[c.n++] = 4;
  for (int k = 1; k <= period && c.n < kBlockCands; ++k)
    if (period % k == 0) c.h[c.n++] = period / k;
  return c;
}

static int cells_per_wave(const Dev& d) { return 64 / (d.mf == 4 ? SlotLanes<4>::n : SlotLanes<kMaxFaces>::n); }

void lay_out_blocks(const Dev& d, MacroSweeps& f, hipStream_t st) {
  // an error that is there already is the caller's to report: the layout waits for the next call
  if (f.laid_out || f.plan.m == 0 || f.plan.local || hipPeekAtLastError() != hipSuccess) return;
  f.laid_out = true;
  const int blocks = f.block.blocks;
  BlockCands c = block_windows(f.plan.m);
  int32_t most[kBlockCands] = {};
  clear_sweep_words(f, d.nc, st);
  hipLaunchKernelGGL(k_block_plan, dim3(blocks, c.n), dim3(kPlanThreads), 3 * (size_t)d.nc, st, d, f.plan, f.block, c,
                     cells_per_wave(d), 0);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(most, f.block.most, sizeof most, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  // 8 wavefronts where a window fits them, two a SIMD; 16 only where none does (a longer window with 16 gains
  // nothing: the wavefronts of a colour share a SIMD)
  int k = 0;
  while (k < c.n && most[k] > kBlockWaves) ++k;
  f.block.wide = k == c.n;
  if (f.block.wide)
    for (k = 0; k < c.n && most[k] > kWideBlockWaves; ++k) {}
  if (e == hipSuccess && k < c.n) {
    f.block.h = c.h[0] = c.h[k];
    hipLaunchKernelGGL(k_block_plan, dim3(blocks), dim3(kPlanThreads), 3 * (size_t)d.nc, st, d, f.plan, f.block, c,
                       cells_per_wave(d), 1);
    hipLaunchKernelGGL(k_block_acks, dim3(1), dim3(kBlockMax), 0, st, f.block, blocks, f.block.h >= f.plan.m ? 1 : 0);
    e = hipGetLastError();
  }
  if (e != hipSuccess || k == c.n) {
    (void)hipGetLastError();
    f.plan.m = 0;
  }
}

bool blocks_pay(const MacroSweeps& f, int n_pairs, int64_t others) {
  return 10.0 + 2.0 * sequence_length(f.plan.m, n_pairs) > 1.2 * (double)others;
}

bool launch_macro_sweeps(const Dev& d, const Bufs& b, const Work& w, MacroSweeps& f, int n_macro, hipStream_t st) {
  if (!f.ready()) return false;
  int steps = sequence_length(f.plan.m, n_macro);
  uint32_t tag0 = take_tags(d, f, steps, st), polls = take_polls(f);
  Dev dd = d;
  const double *W = b.W, *q = b.q;
  Work ww = w;
  void* args[] = {&dd, &W, &q, &ww, &f.plan, &f.block, &f.words, &tag0, &polls, &steps};
  return run(d, false, f, args, st);
}

bool launch_adj_macro_sweeps(const Dev& d, const Bufs& b, MacroSweeps& f, const double* t, double* u, int n_pairs,
                             int32_t* flag, hipStream_t st) {
  if (!f.ready()) return false;
  int steps = sequence_length(f.plan.m, n_pairs);
  uint32_t tag0 = take_tags(d, f, steps, st), polls = take_polls(f);
  Dev dd = d;
  const double* W = b.W;
  void* args[] = {&dd, &W, &t, &u, &flag, &f.plan, &f.block, &f.words, &tag0, &polls, &steps};
  return run(d, true, f, args, st);
}

}  // namespace cis
