// gfx950 kernels of the macroscopic systems' coloured PR-SGS sweeps (Eq. 43 and its transpose) as one launch.
//
// A sweep pair over m colours is 2(m - 1) dependent relaxations of a few thousand six-component cells: bound by
// the latency of one step, not by arithmetic or bytes.  With one launch per relaxation a step costs a launch and
// its drain (4 to 5.3 us), 161 times for 40 pairs of 3 colours, whatever the mesh.  Here every cell keeps its
// operands in the registers of the lanes that own it (one lane per face slot) for all sweeps.  A mesh of up to 16
// wavefronts runs in one workgroup: increments in LDS, one barrier a step.  A larger one, one wavefront a
// workgroup, runs as a dataflow: a cell's relaxation waits for the versions of its neighbours' increments that
// the coloured order asks for, and for nothing else.
//
// Measured: a step costs 0.48 us in one workgroup (48 tetrahedra), 1.55 us as a dataflow on 1 296 tetrahedra (81
// wavefronts; 0.5 us of it one word's way from a store to a load on another XCD, the rest the poll, the flux
// and its divisions) and 1.7 us on 4 608; against the launch per colour and its separate preparation the stage
// went from 400-450 to 77 us, from 530-640 to 250 us and from 560-680 to 274 us.
//
// Exchange: the six doubles of an increment travel as twelve 64-bit words, each holding 32 bits of payload and
// the 32-bit tag of its version, written with relaxed 64-bit atomics of agent scope (one word is always
// consistent, so a reader that finds the awaited tag in all twelve has the whole version: one memory round trip
// and no fence).  A wavefront reads the lines of its 64 neighbours with 16-byte LDS-DMA loads of device scope
// (eight lanes a line, 64 line requests a poll instead of the 768 of one load per lane and word).  A single buffer
// is enough: a neighbour publishes its next version only after it has read this cell's, which this cell publishes
// after reading the neighbour's current one.
//
// Progress: a wavefront relaxes cells of one colour, takes its relaxations in sweep order and waits only for
// versions of earlier positions of the sequence, so the wavefront at the lowest position can go on, provided that
// it is resident and gets to issue.  Resident: the launch is cooperative (the runtime refuses a grid that does
// not fit and runs no two of them at once).  Issue: a SIMD serves its oldest wavefront first, and two or three
// polling ones kept a younger one of the same SIMD from ever publishing (seen with 3 wavefronts a SIMD, in LDS
// and in memory alike), so the kernels are allocated one wavefront per SIMD.  Every wait is bounded besides
// (kSpinMax).
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
template <int NF> struct FlowLanes { static constexpr int n = NF <= 4 ? 4 : 8; };

// The value of slot q's lane, in the lanes of a cell's first quad (4 lanes: a quad permutation; 8 lanes: slots
// 4 and 5 come from the second quad by a mirror of the eight).
template <int NF, int Q> __device__ inline double slot_value(double x) {
  if constexpr (Q < 4) return dpp_move<Q * 0x55>(x);
  else return dpp_move<0x141>(dpp_move<(Q - 4) * 0x55>(x));
}
// acc + x_0 + x_1 .., acc - x_0 - x_1 .. and acc + x_0 y_0 + x_1 y_1 .. (fused) over the slots, in slot order
template <int NF, int Q = 0> __device__ inline void slot_sum(double& acc, double x) {
  if constexpr (Q < NF) {
    acc += slot_value<NF, Q>(x);
    slot_sum<NF, Q + 1>(acc, x);
  }
}
template <int NF, int Q = 0> __device__ inline void slot_fma(double& acc, double x, double y) {
  if constexpr (Q < NF) {
    acc = __builtin_fma(slot_value<NF, Q>(x), slot_value<NF, Q>(y), acc);
    slot_fma<NF, Q + 1>(acc, x, y);
  }
}
template <int NF, int Q = 0> __device__ inline void slot_subtract(double& acc, double x) {
  if constexpr (Q < NF) {
    acc -= slot_value<NF, Q>(x);
    slot_subtract<NF, Q + 1>(acc, x);
  }
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

// The sequence of positions is 0, 1, .., m-1, m-2, .., 0, 1, ..: colour c is relaxed on the way up and on the way
// down, the two end colours once per turn.  Relaxations of colour c in a sequence of n positions:
__device__ inline int relaxations(int c, int n, int m) {
  if (m == 1) return n > 0 ? 1 : 0;
  const int period = 2 * (m - 1), full = n / period, t = n % period;
  const bool end = c == 0 || c == m - 1;
  return full * (end ? 1 : 2) + (t > c ? 1 : 0) + (!end && t > period - c ? 1 : 0);
}
// Versions of a neighbour of colour k that the successive relaxations of a cell of colour c read: the first one
// reads `first`; from one way up to the next way down the neighbour is relaxed `up` times, and from a way down
// to the next way up `down` times (an end colour turns round at once: `up` and `down` in every gap).
struct Versions {
  uint32_t v, up, down;
};
__device__ inline Versions versions_of(int c, int k, int m) {
  const uint32_t gap = k == 0 || k == m - 1 ? 1u : 2u;
  Versions x{k < c ? 1u : 0u, k > c ? gap : 0u, k < c ? gap : 0u};
  if (c == 0 || c == m - 1) x.up = x.down = gap;
  return x;
}
__host__ __device__ inline int sequence_length(int m, int pairs) {
  return pairs == 0 ? 0 : m == 1 ? 1 : pairs * 2 * (m - 1) + 1;
}

// Polls of one wait before the kernel gives up (each at least a memory round trip); a wait that long means a
// wavefront is missing, and the flag turns the call into an error.
constexpr uint32_t kSpinMax = 1u << 18;
// Wavefronts of a dataflow launch per compute unit: one per SIMD (16 384 tetrahedra or 8 192 cells of 6 face slots on
// 256 compute units).  Larger meshes keep a launch per colour; their macro stage is 4-7% of an iteration.
constexpr int kFlowWavesPerCu = 4;
// Cache policy of the polls: device scope (the sc1 bit).
constexpr int kSc1 = 16;

// A lane's cell and neighbour
template <int NF> struct FlowLane {
  static constexpr int NL = FlowLanes<NF>::n, CW = 64 / NL;
  int64_t i = 0, nb = kNoFace;  // cell, neighbour through this lane's slot (< 0: none)
  int a = 0, color = -1, nb_color = 0;
  bool valid = false;

  // color = -1 where the wavefront owns no cells
  __device__ void find(const Dev& d, const FlowPlan& pl, int wave) {
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
    if (nb >= 0)
      while (nb_color + 1 < m && nb >= pl.off[nb_color + 1]) ++nb_color;
  }
};

// Lane a of a cell's first quad stores doubles a and a + 4 of the cell's six
template <class Put> __device__ inline void spread(int a, const double* x, Put&& put) {
  double y[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    y[q] = x[q];
    asm("" : "+v"(y[q]));  // in registers: the selects below would otherwise become an indexed load from scratch
  }
  if (a >= 4) return;
  put(a, a == 0 ? y[0] : a == 1 ? y[1] : a == 2 ? y[2] : y[3]);
  if (a < 2) put(a + 4, a == 0 ? y[4] : y[5]);
}

// The sweeps in one workgroup.  inc: the cells' increments in LDS, [nc][6].  relax(xj, x): one relaxation from the
// neighbour's increment xj to the cell's x.
template <int NF, class Relax>
__device__ inline void sweeps_in_lds(const FlowLane<NF>& L, int64_t nc, int m, int steps, double* inc, double* x,
                                     Relax&& relax) {
  for (int64_t k = threadIdx.x; k < 6 * nc; k += blockDim.x) inc[k] = 0.0;
  __syncthreads();
  int c = 0, up = 1;
  for (int p = 0; p < steps; ++p) {
    if (c == L.color) {
      double xj[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) xj[q] = L.nb >= 0 ? inc[6 * L.nb + q] : 0.0;
      relax(xj, x);
      if (L.valid) spread(L.a, x, [&](int q, double v) { inc[6 * L.i + q] = v; });
    }
    __syncthreads();
    if (m > 1) {
      if (c == m - 1) up = -1;
      if (c == 0) up = 1;
      c += up;
    }
  }
}

// The sweeps as a dataflow over workgroups of one wavefront.  words: the exchange buffer; stage: LDS for the
// lines of the 64 lanes' neighbours.  false: a wait ran out.
template <int NF, class Relax>
__device__ inline bool sweeps_as_flow(const FlowLane<NF>& L, int m, int steps, uint64_t* words, uint64_t* stage,
                                      uint32_t tag0, double* x, Relax&& relax) {
  const int lane = threadIdx.x & 63;
  const int line = (int)(L.nb >= 0 ? L.nb : L.i);
  uint32_t src[8];  // byte offsets of the chunks that this lane loads: of the neighbours of lanes 8k + lane / 8
#pragma unroll
  for (int k = 0; k < 8; ++k)
    src[k] = (uint32_t)__shfl(line, 8 * k + lane / 8, 64) * (uint32_t)(8 * kFlowWords) + 16u * (lane & 7);
  Versions need = L.nb >= 0 ? versions_of(L.color, L.nb_color, m) : Versions{0, 0, 0};
  const int count = relaxations(L.color, steps, m);
  for (int n = 0; n < count; ++n) {
    // the neighbour's increment of version need.v (0: before its first relaxation)
    double xj[6] = {0, 0, 0, 0, 0, 0};
    const uint32_t tag = tag0 + need.v;
    bool ok = need.v == 0u;
    uint32_t spins = 0;
    for (uint64_t wanted = __ballot(!ok); wanted != 0; wanted = __ballot(!ok)) {
      if (++spins > kSpinMax) return false;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if ((wanted >> (8 * k)) & 0xffu)
          __builtin_amdgcn_global_load_lds(
              (__attribute__((address_space(1))) const void*)(reinterpret_cast<const char*>(words) + src[k]),
              (__attribute__((address_space(3))) void*)(stage + 8 * kFlowWords * k), 16, 0, kSc1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const uint64_t* r = stage + kFlowWords * lane;
      uint32_t miss = 0;
      uint64_t lo[6], hi[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        lo[c] = r[2 * (c ^ (line & 7))];
        hi[c] = r[2 * (c ^ (line & 7)) + 1];
        miss |= ((uint32_t)(lo[c] >> 32) ^ tag) | ((uint32_t)(hi[c] >> 32) ^ tag);
      }
      asm volatile("" ::: "memory");
      if (!ok && miss == 0u) {
        ok = true;
#pragma unroll
        for (int c = 0; c < 6; ++c) xj[c] = __builtin_bit_cast(double, (uint64_t)(uint32_t)lo[c] | (hi[c] << 32));
      }
    }
    relax(xj, x);
    if (L.valid)
      spread(L.a, x, [&](int c, double v) {
        const uint64_t t = (uint64_t)(tag0 + (uint32_t)n + 1u) << 32, u = __builtin_bit_cast(uint64_t, v);
        uint64_t* dst = words + kFlowWords * L.i + 2 * (c ^ ((int)L.i & 7));
        __hip_atomic_store(dst, t | (uint32_t)u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(dst + 1, t | (u >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      });
    need.v += n & 1 ? need.down : need.up;
  }
  return true;
}

// Both kernels: one workgroup of kFlowLocal threads (Local), else one wavefront a workgroup and a SIMD
#define CIS_FLOW_KERNEL __global__ __launch_bounds__(Local ? kFlowLocal : 64) \
    __attribute__((amdgpu_waves_per_eu(Local ? 4 : 1, Local ? 4 : 1)))

// Step 4 (Eqs. 38-43): macro flux per cell (Eq. 37), spectral radii r_ij (Eq. 41), diagonal and right-hand side
// of Eq. 43, the sweeps (matrix-free increment G(W_j + dW_j) - G(W_j)) and the predicted state with its
// equilibrium coefficients (q~ = q^n).
template <int NF, bool Local>
CIS_FLOW_KERNEL void k_macro_flow(Dev d, const double* W, const double* q,
                                                                            Work w, FlowPlan pl, uint64_t* words,
                                                                            uint32_t tag0, int steps) {
  extern __shared__ __align__(16) uint64_t lds_words[];
  FlowLane<NF> L;
  L.find(d, pl, Local ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : (int)blockIdx.x);
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
  D += inv_dt_cell(d, geo[2]);
  const double iD = 1.0 / D, D5 = D + 1.0 / (g.Z * tau);
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    double F = 0.0;
    slot_fma<NF>(F, fsum[m], iV);
    if (L.valid && L.a == 0) w.Fmac[6 * i + m] = F;
    res[m] = -F;
  }
  res[5] += fma_(pa.rho * g.R, pa.T, -Wi[5]) / (g.Z * tau);
  double dW[6] = {0, 0, 0, 0, 0, 0};
  auto relax = [&](const double* dWj, double* x) {
    double term[6] = {0, 0, 0, 0, 0, 0};
    if (L.nb >= 0) {
      double Wp[6], dG[6];
#pragma unroll
      for (int m = 0; m < 6; ++m) Wp[m] = Wj[m] + dWj[m];
      macro_flux_increment(Wp, nx, ny, nz, G0, dG);
#pragma unroll
      for (int m = 0; m < 6; ++m) term[m] = hav * fma_(-r, dWj[m], dG[m]);
    }
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      double acc = res[m];
      slot_subtract<NF>(acc, term[m]);
      x[m] = m == 5 ? acc / D5 : acc * iD;
    }
  };
  if constexpr (Local) {
    sweeps_in_lds<NF>(L, d.nc, pl.m, steps, reinterpret_cast<double*>(lds_words), dW, relax);
  } else if (!sweeps_as_flow<NF>(L, pl.m, steps, words, lds_words, tag0, dW, relax)) {
    atomicOr(&w.flag[0], kFlowStuck);
    return;
  }
  if (!L.valid || L.a != 0) return;
  // W~ = W^n + dW~; predicted equilibrium coefficients with q~ = q^n
  double Wt[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    w.dW[6 * i + m] = dW[m];
    Wt[m] = Wi[m] + dW[m];
    w.Wt[6 * i + m] = Wt[m];
  }
  const Prim p = macro_prim(Wt, g.R);
  if (!(p.rho > 0.0) || !(p.T > 0.0) || !(p.Ttr > 0.0) || !(p.Trot > 0.0)) atomicOr(&w.flag[0], 1);
  double* e = w.eq + ER * i;
  eq_coeffs(p, q + 6 * i, g, e);
  const double taut = macro_tau(p, g);
  e[7] = taut;
  w.mbase[i] = inv_dt_cell(d, geo[2]) + 1.0 / taut;
}

// Mac^T u = t: row i couples the neighbours j through Mac_ji^T = -(A_f/V_j)(dG_n/dW (W_i)^T + r_f I)/2 with n out
// of cell i (the flux Jacobian is odd in n and r_f is the same from both sides); Mac is the steady macro system,
// D_i = sum_f (A_f/V_i) r_f / 2 (+ 1/(Z tau_i) for rho E_rot).
template <int NF, bool Local>
CIS_FLOW_KERNEL void k_adj_macro_flow(Dev d, const double* W,
                                                                                const double* t, double* u,
                                                                                int32_t* flag, FlowPlan pl,
                                                                                uint64_t* words, uint32_t tag0,
                                                                                int steps) {
  extern __shared__ __align__(16) uint64_t lds_words[];
  FlowLane<NF> L;
  L.find(d, pl, Local ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : (int)blockIdx.x);
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
  const double iD = 1.0 / D, iD5 = 1.0 / (D + 1.0 / (g.Z * tau));
  double ti[6], x[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int m = 0; m < 6; ++m) ti[m] = t[6 * i + m];
  auto relax = [&](const double* uj, double* ui) {
    double term[6] = {0, 0, 0, 0, 0, 0};
    if (L.nb >= 0) {
      double gj[6];
      euler_flux_vjp(Wi, nx, ny, nz, uj, gj);
#pragma unroll
      for (int m = 0; m < 6; ++m) term[m] = half_av * (gj[m] + r * uj[m]);
    }
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      double acc = ti[m];
      slot_sum<NF>(acc, term[m]);
      ui[m] = acc * (m == 5 ? iD5 : iD);
    }
  };
  if constexpr (Local) {
    sweeps_in_lds<NF>(L, d.nc, pl.m, steps, reinterpret_cast<double*>(lds_words), x, relax);
  } else if (!sweeps_as_flow<NF>(L, pl.m, steps, words, lds_words, tag0, x, relax)) {
    atomicOr(flag, kFlowStuck);
    return;
  }
  if (!L.valid || L.a != 0) return;
#pragma unroll
  for (int m = 0; m < 6; ++m) u[6 * i + m] = x[m];
}

constexpr size_t kStageBytes = 64 * sizeof(uint64_t) * kFlowWords;

// Whether `waves` workgroups of the kernel are within the launch's bound and resident at once.
bool all_resident(const void* kernel, int waves) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, 64, kStageBytes) != hipSuccess) return false;
  return waves <= cus * std::min(per, kFlowWavesPerCu);
}

template <int NF> hipError_t run(bool adjoint, const FlowPlan& pl, int64_t nc, void** args, hipStream_t st) {
  const void* kl = adjoint ? (const void*)k_adj_macro_flow<NF, true> : (const void*)k_macro_flow<NF, true>;
  const void* kg = adjoint ? (const void*)k_adj_macro_flow<NF, false> : (const void*)k_macro_flow<NF, false>;
  if (pl.local)
    return hipLaunchKernel(kl, dim3(1), dim3(kFlowLocal), args, 6 * sizeof(double) * (size_t)nc, st);
  return hipLaunchCooperativeKernel(kg, dim3((unsigned)pl.wave0[pl.m]), dim3(64), args, (unsigned)kStageBytes, st);
}

// The tags of one launch: versions 1 .. of this call follow the last call's, so no word left behind by an earlier
// call carries an awaited tag.
uint32_t take_tags(Flow& f, int steps) {
  const uint32_t t0 = f.tag;
  f.tag += (uint32_t)steps + 1u;
  return t0;
}

}  // namespace

FlowPlan flow_plan(const Dev& d, const int64_t* color_off, int64_t n_colors) {
  FlowPlan pl;
  const int cw = 64 / (d.mf == 4 ? FlowLanes<4>::n : FlowLanes<kMaxFaces>::n);
  int m = 0, waves = 0;
  for (int64_t c = 0; c < n_colors; ++c) {
    const int64_t n = color_off[c + 1] - color_off[c];
    if (n <= 0) continue;
    if (m == kFlowColors || n > (int64_t)1 << 24) return FlowPlan();
    pl.off[m] = (int32_t)color_off[c];
    pl.n[m] = (int32_t)n;
    pl.wave0[m] = waves;
    waves += (int)((n + cw - 1) / cw);
    pl.wave0[++m] = waves;
  }
  if (m == 0) return FlowPlan();
  pl.local = waves <= kFlowLocal / 64;
  if (!pl.local) {
    const bool tet = d.mf == 4;
    const void* k0 = tet ? (const void*)k_macro_flow<4, false> : (const void*)k_macro_flow<kMaxFaces, false>;
    const void* k1 = tet ? (const void*)k_adj_macro_flow<4, false> : (const void*)k_adj_macro_flow<kMaxFaces, false>;
    if (!all_resident(k0, waves) || !all_resident(k1, waves)) return FlowPlan();
  }
  pl.m = m;
  return pl;
}

hipError_t launch_macro_flow(const Dev& d, const Bufs& b, const Work& w, Flow& f, int n_macro, hipStream_t st) {
  int steps = sequence_length(f.plan.m, n_macro);
  uint32_t tag0 = take_tags(f, steps);
  Dev dd = d;
  const double *W = b.W, *q = b.q;
  Work ww = w;
  void* args[] = {&dd, &W, &q, &ww, &f.plan, &f.words, &tag0, &steps};
  return d.mf == 4 ? run<4>(false, f.plan, d.nc, args, st) : run<kMaxFaces>(false, f.plan, d.nc, args, st);
}

hipError_t launch_adj_macro_flow(const Dev& d, const Bufs& b, Flow& f, const double* t, double* u, int n_pairs,
                                 int32_t* flag, hipStream_t st) {
  int steps = sequence_length(f.plan.m, n_pairs);
  uint32_t tag0 = take_tags(f, steps);
  Dev dd = d;
  const double* W = b.W;
  void* args[] = {&dd, &W, &t, &u, &flag, &f.plan, &f.words, &tag0, &steps};
  return d.mf == 4 ? run<4>(true, f.plan, d.nc, args, st) : run<kMaxFaces>(true, f.plan, d.nc, args, st);
}

}  // namespace cis
