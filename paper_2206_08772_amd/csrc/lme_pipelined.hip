// Shape functions (Sec. 2.3) of large bodies in float64 arithmetic: the same
// Newton solve as lme.hip's kernel (its reading stands there), laid out so that
// memory and arithmetic overlap.
//
// A group of kG = 4 lanes (lanes c, c + 16, c + 32, c + 48 of a wave) works on
// one MP; each keeps up to kPpl = 10 of the MP's pairs in registers (offset
// d = x_p - x_I and weight e; pair 4k + l of the row in slot k of member l).  The
// supports of the lattice-like bodies hold 20-33 nodes (radius 1.86 h), up to 40
// with a list skin of 0.1 h; MPs with more than 40 pairs are left to a second
// pass that re-reads their pairs from memory at every evaluation.
//
// Measured on a rod of 1.13M MPs, shape functions with the fused assembly from the
// last multiplier: 618 us against 691 with lme.hip's kernel at 27 pairs per MP, 689
// against 823 at 32 (a list skin of 0.1 h), 755 against 1366 at 35, where one MP in
// four has more than the 36 pairs that kernel holds (lme.hip's dispatch has the sizes
// and lengths where it is the slower one).  No unit is full: the VALU is 39 % busy, the
// L1s' data path 80 %, and the waves wait a third of their time, two per SIMD, for
// the chain of one MP's Newton steps.  14.7 write requests per MP leave for the L2
// (34.8 from lme.hip's kernel with float32 grad N).
//
//  - Workgroups are persistent and their rounds (64 MPs) pipelined: vector
//    memory operations complete in order, so a wait for loads issued after a
//    round's stores waits for the stores too.  Everything a round starts from
//    (node positions, multiplier) is therefore requested before the stores of
//    the round before it, which then drain during the next Newton solve.
//  - The stores leave as whole lines: a wave's 16 rows are one run of the pair
//    arrays, put in order in LDS and written 16 bytes per lane with
//    bounds-checked buffer stores, whose unused lanes are dropped without a
//    branch (a branch would hide the number of stores in flight from the
//    compiler, and it would wait for all of them).
//  - No branch per pair: the first 24 pairs of a row are evaluated together, so
//    that the exponentials' dependent chains overlap.
//  - A step that changes no exponent by more than 1/32 multiplies the weights
//    by the degree-7 Taylor polynomial of exp (truncation below 2.3e-17) instead
//    of evaluating them anew, and needs no line search: with the cumulants
//    kappa_k of delta . d, kappa_1 = -kappa_2 for a Newton step, the change of
//    log Z, sum_k kappa_k / k!, is below -0.47 kappa_2, far past the Armijo bound
//    1e-4 slope = -1e-4 kappa_2.  At most kSmallSteps such steps follow one
//    another (roundings add up); every other evaluation forms the weights anew.
//  - The sums over a group run on the matrix cores.
#include <type_traits>

#include "launch.h"
#include "lme.h"
#include "otm_common.h"

namespace otm {

__constant__ double kExpTaylorPipelined[13] = OTM_EXP_TAYLOR;

namespace {

OTM_DEV double lme_exp(double x) { return otm::lme_exp(kExpTaylorPipelined, x); }

constexpr int kG = 4;              // lanes per MP
constexpr int kPpl = 10;           // pairs per lane
constexpr int kRowMax = kG * kPpl; // pairs of a row kept in registers
constexpr int kWaveMps = kWave / kG;
constexpr int kPerRound = 256 / kG;
// staging of one wave's rows: its pairs, one more for a start at an odd entry,
// and a place for what unused slots write
constexpr int kStage = kWaveMps * kRowMax;
constexpr int kPieces = kStage / (2 * kWave);  // two entries per lane each
constexpr double kLeft = -1.0;     // N of a row left to be solved from memory

// Node coordinates: the packed (x, y, z, 0) records the step keeps in its
// workspace (PACKED: one line per node), or SoA arrays.
template <bool PACKED>
struct NodeSrc {
  const double* x;       // [3][n] (PACKED: unused)
  const double4* packed; // record 2 I = (x, y, z, du_x)
  int64_t n;
  OTM_DEV void get(int32_t I, double& a, double& b, double& c) const {
    if constexpr (PACKED) {
      const double4 v = packed[2 * (int64_t)I];
      a = v.x; b = v.y; c = v.z;
    } else {
      a = x[I]; b = x[n + I]; c = x[2 * n + I];
    }
  }
};

// exp(t) for |t| <= kSmallStep.
constexpr double kSmallStep = 1.0 / 32.0;
constexpr int kSmallSteps = 8;  // in a row
OTM_DEV double lme_exp_small(double t) {
  double p = kExpTaylorPipelined[7];
#pragma unroll
  for (int i = 6; i >= 0; --i) p = fma(p, t, kExpTaylorPipelined[i]);
  return p;
}

// Sum over the four lanes of an MP's group (lanes c, c + 16, c + 32, c + 48 of
// the wave), in each of them: the product of a 4x4 block of ones with the four
// lanes' values on the matrix cores, which leaves the vector ALU to the other
// waves (one instruction for six).  Only where the whole wave is active: the
// matrix cores write every lane's result, also those of lanes that a branch or
// a loop has switched off, whose values the same registers may still hold.
OTM_DEV double rows_sum(double v) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, v, 0.0, 0, 0, 0);
}
// The same where groups have parted (each group's lanes stay together).
OTM_DEV double rows_sum_parted(double v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}
OTM_DEV double rows_max(double v) {
  v = fmax(v, __shfl_xor(v, 16));
  return fmax(v, __shfl_xor(v, 32));
}

// The sums of one evaluation (Z, r, S = sum e d d^T as xx yy zz xy yz xz).
struct Sums {
  double Z, r0, r1, r2, s0, s1, s2, s3, s4, s5;
  OTM_DEV void clear() { Z = r0 = r1 = r2 = s0 = s1 = s2 = s3 = s4 = s5 = 0.0; }
  OTM_DEV void add(double e, double dx, double dy, double dz) {
    Z += e;
    r0 += e * dx; r1 += e * dy; r2 += e * dz;
    s0 += e * dx * dx; s1 += e * dy * dy; s2 += e * dz * dz;
    s3 += e * dx * dy; s4 += e * dy * dz; s5 += e * dx * dz;
  }
  OTM_DEV void reduce() {  // the whole wave's groups together
    Z = rows_sum(Z);
    r0 = rows_sum(r0); r1 = rows_sum(r1); r2 = rows_sum(r2);
    s0 = rows_sum(s0); s1 = rows_sum(s1); s2 = rows_sum(s2);
    s3 = rows_sum(s3); s4 = rows_sum(s4); s5 = rows_sum(s5);
  }
  OTM_DEV void reduce_parted() {
    Z = rows_sum_parted(Z);
    r0 = rows_sum_parted(r0); r1 = rows_sum_parted(r1); r2 = rows_sum_parted(r2);
    s0 = rows_sum_parted(s0); s1 = rows_sum_parted(s1); s2 = rows_sum_parted(s2);
    s3 = rows_sum_parted(s3); s4 = rows_sum_parted(s4); s5 = rows_sum_parted(s5);
  }
};

// What the iteration takes from the sums: residual r and J = S / Z - r r^T.
struct Eval {
  double iz;
  double r[3];
  double J[6];  // xx yy zz xy yz xz
  OTM_DEV void from(const Sums& s) {
    iz = 1.0 / s.Z;
    r[0] = s.r0 * iz; r[1] = s.r1 * iz; r[2] = s.r2 * iz;
    J[0] = s.s0 * iz - r[0] * r[0];
    J[1] = s.s1 * iz - r[1] * r[1];
    J[2] = s.s2 * iz - r[2] * r[2];
    J[3] = s.s3 * iz - r[0] * r[1];
    J[4] = s.s4 * iz - r[1] * r[2];
    J[5] = s.s5 * iz - r[0] * r[2];
  }
};

// Newton step of an evaluation with J^{-1}; false if J is not safely positive
// definite (the multiplier ran away).
OTM_DEV bool newton_step(const Eval& ev, const double (&Mi)[6], double det, double (&delta)[3]) {
  const double tr = ev.J[0] + ev.J[1] + ev.J[2];
  if (!(det > 1e-30 * tr * tr * tr) || !isfinite(det)) return false;
  sym_mul_vec(Mi, ev.r, delta);
  delta[0] = -delta[0]; delta[1] = -delta[1]; delta[2] = -delta[2];
  return true;
}

OTM_DEV void wave_order() {
  // the wave's lanes read each other's LDS writes after this point
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Which slots a wave runs (slot k of a lane holds a pair if k kG < lim; the
// others are masked by weights of 0).  The first six always run, together, so
// that their dependent chains (the exponentials' above all) overlap; the ones
// past 24 and past 32 pairs only where a row of the wave has them.  The
// choices are the wave's, so that no lane is ever switched off: the matrix
// cores sum over all of them.
struct Slots {
  int lim;
  bool past6, past8;
  OTM_DEV explicit Slots(int l) : lim(l) {
    static_assert(kPpl == 10, "slots in groups of 6, 2 and 2");
    past6 = __ballot(l > 6 * kG) != 0;
    past8 = __ballot(l > 8 * kG) != 0;
  }
  OTM_DEV bool has(int k) const { return k * kG < lim; }
  template <class F>
  OTM_DEV void each(F&& f) const {
    f(0); f(1); f(2); f(3); f(4); f(5);
    if (past6) { f(6); f(7); }
    if (past8) { f(8); f(9); }
  }
};

// Float64 atomic add to device memory (never a generic-address one, whose
// completion order the compiler cannot count on).
OTM_DEV void global_add(double* p, double v) {
  __builtin_amdgcn_global_atomic_fadd_f64((__attribute__((address_space(1))) double*)p, v);
}

// What happens to each finished pair besides storing N and grad N: a sink.  For
// rows in registers it is first shown the lane's node ids (claim) and then, once
// the solve is done, the row (add_row) with its MP (Mp::load, waited for in
// ready); a row re-read from memory shows its pairs one by one, by their place
// in the lists (add).  flush ends a span of rounds.

struct NoTable {};
struct NoSink {
  struct In {};
  using Table = NoTable;
  static constexpr bool kTable = false;
  struct Mp {
    OTM_DEV void load(const In&, int64_t, int64_t) {}
    OTM_DEV void ready() const {}
  };
  OTM_DEV void setup(Table&) {}
  OTM_DEV void claim(const int32_t (&)[kPpl], const int32_t*, uint16_t*, const Slots&, int, int) {}
  OTM_DEV void add_row(const In&, const Mp&, const Slots&, int64_t, const double (&)[kPpl],
                       const double (&)[kPpl][3], int) {}
  OTM_DEV void add(const In&, const Mp&, int64_t, double, const double*) {}
  OTM_DEV void flush(const In&, int) {}
};

// An MP's mass, volume and stress.
struct MpForce {
  double mp, vd;
  double s0, s1, s2, s3, s4, s5;
  OTM_DEV void load(const double* mass, const double* vol, const double* sigma, int64_t n_mp,
                    int64_t p) {
    mp = mass[p];
    vd = vol[p];
    s0 = sigma[p]; s1 = sigma[n_mp + p]; s2 = sigma[2 * n_mp + p];
    s3 = sigma[3 * n_mp + p]; s4 = sigma[4 * n_mp + p]; s5 = sigma[5 * n_mp + p];
  }
  OTM_DEV void ready() const {
    hold(mp); hold(vd);
    hold(s0); hold(s1); hold(s2); hold(s3); hold(s4); hold(s5);
  }
};

// Fused nodal assembly (nodal mass and residual equations, Sec. 2.1): the
// pair's m and f contributions, with the same arithmetic as the standalone
// assembly kernel, go into the workgroup's node table.  With conduction (HEAT)
// the table also sums N m_p T_p and v_p q_p . grad N.
// The table slots of the lane's nodes are claimed before the Newton solve, all
// probes in flight together; the sums then need no LDS round trip.
template <bool HEAT>
struct AsmSink {
  static constexpr int V = HEAT ? 6 : 4;
  struct In {
    AsmIn a;
    const int32_t* idx;
  };
  struct Table {
    NodeTableV<V> nodes;
    uint16_t slots[4 * kPpl * kWave];  // the waves' table slots (0xFFFF: none)
  };
  static constexpr bool kTable = true;
  struct Mp : MpForce {
    double T, q0, q1, q2;
    OTM_DEV void load(const In& in, int64_t n_mp, int64_t p) {
      MpForce::load(in.a.mass, in.a.vol, (const double*)in.a.sigma, n_mp, p);
      if constexpr (HEAT) {
        T = in.a.T[p];
        q0 = in.a.q[p]; q1 = in.a.q[n_mp + p]; q2 = in.a.q[2 * n_mp + p];
      }
    }
    OTM_DEV void ready() const {
      MpForce::ready();
      if constexpr (HEAT) { hold(T); hold(q0); hold(q1); hold(q2); }
    }
  };
  NodeTableV<V>* t;
  uint16_t* slots;
  OTM_DEV void setup(Table& table) {
    t = &table.nodes;
    slots = table.slots;
  }
  OTM_DEV static NodeDst<V> dst(const In& in) {
    NodeDst<V> d;
    d.d[0] = in.a.m;
    d.d[1] = in.a.f;
    d.d[2] = in.a.f + in.a.n_nodes;
    d.d[3] = in.a.f + 2 * in.a.n_nodes;
    if constexpr (HEAT) {
      d.d[4] = in.a.heat;
      d.d[5] = in.a.heat + in.a.n_nodes;
    }
    return d;
  }
  // Table slots of the wave's nodes.  ids (LDS) holds slot k's node of lane l at
  // k kWave + l, I those of this lane.  A node's places are the four of its
  // bucket, which one 16-byte read looks through (lanes that read one bucket
  // share the read, where compare-and-swaps on it would queue), and then the
  // following ones.  Nodes not seen in their bucket, new ones mostly, are
  // gathered from the whole wave into a queue (over the N stage's later part)
  // and claimed by compare-and-swap, 64 at a time.
  OTM_DEV void claim(const int32_t (&I)[kPpl], const int32_t* ids, uint16_t* queue,
                     const Slots& sl, int wave, int wl) {
    uint16_t* const to = slots + wave * (kPpl * kWave);
    int n = 0;
    // half of the slots at a time: their buckets are all read before one is used
    auto half = [&](auto first) {
      constexpr int k0 = decltype(first)::value, NB = kPpl / 2;
      int32_t b[NB];
      int4 key[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        b[j] = table_hash(I[k0 + j]) & ~3;
        key[j] = *reinterpret_cast<const int4*>(&t->keys[b[j]]);
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int k = k0 + j;
        int32_t at = -1;
        at = key[j].x == I[k] ? b[j] : at;
        at = key[j].y == I[k] ? b[j] + 1 : at;
        at = key[j].z == I[k] ? b[j] + 2 : at;
        at = key[j].w == I[k] ? b[j] + 3 : at;
        to[k * kWave + wl] = (uint16_t)at;
        const bool miss = at < 0 && sl.has(k);
        const uint64_t m = __ballot(miss);
        const int pos = n + (int)__builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        queue[miss ? pos : kPpl * kWave] = (uint16_t)(k * kWave + wl);
        n += __builtin_popcountll(m);
      }
    };
    half(std::integral_constant<int, 0>{});
    half(std::integral_constant<int, kPpl / 2>{});
    wave_order();
    for (int i = wl; i < n; i += kWave) {
      const int at = queue[i];
      const int32_t node = ids[at];
      to[at] = (uint16_t)table_probe<V>(*t, node, table_hash(node) & ~3);
    }
    wave_order();
  }
  OTM_DEV static void values(const Mp& m, double Nq, const double* g, double (&c)[V]) {
    c[0] = Nq * m.mp;
    pair_force<double>(m.vd, m.s0, m.s1, m.s2, m.s3, m.s4, m.s5, g[0], g[1], g[2], c[1], c[2], c[3]);
    if constexpr (HEAT) {
      c[4] = c[0] * m.T;
      c[5] = m.vd * ((m.q0 * g[0] + m.q1 * g[1]) + m.q2 * g[2]);
    }
  }
  OTM_DEV void add_row(const In& in, const Mp& m, const Slots& sl, int64_t q,
                       const double (&N)[kPpl], const double (&g)[kPpl][3], int tid) {
    static_assert(kTableSlots < 0xFFFF, "16-bit slots");
    const uint16_t* from = slots + tid / kWave * (kPpl * kWave) + tid % kWave;
    uint32_t slot[kPpl];
#pragma unroll
    for (int k = 0; k < kPpl; ++k) slot[k] = from[k * kWave];
    sl.each([&](int k) {
      double c[V];
      values(m, N[k], g[k], c);
      if (sl.has(k)) {
        if (slot[k] != 0xFFFFu) {
#pragma unroll
          for (int v = 0; v < V; ++v) atomicAdd(&t->vals[v][slot[k]], c[v]);
        } else {  // no slot (crowded table): straight to memory
          const NodeDst<V> to = dst(in);
          const int32_t I = in.idx[q + k * kG];
#pragma unroll
          for (int v = 0; v < V; ++v) global_add(to.d[v] + I, c[v]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  OTM_DEV void add(const In& in, const Mp& m, int64_t q, double Nq, const double* g) {
    double c[V];
    values(m, Nq, g, c);
    table_insert<V>(*t, in.idx[q], c, dst(in));
  }
  OTM_DEV void flush(const In& in, int tid) { table_flush(*t, tid, 256, dst(in)); }
};

// Fused contribution store of the deterministic assembly: the pair's four
// contributions (the standalone contribution kernel's arithmetic) go to its
// place in the node-sorted order, where each node later sums them in order.
struct SegSink {
  using In = SegIn;
  using Table = NoTable;
  static constexpr bool kTable = false;
  struct Mp : MpForce {
    OTM_DEV void load(const In& in, int64_t n_mp, int64_t p) {
      MpForce::load(in.mass, in.vol, (const double*)in.sigma, n_mp, p);
    }
  };
  OTM_DEV void setup(Table&) {}
  OTM_DEV void claim(const int32_t (&)[kPpl], const int32_t*, uint16_t*, const Slots&, int, int) {}
  OTM_DEV void add_row(const In& in, const Mp& m, const Slots& sl, int64_t q,
                       const double (&N)[kPpl], const double (&g)[kPpl][3], int) {
    sl.each([&](int k) {
      if (sl.has(k)) add(in, m, q + k * kG, N[k], g[k]);
    });
  }
  OTM_DEV void add(const In& in, const Mp& m, int64_t q, double Nq, const double* g) {
    double c1, c2, c3;
    pair_force<double>(m.vd, m.s0, m.s1, m.s2, m.s3, m.s4, m.s5, g[0], g[1], g[2], c1, c2, c3);
    in.contrib[in.pos_of[q]] = make_double4(Nq * m.mp, c1, c2, c3);
  }
  OTM_DEV void flush(const In&, int) {}
};

// Everything an MP's solve reads and writes.
template <bool PACKED>
struct LmeArgs {
  NodeSrc<PACKED> ns;
  int64_t n_mp;
  const double* __restrict__ xp;
  const int64_t* __restrict__ offsets;
  const int32_t* __restrict__ idx;
  int64_t cap;
  double beta, tol;
  int max_iter;
  double* __restrict__ lam;
  double* __restrict__ N;
  double* __restrict__ dN;
  otm_diag* diag;
};

// Newton iteration of the wave's rows in registers (every lane takes part; rows
// without pairs, and done ones, go along with steps of 0).  The multiplier is
// advanced in place, e ends as the weights (0 past the row) and Mi as J^{-1}
// at it.  Solve::Leave: not a row (live false), or sums that are not numbers;
// the row is to be solved from memory.
enum class Solve { Converged, Failed, Leave };

OTM_DEV Solve lme_solve(const double (&d)[kPpl][3], double (&e)[kPpl], const Slots& sl, bool live,
                        double beta, double tol, int max_iter, double (&lam)[3], double& iz,
                        double (&Mi)[6]) {
  // beta times a bound of the row's |d|^2 (the sum of its lanes' largest; unused
  // slots repeat its first pair), in float32: it is only compared with
  double r2 = 0.0;
#pragma unroll
  for (int k = 0; k < kPpl; ++k)
    r2 = fmax(r2, fma(d[k][0], d[k][0], fma(d[k][1], d[k][1], d[k][2] * d[k][2])));
  const float br2 = fmaxf((float)(beta * rows_sum(r2)) * 1.00001f, 1e-30f);
  Sums s;
  double shift;
  // the weights at lam, formed from the prior, their exponents shifted by the
  // row's largest (an unused slot's is its first pair's)
  auto anew = [&]() {
    double top = -INFINITY, b = beta;
    __asm__ volatile("" : "+s"(b));  // (kept from holding the priors in registers)
    sl.each([&](int k) {
      e[k] = (lam[0] - b * d[k][0]) * d[k][0] + (lam[1] - b * d[k][1]) * d[k][1] +
             (lam[2] - b * d[k][2]) * d[k][2];
      top = fmax(top, e[k]);
    });
    shift = rows_max(top);
    s.clear();
    sl.each([&](int k) {
      const double w = lme_exp(e[k] - shift);
      e[k] = sl.has(k) ? w : 0.0;
      s.add(e[k], d[k][0], d[k][1], d[k][2]);
    });
    s.reduce();
  };
  Solve res = Solve::Leave;
  const double tol2 = tol * tol;
  double a[3] = {0.0, 0.0, 0.0}, from = 0.0, drop = 0.0;
  bool open = false;
  for (int it = 0;;) {
    // trials at 1, 1/2, 1/4, ... of the steps that are not small (at first, the
    // start), the weights formed anew at each: a rejected trial can be so far
    // off that weights which matter vanish at it, and no factor brings them back
    for (int h = 0;; ++h) {
      anew();
      open = open && !(log(s.Z) + shift <= from + drop);
      if (h == 30 || __ballot(open) == 0) break;
      const double back = !open ? 0.0 : (h == 0 ? -0.5 : 0.5);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        a[c] *= back;
        lam[c] += a[c];
      }
      drop *= 0.5;
    }
    // Newton steps from the weights at lam, up to one that is not small
    for (int since = 0;; ++since, ++it) {
      Eval ev;
      ev.from(s);
      iz = ev.iz;
      double det;
      sym_inv(ev.J, Mi, det);
      const bool step = newton_step(ev, Mi, det, a);
      if (live) {
        if (ev.r[0] * ev.r[0] + ev.r[1] * ev.r[1] + ev.r[2] * ev.r[2] <= tol2)
          res = Solve::Converged;
        else if (s.Z < INFINITY && (it >= max_iter || !step))
          res = Solve::Failed;
        else
          live = s.Z < INFINITY;
        live = live && res == Solve::Leave;
      }
      if (__ballot(live) == 0) return res;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        a[c] = live ? a[c] : 0.0;
        lam[c] += a[c];
      }
      const double a2 = a[0] * a[0] + a[1] * a[1] + a[2] * a[2];
      open = live && !(a2 * (double)br2 <= kSmallStep * kSmallStep * beta);
      if (__ballot(open) != 0 || since == kSmallSteps) {
        from = log(s.Z) + shift;
        from += 1e-12 * (1.0 + fabs(from));
        drop = 1e-4 * (ev.r[0] * a[0] + ev.r[1] * a[1] + ev.r[2] * a[2]);
        ++it;
        break;
      }
      // the weights moved with the multiplier
      s.clear();
      sl.each([&](int k) {
        e[k] *= lme_exp_small(a[0] * d[k][0] + a[1] * d[k][1] + a[2] * d[k][2]);
        s.add(e[k], d[k][0], d[k][1], d[k][2]);
      });
      s.reduce();
    }
  }
}

// One MP's solve with its pairs re-read from memory at every evaluation, and
// its stores.  The wave's MPs go their own ways in it.
template <bool PACKED, class Sink>
OTM_DEV void lme_uncached(const LmeArgs<PACKED>& a, const typename Sink::In& in, int64_t p,
                          int lane, int64_t off, int K, Sink& sink) {
  const int64_t n_mp = a.n_mp;
  const double px = a.xp[p], py = a.xp[n_mp + p], pz = a.xp[2 * n_mp + p];
  double lam[3] = {a.lam[p], a.lam[n_mp + p], a.lam[2 * n_mp + p]};
  double dx, dy, dz, shift;
  Sums s;
  auto pair = [&](int q) {
    double x, y, z;
    a.ns.get(a.idx[off + q], x, y, z);
    dx = px - x; dy = py - y; dz = pz - z;
    return -a.beta * ((dx * dx + dy * dy) + dz * dz) + (lam[0] * dx + lam[1] * dy + lam[2] * dz);
  };
  auto anew = [&]() {
    double fm = -INFINITY;
    for (int q = lane; q < K; q += kG) fm = fmax(fm, pair(q));
    shift = rows_max(fm);
    s.clear();
    for (int q = lane; q < K; q += kG) {
      const double f = pair(q);
      s.add(lme_exp(f - shift), dx, dy, dz);
    }
    s.reduce_parted();
  };
  const double tol2 = a.tol * a.tol;
  Eval ev;
  double Mi[6], det;
  bool converged = false;
  anew();
  for (int it = 0;; ++it) {
    ev.from(s);
    sym_inv(ev.J, Mi, det);
    if (ev.r[0] * ev.r[0] + ev.r[1] * ev.r[1] + ev.r[2] * ev.r[2] <= tol2) {
      converged = true;
      break;
    }
    double delta[3];
    if (it >= a.max_iter || !newton_step(ev, Mi, det, delta)) break;
    const double slope = ev.r[0] * delta[0] + ev.r[1] * delta[1] + ev.r[2] * delta[2];
    const double lz0 = log(s.Z) + shift, l0[3] = {lam[0], lam[1], lam[2]};
    double t = 1.0;
    for (int h = 0; h < 31; ++h) {
      lam[0] = l0[0] + t * delta[0];
      lam[1] = l0[1] + t * delta[1];
      lam[2] = l0[2] + t * delta[2];
      anew();
      if (log(s.Z) + shift <= lz0 + 1e-4 * t * slope + 1e-12 * (1.0 + fabs(lz0))) break;
      t *= 0.5;
    }
  }
  if (lane == 0) {
    a.lam[p] = lam[0]; a.lam[n_mp + p] = lam[1]; a.lam[2 * n_mp + p] = lam[2];
    if (!converged) diag_fail(a.diag, OTM_ERR_LME_NOCONV, (uint64_t)p);
  }
  typename Sink::Mp mp;
  mp.load(in, n_mp, p);
  for (int q = lane; q < K; q += kG) {
    const double f = pair(q);
    const double Nq = lme_exp(f - shift) * ev.iz;
    const double d3[3] = {dx, dy, dz};
    double g[3];
    sym_mul_vec(Mi, d3, g);
    g[0] *= -Nq; g[1] *= -Nq; g[2] *= -Nq;
    a.N[off + q] = Nq;
    a.dN[off + q] = g[0];
    a.dN[a.cap + off + q] = g[1];
    a.dN[2 * a.cap + off + q] = g[2];
    sink.add(in, mp, off + q, Nq, g);
  }
}

OTM_DEV int64_t first_lane(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Raw buffer over memory from p on (32-bit byte offsets below 2^31; a store at
// kDrop is out of bounds and dropped).
constexpr uint32_t kDrop = 0x80000000u;
OTM_DEV __amdgpu_buffer_rsrc_t buffer_at(void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)0x7FFFFFFF, 0x00020000);
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Writes a wave's run of entries [front, end) (places past the run's
// rounded-down start) of one array from LDS: kPieces stores of two entries
// per lane, then the entries without a partner (an odd start in lane 0, an odd
// end in lane 1).  Every lane and instruction is always issued.
OTM_DEV void store_run(double* base, const double* st, int lane, int front, int end) {
  const __amdgpu_buffer_rsrc_t rs = buffer_at((void*)first_lane((int64_t)base));
#pragma unroll
  for (int i = 0; i < kPieces; ++i) {
    const int e = 2 * (kWave * i + lane);
    const bool full = e >= front && e + 1 < end;
    const int o = full ? e * (int)sizeof(double) : (int)kDrop;
    __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(st + e), rs, o, 0, 0);
  }
  const bool odd = (lane == 0 && front == 1 && front < end) ||
                   (lane == 1 && (end & 1) != 0 && end - 1 >= front && !(front == 1 && end == 1));
  const int e = lane == 0 ? 1 : (end > 0 ? end - 1 : 0);
  const int o = odd ? e * (int)sizeof(double) : (int)kDrop;
  __builtin_amdgcn_raw_buffer_store_b64(*reinterpret_cast<const u32x2*>(st + e), rs, o, 0, 0);
}

// Workgroup barrier that orders LDS only: __syncthreads() would also wait for
// the stores and atomics under way.
OTM_DEV void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One dword per lane from memory to LDS (lane l's at dst + 4 l), and the wait
// for such loads (and all others).
OTM_DEV void load_to_lds(const int32_t* src, int32_t* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
}
OTM_DEV void wait_loads() { __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Shape functions of all MPs, with the sink's part of the assembly.  A fixed
// grid of kLmeBlocks workgroups (two per CU at this kernel's register use)
// each take chunks of `chunk` consecutive MPs (spatially compact) in rounds of
// 64 (a chunk's last round may be partial).  A sink with a node table flushes
// it to memory every kFlushRounds rounds and at the end of each chunk.  The
// round count is the same for every lane of a workgroup, so the barriers
// around a flush are reached by all of them.
constexpr int kLmeBlocks = 512;
constexpr int kFlushRounds = 8;
static_assert(kLmeBlocks % 8 == 0, "the workgroups split evenly over the 8 XCDs");

// Chunk size.  With four or more chunks of 512 MPs per workgroup, 512 (the
// chunks are dealt round-robin); otherwise one contiguous range per
// workgroup, every workgroup busy (smaller chunks would add flushes faster
// than they even out the work).
inline int lme_chunk(int64_t n_mp) {
  const int64_t per_wg = (n_mp + kLmeBlocks - 1) / kLmeBlocks;
  return per_wg >= 4 * 512 ? 512 : (int)per_wg;
}

template <bool PACKED, class Sink>
struct LmeCall {
  LmeArgs<PACKED> a;
  typename Sink::In in;
  PairWindow mine;
  int chunk;
};

// The kernel's argument, read anew wherever this is called: held in scalar
// registers over the whole pass, the pointers would spill them.
template <class T>
OTM_DEV const T& kernel_arg() {
  auto p = (const __attribute__((address_space(4))) T*)__builtin_amdgcn_kernarg_segment_ptr();
  __asm__ volatile("" : "+s"(p));
  return *(const T*)p;
}

template <bool PACKED, class Sink>
__global__ __launch_bounds__(256, 2) void k_lme(LmeCall<PACKED, Sink> call) {
  using Call = LmeCall<PACKED, Sink>;
  __shared__ typename Sink::Table table;
  __shared__ __align__(16) double stage[4][kStage + 2];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t n_mp = call.a.n_mp, pairs = call.a.offsets[n_mp];
  if (!call.mine.holds(pairs)) return;
  const int chunk = call.chunk;
  const int rpc = (chunk + kPerRound - 1) / kPerRound;  // rounds per chunk
  Sink sink;
  sink.setup(table);
  if constexpr (Sink::kTable) {
    table_clear(table.nodes, threadIdx.x, 256);
    __syncthreads();
  }
  double* const st = stage[wave];
  int32_t* const st32 = reinterpret_cast<int32_t*>(st);
  // Each XCD takes a contiguous eighth of the chunks (its workgroups' gathers
  // then share its L2) and deals them round-robin to its workgroups.  With
  // several chunks per workgroup, a workgroup's chunks come from across its
  // XCD's range, so regions of slow MPs (more pairs, more Newton steps) are
  // shared out instead of setting one workgroup's, and the kernel's, end;
  // with one, each workgroup has a contiguous range.
  const int n_chunks = (int)((n_mp + chunk - 1) / chunk);
  const int xcd = blockIdx.x % 8u, wgs = gridDim.x / 8u;
  const int c_hi = (int)((int64_t)n_chunks * (xcd + 1) / 8);
  const bool ok = pairs <= call.a.cap;  // lists were written (capacity)
  // Round k of chunk c, and its first MP.
  struct Place {
    int c, k;
    int64_t mp;
  };
  auto chunk_at = [&](int c) { return Place{c, 0, (int64_t)c * chunk}; };
  auto after = [&](const Place& w) {
    return w.k + 1 == rpc ? chunk_at(w.c + wgs) : Place{w.c, w.k + 1, w.mp + kPerRound};
  };
  auto count = [&](const Place& w) {  // its MPs
    if (!ok || w.c >= c_hi) return 0;
    const int in_chunk = chunk - w.k * kPerRound;
    const int64_t in_all = n_mp - w.mp;
    const int m = in_all < kPerRound ? (int)in_all : kPerRound;
    return in_chunk < m ? in_chunk : m;
  };
  // The pipeline: in the pass of round r the node ids of round r + 1 are
  // requested first (into LDS), and after the Newton solve, before the stores of
  // round r, the node positions of round r + 1 and the row bounds of round r + 2.
  // The first pass has no round of its own (n0 = 0).
  const Place start = chunk_at((int)((int64_t)n_chunks * xcd / 8) + (int)(blockIdx.x / 8u));
  Place w0{0, 0, 0}, w1 = start;
  bool real = false, some_left = false;
  int n0 = 0, n1 = count(w1);        // MPs of the round
  // this group's row: its pairs start rel after `even`, the wave's first
  // entry rounded down to even
  int64_t even0 = 0, even1 = 0;
  int front0 = 0, front1 = 0, rel0 = 0, rel1 = 0, K0 = 0, K1 = 0;
  double x0[kPpl][3] = {}, px = 0.0, py = 0.0, pz = 0.0, lam[3] = {};
  // (loads without a branch, from a place that exists where there is no row: a
  // branch would be followed by a wait for them)
  auto row_of = [&](const Place& w, int mine) {
    const int64_t p = w.mp + mine;
    return p < n_mp ? p : n_mp - 1;
  };
  auto set_row = [&](int64_t off, int64_t end, bool has, int64_t& even, int& front, int& rel,
                     int& K) {
    const int64_t run0 = first_lane(off);
    even = run0 & ~(int64_t)1;
    front = (int)(run0 - even);
    rel = (int)(off - even);
    K = has ? (int)(end - off) : 0;
  };
  {
    const int mine = wave * kWaveMps + threadIdx.x % kWaveMps;
    const int64_t* o = call.a.offsets + row_of(w1, mine);
    set_row(o[0], o[1], mine < n1, even1, front1, rel1, K1);
  }
  for (;;) {
    // (places recomputed in each pass, and after the solve, rather than held in
    // registers)
    int tv, wl, lane, mine;
    auto places = [&]() {
      tv = (int)(wave * kWave + __lane_id());
      __asm__ volatile("" : "+v"(tv));
      wl = tv % kWave;
      lane = wl / kWaveMps;
      mine = tv / kWave * kWaveMps + wl % kWaveMps;
    };
    places();
    const Place w2 = after(w1);
    const int n2 = count(w2);
    const bool fits1 = K1 > 0 && K1 <= kRowMax;
    // node ids of the next round, slot k of the wave's lanes at ids[k]
    const Call& c0 = kernel_arg<Call>();
    const int32_t* ids1 = c0.a.idx + (even1 < c0.a.cap ? even1 : (int64_t)0);
    wave_order();
#pragma unroll
    for (int k = 0; k < kPpl; ++k) {
      const int q = k * kG + lane < K1 ? k * kG + lane : 0;
      load_to_lds(ids1 + (fits1 ? rel1 + q : 0), st32 + k * kWave);
    }

    // this round
    const bool fits = K0 > 0 && K0 <= kRowMax;
    const int lim = fits ? K0 - lane : 0;
    double d[kPpl][3], e[kPpl], iz = 0.0, Mi[6] = {};
#pragma unroll
    for (int k = 0; k < kPpl; ++k) {
      d[k][0] = px - x0[k][0];
      d[k][1] = py - x0[k][1];
      d[k][2] = pz - x0[k][2];
      e[k] = 0.0;
    }
    const Slots sl(lim);
    Solve res = Solve::Leave;
    if (__ballot(fits) != 0)  // (the first pass, and waves of long rows, have none)
      res = lme_solve(d, e, sl, fits, c0.a.beta, c0.a.tol, c0.a.max_iter, lam, iz, Mi);
    places();
    const Call& c1 = kernel_arg<Call>();
    const bool add = res != Solve::Leave;
    if (lane == 0 && add) {
      const int64_t p0 = w0.mp + mine;
      double* to = c1.a.lam + p0;
      to[0] = lam[0]; to[n_mp] = lam[1]; to[2 * n_mp] = lam[2];
      if (res != Solve::Converged) diag_fail(c1.a.diag, OTM_ERR_LME_NOCONV, (uint64_t)p0);
    }
    some_left |= mine < n0 && !add;
    __builtin_amdgcn_sched_barrier(0);
    typename Sink::Mp mp;
    mp.load(c1.in, n_mp, mine < n0 ? w0.mp + mine : 0);
    // N and grad N in place of the weights and offsets (a left row's N are marked)
#pragma unroll
    for (int k = 0; k < kPpl; ++k) {
      if (k >= 8 && !sl.past8) continue;
      const double Nq = e[k] * iz;
      double g[3];
      sym_mul_vec(Mi, d[k], g);
      d[k][0] = g[0] * -Nq; d[k][1] = g[1] * -Nq; d[k][2] = g[2] * -Nq;
      e[k] = add ? Nq : kLeft;
    }
    mp.ready();
    __builtin_amdgcn_sched_barrier(0);
    sink.add_row(c1.in, mp, Slots(add ? lim : 0), even0 + (rel0 + lane), e, d, tv);
    // the wave's run: its rows follow one another in the lists (MPs without a
    // round are the last ones)
    const uint32_t have = (uint32_t)__ballot(mine < n0) & 0xFFFFu;
    const int end0 = have ? __builtin_amdgcn_readlane(rel0 + K0, 31 - __builtin_clz(have)) : 0;
    const bool run = __ballot(K0 > kRowMax) == 0 && end0 <= kStage;
    if (!run && fits) {  // a row is not in registers, or the run is too long: row by row
#pragma unroll
      for (int k = 0; k < kPpl; ++k) {
        const int q = k * kG + lane;
        if (q < K0) {
          const int64_t at = even0 + (rel0 + q);
          c1.a.N[at] = e[k];
          c1.a.dN[at] = d[k][0];
          c1.a.dN[c1.a.cap + at] = d[k][1];
          c1.a.dN[2 * c1.a.cap + at] = d[k][2];
        }
      }
    }
    // the ids (requested before the solve), and the table slots of the next round
    wait_loads();
    int32_t I1[kPpl];
#pragma unroll
    for (int k = 0; k < kPpl; ++k) I1[k] = st32[k * kWave + wl];
    if constexpr (Sink::kTable) {
      if (real && (w0.k + 1 == rpc || (w0.k + 1) % kFlushRounds == 0)) {
        lds_barrier();
        sink.flush(c1.in, tv);
        lds_barrier();
      }
      sink.claim(I1, st32, reinterpret_cast<uint16_t*>(st32 + kPpl * kWave),
                 Slots(fits1 ? K1 - lane : 0), (int)wave, wl);
    }
    // N to the stage (its registers are free then), the next round's positions
    // and multiplier and the row bounds requested, and the stores
    const int staged = run ? K0 - lane : 0;
    auto put = [&](auto* to, auto get) {
      using T = std::remove_pointer_t<decltype(to)>;
      int at = rel0 + lane;  // (kept from sharing ten places between the four arrays)
      __asm__ volatile("" : "+v"(at));
      wave_order();
#pragma unroll
      for (int k = 0; k < kPpl; ++k) {
        if (k >= 8 && !sl.past8) continue;
        to[k * kG < staged ? at + k * kG : kStage] = (T)get(k);
      }
      wave_order();
    };
    put(st, [&](int k) { return e[k]; });
    const Call& c2 = kernel_arg<Call>();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kPpl; ++k) c2.a.ns.get(fits1 ? I1[k] : 0, x0[k][0], x0[k][1], x0[k][2]);
    const int64_t pn = row_of(w1, mine);
    const double *nxp = c2.a.xp + pn, *nlam = c2.a.lam + pn;
    px = nxp[0]; py = nxp[n_mp]; pz = nxp[2 * n_mp];
    lam[0] = nlam[0]; lam[1] = nlam[n_mp]; lam[2] = nlam[2 * n_mp];
    const int64_t* o2 = c2.a.offsets + row_of(w2, mine);
    const int64_t off2 = o2[0], end2 = o2[1];
    __builtin_amdgcn_sched_barrier(0);
    const int end = run ? end0 : 0;
    store_run(c2.a.N + even0, st, wl, front0, end);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      __builtin_amdgcn_sched_barrier(0);
      put(st, [&](int k) { return d[k][c]; });
      store_run(c2.a.dN + c * c2.a.cap + even0, st, wl, front0, end);
    }
    // (both words of each bound, so that no register of the loads is reused
    // while they are under way, which would wait for them before the stores)
    __asm__ volatile("" ::"v"(off2), "v"(end2));
    if (w1.c >= c_hi) break;
    w0 = w1;
    w1 = w2;
    real = true;
    n0 = n1; even0 = even1; front0 = front1; rel0 = rel1; K0 = K1;
    n1 = n2;
    set_row(off2, end2, mine < n2, even1, front1, rel1, K1);
  }
  // rows that were left (their stores are done at the barrier): the same
  // rounds again
  if (__syncthreads_or(some_left)) {
    const Call& cl = kernel_arg<Call>();
    const int wl = (int)__lane_id(), tid = (int)wave * kWave + wl;
    const int lane = wl / kWaveMps, mine = (int)wave * kWaveMps + wl % kWaveMps;
    for (Place w = start; w.c < c_hi; w = after(w)) {
      if (mine < count(w)) {
        const int64_t p = w.mp + mine;
        const int64_t off = cl.a.offsets[p];
        const int K = (int)(cl.a.offsets[p + 1] - off);
        if (K == 0 || K > kRowMax || cl.a.N[off] == kLeft)
          lme_uncached(cl.a, cl.in, p, lane, off, K, sink);
      }
      if constexpr (Sink::kTable) {
        if (w.k + 1 == rpc || (w.k + 1) % kFlushRounds == 0) {
          __syncthreads();
          sink.flush(cl.in, tid);
          __syncthreads();
        }
      }
    }
  }
}

template <class T>
struct Type {
  using type = T;
};

}  // namespace

void launch_lme_pipelined(int64_t n_nodes, const double* x_nodes, int64_t n_mp,
                          const double* x_mp, const int64_t* nbr_offsets, const int32_t* nbr_idx,
                          int64_t pair_capacity, double beta, double tol, int32_t max_iter,
                          double* lam, double* N, double* dN, const double4* packed,
                          otm_diag* diag, PairWindow mine, hipStream_t s, const AsmIn* fused,
                          const SegIn* seg) {
  if (n_mp <= 0) return;
  const int chunk = lme_chunk(n_mp);
  auto run = [&](auto tag, auto pk, auto in) {
    using Sink = typename decltype(tag)::type;
    constexpr bool PACKED = decltype(pk)::value;
    const LmeCall<PACKED, Sink> call{
        LmeArgs<PACKED>{NodeSrc<PACKED>{x_nodes, packed, n_nodes}, n_mp, x_mp, nbr_offsets,
                        nbr_idx, pair_capacity, beta, tol, max_iter, lam, N, dN, diag},
        in, mine, chunk};
    k_lme<PACKED, Sink><<<kLmeBlocks, 256, 0, s>>>(call);
  };
  // (the step's calls, the ones with a sink, always bring node records)
  constexpr std::true_type yes;
  if (fused != nullptr && fused->heat != nullptr)
    run(Type<AsmSink<true>>{}, yes, AsmSink<true>::In{*fused, nbr_idx});
  else if (fused != nullptr)
    run(Type<AsmSink<false>>{}, yes, AsmSink<false>::In{*fused, nbr_idx});
  else if (seg != nullptr)
    run(Type<SegSink>{}, yes, *seg);
  else if (packed != nullptr)
    run(Type<NoSink>{}, yes, NoSink::In{});
  else
    run(Type<NoSink>{}, std::false_type{}, NoSink::In{});
}

}  // namespace otm
