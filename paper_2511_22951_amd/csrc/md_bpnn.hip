// Behler-Parrinello network potential (Sec. 2.1) in FP64: symmetry functions,
// the atomic network with its backward pass, and forces by the chain rule (eq. force).
//
// One wavefront per atom.  Its neighbours within r_cut are compacted into LDS; the
// radial functions take lanes over neighbours, the angular ones lanes over the unordered
// pairs {j, k} with R_jk < r_cut, compacted a wavefront at a time (the summand is
// symmetric in j and k, so each unordered pair stands for both ordered ones).  The G4
// set is a grid of distinct eta values (index u) and distinct (zeta, lambda) pairs
// (index v): per pair the
// lane evaluates exp(-eta_u s2) and (1 + lambda_v cos)^zeta_v once each and
// accumulates their products on the grid, so the cost per pair does not grow with
// the number of G4 functions that share them.
//
// Bound by FP64 VALU issue (131,072 Cu atoms: 90 % busy in the symmetry functions and 76 % in the
// forces, LDS 47 and 52 %, profiles/pass_counters.txt): about 1400 of an atom's 3003
// unordered pairs (Cu, r_c 6 A) lie within the cutoff, each worth some 170 (symmetry functions)
// or 260 (forces) FP64 instructions.  What keeps the count there: exponentials from an LDS table
// with a short Taylor factor and powers by shared squarings (FAST below; library exp and a
// powering loop otherwise), cutoff functions of R_jk as polynomials in R_jk^2 (no square root,
// sine or division per pair), pairs enumerated so that the lanes of one step meet different
// neighbours (their LDS sums do not serialise), wave-uniform loop bounds (the accumulators stay
// in place).  51 functions, forces and energies: 32,000 Cu atoms 1.24 ms (5.33 ms with the pairs
// by triangle rows, library exponentials and the network inside the first pass); 864 atoms 0.100
// ms (4.12 ms with a whole tile of 64 atoms per block, which left all but 14 CUs idle).
#include <math.h>

#include <type_traits>

#include "md_internal.h"

namespace {

constexpr int NE = 8;  // distinct G4 eta values
constexpr int NZ = 8;  // distinct (zeta, lambda) pairs
constexpr int NL = NZ / 2;  // FAST: distinct zeta values, each with both signs of lambda
constexpr int NT = 512;     // FAST: rows of the exponential table
constexpr int WPB = 4; // waves (atoms in flight) per block
constexpr double PI = 3.14159265358979323846;

struct BpnnDev {
  double rc, rc2, rs;
  double inv_rc2, t_h, t_inv_h;  // 1 / r_c^2; interval of the exponential table and its inverse
  int n2, n4, ng, h1, h2, n_eta, n_zl;
  double g2_eta[MD_BPNN_MAX_G];
  double eta_u[NE], zeta_v[NZ], lam_v[NZ];
  int izeta_v[NZ];  // zeta as an integer (>= 1) or 0 when not integral
  double pref[MD_BPNN_MAX_G];
  unsigned char u_of[MD_BPNN_MAX_G], v_of[MD_BPNN_MAX_G];
  const double* w;  // w01 [ng][h1], b1 [h1], w12 [h1][h2], b2 [h2], w23 [h2], b3
  // FAST sets (fast_grid): v = 2 level + (lambda < 0), zeta of a level reached from the one
  // below by n_sq squarings; eta_u[0] = 0 (u0_one) or not
  int fast, u0_one, n_sq[NL];
};

// One atom's neighbours within r_cut, compacted in LDS.
struct Nb {
  double2 xy[MD_BPNN_MAX_NB];   // x, y of the vector a = x_j - x_i
  double2 zi[MD_BPNN_MAX_NB];   // z, 1 / R
  double2 rf[MD_BPNN_MAX_NB];   // R^2, f_c(R)
  alignas(16) double C[NE * NZ];
  unsigned short pq[4 * MD_WAVE];  // ring of neighbour pairs j | k << 8 (for_pairs_in_cutoff)
};
// ... and what the forces need beyond that.
struct NbForce : Nb {
  double df[MD_BPNN_MAX_NB];    // f_c'(R) / R
  double gx[MD_BPNN_MAX_NB], gy[MD_BPNN_MAX_NB], gz[MD_BPNN_MAX_NB];
  int j[MD_BPNN_MAX_NB];
};

// LDS written by this wavefront's other lanes is read next.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void cutoff(double R, double rc, double& fc, double& dfc) {
  if (R < rc) {
    double s, c;
    sincospi(R / rc, &s, &c);  // sin and cos of pi R / r_c (argument reduction is exact)
    fc = 0.5 * (c + 1.0);
    dfc = -0.5 * PI / rc * s;
  } else {
    fc = 0.0;
    dfc = 0.0;
  }
}

// The cutoff function of a squared distance, f_c = (cos(pi sqrt z) + 1) / 2 with
// z = R^2 / r_c^2 in [0, 1): entire in z, here its degree-10 Chebyshev interpolant about
// z = 1/2 (interpolation error 2e-17, below the rounding of 1e-16).
__device__ __forceinline__ double cutoff_z(double z) {
  const double c[11] = {0.1971500664605933,     -0.883792937313192,    1.1891487278891328,
                        -0.4622581725759399,    0.08880490245644401,   -0.010269231077289684,
                        0.0007960256795973061,  -4.4311202098765786e-05, 1.858761615541518e-06,
                        -6.091765597466249e-08, 1.6020184778650159e-09};
  const double t = z - 0.5;
  double r = c[10];
#pragma unroll
  for (int q = 9; q >= 0; --q) r = fma(r, t, c[q]);
  return r;
}
// Its derivative in z, -pi sin(pi sqrt z) / (4 sqrt z), the same way (error 4e-18);
// f_c'(R) / R = 2 / r_c^2 times this.
__device__ __forceinline__ double cutoff_dz(double z) {
  const double c[11] = {-0.8837929373131916,    2.3782974557782657,    -1.3867745177279067,
                        0.3552196098257719,     -0.0513461553831983,   0.004776154077654175,
                        -0.0003101784562931979, 1.4870092495597676e-05, -5.480449504404572e-07,
                        1.6021042248930055e-08, -3.8036293555090147e-10};
  const double t = z - 0.5;
  double r = c[10];
#pragma unroll
  for (int q = 9; q >= 0; --q) r = fma(r, t, c[q]);
  return r;
}

// x^n for an integer n >= 0 by binary powering, or pow(x, y) when n = 0 marks a
// non-integral exponent.
__device__ __forceinline__ double powi(double x, int n, double y) {
  if (n <= 0) return n == 0 && y != 0.0 ? pow(x, y) : 1.0;
  double r = 1.0;
  while (n) {
    if (n & 1) r *= x;
    x *= x;
    n >>= 1;
  }
  return r;
}

// Stage atom i's neighbours within r_cut into LDS (lane-parallel, order of the list);
// returns how many there are.
template <typename S>
__device__ int gather_neighbours(const BpnnDev& P, const md_domain& D, const double4* pos,
                                 const md_nlist& nl, size_t npad, int i, S& s, bool& over) {
  const int lane = threadIdx.x & (MD_WAVE - 1);
  const int nn = __builtin_amdgcn_readfirstlane(nl.nneigh[i] & MD_NN_MASK);
  const double4 pi = pos[i];
  int base = 0;
  for (int m0 = 0; m0 < nn; m0 += MD_WAVE) {
    const int m = m0 + lane;
    bool keep = false;
    double a[3] = {0, 0, 0}, r2 = 0.0;
    int j = 0;
    if (m < nn) {
      j = nl.neigh[((size_t)(m / nl.lanes) * npad + (size_t)i) * nl.lanes + (m % nl.lanes)];
      const double4 pj = pos[j];
      a[0] = pj.x - pi.x;
      a[1] = pj.y - pi.y;
      a[2] = pj.z - pi.z;
#pragma unroll
      for (int q = 0; q < 3; ++q)
        if (D.periodic[q]) a[q] -= D.len[q] * rint(a[q] * D.inv_len[q]);
      r2 = a[0] * a[0] + a[1] * a[1] + a[2] * a[2];
      keep = r2 < P.rc2;
    }
    const unsigned long long mask = __ballot(keep);
    const int slot = base + __popcll(mask & ((1ull << lane) - 1ull));
    if (keep && slot < MD_BPNN_MAX_NB) {
      const double R = sqrt(r2), iR = 1.0 / R;  // divisions per pair become products
      double fc, dfc;
      cutoff(R, P.rc, fc, dfc);
      s.xy[slot] = make_double2(a[0], a[1]);
      s.zi[slot] = make_double2(a[2], iR);
      s.rf[slot] = make_double2(r2, fc);
      if constexpr (std::is_same<S, NbForce>::value) {
        s.df[slot] = dfc * iR;
        s.gx[slot] = 0.0;
        s.gy[slot] = 0.0;
        s.gz[slot] = 0.0;
        s.j[slot] = j;
      }
    }
    base += __popcll(mask);
  }
  if (base > MD_BPNN_MAX_NB) over = true;
  wave_sync();
  return __builtin_amdgcn_readfirstlane(min(base, MD_BPNN_MAX_NB));  // (uniform loops follow)
}

// Geometry of the pair (j, k) of neighbours of the centre atom.
struct Trip {
  double cos, fAB, fC, s2, z;  // f_c(R_j) f_c(R_k), f_c(R_jk), z = R_jk^2 / r_c^2
};

__device__ __forceinline__ Trip triplet(const BpnnDev& P, const Nb& s, int j, int k) {
  Trip t;
  const double2 xj = s.xy[j], xk = s.xy[k], zj = s.zi[j], zk = s.zi[k], rj = s.rf[j],
                rk = s.rf[k];
  const double dx = xk.x - xj.x, dy = xk.y - xj.y, dz = zk.x - zj.x;
  const double C2 = dx * dx + dy * dy + dz * dz;
  t.z = C2 * P.inv_rc2;
  t.fC = cutoff_z(t.z);
  // |cos| <= 1 up to rounding; clamped so that a non-integral zeta never meets a
  // negative base
  t.cos = fmin(1.0, fmax(-1.0, (xj.x * xk.x + xj.y * xk.y + zj.x * zk.x) * (zj.y * zk.y)));
  t.s2 = rj.x + rk.x + C2;
  t.fAB = rj.y * rk.y;
  return t;
}

// The centre atom's unordered neighbour pairs with R_jk < r_cut, a wavefront at a
// time.  Lanes test 64 flat pair indices per trip and append the accepted pairs to an LDS
// queue; each full wavefront of queued pairs, and the remainder at the end, goes to
// body(j, k, active).  A pair beyond the cutoff adds nothing to G4 or to its derivatives
// (f_c(R_jk) = f_c'(R_jk) = 0), and about half the pairs of a neighbour sphere are such
// pairs: compacting them away keeps the lanes on pairs that contribute.
//
// Flat index t = q nc + m stands for the pair (m, m + q + 1 mod nc): t < nc (nc - 1) / 2 gives
// every unordered pair once (for even nc the last rotation holds half a round), and the lanes
// of a trip hold consecutive m, so that their LDS reads and sums fall on different neighbours.
// Going by rows j of the triangle instead gave a whole wavefront the same j, whose atomic adds
// then ran one after the other, and cost a square root per pair for the index.
template <typename Body>
__device__ __forceinline__ void for_pairs_in_cutoff(const BpnnDev& P, Nb& s, int nc, Body body) {
  if (nc < 2) return;
  const int lane = threadIdx.x & (MD_WAVE - 1);
  const int npairs = nc * (nc - 1) / 2;
  const int step_q = MD_WAVE / nc, step_m = MD_WAVE % nc;
  int q = lane / nc, m = lane % nc;
  int head = 0, tail = 0, t0 = 0;  // the ring's ends (below 64 entries between trips); pairs tested
  auto fill = [&]() {
    while (tail - head < MD_WAVE && t0 < npairs) {
      // two chunks of 64, so that their LDS reads overlap
      bool ok[2];
      int e[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int k = m + q + 1;
        k = k >= nc ? k - nc : k;
        ok[h] = t0 + lane < npairs;
        const int mm = ok[h] ? m : 0, kk = ok[h] ? k : 0;
        const double2 xj = s.xy[mm], xk = s.xy[kk];
        const double dx = xk.x - xj.x, dy = xk.y - xj.y, dz = s.zi[kk].x - s.zi[mm].x;
        ok[h] &= dx * dx + dy * dy + dz * dz < P.rc2;
        e[h] = m | (k << 8);
        t0 += MD_WAVE;
        q += step_q;
        m += step_m;
        if (m >= nc) {
          m -= nc;
          ++q;
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const unsigned long long acc = __builtin_amdgcn_ballot_w64(ok[h]);
        const int at = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(acc >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((unsigned)acc, tail));
        if (ok[h]) s.pq[at & (4 * MD_WAVE - 1)] = (unsigned short)e[h];
        tail += __popcll(acc);
      }
    }
  };
  fill();
  for (int take = min(MD_WAVE, tail); take > 0; take = min(MD_WAVE, tail - head)) {
    wave_sync();
    const unsigned e = lane < take ? s.pq[(head + lane) & (4 * MD_WAVE - 1)] : 0u;
    wave_sync();
    head += take;
    body((int)(e & 255u), (int)(e >> 8), lane < take);
    fill();
  }
  wave_sync();
}

// FAST: exp(-eta_u s) for s in [0, 3 r_c^2) as T_u(s_m) exp(eta_u (s_m - s)), s_m the centre
// of the s's interval (of NT): the table holds the first factor, and the second is its Taylor
// polynomial, whose argument fast_grid bounds by X_MAX (remainder x^7 / 5040 <= 1e-17).
constexpr double X_MAX = 0.0125;

template <int NEU>
__device__ __forceinline__ void fill_exp_table(const BpnnDev& P, double (*T)[NEU]) {
  for (int m = threadIdx.x; m < NT; m += blockDim.x)
    for (int u = 0; u < NEU; ++u) T[m][u] = exp(-P.eta_u[u] * (P.t_h * (m + 0.5)));
  __syncthreads();
}

// exp(-eta_u s2) for u = U, U + 1 (1 where the set has fewer eta values: P.eta_u is 0 there).
// at: the pair's place on the table, row and s_m - s2.  Two at a time, consumed before the next
// two: all of them at once cost the registers that the sums need.
struct ExpAt {
  int m;
  double ds;
};
template <bool FAST>
__device__ __forceinline__ ExpAt exp_at(const BpnnDev& P, double s2) {
  if constexpr (!FAST) return ExpAt{0, s2};
  const int m = min((int)(s2 * P.t_inv_h), NT - 1);
  return ExpAt{m, fma(P.t_h, (double)m + 0.5, -s2)};
}
template <int U, int NEU, bool FAST>
__device__ __forceinline__ void pair_exps(const BpnnDev& P, const double (*T)[NEU], const ExpAt& at,
                                          double (&X)[2]) {
  if constexpr (FAST) {
    const double2 t = *reinterpret_cast<const double2*>(&T[at.m][U]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (U == 0 && u == 0 && P.u0_one) {  // uniform
        X[0] = 1.0;
        continue;
      }
      const double x = P.eta_u[U + u] * at.ds;
      double e = fma(x, 1.0 / 720.0, 1.0 / 120.0);
      e = fma(e, x, 1.0 / 24.0);
      e = fma(e, x, 1.0 / 6.0);
      e = fma(e, x, 0.5);
      e = fma(e, x, 1.0);
      e = fma(e, x, 1.0);
      X[u] = (u == 0 ? t.x : t.y) * e;
    }
  } else {
#pragma unroll
    for (int u = 0; u < 2; ++u) X[u] = U + u < P.n_eta ? exp(-P.eta_u[U + u] * at.ds) : 1.0;
  }
}

// body(U, exponentials of eta U and U + 1) for U = 0, 2, .. NEU - 2.
template <int U, int NEU, bool FAST, typename Body>
__device__ __forceinline__ void for_exp_pairs(const BpnnDev& P, const double (*T)[NEU],
                                              const ExpAt& at, Body body) {
  if constexpr (U < NEU) {
    double X[2];
    pair_exps<U, NEU, FAST>(P, T, at, X);
    body(std::integral_constant<int, U>{}, X);
    __builtin_amdgcn_sched_barrier(0);
    for_exp_pairs<U + 2, NEU, FAST>(P, T, at, body);
  }
}

// (1 + lambda_v cos)^zeta_v, and with DER also zeta_v lambda_v times the power below it.
// FAST: both signs of lambda run through the ascending zeta levels by squarings
// (x^(2n - 1) = x^(n - 1) x^n).
template <bool FAST, bool DER>
__device__ __forceinline__ void pair_powers(const BpnnDev& P, double cos, double (&Pw)[NZ],
                                            double (&Pd)[NZ]) {
  if constexpr (FAST) {
    double a = 1.0 + cos, b = 1.0 - cos, a1 = 1.0, b1 = 1.0;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      for (int q = 0; q < P.n_sq[l]; ++q) {
        if (DER) {
          a1 *= a;
          b1 *= b;
        }
        a *= a;
        b *= b;
      }
      Pw[2 * l] = a;
      Pw[2 * l + 1] = b;
      if (DER) {
        Pd[2 * l] = P.zeta_v[2 * l] * a1;
        Pd[2 * l + 1] = -P.zeta_v[2 * l] * b1;
      }
    }
  } else {
#pragma unroll
    for (int v = 0; v < NZ; ++v) {
      const double base = 1.0 + P.lam_v[v] * cos;
      const int iz = P.izeta_v[v];
      if (DER) {
        const double p1 = v < P.n_zl ? powi(base, iz > 0 ? iz - 1 : 0, P.zeta_v[v] - 1.0) : 0.0;
        Pw[v] = p1 * base;
        Pd[v] = P.zeta_v[v] * P.lam_v[v] * p1;
      } else {
        Pw[v] = v < P.n_zl ? powi(base, iz, P.zeta_v[v]) : 0.0;
      }
    }
  }
}

// Wave-wide sums of v[0..N) spread over the lanes: each stage halves the values a lane still
// carries by exchanging the other half with its partner (a stage with an odd number adds them
// all).  On return v[0..rest) holds the sums of elements base .. base + rest - 1; rest is the
// return value.
template <int N, int O, int W>
__device__ __forceinline__ int wave_sum_scatter(double (&v)[W], int& base) {
  if constexpr (O == 0) {
    return N;
  } else if constexpr (N % 2 == 0) {
    const bool up = (threadIdx.x & O) != 0;
#pragma unroll
    for (int q = 0; q < N / 2; ++q) {
      const double keep = up ? v[q + N / 2] : v[q], give = up ? v[q] : v[q + N / 2];
      v[q] = keep + __shfl_xor(give, O, MD_WAVE);
    }
    base += up ? N / 2 : 0;
    return wave_sum_scatter<N / 2, O / 2, W>(v, base);
  } else {
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] += __shfl_xor(v[q], O, MD_WAVE);
    return wave_sum_scatter<N, O / 2, W>(v, base);
  }
}

// Block -> (tile, first atom of the tile): a tile's 64 atoms are split over 16 / K blocks of
// WPB wavefronts, K atoms each.
struct BlockAtoms {
  int tile, first;
};
__device__ __forceinline__ BlockAtoms block_atoms(int K) {
  const int per = MD_TILE / (WPB * K);
  return BlockAtoms{(int)blockIdx.x / per, (int)blockIdx.x % per * WPB * K};
}

// Pass 1: symmetry functions G of every atom.  NEU eta values are kept in the
// per-lane accumulator grid (NEU x NZ registers): 6 for sets with at most six distinct
// eta values (the common case), else NE.
template <int NEU, bool FAST>
__global__ __launch_bounds__(64 * WPB, FAST && NEU <= 6 ? 3 : 2) void k_bpnn_desc(md_batch b, BpnnDev P, const double4* pos,
                                                        md_nlist nl, size_t npad, int K,
                                                        double* G_all, md_ctl_dev* ctl) {
  __shared__ Nb sh[WPB];
  __shared__ alignas(16) double s_exp[FAST ? NT : 1][NEU];
  md_step_bookkeeping(ctl);
  if constexpr (FAST) fill_exp_table<NEU>(P, s_exp);
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / MD_WAVE);
  const int lane = threadIdx.x & (MD_WAVE - 1);
  Nb& s = sh[w];
  const BlockAtoms B = block_atoms(K);
  const md_tile T = b.tiles[B.tile];
  const md_domain& D = b.domains[T.rep];
  bool over = false;
  for (int a = B.first + w; a < min(T.count, B.first + WPB * K); a += WPB) {
    const int i = T.first + a;
    const int nc = gather_neighbours(P, D, pos, nl, npad, i, s, over);
    double* G = G_all + (size_t)i * P.ng;
    // radial functions: lanes over neighbours, eight functions at a time
    for (int mu0 = 0; mu0 < P.n2; mu0 += 8) {
      double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      for (int m = lane; m < nc; m += MD_WAVE) {
        const double2 rf = s.rf[m];
        const double d = sqrt(rf.x) - P.rs;
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (mu0 + u < P.n2) acc[u] += exp(-P.g2_eta[mu0 + u] * d * d) * rf.y;
      }
      int at = mu0;
      wave_sum_scatter<8, MD_WAVE / 2>(acc, at);
      if (at < P.n2) G[at] = acc[0];  // (lanes that share an element hold the same sum)
    }
    // angular functions: lanes over the unordered pairs within the cutoff
    double g[NEU * NZ];
#pragma unroll
    for (int q = 0; q < NEU * NZ; ++q) g[q] = 0.0;
    for_pairs_in_cutoff(P, s, nc, [&](int j, int k, bool active) {
      const Trip t = triplet(P, s, j, k);
      const double f3 = active ? t.fAB * t.fC : 0.0;
      const bool on = f3 != 0.0;  // (an idle lane's powers may overflow: 0 times them is not 0)
      double Pw[NZ], none[NZ];
      pair_powers<FAST, false>(P, on ? t.cos : 0.0, Pw, none);
      for_exp_pairs<0, NEU, FAST>(P, s_exp, exp_at<FAST>(P, on ? t.s2 : 0.0),
                                  [&](auto U, const double (&X)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const double x = X[u] * f3;
#pragma unroll
          for (int v = 0; v < NZ; ++v)
            g[(U + u) * NZ + v] = fma(x, Pw[v], g[(U + u) * NZ + v]);
        }
      });
    });
    // (one eta value's sums at a time: all of them at once spill registers)
#pragma unroll
    for (int u = 0; u < NEU; ++u) {
      double r[NZ];
#pragma unroll
      for (int v = 0; v < NZ; ++v) r[v] = g[u * NZ + v];
      int at = u * NZ;
      wave_sum_scatter<NZ, MD_WAVE / 2>(r, at);
      s.C[at] = r[0];
      __builtin_amdgcn_sched_barrier(0);
    }
    wave_sync();
    if (lane < P.n4)
      G[P.n2 + lane] = 2.0 * P.pref[lane] * s.C[P.u_of[lane] * NZ + P.v_of[lane]];
    wave_sync();
  }
  if (__any(over) && lane == 0) md_flag(ctl, MD_FLAG_NEIGH_OVERFLOW);
}

// The atomic network and its backward pass: a tile's 64 atoms per block, an atom per lane,
// hidden units and inputs dealt out to the block's wavefronts; the weights, the same for every
// lane, come through the scalar cache.  G [n][ng] is replaced by dE_i/dG.  As part of the
// symmetry-function kernel (one atom per wavefront, ten lanes at work) it was a chain of some
// 200 dependent loads per atom.
__global__ __launch_bounds__(64 * WPB) void k_bpnn_net(md_batch b, BpnnDev P, double* G_all,
                                                      double* e_buf) {
  constexpr int LD = MD_TILE + 1;
  __shared__ double s_G[MD_BPNN_MAX_G * LD];
  __shared__ double s_h1[MD_BPNN_MAX_HIDDEN][MD_TILE], s_h2[MD_BPNN_MAX_HIDDEN][MD_TILE];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / MD_WAVE);
  const int lane = threadIdx.x & (MD_WAVE - 1);
  const md_tile T = b.tiles[blockIdx.x];
  const int ng = P.ng, h1 = P.h1, h2 = P.h2;
  double* G = G_all + (size_t)T.first * ng;
  for (int q = threadIdx.x; q < MD_TILE * ng; q += blockDim.x)
    s_G[q % ng * LD + q / ng] = q < T.count * ng ? G[q] : 0.0;
  const double* __restrict__ w01 = P.w;
  const double* __restrict__ b1 = w01 + (size_t)ng * h1;
  const double* __restrict__ w12 = b1 + h1;
  const double* __restrict__ b2 = w12 + (size_t)h1 * h2;
  const double* __restrict__ w23 = b2 + h2;
  __syncthreads();
  for (int q = w; q < h1; q += WPB) {
    double x = b1[q];
#pragma unroll 8
    for (int mu = 0; mu < ng; ++mu) x += s_G[mu * LD + lane] * w01[mu * h1 + q];
    s_h1[q][lane] = tanh(x);
  }
  __syncthreads();
  for (int q = w; q < h2; q += WPB) {
    double x = b2[q];
#pragma unroll 4
    for (int p = 0; p < h1; ++p) x += s_h1[p][lane] * w12[p * h2 + q];
    s_h2[q][lane] = tanh(x);
  }
  __syncthreads();
  if (w == 0) {
    double e = 0.0;
    for (int q = 0; q < h2; ++q) e += w23[q] * s_h2[q][lane];
    if (lane < T.count) e_buf[T.first + lane] = w23[h2] + e;
  }
  for (int p = w; p < h1; p += WPB) {  // s_h1 becomes dE/d(hidden 1 input)
    double x = 0.0;
#pragma unroll 4
    for (int q = 0; q < h2; ++q) {
      const double h = s_h2[q][lane];
      x += w12[p * h2 + q] * (w23[q] * (1.0 - h * h));
    }
    const double h = s_h1[p][lane];
    s_h1[p][lane] = x * (1.0 - h * h);
  }
  __syncthreads();
  for (int mu = w; mu < ng; mu += WPB) {
    double x = 0.0;
#pragma unroll 4
    for (int p = 0; p < h1; ++p) x += w01[mu * h1 + p] * s_h1[p][lane];
    s_G[mu * LD + lane] = x;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < T.count * ng; q += blockDim.x) G[q] = s_G[q % ng * LD + q / ng];
}

// Add a block's sums v[0..7) (E, W[6]) into the record as fixed point.
__device__ __forceinline__ void block_record_add(double (&v)[7], double* red, long long* slot,
                                                 int rep) {
  const int w = threadIdx.x / MD_WAVE, lane = threadIdx.x & (MD_WAVE - 1);
#pragma unroll
  for (int q = 0; q < 7; ++q) v[q] = md_wave_sum(v[q]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 7; ++q) red[w * 7 + q] = v[q];
  __syncthreads();
  if (threadIdx.x < 7) {
    double s = 0.0;
    for (int q = 0; q < WPB; ++q) s += red[q * 7 + threadIdx.x];
    atomicAdd((unsigned long long*)&slot[(size_t)rep * MD_EV_LEN + threadIdx.x],
              (unsigned long long)(long long)rint(s * MD_EV_SCALE));
  }
}

// Pass 2: forces.  g_m = dE_i/d a_m for every neighbour vector a_m = x_j - x_i;
// F_j -= g_m, F_i += sum_m g_m, W -= a_m (x) g_m.
template <int NEU, bool FAST>
__global__ __launch_bounds__(64 * WPB, 2) void k_bpnn_force(md_batch b, BpnnDev P,
                                                         const double4* pos, md_nlist nl,
                                                         size_t npad, int K, const double* dEdG,
                                                         const double* e_buf, double* force,
                                                         long long* ev, int ev_cap,
                                                         md_ctl_dev* ctl) {
  __shared__ NbForce sh[WPB];
  __shared__ alignas(16) double s_exp[FAST ? NT : 1][NEU];
  __shared__ double red[WPB * 7];
  if constexpr (FAST) fill_exp_table<NEU>(P, s_exp);
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / MD_WAVE);
  const int lane = threadIdx.x & (MD_WAVE - 1);
  NbForce& s = sh[w];
  const BlockAtoms B = block_atoms(K);
  const md_tile T = b.tiles[B.tile];
  const md_domain& D = b.domains[T.rep];
  const int n = b.n_atoms;
  bool over = false;
  double acc[7] = {0, 0, 0, 0, 0, 0, 0};  // E, W xx yy zz xy xz yz
  for (int a = B.first + w; a < min(T.count, B.first + WPB * K); a += WPB) {
    const int i = T.first + a;
    const int nc = gather_neighbours(P, D, pos, nl, npad, i, s, over);
    const double* c = dEdG + (size_t)i * P.ng;
    // grid weights of the angular terms
    for (int q = lane; q < NE * NZ; q += MD_WAVE) s.C[q] = 0.0;
    wave_sync();
    if (lane < P.n4)  // both orders of each pair
      atomicAdd(&s.C[P.u_of[lane] * NZ + P.v_of[lane]], 2.0 * c[P.n2 + lane] * P.pref[lane]);
    wave_sync();
    // radial terms: lanes over neighbours
    for (int m = lane; m < nc; m += MD_WAVE) {
      const double2 xy = s.xy[m], zi = s.zi[m], rf = s.rf[m];
      const double R = sqrt(rf.x), d = R - P.rs, fc = rf.y, dfc = s.df[m] * R;
      double dR = 0.0;
      for (int mu = 0; mu < P.n2; ++mu) {
        const double eta = P.g2_eta[mu];
        dR += c[mu] * exp(-eta * d * d) * (dfc - 2.0 * eta * d * fc);
      }
      const double q = dR / R;
      s.gx[m] += q * xy.x;
      s.gy[m] += q * xy.y;
      s.gz[m] += q * zi.x;
    }
    wave_sync();
    // angular terms: lanes over the unordered pairs within the cutoff.  The pair
    // (j, k) adds g_a to neighbour j and g_b to k; the reversed order adds the same
    // vectors with the roles swapped, which the factor 2 in the grid weights C accounts
    // for.  Lanes of one step can share a neighbour, so the LDS sums take atomic adds.
    // Up to six eta values the weights stay in registers.
    constexpr bool REG = NEU <= 6;
    double cw[REG ? NEU * NZ : 1];
    if constexpr (REG) {
#pragma unroll
      for (int q = 0; q < NEU * NZ; q += 2) {
        const double2 v = *reinterpret_cast<const double2*>(&s.C[q]);
        cw[q] = v.x;
        cw[q + 1] = v.y;
      }
    }
    for_pairs_in_cutoff(P, s, nc, [&](int j, int k, bool active) {
      if (!active) return;
      const Trip t = triplet(P, s, j, k);
      double Pw[NZ], Pd[NZ];
      pair_powers<FAST, true>(P, t.cos, Pw, Pd);
      double q1 = 0.0, qe = 0.0, qc = 0.0;
      for_exp_pairs<0, NEU, FAST>(P, s_exp, exp_at<FAST>(P, t.s2),
                                  [&](auto U, const double (&X)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          double S = 0.0, Q = 0.0;  // sum_v C_uv (power), sum_v C_uv (its derivative in cos)
#pragma unroll
          for (int v = 0; v < NZ; ++v) {
            const double cuv = REG ? cw[REG ? (U + u) * NZ + v : 0] : s.C[(U + u) * NZ + v];
            S = fma(cuv, Pw[v], S);
            Q = fma(cuv, Pd[v], Q);
          }
          q1 = fma(X[u], S, q1);
          qe = fma(P.eta_u[U + u] * X[u], S, qe);
          qc = fma(X[u], Q, qc);
        }
      });
      const double2 xj = s.xy[j], xk = s.xy[k], zj = s.zi[j], zk = s.zi[k];
      const double fA = s.rf[j].y, fB = s.rf[k].y, dfA = s.df[j], dfB = s.df[k];
      const double dfC = 2.0 * P.inv_rc2 * cutoff_dz(t.z);  // f_c'(R) / R, as df
      const double f3 = t.fAB * t.fC, s_cos = qc * f3, e2 = 2.0 * qe * f3;
      const double rA = q1 * dfA * fB * t.fC - e2;
      const double rB = q1 * fA * dfB * t.fC - e2;
      const double rC = q1 * t.fAB * dfC - e2;
      const double iAB = s_cos * (zj.y * zk.y);
      const double cA = rA - s_cos * t.cos * (zj.y * zj.y);
      const double cB = rB - s_cos * t.cos * (zk.y * zk.y);
      const double aj[3] = {xj.x, xj.y, zj.x}, ak[3] = {xk.x, xk.y, zk.x};
      double ga[3], gb[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const double d = ak[q] - aj[q];
        ga[q] = iAB * ak[q] + cA * aj[q] - rC * d;
        gb[q] = iAB * aj[q] + cB * ak[q] + rC * d;
      }
      atomicAdd(&s.gx[j], ga[0]);
      atomicAdd(&s.gy[j], ga[1]);
      atomicAdd(&s.gz[j], ga[2]);
      atomicAdd(&s.gx[k], gb[0]);
      atomicAdd(&s.gy[k], gb[1]);
      atomicAdd(&s.gz[k], gb[2]);
    });
    wave_sync();
    // scatter: F_j -= g, F_i += sum g, W -= a (x) g
    double fi[3] = {0, 0, 0}, wv[6] = {0, 0, 0, 0, 0, 0};
    for (int m = lane; m < nc; m += MD_WAVE) {
      const double2 xy = s.xy[m];
      const double g[3] = {s.gx[m], s.gy[m], s.gz[m]};
      const double av[3] = {xy.x, xy.y, s.zi[m].x};
      const int j = s.j[m];
      atomicAdd(&force[j], -g[0]);
      atomicAdd(&force[n + j], -g[1]);
      atomicAdd(&force[2 * n + j], -g[2]);
      fi[0] += g[0];
      fi[1] += g[1];
      fi[2] += g[2];
      wv[0] -= av[0] * g[0];
      wv[1] -= av[1] * g[1];
      wv[2] -= av[2] * g[2];
      wv[3] -= av[0] * g[1];
      wv[4] -= av[0] * g[2];
      wv[5] -= av[1] * g[2];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) fi[q] = md_wave_sum(fi[q]);
    if (lane == 0) {
      atomicAdd(&force[i], fi[0]);
      atomicAdd(&force[n + i], fi[1]);
      atomicAdd(&force[2 * n + i], fi[2]);
      acc[0] += e_buf[i];
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) acc[1 + q] += wv[q];
    wave_sync();
  }
  if (ev) block_record_add(acc, red, ev + (size_t)(ctl->step % ev_cap) * b.n_rep * MD_EV_LEN,
                           T.rep);
}

// Zero the forces and the record slot of the step being evaluated.
__global__ void k_bpnn_zero(md_batch b, double* force, long long* ev, int ev_cap,
                            const md_ctl_dev* ctl) {
  const size_t n3 = (size_t)3 * b.n_atoms;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n3;
       k += (size_t)gridDim.x * blockDim.x)
    force[k] = 0.0;
  if (ev && blockIdx.x == 0) {
    long long* slot = ev + (size_t)(ctl->step_next % ev_cap) * b.n_rep * MD_EV_LEN;
    for (int q = threadIdx.x; q < b.n_rep * MD_EV_LEN; q += blockDim.x) slot[q] = 0;
  }
}

// Trailing half kick v += half_dt f/m and the kinetic energy into the record.
__global__ __launch_bounds__(MD_ATOM_BLOCK) void k_bpnn_kick(md_batch b, const double* force,
                                                             double* vel, double c, double inv_mass,
                                                             long long* ev, int ev_cap,
                                                             const md_ctl_dev* ctl) {
  const int n = b.n_atoms;
  const int lane = threadIdx.x & (MD_WAVE - 1);
  const int tile = blockIdx.x * (MD_ATOM_BLOCK / MD_WAVE) + threadIdx.x / MD_WAVE;
  double k = 0.0;
  int rep = -1;
  if (tile < b.n_tiles) {
    const md_tile T = b.tiles[tile];
    rep = T.rep;
    if (lane < T.count) {
      const int i = T.first + lane;
      double v[3];
      for (int q = 0; q < 3; ++q) {
        v[q] = vel[(size_t)q * n + i] + c * force[(size_t)q * n + i];
        vel[(size_t)q * n + i] = v[q];
      }
      k = 0.5 / (inv_mass * MD_ACCEL) * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    }
  }
  k = md_wave_sum(k);
  if (ev && lane == 0 && rep >= 0)
    atomicAdd((unsigned long long*)&ev[((size_t)(ctl->step % ev_cap) * b.n_rep + rep) * MD_EV_LEN + 7],
              (unsigned long long)(long long)rint(k * MD_EV_SCALE));
}

// Whether the set can take the FAST evaluation, and its grid in that order.  The rule is what
// the evaluation can represent: every zeta a power of two with at most NL distinct values (up to
// 512: both signs of lambda are formed, and 1024 2^1023 overflows in the one that no function has), and
// |eta| small enough for the exponential table's Taylor factor, |eta| 3 r_c^2 / (2 NT) <= X_MAX
// (|eta| r_c^2 <= 4.2).  Wherever it holds it is the faster one: 32,000 Cu atoms 1.37 ms against
// 2.48 ms for the general form (48 functions with one zeta of 3 in place of 4), 864 atoms 0.100
// against 0.165 ms.
void fast_grid(BpnnDev* d) {
  int lev[NZ], nlev = 0;  // distinct zeta, ascending
  for (int v = 0; v < d->n_zl; ++v) {
    const int z = d->izeta_v[v];
    if (z < 1 || z > 512 || (z & (z - 1))) return;
    int l = 0;
    while (l < nlev && lev[l] < z) ++l;
    if (l < nlev && lev[l] == z) continue;
    if (nlev == NL) return;
    for (int q = nlev; q > l; --q) lev[q] = lev[q - 1];
    lev[l] = z;
    ++nlev;
  }
  for (int u = 0; u < d->n_eta; ++u)
    if (!(fabs(d->eta_u[u]) * 3.0 * d->rc2 <= 2.0 * NT * X_MAX)) return;
  if (d->n4 == 0) return;
  unsigned char v_new[NZ];
  for (int v = 0; v < d->n_zl; ++v) {
    int l = 0;
    while (lev[l] != d->izeta_v[v]) ++l;
    v_new[v] = (unsigned char)(2 * l + (d->lam_v[v] < 0.0));
  }
  int u0 = 0;
  while (u0 < d->n_eta && d->eta_u[u0] != 0.0) ++u0;
  d->u0_one = u0 < d->n_eta;
  if (d->u0_one) {
    d->eta_u[u0] = d->eta_u[0];
    d->eta_u[0] = 0.0;
  }
  for (int q = 0; q < d->n4; ++q) {
    d->v_of[q] = v_new[d->v_of[q]];
    if (d->u0_one)
      d->u_of[q] = (unsigned char)(d->u_of[q] == u0 ? 0 : (d->u_of[q] == 0 ? u0 : d->u_of[q]));
  }
  for (int l = 0; l < NL; ++l) {
    d->n_sq[l] = 0;
    for (int z = l ? (l < nlev ? lev[l - 1] : 0) : 1; l < nlev && z < lev[l]; z *= 2) ++d->n_sq[l];
    d->zeta_v[2 * l] = l < nlev ? lev[l] : 0.0;
  }
  d->fast = 1;
}

int load_params(const md_bpnn* p, BpnnDev* d) {
  *d = BpnnDev{};
  if (!p || !p->weights || !(p->r_cut > 0.0) || p->n_g2 < 0 || p->n_g4 < 0 ||
      p->n_g2 + p->n_g4 < 1 || p->n_g2 + p->n_g4 > MD_BPNN_MAX_G || p->h1 < 1 || p->h2 < 1 ||
      p->h1 > MD_BPNN_MAX_HIDDEN || p->h2 > MD_BPNN_MAX_HIDDEN)
    return MD_ERR_ARG;
  d->rc = p->r_cut;
  d->rc2 = p->r_cut * p->r_cut;
  d->rs = p->r_s;
  d->inv_rc2 = 1.0 / d->rc2;
  d->t_h = 3.0 * d->rc2 / NT;
  d->t_inv_h = NT / (3.0 * d->rc2);
  d->n2 = p->n_g2;
  d->n4 = p->n_g4;
  d->ng = p->n_g2 + p->n_g4;
  d->h1 = p->h1;
  d->h2 = p->h2;
  d->w = p->weights;
  for (int q = 0; q < p->n_g2; ++q) d->g2_eta[q] = p->g2_eta[q];
  for (int q = 0; q < p->n_g4; ++q) {
    const double eta = p->g4_eta[q], zeta = p->g4_zeta[q], lam = p->g4_lambda[q];
    if (!(zeta >= 1.0) || !(lam == 1.0 || lam == -1.0) || !isfinite(eta)) return MD_ERR_ARG;
    int u = 0;
    while (u < d->n_eta && d->eta_u[u] != eta) ++u;
    if (u == d->n_eta) {
      if (u == NE) return MD_ERR_ARG;
      d->eta_u[d->n_eta++] = eta;
    }
    int v = 0;
    while (v < d->n_zl && !(d->zeta_v[v] == zeta && d->lam_v[v] == lam)) ++v;
    if (v == d->n_zl) {
      if (v == NZ) return MD_ERR_ARG;
      d->zeta_v[v] = zeta;
      d->lam_v[v] = lam;
      d->izeta_v[v] = (zeta == floor(zeta) && zeta <= 1024.0) ? (int)zeta : 0;
      ++d->n_zl;
    }
    d->u_of[q] = (unsigned char)u;
    d->v_of[q] = (unsigned char)v;
    d->pref[q] = pow(2.0, 1.0 - zeta);
  }
  fast_grid(d);
  return MD_OK;
}

}  // namespace

extern "C" size_t md_bpnn_workspace_bytes(const md_batch* b, const md_bpnn* p) {
  if (!b || !p || p->n_g2 + p->n_g4 < 1) return 0;
  return md_align256((size_t)b->n_atoms * (size_t)(p->n_g2 + p->n_g4 + 1) * sizeof(double));
}

extern "C" int md_bpnn_forces(const md_batch* b, const md_bpnn* p, const double* pos,
                              const md_nlist* nl, double* force, double* e_atom, double* vel,
                              double inv_mass, double half_dt, long long* ev, int ev_cap,
                              void* ws, void* ctl, void* stream) {
  if (!md_batch_ok(b)) return MD_ERR_ARG;
  if (!pos || !nl || !nl->neigh || !nl->nneigh || !force || !ws || !ctl) return MD_ERR_ARG;
  if (nl->lanes < 1 || nl->lanes > MD_MAX_LANES || nl->max_neigh < nl->lanes) return MD_ERR_ARG;
  if (ev && ev_cap < 1) return MD_ERR_ARG;
  if (vel && !(inv_mass > 0.0)) return MD_ERR_ARG;
  BpnnDev P;
  if (load_params(p, &P) != MD_OK) return MD_ERR_ARG;
  if (b->n_atoms == 0) return MD_OK;
  hipStream_t st = (hipStream_t)stream;
  md_ctl_dev* c = (md_ctl_dev*)ctl;
  const size_t npad = (size_t)md_npad(b->n_atoms);
  double* dEdG = (double*)ws;
  double* e_buf = e_atom ? e_atom : dEdG + (size_t)b->n_atoms * P.ng;
  hipLaunchKernelGGL(k_bpnn_zero, dim3(1024), dim3(256), 0, st, *b, force, (long long*)ev, ev_cap,
                     c);
  MD_LAUNCH_CHECK();
  // Atoms per wavefront: one while that leaves at most eight rounds of the 2048 wavefronts the
  // chip holds of these kernels, more beyond (fewer tables and record sums per atom).  At 864
  // atoms one per wavefront takes 0.107 ms where sixteen per wavefront took milliseconds.
  int K = 1;
  while (K < MD_TILE / WPB && (size_t)b->n_atoms > (size_t)16384 * K) K *= 2;
  const dim3 grid(b->n_tiles * (MD_TILE / (WPB * K))), block(64 * WPB);
#define MD_BPNN_LAUNCH(NEU, FAST)                                                                \
  do {                                                                                           \
    MD_LAUNCH_TIMED(MD_KERNEL_BPNN_DESC, (k_bpnn_desc<NEU, FAST>), grid, block, 0, st, *b, P,    \
                    (const double4*)pos, *nl, npad, K, dEdG, c);                                 \
    MD_LAUNCH_CHECK();                                                                           \
    hipLaunchKernelGGL(k_bpnn_net, dim3(b->n_tiles), block, 0, st, *b, P, dEdG, e_buf);          \
    MD_LAUNCH_CHECK();                                                                           \
    MD_LAUNCH_TIMED(MD_KERNEL_BPNN_FORCE, (k_bpnn_force<NEU, FAST>), grid, block, 0, st, *b, P,  \
                    (const double4*)pos, *nl, npad, K, (const double*)dEdG,                      \
                    (const double*)e_buf, force, (long long*)ev, ev_cap, c);                     \
    MD_LAUNCH_CHECK();                                                                           \
  } while (0)
  if (P.n_eta <= 6) {
    if (P.fast) MD_BPNN_LAUNCH(6, true);
    else MD_BPNN_LAUNCH(6, false);
  } else {
    if (P.fast) MD_BPNN_LAUNCH(NE, true);
    else MD_BPNN_LAUNCH(NE, false);
  }
#undef MD_BPNN_LAUNCH
  if (vel) {
    const int nb = (b->n_tiles + MD_ATOM_BLOCK / MD_WAVE - 1) / (MD_ATOM_BLOCK / MD_WAVE);
    hipLaunchKernelGGL(k_bpnn_kick, dim3(nb), dim3(MD_ATOM_BLOCK), 0, st, *b,
                       (const double*)force, vel, half_dt * inv_mass * MD_ACCEL, inv_mass,
                       (long long*)ev, ev_cap, c);
    MD_LAUNCH_CHECK();
  }
  return MD_OK;
}
