// gfx950 kernels of the coupled lattice-Boltzmann / dynamic immersed-boundary
// step (Coclite, de Tullio, Pascazio, Politi, arXiv 2207.06043, section
// "Numerical method and computational procedure").
//
// One coupled step is four launches on one stream (a step without bodies:
// the fluid launch alone):
//   k_ib_force   marker blocks: MLS interpolation of the streamed (pre-force)
//                velocity at the face centroids, direct forcing and spreading
//                (fixed-point atomics, deterministic); element blocks:
//                stretching and bending forces; diagnostics blocks: volume,
//                area, bounding box and damage check of the positions;
//   k_fluid_all  (k_fluid_bulk and k_fluid_rec on two streams for large
//                grids) fused pull-stream + wall links (interpolated
//                bounce-back) + Zou-He + moments + forced BGK collision; bulk
//                nodes as SoA loads/stores of V consecutive nodes (or one node
//                per thread from a list), boundary nodes from compact records;
//   k_mls_post   hydrodynamic probes (pressure and viscous stress from MLS
//                fits at +-1.2 dx), repulsion, MLS velocity at the vertices,
//                clearing of the previous step's spread buffer;
//   k_body_post  vertex forces and Verlet (soft) / Newton-Euler (rigid).
// One thread of a step's last launch counts the step.
// Populations are stored as deviations g_i = f_i - w_i from the rest
// equilibrium; the collision is written for g (algebraically identical to the
// BGK rule on f, with smaller rounding).
#include <float.h>
#include <limits.h>
#include <math.h>

#include <mutex>

#include "lbm_internal.h"

namespace lbm {

// D3Q19 velocity set in the order of the paper's Eq. e_i.
constexpr int EX[19] = {0, 1, -1, 0, 0, 0, 0, 1, 1, 1, 1, -1, -1, -1, -1, 0, 0, 0, 0};
constexpr int EY[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1};
constexpr int EZ[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 1, -1, 1, -1};
constexpr int OPP[19] = {0, 2, 1, 4, 3, 6, 5, 12, 11, 14, 13, 8, 7, 10, 9, 18, 17, 16, 15};
constexpr double WD[19] = {1.0 / 3,  1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18,
                           1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                           1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

// ---------------------------------------------------------------- storage
__device__ __forceinline__ double to_c(double v) { return v; }
__device__ __forceinline__ float to_c(float v) { return v; }
__device__ __forceinline__ float to_c(_Float16 v) { return (float)v; }

template <class S>
struct Store;
template <>
struct Store<double> {
  typedef double C;
};
template <>
struct Store<float> {
  typedef float C;
};
template <>
struct Store<_Float16> {
  typedef float C;
};
// V consecutive populations of one plane: aligned and element-aligned forms.
template <class S, int V>
struct Vec {
  typedef S a __attribute__((ext_vector_type(V)));
  typedef S u __attribute__((ext_vector_type(V), aligned(sizeof(S))));
};
template <int V>
struct ClsWord;
template <>
struct ClsWord<1> { typedef uint8_t T; };
template <>
struct ClsWord<2> { typedef uint16_t T; };
template <>
struct ClsWord<4> { typedef uint32_t T; };
template <>
struct ClsWord<8> { typedef uint64_t T; };

// ------------------------------------------------------------ index helpers
__device__ __forceinline__ int wrap2(int c, int n) {  // |c| excursion <= 2 cells
  c = c < 0 ? c + n : (c >= n ? c - n : c);
  return c < 0 ? c + n : (c >= n ? c - n : c);
}
__device__ __forceinline__ long long nbr(const Grid& G, int x, int y, int z, int dx, int dy,
                                         int dz) {
  x = wrap2(x + dx, G.nx);
  y = wrap2(y + dy, G.ny);
  z = wrap2(z + dz, G.nz);
  return x + (long long)G.px * (y + (long long)G.ny * z);
}

__device__ __forceinline__ unsigned int udiv31(unsigned int u, unsigned int m, int s) {
  return (unsigned int)(((unsigned long long)u * m) >> s);
}
__device__ __forceinline__ void coords(const Grid& G, long long n, int& x, int& y, int& z) {
  const unsigned int u = (unsigned int)n;  // padded index < 2^31
  const unsigned int t = u / (unsigned int)G.px;
  x = (int)(u - t * (unsigned int)G.px);
  z = (int)(t / (unsigned int)G.ny);
  y = (int)(t - (unsigned int)z * (unsigned int)G.ny);
}
// The same with the divisions as multiply-shifts (fewer instructions; the
// fluid kernels, where the instruction count bounds the FP16S sweep).
__device__ __forceinline__ void coords_ms(const Grid& G, long long n, int& x, int& y, int& z) {
  const unsigned int u = (unsigned int)n;
  const unsigned int t = udiv31(u, G.mpx, G.spx);
  x = (int)(u - t * (unsigned int)G.px);
  z = (int)udiv31(t, G.mny, G.sny);
  y = (int)(t - (unsigned int)z * (unsigned int)G.ny);
}

// The wrapped neighbourhood of a node for offsets -2..2 on each axis, as the
// three terms of a padded index (x, px y, px ny z): at() gives the same index
// as nbr(), with the wraps done once per node instead of once per neighbour.
struct Hood {
  int tx[5], ty[5], tz[5];
  __device__ __forceinline__ int at(int dx, int dy, int dz) const {
    return tx[dx + 2] + ty[dy + 2] + tz[dz + 2];
  }
};
__device__ __forceinline__ Hood hood(const Grid& G, int x, int y, int z) {
  Hood h;
#pragma unroll
  for (int d = 0; d < 5; d++) {
    h.tx[d] = wrap2(x + d - 2, G.nx);
    h.ty[d] = G.px * wrap2(y + d - 2, G.ny);
    h.tz[d] = G.px * G.ny * wrap2(z + d - 2, G.nz);
  }
  return h;
}

// Blocks are dispatched round-robin over the 8 XCDs; give every XCD a
// contiguous run of tiles so that neighbouring rows share its L2.
__device__ __forceinline__ int xcd_remap(int b, int n) {
  int full = n & ~7;
  if (b >= full) return b;
  return (b & 7) * (full >> 3) + (b >> 3);
}

__device__ __forceinline__ void fx_add(long long* p, double v, DevFlags* fl) {
  if (!(fabs(v) <= 1.0)) {
    // out of the fixed-point range: dropped and flagged
    atomicOr(&fl->overflow, 1u);
    v = 0.0;
  }
  long long q = __double2ll_rn(v * FX_SCALE);
  atomicAdd((unsigned long long*)p, (unsigned long long)q);
}

// ---------------------------------------------------------------- collision
// Sum of the 19 deviations (the density deviation rho - 1).  The deviations
// of a direction and its opposite are close to +-3 w e.u and nearly cancel,
// so they are added pairwise first: those sums are exact or nearly so, and
// the density deviation keeps its relative precision in float as well,
// instead of carrying rounding of the size of the large terms.
template <class C>
__device__ __forceinline__ C dev_sum(const C (&g)[19]) {
  const C ax = ((g[1] + g[2]) + (g[3] + g[4])) + (g[5] + g[6]);
  const C d1 = ((g[7] + g[12]) + (g[8] + g[11])) + ((g[9] + g[14]) + (g[10] + g[13]));
  const C d2 = (g[15] + g[18]) + (g[16] + g[17]);
  return g[0] + ((ax + d1) + d2);
}

// e v for a lattice velocity component e in {-1, 0, 1}.  The zero term is
// -0, which an addition drops exactly, so the unrolled dot products below
// keep only their non-zero terms: the same values as the full products
// (0 v + w = w), without the multiplications by zero that IEEE arithmetic
// would otherwise have to carry out.
template <class C>
__device__ __forceinline__ C eterm(int e, C v) {
  return e == 0 ? C(-0.0) : (e > 0 ? v : -v);
}

// BGK with the forcing term on deviations g = f - w (Eqs. evoleq, eqfunc,
// forcing): rho = 1 + sum g, rho u = sum g e + F/2,
// g^eq_i = w_i (drho + rho (3 e.u + 9/2 (e.u)^2 - 3/2 u.u)),
// F_i = (1 - 1/(2 tau)) w_i (3 (e_i - u) + 9 (e_i.u) e_i).F.
template <class C>
__device__ __forceinline__ void collide(C (&g)[19], C Fx, C Fy, C Fz, C omega, C& drho_out, C& ux,
                                        C& uy, C& uz) {
  const C drho = dev_sum(g);
  drho_out = drho;
  C mx = (g[1] - g[2]) + (g[7] + g[8]) + (g[9] + g[10]) - (g[11] + g[12]) - (g[13] + g[14]);
  C my = (g[3] - g[4]) + (g[7] - g[8]) + (g[11] - g[12]) + (g[15] + g[16]) - (g[17] + g[18]);
  C mz = (g[5] - g[6]) + (g[9] - g[10]) + (g[13] - g[14]) + (g[15] - g[16]) + (g[17] - g[18]);
  const C rho = C(1) + drho;
  C ir = C(1) / rho;
  ux = (mx + C(0.5) * Fx) * ir;
  uy = (my + C(0.5) * Fy) * ir;
  uz = (mz + C(0.5) * Fz) * ir;
  C usq = ux * ux + uy * uy + uz * uz;
  C uF = ux * Fx + uy * Fy + uz * Fz;
  C kf = C(1) - C(0.5) * omega;
#pragma unroll
  for (int i = 0; i < 19; i++) {
    C eu = eterm(EX[i], ux) + eterm(EY[i], uy) + eterm(EZ[i], uz);
    C eF = eterm(EX[i], Fx) + eterm(EY[i], Fy) + eterm(EZ[i], Fz);
    C w = C(WD[i]);
    C geq = w * (drho + rho * (C(3) * eu + C(4.5) * eu * eu - C(1.5) * usq));
    C Gi = kf * w * (C(3) * (eF - uF) + C(9) * eu * eF);
    g[i] = g[i] - omega * (g[i] - geq) + Gi;
  }
  if constexpr (sizeof(C) < sizeof(double)) {
    // The collision keeps the mass (rho - 1) and turns the momentum m into
    // m + F exactly; with the weights rounded to float it does not (their
    // sums are off by ~1e-8, the same sign at every node and step), so the
    // residuals are put back: mass on the rest population, momentum on the
    // axis pairs.
    const C mx1 = (g[1] - g[2]) + (g[7] + g[8]) + (g[9] + g[10]) - (g[11] + g[12]) - (g[13] + g[14]);
    const C my1 = (g[3] - g[4]) + (g[7] - g[8]) + (g[11] - g[12]) + (g[15] + g[16]) - (g[17] + g[18]);
    const C mz1 = (g[5] - g[6]) + (g[9] - g[10]) + (g[13] - g[14]) + (g[15] - g[16]) + (g[17] - g[18]);
    const C rx = C(0.5) * ((mx + Fx) - mx1), ry = C(0.5) * ((my + Fy) - my1), rz = C(0.5) * ((mz + Fz) - mz1);
    g[1] += rx;
    g[2] -= rx;
    g[3] += ry;
    g[4] -= ry;
    g[5] += rz;
    g[6] -= rz;
    g[0] += drho - dev_sum(g);
  }
}

// ----------------------------------------------------- boundary nodes (S1/S2)
template <class S>
__device__ __forceinline__ typename Store<S>::C ldA(const FluidArgs& a, int j, long long node) {
  return to_c(((const S*)a.A)[(long long)j * a.g.plane + node]);
}

// Zou-He on an open face (Eq. extbound, general inward normal n = s e_ax),
// on deviations: rho_w = (1 + G0 + 2 Gout)/(1 - u_n) for a velocity face,
// u_n = (rho_w - 1 - G0 - 2 Gout)/rho_w for a density face (tangential u = 0);
// unknowns (e.n = +1): axis  g = g_opp + rho_w/3 u_n,
// diagonal e = n + t: g = g_opp + rho_w/6 (u_n + u.t) - N_t with
// N_t = 1/2 sum_{e.n = 0} g (e.t) - rho_w/3 u.t.  Written with selects on the
// runtime face so that the code stays small.
template <class C>
__device__ void zouhe(C (&g)[19], int face, int kind, C bx, C by, C bz, C brho) {
  const int ax = face >> 1;
  const int s = (face & 1) ? -1 : 1;
  C G0 = 0, Gout = 0, T[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < 19; j++) {
    const int e_ax = ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j]);
    const int en = s * e_ax;
    G0 += en == 0 ? g[j] : C(0);
    Gout += en == -1 ? g[j] : C(0);
    if (EX[j]) T[0] += en == 0 ? C(EX[j]) * g[j] : C(0);
    if (EY[j]) T[1] += en == 0 ? C(EY[j]) * g[j] : C(0);
    if (EZ[j]) T[2] += en == 0 ? C(EZ[j]) * g[j] : C(0);
  }
  C u[3] = {bx, by, bz};
  C rho, un;
  if (kind == 0) {
    un = C(s) * (ax == 0 ? u[0] : (ax == 1 ? u[1] : u[2]));
    rho = (C(1) + G0 + C(2) * Gout) / (C(1) - un);
  } else {
    rho = brho;
    un = (rho - C(1) - G0 - C(2) * Gout) / rho;
    u[0] = ax == 0 ? C(s) * un : C(0);
    u[1] = ax == 1 ? C(s) * un : C(0);
    u[2] = ax == 2 ? C(s) * un : C(0);
  }
  C N[3];
#pragma unroll
  for (int k = 0; k < 3; k++) N[k] = C(0.5) * T[k] - rho / C(3) * u[k];
  C out[19];
#pragma unroll
  for (int j = 0; j < 19; j++) {
    const int e_ax = ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j]);
    // tangential part t = e_j - n (zero on the normal axis)
    const C tx = ax == 0 ? C(0) : C(EX[j]), ty = ax == 1 ? C(0) : C(EY[j]), tz = ax == 2 ? C(0) : C(EZ[j]);
    const C ut = u[0] * tx + u[1] * ty + u[2] * tz;
    const C Nt = N[0] * tx + N[1] * ty + N[2] * tz;
    const bool axis = tx == C(0) && ty == C(0) && tz == C(0);
    const C fill = axis ? g[OPP[j]] + rho / C(3) * un : g[OPP[j]] + rho / C(6) * (un + ut) - Nt;
    out[j] = (s * e_ax == 1) ? fill : g[j];
  }
#pragma unroll
  for (int j = 0; j < 19; j++) g[j] = out[j];
}

// Interpolated bounce-back of the linked direction j at node x (Eq.
// bbouzidi): k0 f*_i(x) + k1 t1 + k2 t2 with i the opposite of j and, by the
// link's branch, t1 = f*_i(x - e_i), t2 = f*_i(x - 2e_i) (q < 1/2) or
// t1 = f*_j(x), t2 = f*_j(x - e_i) (q >= 1/2); k1, k2 are zero where the
// fluid neighbours are missing.

// Direction arithmetic for a direction known only at run time: the
// components of e_j (two bits each, biased by one) and the opposite.
constexpr unsigned long long dir_bits(const int (&e)[19]) {
  unsigned long long b = 0;
  for (int j = 0; j < 19; j++) b |= (unsigned long long)(e[j] + 1) << (2 * j);
  return b;
}
__device__ __forceinline__ int dir_of(unsigned long long bits, int j) { return (int)((bits >> (2 * j)) & 3u) - 1; }
__device__ __forceinline__ int opp_of(int j) {
  return j < 7 ? ((j - 1) ^ 1) + 1 : (j < 15 ? 7 + ((j - 7) ^ 5) : 15 + ((j - 15) ^ 3));
}

// Streamed populations of a block of boundary records, one record per thread
// (record r0 + threadIdx.x; every thread of the block calls, those past the
// last record repeat it): plain pulls (periodic wrap), interpolated
// bounce-back on wall links, and Zou-He for the populations entering through
// an open face.
//
// A record has 4 to 5 links on average out of 18 directions.  Issued per
// record and direction, the rule's six loads made 133 loads per thread (and
// the registers to hold them) where about 45 are needed.  Here the links of
// the block's records, which are consecutive, are spread over its threads,
// one link per thread and pass: the link's node and word (direction, branch),
// then its coefficients and three populations, its value out to LDS, where
// the record picks it up.  The words of LINK_PASSES passes are loaded in one
// batch ahead of the plain pulls, and their populations in one batch after
// them, so that a block waits for the same few rounds of loads whatever its
// number of links.  A plain pull from a solid node or from outside the box
// reads the node's own rest value (no traffic) and is not used.
// Measured against the per-record form (record launch of the D = 96 pipe in
// FP16S 73 -> 49 us; the merged launch of a ten-instance sweep 77 -> 69 us,
// of the 16-capsule channel 52.6 -> 50.3 us, of the bifurcation with one
// capsule 15.0 -> 14.5 us).  Links in padded groups per wave, whose words
// need no start index, were slower (15.6 us there): the padding costs more
// passes than the saved wait.
//
// s_dyn (dynamic LDS): the links of the fullest block of this size.
extern __shared__ double s_dyn[];
constexpr int LINK_PASSES = 5;

template <class S, int NP>
__device__ __forceinline__ void link_values(const FluidArgs& a, int l0, int l1, int first, const int (&nd)[NP],
                                            const unsigned int (&w)[NP], typename Store<S>::C* s_link) {
  typedef typename Store<S>::C C;
  const Grid& G = a.g;
  const S* A = (const S*)a.A;
  const C* lc = (const C*)a.lk_c;
  const long long nl = a.nlinks;
  int n1[NP], n2[NP];  // x - e_i, x - 2 e_i where they are fluid nodes, else x
  const bool per = G.per[0] | G.per[1] | G.per[2];
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int j = w[p] & 31u;
    const int ex = dir_of(dir_bits(EX), j), ey = dir_of(dir_bits(EY), j), ez = dir_of(dir_bits(EZ), j);
    const int d = ex + G.px * (ey + G.ny * ez);
    n1[p] = nd[p] + d;
    n2[p] = nd[p] + 2 * d;
  }
  if (per) {
#pragma unroll 1
    for (int p = 0; p < NP; p++) {
      const int j = w[p] & 31u;
      const int ex = dir_of(dir_bits(EX), j), ey = dir_of(dir_bits(EY), j), ez = dir_of(dir_bits(EZ), j);
      int x, y, z;
      coords(G, nd[p], x, y, z);
      n1[p] = (int)nbr(G, x, y, z, ex, ey, ez);
      n2[p] = (int)nbr(G, x, y, z, 2 * ex, 2 * ey, 2 * ez);
    }
  }
  C k0[NP], k1[NP], k2[NP], v0[NP], v1[NP], v2[NP];
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int l = max(min(first + p * (int)blockDim.x, l1 - 1), 0);
    const int j = w[p] & 31u, i = opp_of(j);
    const bool hq = (w[p] >> 5) & 1u, h1 = (w[p] >> 6) & 1u, h2 = (w[p] >> 7) & 1u;
    const int m1 = h1 ? n1[p] : nd[p], m2 = h2 ? n2[p] : nd[p];
    const S* Ai = A + (long long)i * G.plane;
    const S* At = hq ? A + (long long)j * G.plane : Ai;
    v0[p] = to_c(Ai[nd[p]]);
    v1[p] = to_c(At[hq ? nd[p] : m1]);
    v2[p] = to_c(At[hq ? m1 : m2]);
    k0[p] = lc[l];
    k1[p] = lc[nl + l];
    k2[p] = lc[2 * nl + l];
  }
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int l = first + p * (int)blockDim.x;
    if (l < l1) s_link[l - l0] = k0[p] * v0[p] + k1[p] * v1[p] + k2[p] * v2[p];
  }
}

template <class S>
__device__ __forceinline__ void pull_records(const FluidArgs& a, int r0, typename Store<S>::C (&g)[19], int& node,
                                             bool& on, bool& flagged) {
  typedef typename Store<S>::C C;
  const Grid& G = a.g;
  const S* A = (const S*)a.A;
  const int t = threadIdx.x, nt = (int)blockDim.x;
  C* s_link = (C*)s_dyn;
  on = r0 + t < a.nrec;
  const int r = on ? r0 + t : a.nrec - 1;
  const int l0 = a.rec_link0[r0], l1 = a.rec_link0[min(r0 + nt, a.nrec)];
  node = a.rec_node[r];
  const uint32_t mask = a.rec_mask[r];
  const int lk0 = a.rec_link0[r];
  const int fc = a.rec_face[r];
  int nd[LINK_PASSES];
  unsigned int w[LINK_PASSES];
#pragma unroll
  for (int p = 0; p < LINK_PASSES; p++) {
    const int l = max(min(l0 + t + p * nt, l1 - 1), 0);
    nd[p] = a.lk_node[l];
    w[p] = a.lk_w[l];
  }
  // what comes after the pulls is loaded with them: the node's force flag and
  // the imposed values of an open face
  const uint8_t tfl = a.tflag ? a.tflag[node >> TILE_SHIFT] : 0;
  double bc[4] = {0.0, 0.0, 0.0, 0.0};
  if (fc != 0xff) {
#pragma unroll
    for (int k = 0; k < 4; k++) bc[k] = a.rec_bc[(long long)k * a.nrec + r];
  }
  int x, y, z;
  coords(G, node, x, y, z);
  const int face = fc & 7, kind = (fc >> 4) & 1;
  const int ax = face >> 1, s = (face & 1) ? -1 : 1;
  C pl[19];
  {
    const Hood h = hood(G, x, y, z);
    pl[0] = ldA<S>(a, 0, node);
#pragma unroll
    for (int j = 1; j < 19; j++) {
      const bool unknown = fc != 0xff && s * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j])) == 1;
      const bool plain = !((mask >> j) & 1u) && !unknown;
      pl[j] = to_c(A[plain ? (long long)j * G.plane + h.at(-EX[j], -EY[j], -EZ[j]) : (long long)node]);
    }
  }
  link_values<S, LINK_PASSES>(a, l0, l1, l0 + t, nd, w, s_link);
  for (int l = l0 + t + LINK_PASSES * nt; l < l1; l += nt) {  // a block with more links than the batch holds
    const int nd1[1] = {a.lk_node[l]};
    const unsigned int w1[1] = {a.lk_w[l]};
    link_values<S, 1>(a, l0, l1, l, nd1, w1, s_link);
  }
  __syncthreads();
  g[0] = pl[0];
#pragma unroll
  for (int j = 1; j < 19; j++) {
    const bool linked = (mask >> j) & 1u;
    const bool unknown = fc != 0xff && s * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j])) == 1;
    g[j] = unknown ? C(0) : pl[j];
    if (linked) g[j] = s_link[lk0 - l0 + __popc(mask & ((1u << j) - 1u))];
  }
  if (fc != 0xff) {
    zouhe<C>(g, face, kind, (C)bc[0], (C)bc[1], (C)bc[2], (C)bc[3]);
  }
  flagged = tfl != 0;
}

template <class C>
__device__ __forceinline__ void node_force(const FluidArgs& a, long long node, bool flagged, C& Fx,
                                           C& Fy, C& Fz) {
  double fx = a.gx, fy = a.gy, fz = a.gz;
  if (flagged) {
    fx += (double)a.fx[node] * FX_INV;
    fy += (double)a.fx[a.g.Np + node] * FX_INV;
    fz += (double)a.fx[2 * a.g.Np + node] * FX_INV;
  }
  Fx = (C)fx;
  Fy = (C)fy;
  Fz = (C)fz;
}

// ------------------------------------------------------------ step closing
// Blocks of a kernel that closes a piece of work count themselves on a
// device counter; the last one to arrive combines the kernel's results.
// No agent-scope fence (on gfx950 that writes back the whole L2): the few
// values the last block reads are written with device-coherent atomic
// stores or read-modify-writes, and each writing wave waits for them to
// complete before its block is counted.
__device__ __forceinline__ void wait_mem() { __builtin_amdgcn_s_waitcnt(0); }

__device__ __forceinline__ void store_coherent(double* p, double v) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_coherent(const double* p) {
  return __longlong_as_double((long long)__hip_atomic_load((unsigned long long*)p, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT));
}

__device__ __forceinline__ void raise_pending(DevFlags* flags, int par, unsigned int bits) {
  atomicOr(par ? &flags->pend1 : &flags->pend0, bits);
}

// Non-zero when the run stopped before this step: a sticky bit, or one that
// the previous step raised.
__device__ __forceinline__ unsigned int halted_before(const DevFlags* flags, int par) {
  const uint4 w = *(const uint4*)flags;  // stop, pend0, check, pend1
  return w.x | (par ? w.y : w.w);
}
// The same for the launches after the step's forcing, whose position check may
// have stopped it as well.
__device__ __forceinline__ unsigned int halted(const DevFlags* flags, int par) {
  const uint4 w = *(const uint4*)flags;
  return w.x | w.z | (par ? w.y : w.w);
}

// Closes a step, by one thread of its last launch (halt: halted() as that
// launch saw it).
__device__ __forceinline__ void close_step(DevFlags* flags, unsigned int halt) {
  if (halt) atomicOr(&flags->stop, halt);
  else flags->steps_done += 1;
}

__device__ __forceinline__ bool last_block(unsigned int* counter, unsigned int nblocks) {
  __shared__ int is_last;
  wait_mem();
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned int done = atomicAdd(counter, 1u);
    is_last = (done == nblocks - 1);
  }
  __syncthreads();
  return is_last != 0;
}

// ------------------------------------------------------------- k_fluid
// One thread = V consecutive nodes of a row.  The populations carry guard
// regions of one z-plane plus one row on both sides, so the 19 vector loads
// stay inside the allocation for any group; values pulled for solid or
// boundary-record nodes are computed and discarded.
template <class S, int V, bool PERX>
__device__ void fluid_bulk(const FluidArgs& a, int blk, unsigned int halt) {
  typedef typename Store<S>::C C;
  typedef typename Vec<S, V>::a vec;
  typedef typename Vec<S, V>::u vecu;
  const Grid& G = a.g;
  long long base;
  if (V == 1 && a.bulk_list) {
    // list form: one bulk node per thread from the sorted list of bulk
    // nodes (no idle lanes on sparse geometries; runs along x stay coalesced)
    const long long i = (long long)blk * blockDim.x + threadIdx.x;
    if (i >= a.nbulk_nodes) return;
    base = a.bulk_list[i];
  } else {
    const long long tile = a.tile_list[blk];
    base = tile * ((long long)blockDim.x * V) + (long long)threadIdx.x * V;
  }
  if (base >= G.Np) return;
  bool isb[V];
  bool all = true, any = false;
  if (V == 1 && a.bulk_list) {
    isb[0] = any = true;  // the list holds bulk nodes only
  } else {
    const typename ClsWord<V>::T cw = *(const typename ClsWord<V>::T*)(a.ncls + base);
#pragma unroll
    for (int k = 0; k < V; k++) {
      isb[k] = ((cw >> (8 * k)) & 0xff) == CLS_BULK;
      all = all && isb[k];
      any = any || isb[k];
    }
  }
  if (!any) return;
  const uint8_t tfl = a.tflag ? a.tflag[base >> TILE_SHIFT] : 0;
  const S* A = (const S*)a.A;
  S* B = (S*)a.B;
  const C omega = (C)a.omega;
  int x0, y, z;
  coords_ms(G, base, x0, y, z);
  // The nine source rows (y - e_y, z - e_z), wrapped once on periodic axes
  // (on closed ones the guard rows take the discarded pulls), as element
  // offsets from the start of a plane: padded indices, guards included,
  // stay inside int range (checked when the lattice is created).
  int rows[3][3];
  {
    const int pxy = G.px * G.ny;
    int ty[3], tz[3];
#pragma unroll
    for (int d = 0; d < 3; d++) {
      ty[d] = G.px * (G.per[1] ? wrap2(y + d - 1, G.ny) : y + d - 1);
      tz[d] = pxy * (G.per[2] ? wrap2(z + d - 1, G.nz) : z + d - 1);
    }
#pragma unroll
    for (int dz = 0; dz < 3; dz++)
#pragma unroll
      for (int dy = 0; dy < 3; dy++) rows[dz][dy] = (ty[dy] + x0) + tz[dz];
  }
  // periodic x: groups touching x = 0 or x = nx-1 gather element by element
  const bool xedge = PERX && (x0 == 0 || x0 + V > G.nx - 1);
  vec in[19];
  if (!PERX || !xedge) {
#pragma unroll
    for (int j = 0; j < 19; j++) {
      const S* pl = A + (long long)j * G.plane;
      const int o = rows[1 - EZ[j]][1 - EY[j]];
      if (EX[j] == 0)
        in[j] = *(const vec*)(pl + o);
      else
        in[j] = *(const vecu*)(pl + (o - EX[j]));
    }
  } else {
#pragma unroll
    for (int j = 0; j < 19; j++) {
      const S* pl = A + (long long)j * G.plane + (rows[1 - EZ[j]][1 - EY[j]] - x0);
#pragma unroll
      for (int k = 0; k < V; k++) in[j][k] = pl[wrap2(x0 + k - EX[j], G.nx)];
    }
  }
  if (halt) return;
  const bool flagged = tfl != 0;
  bool bad = false;
#pragma unroll
  for (int k = 0; k < V; k++) {
    C g[19];
#pragma unroll
    for (int j = 0; j < 19; j++) g[j] = to_c(in[j][k]);
    C Fx, Fy, Fz, drho, ux, uy, uz;
    node_force<C>(a, base + k, flagged && isb[k], Fx, Fy, Fz);
    collide<C>(g, Fx, Fy, Fz, omega, drho, ux, uy, uz);
    if (a.mac && isb[k]) store_mac<C>(a, base + k, drho, ux, uy, uz);
    bad = bad || (isb[k] && !(ux * ux + uy * uy + uz * uz <= C(0.09)));
#pragma unroll
    for (int j = 0; j < 19; j++) in[j][k] = (S)g[j];
  }
  const int b32 = (int)base;
  if (all) {
#pragma unroll
    for (int j = 0; j < 19; j++) *(vec*)(B + (long long)j * G.plane + b32) = in[j];
  } else {
#pragma unroll
    for (int j = 0; j < 19; j++)
#pragma unroll
      for (int k = 0; k < V; k++)
        if (isb[k]) B[(long long)j * G.plane + (b32 + k)] = in[j][k];
  }
  if (bad) raise_pending(a.flags, a.par, ST_UNSTABLE);
}

// Marks the solid nodes of the macro field (and the padding), which the
// fluid launches never write: the fits tell them by it.
template <class C>
__global__ void k_mac_solid(Grid G, C* mac, const uint8_t* ncls) {
  const long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (p < G.Np && ncls[p] == CLS_SOLID) mac[4 * p] = C(MAC_SOLID);
}

// This step's rho - 1 and u at a node (what the probes and the vertex
// velocities interpolate), [Np][4] in the compute type.
template <class C>
__device__ __forceinline__ void store_mac(const FluidArgs& a, long long node, C drho, C ux, C uy, C uz) {
  typedef C C4 __attribute__((ext_vector_type(4)));
  C4 v;
  v.x = drho;
  v.y = ux;
  v.z = uy;
  v.w = uz;
  ((C4*)a.mac)[node] = v;
}

template <class S>
__device__ __forceinline__ void load_mac(const FluidArgs& a, long long node, double& drho, double& ux,
                                         double& uy, double& uz) {
  typedef typename Store<S>::C C;
  typedef C C4 __attribute__((ext_vector_type(4)));
  const C4 v = ((const C4*)a.mac)[node];
  drho = (double)v.x;
  ux = (double)v.y;
  uy = (double)v.z;
  uz = (double)v.w;
}

// A block of boundary records: pull_records, then the forced collision, one
// record per thread.  Consecutive records are consecutive nodes, so the
// loads of a wave are coalesced along x.
template <class S>
__device__ void fluid_record_block(const FluidArgs& a, int blk, unsigned int halt) {
  typedef typename Store<S>::C C;
  C g[19];
  int node;
  bool on, flagged;
  pull_records<S>(a, blk * (int)blockDim.x, g, node, on, flagged);
  if (!on || halt) return;
  C Fx, Fy, Fz, drho, ux, uy, uz;
  node_force<C>(a, node, flagged, Fx, Fy, Fz);
  collide<C>(g, Fx, Fy, Fz, (C)a.omega, drho, ux, uy, uz);
  if (a.mac) store_mac<C>(a, node, drho, ux, uy, uz);
  S* B = (S*)a.B;
#pragma unroll
  for (int j = 0; j < 19; j++) B[(long long)j * a.g.plane + node] = (S)g[j];
  if (!(ux * ux + uy * uy + uz * uz <= C(0.09))) raise_pending(a.flags, a.par, ST_UNSTABLE);
}

// The bulk tiles and the boundary records are two kernels: the records
// need several times the registers of the bulk path, and sharing one kernel
// would cap the occupancy of the bandwidth-bound part.  The two launches
// read A and write disjoint nodes of B and may run concurrently.
template <class S, int V, bool PERX>
__global__ __launch_bounds__(256) void k_fluid_bulk(FluidArgs a) {
  const unsigned int halt = halted(a.flags, a.par);
  if (a.close_step == 1 && blockIdx.x == 0 && threadIdx.x == 0) close_step(a.flags, halt);
  fluid_bulk<S, V, PERX>(a, xcd_remap(blockIdx.x, a.nbulk_blocks), halt);
}

template <class S>
__global__ __launch_bounds__(256) void k_fluid_rec(FluidArgs a) {
  const unsigned int halt = halted(a.flags, a.par);
  if (a.close_step == 2 && blockIdx.x == 0 && threadIdx.x == 0) close_step(a.flags, halt);
  fluid_record_block<S>(a, xcd_remap(blockIdx.x, gridDim.x), halt);
}

// Small (cache-resident, latency-bound) grids: records and bulk tiles in one
// launch, the record blocks first (they take longest), so that a step has
// no fork and join between two streams.  Both parts use blocks of the same
// size.
template <class S, int V, bool PERX>
__device__ __forceinline__ void fluid_unit(const FluidArgs& a, int nrb, int u, unsigned int halt) {
  if (u < nrb) fluid_record_block<S>(a, u, halt);
  else fluid_bulk<S, V, PERX>(a, u - nrb, halt);
}

template <class S, int V, bool PERX>
__global__ __launch_bounds__(256) void k_fluid_all(FluidArgs a, int nrb) {
  const int b = blockIdx.x;
  const unsigned int halt = halted(a.flags, a.par);
  if (a.close_step && b == (a.close_step == 1 ? nrb : 0) && threadIdx.x == 0) close_step(a.flags, halt);
  fluid_unit<S, V, PERX>(a, nrb, b < nrb ? xcd_remap(b, nrb) : nrb + xcd_remap(b - nrb, a.nbulk_blocks), halt);
}

// Closes a step that no launch of its own closes (one thread): a lattice
// without fluid nodes, and the adjoint's recomputed steps, which all run at
// parity 0.
__global__ void k_close(DevFlags* flags) {
  if (flags->stop) return;
  if (flags->check) {
    flags->stop = flags->check;
    return;
  }
  flags->steps_done += 1;
  flags->stop = flags->pend0 | flags->pend1;
  flags->pend0 = flags->pend1 = 0u;
}

// ---------------------------------------------------------------- init
template <class S>
__global__ void k_init(Grid G, S* f, const uint8_t* ncls, const double* rho0, const double* u0) {
  long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (n >= (long long)G.nx * G.ny * G.nz) return;
  int x = (int)(n % G.nx);
  long long t = n / G.nx;
  int y = (int)(t % G.ny), z = (int)(t / G.ny);
  long long p = x + (long long)G.px * (y + (long long)G.ny * z);
  const long long N = (long long)G.nx * G.ny * G.nz;
  double r = rho0 ? rho0[n] : 1.0;
  double ux = u0 ? u0[n] : 0.0, uy = u0 ? u0[N + n] : 0.0, uz = u0 ? u0[2 * N + n] : 0.0;
  bool solid = ncls[p] == CLS_SOLID;
  double usq = ux * ux + uy * uy + uz * uz;
  for (int i = 0; i < 19; i++) {
    double eu = EX[i] * ux + EY[i] * uy + EZ[i] * uz;
    double geq = WD[i] * ((r - 1.0) + r * (3.0 * eu + 4.5 * eu * eu - 1.5 * usq));
    f[(long long)i * G.plane + p] = solid ? (S)0 : (S)geq;
  }
}

// -------------------------------------------------------------------- MLS
// 32 lanes per point; lane k < 27 owns the stencil node b + (k%3-1,
// (k/3)%3-1, k/9-1) with b = floor(p + 1/2) (Eqs. uLag, l2norm, intKernel):
// W = exp(-(r/0.3)^2), r = |x_k - p| / 2.6, linear basis (1, x_k - p); solid
// nodes and nodes outside a non-periodic face are excluded.
struct Slot {
  long long node;
  double W, dx, dy, dz;
  int cx, cy, cz;  // node coordinates before periodic wrap
  bool valid;
};

__device__ __forceinline__ Slot stencil_slot(const Grid& G, const uint8_t* ncls, double X,
                                             double Y, double Z, int k) {
  Slot s;
  s.valid = false;
  s.W = 0.0;
  s.node = 0;
  s.dx = s.dy = s.dz = 0.0;
  if (k >= 27) return s;
  const int bx = (int)floor(X + 0.5), by = (int)floor(Y + 0.5), bz = (int)floor(Z + 0.5);
  int c[3] = {bx + k % 3 - 1, by + (k / 3) % 3 - 1, bz + k / 9 - 1};
  s.cx = c[0];
  s.cy = c[1];
  s.cz = c[2];
  s.dx = c[0] - X;
  s.dy = c[1] - Y;
  s.dz = c[2] - Z;
  const int dim[3] = {G.nx, G.ny, G.nz};
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    if (c[a] < 0 || c[a] >= dim[a]) {
      if (G.per[a]) c[a] = ((c[a] % dim[a]) + dim[a]) % dim[a];
      else ok = false;
    }
  }
  if (ok) {
    s.node = c[0] + (long long)G.px * (c[1] + (long long)G.ny * c[2]);
    ok = ncls[s.node] != CLS_SOLID;
  }
  const double r = sqrt(s.dx * s.dx + s.dy * s.dy + s.dz * s.dz) / 2.6;
  s.W = (ok && r <= 1.0) ? exp(-(r / 0.3) * (r / 0.3)) : 0.0;
  s.valid = ok;
  return s;
}

__device__ __forceinline__ double red32(double v) {
#pragma unroll
  for (int m = 16; m >= 1; m >>= 1) v += __shfl_xor(v, m, 32);
  return v;
}
__device__ __forceinline__ double red64(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Moment matrix A = sum W p p^T over the 32-lane group, Cholesky, and
// psi = W A^{-1} p for this lane (psi[0] = phi).  Singular (pivot below
// 1e-10 of the largest diagonal): psi = 0, returns false.
__device__ bool mls_psi(const Slot& s, double (&psi)[4]) {
  const double P[4] = {1.0, s.dx, s.dy, s.dz};
  double A[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = i; j < 4; j++) {
      A[i][j] = red32(s.W * P[i] * P[j]);
      A[j][i] = A[i][j];
    }
  double dmax = fmax(fmax(A[0][0], A[1][1]), fmax(A[2][2], A[3][3]));
  double L[4][4] = {{0}};
  bool ok = dmax > 0.0;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    double d = A[j][j];
#pragma unroll
    for (int k = 0; k < j; k++) d -= L[j][k] * L[j][k];
    if (!(d > 1e-10 * dmax)) ok = false;
    L[j][j] = ok ? sqrt(d) : 1.0;
#pragma unroll
    for (int i = j + 1; i < 4; i++) {
      double v = A[i][j];
#pragma unroll
      for (int k = 0; k < j; k++) v -= L[i][k] * L[j][k];
      L[i][j] = v / L[j][j];
    }
  }
  if (!ok) {
    psi[0] = psi[1] = psi[2] = psi[3] = 0.0;
    return false;
  }
  // y = L^{-1} P, psi = W L^{-T} y
  double y[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    double v = P[i];
#pragma unroll
    for (int k = 0; k < i; k++) v -= L[i][k] * y[k];
    y[i] = v / L[i][i];
  }
  double z[4];
#pragma unroll
  for (int i = 3; i >= 0; i--) {
    double v = y[i];
#pragma unroll
    for (int k = i + 1; k < 4; k++) v -= L[k][i] * z[k];
    z[i] = v / L[i][i];
  }
#pragma unroll
  for (int i = 0; i < 4; i++) psi[i] = s.W * z[i];
  return true;
}

// Post-collision macroscopic fields at a node: rho = sum f*, and the
// velocity of the step u = (sum f* e - F/2)/rho (the collision adds F to the
// momentum).
template <class S>
__device__ __forceinline__ void macro_at(const Grid& G, const S* f, const long long* fx,
                                         const uint8_t* tf, double gx, double gy, double gz,
                                         long long node, double& rho, double& ux, double& uy,
                                         double& uz) {
  // moments in double whatever the storage (off the bandwidth-bound path)
  double g[19];
#pragma unroll
  for (int j = 0; j < 19; j++) g[j] = (double)to_c(f[(long long)j * G.plane + node]);
  const double drho = dev_sum(g);
  const double mx = (g[1] - g[2]) + (g[7] + g[8]) + (g[9] + g[10]) - (g[11] + g[12]) - (g[13] + g[14]);
  const double my = (g[3] - g[4]) + (g[7] - g[8]) + (g[11] - g[12]) + (g[15] + g[16]) - (g[17] + g[18]);
  const double mz = (g[5] - g[6]) + (g[9] - g[10]) + (g[13] - g[14]) + (g[15] - g[16]) + (g[17] - g[18]);
  double Fx = gx, Fy = gy, Fz = gz;
  if (fx && tf && tf[node >> TILE_SHIFT]) {
    Fx += (double)fx[node] * FX_INV;
    Fy += (double)fx[G.Np + node] * FX_INV;
    Fz += (double)fx[2 * G.Np + node] * FX_INV;
  }
  rho = 1.0 + (double)drho;
  ux = ((double)mx - 0.5 * Fx) / rho;
  uy = ((double)my - 0.5 * Fy) / rho;
  uz = ((double)mz - 0.5 * Fz) / rho;
}

__device__ __forceinline__ void face_geom_pts(const double (&pa)[3], const double (&pb)[3],
                                              const double (&pd)[3], double (&c)[3], double (&n)[3],
                                              double& area) {
  double u[3] = {pb[0] - pa[0], pb[1] - pa[1], pb[2] - pa[2]};
  double v[3] = {pd[0] - pa[0], pd[1] - pa[1], pd[2] - pa[2]};
  double N[3] = {u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]};
  const double q = N[0] * N[0] + N[1] * N[1] + N[2] * N[2];
  const double l = sqrt(q), il = 1.0 / l;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    c[k] = (pa[k] + pb[k] + pd[k]) * (1.0 / 3.0);
    n[k] = N[k] * il;
  }
  area = 0.5 * l;
}

__device__ __forceinline__ void face_geom(const double* X, const int32_t* faces, int f,
                                          double (&c)[3], double (&n)[3], double& area) {
  const int a = faces[3 * f], b = faces[3 * f + 1], d = faces[3 * f + 2];
  double pa[3], pb[3], pd[3];
#pragma unroll
  for (int k = 0; k < 3; k++) {
    pa[k] = X[3 * a + k];
    pb[k] = X[3 * b + k];
    pd[k] = X[3 * d + k];
  }
  face_geom_pts(pa, pb, pd, c, n, area);
}

__device__ __forceinline__ void cross3(const double* a, const double* b, double* c) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}

// Signed dihedral angle of hinge (a, b, c, d) (faces (a,b,c) and (b,a,d),
// outward normals, positive for a convex fold) and its gradient with
// respect to the four vertices: the wing gradients are -|e| n/|n|^2; the
// edge-end gradients follow from translation and rotation invariance.
__device__ void hinge_all(const double* X, const int32_t* h, double& theta, double (&gr)[4][3]) {
  const double* pa = X + 3 * h[0];
  const double* pb = X + 3 * h[1];
  const double* pc = X + 3 * h[2];
  const double* pd = X + 3 * h[3];
  double e[3], ca[3], da[3], ab[3], db[3], n1[3], n2[3];
  for (int k = 0; k < 3; k++) {
    e[k] = pb[k] - pa[k];
    ca[k] = pc[k] - pa[k];
    da[k] = pd[k] - pa[k];
    ab[k] = pa[k] - pb[k];
    db[k] = pd[k] - pb[k];
  }
  cross3(e, ca, n1);
  cross3(ab, db, n2);
  const double q1 = n1[0] * n1[0] + n1[1] * n1[1] + n1[2] * n1[2];
  const double q2 = n2[0] * n2[0] + n2[1] * n2[1] + n2[2] * n2[2];
  const double le2 = e[0] * e[0] + e[1] * e[1] + e[2] * e[2];
  const double le = sqrt(le2);
  const double l1 = sqrt(q1), l2 = sqrt(q2);
  double m1[3], m2[3], t[3];
  for (int k = 0; k < 3; k++) {
    m1[k] = n1[k] / l1;
    m2[k] = n2[k] / l2;
  }
  cross3(m1, m2, t);
  theta = atan2((t[0] * e[0] + t[1] * e[1] + t[2] * e[2]) / le,
                m1[0] * m2[0] + m1[1] * m2[1] + m1[2] * m2[2]);
  const double al_c = (ca[0] * e[0] + ca[1] * e[1] + ca[2] * e[2]) / le2;
  const double al_d = (da[0] * e[0] + da[1] * e[1] + da[2] * e[2]) / le2;
  for (int k = 0; k < 3; k++) {
    const double gc = -le * n1[k] / q1;
    const double gd = -le * n2[k] / q2;
    gr[0][k] = -((1.0 - al_c) * gc + (1.0 - al_d) * gd);
    gr[1][k] = -(al_c * gc + al_d * gd);
    gr[2][k] = gc;
    gr[3][k] = gd;
  }
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  // deterministic: fixed lane tree in each wave, then fixed order over waves
  v = red64(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  for (int k = 0; k < (int)(blockDim.x >> 6); k++) t += sh[k];
  return t;
}

// ------------------------------------------------------------ diagnostics
// One block of one body (one face, vertex and edge per thread): partial
// volume sum a.(b x c)/6, area, bounding box, NaN and largest stretch
// l/l0 of the positions X, written to diag_part[dblk].
__device__ void diag_block(const BodyArgs& b, const double* X, int dblk) {
  __shared__ double sh[8];
  __shared__ double shm[4][9];
  const int body = b.dblk_body[dblk];
  const int i = (dblk - b.b_dblk0[body]) * 256 + threadIdx.x;
  // reference centre of the bounding sphere (the previous box centre)
  const double* cref = b.b_diag + 16 * body + 13;
  double V = 0.0, S = 0.0, strain = 0.0, nan = 0.0, r2 = 0.0;
  double lo[3] = {DBL_MAX, DBL_MAX, DBL_MAX}, hi[3] = {-DBL_MAX, -DBL_MAX, -DBL_MAX};
  if (i < b.b_nf[body]) {
    const int f = b.b_face0[body] + i;
    const int* F = b.faces + 3 * f;
    double bc[3];
    cross3(X + 3 * F[1], X + 3 * F[2], bc);
    const double* pa = X + 3 * F[0];
    V = (pa[0] * bc[0] + pa[1] * bc[1] + pa[2] * bc[2]) / 6.0;
    double c[3], n[3];
    face_geom(X, b.faces, f, c, n, S);
  }
  if (i < b.b_nv[body]) {
    const int v = b.b_vert0[body] + i;
    for (int k = 0; k < 3; k++) {
      const double c = X[3 * v + k];
      if (!(c == c)) nan = 1.0;
      lo[k] = c;
      hi[k] = c;
      r2 += (c - cref[k]) * (c - cref[k]);
    }
  }
  if (i < b.b_ne[body]) {
    const int e = b.b_edge0[body] + i;
    const int p = b.edges[2 * e], c = b.edges[2 * e + 1];
    const double r[3] = {X[3 * p] - X[3 * c], X[3 * p + 1] - X[3 * c + 1], X[3 * p + 2] - X[3 * c + 2]};
    strain = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]) / b.l0[e];
  }
  V = block_sum(V, sh);
  S = block_sum(S, sh);
  for (int k = 0; k < 3; k++)
    for (int m = 32; m >= 1; m >>= 1) {
      lo[k] = fmin(lo[k], __shfl_xor(lo[k], m, 64));
      hi[k] = fmax(hi[k], __shfl_xor(hi[k], m, 64));
    }
  for (int m = 32; m >= 1; m >>= 1) {
    strain = fmax(strain, __shfl_xor(strain, m, 64));
    nan = fmax(nan, __shfl_xor(nan, m, 64));
    r2 = fmax(r2, __shfl_xor(r2, m, 64));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    for (int k = 0; k < 3; k++) {
      shm[w][k] = lo[k];
      shm[w][3 + k] = hi[k];
    }
    shm[w][6] = strain;
    shm[w][7] = nan;
    shm[w][8] = r2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* P = b.diag_part + 12 * (long long)dblk;
    store_coherent(P, V);
    store_coherent(P + 1, S);
    for (int k = 0; k < 9; k++) {
      double m = shm[0][k];
      for (int q = 1; q < (int)(blockDim.x >> 6); q++) m = (k < 3) ? fmin(m, shm[q][k]) : fmax(m, shm[q][k]);
      store_coherent(P + 2 + k, m);
    }
  }
}

// Combine the partials of every body in block order (run by the last
// block); returns the DAMAGED / UNSTABLE bits found by this thread.
__device__ unsigned int diag_finalize(const BodyArgs& b) {
  unsigned int raised = 0u;
  // one wave per body; its lanes take the partial blocks (all loads in
  // flight at once), then a fixed-order xor reduction
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63, nw = blockDim.x >> 6;
  for (int body = wv; body < b.nbody; body += nw) {
    double V = 0.0, S = 0.0, lo[3], hi[3], strain = 0.0, nan = 0.0, r2 = 0.0;
    for (int k = 0; k < 3; k++) {
      lo[k] = DBL_MAX;
      hi[k] = -DBL_MAX;
    }
    for (int q = b.b_dblk0[body] + ln; q < b.b_dblk0[body + 1]; q += 64) {
      const double* P = b.diag_part + 12 * (long long)q;
      double p[11];
#pragma unroll
      for (int k = 0; k < 11; k++) p[k] = load_coherent(P + k);
      V += p[0];
      S += p[1];
      for (int k = 0; k < 3; k++) {
        lo[k] = fmin(lo[k], p[2 + k]);
        hi[k] = fmax(hi[k], p[5 + k]);
      }
      strain = fmax(strain, p[8]);
      nan = fmax(nan, p[9]);
      r2 = fmax(r2, p[10]);
    }
    V = red64(V);
    S = red64(S);
    for (int m = 32; m >= 1; m >>= 1) {
      for (int k = 0; k < 3; k++) {
        lo[k] = fmin(lo[k], __shfl_xor(lo[k], m, 64));
        hi[k] = fmax(hi[k], __shfl_xor(hi[k], m, 64));
      }
      strain = fmax(strain, __shfl_xor(strain, m, 64));
      nan = fmax(nan, __shfl_xor(nan, m, 64));
      r2 = fmax(r2, __shfl_xor(r2, m, 64));
    }
    if (ln != 0) continue;
    double* d = b.b_diag + 16 * body;
    d[0] = V;
    d[1] = S;
    for (int k = 0; k < 3; k++) {
      d[2 + k] = lo[k];
      d[5 + k] = hi[k];
    }
    d[8] = strain;
    // bounding sphere of the vertices (and so of the face centroids): the
    // reference centre the blocks measured from, and the largest distance;
    // the next reference is this box's centre
    for (int k = 0; k < 3; k++) {
      d[9 + k] = d[13 + k];
      d[13 + k] = 0.5 * (lo[k] + hi[k]);
    }
    d[12] = sqrt(r2);
    // a link whose length doubles its rest length is damaged (computation stops)
    if (!b.b_rigid[body] && strain >= 2.0) raised |= ST_DAMAGED;
    if (nan > 0.0) raised |= ST_UNSTABLE;
  }
  return raised;
}

// ---------------------------------------------------------- k_ib_force
// First launch of a coupled step, three kinds of blocks (the diagnostics first
// in the grid, the elements last):
//  markers   direct forcing at the face centroids (Eqs. uLag, the direct
//            forcing equation, bodyforce): U = sum phi u* with u* = sum f e
//            / rho of the streamed populations (no force), F_l = U_b - U,
//            spread of c_l phi_k F_l (c_l = face area) in fixed point;
//  elements  stretching force per edge (Eq. strainFor) and bending force per
//            hinge, F = -k_b sin(theta - theta0) dtheta/dx (soft bodies);
//  diag      volume, area, bounding box and stretch of x^n; the last block
//            combines them and stops the computation before anything of
//            this step is written when x^n is damaged or not finite.
// Out of the fixed-point range: the step ends as unstable.
__device__ __forceinline__ void fx_over(const FluidArgs& a) {
  atomicOr(&a.flags->overflow, 1u);
  raise_pending(a.flags, a.par, ST_UNSTABLE);
}

__device__ __forceinline__ long long fx_quant(double v, const FluidArgs& a) {
  if (!(fabs(v) <= 1.0)) {
    fx_over(a);
    v = 0.0;
  }
  return __double2ll_rn(v * FX_SCALE);
}

// ---------------------------------------------- MLS, one point per lane
// Support k (0..26) of a point with stencil base bs = floor(p + 1/2) is the
// node bs + (k%3-1, (k/3)%3-1, k/9-1); it is used when it lies in the box
// (periodic faces wrap) and is not solid.
__device__ __forceinline__ bool support_node(const Grid& G, const uint8_t* ncls, int cx, int cy,
                                             int cz, long long& node) {
  int c[3] = {cx, cy, cz};
  const int dim[3] = {G.nx, G.ny, G.nz};
#pragma unroll
  for (int k = 0; k < 3; k++) {
    if (c[k] < 0 || c[k] >= dim[k]) {
      if (!G.per[k]) return false;
      c[k] = ((c[k] % dim[k]) + dim[k]) % dim[k];
    }
  }
  node = c[0] + (long long)G.px * (c[1] + (long long)G.ny * c[2]);
  return ncls[node] != CLS_SOLID;
}

// W = exp(-(r/0.3)^2), r = |x_k - p| / 2.6 (Eqs. l2norm, intKernel).  On
// the 3x3x3 stencil around floor(p + 1/2) every |x_k - p| <= 1.5 sqrt(3)
// < 2.6, so r <= 1 always holds and W factors into one term per axis:
// W = w(dx) w(dy) w(dz) with w(d) = exp(-d^2 / (2.6^2 0.09)); the nine
// per-axis terms of a point are computed once (quad_weights).
constexpr double MLS_K = 1.0 / (2.6 * 2.6 * 0.09);

// Cholesky A = L L^T; singular (a pivot below 1e-10 of the largest
// diagonal) returns false.  r holds 1/L_ii.
struct Chol4 {
  double L[4][4];
  double r[4];
};

__device__ __forceinline__ bool chol4(const double (&A)[10], Chol4& c) {
  const double M[4][4] = {{A[0], A[1], A[2], A[3]},
                          {A[1], A[4], A[5], A[6]},
                          {A[2], A[5], A[7], A[8]},
                          {A[3], A[6], A[8], A[9]}};
  const double dmax = fmax(fmax(A[0], A[4]), fmax(A[7], A[9]));
  bool ok = dmax > 0.0;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    double d = M[j][j];
#pragma unroll
    for (int k = 0; k < j; k++) d -= c.L[j][k] * c.L[j][k];
    if (!(d > 1e-10 * dmax)) ok = false;
    c.r[j] = ok ? rsqrt(d) : 1.0;
#pragma unroll
    for (int i = j + 1; i < 4; i++) {
      double v = M[i][j];
#pragma unroll
      for (int k = 0; k < j; k++) v -= c.L[i][k] * c.L[j][k];
      c.L[i][j] = v * c.r[j];
    }
  }
  return ok;
}

// x = A^{-1} b
__device__ __forceinline__ void chol_solve(const Chol4& c, const double (&b)[4], double (&x)[4]) {
  double y[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    double v = b[i];
#pragma unroll
    for (int k = 0; k < i; k++) v -= c.L[i][k] * y[k];
    y[i] = v * c.r[i];
  }
#pragma unroll
  for (int i = 3; i >= 0; i--) {
    double v = y[i];
#pragma unroll
    for (int k = i + 1; k < 4; k++) v -= c.L[k][i] * x[k];
    x[i] = v * c.r[i];
  }
}

// ------------------------------------------------ forcing markers (S4)
// A block takes MARKERS_PER_BLOCK consecutive faces (neighbouring faces of
// the mesh); four lanes (a quad) serve each marker:
//  1. centroid, area and marker velocity U_b of the face;
//  2. the block's bounding box of support nodes; all its threads compute
//     u* = sum f e / rho of the streamed populations (no force) at every
//     node of the box into LDS;
//  3. per marker: A = sum W p p^T and sum W p u* over the 27 supports, split
//     over the quad (lane q takes supports q, q+4, ...) and combined by a
//     fixed xor tree, one Cholesky, U = e0 . A^{-1} sum W p u*,
//     F_l = U_b - U (Eqs. uLag and the direct-forcing equation);
//  4. spreading (Eq. bodyforce): c_l phi_k F_l with c_l = face area and
//     phi_k = W_k p_k . A^{-1} e0, in fixed point, summed per node in LDS,
//     then one device atomic per node and component (integer sums: the
//     result does not depend on the order).
// A box larger than BOX_CELLS takes the direct path: u* per support from
// global memory and one device atomic per contribution.
__device__ __forceinline__ double sel3(int i, const double (&w)[3]) {
  return i == 0 ? w[0] : (i == 1 ? w[1] : w[2]);
}

// Exchanges inside a quad of lanes as DPP moves (a shuffle would go through
// the LDS pipe): lane i takes the value of lane SEL_i, two bits each in CTRL.
template <int CTRL>
__device__ __forceinline__ double quad_perm(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double quad_sum(double v) {
  v += quad_perm<0xB1>(v);  // lanes 1 0 3 2
  v += quad_perm<0x4E>(v);  // lanes 2 3 0 1
  return v;
}
template <int L>
__device__ __forceinline__ double quad_lane(double v) {
  return quad_perm<0x55 * L>(v);
}

// The nine per-axis weights of a quad's point, three exponentials per lane
// (sub: lane in the quad) instead of nine.
__device__ __forceinline__ void quad_weights(int sub, const double (&p)[3], const int (&base)[3], double (&wx)[3],
                                             double (&wy)[3], double (&wz)[3]) {
  auto w = [](double pa, int ba, int off) {
    const double d = (double)(ba + off - 1) - pa;
    return exp(-(d * d) * MLS_K);
  };
  const double e0 = sub == 3 ? w(p[1], base[1], 0) : w(p[0], base[0], sub);
  const double e1 = w(sub < 2 ? p[1] : p[2], sub < 2 ? base[1] : base[2], sub < 2 ? sub + 1 : sub - 2);
  const double e2 = w(p[2], base[2], 2);
  wx[0] = quad_lane<0>(e0);
  wx[1] = quad_lane<1>(e0);
  wx[2] = quad_lane<2>(e0);
  wy[0] = quad_lane<3>(e0);
  wy[1] = quad_lane<0>(e1);
  wy[2] = quad_lane<1>(e1);
  wz[0] = quad_lane<2>(e1);
  wz[1] = quad_lane<3>(e1);
  wz[2] = e2;
}

// A quad's share of the 27 supports: nine rows of three along x, row r at
// (y, z) offsets (r % 3, r / 3).  Lane sub takes rows sub and sub + 4 and, of
// row 8, the support at x offset sub (lane 3: none).  A row is summed along x
// first, then enters the sums of the fit with its weight in y and z: half the
// operations of adding support by support.
__device__ __forceinline__ void row_yz(int r, int& ky, int& kz) {
  kz = (r >= 3) + (r >= 6);
  ky = r - 3 * kz;
}

// Sums of one row: wx, wx dx, wx dx^2 over its usable supports, and per field
// f the sums of wx f, wx dx f.
template <int NF>
struct RowSums {
  double m0, m1, m2, f0[NF], f1[NF];
  __device__ __forceinline__ void clear() {
    m0 = m1 = m2 = 0.0;
#pragma unroll
    for (int q = 0; q < NF; q++) f0[q] = f1[q] = 0.0;
  }
  __device__ __forceinline__ void add(double w, double d, const double (&f)[NF]) {
    const double wd = w * d;
    m0 += w;
    m1 += wd;
    m2 += wd * d;
#pragma unroll
    for (int q = 0; q < NF; q++) {
      f0[q] += w * f[q];
      f1[q] += wd * f[q];
    }
  }
};

// The moment matrix sum W p p^T with p = (1, dx, dy, dz), packed a00 a01 a02
// a03 a11 a12 a13 a22 a23 a33, and the right-hand sides sum W p f of a fit.
template <int NF>
struct FitSums {
  double A[10], b[NF][4];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < 10; k++) A[k] = 0.0;
#pragma unroll
    for (int q = 0; q < NF; q++)
#pragma unroll
      for (int k = 0; k < 4; k++) b[q][k] = 0.0;
  }
  __device__ __forceinline__ void add(const RowSums<NF>& s, double w, double dy, double dz) {
    const double wy = w * dy, wz = w * dz;
    A[0] += w * s.m0;
    A[1] += w * s.m1;
    A[2] += wy * s.m0;
    A[3] += wz * s.m0;
    A[4] += w * s.m2;
    A[5] += wy * s.m1;
    A[6] += wz * s.m1;
    A[7] += wy * dy * s.m0;
    A[8] += wy * dz * s.m0;
    A[9] += wz * dz * s.m0;
#pragma unroll
    for (int q = 0; q < NF; q++) {
      b[q][0] += w * s.f0[q];
      b[q][1] += w * s.f1[q];
      b[q][2] += wy * s.f0[q];
      b[q][3] += wz * s.f0[q];
    }
  }
  __device__ __forceinline__ void quad() {
#pragma unroll
    for (int k = 0; k < 10; k++) A[k] = quad_sum(A[k]);
#pragma unroll
    for (int q = 0; q < NF; q++)
#pragma unroll
      for (int k = 0; k < 4; k++) b[q][k] = quad_sum(b[q][k]);
  }
};

// The three coordinates base - 1 .. base + 1 on an axis of n nodes as terms
// of a padded index (stride st), and whether they lie in the box (a periodic
// axis wraps; positions may have left the box by any number of periods).
__device__ __forceinline__ void axis_nodes(int base, int n, int periodic, int st, int (&o)[3], bool (&in)[3]) {
  if (periodic && (base < 0 || base >= n)) base = ((base % n) + n) % n;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    int c = base + i - 1;
    in[i] = periodic || (c >= 0 && c < n);
    if (periodic) c = c < 0 ? c + n : (c >= n ? c - n : c);
    o[i] = in[i] ? st * c : 0;
  }
}
__device__ __forceinline__ int sel3i(int i, const int (&w)[3]) { return i == 0 ? w[0] : (i == 1 ? w[1] : w[2]); }
__device__ __forceinline__ bool sel3b(int i, const bool (&w)[3]) { return i == 0 ? w[0] : (i == 1 ? w[1] : w[2]); }

// u* = sum f e / rho of the streamed populations (no force) at the node
// (x, y, z), inside the box, of padded index node; false at a solid node.  The
// 19 plain pulls go out with the node's class; a boundary record then replaces
// those that come from a wall link (three links per batch of loads) and, on an
// open face, takes rho and u from the known populations (Zou-He).  Entries of
// solid nodes are loaded (the class and the links' words would come a round
// earlier than the loads otherwise) but enter no value: in a state of the
// adjoint's sweep they hold whatever the memory held before, NaN included.
template <class S>
__device__ __forceinline__ bool cell_velocity(const FluidArgs& a, int node, int x, int y, int z, double (&u)[3]) {
  typedef typename Store<S>::C C;
  const Grid& G = a.g;
  const S* A = (const S*)a.A;
  const int r = a.rec_of[node];
  S pl[19];
  {
    const int pxy = G.px * G.ny;
    const int xs[3] = {x == 0 ? G.nx - 1 : x - 1, x, x == G.nx - 1 ? 0 : x + 1};
    const int ys[3] = {G.px * (y == 0 ? G.ny - 1 : y - 1), G.px * y, G.px * (y == G.ny - 1 ? 0 : y + 1)};
    const int zs[3] = {pxy * (z == 0 ? G.nz - 1 : z - 1), pxy * z, pxy * (z == G.nz - 1 ? 0 : z + 1)};
#pragma unroll
    for (int j = 0; j < 19; j++)
      pl[j] = (A + (long long)j * G.plane)[xs[1 - EX[j]] + ys[1 - EY[j]] + zs[1 - EZ[j]]];
  }
  if (r == REC_SOLID) return false;
  double g[19], dl = 0.0, ml[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 19; j++) g[j] = (double)to_c(pl[j]);
  if (r >= 0) {
    const uint32_t mask = a.rec_mask[r], hqm = a.rec_mb[r];
    const int lk0 = a.rec_link0[r], fc = a.rec_face[r];
    const int ax = (fc & 7) >> 1, sg = (fc & 1) ? -1 : 1;
    double bc[4] = {0.0, 0.0, 0.0, 0.0};
    if (fc != 0xff) {
#pragma unroll
      for (int k = 0; k < 4; k++) bc[k] = a.rec_bc[(long long)k * a.nrec + r];
    }
    double G0 = 0.0, Gout = 0.0;
    const C* lc = (const C*)a.lk_c;
    const long long nl = a.nlinks;
    uint32_t m = mask;
    for (int l = lk0; m; l += 3) {
      int jj[3];
      C v[3][6];
#pragma unroll
      for (int q = 0; q < 3; q++) {
        const bool on = m != 0;
        const int j = on ? __ffs(m) - 1 : 1;
        jj[q] = on ? j : 0;
        m &= m - 1;
        const int i = opp_of(j), lq = on ? l + q : lk0;
        const bool hq = (hqm >> j) & 1u;
        const int ex = dir_of(dir_bits(EX), j), ey = dir_of(dir_bits(EY), j), ez = dir_of(dir_bits(EZ), j);
        const long long n1 = nbr(G, x, y, z, ex, ey, ez), n2 = nbr(G, x, y, z, 2 * ex, 2 * ey, 2 * ez);
        v[q][0] = lc[lq];
        v[q][1] = lc[nl + lq];
        v[q][2] = lc[2 * nl + lq];
        v[q][3] = ldA<S>(a, i, node);
        v[q][4] = ldA<S>(a, hq ? j : i, hq ? (long long)node : n1);
        v[q][5] = ldA<S>(a, hq ? j : i, hq ? n1 : n2);
      }
#pragma unroll
      for (int q = 0; q < 3; q++) {
        const int j = jj[q];
        // (a zero coefficient drops what it stands at: a node behind that is
        // not fluid, whose entry may hold anything)
        const C t1 = v[q][1] != C(0) ? v[q][4] : C(0), t2 = v[q][2] != C(0) ? v[q][5] : C(0);
        const double w = j ? (double)(v[q][0] * v[q][3] + v[q][1] * t1 + v[q][2] * t2) : 0.0;
        const int ex = dir_of(dir_bits(EX), j), ey = dir_of(dir_bits(EY), j), ez = dir_of(dir_bits(EZ), j);
        const int en = sg * (ax == 0 ? ex : (ax == 1 ? ey : ez));
        dl += w;
        ml[0] += ex * w;
        ml[1] += ey * w;
        ml[2] += ez * w;
        G0 += en == 0 ? w : 0.0;
        Gout += en == -1 ? w : 0.0;
      }
    }
#pragma unroll
    for (int j = 1; j < 19; j++) {
      const int en = sg * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j]));
      if (((mask >> j) & 1u) || (fc != 0xff && en == 1)) g[j] = 0.0;
    }
    if (fc != 0xff) {
#pragma unroll
      for (int j = 0; j < 19; j++) {
        const int en = sg * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j]));
        G0 += en == 0 ? g[j] : 0.0;
        Gout += en == -1 ? g[j] : 0.0;
      }
      double un, ut[3] = {0.0, 0.0, 0.0};
      if (((fc >> 4) & 1) == 0) {
        un = sg * (ax == 0 ? bc[0] : (ax == 1 ? bc[1] : bc[2]));
#pragma unroll
        for (int k = 0; k < 3; k++) ut[k] = bc[k];
      } else {
        un = (bc[3] - 1.0 - G0 - 2.0 * Gout) / bc[3];
      }
#pragma unroll
      for (int k = 0; k < 3; k++) u[k] = k == ax ? sg * un : ut[k];
      return true;
    }
  }
  const double ir = 1.0 / (1.0 + (dev_sum(g) + dl));
  const double mx = (g[1] - g[2]) + (g[7] + g[8]) + (g[9] + g[10]) - (g[11] + g[12]) - (g[13] + g[14]);
  const double my = (g[3] - g[4]) + (g[7] - g[8]) + (g[11] - g[12]) + (g[15] + g[16]) - (g[17] + g[18]);
  const double mz = (g[5] - g[6]) + (g[9] - g[10]) + (g[13] - g[14]) + (g[15] - g[16]) + (g[17] - g[18]);
  u[0] = (mx + ml[0]) * ir;
  u[1] = (my + ml[1]) * ir;
  u[2] = (mz + ml[2]) * ir;
  return true;
}

// Extents e of the box of stencil bases lo..hi (lo <= hi) with the supports
// around them; false when its cells exceed BOX_CELLS.  The differences are
// taken unsigned: points that have left the box may lie 2^31 or more apart,
// where a signed extent turns negative and its product looks small.
__device__ __forceinline__ bool box_fits(const int (&lo)[3], const int (&hi)[3], int (&e)[3]) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const unsigned int d = (unsigned int)hi[k] - (unsigned int)lo[k];
    ok = ok && d < (unsigned int)BOX_CELLS;
    e[k] = (int)(d + 3u);
  }
  return ok && (unsigned int)e[0] * (unsigned int)e[1] * (unsigned int)e[2] <= (unsigned int)BOX_CELLS;
}
static_assert((BOX_CELLS + 2LL) * (BOX_CELLS + 2LL) * (BOX_CELLS + 2LL) <= 0xffffffffLL, "the product is formed in 32 bits");

// Smallest (largest with MAX) of v over the wave, for values that agree inside
// a quad; on every lane.
template <bool MAX>
__device__ __forceinline__ int wave_ext(int v) {
  auto ext = [](int p, int q) { return MAX ? max(p, q) : min(p, q); };
  v = ext(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true));  // the other quad of eight lanes
  v = ext(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true));  // the other eight of sixteen
  return ext(ext(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             ext(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// The three components of a contribution into the fixed-point sums at p,
// p + stride, p + 2 stride.
template <class T>
__device__ __forceinline__ void spread_add(const FluidArgs& a, T* p, long long stride, double c, const double (&F)[3]) {
#pragma unroll
  for (int q = 0; q < 3; q++)
    atomicAdd((unsigned long long*)(p + q * stride), (unsigned long long)fx_quant(c * F[q], a));
}

template <class S>
__device__ void marker_block(const FluidArgs& a, const BodyArgs& b, int blk, long long* fxc,
                             uint8_t* tfc, unsigned int halt) {
  // u* of the box (as the bits of doubles), then, once every marker has read
  // it, the box's force sums
  __shared__ long long s_acc[3][BOX_CELLS];
  __shared__ int s_node[BOX_CELLS];  // padded node index (< 2^31) or -1
  __shared__ int s_wbox[4][6];
  __shared__ unsigned short s_list[BOX_CELLS];
  __shared__ int s_used;
  const Grid& G = a.g;
  const int t = threadIdx.x, sub = t & 3;
  const int nchunk = b.chunk_n[blk], s0 = b.chunk_s0[blk];
  if (nchunk == 0) {
    // an unused chunk: its box stays empty (the repulsion and the owner
    // pass skip it), and nothing else is done
    if (t < 6 && !halt) b.chunk_box[6 * blk + t] = t < 3 ? INT_MAX : INT_MIN;
    return;
  }
  const int m = s0 + (t >> 2);  // slot
  const bool mk = (t >> 2) < nchunk;
  double cen[3] = {0.0, 0.0, 0.0}, Ub[3] = {0.0, 0.0, 0.0}, area = 0.0;
  int bs[3] = {0, 0, 0};
  if (mk) {
    // two rounds of loads: the slot's vertex ids and body, then everything
    // that depends on them at once (positions, vertex velocities, rigid
    // state; the unused of the last two are discarded)
    const int4 sf = *(const int4*)(b.slot_f + 4 * (long long)m);
    const int v0 = sf.x, v1 = sf.y, v2 = sf.z;
    const int body = sf.w;
    double pa[3], pb[3], pd[3], va[3], vb[3], vd[3], rs[12];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      pa[k] = b.Xcur[3 * v0 + k];
      pb[k] = b.Xcur[3 * v1 + k];
      pd[k] = b.Xcur[3 * v2 + k];
      va[k] = b.Vel[3 * v0 + k];
      vb[k] = b.Vel[3 * v1 + k];
      vd[k] = b.Vel[3 * v2 + k];
    }
    int rigid = 0;
    if (b.n_rigid) {
#pragma unroll
      for (int k = 0; k < 12; k++) rs[k] = b.b_rig[32 * body + k];
      rigid = b.b_rigid[body];
    }
    double nrm[3];
    face_geom_pts(pa, pb, pd, cen, nrm, area);
    if (rigid) {
      const double r[3] = {cen[0] - rs[0], cen[1] - rs[1], cen[2] - rs[2]};
      const double* w = rs + 9;
      Ub[0] = rs[3] + (w[1] * r[2] - w[2] * r[1]);
      Ub[1] = rs[4] + (w[2] * r[0] - w[0] * r[2]);
      Ub[2] = rs[5] + (w[0] * r[1] - w[1] * r[0]);
    } else {
#pragma unroll
      for (int k = 0; k < 3; k++) Ub[k] = (va[k] + vb[k] + vd[k]) * (1.0 / 3.0);
    }
#pragma unroll
    for (int k = 0; k < 3; k++) bs[k] = (int)floor(cen[k] + 0.5);
  }
  if (halt) return;
  if (mk && sub == 0) {
#pragma unroll
    for (int k = 0; k < 3; k++) b.centroid[3 * m + k] = cen[k];
  }
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int lo = wave_ext<false>(mk ? bs[k] : INT_MAX), hi = wave_ext<true>(mk ? bs[k] : INT_MIN);
    if ((t & 63) == 0) {
      s_wbox[t >> 6][k] = lo;
      s_wbox[t >> 6][3 + k] = hi;
    }
  }
  __syncthreads();
  int lo[3], hi[3];
#pragma unroll
  for (int k = 0; k < 3; k++) {
    lo[k] = min(min(s_wbox[0][k], s_wbox[1][k]), min(s_wbox[2][k], s_wbox[3][k]));
    hi[k] = max(max(s_wbox[0][3 + k], s_wbox[1][3 + k]), max(s_wbox[2][3 + k], s_wbox[3][3 + k]));
  }
  // this block's slots form one chunk: its box of stencil bases lets the
  // repulsion skip the chunk when a face is farther than dx from it (an
  // unused chunk keeps the empty box)
  if (t == 0) {
#pragma unroll
    for (int k = 0; k < 3; k++) {
      b.chunk_box[6 * blk + k] = lo[k];
      b.chunk_box[6 * blk + 3 + k] = hi[k];
    }
  }
  const int x0 = lo[0] - 1, y0 = lo[1] - 1, z0 = lo[2] - 1;
  int be[3];
  const bool fits = box_fits(lo, hi, be);
  const int ex = be[0], ey = be[1], ez = be[2];
  const int ncell = fits ? ex * ey * ez : 0;
  const float iex = 1.0f / (float)ex, iey = 1.0f / (float)ey;
  // Boxes of more cells than threads: only the cells that some marker uses are
  // computed (the box of a curved patch is about half empty), from a list of
  // them in any order.
  const bool list = ncell > 256;
  if (list) {
    for (int c = t; c < ncell; c += 256) s_node[c] = -1;
    if (t == 0) s_used = 0;
    __syncthreads();
    if (mk) {
      const int c0 = (bs[0] - 1 - x0) + ex * ((bs[1] - 1 - y0) + ey * (bs[2] - 1 - z0));
#pragma unroll
      for (int i = 0; i < 7; i++) {
        const int k = 4 * i + sub;
        if (k < 27) s_node[c0 + k % 3 + ex * ((k / 3) % 3 + ey * (k / 9))] = 0;
      }
    }
    __syncthreads();
    for (int c = t; c < ncell; c += 256)
      if (s_node[c] == 0) s_list[atomicAdd(&s_used, 1)] = (unsigned short)c;
    __syncthreads();
  }
  const int nuse = list ? s_used : ncell;
  for (int i = t; i < nuse; i += 256) {
    const int c = list ? (int)s_list[i] : i;
    // c / ex and so on for c < 1400: the half keeps the product off the integers
    const int q = (int)(((float)c + 0.5f) * iex), cz = (int)(((float)q + 0.5f) * iey);
    int p[3] = {x0 + c - q * ex, y0 + q - cz * ey, z0 + cz};
    const int dim[3] = {G.nx, G.ny, G.nz};
    bool in = true;
#pragma unroll
    for (int k = 0; k < 3; k++)
      if (p[k] < 0 || p[k] >= dim[k]) {
        if (G.per[k]) p[k] = ((p[k] % dim[k]) + dim[k]) % dim[k];
        else in = false;
      }
    const int node = in ? p[0] + G.px * (p[1] + G.ny * p[2]) : 0;
    double u3[3] = {0.0, 0.0, 0.0};
    const bool ok = in && cell_velocity<S>(a, node, p[0], p[1], p[2], u3);
#pragma unroll
    for (int k = 0; k < 3; k++) s_acc[k][c] = __double_as_longlong(u3[k]);
    s_node[c] = ok ? node : -1;
    if (ok && b.support_tf) b.support_tf[node >> TILE_SHIFT] = 1;
  }
  // a quad always holds one marker (or none), so the quad sums below see
  // four lanes that agree on mk
  double wx[3], wy[3], wz[3], dx[3];
  quad_weights(sub, cen, bs, wx, wy, wz);
#pragma unroll
  for (int k = 0; k < 3; k++) dx[k] = (double)(bs[0] + k - 1) - cen[0];
  __syncthreads();
  FitSums<3> fs;
  fs.clear();
  const int c00 = (bs[0] - 1 - x0) + ex * ((bs[1] - 1 - y0) + ey * (bs[2] - 1 - z0));
  if (mk && fits) {
#pragma unroll
    for (int i = 0; i < 3; i++) {
      int ky = 2, kz = 2;
      if (i < 2) row_yz(sub + 4 * i, ky, kz);
      const int cr = c00 + ex * (ky + ey * kz) + (i < 2 ? 0 : min(sub, 2));
      RowSums<3> rs;
      rs.clear();
#pragma unroll
      for (int k = 0; k < (i < 2 ? 3 : 1); k++) {
        const bool on = s_node[cr + k] >= 0 && (i < 2 || sub < 3);
        const double w = on ? (i < 2 ? wx[k] : sel3(sub, wx)) : 0.0, d = i < 2 ? dx[k] : sel3(sub, dx);
        const double f[3] = {__longlong_as_double(s_acc[0][cr + k]), __longlong_as_double(s_acc[1][cr + k]),
                             __longlong_as_double(s_acc[2][cr + k])};
        rs.add(w, d, f);
      }
      fs.add(rs, sel3(ky, wy) * sel3(kz, wz), (double)(bs[1] + ky - 1) - cen[1], (double)(bs[2] + kz - 1) - cen[2]);
    }
  } else if (mk) {
#pragma unroll 1
    for (int k = sub; k < 27; k += 4) {
      const int kx = k % 3, ky = (k / 3) % 3, kz = k / 9;
      const int cx = bs[0] + kx - 1, cy = bs[1] + ky - 1, cz = bs[2] + kz - 1;
      long long node;
      double u3[3] = {0.0, 0.0, 0.0};
      bool ok = support_node(G, a.ncls, cx, cy, cz, node);
      if (ok) {
        int x, y, z;
        coords(G, node, x, y, z);
        ok = cell_velocity<S>(a, (int)node, x, y, z, u3);
        if (b.support_tf) b.support_tf[node >> TILE_SHIFT] = 1;
      }
      RowSums<3> rs;
      rs.clear();
      rs.add(ok ? sel3(kx, wx) : 0.0, cx - cen[0], u3);
      fs.add(rs, sel3(ky, wy) * sel3(kz, wz), cy - cen[1], cz - cen[2]);
    }
  }
  __syncthreads();
  for (int c = t; c < ncell; c += blockDim.x) {
#pragma unroll
    for (int k = 0; k < 3; k++) s_acc[k][c] = 0;
  }
  fs.quad();
  double F[3] = {0.0, 0.0, 0.0}, cc[4] = {0.0, 0.0, 0.0, 0.0};
  if (mk) {
    Chol4 ch;
    if (chol4(fs.A, ch)) {
      const double e0[4] = {1.0, 0.0, 0.0, 0.0};
      chol_solve(ch, e0, cc);
    } else if (sub == 0) {
      atomicAdd(&a.flags->mls_singular, 1);
    }
#pragma unroll
    for (int q = 0; q < 3; q++)
      F[q] = Ub[q] - (cc[0] * fs.b[q][0] + cc[1] * fs.b[q][1] + cc[2] * fs.b[q][2] + cc[3] * fs.b[q][3]);
  }
  __syncthreads();
  if (mk && fits) {
    // straight-line, no branch per cell: a cell without a node gets zeros
    bool over = false;
#pragma unroll
    for (int i = 0; i < 3; i++) {
      int ky = 2, kz = 2;
      if (i < 2) row_yz(sub + 4 * i, ky, kz);
      const double dy = (double)(bs[1] + ky - 1) - cen[1], dz = (double)(bs[2] + kz - 1) - cen[2];
      const double w = area * (sel3(ky, wy) * sel3(kz, wz)), t0 = cc[0] + cc[2] * dy + cc[3] * dz;
      const int cr = c00 + ex * (ky + ey * kz) + (i < 2 ? 0 : min(sub, 2));
#pragma unroll
      for (int k = 0; k < (i < 2 ? 3 : 1); k++) {
        const double c = i < 2 ? w * wx[k] * (t0 + cc[1] * dx[k]) : w * sel3(sub, wx) * (t0 + cc[1] * sel3(sub, dx));
        const bool on = s_node[cr + k] >= 0 && (i < 2 || sub < 3) && c != 0.0;
#pragma unroll
        for (int q = 0; q < 3; q++) {
          const double v = c * F[q];
          const bool in = fabs(v) <= 1.0;
          over = over || (on && !in);
          atomicAdd((unsigned long long*)&s_acc[q][cr + k], (unsigned long long)__double2ll_rn(on && in ? v * FX_SCALE : 0.0));
        }
      }
    }
    if (over) fx_over(a);
  } else if (mk) {
#pragma unroll 1
    for (int k = sub; k < 27; k += 4) {
      const int kx = k % 3, ky = (k / 3) % 3, kz = k / 9;
      const int cx = bs[0] + kx - 1, cy = bs[1] + ky - 1, cz = bs[2] + kz - 1;
      const double ddx = cx - cen[0], dy = cy - cen[1], dz = cz - cen[2];
      long long node;
      const bool ok = support_node(G, a.ncls, cx, cy, cz, node);
      const double c = area * sel3(kx, wx) * sel3(ky, wy) * sel3(kz, wz) * (cc[0] + cc[1] * ddx + cc[2] * dy + cc[3] * dz);
      if (ok && c != 0.0) {
        spread_add(a, fxc + node, G.Np, c, F);
        tfc[node >> TILE_SHIFT] = 1;
      }
    }
  }
  __syncthreads();
  if (b.stage) {
    // two-pass spread: the block's sums go to its staging box; the owner
    // pass (k_spread_owner) adds them up across blocks without atomics
    long long* st = b.stage + (long long)blk * BOX_CELLS * 3;
    int* sn = b.stage_node + (long long)blk * BOX_CELLS;
    for (int c = t; c < ncell; c += blockDim.x) {
      sn[c] = s_node[c];
#pragma unroll
      for (int q = 0; q < 3; q++) st[3 * c + q] = s_acc[q][c];
    }
    return;
  }
  for (int c = t; c < ncell; c += blockDim.x) {
    const long long node = s_node[c];
    if (node < 0) continue;
    bool any = false;
#pragma unroll
    for (int q = 0; q < 3; q++) {
      const long long v = s_acc[q][c];
      if (v != 0) {
        atomicAdd((unsigned long long*)(fxc + q * G.Np + node), (unsigned long long)v);
        any = true;
      }
    }
    if (any) tfc[node >> TILE_SHIFT] = 1;
  }
}

// Cell of node (x, y, z) in a chunk's box (origin o, extents e), trying the
// periodic images one period away; -1 if outside.
__device__ __forceinline__ int box_cell(const Grid& G, const int (&o)[3], const int (&e)[3], int x, int y, int z) {
  const int p[3] = {x, y, z}, n[3] = {G.nx, G.ny, G.nz};
  int c[3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    int d = p[a] - o[a];
    if (G.per[a] && (d < 0 || d >= e[a])) d = d < 0 ? d + n[a] : d - n[a];
    if (d < 0 || d >= e[a]) return -1;
    c[a] = d;
  }
  return c[0] + e[0] * (c[1] + e[1] * c[2]);
}

// The box of chunk k from its bases (cb: its six ints); false when the chunk
// did not fit LDS (its block added its sums with atomics) or is empty.
__device__ __forceinline__ bool chunk_geom(const int* cb, int (&o)[3], int (&e)[3]) {
  if (cb[3] < cb[0]) return false;
  const int lo[3] = {cb[0], cb[1], cb[2]}, hi[3] = {cb[3], cb[4], cb[5]};
#pragma unroll
  for (int a = 0; a < 3; a++) o[a] = lo[a] - 1;
  return box_fits(lo, hi, e);
}

// Owner pass of the two-pass spread: thread (chunk c, cell i) holds node n;
// it is the owner when no lower chunk's box holds n, and then adds the
// staged sums of every chunk that holds n, in chunk order, into the force
// field (plain stores: one owner per node), and flags the tile.
__global__ __launch_bounds__(256) void k_spread_owner(Grid G, BodyArgs b, long long* fxc, uint8_t* tfc,
                                                      const DevFlags* flags) {
  if (halted(flags, b.par)) return;
  const int nch = b.n_marker_blocks, c = blockIdx.y;
  int o[3], e[3];
  if (!chunk_geom(b.chunk_box + 6 * c, o, e)) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= e[0] * e[1] * e[2]) return;
  const int node = b.stage_node[(long long)c * BOX_CELLS + i];
  if (node < 0) return;
  int x, y, z;
  coords(G, node, x, y, z);
  for (int k = 0; k < c; k++) {
    int ok[3], ek[3];
    if (!chunk_geom(b.chunk_box + 6 * k, ok, ek)) continue;
    const int j = box_cell(G, ok, ek, x, y, z);
    if (j >= 0 && b.stage_node[(long long)k * BOX_CELLS + j] == node) return;  // not the owner
  }
  long long acc[3] = {0, 0, 0};
  for (int k = c; k < nch; k++) {
    int ok[3], ek[3];
    if (!chunk_geom(b.chunk_box + 6 * k, ok, ek)) continue;
    const int j = box_cell(G, ok, ek, x, y, z);
    if (j < 0 || b.stage_node[(long long)k * BOX_CELLS + j] != node) continue;
    const long long* st = b.stage + ((long long)k * BOX_CELLS + j) * 3;
#pragma unroll
    for (int q = 0; q < 3; q++) acc[q] += st[q];
  }
  if (acc[0] == 0 && acc[1] == 0 && acc[2] == 0) return;
#pragma unroll
  for (int q = 0; q < 3; q++) fxc[q * G.Np + node] += acc[q];
  tfc[node >> TILE_SHIFT] = 1;
}

// ------------------------------------------------------------ face binning
// The marker order.  One block per body: each face's key is the position of
// its stencil base floor(c + 1/2) (relative to the body's smallest base, 10
// bits per axis) along the 3-D Hilbert curve, above the face's index within
// the body; the keys are bitonic-sorted (in LDS up to BIN_LDS_KEYS faces,
// else in the body's part of bin_keys) and slot f0 + r takes the face of
// rank r.  The keys are distinct, so the order is a function of the
// positions alone.  The Hilbert curve (unlike the Morton order) has no
// jumps, so 64 consecutive faces stay one compact patch of the membrane.
__device__ __forceinline__ unsigned int spread_bits10(unsigned int x) {
  x &= 1023u;
  x = (x | (x << 16)) & 0x030000FFu;
  x = (x | (x << 8)) & 0x0300F00Fu;
  x = (x | (x << 4)) & 0x030C30C3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

// Hilbert index of a point of [0, 1024)^3, by Skilling's transpose method
// (J. Skilling, "Programming the Hilbert curve", AIP Conf. Proc. 707, 2004):
// the coordinates are turned, level by level from the top, into the
// transposed index, whose bits interleaved give the distance along the
// curve.
__device__ __forceinline__ unsigned int hilbert10(int a, int b, int c) {
  unsigned int X[3] = {(unsigned int)min(max(a, 0), 1023), (unsigned int)min(max(b, 0), 1023),
                       (unsigned int)min(max(c, 0), 1023)};
  for (unsigned int Q = 512u; Q > 1u; Q >>= 1) {
    const unsigned int P = Q - 1u;
#pragma unroll
    for (int i = 0; i < 3; i++) {
      if (X[i] & Q) {
        X[0] ^= P;  // invert the low bits of the first axis
      } else {      // exchange the low bits of axes 0 and i
        const unsigned int t = (X[0] ^ X[i]) & P;
        X[0] ^= t;
        X[i] ^= t;
      }
    }
  }
  X[1] ^= X[0];  // Gray encode
  X[2] ^= X[1];
  unsigned int t = 0u;
  for (unsigned int Q = 512u; Q > 1u; Q >>= 1)
    if (X[2] & Q) t ^= Q - 1u;
  X[0] ^= t;
  X[1] ^= t;
  X[2] ^= t;
  return (spread_bits10(X[0]) << 2) | (spread_bits10(X[1]) << 1) | spread_bits10(X[2]);
}

__device__ __forceinline__ void face_base(const double* X, const int32_t* faces, int f, int (&bs)[3]) {
  const int v0 = faces[3 * f], v1 = faces[3 * f + 1], v2 = faces[3 * f + 2];
#pragma unroll
  for (int k = 0; k < 3; k++) bs[k] = (int)floor((X[3 * v0 + k] + X[3 * v1 + k] + X[3 * v2 + k]) / 3.0 + 0.5);
}

// Keys and sort of one body; K is LDS or global memory (inlined separately
// for each, so that LDS accesses stay LDS instructions).  On return K[0..nf)
// holds the body's keys in increasing order.
__device__ __forceinline__ void hilbert_sort(const BodyArgs& b, int f0, int nf, int n2, const int (&lo)[3],
                                             unsigned long long* K) {
  const int t = threadIdx.x;
  for (int i = t; i < n2; i += blockDim.x) {
    unsigned long long key = ~0ull;  // padding sorts last
    if (i < nf) {
      int bs[3];
      face_base(b.Xcur, b.faces, f0 + i, bs);
      key = ((unsigned long long)hilbert10(bs[0] - lo[0], bs[1] - lo[1], bs[2] - lo[2]) << 32) | (unsigned int)i;
    }
    K[i] = key;
  }
  __syncthreads();
  for (int k = 2; k <= n2; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = t; i < n2; i += blockDim.x) {
        const int p = i ^ j;
        if (p > i) {
          const unsigned long long x = K[i], y = K[p];
          if ((x > y) == ((i & k) == 0)) {
            K[i] = y;
            K[p] = x;
          }
        }
      }
      __syncthreads();
    }
}

__device__ __forceinline__ unsigned int compact_bits10(unsigned int x) {
  x &= 0x09249249u;
  x = (x | (x >> 2)) & 0x030C30C3u;
  x = (x | (x >> 4)) & 0x0300F00Fu;
  x = (x | (x >> 8)) & 0x030000FFu;
  x = (x | (x >> 16)) & 0x000003FFu;
  return x;
}

// The point of [0, 1024)^3 at Hilbert index h (the inverse of hilbert10:
// Gray decode, then the exchanges and inversions undone from the bottom
// level up).
__device__ __forceinline__ void hilbert10_point(unsigned int h, int (&c)[3]) {
  unsigned int X[3] = {compact_bits10(h >> 2), compact_bits10(h >> 1), compact_bits10(h)};
  const unsigned int t = X[2] >> 1;
  X[2] ^= X[1];
  X[1] ^= X[0];
  X[0] ^= t;
  for (unsigned int Q = 2u; Q != 1024u; Q <<= 1) {
    const unsigned int P = Q - 1u;
#pragma unroll
    for (int i = 2; i >= 0; i--) {
      if (X[i] & Q) {
        X[0] ^= P;
      } else {
        const unsigned int u = (X[0] ^ X[i]) & P;
        X[0] ^= u;
        X[i] ^= u;
      }
    }
  }
  c[0] = (int)X[0];
  c[1] = (int)X[1];
  c[2] = (int)X[2];
}

// Exclusive prefix sum over the block's threads in thread order; total gets
// the sum.  s_tmp holds BIN_THREADS / 64 + 1 values.
template <class T>
__device__ __forceinline__ T block_scan(T v, T* s_tmp, T& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  T x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) s_tmp[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    T acc = 0;
    for (int k = 0; k < nw; k++) {
      const T c = s_tmp[k];
      s_tmp[k] = acc;
      acc += c;
    }
    s_tmp[nw] = acc;
  }
  __syncthreads();
  const T ex = s_tmp[w] + x - v;
  total = s_tmp[nw];
  __syncthreads();
  return ex;
}

// Chunks of at most 64 consecutive slots, in order: nrun runs of 64 (the
// last one shorter), the rest of the body's chunks unused.
// Slot s takes face f: the permutation and the face's vertex ids and body.
__device__ __forceinline__ void set_slot(const BodyArgs& b, int s, int f) {
  b.perm[s] = f;
  const int4 v = make_int4(b.faces[3 * f], b.faces[3 * f + 1], b.faces[3 * f + 2], b.face_body[f]);
  *(int4*)(b.slot_f + 4 * (long long)s) = v;
}

__device__ __forceinline__ void fixed_chunks(const BodyArgs& b, int f0, int nf, int c0, int cap) {
  const int nrun = (nf + MARKERS_PER_BLOCK - 1) / MARKERS_PER_BLOCK;
  for (int c = threadIdx.x; c < cap; c += blockDim.x) {
    b.chunk_s0[c0 + c] = f0 + min(c, nrun) * MARKERS_PER_BLOCK;
    b.chunk_n[c0 + c] = c < nrun ? min(MARKERS_PER_BLOCK, nf - c * MARKERS_PER_BLOCK) : 0;
  }
}

__global__ __launch_bounds__(BIN_THREADS) void k_bin_faces(BodyArgs b) {
  __shared__ unsigned long long s_keys[BIN_LDS_KEYS];
  __shared__ unsigned long long s_tmp[BIN_THREADS / 64 + 1];
  __shared__ int s_min[3];
  const int body = blockIdx.x, t = threadIdx.x;
  const int f0 = b.b_face0[body], nf = b.b_nf[body];
  const int c0 = b.b_chunk0[body], cap = b.b_chunk0[body + 1] - c0;
  int n2 = 1;
  while (n2 < nf) n2 <<= 1;
  if (t < 3) s_min[t] = INT_MAX;
  __syncthreads();
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX};
  for (int i = t; i < nf; i += blockDim.x) {
    int bs[3];
    face_base(b.Xcur, b.faces, f0 + i, bs);
#pragma unroll
    for (int k = 0; k < 3; k++) lo[k] = min(lo[k], bs[k]);
  }
#pragma unroll
  for (int k = 0; k < 3; k++) atomicMin(&s_min[k], lo[k]);
  __syncthreads();
  const int mn[3] = {s_min[0], s_min[1], s_min[2]};
  if (n2 > BIN_LDS_KEYS) {
    // large body: sorted in global memory, cut in runs of 64
    unsigned long long* K = b.bin_keys + b.b_key0[body];
    hilbert_sort(b, f0, nf, n2, mn, K);
    for (int i = t; i < nf; i += blockDim.x) set_slot(b, f0 + i, f0 + (int)(K[i] & 0xffffffffull));
    fixed_chunks(b, f0, nf, c0, cap);
    return;
  }
  hilbert_sort(b, f0, nf, n2, mn, s_keys);
  // Chunks: thread t owns the sorted positions t R .. t R + R - 1.  A
  // position starts a segment where its base is more than J (Chebyshev)
  // from the previous one's; each segment of length L is cut into
  // ceil(L / 64) near-equal chunks.  J is the smallest of 1..4 whose
  // segments fit the body's chunks (else plain runs of 64).
  const int R = (nf + BIN_THREADS - 1) / BIN_THREADS;  // <= 8
  unsigned int jm[4] = {0u, 0u, 0u, 0u};
  {
    int prev[3] = {0, 0, 0};
    const int i0 = t * R;
    if (i0 >= 1 && i0 - 1 < nf) hilbert10_point((unsigned int)(s_keys[i0 - 1] >> 32), prev);
    for (int r = 0; r < R; r++) {
      const int i = i0 + r;
      if (i >= nf) break;
      const unsigned long long key = s_keys[i];
      set_slot(b, f0 + i, f0 + (int)(key & 0xffffffffull));
      int c[3];
      hilbert10_point((unsigned int)(key >> 32), c);
      const int d = max(abs(c[0] - prev[0]), max(abs(c[1] - prev[1]), abs(c[2] - prev[2])));
#pragma unroll
      for (int J = 0; J < 4; J++)
        if (i == 0 || d > J + 1) jm[J] |= 1u << r;
      prev[0] = c[0];
      prev[1] = c[1];
      prev[2] = c[2];
    }
  }
  unsigned long long packed = 0ull;
#pragma unroll
  for (int J = 0; J < 4; J++) packed |= (unsigned long long)__popc(jm[J]) << (16 * J);
  unsigned long long tot;
  const unsigned long long ex = block_scan(packed, s_tmp, tot);  // syncs: the keys are free after
  const int nrun = (nf + MARKERS_PER_BLOCK - 1) / MARKERS_PER_BLOCK;
  int J = -1;
  for (int q = 3; q >= 0; q--)
    if ((int)((tot >> (16 * q)) & 0xffffull) + nrun <= cap) J = q;
  if (J < 0) {
    fixed_chunks(b, f0, nf, c0, cap);
    return;
  }
  const int S = (int)((tot >> (16 * J)) & 0xffffull);
  int* SS = reinterpret_cast<int*>(s_keys);  // segment starts [S + 1]
  {
    int o = (int)((ex >> (16 * J)) & 0xffffull);
    for (int r = 0; r < R; r++)
      if (jm[J] & (1u << r)) SS[o++] = t * R + r;
    if (t == 0) SS[S] = nf;
  }
  __syncthreads();
  // chunks of thread t's segments t Rs .. t Rs + Rs - 1
  const int Rs = (S + BIN_THREADS - 1) / BIN_THREADS;
  int nk = 0;
  for (int s = t * Rs; s < min(S, t * Rs + Rs); s++) nk += (SS[s + 1] - SS[s] + MARKERS_PER_BLOCK - 1) / MARKERS_PER_BLOCK;
  unsigned long long ntot;
  int cc = c0 + (int)block_scan((unsigned long long)nk, s_tmp, ntot);
  for (int s = t * Rs; s < min(S, t * Rs + Rs); s++) {
    const int a = SS[s], L = SS[s + 1] - a;
    const int k = (L + MARKERS_PER_BLOCK - 1) / MARKERS_PER_BLOCK;
    for (int q = 0; q < k; q++, cc++) {
      const int lo_q = (L * q) / k, hi_q = (L * (q + 1)) / k;
      b.chunk_s0[cc] = f0 + a + lo_q;
      b.chunk_n[cc] = hi_q - lo_q;
    }
  }
  for (int c = (int)ntot + t; c < cap; c += blockDim.x) {
    b.chunk_s0[c0 + c] = f0 + nf;
    b.chunk_n[c0 + c] = 0;
  }
}

// Zeroes the spread force of the previous step in the tiles it flagged, and
// the flags.  That buffer is not read again once this step has started, and
// the next step adds into it.  Block cb of ncb reads the flags of its tiles
// cb, cb + ncb, ... all at once (one per thread), lists the set ones in LDS,
// then clears them one after the other with all its threads.
__device__ void clear_tiles(const Grid& G, long long* fxp, uint8_t* tfp, int cb, int ncb) {
  __shared__ int s_n;
  __shared__ int s_list[256];
  const long long ntiles = (G.Np >> TILE_SHIFT) + 1;
  for (long long first = cb; first < ntiles; first += (long long)ncb * blockDim.x) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const long long tl = first + (long long)threadIdx.x * ncb;
    if (tl < ntiles && tfp[tl]) s_list[atomicAdd(&s_n, 1)] = (int)tl;
    __syncthreads();
    const int n = s_n;
    // the listed tiles' nodes, all threads at once
    for (int k = threadIdx.x; k < (n << TILE_SHIFT); k += blockDim.x) {
      const long long q = ((long long)s_list[k >> TILE_SHIFT] << TILE_SHIFT) + (k & ((1 << TILE_SHIFT) - 1));
      if (q < G.Np) {
        fxp[q] = 0;
        fxp[G.Np + q] = 0;
        fxp[2 * G.Np + q] = 0;
      }
    }
    if ((int)threadIdx.x < n) tfp[s_list[threadIdx.x]] = 0;
    __syncthreads();
  }
}

__device__ void membrane_element(const BodyArgs& b, int idx) {
  if (idx < b.ne) {
    const int e = idx;
    const int va = b.edges[2 * e], vb = b.edges[2 * e + 1];
    if (b.b_rigid[b.vert_body[va]]) return;
    // F_a = -k (l - l0) (x_a - x_b) / l
    const double r[3] = {b.Xcur[3 * va] - b.Xcur[3 * vb], b.Xcur[3 * va + 1] - b.Xcur[3 * vb + 1],
                         b.Xcur[3 * va + 2] - b.Xcur[3 * vb + 2]};
    const double l = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    const double c = -b.kl[e] * (l - b.l0[e]) / l;
    const int sa = b.sl_edge[2 * e], sb = b.sl_edge[2 * e + 1];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      b.f_slot[((long long)sa * 3 + k) * b.nv + va] = c * r[k];
      b.f_slot[((long long)sb * 3 + k) * b.nv + vb] = -(c * r[k]);
    }
  } else if (idx < b.ne + b.nh) {
    const int h = idx - b.ne;
    const int32_t* H = b.hinges + 4 * h;
    if (b.b_rigid[b.vert_body[H[0]]]) return;
    double th, gr[4][3];
    hinge_all(b.Xcur, H, th, gr);
    const double amp = -b.kb[h] * sin(th - b.theta0[h]);
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const long long sl = b.sl_hinge[4 * h + r];
#pragma unroll
      for (int k = 0; k < 3; k++) b.f_slot[(sl * 3 + k) * b.nv + H[r]] = amp * gr[r][k];
    }
  }
}

template <class S>
__device__ __forceinline__ void ib_force_block(const FluidArgs& a, const BodyArgs& b, long long* fxc,
                                               uint8_t* tfc, unsigned int* counter, int blk) {
  // (not halted(): the check below is of this launch, and a block whose waves
  // saw it at different times would lose some of them before its barriers)
  const unsigned int halt = halted_before(a.flags, a.par);
  const int nmk = b.n_marker_blocks, ndg = b.n_diag_blocks;
  // The diagnostics first: their last block waits for all of them.  The short
  // element blocks last, where they fill the places that the markers leave.
  if (blk < ndg) {
    if (halt) return;
    diag_block(b, b.Xcur, blk);
    // the diagnostics blocks count themselves; the last one combines them
    if (last_block(counter, b.n_diag_blocks)) {
      const unsigned int raised = diag_finalize(b);
      if (raised) atomicOr(&a.flags->check, raised);
      __syncthreads();
      if (threadIdx.x == 0) *counter = 0u;
    }
  } else if (blk < ndg + nmk) {
    marker_block<S>(a, b, blk - ndg, fxc, tfc, halt);
  } else if (!halt) {
    membrane_element(b, (blk - ndg - nmk) * 256 + threadIdx.x);
  }
}

// The marker blocks are chains of dependent loads (about 1 us per round trip
// to memory another XCD wrote last) with little arithmetic, 4 waves on a CU:
// the launch lasts as long as its longest chain.  So: flags, chunk and slot
// tables in two rounds, the 19 pulls of a cell with its class instead of
// after it, three links of a boundary node per round, sums row by row and
// through DPP moves, and one LDS array for u* and then the sums (42 KB, 218
// registers: two waves per SIMD; asking for three or four spills and is
// slower, 15.4 and 17.8 us on one capsule; 17.1 with the spread below).  Of a
// block's 10 us the pulls take 2.5 (7 where links are near), the tables 2.3,
// the spread into LDS 1.6 (2.7 with a branch per cell), the sums 1.1.  A box of
// more than 256 cells computes the used ones only (a coarse sphere of 320 faces
// at r = 4: 3 passes of the pulls become 2, a train of three 3 become 1), and
// the diagnostics, whose last block waits for the others, come first in the
// grid (16 capsules 79 -> 71 us, one 13.7 -> 12.0).  Measured per launch, at
// first -> now: one capsule of 5120 faces 18.7 -> 11.9 us, a train of three
// 32 -> 17, 16 capsules 110 -> 72, a sweep of ten 43 -> 30; in FP64 a rigid
// sphere of 320 faces 28 -> 12.5 in a 48x20x20 pipe (r = 4 in R = 8) and
// 28 -> 17.5 in a 24x12x12 one (r = 2.5 in R = 4.5: links near every cell).
template <class S>
__global__ __launch_bounds__(256, 2) void k_ib_force(FluidArgs a, BodyArgs b, long long* fxc,
                                                  uint8_t* tfc, unsigned int* counter) {
  ib_force_block<S>(a, b, fxc, tfc, counter, blockIdx.x);
}

// Diagnostics of the current positions only (set-up and synchronisation
// points): fills the body table and stops on damage or non-finite values.  Not
// after a stop, one that the last step raised and the next would latch
// included: the run's status is what stopped it.
__global__ __launch_bounds__(256) void k_check(BodyArgs b, const double* X0, const double* X1,
                                               DevFlags* flags, unsigned int* counter) {
  if (flags->stop | flags->pend0 | flags->pend1) return;
  const double* X = (flags->steps_done & 1) ? X1 : X0;
  if ((int)blockIdx.x < b.n_diag_blocks) diag_block(b, X, blockIdx.x);
  if (last_block(counter, gridDim.x)) {
    const unsigned int raised = diag_finalize(b);
    if (raised) atomicOr(&flags->stop, raised);
    __syncthreads();
    if (threadIdx.x == 0) *counter = 0u;
  }
}

// ---------------------------------------------------------- k_mls_post
// One MLS point per quad of lanes, supports read from this step's rho - 1
// and u.  Face waves (8 faces each): lanes 0-31 take the probes 1.2 dx outside
// their faces, lanes 32-63 the probes inside the same faces; each fits rho
// (value) and u (gradient) by moving least squares (the linear-fit
// coefficients), then the outer lane forms the traction: pressure p = rho/3
// and viscous stress rho nu (grad u + grad u^T) (Eqs. hydroForP,
// hydroForNu), the repulsion of centroids of other bodies closer than dx
// (Eq. collision) and, for soft bodies, the volume penalty
// k_v (1 - V/V0) A n (Eq. volFor, outward n).  A singular fit gives 0.
// Vertex waves (16 soft vertices each): the MLS velocity u_v,0 at x_v^n.
// Bound by waiting for dependent loads and, with many faces, by instruction
// issue: the tables a face needs are loaded in two rounds ahead of the fit (the
// traction's among them), solid nodes are told by the macro field itself, a
// quad shares its nine exponentials and adds its partial sums by DPP moves, and
// supports are summed row by row.  Measured per launch, before -> after: one
// capsule 10.3 -> 7.6 us, a train of three 14.4 -> 10.9, a small sphere in
// FP64 8.5 -> 6.7, 16 capsules 72 -> 52, a sweep of ten instances 24.7 -> 17.9.
template <class S, bool GRAD>
__device__ __forceinline__ void fit_point(const FluidArgs& a, unsigned int halt, int sub, const double (&p)[3],
                                          double& rfit, double (&val)[3], double (&grad)[3][3]) {
  typedef typename Store<S>::C C;
  typedef C C4 __attribute__((ext_vector_type(4)));
  const Grid& G = a.g;
  const int bs[3] = {(int)floor(p[0] + 0.5), (int)floor(p[1] + 0.5), (int)floor(p[2] + 0.5)};
  // this lane's seven supports: loads first, all together (out-of-box supports
  // read a node of the box and are not used; solid nodes hold MAC_SOLID)
  int ox[3], oy[3], oz[3];
  bool ix[3], iy[3], iz[3];
  axis_nodes(bs[0], G.nx, G.per[0], 1, ox, ix);
  axis_nodes(bs[1], G.ny, G.per[1], G.px, oy, iy);
  axis_nodes(bs[2], G.nz, G.per[2], G.px * G.ny, oz, iz);
  const C4* mac = (const C4*)a.mac;
  C4 mv[7];
  bool in[7];
  int ky[3], kz[3];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    row_yz(sub + 4 * i, ky[i], kz[i]);
    const int row = sel3i(ky[i], oy) + sel3i(kz[i], oz);
    const bool rin = sel3b(ky[i], iy) && sel3b(kz[i], iz);
#pragma unroll
    for (int k = 0; k < 3; k++) {
      mv[3 * i + k] = mac[ox[k] + row];
      in[3 * i + k] = rin && ix[k];
    }
  }
  ky[2] = kz[2] = 2;
  mv[6] = mac[sel3i(sub, ox) + oy[2] + oz[2]];
  in[6] = sub < 3 && sel3b(sub, ix) && iy[2] && iz[2];
  double wx[3], wy[3], wz[3], dx[3];
  quad_weights(sub, p, bs, wx, wy, wz);
#pragma unroll
  for (int k = 0; k < 3; k++) dx[k] = (double)(bs[0] + k - 1) - p[0];
  constexpr int NF = GRAD ? 4 : 3;  // u and, at the probes, rho - 1
  FitSums<NF> fs;
  fs.clear();
#pragma unroll
  for (int i = 0; i < 3; i++) {
    RowSums<NF> rs;
    rs.clear();
#pragma unroll
    for (int k = 0; k < (i < 2 ? 3 : 1); k++) {
      const C4& v = mv[3 * i + k];
      const bool u = in[3 * i + k] && !(v.x <= C(MAC_SOLID));
      const double w = u ? (i < 2 ? wx[k] : sel3(sub, wx)) : 0.0, d = i < 2 ? dx[k] : sel3(sub, dx);
      double f[NF];
      f[0] = u ? (double)v.y : 0.0;
      f[1] = u ? (double)v.z : 0.0;
      f[2] = u ? (double)v.w : 0.0;
      if (GRAD) f[NF - 1] = u ? (double)v.x : 0.0;
      rs.add(w, d, f);
    }
    const double dy = (double)(bs[1] + ky[i] - 1) - p[1], dz = (double)(bs[2] + kz[i] - 1) - p[2];
    fs.add(rs, sel3(ky[i], wy) * sel3(kz[i], wz), dy, dz);
  }
  fs.quad();  // the quad's four partial sums, in a fixed order
  Chol4 ch;
  const bool ok = chol4(fs.A, ch);
  if (!ok && sub == 0 && !halt) atomicAdd(&a.flags->mls_singular, 1);
  double cc[4] = {0.0, 0.0, 0.0, 0.0};
  if (ok) {
    const double e0[4] = {1.0, 0.0, 0.0, 0.0};
    chol_solve(ch, e0, cc);
  }
  // the weights add up to 1, so the fit of rho is 1 + the fit of rho - 1
  if (GRAD) {
    const double (&br)[4] = fs.b[NF - 1];
    rfit = ok ? 1.0 + (cc[0] * br[0] + cc[1] * br[1] + cc[2] * br[2] + cc[3] * br[3]) : 0.0;
  }
#pragma unroll
  for (int q = 0; q < 3; q++) {
    const double (&bu)[4] = fs.b[q];
    if (!GRAD) val[q] = cc[0] * bu[0] + cc[1] * bu[1] + cc[2] * bu[2] + cc[3] * bu[3];
    if (GRAD) {
      double x[4] = {0.0, 0.0, 0.0, 0.0};
      if (ok) chol_solve(ch, bu, x);
#pragma unroll
      for (int c = 0; c < 3; c++) grad[q][c] = x[1 + c];
    }
  }
}

// Face waves take 8 faces: the quad of lanes 4f..4f+3 (f < 8) fits the probe
// outside face f, lanes 32 + 4f.. the probe inside; vertex waves take 16
// soft vertices, one quad each.

template <class S>
__device__ __forceinline__ void mls_post_block(const FluidArgs& a, const BodyArgs& b, int blk, unsigned int halt) {
  const int gw = (blk * 256 + threadIdx.x) >> 6;
  const int l = threadIdx.x & 63, sub = l & 3;
  const int nfw = (b.nf + MLS_FACES_PER_WAVE - 1) / MLS_FACES_PER_WAVE;
  if (gw < nfw) {
    const int f = gw * MLS_FACES_PER_WAVE + ((l & 31) >> 2);
    const bool valid = f < b.nf;
    const int fv = valid ? f : b.nf - 1;  // spare lanes repeat a face and write nothing
    // two rounds of loads ahead of the fit: the face's tables, then everything
    // that they lead to (what the traction needs at the end among it)
    const int fvx[3] = {b.faces[3 * fv], b.faces[3 * fv + 1], b.faces[3 * fv + 2]};
    const int fsl[3] = {b.sl_face[3 * fv], b.sl_face[3 * fv + 1], b.sl_face[3 * fv + 2]};
    const int body = b.face_body[fv];
    double pa[3], pb[3], pd[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      pa[k] = b.Xcur[3 * fvx[0] + k];
      pb[k] = b.Xcur[3 * fvx[1] + k];
      pd[k] = b.Xcur[3 * fvx[2] + k];
    }
    const double V0 = b.b_param[8 * body], kv = b.b_param[8 * body + 2], V = b.b_diag[16 * body];
    const int rigid = b.b_rigid[body];
    // a wave whose faces belong to one body, and up to 64 bodies: lane o tests
    // body o's box against theirs, so that a body with no neighbour near it
    // (the rule) leaves the repulsion at once
    bool near = b.nbody > 1;
    if (near && b.nbody <= 64) {
      const int q0 = __builtin_amdgcn_readfirstlane(body), o = l < b.nbody ? l : 0;
      const double* bb = b.b_diag + 16 * q0 + 2;
      const double* ob = b.b_diag + 16 * o + 2;
      bool close = l < b.nbody && o != q0;
#pragma unroll
      for (int k = 0; k < 3; k++)
        if (bb[k] > ob[3 + k] + 1.0 || ob[k] > bb[3 + k] + 1.0) close = false;
      near = __ballot(close) != 0ull || __ballot(body != q0) != 0ull;
    }
    double cen[3], nrm[3], area;
    face_geom_pts(pa, pb, pd, cen, nrm, area);
    const double sg = l < 32 ? 1.2 : -1.2;
    double rfit, val[3], G[3][3];
    const double probe[3] = {cen[0] + sg * nrm[0], cen[1] + sg * nrm[1], cen[2] + sg * nrm[2]};
    fit_point<S, true>(a, halt, sub, probe, rfit, val, G);
    if (halt) return;
    // the inner probe of this lane's face
    const double r_in = __shfl(rfit, l + 32, 64);
    double Gin[3][3];
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
      for (int c = 0; c < 3; c++) Gin[i][c] = __shfl(G[i][c], l + 32, 64);
    double acc = 0.0;
    if (near) {
      // repulsion.  First the lanes test the (face q of the wave, other body
      // o) pairs in parallel: o's box must come within dx of q's body's box
      // and of the face itself, and its bounding sphere within dx of the
      // face.  Then, for each surviving pair in (q, o) order, all lanes scan
      // o's centroids.
      const int npair = MLS_FACES_PER_WAVE * b.nbody;
      int cur_q = -1;
      double part = 0.0;
      for (int base = 0; base < npair; base += 64) {
        const int pi = base + l < npair ? base + l : npair - 1;
        const int pq = pi / b.nbody, po = pi - pq * b.nbody;
        const double px = __shfl(cen[0], 4 * pq, 64), py = __shfl(cen[1], 4 * pq, 64),
                     pz = __shfl(cen[2], 4 * pq, 64);
        const int pb = __shfl(body, 4 * pq, 64);
        bool cand = base + l < npair && po != pb;
        {
          const double* bb = b.b_diag + 16 * pb + 2;
          const double* ob = b.b_diag + 16 * po + 2;
          const double* os = b.b_diag + 16 * po + 9;
#pragma unroll
          for (int k = 0; k < 3; k++)
            if (bb[k] > ob[3 + k] + 1.0 || ob[k] > bb[3 + k] + 1.0) cand = false;
          if (px < ob[0] - 1.0 || px > ob[3] + 1.0 || py < ob[1] - 1.0 || py > ob[4] + 1.0 ||
              pz < ob[2] - 1.0 || pz > ob[5] + 1.0)
            cand = false;
          const double sx = px - os[0], sy = py - os[1], sz = pz - os[2];
          if (sx * sx + sy * sy + sz * sz > (os[3] + 1.0) * (os[3] + 1.0)) cand = false;
        }
        unsigned long long m = __ballot(cand);
        while (m) {
          const int bit = __ffsll((unsigned long long)m) - 1;
          m &= m - 1;
          const int q = (base + bit) / b.nbody, o = base + bit - q * b.nbody;
          if (q != cur_q) {
            if (cur_q >= 0) {
              const double tot = red64(part);
              if ((l >> 2) == cur_q) acc = tot;
            }
            cur_q = q;
            part = 0.0;
          }
          const double qx = __shfl(cen[0], 4 * q, 64), qy = __shfl(cen[1], 4 * q, 64),
                       qz = __shfl(cen[2], 4 * q, 64);
          // the lanes test o's chunks in parallel (a centroid c of a chunk
          // has floor(c + 1/2) inside the chunk's box of bases, so a face
          // farther than 1.5 from that box has no partner there); the
          // surviving chunks are scanned one centroid per lane (centroids
          // are stored by slot)
          const int c0 = b.b_chunk0[o], c1 = b.b_chunk0[o + 1] - 1;
          for (int cb0 = c0; cb0 <= c1; cb0 += 64) {
            bool near = false;
            if (cb0 + l <= c1) {
              const int* cb = b.chunk_box + 6 * (cb0 + l);
              near = !(qx < cb[0] - 1.5 || qx > cb[3] + 1.5 || qy < cb[1] - 1.5 || qy > cb[4] + 1.5 ||
                       qz < cb[2] - 1.5 || qz > cb[5] + 1.5);
            }
            unsigned long long mc = __ballot(near);
            while (mc) {
              const int cbit = __ffsll((unsigned long long)mc) - 1;
              mc &= mc - 1;
              const int cb = cb0 + cbit;
              if (l < b.chunk_n[cb]) {
                const int g = b.chunk_s0[cb] + l;
                const double* cj = b.centroid + 3 * g;
                const double ddx = qx - cj[0], ddy = qy - cj[1], ddz = qz - cj[2];
                const double d = sqrt(ddx * ddx + ddy * ddy + ddz * ddz);
                if (d < 1.0 && d > 0.0) part += 1.0 / sqrt(d * d * d * d * d);
              }
            }
          }
        }
      }
      if (cur_q >= 0) {
        const double tot = red64(part);
        if ((l >> 2) == cur_q) acc = tot;
      }
    }
    if (l < 32 && sub == 0 && valid) {
      const double nu = b.nu;
      const double dp = (rfit - r_in) / 3.0;
      double F[3];
#pragma unroll
      for (int i = 0; i < 3; i++) {
        double tn = 0.0;
#pragma unroll
        for (int c = 0; c < 3; c++) {
          const double tp = rfit * nu * (G[i][c] + G[c][i]);
          const double tm = r_in * nu * (Gin[i][c] + Gin[c][i]);
          tn += (tp - tm) * nrm[c];
        }
        F[i] = (-dp * nrm[i] + tn) * area;
      }
      const double pref = b.umax / (8.0 * sqrt(2.0));
      const double cv = rigid ? 0.0 : kv * (1.0 - V / V0) * area;
      double Ft[3];
#pragma unroll
      for (int i = 0; i < 3; i++) {
        Ft[i] = F[i] - pref * acc * nrm[i] + cv * nrm[i];
        b.fext[6 * f + i] = Ft[i];
        b.fext[6 * f + 3 + i] = cen[i];
      }
      // a third of the face force at each of its vertices
#pragma unroll
      for (int r = 0; r < 3; r++) {
        const long long sl = fsl[r];
        const int vr = fvx[r];
#pragma unroll
        for (int i = 0; i < 3; i++) b.f_slot[(sl * 3 + i) * b.nv + vr] = Ft[i] * (1.0 / 3.0);
      }
    }
    return;
  }
  if (b.nsoft_v == 0) return;
  const int idx = (gw - nfw) * MLS_VERTS_PER_WAVE + (l >> 2);
  const bool valid = idx < b.nsoft_v;
  const int v = b.soft_vlist[valid ? idx : b.nsoft_v - 1];
  double rfit, U[3], G[3][3];
  const double xv[3] = {b.Xcur[3 * v], b.Xcur[3 * v + 1], b.Xcur[3 * v + 2]};
  fit_point<S, false>(a, halt, sub, xv, rfit, U, G);
  if (valid && sub == 0 && !halt) {
    b.u0v[3 * v] = U[0];
    b.u0v[3 * v + 1] = U[1];
    b.u0v[3 * v + 2] = U[2];
  }
}

// Blocks of the probe / vertex-velocity part of the launch.
__host__ __device__ __forceinline__ int mls_post_blocks(const BodyArgs& b) {
  const long long waves = (long long)(b.nf + MLS_FACES_PER_WAVE - 1) / MLS_FACES_PER_WAVE +
                          (b.nsoft_v + MLS_VERTS_PER_WAVE - 1) / MLS_VERTS_PER_WAVE;
  return (int)((waves * 64 + 255) / 256);
}

// The launch also clears the force tiles of the previous step (the buffer
// the next step spreads into).  It runs after the forcing launch has checked
// the positions: a damage stop raised there skips this launch, so the force
// of the last completed step survives the stop.
template <class S>
__device__ __forceinline__ void mls_post_unit(const FluidArgs& a, const BodyArgs& b, long long* fxp,
                                              uint8_t* tfp, int blk) {
  const unsigned int halt = halted(a.flags, a.par);
  const int nm = mls_post_blocks(b);
  if (blk < nm) mls_post_block<S>(a, b, blk, halt);
  else if (!halt) clear_tiles(a.g, fxp, tfp, blk - nm, b.n_clear_blocks);
}

template <class S>
__global__ __launch_bounds__(256) void k_mls_post(FluidArgs a, BodyArgs b, long long* fxp, uint8_t* tfp) {
  mls_post_unit<S>(a, b, fxp, tfp, blockIdx.x);
}

// ----------------------------------------------------------- k_body_post
__device__ void rodrigues(const double* phi, double* R) {
  const double th = sqrt(phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2]);
  if (th == 0.0) {
    for (int k = 0; k < 9; k++) R[k] = (k % 4 == 0) ? 1.0 : 0.0;
    return;
  }
  const double k0 = phi[0] / th, k1 = phi[1] / th, k2 = phi[2] / th;
  const double c = cos(th), sn = sin(th), omc = 2.0 * sin(0.5 * th) * sin(0.5 * th);
  const double kk[3] = {k0, k1, k2};
  const double K[9] = {0, -k2, k1, k2, 0, -k0, -k1, k0, 0};
  for (int i = 0; i < 3; i++)
    for (int j = 0; j < 3; j++) R[3 * i + j] = (i == j ? c : 0.0) + sn * K[3 * i + j] + omc * kk[i] * kk[j];
}

__device__ double det3(const double* A) {
  return A[0] * (A[4] * A[8] - A[5] * A[7]) - A[1] * (A[3] * A[8] - A[5] * A[6]) +
         A[2] * (A[3] * A[7] - A[4] * A[6]);
}

// Rigid body (one block): total force and moment about the centre of mass
// (a third of a face's force at each of its vertices: the whole of it at the
// centroid), second-order backward update of u and omega (Eq. angularVelRig
// with the Newton-Euler system, inertia rotated with the body), x_c += u,
// rotation by omega (Rodrigues).  Latency-bound: the launch has 256 threads
// per block when a body is rigid, the face forces come with their centroids
// (one load round instead of three), the six sums share one pass over LDS.
__device__ void rigid_block(const BodyArgs& b, int body, unsigned int halt) {
  __shared__ double sh[4][6];
  __shared__ double rs[32];
  const int v0 = b.b_vert0[body], nv = b.b_nv[body];
  double* st = b.b_rig + 32 * body;
  if (b.b_fixed[body]) {
    if (halt) return;
    for (int v = threadIdx.x; v < nv; v += blockDim.x)
      for (int k = 0; k < 3; k++) {
        b.Xnext[3 * (v0 + v) + k] = b.Xcur[3 * (v0 + v) + k];
        b.Vel[3 * (v0 + v) + k] = 0.0;
      }
    return;
  }
  const int f0 = b.b_face0[body], nf = b.b_nf[body];
  double S[6] = {0, 0, 0, 0, 0, 0};  // force, moment
  const double xc[3] = {st[0], st[1], st[2]};
  double stl[24], Ibm[9];  // thread 0's: the state and the body-frame inertia tensor
  double mass = 1.0;
  if (threadIdx.x == 0) {
    for (int k = 0; k < 24; k++) stl[k] = st[k];
    for (int k = 0; k < 9; k++) Ibm[k] = b.b_param[8 * b.nbody + 9 * body + k];
    mass = b.b_param[8 * body + 4];
  }
#pragma unroll 4
  for (int f = threadIdx.x; f < nf; f += blockDim.x) {
    const double* Ff = b.fext + 6 * (long long)(f0 + f);
    const double F[3] = {Ff[0], Ff[1], Ff[2]};
    const double r[3] = {Ff[3] - xc[0], Ff[4] - xc[1], Ff[5] - xc[2]};
    double t[3];
    cross3(r, F, t);
    for (int k = 0; k < 3; k++) {
      S[k] += F[k];
      S[3 + k] += t[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 6; k++) S[k] = red64(S[k]);
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 6; k++) sh[threadIdx.x >> 6][k] = S[k];
  __syncthreads();
  if (halt) return;
  if (threadIdx.x == 0) {
    // state: x_c 0-2, u 3-5, u_prev 6-8, omega 9-11, omega_prev 12-14, R 15-23
    double F[3] = {0, 0, 0}, M[3] = {0, 0, 0};
    for (int w = 0; w < (int)(blockDim.x >> 6); w++)
      for (int k = 0; k < 3; k++) {
        F[k] += sh[w][k];
        M[k] += sh[w][3 + k];
      }
    const double* R = stl + 15;
    double RI[9], Iw[9];
    for (int i = 0; i < 3; i++)
      for (int j = 0; j < 3; j++) {
        double v = 0.0;
        for (int k = 0; k < 3; k++) v += R[3 * i + k] * Ibm[3 * k + j];
        RI[3 * i + j] = v;
      }
    for (int i = 0; i < 3; i++)
      for (int j = 0; j < 3; j++) {
        double v = 0.0;
        for (int k = 0; k < 3; k++) v += RI[3 * i + k] * R[3 * j + k];
        Iw[3 * i + j] = v;
      }
    double al[3];
    const double dI = det3(Iw);
    for (int c = 0; c < 3; c++) {
      double Mm[9];
      for (int k = 0; k < 9; k++) Mm[k] = Iw[k];
      for (int r = 0; r < 3; r++) Mm[3 * r + c] = M[r];
      al[c] = det3(Mm) / dI;
    }
    double un[3], wn[3];
    for (int k = 0; k < 3; k++) {
      un[k] = 2.0 / 3.0 * (2.0 * stl[3 + k] - 0.5 * stl[6 + k] + F[k] / mass);
      wn[k] = 2.0 / 3.0 * (2.0 * stl[9 + k] - 0.5 * stl[12 + k] + al[k]);
    }
    for (int k = 0; k < 3; k++) {
      stl[6 + k] = stl[3 + k];
      stl[3 + k] = un[k];
      stl[12 + k] = stl[9 + k];
      stl[9 + k] = wn[k];
      stl[k] += un[k];
    }
    double Rr[9], Rn[9];
    rodrigues(wn, Rr);
    for (int i = 0; i < 3; i++)
      for (int j = 0; j < 3; j++) {
        double v = 0.0;
        for (int k = 0; k < 3; k++) v += Rr[3 * i + k] * R[3 * k + j];
        Rn[3 * i + j] = v;
      }
    for (int k = 0; k < 9; k++) stl[15 + k] = Rn[k];
    for (int k = 0; k < 24; k++) rs[k] = st[k] = stl[k];
  }
  __syncthreads();
  for (int v = threadIdx.x; v < nv; v += blockDim.x) {
    const double* Xb = b.Xbody + 3 * (v0 + v);
    double r[3], wr[3];
    for (int i = 0; i < 3; i++) r[i] = rs[15 + 3 * i] * Xb[0] + rs[15 + 3 * i + 1] * Xb[1] + rs[15 + 3 * i + 2] * Xb[2];
    cross3(rs + 9, r, wr);
    for (int k = 0; k < 3; k++) {
      b.Xnext[3 * (v0 + v) + k] = rs[k] + r[k];
      b.Vel[3 * (v0 + v) + k] = rs[3 + k] + wr[k];
    }
  }
}

// Soft vertex: gather the element forces (stretching per edge, bending per
// hinge, one third of each face's volume + hydrodynamic + repulsion force),
// then the Verlet update with the MLS tentative velocity (Eqs. verletPos,
// verletVel, verletPosC, dt = 1).
template <int NS>
__device__ __forceinline__ void soft_vertex(const BodyArgs& b, int idx, unsigned int halt) {
  const int v = b.soft_vlist[idx];
  const int body = b.vert_body[v];
  const double* x = b.Xcur;
  // sum of the element forces written into this vertex's slots (stretching,
  // bending, a third of each incident face's force), in slot order; the
  // slot-major layout makes every load coalesced across the wave
  double F[3] = {0.0, 0.0, 0.0};
  double val[NS][3];
#pragma unroll
  for (int k = 0; k < NS; k++)
#pragma unroll
    for (int c = 0; c < 3; c++) val[k][c] = b.f_slot[((long long)k * 3 + c) * b.nv + v];
  double xv[3], u0[3], xp[3];
#pragma unroll
  for (int k = 0; k < 3; k++) {
    xv[k] = x[3 * v + k];
    u0[k] = b.u0v[3 * v + k];
    xp[k] = b.Xnext[3 * v + k];
  }
  const double mv = b.b_param[8 * body + 3];
#pragma unroll
  for (int k = 0; k < NS; k++)
#pragma unroll
    for (int c = 0; c < 3; c++) F[c] += val[k][c];
  if (halt) return;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const double acc = 0.5 * F[k] / mv;
    const double xt = xv[k] + u0[k] + acc;                    // predictor
    const double un = 1.5 * xt - 2.0 * xv[k] + 0.5 * xp[k];  // velocity
    b.Xnext[3 * v + k] = xv[k] + un + acc;                    // corrector
    b.Vel[3 * v + k] = un;
  }
}

// Last IB launch of a coupled step, in units: one per body (rigid ones), then
// 64 soft vertices each, one per thread (few vertices per block: their loads
// are spread over many CUs).  With rigid bodies the blocks have 256 threads,
// of which the soft units use the first wave.  The first unit closes the
// step, without waiting for the others: nothing of the next step depends on
// the count, and a bit raised in this step stops the next one (DevFlags).
// Counting the blocks and closing in the last one instead cost each block a
// wait for its stores and the last one three more round trips; a one-thread
// launch of its own 4.6 us.
// Measured per launch, before -> after: one capsule 6.1 -> 4.8 us, the train
// with a rigid sphere of 1280 faces 22.5 -> 9.7, a small rigid sphere in FP64
// 9.0 -> 5.9, 16 capsules 10.1 + 4.6 (closing launch) -> 7.0, a sweep of ten
// instances 6.3 + 4.6 -> 5.1.
__device__ __forceinline__ void body_post_unit(const BodyArgs& b, int u, unsigned int halt) {
  if (u < b.nbody) {
    if (b.n_rigid && b.b_rigid[u]) rigid_block(b, u, halt);
  } else {
    const int idx = (u - b.nbody) * 64 + threadIdx.x;
    if (threadIdx.x < 64 && idx < b.nsoft_v) {
      if (b.nslot == VT_SLOTS_LOW) soft_vertex<VT_SLOTS_LOW>(b, idx, halt);
      else soft_vertex<VT_SLOTS>(b, idx, halt);
    }
  }
}

__global__ __launch_bounds__(256) void k_body_post(BodyArgs b, DevFlags* flags, int close) {
  const unsigned int halt = halted(flags, b.par);
  body_post_unit(b, blockIdx.x, halt);
  if (close && blockIdx.x == 0 && threadIdx.x == 0) close_step(flags, halt);
}

// ------------------------------------------------------------ batches
// A batch advances independent contexts together: each phase of a coupled
// step is one launch over the work units of all of them.  Block g of a
// phase takes unit map[g] = (instance, block of that instance's own launch);
// the instance's arguments are read from a device table (per step parity).
// The tables are read through the constant address space: with a uniform
// address such a load is a scalar load into SGPRs, and the compiler may
// reload a field where it is used instead of holding it (a plain global
// pointer gets vector loads, and every field then held in a VGPR).
typedef const __attribute__((address_space(4))) BatchItem CBatchItem;
typedef const __attribute__((address_space(4))) int CInt;
__device__ __forceinline__ int2 batch_unit_at(const int2* map, int u) {
  const CInt* p = (const CInt*)map;
  return make_int2(p[2 * u], p[2 * u + 1]);
}
__device__ __forceinline__ int2 batch_unit(const int2* map) { return batch_unit_at(map, blockIdx.x); }
__device__ __forceinline__ const BatchItem& batch_item(const BatchItem* items, int k) {
  return *(const BatchItem*)&((CBatchItem*)items)[k];
}

template <class S>
__global__ __launch_bounds__(256, 2) void kb_ib_force(const BatchItem* items,
                                                                          const int2* map) {
  const int2 m = batch_unit(map);
  const BatchItem& it = batch_item(items, m.x);
  ib_force_block<S>(it.a, it.b, it.fxc, it.tfc, it.counter, m.y);
}

// Fluid phase.  Merged form: records and bulk tiles of every instance in
// one launch (unit = record block or bulk tile).  Split form: the record
// blocks of all instances, then the bulk tiles of all instances, each
// kernel with its own register budget (the bulk kernel keeps the occupancy
// that the bandwidth-bound part needs).  The host orders every map so that
// each XCD takes a contiguous run of units (whole instances where possible).
template <class S, int V, bool PERX>
__global__ __launch_bounds__(256) void kb_fluid_all(const BatchItem* items, const int2* map, int close) {
  const int2 m = batch_unit(map);
  const FluidArgs a = batch_item(items, m.x).a;
  const int nrb = batch_item(items, m.x).nrb;
  const unsigned int halt = halted(a.flags, a.par);
  if (close && a.close_step && m.y == (a.close_step == 1 ? nrb : 0) && threadIdx.x == 0) close_step(a.flags, halt);
  fluid_unit<S, V, PERX>(a, nrb, m.y, halt);
}

// Persistent form (its own kernel: holding an instance's arguments across
// units takes registers the one-unit form does not need): per_xcd blocks on
// each of the 8 XCDs walk the XCD's contiguous share of the units; an
// instance's arguments are loaded once per run of its units.
template <class S, int V, bool PERX>
__global__ __launch_bounds__(256) void kb_fluid_all_persist(const BatchItem* items, const int2* map,
                                                            int nunits, int per_xcd, int close) {
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int u0 = (int)(((long long)nunits * x) >> 3), u1 = (int)(((long long)nunits * (x + 1)) >> 3);
  int cur = -1, nrb = 0;
  unsigned int halt = 1u;
  FluidArgs a;
  for (int u = u0 + j; u < u1; u += per_xcd) {
    const int2 m = batch_unit_at(map, u);
    if (m.x != cur) {
      cur = m.x;
      a = batch_item(items, m.x).a;
      nrb = batch_item(items, m.x).nrb;
      halt = halted(a.flags, a.par);
    }
    if (close && a.close_step && m.y == (a.close_step == 1 ? nrb : 0) && threadIdx.x == 0) close_step(a.flags, halt);
    if (!halt) fluid_unit<S, V, PERX>(a, nrb, m.y, 0u);
    __syncthreads();  // the next unit reuses the records' LDS
  }
}

template <class S>
__global__ __launch_bounds__(256) void kb_fluid_rec(const BatchItem* items, const int2* map, int close) {
  const int2 m = batch_unit(map);
  const FluidArgs a = batch_item(items, m.x).a;
  const unsigned int halt = halted(a.flags, a.par);
  if (close && a.close_step == 2 && m.y == 0 && threadIdx.x == 0) close_step(a.flags, halt);
  fluid_record_block<S>(a, m.y, halt);
}

// Bulk tiles; per_xcd > 0 is the persistent form: per_xcd blocks on each of
// the 8 XCDs walk the XCD's contiguous share of the units in strides of
// per_xcd.
template <class S, int V, bool PERX>
__global__ __launch_bounds__(256) void kb_fluid_bulk(const BatchItem* items, const int2* map, int close) {
  const int2 m = batch_unit(map);
  const FluidArgs a = batch_item(items, m.x).a;
  const unsigned int halt = halted(a.flags, a.par);
  if (close && a.close_step == 1 && m.y == 0 && threadIdx.x == 0) close_step(a.flags, halt);
  fluid_bulk<S, V, PERX>(a, m.y, halt);
}

template <class S, int V, bool PERX>
__global__ __launch_bounds__(256) void kb_fluid_bulk_persist(const BatchItem* items, const int2* map,
                                                             int nunits, int per_xcd, int close) {
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int u0 = (int)(((long long)nunits * x) >> 3), u1 = (int)(((long long)nunits * (x + 1)) >> 3);
  int cur = -1;
  unsigned int halt = 1u;
  FluidArgs a;
  for (int u = u0 + j; u < u1; u += per_xcd) {
    const int2 m = batch_unit_at(map, u);
    if (m.x != cur) {  // an instance's arguments once per run of its units
      cur = m.x;
      a = batch_item(items, m.x).a;
      halt = halted(a.flags, a.par);
    }
    if (close && a.close_step == 1 && m.y == 0 && threadIdx.x == 0) close_step(a.flags, halt);
    if (!halt) fluid_bulk<S, V, PERX>(a, m.y, 0u);
  }
}

template <class S>
__global__ __launch_bounds__(256) void kb_mls_post(const BatchItem* items, const int2* map) {
  const int2 m = batch_unit(map);
  const BatchItem& it = batch_item(items, m.x);
  mls_post_unit<S>(it.a, it.b, it.fxp, it.tfp, m.y);
}

__global__ __launch_bounds__(256) void kb_body_post(const BatchItem* items, const int2* map) {
  const int2 m = batch_unit(map);
  const BatchItem& it = batch_item(items, m.x);
  const unsigned int halt = halted(it.a.flags, it.a.par);
  body_post_unit(it.b, m.y, halt);
  if (m.y == 0 && threadIdx.x == 0) close_step(it.a.flags, halt);
}

// ------------------------------------------------------------ API kernels
template <class S>
__global__ void k_get_fields(Grid G, const S* f0, const S* f1, const uint8_t* ncls,
                             const long long* fx0, const long long* fx1, const uint8_t* tf0,
                             const uint8_t* tf1, double gx, double gy, double gz,
                             const DevFlags* flags, double* rho, double* u, double* pops,
                             double* fib) {
  const long long N = (long long)G.nx * G.ny * G.nz;
  long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (n >= N) return;
  const long long sd = flags->steps_done;
  const S* f = (sd & 1) ? f1 : f0;
  const int lp = (int)((sd - 1) & 1);
  const long long* fx = sd > 0 ? (lp ? fx1 : fx0) : nullptr;
  const uint8_t* tf = sd > 0 ? (lp ? tf1 : tf0) : nullptr;
  int x = (int)(n % G.nx);
  long long t = n / G.nx;
  int y = (int)(t % G.ny), z = (int)(t / G.ny);
  long long p = x + (long long)G.px * (y + (long long)G.ny * z);
  const bool solid = ncls[p] == CLS_SOLID;
  double bgx = sd > 0 ? gx : 0.0, bgy = sd > 0 ? gy : 0.0, bgz = sd > 0 ? gz : 0.0;
  if (rho || u) {
    double r = 0, ux = 0, uy = 0, uz = 0;
    if (!solid) macro_at<S>(G, f, fx, tf, bgx, bgy, bgz, p, r, ux, uy, uz);
    if (rho) rho[n] = r;
    if (u) {
      u[n] = ux;
      u[N + n] = uy;
      u[2 * N + n] = uz;
    }
  }
  if (pops)
    for (int i = 0; i < 19; i++)
      pops[(long long)i * N + n] = solid ? 0.0 : (double)to_c(f[(long long)i * G.plane + p]) + WD[i];
  if (fib) {
    const bool fl = fx && tf && tf[p >> TILE_SHIFT];
    for (int c = 0; c < 3; c++) fib[(long long)c * N + n] = fl ? (double)fx[c * G.Np + p] * FX_INV : 0.0;
  }
}

template <class S>
__global__ __launch_bounds__(256) void k_interp(Grid G, const S* f0, const S* f1,
                                                const uint8_t* ncls, const long long* fx0,
                                                const long long* fx1, const uint8_t* tf0,
                                                const uint8_t* tf1, double gx, double gy,
                                                double gz, const DevFlags* flags, long long n,
                                                const double* pts, const double* field,
                                                double* out) {
  const long long m = (blockIdx.x * 256LL + threadIdx.x) >> 5;
  const int lane = threadIdx.x & 31;
  if (m >= n) return;
  const long long N = (long long)G.nx * G.ny * G.nz;
  const Slot s = stencil_slot(G, ncls, pts[3 * m], pts[3 * m + 1], pts[3 * m + 2], lane);
  double u[3] = {0.0, 0.0, 0.0};
  if (s.valid) {
    if (field) {
      int x, y, z;
      coords(G, s.node, x, y, z);
      const long long ln = x + (long long)G.nx * (y + (long long)G.ny * z);
      u[0] = field[ln];
      u[1] = field[N + ln];
      u[2] = field[2 * N + ln];
    } else {
      const long long sd = flags->steps_done;
      const S* f = (sd & 1) ? f1 : f0;
      const int lp = (int)((sd - 1) & 1);
      const long long* fx = sd > 0 ? (lp ? fx1 : fx0) : nullptr;
      const uint8_t* tf = sd > 0 ? (lp ? tf1 : tf0) : nullptr;
      double r;
      macro_at<S>(G, f, fx, tf, sd > 0 ? gx : 0.0, sd > 0 ? gy : 0.0, sd > 0 ? gz : 0.0, s.node,
                  r, u[0], u[1], u[2]);
    }
  }
  double psi[4];
  mls_psi(s, psi);
  double U[3];
  for (int k = 0; k < 3; k++) U[k] = red32(psi[0] * u[k]);
  if (lane == 0)
    for (int k = 0; k < 3; k++) out[3 * m + k] = U[k];
}

__global__ __launch_bounds__(256) void k_spread_api(Grid G, const uint8_t* ncls, long long n,
                                                    const double* pts, const double* F,
                                                    const double* c, long long* fx,
                                                    DevFlags* flags) {
  const long long m = (blockIdx.x * 256LL + threadIdx.x) >> 5;
  const int lane = threadIdx.x & 31;
  if (m >= n) return;
  const Slot s = stencil_slot(G, ncls, pts[3 * m], pts[3 * m + 1], pts[3 * m + 2], lane);
  double psi[4];
  mls_psi(s, psi);
  if (s.valid && psi[0] != 0.0) {
    const double cp = c[m] * psi[0];
    fx_add(fx + s.node, cp * F[3 * m], flags);
    fx_add(fx + G.Np + s.node, cp * F[3 * m + 1], flags);
    fx_add(fx + 2 * G.Np + s.node, cp * F[3 * m + 2], flags);
  }
}

__global__ void k_flush_fx(Grid G, long long* fx, double* fib) {
  const long long N = (long long)G.nx * G.ny * G.nz;
  long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (n >= N) return;
  int x = (int)(n % G.nx);
  long long t = n / G.nx;
  int y = (int)(t % G.ny), z = (int)(t / G.ny);
  long long p = x + (long long)G.px * (y + (long long)G.ny * z);
  for (int c = 0; c < 3; c++) {
    long long v = fx[c * G.Np + p];
    if (v != 0) {
      fib[c * N + n] += (double)v * FX_INV;
      fx[c * G.Np + p] = 0;
    }
  }
}

// --------------------------------------------------------------- launchers
#define DISPATCH(prec, KER, ...)                                 \
  switch (prec) {                                                \
    case 0: KER<double> __VA_ARGS__; break;                      \
    case 1: KER<float> __VA_ARGS__; break;                       \
    default: KER<_Float16> __VA_ARGS__; break;                   \
  }

static inline unsigned cdiv(long long a, long long b) { return (unsigned)((a + b - 1) / b); }

// Dynamic LDS of a launch whose record blocks have this many threads.
template <class S>
static unsigned link_lds(const FluidArgs& a, int block) {
  return (unsigned)((block == 64 ? a.lds_links[0] : (block == 128 ? a.lds_links[1] : a.lds_links[2])) *
                    sizeof(typename Store<S>::C));
}

hipError_t launch_init(int prec, const Grid& g, void* f, const uint8_t* ncls, const double* rho,
                       const double* u, hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  switch (prec) {
    case 0: k_init<double><<<cdiv(N, 256), 256, 0, s>>>(g, (double*)f, ncls, rho, u); break;
    case 1: k_init<float><<<cdiv(N, 256), 256, 0, s>>>(g, (float*)f, ncls, rho, u); break;
    default: k_init<_Float16><<<cdiv(N, 256), 256, 0, s>>>(g, (_Float16*)f, ncls, rho, u); break;
  }
  return hipGetLastError();
}

template <class S, int V>
static void bulk_launch(const FluidArgs& a, unsigned grid, hipStream_t s) {
  if (a.g.per[0]) k_fluid_bulk<S, V, true><<<grid, a.bulk_block, 0, s>>>(a);
  else k_fluid_bulk<S, V, false><<<grid, a.bulk_block, 0, s>>>(a);
}

hipError_t launch_fluid_bulk(int prec, const FluidArgs& a, hipStream_t s) {
  if (a.nbulk_blocks == 0) return hipSuccess;
  const unsigned grid = (unsigned)a.nbulk_blocks;
  switch (prec * 16 + (a.bulk_v == 0 ? 1 : a.bulk_v)) {  // 0: list form, one node per thread
    case 0 * 16 + 1: bulk_launch<double, 1>(a, grid, s); break;
    case 0 * 16 + 2: bulk_launch<double, 2>(a, grid, s); break;
    case 1 * 16 + 1: bulk_launch<float, 1>(a, grid, s); break;
    case 1 * 16 + 2: bulk_launch<float, 2>(a, grid, s); break;
    case 1 * 16 + 4: bulk_launch<float, 4>(a, grid, s); break;
    case 2 * 16 + 1: bulk_launch<_Float16, 1>(a, grid, s); break;
    case 2 * 16 + 2: bulk_launch<_Float16, 2>(a, grid, s); break;
    case 2 * 16 + 4: bulk_launch<_Float16, 4>(a, grid, s); break;
    case 2 * 16 + 8: bulk_launch<_Float16, 8>(a, grid, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_mac_solid(int prec, const Grid& g, void* mac, const uint8_t* ncls, hipStream_t s) {
  if (prec == 0) k_mac_solid<double><<<cdiv(g.Np, 256), 256, 0, s>>>(g, (double*)mac, ncls);
  else k_mac_solid<float><<<cdiv(g.Np, 256), 256, 0, s>>>(g, (float*)mac, ncls);
  return hipGetLastError();
}

hipError_t launch_fluid_rec(int prec, const FluidArgs& a, hipStream_t s) {
  if (a.nrec == 0) return hipSuccess;
  const unsigned grid = cdiv(a.nrec, a.rec_block);
  const unsigned blk = (unsigned)a.rec_block;
  switch (prec) {
    case 0: k_fluid_rec<double><<<grid, blk, link_lds<double>(a, blk), s>>>(a); break;
    case 1: k_fluid_rec<float><<<grid, blk, link_lds<float>(a, blk), s>>>(a); break;
    default: k_fluid_rec<_Float16><<<grid, blk, link_lds<_Float16>(a, blk), s>>>(a); break;
  }
  return hipGetLastError();
}

template <class S, int V>
static void all_launch(const FluidArgs& a, int nrb, unsigned grid, hipStream_t s) {
  const unsigned lds = nrb > 0 ? link_lds<S>(a, a.bulk_block) : 0u;
  if (a.g.per[0]) k_fluid_all<S, V, true><<<grid, a.bulk_block, lds, s>>>(a, nrb);
  else k_fluid_all<S, V, false><<<grid, a.bulk_block, lds, s>>>(a, nrb);
}

hipError_t launch_fluid_all(int prec, const FluidArgs& a, hipStream_t s) {
  // no boundary records (an all-fluid periodic box): the bulk kernel, which
  // has the smaller register budget (FP64: 76 registers against 131)
  if (a.nrec == 0) return launch_fluid_bulk(prec, a, s);
  const int nrb = a.nrec > 0 ? (int)cdiv(a.nrec, a.bulk_block) : 0;
  const unsigned grid = (unsigned)(nrb + a.nbulk_blocks);
  if (grid == 0) return hipSuccess;
  switch (prec * 16 + (a.bulk_v == 0 ? 1 : a.bulk_v)) {  // 0: list form
    case 0 * 16 + 1: all_launch<double, 1>(a, nrb, grid, s); break;
    case 0 * 16 + 2: all_launch<double, 2>(a, nrb, grid, s); break;
    case 1 * 16 + 1: all_launch<float, 1>(a, nrb, grid, s); break;
    case 1 * 16 + 2: all_launch<float, 2>(a, nrb, grid, s); break;
    case 1 * 16 + 4: all_launch<float, 4>(a, nrb, grid, s); break;
    case 2 * 16 + 1: all_launch<_Float16, 1>(a, nrb, grid, s); break;
    case 2 * 16 + 2: all_launch<_Float16, 2>(a, nrb, grid, s); break;
    case 2 * 16 + 4: all_launch<_Float16, 4>(a, nrb, grid, s); break;
    case 2 * 16 + 8: all_launch<_Float16, 8>(a, nrb, grid, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_close(DevFlags* flags, hipStream_t s) {
  k_close<<<1, 1, 0, s>>>(flags);
  return hipGetLastError();
}

hipError_t launch_ib_force(int prec, const FluidArgs& a, const BodyArgs& b, long long* fxc,
                           uint8_t* tfc, unsigned int* counter, hipStream_t s) {
  const unsigned grid = (unsigned)(b.n_marker_blocks + b.n_elem_blocks + b.n_diag_blocks);
  if (grid == 0) return hipSuccess;
  switch (prec) {
    case 0: k_ib_force<double><<<grid, 256, 0, s>>>(a, b, fxc, tfc, counter); break;
    case 1: k_ib_force<float><<<grid, 256, 0, s>>>(a, b, fxc, tfc, counter); break;
    default: k_ib_force<_Float16><<<grid, 256, 0, s>>>(a, b, fxc, tfc, counter); break;
  }
  return hipGetLastError();
}

hipError_t launch_mls_post(int prec, const FluidArgs& a, const BodyArgs& b, long long* fxp, uint8_t* tfp,
                           hipStream_t s) {
  if (b.nf == 0) return hipSuccess;
  const unsigned grid = (unsigned)(mls_post_blocks(b) + b.n_clear_blocks);
  switch (prec) {
    case 0: k_mls_post<double><<<grid, 256, 0, s>>>(a, b, fxp, tfp); break;
    case 1: k_mls_post<float><<<grid, 256, 0, s>>>(a, b, fxp, tfp); break;
    default: k_mls_post<_Float16><<<grid, 256, 0, s>>>(a, b, fxp, tfp); break;
  }
  return hipGetLastError();
}

hipError_t launch_body_post(const BodyArgs& b, DevFlags* flags, int close, hipStream_t s) {
  k_body_post<<<body_post_blocks(b), b.n_rigid ? 256 : 64, 0, s>>>(b, flags, close);
  return hipGetLastError();
}

hipError_t launch_batch_ib_force(int prec, const BatchItem* items, const int2* map, int n,
                                 hipStream_t s) {
  if (n == 0) return hipSuccess;
  switch (prec) {
    case 0: kb_ib_force<double><<<n, 256, 0, s>>>(items, map); break;
    case 1: kb_ib_force<float><<<n, 256, 0, s>>>(items, map); break;
    default: kb_ib_force<_Float16><<<n, 256, 0, s>>>(items, map); break;
  }
  return hipGetLastError();
}

template <class S, int V>
static void batch_fluid_launch(const BatchFluid& f, const BatchItem* items, hipStream_t s) {
  const unsigned lds = (unsigned)(f.lds_links * sizeof(typename Store<S>::C));
  if (f.mode == 0) {
    if (f.n_all && f.per_xcd > 0)
      kb_fluid_all_persist<S, V, false>
          <<<8u * f.per_xcd, f.block, lds, s>>>(items, f.map_all, f.n_all, f.per_xcd, f.close);
    else if (f.n_all)
      kb_fluid_all<S, V, false><<<f.n_all, f.block, lds, s>>>(items, f.map_all, f.close);
    return;
  }
  if (f.n_rec) kb_fluid_rec<S><<<f.n_rec, f.block, lds, s>>>(items, f.map_rec, f.close);
  if (f.n_bulk && f.per_xcd > 0)
    kb_fluid_bulk_persist<S, V, false>
        <<<8u * f.per_xcd, f.block, 0, s>>>(items, f.map_bulk, f.n_bulk, f.per_xcd, f.close);
  else if (f.n_bulk)
    kb_fluid_bulk<S, V, false><<<f.n_bulk, f.block, 0, s>>>(items, f.map_bulk, f.close);
}

hipError_t launch_batch_fluid(int prec, const BatchFluid& f, const BatchItem* items, hipStream_t s) {
  switch (prec * 16 + (f.V == 0 ? 1 : f.V)) {  // 0: list form
    case 0 * 16 + 1: batch_fluid_launch<double, 1>(f, items, s); break;
    case 0 * 16 + 2: batch_fluid_launch<double, 2>(f, items, s); break;
    case 1 * 16 + 1: batch_fluid_launch<float, 1>(f, items, s); break;
    case 1 * 16 + 2: batch_fluid_launch<float, 2>(f, items, s); break;
    case 1 * 16 + 4: batch_fluid_launch<float, 4>(f, items, s); break;
    case 2 * 16 + 1: batch_fluid_launch<_Float16, 1>(f, items, s); break;
    case 2 * 16 + 2: batch_fluid_launch<_Float16, 2>(f, items, s); break;
    case 2 * 16 + 4: batch_fluid_launch<_Float16, 4>(f, items, s); break;
    case 2 * 16 + 8: batch_fluid_launch<_Float16, 8>(f, items, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_batch_mls_post(int prec, const BatchItem* items, const int2* map, int n,
                                 hipStream_t s) {
  if (n == 0) return hipSuccess;
  switch (prec) {
    case 0: kb_mls_post<double><<<n, 256, 0, s>>>(items, map); break;
    case 1: kb_mls_post<float><<<n, 256, 0, s>>>(items, map); break;
    default: kb_mls_post<_Float16><<<n, 256, 0, s>>>(items, map); break;
  }
  return hipGetLastError();
}

hipError_t launch_batch_body_post(const BatchItem* items, const int2* map, int n, int block, hipStream_t s) {
  if (n == 0) return hipSuccess;
  kb_body_post<<<n, block, 0, s>>>(items, map);
  return hipGetLastError();
}

// Global FP64 mass and momentum of the populations of the last completed
// step: per block, each thread sums its nodes in index order, then a fixed
// tree; k_diag_final sums the blocks in a fixed order (bitwise reproducible).
constexpr int DIAG_SUM_BLOCKS = 1024;

template <class S>
__global__ __launch_bounds__(256) void k_diag_sum(Grid G, const S* f0, const S* f1, const uint8_t* ncls,
                                                  const DevFlags* flags, double* part) {
  __shared__ double sh[8];
  const S* f = (flags->steps_done & 1) ? f1 : f0;
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};  // non-solid nodes, sum of deviations, momentum
  for (long long p = blockIdx.x * 256LL + threadIdx.x; p < G.Np; p += (long long)gridDim.x * 256) {
    if (ncls[p] == CLS_SOLID) continue;
    v[0] += 1.0;
#pragma unroll
    for (int i = 0; i < 19; i++) {
      const double g = (double)to_c(f[(long long)i * G.plane + p]);
      v[1] += g;
      v[2] += EX[i] * g;
      v[3] += EY[i] * g;
      v[4] += EZ[i] * g;
    }
  }
#pragma unroll
  for (int k = 0; k < 5; k++) {
    const double t = block_sum(v[k], sh);
    if (threadIdx.x == 0) part[5 * blockIdx.x + k] = t;
  }
}

__global__ __launch_bounds__(256) void k_diag_final(const double* part, int nblk, double* out) {
  __shared__ double sh[8];
  for (int k = 0; k < 5; k++) {
    double v = 0.0;
    for (int j = threadIdx.x; j < nblk; j += blockDim.x) v += part[5 * j + k];
    v = block_sum(v, sh);
    if (threadIdx.x == 0) out[k] = v;
  }
}

hipError_t launch_diag_sums(int prec, const Grid& g, const void* f0, const void* f1, const uint8_t* ncls,
                            const DevFlags* flags, double* part, double* out, hipStream_t s) {
  switch (prec) {
    case 0: k_diag_sum<double><<<DIAG_SUM_BLOCKS, 256, 0, s>>>(g, (const double*)f0, (const double*)f1, ncls, flags, part); break;
    case 1: k_diag_sum<float><<<DIAG_SUM_BLOCKS, 256, 0, s>>>(g, (const float*)f0, (const float*)f1, ncls, flags, part); break;
    default: k_diag_sum<_Float16><<<DIAG_SUM_BLOCKS, 256, 0, s>>>(g, (const _Float16*)f0, (const _Float16*)f1, ncls, flags, part); break;
  }
  k_diag_final<<<1, 256, 0, s>>>(part, DIAG_SUM_BLOCKS, out);
  return hipGetLastError();
}

// ------------------------------------------------------------- adjoint
// Discrete adjoint of the fluid step (FP64, no bodies).  One step maps the
// post-collision deviations g^k to g^{k+1} = C(P(g^k)): P is the streaming
// (plain pulls, interpolated bounce-back, Zou-He -- affine in g^k) and C
// the forced BGK collision of each node.  Given lam = dJ/dg^{k+1}, the step
// back is mu = (dC/dh)^T lam node by node, then lam' = P^T mu.
__device__ __forceinline__ bool zh_unknown(int fc, int j) {
  const int face = fc & 7, ax = face >> 1, sg = (face & 1) ? -1 : 1;
  return fc != 0xff && sg * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j])) == 1;
}

// One forward step of the fluid in the context's precision (storage S, the
// same pull and collision as the stream-collide kernels) from a.A into a.B
// (null: only rho and u, into a.mac):
// bulk node t of a.bulk_list, or
// boundary record r.  Solid nodes are not written and no value is formed
// from their entries.  hrec (may be null): [19][nrec], the records'
// populations entering the collision (after Zou-He), kept for the step back.
template <class S>
__device__ __forceinline__ void adj_fwd_bulk_one(const FluidArgs& a, int t) {
  typedef typename Store<S>::C C;
  const Grid& G = a.g;
  const long long n = a.bulk_list[t];
  S* B = (S*)a.B;
  int x, y, z;
  coords(G, n, x, y, z);
  C g[19], dr, ux, uy, uz, Fx, Fy, Fz;
  const Hood h = hood(G, x, y, z);
#pragma unroll
  for (int j = 0; j < 19; j++) g[j] = ldA<S>(a, j, h.at(-EX[j], -EY[j], -EZ[j]));
  node_force<C>(a, n, a.tflag && a.tflag[n >> TILE_SHIFT], Fx, Fy, Fz);
  collide<C>(g, Fx, Fy, Fz, (C)a.omega, dr, ux, uy, uz);
  if (a.mac) store_mac<C>(a, n, dr, ux, uy, uz);
  if (!B) return;  // the step back needs the fields alone
#pragma unroll
  for (int j = 0; j < 19; j++) B[(long long)j * G.plane + n] = (S)g[j];
}

template <class S>
__device__ __forceinline__ void adj_fwd_rec_block(const FluidArgs& a, double* hrec, int blk) {
  typedef typename Store<S>::C C;
  C g[19], dr, ux, uy, uz, Fx, Fy, Fz;
  int n;
  bool on, flagged;
  pull_records<S>(a, blk * (int)blockDim.x, g, n, on, flagged);
  if (!on) return;
  if (hrec) {
    const int r = blk * (int)blockDim.x + threadIdx.x;
#pragma unroll
    for (int j = 0; j < 19; j++) hrec[(long long)j * a.nrec + r] = (double)g[j];
  }
  node_force<C>(a, n, flagged, Fx, Fy, Fz);
  collide<C>(g, Fx, Fy, Fz, (C)a.omega, dr, ux, uy, uz);
  if (a.mac) store_mac<C>(a, n, dr, ux, uy, uz);
  S* B = (S*)a.B;
  if (!B) return;
#pragma unroll
  for (int j = 0; j < 19; j++) B[(long long)j * a.g.plane + n] = (S)g[j];
}

// Split form: the bulk kernel keeps the small register budget of the plain
// pull; merged form (small grids): the records' latency-bound blocks run
// alongside the bulk blocks in one launch (blocks below rec_blocks take
// records).
template <class S>
__global__ __launch_bounds__(256) void k_adj_fwd_bulk(FluidArgs a) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < a.nbulk_nodes) adj_fwd_bulk_one<S>(a, t);
}

template <class S>
__global__ __launch_bounds__(256) void k_adj_fwd_rec(FluidArgs a, double* hrec) {
  adj_fwd_rec_block<S>(a, hrec, blockIdx.x);
}

// Block b of a merged launch -> record block or bulk block, each part's
// blocks remapped so that every XCD takes a contiguous run (neighbouring
// rows share its L2).
__device__ __forceinline__ int adj_unit(int b, int rec_blocks, int nblocks) {
  return b < rec_blocks ? xcd_remap(b, rec_blocks) : rec_blocks + xcd_remap(b - rec_blocks, nblocks - rec_blocks);
}

template <class S>
__global__ __launch_bounds__(256) void k_adj_fwd_all(FluidArgs a, double* hrec, int rec_blocks) {
  const int u = adj_unit(blockIdx.x, rec_blocks, gridDim.x);
  if (u < rec_blocks) {
    adj_fwd_rec_block<S>(a, hrec, u);
  } else {
    const int t = (u - rec_blocks) * 256 + threadIdx.x;
    if (t < a.nbulk_nodes) adj_fwd_bulk_one<S>(a, t);
  }
}

// The transpose of the collision's Jacobian, written out: with
// Phi = sum_i l_i (omega g^eq_i + G_i) as a function of (rho - 1, u, F),
//   P   = dPhi/d(rho - 1) at fixed u,  U_a = dPhi/du_a,  Q_a = dPhi/dF_a at fixed u,
// and du_a/dh_j = (e_ja - u_a)/rho, d(rho - 1)/dh_j = 1, du_a/dF_a = 1/(2 rho):
//   mu_j = (1 - omega) l_j + P + sum_a U_a (e_ja - u_a)/rho,
//   dJ/dF_a += Q_a + U_a/(2 rho).
// With the sums over i of w_i l_i times 1, (1 + 3 e.u + 9/2 (e.u)^2 - 3/2 u.u),
// (3 + 9 e.u) e_a and (e.F) e_a (SL, P', V_a, Z_a), all of them combinations
// of the ten moments of w_i l_i up to second order (which costs a third of the
// operations of summing each over the directions):
//   P = omega P',  U_a = omega rho V_a + 9 kf Z_a - 3 (omega rho u_a + kf F_a) SL,
//   Q_a = kf (V_a - 3 u_a SL),  kf = 1 - omega/2.
// dF[3] += dJ/d(omega) at fixed h: sum_i l_i (g^eq_i - h_i - G_i / (2 kf)).
// With bodies, x7 adds adjoint sources at the node: x7[0] = dJ/drho and
// x7[1..3] = dJ/du of the step's fields (read by the probes and the vertex
// velocities; u depends on F, so they enter dJ/dF too), x7[4..6] = dJ/du*
// of the pre-force velocity u* = m / rho that the forcing markers read
// (mu_j += dJ/du* . (e_j - u*) / rho).  dFn: this node's dJ/dF, dw: dJ/d(omega).
// The populations h enter through their moments and sum l h alone (AdjIn),
// which are formed as soon as they are loaded: h need not be held.
struct AdjIn {
  double drho, mx, my, mz, lh;
};
template <class C>
__device__ __forceinline__ AdjIn adj_in(const C (&hc)[19], const double (&l)[19]) {
  double h[19];
  AdjIn s;
  s.lh = 0.0;
#pragma unroll
  for (int j = 0; j < 19; j++) {
    h[j] = (double)hc[j];
    s.lh += l[j] * h[j];
  }
  s.drho = dev_sum(h);
  s.mx = (h[1] - h[2]) + (h[7] + h[8]) + (h[9] + h[10]) - (h[11] + h[12]) - (h[13] + h[14]);
  s.my = (h[3] - h[4]) + (h[7] - h[8]) + (h[11] - h[12]) + (h[15] + h[16]) - (h[17] + h[18]);
  s.mz = (h[5] - h[6]) + (h[9] - h[10]) + (h[13] - h[14]) + (h[15] - h[16]) + (h[17] - h[18]);
  return s;
}

// Entry i (padded index) of plane j of an adjoint field, or of a state: a
// uniform base and a 32-bit byte offset, so that a load takes one address
// register instead of two (a sweep's six FP64 fields of 19 planes fit the
// device only below 2^29 padded nodes).
template <class T>
__device__ __forceinline__ T& plane_at(T* f, const Grid& G, int j, unsigned int i) {
  return *(T*)((char*)(f + (long long)j * G.plane) + (size_t)(i * (unsigned int)sizeof(T)));
}

// mu_j = (1 - omega) l_j + A0 + e_j.(a0, a1, a2)
struct AdjOut {
  double A0, a0, a1, a2;
  __device__ __forceinline__ double mu(int j, double lj, double omega) const {
    return (1.0 - omega) * lj + A0 + (eterm(EX[j], a0) + eterm(EY[j], a1) + eterm(EZ[j], a2));
  }
};

__device__ __forceinline__ AdjOut collide_vjp(const AdjIn& in, const double (&l)[19], double Fx, double Fy, double Fz,
                                              double omega, const double (&x7)[7], double (&dFn)[3], double& dw) {
  const double drho = in.drho, mx = in.mx, my = in.my, mz = in.mz;
  const double rho = 1.0 + drho, ir = 1.0 / rho;
  const double ux = (mx + 0.5 * Fx) * ir, uy = (my + 0.5 * Fy) * ir, uz = (mz + 0.5 * Fz) * ir;
  const double usq = ux * ux + uy * uy + uz * uz;
  const double kf = 1.0 - 0.5 * omega;
  const double uF = ux * Fx + uy * Fy + uz * Fz;
  double SL = 0.0, M0 = 0.0, M1 = 0.0, M2 = 0.0, XX = 0.0, YY = 0.0, ZZ = 0.0, XY = 0.0, XZ = 0.0, YZ = 0.0;
#pragma unroll
  for (int i = 0; i < 19; i++) {
    const double wl = WD[i] * l[i];
    SL += wl;
    if (EX[i]) { M0 += EX[i] * wl; XX += wl; }
    if (EY[i]) { M1 += EY[i] * wl; YY += wl; }
    if (EZ[i]) { M2 += EZ[i] * wl; ZZ += wl; }
    if (EX[i] * EY[i]) XY += EX[i] * EY[i] * wl;
    if (EX[i] * EZ[i]) XZ += EX[i] * EZ[i] * wl;
    if (EY[i] * EZ[i]) YZ += EY[i] * EZ[i] * wl;
  }
  const double Mu0 = XX * ux + XY * uy + XZ * uz, Mu1 = XY * ux + YY * uy + YZ * uz, Mu2 = XZ * ux + YZ * uy + ZZ * uz;
  const double Z0 = XX * Fx + XY * Fy + XZ * Fz, Z1 = XY * Fx + YY * Fy + YZ * Fz, Z2 = XZ * Fx + YZ * Fy + ZZ * Fz;
  const double V0 = 3.0 * M0 + 9.0 * Mu0, V1 = 3.0 * M1 + 9.0 * Mu1, V2 = 3.0 * M2 + 9.0 * Mu2;
  // sum w l (3 e.u + 9/2 (e.u)^2 - 3/2 u.u)
  const double Pe = 3.0 * (M0 * ux + M1 * uy + M2 * uz) + 4.5 * (Mu0 * ux + Mu1 * uy + Mu2 * uz) - 1.5 * usq * SL;
  const double Pp = SL + Pe;
  // d(out_i)/d(omega) = -(h_i - g^eq_i) - 1/2 w_i (3 (e.F - u.F) + 9 (e.u)(e.F))
  const double Dw = drho * SL + rho * Pe -
                    0.5 * (3.0 * (M0 * Fx + M1 * Fy + M2 * Fz - uF * SL) + 9.0 * (Mu0 * Fx + Mu1 * Fy + Mu2 * Fz));
  const double orho = omega * rho;
  const double U0 = orho * V0 + 9.0 * kf * Z0 - 3.0 * (orho * ux + kf * Fx) * SL + x7[1];
  const double U1 = orho * V1 + 9.0 * kf * Z1 - 3.0 * (orho * uy + kf * Fy) * SL + x7[2];
  const double U2 = orho * V2 + 9.0 * kf * Z2 - 3.0 * (orho * uz + kf * Fz) * SL + x7[3];
  double A0 = omega * Pp + x7[0] - (U0 * ux + U1 * uy + U2 * uz) * ir;
  double a0 = U0 * ir, a1 = U1 * ir, a2 = U2 * ir;
  dFn[0] = kf * (V0 - 3.0 * ux * SL) + 0.5 * a0;
  dFn[1] = kf * (V1 - 3.0 * uy * SL) + 0.5 * a1;
  dFn[2] = kf * (V2 - 3.0 * uz * SL) + 0.5 * a2;
  dw = Dw - in.lh;
  // u* = m / rho (no force): mu_j += x7[4..6] . (e_j - u*) / rho
  A0 -= (x7[4] * mx + x7[5] * my + x7[6] * mz) * ir * ir;
  a0 += x7[4] * ir;
  a1 += x7[5] * ir;
  a2 += x7[6] * ir;
  return AdjOut{A0, a0, a1, a2};
}

// Zou-He's transpose (the rule of zouhe(), affine in the known populations
// for a fixed wall velocity or density): m = dJ/d(populations after the
// rule) -> dJ/d(populations before it), in place; gs += dJ/ds with s the
// scale of the wall velocity of a velocity face.  G0, Gout: the sums of the
// populations after the rule (its known entries are the ones before) with
// e.n = 0 and -1.  With c_i = 1, 2, 0 for
// e_i.n = 0, -1, +1, rho_w depends on g_i through c_i / (1 - u_n) (velocity
// face) and u_n through -c_i / rho_w (density face); the tangential sums T
// through e_i (e_i.n = 0); each unknown j adds m_j to its opposite input.
__device__ __forceinline__ void zouhe_sums(const double (&hz)[19], int face, double& G0, double& Gout) {
  const int ax = face >> 1, sg = (face & 1) ? -1 : 1;
  G0 = Gout = 0.0;
#pragma unroll
  for (int j = 0; j < 19; j++) {
    const int en = sg * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j]));
    G0 += en == 0 ? hz[j] : 0.0;
    Gout += en == -1 ? hz[j] : 0.0;
  }
}
__device__ __forceinline__ void zouhe_vjp(double G0, double Gout, double (&m)[19], int face, int kind,
                                          const double* bc, double& gs) {
  const int ax = face >> 1;
  const int sg = (face & 1) ? -1 : 1;
  double u[3] = {bc[0], bc[1], bc[2]};
  double rho, un;
  if (kind == 0) {
    un = sg * u[ax];
    rho = (1.0 + G0 + 2.0 * Gout) / (1.0 - un);
  } else {
    rho = bc[3];
    un = (rho - 1.0 - G0 - 2.0 * Gout) / rho;
    u[0] = ax == 0 ? sg * un : 0.0;
    u[1] = ax == 1 ? sg * un : 0.0;
    u[2] = ax == 2 ? sg * un : 0.0;
  }
  // R = sum over unknowns of m_j d(fill_j)/d(rho_w) (velocity face) or
  // d(fill_j)/d(u_n) (density face); W = sum over diagonal unknowns of m_j t_j
  double R = 0.0, W[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 19; j++) {
    const int en = sg * (ax == 0 ? EX[j] : (ax == 1 ? EY[j] : EZ[j]));
    if (en != 1) continue;
    const double t[3] = {ax == 0 ? 0.0 : (double)EX[j], ax == 1 ? 0.0 : (double)EY[j], ax == 2 ? 0.0 : (double)EZ[j]};
    const bool axis = t[0] == 0.0 && t[1] == 0.0 && t[2] == 0.0;
    const double ut = u[0] * t[0] + u[1] * t[1] + u[2] * t[2];
    const double coef = kind == 0 ? (axis ? un / 3.0 : (un + ut) / 6.0 + ut / 3.0) : (axis ? rho / 3.0 : rho / 6.0);
    R += m[j] * coef;
    if (!axis) {
      W[0] += m[j] * t[0];
      W[1] += m[j] * t[1];
      W[2] += m[j] * t[2];
    }
  }
  double out[19];
#pragma unroll
  for (int i = 0; i < 19; i++) {
    const int en = sg * (ax == 0 ? EX[i] : (ax == 1 ? EY[i] : EZ[i]));
    const double c = en == 0 ? 1.0 : (en == -1 ? 2.0 : 0.0);
    double v = en != 1 ? m[i] : 0.0;
    if (en == -1) v += m[OPP[i]];  // the unknown opposite copies this input
    v += R * (kind == 0 ? c / (1.0 - un) : -c / rho);
    if (en == 0) v -= 0.5 * (W[0] * EX[i] + W[1] * EY[i] + W[2] * EZ[i]);
    out[i] = v;
  }
#pragma unroll
  for (int i = 0; i < 19; i++) m[i] = out[i];
  if (kind == 0) gs += (rho * un / (1.0 - un) + rho) * R;
}


// The bounce-back transposes of a block's records (r0 + 0..255): the mu of
// each linked direction, which the records left in s_dyn by link, goes back,
// with the rule's coefficients, to the three populations the rule read (FP64
// atomics: several links may feed one).  As in pull_records the links are
// spread over the threads, and their words and coefficients are loaded in one
// batch ahead of the barrier: one record after another took its links in turn,
// three loads and a wait each (record launch of the bifurcation, 133052 links:
// 52 -> 41 us).  Every thread of the block calls.
template <class S, int NP>
__device__ __forceinline__ void adj_link_adds(const FluidArgs& a, int l0, int l1, int first, const int (&nd)[NP],
                                              const unsigned int (&w)[NP], const typename Store<S>::C (&k)[NP][3],
                                              double* acc) {
  const Grid& G = a.g;
  const double* s_m = s_dyn;
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int l = first + p * 256;
    if (l >= l1) continue;
    const double m = s_m[l - l0];
    const int j = w[p] & 31u, i = opp_of(j);
    const bool hq = (w[p] >> 5) & 1u;
    const int ex = dir_of(dir_bits(EX), j), ey = dir_of(dir_bits(EY), j), ez = dir_of(dir_bits(EZ), j);
    int x, y, z;
    coords(G, nd[p], x, y, z);
    const long long n0 = nd[p], n1 = nbr(G, x, y, z, ex, ey, ez), n2 = nbr(G, x, y, z, 2 * ex, 2 * ey, 2 * ez);
    double *ai = acc + (long long)i * G.plane, *at = hq ? acc + (long long)j * G.plane : ai;
    const double k0 = (double)k[p][0], k1 = (double)k[p][1], k2 = (double)k[p][2];
    if (k0 != 0.0) atomicAdd(ai + n0, k0 * m);
    if (k1 != 0.0) atomicAdd(at + (hq ? n0 : n1), k1 * m);
    if (k2 != 0.0) atomicAdd(at + (hq ? n1 : n2), k2 * m);
  }
}

template <class S, int NP>
__device__ __forceinline__ void adj_link_words(const FluidArgs& a, int l1, int first, int (&nd)[NP],
                                               unsigned int (&w)[NP], typename Store<S>::C (&k)[NP][3]) {
  const typename Store<S>::C* lc = (const typename Store<S>::C*)a.lk_c;
  const long long nl = a.nlinks;
#pragma unroll
  for (int p = 0; p < NP; p++) {
    const int l = max(min(first + p * 256, l1 - 1), 0);
    nd[p] = a.lk_node[l];
    w[p] = a.lk_w[l];
#pragma unroll
    for (int q = 0; q < 3; q++) k[p][q] = lc[q * nl + l];
  }
}

template <class S>
__device__ __forceinline__ void adj_links_block(const FluidArgs& a, int r0, double* acc) {
  const int l0 = a.rec_link0[r0], l1 = a.rec_link0[min(r0 + 256, a.nrec)];
  const int first = l0 + (int)threadIdx.x;
  {
    int nd[LINK_PASSES];
    unsigned int w[LINK_PASSES];
    typename Store<S>::C k[LINK_PASSES][3];
    adj_link_words<S, LINK_PASSES>(a, l1, first, nd, w, k);
    __syncthreads();
    adj_link_adds<S, LINK_PASSES>(a, l0, l1, first, nd, w, k, acc);
  }
  for (int l = first + LINK_PASSES * 256; l < l1; l += 256) {  // a block with more links than the batch holds
    int nd[1];
    unsigned int w[1];
    typename Store<S>::C k[1][3];
    adj_link_words<S, 1>(a, l1, l, nd, w, k);
    adj_link_adds<S, 1>(a, l0, l1, l, nd, w, k, acc);
  }
}

// One node of the reverse step: lam = P^T mu_next at the node (plain pulls
// transposed: mu_next of direction j at the node that pulled j from here;
// plus the bounce-back transposes gathered in acc_in), then mu = (dC/dh)^T
// (lam + w) for bulk node t of a.bulk_list (REC false) or boundary record t
// (REC true; h: the populations that entered the collision, Zou-He applied,
// as the recompute kept them in hrec; at open-face records mu is then taken
// back through Zou-He, and that of the linked directions is left in s_dyn for
// adj_links_block).  dF, gs += the node's derivatives of the body force and of
// the inlet-velocity scale.
template <bool REC, class S>
__device__ __forceinline__ void adj_reverse_one(const FluidArgs& a, const AdjStep& st, int t, double (&dF)[4],
                                                double& gs) {
  typedef typename Store<S>::C C;
  const Grid& G = a.g;
  const int n = REC ? a.rec_node[t] : a.bulk_list[t];
  const int q = REC ? a.nbulk_nodes + t : t;
  const uint32_t am = st.amask[q], pm = st.lam ? 0u : st.pmask[q];
  const int fc = REC ? a.rec_face[t] : 0xff;
  // with bodies: the IB force at the node, and whether the force-adjoint
  // pass (mode 1) has anything to do here
  // (mode 1 also visits the tiles of every marker's supports, flagged in etf
  // beforehand: dJ/dF is needed there even where the step's force is zero)
  const uint8_t fft = st.ftf ? st.ftf[n >> TILE_SHIFT] : 0, eft = st.etf ? st.etf[n >> TILE_SHIFT] : 0;
  if (st.mode == 1 && !fft && !eft) return;
  int x, y, z;
  coords(G, n, x, y, z);
  const Hood hd = hood(G, x, y, z);
  double l[19];
  if (st.lam) {
#pragma unroll
    for (int j = 0; j < 19; j++) l[j] = plane_at(st.lam, G, j, n);
  } else {
    // (a pull that another rule replaces reads the node's own entry and drops it)
#pragma unroll
    for (int j = 0; j < 19; j++) {
      const bool on = (pm >> j) & 1u;
      const double v = plane_at(st.mu_next, G, j, j == 0 || !on ? n : hd.at(EX[j], EY[j], EZ[j]));
      l[j] = on ? v : 0.0;
    }
  }
  AdjIn in;
  double G0 = 0.0, Gout = 0.0;
  double hr[REC ? 19 : 1];
  C hb[REC ? 1 : 19];
  if constexpr (REC) {
#pragma unroll
    for (int j = 0; j < 19; j++) hr[j] = st.hrec[(long long)j * a.nrec + t];
  } else {
#pragma unroll
    for (int j = 0; j < 19; j++) hb[j] = to_c(plane_at((const S*)a.A, G, j, hd.at(-EX[j], -EY[j], -EZ[j])));
  }
  if (!st.lam && (am & 0x7ffffu)) {
#pragma unroll
    for (int j = 0; j < 19; j++) {
      if ((am >> j) & 1u) {
        double& pa = plane_at(st.acc_in, G, j, n);
        l[j] += pa;
        if (st.mode == 0) pa = 0.0;
      }
    }
  }
  if (st.w && (am >> 31)) {  // w is non-zero at this node
#pragma unroll
    for (int j = 0; j < 19; j++) l[j] += plane_at(st.w, G, j, n);
  }
  double Fx = a.gx, Fy = a.gy, Fz = a.gz;
  if (fft) {
    Fx += (double)st.fx[n] * FX_INV;
    Fy += (double)st.fx[G.Np + n] * FX_INV;
    Fz += (double)st.fx[2 * G.Np + n] * FX_INV;
  }
  double x7[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (eft) {
#pragma unroll
    for (int k = 0; k < 7; k++) x7[k] = st.ext[(long long)k * G.Np + n];
  }
  if constexpr (REC) {
    in = adj_in(hr, l);
    if (fc != 0xff) zouhe_sums(hr, fc & 7, G0, Gout);
  } else {
    in = adj_in(hb, l);
  }
  double dFn[3], dw;
  const AdjOut o = collide_vjp(in, l, Fx, Fy, Fz, a.omega, x7, dFn, dw);
  if (st.mode == 1) {
#pragma unroll
    for (int k = 0; k < 3; k++) st.fbar[k * G.Np + n] = dFn[k];
    return;
  }
  dF[0] += dFn[0];
  dF[1] += dFn[1];
  dF[2] += dFn[2];
  dF[3] += dw;
  if constexpr (REC) {
#pragma unroll
    for (int j = 0; j < 19; j++) l[j] = o.mu(j, l[j], a.omega);
    if (fc != 0xff) {
      double bc[4];
      for (int k = 0; k < 4; k++) bc[k] = a.rec_bc[(long long)k * a.nrec + t];
      zouhe_vjp(G0, Gout, l, fc & 7, (fc >> 4) & 1, bc, gs);
    }
#pragma unroll
    for (int j = 0; j < 19; j++) plane_at(st.mu, G, j, n) = l[j];
    const uint32_t mask = a.rec_mask[t];
    const int lk = a.rec_link0[t] - a.rec_link0[t & ~255];
#pragma unroll
    for (int j = 1; j < 19; j++)
      if ((mask >> j) & 1u) s_dyn[lk + __popc(mask & ((1u << j) - 1u))] = l[j];
  } else {
#pragma unroll
    for (int j = 0; j < 19; j++) plane_at(st.mu, G, j, n) = o.mu(j, l[j], a.omega);
  }
}

// part[block][0..4] += the block's sums of dJ/ds, dJ/dF, dJ/d(omega)
// (fixed order: bitwise reproducible).
__device__ __forceinline__ void adj_part_add(double* part, double gs, const double (&dF)[4]) {
  __shared__ double sh[8];
  const double t0 = block_sum(gs, sh);
  const double t1 = block_sum(dF[0], sh);
  const double t2 = block_sum(dF[1], sh);
  const double t3 = block_sum(dF[2], sh);
  const double t4 = block_sum(dF[3], sh);
  if (threadIdx.x == 0) {
    double* p = part + ADJ_PART * blockIdx.x;
    p[0] += t0;
    p[1] += t1;
    p[2] += t2;
    p[3] += t3;
    p[4] += t4;
  }
}

// Split form: bulk (REC false) and records (REC true) in two launches,
// grid-stride over at most ADJ_BLOCKS blocks each (partials of the record
// launch in the second half of part).
template <bool REC, class S>
__global__ __launch_bounds__(256, 2) void k_adj_reverse(FluidArgs a, AdjStep st) {
  double dF[4] = {0.0, 0.0, 0.0, 0.0}, gs = 0.0;
  const int count = REC ? a.nrec : a.nbulk_nodes;
  for (int t0 = blockIdx.x * 256; t0 < count; t0 += gridDim.x * 256) {
    const int t = t0 + (int)threadIdx.x;
    if (t < count) adj_reverse_one<REC, S>(a, st, t, dF, gs);
    if (REC && st.mode == 0) {
      adj_links_block<S>(a, t0, st.acc_out);
      __syncthreads();  // the next records reuse the links' LDS
    }
  }
  if (st.mode == 0) adj_part_add(st.part + (REC ? ADJ_PART * ADJ_BLOCKS : 0), gs, dF);
}

// Merged form: blocks below rec_blocks take records, the rest bulk nodes.
// Bound by the waits for its loads at two waves per SIMD (221 registers; at
// the 168 of three it spills 96): bifurcation, 175612 nodes, FP32 states,
// 64 -> 51 us a step, the force-adjoint pass (mode 1) 20 -> 7.4 us.
template <class S>
__global__ __launch_bounds__(256, 2) void k_adj_reverse_all(FluidArgs a, AdjStep st, int rec_blocks) {
  double dF[4] = {0.0, 0.0, 0.0, 0.0}, gs = 0.0;
  const int u = adj_unit(blockIdx.x, rec_blocks, gridDim.x);
  if (u < rec_blocks) {
    const int t = u * 256 + threadIdx.x;
    if (t < a.nrec) adj_reverse_one<true, S>(a, st, t, dF, gs);
    if (st.mode == 0) adj_links_block<S>(a, u * 256, st.acc_out);
  } else {
    const int t = (u - rec_blocks) * 256 + threadIdx.x;
    if (t < a.nbulk_nodes) adj_reverse_one<false, S>(a, st, t, dF, gs);
  }
  if (st.mode == 0) adj_part_add(st.part, gs, dF);
}

// Per non-solid node y (bulk list, then the records), once per sweep:
// pmask bit j: node y + e_j pulls direction j plainly from y; amask bit 31:
// the observable w is non-zero at y; amask bit d < 19:
// population d of y can receive a bounce-back transpose, i.e. some link
// reads it: the link of direction opp(d) or d at y, of opp(d) at y + e_d
// or y + 2 e_d, or of d at y - e_d (a superset: the coefficient and the
// branch of each link are not looked at).
__device__ __forceinline__ bool adj_linked(const FluidArgs& a, long long x, int j) {
  if (a.ncls[x] != CLS_GENERAL) return false;
  return (a.rec_mask[a.rec_of[x]] >> j) & 1u;
}

__global__ __launch_bounds__(256) void k_adj_mask(FluidArgs a, const double* w, uint32_t* pmask, uint32_t* amask) {
  const Grid& G = a.g;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= a.nbulk_nodes + a.nrec) return;
  const long long y = t < a.nbulk_nodes ? (long long)a.bulk_list[t] : (long long)a.rec_node[t - a.nbulk_nodes];
  int px, py, pz;
  coords(G, y, px, py, pz);
  uint32_t m = 0, am = 0;
  for (int j = 0; j < 19; j++) {
    const long long x = j == 0 ? y : nbr(G, px, py, pz, EX[j], EY[j], EZ[j]);
    const uint8_t c = a.ncls[x];
    bool plain = c == CLS_BULK;
    if (c == CLS_GENERAL) {
      const int r = a.rec_of[x];
      plain = j == 0 || (!((a.rec_mask[r] >> j) & 1u) && !zh_unknown(a.rec_face[r], j));
    }
    m |= plain ? (1u << j) : 0u;
    if (j > 0) {
      const int o = OPP[j];
      const bool recv = adj_linked(a, y, o) || adj_linked(a, y, j) ||
                        adj_linked(a, nbr(G, px, py, pz, EX[j], EY[j], EZ[j]), o) ||
                        adj_linked(a, nbr(G, px, py, pz, 2 * EX[j], 2 * EY[j], 2 * EZ[j]), o) ||
                        adj_linked(a, nbr(G, px, py, pz, -EX[j], -EY[j], -EZ[j]), j);
      am |= recv ? (1u << j) : 0u;
    }
  }
  if (w) {
    bool nz = false;
    for (int j = 0; j < 19; j++) nz |= w[(long long)j * G.plane + y] != 0.0;
    am |= nz ? (1u << 31) : 0u;
  }
  pmask[t] = m;
  amask[t] = am;
}

// The last step of the sweep's transpose, lam = P^T mu: the plain pulls
// transposed plus the bounce-back transposes gathered in acc, at every
// non-solid node (bulk list, then the records).
__global__ __launch_bounds__(256) void k_adj_gather(FluidArgs a, const uint32_t* pmask, const uint32_t* amask,
                                                    const double* mu, const double* acc, double* lam) {
  const Grid& G = a.g;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= a.nbulk_nodes + a.nrec) return;
  const long long y = t < a.nbulk_nodes ? (long long)a.bulk_list[t] : (long long)a.rec_node[t - a.nbulk_nodes];
  const uint32_t m = pmask[t], am = amask[t];
  int px, py, pz;
  coords(G, y, px, py, pz);
#pragma unroll
  for (int j = 0; j < 19; j++) {
    const long long x = j == 0 ? y : nbr(G, px, py, pz, EX[j], EY[j], EZ[j]);
    double v = ((m >> j) & 1u) ? mu[(long long)j * G.plane + x] : 0.0;
    if ((am >> j) & 1u) v += acc[(long long)j * G.plane + y];
    lam[(long long)j * G.plane + y] = v;
  }
}

// [19][N] with x fastest (N = nx ny nz) <-> the padded [19][plane] layout;
// towards the padded side only the non-solid nodes are written, and solid
// ones come out zero.
__global__ void k_adj_layout(Grid G, const uint8_t* ncls, const double* in, double* out, int to_padded) {
  const long long p = blockIdx.x * 256LL + threadIdx.x;
  if (p >= G.Np) return;
  const long long N = (long long)G.nx * G.ny * G.nz;
  const unsigned int t = (unsigned int)(p / G.px);
  const int x = (int)(p - (long long)t * G.px);
  const long long n = x + (long long)G.nx * t;
  const bool solid = ncls[p] == CLS_SOLID;  // padding included
  for (int j = 0; j < 19; j++) {
    if (to_padded) {
      if (!solid) out[(long long)j * G.plane + p] = in[(long long)j * N + n];
    } else if (x < G.nx) {
      out[(long long)j * N + n] = solid ? 0.0 : in[(long long)j * G.plane + p];
    }
  }
}

// grad[0..4] = dJ/ds, dJ/dF, dJ/dtau = -omega^2 dJ/d(omega), summed over the
// blocks in a fixed order: one block, every thread its own blocks' partials,
// then a fixed tree (one thread per component took 466 us for 2800 blocks).
__global__ __launch_bounds__(256) void k_adj_grad_final(const double* part, int nblk, double omega, const double* ibsum,
                                                        int nout, double* grad) {
  __shared__ double sh[8];
  double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nblk; b += 256)
#pragma unroll
    for (int q = 0; q < 5; q++) t[q] += part[ADJ_PART * b + q];
#pragma unroll
  for (int q = 0; q < 5; q++) t[q] = block_sum(t[q], sh);
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int q = 0; q < 4; q++) grad[q] = t[q];
  grad[4] = -omega * omega * t[4] + (ibsum ? ibsum[0] : 0.0);
  if (nout > 5) grad[5] = ibsum ? ibsum[1] : 0.0;
}

template <class S>
static void adj_forward(const FluidArgs& a, double* hrec, int merged, hipStream_t s) {
  const int rb = (int)cdiv(a.nrec, 256), bb = (int)cdiv(a.nbulk_nodes, 256);
  const unsigned lds = link_lds<S>(a, 256);
  if (merged) {
    if (rb + bb > 0) k_adj_fwd_all<S><<<rb + bb, 256, lds, s>>>(a, hrec, rb);
  } else {
    if (bb > 0) k_adj_fwd_bulk<S><<<bb, 256, 0, s>>>(a);
    if (rb > 0) k_adj_fwd_rec<S><<<rb, 256, lds, s>>>(a, hrec);
  }
}

hipError_t launch_adjoint_forward(int prec, const FluidArgs& a, double* hrec, int merged, hipStream_t s) {
  if (prec == 0) adj_forward<double>(a, hrec, merged, s);
  else if (prec == 1) adj_forward<float>(a, hrec, merged, s);
  else adj_forward<_Float16>(a, hrec, merged, s);
  return hipGetLastError();
}

hipError_t launch_adjoint_mask(const FluidArgs& a, const double* w, uint32_t* pmask, uint32_t* amask,
                               hipStream_t s) {
  if (a.nbulk_nodes + a.nrec > 0) k_adj_mask<<<cdiv(a.nbulk_nodes + a.nrec, 256), 256, 0, s>>>(a, w, pmask, amask);
  return hipGetLastError();
}

template <class S>
static void adj_reverse(const FluidArgs& a, const AdjStep& st, int merged, hipStream_t s) {
  const int rb = (int)cdiv(a.nrec, 256), bb = (int)cdiv(a.nbulk_nodes, 256);
  const unsigned lds = (unsigned)(a.lds_links[2] * sizeof(double));  // a block's links
  if (merged) {
    if (rb + bb > 0) k_adj_reverse_all<S><<<rb + bb, 256, rb > 0 ? lds : 0u, s>>>(a, st, rb);
  } else {
    if (bb > 0) k_adj_reverse<false, S><<<std::min(bb, ADJ_BLOCKS), 256, 0, s>>>(a, st);
    if (rb > 0) k_adj_reverse<true, S><<<std::min(rb, ADJ_BLOCKS), 256, lds, s>>>(a, st);
  }
}

hipError_t launch_adjoint_reverse(int prec, const FluidArgs& a, const AdjStep& st, int merged, hipStream_t s) {
  if (prec == 0) adj_reverse<double>(a, st, merged, s);
  else if (prec == 1) adj_reverse<float>(a, st, merged, s);
  else adj_reverse<_Float16>(a, st, merged, s);
  return hipGetLastError();
}

hipError_t launch_adjoint_gather(const FluidArgs& a, const uint32_t* pmask, const uint32_t* amask, const double* mu,
                                 const double* acc, double* lam, hipStream_t s) {
  if (a.nbulk_nodes + a.nrec > 0) {
    k_adj_gather<<<cdiv(a.nbulk_nodes + a.nrec, 256), 256, 0, s>>>(a, pmask, amask, mu, acc, lam);
  }
  return hipGetLastError();
}

hipError_t launch_adjoint_layout(const Grid& g, const uint8_t* ncls, const double* in, double* out, int to_padded,
                                 hipStream_t s) {
  k_adj_layout<<<cdiv(g.Np, 256), 256, 0, s>>>(g, ncls, in, out, to_padded);
  return hipGetLastError();
}

hipError_t launch_adjoint_grad(const double* part, int nblk, double omega, const double* ibsum, int nout,
                               double* grad, hipStream_t s) {
  k_adj_grad_final<<<1, 256, 0, s>>>(part, nblk, omega, ibsum, nout, grad);
  return hipGetLastError();
}

hipError_t launch_spread_owner(const Grid& g, const BodyArgs& b, long long* fxc, uint8_t* tfc,
                               const DevFlags* flags, hipStream_t s) {
  if (b.nbody == 0 || !b.stage) return hipSuccess;
  const dim3 grid((BOX_CELLS + 255) / 256, (unsigned)b.n_marker_blocks);
  k_spread_owner<<<grid, 256, 0, s>>>(g, b, fxc, tfc, flags);
  return hipGetLastError();
}

hipError_t launch_bin_faces(const BodyArgs& b, hipStream_t s) {
  if (b.nbody == 0) return hipSuccess;
  k_bin_faces<<<(unsigned)b.nbody, BIN_THREADS, 0, s>>>(b);
  return hipGetLastError();
}

hipError_t launch_check(const BodyArgs& b, const double* X0, const double* X1, DevFlags* flags,
                        unsigned int* counter, hipStream_t s) {
  if (b.nbody == 0) return hipSuccess;
  k_check<<<(unsigned)b.n_diag_blocks, 256, 0, s>>>(b, X0, X1, flags, counter);
  return hipGetLastError();
}

// The inverse of the populations output: the current state (the buffer of
// the completed step count's parity) takes f - w_i at every non-solid node,
// rounded to the storage type; solid nodes keep zero.
template <class S>
__global__ void k_set_pops(Grid G, S* f0, S* f1, const uint8_t* ncls, const DevFlags* flags, const double* pops) {
  const long long N = (long long)G.nx * G.ny * G.nz;
  const long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (n >= N) return;
  S* f = (flags->steps_done & 1) ? f1 : f0;
  const int x = (int)(n % G.nx);
  const long long t = n / G.nx;
  const long long p = x + (long long)G.px * t;
  if (ncls[p] == CLS_SOLID) return;
  for (int i = 0; i < 19; i++) f[(long long)i * G.plane + p] = (S)(pops[(long long)i * N + n] - WD[i]);
}

hipError_t launch_set_populations(int prec, const Grid& g, void* f0, void* f1, const uint8_t* ncls,
                                  const DevFlags* flags, const double* pops, hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  switch (prec) {
    case 0: k_set_pops<double><<<cdiv(N, 256), 256, 0, s>>>(g, (double*)f0, (double*)f1, ncls, flags, pops); break;
    case 1: k_set_pops<float><<<cdiv(N, 256), 256, 0, s>>>(g, (float*)f0, (float*)f1, ncls, flags, pops); break;
    default:
      k_set_pops<_Float16><<<cdiv(N, 256), 256, 0, s>>>(g, (_Float16*)f0, (_Float16*)f1, ncls, flags, pops);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_get_fields(int prec, const Grid& g, const void* f0, const void* f1,
                             const uint8_t* ncls, const long long* fx0, const long long* fx1,
                             const uint8_t* tf0, const uint8_t* tf1, double gx, double gy,
                             double gz, const DevFlags* flags, double* rho, double* u,
                             double* pops, double* fib, hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  switch (prec) {
    case 0:
      k_get_fields<double><<<cdiv(N, 256), 256, 0, s>>>(g, (const double*)f0, (const double*)f1,
                                                        ncls, fx0, fx1, tf0, tf1, gx, gy, gz,
                                                        flags, rho, u, pops, fib);
      break;
    case 1:
      k_get_fields<float><<<cdiv(N, 256), 256, 0, s>>>(g, (const float*)f0, (const float*)f1, ncls,
                                                       fx0, fx1, tf0, tf1, gx, gy, gz, flags,
                                                       rho, u, pops, fib);
      break;
    default:
      k_get_fields<_Float16><<<cdiv(N, 256), 256, 0, s>>>(
          g, (const _Float16*)f0, (const _Float16*)f1, ncls, fx0, fx1, tf0, tf1, gx, gy, gz, flags,
          rho, u, pops, fib);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_interp(int prec, const Grid& g, const void* f0, const void* f1,
                         const uint8_t* ncls, const long long* fx0, const long long* fx1,
                         const uint8_t* tf0, const uint8_t* tf1, double gx, double gy, double gz,
                         const DevFlags* flags, long long n, const double* pts,
                         const double* field, double* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const unsigned grid = cdiv(n * 32, 256);
  switch (prec) {
    case 0:
      k_interp<double><<<grid, 256, 0, s>>>(g, (const double*)f0, (const double*)f1, ncls, fx0, fx1,
                                            tf0, tf1, gx, gy, gz, flags, n, pts, field, out);
      break;
    case 1:
      k_interp<float><<<grid, 256, 0, s>>>(g, (const float*)f0, (const float*)f1, ncls, fx0, fx1,
                                           tf0, tf1, gx, gy, gz, flags, n, pts, field, out);
      break;
    default:
      k_interp<_Float16><<<grid, 256, 0, s>>>(g, (const _Float16*)f0, (const _Float16*)f1, ncls, fx0,
                                              fx1, tf0, tf1, gx, gy, gz, flags, n, pts, field, out);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_spread_api(const Grid& g, const uint8_t* ncls, long long n, const double* pts,
                             const double* F, const double* c, long long* fx, DevFlags* flags,
                             hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_spread_api<<<cdiv(n * 32, 256), 256, 0, s>>>(g, ncls, n, pts, F, c, fx, flags);
  return hipGetLastError();
}

hipError_t launch_flush_fx(const Grid& g, long long* fx, double* fib, hipStream_t s) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  k_flush_fx<<<cdiv(N, 256), 256, 0, s>>>(g, fx, fib);
  return hipGetLastError();
}

// ------------------------------------------------- allocation-free spread
// Fixed-point force sums of the allocation-free spread, then its flags.  In
// host code the name stands for nothing on the device: the kernels get the
// address that hipGetSymbolAddress returned for the device in use.
static __device__ __align__(256) long long scratch[3 * NOALLOC_MAX_NODES + NOALLOC_FLAG_WORDS];

namespace {
std::mutex scratch_mu;
long long* scratch_dev[NOALLOC_MAX_DEVICES] = {};

__global__ void k_zero_words(long long* p, long long n) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}
}  // namespace

hipError_t noalloc_scratch(int device, long long** out) {
  if (device < 0 || device >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_dev[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) {
      const hipError_t e2 = hipSetDevice(cur);
      if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_dev[device] = (long long*)p;
  }
  *out = scratch_dev[device];
  return hipSuccess;
}

hipError_t launch_spread_noalloc(const Grid& g, const uint8_t* ncls, long long n, const double* pts,
                                 const double* F, const double* c, double* fib, long long* scr,
                                 hipStream_t s) {
  if (g.Np > NOALLOC_MAX_NODES) return hipErrorInvalidValue;
  long long* flag_words = scr + 3 * NOALLOC_MAX_NODES;
  // the last call's sums are normally flushed to zero already; clear anyway
  // (a fill kernel, not a memset, so that the sequence can be captured)
  k_zero_words<<<cdiv(3 * g.Np, 256), 256, 0, s>>>(scr, 3 * g.Np);
  k_zero_words<<<1, 64, 0, s>>>(flag_words, NOALLOC_FLAG_WORDS);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_spread_api(g, ncls, n, pts, F, c, scr, (DevFlags*)flag_words, s);
  if (e != hipSuccess) return e;
  return launch_flush_fx(g, scr, fib, s);
}

// ====================================================== coupled adjoint (IB)
// The immersed-boundary part of the discrete adjoint of a coupled step, for
// soft bodies.  The step maps (g, P, Q, V) -> (g', P', Q', V'), with P the
// vertex positions x^n, Q = x^{n-1} and V the vertex velocities; going
// back, the transposes of the Verlet update (Eqs. verletPos, verletVel,
// verletPosC), the membrane forces (Eqs. strainFor, bendFor, volFor), the
// probe tractions (Eqs. hydroForP, hydroForNu), the MLS vertex velocities
// and the direct forcing with its spreading (Eqs. uLag, l2norm, intKernel,
// bodyforce) are applied, each with the derivative of its weights with
// respect to the moving points.  All in FP64.

// Forward-mode dual numbers (value and N partial derivatives), for the bending
// force's derivative along a direction (adjb_element).
template <int N>
struct Dual {
  double v;
  double d[N];
};

#define DUAL_BIN(OP, VEXPR, DEXPR)                                                           \
  template <int N>                                                                           \
  __device__ __forceinline__ Dual<N> operator OP(const Dual<N>& a, const Dual<N>& b) {       \
    Dual<N> r;                                                                               \
    r.v = VEXPR;                                                                             \
    _Pragma("unroll") for (int i = 0; i < N; i++) r.d[i] = DEXPR;                           \
    return r;                                                                                \
  }
DUAL_BIN(+, a.v + b.v, a.d[i] + b.d[i])
DUAL_BIN(-, a.v - b.v, a.d[i] - b.d[i])
DUAL_BIN(*, a.v * b.v, a.d[i] * b.v + a.v * b.d[i])
DUAL_BIN(/, a.v / b.v, (a.d[i] * b.v - a.v * b.d[i]) / (b.v * b.v))
#undef DUAL_BIN
template <int N>
__device__ __forceinline__ Dual<N> operator-(const Dual<N>& a, double b) {
  Dual<N> r = a;
  r.v -= b;
  return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator-(const Dual<N>& a) {
  Dual<N> r;
  r.v = -a.v;
#pragma unroll
  for (int i = 0; i < N; i++) r.d[i] = -a.d[i];
  return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator-(double b, const Dual<N>& a) {
  Dual<N> r = -a;
  r.v += b;
  return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator*(const Dual<N>& a, double b) {
  Dual<N> r;
  r.v = a.v * b;
#pragma unroll
  for (int i = 0; i < N; i++) r.d[i] = a.d[i] * b;
  return r;
}
// chain rule of a scalar function: value f, derivative df at a.v
template <int N>
__device__ __forceinline__ Dual<N> dchain(const Dual<N>& a, double f, double df) {
  Dual<N> r;
  r.v = f;
#pragma unroll
  for (int i = 0; i < N; i++) r.d[i] = df * a.d[i];
  return r;
}
template <int N>
__device__ __forceinline__ Dual<N> dsqrt(const Dual<N>& a) {
  const double r = sqrt(a.v);
  return dchain(a, r, 0.5 / r);
}
template <int N>
__device__ __forceinline__ Dual<N> dsin(const Dual<N>& a) {
  return dchain(a, sin(a.v), cos(a.v));
}
template <int N>
__device__ __forceinline__ Dual<N> datan2(const Dual<N>& y, const Dual<N>& x) {
  Dual<N> r;
  r.v = atan2(y.v, x.v);
  const double q = 1.0 / (x.v * x.v + y.v * y.v);
#pragma unroll
  for (int i = 0; i < N; i++) r.d[i] = (x.v * y.d[i] - y.v * x.d[i]) * q;
  return r;
}

template <class T>
__device__ __forceinline__ void cross_t(const T (&a)[3], const T (&b)[3], T (&c)[3]) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}
template <class T>
__device__ __forceinline__ T dot_t(const T (&a)[3], const T (&b)[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// The fits' derivatives with respect to their point p, in closed form.  With
// d = x_k - p, P = (1, d), W = exp(-K |d|^2), A = sum W P P^T, b = sum W P f
// and c = A^-1 b: dW/dp_m = 2 K d_m W and dP/dp_m = -(0, e_m) give
//   dc/dp_m = c_m e_0 + 2 K A^-1 sum_k W d_m P (f_k - P.c)
// (the terms in sum W P (f - P.c) vanish: the normal equations).  A functional
// s.c of the coefficients, z = A^-1 s, has then the derivative
//   c_m s_0 + 2 K sum_k W d_m (z.P) (f_k - P.c)
// and depends on the node values through W (z.P): one more pass over the
// supports with a few products each, where dual numbers carried three
// derivatives through the moment matrix, its factor and 27 solves.
//
// A quad of lanes per point, its lane's seven supports as in the step's fits
// (rows sub, sub + 4 and a third of row 8).
struct QuadSupports {
  int node[7];  // padded index, -1 where there is no usable support
  int cell[7];  // x + 3 (y + 3 z) offsets as kx | ky << 2 | kz << 4
  double W[7], dx[7], dy[3], dz[3];
};
__device__ __forceinline__ void quad_supports(const FluidArgs& a, int sub, const double (&p)[3], const int (&bs)[3],
                                              QuadSupports& q) {
  const Grid& G = a.g;
  int ox[3], oy[3], oz[3];
  bool ix[3], iy[3], iz[3];
  axis_nodes(bs[0], G.nx, G.per[0], 1, ox, ix);
  axis_nodes(bs[1], G.ny, G.per[1], G.px, oy, iy);
  axis_nodes(bs[2], G.nz, G.per[2], G.px * G.ny, oz, iz);
  uint8_t cls[7];
  double wr[3];
  double wx[3], wy[3], wz[3], dx[3];
  quad_weights(sub, p, bs, wx, wy, wz);
#pragma unroll
  for (int k = 0; k < 3; k++) dx[k] = (double)(bs[0] + k - 1) - p[0];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    int ky = 2, kz = 2;
    if (i < 2) row_yz(sub + 4 * i, ky, kz);
    const int row = sel3i(ky, oy) + sel3i(kz, oz);
    const bool rin = sel3b(ky, iy) && sel3b(kz, iz);
    q.dy[i] = (double)(bs[1] + ky - 1) - p[1];
    q.dz[i] = (double)(bs[2] + kz - 1) - p[2];
    wr[i] = sel3(ky, wy) * sel3(kz, wz);
#pragma unroll
    for (int k = 0; k < (i < 2 ? 3 : 1); k++) {
      const int n = (i < 2 ? ox[k] : sel3i(sub, ox)) + row;
      const bool in = rin && (i < 2 ? ix[k] : sub < 3 && sel3b(sub, ix));
      cls[3 * i + k] = a.ncls[n];
      q.node[3 * i + k] = in ? n : -1;
      q.cell[3 * i + k] = (i < 2 ? k : min(sub, 2)) | ky << 2 | kz << 4;
      q.dx[3 * i + k] = i < 2 ? dx[k] : sel3(sub, dx);
      q.W[3 * i + k] = (i < 2 ? wx[k] : sel3(sub, wx)) * wr[i];
    }
  }
#pragma unroll
  for (int k = 0; k < 7; k++)
    if (q.node[k] < 0 || cls[k] == CLS_SOLID) {
      q.node[k] = -1;
      q.W[k] = 0.0;
    }
}

// Moments of the supports with the fields f[7][NF].
template <int NF>
__device__ __forceinline__ void quad_moments(const QuadSupports& q, const double (&f)[7][NF], FitSums<NF>& fs) {
  fs.clear();
#pragma unroll
  for (int i = 0; i < 3; i++) {
    RowSums<NF> rs;
    rs.clear();
#pragma unroll
    for (int k = 0; k < (i < 2 ? 3 : 1); k++) rs.add(q.W[3 * i + k], q.dx[3 * i + k], f[3 * i + k]);
    fs.add(rs, 1.0, q.dy[i], q.dz[i]);
  }
  fs.quad();
}

__device__ __forceinline__ double lin4(const double (&c)[4], double dx, double dy, double dz) {
  return c[0] + c[1] * dx + c[2] * dy + c[3] * dz;
}

// Box of stencil bases of a block's points (bs of the quads with on set), its
// cells with the supports around them; false when they exceed BOX_CELLS or no
// quad is on.  s_wbox: [4][6] ints.  Every thread calls (two barriers).
struct Box {
  int x0, y0, z0, ex, ey, ez;
  __device__ __forceinline__ int cells() const { return ex * ey * ez; }
  __device__ __forceinline__ int corner(const int (&bs)[3]) const {
    return (bs[0] - 1 - x0) + ex * ((bs[1] - 1 - y0) + ey * (bs[2] - 1 - z0));
  }
  __device__ __forceinline__ int at(int c00, int cell) const {
    return c00 + (cell & 3) + ex * (((cell >> 2) & 3) + ey * (cell >> 4));
  }
};
__device__ __forceinline__ bool block_box(const int (&bs)[3], bool on, int (*s_wbox)[6], Box& bx) {
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int lo = wave_ext<false>(on ? bs[k] : INT_MAX), hi = wave_ext<true>(on ? bs[k] : INT_MIN);
    if ((threadIdx.x & 63) == 0) {
      s_wbox[threadIdx.x >> 6][k] = lo;
      s_wbox[threadIdx.x >> 6][3 + k] = hi;
    }
  }
  __syncthreads();
  int lo[3], hi[3];
#pragma unroll
  for (int k = 0; k < 3; k++) {
    lo[k] = min(min(s_wbox[0][k], s_wbox[1][k]), min(s_wbox[2][k], s_wbox[3][k]));
    hi[k] = max(max(s_wbox[0][3 + k], s_wbox[1][3 + k]), max(s_wbox[2][3 + k], s_wbox[3][3 + k]));
  }
  if (hi[0] < lo[0]) {
    bx = Box{0, 0, 0, 0, 0, 0};
    return false;
  }
  int e[3];
  const bool fits = box_fits(lo, hi, e);
  bx = Box{lo[0] - 1, lo[1] - 1, lo[2] - 1, e[0], e[1], e[2]};
  return fits;
}

// The cell c of a box: node coordinates in the periodic box; false outside.
__device__ __forceinline__ bool box_node(const Grid& G, const Box& bx, int c, int (&p)[3], int& node) {
  const int q = (int)(((float)c + 0.5f) / (float)bx.ex), cz = (int)(((float)q + 0.5f) / (float)bx.ey);
  p[0] = bx.x0 + c - q * bx.ex;
  p[1] = bx.y0 + q - cz * bx.ey;
  p[2] = bx.z0 + cz;
  const int dim[3] = {G.nx, G.ny, G.nz};
#pragma unroll
  for (int k = 0; k < 3; k++)
    if (p[k] < 0 || p[k] >= dim[k]) {
      if (!G.per[k]) return false;
      p[k] = ((p[k] % dim[k]) + dim[k]) % dim[k];
    }
  node = p[0] + G.px * (p[1] + G.ny * p[2]);
  return true;
}

// The bending force of a hinge (a, b, c, d) in any scalar type: the signed
// dihedral angle and F_r = -k_b sin(theta - theta0) dtheta/dx_r, with the
// closed-form angle gradient of the step.
template <class T>
__device__ void hinge_force_t(const T (&X)[4][3], double kb, double th0, T (&F)[4][3]) {
  T e[3], ca[3], da[3], ab[3], db[3], n1[3], n2[3];
  for (int k = 0; k < 3; k++) {
    e[k] = X[1][k] - X[0][k];
    ca[k] = X[2][k] - X[0][k];
    da[k] = X[3][k] - X[0][k];
    ab[k] = X[0][k] - X[1][k];
    db[k] = X[3][k] - X[1][k];
  }
  cross_t(e, ca, n1);
  cross_t(ab, db, n2);
  const T q1 = dot_t(n1, n1), q2 = dot_t(n2, n2), le2 = dot_t(e, e);
  const T le = dsqrt(le2), l1 = dsqrt(q1), l2 = dsqrt(q2);
  T m1[3], m2[3], t[3];
  for (int k = 0; k < 3; k++) {
    m1[k] = n1[k] / l1;
    m2[k] = n2[k] / l2;
  }
  cross_t(m1, m2, t);
  const T theta = datan2(dot_t(t, e) / le, dot_t(m1, m2));
  const T al_c = dot_t(ca, e) / le2, al_d = dot_t(da, e) / le2;
  const T amp = dsin(theta - th0) * (-kb);
  for (int k = 0; k < 3; k++) {
    const T gc = -(le * n1[k]) / q1;
    const T gd = -(le * n2[k]) / q2;
    F[0][k] = amp * (-((1.0 - al_c) * gc + (1.0 - al_d) * gd));
    F[1][k] = amp * (-(al_c * gc + al_d * gd));
    F[2][k] = amp * gc;
    F[3][k] = amp * gd;
  }
}

__device__ __forceinline__ void set_tile(uint8_t* tf, long long node) {
  if (!tf[node >> TILE_SHIFT]) tf[node >> TILE_SHIFT] = 1;
}

// The vertex update transposed.  With P' = P/2 + 3/2 u0 + 5/2 acc + Q/2,
// V' = -P/2 + 3/2 u0 + 3/2 acc + Q/2, Q' = P and acc = F / (2 m_v):
// dJ/du0 = 3/2 (aP + aV), dJ/dF = (5/2 aP + 3/2 aV) / (2 m_v),
// dJ/dQ = (aP + aV)/2, dJ/dP = aP/2 - aV/2 + aQ (more added by the later
// launches), dJ/dV = 0 (the forcing markers add theirs).
__global__ __launch_bounds__(256) void k_adjb_vertex(BodyArgs b, AdjIB ib) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx < b.nbody) ib.gsum[2 + idx] = 0.0;  // sum of A n . dJ/dFt per body (k_adjb_body adds it)
  if (idx >= b.nsoft_v) return;
  const int v = b.soft_vlist[idx];
  const double mv = b.b_param[8 * b.vert_body[v] + 3];
  for (int q = 0; q < 3; q++) {
    const int i = 3 * v + q;
    const double aX = ib.aP[i], aV = ib.aV[i], aQ = ib.aQ[i];
    ib.ub0[i] = 1.5 * (aX + aV);
    ib.Fb[i] = (2.5 * aX + 1.5 * aV) * 0.5 / mv;
    ib.Qn[i] = 0.5 * aX + 0.5 * aV;
    ib.LP[i] = 0.5 * aX - 0.5 * aV + aQ;
    ib.Vn[i] = 0.0;
  }
}

// Edges and hinges transposed, one thread each (whole waves of them): dJ/dkappa
// is summed over the wave first, one atomic per wave.
__device__ __forceinline__ void adjb_element(const BodyArgs& b, const AdjIB& ib, long long gt) {
  const double* X = b.Xcur;
  const int it = gt < b.ne + b.nh ? (int)gt : -1;
  double fy = 0.0;
  if (it >= 0 && it < b.ne) {
    // stretching (Eq. strainFor): F_a = -k (l - l0) r / l, r = x_a - x_b; its
    // Jacobian K = -k [(1 - l0/l) 1 + l0 r r^T / l^3] is symmetric, and
    // dF_b = -dF_a
    const int e = it, va = b.edges[2 * e], vb = b.edges[2 * e + 1];
    double r[3], y[3];
    for (int k = 0; k < 3; k++) {
      r[k] = X[3 * va + k] - X[3 * vb + k];
      y[k] = ib.Fb[3 * va + k] - ib.Fb[3 * vb + k];
    }
    const double l = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    const double kl = b.kl[e], l0 = b.l0[e];
    const double ry = r[0] * y[0] + r[1] * y[1] + r[2] * y[2];
    for (int k = 0; k < 3; k++) {
      const double g = -kl * ((1.0 - l0 / l) * y[k] + l0 * ry * r[k] / (l * l * l));
      atomicAdd(ib.LP + 3 * va + k, g);
      atomicAdd(ib.LP + 3 * vb + k, -g);
      fy += -kl * (l - l0) * r[k] / l * y[k];  // the force is linear in the modulus
    }
  } else if (it >= 0) {
    // bending: the force is minus the gradient of the hinge energy, so its
    // Jacobian is symmetric and the transposed product is the derivative
    // along the adjoint itself (one dual direction)
    const int h = it - b.ne;
    const int32_t* H = b.hinges + 4 * h;
    Dual<1> P[4][3], F[4][3];
    for (int r = 0; r < 4; r++)
      for (int k = 0; k < 3; k++) {
        P[r][k].v = X[3 * H[r] + k];
        P[r][k].d[0] = ib.Fb[3 * H[r] + k];
      }
    hinge_force_t(P, b.kb[h], b.theta0[h], F);
    for (int r = 0; r < 4; r++)
      for (int k = 0; k < 3; k++) {
        atomicAdd(ib.LP + 3 * H[r] + k, F[r][k].d[0]);
        fy += F[r][k].v * ib.Fb[3 * H[r] + k];
      }
  }
  fy = red64(fy);
  if ((threadIdx.x & 63) == 0 && fy != 0.0) atomicAdd(ib.gsum + 1, fy / ib.kappa);
}

// Field values of a quad's supports from the macro field: u and rho - 1.
template <class S>
__device__ __forceinline__ void mac_fields(const FluidArgs& a, const QuadSupports& q, double (&f)[7][4]) {
#pragma unroll
  for (int k = 0; k < 7; k++) {
    double v[4];
    load_mac<S>(a, q.node[k] < 0 ? 0 : q.node[k], v[3], v[0], v[1], v[2]);
#pragma unroll
    for (int c = 0; c < 4; c++) f[k][c] = q.node[k] < 0 ? 0.0 : v[c];
  }
}

// The tractions of a marker chunk's faces transposed (a block per chunk, a
// quad per face, its outer probe and then its inner one):
//   s = sum over the sides of sg A r Q + k_v (1 - V/V0) A ab.n,
//   Q = -ab.n / 3 + nu S:G,  S = ab n^T + n ab^T,
// with ab the mean of the vertices' dJ/dF, r and G the fitted density and
// velocity gradient at the probe c +- 1.2 n.  The sources at the nodes are
// summed in LDS over the chunk's box of supports and added to ext once per node
// and component; the derivatives in n, A and c go to the vertices at the end.
template <class S>
__device__ void adjb_probes(const FluidArgs& a, const BodyArgs& b, const AdjIB& ib, int blk) {
  __shared__ double s_ext[4][BOX_CELLS];
  __shared__ int s_wbox[4][6];
  __shared__ double s_sum[4][3];
  const Grid& G = a.g;
  const int t = threadIdx.x, sub = t & 3;
  const int nchunk = b.chunk_n[blk], s0 = b.chunk_s0[blk];
  if (nchunk == 0) return;
  const bool mk = (t >> 2) < nchunk;
  const int4 sf = *(const int4*)(b.slot_f + 4 * (long long)(s0 + (mk ? t >> 2 : 0)));
  const int vv[3] = {sf.x, sf.y, sf.z}, body = sf.w;
  double X[3][3], ab[3];
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int k = 0; k < 3; k++) X[r][k] = b.Xcur[3 * vv[r] + k];
#pragma unroll
  for (int k = 0; k < 3; k++)
    ab[k] = (ib.Fb[3 * vv[0] + k] + ib.Fb[3 * vv[1] + k] + ib.Fb[3 * vv[2] + k]) * (1.0 / 3.0);
  const double nu = b.nu, V0 = b.b_param[8 * body], kv = b.b_param[8 * body + 2];
  const double cv = kv * (1.0 - b.b_diag[16 * body] / V0);
  const bool kvd = b.b_param[8 * body + 6] != 0.0;
  double cen[3], n[3], A;
  face_geom_pts(X[0], X[1], X[2], cen, n, A);
  const double an = ab[0] * n[0] + ab[1] * n[1] + ab[2] * n[2];
  // derivatives of s in the area, the normal and the centroid
  double gA = cv * an, gn[3] = {cv * A * ab[0], cv * A * ab[1], cv * A * ab[2]}, gc[3] = {0.0, 0.0, 0.0};
  double visc = 0.0;
#pragma unroll 1
  for (int side = 0; side < 2; side++) {
    const double off = side == 0 ? 1.2 : -1.2, sg = side == 0 ? 1.0 : -1.0;
    const double p[3] = {cen[0] + off * n[0], cen[1] + off * n[1], cen[2] + off * n[2]};
    const int bs[3] = {(int)floor(p[0] + 0.5), (int)floor(p[1] + 0.5), (int)floor(p[2] + 0.5)};
    Box bx;
    const bool fits = block_box(bs, mk, s_wbox, bx);
    const int ncell = fits ? bx.cells() : 0;
    for (int c = t; c < ncell; c += blockDim.x)
#pragma unroll
      for (int k = 0; k < 4; k++) s_ext[k][c] = 0.0;
    QuadSupports q;
    quad_supports(a, sub, p, bs, q);
    double f[7][4];
    mac_fields<S>(a, q, f);
    FitSums<4> fs;
    quad_moments(q, f, fs);
    Chol4 ch;
    const bool ok = mk && chol4(fs.A, ch);  // a singular fit gives 0
    __syncthreads();
    if (ok) {
      double cc[4], c[4][4], z[3][4], Q = 0.0, qc[3] = {0.0, 0.0, 0.0};
      const double e0[4] = {1.0, 0.0, 0.0, 0.0};
      chol_solve(ch, e0, cc);
#pragma unroll
      for (int i = 0; i < 4; i++) chol_solve(ch, fs.b[i], c[i]);
#pragma unroll
      for (int i = 0; i < 3; i++) {
        const double si[4] = {0.0, ab[i] * n[0] + ab[0] * n[i], ab[i] * n[1] + ab[1] * n[i],
                              ab[i] * n[2] + ab[2] * n[i]};
        chol_solve(ch, si, z[i]);
#pragma unroll
        for (int k = 0; k < 3; k++) {
          Q += si[1 + k] * c[i][1 + k];
          qc[k] += ab[i] * (c[i][1 + k] + c[k][1 + i]);
        }
      }
      const double r = 1.0 + c[3][0], sv = Q;  // the weights add up to 1: rho = 1 + the fit of rho - 1
      const double Qt = -an * (1.0 / 3.0) + nu * sv;
      // sources: dJ/drho_k = A sg Qt phi_k, dJ/du_ik = A sg nu r W z_i.P
      const double rb = A * sg * Qt, ub = A * sg * nu * r;
      double H[3] = {0.0, 0.0, 0.0}, R[3] = {0.0, 0.0, 0.0};
      const int c00 = fits ? bx.corner(bs) : 0;
#pragma unroll
      for (int k = 0; k < 7; k++) {
        if (q.node[k] < 0) continue;
        const double dx = q.dx[k], dy = q.dy[k / 3], dz = q.dz[k / 3];
        const double phi = q.W[k] * lin4(cc, dx, dy, dz);
        double wz[3], h = 0.0;
#pragma unroll
        for (int i = 0; i < 3; i++) {
          wz[i] = q.W[k] * lin4(z[i], dx, dy, dz);
          h += wz[i] * (f[k][i] - lin4(c[i], dx, dy, dz));
        }
        const double rr = phi * (f[k][3] - lin4(c[3], dx, dy, dz));
        H[0] += h * dx;
        H[1] += h * dy;
        H[2] += h * dz;
        R[0] += rr * dx;
        R[1] += rr * dy;
        R[2] += rr * dz;
        const double e[4] = {rb * phi, ub * wz[0], ub * wz[1], ub * wz[2]};
        if (fits) {
          const int cl = bx.at(c00, q.cell[k]);
#pragma unroll
          for (int i = 0; i < 4; i++) atomicAdd(&s_ext[i][cl], e[i]);
        } else {
#pragma unroll
          for (int i = 0; i < 4; i++) atomicAdd(ib.ext + (long long)i * G.Np + q.node[k], e[i]);
          set_tile(ib.etf, q.node[k]);
        }
      }
      gA += sg * r * Qt;
      visc += A * sg * r * sv;
#pragma unroll
      for (int m = 0; m < 3; m++) {
        const double dr = c[3][1 + m] + 2.0 * MLS_K * quad_sum(R[m]), dq = 2.0 * MLS_K * quad_sum(H[m]);
        const double gp = A * sg * (dr * Qt + r * nu * dq);
        gc[m] += gp;
        gn[m] += off * gp + A * sg * r * (nu * qc[m] - ab[m] * (1.0 / 3.0));
      }
    }
    __syncthreads();
    for (int c = t; c < ncell; c += blockDim.x) {
      double v[4];
#pragma unroll
      for (int k = 0; k < 4; k++) v[k] = s_ext[k][c];
      if (v[0] == 0.0 && v[1] == 0.0 && v[2] == 0.0 && v[3] == 0.0) continue;
      int x[3], node;
      if (!box_node(G, bx, c, x, node)) continue;
#pragma unroll
      for (int k = 0; k < 4; k++) atomicAdd(ib.ext + (long long)k * G.Np + node, v[k]);
      set_tile(ib.etf, node);
    }
  }
  // the scalar gradients: one atomic per block
  const bool lead = mk && sub == 0;
  const double sums[3] = {red64(lead ? visc * (1.0 / 3.0) : 0.0),  // nu = (tau - 1/2) / 3
                          red64(lead && kvd ? cv * A * an : 0.0), red64(lead ? A * an : 0.0)};
  if ((t & 63) == 0)
    for (int k = 0; k < 3; k++) s_sum[t >> 6][k] = sums[k];
  __syncthreads();
  if (t == 0) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int w = 0; w < 4; w++)
      for (int k = 0; k < 3; k++) v[k] += s_sum[w][k];
    atomicAdd(ib.gsum, v[0]);
    if (v[1] != 0.0) atomicAdd(ib.gsum + 1, v[1] / ib.kappa);
    atomicAdd(ib.gsum + 2 + body, v[2]);  // a chunk's faces belong to one body
  }
  if (!lead) return;
  // to the vertices: N = u x w, n = N / |N|, A = |N| / 2, c the mean
  const double u[3] = {X[1][0] - X[0][0], X[1][1] - X[0][1], X[1][2] - X[0][2]};
  const double w[3] = {X[2][0] - X[0][0], X[2][1] - X[0][1], X[2][2] - X[0][2]};
  const double ng = n[0] * gn[0] + n[1] * gn[1] + n[2] * gn[2], il = 0.5 / A;
  double gN[3], gu[3], gw[3];
#pragma unroll
  for (int k = 0; k < 3; k++) gN[k] = (gn[k] - n[k] * ng) * il + 0.5 * gA * n[k];
  cross3(w, gN, gu);
  cross3(gN, u, gw);
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const double m = gc[k] * (1.0 / 3.0);
    atomicAdd(ib.LP + 3 * vv[0] + k, m - gu[k] - gw[k]);
    atomicAdd(ib.LP + 3 * vv[1] + k, m + gu[k]);
    atomicAdd(ib.LP + 3 * vv[2] + k, m + gw[k]);
  }
}

// The MLS velocity at a soft vertex transposed (a quad each): u0 = sum phi_k u_k.
template <class S>
__device__ __forceinline__ void adjb_vertex_velocity(const FluidArgs& a, const BodyArgs& b, const AdjIB& ib, int idx) {
  if (idx >= b.nsoft_v) return;  // whole quads
  const int v = b.soft_vlist[idx], sub = threadIdx.x & 3;
  const double p[3] = {b.Xcur[3 * v], b.Xcur[3 * v + 1], b.Xcur[3 * v + 2]};
  const double ub[3] = {ib.ub0[3 * v], ib.ub0[3 * v + 1], ib.ub0[3 * v + 2]};
  const int bs[3] = {(int)floor(p[0] + 0.5), (int)floor(p[1] + 0.5), (int)floor(p[2] + 0.5)};
  QuadSupports q;
  quad_supports(a, sub, p, bs, q);
  double f[7][4], h[7][1];
  mac_fields<S>(a, q, f);
#pragma unroll
  for (int k = 0; k < 7; k++) h[k][0] = ub[0] * f[k][0] + ub[1] * f[k][1] + ub[2] * f[k][2];
  FitSums<1> fs;
  quad_moments(q, h, fs);
  Chol4 ch;
  if (!chol4(fs.A, ch)) return;
  double cc[4], c[4], H[3] = {0.0, 0.0, 0.0};
  const double e0[4] = {1.0, 0.0, 0.0, 0.0};
  chol_solve(ch, e0, cc);
  chol_solve(ch, fs.b[0], c);
#pragma unroll
  for (int k = 0; k < 7; k++) {
    if (q.node[k] < 0) continue;
    const double dx = q.dx[k], dy = q.dy[k / 3], dz = q.dz[k / 3];
    const double phi = q.W[k] * lin4(cc, dx, dy, dz), r = phi * (h[k][0] - lin4(c, dx, dy, dz));
    H[0] += r * dx;
    H[1] += r * dy;
    H[2] += r * dz;
#pragma unroll
    for (int i = 0; i < 3; i++) atomicAdd(ib.ext + (long long)(1 + i) * a.g.Np + q.node[k], phi * ub[i]);
    set_tile(ib.etf, q.node[k]);
  }
#pragma unroll
  for (int m = 0; m < 3; m++) H[m] = c[1 + m] + 2.0 * MLS_K * quad_sum(H[m]);
  if (sub < 3) atomicAdd(ib.LP + 3 * v + sub, sel3(sub, H));
}

// Elements, probes and vertex velocities transposed, in blocks: the marker
// chunks (probes of their faces), 256 edges and hinges each, 64 soft vertices
// each.  Measured per launch on the 2562-vertex capsule: 105 us with dual
// numbers through every fit and 1.3 million atomics on the node sources,
// 28 us.
template <class S>
__global__ __launch_bounds__(256, 1) void k_adjb_body(FluidArgs a, BodyArgs b, AdjIB ib) {
  const int nmk = b.n_marker_blocks, nel = b.n_elem_blocks, u = blockIdx.x;
  if (u < nmk) adjb_probes<S>(a, b, ib, u);
  else if (u < nmk + nel) adjb_element(b, ib, (long long)(u - nmk) * 256 + threadIdx.x);
  else adjb_vertex_velocity<S>(a, b, ib, (u - nmk - nel) * 64 + (threadIdx.x >> 2));
}

// The volume force through V: Ft_f contains k_v (1 - V/V0) A_f n_f, and
// dV/dx_v is a third of the sum of A n over the faces at v.
__global__ __launch_bounds__(256) void k_adjb_volume(BodyArgs b, AdjIB ib) {
  const int f = blockIdx.x * 256 + threadIdx.x;
  if (f >= b.nf) return;
  const int body = b.face_body[f];
  const double V0 = b.b_param[8 * body], kv = b.b_param[8 * body + 2];
  const double c = -kv / V0 * ib.gsum[2 + body] / 3.0;
  double cen[3], n[3], area;
  face_geom(b.Xcur, b.faces, f, cen, n, area);
  for (int r = 0; r < 3; r++)
    for (int k = 0; k < 3; k++) atomicAdd(ib.LP + 3 * b.faces[3 * f + r] + k, c * area * n[k]);
}

// The forcing markers transposed (a block per marker chunk, a quad per face):
// U = sum phi u*, F_l = U_b - U, f_ib += A phi F_l.  With Fs = sum phi dJ/dF_k:
// dJ/dF_l = A Fs, of which a third goes to each vertex velocity; dJ/du*_k =
// -phi_k A Fs; and the positions through the area (F_l.Fs) and the centroid
// (the derivative of sum phi h, h = A F_l.dJ/dF_k - u*_k.A Fs).  As in the
// forcing itself u* is formed once per node of the chunk's box in LDS (twice
// per support and face before), and the node sources are summed there.
// Measured per launch on the 2562-vertex capsule: 50 -> 17 us.
template <class S>
__global__ __launch_bounds__(256, 1) void k_adjb_markers(FluidArgs a, BodyArgs b, AdjIB ib) {
  __shared__ double s_v[6][BOX_CELLS];  // u*, dJ/dF; then the sums of dJ/du* in the first three
  __shared__ int s_wbox[4][6];
  const Grid& G = a.g;
  const int t = threadIdx.x, sub = t & 3, blk = blockIdx.x;
  const int nchunk = b.chunk_n[blk], s0 = b.chunk_s0[blk];
  if (nchunk == 0) return;
  const bool mk = (t >> 2) < nchunk;
  const int4 sf = *(const int4*)(b.slot_f + 4 * (long long)(s0 + (mk ? t >> 2 : 0)));
  const int vv[3] = {sf.x, sf.y, sf.z};
  double X[3][3], Ub[3];
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int k = 0; k < 3; k++) X[r][k] = b.Xcur[3 * vv[r] + k];
#pragma unroll
  for (int k = 0; k < 3; k++)
    Ub[k] = (b.Vel[3 * vv[0] + k] + b.Vel[3 * vv[1] + k] + b.Vel[3 * vv[2] + k]) * (1.0 / 3.0);
  double cen[3], n[3], area;
  face_geom_pts(X[0], X[1], X[2], cen, n, area);
  const int bs[3] = {(int)floor(cen[0] + 0.5), (int)floor(cen[1] + 0.5), (int)floor(cen[2] + 0.5)};
  Box bx;
  const bool fits = block_box(bs, mk, s_wbox, bx);
  const int ncell = fits ? bx.cells() : 0;
  auto fields = [&](int x, int y, int z, int node, double (&v)[6]) {
    double us[3] = {0.0, 0.0, 0.0};
    const bool ok = cell_velocity<S>(a, node, x, y, z, us);
#pragma unroll
    for (int k = 0; k < 3; k++) {
      v[k] = ok ? us[k] : 0.0;
      v[3 + k] = ok ? ib.fbar[(long long)k * G.Np + node] : 0.0;
    }
  };
  for (int c = t; c < ncell; c += blockDim.x) {
    int x[3], node;
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (box_node(G, bx, c, x, node)) fields(x[0], x[1], x[2], node, v);
#pragma unroll
    for (int k = 0; k < 6; k++) s_v[k][c] = v[k];
  }
  QuadSupports q;
  quad_supports(a, sub, cen, bs, q);
  __syncthreads();
  double f[7][6];
  const int c00 = fits ? bx.corner(bs) : 0;
#pragma unroll
  for (int k = 0; k < 7; k++) {
    const int cl = fits && mk ? bx.at(c00, q.cell[k]) : 0;
#pragma unroll
    for (int i = 0; i < 6; i++) f[k][i] = fits && q.node[k] >= 0 ? s_v[i][cl] : 0.0;
  }
  if (!fits && mk) {  // a box beyond the LDS capacity: support by support
#pragma unroll 1
    for (int k = 0; k < 7; k++) {
      int node = -1;
      double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 7; i++) node = i == k ? q.node[i] : node;
      if (node >= 0) {
        int x, y, z;
        coords(G, node, x, y, z);
        fields(x, y, z, node, v);
      }
#pragma unroll
      for (int i = 0; i < 7; i++)
        if (i == k)
#pragma unroll
          for (int m = 0; m < 6; m++) f[i][m] = v[m];
    }
  }
  FitSums<6> fs;
  quad_moments(q, f, fs);
  __syncthreads();
  for (int c = t; c < ncell; c += blockDim.x)
#pragma unroll
    for (int k = 0; k < 3; k++) s_v[k][c] = 0.0;
  Chol4 ch;
  const bool ok = mk && chol4(fs.A, ch);  // a singular fit has U = 0 and spreads nothing
  __syncthreads();
  if (ok) {
    double cc[4], Fl[3], Fbl[3], bh[4] = {0.0, 0.0, 0.0, 0.0}, c[4], H[3] = {0.0, 0.0, 0.0}, Ab = 0.0;
    const double e0[4] = {1.0, 0.0, 0.0, 0.0};
    chol_solve(ch, e0, cc);
#pragma unroll
    for (int k = 0; k < 3; k++) {
      double U = 0.0, Fs = 0.0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        U += cc[i] * fs.b[k][i];
        Fs += cc[i] * fs.b[3 + k][i];
      }
      Fl[k] = Ub[k] - U;
      Fbl[k] = area * Fs;
      Ab += Fl[k] * Fs;
#pragma unroll
      for (int i = 0; i < 4; i++) bh[i] += area * Fl[k] * fs.b[3 + k][i] - Fbl[k] * fs.b[k][i];
    }
    chol_solve(ch, bh, c);
#pragma unroll
    for (int k = 0; k < 7; k++) {
      if (q.node[k] < 0) continue;
      const double dx = q.dx[k], dy = q.dy[k / 3], dz = q.dz[k / 3];
      double h = 0.0;
#pragma unroll
      for (int i = 0; i < 3; i++) h += area * Fl[i] * f[k][3 + i] - Fbl[i] * f[k][i];
      const double phi = q.W[k] * lin4(cc, dx, dy, dz), r = phi * (h - lin4(c, dx, dy, dz));
      H[0] += r * dx;
      H[1] += r * dy;
      H[2] += r * dz;
      if (fits) {
        const int cl = bx.at(c00, q.cell[k]);
#pragma unroll
        for (int i = 0; i < 3; i++) atomicAdd(&s_v[i][cl], -phi * Fbl[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 3; i++) atomicAdd(ib.ext + (long long)(4 + i) * G.Np + q.node[k], -phi * Fbl[i]);
        set_tile(ib.etf, q.node[k]);
      }
    }
#pragma unroll
    for (int m = 0; m < 3; m++) H[m] = c[1 + m] + 2.0 * MLS_K * quad_sum(H[m]);
    if (sub < 3) {
      // lane r takes vertex r; d area / d vertex: (1/2) n x (opposite edge), counter-clockwise
      const int r = sub, r1 = r == 2 ? 0 : r + 1, r2 = r == 0 ? 2 : r - 1;
      double e[3], dA[3];
#pragma unroll
      for (int k = 0; k < 3; k++) {
        const double xk[3] = {X[0][k], X[1][k], X[2][k]};
        e[k] = sel3(r2, xk) - sel3(r1, xk);
      }
      cross3(n, e, dA);
      const int v = sel3i(r, vv);
#pragma unroll
      for (int k = 0; k < 3; k++) {
        atomicAdd(ib.LP + 3 * v + k, H[k] * (1.0 / 3.0) + Ab * 0.5 * dA[k]);
        atomicAdd(ib.Vn + 3 * v + k, Fbl[k] * (1.0 / 3.0));
      }
    }
  }
  __syncthreads();
  for (int c = t; c < ncell; c += blockDim.x) {
    const double v[3] = {s_v[0][c], s_v[1][c], s_v[2][c]};
    if (v[0] == 0.0 && v[1] == 0.0 && v[2] == 0.0) continue;
    int x[3], node;
    if (!box_node(G, bx, c, x, node)) continue;
#pragma unroll
    for (int k = 0; k < 3; k++) atomicAdd(ib.ext + (long long)(4 + k) * G.Np + node, v[k]);
    set_tile(ib.etf, node);
  }
}

// Eigen-decomposition of a symmetric 3x3 matrix by cyclic Jacobi rotations:
// eigenvalues in d, eigenvectors in the columns of V.
__device__ void jacobi3(double (&M)[3][3], double (&d)[3], double (&V)[3][3]) {
  for (int i = 0; i < 3; i++)
    for (int j = 0; j < 3; j++) V[i][j] = i == j ? 1.0 : 0.0;
  for (int sweep = 0; sweep < 50; sweep++) {
    const double off = M[0][1] * M[0][1] + M[0][2] * M[0][2] + M[1][2] * M[1][2];
    const double dg = M[0][0] * M[0][0] + M[1][1] * M[1][1] + M[2][2] * M[2][2];
    if (off <= 1e-36 * dg) break;
    for (int p = 0; p < 2; p++)
      for (int q = p + 1; q < 3; q++) {
        if (M[p][q] == 0.0) continue;
        const double th = (M[q][q] - M[p][p]) / (2.0 * M[p][q]);
        const double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
        const double c = 1.0 / sqrt(t * t + 1.0), sn = t * c;
        for (int k = 0; k < 3; k++) {  // M <- M J
          const double mkp = M[k][p], mkq = M[k][q];
          M[k][p] = c * mkp - sn * mkq;
          M[k][q] = sn * mkp + c * mkq;
        }
        for (int k = 0; k < 3; k++) {  // M <- J^T M
          const double mpk = M[p][k], mqk = M[q][k];
          M[p][k] = c * mpk - sn * mqk;
          M[q][k] = sn * mpk + c * mqk;
        }
        for (int k = 0; k < 3; k++) {
          const double vkp = V[k][p], vkq = V[k][q];
          V[k][p] = c * vkp - sn * vkq;
          V[k][q] = sn * vkp + c * vkq;
        }
      }
  }
  for (int i = 0; i < 3; i++) d[i] = M[i][i];
}

// Taylor deformation of a body, D = (sqrt(l1) - sqrt(l3)) / (sqrt(l1) +
// sqrt(l3)) from the largest and smallest eigenvalues of the vertex
// second-moment tensor M = sum (x - xbar)(x - xbar)^T / n; one block.  Adds
// D to *jsum, or theta dD/dx = theta (2/n) G (x - xbar) to aP, with G =
// dD/dl1 v1 v1^T + dD/dl3 v3 v3^T.
// Latency-bound (one block): 512 threads keep their first six vertices in
// registers and add their sums in one exchange each for the mean and the
// moments (256 threads, vertices read three times and a sum at a time: 17 us
// for 2562 vertices, 13 us now).
constexpr int TAYLOR_THREADS = 512, TAYLOR_KEEP = 6;
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*sh)[8]) {
#pragma unroll
  for (int k = 0; k < N; k++) v[k] = red64(v[k]);
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < N; k++) sh[threadIdx.x >> 6][k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; k++) {
    v[k] = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); w++) v[k] += sh[w][k];
  }
}
__global__ __launch_bounds__(TAYLOR_THREADS) void k_taylor(BodyArgs b, const double* X, int body, double theta,
                                                           double* aP, double* jsum) {
  __shared__ double sh[TAYLOR_THREADS / 64][8];
  __shared__ double s_G[9];
  const int v0 = b.b_vert0[body], nvb = b.b_nv[body], t = threadIdx.x;
  double x[TAYLOR_KEEP][3], m[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < TAYLOR_KEEP; i++) {
    const int v = t + i * TAYLOR_THREADS;
#pragma unroll
    for (int k = 0; k < 3; k++) {
      x[i][k] = v < nvb ? X[3 * (v0 + v) + k] : 0.0;
      m[k] += x[i][k];
    }
  }
  for (int v = t + TAYLOR_KEEP * TAYLOR_THREADS; v < nvb; v += TAYLOR_THREADS)
    for (int k = 0; k < 3; k++) m[k] += X[3 * (v0 + v) + k];
  block_sums(m, sh);
#pragma unroll
  for (int k = 0; k < 3; k++) m[k] /= nvb;
  double M6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  auto moment = [&](const double (&d)[3]) {
    M6[0] += d[0] * d[0];
    M6[1] += d[0] * d[1];
    M6[2] += d[0] * d[2];
    M6[3] += d[1] * d[1];
    M6[4] += d[1] * d[2];
    M6[5] += d[2] * d[2];
  };
#pragma unroll
  for (int i = 0; i < TAYLOR_KEEP; i++) {
    const double d[3] = {x[i][0] - m[0], x[i][1] - m[1], x[i][2] - m[2]};
    if (t + i * TAYLOR_THREADS < nvb) moment(d);
  }
  for (int v = t + TAYLOR_KEEP * TAYLOR_THREADS; v < nvb; v += TAYLOR_THREADS) {
    const double* p = X + 3 * (long long)(v0 + v);
    const double d[3] = {p[0] - m[0], p[1] - m[1], p[2] - m[2]};
    moment(d);
  }
  block_sums(M6, sh);
  if (t == 0) {
    for (int k = 0; k < 6; k++) M6[k] /= nvb;
    double M[3][3] = {{M6[0], M6[1], M6[2]}, {M6[1], M6[3], M6[4]}, {M6[2], M6[4], M6[5]}};
    double d[3], V[3][3];
    jacobi3(M, d, V);
    int i1 = 0, i3 = 0;
    for (int i = 1; i < 3; i++) {
      if (d[i] > d[i1]) i1 = i;
      if (d[i] < d[i3]) i3 = i;
    }
    const double a = sqrt(d[i1]), c = sqrt(d[i3]), s2 = (a + c) * (a + c);
    if (jsum) *jsum += (a - c) / (a + c);
    const double g1 = c / (a * s2), g3 = -a / (c * s2);  // dD/dl1, dD/dl3
    for (int i = 0; i < 3; i++)
      for (int j = 0; j < 3; j++) s_G[3 * i + j] = g1 * V[i][i1] * V[j][i1] + g3 * V[i][i3] * V[j][i3];
  }
  if (!aP) return;
  __syncthreads();
  const double f = theta * 2.0 / nvb;
  auto add = [&](int v, const double (&d)[3]) {
#pragma unroll
    for (int i = 0; i < 3; i++)
      aP[3 * (v0 + v) + i] += f * (s_G[3 * i] * d[0] + s_G[3 * i + 1] * d[1] + s_G[3 * i + 2] * d[2]);
  };
#pragma unroll
  for (int i = 0; i < TAYLOR_KEEP; i++) {
    const double d[3] = {x[i][0] - m[0], x[i][1] - m[1], x[i][2] - m[2]};
    if (t + i * TAYLOR_THREADS < nvb) add(t + i * TAYLOR_THREADS, d);
  }
  for (int v = t + TAYLOR_KEEP * TAYLOR_THREADS; v < nvb; v += TAYLOR_THREADS) {
    const double* p = X + 3 * (long long)(v0 + v);
    const double d[3] = {p[0] - m[0], p[1] - m[1], p[2] - m[2]};
    add(v, d);
  }
}

// Zero the extra adjoint sources and the fixed-point force in flagged tiles,
// and the flags: a block reads the flags of 256 tiles, then clears the listed
// ones with all its threads.
__global__ __launch_bounds__(256) void k_adjb_clear(Grid G, long long ntiles, double* ext, uint8_t* etf, long long* fx,
                                                    uint8_t* ftf) {
  __shared__ int s_n;
  __shared__ int s_list[256];
  const int t = threadIdx.x;
  if (t == 0) s_n = 0;
  __syncthreads();
  const long long tl = blockIdx.x * 256LL + t;
  if (tl < ntiles) {
    const bool e = etf[tl] != 0, f = ftf[tl] != 0;
    if (e || f) s_list[atomicAdd(&s_n, 1)] = t | (e ? 256 : 0) | (f ? 512 : 0);
    if (e) etf[tl] = 0;
    if (f) ftf[tl] = 0;
  }
  __syncthreads();
  for (int k = t; k < (s_n << TILE_SHIFT); k += 256) {
    const int w = s_list[k >> TILE_SHIFT];
    const long long n = ((blockIdx.x * 256LL + (w & 255)) << TILE_SHIFT) + (k & ((1 << TILE_SHIFT) - 1));
    if (n >= G.Np) continue;
    if (w & 256)
#pragma unroll
      for (int q = 0; q < 7; q++) ext[(long long)q * G.Np + n] = 0.0;
    if (w & 512)
#pragma unroll
      for (int q = 0; q < 3; q++) fx[(long long)q * G.Np + n] = 0;
  }
}

// <w, g> at the non-solid nodes (those with amask bit 31 when use_mask),
// each block adding its sum to part[block] (grid-stride, fixed order).
template <class S>
__global__ __launch_bounds__(256) void k_adj_wdot(FluidArgs a, const S* g, const double* w, const uint32_t* amask,
                                                  int use_mask, double* part) {
  __shared__ double sh[8];
  const Grid& G = a.g;
  double acc = 0.0;
  const int count = a.nbulk_nodes + a.nrec;
  for (int t = blockIdx.x * 256 + threadIdx.x; t < count; t += gridDim.x * 256) {
    if (use_mask && !(amask[t] >> 31)) continue;
    const long long n = t < a.nbulk_nodes ? (long long)a.bulk_list[t] : (long long)a.rec_node[t - a.nbulk_nodes];
    for (int j = 0; j < 19; j++)
      acc += w[(long long)j * G.plane + n] * (double)to_c(g[(long long)j * G.plane + n]);
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] += acc;
}

__global__ __launch_bounds__(256) void k_adj_sum(const double* part, int n, double* out) {
  __shared__ double sh[8];
  double t = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) t += part[k];
  t = block_sum(t, sh);
  if (threadIdx.x == 0) *out = t;
}

hipError_t launch_adjb_vertex(const BodyArgs& b, const AdjIB& ib, hipStream_t s) {
  const int n = std::max(b.nsoft_v, b.nbody);
  if (n > 0) k_adjb_vertex<<<cdiv(n, 256), 256, 0, s>>>(b, ib);
  return hipGetLastError();
}

// The body state of a coupled step's output slot before the step: x^n
// where x^{n+1} will be written, x^{n-1} = the input's x^n, and the input's
// velocities (three arrays of nv3 doubles each).
__global__ __launch_bounds__(256) void k_body_slots(const double* from, double* to, long long nv3) {
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= nv3) return;
  to[i] = from[nv3 + i];
  to[nv3 + i] = from[i];
  to[2 * nv3 + i] = from[2 * nv3 + i];
}

hipError_t launch_body_slots(const double* from, double* to, long long nv3, hipStream_t s) {
  if (nv3 > 0) k_body_slots<<<cdiv(nv3, 256), 256, 0, s>>>(from, to, nv3);
  return hipGetLastError();
}

hipError_t launch_adjb_body(int prec, const FluidArgs& a, const BodyArgs& b, const AdjIB& ib, hipStream_t s) {
  const unsigned grid = (unsigned)(b.n_marker_blocks + b.n_elem_blocks) + cdiv(b.nsoft_v, 64);
  if (grid == 0) return hipSuccess;
  switch (prec) {
    case 0: k_adjb_body<double><<<grid, 256, 0, s>>>(a, b, ib); break;
    case 1: k_adjb_body<float><<<grid, 256, 0, s>>>(a, b, ib); break;
    default: k_adjb_body<_Float16><<<grid, 256, 0, s>>>(a, b, ib); break;
  }
  return hipGetLastError();
}

hipError_t launch_adjb_volume(const BodyArgs& b, const AdjIB& ib, hipStream_t s) {
  if (b.nf > 0) k_adjb_volume<<<cdiv(b.nf, 256), 256, 0, s>>>(b, ib);
  return hipGetLastError();
}

hipError_t launch_adjb_markers(int prec, const FluidArgs& a, const BodyArgs& b, const AdjIB& ib, hipStream_t s) {
  if (b.nf == 0) return hipSuccess;
  const unsigned grid = (unsigned)b.n_marker_blocks;
  switch (prec) {
    case 0: k_adjb_markers<double><<<grid, 256, 0, s>>>(a, b, ib); break;
    case 1: k_adjb_markers<float><<<grid, 256, 0, s>>>(a, b, ib); break;
    default: k_adjb_markers<_Float16><<<grid, 256, 0, s>>>(a, b, ib); break;
  }
  return hipGetLastError();
}

hipError_t launch_taylor(const BodyArgs& b, const double* X, int body, double theta, double* aP, double* jsum,
                         hipStream_t s) {
  k_taylor<<<1, TAYLOR_THREADS, 0, s>>>(b, X, body, theta, aP, jsum);
  return hipGetLastError();
}

hipError_t launch_adjb_clear(const Grid& g, double* ext, uint8_t* etf, long long* fx, uint8_t* ftf, hipStream_t s) {
  const long long ntiles = (g.Np >> TILE_SHIFT) + 1;
  k_adjb_clear<<<cdiv(ntiles, 256), 256, 0, s>>>(g, ntiles, ext, etf, fx, ftf);
  return hipGetLastError();
}

hipError_t launch_adj_wdot(int prec, const FluidArgs& a, const void* g, const double* w, const uint32_t* amask,
                           int use_mask, double* part, hipStream_t s) {
  const int count = a.nbulk_nodes + a.nrec;
  if (count == 0) return hipSuccess;
  const unsigned grid = std::min<unsigned>(cdiv(count, 256), ADJ_BLOCKS);
  switch (prec) {
    case 0: k_adj_wdot<double><<<grid, 256, 0, s>>>(a, (const double*)g, w, amask, use_mask, part); break;
    case 1: k_adj_wdot<float><<<grid, 256, 0, s>>>(a, (const float*)g, w, amask, use_mask, part); break;
    default: k_adj_wdot<_Float16><<<grid, 256, 0, s>>>(a, (const _Float16*)g, w, amask, use_mask, part); break;
  }
  return hipGetLastError();
}

hipError_t launch_adj_sum(const double* part, int n, double* out, hipStream_t s) {
  k_adj_sum<<<1, 256, 0, s>>>(part, n, out);
  return hipGetLastError();
}

}  // namespace lbm
