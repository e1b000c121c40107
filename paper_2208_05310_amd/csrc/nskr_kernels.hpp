// nskr_kernels.hpp -- gfx950 kernels of the DGSEM right-hand side and the
// low-storage RK update for relaxation models 1 and 2 of the non-isothermal
// NSK equations with a van der Waals fluid (arXiv 2208.05310, Sec. 2.3.2, 2.4,
// 3).
//
// Execution model
//   One workgroup owns a few elements (StageTile: each kernel of a stage has
//   its own number), one thread a volume node.  Element tiles are staged in
//   LDS for the 1D derivative sweeps along xi, eta, zeta; face work runs one
//   face point, or one grid line normal to a face pair, per thread.  State is
//   structure-of-arrays [var][element][node]; face traces are face-major
//   [element][face][var][point] so that each element writes its own six faces
//   contiguously and reads all fields of a neighbour's face as one contiguous
//   run.
//
// Data flow of one stage (BR1 needs three neighbour exchanges).  Only what a
// later kernel cannot rebuild from the state goes through memory: the lifted
// gradients never do.
//   k_lift1  : c + neighbour c traces -> lifted grad c; own-face traces of
//              (grad c) . n, of |grad c|^2 and, on walls, of grad c (T2).
//   k_lift2  : U + both sides' conserved and T2 traces -> all lifted
//              gradients, nodal and face temperatures, grad T, lap c; the
//              volume integral of the contravariant fluxes and the point-wise
//              source, into the RK register; the own-face flux traces:
//              convective flux with the own half of the Rusanov dissipation
//              (model 2: the HLLC flux) and viscous flux, or the complete wall
//              flux on wall faces (TF).
//   k_update : TF of both sides -> surface integral, RK stage update, and the
//              conserved face traces of the new state for the next stage.
// Everything that needs the gradients is done in the one kernel that lifts
// them.  Where the update kernel lifted them again for the volume integral,
// the three kernels took 132, 412 and 570 us on 32^3 elements of N = 5 in
// FP64 (71, 232 and 317 us on 48x48x24 of N = 3); this split takes 97, 460
// and 363 us (49, 281 and 212) with the workgroups below, moves 11 % fewer
// bytes and evaluates half as many sweeps.
// The conserved traces rotate over three buffers: stage s reads buffer b(s)
// and writes b(s+1), b = 0 1 0 1 2 (0), so no kernel overwrites traces that
// a neighbouring workgroup may still read.
// Metric terms are per element (affine elements).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nskr {

constexpr int kBlock = 256;

// Global accesses of node- and element-indexed arrays through a wave-uniform
// base pointer and a 32-bit element index: the base stays in scalar
// registers (read-first-lane keeps the compiler from folding it into per-lane
// 64-bit address arithmetic) and the byte offset is one 32-bit vector
// register shared by every field at the same node, so a load or store costs
// no vector address instruction.  Every array addressed this way is below
// 4 GiB (the mesh upload checks it).  Face traces keep 64-bit addresses: one
// per face point, with the field offsets as immediates.
template <typename P> __device__ __forceinline__ P *uniform_ptr(P *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (P *)(((uint64_t)hi << 32) | lo);
}
template <typename T> __device__ __forceinline__ T gld(const T *base, uint32_t i)
{
    typedef __attribute__((address_space(1))) const char gc;
    return *(__attribute__((address_space(1))) const T *)((gc *)uniform_ptr(base) + i * (uint32_t)sizeof(T));
}
template <typename T> __device__ __forceinline__ void gst(T *base, uint32_t i, T v)
{
    typedef __attribute__((address_space(1))) char gc;
    *(__attribute__((address_space(1))) T *)((gc *)uniform_ptr(base) + i * (uint32_t)sizeof(T)) = v;
}
// The same accesses with the non-temporal hint (NT), for the update
// kernel's node arrays on meshes whose node data would fill much of the
// last-level cache: they stream through it instead of displacing the face
// traces that the next kernels read again.
template <bool NT, typename T> __device__ __forceinline__ T gldn(const T *base, uint32_t i)
{
    typedef __attribute__((address_space(1))) const char gc;
    const auto *p = (__attribute__((address_space(1))) const T *)((gc *)uniform_ptr(base) + i * (uint32_t)sizeof(T));
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT, typename T> __device__ __forceinline__ void gstn(T *base, uint32_t i, T v)
{
    typedef __attribute__((address_space(1))) char gc;
    auto *p = (__attribute__((address_space(1))) T *)((gc *)uniform_ptr(base) + i * (uint32_t)sizeof(T));
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

struct Phys {
    double R, a, b, cv, mu, kappa, gam, alpha, beta;
    double inv_Rcv;   // 1 / (R c_v)
    double cs_fac;    // (1 + 1/c_v) R
    double ap;        // alpha for relaxation model 2 (p_alpha = p + ap/2 rho^2), 0 for model 1
    double alpha_2, gam_2, ap_2, a2;  // alpha/2, gamma/2, ap/2, 2 a
    int model;        // 1 or 2
};

// The constants that the fluxes and the source use, in the element type: a
// conversion or product of wave-uniform values is a vector instruction in every
// wave that does it.
template <typename T> struct PhysT {
    T mu, kappa, gam, alpha, beta, gb;  // gb = gamma beta
};

struct BcDev {
    int kind;         // 1 no-slip isothermal with contact angle (moving with uw),
                      // 2 slip adiabatic neutral, 3 generalized Navier slip
    int iso;          // 1: T* = twall in the lifting and k grad T . n (kind 1; kind 3 with gamma3 infinite)
    double twall;
    double rv, rl;    // Maxwell densities at twall
    double gcoef;     // static contact-angle flux g(c) = gcoef (c - rl)(c - rv)
    double uw[3];     // tangential wall velocity (kinds 1, 3)
    double g1, g2, g3, g4;  // gamma_1..gamma_4 (kind 3; zero otherwise)
    double g1_gam;    // gamma_1 / gamma: the dynamic part of g, times div u
    double inv_tw;    // 1 / twall
    int var;          // wall temperature twall + tg . x + rate t (table lookup per face point)
    double tg[3];
    double rate;
    double cg;        // -6 cos(theta) / gamma: gcoef = cg sigma / (rl - rv)^3
    double s2g;       // sqrt(2 gamma): sigma = s2g * (tabulated sigma / sqrt(2 gamma))
};

// Wall-temperature table (Sec. 3.2): kTabN equidistant temperatures on
// [kTabT0, kTabT1], entries (sigma / sqrt(2 gamma), rho_v, rho_l).
constexpr int kTabN = 10000;
constexpr double kTabT0 = 0.3, kTabT1 = 1.0;

// 1D operators for one polynomial degree (host computed, FP64).
struct Basis {
    double Dh[36];    // Dhat[i*P + l] = -(w_l / w_i) D_li
    double L[2][6];   // l_j(-1), l_j(+1)
    double Lh[2][6];  // l_j(-1)/w_j, l_j(+1)/w_j
    double w[6];      // Gauss weights
    double x[6];      // Gauss nodes
};

struct MeshDev {
    int E;
    const int *nbr;      // [E][6] neighbour face and orientation, (6 nb + nf) 8 + o, or -1 on a wall
    const int *bcid;     // [E][6] 0 interior, else 1-based wall index
    // affine elements (the kernels' CV = false instances)
    const double *emet;  // [E][10] Ja[d*3+m], J
    const void *em;      // [E][kEm] what the stage kernels read of an element, in the element type of
                         // the precision: [6][4] outward unit normal and surface element of its
                         // faces, Ja[d*3+m], 1/J
    const double *egeo;  // [E][12] corner 0 and the three edge vectors
    // curved elements (CV = true), in the element type of the precision
    const void *nmet;    // [10][nodes] Ja[d*3+m] and J at every node
    const void *fnrm;    // [E][6][P^2][4] outward unit normal and surface element at every face point
    const double *xnode; // [3][nodes] node coordinates (initial state)
    const BcDev *bcs;
    int wall;            // some face is a wall
    int dyn;             // some Navier-slip wall has gamma_1 != 0 (g needs div u at the wall)
    const double *stab;  // [kTabN][3] wall-temperature table (walls with a temperature gradient)
    int var;             // some wall has a temperature gradient or rate
};

// Values of a record of MeshDev::em, and where Ja and 1/J stand in it.
constexpr int kEm = 36, kEmJa = 24, kEmIJ = 33;

template <int P, int BS = kBlock, int EPB_ = BS / (P * P * P)> struct Tile {
    static constexpr int n2 = P * P, n3 = P * P * P;
    static constexpr int EPB = EPB_;            // elements per block
    static constexpr int NV = EPB * n3;         // nodes per block
    static constexpr int NF = EPB * 6 * n2;     // face points per block
    // Threads per element of the node phases: whole waves where the block has
    // room for it, so that a wave's element (and with it everything read per
    // element) is uniform.
    static constexpr int kWaves = (n3 + 63) / 64 * 64;
    static constexpr bool kUni = EPB * kWaves <= BS;
    static constexpr int TPE = kUni ? kWaves : n3;
};

// Tiles of the stage kernels: elements per workgroup of each kernel and of
// the unit (kTile) in which elements are dealt to the XCDs, a multiple of all
// of them.  Each kernel has its own, since they are bound by different things.
// The update streams and likes groups whose node arrays end on cache lines
// (4 elements of N = 5 are 27 lines of 128 bytes in FP32, 2 in FP64; shared
// lines are fetched and written by two workgroups): 32^3 N = 5, 1 / 2 / 4
// elements: 402 / 368 / 363 us in FP64 and 304 / 261 / 229 in FP32-mixed;
// 16^3 N = 4: 26.9 / 26.6 / 25.5 and 19.2 / 17.2 / 16.3.  k_lift1 at N = 5 takes
// 105 us with one element and 134 with two: short phases between barriers.
template <int P> struct StageTile {
    static constexpr int kLift1 = P == 3 ? 9 : (P == 6 ? 1 : 2);
    static constexpr int kLift2 = P >= 5 ? 1 : (P == 4 ? 2 : 3);
    static constexpr int kUpdate = P == 3 ? 9 : (P == 4 ? 2 : 4);
    static constexpr int kTile = P == 3 ? 9 : (P == 4 ? 2 : 4);
    static constexpr int kFew = P >= 5 ? 1 : kUpdate;  // k_update on meshes of few tiles
    static_assert(kTile % kFew == 0 && kTile % kLift1 == 0 && kTile % kLift2 == 0 && kTile % kUpdate == 0, "tile");
};
// Workgroup of EPB elements in whole waves, with a thread for every node and
// (FACES) for every face point.
template <int P, int EPB, bool FACES> struct Group {
    static constexpr int kNodes = EPB * P * P * P, kFaces = EPB * 6 * P * P;
    static constexpr int NT = ((FACES && kFaces > kNodes ? kFaces : kNodes) + 63) / 64 * 64;
    using G = Tile<P, NT, EPB>;
    static constexpr int kSub = StageTile<P>::kTile / EPB;  // workgroups per tile
    // workgroups of `tiles` tiles: the tiles of each XCD (tile mod 8, as the
    // hardware deals out workgroups) keep their XCD
    static int grid(int tiles) { return kSub == 1 ? tiles : (tiles + 7) / 8 * 8 * kSub; }
    // the tile of workgroup b and its place in it, in elements
    static __device__ __forceinline__ int tile(int b) { return kSub == 1 ? b : b / (8 * kSub) * 8 + b % 8; }
    static __device__ __forceinline__ int part(int b) { return kSub == 1 ? 0 : b / 8 % kSub * EPB; }
};

// Node thread of a workgroup: local element, node of the element, and the
// node's place in the workgroup's tile.
template <typename G> struct NodeTask {
    int le, nd, q;
    bool in;
    __device__ __forceinline__ NodeTask(int t)
    {
        le = t / G::TPE;
        nd = t - le * G::TPE;
        in = le < G::EPB && nd < G::n3;
        q = le * G::n3 + nd;
    }
};

// Value r of element e's record; UNI: e is the same for all lanes of the wave
// and the load a scalar one, whatever the kernel has stored before it (the
// records do not change while a kernel runs).
template <bool UNI, typename T> __device__ __forceinline__ T em_at(const MeshDev &m, int e, int r)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (UNI) {
        const uint32_t u = __builtin_amdgcn_readfirstlane(e);
        return ((const __attribute__((address_space(4))) T *)m.em)[(size_t)u * kEm + r];
    }
#endif
    return gld((const T *)m.em, (uint32_t)e * kEm + r);
}

template <int P> __device__ __forceinline__ int line_node(int d, int l, int p, int q)
{
    return d == 0 ? l + P * (p + P * q) : (d == 1 ? p + P * (l + P * q) : p + P * (q + P * l));
}

// Face point of the neighbour that matches face point fp = p + P q of the
// own face (p, q: the two remaining node indices in increasing axis order)
// under orientation o: (a, b) = (q, p) if o & 4 else (p, q); a -> P-1-a if
// o & 1; b -> P-1-b if o & 2; the neighbour's point is a + P b.
template <int P> __device__ __forceinline__ int orient_fp(int fp, int o)
{
    int a = fp % P, b = fp / P;
    if (o & 4) {
        const int t = a;
        a = b;
        b = t;
    }
    if (o & 1) a = P - 1 - a;
    if (o & 2) b = P - 1 - b;
    return a + P * b;
}

// Face index (6 element + local face) of the neighbour across a face with
// connectivity code `code` >= 0, and the neighbour's matching point.
template <int P> __device__ __forceinline__ size_t nbr_face(int code) { return (size_t)(code >> 3); }
template <int P> __device__ __forceinline__ int nbr_point(int code, int fp) { return orient_fp<P>(fp, code & 7); }

// Outward unit normal and surface element at face point fp of face
// `face` (= 6 element + local face): per face on affine elements, per face
// point on curved ones.
template <int P, typename T, bool CV>
__device__ __forceinline__ void face_normal(const MeshDev &m, size_t face, int fp, T n[3], T &dS)
{
    if (CV) {
        const uint32_t q = ((uint32_t)face * (P * P) + fp) * 4;
        const T *fn = (const T *)m.fnrm;
        n[0] = gld(fn, q);
        n[1] = gld(fn, q + 1);
        n[2] = gld(fn, q + 2);
        dS = gld(fn, q + 3);
    } else {
        const T *em = (const T *)m.em;
        const uint32_t q = (uint32_t)face / 6 * (kEm - 24) + (uint32_t)face * 4;
        n[0] = gld(em, q);
        n[1] = gld(em, q + 1);
        n[2] = gld(em, q + 2);
        dS = gld(em, q + 3);
    }
}
template <int P, typename T, bool CV> __device__ __forceinline__ T face_dS(const MeshDev &m, size_t face, int fp)
{
    if (CV) return gld((const T *)m.fnrm, ((uint32_t)face * (P * P) + fp) * 4 + 3);
    return gld((const T *)m.em, (uint32_t)face / 6 * (kEm - 24) + (uint32_t)face * 4 + 3);
}

// ---------------------------------------------------------------- physics
// 1/x in FP64.  FAST (the FP32-mixed instances, whose inputs carry FP32
// precision): the hardware FP32 reciprocal refined by one Newton step in FP64,
// r + r (1 - x r), relative error about 1e-14 (the square of the FP32
// estimate's); else the correctly rounded division.
template <bool FAST> __device__ __forceinline__ double recip(double x)
{
    if (FAST) {
        const double r = (double)__builtin_amdgcn_rcpf((float)x);
        return fma(r, fma(-x, r, 1.0), r);
    }
    return 1.0 / x;
}

// 1/x in the element type: of FP32 instances the refined reciprocal, rounded,
// which the temperature and the equation of state form anyway.
template <typename T> __device__ __forceinline__ T recip_to(T x) { return T(recip<sizeof(T) == 4>((double)x)); }

// Temperature recovery of eq. totalenergyalpha with eps = R c_v T - a rho
// (always FP64 arithmetic: it cancels large terms near the spinodal).
template <bool FAST = false>
__device__ __forceinline__ double temperature_g2(const Phys &ph, double rho, double m0, double m1, double m2,
                                                 double E, double c, double g2)
{
    const double ir = recip<FAST>(rho);
    double kin = 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) * ir;
    double rel = ph.alpha_2 * (rho - c) * (rho - c);
    double grd = ph.gam_2 * g2;
    return ((E - kin - rel - grd) * ir + ph.a * rho) * ph.inv_Rcv;
}
template <bool FAST = false>
__device__ __forceinline__ double temperature(const Phys &ph, double rho, double m0, double m1, double m2,
                                              double E, double c, double q0, double q1, double q2)
{
    return temperature_g2<FAST>(ph, rho, m0, m1, m2, E, c, q0 * q0 + q1 * q1 + q2 * q2);
}

// van der Waals pressure (eq. pressure) and isentropic sound speed squared
// (eq. speedofsound for the Helmholtz energy of Sec. 2.1), FP64.
template <bool FAST = false>
__device__ __forceinline__ void eos(const Phys &ph, double rho, double T, double &p, double &cs2)
{
    double q = recip<FAST>(1.0 - ph.b * rho);
    p = rho * ph.R * T * q - ph.a * rho * rho;
    cs2 = ph.cs_fac * T * q * q - ph.a2 * rho;
}

// The FP32-mixed instances take the refined reciprocals above.
template <typename T> constexpr bool fast_fp64() { return sizeof(T) == 4; }

// sqrt of a non-negative FP64 value into the element type: FP32 instances
// round the argument and take the FP32 square root.
template <typename T> __device__ __forceinline__ T sqrt_to(double x)
{
    if (sizeof(T) == 4) return T(sqrtf((float)x));
    return T(sqrt(x));
}

// HLLC flux (Toro 2009, Sec. 10.4) of the convective part for relaxation
// model 2 along the unit normal n from the own side (left, uL) to the
// neighbour (right, uR): p is p_alpha, a = sqrt((dp_alpha/drho)_s); Davis wave
// speeds S_L = min(u_L - a_L, u_R - a_R), S_R = max(u_L + a_L, u_R + a_R);
// contact speed S*; the star state keeps its side's tangential velocity and
// c/rho (the order parameter as a passive scalar).
template <typename T>
__device__ __forceinline__ void hllc(const T uL[6], T pL, T aL, const T uR[6], T pR, T aR, const T n[3], T out[6])
{
    const T irL = T(1) / uL[0], irR = T(1) / uR[0];
    const T unL = (uL[1] * n[0] + uL[2] * n[1] + uL[3] * n[2]) * irL;
    const T unR = (uR[1] * n[0] + uR[2] * n[1] + uR[3] * n[2]) * irR;
    const T SL = fmin(unL - aL, unR - aR), SR = fmax(unL + aL, unR + aR);
    // the side whose flux (and star state) is taken
    const T Ss = (pR - pL + uL[0] * unL * (SL - unL) - uR[0] * unR * (SR - unR)) /
                 (uL[0] * (SL - unL) - uR[0] * (SR - unR));
    const bool left = SL >= T(0) || (SR > T(0) && Ss >= T(0));
    const T *u = left ? uL : uR;
    const T un = left ? unL : unR, p = left ? pL : pR, ir = left ? irL : irR;
    const T S = left ? SL : SR;
    out[0] = u[0] * un;
    out[1] = u[1] * un + p * n[0];
    out[2] = u[2] * un + p * n[1];
    out[3] = u[3] * un + p * n[2];
    out[4] = (u[4] + p) * un;
    out[5] = u[5] * un;
    if (SL >= T(0) || SR <= T(0)) return;  // supersonic: the upwind flux
    const T f = u[0] * (S - un) / (S - Ss);
    T us[6];
    us[0] = f;
#pragma unroll
    for (int m = 0; m < 3; ++m) us[1 + m] = f * (u[1 + m] * ir + (Ss - un) * n[m]);
    us[4] = f * (u[4] * ir + (Ss - un) * (Ss + p / (u[0] * (S - un))));
    us[5] = f * u[5] * ir;
#pragma unroll
    for (int v = 0; v < 6; ++v) out[v] += S * (us[v] - u[v]);
}

// Non-conservative source of relaxation model 1, evaluated point-wise with the
// lifted gradients (Sec. 3.1): momentum alpha rho grad(c - rho), energy
// alpha rho grad(c - rho).u + alpha/2 (c^2 - rho^2) div u + gamma (|grad c|^2/2
// div u - grad c (x) grad c : grad u), order parameter alpha beta (rho - c).
// Relaxation model 2 (eq. navierstokeskorteweg_palpha) drops the alpha rho
// grad rho and alpha/2 rho^2 div u parts, which its pressure p_alpha carries.
template <typename T>
__device__ __forceinline__ void source(const PhysT<T> &pt, bool m2, T rho, T c, const T u[3], const T grho[3], const T gu[3][3],
                                       const T gc[3], T S[6])
{
    const T div = gu[0][0] + gu[1][1] + gu[2][2];
    const T al = pt.alpha;
    T d[3], gg = T(0), cc = T(0), du = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        d[i] = m2 ? gc[i] : gc[i] - grho[i];
        gg += gc[i] * gc[i];
        du += d[i] * u[i];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        T r = T(0);
#pragma unroll
        for (int j = 0; j < 3; ++j) r += gc[j] * gu[j][i];
        cc += gc[i] * r;
    }
    S[0] = T(0);
    S[1] = al * rho * d[0];
    S[2] = al * rho * d[1];
    S[3] = al * rho * d[2];
    S[4] = al * rho * du + T(0.5) * al * (m2 ? c * c : c * c - rho * rho) * div +
           pt.gam * (T(0.5) * gg * div - cc);
    S[5] = al * pt.beta * (rho - c);
}

// ------------------------------------------------------------ kernel args
// One problem instance as the kernels see it: caller state, library scratch,
// mesh, physics and its own time step.
template <typename T> struct Inst {
    T *U, *R, *Ut;             // state, RK register, U_t output (rhs)
    T *Ck;                     // compensation of the state update (FP32 Kahan), or null
    T *Q, *TH;                 // grad(rho,u,c) [15] and T, for the API outputs (kUtParts: Q holds the source)
    T *G2;                     // grad T + lap c [4], for the API output only
    T *T2, *TF, *TU;           // face traces: grad c . n, |grad c|^2 (+ grad c on walls) [kT2<T>()],
                               // flux [6],
                               // conserved state [3 buffers][6]; within an array
                               // (a buffer) face-major: [face][field][point]
    MeshDev mesh;
    Phys ph;
    PhysT<T> pt;
    size_t NN;                 // nodes of the instance
    double dt;
    const int *clk;            // batch: steps taken since admission, for walls whose
                               // temperature changes in time (null otherwise)
    double t0;                 // batch: the instance's time at admission
};

// What the stage kernels write.
// kUtParts: U_t in FP32 for model 2, where the divergence of p_alpha (p + alpha/2
// rho^2) and the source alpha rho grad c all but cancel, so that each rounding of
// a value of the size of p_alpha shows.  Of the momenta and the energy (v = 1..4)
// the volume sum and the source go through memory apart (Ut and Q) and meet the
// surface sum unrounded, and so do the convective flux and the own side's
// viscous one (TF, and the traces' second buffer, which only a step uses): U_t
// then differs by 1e-6 (2-norm) from an evaluation with one accumulator, by up to
// 1.3e-4 where they are summed first (33x27x28 elements of N = 4; round-off against
// FP64 6.6e-4 in both).  Its price, on 41x33x35 elements of N = 3: 283 -> 339 us.
// A step keeps the sums: its state does not resolve the difference.  Model 1's U_t
// moves by 3e-6 at most.
enum { kUt, kRk, kG2, kUtParts };

// Kernel argument: a single instance by value, or (BATCH) a device table of
// instances with a block map (instance and first element of every block),
// plus what is common to the launch.
template <typename T> struct Launch {
    Inst<T> one;
    const Inst<T> *tab;
    const int *blk_inst, *blk_e0;
    const int *blk_map;  // single instance: first element of every tile
    Basis bas;
    int mode;        // kUt write U_t; kRk RK stage (update U, R, write traces); kG2 write grad T and lap c
                     // (k_lift2); kUtParts write U_t from its parts
    int first;       // RK: assign R at the first stage
    int last;        // RK: the step's last stage, whose update does not store R (the
                     // next stage to read it is a first stage, which assigns it)
    int tb, tw;      // conserved-trace buffer read by this stage, written for the next
    int full;        // host side: launch the k_lift1 variant that also writes Q and TH
    double A, B;     // RK coefficients of this stage
    double t;        // time of this stage (walls whose temperature changes in time)
    double cs;       // batch: the stage's time fraction c_s of the step
};

// Time of RK stage s of step n from t0: (t0 + n dt) + c_s dt, rounded as the
// host rounds it for a single instance (no fused multiply-adds), so that an
// instance sees bitwise the same stage times alone and in a batch.
__device__ __forceinline__ double stage_time(double t0, int n, double dt, double cs)
{
#pragma clang fp contract(off)
    return (t0 + (double)n * dt) + cs * dt;
}

// Face traces are stored face by face: the K fields of one face's N2 points
// are contiguous ([face][field][point], face = 6 e + f). A block reading a
// neighbour's face then fetches its fields as one run of whole cache lines,
// not K runs of N2 values each that straddle line boundaries, and the field
// offsets are compile-time constants.
// Fields of the T2 face trace: (grad c) . n with the element's own outward
// normal, |grad c|^2, and on wall faces only the vector grad c (the
// tangential gradient of a Navier-slip wall). Interior faces need only the
// first two: the divergence lifting of grad c takes the central normal
// component, and the neighbour's outward normal is minus the own one; the
// face temperature of either side follows from its |grad c|^2 and its
// conserved trace, so the kernel that needs it recovers it there and the one
// that lifts grad c reads one field of the state instead of six.
// FP32 instances store |grad c|^2, formed in FP64, as two floats, the
// rounded value and the rounding error in the field after it, so that the
// face temperature is the one recovered in FP64 (about 48 bits).
template <typename T> constexpr int kT2() { return sizeof(T) == 4 ? 6 : 5; }
template <typename T> constexpr int kT2gc() { return sizeof(T) == 4 ? 3 : 2; }  // first wall grad c field

template <int N2> struct FaceIx {
    size_t face;
    int fp;
    __device__ __forceinline__ FaceIx(size_t fc, int p) : face(fc), fp(p) {}
    // element of field k of a K-field trace array (64-bit: one address per
    // face point, the field offsets folded into the instructions' immediates)
    __device__ __forceinline__ size_t at(int K, int k) const { return (face * K + k) * N2 + fp; }
};


// A pointer read from ordinary device memory is generic to the compiler,
// which then emits flat loads and stores for everything addressed through it.
// The instance table is read-only while a kernel runs, so read it through the
// constant address space: pointers loaded from there are known to point to
// global memory, and accesses through them compile to global loads and stores
// exactly as for pointers passed by value in the kernel arguments.
template <typename P> __device__ __forceinline__ P load_const(const P *p, int i)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return ((const __attribute__((address_space(4))) P *)p)[i];
#else
    return p[i];  // host pass: the body is never run on the host
#endif
}

// The instance and the first element of this workgroup (of `tiles` tiles); false
// for a workgroup past the last tile.
template <int P, typename W, bool BATCH, typename T>
__device__ __forceinline__ bool instance_of(const Launch<T> &L, Inst<T> &a, int &e0, int tiles)
{
    const int b = W::tile(blockIdx.x);
    if (b >= tiles) return false;
    if (BATCH) {
        const int k = load_const(L.blk_inst, b);
        e0 = load_const(L.blk_e0, b);
        a = load_const(L.tab, k);
    } else {
        a = L.one;
        e0 = load_const(L.blk_map, b);
    }
    e0 += W::part(blockIdx.x);
    return true;
}

// Pairs of fields.  The LDS delivers 128-bit reads at the same rate per
// instruction as 64-bit ones (measured: 4.5 against 4.4 cycles per wave
// instruction, 137 against 71 TB/s over the chip; 5.4 and 5.3 along the lines
// of an N = 5 element), and the stage kernels read every node value once per
// node of its three lines, so fields that are swept together lie together.
template <typename T> using V2 = T __attribute__((ext_vector_type(2)));

// 1D operators in LDS (the rows each thread needs differ per lane), in the
// element type of the kernel: FP32 instances then read and multiply floats
// (the values are the FP64 host basis rounded once, as a conversion at every
// use would round them).  Rows are padded to whole pairs.
template <int P, typename T> struct alignas(16) BasisS {
    static constexpr int PS = (P + 1) / 2 * 2;
    T Dh[P * PS];     // Dhat, row i at i PS
    T Lf[2 * PS];     // l_j(-1), l_j(+1)
    V2<T> L[P];       // (l_j(-1), l_j(+1))
    V2<T> Lh[P];      // (l_j(-1), l_j(+1)) / w_j
    __device__ __forceinline__ void load(const Basis &b)
    {
        const int t = threadIdx.x;
        if (t < P * P) Dh[t / P * PS + t % P] = T(b.Dh[t]);
        if (t < 2 * P) Lf[t / P * PS + t % P] = T(b.L[t / P][t % P]);
        if (t < P) {
            L[t] = V2<T>{T(b.L[0][t]), T(b.L[1][t])};
            Lh[t] = V2<T>{T(b.Lh[0][t]), T(b.Lh[1][t])};
        }
    }
    // a padded row of P values
    static __device__ __forceinline__ void row(const T *r, T out[P])
    {
        const V2<T> *v = (const V2<T> *)r;
#pragma unroll
        for (int l = 0; l < P / 2; ++l) {
            const V2<T> q = v[l];
            out[2 * l] = q.x;
            out[2 * l + 1] = q.y;
        }
        if constexpr (P % 2) out[P - 1] = r[P - 1];
    }
};

// Line task: the line of P nodes through face point (p,q) along direction d
// of local element le; it carries the two face points of faces 2d (xi^d = -1)
// and 2d+1 (+1), so each LDS value of the line is read once for both faces.
template <int P> struct LineTask {
    int le, d, fp, p, q;
    int off, str;  // node l of the line is off + l * str (element-local)
    __device__ __forceinline__ LineTask(int task)
    {
        le = task / (3 * P * P);
        const int r = task - le * 3 * P * P;
        d = r / (P * P);
        fp = r - d * P * P;
        p = fp % P;
        q = fp / P;
        // d = 0: (l, p, q); d = 1: (p, l, q); d = 2: (p, q, l)
        off = d == 0 ? P * fp : (d == 1 ? p + P * P * q : fp);
        str = d == 0 ? 1 : (d == 1 ? P : P * P);
    }
};

// Bounds the loads that a sweep keeps in flight: what has been loaded is
// summed into a[0..n) before anything that follows is loaded.  Without it the
// compiler requests a whole line of every field at once and needs the
// registers of one or two waves per SIMD for it.
template <typename T> __device__ __forceinline__ void bound(T *a, int n)
{
#pragma unroll
    for (int k = 0; k < n; ++k) asm volatile("" : "+v"(a[k]));
    __builtin_amdgcn_sched_barrier(0);
}

// Prolongation of one LDS field of an element, or of a pair of fields, to
// both faces of a line.
template <int P, typename T>
__device__ __forceinline__ void prolong2(const T *s, int base, const BasisS<P, T> &B, const LineTask<P> &lt, T &vm,
                                         T &vp)
{
    T am = T(0), ap = T(0);
    const T *ln = s + base + lt.off;
#pragma unroll
    for (int l = 0; l < P; ++l) {
        const T v = ln[l * lt.str];
        const V2<T> w = B.L[l];
        am += w.x * v;
        ap += w.y * v;
    }
    vm = am;
    vp = ap;
}
template <int P, typename T, bool LIM = false>
__device__ __forceinline__ void prolong2(const V2<T> *s, int base, const BasisS<P, T> &B, const LineTask<P> &lt,
                                         T *vm, T *vp)
{
    T a[4] = {T(0), T(0), T(0), T(0)};
    const V2<T> *ln = s + base + lt.off;
#pragma unroll
    for (int l = 0; l < P; ++l) {
        const V2<T> v = ln[l * lt.str], w = B.L[l];
        a[0] += w.x * v.x;
        a[1] += w.y * v.x;
        a[2] += w.x * v.y;
        a[3] += w.y * v.y;
        if (LIM && l % 2 == 1) bound(a, 4);
    }
    vm[0] = a[0];
    vm[1] = a[2];
    vp[0] = a[1];
    vp[1] = a[3];
}

// Face task: face point fp of face f of local element le, with the line of
// the element that ends on it (node l of the line is off + l * str).
template <int P> struct FaceTask {
    int le, f, fp, off, str;
    __device__ __forceinline__ FaceTask(int task)
    {
        constexpr int n2 = P * P;
        le = task / (6 * n2);
        const int r = task - le * 6 * n2;
        f = r / n2;
        fp = r - f * n2;
        const int d = f >> 1, p = fp % P, q = fp / P;
        off = d == 0 ? P * fp : (d == 1 ? p + P * P * q : fp);
        str = d == 0 ? 1 : (d == 1 ? P : P * P);
    }
};

template <typename G> __device__ __forceinline__ constexpr int n_lines() { return G::EPB * 3 * G::n2; }

// Line task of thread t, or -1.  The lines fill the first waves of the
// workgroup lane by lane, so waves without lines issue no instructions for
// the line phases (at N = 5, 108 lines take two waves, not 27 lanes in each
// of four: lift1 9-10 % faster on the 32^3 case in both precisions).
template <typename G> __device__ __forceinline__ int line_of_thread(int t)
{
    return t < n_lines<G>() ? t : -1;
}

// ------------------------------------------------------------ shared pieces
// Primitive variables (rho, u, v, w, c) of a conserved state.  SHARED: with the
// reciprocal that the temperature of the same state forms.
template <typename T, bool SHARED = false> __device__ __forceinline__ void primitives(const T u6[6], T w[5])
{
    const T ir = SHARED ? recip_to(u6[0]) : T(1) / u6[0];
    w[0] = u6[0];
    w[1] = u6[1] * ir;
    w[2] = u6[2] * ir;
    w[3] = u6[3] * ir;
    w[4] = u6[5];
}

// BR1 face values of the primitives on a wall face: the interior values with
// the velocity set to the wall's (no-slip) or stripped of its normal part
// (slip and Navier-slip walls).
template <typename T>
__device__ __forceinline__ void wall_primitives(const MeshDev &m, int el, int f, const T n[3], T w[5])
{
    const BcDev &bc = m.bcs[m.bcid[el * 6 + f] - 1];
    if (bc.kind == 1) {
        w[1] = T(bc.uw[0]);
        w[2] = T(bc.uw[1]);
        w[3] = T(bc.uw[2]);
    } else {
        const T un = w[1] * n[0] + w[2] * n[1] + w[3] * n[2];
        w[1] -= un * n[0];
        w[2] -= un * n[1];
        w[3] -= un * n[2];
    }
}

// Wall temperature twall + tg . x + rate t at a wall face point (x from the
// element's corner and edge vectors at the face point's reference
// coordinates: +-1 along the face's axis, the Gauss nodes of its two
// tangential indices along the others).
template <int P>
__device__ __forceinline__ double wall_temperature(const MeshDev &m, const Basis &bas, const BcDev &bc, int el, int f,
                                                   int fp, double t)
{
    const int d = f >> 1;
    const double xn = (f & 1) ? 1.0 : -1.0, xa = bas.x[fp % P], xb = bas.x[fp / P];
    const double r0 = d == 0 ? xn : xa, r1 = d == 1 ? xn : (d == 0 ? xa : xb), r2 = d == 2 ? xn : xb;
    const double *g = m.egeo + (size_t)el * 12;
    double Tw = bc.twall;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        Tw += bc.tg[k] * (g[k] + 0.5 * ((r0 + 1.0) * g[3 + k] + (r1 + 1.0) * g[6 + k] + (r2 + 1.0) * g[9 + k]));
    return Tw + bc.rate * t;
}

// Wall temperature and contact-angle constants at one wall face point: the
// wall's constants for a fixed temperature; for a temperature varying along
// the wall, sigma, rho_v, rho_l interpolated linearly in the table at T_w.
struct WallPt {
    double Tw, rv, rl, gcoef;
};
template <int P>
__device__ __forceinline__ WallPt wall_point(const MeshDev &m, const Basis &bas, const BcDev &bc, int el, int f, int fp,
                                             double t)
{
    WallPt w{bc.twall, bc.rv, bc.rl, bc.gcoef};
    if (!bc.var) return w;
    const double Tw = wall_temperature<P>(m, bas, bc, el, f, fp, t);
    const double sx = (Tw - kTabT0) / ((kTabT1 - kTabT0) / (kTabN - 1));
    int k = (int)floor(sx);
    k = k < 0 ? 0 : (k > kTabN - 2 ? kTabN - 2 : k);
    const double wt = sx - k;
    const double *t0 = m.stab + 3 * k;
    const double sig = bc.s2g * ((1.0 - wt) * t0[0] + wt * t0[3]);
    w.Tw = Tw;
    w.rv = (1.0 - wt) * t0[1] + wt * t0[4];
    w.rl = (1.0 - wt) * t0[2] + wt * t0[5];
    const double dd = w.rl - w.rv;
    w.gcoef = bc.cg * sig / (dd * dd * dd);
    return w;
}

// BR1 lifted gradient of one field at element-local node (i, j, k):
// J q_m = sum_d Ja^d_m (Dhat w + lhat(+1) w*_+ - lhat(-1) w*_-), from the node
// values fw (element starting at base) and face values fs (element's face
// points starting at fbase) in LDS.
template <int P, typename T, bool LIM = false>
__device__ __forceinline__ void lifted_grad(const T *fw, const T *fs, int base, int fbase, int i, int j, int k,
                                            const BasisS<P, T> &B, const T Ja[9], T iJ, T q[3])
{
    constexpr int n2 = P * P;
    const int idx[3] = {i, j, k};
    const int fpd[3] = {j + P * k, i + P * k, i + P * j};
    T gd[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T acc = T(0), D[P];
        const int p = d == 0 ? j : i, r = d == 2 ? j : k;
        B.row(B.Dh + idx[d] * B.PS, D);
#pragma unroll
        for (int l = 0; l < P; ++l) acc += D[l] * fw[base + line_node<P>(d, l, p, r)];
        if (LIM) bound(&acc, 1);
        const V2<T> lh = B.Lh[idx[d]];
        acc += lh.y * fs[fbase + (2 * d + 1) * n2 + fpd[d]];
        acc -= lh.x * fs[fbase + (2 * d) * n2 + fpd[d]];
        gd[d] = acc;
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) q[m] = iJ * (Ja[m] * gd[0] + Ja[3 + m] * gd[1] + Ja[6 + m] * gd[2]);
}

// Five fields of a tile: two rows of pairs and one single row.
template <typename T> struct Five {
    const V2<T> *a, *b;
    const T *c;
    __device__ __forceinline__ void at(int n, T v[5]) const
    {
        const V2<T> x = a[n], y = b[n];
        v[0] = x.x;
        v[1] = x.y;
        v[2] = y.x;
        v[3] = y.y;
        v[4] = c[n];
    }
};

// The same lifted gradient for five fields at once, sweeping direction by
// direction so that only one row of Dhat is live: the reference derivatives
// gd[f][d], before the metric transform.
template <int P, typename T>
__device__ __forceinline__ void lifted_grads(const Five<T> &w, const Five<T> &s, int base, int fbase, int i, int j,
                                             int k, const BasisS<P, T> &B, T gd[5][3])
{
    constexpr int n2 = P * P;
    const int idx[3] = {i, j, k};
    const int fpd[3] = {j + P * k, i + P * k, i + P * j};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = d == 0 ? j : i, r = d == 2 ? j : k;
        T D[P], acc[5] = {T(0), T(0), T(0), T(0), T(0)}, v[5];
        B.row(B.Dh + idx[d] * B.PS, D);
#pragma unroll
        for (int l = 0; l < P; ++l) {
            w.at(base + line_node<P>(d, l, p, r), v);
#pragma unroll
            for (int f = 0; f < 5; ++f) acc[f] += D[l] * v[f];
            if (l % 2 == 1) bound(acc, 5);
        }
        bound(acc, 5);
        const V2<T> lh = B.Lh[idx[d]];
        s.at(fbase + (2 * d + 1) * n2 + fpd[d], v);
#pragma unroll
        for (int f = 0; f < 5; ++f) acc[f] += lh.y * v[f];
        s.at(fbase + (2 * d) * n2 + fpd[d], v);
#pragma unroll
        for (int f = 0; f < 5; ++f) gd[f][d] = acc[f] - lh.x * v[f];
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Curved elements: the same BR1 lifting in the conservative form with the
// metrics inside the derivative, J q_m = sum_d sum_l Dhat (Ja^d_m w)_l +
// sum_faces lhat w* (n dS)_m, for NFLD fields; node(n, v) and face(n, v) give
// the fields at a tile node and a face point; sJ and sJz hold Ja^d (pair and
// third component, row d) at every node of the tile, sN the outward n dS at
// every face point.  Returns the physical gradients times 1/J (iJ of this node).
template <int P, int NFLD, int NVS, int NFS, typename T, typename FN, typename FS>
__device__ __forceinline__ void lifted_grads_curved(FN node, FS face, const V2<T> (*sJ)[NVS], const T (*sJz)[NVS],
                                                    const T (*sN)[NFS], int base, int fbase, int i, int j, int k,
                                                    const BasisS<P, T> &B, T iJ, T q[NFLD][3])
{
    constexpr int n2 = P * P;
    const int idx[3] = {i, j, k};
    const int fpd[3] = {j + P * k, i + P * k, i + P * j};
#pragma unroll
    for (int f = 0; f < NFLD; ++f) q[f][0] = q[f][1] = q[f][2] = T(0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = d == 0 ? j : i, r = d == 2 ? j : k;
        T D[P], v[NFLD];
        B.row(B.Dh + idx[d] * B.PS, D);
#pragma unroll
        for (int l = 0; l < P; ++l) {
            const int n = base + line_node<P>(d, l, p, r);
            const V2<T> jj = sJ[d][n];
            const T a0 = D[l] * jj.x, a1 = D[l] * jj.y, a2 = D[l] * sJz[d][n];
            node(n, v);
#pragma unroll
            for (int f = 0; f < NFLD; ++f) {
                q[f][0] += a0 * v[f];
                q[f][1] += a1 * v[f];
                q[f][2] += a2 * v[f];
            }
        }
        const V2<T> lh = B.Lh[idx[d]];
        // the two faces' terms enter as one correction: they all but cancel, and
        // added one after the other their round-off moves an FP32 U_t by 1.5e-5
        // (2-norm, 6x6x5 elements of N = 5; 58.1 against 57.0 us in FP64 on 16^3
        // elements of N = 4)
        const int pp = fbase + (2 * d + 1) * n2 + fpd[d], pm = fbase + (2 * d) * n2 + fpd[d];
        T vm[NFLD];
        face(pp, v);
        face(pm, vm);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const T np = lh.y * sN[m][pp], nm = lh.x * sN[m][pm];
#pragma unroll
            for (int f = 0; f < NFLD; ++f) q[f][m] += np * v[f] + nm * vm[f];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int f = 0; f < NFLD; ++f)
#pragma unroll
        for (int m = 0; m < 3; ++m) q[f][m] *= iJ;
}

// Per-node metrics of a curved element tile into LDS (Ja^d as a pair and the
// third component) and this node's 1/J; q is the node's place in the tile, g
// its global node index.
template <typename T, int NVS>
__device__ __forceinline__ T stage_node_metrics(const MeshDev &m, size_t NN, size_t g, int q, V2<T> (*sJ)[NVS],
                                                T (*sJz)[NVS])
{
    const T *nm = (const T *)m.nmet;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        sJ[d][q] = V2<T>{gld(nm + (3 * d) * NN, (uint32_t)g), gld(nm + (3 * d + 1) * NN, (uint32_t)g)};
        sJz[d][q] = gld(nm + (3 * d + 2) * NN, (uint32_t)g);
    }
    return T(1) / gld(nm + 9 * NN, (uint32_t)g);
}

// Physical gradient from the reference derivatives: 1/J times the sum of Ja^d
// times derivative d; on a box along the axes (DIAG) bitwise the general form,
// whose other products are zero there.  The sum is scaled and not Ja^d by 1/J
// beforehand: that factor's rounding is the same at every node of an element,
// and one in grad c or grad rho does not cancel in the source (FP32, 7x6x5
// elements of N = 3: 1.75e-6 of U_t in the 2-norm, of 2.3e-5 in all).
template <bool DIAG, typename T>
__device__ __forceinline__ void to_physical(const T Ja[9], T iJ, const T gd[3], T q[3])
{
    if constexpr (DIAG) {  // Ja^d along axis d
#pragma unroll
        for (int m = 0; m < 3; ++m) q[m] = iJ * (Ja[4 * m] * gd[m]);
        return;
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) q[m] = iJ * (Ja[m] * gd[0] + Ja[3 + m] * gd[1] + Ja[6 + m] * gd[2]);
}

template <bool UNI, typename T> __device__ __forceinline__ void element_metrics(const MeshDev &m, int e, T Ja[9], T &iJ)
{
#pragma unroll
    for (int r = 0; r < 9; ++r) Ja[r] = em_at<UNI, T>(m, e, kEmJa + r);
    iJ = em_at<UNI, T>(m, e, kEmIJ);
}

// ------------------------------------------------------------ k_prolong
// Conserved face traces of the state (into trace buffer L.tw).
template <int P> using ProlongGroup = Group<P, StageTile<P>::kLift1, false>;

template <int P, typename T>
__global__ __launch_bounds__(ProlongGroup<P>::NT) void k_prolong(Launch<T> L, int tiles)
{
    using W = ProlongGroup<P>;
    using G = typename W::G;
    constexpr int BS = W::NT;
    Inst<T> a;
    int e0;
    if (!instance_of<P, W, false>(L, a, e0, tiles)) return;
    __shared__ V2<T> sU[3][G::NV];
    __shared__ BasisS<P, T> B;
    B.load(L.bas);
    const int E = a.mesh.E;
    const int t = threadIdx.x;
    const NodeTask<G> nt(t);
    if (nt.in && e0 + nt.le < E) {
        const uint32_t g32 = (uint32_t)e0 * G::n3 + nt.q;
#pragma unroll
        for (int v = 0; v < 3; ++v) sU[v][nt.q] = V2<T>{gld(a.U + (2 * v) * a.NN, g32), gld(a.U + (2 * v + 1) * a.NN, g32)};
    }
    __syncthreads();
    const size_t NF = (size_t)E * 6 * G::n2;
    T *TU = a.TU + (size_t)L.tw * 6 * NF;
    for (int task = t; task < n_lines<G>(); task += BS) {
        LineTask<P> lt(task);
        const int e = e0 + lt.le;
        if (e >= E) continue;
        const int base = lt.le * G::n3;
        T um[6], up[6];
#pragma unroll
        for (int v = 0; v < 3; ++v) prolong2<P, T>(sU[v], base, B, lt, um + 2 * v, up + 2 * v);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const FaceIx<G::n2> o((size_t)e * 6 + 2 * lt.d + s, lt.fp);
#pragma unroll
            for (int v = 0; v < 6; ++v) TU[o.at(6, v)] = s ? up[v] : um[v];
        }
    }
}

// ------------------------------------------------------------ k_lift1
// Lifted grad c, and the own-face traces of grad c and of the face
// temperature.  FULL: also every lifted gradient and the nodal temperature
// (Q, TH) for the API outputs.
// The per-stage instances are bound by the latency of their short phases and
// keep as many waves per SIMD as their registers allow without spills.
// PIPE (meshes of many groups per resident workgroup): the workgroup takes
// every gridDim-th group of elements and has the next group's c, connectivity
// and neighbour traces in flight while it works on one.  One group per
// workgroup / pipelined: 32^3 N = 5 112 / 97 us in FP64, 85 / 70 in FP32-mixed;
// 50^3 N = 3 FP64 116 / 103; where the groups are few the loop only costs
// (16^3 N = 4 FP64 8.6 / 9.3, 4^3 N = 3 4.2 / 5.4).
template <int P, typename T, bool FULL, bool CV, bool PIPE> constexpr int lift1_waves()
{
    if (FULL || CV) return 1;
    if (PIPE) return sizeof(T) == 4 || P == 4 ? 8 : 6;  // (P == 6 FP64 at 7: 13 spills, 126 us against 97)
    return sizeof(T) == 4 ? 7 : (P == 6 ? 8 : (P == 4 ? 6 : 1));
}
template <int P> using Lift1Group = Group<P, StageTile<P>::kLift1, false>;

template <int P, typename T, bool BATCH, bool FULL = false, bool CV = false, bool PIPE = false>
__global__ __launch_bounds__(Lift1Group<P>::NT, (lift1_waves<P, T, FULL, CV, PIPE>())) void k_lift1(Launch<T> L, int tiles)
{
    using W = Lift1Group<P>;
    using G = typename W::G;
    constexpr int BS = W::NT;
    Inst<T> a;
    int e0;
    if (!instance_of<P, W, BATCH>(L, a, e0, tiles)) return;
    static_assert(!PIPE || (!BATCH && !FULL && !CV), "one instance, affine elements");
    static_assert(n_lines<G>() <= BS, "one line per thread");
    // state (c only, or with FULL all of it) and primitives (FULL), BR1 face
    // values of c or of all primitives
    constexpr int NU = FULL ? 6 : 1, NS = FULL ? 5 : 1, kC = NU - 1;
    // curved elements: the metrics of every node and n dS of every face point
    constexpr int NJ = CV ? 3 : 1, NQ = CV ? 3 : 1, NJV = CV ? G::NV : 1, NQF = CV ? G::NF : 1;
    __shared__ T sU[NU][G::NV];
    __shared__ T sW[FULL ? 5 : 1][FULL ? G::NV : 1];
    __shared__ T sS[NS][G::NF];
    __shared__ V2<T> sG[G::NV];    // grad c
    __shared__ T sGz[G::NV];
    __shared__ V2<T> sJ[NJ][NJV];
    __shared__ T sJz[NJ][NJV];
    __shared__ T sN[NQ][NQF];
    __shared__ BasisS<P, T> B;
    B.load(L.bas);
    const int E = a.mesh.E;
    const size_t NF = (size_t)E * 6 * G::n2;
    constexpr bool full = FULL;
    const T *TU = a.TU + (size_t)L.tb * 6 * NF;

    // early loads: own nodes, and the neighbour traces of this thread's line
    int nbm = -1, nbp = -1;
    T wn[2][6], c0 = T(0);
    auto load_codes = [&](int t, int first, int &cm, int &cp) {
        cm = cp = -1;
        const int ltask = line_of_thread<G>(t);
        const LineTask<P> lt(ltask < 0 ? 0 : ltask);
        const int el = first + lt.le;
        if (ltask < 0 || el >= E) return;
        cm = gld(a.mesh.nbr, el * 6 + 2 * lt.d);
        cp = gld(a.mesh.nbr, el * 6 + 2 * lt.d + 1);
    };
    auto load_traces = [&](int t, int cm, int cp, T w[2][6]) {
        const int ltask = line_of_thread<G>(t);
        const LineTask<P> lt(ltask < 0 ? 0 : ltask);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int nb = s ? cp : cm;
            if (nb >= 0) {
                const FaceIx<G::n2> o(nbr_face<P>(nb), nbr_point<P>(nb, lt.fp));
                if (full) {
#pragma unroll
                    for (int v = 0; v < 6; ++v)
                        if (v != 4) w[s][v] = TU[o.at(6, v)];
                } else {
                    w[s][5] = TU[o.at(6, 5)];
                }
            }
        }
    };
    auto load_c = [&](int t, int first) -> T {
        const NodeTask<G> nt(t);
        const int le = nt.le, tq = nt.q;
        return nt.in && first + le < E ? gld(a.U + 5 * a.NN, (uint32_t)first * G::n3 + tq) : T(0);
    };
    load_codes(threadIdx.x, e0, nbm, nbp);
    if (!FULL) c0 = load_c(threadIdx.x, e0);
    load_traces(threadIdx.x, nbm, nbp, wn);
    // the group after this one: its first element (-1: none) and codes
    int vb = blockIdx.x, en = -1, cnm = -1, cnp = -1;
    auto next_group = [&]() {
        vb += gridDim.x;
        const int tile = W::tile(vb);
        return tile < tiles ? load_const(L.blk_map, tile) + W::part(vb) : -1;
    };
    if constexpr (PIPE) {
        en = next_group();
        if (en >= 0) load_codes(threadIdx.x, en, cnm, cnp);
    }
    for (;;) {
        // (an opaque thread index: what follows from it is formed again for each
        // group instead of being kept in registers across them)
        int t = threadIdx.x;
        if constexpr (PIPE) asm volatile("" : "+v"(t));
        const NodeTask<G> nt(t);
        const int le = nt.le, nd = nt.nd, tq = nt.q;
        const int ltask = line_of_thread<G>(t);
        const LineTask<P> lt(ltask < 0 ? 0 : ltask);
        const int e = e0 + le, el = e0 + lt.le;
        const bool act = nt.in && e < E, lact = ltask >= 0 && el < E;
        const size_t g = (size_t)e0 * G::n3 + tq;
        const uint32_t g32 = (uint32_t)g;
        T iJn = T(0);
        if (act) {
            if constexpr (FULL) {
                T u6[6], w[5];
#pragma unroll
                for (int v = 0; v < 6; ++v) { u6[v] = gld(a.U + (v) * a.NN, g32); sU[v][tq] = u6[v]; }
                primitives(u6, w);
#pragma unroll
                for (int k = 0; k < 5; ++k) sW[k][tq] = w[k];
            } else {
                sU[kC][tq] = c0;
            }
            if constexpr (CV) iJn = stage_node_metrics<T, NJV>(a.mesh, a.NN, g, tq, sJ, sJz);
        }
        T w1[2][6];
        T c1 = T(0);
        int e2 = -1, c2m = -1, c2p = -1;
        if constexpr (PIPE) {
            if (en >= 0) {
                load_traces(t, cnm, cnp, w1);
                c1 = load_c(t, en);
                e2 = next_group();
                if (e2 >= 0) load_codes(t, e2, c2m, c2p);
            }
        }
        __syncthreads();
        // BR1 face values w* on both faces of the line
        if (lact) {
            const int base = lt.le * G::n3;
            T uf[2][6];
            if constexpr (FULL) {
#pragma unroll
                for (int v = 0; v < 6; ++v) prolong2<P, T>(sU[v], base, B, lt, uf[0][v], uf[1][v]);
            } else {
                prolong2<P, T>(sU[kC], base, B, lt, uf[0][5], uf[1][5]);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int f = 2 * lt.d + s;
                const int nb = s ? nbp : nbm;
                const int slot = lt.le * 6 * G::n2 + f * G::n2 + lt.fp;
                if constexpr (CV) {
                    T n[3], dS;
                    face_normal<P, T, true>(a.mesh, (size_t)el * 6 + f, lt.fp, n, dS);
#pragma unroll
                    for (int m = 0; m < 3; ++m) sN[m][slot] = n[m] * dS;
                }
                if (full) {
                    T w[5];
                    primitives(uf[s], w);
                    if (nb >= 0) {
                        T v5[5];
                        primitives(wn[s], v5);
#pragma unroll
                        for (int k = 0; k < 5; ++k) w[k] = T(0.5) * (w[k] + v5[k]);
                    } else {
                        T n[3], dS;
                        face_normal<P, T, CV>(a.mesh, (size_t)el * 6 + f, lt.fp, n, dS);
                        wall_primitives(a.mesh, el, f, n, w);
                    }
#pragma unroll
                    for (int k = 0; k < NS; ++k) sS[k][slot] = w[k];
                } else {
                    sS[NS - 1][slot] = nb >= 0 ? T(0.5) * (uf[s][5] + wn[s][5]) : uf[s][5];
                }
            }
        }
        __syncthreads();
        T qc[3] = {T(0), T(0), T(0)};
        if (act) {
            const int i = nd % P, j = (nd / P) % P, k = nd / (P * P);
            const int base = le * G::n3, fbase = le * 6 * G::n2;
            if constexpr (CV) {
                constexpr int NG = FULL ? 5 : 1;
                auto node = [&](int n, T v[NG]) {
#pragma unroll
                    for (int f = 0; f < NG; ++f) v[f] = FULL ? sW[f][FULL ? n : 0] : sU[kC][n];
                };
                auto face = [&](int n, T v[NG]) {
#pragma unroll
                    for (int f = 0; f < NG; ++f) v[f] = sS[f][n];
                };
                T q[NG][3];
                lifted_grads_curved<P, NG, G::NV, G::NF>(node, face, sJ, sJz, sN, base, fbase, i, j, k, B, iJn, q);
                if constexpr (FULL) {
#pragma unroll
                    for (int w = 0; w < 4; ++w)
#pragma unroll
                        for (int m = 0; m < 3; ++m) gst(a.Q + ((3 * w + m)) * a.NN, g32, T(q[w][m]));
                }
#pragma unroll
                for (int m = 0; m < 3; ++m) qc[m] = q[NG - 1][m];
            } else {
                T Ja[9], iJ;
                element_metrics<G::kUni>(a.mesh, e, Ja, iJ);
                if (full) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        T q[3];
                        lifted_grad<P, T>(sW[w], sS[w], base, fbase, i, j, k, B, Ja, iJ, q);
#pragma unroll
                        for (int m = 0; m < 3; ++m) gst(a.Q + ((3 * w + m)) * a.NN, g32, T(q[m]));
                    }
                }
                lifted_grad<P, T, PIPE>(sU[kC], sS[NS - 1], base, fbase, i, j, k, B, Ja, iJ, qc);
            }
            if constexpr (FULL) {
#pragma unroll
                for (int m = 0; m < 3; ++m) gst(a.Q + ((12 + m)) * a.NN, g32, T(qc[m]));
                const double Tn = temperature<fast_fp64<T>()>(a.ph, (double)sU[0][tq], (double)sU[1][tq], (double)sU[2][tq], (double)sU[3][tq],
                                              (double)sU[4][tq], (double)sU[5][tq], (double)qc[0], (double)qc[1],
                                              (double)qc[2]);
                gst(a.TH, g32, T(Tn));
            }
        }
        if (act) {
            sG[tq] = V2<T>{qc[0], qc[1]};
            sGz[tq] = qc[2];
        }
        __syncthreads();
        if (lact) {
            const int base = lt.le * G::n3;
            T qf[2][3];
            prolong2<P, T, PIPE>(sG, base, B, lt, qf[0], qf[1]);
            prolong2<P, T>(sGz, base, B, lt, qf[0][2], qf[1][2]);
            // outward normal of each face of this line: on affine elements the -
            // face's is the exact negative of the + face's, as the mesh upload
            // forms them
            T nf[2][3];
            if constexpr (CV) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    T dS;
                    face_normal<P, T, true>(a.mesh, (size_t)el * 6 + 2 * lt.d + s, lt.fp, nf[s], dS);
                }
            } else {
                T dS;
                face_normal<P, T, false>(a.mesh, (size_t)el * 6 + 2 * lt.d + 1, lt.fp, nf[1], dS);
#pragma unroll
                for (int m = 0; m < 3; ++m) nf[0][m] = -nf[1][m];
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const FaceIx<G::n2> o((size_t)el * 6 + 2 * lt.d + s, lt.fp);
                a.T2[o.at(kT2<T>(), 0)] = qf[s][0] * nf[s][0] + qf[s][1] * nf[s][1] + qf[s][2] * nf[s][2];
                const double q0 = (double)qf[s][0], q1 = (double)qf[s][1], q2 = (double)qf[s][2];
                const double g2 = q0 * q0 + q1 * q1 + q2 * q2;
                const T gh = T(g2);
                a.T2[o.at(kT2<T>(), 1)] = gh;
                if constexpr (sizeof(T) == 4) a.T2[o.at(kT2<T>(), 2)] = T(g2 - (double)gh);
            }
            // wall faces also keep the vector grad c (Navier-slip traction), in
            // a loop of its own: inside the one above the branch costs ~40 VGPRs
#pragma unroll
            for (int s = 0; s < 2; ++s)
                if ((s ? nbp : nbm) < 0) {
                    const FaceIx<G::n2> o((size_t)el * 6 + 2 * lt.d + s, lt.fp);
                    a.T2[o.at(kT2<T>(), kT2gc<T>())] = qf[s][0];
                    a.T2[o.at(kT2<T>(), kT2gc<T>() + 1)] = qf[s][1];
                    a.T2[o.at(kT2<T>(), kT2gc<T>() + 2)] = qf[s][2];
                }
        }
        if (!PIPE || en < 0) return;
        e0 = en;
        en = e2;
        nbm = cnm;
        nbp = cnp;
        cnm = c2m;
        cnp = c2p;
        c0 = c1;
        wn[0][5] = w1[0][5];
        wn[1][5] = w1[1][5];
    }
}

// ------------------------------------------------------------ k_lift2
// Tile of k_lift2: its own, since its workgroups are bound by the registers
// and the LDS of the node phases and by the rounds of the face phases, not by
// what the streaming kernels of the stage like.  One element per workgroup at
// N = 4 and 5, two at N = 3, three at N = 2 and as many threads as the face
// points need, in whole waves, so that the face phases take one round: the
// second round of a few face points cost a workgroup the latency of a whole one
// (N = 3 on 48x48x24: 387 us with two rounds, 291 with one; with one element
// 325, with four 378; N = 5 on 32^3 with two elements 604 against 460).
// FP64 instances are bound by memory latency at 4 waves per SIMD, LDS and
// vector unit each busy for 60 % of the time (32^3 N = 5: 465 us, 3.7 TB/s of
// algorithmic bytes); FP32 ones by instruction issue, 88 % busy (274 us).
template <int P> using Lift2Group = Group<P, StageTile<P>::kLift2, true>;

// Registers: affine FP64 instances fit in the 128 of 4 waves per SIMD and affine
// FP32 ones in the 80 of 6 (the walls' would take 96: 48 against 52 us on a
// sliding 51x25x13 mesh at N = 3; at 7 waves the spills cost more, 55 us).
// Curved ones take what they need.
template <int P, typename T, bool CV> constexpr int lift2_waves() { return CV ? 1 : (sizeof(T) == 8 ? 4 : 6); }

// WALL: the mesh (or a batch's) has wall faces; without them the wall pass and
// its registers are left out.  DIAG: every element is a box along the axes, Ja^d
// a positive multiple of e_d (the other components are exactly zero, and leaving
// them out changes no finite result) and the normal of face 2d+1 e_d: three
// products for a gradient instead of twelve, and no normal components of the
// stress to form.
template <int P, typename T, bool BATCH, bool CV, bool WALL, bool DIAG>
__global__ __launch_bounds__(Lift2Group<P>::NT, (lift2_waves<P, T, CV>())) void k_lift2(Launch<T> L, int tiles)
{
    using W = Lift2Group<P>;
    using G = typename W::G;
    constexpr int NT = W::NT;
    Inst<T> a;
    int e0;
    if (!instance_of<P, W, BATCH>(L, a, e0, tiles)) return;
    const int E = a.mesh.E;
    // LDS, in rows of pairs of NV nodes: the primitives (rho, u), (v, w) and c
    // and their BR1 face values while they are lifted; then
    //   rows 0..2  (tau . n_d)_0, (tau . n_d)_1 of direction d
    //   rows 3..5  (tau . n_d)_2, div u
    //   rows 6..8  T, grad c . n_d; then grad T . n_d, lap c
    // so that a face task reads three pairs; and the contravariant fluxes of
    // the volume integral over rows 6..8 (directions 0 and 2) and rows 0, 3, 1
    // (direction 1, whose values every thread has read by then).
    // Curved elements, whose normal varies along a face: rows 0..4 grad u,
    // rows 5..7 T, contravariant grad c_d, then 5, 6 grad T, lap c; fluxes
    // over rows 5..7 and rows 8..10.
    constexpr int kRows = CV ? 11 : 9, kT = CV ? 5 : 6;
    constexpr int kLift = 5 * G::NV + 5 * G::NF;
    constexpr int kX0 = (kLift + 1) / 2 + 2 * G::NV;                  // pairs, with the state beside them
    constexpr int kX = kRows * G::NV > kX0 ? kRows * G::NV : kX0;
    // curved elements: the metrics of every node and n dS of every face point
    constexpr int NJ = CV ? 3 : 1, NQ = CV ? 3 : 1, NJV = CV ? G::NV : 1, NQF = CV ? G::NF : 1;
    __shared__ V2<T> sX[kX];
    __shared__ V2<T> sTF[G::NF];   // T*, (grad c)* . n dS
    __shared__ V2<T> sJ[NJ][NJV];
    __shared__ T sJz[NJ][NJV];
    __shared__ T sN[NQ][NQF];
    __shared__ BasisS<P, T> B;
    V2<T>(*sR)[G::NV] = reinterpret_cast<V2<T>(*)[G::NV]>(sX);
    V2<T> *sSa = sX + 2 * G::NV, *sSb = sSa + G::NF;
    T *sWc = reinterpret_cast<T *>(sSb + G::NF), *sSc = sWc + G::NV;
    V2<T> *sM = sX + kX - 2 * G::NV;  // (m_x, m_y), (m_z, rho e)
    const Five<T> fw{sX, sX + G::NV, sWc}, fs{sSa, sSb, sSc};
    B.load(L.bas);
    const int t = threadIdx.x;
    const NodeTask<G> nt(t);
    const int le = nt.le, nd = nt.nd, tq = nt.q;
    const int e = e0 + le;
    const bool act = nt.in && e < E;
    const size_t g = (size_t)e0 * G::n3 + tq;
    const uint32_t g32 = (uint32_t)g;
    const size_t NF = (size_t)E * 6 * G::n2;
    const T *TU = a.TU + (size_t)L.tb * 6 * NF;

    // face work: one face point per thread, as loops of at most one turn (as
    // plain conditions the compiler keeps what the phases share in registers and
    // spills 5 to 8 of them in the FP32 instances with walls).  The traces are
    // loaded before the node loads: both sides' conserved state (the own side's
    // is the prolongation of the state, written by the previous stage), (grad
    // c) . n and |grad c|^2.  The convective part of the flux and the face values
    // that its viscous part needs stay in registers until that part is known.
    static_assert(G::NF <= NT, "one face point per thread");
    // FP64: the face point's normal and surface element are loaded with its
    // traces too (in FP32 the registers would cost a wave per SIMD)
    constexpr bool kOne = sizeof(T) == 8;
    const bool parts = sizeof(T) == 4 && !BATCH && L.mode == kUtParts;
    struct Tr {
        int nb;
        T own[3], oth[3], wn[6], uo[6];
        T n[3], dS;
    };
    auto load_tr = [&](int task, Tr &r) {
        const FaceTask<P> ft(task);
        const int el = e0 + ft.le;
        r.nb = -1;
        if (el >= E) return;
        const FaceIx<G::n2> o((size_t)el * 6 + ft.f, ft.fp);
#pragma unroll
        for (int k = 0; k < kT2gc<T>(); ++k) r.own[k] = a.T2[o.at(kT2<T>(), k)];
#pragma unroll
        for (int v = 0; v < 6; ++v) r.uo[v] = TU[o.at(6, v)];
        r.nb = gld(a.mesh.nbr, el * 6 + ft.f);
        if constexpr (kOne) face_normal<P, T, CV>(a.mesh, (size_t)el * 6 + ft.f, ft.fp, r.n, r.dS);
        if (!WALL || r.nb >= 0) {
            const FaceIx<G::n2> on(nbr_face<P>(r.nb), nbr_point<P>(r.nb, ft.fp));
#pragma unroll
            for (int k = 0; k < kT2gc<T>(); ++k) r.oth[k] = a.T2[on.at(kT2<T>(), k)];
#pragma unroll
            for (int v = 0; v < 6; ++v) r.wn[v] = TU[on.at(6, v)];
        }
    };
    // face temperature from a conserved trace and |grad c|^2 (FP32: value and
    // rounding error; always FP64 arithmetic)
    auto face_T = [&](const T u[6], const T q[3]) {
        double g2 = (double)q[1];
        if constexpr (sizeof(T) == 4) g2 += (double)q[2];
        return temperature_g2<fast_fp64<T>()>(a.ph, (double)u[0], (double)u[1], (double)u[2], (double)u[3],
                                              (double)u[4], (double)u[5], g2);
    };
    // pressure (p_alpha for model 2) and sound speed of the convective flux
    auto face_eos = [&](T rho, double Tf, T &p, T &cw) {
        double pd, cs2;
        eos<fast_fp64<T>()>(a.ph, (double)rho, Tf, pd, cs2);
        p = T(pd + a.ph.ap_2 * (double)rho * (double)rho);
        cw = sqrt_to<T>(fabs(cs2 + a.ph.ap * (double)rho));
    };
    Tr tr;
    if (t < G::NF) load_tr(t, tr);
    // the state waits in LDS (rho and c among the primitives) while the face
    // values are formed, where its registers are needed
    T un[6];
    T iJn = T(0);
    if (act) {
        T w[5];
#pragma unroll
        for (int v = 0; v < 6; ++v) un[v] = gld(a.U + (v) * a.NN, g32);
        primitives<T, true>(un, w);
        sM[tq] = V2<T>{un[1], un[2]};
        sM[G::NV + tq] = V2<T>{un[3], un[4]};
        sR[0][tq] = V2<T>{w[0], w[1]};
        sR[1][tq] = V2<T>{w[2], w[3]};
        sWc[tq] = w[4];
        if constexpr (CV) iJn = stage_node_metrics<T, NJV>(a.mesh, a.NN, g, tq, sJ, sJz);
    }
    // what the flux pass needs of this face point
    T Kc[6], fu[3], fc = T(0), frc = T(0), fgn = T(0), fdS = T(0);
    bool fwall = true;
    // face values: BR1 w* of the primitives; T* and (grad c)* . n dS of the
    // second lifting; and on interior faces the convective part of the flux:
    // the own side's flux with half of the Rusanov dissipation, F^C(u) . n +
    // lam/2 (u - u_nbr), so that half the difference of the two sides' values
    // (each with its own normal) is the central flux plus the dissipation
    // (model 2: the HLLC flux, of which half the difference is itself)
    for (int task = t; task < G::NF; task += NT) {
        const FaceTask<P> ft(task);
        const int el = e0 + ft.le, f = ft.f;
        if (el >= E) break;
        T n[3], dS;
        if constexpr (kOne) {
            n[0] = tr.n[0];
            n[1] = tr.n[1];
            n[2] = tr.n[2];
            dS = tr.dS;
        } else {
            face_normal<P, T, CV>(a.mesh, (size_t)el * 6 + f, ft.fp, n, dS);
        }
        const int slot = ft.le * 6 * G::n2 + f * G::n2 + ft.fp;
        const T *uf = tr.uo;
        T w[5];
        primitives<T, true>(uf, w);
        const double To = face_T(uf, tr.own);
        T Ts, Fs;
        if (!WALL || tr.nb >= 0) {
            T v5[5];
            primitives<T, true>(tr.wn, v5);
            T po, co, pn, cn;
            face_eos(uf[0], To, po, co);
            __builtin_amdgcn_sched_barrier(0);  // one side after the other: registers
            const double Tn = face_T(tr.wn, tr.oth);
            face_eos(tr.wn[0], Tn, pn, cn);
            __builtin_amdgcn_sched_barrier(0);
            T K[6];
            if (a.ph.model == 2) {
                hllc(uf, po, co, tr.wn, pn, cn, n, K);
                if (parts) {
                    const FaceIx<G::n2> o((size_t)el * 6 + f, ft.fp);
#pragma unroll
                    for (int v = 1; v < 5; ++v) {
                        a.TF[o.at(6, v)] = K[v];
                        K[v] = T(0);
                    }
                }
            } else {
                const T mn = uf[1] * n[0] + uf[2] * n[1] + uf[3] * n[2];
                const T mo = tr.wn[1] * n[0] + tr.wn[2] * n[1] + tr.wn[3] * n[2];
                const T vn = mn * recip_to(uf[0]);
                const T lo = fabs(vn) + co, ln = fabs(mo * recip_to(tr.wn[0])) + cn;
                const T hl = T(0.5) * (lo > ln ? lo : ln);
                K[0] = mn + hl * (uf[0] - tr.wn[0]);
                K[1] = uf[1] * vn + po * n[0] + hl * (uf[1] - tr.wn[1]);
                K[2] = uf[2] * vn + po * n[1] + hl * (uf[2] - tr.wn[2]);
                K[3] = uf[3] * vn + po * n[2] + hl * (uf[3] - tr.wn[3]);
                K[4] = (uf[4] + po) * vn + hl * (uf[4] - tr.wn[4]);
                K[5] = uf[5] * vn + hl * (uf[5] - tr.wn[5]);
            }
#pragma unroll
            for (int v = 0; v < 6; ++v) Kc[v] = K[v];
            fu[0] = w[1];
            fu[1] = w[2];
            fu[2] = w[3];
            fc = uf[5];
            frc = uf[0] - uf[5];
            fgn = tr.own[0];
            fdS = dS;
            fwall = false;
#pragma unroll
            for (int k = 0; k < 5; ++k) w[k] = T(0.5) * (w[k] + v5[k]);
            Ts = T(0.5) * (T(To) + T(Tn));
            Fs = T(0.5) * (tr.own[0] - tr.oth[0]) * dS;
        } else {
            wall_primitives(a.mesh, el, f, n, w);
            const BcDev &bc = a.mesh.bcs[a.mesh.bcid[el * 6 + f] - 1];
            Ts = bc.iso ? T(bc.twall) : T(To);
            if (bc.kind != 2) {
                // static part of the contact-angle flux (a varying wall
                // temperature is applied in the pass below; the dynamic part,
                // gamma_1 div u, once grad u is lifted)
                const T c = uf[5];
                Fs = T(bc.gcoef) * (c - T(bc.rl)) * (c - T(bc.rv)) * dS;
            } else {
                Fs = T(0);
            }
        }
        sSa[slot] = V2<T>{w[0], w[1]};
        sSb[slot] = V2<T>{w[2], w[3]};
        sSc[slot] = w[4];
        sTF[slot] = V2<T>{Ts, Fs};
        if constexpr (CV) {
#pragma unroll
            for (int m = 0; m < 3; ++m) sN[m][slot] = n[m] * dS;
        }
    }
    if (WALL && a.mesh.var) {
        // walls whose temperature varies along them: T* and the static
        // contact-angle flux at the local wall temperature, through the table
        // (each thread rewrites only the face point it wrote above)
        double tb = 0.0;  // a batch instance's stage time
        if (BATCH && a.clk) tb = stage_time(a.t0, *a.clk, a.dt, L.cs);
        for (int task = t; task < G::NF; task += NT) {
            const FaceTask<P> ft(task);
            const int el = e0 + ft.le, f = ft.f;
            if (el >= E) continue;
            if (gld(a.mesh.nbr, el * 6 + f) >= 0) continue;  // interior: no wall-table entry
            const BcDev &bc = a.mesh.bcs[a.mesh.bcid[el * 6 + f] - 1];
            if (!bc.var) continue;
            const WallPt wp = wall_point<P>(a.mesh, L.bas, bc, el, f, ft.fp, BATCH ? tb : L.t);
            const int slot = ft.le * 6 * G::n2 + f * G::n2 + ft.fp;
            const FaceIx<G::n2> o((size_t)el * 6 + f, ft.fp);
            if (bc.iso) sTF[slot].x = T(wp.Tw);
            else a.TF[o.at(6, 0)] = T(1.0 / wp.Tw);  // for the heat-transfer flux below, which then overwrites it
            const T c = TU[o.at(6, 5)];
            sTF[slot].y = T(wp.gcoef) * (c - T(wp.rl)) * (c - T(wp.rv)) * face_dS<P, T, CV>(a.mesh, (size_t)el * 6 + f, ft.fp);
        }
    }
    __syncthreads();
    // lifted gradients, nodal temperature and pressure, and the source
    const int i = nd % P, j = (nd / P) % P, k = nd / (P * P);
    const int base = le * G::n3, fbase = le * 6 * G::n2;
    T gc[3] = {T(0), T(0), T(0)}, S[6];
    T iJ = T(0), div = T(0), p = T(0), irn = T(0);
    double Tn = 0.0;
    T gu[3][3];
    if (act) {
        T grho[3];
        if constexpr (CV) {
            T q[5][3];
            lifted_grads_curved<P, 5, G::NV, G::NF>([&](int n, T v[5]) { fw.at(n, v); }, [&](int n, T v[5]) { fs.at(n, v); },
                                                    sJ, sJz, sN, base, fbase, i, j, k, B, iJn, q);
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                grho[m] = q[0][m];
                gu[0][m] = q[1][m];
                gu[1][m] = q[2][m];
                gu[2][m] = q[3][m];
                gc[m] = q[4][m];
            }
            iJ = iJn;
        } else {
            T gd[5][3], Ja[9];
            lifted_grads<P, T>(fw, fs, base, fbase, i, j, k, B, gd);
            element_metrics<G::kUni>(a.mesh, e, Ja, iJ);
            to_physical<DIAG>(Ja, iJ, gd[0], grho);
#pragma unroll
            for (int m = 0; m < 3; ++m) to_physical<DIAG>(Ja, iJ, gd[1 + m], gu[m]);
            to_physical<DIAG>(Ja, iJ, gd[4], gc);
        }
        {
            const V2<T> m01 = sM[tq], m2e = sM[G::NV + tq];
            un[0] = sR[0][tq].x;
            un[1] = m01.x;
            un[2] = m01.y;
            un[3] = m2e.x;
            un[4] = m2e.y;
            un[5] = sWc[tq];
        }
        Tn = temperature<fast_fp64<T>()>(a.ph, (double)un[0], (double)un[1], (double)un[2], (double)un[3], (double)un[4],
                                         (double)un[5], (double)gc[0], (double)gc[1], (double)gc[2]);
        div = gu[0][0] + gu[1][1] + gu[2][2];
        double pd, cs2;
        eos<fast_fp64<T>()>(a.ph, (double)un[0], Tn, pd, cs2);
        p = T(pd + a.ph.ap_2 * (double)un[0] * (double)un[0]);  // p_alpha for model 2
        irn = recip_to(un[0]);
        const T u[3] = {un[1] * irn, un[2] * irn, un[3] * irn};
        source(a.pt, a.ph.model == 2, un[0], un[5], u, grho, gu, gc, S);
    }
    __syncthreads();
    if (act) {
        if constexpr (CV) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sR[r][tq] = V2<T>{gu[2 * r / 3][2 * r % 3], gu[(2 * r + 1) / 3][(2 * r + 1) % 3]};
            sR[4][tq].x = gu[2][2];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const V2<T> jj = sJ[d][tq];
                sR[kT + d][tq] = V2<T>{T(Tn), jj.x * gc[0] + jj.y * gc[1] + sJz[d][tq] * gc[2]};
            }
        } else {
            // per direction d, at the nodes: tau . n_d with n_d the outward
            // normal of face 2d+1 (face 2d has exactly -n_d on these affine
            // elements); its face values are the prolongations of these nodal
            // values (n_d is constant on the face), so a face task prolongs
            // 6 fields instead of 13
            // (gc: the components along the n_d from here on.  They and the fluxes
            // below are scaled by the surface element after they are summed: scaled
            // node by node in FP32, each node's rounding is differentiated)
            const T mu = a.pt.mu, td = T(2.0 / 3.0) * div, g0 = gc[0], g1 = gc[1], g2 = gc[2];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int fr = (2 * d + 1) * 4;
                T tn[3];
                if constexpr (DIAG) {  // n_d is the unit vector of axis d
#pragma unroll
                    for (int m = 0; m < 3; ++m) tn[m] = mu * ((gu[m][d] + gu[d][m]) - (m == d ? td : T(0)));
                } else {
                    const T n0 = em_at<G::kUni, T>(a.mesh, e, fr), n1 = em_at<G::kUni, T>(a.mesh, e, fr + 1),
                            n2 = em_at<G::kUni, T>(a.mesh, e, fr + 2);
                    gc[d] = n0 * g0 + n1 * g1 + n2 * g2;
#pragma unroll
                    for (int m = 0; m < 3; ++m)
                        tn[m] = mu * ((gu[m][0] + gu[0][m]) * n0 + (gu[m][1] + gu[1][m]) * n1 +
                                      (gu[m][2] + gu[2][m]) * n2 - td * (m == 0 ? n0 : (m == 1 ? n1 : n2)));
                }
                sR[d][tq] = V2<T>{tn[0], tn[1]};
                sR[3 + d][tq] = V2<T>{tn[2], div};
                sR[kT + d][tq] = V2<T>{T(Tn), gc[d]};
            }
        }
    }
    __syncthreads();
    if (WALL && a.mesh.dyn) {
        // Navier-slip walls with gamma_1 != 0: the contact-angle flux gains
        // (gamma_1/gamma) div u, div u the trace of the lifted velocity gradient
        for (int task = t; task < G::NF; task += NT) {
            const FaceTask<P> ft(task);
            const int el = e0 + ft.le, f = ft.f;
            if (el >= E) continue;
            if (gld(a.mesh.nbr, el * 6 + f) >= 0) continue;  // interior: no wall-table entry
            const BcDev &bc = a.mesh.bcs[a.mesh.bcid[el * 6 + f] - 1];
            if (bc.kind != 3 || bc.g1 == 0.0) continue;
            const T *Lf = B.Lf + (f & 1) * B.PS;
            const int lo = ft.le * G::n3 + ft.off, ls = ft.str;
            T d0 = T(0);
#pragma unroll
            for (int l = 0; l < P; ++l) {
                const int q = lo + l * ls;
                d0 += Lf[l] * (CV ? sR[0][q].x + sR[2][q].x + sR[4][q].x : sR[3][q].y);
            }
            const T dS = face_dS<P, T, CV>(a.mesh, (size_t)el * 6 + f, ft.fp);
            sTF[ft.le * 6 * G::n2 + f * G::n2 + ft.fp].y += T(bc.g1_gam) * d0 * dS;
        }
        __syncthreads();
    }
    // grad T (BR1 with T*) and lap c (divergence lifting of grad c from its
    // components along the normals; curved: its contravariant components)
    T gT[3] = {T(0), T(0), T(0)}, lap = T(0);
    if (act) {
        const int idx[3] = {i, j, k};
        const int fpd[3] = {j + P * k, i + P * k, i + P * j};
        T gd[3], dl = T(0);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int p = d == 0 ? j : i, q = d == 2 ? j : k;
            T accT = T(0), ad = T(0), D[P];
            B.row(B.Dh + idx[d] * B.PS, D);
#pragma unroll
            for (int l = 0; l < P; ++l) {
                const V2<T> v = sR[kT + d][base + line_node<P>(d, l, p, q)];
                if constexpr (!CV) accT += D[l] * v.x;
                ad += D[l] * v.y;
            }
            const V2<T> lh = B.Lh[idx[d]], vp = sTF[fbase + (2 * d + 1) * G::n2 + fpd[d]], vm = sTF[fbase + (2 * d) * G::n2 + fpd[d]];
            if constexpr (!CV) gd[d] = accT + (lh.y * vp.x - lh.x * vm.x);
            if constexpr (!CV) ad = em_at<G::kUni, T>(a.mesh, e, (2 * d + 1) * 4 + 3) * ad;
            dl += ad + lh.y * vp.y + lh.x * vm.y;
        }
        if constexpr (CV) {
            T qT[1][3];
            lifted_grads_curved<P, 1, G::NV, G::NF>([&](int n, T v[1]) { v[0] = sR[kT][n].x; }, [&](int n, T v[1]) { v[0] = sTF[n].x; },
                                                    sJ, sJz, sN, base, fbase, i, j, k, B, iJ, qT);
#pragma unroll
            for (int m = 0; m < 3; ++m) gT[m] = qT[0][m];
        } else {
            T Ja[9], iJ2;
            element_metrics<G::kUni>(a.mesh, e, Ja, iJ2);
            to_physical<DIAG>(Ja, iJ, gd, gT);
        }
        lap = iJ * dl;
        if (L.mode == kG2) {  // the second lifting's output alone
            gst(a.G2 + (0) * a.NN, g32, T(gT[0]));
            gst(a.G2 + (1) * a.NN, g32, T(gT[1]));
            gst(a.G2 + (2) * a.NN, g32, T(gT[2]));
            gst(a.G2 + (3) * a.NN, g32, T(lap));
        }
    }
    if (L.mode == kG2) return;
    T zc;
    __syncthreads();
    if (act) {
        // j_e = k grad T + (gamma zeta - gamma c div u) grad c
        zc = a.pt.gam * (a.pt.beta * (a.pt.gam * lap + a.pt.alpha * (un[0] - un[5])) - un[5] * div);
        if constexpr (CV) {
            sR[kT][tq] = V2<T>{gT[0], gT[1]};
            sR[kT + 1][tq] = V2<T>{gT[2], lap};
        } else {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int fr = (2 * d + 1) * 4;
                T gn = gT[d];
                if constexpr (!DIAG)
                    gn = gT[0] * em_at<G::kUni, T>(a.mesh, e, fr) + gT[1] * em_at<G::kUni, T>(a.mesh, e, fr + 1) +
                         gT[2] * em_at<G::kUni, T>(a.mesh, e, fr + 2);
                sR[kT + d][tq] = V2<T>{gn, lap};
            }
        }
    }
    __syncthreads();
    // own-face flux traces, one face point per task: on interior faces half
    // of the convective part from above and of -F^V . n, times dS, so that the
    // numerical flux is the difference of the two sides' traces; on walls (a
    // pass of its own, whose values would cost the common one registers) the
    // complete wall flux times dS
    struct Pro {  // prolongation of one row of sX to a face point
        const T *Lr;
        int lo, ls;
        __device__ __forceinline__ V2<T> operator()(const V2<T> *fld) const
        {
            T w[P], x = T(0), y = T(0);
            BasisS<P, T>::row(Lr, w);
#pragma unroll
            for (int l = 0; l < P; ++l) {
                const V2<T> v = fld[lo + l * ls];
                x += w[l] * v.x;
                y += w[l] * v.y;
            }
            T r[2] = {x, y};
            bound(r, 2);
            return V2<T>{r[0], r[1]};
        }
    };
    // the face values of tau n (traction mu ((grad u + grad u^T) n - 2/3 div u
    // n)), div u, grad T . n and lap c.  Affine elements: from the nodal
    // normal components of direction f/2, with the face's sign; curved: from
    // the prolonged gradients and the normal of this face point.
    auto viscous = [&](const Pro &pro, int f, const T n[3], T tn[3], T &dv, T &gTn, T &lapf) {
        if constexpr (CV) {
            T gf[10];
#pragma unroll
            for (int r = 0; r < 5; ++r) {
                const V2<T> v = pro(sR[r]);
                gf[2 * r] = v.x;  // gf[3 j + i] = d u_j / d x_i
                gf[2 * r + 1] = v.y;
            }
            dv = gf[0] + gf[4] + gf[8];
            const T td = T(2.0 / 3.0) * dv, mu = a.pt.mu;
            tn[0] = mu * ((gf[0] + gf[0]) * n[0] + (gf[1] + gf[3]) * n[1] + (gf[2] + gf[6]) * n[2] - td * n[0]);
            tn[1] = mu * ((gf[3] + gf[1]) * n[0] + (gf[4] + gf[4]) * n[1] + (gf[5] + gf[7]) * n[2] - td * n[1]);
            tn[2] = mu * ((gf[6] + gf[2]) * n[0] + (gf[7] + gf[5]) * n[1] + (gf[8] + gf[8]) * n[2] - td * n[2]);
            const V2<T> x = pro(sR[kT]), y = pro(sR[kT + 1]);
            gTn = x.x * n[0] + x.y * n[1] + y.x * n[2];
            lapf = y.y;
        } else {
            const T sgn = (f & 1) ? T(1) : T(-1);
            const int d = f >> 1;
            const V2<T> x = pro(sR[d]), y = pro(sR[3 + d]), z = pro(sR[kT + d]);
            tn[0] = sgn * x.x;
            tn[1] = sgn * x.y;
            tn[2] = sgn * y.x;
            dv = y.y;
            gTn = sgn * z.x;
            lapf = z.y;
        }
    };
    for (int task = t; task < G::NF; task += NT) {
        const FaceTask<P> ft(task);
        const int el = e0 + ft.le, f = ft.f;
        if (el >= E) break;
        if (WALL && fwall) continue;
        const Pro pro{B.Lf + (f & 1) * B.PS, ft.le * G::n3 + ft.off, ft.str};
        const FaceIx<G::n2> o((size_t)el * 6 + f, ft.fp);
        T K[6], dS = fdS, n[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int v = 0; v < 6; ++v) K[v] = Kc[v];
        if constexpr (CV) face_normal<P, T, CV>(a.mesh, (size_t)el * 6 + f, ft.fp, n, dS);
        // scheduling barriers keep each field group's LDS loads next to the
        // arithmetic that consumes them (otherwise all of them are hoisted
        // and the register demand limits occupancy)
        __builtin_amdgcn_sched_barrier(0);
        T tn[3], dv, gTn, lapc;
        viscous(pro, f, n, tn, dv, gTn, lapc);
        K[1] -= tn[0];
        K[2] -= tn[1];
        K[3] -= tn[2];
        K[4] -= tn[0] * fu[0] + tn[1] * fu[1] + tn[2] * fu[2];
        K[4] -= a.pt.kappa * gTn;
        // order-parameter terms of j_e and F^V_c
        const T zeta = a.pt.beta * (a.pt.gam * lapc + a.pt.alpha * frc);
        K[4] -= -a.pt.gam * fc * fgn * dv + a.pt.gam * fgn * zeta;
        K[5] -= a.pt.gb * fgn;
        dS *= T(0.5);
        T *TV = a.TU + 6 * NF;
        if (parts) {
#pragma unroll
            for (int v = 1; v < 5; ++v) TV[o.at(4, v - 1)] = K[v];
            a.TF[o.at(6, 0)] = K[0] * dS;
            a.TF[o.at(6, 5)] = K[5] * dS;
        } else {
#pragma unroll
            for (int v = 0; v < 6; ++v) a.TF[o.at(6, v)] = K[v] * dS;
        }
    }
    for (int task = t; WALL && a.mesh.wall && task < G::NF; task += NT) {
        const FaceTask<P> ft(task);
        const int el = e0 + ft.le, f = ft.f;
        if (el >= E) break;
        if (gld(a.mesh.nbr, el * 6 + f) >= 0) continue;
        const BcDev &bc = a.mesh.bcs[a.mesh.bcid[el * 6 + f] - 1];
        const int kind = bc.kind;
        const Pro pro{B.Lf + (f & 1) * B.PS, ft.le * G::n3 + ft.off, ft.str};
        const FaceIx<G::n2> o((size_t)el * 6 + f, ft.fp);
        T K[6], n[3], dS;
        // the prolongations before the traces are loaded, and before the normal
        // where they do without it: in the other order the pass needs more
        // registers than the kernel has, and spills
        if constexpr (CV) face_normal<P, T, CV>(a.mesh, (size_t)el * 6 + f, ft.fp, n, dS);
        T tn[3], dv, gTn, lapc;
        viscous(pro, f, n, tn, dv, gTn, lapc);
        bound(tn, 3);
        if constexpr (!CV) face_normal<P, T, CV>(a.mesh, (size_t)el * 6 + f, ft.fp, n, dS);
        T u6[6], q[3];
#pragma unroll
        for (int v = 0; v < 6; ++v) u6[v] = TU[o.at(6, v)];
#pragma unroll
        for (int k2 = 0; k2 < kT2gc<T>(); ++k2) q[k2] = a.T2[o.at(kT2<T>(), k2)];
        const double Tf = face_T(u6, q);
        T p, cw;
        face_eos(u6[0], Tf, p, cw);
        const T rho = u6[0], c = u6[5], ir = T(1) / rho;
        const T u0 = u6[1] * ir, u1 = u6[2] * ir, u2 = u6[3] * ir;
        const T mn = u6[1] * n[0] + u6[2] * n[1] + u6[3] * n[2], vn = mn * ir, lam = fabs(vn) + cw;
        const T w0 = T(bc.uw[0]), w1 = T(bc.uw[1]), w2 = T(bc.uw[2]);
        K[0] = K[4] = K[5] = T(0);
        if (kind == 1) {
            // ghost velocity 2 u_w - u (same rho, c, T); energy: -(u.n + lam)/2
            // times the ghost's extra kinetic energy 2 rho (|u_w|^2 - u_w . u);
            // the traction, and its work at the wall velocity
            const T r0 = u6[1] - rho * w0, r1 = u6[2] - rho * w1, r2 = u6[3] - rho * w2;
            K[1] = r0 * vn + p * n[0] + lam * r0 - tn[0];
            K[2] = r1 * vn + p * n[1] + lam * r1 - tn[1];
            K[3] = r2 * vn + p * n[2] + lam * r2 - tn[2];
            K[4] = -(vn + lam) * rho * (w0 * (w0 - u0) + w1 * (w1 - u1) + w2 * (w2 - u2));
            K[4] -= tn[0] * w0 + tn[1] * w1 + tn[2] * w2;
        } else {
            // mirrored normal velocity only; normal part of the traction
            const T s_ = mn * vn + p + lam * mn - (tn[0] * n[0] + tn[1] * n[1] + tn[2] * n[2]);
            K[1] = s_ * n[0];
            K[2] = s_ * n[1];
            K[3] = s_ * n[2];
            if (kind == 3) {
                // Navier slip: tangential traction gamma_1 div u grad_G c -
                // gamma_2 (u_t - u_w,t), and its work on u_t
                const T gc0 = a.T2[o.at(kT2<T>(), kT2gc<T>())], gc1 = a.T2[o.at(kT2<T>(), kT2gc<T>() + 1)],
                        gc2 = a.T2[o.at(kT2<T>(), kT2gc<T>() + 2)];
                const T gcn = gc0 * n[0] + gc1 * n[1] + gc2 * n[2];
                const T wn = w0 * n[0] + w1 * n[1] + w2 * n[2];
                const T a1 = T(bc.g1) * dv, a2 = T(bc.g2);
                const T ut0 = u0 - vn * n[0], ut1 = u1 - vn * n[1], ut2 = u2 - vn * n[2];
                const T t0 = a1 * (gc0 - gcn * n[0]) - a2 * (ut0 - (w0 - wn * n[0]));
                const T t1 = a1 * (gc1 - gcn * n[1]) - a2 * (ut1 - (w1 - wn * n[1]));
                const T t2 = a1 * (gc2 - gcn * n[2]) - a2 * (ut2 - (w2 - wn * n[2]));
                K[1] -= t0;
                K[2] -= t1;
                K[3] -= t2;
                K[4] -= t0 * ut0 + t1 * ut1 + t2 * ut2;
            }
        }
        if (kind != 2) {
            if (bc.iso) {
                K[4] -= a.pt.kappa * gTn;
            } else {  // heat transfer, eq. bc_energy_alpha
                const double itw = bc.var ? (double)a.TF[o.at(6, 0)] : bc.inv_tw;
                K[4] -= T(-bc.g3 * (itw - 1.0 / Tf));
            }
            // contact-angle flux g (with gamma_1 div u on Navier-slip
            // walls), as the second lifting used it: sTF holds g dS; and
            // the wall value zeta_c = -gamma_1 gamma_4 div u
            const T gw = sTF[ft.le * 6 * G::n2 + f * G::n2 + ft.fp].y / dS;
            const T zeta = -T(bc.g1 * bc.g4) * dv;
            K[4] -= -a.pt.gam * c * gw * dv + a.pt.gam * gw * zeta;
            K[5] -= a.pt.gb * gw;
        }
#pragma unroll
        for (int v = 0; v < 6; ++v) a.TF[o.at(6, v)] = K[v] * dS;
    }
    // the RK register of this node, requested now so that the loads complete
    // during the volume integral
    T Rn[6];
    if (L.mode == kRk && act && !L.first) {
#pragma unroll
        for (int v = 0; v < 6; ++v) Rn[v] = gld(a.R + (v) * a.NN, g32);
    }
    // volume integral sum_d Dhat_d (Ja^d . F): the contravariant fluxes of
    // direction d+1 are written while direction d is read, one barrier per
    // direction
    T acc[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
    // row q of the fluxes of direction 1 (odd) or 0 and 2
    auto frow = [&](bool odd, int q) { return odd ? (CV ? 8 + q : (q == 0 ? 0 : (q == 1 ? 3 : 1))) : kT + q; };
    // (F^C - F^V), F^V = (0, tau, tau u + j_e, gamma beta grad c): curved elements
    // form the tensor, whose rows Ja^d takes at each node; affine ones the flux
    // along n_d, times dS_d
    T Fx[CV ? 6 : 1][3];
    if constexpr (CV) {
        if (act) {
            T gg[10];
#pragma unroll
            for (int r = 0; r < 5; ++r) {
                const V2<T> v = sR[r][tq];
                gg[2 * r] = v.x;
                gg[2 * r + 1] = v.y;
            }
            const T u[3] = {un[1] * irn, un[2] * irn, un[3] * irn};
            const T mu = a.pt.mu, td = T(2.0 / 3.0) * div;
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                T tau[3];
#pragma unroll
                for (int m = 0; m < 3; ++m) tau[m] = mu * (gg[3 * m + r] + gg[3 * r + m] - (m == r ? td : T(0)));
                Fx[0][r] = un[1 + r];
#pragma unroll
                for (int m = 0; m < 3; ++m) Fx[1 + m][r] = un[1 + m] * u[r] + (m == r ? p : T(0)) - tau[m];
                Fx[4][r] = (un[4] + p) * u[r] - (tau[0] * u[0] + tau[1] * u[1] + tau[2] * u[2]) -
                           (a.pt.kappa * gT[r] + zc * gc[r]);
                Fx[5][r] = un[5] * u[r] - a.pt.gb * gc[r];
            }
        }
    }
    auto put_flux = [&](int d) {
        T f[6];
        if constexpr (CV) {
            const V2<T> jj = sJ[d][tq];
            const T jz = sJz[d][tq];
#pragma unroll
            for (int v = 0; v < 6; ++v) f[v] = jj.x * Fx[v][0] + jj.y * Fx[v][1] + jz * Fx[v][2];
        } else {
            const int fr = (2 * d + 1) * 4;
            const T gn = d == 0 ? gc[0] : (d == 1 ? gc[1] : gc[2]);
            T n[3], mn, qn;
            if constexpr (DIAG) {
                mn = un[1 + d];
                qn = gT[d];
            } else {
#pragma unroll
                for (int m = 0; m < 3; ++m) n[m] = em_at<G::kUni, T>(a.mesh, e, fr + m);
                mn = n[0] * un[1] + n[1] * un[2] + n[2] * un[3];
                qn = n[0] * gT[0] + n[1] * gT[1] + n[2] * gT[2];
            }
            const V2<T> x = sR[d][tq], y = sR[3 + d][tq];
            const T tn[3] = {x.x, x.y, y.x}, vn = mn * irn, dS = em_at<G::kUni, T>(a.mesh, e, fr + 3);
            f[0] = mn;
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                if constexpr (DIAG) f[1 + m] = un[1 + m] * vn + (m == d ? p : T(0)) - tn[m];
                else f[1 + m] = un[1 + m] * vn + p * n[m] - tn[m];
            }
            f[4] = (un[4] + p) * vn - (tn[0] * un[1] + tn[1] * un[2] + tn[2] * un[3]) * irn - (a.pt.kappa * qn + zc * gn);
            f[5] = un[5] * vn - a.pt.gb * gn;
#pragma unroll
            for (int v = 0; v < 6; ++v) f[v] *= dS;
        }
#pragma unroll
        for (int r = 0; r < 3; ++r) sR[frow(d & 1, r)][tq] = V2<T>{f[2 * r], f[2 * r + 1]};
    };
    __syncthreads();
    if (act) put_flux(0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        __syncthreads();
        if (act) {
            if (d < 2) put_flux(d + 1);
            __builtin_amdgcn_sched_barrier(0);
            const V2<T> *r0 = sR[frow(d & 1, 0)], *r1 = sR[frow(d & 1, 1)], *r2 = sR[frow(d & 1, 2)];
            const int id = d == 0 ? i : (d == 1 ? j : k);
            const int str = d == 0 ? 1 : (d == 1 ? P : P * P);
            const int lo = base + line_node<P>(d, 0, d == 0 ? j : i, d == 2 ? j : k);
            T D[P];
            B.row(B.Dh + id * B.PS, D);
#pragma unroll
            for (int l = 0; l < P; ++l) {
                const V2<T> x = r0[lo + l * str], y = r1[lo + l * str], z = r2[lo + l * str];
                acc[0] += D[l] * x.x;
                acc[1] += D[l] * x.y;
                acc[2] += D[l] * y.x;
                acc[3] += D[l] * y.y;
                acc[4] += D[l] * z.x;
                acc[5] += D[l] * z.y;
                if (l % 2 == 1) bound(acc, 6);
            }
        }
    }
    // the volume part W = S - iJ acc of U_t, into the register (RK) or the
    // output (U_t alone); k_update adds the surface part (kUtParts: the sum and
    // the source)
    if (!act) return;
    const T A = T(L.A), dt = T(a.dt);
#pragma unroll
    for (int v = 0; v < 6; ++v) {
        const T W = -acc[v] * iJ + S[v];
        if (parts && v % 5) {
            gst(a.Ut + (v) * a.NN, g32, acc[v]);
            gst(a.Q + (v) * a.NN, g32, S[v]);
        } else if (L.mode != kRk) gst(a.Ut + (v) * a.NN, g32, W);
        else gst(a.R + (v) * a.NN, g32, L.first ? dt * W : A * Rn[v] + dt * W);
    }
}

// ------------------------------------------------------------ k_update
// Bound by memory: 32^3 N = 5 in FP64 363 us, 5.4 TB/s of algorithmic bytes, where
// a large copy takes 5.07; with the gradients lifted again and the volume
// integral in this kernel it took 570 us.  The flux traces come as differences
// to take, so no normals, states or wave speeds are read, and the register
// already holds the volume part.  A thread per face point where the faces
// outnumber the nodes (N = 3, two elements: 513 -> 505 us on 50^3).
template <int P, bool FEW> using UpdateGroup = Group<P, FEW ? StageTile<P>::kFew : StageTile<P>::kUpdate, P == 4 || FEW>;


template <int P, typename T, bool BATCH, bool CV = false, bool NT = false, bool FEW = false>
__global__ __launch_bounds__((UpdateGroup<P, FEW>::NT)) void k_update(Launch<T> L, int tiles)
{
    using W = UpdateGroup<P, FEW>;
    using G = typename W::G;
    constexpr int BS = W::NT;
    Inst<T> a;
    int e0;
    if (!instance_of<P, W, BATCH>(L, a, e0, tiles)) return;
    __shared__ V2<T> sF[3][G::NV];     // new state
    __shared__ V2<T> sFs[3][G::NF];    // surface flux (F* . n) dS
    __shared__ BasisS<P, T> B;
    B.load(L.bas);
    const int E = a.mesh.E;
    const int t = threadIdx.x;
    const NodeTask<G> nt(t);
    const int le = nt.le, nd = nt.nd, tq = nt.q;
    const int e = e0 + le;
    const bool act = nt.in && e < E;
    const size_t g = (size_t)e0 * G::n3 + tq;
    const uint32_t g32 = (uint32_t)g;
    const size_t NF = (size_t)E * 6 * G::n2;

    // per face point: (F* . n) dS, the difference of the two sides' flux
    // traces (the wall flux on walls; kUtParts: the own side's convective flux
    // plus half the difference of the viscous ones, both still times dS)
    const bool parts = sizeof(T) == 4 && !BATCH && L.mode == kUtParts;
    const T *TV = a.TU + 6 * NF;
    for (int task = t; task < G::NF; task += BS) {
        const FaceTask<P> ft(task);
        const int el = e0 + ft.le;
        if (el >= E) continue;
        const FaceIx<G::n2> o((size_t)el * 6 + ft.f, ft.fp);
        const int nb = gld(a.mesh.nbr, el * 6 + ft.f);
        T K[6], Kn[6];
#pragma unroll
        for (int v = 0; v < 6; ++v) K[v] = a.TF[o.at(6, v)];
        if (nb >= 0) {
            const FaceIx<G::n2> on(nbr_face<P>(nb), nbr_point<P>(nb, ft.fp));
#pragma unroll
            for (int v = 0; v < 6; ++v) Kn[v] = parts && v % 5 ? TV[on.at(4, v - 1)] : a.TF[on.at(6, v)];
            if (parts) {
                const T dS = face_dS<P, T, CV>(a.mesh, (size_t)el * 6 + ft.f, ft.fp);
#pragma unroll
                for (int v = 1; v < 5; ++v) {
                    const T vis = T(0.5) * (TV[o.at(4, v - 1)] - Kn[v]) * dS;
                    K[v] = vis + K[v] * dS;
                    Kn[v] = T(0);
                }
            }
#pragma unroll
            for (int v = 0; v < 6; ++v) K[v] -= Kn[v];
        }
        const int slot = ft.le * 6 * G::n2 + ft.f * G::n2 + ft.fp;
#pragma unroll
        for (int v = 0; v < 3; ++v) sFs[v][slot] = V2<T>{K[2 * v], K[2 * v + 1]};
    }
    // this node's state and register (and compensation of an FP32 instance)
    T u6[6], Rn[6], Cn[6], iJ = T(0);
    const bool rk = L.mode == kRk;
    if (act) {
        T *R = rk ? a.R : a.Ut;  // holds the volume part (kUtParts: its sum)
#pragma unroll
        for (int v = 0; v < 6; ++v) Rn[v] = gldn<NT>(R + (v) * a.NN, g32);
        if (rk) {
#pragma unroll
            for (int v = 0; v < 6; ++v) {
                u6[v] = gldn<NT>(a.U + (v) * a.NN, g32);
                if constexpr (sizeof(T) == 4) Cn[v] = a.Ck ? gldn<NT>(a.Ck + (v) * a.NN, g32) : T(0);
            }
        }
        if constexpr (CV) iJ = T(1) / gld((const T *)a.mesh.nmet + 9 * a.NN, g32);
        else iJ = em_at<G::kUni, T>(a.mesh, e, kEmIJ);
    }
    __syncthreads();
    T acc[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
    if (act) {
        const int i = nd % P, j = (nd / P) % P, k = nd / (P * P);
        const int idx[3] = {i, j, k};
        const int fpd[3] = {j + P * k, i + P * k, i + P * j};
        const int fbase = le * 6 * G::n2;
        if (parts) {
#pragma unroll
            for (int v = 1; v < 5; ++v) acc[v] = Rn[v];
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const V2<T> lh = B.Lh[idx[d]];
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                const V2<T> fp = sFs[v][fbase + (2 * d + 1) * G::n2 + fpd[d]], fm = sFs[v][fbase + (2 * d) * G::n2 + fpd[d]];
                acc[2 * v] += lh.y * fp.x + lh.x * fm.x;
                acc[2 * v + 1] += lh.y * fp.y + lh.x * fm.y;
            }
        }
        if (!rk) {
#pragma unroll
            for (int v = 0; v < 6; ++v) {
                const T W = parts && v % 5 ? gld(a.Q + v * a.NN, g32) : Rn[v];
                gst(a.Ut + (v) * a.NN, g32, W - acc[v] * iJ);
            }
        }
    }
    if (!rk) return;
    // low-storage RK stage
    if (act) {
        const T B = T(L.B), dt = T(a.dt);
#pragma unroll
        for (int v = 0; v < 6; ++v) {
            // (1/J first, as in the volume part: dt / J would round for the surface
            // part alone, the same way in every step)
            const T r = Rn[v] - dt * (acc[v] * iJ);
            if (!L.last) gstn<NT>(a.R + (v) * a.NN, g32, T(r));
            T u;
            if (sizeof(T) == 4 && a.Ck) {
                // compensated summation: the low-order part lost by u6 + B r is
                // kept in Ck and fed into the next stage's increment
                const T y = B * r - Cn[v];
                u = u6[v] + y;
                gstn<NT>(a.Ck + (v) * a.NN, g32, T((u - u6[v]) - y));
            } else {
                u = u6[v] + B * r;
            }
            gstn<NT>(a.U + (v) * a.NN, g32, T(u));
            u6[v] = u;
        }
#pragma unroll
        for (int v = 0; v < 3; ++v) sF[v][tq] = V2<T>{u6[2 * v], u6[2 * v + 1]};
    }
    __syncthreads();
    const int ltask = line_of_thread<G>(t);
    const LineTask<P> lt(ltask < 0 ? 0 : ltask);
    const int el = e0 + lt.le;
    const bool lact = ltask >= 0 && el < E;
    if (lact) {
        T *TUw = a.TU + (size_t)L.tw * 6 * NF;
        const int b2 = lt.le * G::n3;
        T um[6], up[6];
#pragma unroll
        for (int v = 0; v < 3; ++v) prolong2<P, T>(sF[v], b2, B, lt, um + 2 * v, up + 2 * v);
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
            const FaceIx<G::n2> o((size_t)el * 6 + 2 * lt.d + sd, lt.fp);
#pragma unroll
            for (int v = 0; v < 6; ++v) TUw[o.at(6, v)] = sd ? up[v] : um[v];
        }
    }
}

}  // namespace nskr
