// Internal declarations of the gfx950 thermal LBM library: lattice traits, the
// per-cell arithmetic shared by the kernels, kernel argument blocks and the
// launchers called by the C ABI layer.
//
// Method (Li & Shan, arXiv:2302.04741, Sec. 2):
//   stored variable f~ (auxiliary variable of the trapezoidal time integration);
//   mid-point moments rho, u = u~ + g/2, theta = (E/rho - |u~|^2 + |g|^2/4)/D;
//   equilibrium = Hermite expansion of the Maxwellian to order N, eq. (fN);
//   force       = Hermite expansion eq. (F) to the third moment, eq. (fi);
//   sigma-bar   = -(1 - 1/(2 tau^)) sum_i (f~_i - f0_i)(xi_i - u)(xi_i - u), traceless;
//   step        = eq. (lbm): f~(x + xi_i, t+1) = f~ - (f~ - f0)/tau^ + (1 - 1/(2 tau^)) F.
// Everything here is written as closed-form polynomials in the integer velocity
// components with per-cell coefficients, and shares the sign parts of each orbit
// of velocities that differ in signs only.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "fastdiv.h"
#include "lattice_tables.h"

namespace lbm {

// ---------------------------------------------------------------------------
// compile-time loops
// ---------------------------------------------------------------------------
template <int I, typename F, int... K>
__host__ __device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, K...>)
{
    (f(std::integral_constant<int, I + K>{}), ...);
}
template <int I, int N, typename F> __host__ __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N)
        static_for_seq<I>(static_cast<F &&>(f), std::make_integer_sequence<int, N - I>{});
}

// fused multiply-add in the precision of its arguments
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// ---------------------------------------------------------------------------
// buffer access to the population planes: scalar resource (plane base, size),
// scalar row offset, per-lane 32-bit x offset.  Addressing costs no VALU work,
// and the hardware range check drops accesses past the plane.
// ---------------------------------------------------------------------------
constexpr int BUF_DWORD3 = 0x00020000;  // raw buffer, 32-bit data format
// Cache bits of a buffer access (gfx940 and later): 1 sc0, 2 nt, 16 sc1.  Stores
// with sc0 sc1 are written through the L2 to the memory side; with nt they are
// streamed (the memory-side cache does not keep them).
constexpr int BUF_DEFAULT = 0, BUF_NT = 2, BUF_THROUGH = 17, BUF_STREAM = 18;

// Cache policy of the step's population traffic: every element is read once and
// written once a step, and what one step writes is what the next one reads, so
// the 256 MB memory-side cache can serve part of a step's reads where the stores
// leave their lines in it.  T: bytes of one population buffer, whole 128-byte
// lines.
//
// RESIDENT (both buffers fit): default loads, stores written through (written back
//   by default they cost the same, but leave the L2's dirty lines to the end of
//   the launch).
// STREAM (larger): stores streamed past the cache, except the last W bytes of a
//   sweep, which are written through (KEEP); the next step sweeps the other way
//   and reads those first.  Loads of the kept part are marked nt, so that what is
//   being kept is not displaced by what is being read.
// STREAM_NT: STREAM with every load nt.
//
// us a step, STREAM against every store nt (the rest as here):
//   D2Q37 FP32 1024^2 (T 155 MB) 52.5 / 62.7, 1200^2 (219) 70 / 81, 1400^2 (308) 100 /
//   107, 2048^2 (621) 207 / 220, 3000^2 (1332) 462 / 476; FP64 900^2 (248) 77 / 88,
//   1537x1021 (465) 165 / 179; F16 1800^2 (250) 83 / 91, D3Q39 256^3 (1309) 471 / 484;
//   D3Q39 FP32 120^3 (288) 100 / 118, 160^3 (639) 230 / 239, 256^3 (2617) 940 / 948.
// RESIDENT against the same: D2Q37 FP32 512^2 (39) 14.7 / 18.0, 900^2 (124) 39 / 46;
//   D3Q39 F16 96^3 (71) 26 / 40.
enum class Policy { RESIDENT, STREAM, STREAM_NT, KEEP };
template <Policy P> struct CacheBits;
template <> struct CacheBits<Policy::RESIDENT> {
    static constexpr int load = BUF_DEFAULT, store = BUF_THROUGH;
};
template <> struct CacheBits<Policy::STREAM> {
    static constexpr int load = BUF_DEFAULT, store = BUF_STREAM;
};
template <> struct CacheBits<Policy::STREAM_NT> {
    static constexpr int load = BUF_NT, store = BUF_STREAM;
};
template <> struct CacheBits<Policy::KEEP> {
    static constexpr int load = BUF_NT, store = BUF_THROUGH;
};

// The LLVM intrinsics by name (a compiler without them fails at the link).  clang's
// builtins take a resource that only __builtin_amdgcn_make_buffer_rsrc forms, which masks
// the address on every access: one scalar instruction more each, 0.2-0.4% of a step, and
// 20 to 28 bytes of scratch in the FP64 D3Q39 step (129x95x110, 8 steps, 1565 us against
// 1525; 256^3 1940 against 1887).
typedef int RsrcWords __attribute__((ext_vector_type(4)));
typedef int Words2 __attribute__((ext_vector_type(2)));
__device__ float buf_load_f32(RsrcWords, int, int, int) __asm("llvm.amdgcn.raw.buffer.load.f32");
__device__ Words2 buf_load_2i32(RsrcWords, int, int, int) __asm("llvm.amdgcn.raw.buffer.load.v2i32");
__device__ short buf_load_i16(RsrcWords, int, int, int) __asm("llvm.amdgcn.raw.buffer.load.i16");
__device__ void buf_store_f32(float, RsrcWords, int, int,
                              int) __asm("llvm.amdgcn.raw.buffer.store.f32");
__device__ void buf_store_2i32(Words2, RsrcWords, int, int,
                               int) __asm("llvm.amdgcn.raw.buffer.store.v2i32");
__device__ void buf_store_i16(short, RsrcWords, int, int,
                              int) __asm("llvm.amdgcn.raw.buffer.store.i16");

// The planes of one population buffer, one after the other: the next plane's
// resource is two scalar adds away from the last one's (a resource made afresh
// for each plane took about ten scalar instructions, and a wavefront issues one
// scalar instruction in the time of one vector instruction).
struct PlaneWalk {
    uint64_t base;  // device address of the current plane (48 bits)
    uint32_t bytes;
    int plane;
    __device__ __forceinline__ PlaneWalk(const void *p, uint32_t plane_bytes)
        : base(reinterpret_cast<uint64_t>(p)), bytes(plane_bytes), plane(0)
    {
    }
    // resource of plane i (a compile-time index)
    __device__ __forceinline__ RsrcWords at(int i)
    {
        if (i >= plane) base += uint64_t(bytes) * uint32_t(i - plane);
        else base -= uint64_t(bytes) * uint32_t(plane - i);
        plane = i;
        return RsrcWords{int(uint32_t(base)), int(uint32_t(base >> 32)), int(bytes), BUF_DWORD3};
    }
};

template <class S> struct BufIO;
template <> struct BufIO<float> {
    template <int LD>
    __device__ static __forceinline__ float load(RsrcWords r, uint32_t v, uint32_t s)
    {
        return buf_load_f32(r, int(v), int(s), LD);
    }
    template <int ST>
    __device__ static __forceinline__ void store(float x, RsrcWords r, uint32_t v, uint32_t s)
    {
        buf_store_f32(x, r, int(v), int(s), ST);
    }
};
template <> struct BufIO<double> {
    template <int LD>
    __device__ static __forceinline__ double load(RsrcWords r, uint32_t v, uint32_t s)
    {
        return __builtin_bit_cast(double, buf_load_2i32(r, int(v), int(s), LD));
    }
    template <int ST>
    __device__ static __forceinline__ void store(double x, RsrcWords r, uint32_t v, uint32_t s)
    {
        buf_store_2i32(__builtin_bit_cast(Words2, x), r, int(v), int(s), ST);
    }
};
template <> struct BufIO<__half> {
    template <int LD>
    __device__ static __forceinline__ __half load(RsrcWords r, uint32_t v, uint32_t s)
    {
        return __builtin_bit_cast(__half, buf_load_i16(r, int(v), int(s), LD));
    }
    template <int ST>
    __device__ static __forceinline__ void store(__half x, RsrcWords r, uint32_t v, uint32_t s)
    {
        buf_store_i16(__builtin_bit_cast(short, x), r, int(v), int(s), ST);
    }
};

// ---------------------------------------------------------------------------
// lattice traits (velocity order: rest, then +c/-c pairs shell by shell)
// ---------------------------------------------------------------------------
template <int LAT> struct Lattice;

template <> struct Lattice<0> {
    static constexpr int D = D2Q37_D, Q = D2Q37_Q, NS = D2Q37_NSHELL, MAXEQ = 4;
    // r^2 as R*R (not the separately rounded r^2) keeps xi^2 consistent with xi = R c
    static constexpr double R = d2q37_R, R2 = d2q37_R * d2q37_R;
    static constexpr int c(int i, int a) { return d2q37_C[i][a]; }
    static constexpr int shell(int i) { return d2q37_SHELL[i]; }
    static constexpr double wshell(int s) { return d2q37_WSHELL[s]; }
};

template <> struct Lattice<1> {
    static constexpr int D = D3Q39_D, Q = D3Q39_Q, NS = D3Q39_NSHELL, MAXEQ = 3;
    static constexpr double R = d3q39_R, R2 = d3q39_R * d3q39_R;
    static constexpr int c(int i, int a) { return d3q39_C[i][a]; }
    static constexpr int shell(int i) { return d3q39_SHELL[i]; }
    static constexpr double wshell(int s) { return d3q39_WSHELL[s]; }
};

template <class L> constexpr int c2(int i)
{
    return L::c(i, 0) * L::c(i, 0) + L::c(i, 1) * L::c(i, 1) + L::c(i, 2) * L::c(i, 2);
}

// Velocities come in orbits of sign flips: |c| = (k_x, k_y, k_z) with every sign
// of every nonzero component, 2, 4 or 8 velocities of one shell.  orbit_rep: i
// is the orbit's member without negative components; velocity_of: the index of
// a vector of the set.
template <class L> constexpr bool orbit_rep(int i)
{
    return i > 0 && L::c(i, 0) >= 0 && L::c(i, 1) >= 0 && L::c(i, 2) >= 0;
}
template <class L> constexpr int velocity_of(int x, int y, int z)
{
    for (int i = 0; i < L::Q; ++i)
        if (L::c(i, 0) == x && L::c(i, 1) == y && L::c(i, 2) == z) return i;
    return -1;
}
template <class L> constexpr int opposite(int i)
{
    return velocity_of<L>(-L::c(i, 0), -L::c(i, 1), -L::c(i, 2));
}
// The orbit of rep seen as +c/-c pairs: pair s flips the sign of the last nonzero
// axis by bit 0 of s and, of three, that of the second by bit 1; the planes of
// the pairs then ascend.
template <class L> struct Orbit {
    int n, ax[3];  // nonzero components and their axes
    constexpr explicit Orbit(int rep) : n(0), ax{0, 0, 0}
    {
        for (int a = 0; a < 3; ++a)
            if (L::c(rep, a) != 0) ax[n++] = a;
    }
    constexpr int pairs() const { return n == 1 ? 1 : (n == 2 ? 2 : 4); }
    constexpr int plus(int rep, int s) const
    {
        int c[3] = {L::c(rep, 0), L::c(rep, 1), L::c(rep, 2)};
        if (n > 1 && (s & 1)) c[ax[n - 1]] = -c[ax[n - 1]];
        if (s & 2) c[ax[1]] = -c[ax[1]];
        return velocity_of<L>(c[0], c[1], c[2]);
    }
};

// The orbits' representatives, those on the axes first, then by nonzero components
// and plane.
template <class L> struct OrbitList {
    int n, rep[L::Q];
    constexpr OrbitList() : n(0), rep{}
    {
        for (int k = 1; k <= 3; ++k)
            for (int i = 1; i < L::Q; ++i)
                if (orbit_rep<L>(i) && Orbit<L>(i).n == k) rep[n++] = i;
    }
};
template <class L> constexpr OrbitList<L> ORBITS{};

// ---------------------------------------------------------------------------
// storage conversion
// ---------------------------------------------------------------------------
// Every storage type holds the deviations h_i = f_i - w_i rho0.  LBM_F16DEV
// stores h_i * 2^k_i as binary16, with k_i = round(-log2 w_i): the exact
// power-of-two scale brings deviations of the size of w_i to about one, far
// from the subnormal range of binary16.
// The factor a stored value carries relative to the deviation it stands for:
// 1 for FP64 and FP32 storage (reduced-precision storage supplies its own).
struct UnitScale {
    template <int I> static constexpr double scale() { return 1.0; }
};

template <class L> struct DevScale {
    static constexpr int k(int i)
    {
        // k_i = round(-log2(w_i)): an exact power of two, chosen so that a
        // deviation comparable to w_i is stored near 1.
        double w = L::wshell(L::shell(i));
        int e = 0;
        while (w < 0.70710678118654752) {
            w *= 2.0;
            ++e;
        }
        return e;
    }
};

// ---------------------------------------------------------------------------
// argument blocks
// ---------------------------------------------------------------------------
// Population planes store rows of px >= nx values (nx rounded up to a multiple
// of 64), so that every row starts on a 128-byte line and a wavefront's run of
// 64 consecutive cells touches the fewest lines; values at x >= nx are never
// read or written.  Field arrays (moments, forces) are dense: cell =
// (z*ny + y)*nx + x.
constexpr int ROW_ALIGN = 64;

struct GridDims {
    int32_t nx, ny, nz;
    int32_t px;     // row pitch of the population planes
    int64_t N;      // cells, nx*ny*nz
    int64_t P;      // values per population plane, px*ny*nz
    DivU32 by_wpr;  // division by the wavefronts per row, ceil(nx / 64)
    DivU32 by_ny;   // division by ny
};

inline GridDims make_grid_dims(int64_t nx, int64_t ny, int64_t nz, int64_t px)
{
    return GridDims{int32_t(nx), int32_t(ny), int32_t(nz), int32_t(px), nx * ny * nz,
                    px * ny * nz, make_divu32(uint32_t((nx + 63) / 64)),
                    make_divu32(uint32_t(ny))};
}

struct ForceDesc {
    int32_t kind;  // 0 uniform, 1 axis profile, 2 field
    int32_t axis;  // profile axis
    int64_t len;   // profile length
    double g[3];   // uniform value
    const void *tab;  // profile (D*len) or field (D*N), arithmetic precision
};

struct StepCoef {
    double om;   // 1/tau^
    double cf;   // 1 - 1/(2 tau^)
    double rho0; // reference density of the stored deviations
    double mu;   // > 0: per-cell tau^ = mu/(rho theta) + 1/2 replaces om and cf
};

// Plates normal to y at y = -1/2 and y = ny - 1/2 (lbm_set_walls): a population
// whose streaming source lies behind a plate is the plate's emission
// rw[side][column of the source] * e[side][i]; populations streaming into a
// plate stay in their slots at the node they leave (the "crossing" slots).
// A plate's density rw over column (x, z) is the sum of the
// slots of the rows next to it whose next move crosses it, over the plate's
// normalisation e_Q.  Those sums are kept per row ("partial sums": rows 0, 1, 2
// for the bottom plate, ny-3+k for the top one; the same rows for both when
// ny < 3), for each of the two population buffers: the step that writes a
// buffer also writes its partial sums, and the next step adds the (at most 3)
// rows of a column in order.
struct WallDesc {
    int32_t on;
    int32_t par;      // buffer holding the state read (0 or 1): its sums are part[par]
    double *part;     // [2 buffer][2 plate][3 row][nx*nz] partial sums (bottom, top)
    const double *e;  // [2][Q + 1]: e_i = f0_i(1, (U_w, 0, 0), theta_w), then the normalisation
};

__host__ __device__ inline int64_t wall_part_index(int par, int side, int k, int64_t ncol,
                                                   int64_t col)
{
    return ((int64_t(par) * 2 + side) * 3 + k) * ncol + col;
}

// One member of a multi-grid batch (device table entry).  Its tiles are runs
// of 64 cells along x (one wavefront each): chunks_x per grid row, rows in
// (z, y) order.
struct TileSim {
    const void *pop[2];  // the two population buffers
    uint32_t *ctr;       // step counter pair (F16 stochastic rounding keys), see LaunchCfg
    int32_t cur;         // buffer holding the state when the table was built
    int32_t chunks_x;    // tiles per grid row, ceil(nx / 64)
    int64_t tile_begin;  // first tile of this simulation in the list
    GridDims gd;
    ForceDesc fd;
    StepCoef co;
    WallDesc wd;         // plates (off for a periodic member); wd.par is set per step
};

// ---------------------------------------------------------------------------
// body force at a cell
// ---------------------------------------------------------------------------
// TT: element type of the force table (the arithmetic precision of the
// storage), TO: output type.
template <class TT, class TO, int D>
__device__ __forceinline__ void load_force(const ForceDesc &fd, const GridDims &gd, int x, int y,
                                           int z, int64_t cell, TO g[3])
{
    g[0] = g[1] = g[2] = TO(0);
    if (fd.kind == 0) {
        for (int a = 0; a < D; ++a) g[a] = TO(TT(fd.g[a]));
    } else if (fd.kind == 1) {
        const TT *tab = static_cast<const TT *>(fd.tab);
        const int k = fd.axis == 0 ? x : (fd.axis == 1 ? y : z);
        for (int a = 0; a < D; ++a) g[a] = TO(tab[a * fd.len + k]);
    } else {
        const TT *tab = static_cast<const TT *>(fd.tab);
        for (int a = 0; a < D; ++a) g[a] = TO(tab[a * gd.N + cell]);
    }
}

// ---------------------------------------------------------------------------
// per-cell state after the moment pass
// ---------------------------------------------------------------------------
template <class T> struct CellState {
    T rho;
    T drho;      // rho - rho0
    T ub[3];     // mid-point velocity u~ + g/2
    T th;        // mid-point temperature
    T g[3];
    T sig[3][3]; // mid-point deviatoric stress (traceless), zero unless needed
    T om;        // 1/tau^ of this cell
    T cf;        // 1 - 1/(2 tau^) of this cell
};

// Raw sums of one cell over the stored deviations h_i = f_i - w_i rho0:
// drho = sum h, j = sum h c (integer c), P = sum h c c.  Because the weights
// satisfy sum w = 1, sum w c = 0 and sum w c c = delta / r^2, the moments of f
// follow as rho = rho0 + drho, sum f xi = r j, sum f xi xi = rho0 delta + r^2 P.
template <class T> struct RawSums {
    T drho, j[3], P[3][3];
};

//
// SC::scale<i>() is the factor the values carry (1, or the power of two of
// reduced-precision storage, the same for every velocity of a shell): the
// sums take it out through their constants.
//
// The sums go orbit by orbit: the 2, 4 or 8 populations of an orbit are first
// transformed into their sign sums (a Hadamard transform: S = sum, X_a = sum
// sign_a, E_ab = sum sign_a sign_b), of which each moment needs one term per
// orbit; the diagonal of P shares its running sums by |c_a| = 1, 2, 3.
template <class L, class T, class SC = UnitScale>
__device__ __forceinline__ RawSums<T> raw_sums(const T (&h)[L::Q])
{
    constexpr int D = L::D;
    RawSums<T> s;
    for (int a = 0; a < 3; ++a) {
        s.j[a] = T(0);
        for (int b = 0; b < 3; ++b) s.P[a][b] = T(0);
    }
    T by_k[3][3];  // [axis][|c_a| - 1]: sum of the orbits' S
    T rest;        // orbits without an x component
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) by_k[a][k] = T(0);
    constexpr double u0 = 1.0 / SC::template scale<0>();
    rest = (u0 == 1.0) ? h[0] : h[0] * T(u0);
    // acc += m * v, one rounding; the scale is folded into m
    auto add = [](T &acc, double m, T v) {
        if (m == 1.0) acc += v;
        else acc = fma_t(v, T(m), acc);
    };
    static_for<0, ORBITS<L>.n>([&](auto I) {
        constexpr int i = ORBITS<L>.rep[decltype(I)::value];
        constexpr Orbit<L> o(i);
        constexpr double u = 1.0 / SC::template scale<i>();  // exact: a power of two
        constexpr int a0 = o.ax[0], a1 = o.ax[1], a2 = o.ax[2];
        constexpr int k0 = L::c(i, a0), k1 = L::c(i, a1), k2 = L::c(i, a2);
        T sp[4], dm[4];
        static_for<0, o.pairs()>([&](auto J) {
            constexpr int j = decltype(J)::value;
            constexpr int ip = o.plus(i, j);
            constexpr int im = opposite<L>(ip);
            sp[j] = h[ip] + h[im];
            dm[j] = h[ip] - h[im];
        });
        T S;
        if constexpr (o.n == 1) {
            S = sp[0];
            add(s.j[a0], u * k0, dm[0]);
        } else if constexpr (o.n == 2) {
            S = sp[0] + sp[1];
            add(s.P[a0][a1], u * (k0 * k1), sp[0] - sp[1]);
            add(s.j[a0], u * k0, dm[0] + dm[1]);
            add(s.j[a1], u * k1, dm[0] - dm[1]);
        } else {
            const T pa = sp[0] + sp[1], ma = sp[0] - sp[1];
            const T pb = sp[2] + sp[3], mb = sp[2] - sp[3];
            S = pa + pb;
            add(s.P[a0][a2], u * (k0 * k2), ma + mb);
            add(s.P[a0][a1], u * (k0 * k1), pa - pb);
            add(s.P[a1][a2], u * (k1 * k2), ma - mb);
            const T qa = dm[0] + dm[1], na = dm[0] - dm[1];
            const T qb = dm[2] + dm[3], nb = dm[2] - dm[3];
            add(s.j[a0], u * k0, qa + qb);
            add(s.j[a2], u * k2, na + nb);
            add(s.j[a1], u * k1, qa - qb);
        }
        add(by_k[a0][k0 - 1], u, S);
        if constexpr (o.n >= 2) add(by_k[a1][k1 - 1], u, S);
        if constexpr (o.n >= 3) add(by_k[a2][k2 - 1], u, S);
        if constexpr (L::c(i, 0) == 0) add(rest, u, S);
    });
    s.drho = rest + ((by_k[0][0] + by_k[0][1]) + by_k[0][2]);
    for (int a = 0; a < D; ++a)
        s.P[a][a] = fma_t(T(9), by_k[a][2], fma_t(T(4), by_k[a][1], by_k[a][0]));
    return s;
}

// Mid-point moments, relaxation coefficients and (if WITH_SIGMA) sigma-bar
// from the raw sums.
//   rho = rho0 + drho, u = r j / rho + g/2,
//   theta = (E/rho - |u~|^2 + |g|^2/4)/D with E = rho0 D + r^2 tr P;
//   tau^ = the run's constant, or mu/(rho theta) + 1/2 when mu > 0 (the
//   relaxation time that keeps the dynamic viscosity constant, Sec. 3);
//   sigma-bar = -cf [sum f xi xi - rho(u u + theta delta) + rho (u g + g u)/2]
//   with its trace removed.  The isotropic parts (rho0 delta and
//   rho theta delta) drop out of the traceless projection exactly, so they are
//   left out: sigma-bar = dev(-cf [r^2 P - rho u u + rho (u g + g u)/2]).
template <class L, class T, bool WITH_SIGMA>
__device__ __forceinline__ void finish_moments(const RawSums<T> &s, const T g[3],
                                               const StepCoef &co, CellState<T> &cs)
{
    constexpr int D = L::D;
    const T r = T(L::R), r2 = T(L::R2);
    const T rho0 = T(co.rho0);
    const T rho = rho0 + s.drho;
    const T inv = T(1) / rho;
    T ut2 = T(0), g2 = T(0), tr = T(0);
    cs.rho = rho;
    cs.drho = s.drho;
    for (int a = 0; a < 3; ++a) {
        cs.g[a] = g[a];
        cs.ub[a] = T(0);
    }
    for (int a = 0; a < D; ++a) {
        const T ut = r * s.j[a] * inv;
        cs.ub[a] = ut + T(0.5) * g[a];
        ut2 += ut * ut;
        g2 += g[a] * g[a];
        tr += s.P[a][a];
    }
    const T E = rho0 * T(D) + r2 * tr;
    cs.th = (E * inv - ut2 + T(0.25) * g2) * T(1.0 / D);
    cs.om = T(co.om);
    cs.cf = T(co.cf);
    if (co.mu > 0.0) {  // uniform over the launch
        cs.om = T(1) / (T(co.mu) / (rho * cs.th) + T(0.5));
        cs.cf = T(1) - T(0.5) * cs.om;
    }
    const T cf = cs.cf;
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) cs.sig[a][b] = T(0);
    if constexpr (WITH_SIGMA) {
        T str = T(0);
        for (int a = 0; a < D; ++a) {
            for (int b = a; b < D; ++b) {
                T v = r2 * s.P[a][b] - rho * cs.ub[a] * cs.ub[b]
                      + T(0.5) * rho * (cs.ub[a] * g[b] + g[a] * cs.ub[b]);
                v *= -cf;
                cs.sig[a][b] = v;
                cs.sig[b][a] = v;
            }
            str += cs.sig[a][a];
        }
        for (int a = 0; a < D; ++a) cs.sig[a][a] -= str * T(1.0 / D);
    }
}

// ---------------------------------------------------------------------------
// alpha * f0 + beta * F for every velocity, in even/odd pair form.
//
// For velocity xi_i in shell s (xi^2 = X2) with xu = xi.u, xg = xi.g,
// u2 = |u|^2, t = theta - 1, gu = g.u:
//   f0 = w rho [ e(xu^2) + o(xu) ],  e even, o odd in xi:
//     e = 1 + (xu^2 - u2 + t(X2 - D))/2
//         + [xu^4 - 6 xu^2 u2 + 3 u2^2 + 6t(xu^2(X2 - D - 4) + u2(D + 2 - X2))
//            + 3t^2(X2^2 - 2(D+2) X2 + D(D+2))]/24            (N = 4)
//     o = xu [1 + (xu^2 - 3 u2 + 3t(X2 - D - 2))/6]           (N >= 3; xu for N = 2)
//   F (eq. (fi)) even part  w rho (xg xu - gu)                (order >= 2)
//     odd part  w rho xg                                       (order 1, 2)
//               w rho [xg (1 + (xu^2 - u2 + t(X2 - D - 2))/2) - gu xu]   (order >= 3)
//               - (w/2) [xg (xi.sigma.xi) - 2 xi.sigma.g]     (order 4)
// The even part omits alpha * w * rho (the leading term of f0) and has w * base added
// (callers pass the rounded increment of that leading term, or add it themselves).
// With a scale SC every w is w * SC::scale<i>() (a power of two): even and odd come
// out multiplied by it exactly.
// The callback receives (i_plus, i_minus, even, odd) for each pair and
// (0, -1, even, 0) for the rest velocity; the indices are passed as
// std::integral_constant so that callers index register arrays statically.
//
// Evaluation.  In the integer components c of xi = r c, even/w and odd/w are
// polynomials of degree <= 4 whose coefficients depend on the cell only, so
// they are computed once a cell and each orbit of sign flips needs its sign
// parts only: with |c| = (k_x, k_y, k_z)
//   even/w = E + sum_{a<b} sign_a sign_b E_ab,  odd/w = sum_a sign_a O_a (+ sign_xyz O_xyz),
//   E    = C + T (X2 - D) + sum_a k_a^2 (K_a + k_a^2 Q_a) + k_x^2 k_y^2 Q_xy
//                                                     (T = alpha rho t/2; Q: N = 4, D = 2)
//   E_ab = k_a k_b (K_ab + k_a^2 Q_aab + k_b^2 Q_abb)
//   O_a  = k_a (G_a + sum_b k_b^2 H_ab),   O_xyz = k_x k_y k_z H_xyz
// and the 2, 4 or 8 velocities of the orbit are the butterflies of those parts.
// Against xi.u, xi.g and xi.sigma.xi dotted out for each pair this halves the
// step's vector instructions (counts and times at step_cell).
//
// A rounding error of a coefficient that all populations share goes into the conserved
// sums whole, as sum w = 1.  So the large isotropic term T (X2 - D) is added shell by
// shell, and C is what makes the even parts sum to base for the K and Q as they were
// rounded (sum w c_a^2 = 1/r^2, sum w c_a^4 = 3/r^4, sum w c_a^2 c_b^2 = 1/r^4).  Rms
// change of the mass in one FP32 collision, speeds to 0.05: D2Q37 1.4e-9, D3Q39
// 1.7e-9; with the closed form of C and all of it in one constant 2.9e-9 and 3.6e-9,
// with xi.u dotted out for each pair 2.5e-9 and 2.6e-9; speeds to 1.5 along x 6.6e-8
// and 7.5e-8 against 9.3e-8 and 1.0e-7 pair by pair.
// ---------------------------------------------------------------------------
template <class L, class T, int EQ, int FO, class SC = UnitScale, class CB>
__device__ __forceinline__ void combo_pairs(const CellState<T> &cs, T alpha, T beta, T base,
                                            CB &&cb)
{
    constexpr int D = L::D;
    static_assert(EQ < 4 || D == 2, "the fourth order is written out for two dimensions");
    const T r = T(L::R), r2 = T(L::R2);
    T U[3], G[3], u2 = T(0), gu = T(0);
    for (int a = 0; a < 3; ++a) {
        U[a] = r * cs.ub[a];
        G[a] = r * cs.g[a];
    }
    for (int a = 0; a < D; ++a) {
        u2 = fma_t(cs.ub[a], cs.ub[a], u2);
        gu = fma_t(cs.g[a], cs.ub[a], gu);
    }
    const T t = cs.th - T(1);
    const T arho = alpha * cs.rho, brho = beta * cs.rho, brgu = brho * gu;
    const T half_t = T(0.5) * t;

    // polynomials in X2 of the even part's xu^2 factor D0 + D1 X2 and of the odd
    // part's xu factor G0 + G1 X2
    T D0 = T(0.5), D1 = T(0), tt = T(0), tu = T(0);
    if constexpr (EQ == 4) {
        tt = t * t;
        tu = t * u2;
        // (t (X2 - D - 4) - u2) / 4
        D0 -= T(0.25) * fma_t(T(D + 4), t, u2);
        D1 = T(0.25) * t;
    }
    const T G0 = T(1) - fma_t(half_t, T(D + 2), T(0.5) * u2), G1 = half_t;

    // odd coefficients (first: the other way round the FP64 step on D3Q39 takes 8
    // registers more a lane, and its batch kernel drops to two wavefronts a SIMD)
    constexpr bool CUBIC = EQ >= 3 || FO >= 3;
    T O[3], H[3][3], Hxyz = T(0);
    {
        T Z[3][3];  // FO >= 3: G_a's quadratic forms, rho xu^2 / 2 - xi.sigma.xi / 2 (times beta)
        if constexpr (FO == 4) {
            const T hb2 = T(0.5 * L::R2) * beta;
            for (int a = 0; a < D; ++a)
                for (int b = a; b < D; ++b) Z[a][b] = Z[b][a] = -hb2 * cs.sig[a][b];
            // the linear term of sigma, 2 (beta/2) xi.sigma.g
            for (int a = 0; a < D; ++a) {
                T sg = T(0);
                for (int b = 0; b < D; ++b) sg = fma_t(Z[a][b], G[b], sg);
                O[a] = T(-2.0 / L::R2) * sg;
            }
        }
        if constexpr (FO >= 3) {
            const T hbrho = T(0.5) * brho;
            for (int a = 0; a < D; ++a) {
                const T hu = hbrho * U[a];
                for (int b = a; b < D; ++b)
                    Z[a][b] = Z[b][a] = FO == 4 ? fma_t(hu, U[b], Z[a][b]) : hu * U[b];
            }
        }
        for (int a = 0; a < D; ++a) {
            const T au = arho * U[a];
            const T bg = brho * G[a];
            // linear
            T lin;
            if constexpr (EQ >= 3 && FO >= 3) lin = fma_t(G0, au + bg, -brgu * U[a]);
            else if constexpr (EQ >= 3) lin = fma_t(G0, au, bg);
            else if constexpr (FO >= 3) lin = fma_t(G0, bg, fma_t(-brgu, U[a], au));
            else lin = au + bg;
            O[a] = FO == 4 ? O[a] + lin : lin;
            // cubic: c_a c_b^2
            if constexpr (CUBIC) {
                const T iso = G1 * r2 * (EQ >= 3 && FO >= 3 ? au + bg : (EQ >= 3 ? au : bg));
                for (int b = 0; b < D; ++b) {
                    T v = iso;
                    if constexpr (EQ >= 3) v = fma_t(T(a == b ? 1.0 / 6.0 : 0.5) * au, U[b] * U[b], v);
                    if constexpr (FO >= 3) {
                        v = fma_t(G[a], Z[b][b], v);
                        if (a != b) v = fma_t(T(2) * G[b], Z[a][b], v);
                    }
                    H[a][b] = v;
                }
            }
        }
        if constexpr (CUBIC && D == 3) {
            if constexpr (EQ >= 3) Hxyz = arho * U[0] * U[1] * U[2];
            if constexpr (FO >= 3)
                Hxyz = fma_t(T(2), fma_t(G[0], Z[1][2], fma_t(G[1], Z[0][2], G[2] * Z[0][1])),
                             Hxyz);
        }
    }

    // even coefficients
    const T iso = arho * half_t;
    T K[3], Kab[3][3], Q[3] = {T(0), T(0), T(0)}, Qxy = T(0), Qab[2] = {T(0), T(0)}, C;
    {
        const T m = arho * D0;
        T V[3];  // half the quadratic form's vector: K_ab = U_a V_b + U_b V_a
        for (int a = 0; a < D; ++a) V[a] = FO >= 2 ? fma_t(m, U[a], brho * G[a]) : m * U[a];
        // the fourth order's X2 and X2^2: -t (u2 + (D + 2) t) / 4 and t^2 / 8
        const T e1 = arho * T(-0.25 * L::R2) * fma_t(T(D + 2), tt, tu);
        for (int a = 0; a < D; ++a) {
            K[a] = EQ == 4 ? fma_t(U[a], V[a], e1) : U[a] * V[a];
            for (int b = a + 1; b < D; ++b) Kab[a][b] = fma_t(U[a], V[b], U[b] * V[a]);
        }
        T sum = K[0];
        for (int a = 1; a < D; ++a) sum += K[a];
        if constexpr (EQ == 4) {
            const T e2 = arho * tt * T(0.125 * L::R2 * L::R2);
            const T d1 = arho * D1 * r2;
            const T a24 = arho * T(1.0 / 24.0);
            const T xx = U[0] * U[0], yy = U[1] * U[1], xy = U[0] * U[1];
            Q[0] = fma_t(xx, fma_t(a24, xx, d1), e2);
            Q[1] = fma_t(yy, fma_t(a24, yy, d1), e2);
            Qxy = fma_t(d1, xx + yy, fma_t(T(6) * a24 * xx, yy, T(2) * e2));
            Qab[0] = xy * fma_t(T(4) * a24, xx, T(2) * d1);
            Qab[1] = xy * fma_t(T(4) * a24, yy, T(2) * d1);
            sum = fma_t(T(1.0 / L::R2), fma_t(T(3), Q[0] + Q[1], Qxy), sum);
        }
        C = fma_t(T(-1.0 / L::R2), sum, base);
    }
    // C + T (X2 - D) of a shell
    auto isotropic = [&](double X2) { return fma_t(T(X2 - D), iso, C); };
    // rest velocity
    constexpr double w0 = L::wshell(L::shell(0)) * SC::template scale<0>();
    cb(std::integral_constant<int, 0>{}, std::integral_constant<int, -1>{},
       T(w0) * isotropic(0.0), T(0));

    // orbits on the axes first: they need no mixed coefficient, so the populations
    // they take are gone before those are formed (two FP64 registers a lane)
    static_for<0, ORBITS<L>.n>([&](auto I) {
        constexpr int i = ORBITS<L>.rep[decltype(I)::value];
        constexpr Orbit<L> o(i);
        constexpr double w = L::wshell(L::shell(i)) * SC::template scale<i>();
        constexpr int a0 = o.ax[0], a1 = o.ax[1], a2 = o.ax[2];
        constexpr int k0 = L::c(i, a0), k1 = L::c(i, a1), k2 = L::c(i, a2);
        // k^2 (K + k^2 Q) of one axis, and the odd part's G + k^2 H
        auto even1 = [&](auto A, T acc) {
            constexpr int a = decltype(A)::value, k = L::c(i, a);
            if constexpr (EQ == 4) return fma_t(T(k * k), fma_t(T(k * k), Q[a], K[a]), acc);
            else return fma_t(T(k * k), K[a], acc);
        };
        auto odd1 = [&](auto A) {
            constexpr int a = decltype(A)::value, k = L::c(i, a);
            T v = O[a];
            if constexpr (CUBIC) {
                v = fma_t(T(k * k), H[a][a], v);
                static_for<0, D>([&](auto B) {
                    constexpr int b = decltype(B)::value, kb = L::c(i, b);
                    if constexpr (b != a && kb != 0) v = fma_t(T(kb * kb), H[a][b], v);
                });
            }
            return T(w * k) * v;
        };
        auto cross = [&](auto A, auto B) {
            constexpr int a = decltype(A)::value, b = decltype(B)::value;
            constexpr int ka = L::c(i, a), kb = L::c(i, b);
            T v = Kab[a][b];
            if constexpr (EQ == 4)
                v = fma_t(T(kb * kb), Qab[1], fma_t(T(ka * ka), Qab[0], v));
            return T(w * ka * kb) * v;
        };
        auto emit = [&](auto J, T ev, T od) {
            constexpr int ip = o.plus(i, decltype(J)::value);
            constexpr int im = opposite<L>(ip);
            cb(std::integral_constant<int, ip>{}, std::integral_constant<int, im>{}, ev, od);
        };
        using A0 = std::integral_constant<int, a0>;
        using A1 = std::integral_constant<int, a1>;
        using A2 = std::integral_constant<int, a2>;
        T e = even1(A0{}, isotropic(L::R2 * c2<L>(i)));
        if constexpr (o.n == 1) {
            emit(std::integral_constant<int, 0>{}, T(w) * e, odd1(A0{}));
        } else if constexpr (o.n == 2) {
            e = even1(A1{}, e);
            if constexpr (EQ == 4) e = fma_t(T(k0 * k0 * k1 * k1), Qxy, e);
            e *= T(w);
            const T x = cross(A0{}, A1{});
            const T p = odd1(A0{}), q = odd1(A1{});
            emit(std::integral_constant<int, 0>{}, e + x, p + q);
            emit(std::integral_constant<int, 1>{}, e - x, p - q);
        } else {
            e = T(w) * even1(A2{}, even1(A1{}, e));
            const T x = cross(A0{}, A1{}), y = cross(A0{}, A2{}), z = cross(A1{}, A2{});
            const T p = odd1(A0{}), q = odd1(A1{}), v = odd1(A2{});
            const T h = CUBIC ? T(w * k0 * k1 * k2) * Hxyz : T(0);
            // signs (+, s1, s2): even e + s1 x + s2 y + s1 s2 z, odd p + s1 q + s2 v + s1 s2 h
            const T ex = e + x, em = e - x, yz = y + z, ym = y - z;
            const T pq = p + q, pm = p - q, vh = v + h, vm = v - h;
            emit(std::integral_constant<int, 0>{}, ex + yz, pq + vh);
            emit(std::integral_constant<int, 1>{}, ex - yz, pq - vh);
            emit(std::integral_constant<int, 2>{}, em + ym, pm + vm);
            emit(std::integral_constant<int, 3>{}, em - ym, pm - vm);
        }
    });
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

struct LaunchCfg {
    int block;  // threads along x per block
    hipStream_t stream;
    WallDesc walls;  // off unless the handle has plates
    uint32_t *ctr;   // the handle's step counter pair (keys of the F16 stochastic rounding)
    int cur;         // buffer holding the state read: the step reads ctr[cur], writes ctr[cur ^ 1]
};

// Generic entry points (lbm_dispatch.hip), switching on lattice and storage.
hipError_t launch_pattern(int lat, int storage, const void *A, void *B, const GridDims &gd,
                          const LaunchCfg &lc);
hipError_t launch_step(int lat, int storage, int eq, int fo, const void *A, void *B,
                       const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                       const LaunchCfg &lc);
hipError_t launch_init(int lat, int storage, int eq, int fo, const double *rho, const double *u,
                       const double *theta, void *A, const GridDims &gd, const ForceDesc &fd,
                       const StepCoef &co, const LaunchCfg &lc);
hipError_t launch_rebuild(int lat, int storage, int eq, int fo, const void *A, void *B,
                          const GridDims &gd, const ForceDesc &old_force, const ForceDesc &force,
                          const StepCoef &co, const LaunchCfg &lc);
hipError_t launch_moments(int lat, int storage, const void *A, double *rho, double *u,
                          double *theta, const GridDims &gd, const ForceDesc &fd,
                          const StepCoef &co, const LaunchCfg &lc);
hipError_t launch_heat_flux(int lat, int storage, int eq, int fo, const void *A, double *q,
                            const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                            const LaunchCfg &lc);
hipError_t launch_totals(int lat, int storage, const void *A, double *partials, double *out_dev,
                         const GridDims &gd, const StepCoef &co, hipStream_t stream);
hipError_t launch_convert(int storage, const double *src, void *dst, int64_t n,
                          hipStream_t stream);
// dense rows (nx values each, back to back) out of (exporting) or into the padded
// rows of all Q planes; `dense` aligned to the stored type (rows.hip)
hipError_t launch_copy_rows(int storage, void *padded, void *dense, const GridDims &gd, int Q,
                            bool exporting, hipStream_t stream);
constexpr int64_t MIB = int64_t(1) << 20;
constexpr int64_t STEP_CACHED_BYTES = 128 * MIB;  // two such buffers fit the memory-side cache
// One launch of the multi-grid step: tile list, its members, launch shape.
struct BatchLaunch {
    const int64_t *begin;   // device: first tile of member k (k < nsims), ascending
    const TileSim *table;   // device: the members
    int nsims;
    int64_t tile0;          // the first member's first tile
    int64_t ntiles;         // tiles of these members
    int parity;             // batch steps since the table was built, mod 2
    int threads;            // threads per block (64, 128 or 256: 1, 2 or 4 tiles), 0: default
    int64_t blocks;         // 0: one block per tile; > 0: persistent walk
    hipStream_t stream;
    bool walls;             // some member of the batch has plates (the kernel variant)
    int64_t bytes;          // one population buffer of these members together, whole lines
};
hipError_t launch_multi_step(int lat, int storage, int eq, int fo, const BatchLaunch &bl);
// plates: emission tables, the row sums of a state no step produced, and the
// step of a grid between plates
hipError_t launch_wall_setup(int lat, int eq, const double *theta, const double *uw, int64_t ny,
                             double *e, hipStream_t stream);
hipError_t launch_wall_mass(int lat, int storage, const void *A, const GridDims &gd,
                            const StepCoef &co, const LaunchCfg &lc);
hipError_t launch_wall_step(int lat, int storage, int eq, int fo, const void *A, void *B,
                            const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                            const LaunchCfg &lc);

// Per-lattice / per-storage pieces, each explicitly instantiated in its own
// translation unit (step_*.hip, aux_*.hip) so that the build parallelises.
template <int LAT, class S>
hipError_t launch_step_ls(int eq, int fo, const void *A, void *B, const GridDims &gd,
                          const ForceDesc &fd, const StepCoef &co, const LaunchCfg &lc);
template <int LAT, class S>
hipError_t launch_multi_step_ls(int eq, int fo, const BatchLaunch &bl);
template <int LAT, class S>
hipError_t launch_wall_step_ls(int eq, int fo, const void *A, void *B, const GridDims &gd,
                               const ForceDesc &fd, const StepCoef &co, const LaunchCfg &lc);
template <int LAT, class S>
hipError_t launch_pattern_ls(const void *A, void *B, const GridDims &gd, const LaunchCfg &lc);
template <int LAT>
hipError_t launch_wall_setup_l(int eq, const double *theta, const double *uw, int64_t ny,
                               double *e, hipStream_t stream);
template <int LAT>
hipError_t launch_wall_mass_l(int storage, const void *A, const GridDims &gd, const StepCoef &co,
                              const LaunchCfg &lc);
template <int LAT, class S>
hipError_t launch_init_ls(int eq, int fo, const double *rho, const double *u, const double *theta,
                          void *A, const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                          const LaunchCfg &lc);
template <int LAT, class S>
hipError_t launch_rebuild_ls(int eq, int fo, const void *A, void *B, const GridDims &gd,
                             const ForceDesc &old_force, const ForceDesc &force,
                             const StepCoef &co, const LaunchCfg &lc);
template <int LAT, class S>
hipError_t launch_moments_ls(const void *A, double *rho, double *u, double *theta,
                             const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                             const LaunchCfg &lc);
template <int LAT, class S>
hipError_t launch_heat_flux_ls(int eq, int fo, const void *A, double *q, const GridDims &gd,
                               const ForceDesc &fd, const StepCoef &co, const LaunchCfg &lc);
template <int LAT>
hipError_t launch_totals_l(int storage, const void *A, double *partials, double *out_dev,
                           const GridDims &gd, const StepCoef &co, hipStream_t stream);

constexpr int TOTALS_BLOCKS = 512;  // fixed partition: results independent of launch shape

}  // namespace lbm
