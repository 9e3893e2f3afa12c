// HIP kernel templates of the gfx950 thermal LBM library.
//
//   step_kernel      one fused time step of eq. (lbm) (Li & Shan, arXiv:2302.04741,
//                    Sec. 2): pull streaming, moments, mid-point values,
//                    sigma-bar, Hermite equilibrium, Hermite force eq. (fi), BGK
//                    relaxation, store.  One thread per cell, SoA populations.
//   init_kernel      f~ = f0 - F/2 at step 0 (sigma = 0), written in pull layout.
//   moments_kernel   physical rho, u + g/2, theta in FP64.
//   heatflux_kernel  q = 1/2 sum_i f_i |xi_i - u|^2 (xi_i - u) of the physical f.
//   totals kernels   FP64 sums of the stored populations in a fixed order.
//
// Layout: populations are SoA planes, A[i*P + (z*ny + y)*px + x], rows padded
// to px = nx rounded up to 64 values (P = px*ny*nz), holding the deviations
// h_i = f~_i - w_i rho0 (scaled by 2^k_i for F16); the padding is never read.
// The stored state is post-collision ("pull" layout): the pre-collision value
// of velocity i at cell x is plane i at x - c_i (periodic).  A step reads every
// grid element of A exactly once (a permutation per plane) and writes every
// grid element of B exactly once, at the thread's own cell.
#pragma once

#include <algorithm>

#include "lbm_internal.h"

namespace lbm {

// ---------------------------------------------------------------------------
// storage codecs: S = stored type, T = arithmetic type; both sides are h_i
// ---------------------------------------------------------------------------
template <class S> struct ArithOf;
template <> struct ArithOf<double> { using type = double; };
template <> struct ArithOf<float> { using type = float; };
template <> struct ArithOf<__half> { using type = float; };

// Random bits of the F16 stochastic rounding.  One 32-bit key per (cell,
// step): the cell index and the step number combined linearly, then the
// 32-bit finalizer of MurmurHash3 (Appleby) to spread every input bit over
// the word.  From that key runs a 32-bit linear congruential sequence (Knuth's
// multiplier 6364136223846793005 reduced to its low word, odd increment), and
// the population of plane i takes word i of it, whole, as the seed of its
// conversion (half_sr reads its top 13 bits, the sequence's best ones).  Nothing
// depends on the launch shape, the batch, the other members or the order in
// which the planes are stored.
__device__ __forceinline__ uint32_t sr_key(uint32_t cell, uint32_t step)
{
    uint32_t h = cell * 0x9E3779B1u + step * 0x85EBCA77u;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}
// The sequence d words on, for d in [-N, N]: x -> mul[d + N] x + add[d + N]  (mod 2^32).
struct SrJump {
    static constexpr int N = 40;
    uint32_t mul[2 * N + 1], add[2 * N + 1];
    constexpr SrJump() : mul{}, add{}
    {
        constexpr uint32_t m = 0x4C957F2Du, a = 0x2545F491u;
        uint32_t inv = m;  // 1 / m mod 2^32: Newton's iteration doubles the correct bits
        for (int k = 0; k < 5; ++k) inv *= 2u - m * inv;
        mul[N] = 1u;
        for (int d = 1; d <= N; ++d) {
            mul[N + d] = mul[N + d - 1] * m;
            add[N + d] = add[N + d - 1] * m + a;
            mul[N - d] = mul[N - d + 1] * inv;
            add[N - d] = (add[N - d + 1] - a) * inv;
        }
    }
};
static constexpr SrJump SR_JUMP{};
struct SrStream {
    uint32_t x;  // word `at`
    int at;
    // word i (a compile-time index: planes stored in sequence cost one step each,
    // the four gaps in the order of the orbits a step with other constants)
    __device__ __forceinline__ uint32_t word(int i)
    {
        const int d = i - at + SrJump::N;
        x = x * SR_JUMP.mul[d] + SR_JUMP.add[d];
        at = i;
        return x;
    }
};

// float -> binary16 with stochastic rounding: a value between two
// neighbouring halves a < v < b rounds to b with probability (v - a)/(b - a),
// so the rounding error has zero mean whatever v is.  gfx950 does this in one
// instruction (v_cvt_sr_f16_f32).  Measured on an MI355X over 196,608 random
// values in the normal half range, it equals: add the seed's top 13 bits
// (seed >> 19) to the FP32 bit pattern (sign and magnitude) below the 13 bits
// binary16 drops, then drop them; in the subnormal half range it rounds
// stochastically at the subnormal spacing 2^-24 (the up-rounding frequency
// matched the fraction within sampling error on 32 values x 32,768 seeds).
__device__ __forceinline__ __half half_sr(float v, uint32_t seed)
{
    // the instruction writes the low half of its destination and keeps the
    // high half of the tied operand, here v's own register (no extra move)
    typedef _Float16 H2 __attribute__((ext_vector_type(2)));
    const H2 r = __builtin_amdgcn_cvt_sr_f16_f32(__builtin_bit_cast(H2, v), v, seed, false);
    return __builtin_bit_cast(__half, r.x);
}

// load/store convert between a stored value and the deviation h_i it stands
// for; load_scaled/store_scaled keep the factor scale<I>() the stored value
// carries (the fused step works on scaled values: see raw_sums, combo_pairs).
template <class L, class S> struct Codec {
    static constexpr bool STOCHASTIC = false;
    template <int I> static constexpr double scale() { return 1.0; }
    template <int I, class T> __device__ static __forceinline__ T load(S v) { return T(v); }
    template <int I, class T> __device__ static __forceinline__ S store(T h) { return S(h); }
    template <int I, class T> __device__ static __forceinline__ T load_scaled(S v) { return T(v); }
    template <int I, class T> __device__ static __forceinline__ S store_scaled(T h, SrStream &)
    {
        return S(h);
    }
};

// F16 deviations: stored value h_i 2^k_i, k_i = round(-log2 w_i).  The step
// stores with stochastic rounding (store_scaled); the initial state and the
// kernels off the step path round to nearest (store).
template <class L> struct Codec<L, __half> {
    static constexpr bool STOCHASTIC = true;
    template <int I> static constexpr double scale()
    {
        double s = 1.0;
        for (int e = 0; e < DevScale<L>::k(I); ++e) s *= 2.0;
        return s;
    }
    template <int I, class T> __device__ static __forceinline__ T load(__half v)
    {
        constexpr double inv = 1.0 / scale<I>();  // exact: a power of two
        return T(__half2float(v)) * T(inv);
    }
    template <int I, class T> __device__ static __forceinline__ __half store(T h)
    {
        constexpr double sc = scale<I>();
        return __float2half_rn(float(h * T(sc)));
    }
    template <int I, class T> __device__ static __forceinline__ T load_scaled(__half v)
    {
        return T(__half2float(v));
    }
    // stochastic rounding (half_sr), seeded by the plane's word of the cell's stream
    template <int I, class T> __device__ static __forceinline__ __half store_scaled(T h,
                                                                                   SrStream &rng)
    {
        return half_sr(float(h), rng.word(I));
    }
};

// ---------------------------------------------------------------------------
// pull gather: h_i = A[i][x - c_i (periodic)]
// ---------------------------------------------------------------------------
// Distinct column shifts (c_x, c_z) of the velocities that can cross a plate.
template <class L> struct WallShifts {
    int n, cx[L::Q], cz[L::Q], of[L::Q];
    constexpr WallShifts() : n(0), cx{}, cz{}, of{}
    {
        for (int i = 0; i < L::Q; ++i) {
            of[i] = -1;
            if (L::c(i, 1) == 0) continue;
            for (int k = 0; k < n; ++k)
                if (cx[k] == L::c(i, 0) && cz[k] == L::c(i, 2)) of[i] = k;
            if (of[i] < 0) {
                cx[n] = L::c(i, 0);
                cz[n] = L::c(i, 2);
                of[i] = n++;
            }
        }
    }
};
template <class L> constexpr WallShifts<L> WALL_SHIFTS{};

// sum of the weights of the velocities with c_y = k (or -k)
template <class L> constexpr double wall_weight(int k)
{
    double w = 0.0;
    for (int i = 0; i < L::Q; ++i)
        if (L::c(i, 1) == k) w += L::wshell(L::shell(i));
    return w;
}

// f(I) for every population, in the order in which combo_pairs hands them out
template <class L, class F> __device__ __forceinline__ void in_step_order(F &&f)
{
    f(std::integral_constant<int, 0>{});
    static_for<0, ORBITS<L>.n>([&](auto I) {
        constexpr int i = ORBITS<L>.rep[decltype(I)::value];
        constexpr Orbit<L> o(i);
        static_for<0, o.pairs()>([&](auto J) {
            constexpr int ip = o.plus(i, decltype(J)::value);
            f(std::integral_constant<int, ip>{});
            f(std::integral_constant<int, opposite<L>(ip)>{});
        });
    });
}

// The plates' partial sums of one node of row y: ps[c_y + 3] holds the sum of the
// node's stored deviations with that c_y, added in in_step_order (a step and the pass
// over a state that no step produced then give the same bits).
template <class L>
__device__ __forceinline__ void crossing_sums(const double (&ps)[7], int y, int ny, double rho0,
                                              double &below, double &above)
{
    below = above = 0.0;
    static_for<1, 4>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr double w = wall_weight<L>(k);
        if (y - k < 0) below += fma_t(w, rho0, ps[3 - k]);
        if (y + k >= ny) above += fma_t(w, rho0, ps[3 + k]);
    });
}

// A plate's densities over the columns (x, z) - (c_x, c_z): the columns' row sums,
// in order, over the plate's normalisation (side 0: the plate below, 1: above).
template <class L>
__device__ __forceinline__ void wall_densities_of(const WallDesc &wd, const GridDims &gd, int side,
                                                  int x, int z,
                                                  double (&rw)[WALL_SHIFTS<L>.n])
{
    const int64_t ncol = int64_t(gd.nx) * gd.nz;
    const double *rows = wd.part + wall_part_index(wd.par, side, 0, ncol, 0);
    const double norm = wd.e[side * (L::Q + 1) + L::Q], inv = 1.0 / norm;
    static_for<0, WALL_SHIFTS<L>.n>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cx = WALL_SHIFTS<L>.cx[k], cz = WALL_SHIFTS<L>.cz[k];
        const uint32_t xv = wrap_back(uint32_t(x), cx, uint32_t(gd.nx));
        const uint32_t zv = L::D == 3 ? wrap_back(uint32_t(z), cz, uint32_t(gd.nz)) : 0u;
        const int64_t col = int64_t(zv) * gd.nx + xv;
        double m = rows[col];
        if (gd.ny > 1) m += rows[ncol + col];
        if (gd.ny > 2) m += rows[2 * ncol + col];
        rw[k] = quotient(m, norm, inv);
    });
}

// Byte offsets of the pull sources x - c of one wavefront's cells: 7 per lane along
// x; y and z are uniform over the wavefront, so each row offset is a scalar.  A
// plane is < 4 GiB (checked at creation), so are all of them.
template <class L, class S> struct PullOffsets {
    uint32_t xs[7], ys[7], zs[7];
    __device__ __forceinline__ PullOffsets(const GridDims &gd, int x, int y, int z, bool pin)
    {
        const uint32_t pitch = uint32_t(gd.px) * uint32_t(sizeof(S));
        const uint32_t slab = pitch * uint32_t(gd.ny);
#pragma unroll
        for (int d = -3; d <= 3; ++d) {
            xs[d + 3] = wrap_back(uint32_t(x), d, uint32_t(gd.nx)) * uint32_t(sizeof(S));
            ys[d + 3] = wrap_back(uint32_t(y), d, uint32_t(gd.ny)) * pitch;
            zs[d + 3] = (L::D == 3) ? wrap_back(uint32_t(z), d, uint32_t(gd.nz)) * slab : 0u;
            if (pin) {  // uniform, but around branches some end up on the vector unit
                ys[d + 3] = __builtin_amdgcn_readfirstlane(ys[d + 3]);
                zs[d + 3] = __builtin_amdgcn_readfirstlane(zs[d + 3]);
            }
        }
    }
    __device__ __forceinline__ uint32_t row(int cy, int cz) const
    {
        return zs[cz + 3] + ys[cy + 3];
    }
};

// With plates (WALLS, the rows next to one), a population whose source lies behind
// the plate is the plate's emission into it, h_i = rw e_i - w_i rho0 with rw the
// plate's density over the source's column.  Which ones do depends on c_y alone:
// a uniform test for each c_y; the densities' and the other populations' loads are
// all in flight before the first emission is formed.  (A test, three dependent
// loads and a division for each slot made the row wavefronts of the plated 3 x 150
// FP64 channel twice as long as the others': 10.6 -> 6.1 us a step, 8254 -> 2671
// instructions in the kernel.)
template <class L, class S, class T, bool WALLS = false, int LD = BUF_DEFAULT>
__device__ __forceinline__ void gather(const S *__restrict__ A, const GridDims &gd, int x, int y,
                                       int z, T (&h)[L::Q], const WallDesc *wd = nullptr,
                                       double rho0 = 0.0)
{
    const PullOffsets<L, S> at(gd, x, y, z, WALLS);
    const PlaneWalk first(A, uint32_t(gd.P * int64_t(sizeof(S))));
    auto fetch = [&](auto I, PlaneWalk &planes) {
        constexpr int i = decltype(I)::value;
        constexpr int cx = L::c(i, 0), cy = L::c(i, 1), cz = L::c(i, 2);
        h[i] = Codec<L, S>::template load_scaled<i, T>(
            BufIO<S>::template load<LD>(planes.at(i), at.xs[cx + 3], at.row(cy, cz)));
    };
    if constexpr (!WALLS) {
        PlaneWalk planes = first;
        static_for<0, L::Q>([&](auto I) { fetch(I, planes); });
    } else {
        double rw[2][WALL_SHIFTS<L>.n] = {};
        if (y < 3) wall_densities_of<L>(*wd, gd, 0, x, z, rw[0]);
        if (y >= gd.ny - 3) wall_densities_of<L>(*wd, gd, 1, x, z, rw[1]);
        // every population of one c_y (upward ones can come from the plate below)
        auto rows = [&](auto CY, auto &&f) {
            static_for<0, L::Q>([&](auto I) {
                if constexpr (L::c(decltype(I)::value, 1) == decltype(CY)::value) f(I);
            });
        };
        auto behind = [&](int cy) { return y - cy < 0 || y - cy >= gd.ny; };
        static_for<-3, 4>([&](auto CY) {
            if (!behind(decltype(CY)::value)) {
                PlaneWalk planes = first;
                rows(CY, [&](auto I) { fetch(I, planes); });
            }
        });
        static_for<-3, 4>([&](auto CY) {
            constexpr int cy = decltype(CY)::value;
            constexpr int side = cy > 0 ? 0 : 1;
            if (cy != 0 && behind(cy))
                rows(CY, [&](auto I) {
                    constexpr int i = decltype(I)::value;
                    constexpr int k = cy != 0 ? WALL_SHIFTS<L>.of[i] : 0;
                    constexpr double sc = Codec<L, S>::template scale<i>();  // a power of two
                    constexpr double w = L::wshell(L::shell(i));
                    h[i] = T(sc * (rw[side][k] * wd->e[side * (L::Q + 1) + i] - w * rho0));
                });
        });
    }
}

// ---------------------------------------------------------------------------
// K1: fused step
// ---------------------------------------------------------------------------
// Largest block of the step kernel: FP64 arithmetic needs more than 128 VGPRs
// per lane, so its blocks stay at 256 threads (4 waves).
template <class S> constexpr int step_max_threads()
{
    return sizeof(typename ArithOf<S>::type) == 8 ? 256 : 1024;
}

// Launch shape of the step: threads per block, and the LDS bytes a block asks for
// (unused: they only limit how many blocks share a CU).
struct StepShape {
    int threads;
    unsigned lds;
};

// Default, measured.  FP64: 128 threads (D3Q39 256^3: +6%, D2Q37 1024^2: +4% over
// 256, which is its largest).  FP32 and F16: 256, except FP32 populations past the
// 256 MB memory-side cache by far (a buffer of 400 MB and more): there the rate
// falls with the wavefronts in flight, whose loads and stores open ever more
// places of the 78 plane streams at once, and the arithmetic needs few of them,
// so a CU gets 8 wavefronts, one block of 512 threads.  FP32 us a step, 8
// wavefronts against as many as the registers allow (256 threads): D3Q39 160^3
// 227 / 234, 224^3 614 / 657, 256^3 913 / 957 (1024 threads, 16 wavefronts: 942),
// D2Q37 2048^2 220 / 226, 3000^2 475 / 500; below that size it gains or loses 2%,
// and F16, with half the bytes a wavefront, loses (256^3 700 / 496); F16 of 1 GiB a
// buffer and more takes 512 threads unlimited (256^3 476 / 490, D2Q37 4096^2 441 /
// 458; below it is within 2% either way).  FP64 on D3Q39 from 1 GiB a buffer: 256
// threads and 8 wavefronts a CU (against 128 threads, 12 wavefronts: 160^3 452 / 459,
// 224^3 1280 / 1337, 256^3 1902 / 1934, 280^3 2527 / 2637, 320^3 3803 / 3856, 64x300x250
// 534 / 530; 256 threads unlimited 459, 1306, 1934, 2645, 3960); below it, and on D2Q37,
// within 2% either way.
constexpr int64_t STEP_LARGE_BYTES = 400 * MIB;
constexpr unsigned STEP_LDS_PER_CU = 160u << 10;

// Grids of a few wavefronts a SIMD (1024 SIMDs on the chip), both buffers cached:
// what counts there is how the blocks spread over the CUs in one round, and the
// widths measured best follow the number of wavefronts (us a step, against 256
// threads, 128 for FP64):
//   up to 256: 64 threads, a wavefront a CU (FP64 64^2 3.8 / 4.1, 12^3 4.4 / 5.4,
//     FP32 100x128 3.8 / 4.3, plated 3 x 150 FP64 10.6 / 12.1);
//   FP64 to 4096: 64 (256^2 9.3 / 10.5, 40^3 8.7 / 9.9, 64^3 24 / 35);
//   FP32 512-1280: 512 (200^2 5.4 / 6.0, 250x300 7.0 / 8.9, 33^3 5.6 / 6.2); F16 on
//     D2Q37 1100-2048: 512 (320^2 6.6 / 7.3);
//   FP32 to 2048: 1024 on D2Q37 (320^2 8.4 / 9.6), 64 on D3Q39 (40^3 7.0 / 8.0);
//   FP32 and F16 to 4096 (F16 on D3Q39 from 3072): 1024, one block a CU at most
//     (FP32 400x300 8.6 / 10.7, 512^2 12.9 / 14.9, F16 512^2 8.3 / 10.5, 64^3 8.1 / 11.2);
//   beyond, FP32 on D2Q37: 512 (600^2 17.1 / 18.5, 700^2 23.3 / 24.8).
// 0: no preference.
template <int LAT, class S> inline int small_grid_threads(int64_t waves)
{
    if (waves <= 256) return 64;
    if (sizeof(S) == 8) return waves <= 4096 ? 64 : 0;
    if (sizeof(S) == 4) {
        if (waves <= 512) return 0;
        if (waves <= 1280) return 512;
        if (waves <= 2048) return LAT == 0 ? 1024 : 64;
        if (waves <= 4096) return 1024;
        return LAT == 0 ? 512 : 0;
    }
    if (LAT == 0 && waves > 1100 && waves <= 2048) return 512;
    return waves > (LAT == 0 ? 2048 : 3072) && waves <= 4096 ? 1024 : 0;
}

template <int LAT, class S>
inline StepShape step_shape(int64_t buffer_bytes, int64_t waves, int threads)
{
    const bool large = sizeof(S) == 4 && buffer_bytes >= STEP_LARGE_BYTES;
    int bx = threads;
    if (bx <= 0 && buffer_bytes <= STEP_CACHED_BYTES) bx = small_grid_threads<LAT, S>(waves);
    const bool wide = large || (sizeof(S) == 2 && buffer_bytes >= 1024 * MIB);
    const bool large64 = LAT == 1 && sizeof(S) == 8 && buffer_bytes >= 1024 * MIB;
    if (bx <= 0) bx = sizeof(S) == 8 ? (large64 ? 256 : 128) : (wide ? 512 : 256);
    bx = bx < step_max_threads<S>() ? bx : step_max_threads<S>();
    const bool limit = (large || large64) && (bx == 256 || bx == 512);
    return StepShape{bx, limit ? STEP_LDS_PER_CU * unsigned(bx) / 512u : 0u};
}

// Cache policy for a population buffer of T bytes (whole lines), measured from
// T = 10 MB to 5 GB.  Both buffers fit the memory-side cache up to 128 MiB each.
// Past it the kept part W is what the cache holds beside the traffic: measured best
// between 0.5 and 0.6 T up to T = 300 MB, and flat from 160 to 240 MB above.  D3Q39
// FP64 between 250 and 700 MB gains from nt loads throughout and W = 240 MB
// (129x95x110 170 us against 178, 116^3 180 / 191, 126^3 225 / 228; 136^3, 785 MB,
// loses, 306 / 303; the others lose everywhere).
struct StepPolicy {
    Policy policy;
    double keep;  // share of the sweep, at its end, whose stores are kept; 0: no reversal
};
template <int LAT, class S> inline StepPolicy step_policy(int64_t T)
{
    if (T <= STEP_CACHED_BYTES) return {Policy::RESIDENT, 0.0};
    const double t = double(T);
    if (LAT == 1 && sizeof(S) == 8 && t > 250e6 && t <= 700e6)
        return {Policy::STREAM_NT, std::min(0.57, 240e6 / t)};
    return {Policy::STREAM, std::min(0.55, 200e6 / t)};
}
// The order of one step's sweep over its work items (one argument of the kernels:
// each costs the host a share of the launch).
struct Sweep {
    int64_t first;  // a batch: first tile of the launch
    int64_t keep;   // first item, in the order of the sweep, whose stores are kept
    int cur;        // buffer the step reads (a batch: flips each member's own)
    int backwards;  // odd steps of a policy that keeps: last item first
};
inline Sweep sweep_of(const StepPolicy &sp, int64_t items, int cur, int64_t first = 0)
{
    if (sp.keep <= 0) return {first, items, cur, 0};
    return {first, items - int64_t(double(items) * sp.keep), cur, cur};
}
// Bytes of one population buffer in whole 128-byte lines.
template <int LAT, class S> inline int64_t buffer_lines_bytes(const GridDims &gd)
{
    return int64_t(Lattice<LAT>::Q) * gd.ny * gd.nz *
           ((int64_t(gd.nx) * int64_t(sizeof(S)) + 127) / 128 * 128);
}

// The fused update of one cell (x, y, z): gather, moments, equilibrium, stress,
// force, relaxation, store.  y and z must be uniform over the wavefront.
// `step` is the step number (the state read is after `step` steps): with F16
// storage it keys the stochastic rounding of every value stored.
//
// Bound by memory on large grids and by the length of its instruction stream on
// small ones (one wavefront a SIMD or fewer: each instruction is latency).  The
// stream is 938 instructions for D2Q37 FP32 (535 vector, 325 scalar) and 1058 for
// D3Q39 FP32 (586, 388); with the pair-by-pair evaluation, looping wraps and a
// resource made for each access it was 1860 and 2211.  Step of D2Q37 64^2 FP64:
// 5.7 -> 4.7 us, of the plated 3 x 150 channel 15.3 -> 12.2 us, of D2Q37 256^2 FP32
// 8.4 -> 7.9 us; at 1024^2 and above the memory time hid most of it already.
template <int LAT, class S, int EQ, int FO, Policy P, bool WALLS = false>
__device__ __forceinline__ void step_cell(const S *__restrict__ A, S *__restrict__ B,
                                          const GridDims &gd, const ForceDesc &fd,
                                          const StepCoef &co, int x, int y, int z,
                                          uint32_t step, const WallDesc *wd = nullptr)
{
    using L = Lattice<LAT>;
    using T = typename ArithOf<S>::type;
    const int64_t row = int64_t(z) * gd.ny + y;  // uniform
    const int64_t rowbase = row * gd.px;          // padded population row
    const int64_t cell = row * gd.nx + x;         // dense field index

    // h holds the deviations as stored, times Codec::scale<i>() (1 unless the
    // storage is reduced-precision); the sums and the pair terms take the
    // scale through their constants, so no value is rescaled on the way.
    using C = Codec<L, S>;
    SrStream rng{C::STOCHASTIC ? sr_key(uint32_t(cell), step) : 0u, 0};
    T h[L::Q];
    gather<L, S, T, WALLS, CacheBits<P>::load>(A, gd, x, y, z, h, wd, co.rho0);
    T g[3];
    load_force<T, T, L::D>(fd, gd, x, y, z, cell, g);

    const RawSums<T> rs = raw_sums<L, T, C>(h);
    CellState<T> cs;
    finish_moments<L, T, FO == 4>(rs, g, co, cs);

    // h* = h + om (f0 - f) + cf F with f0 - f = w drho + (f0 - w rho) - h, so
    // h* = (1 - om) h + [om w drho + om (f0 - w rho) + cf F]; the bracket is what
    // combo_pairs returns with base = om drho (even +- odd part), each population one
    // fma of it (1 - om is exact for om = 1/tau^ in [1/2, 2]).  Every term is a small
    // deviation, so the rounding stays at the size of h.
    const T om = cs.om;
    const T omc = T(1) - om;
    const uint32_t xo = uint32_t(x) * uint32_t(sizeof(S));
    const uint32_t ro = uint32_t(rowbase) * uint32_t(sizeof(S));
    PlaneWalk planes(B, uint32_t(gd.P * int64_t(sizeof(S))));
    // with plates: the partial sums of the state written here (the slots whose
    // next move crosses a plate, as stored), for the next step's emission; kept by
    // c_y, which decides what crosses
    double ps[7] = {};
    auto account = [&](auto II, S stored) {
        if constexpr (WALLS) {
            constexpr int i = decltype(II)::value;
            constexpr int cy = L::c(i, 1);
            if constexpr (cy != 0)
                ps[cy + 3] += Codec<L, S>::template load<i, double>(stored);
        }
    };
    combo_pairs<L, T, EQ, FO, C>(cs, om, cs.cf, om * cs.drho, [&](auto IP, auto IM, T ev, T od) {
        constexpr int ip = decltype(IP)::value;
        constexpr int im = decltype(IM)::value;
        auto relaxed = [&](T hi, T sign_od) { return fma_t(omc, hi, ev + sign_od); };
        const S sp = C::template store_scaled<ip, T>(relaxed(h[ip], od), rng);
        constexpr int ST = CacheBits<P>::store;
        BufIO<S>::template store<ST>(sp, planes.at(ip), xo, ro);
        account(IP, sp);
        if constexpr (im >= 0) {
            const S sm = C::template store_scaled<im, T>(relaxed(h[im], -od), rng);
            BufIO<S>::template store<ST>(sm, planes.at(im), xo, ro);
            account(IM, sm);
        }
    });
    if constexpr (WALLS) {
        const int64_t ncol = int64_t(gd.nx) * gd.nz;
        const int64_t col = int64_t(z) * gd.nx + x;
        const int y1 = gd.ny > 3 ? gd.ny - 3 : 0;  // first row of the top plate's sums
        double below, above;
        crossing_sums<L>(ps, y, gd.ny, co.rho0, below, above);
        if (y < 3) wd->part[wall_part_index(wd->par ^ 1, 0, y, ncol, col)] = below;
        if (y >= y1) wd->part[wall_part_index(wd->par ^ 1, 1, y - y1, ncol, col)] = above;
    }
}

// Step counter of a handle (F16 storage only): a pair of words; a step that
// reads buffer `cur` reads the step number from ctr[cur] and one lane writes
// the next number to ctr[cur ^ 1], which the next step reads.  The launches
// of a step loop, eager or captured in a graph, so carry the count without
// the host.
template <class S> __device__ __forceinline__ uint32_t step_number(const uint32_t *ctr, int cur)
{
    if constexpr (Codec<Lattice<0>, S>::STOCHASTIC) return __builtin_amdgcn_readfirstlane(ctr[cur]);
    else return 0u;
}
template <class S>
__device__ __forceinline__ void advance_step_number(uint32_t *ctr, int cur, uint32_t step,
                                                    bool writer)
{
    if constexpr (Codec<Lattice<0>, S>::STOCHASTIC) {
        if (writer) ctr[cur ^ 1] = step + 1u;
    }
}

// Work split: one wavefront updates 64 consecutive cells of one row
// (wavefronts numbered row by row, ceil(nx/64) per row); a block is any run of
// consecutive wavefronts, so blocks may straddle rows and none is left partly
// empty at the end of a row.  The wavefront's row is a scalar.
__device__ __forceinline__ bool wave_cell(const GridDims &gd, uint32_t wave, int &x, int &y,
                                          int &z)
{
    const uint32_t k = (uint32_t(gd.nx) + 63u) >> 6;  // wavefronts per row
    const uint32_t row = divu(gd.by_wpr, wave);
    if (row >= uint32_t(gd.ny) * uint32_t(gd.nz)) return false;
    x = int((wave - row * k) * 64u + (threadIdx.x & 63u));
    const uint32_t zz = divu(gd.by_ny, row);
    y = int(row - zz * uint32_t(gd.ny));
    z = int(zz);
    return x < gd.nx;
}

// The wavefront's number in a launch of whole wavefronts.
__device__ __forceinline__ uint32_t block_wave()
{
    return __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
}

// Wavefronts per SIMD the compiler must leave room for: FP32 arithmetic fits
// five without spills; FP64 needs three (168 registers; left free, the D3Q39
// schedule takes 170).
template <class S> constexpr int step_min_waves() { return sizeof(S) == 8 ? 3 : 5; }

// Between two inlined cell updates: left to itself the compiler forms the scalars of
// both before the branch between them, more than the scalar registers hold (106 used
// and spilled against 55).
__device__ __forceinline__ void keep_apart() { asm volatile("" ::: "memory"); }

// The block's place on the grid: odd steps sweep it backwards (see Policy).
__device__ __forceinline__ uint32_t swept_block(int backwards)
{
    return backwards ? gridDim.x - 1u - blockIdx.x : blockIdx.x;
}

template <int LAT, class S, int EQ, int FO, Policy P>
__global__ void __launch_bounds__(step_max_threads<S>())
    __attribute__((amdgpu_waves_per_eu(step_min_waves<S>(), 8)))
    step_kernel(const S *__restrict__ A, S *__restrict__ B, GridDims gd, ForceDesc fd,
                StepCoef co, uint32_t *ctr, Sweep sw)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(
        swept_block(sw.backwards) * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const uint32_t step = step_number<S>(ctr, sw.cur);
    advance_step_number<S>(ctr, sw.cur, step, wave == 0 && threadIdx.x == 0);
    int x, y, z;
    if (!wave_cell(gd, wave, x, y, z)) return;
    if (P != Policy::RESIDENT && blockIdx.x >= uint32_t(sw.keep)) {  // the sweep's last blocks (see Policy)
        keep_apart();
        step_cell<LAT, S, EQ, FO, P == Policy::RESIDENT ? P : Policy::KEEP>(A, B, gd, fd, co, x, y,
                                                                            z, step);
    } else {
        step_cell<LAT, S, EQ, FO, P>(A, B, gd, fd, co, x, y, z, step);
    }
}

// K7 (diagnostic): the memory traffic of K1 alone -- every population read
// from its pull source and written unchanged at the cell's own slot of the
// other buffer, K1's work split, no arithmetic.  Every pass sweeps forward and, above
// the cached size, streams every store: the rate of K1's loads and stores from and to
// memory.  K1 passes it where the memory-side cache serves part of its reads (see Policy).
template <int LAT, class S, Policy P>
__global__ void __launch_bounds__(step_max_threads<S>())
    pattern_kernel(const S *__restrict__ A, S *__restrict__ B, GridDims gd)
{
    using L = Lattice<LAT>;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) +
                                                         (threadIdx.x >> 6));
    int x, y, z;
    if (!wave_cell(gd, wave, x, y, z)) return;
    S h[L::Q];
    gather<L, S, S, false, CacheBits<P>::load>(A, gd, x, y, z, h);
    const uint32_t xo = uint32_t(x) * uint32_t(sizeof(S));
    const uint32_t ro = uint32_t((int64_t(z) * gd.ny + y) * gd.px) * uint32_t(sizeof(S));
    PlaneWalk planes(B, uint32_t(gd.P * int64_t(sizeof(S))));
    static_for<0, L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        BufIO<S>::template store<CacheBits<P>::store>(h[i], planes.at(i), xo, ro);
    });
}

// K1c: the step of a grid between plates, in one launch: K1's work split;
// the wavefronts of the rows next to a plate (y < 3 or y >= ny - 3, a uniform
// test) take the plates' emission in place of the sources behind them and
// write the partial sums of the state they produce.
template <int LAT, class S, int EQ, int FO, Policy P>
__global__ void __launch_bounds__(step_max_threads<S>())
    wall_step_kernel(const S *__restrict__ A, S *__restrict__ B, GridDims gd, ForceDesc fd,
                     StepCoef co, WallDesc wd, uint32_t *ctr, int cur)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) +
                                                         (threadIdx.x >> 6));
    const uint32_t step = step_number<S>(ctr, cur);
    advance_step_number<S>(ctr, cur, step, wave == 0 && threadIdx.x == 0);
    int x, y, z;
    if (!wave_cell(gd, wave, x, y, z)) return;
    if (y < 3 || y >= gd.ny - 3)
        step_cell<LAT, S, EQ, FO, P, true>(A, B, gd, fd, co, x, y, z, step, &wd);
    else
        step_cell<LAT, S, EQ, FO, P>(A, B, gd, fd, co, x, y, z, step);
}

// ---------------------------------------------------------------------------
// K1b: multi-grid step.  Several simulations (same lattice, storage and
// orders; any grid sizes, relaxation times and forces) advance one step in one
// launch.  The work is a list of tiles -- one tile is 64 consecutive cells of
// one grid row of one simulation, updated by one wavefront -- and wavefront w
// of the launch takes tiles w, w + W, ... (W wavefronts launched): with one
// wavefront per tile the hardware balances uneven members; with fewer blocks
// the grid is persistent and every wavefront exits after at most
// ceil(ntiles / W) tiles.  Each cell is updated by exactly one thread with the
// arithmetic of the single-grid step, so no result depends on the launch shape
// or on the other members.  The WALLS variant (launched when some member has
// plates) updates the rows next to a member's plates as K1c does; periodic
// batches keep the variant without that code.
// ---------------------------------------------------------------------------
template <int LAT, class S, int EQ, int FO, Policy P, bool WALLS>
__global__ void __launch_bounds__(256)
    multi_step_kernel(const int64_t *__restrict__ begin, const TileSim *__restrict__ sims,
                      int nsims, int64_t ntiles, Sweep sw)
{
    const int64_t nw = int64_t(gridDim.x) * (blockDim.x >> 6);
    int64_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    for (; w < ntiles; w += nw) {
        const int64_t t = sw.first + (sw.backwards ? ntiles - 1 - w : w);
        // the simulation owning tile t: last k with begin[k] <= t (uniform)
        int lo = 0, hi = nsims - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (begin[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const TileSim &sd = sims[lo];
        // tiles of one simulation number fewer than its cells (< 2^32)
        const uint32_t k = uint32_t(t - begin[lo]);
        const uint32_t cx = uint32_t(sd.chunks_x);
        const uint32_t row = divu(sd.gd.by_wpr, k);  // chunks_x = ceil(nx / 64)
        const uint32_t xc = k - row * cx;
        const uint32_t zz = divu(sd.gd.by_ny, row);
        const int y = int(row - zz * uint32_t(sd.gd.ny)), z = int(zz);
        const int x = int(xc * 64u + (threadIdx.x & 63u));
        const int c = sd.cur ^ sw.cur;
        const S *A = static_cast<const S *>(sd.pop[c]);
        S *B = static_cast<S *>(const_cast<void *>(sd.pop[c ^ 1]));
        // the member's step number; its first tile's wavefront advances it
        const uint32_t step = step_number<S>(sd.ctr, c);
        advance_step_number<S>(sd.ctr, c, step, k == 0 && (threadIdx.x & 63u) == 0);
        if (x >= sd.gd.nx) continue;
        if constexpr (WALLS) {
            // a member between plates: its rows next to a plate as in K1c
            if (sd.wd.on && (y < 3 || y >= sd.gd.ny - 3)) {
                WallDesc wd = sd.wd;
                wd.par = c;
                step_cell<LAT, S, EQ, FO, P, true>(A, B, sd.gd, sd.fd, sd.co, x, y, z, step,
                                                   &wd);
                continue;
            }
        }
        if (!WALLS && P != Policy::RESIDENT && w >= sw.keep) {  // the sweep's last tiles
            keep_apart();
            step_cell<LAT, S, EQ, FO, WALLS || P == Policy::RESIDENT ? P : Policy::KEEP>(
                A, B, sd.gd, sd.fd, sd.co, x, y, z, step);
        } else {
            step_cell<LAT, S, EQ, FO, P>(A, B, sd.gd, sd.fd, sd.co, x, y, z, step);
        }
    }
}

// ---------------------------------------------------------------------------
// kernels off the step path: one thread per cell, the step's work split in blocks
// of 256 threads, arithmetic in the storage's own
// precision (FP64 for FP64 storage, FP32 for FP32 and F16 storage; the
// fields handed in and out stay FP64)
// ---------------------------------------------------------------------------
// Each comes in two variants, without plates and with (WALLS: launched for a handle
// that has them; every row then takes the gather that tests for a plate).  One
// kernel choosing between two gathers had its 39 loads in two branches and waited
// for some of them one by one.
// ---------------------------------------------------------------------------
// K2: initial state f~ = f0 - F/2 (sigma = 0), stored as h = f~ - w rho0 and
// scattered so that the pull gather of the first step finds h_i(x) at
// A[i][x - c_i].  Bound by memory, by its shifted stores above all: default
// (write-back) stores, since lines are completed by neighbouring wavefronts
// (streamed or written through they cost 20-120% more).
// ---------------------------------------------------------------------------
template <class L, class S, class T, int EQ, int FO, bool WALLS>
__device__ __forceinline__ void scatter_initial(const CellState<T> &cs, S *__restrict__ A,
                                                const GridDims &gd, int x, int y, int z)
{
    const int64_t row = int64_t(z) * gd.ny + y;
    // the slot the first step pulls velocity i of this cell from is x - c_i
    const PullOffsets<L, S> at(gd, x, y, z, true);
    const uint32_t xo = uint32_t(x) * uint32_t(sizeof(S));
    const uint32_t ro = uint32_t(row * gd.px) * uint32_t(sizeof(S));
    PlaneWalk planes(A, uint32_t(gd.P * int64_t(sizeof(S))));
    constexpr int FOI = FO == 4 ? 3 : FO;  // sigma = 0 at the start
    // h = w (rho - rho0) + (f0 - w rho) - F/2
    combo_pairs<L, T, EQ, FOI>(cs, T(1), T(-0.5), T(0), [&](auto IP, auto IM, T ev, T od) {
        constexpr double w = L::wshell(L::shell(decltype(IP)::value));
        auto put = [&](auto II, T v) {
            constexpr int i = decltype(II)::value;
            constexpr int cx = L::c(i, 0), cy = L::c(i, 1), cz = L::c(i, 2);
            const S sv = Codec<L, S>::template store<i, T>(v);
            const RsrcWords plane = planes.at(i);
            if constexpr (cy != 0 && WALLS) {
                // with plates: a population arriving from behind a plate has no
                // slot (the plate emits it); one about to stream into a plate
                // stays in its own node's slot
                if (y + cy < 0 || y + cy >= gd.ny)
                    BufIO<S>::template store<BUF_DEFAULT>(sv, plane, xo, ro);
                if (y - cy < 0 || y - cy >= gd.ny) return;
            }
            BufIO<S>::template store<BUF_DEFAULT>(sv, plane, at.xs[cx + 3], at.row(cy, cz));
        };
        put(IP, fma_t(T(w), cs.drho, ev + od));
        if constexpr (decltype(IM)::value >= 0) put(IM, fma_t(T(w), cs.drho, ev - od));
    });
}

template <int LAT, class S, int EQ, int FO, bool WALLS>
__global__ void __launch_bounds__(512)
    init_kernel(const double *__restrict__ rho, const double *__restrict__ u,
                const double *__restrict__ theta, S *__restrict__ A, GridDims gd, ForceDesc fd,
                StepCoef co)
{
    using L = Lattice<LAT>;
    using T = typename ArithOf<S>::type;
    int x, y, z;
    if (!wave_cell(gd, block_wave(), x, y, z)) return;
    const int64_t N = gd.N;
    const int64_t cell = (int64_t(z) * gd.ny + y) * gd.nx + x;

    T g[3];
    load_force<T, T, L::D>(fd, gd, x, y, z, cell, g);
    CellState<T> cs;
    cs.rho = T(rho[cell]);
    cs.drho = T(rho[cell] - co.rho0);  // the deviation rounded once
    cs.th = T(theta[cell]);
    for (int a = 0; a < 3; ++a) {
        cs.ub[a] = (a < L::D) ? T(u[int64_t(a) * N + cell]) : T(0);
        cs.g[a] = g[a];
        for (int b = 0; b < 3; ++b) cs.sig[a][b] = T(0);
    }
    scatter_initial<L, S, T, EQ, FO, WALLS>(cs, A, gd, x, y, z);
}

// K2b: the state rebuilt for another force before the first step, in one pass: the
// moments of the state in A under the old force, f~ = f0 - F/2 with the new one
// scattered into B.  Through FP64 fields in between (K3, then K2) it moves 80 bytes a
// cell more: D3Q39 FP32 160^3 314 us, in one pass 259 (256^3: 1213 / 980).  The
// values are the same: K3
// writes T widened to FP64, K2 narrows it back.
template <int LAT, class S, int EQ, int FO>
__global__ void __launch_bounds__(512)
    rebuild_kernel(const S *__restrict__ A, S *__restrict__ B, GridDims gd, ForceDesc old_force,
                   ForceDesc force, StepCoef co, uint32_t *ctr, int cur)
{
    using L = Lattice<LAT>;
    using T = typename ArithOf<S>::type;
    using C = Codec<L, S>;
    const uint32_t wave = block_wave();
    // the step number goes with the state
    if (C::STOCHASTIC && wave == 0 && threadIdx.x == 0) ctr[cur ^ 1] = ctr[cur];
    int x, y, z;
    if (!wave_cell(gd, wave, x, y, z)) return;
    const int64_t cell = (int64_t(z) * gd.ny + y) * gd.nx + x;
    CellState<T> cs;
    {
        T h[L::Q], g[3];
        gather<L, S, T>(A, gd, x, y, z, h);
        load_force<T, T, L::D>(old_force, gd, x, y, z, cell, g);
        const RawSums<T> rs = raw_sums<L, T, C>(h);
        finish_moments<L, T, false>(rs, g, co, cs);
    }
    T g[3];
    load_force<T, T, L::D>(force, gd, x, y, z, cell, g);
    cs.drho = T(double(cs.rho) - co.rho0);
    for (int a = 0; a < 3; ++a) cs.g[a] = g[a];
    scatter_initial<L, S, T, EQ, FO, false>(cs, B, gd, x, y, z);
}

// ---------------------------------------------------------------------------
// K3: physical moments rho, u + g/2, theta of the state
// ---------------------------------------------------------------------------
template <int LAT, class S, bool WALLS>
__global__ void __launch_bounds__(256)
    moments_kernel(const S *__restrict__ A, double *__restrict__ rho, double *__restrict__ u,
                   double *__restrict__ theta, GridDims gd, ForceDesc fd, StepCoef co,
                   WallDesc wd)
{
    using L = Lattice<LAT>;
    using T = typename ArithOf<S>::type;
    using C = Codec<L, S>;
    int x, y, z;
    if (!wave_cell(gd, block_wave(), x, y, z)) return;
    const int64_t N = gd.N;
    const int64_t cell = (int64_t(z) * gd.ny + y) * gd.nx + x;
    T h[L::Q];  // as stored (scaled for F16): raw_sums takes the scale out
    gather<L, S, T, WALLS>(A, gd, x, y, z, h, &wd, co.rho0);
    T g[3];
    load_force<T, T, L::D>(fd, gd, x, y, z, cell, g);
    const RawSums<T> rs = raw_sums<L, T, C>(h);
    CellState<T> cs;
    finish_moments<L, T, false>(rs, g, co, cs);
    if (rho) rho[cell] = double(cs.rho);
    if (theta) theta[cell] = double(cs.th);
    if (u)
        for (int a = 0; a < L::D; ++a) u[int64_t(a) * N + cell] = double(cs.ub[a]);
}

// ---------------------------------------------------------------------------
// K5: heat flux q = 1/2 sum_i f_i |xi_i - u|^2 (xi_i - u) of the physical
// distribution f = f0 + cf (f~ - f0 + F/2).  With the equilibrium of order
// N >= 3 the rule reproduces the Maxwellian's moments up to order N + 3, so
// sum_i f0_i |c_i|^2 c_i (c = xi - u) is the Maxwellian's third central
// moment, zero: q = 1/2 sum_i (f_i - f0_i) |c_i|^2 c_i, a sum of small terms
//   f - f0 = cf (h - w drho) - cf (f0 - w rho) + (cf/2) F.
// For N = 2 the equilibrium's own part is added, sum_i f0_i |c_i|^2 c_i =
// -rho u (D + 2 + |u|^2) (the rule's moments to degree 3) + sum_i (f0 - w rho)_i |c_i|^2 c_i.
// ---------------------------------------------------------------------------
template <int LAT, class S, int EQ, int FO, bool WALLS>
__global__ void __launch_bounds__(256)
    heatflux_kernel(const S *__restrict__ A, double *__restrict__ q, GridDims gd, ForceDesc fd,
                    StepCoef co, WallDesc wd)
{
    using L = Lattice<LAT>;
    using T = typename ArithOf<S>::type;
    using C = Codec<L, S>;
    int x, y, z;
    if (!wave_cell(gd, block_wave(), x, y, z)) return;
    const int64_t N = gd.N;
    const int64_t cell = (int64_t(z) * gd.ny + y) * gd.nx + x;
    T h[L::Q];
    gather<L, S, T, WALLS>(A, gd, x, y, z, h, &wd, co.rho0);
    T g[3];
    load_force<T, T, L::D>(fd, gd, x, y, z, cell, g);
    const RawSums<T> rs = raw_sums<L, T, C>(h);
    CellState<T> cs;
    finish_moments<L, T, FO == 4>(rs, g, co, cs);
    static_for<0, L::Q>([&](auto I) {  // the deviations themselves (exact: powers of two)
        constexpr int i = decltype(I)::value;
        constexpr double inv = 1.0 / C::template scale<i>();
        if constexpr (inv != 1.0) h[i] *= T(inv);
    });
    const T cf = cs.cf;
    T qa[3] = {T(0), T(0), T(0)};
    auto acc = [&](auto II, T d) {
        constexpr int i = decltype(II)::value;
        T cv[3], cc = T(0);
        for (int a = 0; a < L::D; ++a) {
            cv[a] = T(L::R * double(L::c(i, a))) - cs.ub[a];
            cc += cv[a] * cv[a];
        }
        for (int a = 0; a < L::D; ++a) qa[a] += d * cc * cv[a];
    };
    // h - w drho first: both are of the size of drho (with rho0 = 0, of rho)
    combo_pairs<L, T, EQ, FO>(cs, -cf, T(0.5) * cf, T(0), [&](auto IP, auto IM, T ev, T od) {
        constexpr int ip = decltype(IP)::value;
        constexpr int im = decltype(IM)::value;
        constexpr double w = L::wshell(L::shell(ip));
        acc(IP, fma_t(cf, fma_t(T(-w), cs.drho, h[ip]), ev + od));
        if constexpr (im >= 0) acc(IM, fma_t(cf, fma_t(T(-w), cs.drho, h[im]), ev - od));
    });
    if constexpr (EQ == 2) {
        T u2 = T(0);
        for (int a = 0; a < L::D; ++a) u2 += cs.ub[a] * cs.ub[a];
        for (int a = 0; a < L::D; ++a) qa[a] -= cs.rho * cs.ub[a] * (T(L::D + 2) + u2);
        combo_pairs<L, T, 2, 1>(cs, T(1), T(0), T(0), [&](auto IP, auto IM, T ev, T od) {
            acc(IP, ev + od);
            if constexpr (decltype(IM)::value >= 0) acc(IM, ev - od);
        });
    }
    for (int a = 0; a < L::D; ++a) q[int64_t(a) * N + cell] = double(T(0.5) * qa[a]);
}

// ---------------------------------------------------------------------------
// K6: plates.  wall_setup_kernel: e_i = f0_i(1, (U_w, 0, 0), theta_w) of both
// plates in FP64 and the normalisation sum_{i entering} min(|c_iy|, ny) e_i.
// wall_mass_kernel: per (x, z) column, plate and row next to the plate, the
// mass of the crossing slots (populations about to stream into the plate),
// for a state no step produced (after initialisation or an external write);
// a step writes the same sums, bit for bit, for the state it produces.  The plate's density
// rw over a column, at which it re-emits exactly what it absorbs, is the sum
// of its rows' sums over the normalisation.
// ---------------------------------------------------------------------------
template <int LAT, int EQ>
__global__ void __launch_bounds__(64)
    wall_setup_kernel(double th_b, double th_t, double u_b, double u_t, int64_t ny,
                      double *__restrict__ e)
{
    using L = Lattice<LAT>;
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    for (int side = 0; side < 2; ++side) {
        CellState<double> cs;
        cs.rho = 1.0;
        cs.drho = 0.0;
        cs.th = side == 0 ? th_b : th_t;
        for (int a = 0; a < 3; ++a) {
            cs.ub[a] = 0.0;
            cs.g[a] = 0.0;
            for (int b = 0; b < 3; ++b) cs.sig[a][b] = 0.0;
        }
        cs.ub[0] = side == 0 ? u_b : u_t;
        cs.om = 0.0;
        cs.cf = 0.0;
        double *es = e + side * (L::Q + 1);
        // f0 = w rho + (f0 - w rho); the bracket is what combo_pairs returns
        combo_pairs<L, double, EQ, 1>(cs, 1.0, 0.0, 0.0, [&](auto IP, auto IM, double ev,
                                                           double od) {
            constexpr int ip = decltype(IP)::value;
            constexpr int im = decltype(IM)::value;
            constexpr double w = L::wshell(L::shell(ip));
            es[ip] = w + (ev + od);
            if constexpr (im >= 0) es[im] = w + (ev - od);
        });
        double z = 0.0;
        for (int i = 0; i < L::Q; ++i) {
            const int cy = L::c(i, 1);
            if (side == 0 ? cy > 0 : cy < 0) {
                const int64_t k = cy < 0 ? -cy : cy;
                z += double(k < ny ? k : ny) * es[i];
            }
        }
        es[L::Q] = z;
    }
}

template <class L, class S>
__device__ __forceinline__ void wall_column_density(const S *__restrict__ A, const GridDims &gd,
                                                    const StepCoef &co, const WallDesc &wd,
                                                    int64_t col)
{
    // The partial sums of state A (buffer wd.par) over one column: per row next
    // to a plate, its slots whose next move crosses the plate -- rows y = k
    // with c_y < -k (bottom), rows y = ny-3+k with c_y >= 3 - k (top).  Every load
    // of a row is unconditional and independent (crossing_sums selects the terms),
    // so they are all in flight at once.
    const int64_t ncol = int64_t(gd.nx) * gd.nz;
    const int x = int(col % gd.nx), z = int(col / gd.nx);
    static_for<0, 2>([&](auto SIDE) {
        constexpr int side = decltype(SIDE)::value;
        const int y0 = side == 0 ? 0 : (gd.ny > 3 ? gd.ny - 3 : 0);
        static_for<0, 3>([&](auto K) {
            constexpr int k = decltype(K)::value;
            const int y = y0 + k;
            if (y >= gd.ny) return;  // uniform: only when ny < 3
            const int64_t own = (int64_t(z) * gd.ny + y) * gd.px + x;
            double ps[7] = {};
            in_step_order<L>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cy = L::c(i, 1);
                // a slot can cross only toward its plate
                if constexpr (side == 0 ? cy < 0 : cy > 0)
                    ps[cy + 3] += Codec<L, S>::template load<i, double>(A[int64_t(i) * gd.P + own]);
            });
            double below, above;
            crossing_sums<L>(ps, y, gd.ny, co.rho0, below, above);
            wd.part[wall_part_index(wd.par, side, k, ncol, col)] = side == 0 ? below : above;
        });
    });
}

template <int LAT, class S>
__global__ void __launch_bounds__(256)
    wall_mass_kernel(const S *__restrict__ A, GridDims gd, StepCoef co, WallDesc wd)
{
    const int64_t ncol = int64_t(gd.nx) * gd.nz;
    const int64_t col = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (col < ncol) wall_column_density<Lattice<LAT>, S>(A, gd, co, wd, col);
}

// ---------------------------------------------------------------------------
// K4: totals.  Stage 1: block b sums a fixed slice of every population plane
// of h; stage 2: one block adds the slices in order and forms the moments of
// f = w rho0 + h using sum w = 1, sum w c = 0 and sum w |c|^2 r^2 = D:
//   mass = N rho0 + sum H_i, momentum = r sum c_i H_i,
//   energy = N rho0 D + r^2 sum |c_i|^2 H_i,  with H_i = sum_x h_i(x).
// The partition and the reduction order do not depend on the grid or launch
// shape of the step, so the result is bitwise reproducible.
// ---------------------------------------------------------------------------
// Stage 1: block b sums the cells of a fixed run of grid rows, every lane
// holding one FP64 accumulator per population: the block's cells are taken
// in order, lane t the t-th of every 256, all Q planes of a cell loaded
// together; then each accumulator is reduced across the block in a fixed tree.
template <int LAT, class S>
__global__ void __launch_bounds__(256)
    totals_stage1(const S *__restrict__ A, double *__restrict__ partials, GridDims gd,
                  DivU32 by_nx)
{
    using L = Lattice<LAT>;
    __shared__ double lds[4][L::Q];
    const int64_t rows = int64_t(gd.ny) * gd.nz;
    const int64_t chunk = (rows + TOTALS_BLOCKS - 1) / TOTALS_BLOCKS;
    const int64_t lo = int64_t(blockIdx.x) * chunk;
    const int64_t hi = (lo + chunk < rows) ? lo + chunk : rows;
    double acc[L::Q];
    static_for<0, L::Q>([&](auto I) { acc[decltype(I)::value] = 0.0; });
    // cells of the block, < 2^32: a block holds at most ceil(rows / 512) rows
    const uint32_t ncell = hi > lo ? uint32_t((hi - lo) * gd.nx) : 0u;
    for (uint32_t k = threadIdx.x; k < ncell; k += 256) {
        const uint32_t dr = divu(by_nx, k);
        const int64_t idx = (lo + dr) * gd.px + (k - dr * uint32_t(gd.nx));
        static_for<0, L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            acc[i] += Codec<L, S>::template load<i, double>(A[int64_t(i) * gd.P + idx]);
        });
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    static_for<0, L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        double v = acc[i];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) lds[wid][i] = v;
    });
    __syncthreads();
    if (threadIdx.x < L::Q) {
        const int i = threadIdx.x;
        partials[int64_t(i) * TOTALS_BLOCKS + blockIdx.x] =
            (lds[0][i] + lds[1][i]) + (lds[2][i] + lds[3][i]);
    }
}

// Stage 2: a wavefront adds the 512 slices of one plane (8 a lane, then a tree),
// 16 planes at a time: 4 us.  One block adding plane after plane, with two barriers
// each, took 37 us, more than stage 1 of every grid below 10^6 cells.
template <int LAT>
__global__ void __launch_bounds__(1024) totals_stage2(const double *__restrict__ partials,
                                                      double *__restrict__ out, GridDims gd,
                                                      StepCoef co)
{
    using L = Lattice<LAT>;
    __shared__ double Hi[L::Q];
    const int lane = threadIdx.x & 63;
    for (int i = threadIdx.x >> 6; i < L::Q; i += 16) {
        const double *p = partials + int64_t(i) * TOTALS_BLOCKS + lane;
        double v = p[0];
#pragma unroll
        for (int k = 1; k < TOTALS_BLOCKS / 64; ++k) v += p[64 * k];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) Hi[i] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0, p[3] = {0.0, 0.0, 0.0}, e = 0.0;
        static_for<0, L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            m += Hi[i];
            for (int a = 0; a < L::D; ++a) p[a] += double(L::c(i, a)) * Hi[i];
            e += double(c2<L>(i)) * Hi[i];
        });
        const double base = double(gd.N) * co.rho0;
        out[0] = base + m;
        for (int a = 0; a < L::D; ++a) out[1 + a] = L::R * p[a];
        out[1 + L::D] = base * double(L::D) + L::R2 * e;
    }
}

}  // namespace lbm
