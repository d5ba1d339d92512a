// HIP kernels (gfx950, wave64) of the two-fluid colour LBM time step over a sparse pore list.
//
// Method (arXiv 2007.12266, section "Color Lattice-Boltzmann Model"): two D3Q7 mass LBEs whose
// post-collision populations are the recoloured equilibria
//   A*_q = w_q N_a [1 + u.xi_q / cs^2 + beta (N_b/N) n.xi_q],
//   B*_q = w_q N_b [1 + u.xi_q / cs^2 - beta (N_a/N) n.xi_q],   cs^2 = 2/9,
// coupled through phi = (N_a - N_b)/(N_a + N_b), C = grad phi and n = C/|C| to a D3Q19 MRT LBE
// with the alpha|C| terms in the equilibria of the energy and stress moments and a constant body
// force t_q xi_q.F / cs^2 (cs^2 = 1/3).
//
// Kernel design for MI355X:
//  * Structure of arrays: population q of pore voxel i lives at X[q*ld + i]; one thread per pore
//    voxel, so every wavefront touches 64 consecutive doubles per population (coalesced).
//  * AA pattern in place for the D3Q19 populations (one copy of the array). Even steps read the
//    voxel's own slots and write the post-collision value of direction q into its own slot
//    opp(q). Odd steps read incoming f_q from slot opp(q) of the upstream neighbour and write
//    f*_q into slot q of the downstream neighbour. A solid (or out-of-domain) neighbour turns
//    either access into the voxel's own opposite slot, which is halfway bounce-back. Each thread
//    reads and writes the same set of addresses, so the pattern is race-free without a second
//    buffer.
//  * The D3Q7 component populations are streamed in moment form. The mass LBEs relax fully: the
//    seven outgoing A*_q of a voxel are fixed by N_a, u and G = beta (N_a N_b / N) n (and B*_q by
//    N_b, u, -G). The collide kernel therefore stores u and G per voxel, coalesced, in the voxel's
//    own slots; N_a and N_b follow from the phi and N that the phase kernel stored for it, which
//    are kept for one more step in buffers that alternate by step parity. The phase kernel
//    rebuilds each incoming A_q(x) = A*_q(x - xi_q) from the upstream neighbour's 8 numbers with
//    the same arithmetic the populations would have been formed with (at a wall, from the voxel's
//    own opposite outgoing population). This moves 14 values per voxel and step instead of 28, and
//    turns the odd step's 14 scattered A/B writes into 6 coalesced ones. (With N_a and N_b stored
//    again by the collide kernel, 512^3 FP64 took 1.9% longer, 320^3 FP32-mixed 2.4%; the phase
//    kernel's loads, two where a pair was one, cost 8% of its own time.) A state that no step has
//    made, initial or loaded, holds the densities themselves (a per-domain device flag, cleared by
//    the first collide). The slots are 3 rows of value pairs, (u_x, G_x), (u_y, G_y), (u_z, G_z),
//    so that what a neighbour contributes along one axis is one wide load; storing each voxel's
//    values contiguously was measured slower on both kernels.
//  * Neighbours come from an int32 table with opposite directions interleaved (one 8-byte load
//    per pair), or from the voxel's packed coordinate and per-64-voxel row records (the rank
//    lookup: less memory, a dependent load more, measured slower). The step kernels are
//    compiled for each lookup.
//  * The MRT collision is evaluated in its two-relaxation-time form: the relaxation matrix has
//    one rate (s+ = 1/tau) on every even moment and one rate (s- = 8(2-s+)/(8-s+)) on every odd
//    one (the conserved moments have zero non-equilibrium part, so their rate is immaterial).
//    For an orthogonal basis whose rows are each even or odd in xi this makes
//    M^-1 S M = s+ P_even + s- P_odd, so the 19x19 transforms reduce to sums and differences of
//    opposite pairs. The equilibrium in population space is the second-order polynomial plus the
//    image of the alpha|C| moment terms under M^-1 (closed form below).
//  * Workgroup -> tile mapping can be XCD-aware: the hardware deals workgroups round-robin to
//    the 8 XCDs, so each XCD is given runs of consecutive tiles, the XCDs' runs
//    interleaved. Neighbouring tiles then share an L2 (the cache lines a wave's scattered
//    accesses leave half used are completed by the next tile on the same XCD) while all XCDs
//    still stream through the pore list together.
//  * Three storage precisions share every kernel body through a precision policy: FP64 stores
//    f, the moment slots, phi and N in double and computes in double; FP32-deviation stores f as
//    the deviation f_q - t_q from the rest equilibrium (rho0 = 1), the rest as float, and
//    computes in float on those deviations; the mixed form stores f as FP32 deviations but keeps
//    the phase field (moment slots, phi, N) in double and computes in double, because rounding
//    the phase field to float every step is what moves the Darcy flux of a two-phase state, not
//    rounding f. The two-rate collision is invariant under the deviation shift (t_q is the same
//    for q and opp(q)), so the same formulas serve all three.
//  * No MFMA: nothing here is a dense contraction. The kernel is bound by HBM traffic.

#include <algorithm>
#include <cmath>

#include "lbm_internal.h"

namespace lbm {
namespace {

// D3Q19 velocities (order: rest; +x -x +y -y +z -z; xy, xz, yz diagonals) and opposites.
constexpr int CX[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
constexpr int CY[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
constexpr int CZ[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
constexpr int OPP[19] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};

__host__ __device__ constexpr double tw(int q) {   // D3Q19 weights t_q
    return q == 0 ? 1.0 / 3.0 : (q < 7 ? 1.0 / 18.0 : 1.0 / 36.0);
}

// Precision policies. F: storage type of f. S: storage type of the moment slots, phi and N.
// R: arithmetic type. kDev: f is stored as f_q - t_q. kCMin: smallest resolved colour-gradient
// magnitude (a few orders above the rounding noise of C in the arithmetic type); a smaller |C|
// counts as zero.
template <int PREC> struct Prec;
template <> struct Prec<LBM_FP64> {
    using F = double;
    using S = double;
    using R = double;
    static constexpr bool kDev = false;
    static constexpr double kCMin = 1e-10;
};
template <> struct Prec<LBM_FP32_DEV> {
    using F = float;
    using S = float;
    using R = float;
    static constexpr bool kDev = true;
    static constexpr double kCMin = 1e-5;
};
template <> struct Prec<LBM_FP32_MIXED> {
    using F = float;
    using S = double;
    using R = double;
    static constexpr bool kDev = true;
    static constexpr double kCMin = 1e-10;
};

// Neighbour lookup, fixed at compile time for the single-domain step kernels and chosen per
// domain at run time (words != null selects the rank lookup, cwave != null the compact one) where
// domains of several kinds meet.
enum { NB_DYN = 0, NB_TABLE = 1, NB_RANK = 2, NB_COMPACT = 3 };

// Hardware block b runs on XCD b % 8 as that XCD's (b / 8)-th block; it takes logical tile
// ((j / C) * 8 + x) * C + j % C (x = b % 8, j = b / 8, C = run length; C = 1 is launch order).
// With gridDim.x a multiple of 8 C this is a bijection of [0, gridDim.x). j / C is a product with
// m = ceil(2^31 / C): exact for j < 2^25, as m C - 2^31 < C <= 64 and a grid holds at most
// 2^30 / 64 blocks.
__device__ __forceinline__ int xcd_run_tile(int b, int C, uint32_t m) {
    const uint32_t x = b & 7, j = (uint32_t)b >> 3;
    const uint32_t r = (uint32_t)(((uint64_t)j * m) >> 31);
    return (int)((r * 8 + x) * C + (j - r * C));
}

// Has the arguments a step kernel's loads need in scalar registers from here on. Left alone, the
// compiler loads each where it is first used, and the address of every next load waits for
// another trip to the arguments (a quarter of a small kernel's time).
template <int NB>
__device__ __forceinline__ void load_args(const StepArgs& a) {
    asm volatile("" ::"s"(a.N), "s"(a.ld), "s"(a.f), "s"(a.M), "s"(a.phi), "s"(a.ntot),
                 "s"(a.phi_prev), "s"(a.ntot_prev),
                 "s"(a.fresh), "s"(a.face), "s"(a.block), "s"(a.xcd_run), "s"(a.xcd_mul),
                 "s"(a.tile_first), "s"(a.tile_sign));
    if (NB == NB_COMPACT)
        asm volatile("" ::"s"(a.cwave), "s"(a.cn8), "s"(a.cn16), "s"(a.cwide), "s"(a.cex));
    if (NB == NB_TABLE) asm volatile("" ::"s"(a.nbr));
}

// First voxel of this workgroup's tile. In the order from the end (a.tile_sign = -1) the tiles
// run from the end of the (padded) grid, so a kernel launched after one in forward order starts
// on the tiles the other finished last, whose lines may still be in the caches; on a padded grid
// the tiles beyond the pore list still exit. No branch and no value from outside the arguments:
// the whole prologue waits for one load of them (it took four loads in turn).
__device__ __forceinline__ int tile_start(const StepArgs& a) {
    const int t = xcd_run_tile((int)blockIdx.x, a.xcd_run, a.xcd_mul);
    return (a.tile_first + a.tile_sign * t) * a.block;
}

// The D3Q7 moment slots of a voxel are stored as three pairs, one row of 2*ld values per pair:
// (u_x, G_x), (u_y, G_y), (u_z, G_z), each a single 16-byte (FP64) or 8-byte (FP32) access.
template <typename S> struct PairOf;
template <> struct PairOf<double> { using T = double2; };
template <> struct PairOf<float> { using T = float2; };

// Streaming accesses (STREAM). Per launch the step touches most of its data once: the
// populations of the even step (read and written in place), the neighbour table, the moment
// slots and phi written for the next kernel. On a domain far larger than the caches, marking
// those accesses non-temporal lets the L2 give their lines up first, which keeps resident the
// lines that neighbouring voxels re-read within the launch (phi in the collide kernel, the
// moment slots in the phase kernel). On a domain that fits the 256 MB Infinity Cache (and in
// pools, whose members run in cache-sized groups) the same hint costs the reuse from one step
// to the next, so it is a launch option (lbm_tuning). The odd step's populations stay ordinary
// accesses either way: they land one neighbour away, so a cache line is shared between adjacent
// waves and must be merged in the L2.
template <bool STREAM, typename T>
__device__ __forceinline__ T load_once(const T* p) {
    if (STREAM) return __builtin_nontemporal_load(p);
    return *p;
}

template <bool STREAM, typename T>
__device__ __forceinline__ void store_once(T v, T* p) {
    if (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <typename S>
__device__ __forceinline__ typename PairOf<S>::T load_pair(const S* __restrict__ M, size_t ld,
                                                          int k, int y) {
    return reinterpret_cast<const typename PairOf<S>::T*>(M)[(size_t)k * ld + y];
}

// One 16-byte (FP64) or 8-byte (FP32) store of a pair of slots.
template <typename S, bool STREAM = false>
__device__ __forceinline__ void store_pair(S* __restrict__ M, size_t ld, int k, int i, S x, S y) {
    typedef S Vec2 __attribute__((ext_vector_type(2)));
    Vec2 v;
    v.x = x;
    v.y = y;
    store_once<STREAM>(v, reinterpret_cast<Vec2*>(M) + ((size_t)k * ld + i));
}

template <int NB>
__device__ __forceinline__ bool use_compact(const StepArgs& a) {
    return NB == NB_COMPACT || (NB == NB_DYN && a.cwave);
}

template <int NB>
__device__ __forceinline__ bool use_table(const StepArgs& a) {
    return NB == NB_TABLE || (NB == NB_DYN && !a.words && !a.cwave);
}

template <int NB>
__device__ __forceinline__ bool use_rank(const StepArgs& a) {
    return NB == NB_RANK || (NB == NB_DYN && a.words);
}

// Memory that no thread writes during a launch, read through the constant address space: where
// the address is the same for every lane of a wave the compiler can use scalar loads.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* as_const(const T* p) {
    return (const __attribute__((address_space(4))) T*)p;
}

// What a voxel's neighbour lookups share: its coordinates (rank lookup) or its 18 decoded
// neighbours (compact lookup).
struct Pos {
    int x, y, z;
    int cn[18];
};

// Compact lookup of all 18 neighbours of pore voxel i: a code above the wave's pore or tail base
// for each direction (a mask bit chooses), 8 bits wide in byte waves and 16 bits in the others,
// or the int32 entries of an exception wave (layout in lbm_prepass.h). The wave record is read
// once per voxel; with WAVE, the caller's waves hold 64 consecutive pore voxels (tiles of a
// multiple of 64 starting at a multiple of 64), so the record's address is wave-uniform: it is
// read with scalar loads and the tests of the wave's kind are scalar branches. Directions a
// kernel never asks for are dead code (the phase kernel reads only n8 of a byte wave, and only
// wide of a 16-bit one). Byte codes take 13 and 6 bytes per voxel off the two kernels (80% byte
// waves); with 16-bit codes alone 256^3 FP64 took 2.5% longer, 320^3 FP32-mixed 3.1%, 512^3
// FP64 2.5%, a pool of 16 FP32-mixed members 4.5%. Giving exception waves byte codes too, above
// bases for each of up to four stretches of lanes, saved no time.
template <bool WAVE, bool STREAM>
__device__ __forceinline__ void compact_all(const StepArgs& a, int i, int (&cn)[18]) {
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));
    typedef uint32_t U2 __attribute__((ext_vector_type(2)));
    const int w = WAVE ? __builtin_amdgcn_readfirstlane(i >> 6) : (i >> 6);
    const auto* rec = as_const(a.cwave) + (size_t)w * kCompactWaveInts;
    const int32_t row = rec[kCompactExRow], kind = rec[kCompactKind];
    if (row >= 0) {
        const int32_t* ex = a.cex + (size_t)row * 18 * 64 + (i & 63);
#pragma unroll
        for (int q = 1; q < 19; ++q) cn[q - 1] = load_once<STREAM>(ex + (q - 1) * 64);
        return;
    }
    const U2 n8 = load_once<STREAM>(reinterpret_cast<const U2*>(a.cn8) + i);
    const U4 n16 = load_once<STREAM>(reinterpret_cast<const U4*>(a.cn16) + i);
    // Byte code and mask bit of direction q.
    auto byte_code = [&](int q) {
        const uint32_t words[5] = {n8.x, n8.y, n16.x, n16.y, n16.z};
        const int k = q < 7 ? q - 1 : q + 1;
        return (words[k >> 2] >> (8 * (k & 3))) & 0xffu;
    };
    auto byte_tail = [&](int q) { return (q < 7 ? n8.y >> (16 + q - 1) : n16.w >> (q - 7)) & 1u; };
    // Both bases as wave-uniform values, then a per-lane select (a select of the two addresses
    // would turn the scalar loads into vector ones).
    auto target = [&](int q, uint32_t tail, uint32_t code) {
        const int32_t pb = WAVE ? __builtin_amdgcn_readfirstlane(rec[q - 1]) : rec[q - 1];
        const int32_t tb = WAVE ? __builtin_amdgcn_readfirstlane(rec[18 + q - 1]) : rec[18 + q - 1];
        return (tail ? tb : pb) + (int)code;
    };
    if (kind == 1) {
#pragma unroll
        for (int q = 1; q < 19; ++q) cn[q - 1] = target(q, byte_tail(q), byte_code(q));
        return;
    }
    const U4 wide = load_once<STREAM>(reinterpret_cast<const U4*>(a.cwide) + i);
    const uint32_t words[9] = {wide.y, wide.z, wide.w, n16.x, n16.y, n16.z, n16.w, n8.x, n8.y};
#pragma unroll
    for (int q = 1; q < 19; ++q) {
        const uint32_t word = words[(q - 1) >> 1];
        cn[q - 1] = target(q, (wide.x >> q) & 1u, (q & 1) ? (word & 0xffffu) : (word >> 16));
    }
}

// Pressure face of pore voxel i: 0, 1 (inlet) or 2 (outlet). With the compact lookup a mark in the
// wave's record says whether the wave holds any, so the others read no flags.
template <int NB>
__device__ __forceinline__ int face_of(const StepArgs& a, int i) {
    if (!a.face) return 0;
    if (NB == NB_COMPACT) {
        const int w = __builtin_amdgcn_readfirstlane(i >> 6);
        if (!(as_const(a.cwave) + (size_t)w * kCompactWaveInts)[kCompactFace]) return 0;
    }
    return a.face[i];
}

// Per-voxel lookup state of pore voxel i (see Pos).
template <int NB = NB_DYN, bool WAVE = false, bool STREAM = false>
__device__ __forceinline__ Pos pos_of(const StepArgs& a, int i) {
    Pos p;
    p.x = p.y = p.z = 0;
    if (use_compact<NB>(a)) {
        compact_all<WAVE, STREAM>(a, i, p.cn);
        return p;
    }
    if (!use_rank<NB>(a)) return p;
    const uint32_t c = a.coord[i];
    p.x = (int)(c & ((1u << kCoordXBits) - 1));
    p.y = (int)((c >> kCoordXBits) & ((1u << kCoordYBits) - 1));
    p.z = (int)(c >> (kCoordXBits + kCoordYBits));
    return p;
}

// Pore index, or N + tail index for a solid, of the in-domain voxel (x, y, z): the segment's
// first index plus the number of pore (or tail-solid) voxels before x in the segment.
__device__ __forceinline__ int rank_index(const StepArgs& a, int x, int y, int z) {
    const RowWord rw = a.words[((size_t)y + (size_t)a.ny * z) * a.W + (x >> 6)];
    const int b = x & 63;
    const uint64_t below = (1ull << b) - 1ull;
    if ((rw.pore >> b) & 1ull) return rw.pore_base + __popcll(rw.pore & below);
    return a.N + rw.tail_base + __popcll(rw.tail & below);
}

// Neighbour of pore voxel i along direction q (1..18) for the colour gradient: a pore index
// (< N) or N + tail index (a solid's phi_s, or the wall's). `mirror` is set for a z neighbour
// beyond a pressure face in the rank lookup: its phi is the in-plane voxel's, but streaming
// bounces back there (stream index N). With the explicit table, such neighbours are tail
// ghosts, already >= N.
template <int NB = NB_DYN, bool STREAM = false>
__device__ __forceinline__ int nb(const StepArgs& a, int q, int i, Pos p, bool& mirror) {
    mirror = false;
    if (use_table<NB>(a)) {
        // Opposite directions (q, q + 1 for odd q) share one 8-byte entry.
        const int64_t e =
            load_once<STREAM>(reinterpret_cast<const int64_t*>(a.nbr) + ((size_t)((q - 1) >> 1) * a.ld + i));
        return (q & 1) ? (int)(uint32_t)e : (int)(e >> 32);
    }
    if (use_compact<NB>(a)) return p.cn[q - 1];
    int cx = p.x + CX[q], cy = p.y + CY[q], cz = p.z + CZ[q];
    if (CX[q] && (cx < 0 || cx >= a.nx)) {
        if (!(a.periodic & 1)) return a.N;
        cx = cx < 0 ? cx + a.nx : cx - a.nx;
    }
    if (CY[q] && (cy < 0 || cy >= a.ny)) {
        if (!(a.periodic & 2)) return a.N;
        cy = cy < 0 ? cy + a.ny : cy - a.ny;
    }
    if (CZ[q] && (cz < 0 || cz >= a.nz)) {
        if (a.periodic & 4) {
            cz = cz < 0 ? cz + a.nz : cz - a.nz;
        } else if (a.bc_z) {
            cz = p.z;
            mirror = true;
        } else {
            return a.N;
        }
    }
    return rank_index(a, cx, cy, cz);
}

// Streaming neighbour of pore voxel i along q: a pore index, or >= N for a wall (bounce-back).
template <int NB = NB_DYN, bool STREAM = false>
__device__ __forceinline__ int nb_stream(const StepArgs& a, int q, int i, Pos p) {
    bool mirror;
    const int r = nb<NB, STREAM>(a, q, i, p, mirror);
    return mirror ? a.N : r;
}

// Incoming population q of voxel i (D3Q19 or D3Q7 array X).
template <bool ODD, typename S, bool STREAM = false>
__device__ __forceinline__ S load_in(const S* __restrict__ X, const StepArgs& a, int q, int i,
                                     int r_up) {
    if (!ODD) return load_once<STREAM>(&X[(size_t)q * a.ld + i]);
    if (q == 0) return X[i];
    // r_up: neighbour along opp(q), i.e. the upstream voxel i - xi_q.
    return r_up < a.N ? X[(size_t)OPP[q] * a.ld + r_up] : X[(size_t)q * a.ld + i];
}

// Store the post-collision population q of voxel i.
template <bool ODD, typename S, bool STREAM = false>
__device__ __forceinline__ void store_out(S* __restrict__ X, const StepArgs& a, int q, int i,
                                          int r_down, S v) {
    if (!ODD) {
        store_once<STREAM>(v, &X[(size_t)OPP[q] * a.ld + i]);
    } else if (q == 0) {
        X[i] = v;
    } else {
        // r_down: neighbour along q, the downstream voxel i + xi_q; a wall sends the population
        // back into the voxel's own opposite slot. One store to the selected address.
        const bool in = r_down < a.N;
        X[in ? (size_t)q * a.ld + r_down : (size_t)OPP[q] * a.ld + i] = v;
    }
}

// ------------------------------------------------------------------------------------------
// Initial state: rest equilibrium, rho = 1, u = 0, N_a = (1 + phi0)/2, N_b = (1 - phi0)/2.
// Natural layout (step 0 is even).
// ------------------------------------------------------------------------------------------
template <int PREC>
__global__ void __launch_bounds__(256) init_kernel(StepArgs a, const double* __restrict__ phi0) {
    using P = Prec<PREC>;
    using F = typename P::F;
    using S = typename P::S;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.N) return;
    F* f = (F*)a.f;
    S* M = (S*)a.M;
    const double na = 0.5 * (1.0 + phi0[i]), nbv = 0.5 * (1.0 - phi0[i]);
#pragma unroll
    for (int q = 0; q < 19; ++q) f[(size_t)q * a.ld + i] = (F)(P::kDev ? 0.0 : tw(q));
    // A fresh state: the densities themselves (the fresh flag is set by the host).
    ((S*)a.phi_prev)[i] = (S)na;
    ((S*)a.ntot_prev)[i] = (S)nbv;
#pragma unroll
    for (int k = 0; k < 3; ++k) store_pair<S>(M, a.ld, k, i, (S)0, (S)0);
}

// a b + c rounded once. The step's arithmetic states each fused operation: left to the compiler,
// which product of a sum of two is rounded on its own depends on what surrounds it, and the
// variants of a kernel (lookup, streaming, load order, batched) would differ in the last bit.
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// s + v with no contraction into a preceding product.
__device__ __forceinline__ double add_rounded(double s, double v) {
#pragma clang fp contract(off)
    return s + v;
}

// Outgoing D3Q7 populations along an axis direction of sign sgn (+1 or -1), from one voxel's
// densities N_a, N_b and moment slots u_c, G_c of the direction's axis c:
// A* = w [N_a (1 + sgn u_c / cs^2) + sgn G_c], B* = w [N_b (1 + sgn u_c / cs^2) - sgn G_c],
// w = 1/9, cs^2 = 2/9.
template <typename R>
__device__ __forceinline__ void ab_out(R na, R nb, R uc, R gc, R sgn, R& ao, R& bo) {
    const R eu = fused((R)4.5, sgn * uc, (R)1);
    const R en = sgn * gc;
    ao = (R)(1.0 / 9.0) * fused(na, eu, en);
    bo = (R)(1.0 / 9.0) * fused(nb, eu, -en);
}

// Densities that a voxel's components left with, from the phi and N of the step that sent them
// (the arithmetic with which the collide kernel formed them), or as they are (raw).
template <typename R>
__device__ __forceinline__ void sent(R p, R n, bool raw, R& na, R& nb) {
    na = raw ? p : (R)0.5 * n * ((R)1 + p);
    nb = raw ? n : (R)0.5 * n * ((R)1 - p);
}

// Component densities N_a, N_b of pore voxel i in the current state: the sum of the incoming
// D3Q7 populations (rebuilt from the upstream neighbours' moment slots, or from the voxel's own
// opposite outgoing population where the upstream neighbour is solid: halfway bounce-back).
// Pressure-face voxels carry their imposed composition; a fresh state its initial densities.
// All six neighbour indices are read first and every slot load is unconditional (a solid
// upstream neighbour selects the voxel's own slots and flips the sign), so the loads of one
// voxel are in flight together.
// Callers keep each wave on 64 consecutive pore voxels (see compact_all).
// `ghost`: for a voxel of a pressure face the tail entry that mirrors its phi across the face (the
// target beyond the face), else -1; the rank lookup has no such entries.
// FACE: the domain may have pressure faces.
// REST: the state may be at rest, where the neighbours' numbers count for nothing and are not
// fetched (us a count of the phase right after a growth, fetched / not, 256^3 FP64 118 / 59, 320^3
// 220 / 89). The kernels of a step have no such test: its wait for the flag ahead of the fetches
// costs them 1% up to 150^3, and a step from rest is the first of many. Nor have the reductions and
// fields, which would take 1 to 10% longer for every state (320^3 FP32-dev 263 -> 291 us).
template <int PREC, int NB = NB_DYN, bool STREAM = false, bool FACE = true, bool REST = false>
__device__ __forceinline__ void densities(const StepArgs& a, int i, int fresh, double& na,
                                          double& nbv, int& ghost) {
    using P = Prec<PREC>;
    using S = typename P::S;
    using R = typename P::R;
    const S* M = (const S*)a.M;
    const S* __restrict__ pp = (const S*)a.phi_prev;
    const S* __restrict__ np = (const S*)a.ntot_prev;
    R ain[7], bin[7];
    const S own_p = pp[i], own_n = np[i];
    const bool rest = REST && fresh == 1;
    int fc = REST && FACE ? face_of<NB>(a, i) : 0;
    int up[7] = {i, i, i, i, i, i, i};
    if (!rest || fc) {   // a face voxel's ghost is found by its lookup
        const Pos pos = pos_of<NB, true, STREAM>(a, i);
#pragma unroll
        for (int q = 1; q < 7; ++q) up[q] = nb_stream<NB, STREAM>(a, OPP[q], i, pos);  // i - xi_q
    }
    if (!REST && FACE) fc = face_of<NB>(a, i);
    ghost = fc && !use_rank<NB>(a) ? (fc == 1 ? up[5] : up[6]) : -1;   // along -z, along +z
    R sna[7], snb[7], suc[7], sgc[7], ouc[3], ogc[3];   // ouc, ogc: the voxel's own
    constexpr bool kFloat = sizeof(S) == sizeof(float);
    if (rest) {
#pragma unroll
        for (int q = 1; q < 7; ++q) sna[q] = snb[q] = suc[q] = sgc[q] = (R)0;
#pragma unroll
        for (int c = 0; c < 3; ++c) ouc[c] = ogc[c] = (R)0;
    } else {
#pragma unroll
        for (int q = 1; q < 7; ++q) {
            const int c = (q - 1) >> 1;
            const int y = up[q] < a.N ? up[q] : i;
            sna[q] = (R)pp[y];
            snb[q] = (R)np[y];
            const auto g = load_pair<S>(M, a.ld, c, y);
            suc[q] = (R)g.x;
            sgc[q] = (R)g.y;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (kFloat) {
                const auto g = load_pair<S>(M, a.ld, c, i);
                ouc[c] = (R)g.x;
                ogc[c] = (R)g.y;
            }
    }
#pragma unroll
    for (int q = 1; q < 7; ++q) {
        const R sq = (q & 1) ? (R)1 : (R)-1;
        sent<R>(sna[q], snb[q], fresh != 0, sna[q], snb[q]);
        ab_out<R>(sna[q], snb[q], suc[q], sgc[q], up[q] < a.N ? sq : -sq, ain[q], bin[q]);
    }
    R own_a, own_b;
    sent<R>((R)own_p, (R)own_n, fresh != 0, own_a, own_b);
    if (kFloat) {
        // The rest population is what the six moving ones leave of N (the rounded float weights
        // would otherwise add 1.5e-8 of mass per step); sums in double, see below.
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int q = 1; q < 7; ++q) {
            R ao, bo;
            const int c = (q - 1) >> 1;
            ab_out<R>(own_a, own_b, ouc[c], ogc[c], (q & 1) ? (R)1 : (R)-1, ao, bo);
            sa += (double)ao;
            sb += (double)bo;
        }
        ain[0] = (R)0;
        bin[0] = (R)0;
        na = (double)own_a - sa;
        nbv = (double)own_b - sb;
    } else {
        ain[0] = (R)(1.0 / 3.0) * own_a;
        bin[0] = (R)(1.0 / 3.0) * own_b;
        na = 0.0;
        nbv = 0.0;
    }
    // Accumulated in double in both precisions: a float running sum of seven populations
    // carries a mean rounding bias of a few 1e-9, which would create that much mass per step.
    // Each population is rounded on its own before it enters the sum (no fused multiply-add
    // across the two), as in an evaluation that stores the populations.
#pragma unroll
    for (int q = 0; q < 7; ++q) {
        na = add_rounded(na, (double)ain[q]);
        nbv = add_rounded(nbv, (double)bin[q]);
    }
    // The exceptions come last, so that no load above waits for a face flag or the fresh flag.
    if (fc) {
        na = fc == 1 ? 1.0 : 0.0;
        nbv = 1.0 - na;
    }
    if (fresh == 1) {
        // The initial populations are w_q N at rest; summing them (rather than taking N) keeps
        // the initial phase bitwise equal to a population-based evaluation.
        const R n0 = own_a, n1 = own_b;
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            const R w = q == 0 ? (R)(1.0 / 3.0) : (R)(1.0 / 9.0);
            ain[q] = w * n0;
            bin[q] = w * n1;
        }
        na = 0.0;
        nbv = 0.0;
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            na += (double)ain[q];
            nbv += (double)bin[q];
        }
    }
}

// ------------------------------------------------------------------------------------------
// Densities and phase indicator: N_a = sum_q A_q, N_b = sum_q B_q (q = 0..6) of the streamed-in
// D3Q7 populations; phi = (N_a - N_b)/(N_a + N_b); N = N_a + N_b.
// ------------------------------------------------------------------------------------------
template <int PREC, int NB, bool STREAM, bool FACE, bool REST = false>
__device__ __forceinline__ void phase_voxel(const StepArgs& a, int i, int fresh) {
    using S = typename Prec<PREC>::S;
    double na, nbv;
    int ghost;
    densities<PREC, NB, STREAM, FACE, REST>(a, i, fresh, na, nbv, ghost);
    const double nt = na + nbv;
    const S phi = (S)((na - nbv) / nt);
    store_once<STREAM>(phi, (S*)a.phi + i);
    store_once<STREAM>((S)nt, (S*)a.ntot + i);
    if (FACE) {
        if (ghost >= 0) ((S*)a.phi)[ghost] = phi;
        if (i == 0) a.fresh[1] = fresh != 0 ? 1 : 0;
    }
}

template <int PREC, int NB, bool STREAM, bool FACE, bool REST>
__global__ void __launch_bounds__(256) phase_kernel(StepArgs a) {
    load_args<NB>(a);
    const int i = tile_start(a) + (int)threadIdx.x;
    if (i < a.N) phase_voxel<PREC, NB, STREAM, FACE, REST>(a, i, *a.fresh);
}

// ------------------------------------------------------------------------------------------
// Fused colour gradient + MRT collision with interfacial terms and body force + recolouring +
// AA streaming.
// ------------------------------------------------------------------------------------------
// Zou-He pressure condition of density rho on the streamed populations of a voxel of the inlet
// (fc = 1, z = 0) or the outlet (2, z = nz - 1): the unknowns, whose xi_z points into the domain,
// follow from the others, so applying the condition again gives the same values. The composition
// of the face planes (pure a, N = 1, at the inlet; pure b at the outlet) is imposed where
// densities are formed (the face flag), which equals resetting their D3Q7 populations to
// equilibrium.
template <int PREC>
__device__ __forceinline__ void pressure_face(typename Prec<PREC>::F (&f)[19], int fc, double rho) {
#pragma clang fp contract(off)
    using P = Prec<PREC>;
    using F = typename P::F;
    const int dir = fc == 1 ? 1 : -1;
    double fl[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) fl[q] = (double)f[q] + (P::kDev ? tw(q) : 0.0);
    double s0 = 0.0, up = 0.0, down = 0.0, tx = 0.0, ty = 0.0;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        if (CZ[q] == 0) {
            s0 += fl[q];
            if (CX[q]) tx += CX[q] * fl[q];
            if (CY[q]) ty += CY[q] * fl[q];
        } else if (CZ[q] > 0) {
            up += fl[q];
        } else {
            down += fl[q];
        }
    }
    const double jz = dir * (rho - s0 - 2.0 * (dir > 0 ? down : up));
#pragma unroll
    for (int q = 1; q < 19; ++q) {
        if (CZ[q] == 0) continue;
        double val = fused(6.0 * tw(q) * CZ[q], jz, fl[OPP[q]]);
        if (CX[q]) val -= 0.5 * (CX[q] * tx);
        if (CY[q]) val -= 0.5 * (CY[q] * ty);
        if (CZ[q] == dir) f[q] = (F)(val - (P::kDev ? tw(q) : 0.0));
    }
}

// EARLY: every load of a voxel is issued before the first value is used: the even step's own
// populations first, as they need no index, then (indices known) the neighbours' phi and the odd
// step's populations. The scheduler otherwise issues the populations after the gradient has
// waited for phi, one more round trip per voxel. That is time where a launch has few waves per
// CU to hide it (32^3 bead pack in FP64, with load_args: 8.7 -> 8.1 us a step; 64^3 in
// FP32-mixed 9.2 -> 8.5), nothing in a pool, and a loss where the waves in flight compete for the
// L2 (256^3 FP64 -0.7%, 320^3 FP32-mixed -0.9%): on for domains up to kEarlyVoxels.
template <int PREC, bool ODD, int NB, bool STREAM, bool EARLY, bool FACE>
__device__ __forceinline__ void collide_voxel(const StepArgs& a, int i) {
#pragma clang fp contract(off)
    using P = Prec<PREC>;
    using F = typename P::F;
    using S = typename P::S;
    using R = typename P::R;
    F* f = (F*)a.f;
    const S* __restrict__ ph = (const S*)a.phi;

    F fraw[19];
    if (EARLY && !ODD) {
#pragma unroll
        for (int q = 0; q < 19; ++q) fraw[q] = load_in<ODD, F, STREAM>(f, a, q, i, 0);
    }
    S phi_own = 0, n_own = 0;
    if (EARLY) {
        phi_own = ph[i];
        n_own = ((const S*)a.ntot)[i];
    }

    int r[19];           // gradient neighbours (phi index)
    uint32_t mirror = 0; // bit q: streaming along q bounces back although r[q] is a pore index
    r[0] = i;
    {
        const Pos pos = pos_of<NB, true, STREAM>(a, i);
#pragma unroll
        for (int q = 1; q < 19; ++q) {
            bool m;
            r[q] = nb<NB, STREAM>(a, q, i, pos, m);
            mirror |= (m ? 1u : 0u) << q;
        }
    }
#define RS(q) (((mirror >> (q)) & 1u) ? a.N : r[(q)])

    // Colour gradient: weight 1 on the axis links and 1/2 on the diagonals, so that C -> 6 grad
    // phi and the flat-interface tension is exactly 6 alpha. Each component is accumulated in
    // increasing q, one term at a time: every product is exact (a power of two times phi), so
    // the sum is the same correctly rounded chain in any implementation that keeps this order.
    // That matters where |C| is small, since n = C/|C| amplifies a rounding difference in C.
    S praw[19];
#pragma unroll
    for (int q = 1; q < 19; ++q) praw[q] = ph[r[q]];
    if (EARLY && ODD) {
#pragma unroll
        for (int q = 0; q < 19; ++q)
            fraw[q] = load_in<ODD, F, STREAM>(f, a, q, i, RS(OPP[q]));
    }
    if (EARLY) __builtin_amdgcn_sched_barrier(0);
    const int fc = FACE && a.face_bc ? face_of<NB>(a, i) : 0;
    R p[19];
#pragma unroll
    for (int q = 1; q < 19; ++q) p[q] = (R)praw[q];
    R Cx = 0, Cy = 0, Cz = 0;
#pragma unroll
    for (int q = 1; q < 19; ++q) {
        const R w = q < 7 ? (R)1 : (R)0.5;
        if (CX[q]) Cx = fused(w * CX[q], p[q], Cx);
        if (CY[q]) Cy = fused(w * CY[q], p[q], Cy);
        if (CZ[q]) Cz = fused(w * CZ[q], p[q], Cz);
    }
    // |C| <= kCMin is an unresolved gradient (a cancellation whose residue is rounding): it
    // counts as zero, so that n never takes a direction decided by rounding.
    const R c2 = fused(Cz, Cz, fused(Cy, Cy, Cx * Cx));
    const bool resolved = c2 > (R)(P::kCMin * P::kCMin);
    const R cm = resolved ? sqrt(c2) : (R)0;
    const R ic = resolved ? (R)1 / cm : (R)0;
    const R nx = Cx * ic, ny = Cy * ic, nz = Cz * ic;

    // Incoming populations (f, or f - t in deviation storage).
    if (!EARLY) {
#pragma unroll
        for (int q = 0; q < 19; ++q)
            fraw[q] = load_in<ODD, F, STREAM>(f, a, q, i, RS(OPP[q]));
        phi_own = ph[i];
        n_own = ((const S*)a.ntot)[i];
    }
    // A select, not rho_face[fc - 1]: a pool's kernels hold their arguments in registers, and an
    // index known only at run time puts all 280 bytes of them in scratch for every lane (us a step of
    // 15 periodic members of 64^3 and one with faces, index / select: FP64 204 / 108, FP32-mixed
    // 166 / 67.5, FP32-dev 139 / 57.9; of 16 with faces 281 / 154, 252 / 109, 227 / 76.4). The
    // domain's own kernels lose 8 (FP64) and 18 registers with it.
    if (FACE && fc && !a.fresh[1])
        pressure_face<PREC>(fraw, fc, fc == 1 ? a.rho_face[0] : a.rho_face[1]);
    R fl[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) fl[q] = (R)fraw[q];

    // rho (or rho - 1 in deviation storage) and j.
    R rho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        rho += fl[q];
        if (CX[q]) jx += CX[q] * fl[q];
        if (CY[q]) jy += CY[q] * fl[q];
        if (CZ[q]) jz += CZ[q] * fl[q];
    }
    const R jj = fused(jz, jz, fused(jy, jy, jx * jx));

    const R phi_i = (R)phi_own;
    const R nt = (R)n_own;
    // Recolouring with the flow velocity u = j + F/2 (rho0 = 1): the outgoing D3Q7 populations
    // are w_q [N_a (1 + u.xi_q/cs^2) + G.xi_q] and w_q [N_b (1 + u.xi_q/cs^2) - G.xi_q] with
    // G = beta (N_a N_b / N) n. Of their 8 defining numbers u and G go to the voxel's own moment
    // slots; N_a and N_b follow from phi and N, which the phase kernel reads again.
    const R ux = jx + (R)(0.5 * a.F[0]), uy = jy + (R)(0.5 * a.F[1]);
    const R uz = jz + (R)(0.5 * a.F[2]);
    const R na = (R)0.5 * nt * ((R)1 + phi_i);
    const R nbv = (R)0.5 * nt * ((R)1 - phi_i);
    const R seg = (R)a.beta * na * nbv / nt;
    S* M = (S*)a.M;
    const size_t ld = (size_t)a.ld;
    store_pair<S, STREAM>(M, ld, 0, i, (S)ux, (S)(seg * nx));
    store_pair<S, STREAM>(M, ld, 1, i, (S)uy, (S)(seg * ny));
    store_pair<S, STREAM>(M, ld, 2, i, (S)uz, (S)(seg * nz));

    const R nu = fused((R)0.5 * ((R)1 + phi_i), (R)a.nu_a, (R)0.5 * ((R)1 - phi_i) * (R)a.nu_b);
    const R sp = (R)1 / fused((R)3, nu, (R)0.5);
    const R sm = (R)8 * ((R)2 - sp) / ((R)8 - sp);

    // Image of the alpha|C| equilibrium-moment terms in population space (even in xi):
    // e-row -19 g, 3pxx (g/2)(3nx^2-1), pww (g/2)(ny^2-nz^2), pxy (g/2)nx ny, ... ; g = alpha|C|.
    const R g = (R)a.alpha * cm;
    const R hxx = g * fused((R)3 * nx, nx, (R)-1);
    const R hww = g * fused(ny, ny, -(nz * nz));
    const R hx36 = hxx * (R)(1.0 / 36.0), hx72 = hxx * (R)(1.0 / 72.0);
    const R c_ax = (R)(11.0 / 126.0), c_dg = (R)(-8.0 / 126.0), c_w = (R)(1.0 / 24.0);
    const R dX = fused(g, c_ax, hx36), dYZ = fused(g, c_dg, -hx36);
    const R dY = fused(hww, c_w, fused(g, c_ax, -hx72));
    const R dZ = fused(hww, -c_w, fused(g, c_ax, -hx72));
    const R dXY = fused(hww, c_w, fused(g, c_dg, hx72));
    const R dXZ = fused(hww, -c_w, fused(g, c_dg, hx72));
    const R gxy = g * nx * ny * (R)0.125, gxz = g * nx * nz * (R)0.125;
    const R gyz = g * ny * nz * (R)0.125;

    // Even equilibrium part (per velocity class) and odd part 3 t xi.j. The rest weight t_q
    // multiplies rho in the even part; with deviation storage both sides carry -t_q.
    const R base = fused((R)-1.5, jj, rho);
    R fs[19];
    const R e0 = fused(g, (R)(5.0 / 21.0), (R)(1.0 / 3.0) * base);
    fs[0] = fused(-sp, fl[0] - e0, fl[0]);
#pragma unroll
    for (int q = 1; q < 19; q += 2) {
        const int qb = q + 1;
        const R t = (R)tw(q);
        const R e3[3] = {CX[q] * jx, CY[q] * jy, CZ[q] * jz};
        const R ej = CX[q] && CY[q] ? e3[0] + e3[1]
                     : CX[q] && CZ[q] ? e3[0] + e3[2]
                     : CY[q] && CZ[q] ? e3[1] + e3[2]
                     : CX[q] ? e3[0] : CY[q] ? e3[1] : e3[2];
        const R ef = (R)(CX[q] * a.F[0] + CY[q] * a.F[1] + CZ[q] * a.F[2]);
        R dq;
        if (q == 1) dq = dX;
        else if (q == 3) dq = dY;
        else if (q == 5) dq = dZ;
        else if (q < 11) dq = dXY + gxy * (R)(CX[q] * CY[q]);
        else if (q < 15) dq = dXZ + gxz * (R)(CX[q] * CZ[q]);
        else dq = dYZ + gyz * (R)(CY[q] * CZ[q]);
        const R ep = fused(t, fused((R)4.5 * ej, ej, base), dq);
        const R em = (R)3 * t * ej;
        const R rp = fused((R)0.5, fl[q] + fl[qb], -ep);
        const R rm = fused((R)0.5, fl[q] - fl[qb], -em);
        fs[q] = fused((R)3 * t, ef, fused(-sm, rm, fused(-sp, rp, fl[q])));
        fs[qb] = fused((R)-3 * t, ef, fused(sm, rm, fused(-sp, rp, fl[qb])));
    }

#pragma unroll
    for (int q = 0; q < 19; ++q) store_out<ODD, F, STREAM>(f, a, q, i, RS(q), (F)fs[q]);
#undef RS
    if (i == 0) *a.fresh = 0;        // the state now holds outgoing moments
}

template <int PREC, bool ODD, int NB, bool STREAM, bool EARLY, bool FACE>
__global__ void __launch_bounds__(256) collide_kernel(StepArgs a) {
    load_args<NB>(a);
    const int i = tile_start(a) + (int)threadIdx.x;
    if (i < a.N) collide_voxel<PREC, ODD, NB, STREAM, EARLY, FACE>(a, i);
}

// ------------------------------------------------------------------------------------------
// Batched steps: one launch covers every live domain of a pool. The pore list of each domain is
// cut into tiles of blockDim.x voxels; tile t belongs to slot tile_dom[t] and is that slot's
// (t - tile_first[slot])-th tile. A fixed grid strides over the tiles (persistent launch); the
// tile count is read from device memory so that a captured graph stays valid when the pool's
// membership changes. Per-voxel arithmetic is the single-domain one, so every domain's result
// is bitwise the same alone and in the mix.
// ------------------------------------------------------------------------------------------
// The tile table and the per-slot arguments are read-only during a launch and every index into
// them is uniform over the workgroup: reading them through the constant address space (as_const)
// lets the compiler use scalar loads, so a slot's arguments live in scalar registers.

// A whole record through the constant address space, one 32-bit word at a time (the compiler
// merges the words into wide scalar loads).
template <typename T>
__device__ __forceinline__ T load_const(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "record size must be a multiple of 4 bytes");
    T out;
    const auto* src = as_const(reinterpret_cast<const int32_t*>(p));
    int32_t* dst = reinterpret_cast<int32_t*>(&out);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) dst[k] = src[k];
    return out;
}

// Arguments of slot d at the step's parity.
__device__ __forceinline__ StepArgs batch_args(const BatchArgs& b, int d) {
    StepArgs a = load_const(b.doms + d);
    void *phi = a.phi, *ntot = a.ntot;
    a.phi = b.odd ? a.phi_prev : phi;
    a.ntot = b.odd ? a.ntot_prev : ntot;
    a.phi_prev = b.odd ? phi : a.phi_prev;
    a.ntot_prev = b.odd ? ntot : a.ntot_prev;
    return a;
}

template <int PREC, int NB, bool FACE>
__global__ void __launch_bounds__(256) phase_batched(BatchArgs b) {
    const int nt = *as_const(b.ntiles);
    const int first = b.xcd ? xcd_run_tile((int)blockIdx.x, kXcdRun, xcd_mul_of(kXcdRun))
                            : (int)blockIdx.x;
    for (int t = first; t < nt; t += gridDim.x) {
        const int d = as_const(b.tile_dom)[t];
        const StepArgs a = batch_args(b, d);
        const int i = (t - as_const(b.tile_first)[d]) * blockDim.x + threadIdx.x;
        if (i < a.N) phase_voxel<PREC, NB, false, FACE>(a, i, *a.fresh);
    }
}

template <int PREC, bool ODD, int NB, bool FACE>
__global__ void __launch_bounds__(256) collide_batched(BatchArgs b) {
    const int nt = *as_const(b.ntiles);
    const int first = b.xcd ? xcd_run_tile((int)blockIdx.x, kXcdRun, xcd_mul_of(kXcdRun))
                            : (int)blockIdx.x;
    for (int t = first; t < nt; t += gridDim.x) {
        const int d = as_const(b.tile_dom)[t];
        const StepArgs a = batch_args(b, d);
        const int i = (t - as_const(b.tile_first)[d]) * blockDim.x + threadIdx.x;
        if (i < a.N) collide_voxel<PREC, ODD, NB, false, false, FACE>(a, i);
    }
}

// ------------------------------------------------------------------------------------------
// Per-voxel read-out in FP64 from either storage: rho and j, and with the densities N_a, N_b.
// ------------------------------------------------------------------------------------------
template <int PREC, bool ODD>
__device__ __forceinline__ void voxel_flow(const StepArgs& a, int i, double& rho, double& jx,
                                           double& jy, double& jz) {
    using P = Prec<PREC>;
    using F = typename P::F;
    const F* f = (const F*)a.f;
    int r[19];
    r[0] = i;
    const Pos pos = pos_of(a, i);
#pragma unroll
    for (int q = 1; q < 19; ++q) r[q] = ODD ? nb_stream(a, q, i, pos) : 0;
    rho = 0.0;
    jx = jy = jz = 0.0;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        const double v = (double)load_in<ODD>(f, a, q, i, r[OPP[q]]);
        rho += v;
        jx += CX[q] * v;
        jy += CY[q] * v;
        jz += CZ[q] * v;
    }
    if (P::kDev) rho += 1.0;
}

template <int PREC, bool ODD>
__device__ __forceinline__ void voxel_state(const StepArgs& a, int i, double& na, double& nbv,
                                            double& rho, double& jx, double& jy, double& jz) {
    int ghost;
    densities<PREC>(a, i, *a.fresh, na, nbv, ghost);   // callers' waves are aligned
    voxel_flow<PREC, ODD>(a, i, rho, jx, jy, jz);
}

// ------------------------------------------------------------------------------------------
// Reductions (FP64, deterministic: fixed grid, fixed per-thread stride, fixed butterfly).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Partial sums of reduction block `blk` (of kRedBlocks): voxels blk*T + tid + k*kRedBlocks*T.
template <int PREC, bool ODD>
__device__ __forceinline__ void reduce_block(const StepArgs& a, int blk,
                                             double* __restrict__ partials) {
    if ((int64_t)blk * kRedThreads >= a.N) {   // no voxel: a small domain has few blocks that do
        if (threadIdx.x < kNRed) partials[(size_t)blk * kNRed + threadIdx.x] = 0.0;
        return;
    }
    double acc[kNRed];
#pragma unroll
    for (int k = 0; k < kNRed; ++k) acc[k] = 0.0;
    const int stride = kRedBlocks * kRedThreads;
    for (int i = blk * kRedThreads + threadIdx.x; i < a.N; i += stride) {
        double na, nbv, rho, jx, jy, jz;
        voxel_state<PREC, ODD>(a, i, na, nbv, rho, jx, jy, jz);
        const double phi = (na - nbv) / (na + nbv);
        const double u[3] = {jx + 0.5 * a.F[0], jy + 0.5 * a.F[1], jz + 0.5 * a.F[2]};
        const bool bad = !(isfinite(na) && isfinite(nbv) && isfinite(rho) && isfinite(u[0]) &&
                           isfinite(u[1]) && isfinite(u[2]));
        const double wa = 0.5 * (1.0 + phi), wb = 0.5 * (1.0 - phi);
        acc[0] += na;
        acc[1] += nbv;
        acc[2] += wa;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            acc[5 + c] += u[c];
            acc[8 + c] += wa * u[c];
            acc[11 + c] += wb * u[c];
        }
        if (phi > 0.0) {
            acc[3] += 1.0;
            acc[14] += rho;
            acc[22] += rho / 3.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[16 + c] += rho * u[c];
        } else if (phi < 0.0) {
            acc[4] += 1.0;
            acc[15] += rho;
            acc[23] += rho / 3.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[19 + c] += rho * u[c];
        }
        acc[24] += bad ? 1.0 : 0.0;
    }
    __shared__ double lds[kRedThreads / 64][kNRed];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kNRed; ++k) {
        const double s = wave_sum(acc[k]);
        if (lane == 0) lds[wave][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < kNRed) {
        double s = 0.0;
        for (int w = 0; w < kRedThreads / 64; ++w) s += lds[w][threadIdx.x];
        partials[(size_t)blk * kNRed + threadIdx.x] = s;
    }
}

template <int PREC, bool ODD>
__global__ void __launch_bounds__(kRedThreads) reduce_kernel(StepArgs a,
                                                             double* __restrict__ partials) {
    reduce_block<PREC, ODD>(a, blockIdx.x, partials);
}

// One group of kRedBlocks blocks per pool slot, with the single-domain decomposition, so a
// slot's sums are bitwise those of lbm_reduce on the domain alone. Empty slots (N = 0) give 0.
template <int PREC, bool ODD>
__global__ void __launch_bounds__(kRedThreads) reduce_batched(BatchArgs b,
                                                              double* __restrict__ partials) {
    const int slot = blockIdx.x / kRedBlocks;
    const StepArgs a = batch_args(b, slot);
    reduce_block<PREC, ODD>(a, blockIdx.x % kRedBlocks,
                            partials + (size_t)slot * kRedBlocks * kNRed);
}

// Sum of each group's nblocks partial records (kNRed values each); one workgroup of
// kFinalThreads per group. Thread t adds the records t, t + kFinalThreads, ... in that order,
// each wave combines its threads with the fixed butterfly, and the waves' sums are added in
// wave order: the same order on every call, whatever the timing.
constexpr int kFinalThreads = 256;

__global__ void __launch_bounds__(kFinalThreads) reduce_final_kernel(
    const double* __restrict__ partials, int nblocks, double* __restrict__ out) {
    const double* p = partials + (size_t)blockIdx.x * nblocks * kNRed;
    double acc[kNRed];
#pragma unroll
    for (int k = 0; k < kNRed; ++k) acc[k] = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kFinalThreads) {
#pragma unroll
        for (int k = 0; k < kNRed; ++k) acc[k] += p[(size_t)b * kNRed + k];
    }
    __shared__ double lds[kFinalThreads / 64][kNRed];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kNRed; ++k) {
        const double s = wave_sum(acc[k]);
        if (lane == 0) lds[wave][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < kNRed) {
        double s = 0.0;
        for (int w = 0; w < kFinalThreads / 64; ++w) s += lds[w][threadIdx.x];
        out[(size_t)blockIdx.x * kNRed + threadIdx.x] = s;
    }
}

// ------------------------------------------------------------------------------------------
// Field read-back for pore voxels (pore order), in FP64.
// ------------------------------------------------------------------------------------------
template <int PREC, bool ODD>
__global__ void __launch_bounds__(256) field_kernel(StepArgs a, int field,
                                                    double* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.N) return;
    double v;
    if (field <= LBM_FIELD_PHI) {   // N_a, N_b, phi: the components alone (a third of the bytes)
        double na, nbv;
        int ghost;
        densities<PREC>(a, i, *a.fresh, na, nbv, ghost);
        out[i] = field == LBM_FIELD_NA   ? na
                 : field == LBM_FIELD_NB ? nbv
                                         : (na - nbv) / (na + nbv);
        return;
    }
    double rho, jx, jy, jz;
    voxel_flow<PREC, ODD>(a, i, rho, jx, jy, jz);
    switch (field) {
    case LBM_FIELD_RHO: v = rho; break;
    case LBM_FIELD_P: v = rho / 3.0; break;
    case LBM_FIELD_UX: v = jx + 0.5 * a.F[0]; break;
    case LBM_FIELD_UY: v = jy + 0.5 * a.F[1]; break;
    default: v = jz + 0.5 * a.F[2]; break;
    }
    out[i] = v;
}

// ------------------------------------------------------------------------------------------
// Pressure faces. Across the z faces the colour gradient mirrors the plane: the tail entry that
// stands for an out-of-domain z neighbour carries the phi of the in-plane voxel, written by the
// phase kernel beside that voxel's own. The collide kernel applies the pressure condition to the
// populations of a face voxel as it reads them; pressure_bc_kernel applies it to the stored state
// where a stretch of steps ends, and after every step of a flux inlet, whose density is known
// only then. (With a kernel of their own each, ghosts and faces took 10 of 128^3's 55 us a step.)
// The kernel reads and writes in the layout of the next step (parity ODD); the unknowns always
// sit in the voxel's own slot q, because their upstream neighbour is outside. The first collide
// kernel on a state that no step of this domain has made takes its face populations as they are
// (fresh[1]): at rest there is no condition yet, and a loaded state was settled where it was saved,
// perhaps under other densities than this domain's.
// ------------------------------------------------------------------------------------------
template <int PREC, bool ODD>
__global__ void __launch_bounds__(256) pressure_bc_kernel(StepArgs a,
                                                          const int32_t* __restrict__ faces,
                                                          int n_in, int n_out, double rho_in,
                                                          double rho_out,
                                                          const double* __restrict__ rho_in_dev) {
    using P = Prec<PREC>;
    using F = typename P::F;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_in + n_out) return;
    const int i = faces[k];
    const int fc = k < n_in ? 1 : 2;
    F* f = (F*)a.f;
    int r[19];
    r[0] = i;
    const Pos pos = pos_of(a, i);
#pragma unroll
    for (int q = 1; q < 19; ++q) r[q] = nb_stream(a, q, i, pos);
    F fl[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) fl[q] = load_in<ODD>(f, a, q, i, r[OPP[q]]);
    pressure_face<PREC>(fl, fc, fc == 1 ? (rho_in_dev ? *rho_in_dev : rho_in) : rho_out);
#pragma unroll
    for (int q = 1; q < 19; ++q)
        if (CZ[q] == (fc == 1 ? 1 : -1)) f[(size_t)q * a.ld + i] = fl[q];
}

// Flux inlet: sum over the inlet voxels of s0 + 2 sout (the known part of each voxel's
// j_z = rho - s0 - 2 sout under the pressure condition), then the density that makes the summed
// flow velocity u_z = j_z + F_z/2 equal the imposed flux. A fixed grid of kInletBlocks
// workgroups of kInletThreads threads with a fixed stride writes one partial sum per workgroup;
// one workgroup adds them in a fixed tree order, so the result does not depend on timing.
constexpr int kInletBlocks = 256;
constexpr int kInletThreads = 256;

template <int PREC, bool ODD>
__global__ void __launch_bounds__(kInletThreads) inlet_partial_kernel(
    StepArgs a, const int32_t* __restrict__ faces, int n_in, double* __restrict__ partial) {
    using P = Prec<PREC>;
    using F = typename P::F;
    __shared__ double acc[kInletThreads];
    const F* f = (const F*)a.f;
    double s = 0.0;
    for (int k = blockIdx.x * kInletThreads + threadIdx.x; k < n_in;
         k += kInletBlocks * kInletThreads) {
        const int i = faces[k];
        int r[19];
        r[0] = i;
        const Pos pos = pos_of(a, i);
#pragma unroll
        for (int q = 1; q < 19; ++q) r[q] = nb_stream(a, q, i, pos);
        double s0 = 0.0, sout = 0.0;
#pragma unroll
        for (int q = 0; q < 19; ++q) {
            const double fq = (double)load_in<ODD>(f, a, q, i, r[OPP[q]]) + (P::kDev ? tw(q) : 0.0);
            if (CZ[q] == 0) s0 += fq;
            else if (CZ[q] == -1) sout += fq;
        }
        s += s0 + 2.0 * sout;
    }
    acc[threadIdx.x] = s;
    __syncthreads();
    for (int h = kInletThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) acc[threadIdx.x] += acc[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = acc[0];
}

__global__ void __launch_bounds__(kInletBlocks) inlet_finish_kernel(
    const double* __restrict__ partial, int n_in, double flux, double fz,
    double* __restrict__ rho_in_dev) {
    __shared__ double acc[kInletBlocks];
    acc[threadIdx.x] = partial[threadIdx.x];
    __syncthreads();
    for (int h = kInletBlocks / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) acc[threadIdx.x] += acc[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        rho_in_dev[0] = (flux - (double)n_in * 0.5 * fz + acc[0]) / (double)n_in;
}

int grid_for(const StepArgs& a, int block) { return (a.N + block - 1) / block; }

}  // namespace

// ------------------------------------------------------------------------------------------
// Launchers: dispatch on precision and step parity (the step kernels also on the lookup).
// ------------------------------------------------------------------------------------------
// One launch of KERNEL<P, odd> (or KERNEL<P, odd, NB>) for the precision P of the domain.
#define LBM_LAUNCH_ODD(KERNEL, P, GRID, BLOCK, ...)                                            \
    do {                                                                                       \
        if (odd)                                                                               \
            hipLaunchKernelGGL((KERNEL<P, true>), GRID, BLOCK, 0, s, __VA_ARGS__);             \
        else                                                                                   \
            hipLaunchKernelGGL((KERNEL<P, false>), GRID, BLOCK, 0, s, __VA_ARGS__);            \
    } while (0)

#define LBM_LAUNCH_ODD_NB(KERNEL, P, NBV, GRID, BLOCK, ...)                                    \
    do {                                                                                       \
        if (odd && face)                                                                       \
            hipLaunchKernelGGL((KERNEL<P, true, NBV, true>), GRID, BLOCK, 0, s, __VA_ARGS__);  \
        else if (odd)                                                                          \
            hipLaunchKernelGGL((KERNEL<P, true, NBV, false>), GRID, BLOCK, 0, s, __VA_ARGS__); \
        else if (face)                                                                         \
            hipLaunchKernelGGL((KERNEL<P, false, NBV, true>), GRID, BLOCK, 0, s, __VA_ARGS__); \
        else                                                                                   \
            hipLaunchKernelGGL((KERNEL<P, false, NBV, false>), GRID, BLOCK, 0, s, __VA_ARGS__); \
    } while (0)

#define LBM_PREC_SWITCH(PREC, LAUNCH, KERNEL, ...)                                             \
    do {                                                                                       \
        if ((PREC) == LBM_FP32_DEV)                                                            \
            LAUNCH(KERNEL, LBM_FP32_DEV, __VA_ARGS__);                                         \
        else if ((PREC) == LBM_FP32_MIXED)                                                     \
            LAUNCH(KERNEL, LBM_FP32_MIXED, __VA_ARGS__);                                       \
        else                                                                                   \
            LAUNCH(KERNEL, LBM_FP64, __VA_ARGS__);                                             \
    } while (0)

#define LBM_DISPATCH(KERNEL, GRID, BLOCK, ...)                                                 \
    LBM_PREC_SWITCH(a.prec, LBM_LAUNCH_ODD, KERNEL, GRID, BLOCK, __VA_ARGS__)

hipError_t launch_init(const StepArgs& a, const double* phi0, int block, hipStream_t s) {
    (void)block;
    if (a.prec == LBM_FP32_DEV)
        hipLaunchKernelGGL(init_kernel<LBM_FP32_DEV>, dim3(grid_for(a, 256)), dim3(256), 0, s,
                           a, phi0);
    else if (a.prec == LBM_FP32_MIXED)
        hipLaunchKernelGGL(init_kernel<LBM_FP32_MIXED>, dim3(grid_for(a, 256)), dim3(256), 0, s,
                           a, phi0);
    else
        hipLaunchKernelGGL(init_kernel<LBM_FP64>, dim3(grid_for(a, 256)), dim3(256), 0, s, a,
                           phi0);
    return hipGetLastError();
}

// The step kernel (0: phase, 1: collide, 2: phase outside a step) of a domain, by precision, parity,
// neighbour lookup, streaming accesses, load order and pressure faces (whose code costs the collide
// kernel registers: with the compact lookup 158 for 120 to 128 in FP64, 140 for 120 to 124 in
// FP32-mixed, 120 for 77 to 113 in FP32-dev). The phase kernel is the same at both parities.
using StepKernel = void (*)(StepArgs);

template <int P, int NB, bool ST, bool FACE>
static StepKernel step_kernel_fn(const StepArgs& a, int kernel, bool odd) {
    if (kernel == 0) return phase_kernel<P, NB, ST, FACE, false>;
    if (kernel == 2) return phase_kernel<P, NB, ST, FACE, true>;
    if (!ST && a.N <= kEarlyVoxels)
        return odd ? collide_kernel<P, true, NB, false, true, FACE>
                   : collide_kernel<P, false, NB, false, true, FACE>;
    return odd ? collide_kernel<P, true, NB, ST, false, FACE>
               : collide_kernel<P, false, NB, ST, false, FACE>;
}

// The collide kernel needs its face code only where it applies the condition itself (a flux inlet
// and a single plane have kernels for that after every step); the phase kernel for any face.
template <int P, int NB, bool ST>
static StepKernel step_kernel_fn(const StepArgs& a, int kernel, bool odd) {
    return (kernel != 1 ? a.face != nullptr : a.face_bc != 0)
               ? step_kernel_fn<P, NB, ST, true>(a, kernel, odd)
               : step_kernel_fn<P, NB, ST, false>(a, kernel, odd);
}

template <int P, bool ST>
static StepKernel step_kernel_fn_nb(const StepArgs& a, int kernel, bool odd) {
    return a.words ? step_kernel_fn<P, NB_RANK, ST>(a, kernel, odd)
           : a.cwave ? step_kernel_fn<P, NB_COMPACT, ST>(a, kernel, odd)
                     : step_kernel_fn<P, NB_TABLE, ST>(a, kernel, odd);
}

template <bool ST>
static StepKernel step_kernel_fn_prec(const StepArgs& a, int kernel, bool odd) {
    if (a.prec == LBM_FP32_DEV) return step_kernel_fn_nb<LBM_FP32_DEV, ST>(a, kernel, odd);
    if (a.prec == LBM_FP32_MIXED) return step_kernel_fn_nb<LBM_FP32_MIXED, ST>(a, kernel, odd);
    return step_kernel_fn_nb<LBM_FP64, ST>(a, kernel, odd);
}

static StepKernel step_kernel(const StepArgs& a, int kernel, bool odd, bool stream) {
    return stream ? step_kernel_fn_prec<true>(a, kernel, odd)
                  : step_kernel_fn_prec<false>(a, kernel, odd);
}

// `lds`: dynamic LDS per workgroup, which the step kernels do not use; it only bounds how many
// workgroups a CU holds at once (see step_kernel_lds).
hipError_t launch_phase(const StepArgs& a, bool odd, int block, bool stream, unsigned lds,
                        hipStream_t s, bool in_step) {
    hipLaunchKernelGGL(step_kernel(a, in_step || a.N <= kEarlyVoxels ? 0 : 2, odd, stream), dim3(a.grid), dim3(block), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_collide(const StepArgs& a, bool odd, int block, bool stream, unsigned lds,
                          hipStream_t s) {
    hipLaunchKernelGGL(step_kernel(a, 1, odd, stream), dim3(a.grid), dim3(block), lds, s, a);
    return hipGetLastError();
}

// Occupancy limit. Fewer resident waves can be faster for these kernels: their in-flight
// working set (a wave's gathers, the partially written lines of the odd step) competes for the
// 4 MB L2 of an XCD, and past some occupancy the lines neighbouring voxels share are evicted
// before they are reused. The hardware holds a workgroup only where its LDS fits, so reserving
// LDS that the kernel never touches bounds the workgroups per CU. The smallest such reservation
// (in 256-byte steps) that keeps both parities of the kernel at or below `wg` workgroups per CU
// is found with the runtime's occupancy calculator; 0 where the registers already allow no
// more, or for wg == 0 (no limit).
hipError_t step_kernel_lds(const StepArgs& a, int kernel, int block, bool stream, int wg,
                           unsigned* lds) {
    *lds = 0;
    if (wg <= 0) return hipSuccess;
    int dev = 0, max_lds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    unsigned need = 0;
    for (int odd = 0; odd < 2; ++odd) {
        const void* fn = (const void*)step_kernel(a, kernel, odd != 0, stream);
        auto blocks = [&](unsigned bytes, int* n) {
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, fn, block, bytes);
        };
        int n = 0;
        if ((e = blocks(0, &n)) != hipSuccess) return e;
        if (n <= wg) continue;
        unsigned lo = 0, hi = (unsigned)max_lds & ~255u;   // blocks(lo) > wg
        if ((e = blocks(hi, &n)) != hipSuccess) return e;
        if (n > wg) {   // even the largest reservation cannot bound it this far
            need = std::max(need, hi);
            continue;
        }
        while (hi - lo > 256) {
            const unsigned mid = ((lo + hi) / 2) & ~255u;
            if ((e = blocks(mid, &n)) != hipSuccess) return e;
            (n <= wg ? hi : lo) = mid;
        }
        need = std::max(need, hi);
    }
    *lds = need;
    return hipSuccess;
}

hipError_t launch_reduce(const StepArgs& a, bool odd, double* partials, double* out,
                         hipStream_t s) {
    LBM_DISPATCH(reduce_kernel, dim3(kRedBlocks), dim3(kRedThreads), a, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(kFinalThreads), 0, s, partials,
                       kRedBlocks, out);
    return hipGetLastError();
}

#define LBM_DISPATCH_B(KERNEL, GRID, BLOCK, ...)                                               \
    LBM_PREC_SWITCH(prec, LBM_LAUNCH_ODD, KERNEL, GRID, BLOCK, __VA_ARGS__)

#define LBM_LAUNCH_NB(KERNEL, P, NBV, GRID, BLOCK, ...)                                        \
    do {                                                                                       \
        if (face)                                                                              \
            hipLaunchKernelGGL((KERNEL<P, NBV, true>), GRID, BLOCK, 0, s, __VA_ARGS__);        \
        else                                                                                   \
            hipLaunchKernelGGL((KERNEL<P, NBV, false>), GRID, BLOCK, 0, s, __VA_ARGS__);       \
    } while (0)

#define LBM_DISPATCH_B_NB(LAUNCH, KERNEL, GRID, BLOCK, ...)                                            \
    do {                                                                                       \
        if (lookup == LBM_NBR_TABLE)                                                           \
            LBM_PREC_SWITCH(prec, LAUNCH, KERNEL, NB_TABLE, GRID, BLOCK, __VA_ARGS__); \
        else if (lookup == LBM_NBR_COMPACT)                                                    \
            LBM_PREC_SWITCH(prec, LAUNCH, KERNEL, NB_COMPACT, GRID, BLOCK,          \
                            __VA_ARGS__);                                                      \
        else if (lookup == LBM_NBR_RANK)                                                       \
            LBM_PREC_SWITCH(prec, LAUNCH, KERNEL, NB_RANK, GRID, BLOCK, __VA_ARGS__); \
        else                                                                                   \
            LBM_PREC_SWITCH(prec, LAUNCH, KERNEL, NB_DYN, GRID, BLOCK, __VA_ARGS__); \
    } while (0)

hipError_t launch_phase_batched(const BatchArgs& b, int prec, int lookup, bool face, int grid,
                                int block, hipStream_t s) {
    LBM_DISPATCH_B_NB(LBM_LAUNCH_NB, phase_batched, dim3(grid), dim3(block), b);
    return hipGetLastError();
}

hipError_t launch_collide_batched(const BatchArgs& b, int prec, bool odd, int lookup, bool face,
                                  int grid, int block, hipStream_t s) {
    LBM_DISPATCH_B_NB(LBM_LAUNCH_ODD_NB, collide_batched, dim3(grid), dim3(block), b);
    return hipGetLastError();
}

hipError_t launch_reduce_batched(const BatchArgs& b, int prec, bool odd, int nslots,
                                 double* partials, double* out, hipStream_t s) {
    if (nslots <= 0) return hipSuccess;
    LBM_DISPATCH_B(reduce_batched, dim3(nslots * kRedBlocks), dim3(kRedThreads), b, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_final_kernel, dim3(nslots), dim3(kFinalThreads), 0, s, partials,
                       kRedBlocks, out);
    return hipGetLastError();
}

hipError_t launch_field(const StepArgs& a, bool odd, int field, double* out, int block,
                        hipStream_t s) {
    (void)block;
    LBM_DISPATCH(field_kernel, dim3(grid_for(a, 256)), dim3(256), a, field, out);
    return hipGetLastError();
}

// ---- Densities of a saved state
namespace {
template <typename S>
__global__ void __launch_bounds__(256) densities_out_kernel(StepArgs a, int i0, int n,
                                                            S* __restrict__ pairs) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    S na, nb;
    sent<S>(((const S*)a.phi_prev)[i0 + k], ((const S*)a.ntot_prev)[i0 + k], *a.fresh != 0, na, nb);
    store_pair<S>(pairs, 0, 0, k, na, nb);
}

template <typename S>
__global__ void __launch_bounds__(256) densities_in_kernel(StepArgs a,
                                                           const S* __restrict__ pairs) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.N) return;
    const auto v = load_pair<S>(pairs, 0, 0, i);
    ((S*)a.phi_prev)[i] = v.x;
    ((S*)a.ntot_prev)[i] = v.y;
}
}  // namespace

hipError_t launch_densities_out(const StepArgs& a, int32_t i0, int32_t n, void* pairs,
                                hipStream_t s) {
    const dim3 grid((n + 255) / 256);
    if (a.prec == LBM_FP32_DEV)
        hipLaunchKernelGGL(densities_out_kernel<float>, grid, dim3(256), 0, s, a, i0, n,
                           (float*)pairs);
    else
        hipLaunchKernelGGL(densities_out_kernel<double>, grid, dim3(256), 0, s, a, i0, n,
                           (double*)pairs);
    return hipGetLastError();
}

hipError_t launch_densities_in(const StepArgs& a, const void* pairs, hipStream_t s) {
    const dim3 grid(grid_for(a, 256));
    if (a.prec == LBM_FP32_DEV)
        hipLaunchKernelGGL(densities_in_kernel<float>, grid, dim3(256), 0, s, a,
                           (const float*)pairs);
    else
        hipLaunchKernelGGL(densities_in_kernel<double>, grid, dim3(256), 0, s, a,
                           (const double*)pairs);
    return hipGetLastError();
}

hipError_t launch_pressure_bc(const StepArgs& a, bool next_odd, const int32_t* faces,
                              int32_t n_in, int32_t n_out, double rho_in, double rho_out,
                              const double* rho_in_dev, hipStream_t s) {
    const int n = n_in + n_out;
    if (n <= 0) return hipSuccess;
    const dim3 grid((n + 255) / 256);
    const bool odd = next_odd;
    LBM_DISPATCH(pressure_bc_kernel, grid, dim3(256), a, faces, n_in, n_out, rho_in, rho_out,
                 rho_in_dev);
    return hipGetLastError();
}

hipError_t launch_inlet_density(const StepArgs& a, bool next_odd, const int32_t* faces,
                                int32_t n_in, double flux, double* rho_in_dev, double* partial,
                                hipStream_t s) {
    if (n_in <= 0) return hipSuccess;
    const bool odd = next_odd;
    LBM_DISPATCH(inlet_partial_kernel, dim3(kInletBlocks), dim3(kInletThreads), a, faces, n_in,
                 partial);
    if (hipError_t e = hipGetLastError()) return e;
    hipLaunchKernelGGL(inlet_finish_kernel, dim3(1), dim3(kInletBlocks), 0, s,
                       (const double*)partial, n_in, flux, a.F[2], rho_in_dev);
    return hipGetLastError();
}

}  // namespace lbm
