// Internal declarations shared by the runtime (lbm_runtime.hip), the pre-pass
// (lbm_prepass.cpp) and the kernels (lbm_kernels.hip). Not part of the C-ABI.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include <hip/hip_runtime.h>

#include "../../include/lbm.h"
#include "lbm_prepass.h"

namespace lbm {

// Number of FP64 accumulators of the reduction kernel, in this order:
//  0 M_a  1 M_b  2 sum (1+phi)/2  3 V_a (#phi>0)  4 V_b (#phi<0)  5..7 sum u
//  8..10 sum (1+phi)/2 u  11..13 sum (1-phi)/2 u  14 sum rho over phi>0  15 over phi<0
//  16..18 sum rho u over phi>0  19..21 over phi<0  22 sum p over phi>0  23 over phi<0
//  24 count of non-finite voxels
constexpr int kNRed = 25;
constexpr int kRedBlocks = 512;   // fixed launch shape of the reduction => fixed summation order
constexpr int kRedThreads = 256;

// Arguments of the step kernels (passed by value).
struct StepArgs {
    int32_t N;          // pore voxels
    int32_t block;      // threads per workgroup of the step kernels (voxels per tile)
    int64_t ld;         // leading dimension of population arrays
    const int32_t* nbr; // [9][ld][2]: neighbours along (q, q + 1) for q = 1, 3, ..., 17
    void* phi;          // [N + n_tail] in the storage type: this step's phase indicator, written by
    void* ntot;         //   the phase kernel; the tail holds phi_s. [N]: this step's N = N_a + N_b
    void* phi_prev;     // the same of the step before, from which the phase kernel has the
    void* ntot_prev;    //   densities that the components left with (see `fresh` for a state that
                        //   no step has made). The pairs of buffers alternate by step parity.
    void* f;            // [19][ld] populations (storage type per precision)
    void* M;            // [3][ld][2] D3Q7 moment slot pairs: (u_x, G_x), (u_y, G_y), (u_z, G_z)
    int32_t* fresh;     // device flags: [0] 0 while phi_prev and ntot_prev are a step's; else they
                        // hold N_a and N_b themselves: 1 in a state at rest (initial, or after a
                        // morphological step), 2 in a state that was loaded; [1] whether [0] was
                        // set at the step's phase kernel, for the collide kernel that clears [0]
                        // and takes the face populations of such a state as they are
    const int8_t* face; // per pore voxel: 0, 1 (inlet face), 2 (outlet face); null without faces
    double nu_a, nu_b;  // kinematic viscosities
    double alpha, beta;
    double F[3];
    double rho_face[2]; // imposed densities of the inlet and the outlet face
    int32_t face_bc;    // 1: the collide kernel applies the pressure condition (fixed densities)
    int32_t grid;       // workgroups of a step kernel's launch
    int32_t xcd_run;    // tiles per run of the XCD-aware order (1: launch order)
    uint32_t xcd_mul;   // xcd_mul_of(xcd_run)
    int32_t tile_first; // a workgroup takes tile tile_first + tile_sign * (its place in the
    int32_t tile_sign;  //   order): 0 and 1, or grid - 1 and -1 for the order from the end
    int32_t prec;       // lbm_precision
    // Rank lookup of neighbours (used instead of nbr when words != null):
    const uint32_t* coord;   // [ld] packed (x, y, z) of each pore voxel
    const RowWord* words;    // [nz][ny][W] 64-voxel row segments
    // Compact lookup (used instead of nbr when cwave != null; layout in lbm_prepass.h):
    const uint2* cn8;        // [ld] byte waves: axis codes; 16-bit waves: codes of q = 15..18
    const uint4* cn16;       // [ld] codes of q = 7..18 (byte waves) or 7..14
    const uint4* cwide;      // [ld] 16-bit waves: mask and codes of q = 1..6
    const int32_t* cwave;    // [ld / 64][kCompactWaveInts] bases, exception row, kind
    const int32_t* cex;      // [exception waves][18][64] int32 targets
    int32_t nx, ny, nz, W;
    int32_t periodic;        // bit a set: axis a is periodic
    int32_t bc_z;            // 1: z neighbours beyond the faces mirror the plane
};

// Arguments of the batched (pool) kernels. All arrays live in device memory.
// XCD-aware tile order: the hardware deals workgroups round-robin to the 8 XCDs; each XCD is
// given runs of consecutive tiles, the runs interleaved (grid a multiple of 8 runs). kXcdRun is
// the run length of the batched launches and the default of a domain's own launches, which may
// choose any length up to kMaxXcdRun for each kernel and step parity (lbm_tuning).
constexpr int kXcdRun = 16;
// The factor whose product with j, shifted right by 31, is j / run (see xcd_run_tile).
constexpr uint32_t xcd_mul_of(int run) {
    return (uint32_t)(((uint64_t(1) << 31) + (uint32_t)run - 1) / (uint32_t)run);
}
constexpr int kMaxXcdRun = 64;

// Steps in the captured chunk of the single-domain step loop (even, so every chunk starts and
// ends on an even step).
constexpr int64_t kStepGraphChunk = 64;

// Device memory above which a new domain launches its step kernels with streaming
// (non-temporal) accesses and the collide runs that go with them: one and a half times the
// MI355X Infinity Cache (256 MB) in FP64 and FP32-mixed, twice in FP32-dev, so that a domain the
// cache holds from one step to the next keeps that reuse. us a step without / with, porosity 0.2:
// FP64 302 MB 105.1 / 105.2, 370 MB 134.3 / 134.5, 447 MB 166.3 / 153.2, 541 MB 206 / 186;
// FP32-mixed 336 MB 118.6 / 118.2, 406 MB 148.1 / 142.5, 500 MB 186 / 169; FP32-dev 329 MB
// 111.7 / 115.1, 405 MB 136.0 / 137.6. With the rank lookup, whose row records are read again and
// again, twice the cache in every precision, and no workgroup limits below it: their dependent
// loads need the waves. us a step without / with what the other lookups get, porosity 0.25: 1.0 M
// voxels FP64 104.9 / 122.4, FP32-mixed 88.9 / 97.6, FP32-dev 80.1 / 89.2; 2.0 M voxels FP64
// 277.7 / 298.5, FP32-mixed 223.2 / 236.6, FP32-dev 144.4 / 166.0; 4.1 M (both stream) 623.2 / 625.3,
// 500.8 / 493.8, 426.2 / 417.5.
constexpr int64_t stream_bytes(int32_t precision, bool rank) {
    return int64_t(precision == LBM_FP32_DEV || rank ? 512 : 384) << 20;
}

// Fewest pore voxels of a domain (not with the rank lookup) whose kernels get the per-CU workgroup
// limits of a large one without its streaming. us a step without / with limits: FP64 0.79 M voxels 68.5 / 68.5, 0.98 M
// 105.1 / 101.9, 1.2 M 134.3 / 131.3; FP32-mixed 0.79 M 51.1 / 50.3, 1.2 M 89.1 / 87.0; FP32-dev
// 0.98 M 51.8 / 51.4. Below, they gain nothing in FP64 (0.6 M: 54.1 / 54.1) and cost a 524
// thousand voxel domain in FP32-dev a percent.
constexpr int64_t kLimitVoxels = int64_t(3) << 18;

// Most pore voxels of a domain that steps in workgroups of 64 by default: with 256, fewer than
// half of the CUs have one. us a step with 256 / 64: FP64 19,660 voxels 8.06 / 7.06, 27,648 8.29 /
// 7.48; FP32-dev 19,660 7.29 / 6.47; but 65,536 voxels in FP32-mixed 8.29 / 8.73.
constexpr int64_t kSmallVoxels = int64_t(1) << 15;

// Most pore voxels of a domain whose collide kernel issues all its loads first (EARLY in
// lbm_kernels.hip): up to about four waves per SIMD. Above, other waves hide the round trip that
// it saves, and its registers only cost occupancy. Measured as a whole pass: 20 thousand voxels
// +6%, 65 thousand +7%, 524 thousand -0.2% (FP64) and -1.2% (FP32-dev, 110 registers for 76).
constexpr int32_t kEarlyVoxels = 1 << 18;

// Largest per-CU workgroup limit a launch configuration may ask for (lbm_tuning.*_wg).
constexpr int kMaxWgPerCu = 16;

struct BatchArgs {
    const StepArgs* doms;       // per-slot kernel arguments (N = 0 for an empty slot)
    const int32_t* tile_dom;    // slot of each tile
    const int32_t* tile_first;  // first tile of each slot
    const int32_t* ntiles;      // number of tiles in use (device scalar)
    int32_t xcd;                // 1: XCD-aware tile order (grid a multiple of 8 * 16)
    int32_t odd;                // parity of the step (doms holds the arguments of even steps)
};

// Kernel launchers (lbm_kernels.hip). `odd` is the parity of the step being taken.
hipError_t launch_init(const StepArgs& a, const double* phi0, int block, hipStream_t s);
// in_step false: the phase of the current state for a reader, which may find it at rest.
hipError_t launch_phase(const StepArgs& a, bool odd, int block, bool stream, unsigned lds,
                        hipStream_t s, bool in_step = true);
hipError_t launch_collide(const StepArgs& a, bool odd, int block, bool stream, unsigned lds,
                          hipStream_t s);
// Dynamic LDS that bounds a step kernel (0: phase, 1: collide) to `wg` workgroups per CU.
hipError_t step_kernel_lds(const StepArgs& a, int kernel, int block, bool stream, int wg,
                           unsigned* lds);
// faces: inlet pore indices (n_in) followed by outlet ones (n_out); next_odd: parity of the
// step that will read the state the condition is applied to.
// rho_in_dev (nullable): device scalar that replaces rho_in (flux inlet).
hipError_t launch_pressure_bc(const StepArgs& a, bool next_odd, const int32_t* faces,
                              int32_t n_in, int32_t n_out, double rho_in, double rho_out,
                              const double* rho_in_dev, hipStream_t s);
// Flux inlet: the inlet density for which the flow velocity summed over the n_in inlet voxels
// (faces[0..n_in)) equals flux, written to *rho_in_dev (fixed grid and order; partial holds at
// least 256 doubles of scratch).
hipError_t launch_inlet_density(const StepArgs& a, bool next_odd, const int32_t* faces,
                                int32_t n_in, double flux, double* rho_in_dev, double* partial,
                                hipStream_t s);
hipError_t launch_reduce(const StepArgs& a, bool odd, double* partials, double* out,
                         hipStream_t s);
// lookup: LBM_NBR_TABLE or LBM_NBR_RANK when every member uses that neighbour lookup, else
// LBM_NBR_AUTO (each tile tests its domain's lookup at run time).
// face: whether any member has pressure faces; for the collide kernel, faces whose condition it
// applies itself.
hipError_t launch_phase_batched(const BatchArgs& b, int prec, int lookup, bool face, int grid,
                                int block, hipStream_t s);
hipError_t launch_collide_batched(const BatchArgs& b, int prec, bool odd, int lookup, bool face,
                                  int grid, int block, hipStream_t s);
// Reductions of slots 0..nslots-1 into out[nslots][kNRed]; partials holds nslots*kRedBlocks rows.
hipError_t launch_reduce_batched(const BatchArgs& b, int prec, bool odd, int nslots,
                                 double* partials, double* out, hipStream_t s);
hipError_t launch_field(const StepArgs& a, bool odd, int field, double* out, int block,
                        hipStream_t s);
// The densities (N_a, N_b) that the components of voxels i0 .. i0 + n - 1 left with, as pairs in
// the storage type (saved states hold them), and back for all voxels (flag 2 of `fresh`).
hipError_t launch_densities_out(const StepArgs& a, int32_t i0, int32_t n, void* pairs, hipStream_t s);
hipError_t launch_densities_in(const StepArgs& a, const void* pairs, hipStream_t s);

// Host <-> device copies of large caller buffers (lbm_transfer.hip): staged through pinned
// memory by several host threads while the previous chunk's DMA runs. Ordered on stream s after
// its earlier work; they return once the copy is complete (the stream is synchronised).
hipError_t copy_to_device(void* dst, const void* src, size_t bytes, hipStream_t s);
hipError_t copy_to_host(void* dst, const void* src, size_t bytes, hipStream_t s);

// Pinned host memory of up to kPinnedBytes that a kernel of this call writes its result into (the
// host address is valid on every device). ptr() is null when `bytes` is larger or no memory is to
// be had: the caller then goes through a device buffer.
constexpr size_t kPinnedBytes = size_t(8) << 20;
class PinnedOut {
public:
    explicit PinnedOut(size_t bytes);
    ~PinnedOut();
    PinnedOut(const PinnedOut&) = delete;
    PinnedOut& operator=(const PinnedOut&) = delete;
    void* ptr() const { return ptr_; }
    // Waits for stream s, on which the kernel was launched, and copies the result to dst. Must
    // also run (or the stream be waited for) before the object goes if a launch used ptr().
    hipError_t take(void* dst, size_t bytes, hipStream_t s);

private:
    void* ptr_ = nullptr;
};

// Squared distances between voxel centres for the morphological step (lbm_prep.hip), clipped
// at cap (<= 255): to_a[v] to the nearest voxel whose bit is set in label_bits (rows packed as
// 64-voxel words), to_other[v] to the nearest voxel whose bit is clear or beyond a non-periodic
// face (periodic: bit a for axis a). other_bits receives the complement bits; tmp, to_a and
// to_other hold nx*ny*nz bytes each.
lbm_status morph_distance(int nx, int ny, int nz, int periodic, const uint64_t* label_bits,
                          uint64_t* other_bits, int32_t cap, uint8_t* tmp, uint8_t* to_a,
                          uint8_t* to_other, hipStream_t s);

}  // namespace lbm
