// rmhdlb_internal.h -- declarations shared by the kernels and the C ABI
// implementation of the HIP library (not part of the public interface).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rmhdlb.h"
#include "rmhdlb_device.h"

namespace rmhd {

constexpr int NPART = 26;  // partial diagnostic sums per block: 9 (see k_moments), 16 Newton bins, fallbacks
constexpr int RED_WAVES = 4;

struct InPtrs {
    const double *n, *p;
    const double *u[3], *E[3], *B[3];
    const double* rho_c;
};

// Prescribed fields of a driven face (nx * ny values each).
struct FacePtrs {
    const double *n, *p;
    const double *u[3], *B[3];
};

struct OutPtrs {
    double *n, *p, *eps;
    double *u[3], *E[3], *B[3], *J[3];
    double* rho_c;
};

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
    return x;
}

// Deterministic block sums of W values per thread: butterfly within each
// 64-wide wavefront, then the 4 wavefront results in fixed order.  Thread j
// (j < W) writes sum j to out[j].
template <int W>
__device__ __forceinline__ void block_sum(const double (&v)[W], double* __restrict__ out) {
    __shared__ double sh[W][RED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const double s = wave_sum(v[j]);
        if (lane == 0) sh[j][wave] = s;
    }
    __syncthreads();
    if (threadIdx.x < W) {
        const int j = threadIdx.x;
        out[j] = ((sh[j][0] + sh[j][1]) + (sh[j][2] + sh[j][3]));
    }
}

__device__ __forceinline__ void block_max1(double v, double* __restrict__ out) {
    __shared__ double sh[RED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double m = wave_max(v);
    if (lane == 0) sh[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

__device__ __forceinline__ double block_sum_value(double v) {
    __shared__ double sh[RED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double s = wave_sum(v);
    if (lane == 0) sh[wave] = s;
    __syncthreads();
    const double r = ((sh[0] + sh[1]) + (sh[2] + sh[3]));
    __syncthreads();
    return r;
}

__device__ __forceinline__ double block_max_value(double v) {
    __shared__ double sh[RED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double m = wave_max(v);
    if (lane == 0) sh[wave] = m;
    __syncthreads();
    const double r = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    __syncthreads();
    return r;
}

int num_tiles(const Consts& K);

// Arrays of the raw (interface) state: F[19], G[19], h*[25], E_prev[3], and
// B_prev[3] with the previous-B reading.
__host__ __device__ inline int state_arrays(const Consts& K) { return NSTATE + (K.bprev ? 3 : 0); }

// Launch shape of the fused step: z-planes walked per block, the tile width
// along x (64, 32 or 16 cells; a row group has cells_per_block cells, in
// StepWalk::zt planes), the number of blocks that walk a column's chunk of
// zg * zb planes interleaved, and the row groups per block stacked along y.
struct StepTuning {
    int zb;
    int px;
    int zg = 1;
    int yw = 1;
};

// One instance of a batched step: its constants, both state buffers, its
// face-pass output, its launch geometry and its first block and face-pass thread in the batched launches.
struct BatchInst {
    Consts K;
    char* buf[2];
    double* faceB;
    int tiles_x, ncol, zb, zt, yw, nblk;
    int64_t blk0;
    int64_t face0;
};

struct GuessTables;

// Normalisation of the learned guess's inputs and targets (training-set
// mean and standard deviation).
struct Norm4 {
    double mu_x[6], sd_x[6], mu_t[2], sd_t[2];
};

constexpr int SAMPLE_SUMS = 17;  // per-block sums of the sampling pass: F, F^2 (6 each), T, T^2 (2 each), failed

struct TrainArgs {
    const float* X;   // n x 6 normalised inputs
    const float* Yt;  // n x 2 normalised targets
    int n, batch, iters, stride;
    float lr;
    float* w;         // MLP_NP master weights: initial on entry, trained on exit
    float* m;         // Adam moments (zero on entry)
    float* v;
    float* losses;    // loss of every iteration (may be null)
    float* grad;      // gradient-only mode: the gradient of the batch
    float* y;         // gradient-only mode: the outputs, n x 2 (may be null)
    int grad_only;
};



// Storage type -> (E_prev storage type, arithmetic type of the step).
template <typename TS>
struct StoreTypes;
template <>
struct StoreTypes<double> {
    using E = double;
    using V = double;
};
template <>
struct StoreTypes<float> {
    using E = float;
    using V = float;
};
template <>
struct StoreTypes<_Float16> {
    using E = float;
    using V = float;
};

// Device buffers of the diagnostics pass.
struct DiagBufs {
    double* faceB;    // adjusted normal B of the open-face cells (Consts::fo layout)
    double* scratch;  // 4 N: B of every cell, then E^z
    double* part;     // NPART per tile
    double* part2;    // max |div B| per tile
    double* nullp;    // (key, cell) per tile
    const double* ez0;  // initial E^z
    const double* b0;   // max |B| of the initial fields
    double* result;   // NPART sums, max |div B|, R, null cell, B0
};

// gt: inference tables of the learned recovery guess, or nullptr for the
// plain recovery (Newton from E_f).
template <typename TS>
hipError_t launch_step(const char* src, char* dst, const Consts& K, const StepTuning& tune,
                       double* faceB, const GuessTables* gt, hipStream_t s);
template <typename TS>
hipError_t launch_moments(const char* src, const Consts& K, const OutPtrs& out, const DiagBufs& D,
                          const GuessTables* gt, hipStream_t s);
hipError_t launch_face_check(const FacePtrs& in, const Consts& K, double* part, double* result, hipStream_t s);
template <typename TS>
hipError_t launch_ghost(const FacePtrs& in, const Consts& K, char* dst, hipStream_t s);
hipError_t launch_init_ref(const InPtrs& in, const Consts& K, double* part, double* result, hipStream_t s);
template <typename TS>
hipError_t launch_face_b(const char* src, const Consts& K, double* faceB, hipStream_t s);
// Whether the step takes the kernels for a single z-plane: there every
// z-displacement of the stencil leads back to the cell itself (periodic or
// open z; a driven face has planes below it), and 54 of a cell's 168 reads of
// f fall on points already read.  ms per step, general -> flat: KH slab
// 1024 x 2048 FP64 0.581 -> 0.541, sweep of 25.2 M cells FP32 4.19 -> 3.60.
inline bool flat_grid(const Consts& K) { return K.nz == 1 && !K.drv; }
// Cells per row group of a fused-step block: 128 in the pair layout (FP64 storage, elem = 8 bytes, two lanes
// per cell), 256 in the quad and double-quad layouts (FP32 and FP16 storage, one lane per cell).
__host__ __device__ constexpr int cells_per_block(int elem) { return elem == 8 ? 128 : 256; }
// Most z-planes of a fused-step tile: two in FP64 and FP32 where the rows suffice
// (at least four), so that half of the z-neighbour planes of the stencil are
// the tile's own: 56 instead of 68 lines of L1 per 128 cells and direction
// (FP64 at px = 32), ms per step at 256x256x512 one / two planes FP64 9.9 / 9.36, FP32
// 4.9 / 4.75 (wavefronts in step).  FP16 is 1 % faster with one plane.
__host__ __device__ constexpr int most_planes(int elem, int px, bool flat) {
    return flat || elem == 2 || cells_per_block(elem) / px < 4 ? 1 : 2;
}
// Blocks of a step whose tiles hold one plane and walk one.
inline int64_t plane_blocks(const Consts& K, int px, int yw, int elem) {
    const int py = cells_per_block(elem) / px * yw;
    return (int64_t)((K.nx + px - 1) / px) * ((K.ny + py - 1) / py) * K.nz;
}
// What a tuning's zb becomes: the planes of a tile and those that a block
// walks, at most the grid's and whole tiles (an odd number is rounded up).
// A walk of a single plane takes tiles of one where the step then has a block
// for every CU (blocks: plane_blocks, or their sum in a batch): in tiles of two half of
// every block finds no rows (64x64x32 cells, 512 blocks of FP32 64-wide, 22.5 us per step with one
// plane, 26.5 with two; FP64 32-wide 1024 blocks 40.3 and 51.1).  With fewer
// blocks the half-filled ones spread the same wavefronts over twice as many CUs (64x32x8, 64 blocks,
// FP32 12.7 and 11.7; FP64 128 blocks 13.7 and 12.4); at 256 the two are equal within 2 %.
constexpr int FULL_CHIP = 256;  // compute units
struct StepWalk {
    int zb, zt;
};
inline StepWalk step_walk(const Consts& K, int px, int zb, int elem, bool flat, int64_t blocks) {
    StepWalk w;
    w.zb = zb < 1 ? 1 : (zb < K.nz ? zb : K.nz);
    w.zt = w.zb == 1 && blocks >= FULL_CHIP ? 1 : most_planes(elem, px, flat);
    if (w.zt == 2 && w.zb > 1) w.zb += w.zb & 1;
    return w;
}
// Launch geometry of the fused step for a tile width px, w.zb planes per block
// and zg blocks per column and chunk of zg * zb planes: tiles along x,
// columns, blocks.
void step_geometry(const Consts& K, int px, const StepWalk& w, int zg, int yw, int elem, int& tiles_x, int& ncol,
                   int& nblk);
inline bool quad_storage(int32_t storage) { return storage != RMHDLB_STORE_F64; }
inline int storage_bytes(int32_t storage) {
    return storage == RMHDLB_STORE_F64 ? 8 : (storage == RMHDLB_STORE_F32 ? 4 : 2);
}
// One batched step (face pass of the instances that need it, then the fused
// step of all) reading buffer `parity` of every instance; px the tile width
// (128, 64, 32, 16), waves the occupancy variant (FP32: 2 or 3); flat: every
// instance satisfies flat_grid.
template <typename TS>
hipError_t launch_batch(const BatchInst* dev, int ninst, int total_blocks, int64_t total_face, bool flat, int px,
                        int waves, int parity, hipStream_t s);
// nsteps batched steps in one cooperative launch of the persistent batch
// kernel (grid barriers between the steps), starting from buffer `parity`;
// next: 16 ints of device memory for its tile counters (cleared here).  No
// face pass: the caller steps batches that need one by graph replays.
template <typename TS>
hipError_t launch_batch_persistent(const BatchInst* dev, int ninst, int total_blocks, bool flat, int px, int waves,
                                   int parity, int nsteps, int* next, hipStream_t s);
template <typename TS>
hipError_t launch_guess_samples(const char* src, const Consts& K, double* faceB, int ns, double* F, double* T,
                                double* part, double* result, hipStream_t s);
hipError_t launch_guess_normalise(const double* F, const double* T, int ns, const Norm4& nm, float* X, float* Y,
                                  hipStream_t s);
hipError_t launch_train(const TrainArgs& A, hipStream_t s);
// Initial state from the fields in, with the references of the reconnection
// rate: E^z_0 into ez0 and max |B| into b0 (part: one value per tile).
template <typename TS>
hipError_t launch_init(const InPtrs& in, const Consts& K, double* scr, char* dst, double* ez0, double* part,
                       double* b0, hipStream_t s);
// Plain copy of n16 16-byte words (the HBM reference rate).
hipError_t launch_copy16(const void* src, void* dst, int64_t n16, hipStream_t s);
template <typename TS>
hipError_t launch_export(const char* src, double* dst, const Consts& K, hipStream_t s);
template <typename TS>
hipError_t launch_import(const double* src, char* dst, const Consts& K, hipStream_t s);

}  // namespace rmhd
