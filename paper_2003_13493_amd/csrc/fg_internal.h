// Internal declarations shared by the kernels and the host runtime of
// libfastgrid.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastgrid.h"

// Device-side description of one detection job (one frame).
struct fg_job {
    uint8_t *lvl[FAST_MAX_LEVELS];   // level planes; [0] is the input
    int32_t w[FAST_MAX_LEVELS];
    int32_t h[FAST_MAX_LEVELS];
    int32_t pitch[FAST_MAX_LEVELS];
    int32_t levels, t, n, cell;
    int32_t score;                   // corner score kind (FAST_SCORE_*)
    uint16_t *smap[FAST_MAX_LEVELS]; // score maps (score-map and standalone-NMS entry points)
    int32_t smap_pitch[FAST_MAX_LEVELS];   // their pitches in elements
    fast_feature *out;               // gw*gh slots
    int32_t gw, gh;                  // grid size in cells
    int32_t rcells;                  // cells per region side
    int32_t rx, ry;                  // regions across, down
};

// Launch shape knobs (set per context by fast_set_launch / the autotuner).
struct fg_launch {
    int region;          // target region side in level-0 pixels, batches
    int plain_region;    // the same for one-frame calls; 0 = chosen per frame
    int block;           // threads per workgroup
    int blocks_per_cu;   // persistent kernel occupancy target
    int num_cu;          // compute units on the device
};

// Dynamic LDS bytes of the detect kernels for a workgroup size.
size_t fg_smem_bytes(int block);

// Fill the derived fields of a job (grid, regions) for a launch shape.
void fg_job_layout(fg_job &j, const fg_launch &L);

// Lucas-Kanade tracking of nfeat features, one wave64 each.
struct fg_track_args {
    const uint8_t *tpl[FAST_MAX_LEVELS];
    const uint8_t *img[FAST_MAX_LEVELS];
    int32_t w[FAST_MAX_LEVELS], h[FAST_MAX_LEVELS];
    int32_t tpitch[FAST_MAX_LEVELS], ipitch[FAST_MAX_LEVELS];
    int32_t levels;
    const float *feats;   // nfeat x (x, y)
    float *q;             // nfeat x (tx, ty, alpha, beta), in and out
    int32_t *status;
    int32_t *iters;       // or null
    int32_t nfeat, mode, max_iter;
    float eps;
};
hipError_t fg_launch_track(const fg_track_args &A, hipStream_t s);

// One camera stream's step of the detect-and-track loop (fast_frontend_step):
// tracking arguments (tpl = previous pyramid, img = current; feats, q and
// status hold `capacity` entries; nfeat unused: the live count is *count),
// this frame's cell winners, and the selection rule.
struct fg_fe_job {
    fg_track_args A;
    const fast_feature *slots;   // gw*gh cell winners of the current frame
    int32_t *count;              // live features: in, tracked from the previous frame; out, after the step
    int32_t *info;               // out: tracked, re-detected (0/1), live, 0
    int32_t cell, gw, gh;
    int32_t capacity;            // the target track count
    int32_t redetect_below;      // re-detect when fewer live tracks remain
    int32_t has_prev;            // 0 on a stream's first frame: nothing to track
    int32_t feat_base;           // first wave of this job in the tracking launch
};

// Tracking of every job's live features (one wave per feature slot, total_slots
// = sum of capacities), then the update of every job's feature list.
hipError_t fg_launch_frontend(const fg_fe_job *jobs_dev, int njobs, int total_slots, hipStream_t s);

// Plain path: one frame.  Enqueues the pyramid (levels 1..L-1) and detection.
hipError_t fg_launch_plain(const fg_job &j, const fg_launch &L, hipStream_t s);

// Pyramid only, one frame.
hipError_t fg_launch_pyramid(const fg_job &j, hipStream_t s);

// One frame's score maps (j.smap): builds levels 1.. like fg_launch_plain and
// writes every level's scores instead of selecting features.
hipError_t fg_launch_score_maps(const fg_job &j, const fg_launch &L, hipStream_t s);

// Standalone NMS over (2 radius + 1)^2 neighbourhoods and the cell arg-max
// from j.smap (j.lvl unused) into j.out.
hipError_t fg_launch_nms_grid(const fg_job &j, int radius, hipStream_t s);

// The persistent batched kernels' counter buffer: FG_QUEUES work queues, the
// head of queue c at word FG_QUEUE_STRIDE * c, and the exit count at word
// FG_QUEUES * FG_QUEUE_STRIDE.  The heads sit 256 bytes apart, on separate
// cache lines: one shared head serialises every ticket of a launch (about
// 13 ns each on MI355X, which alone bounded the 64-frame batch near 100 us).
constexpr int FG_QUEUES = 8;
constexpr int FG_QUEUE_STRIDE = 64;
constexpr int FG_EXIT_WORD = FG_QUEUES * FG_QUEUE_STRIDE;
constexpr int FG_COUNTER_WORDS = FG_EXIT_WORD + FG_QUEUE_STRIDE;
// Consecutive work items a queue hands out before the next queue's run: 16
// neighbouring 64x64 regions on one XCD cut the batch's fetched bytes 3x
// against runs of one; runs of 64 cut them further but leave the queues
// (and XCDs) finishing up to 2% apart.
constexpr int FG_QUEUE_RUN = 16;

// Regions of at most this side (level-0 pixels) are one fused sub-tile.
constexpr int FG_SUB = 64;

// One work item of the batched kernels: a region of a job, its row << 16 | its
// column (below 2^12 each), with FG_WHOLE set for a whole region of 64 x 64
// pixels of a job of three levels and more.
struct fg_item {
    uint32_t job;
    uint32_t region;
};
constexpr uint32_t FG_WHOLE = 1u << 15;

// Pyramid levels detected from one level-0 load; each FG_MAX_FUSED levels
// further up take one more pass (levels 3-5, then 6-7).
constexpr int FG_MAX_FUSED = 3;

// Whole regions of a job (FG_WHOLE).
__host__ __device__ constexpr int fg_whole_regions(const fg_job &j) {
    return j.rcells * j.cell == FG_SUB && j.levels >= FG_MAX_FUSED ? (j.w[0] / FG_SUB) * (j.h[0] / FG_SUB) : 0;
}

// Cells per side of an upper region, the part of a frame one workgroup takes
// in the passes over levels 3.. : 128 level-0 pixels (16 of level 3), at most
// 16 cells, and never less than a region of the level-0 pass, so that a frame
// has no more upper regions than regions.  Measured for levels 3.. of one
// frame: 1920x1080, 4 levels, 7.9 us with 128 (135 workgroups) and 9.0 with
// 256 (40 of 256 CUs busy); 4096x2160, 5 levels, 10.3 us with 128 and 9.4 with
// 256; 64 or fewer spend a workgroup's whole chain of loads and passes on 64
// pixels of level 3 (27 us for that frame's 2176 regions).  The pass over levels 6
// and 7 takes the same regions, 2 pixels of level 6 a side: up to 4096x2160 its
// workgroups (544) are all resident at once, so it lasts one chain (6 to 7 us)
// whatever their size.
constexpr int FG_UPPER_SIDE = 128;
__host__ __device__ constexpr int fg_upper_cells(int cell, int rcells) {
    const int c = FG_UPPER_SIDE / cell;
    return c < rcells ? rcells : (c > 16 ? 16 : c);
}
__host__ __device__ constexpr int fg_upper_regions(const fg_job &j) {
    const int c = fg_upper_cells(j.cell, j.rcells);
    return ((j.gw + c - 1) / c) * ((j.gh + c - 1) / c);
}

// The level-0 work of a batch: its regions, those that are whole, and whether
// every job's regions are single 64x64 sub-tiles.
struct fg_batch_work {
    int total, whole;
    bool all_single;
};

// The kernel that takes it.
//   GENERIC       any region and workgroup size;
//   GENERIC_WIDE  the same with at most 128 registers;
//   ANY           regions that are single sub-tiles, workgroups of 256 threads and
//                 more, at most 128 registers;
//   WHOLE         the same with 168 and a path of its own for whole regions.
// WHOLE takes a whole region in 0.88 of ANY's time and another one (of one or two
// levels, or of cells that do not make 64 pixels) in 1.1 of it, so the line lies at
// one whole region in four.  64 frames of three sizes, 16, 24, 32 and 40 of them of
// three levels and the others of one: ANY 94.0, 96.2, 99.4 and 101.7 us, WHOLE 94.4,
// 93.4, 93.9 and 93.7; the others of 48-pixel cells: ANY 132.2, 130.1, 125.8 and
// 122.3, WHOLE 136.2, 130.7, 123.0 and 116.5.
//
// With more than 128 registers, three waves a SIMD, one workgroup past 256 threads
// (two waves on a SIMD) is resident where 128 let two be.  64 frames of three levels with 320 threads and 3 workgroups a CU: WHOLE
// 203 us, ANY 140; 384 and 2, 198 and 136; 512 and 2, 186 and 129; 512 and 1, 171
// and 195.
enum class fg_batch_kernel { GENERIC, GENERIC_WIDE, ANY, WHOLE };
constexpr fg_batch_kernel fg_choose_batch(const fg_batch_work &w, const fg_launch &L) {
    const bool wide = L.block > 256 && L.blocks_per_cu > 1;
    if (!w.all_single || L.block < 256) return wide ? fg_batch_kernel::GENERIC_WIDE : fg_batch_kernel::GENERIC;
    return !wide && 4LL * w.whole >= w.total ? fg_batch_kernel::WHOLE : fg_batch_kernel::ANY;
}

// Copy `bytes` (a multiple of 8) of coherent pinned host memory to device
// memory by a kernel on `s`.
hipError_t fg_launch_upload(void *dev, const void *host, size_t bytes, hipStream_t s);

// Batched path: `jobs_dev` is a device copy of the jobs.  items[0 .. work.total)
// lists every region of every job once, in any order; the next total_upper items
// list every upper region of the jobs with more than FG_MAX_FUSED levels.
// `counter` holds FG_COUNTER_WORDS zero-initialised words that the kernel re-arms
// itself on exit.
hipError_t fg_launch_batch(const fg_job *jobs_dev, const fg_item *items, const fg_batch_work &work, int total_upper,
                           int max_levels, unsigned *counter, const fg_launch &L, hipStream_t s);
