// Internal declarations shared by the host runtime and the gfx950 kernels of
// libags.  Not part of the public C-ABI (include/ags.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ags.h"

namespace ags {

// One tile block = 256 threads = four wave64s; each thread owns groups of
// 8 consecutive elements (one 16-byte bf16 load or two 16-byte fp32 loads
// per replica).  A tile is at most kTileElems elements of ONE layer, so a
// tile's partial sums belong to exactly one layer.  The default tile is one
// group per thread: on MI355X (ResNet-50 layout, K = 16 bf16) 2048-element
// tiles ran the step kernel in 186 us against 195 us for 4096 and 202 us
// for 8192 (the many short blocks balance the 256 CUs best).
constexpr int kBlock = 256;
constexpr int kVec = 8;
// Threads of a block of the kernels that walk tiles (step, correction and
// LARS update); a round of such a block covers kTileBlock * kVec elements.
#ifndef AGS_TILE_BLOCK
#define AGS_TILE_BLOCK 256
#endif
constexpr int kTileBlock = AGS_TILE_BLOCK;
static_assert(kTileBlock % 64 == 0 && kTileBlock >= 64 && kTileBlock <= 1024, "whole waves");
#ifndef AGS_TILE_ELEMS
#define AGS_TILE_ELEMS (AGS_TILE_BLOCK * 8)
#endif
constexpr int kTileElems = AGS_TILE_ELEMS;  // a multiple of kTileBlock * kVec
static_assert(kTileElems % (kTileBlock * kVec) == 0, "tile must hold whole block rounds");
// A layer is cut into at most this many tiles (bigger layers get tiles of a
// multiple of kTileElems).
#ifndef AGS_MAX_TILES_PER_LAYER
#define AGS_MAX_TILES_PER_LAYER (1 << 30)
#endif
constexpr int64_t kMaxTilesPerLayer = AGS_MAX_TILES_PER_LAYER;
// The finalize kernel sums at most this many tile partials per block (16 per
// thread); a layer with more tiles is finalized by several blocks whose sums
// the last of them combines.
constexpr int kFinTilesPerChunk = 4096;
// Consecutive tiles that one XCD takes at a time (tile_of_block in
// ags_kernels.hip, which holds the measurements).
constexpr int kXcdGroup = 8;

// Once w and m (8 bytes per element) pass this size they cannot stay in the
// 256 MB Infinity Cache between steps, and every step streams them from HBM
// with the replicas.
#ifndef AGS_OCCUPANCY_CAP_MIN_BYTES
#define AGS_OCCUPANCY_CAP_MIN_BYTES (256ll << 20)
#endif
constexpr int64_t kOccupancyCapMinBytes = AGS_OCCUPANCY_CAP_MIN_BYTES;

// Does a LARS step keep the replica mean between its passes?  When re-reading
// the replicas there would cost more than writing and reading one fp32 per
// element.
constexpr bool keeps_mean(int row_bytes) { return row_bytes > 8; }

// How the streaming kernels of a handle (or of a statistics call without
// one) are launched: the most blocks that share a CU, 0 = as many as the
// registers allow.
struct LaunchShape {
    int step_blocks;    // step kernel with the update
    int stats_blocks;   // step kernel, statistics only
    int update_blocks;  // LARS update
    // Non-temporal (streaming) accesses: to w and m in the step kernel and in
    // the LARS update, and the stores of the replica mean between them.
    bool stream_step, stream_update, stream_gbar;
    bool grouped_step;  // tile order of the step kernel with the update
};

// The rule behind a LaunchShape, by the bytes of w and m together ("size"
// below), the replica bytes per element ("row"), type and kernel.  All
// figures are whole calls on MI355X in us: three handles in turn; one handle
// back to back; one step after a 1 GiB read that evicts the caches.  Layouts
// without a name are layers of 2048 to 2.4 million elements.
//
// Streaming accesses to w and m.  Ordinary ones leave the new w and m as
// dirty lines in the Infinity Cache.  If the next step finds them there (one
// handle back to back, w and m fit) that saves HBM traffic; if other work
// evicts them first (a training step's forward and backward passes, or
// another handle), their write-backs are scattered among the reads of what
// runs next, and the reads stall on the DRAM's turn-arounds: 204 MB of
// writes that take 33 us by themselves cost 95 us within a K = 16 step and
// 170 us within a K = 64 one.  Streaming accesses write straight through but
// find nothing on the next step.  They are taken where their gain in turn
// outweighs (in percent) what they lose back to back and after an eviction
// (which leaves the ordinary accesses' write-backs out of the time); what is
// lost back to back there is a chosen loss.  Ordinary -> streaming:
//   row >= 64 (K = 16 fp32, 32 bf16): from 8 MiB on.  8 MiB fp32 23 -> 23;
//     21 -> 22; 26 -> 26, 24 MiB fp32 52 -> 49; 50 -> 48; 55 -> 52, bf16 52
//     -> 52; 51 -> 50; 56 -> 55, 85 MiB bf16 177 -> 167; 167 -> 165; 182 ->
//     179; ResNet-50 (195 MiB) bf16 K = 32 384 -> 357; 341 -> 360; 360 ->
//     362, K = 64 679 -> 651; 633 -> 655; 646 -> 659, fp32 K = 16 392 ->
//     352; 340 -> 355; 361 -> 361;
//   row 32 to 63, fp32: from 128 MiB on.  K = 8 85 MiB 95 -> 97; 89 -> 95;
//     98 -> 102, 112 MiB 133 -> 122; 113 -> 121; 125 -> 127, 144 MiB 171 ->
//     155; 141 -> 154; 157 -> 162, ResNet-50 235 -> 207; 190 -> 209; 213 ->
//     214, VGG-16's size (1056 MiB) 1145 -> 1060; 1086 -> 1057; 1112 -> 1063;
//   row 40 to 63, bf16, and 20 to 31, fp32: once w and m outgrow the cache.
//     K = 20 bf16 280 MiB 385 -> 360; 337 -> 362; 365 -> 366, 480 MiB 667 ->
//     646; 620 -> 640; 650 -> 648, K = 24 280 MiB 446 -> 417; 396 -> 416; 425
//     -> 421, K = 6 fp32 280 MiB 259 -> 239; 226 -> 239; 245 -> 243, 480 MiB
//     431 -> 411; 396 -> 406; 416 -> 409; ResNet-50 K = 24 bf16 310 -> 285; 267
//     -> 288; 287 -> 293;
//   row 32 to 39, bf16, and 16 to 19, fp32: from 512 MiB on.  K = 16 bf16
//     ResNet-50 230 -> 215; 188 -> 214; 213 -> 219, 280 MiB 325 -> 313; 283
//     -> 313; 313 -> 317, 450 MiB 517 -> 500; 475 -> 499; 508 -> 503, 600
//     MiB 686 -> 670; 649 -> 671; 679 -> 677, 1056 MiB 1179 -> 1162; 1144
//     -> 1169; 1171 -> 1170; K = 4 fp32 195 MiB 153 -> 140; 123 -> 140; 135
//     -> 146, 280 MiB 206 -> 195; 182 -> 196; 194 -> 200, 450 MiB 322 ->
//     312; 302 -> 308; 311 -> 318, 600 MiB 425 -> 407; 402 -> 405; 408 -> 418;
//   row < 16: fp32 once w and m outgrow the cache (K = 1 230 MiB 116 -> 105;
//     97 -> 104; 101 -> 110, 280 MiB at the two blocks per CU that were best
//     before 139 -> 125; 131 -> 125; 130 -> 129, 1056 MiB 478 -> 460; 466 ->
//     464; 460 -> 447), bf16 never (K = 4 1056 MiB 573 -> 632; 531 -> 628;
//     532 -> 630, nor with row 16 to 31: K = 8 768 -> 776; 739 -> 777; 733
//     -> 776);
//   element scales (w and m loads only, the stores always stream): bf16
//     never (K = 16 195 MiB 280 -> 269; 239 -> 270; 262 -> 277, 1056 MiB 1349
//     -> 1405; 1328 -> 1395; 1343 -> 1396); fp32 row >= 64 from 128 MiB on
//     (K = 16 85 MiB 171 -> 181; 169 -> 179; 179 -> 184, 144 MiB 322 -> 289;
//     278 -> 288; 296 -> 295, 195 MiB 433 -> 388; 370 -> 383; 392 -> 387),
//     40 to 63 once w and m outgrow the cache (K = 10 195 MiB 303 -> 280; 257
//     -> 280; 287 -> 285, 280 MiB 425 -> 397; 364 -> 395; 397 -> 395, 450 MiB
//     667 -> 631; 601 -> 635; 638 -> 628), 24 to 39 from 512 MiB on (K = 8 195
//     MiB 262 -> 249; 223 -> 246; 246 -> 252, 450 MiB 577 -> 554; 519 -> 560;
//     549 -> 555, 600 MiB 768 -> 746; 714 -> 740; 730 -> 731, 1056 MiB 1325 ->
//     1289; 1265 -> 1295; 1288 -> 1264, K = 7 280 MiB 351 -> 323; 290 -> 322;
//     314 -> 327, 600 MiB 706 -> 675; 658 -> 672; 680 -> 678), less never (K =
//     4 280 MiB 265 -> 257; 225 -> 257; 233 -> 265, 1056 MiB 940 -> 944; 911 ->
//     940; 918 -> 967).
// LARS's update has just one row (the mean) beside w and m: from 64 MiB on.
// K = 8 fp32 56 MiB 79 -> 78; 76 -> 78; 83 -> 82, 72 MiB 98 -> 93; 92 -> 93;
// 98 -> 98; K = 16 bf16 56 MiB 86 -> 86; 82 -> 86; 90 -> 92, 72 MiB 107 ->
// 104; 101 -> 105; 107 -> 108, 195 MiB 270 -> 255; 246 -> 249; 245 -> 254.
// The mean itself streams once it alone outgrows the cache (w and m: 512
// MiB).  K = 8 fp32 480 MiB 596 -> 580; 556 -> 581; 564 -> 581, 560 MiB 705
// -> 673; 687 -> 675; 695 -> 682; K = 16 bf16 480 MiB 641 -> 632; 612 ->
// 622; 618 -> 632, 560 MiB 742 -> 726; 736 -> 718; 743 -> 723.
//
// Blocks per CU.  Fewer resident blocks mean fewer row streams open at once
// (K + 2 per block), so the DRAM rows are used better, until too few reads
// are in flight; small layouts, whose blocks the chip holds at once, only
// lose.
//   Step kernel, ordinary accesses, w and m fit: 4 from 40 MiB on against no
//     cap (bf16 K = 1 32 MiB 24.5 -> 24.9; 23.0 -> 23.1; 28.0 -> 28.0, 48 MiB
//     31.7 -> 30.6; 30.7 -> 30.0; 35.1 -> 33.6, 195 MiB 96 -> 92; 84 -> 82; 86
//     -> 83, fp32 K = 4 32 MiB 30.4 -> 30.9; 30.1 -> 30.4; 34.3 -> 34.6, bf16
//     K = 8 195 MiB 156 -> 152; 128 -> 125; 143 -> 141, K = 16 and fp32 within
//     1%; element scales bf16 K = 1 32 MiB 31.3 -> 31.7; 30.7 -> 30.8; 35.0 ->
//     35.4, 85 MiB 62.5 -> 61.5; 61.3 -> 60.2; 64.2 -> 63.5, 195 MiB 138 ->
//     136; 123 -> 120; 125 -> 124, row >= 16 the same).
//   Ordinary accesses, larger: row < 16 4 (bf16 K = 4 1056 MiB 573 -> 606 at
//     2), else 2 against 4 (fp32 K = 4 280 MiB 216 -> 206; 175 -> 182; 187 ->
//     194, 450 MiB 348 -> 322; 298 -> 302; 306 -> 311, bf16 K = 8 1056 MiB 768
//     -> 755; 739 -> 729; 733 -> 741, K = 16 1254 -> 1179; 1152 -> 1144; 1179
//     -> 1171).  Element scales: row < 16 3 against 4 (fp32 K = 1 600 MiB 405
//     -> 380; 353 -> 343; 363 -> 351, bf16 K = 4 473 -> 456; 432 -> 424; 439
//     -> 428); else 2 against 3 for bf16 (K = 16 280 MiB 389 -> 378; 339 ->
//     350; 364 -> 366, 1056 MiB 1431 -> 1349; 1372 -> 1328; 1384 -> 1343), for
//     fp32 from 512 MiB on (K = 4 450 MiB 420 -> 413; 370 -> 392; 380 -> 398,
//     600 MiB 563 -> 541; 509 -> 519; 520 -> 529, 1056 MiB 1011 -> 940; 935 ->
//     911; 945 -> 918; K = 8 the same either way).
//   Streaming accesses: row < 16 3 against 2 (fp32 K = 1 280 MiB 125 / 130;
//     125 / 131; 129 / 138), else 2 against 3 (fp32 K = 8 280 MiB 302 -> 287;
//     303 -> 286; 303 -> 291, K = 16 element scales 195 MiB 403 -> 388; 400 ->
//     383; 406 -> 387, bf16 K = 16 and 32 the same) or none (K = 16 fp32 24
//     MiB 51 -> 49; 50 -> 48; 55 -> 52, 85 MiB 163 -> 154; 161 -> 153; 167 ->
//     156).
//   Statistics (alone, handles in turn; no cap / 4 / 3): row < 16 none (bf16
//     K = 1 195 MiB 31 / 40 / 47); else from 64 MiB on 3 for fp32 (K = 8 16
//     MiB 19.7 / 19.7 / 20.8, 64 MiB 53.0 / 52.1 / 52.6, 85 MiB 67.4 / 66.6 /
//     66.4, 1056 MiB 718 / 700 / 689; LARS's whole step 64 MiB 84.9 -> 86.0 at
//     3, 85 MiB 108.2 -> 108.2, 195 MiB 238 -> 234) and 4 for bf16 (K = 8 64 MiB 34.1 / 34.9 / 36.8, 450 MiB
//     184 / 180 / 187; K >= 16 the same).
//   LARS update (whole step): 4 from 64 MiB on, from 40 on where it reads the
//     replicas again (row <= 8: K = 1 bf16 32 MiB 27.2 -> 27.2; 26.1 -> 26.1;
//     31.1 -> 31.0, 48 MiB 35.3 -> 34.2; 34.4 -> 34.0; 40.3 -> 37.6; K = 4 fp32
//     48 MiB 48.0 -> 48.0; 47.1 -> 48.4; 53.4 -> 53.5; K = 16 bf16 195 MiB 256
//     -> 252; 250 -> 247; 256 -> 252); larger 3 (K = 8 fp32 400 MiB 483 -> 482;
//     480 -> 479; 486 -> 482, 1056 MiB 1297 -> 1275; 1312 -> 1289; 1321 -> 1280).
//
// The grouped tile order (tile_of_block) serves every kernel but the step
// kernel with element scales of bf16 replicas, whose four fp32 streams
// outweigh the rows: grouped against dispatch order (kernel alone, in turn)
// VGG-16 K = 16 1349 -> 1293, K = 8 973 -> 941, K = 1 638 -> 617, ResNet-50
// K = 16 255 -> 253.
inline LaunchShape launch_shape(const ags_config& c) {
    const int row = c.K * (c.grad_dtype == AGS_BF16 ? 2 : 4);  // replica bytes per element
    const int64_t size = 8 * c.n_flat;                         // bytes of w and m
    const bool large = size > kOccupancyCapMinBytes, larger = size > 2 * kOccupancyCapMinBytes;
    const bool f32 = c.grad_dtype == AGS_F32, ew = c.elementwise != 0;
    constexpr int64_t MiB = 1 << 20;
    LaunchShape s;
    s.grouped_step = f32 || !ew;
    if (ew) s.stream_step = f32 && (row >= 64 ? size > 128 * MiB : row >= 40 ? large : row >= 24 && larger);
    else if (row >= 64) s.stream_step = size > 8 * MiB;
    else if (row >= 32 && f32) s.stream_step = size > 128 * MiB;
    else if (row >= (f32 ? 20 : 40)) s.stream_step = large;
    else if (row >= (f32 ? 16 : 32)) s.stream_step = larger;
    else s.stream_step = f32 && large;
    s.stream_update = size > 64 * MiB;
    s.stream_gbar = larger;
    if (s.stream_step) s.step_blocks = row >= 16 ? 2 : 3;
    else if (!large) s.step_blocks = size > 40 * MiB ? 4 : 0;
    else if (ew) s.step_blocks = row >= 16 && (!f32 || larger) ? 2 : 3;
    else s.step_blocks = row >= 16 ? 2 : 4;
    s.stats_blocks = row < 16 || size <= 64 * MiB ? 0 : (f32 ? 3 : 4);
    s.update_blocks = large ? 3 : size > (keeps_mean(row) ? 64 : 40) * MiB ? 4 : 0;
    return s;
}

// The replica counts with kernels of their own; 0 for any other (then K >= 3).
constexpr int compiled_replicas(int K) {
    return K == 1 || K == 2 || K == 4 || K == 8 || K == 16 || K == 32 || K == 64 ? K : 0;
}
// What launch_shape and keeps_mean can ask of the kernels of a compiled
// replica count (or of any other, kt = 0); only those are built.
constexpr bool can_stream_step(bool f32, int kt, bool ew) {
    if (ew) return f32 && (kt == 0 || kt >= 8);
    return f32 || kt == 0 || kt >= 16;
}
constexpr bool can_keep_mean(bool f32, int kt) { return kt == 0 || keeps_mean(kt * (f32 ? 4 : 2)); }
constexpr bool can_drop_mean(bool f32, int kt) { return !keeps_mean((kt ? kt : 3) * (f32 ? 4 : 2)); }

// Elements per tile of a layer of numel elements.
__host__ __device__ inline int64_t tile_elems_for(int64_t numel) {
    const int64_t per = (int64_t)kTileElems * kMaxTilesPerLayer;
    const int64_t mult = (numel + per - 1) / per;
    return (int64_t)kTileElems * (mult > 0 ? mult : 1);
}
#ifndef AGS_CORRECT_BLOCKS
#define AGS_CORRECT_BLOCKS 512
#endif
// Grid of the correction pass: small, because on most steps the pass only
// reads its list's length and exits.
constexpr int kCorrectBlocks = AGS_CORRECT_BLOCKS;

struct Tile {
    int64_t begin;  // first element (flat index), a multiple of kVec
    int32_t count;  // elements in the tile, 1..kTileElems
    int32_t layer;
};

struct LayerDev {
    int32_t tile_begin, tile_end;    // tiles [tile_begin, tile_end) cover the layer
    uint32_t flags;
    int32_t chunk_begin, chunk_end;  // finalize chunks of the layer
    int32_t pad_;
    int64_t numel;
};

// A finalize block's share: tiles [tile_begin, tile_end) of one layer.
struct FinChunk {
    int32_t layer, tile_begin, tile_end, pad_;
};

struct ChunkSum {
    double w, g, d, s, x;  // x: sum of the refreshed element scales
};

// Device-resident AGS state, updated by the last finalize block of a committed step.
struct DevState {
    double g_prev;      // ||G||^2 of the last committed step (0 before the first)
    int64_t step;       // steps completed
    int32_t last_sens;  // the sensitive bit of the last committed step
    int32_t ew_cur;     // element scales: which of the two buffers is in force
    float lr;           // learning rate in force (ags_set_lr writes it on the handle's
                        // stream, so a step replayed from a graph uses the current one)
    int32_t pad_;
};

// Per-tile fp32 partial sums: W (sum w^2), G (sum gbar^2), D (sum over
// elements of sum_k (g_k - gbar)^2, not yet divided by K), S (small-batch
// sum of squares).
struct Partial {
    float w, g, d, s;
};

// Arguments of the step kernel (statistics of every tile and -- when update
// is on -- the momentum-SGD update with the predicted coefficients) and of
// the finalize kernel (per-layer and global statistics, the decision).
struct StepArgs {
    const void* grads;
    int64_t stride;
    float* w;
    float* m;
    float* gbar;             // store the replica mean here (or nullptr)
    const Tile* tiles;
    Partial* partials;
    const LayerDev* layers;
    int n_layers;
    int K;
    float invK;
    int small_replica;       // -1, or 0..K-1
    int mode;                // ags_mode
    int commit;              // 1: a step (state advances), 0: statistics only
    int refresh_every;
    float momentum;          // used when the kernel updates w and m (lr: state->lr)
    double delta, eps, s_max, trust_coef, weight_decay, static_scale;
    double* gradscale;       // [n_layers]; with element scales, their layer means
    DevState* state;
    double* g_prev_l;        // [n_layers] G_l of the last committed step
    int32_t* last_sens_l;    // [n_layers] the bit that decided each layer then
    int delta_scope;         // ags_delta_scope
    float2* coef;            // [n_layers] LARS: (a_l, b_l), fp32
    float2* corr;            // [n_layers] correction c = x + y * scale_j (fp32) of listed layers
    int* corr_list;          // [n_layers] the layers that need the correction pass
    int* corr_count;         // how many
    int updated;             // the step kernel applied predicted coefficients
    // Step kernel: tiles in reverse order.  Once w and m outgrow the
    // Infinity Cache the host alternates the direction from step to step, so
    // that a step starts on the lines the step before touched last instead of
    // sweeping a working set larger than the cache in one direction.  One
    // direction / alternating, whole step, ordinary accesses to w and m, back
    // to back: VGG-16 K = 8 bf16 754 / 725 us, with element scales 957 / 941,
    // 300 MiB of w and m K = 8 bf16 224 / 208 (in turn the same); streaming
    // ones leave less to find: VGG-16 K = 8 fp32 1090 / 1091 back to back,
    // 1069 / 1061 in turn, with element scales 1302 / 1292 both ways.  Layouts
    // that fit the cache gain nothing.
    int reverse;
    unsigned* done_count;    // layers finished (reset by the last block)
    const FinChunk* chunks;  // finalize blocks
    ChunkSum* chunk_sums;    // [n_chunks] sums of multi-chunk layers
    unsigned* layer_chunk_count;  // [n_layers] chunks finished (reset by the last)
    ags_layer_stats* lstats;
    ags_global_stats* gstats;
    // Element scales (elementwise AGS; all null / 0 otherwise).  The buffer
    // in force and whether a step refreshes are read from the device state
    // (state->ew_cur, state->step), so a captured step replays correctly.
    int ew;                  // 0: a scale per layer, 1: per element
    float* ew_buf;           // [2][n_flat] the two scale buffers
    int64_t n_flat;
    float* ew_partials;      // [n_tiles] per-tile sums of the refreshed scales
    // LARS: per-tile sums of w^2 written by the last update pass; when set,
    // the statistics-only step kernel takes W from them and skips w.
    const float* w_norm_in;
    // Bytes of dynamic LDS the step kernel is launched with (it uses none):
    // a pad that caps the blocks resident per CU (launch_shape).
    int lds_pad;
    int stream_wm;    // streaming accesses to w and m (launch_shape)
    int stream_gbar;  // streaming stores of the replica mean
    int grouped;      // grouped tile order (tile_of_block)
};

struct UpdateArgs {
    const Tile* tiles;
    int n_tiles;
    const float* gbar;    // materialised replica mean, or nullptr to recompute
    const void* grads;
    int64_t stride;
    int K;
    float invK;
    float* w;
    float* m;
    const float2* coef;   // LARS update: (a_l, b_l)
    const LayerDev* layers;  // correction pass: the listed layers' tiles
    const float2* corr;   // correction pass: c = x + y * gs_old_j of a listed layer
    const int* corr_list;
    const int* corr_count;
    const float* ew_buf;  // [2][n_flat] element scales (or null)
    int64_t n_flat;
    const DevState* state;  // after the step: the buffer in force and the step count
    int refresh_every;
    float momentum;          // lr: state->lr
    // LARS update: per-tile sums of the new w^2, summed as the statistics
    // pass sums w^2 (or nullptr).
    float* w_norm_out;
    // Dynamic LDS of the LARS update launch (0: none), a cap on its blocks
    // per CU, and its streaming accesses to w and m (launch_shape).
    int lds_pad;
    int stream_wm;
    // LARS update: the tiles in reverse order (the last tiles first).  The
    // pass then ends on the first tiles, whose replica mean the next
    // statistics pass writes first, and those lines are still in the Infinity
    // Cache: that pass measured 154.4 -> 151.0 us (ResNet-50
    // K = 16 bf16; K = 64 582 -> 574 us) with the update pass unchanged.
    // Used while w and m fit the cache (VGG-16's step lost 0.8% with it).
    int reverse;
};

// Text for ags_last_error(NULL) on this thread (ags_api.hip).
void set_thread_error(const char* why);

// Events a launch records at its kernel's start and end (both null: none).
// They belong to the kernel's own dispatch, so their elapsed time is the
// kernel's execution alone, without the marker packets and cache
// write-backs of a separate hipEventRecord between kernels.
struct KernelEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};

// Launchers (ags_kernels.hip).  They only enqueue; the return value is the
// launch status.  update != 0 makes the step kernel apply the update.
hipError_t launch_step(const StepArgs& a, ags_dtype dt, int n_tiles, bool update, hipStream_t s,
                       KernelEvents ev);
hipError_t launch_finalize(const StepArgs& a, int n_chunks, hipStream_t s, KernelEvents ev);
hipError_t launch_update(const UpdateArgs& a, ags_dtype dt, hipStream_t s, KernelEvents ev);
hipError_t launch_correct(const UpdateArgs& a, ags_dtype dt, hipStream_t s, KernelEvents ev);
// Writes the learning rate in force into the device state (one thread).
hipError_t launch_set_lr(DevState* state, float lr, hipStream_t s);

}  // namespace ags
