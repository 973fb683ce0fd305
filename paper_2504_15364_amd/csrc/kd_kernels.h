// Internal launcher interface between the C-ABI host layer and the gfx950 kernels.
//
// One block step is two launches:
//   step_main  append (Eq. 5) + split-KV flash attention partials (Eq. 1-2)
//              + running key sum S' = S + sum of the block's keys (the anchor is S' / n)
//              + cosine score of every row, taken from the K tiles while they sit in LDS
//              (step_few instead where a KV head has few query rows and many keys)
//   step_post  merge of the attention partials  ||  selection of the rows to evict
//              and compaction, one workgroup per head (Eq. 6-7)
// For the ORDERED layout the rows are shifted in place by the selection's workgroup itself (short caches), by the workgroups around it in
// the same launch (step_post_shift) or, where the chip does not hold all rows in registers, by one more launch.
// With the eviction deferred the second launch is the merge alone, and the selection and
// compaction ride in the step_main launch of the next cache (launch_step_main_carry).
// step_score scores a cache outside a block step (keydiff_scores).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kd {

constexpr int TILE_KEYS = 64;       // keys per attention K/V tile
constexpr int MAIN_WAVES = 8;       // waves (of 32 query rows) per step_main workgroup
constexpr int FEW_KEYS = 32;        // keys per wave and tile in step_few
constexpr int FEW_ROWS = 32;        // query rows per KV head up to which a step may run step_few instead of step_main (the plan decides)
constexpr int POST_THREADS = 1024;  // workgroup size of step_post
constexpr int SCORE_THREADS = 256;  // workgroup size of step_score
constexpr int SCORE_ROWS = 128;     // rows per step_score workgroup: 32 per wave
constexpr int HIST_BINS = 4096;     // score histogram resolution in step_post (bins over [-1, 1])
// Bound of |approximate score - exact score| (step_main with score_approx).  With |k| and |mu| the norms and the sums of
// the matrix pipe off by at most 2^-23 of the running magnitude per term: 128 terms of mu.k 1.6e-5 |mu||k| (the second
// bf16 vector of the anchor adds a 256th of that), the anchor as two bf16 vectors 2^-18, |k| 128 / 2 terms 7.7e-6, square
// roots, reciprocal and products 1e-6: 2.9e-5 in all, as |score| <= 1.
constexpr float SCORE_SLACK = 3e-5f;
constexpr int CHUNK_ROWS = 128;     // rows per workgroup in the from-scratch key-sum pass
constexpr int LAYOUT_SHIFT_HERE = 2;  // StepParams::layout: ORDERED, and the selection shifts the rows too (short caches, shift_fits_selection)
constexpr int ORD_ROWS = 128;       // rows per workgroup of the ordered compaction
constexpr int ORD_THREADS = 1024;   // ... and its threads: 4 16-byte units each
constexpr int ORD_MIN_ROWS = 32;    // fewest rows a workgroup of a shift takes: one flag each in the metadata
constexpr int TICKET_STRIDE = 32;   // words from one head's ticket counter to the next: a cache line
constexpr int AROUND_UNITS = 20;    // most 16-byte units a thread of a shift around the selection holds in registers
constexpr int ORD_SPIN_LIMIT = 1 << 20;  // polls of a predecessor's flag before giving up
constexpr int MAX_CAP = 32768;      // budget_N + block_B limit (selection bitmaps, ownership)

// status bits kernels may raise (device word in the metadata buffer)
constexpr int STATUS_SELECT_COUNT = 1;  // selection evicted a number of rows other than n - N
constexpr int STATUS_ORDER_TIMEOUT = 2; // ordered compaction: a workgroup gave up waiting for its predecessors

// (256 bytes: four lines of argument memory, which is cold in every launch)
struct StepParams {
    // tensors of the call
    const uint16_t *q;               // [batch][hq][Bt][D]
    const uint16_t *k_new, *v_new;   // [batch][hkv][Bt][D]
    uint16_t *out;                   // [batch][hq][Bt][D]
    float *scores_out;               // nullable [BH][n]
    // caller-owned state
    uint16_t *k, *v;                 // caches [BH][cap][D]
    int32_t *pos;                    // [BH][cap] token position of every row
    const double *ksum;              // [BH][D] running sum of the (raw or unit) keys in the cache before this step
    double *ksum_next;               // [BH][D] ... after it (the other half of a double buffer): written by
                                     // step_main (+ the block's keys), then by step_post (- the evicted keys)
    int32_t *status;
    // scratch
    _Float16 *part_o;                // [splits][BH][blocks of 32 rows][D/8 slabs][64 lanes][4] partial outputs in the
                                     // MFMA accumulator layout, each normalised by its row sum
    float2 *part_ml;                 // [splits][BH * G * Bt]     (reference max in log2 units, row sum)
    float *scores;                   // [BH][cap]; approximate if score_approx
    double *anchor;                  // [BH][D] the step's anchor (score_approx)
    int32_t *dstmap;                 // [BH][cap] ORDERED layout: destination row or -1
    int32_t *lists;                  // [BH][4 * B]: the E evicted rows in ascending order (the rest is not used)
    unsigned long long *argmax_rec;  // nullable [BH][splits][2]: the generation phase (one row to evict, no window):
                                     // per step_few workgroup the largest (orderable score bits << 32 | row) among the
                                     // rows it scored, and whether another of its rows has the same score bits
    // sizes
    int batch, hkv, G, D, Bt, len, n, N, B, cap;
    int splits, mtiles, ntiles;      // splits: ranges of keys per head, one partial per output row each (1: the attention writes `out`)
    int few;                         // the step runs step_few (at most FEW_ROWS query rows per KV head, see the plan): its partials are
                                     // float [splits][BH][G * Bt][D] in part_o
    int edge_cost;                   // weight (in plain tiles: 1 or 2) of a tile holding rows of the block when
                                     // the key tiles are divided over the splits
    int lists_in_lds;                // selection lists live in LDS (else in `lists`)
    int merge_wgs;                   // merge workgroups in step_post (0 when splits == 1)
    int do_score, do_evict;
    int score_approx;                // the step's scores are within SCORE_SLACK of the exact ones (or NaN: not known)
    int anchor_mode, layout, window_W;
    int32_t pos0, window_pos_min;
    float scale_log2e;
    double eps;
#ifdef KD_TIMELINE
    unsigned long long *timeline;    // [workgroup][32] wall-clock stamps of this launch (profiling build only)
#endif
};
#ifndef KD_TIMELINE
static_assert(sizeof(StepParams) == 256, "a field that crosses into a fifth line costs every launch that reads it a trip to memory");
#endif

// The same block step of several layers at once (keydiff_prefill_block_layers): one launch whose grid's second dimension is
// the layer.  All have the same sizes; pointers, and what follows from them, are each layer's own.
constexpr int GROUP_LAYERS = 16;     // (4 KB of arguments)
struct LayerSteps {
    StepParams p[GROUP_LAYERS];
};
// The row shift of one ORDERED cache by the destination map its selection wrote (flags: [BH][chunks of ORD_ROWS rows] int32 in
// zero-initialised device memory; epoch: a value no earlier shift of this cache used)
struct ShiftStep {
    uint16_t *k, *v;
    const int32_t *dstmap;
    int32_t *status, *flags;
    int BH, n, N, cap;
    int32_t epoch;
    uint32_t *tickets;   // as in ShiftAround
    uint32_t first_ticket;
};
struct ShiftSteps {
    ShiftStep s[GROUP_LAYERS];
};

// The same shift by the workgroups around the selection that decides it, in one launch with it (step_post_shift): the rows wait in
// registers while the selection runs, which hands over its eviction bitmap word by word, each with the epoch beside it.
struct ShiftAround {
    unsigned long long *words;   // [BH][stride] zero-initialised: a word that says whether there is something to move, then the bitmap
    int32_t *flags;              // [BH][chunks]: the chunk's rows are in registers
    uint32_t *tickets;           // [BH][TICKET_STRIDE] zero-initialised: workgroups of the head that have started, over all launches
    uint32_t first_ticket;       // ... before this launch
    int32_t epoch, stride;
    int32_t units, chunks;       // 16-byte units a thread holds; workgroups a head
};
struct ShiftArounds {
    ShiftAround s[GROUP_LAYERS];
};

// Pieces (of four output values) a thread of the merge takes: with few splits several
constexpr int MERGE_FEW_SPLITS = 4, MERGE_PIECES = 4;
__host__ __device__ constexpr int merge_pieces(int splits) { return splits <= MERGE_FEW_SPLITS ? MERGE_PIECES : 1; }

hipError_t configure_kernels();      // one-time function attributes (dynamic LDS sizes)
hipError_t launch_step_main(const StepParams &p, hipStream_t s);
// ... of `layers` layers in one launch (2 .. GROUP_LAYERS of them, none with step_few)
hipError_t launch_step_main_layers(const LayerSteps &steps, int layers, hipStream_t s);
// the same step where the plan chose step_few (p.few)
hipError_t launch_step_few(const StepParams &p, hipStream_t s);
// How the selection of step `cy` would ride in another launch: not at all, reading its scores and positions from memory in
// every pass, or from copies in LDS.
enum class Ride { none, memory, lds };
Ride ride_of(const StepParams &cy);
// whether some waves of the step's row tiles have no query row (they copy tiles and score)
bool main_runs_help(const StepParams &p);
// step_main of `p` whose first workgroups run the selection and compaction `cy` describes (the
// parameters of an earlier step of another cache; for the ORDERED layout the caller still launches
// the row shift afterwards); can_carry says whether the pair fits
bool can_carry(const StepParams &p, const StepParams &cy);
hipError_t launch_step_main_carry(const StepParams &p, const StepParams &cy, hipStream_t s);
// An ORDERED cache's row shift riding in an attention launch: `p` is the step whose selection wrote the
// destination map, `parts` workgroups per head share the head's chunks (flags, epoch: as for
// launch_compact_ordered).  can_host_shift says whether the attention step `p` can take it along.
struct ShiftRide {
    StepParams p;
    int32_t *flags;
    int nchunks, parts, nshift;
    int32_t epoch;
    uint32_t *tickets;   // as in ShiftAround
    uint32_t first_ticket;
};
bool can_host_shift(const StepParams &p, const StepParams &shifted);
// step_main of `p` with passengers: the selection `cy` (or none: nullptr) and the shift `ride`
hipError_t launch_step_main_ride(const StepParams &p, const StepParams *cy, const ShiftRide &ride, hipStream_t s);
hipError_t launch_step_score(const StepParams &p, hipStream_t s);
hipError_t launch_step_post(const StepParams &p, hipStream_t s);
hipError_t launch_step_post_layers(const LayerSteps &steps, int layers, hipStream_t s);
// Units a thread and chunks a head of a shift around the selection of `layers` caches shaped like p's on `cus` compute units; false: not that way
bool plan_shift_around(const StepParams &p, int layers, int cus, int32_t *units, int32_t *chunks);
hipError_t launch_step_post_shift(const StepParams &p, const ShiftAround &around, hipStream_t s);
hipError_t launch_step_post_shift_layers(const LayerSteps &steps, const ShiftArounds &arounds, int layers, hipStream_t s);
// the ordered shift of one cache (p: its step), and of `layers` caches of the same sizes
hipError_t launch_compact_ordered(const StepParams &p, const ShiftStep &shift, hipStream_t s);
hipError_t launch_compact_layers(const ShiftSteps &steps, int layers, int D, hipStream_t s);
// the merge of pm's partials and the ordered shift of another cache in one launch (same head_dim)
hipError_t launch_merge_shift(const StepParams &pm, const ShiftStep &shift, hipStream_t s);
hipError_t launch_ksum_rebuild(const StepParams &p, double *partials, hipStream_t s);
// rotary embedding of the blocks' queries (q_rows rows each) and keys (k_rows rows), Bt tokens per (sequence,
// head) at positions pos0 + j, by the caller's float tables [position][D / 2]
constexpr int ROPE_LAYERS = 32;      // blocks one launch rotates
struct RopeBatch {
    const uint16_t *q[ROPE_LAYERS], *k[ROPE_LAYERS];
    uint16_t *q_rot[ROPE_LAYERS], *k_rot[ROPE_LAYERS];
    int layers;
};
hipError_t launch_rope(const RopeBatch &b, const float *cos_t, const float *sin_t, int q_rows, int k_rows, int Bt, int D,
                       int32_t pos0, hipStream_t s);
hipError_t launch_zero_words(int32_t *p, size_t nwords, hipStream_t s);
hipError_t launch_load_rows(const uint16_t *src, uint16_t *dst, int BH, int cap, int D, int len,
                            hipStream_t s);
hipError_t launch_load_pos(const int32_t *src, int32_t *dst, int BH, int cap, int len, int to_cache,
                           hipStream_t s);

bool lists_fit_lds(int n, int N);
// whether the selection of an ORDERED step (a launch of its own) had better shift the rows itself
bool shift_fits_selection(const StepParams &p);

}  // namespace kd
