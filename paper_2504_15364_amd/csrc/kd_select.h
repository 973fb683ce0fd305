// Selection of the rows to evict and compaction of one head (Eq. 6-7), as device code shared by
// the kernels that can run it: step_post (one workgroup of 1024 threads per head) and the variant of
// step_main that carries another cache's pending eviction (workgroups of 512 threads).
//
// One workgroup takes the head's scores and positions once -- into registers (step_post) or into LDS
// (asynchronously, the passenger) -- bins the scores into a 4096-bin LDS histogram (a monotone map of the float), scans it for the bin
// that holds the E-th largest score, evicts everything above that bin and ranks the few rows inside
// it exactly by (score bits, position): equal scores keep the lower position.  It then compacts the
// cache and takes the evicted keys out of ksum.
//
// The passenger's passes over the rows are short rolled loops over the LDS copy.  As a passenger the selection
// runs on one compute unit per head, whose instruction cache nothing has warmed, while the
// attention saturates the memory system: with the rows in registers and every pass unrolled
// (25 KB of straight-line code) it spent most of its time waiting for its own instructions.  In step_post,
// where sixteen waves share the fetch and the caller waits for the end, the registers are the shorter way.
//
// What bounds it there is the issue of its instructions: sixteen waves on four SIMDs, 16 cycles for each instruction that all of
// them execute (288 rows took 8.2 us of the 11.2 that 4224 take).  Hence: a row's place in the histogram is worked out once and
// compared as a float afterwards; the eviction bitmap is put together from the rows a wave holds (no atomics but for the
// few candidates) and gives the list of evicted rows in order; block-wide scans fold the totals of the waves across
// lanes; half of the waves take K rows, the other half V rows, so that a wave's addresses differ by constants;
// and a K row's piece is read by the thread that overwrites it, so that the moves wait for no barrier and the sum of the
// evicted keys is formed behind them.  Launches of step_post before and after, us: 8 heads of 128, 128 rows evicted of 4224
// 11.15 -> 9.0, of 8320 in the ORDERED layout 12.6 -> 11.0, 512 of 16896 26.6 -> 20.8; of 64, 32 of 288 ORDERED 8.2 -> 6.5, 64 of 576
// (8 heads) 9.8 -> 7.6.  Not kept: 512 threads (4224 rows 2 us slower, 2112 rows 0.5 us faster), 256 (slower at all sizes).
#pragma once
#include "kd_kernels.h"
#include "kd_device.h"

namespace kd {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

constexpr int CAND_MAX = 1024;  // rows of the threshold bin ranked in LDS; more fall back to a radix select
constexpr int MAX_SELECT_WAVES = POST_THREADS / 64;   // PostShared is laid out for the largest workgroup
constexpr int CARRY_THREADS = 512;                  // workgroup size of the step_main variant that carries a selection
constexpr int KEY_PARTS = 8;                        // partial sums of the evicted keys
constexpr int SELECT_TAILU = 8;                     // 16-byte units of the tail rows [N, n) a thread keeps in registers

// float -> unsigned key with the same order
__device__ __forceinline__ uint32_t orderable(float s)
{
    const uint32_t b = __float_as_uint(s);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Monotone non-decreasing map of a score onto [0, HIST_BINS): the integer part of score_place, which is clamped (a NaN to 0).
__device__ __forceinline__ float score_place(float s)
{
    return __builtin_amdgcn_fmed3f(__builtin_fmaf(s, (float)(HIST_BINS / 2), (float)(HIST_BINS / 2)), 0.f, (float)(HIST_BINS - 1));
}
__device__ __forceinline__ int score_bin(float s) { return (int)score_place(s); }

struct PostShared {
    uint32_t hist[HIST_BINS];  // score histogram of the head (a monotone map of the float)
    uint32_t wave_tot[MAX_SELECT_WAVES], wave_tot2[MAX_SELECT_WAVES];
    uint64_t wave_tot64[MAX_SELECT_WAVES];
    uint32_t radix_hist[256];
    uint32_t sel_bin, sel_rank, sel_cnt;
    int tb;           // threshold bin
    uint32_t ncand, nev;
    uint32_t cand_slot[CAND_MAX];
    uint32_t cand_key[CAND_MAX];
    int32_t cand_pos[CAND_MAX];
    double colsum[MAX_SELECT_WAVES][128];
    double mu[128], mu2[8];   // the anchor and |mu|^2 in pieces (approximate scores: exact ones of the rows near the threshold)
    int bad;                  // a row's score is not known even approximately
};

// bytes of dynamic LDS a carried selection places PostShared in, ahead of its bitmap and lists
__host__ __device__ constexpr size_t carry_shared_bytes() { return (sizeof(PostShared) + 255) & ~(size_t)255; }

// value of the lane `ctrl` names (DPP), 0 where that lane lies outside the row or the row is masked out
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_fetch(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xF, true);
}

// inclusive prefix sum over the 64 lanes of a wave, on the vector ALU alone: Hillis-Steele inside
// each row of 16 lanes (row_shr 1, 2, 4, 8), then lane 15 of rows 0 and 2 into rows 1 and 3
// (row_bcast:15), then lane 31 into rows 2 and 3 (row_bcast:31)
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x)
{
    x += dpp_fetch<0x111, 0xF>(x);
    x += dpp_fetch<0x112, 0xF>(x);
    x += dpp_fetch<0x114, 0xF>(x);
    x += dpp_fetch<0x118, 0xF>(x);
    x += dpp_fetch<0x142, 0xA>(x);
    x += dpp_fetch<0x143, 0xC>(x);
    return x;
}
// exclusive prefix sum over the workgroup; `wave_tot`: LDS words of the waves that no thread still reads
template <int THREADS, typename T>
__device__ __forceinline__ T block_exclusive_scan_t(T v, T *wave_tot, T *total)
{
    constexpr int NWAVES = THREADS / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T inc = wave_inclusive_scan(v);
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    // the totals of the waves, one a lane, scanned the same way (every thread adding them up by itself: 0.4 us a scan of 16 waves)
    static_assert(NWAVES <= 16, "the totals fit one row of lanes");
    const T totals = wave_inclusive_scan(lane < NWAVES ? wave_tot[lane & (NWAVES - 1)] : (T)0);
    *total = (T)__builtin_amdgcn_readlane((int)totals, NWAVES - 1);
    const T base = wave == 0 ? (T)0 : (T)__builtin_amdgcn_readlane((int)totals, __builtin_amdgcn_readfirstlane(wave - 1));
    return base + inc - v;
}

// ---------------------------------------------------- slow path: radix select in a bin
// More than CAND_MAX rows share the threshold bin (near-identical keys).  MSB-first
// 8-bit radix select over the 64-bit key (orderable score : position) restricted to
// that bin; reads scores and positions again on every pass.  Marks the
// `need` largest in the evict bitmap.
template <int THREADS>
__device__ void radix_select_in_bin(const StepParams &p, PostShared &sh, const float *sc, const int32_t *pos,
                                    uint32_t *evbits, int tb, uint32_t need)
{
    const int tid = threadIdx.x, lane = tid & 63;
    uint64_t prefix = 0;
    uint32_t rank = need;
    int resolved = 0;
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
        for (int i = tid; i < 256; i += THREADS) sh.radix_hist[i] = 0;
        __syncthreads();
        for (int i0 = 0; i0 < p.n; i0 += THREADS) {
            const int i = i0 + tid;
            bool part = false;
            uint32_t digit = 0;
            if (i < p.n) {
                const float s = sc[i];
                const bool exempt = p.window_W > 0 && pos[i] >= p.window_pos_min;
                if (!exempt && score_bin(s) == tb) {
                    const uint64_t key = ((uint64_t)orderable(s) << 32) | (uint32_t)pos[i];
                    part = pass == 0 || (key >> (shift + 8)) == prefix;
                    digit = (uint32_t)(key >> shift) & 255u;
                }
            }
            const uint64_t active = __ballot(part);
            if (active) {
                const int leader = __ffsll((unsigned long long)active) - 1;
                const uint32_t ld = __shfl(digit, leader);
                const uint64_t same = __ballot(part && digit == ld);
                if (lane == leader) atomicAdd(&sh.radix_hist[ld], (uint32_t)__popcll(same));
                else if (part && digit != ld) atomicAdd(&sh.radix_hist[digit], 1u);
            }
        }
        __syncthreads();
        if (tid < 64) {
            const uint32_t c0 = sh.radix_hist[4 * lane], c1 = sh.radix_hist[4 * lane + 1],
                           c2 = sh.radix_hist[4 * lane + 2], c3 = sh.radix_hist[4 * lane + 3];
            const uint32_t mine = c0 + c1 + c2 + c3;
            uint32_t suf = mine;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t t = __shfl_down(suf, off);
                if (lane + off < 64) suf += t;
            }
            const uint64_t reach = __ballot(suf >= rank);
            const int owner = reach ? 63 - __clzll((unsigned long long)reach) : 0;
            if (lane == owner) {
                uint32_t above = suf - mine, bin, cnt;
                if (above + c3 >= rank) { bin = 3; cnt = c3; }
                else if ((above += c3) + c2 >= rank) { bin = 2; cnt = c2; }
                else if ((above += c2) + c1 >= rank) { bin = 1; cnt = c1; }
                else { above += c1; bin = 0; cnt = c0; }
                sh.sel_bin = 4 * lane + bin;
                sh.sel_rank = rank - above;
                sh.sel_cnt = cnt;
            }
        }
        __syncthreads();
        prefix = (prefix << 8) | sh.sel_bin;
        rank = sh.sel_rank;
        resolved = 8 * (pass + 1);
        const bool done = sh.sel_cnt == rank;
        __syncthreads();
        if (done) break;
    }
    for (int i = tid; i < p.n; i += THREADS) {
        const float s = sc[i];
        const bool exempt = p.window_W > 0 && pos[i] >= p.window_pos_min;
        if (!exempt && score_bin(s) == tb) {
            const uint64_t key = ((uint64_t)orderable(s) << 32) | (uint32_t)pos[i];
            if ((key >> (64 - resolved)) >= prefix) atomicOr(&evbits[i >> 5], 1u << (i & 31));
        }
    }
    __syncthreads();
}

// Where the passes over the rows find scores and positions: in memory, in LDS copies, or in the registers of
// the thread that owns the row (SRC = the number of 16-byte loads per thread: rows 4 (q THREADS + tid) .. + 3)
constexpr int SRC_MEMORY = 0, SRC_LDS = -1;

// bytes of dynamic LDS the selection of a step uses behind PostShared: the eviction bitmap, the
// lists (when they fit) and, for the passenger, the copies of the scores and positions
__host__ __device__ inline size_t select_dyn_bytes(int n, int N, int cap, bool lists_in_lds, bool resident)
{
    size_t b = ((size_t)((n + 31) / 32) * 4 + 15) & ~(size_t)15;
    if (lists_in_lds) b += ((size_t)(n - N) * 4 + 15) & ~(size_t)15;
    if (resident) b += (size_t)cap * 8;
    return b;
}

// What a selection does once its eviction bitmap is final and the evicted keys have been read: nothing, or hand the bitmap to the
// workgroups of the same launch that hold the rows (ShiftAround).  Every word travels with the epoch of the launch in one 8-byte
// store, so a reader needs no order between words: it reads one until it carries the epoch.
struct NoPublish {
    static constexpr bool ON = false;
    __device__ void arrive() const {}
    __device__ bool mine() const { return true; }
    __device__ void operator()(int, const uint32_t *, int) const {}
    __device__ void nothing(int) const {}
};
struct PublishWords {
    static constexpr bool ON = true;
    const ShiftAround &around;
    uint32_t drawn;      // thread 0: what the counter held, perhaps still on its way
    uint32_t *ticket;    // LDS
    // the ticket is needed before anything is written, and travels behind the scores till then: thread 0 hands it out ahead of a barrier, and
    // behind it the workgroup learns whether the selection is its own
    __device__ __forceinline__ void arrive() const
    {
        if (threadIdx.x == 0) *ticket = drawn - around.first_ticket;
    }
    __device__ __forceinline__ bool mine() const { return *ticket == 0; }
    __device__ __forceinline__ void put(int bh, int i, uint32_t w) const
    {
        __hip_atomic_store(around.words + (size_t)bh * around.stride + i, ((unsigned long long)(uint32_t)around.epoch << 32) | w,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // (by all threads of the workgroup)
    __device__ __forceinline__ void operator()(int bh, const uint32_t *evbits, int nwords) const
    {
        for (int i = threadIdx.x; i < nwords; i += blockDim.x) put(bh, 1 + i, evbits[i]);
        if (threadIdx.x == 0) put(bh, 0, 1);
    }
    __device__ __forceinline__ void nothing(int bh) const   // (impossible: the rows stay where they are)
    {
        if (threadIdx.x == 0) put(bh, 0, 2);
    }
};

// ------------------------------------------------------------- select + compaction
// `dyn`: dynamic LDS of select_dyn_bytes(...) bytes, 16-byte aligned.  The list of evicted rows lies in LDS when it fits, else in
// the scratch buffer.
// The caller keeps n <= 32 * THREADS (a thread owns one word of the eviction bitmap) and, with SRC > 0,
// n <= 4 * SRC * THREADS.
// (inlined: outlined, the parameter block would be passed through scratch memory)
// APPROX: the scores may be approximate (p.score_approx says).
template <int D, int SRC, int THREADS, bool APPROX, class Publish = NoPublish>
__device__ __forceinline__ void select_and_compact(const StepParams &p, PostShared &sh, unsigned char *dyn, int bh, const Publish &publish = {})
{
    constexpr int UPR = D / 8;
    constexpr int TAILU = THREADS > 512 || D == 64 ? SELECT_TAILU / 2 : SELECT_TAILU;   // (128 rows a batch, 256 of 64 with 1024 threads)
    // The rows [N, n), the only ones that can move (FILL layout), are requested with the scores; scoring rows exactly takes
    // the registers they would wait in, and they are then requested with the evicted keys.
    constexpr bool EARLY_TAIL = !APPROX;
    constexpr int NWAVES = THREADS / 64;
    constexpr bool RES = SRC == SRC_LDS;
    constexpr int NQ4 = SRC > 0 ? SRC : 1;
    constexpr bool PREG = SRC > 0 && SRC <= 3;   // positions in registers too (else read where they are needed)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int E = p.n - p.N;
    const float *sc_g = p.scores + (size_t)bh * p.cap;
    int32_t *pos = p.pos + (size_t)bh * p.cap;
    uint16_t *kb = p.k + (size_t)bh * p.cap * D;
    uint16_t *vb = p.v + (size_t)bh * p.cap * D;
    const int nwords = (p.n + 31) / 32;
    uint32_t *evbits = reinterpret_cast<uint32_t *>(dyn);
    size_t dyn_off = ((size_t)nwords * 4 + 15) & ~(size_t)15;
    int32_t *lists = p.lists + (size_t)bh * 4 * p.B;
    if (p.lists_in_lds) {
        lists = reinterpret_cast<int32_t *>(dyn + dyn_off);
        dyn_off += ((size_t)E * 4 + 15) & ~(size_t)15;
    }
    float *sc_l = reinterpret_cast<float *>(dyn + dyn_off);
    int32_t *pos_l = reinterpret_cast<int32_t *>(dyn + dyn_off + (size_t)p.cap * 4);
    // the LDS copies as LDS pointers, so that the loops use ds_read
    typedef __attribute__((address_space(3))) const float lds_cf32;
    typedef __attribute__((address_space(3))) const int32_t lds_ci32;
    typedef __attribute__((address_space(3))) const i32x4 lds_ci32x4;
    lds_cf32 *sc_s = (lds_cf32 *)sc_l;
    lds_ci32 *pos_s = (lds_ci32 *)pos_l;
    f32x4 sreg[NQ4];
    // score_place of the rows in registers, -1: not there, or exempt (with approximate scores a bit of `live` for each row that is neither)
    f32x4 place[APPROX ? 1 : NQ4];
    uint32_t live = 0;
    static_assert(4 * NQ4 <= 32, "one bit a row");
    i32x4 preg[PREG ? NQ4 : 1];
    // visit(row, score, position, k) for every row this thread owns, the k-th of at most 32.  Positions that lie in neither
    // registers nor LDS are read (and handed to visit) only where a pass asks for them: with a window, or to choose by them.
    auto for_rows = [&](bool positions, auto &&visit) {
        if constexpr (SRC > 0) {
#pragma unroll
            for (int q = 0; q < NQ4; ++q) {
                if (q * 4 * THREADS >= p.n) break;   // uniform
                const int i0 = 4 * (q * THREADS + tid);
                i32x4 pq = {0, 0, 0, 0};
                if constexpr (PREG) pq = preg[q];
                else if (positions && i0 < p.n) pq = *reinterpret_cast<const i32x4 *>(pos + i0);   // (a multiple of four rows)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i0 + e < p.n) visit(i0 + e, sreg[q][e], (int32_t)pq[e], 4 * q + e);
            }
        } else {
            if constexpr (RES) {
#pragma unroll 2
                for (int i = tid, k = 0; i < p.n; i += THREADS, ++k) visit(i, (float)sc_s[i], (int32_t)pos_s[i], k);
            } else if (positions) {
#pragma unroll 2
                for (int i = tid, k = 0; i < p.n; i += THREADS, ++k) visit(i, sc_g[i], pos[i], k);
            } else {
#pragma unroll 4
                for (int i = tid, k = 0; i < p.n; i += THREADS, ++k) visit(i, sc_g[i], 0, k);
            }
        }
    };
    auto exempt = [&](int32_t pi) { return p.window_W > 0 && pi >= p.window_pos_min; };
    KD_TL_DECL
    KD_TL(0);
#ifdef KD_TIMELINE
    if (threadIdx.x == 0) kd_tl[31] = 2;   // record kind: selection workgroup
#define KD_SEL_RETURN do { KD_TL(12); KD_TL_DUMP(p.timeline, blockIdx.x); return; } while (0)
#else
#define KD_SEL_RETURN return
#endif

    // ---- 0. every load that does not depend on the selection is issued here, so that the chain
    // below costs one memory round trip now and one for the evicted rows later: the scores and
    // positions of all rows (into registers, or by asynchronous copies into LDS, 1 KB per wave and
    // instruction; the buffers hold a multiple of four rows) and the running key sum.
    if constexpr (SRC > 0) {
#pragma unroll
        for (int q = 0; q < NQ4; ++q) {
            const int i = 4 * (q * THREADS + tid);
            sreg[q] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (i < p.n) sreg[q] = *reinterpret_cast<const f32x4 *>(sc_g + i);
            if constexpr (PREG) {
                preg[q] = i32x4{0, 0, 0, 0};
                if (i < p.n) preg[q] = *reinterpret_cast<const i32x4 *>(pos + i);
            }
        }
    }
    if (RES) {
        const int nchunks = (p.cap * 4 + 1023) / 1024;
        for (int c = wave; c < 2 * nchunks; c += NWAVES) {      // wave uniform
            const bool second = c >= nchunks;
            const int w0 = (second ? c - nchunks : c) * 256 + 4 * lane;   // first of this lane's four words
            const uint32_t dst = (uint32_t)(uintptr_t)(second ? (void *)pos_l : (void *)sc_l) + (uint32_t)(w0 - 4 * lane) * 4u;
            if (w0 < p.cap) lds_copy16(dst, second ? (const void *)(pos + w0) : (const void *)(sc_g + w0));
        }
    }
    const double ksum_old = tid < D ? p.ksum_next[(size_t)bh * D + tid] : 0.0;  // the sum step_main just wrote
    // The first half of the waves takes the K rows of the tail, the second half the V rows: thread (tail_row0, unit) the rows
    // tail_row0, tail_row0 + TROWS, ..
    constexpr int TROWS = THREADS / 2 / UPR;
    auto tail_row0 = [&]() { return (tid % (THREADS / 2)) / UPR; };
    auto tail_rows = [&]() { return wave >= NWAVES / 2 ? vb : kb; };
    const uint32_t unit_off = (uint32_t)(tid % UPR) * 8;
    u32x4 tailv[TAILU];
    auto request_rows = [&](int r0) {   // rows N + r0 + tail_row0, + TROWS, .. of the tail
#pragma unroll
        for (int q = 0; q < TAILU; ++q) {
            const int r = r0 + q * TROWS;   // uniform
            tailv[q] = u32x4{0u, 0u, 0u, 0u};
            if (r < E && r + tail_row0() < E)
                tailv[q] = *reinterpret_cast<const u32x4 *>(tail_rows() + (size_t)(p.N + r) * D + (uint32_t)(tail_row0() * D) + unit_off);
        }
    };
    auto request_tail = [&]() {
        if (p.layout == 1) request_rows(0);
    };
    if constexpr (EARLY_TAIL) request_tail();
    for (int i = tid; i < nwords; i += THREADS) evbits[i] = 0;
    const bool use_rec = E == 1 && p.argmax_rec != nullptr && p.window_W == 0 && 4 * p.splits <= HIST_BINS;   // uniform
    if (use_rec) {
        // the arg-max records of the attention launch travel with the loads above (the histogram's space
        // holds them: a single eviction builds no histogram)
        uint64_t *recs = reinterpret_cast<uint64_t *>(sh.hist);
        for (int s_ = tid; s_ < 2 * p.splits; s_ += THREADS) recs[s_] = p.argmax_rec[(size_t)bh * p.splits * 2 + s_];
    } else {
        for (int i = tid; i < HIST_BINS; i += THREADS) sh.hist[i] = 0;
    }
    bool approx = APPROX && p.score_approx != 0;   // uniform
    double mu = 0.0;   // the anchor as the attention left it (first used behind a later barrier)
    if (approx && tid < D) mu = p.anchor[(size_t)bh * D + tid];
    if (tid == 0) {
        sh.ncand = 0;
        sh.nev = 0;
        sh.tb = 0;
        sh.bad = 0;
    }
    KD_TL(1);   // loads issued
    if (RES) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's copies have landed
    if (E == 1) publish.arrive();
    __syncthreads();   // every wave's part of the copies; the cleared histogram and bitmap
    if (E == 1 && !publish.mine()) return;   // uniform, like the one below; nothing has been written yet
    KD_TL(2);   // scores and positions in LDS

    if (E == 1 && !approx) {
        // ---- 1'. a single row to evict (the generation phase): the arg-max by (score bits, position)
        // replaces histogram, threshold and ranking
        // The attention launch may have left the arg-max by (score bits, row) of every workgroup's rows
        // (p.argmax_rec): unless two rows share the largest score bits -- then the lower position has to
        // win, and positions are not row numbers -- the row to evict is read off those few records.
        uint64_t gbest = 0;
        bool known = false;
        if (use_rec) {
            if (wave == 0) {
                // the lanes share the records (a workgroup of the attention left each), then fold
                const uint64_t *recs = reinterpret_cast<const uint64_t *>(sh.hist);
                uint64_t b0 = 0;
                bool tie = false;
                auto fold = [&](uint64_t ob, bool ot) {   // (no record is folded in twice)
                    const uint32_t hb = (uint32_t)(b0 >> 32), ho = (uint32_t)(ob >> 32);
                    if (ho > hb) {
                        b0 = ob;
                        tie = ot;
                    } else if (ho == hb && ob != 0) {
                        tie = true;
                        b0 = ob > b0 ? ob : b0;
                    }
                };
                for (int s_ = lane; s_ < p.splits; s_ += 64) fold(recs[2 * s_], recs[2 * s_ + 1] != 0);
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t lo = __shfl_xor((uint32_t)b0, off), hi = __shfl_xor((uint32_t)(b0 >> 32), off);
                    const bool ot = __shfl_xor((int)tie, off) != 0;
                    fold(((uint64_t)hi << 32) | lo, ot);
                }
                if (lane == 0) {
                    sh.sel_cnt = (b0 != 0 && !tie) ? 1u : 0u;
                    sh.tb = (int)(uint32_t)b0;
                    if (b0 != 0 && !tie) evbits[(uint32_t)b0 >> 5] |= 1u << ((uint32_t)b0 & 31);
                }
            }
            __syncthreads();
            known = sh.sel_cnt != 0;   // uniform
            gbest = known ? 1 : 0;
        }
        if (!known) {
            uint64_t best = 0;   // 0: no row (every real key is larger: orderable() of a finite score is > 0)
            int besti = -1;
            for_rows(true, [&](int i, float s, int32_t pi, int) {
                if (!exempt(pi)) {
                    const uint64_t key = ((uint64_t)orderable(s) << 32) | (uint32_t)pi;
                    if (key > best) {
                        best = key;
                        besti = i;
                    }
                }
            });
            uint64_t wbest = best;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t lo = __shfl_xor((uint32_t)wbest, off), hi = __shfl_xor((uint32_t)(wbest >> 32), off);
                const uint64_t o = ((uint64_t)hi << 32) | lo;
                wbest = o > wbest ? o : wbest;
            }
            if (lane == 0) sh.wave_tot64[wave] = wbest;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) gbest = sh.wave_tot64[w] > gbest ? sh.wave_tot64[w] : gbest;
            // positions are unique within a head, so exactly one thread holds the winning key
            if (besti >= 0 && best == gbest) {
                atomicOr(&evbits[besti >> 5], 1u << (besti & 31));
                sh.tb = besti;
            }
            __syncthreads();
        }
        if (p.layout == 1 && gbest != 0) {
            // FILL: the one tail row (row N, this step's token) travels with the evicted key: the rest of the work
            // is one row read and at most one row moved, done here without lists
            const int e = sh.tb;
            double x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = 0.0;
            u32x4 tail = {0u, 0u, 0u, 0u};
            if constexpr (EARLY_TAIL) tail = tailv[0];
            else if (tail_row0() == 0) tail = *reinterpret_cast<const u32x4 *>(tail_rows() + (size_t)p.N * D + unit_off);
            if (tid < UPR) {
                const u32x4 w = *reinterpret_cast<const u32x4 *>(kb + (size_t)e * D + tid * 8);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[2 * i] = bf16_lo(w[i]);
                    x[2 * i + 1] = bf16_hi(w[i]);
                }
            }
            if (p.anchor_mode == 1 && tid < 64) {  // unit key: x / |k|; the row's UPR lanes are the first of wave 0
                double k2 = 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) k2 += x[i] * x[i];
                k2 = row_allreduce_f64<UPR>(k2);
                const double nk = sqrt(k2);
                const double inv = nk > 0.0 ? 1.0 / nk : 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] *= inv;
            }
            if (tid < UPR) {
#pragma unroll
                for (int i = 0; i < 8; ++i) sh.colsum[0][tid * 8 + i] = x[i];
            }
            // the evicted key has been read: its slot may take the tail row (the thread that read
            // unit u of K is the one that writes unit u of K)
            if (e != p.N && tail_row0() == 0) {
                *reinterpret_cast<u32x4 *>(tail_rows() + (size_t)e * D + unit_off) = tail;
                if (tid == 0) pos[e] = p.pos0 + (p.N - p.len);
            }
            __syncthreads();
            if (tid < D) p.ksum_next[(size_t)bh * D + tid] = ksum_old - sh.colsum[0][tid];
            KD_SEL_RETURN;
        }
        // (ORDERED: the evicted row goes the way of the others below; where nothing
        // could be evicted -- impossible -- the bitmap stays empty and the count check reports it)
    } else {
    // Exact score of row i, in the arithmetic of the attention's exact scores: the UPR lanes that share it call this together, each with its 16-byte unit.
    auto exact_score = [&](int i) {
        const int u = tid % UPR;
        const u32x4 w = *reinterpret_cast<const u32x4 *>(kb + (size_t)i * D + u * 8);
        double dot = 0.0, k2 = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double x0 = bf16_lo(w[j]), x1 = bf16_hi(w[j]);
            dot = __builtin_fma(sh.mu[u * 8 + 2 * j], x0, dot);
            k2 = __builtin_fma(x0, x0, k2);
            dot = __builtin_fma(sh.mu[u * 8 + 2 * j + 1], x1, dot);
            k2 = __builtin_fma(x1, x1, k2);
        }
        return finish_score(row_score_sum_f64<UPR>(dot), row_score_sum_f64<UPR>(k2), sum_of_pieces<D>(sh.mu2), p.eps);
    };
    for (;;) {   // (a second time, with exact scores of all rows, where approximate ones do not do)
    // ---- 1. histogram of the non-exempt scores in LDS
    auto count = [&](float s, float at) {
        atomicAdd(&sh.hist[(int)at], 1u);
        if (APPROX && s != s) sh.bad = 1;
    };
    if constexpr (SRC > 0) {
#pragma unroll
        for (int q = 0; q < NQ4; ++q) {
            if (q * 4 * THREADS >= p.n) break;   // uniform
            const int i0 = 4 * (q * THREADS + tid);
            i32x4 pq = {0, 0, 0, 0};
            if constexpr (PREG) pq = preg[q];
            else if (p.window_W > 0 && i0 < p.n) pq = *reinterpret_cast<const i32x4 *>(pos + i0);   // (a multiple of four rows)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float at = i0 + e >= p.n || exempt((int32_t)pq[e]) ? -1.f : score_place(sreg[q][e]);
                if constexpr (APPROX) live |= at >= 0.f ? 1u << (4 * q + e) : 0u;
                else place[q][e] = at;
                if (at >= 0.f) count(sreg[q][e], at);
            }
        }
    } else {
        for_rows(p.window_W > 0, [&](int, float s, int32_t pi, int) {
            if (!exempt(pi)) count(s, score_place(s));
        });
    }
    publish.arrive();
    __syncthreads();
    if (!publish.mine()) return;
    if (approx && tid < D) {   // (whole waves)
        sh.mu[tid] = mu;
        const double sq = row_allreduce_f64<16>(mu * mu);
        if ((lane & 15) == 0) sh.mu2[tid / 16] = sq;
    }
    KD_TL(3);   // scores binned

    // ---- 2. threshold bin: thread t owns the HIST_BINS / THREADS bins below its top one, highest first
    uint32_t cnt[HIST_BINS / THREADS];
    uint32_t mine = 0;
    const int top = HIST_BINS - 1 - (HIST_BINS / THREADS) * tid;
#pragma unroll
    for (int j = 0; j < HIST_BINS / THREADS; ++j) {
        cnt[j] = sh.hist[top - j];
        mine += cnt[j];
    }
    uint32_t total;
    uint32_t above = block_exclusive_scan_t<THREADS, uint32_t>(mine, sh.wave_tot, &total);
    if (above < (uint32_t)E && above + mine >= (uint32_t)E) {
#pragma unroll
        for (int j = 0; j < HIST_BINS / THREADS; ++j) {
            if (above + cnt[j] >= (uint32_t)E) {
                sh.tb = top - j;
                break;
            }
            above += cnt[j];
        }
    }
    if (tid == 0 && total < (uint32_t)E) atomicOr(p.status, STATUS_SELECT_COUNT);  // cannot happen: E <= candidates
    __syncthreads();
    const int tb = sh.tb;
    KD_TL(4);   // threshold bin known

    // Above the bin -> evicted, inside it -> candidate for the exact ranking.  The E-th largest approximate score lies in the
    // bin and the E-th largest exact one within the slack of it: a row more than twice the slack above the bin is evicted
    // whatever its exact score, one as far below it stays, and those between are candidates (the last term covers the
    // rounding of the bin edges).
    const float above_from = (float)(tb + 1);   // (no place of the top bin reaches it)
    const float reach = approx ? 2.f * SCORE_SLACK + 1e-6f : 0.f;
    uint32_t nabove = 0;   // of the rows this lane has looked at (or, on rows in LDS or memory, its wave)
    // a row that may be chosen, with its place: true if it lies above the bin; in the bin, it joins the candidates
    auto classify = [&](int i, float s, float at, int32_t pi) {
        bool above_bin, in_bin;
        if constexpr (APPROX) {
            above_bin = score_bin(s - reach) > tb;
            in_bin = score_bin(s + reach) >= tb;
        } else {
            above_bin = at >= above_from;
            in_bin = at >= (float)tb;
        }
        if (!above_bin && in_bin) {
            const uint32_t c = atomicAdd(&sh.ncand, 1u);
            if (c < CAND_MAX) {
                sh.cand_slot[c] = (uint32_t)i;
                sh.cand_key[c] = orderable(s);
                sh.cand_pos[c] = pi;
            }
        }
        return above_bin;
    };
    // The bitmap is written word by word, without atomics: a wave holds whole words of it.
    if constexpr (SRC > 0) {
#pragma unroll
        for (int q = 0; q < NQ4; ++q) {
            if (q * 4 * THREADS >= p.n) break;   // uniform
            const int i0 = 4 * (q * THREADS + tid);
            uint32_t four = 0;   // the thread's four rows; eight lanes make a word
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float at = APPROX ? 0.f : place[APPROX ? 0 : q][e];
                if ((!APPROX || ((live >> (4 * q + e)) & 1u)) && classify(i0 + e, sreg[q][e], at, PREG ? (int32_t)preg[PREG ? q : 0][e] : 0))
                    four |= 1u << e;
            }
            nabove += (uint32_t)__popc(four);
            uint32_t word = four << (4 * (lane & 7));
            word |= dpp_fetch<0xB1, 0xF>(word);    // quad_perm [1,0,3,2]
            word |= dpp_fetch<0x4E, 0xF>(word);    // quad_perm [2,3,0,1]
            word |= dpp_fetch<0x141, 0xF>(word);   // row_half_mirror
            if ((lane & 7) == 0 && i0 < p.n) evbits[i0 >> 5] = word;
        }
        nabove = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(nabove), 63);
    } else {
        auto mark = [&](int i, bool above_bin) {   // (rows i of the wave's lanes: 64 in a row from a multiple of 64)
            const uint64_t m = __ballot(above_bin);
            if (lane == 0) *reinterpret_cast<uint64_t *>(evbits + (i >> 5)) = m;
            nabove += (uint32_t)__popcll(m);
        };
#pragma unroll 2
        for (int i0 = 64 * wave; i0 < p.n; i0 += THREADS) {   // uniform per wave
            const int i = i0 + lane;
            bool above_bin = false;
            if (i < p.n) {
                const float s = RES ? (float)sc_s[i] : sc_g[i];
                const int32_t pi = RES ? (int32_t)pos_s[i] : p.window_W > 0 ? pos[i] : 0;
                if (!exempt(pi)) above_bin = classify(i, s, APPROX ? 0.f : score_place(s), pi);
            }
            mark(i0, above_bin);
        }
    }
    if (lane == 0 && nabove != 0) atomicAdd(&sh.nev, nabove);
    __syncthreads();
    const uint32_t ncand = sh.ncand, need = (uint32_t)E - sh.nev;
    if constexpr (APPROX) {
    if (approx && (sh.bad || ncand > CAND_MAX)) {   // uniform
        // rare: nearly identical keys, or keys out of the range of the approximation
        for (int r0 = 0; r0 < p.n; r0 += THREADS / UPR) {   // uniform
            const int i = r0 + tid / UPR;
            const float s = exact_score(min(i, p.n - 1));
            if (i < p.n && tid % UPR == 0) {
                if constexpr (RES) sc_l[i] = s;
                else p.scores[(size_t)bh * p.cap + i] = s;
            }
        }
        for (int i = tid; i < HIST_BINS; i += THREADS) sh.hist[i] = 0;
        for (int i = tid; i < nwords; i += THREADS) evbits[i] = 0;
        __syncthreads();
        if (tid == 0) sh.ncand = sh.nev = 0;
        live = 0;
        if constexpr (SRC > 0) {
#pragma unroll
            for (int q = 0; q < NQ4; ++q) {
                const int i = 4 * (q * THREADS + tid);
                if (i < p.n) sreg[q] = *reinterpret_cast<const f32x4 *>(sc_g + i);
            }
        }
        approx = false;
        __syncthreads();
        continue;
    }
    if (approx) {
        for (uint32_t c0 = 0; c0 < ncand; c0 += THREADS / UPR) {   // uniform
            const uint32_t c = c0 + tid / UPR;
            const float s = exact_score((int)sh.cand_slot[min(c, ncand - 1)]);
            if (c < ncand && tid % UPR == 0) sh.cand_key[c] = orderable(s);
        }
        __syncthreads();
    }
    }   // APPROX
    if constexpr (!RES && !PREG) {
        for (uint32_t c = tid; c < min(ncand, (uint32_t)CAND_MAX); c += THREADS) sh.cand_pos[c] = pos[sh.cand_slot[c]];
        __syncthreads();
    }
    KD_TL(5);   // candidates collected

    // ---- 3. exact ranking inside the bin by (score bits, position), largest first: a wave takes a
    // candidate, its lanes compare it with 64 others at a time and count by ballot
    if (ncand <= CAND_MAX) {
        for (uint32_t c = wave; c < ncand; c += NWAVES) {   // uniform per wave
            const uint32_t key = sh.cand_key[c];
            const int32_t cp = sh.cand_pos[c];
            uint32_t rank = 0;
            for (uint32_t o0 = 0; o0 < ncand; o0 += 64) {
                const uint32_t o = o0 + lane;
                bool gt = false;
                if (o < ncand) {
                    const uint32_t ok = sh.cand_key[o];
                    gt = (ok > key) || (ok == key && sh.cand_pos[o] > cp);
                }
                rank += (uint32_t)__popcll(__ballot(gt));
            }
            if (lane == 0 && rank < need) atomicOr(&evbits[sh.cand_slot[c] >> 5], 1u << (sh.cand_slot[c] & 31));
        }
        __syncthreads();
    } else {
        radix_select_in_bin<THREADS>(p, sh, RES ? sc_l : sc_g, RES ? pos_l : pos, evbits, tb, need);   // (exact scores here)
    }
    break;
    }   // for (;;)
    }   // E > 1, or approximate scores
    KD_TL(6);   // ranking done: the eviction bitmap and the list of evicted rows are final

    // ---- 4. the evicted rows in ascending order, from the bitmap: thread t owns word t = rows [32 t, 32 t + 32), or its share of a word
    // where there are threads enough (it lists its rows one after the other: with whole words the list of 32 of 288 rows took 1.4 us of the
    // 6.7 behind the start of a selection).  The count of
    // evicted rows before each word also gives the destinations of the ORDERED layout, and of the FILL layout the rank of a hole
    // (the k-th evicted row below N is hole k) and of a mover.
    int32_t *evlist = lists;
    if constexpr (!EARLY_TAIL) request_tail();
    uint32_t *word_base = sh.cand_slot;   // the candidate arrays are free by now
    static_assert(MAX_CAP / 32 <= CAND_MAX, "one count per bitmap word");
    {
        uint32_t total;
        const int split = 4 * nwords <= THREADS ? 2 : 2 * nwords <= THREADS ? 1 : 0, bits = 32 >> split;   // uniform
        const int word = tid >> split, first = bits * (tid & ((1 << split) - 1));
        uint32_t w = word < nwords ? (evbits[word] >> first) & (0xFFFFFFFFu >> (32 - bits)) : 0u;
        uint32_t at = block_exclusive_scan_t<THREADS, uint32_t>((uint32_t)__popc(w), sh.wave_tot2, &total);
        // an impossible count is reported and nothing is moved (keeps every index in range)
        if (total != (uint32_t)E) {   // uniform
            if (tid == 0) atomicOr(p.status, STATUS_SELECT_COUNT);
            publish.nothing(bh);
            KD_SEL_RETURN;
        }
        if (word < nwords && first == 0) word_base[word] = at;
        for (; w; w &= w - 1) evlist[at++] = 32 * word + first + __ffs(w) - 1;
    }
    __syncthreads();
    auto before = [&](int i) { return (int)(word_base[i >> 5] + (uint32_t)__popc(evbits[i >> 5] & ((1u << (i & 31)) - 1u))); };
    auto evicted = [&](int i) { return ((evbits[i >> 5] >> (i & 31)) & 1u) != 0; };
    KD_TL(7);   // evicted rows listed

    // ---- 5. compaction, and the evicted keys taken out of the running key sum.  A sum of doubles depends in its last bit on the
    // order of its terms: E terms are dealt to KEY_PARTS parts in rounds of 64 / UPR (the lanes of a wave that share no row), in the order of the
    // tail rows they make room for (FILL) or of the rows themselves (ORDERED), whatever the number of threads, so that the
    // passenger leaves the very sum step_post does.
    constexpr int RPW = 64 / UPR, KWAVES = NWAVES / 2, TURNS = KEY_PARTS / KWAVES;
    static_assert(TURNS >= 1 && TURNS * KWAVES == KEY_PARTS && TAILU % TURNS == 0, "a round's part follows from its place in a batch");
    static_assert(TROWS == RPW * KWAVES, "a wave of the first half takes RPW rows a round");
    const bool keys = wave < KWAVES;   // uniform per wave: takes K rows (the others V rows)
    constexpr int KEY_ROWS = KEY_PARTS * RPW;   // ORDERED: rows a round
    const bool part_waves = wave < KEY_PARTS;   // uniform per wave
    static_assert(NWAVES >= KEY_PARTS, "a wave for every part");
    double acc[TURNS][8];
#pragma unroll
    for (int t = 0; t < TURNS; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[t][i] = 0.0;
    auto add_key = [&](const u32x4 &w, double (&a)[8]) {
        double x[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = bf16_lo(w[i]);
            x[2 * i + 1] = bf16_hi(w[i]);
        }
        double inv = 1.0;
        if (p.anchor_mode == 1) {  // unit key: x / |k|
            double k2 = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) k2 += x[i] * x[i];
            k2 = row_allreduce_f64<UPR>(k2);
            const double nk = sqrt(k2);
            inv = nk > 0.0 ? 1.0 / nk : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] += (p.anchor_mode == 1) ? x[i] * inv : x[i];
    };
    if (p.layout == 1) {
        // FILL: the k-th surviving row of [N, n) moves into the k-th evicted slot of [0, N).  Rows from N on belong to this step's
        // block: row i holds token pos0 + (i - len).  The thread that brings a piece of a K row takes the piece it overwrites
        // along (a load ahead of a store of the same thread to the same place), and of a tail row that is itself evicted the
        // piece it already holds: no wave waits for another.
        const int nholes = before(p.N);   // (row N exists: n > N)
        for (int r0 = 0; r0 < E; r0 += TAILU * TROWS) {   // uniform
            if (r0 > 0) request_rows(r0);
            int to[TAILU];
#pragma unroll
            for (int q = 0; q < TAILU; ++q) {
                const int r = r0 + q * TROWS + tail_row0();
                to[q] = -1;
                if (r0 + q * TROWS < E && r < E && !evicted(p.N + r)) to[q] = evlist[r - (before(p.N + r) - nholes)];
            }
            u32x4 old[TAILU];
            if (keys) {
#pragma unroll
                for (int q = 0; q < TAILU; ++q) {
                    old[q] = tailv[q];   // (zeros past the last row)
                    if (to[q] >= 0) old[q] = *reinterpret_cast<const u32x4 *>(kb + (size_t)to[q] * D + unit_off);
                }
            }
#pragma unroll
            for (int q = 0; q < TAILU; ++q)
                if (to[q] >= 0) *reinterpret_cast<u32x4 *>(tail_rows() + (size_t)to[q] * D + unit_off) = tailv[q];
            if (keys) {
#pragma unroll
                for (int q = 0; q < TAILU; ++q)
                    if (r0 + q * TROWS < E) add_key(old[q], acc[q % TURNS]);
            } else if (unit_off == 0) {
#pragma unroll
                for (int q = 0; q < TAILU; ++q)
                    if (to[q] >= 0) pos[to[q]] = p.pos0 + (p.N + r0 + q * TROWS + tail_row0() - p.len);
            }
        }
    } else {
        // ORDERED: kept row i moves to i - (evicted rows before i); positions are compacted here, the
        // K/V rows by compact_ordered_kernel.  A position lands at or below the row it came from: from registers or
        // the LDS copy nothing can be overwritten before it is read; reading from memory, the rows are taken in
        // ascending chunks, each read, then (barrier) written.
        // Nothing moves here, so KEY_PARTS waves take keys, one part each (a passenger: all of its waves).  The keys are added ahead
        // of the positions: behind their stores, the wait for the keys would be one for the stores too.
        u32x4 old[TAILU];
        for (int r0 = 0; r0 < E && part_waves; r0 += TAILU * KEY_ROWS) {   // uniform per wave
#pragma unroll
            for (int q = 0; q < TAILU; ++q) {
                const int r = r0 + q * KEY_ROWS + tid / UPR;
                old[q] = u32x4{0u, 0u, 0u, 0u};
                if (r < E) old[q] = *reinterpret_cast<const u32x4 *>(kb + (size_t)evlist[r] * D + unit_off);
            }
#pragma unroll
            for (int q = 0; q < TAILU; ++q)
                if (r0 + q * KEY_ROWS < E) add_key(old[q], acc[0]);
        }
        if constexpr (Publish::ON) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the evicted keys are in registers: their rows may be overwritten
            __syncthreads();
            publish(bh, evbits, nwords);
        }
        int32_t *dst = p.dstmap + (size_t)bh * p.cap;
        // four rows, which share a bitmap word (the buffers hold a multiple of four rows)
        auto place_rows = [&](int i, const i32x4 &at) {
            const uint32_t word = evbits[i >> 5], bit = (uint32_t)i & 31u;
            int to = i - (int)(word_base[i >> 5] + (uint32_t)__popc(word & ((1u << bit) - 1u)));
            i32x4 d;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool gone = ((word >> (bit + e)) & 1u) != 0;
                d[e] = gone ? -1 : to;
                if (!gone && i + e < p.n) pos[to] = at[e];
                to += gone ? 0 : 1;
            }
            if (!Publish::ON && p.layout != LAYOUT_SHIFT_HERE) *reinterpret_cast<i32x4 *>(dst + i) = d;
        };
        if constexpr (PREG) {
#pragma unroll
            for (int q = 0; q < NQ4; ++q) {
                const int i = 4 * (q * THREADS + tid);
                if (i < p.n) place_rows(i, preg[q]);
            }
        } else if constexpr (RES) {
            for (int i = 4 * tid; i < p.n; i += 4 * THREADS) place_rows(i, (i32x4)*(lds_ci32x4 *)(pos_s + i));
        } else {
            for (int i0 = 0; i0 < p.n; i0 += THREADS) {   // uniform
                const int i = i0 + tid;
                int32_t pi = 0;
                if (i < p.n) pi = pos[i];
                __syncthreads();
                if (i < p.n) {
                    if (evicted(i)) dst[i] = -1;
                    else {
                        const int to = i - before(i);
                        dst[i] = to;
                        pos[to] = pi;
                    }
                }
            }
        }
    }
    // ORDERED, a short cache: the rows behind the first evicted one are shifted here, pass by pass in ascending order (a row
    // moves down, so no pass overwrites what a later one has to read); the first pass is requested ahead of the key sum.
    constexpr int SHIFTU = 8;
    const bool shift_here = PREG && p.layout == LAYOUT_SHIFT_HERE;   // uniform (such a cache has at most 768 rows: positions in registers)
    u32x4 moved[SHIFTU];
    auto request_shift = [&](int i0) {
#pragma unroll
        for (int q = 0; q < SHIFTU; ++q) {
            const int i = i0 + q * TROWS + tail_row0();
            if (i < p.n) moved[q] = *reinterpret_cast<const u32x4 *>(tail_rows() + (size_t)i * D + unit_off);
        }
    };
    if (shift_here) request_shift(evlist[0]);
    KD_TL(8);   // moves issued
    if (p.layout == 1 ? keys : part_waves) {
#pragma unroll
        for (int t = 0; t < TURNS; ++t) {
            if (t > 0 && p.layout != 1) break;   // uniform
#pragma unroll
            for (int i = 0; i < 8; ++i) {   // the rows of the wave (lanes with the same unit)
                acc[t][i] = sum_over_units_f64<UPR>(acc[t][i]);
            }
            if (lane < UPR) {
#pragma unroll
                for (int i = 0; i < 8; ++i) sh.colsum[t * KWAVES + wave][lane * 8 + i] = acc[t][i];
            }
        }
    }
    if (shift_here) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the rows of the first pass (and the evicted keys) are in registers
    __syncthreads();
    if (shift_here) {
        for (int i0 = evlist[0]; i0 < p.n; i0 += SHIFTU * TROWS) {   // uniform
            if (i0 > evlist[0]) {
                request_shift(i0);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
            }
#pragma unroll
            for (int q = 0; q < SHIFTU; ++q) {
                const int i = i0 + q * TROWS + tail_row0();
                if (i < p.n && !evicted(i))
                    *reinterpret_cast<u32x4 *>(tail_rows() + (size_t)(i - before(i)) * D + unit_off) = moved[q];
            }
        }
    }
    if (tid < D) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < KEY_PARTS; ++w) s += sh.colsum[w][tid];
        p.ksum_next[(size_t)bh * D + tid] = ksum_old - s;
    }
    KD_TL(9);   // key sum stored
#ifdef KD_TIMELINE
    __builtin_amdgcn_s_waitcnt(0x0F70);
    KD_SEL_RETURN;
#endif
#undef KD_SEL_RETURN
}

}  // namespace kd
