// step_post: selection and compaction (Eq. 6-7) running next to the log-sum-exp merge of the
// attention partials; step_score: the cosine score (appendix "FLOP count of KeyDiff") of a cache
// outside a block step (inside one, step_main scores the keys while it holds them in LDS).
//
// The score that decides an eviction is IEEE double arithmetic on the bf16 data,
// rounded once to float: s_i = mu.k_i / max(|mu||k_i|, eps) with mu = ksum / n, so
// the retained set does not depend on summation order beyond the last bit of a double.
//
// Selection.  One workgroup per head loads the head's scores once, bins them into a
// 4096-bin LDS histogram (a monotone map of the float), scans it for the bin that
// holds the E-th largest score, evicts everything above that bin and ranks the few
// rows inside it exactly by (score bits, position): equal scores keep the lower
// position.  It then compacts the cache and takes the evicted keys out of ksum.
#include "kd_kernels.h"
#include "kd_device.h"
#include "kd_select.h"

namespace kd {

constexpr int SCORE_WAVES = SCORE_THREADS / 64;
constexpr int MERGE_THREADS = 256;   // workgroup size of the stand-alone merge


// ------------------------------------------------------------------------ scores
struct ScoreShared {
    double mu[128];
    double red[SCORE_WAVES];
    double dot[SCORE_WAVES][64];  // per-wave staging of (mu.k, |k|^2) so that sqrt and divide run on full waves
    double k2[SCORE_WAVES][64];
};

// Rows [row0, row1) of head bh (at most SCORE_ROWS), scored against the anchor ksum / n.  D/8 lanes
// share a row (one 16-byte unit each); a wave takes SCORE_ROWS / SCORE_WAVES consecutive rows, stages
// (mu.k, |k|^2) of each row in LDS and then lane i finishes row i of them.  Small row counts per wave
// and two waves per SIMD: the pass is one memory round trip plus a chain of double-precision
// arithmetic, and what hides either is other waves.
template <int D>
__device__ __forceinline__ void score_rows(const StepParams &p, ScoreShared &sh, int bh, int row0, int row1)
{
    constexpr int UPR = D / 8;
    constexpr int RPW = 64 / UPR;                   // rows per wave per pass
    constexpr int WROWS = SCORE_ROWS / SCORE_WAVES; // rows per wave
    constexpr int NP = WROWS / RPW;                 // passes per wave
    static_assert(NP >= 2 && NP % 2 == 0 && WROWS <= 64, "a wave takes an even number of passes and at most 64 rows");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int u = lane % UPR, rl = lane / UPR;
    const uint16_t *kb = p.k + (size_t)bh * p.cap * D;
    // the rows are requested ahead of the key sum
    const int base = row0 + wave * WROWS;
    u32x4 w[NP];
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) {
        const int row = base + ps * RPW + rl;
        u32x4 z = {0u, 0u, 0u, 0u};
        if (row < row1) z = *reinterpret_cast<const u32x4 *>(kb + (size_t)row * D + u * 8);
        w[ps] = z;
    }
    // anchor = ksum / n (Method, "Efficient Variant"); |mu| by a fixed-shape reduction
    double m = 0.0;
    if (tid < D) {
        m = p.ksum[(size_t)bh * D + tid] / (double)p.n;
        sh.mu[tid] = m;
    }
    double sq = m * m;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) sq += shfl_xor_f64(sq, off);
    if (lane == 0) sh.red[wave] = sq;
    __syncthreads();
    double mu2 = 0.0;
#pragma unroll
    for (int wv = 0; wv < SCORE_WAVES; ++wv) mu2 += sh.red[wv];

    double mreg[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) mreg[i] = sh.mu[u * 8 + i];
    // products of two bf16 values are exact in double, so fma(a, a, .) is the plain sum of squares;
    // mu.k takes one rounding per term either way
    auto partial = [&](const u32x4 &wv, double &dot, double &k2) {
        dot = 0.0;
        k2 = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double a = bf16_lo(wv[i]), b = bf16_hi(wv[i]);
            dot = __builtin_fma(mreg[2 * i], a, dot);
            k2 = __builtin_fma(a, a, k2);
            dot = __builtin_fma(mreg[2 * i + 1], b, dot);
            k2 = __builtin_fma(b, b, k2);
        }
    };
    if constexpr (UPR == 16) {
        // two passes at a time: the four quantities are summed over the 16 lanes of a row with 5
        // additions per lane; lanes 0-3 of a row end with mu.k of the first pass, 4-7 with its
        // |k|^2, 8-11 and 12-15 with those of the second
#pragma unroll
        for (int ps = 0; ps < NP; ps += 2) {
            double d0, q0, d1, q1;
            partial(w[ps], d0, q0);
            partial(w[ps + 1], d1, q1);
            const double v = row_reduce_scatter4_f64(d0, q0, d1, q1, u);
            if ((u & 3) == 0) {
                const int slot = (ps + (u >> 3)) * RPW + rl;
                if (u & 4) sh.k2[wave][slot] = v;
                else sh.dot[wave][slot] = v;
            }
        }
    } else {
#pragma unroll
        for (int ps = 0; ps < NP; ++ps) {
            double dot, k2;
            partial(w[ps], dot, k2);
            dot = row_allreduce_f64<UPR>(dot);
            k2 = row_allreduce_f64<UPR>(k2);
            if (u == 0) {
                sh.dot[wave][ps * RPW + rl] = dot;
                sh.k2[wave][ps * RPW + rl] = k2;
            }
        }
    }
    // same wave wrote and reads: the LDS accesses of one wave complete in order; the fence only
    // keeps the compiler from moving the reads above the writes
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int row = base + lane;
    if (lane < WROWS && row < row1) {
        const double dot = sh.dot[wave][lane], k2 = sh.k2[wave][lane];
        const float sc = finish_score(dot, k2, mu2, p.eps);
        p.scores[(size_t)bh * p.cap + row] = sc;
        if (p.scores_out) p.scores_out[(size_t)bh * p.n + row] = sc;
    }
}


// ------------------------------------------------------------------------ merge
// Thread gid takes four output values: step_main leaves a partial in its accumulator layout -- per
// 32-row block D/8 slabs of 512 bytes, slab 4 db + jj holding for lane (h, l32) the values
// d = 32 db + 8 jj + 4 h .. + 3 of row l32 -- and consecutive threads read consecutive lanes of a slab.
// MB: splits requested together
template <int D, int MB = 16>
__device__ __forceinline__ void merge_rows(const StepParams &p, size_t gid)
{
    constexpr int SLABS = D / 8;
    const int BH = p.batch * p.hkv;
    const int Mtot = p.G * p.Bt;
    const int nblk = (Mtot + 31) / 32;
    const size_t rows = (size_t)BH * Mtot;
    const int L = (int)(gid % 64), slab = (int)((gid / 64) % SLABS);
    const size_t blkid = gid / (64 * SLABS);   // (head, 32-row block)
    if (blkid >= (size_t)BH * nblk) return;
    const int bh = (int)(blkid / nblk), m = (int)(blkid % nblk) * 32 + (L & 31);
    if (m >= Mtot) return;
    const size_t row = (size_t)bh * Mtot + m;
    const size_t pstride = (size_t)BH * nblk * SLABS * 64 * 4;          // halfs per split
    const _Float16 *pbase = p.part_o + ((blkid * SLABS + slab) * 64 + L) * 4;
    // One memory round trip: the (max, sum) pairs and the partial rows of a batch of splits are
    // requested together; only with more splits than a batch holds does a second batch follow, and
    // the running result is then rescaled to the larger reference (as inside the attention).
    float mx = -INFINITY;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float Lsum = 0.f;
    for (int s0 = 0; s0 < p.splits; s0 += MB) {
        float2 ml[MB];
        f16x4 o[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const bool live = s0 + i < p.splits;
            const f16x4 zero = {(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
            ml[i] = live ? p.part_ml[(size_t)(s0 + i) * rows + row] : make_float2(-INFINITY, 0.f);
            o[i] = live ? *reinterpret_cast<const f16x4 *>(pbase + (size_t)(s0 + i) * pstride) : zero;
        }
        float bm = ml[0].x;
#pragma unroll
        for (int i = 1; i < MB; ++i) bm = fmaxf(bm, ml[i].x);
        if (bm > mx) {
            const float down = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx - bm);
            acc.x *= down;
            acc.y *= down;
            acc.z *= down;
            acc.w *= down;
            Lsum *= down;
            mx = bm;
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            // a partial is its split's output normalised by its own row sum: weight it by that sum
            const float w = ml[i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[i].x - mx) * ml[i].y;
            acc.x += w * (float)o[i][0];
            acc.y += w * (float)o[i][1];
            acc.z += w * (float)o[i][2];
            acc.w += w * (float)o[i][3];
            Lsum += w;
        }
    }
    const float inv = 1.f / Lsum;
    const int g = m / p.Bt, j = m % p.Bt;
    const int d0 = 8 * slab + 4 * (L >> 5);
    bf16x4 o;
    o[0] = (__bf16)(acc.x * inv);
    o[1] = (__bf16)(acc.y * inv);
    o[2] = (__bf16)(acc.z * inv);
    o[3] = (__bf16)(acc.w * inv);
    *reinterpret_cast<bf16x4 *>(p.out + (((size_t)bh * p.G + g) * p.Bt + j) * D + d0) = o;
}

// The same for at most four splits, MERGE_PIECES pieces of four values a thread (gid0, gid0 + stride, ..), all of them requested
// together: a piece is a few loads then, and what the merge takes is as many bytes in flight from fewer workgroups (merge of 4 splits of
// 2048 rows a head, 8 heads: 9.4 -> 6.3 us; beside the selections of four layers 12.5 -> 11.9).  With five to eight splits, two pieces a thread
// were slower (5 splits, three layers: 4.5 -> 5.4 us).
template <int D>
__device__ __forceinline__ void merge_rows_few_splits(const StepParams &p, size_t gid0, size_t stride)
{
    constexpr int SLABS = D / 8, MB = MERGE_FEW_SPLITS, ITEMS = MERGE_PIECES;
    const int BH = p.batch * p.hkv, Mtot = p.G * p.Bt, nblk = (Mtot + 31) / 32;
    const size_t rows = (size_t)BH * Mtot, pstride = (size_t)BH * nblk * SLABS * 64 * 4;
    float2 ml[ITEMS][MB];
    f16x4 o[ITEMS][MB];
    size_t row[ITEMS];
    int d0[ITEMS];
    bool there[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const size_t gid = gid0 + it * stride;
        const int L = (int)(gid % 64), slab = (int)((gid / 64) % SLABS);
        const size_t blkid = gid / (64 * SLABS);
        const int bh = (int)(blkid / nblk), m = (int)(blkid % nblk) * 32 + (L & 31);
        there[it] = blkid < (size_t)BH * nblk && m < Mtot;
        row[it] = (size_t)bh * Mtot + m;
        d0[it] = 8 * slab + 4 * (L >> 5);
        const _Float16 *pbase = p.part_o + gid * 4;   // ((block, slab, lane) in this order is what gid counts)
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const bool live = there[it] && i < p.splits;
            const f16x4 zero = {(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
            ml[it][i] = live ? p.part_ml[(size_t)i * rows + row[it]] : make_float2(-INFINITY, 0.f);
            o[it][i] = live ? *reinterpret_cast<const f16x4 *>(pbase + (size_t)i * pstride) : zero;
        }
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (!there[it]) continue;
        float mx = ml[it][0].x;
#pragma unroll
        for (int i = 1; i < MB; ++i) mx = fmaxf(mx, ml[it][i].x);
        float acc[4] = {0.f, 0.f, 0.f, 0.f}, Lsum = 0.f;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const float w = ml[it][i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[it][i].x - mx) * ml[it][i].y;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] += w * (float)o[it][i][r];
            Lsum += w;
        }
        const float inv = 1.f / Lsum;
        bf16x4 out;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = (__bf16)(acc[r] * inv);
        *reinterpret_cast<bf16x4 *>(p.out + row[it] * D + d0[it]) = out;
    }
}

// `thread` of `threads` that merge, each merge_pieces pieces
template <int D>
__device__ __forceinline__ void merge_thread(const StepParams &p, size_t thread, size_t threads)
{
    // (many splits first: a launch of a few workgroups lasts as long as its code and two trips take to arrive; 32 splits of 36 rows,
    // behind the other two 13.7 us, first 13.1)
    if (__builtin_expect(p.splits > 8, 1)) merge_rows<D>(p, thread);   // uniform
    else if (p.splits > MERGE_FEW_SPLITS) merge_rows<D, 8>(p, thread);
    else merge_rows_few_splits<D>(p, thread, threads);
}

// The merge of step_few's partials (float, [psplits][BH][G * Bt][D], each normalised by its row sum): workgroup
// `part` of `parts` of a head takes its share of the rows, a thread four output values and a share of the splits.  What bounds it is the
// trip to memory: the splits are dealt over the threads eight ways, so
// that 32 splits are one round of loads, not 32 loads in a row, and the shares are added up through LDS; and a compute unit takes in
// some 57 KB a microsecond, 4 rows of 128 in 32 splits are 64 KB: a workgroup a row ends with the eviction beside it (2.9 -> 2.4 us).
template <int D>
__device__ __forceinline__ void merge_few(const StepParams &p, float *lds, int bh, int part_, int parts)
{
    constexpr int MB = 8;                       // splits requested together
    constexpr int SHARES = 8;
    const int BH = p.batch * p.hkv, Mtot = p.G * p.Bt;
    const int m0 = part_ * Mtot / parts, rows = (part_ + 1) * Mtot / parts - m0;
    const int items = rows * (D / 4);           // at most POST_THREADS (32 rows of 128)
    const int shares = min(min(POST_THREADS / items, SHARES), p.splits);
    const int it = (int)threadIdx.x % items, share = (int)threadIdx.x / items;
    const float *part = reinterpret_cast<const float *>(p.part_o) + ((size_t)bh * Mtot + m0) * D + (size_t)it * 4;
    const float2 *mls = p.part_ml + (size_t)bh * Mtot + m0 + it / (D / 4);
    const size_t pstride = (size_t)BH * Mtot * D, mstride = (size_t)BH * Mtot;
    float mx = -INFINITY, Lsum = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (share < shares) {
        for (int s0 = share; s0 < p.splits; s0 += MB * shares) {
            float2 ml[MB];
            f32x4 o[MB];
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int s_ = s0 + i * shares;
                const bool live = s_ < p.splits;
                ml[i] = live ? mls[(size_t)s_ * mstride] : make_float2(-INFINITY, 0.f);
                o[i] = live ? *reinterpret_cast<const f32x4 *>(part + (size_t)s_ * pstride) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
            float bm = mx;
#pragma unroll
            for (int i = 0; i < MB; ++i) bm = fmaxf(bm, ml[i].x);
            const float down = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx - bm);
            mx = bm;
            Lsum *= down;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] *= down;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const float w = ml[i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[i].x - mx) * ml[i].y;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] += w * o[i][r];
                Lsum += w;
            }
        }
    }
    if (shares > 1) {   // uniform
        float *mine = lds + (size_t)threadIdx.x * 6;
        mine[0] = mx;
        mine[1] = Lsum;
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[2 + r] = acc[r];
        __syncthreads();
        if (share > 0) return;
        float bm = mx;
        for (int s_ = 1; s_ < shares; ++s_) bm = fmaxf(bm, lds[(size_t)(it + s_ * items) * 6]);
        const float down = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx - bm);
        Lsum *= down;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] *= down;
        for (int s_ = 1; s_ < shares; ++s_) {
            const float *o = lds + (size_t)(it + s_ * items) * 6;
            const float w = o[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(o[0] - bm);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] += w * o[2 + r];
            Lsum += w * o[1];
        }
    } else if (share > 0) {
        return;
    }
    const float inv = 1.f / Lsum;
    bf16x4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = (__bf16)(acc[r] * inv);
    *reinterpret_cast<bf16x4 *>(p.out + ((size_t)bh * Mtot + m0) * D + (size_t)it * 4) = o;
}

// The merge as a kernel of its own (a step whose eviction is deferred has nothing else to run
// here): small workgroups, so that the rows spread over every compute unit.
// Workgroup i takes head i % BH, like the workgroups of step_main: on a chip whose workgroups go
// round-robin over the XCDs the partials of a head are then read on the XCD that wrote them.
template <int D>
__device__ __forceinline__ void merge_body(const StepParams &p)
{
    const int BH = p.batch * p.hkv;
    const size_t per_head = (size_t)((p.G * p.Bt + 31) / 32) * (D / 8) * 64, threads = per_head / merge_pieces(p.splits);
    const int bh = blockIdx.x % BH;
    const size_t local = (size_t)(blockIdx.x / BH) * MERGE_THREADS + threadIdx.x;
    if (local < threads) merge_thread<D>(p, (size_t)bh * per_head + local, threads);
}
template <int D>
__global__ __launch_bounds__(MERGE_THREADS) void merge_kernel(StepParams p)
{
    merge_body<D>(p);
}
// ... of several layers, blockIdx.y each
template <int D>
__global__ __launch_bounds__(MERGE_THREADS) void merge_layers_kernel(LayerSteps steps)
{
    warm_arguments<sizeof(StepParams)>(blockIdx.y * (uint32_t)sizeof(StepParams));
    merge_body<D>(steps.p[blockIdx.y]);
}

// step_score: every workgroup scores SCORE_ROWS rows of one head.  The launch boundary after it
// makes the scores visible to step_post.
template <int D>
__global__ __launch_bounds__(SCORE_THREADS) void step_score_kernel(StepParams p)
{
    __shared__ ScoreShared sh;
    const int BH = p.batch * p.hkv;
    const int bh = blockIdx.x % BH, chunk = blockIdx.x / BH;
    const int row0 = chunk * SCORE_ROWS, row1 = min(p.n, row0 + SCORE_ROWS);
    score_rows<D>(p, sh, bh, row0, row1);
}

// step_post: workgroups [0, BH) select and compact one head each (when this step evicts); the
// rest merge the attention partials.  SRC: 16-byte loads of scores (and of positions) a thread of the
// selection holds in registers; 0: it reads them from memory where it needs them at all.
template <int D, int SRC, bool APPROX>
__device__ __forceinline__ void post_body(const StepParams &p, int block)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ PostShared sh;
    const int n_select = p.do_evict ? p.batch * p.hkv : 0;
    if (block >= n_select) {
#ifdef KD_TIMELINE
        const unsigned long long started = wall_clock64();
#endif
        static_assert(sizeof(PostShared) >= POST_THREADS * 6 * sizeof(float), "the merge of step_few's partials uses the selection's tables");
        const int BH = p.batch * p.hkv, i = block - n_select;
        // (behind the other merges: ahead of them a pass of blocks of 128 at 4096 keys took 3442 us, 3393 this way)
        if (__builtin_expect(p.few != 0, 0)) merge_few<D>(p, reinterpret_cast<float *>(&sh), i % BH, i / BH, p.merge_wgs / BH);
        else merge_thread<D>(p, (size_t)(block - n_select) * POST_THREADS + threadIdx.x, (size_t)p.merge_wgs * POST_THREADS);
#ifdef KD_TIMELINE
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        const unsigned long long ended = wall_clock64();
        if (p.timeline && threadIdx.x < 32) {   // record kind 4: merging workgroup
            const unsigned long long v = threadIdx.x == 0 ? started : threadIdx.x == 12 ? ended : threadIdx.x == 31 ? 4 : 0;
            p.timeline[(size_t)block * 32 + threadIdx.x] = v;
        }
#endif
        return;
    }
    select_and_compact<D, SRC, POST_THREADS, APPROX>(p, sh, smem_raw, block);
}
template <int D, int SRC, bool APPROX>
__global__ __launch_bounds__(POST_THREADS) void step_post_kernel(StepParams p)
{
    warm_arguments<sizeof(StepParams)>();
    post_body<D, SRC, APPROX>(p, (int)blockIdx.x);
}
// ... of several layers: blockIdx.x is the layer, so that the selections, which take longest, are dispatched first
template <int D, int SRC>
__global__ __launch_bounds__(POST_THREADS) void step_post_layers_kernel(LayerSteps steps)
{
    warm_arguments<sizeof(StepParams)>(blockIdx.x * (uint32_t)sizeof(StepParams));
    post_body<D, SRC, false>(steps.p[blockIdx.x], (int)blockIdx.y);
}

// ------------------------------------------------------------- selection and ordered compaction in one launch
// The shift behind a selection needs its bitmap and nothing else of it, and reading the rows, half of the shift's work, needs not
// even that.  So the two run in one launch: workgroup `index` behind the selections requests its rows into registers, merges its share of the
// attention partials, and waits for the bitmap of its head and for the chunks below it that its rows may land in; then it stores.  The grid is
// no larger than the chip.
// Who does what is dealt by tickets: the first workgroup of a head that starts selects, the ones after it take the chunks from the lowest up.  So
// a workgroup waits only for ones that have started, and those need nothing but their turn on the compute unit they hold -- whatever order the XCDs
// start workgroups in, and whatever other launches (other caches on other streams) hold or wait for the rest of the chip.  By block number instead,
// two such launches could each fill an XCD with workgroups that wait for one queued on the other's.  Workgroups [0, BH) expect the first ticket and
// begin the selection while it travels (PublishWords); the others merge before they draw, else they often are the first and select late
// (a step of 8192 rows 5 us longer).  Measured by block number / by tickets, us: 96 blocks of 128, 32 of which evict, 32 / 8 heads, 8192 rows
// 2549 / 2584;  96 blocks through three layers, 64 evict, 24 / 8 heads, 4096 rows 4564 / 4615.  Waits are bounded all the same: one that expires is reported in the status word, and its workgroup stores nothing.
// Thread: K rows in the first half of the workgroup, V rows in the second, TROWS rows apart.
// What bounds it: the selection up to its bitmap (8 us at 8320 rows), then one store of the rows, with the hint that nothing reads them
// again here (1.5 to 3 % of a step less than without).  The merge goes first: behind the requests of the rows, which hold registers, it
// took 1 % of a step more.  A step with both launches / with this one (roles by block number), us: 8 heads of 128, 32 query heads, blocks of 128, 2048 rows
// 31.8 / 29.9, 4096 40.7 / 35.9, 8192 54.9 / 43.1, 11000 68.0 / 53.8;  2 heads, 8192 rows 38.5 / 33.8;  8 of 64, two sequences, 4096 rows 39.4 / 33.1.
template <int D>
__device__ __forceinline__ void merge_around(const StepParams &p, const ShiftAround &sa, PostShared &sh, int index)
{
    constexpr int SLABS = D / 8;
    const int BH = p.batch * p.hkv;
    if (p.splits <= 1) return;   // uniform, like the branches below
    if (__builtin_expect(p.few != 0, 0)) {
        const int parts = min(p.merge_wgs / BH, sa.chunks);
        if (index / BH < parts) merge_few<D>(p, reinterpret_cast<float *>(&sh), index % BH, index / BH, parts);
    } else {
        // By the number of splits as in merge_thread, but four pieces a thread only where one each takes it more than two rounds.  Always with
        // the body for many splits / this way, us: 28 / 4 heads, four sequences, 1024 keys, blocks of 200 (three rounds) 46.0 / 39.0;  two layers of 24 / 8,
        // two sequences, 2048 keys, blocks of 256 63.6 / 59.0;  three of 32 / 8, 4096 keys 54.7 / 53.4;  two of 28 / 4, 8192 keys, blocks of 256 (two
        // rounds) 85.3 / 84.7, with four pieces 86.2.
        const size_t items = (size_t)BH * ((p.G * p.Bt + 31) / 32) * SLABS * 64, step = (size_t)BH * sa.chunks * POST_THREADS;
        const size_t first = (size_t)index * POST_THREADS + threadIdx.x;
        if (__builtin_expect(p.splits > 8, 1)) {
            for (size_t g = first; g < items; g += step) merge_rows<D>(p, g);
        } else if (p.splits > MERGE_FEW_SPLITS || items <= 2 * step) {
            for (size_t g = first; g < items; g += step) merge_rows<D, 8>(p, g);
        } else {
            for (size_t g = first; g < items / MERGE_PIECES; g += step) merge_rows_few_splits<D>(p, g, items / MERGE_PIECES);
        }
    }
}
template <int D>
__device__ __forceinline__ void shift_around(const StepParams &p, const ShiftAround &sa, PostShared &sh, int &go, int bh, int chunk)
{
    constexpr int UPR = D / 8, TROWS = POST_THREADS / 2 / UPR;
    const int tid = threadIdx.x, rows = sa.units * TROWS;
    const int row0 = chunk * rows + tid % (POST_THREADS / 2) / UPR;
    uint16_t *base = (tid >= POST_THREADS / 2 ? p.v : p.k) + (size_t)bh * p.cap * D + tid % UPR * 8;
    u32x4 val[AROUND_UNITS];
#pragma unroll
    for (int q = 0; q < AROUND_UNITS; ++q)
        if (q < sa.units) val[q] = *reinterpret_cast<const u32x4 *>(base + (size_t)min(row0 + q * TROWS, p.n - 1) * D);
    if (tid == 0) go = 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // every row of this chunk is in registers
    __syncthreads();
    int32_t *flags = sa.flags + (size_t)bh * sa.chunks;
    const unsigned long long *words = sa.words + (size_t)bh * sa.stride;
    if (tid == 0) __hip_atomic_store(&flags[chunk], sa.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto expired = [&]() {
        atomicOr(p.status, STATUS_ORDER_TIMEOUT);
        go = 0;
    };
    // the word of the epoch
    auto word_at = [&](int i) {
        for (int spins = 0; spins <= ORD_SPIN_LIMIT; ++spins) {
            const unsigned long long w = __hip_atomic_load(&words[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((int32_t)(w >> 32) == sa.epoch) return (uint32_t)w;
            __builtin_amdgcn_s_sleep(1);
        }
        expired();
        return 0u;
    };
    const int reach = (p.n - p.N + rows - 1) / rows, below = chunk - 1 - (tid - 64);   // chunks below this one its rows can land in
    if (tid == 0) {
        if (word_at(0) != 1) go = 0;
    } else if (tid >= 64 && tid < 64 + reach && below >= 0) {
        int spins = 0;
        while (__hip_atomic_load(&flags[below], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != sa.epoch) {
            if (++spins > ORD_SPIN_LIMIT) {
                expired();
                break;
            }
            __builtin_amdgcn_s_sleep(4);
        }
    }
    __syncthreads();
    if (go == 0) return;   // uniform: nothing to move, or a wait has expired
    __syncthreads();       // (everybody has looked, before a word that does not come changes it)
    const int nwords = (p.n + 31) / 32;
    uint32_t *bits = sh.hist, *before = sh.hist + MAX_CAP / 32;
    static_assert(2 * (MAX_CAP / 32) <= HIST_BINS && MAX_CAP / 32 <= POST_THREADS, "the bitmap and its counts use the histogram's place, a word a thread");
    const uint32_t w = tid < nwords ? word_at(1 + tid) : 0u;
    uint32_t total;
    const uint32_t at = block_exclusive_scan_t<POST_THREADS, uint32_t>((uint32_t)__popc(w), sh.wave_tot, &total);
    bits[tid] = w;
    before[tid] = at;
    __syncthreads();
    if (go == 0) return;   // uniform
#pragma unroll
    for (int q = 0; q < AROUND_UNITS; ++q) {
        const int row = row0 + q * TROWS;
        if (q < sa.units && row < p.n) {
            const uint32_t word = bits[row >> 5], bit = (uint32_t)row & 31u;
            const int to = row - (int)(before[row >> 5] + (uint32_t)__popc(word & ((1u << bit) - 1u)));
            if (((word >> bit) & 1u) == 0 && to != row) __builtin_nontemporal_store(val[q], reinterpret_cast<u32x4 *>(base + (size_t)to * D));
        }
    }
}
template <int D>
__device__ __forceinline__ void post_shift_body(const StepParams &p, const ShiftAround &sa, int block)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ PostShared sh;
    __shared__ uint32_t ticket;
    __shared__ int go;
    const int BH = p.batch * p.hkv, bh = block % BH;
    bool select = block < BH;   // uniform, like the branches below
    if (!select) merge_around<D>(p, sa, sh, block - BH);
    uint32_t drawn = 0;
    if (threadIdx.x == 0) drawn = draw_ticket(sa.tickets + (size_t)bh * TICKET_STRIDE);
    const PublishWords publish{sa, drawn, &ticket};
    if (!select) {
        publish.arrive();
        __syncthreads();
        select = publish.mine();
    }
    if (select) {
        select_and_compact<D, 3, POST_THREADS, false>(p, sh, smem_raw, bh, publish);
        if (publish.mine()) return;
    }
    if (ticket > (uint32_t)sa.chunks) {   // (impossible)
        if (threadIdx.x == 0) atomicOr(p.status, STATUS_ORDER_TIMEOUT);
        return;
    }
    shift_around<D>(p, sa, sh, go, bh, (int)ticket - 1);
}
template <int D>
__global__ __launch_bounds__(POST_THREADS) void step_post_shift_kernel(StepParams p, ShiftAround sa)
{
    warm_arguments<sizeof(StepParams) + sizeof(ShiftAround)>();
    post_shift_body<D>(p, sa, (int)blockIdx.x);
}
// ... of several layers: blockIdx.x is the layer
template <int D>
__global__ __launch_bounds__(POST_THREADS) void step_post_shift_layers_kernel(LayerSteps steps, ShiftArounds arounds)
{
    warm_arguments<sizeof(StepParams)>(blockIdx.x * (uint32_t)sizeof(StepParams));
    post_shift_body<D>(steps.p[blockIdx.x], arounds.s[blockIdx.x], (int)blockIdx.y);
}

// ------------------------------------------------------------- ordered compaction
// Stable in-place shift: kept row i moves to dst[i] = i - (evicted rows before i), so a row moves
// down by at most E = n - N rows.  One workgroup per ORD_ROWS rows reads its moving rows into
// registers, announces that (flag = epoch of this launch), waits until the workgroups whose rows
// it may overwrite -- the ceil(E / ORD_ROWS) chunks before it -- have announced the same, and
// stores.  The workgroups of a head take its chunks from the lowest up in the order in which they start (tickets, as above), so a
// workgroup only ever waits for ones that have started (by block number / by tickets, us a step: 32 / 8 heads of 128, 13000 rows 76.5 / 77.5;  two
// layers of 12288 115.5 / 118.2;  8 / 2 of 64, 16000 rows 40.8 / 42.6); the wait is bounded and reports a timeout in the status word instead of hanging.
// (Step: StepParams or ShiftStep)
template <int D, class Step>
__device__ __forceinline__ void shift_chunk(const Step &p, int BH, int32_t *flags, int nchunks, int32_t epoch, uint32_t *tickets, uint32_t first_ticket,
                                            int block)
{
    constexpr int UPR = D / 8;
    constexpr int UPT = ORD_ROWS * UPR * 2 / ORD_THREADS;   // 16-byte units (K and V) per thread
    static_assert(UPT * ORD_THREADS == ORD_ROWS * UPR * 2, "the chunk must divide over the threads");
    __shared__ uint32_t ticket;
    const int bh = block % BH, tid = threadIdx.x;
    if (tid == 0) ticket = draw_ticket(tickets + (size_t)bh * TICKET_STRIDE) - first_ticket;
    __syncthreads();
    if (ticket >= (uint32_t)nchunks) {   // (impossible)
        if (tid == 0) atomicOr(p.status, STATUS_ORDER_TIMEOUT);
        return;
    }
    const int chunk = (int)ticket;
    uint16_t *kb = p.k + (size_t)bh * p.cap * D;
    uint16_t *vb = p.v + (size_t)bh * p.cap * D;
    const int32_t *dst = p.dstmap + (size_t)bh * p.cap;
    const int r0 = chunk * ORD_ROWS;
    u32x4 val[UPT];
    int drow[UPT];
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
        const int w = q * ORD_THREADS + tid;
        const int which = w >= ORD_ROWS * UPR, rem = w - which * ORD_ROWS * UPR;
        const int row = r0 + rem / UPR, u = rem % UPR;
        // the row is requested together with its destination, not after it: one memory round trip
        // (rows that turn out to stay, or to be evicted, are the few ahead of the first eviction and
        // the evicted ones themselves)
        drow[q] = -1;
        val[q] = u32x4{0u, 0u, 0u, 0u};
        if (row < p.n) {
            val[q] = *reinterpret_cast<const u32x4 *>((which ? vb : kb) + (size_t)row * D + u * 8);
            const int d = dst[row];
            if (d >= 0 && d != row) drow[q] = d;
        }
    }
    __shared__ int go;
    if (tid == 0) go = 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // every row of this chunk is in registers
    __syncthreads();
    int32_t *myflags = flags + (size_t)bh * nchunks;
    if (tid == 0) __hip_atomic_store(&myflags[chunk], epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int reach = (p.n - p.N + ORD_ROWS - 1) / ORD_ROWS;   // chunks below this one its rows can land in
    if (tid < reach && chunk - 1 - tid >= 0) {
        int spins = 0;
        while (__hip_atomic_load(&myflags[chunk - 1 - tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch) {
            if (++spins > ORD_SPIN_LIMIT) {
                atomicOr(p.status, STATUS_ORDER_TIMEOUT);
                go = 0;   // rows that have not been read must not be stored over
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
    }
    __syncthreads();
    if (go == 0) return;   // uniform
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
        const int w = q * ORD_THREADS + tid;
        const int which = w >= ORD_ROWS * UPR, rem = w - which * ORD_ROWS * UPR;
        if (drow[q] >= 0)
            *reinterpret_cast<u32x4 *>((which ? vb : kb) + (size_t)drow[q] * D + (rem % UPR) * 8) = val[q];
    }
}

// One cache, by the parameters of its step.  (From a block of all the shift needs, 64 bytes, or from an array of them, the launch
// takes 0.4 to 1 us more: 16 of 8208 rows 11.9 us, 12.8 and 13.2; 9 of 10009 15.5 and 16.1.  Reading what the announcement needs
// ahead of the rows does not change that.)
template <int D>
__global__ __launch_bounds__(ORD_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) void compact_ordered_kernel(StepParams p, int32_t *flags, int nchunks, int32_t epoch, uint32_t *tickets, uint32_t first_ticket)
{
    shift_chunk<D>(p, p.batch * p.hkv, flags, nchunks, epoch, tickets, first_ticket, (int)blockIdx.x);
}
__host__ __device__ static inline int shift_chunks(const ShiftStep &sh) { return (sh.n + ORD_ROWS - 1) / ORD_ROWS; }
// ... of several caches, blockIdx.y each
template <int D>
__global__ __launch_bounds__(ORD_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) void compact_layers_kernel(ShiftSteps steps)
{
    const ShiftStep &p = steps.s[blockIdx.y];
    shift_chunk<D>(p, p.BH, p.flags, shift_chunks(p), p.epoch, p.tickets, p.first_ticket, (int)blockIdx.x);
}

// The merge of one cache's attention partials and the ordered shift of another cache in one launch
// (eviction deferred, ORDERED layout: the selection of the other cache rode in the attention launch
// just before, and its rows have no reader until that cache's next step).  The merge is a memory
// round trip on a chip it leaves mostly idle; the shift is bound by HBM traffic: together they take
// what the shift takes alone.  Workgroups [0, merge_wgs) merge -- they are dispatched first and
// the caller waits for their output -- the others shift one chunk each.
template <int D>
__global__ __launch_bounds__(ORD_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) void merge_shift_kernel(StepParams pm, ShiftStep shift, int merge_wgs)
{
    if ((int)blockIdx.x < merge_wgs) {
        // (few splits per round trip: the launch lasts as long as the shift does, and the registers
        // decide how many of its workgroups a compute unit holds)
        merge_rows<D, 4>(pm, (size_t)blockIdx.x * ORD_THREADS + threadIdx.x);
        return;
    }
    shift_chunk<D>(shift, shift.BH, shift.flags, shift_chunks(shift), shift.epoch, shift.tickets, shift.first_ticket, (int)blockIdx.x - merge_wgs);
}

// --------------------------------------------------- key sum from scratch (cache load)
// Column sums of CHUNK_ROWS rows in double; unit keys for anchor mode 1.
template <int D>
__global__ __launch_bounds__(256) void ksum_partial_kernel(StepParams p, double *partials, int nchunks)
{
    constexpr int UPR = D / 8;
    constexpr int RL = 256 / UPR;
    __shared__ double red[RL][D];
    const int bh = blockIdx.y, chunk = blockIdx.x;
    const int u = threadIdx.x % UPR, rl = threadIdx.x / UPR;
    const uint16_t *kb = p.k + (size_t)bh * p.cap * D;
    double acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
    const int r0 = chunk * CHUNK_ROWS;
    for (int r = rl; r < CHUNK_ROWS; r += RL) {
        const int row = r0 + r;
        double x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = 0.0;
        if (row < p.n) {
            const u32x4 w = *reinterpret_cast<const u32x4 *>(kb + (size_t)row * D + u * 8);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[2 * i] = bf16_lo(w[i]);
                x[2 * i + 1] = bf16_hi(w[i]);
            }
        }
        double inv = 1.0;
        if (p.anchor_mode == 1) {
            double k2 = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) k2 += x[i] * x[i];
#pragma unroll
            for (int m = 1; m < UPR; m <<= 1) k2 += shfl_xor_f64(k2, m);
            const double nk = sqrt(k2);
            inv = nk > 0.0 ? 1.0 / nk : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += (p.anchor_mode == 1) ? x[i] * inv : x[i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) red[rl][u * 8 + i] = acc[i];
    __syncthreads();
    if (threadIdx.x < D) {
        double s = 0.0;
        for (int r = 0; r < RL; ++r) s += red[r][threadIdx.x];
        partials[((size_t)bh * nchunks + chunk) * D + threadIdx.x] = s;
    }
}

// The sums of the chunks of a head: eight shares of the chunks side by side, each eight loads at a time (one thread a
// column that read them one after the other took 17.4 us for 64 chunks; now 3.9).
constexpr int KSUM_SHARES = 8;
__global__ __launch_bounds__(KSUM_SHARES * 128) void ksum_final_kernel(const double *partials, double *ksum, int nchunks, int D)
{
    __shared__ double part[KSUM_SHARES][128];
    const int bh = blockIdx.x, c = threadIdx.x % D, share = threadIdx.x / D;
    double s = 0.0;
#pragma unroll 8
    for (int k = share; k < nchunks; k += KSUM_SHARES) s += partials[((size_t)bh * nchunks + k) * D + c];
    part[share][c] = s;
    __syncthreads();
    if (share == 0) {
        for (int i = 1; i < KSUM_SHARES; ++i) s += part[i][c];
        ksum[(size_t)bh * D + c] = s;
    }
}

// ------------------------------------------------------------------ rotary embedding
// Fig. 1 step (1), the part of it that can live inside this boundary: the block's queries and keys
// arrive as the projections produced them and are rotated here, at the positions pos0 + j, into
// buffers the block step then reads.  Half-split pairing (i, i + D/2); cos and sin come from the
// caller's float tables [position][D/2]; x1 cos - x2 sin and x2 cos + x1 sin with every product and
// sum rounded to float on its own, then one rounding to bf16.
// rows: all (sequence, head) rows of q followed by those of k_new, Bt tokens each; a thread takes the
// 8 + 8 paired elements of one 16-byte unit of the first half.
// blockIdx.y: the layer (a call through several layers rotates the blocks of all of them in one launch: with one launch a
// layer the rotation of a 128-token block, 24 / 8 heads, took 3.7 us of kernel and a launch of its own in every layer).
template <int D>
__global__ __launch_bounds__(256) void rope_kernel(RopeBatch in, const float *cos_t, const float *sin_t, int q_rows, int k_rows,
                                                   int Bt, int32_t pos0)
{
    const uint16_t *q = in.q[blockIdx.y], *k = in.k[blockIdx.y];
    uint16_t *q_rot = in.q_rot[blockIdx.y], *k_rot = in.k_rot[blockIdx.y];
    constexpr int UPH = D / 16;   // 16-byte units per half row
    const size_t gid = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t row = gid / UPH;
    const int unit = (int)(gid % UPH);
    if (row >= (size_t)q_rows + k_rows) return;
    const bool isk = row >= (size_t)q_rows;
    const size_t r = isk ? row - q_rows : row;
    const uint16_t *src = (isk ? k : q) + r * D;
    uint16_t *dst = (isk ? k_rot : q_rot) + r * D;
    const int j = (int)(r % Bt);
    const float *cs = cos_t + ((size_t)pos0 + j) * (D / 2) + unit * 8;
    const float *sn = sin_t + ((size_t)pos0 + j) * (D / 2) + unit * 8;
    const u32x4 a = *reinterpret_cast<const u32x4 *>(src + unit * 8);           // x1: elements 8 unit .. + 7
    const u32x4 b = *reinterpret_cast<const u32x4 *>(src + D / 2 + unit * 8);   // x2: the paired elements
    const f32x4 c0 = *reinterpret_cast<const f32x4 *>(cs), c1 = *reinterpret_cast<const f32x4 *>(cs + 4);
    const f32x4 s0 = *reinterpret_cast<const f32x4 *>(sn), s1 = *reinterpret_cast<const f32x4 *>(sn + 4);
    u32x4 o1, o2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float y1[2], y2[2];
#pragma unroll
        for (int hw = 0; hw < 2; ++hw) {
            const float x1 = __uint_as_float(hw ? (a[i] & 0xFFFF0000u) : (a[i] << 16));
            const float x2 = __uint_as_float(hw ? (b[i] & 0xFFFF0000u) : (b[i] << 16));
            const int e = 2 * i + hw;
            const float c = e < 4 ? c0[e] : c1[e - 4], sgn = e < 4 ? s0[e] : s1[e - 4];
            y1[hw] = __fsub_rn(__fmul_rn(x1, c), __fmul_rn(x2, sgn));
            y2[hw] = __fadd_rn(__fmul_rn(x2, c), __fmul_rn(x1, sgn));
        }
        const __bf16 l1 = (__bf16)y1[0], h1 = (__bf16)y1[1], l2 = (__bf16)y2[0], h2 = (__bf16)y2[1];
        o1[i] = (uint32_t)__builtin_bit_cast(uint16_t, l1) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
        o2[i] = (uint32_t)__builtin_bit_cast(uint16_t, l2) | ((uint32_t)__builtin_bit_cast(uint16_t, h2) << 16);
    }
    *reinterpret_cast<u32x4 *>(dst + unit * 8) = o1;
    *reinterpret_cast<u32x4 *>(dst + D / 2 + unit * 8) = o2;
}

// ------------------------------------------------------------------ small helpers
__global__ void zero_words_kernel(int32_t *p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

// rows [BH][len][D] (dense) -> cache rows [BH][cap][D]
__global__ void load_rows_kernel(const uint16_t *src, uint16_t *dst, int cap, int D, int len)
{
    const int bh = blockIdx.y;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // 16-byte unit within the head
    const size_t units = (size_t)len * (D / 8);
    if (i < units)
        *reinterpret_cast<u32x4 *>(dst + (size_t)bh * cap * D + i * 8) =
            *reinterpret_cast<const u32x4 *>(src + (size_t)bh * len * D + i * 8);
}

// int32 [BH][len] dense <-> [BH][cap] strided
__global__ void load_pos_kernel(const int32_t *src, int32_t *dst, int cap, int len, int to_cache)
{
    const int bh = blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < len) {
        if (to_cache) dst[(size_t)bh * cap + i] = src[(size_t)bh * len + i];
        else dst[(size_t)bh * len + i] = src[(size_t)bh * cap + i];
    }
}

// ---------------------------------------------------------------------- launchers
constexpr size_t LISTS_LDS_MAX = 48 * 1024;

// A compute unit shifts the rows of a head at some 100 GB/s; a launch of its own with the rows spread over the chip costs 3 us and
// its gap.  Measured, us a step with the shift apart / inside the selection (4 / 1 heads of 64, 8 / 2 of 64 and 24 / 8 of 128):
// 128 rows 16.0 / 14.6, 16.5 / 14.7, 17.4 / 15.4;  288 rows 16.4 / 14.7, 16.7 / 14.9, 18.3 / 16.7;  512 rows 16.5 / 15.3,
// 17.1 / 15.5, 18.2 / 17.9;  544 rows 17.9 / 16.6, 18.1 / 16.9, 19.6 / 20.1;  1024 rows 17.1 / 17.5, 17.6 / 17.7, 19.2 / 22.8.
constexpr int SHIFT_HERE_MAX = 48 * 1024;   // elements of a head's K
bool shift_fits_selection(const StepParams &p) { return (long)p.n * p.D <= SHIFT_HERE_MAX; }
static_assert(SHIFT_HERE_MAX / 64 <= 3 * 4 * POST_THREADS, "the selection holds the scores and positions of such a cache in registers");

bool lists_fit_lds(int n, int N) { return n > N && (size_t)(n - N) * 4 <= LISTS_LDS_MAX; }

// dynamic LDS a step_post launch may ask for next to its static tables (160 KB per compute unit)
constexpr size_t POST_DYN_MAX = 64 * 1024;

hipError_t configure_main_kernels();
hipError_t configure_few_kernels();

hipError_t configure_kernels()
{
    hipError_t e = configure_main_kernels();
    if (e != hipSuccess) return e;
    e = configure_few_kernels();
    if (e != hipSuccess) return e;
    static_assert(MAX_CAP / 8 + LISTS_LDS_MAX + 16 <= POST_DYN_MAX, "the non-resident selection always fits");
    const void *post_fns[] = {
#define KD_FN(DD, SRC)                                                           \
    reinterpret_cast<const void *>(step_post_kernel<DD, SRC, false>),             \
        reinterpret_cast<const void *>(step_post_layers_kernel<DD, SRC>)
#define KD_FNS(DD)                                                               \
    KD_FN(DD, 0), KD_FN(DD, 3), KD_FN(DD, 5), reinterpret_cast<const void *>(step_post_kernel<DD, 0, true>), \
        reinterpret_cast<const void *>(step_post_kernel<DD, 3, true>)
        KD_FNS(128), KD_FNS(64),
        reinterpret_cast<const void *>(step_post_shift_kernel<128>), reinterpret_cast<const void *>(step_post_shift_layers_kernel<128>),
        reinterpret_cast<const void *>(step_post_shift_kernel<64>), reinterpret_cast<const void *>(step_post_shift_layers_kernel<64>)};
#undef KD_FNS
#undef KD_FN
    for (const void *fn : post_fns) {
        e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)POST_DYN_MAX);
        if (e != hipSuccess) return e;
    }
    return e;
}

hipError_t launch_step_score(const StepParams &p, hipStream_t s)
{
    const int grid = p.batch * p.hkv * ((p.n + SCORE_ROWS - 1) / SCORE_ROWS);
    if (p.D == 128) hipLaunchKernelGGL((step_score_kernel<128>), dim3(grid), dim3(SCORE_THREADS), 0, s, p);
    else if (p.D == 64) hipLaunchKernelGGL((step_score_kernel<64>), dim3(grid), dim3(SCORE_THREADS), 0, s, p);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// Three 16-byte loads of scores and of positions a thread up to 12288 rows, five of scores alone up to 20480 (a pass that
// needs every row's position reads those from memory); the registers hold no more beside the rows that may move, so
// larger caches are read from memory in every pass (with approximate scores, whose exact ones take registers, beyond 12288 rows).  With the arg-max records of the attention launch the scores are hardly
// ever looked at.
static int post_source(const StepParams &p)
{
    return p.argmax_rec || p.n > (p.score_approx ? 3 : 5) * 4 * POST_THREADS ? 0 : p.n <= 3 * 4 * POST_THREADS ? 3 : 5;
}

hipError_t launch_step_post(const StepParams &p, hipStream_t s)
{
    const int grid = (p.do_evict ? p.batch * p.hkv : 0) + p.merge_wgs;
    if (grid == 0) return hipSuccess;
    if (!p.do_evict && p.few) {
        if (p.D == 128) hipLaunchKernelGGL((step_post_kernel<128, 0, false>), dim3(grid), dim3(POST_THREADS), 0, s, p);
        else if (p.D == 64) hipLaunchKernelGGL((step_post_kernel<64, 0, false>), dim3(grid), dim3(POST_THREADS), 0, s, p);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (!p.do_evict) {   // merge only
        const size_t per_head = (size_t)((p.G * p.Bt + 31) / 32) * (p.D / 8) * 64 / merge_pieces(p.splits);
        const int mgrid = p.batch * p.hkv * (int)((per_head + MERGE_THREADS - 1) / MERGE_THREADS);
        if (p.D == 128) hipLaunchKernelGGL((merge_kernel<128>), dim3(mgrid), dim3(MERGE_THREADS), 0, s, p);
        else if (p.D == 64) hipLaunchKernelGGL((merge_kernel<64>), dim3(mgrid), dim3(MERGE_THREADS), 0, s, p);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (p.n > 32 * POST_THREADS) return hipErrorInvalidValue;   // a thread owns one word of the eviction bitmap
    const int src = post_source(p);
    const size_t lds = select_dyn_bytes(p.n, p.N, p.cap, p.lists_in_lds != 0, false);
#define KD_GO2(DD, SRC)                                                                                                    \
    if (p.score_approx) hipLaunchKernelGGL((step_post_kernel<DD, SRC, true>), dim3(grid), dim3(POST_THREADS), lds, s, p);   \
    else hipLaunchKernelGGL((step_post_kernel<DD, SRC, false>), dim3(grid), dim3(POST_THREADS), lds, s, p);
#define KD_GO(DD)                       \
    if (src == 0) { KD_GO2(DD, 0) }      \
    else if (src == 3) { KD_GO2(DD, 3) } \
    else hipLaunchKernelGGL((step_post_kernel<DD, 5, false>), dim3(grid), dim3(POST_THREADS), lds, s, p);
    if (p.D == 128) { KD_GO(128) }
    else if (p.D == 64) { KD_GO(64) }
#undef KD_GO
#undef KD_GO2
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_step_post_layers(const LayerSteps &steps, int layers, hipStream_t s)
{
    const StepParams &p = steps.p[0];
    if (layers < 2 || layers > GROUP_LAYERS || p.few || p.argmax_rec || p.score_approx) return hipErrorInvalidValue;
    const int per_layer = (p.do_evict ? p.batch * p.hkv : 0) + p.merge_wgs;
    if (per_layer == 0) return hipSuccess;
    if (!p.do_evict) {
        const size_t per_head = (size_t)((p.G * p.Bt + 31) / 32) * (p.D / 8) * 64 / merge_pieces(p.splits);
        const dim3 grid((unsigned)(p.batch * p.hkv * ((per_head + MERGE_THREADS - 1) / MERGE_THREADS)), (unsigned)layers);
        if (p.D == 128) hipLaunchKernelGGL((merge_layers_kernel<128>), grid, dim3(MERGE_THREADS), 0, s, steps);
        else if (p.D == 64) hipLaunchKernelGGL((merge_layers_kernel<64>), grid, dim3(MERGE_THREADS), 0, s, steps);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (p.n > 32 * POST_THREADS) return hipErrorInvalidValue;
    const int src = post_source(p);
    const size_t lds = select_dyn_bytes(p.n, p.N, p.cap, p.lists_in_lds != 0, false);
    const dim3 grid((unsigned)layers, (unsigned)per_layer);
#define KD_GO(DD)                                                                                                          \
    if (src == 0) hipLaunchKernelGGL((step_post_layers_kernel<DD, 0>), grid, dim3(POST_THREADS), lds, s, steps);             \
    else if (src == 3) hipLaunchKernelGGL((step_post_layers_kernel<DD, 3>), grid, dim3(POST_THREADS), lds, s, steps);        \
    else hipLaunchKernelGGL((step_post_layers_kernel<DD, 5>), grid, dim3(POST_THREADS), lds, s, steps);
    if (p.D == 128) { KD_GO(128) }
    else if (p.D == 64) { KD_GO(64) }
#undef KD_GO
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// The fewest units a thread with which selections and chunks are on the chip together, one workgroup a compute unit (their registers hold
// no second one): the more compute units take part, the sooner the rows are read and stored.
bool plan_shift_around(const StepParams &p, int layers, int cus, int32_t *units, int32_t *chunks)
{
    if (!p.do_evict || p.score_approx || post_source(p) != 3) return false;
    const int BH = p.batch * p.hkv;
    for (int u = 1; u <= AROUND_UNITS; ++u) {
        const int rows = u * (POST_THREADS / 2 / (p.D / 8)), n = (p.n + rows - 1) / rows;
        static_assert(POST_THREADS / 2 / (128 / 8) >= ORD_MIN_ROWS, "one flag for every chunk");
        if (layers * BH * (n + 1) > cus || (p.n - p.N + rows - 1) / rows > POST_THREADS - 64) continue;
        *units = u;
        *chunks = n;
        return true;
    }
    return false;
}

hipError_t launch_step_post_shift(const StepParams &p, const ShiftAround &around, hipStream_t s)
{
    const dim3 grid((unsigned)(p.batch * p.hkv * (1 + around.chunks)));
    const size_t lds = select_dyn_bytes(p.n, p.N, p.cap, p.lists_in_lds != 0, false);
    if (!p.do_evict || p.score_approx || post_source(p) != 3 || around.units < 1 || around.units > AROUND_UNITS) return hipErrorInvalidValue;
    if (p.D == 128) hipLaunchKernelGGL((step_post_shift_kernel<128>), grid, dim3(POST_THREADS), lds, s, p, around);
    else if (p.D == 64) hipLaunchKernelGGL((step_post_shift_kernel<64>), grid, dim3(POST_THREADS), lds, s, p, around);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_step_post_shift_layers(const LayerSteps &steps, const ShiftArounds &arounds, int layers, hipStream_t s)
{
    const StepParams &p = steps.p[0];
    const ShiftAround &a = arounds.s[0];
    if (layers < 2 || layers > GROUP_LAYERS || !p.do_evict || p.score_approx || post_source(p) != 3 || a.units < 1 || a.units > AROUND_UNITS)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)layers, (unsigned)(p.batch * p.hkv * (1 + a.chunks)));
    const size_t lds = select_dyn_bytes(p.n, p.N, p.cap, p.lists_in_lds != 0, false);
    if (p.D == 128) hipLaunchKernelGGL((step_post_shift_layers_kernel<128>), grid, dim3(POST_THREADS), lds, s, steps, arounds);
    else if (p.D == 64) hipLaunchKernelGGL((step_post_shift_layers_kernel<64>), grid, dim3(POST_THREADS), lds, s, steps, arounds);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// one waiting thread per chunk in reach
static bool shift_fits(const ShiftStep &sh) { return sh.n - sh.N <= ORD_THREADS * ORD_ROWS; }

hipError_t launch_compact_ordered(const StepParams &p, const ShiftStep &shift, hipStream_t s)
{
    if (!shift_fits(shift)) return hipErrorInvalidValue;
    const int chunks = shift_chunks(shift);
    const dim3 grid((unsigned)(shift.BH * chunks));
    if (p.D == 128) hipLaunchKernelGGL((compact_ordered_kernel<128>), grid, dim3(ORD_THREADS), 0, s, p, shift.flags, chunks, shift.epoch, shift.tickets, shift.first_ticket);
    else if (p.D == 64) hipLaunchKernelGGL((compact_ordered_kernel<64>), grid, dim3(ORD_THREADS), 0, s, p, shift.flags, chunks, shift.epoch, shift.tickets, shift.first_ticket);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_compact_layers(const ShiftSteps &steps, int layers, int D, hipStream_t s)
{
    if (layers < 2 || layers > GROUP_LAYERS || !shift_fits(steps.s[0])) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(steps.s[0].BH * shift_chunks(steps.s[0])), (unsigned)layers);
    if (D == 128) hipLaunchKernelGGL((compact_layers_kernel<128>), grid, dim3(ORD_THREADS), 0, s, steps);
    else if (D == 64) hipLaunchKernelGGL((compact_layers_kernel<64>), grid, dim3(ORD_THREADS), 0, s, steps);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// pm: the step whose partials are merged; shift: the other cache's
hipError_t launch_merge_shift(const StepParams &pm, const ShiftStep &shift, hipStream_t s)
{
    const size_t merge_threads = (size_t)pm.batch * pm.hkv * ((pm.G * pm.Bt + 31) / 32) * (pm.D / 8) * 64;
    const int mw = (int)((merge_threads + ORD_THREADS - 1) / ORD_THREADS);
    const int grid = mw + shift.BH * shift_chunks(shift);
    if (!shift_fits(shift) || pm.splits < 2 || pm.few) return hipErrorInvalidValue;
    if (pm.D == 128) hipLaunchKernelGGL((merge_shift_kernel<128>), dim3(grid), dim3(ORD_THREADS), 0, s, pm, shift, mw);
    else if (pm.D == 64) hipLaunchKernelGGL((merge_shift_kernel<64>), dim3(grid), dim3(ORD_THREADS), 0, s, pm, shift, mw);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_ksum_rebuild(const StepParams &p, double *partials, hipStream_t s)
{
    const int BH = p.batch * p.hkv;
    if (p.n == 0) return launch_zero_words(reinterpret_cast<int32_t *>(const_cast<double *>(p.ksum)), (size_t)BH * p.D * 2, s);
    const int nchunks = (p.n + CHUNK_ROWS - 1) / CHUNK_ROWS;
    dim3 grid(nchunks, BH);
    if (p.D == 128) hipLaunchKernelGGL((ksum_partial_kernel<128>), grid, dim3(256), 0, s, p, partials, nchunks);
    else if (p.D == 64) hipLaunchKernelGGL((ksum_partial_kernel<64>), grid, dim3(256), 0, s, p, partials, nchunks);
    else return hipErrorInvalidValue;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ksum_final_kernel, dim3(BH), dim3(KSUM_SHARES * p.D), 0, s, partials, const_cast<double *>(p.ksum), nchunks, p.D);
    return hipGetLastError();
}

hipError_t launch_rope(const RopeBatch &b, const float *cos_t, const float *sin_t, int q_rows, int k_rows, int Bt, int D,
                       int32_t pos0, hipStream_t s)
{
    if (b.layers < 1 || b.layers > ROPE_LAYERS) return hipErrorInvalidValue;
    const size_t threads = ((size_t)q_rows + k_rows) * (D / 16);
    const dim3 grid((unsigned)((threads + 255) / 256), (unsigned)b.layers);
    if (D == 128) hipLaunchKernelGGL((rope_kernel<128>), grid, dim3(256), 0, s, b, cos_t, sin_t, q_rows, k_rows, Bt, pos0);
    else if (D == 64) hipLaunchKernelGGL((rope_kernel<64>), grid, dim3(256), 0, s, b, cos_t, sin_t, q_rows, k_rows, Bt, pos0);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_zero_words(int32_t *ptr, size_t nwords, hipStream_t s)
{
    if (nwords == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, s, ptr, nwords);
    return hipGetLastError();
}

hipError_t launch_load_rows(const uint16_t *src, uint16_t *dst, int BH, int cap, int D, int len, hipStream_t s)
{
    if (len == 0) return hipSuccess;
    const size_t units = (size_t)len * (D / 8);
    hipLaunchKernelGGL(load_rows_kernel, dim3((unsigned)((units + 255) / 256), BH), dim3(256), 0, s, src, dst,
                       cap, D, len);
    return hipGetLastError();
}

hipError_t launch_load_pos(const int32_t *src, int32_t *dst, int BH, int cap, int len, int to_cache,
                           hipStream_t s)
{
    if (len == 0) return hipSuccess;
    hipLaunchKernelGGL(load_pos_kernel, dim3((len + 255) / 256, BH), dim3(256), 0, s, src, dst, cap, len,
                       to_cache);
    return hipGetLastError();
}

}  // namespace kd
