// step_few: the attention launch of a block step whose KV heads have few query rows (G * Bt <= 32: the
// generation phase above all) and enough keys for it to pay (the plan has the rule and both sides' times).  Same work as step_main -- append (Eq. 5), block attention over cache ||
// block (Eq. 1-2), anchor and cosine score of every key -- cut for a step that is bound by reading the
// cache once, not by the matrix cores.
//
// What bounds it: the stream of K and V from HBM (4 D bytes per key and KV head).  step_main puts 256
// query rows on a workgroup and shares every key tile among its waves, a barrier per tile; with 4 rows
// that leaves two waves doing all the attention for 32 columns of which 4 exist.  Here a wave is on its
// own: it takes 32 keys at a time (tiles interleaved over the eight waves, so a workgroup still reads a
// contiguous range), holds 16 query rows (16x16x32 MFMA; more than 16 rows take a second workgroup on the same
// keys), keeps its own maximum, row
// sum and output, and scores its keys from the registers they arrived in.  No barrier inside the loop;
// the next tile's K and V are in flight (16 KB per wave, 128 KB per compute unit) while one is worked on.
// The eight results are merged through LDS once at the end, and the key ranges of different workgroups by
// step_post from float partials.  Measured per step against step_main with two waves sharing the key tiles
// (attention + merge and selection, 32 / 8 heads, N = 8192): one sequence 14.3 + 22.9 -> 15.0 + 4.0 us,
// sixteen sequences 106.9 + 6.9 -> 98 + 4.8 us (537 MB: 5.5 TB/s).  By the stamps of one sequence the
// anchor is formed 4.2 us after the launch began (5.9 behind barriers for which every wave had to have requested its tiles), the tiles are done
// at 6.3 (8.1) and the partials stored at 9.0 (10.5); of the chain behind the data the arg-max (six exchanges of 64-bit pairs through LDS, then
// one thread over eight records) took 2 us more once: it is the work of one wave that has nothing to merge, on the vector ALU.
//
//   S^T = K Q^T  A = K rows, loaded straight from memory in operand layout (lane: row l % 16, 16 bytes at
//                32 c + 8 (l / 16): 64 contiguous bytes per row and instruction); B = Q^T (registers)
//   O^T = V^T P^T  V goes through a wave-private piece of LDS: written as rows, read back with the
//                transposing ds_read_b64_tr_b16; B = P^T straight from the accumulators: the 32 keys are
//                enumerated in accumulator order (k-slot 8 g + i of lane group g is key 4 g + i for i < 4
//                and 16 + 4 g + i - 4 otherwise), and the two transposing reads fetch exactly those.
#include "kd_kernels.h"
#include "kd_device.h"
#include "kd_select.h"

namespace kd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int FEW_WAVES = 8;
constexpr float FEW_RESCALE_SLACK = 64.f;   // the reference maximum may lag by 2^64, as in step_main

template <int D>
constexpr size_t few_lds_bytes()
{
    // V tiles of the waves, and their outputs (float, 16 rows each) in a place of their own: a wave that is done waits for no other's V
    return (size_t)FEW_WAVES * FEW_KEYS * D * 2 + (size_t)FEW_WAVES * 16 * D * 4;
}

// max over the four 16-lane rows of a wave, position by position (every lane gets it)
__device__ __forceinline__ float max_over_rows(float x)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Two quantities reduced over a pair of lane halves (H32: lanes i and i ^ 32) or of 16-lane rows (lanes i
// and i ^ 16) with one addition: the even side ends with the sum of x, the odd side with the sum of y.
template <bool H32>
__device__ __forceinline__ double pair_split_f64(double x, double y)
{
    const uint32_t xl = (uint32_t)__double2loint(x), xh = (uint32_t)__double2hiint(x);
    const uint32_t yl = (uint32_t)__double2loint(y), yh = (uint32_t)__double2hiint(y);
    const auto l = H32 ? __builtin_amdgcn_permlane32_swap(xl, yl, false, false)
                       : __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto h = H32 ? __builtin_amdgcn_permlane32_swap(xh, yh, false, false)
                       : __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

// Arg-max over a wave of (orderable score bits << 32 | row) with a tie flag: every lane gets the record with the largest score bits
// and whether another one has them too (or the winner's own flag is set).  0: no row.  On the vector ALU alone.
__device__ __forceinline__ void wave_argmax(unsigned long long &best, bool &tie)
{
    const uint32_t hi = (uint32_t)(best >> 32);
    uint32_t m = hi;   // maximum of the lanes below and this one, as in wave_inclusive_scan; lane 63: of all
    m = max(m, dpp_fetch<0x111, 0xF>(m));
    m = max(m, dpp_fetch<0x112, 0xF>(m));
    m = max(m, dpp_fetch<0x114, 0xF>(m));
    m = max(m, dpp_fetch<0x118, 0xF>(m));
    m = max(m, dpp_fetch<0x142, 0xA>(m));
    m = max(m, dpp_fetch<0x143, 0xC>(m));
    m = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    const uint64_t with = __builtin_amdgcn_ballot_w64(hi == m);   // (of 64 lanes without a row: all, with m == 0)
    const int first = __builtin_ctzll(with);
    const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, first);
    tie = m != 0 && (__popcll(with) > 1 || __builtin_amdgcn_ballot_w64(hi == m && tie) != 0);
    best = ((unsigned long long)m << 32) | row;
}

// STREAM: the cached rows are read with the non-temporal hint (see launch_step_few)
template <int D, bool STREAM>
__global__ __launch_bounds__(64 * FEW_WAVES) void step_few_kernel(StepParams p)
{
    warm_arguments<sizeof(StepParams)>();
    constexpr int NW = FEW_WAVES, NT = 64 * NW;
    constexpr int UPR = D / 8;                 // 16-byte units per row
    constexpr int NC = D / 32;                 // k-chunks of the first product
    constexpr int NDB = D / 16;                // 16-wide d blocks of the output
    constexpr int ROWB = D * 2;
    constexpr int RPL = 64 / UPR;              // rows a wave-wide 16-byte load covers
    constexpr int NV = FEW_KEYS / RPL;         // ... loads per V tile
    constexpr int VSW = UPR / 4;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ double bs_part[NW][D];
    __shared__ double mu_s[D], mu_w[NW][D];
    __shared__ double red[D / 16];
    __shared__ float2 ml_s[NW][16];
    __shared__ unsigned long long rec_s[NW][64];   // every lane's best row, its tie flag in bit 31

    KD_TL_DECL
    KD_TL(0);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, g = lane >> 4;
    const int BH = p.batch * p.hkv;
    const int bh = (int)blockIdx.x % BH, mt = (int)blockIdx.x / BH % p.mtiles, sp = (int)blockIdx.x / BH / p.mtiles;
    const int Mtot = p.G * p.Bt;
    const int m0 = 16 * mt, mrows = min(16, Mtot - m0);   // this workgroup's query rows
    const int nt = (p.n + FEW_KEYS - 1) / FEW_KEYS;
    const int t0 = (int)((long)sp * nt / p.splits), t1 = (int)((long)(sp + 1) * nt / p.splits);

    const uint16_t *kcache = p.k + (size_t)bh * p.cap * D;
    const uint16_t *vcache = p.v + (size_t)bh * p.cap * D;
    const uint16_t *knew = p.k_new + (size_t)bh * p.Bt * D;
    const uint16_t *vnew = p.v_new + (size_t)bh * p.Bt * D;

    auto ld = [](const uint16_t *g) -> u32x4 {
        if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(g));
        else return *reinterpret_cast<const u32x4 *>(g);
    };
    // ---- requested first, because loads return in order and the anchor's chain is the longest: the first
    // block row of this thread, the key sum, and this workgroup's slice of the rows to append (Eq. 5; the
    // rows are stored at once: nothing in this launch reads a cache row from len on)
    const bool writer = sp == 0 && mt == 0;
    const bool scoring = p.do_score != 0 && mt == 0;   // one of the workgroups that share a key range scores it
    const bool need_sum = scoring || writer;
    const int bu = tid % UPR, brl = tid / UPR;
    // One token and the plain anchor: every wave forms the anchor by itself, columns lane and lane + 64, in the arithmetic of the general way.
    // Nothing waits for the other waves, which are still requesting their tiles (two barriers there ended 5.9 us after the launch began).
    const bool alone = p.Bt == 1 && p.anchor_mode == 0;   // uniform
    constexpr int WC = D / 64;   // columns a lane
    u32x4 brow = {0u, 0u, 0u, 0u};
    double ksum_before = 0.0, wsum[WC];
    uint16_t wkey[WC];
    if (alone) {
#pragma unroll
        for (int i = 0; i < WC; ++i) {
            wkey[i] = knew[lane + 64 * i];
            wsum[i] = p.ksum[(size_t)bh * D + lane + 64 * i];
        }
    } else if (need_sum) {
        if (brl < p.Bt) brow = *reinterpret_cast<const u32x4 *>(knew + (size_t)brl * D + bu * 8);
        if (tid < D) ksum_before = p.ksum[(size_t)bh * D + tid];
    }
    {
        const int W = p.splits * p.mtiles, w = sp * p.mtiles + mt;
        const int j0 = (int)((long)w * p.Bt / W), j1 = (int)((long)(w + 1) * p.Bt / W);
        for (int u = tid; u < (j1 - j0) * UPR * 2; u += NT) {
            const int which = u >= (j1 - j0) * UPR, rem = u - which * (j1 - j0) * UPR;
            const int j = j0 + rem / UPR, unit = rem % UPR;
            *reinterpret_cast<u32x4 *>((which ? p.v : p.k) + ((size_t)bh * p.cap + p.len + j) * D + unit * 8) =
                *reinterpret_cast<const u32x4 *>((which ? vnew : knew) + (size_t)j * D + unit * 8);
        }
        for (int j = j0 + tid; j < j1; j += NT) p.pos[(size_t)bh * p.cap + p.len + j] = p.pos0 + j;
    }

    // ---- loads of one tile.  Rows past n repeat row n - 1 (finite data whose weights are masked to zero).
    auto load_k = [&](int t, u32x4 (&kr)[2][NC]) {
        const int r0 = t * FEW_KEYS;
        if (r0 + FEW_KEYS <= p.len) {   // uniform: every row is a cached one
            const uint16_t *kb = kcache + (size_t)r0 * D + (size_t)c16 * D + 8 * g;
#pragma unroll
            for (int kg = 0; kg < 2; ++kg)
#pragma unroll
                for (int c = 0; c < NC; ++c) kr[kg][c] = ld(kb + kg * 16 * D + c * 32);
        } else {
#pragma unroll
            for (int kg = 0; kg < 2; ++kg) {
                const int r = min(r0 + 16 * kg + c16, p.n - 1);
                const uint16_t *kb = (r < p.len ? kcache + (size_t)r * D : knew + (size_t)(r - p.len) * D) + 8 * g;
#pragma unroll
                for (int c = 0; c < NC; ++c) kr[kg][c] = *reinterpret_cast<const u32x4 *>(kb + c * 32);
            }
        }
    };
    auto load_v = [&](int t, u32x4 (&vr)[NV]) {
        const int r0 = t * FEW_KEYS;
        if (r0 + FEW_KEYS <= p.len) {
            const uint16_t *vb = vcache + (size_t)r0 * D + (size_t)lane * 8;
#pragma unroll
            for (int i = 0; i < NV; ++i) vr[i] = ld(vb + i * 64 * 8);
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int r = min(r0 + i * RPL + lane / UPR, p.n - 1);
                const uint16_t *vb = r < p.len ? vcache + (size_t)r * D : vnew + (size_t)(r - p.len) * D;
                vr[i] = *reinterpret_cast<const u32x4 *>(vb + (lane % UPR) * 8);
            }
        }
    };
    // K is requested two tiles ahead (two sets of registers; a set is requested again as soon as its tile has been
    // scored), V one tile ahead.
    u32x4 ka[2][NC], kb2[2][NC], vr[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) vr[i] = u32x4{0u, 0u, 0u, 0u};
    int t = t0 + wave;
    if (t < t1) {
        load_k(t, ka);
        load_v(t, vr);
        if (t + NW < t1) load_k(t + NW, kb2);
    }

    KD_TL(1);   // first tiles requested
    // ---- query rows: B operand of the first product, column c16; rows past the last repeat it
    bf16x8 qreg[NC];
    int vis;   // rows [0, vis) are visible to the lane's query: all cached rows, block rows 0 .. j
    {
        const uint16_t *qhead = p.q + (size_t)bh * p.G * p.Bt * D;
        const int m = min(m0 + c16, Mtot - 1);
        vis = p.len + m % p.Bt + 1;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            qreg[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(qhead + (size_t)m * D + c * 32 + 8 * g));
    }

    // ---- anchor: key sum after this step = key sum before it + the block's keys (at most 32 rows)
    double ksum_after = 0.0;
    double nmu2 = 0.0;   // |mu|^2
    const double *mu = alone ? mu_w[wave] : mu_s;
    if (alone) {
        double sq[WC];
#pragma unroll
        for (int i = 0; i < WC; ++i) {
            wsum[i] += bf16_hi((uint32_t)wkey[i] << 16);
            const double m = wsum[i] / (double)p.n;
            mu_w[wave][lane + 64 * i] = m;
            sq[i] = row_allreduce_f64<16>(m * m);
        }
#pragma unroll
        for (int i = 0; i < D / 16; ++i) {   // piece i is in the lanes of row i % 4
            const int from = 16 * (i % 4);
            nmu2 += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(sq[i / 4]), from),
                                     __builtin_amdgcn_readlane(__double2loint(sq[i / 4]), from));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (the wave reads what it wrote)
    } else if (need_sum) {
        double bacc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) bacc[i] = 0.0;
        static_assert(FEW_ROWS <= NT / UPR, "the block's rows fit one pass");
        {
            const u32x4 w = brow;   // (threads past the block hold zeros, which add nothing)
            double x[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[2 * i] = bf16_lo(w[i]);
                x[2 * i + 1] = bf16_hi(w[i]);
            }
            double inv = 1.0;
            if (p.anchor_mode == 1) {   // unit keys (Eq. 7): x / |k_j|, a zero key adds nothing
                double k2 = 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) k2 += x[i] * x[i];
                k2 = row_allreduce_f64<UPR>(k2);
                const double nk = sqrt(k2);
                inv = nk > 0.0 ? 1.0 / nk : 0.0;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) bacc[i] += (p.anchor_mode == 1) ? x[i] * inv : x[i];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            bacc[i] = sum_over_units_f64<UPR>(bacc[i]);
        }
        if (lane < UPR) {
#pragma unroll
            for (int i = 0; i < 8; ++i) bs_part[wave][bu * 8 + i] = bacc[i];
        }
        __syncthreads();
        double sq = 0.0;
        if (tid < D) {
            double tot = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) tot += bs_part[w][tid];
            ksum_after = ksum_before + tot;
            const double m = ksum_after / (double)p.n;
            mu_s[tid] = m;
            sq = m * m;
        }
        sq = row_allreduce_f64<16>(sq);
        if (tid < D && (lane & 15) == 0) red[tid / 16] = sq;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < D / 16; ++i) nmu2 += red[i];
    }

    KD_TL(2);   // anchor formed
    // ---- state of the wave
    f32x4 oacc[NDB], lacc = {0.f, 0.f, 0.f, 0.f};
    float mref = -INFINITY;
#pragma unroll
    for (int db = 0; db < NDB; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;

    unsigned char *vt = smem + (size_t)wave * FEW_KEYS * ROWB;
    // V rows are stored with their 16-byte units permuted so that what a transposing read gathers lies in
    // different banks: unit ^ VSW (row & 3) ^ 2 (row / 4 & 1) (16 units per row; 8 units: the first term alone)
    auto vswz = [](int row) { return UPR == 16 ? (VSW * (row & 3)) ^ (2 * ((row >> 2) & 1)) : VSW * (row & 3); };
    const int vwr = lane / UPR;   // row of load 0 of this lane; load i adds RPL i
    const int vrd_row = 4 * g + (c16 >> 2);
    const int vrd0 = vrd_row * ROWB + (c16 & 1) * 8;
    const int vrd_unit = ((c16 & 3) >> 1) ^ vswz(vrd_row);   // (rows + 16 have the same swizzle)

    // best row this lane has finished as (orderable score bits << 32 | row), and whether it met the same bits twice
    unsigned long long am_best = 0;
    bool am_tie = false;
    double held_dot = 0.0, held_k2 = 0.0;   // (mu.k, |k|^2) of the lane's row of the two tiles scored last
    int held_row = 0x7fffffff;
    auto flush_scores = [&]() {   // sqrt and divide on full waves: 64 rows of two tiles
        if (held_row < p.n) {
            const float sc = finish_score(held_dot, held_k2, nmu2, p.eps);
            p.scores[(size_t)bh * p.cap + held_row] = sc;
            if (p.scores_out) p.scores_out[(size_t)bh * p.n + held_row] = sc;
            const uint32_t bits = orderable(sc), top = (uint32_t)(am_best >> 32);
            am_tie = bits > top ? false : am_tie || bits == top;
            if (bits > top) am_best = ((unsigned long long)bits << 32) | (uint32_t)held_row;
        }
        held_row = 0x7fffffff;
    };

    auto tile = [&](int t, bool odd, u32x4 (&kc)[2][NC]) {
        // V of this tile to LDS (the reads of the tile before it have been consumed), then the next tile's loads
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = vwr + RPL * i;
            *reinterpret_cast<u32x4 *>(vt + row * ROWB + (((lane % UPR) ^ vswz(row)) * 16)) = vr[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (t + NW < t1) load_v(t + NW, vr);
        __builtin_amdgcn_sched_barrier(0);

        KD_TL(3);   // V of the tile in LDS
        // logits: element i of s[kg] is key 32 t + 16 kg + 4 g + i of query column c16
        f32x4 s[2];
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) s[kg] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int kg = 0; kg < 2; ++kg)
                s[kg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kc[kg][c]), qreg[c], s[kg], 0, 0, 0);

        // cosine score (appendix "FLOP count of KeyDiff"): the lane holds a quarter of row 16 kg + c16 of the tile
        if (scoring) {
            double dot[2], k2[2];
#pragma unroll
            for (int kg = 0; kg < 2; ++kg) dot[kg] = k2[kg] = 0.0;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double m8[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) m8[i] = mu[32 * c + 8 * g + i];
#pragma unroll
                for (int kg = 0; kg < 2; ++kg)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double x0 = bf16_lo(kc[kg][c][i]), x1 = bf16_hi(kc[kg][c][i]);
                        dot[kg] = __builtin_fma(m8[2 * i], x0, dot[kg]);
                        k2[kg] = __builtin_fma(x0, x0, k2[kg]);
                        dot[kg] = __builtin_fma(m8[2 * i + 1], x1, dot[kg]);
                        k2[kg] = __builtin_fma(x1, x1, k2[kg]);
                    }
            }
            // the four lanes of a row summed: lanes 0-15 end with mu.k of group 0, 16-31 with its |k|^2, 32-47 and 48-63
            // with those of group 1; then both halves of a pair get both numbers
            const double z = pair_split_f64<false>(pair_split_f64<true>(dot[0], dot[1]), pair_split_f64<true>(k2[0], k2[1]));
            const uint32_t zl = (uint32_t)__double2loint(z), zh = (uint32_t)__double2hiint(z);
            const auto l = __builtin_amdgcn_permlane16_swap(zl, zl, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap(zh, zh, false, false);
            if (odd == ((g & 1) != 0)) {
                held_dot = __hiloint2double((int)h[0], (int)l[0]);
                held_k2 = __hiloint2double((int)h[1], (int)l[1]);
                held_row = t * FEW_KEYS + 16 * (g >> 1) + c16;
            }
            if (odd) flush_scores();
        }
        if (t + 2 * NW < t1) load_k(t + 2 * NW, kc);   // kc is free
        __builtin_amdgcn_sched_barrier(0);
        KD_TL(4);   // tile scored

        // weights
        if ((t + 1) * FEW_KEYS > p.len) {   // uniform: rows of the block or past the end
            const int lim = vis - t * FEW_KEYS - 4 * g;
#pragma unroll
            for (int kg = 0; kg < 2; ++kg)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[kg][i] = 16 * kg + i < lim ? s[kg][i] : -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                         fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
        mx = max_over_rows(mx) * p.scale_log2e;
        const bool need = mx > mref + FEW_RESCALE_SLACK;
        if (__builtin_amdgcn_ballot_w64(need) != 0) {
            const float alpha = need ? __builtin_amdgcn_exp2f(mref - mx) : 1.f;
            mref = need ? mx : mref;
#pragma unroll
            for (int i = 0; i < 4; ++i) lacc[i] *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int i = 0; i < 4; ++i) oacc[db][i] *= alpha;
        }
        const float nm = mref == -INFINITY ? 0.f : -mref;
        bf16x8 pk;
#pragma unroll
        for (int kg = 0; kg < 2; ++kg)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                pk[4 * kg + i] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[kg][i], p.scale_log2e, nm));
        lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pk, lacc, 0, 0, 0);   // row sum of the rounded weights
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            const unsigned char *ap = vt + vrd0 + (((2 * db) ^ vrd_unit) * 16);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(ap));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(ap + 16 * ROWB));
            const bf16x8 va = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pk, oacc[db], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    for (; t < t1; t += 2 * NW) {
        tile(t, false, ka);
        if (t + NW < t1) tile(t + NW, true, kb2);
    }
    KD_TL(5);   // tiles done
    if (scoring) flush_scores();   // (an odd number of tiles leaves half a wave's rows)

    if (writer) {
        if (alone) {
#pragma unroll
            for (int i = 0; i < WC; ++i)
                if (wave == 0) p.ksum_next[(size_t)bh * D + lane + 64 * i] = wsum[i];
        } else if (tid < D) p.ksum_next[(size_t)bh * D + tid] = ksum_after;
    }

    // ---- the eight results become one
    KD_TL(6);   // scores finished
    float *const outs = reinterpret_cast<float *>(smem + (size_t)NW * FEW_KEYS * ROWB);
    float *ow = outs + (size_t)wave * 16 * D;
    if (c16 < mrows) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) *reinterpret_cast<f32x4 *>(ow + c16 * D + 16 * db + 4 * g) = oacc[db];
        if (g == 0) ml_s[wave][c16] = make_float2(mref, lacc[0]);
    }
    if (scoring && p.argmax_rec) rec_s[wave][lane] = am_best | (am_tie ? 0x80000000ull : 0ull);   // uniform (a row number takes 15 bits)
    __syncthreads();
    KD_TL(8);   // results and arg-max records in LDS
    if (scoring && p.argmax_rec && wave == NW - 1) {   // (the last wave: with few query rows it has nothing to merge)
        unsigned long long best = 0;
        bool tie = false;
#pragma unroll
        for (int w = 0; w < NW; ++w) {   // (as the records of different lanes are combined)
            const unsigned long long r = rec_s[w][lane], row = r & ~0x80000000ull;
            const bool rt = (r & 0x80000000ull) != 0;
            const uint32_t hr = (uint32_t)(r >> 32), hb = (uint32_t)(best >> 32);
            if (hr > hb) {
                best = row;
                tie = rt;
            } else if (hr == hb && hr != 0) tie = true;
        }
        wave_argmax(best, tie);
        if (lane == 0) {
            unsigned long long *rec = p.argmax_rec + ((size_t)bh * p.splits + sp) * 2;
            rec[0] = best;
            rec[1] = tie ? 1ull : 0ull;
        }
    }
    for (int it = tid; it < mrows * (D / 4); it += NT) {
        const int m = it / (D / 4), d0 = it % (D / 4) * 4;
        float mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) mx = fmaxf(mx, ml_s[w][m].x);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float2 ml = ml_s[w][m];
            const float f = ml.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - mx);
            const f32x4 o = *reinterpret_cast<const f32x4 *>(outs + ((size_t)w * 16 + m) * D + d0);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += f * o[i];
            L += f * ml.y;
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;   // a row may see no key of this workgroup's range
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] *= inv;
        if (p.splits > 1) {
            *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(p.part_o) + (((size_t)sp * BH + bh) * Mtot + m0 + m) * D + d0) = acc;
            if (d0 == 0) p.part_ml[((size_t)sp * BH + bh) * Mtot + m0 + m] = make_float2(mx, L);
        } else {
            bf16x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (__bf16)acc[i];
            *reinterpret_cast<bf16x4 *>(p.out + ((size_t)bh * p.G * p.Bt + m0 + m) * D + d0) = o;
        }
    }
    KD_TL(9);   // partial stored
#ifdef KD_TIMELINE
    __builtin_amdgcn_s_waitcnt(0x0F70);
    KD_TL(12);
    if (threadIdx.x == 0) kd_tl[31] = 5;   // record kind: step_few workgroup
    KD_TL_DUMP(p.timeline, blockIdx.x);
#endif
}

hipError_t configure_few_kernels()
{
    hipError_t e;
#define KD_SET(D, ST)                                                                                                        \
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(step_few_kernel<D, ST>), hipFuncAttributeMaxDynamicSharedMemorySize, \
                            (int)few_lds_bytes<D>());                                                                        \
    if (e != hipSuccess) return e;
    KD_SET(128, false)
    KD_SET(128, true)
    KD_SET(64, false)
    KD_SET(64, true)
#undef KD_SET
    return hipSuccess;
}

hipError_t launch_step_few(const StepParams &p, hipStream_t s)
{
    const int M = p.G * p.Bt;
    if (!p.few || M > FEW_ROWS || p.mtiles != (M + 15) / 16) return hipErrorInvalidValue;
    const int grid = p.batch * p.hkv * p.mtiles * p.splits;
    // Caches that do not fit the 256 MB last-level cache cannot be found there by the next step: they are read with the
    // non-temporal hint (537 MB, 16 sequences: 109 -> 98 us a launch; a plain read of the same bytes 92 -> 82 us).  Smaller
    // ones would lose what the last-level cache holds of them (14 MB a layer: 4 to 6 % slower with the hint).
    const bool stream = 4.0 * p.batch * p.hkv * (double)p.n * p.D > 256.0 * 1024 * 1024;
#define KD_GO(D)                                                                                                                \
    if (stream) hipLaunchKernelGGL((step_few_kernel<D, true>), dim3(grid), dim3(64 * FEW_WAVES), (few_lds_bytes<D>()), s, p); \
    else hipLaunchKernelGGL((step_few_kernel<D, false>), dim3(grid), dim3(64 * FEW_WAVES), (few_lds_bytes<D>()), s, p);
    if (p.D == 128) { KD_GO(128) }
    else if (p.D == 64) { KD_GO(64) }
    else return hipErrorInvalidValue;
#undef KD_GO
    return hipGetLastError();
}

}  // namespace kd
