/*
 * gfx950 kernels for Eq. 1 on the dose-coefficient matrix D_ij.
 *
 *   beamlet-row CSR (what the fill writes: row j = beamlet, columns = voxels)
 *     k_fluence_dose      dose_i += w_j D_ij, summed over neighbouring rows in LDS, then FP32
 *                         atomics                            -- one wave per share of 8 or 32 rows
 *     k_fluence_gradient  g_j = sum_i D_ij r_i, fixed order      -- one workgroup per row
 *   voxel-row CSR (row i = voxel, columns = beamlets): the transpose, a stable
 *   sort of the row-major entries by column
 *     k_run_count, scan, k_run_sizes   runs of each piece of a row (stretches within
 *                                      one 32-column bucket), their pointers, the
 *                                      path flags
 *     run path (the default for D, whose rows are long stretches of columns):
 *       k_run_emit                     run records: bucket, row, first entry and a
 *                                      32-bit column mask (ascending rows) or length
 *       k_rs_hist, scan, k_run_scatter stable LSD radix sort of the runs by bucket
 *       k_bucket_bounds                bucket pointers
 *       rows ascending:   k_bucket_count (column counts from the masks), scan (the
 *                         voxel-row pointers), k_place_sorted -- runs' values in
 *                         registers by column, written out column by column
 *       rows in any order: k_key_count + scan (pointers), k_place_any
 *     entry path (short stretches): k_key_count + scan, k_expand_rows, then
 *       k_rs_hist, scan, k_rs_scatter per 8 bits of the column
 *     k_voxel_dose        dose_i = sum_j D_ij w_j, fixed order  -- 8 lanes per voxel row
 *
 * Both sorts are stable and the input rows are in ascending beamlet order, so
 * every voxel row lists its beamlets in ascending order: the transpose is
 * canonical and bit-reproducible.  It runs without host synchronisation.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <utility>

#include "fspb_device.h"

namespace fspb {

namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;          // digits per pass
constexpr int kSortBlock = 512;                  // threads of a scatter workgroup
constexpr int kSortWaves = kSortBlock / kWave;
constexpr int kSortItems = 8;                    // entries per thread of a tile
constexpr int kSortTile = kSortBlock * kSortItems;   // 4096 entries per sort tile
constexpr int kScanRounds = 4;
constexpr int kScanChunk = 4 * kBlock * kScanRounds;   // 4096 values per scan block
constexpr int kScanTop = 1024;

static_assert(kRadix == kBlock && kRadix <= kSortBlock, "one thread per digit");

/* Item of workgroup blockIdx.x where each XCD is to take GROUP consecutive items: workgroups are handed
 * to the 8 XCDs in turn. */
constexpr int kXcds = 8;
template <int GROUP>
__device__ inline int xcd_item()
{
    const int x = (int)(blockIdx.x % kXcds), k = (int)(blockIdx.x / kXcds);
    return ((k / GROUP) * kXcds + x) * GROUP + k % GROUP;
}

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ inline int mbcnt64(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

template <typename T>
__device__ inline T wave_sum(T x)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, kWave);
    return x;
}

/*
 * Inclusive scan of a wave's 32-bit integers by DPP: row shifts by 1, 2, 4 and
 * 8 lanes scan each row of 16 lanes (lanes shifted in from outside the row read
 * 0); rows 1 and 3 then add the last lane of the row below (row_bcast:15) and
 * rows 2 and 3 add lane 31 (row_bcast:31).  Every lane of the wave must be
 * active.
 */
__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return (uint32_t)x;
}

/* Wave total of 32-bit integers (every lane active), the same on every lane. */
__device__ inline uint32_t wave_sum(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(x), kWave - 1);
}

/* Exclusive scan of one value per thread over a block of W waves; *total gets the sum. */
template <int W = kWavesPerBlock>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t *s_w, uint32_t *total)
{
    const int l = lane_id(), w = threadIdx.x >> 6;
    uint32_t x = wave_incl_scan(v);
    if (l == kWave - 1) s_w[w] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const uint32_t t = s_w[k];
        off += k < w ? t : 0u;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

/* ------------------------------------------------------------ Eq. 1 */

__global__ __launch_bounds__(kBlock) void k_zero(float *__restrict__ x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) x[i] = 0.0f;
}

__global__ __launch_bounds__(kBlock) void k_zero_u32(uint32_t *__restrict__ x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) x[i] = 0u;
}

/*
 * dose[i] += w_j D_ij.  One global FP32 atomic per entry is bound at the memory
 * side, to which every request is forwarded (3.40 ms for 6.5e8 entries on a
 * 128^3 grid, 1.5 TB/s of matrix), and LDS float atomics take about two cycles
 * per lane (4.0 ms); but neighbouring beamlets cover nearly the same voxels.
 * So a wave takes a share (the same fraction of each) of `group` consecutive
 * rows and walks it in windows of kDoseWindow columns, each starting at the
 * lowest column not yet added: all rows' entries of the window are added with
 * plain reads and writes to the wave's own LDS, then each touched voxel goes
 * out with one coalesced atomic.  Lane r finds the end of row r's part of the
 * window by bisection (at most kDoseWindow entries, when columns ascend),
 * starting from the length of its last part.  1.55 ms (3.4 TB/s of matrix): the
 * waves stream at 5 TB/s but search for a third of their time.
 *
 * Nothing is assumed about the order of a row's columns: entries a window does
 * not hold, and 64-entry sets whose columns do not ascend strictly (plain adds
 * need them distinct), go to memory one by one, and so does what is left of a
 * share whose rows lie too far apart for windows to pay.
 *
 * A group whose shares would have fewer than kDoseShare entries, or one of whose
 * rows does not ascend from its first entry to its middle one and its last, takes no
 * shares: its waves take whole rows, or pieces of rows, and send every entry to
 * memory.  The searches of a window cost about what a thousand atomics do (2000 rows
 * of 1000 entries: 13.6 us, 29.8 in shares of 500; 9000 shuffled rows of 300: 48 and
 * 98; 64^3 and 8100 beamlets with a 1 cm cutoff, shares of 2245: 74 in windows, 143
 * straight to memory).
 */
constexpr int kDoseRows = 32;
constexpr int kDoseWindow = 2048;              // 8 KB of LDS per wave
constexpr int kDoseSets = 4;                   // 64-entry sets whose loads are issued together
constexpr int kDoseMinEntries = 64;            // windows pay with more entries than this each and at
constexpr int kDoseSlack = 1024;               // least 4/3 per touched voxel, give or take a share's
                                               // ragged ends
constexpr int kDoseShare = 2048;               // fewest entries of a share
constexpr int kDosePiece = 128;                // fewest entries of a piece of a row, on average
constexpr int kDoseSpread = 8;                 // most columns per entry over which a share's rows lie
constexpr int kDoseGuess = 24;                 // width of the first guess at a row's part of a window

/* Orders a wave's LDS accesses: they complete in issue order, so the compiler only has to keep theirs. */
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline int64_t readlane64(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ inline uint32_t wave_min(uint32_t v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, d, kWave));
    return v;
}

/* Columns between the lowest and the highest end of the rows' parts [p, end) of a share. */
__device__ inline int64_t dose_span(const int32_t *__restrict__ indices, int64_t p, int64_t end)
{
    const uint32_t a = p < end ? (uint32_t)indices[p] : 0xffffffffu, b = p < end ? (uint32_t)indices[end - 1] : 0xffffffffu;
    const uint32_t lo = wave_min(min(a, b)), hi = ~wave_min(p < end ? ~max(a, b) : 0xffffffffu);
    return hi > lo ? (int64_t)(hi - lo) : 0;
}

__global__ __launch_bounds__(kBlock) void k_fluence_dose(const int64_t *__restrict__ indptr,
                                                         const int32_t *__restrict__ indices,
                                                         const float *__restrict__ values, int n_rows,
                                                         int n_voxels, const float *__restrict__ w,
                                                         float *__restrict__ dose, int group)
{
    __shared__ float s_acc[kWavesPerBlock][kDoseWindow];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    float *acc = s_acc[wave];
    const uint32_t n = (uint32_t)n_voxels;
    // lane r < group (at most kDoseRows): row r of the group, its share [p, end); a row of weight 0
    // adds nothing
    const int j = blockIdx.x * group + lane;
    const float wj = lane < group && j < n_rows ? w[j] : 0.0f;
    const int64_t e0 = wj != 0.0f ? indptr[j] : 0, e1 = wj != 0.0f ? indptr[j + 1] : 0;
    const int64_t len = max(e1 - e0, (int64_t)0), all = wave_sum(len);
    const int waves = (int)gridDim.y * kWavesPerBlock, me = (int)blockIdx.y * kWavesPerBlock + wave;
    // where the k-th of n equal parts of the lane's row begins
    auto cut = [&](int k, int n) { return e0 + len / n * k + len % n * k / n; };
    int64_t p = e0, end = e0;
    bool windowed = false, shares = all >= (int64_t)kDoseShare * waves;
    if (shares) {
        // the same rows and entries for every wave of the group: it takes shares, or it does not
        const uint32_t a = len ? (uint32_t)indices[e0] : 0u, m = len ? (uint32_t)indices[e0 + (len >> 1)] : 0u;
        const uint32_t b = len ? (uint32_t)indices[e1 - 1] : 0u;
        p = cut(me, waves);
        end = cut(me + 1, waves);
        windowed = dose_span(indices, p, end) <= kDoseSpread * wave_sum(end - p);
        shares = __ballot(a > m || m > b) == 0;
    }
    if (!shares) {   // rows, or pieces of rows where there are more waves than rows
        const int rows = min(group, n_rows - (int)blockIdx.x * group);
        const int pieces = (int)max((int64_t)1, min((int64_t)(waves / rows), all / rows / kDosePiece));
        const int step = pieces > 1 ? rows : min(waves, rows), r = me / pieces, k = me - r * pieces;
        const bool mine = r < step && lane % step == r;
        p = mine ? cut(k, pieces) : e0;
        end = mine ? cut(k + 1, pieces) : e0;
        windowed = false;
    }
    if (windowed) {
        for (int i = lane; i < kDoseWindow; i += kWave) acc[i] = 0.0f;
        wave_lds_fence();
    }

    struct Group {
        uint32_t i[kDoseSets];
        float v[kDoseSets], w[kDoseSets];
        int n[kDoseSets];
    };
    int64_t seen = 0;
    int guess = -1;
    int64_t out = 0;
    for (int64_t windows = 1; windowed && __ballot(p < end); ++windows) {
        // the window [base, base + kDoseWindow), aligned for coalesced atomics
        const uint32_t base = wave_min(p < end ? (uint32_t)indices[p] : 0xffffffffu) & ~31u;
        const uint32_t stop = base < 0xffffffffu - kDoseWindow ? base + kDoseWindow : 0xffffffffu;
        int64_t lo = p, hi = min(end, p + kDoseWindow);
        if (guess >= 0) {   // the last window's count, give or take
            const int64_t qa = lo + guess - kDoseGuess, qb = lo + guess + kDoseGuess;
            const bool ia = qa >= lo && qa < hi, ib = qb < hi;
            const uint32_t ca = ia ? (uint32_t)indices[qa] : 0u, cb = ib ? (uint32_t)indices[qb] : 0u;
            if (ib) {
                if (cb < stop) lo = qb + 1;
                else hi = qb;
            }
            if (ia && qa >= lo) {
                if (ca < stop) lo = qa + 1;
                else hi = qa;
            }
        }
        while (__ballot(lo < hi)) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if (lo < hi) {
                if ((uint32_t)indices[mid] < stop) lo = mid + 1;
                else hi = mid;
            }
        }
        const int cnt = (int)(lo - p);
        guess = cnt;
        if (!__ballot(cnt > 0)) break;   // only columns outside the grid next
        seen += wave_sum((uint32_t)cnt);
        // the rows with entries in the window in sets of 64, kDoseSets of them at a time, two such
        // groups in flight while a third is added
        uint64_t rows = __ballot(cnt > 0);
        int left = 0;
        int64_t at = 0;
        float wr = 0.0f;
        auto load = [&](Group &G) {
#pragma unroll
            for (int k = 0; k < kDoseSets; ++k) {
                if (left <= 0 && rows) {
                    const int r = (int)__builtin_ctzll(rows);
                    rows &= rows - 1;
                    left = __builtin_amdgcn_readlane(cnt, r);
                    at = readlane64(p, r);
                    wr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wj), r));
                }
                G.n[k] = left;
                G.w[k] = wr;
                const bool in = lane < left;
                G.i[k] = in ? (uint32_t)__builtin_nontemporal_load(indices + at + lane) : 0xffffffffu;
                G.v[k] = in ? __builtin_nontemporal_load(values + at + lane) : 0.0f;
                left -= kWave;
                at += kWave;
            }
        };
        auto add = [&](const Group &G) {
#pragma unroll
            for (int k = 0; k < kDoseSets; ++k) {
                if (G.n[k] <= 0) break;
                const uint32_t c = G.i[k];
                const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x138, 0xf, 0xf, false);
                const bool down = lane > 0 && lane < G.n[k] && c <= below;
                const float x = G.w[k] * G.v[k];
                if (__ballot(down) == 0 && c < n && c - base < (uint32_t)kDoseWindow) acc[c - base] += x;
                else if (c < n) atomicAdd(dose + c, x);
                wave_lds_fence();
            }
        };
        Group g0, g1, g2;
        load(g0);
        load(g1);
        for (;;) {
            load(g2);
            add(g0);
            if (g1.n[0] <= 0) break;
            load(g0);
            add(g1);
            if (g2.n[0] <= 0) break;
            load(g1);
            add(g2);
            if (g0.n[0] <= 0) break;
        }
        // the touched voxels (adding 0 changes nothing)
        uint32_t touched = 0;
#pragma unroll 4
        for (int i = lane; i < kDoseWindow; i += kWave) {
            const float x = acc[i];
            if (x != 0.0f) {
                atomicAdd(dose + base + i, x);
                ++touched;
            }
            acc[i] = 0.0f;
        }
        wave_lds_fence();
        p = lo;
        out += wave_sum(touched);
        if (4 * out > 3 * seen + kDoseSlack || seen + kDoseSlack < windows * kDoseMinEntries) break;
    }
    // what is left, straight to memory: four rows at a time, or two or four parts of a row
    uint64_t rows = __ballot(p < end);
    const int many = __popcll(rows), q = many >= 4 ? 1 : many >= 2 ? 2 : 4;
    while (rows) {
        int64_t a[4], b[4];
        float wr[4];
        bool more = false, row = false;
        int r = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if ((k & (q - 1)) == 0) {
                row = rows != 0;
                r = row ? (int)__builtin_ctzll(rows) : 0;
                rows &= rows - 1;
            }
            a[k] = row ? readlane64(p, r) + kWave * (k & (q - 1)) : 0;
            b[k] = row ? readlane64(end, r) : 0;
            wr[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wj), r));
            more = more || a[k] < b[k];
        }
        while (more) {
            uint32_t i[4];
            float v[4];
            more = false;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in = a[k] + lane < b[k];
                i[k] = in ? (uint32_t)indices[a[k] + lane] : 0xffffffffu;
                v[k] = in ? values[a[k] + lane] : 0.0f;
                a[k] += q * kWave;
                more = more || a[k] < b[k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i[k] < n) atomicAdd(dose + i[k], wr[k] * v[k]);
        }
    }
}

/*
 * Entries [e0, e1) of a CSR row split for 16-byte loads: [e0, a) head, [a, b) whole
 * steps of `step` entries (4 consecutive per lane), [b, e1) tail; the head is
 * shorter than 4 entries.  Only when indices and values have the same offset
 * modulo 16 bytes; otherwise head and steps are empty and the whole row is tail.
 */
struct RowSplit { int64_t a, b; };

__device__ inline RowSplit row_split(const int32_t *indices, const float *values, int64_t e0, int64_t e1,
                                     int step)
{
    const uintptr_t oi = (uintptr_t)indices, ov = (uintptr_t)values;
    if ((oi & 3) || (ov & 3) || ((oi ^ ov) & 15)) return {e0, e0};
    const int64_t mis = (int64_t)((oi >> 2) & 3);          // element offset of the array modulo 4
    const int64_t a = min(e1, ((e0 + mis + 3) & ~(int64_t)3) - mis);
    return {a, a + (e1 - a) / step * step};
}

typedef int vi4 __attribute__((ext_vector_type(4)));
typedef float vf4 __attribute__((ext_vector_type(4)));

/*
 * g_j = sum_i D_ij r_i; one workgroup per row.  The row's middle goes in steps
 * of PER BLOCK entries: lane l of wave w takes entries 64 PER w + l + 64 k
 * (k < PER) of a step, so that each gather of r reads 64 consecutive columns;
 * the next step's indices and values are loaded after this step's gathers are
 * issued, so they are in flight while the gathered values are awaited.  The tail
 * is lane-strided, four entries of a lane at a time and the first four loaded with the first
 * step; lane partial sums, a fixed butterfly per wave and the wave totals added in
 * wave order.  Columns outside [0, n_voxels) are skipped.
 *
 * Bound by the read of D.  Rows start anywhere, so steps share cache lines: marked
 * as streamed the loads fetch them twice (128^3, 9 beams of 900, 8.1e4 entries a
 * row, with groups of 16 rows as below: 1027 us against 977).
 *
 * The width follows the number of rows, all that the host knows of the matrix.  Few
 * rows get 1024 threads each, or most of the chip idles (240 rows of 8e4 entries:
 * 33 us, 88 with 256).  Many rows may be short, and then what counts is how many
 * waves have to be launched: 256 threads (9000 rows of 50 entries: 7.6 us, 20.5 with
 * 1024; of 1000: 18.1 and 31.6; at 2000 rows of 50 the widths are equal, at 4000
 * they take 7.8 and 10.2).  Long rows then need many entries in flight per lane, or
 * so many rows are open at once that r falls out of the L2: PER 8 takes 977 us on
 * that slab, PER 4 999; above kGradMany rows, where rows are shorter still, PER 4
 * (40000 of 2000: 119 us, PER 8 131).
 *
 * With 256 threads kGradXcd consecutive rows go to one XCD (workgroups are dealt to
 * the XCDs in turn), since neighbouring beamlets gather the same voxels of r.  That slab:
 * 959 us (1024 threads a row 945, 256 as before them 1070), 977 in groups of 16, 1047
 * one by one; groups of 64 take 960 but on 256x256x100 with 9 beams of 576 642 against 623,
 * of 256 994 and 699.
 */
constexpr int kGradFew = 2048;
constexpr int kGradMany = 32768;
constexpr int kGradXcd = 32;
template <int GROUP>
__device__ inline int grad_row(int n_rows)
{
    const int b = blockIdx.x;
    if constexpr (GROUP == 0) return b;
    else return b < n_rows - n_rows % (kXcds * GROUP) ? xcd_item<GROUP>() : b;   // the last, partial set: one by one
}
template <int BLOCK, int PER, int GROUP>
__global__ __launch_bounds__(BLOCK) void k_fluence_gradient(const int64_t *__restrict__ indptr,
                                                            const int32_t *__restrict__ indices,
                                                            const float *__restrict__ values, int n_rows,
                                                            int n_voxels, const float *__restrict__ r,
                                                            float *__restrict__ g)
{
    constexpr int kStep = PER * BLOCK;
    constexpr int kWaves = BLOCK / kWave;
    __shared__ float s_w[kWaves];
    const int j = grad_row<GROUP>(n_rows);
    const int t = threadIdx.x;
    const uint32_t n = (uint32_t)n_voxels;
    const int64_t e0 = indptr[j], e1 = indptr[j + 1];
    // whole steps from the row's start (4-byte loads need no alignment), then the tail
    const int64_t b = e0 + (e1 - e0) / kStep * kStep;
    float acc0 = 0.0f, acc1 = 0.0f;
    int64_t e = e0 + PER * kWave * (t >> 6) + (t & (kWave - 1));
    uint32_t i0[PER], ti[4];
    float v0[PER], tv[4];
    if (e0 < b) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            i0[k] = (uint32_t)indices[e + kWave * k];
            v0[k] = values[e + kWave * k];
        }
    }
    auto load_tail = [&](int64_t at) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            ti[k] = ~0u;
            if (at + t + BLOCK * k < e1) {
                ti[k] = (uint32_t)indices[at + t + BLOCK * k];
                tv[k] = values[at + t + BLOCK * k];
            }
        }
    };
    load_tail(b);
    if (e0 < b) {   // the same for the whole workgroup, as is every step test below
        for (;;) {
            const int64_t en = e + kStep;
            float x[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) x[k] = i0[k] < n ? r[i0[k]] : 0.0f;
            uint32_t i1[PER];
            float v1[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                i1[k] = i0[k];
                v1[k] = v0[k];
            }
            if (en < b) {
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    i1[k] = (uint32_t)indices[en + kWave * k];
                    v1[k] = values[en + kWave * k];
                }
            }
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if (i0[k] < n) acc0 = fmaf(v0[k], x[k], acc0);
            if (en >= b) break;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                i0[k] = i1[k];
                v0[k] = v1[k];
            }
            e = en;
        }
    }
#pragma unroll
    for (int q = 0; q < PER; q += 4) {
        if (q && b + BLOCK * q >= e1) break;
        if (q) load_tail(b + BLOCK * q);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (ti[k] < n) acc1 = fmaf(tv[k], r[ti[k]], acc1);
    }
    const float s = wave_sum(acc0 + acc1);
    if (lane_id() == 0) s_w[t >> 6] = s;
    __syncthreads();
    if (t == 0) {
        float tot = s_w[0];
        for (int k = 1; k < kWaves; ++k) tot += s_w[k];
        g[j] = tot;
    }
}

/*
 * dose_i = sum_j D_ij w_j over voxel row i, in a fixed order: 8 lanes per row,
 * steps of 32 entries by 16-byte loads of four consecutive ones per lane, the
 * next step's loads in flight while this step's entries are added; a row's head,
 * tail and first step are loaded together, and the pointers of the next row
 * before them.  Lane-strided partial sums, a fixed butterfly.  Beamlets outside
 * [0, n_w) are skipped.
 *
 * Bound by the read of D.  Neighbouring rows and steps share cache lines, so the
 * loads are not marked as streamed (16 lanes: 1148 us, marked 1214).  8 lanes,
 * because many rows are shorter than a step of 16 or 32 (64x64x64, one beam of
 * 100: 8 us, 13 with 16 lanes, 25 with 32).  w comes from LDS where a CU can hold
 * four copies and so all its waves (128^3, 9 beams of 900: 1020 us, gathered
 * through the cache 1202; 12500 beamlets 117 and 102) and the matrix has a third of an
 * entry for each word copied (64^3, 8100 beamlets: with 2.5 entries per word 144 and 184,
 * with 0.27 23.3 and 18.9, with 0.02 13.5 and 7.6; 9000 on 2e6 voxels, 0.49: 102 and 87
 * where neighbouring voxels meet the same beamlets, 105 and 158 where any).
 *
 * Workgroups stay for many rows: 8191 of them (128^3, 9 beams of 900 with 4095: 1082 us,
 * 8191: 1028, 12287: 1016; 256x256x100, 9 beams of 576: 910, 896, 1016), an odd number, so
 * that no workgroup's rows keep the same place in the grid's lines (that matrix with 8064
 * 1095, with 8189, 8190, 8192 and 8193 908, 844, 1205 and 912; 9 beams of 1600 and a 1 cm
 * cutoff 350 with the odd numbers, 493 with 8064, 531 with 8192; on 128^3 all within 4 %).
 * 128^3, 9 beams of 900, 6.5e8 entries: 1028 us (5.1 TB/s), 1469 with 16 lanes per
 * row, a workgroup per 16 rows, the tail after the steps and w from the cache;
 * 256x256x100, 9 beams of 576: 1916 -> 896.
 */
constexpr int kVoxelBlock = 512;
constexpr int kVoxelLanes = 8;
constexpr int kVoxelRows = kVoxelBlock / kVoxelLanes;
constexpr int kVoxelStep = 4 * kVoxelLanes;
constexpr int kVoxelLdsWords = 10240;              // 40 KB: four workgroups, 32 waves per CU
constexpr int kVoxelGroups = 8191;
constexpr int kVoxelReuse = 3;                     // words of w copied to LDS per entry, at most
constexpr int kVoxelFewWords = 1024;               // copied in any case: the entries' number is one load later
template <bool LDS>
__device__ __attribute__((always_inline)) inline void voxel_rows(const int64_t *__restrict__ t_indptr,
                                                                 const int32_t *__restrict__ t_indices,
                                                                 const float *__restrict__ t_values, int n_voxels,
                                                                 int n_w, const float *w, float *__restrict__ dose)
{
    extern __shared__ float s_w[];
    const float *wt = LDS ? s_w : w;
    const int l = threadIdx.x & (kVoxelLanes - 1);
    const uint32_t n = (uint32_t)n_w;
    const int64_t stride = (int64_t)gridDim.x * kVoxelRows;
    int64_t i = (int64_t)blockIdx.x * kVoxelRows + threadIdx.x / kVoxelLanes;
    if (i >= n_voxels) return;
    int64_t e0 = t_indptr[i], e1 = t_indptr[i + 1];
    for (;;) {
        const int64_t in = i + stride;
        int64_t n0 = 0, n1 = 0;
        if (in < n_voxels) {
            n0 = t_indptr[in];
            n1 = t_indptr[in + 1];
        }
        const RowSplit sp = row_split(t_indices, t_values, e0, e1, kVoxelStep);
        uint32_t hi = ~0u, ti[4];
        float hv, tv[4];
        if (e0 + l < sp.a) {
            hi = (uint32_t)t_indices[e0 + l];
            hv = t_values[e0 + l];
        }
        int64_t e = sp.a + 4 * l, te = sp.b + l;
        vi4 a;
        vf4 c;
        if (e < sp.b) {
            a = *reinterpret_cast<const vi4 *>(t_indices + e);
            c = *reinterpret_cast<const vf4 *>(t_values + e);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ti[u] = ~0u;
            if (te + kVoxelLanes * u < e1) {
                ti[u] = (uint32_t)t_indices[te + kVoxelLanes * u];
                tv[u] = t_values[te + kVoxelLanes * u];
            }
        }
        float acc[2] = {0.0f, 0.0f};
        while (e < sp.b) {
            e += kVoxelStep;
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if ((uint32_t)a[u] < n) x[u] = wt[(uint32_t)a[u]];
            const vi4 ap = a;
            const vf4 cp = c;
            if (e < sp.b) {
                a = *reinterpret_cast<const vi4 *>(t_indices + e);
                c = *reinterpret_cast<const vf4 *>(t_values + e);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if ((uint32_t)ap[u] < n) acc[u & 1] = fmaf(cp[u], x[u], acc[u & 1]);
        }
        float s = 0.0f;
        if (hi < n) s = hv * wt[hi];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (ti[u] < n) s = fmaf(tv[u], wt[ti[u]], s);
        for (te += kVoxelStep; te < e1; te += kVoxelLanes) {   // a tail longer than a step: unequal offsets
            const uint32_t j = (uint32_t)t_indices[te];
            if (j < n) s = fmaf(t_values[te], wt[j], s);
        }
        s += acc[0] + acc[1];
#pragma unroll
        for (int d = kVoxelLanes / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, kWave);
        if (l == 0) dose[i] = s;
        if (in >= n_voxels) break;
        i = in;
        e0 = n0;
        e1 = n1;
    }
}

/* Where w is read: through the cache, from LDS, or by the number of entries (kVoxelReuse).  Eight waves
 * per SIMD: with 66 registers instead of 64 there were seven (240 rows of 8e4 entries on 128^3: 60 us
 * instead of 49). */
enum class WHome { kCache, kLds, kEither };
template <WHome HOME>
__global__ __launch_bounds__(kVoxelBlock, 8) void k_voxel_dose(const int64_t *__restrict__ t_indptr,
                                                               const int32_t *__restrict__ t_indices,
                                                               const float *__restrict__ t_values, int n_voxels,
                                                               int n_w, const float *__restrict__ w,
                                                               float *__restrict__ dose)
{
    extern __shared__ float s_w[];
    if (HOME == WHome::kLds || (HOME == WHome::kEither && (int64_t)n_w * gridDim.x <=
                                                              kVoxelReuse * (t_indptr[n_voxels] - t_indptr[0]))) {
        for (int j = threadIdx.x; j < n_w; j += kVoxelBlock) s_w[j] = w[j];
        __syncthreads();
        voxel_rows<true>(t_indptr, t_indices, t_values, n_voxels, n_w, w, dose);
    } else {
        voxel_rows<false>(t_indptr, t_indices, t_values, n_voxels, n_w, w, dose);
    }
}

/* ------------------------------------------------------------ transpose */

/*
 * The transpose never synchronises the host: both of its sort paths are
 * enqueued, and a flag the device computes from the data (how long the
 * stretches of each row within a bucket of columns are) lets one of them run;
 * the other's kernels return at once.  Sizes only the device knows (the number
 * of stretches) are read by the kernels themselves, which walk their work
 * grid-stride from a grid sized by a host bound.
 */
struct Gate {
    const int32_t *flag;   // nullptr: always run
    int32_t want;
};
__device__ inline bool gate_closed(Gate g) { return g.flag && *g.flag != g.want; }

/* An element count known on the host (dev == nullptr) or read from device memory. */
struct Count {
    int64_t n;
    const int64_t *dev;
};
__device__ inline int64_t count_of(Count c) { return c.dev ? *c.dev : c.n; }

/* rows[e] = j for every entry e of row j (clamped to [0, nnz)); one wave per row. */
__global__ __launch_bounds__(kBlock) void k_expand_rows(const int64_t *__restrict__ indptr, int n_rows, int64_t nnz,
                                                        int32_t *__restrict__ rows, Gate g)
{
    if (gate_closed(g)) return;
    const int j = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (j >= n_rows) return;
    const int64_t e0 = indptr[j] > 0 ? indptr[j] : 0, e1 = indptr[j + 1] < nnz ? indptr[j + 1] : nnz;
    for (int64_t e = e0 + lane_id(); e < e1; e += kWave) rows[e] = j;
}

/* Values base .. base + 3 of in[0, n), 0 past the end (in: 16-byte aligned, base a multiple of 4). */
__device__ inline uint4 load_four(const uint32_t *in, int64_t base, int64_t n)
{
    if (base + 3 < n) return *reinterpret_cast<const uint4 *>(in + base);
    return make_uint4(base < n ? in[base] : 0u, base + 1 < n ? in[base + 1] : 0u, base + 2 < n ? in[base + 2] : 0u, 0u);
}

/* Scan, phase 1: sum of each kScanChunk-value chunk (grid-stride over chunks).  In both this and
 * phase 3 a thread takes four consecutive values a round, so that a wave reads 1 KB in one go. */
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t *__restrict__ in, Count n_in,
                                                        uint32_t *__restrict__ partial, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ uint32_t s_w[kWavesPerBlock];
    const int64_t n = count_of(n_in), nch = (n + kScanChunk - 1) / kScanChunk;
    for (int64_t c = blockIdx.x; c < nch; c += gridDim.x) {
        uint32_t v = 0;
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r) {
            const uint4 x = load_four(in, c * kScanChunk + (r * kBlock + (int)threadIdx.x) * 4, n);
            v += x.x + x.y + x.z + x.w;
        }
        v = wave_sum(v);
        if (lane_id() == 0) s_w[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = 0;
            for (int k = 0; k < kWavesPerBlock; ++k) t += s_w[k];
            partial[c] = t;
        }
        __syncthreads();
    }
}

/* Scan, phase 2: exclusive scan of the chunk sums in place (one workgroup);
 * partial[nb] = total, also stored to *total64 when given. */
__global__ __launch_bounds__(kScanTop) void k_scan_top(uint32_t *__restrict__ partial, Count n_in,
                                                       int64_t *__restrict__ total64, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ uint32_t s_w[kScanTop / kWave];
    const int64_t nb = (count_of(n_in) + kScanChunk - 1) / kScanChunk;
    const int l = lane_id(), w = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kScanTop) {
        const int64_t i = b0 + threadIdx.x;
        const uint32_t v = i < nb ? partial[i] : 0u;
        uint32_t x = wave_incl_scan(v);
        if (l == kWave - 1) s_w[w] = x;
        __syncthreads();
        uint32_t off = 0, tot = 0;
        for (int k = 0; k < kScanTop / kWave; ++k) {
            off += k < w ? s_w[k] : 0u;
            tot += s_w[k];
        }
        if (i < nb) partial[i] = carry + off + x - v;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[nb] = carry;
        if (total64) *total64 = (int64_t)carry;
    }
}

/* Scan, phase 3: exclusive scan within each chunk plus its chunk offset (grid-stride); out may
 * be in (each round is read before it is written). */
template <typename OUT>
__global__ __launch_bounds__(kBlock) void k_scan_down(const uint32_t *in, Count n_in, const uint32_t *__restrict__ partial,
                                                      OUT *out, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ uint32_t s_w[kWavesPerBlock];
    const int64_t n = count_of(n_in), nch = (n + kScanChunk - 1) / kScanChunk;
    for (int64_t c = blockIdx.x; c < nch; c += gridDim.x) {
        uint32_t run = partial[c];
        uint4 x[kScanRounds];
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r)
            x[r] = load_four(in, c * kScanChunk + (r * kBlock + (int)threadIdx.x) * 4, n);
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r) {
            const int64_t i = c * kScanChunk + (r * kBlock + (int)threadIdx.x) * 4;
            uint32_t total;
            const uint32_t e = run + block_excl_scan(x[r].x + x[r].y + x[r].z + x[r].w, s_w, &total);
            run += total;
            if (i < n) out[i] = (OUT)e;
            if (i + 1 < n) out[i + 1] = (OUT)(e + x[r].x);
            if (i + 2 < n) out[i + 2] = (OUT)(e + x[r].x + x[r].y);
            if (i + 3 < n) out[i + 3] = (OUT)(e + x[r].x + x[r].y + x[r].z);
        }
    }
}

/* Radix pass, phase 1: digit histogram of each kSortTile-entry tile, stored
 * digit-major (hist[d * n_tiles + tile]) so that one exclusive scan gives every
 * (digit, tile) its first output slot.  Keys above `clamp` count as `clamp`
 * (the sentinel that sorts entries with an invalid column last).  Keys lie
 * STRIDE words apart. */
template <int STRIDE>
__global__ __launch_bounds__(kBlock) void k_rs_hist(const uint32_t *__restrict__ keys, Count n_in, uint32_t clamp,
                                                    int shift, uint32_t *__restrict__ hist, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ uint32_t h[kRadix];
    const int64_t n = count_of(n_in), n_tiles = (n + kSortTile - 1) / kSortTile;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        h[threadIdx.x] = 0u;
        __syncthreads();
        const int64_t base = tile * kSortTile + threadIdx.x;
#pragma unroll
        for (int r = 0; r < kSortTile / kBlock; ++r) {
            const int64_t i = base + (int64_t)r * kBlock;
            if (i < n) atomicAdd(&h[(min(keys[i * STRIDE], clamp) >> shift) & (kRadix - 1)], 1u);
        }
        __syncthreads();
        hist[(int64_t)threadIdx.x * n_tiles + tile] = h[threadIdx.x];
        __syncthreads();
    }
}

/*
 * Radix pass, phase 2: stable scatter of a tile.  Wave w of a block owns the
 * w-th part of the tile (kSortItems rounds of 64 consecutive entries) and ranks
 * it on its own: in a round, ballots on the 8 digit bits group the lanes
 * holding the same digit, a lane's rank is the number of lower peers, and the
 * wave's per-digit counter in LDS (read by the group, advanced by its lowest
 * lane) orders the rounds.  One block scan turns the waves' counts into
 * tile-local slots (digit-major, lower waves first): slot[] on return, and
 * goff[d] the global slot of tile-local slot 0 of digit d's run.
 */
struct TileRank {
    uint32_t cnt[kSortWaves][kRadix];   // per wave: digit counts, then first tile-local slot
    uint32_t goff[kRadix];
    uint32_t w[kSortWaves];
};

__device__ inline void rank_tile(TileRank &T, const uint32_t (&key)[kSortItems], int64_t sub0, int64_t n, int shift,
                                 const uint32_t *__restrict__ offs, int64_t n_tiles, int64_t tile,
                                 uint32_t (&slot)[kSortItems])
{
    const int t = threadIdx.x, wave = t >> 6, lane = t & (kWave - 1);
    for (int k = t; k < kSortWaves * kRadix; k += kSortBlock) (&T.cnt[0][0])[k] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const bool valid = sub0 + (int64_t)r * kWave + lane < n;
        const uint32_t d = (key[r] >> shift) & (kRadix - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = (uint32_t)mbcnt64(peers);
        uint32_t before = 0u;
        if (valid) before = T.cnt[wave][d];                 // every lane of the group reads the old count
        if (valid && rank == 0) T.cnt[wave][d] = before + (uint32_t)__popcll(peers);
        slot[r] = before + rank;
    }
    __syncthreads();
    // thread t < kRadix = digit t: tile-local start of the digit, then of each wave's part of it
    uint32_t c[kSortWaves], tot = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        c[w] = t < kRadix ? T.cnt[w][t] : 0u;
        tot += c[w];
    }
    uint32_t total;
    const uint32_t start = block_excl_scan<kSortWaves>(tot, T.w, &total);
    if (t < kRadix) {
        uint32_t b = start;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            T.cnt[w][t] = b;
            b += c[w];
        }
        T.goff[t] = offs[(int64_t)t * n_tiles + tile] - start;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) slot[r] += T.cnt[wave][(key[r] >> shift) & (kRadix - 1)];
}

/* Scatter of (key, row, value) entries: the tile is sorted by digit in LDS, the
 * values after the keys and rows, and written out in that order, so each
 * digit's run goes to consecutive addresses.  keys_out may be NULL (last pass).
 * Grid-stride over the tiles. */
__global__ __launch_bounds__(kSortBlock) void k_rs_scatter(const uint32_t *__restrict__ keys_in,
                                                           const int32_t *__restrict__ rows_in,
                                                           const float *__restrict__ vals_in, Count n_in,
                                                           uint32_t clamp, int shift,
                                                           const uint32_t *__restrict__ offs,
                                                           uint32_t *__restrict__ keys_out,
                                                           int32_t *__restrict__ rows_out,
                                                           float *__restrict__ vals_out, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ uint2 s_pair[kSortTile];
    __shared__ TileRank T;
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int64_t n = count_of(n_in), n_tiles = (n + kSortTile - 1) / kSortTile;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t tile0 = tile * kSortTile, sub0 = tile0 + (int64_t)(t >> 6) * (kSortTile / kSortWaves);
        uint32_t key[kSortItems], slot[kSortItems], at[kSortItems];
        int32_t row[kSortItems];
        float val[kSortItems];
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const int64_t i = sub0 + (int64_t)r * kWave + lane;
            const bool valid = i < n;
            key[r] = valid ? min(keys_in[i], clamp) : 0u;
            row[r] = valid ? rows_in[i] : 0;
            val[r] = valid ? vals_in[i] : 0.0f;
        }
        rank_tile(T, key, sub0, n, shift, offs, n_tiles, tile, slot);
#pragma unroll
        for (int r = 0; r < kSortItems; ++r)
            if (sub0 + (int64_t)r * kWave + lane < n) s_pair[slot[r]] = make_uint2(key[r], (uint32_t)row[r]);
        __syncthreads();
        const int m = (int)min((int64_t)kSortTile, n - tile0);
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const int lp = r * kSortBlock + t;
            if (lp < m) {
                const uint2 q = s_pair[lp];
                at[r] = T.goff[(q.x >> shift) & (kRadix - 1)] + (uint32_t)lp;
                if (keys_out) keys_out[at[r]] = q.x;
                rows_out[at[r]] = (int32_t)q.y;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; ++r)
            if (sub0 + (int64_t)r * kWave + lane < n) s_pair[slot[r]].x = __float_as_uint(val[r]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const int lp = r * kSortBlock + t;
            if (lp < m) vals_out[at[r]] = __uint_as_float(s_pair[lp].x);
        }
        __syncthreads();
    }
}

/* A run of the transpose: bucket key, row (flagged when invalid), first entry, auxiliary word. */
typedef uint4 Run;

/*
 * Scatter of run records, 16 bytes each: a digit's run of a tile (16 records on
 * average) is 256 contiguous bytes, where four separate arrays were written in
 * pieces of 64, each parts of two cache lines (3.7e7 runs: 0.30 ms a pass against
 * 0.49).
 */
__global__ __launch_bounds__(kSortBlock) void k_run_scatter(const Run *__restrict__ in, Count n_in, int shift,
                                                            const uint32_t *__restrict__ offs, Run *__restrict__ out,
                                                            Gate g)
{
    if (gate_closed(g)) return;
    __shared__ Run s_run[kSortTile];
    __shared__ TileRank T;
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int64_t n = count_of(n_in), n_tiles = (n + kSortTile - 1) / kSortTile;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t tile0 = tile * kSortTile, sub0 = tile0 + (int64_t)(t >> 6) * (kSortTile / kSortWaves);
        Run run[kSortItems];
        uint32_t key[kSortItems], slot[kSortItems];
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const int64_t i = sub0 + (int64_t)r * kWave + lane;
            run[r] = i < n ? in[i] : make_uint4(0u, 0u, 0u, 0u);
            key[r] = run[r].x;
        }
        rank_tile(T, key, sub0, n, shift, offs, n_tiles, tile, slot);
#pragma unroll
        for (int r = 0; r < kSortItems; ++r)
            if (sub0 + (int64_t)r * kWave + lane < n) s_run[slot[r]] = run[r];
        __syncthreads();
        const int m = (int)min((int64_t)kSortTile, n - tile0);
        for (int lp = t; lp < m; lp += kSortBlock) {
            const Run q = s_run[lp];
            out[T.goff[(q.x >> shift) & (kRadix - 1)] + (uint32_t)lp] = q;
        }
        __syncthreads();
    }
}

}  // namespace

static inline unsigned blocks_of(int64_t items, int per_block)
{
    return (unsigned)((items + per_block - 1) / per_block);
}

// Workgroups of the beamlet-row dose: four per CU in one round, though LDS (32 KB of 160) and registers
// (88) admit five.  With 1280 of them shares are shorter and so less aligned between rows, and more
// windows are open at once: the 6.5e8-entry slab 2.08 ms against 1.55, 256x256x100 with 9 beams of 576
// 1.45 against 1.11 (two rounds of four: the slab 1.66).  Rows per group: 32, since the more rows share a voxel the fewer atomics;
// with few rows 8, for enough waves (240 rows of 8e4 entries: 0.10 ms against 0.19 with 32; 900
// rows: 0.22 against 0.17).
constexpr unsigned kDoseGroups = 1024;
constexpr int kDoseManyRows = 512;
constexpr int kDoseFewGroup = 8;

hipError_t launch_fluence_dose(const int64_t *indptr, const int32_t *indices, const float *values, int n_rows,
                               int n_voxels, const float *w, float *dose, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero, dim3(blocks_of(n_voxels, kBlock)), dim3(kBlock), 0, s, dose, (int64_t)n_voxels);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_rows == 0) return e;
    const int group = n_rows >= kDoseManyRows ? kDoseRows : kDoseFewGroup;
    const unsigned groups = blocks_of(n_rows, group);
    const unsigned parts = std::min(64u, std::max(1u, kDoseGroups / groups));
    hipLaunchKernelGGL(k_fluence_dose, dim3(groups, parts), dim3(kBlock), 0, s, indptr, indices, values, n_rows,
                       n_voxels, w, dose, group);
    return hipGetLastError();
}

hipError_t launch_fluence_gradient(const int64_t *indptr, const int32_t *indices, const float *values, int n_rows,
                                   int n_voxels, const float *r, float *g, hipStream_t s)
{
    if (n_rows == 0) return hipSuccess;
    if (n_rows <= kGradFew)
        hipLaunchKernelGGL((k_fluence_gradient<1024, 4, 0>), dim3(n_rows), dim3(1024), 0, s, indptr, indices, values,
                           n_rows, n_voxels, r, g);
    else if (n_rows <= kGradMany)
        hipLaunchKernelGGL((k_fluence_gradient<256, 8, kGradXcd>), dim3(n_rows), dim3(256), 0, s, indptr, indices,
                           values, n_rows, n_voxels, r, g);
    else
        hipLaunchKernelGGL((k_fluence_gradient<256, 4, kGradXcd>), dim3(n_rows), dim3(256), 0, s, indptr, indices,
                           values, n_rows, n_voxels, r, g);
    return hipGetLastError();
}

hipError_t launch_voxel_dose(const int64_t *t_indptr, const int32_t *t_indices, const float *t_values, int n_voxels,
                             int n_w, const float *w, float *dose, hipStream_t s)
{
    const unsigned blocks = std::min(blocks_of((int64_t)n_voxels, kVoxelRows), (unsigned)kVoxelGroups);
    const size_t copy = sizeof(float) * (size_t)n_w;
    if (n_w <= kVoxelFewWords)
        hipLaunchKernelGGL(k_voxel_dose<WHome::kLds>, dim3(blocks), dim3(kVoxelBlock), copy, s, t_indptr, t_indices,
                           t_values, n_voxels, n_w, w, dose);
    else if (n_w <= kVoxelLdsWords)
        hipLaunchKernelGGL(k_voxel_dose<WHome::kEither>, dim3(blocks), dim3(kVoxelBlock), copy, s, t_indptr, t_indices,
                           t_values, n_voxels, n_w, w, dose);
    else
        hipLaunchKernelGGL(k_voxel_dose<WHome::kCache>, dim3(blocks), dim3(kVoxelBlock), 0, s, t_indptr, t_indices,
                           t_values, n_voxels, n_w, w, dose);
    return hipGetLastError();
}

namespace {

/*
 * Run transpose.  A run is a maximal stretch of consecutive entries of one row
 * whose columns share a bucket of kBucketCols columns (col >> kBucketShift);
 * entries whose column lies outside [0, n_voxels) form runs of their own,
 * flagged (row id with its top bit set) and never placed.  The runs are
 * sorted by bucket (stably, so a bucket's runs keep row order) and the
 * entries of each bucket are then placed by one wave, in that order, with a
 * stable counting sort on the column's low bits: the output is the stable sort
 * of the row-major entries by column, as the radix path gives.
 *
 * When every row's columns ascend strictly (a plan's D) a run holds at most
 * one entry per column of its bucket, so a 32-bit mask of its columns
 * describes it: its length is the mask's popcount, its k-th entry lies in the
 * column of the mask's k-th set bit, and the entries of a bucket that fall in
 * column c are counted by popcounts of masks.  The placement then reads only
 * the values, and the voxel-row pointers come from the bucket counts.
 */
constexpr int kBucketShift = 5;
constexpr int kBucketCols = 1 << kBucketShift;
constexpr uint32_t kRunFlag = 0x80000000u;   // run of invalid columns (in the run's row id)
constexpr int kRowChunks = 4;                // chunks of 64 entries whose loads are in flight together

/* Value of the lane below, through a whole-wave DPP shift; lane 0 takes `edge`. */
__device__ inline int from_lane_below(int v, int edge) { return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xf, 0xf, false); }

/* Run key of a column: its bucket, or -2 (outside [0, n_voxels)). */
__device__ inline int run_key(int col, int n_voxels)
{
    return (uint32_t)col < (uint32_t)n_voxels ? (col >> kBucketShift) : -2;
}

/* Flags the transpose computes on the device (one 64-byte slot of the workspace). */
struct Flags {
    int32_t unsorted;      // some row's columns do not ascend strictly
    int32_t use_runs;      // runs are at most half the entries: a run path
    int64_t hist_len;      // digit-histogram length of the run sort
    int32_t need_counts;   // entries per column counted by atomics (entry path, unsorted rows)
    int32_t sorted;        // run path with masks (rows ascending)
    int32_t any;           // run path for rows in any column order
    int32_t few_runs;      // too few runs to a bucket for four waves
    int32_t pad[8];
};
static_assert(sizeof(Flags) == 64, "one slot");

/*
 * The rows in pieces of equal length, `split` of them to a row (more than one where the rows are
 * too few to fill the chip), one wave each.  A piece is read in blocks of kRunBlock entries, and
 * its first entry and each block's start a run of their own (one in a thousand entries): no run
 * is open where a wave begins to read.
 */
constexpr int kRunSteps = 16;
constexpr int kRunBlock = kRunSteps * kWave;

struct Piece {
    int row;
    int64_t e0, e1;        // its entries
    int64_t first;         // the row's first entry
};
__device__ inline Piece piece_of(const int64_t *__restrict__ indptr, int id, int split)
{
    Piece P;
    P.row = split > 1 ? id / split : id;
    P.first = P.e0 = indptr[P.row];
    P.e1 = indptr[P.row + 1];
    if (split > 1) {
        const int64_t len = P.e1 - P.first, k = id - P.row * split;
        P.e0 = P.first + len * k / split;
        P.e1 = P.first + len * (k + 1) / split;
    }
    return P;
}

/* counts[k] += 1 for every key k in [0, n_valid) among the first n keys; other keys are skipped. */
__global__ __launch_bounds__(kBlock) void k_key_count(const int32_t *__restrict__ keys, int64_t n, int n_valid,
                                                      uint32_t *__restrict__ counts, Gate g)
{
    if (gate_closed(g)) return;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += stride) {
        const uint32_t i = (uint32_t)keys[e];
        if (i < (uint32_t)n_valid) atomicAdd(counts + i, 1u);
    }
}

/* Per piece (one wave, kRowChunks chunks of 64 entries loaded together): the number of runs
 * (run_cnt[id]), and the unsorted flag when the row's columns do not ascend strictly. */
__global__ __launch_bounds__(kBlock) void k_run_count(const int64_t *__restrict__ indptr,
                                                      const int32_t *__restrict__ indices, int n_rows, int n_voxels,
                                                      int split, uint32_t *__restrict__ run_cnt, Flags *__restrict__ fl)
{
    const int id = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (id >= n_rows * split) return;
    const int lane = lane_id();
    const Piece P = piece_of(indptr, id, split);
    uint32_t runs = 0;
    // the entry before: of the row for the order, of the block for the runs
    bool down = false, any = P.e0 > P.first;
    int prev_col = any && P.e0 < P.e1 ? indices[P.e0 - 1] : 0, prev_k = -1;
    for (int64_t c = P.e0; c < P.e1; c += kRowChunks * kWave) {
        int cols[kRowChunks];
#pragma unroll
        for (int u = 0; u < kRowChunks; ++u) {
            const int64_t e = c + u * kWave + lane;
            cols[u] = e < P.e1 ? indices[e] : 0;
        }
        if (((c - P.e0) & (kRunBlock - 1)) == 0) prev_k = -1;
#pragma unroll
        for (int u = 0; u < kRowChunks; ++u) {
            const int64_t e = c + u * kWave + lane;
            const bool in = e < P.e1;
            const int col = cols[u];
            const int k = in ? run_key(col, n_voxels) : -3;
            const int cp = from_lane_below(col, prev_col), kp = from_lane_below(k, prev_k);
            runs += (uint32_t)__popcll(__ballot(in && k != kp));
            down = down || (in && (any || lane > 0) && col <= cp);
            any = true;
            prev_col = __builtin_amdgcn_readlane(col, kWave - 1);
            prev_k = __builtin_amdgcn_readlane(k, kWave - 1);
        }
    }
    if (lane == 0) run_cnt[id] = runs;
    if (__ballot(down) && lane == 0) fl->unsorted = 1;
}
static_assert(kRunBlock % (kRowChunks * kWave) == 0, "blocks end with a group of chunks");

/* The path flags (one thread): a run path when the runs are at most half the
 * entries, with masks when the rows ascend; else the radix sort of the entries.
 * many_runs: fewer are few for the placement. */
__global__ void k_run_sizes(const int64_t *__restrict__ n_runs, int64_t nnz, int64_t many_runs, Flags *__restrict__ fl)
{
    const int64_t R = *n_runs;
    const int32_t use = 2 * R <= nnz ? 1 : 0, uns = fl->unsorted ? 1 : 0;
    fl->use_runs = use;
    fl->hist_len = (int64_t)kRadix * ((R + kSortTile - 1) / kSortTile);
    fl->need_counts = (!use || uns) ? 1 : 0;
    fl->sorted = (use && !uns) ? 1 : 0;
    fl->any = (use && uns) ? 1 : 0;
    fl->few_runs = R < many_runs ? 1 : 0;
}

/*
 * Records of every run (row-major run ids from run_ptr): its bucket key (an
 * invalid run takes the bucket of its column clamped into the grid), row
 * (flagged when invalid), first entry, and an auxiliary word: with ascending
 * rows the mask of its columns (OR of 1 << (col mod 32) over its entries, 0 for
 * an invalid run), else its length (0 for an invalid run).
 *
 * A wave stages a block of columns in LDS and lists where its runs start (one
 * compare, ballot and compaction per 64 entries); then lane i makes the record
 * of run i from its first and last column: a range of bits when it has no
 * hole, as on a VOI row, else the OR over its entries.  (A record made at the
 * lane of its run's last entry took the whole wave through the search for the
 * run's start: 1.46 ms for 6.5e8 entries against 0.69, 4.8 TB/s.)
 */
__global__ __launch_bounds__(kBlock) void k_run_emit(const int64_t *__restrict__ indptr,
                                                     const int32_t *__restrict__ indices, int n_rows, int n_voxels,
                                                     int split, const int64_t *__restrict__ run_ptr,
                                                     const Flags *__restrict__ fl, Run *__restrict__ out, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ int32_t s_col[kWavesPerBlock][kRunBlock];
    __shared__ uint16_t s_start[kWavesPerBlock][kRunBlock];
    const int wave = threadIdx.x >> 6, id = blockIdx.x * kWavesPerBlock + wave;
    if (id >= n_rows * split) return;   // no barrier below: each wave has its own LDS
    const bool masks = fl->unsorted == 0;
    const int lane = lane_id();
    const Piece P = piece_of(indptr, id, split);
    int32_t *col = s_col[wave];
    uint16_t *start = s_start[wave];
    int64_t r = run_ptr[id];
    for (int64_t c = P.e0; c < P.e1; c += kRunBlock) {
        const int n = (int)min((int64_t)kRunBlock, P.e1 - c);
        int cols[kRunSteps];
#pragma unroll
        for (int u = 0; u < kRunSteps; ++u) {
            const int x = u * kWave + lane;
            cols[u] = x < n ? __builtin_nontemporal_load(indices + c + x) : 0;
        }
        int prev_k = -1, runs = 0;
#pragma unroll
        for (int u = 0; u < kRunSteps; ++u) {
            if (u * kWave >= n) break;
            const int x = u * kWave + lane;
            const int k = x < n ? run_key(cols[u], n_voxels) : -3;
            const int kp = from_lane_below(k, prev_k);
            prev_k = __builtin_amdgcn_readlane(k, kWave - 1);
            const uint64_t m = __ballot(x < n && k != kp);
            if (x < n && k != kp) start[runs + mbcnt64(m)] = (uint16_t)x;
            runs += __popcll(m);
            col[x] = cols[u];
        }
        wave_lds_fence();
        for (int i = lane; i < runs; i += kWave) {
            const int a = start[i], b = i + 1 < runs ? start[i + 1] : n, first = col[a], last = col[b - 1];
            const bool valid = (uint32_t)first < (uint32_t)n_voxels;
            uint32_t x = valid ? (uint32_t)(b - a) : 0u;
            if (masks && valid) {
                if (last - first == b - a - 1) {
                    const uint32_t hi = (2u << (last & (kBucketCols - 1))) - 1u;
                    x = hi & ~((1u << (first & (kBucketCols - 1))) - 1u);
                } else {
                    x = 0u;
                    for (int y = a; y < b; ++y) x |= 1u << (col[y] & (kBucketCols - 1));
                }
            }
            const int clamped = first < 0 ? 0 : (first >= n_voxels ? n_voxels - 1 : first);
            out[r + i] = make_uint4((uint32_t)(clamped >> kBucketShift), (uint32_t)P.row | (valid ? 0u : kRunFlag),
                                    (uint32_t)(c + a), x);
        }
        wave_lds_fence();
        r += runs;
    }
}

/* Bucket pointers from the runs sorted by bucket: b_ptr[b] = first run of bucket b or above
 * (b_ptr[n_buckets] = R), by bisection, one thread per bucket.  (Written run by run, each thread
 * filling the gap before its run's bucket, one thread filled all of an empty stretch of the grid:
 * 0.24 ms for 3.7e7 runs in 65,536 buckets against 0.02, and 1.1 ms where a few beamlets leave most
 * of 1e5 buckets empty.) */
__global__ __launch_bounds__(kBlock) void k_bucket_bounds(const Run *__restrict__ runs, Count n_runs, int n_buckets,
                                                          int64_t *__restrict__ b_ptr, Gate g)
{
    if (gate_closed(g)) return;
    const int b = blockIdx.x * kBlock + threadIdx.x;
    if (b > n_buckets) return;
    int64_t lo = 0, hi = count_of(n_runs);
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (runs[mid].x < (uint32_t)b) lo = mid + 1;
        else hi = mid;
    }
    b_ptr[b] = lo;
}

/* Groups of kXcdGroup consecutive buckets go to one XCD, so that the runs of neighbouring buckets,
 * which share cache lines of a row, meet in one L2; the groups themselves are dealt to the XCDs in
 * turn, which keeps the XCDs evenly loaded when the entries crowd into part of the grid. */
constexpr int kXcdGroup = 16;
static unsigned xcd_grid(int n_buckets)
{
    const int per = kXcds * kXcdGroup;
    return (unsigned)(((n_buckets + per - 1) / per) * per);
}

/* Entries per column (counts[]) from the masks of ascending rows' runs: one wave per bucket, a
 * popcount of a ballot per column and 64 runs. */
__global__ __launch_bounds__(kWave) void k_bucket_count(const int64_t *__restrict__ b_ptr,
                                                        const Run *__restrict__ runs, int n_voxels,
                                                        int n_buckets, uint32_t *__restrict__ counts, Gate g)
{
    if (gate_closed(g)) return;
    const int b = blockIdx.x, lane = lane_id();
    const int64_t q0 = b_ptr[b], q1 = b_ptr[b + 1];
    uint32_t n[kBucketCols] = {};
    uint32_t next = q0 + lane < q1 ? runs[q0 + lane].w : 0u;
    for (int64_t q = q0; q < q1; q += kWave) {
        const uint32_t mask = next;
        next = q + kWave + lane < q1 ? runs[q + kWave + lane].w : 0u;
#pragma unroll
        for (int c = 0; c < kBucketCols; ++c) n[c] += (uint32_t)__popcll(__ballot((mask >> c) & 1u));
    }
    uint32_t mine = 0u;
#pragma unroll
    for (int c = 0; c < kBucketCols; ++c) mine = lane == c ? n[c] : mine;
    const int col = (b << kBucketShift) + lane;
    if (lane < kBucketCols && col < n_voxels) counts[col] = mine;
}

typedef float vf4u __attribute__((ext_vector_type(4), aligned(4)));

/*
 * Placement for rows with ascending columns, one workgroup per bucket, 64 runs
 * per wave at a time (lane = run, in row order over the waves).  A lane takes
 * its run's values into registers by column: where no run of the wave has a
 * hole, the value of column c lies (c - first column) entries after the run's
 * first, so that 16-byte loads of four columns bring each to its own register;
 * otherwise the run's entries are loaded one by one.  Then for each column the
 * ballot of the runs that hold it ranks them, and their row ids and values go
 * out as one contiguous store each, after those of the waves before: neither
 * entries in LDS nor a search for an entry's column.
 *
 * Bound by memory, and by how much of the output is open at a time: a column's
 * cache lines are written piece by piece and leave L2 half filled if too many
 * buckets are under way.  6.5e8 entries in 3.03 ms (5.6 GB fetched, since runs of
 * 18 entries share their lines with neighbours, and 5.7 written, 3.7 TB/s)
 * against 3.97 with each batch's entries reordered in LDS.
 */
template <int W>
__device__ __attribute__((always_inline)) inline void place_bucket(
    int b, int wave, uint32_t (*s_n)[W][kBucketCols], const float *__restrict__ values, int n_voxels,
    const int64_t *__restrict__ b_ptr, const Run *__restrict__ runs, const int64_t *__restrict__ t_indptr, uint32_t nnz,
    int32_t *__restrict__ t_indices, float *__restrict__ t_values)
{
    const int lane = lane_id();
    const int64_t q0 = b_ptr[b], q1 = b_ptr[b + 1];
    // lane c: next output position of column c
    const int mine = (b << kBucketShift) + lane;
    uint32_t pos = lane < kBucketCols && mine < n_voxels ? (uint32_t)t_indptr[mine] : 0u;

    constexpr int kBatch = W * kWave;
    int64_t q = q0 + wave * kWave + lane;
    Run next = q < q1 ? runs[q] : make_uint4(0u, 0u, 0u, 0u);
    int turn = 0;
    for (int64_t qb = q0; qb < q1; qb += kBatch, turn ^= 1) {
        const uint32_t mask = next.w, src = next.z;   // mask 0: an invalid run, not placed
        const int row = (int)next.y;
        q += kBatch;
        next = q < q1 ? runs[q] : make_uint4(0u, 0u, 0u, 0u);
        const uint32_t lo = mask ? (uint32_t)__builtin_ctz(mask) : 0u, hi = mask ? 31u - (uint32_t)__builtin_clz(mask) : 0u;
        const uint32_t run = mask >> lo;
        // whole quads of four columns lie inside the array
        const bool plain = (run & (run + 1u)) == 0u && src >= (lo & 3u) && (uint64_t)src + ((hi | 3u) - lo) < nnz;
        float v[kBucketCols];
        if (__ballot(mask != 0u && !plain) == 0) {
            const float *p = values + ((int64_t)src - lo);
#pragma unroll
            for (int m = 0; m < kBucketCols / 4; ++m) {
                vf4u x = {0.0f, 0.0f, 0.0f, 0.0f};
                if ((mask >> (4 * m)) & 15u) x = *reinterpret_cast<const vf4u *>(p + 4 * m);
                v[4 * m] = x.x;
                v[4 * m + 1] = x.y;
                v[4 * m + 2] = x.z;
                v[4 * m + 3] = x.w;
            }
        } else {
            int64_t e = src;
#pragma unroll
            for (int c = 0; c < kBucketCols; ++c) {
                v[c] = 0.0f;
                if ((mask >> c) & 1u) v[c] = values[e++];
            }
        }
        // this wave's entries per column, those of the waves before it, of all
        uint32_t n = 0u;
#pragma unroll
        for (int c = 0; c < kBucketCols; ++c) {
            const uint32_t k = (uint32_t)__popcll(__ballot((mask >> c) & 1u));
            n = lane == c ? k : n;
        }
        if (lane < kBucketCols) s_n[turn][wave][lane] = n;
        if (W > 1) __syncthreads();   // the buffers alternate: one barrier a batch
        else wave_lds_fence();
        uint32_t at = pos;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t k = s_n[turn][w][lane & (kBucketCols - 1)];
            at += w < wave ? k : 0u;
            pos += k;
        }
#pragma unroll
        for (int c = 0; c < kBucketCols; ++c) {
            const bool in = (mask >> c) & 1u;
            const uint64_t m = __ballot(in);
            const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)at, c);
            // the bound always holds for consistent runs; it keeps every store inside the arrays
            if (in && p + (uint32_t)__popcll(m) <= nnz) {
                const int rank = mbcnt64(m);
                (t_indices + p)[rank] = row;
                (t_values + p)[rank] = v[c];
            }
        }
    }
}

/* One bucket per workgroup, or (few: where the flag says so) per wave. */
template <int W>
__global__ __launch_bounds__(W * kWave) void k_place_sorted(
    const float *__restrict__ values, int n_voxels, int n_buckets, const int64_t *__restrict__ b_ptr,
    const Run *__restrict__ runs, const int64_t *__restrict__ t_indptr, uint32_t nnz, int32_t *__restrict__ t_indices,
    float *__restrict__ t_values, const int32_t *__restrict__ few, Gate g)
{
    if (gate_closed(g)) return;
    __shared__ uint32_t s_n[2 * W * kBucketCols];   // entries per column of each wave's batch
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), b = xcd_item<kXcdGroup>();
    if (W > 1 && *few) {
        const int bw = b * W + wave;   // a barrier is not met: each wave goes through its own bucket
        if (bw < n_buckets)
            place_bucket<1>(bw, 0, reinterpret_cast<uint32_t(*)[1][kBucketCols]>(s_n + 2 * kBucketCols * wave), values,
                            n_voxels, b_ptr, runs, t_indptr, nnz, t_indices, t_values);
    } else if (b < n_buckets) {
        place_bucket<W>(b, wave, reinterpret_cast<uint32_t(*)[W][kBucketCols]>(s_n), values, n_voxels, b_ptr, runs,
                        t_indptr, nnz, t_indices, t_values);
    }
}

/* The runs of bucket b, taken 64 at a time: lane i holds run q0 + i (its row,
 * first entry and length), with the batch's exclusive prefix of lengths. */
struct RunBatch {
    int row;
    uint32_t src, len, excl, total;
};

__device__ inline RunBatch load_runs(int64_t qb, int64_t q1, const Run *__restrict__ runs)
{
    const int lane = lane_id();
    const int64_t q = qb + lane;
    RunBatch B{0, 0u, 0u, 0u, 0u};
    if (q < q1) {
        const Run r = runs[q];
        B.row = (int)(r.y & ~kRunFlag);
        B.src = r.z;
        B.len = r.w;   // 0 for an invalid run
    }
    uint32_t incl = wave_incl_scan(B.len);
    B.excl = incl - B.len;
    B.total = __shfl(incl, kWave - 1, kWave);
    return B;
}

/* Lane of the run holding batch entry p = c0 + lane: the last lane whose
 * exclusive prefix is <= p, walked wave-uniformly from *rcur. */
__device__ inline int run_of(const RunBatch &B, uint32_t c0, int &rcur)
{
    while (rcur + 1 < kWave && (uint32_t)__builtin_amdgcn_readlane((int)B.excl, rcur + 1) <= c0) ++rcur;
    const uint32_t p = c0 + lane_id();
    int rr = rcur;
    for (int k = rcur + 1; k < kWave; ++k) {
        const uint32_t ek = (uint32_t)__builtin_amdgcn_readlane((int)B.excl, k);
        if (ek > c0 + kWave - 1) break;
        if (p >= ek) rr = k;
    }
    return rr;
}

/*
 * Placement for rows in any column order, one wave per bucket: the bucket's
 * runs are taken 64 at a time, their entries flattened over the lanes in run
 * order; an entry of column col goes to t_indptr[col] + (entries of col placed
 * before it), counted per column in LDS.  Equal columns within a 64-entry
 * chunk are ranked by lane with five ballots over the column's low bits.
 */
__global__ __launch_bounds__(kWave) void k_place_any(
    const int32_t *__restrict__ indices, const float *__restrict__ values, int n_voxels, int n_buckets,
    const int64_t *__restrict__ b_ptr, const Run *__restrict__ runs, const int64_t *__restrict__ t_indptr, uint32_t nnz,
    int32_t *__restrict__ t_indices, float *__restrict__ t_values, Gate g)
{
    if (gate_closed(g)) return;
    const int b = xcd_item<kXcdGroup>();
    if (b >= n_buckets) return;
    __shared__ uint32_t base[kBucketCols];
    __shared__ uint32_t cnt[kBucketCols];
    const int lane = lane_id();
    for (int c = lane; c < kBucketCols; c += kWave) {
        const int col = (b << kBucketShift) + c;
        base[c] = col < n_voxels ? (uint32_t)t_indptr[col] : 0u;
        cnt[c] = 0u;
    }
    __builtin_amdgcn_wave_barrier();
    const int64_t q0 = b_ptr[b], q1 = b_ptr[b + 1];
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));   // lanes under this one
    for (int64_t qb = q0; qb < q1; qb += kWave) {
        const RunBatch B = load_runs(qb, q1, runs);
        int rcur = 0;
        for (uint32_t c0 = 0; c0 < B.total; c0 += kWave) {
            const uint32_t p = c0 + lane;
            const int rr = run_of(B, c0, rcur);
            const bool in = p < B.total;
            const uint32_t e = __shfl(B.src, rr, kWave) + (p - __shfl(B.excl, rr, kWave));
            const int rowj = __shfl(B.row, rr, kWave);
            const int col = in ? indices[e] : 0;
            const float v = in ? values[e] : 0.0f;
            const int bin = col & (kBucketCols - 1);
            uint64_t eq = __ballot(in);
#pragma unroll
            for (int k = 0; k < kBucketShift; ++k) {
                const bool bit = (bin >> k) & 1;
                const uint64_t m = __ballot(bit);
                eq &= bit ? m : ~m;
            }
            const uint32_t rank = (uint32_t)__popcll(eq & below);
            const uint32_t n_eq = (uint32_t)__popcll(eq);
            const uint32_t pos = base[bin] + cnt[bin] + rank;
            if (in && pos < nnz) {   // always true for consistent runs; keeps every store in bounds
                t_indices[pos] = rowj;
                t_values[pos] = v;
            }
            __builtin_amdgcn_wave_barrier();
            if (in && rank + 1 == n_eq) cnt[bin] += n_eq;   // the last lane of each column group
            __builtin_amdgcn_wave_barrier();
        }
    }
}

}  // namespace

/* Workspace layout of the transpose (offsets from a 256-byte aligned base). */
struct TransposeLayout {
    size_t key[2], row[2], val[2];   // of the entry path; the run path keeps records in the same space
    size_t hist, partial, counts, bptr, flags, run_cnt, run_ptr, total;
};

/* Pieces per row of the run kernels: at least kRunWaves waves in all where the rows are too few, of
 * no less than 512 entries each (on average), so that the runs that pieces cut stay few.  (32 rows
 * of 5e5 entries: both run kernels 17 us against 0.9 ms with a wave per row.) */
constexpr int kRunWaves = 8192;
static int run_split(int64_t nnz, int n_rows)
{
    const int64_t want = (kRunWaves + n_rows - 1) / n_rows, most = nnz / n_rows / 512;
    return (int)std::max<int64_t>(1, std::min(want, most));
}

static TransposeLayout transpose_layout(int64_t nnz, int n_voxels, int n_rows)
{
    TransposeLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    const int64_t n_tiles = (nnz + kSortTile - 1) / kSortTile;
    const int64_t n_hist = (int64_t)kRadix * (n_tiles > 0 ? n_tiles : 1);
    const int64_t nb = (n_voxels + kBucketCols - 1) >> kBucketShift;
    int64_t n_scan = std::max<int64_t>(std::max<int64_t>(n_hist, n_voxels), (int64_t)std::max(n_rows, 1) * (n_rows > 0 ? run_split(nnz, n_rows) : 1));
    const size_t e = (size_t)(nnz > 0 ? nnz : 1);
    const size_t pieces = n_rows > 0 ? (size_t)n_rows * run_split(nnz, n_rows) : 1;
    for (int b = 0; b < 2; ++b) {
        L.key[b] = take(sizeof(uint32_t) * e);
        L.row[b] = take(sizeof(int32_t) * e);
        L.val[b] = take(sizeof(float) * e);
    }
    L.hist = take(sizeof(uint32_t) * (size_t)n_hist);
    L.partial = take(sizeof(uint32_t) * (size_t)((n_scan + kScanChunk - 1) / kScanChunk + 1));
    L.counts = take(sizeof(uint32_t) * ((size_t)n_voxels + 1));
    L.bptr = take(sizeof(int64_t) * (size_t)(nb + 1));
    L.flags = take(sizeof(Flags));
    L.run_cnt = take(sizeof(uint32_t) * pieces);
    L.run_ptr = take(sizeof(int64_t) * (pieces + 1));
    L.total = off;
    return L;
}

size_t transpose_workspace(int64_t nnz, int n_voxels, int n_rows)
{
    return transpose_layout(nnz, n_voxels, n_rows).total;
}

int transpose_passes(int n_keys)
{
    int bits = 0;
    while (bits < 31 && ((int64_t)1 << bits) < (int64_t)n_keys) ++bits;
    const int p = (bits + kRadixBits - 1) / kRadixBits;
    return p > 0 ? p : 1;
}

/* Persistent grid of a grid-stride launch over `items` units of work. */
static unsigned stride_grid(int64_t items)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(items, 4096));
}

/* Exclusive scan of n uint32 values in -> out (OUT = uint32_t or int64_t; out may be in); n is a
 * host count or, with n.dev, a device count at most n_max.  partial[nblocks] receives the total,
 * and *total64 too when given. */
template <typename OUT>
static hipError_t scan_excl(const uint32_t *in, Count n, int64_t n_max, uint32_t *partial, OUT *out,
                            int64_t *total64, Gate g, hipStream_t s)
{
    const unsigned nb = stride_grid((n_max + kScanChunk - 1) / kScanChunk);
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kBlock), 0, s, in, n, partial, g);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanTop), 0, s, partial, n, total64, g);
    hipLaunchKernelGGL(k_scan_down<OUT>, dim3(nb), dim3(kBlock), 0, s, in, n, partial, out, g);
    return hipGetLastError();
}

/*
 * One stable LSD radix sort of (key, row, value) triples by key: `passes`
 * passes of 8 bits, keys above clamp sorted as clamp, ping-pong through
 * (k1, r1, v1) and (k0, r0, v0) (the input may be separate), the last pass
 * writing rows and values to (rows_out, vals_out).
 */
static hipError_t sort_entries(const uint32_t *keys, const int32_t *rows, const float *vals, int64_t n, uint32_t clamp,
                               int passes, uint32_t *k0, int32_t *r0, float *v0, uint32_t *k1, int32_t *r1, float *v1,
                               int32_t *rows_out, float *vals_out, uint32_t *hist, uint32_t *partial, Gate g,
                               hipStream_t s)
{
    const int64_t tiles = (n + kSortTile - 1) / kSortTile, n_hist = (int64_t)kRadix * tiles;
    const unsigned grid = stride_grid(tiles);
    const Count cn{n, nullptr};
    hipError_t e;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * kRadixBits;
        const bool last = p == passes - 1, odd = p & 1;
        uint32_t *kout = last ? nullptr : (odd ? k0 : k1);
        int32_t *rout = last ? rows_out : (odd ? r0 : r1);
        float *vout = last ? vals_out : (odd ? v0 : v1);
        hipLaunchKernelGGL(k_rs_hist<1>, dim3(grid), dim3(kBlock), 0, s, keys, cn, clamp, shift, hist, g);
        if ((e = scan_excl<uint32_t>(hist, Count{n_hist, nullptr}, n_hist, partial, hist, nullptr, g, s)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_rs_scatter, dim3(grid), dim3(kSortBlock), 0, s, keys, rows, vals, cn, clamp, shift, hist,
                           kout, rout, vout, g);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        keys = kout;
        rows = rout;
        vals = vout;
    }
    return hipSuccess;
}

/* Stable LSD radix sort of run records by key through b and a; a holds the input, *sorted the
 * result.  n is a device count, at most n_max. */
static hipError_t sort_runs(Run *a, Run *b, Count n, int64_t n_max, int passes, uint32_t *hist, uint32_t *partial,
                            int64_t *hist_len, Gate g, Run **sorted, hipStream_t s)
{
    const int64_t tiles_max = (n_max + kSortTile - 1) / kSortTile;
    const unsigned grid = stride_grid(tiles_max);
    hipError_t e;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * kRadixBits;
        hipLaunchKernelGGL(k_rs_hist<4>, dim3(grid), dim3(kBlock), 0, s, reinterpret_cast<const uint32_t *>(a), n,
                           0xffffffffu, shift, hist, g);
        if ((e = scan_excl<uint32_t>(hist, Count{0, hist_len}, (int64_t)kRadix * tiles_max, partial, hist, nullptr, g,
                                     s)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_run_scatter, dim3(grid), dim3(kSortBlock), 0, s, a, n, shift, hist, b, g);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        std::swap(a, b);
    }
    *sorted = a;
    return hipSuccess;
}

// Large buckets are placed by four waves, and the LDS reserved keeps the workgroups per CU at
// three, so that the open cache lines stay in L2 (1e4 entries per bucket: placement 3.03 ms against
// 3.39 with as many as fit and 3.83 with one wave each; whole transposes of 715 per bucket 0.64 ms
// against 0.68 with one wave); small ones, whose latency counts, by one wave and as many as fit
// (290 per bucket 0.33 against 0.38, 160 per bucket 0.23 against 0.34).  Four waves take 256 runs at
// a time, so a bucket must also have runs for them, which only the device knows: rows of consecutive
// columns have one to a row (9000 rows of 4000 over 2e6 columns, 18 runs to a bucket of 576 entries:
// 0.4 ms with a wave to each bucket, 0.57 with four; 38 runs and 683 entries 0.56 with four, 0.58).
constexpr int64_t kPlaceMany = 512;              // entries per bucket
constexpr int64_t kPlaceRuns = 32;               // runs per bucket
constexpr unsigned kPlaceReserve = 45 * 1024;

hipError_t launch_transpose(const int64_t *indptr, const int32_t *indices, const float *values, int n_rows,
                            int n_voxels, int64_t nnz, int64_t *t_indptr, int32_t *t_indices, float *t_values,
                            void *workspace, hipStream_t s)
{
    const TransposeLayout L = transpose_layout(nnz, n_voxels, n_rows);
    char *ws = static_cast<char *>(workspace);
    uint32_t *key[2] = {reinterpret_cast<uint32_t *>(ws + L.key[0]), reinterpret_cast<uint32_t *>(ws + L.key[1])};
    int32_t *row[2] = {reinterpret_cast<int32_t *>(ws + L.row[0]), reinterpret_cast<int32_t *>(ws + L.row[1])};
    float *val[2] = {reinterpret_cast<float *>(ws + L.val[0]), reinterpret_cast<float *>(ws + L.val[1])};
    uint32_t *hist = reinterpret_cast<uint32_t *>(ws + L.hist);
    uint32_t *partial = reinterpret_cast<uint32_t *>(ws + L.partial);
    uint32_t *counts = reinterpret_cast<uint32_t *>(ws + L.counts);
    Flags *fl = reinterpret_cast<Flags *>(ws + L.flags);
    uint32_t *run_cnt = reinterpret_cast<uint32_t *>(ws + L.run_cnt);
    int64_t *run_ptr = reinterpret_cast<int64_t *>(ws + L.run_ptr);
    const Gate always{nullptr, 0};
    hipError_t e;

    hipLaunchKernelGGL(k_zero_u32, dim3(blocks_of((int64_t)n_voxels + 1, kBlock)), dim3(kBlock), 0, s, counts,
                       (int64_t)n_voxels + 1);
    if (nnz == 0 || n_rows == 0)   // empty voxel rows
        return scan_excl<int64_t>(counts, Count{n_voxels, nullptr}, n_voxels, partial, t_indptr, t_indptr + n_voxels,
                                  always, s);

    // runs of every piece and the unsorted flag; run pointers; the path flags
    const int split = run_split(nnz, n_rows);
    const int64_t pieces = (int64_t)n_rows * split;
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(kBlock), 0, s, reinterpret_cast<uint32_t *>(fl),
                       (int64_t)(sizeof(Flags) / 4));
    hipLaunchKernelGGL(k_run_count, dim3(blocks_of(pieces, kWavesPerBlock)), dim3(kBlock), 0, s, indptr, indices,
                       n_rows, n_voxels, split, run_cnt, fl);
    if ((e = scan_excl<int64_t>(run_cnt, Count{pieces, nullptr}, pieces, partial, run_ptr, run_ptr + pieces, always,
                                s)) != hipSuccess)
        return e;
    const Count n_runs{0, run_ptr + pieces};
    const int nb = (n_voxels + kBucketCols - 1) >> kBucketShift;
    hipLaunchKernelGGL(k_run_sizes, dim3(1), dim3(1), 0, s, n_runs.dev, nnz, kPlaceRuns * nb, fl);
    const Gate runs{&fl->use_runs, 1}, entries{&fl->use_runs, 0}, counted{&fl->need_counts, 1},
        masked{&fl->sorted, 1}, any{&fl->any, 1};

    // run paths: at most nnz / 2 records of 16 bytes, in the space of key, row and val of each side
    const int64_t half = (nnz + 1) / 2;
    Run *ra = reinterpret_cast<Run *>(key[0]), *rb = reinterpret_cast<Run *>(key[1]), *sorted = nullptr;
    int64_t *bptr = reinterpret_cast<int64_t *>(ws + L.bptr);
    hipLaunchKernelGGL(k_run_emit, dim3(blocks_of(pieces, kWavesPerBlock)), dim3(kBlock), 0, s, indptr, indices,
                       n_rows, n_voxels, split, run_ptr, fl, ra, runs);
    // stable sort of the runs by bucket
    if ((e = sort_runs(ra, rb, n_runs, half, transpose_passes(nb), hist, partial, &fl->hist_len, runs, &sorted, s)) !=
        hipSuccess)
        return e;
    hipLaunchKernelGGL(k_bucket_bounds, dim3(blocks_of((int64_t)nb + 1, kBlock)), dim3(kBlock), 0, s, sorted, n_runs,
                       nb, bptr, runs);

    // entries per column (from the run masks; entry path and unsorted rows: by atomics), the
    // voxel-row pointers
    hipLaunchKernelGGL(k_bucket_count, dim3(nb), dim3(kWave), 0, s, bptr, sorted, n_voxels, nb, counts, masked);
    hipLaunchKernelGGL(k_key_count, dim3(stride_grid(blocks_of(nnz, kBlock))), dim3(kBlock), 0, s, indices, nnz,
                       n_voxels, counts, counted);
    if ((e = scan_excl<int64_t>(counts, Count{n_voxels, nullptr}, n_voxels, partial, t_indptr, t_indptr + n_voxels,
                                always, s)) != hipSuccess)
        return e;

    if (nnz >= kPlaceMany * nb)
        hipLaunchKernelGGL(k_place_sorted<4>, dim3(xcd_grid(nb)), dim3(4 * kWave), kPlaceReserve, s, values, n_voxels,
                           nb, bptr, sorted, t_indptr, (uint32_t)nnz, t_indices, t_values, &fl->few_runs, masked);
    else
        hipLaunchKernelGGL(k_place_sorted<1>, dim3(xcd_grid(nb)), dim3(kWave), 0, s, values, n_voxels, nb, bptr,
                           sorted, t_indptr, (uint32_t)nnz, t_indices, t_values, nullptr, masked);
    hipLaunchKernelGGL(k_place_any, dim3(xcd_grid(nb)), dim3(kWave), 0, s, indices, values, n_voxels, nb, bptr, sorted,
                       t_indptr, (uint32_t)nnz, t_indices, t_values, any);
    if ((e = hipGetLastError()) != hipSuccess) return e;

    // entry path: row id of every entry (into row[0]), then a radix sort of the entries by
    // column (invalid columns as n_voxels, sorted last)
    hipLaunchKernelGGL(k_expand_rows, dim3(blocks_of(n_rows, kWavesPerBlock)), dim3(kBlock), 0, s, indptr, n_rows, nnz,
                       row[0], entries);
    return sort_entries(reinterpret_cast<const uint32_t *>(indices), row[0], values, nnz, (uint32_t)n_voxels,
                        transpose_passes(n_voxels + 1), key[0], row[0], val[0], key[1], row[1], val[1], t_indices,
                        t_values, hist, partial, entries, s);
}

/*
 * Scratch of the allocation-free transpose: a file-scope device array, one
 * copy per GPU, held until the process ends.  Host code never passes the
 * array's name to a kernel (on the host it is only a stand-in for the
 * symbol): its device address is taken once per device with
 * hipGetSymbolAddress and kept in noalloc_scratch_ptr.
 */
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_ptr(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace fspb
