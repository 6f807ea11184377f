// Both score passes of attn_mass.hip for launches that cannot fill the chip with its workgroups
// (few slices, short sequences; Section 2.4 Eq. (1), Section 4.2 Eq. (7)).
//
//   attn_lse_split_kernel     row log-sum-exps, L_t = log2 sum_j exp2(c s_tj)
//   attn_lse_split16_kernel, attn_colsum_split16_kernel  the same with 16 rows a workgroup, the smallest fp32 launches
//   attn_colsum_split_kernel  column sums, mass_j = sum_g sum_{t>=j} exp2(c s_tj - L_t)
//
// What bounds such a launch is the longest serial chain of a workgroup and the number of idle compute
// units, not a rate: 256 stationary rows per workgroup leave 128 workgroups for 32 slices of 1000
// tokens, and with G query heads per KV head the one workgroup of a key tile walks all G heads.
// Here a workgroup owns a QUARTER of the rows (32 per MFMA block, NBLK blocks: 64 rows, 32 for fp32),
// all its waves hold the same rows in registers and the streamed 32-row tiles are dealt to the waves
// in turn, so four times as many workgroups run and each wave's chain is 1/W as long.  Every wave has
// its own two LDS stages and waits for nobody until the partial results are combined through LDS
// in the order of the waves (deterministic).  Each wave reads its tiles for 64 stationary rows only,
// where a workgroup of attn_mass.hip reads them once for 256 (attn_pipe.hip: 512): four (eight) times the L2
// traffic, which is why full launches stay with those kernels (the rule is at attn_split_waves).
#include <algorithm>

#include "attn_tile.h"

namespace kvm {

// A wave's private stream: 32 rows of CHUNKS 16-byte chunks per stage, swizzled like Tile.
template <typename T> struct Stream {
    static constexpr int CH = Mma<T>::CHUNKS;
    static constexpr int SLOTS = 32 * CH;
    static constexpr int LOADS = SLOTS / WAVE;               // global_load_lds instructions per tile
    static constexpr int ROWS_PER_LOAD = WAVE / CH;
    // rows [row0, row0+32) of the matrix at `base`; rows past n_valid repeat the last valid one (row0 < n_valid)
    static __device__ __forceinline__ void issue(const T *base, int row0, int n_valid, u32x4 *stage, int lane) {
        const int last = n_valid - 1 - row0;
        const char *first_row = reinterpret_cast<const char *>(base + (size_t)row0 * HEAD_DIM);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int row = i * ROWS_PER_LOAD + lane / CH, pos = lane % CH;
            const uint32_t off = (uint32_t)(min(row, last) * (HEAD_DIM * (int)sizeof(T)) + ((pos ^ (row & (CH - 1))) * 16));
            __builtin_amdgcn_global_load_lds((gptr_t)(first_row + off), (lptr_t)(stage + i * WAVE), 16, 0, 0);
        }
    }
    static __device__ __forceinline__ u32x4 frag(const u32x4 *stage, int f, int lane) {
        const int row = lane & 31;
        return stage[row * CH + ((2 * f + (lane >> 5)) ^ (row & (CH - 1)))];
    }
};

// the wave's own tile has landed, and its LDS reads of the stage that is overwritten next are done
__device__ __forceinline__ void wait_own_tile() { __builtin_amdgcn_s_waitcnt(7 << 4); }   // vmcnt(0) lgkmcnt(0)

// The stationary rows [row0, row0 + 32 NBLK) of a workgroup, which all its waves hold: once from memory into LDS, the loads dealt to the
// waves, and from there into every wave's registers.  (Straight from memory a fragment is 16 bytes of each of 32 rows, which the path to
// the caches serves at 17 bytes a cycle and compute unit instead of 60, and every wave would ask for all of them.)  `space`: 1024 slots that
// no load is under way to; the caller puts a barrier between this and the first load into them.  Rows past n_valid repeat the last valid one.
// us, both passes, fragments from memory by every wave / this: 8 slices of 4096 tokens 61.7 / 52.2, 32 of them 189 / 172, 32 ragged ones of up to
// 1000 23.4 / 19.7, 16 of them, G = 4, 40.5 / 34.7, one of 16384 132 / 129; fp32: 8 of up to 2000 89 / 88.
template <typename T, int W>
__device__ __forceinline__ void issue_stationary(const T *base, int row0, int n_valid, u32x4 *space, int wave, int lane) {
    constexpr int CH = Mma<T>::CHUNKS;
    const int last = n_valid - 1 - row0;
    const char *first_row = reinterpret_cast<const char *>(base + (size_t)row0 * HEAD_DIM);
#pragma unroll
    for (int i = 0; i < 32 * Mma<T>::NBLK * CH / WAVE / W; ++i) {
        const int j = i * W + wave, row = j * (WAVE / CH) + lane / CH, pos = lane % CH;
        const uint32_t off = (uint32_t)(min(row, last) * (HEAD_DIM * (int)sizeof(T)) + ((pos ^ (row & (CH - 1))) * 16));
        __builtin_amdgcn_global_load_lds((gptr_t)(first_row + off), (lptr_t)(space + j * WAVE), 16, 0, 0);
    }
}
template <typename T>
__device__ __forceinline__ void read_stationary(const u32x4 *space, int lane, u32x4 (*frags)[Mma<T>::FRAGS]) {
    constexpr int CH = Mma<T>::CHUNKS;
    const int row = lane & 31;
#pragma unroll
    for (int b = 0; b < Mma<T>::NBLK; ++b)
#pragma unroll
        for (int f = 0; f < Mma<T>::FRAGS; ++f) frags[b][f] = space[(32 * b + row) * CH + ((2 * f + (lane >> 5)) ^ (row & (CH - 1)))];
}

// scores of a streamed 32-row block against one stationary block
template <typename T>
__device__ __forceinline__ f32x16 stream_scores(const u32x4 *a, const u32x4 *bfrag) {
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int f = 0; f < Mma<T>::FRAGS; ++f) Mma<T>::mma(acc, a[f], bfrag[f]);
    return acc;
}

// blockIdx -> (slice, rank), rank 0 the longest tile.  Workgroups are dealt round-robin to the eight XCDs, each with its own
// L2, so p slices that take turns, p a power of two up to eight, leave a slice's tiles on 8 / p of them.  All slices in turn,
// longest tiles first, does that for multiples of four; an odd number puts every slice on every XCD: column sums of 51
// slices of 2500 tokens, G = 4, 385 us (full kernel 301), both passes of 31 slices of 4096 229 (180), of 53 slices of 1500 83
// (77).  Other numbers of slices therefore go out as one, two and four of them, as needed, and then in whole groups of eight, in
// each part the longest tiles first: 202, 178 and 60.  Fewer than eight slices do so eight ranks at a time, or the short tiles of
// one part would start before the long ones of the next (6 slices of 8192: 139 in turn, 157 in parts, 141 like this; 7 of 6000 115,
// 107 and 97), and not below 32 tiles, where they find everything in any L2 (7 of 600: 15.0 in turn, 15.3).
// In turn the work is spread evenly, though, which is worth more where the lengths differ (by the first 64 rows of the
// batch: 21 slices of up to 6000 tokens 148 in turn, 214 in parts; all 6000 long 294 and 235) and for fp32, where the
// traffic hides behind the matrix pipe (5 slices of 3000: 121 and 135).
struct SplitBlock { int slice, rank; };
template <typename T>
__device__ __forceinline__ SplitBlock split_block(int n_slices, int tiles, const int32_t *seq_lens, int rows, int lane) {
    int i = blockIdx.x;
    bool in_turn = sizeof(T) == 4 || n_slices % 4 == 0 || n_slices <= 2 || (n_slices < 8 && tiles < 32);
    if (!in_turn && seq_lens) {
        const int len = seq_lens[min(lane, rows - 1)];
        in_turn = __ballot(len != __builtin_amdgcn_readfirstlane(len)) != 0;
    }
    if (in_turn) return {i % n_slices, i / n_slices};
    const int chunk = n_slices < 8 ? 8 : tiles;              // ranks that are dealt out before the next
    const int rank0 = i / (chunk * n_slices) * chunk, ranks = min(chunk, tiles - rank0);
    i -= rank0 * n_slices;
    int first = 0, p = 1;
    for (; p < 8; p *= 2) {
        if (!(n_slices & p)) continue;
        if (i < p * ranks) break;
        i -= p * ranks;
        first += p;
    }
    if (p == 8) p = n_slices - first;
    return {first + i % p, rank0 + i / p};
}

template <typename T, int W>
__global__ __launch_bounds__(W * WAVE, sizeof(T) == 2 && W == 4 ? 2 : 1) void attn_lse_split_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, float *__restrict__ lse, const int32_t *__restrict__ seq_lens,
    int n_qslices, int HG, int G, int N, int n_pad, int tiles_per_slice, float c, float out_scale, float pad)
{
    using M = Mma<T>;
    using S = Stream<T>;
    constexpr int NB = M::NBLK, ROWS = 32 * NB;
    __shared__ u32x4 lds_a[W][S::SLOTS], lds_b[W][S::SLOTS];  // (two objects: see attn_lse_kernel)
    __shared__ float part_m[W][ROWS], part_l[W][ROWS];

    const int lane = threadIdx.x & 63;
    const SplitBlock sb = split_block<T>(n_qslices, tiles_per_slice, seq_lens, n_qslices / HG, lane);
    const int qslice = sb.slice;
    const int tile = tiles_per_slice - 1 - sb.rank;           // the last tile has the longest rows
    const int b = qslice / HG;
    const int kvslice = b * (HG / G) + (qslice % HG) / G;
    const int n = clamp_len(seq_lens, b, N);
    const int q0 = tile * ROWS;
    if (q0 >= n) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T *Qs = Q + (size_t)qslice * N * HEAD_DIM;
    const T *Ks = K + (size_t)kvslice * N * HEAD_DIM;

    const int diag0 = tile * NB;                              // key block on the diagonal of query block 0
    const int count = min(diag0 + NB, (n + 31) / 32);         // key blocks 0 .. count-1, this wave's: wave, wave+W, ...
    int next = wave;
    auto issue_next = [&](u32x4 *stage) {
        if (next < count) S::issue(Ks, next * 32, n, stage, lane);
        next += W;
    };
    issue_stationary<T, W>(Qs, q0, n, lds_b[0], wave, lane);
    issue_next(lds_a[wave]);
    if (wave < count) wait_vmcnt<S::LOADS>();                 // the rows are here, the first tile may be under way
    else wait_vmcnt<0>();
    barrier_no_fence();
    u32x4 qf[NB][M::FRAGS];
    read_stationary<T>(lds_b[0], lane, qf);
    wait_lds();
    barrier_no_fence();
    float m_run[NB], l_run[NB];

    // 16-bit types: the reference of a wave's sums is the maximum of its first block and is held to the diagonal (see
    // rowsum_held).  Should a later score be so far above it that a sum leaves the range in which it can be put on
    // another reference without loss (HELD_SUM_MAX), the workgroup does all of it once more with the maximum updated at every
    // block.  That is looked at before the diagonal, whose maximum may scale the held sum to nothing, and before the waves' sums are combined.
    // Held or not, us: 32 slices of 4000 tokens 87.5 / 92.0, 16 of 2000 18.6 / 19.9, one of 16384 63.9 / 69.5.
    bool hold = sizeof(T) == 2, fits = true;
    auto step = [&](int t, const u32x4 *cur, u32x4 *nxt) {
        wait_own_tile();
        issue_next(nxt);
        u32x4 a[M::FRAGS];
#pragma unroll
        for (int f = 0; f < M::FRAGS; ++f) a[f] = S::frag(cur, f, lane);
        if (sizeof(T) == 2 && hold && t > wave && t < diag0) {
#pragma unroll
            for (int qb = 0; qb < NB; ++qb) rowsum_held(stream_scores<T>(a, qf[qb]), c, m_run[qb] * c, l_run[qb]);
            return;
        }
        if (sizeof(T) == 2 && hold) {
#pragma unroll
            for (int qb = 0; qb < NB; ++qb) fits = fits && l_run[qb] <= HELD_SUM_MAX;
        }
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) {
            if (t > diag0 + qb) continue;                     // every key of the block is in the future
            f32x16 acc = stream_scores<T>(a, qf[qb]);
            if (t == diag0 + qb) mask_rows_above_col(acc, lane);          // accumulator rows are keys, columns queries
            rowstat_update(acc, c, m_run[qb], l_run[qb]);
        }
    };
    for (;;) {
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) { m_run[qb] = M_INIT; l_run[qb] = 0.f; }
        for (int t = wave; t < count; t += 2 * W) {
            step(t, lds_a[wave], lds_b[wave]);
            if (t + W < count) step(t + W, lds_b[wave], lds_a[wave]);
        }
        // lanes l and l+32 hold the two halves of a row's keys; then the waves are combined
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) {
            fits = fits && l_run[qb] <= HELD_SUM_MAX;         // false for NaN
            const float m_o = __shfl_xor(m_run[qb], 32, WAVE), l_o = __shfl_xor(l_run[qb], 32, WAVE);
            const float m = fmaxf(m_run[qb], m_o);
            const float l = l_run[qb] * __builtin_amdgcn_exp2f((m_run[qb] - m) * c) + l_o * __builtin_amdgcn_exp2f((m_o - m) * c);
            if (lane < 32) { part_m[wave][32 * qb + lane] = m; part_l[wave][32 * qb + lane] = l; }
        }
        if (!__syncthreads_or(hold && !fits)) break;
        hold = false;
        next = wave;
        issue_next(lds_a[wave]);
    }
    const int q = q0 + threadIdx.x;
    if (threadIdx.x < ROWS && q < n_pad) {
        float m = part_m[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < W; ++w) m = fmaxf(m, part_m[w][threadIdx.x]);
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) l += part_l[w][threadIdx.x] * __builtin_amdgcn_exp2f((part_m[w][threadIdx.x] - m) * c);
        lse[(size_t)qslice * n_pad + q] = q < n ? (m * c + __log2f(l)) * out_scale : pad;
    }
}

template <typename T, int W>
__global__ __launch_bounds__(W * WAVE, sizeof(T) == 2 && W == 4 ? 2 : 1) void attn_colsum_split_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const float *__restrict__ lse, float *__restrict__ mass,
    float *__restrict__ sim_opt, const int32_t *__restrict__ seq_lens, int n_kvslices, int H, int G, int N, int n_pad,
    int tiles_per_slice, float c)
{
    using M = Mma<T>;
    using S = Stream<T>;
    constexpr int NB = M::NBLK, KEYS = 32 * NB;
    __shared__ u32x4 lds_a[W][S::SLOTS], lds_b[W][S::SLOTS];
    __shared__ __attribute__((aligned(16))) float lse_a[W][32], lse_b[W][32];
    __shared__ float part_s[W][KEYS];

    const int lane = threadIdx.x & 63;
    const SplitBlock sb = split_block<T>(n_kvslices, tiles_per_slice, seq_lens, n_kvslices / H, lane);
    const int kvslice = sb.slice;
    const int tile = sb.rank;                                 // tile 0 has the most rows below it
    const int b = kvslice / H, h = kvslice % H;
    const int n = clamp_len(seq_lens, b, N);
    const int k0 = tile * KEYS;
    float *mass_s = mass + (size_t)kvslice * N;
    float *sim_s = sim_opt ? sim_opt + (size_t)kvslice * N : nullptr;
    if (k0 >= n) {                                            // padding only: defined zeros
        const int j = k0 + threadIdx.x;
        if (threadIdx.x < KEYS && j < N) {
            mass_s[j] = 0.f;
            if (sim_s) sim_s[j] = 0.f;
        }
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T *Ks = K + (size_t)kvslice * N * HEAD_DIM;

    // the 32-row query blocks that see these keys, head after head: block u of the list is block
    // diag0 + u % per_head of head u / per_head; this wave's: wave, wave+W, ...
    const int diag0 = tile * NB;
    const int per_head = (n + 31) / 32 - diag0;
    const int count = per_head * G;
    int next = wave, next_g = wave / per_head, next_qb = wave % per_head;
    auto issue_next = [&](u32x4 *stage, float *stage_lse) {
        if (next < count) {
            const size_t qslice = ((size_t)b * H + h) * G + next_g;
            const int row0 = (diag0 + next_qb) * 32;
            S::issue(Q + qslice * N * HEAD_DIM, row0, n, stage, lane);
            if (lane < 32)
                __builtin_amdgcn_global_load_lds((gptr_t)(lse + qslice * n_pad + row0 + lane), (lptr_t)stage_lse, 4, 0, 0);
        }
        next += W;
        next_qb += W;
        while (next_qb >= per_head) { next_qb -= per_head; ++next_g; }
    };
    issue_stationary<T, W>(Ks, k0, n, lds_b[0], wave, lane);
    issue_next(lds_a[wave], lse_a[wave]);
    if (wave < count) wait_vmcnt<S::LOADS + 1>();             // the rows are here, the first tile may be under way
    else wait_vmcnt<0>();
    barrier_no_fence();
    u32x4 kf[NB][M::FRAGS];
    read_stationary<T>(lds_b[0], lane, kf);
    wait_lds();
    barrier_no_fence();
    if constexpr (sizeof(T) == 2) {
        if (sim_s) {                                          // the keys are here anyway: wave kb takes block kb's similarities
#pragma unroll
            for (int kb = 0; kb < NB; ++kb)
                if (wave == kb) {
                    const u32x4 before = load_predecessor<T>(Ks, k0 + 32 * kb, n, lane);
                    stationary_cosine<T>(k0 + 32 * kb, n, N, lane, kf[kb], before, sim_s);
                }
        }
    }
    float part[NB][2];
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) part[kb][0] = part[kb][1] = 0.f;

    int qb_cur = wave % per_head;                             // query block of the current step, from diag0
    auto step = [&](const u32x4 *cur, const float *cur_lse, u32x4 *nxt, float *nxt_lse) {
        wait_own_tile();
        issue_next(nxt, nxt_lse);
        u32x4 a[M::FRAGS];
#pragma unroll
        for (int f = 0; f < M::FRAGS; ++f) a[f] = S::frag(cur, f, lane);
        const RowStats L = load_rowstats(cur_lse, 0, lane);
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
            if (qb_cur < kb) continue;                        // every query of the block precedes the keys
            f32x16 acc = stream_scores<T>(a, kf[kb]);
            if (qb_cur == kb) mask_rows_below_col(acc, lane); // accumulator rows are queries, columns keys
            colsum_update(acc, L, c, part[kb]);
        }
        qb_cur += W;
        while (qb_cur >= per_head) qb_cur -= per_head;
    };
    for (int u = wave; u < count; u += 2 * W) {
        step(lds_a[wave], lse_a[wave], lds_b[wave], lse_b[wave]);
        if (u + W < count) step(lds_b[wave], lse_b[wave], lds_a[wave], lse_a[wave]);
    }
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) {
        const float colsum = part[kb][0] + part[kb][1];
        const float total = colsum + __shfl_xor(colsum, 32, WAVE);
        if (lane < 32) part_s[wave][32 * kb + lane] = total;
    }
    __syncthreads();
    const int key = k0 + threadIdx.x;
    if (threadIdx.x < KEYS && key < N) {
        float total = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) total += part_s[w][threadIdx.x];
        mass_s[key] = key < n ? total : 0.f;
    }
}

// ------------------------------------------------------------------------------------------
// fp32, the smallest launches: 16 rows a workgroup
// ------------------------------------------------------------------------------------------
//
// In fp32 the chain of a workgroup is matrix time: a 32x32 block is 64 MFMAs of 64 cycles on the one pipe of a wave, and more waves
// share the same four pipes.  What shortens it is more compute units: blocks of 16x16 (32 MFMAs 16x16x4 of 32 cycles, the same
// rate) put half the rows on each of twice as many workgroups, against twice the tile traffic.
struct Rows16 {
    static constexpr int CH = 32;                            // 16-byte chunks per row
    static constexpr int SLOTS = 16 * CH;
    static constexpr int FRAGS = 8;                          // fragment f of lane l: chunk 4 f + l / 16 of row l % 16
    // rows [row0, row0+16) of the matrix at `base` -> a stage, swizzled; rows past n_valid repeat the last valid one
    static __device__ __forceinline__ void issue(const float *base, int row0, int n_valid, u32x4 *stage, int lane) {
        const int last = n_valid - 1 - row0;
        const char *first_row = reinterpret_cast<const char *>(base + (size_t)row0 * HEAD_DIM);
#pragma unroll
        for (int i = 0; i < SLOTS / WAVE; ++i) {
            const int row = 2 * i + lane / CH, pos = lane % CH;
            const uint32_t off = (uint32_t)(min(row, last) * (HEAD_DIM * 4) + ((pos ^ row) * 16));
            __builtin_amdgcn_global_load_lds((gptr_t)(first_row + off), (lptr_t)(stage + i * WAVE), 16, 0, 0);
        }
    }
    static __device__ __forceinline__ u32x4 frag(const u32x4 *stage, int f, int lane) {
        const int row = lane & 15;
        return stage[row * CH + ((4 * f + (lane >> 4)) ^ row)];
    }
    // the stationary rows, as issue_stationary and read_stationary
    template <int W> static __device__ __forceinline__ void issue_rows(const float *base, int row0, int n_valid, u32x4 *space, int wave, int lane) {
        const int last = n_valid - 1 - row0;
        const char *first_row = reinterpret_cast<const char *>(base + (size_t)row0 * HEAD_DIM);
#pragma unroll
        for (int i = 0; i < SLOTS / WAVE / W; ++i) {
            const int j = i * W + wave, row = 2 * j + lane / CH, pos = lane % CH;
            const uint32_t off = (uint32_t)(min(row, last) * (HEAD_DIM * 4) + ((pos ^ row) * 16));
            __builtin_amdgcn_global_load_lds((gptr_t)(first_row + off), (lptr_t)(space + j * WAVE), 16, 0, 0);
        }
    }
    static __device__ __forceinline__ void read_rows(const u32x4 *space, int lane, u32x4 *frags) {
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) frags[f] = frag(space, f, lane);
    }
    // Result i of lane l is streamed row 4 (l / 16) + i, stationary row l % 16.  (Two chains: an MFMA does not wait for the one before.)
    static __device__ __forceinline__ f32x4 scores(const u32x4 *stage, const u32x4 *b, int lane) {
        u32x4 a[FRAGS];
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) a[f] = frag(stage, f, lane);
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int f = 0; f < FRAGS; ++f)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t ai = a[f][i], bi = b[f][i];
                acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, ai), __builtin_bit_cast(float, bi), acc[i & 1], 0, 0, 0);
            }
        return acc[0] + acc[1];
    }
};

template <int W>
__global__ __launch_bounds__(W * WAVE, 1) void attn_lse_split16_kernel(
    const float *__restrict__ Q, const float *__restrict__ K, float *__restrict__ lse, const int32_t *__restrict__ seq_lens,
    int n_qslices, int HG, int G, int N, int n_pad, int tiles_per_slice, float c, float out_scale, float pad)
{
    __shared__ u32x4 lds_a[W][Rows16::SLOTS], lds_b[W][Rows16::SLOTS];
    __shared__ float part_m[W][16], part_l[W][16];
    const int lane = threadIdx.x & 63;
    const int qslice = blockIdx.x % n_qslices;
    const int tile = tiles_per_slice - 1 - (int)(blockIdx.x / n_qslices);    // the last tile has the longest rows
    const int b = qslice / HG;
    const int kvslice = b * (HG / G) + (qslice % HG) / G;
    const int n = clamp_len(seq_lens, b, N);
    const int q0 = tile * 16;
    const int q = q0 + (int)threadIdx.x;
    if (q0 >= n) {                                            // (the second pass may read them, in a streamed block of 32 rows)
        if (threadIdx.x < 16 && q < n_pad) lse[(size_t)qslice * n_pad + q] = pad;
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float *Ks = K + (size_t)kvslice * N * HEAD_DIM;
    const int count = tile + 1;                               // key blocks 0 .. tile, this wave's: wave, wave+W, ...
    int next = wave;
    auto issue_next = [&](u32x4 *stage) {
        if (next < count) Rows16::issue(Ks, next * 16, n, stage, lane);
        next += W;
    };
    Rows16::issue_rows<W>(Q + (size_t)qslice * N * HEAD_DIM, q0, n, lds_b[0], wave, lane);
    issue_next(lds_a[wave]);
    if (wave < count) wait_vmcnt<Rows16::SLOTS / WAVE>();
    else wait_vmcnt<0>();
    barrier_no_fence();
    u32x4 qf[Rows16::FRAGS];
    Rows16::read_rows(lds_b[0], lane, qf);
    wait_lds();
    barrier_no_fence();
    float m_run = M_INIT, l_run = 0.f;
    auto step = [&](int t, const u32x4 *cur, u32x4 *nxt) {
        wait_own_tile();
        issue_next(nxt);
        f32x4 s = Rows16::scores(cur, qf, lane);
        if (t == tile) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * (lane >> 4) + i > (lane & 15)) s[i] = -INFINITY;
        }
        const float m = fmaxf(m_run, fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) p += __builtin_amdgcn_exp2f(fmaf(s[i], c, -m * c));
        l_run = l_run * __builtin_amdgcn_exp2f((m_run - m) * c) + p;
        m_run = m;
    };
    for (int t = wave; t < count; t += 2 * W) {
        step(t, lds_a[wave], lds_b[wave]);
        if (t + W < count) step(t + W, lds_b[wave], lds_a[wave]);
    }
    // the four lanes l % 16 hold the quarters of a row's keys; then the waves are combined
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {
        const float m_o = __shfl_xor(m_run, off, WAVE), l_o = __shfl_xor(l_run, off, WAVE);
        const float m = fmaxf(m_run, m_o);
        l_run = l_run * __builtin_amdgcn_exp2f((m_run - m) * c) + l_o * __builtin_amdgcn_exp2f((m_o - m) * c);
        m_run = m;
    }
    if (lane < 16) { part_m[wave][lane] = m_run; part_l[wave][lane] = l_run; }
    __syncthreads();
    if (threadIdx.x < 16 && q < n_pad) {
        float m = part_m[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < W; ++w) m = fmaxf(m, part_m[w][threadIdx.x]);
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) l += part_l[w][threadIdx.x] * __builtin_amdgcn_exp2f((part_m[w][threadIdx.x] - m) * c);
        lse[(size_t)qslice * n_pad + q] = q < n ? (m * c + __log2f(l)) * out_scale : pad;
    }
}

template <int W>
__global__ __launch_bounds__(W * WAVE, 1) void attn_colsum_split16_kernel(
    const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ lse, float *__restrict__ mass,
    const int32_t *__restrict__ seq_lens, int n_kvslices, int H, int G, int N, int n_pad, int tiles_per_slice, float c)
{
    __shared__ u32x4 lds_a[W][Rows16::SLOTS], lds_b[W][Rows16::SLOTS];
    __shared__ __attribute__((aligned(16))) float lse_a[W][16], lse_b[W][16];
    __shared__ float part_s[W][16];
    const int lane = threadIdx.x & 63;
    const int kvslice = blockIdx.x % n_kvslices, tile = blockIdx.x / n_kvslices;   // tile 0 has the most rows below it
    const int b = kvslice / H, h = kvslice % H;
    const int n = clamp_len(seq_lens, b, N);
    const int k0 = tile * 16;
    float *mass_s = mass + (size_t)kvslice * N;
    const int key = k0 + (int)threadIdx.x;
    if (k0 >= n) {                                            // padding only: defined zeros
        if (threadIdx.x < 16 && key < N) mass_s[key] = 0.f;
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the 16-row query blocks that see these keys, head after head (see attn_colsum_split_kernel)
    const int per_head = (n + 15) / 16 - tile;
    const int count = per_head * G;
    int next = wave, next_g = wave / per_head, next_qb = wave % per_head;
    auto issue_next = [&](u32x4 *stage, float *stage_lse) {
        if (next < count) {
            const size_t qslice = ((size_t)b * H + h) * G + next_g;
            const int row0 = (tile + next_qb) * 16;
            Rows16::issue(Q + qslice * N * HEAD_DIM, row0, n, stage, lane);
            if (lane < 16)
                __builtin_amdgcn_global_load_lds((gptr_t)(lse + qslice * n_pad + row0 + lane), (lptr_t)stage_lse, 4, 0, 0);
        }
        next += W;
        next_qb += W;
        while (next_qb >= per_head) { next_qb -= per_head; ++next_g; }
    };
    Rows16::issue_rows<W>(K + (size_t)kvslice * N * HEAD_DIM, k0, n, lds_b[0], wave, lane);
    issue_next(lds_a[wave], lse_a[wave]);
    if (wave < count) wait_vmcnt<Rows16::SLOTS / WAVE + 1>();
    else wait_vmcnt<0>();
    barrier_no_fence();
    u32x4 kf[Rows16::FRAGS];
    Rows16::read_rows(lds_b[0], lane, kf);
    wait_lds();
    barrier_no_fence();
    float part = 0.f;
    int qb_cur = wave % per_head;
    auto step = [&](const u32x4 *cur, const float *cur_lse, u32x4 *nxt, float *nxt_lse) {
        wait_own_tile();
        issue_next(nxt, nxt_lse);
        f32x4 s = Rows16::scores(cur, kf, lane);
        const f32x4 L = *reinterpret_cast<const f32x4 *>(&cur_lse[4 * (lane >> 4)]);
        if (qb_cur == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * (lane >> 4) + i < (lane & 15)) s[i] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) part += __builtin_amdgcn_exp2f(fmaf(s[i], c, -L[i]));
        qb_cur += W;
        while (qb_cur >= per_head) qb_cur -= per_head;
    };
    for (int u = wave; u < count; u += 2 * W) {
        step(lds_a[wave], lse_a[wave], lds_b[wave], lse_b[wave]);
        if (u + W < count) step(lds_b[wave], lse_b[wave], lds_a[wave], lse_a[wave]);
    }
    part += __shfl_xor(part, 16, WAVE);
    part += __shfl_xor(part, 32, WAVE);
    if (lane < 16) part_s[wave][lane] = part;
    __syncthreads();
    if (threadIdx.x < 16 && key < N) {
        float total = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) total += part_s[w][threadIdx.x];
        mass_s[key] = key < n ? total : 0.f;
    }
}

// ------------------------------------------------------------------------------------------
// host launchers
// ------------------------------------------------------------------------------------------

constexpr int SPLIT16 = 16;              // added to the waves: the fp32 kernels of 16 rows

// Waves per workgroup of a split launch; 0: the full kernels are the better choice.
//   N, slices  stationary rows per slice, slices of the launch;  heads  streamed sequences per slice (G in the column sums, else 1)
//   tiles      256-row (fp32: 128) tiles per slice of the full kernel;  full_wgs  workgroups it would launch
// Measured per pass, row statistics and column sums, full / split kernel, us (full_wgs in brackets): 32 slices of 1000 tokens f16 (128) 25.0, 25.9 / 12.8,
// 12.7; 8 of 4096 (64) 84.9, 90.2 / 29.8, 29.1, with G = 4 the column sums 328 / 91; 32 of 4096 (256) 91.8, 96.6 / 88.5, 89.8; 51 of 2500 (255) 79.1, 82.8 /
// 60.0, 58.7; one of 16384 (32) 312, 457 / 67, 73; of 131072 (256) 11340, 11820 / 2460, 2650; 8 of 16384 with G = 4 (256) column sums 1830 / 1290, although
// the column sums of such lengths have a kernel of 512 keys a workgroup and read every tile eight times as often as that; but 160 of 2048 (640)
// 110, 112 / 128, 125 and 24 of 2500 with G = 4 (480) row statistics 93.9 / 107.8.
// Below 8 tiles a full workgroup's load is not evened out by pairing, and the split kernels still win at 384 (96 slices of
// 1000: 34.4, 36.2 / 26.0, 24.8).  In one or two tiles the full kernels' chains are short as well, and the split ones need a chain, heads
// after each other, to earn their traffic.  G = 1: 160 slices of 512 (320) 21.0, 21.4 / 19.3, 16.2; 128 of 256 11.2, 11.4 / 7.9, 7.0, 192 of them
// 11.4, 11.3 / 11.0, 10.0; 256 of 128 8.2, 8.0 / 7.2, 6.6, of 64 6.4, 6.6 / 6.4, 6.1.  Column sums, G = 2: 256 slices of 256 18.3 / 15.2; G = 4: 320 of
// 256 33.9 / 30.0, 384 of 200 32.0 / 27.4, but 384 of 256 34.7 / 36.0.
// These are the present kernels, whose stationary rows go through LDS; the lines were drawn with the ones before, 3 to 19 % slower, and lie short of
// where the two sides meet now: 64 slices of 2500 (320) 83.3, 86.5 / 73.3, 71.6, 96 of 2000 (384) 75.1, 78.1 / 72.6, 70.3; 128 of 1000 (512) 35.9, 37.4 / 33.7,
// 31.7; 192 of 512 (384) 22.2, 23.0 / 20.8, 18.1; 256 of 256 column sums 11.9 / 10.7; 384 of 200, G = 2, column sums 21.1 / 19.2.
// fp32, where the matrix pipe is sixteen times slower and the latencies hide behind it: 8 slices of 4096 (128) 282, 287 / 167, 169, 32 of
// 1000 (128) 82, 83 / 55, 55, 64 of them (256) 86, 87 / 104, 102.  The kernels of 16 rows, both passes, 32 rows / 16 rows and four waves / eight: one slice
// of 130 16.9 / 11.2 / 11.9, of 1000 44 / 31 / 28.5, of 4000 145 / 100 / 85.5, 8 of 1000 (256 workgroups of 32 rows) 45.5 / 39.7 / 36.5,
// 16 of 512 (256, short chains) 27.0 / 23.7 / 25.4, 32 of 200 18.2 / 14.8 / 18.5, 4 of 3000 (376) 112 / 103 / 113; and 16 of 1000 (512) 55 / 58 /
// 65: hence up to 384 blocks of 32 rows, and eight waves, whose workgroups of 130 KB of LDS take a compute unit each, where the up to 512 of
// them (two of 16 rows a block) are through in two rounds and the chain is long.
// Eight waves instead of four halve the chain but leave one workgroup per compute unit: worth it where all of them
// are resident in two rounds and the chain is long (8 slices of 1000, G = 4, column sums: 30 with four, 24 with
// eight; of 4096: 117 and 93; 32 slices of 1000, chain of 32: 15 and 17).
int attn_split_waves(bool colsum, int dtype, int N, long long slices, int heads, int tiles, long long full_wgs)
{
    const int blocks = (N + 31) / 32;                         // streamed 32-row blocks per head
    if (dtype == KVM_F32) {
        if (full_wgs > 128) return 0;
        if (slices * blocks <= 256 && (long long)blocks * heads >= 24) return SPLIT16 + 8;
        return slices * blocks <= 384 ? SPLIT16 + 4 : 4;
    }
    int most = tiles >= 8 ? 256 : 384;
    if (heads == 1 && tiles == 2 && blocks > 14) most = 320;
    else if (heads == 1 && tiles == 1) most = blocks <= 3 ? 256 : colsum ? 128 : blocks <= 6 ? 256 : 192;
    else if (tiles == 1) most -= 64 * std::max(0, blocks - (heads < 4 ? 6 : 7));
    if (full_wgs > most) return 0;
    return slices * ((blocks + 1) / 2) <= 512 && (long long)blocks * heads >= 64 ? 8 : 4;
}

template <typename T, int W>
static void lse_t(const kvm_shape &sh, const void *Q, const void *K, float *lse, int n_pad, float c, float out_scale, float pad,
                  hipStream_t st)
{
    constexpr int ROWS = 32 * Mma<T>::NBLK;
    const int tiles = (sh.N + ROWS - 1) / ROWS, n_q = sh.B * sh.H_kv * sh.G;
    hipLaunchKernelGGL((attn_lse_split_kernel<T, W>), dim3((unsigned)((long long)n_q * tiles)), dim3(W * WAVE), 0, st, (const T *)Q,
                       (const T *)K, lse, sh.seq_lens, n_q, sh.H_kv * sh.G, sh.G, sh.N, n_pad, tiles, c, out_scale, pad);
}

template <typename T, int W>
static void colsum_t(const kvm_shape &sh, const void *Q, const void *K, const float *lse, float *mass, float *sim_opt, int n_pad,
                     float c, hipStream_t st)
{
    constexpr int KEYS = 32 * Mma<T>::NBLK;
    const int tiles = (sh.N + KEYS - 1) / KEYS, n_kv = sh.B * sh.H_kv;
    hipLaunchKernelGGL((attn_colsum_split_kernel<T, W>), dim3((unsigned)((long long)n_kv * tiles)), dim3(W * WAVE), 0, st, (const T *)Q,
                       (const T *)K, lse, mass, sizeof(T) == 2 ? sim_opt : nullptr, sh.seq_lens, n_kv, sh.H_kv, sh.G, sh.N, n_pad, tiles, c);
}

template <int W>
static void lse16_t(const kvm_shape &sh, const void *Q, const void *K, float *lse, int n_pad, float c, float out_scale, float pad,
                    hipStream_t st)
{
    const int tiles = (sh.N + 31) / 32 * 2, n_q = sh.B * sh.H_kv * sh.G;   // (whole 32-row blocks: the second pass may be the other kernel)
    hipLaunchKernelGGL(attn_lse_split16_kernel<W>, dim3((unsigned)((long long)n_q * tiles)), dim3(W * WAVE), 0, st, (const float *)Q,
                       (const float *)K, lse, sh.seq_lens, n_q, sh.H_kv * sh.G, sh.G, sh.N, n_pad, tiles, c, out_scale, pad);
}

template <int W>
static void colsum16_t(const kvm_shape &sh, const void *Q, const void *K, const float *lse, float *mass, int n_pad, float c, hipStream_t st)
{
    const int tiles = (sh.N + 15) / 16, n_kv = sh.B * sh.H_kv;
    hipLaunchKernelGGL(attn_colsum_split16_kernel<W>, dim3((unsigned)((long long)n_kv * tiles)), dim3(W * WAVE), 0, st, (const float *)Q,
                       (const float *)K, lse, mass, sh.seq_lens, n_kv, sh.H_kv, sh.G, sh.N, n_pad, tiles, c);
}

void launch_lse_split(int waves, const kvm_shape &sh, const void *Q, const void *K, float *lse, int n_pad, float c, float out_scale,
                      float pad, hipStream_t st)
{
    if (sh.dtype == KVM_F32 && waves == SPLIT16 + 8) lse16_t<8>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
    else if (sh.dtype == KVM_F32 && waves > SPLIT16) lse16_t<4>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
    else if (sh.dtype == KVM_F32) lse_t<float, 4>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
    else if (sh.dtype == KVM_F16 && waves == 4) lse_t<half_t, 4>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
    else if (sh.dtype == KVM_F16) lse_t<half_t, 8>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
    else if (waves == 4) lse_t<bf16_t, 4>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
    else lse_t<bf16_t, 8>(sh, Q, K, lse, n_pad, c, out_scale, pad, st);
}

void launch_colsum_split(int waves, const kvm_shape &sh, const void *Q, const void *K, const float *lse, float *mass, float *sim_opt,
                         int n_pad, float c, hipStream_t st)
{
    if (sh.dtype == KVM_F32 && waves == SPLIT16 + 8) colsum16_t<8>(sh, Q, K, lse, mass, n_pad, c, st);
    else if (sh.dtype == KVM_F32 && waves > SPLIT16) colsum16_t<4>(sh, Q, K, lse, mass, n_pad, c, st);
    else if (sh.dtype == KVM_F32) colsum_t<float, 4>(sh, Q, K, lse, mass, sim_opt, n_pad, c, st);
    else if (sh.dtype == KVM_F16 && waves == 4) colsum_t<half_t, 4>(sh, Q, K, lse, mass, sim_opt, n_pad, c, st);
    else if (sh.dtype == KVM_F16) colsum_t<half_t, 8>(sh, Q, K, lse, mass, sim_opt, n_pad, c, st);
    else if (waves == 4) colsum_t<bf16_t, 4>(sh, Q, K, lse, mass, sim_opt, n_pad, c, st);
    else colsum_t<bf16_t, 8>(sh, Q, K, lse, mass, sim_opt, n_pad, c, st);
}

}  // namespace kvm
