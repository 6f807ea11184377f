// The aggregated scores of short sequences in one score pass (Section 2.4 Eq. (1), Section 4.2 Eq. (7)).
//
//   attn_single_kernel       exponentials, row sums and column sums of 32 rows (fp32: 16) at a time, from one QK^T
//   attn_single_sum_kernel   adds the column sums of a slice's workgroups up, in their order (column_parts.h)
//
// The two passes of attn_mass.hip and attn_split.hip form the score matrix twice, with an exponential a score each time, because
// a row's sum has to be known before its terms can go to the columns.  Up to 2048 keys (fp32: 4096) the terms of 32 (16) rows fit
// the registers of a workgroup, though: its waves share the keys out, each keeps exp2(c s - r) of its own, r a reference of the
// rows, the waves exchange their parts of the row sums, and each term goes to its column with one multiplication.  Half the
// matrix work and half the exponentials; the price is that every key tile is read for 32 rows instead of 64 to 512.
//
// What bounds it (32 rows, 1024 slices of 1000 fp16 tokens): the 32 KB of keys that four SIMDs take in for 32x32 scores each are
// 550 cycles of the path from the caches (60 bytes a cycle and compute unit, measured), their arithmetic is 400 cycles of the vector
// ALU and 256 of the matrix pipe, and the exchange of the row sums leaves a wave idle once in 32 rows; the counters show the vector ALU
// busy for half of the time, with two waves a SIMD (256 registers).  64 rows a workgroup would halve the traffic and were
// twice as slow: eight waves then hold one compute unit, and nothing covers their exchanges.  fp32 is matrix time; its rows
// of more than 2048 tokens spill 55 of their 256 registers, most of them around the last tiles of the longest rows and the loops.
// us, both passes / this with its sum kernel: 1024 slices of 1000 fp16 tokens 436 / 334, 256 of them 118 / 77, 32 of them 19.0 / 16.0, 8 of them 18.1 /
// 12.2; 1024 of 512 134 / 99, of 250 53 / 32, of 128 33 / 20; 32 of 2000 51 / 42; 8 of 1000, G = 4, in bf16 28.3 / 19.5; fp32: 256 of 1000 587 /
// 348, 32 of 4096 1052 / 750, one of 512 18.0 / 12.7.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "attn_tile.h"
#include "column_parts.h"
#include "row_window.h"

namespace kvm {

template <typename T> struct Single;
// 16-bit types: 32 rows as two operands of the 16x16x32 MFMA against tiles of 32 keys; fp32: 16 rows and keys, 16x16x4.
template <typename T> struct SingleHalf {
    static constexpr int CH = 16, FRAGS = 4, SUB = 2;         // 16-byte chunks a row, fragments a lane and 16 rows, 16 keys a tile
};
template <> struct Single<half_t> : SingleHalf<half_t> {
    static __device__ __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, const f32x4 &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};
template <> struct Single<bf16_t> : SingleHalf<bf16_t> {
    static __device__ __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, const f32x4 &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
// fp32 scores are two sums of 64 products: as one of 128 they were less exact than those of the 16-row split kernels (error of the aggregated scores
// against 64 bits, 2-norm, those / one sum / two: 4 slices of 1000, scores like N(0, 8^2), 4.9e-7 / 6.5e-7 / 3.8e-7, one of 500, N(0, 4^2),
// 1.8e-7 / 2.6e-7 / 1.5e-7).  It costs 1 to 2 %, from 2049 tokens on 1 to 5 (32 of 4096 721 / 756 us).
template <> struct Single<float> {
    static constexpr int CH = 32, FRAGS = 8, SUB = 1;
    static __device__ __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, f32x4 c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t ai = a[i], bi = b[i];
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, ai), __builtin_bit_cast(float, bi), c, 0, 0, 0);
        }
        return c;
    }
};

// A row's terms are formed against one reference for all rows of the unit: the least log-sum-exp of the unit before, which is of the same query
// head (a workgroup stays with one).  Row sums between these bounds lose nothing by it: no term overflows, and one below 2^-126, which exp2
// flushes to zero, is below 2^-94 of the sum.  Other rows (22 natural orders below the least one of the unit before, or 83 above it)
// get a reference of their own, which costs their unit two more walks.
// us, two passes / reference of the first row of the unit before, whichever head's / this, scores like N(0, s^2): 256 slices of 1000 fp16 tokens, G = 4,
// s = 1 in every other head and 8 in the others 402 / 348 / 288, s = 20 538 / 614 / 300, s = 40 584 / 944 / 632; 32 of 1000, G = 1,
// s = 20 30 / 38 / 25, s = 40 30 / 39 / 35; fp32, 8 of 1000, G = 4, s = 20 101 / 144 / 81, s = 40 101 / 150 / 138; s = 1: within 2 %.
constexpr float SUM_MIN = 0x1p-32f, SUM_MAX = 0x1p120f;

// f(0), f(1), .. f(N-1) with constant arguments
template <int I, int N, typename F> __device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// 64 times 16 bytes of a window (scalar) of the matrix at base into consecutive LDS slots; what lies beyond its end reads as zeros
__device__ __forceinline__ void load_lds(const char *base, RowWindow w, int lane_offset, u32x4 *dst) {
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)(base + w.begin), 0, w.bytes, 0x00027000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)dst, 16, lane_offset, 0, 0, 0);
#endif
}

// lane N of each row of 16 lanes, in all of them
template <int N> __device__ __forceinline__ float row16_lane(float v) { return dpp_f<0x150 + N>(v); }

// the least of the four 16-lane rows of a wave (same lane position in each), in all of them
__device__ __forceinline__ float rows4_min(float v) {
    const uint32_t a = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    const uint32_t b = __builtin_bit_cast(uint32_t, fminf(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)));
    const auto t = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    const uint32_t t0 = t[0], t1 = t[1];
    return fminf(__builtin_bit_cast(float, t0), __builtin_bit_cast(float, t1));
}

// (max, sum) of a row and of more of its scores, in the reference of the larger maximum
__device__ __forceinline__ void join(float &m0, float &l0, float m1, float l1, float c) {
    const float m = fmaxf(m0, m1);
    l0 = l0 * __builtin_amdgcn_exp2f((m0 - m) * c) + l1 * __builtin_amdgcn_exp2f((m1 - m) * c);
    m0 = m;
}

// blockIdx -> (slice, workgroup of the slice).  Workgroups are dealt round-robin to the eight XCDs, each with its own L2.  Eight slices that take turns
// keep each on one of them; what is left over by whole eights goes out before them as four, two and one, which leave a slice on two,
// four or all eight.  (In turn as they are, 33 or 57 slices put every slice on every XCD; rounded up to whole eights with empty workgroups, 65
// slices keep one XCD an eighth longer than the others.  us, those / this, each with its best number of workgroups: 57 slices of 1000 fp16 tokens 40 / 25,
// 33 of 2000 80 / 46, 100 of 1000 38.9 / 35.9.)  From 64 slices on an eight's
// workgroups go out together, or too many keys are asked for at a time.
struct SingleBlock { int slice, p; };
__device__ __forceinline__ SingleBlock single_block(int n_slices, int P) {
    int i = blockIdx.x;
    if (n_slices < 8) return {i % n_slices, i / n_slices};
    const int rest = n_slices & 7, whole = n_slices - rest;
    if (i < rest * P) {
        int first = whole, size = 4;
        for (; size > 1; size >>= 1) {
            if (!(rest & size)) continue;
            if (i < size * P) break;
            i -= size * P;
            first += size;
        }
        return {first + i % size, i / size};
    }
    i -= rest * P;
    if (whole < 64) return {i % whole, i / whole};
    const int eight = i / (8 * P);
    i -= eight * 8 * P;
    return {8 * eight + (i & 7), i >> 3};
}

// Units of work of a slice: a group of rows of one query head.  P workgroups share the slice, P a multiple of G; workgroup p takes units of head
// p % G, counted off from the longest: r = p / G, 2S-1-r, 2S+r, .. with S = P / G, a long one, then short ones.
template <typename T, int RT, int W, int NT, int OCC>
__global__ __launch_bounds__(W * WAVE, OCC) void attn_single_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, float *__restrict__ out, int n_slices, int G, int n, int n_pad,
    int sharers, float c)
{
    using A = Single<T>;
    static_assert(RT == A::SUB, "one tile on the diagonal");
    constexpr int SUB = A::SUB, ROWS = 16 * RT, KEYS = 16 * SUB, FR = A::FRAGS, CH = A::CH, R = 4 * RT;
    constexpr int SLOTS = KEYS * CH, ROW_BYTES = HEAD_DIM * (int)sizeof(T);
    __shared__ u32x4 stage[W][SLOTS];
    __shared__ __attribute__((aligned(16))) float part[2][W][ROWS];
    __shared__ u32x4 rows_q[ROWS * CH];

    const int lane = threadIdx.x & 63, group = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int P = sharers * G;                                // workgroups of a slice, `sharers` of a head
    const SingleBlock sb = single_block(n_slices, P);
    const int slice = sb.slice, p = sb.p;
    const int units = (n + ROWS - 1) / ROWS, rank = G == 1 ? p : p / G;   // of a head: units, which of its workgroups
    const char *Ks = reinterpret_cast<const char *>(K + (size_t)slice * n * HEAD_DIM);
    const char *Qs = reinterpret_cast<const char *>(Q + ((size_t)slice * G + (p - rank * G)) * n * HEAD_DIM);

    // Rows [16 m, 16 m + 16) of a matrix into 16 rows of LDS, HALF load instructions; chunk ch of row r goes to position ch ^ r, which
    // is done on the source side (the instruction writes 64 consecutive slots).  Rows past the slice's last one read as zeros.
    constexpr int HALF = 16 * CH / WAVE;
    // (The offsets of load i are those of load 0 with some bits turned, as are the slots of fragment f: where the terms fill the registers they
    // are worked out each time.)
    constexpr bool TIGHT = NT * SUB * RT > 16 && sizeof(T) == 4;
    constexpr int OFFS = TIGHT ? 1 : HALF, SLOTS_KEPT = TIGHT ? 1 : FR, TURN = 16 * WAVE + 16 * (WAVE / CH);
    int voff[OFFS], slot[SLOTS_KEPT];
#pragma unroll
    for (int i = 0; i < OFFS; ++i) voff[i] = row_of_lane(i, lane, CH) * ROW_BYTES + offset_in_row(row_of_lane(i, lane, CH), lane, CH);
#pragma unroll
    for (int f = 0; f < SLOTS_KEPT; ++f) slot[f] = col * CH + ((4 * f + group) ^ col);

    auto issue = [&](int t) __attribute__((always_inline)) {
        asm volatile("" : "+s"(t));                           // (or the offsets of all tiles are kept in registers from unit to unit)
        int first = voff[0];
        if (TIGHT) asm volatile("" : "+v"(first));
#pragma unroll
        for (int h = 0; h < SUB; ++h) {
            const RowWindow w = row_window(n, t * KEYS + 16 * h, ROW_BYTES);
#pragma unroll
            for (int i = 0; i < HALF; ++i) load_lds(Ks, w, TIGHT ? first ^ i * TURN : voff[TIGHT ? 0 : i], stage[wave] + (h * HALF + i) * WAVE);
        }
    };

    // unit o: its first tile, and its rows, which are dealt to the waves (rows past the end repeat the last one: sums that count for nothing)
    u32x4 qf[RT][FR];
    int q0 = 0, cnt = 0, diag = 0;
    auto unit = [&](int k) __attribute__((always_inline)) { return k * sharers + ((k & 1) ? sharers - 1 - rank : rank); };
    auto begin = [&](int o) __attribute__((always_inline)) {
        q0 = (units - 1 - o) * ROWS;
        diag = q0 / KEYS;                                     // key tile on the diagonal
        cnt = (diag + W - wave) / W;                          // tiles of this wave: wave, wave + W, ..
        if (cnt > 0) issue(wave);
    };
    auto load_rows = [&]() __attribute__((always_inline)) {
        const int lane_now = fresh_lane();
        const RowWindow w = row_window(n, q0, ROW_BYTES);
#pragma unroll
        for (int i = 0; i < ROWS * CH / WAVE / W; ++i) {
            const int j = i * W + wave, row = row_of_lane(j, lane_now, CH);
            load_lds(Qs, w, min(row, n - 1 - q0) * ROW_BYTES + offset_in_row(row, lane_now, CH), rows_q + j * WAVE);
        }
    };
    auto read_rows = [&]() __attribute__((always_inline)) {
        const int lane_now = fresh_lane();                    // (addresses that need not stay in registers)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int f = 0; f < FR; ++f) qf[rt][f] = rows_q[(lane_now & 15) * CH + ((4 * f + (lane_now >> 4)) ^ (lane_now & 15)) + 16 * CH * rt];
        wait_lds();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int f = 0; f < FR; ++f) asm volatile("" : "+v"(qf[rt][f]));
    };
    auto read_frags = [&](u32x4 (*kf)[FR]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < SUB; ++j)
#pragma unroll
            for (int f = 0; f < FR; ++f) kf[j][f] = stage[wave][slot[TIGHT ? 0 : f] + 16 * CH * j];
    };
    auto scores = [&](const u32x4 (*kf)[FR], f32x4 (*s)[RT]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < SUB; ++j) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) s[j][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int f = 0; f < FR; ++f)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) s[j][rt] = A::mma(qf[rt][f], kf[j][f], s[j][rt]);
            } else {                                          // (two sums of 64 products, see Single<float>)
                f32x4 half = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < FR / 2; ++f) {
                    s[j][0] = A::mma(qf[0][f], kf[j][f], s[j][0]);
                    half = A::mma(qf[0][FR / 2 + f], kf[j][FR / 2 + f], half);
                }
                s[j][0] += half;
            }
        }
    };
    // the scores of the tile that is in the stage; read() comes once its rows are in registers
    auto stage_scores = [&](f32x4 (*s)[RT], auto read) __attribute__((always_inline)) {
        if constexpr (TIGHT) {                                // half of the fragments at a time
            f32x4 sum[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
            int first = slot[0];
            asm volatile("" : "+v"(first));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 kf[FR / 2];
#pragma unroll
                for (int f = 0; f < FR / 2; ++f) kf[f] = stage[wave][first ^ 4 * (h * (FR / 2) + f)];
                __builtin_amdgcn_sched_barrier(0);
                wait_lds();
                if (h == 1) read();
#pragma unroll
                for (int f = 0; f < FR / 2; ++f) sum[h] = A::mma(qf[0][h * (FR / 2) + f], kf[f], sum[h]);
                if (h == 0) __builtin_amdgcn_sched_barrier(0);
            }
            s[0][0] = sum[0] + sum[1];
        } else {
            u32x4 kf[SUB][FR];
            read_frags(kf);
            wait_lds();
            read();
            scores(kf, s);
        }
    };
    auto mask = [&](f32x4 (*s)[RT]) __attribute__((always_inline)) {      // the tile on the diagonal: keys after their row
        const int lane_now = fresh_lane();
        const int ahead = (lane_now & 15) - 4 * (lane_now >> 4);
#pragma unroll
        for (int j = 0; j < SUB; ++j)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (16 * (r / 4) + r % 4 < 16 * j + ahead) s[j][r / 4][r % 4] = -INFINITY;
    };

    float colsum[NT][SUB];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < SUB; ++j) colsum[i][j] = 0.f;
    int covered = 0;
    float base = 0.f;                                         // the reference; the first: the first unit's first row, its largest score with four keys before it
    if (rank < units) {
        begin(rank);
        load_rows();
        covered = cnt;
        const typename Elem<T>::Raw first_row = Elem<T>::load(reinterpret_cast<const T *>(Qs) + (size_t)q0 * HEAD_DIM, col);
        const typename Elem<T>::Raw key = Elem<T>::load(reinterpret_cast<const T *>(Ks) + (size_t)((q0 * group) >> 2) * HEAD_DIM, col);
        const float most = -c * rows4_min(-row16_sum(RowDot<T>::dot(first_row, key)));
        if (fabsf(most) < 0x1p60f) base = most;
    }
    int par = 0;
    uint64_t redo = 0;
    for (int k = 0, o = rank; o < units;) {
        float l[R];
        f32x4 t_[NT][SUB][RT];
        const int q0_now = q0, cnt_now = cnt, diag_now = diag;
        wait_vmcnt<0>();                                      // the wave's part of the rows and its first tile are here
        barrier_no_fence();
        read_rows();
        if (cnt > 0) {
            stage_scores(t_[0], [&]() __attribute__((always_inline)) { if (1 < cnt) issue(W + wave); });
        }
#pragma unroll
        for (int r = 0; r < R; ++r) l[r] = 0.f;
        auto terms = [&](f32x4 *s) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < R; ++r) s[r / 4][r % 4] = __builtin_amdgcn_exp2f(fmaf(s[r / 4][r % 4], c, -base));
#pragma unroll
            for (int r = 0; r < R; ++r) l[r] += s[r / 4][r % 4];
        };
        // The terms of a tile are formed under the LDS reads of the next one and between its MFMAs.
        static_for<1, NT + 1>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = ic;
            if (i < NT && i < cnt) {
                if constexpr (i < NT) {
                    wait_vmcnt<0>();
                    const auto next = [&]() __attribute__((always_inline)) { if (i + 1 < NT && i + 1 < cnt) issue((i + 1) * W + wave); };
                    if constexpr (SUB > 1) {
                        u32x4 kf[SUB][FR];
                        read_frags(kf);
                        terms(t_[i - 1][0]);
                        __builtin_amdgcn_sched_barrier(0);
                        wait_lds();
                        next();
                        scores(kf, t_[i]);
                    } else {
                        stage_scores(t_[i], next);
                    }
                    terms(t_[i - 1][SUB - 1]);
                    if constexpr (sizeof(T) == 2) {
#pragma unroll
                        for (int q = 0; q < 4 * RT; ++q) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // MFMA
                            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);   // VALU
                            __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);   // TRANS
                        }
                    }
                }
            } else if (i == cnt) {
                if ((i - 1) * W + wave == diag_now) mask(t_[i - 1]);
#pragma unroll
                for (int j = 0; j < SUB; ++j) terms(t_[i - 1][j]);
                asm volatile("");                             // (keeps the ends of all tiles apart: merged, they address t_ by a variable, in scratch)
            }
        });
        // the next unit's first tile is on its way while this one's sums are exchanged, its rows while the terms go to the columns
        ++k;
        o = unit(k);
        if (o < units) begin(o);
#pragma unroll
        for (int r = 0; r < R; ++r) l[r] = row16_sum(l[r]);
        if (const int lane_w = fresh_lane(); (lane_w & 15) == 0) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                *reinterpret_cast<f32x4 *>(&part[par][wave][16 * rt + (lane_w >> 4) * 4]) = f32x4{l[4 * rt], l[4 * rt + 1], l[4 * rt + 2], l[4 * rt + 3]};
        }
        wait_lds();
        barrier_no_fence();                                   // (and every wave has long read this unit's rows)
        if (o < units) load_rows();
        // lane `col` of a row of lanes adds up the sum of that row's own score row col
        const int lane_now = fresh_lane();
        const int myrow = 16 * ((lane_now >> 2) & (RT - 1)) + 4 * (lane_now >> 4) + (lane_now & 3);
        float sum = part[par][0][myrow];
#pragma unroll
        for (int w = 1; w < W; ++w) sum += part[par][w][myrow];
        const bool counts = q0_now + myrow < n;
        float least = counts ? sum : INFINITY;                // of the unit's rows, in every lane
        least = fminf(least, dpp_f<0xB1>(least));
        least = fminf(least, dpp_f<0x4E>(least));
        if (RT > 1) least = fminf(least, dpp_f<0x141>(least));
        least = rows4_min(least);
        if (__ballot(counts && !(sum >= SUM_MIN && sum <= SUM_MAX)) == 0) {   // (the same rows in every wave)
            const float inv = counts ? 1.0f / sum : 0.f;
            float wgt[R];
            static_for<0, R>([&](auto ic) __attribute__((always_inline)) { wgt[ic] = row16_lane<ic>(inv); });
            static_for<0, NT>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = ic;
                if (i < cnt_now) {
#pragma unroll
                    for (int j = 0; j < SUB; ++j)
#pragma unroll
                        for (int r = 0; r < R; ++r) colsum[i][j] = fmaf(t_[i][j][r / 4][r % 4], wgt[r], colsum[i][j]);
                }
            });
        } else {
            redo |= 1ull << (k - 1);
        }
        base += fminf(fmaxf(__log2f(least), -100.f), 100.f);
        par ^= 1;
    }
    // Units whose rows no common reference fitted: the statistics of their rows with a maximum of their own, then the terms from them, in two
    // more walks over the tiles.
    for (; redo; redo &= redo - 1) {
        const int k = __builtin_ctzll(redo);
        __syncthreads();                                      // nobody reads the rows or sums of the unit before
        begin(unit(k));
        load_rows();
        wait_vmcnt<0>();
        __syncthreads();
        read_rows();
        float m[R], l[R];
#pragma unroll
        for (int r = 0; r < R; ++r) { m[r] = M_INIT; l[r] = 0.f; }
        f32x4 s[SUB][RT];
        auto scores_of = [&](int i, int next) __attribute__((always_inline)) {
            wait_vmcnt<0>();
            stage_scores(s, [&]() __attribute__((always_inline)) { if (next < cnt) issue(next * W + wave); });
            if (i * W + wave == diag) mask(s);
        };
#pragma clang loop unroll(disable)
        for (int i = 0; i < cnt; ++i) {
            scores_of(i, i + 1);
#pragma unroll
            for (int j = 0; j < SUB; ++j)
#pragma unroll
                for (int r = 0; r < R; ++r) join(m[r], l[r], s[j][r / 4][r % 4], 1.f, c);
        }
        if (cnt > 0) issue(wave);                             // for the second walk
#pragma unroll
        for (int r = 0; r < R; ++r) {
            join(m[r], l[r], dpp_f<0xB1>(m[r]), dpp_f<0xB1>(l[r]), c);
            join(m[r], l[r], dpp_f<0x4E>(m[r]), dpp_f<0x4E>(l[r]), c);
            join(m[r], l[r], dpp_f<0x141>(m[r]), dpp_f<0x141>(l[r]), c);
            join(m[r], l[r], dpp_f<0x140>(m[r]), dpp_f<0x140>(l[r]), c);
        }
        if (col == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                part[0][wave][16 * (r / 4) + 4 * group + r % 4] = m[r];
                part[1][wave][16 * (r / 4) + 4 * group + r % 4] = l[r];
            }
        }
        __syncthreads();
        const int myrow = 16 * ((col >> 2) & (RT - 1)) + 4 * group + (col & 3);
        float mm = part[0][0][myrow], ll = part[1][0][myrow];
        for (int w = 1; w < W; ++w) join(mm, ll, part[0][w][myrow], part[1][w][myrow], c);
        // (by maximum and sum, not by their log-sum-exp: rounded at 2^36, its error would be the exponent of an infinite term)
        const float inv = q0 + myrow < n ? 1.0f / ll : 0.f;
        float most[R], wgt[R];
        static_for<0, R>([&](auto ic) __attribute__((always_inline)) { most[ic] = row16_lane<ic>(mm); wgt[ic] = row16_lane<ic>(inv); });
#pragma clang loop unroll(disable)
        for (int i = 0; i < cnt; ++i) {
            scores_of(i, i + 1);
#pragma unroll
            for (int j = 0; j < SUB; ++j) {
                float v = 0.f;
#pragma unroll
                for (int r = 0; r < R; ++r) v = fmaf(__builtin_amdgcn_exp2f((s[j][r / 4][r % 4] - most[r]) * c), wgt[r], v);
                static_for<0, NT>([&](auto ic) __attribute__((always_inline)) { colsum[ic][j] += ic == i ? v : 0.f; });
            }
        }
    }
    float *dst = out + ((size_t)slice * P + p) * n_pad;
    static_for<0, NT>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = ic;
        if (i < covered) {
#pragma unroll
            for (int j = 0; j < SUB; ++j) {
                const float v = rows4_sum(colsum[i][j]);
                if (lane < 16) dst[(i * W + wave) * KEYS + 16 * j + lane] = v;
            }
        }
    });
}

__global__ __launch_bounds__(COLUMN_BLOCK) void attn_single_sum_kernel(ColumnParts a)
{
    __shared__ float sums[4][64];
    add_column_parts(a, blockIdx.x, sums);
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------

struct SinglePlan {
    int waves = 0, tiles = 0, parts = 0;                     // waves of a workgroup, key tiles of a wave, workgroups of a slice
};

static int single_rows(const kvm_shape &sh) { return sh.dtype == KVM_F32 ? 16 : 32; }
static int single_stride(int N) { return (N + 31) / 32 * 32; }

// parts == 0: the two passes are the better choice.
//   waves, tiles  the fewest registers that hold the terms of the longest row; fewer waves a workgroup are more workgroups a compute unit
//          that cover each other's exchanges (1024 slices of 250 fp16 tokens, us, two waves of four tiles / four of four 37 / 47; of 128, one wave / two 21 / 23, both before the other changes to this kernel)
//   parts  as many as fill one to eight rounds of the workgroups that the chip holds, whichever takes the least: rounds times (the largest share
//          of units, in key tiles of a wave, each unit three more for its exchange, and three for a workgroup's start), and a twentieth of a
//          tile for every row of column sums beyond 32 that the sum kernel reads.  (Two rounds rounded up run into a third: us, two passes / that /
//          this, 36 slices of 1000 fp16 tokens 21.4 / 21.9 / 17.5, 40 of 2000 63 / 64.5 / 54.7, 200 of 1200 121 / 140 / 120; fp32, 33 of 2000 534 / 252 / 191.)  At least four a slice, or the slices that run at a time on an XCD outgrow its L2 (1024 slices of 1000, us,
//          1 / 2 / 4 / 8 / 16 / 32 parts 659 / 363 / 327 / 351 / 389 / 451), as many for every head, and no more than 64 units each (see redo)
// Longer rows.  16-bit types from 1025 tokens on: eight waves fill a compute unit alone, which a full launch of the other kernels beats (us, two passes /
// this: 1024 slices of 1100 467 / 577, 520 of 1100 229 / 267, 300 of 1200 1.04 times as long here), and a small one does not (200 of 1200 121 / 120, 128 of
// 2048 168 / 158, 96 of 1500 104 / 97, 40 of 2000 63 / 55, 8 of 2000 30 / 21; G = 4: 33 of 1500 115 / 109, 24 of 1500 94 / 92): up to 2^18
// query rows.  Longest against the split kernels at 33 to 72 heads of 1025 to 1280 tokens, up to 8 % (52 of 1030 29.6 / 31.8).  From 1300 tokens on the
// line would lie further out (256 of 2000 311 / 298).  fp32: 256 of 4096 8170 / 6120.
// And 513 to 768 tokens, where the other kernels' three row tiles are full and six key tiles a wave are held in the registers of eight: from 2^20 keys on
// (1024 slices of 700 0.94 times as long as two passes, of 768 0.96; 1800 of 700 1.05, 2048 of 768 1.07; G = 4: 520 of 700 1.02).
// Batches of differing lengths would gain as well (512 slices of 250 to 1000 tokens 142 / 94) and keep the two passes: there the column-sum
// kernels also write the similarities of kvm_attn_mass_sim, whose scores are bit for bit those of kvm_attn_mass.
constexpr long long SINGLE_LONG_ROWS = 1ll << 18, SINGLE_MID_KEYS = 1ll << 20;

constexpr int SINGLE_ROUNDS = 8, SINGLE_UNIT = 3, SINGLE_START = 3;

// the largest share of a head's units that one of its workgroups has, in key tiles of a wave
static int single_share(int units, int sharers, int waves)
{
    int first = 0, last = 0;                                 // of the workgroups 0 and sharers - 1: the others lie between
    for (int u = 0, k = 0; u < units; u += sharers, ++k) {
        const int near = (k & 1) ? u + sharers - 1 : u, far = 2 * u + sharers - 1 - near;
        if (near < units) first += (units - near + waves - 1) / waves + SINGLE_UNIT;
        if (far < units) last += (units - far + waves - 1) / waves + SINGLE_UNIT;
    }
    return std::max(first, last);
}

static SinglePlan single_plan(const kvm_shape &sh)
{
    SinglePlan pl;
    const bool f32 = sh.dtype == KVM_F32;
    const long long slices = (long long)sh.B * sh.H_kv;
    if (slices * sh.N == 0 || sh.seq_lens || sh.N > (f32 ? 4096 : 2048) || sh.G > 1024) return pl;
    if (!f32 && sh.N > 1024 && slices * sh.G * sh.N > SINGLE_LONG_ROWS) return pl;
    if (!f32 && sh.N > 512 && sh.N <= 768 && slices * sh.N > SINGLE_MID_KEYS) return pl;
    int resident;                                            // workgroups a compute unit holds
    if (f32) {
        pl.waves = sh.N <= 1024 ? 4 : 8;
        pl.tiles = sh.N <= 256 ? 4 : sh.N <= 512 ? 8 : sh.N <= 2048 ? 16 : 32;
        resident = sh.N <= 512 ? 3 : sh.N <= 1024 ? 2 : 1;
    } else {
        pl.waves = sh.N <= 128 ? 1 : sh.N <= 256 ? 2 : sh.N <= 1024 ? 4 : 8;
        pl.tiles = sh.N <= 512 ? 4 : 8;
        resident = sh.N <= 128 ? 9 : sh.N <= 256 ? 6 : sh.N <= 512 ? 3 : sh.N <= 1024 ? 2 : 1;
    }
    const long long units = (sh.N + single_rows(sh) - 1) / single_rows(sh);   // of a head
    const long long slots = 256ll * resident, heads = slices * sh.G, least = std::min(units, std::max((4ll + sh.G - 1) / sh.G, (units + 63) / 64));
    long long sharers = units, best = LLONG_MAX;
    for (long long rounds = 1, last = 0; rounds <= SINGLE_ROUNDS && last < units; ++rounds) {
        const long long s = std::min(units, std::max(least, rounds * slots / heads));
        if (s == last) continue;
        last = s;
        const long long cost = (heads * s + slots - 1) / slots * (single_share((int)units, (int)s, pl.waves) + SINGLE_START) * 20 + std::max(0ll, s * sh.G - 32);
        if (cost < best) best = cost, sharers = s;
    }
    const long long parts = sharers * sh.G;
    const long long limit = 1ll << 32;                       // threads of a launch
    if (slices * parts * pl.waves * WAVE >= limit || slices * ((sh.N + 63) / 64 + (sh.N + 255) / 256) * COLUMN_BLOCK >= limit)
        return SinglePlan();                                 // (the second launch may scan the keys as well)
    pl.parts = (int)parts;
    return pl;
}

// Workspace of the single pass (0: not taken): the workgroups' column sums.
size_t attn_single_bytes(const kvm_shape &sh)
{
    return (size_t)sh.B * sh.H_kv * single_plan(sh).parts * single_stride(sh.N) * sizeof(float);
}

template <typename T, int W, int NT, int OCC>
static void single_t(const kvm_shape &sh, const void *Q, const void *K, float *part, int P, float c, hipStream_t st)
{
    const int n_kv = sh.B * sh.H_kv;
    const long long blocks = (long long)n_kv * P;
    hipLaunchKernelGGL((attn_single_kernel<T, sizeof(T) == 2 ? 2 : 1, W, NT, OCC>), dim3((unsigned)blocks), dim3(W * WAVE), 0, st, (const T *)Q,
                       (const T *)K, part, n_kv, sh.G, sh.N, single_stride(sh.N), P / sh.G, c);
}

template <typename T>
static void single_dispatch(const SinglePlan &pl, const kvm_shape &sh, const void *Q, const void *K, float *part, float c, hipStream_t st)
{
    if constexpr (sizeof(T) == 2) {
        if (pl.waves == 1) single_t<T, 1, 4, 3>(sh, Q, K, part, pl.parts, c, st);
        else if (pl.waves == 2) single_t<T, 2, 4, 3>(sh, Q, K, part, pl.parts, c, st);
        else if (pl.waves == 4 && pl.tiles == 4) single_t<T, 4, 4, 3>(sh, Q, K, part, pl.parts, c, st);
        else if (pl.waves == 4) single_t<T, 4, 8, 2>(sh, Q, K, part, pl.parts, c, st);
        else single_t<T, 8, 8, 2>(sh, Q, K, part, pl.parts, c, st);
    } else {
        if (pl.tiles == 4) single_t<T, 4, 4, 3>(sh, Q, K, part, pl.parts, c, st);
        else if (pl.tiles == 8) single_t<T, 4, 8, 3>(sh, Q, K, part, pl.parts, c, st);
        else if (pl.waves == 4) single_t<T, 4, 16, 2>(sh, Q, K, part, pl.parts, c, st);
        else if (pl.tiles == 16) single_t<T, 8, 16, 2>(sh, Q, K, part, pl.parts, c, st);
        else single_t<T, 8, 32, 2>(sh, Q, K, part, pl.parts, c, st);
    }
}

// sim != nullptr: the similarities as well.
kvm_status launch_attn_single(const kvm_shape &sh, const void *Q, const void *K, float *mass, float *part, float *sim, hipStream_t st)
{
    const float c = (float)(1.4426950408889634 / sqrt((double)sh.d));
    const SinglePlan pl = single_plan(sh);
    {
        ProfScope prof("attn_single_kernel", st);
        if (sh.dtype == KVM_F32) single_dispatch<float>(pl, sh, Q, K, part, c, st);
        else if (sh.dtype == KVM_F16) single_dispatch<half_t>(pl, sh, Q, K, part, c, st);
        else single_dispatch<bf16_t>(pl, sh, Q, K, part, c, st);
        kvm_status rc = check_launch("attn_single_kernel");
        if (rc != KVM_OK) return rc;
    }
    ColumnParts sums;
    sums.part = part;
    sums.mass = mass;
    sums.G = sh.G;
    sums.n = sh.N;
    sums.n_pad = single_stride(sh.N);
    sums.P = pl.parts;
    sums.rows = single_rows(sh);
    sums.blocks_per_slice = (sh.N + 63) / 64;
    if (sim) return launch_cosine_scan_and_sums(sh, K, sim, sums, st);
    ProfScope prof("attn_single_sum_kernel", st);
    hipLaunchKernelGGL(attn_single_sum_kernel, dim3((unsigned)((long long)sums.blocks_per_slice * sh.B * sh.H_kv)), dim3(COLUMN_BLOCK), 0, st, sums);
    return check_launch("attn_single_sum_kernel");
}

}  // namespace kvm
