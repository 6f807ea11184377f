// Decode-time update of the aggregated attention scores: the newest token's query attends to
// all keys of the cache (Section 2.4 Eq. (1) for one query row), and the row is added into
// the column sums (Section 4.2 Eq. (7): a sum over query rows, so one more row is one more
// term per key).
//
// One query row against N keys is a matrix-vector product: every key is read once and used
// for G dot products, so the update is bound by the HBM read of K (N d s bytes per slice) and
// the matrix cores have nothing to offer.  Two launches, because the softmax denominator
// spans the whole row:
//   append_scores_kernel      thread j of a workgroup owns key j of a 256-key tile; a row is
//                             spread over 16 lanes as in the other streaming kernels.  Scores
//                             (base-2 logarithm units) go to the workspace, with the maximum
//                             and the sum of exponentials of every wave's 64 keys beside them
//                             (no exchange between waves, so no barrier).
//   append_accumulate_kernel  merges the pieces' statistics of every query head into its
//                             log-sum-exp and adds exp2(score - lse) of all G heads to mass.
#include <algorithm>

#include "kvm_common.h"

namespace kvm {

constexpr int APP_BLOCK = 256;
constexpr int APP_ROWS_PER_GROUP = 16;                      // one row per lane of the group in the end
constexpr int APP_WAVES = APP_BLOCK / WAVE;
constexpr int ACC_PER_THREAD = 4;                           // keys per thread of the second kernel
constexpr int ACC_HEADS = 16;                               // query heads between two barriers of it
constexpr int ACC_CHUNK = APP_BLOCK * ACC_PER_THREAD;
constexpr int ACC_MAX_CHUNKS = 256;                         // workgroups per slice
constexpr int ACC_SHARED_PIECES = 512;                      // longer lists of statistics may be walked by all waves

int attn_lse_stride(int N);

// A wave's 64 values under a commutative operation, every lane gets the result: lanes i and i ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1 in turn, the rows by
// swaps and then within a row by rotations (what they combine repeats every 16, 8, 4, 2 lanes, so a rotation by half of that is the
// exchange).  On the vector ALU: by LDS moves the twelve exchanges of a query head are a chain of twelve LDS round trips (score kernel, us, LDS / this: 8
// slices of 2000 fp16 tokens, G = 8, 13.4 / 12.4, 32 of 3000 in fp32 21.2 / 20.2, of 1000, G = 1, 6.8 / 6.4).
template <typename F> __device__ __forceinline__ float wave_all(float v, F op) {
    const uint32_t a = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    const uint32_t b = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)));
    const auto t = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    const uint32_t t0 = t[0], t1 = t[1];
    v = op(__builtin_bit_cast(float, t0), __builtin_bit_cast(float, t1));
    v = op(v, dpp_f<0x128>(v));                               // row_ror:8
    v = op(v, dpp_f<0x124>(v));
    v = op(v, dpp_f<0x122>(v));
    return op(v, dpp_f<0x121>(v));
}
__device__ __forceinline__ float wave_max(float v) { return wave_all(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float wave_sum(float v) { return wave_all(v, [](float a, float b) { return a + b; }); }

// The next head's query is loaded while a head is worked out (us, without / with: 8 slices of 2000 fp16 tokens, G = 8, 12.5 / 11.1, 32 of 3000 in bf16,
// G = 4, 11.3 / 10.8); six waves a SIMD in 16 bit, as without it.
template <typename T>
__global__ __launch_bounds__(APP_BLOCK, sizeof(T) == 2 ? 6 : 3) void append_scores_kernel(const T *__restrict__ q_new, const T *__restrict__ K,
                                                                   float *__restrict__ scores, float *__restrict__ stats,
                                                                   const int32_t *__restrict__ seq_lens, int H, int G,
                                                                   int N, int n_pad, int tiles_per_slice, int stream_from, float c)
{
    typedef typename Elem<T>::Raw Raw;
    const int slice = blockIdx.x / tiles_per_slice;          // (b, h)
    const int tile = blockIdx.x - slice * tiles_per_slice;
    const int b = slice / H;
    const int n = clamp_len(seq_lens, b, N);
    const int j_wave = tile * APP_BLOCK + (threadIdx.x & ~63);   // a wave's 64 keys share one pair of statistics
    if (j_wave >= n) return;                                 // the other kernel looks at keys below n only
    const int lane16 = threadIdx.x & 15, group = threadIdx.x >> 4;
    const int j0 = tile * APP_BLOCK + group * APP_ROWS_PER_GROUP;
    const T *Ks = K + (size_t)slice * N * HEAD_DIM;

    // all rows of the group at once; rows past the end repeat the last valid one and are masked below
    Raw raw[APP_ROWS_PER_GROUP];
    load_rows_once<T, APP_ROWS_PER_GROUP>(Ks, j0, n, lane16, stream_from, raw);

    const T *q_row = q_new + (size_t)slice * G * HEAD_DIM;
    Raw q_next = Elem<T>::load(q_row, lane16);
    const int j = tile * APP_BLOCK + threadIdx.x;            // the key whose score this thread keeps
    const int stats_per_row = n_pad / WAVE;
    for (int g = 0; g < G; ++g) {
        const size_t qslice = (size_t)slice * G + g;
        const Raw q = q_next;
        if (g + 1 < G) q_next = Elem<T>::load(q_row + (size_t)(g + 1) * HEAD_DIM, lane16);   // on its way while this head is worked out
        float mine = 0.f;
#pragma unroll
        for (int i = 0; i < APP_ROWS_PER_GROUP; ++i) {
            const float dot = row16_sum(RowDot<T>::dot(raw[i], q));
            if (lane16 == i) mine = dot;
        }
        const float x = j < n ? mine * c : -INFINITY;
        if (j < n) scores[qslice * n_pad + j] = x;
        const float m = wave_max(x);                         // finite: key j_wave is below n
        const float l = wave_sum(__builtin_amdgcn_exp2f(x - m));
        if ((threadIdx.x & 63) == 0) {
            float *st = stats + (qslice * stats_per_row + j_wave / WAVE) * 2;
            st[0] = m;
            st[1] = l;
        }
    }
}

// Statistics [first, last) of a query row put on their maximum m, by one wave: the sum of exponentials (maximum first, sums
// scaled to it).  Every lane gets both.
__device__ __forceinline__ float row_sum(const float *st, int first, int last, float &m) {
    const int lane = threadIdx.x & 63;
    float tm = -INFINITY;
    for (int t = first + lane; t < last; t += WAVE) tm = fmaxf(tm, st[2 * t]);
    m = wave_max(tm);
    float tl = 0.f;
    for (int t = first + lane; t < last; t += WAVE) tl += st[2 * t + 1] * __builtin_amdgcn_exp2f(st[2 * t] - m);
    return wave_sum(tl);
}

// The log-sum-exps of query heads [g0, g0 + heads), heads <= ACC_HEADS, by a workgroup, -> lse_of in LDS.  The waves take the heads in
// turn.  SHARED: a quarter of every list a wave, for long lists and heads that do not come out even, where the waves without a list
// would wait for the others.  us, in turn / shared: one slice of 131072 keys, one head, 15.1 / 8.3, two 16.9 / 11.9, four 17.9 / 19.4,
// eight 30.8 / 34.0; of 32768, one head 7.6 / 6.1, three 8.7 / 9.0, four 9.4 / 10.5.
template <bool SHARED>
__device__ __forceinline__ void row_lses(const float *stats, int stats_per_row, int g0, int heads, int pieces, float *lse_of, float2 (*part)[APP_WAVES]) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (!SHARED) {
        for (int g = wave; g < heads; g += APP_WAVES) {
            float m;
            const float l = row_sum(stats + (size_t)(g0 + g) * stats_per_row * 2, 0, pieces, m);
            if (lane == 0) lse_of[g] = m + __log2f(l);
        }
        __syncthreads();
        return;
    }
    const int quarter = (pieces + APP_WAVES - 1) / APP_WAVES;
    for (int g = 0; g < heads; ++g) {
        float m;
        const float l = row_sum(stats + (size_t)(g0 + g) * stats_per_row * 2, wave * quarter, min((wave + 1) * quarter, pieces), m);
        if (lane == 0) part[g][wave] = make_float2(m, l);
    }
    __syncthreads();
    if ((int)threadIdx.x < heads) {
        float m = -INFINITY, l = 0.f;
#pragma unroll
        for (int w = 0; w < APP_WAVES; ++w) m = fmaxf(m, part[threadIdx.x][w].x);
#pragma unroll
        for (int w = 0; w < APP_WAVES; ++w) l += part[threadIdx.x][w].y * __builtin_amdgcn_exp2f(part[threadIdx.x][w].x - m);
        lse_of[threadIdx.x] = m + __log2f(l);
    }
    __syncthreads();
}

// ACC_HEADS query heads between two barriers; a single head of a short list is worked out by every wave for itself.
// (All waves on one head after the other with three barriers each, and eight keys a thread, before / now, us: 32 slices of 3000
// keys, G = 4, 18.4 / 7.3; 8 of 1000, G = 8, 20.9 / 9.3; 64 of 16000, G = 2, 14.3 / 8.5; 1024 of 4096 18.2 / 15.2.)
// Every workgroup needs the statistics of all keys, N / 64 pairs a head, so no slice gets more than ACC_MAX_CHUNKS of them: beyond,
// they take several chunks of keys each, or the reads would grow with the square of N (us, a workgroup per chunk / this, and the lists
// shared: one slice of 262144 keys 28.6 / 12.0, of 1048576 99.8 / 31.6, of 4194304 1113 / 115).  LONG: rows that may need either.
template <bool LONG>
__global__ __launch_bounds__(APP_BLOCK) void append_accumulate_kernel(const float *__restrict__ scores,
                                                                       const float *__restrict__ stats, float *__restrict__ mass,
                                                                       const int32_t *__restrict__ seq_lens, int H, int G, int N,
                                                                       int n_pad, int chunks_per_slice)
{
    __shared__ float lse_of[ACC_HEADS];
    __shared__ float2 part[ACC_HEADS][APP_WAVES];
    const int slice = blockIdx.x / chunks_per_slice;
    const int n = clamp_len(seq_lens, slice / H, N);
    const int keys = LONG ? (n + ACC_CHUNK * ACC_MAX_CHUNKS - 1) / (ACC_CHUNK * ACC_MAX_CHUNKS) * ACC_CHUNK : ACC_CHUNK;   // of this workgroup
    const int j_first = (blockIdx.x - slice * chunks_per_slice) * keys;
    if (j_first >= n) return;
    const int pieces = (n + WAVE - 1) / WAVE;                // statistics come per 64 keys
    const int stats_per_row = n_pad / WAVE;
    const float *row = scores + (size_t)slice * G * n_pad, *st = stats + (size_t)slice * G * stats_per_row * 2;
    float *a = mass + (size_t)slice * N;
    float own_lse = 0.f;
    for (int j_block = j_first; j_block < min(j_first + keys, n); j_block += ACC_CHUNK) {
    float add[ACC_PER_THREAD], before[ACC_PER_THREAD];
#pragma unroll
    for (int u = 0; u < ACC_PER_THREAD; ++u) {
        const int j = j_block + u * APP_BLOCK + threadIdx.x;
        add[u] = 0.f;
        before[u] = j < n - 1 ? a[j] : 0.f;                  // the newest token's entry starts here
    }
    for (int g0 = 0; g0 < G; g0 += ACC_HEADS) {
        const int heads = min(ACC_HEADS, G - g0);
        float x[ACC_PER_THREAD];                             // the first head's scores, on their way meanwhile
#pragma unroll
        for (int u = 0; u < ACC_PER_THREAD; ++u) {
            const int j = j_block + u * APP_BLOCK + threadIdx.x;
            x[u] = j < n ? row[(size_t)g0 * n_pad + j] : -INFINITY;
        }
        const bool shared = LONG && pieces > ACC_SHARED_PIECES && heads % APP_WAVES != 0, alone = heads == 1 && !shared;
        if (j_block == j_first || G > ACC_HEADS) {           // (else they are there from the chunk before)
            if (alone) {
                float m;
                const float l = row_sum(st + (size_t)g0 * stats_per_row * 2, 0, pieces, m);
                own_lse = m + __log2f(l);
            } else {
                if (g0 > 0 || j_block > j_first) __syncthreads();   // the heads before have been read
                if (shared) row_lses<true>(st, stats_per_row, g0, heads, pieces, lse_of, part);
                else row_lses<false>(st, stats_per_row, g0, heads, pieces, lse_of, part);
            }
        }
        float lse = alone ? own_lse : lse_of[0];
        for (int g = 0;;) {
            const float l = lse;
            float next[ACC_PER_THREAD];
            const bool more = g + 1 < heads;
            if (more) {
                lse = lse_of[g + 1];
#pragma unroll
                for (int u = 0; u < ACC_PER_THREAD; ++u) {
                    const int j = j_block + u * APP_BLOCK + threadIdx.x;
                    next[u] = j < n ? row[(size_t)(g0 + g + 1) * n_pad + j] : -INFINITY;
                }
            }
#pragma unroll
            for (int u = 0; u < ACC_PER_THREAD; ++u) add[u] += __builtin_amdgcn_exp2f(x[u] - l);
            if (!more) break;
            ++g;
#pragma unroll
            for (int u = 0; u < ACC_PER_THREAD; ++u) x[u] = next[u];
        }
    }
#pragma unroll
    for (int u = 0; u < ACC_PER_THREAD; ++u) {
        const int j = j_block + u * APP_BLOCK + threadIdx.x;
        if (j < n) a[j] = before[u] + add[u];
    }
    }
}

template <typename T>
static kvm_status launch_t(const kvm_shape &sh, const void *q_new, const void *K, float *mass, float *ws, hipStream_t st)
{
    const int tiles = (sh.N + APP_BLOCK - 1) / APP_BLOCK;
    const int n_pad = attn_lse_stride(sh.N);
    const size_t n_q = (size_t)sh.B * sh.H_kv * sh.G;
    float *scores = ws, *stats = ws + n_q * n_pad;
    const float c = (float)(1.4426950408889634 / sqrt((double)sh.d));
    const long long blocks = (long long)sh.B * sh.H_kv * tiles;
    {
        ProfScope prof("append_scores_kernel", st);
        // From half the last-level cache on the keys are read with the non-temporal hint: with them the compacted rows that
        // the refresh moves next, as large again, would not fit.  Token loop, us, plain / hint: 32 slices of 8192 tokens
        // (64 MiB) 92 / 93, of 12288 114 / 117, of 16384 151 / 143, of 32768 442 / 364; 1024 of 4096 449 / 403 (this kernel 236 / 190).
        hipLaunchKernelGGL(append_scores_kernel<T>, dim3((unsigned)blocks), dim3(APP_BLOCK), 0, st, (const T *)q_new, (const T *)K,
                           scores, stats, sh.seq_lens, sh.H_kv, sh.G, sh.N, n_pad, tiles, stream_length(sh, LLC_BYTES / 2), c);
    }
    kvm_status rc = check_launch("append_scores_kernel");
    if (rc != KVM_OK) return rc;
    ProfScope prof("append_accumulate_kernel", st);
    const int chunks = std::min((sh.N + ACC_CHUNK - 1) / ACC_CHUNK, ACC_MAX_CHUNKS);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((long long)sh.B * sh.H_kv * chunks)), dim3(APP_BLOCK), 0, st, (const float *)scores,
                           (const float *)stats, mass, sh.seq_lens, sh.H_kv, sh.G, sh.N, n_pad, chunks);
    };
    if (sh.N > ACC_SHARED_PIECES * WAVE) run(append_accumulate_kernel<true>);
    else run(append_accumulate_kernel<false>);
    return check_launch("append_accumulate_kernel");
}

// ws: scores (B H_kv G, stride attn_lse_stride(N)) followed by two floats per (query slice, 64 keys).
kvm_status launch_attn_append(const kvm_shape &sh, const void *q_new, const void *K, float *mass, float *ws, hipStream_t st)
{
    if ((long long)sh.B * sh.H_kv == 0 || sh.N == 0) return KVM_OK;
    switch (sh.dtype) {
    case KVM_F32: return launch_t<float>(sh, q_new, K, mass, ws, st);
    case KVM_F16: return launch_t<half_t>(sh, q_new, K, mass, ws, st);
    default: return launch_t<bf16_t>(sh, q_new, K, mass, ws, st);
    }
}

}  // namespace kvm
