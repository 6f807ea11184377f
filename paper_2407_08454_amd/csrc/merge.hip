// Gaussian-kernel weighted merging with a compacting write (Section 4.2: Def. 4.2 Eq. (4),
// Eq. (5), (6); Algorithm 2).
//
// Work is dealt out by tokens, not by sets, because set lengths are very uneven (most sets
// are conserved singletons, most tokens sit in sets of 17..128): one wave owns the sets that
// start inside its tile of 16 or 32 tokens, and finds the first of them itself.  A row of 128 elements is spread over 16 lanes
// (8 elements = 16 B each for 16-bit types), so one wave instruction moves four rows.  Per
// set: one sweep over its keys for the distances to the pivot (sigma), a second sweep (served
// by L2, the set was just read) that forms the weights and accumulates keys and values in
// fp32, then one rounded row is written per output.  Loads are issued 16 rows at a time; a
// set of up to 16 tokens is read exactly once and held in registers.  Runs of singleton sets
// are copied bit for bit.  HBM traffic: K once, V once, 2 M rows out.
//
// Kernels:
//   merge_kernel        one wave per tile (merge_one_set per set, runs of singletons copied); in small launches
//                       four tiles a workgroup, whose waves merge the longer sets together (merge_set_team)
//   merge_long_kernel   the sets of more than LONG_SET_MIN tokens, one 1024-thread workgroup per slice
//   refresh_kernel      decode time: compares the new maps with the previous ones, moves the rows of
//                       unchanged sets in place and merges the changed sets again
#include <limits.h>

#include "kvm_common.h"

namespace kvm {

// Tokens per wave (its sets are those that start in the tile).  A wave merges its sets one after the other, a
// memory round trip or more for each, so short chains of many waves cover the latency better than long ones;
// against them stands the look-up of the first set, two or three dependent loads a wave.  Measured, us, with
// tiles of 64 from a table that a launch of its own filled / 32 / 16: 8 slices of 1000 tokens 27.4 / 16.3 /
// 14.1; 64 of 4096 60 / 47 / 44.5; 256 of 1024 in fp32 110 / 106 / 90; 128 of 4096 110 / 92 / 96; 256 of
// 4096 201 / 180 / 185; 1024 of 4096 628 / 597 / -.  Tiles of 64 with the look-up: 1024 slices of 4096 1-2 % slower
// than with the table.  Hence 16 up to 2^18 tokens, where the waves fit the chip four times over, 32 beyond.
// In the larger launches the slices go out in groups of eight, so that a slice's tiles, which read the same map entries,
// stay on one XCD: workgroups are dealt round-robin to the eight of them.  Dealt out slice by slice, a slice of 256 tokens
// sends its tile t, with the work of that part of a sequence, to XCD t every time.  Within an XCD two or four tiles a slice
// fall into step with its units in the same way, so the first tile of a slice moves on with the group, in steps of no period.
// The XCD of a slice's place in its group moves on as well: lengths that repeat every four rows would leave the same XCDs idle
// (300 slices of 1024 to 4096 tokens 168 / 131, slice by slice 136; 9000 of 25 to 100 126 / 100).
// Launches of 2^18 tokens or fewer are resident at once and gain nothing, and eight long slices at a time, one an XCD, differ too
// much in their work (256 slices of 16384 576 / 596, 8 of 65536 113 / 117).  Measured, us, slice by slice / in groups / in groups
// with moving first tile: 4096 slices of 256 tokens, budget 0.35, 221 / 165 / 149 (tiles of 64 from a table: 193); 9000 of 100
// 232 / 227 / 145 (190); 16000 of 64 198 / 193 / 156 (167); 1024 of 1024 214 / 155 / 155 (216); 1024 of 4096 572 / 532 / 532 (611).
constexpr int MERGE_TILE_FEW = 16, MERGE_TILE = 32;
constexpr long long MERGE_FEW_TOKENS = 1 << 18;
constexpr int MERGE_GROUPED_TILES = 128;                     // per slice
// In a small launch the longest set is what everything waits for: a wave takes about 1200 cycles for 16 of its rows and sweep, 15 us
// for 250 tokens, when the median wave is done in one.  So up to 96 K tokens four waves share a workgroup, and after their
// tiles merge the sets of more than SPLIT_SET_MIN tokens together, a quarter each.  us, one wave a workgroup / four: one slice of 512
// fp32 tokens 13.8 / 10.8, 32 of 1000 20.9 / 16.2, of 2000 29.4 / 22.0, of 3000 27.6 / 25.9 (fp32 33.1 / 33.0), 8 of 8000 29.1 / 21.5;
// beyond, where the waves of a workgroup that wait for the slowest leave their places empty: 100 of 1000 26.5 / 29.5, 32 of 4000
// 26.6 / 28.7, 64 of 8000 75 / 91, 1024 of 4096 577 / 980.
constexpr long long MERGE_TEAM_TOKENS = 3 << 15;
// The merged rows go out with the non-temporal hint where keys, values and the compacted cache come to more than the last-level cache holds:
// that keeps the keys for their second sweep and what is left of the inputs in it.  In smaller launches who reads the compacted cache
// next, the attention of the next token, finds it in the cache.  Budget 0.5, us, compaction / compaction and a read of the merged rows, plain / hint:
// 40 slices of 3000 fp16 tokens (29 MiB of keys) 43.4 / 43.2 and 59.4 / 60.4, 64 of 4096 (64 MiB) 63.8 / 63.5 and 86.4 / 87.1, 96 of them 91.4 / 84.5 and
// 119.5 / 115.6, 128 110.8 / 106.7 and 146.5 / 144.3; fp32: 40 of 3000 57.6 / 57.9 and 76.5 / 77.9, 64 of 3000 83.2 / 79.2 and 107.2 / 106.9; merge alone,
// 1024 of 4096 in fp16 567 / 550, in fp32 1100 / 1068.
static bool streams_rows(const kvm_shape &sh, int cap_rows) { return 2 * token_bytes(sh) * ((long long)sh.N + cap_rows) >= LLC_BYTES; }
// Sets of more than LONG_SET_MIN tokens are left to merge_long_kernel, which puts a whole workgroup
// on each of them: one wave would stream such a set for hundreds of dependent round trips while
// the rest of the chip has nothing to do (identical keys make one set of a whole slice).
constexpr int LONG_SET_MIN = 512;
constexpr int LONG_SET_BLOCK = 1024;
constexpr int LONG_SET_LOOK = 4;         // sets a thread looks at between two barriers of the look-up
// 4-row groups whose loads are issued together: 16 rows of K and of V.  Larger batches read
// more sets in a single sweep but cost registers; the kernel is bound by memory latency, and
// four waves per SIMD with 16-row batches beat two waves with 32-row batches.
template <typename T> struct MergeUnroll { static constexpr int value = 4; };

// int32 entries of workspace per slice that the callers of a merge bring.  The refresh keeps its list of long
// sets in the last N / (LONG_SET_MIN + 1) + 2 of them; a full merge needs none, but its entry points go on
// asking for the same size (kvm_workspace_bytes, the limit of kvm_merge_static).
static int long_list_offset(int N) { return (N + 63) / 64 + 1; }   // the number of listed sets, their indices after it
static __host__ __device__ int max_long_sets(int N) { return N / (LONG_SET_MIN + 1) + 1; }
static int merge_ws_stride(int N) { return long_list_offset(N) + 1 + max_long_sets(N); }

size_t merge_workspace_bytes(const kvm_shape &sh)
{
    return (size_t)sh.B * sh.H_kv * merge_ws_stride(sh.N) * sizeof(int32_t);
}

struct MergeArgs {
    const int32_t *set_start, *pivot, *n_sets, *seq_lens;
    float *w_opt;
    const int32_t *long_list;   // NULL (every long set of the maps is merged), or per slice, list_stride entries
                                // apart: the number of long sets to merge, then their indices
    int list_stride;
    int slices, H, N, cap_rows;
    int tile, tiles_per_slice;  // tokens per wave (merge_kernel)
    int mode;               // MERGE_ADAPTIVE, MERGE_FIXED (uses inv_two_sigma_sq) or MERGE_AVERAGE
    float inv_two_sigma_sq; // 1 / (2 sigma^2) for the fixed-sigma mode
    int value_scale;
};

// Smallest s in [0, M] with set_start[s] >= edge (M if there is none), by one wave: 64 probes of the
// remaining range a round, so two dependent loads up to 4160 sets and three up to 266304.  The starts of
// consistent maps ascend; for any other maps the result is some value in [0, M].
__device__ __forceinline__ int first_set_at(const int32_t *sst, int M, int edge, int lane) {
    int lo = 0, len = M;                                     // the result lies in [lo, lo + len]
    while (len > 0) {
        const int step = (len + WAVE - 1) / WAVE;
        const int at = lane * step;
        const int below = __popcll(__ballot(at < len && sst[lo + min(at, len - 1)] < edge));
        if (below == 0) break;
        const int skip = (below - 1) * step + 1;             // <= len: probe below - 1 lies inside the range
        lo += skip;
        len = min(step - 1, len - skip);
    }
    return lo;
}

// LDS written by some lanes of a wave is read by others of the same wave after this: the hardware keeps a wave's LDS operations
// in order, so it only holds the compiler.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// In the launches that stream their merged rows, 16-bit rows that are read once carry the hint too: values, and keys of single tokens and of
// sets of up to 16.  It leaves the caches to the keys of the longer sets' second sweep.  us, without / with: sets and merge of 1600 slices of 500 bf16
// tokens 135 / 126, 1024 of 2000 fp16 376 / 367, 1024 of 4096 759 / 748, 1600 of 4096 in bf16 1085 / 1071, 640 of 16384 1751 / 1743.  Not
// in fp32, where it costs time: 1024 of 4096 1474 / 1540.
template <typename T, bool STREAM> constexpr bool reads_once() { return STREAM && sizeof(T) == 2; }

// Chunk c of a row of a slice.  A slice has less than 2^32 bytes, so scalar base and 32-bit offset: half the address arithmetic and a
// register instead of two.
template <typename T, bool ONCE = false>
__device__ __forceinline__ typename Elem<T>::Raw row_chunk(const T *slice, int row, int c) {
    const uint32_t at = (uint32_t)row * (uint32_t)(HEAD_DIM * sizeof(T)) + (uint32_t)c * (uint32_t)(8 * sizeof(T));
    const T *row_at = reinterpret_cast<const T *>(reinterpret_cast<const char *>(slice) + at);
    if constexpr (ONCE) return Elem<T>::load_stream(row_at, 0);
    else return Elem<T>::load(row_at, 0);
}

// A row that is copied: lane c of 16 moves the pieces c, c + 16 of 16 bytes, so that every store of a wave writes whole rows or half rows
// (where an fp32 lane stored its 32 bytes in two, each store wrote every other 16 bytes, and the non-temporal hint sent them out like that: copies of all
// tokens of 64 slices of 4096 in fp32, plain / that with the hint / this 105 / 93 / 86 us, of 512 slices 806 / 916 / 851; merge of 1024 of AR(1) keys
// 1148 / 1110 / 1068).
template <typename T> struct CopiedRow {
    u32x4 piece[sizeof(T) / 2];
    template <bool ONCE> __device__ __forceinline__ void load(const T *slice, int row, int c) {
        const uint32_t at = (uint32_t)row * (uint32_t)(HEAD_DIM * sizeof(T)) + (uint32_t)c * 16u;
#pragma unroll
        for (int h = 0; h < (int)sizeof(T) / 2; ++h)
            if constexpr (ONCE) piece[h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(slice) + at + 256 * h));
            else piece[h] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(slice) + at + 256 * h);
    }
    template <bool STREAM> __device__ __forceinline__ void store(T *row, int c) const {
        u32x4 *p = reinterpret_cast<u32x4 *>(row) + c;
#pragma unroll
        for (int h = 0; h < (int)sizeof(T) / 2; ++h) {
            if constexpr (STREAM) __builtin_nontemporal_store(piece[h], p + 16 * h);
            else p[16 * h] = piece[h];
        }
    }
};

// Squared distance of 8 elements, summed over the 16 lanes of the row.
__device__ __forceinline__ float sq_dist16(const float *kp, const float *x) {
    float d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = kp[e] - x[e];
    const float s0 = fmaf(d[1], d[1], d[0] * d[0]), s1 = fmaf(d[3], d[3], d[2] * d[2]);
    const float s2 = fmaf(d[5], d[5], d[4] * d[4]), s3 = fmaf(d[7], d[7], d[6] * d[6]);
    return row16_sum((s0 + s1) + (s2 + s3));
}

// WITH_W: also write the per-token weights.  MODE: how the weights are formed -- Gaussian
// kernel with sigma derived from the set, Gaussian kernel with a given sigma, or uniform
// (average weighted merging).  Both are compile-time so that the row loops stay free of
// branches and the compiler can interleave the independent rows.
enum { MERGE_ADAPTIVE = 0, MERGE_FIXED = 1, MERGE_AVERAGE = 2 };

// The part of a merged row that is written: all of keys and values, or the chunks [c0, c1) of one of them (which: 0 keys, 1 values).
struct RowPart {
    int which = -1, c0 = 0, c1 = 16;
    __device__ __forceinline__ bool holds(int row, int c) const { return which < 0 || (row == which && c >= c0 && c < c1); }
};

// Partial sums of a set, of the rows a lane has seen (8 columns of every fourth row): keys, values, weights.
struct SetSums { float k[8], v[8], g; };
__device__ __forceinline__ void clear(SetSums &s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s.k[e] = s.v[e] = 0.f;
    s.g = 0.f;
}
// a lane's sums in LDS: 17 floats, WAVE apart
constexpr int PARKED = 17 * WAVE;
__device__ __forceinline__ void park(const SetSums &s, float *at) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { at[e * WAVE] = s.k[e]; at[(8 + e) * WAVE] = s.v[e]; }
    at[16 * WAVE] = s.g;
}
__device__ __forceinline__ void add_parked(SetSums &s, const float *at) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { s.k[e] += at[e * WAVE]; s.v[e] += at[(8 + e) * WAVE]; }
    s.g += at[16 * WAVE];
}

// A set of more than SPLIT_SET_MIN tokens is summed in four parts, whole 16-row batches, and the parts are added
// up in order: by one wave, one part after the other, or by four waves at once.  Either way a set gets the same bits.
constexpr int SPLIT_SET_MIN = 128;
constexpr int SPLIT_PARTS = 4;
__device__ __forceinline__ int part_rows(int m) { return ((m + 15) / 16 + SPLIT_PARTS - 1) / SPLIT_PARTS * 16; }

// The steps of merging one set [lo, hi) with pivot p, 16 rows at a time, each for its rows [from, to) (counted from lo, from a
// multiple of 16).
template <typename T, bool WITH_W, int MODE, bool STREAM> struct SetMerge {
    using E = Elem<T>;
    using Raw = typename E::Raw;
    static constexpr int U = MergeUnroll<T>::value;            // row groups (of 4 rows) in flight
    static constexpr bool READ_ONCE = reads_once<T, STREAM>();
    const T *Ks, *Vs;
    float *wo;
    const MergeArgs &a;
    int lo, hi, lane, slot, c;                                 // slot: which of the four rows of an instruction; c: which 8-element chunk of the row
    float kp[8];

    __device__ __forceinline__ SetMerge(const T *Ks, const T *Vs, float *wo, const MergeArgs &a, int lo, int hi, int lane)
        : Ks(Ks), Vs(Vs), wo(wo), a(a), lo(lo), hi(hi), lane(lane), slot(lane >> 4), c(lane & 15) {}
    // Rows past the end of the set are clamped to its last row and given weight zero, so
    // that every lane runs the same straight-line code.
    template <bool ONCE = false> __device__ __forceinline__ void load_rows(const T *base, int j0, Raw *r) const {
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = row_chunk<T, ONCE>(base, min(j0 + 4 * u + slot, hi - 1), c);
    }
    // distances to the pivot -> dist (LDS, one per row)
    __device__ __forceinline__ void batch_distances(int j0, const Raw *kr, float *dist) const {
        float mine = 0.f;                                     // lane c of a row group keeps the distance of row group c
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float x[8];
            E::to_float(kr[u], x);
            const float d = __builtin_amdgcn_sqrtf(sq_dist16(kp, x));
            mine = c == u ? d : mine;
        }
        if (c < U) dist[j0 - lo + 4 * c + slot] = mine;
    }
    // (two batches on their way at a time: there are registers for them here, not in the sums)
    __device__ __forceinline__ void distances(int from, int to, float *dist) const {
        int j0 = lo + from;
        for (; j0 + 4 * U < lo + to; j0 += 8 * U) {
            Raw kr[2][U];
            load_rows(Ks, j0, kr[0]);
            load_rows(Ks, j0 + 4 * U, kr[1]);
            __builtin_amdgcn_sched_barrier(0);
            batch_distances(j0, kr[0], dist);
            batch_distances(j0 + 4 * U, kr[1], dist);
        }
        if (j0 < lo + to) {
            Raw kr[U];
            load_rows(Ks, j0, kr);
            batch_distances(j0, kr, dist);
        }
    }
    // g_j = exp(-D_j^2 / (2 sigma^2)); with sigma = dsum / (sqrt(2) m) that is exp(-(D_j m / dsum)^2).  One row a lane; zero past
    // the end of the set.  From the distances of all rows.
    __device__ __forceinline__ void weights(int from, int to, const float *dist, float *w) const {
        const int m = hi - lo;
        float dsum = 0.f;
        for (int i = lane; i < m; i += WAVE) dsum += dist[i];
        dsum = rows4_sum(row16_sum(dsum));
        const float inv_mean = dsum > 0.f ? (float)m / dsum : 0.f;
        for (int i = from + lane; i < ((to + 4 * U - 1) & -(4 * U)); i += WAVE) {
            const float r = dist[i] * inv_mean;
            const float g = i < m ? __expf(-r * r) : 0.f;
            w[i] = g;
            if (WITH_W && i < m) wo[lo + i] = g;
        }
    }
    // weighted sums; the weights from LDS, or for the fixed modes as they come
    __device__ __forceinline__ void batch_sums(int j0, const Raw *kr, const Raw *vr, const float *w, SetSums &s) const {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = j0 + 4 * u + slot;
            float x[8], v[8], g;
            E::to_float(kr[u], x);
            if (MODE == MERGE_ADAPTIVE) {
                g = w[row - lo];
            } else {
                g = MODE == MERGE_AVERAGE ? 1.f : __expf(-sq_dist16(kp, x) * a.inv_two_sigma_sq);
                g = row < hi ? g : 0.f;
                if (WITH_W && c == 0 && row < hi) wo[row] = g;
            }
            E::to_float(vr[u], v);
            s.g += g;
#pragma unroll
            for (int e = 0; e < 8; ++e) { s.k[e] = fmaf(g, x[e], s.k[e]); s.v[e] = fmaf(g, v[e], s.v[e]); }
        }
    }
    __device__ __forceinline__ void add_sums(int from, int to, const float *w, SetSums &s) const {
        for (int j0 = lo + from; j0 < lo + to; j0 += 4 * U) {
            Raw kr[U], vr[U];
            load_rows(Ks, j0, kr);
            load_rows<READ_ONCE>(Vs, j0, vr);
            __builtin_amdgcn_sched_barrier(0);                // (left alone, the compiler saves registers by taking the groups one by one)
            batch_sums(j0, kr, vr, w, s);
        }
    }
    __device__ __forceinline__ void sums(int from, int to, const float *w, SetSums &s) const {
        clear(s);
        add_sums(from, to, w, s);
    }
    // A set of two batches (17 .. 32 tokens): the second batch stays in registers from the distances to the sums, with its values, so half
    // the keys are read once, and the first one's second read is a batch after its first.  (Both batches in registers spill, 29 to
    // 50 of them, and so does the first batch's reload if it may start before the second's sums: hence the fence.  A last batch
    // kept for every length helps these and hurts the longer ones: 1024 slices of up to 16384 tokens 1216 / 1317.)  us, two
    // sweeps / this, the two batches on their way in distances and the 32-bit row offsets together: 1024 slices of 4096 565 / 547,
    // 256 of them 161 / 152, 1600 of 4096 in bf16 780 / 760, 1600 of 500 116 / 108, 64 of 4096 in fp32 72.6 / 68.8.
    __device__ __forceinline__ void sums_pair(int p, float *set_w, SetSums &s) {
        Raw k1[U], v1[U];
        load_rows(Ks, lo + 4 * U, k1);
        load_rows<READ_ONCE>(Vs, lo + 4 * U, v1);
        load_pivot(p);
        distances(0, 4 * U, set_w);
        batch_distances(lo + 4 * U, k1, set_w);
        wave_lds_fence();
        weights(0, hi - lo, set_w, set_w);
        wave_lds_fence();
        clear(s);
        batch_sums(lo + 4 * U, k1, v1, set_w, s);
        __builtin_amdgcn_sched_barrier(0);
        add_sums(0, 4 * U, set_w, s);
    }
    // a set of up to 16 tokens is read once: all loads issued together, both sweeps from registers.  (Left alone, the compiler
    // moves the pivot's load and the wait for it ahead of the branch on the length, and in fp16 takes the rows of the fixed mode
    // one by one, a round trip each: 512 slices of 4096 tokens in sets of three, fixed sigma, fp16, 880 / 483 us.)
    __device__ __forceinline__ void sums_short(int p, SetSums &s) {
        if constexpr (sizeof(T) == 2) asm volatile("");
        clear(s);
        const Raw kp_raw = row_chunk<T>(Ks, p, c);
        Raw kr[U], vr[U];
        load_rows<READ_ONCE>(Ks, lo, kr);
        load_rows<READ_ONCE>(Vs, lo, vr);
        if (MODE == MERGE_FIXED) __builtin_amdgcn_sched_barrier(0);
        E::to_float(kp_raw, kp);
        if (MODE != MERGE_ADAPTIVE) {
            batch_sums(lo, kr, vr, nullptr, s);
            return;
        }
        float d[U], dsum = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float x[8];
            E::to_float(kr[u], x);
            d[u] = sq_dist16(kp, x);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            d[u] = __builtin_amdgcn_sqrtf(d[u]);
            dsum += lo + 4 * u + slot < hi ? d[u] : 0.f;
        }
        dsum = rows4_sum(dsum);
        const float inv_mean = dsum > 0.f ? (float)(hi - lo) / dsum : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = lo + 4 * u + slot;
            float x[8], v[8];
            const float r = d[u] * inv_mean;
            float g = __expf(-r * r);
            g = row < hi ? g : 0.f;
            if (WITH_W && c == 0 && row < hi) wo[row] = g;
            E::to_float(kr[u], x);
            E::to_float(vr[u], v);
            s.g += g;
#pragma unroll
            for (int e = 0; e < 8; ++e) { s.k[e] = fmaf(g, x[e], s.k[e]); s.v[e] = fmaf(g, v[e], s.v[e]); }
        }
    }
    __device__ __forceinline__ void load_pivot(int p) { E::to_float(row_chunk<T>(Ks, p, c), kp); }
    // the merged rows.  The weights that are normalised here were written by other lanes, in a team by other waves: the caller puts a fence
    // (a barrier in a team) between those stores and this.
    __device__ __forceinline__ void finish(SetSums &s, T *k_row, T *v_row, const RowPart part) const {
        const int m = hi - lo;
        const float inv_g = 1.f / rows4_sum(s.g);
        // Keys come out in the even rows of the wave, values in the odd ones.  us, two sums for every column / one: 512 slices of 4096 tokens in sets
        // of two 826 / 725, of eight 252 / 236, 64 of 4096 in sets of three 80 / 68, 32 of 1000 AR(1) keys 16.5 / 15.3.  (What depends on the
        // row is worked out here, for every set: kept across the sets it spills.)
        int row = slot;
        asm volatile("" : "+v"(row));
        const float scale = (row & 1) && a.value_scale ? inv_g * (float)m : inv_g;
        float out[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = rows4_sum_pair(s.k[e], s.v[e]) * scale;
        if (row < 2 && part.holds(row, c)) {
            if constexpr (STREAM) E::store_stream(row == 0 ? k_row : v_row, c, E::from_float(out));
            else E::store(row == 0 ? k_row : v_row, c, E::from_float(out));
        }
        if (WITH_W) {
            for (int i = lane; i < m; i += WAVE) wo[lo + i] *= inv_g;
        }
    }
};

// One set [lo, hi) of 1 .. LONG_SET_MIN tokens with pivot p (lo <= p < hi), merged by one wave into
// the rows k_row, v_row.  Shared by merge_kernel and the refresh of single sets, so that a set gives
// the same bits wherever it is merged.  set_w: LDS of the wave, a float per token (a multiple of 16).
// Sets of more than 16 tokens take two sweeps; the first leaves the distances in LDS, one lane a row turns them into weights, and the
// second is multiply-adds.  (With distances worked out again in the second sweep, sixteen times over in the lanes of a row, a lone
// wave's arithmetic took as long as its loads: us, before / now, this and the sums on swaps instead of LDS moves together, one slice
// of 512 fp32 tokens 15.1 / 13.6, 1 of 16000 17.4 / 14.2, 32 of 2000 31.8 / 29.4, 1600 of 500 in bf16, now four waves a SIMD
// instead of three, 115 / 103.)
template <typename T, bool WITH_W, int MODE, bool ANY_LENGTH, bool STREAM>
__device__ __forceinline__ void merge_one_set(const T *Ks, const T *Vs, T *k_row, T *v_row, float *wo, int lo, int hi, int p,
                                              const MergeArgs &a, int lane, float *set_w, const RowPart part = RowPart())
{
    SetMerge<T, WITH_W, MODE, STREAM> set(Ks, Vs, wo, a, lo, hi, lane);
    constexpr int BATCH = 4 * SetMerge<T, WITH_W, MODE, STREAM>::U;
    const int m = hi - lo;
    SetSums s;
    if (m <= BATCH) {
        set.sums_short(p, s);
    } else if (MODE == MERGE_ADAPTIVE && m <= 2 * BATCH) {
        set.sums_pair(p, set_w, s);
        wave_lds_fence();
    } else {
        set.load_pivot(p);
        if (MODE == MERGE_ADAPTIVE) {
            set.distances(0, m, set_w);
            wave_lds_fence();
            set.weights(0, m, set_w, set_w);
            wave_lds_fence();
        }
        if (!ANY_LENGTH || m <= SPLIT_SET_MIN) {
            set.sums(0, m, set_w, s);
        } else {
            // (the running totals wait in LDS: in registers they cost every set of the kernel its fourth wave a SIMD, or spills)
            float *total = set_w + LONG_SET_MIN + lane;
            for (int from = 0;;) {
                const int to = min(from + part_rows(m), m);
                set.sums(from, to, set_w, s);
                if (from > 0) add_parked(s, total);
                if (to == m) break;
                park(s, total);
                from = to;
            }
        }
        wave_lds_fence();                                     // the next set's distances come to the same place
    }
    if (WITH_W) wave_lds_fence();
    set.finish(s, k_row, v_row, part);
}

// The same for a set of more than SPLIT_SET_MIN tokens by four waves of a workgroup, one part each.  All threads of the workgroup call
// it together (barriers inside); a team without a set passes an empty one.
struct TeamShared {
    float dist[LONG_SET_MIN], w[LONG_SET_MIN];
    float part[SPLIT_PARTS - 1][PARKED];
};
template <typename T, bool WITH_W, int MODE>
__device__ __forceinline__ void merge_set_team(const T *Ks, const T *Vs, T *k_row, T *v_row, float *wo, int lo, int hi, int p,
                                               const MergeArgs &a, int lane, int part_id, TeamShared &sh, const RowPart part = RowPart())
{
    SetMerge<T, WITH_W, MODE, false> set(Ks, Vs, wo, a, lo, hi, lane);
    SetSums s;
    const int from = part_id * part_rows(hi - lo), to = min(from + part_rows(hi - lo), hi - lo);   // (may be empty)
    if (hi > lo) set.load_pivot(p);
    if (MODE == MERGE_ADAPTIVE) {
        set.distances(from, to, sh.dist);
        __syncthreads();
        if (hi > lo) set.weights(from, to, sh.dist, sh.w);
        wave_lds_fence();                                     // a wave reads its own weights only
    }
    set.sums(from, to, sh.w, s);
    if (MODE != MERGE_ADAPTIVE) __syncthreads();              // the first wave has taken the parts of the set before
    if (part_id > 0) park(s, sh.part[part_id - 1] + lane);
    __syncthreads();
    if (part_id == 0 && hi > lo) {
        for (int q = 0; q < SPLIT_PARTS - 1; ++q) add_parked(s, sh.part[q] + lane);
        set.finish(s, k_row, v_row, part);
    }
}

// WAVES 1: a wave is a workgroup of its own.  WAVES 4: four tiles a workgroup, whose waves then merge the sets of more than
// SPLIT_SET_MIN tokens together.
// Four waves a SIMD in 16 bit; three where fixed sigma with the weights written would spill for it (512 slices of 4096 tokens in sets of two 1135 / 991 us,
// of sixteen 254 / 231, 256 slices of AR(1) keys 183 / 170).
template <typename T, bool WITH_W, int MODE> constexpr int merge_waves_per_simd() {
    return sizeof(T) == 4 ? 2 : WITH_W && MODE == MERGE_FIXED ? 3 : 4;
}
template <typename T, bool WITH_W, int MODE, int WAVES, bool STREAM>
__global__ __launch_bounds__(WAVES * WAVE, (merge_waves_per_simd<T, WITH_W, MODE>())) void merge_kernel(const T *__restrict__ K, const T *__restrict__ V,
                                                            T *__restrict__ K_out, T *__restrict__ V_out, MergeArgs a)
{
    constexpr int US = 4;                      // row groups (of 4 rows) in flight in runs of singleton sets
    constexpr bool TEAM = WAVES == SPLIT_PARTS;
    __shared__ float set_w[WAVES][TEAM ? SPLIT_SET_MIN : LONG_SET_MIN + PARKED];   // (merge_one_set)
    const int wave = TEAM ? (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int per_slice = (a.tiles_per_slice + WAVES - 1) / WAVES;        // workgroups
    int slice = blockIdx.x / per_slice, tile = (blockIdx.x - slice * per_slice) * WAVES + wave;
    const int group = slice / 8;
    if (!TEAM && a.tile == MERGE_TILE && a.tiles_per_slice <= MERGE_GROUPED_TILES && group < a.slices / 8) {
        const int at = blockIdx.x - 8 * group * a.tiles_per_slice;
        slice = 8 * group + (at + group) % 8;
        tile = (at / 8 + group + group / 4 + group / 16) % a.tiles_per_slice;
    }
    const int lane = threadIdx.x & 63;
    const int slot = lane >> 4;          // which of the four rows of an instruction
    const int c = lane & 15;             // which 8-element chunk of the row
    const int n = clamp_len(a.seq_lens, slice / a.H, a.N);
    const int edge = tile * a.tile;
    if (!TEAM && edge >= n) return;
    const int M = edge < n ? min(max(a.n_sets[slice], 0), a.cap_rows) : 0;
    const int32_t *sst = a.set_start + (size_t)slice * (a.cap_rows + 1);
    const int32_t *piv = a.pivot + (size_t)slice * a.cap_rows;
    // lane i looks at set s_lo+i (the pivot is fetched along, before it is known to be needed); cnt sets from
    // s_lo on start inside this tile, followed by the start of the next set, the end of the last one
    const int s_lo = first_set_at(sst, M, edge, lane);
    const int start_raw = s_lo + lane <= M ? sst[s_lo + lane] : INT_MAX;
    const int my_piv = s_lo + lane < M ? piv[s_lo + lane] : 0;
    const unsigned long long beyond = ~__ballot(s_lo + lane < M && start_raw < edge + a.tile);
    const int cnt = beyond ? __builtin_ctzll(beyond) : WAVE;
    if (!TEAM && cnt == 0) return;

    const T *Ks = K + (size_t)slice * a.N * HEAD_DIM;
    const T *Vs = V + (size_t)slice * a.N * HEAD_DIM;
    T *Ko = K_out + (size_t)slice * a.cap_rows * HEAD_DIM;
    T *Vo = V_out + (size_t)slice * a.cap_rows * HEAD_DIM;
    float *wo = WITH_W ? a.w_opt + (size_t)slice * a.N : nullptr;

    const int my_start = min(max(start_raw, 0), n);
    int my_next = __shfl_down(my_start, 1, WAVE);
    if (cnt == WAVE && lane == WAVE - 1) my_next = min(max(sst[s_lo + WAVE], 0), n);
    const unsigned long long single_mask = __ballot(lane < cnt && my_next - my_start == 1);

    struct Posted { int s, lo, hi, p; };
    __shared__ Posted posted[TEAM ? WAVES * WAVE : 1];        // (a wave looks at no more than 64 sets)
    __shared__ int n_posted;
    __shared__ char team_mem[TEAM ? sizeof(TeamShared) : 1] __attribute__((aligned(16)));
    if (TEAM) {
        if (threadIdx.x == 0) n_posted = 0;
        __syncthreads();
    }
    int i = 0;
    while (i < cnt) {
        // ---- runs of singleton sets: plain copy, up to 4*U sets per step, all loads in flight ------
        if ((single_mask >> i) & 1ull) {
            const unsigned long long others = ~(single_mask >> i);        // (no bit of the mask is set beyond cnt)
            const int run = min(others ? __builtin_ctzll(others) : WAVE, 4 * US);
            CopiedRow<T> rk[US], rv[US];
            int src[US];
#pragma unroll
            for (int u = 0; u < US; ++u) {
                const int r = 4 * u + slot;
                src[u] = __shfl(my_start, i + min(r, run - 1), WAVE);
                if (r < run) {
                    rk[u].template load<reads_once<T, STREAM>()>(Ks, src[u], c);
                    rv[u].template load<reads_once<T, STREAM>()>(Vs, src[u], c);
                }
            }
#pragma unroll
            for (int u = 0; u < US; ++u) {
                const int r = 4 * u + slot;
                if (r < run) {
                    rk[u].template store<STREAM>(Ko + (size_t)(s_lo + i + r) * HEAD_DIM, c);
                    rv[u].template store<STREAM>(Vo + (size_t)(s_lo + i + r) * HEAD_DIM, c);
                    if (WITH_W && c == 0) wo[src[u]] = 1.f;
                }
            }
            i += run;
            continue;
        }
        // ---- a set with several tokens --------------------------------------------------------------
        const int lo = __builtin_amdgcn_readlane(my_start, i);
        const int hi = __builtin_amdgcn_readlane(my_next, i);
        const int m = hi - lo;
        if (m <= 0 || m > LONG_SET_MIN) { ++i; continue; }                // inconsistent map: nothing to merge; long set: merge_long_kernel
        int p = __builtin_amdgcn_readlane(my_piv, i);
        p = min(max(p, lo), hi - 1);
        if (TEAM && m > SPLIT_SET_MIN) {
            if (lane == 0) posted[atomicAdd(&n_posted, 1)] = {s_lo + i, lo, hi, p};
            ++i;
            continue;
        }
        merge_one_set<T, WITH_W, MODE, !TEAM, STREAM>(Ks, Vs, Ko + (size_t)(s_lo + i) * HEAD_DIM, Vo + (size_t)(s_lo + i) * HEAD_DIM, wo, lo, hi, p,
                                              a, lane, set_w[wave]);
        ++i;
    }
    if constexpr (TEAM) {
        __syncthreads();
        const int n_team = n_posted;
        for (int k = 0; k < n_team; ++k) {
            const int s = __builtin_amdgcn_readfirstlane(posted[k].s), lo = __builtin_amdgcn_readfirstlane(posted[k].lo);
            const int hi = __builtin_amdgcn_readfirstlane(posted[k].hi), p = __builtin_amdgcn_readfirstlane(posted[k].p);
            merge_set_team<T, WITH_W, MODE>(Ks, Vs, Ko + (size_t)s * HEAD_DIM, Vo + (size_t)s * HEAD_DIM, wo, lo, hi, p, a, lane, wave,
                                            *reinterpret_cast<TeamShared *>(team_mem));
        }
    }
}

// One set of more than LONG_SET_MIN tokens by the 64 sixteen-lane groups of a 1024-thread workgroup: group g takes the set's rows
// g, g + 64, ... (four of them in flight), the distance sum and then the weighted sums are added up across the groups through
// LDS.  Same arithmetic per row as merge_one_set; only the order of the fp32 additions differs.  All threads call it together.
struct LongShared {
    float red[LONG_SET_BLOCK / WAVE][16][17];                 // per wave and chunk lane: 8 key sums, 8 value sums, weight sum
    float red1[LONG_SET_BLOCK / WAVE];
};
template <typename T, bool WITH_W, int MODE>
__device__ __forceinline__ void merge_long_set(const T *Ks, const T *Vs, T *k_row, T *v_row, float *wo, int lo, int hi, int p, const MergeArgs &a,
                                               int tid, LongShared &sh, const RowPart part = RowPart())
{
    using E = Elem<T>;
    using Raw = typename E::Raw;
    constexpr int U = 4;                                     // rows of a group in flight
    constexpr int GROUPS = LONG_SET_BLOCK / 16, WAVES = LONG_SET_BLOCK / WAVE;
    const int lane = tid & 63, wave = tid >> 6, c = tid & 15, group = tid >> 4;
    const int m = hi - lo;
    float kp[8];
    E::to_float(E::load(Ks + (size_t)p * HEAD_DIM, c), kp);
    float inv_mean = 0.f;
    if (MODE == MERGE_ADAPTIVE) {
        float dsum = 0.f;
        for (int j0 = lo + group; j0 < hi; j0 += GROUPS * U) {
            Raw kr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) kr[u] = E::load(Ks + (size_t)min(j0 + GROUPS * u, hi - 1) * HEAD_DIM, c);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float x[8];
                E::to_float(kr[u], x);
                const float dist = __builtin_amdgcn_sqrtf(sq_dist16(kp, x));
                dsum += (j0 + GROUPS * u < hi) ? dist : 0.f;
            }
        }
        dsum = rows4_sum(dsum);                           // the wave's four groups
        __syncthreads();                                  // sh.red1 may still be read from the set before
        if (lane == 0) sh.red1[wave] = dsum;
        __syncthreads();
        float total = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < WAVES; ++w2) total += sh.red1[w2];
        inv_mean = total > 0.f ? (float)m / total : 0.f;
    }
    float ak[8], av[8], gsum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) { ak[e] = 0.f; av[e] = 0.f; }
    for (int j0 = lo + group; j0 < hi; j0 += GROUPS * U) {
        Raw kr[U], vr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t row = (size_t)min(j0 + GROUPS * u, hi - 1) * HEAD_DIM;
            kr[u] = E::load(Ks + row, c);
            vr[u] = E::load(Vs + row, c);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = j0 + GROUPS * u;
            float x[8], v[8];
            E::to_float(kr[u], x);
            float g;
            if (MODE == MERGE_AVERAGE) {
                g = 1.f;
            } else if (MODE == MERGE_FIXED) {
                g = __expf(-sq_dist16(kp, x) * a.inv_two_sigma_sq);
            } else {
                const float r = __builtin_amdgcn_sqrtf(sq_dist16(kp, x)) * inv_mean;
                g = __expf(-r * r);
            }
            g = row < hi ? g : 0.f;
            gsum += g;
            E::to_float(vr[u], v);
#pragma unroll
            for (int e = 0; e < 8; ++e) { ak[e] = fmaf(g, x[e], ak[e]); av[e] = fmaf(g, v[e], av[e]); }
            if (WITH_W && c == 0 && row < hi) wo[row] = g;
        }
    }
    gsum = rows4_sum(gsum);
#pragma unroll
    for (int e = 0; e < 8; ++e) { ak[e] = rows4_sum(ak[e]); av[e] = rows4_sum(av[e]); }
    __syncthreads();                                      // sh.red may still be read from the set before
    if (lane < 16) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { sh.red[wave][c][e] = ak[e]; sh.red[wave][c][8 + e] = av[e]; }
        sh.red[wave][c][16] = gsum;
    }
    __syncthreads();
    float gtot = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < WAVES; ++w2) gtot += sh.red[w2][0][16];
    const float inv_g = 1.f / gtot;
    if (tid < 32) {                                       // lanes 0..15: the key row, 16..31: the value row
        const bool is_v = tid >= 16;
        const float scale = is_v && a.value_scale ? inv_g * (float)m : inv_g;
        float out[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float t = 0.f;
#pragma unroll
            for (int w2 = 0; w2 < WAVES; ++w2) t += sh.red[w2][c][(is_v ? 8 : 0) + e];
            out[e] = t * scale;
        }
        if (part.holds(is_v, c)) E::store(is_v ? v_row : k_row, c, E::from_float(out));
    }
    if (WITH_W && c == 0) {                               // each writer normalises its own g_j
        for (int row = lo + group; row < hi; row += GROUPS) wo[row] *= inv_g;
    }
}

// Sets of more than LONG_SET_MIN tokens, one after the other, by a 1024-thread workgroup per slice.  The workgroup looks the long sets up in the maps itself (or takes the refresh's list), 4096 sets
// at a time, in no particular order: each is merged on its own.  The registers of one workgroup per
// compute unit are given to it outright (waves_per_eu), because the compiler otherwise saves them by
// taking the four rows of a group one after the other; a set's number is moved to a scalar, because
// one that comes out of LDS counts as different in every lane.  Measured, us, this kernel: one
// slice of 262144 equal keys 1305 / 954 (935 with the sets listed by a launch of 176 us before it), 512
// of 4096 117 / 97 (98 and 10); one of 2^20 tokens without long sets 292 / 132 (6 and 850).
template <typename T, bool WITH_W, int MODE>
__global__ __launch_bounds__(LONG_SET_BLOCK) __attribute__((amdgpu_waves_per_eu(4, 4))) void merge_long_kernel(const T *__restrict__ K, const T *__restrict__ V,
                                                                T *__restrict__ K_out, T *__restrict__ V_out, MergeArgs a)
{
    __shared__ LongShared sums;
    __shared__ int found[LONG_SET_BLOCK * LONG_SET_LOOK], n_found[2];   // (two counters in turn: one is cleared while the other is read)
    const int slice = blockIdx.x;
    const int tid = threadIdx.x;
    const int n = clamp_len(a.seq_lens, slice / a.H, a.N);
    const int M = min(max(a.n_sets[slice], 0), a.cap_rows);
    const int32_t *sst = a.set_start + (size_t)slice * (a.cap_rows + 1);
    const int32_t *piv = a.pivot + (size_t)slice * a.cap_rows;
    const T *Ks = K + (size_t)slice * a.N * HEAD_DIM;
    const T *Vs = V + (size_t)slice * a.N * HEAD_DIM;
    T *Ko = K_out + (size_t)slice * a.cap_rows * HEAD_DIM;
    T *Vo = V_out + (size_t)slice * a.cap_rows * HEAD_DIM;
    float *wo = WITH_W ? a.w_opt + (size_t)slice * a.N : nullptr;

    const int32_t *pl = a.long_list ? a.long_list + (size_t)slice * a.list_stride : nullptr;
    int left = max_long_sets(a.N);                            // consistent maps never have more
    const int candidates = pl ? min(max(pl[0], 0), left) : M;
    if (candidates == 0 || M == 0) return;
    if (tid < 2) n_found[tid] = 0;
    __syncthreads();
    for (int first = 0, turn = 0; first < candidates; first += LONG_SET_BLOCK * LONG_SET_LOOK, turn ^= 1) {
    // (all loads before the first test; beyond the last set the last one is looked at again, and not taken)
    int s_at[LONG_SET_LOOK], from[LONG_SET_LOOK], to[LONG_SET_LOOK];
#pragma unroll
    for (int u = 0; u < LONG_SET_LOOK; ++u) s_at[u] = min(first + u * LONG_SET_BLOCK + tid, candidates - 1);
    if (pl) {
#pragma unroll
        for (int u = 0; u < LONG_SET_LOOK; ++u) s_at[u] = min(max(pl[1 + s_at[u]], 0), M - 1);
    }
#pragma unroll
    for (int u = 0; u < LONG_SET_LOOK; ++u) { from[u] = sst[s_at[u]]; to[u] = sst[s_at[u] + 1]; }
#pragma unroll
    for (int u = 0; u < LONG_SET_LOOK; ++u)
        if (first + u * LONG_SET_BLOCK + tid < candidates && min(max(to[u], 0), n) - min(max(from[u], 0), n) > LONG_SET_MIN)
            found[atomicAdd(&n_found[turn], 1)] = s_at[u];
    __syncthreads();
    const int n_long = __builtin_amdgcn_readfirstlane(min(n_found[turn], left));
    left -= n_long;
    if (tid == 0) n_found[turn ^ 1] = 0;                      // read last before this turn's barrier above
    for (int k = 0; k < n_long; ++k) {
        const int s = __builtin_amdgcn_readfirstlane(found[k]);   // scalar, and the loops below with it
        const int lo = min(max(sst[s], 0), n), hi = min(max(sst[s + 1], 0), n);
        const int p = max(min(max(piv[s], lo), hi - 1), 0);   // (the bounds are read a second time: inside the slice whatever they are)
        merge_long_set<T, WITH_W, MODE>(Ks, Vs, Ko + (size_t)s * HEAD_DIM, Vo + (size_t)s * HEAD_DIM, wo, lo, hi, p, a, tid, sums);
    }
    if (first + LONG_SET_BLOCK * LONG_SET_LOOK < candidates) __syncthreads();  // found is filled again; the cleared counter is seen
    }
}

template <typename T, int WAVES, bool STREAM>
static void launch_merge_t(const kvm_shape &sh, const void *K, const void *V, void *K_out, void *V_out,
                           const MergeArgs &a, hipStream_t st)
{
    const long long blocks = (long long)sh.B * sh.H_kv * ((a.tiles_per_slice + WAVES - 1) / WAVES);
    ProfScope prof("merge_kernel", st);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(WAVES * WAVE), 0, st, (const T *)K, (const T *)V, (T *)K_out, (T *)V_out, a);
    };
    if (a.w_opt) {
        if (a.mode == MERGE_AVERAGE) run(merge_kernel<T, true, MERGE_AVERAGE, WAVES, STREAM>);
        else if (a.mode == MERGE_FIXED) run(merge_kernel<T, true, MERGE_FIXED, WAVES, STREAM>);
        else run(merge_kernel<T, true, MERGE_ADAPTIVE, WAVES, STREAM>);
    } else {
        if (a.mode == MERGE_AVERAGE) run(merge_kernel<T, false, MERGE_AVERAGE, WAVES, STREAM>);
        else if (a.mode == MERGE_FIXED) run(merge_kernel<T, false, MERGE_FIXED, WAVES, STREAM>);
        else run(merge_kernel<T, false, MERGE_ADAPTIVE, WAVES, STREAM>);
    }
}

template <typename T>
static void launch_merge_long_t(const kvm_shape &sh, const void *K, const void *V, void *K_out, void *V_out,
                                const MergeArgs &a, hipStream_t st)
{
    ProfScope prof("merge_long_kernel", st);
    const dim3 grid((unsigned)((long long)sh.B * sh.H_kv)), block(LONG_SET_BLOCK);
    const T *k = (const T *)K, *v = (const T *)V;
    T *ko = (T *)K_out, *vo = (T *)V_out;
    if (a.w_opt) {
        if (a.mode == MERGE_AVERAGE) hipLaunchKernelGGL((merge_long_kernel<T, true, MERGE_AVERAGE>), grid, block, 0, st, k, v, ko, vo, a);
        else if (a.mode == MERGE_FIXED) hipLaunchKernelGGL((merge_long_kernel<T, true, MERGE_FIXED>), grid, block, 0, st, k, v, ko, vo, a);
        else hipLaunchKernelGGL((merge_long_kernel<T, true, MERGE_ADAPTIVE>), grid, block, 0, st, k, v, ko, vo, a);
    } else {
        if (a.mode == MERGE_AVERAGE) hipLaunchKernelGGL((merge_long_kernel<T, false, MERGE_AVERAGE>), grid, block, 0, st, k, v, ko, vo, a);
        else if (a.mode == MERGE_FIXED) hipLaunchKernelGGL((merge_long_kernel<T, false, MERGE_FIXED>), grid, block, 0, st, k, v, ko, vo, a);
        else hipLaunchKernelGGL((merge_long_kernel<T, false, MERGE_ADAPTIVE>), grid, block, 0, st, k, v, ko, vo, a);
    }
}

kvm_status launch_merge(const kvm_shape &sh, const kvm_params &pr, int cap_rows, const void *K, const void *V,
                        const int32_t *set_start, const int32_t *pivot, const int32_t *n_sets, void *K_out,
                        void *V_out, float *w_opt, hipStream_t st)
{
    if ((long long)sh.B * sh.H_kv == 0 || cap_rows == 0 || sh.N == 0) return KVM_OK;
    MergeArgs a;
    a.set_start = set_start;
    a.pivot = pivot;
    a.n_sets = n_sets;
    a.seq_lens = sh.seq_lens;
    a.w_opt = w_opt;
    a.long_list = nullptr;
    a.slices = sh.B * sh.H_kv;
    a.H = sh.H_kv;
    a.N = sh.N;
    a.cap_rows = cap_rows;
    a.tile = (long long)sh.B * sh.H_kv * sh.N <= MERGE_FEW_TOKENS ? MERGE_TILE_FEW : MERGE_TILE;
    a.tiles_per_slice = (sh.N + a.tile - 1) / a.tile;
    a.list_stride = 0;
    a.mode = pr.weights == KVM_WEIGHTS_AVERAGE ? MERGE_AVERAGE : (pr.sigma_mode == KVM_SIGMA_FIXED ? MERGE_FIXED : MERGE_ADAPTIVE);
    a.inv_two_sigma_sq = a.mode == MERGE_FIXED ? 1.f / (2.f * pr.sigma * pr.sigma) : 0.f;
    a.value_scale = pr.value_scale_by_set_size;
    const bool team = (long long)sh.B * sh.H_kv * sh.N <= MERGE_TEAM_TOKENS;
    const bool stream = streams_rows(sh, cap_rows);
    const auto launch = [&](auto elem) {
        using T = decltype(elem);
        if (team) launch_merge_t<T, 4, false>(sh, K, V, K_out, V_out, a, st);
        else if (stream) launch_merge_t<T, 1, true>(sh, K, V, K_out, V_out, a, st);
        else launch_merge_t<T, 1, false>(sh, K, V, K_out, V_out, a, st);
    };
    switch (sh.dtype) {
    case KVM_F32: launch(float()); break;
    case KVM_F16: launch(half_t()); break;
    default: launch(bf16_t()); break;
    }
    kvm_status rc = check_launch("merge_kernel");
    if (rc != KVM_OK || sh.N <= LONG_SET_MIN) return rc;          // (no slice can hold a long set)
    switch (sh.dtype) {
    case KVM_F32: launch_merge_long_t<float>(sh, K, V, K_out, V_out, a, st); break;
    case KVM_F16: launch_merge_long_t<half_t>(sh, K, V, K_out, V_out, a, st); break;
    default: launch_merge_long_t<bf16_t>(sh, K, V, K_out, V_out, a, st); break;
    }
    return check_launch("merge_long_kernel");
}

// ------------------------------------------------------------------------------------------
// Refresh of a compacted cache after the index maps changed a little (decode time: one more
// token moves the recent window, the top-k and a few pivots).  A set of the new maps whose
// extent and pivot already existed in the previous maps has the same merged row as before:
// the row only moves to its new index; the others are merged again.  Result: bit for bit what
// merge_kernel / merge_long_kernel give on the new maps.
//
// refresh_kernel, one workgroup per slice (or two or four, see REFRESH_MAX_PARTS), three phases with a barrier between them:
//   compare   src[s] = row of the previous cache that new row s is (-1: merge again), the list
//             of short sets to merge again, and the long ones in the layout merge_long_kernel
//             reads (that kernel follows)
//   move      rows in place.  src is increasing over the rows that move, so rows moving up
//             never need a row that rows moving down overwrite and vice versa; rows moving up
//             are taken from the top down, rows moving down from the bottom up, a batch at a time,
//             all reads of a batch before its writes.
//   merge     one wave per listed set (merge_one_set), the workgroup's waves in turn.  A
//             slice that has little to move gets here early, so the longest set of the launch
//             (one wave, up to LONG_SET_MIN rows) overlaps the other slices' moves.
// ------------------------------------------------------------------------------------------

struct RefreshArgs {
    const int32_t *prev_set_id, *prev_set_start, *prev_pivot, *prev_n_sets;
    int32_t *src;          // (slices, cap_rows), written alike by all workgroups of a slice (see REFRESH_MAX_PARTS)
    int32_t *lists;        // (slices, cap_rows + 1): number of short sets to merge again, then their indices
    int32_t *long_list;    // what MergeArgs::long_list points to
    int32_t *n_changed;    // (slices) or NULL: sets merged again
    int32_t *part_lists;   // (parts - 1, slices, cap_rows + 2 + max_long_sets): the lists of the workgroups of a slice beyond the first, long ones after the short
    int parts;             // workgroups per slice: 1, or 2 or 4 (refresh_kernel<..., SPLIT>)
};

constexpr int REFRESH_POSTED = 256;                          // sets that are merged again in one turn
constexpr int REFRESH_LOOK = 4;                              // sets a thread compares at a time
// Threads per slice: 512, two workgroups per compute unit (128 registers each), or 1024 where every slice has a compute unit to itself:
// half as many batches to move one after the other, and the long sets are merged by the same workgroup instead of by a launch of their own.
// Whole decode step, us, 512 / 1024: 32 slices of 3000 bf16 tokens, G = 4, 54.3 / 48.4, of 1000 41.8 / 38.9, 8 of 9000 81.8 / 75.0, of 2000 in fp32
// 43.0 / 40.2, 256 of 2000 68.6 / 65.2, 240 of 4096 110.8 / 106.6.  Where no set can be long there is no launch to save and little to move, and
// the larger workgroup only starts later (refresh: 128 slices of 100 fp16 tokens 11.4 / 12.8, of 300 15.6 / 16.6, one of 300 9.1 / 10.0).
constexpr int REFRESH_BLOCK = 512, REFRESH_BLOCK_FEW = LONG_SET_BLOCK;
constexpr long long REFRESH_FEW_SLICES = 256;
static bool refresh_few(const kvm_shape &sh) { return (long long)sh.B * sh.H_kv <= REFRESH_FEW_SLICES && sh.N > LONG_SET_MIN; }
constexpr int REFRESH_MAX_PARTS = 4;
template <typename T> struct MovePerGroup { static constexpr int value = 16 / sizeof(T); };   // rows a 16-lane group moves per batch
constexpr int REFRESH_MOVE_ROWS = REFRESH_BLOCK_FEW / 16 * MovePerGroup<half_t>::value;       // 16-bit rows of a batch of one workgroup a slice
// Up to 128 slices, where compute units are left over, two or four workgroups share a slice by columns: one or two move and write keys, the
// others values, half a row each where there are four.  No bytes of the rows are shared, so they still move in place without waiting for another
// workgroup; each compares the maps and merges the changed sets for itself, with lists of its own.  The sources (src) they do share: every
// workgroup of a slice writes all of them and reads what it wrote, the same values as the others, since they follow from the maps alone.  What
// depends on the workgroup must not go there.  What a workgroup has to move is then a half or a
// quarter (one compute unit moves about 0.1 TB/s), where it takes it more than two batches: below, the refresh is a chain of latencies
// that does not get shorter (8 slices of 1000 bf16 tokens 16.0 / 17.5).  Four, not eight: a quarter of a 16-bit row would be half a cache line.
// Refresh, us, one workgroup a slice / split: 32 slices of 3000 bf16 tokens 23.3 / 20.4, 8 of 2200 21.1 / 18.4, of 16384 54.7 / 30.8, 64 of 4096
// 31.5 / 25.6, 128 38.6 / 35.3; fp32: 32 of 2000 28.5 / 21.4, 128 41.0 / 36.1, 8 of 2000 at 35 percent 16.8 / 14.7, 40 of 1100 22.2 / 19.2.

template <typename T, int MODE, int BLOCK, bool SPLIT>
__global__ __launch_bounds__(BLOCK, 4) void refresh_kernel(const T *__restrict__ K, const T *__restrict__ V,
                                                                T *__restrict__ K_out, T *__restrict__ V_out, MergeArgs a,
                                                                RefreshArgs r)
{
    using E = Elem<T>;
    using Raw = typename E::Raw;
    constexpr int MOVE_PER_GROUP = SPLIT ? 8 : MovePerGroup<T>::value;   // (split, one of keys and values)
    __shared__ int n_short, n_long, first_moved, any_up, any_down;
    constexpr int TEAMS = BLOCK / WAVE / SPLIT_PARTS;
    __shared__ float set_w[BLOCK / WAVE][SPLIT_SET_MIN];
    __shared__ TeamShared team_mem[TEAMS];
    __shared__ int posted[REFRESH_POSTED], n_posted;
    const int slice = SPLIT ? blockIdx.x % a.slices : blockIdx.x, part_id = SPLIT ? blockIdx.x / a.slices : 0;
    const int tid = threadIdx.x;
    const int lanes = SPLIT ? 32 / r.parts : 16;             // of a row that is moved
    const int groups = BLOCK / lanes, group = tid / lanes, c = (part_id >> 1) * lanes + tid % lanes;
    const int move_batch_rows = groups * MOVE_PER_GROUP;     // rows the workgroup moves per batch
    RowPart part;
    if (SPLIT) part.which = part_id & 1, part.c0 = (part_id >> 1) * lanes, part.c1 = part.c0 + lanes;
    const int n = clamp_len(a.seq_lens, slice / a.H, a.N);
    const int M = min(max(a.n_sets[slice], 0), a.cap_rows);
    const int M_old = min(max(r.prev_n_sets[slice], 0), a.cap_rows);
    const int32_t *sst = a.set_start + (size_t)slice * (a.cap_rows + 1);
    const int32_t *piv = a.pivot + (size_t)slice * a.cap_rows;
    const int32_t *osst = r.prev_set_start + (size_t)slice * (a.cap_rows + 1);
    const int32_t *opiv = r.prev_pivot + (size_t)slice * a.cap_rows;
    const int32_t *osid = r.prev_set_id + (size_t)slice * a.N;
    int32_t *src = r.src + (size_t)slice * a.cap_rows;
    const int max_long = max_long_sets(a.N);
    int32_t *list = r.lists + (size_t)slice * (a.cap_rows + 1);
    int32_t *pl = r.long_list + (size_t)slice * a.list_stride;
    if (SPLIT && part_id > 0) {
        list = r.part_lists + ((size_t)(part_id - 1) * a.slices + slice) * (a.cap_rows + 2 + max_long);
        pl = list + a.cap_rows + 1;
    }
    T *Ko = K_out + (size_t)slice * a.cap_rows * HEAD_DIM;
    T *Vo = V_out + (size_t)slice * a.cap_rows * HEAD_DIM;

    // ---- compare ------------------------------------------------------------------------------
    if (tid == 0) { n_short = 0; n_long = 0; first_moved = a.cap_rows; any_up = 0; any_down = 0; }
    int my_first = M;
    bool my_up = false, my_down = false;
    for (int base = 0; base == 0 || base < M; base += BLOCK * REFRESH_LOOK) {   // (the first turn's loads do not wait for M)
        // Three round trips for four sets a thread: the sets' own bounds and pivots, their first tokens' previous sets, those sets' bounds and
        // pivots.  (One set at a time, a test between one load and the next, they were five for each.  Whole decode step, us, before / now:
        // 1024 slices of 4096 fp16 tokens 381 / 374, 32 of 3000 in bf16 48.5 / 47.0, 8 of 16384 93.7 / 90.1.)  Indices are clamped into the
        // buffers, and what a clamped one reads is not taken.
        int start[REFRESH_LOOK], end[REFRESH_LOOK], p[REFRESH_LOOK], so[REFRESH_LOOK], o_start[REFRESH_LOOK], o_end[REFRESH_LOOK], o_p[REFRESH_LOOK];
#pragma unroll
        for (int u = 0; u < REFRESH_LOOK; ++u) {
            const int s = min(base + u * BLOCK + tid, a.cap_rows - 1);
            start[u] = sst[s]; end[u] = sst[s + 1]; p[u] = piv[s];
        }
#pragma unroll
        for (int u = 0; u < REFRESH_LOOK; ++u) so[u] = osid[max(min(start[u], n - 1), 0)];
#pragma unroll
        for (int u = 0; u < REFRESH_LOOK; ++u) {
            const int at = min(max(so[u], 0), a.cap_rows - 1);
            o_start[u] = osst[at]; o_end[u] = osst[at + 1]; o_p[u] = opiv[at];
        }
        // (left alone, the compiler moves the last loads behind the tests that need them)
        static_assert(REFRESH_LOOK == 4, "the operands below");
        asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]), "+v"(o_start[0]), "+v"(o_start[1]), "+v"(o_start[2]), "+v"(o_start[3]),
                          "+v"(o_end[0]), "+v"(o_end[1]), "+v"(o_end[2]), "+v"(o_end[3]), "+v"(o_p[0]), "+v"(o_p[1]), "+v"(o_p[2]), "+v"(o_p[3]));
        if (base == 0) __syncthreads();                       // the counters are cleared
#pragma unroll
        for (int u = 0; u < REFRESH_LOOK; ++u) {
            const int s = base + u * BLOCK + tid;
            if (s >= M) continue;
            const int lo = min(max(start[u], 0), n), hi = min(max(end[u], 0), n);
            const bool same = hi > lo && so[u] >= 0 && so[u] < M_old && o_start[u] == start[u] && o_end[u] == end[u] && o_p[u] == p[u];
            const int from = same ? so[u] : -1;
            src[s] = from;                                    // (from the maps alone: the same from every workgroup of the slice)
            if (from < 0) {
                if (hi - lo > LONG_SET_MIN) {
                    const int k = atomicAdd(&n_long, 1);
                    if (k < max_long) pl[1 + k] = s;
                } else {
                    list[1 + atomicAdd(&n_short, 1)] = s;
                }
            } else if (from != s) {
                my_first = min(my_first, s);
                my_up |= from < s;
                my_down |= from > s;
            }
        }
    }
    if (my_first < M) atomicMin(&first_moved, my_first);
    if (my_up) any_up = 1;
    if (my_down) any_down = 1;
    __syncthreads();                                          // src and list are read below by other threads of this workgroup
    const int first = min(first_moved, M);
    const bool moves_up = any_up != 0, moves_down = any_down != 0;
    const int cnt = n_short;
    if (tid == 0) {
        list[0] = cnt;
        pl[0] = min(n_long, max_long);
        if (r.n_changed && part_id == 0) r.n_changed[slice] = cnt + n_long;
    }

    // ---- move ---------------------------------------------------------------------------------
    // (a direction that no row takes is skipped as a whole: after one more token nearly all rows
    // that move go the same way)
    const int b_lo = first / move_batch_rows, b_hi = (M - 1) / move_batch_rows;
    T *const X = SPLIT && part.which == 1 ? Vo : Ko;
    int s[MOVE_PER_GROUP], f[MOVE_PER_GROUP], f_next[MOVE_PER_GROUP];
    Raw rk[MOVE_PER_GROUP], rv[SPLIT ? 1 : MOVE_PER_GROUP];
    auto sources = [&](int bt, int *out) {                    // the batch's sources, before the direction filter
#pragma unroll
        for (int u = 0; u < MOVE_PER_GROUP; ++u) {
            const int row = bt * move_batch_rows + u * groups + group;
            out[u] = src[min(row, M - 1)];                    // (rows move, so there are some)
        }
    };
    auto move_batch = [&](int bt, bool up, int bt_next, bool more) {
        bool any = false;
#pragma unroll
        for (int u = 0; u < MOVE_PER_GROUP; ++u) {
            s[u] = bt * move_batch_rows + u * groups + group;
            f[u] = s[u] < M ? f_next[u] : -1;
            if (!(up ? (f[u] >= 0 && f[u] < s[u]) : f[u] > s[u])) f[u] = -1;
            any |= f[u] >= 0;
        }
        if (more) sources(bt_next, f_next);                   // in flight across the barriers
        if (!__syncthreads_or(any ? 1 : 0)) return;
#pragma unroll
        for (int u = 0; u < MOVE_PER_GROUP; ++u)
            if (f[u] >= 0) {
                rk[u] = E::load(X + (size_t)f[u] * HEAD_DIM, c);
                if constexpr (!SPLIT) rv[u] = E::load(Vo + (size_t)f[u] * HEAD_DIM, c);
            }
        __syncthreads();                                      // every source row of the batch is in registers
#pragma unroll
        for (int u = 0; u < MOVE_PER_GROUP; ++u)
            if (f[u] >= 0) {
                E::store(X + (size_t)s[u] * HEAD_DIM, c, rk[u]);
                if constexpr (!SPLIT) E::store(Vo + (size_t)s[u] * HEAD_DIM, c, rv[u]);
            }
    };
    if (moves_up) {                                           // new index above the old one: batches from the top down
        sources(b_hi, f_next);
        for (int bt = b_hi; bt >= b_lo; --bt) move_batch(bt, true, bt - 1, bt > b_lo);
    }
    if (moves_up && moves_down) __syncthreads();
    if (moves_down) {                                         // batches from the bottom up
        sources(b_lo, f_next);
        for (int bt = b_lo; bt <= b_hi; ++bt) move_batch(bt, false, bt + 1, bt < b_hi);
    }
    if (moves_up || moves_down) __syncthreads();              // a row merged below may be one that was a source above

    // ---- merge the listed sets again -------------------------------------------------------------
    // (a wave each; sets of more than SPLIT_SET_MIN tokens are left for teams of four waves)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T *Ks = K + (size_t)slice * a.N * HEAD_DIM;
    const T *Vs = V + (size_t)slice * a.N * HEAD_DIM;
    for (int base = 0; base < cnt; base += REFRESH_POSTED) {  // (the same for the whole workgroup)
        __syncthreads();                                      // the list of the turn before has been read
        if (tid == 0) n_posted = 0;
        __syncthreads();
        for (int k = base + wave; k < min(base + REFRESH_POSTED, cnt); k += BLOCK / WAVE) {
            const int s = __builtin_amdgcn_readfirstlane(list[1 + k]);
            if (s < 0 || s >= M) continue;                    // (the same for the whole wave)
            const int lo = min(max(sst[s], 0), n), hi = min(max(sst[s + 1], 0), n);
            if (hi - lo <= 0 || hi - lo > LONG_SET_MIN) continue;
            if (hi - lo > SPLIT_SET_MIN) {
                if (lane == 0) posted[atomicAdd(&n_posted, 1)] = s;
                continue;
            }
            const int p = min(max(piv[s], lo), hi - 1);
            merge_one_set<T, false, MODE, false, false>(Ks, Vs, Ko + (size_t)s * HEAD_DIM, Vo + (size_t)s * HEAD_DIM, nullptr, lo, hi, p, a, lane,
                                                 set_w[wave], part);
        }
        __syncthreads();
        const int n_team = n_posted;
        for (int k = wave / SPLIT_PARTS; k < (n_team + TEAMS - 1) / TEAMS * TEAMS; k += TEAMS) {   // (as many turns for every team)
            const int s = __builtin_amdgcn_readfirstlane(posted[min(k, n_team - 1)]);
            const int lo = min(max(sst[s], 0), n), hi = k < n_team ? max(min(max(sst[s + 1], 0), n), lo) : lo;
            const int p = max(min(max(piv[s], lo), hi - 1), 0);
            merge_set_team<T, false, MODE>(Ks, Vs, Ko + (size_t)s * HEAD_DIM, Vo + (size_t)s * HEAD_DIM, nullptr, lo, min(hi, lo + LONG_SET_MIN), p, a,
                                           lane, wave % SPLIT_PARTS, team_mem[wave / SPLIT_PARTS], part);
        }
    }
    if constexpr (BLOCK == LONG_SET_BLOCK) {
        __shared__ LongShared long_sums;
        for (int k = 0; k < min(n_long, max_long); ++k) {     // (the same for the whole workgroup)
            const int s = __builtin_amdgcn_readfirstlane(pl[1 + k]);
            if (s < 0 || s >= M) continue;
            const int lo = min(max(sst[s], 0), n), hi = min(max(sst[s + 1], 0), n);
            if (hi <= lo) continue;
            const int p = min(max(piv[s], lo), hi - 1);
            merge_long_set<T, false, MODE>(Ks, Vs, Ko + (size_t)s * HEAD_DIM, Vo + (size_t)s * HEAD_DIM, nullptr, lo, hi, p, a, tid, long_sums, part);
        }
    }
}

template <typename T>
static kvm_status launch_refresh_t(const kvm_shape &sh, const void *K, const void *V, void *K_out, void *V_out,
                                   const MergeArgs &ma, const RefreshArgs &ra, hipStream_t st)
{
    const long long slices = (long long)sh.B * sh.H_kv;
    const bool few = refresh_few(sh);
    {
        ProfScope prof(ra.parts > 2 ? "refresh_kernel_4" : ra.parts > 1 ? "refresh_kernel_2" : few ? "refresh_kernel_few" : "refresh_kernel", st);
        const auto run = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(slices * ra.parts)), dim3(few ? REFRESH_BLOCK_FEW : REFRESH_BLOCK), 0, st, (const T *)K,
                               (const T *)V, (T *)K_out, (T *)V_out, ma, ra);
        };
        const auto pick = [&](auto mode) {
            constexpr int MODE = decltype(mode)::value;
            if (ra.parts > 1) run(refresh_kernel<T, MODE, REFRESH_BLOCK_FEW, true>);
            else if (few) run(refresh_kernel<T, MODE, REFRESH_BLOCK_FEW, false>);
            else run(refresh_kernel<T, MODE, REFRESH_BLOCK, false>);
        };
        if (ma.mode == MERGE_AVERAGE) pick(std::integral_constant<int, MERGE_AVERAGE>());
        else if (ma.mode == MERGE_FIXED) pick(std::integral_constant<int, MERGE_FIXED>());
        else pick(std::integral_constant<int, MERGE_ADAPTIVE>());
    }
    kvm_status rc = check_launch("refresh_kernel");
    if (rc != KVM_OK || few || sh.N <= LONG_SET_MIN) return rc;
    launch_merge_long_t<T>(sh, K, V, K_out, V_out, ma, st);
    return check_launch("merge_long_kernel");
}

size_t merge_refresh_workspace_bytes(const kvm_shape &sh, int cap_rows)
{
    return (size_t)sh.B * sh.H_kv * ((size_t)merge_ws_stride(sh.N) + 2 * (size_t)cap_rows + 1) * sizeof(int32_t);
}

// Workgroups per slice of a refresh that has ws_bytes of workspace (the lists of the ones beyond the first stand behind the rest; the size that
// kvm_workspace_bytes gives has room for four up to a budget of 0.64, for two always).
static int refresh_parts(const kvm_shape &sh, int cap_rows, size_t ws_bytes)
{
    const size_t slices = (size_t)sh.B * sh.H_kv;
    const size_t each = slices * ((size_t)cap_rows + 2 + max_long_sets(sh.N)) * sizeof(int32_t);   // lists of one more workgroup a slice
    int parts = 1;
    if (!refresh_few(sh) || cap_rows <= 2 * REFRESH_MOVE_ROWS / (sh.dtype == KVM_F32 ? 2 : 1)) return parts;
    while (parts < REFRESH_MAX_PARTS && (long long)slices * 2 * parts <= REFRESH_FEW_SLICES &&
           merge_refresh_workspace_bytes(sh, cap_rows) + (2 * parts - 1) * each <= ws_bytes)
        parts *= 2;
    return parts;
}

kvm_status launch_merge_refresh(const kvm_shape &sh, const kvm_params &pr, int cap_rows, const void *K, const void *V,
                                const int32_t *prev_set_id, const int32_t *prev_set_start, const int32_t *prev_pivot,
                                const int32_t *prev_n_sets, const int32_t *set_start, const int32_t *pivot,
                                const int32_t *n_sets, void *K_out, void *V_out, int32_t *n_changed, int32_t *ws, size_t ws_bytes, hipStream_t st)
{
    const size_t slices = (size_t)sh.B * sh.H_kv;
    if (slices == 0 || cap_rows == 0 || sh.N == 0) return KVM_OK;
    const int stride = merge_ws_stride(sh.N);
    RefreshArgs ra;
    ra.prev_set_id = prev_set_id;
    ra.prev_set_start = prev_set_start;
    ra.prev_pivot = prev_pivot;
    ra.prev_n_sets = prev_n_sets;
    ra.src = ws + slices * stride;
    ra.lists = ra.src + slices * cap_rows;
    ra.long_list = ws + long_list_offset(sh.N);
    ra.n_changed = n_changed;
    ra.part_lists = ra.lists + slices * (cap_rows + 1);
    ra.parts = refresh_parts(sh, cap_rows, ws_bytes);
    MergeArgs ma;
    ma.set_start = set_start;
    ma.pivot = pivot;
    ma.n_sets = n_sets;
    ma.seq_lens = sh.seq_lens;
    ma.w_opt = nullptr;
    ma.long_list = ra.long_list;
    ma.list_stride = stride;
    ma.slices = sh.B * sh.H_kv;
    ma.H = sh.H_kv;
    ma.N = sh.N;
    ma.cap_rows = cap_rows;
    ma.tile = ma.tiles_per_slice = 0;                        // (merge_kernel is not launched)
    ma.mode = pr.weights == KVM_WEIGHTS_AVERAGE ? MERGE_AVERAGE : (pr.sigma_mode == KVM_SIGMA_FIXED ? MERGE_FIXED : MERGE_ADAPTIVE);
    ma.inv_two_sigma_sq = ma.mode == MERGE_FIXED ? 1.f / (2.f * pr.sigma * pr.sigma) : 0.f;
    ma.value_scale = pr.value_scale_by_set_size;
    switch (sh.dtype) {
    case KVM_F32: return launch_refresh_t<float>(sh, K, V, K_out, V_out, ma, ra, st);
    case KVM_F16: return launch_refresh_t<half_t>(sh, K, V, K_out, V_out, ma, ra, st);
    default: return launch_refresh_t<bf16_t>(sh, K, V, K_out, V_out, ma, ra, st);
    }
}

// ------------------------------------------------------------------------------------------
// The merge for callers that cannot bring a workspace.  Nothing is kept between its kernels; the size
// limit of the entry point, once that of a work plan in a buffer of the library, is part of its contract.
// ------------------------------------------------------------------------------------------

constexpr size_t STATIC_MAX_ENTRIES = (size_t)KVM_MERGE_STATIC_MAX_PLAN_ENTRIES;

kvm_status launch_merge_static(const kvm_shape &sh, const kvm_params &pr, int cap_rows, const void *K, const void *V,
                               const int32_t *set_start, const int32_t *pivot, const int32_t *n_sets, void *K_out,
                               void *V_out, float *w_opt, hipStream_t st)
{
    const size_t need = merge_workspace_bytes(sh) / sizeof(int32_t);
    if (need > STATIC_MAX_ENTRIES) {
        set_error("kvm_merge_static: the shape counts %zu entries (B*H_kv*(ceil(N/64)+floor(N/513)+3)), the limit of this call is %zu "
                  "(the size of a built-in buffer it once used); use kvm_merge with a workspace", need, STATIC_MAX_ENTRIES);
        return KVM_ERR_WORKSPACE;
    }
    return launch_merge(sh, pr, cap_rows, K, V, set_start, pivot, n_sets, K_out, V_out, w_opt, st);
}

}  // namespace kvm
