// Order-preserving dictionary encoding of fixed-width string columns.
//
// A string column is a zero-padded byte matrix [n][L] (L a multiple of 4,
// at most 32; strings hold no zero bytes).  Its dictionary is the sorted
// list of distinct strings, one per row of a [d][L] byte matrix, and a
// string's code is its position there, so codes compare as the strings do
// and equal strings have equal codes: the codes serve as int32 keys of the
// filter, join and group-by operators.
//
// Build (one call, asynchronous): every row inserts itself into an
// open-addressing table of row ids keyed by the string (a slot keeps the
// first row that claimed it; a later row with the same string finds it by
// comparing the words) and records its slot; the occupied slots are
// compacted to one representative row per distinct string; the
// representatives are sorted by string (tiles of 1024 in LDS, then merges of
// 16 runs); the position of each becomes the code of its slot and its bytes
// the dictionary row; finally every row reads its code through its slot.
// Lookup searches a sample of every S-th dictionary string held in LDS, then
// the one run of S strings in memory.  Strings compare as sequences of
// big-endian 32-bit words, which is byte-wise lexicographic order with the
// zero padding sorting first.
#include "common.hpp"

namespace tdp {

namespace {

constexpr int kDictMaxWords = 8;  // 32 bytes

// The W words of one string as they lie in memory: loads of up to 16 bytes
// when the string starts that aligned.
template <int W>
__device__ __forceinline__ void load_raw(const uint32_t* s, bool aligned, uint32_t w[W]) {
    constexpr int V = W % 4 == 0 ? 4 : W % 2 == 0 ? 2 : 1;
    typedef uint32_t vec __attribute__((ext_vector_type(V)));
    if (V > 1 && aligned) {
#pragma unroll
        for (int k = 0; k < W; k += V) {
            const vec q = *(const vec*)(s + k);
#pragma unroll
            for (int e = 0; e < V; ++e) w[k + e] = ((const uint32_t*)&q)[e];
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < W; ++k) w[k] = s[k];
}

// The W words of one string as big-endian values (zero past W): 16-byte
// loads when the string starts 16-byte aligned and W is a multiple of 4 (a
// search step is then one load instruction, not four whose lanes each touch
// another cache line), 4-byte loads otherwise.
__device__ __forceinline__ void load_words(const uint32_t* s, int W, uint32_t w[kDictMaxWords]) {
    if ((W & 3) == 0 && ((uintptr_t)s & 15) == 0) {
#pragma unroll
        for (int k = 0; k < kDictMaxWords; k += 4) {
            uint4 q = make_uint4(0u, 0u, 0u, 0u);
            if (k < W) q = *(const uint4*)(s + k);
            w[k] = __builtin_bswap32(q.x);
            w[k + 1] = __builtin_bswap32(q.y);
            w[k + 2] = __builtin_bswap32(q.z);
            w[k + 3] = __builtin_bswap32(q.w);
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < kDictMaxWords; ++k) w[k] = k < W ? __builtin_bswap32(s[k]) : 0u;
}

// -1, 0, 1 as a < b, a == b, a > b (big-endian words, lexicographic).
__device__ __forceinline__ int cmp_words(const uint32_t a[kDictMaxWords], const uint32_t b[kDictMaxWords], int W) {
#pragma unroll
    for (int k = 0; k < kDictMaxWords; ++k) {
        if (k >= W) break;
        if (a[k] != b[k]) return a[k] < b[k] ? -1 : 1;
    }
    return 0;
}

template <int W>
__device__ __forceinline__ uint32_t hash_raw(const uint32_t w[W]) {
    uint32_t h = 0x9E3779B9u;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        h = (h ^ w[k]) * 0x85EBCA6Bu;
        h ^= h >> 15;
    }
    return hash32(h);
}

template <int W>
__device__ __forceinline__ bool same_raw(const uint32_t a[W], const uint32_t b[W]) {
    uint32_t d = 0;
#pragma unroll
    for (int k = 0; k < W; ++k) d |= a[k] ^ b[k];
    return d == 0;
}

__global__ void dict_fill_kernel(int32_t* p, int64_t n, int32_t v, int64_t* d_count, int32_t* status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *d_count = 0;
        if (status) *status = 0;
    }
}

// The rows of a pass over a column whose rows repeat their strings: of every
// group of 16 units of kUnitRows rows one unit is the sample, at a place that
// varies from group to group, so that the sample shows the strings of a sorted
// or clustered column too, and of one that repeats every so many rows.
// PASS_FIRST takes the sample of one of every four groups (again at varying
// places), PASS_SAMPLE that of the others, PASS_REST the units outside it.
enum DictPass { PASS_ALL, PASS_FIRST, PASS_SAMPLE, PASS_REST };
constexpr int kUnitRows = 8;
constexpr int kGroupUnits = 16;

// The j-th number from 0 on whose place among every N, in quotient q = j / (N - 1)
// of them, is not `taken`.
template <int N>
__device__ __forceinline__ uint32_t skip_one(uint32_t j, uint32_t q, uint32_t taken) {
    const uint32_t o = j - q * (N - 1);
    return q * N + o + (o >= taken);
}

// k-th row of a pass (some lie past the column's end), and their number.
template <int PASS>
__device__ __forceinline__ int64_t pass_row(int64_t k) {
    if (PASS == PASS_ALL) return k;
    const uint32_t j = (uint32_t)(k / kUnitRows);
    auto unit_of = [](uint32_t g) { return hash32(g) % kGroupUnits; };
    auto quarter_of = [](uint32_t q) { return hash32(~q) % 4; };
    uint32_t unit;
    if (PASS == PASS_REST) {
        const uint32_t g = j / (kGroupUnits - 1);
        unit = skip_one<kGroupUnits>(j, g, unit_of(g));
    } else {
        const uint32_t g = PASS == PASS_FIRST ? 4 * j + quarter_of(j) : skip_one<4>(j, j / 3, quarter_of(j / 3));
        unit = g * kGroupUnits + unit_of(g);
    }
    return (int64_t)unit * kUnitRows + k % kUnitRows;
}

int64_t pass_rows(int pass, int64_t n) {
    const int64_t groups = ceil_div(n, (int64_t)kGroupUnits * kUnitRows), quarters = ceil_div(groups, (int64_t)4);
    switch (pass) {
        case PASS_FIRST: return quarters * kUnitRows;
        case PASS_SAMPLE: return quarters * 3 * kUnitRows;
        case PASS_REST: return groups * (kGroupUnits - 1) * kUnitRows;
        default: return n;
    }
}

// Each of the pass's `rows` rows finds or claims the slot of its string;
// row_slot[i] = the slot.  PASS_REST: `seen` holds copies of the strings whose
// slots the sample claimed, [slot][W], so a row whose string
// is among them reads one line of a small array instead of a slot and then a
// row of the column at a random place (the column's lines, 128 bytes for each
// row's 16, were the bound of the one-launch form: 235 us for 10M rows of
// 100K distinct 16-byte strings).  A copy that begins with a zero word is no
// copy: the slot was free then, or holds the empty string.
// A thread takes kRows rows at a time, 256 apart, and walks their probe
// sequences together: a wave lasts as long as its longest sequence, so one
// row after the other would add up the longest of each.
template <int W, int PASS>
__global__ __launch_bounds__(256) void dict_insert_kernel(const uint32_t* __restrict__ strs, int64_t rows, int64_t n,
                                                          int32_t* table, uint32_t mask,
                                                          const uint32_t* __restrict__ seen, int32_t* row_slot,
                                                          int32_t* status) {
    constexpr bool SEEN = PASS == PASS_REST;
    constexpr int kRows = SEEN ? (W <= 4 ? 4 : 2) : 1;
    const int64_t step = 256 * kRows;
    const bool aligned = ((uintptr_t)strs & 15) == 0;
    for (int64_t k0 = (int64_t)blockIdx.x * step; k0 < rows; k0 += (int64_t)gridDim.x * step) {
        int64_t row[kRows];
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
            const int64_t k = k0 + e * 256 + threadIdx.x;
            row[e] = k < rows ? pass_row<PASS>(k) : n;
        }
        uint32_t w[kRows][W], s[kRows];
        bool found[kRows];
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
            load_raw<W>(strs + (row[e] < n ? row[e] : n - 1) * W, aligned, w[e]);
        }
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
            s[e] = hash_raw<W>(w[e]) & mask;
            found[e] = false;
        }
        uint32_t probes = 0;  // of the rows that probed longest
        if (SEEN) {
            bool walk[kRows], any = true;
#pragma unroll
            for (int e = 0; e < kRows; ++e) walk[e] = true;
            for (; any && probes <= mask; ++probes) {
                uint32_t o[kRows][W];
#pragma unroll
                for (int e = 0; e < kRows; ++e)
                    if (walk[e]) load_raw<W>(seen + (int64_t)s[e] * W, true, o[e]);
                any = false;
#pragma unroll
                for (int e = 0; e < kRows; ++e) {
                    if (!walk[e]) continue;
                    found[e] = o[e][0] != 0 && same_raw<W>(w[e], o[e]);
                    walk[e] = o[e][0] != 0 && !found[e];
                    if (walk[e]) s[e] = (s[e] + 1) & mask;
                    any |= walk[e];
                }
            }
        }
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
            const int64_t i = row[e];
            if (i >= n) continue;
            int32_t slot = found[e] ? (int32_t)s[e] : -1;
            for (uint32_t p = 0; slot < 0 && p <= mask; ++p) {
                // a claimed slot never changes, so a plain (cached) read that
                // sees a row is final; one that sees the slot empty may be
                // stale, and the compare-and-swap then returns the slot's
                // current value
                int32_t cur = table[s[e]];
                if (cur < 0) cur = atomicCAS(&table[s[e]], -1, (int32_t)i);
                bool mine = cur < 0;
                if (!mine) {
                    uint32_t o[W];
                    load_raw<W>(strs + (int64_t)cur * W, aligned, o);
                    mine = same_raw<W>(w[e], o);
                }
                if (mine) slot = (int32_t)s[e];
                else s[e] = (s[e] + 1) & mask;
            }
            if (slot < 0) raise_flag(status, TDP_FLAG_TABLE_FULL);
            row_slot[i] = slot;
        }
    }
}

// Copies of the claimed slots' strings (zeros for free slots).
__global__ void dict_seen_kernel(const uint32_t* __restrict__ strs, int W, const int32_t* table, int64_t n_slots,
                                 uint32_t* seen) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_slots * W; e += stride) {
        const int32_t r = table[e / W];
        seen[e] = r >= 0 ? strs[(int64_t)r * W + e % W] : 0u;
    }
}

// One representative row per occupied slot, in any order; more than `cap`
// distinct strings raise the flag.  A workgroup reserves the positions of its
// 4096 slots with one atomic add: an add per wave serialised on the one
// counter (51 us for 2^18 slots; 5 us now).
constexpr int kCompactThreads = 1024;

__global__ __launch_bounds__(kCompactThreads) void dict_compact_kernel(const int32_t* table, int64_t n_slots,
                                                                       int32_t* reps, int64_t cap, int64_t* d_count,
                                                                       int32_t* status) {
    __shared__ uint32_t s_wave[kCompactThreads / kWave];
    __shared__ unsigned long long s_first;
    const int wave = threadIdx.x / kWave;
    const int64_t step = (int64_t)kCompactThreads * 4;
    for (int64_t s0 = (int64_t)blockIdx.x * step; s0 < n_slots; s0 += (int64_t)gridDim.x * step) {
        const int64_t s = s0 + threadIdx.x * 4;  // n_slots is a multiple of 4
        int4 r = make_int4(-1, -1, -1, -1);
        if (s < n_slots) r = *(const int4*)&table[s];
        uint32_t below, total;
        wave_count_scan<3>((uint32_t)((r.x >= 0) + (r.y >= 0) + (r.z >= 0) + (r.w >= 0)), below, total);
        if (lane_id() == 0) s_wave[wave] = total;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t sum = 0;
            for (int w = 0; w < kCompactThreads / kWave; ++w) {
                const uint32_t c = s_wave[w];
                s_wave[w] = sum;
                sum += c;
            }
            s_first = sum ? atomicAdd((unsigned long long*)d_count, (unsigned long long)sum) : 0;
        }
        __syncthreads();
        int64_t k = (int64_t)s_first + s_wave[wave] + below;
        const int32_t v[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (v[e] < 0) continue;
            if (k < cap) reps[k] = v[e];
            else raise_flag(status, TDP_FLAG_TABLE_FULL);
            ++k;
        }
        __syncthreads();
    }
}

// The representatives are sorted by tiles of kTile in LDS, then by merges of
// kMergeWay sorted runs at a time in which every representative finds its
// place by binary searches of the other runs of its group: one launch per
// factor of kMergeWay (two for 100K strings, where a bitonic network over the
// same tiles took 28 launches and 212 us).  A launch works on the first
// *d_count representatives (at most cap) and does little past them.
constexpr int kTile = 1024;
constexpr int kSortThreads = kTile / 2;
constexpr int kMergeWay = 16;
constexpr int kMergeWaves = 4;  // waves that share the searches of 64 representatives
constexpr int kMergeGrid = 1 << 15;  // most workgroups of a merge

// Word pair p of a string, most significant word first.
__device__ __forceinline__ uint64_t load_pair(const uint32_t* s, int W, int p) {
    const uint64_t hi = (uint64_t)__builtin_bswap32(s[2 * p]) << 32;
    return 2 * p + 1 < W ? hi | __builtin_bswap32(s[2 * p + 1]) : hi;
}

// d representatives in order: their rows, and their strings as columns of word
// pairs (pair p of representative i from words[2 * (p * d + i)] on, then a
// column of single words where W is odd), so that they take as many bytes as d
// rows of the dictionary, whose buffer holds one of the two runs of a merge.
struct DictRun {
    int32_t* rep;
    uint32_t* words;
};
typedef uint64_t __attribute__((aligned(4))) u64a4;

template <int W>
__device__ __forceinline__ uint64_t run_pair(const DictRun& r, int64_t d, int p, int64_t i) {
    if (2 * p + 1 == W) return (uint64_t)r.words[2 * p * d + i] << 32;
    return *(const u64a4*)&r.words[2 * (p * d + i)];
}

template <int W>
__device__ __forceinline__ void put_pair(const DictRun& r, int64_t d, int p, int64_t i, uint64_t v) {
    if (2 * p + 1 == W) r.words[2 * p * d + i] = (uint32_t)(v >> 32);
    else *(u64a4*)&r.words[2 * (p * d + i)] = v;
}

// A bitonic network over one tile.  Only the first pair and the tile position
// move; a tie reads the other pairs where they were loaded.  Strides of at
// most a wave's 128 elements need no workgroup barrier.
template <int W>
__global__ __launch_bounds__(kSortThreads) void dict_tile_sort_kernel(const uint32_t* __restrict__ strs,
                                                                      const int32_t* reps, const int64_t* d_count,
                                                                      int64_t cap, DictRun out) {
    constexpr int P = (W + 1) / 2;      // word pairs
    constexpr uint16_t kNone = 0xFFFF;  // no string: sorts last
    __shared__ uint64_t s_key[kTile];
    __shared__ uint64_t s_rest[P > 1 ? P - 1 : 1][kTile];
    __shared__ uint16_t s_at[kTile];
    const int64_t d = *d_count < cap ? *d_count : cap;
    const int64_t base = (int64_t)blockIdx.x * kTile;
    if (base >= d) return;
    const int m = (int)(d - base < kTile ? d - base : kTile);
#pragma unroll
    for (int e = threadIdx.x; e < kTile; e += kSortThreads) {
        const uint32_t* q = strs + (int64_t)reps[base + (e < m ? e : 0)] * W;
        s_at[e] = e < m ? (uint16_t)e : kNone;
        s_key[e] = e < m ? load_pair(q, W, 0) : ~0ull;
#pragma unroll
        for (int p = 1; p < P; ++p) s_rest[p - 1][e] = load_pair(q, W, p);
    }
    __syncthreads();
    int span = 2;  // the tile's power of two
    while (span < m) span <<= 1;
    for (int kk = 2; kk <= span; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
            const int t = threadIdx.x;
            const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
            const int l = i | j;
            if (i < span) {
                const uint64_t x = s_key[i], y = s_key[l];
                const uint16_t ax = s_at[i], ay = s_at[l];
                bool gt = x > y;
                if (x == y) {
                    gt = ax == kNone && ay != kNone;
                    if (P > 1 && ax != kNone && ay != kNone) {
                        bool open = true;
#pragma unroll
                        for (int p = 0; p < P - 1; ++p) {
                            const uint64_t a = s_rest[p][ax], b = s_rest[p][ay];
                            if (open && a != b) {
                                gt = a > b;
                                open = false;
                            }
                        }
                    }
                }
                // strings are distinct, so "not greater" is "smaller" except between two missing ones
                if (gt == ((i & kk) == 0)) {
                    s_key[i] = y;
                    s_key[l] = x;
                    s_at[i] = ay;
                    s_at[l] = ax;
                }
            }
            if (j > kWave) __syncthreads();
            else wave_lds_sync();
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < m; e += kSortThreads) {
        const int at = s_at[e];
        out.rep[base + e] = reps[base + at];
        put_pair<W>(out, d, 0, base + e, s_key[e]);
#pragma unroll
        for (int p = 1; p < P; ++p) put_pair<W>(out, d, p, base + e, s_rest[p - 1][at]);
    }
}

// One merge of up to kMergeWay sorted runs of `run` representatives: the place
// of each in the merged run is its place in its own run plus the number of
// smaller strings in each other run of the group.  A workgroup takes 64
// neighbours of one run, whose searches touch the same few lines, and its
// waves share the runs, four searches in flight per lane.  LAST (one group in
// all): the place is the string's code and its row of the dictionary.
template <int W, bool LAST>
__global__ __launch_bounds__(kMergeWaves * kWave) void dict_merge_kernel(DictRun in, DictRun out, int64_t run,
                                                                         const int64_t* d_count, int64_t cap,
                                                                         const int32_t* row_slot, int32_t* slot_code,
                                                                         uint32_t* dict) {
    constexpr int P = (W + 1) / 2;
    constexpr int kPer = kMergeWay / kMergeWaves;
    __shared__ int32_t s_part[kMergeWaves][kWave];
    const int64_t d = *d_count < cap ? *d_count : cap;
    const int wave = threadIdx.x / kWave;
    for (int64_t i0 = (int64_t)blockIdx.x * kWave; i0 < d; i0 += (int64_t)gridDim.x * kWave) {
        const int64_t i = i0 + lane_id();
        const bool have = i < d;
        uint64_t key[P];
#pragma unroll
        for (int p = 0; p < P; ++p) key[p] = run_pair<W>(in, d, p, have ? i : d - 1);
        const int64_t own = i0 / run;                           // run is a multiple of 64
        const int64_t g0 = own / kMergeWay * kMergeWay;         // first run of the group
        int64_t first[kPer];
        int32_t lo[kPer], len[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int64_t r = g0 + wave * kPer + k;
            first[k] = r * run;
            const int64_t left = d - first[k];
            len[k] = r == own || left <= 0 ? 0 : (int32_t)(left < run ? left : run);
            if (len[k] == 0) first[k] = 0;
            lo[k] = 0;
        }
        // lo counts strings known to be smaller; the last step can find the whole run smaller
        for (int64_t step = run / 2; step >= 0; step = step > 1 ? step >> 1 : step - 1) {
            const int32_t s = step > 0 ? (int32_t)step : 1;
            uint64_t x[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) x[k] = run_pair<W>(in, d, 0, first[k] + (lo[k] + s <= len[k] ? lo[k] + s - 1 : 0));
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                if (lo[k] + s > len[k]) continue;
                bool less = x[k] < key[0];
                if (P > 1 && x[k] == key[0]) {
                    bool open = true;
#pragma unroll
                    for (int p = 1; p < P; ++p) {
                        const uint64_t y = run_pair<W>(in, d, p, first[k] + lo[k] + s - 1);
                        if (open && y != key[p]) {
                            less = y < key[p];
                            open = false;
                        }
                    }
                }
                if (less) lo[k] += s;
            }
        }
        int32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) sum += lo[k];
        s_part[wave][lane_id()] = sum;
        __syncthreads();
        if (wave == 0 && have) {
            int64_t rank = g0 * run + i - own * run;
#pragma unroll
            for (int w = 0; w < kMergeWaves; ++w) rank += s_part[w][lane_id()];
            const int32_t row = in.rep[i];
            if (LAST) {
                slot_code[row_slot[row]] = (int32_t)rank;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    dict[rank * W + 2 * p] = __builtin_bswap32((uint32_t)(key[p] >> 32));
                    if (2 * p + 1 < W) dict[rank * W + 2 * p + 1] = __builtin_bswap32((uint32_t)key[p]);
                }
            } else {
                out.rep[rank] = row;
#pragma unroll
                for (int p = 0; p < P; ++p) put_pair<W>(out, d, p, rank, key[p]);
            }
        }
        __syncthreads();  // the counts have been read
    }
}

// Four rows per thread and step when `codes` is 16-byte aligned (16-byte
// loads of the workspace's row slots and stores of codes), the tail of
// fewer than four rows one by one.
__global__ void dict_codes_kernel(const int32_t* row_slot, int64_t n, const int32_t* slot_code, int32_t* codes) {
    const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t tail = 0;
    if (((uintptr_t)codes & 15) == 0) {
        const int64_t n4 = n / 4;
        for (int64_t q = t; q < n4; q += nthreads) {
            const int4 s = *(const int4*)&row_slot[q * 4];
            int4 c;
            c.x = s.x >= 0 ? slot_code[s.x] : -1;
            c.y = s.y >= 0 ? slot_code[s.y] : -1;
            c.z = s.z >= 0 ? slot_code[s.z] : -1;
            c.w = s.w >= 0 ? slot_code[s.w] : -1;
            *(int4*)&codes[q * 4] = c;
        }
        tail = n4 * 4;
    }
    for (int64_t j = tail + t; j < n; j += nthreads) {
        const int32_t s = row_slot[j];
        codes[j] = s >= 0 ? slot_code[s] : -1;
    }
}

// Lower bound of each string in the sorted dictionary, and whether it is
// there: first among the samples dict[0], dict[S], dict[2S], ... (held in
// LDS), which leaves one run of fewer than S strings to search in memory.
constexpr int kLookupThreads = 1024;
constexpr int kLookupLdsBytes = 48 * 1024;

__global__ __launch_bounds__(kLookupThreads) void dict_lookup_kernel(const uint32_t* __restrict__ dict, int64_t d,
                                                                     int W, const uint32_t* __restrict__ strs,
                                                                     int64_t n, int sshift, int ns, int32_t* pos,
                                                                     int8_t* found) {
    extern __shared__ uint32_t s_samp[];  // [ns][W] big-endian words
    for (int e = threadIdx.x; e < ns * W; e += blockDim.x) {
        const int q = e / W, k = e - q * W;
        s_samp[e] = __builtin_bswap32(dict[((int64_t)q << sshift) * W + k]);
    }
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint32_t w[kDictMaxWords];
        load_words(strs + i * W, W, w);
        int slo = 0, shi = ns;  // first sample >= w
        while (slo < shi) {
            const int mid = (slo + shi) >> 1;
            uint32_t m[kDictMaxWords];
#pragma unroll
            for (int k = 0; k < kDictMaxWords; ++k) m[k] = k < W ? s_samp[mid * W + k] : 0u;
            if (cmp_words(m, w, W) < 0) slo = mid + 1;
            else shi = mid;
        }
        // the lower bound lies in ((slo - 1) * S, min(slo * S, d)]
        int64_t lo = slo == 0 ? 0 : ((int64_t)(slo - 1) << sshift) + 1;
        int64_t hi = ((int64_t)slo << sshift) < d ? ((int64_t)slo << sshift) : d;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            uint32_t m[kDictMaxWords];
            load_words(dict + mid * W, W, m);
            if (cmp_words(m, w, W) < 0) lo = mid + 1;
            else hi = mid;
        }
        int8_t f = 0;
        if (lo < d) {
            uint32_t m[kDictMaxWords];
            load_words(dict + lo * W, W, m);
            f = cmp_words(m, w, W) == 0 ? 1 : 0;
        }
        pos[i] = (int32_t)lo;
        if (found) found[i] = f;
    }
}

__global__ void dict_decode_kernel(const int32_t* codes, int64_t n, const uint32_t* dict, int64_t d, int W,
                                   uint32_t* out, int32_t* status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t c = codes[i];
        const bool in = c >= 0 && c < d;
        if (!in) raise_flag(status, TDP_FLAG_KEY_DOMAIN);
        for (int k = 0; k < W; ++k) out[i * W + k] = in ? dict[(int64_t)c * W + k] : 0u;
    }
}

// When the bound promises at least kSeenRepeat rows per string, a sixteenth of
// the rows claims most slots and the rest read the copies of their strings; a
// quarter of that sample goes alone, so that few rows at a time find a
// slot empty (each such row is a device-scope compare-and-swap, about 11 G/s:
// 46 us for a sixteenth of 10M rows in one launch, 2 x 20 us in two).  These
// builds get four slots per string: a wave waits for its longest probe
// sequence (10M rows, 100K strings: 298 us for the whole encoding with four
// slots, 318 with two, 585 at 76% load, 330 with eight).
constexpr int64_t kSeenMinRows = 1 << 17;
constexpr int64_t kSeenRepeat = 8;

struct DictWs {
    int32_t* table;
    int32_t* slot_code;
    int32_t* row_slot;
    int32_t* reps;
    uint32_t* seen;  // string copies by slot, for builds whose rows repeat their strings (null otherwise)
    uint32_t* words; // strings of the sorted run that is not in the dictionary's buffer
    int64_t n_slots;
};

DictWs dict_layout(void* ws, int64_t n, int64_t max_distinct, int W, size_t* bytes) {
    DictWs w;
    int64_t slots = 256;
    const bool repeats = n >= kSeenMinRows && n >= kSeenRepeat * max_distinct;
    // slots are int32 (a bound above 2^30 fills its table beyond a half)
    while (slots < (repeats ? 4 : 2) * max_distinct && slots < (int64_t)1 << 31) slots <<= 1;
    WsAlloc wa(ws);
    w.table = wa.take<int32_t>(slots);
    w.slot_code = wa.take<int32_t>(slots);
    w.row_slot = wa.take<int32_t>(std::max<int64_t>(n, 1));
    w.reps = wa.take<int32_t>(max_distinct);
    w.words = wa.take<uint32_t>(max_distinct * W);
    w.seen = repeats ? wa.take<uint32_t>(slots * W) : nullptr;
    w.n_slots = slots;
    if (bytes) *bytes = wa.bytes();
    return w;
}

int dict_grid(int64_t n) { return (int)std::min<int64_t>(std::max<int64_t>(ceil_div(n, 256), 1), 8192); }

template <int W>
void dict_insert(const uint32_t* strs, int64_t n, const DictWs& w, int32_t* status, hipStream_t stream) {
    const uint32_t mask = (uint32_t)(w.n_slots - 1);
    auto run = [&](auto kernel, int pass, int rows_per_thread) {
        const int64_t rows = pass_rows(pass, n);
        if (rows > 0)
            kernel<<<dict_grid(ceil_div(rows, (int64_t)rows_per_thread)), 256, 0, stream>>>(strs, rows, n, w.table, mask,
                                                                                          w.seen, w.row_slot, status);
    };
    if (!w.seen) return run(dict_insert_kernel<W, PASS_ALL>, PASS_ALL, 1);
    run(dict_insert_kernel<W, PASS_FIRST>, PASS_FIRST, 1);
    run(dict_insert_kernel<W, PASS_SAMPLE>, PASS_SAMPLE, 1);
    dict_seen_kernel<<<dict_grid(w.n_slots * W), 256, 0, stream>>>(strs, W, w.table, w.n_slots, w.seen);
    run(dict_insert_kernel<W, PASS_REST>, PASS_REST, 4);
}

template <int W>
void dict_sort(const uint32_t* strs, const DictWs& w, int64_t cap, const int64_t* d_count, uint32_t* dict,
               hipStream_t stream) {
    // The last merge writes the dictionary, so it reads the run in the workspace;
    // the tile sort starts in the one from which the merges before it end there.
    // The table is read no more, and holds the rows of the run that the tile
    // sort, which still reads reps, writes.
    int merges = 0;
    for (int64_t run = kTile; run * kMergeWay < cap; run *= kMergeWay) ++merges;
    int at = merges & 1;
    DictRun runs[2] = {{w.reps, w.words}, {w.reps, dict}};
    runs[at].rep = w.table;
    dict_tile_sort_kernel<W><<<(unsigned)ceil_div(cap, kTile), kSortThreads, 0, stream>>>(strs, w.reps, d_count, cap,
                                                                                         runs[at]);
    const unsigned grid = (unsigned)std::min<int64_t>(ceil_div(cap, kWave), kMergeGrid);
    int64_t run = kTile;
    for (; merges > 0; --merges, run *= kMergeWay, at ^= 1)
        dict_merge_kernel<W, false><<<grid, kMergeWaves * kWave, 0, stream>>>(runs[at], runs[at ^ 1], run, d_count, cap,
                                                                              nullptr, nullptr, nullptr);
    dict_merge_kernel<W, true><<<grid, kMergeWaves * kWave, 0, stream>>>(runs[at], runs[at ^ 1], run, d_count, cap,
                                                                         w.row_slot, w.slot_code, dict);
}

int dict_check_width(int32_t L, const char* fn) {
    if (L < 4 || L > 4 * kDictMaxWords || (L & 3)) return fail(TDP_EINVAL, "%s: width %d is not a multiple of 4 in 4..32", fn, L);
    return TDP_OK;
}

}  // namespace

}  // namespace tdp

using namespace tdp;

namespace {
// The distinct-string bound a build works with: max_distinct, 0 meaning n.
int64_t dict_bound(int64_t n, int64_t max_distinct) {
    return std::max<int64_t>(max_distinct == 0 ? n : std::min(max_distinct, n), 1);
}
}  // namespace

extern "C" size_t tdp_dict_build_workspace_size(int64_t n, int64_t max_distinct) {
    size_t b;
    dict_layout(nullptr, std::max<int64_t>(n, 0), dict_bound(std::max<int64_t>(n, 0), std::max<int64_t>(max_distinct, 0)),
                kDictMaxWords, &b);  // the widest strings
    return b;
}

extern "C" int tdp_dict_build(const uint8_t* strs, int64_t n, int32_t L, int64_t max_distinct, uint8_t* dict,
                              int64_t* d_n_dict, int32_t* codes, int32_t* d_status, void* ws, size_t ws_bytes,
                              hipStream_t stream) {
    int rc = dict_check_width(L, "tdp_dict_build");
    if (rc) return rc;
    if (n < 0 || n > INT32_MAX || max_distinct < 0) return fail(TDP_EINVAL, "tdp_dict_build: n=%lld max_distinct=%lld", (long long)n, (long long)max_distinct);
    if (!d_n_dict || (n > 0 && (!strs || !dict || !codes))) return fail(TDP_EINVAL, "tdp_dict_build: null pointer");
    if ((uintptr_t)strs & 3 || (uintptr_t)dict & 3) return fail(TDP_EINVAL, "tdp_dict_build: strings and dictionary must be 4-byte aligned");
    const int64_t md = dict_bound(n, max_distinct);
    size_t need;
    dict_layout(nullptr, n, md, kDictMaxWords, &need);
    if (!ws || ws_bytes < need) return fail_need(TDP_EWORKSPACE, (int64_t)need, "tdp_dict_build: workspace %zu < %zu", ws_bytes, need);
    if ((uintptr_t)ws & 255) return fail(TDP_EINVAL, "tdp_dict_build: workspace not 256-byte aligned");
    const int W = L / 4;
    DictWs w = dict_layout(ws, n, md, W, nullptr);
    const uint32_t* s32 = (const uint32_t*)strs;
    dict_fill_kernel<<<dict_grid(w.n_slots), 256, 0, stream>>>(w.table, w.n_slots, -1, d_n_dict, d_status);
    if (n > 0) {
        switch (W) {
            case 1: dict_insert<1>(s32, n, w, d_status, stream); break;
            case 2: dict_insert<2>(s32, n, w, d_status, stream); break;
            case 3: dict_insert<3>(s32, n, w, d_status, stream); break;
            case 4: dict_insert<4>(s32, n, w, d_status, stream); break;
            case 5: dict_insert<5>(s32, n, w, d_status, stream); break;
            case 6: dict_insert<6>(s32, n, w, d_status, stream); break;
            case 7: dict_insert<7>(s32, n, w, d_status, stream); break;
            default: dict_insert<8>(s32, n, w, d_status, stream); break;
        }
        dict_compact_kernel<<<(unsigned)std::min<int64_t>(ceil_div(w.n_slots, 4 * kCompactThreads), kCUs), kCompactThreads, 0, stream>>>(
            w.table, w.n_slots, w.reps, md, d_n_dict, d_status);
        uint32_t* out = (uint32_t*)dict;
        switch (W) {
            case 1: dict_sort<1>(s32, w, md, d_n_dict, out, stream); break;
            case 2: dict_sort<2>(s32, w, md, d_n_dict, out, stream); break;
            case 3: dict_sort<3>(s32, w, md, d_n_dict, out, stream); break;
            case 4: dict_sort<4>(s32, w, md, d_n_dict, out, stream); break;
            case 5: dict_sort<5>(s32, w, md, d_n_dict, out, stream); break;
            case 6: dict_sort<6>(s32, w, md, d_n_dict, out, stream); break;
            case 7: dict_sort<7>(s32, w, md, d_n_dict, out, stream); break;
            default: dict_sort<8>(s32, w, md, d_n_dict, out, stream); break;
        }
        dict_codes_kernel<<<dict_grid(ceil_div(n, 4)), 256, 0, stream>>>(w.row_slot, n, w.slot_code, codes);
    }
    return launch_status("tdp_dict_build");
}

extern "C" int tdp_dict_lookup(const uint8_t* dict, int64_t n_dict, int32_t L, const uint8_t* strs, int64_t n,
                               int32_t* pos, int8_t* found, hipStream_t stream) {
    int rc = dict_check_width(L, "tdp_dict_lookup");
    if (rc) return rc;
    if (n < 0 || n_dict < 0 || n_dict > INT32_MAX || (n > 0 && (!strs || !pos)) || (n_dict > 0 && !dict))
        return fail(TDP_EINVAL, "tdp_dict_lookup: null pointer or negative size");
    if ((uintptr_t)strs & 3 || (uintptr_t)dict & 3) return fail(TDP_EINVAL, "tdp_dict_lookup: arrays must be 4-byte aligned");
    if (n == 0) return TDP_OK;
    // samples every S = 2^sshift strings, as many as fit the LDS budget
    const int W = L / 4;
    const int64_t max_samples = kLookupLdsBytes / (W * (int64_t)sizeof(uint32_t));
    int sshift = 0;
    while (ceil_div(n_dict, (int64_t)1 << sshift) > max_samples) ++sshift;
    const int ns = (int)ceil_div(n_dict, (int64_t)1 << sshift);
    const int grid = (int)std::min<int64_t>(std::max<int64_t>(ceil_div(n, kLookupThreads), 1), 4 * kCUs);
    dict_lookup_kernel<<<grid, kLookupThreads, (size_t)ns * W * sizeof(uint32_t), stream>>>(
        (const uint32_t*)dict, n_dict, W, (const uint32_t*)strs, n, sshift, ns, pos, found);
    return launch_status("tdp_dict_lookup");
}

extern "C" int tdp_dict_decode(const int32_t* codes, int64_t n, const uint8_t* dict, int64_t n_dict, int32_t L,
                               uint8_t* out, int32_t* d_status, hipStream_t stream) {
    int rc = dict_check_width(L, "tdp_dict_decode");
    if (rc) return rc;
    if (n < 0 || n_dict < 0 || (n > 0 && (!codes || !out)) || (n_dict > 0 && !dict))
        return fail(TDP_EINVAL, "tdp_dict_decode: null pointer or negative size");
    if ((uintptr_t)out & 3 || (uintptr_t)dict & 3) return fail(TDP_EINVAL, "tdp_dict_decode: arrays must be 4-byte aligned");
    if (n == 0) return TDP_OK;
    dict_decode_kernel<<<dict_grid(n), 256, 0, stream>>>(codes, n, (const uint32_t*)dict, n_dict, L / 4, (uint32_t*)out,
                                                         d_status);
    return launch_status("tdp_dict_decode");
}
