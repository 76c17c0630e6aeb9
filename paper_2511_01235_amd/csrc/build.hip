// Bi-CSR construction on the device (Section 5.1): the same rows, slots, pair
// links and slack as build_bicsr in bicsr.cpp makes on the host.
//
// Every edge (u, v, c) becomes two entries, (u, v, c) and (v, u, 0), keyed by
// row and column.  A radix sort brings equal pairs together; one pass merges
// them (repeated pairs add up, an absent reverse direction keeps capacity 0);
// row lengths plus slack are scanned into row starts; a last pass writes each
// entry's slot and finds its reverse by a binary search in the other row.
//
// Bound by memory traffic: 12 bytes per entry, read twice and written once per
// 8-bit digit of the key, and by the upload of the edges (12 bytes each).
// Loading an RMAT-16 graph (1.05 M edges) takes 1.7 ms with it against 99 ms
// with the host builder (two sorts of pairs by one thread), RMAT-20 (16.8 M)
// 16 ms against 2.37 s.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "mf_internal.h"
#include "slot_index.h"

namespace mf {

namespace {

constexpr int WAVE = 64;
constexpr int BLOCK = 256;
constexpr int WAVES = BLOCK / WAVE;
// A sort tile: each wave takes 1024 consecutive entries, 64 at a time, so that
// entries with equal digits keep their order.
constexpr int ROUNDS = 16;
constexpr int WAVE_ITEMS = ROUNDS * WAVE;
constexpr int TILE = WAVES * WAVE_ITEMS;
constexpr int DIGITS = 256;

// What the host reads back.
struct BuildCounts {
    int invalid;                      // an edge out of range, u == v or c < 0
    int overflow;                     // c(u,v) + c(v,u) of a merged pair above int32
    int long_rows;                    // a row of more than CUT_LONG slots
    int pad;
    long long entries;                // merged entries (slots in use)
    unsigned long long with_capacity; // ... with capacity > 0
};

__device__ __forceinline__ int digit_of(unsigned long long key, int shift) { return (int)(key >> shift) & (DIGITS - 1); }

// exclusive sum of x over the block; *total the block's sum (every thread calls it)
__device__ __forceinline__ long long block_excl(long long x, long long* s_part, long long* total) {
    const int lane = __lane_id(), w = threadIdx.x / WAVE;
    long long inc = x;
    for (int d = 1; d < WAVE; d <<= 1) {
        const long long y = __shfl_up(inc, d, WAVE);
        if (lane >= d) inc += y;
    }
    if (lane == WAVE - 1) s_part[w] = inc;
    __syncthreads();
    long long before = 0, all = 0;
    for (int i = 0; i < WAVES; ++i) {
        if (i < w) before += s_part[i];
        all += s_part[i];
    }
    __syncthreads();
    *total = all;
    return before + inc - x;
}

__global__ void __launch_bounds__(BLOCK) k_build_expand(int n, int64_t m, const int32_t* src, const int32_t* dst,
                                                        const int32_t* cap, int bits, unsigned long long* key,
                                                        int32_t* val, BuildCounts* bc) {
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (i >= m) return;
    const int u = src[i], v = dst[i], c = cap[i];
    if (u < 0 || u >= n || v < 0 || v >= n || u == v || c < 0) {
        bc->invalid = 1;
        key[2 * i] = key[2 * i + 1] = 0;   // in range for the passes behind this one
        val[2 * i] = val[2 * i + 1] = 0;
        return;
    }
    key[2 * i] = (unsigned long long)(unsigned)u << bits | (unsigned)v;
    key[2 * i + 1] = (unsigned long long)(unsigned)v << bits | (unsigned)u;
    val[2 * i] = c;
    val[2 * i + 1] = 0;
}

// entries per digit of one tile -> hist[digit * tiles + tile]
__global__ void __launch_bounds__(BLOCK) k_sort_hist(const unsigned long long* key, int64_t count, int shift,
                                                     unsigned* hist, int tiles) {
    __shared__ unsigned s_h[DIGITS];
    s_h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * TILE;
    for (int r = 0; r < TILE / BLOCK; ++r) {
        const int64_t i = base + r * BLOCK + threadIdx.x;
        if (i < count) atomicAdd(&s_h[digit_of(key[i], shift)], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * tiles + blockIdx.x] = s_h[threadIdx.x];
}

// one block per digit: exclusive sums of its tile counts, and its total
__global__ void __launch_bounds__(BLOCK) k_sort_scan(unsigned* hist, int tiles, unsigned* totals) {
    __shared__ long long s_part[WAVES];
    unsigned* h = hist + (size_t)blockIdx.x * tiles;
    long long carry = 0;
    for (int b = 0; b < tiles; b += BLOCK) {
        const int i = b + threadIdx.x;
        const long long x = i < tiles ? h[i] : 0;
        long long total;
        const long long ex = block_excl(x, s_part, &total);
        if (i < tiles) h[i] = (unsigned)(carry + ex);
        carry += total;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = (unsigned)carry;
}

// Stable scatter of one tile by digit.  A wave ranks its 64 entries of a round
// by matching digits with eight ballots; a counter per wave and digit in LDS
// carries the ranks from round to round, and the waves' counters are summed
// in wave order.
__global__ void __launch_bounds__(BLOCK) k_sort_scatter(const unsigned long long* key, const int32_t* val,
                                                        unsigned long long* key_out, int32_t* val_out, int64_t count,
                                                        int shift, const unsigned* hist, int tiles,
                                                        const unsigned* totals) {
    __shared__ unsigned s_cnt[WAVES][DIGITS];
    __shared__ long long s_part[WAVES];
    const int tid = threadIdx.x, lane = __lane_id(), w = tid / WAVE;
    for (int i = 0; i < WAVES; ++i) s_cnt[i][tid] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * TILE + (int64_t)w * WAVE_ITEMS;
    unsigned long long k[ROUNDS];
    int32_t x[ROUNDS];
    unsigned rank[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = base + r * WAVE + lane;
        const int64_t j = i < count ? i : count - 1;
        k[r] = key[j];
        x[r] = val[j];
    }
    volatile unsigned* cnt = s_cnt[w];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const bool in = base + r * WAVE + lane < count;
        const int d = digit_of(k[r], shift);
        unsigned long long same = __ballot(in);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const unsigned long long m = __ballot(d >> b & 1);
            same &= d >> b & 1 ? m : ~m;
        }
        const unsigned below = (unsigned)__popcll(same & ((1ull << lane) - 1ull));
        const unsigned before = cnt[d];
        rank[r] = before + below;
        __builtin_amdgcn_wave_barrier();
        if (in && below == 0) cnt[d] = before + (unsigned)__popcll(same);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {   // thread d: where each wave's entries of digit d start
        long long all;
        const long long digit_base = block_excl(totals[tid], s_part, &all);
        unsigned at = (unsigned)digit_base + hist[(size_t)tid * tiles + blockIdx.x];
        for (int i = 0; i < WAVES; ++i) {
            const unsigned c = s_cnt[i][tid];
            s_cnt[i][tid] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        if (base + r * WAVE + lane >= count) continue;
        const unsigned p = s_cnt[w][digit_of(k[r], shift)] + rank[r];
        key_out[p] = k[r];
        val_out[p] = x[r];
    }
}

// distinct keys that start in each tile of the sorted entries
__global__ void __launch_bounds__(BLOCK) k_merge_count(const unsigned long long* key, int64_t count, long long* tile) {
    __shared__ long long s_part[WAVES];
    long long c = 0;
    for (int r = 0; r < TILE / BLOCK; ++r) {
        const int64_t i = (int64_t)blockIdx.x * TILE + r * BLOCK + threadIdx.x;
        if (i < count) c += i == 0 || key[i] != key[i - 1];
    }
    long long total;
    block_excl(c, s_part, &total);
    if (threadIdx.x == 0) tile[blockIdx.x] = total;
}

__global__ void __launch_bounds__(BLOCK) k_merge_scan(long long* tile, int tiles, BuildCounts* bc) {
    __shared__ long long s_part[WAVES];
    long long carry = 0;
    for (int b = 0; b < tiles; b += BLOCK) {
        const int i = b + threadIdx.x;
        const long long x = i < tiles ? tile[i] : 0;
        long long total;
        const long long ex = block_excl(x, s_part, &total);
        if (i < tiles) tile[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) bc->entries = carry;
}

// merged entry e: its key, the sum of its capacities (sum[] starts at 0), and
// the first and end entry of every row
__global__ void __launch_bounds__(BLOCK) k_merge(const unsigned long long* key, const int32_t* val, int64_t count,
                                                 const long long* tile, int bits, unsigned long long* mkey,
                                                 unsigned long long* sum, int32_t* first, int32_t* end) {
    __shared__ long long s_part[WAVES];
    long long at = tile[blockIdx.x];
    for (int r = 0; r < TILE / BLOCK; ++r) {
        const int64_t i = (int64_t)blockIdx.x * TILE + r * BLOCK + threadIdx.x;
        const bool in = i < count;
        const unsigned long long k = in ? key[i] : 0ull;
        const unsigned long long p = in && i > 0 ? key[i - 1] : ~0ull;
        const bool head = in && (i == 0 || k != p);
        long long total;
        const long long e = at + block_excl(head, s_part, &total) + head - 1;
        if (head) {
            mkey[e] = k;
            const int row = (int)(k >> bits);
            if (i == 0 || (int)(p >> bits) != row) {
                first[row] = (int32_t)e;
                if (i > 0) end[(int)(p >> bits)] = (int32_t)e;
            }
        }
        if (in && val[i]) atomicAdd(&sum[e], (unsigned long long)val[i]);
        if (in && i == count - 1) end[(int)(k >> bits)] = (int32_t)(e + 1);
        at += total;
    }
}

__global__ void __launch_bounds__(BLOCK) k_build_rows(int n, const int32_t* first, const int32_t* end, int slack_min,
                                                      int slack_pct, int32_t* row_len, int32_t* row_sorted,
                                                      int64_t* size, BuildCounts* bc) {
    const int v = blockIdx.x * BLOCK + threadIdx.x;
    if (v >= n) return;
    const int len = end[v] - first[v];
    if (len > CUT_LONG) bc->long_rows = 1;
    const long long sl = ((long long)len * slack_pct + 99) / 100;
    row_len[v] = len;
    row_sorted[v] = len;
    size[v] = len + (sl < slack_min ? slack_min : sl);
}

__global__ void __launch_bounds__(BLOCK) k_build_row_ptr(int n, const int64_t* start, int32_t* row_ptr) {
    const int v = blockIdx.x * BLOCK + threadIdx.x;
    if (v <= n) row_ptr[v] = (int32_t)start[v];
}

// free slots: {own row, 0}, unlinked (eight lanes per row)
__global__ void __launch_bounds__(BLOCK) k_build_slack(int n, const int32_t* row_ptr, const int32_t* row_len,
                                                       SlotArrays a) {
    const int64_t stride = (int64_t)gridDim.x * BLOCK;
    for (int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x; t < 8 * (int64_t)n; t += stride) {
        const int v = (int)(t / 8);
        strided((int64_t)row_ptr[v] + row_len[v] + t % 8, row_ptr[v + 1], 8, [&](int j) {
            a.cr[j] = make_int2(v, 0);
            a.rev[j] = -1;
            a.cap[j] = 0;
            a.capsum[j] = 0;
        });
    }
}

// entry e into its slot, linked to its reverse (always there)
__global__ void __launch_bounds__(BLOCK) k_build_slots(int64_t entries, int bits, const unsigned long long* mkey,
                                                       const unsigned long long* sum, const int32_t* first,
                                                       const int32_t* end, const int32_t* row_ptr, SlotArrays a,
                                                       BuildCounts* bc) {
    __shared__ long long s_part[WAVES];
    const int64_t e = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    const unsigned long long low = (1ull << bits) - 1;
    int has = 0;
    if (e < entries) {
        const unsigned long long k = mkey[e];
        const int u = (int)(k >> bits), v = (int)(k & low);
        const unsigned long long back = (unsigned long long)(unsigned)v << bits | (unsigned)u;
        const int lo = first_at_least(mkey, first[v], end[v], back);
        const int j = row_ptr[u] + (int)(e - first[u]), jr = row_ptr[v] + (lo - first[v]);
        const unsigned long long c = sum[e], both = c + sum[lo];
        if (both > (unsigned long long)INT_MAX) bc->overflow = 1;
        a.cr[j] = make_int2(v, (int)c);
        a.rev[j] = jr;
        a.cap[j] = (int)c;
        a.capsum[j] = (int)both;
        has = c > 0;
    }
    long long total;
    block_excl(has, s_part, &total);
    if (threadIdx.x == 0 && total) atomicAdd(&bc->with_capacity, (unsigned long long)total);
}

// What a handle holds, about: the slot arrays and the idle winner (24 bytes a
// slot); excess, heights, lists and queues (a vertex); the mid-size levels'
// segments and the counters.
constexpr size_t HANDLE_SLOT_BYTES = 24, HANDLE_VERTEX_BYTES = 96, HANDLE_BYTES = 64u << 20;

unsigned blocks_for(int64_t items, int per) { return (unsigned)std::max<int64_t>(1, (items + per - 1) / per); }

// Pieces of one allocation.
struct Arena {
    char* base = nullptr;
    size_t used = 0;
    template <class T>
    T* take(int64_t count) {
        T* p = reinterpret_cast<T*>(base + used);
        used += (sizeof(T) * (size_t)count + 255) & ~(size_t)255;
        return p;
    }
};

}  // namespace

mf_status build_bicsr_device(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, const int32_t* cap,
                             int32_t slack_min, int32_t slack_pct, hipStream_t st, const DeviceAllocator& mem,
                             DeviceBiCSR* out, bool* no_room) {
    *no_room = false;
    const int64_t count = 2 * m;
    int bits = 1;
    while ((1ll << bits) < n) ++bits;
    const int tiles = (int)blocks_for(count, TILE);
    Arena a;
    auto carve = [&](Arena& ar, int32_t** in, unsigned long long** key, int32_t** val, unsigned** hist, unsigned** totals,
                     unsigned long long** sum, int32_t** first, int32_t** end, int64_t** size, int64_t** start,
                     int64_t** tile, long long** mtile, BuildCounts** bc) {
        for (int i = 0; i < 2; ++i) key[i] = ar.take<unsigned long long>(count);
        for (int i = 0; i < 2; ++i) val[i] = ar.take<int32_t>(count);
        *in = ar.take<int32_t>(3 * m);
        *hist = ar.take<unsigned>((int64_t)DIGITS * tiles);
        *totals = ar.take<unsigned>(DIGITS);
        *sum = ar.take<unsigned long long>(count);
        *first = ar.take<int32_t>(n);
        *end = ar.take<int32_t>(n);
        *size = ar.take<int64_t>(n);
        *start = ar.take<int64_t>((int64_t)n + 1);
        *tile = ar.take<int64_t>(relayout_tiles(n));
        *mtile = ar.take<long long>(tiles);
        *bc = ar.take<BuildCounts>(1);
    };
    int32_t *in, *val[2], *first, *end;
    unsigned long long *key[2], *sum;
    unsigned *hist, *totals;
    int64_t *size, *start, *tile;
    long long* mtile;
    BuildCounts* bc;
    carve(a, &in, key, val, &hist, &totals, &sum, &first, &end, &size, &start, &tile, &mtile, &bc);  // sizes only
    // Scratch of this call only, not the handle's: from the device itself, so
    // that an allocator sized for the handle's buffers still suffices.  The
    // slot arrays are allocated beside it, so it is taken only where it and
    // the whole handle fit in half of the free memory (the other half is for
    // what other threads load and repair meanwhile); elsewhere the host
    // builder needs none.  (The query takes 5 us.)
    const int64_t most_slots = std::min<int64_t>(count + n + (int64_t)n * slack_min + count / 100 * slack_pct, INT_MAX);
    const size_t handle = HANDLE_SLOT_BYTES * (size_t)most_slots + HANDLE_VERTEX_BYTES * (size_t)n + HANDLE_BYTES;
    size_t free_bytes = 0, total_bytes = 0;
    void* block = nullptr;
    if (hipMemGetInfo(&free_bytes, &total_bytes) != hipSuccess || a.used + handle > free_bytes / 2 ||
        hipMallocAsync(&block, a.used, st) != hipSuccess) {
        (void)hipGetLastError();
        *no_room = true;
        return MF_ERR_OUT_OF_MEMORY;
    }
    a = Arena{(char*)block, 0};
    carve(a, &in, key, val, &hist, &totals, &sum, &first, &end, &size, &start, &tile, &mtile, &bc);
    // given back in the stream's order (hipFree would wait for the whole
    // device: a load beside a 125 ms kernel of another stream took 125 ms,
    // 4 ms this way); the wait behind it lets the pool return it to the device
    struct Release {
        void* p;
        hipStream_t st;
        void give_back() {
            if (p) (void)hipFreeAsync(p, st);
            p = nullptr;
        }
        ~Release() {
            if (!p) return;
            give_back();
            (void)hipStreamSynchronize(st);
        }
    } release{block, st};
#define BUILD_HIP(call) \
    do {                \
        if ((call) != hipSuccess) return MF_ERR_DEVICE; \
    } while (0)
    BUILD_HIP(hipMemcpyAsync(in, src, 4 * (size_t)m, hipMemcpyHostToDevice, st));
    BUILD_HIP(hipMemcpyAsync(in + m, dst, 4 * (size_t)m, hipMemcpyHostToDevice, st));
    BUILD_HIP(hipMemcpyAsync(in + 2 * m, cap, 4 * (size_t)m, hipMemcpyHostToDevice, st));
    launch_fill_i32(reinterpret_cast<int32_t*>(bc), 0, sizeof(BuildCounts) / 4, st);
    launch_fill_i32(reinterpret_cast<int32_t*>(sum), 0, 2 * count, st);
    launch_fill_i32(first, 0, n, st);
    launch_fill_i32(end, 0, n, st);
    k_build_expand<<<blocks_for(m, BLOCK), BLOCK, 0, st>>>(n, m, in, in + m, in + 2 * m, bits, key[0], val[0], bc);
    int cur = 0;
    for (int shift = 0; shift < 2 * bits; shift += 8, cur ^= 1) {
        k_sort_hist<<<tiles, BLOCK, 0, st>>>(key[cur], count, shift, hist, tiles);
        k_sort_scan<<<DIGITS, BLOCK, 0, st>>>(hist, tiles, totals);
        k_sort_scatter<<<tiles, BLOCK, 0, st>>>(key[cur], val[cur], key[cur ^ 1], val[cur ^ 1], count, shift, hist,
                                                tiles, totals);
    }
    unsigned long long* mkey = key[cur ^ 1];
    k_merge_count<<<tiles, BLOCK, 0, st>>>(key[cur], count, mtile);
    k_merge_scan<<<1, BLOCK, 0, st>>>(mtile, tiles, bc);
    k_merge<<<tiles, BLOCK, 0, st>>>(key[cur], val[cur], count, mtile, bits, mkey, sum, first, end);
    k_build_rows<<<blocks_for(n, BLOCK), BLOCK, 0, st>>>(n, first, end, slack_min, slack_pct, out->row_len,
                                                         out->row_sorted, size, bc);
    launch_scan_sizes(n, size, start, tile, st);
    BUILD_HIP(hipGetLastError());
    int64_t S = 0;
    BuildCounts c{};
    BUILD_HIP(hipMemcpyAsync(&S, start + n, sizeof(S), hipMemcpyDeviceToHost, st));
    BUILD_HIP(hipMemcpyAsync(&c, bc, sizeof(c), hipMemcpyDeviceToHost, st));
    BUILD_HIP(hipStreamSynchronize(st));
    if (c.invalid) return MF_ERR_INVALID;
    if (S > INT_MAX) return MF_ERR_OVERFLOW;
    if (mem.allocate((void**)&out->a.cr, sizeof(int2) * (size_t)S) != hipSuccess ||
        mem.allocate((void**)&out->a.rev, 4 * (size_t)S) != hipSuccess ||
        mem.allocate((void**)&out->a.cap, 4 * (size_t)S) != hipSuccess ||
        mem.allocate((void**)&out->a.capsum, 4 * (size_t)S) != hipSuccess) {
        // (another thread took the room meanwhile: once more without the
        // scratch; a caller's allocator that refuses is taken at its word)
        *no_room = !mem.alloc_fn;
        return MF_ERR_OUT_OF_MEMORY;
    }
    k_build_row_ptr<<<blocks_for((int64_t)n + 1, BLOCK), BLOCK, 0, st>>>(n, start, out->row_ptr);
    k_build_slack<<<stride_blocks(8 * (int64_t)n, BLOCK), BLOCK, 0, st>>>(n, out->row_ptr, out->row_len, out->a);
    k_build_slots<<<blocks_for(c.entries, BLOCK), BLOCK, 0, st>>>(c.entries, bits, mkey, sum, first, end,
                                                                  out->row_ptr, out->a, bc);
    BUILD_HIP(hipGetLastError());
    BUILD_HIP(hipMemcpyAsync(&c, bc, sizeof(c), hipMemcpyDeviceToHost, st));
    release.give_back();  // (behind the copy; one wait for both)
    BUILD_HIP(hipStreamSynchronize(st));
    if (c.overflow) return MF_ERR_OVERFLOW;
    out->slots = S;
    out->pairs = c.entries;
    out->m_unique = (int64_t)c.with_capacity;
    out->long_rows = c.long_rows != 0;
    return MF_OK;
#undef BUILD_HIP
}

}  // namespace mf
