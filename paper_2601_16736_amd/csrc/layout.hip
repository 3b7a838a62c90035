// Spatial ordering of primitives (Morton / Z-order of the means) and row
// gather, used to lay a scene out so that the primitives one view sees sit in
// long contiguous index runs.
#include <algorithm>
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include "internal.h"
#include "trace.h"

namespace gs {

gs_status set_error(gs_status s, const char* msg);
void clear_error();

namespace {

constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// order-preserving map of FP32 onto uint32 (for atomic min/max)
__device__ __forceinline__ uint32_t f2ord(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float ord2f(uint32_t o)
{
    const uint32_t u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    return __uint_as_float(u);
}

// The union of the boxes of a block of 64 * Waves threads, left in every thread.
template <int Waves>
__device__ __forceinline__ void join_boxes(uint32_t (&lo)[3], uint32_t (&hi)[3])
{
    __shared__ uint32_t s_box[Waves][6];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int off = 32; off > 0; off >>= 1) {
            lo[a] = min(lo[a], (uint32_t)__shfl_xor((int)lo[a], off));
            hi[a] = max(hi[a], (uint32_t)__shfl_xor((int)hi[a], off));
        }
        if (threadIdx.x % 64 == 0) {
            s_box[threadIdx.x / 64][a] = lo[a];
            s_box[threadIdx.x / 64][3 + a] = hi[a];
        }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int w = 0; w < Waves; ++w) {
            lo[a] = min(lo[a], s_box[w][a]);
            hi[a] = max(hi[a], s_box[w][3 + a]);
        }
    }
}

// Bounding box of the means, one per block; the Morton kernel joins them.
constexpr int kBoxBlocks = 256, kBoxThreads = 1024;

__global__ __launch_bounds__(kBoxThreads) void bbox_kernel(const float* __restrict__ means, int64_t ms, int64_t n,
                                                           uint32_t* __restrict__ boxes)
{
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float x = means[ms * i + a];
            if (x == x) {                      // NaN means take no part in the box
                const uint32_t o = f2ord(x);
                lo[a] = min(lo[a], o);
                hi[a] = max(hi[a], o);
            }
        }
    }
    join_boxes<kBoxThreads / 64>(lo, hi);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            boxes[blockIdx.x * 6 + a] = lo[a];
            boxes[blockIdx.x * 6 + 3 + a] = hi[a];
        }
    }
}

// 10 bits spread to every third bit position
__device__ __forceinline__ uint32_t spread3(uint32_t x)
{
    x &= 0x3FFu;
    x = (x | (x << 16)) & 0x030000FFu;
    x = (x | (x << 8)) & 0x0300F00Fu;
    x = (x | (x << 4)) & 0x030C30C3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

// The order is a stable radix sort of the 30-bit codes, three passes of ten
// bits.  Each pass counts the digits of every tile (the first pass while it
// makes the codes), turns the counts into places, and moves (code, index)
// pairs there; the last pass writes indices alone.  The arrays are small (a
// pass over 1M pairs moves 20 MB, 4 us), so launches and the latency inside
// each set the time: ten bits rather than eight save three launches, and no
// tile waits for another one.  Runs of a digit in a tile are short (four pairs),
// which the L2 caches join.  1M primitives: 70 us, with the library's sort 184;
// 3M: 120 against 195; 200k: 53 against 81.
constexpr int kDigitBits = 10;
constexpr int kDigits = 1 << kDigitBits;
constexpr int kTileRounds = 8;
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kTile = kTileThreads * kTileRounds;      // each wave on kTileRounds * 64 places in a row

__device__ __forceinline__ int tile_place(int u)
{
    return (threadIdx.x / 64) * (kTileRounds * 64) + u * 64 + threadIdx.x % 64;
}

// Adds the tile's digits up in LDS and writes them as row blockIdx.x of counts.
struct DigitCounter {
    uint32_t* s_count;
    __device__ void clear() const
    {
#pragma unroll
        for (int k = threadIdx.x; k < kDigits; k += kTileThreads) s_count[k] = 0u;
        __syncthreads();
    }
    __device__ void add(uint32_t digit) const { atomicAdd(&s_count[digit], 1u); }
    __device__ void write(uint32_t* counts) const
    {
        __syncthreads();
#pragma unroll
        for (int k = threadIdx.x; k < kDigits; k += kTileThreads)
            counts[(int64_t)blockIdx.x * kDigits + k] = s_count[k];
    }
};

template <bool Count>
__global__ __launch_bounds__(kTileThreads) void morton_kernel(const float* __restrict__ means, int64_t ms, int64_t n,
                                                     const uint32_t* __restrict__ boxes, int n_boxes, uint32_t* __restrict__ keys,
                                                     uint32_t* __restrict__ counts)
{
    __shared__ uint32_t s_count[kDigits];
    const DigitCounter counter{s_count};
    uint32_t blo[3], bhi[3];
    static_assert(kTileThreads >= kBoxBlocks, "each thread joins one block's box");
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        blo[a] = boxes[threadIdx.x % n_boxes * 6 + a];
        bhi[a] = boxes[threadIdx.x % n_boxes * 6 + 3 + a];
    }
    if (Count) counter.clear();
    join_boxes<kTileWaves>(blo, bhi);
    float lo[3], scale[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = ord2f(blo[a]);
        const float ext = ord2f(bhi[a]) - lo[a];
        scale[a] = ext > 0.0f ? 1024.0f / ext : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < (Count ? kTileRounds : 1); ++u) {
        const int64_t i = Count ? (int64_t)blockIdx.x * kTile + tile_place(u)
                                : (int64_t)blockIdx.x * kTileThreads + threadIdx.x;
        if (i >= n) continue;
        uint32_t q[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float t = (means[ms * i + a] - lo[a]) * scale[a];
            q[a] = t >= 0.0f ? (uint32_t)min(t, 1023.0f) : 0u;        // NaN -> 0
        }
        const uint32_t key = spread3(q[0]) | (spread3(q[1]) << 1) | (spread3(q[2]) << 2);
        keys[i] = key;
        if (Count) counter.add(key % kDigits);
    }
    if (Count) counter.write(counts);
}

__global__ __launch_bounds__(kTileThreads) void count_digits_kernel(const uint2* __restrict__ pairs, int64_t n, int shift,
                                                           uint32_t* __restrict__ counts)
{
    __shared__ uint32_t s_count[kDigits];
    const DigitCounter counter{s_count};
    counter.clear();
#pragma unroll
    for (int u = 0; u < kTileRounds; ++u) {
        const int64_t i = (int64_t)blockIdx.x * kTile + tile_place(u);
        if (i < n) counter.add((pairs[i].x >> shift) % kDigits);
    }
    counter.write(counts);
}

// counts[t][d] becomes the sum over the tiles before t, totals[d] the sum over
// all of them.  A block takes kScanDigits digits; its 1024 threads are so many
// columns of the table, split in runs of tiles.
constexpr int kScanDigits = 16;
constexpr int kScanRuns = 1024 / kScanDigits;

__global__ __launch_bounds__(1024) void scan_tiles_kernel(uint32_t* __restrict__ counts, int64_t tiles,
                                                          uint32_t* __restrict__ totals)
{
    __shared__ uint32_t s_run[kScanRuns][kScanDigits];
    const int d = blockIdx.x * kScanDigits + threadIdx.x % kScanDigits;
    const int run = threadIdx.x / kScanDigits;
    const int64_t per = (tiles + kScanRuns - 1) / kScanRuns;
    const int64_t t0 = min(run * per, tiles), t1 = min(t0 + per, tiles);
    uint32_t sum = 0u;
#pragma unroll 8
    for (int64_t t = t0; t < t1; ++t) sum += counts[t * kDigits + d];
    s_run[run][threadIdx.x % kScanDigits] = sum;
    __syncthreads();
    // inclusive sums over the runs, in log2 steps
    for (int off = 1; off < kScanRuns; off *= 2) {
        const uint32_t add = run >= off ? s_run[run - off][threadIdx.x % kScanDigits] : 0u;
        __syncthreads();
        s_run[run][threadIdx.x % kScanDigits] += add;
        __syncthreads();
    }
    uint32_t before = s_run[run][threadIdx.x % kScanDigits] - sum;
    if (run == kScanRuns - 1) totals[d] = before + sum;
#pragma unroll 8
    for (int64_t t = t0; t < t1; ++t) {
        const uint32_t c = counts[t * kDigits + d];
        counts[t * kDigits + d] = before;
        before += c;
    }
}

// Sum over the threads before this one, of all 512.
__device__ __forceinline__ uint32_t sum_before(uint32_t own, uint32_t (&s_sum)[kTileWaves])
{
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    uint32_t upto = own;
#pragma unroll
    for (int off = 1; off < 64; off *= 2) {
        const uint32_t x = (uint32_t)__shfl_up((int)upto, off);
        if (lane >= off) upto += x;
    }
    if (lane == 63) s_sum[wave] = upto;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) upto += w < wave ? s_sum[w] : 0u;
    return upto - own;
}

// Moves a tile's pairs to their places.  A wave ranks its places 64 at a time:
// ten ballots find the lanes with a lane's digit, and the wave's own table in
// LDS how many came before.  The pairs go through LDS in the order of their
// digits, so that a run's writes leave together (3M pairs: 21 us, written from
// the registers 35 us).  Eight rounds by eight waves rather than sixteen by
// four: the rounds are a serial chain (200k pairs: 8.5 against 10.4 us).
// First: keys alone, the index is the place.  Last: indices alone are written.
template <bool First, bool Last>
__global__ __launch_bounds__(kTileThreads) void move_pairs_kernel(const void* __restrict__ in, void* __restrict__ out,
                                                                  int64_t n, int shift,
                                                                  const uint32_t* __restrict__ counts,
                                                                  const uint32_t* __restrict__ totals)
{
    __shared__ uint16_t s_rank[kTileWaves][kDigits];
    __shared__ uint32_t s_shift[kDigits];          // from a digit's place in the tile to that in the output
    __shared__ uint32_t s_total[kTileWaves], s_count[kTileWaves];
    __shared__ uint2 s_pair[kTile];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int64_t first = (int64_t)blockIdx.x * kTile;
    uint2 pair[kTileRounds];
#pragma unroll
    for (int u = 0; u < kTileRounds; ++u) {
        const int64_t i = first + tile_place(u);
        pair[u] = make_uint2(0u, 0u);
        if (i < n) pair[u] = First ? make_uint2(static_cast<const uint32_t*>(in)[i], (uint32_t)i)
                                   : static_cast<const uint2*>(in)[i];
    }
    // thread k has digits 2k and 2k + 1
    static_assert(kDigits == 2 * kTileThreads, "two digits per thread");
    const uint2 total = reinterpret_cast<const uint2*>(totals)[threadIdx.x];
    const uint2 count = reinterpret_cast<const uint2*>(counts)[(int64_t)blockIdx.x * (kDigits / 2) + threadIdx.x];
#pragma unroll
    for (int k = 0; k < kDigits / 64; ++k) s_rank[wave][k * 64 + lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();

    uint32_t rank[kTileRounds];
#pragma unroll
    for (int u = 0; u < kTileRounds; ++u) {
        const bool ok = first + tile_place(u) < n;
        const uint32_t digit = (pair[u].x >> shift) % kDigits;
        uint64_t same = __ballot(ok);
#pragma unroll
        for (int b = 0; b < kDigitBits; ++b) {
            const bool bit = (digit >> b) & 1u;
            const uint64_t set = __ballot(bit);
            same &= bit ? set : ~set;
        }
        rank[u] = s_rank[wave][digit] + __popcll(same & ((1ull << lane) - 1ull));
        // the last lane of a digit counts for all of them; the table is the wave's own
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (ok && (same >> lane) == 1ull) s_rank[wave][digit] = (uint16_t)(rank[u] + 1u);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    const uint32_t global = sum_before(total.x + total.y, s_total);       // has a barrier: the tables are whole
    uint32_t n0 = 0u, n1 = 0u;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) {
        n0 += s_rank[w][2 * threadIdx.x];
        n1 += s_rank[w][2 * threadIdx.x + 1];
    }
    uint32_t at0 = sum_before(n0 + n1, s_count), at1 = at0 + n0;
    s_shift[2 * threadIdx.x] = global + count.x - at0;
    s_shift[2 * threadIdx.x + 1] = global + total.x + count.y - at1;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) {
        const uint32_t c0 = s_rank[w][2 * threadIdx.x], c1 = s_rank[w][2 * threadIdx.x + 1];
        s_rank[w][2 * threadIdx.x] = (uint16_t)at0;
        s_rank[w][2 * threadIdx.x + 1] = (uint16_t)at1;
        at0 += c0;
        at1 += c1;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kTileRounds; ++u)
        if (first + tile_place(u) < n) s_pair[s_rank[wave][(pair[u].x >> shift) % kDigits] + rank[u]] = pair[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kTileRounds; ++u) {
        const int k = u * kTileThreads + threadIdx.x;
        if (first + k >= n) continue;
        const uint2 p = s_pair[k];
        const uint32_t at = k + s_shift[(p.x >> shift) % kDigits];
        if (Last) static_cast<uint32_t*>(out)[at] = p.y;
        else static_cast<uint2*>(out)[at] = p;
    }
}

// Row gather in chunks of T: thread k of the flattened (row, chunk) space
// moves chunk k, so consecutive lanes move consecutive chunks.  A block finds
// its first chunk's row with one 64-bit division that all lanes share; the
// lanes then divide 32-bit places.  One chunk per thread: the lines of the
// sources set the time (about 5 TB/s of whole lines), and more, shorter waves
// spread over them better than more loads in flight (eight chunks per thread
// from a row list in LDS: 151 against 86 us for 1M random rows of 180 bytes).
// Chunks of one or two bytes take four per thread, to load fewer indices.
constexpr int kGatherThreads = 256;
template <typename T> constexpr int kGatherUnroll = sizeof(T) <= 2 ? 4 : 1;

// Three words, word alignment: a 12-byte row, or a fifteenth of the 45 SH-rest
// values, in one access instead of three.  1M random rows of 180 bytes: 86 us,
// with 4-byte chunks and a 64-bit division for each 135 us; rows of 90 bytes
// in 2-byte chunks 77 us, byte by byte 134 us.
struct Chunk12 { uint32_t a, b, c; };

template <typename T>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(const T* __restrict__ src, T* __restrict__ dst,
                                                                const int32_t* __restrict__ perm, int64_t n,
                                                                uint32_t cpr, float inv)
{
    constexpr int U = kGatherUnroll<T>;
    const int64_t k0 = (int64_t)blockIdx.x * (kGatherThreads * U);
    const int64_t row0 = k0 / cpr;
    const uint32_t c0 = (uint32_t)(k0 - row0 * cpr);
    const int64_t total = n * cpr;
    T x[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t k = c0 + u * kGatherThreads + threadIdx.x;
        // k / cpr: exact but for one, which the next lines mend
        uint32_t r = (uint32_t)((float)k * inv);
        int32_t c = (int32_t)(k - r * cpr);
        if (c < 0) { c += (int32_t)cpr; --r; }
        if (c >= (int32_t)cpr) { c -= (int32_t)cpr; ++r; }
        ok[u] = k0 + u * kGatherThreads + threadIdx.x < total;
        const int32_t p = ok[u] ? perm[row0 + r] : -1;
        ok[u] = (uint32_t)p < (uint64_t)n;                  // out-of-range entries are skipped
        if (ok[u]) x[u] = src[(int64_t)p * cpr + c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (ok[u]) dst[k0 + u * kGatherThreads + threadIdx.x] = x[u];
}

// Threads stride over the chunks, with a 64-bit division for each: for rows
// too long or chunks too many for one dispatch of the kernel above, and for
// 16-byte chunks, where the division hides behind the loads (1M random rows of
// 192 bytes: 72 us, above 76 us).
template <typename T>
__global__ __launch_bounds__(kGatherThreads) void gather_strided_kernel(const T* __restrict__ src, T* __restrict__ dst,
                                                                        const int32_t* __restrict__ perm, int64_t n,
                                                                        int64_t cpr)
{
    const int64_t total = n * cpr;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = k / cpr;
        const int32_t p = perm[i];
        if ((uint32_t)p < (uint64_t)n) dst[k] = src[(int64_t)p * cpr + (k - i * cpr)];
    }
}

template <typename T>
void launch_gather(const void* src, void* dst, const int32_t* perm, int64_t n, int64_t row_bytes, hipStream_t stream)
{
    const int64_t cpr = row_bytes / (int64_t)sizeof(T);
    if constexpr (sizeof(T) < 16) {
        // places in a row and a block are exact in FP32 below 2^24
        const int64_t per = kGatherThreads * kGatherUnroll<T>;
        if (cpr <= (int64_t)1 << 22 && cpr <= kMaxGridBlocks * per / n) {
            const unsigned blocks = (unsigned)((n * cpr + per - 1) / per);
            hipLaunchKernelGGL(gather_kernel<T>, dim3(blocks), dim3(kGatherThreads), 0, stream, (const T*)src, (T*)dst,
                               perm, n, (uint32_t)cpr, 1.0f / (float)cpr);
            return;
        }
    }
    hipLaunchKernelGGL(gather_strided_kernel<T>, dim3(8192), dim3(kGatherThreads), 0, stream, (const T*)src, (T*)dst,
                       perm, n, cpr);
}

// Below this many primitives ten launches take longer than the library's sort,
// which takes fewer the fewer there are: the order of 20,000 takes 43 us with
// it, 49 without; of 60,000 47.5 and 50.5; of 200,000 81 and 53.
constexpr int64_t kOwnSortMin = 65536;

size_t small_sort_bytes(int64_t n)
{
    size_t bytes = 0;
    (void)rocprim::radix_sort_pairs(nullptr, bytes, (const uint32_t*)nullptr, (uint32_t*)nullptr,
                                    rocprim::counting_iterator<int32_t>(0), (int32_t*)nullptr, (size_t)n, 0, 30);
    return bytes;
}

// The parts of the workspace.  The keys lie where the second pass puts its
// pairs, or the library's sort its keys' copy: they are read by then.  The boxes
// lie where the first pass or that sort writes first.
struct OrderSpace {
    bool own;
    int boxes_n;
    int64_t tiles;
    size_t totals, counts, keys, pairs, bytes;
    explicit OrderSpace(int64_t n)
    {
        own = n >= kOwnSortMin;
        boxes_n = (int)std::min<int64_t>((n + kBoxThreads - 1) / kBoxThreads, kBoxBlocks);
        tiles = (n + kTile - 1) / kTile;
        totals = counts = keys = pairs = bytes = 0;
        if (own) {
            counts = align_up(kDigits * 4);
            keys = counts + align_up((size_t)tiles * kDigits * 4);
            pairs = keys + align_up((size_t)n * 8);
            bytes = pairs + align_up((size_t)n * 8);
        } else {
            keys = 0;
            pairs = align_up((size_t)n * 4);
            counts = 2 * align_up((size_t)n * 4);       // the sort's own
            bytes = counts + align_up(small_sort_bytes(n));
        }
    }
};

}  // namespace

}  // namespace gs

using namespace gs;

extern "C" size_t gs_spatial_order_workspace_size(int64_t n)
{
    if (n < 0) return 0;
    return OrderSpace(n).bytes;
}

extern "C" gs_status gs_spatial_order(const float* means, int64_t means_stride, int64_t n, int32_t* perm,
                                      void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    clear_error();
    if (n < 0 || n >= ((int64_t)1 << 31)) return set_error(GS_EINVAL, "gs_spatial_order: n must be in [0, 2^31)");
    const int64_t ms = means_stride == 0 ? 3 : means_stride;
    if (ms < 3 || ms > 65536 || ms * n >= ((int64_t)1 << 40))
        return set_error(GS_EINVAL, "gs_spatial_order: means_stride must be 0 or in [3, 65536]");
    if (n == 0) return GS_OK;
    if (means == nullptr || perm == nullptr || workspace == nullptr)
        return set_error(GS_EINVAL, "gs_spatial_order: means, perm and workspace are required");
    if ((uintptr_t)means % 4 || (uintptr_t)perm % 4 || (uintptr_t)workspace % kAlign)
        return set_error(GS_EINVAL, "gs_spatial_order: misaligned pointer (workspace needs 256 bytes)");
    if (workspace_bytes < gs_spatial_order_workspace_size(n))
        return set_error(GS_EINVAL, "gs_spatial_order: workspace too small");
    char* ws = static_cast<char*>(workspace);
    const OrderSpace at(n);
    uint32_t* keys = reinterpret_cast<uint32_t*>(ws + at.keys);
    uint32_t* boxes = reinterpret_cast<uint32_t*>(ws + at.pairs);
    void* pairs = ws + at.pairs;
    const dim3 tiles((unsigned)at.tiles), block(kTileThreads), scans(kDigits / kScanDigits), scan_block(1024);
    hipLaunchKernelGGL(bbox_kernel, dim3(at.boxes_n), dim3(kBoxThreads), 0, stream, means, ms, n, boxes);
    if (!at.own) {
        hipLaunchKernelGGL(morton_kernel<false>, dim3((unsigned)((n + kTileThreads - 1) / kTileThreads)), block, 0,
                           stream, means, ms, n, boxes, at.boxes_n, keys, nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return set_error(GS_EHIP, hipGetErrorString(e));
        size_t bytes = small_sort_bytes(n);
        e = rocprim::radix_sort_pairs(ws + at.counts, bytes, (const uint32_t*)keys, (uint32_t*)pairs,
                                      rocprim::counting_iterator<int32_t>(0), perm, (size_t)n, 0, 30, stream);
        return e == hipSuccess ? GS_OK : set_error(GS_EHIP, hipGetErrorString(e));
    }
    uint32_t* totals = reinterpret_cast<uint32_t*>(ws + at.totals);
    uint32_t* counts = reinterpret_cast<uint32_t*>(ws + at.counts);
    hipLaunchKernelGGL(morton_kernel<true>, tiles, block, 0, stream, means, ms, n, boxes, at.boxes_n, keys, counts);
    hipLaunchKernelGGL(scan_tiles_kernel, scans, scan_block, 0, stream, counts, at.tiles, totals);
    hipLaunchKernelGGL((move_pairs_kernel<true, false>), tiles, block, 0, stream, keys, pairs, n, 0, counts, totals);
    hipLaunchKernelGGL(count_digits_kernel, tiles, block, 0, stream, (const uint2*)pairs, n, kDigitBits, counts);
    hipLaunchKernelGGL(scan_tiles_kernel, scans, scan_block, 0, stream, counts, at.tiles, totals);
    hipLaunchKernelGGL((move_pairs_kernel<false, false>), tiles, block, 0, stream, pairs, keys, n, kDigitBits, counts,
                       totals);
    hipLaunchKernelGGL(count_digits_kernel, tiles, block, 0, stream, (const uint2*)keys, n, 2 * kDigitBits, counts);
    hipLaunchKernelGGL(scan_tiles_kernel, scans, scan_block, 0, stream, counts, at.tiles, totals);
    hipLaunchKernelGGL((move_pairs_kernel<false, true>), tiles, block, 0, stream, keys, perm, n, 2 * kDigitBits,
                       counts, totals);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GS_OK : set_error(GS_EHIP, hipGetErrorString(e));
}

extern "C" gs_status gs_gather_rows(const void* src, void* dst, const int32_t* perm, int64_t n, int64_t row_bytes,
                                    hipStream_t stream)
{
    clear_error();
    if (n < 0 || n >= ((int64_t)1 << 31) || row_bytes < 1)
        return set_error(GS_EINVAL, "gs_gather_rows: bad n or row_bytes");
    if (n == 0) return GS_OK;
    if (src == nullptr || dst == nullptr || perm == nullptr)
        return set_error(GS_EINVAL, "gs_gather_rows: NULL pointer");
    if (src == dst) return set_error(GS_EINVAL, "gs_gather_rows: src and dst must differ");
    // the widest chunk that the row length and both arrays allow
    const uintptr_t align = (uintptr_t)src | (uintptr_t)dst | (uintptr_t)row_bytes;
    if (align % 16 == 0) launch_gather<uint4>(src, dst, perm, n, row_bytes, stream);
    else if (align % 8 == 0) launch_gather<uint2>(src, dst, perm, n, row_bytes, stream);
    else if (align % 4 == 0 && row_bytes % 12 == 0) launch_gather<Chunk12>(src, dst, perm, n, row_bytes, stream);
    else if (align % 4 == 0) launch_gather<uint32_t>(src, dst, perm, n, row_bytes, stream);
    else if (align % 2 == 0) launch_gather<uint16_t>(src, dst, perm, n, row_bytes, stream);
    else launch_gather<uint8_t>(src, dst, perm, n, row_bytes, stream);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GS_OK : set_error(GS_EHIP, hipGetErrorString(e));
}
