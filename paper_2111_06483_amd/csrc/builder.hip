// Partition-block builder: worker p's P destination-major CSR blocks
// G_{p,q} (Sec. 3.2 of the paper), plus the derived indexes the aggregation
// kernels launch from: the source-major transpose of every block, degree-class
// ordered row lists, the sorted touched-source list and the all-blocks row
// index.  Integer work only.  Every array is bit-exact and independent of
// scheduling: rows are filled through atomic cursors and then sorted, and the
// launch lists hold the rows of a degree class in their own order.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <map>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "global_ptr.h"
#include "sar_internal.h"

namespace sar {

static thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

}  // namespace sar

extern "C" const char* sar_last_error(void) { return sar::g_err; }
extern "C" int sar_version(void) { return 5; }

namespace {

using sar::Block;

constexpr int kThreads = 256;
constexpr int kScanTile = 2048;   // 256 threads x 8 values
constexpr int kPartTile = 1024;   // nodes per workgroup when ranking nodes in partitions
constexpr int kLdsSort = 8192;    // longer rows up to this length are sorted in LDS

// ---------------------------------------------------------------- scan

__device__ inline int block_exclusive_scan(int v, int* lds4, int* total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) lds4[w] = incl;
    __syncthreads();
    int woff = 0;
    for (int k = 0; k < w; ++k) woff += lds4[k];
    *total = lds4[0] + lds4[1] + lds4[2] + lds4[3];
    __syncthreads();
    return woff + incl - v;
}

// The eight values of a thread, in 16-byte pieces where they are whole (arrays start at a multiple of 16 bytes or pass ALIGNED = false).
template <bool ALIGNED>
__device__ inline int load_eight(const int32_t* in, int64_t base, int64_t n, int (&v)[8])
{
    if (ALIGNED && base + 8 <= n) {
        const int4 a = *reinterpret_cast<const int4*>(in + base), b = *reinterpret_cast<const int4*>(in + base + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = (base + k < n) ? in[base + k] : 0;
    }
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

template <bool ALIGNED>
__global__ __launch_bounds__(kThreads) void k_tile_reduce(const int32_t* __restrict__ in, int64_t n,
                                                          int32_t* __restrict__ tile_sums)
{
    __shared__ int lds4[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
    int v[8], total;
    block_exclusive_scan(load_eight<ALIGNED>(in, base, n, v), lds4, &total);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

// What stands before this workgroup's tile: `before` tiles of it added up here (SUMS: tile_sums holds the tiles' own sums) or
// read (their prefix sums).
template <bool ALIGNED, bool SUMS>
__global__ __launch_bounds__(kThreads) void k_tile_scan(const int32_t* in, int64_t n,
                                                        const int32_t* __restrict__ tile_sums,
                                                        int32_t first, int32_t* out)
{
    __shared__ int lds4[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
    int v[8], total, before = 0;
    const int s = load_eight<ALIGNED>(in, base, n, v);
    if constexpr (SUMS) {
        int part = 0;
        for (int k = threadIdx.x; k < (int)blockIdx.x; k += kThreads) part += tile_sums[k];
        block_exclusive_scan(part, lds4, &before);
    } else if (tile_sums) {
        before = tile_sums[blockIdx.x];
    }
    int run = block_exclusive_scan(s, lds4, &total) + before + first;
    int w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        w[k] = run;
        run += v[k];
    }
    if (ALIGNED && base + 8 <= n) {
        *reinterpret_cast<int4*>(out + base) = make_int4(w[0], w[1], w[2], w[3]);
        *reinterpret_cast<int4*>(out + base + 4) = make_int4(w[4], w[5], w[6], w[7]);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (base + k < n) out[base + k] = w[k];
    }
}

// Device memory of handles and of builder calls.  A handle is some ten arrays of a few to a few
// hundred MB, and a program that rebuilds its handles (a graph that changes, restricted handles batch
// by batch) would pay the driver for mapping and clearing them every time: up to 20 ms of a 25 ms
// call where much memory had been freed before.  What a builder call or sar_blocks_free gives up is
// therefore kept for the next call, at most kPoolMost bytes per device and nothing larger than a
// quarter of that, and all of it is given back when the last handle on the device is freed, when an
// allocation made here fails, or by sar_release_memory.  Nothing enters the pool before the work that used it
// is done.
class Pool {
public:
    static constexpr size_t kPoolMost = (size_t)1 << 30;
    static size_t round(size_t bytes)
    {
        size_t unit = 4096;
        while (unit * 16 < bytes) unit *= 2;         // at most an eighth more than asked for
        return (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
    }
    int take(int dev, void** out, size_t size)       // dev: the current device; size as round() gives it
    {
        const hipError_t e = try_take(dev, out, size);
        return e == hipSuccess ? SAR_OK
                               : sar::fail(SAR_ERR_HIP, "hipMalloc of %zu bytes failed: %s", size, hipGetErrorString(e));
    }
    hipError_t try_take(int dev, void** out, size_t size)      // no error is left behind, here or with the runtime
    {
        std::lock_guard<std::mutex> lock(m_);
        auto& d = devices_[dev];
        auto it = d.idle.lower_bound(size);
        if (it != d.idle.end() && it->first == size) {
            *out = it->second;
            d.bytes -= it->first;
            d.idle.erase(it);
            return hipSuccess;
        }
        hipError_t e = hipMalloc(out, size);
        if (e == hipSuccess) return e;
        (void)hipGetLastError();
        release(d);
        e = hipMalloc(out, size);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }
    void give(int dev, void* p, size_t size)         // memory of `dev` that nothing in flight uses any more
    {
        if (size <= kPoolMost / 4) {
            std::lock_guard<std::mutex> lock(m_);
            auto& d = devices_[dev];
            if (d.bytes + size <= kPoolMost) {
                try {
                    d.idle.emplace(size, p);
                    d.bytes += size;
                    return;
                } catch (const std::bad_alloc&) {   // no host memory for the entry: not kept
                }
            }
        }
        (void)hipFree(p);
    }
    // Whether memory of that size is kept once the builder call that uses it gives it up, and not handed to the driver then or
    // with the call's own handle.
    bool keeps(int dev, size_t size)
    {
        std::lock_guard<std::mutex> lock(m_);
        return size <= kPoolMost / 4 && devices_[dev].handles > 1;
    }
    // A page of pinned host memory for what a call's kernels report to the host and what it sends them: through pageable
    // memory every copy waits for the stream (15.2M edges: twelve copies, the build 1534 us and now 1431).  At most kHostPages idle ones.
    static constexpr size_t kHostPage = 192 << 10;
    static constexpr size_t kHostPages = 4;
    int take_host(void** out)
    {
        {
            std::lock_guard<std::mutex> lock(m_);
            if (!host_.empty()) {
                *out = host_.back();
                host_.pop_back();
                return SAR_OK;
            }
        }
        SAR_HIP(hipHostMalloc(out, kHostPage, hipHostMallocPortable));
        return SAR_OK;
    }
    void give_host(void* p)
    {
        {
            std::lock_guard<std::mutex> lock(m_);
            if (host_.size() < kHostPages) {
                try {
                    host_.push_back(p);
                    return;
                } catch (const std::bad_alloc&) {
                }
            }
        }
        (void)hipHostFree(p);
    }
    void count_handle(int dev, int by)
    {
        std::lock_guard<std::mutex> lock(m_);
        auto& d = devices_[dev];
        d.handles += by;
        if (d.handles > 0) return;
        release(d);
        for (auto& e : devices_)
            if (e.second.handles > 0) return;
        release_host();
    }
    void release_all()
    {
        std::lock_guard<std::mutex> lock(m_);
        for (auto& d : devices_) release(d.second);
        release_host();
    }

private:
    struct Device {
        std::multimap<size_t, void*> idle;
        size_t bytes = 0;
        int64_t handles = 0;
    };
    void release(Device& d)
    {
        for (auto& e : d.idle) (void)hipFree(e.second);
        d.idle.clear();
        d.bytes = 0;
    }
    void release_host()
    {
        for (void* p : host_) (void)hipHostFree(p);
        host_.clear();
    }
    std::mutex m_;
    std::map<int, Device> devices_;
    std::vector<void*> host_;
};

Pool& pool()
{
    static Pool* p = new Pool();     // never destroyed: handles may be freed while the process ends
    return *p;
}

// Scratch of one builder call on one stream.
struct DeviceTemps {
    explicit DeviceTemps(hipStream_t s, int device) : st(s), dev(device) {}
    DeviceTemps(const DeviceTemps&) = delete;
    ~DeviceTemps()
    {
        drop_spare();
        if (ptrs.empty() && !page) return;
        (void)hipStreamSynchronize(st);
        for (auto& p : ptrs) pool().give(dev, p.first, p.second);
        if (page) pool().give_host(page);
    }
    // the call's page of pinned memory: what the device reports first, then `up` bytes to send
    int host(void** out, size_t up = 0)
    {
        if (!page) SAR_TRY(pool().take_host(&page));
        *out = static_cast<char*>(page) + up;
        return SAR_OK;
    }
    template <typename T>
    int alloc(T** out, int64_t count)
    {
        void* p = nullptr;
        const size_t size = Pool::round(std::max<int64_t>(count, 1) * sizeof(T));
        ptrs.reserve(ptrs.size() + 1);      // before there is anything to lose
        SAR_TRY(or_without_spare([&] { return pool().take(dev, &p, size); }));
        ptrs.emplace_back(p, size);
        *out = static_cast<T*>(p);
        return SAR_OK;
    }
    // Several arrays as one piece, where the pool keeps pieces of that size.  A program that frees its only handle gives
    // every piece back to the driver, 240 us each once the few ten MB that the runtime holds on to are full (2.4 million nodes, 8
    // million edges of which an eighth is kept, built and freed: 7.8 ms with a piece for every array, 6.8 with these).
    struct Part {
        void** out;
        size_t bytes;
    };
    int alloc_parts(std::initializer_list<Part> parts)
    {
        size_t total = 0;
        for (const Part& x : parts) total += (x.bytes + 255) / 256 * 256;
        if (Pool::round(total) > Pool::kPoolMost / 4) {
            for (const Part& x : parts) {
                char* p = nullptr;
                SAR_TRY(alloc(&p, (int64_t)x.bytes));
                *x.out = p;
            }
            return SAR_OK;
        }
        char* p = nullptr;
        SAR_TRY(alloc(&p, (int64_t)total));
        for (const Part& x : parts) {
            *x.out = p;
            p += (x.bytes + 255) / 256 * 256;
        }
        return SAR_OK;
    }
    template <typename T>
    static Part part(T** out, int64_t count)
    {
        return {reinterpret_cast<void**>(out), (size_t)std::max<int64_t>(count, 1) * sizeof(T)};
    }
    // Scratch that the call can do without (`spare`, null where there is no room or the pool would not keep it): it makes way for
    // whatever else is asked for.
    void alloc_spare(size_t bytes)
    {
        spare_bytes = Pool::round(bytes);
        if (!pool().keeps(dev, spare_bytes) || pool().try_take(dev, &spare, spare_bytes) != hipSuccess) spare = nullptr;
    }
    void drop_spare()
    {
        if (!spare) return;
        (void)hipStreamSynchronize(st);
        pool().give(dev, spare, spare_bytes);
        spare = nullptr;
    }
    template <typename Fn>
    int or_without_spare(Fn&& take)
    {
        const int rc = take();
        if (rc == SAR_OK || !spare) return rc;
        drop_spare();
        return take();
    }
    hipStream_t st;
    int dev;
    void* page = nullptr;
    void* spare = nullptr;
    size_t spare_bytes = 0;
    std::vector<std::pair<void*, size_t>> ptrs;
};

// Up to so many tiles every workgroup adds up the sums of the tiles before its own, 16 loads a thread at most, and a scan is two
// launches; beyond that the sums are scanned by a pass of their own.  (A build of 15 million edges in 8 blocks has eight scans of up to
// 1.2 million values, bound by launches and their chains of loads: 16 launches of 6.5 us for the scans and 8 of 5.6 for the sums, now 8 of
// 5.0 and 8 of 4.2; the whole build 1340 -> 1260 us.  The scans of a build over N nodes, sums by a pass of their own / added up by every
// workgroup, us: N of 0.5 million 93 / 65, 2 million 110 / 78, 4 million (1954 tiles) 127 / 95, 8 million (3907 tiles) 204 / 135.)
constexpr int64_t kScanOnce = 4096;

// out[k] = base + sum of in[0..k) for k in [0,n); in may equal out.
int exclusive_scan(const int32_t* in, int32_t* out, int64_t n, hipStream_t st, DeviceTemps& tmp, int32_t base = 0)
{
    if (n <= 0) return SAR_OK;
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    auto with = [&](auto aligned) -> int {
        constexpr bool A = decltype(aligned)::value;
        int32_t* sums = nullptr;
        if (tiles > 1) {
            SAR_TRY(tmp.alloc(&sums, tiles));
            k_tile_reduce<A><<<(unsigned)tiles, kThreads, 0, st>>>(in, n, sums);
            SAR_LAUNCH_CHECK();
        }
        if (tiles > 1 && tiles <= kScanOnce) {
            k_tile_scan<A, true><<<(unsigned)tiles, kThreads, 0, st>>>(in, n, sums, base, out);
        } else {
            if (tiles > 1) SAR_TRY(exclusive_scan(sums, sums, tiles, st, tmp));
            k_tile_scan<A, false><<<(unsigned)tiles, kThreads, 0, st>>>(in, n, sums, base, out);
        }
        SAR_LAUNCH_CHECK();
        return SAR_OK;
    };
    return ((uintptr_t)in | (uintptr_t)out) % 16 == 0 ? with(std::true_type{}) : with(std::false_type{});
}

// ------------------------------------------------- local ids of all nodes

__global__ __launch_bounds__(kThreads) void k_part_tile_count(const int32_t* __restrict__ part,
                                                              int64_t N, int P, int64_t n_tiles,
                                                              int32_t* __restrict__ tile_counts,
                                                              int* __restrict__ err)
{
    static_assert(SAR_MAX_PARTS <= kThreads, "one thread per partition");
    __shared__ int hist[SAR_MAX_PARTS];
    if (threadIdx.x < SAR_MAX_PARTS) hist[threadIdx.x] = 0;
    __syncthreads();
    for (int r = 0; r < kPartTile / kThreads; ++r) {
        const int64_t v = (int64_t)blockIdx.x * kPartTile + r * kThreads + threadIdx.x;
        if (v < N) {
            const int pv = part[v];
            if (pv < 0 || pv >= P)
                atomicOr(err, 1);
            else
                atomicAdd(&hist[pv], 1);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < P) tile_counts[(int64_t)threadIdx.x * n_tiles + blockIdx.x] = hist[threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) tile_counts[(int64_t)P * n_tiles] = 0;      // closes the scan
}

// code[v] = (partition of v << tag_shift) | number of nodes u < v in the same partition; owner[v] = the partition.
__global__ __launch_bounds__(kThreads) void k_local_ids(const int32_t* __restrict__ part, int64_t N,
                                                        int P, int64_t n_tiles,
                                                        const int32_t* __restrict__ tile_base, int tag_shift,
                                                        uint32_t* __restrict__ code, uint8_t* __restrict__ owner)
{
    static_assert(SAR_MAX_PARTS <= 256, "a partition fits a byte");
    constexpr int kRounds = kPartTile / kThreads;
    constexpr int kChunks = kPartTile / 64;
    __shared__ int cnt[kChunks][SAR_MAX_PARTS];
    for (int k = threadIdx.x; k < kChunks * SAR_MAX_PARTS; k += kThreads) (&cnt[0][0])[k] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int pv[kRounds], rank[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t v = (int64_t)blockIdx.x * kPartTile + r * kThreads + threadIdx.x;
        int x = (v < N) ? part[v] : -1;
        if (x < 0 || x >= P) x = -1;
        pv[r] = x;
        // lanes holding the same partition id find each other
        unsigned long long mine = 0;
        bool pending = x >= 0;
        unsigned long long todo = __ballot(pending);
        while (todo) {
            const int first = __ffsll((long long)todo) - 1;
            const int val = __shfl(x, first);
            const unsigned long long same = __ballot(pending && x == val);
            if (pending && x == val) {
                mine = same;
                pending = false;
            }
            todo = __ballot(pending);
        }
        const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        rank[r] = __popcll(mine & below);
        if (x >= 0 && rank[r] == 0) cnt[r * (kThreads / 64) + wave][x] = __popcll(mine);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t v = (int64_t)blockIdx.x * kPartTile + r * kThreads + threadIdx.x;
        if (pv[r] < 0) continue;
        const int chunk = r * (kThreads / 64) + wave;
        int pre = 0;
        for (int c = 0; c < chunk; ++c) pre += cnt[c][pv[r]];
        const int64_t col = (int64_t)pv[r] * n_tiles;
        code[v] = ((uint32_t)pv[r] << tag_shift) | (uint32_t)(tile_base[col + blockIdx.x] - tile_base[col] + pre + rank[r]);
        owner[v] = (uint8_t)pv[r];
    }
}

// ------------------------------------------------------ buckets of keys
//
// Both indexes of a block are (key, value) pairs grouped by key with every group ascending: the CSR
// has key = row (block q, destination) and value = source, its transpose key = source and value =
// destination.  Counters in memory, one atomic per pair, serialise on the frequent keys of a
// power-law graph (15.2M edges: count 3.2 ms, scatter 2.1 ms for the CSR, 1.9 + 2.2 ms for the
// transposes, and as many passes again through cursors).  Here the pairs first go to buckets of up to
// 2^w keys and 4 thousand pairs on average: every tile of the input counts its pairs per bucket in
// LDS, one scan over the [bucket][tile] counts gives each tile its place in each bucket, and the
// tile's pairs are written there.  Then a workgroup takes a bucket: counts its keys in LDS; and, with
// the offsets of all keys scanned, places its values in LDS, sorts the groups there and writes them
// out in order.  No atomic leaves the LDS, and what is written does not depend on scheduling.
// The keys are dealt to the buckets in runs of four: neighbouring keys are often frequent together
// (ids in the order of degree), and a bucket of the 1024 most frequent rows of that graph holds half a
// million pairs (641 us for one workgroup, and 14 ms to sort its rows).
// What the kernels now take on those 15.2M edges: pairs to buckets 198 + 70 us from the edge list (the first gathers the
// nodes' codes, the second reads what it left; each for itself, one edge a thread at a time, 216 + 217) and 31 + 120 us from the
// CSR, keys 29, finish 170 each.  The last was 372 us, three quarters
// of it instructions: groups of up to 8 values now take 8 lanes instead of 16, those of 17 to 256 a network in registers.

constexpr int kBucketThreads = 512;
constexpr int kRunBits = 2;             // runs of four keys
constexpr int kBucketSub = 2048;         // input is taken 2048 pairs at a time
constexpr int kMaxBucketBits = 13;       // keys of a bucket: LDS counters of 32 KB at most
constexpr int kBucketCap = 10240;        // values of a bucket that are placed and sorted in LDS
constexpr int kRankLanes = 16;           // groups up to this length are sorted by 16 lanes
constexpr int kWaveSort = 256;           //            up to this length by one wavefront
constexpr int64_t kKeysPerPass = (int64_t)1 << 28;      // at most 32768 buckets at once
constexpr int64_t kMaxBucketCounts = (int64_t)1 << 25;  // entries of the [bucket][tile] counts

struct BucketPlan {
    int w;                   // log2 of the keys a bucket has room for
    int nb;                  // log2 of the buckets
    int64_t tile, n_tiles;   // pairs (input elements) per tile, a multiple of kBucketSub
    int n_buckets() const { return 1 << nb; }
};

// Key k of a pass sits in bucket `bucket` at place `place`; key_at is the inverse.
struct Deal {
    int nb;
    __device__ inline int bucket(int64_t key) const { return (int)(key >> kRunBits) & ((1 << nb) - 1); }
    __device__ inline int place(int64_t key) const
    {
        return ((int)(key >> (kRunBits + nb)) << kRunBits) | (int)(key & ((1 << kRunBits) - 1));
    }
    __device__ inline int64_t key_at(int bucket, int place) const
    {
        return ((((int64_t)(place >> kRunBits) << nb) | bucket) << kRunBits) | (place & ((1 << kRunBits) - 1));
    }
};

// n_keys <= kKeysPerPass.
BucketPlan plan_buckets(int64_t n_keys, int64_t n_items)
{
    BucketPlan b;
    const int64_t per = std::min<int64_t>(4096, std::max<int64_t>(256, n_items / 1024));
    const int64_t want = n_items / per + 1;
    b.nb = 0;
    // as many buckets as wanted, while each has a run; more where a bucket could not count its keys
    while (((int64_t)1 << b.nb) < want && ((int64_t)1 << (b.nb + kRunBits)) < n_keys && b.nb < 15) ++b.nb;
    while (((int64_t)1 << (b.nb + kMaxBucketBits)) < n_keys) ++b.nb;
    b.w = kRunBits;
    while (((int64_t)1 << (b.nb + b.w)) < n_keys) ++b.w;
    // about 512 tiles, fewer where the counts would not fit
    const int64_t tiles = std::min<int64_t>(512, std::max<int64_t>(1, kMaxBucketCounts >> b.nb));
    b.tile = std::max<int64_t>(1, (n_items + tiles - 1) / tiles);
    b.tile = (b.tile + kBucketSub - 1) / kBucketSub * kBucketSub;
    b.n_tiles = std::max<int64_t>(1, (n_items + b.tile - 1) / b.tile);
    return b;
}

// A pair as it travels: the key's place in its bucket above `vbits` bits of value; 32 bits where
// that fits, else 64.
template <typename PairT>
__device__ inline PairT make_pair(int key_in_bucket, uint32_t value, int vbits)
{
    return ((PairT)(uint32_t)key_in_bucket << vbits) | (PairT)value;
}

// The edges of worker p as pairs (q n_dst + destination, source), both local ids.  code[v] =
// (partition << tag_shift) | local id.
template <typename IdxT>
struct EdgeSource {
    const IdxT* src;
    const IdxT* dst;
    const uint32_t* code;
    const uint8_t* owner;    // the partition alone
    int64_t E, N, n_dst;
    int p, tag_shift;
    int* err;
    // Edges e, e + step ... e + (U - 1) step (below end): which are kept, their keys and, with VALUES, their values.  The
    // gathers of the codes wait for memory (10 MB of them for 2.4 million nodes do not stay in a 4 MB L2), so U edges' are
    // under way at once; without VALUES a source is only asked for its partition, a byte a node, which stays there.
    template <int U, bool VALUES>
    __device__ inline void get(int64_t e, int64_t step, int64_t end, bool (&have)[U], int64_t (&key)[U], uint32_t (&value)[U]) const
    {
        int64_t d[U], s[U];
        uint32_t cd[U], cs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = min(e + u * step, E - 1);
            d[u] = (int64_t)dst[at];
            s[u] = (int64_t)src[at];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            have[u] = e + u * step < end;
            if (have[u] && (d[u] < 0 || d[u] >= N || s[u] < 0 || s[u] >= N)) {
                atomicOr(err, 2);
                have[u] = false;
            }
            cd[u] = have[u] ? code[d[u]] : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            have[u] = have[u] && (int)(cd[u] >> tag_shift) == p;
            cs[u] = 0;
            if (have[u]) cs[u] = VALUES ? code[s[u]] : (uint32_t)owner[s[u]];
        }
        const uint32_t mask = (1u << tag_shift) - 1u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            key[u] = (int64_t)(VALUES ? cs[u] >> tag_shift : cs[u]) * n_dst + (int64_t)(cd[u] & mask);
            value[u] = cs[u] & mask;
        }
    }
};

// The same edges as the counting pass left them: (key, value), key ~0 where the edge is not kept.  Where all keys are one
// pass, the pool keeps the memory and nothing else needs the room, the scatter reads these 8 bytes instead of the edge list, and
// gathers no codes (15.2M edges: count and scatter 153 + 194 us, so 198 + 70).  That is some 15% of a build, and less than what the
// driver takes for memory that is not kept: the only handle built and freed, of 8 million edges an eighth kept, 4.6 ms with and
// 1.7 without, all of 2 million 1.8 and 0.9; beside other handles, from more than 256 MiB on (33 million edges), 100 million 17 to 75
// ms from run to run and 15.6, of 60 million an eighth 3.3 to 4.4 and 3.9.
struct StoredEdges {
    const uint2* edges;
    int64_t E;
    template <int U, bool VALUES>
    __device__ inline void get(int64_t e, int64_t step, int64_t end, bool (&have)[U], int64_t (&key)[U], uint32_t (&value)[U]) const
    {
        uint2 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = edges[min(e + u * step, E - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            have[u] = e + u * step < end && x[u].x != ~0u;
            key[u] = x[u].x;
            value[u] = x[u].y;
        }
    }
};

constexpr int kEdgesAhead = 4;

template <typename Src, bool STORE>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_count(Src in, int64_t tile, int64_t n_tiles, int64_t key0,
                                                                 int64_t n_keys, Deal deal,
                                                                 int32_t* __restrict__ counts,
                                                                 unsigned long long* __restrict__ kept,
                                                                 uint2* __restrict__ stored)
{
    extern __shared__ int bucket_hist[];
    const int n_buckets = 1 << deal.nb;
    for (int b = threadIdx.x; b < n_buckets; b += kBucketThreads) bucket_hist[b] = 0;
    __syncthreads();
    const int64_t beg = (int64_t)blockIdx.x * tile, end = min(in.E, beg + tile);
    unsigned long long mine = 0;
    for (int64_t e = beg + threadIdx.x; e < end; e += kBucketThreads * kEdgesAhead) {
        bool have[kEdgesAhead];
        int64_t key[kEdgesAhead];
        uint32_t value[kEdgesAhead];
        in.template get<kEdgesAhead, STORE>(e, kBucketThreads, end, have, key, value);
#pragma unroll
        for (int u = 0; u < kEdgesAhead; ++u) {
            if constexpr (STORE) {
                if (e + u * kBucketThreads < end)
                    stored[e + u * kBucketThreads] = have[u] ? make_uint2((uint32_t)key[u], value[u]) : make_uint2(~0u, 0u);
            }
            if (!have[u]) continue;
            ++mine;
            key[u] -= key0;
            if (key[u] >= 0 && key[u] < n_keys) atomicAdd(&bucket_hist[deal.bucket(key[u])], 1);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n_buckets; b += kBucketThreads) counts[(int64_t)b * n_tiles + blockIdx.x] = bucket_hist[b];
    if (blockIdx.x == 0 && threadIdx.x == 0) counts[(int64_t)n_buckets * n_tiles] = 0;      // closes the scan
    // edges kept for this worker, in 64 bits: the 32-bit offsets that follow must not wrap
    if (kept) {
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
        if ((threadIdx.x & 63) == 0 && mine) atomicAdd(kept, mine);
    }
}

template <typename Src, typename PairT>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_scatter(Src in, int64_t tile, int64_t n_tiles, int64_t key0,
                                                                   int64_t n_keys, Deal deal, int vbits,
                                                                   const int32_t* __restrict__ offsets,
                                                                   PairT* __restrict__ pairs)
{
    extern __shared__ int bucket_cursor[];
    const int n_buckets = 1 << deal.nb;
    for (int b = threadIdx.x; b < n_buckets; b += kBucketThreads)
        bucket_cursor[b] = offsets[(int64_t)b * n_tiles + blockIdx.x];
    __syncthreads();
    const int64_t beg = (int64_t)blockIdx.x * tile, end = min(in.E, beg + tile);
    for (int64_t e = beg + threadIdx.x; e < end; e += kBucketThreads * kEdgesAhead) {
        bool have[kEdgesAhead];
        int64_t key[kEdgesAhead];
        uint32_t value[kEdgesAhead];
        in.template get<kEdgesAhead, true>(e, kBucketThreads, end, have, key, value);
#pragma unroll
        for (int u = 0; u < kEdgesAhead; ++u) {
            key[u] -= key0;
            if (!have[u] || key[u] < 0 || key[u] >= n_keys) continue;
            pairs[atomicAdd(&bucket_cursor[deal.bucket(key[u])], 1)] = make_pair<PairT>(deal.place(key[u]), value[u], vbits);
        }
    }
}

// What the builder's kernels need of every block, in device memory.
struct BlkDev {
    sar::GlobalPtr<const int32_t> indptr;
    sar::GlobalPtr<const int32_t> indices;
    int64_t n_src, coff;     // sources of the block, and of the blocks before it
    int64_t nnz, nnz0;       // edges of the block, and of the blocks before it
    int64_t tile0;           // first tile of the block's edges (k_block_count / k_block_scatter)
    int64_t s_tile0;         // first tile of its sources in the launch lists' counts
    sar::GlobalPtr<uint32_t> rows;          // launch lists
    sar::GlobalPtr<uint32_t> t_rows;
    sar::GlobalPtr<int32_t> t_indptr;
    sar::GlobalPtr<int32_t> t_rank;
};

// The edges of all blocks as pairs (coff[q] + source, destination): a tile lies inside one block.
template <int64_t BlkDev::*FIRST = &BlkDev::tile0>
__device__ inline int block_of_tile(const BlkDev* blk, int P, int64_t tile)
{
    int lo = 0, hi = P - 1;      // the last block that starts at or before the tile and has tiles
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (blk[mid].*FIRST <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(kBucketThreads) void k_block_count(const BlkDev* __restrict__ blk, int P, int64_t tile,
                                                                int64_t n_tiles, int64_t key0, int64_t n_keys, Deal deal,
                                                                int32_t* __restrict__ counts)
{
    extern __shared__ int bucket_hist[];
    const int n_buckets = 1 << deal.nb;
    for (int b = threadIdx.x; b < n_buckets; b += kBucketThreads) bucket_hist[b] = 0;
    __syncthreads();
    const BlkDev& B = blk[block_of_tile(blk, P, blockIdx.x)];
    const int64_t beg = ((int64_t)blockIdx.x - B.tile0) * tile, end = min(B.nnz, beg + tile);
    const int64_t first = B.coff - key0;
    for (int64_t e = beg + threadIdx.x; e < end; e += kBucketThreads * kEdgesAhead) {
        int32_t j[kEdgesAhead];
#pragma unroll
        for (int u = 0; u < kEdgesAhead; ++u) j[u] = B.indices[min(e + u * kBucketThreads, end - 1)];
#pragma unroll
        for (int u = 0; u < kEdgesAhead; ++u) {
            const int64_t key = first + j[u];
            if (e + u * kBucketThreads < end && key >= 0 && key < n_keys) atomicAdd(&bucket_hist[deal.bucket(key)], 1);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n_buckets; b += kBucketThreads) counts[(int64_t)b * n_tiles + blockIdx.x] = bucket_hist[b];
    if (blockIdx.x == 0 && threadIdx.x == 0) counts[(int64_t)n_buckets * n_tiles] = 0;      // closes the scan
}

// The destination of an edge is the row whose range holds it: the rows that start inside the SUB
// edges at hand mark their first edge, and a running maximum over the marks names every edge's row.
// row[k] becomes the row of edge beg + threadIdx.x * kPer + k.  `known` is the row of edge beg - 1 where the workgroup
// has just had it, else -1; it becomes that of the last edge.
template <int THREADS, int SUB>
__device__ inline void rows_of_edges(const BlkDev& B, int64_t n_dst, int64_t beg, int n, int& known, int* mark,
                                     int (&row)[SUB / THREADS])
{
    constexpr int kPer = SUB / THREADS, kWaves = THREADS / 64;
    __shared__ int wave_max[kWaves];
    __shared__ int first_row;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (known < 0 && wave == 0) {
        // the last row that starts at or before `beg`, 64 tries a round (in 32 bits: of 64-bit uniform values the compiler
        // selected the new `lo` by the condition code of another instruction)
        uint32_t lo = 0, hi = (uint32_t)n_dst - 1u;
        const int32_t at = (int32_t)beg;
        while (lo < hi) {
            const uint32_t step = (hi - lo) / 64 + 1;
            const uint32_t c = (uint32_t)__popcll(__ballot(B.indptr[lo + min((lane + 1) * step, hi - lo)] <= at));
            const uint32_t from = min(c * step, hi - lo);
            hi = lo + min((c + 1) * step - 1, hi - lo);
            lo += from;
        }
        if (lane == 0) first_row = (int)lo;
    }
    for (int k = threadIdx.x; k < SUB; k += THREADS) mark[k] = 0;
    __syncthreads();
    const int r0 = known < 0 ? first_row : known;
    for (int64_t r = r0 + 1 + threadIdx.x; r < n_dst; r += THREADS) {
        const int64_t at = B.indptr[r] - beg;
        if (at >= n) break;
        atomicMax(&mark[at], (int)(r - r0));
    }
    __syncthreads();
    int run = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        run = max(run, mark[threadIdx.x * kPer + k]);
        row[k] = run;
    }
    int incl = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(incl, o);
        if (lane >= o) incl = max(incl, x);
    }
    if (lane == 63) wave_max[wave] = incl;
    __syncthreads();
    int before = __shfl_up(incl, 1);
    if (lane == 0) before = 0;
    for (int k = 0; k < wave; ++k) before = max(before, wave_max[k]);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        row[k] = r0 + max(before, row[k]);
        if ((int)threadIdx.x * kPer + k == n - 1) first_row = row[k];
    }
    __syncthreads();
    known = first_row;
}

template <typename PairT>
__global__ __launch_bounds__(kBucketThreads) void k_block_scatter(const BlkDev* __restrict__ blk, int P, int64_t n_dst,
                                                                  int64_t tile, int64_t n_tiles, int64_t key0,
                                                                  int64_t n_keys, Deal deal, int vbits,
                                                                  const int32_t* __restrict__ offsets,
                                                                  PairT* __restrict__ pairs)
{
    constexpr int kPer = kBucketSub / kBucketThreads;
    extern __shared__ int bucket_cursor[];
    __shared__ int mark[kBucketSub];
    const int n_buckets = 1 << deal.nb;
    for (int b = threadIdx.x; b < n_buckets; b += kBucketThreads)
        bucket_cursor[b] = offsets[(int64_t)b * n_tiles + blockIdx.x];
    const BlkDev& B = blk[block_of_tile(blk, P, blockIdx.x)];
    const int64_t t_beg = ((int64_t)blockIdx.x - B.tile0) * tile, t_end = min(B.nnz, t_beg + tile);
    const int64_t first = B.coff - key0;
    int known = -1;
    for (int64_t beg = t_beg; beg < t_end; beg += kBucketSub) {
        const int n = (int)min((int64_t)kBucketSub, t_end - beg);
        int row[kPer];
        rows_of_edges<kBucketThreads, kBucketSub>(B, n_dst, beg, n, known, mark, row);
#pragma unroll
        for (int k = 0; k < kPer; ++k) mark[threadIdx.x * kPer + k] = row[k];
        __syncthreads();
        for (int k = threadIdx.x; k < n; k += kBucketThreads) {
            const int64_t key = first + B.indices[beg + k];
            if (key < 0 || key >= n_keys) continue;
            pairs[atomicAdd(&bucket_cursor[deal.bucket(key)], 1)] =
                make_pair<PairT>(deal.place(key), (uint32_t)mark[k], vbits);
        }
    }
}

// The same for 32-bit pairs and up to 2^kStagedBits buckets: 16 thousand pairs are put in the order of their buckets in
// LDS first, so that neighbouring lanes write neighbouring pairs.  A pair at a time, a wavefront's store went to 64
// different cache lines of which it wrote four bytes each (15.2M pairs: 13M requests beyond the L2s, 187 us; staged 120, half as
// many pairs at a time by two workgroups on a CU 133).
constexpr int kStageThreads = 1024, kStageSub = 4096, kStage = 4 * kStageSub, kStagedBits = 12;
constexpr size_t kStagedLds = (2 * ((size_t)1 << kStagedBits) + kStage + kStage / 2) * sizeof(int);
__global__ __launch_bounds__(kStageThreads) void k_block_scatter_staged(const BlkDev* __restrict__ blk, int P, int64_t n_dst,
                                                                        int64_t tile, int64_t n_tiles, int64_t key0,
                                                                        int64_t n_keys, Deal deal, int vbits,
                                                                        const int32_t* __restrict__ offsets,
                                                                        uint32_t* __restrict__ pairs)
{
    constexpr int kPer = kStageSub / kStageThreads, kSubs = kStage / kStageSub, kWaves = kStageThreads / 64;
    constexpr int kMine = ((1 << kStagedBits) + kStageThreads - 1) / kStageThreads;    // buckets a thread sums up
    extern __shared__ int staged_lds[];
    __shared__ int wave_sum[kWaves];
    int* const start = staged_lds;                                     // pairs of a bucket, then its first place here
    int* const at = start + (1 << kStagedBits);                        // its next place in `pairs`, less `start`
    uint32_t* const stage = (uint32_t*)(at + (1 << kStagedBits));      // first the marks of the rows
    uint16_t* const owner = (uint16_t*)(stage + kStage);               // the bucket of a staged pair
    const int n_buckets = 1 << deal.nb, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const BlkDev& B = blk[block_of_tile(blk, P, blockIdx.x)];
    const int64_t t_beg = ((int64_t)blockIdx.x - B.tile0) * tile, t_end = min(B.nnz, t_beg + tile);
    const int64_t first = B.coff - key0;
    int next[kMine];                                                   // of the thread's own buckets
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int b = threadIdx.x * kMine + k;
        next[k] = b < n_buckets ? offsets[(int64_t)b * n_tiles + blockIdx.x] : 0;
    }
    int known = -1;
    for (int64_t beg = t_beg; beg < t_end; beg += kStage) {
        for (int b = threadIdx.x; b < n_buckets; b += kStageThreads) start[b] = 0;
        uint32_t pair[kSubs * kPer], meta[kSubs * kPer];               // meta: bucket | rank in the stage's bucket << 12
#pragma unroll
        for (int sub = 0; sub < kSubs; ++sub) {
            const int64_t sb = beg + sub * kStageSub;
            const int n = (int)max((int64_t)0, min((int64_t)kStageSub, t_end - sb));
#pragma unroll
            for (int k = 0; k < kPer; ++k) meta[sub * kPer + k] = ~0u;
            if (n == 0) continue;                                      // the same for the whole workgroup
            int row[kPer];
            int32_t j[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) j[k] = B.indices[sb + min((int)threadIdx.x * kPer + k, n - 1)];
            rows_of_edges<kStageThreads, kStageSub>(B, n_dst, sb, n, known, (int*)stage, row);
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int64_t key = first + j[k];
                if ((int)threadIdx.x * kPer + k >= n || key < 0 || key >= n_keys) continue;
                const int b = deal.bucket(key);
                pair[sub * kPer + k] = make_pair<uint32_t>(deal.place(key), (uint32_t)row[k], vbits);
                meta[sub * kPer + k] = (uint32_t)b | (uint32_t)atomicAdd(&start[b], 1) << kStagedBits;
            }
        }
        __syncthreads();
        int count[kMine], sum = 0;
#pragma unroll
        for (int k = 0; k < kMine; ++k) {
            const int b = threadIdx.x * kMine + k;
            count[k] = b < n_buckets ? start[b] : 0;
            sum += count[k];
        }
        int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        int run = incl - sum, total = 0;
        for (int k = 0; k < kWaves; ++k) {
            if (k < wave) run += wave_sum[k];
            total += wave_sum[k];
        }
#pragma unroll
        for (int k = 0; k < kMine; ++k) {
            const int b = threadIdx.x * kMine + k;
            if (b < n_buckets) {
                start[b] = run;
                at[b] = next[k] - run;
            }
            run += count[k];
            next[k] += count[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSubs * kPer; ++k) {
            if (meta[k] == ~0u) continue;
            const int b = (int)(meta[k] & ((1u << kStagedBits) - 1u)), to = start[b] + (int)(meta[k] >> kStagedBits);
            stage[to] = pair[k];
            owner[to] = (uint16_t)b;
        }
        __syncthreads();
        for (int k = threadIdx.x; k < total; k += kStageThreads) pairs[at[owner[k]] + k] = stage[k];
        __syncthreads();
    }
}

// Ascending sort of a[0, len) by the threads `tid` of `nt`: a bitonic network in which every
// comparator is ascending, so the virtual +inf padding behind the end never moves.
template <typename Sync>
__device__ inline void bitonic(int32_t* a, int len, int tid, int nt, Sync&& sync)
{
    int n2 = 1;
    while (n2 < len) n2 <<= 1;
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const bool flip = j == (k >> 1);
            for (int t = tid; t < n2; t += nt) {
                const int partner = flip ? (t ^ (k - 1)) : (t ^ j);
                if (partner > t && partner < len) {
                    const int32_t x = a[t], y = a[partner];
                    if (x > y) {
                        a[t] = y;
                        a[partner] = x;
                    }
                }
            }
            sync();
        }
    }
}

// The value of lane ^ M.
template <int M>
__device__ inline uint32_t lane_xor(uint32_t x)
{
    constexpr int kDpp = M == 1 ? 0xB1 : M == 2 ? 0x4E : M == 3 ? 0x1B : M == 7 ? 0x141 : M == 8 ? 0x128 : M == 15 ? 0x140 : 0;
    if constexpr (kDpp != 0)      // quad_perm, row_half_mirror, row_ror:8, row_mirror
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDpp, 0xf, 0xf, false);
    else if constexpr (M < 32)
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (M << 10) | 0x1f);
    else
        return (uint32_t)__shfl_xor((int)x, M);
}

// Values among the 16 of a DPP row that sort before this lane's (equal ones by lane).
template <int J>
__device__ inline int rank16_step(int32_t x, int l)
{
    if constexpr (J == 0) {
        return 0;
    } else {
        const int32_t y = __builtin_amdgcn_update_dpp(0, x, 0x120 + J, 0xf, 0xf, false);   // row_ror:J
        const int from = (l - J) & 15;
        return rank16_step<J - 1>(x, l) + ((y < x || (y == x && from < l)) ? 1 : 0);
    }
}
__device__ inline int rank16(int32_t x, int l) { return rank16_step<15>(x, l); }

// Values among the 8 of half a DPP row that sort before this lane's.  A lane's partner is lane ^ m, and of equal values the
// one at the lower lane goes first: it is the partner where the lane has m's highest bit.
__device__ inline int rank8(uint32_t x, int l)
{
    const uint32_t b1 = x + (l & 1), b2 = x + (l >> 1 & 1), b4 = x + (l >> 2 & 1);
    const uint32_t far = lane_xor<7>(x);
    return (lane_xor<1>(x) < b1) + (lane_xor<2>(x) < b2) + (lane_xor<3>(x) < b2) + (far < b4) + (lane_xor<1>(far) < b4) +
           (lane_xor<2>(far) < b4) + (lane_xor<3>(far) < b4);
}

// Steps of a bitonic network over 64 N values, lane l holding values N l to N l + N - 1, in which every comparator is
// ascending: value i meets i ^ (K - 1), then i ^ K/4, i ^ K/8 ... 1.
template <int N, int J>
__device__ inline void bitonic_halves(int32_t (&x)[N], int lane)
{
    if constexpr (J >= 1) {
        if constexpr (J >= N) {
#pragma unroll
            for (int r = 0; r < N; ++r) {
                const int32_t y = (int32_t)lane_xor<J / N>((uint32_t)x[r]);
                x[r] = (lane & (J / N)) ? max(x[r], y) : min(x[r], y);
            }
        } else {
#pragma unroll
            for (int r = 0; r < N; ++r)
                if (!(r & J)) {
                    const int32_t lo = min(x[r], x[r | J]);
                    x[r | J] = max(x[r], x[r | J]);
                    x[r] = lo;
                }
        }
        bitonic_halves<N, J / 2>(x, lane);
    }
}
template <int N, int K>
__device__ inline void bitonic_steps(int32_t (&x)[N], int lane)
{
    if constexpr (K > 2) bitonic_steps<N, K / 2>(x, lane);
    if constexpr (K > N) {
        constexpr int M = K / N - 1;
        int32_t y[N];
#pragma unroll
        for (int r = 0; r < N; ++r) y[r] = (int32_t)lane_xor<M>((uint32_t)x[N - 1 - r]);
#pragma unroll
        for (int r = 0; r < N; ++r) x[r] = (lane & ((M + 1) / 2)) ? max(x[r], y[r]) : min(x[r], y[r]);
    } else {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const int o = r ^ (K - 1);
            if (r < o) {
                const int32_t lo = min(x[r], x[o]);
                x[o] = max(x[r], x[o]);
                x[r] = lo;
            }
        }
    }
    bitonic_halves<N, K / 4>(x, lane);
}

// Ascending order of a[0, len), len <= 64 N, by one wavefront, in registers: 256 values are 36 steps, 15 of them
// inside a lane, of the others' exchanges two thirds DPP; under two instructions a value.  (Counting for every value the ones
// before it reads the group from LDS once per value: 13 instructions for each of 256 values, and the long groups were most of
// what the kernel below issued.)
template <int N>
__device__ inline void sort_wave(int32_t* a, int len, int lane)
{
    int32_t x[N];
#pragma unroll
    for (int r = 0; r < N; ++r) x[r] = lane * N + r < len ? a[lane * N + r] : 0x7fffffff;
    bitonic_steps<N, 64 * N>(x, lane);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the reads stay ahead of the writes
#pragma unroll
    for (int r = 0; r < N; ++r)
        if (lane * N + r < len) a[lane * N + r] = x[r];
}

// Ascending order of a[0, len) in LDS by a workgroup of THREADS, len <= kMergeSort: wavefronts sort
// pieces of 256, then pairs of sorted runs are merged in place, every value finding its place by a
// search in the other run.  (A bitonic network spends most of its time in barriers.)
constexpr int kMergeSort = 4096;
template <int THREADS>
__device__ inline void merge_sort(int32_t* a, int len)
{
    constexpr int kPer = kMergeSort / THREADS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c = wave * kWaveSort; c < len; c += THREADS / 64 * kWaveSort)
        sort_wave<kWaveSort / 64>(a + c, min(kWaveSort, len - c), lane);
    __syncthreads();
    for (int width = kWaveSort; width < len; width *= 2) {
        int32_t x[kPer];
        int to[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int e = r * THREADS + threadIdx.x;
            to[r] = -1;
            x[r] = 0;
            if (e >= len) continue;
            x[r] = a[e];
            const int run = e / width, other = (run ^ 1) * width;
            int lo = 0, hi = min(width, max(0, len - other));
            const int32_t bound = x[r] + (run & 1);          // of equal values the first run's go first
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (a[other + mid] < bound)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            to[r] = (run & ~1) * width + (e - run * width) + lo;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPer; ++r)
            if (to[r] >= 0) a[to[r]] = x[r];
        __syncthreads();
    }
}

// off[key] = pairs of the key, for every key of the pass: a workgroup per bucket.  off[n_keys] and the counters
// of the buckets too large for LDS start at 0.
template <typename PairT>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_keys(const PairT* __restrict__ pairs,
                                                                const int32_t* __restrict__ offsets, int64_t n_tiles,
                                                                int w, Deal deal, int64_t n_keys, int vbits,
                                                                int32_t* __restrict__ off, int* __restrict__ big_count)
{
    extern __shared__ int bucket_lds[];
    const int n_slots = 1 << w, b = blockIdx.x;
    if (b == 0 && threadIdx.x == 0) big_count[0] = big_count[1] = off[n_keys] = 0;
    for (int k = threadIdx.x; k < n_slots; k += kBucketThreads) bucket_lds[k] = 0;
    __syncthreads();
    const int beg = offsets[(int64_t)b * n_tiles], end = offsets[(int64_t)(b + 1) * n_tiles];
    for (int e = beg + threadIdx.x; e < end; e += kBucketThreads) atomicAdd(&bucket_lds[(int)(pairs[e] >> vbits)], 1);
    __syncthreads();
    for (int k = threadIdx.x; k < n_slots; k += kBucketThreads) {
        const int64_t key = deal.key_at(b, k);
        if (key < n_keys) off[key] = bucket_lds[k];
    }
}

// One bucket per workgroup: its values in order at off[key], each group ascending.  A bucket of more
// than kBucketCap pairs is placed in memory directly and listed for k_sort_buckets.
template <typename PairT>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_finish(const PairT* __restrict__ pairs,
                                                                  const int32_t* __restrict__ offsets, int64_t n_tiles,
                                                                  int w, Deal deal, int64_t n_keys, int vbits,
                                                                  const int32_t* __restrict__ off,
                                                                  int32_t* __restrict__ values,
                                                                  int32_t* __restrict__ big_list,
                                                                  int* __restrict__ big_count)
{
    constexpr int kWaves = kBucketThreads / 64;
    constexpr int kRunLanes = 16;
    extern __shared__ int bucket_lds[];
    __shared__ int wave_sum[kWaves];
    __shared__ int n_small, n_listed, n_big;
    __shared__ uint16_t small[kBucketCap / (kRankLanes / 2 + 1) + 1];
    __shared__ uint16_t listed[kBucketCap / kRankLanes];
    __shared__ uint16_t big[kBucketCap / kWaveSort];
    const int n_slots = 1 << w;
    int* cnt = bucket_lds;
    int32_t* vals = bucket_lds + n_slots;
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int beg = offsets[(int64_t)b * n_tiles], end = offsets[(int64_t)(b + 1) * n_tiles], n = end - beg;
    const PairT vmask = (PairT)(((uint64_t)1 << vbits) - 1u);
    if (n == 0) return;
    if (n > kBucketCap) {
        for (int k = threadIdx.x; k < n_slots; k += kBucketThreads) {
            const int64_t key = deal.key_at(b, k);
            cnt[k] = key < n_keys ? off[key] : 0;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < n; e += kBucketThreads) {
            const PairT x = pairs[beg + e];
            values[atomicAdd(&cnt[(int)(x >> vbits)], 1)] = (int32_t)(x & vmask);
        }
        if (threadIdx.x == 0) big_list[atomicAdd(big_count, 1)] = b;
        return;
    }
    if (threadIdx.x == 0) n_small = n_listed = n_big = 0;
    for (int k = threadIdx.x; k < n_slots; k += kBucketThreads) {
        const int64_t key = deal.key_at(b, k);
        cnt[k] = key < n_keys ? off[key + 1] - off[key] : 0;
    }
    __syncthreads();
    const int per = (n_slots + kBucketThreads - 1) / kBucketThreads;
    int sum = 0;
    for (int k = 0; k < per; ++k) {
        const int at = threadIdx.x * per + k;
        if (at < n_slots) sum += cnt[at];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(incl, o);
        if (lane >= o) incl += x;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int run = incl - sum;
    for (int k = 0; k < wave; ++k) run += wave_sum[k];
    for (int k = 0; k < per; ++k) {
        const int at = threadIdx.x * per + k;
        if (at < n_slots) {
            const int c = cnt[at];
            cnt[at] = run;
            run += c;
        }
    }
    __syncthreads();
    // each group's start is its cursor; afterwards it is the group's end
    constexpr int kAhead = 8;
    for (int e0 = threadIdx.x; e0 < n; e0 += kBucketThreads * kAhead) {
        PairT x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) x[u] = pairs[beg + min(e0 + u * kBucketThreads, n - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (e0 + u * kBucketThreads < n) vals[atomicAdd(&cnt[(int)(x[u] >> vbits)], 1)] = (int32_t)(x[u] & vmask);
    }
    __syncthreads();
    // Groups of up to 8 values, most of them: 8 lanes each, a lane's value goes to the place that the count of the values
    // before it gives it; the others' values come by DPP, without LDS.
    for (int k0 = threadIdx.x / 8; k0 < n_slots; k0 += kBucketThreads / 8) {
        const int s = k0 ? cnt[k0 - 1] : 0, len = cnt[k0] - s, l = threadIdx.x % 8;
        if (len > 8) {
            if (l != 0) continue;
            if (len > kWaveSort)
                big[atomicAdd(&n_big, 1)] = (uint16_t)k0;
            else if (len > kRankLanes)
                listed[atomicAdd(&n_listed, 1)] = (uint16_t)k0;
            else
                small[atomicAdd(&n_small, 1)] = (uint16_t)k0;
        } else if (len > 1) {
            const uint32_t x = l < len ? (uint32_t)vals[s + l] : 0x7fffffffu;
            const int rank = rank8(x, l);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the reads stay ahead of the writes
            if (l < len) vals[s + rank] = (int32_t)x;
        }
    }
    __syncthreads();
    // up to 16: a DPP row each
    for (int i = threadIdx.x / kRankLanes; i < n_small; i += kBucketThreads / kRankLanes) {
        const int k = small[i], s = k ? cnt[k - 1] : 0, len = cnt[k] - s, l = threadIdx.x % kRankLanes;
        const int32_t x = l < len ? vals[s + l] : 0x7fffffff;
        const int rank = rank16(x, l);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (l < len) vals[s + rank] = x;
    }
    // up to 256: a wavefront each, one to four values to a lane
    for (int i = wave; i < n_listed; i += kWaves) {
        const int k = __builtin_amdgcn_readfirstlane(listed[i]);
        const int s = k ? cnt[k - 1] : 0, len = __builtin_amdgcn_readfirstlane(cnt[k] - s);
        if (len <= 64)
            sort_wave<1>(vals + s, len, lane);
        else if (len <= 128)
            sort_wave<2>(vals + s, len, lane);
        else
            sort_wave<4>(vals + s, len, lane);
    }
    __syncthreads();
    for (int i = 0; i < n_big; ++i) {
        const int k = big[i], s = k ? cnt[k - 1] : 0, len = cnt[k] - s;
        if (len <= kMergeSort)
            merge_sort<kBucketThreads>(vals + s, len);
        else
            bitonic(vals + s, len, threadIdx.x, kBucketThreads, [] { __syncthreads(); });
    }
    __syncthreads();
    // a run of keys is contiguous here and there
    for (int r = threadIdx.x / kRunLanes; r < n_slots >> kRunBits; r += kBucketThreads / kRunLanes) {
        const int k0 = r << kRunBits, s = k0 ? cnt[k0 - 1] : 0, len = cnt[k0 + (1 << kRunBits) - 1] - s;
        if (len == 0) continue;
        int32_t* const out = values + off[deal.key_at(b, k0)];
        for (int e = threadIdx.x % kRunLanes; e < len; e += kRunLanes) out[e] = vals[s + e];
    }
}

// A call's report to the host: flags[0..3] (or zeros), then in[k * step] for k in [0, n).
__global__ __launch_bounds__(kThreads) void k_report(const int32_t* __restrict__ in, int64_t step, int n,
                                                     const int* __restrict__ flags, int32_t* __restrict__ out)
{
    if (threadIdx.x < 4) out[threadIdx.x] = flags ? flags[threadIdx.x] : 0;
    for (int k = threadIdx.x; k < n; k += kThreads) out[4 + k] = in[k * step];
}

// indptr of block q out of the offsets of all blocks' rows
__global__ __launch_bounds__(kThreads) void k_make_indptr(const int32_t* __restrict__ row_off,
                                                          int64_t n_dst, int P,
                                                          int32_t* __restrict__ indptr_all)
{
    const int64_t total = (int64_t)P * (n_dst + 1);
    for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * kThreads) {
        const int64_t q = k / (n_dst + 1), i = k - q * (n_dst + 1);
        indptr_all[k] = row_off[q * n_dst + i] - row_off[q * n_dst];
    }
}

// The groups of the listed buckets (those too large for k_bucket_finish).  A bucket is kSortShares shares, share
// c holding the groups at places c, c + kSortShares ... (a run of neighbouring keys, often long together, falls
// into different shares), and the workgroups take share after share from *next: a bucket's long groups may be
// one or all of its groups, so a fixed deal of shares to workgroups leaves most of them idle (1000 rows of 30
// thousand edges, one to a bucket: build 35.5 ms when workgroup (x, y) took share y of every 32nd bucket,
// 7.9 ms now; 100 rows of 300 thousand 160 and 77 ms).  Every workgroup ends when the shares have been taken.
constexpr int kSortShares = 16;
__global__ __launch_bounds__(kThreads) void k_sort_buckets(const int32_t* __restrict__ off, int32_t* __restrict__ data,
                                                           int w, Deal deal, int64_t n_keys,
                                                           const int32_t* __restrict__ big_list,
                                                           const int* __restrict__ big_count, int* __restrict__ next)
{
    constexpr int kMostPlaces = (1 << kMaxBucketBits) / kSortShares;
    __shared__ int32_t buf[kLdsSort];
    __shared__ int32_t first[kMostPlaces], length[kMostPlaces];
    __shared__ int share, n_groups;
    const int n_shares = *big_count * kSortShares;
    if (n_shares == 0) return;       // the usual case: no atomics then
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {
            share = atomicAdd(next, 1);
            n_groups = 0;
        }
        __syncthreads();
        if (share >= n_shares) break;
        const int b = big_list[share / kSortShares];
        for (int k = share % kSortShares + (int)threadIdx.x * kSortShares; k < (1 << w); k += kThreads * kSortShares) {
            const int64_t key = deal.key_at(b, k);
            if (key >= n_keys) continue;
            const int beg = off[key], len = off[key + 1] - beg;
            if (len <= 1) continue;
            const int at = atomicAdd(&n_groups, 1);
            first[at] = beg;
            length[at] = len;
        }
        __syncthreads();
        const int n = n_groups;
        for (int i = 0; i < n; ++i) {
            const int len = length[i];
            int32_t* g = data + first[i];
            const bool in_lds = len <= kLdsSort;
            if (in_lds) {
                for (int t = threadIdx.x; t < len; t += kThreads) buf[t] = g[t];
            }
            __syncthreads();
            if (len <= kMergeSort)
                merge_sort<kThreads>(buf, len);
            else
                bitonic(in_lds ? buf : g, len, threadIdx.x, kThreads, [] { __syncthreads(); });
            if (in_lds) {
                for (int t = threadIdx.x; t < len; t += kThreads) g[t] = buf[t];
            }
            __syncthreads();
        }
    }
}

// ------------------------------------------------- degree-class row lists

__device__ inline int degree_class(int len) { return len <= 0 ? 0 : 32 - __clz(len); }

// The launch lists: the blocks' own rows, their sources, the rows of all blocks, the sources of all blocks.
enum class Lists { kRows, kSources, kAllRows, kAllSources };
constexpr int kPlacePer = 8, kPlaceRows = kThreads * kPlacePer;      // rows of a tile
// Rows of a tile in every class, [class][tile] for each list one after another (the sources of all blocks: [class][block][tile];
// a block has the tiles of its own sources), and, scanned, how many of the list's class stand before them.
struct ListIn {
    const BlkDev* blk;
    const int32_t* off;      // kAllRows: the all-blocks row offsets
    int64_t n_dst;
    int P;
    int64_t t_rows, t_src;   // tiles of a block's rows, and of all blocks' sources
    bool fused;
    __host__ __device__ inline int64_t first_src() const { return P * sar::kNumClasses * t_rows; }
    __host__ __device__ inline int64_t first_all_rows() const { return first_src() + sar::kNumClasses * t_src; }
    __host__ __device__ inline int64_t first_all_src() const { return first_all_rows() + (fused ? sar::kNumClasses * t_rows : 0); }
    __host__ __device__ inline int64_t size() const { return first_all_src() + sar::kNumClasses * t_src; }
    // where the counts of class c of list l (of block q) start, and how many there are
    __device__ inline int64_t counts(Lists l, int q, int c, int64_t& tiles) const
    {
        if (l == Lists::kSources) {
            tiles = (q + 1 < P ? blk[q + 1].s_tile0 : t_src) - blk[q].s_tile0;
            return first_src() + blk[q].s_tile0 * sar::kNumClasses + c * tiles;
        }
        tiles = l == Lists::kAllSources ? t_src : t_rows;
        const int64_t first = l == Lists::kRows ? (int64_t)q * sar::kNumClasses * t_rows : l == Lists::kAllRows ? first_all_rows() : first_all_src();
        return first + c * tiles;
    }
    // a workgroup's block and its tile there: the blocks' rows (tile, block), all others by the tile
    __device__ inline void place(Lists l, int& q, int64_t& tile) const
    {
        q = (int)blockIdx.y;
        tile = blockIdx.x;
        if (l == Lists::kRows || l == Lists::kAllRows) return;
        q = block_of_tile<&BlkDev::s_tile0>(blk, P, tile);
        tile -= blk[q].s_tile0;
    }
    __device__ inline const int32_t* offsets(Lists l, int y, int64_t& n) const
    {
        const bool sources = l == Lists::kSources || l == Lists::kAllSources;
        n = sources ? blk[y].n_src : n_dst;
        return l == Lists::kAllRows ? off : sources ? blk[y].t_indptr : blk[y].indptr;
    }
};

// The classes of a tile's rows: class c[j] and place at[j] among the tile's rows of the class, in the rows' order, of row
// tile * kPlaceRows + j * kThreads + threadIdx.x (-1: no row); cnt[class] = rows of the class in the tile.
__device__ inline void tile_classes(const int32_t* off, int64_t n, int64_t tile, int (&c)[kPlacePer], int (&at)[kPlacePer],
                                    int* cnt)
{
    constexpr int kChunks = kPlacePer * kThreads / 64;
    __shared__ int chunk[kChunks][sar::kNumClasses];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k = threadIdx.x; k < kChunks * sar::kNumClasses; k += kThreads) (&chunk[0][0])[k] = 0;
#pragma unroll
    for (int j = 0; j < kPlacePer; ++j) {
        const int64_t r = tile * kPlaceRows + j * kThreads + threadIdx.x;
        c[j] = r < n ? degree_class(off[r + 1] - off[r]) : -1;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPlacePer; ++j) {
        at[j] = 0;
        unsigned long long todo = __ballot(c[j] >= 0);
        while (todo) {
            const int first = __ffsll((long long)todo) - 1, of = __shfl(c[j], first);
            const unsigned long long same = __ballot(c[j] == of);
            if (c[j] == of) at[j] = __popcll(same & ((1ull << lane) - 1ull));
            if (lane == first) chunk[j * (kThreads / 64) + wave][of] = __popcll(same);
            todo &= ~same;
        }
    }
    __syncthreads();
    if (threadIdx.x < sar::kNumClasses) {
        int run = 0;
#pragma unroll 8
        for (int k = 0; k < kChunks; ++k) {
            const int x = chunk[k][threadIdx.x];
            chunk[k][threadIdx.x] = run;
            run += x;
        }
        cnt[threadIdx.x] = run;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPlacePer; ++j)
        if (c[j] >= 0) at[j] += chunk[j * (kThreads / 64) + wave][c[j]];
}

__global__ __launch_bounds__(kThreads) void k_class_count(ListIn in, Lists l, int32_t* __restrict__ counts)
{
    __shared__ int cnt[sar::kNumClasses];
    int64_t n, tiles, tile;
    int q;
    in.place(l, q, tile);
    const int32_t* off = in.offsets(l, q, n);
    int c[kPlacePer], at[kPlacePer];
    tile_classes(off, n, tile, c, at, cnt);
    __syncthreads();
    if (threadIdx.x < sar::kNumClasses) {
        counts[in.counts(l, q, threadIdx.x, tiles) + tile] = cnt[threadIdx.x];
        if (l == Lists::kSources) counts[in.counts(Lists::kAllSources, 0, threadIdx.x, tiles) + blockIdx.x] = cnt[threadIdx.x];
    }
    if (l == Lists::kRows && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) counts[in.size()] = 0;
}

// hist[list][class] out of the scanned counts (differences of 32-bit sums): the blocks' rows, their sources, all rows, all sources
__global__ __launch_bounds__(kThreads) void k_class_totals(ListIn in, bool sources, const int32_t* __restrict__ counts,
                                                           int32_t* __restrict__ hist)
{
    for (int k = threadIdx.x; k < (2 * in.P + 2) * sar::kNumClasses; k += kThreads) {
        const int y = k / sar::kNumClasses, c = k % sar::kNumClasses;
        const Lists l = y < in.P ? Lists::kRows : y < 2 * in.P ? Lists::kSources : y == 2 * in.P ? Lists::kAllRows : Lists::kAllSources;
        const bool there = l == Lists::kRows || (l == Lists::kAllRows ? in.fused : sources);
        int64_t tiles;
        const int64_t of = in.counts(l, y % in.P, c, tiles);
        hist[k] = there ? (int32_t)((uint32_t)counts[of + tiles] - (uint32_t)counts[of]) : 0;
    }
}

// start[class] is the first place of the class in the list; value written = r | tag.  Rows stand by class, in a class in their
// own order: the same lists from every build.  Where ids follow degrees the longest rows stand in front; the kernels deal the
// rows after the shared ones from behind (1.5 M edges, rows of up to 10 thousand, forward pass: 219 us; dealt from the front 287,
// and 267 with the rows in the order in which workgroups came to take places for 256 at a time).  Rows without edges (class 0)
// are listed last, in the blocks' own row lists not at all.
__global__ __launch_bounds__(kThreads) void k_class_place(ListIn in, Lists l, int tag_shift, const int* __restrict__ starts,
                                                          const int32_t* __restrict__ counts, uint32_t* __restrict__ out_all)
{
    __shared__ int cnt[sar::kNumClasses];
    __shared__ int base[sar::kNumClasses];
    int64_t n, tiles, tile;
    int q;
    in.place(l, q, tile);
    const int32_t* off = in.offsets(l, q, n);
    const int* start = starts + (l == Lists::kRows || l == Lists::kSources ? q * sar::kNumClasses : 0);
    uint32_t* out = l == Lists::kRows ? in.blk[q].rows.as<uint32_t>() : l == Lists::kSources ? in.blk[q].t_rows.as<uint32_t>() : out_all;
    const uint32_t tag = l == Lists::kAllSources ? (uint32_t)q << tag_shift : 0u;
    int c[kPlacePer], at[kPlacePer];
    tile_classes(off, n, tile, c, at, cnt);
    if (threadIdx.x < sar::kNumClasses) {
        const int64_t of = in.counts(l, q, threadIdx.x, tiles), mine = l == Lists::kAllSources ? (int64_t)blockIdx.x : tile;
        base[threadIdx.x] = start[threadIdx.x] + (int32_t)((uint32_t)counts[of + mine] - (uint32_t)counts[of]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPlacePer; ++j)
        if (c[j] > 0 || (c[j] == 0 && l != Lists::kRows))
            out[base[c[j]] + at[j]] = (uint32_t)(tile * kPlaceRows + j * kThreads + threadIdx.x) | tag;
}

struct ClassLayout {
    int64_t n_rows = 0, n_long = 0, n_shared = 0, n_wide = 0;
    int start[sar::kNumClasses];
};

// Degree class from which a list's rows are shared by the four wavefronts of a workgroup: the
// lowest of 128 / 256 / 512 edges (but not below `floor_class`) that leaves them a small minority
// of the list.  A skewed list then has no single-wavefront row long enough to decide when a
// launch ends; a list of uniformly long rows keeps one wavefront per row (no merges).
int pick_long_class(const int* hist, int floor_class)
{
    int64_t n_rows = 0;
    for (int c = 1; c < sar::kNumClasses; ++c) n_rows += hist[c];
    for (int lc = floor_class; lc < sar::kLongClass; ++lc) {
        int64_t n_long = 0;
        for (int c = lc; c < sar::kNumClasses; ++c) n_long += hist[c];
        if (n_long <= std::max<int64_t>(256, n_rows / 16)) return lc;
    }
    return sar::kLongClass;
}

// Degree class from which a launch over the list shares rows among four wavefronts: that of the long rows, and in a short
// launch a lower one.  A wavefront takes eight edges per round trip to memory, so a row of more edges than a wavefront's
// even share of the launch (4096 of them run at once) is what the launch waits for: with 136 thousand edges in a block, 33 a
// wavefront, the rows of 8 edges and more alone took 38 of the 42 us of its forward launch, rows of 64 to 127 edges 8 to 16
// round trips each; with those of 32 and more shared, evenly cut, 30 us.  A graph of 4096 nodes and 64 thousand edges, 4 heads of 16: forward
// 16.0 -> 10.9, backward 22.5 -> 16.0 us.  (In launches of millions of edges sharing costs: 47 bf16 values, 6 M edges, rows from
// 32 on shared, backward 3 to 9% slower.)  At most 1024 rows: each takes a workgroup, and about as many run at once.
int shared_class(const int* hist, int64_t edges, int long_class)
{
    int c = sar::kSharedClassLeast;
    while (c < long_class && ((int64_t)1 << (c - 1)) < edges / 4096) ++c;
    for (; c < sar::kLongClassBlock && c < long_class; ++c) {
        int64_t n = 0;
        for (int k = c; k < sar::kNumClasses; ++k) n += hist[k];
        if (n <= 1024) return c;
    }
    return long_class;
}

ClassLayout layout_from_hist(const int* hist, int64_t offset, int floor_class, int64_t edges)
{
    const int long_class = pick_long_class(hist, floor_class), shared = shared_class(hist, edges, long_class);
    ClassLayout L;
    int64_t run = offset;
    for (int c = sar::kNumClasses - 1; c >= 1; --c) {
        L.start[c] = (int)run;
        run += hist[c];
        L.n_rows += hist[c];
        if (c >= long_class) L.n_long += hist[c];
        if (c >= shared) L.n_shared += hist[c];
        if (c > sar::kNarrowMaxClass) L.n_wide += hist[c];
    }
    L.start[0] = (int)run;
    return L;
}

// ------------------------------------- sources of one edge, destination-major

struct SingleTabs {
    const int32_t* t_indptr[SAR_MAX_BLOCKS];
    const int32_t* t_rank[SAR_MAX_BLOCKS];   // null: the source's own id is its row
};

// The entries of the all-blocks index whose source has no other edge in its block, in the order
// of the index (ascending destination, block after block inside a destination): (destination,
// tagged source, row of the source in its block's error).  One wavefront per destination row,
// twice: FILL = false counts a row's entries into cnt[r], FILL = true writes them from off[r] on.
template <bool FILL>
__global__ __launch_bounds__(kThreads) void k_single_list(SingleTabs tabs, const int32_t* __restrict__ f_indptr,
                                                          const uint32_t* __restrict__ f_indices, int64_t n_dst,
                                                          int tag_shift, int32_t* __restrict__ cnt,
                                                          const int32_t* __restrict__ off,
                                                          int64_t n_single, int32_t* __restrict__ s_dst,
                                                          uint32_t* __restrict__ s_src, int32_t* __restrict__ s_row)
{
    __shared__ sar::GlobalPtr<const int32_t> ip[SAR_MAX_BLOCKS];
    __shared__ sar::GlobalPtr<const int32_t> rk[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        ip[threadIdx.x] = tabs.t_indptr[threadIdx.x];
        rk[threadIdx.x] = tabs.t_rank[threadIdx.x];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const uint32_t mask = (1u << tag_shift) - 1u;
    const int64_t n_waves = (int64_t)gridDim.x * (kThreads / 64);
    for (int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); r < n_dst; r += n_waves) {
        const int beg = f_indptr[r], end = f_indptr[r + 1];
        int at = FILL ? off[r] : 0;
        for (int c = beg; c < end; c += 64) {
            uint32_t id = 0;
            int q = 0, j = 0;
            bool single = false;
            if (c + lane < end) {
                id = f_indices[c + lane];
                q = (int)(id >> tag_shift);
                j = (int)(id & mask);
                single = ip[q][j + 1] - ip[q][j] == 1;
            }
            const unsigned long long votes = __ballot(single);
            if (FILL && single) {
                const int mine = at + __popcll(votes & ((1ull << lane) - 1ull));
                if (mine < n_single) {
                    s_dst[mine] = (int32_t)r;
                    s_src[mine] = id;
                    s_row[mine] = rk[q] ? rk[q][j] : j;
                }
            }
            at += __popcll(votes);
        }
        if (!FILL && lane == 0) cnt[r] = at;
    }
}

// ------------------------------------------- source side of the blocks

// t_indptr of every block (its sources' offsets, from 0) and flags[j] = 1 if a source has an edge
__global__ __launch_bounds__(kThreads) void k_source_offsets(const BlkDev* __restrict__ blk, const int32_t* __restrict__ off,
                                                             int32_t* __restrict__ flags)
{
    const BlkDev& B = blk[blockIdx.y];
    for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k <= B.n_src; k += (int64_t)gridDim.x * kThreads) {
        const int32_t o = off[B.coff + k];
        B.t_indptr[k] = o - (int32_t)B.nnz0;
        if (k < B.n_src)
            flags[B.coff + k] = off[B.coff + k + 1] > o ? 1 : 0;
        else if (blockIdx.y == gridDim.y - 1)
            flags[B.coff + k] = 0;           // closes the scan
    }
}

// t_rank[j] = touched sources of the block below j (pos: of all blocks), and the ascending touched list
__global__ __launch_bounds__(kThreads) void k_source_ranks(const BlkDev* __restrict__ blk, const int32_t* __restrict__ pos,
                                                           int32_t* __restrict__ touched_all)
{
    const BlkDev& B = blk[blockIdx.y];
    const int32_t base = pos[B.coff];
    for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k <= B.n_src; k += (int64_t)gridDim.x * kThreads) {
        const int32_t at = pos[B.coff + k];
        B.t_rank[k] = at - base;
        if (k < B.n_src && pos[B.coff + k + 1] > at) touched_all[at] = (int32_t)k;
    }
}

// ------------------------------------------------- all-blocks (fused) index

__global__ __launch_bounds__(kThreads) void k_total_degree(const BlkDev* __restrict__ blk, int P, int64_t n_dst,
                                                           int32_t* __restrict__ deg)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i <= n_dst;
         i += (int64_t)gridDim.x * kThreads) {
        int d = 0;
        if (i < n_dst)
            for (int q = 0; q < P; ++q) d += blk[q].indptr[i + 1] - blk[q].indptr[i];
        deg[i] = d;   // deg[n_dst] = 0 closes the scan
    }
}

// Rows of the all-blocks index: a row's sources block after block, tagged with the block.  A wavefront takes `rows` rows
// from as many parts of the list (neighbouring rows are often long together), as many as have a lane each for every block, 4 at
// most: a lane reads its block's range of its row, then 8 lanes copy a range, 32 ranges of one turn under way at once, and
// the whole wavefront the ranges of more than 64.  (One row at a time, 8 lanes to a range of any length: 306 thousand rows
// of 50 in 8 blocks, up to 11 thousand in one, 94 us, now 56.)
__global__ __launch_bounds__(kThreads) void k_fused_copy(const BlkDev* __restrict__ blk, int P, int rows, int64_t n_dst,
                                                         const int32_t* __restrict__ f_indptr, int tag_shift,
                                                         uint32_t* __restrict__ f_indices)
{
    constexpr int kTurn = 4;
    __shared__ sar::GlobalPtr<const int32_t> s_indices[SAR_MAX_BLOCKS];
    __shared__ sar::GlobalPtr<const int32_t> s_indptr[SAR_MAX_BLOCKS];
    if ((int)threadIdx.x < P) {
        s_indices[threadIdx.x] = blk[threadIdx.x].indices;
        s_indptr[threadIdx.x] = blk[threadIdx.x].indptr;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, sub = lane & 7, grp = lane >> 3, ranges = rows * P;
    const int my_row = lane / P, my_q = lane - my_row * P;
    const int64_t part = (n_dst + rows - 1) / rows, step = ((int64_t)gridDim.x * kThreads) >> 6;
    for (int64_t i0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6; i0 < part; i0 += step) {
        const int64_t i = i0 + my_row * part;
        int beg = 0, len = 0, pos = 0;
        if (lane < ranges && i < n_dst) {
            beg = s_indptr[my_q][i];
            len = s_indptr[my_q][i + 1] - beg;
            pos = f_indptr[i];
        }
        int at = len;                          // sum of the row's lengths up to this block's
        for (int o = 1; o < P; o <<= 1) {
            const int x = __shfl_up(at, o);
            if (my_q >= o) at += x;
        }
        at += pos - len;
        constexpr int kLong = 64;
        for (uint64_t todo = __ballot(len > kLong); todo; todo &= todo - 1) {
            const int r = __ffsll((long long)todo) - 1;
            const int b = __shfl(beg, r), n = __shfl(len, r), a = __shfl(at, r), q = __shfl(my_q, r);
            const int32_t* const from = s_indices[q] + b;
            for (int e0 = lane; e0 < n; e0 += 64 * kTurn) {
                uint32_t x[kTurn];
#pragma unroll
                for (int u = 0; u < kTurn; ++u) x[u] = (uint32_t)from[min(e0 + 64 * u, n - 1)];
#pragma unroll
                for (int u = 0; u < kTurn; ++u)
                    if (e0 + 64 * u < n) f_indices[a + e0 + 64 * u] = x[u] | ((uint32_t)q << tag_shift);
            }
        }
        for (int r0 = 0; r0 < ranges; r0 += 8 * kTurn) {
            int b[kTurn], n[kTurn], a[kTurn], q[kTurn];
            uint32_t x[kTurn];
#pragma unroll
            for (int u = 0; u < kTurn; ++u) {
                const int r = r0 + u * 8 + grp, from = min(r, 63);
                b[u] = __shfl(beg, from);
                n[u] = __shfl(len, from);
                a[u] = __shfl(at, from);
                q[u] = __shfl(my_q, from);
                if (r >= ranges || n[u] > kLong) n[u] = 0;
                if (sub < n[u]) x[u] = (uint32_t)s_indices[q[u]][b[u] + sub];
            }
#pragma unroll
            for (int u = 0; u < kTurn; ++u) {
                const uint32_t tag = (uint32_t)q[u] << tag_shift;
                if (sub < n[u]) f_indices[a[u] + sub] = x[u] | tag;
                for (int e = sub + 8; e < n[u]; e += 8) f_indices[a[u] + e] = (uint32_t)s_indices[q[u]][b[u] + e] | tag;
            }
        }
    }
}

// ends[2q], ends[2q+1] = first and last offset of block q
__global__ __launch_bounds__(kThreads) void k_block_ends(const BlkDev* __restrict__ blk, int P, int64_t n_dst,
                                                         int32_t* __restrict__ ends)
{
    const int q = threadIdx.x;
    if (q < P) {
        ends[2 * q] = blk[q].indptr[0];
        ends[2 * q + 1] = blk[q].indptr[n_dst];
    }
}

__global__ __launch_bounds__(kThreads) void k_check_columns(const BlkDev* __restrict__ blk, int64_t n_dst,
                                                            int* __restrict__ err)
{
    const BlkDev& B = blk[blockIdx.y];
    for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < B.nnz;
         k += (int64_t)gridDim.x * kThreads)
        if (B.indices[k] < 0 || B.indices[k] >= B.n_src) atomicOr(err, 4);
    for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < n_dst;
         k += (int64_t)gridDim.x * kThreads)
        if (B.indptr[k + 1] < B.indptr[k]) atomicOr(err, 8);
}

unsigned grid_for(int64_t items, int per_block = kThreads, int64_t cap = 1 << 20)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + per_block - 1) / per_block, cap));
}

template <typename T>
int own(sar_blocks* h, T** out, int64_t count)
{
    void* p = nullptr;
    const size_t size = Pool::round(std::max<int64_t>(count, 1) * sizeof(T));
    h->owned.reserve(h->owned.size() + 1);
    SAR_TRY(pool().take(h->device, &p, size));
    h->owned.emplace_back(p, size);
    *out = static_cast<T*>(p);
    return SAR_OK;
}

int bits_for(int64_t n)
{
    int b = 0;
    while (((int64_t)1 << b) < n) ++b;
    return b;
}

// Bits by which a source's block is tagged above its local id.
int set_tag_shift(sar_blocks* h, int64_t n_src_max)
{
    h->tag_shift = std::max(1, bits_for(std::max<int64_t>(n_src_max, 2)));
    if (h->tag_shift + bits_for(h->P) > 32)
        return sar::fail(SAR_ERR_UNSUPPORTED, "P=%d blocks of up to %lld sources do not fit a 32-bit tagged index",
                         h->P, (long long)n_src_max);
    return SAR_OK;
}

template <typename Fn>
int allow_lds(Fn fn, size_t bytes)
{
    SAR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    return SAR_OK;
}

// Where things stand in a call's pinned page: the newest report, the blocks, the lists' cursors.
constexpr size_t kReportBytes = (4 + (2 * SAR_MAX_PARTS + 2) * sar::kNumClasses + 15) / 16 * 16 * sizeof(int32_t);
constexpr size_t kBlkBytes = SAR_MAX_PARTS * sizeof(BlkDev);
static_assert(2 * kReportBytes + kBlkBytes <= Pool::kHostPage && kReportBytes % alignof(BlkDev) == 0, "");

// Has the stream report flags[0..3] and in[k * step], k < n; without `wait` the stream has to be waited for before `*report` is read.
int send_report(const int32_t* in, int64_t step, int n, const int* flags, bool wait, const int32_t** report,
                DeviceTemps& tmp, hipStream_t st)
{
    void* page = nullptr;
    SAR_TRY(tmp.host(&page));
    k_report<<<1, kThreads, 0, st>>>(in, step, n, flags, static_cast<int32_t*>(page));
    SAR_LAUNCH_CHECK();
    if (wait) SAR_HIP(hipStreamSynchronize(st));
    *report = static_cast<const int32_t*>(page);
    return SAR_OK;
}

int check_flags(int err)
{
    if (err & 1) return sar::fail(SAR_ERR_INVALID_ARG, "part[] holds a value outside [0,P)");
    if (err & 2) return sar::fail(SAR_ERR_INVALID_ARG, "edge list holds a node id outside [0,N)");
    if (err & 4) return sar::fail(SAR_ERR_INVALID_ARG, "indices[] holds a column outside [0,n_src)");
    if (err & 8) return sar::fail(SAR_ERR_INVALID_ARG, "indptr[] is not non-decreasing");
    if (err & 16) return sar::fail(SAR_ERR_INVALID_ARG, "dst_ids[] holds a row outside [0,n_dst)");
    return SAR_OK;
}

// Scratch of a builder call that its two groupings share.
struct PairScratch {
    void* pairs = nullptr;
    size_t bytes = 0;
    int take(DeviceTemps& tmp, size_t want)
    {
        if (want <= bytes) return SAR_OK;
        char* p = nullptr;
        SAR_TRY(tmp.alloc(&p, (int64_t)want));
        pairs = p;
        bytes = want;
        return SAR_OK;
    }
};

// The pairs of the n_keys keys of a pass are in their buckets: off[0..n_keys] their offsets (from `base`
// on), and their values in order.
template <typename PairT>
int finish_buckets(const BucketPlan& plan, const PairT* pairs, const int32_t* counts, int64_t n_keys, int vbits,
                   int32_t base, int32_t* off, int32_t* values, DeviceTemps& tmp, hipStream_t st)
{
    int32_t* list = nullptr;
    SAR_TRY(tmp.alloc(&list, plan.n_buckets() + 2));
    int* count = list + plan.n_buckets();                // buckets listed, and shares of them taken
    const size_t slots = ((size_t)1 << plan.w) * sizeof(int), lds = slots + kBucketCap * sizeof(int32_t);
    const Deal deal{plan.nb};
    k_bucket_keys<PairT><<<(unsigned)plan.n_buckets(), kBucketThreads, slots, st>>>(pairs, counts, plan.n_tiles, plan.w,
                                                                                   deal, n_keys, vbits, off, count);
    SAR_LAUNCH_CHECK();
    SAR_TRY(exclusive_scan(off, off, n_keys + 1, st, tmp, base));
    SAR_TRY(allow_lds(k_bucket_finish<PairT>, lds));
    k_bucket_finish<PairT><<<(unsigned)plan.n_buckets(), kBucketThreads, lds, st>>>(
        pairs, counts, plan.n_tiles, plan.w, deal, n_keys, vbits, off, values, list, count);
    SAR_LAUNCH_CHECK();
    k_sort_buckets<<<(unsigned)std::min(plan.n_buckets() * kSortShares, 1024), kThreads, 0, st>>>(
        off, values, plan.w, deal, n_keys, list, count, count + 1);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// Builds what `flags` asks for on top of per-block CSR arrays already in h->blk.
int derive(sar_blocks* h, DeviceTemps& tmp, PairScratch& scratch, hipStream_t st)
{
    const int P = h->P;
    const int64_t n_dst = h->n_dst;
    if ((h->flags & SAR_BUILD_COMPACT) && !(h->flags & SAR_BUILD_TRANSPOSE))
        return sar::fail(SAR_ERR_INVALID_ARG, "SAR_BUILD_COMPACT needs SAR_BUILD_TRANSPOSE");
    const bool transpose = (h->flags & SAR_BUILD_TRANSPOSE) != 0, fused = (h->flags & SAR_BUILD_FUSED) != 0;

    int64_t nnz_total = 0, n_src_total = 0, n_src_max = 0, nnz_max = 0;
    for (auto& b : h->blk) {
        nnz_total += b.nnz;
        n_src_total += b.n_src;
        n_src_max = std::max(n_src_max, b.n_src);
        nnz_max = std::max(nnz_max, b.nnz);
    }
    if (n_src_total >= ((int64_t)1 << 31))
        return sar::fail(SAR_ERR_UNSUPPORTED, "the %d source partitions hold %lld nodes in total; a handle's work "
                         "lists index fewer than 2^31", P, (long long)n_src_total);
    SAR_TRY(set_tag_shift(h, n_src_max));
    if (fused && nnz_total >= ((int64_t)1 << 31))
        return sar::fail(SAR_ERR_UNSUPPORTED, "all-blocks index needs fewer than 2^31 edges, got %lld",
                         (long long)nnz_total);
    if (transpose && nnz_total >= ((int64_t)1 << 31))
        return sar::fail(SAR_ERR_UNSUPPORTED, "transpose needs fewer than 2^31 edges in total, got %lld",
                         (long long)nnz_total);

    // ---- arrays whose sizes are known; the launch lists at the most they can hold
    const int64_t rows_most = std::min<int64_t>(nnz_total, (int64_t)P * n_dst);
    int32_t *rows_all = nullptr, *t_indices_all = nullptr, *t_indptr_all = nullptr, *t_rank_all = nullptr;
    int32_t *t_rows_all = nullptr, *touched_all = nullptr;
    SAR_TRY(own(h, &h->deg, n_dst + 1));
    SAR_TRY(own(h, &rows_all, rows_most));
    if (fused) {
        SAR_TRY(own(h, &h->f_indptr, n_dst + 1));
        SAR_TRY(own(h, &h->f_indices, nnz_total));
        SAR_TRY(own(h, &h->f_rows, n_dst));
    }
    if (transpose) {
        SAR_TRY(own(h, &t_indices_all, nnz_total));
        SAR_TRY(own(h, &t_indptr_all, n_src_total + P));
        SAR_TRY(own(h, &t_rank_all, n_src_total + P));
        // the launch lists also carry the sources without edges (last), so that the
        // backward kernels write every row of dZ_q; `touched` holds only the others
        SAR_TRY(own(h, &t_rows_all, n_src_total));
        SAR_TRY(own(h, &h->ft_rows, n_src_total));
        SAR_TRY(own(h, &touched_all, std::min(n_src_total, nnz_total)));
    }

    const BucketPlan plan = plan_buckets(std::min(kKeysPerPass, std::max<int64_t>(n_src_total, 1)), nnz_total);
    void* page = nullptr;
    SAR_TRY(tmp.host(&page, kReportBytes));
    BlkDev* const blk = static_cast<BlkDev*>(page);
    int64_t coff = 0, nnz0 = 0, tiles = 0, s_tiles = 0;
    for (int q = 0; q < P; ++q) {
        Block& b = h->blk[q];
        if (transpose) {
            b.t_indptr = t_indptr_all + coff + q;
            b.t_rank = t_rank_all + coff + q;
            b.t_indices = t_indices_all + nnz0;
            b.t_rows = t_rows_all + coff;
        }
        blk[q] = BlkDev{b.indptr, b.indices, b.n_src, coff, b.nnz, nnz0, tiles, s_tiles, nullptr,
                        reinterpret_cast<uint32_t*>(b.t_rows), b.t_indptr, b.t_rank};
        coff += b.n_src;
        nnz0 += b.nnz;
        tiles += (b.nnz + plan.tile - 1) / plan.tile;
        if (transpose) s_tiles += (b.n_src + kPlaceRows - 1) / kPlaceRows;
    }
    BlkDev* blk_d = nullptr;
    const int C = sar::kNumClasses, n_hist = (2 * P + 2) * C;
    int *starts_d = nullptr, *class_counts = nullptr;
    int32_t *col_off = nullptr, *counts = nullptr, *pos = nullptr;      // (the transpose's)
    ListIn in{nullptr, h->f_indptr, n_dst, P, (n_dst + kPlaceRows - 1) / kPlaceRows, s_tiles, fused};
    SAR_TRY(tmp.alloc_parts({tmp.part(&blk_d, P), tmp.part(&starts_d, n_hist), tmp.part(&class_counts, in.size() + 1),
                             tmp.part(&col_off, transpose ? n_src_total + 1 : 0), tmp.part(&pos, transpose ? n_src_total + 1 : 0),
                             tmp.part(&counts, transpose ? (int64_t)plan.n_buckets() * std::max<int64_t>(tiles, 1) + 1 : 0)}));
    in.blk = blk_d;
    SAR_HIP(hipMemcpyAsync(blk_d, blk, P * sizeof(BlkDev), hipMemcpyHostToDevice, st));

    // total in-degree |N(i)|, and the tiles' rows by class
    k_total_degree<<<grid_for(n_dst + 1), kThreads, 0, st>>>(blk_d, P, n_dst, h->deg);
    SAR_LAUNCH_CHECK();
    const dim3 g_rows((unsigned)std::max<int64_t>(1, in.t_rows), P), g_all(g_rows.x, 1), g_tiles((unsigned)std::max<int64_t>(1, in.t_src), 1);
    const dim3 g_src(grid_for(n_src_max + 1, kThreads, std::max(1, 4096 / P)), P);
    const bool lists = n_dst > 0, src_lists = transpose && n_src_max > 0;
    if (lists) {
        k_class_count<<<g_rows, kThreads, 0, st>>>(in, Lists::kRows, class_counts);
        SAR_LAUNCH_CHECK();
    } else {
        SAR_HIP(hipMemsetAsync(class_counts + in.size(), 0, sizeof(int32_t), st));
    }

    // ---- all-blocks destination-major index
    if (fused) {
        SAR_TRY(exclusive_scan(h->deg, h->f_indptr, n_dst + 1, st, tmp));
        const int rows = std::min(4, 64 / P);       // P <= 64
        k_fused_copy<<<grid_for((n_dst + rows - 1) / rows * 64), kThreads, 0, st>>>(blk_d, P, rows, n_dst, h->f_indptr,
                                                                                    h->tag_shift, h->f_indices);
        SAR_LAUNCH_CHECK();
        if (lists) {
            k_class_count<<<g_all, kThreads, 0, st>>>(in, Lists::kAllRows, class_counts);
            SAR_LAUNCH_CHECK();
        }
    }

    // ---- source-major transpose of every block
    if (transpose) {
        const int vbits = bits_for(std::max<int64_t>(n_dst, 1));
        const bool narrow = plan.w + vbits <= 32;
        SAR_TRY(scratch.take(tmp, (size_t)nnz_total * (narrow ? 4 : 8)));
        BucketPlan pass = plan;
        pass.n_tiles = tiles;
        int32_t base = 0;
        if (nnz_total == 0) SAR_HIP(hipMemsetAsync(col_off, 0, (n_src_total + 1) * sizeof(int32_t), st));
        for (int64_t key0 = 0; key0 < n_src_total && nnz_total > 0; key0 += kKeysPerPass) {
            const int64_t nk = std::min(kKeysPerPass, n_src_total - key0);
            const bool last = key0 + nk == n_src_total;
            const int64_t n_counts = (int64_t)pass.n_buckets() * tiles + 1;
            const size_t lds = pass.n_buckets() * sizeof(int);
            const Deal deal{pass.nb};
            SAR_TRY(allow_lds(k_block_count, lds));
            k_block_count<<<(unsigned)tiles, kBucketThreads, lds, st>>>(blk_d, P, pass.tile, tiles, key0, nk, deal,
                                                                        counts);
            SAR_LAUNCH_CHECK();
            SAR_TRY(exclusive_scan(counts, counts, n_counts, st, tmp));
            auto place = [&](auto* pairs) -> int {
                using PairT = std::remove_pointer_t<decltype(pairs)>;
                if (sizeof(PairT) == 4 && pass.nb <= kStagedBits) {
                    SAR_TRY(allow_lds(k_block_scatter_staged, kStagedLds));
                    k_block_scatter_staged<<<(unsigned)tiles, kStageThreads, kStagedLds, st>>>(
                        blk_d, P, n_dst, pass.tile, tiles, key0, nk, deal, vbits, counts, (uint32_t*)pairs);
                } else {
                    SAR_TRY(allow_lds(k_block_scatter<PairT>, lds));
                    k_block_scatter<PairT><<<(unsigned)tiles, kBucketThreads, lds, st>>>(
                        blk_d, P, n_dst, pass.tile, tiles, key0, nk, deal, vbits, counts, pairs);
                }
                SAR_LAUNCH_CHECK();
                return finish_buckets<PairT>(pass, pairs, counts, nk, vbits, base, col_off + key0, t_indices_all, tmp, st);
            };
            SAR_TRY(narrow ? place(static_cast<uint32_t*>(scratch.pairs)) : place(static_cast<uint64_t*>(scratch.pairs)));
            if (!last) {
                int32_t in_pass = 0;
                SAR_HIP(hipMemcpyAsync(&in_pass, counts + n_counts - 1, sizeof(int32_t), hipMemcpyDeviceToHost, st));
                SAR_HIP(hipStreamSynchronize(st));
                base += in_pass;
            }
        }
        // per-block offsets (from 0), the classes of the sources, ranks of the touched ones
        k_source_offsets<<<g_src, kThreads, 0, st>>>(blk_d, col_off, pos);
        SAR_LAUNCH_CHECK();
        if (src_lists) {
            k_class_count<<<g_tiles, kThreads, 0, st>>>(in, Lists::kSources, class_counts);
            SAR_LAUNCH_CHECK();
        }
        SAR_TRY(exclusive_scan(pos, pos, n_src_total + 1, st, tmp));
        k_source_ranks<<<g_src, kThreads, 0, st>>>(blk_d, pos, touched_all);
        SAR_LAUNCH_CHECK();
    }

    // ---- launch lists, longest class first
    SAR_TRY(exclusive_scan(class_counts, class_counts, in.size() + 1, st, tmp));
    SAR_TRY(tmp.host(&page));
    const int32_t* report = static_cast<const int32_t*>(page);
    k_class_totals<<<1, kThreads, 0, st>>>(in, transpose, class_counts, static_cast<int32_t*>(page));
    SAR_LAUNCH_CHECK();
    SAR_HIP(hipStreamSynchronize(st));
    const std::vector<int> hist(report, report + n_hist);
    SAR_TRY(tmp.host(&page, kReportBytes + kBlkBytes));
    int* const cursors = static_cast<int*>(page);
    std::fill(cursors, cursors + n_hist, 0);
    int64_t rows_at = 0, t_rows_at = 0;
    int all_hist[sar::kNumClasses] = {0};
    for (int q = 0; q < P; ++q) {
        Block& b = h->blk[q];
        const int* row_hist = &hist[q * C];
        ClassLayout L = layout_from_hist(row_hist, 0, sar::kLongClassBlock, b.nnz);
        b.n_rows = L.n_rows;
        b.n_long = L.n_long;
        b.n_shared = L.n_shared;
        b.n_rows_wide = L.n_wide;
        for (int c = 1; c < C; ++c)
            if (row_hist[c]) b.hub = (int64_t)1 << (c - 1);
        memcpy(&cursors[q * C], L.start, sizeof(L.start));
        b.rows = rows_all + rows_at;
        blk[q].rows = reinterpret_cast<uint32_t*>(b.rows);
        rows_at += L.n_rows;
        if (transpose) {
            const int* s_hist = &hist[(P + q) * C];
            ClassLayout S = layout_from_hist(s_hist, 0, sar::kLongClassBlock, b.nnz);
            b.n_t_rows = S.n_rows;
            b.n_t_long = S.n_long;
            b.n_t_shared = S.n_shared;
            b.n_t_wide = S.n_wide;
            memcpy(&cursors[(P + q) * C], S.start, sizeof(S.start));
            b.touched = touched_all + t_rows_at;
            t_rows_at += S.n_rows;
            for (int c = 0; c < C; ++c) all_hist[c] += s_hist[c];
        }
    }
    if (fused) {
        ClassLayout L = layout_from_hist(&hist[2 * P * C], 0, sar::kLongClassBlock, nnz_total);
        h->n_f_rows = L.n_rows;
        h->n_f_shared = L.n_shared;
        for (int c = 1; c < C; ++c) {
            if (hist[2 * P * C + c]) h->f_longest = ((int64_t)1 << c) - 1;
            if (c >= sar::kHubClass) h->n_f_hub += hist[2 * P * C + c];
        }
        memcpy(&cursors[2 * P * C], L.start, sizeof(L.start));
    }
    if (transpose) {
        ClassLayout L = layout_from_hist(all_hist, 0, sar::kLongClassBlock, nnz_total);
        h->n_ft_rows = L.n_rows;
        h->n_ft_shared = L.n_shared;
        h->n_ft_wide = L.n_wide;
        for (int c = 1; c < C; ++c)
            if (all_hist[c]) h->ft_longest = ((int64_t)1 << c) - 1;
        memcpy(&cursors[(2 * P + 1) * C], L.start, sizeof(L.start));
    }
    SAR_HIP(hipMemcpyAsync(blk_d, blk, P * sizeof(BlkDev), hipMemcpyHostToDevice, st));
    SAR_HIP(hipMemcpyAsync(starts_d, cursors, n_hist * sizeof(int), hipMemcpyHostToDevice, st));
    if (lists) {
        k_class_place<<<g_rows, kThreads, 0, st>>>(in, Lists::kRows, 0, starts_d, class_counts, nullptr);
        SAR_LAUNCH_CHECK();
    }
    if (fused && lists) {
        k_class_place<<<g_all, kThreads, 0, st>>>(in, Lists::kAllRows, 0, starts_d + 2 * P * C, class_counts,
                                                  reinterpret_cast<uint32_t*>(h->f_rows));
        SAR_LAUNCH_CHECK();
    }
    if (transpose) {
        if (src_lists) {
            k_class_place<<<g_tiles, kThreads, 0, st>>>(in, Lists::kSources, 0, starts_d + P * C, class_counts, nullptr);
            SAR_LAUNCH_CHECK();
            k_class_place<<<g_tiles, kThreads, 0, st>>>(in, Lists::kAllSources, h->tag_shift, starts_d + (2 * P + 1) * C,
                                                        class_counts, h->ft_rows);
            SAR_LAUNCH_CHECK();
        }

        // ---- the sources of one edge, listed from their destinations' side (all-blocks backward):
        // built where they carry at least an eighth of the edges, or on request
        const int64_t n_single = all_hist[1];
        const bool want_singles = (h->flags & SAR_BUILD_SINGLES) ||
                                  (!(h->flags & SAR_BUILD_NO_SINGLES) && n_single * 8 >= nnz_total);
        if (fused && want_singles && n_single > 0) {
            SAR_TRY(own(h, &h->s_dst, n_single));
            SAR_TRY(own(h, &h->s_src, n_single));
            SAR_TRY(own(h, &h->s_row, n_single));
            SingleTabs stabs;
            memset(&stabs, 0, sizeof(stabs));
            for (int q = 0; q < P; ++q) {
                stabs.t_indptr[q] = h->blk[q].t_indptr;
                stabs.t_rank[q] = (h->flags & SAR_BUILD_COMPACT) ? h->blk[q].t_rank : nullptr;
            }
            int32_t *s_cnt = nullptr, *s_off = nullptr;
            SAR_TRY(tmp.alloc_parts({tmp.part(&s_cnt, n_dst + 1), tmp.part(&s_off, n_dst + 1)}));
            SAR_HIP(hipMemsetAsync(s_cnt + n_dst, 0, sizeof(int32_t), st));
            const unsigned g_list = grid_for(n_dst * 64, kThreads, 1 << 16);
            k_single_list<false><<<g_list, kThreads, 0, st>>>(stabs, h->f_indptr, h->f_indices, n_dst, h->tag_shift,
                                                              s_cnt, nullptr, 0, nullptr, nullptr, nullptr);
            SAR_LAUNCH_CHECK();
            SAR_TRY(exclusive_scan(s_cnt, s_off, n_dst + 1, st, tmp));
            SAR_TRY(send_report(s_off + n_dst, 1, 1, nullptr, false, &report, tmp, st));
            k_single_list<true><<<g_list, kThreads, 0, st>>>(stabs, h->f_indptr, h->f_indices, n_dst, h->tag_shift,
                                                             nullptr, s_off, n_single, h->s_dst, h->s_src, h->s_row);
            SAR_LAUNCH_CHECK();
            h->n_single = n_single;
        }
    }
    SAR_HIP(hipStreamSynchronize(st));
    if (h->n_single > 0 && report[4] != h->n_single)
        return sar::fail(SAR_ERR_STATE, "the all-blocks index lists %d sources of one edge, the transposes %lld", report[4],
                         (long long)h->n_single);
    return SAR_OK;
}

int build_from_edges(sar_blocks* h, const void* src, const void* dst, int idx_bytes, int64_t E,
                     const int32_t* part, int64_t N, int P, int p, DeviceTemps& tmp, PairScratch& scratch, hipStream_t st)
{
    int* err_d = nullptr;
    SAR_TRY(tmp.alloc(&err_d, 4));
    unsigned long long* kept_d = reinterpret_cast<unsigned long long*>(err_d + 2);     // reported with the flags
    SAR_HIP(hipMemsetAsync(err_d, 0, 4 * sizeof(int), st));

    // 1. rank of every node inside its partition
    const int64_t n_tiles = std::max<int64_t>(1, (N + kPartTile - 1) / kPartTile);
    int32_t* tile_counts = nullptr;
    uint32_t* code = nullptr;
    uint8_t* owner = nullptr;
    SAR_TRY(tmp.alloc(&tile_counts, (int64_t)P * n_tiles + 1));
    k_part_tile_count<<<(unsigned)n_tiles, kThreads, 0, st>>>(part, N, P, n_tiles, tile_counts, err_d);
    SAR_LAUNCH_CHECK();
    SAR_TRY(exclusive_scan(tile_counts, tile_counts, (int64_t)P * n_tiles + 1, st, tmp));
    std::vector<int32_t> part_first(P + 1);
    const int32_t* report = nullptr;
    SAR_TRY(send_report(tile_counts, n_tiles, P + 1, err_d, true, &report, tmp, st));
    SAR_TRY(check_flags(report[0]));
    std::copy(report + 4, report + 5 + P, part_first.begin());
    const int64_t n_dst = part_first[p + 1] - part_first[p];
    h->n_dst = n_dst;
    h->blk.resize(P);
    int64_t n_src_max = 0;
    for (int q = 0; q < P; ++q) {
        h->blk[q].n_dst = n_dst;
        h->blk[q].n_src = part_first[q + 1] - part_first[q];
        n_src_max = std::max(n_src_max, h->blk[q].n_src);
    }
    SAR_TRY(set_tag_shift(h, n_src_max));
    const int64_t n_rows_all = (int64_t)P * n_dst;
    int32_t* row_off = nullptr;
    SAR_TRY(tmp.alloc_parts({tmp.part(&code, N), tmp.part(&owner, N), tmp.part(&row_off, n_rows_all + 1)}));
    k_local_ids<<<(unsigned)n_tiles, kThreads, 0, st>>>(part, N, P, n_tiles, tile_counts, h->tag_shift, code, owner);
    SAR_LAUNCH_CHECK();

    // 2. the kept edges grouped by (block, destination)
    int32_t *indices_all = nullptr, *indptr_all = nullptr;
    SAR_TRY(own(h, &indptr_all, (int64_t)P * (n_dst + 1)));
    int64_t nnz_total = 0;
    auto group = [&](auto in) -> int {
        const int vbits = h->tag_shift;
        BucketPlan plan = plan_buckets(std::min(kKeysPerPass, std::max<int64_t>(n_rows_all, 1)), E);
        const bool narrow = plan.w + vbits <= 32;
        int32_t* counts = nullptr;
        SAR_TRY(tmp.alloc(&counts, (int64_t)plan.n_buckets() * plan.n_tiles + 1));
        if (n_rows_all <= kKeysPerPass) tmp.alloc_spare((size_t)E * sizeof(uint2));
        int32_t base = 0;
        for (int64_t key0 = 0; key0 < std::max<int64_t>(n_rows_all, 1); key0 += kKeysPerPass) {
            const int64_t nk = std::min(kKeysPerPass, n_rows_all - key0);
            const bool first = key0 == 0, last = key0 + nk >= n_rows_all;
            const int64_t n_counts = (int64_t)plan.n_buckets() * plan.n_tiles + 1;
            const size_t lds = plan.n_buckets() * sizeof(int);
            const Deal deal{plan.nb};
            auto count = [&](auto store) -> int {
                auto fn = k_bucket_count<decltype(in), decltype(store)::value>;
                SAR_TRY(allow_lds(fn, lds));
                fn<<<(unsigned)plan.n_tiles, kBucketThreads, lds, st>>>(in, plan.tile, plan.n_tiles, key0, nk, deal, counts,
                                                                        first ? kept_d : nullptr, static_cast<uint2*>(tmp.spare));
                SAR_LAUNCH_CHECK();
                return SAR_OK;
            };
            SAR_TRY(tmp.spare ? count(std::true_type{}) : count(std::false_type{}));
            SAR_TRY(exclusive_scan(counts, counts, n_counts, st, tmp));
            if (first) {
                unsigned long long kept = 0;
                SAR_TRY(send_report(nullptr, 0, 0, err_d, true, &report, tmp, st));
                SAR_TRY(check_flags(report[0]));
                memcpy(&kept, report + 2, sizeof(kept));
                if (kept >= (1ull << 31))
                    return sar::fail(SAR_ERR_UNSUPPORTED,
                                     "worker %d's share holds %llu in-edges; a handle holds fewer than 2^31", p, kept);
                nnz_total = (int64_t)kept;
                SAR_TRY(tmp.or_without_spare([&] { return own(h, &indices_all, nnz_total); }));
                SAR_TRY(scratch.take(tmp, (size_t)nnz_total * (narrow ? 4 : 8)));
                if (n_rows_all == 0) break;
            }
            auto place = [&](auto* pairs) -> int {
                using PairT = std::remove_pointer_t<decltype(pairs)>;
                auto scatter = [&](auto from) -> int {
                    auto fn = k_bucket_scatter<decltype(from), PairT>;
                    SAR_TRY(allow_lds(fn, lds));
                    fn<<<(unsigned)plan.n_tiles, kBucketThreads, lds, st>>>(from, plan.tile, plan.n_tiles, key0, nk, deal,
                                                                            vbits, counts, pairs);
                    SAR_LAUNCH_CHECK();
                    return SAR_OK;
                };
                SAR_TRY(tmp.spare ? scatter(StoredEdges{static_cast<const uint2*>(tmp.spare), E}) : scatter(in));
                return finish_buckets<PairT>(plan, pairs, counts, nk, vbits, base, row_off + key0, indices_all, tmp, st);
            };
            SAR_TRY(narrow ? place(static_cast<uint32_t*>(scratch.pairs)) : place(static_cast<uint64_t*>(scratch.pairs)));
            if (!last) {
                int32_t in_pass = 0;
                SAR_HIP(hipMemcpyAsync(&in_pass, counts + n_counts - 1, sizeof(int32_t), hipMemcpyDeviceToHost, st));
                SAR_HIP(hipStreamSynchronize(st));
                base += in_pass;
            }
        }
        return SAR_OK;
    };
    if (E > 0) {
        if (idx_bytes == 4)
            SAR_TRY(group(EdgeSource<int32_t>{(const int32_t*)src, (const int32_t*)dst, code, owner, E, N, n_dst, p, h->tag_shift, err_d}));
        else
            SAR_TRY(group(EdgeSource<int64_t>{(const int64_t*)src, (const int64_t*)dst, code, owner, E, N, n_dst, p, h->tag_shift, err_d}));
    }
    if (E == 0 || n_rows_all == 0) {
        SAR_HIP(hipMemsetAsync(row_off, 0, (n_rows_all + 1) * sizeof(int32_t), st));
        if (!indices_all) SAR_TRY(own(h, &indices_all, 0));
    }
    k_make_indptr<<<grid_for((int64_t)P * (n_dst + 1)), kThreads, 0, st>>>(row_off, n_dst, P, indptr_all);
    SAR_LAUNCH_CHECK();
    std::vector<int32_t> block_first(P + 1, 0);
    if (n_dst > 0) {
        SAR_TRY(send_report(row_off, n_dst, P + 1, nullptr, true, &report, tmp, st));
        std::copy(report + 4, report + 5 + P, block_first.begin());
    }
    tmp.drop_spare();      // (its readers are done: the handle's other arrays may take its room)
    for (int q = 0; q < P; ++q) {
        h->blk[q].nnz = block_first[q + 1] - block_first[q];
        h->blk[q].indptr = indptr_all + (int64_t)q * (n_dst + 1);
        h->blk[q].indices = indices_all + block_first[q];
    }
    return SAR_OK;
}

// ------------------------------------------------ destination subsets

// cnt[q n_sub + r] = length of row ids[r] of block q (0 and an error flag for an id out of range)
__global__ __launch_bounds__(kThreads) void k_subset_count(const BlkDev* __restrict__ from, const int32_t* __restrict__ ids,
                                                           int64_t n_sub, int64_t n_dst, int32_t* __restrict__ cnt, int* err)
{
    const int32_t* indptr = from[blockIdx.y].indptr;
    for (int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x; r < n_sub; r += (int64_t)gridDim.x * kThreads) {
        int c = 0;
        const int i = ids[r];
        if (i < 0 || i >= n_dst)
            atomicOr(err, 16);
        else
            c = indptr[i + 1] - indptr[i];
        cnt[(int64_t)blockIdx.y * n_sub + r] = c;
    }
}

// new row r of block q = its old row ids[r], 16 lanes per row
__global__ __launch_bounds__(kThreads) void k_subset_copy(const BlkDev* __restrict__ from,
                                                          const int32_t* __restrict__ ids, int64_t n_sub,
                                                          const int32_t* __restrict__ row_off,
                                                          int32_t* __restrict__ new_indices)
{
    constexpr int kLanes = 16;
    const int32_t* indptr = from[blockIdx.y].indptr;
    const int32_t* indices = from[blockIdx.y].indices;
    const int lane = threadIdx.x & (kLanes - 1);
    const int64_t first = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kLanes;
    const int64_t step = ((int64_t)gridDim.x * kThreads) / kLanes;
    for (int64_t r = first; r < n_sub; r += step) {
        const int i = ids[r];
        const int beg = indptr[i], len = indptr[i + 1] - beg, at = row_off[(int64_t)blockIdx.y * n_sub + r];
        for (int k = lane; k < len; k += kLanes) new_indices[at + k] = indices[beg + k];
    }
}

// Frees the handle's arrays once nothing on its device uses them any more.
void destroy(sar_blocks* h)
{
    if (!h) return;
    int current = h->device;
    (void)hipGetDevice(&current);
    if (current != h->device) (void)hipSetDevice(h->device);
    if (!h->owned.empty()) (void)hipDeviceSynchronize();
    for (auto& p : h->owned) pool().give(h->device, p.first, p.second);
    pool().count_handle(h->device, -1);
    if (current != h->device) (void)hipSetDevice(current);
    delete h;
}

// A handle on the current device.
int new_handle(sar_blocks** out)
{
    sar_blocks* h = new (std::nothrow) sar_blocks();
    if (!h) return sar::fail(SAR_ERR_HIP, "out of host memory");
    const hipError_t e = hipGetDevice(&h->device);
    if (e != hipSuccess) {
        delete h;
        return sar::fail(SAR_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
    }
    pool().count_handle(h->device, +1);
    *out = h;
    return SAR_OK;
}

// What fn returns; a host allocation that fails in it becomes an error code instead of an exception at the C boundary.
template <typename Fn>
int guarded(Fn&& fn)
{
    try {
        return fn();
    } catch (const std::bad_alloc&) {
        return sar::fail(SAR_ERR_HIP, "out of host memory");
    }
}

}  // namespace

namespace {
constexpr int kKnownFlags = SAR_BUILD_TRANSPOSE | SAR_BUILD_FUSED | SAR_BUILD_SKIP_UNTOUCHED | SAR_BUILD_COMPACT |
                            SAR_BUILD_SINGLES | SAR_BUILD_NO_SINGLES;
}

extern "C" int sar_blocks_build(const void* src, const void* dst, int idx_bytes, int64_t E,
                                const int32_t* part, int64_t N, int P, int p, int flags, void* stream,
                                sar_blocks_t** out)
{
    SAR_CHECK_ARG(out != nullptr, "out is null");
    *out = nullptr;
    SAR_CHECK_ARG(idx_bytes == 4 || idx_bytes == 8, "idx_bytes must be 4 or 8, got %d", idx_bytes);
    SAR_CHECK_ARG(E >= 0 && N > 0, "need E >= 0 and N > 0 (E=%lld, N=%lld)", (long long)E, (long long)N);
    SAR_CHECK_ARG(E == 0 || (src && dst), "src/dst is null");
    SAR_CHECK_ARG(part != nullptr, "part is null");
    SAR_CHECK_ARG(P >= 1 && p >= 0 && p < P, "need 0 <= p < P, got p=%d P=%d", p, P);
    SAR_CHECK_ARG((flags & ~kKnownFlags) == 0, "unknown flags 0x%x", flags);
    if (P > SAR_MAX_PARTS)
        return sar::fail(SAR_ERR_UNSUPPORTED, "P=%d exceeds SAR_MAX_PARTS=%d", P, SAR_MAX_PARTS);
    if (P > SAR_MAX_BLOCKS && (flags & SAR_BUILD_FUSED))
        return sar::fail(SAR_ERR_UNSUPPORTED,
                         "P=%d exceeds SAR_MAX_BLOCKS=%d, the most an all-blocks call takes: build without "
                         "SAR_BUILD_FUSED and use the per-block calls", P, SAR_MAX_BLOCKS);
    if (N >= ((int64_t)1 << 31))
        return sar::fail(SAR_ERR_UNSUPPORTED, "N must be below 2^31 (32-bit node ids inside the handle)");
    sar_blocks* h = nullptr;
    SAR_TRY(guarded([&] { return new_handle(&h); }));
    h->P = P;
    h->flags = flags;
    hipStream_t st = sar::as_stream(stream);
    auto body = [&]() -> int {       // the scratch goes back before a failed call's handle, the last one maybe, does
        DeviceTemps tmp(st, h->device);
        PairScratch scratch;
        SAR_TRY(build_from_edges(h, src, dst, idx_bytes, E, part, N, P, p, tmp, scratch, st));
        return derive(h, tmp, scratch, st);
    };
    int rc = guarded(body);
    if (rc != SAR_OK) {
        destroy(h);
        return rc;
    }
    *out = h;
    return SAR_OK;
}

extern "C" int sar_blocks_wrap(int P, int64_t n_dst, const int64_t* n_src, const int32_t* const* indptr,
                               const int32_t* const* indices, int flags, void* stream, sar_blocks_t** out)
{
    SAR_CHECK_ARG(out != nullptr, "out is null");
    *out = nullptr;
    SAR_CHECK_ARG(P >= 1 && n_dst >= 0, "need P >= 1 and n_dst >= 0");
    SAR_CHECK_ARG(n_src && indptr && indices, "n_src/indptr/indices is null");
    SAR_CHECK_ARG((flags & ~kKnownFlags) == 0, "unknown flags 0x%x", flags);
    if (P > SAR_MAX_PARTS)
        return sar::fail(SAR_ERR_UNSUPPORTED, "P=%d exceeds SAR_MAX_PARTS=%d", P, SAR_MAX_PARTS);
    if (P > SAR_MAX_BLOCKS && (flags & SAR_BUILD_FUSED))
        return sar::fail(SAR_ERR_UNSUPPORTED,
                         "P=%d exceeds SAR_MAX_BLOCKS=%d, the most an all-blocks call takes: build without "
                         "SAR_BUILD_FUSED and use the per-block calls", P, SAR_MAX_BLOCKS);
    for (int q = 0; q < P; ++q) {
        SAR_CHECK_ARG(indptr[q] != nullptr, "indptr[%d] is null", q);
        SAR_CHECK_ARG(n_src[q] >= 0 && n_src[q] < ((int64_t)1 << 31), "n_src[%d] out of range", q);
    }
    SAR_CHECK_ARG(n_dst < ((int64_t)1 << 31), "n_dst must be below 2^31");
    hipStream_t st = sar::as_stream(stream);
    sar_blocks* h = nullptr;
    SAR_TRY(guarded([&] { return new_handle(&h); }));
    h->P = P;
    h->n_dst = n_dst;
    h->flags = flags;
    auto body = [&]() -> int {
        h->blk.resize(P);
        DeviceTemps tmp(st, h->device);
        PairScratch scratch;
        int* err_d = nullptr;
        int32_t* ends_d = nullptr;
        BlkDev* blk_d = nullptr;
        SAR_TRY(tmp.alloc(&err_d, 4));
        SAR_TRY(tmp.alloc(&ends_d, 2 * P));
        SAR_TRY(tmp.alloc(&blk_d, P));
        SAR_HIP(hipMemsetAsync(err_d, 0, 4 * sizeof(int), st));
        std::vector<BlkDev> blk(P);
        std::vector<int32_t> ends(2 * P);
        for (int q = 0; q < P; ++q) {
            Block& b = h->blk[q];
            b.n_dst = n_dst;
            b.n_src = n_src[q];
            b.indptr = indptr[q];
            b.indices = indices[q];
            blk[q] = BlkDev{indptr[q], indices[q], n_src[q], 0, 0, 0, 0, 0, nullptr, nullptr, nullptr, nullptr};
        }
        SAR_HIP(hipMemcpyAsync(blk_d, blk.data(), P * sizeof(BlkDev), hipMemcpyHostToDevice, st));
        k_block_ends<<<1, kThreads, 0, st>>>(blk_d, P, n_dst, ends_d);
        SAR_LAUNCH_CHECK();
        SAR_HIP(hipMemcpyAsync(ends.data(), ends_d, 2 * P * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        SAR_HIP(hipStreamSynchronize(st));
        int64_t most = n_dst;
        for (int q = 0; q < P; ++q) {
            SAR_CHECK_ARG(ends[2 * q] == 0 && ends[2 * q + 1] >= 0, "indptr[%d] must start at 0 and end >= 0", q);
            blk[q].nnz = h->blk[q].nnz = ends[2 * q + 1];
            SAR_CHECK_ARG(blk[q].nnz == 0 || indices[q] != nullptr, "indices[%d] is null", q);
            most = std::max(most, blk[q].nnz);
        }
        SAR_HIP(hipMemcpyAsync(blk_d, blk.data(), P * sizeof(BlkDev), hipMemcpyHostToDevice, st));
        k_check_columns<<<dim3(grid_for(most, kThreads, std::max(1, 4096 / P)), P), kThreads, 0, st>>>(blk_d, n_dst, err_d);
        SAR_LAUNCH_CHECK();
        const int32_t* report = nullptr;
        SAR_TRY(send_report(nullptr, 0, 0, err_d, true, &report, tmp, st));
        SAR_TRY(check_flags(report[0]));
        return derive(h, tmp, scratch, st);
    };
    int rc = guarded(body);
    if (rc != SAR_OK) {
        destroy(h);
        return rc;
    }
    *out = h;
    return SAR_OK;
}

extern "C" int sar_blocks_info(const sar_blocks_t* b, int* P, int64_t* n_dst)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    if (P) *P = b->P;
    if (n_dst) *n_dst = b->n_dst;
    return SAR_OK;
}

extern "C" int sar_blocks_singles(const sar_blocks_t* b, int64_t* n, const int32_t** dst, const uint32_t** src,
                                  const int32_t** row, int* tag_shift)
{
    SAR_CHECK_ARG(b != nullptr && n != nullptr, "handle or n is null");
    *n = b->n_single;
    if (dst) *dst = b->s_dst;
    if (src) *src = b->s_src;
    if (row) *row = b->s_row;
    if (tag_shift) *tag_shift = b->tag_shift;
    return SAR_OK;
}

extern "C" int sar_blocks_get(const sar_blocks_t* b, int q, sar_block_view* v)
{
    SAR_CHECK_ARG(b != nullptr && v != nullptr, "handle or view is null");
    SAR_CHECK_ARG(q >= 0 && q < b->P, "block %d out of range [0,%d)", q, b->P);
    const Block& k = b->blk[q];
    v->n_dst = k.n_dst;
    v->n_src = k.n_src;
    v->nnz = k.nnz;
    v->indptr = k.indptr;
    v->indices = k.indices;
    v->t_indptr = k.t_indptr;
    v->t_indices = k.t_indices;
    v->rows = k.rows;
    v->n_rows = k.n_rows;
    v->n_long = k.n_long;
    v->t_rows = k.t_rows;
    v->n_t_rows = k.n_t_rows;
    v->n_t_long = k.n_t_long;
    v->touched = k.touched;
    v->t_rank = k.t_rank;
    return SAR_OK;
}

extern "C" int sar_blocks_degree(const sar_blocks_t* b, const int32_t** deg)
{
    SAR_CHECK_ARG(b != nullptr && deg != nullptr, "handle or deg is null");
    *deg = b->deg;
    return SAR_OK;
}

extern "C" int sar_blocks_free(sar_blocks_t* b)
{
    destroy(b);
    return SAR_OK;
}

extern "C" int sar_release_memory(void)
{
    pool().release_all();
    return SAR_OK;
}

extern "C" int sar_blocks_subset(const sar_blocks_t* b, const int32_t* dst_ids, int64_t n_sub, int flags,
                                 void* stream, sar_blocks_t** out)
{
    SAR_CHECK_ARG(out != nullptr, "out is null");
    *out = nullptr;
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_CHECK_ARG(n_sub >= 0 && n_sub < ((int64_t)1 << 31), "n_sub must be in [0, 2^31)");
    SAR_CHECK_ARG(n_sub == 0 || dst_ids != nullptr, "dst_ids is null");
    SAR_CHECK_ARG((flags & ~kKnownFlags) == 0, "unknown flags 0x%x", flags);
    hipStream_t st = sar::as_stream(stream);
    sar_blocks* h = nullptr;
    SAR_TRY(guarded([&] { return new_handle(&h); }));
    h->P = b->P;
    h->n_dst = n_sub;
    h->flags = flags;
    auto body = [&]() -> int {
        h->blk.resize(b->P);
        DeviceTemps tmp(st, h->device);
        PairScratch scratch;
        const int P = b->P;
        const int64_t n_rows_all = (int64_t)P * n_sub;
        int* err_d = nullptr;
        BlkDev* blk_d = nullptr;
        int32_t *row_off = nullptr, *indptr_all = nullptr, *indices_all = nullptr;
        SAR_TRY(tmp.alloc(&err_d, 4));
        SAR_TRY(tmp.alloc(&blk_d, P));
        SAR_TRY(tmp.alloc(&row_off, n_rows_all + 1));
        SAR_TRY(own(h, &indptr_all, (int64_t)P * (n_sub + 1)));
        std::vector<BlkDev> blk(P);
        for (int q = 0; q < P; ++q) {
            const Block& from = b->blk[q];
            h->blk[q].n_dst = n_sub;
            h->blk[q].n_src = from.n_src;
            blk[q] = BlkDev{from.indptr, from.indices, from.n_src, 0, 0, 0, 0, 0, nullptr, nullptr, nullptr, nullptr};
        }
        SAR_HIP(hipMemcpyAsync(blk_d, blk.data(), P * sizeof(BlkDev), hipMemcpyHostToDevice, st));
        SAR_HIP(hipMemsetAsync(err_d, 0, 4 * sizeof(int), st));
        SAR_HIP(hipMemsetAsync(row_off + n_rows_all, 0, sizeof(int32_t), st));
        std::vector<int32_t> block_first(P + 1, 0);
        if (n_sub > 0) {
            k_subset_count<<<dim3(grid_for(n_sub, kThreads, std::max(1, 4096 / P)), P), kThreads, 0, st>>>(
                blk_d, dst_ids, n_sub, b->n_dst, row_off, err_d);
            SAR_LAUNCH_CHECK();
            SAR_TRY(exclusive_scan(row_off, row_off, n_rows_all + 1, st, tmp));
        }
        const int32_t* report = nullptr;
        SAR_TRY(send_report(row_off, n_sub, n_sub > 0 ? P + 1 : 0, err_d, true, &report, tmp, st));
        SAR_TRY(check_flags(report[0]));         // ids are in range beyond this point
        if (n_sub > 0) std::copy(report + 4, report + 5 + P, block_first.begin());
        // the offsets are 32-bit: repeated ids may list more edges than the handle they come from
        for (int q = 0; q < P; ++q)
            if (block_first[q + 1] < block_first[q])
                return sar::fail(SAR_ERR_UNSUPPORTED, "the subset holds 2^31 edges or more");
        SAR_TRY(own(h, &indices_all, block_first[P]));
        if (block_first[P] > 0) {
            k_subset_copy<<<dim3(grid_for(n_sub * 16, kThreads, std::max(1, (1 << 16) / P)), P), kThreads, 0, st>>>(
                blk_d, dst_ids, n_sub, row_off, indices_all);
            SAR_LAUNCH_CHECK();
        }
        k_make_indptr<<<grid_for((int64_t)P * (n_sub + 1)), kThreads, 0, st>>>(row_off, n_sub, P, indptr_all);
        SAR_LAUNCH_CHECK();
        for (int q = 0; q < P; ++q) {
            h->blk[q].nnz = block_first[q + 1] - block_first[q];
            h->blk[q].indptr = indptr_all + (int64_t)q * (n_sub + 1);
            h->blk[q].indices = indices_all + block_first[q];
        }
        return derive(h, tmp, scratch, st);
    };
    int rc = guarded(body);
    if (rc != SAR_OK) {
        destroy(h);
        return rc;
    }
    *out = h;
    return SAR_OK;
}
