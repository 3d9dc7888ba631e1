// Device primitives: device memory pool, exclusive scan of counts and a
// stable LSD radix sort (keys with 32-bit values), all written for wave64.
#include <algorithm>
#include <chrono>
#include <cstring>
#include <thread>

#include "em_internal.h"
#include "em_wave.h"

namespace em {

// ---------------------------------------------------------------- workspace
Workspace::Workspace(int device) : device_(device), bufs_(S_NUM_SLOTS) {}

Workspace::~Workspace()
{
    release();
    if (mailbox_) (void)hipHostFree(mailbox_);
}

void *Workspace::mailbox()
{
    if (arena_base_) return nullptr;
    if (!mailbox_ && hipHostMalloc(&mailbox_, kMailboxBytes, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();  // the copies do without it
        mailbox_ = nullptr;
    }
    return mailbox_;
}

void Workspace::use_arena(void *base, size_t bytes)
{
    release();
    arena_base_ = static_cast<char *>(base);
    arena_cap_ = bytes;
    arena_used_ = 0;
}

size_t Workspace::arena_free() const
{
    return arena_base_ ? arena_cap_ - arena_used_ : ~size_t(0);
}

void Workspace::release()
{
    if (arena_base_) {
        for (Buf &b : bufs_) b = Buf();
        arena_used_ = 0;
        held_.store(0);
        return;
    }
    for (Buf &b : bufs_)
        if (b.p) {
            if (stream_) (void)hipFreeAsync(b.p, stream_);
            else (void)hipFree(b.p);
            held_.fetch_sub(b.cap);
            b.p = nullptr;
            b.cap = 0;
        }
}

void Workspace::drop(int slot)
{
    if (arena_base_ || slot < 0 || slot >= (int)bufs_.size()) return;
    Buf &b = bufs_[slot];
    if (!b.p) return;
    if (stream_) (void)hipFreeAsync(b.p, stream_);
    else (void)hipFree(b.p);
    held_.fetch_sub(b.cap);
    b = Buf();
}

void *Workspace::get(int slot, size_t bytes)
{
    if (slot < 0 || slot >= (int)bufs_.size()) throw Error{MAP_EINVAL, "workspace slot out of range"};
    Buf &b = bufs_[slot];
    if (bytes == 0) bytes = 256;
    if (arena_base_) {
        if (b.cap >= bytes) return b.p;
        const size_t want = (bytes + 255) & ~size_t(255);
        if (want > arena_cap_ - arena_used_)
            throw Error{MAP_ENOMEM, "the fixed scratch buffer (" + std::to_string(arena_cap_ >> 20) +
                                        " MiB) is too small for this input: " + std::to_string(arena_used_ + want) +
                                        " bytes needed so far"};
        b.p = arena_base_ + arena_used_;
        b.cap = want;
        arena_used_ += want;
        held_.store(arena_used_);
        return b.p;
    }
    if (b.cap < bytes) {
        if (b.p) {
            if (stream_) EM_HIP(hipFreeAsync(b.p, stream_));
            else EM_HIP(hipFree(b.p));
        }
        held_.fetch_sub(b.cap);
        b.p = nullptr;
        b.cap = 0;
        // growth slack: a quarter, at most 256 MiB (buffers of tens of GB are not padded by a quarter)
        size_t want = bytes + std::min(bytes / 4, size_t(256) << 20) + 256;
        want = (want + 255) & ~size_t(255);
        hipError_t e = stream_ ? hipMallocAsync(&b.p, want, stream_) : hipMalloc(&b.p, want);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            throw Error{MAP_ENOMEM, "device allocation of " + std::to_string(want) + " bytes failed"};
        }
        b.cap = want;
        held_.fetch_add(want);
    }
    return b.p;
}

size_t Workspace::bytes_held() const { return held_.load(); }

// ---------------------------------------------------------------- bounded stream waits
static thread_local double t_wait_limit_ms = 0.0;

void set_wait_limit_ms(double ms) { t_wait_limit_ms = ms > 0.0 ? ms : 0.0; }

void stream_sync(hipStream_t s)
{
    if (t_wait_limit_ms <= 0.0) {
        EM_HIP(hipStreamSynchronize(s));
        return;
    }
    const auto t0 = std::chrono::steady_clock::now();
    for (int spin = 0;; spin++) {
        const hipError_t e = hipStreamQuery(s);
        if (e == hipSuccess) return;
        (void)hipGetLastError();  // a not-ready query is no error of the next call
        if (e != hipErrorNotReady)
            throw Error{MAP_EDEVICE, std::string("hipStreamQuery: ") + hipGetErrorString(e)};
        const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        if (ms > t_wait_limit_ms)
            throw Error{MAP_EDEVICE, std::string(kWaitLimitText) + " (" + std::to_string((long long)t_wait_limit_ms) +
                                         " ms)"};
        if (spin < 200) std::this_thread::yield();
        else std::this_thread::sleep_for(std::chrono::microseconds(20));
    }
}

namespace {

constexpr int kReadItems = 6;
struct ReadArgs {
    const uint32_t *from[kReadItems];
    int words[kReadItems], at[kReadItems], n;
};

__global__ void k_read_back(ReadArgs A, uint32_t *mail)
{
    for (int q = 0; q < A.n; q++)
        for (int i = threadIdx.x; i < A.words[q]; i += blockDim.x) mail[A.at[q] + i] = A.from[q][i];
}

}  // namespace

// A copy to pageable memory is a kernel into a staging buffer and a wait of the
// host for each; one kernel that writes all items to pinned memory and one wait
// bring a call on 512 particles (12 copies, now five of these) from 500 to 349 us,
// with the box as a kernel argument and k_stats_final.  Where waits have a limit (the
// server's threads) the stream is polled with sleeps between, and the copies stay:
// twelve served jobs 24.4 ms without them, 23.0 with.
void read_back(Workspace &ws, std::initializer_list<ReadItem> items, hipStream_t s)
{
    uint32_t *mail = t_wait_limit_ms > 0.0 ? nullptr : static_cast<uint32_t *>(ws.mailbox());
    ReadArgs A{};
    size_t at = 0;
    for (const ReadItem &r : items) {
        if (!mail) {
            EM_HIP(hipMemcpyAsync(r.to, r.from, r.bytes, hipMemcpyDeviceToHost, s));
            continue;
        }
        EM_CHECK(A.n < kReadItems && r.bytes % 4 == 0 && at + r.bytes <= kMailboxBytes, MAP_EINVAL,
                 "results do not fit the mailbox");
        A.from[A.n] = static_cast<const uint32_t *>(r.from);
        A.words[A.n] = (int)(r.bytes / 4);
        A.at[A.n++] = (int)(at / 4);
        at += r.bytes;
    }
    if (mail) {
        hipLaunchKernelGGL(k_read_back, dim3(1), dim3(64), 0, s, A, mail);
        EM_HIP(hipGetLastError());
    }
    stream_sync(s);
    at = 0;
    if (mail)
        for (const ReadItem &r : items) {
            std::memcpy(r.to, reinterpret_cast<const char *>(mail) + at, r.bytes);
            at += r.bytes;
        }
}

int device_cu_count()
{
    int dev = 0, cus = 0;
    EM_HIP(hipGetDevice(&dev));
    EM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    return cus > 0 ? cus : 1;
}

// ---------------------------------------------------------------- fills
__global__ void k_iota_u32(uint32_t *p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = (uint32_t)i;
}

__global__ void k_iota_i64(int64_t *p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = i;
}

__global__ void k_zero_u64(uint64_t *p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0;
}

__global__ void k_zero_u8(uint8_t *p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

static int grid_for(int64_t n, int block, int cap = 65536)
{
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

void fill_iota_u32(uint32_t *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_iota_u32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
    EM_HIP(hipGetLastError());
}

void fill_iota_i64(int64_t *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_iota_i64, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
    EM_HIP(hipGetLastError());
}

// Zero a buffer with a kernel (keeps the path free of memset nodes).
void fill_zero_bytes(void *p, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return;
    size_t words = bytes / 8;
    if (words) hipLaunchKernelGGL(k_zero_u64, dim3(grid_for((int64_t)words, 256)), dim3(256), 0, s,
                                  static_cast<uint64_t *>(p), (int64_t)words);
    size_t tail = bytes - words * 8;
    if (tail) hipLaunchKernelGGL(k_zero_u8, dim3(1), dim3(64), 0, s, static_cast<uint8_t *>(p) + words * 8,
                                 (int64_t)tail);
    EM_HIP(hipGetLastError());
}

// ---------------------------------------------------------------- block scan helpers
constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_CHUNK = SCAN_BLOCK * SCAN_ITEMS;

// exclusive scan of one value per thread across a 256-thread block (4 waves)
__device__ inline int64_t block_exclusive_scan(int64_t v, int64_t *total)
{
    __shared__ int64_t wsum[SCAN_BLOCK / 64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    int64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < SCAN_BLOCK / 64; w++) {
        if (w < wave) before += wsum[w];
        all += wsum[w];
    }
    __syncthreads();
    if (total) *total = all;
    return before + x - v;
}

__global__ void k_chunk_sums(const int64_t *in, int64_t n, int64_t *partial)
{
    int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_ITEMS;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++)
        if (base + k < n) s += in[base + k];
    int64_t tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// out[i+1] = prefix[block] + inclusive scan within the chunk; out[0] = 0
__global__ void k_chunk_scan(const int64_t *in, int64_t n, const int64_t *prefix, int64_t *out)
{
    int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_ITEMS;
    int64_t v[SCAN_ITEMS];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        s += v[k];
    }
    int64_t ex = block_exclusive_scan(s, nullptr) + (prefix ? prefix[blockIdx.x] : 0);
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        ex += v[k];
        if (base + k < n) out[base + k + 1] = ex;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0;
}

// The whole scan in one workgroup of 1024 threads.
constexpr int SCAN_ONE_BLOCK = 1024;
constexpr int SCAN_ONE_MAX = SCAN_ONE_BLOCK * SCAN_ITEMS;

__global__ void __launch_bounds__(SCAN_ONE_BLOCK) k_scan_one(const int64_t *in, int64_t n, int64_t *out)
{
    __shared__ int64_t wsum[SCAN_ONE_BLOCK / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = (int64_t)threadIdx.x * SCAN_ITEMS;
    int64_t v[SCAN_ITEMS], sum = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        v[k] = base + k < n ? in[base + k] : 0;
        sum += v[k];
    }
    int64_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int64_t ex = x - sum;
    for (int w = 0; w < SCAN_ONE_BLOCK / 64; w++)
        if (w < wave) ex += wsum[w];
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        ex += v[k];
        if (base + k < n) out[base + k + 1] = ex;
    }
    if (threadIdx.x == 0) out[0] = 0;
}

static void scan_rec(int64_t *tmp, const int64_t *in, int64_t *out, int64_t n, hipStream_t s)
{
    int64_t nb = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    if (nb <= 1) {
        hipLaunchKernelGGL(k_chunk_scan, dim3(1), dim3(SCAN_BLOCK), 0, s, in, n, (const int64_t *)nullptr, out);
        EM_HIP(hipGetLastError());
        return;
    }
    int64_t *partial = tmp;
    int64_t *pscan = tmp + nb;
    int64_t *next = tmp + 2 * nb + 1;
    hipLaunchKernelGGL(k_chunk_sums, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, partial);
    EM_HIP(hipGetLastError());
    scan_rec(next, partial, pscan, nb, s);
    hipLaunchKernelGGL(k_chunk_scan, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, (const int64_t *)pscan, out);
    EM_HIP(hipGetLastError());
}

void scan_counts(Workspace &ws, const int64_t *in, int64_t *out, int64_t n, hipStream_t s)
{
    if (n <= 0) {
        fill_zero_bytes(out, sizeof(int64_t), s);
        return;
    }
    if (n <= SCAN_ONE_MAX) {  // one launch of 5 us; the three of the chunked scan take 11, one chunk after the other here 7 each
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(SCAN_ONE_BLOCK), 0, s, in, n, out);
        EM_HIP(hipGetLastError());
        return;
    }
    // scratch: sum over levels of (2 nb + 1)
    int64_t need = 0, m = n;
    while (m > SCAN_CHUNK) {
        int64_t nb = (m + SCAN_CHUNK - 1) / SCAN_CHUNK;
        need += 2 * nb + 1;
        m = nb;
    }
    int64_t *tmp = ws.get<int64_t>(S_SCAN_TMP, (size_t)need + 8);
    scan_rec(tmp, in, out, n, s);
}

// ---------------------------------------------------------------- box trees
// A workgroup takes 256 parents of one level and goes up the subtree above them,
// nine levels a launch; one launch per level took 2.4 us each, 84 of them for a
// grid of 30,011 sites with five Lloyd steps.
__global__ void __launch_bounds__(256) k_tree_parents(int64_t first, double *boxes)
{
    int64_t level = first;
    int mine = first < 256 ? (int)first : 256;  // parents of this level that are the workgroup's
    for (;;) {
        if ((int)threadIdx.x < mine) {
            const int64_t i = level + (int64_t)blockIdx.x * mine + threadIdx.x;
            const double *a = boxes + 6 * (2 * i), *b = boxes + 6 * (2 * i + 1);
            double *o = boxes + 6 * i;
            for (int d = 0; d < 3; d++) {
                o[d] = fmin(a[d], b[d]);
                o[3 + d] = fmax(a[3 + d], b[3 + d]);
            }
        }
        if (mine == 1) break;
        __syncthreads();
        level >>= 1;
        mine >>= 1;
    }
}

void tree_parent_boxes(double *boxes, int64_t NL, hipStream_t s)
{
    for (int64_t first = NL / 2; first >= 1; first /= 512) {
        hipLaunchKernelGGL(k_tree_parents, dim3((unsigned)((first + 255) / 256)), dim3(256), 0, s, first, boxes);
        EM_HIP(hipGetLastError());
    }
}

// ---------------------------------------------------------------- radix sort
// LSD radix sort with digits of up to 10 bits: a key width of b bits takes
// ceil(b / 10) passes, the width split evenly between them (18-bit keys: two
// passes of 9 bits, so the result lands back in the input buffers).  Short
// lists are sorted by counting instead.
constexpr int RS_BLOCK = 256;
constexpr int RS_WAVES = RS_BLOCK / 64;
constexpr int RS_MAX_BITS = 10;
constexpr int RS_MAX_BUCKETS = 1 << RS_MAX_BITS;

template <typename K, int ITEMS>
__global__ void k_rs_hist(const K *keys, int64_t n, int shift, int rb, int64_t nblocks, int64_t *hist)
{
    __shared__ unsigned cnt[RS_MAX_BUCKETS];
    const int nb = 1 << rb;
    for (int t = threadIdx.x; t < nb; t += RS_BLOCK) cnt[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (RS_BLOCK * ITEMS);
    const unsigned mask = (unsigned)nb - 1u;
    for (int k = 0; k < ITEMS; k++) {
        int64_t i = base + (int64_t)k * RS_BLOCK + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(unsigned)(keys[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nb; t += RS_BLOCK) hist[(int64_t)t * nblocks + blockIdx.x] = cnt[t];
}

// Stable scatter: each wavefront ranks its own consecutive part of the tile, 64
// items at a time, against its own digit counts (the rank of an item among equal
// digits is the count so far plus the equal digits in lower lanes), with no
// barrier; the counts of the wavefronts become places in the tile, the tile is put
// in order in LDS, and neighbouring threads write neighbouring items.  The items
// stay in registers, so a thread's loads are all in flight together.  Bound by the
// scattered stores, runs of 8 items on average at 512 digits: a pass over
// 2,097,152 64-bit keys takes 25 us (46 with 256 items at a time, three barriers
// each, and stores item by item; 49 with the barriers gone alone), one over 14.5e6
// 32-bit keys 95 us (198).
template <typename K, int ITEMS>
__global__ void __launch_bounds__(RS_BLOCK) k_rs_scatter(const K *__restrict__ keys, const uint32_t *__restrict__ vals,
                                                         K *__restrict__ keys_out, uint32_t *__restrict__ vals_out,
                                                         int64_t n, int shift, int rb, int64_t nblocks,
                                                         const int64_t *__restrict__ offsets)
{
    constexpr int TILE = RS_BLOCK * ITEMS, PER = RS_MAX_BUCKETS / RS_BLOCK;
    __shared__ unsigned wcnt[RS_WAVES][RS_MAX_BUCKETS];
    __shared__ unsigned to[RS_MAX_BUCKETS];  // where a digit's items go, less their place in the tile
    __shared__ unsigned wsum[RS_WAVES];
    __shared__ K item[TILE];
    __shared__ uint32_t carried[TILE];
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nb = 1 << rb;
    const unsigned mask = (unsigned)nb - 1u;
    for (int q = lane; q < nb; q += 64) wcnt[wave][q] = 0;
    const int64_t tile = (int64_t)blockIdx.x * TILE, base = tile + (int64_t)wave * (64 * ITEMS) + lane;
    K key[ITEMS];
    uint32_t val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        const int64_t i = base + 64 * k;
        key[k] = i < n ? keys[i] : K(0);
        val[k] = i < n ? vals[i] : 0u;
    }
    lds_sync_wave();
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        const bool valid = base + 64 * k < n;
        const unsigned d = (unsigned)(key[k] >> shift) & mask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < rb; b++) {
            const bool one = (d >> b) & 1u;
            const uint64_t bb = __ballot(one);
            peers &= one ? bb : ~bb;
        }
        const unsigned below = (unsigned)lanes_below(peers), before = valid ? wcnt[wave][d] : 0u;
        rank[k] = before + below;
        lds_sync_wave();
        if (valid && below == 0) wcnt[wave][d] = before + (unsigned)__popcll(peers);
        lds_sync_wave();
    }
    __syncthreads();
    // thread t: digits PER t ..., their items and the items of the digits before (a scan over the threads)
    unsigned sum = 0;
    for (int u = 0; u < PER; u++)
        for (int w = 0; w < RS_WAVES; w++) sum += PER * t + u < nb ? wcnt[w][PER * t + u] : 0u;
    unsigned incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    unsigned at = incl - sum;
    for (int w = 0; w < wave; w++) at += wsum[w];
    for (int u = 0; u < PER; u++) {
        const int q = PER * t + u;
        if (q >= nb) break;
        to[q] = (unsigned)offsets[(int64_t)q * nblocks + blockIdx.x] - at;  // (fewer than 2^32 items)
        for (int w = 0; w < RS_WAVES; w++) {
            const unsigned c = wcnt[w][q];
            wcnt[w][q] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        if (base + 64 * k >= n) continue;
        const unsigned p = wcnt[wave][(unsigned)(key[k] >> shift) & mask] + rank[k];
        item[p] = key[k];
        carried[p] = val[k];
    }
    __syncthreads();
    const int m = (int)(n - tile < TILE ? n - tile : TILE);
    for (int p = t; p < m; p += RS_BLOCK) {
        const K x = item[p];
        const unsigned dest = to[(unsigned)(x >> shift) & mask] + (unsigned)p;
        keys_out[dest] = x;
        vals_out[dest] = carried[p];
    }
}

// Sort of a short list by counting: an item's place is the number of items
// whose (key, index) is less.  A workgroup takes 64 items; each of its 16
// wavefronts counts over a sixteenth of the list, whose keys it reads as
// wave-uniform values (scalar loads; a compare and an add per key), and the
// counts meet in LDS.  The work grows with the square of the list, so the line
// lies a little below the crossing: octrees (63-bit keys with values, whole build)
// of 1,000 particles 117 us by counting and 168 by seven radix passes, 16,384 154
// and 249, 32,768 217 and 272, 40,000 267 and 268, 65,536 403 and 280.
constexpr int64_t kSmallSort = 32768;
constexpr int kRankParts = 16;

template <typename K, bool VALS>
__global__ void __launch_bounds__(64 * kRankParts) k_rank_sort(const K *__restrict__ keys,
                                                               const uint32_t *__restrict__ vals, int64_t n,
                                                               K *__restrict__ keys_out, uint32_t *__restrict__ vals_out)
{
    __shared__ unsigned part[kRankParts][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = (int)blockIdx.x * 64, i = i0 + lane, m = (int)n;
    const K mine = i < m ? keys[i] : K(0);
    const int q = (m + kRankParts - 1) / kRankParts, lo = w * q < m ? w * q : m, hi = lo + q < m ? lo + q : m;
    unsigned less = 0;
    // before the items of this workgroup an equal key counts, after them it does not
    const int a = min(max(lo, i0), hi), b = min(max(a, i0 + 64), hi);
#pragma unroll 16
    for (int j = lo; j < a; j++) less += keys[j] <= mine ? 1u : 0u;
    for (int j = a; j < b; j++) {
        const K k = keys[j];
        less += k < mine || (k == mine && j < i) ? 1u : 0u;
    }
#pragma unroll 16
    for (int j = b; j < hi; j++) less += keys[j] < mine ? 1u : 0u;
    part[w][lane] = less;
    __syncthreads();
    if (w == 0 && i < m) {
        unsigned r = 0;
        for (int k = 0; k < kRankParts; k++) r += part[k][lane];
        keys_out[r] = mine;
        if (VALS) vals_out[r] = vals[i];
    }
}

template <typename K>
__global__ void k_copy_pairs(const K *__restrict__ keys, const uint32_t *__restrict__ vals, int64_t n,
                             K *__restrict__ keys_out, uint32_t *__restrict__ vals_out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys_out[i] = keys[i];
    vals_out[i] = vals[i];
}

template <typename K, int ITEMS>
static void radix_passes(Workspace &ws, K *keys, uint32_t *vals, K *keys2, uint32_t *vals2, int64_t n, int bits,
                         hipStream_t s)
{
    const int passes = (bits + RS_MAX_BITS - 1) / RS_MAX_BITS;
    const int rb = (bits + passes - 1) / passes;
    const int64_t nblocks = (n + RS_BLOCK * ITEMS - 1) / (RS_BLOCK * ITEMS);
    int64_t *hist = ws.get<int64_t>(S_SORT_HIST, (size_t)(nblocks << rb) * 2 + 1);
    int64_t *offs = hist + (nblocks << rb);
    K *src_k = keys, *dst_k = keys2;
    uint32_t *src_v = vals, *dst_v = vals2;
    for (int p = 0; p < passes; p++) {
        const int shift = rb * p;
        hipLaunchKernelGGL((k_rs_hist<K, ITEMS>), dim3((unsigned)nblocks), dim3(RS_BLOCK), 0, s, src_k, n, shift, rb,
                           nblocks, hist);
        EM_HIP(hipGetLastError());
        scan_counts(ws, hist, offs, nblocks << rb, s);
        hipLaunchKernelGGL((k_rs_scatter<K, ITEMS>), dim3((unsigned)nblocks), dim3(RS_BLOCK), 0, s, src_k, src_v,
                           dst_k, dst_v, n, shift, rb, nblocks, (const int64_t *)offs);
        EM_HIP(hipGetLastError());
        std::swap(src_k, dst_k);
        std::swap(src_v, dst_v);
    }
    if (src_k != keys) {
        hipLaunchKernelGGL(k_copy_pairs<K>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const K *)src_k,
                           (const uint32_t *)src_v, n, keys, vals);
        EM_HIP(hipGetLastError());
    }
}

template <typename K>
static void radix_sort(Workspace &ws, K *keys, uint32_t *vals, K *keys2, uint32_t *vals2, int64_t n, int bits,
                       hipStream_t s)
{
    if (n <= 1 || bits <= 0) return;
    if (n <= kSmallSort) {
        hipLaunchKernelGGL((k_rank_sort<K, true>), dim3((unsigned)((n + 63) / 64)), dim3(64 * kRankParts), 0, s, (const K *)keys,
                           (const uint32_t *)vals, n, keys2, vals2);
        EM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_copy_pairs<K>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const K *)keys2,
                           (const uint32_t *)vals2, n, keys, vals);
        EM_HIP(hipGetLastError());
        return;
    }
    // items per thread: enough workgroups to fill the chip, and more items per digit for the stores where there are
    // (a scatter pass with 4, 8 and 16 items: 262,144 keys 9.9, 11.7 and 15.3 us, 700,000 15.7, 14.7 and 16.7,
    // 2,097,152 40, 31 and 26)
    if (n <= (int64_t(1) << 19)) radix_passes<K, 4>(ws, keys, vals, keys2, vals2, n, bits, s);
    else if (n <= (int64_t(1) << 20)) radix_passes<K, 8>(ws, keys, vals, keys2, vals2, n, bits, s);
    else radix_passes<K, 16>(ws, keys, vals, keys2, vals2, n, bits, s);
}

const uint64_t *sort_keys_u64(Workspace &ws, uint64_t *keys, uint64_t *keys2, int64_t n, int bits, hipStream_t s)
{
    if (n <= 1) return keys;
    if (n <= kSmallSort) {
        hipLaunchKernelGGL((k_rank_sort<uint64_t, false>), dim3((unsigned)((n + 63) / 64)), dim3(64 * kRankParts), 0, s,
                           (const uint64_t *)keys, (const uint32_t *)nullptr, n, keys2, (uint32_t *)nullptr);
        EM_HIP(hipGetLastError());
        return keys2;
    }
    uint32_t *v = ws.get<uint32_t>(S_FIX_VAL2, (size_t)(2 * n));
    fill_iota_u32(v, n, s);
    radix_sort<uint64_t>(ws, keys, v, keys2, v + n, n, bits, s);
    return keys;
}

void radix_sort_u32(Workspace &ws, uint32_t *keys, uint32_t *vals, uint32_t *keys2, uint32_t *vals2, int64_t n,
                    int bits, hipStream_t s)
{
    radix_sort<uint32_t>(ws, keys, vals, keys2, vals2, n, bits, s);
}

void radix_sort_u64(Workspace &ws, uint64_t *keys, uint32_t *vals, uint64_t *keys2, uint32_t *vals2, int64_t n,
                    int bits, hipStream_t s)
{
    radix_sort<uint64_t>(ws, keys, vals, keys2, vals2, n, bits, s);
}

}  // namespace em
