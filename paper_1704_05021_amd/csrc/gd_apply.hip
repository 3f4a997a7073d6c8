// Server-side apply of sparse pushes to a parameter shard (Section 3: each
// server owns a shard of the parameters and receives the clients' pieces).
//
// For an index pushed by several clients the values are summed in client
// order starting from +0, and the parameter is updated once:
// p[i] -= lr * s[i].  No atomics, so the result is deterministic.
//
// Two forms, with the same results bit for bit.  The scattered form reads
// and writes only the pushed parameters; the streaming form reads the whole
// shard in order and writes back the 16-byte vectors that change, for pushes
// dense enough that most 128-byte lines of the shard hold an update.
// Quantised pushes (indices, sign bits, centre pairs; Section 5.4) are decoded
// entry by entry where their values are read.
//
// The scattered form: one block per bucket of 2^11 to 2^15 consecutive parameter
// indices (the denser the pushes, the fewer).  The block finds where the bucket starts and ends in every
// client's (ascending) index list, all bounds at once by groups of lanes (a
// 32-way search for four clients, 8-way for sixteen), stages those entries in
// LDS, dealt to the threads whatever client they come from, marks the indices
// pushed more than once, and then gives every index to the lowest client
// holding it, which sums all clients' values for it in client order and
// writes p once.  The parameter writes of a block stay inside its bucket.

#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <thread>
#include <utility>

#include "gd_kernels.h"

namespace gd {

constexpr uint32_t kApplyBucketShift = 15;                   // parameters of a bucket, at most (log2)
constexpr uint32_t kApplyBucketMin = 11;                     // and at least
constexpr uint32_t kApplyBucketEntries = 512;                // entries of a bucket, on average at most
constexpr int kApplyLds = 2048;                              // entries of all clients staged per bucket
constexpr int kBucketWords = (1 << kApplyBucketShift) / 32;  // one bit per index of a bucket

// First position in list[0, n) whose value is >= x, found by a group of L
// lanes together (L a power of two, g the lane within its group): L probes a
// round.  All lanes of the wave call it; groups may search different lists.
__device__ __forceinline__ uint32_t group_lower_bound(const uint32_t* list, uint32_t n, uint32_t x, uint32_t L, uint32_t g) {
    const uint64_t mask = (L == 64 ? ~0ull : (1ull << L) - 1ull) << (lane_id() & ~(L - 1u));
    uint32_t lo = 0, hi = n;
    while (ballot(hi > lo) != 0) {
        const uint32_t len = hi - lo, step = (len + L - 1u) / L;
        uint64_t q = len <= L ? (uint64_t)lo + g : (uint64_t)lo + (uint64_t)(g + 1u) * step - 1u;
        if (len > L && q >= hi) q = hi - 1u;
        // probes rise with g, so the lanes below x form a prefix of the group
        const bool below = q < hi && list[q] < x;
        const uint32_t t = popc64(ballot(below) & mask);
        if (hi > lo) {
            if (len <= L) {
                lo = hi = lo + t;
            } else {
                const uint64_t nlo = (uint64_t)lo + (uint64_t)t * step, nhi = nlo + step;
                lo = nlo < hi ? (uint32_t)nlo : hi;
                hi = nhi < hi ? (uint32_t)nhi : hi;
            }
        }
    }
    return lo;
}

// First position in list[lo, hi) holding x, or hi.
__device__ __forceinline__ uint32_t find_u32(const uint32_t* list, uint32_t lo, uint32_t hi, uint32_t x) {
    uint32_t a = lo, b = hi;
    while (a < b) {
        const uint32_t mid = a + ((b - a) >> 1);
        if (list[mid] < x) a = mid + 1;
        else b = mid;
    }
    return a < hi && list[a] == x ? a : hi;
}

// Layouts of at most this many tensors have their starts copied to LDS, where
// the quantised pushes look up each entry's tensor.
constexpr uint32_t kApplyTensors = 64;

__device__ __forceinline__ void load_starts(const ApplyArgs& a, uint32_t* starts) {
    if (a.qkind != 0 && a.T <= kApplyTensors && threadIdx.x < a.T) starts[threadIdx.x] = a.tensor_off[threadIdx.x];
}

// Centre of a quantised push's entry (index i): the entry's sign picks it from
// the pair of its tensor or column.  starts: the tensors' first elements
// (load_starts), or where they are many, in memory.
__device__ __forceinline__ float push_centre(const ApplyArgs& a, const uint32_t* starts, const float* means, uint32_t i,
                                             uint32_t neg) {
    uint32_t lo = 0, hi = a.T;  // tensor holding i: the last t with start <= i
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        const uint32_t x = a.T <= kApplyTensors ? starts[mid] : a.tensor_off[mid];
        if (x <= i) lo = mid;
        else hi = mid;
    }
    const uint32_t g = a.qkind == kQuantColumnMean ? a.colbase[lo] + (i - a.tensor_off[lo]) % a.columns[lo] : lo;
    return means[2 * g + neg];
}

// Value of entry pos (index i) of push c: sent as is, or the entry's centre.
__device__ __forceinline__ float push_val(const ApplyArgs& a, const uint32_t* starts, uint32_t c, uint32_t pos, uint32_t i) {
    if (a.qkind == 0) return a.val[c][pos];
    return push_centre(a, starts, a.means[c], i, (a.bits[c][pos >> 5] >> (pos & 31)) & 1u);
}

__global__ __launch_bounds__(kBlock) void k_apply(ApplyArgs a) {
    __shared__ uint32_t rng[2 * kMaxPushes];   // bucket's [begin, end) in each client's list
    __shared__ uint32_t base[kMaxPushes + 1];  // first staged entry of each client
    __shared__ uint32_t sidx[kApplyLds];
    __shared__ float sval[kApplyLds];
    __shared__ uint32_t seen[2][kBucketWords];  // [0]: index pushed at least once, [1]: more than once
    __shared__ uint32_t starts[kApplyTensors];
    __shared__ uint16_t again[kApplyLds];  // staged entries whose index another client holds too
    __shared__ uint32_t nagain;
    const int tid = threadIdx.x;
    const uint32_t b = blockIdx.x;
    const uint32_t i_lo = b << a.bshift;
    const uint64_t i_hi64 = ((uint64_t)b + 1) << a.bshift;
    const uint32_t i_hi = i_hi64 < a.n ? (uint32_t)i_hi64 : a.n;
    // 1. the bucket's range in every list, all 2 C bounds at once: groups of
    //    as many lanes as the block has for each
    uint32_t L = 32;
    while (L * 2 * a.C > (uint32_t)kBlock) L >>= 1;
    {
        const uint32_t j = tid / L;  // bound j & 1 of client j >> 1
        const bool has = j < 2 * a.C;
        const uint32_t c = has ? j >> 1 : 0u;
        const uint32_t pos = group_lower_bound(a.idx[c], has ? a.nnz[c] : 0u, j & 1 ? i_hi : i_lo, L, tid & (L - 1u));
        if (has && (tid & (L - 1u)) == 0) rng[j] = pos;
    }
    load_starts(a, starts);
    if (tid == 0) nagain = 0;
    for (uint32_t q = tid; q < (1u << a.bshift) / 32u; q += kBlock) {
        seen[0][q] = 0;
        seen[1][q] = 0;
    }
    __syncthreads();
    if (tid < kWave) {
        // (a list out of order may end before it begins)
        const uint32_t cnt = (uint32_t)tid < a.C && rng[2 * tid + 1] > rng[2 * tid] ? rng[2 * tid + 1] - rng[2 * tid] : 0u;
        const uint32_t incl = wave_incl_scan(cnt);
        base[tid] = incl - cnt;  // (for tid >= C: the total)
        if (tid == kWave - 1) base[kWave] = incl;
    }
    __syncthreads();
    const uint32_t total = base[kMaxPushes];
    if (total == 0) return;
    if (total <= (uint32_t)kApplyLds) {
        // 2. stage the bucket's entries (index, value) of every client, dealt
        //    to the threads in order: entry e belongs to the last client whose
        //    first entry is at or before it.  Indices, values or sign words of
        //    all a thread's entries are in flight together.
        constexpr int kPer = kApplyLds / kBlock;
        uint32_t cl[kPer], pi[kPer], bits[kPer];
        float pv[kPer];
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const uint32_t e = tid + t * kBlock;
            cl[t] = kNoKey;
            pi[t] = kNoKey;
            pv[t] = 0.0f;
            bits[t] = 0;
            if (e >= total) continue;
            uint32_t c = 0;
#pragma unroll
            for (uint32_t st = kMaxPushes / 2; st > 0; st >>= 1)
                if (base[c + st] <= e) c += st;  // (clients past the last have no entry: base is the total)
            const uint32_t pos = rng[2 * c] + (e - base[c]);
            cl[t] = c;
            pi[t] = a.idx[c][pos];
            if (a.qkind == 0) pv[t] = a.val[c][pos];
            else bits[t] = a.bits[c][pos >> 5] >> (pos & 31);
        }
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const uint32_t e = tid + t * kBlock;
            if (e >= total) continue;
            const uint32_t off = pi[t] - i_lo, bit = 1u << (off & 31);
            // an index outside the bucket (a list out of order) is skipped
            if (off >= i_hi - i_lo) pi[t] = kNoKey;
            else if (a.qkind != 0) pv[t] = push_centre(a, starts, a.means[cl[t]], pi[t], bits[t] & 1u);
            sidx[e] = pi[t];
            sval[e] = pv[t];
            if (pi[t] != kNoKey && (atomicOr(&seen[0][off >> 5], bit) & bit)) atomicOr(&seen[1][off >> 5], bit);
        }
        __syncthreads();
        // 3. an index pushed once takes its value; a thread reads the
        //    parameters of all its entries at once, so that their latencies
        //    overlap.  The entries of the others are listed and dealt to the
        //    threads anew (a wave that met a few of them among its own entries
        //    would wait for their searches each time): an entry is skipped if
        //    a lower client holds its index, else it sums every client's value
        //    in client order.
        float pold[kPer];
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            pold[t] = 0.0f;
            if (pi[t] == kNoKey) continue;
            const uint32_t off = pi[t] - i_lo;
            if (seen[1][off >> 5] & (1u << (off & 31))) {
                again[atomicAdd(&nagain, 1u)] = (uint16_t)(tid + t * kBlock);
                pi[t] = kNoKey;
            } else {
                pold[t] = a.p[pi[t]];
            }
        }
        __syncthreads();
        for (uint32_t d = tid; d < nagain; d += kBlock) {
            const uint32_t e = again[d], i = sidx[e];
            uint32_t c = 0;
#pragma unroll
            for (uint32_t st = kMaxPushes / 2; st > 0; st >>= 1)
                if (base[c + st] <= e) c += st;
            const float old = a.p[i];
            bool owner = true;
            for (uint32_t cc = 0; cc < c && owner; ++cc)
                owner = find_u32(sidx, base[cc], base[cc + 1], i) == base[cc + 1];
            if (!owner) continue;
            float sum = 0.0f + sval[e];
            for (uint32_t cc = c + 1; cc < a.C; ++cc) {
                const uint32_t hit = find_u32(sidx, base[cc], base[cc + 1], i);
                if (hit != base[cc + 1]) sum = sum + sval[hit];
            }
            const float step = a.lr * sum;
            a.p[i] = old - step;
        }
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            if (pi[t] == kNoKey) continue;
            const float sum = 0.0f + pv[t], step = a.lr * sum;
            a.p[pi[t]] = pold[t] - step;
        }
        return;
    }
    // More entries than the block can stage: each reads the lists as they lie.
    for (uint32_t e = tid; e < total; e += kBlock) {
        uint32_t c = 0;
        while (base[c + 1] <= e) ++c;  // client of entry e
        const uint32_t q = e - base[c];
        const uint32_t i = a.idx[c][rng[2 * c] + q];
        if (i - i_lo >= i_hi - i_lo) continue;  // outside the bucket: a list out of order
        bool owner = true;
        for (uint32_t cc = 0; cc < c && owner; ++cc)
            owner = find_u32(a.idx[cc], rng[2 * cc], rng[2 * cc + 1], i) == rng[2 * cc + 1];
        if (!owner) continue;
        float s = 0.0f + push_val(a, starts, c, rng[2 * c] + q, i);
        for (uint32_t cc = c + 1; cc < a.C; ++cc) {
            const uint32_t hit = find_u32(a.idx[cc], rng[2 * cc], rng[2 * cc + 1], i);
            if (hit != rng[2 * cc + 1]) s = s + push_val(a, starts, cc, hit, i);
        }
        const float step = a.lr * s;
        a.p[i] = a.p[i] - step;
    }
}

// The streaming form, for pushes dense enough that most 128-byte lines of
// the shard hold an update (the scattered form above then fetches nearly every
// line anyway, one scattered word at a time).  One block per tile of
// kApplyTileLen consecutive parameters reads the tile in order with 16-byte
// loads, forms the sum of every pushed parameter of the tile in LDS, and
// writes back only the 16-byte vectors that an entry touches.
//
// The sums start at +0 and take the clients in turn, between barriers.  No
// two entries of one client's turn share an index (a push holds an index at
// most once), so each LDS sum is formed in client order without atomics, as
// the scattered form forms it, and the parameter then takes p - lr * sum:
// the two forms agree bit for bit.  The tile's range in every client's list
// comes from a bounds table (k_apply_bounds, one pass over the lists before
// this kernel).  Each thread loads kApplyTileEntries entries of the tile at
// once, for all clients together (entry e of the tile belongs to the last
// client whose first entry in the tile is at or before e); a tile with more
// entries takes further rounds, each with the turns of its own clients only
// (with a turn of all 40 clients a round, 40 that push the same 47 rows of a
// 37M shard took 261 us, in the scattered form 219; now 198).
//
// Tiles of 4,096 parameters (four 16-byte vectors per thread, 16.9 KB of
// LDS) keep eight blocks per compute unit in flight, which streams faster on
// this part than fewer blocks holding larger chunks in registers, or
// persistent blocks that load the next tile while they settle the current
// one (both measured slower).
constexpr int kApplyTileShift = 12;
constexpr uint32_t kApplyTileLen = 1u << kApplyTileShift;                          // parameters per block
constexpr int kApplyTileThreads = 256;
constexpr int kApplyTileVecs = (int)kApplyTileLen / 4 / kApplyTileThreads;        // 16-byte vectors per thread
constexpr int kApplyTileEntries = 2;                                                // entries per thread per round
constexpr uint32_t kApplyTileRound = (uint32_t)kApplyTileEntries * kApplyTileThreads;
static_assert(kMaxPushes == kWave, "one lane per client holds its range");

// The bounds table of the streaming form: row c holds, for every tile
// boundary B_b (b * kApplyTileLen for b < tiles, n for b = tiles), the first
// position in client c's list whose index is at least B_b.  With f(x) the
// number of boundaries at or below x, entry e starts the boundaries in
// [f(x_{e-1}), f(x_e)), the list's head [0, f(x_0)) starts at 0 and its tail
// [f(x_last), tiles] at the list's length: one pass over the entries, no
// search.  One row of blocks per client (blockIdx.y); the first tiles + 1
// threads of a row fill the head and tail, the others one entry each.  (A
// list out of order leaves some boundaries unwritten; readers clamp.)
__global__ __launch_bounds__(kBlock) void k_apply_bounds(ApplyArgs a, uint32_t tiles) {
    const uint32_t c = blockIdx.y;
    const uint32_t m = a.nnz[c];
    const uint32_t* list = a.idx[c];
    uint32_t* row = const_cast<uint32_t*>(a.tab) + (size_t)c * a.tstride;
    const uint64_t item = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const auto f = [&](uint32_t x) { return x < a.n ? (x >> kApplyTileShift) + 1u : tiles + 1u; };
    if (item <= tiles) {
        const uint32_t b = (uint32_t)item;
        if (m == 0 || b < f(list[0])) row[b] = 0;
        else if (b >= f(list[m - 1])) row[b] = m;
        return;
    }
    const uint64_t e = item - tiles;  // 1 .. m - 1
    if (e >= m) return;
    const uint32_t hi = f(list[e]);
    for (uint32_t b = f(list[e - 1]); b < hi; ++b) row[b] = (uint32_t)e;
}

__global__ __launch_bounds__(kApplyTileThreads) void k_apply_tile(ApplyArgs a) {
    __shared__ __align__(16) float sum[kApplyTileLen];      // per parameter of the tile
    __shared__ uint32_t touched[kApplyTileLen / 32];       // pushed at least once
    __shared__ uint32_t starts[kApplyTensors];
    const int tid = threadIdx.x, lane = lane_id();
    const uint32_t b = blockIdx.x, C = a.C;
    const uint32_t i_lo = b << kApplyTileShift;
    const bool whole = (uint64_t)i_lo + kApplyTileLen <= a.n;  // the same in every thread
    const uint32_t len = whole ? kApplyTileLen : a.n - i_lo;
    load_starts(a, starts);  // (read after the first barrier below)
    // The tile's range in the list of client `lane` (lanes >= C: none), from
    // the bounds table and clamped to the list, so that any table content
    // stays inside it.  Every wave reads it, so no barrier is needed for it.
    uint32_t r0 = 0, r1 = 0, nz = 0;
    if ((uint32_t)lane < C) {
        const uint32_t* row = a.tab + (size_t)lane * a.tstride + b;
        r0 = row[0];
        r1 = row[1];
    }
    // The tile's parameters: vector v = tid + kApplyTileThreads r holds
    // parameters i_lo + 4v .. 4v + 3 (each row of vectors is one coalesced
    // 4 KB read).
    f4 pv[kApplyTileVecs];
    if (whole) {
#pragma unroll
        for (int r = 0; r < kApplyTileVecs; ++r)
            pv[r] = *reinterpret_cast<const f4*>(a.p + i_lo + 4u * ((uint32_t)tid + (uint32_t)r * kApplyTileThreads));
    } else {
#pragma unroll
        for (int r = 0; r < kApplyTileVecs; ++r) {
            const uint32_t o = 4u * ((uint32_t)tid + (uint32_t)r * kApplyTileThreads);
            pv[r] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (o + q < len) pv[r][q] = a.p[i_lo + o + q];
        }
    }
    for (uint32_t c = 0; c < C; ++c)
        if ((uint32_t)lane == c) nz = a.nnz[c];
    r0 = min(r0, nz);
    r1 = min(r1, nz);
    const uint32_t cnt = r1 > r0 ? r1 - r0 : 0u;
    const uint32_t incl = wave_incl_scan(cnt);
    const uint32_t base = incl - cnt;                        // the client's first entry in the tile
    const uint32_t total = lane_value(incl, kWave - 1);      // the same in every wave
#pragma unroll
    for (int r = 0; r < kApplyTileVecs; ++r)
        reinterpret_cast<f4*>(sum)[tid + r * kApplyTileThreads] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    if (tid < (int)(kApplyTileLen / 32)) touched[tid] = 0;
    if (total == 0) return;  // nothing pushed here (block-uniform): nothing is written
    for (uint32_t e0 = 0; e0 < total; e0 += kApplyTileRound) {
        // this thread's entries e = e0 + tid + kApplyTileThreads k: offset in
        // the tile, client and value, all loaded at once
        uint32_t off[kApplyTileEntries], cl[kApplyTileEntries], bits[kApplyTileEntries];
        float val[kApplyTileEntries];
#pragma unroll
        for (int k = 0; k < kApplyTileEntries; ++k) {
            const uint32_t e = e0 + (uint32_t)tid + (uint32_t)k * kApplyTileThreads;
            uint32_t c = 0, first = 0, at = lane_value(r0, 0);
            const uint32_t* ip = a.idx[0];
            const float* vp = a.val[0];
            for (uint32_t cc = 1; cc < C; ++cc) {
                const uint32_t bc = lane_value(base, (int)cc), rc = lane_value(r0, (int)cc);
                if (e >= bc) {
                    c = cc;
                    first = bc;
                    at = rc;
                    ip = a.idx[cc];
                    vp = a.val[cc];
                }
            }
            cl[k] = kNoKey;
            off[k] = kNoKey;
            val[k] = 0.0f;
            bits[k] = 0;
            if (e < total) {
                const uint32_t pos = at + (e - first);
                const uint32_t i = ip[pos];
                cl[k] = c;
                off[k] = i - i_lo;  // outside the tile (a list out of order): skipped below
                if (a.qkind == 0) val[k] = vp[pos];
                else bits[k] = a.bits[c][pos >> 5] >> (pos & 31);
            }
        }
        __syncthreads();  // sums cleared (first round), or the previous round's turns done
        if (a.qkind != 0) {
#pragma unroll
            for (int k = 0; k < kApplyTileEntries; ++k)
                if (off[k] < len) val[k] = push_centre(a, starts, a.means[cl[k]], i_lo + off[k], bits[k] & 1u);
        }
        // turns of the clients that the round's entries belong to only (the same in every
        // wave: rounds of a tile with many entries hold few clients each)
        const uint32_t e1 = total - e0 > kApplyTileRound ? e0 + kApplyTileRound - 1u : total - 1u;
        const uint32_t c0 = popc64(ballot((uint32_t)lane < C && base <= e0)) - 1u;
        const uint32_t c1 = popc64(ballot((uint32_t)lane < C && base <= e1)) - 1u;
        for (uint32_t t = c0; t <= c1; ++t) {
            if (t > c0) __syncthreads();  // the previous client's turn done
#pragma unroll
            for (int k = 0; k < kApplyTileEntries; ++k) {
                if (cl[k] != t || off[k] >= len) continue;
                sum[off[k]] = sum[off[k]] + val[k];
                atomicOr(&touched[off[k] >> 5], 1u << (off[k] & 31u));
            }
        }
    }
    __syncthreads();  // every sum complete
#pragma unroll
    for (int r = 0; r < kApplyTileVecs; ++r) {
        const uint32_t v = (uint32_t)tid + (uint32_t)r * kApplyTileThreads;
        const uint32_t nib = (touched[v >> 3] >> ((v & 7u) * 4u)) & 0xFu;  // parameters 4v .. 4v + 3
        if (nib == 0) continue;
        const f4 s = reinterpret_cast<const f4*>(sum)[v];
        f4 x = pv[r];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((nib >> q) & 1u) {
                const float step = a.lr * s[q];
                x[q] = x[q] - step;
            }
        }
        if (whole) {
            *reinterpret_cast<f4*>(a.p + i_lo + 4u * v) = x;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4u * v + q < len) a.p[i_lo + 4u * v + q] = x[q];
        }
    }
}

// Form of later applies (a test hook): 0 chosen per call, 1 scattered, 2
// streaming wherever the parameters are 16-byte aligned.
static std::atomic<int> g_apply_form{0};

// The streaming form's bounds table is kept per device and stream, and reused
// by later calls on the same stream: work on one stream runs in order, so a
// call's bounds pass cannot overwrite the table while an earlier call on that
// stream still reads it, and calls on different streams use different tables.
// (A per-call allocation in stream order from a memory pool, or an event
// ordering the calls of all streams on one table, each cost about 5-6 us per
// call.)  The per-thread default stream is one stream per host thread, so
// its tables are kept per thread.  The mutex also keeps the two launches of
// one call together when host threads share a stream.  A call that needs more
// than its stream's table gets a new one of at least twice the size.  No table
// is ever freed: a captured call holds its address for every replay of its
// graph, and nothing tells when the last replay was.  So all tables of a stream
// take less than twice the largest, itself below twice what a call needed.
struct TableKey {
    int dev;
    uintptr_t stream;
    std::thread::id thread;
    bool operator<(const TableKey& o) const {
        if (dev != o.dev) return dev < o.dev;
        if (stream != o.stream) return stream < o.stream;
        return thread < o.thread;
    }
};
static std::mutex g_tab_mu;
static std::map<TableKey, std::pair<void*, size_t>> g_tables;

// hipMalloc by a thread in the relaxed capture mode: in the default mode it is
// refused while any stream in the process is being captured, and breaks that
// capture (of another program part, perhaps, that this call has nothing to do with).
static hipError_t malloc_beside_captures(void** p, size_t bytes) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return hipMalloc(p, bytes);
    const hipError_t e = hipMalloc(p, bytes);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return e;
}

// The table of the current device and stream st, at least `bytes` long, or
// null if it cannot be allocated.  Called with g_tab_mu held.
static uint32_t* stream_table(hipStream_t st, size_t bytes) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    const TableKey key{dev, reinterpret_cast<uintptr_t>(st), st == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id()};
    auto& slot = g_tables[key];
    if (slot.second < bytes) {
        const size_t least = (bytes + 65535u) & ~(size_t)65535u;
        size_t want = std::max(least, 2 * slot.second);
        void* q = nullptr;
        if (malloc_beside_captures(&q, want) != hipSuccess) {
            (void)hipGetLastError();
            want = least;
            if (malloc_beside_captures(&q, want) != hipSuccess) return nullptr;
        }
        slot = {q, want};
    }
    return static_cast<uint32_t*>(slot.first);
}

void set_apply_form(int form) { g_apply_form.store(form); }

hipError_t launch_apply(const ApplyArgs& a, uint32_t max_nnz, hipStream_t st) {
    if (a.C == 0 || max_nnz == 0 || a.n == 0) return hipSuccess;
    uint64_t total = 0;
    for (uint32_t c = 0; c < a.C; ++c) total += a.nnz[c];
    // Streaming reads every line of the shard, in order; scattered reads and
    // writes words, and searches for the indices that several clients hold.
    // How the pushes lie is not known here.  Spread evenly they cost scattered
    // less up to about an entry per 32 parameters, but where most lie in few
    // rows (a vocabulary sorted by frequency) a bucket overflows the staged
    // entries and its block reads the lists in place, while streaming depends
    // little on it.  us, scattered / streaming, evenly and all in the shard's
    // first rows: 37M parameters, an entry per 60: 1 client 24 / 35 and 39 / 30,
    // 4 clients 29 / 38 and 1204 / 79, 8 clients 35 / 45 and 3432 / 172.  So the
    // line of up to 8 clients is where about 40% of the shard's lines hold an
    // entry if they lie evenly: 12 us lost at most there, against 3 ms.
    // With more clients streaming costs a turn of barriers more for each, and
    // evenly the two measure alike at the lines below (16 clients: 9.7M, per 100:
    // 25 / 29, per 50: 28 / 28; 37M, per 50: 50 / 57, per 30: 82 / 59; in the first
    // rows 9.7M, per 100: 1439 / 404; 37M, per 30: 1968 / 413).
    const int form = g_apply_form.load();
    const bool aligned = (reinterpret_cast<uintptr_t>(a.p) & 15u) == 0;
    const bool cached = a.n <= (1u << 24);  // the shard stays in the caches (64 MiB)
    const uint64_t sparse = a.C <= 8u ? 64u : cached ? 128u : 48u;
    bool stream = aligned && form != 1 && (form == 2 || total * sparse >= a.n);
    if (stream && form != 2 && a.C > 8u) {
        // A captured call of more than 8 clients is scattered, so that no
        // first call is needed before the capture, and no replay depends on a
        // table that a later call on the stream may replace.
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        stream = hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone;
        if (!stream) (void)hipGetLastError();
    }
    if (stream) {
        const uint32_t tiles = (uint32_t)(((uint64_t)a.n + kApplyTileLen - 1) >> kApplyTileShift);
        std::lock_guard<std::mutex> lk(g_tab_mu);
        uint32_t* tab = stream_table(st, (size_t)a.C * (tiles + 1u) * sizeof(uint32_t));
        if (tab) {
            ApplyArgs b = a;
            b.tab = tab;
            b.tstride = tiles + 1u;
            uint64_t items = 0;  // head and tail, then the entries after the first
            for (uint32_t c = 0; c < a.C; ++c) items = std::max<uint64_t>(items, tiles + 1u + (a.nnz[c] ? a.nnz[c] - 1u : 0u));
            hipLaunchKernelGGL(k_apply_bounds, dim3((uint32_t)((items + kBlock - 1) / kBlock), a.C), dim3(kBlock), 0, st, b,
                               tiles);
            hipLaunchKernelGGL(k_apply_tile, dim3(tiles), dim3(kApplyTileThreads), 0, st, b);
            return hipGetLastError();
        }
        (void)hipGetLastError();  // no table: the scattered form below
    }
    // Buckets hold at most kApplyBucketEntries entries on average, so that few hold
    // more than are staged.  us, all of 2^15 parameters / by density (37M parameters
    // that are not 16-byte aligned, an entry per 20, 4 clients): evenly 75 / 64, rows
    // by frequency 241 / 81, all in the first rows 395 / 102; against that the blocks
    // without an entry, which only search, where whole rows lie evenly: 40 / 49.
    ApplyArgs b = a;
    b.bshift = kApplyBucketShift;
    while (b.bshift > kApplyBucketMin && (total << b.bshift) > (uint64_t)kApplyBucketEntries * a.n) --b.bshift;
    const uint32_t buckets = (uint32_t)(((uint64_t)a.n + (1ull << b.bshift) - 1) >> b.bshift);
    hipLaunchKernelGGL(k_apply, dim3(buckets), dim3(kBlock), 0, st, b);
    return hipGetLastError();
}

}  // namespace gd
