// 1-bit quantisation of the kept values (Section 5.4), with the
// quantisation error fed back into the residual (gfx950, wave64).
//
// After dropping, each kept value is replaced by one of two centres, chosen by
// its sign (values not below zero are positive).  Section 5.4 compares
// several ways of choosing the centres; all four are here:
//   sign mean    : per tensor, the average of its kept positive values and of
//                  its kept negative values;
//   threshold    : +-T, T the dropping threshold, i.e. the smallest kept
//                  magnitude of the threshold segment;
//   global mean  : one positive and one negative average over every kept
//                  value of the call;
//   column mean  : per column of each tensor's row-major matrix view.
// Per-tensor and global sums are taken in fp64 in a fixed order (per
// candidate tile, then tiles in order; after the direct form per slice of the
// sent list, then slices in order), so they are deterministic; column
// sums are fp64 atomics over the sent entries (in LDS per slice, then once
// per touched column).  The sent bits are packed LSB-first, 32 per word,
// and residual[idx] becomes acc - centre.

#include <algorithm>

#include "gd_kernels.h"

namespace gd {

// Sent entries up to which column sums take slices of 256, of 1,024 and of 2,048.
constexpr uint64_t kColTinyK = 1u << 16, kColSmallK = 1u << 18, kColMidK = 1u << 20;

// Zeros tensor u keeps in the zero mode (every candidate kept, plus zeros):
// its kept count less its candidates; 0 outside the zero mode.
__device__ __forceinline__ uint32_t zeros_kept(const QuantArgs& q, uint32_t u) {
    return q.seg[q.per_tensor ? u : 0u].zero ? q.tensor_counts[u] - (q.ten_cbase[u + 1] - q.ten_cbase[u]) : 0u;
}

// Centres per tensor (every kind but the column mean) and the first output
// slot of each tensor.  One wave per tensor.
__global__ __launch_bounds__(kBlock) void k_means(QuantArgs q) {
    const int w = threadIdx.x >> 6, lane = lane_id();
    const uint32_t t = blockIdx.x * kWavesPerBlock + w;
    if (t >= q.T) return;
    uint32_t before = 0;
    for (uint32_t u = lane; u < t; u += kWave) before += q.tensor_counts[u];
    before = wave_sum(before);
    if (lane == 0) {
        q.qbase[t] = before;
        if (t + 1 == q.T) q.qbase[q.T] = before + q.tensor_counts[t];
    }
    if (q.qkind == kQuantColumnMean) return;
    float pos = 0.0f, neg = 0.0f;
    if (q.qkind == kQuantThreshold) {
        // the smallest kept magnitude of the segment: the exact threshold key,
        // or under a sampled threshold the smallest key sent, the minimum over
        // the segment's tiles
        const uint32_t s = q.per_tensor ? t : 0u;
        uint32_t key = kNoKey;
        if (q.sampled) {
            const uint32_t g0 = q.per_tensor ? q.tile_base[t] : 0u, g1 = q.per_tensor ? q.tile_base[t + 1] : q.tile_base[q.T];
            for (uint32_t g = g0 + lane; g < g1; g += kWave) {
                const uint32_t x = (uint32_t)q.tile_q[4 * (size_t)g + 0];
                key = x < key ? x : key;
            }
            key = wave_min(key);
        } else if (keep_of(q.seg_off[s + 1] - q.seg_off[s], q.keep_ppm) > 0) {
            key = q.seg[s].zero ? 0u : q.seg[s].thr;  // zero mode: T = 0 (the count pass may see no tile)
        }
        if (key != kNoKey) {
            pos = __uint_as_float(key);
            neg = __uint_as_float(key | 0x80000000u);
        }
    } else {
        const bool global = q.qkind == kQuantGlobalMean;
        const uint32_t g0 = global ? 0u : q.tile_base[t], g1 = global ? q.tile_base[q.T] : q.tile_base[t + 1];
        double sp = 0.0, sn = 0.0, np = 0.0, nn = 0.0;
        for (uint32_t g = g0 + lane; g < g1; g += kWave) {
            sp += q.tile_q[4 * (size_t)g + 0];
            sn += q.tile_q[4 * (size_t)g + 1];
            np += q.tile_q[4 * (size_t)g + 2];
            nn += q.tile_q[4 * (size_t)g + 3];
        }
        sp = wave_sum(sp);
        sn = wave_sum(sn);
        np = wave_sum(np);
        nn = wave_sum(nn);
        // zero mode: the kept zeros are in no tile's sums; each counts as a
        // positive value (not below zero) and adds nothing to sp
        uint32_t zk = 0;
        if (global) {
            for (uint32_t u = lane; u < q.T; u += kWave) zk += zeros_kept(q, u);
        } else if (lane == 0) {
            zk = zeros_kept(q, t);
        }
        np += (double)wave_sum(zk);
        pos = np > 0.0 ? (float)(sp / np) : 0.0f;
        neg = nn > 0.0 ? (float)(sn / nn) : 0.0f;
    }
    if (lane == 0) {
        q.means[2 * t + 0] = pos;
        q.means[2 * t + 1] = neg;
    }
}

// After the direct form (exact thresholds only, no tile sums): the sums come
// from the sent list itself.
//
// The first output slot of each tensor, where the sums are taken by slices or
// one block of k_dmeans cannot find them on the way (kMeansLocalT tensors).
constexpr int kMeansThreads = 1024;
constexpr uint32_t kMeansLocalT = kMeansThreads - 1;
// Sent entries that one block per tensor sums directly; more are summed per
// slice first.  One block of 1,024 threads takes about 0.1 us per 1,024 entries.
constexpr uint32_t kMeansDirectK = 65536;

__global__ __launch_bounds__(kMeansThreads) void k_qbase(QuantArgs q) {
    __shared__ uint32_t lds[kMeansThreads / kWave + 1];
    uint32_t carry = 0;
    for (uint32_t t0 = 0; t0 < q.T; t0 += kMeansThreads) {
        const uint32_t t = t0 + threadIdx.x;
        uint32_t total;
        const uint32_t excl = block_excl_scan<kMeansThreads>(t < q.T ? q.tensor_counts[t] : 0u, lds, &total);
        if (t < q.T) q.qbase[t] = carry + excl;
        carry += total;
    }
    if (threadIdx.x == 0) q.qbase[q.T] = carry;
}

// Sums of four doubles over a block of NT threads, in every thread.
template <int NT>
__device__ __forceinline__ void block_sum4(double v[4], double* lds) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = wave_sum(v[i]);
    if (lane_id() == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) lds[4 * (threadIdx.x / kWave) + i] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = lds[i];
        for (int w = 1; w < NT / kWave; ++w) v[i] += lds[4 * w + i];
    }
    __syncthreads();
}

// One more sent value into the sums and counts (positive sum, negative sum,
// positive count, negative count).
__device__ __forceinline__ void add_value(double v[4], float x) {
    if (x < 0.0f) {
        v[1] += (double)x;
        v[3] += 1.0;
    } else {
        v[0] += (double)x;
        v[2] += 1.0;
    }
}

// Sums of every slice of kQSlice sent entries: per tensor under the sign mean
// (slice j and tensor t have record j + t: along the list either grows from
// one pair to the next, so a tensor's records are consecutive), else over all.
// A slice inside one tensor is summed by the block.  Else the slice is staged
// in LDS and its tensors are dealt out, those of at most kQThreadSum entries to
// threads and the others, at most 124, to waves: a slice may hold thousands of
// tensors, and summing each with the block waited at four barriers a tensor
// (100,000 entries of 3,000 tensors: 249 us a call, the candidate form 110; now 67).
constexpr uint32_t kQThreadSum = 32;

__global__ __launch_bounds__(kBlock) void k_qsum(QuantArgs q) {
    __shared__ double lds[4 * kWavesPerBlock];
    __shared__ float xs[kQSlice];
    __shared__ uint32_t more[kQSlice / (kQThreadSum + 1) + 1], nmore;
    const int tid = threadIdx.x;
    constexpr int PER = kQSlice / kBlock;
    const uint64_t j0 = (uint64_t)blockIdx.x * kQSlice, j1 = j0 + kQSlice < q.k_total ? j0 + kQSlice : q.k_total;
    const bool own = q.qkind == kQuantSignMean;
    float x[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint64_t j = j0 + i * kBlock + tid;
        x[i] = j < j1 ? q.val[j] : 0.0f;
    }
    const auto base = [&](uint32_t t) { return q.qbase[t]; };
    const uint32_t t0 = own ? wave_last_at_most(base, q.T, (uint32_t)j0) : 0u;
    if (!own || q.qbase[t0 + 1] >= j1) {  // (block-uniform)
        double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (j0 + i * kBlock + tid < j1) add_value(v, x[i]);
        block_sum4<kBlock>(v, lds);
        if (tid == 0)
            for (int i = 0; i < 4; ++i) q.tq[4 * ((size_t)blockIdx.x + t0) + i] = v[i];
        return;
    }
    const uint32_t t1 = wave_last_at_most(base, q.T, (uint32_t)(j1 - 1));
    if (tid == 0) nmore = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) xs[i * kBlock + tid] = x[i];
    __syncthreads();
    for (uint32_t t = t0 + tid; t <= t1; t += kBlock) {
        const uint32_t b = q.qbase[t] > j0 ? q.qbase[t] - (uint32_t)j0 : 0u;
        const uint32_t e = (uint32_t)((q.qbase[t + 1] < j1 ? q.qbase[t + 1] : j1) - j0);
        if (b >= e) continue;  // no entry of its own: nobody reads the record
        if (e - b > kQThreadSum) {
            more[atomicAdd(&nmore, 1u)] = t;
            continue;
        }
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (uint32_t i = b; i < e; ++i) add_value(v, xs[i]);
        for (int i = 0; i < 4; ++i) q.tq[4 * ((size_t)blockIdx.x + t) + i] = v[i];
    }
    __syncthreads();
    for (uint32_t d = wave_index(); d < nmore; d += kWavesPerBlock) {
        const uint32_t t = more[d];
        const uint32_t b = q.qbase[t] > j0 ? q.qbase[t] - (uint32_t)j0 : 0u;
        const uint32_t e = (uint32_t)((q.qbase[t + 1] < j1 ? q.qbase[t + 1] : j1) - j0);
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (uint32_t i = b + lane_id(); i < e; i += kWave) add_value(v, xs[i]);
        for (int i = 0; i < 4; ++i) {
            v[i] = wave_sum(v[i]);
            if (lane_id() == 0) q.tq[4 * ((size_t)blockIdx.x + t) + i] = v[i];
        }
    }
}

// The centres of tensor t under threshold centres: the smallest kept magnitude
// of the segment is the exact threshold key.
__device__ __forceinline__ void threshold_centres(const QuantArgs& q, uint32_t t, float& pos, float& neg) {
    const uint32_t s = q.per_tensor ? t : 0u;
    pos = neg = 0.0f;
    if (keep_of(q.seg_off[s + 1] - q.seg_off[s], q.keep_ppm) > 0) {
        pos = __uint_as_float(q.seg[s].thr);
        neg = __uint_as_float(q.seg[s].thr | 0x80000000u);
    }
}
__device__ __forceinline__ void mean_centres(const double v[4], float& pos, float& neg) {
    pos = v[2] > 0.0 ? (float)(v[0] / v[2]) : 0.0f;
    neg = v[3] > 0.0 ? (float)(v[1] / v[3]) : 0.0f;
}

// Centres per tensor of more than kMeansLocalT tensors (sign means from the
// slices' sums, threshold centres), a wave each: few entries or records to a
// tensor, so blocks of their own were mostly launch.
__global__ __launch_bounds__(kBlock) void k_tmeans(QuantArgs q) {
    const uint32_t t = blockIdx.x * kWavesPerBlock + wave_index();
    if (t >= q.T) return;
    float pos, neg;
    if (q.qkind == kQuantThreshold) {
        threshold_centres(q, t, pos, neg);
    } else {
        const uint32_t a = q.qbase[t], b = q.qbase[t + 1];
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (uint32_t r = a / kQSlice + lane_id(); a < b && r <= (b - 1) / kQSlice; r += kWave)
            for (int i = 0; i < 4; ++i) v[i] += q.tq[4 * ((size_t)r + t) + i];
        for (int i = 0; i < 4; ++i) v[i] = wave_sum(v[i]);
        mean_centres(v, pos, neg);
    }
    if (lane_id() == 0) {
        q.means[2 * t + 0] = pos;
        q.means[2 * t + 1] = neg;
    }
}

// Centres per tensor (every kind but the column mean) and the first output
// slot of each tensor.  One block per tensor; under the global mean, whose
// centres are the same for every tensor, one block in all (a block per tensor,
// each summing the whole list, took 244 us a call at 62,000 entries and 3,000
// tensors, the candidate form 130; now 98).
__global__ __launch_bounds__(kMeansThreads) void k_dmeans(QuantArgs q, uint32_t sliced, uint32_t have_base) {
    constexpr int NT = kMeansThreads, U = 8;
    __shared__ double lds[4 * (NT / kWave)];
    __shared__ uint32_t first[NT + 1], scan[NT / kWave + 1];
    const int tid = threadIdx.x;
    const uint32_t t = blockIdx.x;
    const uint32_t* qbase = q.qbase;
    if (!have_base) {
        uint32_t total;
        const uint32_t excl = block_excl_scan<NT>((uint32_t)tid < q.T ? q.tensor_counts[tid] : 0u, scan, &total);
        first[tid] = excl;
        if (t == 0 && (uint32_t)tid <= q.T) q.qbase[tid] = excl;
        __syncthreads();
        qbase = first;
    }
    if (q.qkind == kQuantColumnMean) return;
    float pos = 0.0f, neg = 0.0f;
    if (q.qkind == kQuantThreshold) {
        threshold_centres(q, t, pos, neg);
    } else {
        const bool own = q.qkind == kQuantSignMean;
        const uint32_t a = own ? qbase[t] : 0u, b = own ? qbase[t + 1] : qbase[q.T];
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        if (sliced) {
            for (uint32_t r = a / kQSlice + tid; a < b && r <= (b - 1) / kQSlice; r += NT)
                for (int i = 0; i < 4; ++i) v[i] += q.tq[4 * ((size_t)r + (own ? t : 0u)) + i];
        } else {
            for (uint32_t j = a + tid; j < b; j += U * NT) {
                float x[U];
#pragma unroll
                for (int i = 0; i < U; ++i) x[i] = b - j > (uint32_t)i * NT ? q.val[j + i * NT] : 0.0f;
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (b - j > (uint32_t)i * NT) add_value(v, x[i]);
            }
        }
        block_sum4<NT>(v, lds);
        mean_centres(v, pos, neg);
    }
    const uint32_t end = q.qkind == kQuantGlobalMean ? q.T : t + 1;
    for (uint32_t u = t + tid; u < end; u += NT) {
        q.means[2 * (size_t)u + 0] = pos;
        q.means[2 * (size_t)u + 1] = neg;
    }
}

// Column sums of the sent entries, per sign, with the first output slot of
// each tensor where one block can find them on the way (T <= kColLocalT).  Each
// block takes a slice of PER * kBlock consecutive output slots, every thread
// PER of them, loaded at once.  The entries of a tensor with at least kPerCol
// of them per column in the slice are summed in LDS first (fp64 LDS atomics),
// each touched column then added to the global sums once; the entries of the
// others, few to a column, are added directly.  A tensor's columns lie in LDS
// where its entries lie in the slice, so all tensors of a slice have room at
// once, and are cleared, summed and added together: a slice may hold thousands
// of small tensors (1.6M entries of 8,000 one-column tensors, summed one tensor
// after another: 347 us a call; where more than 16 tensors in a slice were
// added directly, 474; now 339).  Bound by the chain of loads, then the global
// atomics (about 16 G/s).  It took 16.8 us for 21,000 entries of a ragged 21M-element
// layout in slices of 4,096, one entry after another, and 27.0 with the passes
// for the first slots, the centres and the values; now 6.8 and 10.7.
constexpr uint32_t kColLocalT = kBlock - 1;

// LOCAL: the first slots found on the way (a choice at run time would read them
// with flat loads, which wait for all the values in flight).
template <int PER, bool LOCAL>
__global__ __launch_bounds__(kBlock) void k_colsum(QuantArgs q) {
    constexpr uint32_t kSlice = PER * kBlock;
    constexpr uint32_t kPerCol = PER > 8 ? 2 : 1, kCols = kSlice / kPerCol;  // 48 KB of sums and counts at most
    __shared__ double ls[2 * kCols];
    __shared__ uint32_t lc[2 * kCols];
    __shared__ uint32_t first[LOCAL ? kBlock : 1], scan[kBlock / kWave + 1];
    const int tid = threadIdx.x;
    const uint64_t j0 = (uint64_t)blockIdx.x * kSlice;
    float x[PER];
    uint32_t ix[PER];
    const auto load = [&] {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint64_t at = j0 + i * kBlock + tid;
            x[i] = at < q.k_total ? __uint_as_float(load_early(reinterpret_cast<const uint32_t*>(q.val) + at)) : 0.0f;
            ix[i] = at < q.k_total ? load_early(q.idx + at) : 0u;
        }
    };
    if (!q.sampled) load();
    if (LOCAL) {
        uint32_t all;
        const uint32_t excl = block_excl_scan<kBlock>((uint32_t)tid < q.T ? q.tensor_counts[tid] : 0u, scan, &all);
        first[tid] = excl;
        if (blockIdx.x == 0 && (uint32_t)tid <= q.T) q.qbase[tid] = excl;
        __syncthreads();
    }
    const auto base = [&](uint32_t t) { return LOCAL ? first[t] : q.qbase[t]; };
    const uint32_t total = base(q.T);
    if (j0 >= total) return;
    if (q.sampled) load();  // (most blocks of a large capacity lie past what is sent)
    const uint32_t j1 = j0 + kSlice < total ? (uint32_t)j0 + kSlice : total;
    const auto clear = [&](uint32_t n) {
        for (uint32_t i = tid; i < n; i += kBlock) {
            ls[i] = 0.0;
            lc[i] = 0;
        }
        __syncthreads();
    };
    const auto add = [&](double* sum, uint32_t* cnt, uint32_t slot, float v) {
        const uint32_t sl = 2 * slot + (v < 0.0f ? 1u : 0u);
        unsafeAtomicAdd(&sum[sl], (double)v);
        atomicAdd(&cnt[sl], 1u);
    };
    const uint32_t t0 = __builtin_amdgcn_readfirstlane(wave_last_at_most(base, q.T, (uint32_t)j0));  // of slot j0
    if (base(t0 + 1) >= j1) {  // the whole slice (block-uniform)
        const uint32_t C = q.columns[t0], cb = q.colbase[t0], off = q.tensor_off[t0];
        const bool lds = (uint64_t)C * kPerCol <= j1 - (uint32_t)j0;
        if (lds) clear(2 * C);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (j0 + i * kBlock + tid >= j1) continue;
            const uint32_t col = (ix[i] - off) % C;
            if (lds) add(ls, lc, col, x[i]);
            else add(q.csum, q.ccnt, cb + col, x[i]);
        }
        __syncthreads();
        for (uint32_t i = tid; lds && i < 2 * C; i += kBlock)
            if (lc[i]) {
                unsafeAtomicAdd(&q.csum[2 * cb + i], ls[i]);
                atomicAdd(&q.ccnt[2 * cb + i], lc[i]);
            }
        return;
    }
    const uint32_t t1 = wave_last_at_most(base, q.T, j1 - 1);
    // tensor of slot j of the slice: the last t with base(t) <= j
    const auto tensor_at = [&](uint32_t j) {
        uint32_t lo = t0, hi = t1 + 1;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (base(mid) <= j) lo = mid;
            else hi = mid;
        }
        return lo;
    };
    // tensor t's first entry in the slice, and its first column in LDS (kPerCol
    // slots on for each further column, the slot still is one of t's entries)
    const auto from = [&](uint32_t t) { return base(t) > (uint32_t)j0 ? base(t) - (uint32_t)j0 : 0u; };
    const auto lds_col = [&](uint32_t t) { return (from(t) + kPerCol - 1) / kPerCol; };
    clear(2 * kCols);
    uint32_t ten[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint64_t at = j0 + i * kBlock + tid;
        ten[i] = tensor_at(at < j1 ? (uint32_t)at : j1 - 1);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (j0 + i * kBlock + tid >= j1) continue;
        const uint32_t t = ten[i], C = q.columns[t], col = (ix[i] - q.tensor_off[t]) % C;
        const uint32_t n = (base(t + 1) < j1 ? base(t + 1) : j1) - (uint32_t)j0 - from(t);  // t's entries in the slice
        if ((uint64_t)C * kPerCol <= n) add(ls, lc, lds_col(t) + col, x[i]);
        else add(q.csum, q.ccnt, q.colbase[t] + col, x[i]);
    }
    __syncthreads();
    for (uint32_t i = tid; i < 2 * kCols; i += kBlock) {
        if (lc[i] == 0) continue;
        const uint32_t t = tensor_at((uint32_t)j0 + (i >> 1) * kPerCol);
        const uint32_t sl = 2 * (q.colbase[t] + (i >> 1) - lds_col(t)) + (i & 1u);
        unsafeAtomicAdd(&q.csum[sl], ls[i]);
        atomicAdd(&q.ccnt[sl], lc[i]);
    }
}

// Column-wise centre from the column's sum and count (no entries: the sum is
// clear and the centre 0; without a branch both loads are in flight at once).
__device__ __forceinline__ float col_centre(const QuantArgs& q, uint32_t g) {
    const uint32_t n = q.ccnt[g];
    return (float)(q.csum[g] / (double)(n ? n : 1u));
}

template <bool COLUMN>
__global__ __launch_bounds__(kBlock) void k_quant(QuantArgs q) {
    const uint64_t j = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    // column-wise centres are given out here, and each entry forms its own
    if (COLUMN && j < q.groups) {
        q.means[2 * j + 0] = col_centre(q, 2 * (uint32_t)j);
        q.means[2 * j + 1] = col_centre(q, 2 * (uint32_t)j + 1);
    }
    // entries sent (the grid covers k_total >= total; the first slots are not formed where that is 0)
    const uint64_t total = !COLUMN || q.k_total ? q.qbase[q.T] : 0u;
    const bool valid = j < total;
    bool neg = false;
    if (valid) {
        // both in flight at once, and during the search (where the index waited for the
        // value, a call that sends 20M entries took 711 us; now 692)
        const uint32_t i = load_early(q.idx + j);
        const float x = __uint_as_float(load_early(reinterpret_cast<const uint32_t*>(q.val) + j));
        neg = x < 0.0f;
        // tensor of output slot j: the last t with qbase[t] <= j
        uint32_t lo = 0, hi = q.T;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (q.qbase[mid] <= j) lo = mid;
            else hi = mid;
        }
        const float centre = COLUMN ? col_centre(q, 2 * (q.colbase[lo] + (i - q.tensor_off[lo]) % q.columns[lo]) + (neg ? 1u : 0u))
                             : neg  ? q.means[2 * lo + 1]
                                    : q.means[2 * lo + 0];
        if (i < q.N) q.res[i] = x - centre;
    }
    const uint64_t m = ballot(valid && neg);
    const uint64_t jw = j - lane_id();  // first slot of this wave, a multiple of 64
    const uint64_t words = (total + 31) / 32;
    if (lane_id() == 0 && jw / 32 < words) q.sign_bits[jw / 32] = (uint32_t)m;
    if (lane_id() == 1 && jw / 32 + 1 < words) q.sign_bits[jw / 32 + 1] = (uint32_t)(m >> 32);
}

static inline uint32_t blocks_for_waves(uint32_t waves) { return (waves + kWavesPerBlock - 1) / kWavesPerBlock; }

hipError_t launch_quant(const QuantArgs& q, hipStream_t st) {
    const bool column = q.qkind == kQuantColumnMean;
    // k_colsum finds the first slots itself, but where most of its blocks may only
    // find that they lie past the entries sent (40M elements, a capacity of all of
    // them, 400,000 sent: 245 us a call, with the first slots by a pass of their
    // own and no values read there 170)
    const bool local = column && q.T <= kColLocalT && !(q.sampled && q.k_total > kColMidK);
    if (!local && q.direct) {
        const bool sums = q.qkind == kQuantSignMean || q.qkind == kQuantGlobalMean;
        const bool many = q.T > kMeansLocalT, own = q.qkind != kQuantGlobalMean;
        const bool sliced = sums && (q.k_total > kMeansDirectK || (many && own && q.k_total > 0)), base = sliced || many;
        if (base) hipLaunchKernelGGL(k_qbase, dim3(1), dim3(kMeansThreads), 0, st, q);
        if (sliced) hipLaunchKernelGGL(k_qsum, dim3((uint32_t)((q.k_total + kQSlice - 1) / kQSlice)), dim3(kBlock), 0, st, q);
        // (column means need the first slots only, of one block)
        if (!column && many && own)
            hipLaunchKernelGGL(k_tmeans, dim3(blocks_for_waves(q.T)), dim3(kBlock), 0, st, q);
        else if (!column || !base)
            hipLaunchKernelGGL(k_dmeans, dim3(column || !own ? 1u : q.T), dim3(kMeansThreads), 0, st, q, sliced ? 1u : 0u,
                               base ? 1u : 0u);
    } else if (!local) {
        hipLaunchKernelGGL(k_means, dim3(blocks_for_waves(q.T)), dim3(kBlock), 0, st, q);
    }
    if (column && q.k_total > 0) {
        // Short slices fill the device from few entries; of many, long ones save
        // adds to columns that many blocks share (a call with slices of 1,024 /
        // 2,048 / 4,096 in us: 120,000 entries over 200 columns x 6 tensors 94 /
        // 96 / 100; 21,000 ragged ones 100 / 103 / 111, of 256 98; 960,000 over 8
        // 132 / 126 / 124; 4.25M over 500 381 / 336 / 322).  Under a sampled
        // threshold k_total is only a bound, and often far above what is sent (this
        // pass at 50,000 sent of 5M in slices of 2,048 / 4,096: 11.5 / 14.5 us).
        const uint32_t per = q.k_total <= kColTinyK ? 1u : q.k_total <= kColSmallK ? 4u : q.k_total <= kColMidK || q.sampled ? 8u : 16u;
        const uint32_t slice = per * kBlock;
        const dim3 g((uint32_t)((q.k_total + slice - 1) / slice));
        auto sums = per == 1   ? (local ? k_colsum<1, true> : k_colsum<1, false>)
                    : per == 4 ? (local ? k_colsum<4, true> : k_colsum<4, false>)
                    : per == 8 ? (local ? k_colsum<8, true> : k_colsum<8, false>)
                               : (local ? k_colsum<16, true> : k_colsum<16, false>);
        hipLaunchKernelGGL(sums, g, dim3(kBlock), 0, st, q);
    }
    const uint64_t items = std::max<uint64_t>(q.k_total, column ? q.groups : 0u);
    if (items > 0) {
        const dim3 g((uint32_t)((items + kBlock - 1) / kBlock));
        if (column) hipLaunchKernelGGL(k_quant<true>, g, dim3(kBlock), 0, st, q);
        else hipLaunchKernelGGL(k_quant<false>, g, dim3(kBlock), 0, st, q);
    }
    return hipGetLastError();
}

}  // namespace gd
