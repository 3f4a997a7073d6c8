// The direct form of the exact compressor, for gradients small enough that
// reading every element in every pass costs less than sampling a bracket and
// compacting candidates (gfx950, wave64).
//
//   k_dacc     : acc = gradient + residual, written back where it changes, and
//                the histogram of the top 11 key bits.
//   k_dhist    : that digit of the k-th largest key, and the histogram of the
//                next 11 bits among the keys that share it.
//   k_dcollect : the second digit; per piece, the keys above the 22-bit prefix
//                and those that share it.
//   k_demit    : the threshold among those, and the kept pairs in order.
//
// Four launches in place of the candidate form's ten, with no sample, so
// nothing can miss.  Each pass is bound by its chain of dependent reads and
// barriers (histogram copies, pick, elements; records, keys, counts) at the
// small end, 5 to 8 us each at 0.67M elements (24.8 us a call; the candidate
// form 52.9), and by reading every element again at the large end.
//
// The flat gradient is cut into chunks of consecutive 1024-element units.  A
// piece is the part of one threshold segment inside one chunk, and has a block
// of its own: a chunk holds one piece under a global threshold, and one per
// overlapping tensor under a per-tensor one (a block that took them one after
// another waited through every pass's chain of reads once per piece: 12.0
// against 5.7 us a pass where one chunk holds three).  Piece (chunk c, segment s) has
// the index c + s: along the gradient c or s grows from each piece to the
// next, so indices are distinct and ascending, and one segment's pieces are
// consecutive.  k_dcollect leaves a record per piece; the emitting block of a
// piece reads its segment's records, resolves the threshold among the bin's
// keys and counts what the earlier pieces keep, so no pass over the data and
// no device-wide atomics are needed between the 22-bit prefix and the sent list
// (but for the counts per tensor under a global threshold).
//
// The line between the forms (kDirectMaxUnits) was drawn under one threshold over
// an MLP; it holds over numbers of tensors and scopes too, evenly cut, direct
// against candidate form, us a call: 0.3M elements, 1 tensor 24 / 52, 1,024 per
// tensor 71 / 159, 10,000 per tensor 119 / 983; 6.2M, global 51 / 69 (1 tensor),
// 72 / 75 (1,025), 75 / 721 (50,000); per tensor 58 / 71 (27), 83 / 101 (256),
// 123 / 196 (1,024), 92 / 197 (1,025), 294 / 1,285 (10,000).

#include <hip/hip_ext.h>

#include "gd_kernels.h"

namespace gd {

constexpr uint32_t kFewBits = 9;                 // low key bits below the prefix that two digits leave
constexpr uint32_t kBinKeys = 1u << kFewBits;    // keys of such a bin
constexpr uint32_t kListKeys = 16;               // a piece with more different keys in the bin stores counts
constexpr uint32_t kDenseFlag = 0x80000000u;     // in PieceInfo::in: suffix counts stored in place of keys

struct Piece {
    uint32_t c, s, ea, eb;  // chunk, segment, elements [ea, eb)
    uint32_t sa, sb;        // the whole segment
};

__device__ __forceinline__ uint32_t chunk_of(const DirectArgs& a, uint32_t e) { return e >> a.cshift; }

// The piece with index j (one block each); false where there is none: segment
// s has pieces chunk_of(start) + s and on, so s is the last segment whose
// first index is at most j.
__device__ __forceinline__ bool piece_of(const DirectArgs& a, uint32_t j, Piece& p) {
    p.s = 0;
    p.sa = 0;
    p.sb = a.N;
    if (a.per_tensor) {
        if (a.S <= (uint32_t)kWave) {  // one load for all of them
            const uint32_t t = lane_id();
            const bool at = t < a.S && chunk_of(a, a.tensor_off[t < a.S ? t : 0u]) + t <= j;
            p.s = popc64(ballot(at)) - 1u;  // (segment 0 starts at index 0)
        } else {
            uint32_t hi = a.S;
            while (hi - p.s > 1) {
                const uint32_t mid = (p.s + hi) >> 1;
                if (chunk_of(a, a.tensor_off[mid]) + mid <= j) p.s = mid;
                else hi = mid;
            }
        }
        p.sa = a.tensor_off[p.s];
        p.sb = a.tensor_off[p.s + 1];
    }
    p.c = j - p.s;
    if (p.sa >= p.sb || p.c > chunk_of(a, p.sb - 1)) return false;
    const uint32_t cs = p.c << a.cshift, len = 1u << a.cshift;
    p.ea = p.sa > cs ? p.sa : cs;
    p.eb = p.sb - cs > len ? cs + len : p.sb;
    return true;
}

// First element of segment s (starting at sa) in the piece with index j.
__device__ __forceinline__ uint32_t piece_start(const DirectArgs& a, uint32_t s, uint32_t sa, uint32_t j) {
    const uint32_t cs = (j - s) << a.cshift;
    return cs > sa ? cs : sa;
}

// Vector of x at element e (a multiple of 4 below N), elements past the end as 0.
__device__ __forceinline__ f4 load4(const float* x, uint32_t e, uint32_t N) {
    if (N - e >= 4) return *reinterpret_cast<const f4*>(x + e);
    f4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 3; ++q)
        if ((uint32_t)q < N - e) v[q] = x[e + q];
    return v;
}

// Rank query on a histogram of NB bins in COPIES copies, by the whole block:
// the bin of the r-th largest key (r >= 1) and the number of keys in higher
// bins.  Returns the histogram's total; digit and above are meaningful only
// when r is at most that.
template <int NT, int NB, int COPIES>
__device__ __forceinline__ uint32_t block_pick(const uint32_t* hist, uint32_t r, uint32_t* lds, uint32_t& digit,
                                               uint32_t& above) {
    constexpr int PER = NB > NT ? NB / NT : 1;
    static_assert(PER == 8 || PER == 4 || PER == 2 || PER == 1, "bins per thread");
    const int tid = threadIdx.x;
    const int top = NB - PER * tid;  // this thread owns bins [top - PER, top) (none when top <= 0)
    uint32_t c[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) c[i] = 0;
    if (PER > 1 || top > 0) {
#pragma unroll
        for (int j = 0; j < COPIES; ++j) {
            const uint32_t* p = hist + j * NB + top - PER;
            if (PER >= 4) {
#pragma unroll
                for (int i = 0; i < PER / 4; ++i) {
                    const uint4 x = reinterpret_cast<const uint4*>(p)[i];
                    c[4 * i % PER] += x.x, c[(4 * i + 1) % PER] += x.y, c[(4 * i + 2) % PER] += x.z, c[(4 * i + 3) % PER] += x.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < PER; ++i) c[i] += p[i];
            }
        }
    }
    uint32_t sum = 0, total;
#pragma unroll
    for (int i = 0; i < PER; ++i) sum += c[i];
    const uint32_t excl = block_excl_scan<NT>(sum, lds, &total);
    uint32_t* out = lds + NT / kWave + 1;
    if (excl < r && r <= excl + sum) {
        uint32_t acc = excl;
        bool found = false;
#pragma unroll
        for (int i = PER - 1; i >= 0; --i) {  // high to low
            if (!found && acc + c[i] >= r) {
                out[0] = (uint32_t)(top - PER + i);
                out[1] = acc;
                found = true;
            }
            acc += c[i];
        }
    }
    __syncthreads();
    digit = __builtin_amdgcn_readfirstlane(out[0]);
    above = __builtin_amdgcn_readfirstlane(out[1]);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(total);
}
template <int NT>
constexpr int kPickLds = NT / kWave + 1 + 2;

// block_pick over kHistCopies copies, or the one that a layout of many tensors keeps.
template <int NT, int NB>
__device__ __forceinline__ uint32_t block_pick_copies(const uint32_t* hist, uint32_t copies, uint32_t r, uint32_t* lds,
                                                      uint32_t& digit, uint32_t& above) {
    return copies == kHistCopies ? block_pick<NT, NB, kHistCopies>(hist, r, lds, digit, above)
                                 : block_pick<NT, NB, 1>(hist, r, lds, digit, above);
}

// Clears the block's LDS histogram (and waits).
template <int NT, int NB = kSelBins>
__device__ __forceinline__ void clear_hist(uint32_t* h) {
    for (int i = threadIdx.x; i < NB; i += NT) h[i] = 0;
    __syncthreads();
}

// Adds the block's LDS histogram to the segment's (and waits at both ends).
template <int NT, int NB = kSelBins>
__device__ __forceinline__ void flush_hist(const uint32_t* h, uint32_t* g) {
    __syncthreads();
    for (int i = threadIdx.x; i < NB; i += NT)
        if (h[i]) atomicAdd(&g[i], h[i]);
    __syncthreads();
}

// Adds 1 to h[bin] for every active lane of the wave; lanes that all hold one
// bin (equal values) add once.
__device__ __forceinline__ void hist_add_wave(uint32_t* h, uint32_t bin, bool active) {
    const uint64_t m = ballot(active);
    if (m == 0) return;
    const int first = __ffsll((unsigned long long)m) - 1;
    const uint32_t b0 = lane_value(bin, first);
    if (ballot(active && bin == b0) == m) {
        if (lane_id() == first) atomicAdd(&h[b0], popc64(m));
    } else if (active) {
        atomicAdd(&h[bin], 1u);
    }
}

// The per-call state that does not depend on the data: the first output slot
// of each segment, where one segment is one tensor the kept counts, and the
// state of the segments that keep nothing, which no later pass touches.
// Run by one block.
template <int NT>
__device__ __forceinline__ void call_prologue(const uint32_t* seg_off, uint32_t S, uint32_t T, uint32_t keep_ppm,
                                              uint64_t* out_base, uint32_t* tensor_counts, SegState* seg,
                                              uint32_t* lds) {
    const int tid = threadIdx.x;
    const bool own = S == T;  // a segment is a tensor: k is its kept count
    uint64_t carry = 0;
    for (uint32_t b0 = 0; b0 < S; b0 += NT) {
        const uint32_t s = b0 + tid;
        const uint32_t k = s < S ? keep_of(seg_off[s + 1] - seg_off[s], keep_ppm) : 0u;
        uint32_t total;
        const uint32_t excl = block_excl_scan<NT>(k, lds, &total);
        if (s < S) {
            out_base[s] = carry + excl;
            if (own) tensor_counts[s] = k;
            if (k == 0) {
                SegState& g = seg[s];
                g.clo = g.miss = g.need = g.zero = 0;
                g.thr = kNoKey;
            }
        }
        carry += total;
    }
    if (!own)
        for (uint32_t t = tid; t < T; t += NT) tensor_counts[t] = 0;  // summed by the emitting pass
}

// What the emitting block of a piece needs to know of its segment.
struct Resolved {
    uint32_t thr;    // the threshold key T
    uint32_t need;   // keys equal to T to keep, lowest index first
    uint32_t above;  // keys above T in the segment's earlier pieces
    uint32_t equal;  // keys equal to T there
};

// What a piece leaves of its keys in the bin: nothing, one value (`in` times),
// a list of `in` keys, or (kDenseFlag) the number of its keys at or above each
// of the bin's values.  Lists are short but for the segment's first and last
// piece, which may be too short to store counts.
__device__ __forceinline__ bool one_key(const PieceInfo& p) { return p.kmin == p.kmax; }
__device__ __forceinline__ bool long_list(const PieceInfo& p) {
    return !(p.in & kDenseFlag) && p.in > kListKeys && !one_key(p);
}
// Keys at or above bin value x (0 to kBinKeys) of a piece that stores counts.
__device__ __forceinline__ uint32_t dense_ge(const DirectArgs& a, uint32_t at, uint32_t x) {
    return x < kBinKeys ? a.ent[at + x] : 0u;
}

// Keys above and equal to thr among the bin's keys of one piece (a long list's
// not counted).
__device__ __forceinline__ void count_piece(const DirectArgs& a, const PieceInfo& p, uint32_t at, uint32_t lo, uint32_t thr,
                                            uint32_t& g, uint32_t& e) {
    const uint32_t n = p.in & ~kDenseFlag;
    if (n == 0 || p.kmax < thr) return;
    if (p.kmin > thr) {
        g += n;
    } else if (one_key(p)) {
        e += n;
    } else if (p.in & kDenseFlag) {
        const uint32_t ge = dense_ge(a, at, thr - lo), gt = dense_ge(a, at, thr - lo + 1);
        g += gt;
        e += ge - gt;
    } else if (!long_list(p)) {
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t k = a.ent[at + i];
            g += k > thr;
            e += k == thr;
        }
    }
}

// Resolves the threshold of segment s (its bin: keys [lo, lo + 2^bits), the
// r-th largest of them) from the pieces' records, and counts the keys above
// and equal to it in the pieces before `pair`.  Called by the whole block;
// h is a kSelBins-word LDS histogram.
//
// Every emitting block does this, so its work is bounded whatever the values: a
// thread reads the records of P / NT pieces (P at most 1,152), a list of at most
// kListKeys keys for each, and where pieces store counts one of them for each
// step of a search over the bin's nine bits.  (Adding up all counts of all
// pieces in every block took 1,735 us a call at 4.7M elements within 4,096
// neighbouring values, the candidate form 1,009; now 110.)
template <int NT>
__device__ Resolved resolve(const DirectArgs& a, uint32_t s, uint32_t sa, uint32_t sb, uint32_t pair, uint32_t lo,
                            uint32_t r, uint32_t* h, uint32_t* lds) {
    const int tid = threadIdx.x;
    const uint32_t j0 = chunk_of(a, sa) + s, j1 = chunk_of(a, sb - 1) + s + 1;
    uint32_t above = 0, kmin = kNoKey, kmax = 0, forms = 0;  // forms: 1, some piece stores counts; 2, a long list
    for (uint32_t j = j0 + tid; j < j1; j += NT) {
        const PieceInfo p = a.info[j];
        if (j < pair) above += p.gt;
        if (p.in) {
            kmin = min(kmin, p.kmin);
            kmax = max(kmax, p.kmax);
            forms |= (p.in >> 31) | (long_list(p) ? 2u : 0u);
        }
    }
    // sums and extremes over the block
    uint32_t* red = lds;  // [NT / 64][4]
    {
        const uint32_t x0 = wave_sum(above), x1 = wave_min(kmin), x2 = lane_value(wave_incl_max(kmax), kWave - 1);
        const uint64_t m1 = ballot((forms & 1u) != 0), m2 = ballot((forms & 2u) != 0);
        if (lane_id() == 0) {
            uint32_t* q = red + 4 * (threadIdx.x / kWave);
            q[0] = x0;
            q[1] = x1;
            q[2] = x2;
            q[3] = (m1 != 0 ? 1u : 0u) | (m2 != 0 ? 2u : 0u);
        }
        __syncthreads();
        above = 0, kmin = kNoKey, kmax = 0, forms = 0;
        for (int i = 0; i < NT / kWave; ++i) {
            above += red[4 * i];
            kmin = min(kmin, red[4 * i + 1]);
            kmax = max(kmax, red[4 * i + 2]);
            forms |= red[4 * i + 3];
        }
        __syncthreads();
        above = __builtin_amdgcn_readfirstlane(above);
        kmin = __builtin_amdgcn_readfirstlane(kmin);
        kmax = __builtin_amdgcn_readfirstlane(kmax);
        forms = __builtin_amdgcn_readfirstlane(forms);
    }
    // sums over the block, in every thread (waits at both ends)
    const auto block_sums = [&](uint32_t& u, uint32_t& v) {
        u = wave_sum(u);
        v = wave_sum(v);
        if (lane_id() == 0) {
            red[2 * (threadIdx.x / kWave)] = u;
            red[2 * (threadIdx.x / kWave) + 1] = v;
        }
        __syncthreads();
        u = v = 0;
        for (int i = 0; i < NT / kWave; ++i) {
            u += red[2 * i];
            v += red[2 * i + 1];
        }
        __syncthreads();
        u = __builtin_amdgcn_readfirstlane(u);
        v = __builtin_amdgcn_readfirstlane(v);
    };
    Resolved z{kmin, r, above, 0u};
    if (kmin < kmax) {  // (one key in the whole bin is the threshold)
        // the keys that are listed, by value
        clear_hist<NT, (int)kBinKeys>(h);
        for (uint32_t j = j0 + tid; j < j1; j += NT) {
            const PieceInfo p = a.info[j];
            if (p.in == 0) continue;
            if (one_key(p)) {
                atomicAdd(&h[p.kmin - lo], p.in);
            } else if (!(p.in & kDenseFlag) && !long_list(p)) {
                const uint32_t at = piece_start(a, s, sa, j);
                for (uint32_t i = 0; i < p.in; ++i) atomicAdd(&h[a.ent[at + i] - lo], 1u);
            }
        }
        // the first and the last piece
        for (uint32_t j = j0; j < j1 && (forms & 2u); j += max(j1 - 1 - j0, 1u)) {
            const PieceInfo p = a.info[j];
            const uint32_t at = piece_start(a, s, sa, j);
            for (uint32_t i = tid; long_list(p) && i < p.in; i += NT) atomicAdd(&h[a.ent[at + i] - lo], 1u);
        }
        __syncthreads();
        uint32_t d, ab;
        if (!(forms & 1u)) {
            block_pick<NT, (int)kBinKeys, 1>(h, r, lds, d, ab);
        } else {
            // h[x] = listed keys at or above x; then the largest x with at least r keys at or above it
            static_assert(kBinKeys == 2 * NT, "two values per thread");
            const int top = (int)kBinKeys - 2 * tid;
            const uint32_t c1 = h[top - 1], c0 = h[top - 2];
            uint32_t total;
            const uint32_t excl = block_excl_scan<NT>(c0 + c1, lds, &total);
            h[top - 1] = excl + c1;
            h[top - 2] = excl + c1 + c0;
            __syncthreads();
            d = 0, ab = 0;
            uint32_t end = kBinKeys;  // fewer than r keys at or above it: ab
            while (end - d > 1) {
                const uint32_t mid = (d + end) >> 1;
                uint32_t c = 0, none = 0;
                for (uint32_t j = j0 + tid; j < j1; j += NT) {
                    const PieceInfo p = a.info[j];
                    if (p.in & kDenseFlag) c += dense_ge(a, piece_start(a, s, sa, j), mid);
                }
                block_sums(c, none);
                c += h[mid];
                if (c >= r) {
                    d = mid;
                } else {
                    end = mid;
                    ab = c;
                }
            }
        }
        z.thr = lo + d;
        z.need = r - ab;
    }
    uint32_t g = 0, e = 0;
    for (uint32_t j = j0 + tid; j < pair; j += NT) count_piece(a, a.info[j], piece_start(a, s, sa, j), lo, z.thr, g, e);
    if ((forms & 2u) && j0 < pair) {  // (the last piece is not before another)
        const PieceInfo p = a.info[j0];
        for (uint32_t i = tid; long_list(p) && i < p.in; i += NT) {
            const uint32_t k = a.ent[sa + i];
            // as count_piece: a list all above or below the threshold is counted there
            if (p.kmin <= z.thr && z.thr <= p.kmax) {
                g += k > z.thr;
                e += k == z.thr;
            }
        }
    }
    block_sums(g, e);
    z.above += g;
    z.equal = e;
    return z;
}
template <int NT>
constexpr int kResolveLds = 4 * (NT / kWave) > kPickLds<NT> ? 4 * (NT / kWave) : kPickLds<NT>;

// A block takes one piece; wave w of it the units [w UPW, (w + 1) UPW) of the
// piece's chunk, each as four rows of 256 elements, one 16-byte vector per lane.
constexpr uint32_t kSmallPiece = 256;  // pieces of at most this many elements skip the LDS histogram

template <int UPW>
struct Rows {
    f4 v[4 * UPW];
};

// This wave's unit j of chunk c (it may lie past the last one).
template <int UPW>
__device__ __forceinline__ uint32_t wave_unit(const DirectArgs& a, uint32_t c, int j) {
    return c * (kDirectThreads / kWave * UPW) + wave_index() * UPW + j;
}
// First element of this lane's vector in row i of unit u (it may lie past the last element).
__device__ __forceinline__ uint32_t row_elem(uint32_t u, int i) { return u * kUnitLen + i * 256 + 4 * lane_id(); }

// acc of the wave's elements: the residual, which holds it, or params - copy.
template <int UPW, bool PULL>
__device__ __forceinline__ void load_rows(const DirectArgs& a, uint32_t c, Rows<UPW>& x) {
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        const uint32_t u = wave_unit<UPW>(a, c, j);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f4 v = {0.f, 0.f, 0.f, 0.f};
            const uint32_t e = row_elem(u, i);
            if (u < a.C && e < a.N) {
                if (PULL) v = load4(a.pull_p, e, a.N) - load4(a.pull_copy, e, a.N);
                else v = load4(a.res, e, a.N);
            }
            x.v[4 * j + i] = v;
        }
    }
}

// Calls f(key, e, valid) for the wave's elements in the units that overlap
// piece p, valid for those inside it.  All lanes call it together.
template <int UPW, typename F>
__device__ __forceinline__ void for_keys(const DirectArgs& a, uint32_t c, const Piece& p, const Rows<UPW>& x, F&& f) {
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        const uint32_t u = wave_unit<UPW>(a, c, j);
        const uint32_t us = u * kUnitLen;
        if (u >= a.C || us >= p.eb || (p.ea > us && p.ea - us >= kUnitLen)) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t e = row_elem(u, i) + q;
                f(key_of(x.v[4 * j + i][q]), e, e - p.ea < p.eb - p.ea);
            }
    }
}

// Pass 1: the top digit from its histogram, then the next 11 bits among the
// keys that share it.  Fewer nonzero keys than k: the threshold is key 0 (the
// zero mode).
template <int NT, int UPW, bool PULL>
__device__ __forceinline__ void direct_hist1(const DirectArgs& a, uint32_t* h, uint32_t* lds) {
    Piece p;
    if (!piece_of(a, blockIdx.x, p)) return;
    const uint32_t c = p.c;
    Rows<UPW> x;
    load_rows<UPW, PULL>(a, c, x);
    const uint32_t k = keep_of(p.sb - p.sa, a.keep_ppm);
    uint32_t d0, above;
    if (k == 0) return;
    const uint32_t nz =
        block_pick_copies<NT, kSelBins>(a.h0 + (size_t)p.s * a.copies * kSelBins, a.copies, k, lds, d0, above);
    const bool zero = nz < k;
    if (p.ea == p.sa && threadIdx.x == 0) {
        SegState& g = a.seg[p.s];
        g.d0 = d0;
        g.r1 = k - above;
        g.clo = nz;
        g.zero = zero;
        g.miss = 0;
    }
    if (zero) return;
    uint32_t* g = a.h1 + ((size_t)p.s * a.copies + blockIdx.x % a.copies) * kSelBins;
    const bool small = p.eb - p.ea <= kSmallPiece;
    if (!small) clear_hist<NT>(h);
    for_keys<UPW>(a, c, p, x, [&](uint32_t key, uint32_t, bool in) {
        const bool hit = in && key >> kSel0Shift == d0;
        if (ballot(hit) == 0) return;
        if (small) {
            if (hit) atomicAdd(&g[(key >> kFewBits) & (kSelBins - 1)], 1u);
        } else {
            hist_add_wave(h, (key >> kFewBits) & (kSelBins - 1), hit);
        }
    });
    if (!small) flush_hist<NT>(h, g);
}

// Pass 2: the second digit; per piece, the keys above the 22-bit prefix, and
// the keys that share it.
template <int NT, int UPW, bool PULL>
__device__ __forceinline__ void direct_collect(const DirectArgs& a, uint32_t* h, uint32_t* lds) {
    Piece p;
    if (!piece_of(a, blockIdx.x, p)) return;
    const uint32_t c = p.c;
    __shared__ __align__(16) uint32_t sum[4];  // keys above, inside, smallest, largest
    Rows<UPW> x;
    load_rows<UPW, PULL>(a, c, x);
    const int tid = threadIdx.x;
    const uint32_t k = keep_of(p.sb - p.sa, a.keep_ppm);
    if (k == 0) return;
    const SegState g = a.seg[p.s];
    uint32_t lo = 0, bits = 0, r = k - g.clo;  // zero mode: the bin is key 0
    if (!g.zero) {
        uint32_t d1, above;
        block_pick_copies<NT, kSelBins>(a.h1 + (size_t)p.s * a.copies * kSelBins, a.copies, g.r1, lds, d1, above);
        lo = (g.d0 << kSel0Shift) | (d1 << kFewBits);
        bits = kFewBits;
        r = g.r1 - above;
    }
    if (tid < 4) sum[tid] = tid == 2 ? kNoKey : 0u;
    for (uint32_t i = tid; i < kBinKeys; i += NT) h[i] = 0;
    __syncthreads();
    uint32_t gt = 0, nz = 0, kmin = kNoKey, kmax = 0;
    for_keys<UPW>(a, c, p, x, [&](uint32_t key, uint32_t, bool in) {
        const uint32_t d = key - lo;
        gt += in && key >= lo && d >> bits != 0;
        const bool hit = in && key >= lo && d >> bits == 0;
        if (bits == 0) {
            nz += hit;
        } else if (hit) {
            a.ent[p.ea + atomicAdd(&sum[1], 1u)] = key;
            atomicAdd(&h[d], 1u);
            kmin = min(kmin, key);
            kmax = max(kmax, key);
        }
    });
    gt = wave_sum(gt);
    nz = wave_sum(nz);
    if (nz) kmin = kmax = lo;
    kmin = wave_min(kmin);
    kmax = lane_value(wave_incl_max(kmax), kWave - 1);
    if (lane_id() == 0) {
        if (gt) atomicAdd(&sum[0], gt);
        if (nz) atomicAdd(&sum[1], nz);
        if (kmin != kNoKey) {
            atomicMin(&sum[2], kmin);
            atomicMax(&sum[3], kmax);
        }
    }
    __syncthreads();
    // a piece with many different keys in the bin stores, in place of the keys,
    // how many are at or above each of its 512 values, if it has room for them
    // (every piece but a segment's first and last does: those are whole chunks)
    const bool dense = bits != 0 && sum[1] > kListKeys && sum[2] != sum[3] && p.eb - p.ea >= kBinKeys;
    if (dense && tid < kWave) {
        uint32_t carry = 0;
        for (uint32_t x = kBinKeys - 1 - tid; x < kBinKeys; x -= kWave) {  // (wraps past 0 at the end)
            const uint32_t incl = wave_incl_scan(h[x]) + carry;
            a.ent[p.ea + x] = incl;
            carry = lane_value(incl, kWave - 1);
        }
    }
    if (tid == 0) {
        a.info[blockIdx.x] = PieceInfo{sum[0], sum[1] | (dense ? kDenseFlag : 0u), sum[2], sum[3]};
        if (p.ea == p.sa) {
            SegState& o = a.seg[p.s];
            o.blo = lo;
            o.r2 = r;
        }
    }
    __syncthreads();
}

// Under one threshold over several tensors: where the tensors that start in unit u
// (elements [us, us + 1024)) begin in the sent list.  Their counts are formed by
// differences: a tensor's start is taken off its own count and added to that of
// the last non-empty tensor before it.  start: the output slot of the unit's first
// kept entry; km: this lane's kept elements, bit 4 i + q.  Called by the whole wave.
//
// Each lane takes a tensor.  Of the tensors that start at one element all but the
// last are empty and keep the count 0: the first and the last of such a run write
// its two marks, and a run past the wave's tensors is skipped by a search.  (One
// tensor after another took 7,110 us a call of 6.1M elements with 20,000 empty
// tensors in a row, the candidate form 162, and 1,411 with 20,000 of one element,
// the candidate form 949; now 67 and 108.)
__device__ __forceinline__ void mark_unit(const DirectArgs& a, uint32_t u, uint64_t start, uint32_t km) {
    const auto off = [&](uint32_t t) { return a.tensor_off[t]; };
    const auto slot = [&](uint64_t pos) { return (uint32_t)(pos < a.capacity ? pos : a.capacity); };
    const uint32_t us = u * kUnitLen, ue = a.N - us > kUnitLen ? us + kUnitLen : a.N;
    const uint32_t info = a.unit_info[u], t0 = info & 0x7FFFFFFFu;  // t0: the last tensor that starts at or before us
    const uint32_t lane = lane_id();
    if (off(t0) == us) {
        uint32_t head = t0;
        if (t0 > 0 && off(t0 - 1) == us) head = us > 0 ? wave_last_at_most(off, t0, us - 1) + 1 : 0u;
        if (lane == 0) {
            atomicSub(&a.tensor_counts[t0], slot(start));
            if (head > 0) atomicAdd(&a.tensor_counts[head - 1], slot(start));
        }
    }
    if (!(info >> 31)) return;
    // kept elements of each row before this lane's, two rows to a word
    const uint32_t n01 = __popc(km & 0xFu) | __popc(km >> 4 & 0xFu) << 16;
    const uint32_t n23 = __popc(km >> 8 & 0xFu) | __popc(km >> 12 & 0xFu) << 16;
    const uint32_t i01 = wave_incl_scan(n01), i23 = wave_incl_scan(n23);
    const uint32_t s01 = lane_value(i01, kWave - 1), s23 = lane_value(i23, kWave - 1);
    const uint32_t row1 = s01 & 0xFFFFu, row2 = row1 + (s01 >> 16), row3 = row2 + (s23 & 0xFFFFu);  // before each row
    for (uint32_t t = t0 + 1; t < a.T;) {
        const uint32_t x = t + lane;
        const uint32_t y = x < a.T ? off(x) : kNoKey;
        const bool in = y < ue;
        // kept elements of the unit before the tensor: in the rows before its row i,
        // in the lanes before the lane l that holds its first element, in that lane
        const uint32_t o = in ? y - us : 0u, i = o >> 8, l = (o & 255u) >> 2;
        const uint32_t b01 = (uint32_t)__shfl((int)(i01 - n01), (int)l), b23 = (uint32_t)__shfl((int)(i23 - n23), (int)l);
        const uint32_t m = (uint32_t)__shfl((int)km, (int)l) >> (4 * i) & ((1u << (o & 3u)) - 1u);
        const uint32_t n = (i == 0 ? 0u : i == 1 ? row1 : i == 2 ? row2 : row3) +
                           (((i & 2u ? b23 : b01) >> (16 * (i & 1u))) & 0xFFFFu) + __popc(m);
        if (in) {  // (off(T) = N is past every start)
            if (off(x + 1) != y) atomicSub(&a.tensor_counts[x], slot(start + n));
            if (off(x - 1) != y) atomicAdd(&a.tensor_counts[x - 1], slot(start + n));
        }
        if (ballot(!in) != 0) break;
        const uint32_t last = lane_value(y, kWave - 1);
        t += kWave;
        if (t < a.T && off(t) == last) t = wave_last_at_most(off, a.T, last);
    }
}

// Pass 3: the kept (index, value) pairs in ascending index order, and their
// residual set to +0 (or added to the pulled copy).
template <int NT, int UPW, bool PULL>
__device__ __forceinline__ void direct_emit(const DirectArgs& a, uint32_t* h, uint32_t* lds) {
    Piece p;
    if (!piece_of(a, blockIdx.x, p)) return;
    const uint32_t c = p.c;
    __shared__ __align__(16) uint32_t wc[2 * (NT / kWave)];
    Rows<UPW> x;
    load_rows<UPW, PULL>(a, c, x);
    const int w = (int)wave_index(), lane = lane_id();
    const uint32_t k = keep_of(p.sb - p.sa, a.keep_ppm);
    if (k == 0) return;
    const SegState g = a.seg[p.s];
    const Resolved z = resolve<NT>(a, p.s, p.sa, p.sb, blockIdx.x, g.blo, g.r2, h, lds);
    if (p.ea == p.sa && threadIdx.x == 0) {
        a.seg[p.s].thr = z.thr;
        a.seg[p.s].need = z.need;
    }
    // keys above and equal to the threshold before this wave's first element
    uint32_t gt = 0, eq = 0;
    for_keys<UPW>(a, c, p, x, [&](uint32_t key, uint32_t, bool in) {
        gt += in && key > z.thr;
        eq += in && key == z.thr;
    });
    gt = wave_sum(gt);
    eq = wave_sum(eq);
    if (lane == 0) {
        wc[2 * w] = gt;
        wc[2 * w + 1] = eq;
    }
    __syncthreads();
    uint32_t bg = z.above, be = z.equal;
    for (int i = 0; i < w; ++i) {
        bg += wc[2 * i];
        be += wc[2 * i + 1];
    }
    const uint64_t ob = a.out_base[p.s];
    const bool marks = a.S != a.T;  // several tensors in the segment: where each one's entries start
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        const uint32_t u = wave_unit<UPW>(a, c, j), us = u * kUnitLen;
        if (u >= a.C || us >= p.eb || (p.ea > us && p.ea - us >= kUnitLen)) continue;
        const uint64_t start = ob + bg + (be < z.need ? be : z.need);
        uint32_t km = 0;  // this lane's kept elements, bit 4 i + q
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f4 v = x.v[4 * j + i];
            const uint32_t e = row_elem(u, i);
            bool isgt[4], iseq[4];
            uint64_t mg[4], me[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = e + q - p.ea < p.eb - p.ea;
                isgt[q] = in && key_of(v[q]) > z.thr;
                iseq[q] = in && key_of(v[q]) == z.thr;
                mg[q] = ballot(isgt[q]);
                me[q] = ballot(iseq[q]);
            }
            if ((mg[0] | mg[1] | mg[2] | mg[3] | me[0] | me[1] | me[2] | me[3]) == 0) continue;
            uint32_t G = bg + lanes_below(mg[0]) + lanes_below(mg[1]) + lanes_below(mg[2]) + lanes_below(mg[3]);
            uint32_t E = be + lanes_below(me[0]) + lanes_below(me[1]) + lanes_below(me[2]) + lanes_below(me[3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (isgt[q] || (iseq[q] && E < z.need)) {
                    const uint64_t pos = ob + G + (E < z.need ? E : z.need);
                    if (pos < a.capacity) {  // (always: the capacity holds k)
                        a.idx[pos] = e + q;
                        a.val[pos] = v[q];
                    }
                    if (PULL) a.pull_copy[e + q] = a.pull_copy[e + q] + v[q];
                    else a.res[e + q] = 0.0f;
                    km |= 1u << (4 * i + q);
                }
                G += isgt[q];
                E += iseq[q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bg += popc64(mg[q]);
                be += popc64(me[q]);
            }
        }
        if (marks) mark_unit(a, u, start, km);
    }
    if (marks && c + 1 == a.G && w == 0) {  // the last non-empty tensor ends with the list
        const uint32_t t = wave_last_at_most([&](uint32_t x) { return a.tensor_off[x]; }, a.T, a.N - 1);
        if (lane == 0) atomicAdd(&a.tensor_counts[t], (uint32_t)(k < a.capacity ? k : a.capacity));
    }
    __syncthreads();
}

// MODE as in the dense pass: 0: gradient + residual; 1: (gradient - base) +
// residual; 2: gradient - base, nothing written.
template <int MODE, int UPW>
__global__ __launch_bounds__(kDirectThreads) void k_dacc(DirectArgs a) {
    constexpr int NT = kDirectThreads;
    __shared__ __align__(16) uint32_t h[kSelBins];
    __shared__ __align__(16) uint32_t lds[kPickLds<NT>];
    const int tid = threadIdx.x;
    {  // the second digit's histograms, which the next pass adds to
        const size_t words = (size_t)a.S * a.copies * (kSelBins / 4);
        uint4* z = reinterpret_cast<uint4*>(a.h1);
        for (size_t i = (size_t)blockIdx.x * NT + tid; i < words; i += (size_t)gridDim.x * NT) z[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (blockIdx.x == 0) call_prologue<NT>(a.seg_off, a.S, a.T, a.keep_ppm, a.out_base, a.tensor_counts, a.seg, lds);
    Piece p;
    if (!piece_of(a, blockIdx.x, p)) return;
    const uint32_t c = p.c;
    const bool small = p.eb - p.ea <= kSmallPiece;
    uint32_t* gh = a.h0 + ((size_t)p.s * a.copies + blockIdx.x % a.copies) * kSelBins;
    if (!small) clear_hist<NT>(h);
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        const uint32_t u = wave_unit<UPW>(a, c, j), us = u * kUnitLen;
        if (u >= a.C || us >= p.eb || (p.ea > us && p.ea - us >= kUnitLen)) continue;
        f4 g[4], b[4], r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t e = row_elem(u, i);
            g[i] = b[i] = r[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (e < a.N) {
                g[i] = load4(a.grad, e, a.N);
                if (MODE >= 1) b[i] = load4(a.base, e, a.N);
                if (MODE != 2) r[i] = load4(a.res, e, a.N);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t e = row_elem(u, i);
            f4 v;
            bool in[4], same = true;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                in[q] = e + q - p.ea < p.eb - p.ea;
                // binary32 roundings, one per operation
                const float d = MODE >= 1 ? g[i][q] - b[i][q] : g[i][q];
                v[q] = MODE == 2 ? d : d + r[i][q];
                same = same && __float_as_uint(v[q]) == __float_as_uint(r[i][q]);
                const uint32_t key = key_of(v[q]);
                if (in[q] && key != 0) {
                    if (small) atomicAdd(&gh[key >> kSel0Shift], 1u);
                    else atomicAdd(&h[key >> kSel0Shift], 1u);
                }
            }
            if (MODE != 2 && !same) {
                if (in[0] && in[3]) {
                    *reinterpret_cast<f4*>(a.res + e) = v;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (in[q]) a.res[e + q] = v[q];
                }
            }
        }
    }
    if (!small) flush_hist<NT>(h, gh);
}

template <int UPW, bool PULL>
__global__ __launch_bounds__(kDirectThreads) void k_dhist(DirectArgs a) {
    __shared__ __align__(16) uint32_t h[kSelBins];
    __shared__ __align__(16) uint32_t lds[kPickLds<kDirectThreads>];
    direct_hist1<kDirectThreads, UPW, PULL>(a, h, lds);
}

template <int UPW, bool PULL>
__global__ __launch_bounds__(kDirectThreads) void k_dcollect(DirectArgs a) {
    __shared__ __align__(16) uint32_t h[kBinKeys];
    __shared__ __align__(16) uint32_t lds[kPickLds<kDirectThreads>];
    {  // the first digit's histograms, for the next call
        const size_t words = (size_t)a.S * a.copies * (kSelBins / 4);
        uint4* z = reinterpret_cast<uint4*>(a.h0);
        for (size_t i = (size_t)blockIdx.x * kDirectThreads + threadIdx.x; i < words; i += (size_t)gridDim.x * kDirectThreads)
            z[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    direct_collect<kDirectThreads, UPW, PULL>(a, h, lds);
}

template <int UPW, bool PULL>
__global__ __launch_bounds__(kDirectThreads) void k_demit(DirectArgs a) {
    __shared__ __align__(16) uint32_t h[kSelBins];
    __shared__ __align__(16) uint32_t lds[kResolveLds<kDirectThreads>];
    clear_col_sums(a.cols);
    direct_emit<kDirectThreads, UPW, PULL>(a, h, lds);
}

template <int UPW>
static hipError_t launch_direct_upw(const DirectArgs& a, int mode, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
    const dim3 g(a.G ? a.G + a.S - 1 : 1u), b(kDirectThreads);  // a block per piece, and per index without one
    auto first = mode == 0 ? k_dacc<0, UPW> : mode == 1 ? k_dacc<1, UPW> : k_dacc<2, UPW>;
    if (t0 != nullptr && t1 != nullptr) hipExtLaunchKernelGGL(first, g, b, 0, st, t0, t1, 0, a);
    else hipLaunchKernelGGL(first, g, b, 0, st, a);
    if (a.G == 0) return hipGetLastError();
    if (mode == 2) {
        hipLaunchKernelGGL((k_dhist<UPW, true>), g, b, 0, st, a);
        hipLaunchKernelGGL((k_dcollect<UPW, true>), g, b, 0, st, a);
        hipLaunchKernelGGL((k_demit<UPW, true>), g, b, 0, st, a);
    } else {
        hipLaunchKernelGGL((k_dhist<UPW, false>), g, b, 0, st, a);
        hipLaunchKernelGGL((k_dcollect<UPW, false>), g, b, 0, st, a);
        hipLaunchKernelGGL((k_demit<UPW, false>), g, b, 0, st, a);
    }
    return hipGetLastError();
}

// Units per wave: one while the chunks are few enough that reading their
// records costs less than the longer chain of two units (4.2M elements: 42 us a
// call with one, 46 with two; 6.1M: 55 and 51).
uint32_t direct_units_per_wave(uint32_t units) { return units <= 4608 ? 1u : 2u; }

// t0, t1: as launch_dense, for the first pass.
hipError_t launch_direct(DirectArgs a, int mode, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
    const uint32_t upw = direct_units_per_wave(a.C), cu = upw * (kDirectThreads / kWave);
    a.cshift = 10;  // log2 of kUnitLen
    while ((kUnitLen << (a.cshift - 10)) < cu * kUnitLen) ++a.cshift;
    a.G = (a.C + cu - 1) / cu;
    return upw == 1 ? launch_direct_upw<1>(a, mode, st, t0, t1) : launch_direct_upw<2>(a, mode, st, t0, t1);
}

}  // namespace gd
