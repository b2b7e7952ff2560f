// Device-side construction of the compressed residual copies and the utility
// kernels of the CCD++ library (gfx950).
//
// Construction (once per handle): the observed set Omega of Section 3 is given
// as triplets.  For each copy, every entry gets a key (segment id, column inside
// its tile) -- the segment order is decided on the host from per-(tile, row)
// counts -- and a radix sort brings the entries into layout order, carrying the
// triplet index along so values and the map between the two copies follow.
// Adjacent equal keys after the user-major sort are repeated positions.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>
#include <rocprim/iterator/counting_iterator.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include <algorithm>
#include <type_traits>

#include "ccdpp_internal.hpp"

namespace ccdk {
namespace {

constexpr int kT = 256;
// Histograms with at most this many bins count in LDS (128 KB per workgroup).
constexpr int32_t kHistLdsBins = 32768;

inline dim3 grid_for(int64_t n, int64_t cap = 1 << 20) {
    int64_t g = (n + kT - 1) / kT;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return dim3((unsigned)g);
}

// The elements a thread visits in the copies between the two orders of the entries: each
// eighth of the range is one XCD's (workgroups go to the XCDs round-robin), walked
// front to back by its workgroups together.  The stores in flight on an XCD then fall
// into few lines of the other order (about one per row of its tile), which its own
// L2 merges.  (Between the copies of 10M ratings: 88 -> 59 us; of 100M: 1230 -> 1190 us.
// The build's maps, which mostly gather, gained nothing from it.)
struct Span {
    int64_t lo, hi, step;
};
__device__ __forceinline__ Span xcd_span(int64_t n) {
    const int64_t per = ((n + 7) / 8 + kT - 1) / kT * kT;
    const int64_t first = (int64_t)(blockIdx.x & 7u) * per;
    return Span{first + (int64_t)(blockIdx.x >> 3) * kT + threadIdx.x, min(n, first + per),
                (int64_t)(gridDim.x >> 3) * kT};
}
inline dim3 xcd_grid(int64_t n) {
    const int64_t per = ((n + 7) / 8 + kT - 1) / kT;
    return dim3((unsigned)(8 * std::max<int64_t>(1, std::min<int64_t>(per, 1 << 17))));
}

// Adds one to count[key] for every valid lane of the wave.  A lane whose key equals
// the previous lane's (a run, as in triplets grouped by row) adds through the run's
// first lane, so a run costs one atomic.  The valid lanes are a prefix of the wave,
// and every lane of the wave calls this.
__device__ inline void count_runs(int32_t key, bool valid, int32_t* count) {
    const int lane = (int)(threadIdx.x & 63);
    const int32_t prev = __shfl_up(key, 1);
    const bool head = valid && (lane == 0 || prev != key);
    const uint64_t heads = __ballot(head);
    const int nvalid = __popcll(__ballot(valid));
    if (head) {
        const uint64_t later = lane == 63 ? 0 : heads >> (lane + 1);
        const int next = later ? lane + __ffsll((unsigned long long)later) : nvalid;
        atomicAdd(&count[key], next - lane);
    }
}

// Range [lo, hi) of entries of workgroup blockIdx.x: contiguous, so that runs stay in
// one wave.
__device__ inline void block_range(int64_t n, int64_t* lo, int64_t* hi) {
    const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 63) / 64 * 64;
    *lo = min(n, (int64_t)blockIdx.x * per);
    *hi = min(n, *lo + per);
}

// count[key[e]] += 1 for every e < n.  bins <= kHistLdsBins: the workgroup counts in
// LDS and adds its non-zero counts at the end; else straight into global memory.
template <bool kLds>
__global__ void __launch_bounds__(1024) k_histogram(const int32_t* __restrict__ key, int64_t n,
                                                    int32_t bins, int32_t* count) {
    extern __shared__ int32_t lds_count[];
    int32_t* c = count;
    if constexpr (kLds) {
        for (int32_t b = threadIdx.x; b < bins; b += blockDim.x) lds_count[b] = 0;
        __syncthreads();
        c = lds_count;
    }
    int64_t lo, hi;
    block_range(n, &lo, &hi);
    for (int64_t base = lo + (threadIdx.x & ~63); base < hi; base += blockDim.x) {
        const int64_t e = base + (threadIdx.x & 63);
        const bool valid = e < hi;
        count_runs(valid ? key[e] : 0, valid, c);
    }
    if constexpr (kLds) {
        __syncthreads();
        for (int32_t b = threadIdx.x; b < bins; b += blockDim.x)
            if (lds_count[b]) atomicAdd(&count[b], lds_count[b]);
    }
}

__global__ void k_add(int32_t* __restrict__ a, int64_t n, int32_t delta) {
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT)
        a[e] += delta;
}

// Entries whose key lies in [lo, hi).
struct KeyInRange {
    const int32_t* key;
    int32_t lo, hi;
    __device__ bool operator()(int32_t e) const { return key[e] >= lo && key[e] < hi; }
};

__global__ void k_map(const int32_t* __restrict__ in, const int32_t* __restrict__ table,
                      int64_t n, int32_t* __restrict__ out) {
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT)
        out[e] = table[in[e]];
}

// Entries per (tile, row) segment: count[(col / T) * rows + row].
__global__ void __launch_bounds__(kT) k_seg_histogram(const int32_t* __restrict__ lrow,
                                                      const int32_t* __restrict__ lcol, int64_t nnz,
                                                      int32_t rows, int32_t T, int32_t* count) {
    int64_t lo, hi;
    block_range(nnz, &lo, &hi);
    for (int64_t base = lo + (threadIdx.x & ~63); base < hi; base += blockDim.x) {
        const int64_t e = base + (threadIdx.x & 63);
        const bool valid = e < hi;
        const int32_t key = valid ? (lcol[e] / T) * rows + lrow[e] : 0;
        count_runs(key, valid, count);
    }
}

// The same with the entries taken in an order that keeps most tiles together (the
// user-major copy's, for the item-major one): a workgroup counts a run of one tile in LDS,
// one word per row, and adds its counts at the run's end; an entry of another tile
// inside what the search took for a run is counted in global memory, so the counts
// are right in any order.  (10M ratings, 6 tiles of 10,681 rows: 0.08 ms; 100M, 36 of
// 17,770: 0.82 ms; one global atomic per entry took 1.7 and 6.0 ms.)
__global__ void __launch_bounds__(1024) k_seg_histogram_runs(
    const int32_t* __restrict__ order, const int32_t* __restrict__ lrow,
    const int32_t* __restrict__ lcol, int64_t nnz, int32_t rows, int32_t T, int32_t* count) {
    extern __shared__ int32_t lds_count[];
    int64_t lo, hi;
    block_range(nnz, &lo, &hi);
    while (lo < hi) {
        const int32_t p = lcol[order[lo]] / T;
        int64_t a = lo + 1, b = hi;  // the run's end: the first entry of another tile
        while (a < b) {
            const int64_t mid = (a + b) >> 1;
            if (lcol[order[mid]] / T == p) a = mid + 1; else b = mid;
        }
        for (int32_t r = threadIdx.x; r < rows; r += blockDim.x) lds_count[r] = 0;
        __syncthreads();
        for (int64_t e = lo + threadIdx.x; e < a; e += blockDim.x) {
            const int32_t t = order[e];
            const int32_t q = lcol[t] / T, r = lrow[t];
            if (q == p)
                atomicAdd(&lds_count[r], 1);
            else
                atomicAdd(&count[(int64_t)q * rows + r], 1);
        }
        __syncthreads();
        for (int32_t r = threadIdx.x; r < rows; r += blockDim.x)
            if (lds_count[r]) atomicAdd(&count[(int64_t)p * rows + r], lds_count[r]);
        __syncthreads();
        lo = a;
    }
}

// Sort key of an entry: its segment id, then its column inside the tile.
__global__ void k_seg_keys(const int32_t* __restrict__ lrow, const int32_t* __restrict__ lcol,
                           const int32_t* __restrict__ segid, int64_t nnz, int32_t rows, int32_t T,
                           int cbits, uint64_t* __restrict__ keys, int32_t* __restrict__ ids) {
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * kT) {
        const int64_t c = lcol[e];
        const int64_t p = c / T;
        const uint64_t s = (uint64_t)segid[p * rows + lrow[e]];
        keys[e] = (s << cbits) | (uint64_t)(c - p * T);
        ids[e] = (int32_t)e;
    }
}

__global__ void k_dup_check(const uint64_t* __restrict__ keys, int64_t nnz, int32_t* flag) {
    for (int64_t p = (int64_t)blockIdx.x * kT + threadIdx.x; p + 1 < nnz;
         p += (int64_t)gridDim.x * kT)
        if (keys[p] == keys[p + 1]) *flag = 1;
}

// Entry q of the sorted order goes to padded position p = q + seg_off[segment]:
// its index to idx[p], its value to val[val_slot(p)]; pos[q] is the value slot.
template <class I, class V>
__global__ void k_layout_fill(const uint64_t* __restrict__ keys, const int32_t* __restrict__ perm,
                              const float* __restrict__ val_in, int64_t nnz, int cbits,
                              uint64_t mask, const int32_t* __restrict__ seg_off, uint32_t swz_lim,
                              I* __restrict__ idx, V* __restrict__ val,
                              int32_t* __restrict__ pos) {
    for (int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x; q < nnz; q += (int64_t)gridDim.x * kT) {
        const uint64_t key = keys[q];
        const int64_t p = q + seg_off[key >> cbits];
        const uint32_t c = (uint32_t)(key & mask);
        const bool first = q == 0 || (keys[q - 1] >> cbits) != (key >> cbits);
        idx[p] = (I)((c < swz_lim ? lds_swizzle(c) : c) | (first ? IndexBits<I>::start : 0u));
        const int64_t f = val_slot<V>(p);
        val[f] = (V)val_in[perm[q]];
        pos[q] = (int32_t)f;
    }
}

template <class I>
__global__ void k_fill_idx(I* __restrict__ idx, I value, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT)
        idx[i] = value;
}

__global__ void k_invert(const int32_t* __restrict__ perm, int64_t n, int32_t* __restrict__ inv) {
    for (int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x; q < n; q += (int64_t)gridDim.x * kT)
        inv[perm[q]] = (int32_t)q;
}

__global__ void k_compose(const int32_t* __restrict__ a, const int32_t* __restrict__ b, int64_t n,
                          int32_t* __restrict__ out) {
    for (int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x; q < n; q += (int64_t)gridDim.x * kT)
        out[q] = a[b[q]];
}

// out[from[e]] = to[e]: a map between value slots of the two copies.
__global__ void k_slot_map(const int32_t* __restrict__ from, const int32_t* __restrict__ to,
                           int64_t n, int32_t* __restrict__ out) {
    for (int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x; q < n; q += (int64_t)gridDim.x * kT)
        out[from[q]] = to[q];
}

// dst[map[f]] = src[f] over the source copy's value slots in order (slots of
// padding entries map to -1): sequential reads, one scattered write per entry.
template <class V>
__global__ void k_copy_slots(const V* __restrict__ src, const int32_t* __restrict__ map,
                             V* __restrict__ dst, int64_t n) {
    const Span sp = xcd_span(n);
    for (int64_t f = sp.lo; f < sp.hi; f += sp.step) {
        const int32_t g = map[f];
        if (g >= 0) dst[g] = src[f];
    }
}

template <class V>
__global__ void k_fill(V* __restrict__ dst, V value, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT)
        dst[i] = value;
}

// Tiles of kFR rows by up to kFT columns of a factor matrix, turned in LDS between the
// column-major order over relabelled ids (rows contiguous) and a row-major one (columns
// contiguous), so that both sides are read and written in whole lines: bound by
// the two streams.  `lanes` (a power of two, at least the tile's columns) threads
// take a row's values together, so that no thread divides.  A workgroup takes the tiles of
// its rows in steps of gridDim.y: all of them, a row's lines being shared by its tiles, or,
// where rows alone make too few workgroups (turn_grid), a share.
constexpr int kFR = 64, kFT = 32, kFE = kFR * kFT / kT;  // kFE values per thread, requested together

// Turns of few values go value by value, in the order of what they write (32-bit
// positions): one value's latency, where a tile adds LDS and a barrier (kTurnSmall).
template <class S, class V>
__global__ void k_factor_in_small(const S* __restrict__ rowmajor, const int32_t* __restrict__ new2old,
                                  uint32_t rows, uint32_t k, V* __restrict__ colmajor) {
    const uint32_t e = blockIdx.x * kT + threadIdx.x;
    if (e >= rows * k) return;
    const uint32_t t = e / rows;
    colmajor[e] = (V)rowmajor[(uint32_t)new2old[e - t * rows] * k + t];
}
template <class V, class S>
__global__ void k_factor_out_small(const V* __restrict__ colmajor, const int32_t* __restrict__ old2new,
                                   uint32_t rows, uint32_t k, uint32_t pitch, S* __restrict__ rowmajor) {
    const uint32_t e = blockIdx.x * kT + threadIdx.x;
    if (e >= rows * pitch) return;
    const uint32_t i = e / pitch, t = e - i * pitch;
    rowmajor[e] = t < k ? (S)colmajor[t * rows + (old2new ? (uint32_t)old2new[i] : i)] : S(0);
}

// colmajor[t * rows + i'] = rowmajor[new2old[i'] * k + t]
template <class S, class V>
__global__ __launch_bounds__(kT) void k_factor_in(const S* __restrict__ rowmajor,
                                                  const int32_t* __restrict__ new2old, int64_t rows,
                                                  int64_t k, int shift, V* __restrict__ colmajor) {
    __shared__ V tile[kFT][kFR + 1];
    const int64_t r0 = (int64_t)blockIdx.x * kFR;
    const int nr = (int)min((int64_t)kFR, rows - r0);
    const int lanes = 1 << shift, last = nr * lanes - 1;
    for (int64_t t0 = (int64_t)blockIdx.y * kFT; t0 < k; t0 += (int64_t)gridDim.y * kFT) {
        const int nt = (int)min((int64_t)kFT, k - t0);
        V v[kFE];
#pragma unroll
        for (int j = 0; j < kFE; ++j) {
            if (j * kT > last) break;
            const int e = min(j * kT + (int)threadIdx.x, last);
            v[j] = (V)rowmajor[(int64_t)new2old[r0 + (e >> shift)] * k + t0 + min(e & (lanes - 1), nt - 1)];
        }
#pragma unroll
        for (int j = 0; j < kFE; ++j) {
            if (j * kT > last) break;
            const int e = j * kT + threadIdx.x, t = e & (lanes - 1);
            if (e <= last && t < nt) tile[t][e >> shift] = v[j];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < nt * kFR; e += kT) {
            const int t = e / kFR, r = e % kFR;
            if (r < nr) colmajor[(t0 + t) * rows + r0 + r] = tile[t][r];
        }
        __syncthreads();
    }
}

// rowmajor[new2old[i'] * pitch + t] = colmajor[t * rows + i'], zero for k <= t < pitch
// (new2old null: row i')
template <class V, class S>
__global__ __launch_bounds__(kT) void k_factor_out(const V* __restrict__ colmajor,
                                                   const int32_t* __restrict__ new2old, int64_t rows,
                                                   int64_t k, int64_t pitch, int shift,
                                                   S* __restrict__ rowmajor) {
    __shared__ V tile[kFT][kFR + 1];
    const int64_t r0 = (int64_t)blockIdx.x * kFR;
    const int nr = (int)min((int64_t)kFR, rows - r0);
    const int lanes = 1 << shift, last = nr * lanes - 1;
    for (int64_t t0 = (int64_t)blockIdx.y * kFT; t0 < pitch; t0 += (int64_t)gridDim.y * kFT) {
        const int nt = (int)min((int64_t)kFT, pitch - t0);
        V v[kFE];
#pragma unroll
        for (int j = 0; j < kFE; ++j) {
            if (j * kT >= nt * kFR) break;
            const int e = j * kT + threadIdx.x, t = min(e / kFR, nt - 1), r = min(e % kFR, nr - 1);
            v[j] = t0 + t < k ? colmajor[(t0 + t) * rows + r0 + r] : V(0);
        }
#pragma unroll
        for (int j = 0; j < kFE; ++j) {
            if (j * kT >= nt * kFR) break;
            const int e = j * kT + threadIdx.x;
            if (e < nt * kFR) tile[e / kFR][e % kFR] = v[j];
        }
        __syncthreads();
#pragma unroll 1
        for (int e = threadIdx.x; e <= last; e += kT) {
            const int r = e >> shift, t = e & (lanes - 1);
            const int64_t i = new2old ? new2old[r0 + r] : r0 + r;
            if (t < nt) rowmajor[i * pitch + t0 + t] = (S)tile[t][r];
        }
        __syncthreads();
    }
}

// Workgroups of a turn of `cols` columns, and the shift of `lanes`.  Rows alone fill the
// chip from kTurnGroups workgroups on.  (64 x 65,536, one workgroup before: out 17.7 ms a call,
// now 1.1; 20,000 x 64, 313 before: in 13.3 us, now 6.6.)
constexpr int64_t kTurnGroups = 1024;
// Up to this many values a turn goes value by value (us, values against tiles: 2,000 x 20
// in 2.7 against 5.0, out 2.8 against 5.2; 6,041 x 40 in 4.6 against 7.8, out 3.9 against 8.0;
// 20,000 x 20 equal); rows of up to four values, whole in one sector, into columns always do
// (480,189 x 4: 9.2 against 10.4).
constexpr int64_t kTurnSmall = 1 << 18, kTurnNarrow = 1 << 28;
inline dim3 turn_grid(int64_t rows, int64_t cols, int* shift) {
    const int64_t gx = (rows + kFR - 1) / kFR, tiles = (cols + kFT - 1) / kFT;
    const int64_t gy = std::min(std::min<int64_t>(tiles, 65535), (kTurnGroups + gx - 1) / gx);
    for (*shift = 0; (1 << *shift) < std::min<int64_t>(cols, kFT);) ++*shift;
    return dim3((unsigned)gx, (unsigned)std::max<int64_t>(1, gy));
}

// Four values of a row of a row-major factor copy whose pitch is a multiple of 4.
template <class V> struct Row4 {
    V v[4];
};
template <class V>
__device__ __forceinline__ Row4<V> load4(const V* p) {
    struct alignas(16) Q {
        V v[4];
    };
    const Q q = *reinterpret_cast<const Q*>(p);
    return Row4<V>{{q.v[0], q.v[1], q.v[2], q.v[3]}};
}

// Rewrites, one wave per window, every window whose lanes' valid entries each climb
// by at most kDeltaMax unswizzled columns into the delta-coded format, and sets its
// bit.  Valid entries come first in a lane (padding only ends a segment); a lane
// of padding alone is coded as its first index with one valid entry.  Every lane
// reads its 16 bytes before the vote, so the window is rewritten in place.
__global__ __launch_bounds__(kT) void k_delta_windows(uint16_t* __restrict__ idx, int64_t nwin,
                                                       uint32_t pad, uint64_t* __restrict__ dmask) {
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t w = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    if (w >= nwin) return;  // whole waves leave together
    uint16_t* blk = idx + w * kWin;
    const uint4 v = *reinterpret_cast<const uint4*>(blk + lane * kE);
    const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
    uint32_t c[8];
    for (int k = 0; k < 8; ++k) c[k] = (wd[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
    int cnt = 0;
    while (cnt < 8 && c[cnt] != pad) ++cnt;
    bool ok = true;
    for (int k = cnt; k < 8; ++k) ok = ok && c[k] == pad;  // padding only after the valid entries
    uint32_t st[7] = {0, 0, 0, 0, 0, 0, 0};
    if (cnt > 0) {
        uint32_t prev = lds_swizzle(c[0] & 0x7FFFu);
        for (int k = 1; k < cnt; ++k) {
            const uint32_t cur = lds_swizzle(c[k]);
            ok = ok && cur >= prev && cur - prev <= kDeltaMax;
            st[k - 1] = (cur - prev) & kDeltaMax;
            prev = cur;
        }
    }
    if (!__all(ok)) return;
    const uint32_t last = (uint32_t)(cnt > 0 ? cnt - 1 : 0);
    uint32_t* words = reinterpret_cast<uint32_t*>(blk);
    words[3 * lane] = c[0] | (st[0] << 16) | (st[1] << 27);
    words[3 * lane + 1] = (st[1] >> 5) | (st[2] << 6) | (st[3] << 17) | (st[4] << 28);
    words[3 * lane + 2] = (st[4] >> 4) | (st[5] << 7) | (st[6] << 18) | (last << 29);
    if (lane == 0) atomicOr(reinterpret_cast<unsigned long long*>(dmask + (w >> 6)),
                            1ull << (w & 63));
}

// One step of a sum over lanes that also deals the values out: of the 2 * N values, the
// lanes whose bit is set keep the upper half and the others the lower one, each
// adding its partner's (the lane CTRL reads, whose bit differs) values of that half.
template <int CTRL>
__device__ __forceinline__ double dpp_from(double x) {
    int2 v = __builtin_bit_cast(int2, x);
    v.x = __builtin_amdgcn_update_dpp(0, v.x, CTRL, 0xF, 0xF, false);
    v.y = __builtin_amdgcn_update_dpp(0, v.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, v);
}
template <int CTRL, int N>
__device__ __forceinline__ void deal(double* v, bool upper) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double keep = upper ? v[N + i] : v[i], give = upper ? v[i] : v[N + i];
        v[i] = keep + dpp_from<CTRL>(give);
    }
}

constexpr int64_t kRebuildWaves = 1536;  // six per compute unit

// Index of entry q as the plain format holds it, from a delta-coded window when
// its bit is set.
template <class I>
__device__ __forceinline__ uint32_t index_at(const I* idx, const uint64_t* dmask, uint32_t pad,
                                             int64_t q) {
    const int64_t w = q / kWin;
    if (dmask && ((dmask[w >> 6] >> (w & 63)) & 1u)) {
        const uint32_t* rec = reinterpret_cast<const uint32_t*>(idx + w * kWin) + 3 * ((q % kWin) / kE);
        uint32_t c[8];
        delta_decode(rec[0], rec[1], rec[2], pad, c);
        return c[q % kE];
    }
    return (uint32_t)idx[q];
}

// k_rebuild below for few entries and features, or without memory for a row-major H: an
// entry per thread, both factors read from their columns.  Entry e's value slot is pos[e].
template <class I, class V>
__global__ void k_rebuild_each(const int64_t* __restrict__ seg_start, int64_t nseg,
                               const int32_t* __restrict__ seg_row, const int32_t* __restrict__ tile_seg,
                               int32_t P, int32_t T, uint32_t swz_lim, const I* __restrict__ idx,
                               const uint64_t* __restrict__ dmask, uint32_t pad,
                               const int32_t* __restrict__ pos, const V* __restrict__ A,
                               const V* __restrict__ W, const V* __restrict__ H, int64_t m,
                               int64_t n, int32_t k, int64_t nnz, V* __restrict__ val) {
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * kT) {
        const int64_t f = pos[e];            // value slot
        const int64_t q = val_entry<V>(f);   // entry position
        int64_t lo = 0, hi = nseg;  // last s with seg_start[s] <= q
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (seg_start[mid] <= q) lo = mid; else hi = mid;
        }
        int32_t plo = 0, phi = P;  // last tile p with tile_seg[p] <= s
        while (phi - plo > 1) {
            const int32_t mid = (plo + phi) >> 1;
            if (tile_seg[mid] <= lo) plo = mid; else phi = mid;
        }
        const int64_t i = seg_row[lo];
        const uint32_t c = index_at<I>(idx, dmask, pad, q) & IndexBits<I>::mask;
        const int64_t j = (int64_t)plo * T + (int64_t)(c < swz_lim ? lds_swizzle(c) : c);
        double pred = 0.0;
        for (int32_t t = 0; t < k; ++t)
            pred = __builtin_fma((double)W[(int64_t)t * m + i], (double)H[(int64_t)t * n + j], pred);
        val[f] = (V)((double)A[f] - pred);
    }
}

// R = A - w_i^T h_j for every entry of the user-major layout (prediction summed in fp64,
// one rounding to the value type).  A wave takes a window: lane l finds the segment of
// its kE entries (they belong to one) and from it the row and the tile, and puts
// their columns in LDS.  Then groups of G lanes take the window's lanes' entries in
// turn, each lane four features of every row h_j at a time, so that a row of HT (H
// row-major, rows of `pitch` values, a multiple of 4, zero past k) is read in whole
// lines, and the lanes' sums are added over the group.  `parts` (a power of two, at most
// G) waves share a window's turns where windows alone are too few (2,000 x 1,000, 50,000
// ratings, k = 40: 30.9 -> 8.2 us).  A holds the ratings in the slots of val.
// Bound by L2: one lane per entry fetched a 128-byte line per 16 bytes of a row, at
// 31 TB/s.  (m = 480,189, n = 17,770, 100.5M ratings, k = 40: 8.3 ms with one
// 4-byte gather per entry and feature, 4.1 with 16-byte ones, 2.9 now.)
template <class I, class V, int G>
__global__ __launch_bounds__(kT) void k_rebuild(
    const int64_t* __restrict__ seg_start, int64_t nseg, const int32_t* __restrict__ seg_row,
    const int32_t* __restrict__ tile_seg, int32_t P, int32_t T, uint32_t swz_lim,
    const I* __restrict__ idx, const uint64_t* __restrict__ dmask, uint32_t pad,
    const V* __restrict__ A, const V* __restrict__ W, const V* __restrict__ HT, int64_t m,
    uint32_t k, uint32_t pitch, int64_t npad, int parts, V* __restrict__ val) {
    constexpr uint32_t kNone = 0xFFFFFFFFu;  // a padding entry
    __shared__ uint4 cols[kT / 64][64][2];
    const int wave = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63u);
    const int grp = lane / G, g = lane % G;
    for (int64_t wp = (int64_t)blockIdx.x * (kT / 64) + wave; wp < npad / kWin * parts;
         wp += (int64_t)gridDim.x * (kT / 64)) {
        const int64_t w = wp / parts;
        const int turns = G / parts, it0 = (int)(wp % parts) * turns;
        const int64_t q0 = w * kWin + lane * kE;
        int64_t lo = 0, hi = nseg;  // last s with seg_start[s] <= q0
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (seg_start[mid] <= q0) lo = mid; else hi = mid;
        }
        int32_t plo = 0, phi = P;  // last tile p with tile_seg[p] <= s
        while (phi - plo > 1) {
            const int32_t mid = (plo + phi) >> 1;
            if (tile_seg[mid] <= lo) plo = mid; else phi = mid;
        }
        const int32_t row = seg_row[lo];
        uint32_t c[kE];
        if constexpr (sizeof(I) == 2) {
            if (dmask && ((dmask[w >> 6] >> (w & 63)) & 1u)) {
                const uint32_t* rec = reinterpret_cast<const uint32_t*>(idx + w * kWin) + 3 * lane;
                delta_decode(rec[0], rec[1], rec[2], pad, c);
            } else {
                const uint4 v = *reinterpret_cast<const uint4*>(idx + q0);
                const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
                for (int e = 0; e < kE; ++e) c[e] = (wd[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
            }
        } else {
            const uint4 v0 = *reinterpret_cast<const uint4*>(idx + q0);
            const uint4 v1 = *reinterpret_cast<const uint4*>(idx + q0 + 4);
            const uint32_t wd[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            for (int e = 0; e < kE; ++e) c[e] = wd[e];
        }
        for (int e = 0; e < kE; ++e) {
            const uint32_t u = c[e] & IndexBits<I>::mask;
            c[e] = u == pad ? kNone : (uint32_t)plo * (uint32_t)T + (u < swz_lim ? lds_swizzle(u) : u);
        }
        __builtin_amdgcn_wave_barrier();  // the last window's reads come before these writes
        cols[wave][lane][0] = make_uint4(c[0], c[1], c[2], c[3]);
        cols[wave][lane][1] = make_uint4(c[4], c[5], c[6], c[7]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int it = it0; it < it0 + turns; ++it) {
            const int b = it * (64 / G) + grp;  // whose entries
            const int64_t i = __shfl(row, b);
            const uint4 ca = cols[wave][b][0], cb = cols[wave][b][1];
            const uint32_t j[kE] = {ca.x, ca.y, ca.z, ca.w, cb.x, cb.y, cb.z, cb.w};
            double pred[kE] = {};
            for (uint32_t t = 4 * g; t < pitch; t += 4 * G) {
                Row4<V> wt;
                for (int u = 0; u < 4; ++u) wt.v[u] = t + u < k ? W[(int64_t)(t + u) * m + i] : V(0);
                Row4<V> h[kE];
#pragma unroll
                for (int e = 0; e < kE; ++e)
                    h[e] = load4(HT + (j[e] == kNone ? 0 : (int64_t)j[e]) * pitch + t);
#pragma unroll
                for (int e = 0; e < kE; ++e)
                    for (int u = 0; u < 4; ++u)
                        pred[e] = __builtin_fma((double)wt.v[u], (double)h[e].v[u], pred[e]);
            }
            // Sums over the group; value v0 + i of the lane's kept ones ends in pred[i].
            int v0;
            if constexpr (G == 16) {
                deal<0x140, 4>(pred, g & 8);  // row_mirror: lane 15 - g
                deal<0x141, 2>(pred, g & 4);  // row_half_mirror: lane 7 - g of its half
                deal<0x4E, 1>(pred, g & 2);   // quad_perm: lane ^ 2
                pred[0] += dpp_from<0xB1>(pred[0]);  // quad_perm: lane ^ 1
                v0 = g >> 1;
            } else if constexpr (G == 8) {
                deal<0x141, 4>(pred, g & 4);
                deal<0x4E, 2>(pred, g & 2);
                deal<0xB1, 1>(pred, g & 1);
                v0 = g;
            } else {
                deal<0x4E, 4>(pred, g & 2);
                deal<0xB1, 2>(pred, g & 1);
                v0 = 2 * g;
            }
            constexpr int N = G == 4 ? 2 : 1;
            if (G < 16 || (g & 1) == 0) {
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const int e = v0 + n;
                    const int64_t f = val_slot<V>(w * kWin + b * kE + e);
                    const bool held = reinterpret_cast<const uint32_t*>(&cols[wave][b][0])[e] != kNone;
                    val[f] = held ? (V)((double)A[f] - pred[n]) : V(0);  // padding keeps value 0
                }
            }
        }
    }
}

template <class S, class V>
__global__ void k_copy_mapped(const S* __restrict__ src, const int32_t* __restrict__ smap,
                              V* __restrict__ dst, const int32_t* __restrict__ dmap,
                              int64_t n) {
    const Span sp = xcd_span(n);
    for (int64_t i = sp.lo; i < sp.hi; i += sp.step)
        dst[dmap ? dmap[i] : i] = (V)src[smap ? smap[i] : i];
}

// Bitwise comparison of the two copies (as unsigned words of the value's size).
template <class V>
__global__ void k_consistency(const V* __restrict__ a, const int32_t* __restrict__ amap,
                              const V* __restrict__ b, const int32_t* __restrict__ bmap,
                              int64_t n, unsigned long long* count) {
    using U = typename std::conditional<sizeof(V) == 4, uint32_t, uint64_t>::type;
    for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT)
        if (__builtin_bit_cast(U, a[amap[i]]) != __builtin_bit_cast(U, b[bmap[i]]))
            atomicAdd(count, 1ull);
}

// splitmix64 (Steele, Lea and Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014): a counter-based 64-bit generator.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// The initial H: entry (j, t) of the row-major n x k matrix over input ids, e = j k + t,
// is 0.1 z, z ~ N(0, 1) by the Box-Muller transform of the counter draws 2e and 2e + 1
// of a stream keyed by the seed, rounded to float; written column-major over
// relabelled ids (H[t n + j'] for j' = old2new[j]).
template <class V>
__global__ void k_initial_h(uint64_t seed, const int32_t* __restrict__ new2old, int64_t n,
                            int32_t k, V* __restrict__ H) {
    const uint64_t key = splitmix64(seed);
    const int64_t total = n * k;
    for (int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x; q < total;
         q += (int64_t)gridDim.x * kT) {
        const int64_t t = q / n;
        const int64_t jn = q - t * n;
        const uint64_t e = (uint64_t)new2old[jn] * (uint64_t)k + (uint64_t)t;
        const double u1 = (double)(splitmix64(key + 2 * e) >> 11) * 0x1.0p-53;
        const double u2 = (double)(splitmix64(key + 2 * e + 1) >> 11) * 0x1.0p-53;
        const double z = __builtin_sqrt(-2.0 * log1p(-u1)) * cos(6.283185307179586 * u2);
        H[q] = (V)(float)(0.1 * z);
    }
}

template <class V>
__global__ void k_seg_spread(const V* __restrict__ F, int64_t rows,
                             const int32_t* __restrict__ seg_row, int64_t S, int32_t k,
                             V* __restrict__ out) {
    const int64_t total = S * k;
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * kT) {
        const int64_t t = e / S;
        const int64_t sg = e - t * S;
        out[e] = F[t * rows + seg_row[sg]];
    }
}

// Workgroup b sums elements b*256 + t + s*(nparts*256) in order per thread, then a
// fixed tree: deterministic for a fixed nparts.
__device__ __forceinline__ void block_total(double acc, double* out) {
    __shared__ double s[kT];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kT / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

template <class V>
__global__ void k_sq_sum(const V* __restrict__ v, int64_t n, double* __restrict__ part) {
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
        const double d = v[i];
        acc = __builtin_fma(d, d, acc);
    }
    block_total(acc, &part[blockIdx.x]);
}

// A held-out triplet that no kernel may use.
__device__ __forceinline__ bool unusable(int32_t r, int32_t c, float a, int64_t m, int64_t n) {
    return r < 0 || (int64_t)r >= m || c < 0 || (int64_t)c >= n || !__builtin_isfinite(a);
}

// Squared prediction errors of held-out triplets, one fixed-order partial per block.
// CHECK: the triplets were not validated on the host; an entry whose indices are out
// of range or whose value is not finite is skipped (never used as an index) and
// counted in rejected[blockIdx.x] and *bad (either may be null).  Valid entries take the
// same arithmetic in the same order either way.
template <class V, bool CHECK>
__global__ void k_test_err(const int32_t* __restrict__ row, const int32_t* __restrict__ col,
                           const float* __restrict__ val, int64_t nnz,
                           const int32_t* __restrict__ rnew, const int32_t* __restrict__ cnew,
                           const V* __restrict__ W, const V* __restrict__ H, int64_t m,
                           int64_t n, int32_t k, double* __restrict__ part,
                           double* __restrict__ rejected, unsigned long long* bad) {
    double acc = 0.0;
    int refused = 0;
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * kT) {
        const int32_t r = row[e], c = col[e];
        const float a = val[e];
        if constexpr (CHECK) {
            if (unusable(r, c, a, m, n)) {
                ++refused;
                continue;
            }
        }
        const int64_t i = rnew[r];
        const int64_t j = cnew[c];
        double pred = 0.0;
#pragma unroll 8
        for (int32_t t = 0; t < k; ++t)
            pred = __builtin_fma((double)W[(int64_t)t * m + i], (double)H[(int64_t)t * n + j], pred);
        const double err = (double)a - pred;
        acc = __builtin_fma(err, err, acc);
    }
    block_total(acc, &part[blockIdx.x]);
    if constexpr (CHECK) {
        if (bad && refused) atomicAdd(bad, (unsigned long long)refused);
        if (rejected) {
            __syncthreads();  // block_total's LDS is reused
            block_total((double)refused, &rejected[blockIdx.x]);
        }
    }
}

// k_test_err with one or both factors as a row-major copy over relabelled ids (rows of
// `pitch` values, a multiple of 4, zero past k): four features per gather instead of one,
// and a row's gathers in the same lines.  WR, HR: which are row-major; the other one is
// column-major.  CHECK: as there.  The same sums in the same order.
template <class V, bool WR, bool HR, bool CHECK>
__global__ void k_test_err_rows(const int32_t* __restrict__ row, const int32_t* __restrict__ col,
                                const float* __restrict__ val, int64_t nnz,
                                const int32_t* __restrict__ rnew, const int32_t* __restrict__ cnew,
                                const V* __restrict__ W, const V* __restrict__ H, int64_t m, int64_t n,
                                uint32_t k, uint32_t pitch, double* __restrict__ part,
                                unsigned long long* bad) {
    double acc = 0.0;
    int refused = 0;
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * kT) {
        const int32_t r = row[e], c = col[e];
        const float a = val[e];
        if constexpr (CHECK) {
            if (unusable(r, c, a, m, n)) {
                ++refused;
                continue;
            }
        }
        const int64_t i = rnew[r], j = cnew[c];
        auto four = [&](auto rows, const V* F, int64_t r, int64_t len, uint32_t t) {
            Row4<V> x;
            if constexpr (decltype(rows)::value) {
                x = load4(F + r * pitch + t);
            } else {
                for (int u = 0; u < 4; ++u) x.v[u] = t + u < k ? F[(int64_t)(t + u) * len + r] : V(0);
            }
            return x;
        };
        double pred = 0.0;
#pragma unroll 4
        for (uint32_t t = 0; t < pitch; t += 4) {
            const Row4<V> w = four(std::bool_constant<WR>{}, W, i, m, t);
            const Row4<V> h = four(std::bool_constant<HR>{}, H, j, n, t);
            for (int u = 0; u < 4; ++u) pred = __builtin_fma((double)w.v[u], (double)h.v[u], pred);
        }
        const double err = (double)a - pred;
        acc = __builtin_fma(err, err, acc);
    }
    block_total(acc, &part[blockIdx.x]);
    if constexpr (CHECK) {
        if (refused) atomicAdd(bad, (unsigned long long)refused);
    }
}

// ---- segments of a tiled copy ----------------------------------------------------------
// A thread per row walks the row's pairs tile by tile: neighbouring threads read
// neighbouring words.  (The host's loops over 31M pairs and 18M segments took 0.4 s.)
__global__ void k_row_stats(const int32_t* __restrict__ cnt, int64_t rows, int32_t P, int32_t cold_tile,
                            int32_t* __restrict__ stats) {
    const int64_t r = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (r >= rows) return;
    int32_t segs = 0, cold = 0, all = 0;
    for (int32_t p = 0; p < P; ++p) {
        const int32_t c = cnt[(int64_t)p * rows + r];
        segs += c > 0;
        all += c;
        if (p >= cold_tile) cold += c;
    }
    stats[r] = segs;
    stats[rows + r] = cold;
    stats[2 * rows + r] = all;
}

// heads[p] = pad at tile p's first pair (heads[P]: past the last pair), heads[P + 1 + p] = segid
// there.
__global__ void k_tile_heads(const int32_t* __restrict__ cnt, const int32_t* __restrict__ segid,
                             const int64_t* __restrict__ pad, int64_t rows, int32_t P,
                             int64_t* __restrict__ heads) {
    const int64_t p = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (p < P) {
        heads[p] = pad[p * rows];
        heads[P + 1 + p] = segid[p * rows];
    } else if (p == P) {
        heads[P] = pad[P * rows - 1] + ((int64_t)cnt[P * rows - 1] + kE - 1) / kE * kE;
    }
}

// (blockIdx.y: the tile)
__global__ void k_seg_emit(const int32_t* __restrict__ cnt, const int32_t* __restrict__ segid,
                           const int64_t* __restrict__ pad, const int32_t* __restrict__ plain,
                           int64_t rows, const int64_t* __restrict__ tile_pad,
                           const int64_t* __restrict__ tile_base, int32_t* __restrict__ seg_row,
                           int64_t* __restrict__ seg_start, int32_t* __restrict__ seg_off) {
    const int p = (int)blockIdx.y;
    for (int64_t r = (int64_t)blockIdx.x * kT + threadIdx.x; r < rows; r += (int64_t)gridDim.x * kT) {
        const int64_t i = (int64_t)p * rows + r;
        if (cnt[i] == 0) continue;
        const int32_t sg = segid[i];
        const int64_t start = tile_base[p] + pad[i] - tile_pad[p];
        seg_row[sg] = (int32_t)r;
        seg_start[sg] = start;
        seg_off[sg] = (int32_t)(start - plain[i]);
    }
}

__global__ void k_mark_cuts(const int32_t* __restrict__ cut_seg, int64_t n, int32_t* __restrict__ cut_of) {
    const int64_t c = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (c < n) cut_of[cut_seg[c]] = (int32_t)c;
}

__global__ void k_row_counts(const int32_t* __restrict__ cnt, const int32_t* __restrict__ segid,
                             int64_t rows, int32_t P, const int32_t* __restrict__ cut_of,
                             const int32_t* __restrict__ cut_off, int32_t* __restrict__ nsegs,
                             int32_t* __restrict__ nslots) {
    const int64_t r = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (r > rows) return;
    int32_t segs = 0, slots = 0;
    for (int32_t p = 0; r < rows && p < P; ++p) {
        const int64_t i = (int64_t)p * rows + r;
        if (cnt[i] == 0) continue;
        const int32_t c = cut_of[segid[i]];
        ++segs;
        slots += c < 0 ? 1 : cut_off[c + 1] - cut_off[c];
    }
    nsegs[r] = segs;
    nslots[r] = slots;
}

__global__ void k_row_lists(const int32_t* __restrict__ cnt, const int32_t* __restrict__ segid,
                            int64_t rows, int32_t P, const int32_t* __restrict__ cut_of,
                            const int32_t* __restrict__ cut_off, const int32_t* __restrict__ cut_slot,
                            const int32_t* __restrict__ seg_ptr, const int32_t* __restrict__ slot_ptr,
                            int32_t* __restrict__ segs, int32_t* __restrict__ slots) {
    const int64_t r = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (r >= rows) return;
    int32_t a = seg_ptr[r], b = slot_ptr[r];
    for (int32_t p = 0; p < P; ++p) {
        const int64_t i = (int64_t)p * rows + r;
        if (cnt[i] == 0) continue;
        const int32_t sg = segid[i], c = cut_of[sg];
        segs[a++] = sg;
        if (c < 0) {
            slots[b++] = sg;
        } else {
            for (int32_t k = cut_off[c]; k < cut_off[c + 1]; ++k) slots[b++] = cut_slot[k];
        }
    }
}

// The same with a wave per row, a lane per tile: for rows too few to fill the chip and tiles
// enough for the lanes (row_waves).  (100 rows, 62,500 tiles: 15, 17 and 18 ms with a thread per
// row.)
__device__ __forceinline__ int32_t wave_total(int32_t x) {
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d);
    return x;
}
__global__ void k_row_stats_wave(const int32_t* __restrict__ cnt, int64_t rows, int32_t P, int32_t cold_tile,
                                 int32_t* __restrict__ stats) {
    const int64_t r = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    const int lane = (int)(threadIdx.x & 63u);
    if (r >= rows) return;  // (whole waves)
    int32_t segs = 0, cold = 0, all = 0;
    for (int64_t p = lane; p < P; p += 64) {
        const int32_t c = cnt[p * rows + r];
        segs += c > 0;
        all += c;
        if (p >= cold_tile) cold += c;
    }
    segs = wave_total(segs);
    cold = wave_total(cold);
    all = wave_total(all);
    if (lane == 0) {
        stats[r] = segs;
        stats[rows + r] = cold;
        stats[2 * rows + r] = all;
    }
}

__global__ void k_row_counts_wave(const int32_t* __restrict__ cnt, const int32_t* __restrict__ segid,
                                  int64_t rows, int32_t P, const int32_t* __restrict__ cut_of,
                                  const int32_t* __restrict__ cut_off, int32_t* __restrict__ nsegs,
                                  int32_t* __restrict__ nslots) {
    const int64_t r = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    const int lane = (int)(threadIdx.x & 63u);
    if (r > rows) return;
    int32_t segs = 0, slots = 0;
    for (int64_t p = lane; r < rows && p < P; p += 64) {
        const int64_t i = p * rows + r;
        if (cnt[i] == 0) continue;
        const int32_t c = cut_of[segid[i]];
        ++segs;
        slots += c < 0 ? 1 : cut_off[c + 1] - cut_off[c];
    }
    segs = wave_total(segs);
    slots = wave_total(slots);
    if (lane == 0) {
        nsegs[r] = segs;
        nslots[r] = slots;
    }
}

__global__ void k_row_lists_wave(const int32_t* __restrict__ cnt, const int32_t* __restrict__ segid,
                                 int64_t rows, int32_t P, const int32_t* __restrict__ cut_of,
                                 const int32_t* __restrict__ cut_off, const int32_t* __restrict__ cut_slot,
                                 const int32_t* __restrict__ seg_ptr, const int32_t* __restrict__ slot_ptr,
                                 int32_t* __restrict__ segs, int32_t* __restrict__ slots) {
    const int64_t r = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    const int lane = (int)(threadIdx.x & 63u);
    if (r >= rows) return;
    int32_t a = seg_ptr[r], b = slot_ptr[r];
    for (int64_t p0 = 0; p0 < P; p0 += 64) {
        const int64_t i = (p0 + lane) * rows + r;
        const bool held = p0 + lane < P && cnt[i] != 0;
        const int32_t sg = held ? segid[i] : 0, c = held ? cut_of[sg] : -1;
        const int32_t n = !held ? 0 : c < 0 ? 1 : cut_off[c + 1] - cut_off[c];
        const uint64_t mask = __ballot(held);
        int32_t upto = n;  // slots of the lanes up to this one
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t x = __shfl_up(upto, d);
            if (lane >= d) upto += x;
        }
        if (held) {
            segs[a + __popcll(mask & ((1ull << lane) - 1))] = sg;
            const int32_t at = b + upto - n;
            if (c < 0) {
                slots[at] = sg;
            } else {
                for (int32_t k = 0; k < n; ++k) slots[at + k] = cut_slot[cut_off[c] + k];
            }
        }
        a += __popcll(mask);
        b += __shfl(upto, 63);
    }
}

struct NonEmpty {
    __host__ __device__ int32_t operator()(int32_t c) const { return c > 0; }
};
struct Padded {
    __host__ __device__ int64_t operator()(int32_t c) const { return ((int64_t)c + kE - 1) / kE * kE; }
};
template <class In, class T>
hipError_t scan_to(In in, T* out, int64_t n, hipStream_t s, const TakeFn& take) {
    size_t need = 0;
    void* tmp = nullptr;
    hipError_t e = rocprim::exclusive_scan(nullptr, need, in, out, T(0), (size_t)n, rocprim::plus<T>(), s);
    if (e == hipSuccess) e = take(&tmp, need);
    if (e != hipSuccess) return e;
    return rocprim::exclusive_scan(tmp, need, in, out, T(0), (size_t)n, rocprim::plus<T>(), s);
}

// Counts triplets that a kernel must not use (one atomic per wave that has any).
__global__ void k_check_triplets(const int32_t* __restrict__ row, const int32_t* __restrict__ col,
                                 const float* __restrict__ val, int64_t nnz, int64_t m, int64_t n,
                                 unsigned long long* bad) {
    int count = 0;
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * kT) {
        count += unusable(row[e], col[e], val[e], m, n);
    }
    if (count) atomicAdd(bad, (unsigned long long)count);
}
template <class S>
__global__ void k_check_finite(const S* __restrict__ v, int64_t n, unsigned long long* bad) {
    int count = 0;
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT)
        count += !__builtin_isfinite(v[e]);
    if (count) atomicAdd(bad, (unsigned long long)count);
}

}  // namespace

// The limits are the process's, so they are always set to the most any call asks for: a create
// on another thread cannot lower them between a set and a launch.
hipError_t build_init() {
    for (const void* k : {(const void*)k_histogram<true>, (const void*)k_seg_histogram_runs}) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kHistLdsBins * 4);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Whether a row's pairs take a wave (a thread per row would leave compute units idle).
static bool row_waves(int64_t rows, int32_t P) { return rows < 16384 && P >= 64; }
hipError_t launch_row_stats(const int32_t* cnt, int64_t rows, int32_t P, int32_t cold_tile,
                            int32_t* stats, hipStream_t s) {
    if (row_waves(rows, P))
        hipLaunchKernelGGL(k_row_stats_wave, grid_for(rows * 64), dim3(kT), 0, s, cnt, rows, P, cold_tile, stats);
    else
        hipLaunchKernelGGL(k_row_stats, grid_for(rows), dim3(kT), 0, s, cnt, rows, P, cold_tile, stats);
    return hipGetLastError();
}
hipError_t launch_tile_heads(const int32_t* cnt, const int32_t* segid, const int64_t* pad, int64_t rows,
                             int32_t P, int64_t* heads, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_heads, grid_for((int64_t)P + 1, 1 << 24), dim3(kT), 0, s, cnt, segid, pad, rows,
                       P, heads);
    return hipGetLastError();
}
hipError_t launch_seg_emit(const int32_t* cnt, const int32_t* segid, const int64_t* pad,
                           const int32_t* plain, int64_t rows, int32_t P, const int64_t* tile_pad,
                           const int64_t* tile_base, int32_t* seg_row, int64_t* seg_start,
                           int32_t* seg_off, hipStream_t s) {
    // (the grid's second dimension is limited to 65,535: more tiles go in turns)
    for (int32_t p = 0; p < P; p += 65535) {
        const int32_t np = std::min(P - p, 65535);
        dim3 grid = grid_for(rows, 4096);
        grid.y = (unsigned)np;
        const int64_t at = (int64_t)p * rows;
        hipLaunchKernelGGL(k_seg_emit, grid, dim3(kT), 0, s, cnt + at, segid + at, pad + at, plain + at,
                           rows, tile_pad + p, tile_base + p, seg_row, seg_start, seg_off);
    }
    return hipGetLastError();
}
hipError_t launch_mark_cuts(const int32_t* cut_seg, int64_t n, int32_t* cut_of, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mark_cuts, grid_for(n), dim3(kT), 0, s, cut_seg, n, cut_of);
    return hipGetLastError();
}
hipError_t launch_row_counts(const int32_t* cnt, const int32_t* segid, int64_t rows, int32_t P,
                             const int32_t* cut_of, const int32_t* cut_off, int32_t* nsegs,
                             int32_t* nslots, hipStream_t s) {
    if (row_waves(rows, P))
        hipLaunchKernelGGL(k_row_counts_wave, grid_for((rows + 1) * 64), dim3(kT), 0, s, cnt, segid, rows, P,
                           cut_of, cut_off, nsegs, nslots);
    else
        hipLaunchKernelGGL(k_row_counts, grid_for(rows + 1), dim3(kT), 0, s, cnt, segid, rows, P, cut_of,
                           cut_off, nsegs, nslots);
    return hipGetLastError();
}
hipError_t launch_row_lists(const int32_t* cnt, const int32_t* segid, int64_t rows, int32_t P,
                            const int32_t* cut_of, const int32_t* cut_off, const int32_t* cut_slot,
                            const int32_t* seg_ptr, const int32_t* slot_ptr, int32_t* segs,
                            int32_t* slots, hipStream_t s) {
    if (row_waves(rows, P))
        hipLaunchKernelGGL(k_row_lists_wave, grid_for(rows * 64), dim3(kT), 0, s, cnt, segid, rows, P, cut_of,
                           cut_off, cut_slot, seg_ptr, slot_ptr, segs, slots);
    else
        hipLaunchKernelGGL(k_row_lists, grid_for(rows), dim3(kT), 0, s, cnt, segid, rows, P, cut_of, cut_off,
                           cut_slot, seg_ptr, slot_ptr, segs, slots);
    return hipGetLastError();
}
hipError_t scan_segments(const int32_t* cnt, int64_t n, int32_t* segid, int64_t* pad, int32_t* plain,
                         hipStream_t s, const TakeFn& take) {
    hipError_t e = scan_to(rocprim::make_transform_iterator(cnt, NonEmpty()), segid, n, s, take);
    if (e == hipSuccess) e = scan_to(rocprim::make_transform_iterator(cnt, Padded()), pad, n, s, take);
    if (e == hipSuccess) e = scan_to(cnt, plain, n, s, take);
    return e;
}
hipError_t scan_counts(int32_t* a, int64_t n, hipStream_t s, const TakeFn& take) {
    return scan_to(a, a, n, s, take);
}

hipError_t launch_check_triplets(const int32_t* row, const int32_t* col, const float* val, int64_t nnz,
                                 int64_t m, int64_t n, unsigned long long* bad, hipStream_t s) {
    if (nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_triplets, grid_for(nnz, 4096), dim3(kT), 0, s, row, col, val, nnz, m, n,
                       bad);
    return hipGetLastError();
}
template <class S>
hipError_t launch_check_finite(const S* v, int64_t n, unsigned long long* bad, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_finite<S>, grid_for(n, 4096), dim3(kT), 0, s, v, n, bad);
    return hipGetLastError();
}
template hipError_t launch_check_finite<float>(const float*, int64_t, unsigned long long*, hipStream_t);
template hipError_t launch_check_finite<double>(const double*, int64_t, unsigned long long*, hipStream_t);

hipError_t launch_histogram(const int32_t* key, int64_t n, int32_t bins, int32_t* count,
                           int32_t workgroups, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (bins <= kHistLdsBins) {
        const size_t lds = (size_t)bins * 4;
        const int64_t g = std::min<int64_t>(workgroups, (n + 1023) / 1024);
        hipLaunchKernelGGL(k_histogram<true>, dim3((unsigned)g), dim3(1024), lds, s, key, n, bins,
                           count);
    } else {
        hipLaunchKernelGGL(k_histogram<false>, grid_for(n, 8192), dim3(kT), 0, s, key, n, bins,
                           count);
    }
    return hipGetLastError();
}

hipError_t launch_map(const int32_t* in, const int32_t* table, int64_t n, int32_t* out,
                      hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_map, grid_for(n), dim3(kT), 0, s, in, table, n, out);
    return hipGetLastError();
}

hipError_t launch_seg_histogram(const int32_t* lrow, const int32_t* lcol, int64_t nnz,
                                int32_t rows, int32_t T, const int32_t* order, int32_t workgroups,
                                int32_t* count, hipStream_t s) {
    if (nnz == 0) return hipSuccess;
    if (order && rows <= kHistLdsBins) {
        const size_t lds = (size_t)rows * 4;
        // (runs of at least two entries per word that a workgroup clears and adds)
        const int64_t g = std::max<int64_t>(1, std::min<int64_t>(workgroups, nnz / (2 * (int64_t)rows + 1)));
        hipLaunchKernelGGL(k_seg_histogram_runs, dim3((unsigned)g), dim3(1024), lds, s, order, lrow, lcol,
                           nnz, rows, T, count);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_seg_histogram, grid_for(nnz, 8192), dim3(kT), 0, s, lrow, lcol, nnz, rows,
                       T, count);
    return hipGetLastError();
}

hipError_t launch_seg_keys(const int32_t* lrow, const int32_t* lcol, const int32_t* segid,
                           int64_t nnz, int32_t rows, int32_t T, int cbits, uint64_t* keys,
                           int32_t* ids, hipStream_t s) {
    if (nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(k_seg_keys, grid_for(nnz), dim3(kT), 0, s, lrow, lcol, segid, nnz, rows, T,
                       cbits, keys, ids);
    return hipGetLastError();
}

hipError_t launch_dup_check(const uint64_t* keys, int64_t nnz, int32_t* flag, hipStream_t s) {
    if (nnz < 2) return hipSuccess;
    hipLaunchKernelGGL(k_dup_check, grid_for(nnz), dim3(kT), 0, s, keys, nnz, flag);
    return hipGetLastError();
}

template <class V>
hipError_t launch_layout_fill(const uint64_t* keys, const int32_t* perm, const float* val_in,
                              int64_t nnz, int cbits, const int32_t* seg_off, uint32_t swz_lim, bool idx16,
                              void* idx, V* val, int32_t* pos, hipStream_t s) {
    if (nnz == 0) return hipSuccess;
    const uint64_t mask = cbits >= 64 ? ~0ull : ((1ull << cbits) - 1);
    if (idx16)
        hipLaunchKernelGGL((k_layout_fill<uint16_t, V>), grid_for(nnz), dim3(kT), 0, s, keys, perm,
                           val_in, nnz, cbits, mask, seg_off, swz_lim, static_cast<uint16_t*>(idx), val,
                           pos);
    else
        hipLaunchKernelGGL((k_layout_fill<int32_t, V>), grid_for(nnz), dim3(kT), 0, s, keys, perm,
                           val_in, nnz, cbits, mask, seg_off, swz_lim, static_cast<int32_t*>(idx), val,
                           pos);
    return hipGetLastError();
}

hipError_t launch_fill_idx(void* idx, bool idx16, int32_t value, int64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (idx16)
        hipLaunchKernelGGL(k_fill_idx<uint16_t>, grid_for(n), dim3(kT), 0, s,
                           static_cast<uint16_t*>(idx), (uint16_t)value, n);
    else
        hipLaunchKernelGGL(k_fill_idx<int32_t>, grid_for(n), dim3(kT), 0, s,
                           static_cast<int32_t*>(idx), value, n);
    return hipGetLastError();
}

hipError_t launch_invert(const int32_t* perm, int64_t n, int32_t* inv, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_invert, grid_for(n), dim3(kT), 0, s, perm, n, inv);
    return hipGetLastError();
}

hipError_t launch_compose(const int32_t* a, const int32_t* b, int64_t n, int32_t* out,
                          hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_compose, grid_for(n), dim3(kT), 0, s, a, b, n, out);
    return hipGetLastError();
}

hipError_t launch_slot_map(const int32_t* from, const int32_t* to, int64_t n, int32_t* out,
                          hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_slot_map, grid_for(n), dim3(kT), 0, s, from, to, n, out);
    return hipGetLastError();
}

template <class V>
hipError_t launch_copy_slots(const V* src, const int32_t* map, V* dst, int64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((k_copy_slots<V>), xcd_grid(n), dim3(kT), 0, s, src, map, dst, n);
    return hipGetLastError();
}

template <class V>
hipError_t launch_fill(V* dst, V value, int64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill<V>, grid_for(n), dim3(kT), 0, s, dst, value, n);
    return hipGetLastError();
}

template <class S, class V>
hipError_t launch_scatter_factor_in(const S* rowmajor, const int32_t* new2old, int64_t rows,
                                    int32_t k, V* colmajor, hipStream_t s) {
    if (rows * k <= (k <= 4 ? kTurnNarrow : kTurnSmall)) {
        hipLaunchKernelGGL((k_factor_in_small<S, V>), grid_for(rows * k), dim3(kT), 0, s, rowmajor,
                           new2old, (uint32_t)rows, (uint32_t)k, colmajor);
        return hipGetLastError();
    }
    int shift;
    const dim3 grid = turn_grid(rows, k, &shift);
    hipLaunchKernelGGL((k_factor_in<S, V>), grid, dim3(kT), 0, s, rowmajor, new2old, rows, (int64_t)k,
                       shift, colmajor);
    return hipGetLastError();
}

template <class V, class S>
hipError_t launch_factor_out(const V* colmajor, const int32_t* new2old, const int32_t* old2new,
                             int64_t rows, int32_t k, int64_t pitch, S* rowmajor, hipStream_t s) {
    if (rows * pitch <= kTurnSmall) {
        hipLaunchKernelGGL((k_factor_out_small<V, S>), grid_for(rows * pitch), dim3(kT), 0, s, colmajor,
                           old2new, (uint32_t)rows, (uint32_t)k, (uint32_t)pitch, rowmajor);
        return hipGetLastError();
    }
    int shift;
    const dim3 grid = turn_grid(rows, pitch, &shift);
    hipLaunchKernelGGL((k_factor_out<V, S>), grid, dim3(kT), 0, s, colmajor, new2old, rows, (int64_t)k,
                       pitch, shift, rowmajor);
    return hipGetLastError();
}

hipError_t launch_delta_windows(void* idx, int64_t npad, int32_t pad, uint64_t* dmask,
                                hipStream_t s) {
    const int64_t nwin = npad / kWin;
    if (nwin == 0) return hipSuccess;
    hipLaunchKernelGGL(k_delta_windows, dim3((unsigned)((nwin + kT / 64 - 1) / (kT / 64))), dim3(kT),
                       0, s, static_cast<uint16_t*>(idx), nwin, (uint32_t)pad, dmask);
    return hipGetLastError();
}

template <class I, class V>
static void rebuild_groups(const Layout& L, const V* A, const V* W, const V* HT, int64_t m, int32_t k,
                           hipStream_t s) {
    // Lanes per row of HT: as many as its values fill, four each.
    const uint32_t pitch = (uint32_t)row_pitch(k);
    const int groups = pitch <= 16 ? 4 : pitch <= 32 ? 8 : 16;
    const int64_t nwin = L.npad / kWin;
    int parts = 1;
    while (parts < groups && nwin * parts < kRebuildWaves) parts *= 2;
    const dim3 grid = grid_for(nwin * parts * 64, 1 << 14);
#define CCDK_REBUILD(G)                                                                            \
    hipLaunchKernelGGL((k_rebuild<I, V, G>), grid, dim3(kT), 0, s, L.seg_start, L.nseg, L.seg_row,   \
                       L.tile_seg, L.P, L.T, L.swz_lim, static_cast<const I*>(L.idx),                \
                       sizeof(I) == 2 ? L.dmask : nullptr, (uint32_t)L.pad, A, W, HT, m,             \
                       (uint32_t)k, pitch, L.npad, parts, static_cast<V*>(L.val))
    if (groups == 4)
        CCDK_REBUILD(4);
    else if (groups == 8)
        CCDK_REBUILD(8);
    else
        CCDK_REBUILD(16);
#undef CCDK_REBUILD
}
template <class I, class V>
static void rebuild_any(const Layout& L, const int32_t* pos, const V* A, const V* W, const V* H,
                        const V* HT, int64_t m, int32_t k, hipStream_t s) {
    if (HT) return rebuild_groups<I, V>(L, A, W, HT, m, k, s);
    hipLaunchKernelGGL((k_rebuild_each<I, V>), grid_for(L.nnz), dim3(kT), 0, s, L.seg_start, L.nseg,
                       L.seg_row, L.tile_seg, L.P, L.T, L.swz_lim, static_cast<const I*>(L.idx),
                       sizeof(I) == 2 ? L.dmask : nullptr, (uint32_t)L.pad, pos, A, W, H, m, L.cols, k,
                       L.nnz, static_cast<V*>(L.val));
}

template <class V>
hipError_t launch_rebuild_residual(const Layout& L, const int32_t* pos, const V* A, const V* W,
                                   const V* H, const V* HT, int64_t m, int32_t k, hipStream_t s) {
    if (L.nnz == 0) return hipSuccess;
    if (L.idx16)
        rebuild_any<uint16_t, V>(L, pos, A, W, H, HT, m, k, s);
    else
        rebuild_any<int32_t, V>(L, pos, A, W, H, HT, m, k, s);
    return hipGetLastError();
}

template <class S, class V>
hipError_t launch_copy_mapped(const S* src, const int32_t* smap, V* dst, const int32_t* dmap,
                              int64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((k_copy_mapped<S, V>), xcd_grid(n), dim3(kT), 0, s, src, smap, dst, dmap, n);
    return hipGetLastError();
}

template <class V>
hipError_t launch_consistency(const V* a, const int32_t* amap, const V* b, const int32_t* bmap,
                              int64_t n, unsigned long long* count, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_consistency<V>, grid_for(n), dim3(kT), 0, s, a, amap, b, bmap, n, count);
    return hipGetLastError();
}

template <class V>
hipError_t launch_initial_h(uint64_t seed, const int32_t* new2old, int64_t n, int32_t k, V* H,
                            hipStream_t s) {
    if (n * k == 0) return hipSuccess;
    hipLaunchKernelGGL(k_initial_h<V>, grid_for(n * k), dim3(kT), 0, s, seed, new2old, n, k, H);
    return hipGetLastError();
}

template <class V>
hipError_t launch_seg_spread(const V* F, int64_t rows, const int32_t* seg_row, int64_t S,
                             int32_t k, V* out, hipStream_t s) {
    if (S == 0 || k == 0) return hipSuccess;
    hipLaunchKernelGGL(k_seg_spread<V>, grid_for(S * k), dim3(kT), 0, s, F, rows, seg_row, S, k,
                       out);
    return hipGetLastError();
}

template <class V>
hipError_t launch_sq_sum(const V* v, int64_t n, double* part, int32_t nparts, hipStream_t s) {
    hipLaunchKernelGGL(k_sq_sum<V>, dim3(nparts), dim3(kT), 0, s, v, n, part);
    return hipGetLastError();
}

template <class V>
hipError_t launch_test_err(const int32_t* row, const int32_t* col, const float* val, int64_t nnz,
                           const int32_t* rold2new, const int32_t* cold2new, const V* W,
                           const V* H, int64_t m, int64_t n, int32_t k, double* part,
                           int32_t nparts, double* rejected, unsigned long long* bad,
                           hipStream_t s) {
    if (rejected || bad)
        hipLaunchKernelGGL((k_test_err<V, true>), dim3(nparts), dim3(kT), 0, s, row, col, val, nnz,
                           rold2new, cold2new, W, H, m, n, k, part, rejected, bad);
    else
        hipLaunchKernelGGL((k_test_err<V, false>), dim3(nparts), dim3(kT), 0, s, row, col, val, nnz,
                           rold2new, cold2new, W, H, m, n, k, part, nullptr, nullptr);
    return hipGetLastError();
}

template <class V>
hipError_t launch_test_err_rows(const int32_t* row, const int32_t* col, const float* val, int64_t nnz,
                                const int32_t* rold2new, const int32_t* cold2new, const V* W,
                                const V* H, const V* WT, const V* HT, int64_t m, int64_t n, int32_t k,
                                double* part, int32_t nparts, unsigned long long* bad, hipStream_t s) {
    const auto kernel = WT && HT ? (bad ? k_test_err_rows<V, true, true, true> : k_test_err_rows<V, true, true, false>)
                        : HT ? (bad ? k_test_err_rows<V, false, true, true> : k_test_err_rows<V, false, true, false>)
                             : (bad ? k_test_err_rows<V, true, false, true> : k_test_err_rows<V, true, false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)nparts), dim3(kT), 0, s, row, col, val, nnz, rold2new, cold2new,
                       WT ? WT : W, HT ? HT : H, m, n, (uint32_t)k, (uint32_t)row_pitch(k), part, bad);
    return hipGetLastError();
}

#define CCDK_BUILD_INSTANTIATE(V)                                                               \
    template hipError_t launch_layout_fill<V>(const uint64_t*, const int32_t*, const float*,    \
                                              int64_t, int, const int32_t*, uint32_t, bool, void*, \
                                              V*, int32_t*, hipStream_t);                       \
    template hipError_t launch_fill<V>(V*, V, int64_t, hipStream_t);                            \
    template hipError_t launch_copy_slots<V>(const V*, const int32_t*, V*, int64_t, hipStream_t); \
    template hipError_t launch_scatter_factor_in<float, V>(const float*, const int32_t*,        \
                                                           int64_t, int32_t, V*, hipStream_t);  \
    template hipError_t launch_scatter_factor_in<double, V>(const double*, const int32_t*,      \
                                                            int64_t, int32_t, V*, hipStream_t); \
    template hipError_t launch_factor_out<V, float>(const V*, const int32_t*, const int32_t*,   \
                                                    int64_t, int32_t, int64_t, float*, hipStream_t); \
    template hipError_t launch_factor_out<V, double>(const V*, const int32_t*, const int32_t*,  \
                                                     int64_t, int32_t, int64_t, double*, hipStream_t); \
    template hipError_t launch_rebuild_residual<V>(const Layout&, const int32_t*, const V*,     \
                                                   const V*, const V*, const V*, int64_t,       \
                                                   int32_t, hipStream_t);                       \
    template hipError_t launch_test_err_rows<V>(const int32_t*, const int32_t*, const float*,   \
                                                int64_t, const int32_t*, const int32_t*,        \
                                                const V*, const V*, const V*, const V*,         \
                                                int64_t, int64_t, int32_t, double*, int32_t,    \
                                                unsigned long long*, hipStream_t);              \
    template hipError_t launch_copy_mapped<V, V>(const V*, const int32_t*, V*, const int32_t*,  \
                                                 int64_t, hipStream_t);                         \
    template hipError_t launch_consistency<V>(const V*, const int32_t*, const V*,               \
                                              const int32_t*, int64_t, unsigned long long*,     \
                                              hipStream_t);                                     \
    template hipError_t launch_seg_spread<V>(const V*, int64_t, const int32_t*, int64_t,        \
                                             int32_t, V*, hipStream_t);                         \
    template hipError_t launch_initial_h<V>(uint64_t, const int32_t*, int64_t, int32_t, V*,     \
                                            hipStream_t);                                       \
    template hipError_t launch_sq_sum<V>(const V*, int64_t, double*, int32_t, hipStream_t);     \
    template hipError_t launch_test_err<V>(const int32_t*, const int32_t*, const float*,        \
                                           int64_t, const int32_t*, const int32_t*, const V*,   \
                                           const V*, int64_t, int64_t, int32_t, double*,        \
                                           int32_t, double*, unsigned long long*, hipStream_t);
CCDK_BUILD_INSTANTIATE(float)
CCDK_BUILD_INSTANTIATE(double)
#undef CCDK_BUILD_INSTANTIATE
template hipError_t launch_copy_mapped<double, float>(const double*, const int32_t*, float*,
                                                      const int32_t*, int64_t, hipStream_t);
template hipError_t launch_copy_mapped<float, double>(const float*, const int32_t*, double*,
                                                      const int32_t*, int64_t, hipStream_t);

// Radix sort of (key, id) pairs on the low `bits` bits of the key.
hipError_t sort_pairs(const uint64_t* kin, uint64_t* kout, const int32_t* vin, int32_t* vout,
                      int64_t n, int bits, hipStream_t s, const TakeFn& take) {
    size_t need = 0;
    void* tmp = nullptr;
    hipError_t e = rocprim::radix_sort_pairs(nullptr, need, kin, kout, vin, vout, (size_t)n, 0u,
                                             (unsigned)bits, s);
    if (e == hipSuccess) e = take(&tmp, need);
    if (e != hipSuccess) return e;
    return rocprim::radix_sort_pairs(tmp, need, kin, kout, vin, vout, (size_t)n, 0u,
                                     (unsigned)bits, s);
}

hipError_t select_range(const int32_t* key, int64_t n, int32_t lo, int32_t hi, int32_t* out,
                        int64_t* count, hipStream_t s, const TakeFn& take) {
    const rocprim::counting_iterator<int32_t> ids(0);
    const KeyInRange pred{key, lo, hi};
    size_t need = 0;
    void* tmp = nullptr;
    hipError_t e = rocprim::select(nullptr, need, ids, out, count, (size_t)n, pred, s);
    if (e == hipSuccess) e = take(&tmp, need);
    if (e != hipSuccess) return e;
    return rocprim::select(tmp, need, ids, out, count, (size_t)n, pred, s);
}

hipError_t launch_add(int32_t* a, int64_t n, int32_t delta, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_add, grid_for(n), dim3(kT), 0, s, a, n, delta);
    return hipGetLastError();
}

}  // namespace ccdk
