// Preprocessing (Section 2.1; Section 3.1 host step 3): per client row, order
// the facilities by (distance, index) and emit the first K = m - p + 1
// entries of the ordering Pi', the gap terms Delta' and the sorted distances
// D'.
//
// One workgroup sorts one row in LDS by a stable least-significant-digit
// radix sort of the distances (Knuth, TAOCP 3, 5.2.5).  The facilities enter
// in index order, so stability alone breaks ties by the lower index, the
// order the paper's Example 1 prints.
#include <algorithm>

#include "common.hpp"

namespace pmp {

namespace {

constexpr int kSortThreads = 512;  // workgroups of the device-memory sort below

// ---------------------------------------------------------------------------
// k_radix_rows: a workgroup of NW waves sorts a row of up to NW I 64
// facilities, wave w holding the I vectors of 64 consecutive facilities from
// w I on in registers.
//
// The row's widest distance (an OR over the row) gives the bits to sort by
// and so the passes: ceil(bits / 8) of bits / passes bits each, 6 at least
// (graph distances below 2^8 take one, a 10^4 grid's two, rows of zeros none).
// A pass counts and ranks: for each of its vectors in order a wave finds the
// lanes with the same digit by a ballot per digit bit, a lane's rank is the
// wave's count of the digit so far plus the equal lanes below it, and the
// lowest of the equal lanes adds their number to the count (a wave's LDS
// accesses execute in order, so the vectors pipeline without waits).  Two
// waves share a 32-bit word of counts, 16 bits each.  An exclusive sum over
// (digit, wave) then gives every wave's first place of each digit, and the
// keys are scattered to their places in LDS.
//
// While every distance is below 2^16 a key is distance << 16 | facility, one
// LDS word; otherwise distances and facilities are scattered to two arrays.
//
// Bound: a vector costs about 4 VALU instructions per digit bit and 20 per
// pass, and the waves wait at four barriers a pass.  A bitonic network in LDS
// (91 compare-exchange stages at m = 5000) took 792 us for 5000 rows of
// 14-bit distances, moving every key through LDS in every stage; this sort
// takes 121 us (350 MB of rows and tables: 2.9 TB/s), 178 us with 21-bit
// distances.  900 rows of 900 (one pass): 37 -> 7 us; 777 rows of 20001 with
// 21 bits: 1.28 ms in device memory -> 0.19 ms.  Shapes (waves, vectors per
// wave) follow m so that at most a few vectors are padding: rows up to 8192
// keep two or more workgroups per CU (16 waves of 5 vectors instead of 8 of
// 10 leave one: 182 us), wider ones take one workgroup of 16 waves and its
// CU's LDS, 6 bytes a facility.
// ---------------------------------------------------------------------------
constexpr int kDigits = 256;

template <int NW>
constexpr int count_words()  // one set of counts: two waves to a word
{
    return NW / 2 * kDigits;
}

// Counts and ranks of one pass (DB digit bits from bit sh of the keys): a
// wave's counts go to its half of the words `mine`, each key's place among
// the wave's keys of its digit to the low half of rank.
template <int DB, int I, bool NARROW>
__device__ __forceinline__ void radix_count(const uint32_t (&key)[I], uint32_t (&rank)[I], int sh,
                                            uint32_t *mine, int half)
{
#pragma unroll
    for (int r = 0; r < I; ++r) {
        const uint32_t d = (key[r] >> sh) & (uint32_t)((1 << DB) - 1);
        uint32_t lo = 0u, hi = 0u;  // lanes with another digit
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            const uint32_t t = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);  // 0 or all ones
            const uint64_t ones = __builtin_amdgcn_ballot_w64(t != 0u);
            lo |= (uint32_t)ones ^ t;
            hi |= (uint32_t)(ones >> 32) ^ t;
        }
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(~hi, __builtin_amdgcn_mbcnt_lo(~lo, 0u));
        // every lane reads before the lowest lane of each digit adds
        const uint32_t before =
            __hip_atomic_load(mine + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (below == 0u)
            __hip_atomic_fetch_add(mine + d,
                                   (uint32_t)(64 - __builtin_popcount(lo) - __builtin_popcount(hi))
                                       << half,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const uint32_t place = ((before >> half) & 0xFFFFu) + below;
        rank[r] = NARROW ? place : (rank[r] & 0xFFFF0000u) | place;
    }
}

template <int NW, int I, bool NARROW>
__device__ __forceinline__ void radix_sort_row(uint32_t (&key)[I], int bits, uint32_t *counts,
                                               uint32_t *wave_total, uint32_t *keys,
                                               uint16_t *idx)
{
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int first = wave * I * 64 + lane;
    // digits of 6, 7 or 8 bits (two waves: at most 7, a digit per thread)
    constexpr int kMost = NW >= 4 ? 8 : 7;
    const int passes = (bits + kMost - 1) / kMost;
    const int db = passes ? max(6, (bits + passes - 1) / passes) : 0;
    // low half: the rank in a pass; high half: the facility (not NARROW)
    uint32_t rank[I];
#pragma unroll
    for (int r = 0; r < I; ++r)
        rank[r] = NARROW ? 0u : (uint32_t)(first + 64 * r) << 16;
    if (passes == 0) {  // all distances zero: index order
#pragma unroll
        for (int r = 0; r < I; ++r) {
            keys[first + 64 * r] = key[r];
            if constexpr (!NARROW)
                idx[first + 64 * r] = (uint16_t)(rank[r] >> 16);
        }
    }
    const int ndig = 1 << db, half = (wave & 1) * 16;
    for (int p = 0; p < passes; ++p) {
        const int sh = p * db + (NARROW ? 16 : 0);
        uint32_t *cnt = counts + (p & 1) * count_words<NW>();
        uint32_t *spare = counts + ((p & 1) ^ 1) * count_words<NW>();
        uint32_t *mine = cnt + (wave >> 1) * kDigits;
        if (db == 6)
            radix_count<6, I, NARROW>(key, rank, sh, mine, half);
        else if (db == 7)
            radix_count<7, I, NARROW>(key, rank, sh, mine, half);
        else if constexpr (kMost == 8)
            radix_count<8, I, NARROW>(key, rank, sh, mine, half);
        __syncthreads();
        // counts -> first places: over the waves of a digit, then the digits
        const int t = (int)threadIdx.x;
        uint32_t at[NW / 2];
        uint32_t sum = 0;
        if (t < ndig) {
#pragma unroll
            for (int q = 0; q < NW / 2; ++q) {
                const uint32_t c = cnt[q * kDigits + t];
                at[q] = sum | ((sum + (c & 0xFFFFu)) << 16);
                sum += (c & 0xFFFFu) + (c >> 16);
            }
        }
        const uint32_t incl = wave_scan_incl(sum, lane);
        if (lane == 63)
            wave_total[wave] = incl;
        for (int k = t; k < count_words<NW>(); k += 64 * NW)
            spare[k] = 0u;  // the next pass's counts
        __syncthreads();
        if (t < ndig) {
            uint32_t base = incl - sum;
#pragma unroll
            for (int v = 0; v < kDigits / 64 - 1; ++v)
                base += v < wave ? wave_total[min(v, NW - 1)] : 0u;
#pragma unroll
            for (int q = 0; q < NW / 2; ++q)
                cnt[q * kDigits + t] = at[q] + base * 0x10001u;
        }
        __syncthreads();
        // (digits are taken from the keys again: kept, they and their
        // addresses would cost 2 I registers)
#pragma unroll
        for (int r = 0; r < I; ++r)
            asm volatile("" : "+v"(key[r]));
#pragma unroll
        for (int r = 0; r < I; ++r) {
            const uint32_t d = (key[r] >> sh) & (uint32_t)(ndig - 1);
            const uint32_t o = ((mine[d] >> half) & 0xFFFFu) + (rank[r] & 0xFFFFu);
            keys[o] = key[r];
            if constexpr (!NARROW)
                idx[o] = (uint16_t)(rank[r] >> 16);
        }
        if (p + 1 < passes) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < I; ++r) {
                key[r] = keys[first + 64 * r];
                if constexpr (!NARROW)
                    rank[r] = (uint32_t)idx[first + 64 * r] << 16;
            }
        }
    }
    __syncthreads();
}

// The first K sorted entries, four per thread (a row of the tables starts on
// a multiple of 64 entries), zeros up to the pitch.
template <int NW, bool NARROW>
__device__ __forceinline__ void emit_sorted(const uint32_t *keys, const uint16_t *idx, int K,
                                            int pitch, int64_t base, uint16_t *pi,
                                            int32_t *delta, int32_t *ds)
{
    for (int k = 4 * (int)threadIdx.x; k < pitch; k += 4 * 64 * NW) {
        const uint4 q = *reinterpret_cast<const uint4 *>(keys + k);
        const uint32_t x[5] = {k ? keys[k - 1] : 0u, q.x, q.y, q.z, q.w};
        ushort4 j = NARROW ? make_ushort4((uint16_t)q.x, (uint16_t)q.y, (uint16_t)q.z,
                                          (uint16_t)q.w)
                           : *reinterpret_cast<const ushort4 *>(idx + k);
        int32_t dist[5];
#pragma unroll
        for (int c = 0; c < 5; ++c)
            dist[c] = (int32_t)(NARROW ? x[c] >> 16 : x[c]);
        if (k + 4 > K) {  // the row's end
            j.x = k < K ? j.x : 0;
            j.y = k + 1 < K ? j.y : 0;
            j.z = k + 2 < K ? j.z : 0;
            j.w = 0;
        }
        int32_t v[4], g[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            v[c] = k + c < K ? dist[c + 1] : 0;
            g[c] = k + c < K ? dist[c + 1] - dist[c] : 0;
        }
        *reinterpret_cast<ushort4 *>(pi + base + k) = j;
        *reinterpret_cast<int4 *>(ds + base + k) = make_int4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<int4 *>(delta + base + k) = make_int4(g[0], g[1], g[2], g[3]);
    }
}

// Waves per SIMD the registers are held to.  More waves hide the barriers and
// the LDS round trips better than a few spilled values cost (4801 rows of
// 3333: 95 us at 6, 92 at 8; 5000 of 5000: 129 at 5, 121 at 6).
constexpr int radix_waves_per_simd(int NW, int I)
{
    return NW == 16 ? 4 : I <= 8 ? 8 : I <= 12 ? 6 : 4;
}

template <int NW, int I>
__global__ __launch_bounds__(64 * NW, radix_waves_per_simd(NW, I)) void k_radix_rows(const int32_t *__restrict__ d, int64_t ld,
                                                        int32_t m, int32_t K, int32_t pitch,
                                                        uint16_t *__restrict__ pi,
                                                        int32_t *__restrict__ delta,
                                                        int32_t *__restrict__ ds,
                                                        uint32_t *__restrict__ row_err,
                                                        unsigned long long *__restrict__ colsum,
                                                        uint32_t *__restrict__ nearc)
{
    extern __shared__ __align__(16) uint32_t lds_words[];
    __shared__ uint32_t wave_word[NW];
    uint32_t *counts = lds_words;                        // two sets
    uint32_t *keys = lds_words + 2 * count_words<NW>();  // NW I 64
    uint16_t *idx = reinterpret_cast<uint16_t *>(keys + NW * I * 64);
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int64_t i = blockIdx.x;
    const int32_t *row = d + i * ld;
    uint32_t key[I];
#pragma unroll
    for (int r = 0; r < I; ++r)  // every load at a valid address
        key[r] = (uint32_t)row[min((wave * I + r) * 64 + lane, m - 1)];
    for (int k = (int)threadIdx.x; k < 2 * count_words<NW>(); k += 64 * NW)
        counts[k] = 0u;
    uint32_t any = 0;
#pragma unroll
    for (int r = 0; r < I; ++r)
        any |= key[r];  // (a clamped load repeats a distance of the row)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        any |= (uint32_t)__shfl_xor((int)any, o);
    if (lane == 0)
        wave_word[wave] = any;
    __syncthreads();
    any = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v)
        any |= wave_word[v];
    any = __builtin_amdgcn_readfirstlane(any);
    __syncthreads();  // (wave_word is used again)
    const int bits = any ? 32 - __builtin_clz(any) : 0;
    if (threadIdx.x == 0)
        row_err[i] = any >> 31;  // a negative distance
    // this row's share of the sums that the next launch adds to
    for (int64_t j = i + (int64_t)gridDim.x * threadIdx.x; j < m;
         j += (int64_t)gridDim.x * 64 * NW) {
        colsum[j] = 0ull;
        nearc[j] = 0u;
    }
    // padding past m: the last keys of every pass's last digit
    if (bits <= 16) {
#pragma unroll
        for (int r = 0; r < I; ++r) {
            const int j = (wave * I + r) * 64 + lane;
            key[r] = j < m ? (key[r] << 16) | (uint32_t)j : ~0u;
        }
        radix_sort_row<NW, I, true>(key, bits, counts, wave_word, keys, idx);
        emit_sorted<NW, true>(keys, idx, K, pitch, i * pitch, pi, delta, ds);
    } else {
#pragma unroll
        for (int r = 0; r < I; ++r)
            key[r] = (wave * I + r) * 64 + lane < m ? key[r] : ~0u;
        radix_sort_row<NW, I, false>(key, bits, counts, wave_word, keys, idx);
        emit_sorted<NW, false>(keys, idx, K, pitch, i * pitch, pi, delta, ds);
    }
}

// ---------------------------------------------------------------------------
// Rows wider than kMaxLdsRow (m up to 65535): a bitonic network (Batcher,
// 1968) on the padded row (m2 64-bit keys distance << 16 | facility, a power
// of two of them), run in device memory.  Each row's keys live in a scratch array; chunks of
// kWideChunk keys are sorted in LDS by every stage of size <= kWideChunk
// (compare directions from the keys' global indices, as in the whole
// network); each larger size runs its strides >= kWideChunk as passes over
// the scratch (a thread per compare-exchange) and its smaller strides in LDS
// again, chunk by chunk.
// ---------------------------------------------------------------------------
constexpr int kWideChunk = PMP_MAX_FACILITIES;  // keys per LDS chunk (64 KB)

// Stages (size, stride) with size in [size_lo, size_hi] and stride < kWideChunk
// on the chunk at global index base (keys in LDS).
__device__ __forceinline__ void bitonic_chunk(uint64_t *key, int base, int size_lo, int size_hi)
{
    const int half = kWideChunk >> 1;
    for (int size = size_lo; size <= size_hi; size <<= 1) {
        for (int stride = min(size, kWideChunk) >> 1; stride > 0; stride >>= 1) {
            for (int t = threadIdx.x; t < half; t += kSortThreads) {
                const int lo = 2 * t - (t & (stride - 1));
                const int hi = lo + stride;
                const bool ascending = ((base + lo) & size) == 0;
                const uint64_t a = key[lo], b = key[hi];
                if ((a > b) == ascending) {
                    key[lo] = b;
                    key[hi] = a;
                }
            }
            __syncthreads();
        }
    }
}

// Load the keys of row blockIdx.y, chunk blockIdx.x (padding past m with
// all-ones keys; negative distances flagged), sort the chunk by every stage
// of size <= kWideChunk, store it to the row's scratch.
__global__ __launch_bounds__(kSortThreads) void k_wide_chunks(
    const int32_t *__restrict__ d, int64_t ld, int32_t row0, int32_t m, int32_t m2,
    uint64_t *__restrict__ scratch, uint32_t *__restrict__ err)
{
    extern __shared__ uint64_t lds_keys[];
    const int32_t i = row0 + (int32_t)blockIdx.y;
    const int base = (int)blockIdx.x * kWideChunk;
    const int32_t *row = d + (int64_t)i * ld;
    uint64_t *out = scratch + (int64_t)blockIdx.y * m2 + base;
    int negative = 0;
    for (int k = threadIdx.x; k < kWideChunk; k += kSortThreads) {
        const int j = base + k;
        uint64_t key = ~0ull;
        if (j < m) {
            const int32_t v = row[j];
            negative |= v < 0;
            key = ((uint64_t)(uint32_t)v << 16) | (uint64_t)j;
        }
        lds_keys[k] = key;
    }
    if (__syncthreads_or(negative) && threadIdx.x == 0)
        atomicOr(err, ERR_NEGATIVE_DISTANCE);
    bitonic_chunk(lds_keys, base, 2, kWideChunk);
    for (int k = threadIdx.x; k < kWideChunk; k += kSortThreads)
        out[k] = lds_keys[k];
}

// One stage (size, stride >= kWideChunk) of every row of the batch: a
// thread per compare-exchange.
__global__ void k_wide_step(uint64_t *__restrict__ scratch, int32_t m2, int32_t size,
                            int32_t stride)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int half = m2 >> 1;
    if (t >= half)
        return;
    uint64_t *key = scratch + (int64_t)blockIdx.y * m2;
    const int lo = 2 * (int)t - ((int)t & (stride - 1));
    const int hi = lo + stride;
    const bool ascending = (lo & size) == 0;
    const uint64_t a = key[lo], b = key[hi];
    if ((a > b) == ascending) {
        key[lo] = b;
        key[hi] = a;
    }
}

// The strides below kWideChunk of stage `size`, chunk by chunk in LDS.
__global__ __launch_bounds__(kSortThreads) void k_wide_local(uint64_t *__restrict__ scratch,
                                                            int32_t m2, int32_t size)
{
    extern __shared__ uint64_t lds_keys[];
    const int base = (int)blockIdx.x * kWideChunk;
    uint64_t *key = scratch + (int64_t)blockIdx.y * m2 + base;
    for (int k = threadIdx.x; k < kWideChunk; k += kSortThreads)
        lds_keys[k] = key[k];
    __syncthreads();
    const int half = kWideChunk >> 1;
    for (int stride = kWideChunk >> 1; stride > 0; stride >>= 1) {
        for (int t = threadIdx.x; t < half; t += kSortThreads) {
            const int lo = 2 * t - (t & (stride - 1));
            const int hi = lo + stride;
            const bool ascending = ((base + lo) & size) == 0;
            const uint64_t a = lds_keys[lo], b = lds_keys[hi];
            if ((a > b) == ascending) {
                lds_keys[lo] = b;
                lds_keys[hi] = a;
            }
        }
        __syncthreads();
    }
    for (int k = threadIdx.x; k < kWideChunk; k += kSortThreads)
        key[k] = lds_keys[k];
}

// Pi', Delta', D' of the batch's rows from their sorted keys.
__global__ __launch_bounds__(kSortThreads) void k_wide_emit(const uint64_t *__restrict__ scratch,
                                                           int32_t row0, int32_t m2, int32_t K,
                                                           int32_t pitch, uint16_t *pi,
                                                           int32_t *delta, int32_t *ds)
{
    const uint64_t *key = scratch + (int64_t)blockIdx.y * m2;
    const int64_t base = (int64_t)(row0 + (int32_t)blockIdx.y) * pitch;
    for (int k = (int)blockIdx.x * kSortThreads + threadIdx.x; k < pitch;
         k += (int)gridDim.x * kSortThreads) {
        uint16_t f = 0;
        int32_t dist = 0, gap = 0;
        if (k < K) {
            const uint64_t x = key[k];
            f = (uint16_t)(x & 0xFFFFu);
            dist = (int32_t)(x >> 16);
            gap = k == 0 ? dist : dist - (int32_t)(key[k - 1] >> 16);
        }
        pi[base + k] = f;
        ds[base + k] = dist;
        delta[base + k] = gap;
    }
}

__global__ void k_zero(uint32_t *p, size_t words)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < words;
         k += stride)
        p[k] = 0;
}

}  // namespace

int wide_sort_rows_per_batch(int32_t m)
{
    int32_t m2 = 2;
    while (m2 < m)
        m2 <<= 1;
    // about 256 MB of scratch keys per batch
    const int64_t rows = (256ll << 20) / ((int64_t)m2 * 8);
    return (int)std::max<int64_t>(1, std::min<int64_t>(rows, 65535));
}

hipError_t launch_sort_rows_wide(const int32_t *d, int64_t ld, int32_t n, int32_t m,
                                 int32_t K, int32_t pitch, uint16_t *pi, int32_t *delta,
                                 int32_t *ds, uint32_t *err, uint64_t *scratch, int32_t batch,
                                 hipStream_t s)
{
    int32_t m2 = 2;
    while (m2 < m)
        m2 <<= 1;
    const int chunks = m2 / kWideChunk;
    const size_t lds = sizeof(uint64_t) * kWideChunk;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_wide_chunks),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_wide_local),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess)
        return e;
    for (int32_t row0 = 0; row0 < n; row0 += batch) {
        const int32_t rows = std::min(batch, n - row0);
        hipLaunchKernelGGL(k_wide_chunks, dim3(chunks, rows), dim3(kSortThreads), lds, s, d, ld,
                           row0, m, m2, scratch, err);
        for (int size = 2 * kWideChunk; size <= m2; size <<= 1) {
            for (int stride = size >> 1; stride >= kWideChunk; stride >>= 1)
                hipLaunchKernelGGL(k_wide_step, dim3((m2 / 2 + 255) / 256, rows), dim3(256), 0,
                                   s, scratch, m2, size, stride);
            hipLaunchKernelGGL(k_wide_local, dim3(chunks, rows), dim3(kSortThreads), lds, s,
                               scratch, m2, size);
        }
        hipLaunchKernelGGL(k_wide_emit, dim3((pitch + kSortThreads - 1) / kSortThreads, rows),
                           dim3(kSortThreads), 0, s, scratch, row0, m2, K, pitch, pi, delta, ds);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

namespace {

template <int NW, int I>
hipError_t launch_radix(const int32_t *d, int64_t ld, int32_t n, int32_t m, int32_t K,
                        int32_t pitch, uint16_t *pi, int32_t *delta, int32_t *ds,
                        uint32_t *row_err, unsigned long long *colsum, uint32_t *nearc,
                        hipStream_t s)
{
    static_assert(NW * I * 64 <= 65535, "places are counted in 16 bits");
    const size_t lds = sizeof(uint32_t) * 2 * count_words<NW>() + 6 * (size_t)(NW * I * 64);
    static_assert(sizeof(uint32_t) * 2 * NW / 2 * kDigits + 6 * NW * I * 64 + 4 * NW <= 163840,
                  "more than a CU's LDS");
    if (lds > 65536) {
        const hipError_t e =
            hipFuncSetAttribute(reinterpret_cast<const void *>(k_radix_rows<NW, I>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL((k_radix_rows<NW, I>), dim3(n), dim3(64 * NW), lds, s, d, ld, m, K, pitch,
                       pi, delta, ds, row_err, colsum, nearc);
    return hipGetLastError();
}

}  // namespace

// m <= kMaxLdsRow.
hipError_t launch_sort_rows(const int32_t *d, int64_t ld, int32_t n, int32_t m,
                            int32_t K, int32_t pitch, uint16_t *pi,
                            int32_t *delta, int32_t *ds, uint32_t *row_err,
                            unsigned long long *colsum, uint32_t *nearc, hipStream_t s)
{
#define PMP_RADIX(NW, I)                                                                \
    if (m <= NW * I * 64)                                                               \
        return launch_radix<NW, I>(d, ld, n, m, K, pitch, pi, delta, ds, row_err, colsum,       \
                                   nearc, s);
    PMP_RADIX(2, 1)
    PMP_RADIX(2, 2)
    PMP_RADIX(4, 2)
    PMP_RADIX(4, 3)
    PMP_RADIX(4, 4)
    PMP_RADIX(4, 6)
    PMP_RADIX(4, 8)
    PMP_RADIX(8, 5)
    PMP_RADIX(8, 6)
    PMP_RADIX(8, 8)
    PMP_RADIX(8, 10)
    PMP_RADIX(8, 12)
    PMP_RADIX(8, 14)
    PMP_RADIX(8, 16)
    PMP_RADIX(16, 10)
    PMP_RADIX(16, 12)
    PMP_RADIX(16, 14)
    PMP_RADIX(16, 16)
    PMP_RADIX(16, 18)
    PMP_RADIX(16, 20)
    PMP_RADIX(16, 23)
#undef PMP_RADIX
    static_assert(kMaxLdsRow == 16 * 23 * 64, "the widest shape above");
    return hipErrorInvalidValue;
}

// Zero a device buffer with a kernel (safe inside stream capture).
hipError_t launch_zero(void *p, size_t bytes, hipStream_t s)
{
    if (bytes == 0)
        return hipSuccess;
    if (bytes % 4 != 0)
        return hipErrorInvalidValue;
    const size_t words = bytes / 4;
    size_t blocks = (words + 255) / 256;
    if (blocks > 1024)
        blocks = 1024;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, s,
                       (uint32_t *)p, words);
    return hipGetLastError();
}

}  // namespace pmp
