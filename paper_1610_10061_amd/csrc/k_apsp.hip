// All-pairs shortest paths by blocked Floyd-Warshall (Floyd, CACM 1962;
// the three-phase tiling of Venkataraman et al., JEA 2003): the step that
// turns a graph instance (edge weights) into the distance matrix d that
// preprocessing sorts.  Distances are uint32 in a padded work matrix with
// INF = 0x7FFFFFFF for "no path"; every finite distance stays below INF (the
// host checks (n - 1) * max weight < INF), so a + b never wraps in 32 bits
// and min(d_ij, a + b) never exceeds d_ij <= INF: an update is one add and
// one min.
//
// Per round kb (tile 64 x 64), two launches:
//  - k_fw_panels: every tile of row kb and column kb times the closed diagonal
//    tile G = (kb, kb): a row tile T becomes min over k of G[., k] + T[k, .],
//    a column tile min over k of T[., k] + G[k, .] (G has a zero diagonal, so
//    T itself is among the sums).  With G closed beforehand these are plain
//    min-plus products, no chain of 64 dependent steps;
//  - k_fw_rest: every other tile (i, j) takes min over k of
//    D(i, kb)[., k] + D(kb, j)[k, .], and the workgroup of the next round's
//    diagonal tile then closes it (the first round's is closed by k_fw_close).
// When every panel workgroup closed the diagonal itself and relaxed its tile
// step by step (128 barriers), a round's panels took 62 us whatever n; they
// take 5 us now, k_fw_rest at n = 2000 23 us (20 before it also closed the
// next diagonal, a chain of 16 barriers).  Whole calls, n = 900 / 2000 / 4096:
// 1.27 / 2.76 / 7.8 -> 0.39 / 0.91 / 3.6 ms.  Bound: at n = 4096 the VALU (an
// add and half a v_min3 per update: 19 of 26 T updates/s), at small n the
// chain panels -> tile -> closing, about 25 us a round.
#include "common.hpp"

namespace pmp {

namespace {

constexpr int kTile = 64;
constexpr uint32_t kInf = 0x7FFFFFFFu;

constexpr int kLd = kTile + 4;  // padded LDS row: 16-byte aligned, columns spread over the banks

__device__ __forceinline__ int64_t tile_row(int ld, int ti, int tj, int r)
{
    return (int64_t)(ti * kTile + r) * ld + tj * kTile;
}

// A 64 x 64 tile staged by 256 threads, as it is or transposed.
__device__ __forceinline__ void stage_tile(uint32_t (&s)[kTile][kLd], const uint32_t *D, int ld,
                                           int ti, int tj, bool transposed)
{
    uint4 q[4];
    const int r = (int)threadIdx.x >> 4, c = 4 * ((int)threadIdx.x & 15);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        q[k] = *reinterpret_cast<const uint4 *>(D + tile_row(ld, ti, tj, r + 16 * k) + c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = r + 16 * k;
        if (transposed) {
            s[c][row] = q[k].x;
            s[c + 1][row] = q[k].y;
            s[c + 2][row] = q[k].z;
            s[c + 3][row] = q[k].w;
        } else {
            *reinterpret_cast<uint4 *>(&s[row][c]) = q[k];
        }
    }
}

// Closes a tile over its own 64 vertices: wave v of 4 holds rows 16 v + r in
// v[r], lane = column.  Four vertices at a time: their rows' owner closes the
// four rows among themselves (register moves only), publishes them, and every
// wave relaxes its rows through them: with the four rows closed, a row's new
// values are the least of its old ones and of (its old entry at the vertex +
// the vertex's row), so the four sums of a row do not wait for each other.
// 16 barriers; 12 us against 29 us for 64 steps with a barrier each.
__device__ __forceinline__ void close_tile(uint32_t (&v)[16], uint32_t (&pub)[2][4][kTile])
{
    const int lane = threadIdx.x & 63, wave = wave_id();
    for (int owner = 0; owner < 4; ++owner) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int k0 = 16 * owner + 4 * g;  // first of the four vertices
            if (wave == owner) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r != k)
                            v[4 * g + r] =
                                min(v[4 * g + r],
                                    (uint32_t)__builtin_amdgcn_readlane((int)v[4 * g + r], k0 + k) +
                                        v[4 * g + k]);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    pub[g & 1][r][lane] = v[4 * g + r];
            }
            __syncthreads();
            uint32_t row[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                row[k] = pub[g & 1][k][lane];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                uint32_t x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    x[k] = (uint32_t)__builtin_amdgcn_readlane((int)v[r], k0 + k) + row[k];
                v[r] = min(min(min(min(v[r], x[0]), x[1]), x[2]), x[3]);  // two v_min3
            }
        }
    }
}

// The rounds of a call whose paths might not fit int32 (a weight above
// `most` = (INF - 1) / (n - 1)) leave the work matrix alone: the host has
// enqueued some or all of them when it learns that the call is refused.
__device__ __forceinline__ bool refused(const uint32_t *wmax, uint32_t most)
{
    return *wmax > most;
}

// Tile (kb, kb) closed; the largest weight goes to the host word for the
// caller's check.
__global__ __launch_bounds__(256) void k_fw_close(uint32_t *D, int ld, int kb,
                                                  const uint32_t *wmax, uint32_t most,
                                                  uint32_t *host_wmax)
{
    __shared__ uint32_t pub[2][4][kTile];
    const int lane = threadIdx.x & 63, wave = wave_id();
    if (threadIdx.x == 0)
        __hip_atomic_store(host_wmax, *wmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (refused(wmax, most))
        return;
    uint32_t v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
        v[r] = D[tile_row(ld, kb, kb, 16 * wave + r) + lane];
    close_tile(v, pub);
#pragma unroll
    for (int r = 0; r < 16; ++r)
        D[tile_row(ld, kb, kb, 16 * wave + r) + lane] = v[r];
}

// Phase 2 of round kb.  A workgroup takes a strip of 16 columns of a tile of
// row kb, or of 16 rows of a tile of column kb (strips depend on themselves
// and G only, so they are replaced in place): 8 (nb - 1) workgroups, four
// sums per step and thread.
__global__ __launch_bounds__(256) void k_fw_panels(uint32_t *D, int ld, int nb, int kb,
                                                   const uint32_t *__restrict__ wmax,
                                                   uint32_t most)
{
    __shared__ __attribute__((aligned(16))) uint32_t G[kTile][kLd];  // row strips: transposed
    __shared__ __attribute__((aligned(16))) uint32_t T[kTile][20];   // T[k][strip position]
    const int strips = 4 * (nb - 1);
    const bool row = (int)blockIdx.x < strips;
    const int x = row ? (int)blockIdx.x : (int)blockIdx.x - strips;
    const int o = x >> 2, q = x & 3, other = o < kb ? o : o + 1;
    const int t = (int)threadIdx.x;
    if (row) {  // columns 16 q .. of tile (kb, other)
        const int k = t >> 2, c = 4 * (t & 3);
        const uint4 e = *reinterpret_cast<const uint4 *>(D + tile_row(ld, kb, other, k) + 16 * q + c);
        *reinterpret_cast<uint4 *>(&T[k][c]) = e;
    } else {  // rows 16 q .. of tile (other, kb)
        const int r = t >> 4, k = 4 * (t & 15);
        const uint4 e = *reinterpret_cast<const uint4 *>(D + tile_row(ld, other, kb, 16 * q + r) + k);
        T[k][r] = e.x;
        T[k + 1][r] = e.y;
        T[k + 2][r] = e.z;
        T[k + 3][r] = e.w;
    }
    stage_tile(G, D, ld, kb, kb, row);
    if (refused(wmax, most))  // (read beside the tiles)
        return;
    __syncthreads();
    // 16 strip positions x 64: this thread's strip position and four others
    const int a = t >> 4, b = t & 15;
    const int pos = row ? b : a, quad = 4 * (row ? a : b);
    uint32_t acc[4] = {~0u, ~0u, ~0u, ~0u};
#pragma unroll 16
    for (int k = 0; k < kTile; ++k) {
        const uint32_t s = T[k][pos];
        const uint4 g = *reinterpret_cast<const uint4 *>(&G[k][quad]);
        acc[0] = min(acc[0], g.x + s);
        acc[1] = min(acc[1], g.y + s);
        acc[2] = min(acc[2], g.z + s);
        acc[3] = min(acc[3], g.w + s);
    }
    if (row) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            D[tile_row(ld, kb, other, quad + r) + 16 * q + pos] = acc[r];
    } else {
        *reinterpret_cast<uint4 *>(D + tile_row(ld, other, kb, 16 * q + pos) + quad) =
            make_uint4(acc[0], acc[1], acc[2], acc[3]);
    }
}

// Phase 3 of round kb: tile (i, j) off row and column kb.  The column-panel
// tile is staged transposed so each thread reads its 4 rows' entries of
// column k with one 16-byte LDS read, and the row-panel tile's 4 columns of
// row k likewise (4 x 4 sums per thread and step).  The workgroup of tile
// (kb + 1, kb + 1), the first dispatched, closes it afterwards: its waves run
// at a higher priority than the ones they share a CU with, so that its chain
// ends with the launch's other work and not after it.
__global__ __launch_bounds__(256) void k_fw_rest(uint32_t *D, int ld, int nb, int kb,
                                                 const uint32_t *__restrict__ wmax,
                                                 uint32_t most)
{
    __shared__ __attribute__((aligned(16))) uint32_t At[kTile][kLd];  // At[k][i] = D(i, kb)[i][k]
    __shared__ __attribute__((aligned(16))) uint32_t B[kTile][kLd];   // B[k][j] = D(kb, j)[k][j]
    __shared__ uint32_t pub[2][4][kTile];
    const int nrest = nb - 1;
    // tiles in order from (kb, kb) of the numbering that leaves out row and
    // column kb: that is tile (kb + 1, kb + 1) while there is one
    int x = (int)blockIdx.x + (kb < nrest ? kb * nrest + kb : 0);
    if (x >= nrest * nrest)
        x -= nrest * nrest;
    const int ii = x / nrest, jj = x - ii * nrest;
    const int ti = ii < kb ? ii : ii + 1, tj = jj < kb ? jj : jj + 1;
    const bool next_diag = ti == kb + 1 && tj == kb + 1;
    if (next_diag)
        __builtin_amdgcn_s_setprio(3);
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    uint32_t acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint4 v =
            *reinterpret_cast<const uint4 *>(D + tile_row(ld, ti, tj, 4 * ty + r) + 4 * tx);
        acc[r][0] = v.x;
        acc[r][1] = v.y;
        acc[r][2] = v.z;
        acc[r][3] = v.w;
    }
    stage_tile(At, D, ld, ti, kb, true);
    stage_tile(B, D, ld, kb, tj, false);
    if (refused(wmax, most))
        return;
    __syncthreads();
#pragma unroll 8
    for (int k = 0; k < kTile; ++k) {
        const uint4 a = *reinterpret_cast<const uint4 *>(&At[k][4 * ty]);
        const uint4 bb = *reinterpret_cast<const uint4 *>(&B[k][4 * tx]);
        const uint32_t av[4] = {a.x, a.y, a.z, a.w};
        const uint32_t bv[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[r][c] = min(acc[r][c], av[r] + bv[c]);
    }
    if (next_diag) {
        __syncthreads();  // (At is read no more)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<uint4 *>(&At[4 * ty + r][4 * tx]) =
                make_uint4(acc[r][0], acc[r][1], acc[r][2], acc[r][3]);
        __syncthreads();
        const int lane = threadIdx.x & 63, wave = wave_id();
        uint32_t v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
            v[r] = At[16 * wave + r][lane];
        close_tile(v, pub);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            D[tile_row(ld, ti, tj, 16 * wave + r) + lane] = v[r];
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *reinterpret_cast<uint4 *>(D + tile_row(ld, ti, tj, 4 * ty + r) + 4 * tx) =
            make_uint4(acc[r][0], acc[r][1], acc[r][2], acc[r][3]);
}

// Rows that a workgroup of k_fw_in and k_fw_out takes (256 columns each).
constexpr int kInRows = 16;

// Work matrix from the weights: INF where there is no edge (w < 0) and in the
// padding, 0 on the diagonal, and the largest weight into *wmax (one atomic
// per workgroup at most: one per wave kept 8192 of them on one address for
// 80 us at n = 2000).
__global__ __launch_bounds__(256) void k_fw_in(const int32_t *w, int64_t ldw, int n, uint32_t *D,
                                               int ld, uint32_t *wmax)
{
    __shared__ uint32_t part[4];
    const int j = (int)blockIdx.x * 256 + (int)threadIdx.x, i0 = (int)blockIdx.y * kInRows;
    uint32_t mx = 0;
    int32_t x[kInRows];
#pragma unroll
    for (int r = 0; r < kInRows; ++r)
        x[r] = w[(int64_t)min(i0 + r, n - 1) * ldw + min(j, n - 1)];
#pragma unroll
    for (int r = 0; r < kInRows; ++r) {
        const int i = i0 + r;
        uint32_t v = kInf;
        if (i < n && j < n && x[r] >= 0) {
            v = (uint32_t)x[r];
            mx = max(mx, v);
        }
        if (i == j)
            v = 0;
        if (i < ld && j < ld)
            D[(int64_t)i * ld + j] = v;
    }
#pragma unroll
    for (int dd = 32; dd > 0; dd >>= 1)
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, dd));
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = max(max(part[0], part[1]), max(part[2], part[3]));
        if (mx > __hip_atomic_load(wmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(wmax, mx);
    }
}

// Distances out: -1 for INF (no path).  Nothing is written when a path length
// might not fit.
__global__ __launch_bounds__(256) void k_fw_out(const uint32_t *D, int ld, int n, int32_t *d,
                                                int64_t ldd, const uint32_t *wmax,
                                                uint32_t most)
{
    if (refused(wmax, most))
        return;
    const int j = (int)blockIdx.x * 256 + (int)threadIdx.x, i0 = (int)blockIdx.y * kInRows;
    if (j >= n)
        return;
#pragma unroll
    for (int r = 0; r < kInRows; ++r) {
        const int i = i0 + r;
        if (i < n) {
            const uint32_t v = D[(int64_t)i * ld + j];
            d[(int64_t)i * ldd + j] = v >= kInf ? -1 : (int32_t)v;
        }
    }
}

}  // namespace

int apsp_padded(int n)
{
    return ((n + kTile - 1) / kTile) * kTile;
}

int apsp_rounds(int n)
{
    return apsp_padded(n) / kTile;
}

hipError_t launch_apsp_in(const int32_t *w, int64_t ldw, int n, uint32_t *D, uint32_t *wmax,
                          hipStream_t s)
{
    const int ld = apsp_padded(n);
    hipLaunchKernelGGL(k_fw_in, dim3((ld + 255) / 256, (ld + kInRows - 1) / kInRows), dim3(256), 0,
                       s, w, ldw, n, D, ld, wmax);
    return hipGetLastError();
}

uint32_t apsp_most_weight(int n)
{
    return n < 2 ? ~0u : (kInf - 1) / (uint32_t)(n - 1);
}

hipError_t launch_apsp_close(uint32_t *D, int n, const uint32_t *wmax, uint32_t *host_wmax,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_fw_close, dim3(1), dim3(256), 0, s, D, apsp_padded(n), 0, wmax,
                       apsp_most_weight(n), host_wmax);
    return hipGetLastError();
}

hipError_t launch_apsp_rounds(uint32_t *D, int n, int first, int last, const uint32_t *wmax,
                              hipStream_t s)
{
    const int ld = apsp_padded(n), nb = ld / kTile;
    const uint32_t most = apsp_most_weight(n);
    for (int kb = first; kb < last && nb > 1; ++kb) {
        hipLaunchKernelGGL(k_fw_panels, dim3(8 * (nb - 1)), dim3(256), 0, s, D, ld, nb, kb, wmax,
                           most);
        hipLaunchKernelGGL(k_fw_rest, dim3((nb - 1) * (nb - 1)), dim3(256), 0, s, D, ld, nb, kb,
                           wmax, most);
    }
    return hipGetLastError();
}

hipError_t launch_apsp_out(const uint32_t *D, int n, int32_t *d, int64_t ldd,
                           const uint32_t *wmax, hipStream_t s)
{
    const int ld = apsp_padded(n);
    hipLaunchKernelGGL(k_fw_out, dim3((n + 255) / 256, (n + kInRows - 1) / kInRows), dim3(256), 0,
                       s, D, ld, n, d, ldd, wmax, apsp_most_weight(n));
    return hipGetLastError();
}

}  // namespace pmp
