// Several Chebyshev products per launch on tiles of a sparse H (gfx950).
//
// A time step is 19 products with H.  One product per launch streams every
// vector through memory each time; here a workgroup owns a tile of rows of one
// vector and forms K consecutive products for it in one launch, with the rows
// within K hops of the tile (its closure) recomputed on chip: product j of K
// is formed for the rows within K - j hops.  p_m and p_m-1 of the closure live
// in two LDS buffers that take turns (p_m+1 replaces p_m-1, one barrier a
// product), H's rows (local columns, values) in registers for all K products,
// and the series sum c_m p_m of the tile's own rows in FP64 registers.  So a
// launch reads the closure's vectors once and writes the tile's once for K
// products, at the price of the closure's extra rows.
//
// What bounds it: memory first where the vectors stream from it (33.5M rows,
// complex128, 10 or 9 products a launch: 4.77 GB in 1.24 ms, 3.8 TB/s or 79% of a
// large copy's rate, with the LDS active 46% and the vector ALUs 36% of a CU's busy
// cycles), the wait for a closure's loads not being covered entirely by the CU's
// second workgroup; LDS bandwidth and issue rate (about one clock per CU for a row
// and product: W gathers, an old value and a store of 16 bytes) where they come
// from the last-level cache; and, where a sample has fewer tiles than the card
// takes at once (512), the latency of a launch: about 10 us for the closure's
// rows and H, waited for in turn, plus the products.
// Measured, against the term and pair kernels: graphene 2048^2, complex128, 16
// steps: 25.7 -> 10.5 ms; graphene 64^2 (one launch a step), 256 steps: 13.9 ->
// 3.6 ms; AB bilayer 1024x512, complex64, blocks of 16: 46.5 -> 31.4 ms; graphene
// 640x480 with 20% vacancies (CSR), complex128 blocks of 4: 11.0 -> 2.7 ms.
// Rows of 12 (third neighbours): five hops reach too far, and the staged term
// kernel stays.
//
// Plan (StepPlan): tiles of at most 1024 rows; per tile the closure's rows in
// order of hop distance (the tile's own first, each layer ascending), the
// number of rows within d hops for d <= depth, and 16-bit local columns of the
// rows within depth - 1 hops (as byte offsets into the closure's vector), and a
// byte per slot that selects its value: its value table index, or without a
// table its stored slot.  step_plan_kernel builds it on the device by
// breadth-first search from the stored ELL columns.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "tbpm_device.h"

namespace tbpm {

constexpr int SWG = 1024;                  // lanes per workgroup
constexpr int SP_CAP = STEP_CLOSURE;       // most rows of a closure the plan kernel takes
constexpr int SP_HASH = 16384;             // slots of its row -> local index table (LDS)

// ---- the plan ----------------------------------------------------------------------------

struct PlanArgs {
    const int32_t *col;                    // stored ELL columns [w][ld]
    int64_t ld;
    int32_t w, depth, cap, fill;
    const int32_t *tiles;                  // [tiles][2]: first row and count, in tile_rows
    const int32_t *tile_rows;              // the tiles' own rows
    int32_t *layer;                        // [tiles][depth + 1]: rows within d hops (0 at depth: more than cap)
    // fill: closures of tile i at entries clo_ptr[i] .. clo_ptr[i+1] - 1
    const int32_t *clo_ptr;
    int32_t *rows;
    uint64_t *lcol;                        // word q of entry e at q * lde + e
    uint32_t *vsel;                        // the same for value bytes, four a word
    int64_t lde;
    const uint32_t *vidx;                  // value table indexes of the rows, or null
    int32_t self;                          // move the slot of the row's own column to the end
    int32_t eshift;                        // log2 of a vector element's bytes: lcol holds byte offsets
};

__device__ __forceinline__ int plan_slot(const int32_t *keys, int32_t c)
{
    int h = (int)(((uint32_t)c * 2654435761u) >> 18);
    while (keys[h] != c)                   // c is in the table
        h = (h + 1) & (SP_HASH - 1);
    return h;
}

__global__ __launch_bounds__(SWG) void step_plan_kernel(PlanArgs a)
{
    __shared__ int32_t keys[SP_HASH];
    __shared__ uint16_t at[SP_HASH];
    __shared__ int32_t list[SP_CAP];
    __shared__ int count;
    const int t = threadIdx.x;
    const int tile = blockIdx.x;
    const int32_t *own = a.tile_rows + a.tiles[2 * tile];
    const int n0 = min(a.tiles[2 * tile + 1], SWG);
    for (int i = t; i < SP_HASH; i += SWG)
        keys[i] = -1;
    if (t == 0)
        count = n0;
    __syncthreads();
    // a new row's slot, or -1 when it is there already
    auto insert = [&](int32_t c) -> bool {
        int h = (int)(((uint32_t)c * 2654435761u) >> 18);
        for (int tries = 0; tries < SP_HASH; ++tries) {
            const int32_t old = atomicCAS(&keys[h], -1, c);
            if (old == -1)
                return true;
            if (old == c)
                return false;
            h = (h + 1) & (SP_HASH - 1);
        }
        return false;
    };
    if (t < n0) {
        list[t] = own[t];
        insert(own[t]);
    }
    __syncthreads();
    int32_t *layer = a.layer + (int64_t)tile * (a.depth + 1);
    if (t == 0)
        layer[0] = n0;
    int f0 = 0, f1 = n0;                    // the newest layer
    for (int d = 1; d <= a.depth; ++d) {
        for (int i = f0 + t; i < f1; i += SWG) {
            const int32_t r = list[i];
            for (int s = 0; s < a.w; ++s) {
                const int32_t c = a.col[(int64_t)s * a.ld + r];
                if (*(volatile int *)&count <= a.cap && insert(c)) {
                    const int p = atomicAdd(&count, 1);
                    if (p < SP_CAP)
                        list[p] = c;
                }
            }
        }
        __syncthreads();
        const int found = count;
        if (found > a.cap) {                // uniform
            if (t == 0)
                layer[a.depth] = 0;
            return;
        }
        // the layer in ascending row order: each row's rank among the layer's
        int32_t mine[SP_CAP / SWG];
        int rank[SP_CAP / SWG];
#pragma unroll
        for (int k = 0; k < SP_CAP / SWG; ++k) {
            const int i = f1 + t + k * SWG;
            rank[k] = 0;
            mine[k] = i < found ? list[i] : 0;
            if (i < found)
                for (int j = f1; j < found; ++j)
                    rank[k] += list[j] < mine[k] ? 1 : 0;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SP_CAP / SWG; ++k)
            if (f1 + t + k * SWG < found)
                list[f1 + rank[k]] = mine[k];
        __syncthreads();
        if (t == 0)
            layer[d] = found;
        f0 = f1;
        f1 = found;
    }
    if (!a.fill)
        return;
    for (int i = t; i < f1; i += SWG)
        at[plan_slot(keys, list[i])] = (uint16_t)i;
    __syncthreads();
    const int64_t e0 = a.clo_ptr[tile];
    const int inner = f0;                   // rows within depth - 1 hops
    for (int i = t; i < f1; i += SWG) {
        a.rows[e0 + i] = list[i];
        const int32_t r = list[i];
        int from = a.w;                     // the slot that goes last
        if (a.self)
            for (int s = a.w - 1; s >= 0; --s)
                from = a.col[(int64_t)s * a.ld + r] == r ? s : from;
        uint64_t word = 0;
        uint32_t sel = 0;
        for (int s = 0; s < a.w; ++s) {
            const int q = s == a.w - 1 && from < a.w ? from : s < from ? s : s + 1;     // the stored slot
            const uint64_t l = i < inner ? at[plan_slot(keys, a.col[(int64_t)q * a.ld + r])] : 0;
            const uint32_t k = a.vidx ? (a.vidx[(int64_t)(q / 4) * a.ld + r] >> (8 * (q % 4))) & 255u : (uint32_t)q;
            word |= (l << a.eshift) << (16 * (s % 4));
            sel |= k << (8 * (s % 4));
            if (s % 4 == 3 || s == a.w - 1) {
                a.lcol[(int64_t)(s / 4) * a.lde + e0 + i] = word;
                a.vsel[(int64_t)(s / 4) * a.lde + e0 + i] = sel;
                word = 0;
                sel = 0;
            }
        }
    }
}

// Cuts a tile in two: its rows (a range of tile_rows) are put in breadth-first
// order, piece after piece, and *cut is half of them, or the end of a piece
// that lies nearer to half than a quarter.  Both parts are left ascending.
__global__ __launch_bounds__(SWG) void step_split_kernel(const int32_t *col, int64_t ld, int32_t w,
                                                         const int32_t *tiles, int32_t *tile_rows, int32_t *cuts)
{
    constexpr int HS = 4096;
    __shared__ int32_t keys[HS];            // row -> its place below
    __shared__ int16_t at[HS];
    __shared__ int32_t rows[SWG];
    __shared__ int16_t order[SWG];          // breadth-first
    __shared__ int32_t seen[SWG];
    __shared__ int count, seed, cut;
    const int t = threadIdx.x;
    int32_t *own = tile_rows + tiles[2 * blockIdx.x];
    const int m = min(tiles[2 * blockIdx.x + 1], SWG);
    for (int i = t; i < HS; i += SWG)
        keys[i] = -1;
    if (t < m)
        rows[t] = own[t];
    seen[t] = 0;
    if (t == 0) {
        count = 0;
        cut = 0;
    }
    __syncthreads();
    if (t < m) {
        int h = (int)(((uint32_t)rows[t] * 2654435761u) >> 20);
        while (atomicCAS(&keys[h], -1, rows[t]) != -1)      // the rows are distinct, and fewer than slots
            h = (h + 1) & (HS - 1);
        at[h] = (int16_t)t;
    }
    __syncthreads();
    int f0 = 0, f1 = 0;                     // the newest layer in order
    while (f1 < m) {
        if (f0 == f1) {                     // a piece is complete: go on from the lowest row not seen
            if (t == 0) {
                if (4 * f1 >= m && 4 * f1 <= 3 * m && (cut == 0 || abs(2 * f1 - m) < abs(2 * cut - m)))
                    cut = f1;
                seed = SWG;
            }
            __syncthreads();
            if (t < m && !seen[t])
                atomicMin(&seed, t);
            __syncthreads();
            if (t == 0) {
                order[f1] = (int16_t)seed;
                seen[seed] = 1;
                count = f1 + 1;
            }
            __syncthreads();
            f1 = f1 + 1;
        }
        const int i = f0 + t;
        if (i < f1) {
            const int32_t r = rows[order[i]];
            for (int s = 0; s < w; ++s) {
                const int32_t c = col[(int64_t)s * ld + r];
                int h = (int)(((uint32_t)c * 2654435761u) >> 20);
                while (keys[h] != c && keys[h] != -1)
                    h = (h + 1) & (HS - 1);
                if (keys[h] == c && atomicExch(&seen[at[h]], 1) == 0)
                    order[atomicAdd(&count, 1)] = at[h];
            }
        }
        __syncthreads();
        const int found = count;
        // the layer in ascending order, so that the result does not depend on timing
        int16_t mine = 0;
        int rank = 0;
        if (f1 + t < found) {
            mine = order[f1 + t];
            for (int j = f1; j < found; ++j)
                rank += order[j] < mine ? 1 : 0;
        }
        __syncthreads();
        if (f1 + t < found)
            order[f1 + rank] = mine;
        __syncthreads();
        f0 = f1;
        f1 = found;
    }
    const int half = cut > 0 ? cut : (m + 1) / 2;
    if (t < m) {
        const int b = t < half ? 0 : half, e = t < half ? half : m;
        int rank = 0;
        for (int j = b; j < e; ++j)
            rank += order[j] < order[t] ? 1 : 0;
        own[b + rank] = rows[order[t]];     // rows[] is ascending
    }
    if (t == 0)
        cuts[blockIdx.x] = half;
}

__global__ __launch_bounds__(WG) void iota_kernel(int32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x; i < n; i += (int64_t)gridDim.x * WG)
        p[i] = (int32_t)i;
}

// what the stored ELL allows: *flag |= 1 when some value has an imaginary part
// other than +-0, |= 2 when some row has no slot in its own column
template <typename T>
__global__ __launch_bounds__(WG) void step_facts_kernel(const int32_t *col, const T *val, int64_t n, int64_t ld,
                                                        int32_t w, int32_t *flag)
{
    int f = 0;
    for (int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x; i < n; i += (int64_t)gridDim.x * WG) {
        bool own = false;
        for (int s = 0; s < w; ++s) {
            f |= val[(int64_t)s * ld + i].y != 0 ? 1 : 0;
            own = own || col[(int64_t)s * ld + i] == i;
        }
        f |= own ? 0 : 2;
    }
    f |= __shfl_xor(f, 32, 64);
    f |= __shfl_xor(f, 16, 64);
    f |= __shfl_xor(f, 8, 64);
    f |= __shfl_xor(f, 4, 64);
    f |= __shfl_xor(f, 2, 64);
    f |= __shfl_xor(f, 1, 64);
    if (threadIdx.x % 64 == 0 && f)
        atomicOr(flag, f);
}

// ---- the products ------------------------------------------------------------------------

constexpr int STW = 512;                   // lanes per workgroup: two workgroups a CU cover each other's loads
constexpr int STW_OWN = 1024 / STW;        // rows of the tile per lane

// Closure rows per lane: H's columns and values of a lane's rows, and their
// p_m and p_m-1, take at most 92 (complex64: 84, its rows need more besides) of
// the 128 registers that two workgroups leave, beyond which some row lengths
// spill; two buffers of the closure's rows take at most half the LDS.  (The series
// spills for none.  The moments, whose sums need registers too, spill 92, 138 and
// 50 registers for complex128 rows of 3, of 4 without and of 5 with the own
// column, real values, and 2 for complex64 rows of 4 with complex ones.)
template <typename T, int W, bool REAL>
constexpr int step_rows()
{
    const int regs = 2 * ((W + 3) / 4) + W * (int)sizeof(T) / (REAL ? 8 : 4) + (int)sizeof(T) / 2;
    const int k = (sizeof(T) == 16 ? 92 : 84) / regs;
    const int most = sizeof(T) == 8 ? 6 : REAL ? 5 : 3;
    return k > most ? most : k < 2 ? 0 : k;        // 0: not compiled (a tile's 1024 rows take two)
}

// Closure rows of a tile: the lanes' registers, and two workgroups a CU: half of
// the 160 KiB, the table's and the sums' 4 KiB apart, holds two vectors of them
template <typename T, int W, bool REAL>
constexpr int step_closure()
{
    const int fit = (81920 - 4096 - 4096) / (2 * (int)sizeof(T));
    const int k = step_rows<T, W, REAL>() * STW;
    const int most = k < fit ? k : fit;
    return most < SP_CAP ? most : SP_CAP;
}

// Sums of three values over a wave: lane l returns that of value l / 16 (0 for
// l >= 48).  Halves, then rows of 16 lanes, trade places so that one addition
// serves two values, and rotations finish each row: 25 instructions, where three
// sums by shuffles take 54 and the LDS crossbar.
__device__ __forceinline__ double swap_add(double x, double y, bool halves)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x), v = (uint64_t)__double_as_longlong(y);
    uint32_t r[2][2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t p = (uint32_t)(u >> (32 * q)), s = (uint32_t)(v >> (32 * q));
        const auto w = halves ? __builtin_amdgcn_permlane32_swap(p, s, false, false)
                              : __builtin_amdgcn_permlane16_swap(p, s, false, false);
        r[0][q] = w[0];
        r[1][q] = w[1];
    }
    return __longlong_as_double((long long)(((uint64_t)r[0][1] << 32) | r[0][0])) +
           __longlong_as_double((long long)(((uint64_t)r[1][1] << 32) | r[1][0]));
}
template <int CTRL>
__device__ __forceinline__ double row_rotate_add(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
    return x + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum3(double s0, double s1, double s2)
{
    // rows of 16: (0, 1, 2, 3) hold parts of s0, s1, s2 and nothing
    double x = swap_add(s0, s2, true);              // halves: s0, s2
    double y = swap_add(s1, 0.0, true);             // halves: s1, 0
    x = swap_add(x, y, false);                      // rows: s0, s1, s2, 0
    x = row_rotate_add<0x128>(x);                   // row_ror 8, 4, 2, 1
    x = row_rotate_add<0x124>(x);
    x = row_rotate_add<0x122>(x);
    return row_rotate_add<0x121>(x);
}

// SELF: the plan has every row's entry in its own column (or a padding slot) in
// its last slot, which reads the lane's register instead of LDS
template <typename T, int W, bool REAL, bool SELF, bool MOM>
__global__ __launch_bounds__(STW) __attribute__((amdgpu_waves_per_eu(4))) void step_kernel(StepArgs a)
{
    using E = Elem<T>;
    using Re = decltype(T{}.x);
    using V = typename std::conditional<REAL, Re, T>::type;
    using A = typename E::acc;
    constexpr int KR = step_rows<T, W, REAL>();
    constexpr int NW = (W + 3) / 4;
    constexpr int G = SELF ? W - 1 : W;             // slots gathered from LDS
    extern __shared__ __attribute__((aligned(16))) char step_lds[];
    // p_m of the closure and p_m+1, by turns
    constexpr int PB = step_closure<T, W, REAL>();
    T *const pa = reinterpret_cast<T *>(step_lds);
    T *const pb = pa + PB;
    V *vtab = reinterpret_cast<V *>(pb + PB);       // value table
    // sums of the waves: <psi0|out>, <out|out>; MOM: <p|p'>, <p|p> of every product
    __shared__ double red[MOM ? STEP_DEPTH : 1][STW / 64][3];

    const int64_t per = (a.ntiles + NXCD - 1) / NXCD;
    const int64_t u = blockIdx.x / NXCD;
    const int64_t tile = (int64_t)(blockIdx.x % NXCD) * per + u / a.B;
    const int b = (int)(u % a.B);
    if (u / a.B >= per || tile >= a.ntiles)
        return;                                     // uniform over the workgroup
    const int64_t e0 = a.clo_ptr[tile];
    const int32_t *__restrict__ layer = a.layer + tile * (a.depth + 1);
    const int K = a.count;                          // products of this launch (<= depth)
    const int n0 = min(layer[0], STW * STW_OWN);
    const int nk = min(layer[K], min(KR * STW, a.max_rows));
    int lim = layer[K - 1];
    const int t = threadIdx.x;
    const int64_t shift = (int64_t)b * a.stride;    // the block's vectors lie one after another
    const T *__restrict__ x = static_cast<const T *>(a.x) + shift;
    const T *__restrict__ y = static_cast<const T *>(a.y) + shift;
    const bool cont = a.y != nullptr;               // p_m-1 and the series so far exist

    // H's local columns, value bytes and the rows of the lane's entries t, t + STW, ...
    int32_t row[KR];
    uint32_t cw[KR][2 * NW];                        // two 16-bit columns a word
    uint32_t vw[KR][NW];
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const int e = t + k * STW;
        row[k] = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q)
            vw[k][q] = cw[k][2 * q] = cw[k][2 * q + 1] = 0;
        if (e < nk) {
            row[k] = a.rows[e0 + e];
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                const uint64_t w = a.lcol[(int64_t)q * a.lde + e0 + e];
                cw[k][2 * q] = (uint32_t)w;
                cw[k][2 * q + 1] = (uint32_t)(w >> 32);
                vw[k][q] = a.vsel[(int64_t)q * a.lde + e0 + e];
            }
        }
    }
    const bool table = a.vtab != nullptr;
    if (table) {
        for (int i = t; i < a.table_size; i += STW) {
            const T h = static_cast<const T *>(a.vtab)[i];
            if constexpr (REAL)
                vtab[i] = h.x;
            else
                vtab[i] = h;
        }
        __syncthreads();
    }
    // vectors and diagonals of every row first, so that they are waited for
    // together; then the values, row by row
    V v[KR][W];
    T own[KR], old[KR];                             // p_m and p_m-1 of the lane's rows
    V dg[SELF ? 1 : KR];                            // the row's diagonal (SELF: in its place, v[k][W - 1])
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        own[k] = old[k] = T{};
        V &diag = SELF ? v[k][W - 1] : dg[SELF ? 0 : k];
        diag = V{};
        if (t + k * STW < nk) {
            own[k] = x[row[k]];
            if (cont)
                old[k] = y[row[k]];
            if (table && a.vdiag) {
                const T h = diag_value(static_cast<const T *>(a.vdiag), a.vdiag_real, row[k]);
                if constexpr (REAL)
                    diag = h.x;
                else
                    diag = h;
            }
        }
    }
    if (table) {
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < W; ++s) {
                const uint32_t i = (vw[k][s / 4] >> (8 * (s % 4))) & 255u;
                const V h = vtab[min(i, (uint32_t)a.table_size - 1u)];
                if (SELF && s == W - 1)             // the one slot that can be the diagonal
                    v[k][s] = i == 255u ? v[k][s] : h;
                else
                    v[k][s] = !SELF && i == 255u ? dg[SELF ? 0 : k] : h;
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < W; ++s) {
                if (s % 2 == 0)
                    __builtin_amdgcn_sched_barrier(0);
                const uint32_t i = (vw[k][s / 4] >> (8 * (s % 4))) & 255u;
                asm("" : "+v"(row[k]));             // (addresses formed anew rather than kept)
                const int64_t at = (int64_t)i * a.ld + row[k];
                if constexpr (REAL)
                    v[k][s] = static_cast<const Re *>(a.val)[2 * at];
                else
                    v[k][s] = static_cast<const T *>(a.val)[at];
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < KR; ++k)
        if (t + k * STW < nk)
            pa[t + k * STW] = own[k];
#pragma unroll
    for (int k = 0; k < STW_OWN; ++k)
        asm("" : "+v"(row[k]));
    // the series of the tile's own rows: this launch's terms
    d2 o[STW_OWN];
#pragma unroll
    for (int k = 0; k < STW_OWN; ++k) {
        o[k] = d2{0.0, 0.0};
        if (!MOM && !cont)
            o[k] = cmul(d2{a.c[0][0], a.c[0][1]}, E::to_d(own[k]));
    }
    __syncthreads();

    // product j: from cur (p_m; its closure at `from`) and prev (p_m-1) to prev
    // and `to`.  Written out for both roles of the two, so that no register is
    // copied and either buffer's place in LDS is an instruction's constant. (Rolled,
    // with local indexes instead of byte offsets: 12 of 43 vector instructions a
    // row more, 3 to 6% slower, and the longer rows spilled.)
    auto product = [&](int j, const T *from, T *to, T (&cur)[KR], T (&prev)[KR]) __attribute__((always_inline)) {
        const int next = j < K ? layer[K - j - 1] : 0;
        const double scale = (!cont && j == 1) ? a.scale1 : a.scale;
        const d2 c{a.c[j][0], a.c[j][1]};
        double m0 = 0.0, m1 = 0.0, m2 = 0.0;
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            const int e = t + k * STW;
            if (k * STW < lim) {                    // uniform
                if (e < lim) {
                    // the columns stay packed: without this the compiler unpacks
                    // every one of them before the loop and runs out of registers
#pragma unroll
                    for (int q = 0; q < (G + 1) / 2; ++q)
                        asm("" : "+v"(cw[k][q]));
                    A acc{0, 0};
                    if constexpr (SELF) {
                        if constexpr (REAL)
                            acc = A{v[k][W - 1] * cur[k].x, v[k][W - 1] * cur[k].y};
                        else
                            cmac(acc, (A)v[k][W - 1], (A)cur[k]);
                    }
#pragma unroll
                    for (int s = 0; s < G; ++s) {
                        const uint32_t at = (cw[k][s / 2] >> (16 * (s % 2))) & 0xFFFFu;
                        const T xv = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(from) + at);
                        if constexpr (REAL) {
                            acc.x += v[k][s] * xv.x;
                            acc.y += v[k][s] * xv.y;
                        } else {
                            cmac(acc, (A)v[k][s], (A)xv);
                        }
                    }
                    const d2 pn = E::acc_to_d(acc) * scale - E::to_d(prev[k]);
                    prev[k] = E::from_d(pn);
                    to[e] = prev[k];
                    if (k < STW_OWN && e < n0) {
                        if constexpr (MOM) {        // p in cur, p' in prev, as stored
                            const d2 xd = E::to_d(cur[k]), yd = E::to_d(prev[k]);
                            m0 += xd.x * yd.x + xd.y * yd.y;
                            m1 += xd.x * yd.y - xd.y * yd.x;
                            m2 += xd.x * xd.x + xd.y * xd.y;
                        } else {
                            o[k < STW_OWN ? k : 0] += cmul(c, pn);
                        }
                    }
                }
            }
        }
        lim = next;
        if constexpr (MOM) {
            const double m = wave_sum3(m0, m1, m2);
            if (t % 16 == 0 && (t & 48) != 48)
                red[j - 1][t / 64][(t & 63) / 16] = m;
        }
        __syncthreads();                            // p_m+1 complete; every read of p_m done
    };
    int j = 1;
    for (; j < K; j += 2) {
        product(j, pa, pb, own, old);
        product(j + 1, pb, pa, old, own);
    }
    if (j == K) {
        product(j, pa, pb, own, old);
#pragma unroll
        for (int k = 0; k < STW_OWN; ++k) {         // the newest in own
            const T q = own[k];
            own[k] = old[k];
            old[k] = q;
        }
    }

    if constexpr (MOM) {
        // (every wave's sums are in: the last product ended in a barrier)
#pragma unroll
        for (int k = 0; k < STW_OWN; ++k)
            if (a.xout && t + k * STW < n0) {
                static_cast<T *>(a.xout)[shift + row[k]] = own[k];
                static_cast<T *>(a.yout)[shift + row[k]] = old[k];
            }
        if (t < 3 * K) {
            double s = 0.0;
            for (int w = 0; w < STW / 64; ++w)
                s += red[t / 3][w][t % 3];
            a.partials[(int64_t)(t / 3) * a.mom_stride + (tile * a.B + b) * 4 + t % 3] = s;
        }
        return;
    }
    T so[STW_OWN], p0[STW_OWN];                     // the series before this launch, psi0
#pragma unroll
    for (int k = 0; k < STW_OWN; ++k) {
        so[k] = p0[k] = T{};
        if (t + k * STW < n0) {
            if (cont)
                so[k] = static_cast<const T *>(a.out)[shift + row[k]];
            if (a.psi0)
                p0[k] = static_cast<const T *>(a.psi0)[shift + row[k]];
        }
    }
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;            // <psi0|out>, <out|out> of the tile
#pragma unroll
    for (int k = 0; k < STW_OWN; ++k) {
        if (t + k * STW < n0) {
            const int64_t at = shift + row[k];
            const T os = E::from_d(E::to_d(so[k]) + o[k]);
            static_cast<T *>(a.out)[at] = os;
            if (a.xout) {                           // the next launch goes on from p_m+K, p_m+K-1
                static_cast<T *>(a.xout)[at] = own[k];
                static_cast<T *>(a.yout)[at] = old[k];
            }
            if (a.psi0) {
                const d2 p = E::to_d(p0[k]);
                const d2 od = E::to_d(os);
                s0 += p.x * od.x + p.y * od.y;
                s1 += p.x * od.y - p.y * od.x;
                s2 += od.x * od.x + od.y * od.y;
            }
        }
    }
    if (a.psi0) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            s0 += __shfl_xor(s0, off, 64);
            s1 += __shfl_xor(s1, off, 64);
            s2 += __shfl_xor(s2, off, 64);
        }
        if (t % 64 == 0) {
            red[0][t / 64][0] = s0;
            red[0][t / 64][1] = s1;
            red[0][t / 64][2] = s2;
        }
        __syncthreads();
        if (t < 3) {
            double s = 0.0;
            for (int w = 0; w < STW / 64; ++w)
                s += red[0][w][t];
            a.partials[(tile * a.B + b) * 4 + t] = s;
        }
    }
}

// ---- host ----------------------------------------------------------------------------------

template <typename T, bool REAL>
static int rows_of(int w)
{
    switch (w) {
    case 3: return step_closure<T, 3, REAL>();
    case 4: return step_closure<T, 4, REAL>();
    case 5: return step_closure<T, 5, REAL>();
    case 8: return step_closure<T, 8, REAL>();
    case 12: return step_closure<T, 12, REAL>();
    default: return 0;
    }
}

int step_closure_max(int dtype, int w, bool real)
{
    if (dtype == TBPM_C128)
        return real ? rows_of<d2, true>(w) : rows_of<d2, false>(w);
    return real ? rows_of<f2, true>(w) : rows_of<f2, false>(w);
}

template <typename T, int W, bool REAL, bool SELF>
static hipError_t launch_w(const StepArgs &a, hipStream_t st)
{
    if constexpr (step_rows<T, W, REAL>() == 0) {
        return hipErrorInvalidValue;
    } else {
        const int64_t per = (a.ntiles + NXCD - 1) / NXCD;
        const size_t lds = (2 * (size_t)step_closure<T, W, REAL>() + (size_t)a.table_size) * sizeof(T);
        const dim3 grid((unsigned)(per * NXCD * a.B));
        if (a.moments)
            hipLaunchKernelGGL((step_kernel<T, W, REAL, SELF, true>), grid, dim3(STW), lds, st, a);
        else
            hipLaunchKernelGGL((step_kernel<T, W, REAL, SELF, false>), grid, dim3(STW), lds, st, a);
        return hipGetLastError();
    }
}

template <typename T, bool REAL>
static hipError_t launch_t(const StepArgs &a, hipStream_t st)
{
    switch (a.w) {
    case 3: return launch_w<T, 3, REAL, false>(a, st);
    case 4: return a.self ? launch_w<T, 4, REAL, true>(a, st) : launch_w<T, 4, REAL, false>(a, st);
    case 5: return a.self ? launch_w<T, 5, REAL, true>(a, st) : launch_w<T, 5, REAL, false>(a, st);
    case 8: return launch_w<T, 8, REAL, false>(a, st);
    case 12: return launch_w<T, 12, REAL, false>(a, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_steps(int dtype, bool real, const StepArgs &a, hipStream_t st)
{
    if (a.ntiles <= 0 || a.B < 1 || a.count < 1 || a.count > a.depth || a.depth > STEP_DEPTH || !a.rows ||
        !a.lcol || !a.vsel || !a.layer || !a.x || (a.moments ? !a.partials || a.psi0 || a.mom_stride < a.ntiles * (int64_t)a.B * 4 : !a.out) ||
        a.max_rows < 1 || a.max_rows > step_closure_max(dtype, a.w, real) ||
        (a.xout && !a.yout) || (a.psi0 && !a.partials) || a.table_size < 0 || a.table_size > 256 ||
        (a.vtab ? a.table_size < 1 : !a.val))
        return hipErrorInvalidValue;
    if (dtype == TBPM_C128)
        return real ? launch_t<d2, true>(a, st) : launch_t<d2, false>(a, st);
    return real ? launch_t<f2, true>(a, st) : launch_t<f2, false>(a, st);
}

hipError_t launch_step_plan(const int32_t *col, int64_t ld, int w, int depth, int cap, int tiles,
                            const int32_t *tile, const int32_t *tile_rows, int32_t *layer,
                            const int32_t *clo_ptr, int32_t *rows, uint64_t *lcol, uint32_t *vsel, int64_t lde,
                            const uint32_t *vidx, bool self, int dtype, hipStream_t st)
{
    if (tiles <= 0 || depth < 1 || depth > STEP_DEPTH || cap < SWG || cap > SP_CAP || w < 1)
        return hipErrorInvalidValue;
    PlanArgs a{col, ld, w, depth, cap, rows ? 1 : 0, tile, tile_rows, layer, clo_ptr, rows, lcol, vsel, lde, vidx,
               self ? 1 : 0, dtype == TBPM_C128 ? 4 : 3};
    hipLaunchKernelGGL(step_plan_kernel, dim3(tiles), dim3(SWG), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_step_split(const int32_t *col, int64_t ld, int w, int tiles, const int32_t *tile, int32_t *tile_rows,
                             int32_t *cuts, hipStream_t st)
{
    if (tiles <= 0 || w < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(step_split_kernel, dim3(tiles), dim3(SWG), 0, st, col, ld, w, tile, tile_rows, cuts);
    return hipGetLastError();
}

hipError_t launch_iota(int32_t *p, int64_t n, hipStream_t st)
{
    hipLaunchKernelGGL(iota_kernel, dim3(std::min(elem_grid(n), 4096)), dim3(WG), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_step_facts(int dtype, const int32_t *col, const void *val, int64_t n, int64_t ld, int w,
                             int32_t *flag, hipStream_t st)
{
    const int g = std::min(elem_grid(n), 2048);
    if (dtype == TBPM_C128)
        hipLaunchKernelGGL(step_facts_kernel<d2>, dim3(g), dim3(WG), 0, st, col, (const d2 *)val, n, ld, w, flag);
    else
        hipLaunchKernelGGL(step_facts_kernel<f2>, dim3(g), dim3(WG), 0, st, col, (const f2 *)val, n, ld, w, flag);
    return hipGetLastError();
}

}  // namespace tbpm
