// Plans for several products with H per launch (tbpm_steps.hip): which rows
// form a tile, and the closure of each tile to a number of hops.
//
// Tiles are compact regions of the sparsity graph of at most 1024 rows: the
// patches of a patch-reordered H, or (plain ELL) regions grown by breadth-first
// search here.  A tile whose closure is too large for the kernel (patches of
// several pieces, above all) is cut into its connected pieces, or in half.
// The closures themselves are built on the device.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "tbpm_internal.h"

namespace tbpm {

namespace {

struct Tiles {
    std::vector<int32_t> ptr{0}, rows;
    int64_t count() const { return (int64_t)ptr.size() - 1; }
    void close() { ptr.push_back((int32_t)rows.size()); }
};

// the stored ELL columns, in host memory
struct Columns {
    std::vector<int32_t> c;
    int64_t ld = 0;
    int w = 0;
};

// breadth-first regions of at most `most` rows, one connected piece each
void grow_tiles(const Columns &h, int64_t n, int most, Tiles &out)
{
    std::vector<uint8_t> taken((size_t)n, 0);
    std::vector<int32_t> queue;
    int64_t low = 0;
    int32_t seed = -1;                      // an untaken neighbour of the previous tile
    while ((int64_t)out.rows.size() < n) {
        if (seed < 0 || taken[(size_t)seed]) {
            while (taken[(size_t)low])
                ++low;
            seed = (int32_t)low;
        }
        queue.assign(1, seed);
        taken[(size_t)seed] = 1;
        seed = -1;
        for (size_t i = 0; i < queue.size(); ++i)
            for (int s = 0; s < h.w; ++s) {
                const int32_t u = h.c[(size_t)(s * h.ld + queue[i])];
                if (taken[(size_t)u])
                    continue;
                if ((int)queue.size() >= most) {
                    if (seed < 0)
                        seed = u;
                    continue;
                }
                taken[(size_t)u] = 1;
                queue.push_back(u);
            }
        std::sort(queue.begin(), queue.end());
        out.rows.insert(out.rows.end(), queue.begin(), queue.end());
        out.close();
    }
}

// cuts rows[0..m) in two: its connected pieces in two groups of about equal
// size, or a single piece in halves of breadth-first order
void split_tile(const Columns &h, const int32_t *rows, int m, Tiles &out)
{
    auto find = [&](int32_t r) -> int {     // rows are ascending
        const int32_t *p = std::lower_bound(rows, rows + m, r);
        return p != rows + m && *p == r ? (int)(p - rows) : -1;
    };
    std::vector<uint8_t> taken((size_t)m, 0);
    std::vector<int> queue;                 // piece after piece
    size_t cut = 0;                         // end of the first group of pieces
    for (int i0 = 0; i0 < m; ++i0) {
        if (taken[(size_t)i0])
            continue;
        if (cut == 0 && 2 * queue.size() >= (size_t)m)
            cut = queue.size();
        size_t i = queue.size();
        queue.push_back(i0);
        taken[(size_t)i0] = 1;
        for (; i < queue.size(); ++i)
            for (int s = 0; s < h.w; ++s) {
                const int j = find(h.c[(size_t)(s * h.ld + rows[queue[i]])]);
                if (j >= 0 && !taken[(size_t)j]) {
                    taken[(size_t)j] = 1;
                    queue.push_back(j);
                }
            }
    }
    if (cut == 0)
        cut = (size_t)(m + 1) / 2;
    for (size_t b = 0, e = cut; b < (size_t)m; b = e, e = (size_t)m) {
        std::sort(queue.begin() + (std::ptrdiff_t)b, queue.begin() + (std::ptrdiff_t)e);
        for (size_t i = b; i < e; ++i)
            out.rows.push_back(rows[queue[i]]);
        out.close();
    }
}

// Time of one tile and launch with two workgroups a CU, in microseconds: the
// closure's vectors and H are waited for about three times in a row, then the
// products run at the rate of the LDS gathers.  Fitted on graphene, complex128
// (depths 5, 7, 10: 15.8, 17.4, 20.8 us at 1565 to 1900 rows), and the AB
// bilayer, complex64 (11.1 us at depth 5 and 1770 rows).
double step_tile_us(int dtype, int w, double rows, double products)
{
    const bool c128 = dtype == TBPM_C128;
    return 3.0 + rows * (c128 ? 0.0045 : 0.0023) + products * (c128 ? 0.00067 : 0.00052) * (w + 4) / 8.0;
}

}  // namespace

void free_steps(tbpm_ham *ham)
{
    tbpm_ham::StepPlan &p = ham->steps;
    ham->ctx->dev_free(p.clo_ptr);
    ham->ctx->dev_free(p.layer);
    ham->ctx->dev_free(p.rows);
    ham->ctx->dev_free(p.lcol);
    ham->ctx->dev_free(p.vsel);
    p = tbpm_ham::StepPlan();
}

// Builds ham->steps on stream st (left empty where no plan fits).  Only device
// errors are returned.
hipError_t build_steps(tbpm_ham *ham, hipStream_t st)
{
    tbpm_ctx *ctx = ham->ctx;
    const int64_t n = ham->n;
    if (ham->format == TBPM_FMT_CSR || ham->patch_rows > 1024 || step_closure_max(ham->dtype, ham->ell_w, true) == 0)
        return hipSuccess;
    Columns h;
    h.ld = ham->ell_ld;
    h.w = ham->ell_w;
    auto fetch = [&]() -> hipError_t {
        if (!h.c.empty())
            return hipSuccess;
        h.c.resize((size_t)h.w * (size_t)h.ld);
        return hipMemcpy(h.c.data(), ham->col, h.c.size() * 4, hipMemcpyDeviceToHost);
    };
    // scratch on the device, freed on every way out
    std::vector<void *> held;
    auto take = [&](size_t bytes) -> void * {
        void *q = ctx->dev_alloc(bytes);
        if (q)
            held.push_back(q);
        return q;
    };
    auto done = [&](hipError_t e) -> hipError_t {
        (void)hipStreamSynchronize(st);
        for (void *q : held)
            ctx->dev_free(q);
        if (e != hipSuccess)
            free_steps(ham);
        return e;
    };
#define PLAN_HIP(expr)                                                                       \
    do {                                                                                     \
        const hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                                \
            return done(e_);                                                                 \
    } while (0)

    int32_t facts = 0;
    int32_t *d_flag = (int32_t *)take(256);
    if (!d_flag)
        return done(hipErrorOutOfMemory);
    PLAN_HIP(hipMemsetAsync(d_flag, 0, 4, st));
    PLAN_HIP(launch_step_facts(ham->dtype, ham->col, ham->val, n, h.ld, h.w, d_flag, st));
    PLAN_HIP(hipMemcpyAsync(&facts, d_flag, 4, hipMemcpyDeviceToHost, st));
    PLAN_HIP(hipStreamSynchronize(st));
    const bool real = (facts & 1) == 0;
    const int cap = step_closure_max(ham->dtype, h.w, real);
    if (cap < 1024)
        return done(hipSuccess);

    Tiles first;
    if (ham->patched) {
        first.rows.resize((size_t)n);
        for (int64_t i = 0; i < n; ++i)
            first.rows[(size_t)i] = (int32_t)i;
        first.ptr = ham->h_patch_ptr;
    } else {
        PLAN_HIP(fetch());
        grow_tiles(h, n, (int)std::min<int64_t>(1024, std::max<int64_t>(64, (n + 255) / 256)), first);
    }
    // the depth of which a time step at the default truncation (19 products) costs least
    struct Choice {
        Tiles tiles;
        std::vector<int32_t> size;
        int depth = 0;
        double tile_us = 0.0, step_us = 1e300;
    } best;
    for (int depth : {19, 10, 7, 5}) {
        // a patch's rows within 19 hops do not fit
        if (depth == 19 && ham->patched)
            continue;
        Tiles good, todo = first;
        std::vector<int32_t> size, layer, over;
        double products = 0.0;              // rows formed, over all products of a launch
        bool fits = true;
        while (fits && todo.count() > 0) {
            const int64_t nt = todo.count();
            const size_t mark = held.size();
            int32_t *d_ptr = (int32_t *)take((size_t)(nt + 1) * 4), *d_rows = (int32_t *)take(todo.rows.size() * 4),
                    *d_layer = (int32_t *)take((size_t)nt * (depth + 1) * 4), *d_over = (int32_t *)take((size_t)nt * 4);
            if (!d_ptr || !d_rows || !d_layer || !d_over)
                return done(hipErrorOutOfMemory);
            layer.resize((size_t)nt * (depth + 1));
            over.resize((size_t)nt);
            PLAN_HIP(hipMemcpyAsync(d_ptr, todo.ptr.data(), (size_t)(nt + 1) * 4, hipMemcpyHostToDevice, st));
            PLAN_HIP(hipMemcpyAsync(d_rows, todo.rows.data(), todo.rows.size() * 4, hipMemcpyHostToDevice, st));
            PLAN_HIP(launch_step_plan(ham->col, h.ld, h.w, depth, cap, (int)nt, d_ptr, d_rows, d_layer, d_over,
                                      nullptr, nullptr, nullptr, nullptr, 0, nullptr, false, st));
            PLAN_HIP(hipMemcpyAsync(layer.data(), d_layer, layer.size() * 4, hipMemcpyDeviceToHost, st));
            PLAN_HIP(hipMemcpyAsync(over.data(), d_over, over.size() * 4, hipMemcpyDeviceToHost, st));
            PLAN_HIP(hipStreamSynchronize(st));
            while (held.size() > mark) {
                ctx->dev_free(held.back());
                held.pop_back();
            }
            Tiles next;
            for (int64_t i = 0; i < nt; ++i) {
                const int32_t b = todo.ptr[(size_t)i], e = todo.ptr[(size_t)i + 1];
                if (!over[(size_t)i]) {
                    good.rows.insert(good.rows.end(), todo.rows.begin() + b, todo.rows.begin() + e);
                    good.close();
                    size.push_back(layer[(size_t)i * (depth + 1) + depth]);
                    for (int d = 0; d < depth; ++d)
                        products += layer[(size_t)i * (depth + 1) + d];
                    continue;
                }
                // a handful of rows that reach too far: the graph grows too fast for this depth
                if (e - b < 8) {
                    fits = false;
                    break;
                }
                PLAN_HIP(fetch());
                split_tile(h, todo.rows.data() + b, e - b, next);
            }
            todo = std::move(next);
            if (good.count() + todo.count() > 4 * first.count() + 1024)
                fits = false;
        }
        int64_t total = 0;
        for (int32_t c : size)
            total += c;
        if (!fits || total > INT32_MAX)
            continue;
        const double nt = (double)good.count();
        const double tile_us = step_tile_us(ham->dtype, h.w, (double)total / nt, products / nt);
        const double step_us = (double)((19 + depth - 1) / depth) * std::max(1.0, nt / STEP_SLOTS) * tile_us;
        if (step_us < best.step_us) {
            best.tiles = std::move(good);
            best.size = std::move(size);
            best.depth = depth;
            best.tile_us = tile_us;
            best.step_us = step_us;
        }
        if (getenv("TBPM_PLAN_LOG"))
            fprintf(stderr, "plan: n %lld first %lld tiles %.0f depth %d mean %.0f amp %.2f avg %.2f real %d tile %.1f us step %.1f us\n", (long long)n, (long long)first.count(), nt, depth, (double)total / nt, (double)total / n, products/depth/n, real, tile_us, step_us);
        if (depth == 19 && nt <= STEP_SLOTS)
            break;                          // every tile at once, one launch a step
    }
    if (best.depth > 0) {
        const int depth = best.depth;
        const int64_t nt = best.tiles.count();
        std::vector<int32_t> cp((size_t)nt + 1, 0);
        for (int64_t i = 0; i < nt; ++i)
            cp[(size_t)i + 1] = cp[(size_t)i] + best.size[(size_t)i];
        tbpm_ham::StepPlan &p = ham->steps;
        p.lde = ((int64_t)cp.back() + 255) / 256 * 256;
        p.clo_ptr = (int32_t *)ctx->dev_alloc((size_t)(nt + 1) * 4);
        p.layer = (int32_t *)ctx->dev_alloc((size_t)nt * (depth + 1) * 4);
        p.rows = (int32_t *)ctx->dev_alloc((size_t)p.lde * 4);
        p.lcol = (uint64_t *)ctx->dev_alloc((size_t)((h.w + 3) / 4) * (size_t)p.lde * 8);
        p.vsel = (uint32_t *)ctx->dev_alloc((size_t)((h.w + 3) / 4) * (size_t)p.lde * 4);
        int32_t *d_ptr = (int32_t *)take((size_t)(nt + 1) * 4), *d_rows = (int32_t *)take((size_t)n * 4),
                *d_over = (int32_t *)take((size_t)nt * 4);
        if (!p.clo_ptr || !p.layer || !p.rows || !p.lcol || !p.vsel || !d_ptr || !d_rows || !d_over)
            return done(hipErrorOutOfMemory);
        PLAN_HIP(hipMemcpyAsync(p.clo_ptr, cp.data(), (size_t)(nt + 1) * 4, hipMemcpyHostToDevice, st));
        PLAN_HIP(hipMemcpyAsync(d_ptr, best.tiles.ptr.data(), (size_t)(nt + 1) * 4, hipMemcpyHostToDevice, st));
        PLAN_HIP(hipMemcpyAsync(d_rows, best.tiles.rows.data(), (size_t)n * 4, hipMemcpyHostToDevice, st));
        PLAN_HIP(launch_step_plan(ham->col, h.ld, h.w, depth, cap, (int)nt, d_ptr, d_rows, p.layer, d_over, p.clo_ptr,
                                  p.rows, p.lcol, p.vsel, p.lde, ham->vidx, (facts & 2) == 0, st));
        PLAN_HIP(hipStreamSynchronize(st));
        p.ntiles = nt;
        p.depth = depth;
        p.max_rows = *std::max_element(best.size.begin(), best.size.end());
        p.tile_us = best.tile_us;
        p.real = real;
        p.self = (facts & 2) == 0;
        ham->bytes += (size_t)(nt + 1) * 4 + (size_t)nt * (depth + 1) * 4 +
                      (size_t)p.lde * (4 + 12 * (size_t)((h.w + 3) / 4));
    }
#undef PLAN_HIP
    return done(hipSuccess);
}

}  // namespace tbpm
