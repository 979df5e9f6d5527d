// Plans for several products with H per launch (tbpm_steps.hip): which rows
// form a tile, to how many hops, and the closure of each tile.
//
// Tiles are compact regions of the sparsity graph of at most 1024 rows: the
// patches of a patch-reordered H, or (plain ELL, CSR) regions grown by
// breadth-first search here.  A tile whose closure is too large for the kernel (patches of
// several pieces, above all) is cut in two until its parts fit.  Everything
// per row happens on the device; the host sees a few numbers per tile.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <initializer_list>
#include <memory>
#include <new>
#include <thread>
#include <vector>

#include "tbpm_internal.h"

namespace tbpm {

namespace {

struct Tile {
    int32_t begin, count;               // rows: a range of the row list
    int32_t size;                       // rows of its closure, 0: not known or too many
    double products;                    // rows formed in all products of a launch
    bool shared;                        // by small pieces
};

// neighbours of a row: of the caller's CSR, or (rp null) of ELL columns c [w][ld]
struct Rows {
    const int64_t *rp;
    const int32_t *c;
    int64_t ld;
    int w;
    template <typename F>
    void each(int32_t r, F f) const
    {
        if (rp)
            for (int64_t k = rp[r]; k < rp[r + 1]; ++k)
                f(c[k]);
        else
            for (int s = 0; s < w; ++s)
                f(c[(size_t)s * (size_t)ld + (size_t)r]);
    }
};

// f(0) .. f(count - 1) on threads of their own, on this one where none can be had;
// throws std::bad_alloc when one of them ran out of memory
template <typename F>
void in_parallel(int count, F f)
{
    std::atomic<bool> failed{false};
    auto one = [&](int i) {
        try {
            f(i);
        } catch (...) {
            failed = true;
        }
    };
    std::vector<std::thread> threads;
    int i = 0;
    try {
        threads.reserve((size_t)count);
        for (; i + 1 < count; ++i)
            threads.emplace_back(one, i);
    } catch (...) {
    }
    for (; i < count; ++i)
        one(i);
    for (std::thread &t : threads)
        t.join();
    if (failed)
        throw std::bad_alloc();
}

// breadth-first pieces of at most `most` rows among the rows lo .. hi - 1, one
// connected piece each: piece[row] and the pieces' numbers of rows
void grow_pieces(const Rows &g, int32_t lo, int32_t hi, int most, int32_t *piece, std::vector<int32_t> &count)
{
    constexpr int32_t NONE = -1;
    std::fill(piece + lo, piece + hi, NONE);
    std::vector<int32_t> queue((size_t)most);
    int32_t low = lo, taken = lo;
    int32_t seed = NONE;                // an untaken neighbour of the previous piece
    while (taken < hi) {
        if (seed == NONE || piece[seed] != NONE) {
            while (piece[low] != NONE)
                ++low;
            seed = low;
        }
        const int32_t id = (int32_t)count.size();
        int end = 1;
        queue[0] = seed;
        piece[seed] = id;
        seed = NONE;
        for (int i = 0; i < end; ++i)
            g.each(queue[(size_t)i], [&](int32_t u) {
                if (u < lo || u >= hi || piece[u] != NONE)
                    return;
                if (end == most) {
                    if (seed == NONE)
                        seed = u;
                    return;
                }
                piece[u] = id;
                queue[(size_t)end++] = u;
            });
        count.push_back(end);
        taken += end;
    }
}

// Tiles of at most `most` rows, one connected piece each, grown in up to eight
// ranges of the rows at once (491,000 rows: 1.6 ms instead of 7.3; the ranges
// depend on n alone).  Pieces of fewer than `small` rows (what growing left over,
// where it ran into other pieces or a range's end; clusters that vacancies cut off)
// share tiles, in the order found, so that no workgroup is spent on a few rows: a
// quarter of a tile, an eighth left 25 more tiles of 714 than growing in one range
// (graphene with 30% vacancies, 499,000 rows, complex64, two vectors, 12 steps: 0.85 ms
// in one range, 0.90 by an eighth, 0.84 by a quarter).  rows: tile after tile, ascending in each piece.
void grow_tiles(const Rows &g, int64_t n, int most, int small, int32_t *rows, std::vector<Tile> &tiles)
{
    const int parts = (int)std::min<int64_t>(8, std::max<int64_t>(1, n / 32768));
    auto from = [&](int i) { return (int32_t)(n * i / parts); };
    std::unique_ptr<int32_t[]> piece(new int32_t[(size_t)n]);
    std::vector<std::vector<int32_t>> count((size_t)parts);
    in_parallel(parts, [&](int i) { grow_pieces(g, from(i), from(i + 1), most, piece.get(), count[(size_t)i]); });
    std::vector<std::vector<int32_t>> tile_of(count);
    int32_t shared = -1;
    for (int i = 0; i < parts; ++i)
        for (size_t q = 0; q < count[(size_t)i].size(); ++q) {
            const int32_t c = count[(size_t)i][q];
            const bool joins = c < small && shared >= 0 && tiles[(size_t)shared].count + c <= most;
            if (!joins) {
                tiles.push_back({0, 0, 0, 0.0, c < small});
                if (c < small)
                    shared = (int32_t)tiles.size() - 1;
            }
            const int32_t t = joins ? shared : (int32_t)tiles.size() - 1;
            tile_of[(size_t)i][q] = t;
            tiles[(size_t)t].count += c;
        }
    std::vector<int32_t> at(tiles.size());
    int32_t begin = 0;
    for (size_t i = 0; i < tiles.size(); ++i) {
        tiles[i].begin = at[i] = begin;
        begin += tiles[i].count;
    }
    // where each piece begins, then its rows
    for (int i = 0; i < parts; ++i)
        for (size_t q = 0; q < count[(size_t)i].size(); ++q) {
            int32_t &t = tile_of[(size_t)i][q];
            const int32_t b = at[(size_t)t];
            at[(size_t)t] += count[(size_t)i][q];
            t = b;
        }
    in_parallel(parts, [&](int i) {
        std::vector<int32_t> &next = tile_of[(size_t)i];
        for (int32_t r = from(i); r < from(i + 1); ++r)
            rows[next[(size_t)piece[(size_t)r]]++] = r;
    });
}

// Time of one tile and launch with two workgroups a CU, in microseconds: the
// closure's vectors and H are waited for about three times in a row, then the
// products run at the rate of the LDS gathers.  Fitted on graphene, complex128
// (depths 5, 7, 10: 15.8, 17.4, 20.8 us at 1565 to 1900 rows), and the AB
// bilayer, complex64 (11.1 us at depth 5 and 1770 rows).
double tile_time(int dtype, int w, double rows, double products)
{
    const bool c128 = dtype == TBPM_C128;
    return 3.0 + rows * (c128 ? 0.0045 : 0.0023) + products * (c128 ? 0.00067 : 0.00052) * (w + 4) / 8.0;
}

// of a time step at the default truncation (19 products), one vector
double step_time(int depth, double tiles, double tile_us)
{
    return (double)((19 + depth - 1) / depth) * std::max(1.0, tiles / STEP_SLOTS) * tile_us;
}

class Builder {
  public:
    Builder(tbpm_ham *h, const tbpm_csr *host_csr, hipStream_t s)
        : ham(h), ctx(h->ctx), csr(host_csr), st(s), col(h->steps.ell_col ? h->steps.ell_col : h->col),
          val(h->steps.ell_val ? h->steps.ell_val : h->val), ld(h->steps.ld), w(h->steps.w)
    {
    }
    ~Builder()
    {
        (void)hipStreamSynchronize(st);
        for (void *q : held)
            ctx->dev_free(q);
    }
    hipError_t run();

  private:
    tbpm_ham *ham;
    tbpm_ctx *ctx;
    const tbpm_csr *csr;                // H as given, in host memory, or null
    hipStream_t st;
    const int32_t *col;                 // H's slots
    const void *val;
    int64_t ld;
    int w;
    std::vector<void *> held;           // scratch on the device
    int32_t *d_rows = nullptr;          // every row, tile after tile
    int32_t *d_tile = nullptr, *d_out = nullptr;
    size_t tile_cap = 0, out_cap = 0;
    std::vector<int32_t> io, out;

    hipError_t take(int32_t *&p, size_t ints)
    {
        p = (int32_t *)ctx->dev_alloc(ints * 4);
        if (!p)
            return hipErrorOutOfMemory;
        held.push_back(p);
        return hipSuccess;
    }
    // the listed tiles' ranges in d_tile, and room for `ints` results in d_out
    hipError_t list(const std::vector<Tile> &tiles, const std::vector<int32_t> &which, size_t ints)
    {
        io.clear();
        for (int32_t i : which) {
            io.push_back(tiles[(size_t)i].begin);
            io.push_back(tiles[(size_t)i].count);
        }
        hipError_t e = hipSuccess;
        if (io.size() > tile_cap)
            e = take(d_tile, tile_cap = io.size());
        if (e == hipSuccess && ints > out_cap)
            e = take(d_out, out_cap = ints);
        if (e == hipSuccess)
            e = hipMemcpyAsync(d_tile, io.data(), io.size() * 4, hipMemcpyHostToDevice, st);
        return e;
    }
    hipError_t results(size_t ints)
    {
        out.resize(ints);
        hipError_t e = hipMemcpyAsync(out.data(), d_out, ints * 4, hipMemcpyDeviceToHost, st);
        return e == hipSuccess ? hipStreamSynchronize(st) : e;
    }
    hipError_t measure(std::vector<Tile> &tiles, const std::vector<int32_t> &which, int depth, int cap);
    hipError_t split(std::vector<Tile> &tiles, const std::vector<int32_t> &which);
    hipError_t fit(std::vector<Tile> &cut, int depth, int cap, double scale, double least, double *us);
};

// closure sizes of the listed tiles
hipError_t Builder::measure(std::vector<Tile> &tiles, const std::vector<int32_t> &which, int depth, int cap)
{
    const size_t ints = which.size() * (size_t)(depth + 1);
    hipError_t e = list(tiles, which, ints);
    if (e == hipSuccess)
        e = launch_step_plan(col, ld, w, depth, cap, (int)which.size(), d_tile, d_rows, d_out,
                             nullptr, nullptr, nullptr, nullptr, 0, nullptr, false, ham->dtype, st);
    if (e == hipSuccess)
        e = results(ints);
    for (size_t k = 0; e == hipSuccess && k < which.size(); ++k) {
        const int32_t *layer = &out[k * (size_t)(depth + 1)];
        Tile &t = tiles[(size_t)which[k]];
        t.size = layer[depth];
        t.products = 0.0;
        for (int d = 0; t.size > 0 && d < depth; ++d)
            t.products += layer[d];
    }
    return e;
}

// every listed tile in two, in its place: breadth-first halves, or (shared: hundreds
// of small pieces one after the other, of which the kernel walks each) list halves
hipError_t Builder::split(std::vector<Tile> &tiles, const std::vector<int32_t> &which)
{
    std::vector<int32_t> walked;
    for (int32_t i : which)
        if (!tiles[(size_t)i].shared)
            walked.push_back(i);
    hipError_t e = hipSuccess;
    if (!walked.empty()) {
        e = list(tiles, walked, walked.size());
        if (e == hipSuccess)
            e = launch_step_split(col, ld, w, (int)walked.size(), d_tile, d_rows, d_out, st);
        if (e == hipSuccess)
            e = results(walked.size());
    }
    if (e != hipSuccess)
        return e;
    std::vector<Tile> next;
    next.reserve(tiles.size() + which.size());
    size_t k = 0, walk = 0;
    for (size_t i = 0; i < tiles.size(); ++i) {
        const Tile t = tiles[i];
        if (k < which.size() && (size_t)which[k] == i) {
            const int32_t at = t.shared ? (t.count + 1) / 2 : out[walk++];
            next.push_back({t.begin, at, 0, 0.0, t.shared});
            next.push_back({t.begin + at, t.count - at, 0, 0.0, t.shared});
            ++k;
        } else {
            next.push_back(t);
        }
    }
    tiles.swap(next);
    return hipSuccess;
}

#define PLAN_HIP(expr)                                                                       \
    do {                                                                                     \
        const hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                                \
            return e_;                                                                       \
    } while (0)

// Cuts the tiles whose closures are over the cap until all fit.  *us: the modelled
// time of a step where the sample has `scale` times these tiles; it ends early, with
// at least `least`, where that is no longer to be undercut.
hipError_t Builder::fit(std::vector<Tile> &cut, int depth, int cap, double scale, double least, double *us)
{
    std::vector<int32_t> which, bad;
    while (true) {
        which.clear();
        for (size_t i = 0; i < cut.size(); ++i)
            if (cut[i].size == 0)
                which.push_back((int32_t)i);
        PLAN_HIP(measure(cut, which, depth, cap));
        double rows = 0.0, products = 0.0;
        bad.clear();
        bool far = false;
        for (int32_t i : which)
            if (cut[(size_t)i].size == 0) {
                bad.push_back(i);
                far = far || cut[(size_t)i].count < 8;      // a handful of rows that reach too far
            }
        for (const Tile &t : cut) {
            rows += t.size == 0 ? cap : t.size;
            products += t.products;
        }
        const double now = (double)(cut.size() + bad.size());
        *us = step_time(depth, now * scale, tile_time(ham->dtype, w, rows / now, products / now));
        if (far)
            *us = std::max(*us, least);
        if (far || *us >= least || bad.empty())
            return hipSuccess;
        PLAN_HIP(split(cut, bad));
    }
}

hipError_t Builder::run()
{
    const int64_t n = ham->n;
    int32_t *d_flag = nullptr, facts = 0;
    PLAN_HIP(take(d_flag, 64));
    PLAN_HIP(hipMemsetAsync(d_flag, 0, 4, st));
    PLAN_HIP(launch_step_facts(ham->dtype, col, val, n, ld, w, d_flag, st));
    PLAN_HIP(hipMemcpyAsync(&facts, d_flag, 4, hipMemcpyDeviceToHost, st));
    PLAN_HIP(hipStreamSynchronize(st));
    const bool real = (facts & 1) == 0, self = (facts & 2) == 0;
    const int cap = step_closure_max(ham->dtype, w, real);
    if (cap < 1024)
        return hipSuccess;              // not compiled

    std::vector<Tile> first;
    int32_t *d_first = nullptr, *d_spare = nullptr;
    PLAN_HIP(take(d_first, (size_t)n));
    PLAN_HIP(take(d_rows, (size_t)n));
    PLAN_HIP(take(d_spare, (size_t)n));
    if (ham->patched) {
        for (int64_t q = 0; q < ham->npatch; ++q) {
            const int32_t b = ham->h_patch_ptr[(size_t)q];
            first.push_back({b, ham->h_patch_ptr[(size_t)q + 1] - b, 0, 0.0, false});
        }
        PLAN_HIP(launch_iota(d_first, n, st));
    } else {
        std::unique_ptr<int32_t[]> c, rows(new int32_t[(size_t)n]);
        Rows g{csr ? csr->row_ptr : nullptr, csr ? csr->col : nullptr, ld, w};
        if (!csr) {
            const size_t slots = (size_t)w * (size_t)ld;
            c.reset(new int32_t[slots]);
            g.c = c.get();
            PLAN_HIP(hipMemcpyAsync(c.get(), col, slots * 4, hipMemcpyDeviceToHost, st));
            PLAN_HIP(hipStreamSynchronize(st));
        }
        const int most = (int)std::min<int64_t>(1024, std::max<int64_t>(64, (n + 255) / 256));
        grow_tiles(g, n, most, ham->format == TBPM_FMT_CSR ? most / 4 : 0, rows.get(), first);
        PLAN_HIP(hipMemcpyAsync(d_first, rows.get(), (size_t)n * 4, hipMemcpyHostToDevice, st));
        PLAN_HIP(hipStreamSynchronize(st));
    }

    // The depth of which a step costs least: for each, tiles whose closures all
    // fit, those over the cap cut in two until they do.  Nothing is planned that
    // the term kernels outrun for one vector and (complex64) for blocks of 8.
    std::vector<Tile> tiles;
    int depth = 0;
    double least = std::max(terms_us(ham, 20, 1), ham->dtype == TBPM_C64 ? terms_us(ham, 20, 8) / 8 : 0.0);
    struct Try {
        int depth;
        double us;                      // as a sample of the tiles has it
    };
    std::vector<Try> order;
    // Many tiles grown here: what each depth would cost is first found on up to 32 of
    // them (not those that small pieces share: they are cut most, and few), from 10
    // on, which wins most often, so that the others end as soon as they cost a tenth
    // more.  The four take 0.5 to 5 ms so (521 tiles of 491,000 rows of 3; 766 of
    // 784,000 rows of 12), on all tiles 7 and 40; of 280 tiles the search on all
    // takes 2 to 3 and a sample no less.  (On patches, whose search is a few percent
    // of storing H, all tiles decide: patches of several pieces make a sample miss.)
    constexpr size_t SAMPLE = 32;
    const bool sampled = !ham->patched && first.size() >= 16 * SAMPLE;
    for (int d : sampled ? std::initializer_list<int>{10, 19, 7, 5} : std::initializer_list<int>{19, 10, 7, 5})
        if (d != 19 || !ham->patched)   // a patch's rows within 19 hops do not fit
            order.push_back({d, 0.0});
    std::vector<Tile> some;
    for (size_t i = 0; sampled && i < SAMPLE; ++i)
        for (size_t k = (2 * i + 1) * first.size() / (2 * SAMPLE); k < (i + 1) * first.size() / SAMPLE; ++k)
            if (!first[k].shared) {
                some.push_back(first[k]);
                break;
            }
    if (!some.empty()) {
        const double scale = (double)first.size() / (double)some.size();
        double bound = 1.1 * least;
        for (Try &t : order) {
            PLAN_HIP(hipMemcpyAsync(d_rows, d_first, (size_t)n * 4, hipMemcpyDeviceToDevice, st));
            std::vector<Tile> cut = some;
            PLAN_HIP(fit(cut, t.depth, cap, scale, bound, &t.us));
            bound = std::min(bound, 1.1 * t.us);
        }
        std::stable_sort(order.begin(), order.end(), [](const Try &a, const Try &b) { return a.us < b.us; });
    }
    for (const Try &t : order) {
        if (t.us >= 1.1 * least)
            continue;                   // (a sample misses by a few percent)
        std::swap(d_rows, d_spare);     // d_spare: the best tiles so far
        PLAN_HIP(hipMemcpyAsync(d_rows, d_first, (size_t)n * 4, hipMemcpyDeviceToDevice, st));
        std::vector<Tile> cut = first;
        double us = least;
        PLAN_HIP(fit(cut, t.depth, cap, 1.0, least, &us));
        if (us < least) {
            least = us;
            depth = t.depth;
            tiles.swap(cut);
        } else {
            std::swap(d_rows, d_spare);
        }
        if (depth == 19 && (double)tiles.size() <= STEP_SLOTS)
            break;                      // every tile at once, one launch a step
    }
    if (depth == 0)
        return hipSuccess;
    const size_t nt = tiles.size();
    std::vector<int32_t> cp(nt + 1, 0);
    int64_t total = 0;
    double products = 0.0;
    int32_t most = 0, own = 0;
    for (size_t i = 0; i < nt; ++i) {
        most = std::max(most, tiles[i].size);
        own = std::max(own, tiles[i].count);
        products += tiles[i].products;
        total += tiles[i].size;
        if (total > INT32_MAX)
            return hipSuccess;
        cp[i + 1] = (int32_t)total;
    }
    tbpm_ham::StepPlan &p = ham->steps;
    const size_t words = (size_t)((w + 3) / 4);
    p.lde = (total + 255) / 256 * 256;
    p.clo_ptr = (int32_t *)ctx->dev_alloc((nt + 1) * 4);
    p.layer = (int32_t *)ctx->dev_alloc(nt * (size_t)(depth + 1) * 4);
    p.rows = (int32_t *)ctx->dev_alloc((size_t)p.lde * 4);
    p.lcol = (uint64_t *)ctx->dev_alloc(words * (size_t)p.lde * 8);
    p.vsel = (uint32_t *)ctx->dev_alloc(words * (size_t)p.lde * 4);
    if (!p.clo_ptr || !p.layer || !p.rows || !p.lcol || !p.vsel)
        return hipErrorOutOfMemory;
    std::vector<int32_t> all(nt);
    for (size_t i = 0; i < nt; ++i)
        all[i] = (int32_t)i;
    PLAN_HIP(list(tiles, all, 1));
    PLAN_HIP(hipMemcpyAsync(p.clo_ptr, cp.data(), (nt + 1) * 4, hipMemcpyHostToDevice, st));
    PLAN_HIP(launch_step_plan(col, ld, w, depth, cap, (int)nt, d_tile, d_rows, p.layer, p.clo_ptr, p.rows, p.lcol,
                              p.vsel, p.lde, ham->vidx, self, ham->dtype, st));
    PLAN_HIP(hipStreamSynchronize(st));
    p.depth = depth;
    p.max_rows = most;
    p.tile_rows = own;
    p.tile_us = tile_time(ham->dtype, w, (double)total / (double)nt, products / (double)nt);
    p.real = real;
    p.self = self;
    p.ntiles = (int64_t)nt;
    ham->bytes += (nt + 1) * 4 + nt * (size_t)(depth + 1) * 4 + (size_t)p.lde * (4 + 12 * words);
    return hipSuccess;
}
#undef PLAN_HIP

}  // namespace

void free_steps(tbpm_ham *ham)
{
    tbpm_ham::StepPlan &p = ham->steps;
    ham->ctx->dev_free(p.clo_ptr);
    ham->ctx->dev_free(p.layer);
    ham->ctx->dev_free(p.rows);
    ham->ctx->dev_free(p.lcol);
    ham->ctx->dev_free(p.vsel);
    ham->ctx->dev_free(p.ell_col);
    ham->ctx->dev_free(p.ell_val);
    p = tbpm_ham::StepPlan();
}

// Rows of uneven length stay in CSR, whose kernels read H's values and gather
// vectors at 4.1 TB/s at best; the tiles' kernel holds H in registers, so the
// padding to the next width it is compiled for costs no more than those.
hipError_t step_slots(tbpm_ham *ham, const int64_t *rp, const int32_t *col, const double *val, hipStream_t st)
{
    tbpm_ham::StepPlan &p = ham->steps;
    for (int w : {3, 4, 5, 8, 12})
        if (p.w == 0 && ham->max_row <= w && step_closure_max(ham->dtype, w, true) > 0)
            p.w = w;
    if (p.w == 0 || ham->max_row == 0)
        return hipSuccess;
    p.ld = (ham->n + 255) / 256 * 256;
    const size_t slots = (size_t)p.w * (size_t)p.ld;
    p.ell_col = (int32_t *)ham->ctx->dev_alloc(slots * 4);
    p.ell_val = ham->ctx->dev_alloc(slots * (ham->dtype == TBPM_C128 ? 16 : 8));
    if (!p.ell_col || !p.ell_val) {
        free_steps(ham);
        return hipSuccess;
    }
    return launch_to_ell(ham->dtype, rp, col, val, ham->n, p.w, p.ld, p.ell_col, p.ell_val, st);
}

// Builds ham->steps on stream st (host_csr: H as given, where that is in host
// memory), left empty where no plan fits or pays, or
// where memory of the device or the host does not suffice for it (the term
// kernels need none).
hipError_t build_steps(tbpm_ham *ham, const tbpm_csr *host_csr, hipStream_t st)
{
    tbpm_ham::StepPlan &p = ham->steps;
    if (ham->format == TBPM_FMT_CSR) {
        if (!p.ell_val)
            return hipSuccess;
    } else {
        p.w = ham->ell_w;
        p.ld = ham->ell_ld;
    }
    if (ham->patch_rows > 1024 || step_closure_max(ham->dtype, p.w, true) == 0)
        return hipSuccess;
    hipError_t e;
    try {
        Builder b(ham, host_csr, st);
        e = b.run();
    } catch (const std::bad_alloc &) {              // host memory: no plan either
        e = hipErrorOutOfMemory;
    }
    if (p.ntiles == 0) {
        free_steps(ham);
    } else if (p.ell_col) {
        ham->ctx->dev_free(p.ell_col);
        p.ell_col = nullptr;
        ham->bytes += (size_t)p.w * (size_t)p.ld * (ham->dtype == TBPM_C128 ? 16 : 8);
    }
    return e == hipErrorOutOfMemory ? hipSuccess : e;
}

}  // namespace tbpm
