// Stores H while large host allocations of the process are refused: H is stored
// without a plan of tiles, no exception leaves the C entry point, and propagations
// with and without the plan agree.  Exits 0 when all of it holds.
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "tbpm.h"

static std::atomic<size_t> limit{0};             // 0: none; else the bytes from which new is refused
static std::atomic<int> refused{0};

void *operator new(std::size_t n)
{
    const size_t l = limit.load();
    if (l && n >= l) {
        ++refused;
        throw std::bad_alloc();
    }
    if (void *p = std::malloc(n ? n : 1))
        return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

static int failures = 0;

static void check(bool ok, const char *what)
{
    std::printf("%s: %s\n", what, ok ? "ok" : "FAILED");
    std::fflush(stdout);
    failures += ok ? 0 : 1;
}

int main(int argc, char **argv)
{
    const int32_t format = argc > 1 ? std::atoi(argv[1]) : TBPM_FMT_ELL;
    // a ring of n sites with on-site energies; every third bond cut where the rows are to be uneven
    const int64_t n = 60000;
    std::vector<int64_t> rp{0};
    std::vector<int32_t> col;
    std::vector<double> val;
    auto bond = [&](int64_t i) { return format == TBPM_FMT_ELL || i % 3 != 0; };   // between i and i + 1
    for (int64_t i = 0; i < n; ++i) {
        const int64_t l = (i + n - 1) % n, r = (i + 1) % n;
        for (int64_t c = 0; c < 3; ++c) {
            const int64_t j = i == 0 ? (c == 0 ? 0 : c == 1 ? 1 : n - 1) : i == n - 1 ? (c == 0 ? 0 : n - 3 + c) : i - 1 + c;
            if ((j == l && l != i && !bond(l)) || (j == r && !bond(i)))
                continue;
            col.push_back((int32_t)j);
            val.push_back(j == i ? 0.1 * std::sin((double)i) : -1.0);
            val.push_back(0.0);
        }
        rp.push_back((int64_t)col.size());
    }
    tbpm_csr csr{};
    csr.n = n;
    csr.nnz = rp.back();
    csr.row_ptr = rp.data();
    csr.col = col.data();
    csr.val = val.data();
    tbpm_ctx *ctx = nullptr;
    check(tbpm_ctx_create(0, nullptr, nullptr, &ctx) == TBPM_OK, "context");
    if (!ctx)
        return 1;
    const int32_t steps = 3;
    std::vector<double> corr[2];
    int64_t tiles[2] = {-1, -1};
    for (int k = 0; k < 2; ++k) {
        tbpm_ham *ham = nullptr;
        tbpm_status s = TBPM_ERR_OOM;
        limit = k == 1 ? 200000 : 0;                 // (the first pass loads the kernels)
        try {
            s = tbpm_build_csr(ctx, &csr, TBPM_C128, format, 0, &ham);
        } catch (const std::bad_alloc &) {
            limit = 0;
            check(false, "no exception from storing H");
        }
        limit = 0;
        check(s == TBPM_OK && ham, k == 1 ? "H stored with host allocations refused" : "H stored");
        if (!ham)
            break;
        check(tbpm_ham_tiles(ham, 1, nullptr, &tiles[k], nullptr) == TBPM_OK, "plan query");
        tbpm_params p{};
        p.rescale = 2.5;
        p.num_time_steps = steps;
        p.num_vectors = 1;
        p.seed = 5;
        corr[k].assign(2 * (steps + 1), 0.0);
        check(tbpm_propagate_dos(ctx, ham, &p, corr[k].data(), nullptr, nullptr, nullptr) == TBPM_OK, "propagation");
        tbpm_ham_destroy(ham);
    }
    check(refused > 0 && tiles[0] > 0 && tiles[1] == 0, "a plan exists only where its memory was given");
    double d = corr[0].size() == corr[1].size() ? 0.0 : 1.0;
    for (size_t i = 0; d < 1.0 && i < corr[0].size(); ++i)
        d = std::fmax(d, std::fabs(corr[0][i] - corr[1][i]));
    check(d <= 1e-10, "results agree");
    tbpm_ctx_destroy(ctx);
    return failures ? 1 : 0;
}
