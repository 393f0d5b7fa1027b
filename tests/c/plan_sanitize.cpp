// The host planner (plan.cpp) under AddressSanitizer, UBSan and libstdc++
// bounds assertions, over the workloads, the test layouts and the rejected
// inputs of the test suite. Prints one summary line; any sanitizer report or
// unexpected status makes the run fail. Every accepted plan's band launches are
// checked against what keeps the kernels in range (see check_items).
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <string>
#include <vector>
#include "plan.hpp"
using namespace nsg;

static int n_ok = 0, n_err = 0, n_bad = 0;

// What the band kernels rely on: an item's elements fit its threads, its
// threads are whole waves of the launch's block (all of it in a tier's launch),
// its matrix-core tiles fit its waves, its sequences fit the launch's LDS, the
// paired load forms stay inside data plus guard, no prime stage in a Bluestein
// length (its first stage takes the kernel's product), and every band of every
// signal is transformed once.
static void check_items(const HostPlan& p, const char* what) {
    auto bad = [&](const char* why, size_t at) {
        printf("UNEXPECTED %s: %s at %zu\n", what, why, at);
        ++n_bad;
    };
    std::vector<int> seen(p.bands.size() * static_cast<size_t>(p.batch), 0);
    size_t total = 0;
    for (const Bucket& bk : p.buckets) {
        if (bk.lds_elems * 8 > 160 * 1024) bad("reserved LDS", 0);
        total += static_cast<size_t>(bk.nitems);
        for (int i = bk.item_off; i < bk.item_off + bk.nitems; ++i) {
            const WorkItem& w = p.items[static_cast<size_t>(i)];
            const size_t at = static_cast<size_t>(i);
            const FftDesc& d = p.ffts[static_cast<size_t>(w.bd.fft)];
            if (w.nt % 64 || w.nt < 64 || w.nt > bk.nt || (!bk.all && w.nt != bk.nt)) bad("threads", at);
            if ((static_cast<int64_t>(w.bd.n) << w.lgnb) > static_cast<int64_t>(w.nt) * bk.ept) bad("elements", at);
            if (lds_slots(w.bd.n, w.lgnb) > bk.lds_elems) bad("LDS", at);
            if (d.n != w.bd.n || d.nstages > kLdsStages) bad("descriptor", at);
            for (int s = 0; s < d.nstages; ++s) {
                const int R = d.st[s].R;
                if (R <= 16) continue;
                if (w.bd.chirp >= 0) bad("prime stage in a Bluestein length", at);
                if (mfma_tiles((w.bd.n / R) << w.lgnb, R) > kMfmaTilesPerWave * (w.nt / 64)) bad("tiles", at);
            }
            const int64_t st = w.nt >> w.lgnb, reach = w.bd.M - 1 + 3 * st;
            if ((w.fast & kItemFastRoute) && (w.bd.k_lo < 1 || w.bd.k_lo + w.bd.M > p.L || 3 * st > p.L ||
                                              w.bd.k_lo + reach >= p.L + kFastGuard || w.bd.off + reach >= p.C + kFastGuard))
                bad("paired router reads", at);
            if ((w.fast & kItemFastCoef) && w.bd.off + reach >= p.C) bad("paired coefficient reads", at);
            if (w.count < 1 || w.count > (1 << w.lgnb) || w.s0 < 0 || w.s0 + w.count > p.batch) {
                bad("signals", at);
                continue;
            }
            for (int k = 0; k < w.count; ++k) ++seen[static_cast<size_t>(w.band) * p.batch + w.s0 + k];
        }
    }
    if (total != p.items.size()) bad("items outside the launches", total);
    // huge bands: every tile of every signal in the column and row pass, and
    // again in the second transform of a Bluestein band
    for (int pass = 0; pass < 4; ++pass) {
        size_t want = 0;
        for (const BigDesc& g : p.bigs) {
            const bool blu = p.banddev[static_cast<size_t>(g.band)].chirp >= 0;
            if (pass >= 2 && !blu) continue;
            const int n = pass % 2 ? g.n1 : g.n2, lg = pass % 2 ? g.lgb : g.lga;
            want += static_cast<size_t>((n + (1 << lg) - 1) >> lg) * static_cast<size_t>(p.batch);
            if (pass == 0)
                for (int k = 0; k < p.batch; ++k) ++seen[static_cast<size_t>(g.band) * p.batch + k];
        }
        if (want != static_cast<size_t>(p.big_n[pass])) bad("huge-band items", static_cast<size_t>(pass));
    }
    for (size_t i = 0; i < seen.size(); ++i)
        if (seen[i] != 1) bad("coverage", i);
}
// The shared launch of a plan: threads of its block and elements per thread.
static void shared(double fs, double fmin, int B, int64_t N, int batch, int nt, int ept) {
    HostPlan p; std::string err;
    const int r = build_host_plan(p, fs, fmin, fs / 2, B, N, batch, false, err);
    const Bucket* all = nullptr;
    for (const Bucket& bk : p.buckets)
        if (bk.all) all = &bk;
    if (r != 0 || !all || all->nt != nt || all->ept != ept) {
        printf("UNEXPECTED shared launch N=%lld: %dx%d\n", (long long)N, all ? all->nt : 0, all ? all->ept : 0);
        ++n_bad;
    }
}
static void cq(double fs, double fmin, double fmax, int B, int64_t N, int batch, bool sliced, bool expect_ok) {
    HostPlan p; std::string err;
    int r = build_host_plan(p, fs, fmin, fmax, B, N, batch, sliced, err);
    if ((r == 0) != expect_ok) {
        printf("UNEXPECTED cq fs=%g N=%lld B=%d r=%d %s\n", fs, (long long)N, B, r, err.c_str());
        ++n_bad;
    }
    if (r == 0) check_items(p, "cq");
    (r == 0 ? n_ok : n_err)++;
}
static void bl(double fs, int64_t N, int batch, const std::vector<BandSpec>& s, bool sliced, bool expect_ok) {
    HostPlan p; std::string err;
    int r = build_host_plan_bands(p, fs, N, batch, s, sliced, err);
    if ((r == 0) != expect_ok) {
        printf("UNEXPECTED bands N=%lld r=%d %s\n", (long long)N, r, err.c_str());
        ++n_bad;
    }
    if (r == 0) check_items(p, "bands");
    (r == 0 ? n_ok : n_err)++;
}
static std::vector<BandSpec> padded(const std::vector<double>& xs, const std::vector<int64_t>& lens, int64_t dc, int64_t ny) {
    std::vector<BandSpec> s;
    s.push_back({0, xs[0], xs[0] * 0.35, dc, 0.0});
    for (size_t i = 0; i < xs.size(); ++i) s.push_back({1, xs[i], xs[i] * 0.35, lens[i], 0.0});
    s.push_back({2, xs.back(), xs.back() * 0.35, ny, 0.0});
    return s;
}
int main() {
    // workloads
    cq(22050, 110, 11025, 12, 16384, 1, false, true);
    cq(44100, 32.7, 22050, 48, 44100, 1, false, true);
    cq(44100, 40, 22050, 24, 220500, 16, false, true);
    cq(22050, 55, 11025, 36, 88200, 128, false, true);
    cq(48000, 20, 24000, 96, 2880000, 1, false, true);
    cq(48000, 20, 24000, 96, 131072, 16, true, true);
    // small test layouts
    cq(4, 0.5, 2, 1, 4, 2, false, true);
    cq(6, 0.7, 3, 1, 6, 2, false, true);
    cq(8, 1, 4, 1, 8, 1, false, true);
    cq(30, 1, 15, 2, 30, 3, false, true);
    cq(250, 4, 125, 4, 500, 2, false, true);
    cq(268, 4, 134, 4, 268, 2, false, true);
    cq(1028, 8, 514, 6, 1028, 3, false, true);
    cq(250, 4, 125, 3, 250, 1, false, true);
    cq(4620, 30, 2310, 12, 4620, 3, false, true);
    cq(8000, 50, 4000, 24, 6000, 5, false, true);
    cq(22050, 110, 11025, 12, 16384, 3, false, true);
    // coarse long layout (wide gather records)
    cq(44100, 20, 22050, 12, 1323000, 1, false, true);
    // shared band launches: each block size, with and without 16 elements per
    // thread, beside a huge-band chain, few bands, long phases
    shared(22050, 110, 12, 16384, 19, 256, 8);
    shared(16000, 50, 24, 50274, 3, 512, 8);
    shared(44100, 40, 24, 132300, 2, 1024, 8);
    shared(44100, 40, 24, 220500, 3, 1024, 16);
    shared(44100, 40, 3, 44100, 3, 1024, 16);
    shared(48000, 40, 12, 240000, 1, 1024, 16);
    shared(48000, 40, 12, 240000, 8, 1024, 8);
    cq(22050, 110, 11025, 12, 16384, 19, false, true);
    cq(16000, 50, 8000, 24, 50274, 3, false, true);
    cq(44100, 40, 22050, 24, 132300, 2, false, true);
    cq(44100, 40, 22050, 24, 220500, 3, false, true);
    cq(44100, 40, 22050, 3, 44100, 3, false, true);
    cq(44100, 690, 22050, 3, 132300, 5, false, true);
    cq(48000, 40, 24000, 12, 240000, 1, false, true);
    cq(48000, 40, 24000, 12, 240000, 8, false, true);
    cq(44100, 40, 22050, 48, 220500, 7, false, true);
    cq(8000, 31, 4000, 17, 65522, 11, false, true);
    // errors
    cq(22050, 110, 11025, 12, 16383, 1, false, false);   // odd N
    cq(22050, 110, 11025, 12, 2, 1, false, false);       // N < 4
    cq(22050, 11025, 11025, 12, 16384, 1, false, false); // fmin at Nyquist
    cq(22050, 110, 50, 12, 16384, 1, false, false);      // fmax < fmin
    cq(22050, 110, 11025, 0, 16384, 1, false, false);    // B < 1
    cq(22050, 110, 11025, 12, 16384, 0, false, false);   // batch < 1
    cq(-1, 110, 11025, 12, 16384, 1, false, false);      // fs <= 0
    // band lists
    std::vector<double> xs12, xs14;
    for (int j = 0; j < 12; ++j) xs12.push_back(8.0 * std::pow(1.35, j));
    for (int j = 0; j < 14; ++j) xs14.push_back(10.0 * std::pow(1.4, j));
    bl(1200, 1200, 2, padded(xs12, {0, 8, 0, 20, 0, 31, 40, 0, 67, 0, 2 * 263, 160}, 16, 1500), false, true);
    bl(4000, 4000, 2, padded(xs14, {0, 0, 0, 0, 0, 0, 8200, 0, 0, 8209, 0, 0, 0, 0}, 0, 9000), false, true);
    bl(4000, 4000, 2, padded(xs14, {512, 513, 2048, 2050, 4096, 4100, 8192, 8200, 16384, 16400, 0, 0, 0, 0}, 0, 0), false, true);
    bl(4000, 4000, 2, padded(xs14, {3, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, 0, 0), false, false);  // length below width
    std::vector<BandSpec> t1;
    table1_specs(t1);
    bl(44100, 65536, 128, t1, false, true);
    bl(44100, 65536, 1, t1, false, true);
    bl(44100, 65536, 16, t1, true, true);
    std::vector<BandSpec> erb; std::string err;
    if (erb_specs(16000, 32000, 50, 8000, 2.0, erb, err) != 0) {
        printf("UNEXPECTED erb %s\n", err.c_str());
        ++n_bad;
    }
    bl(16000, 32000, 2, erb, false, true);
    // maximum huge transform: N = 2^24, a DC band zero-padded to 2^24
    {
        const int64_t N = 1 << 24;
        const double h = double(N / 4);
        std::vector<BandSpec> s = {{0, h, 2.0, N, 0.0}, {1, h, 2.0, 0, 0.0}, {2, h, 2.0, 0, 0.0}};
        bl(48000.0, N, 1, s, false, true);
    }
    // every length a workgroup may transform fits the kernels' stage records
    for (int n = 1; n <= kMaxLdsFft; ++n) {
        std::vector<int> rad;
        if (factor_radices(n, rad) && rad.size() > static_cast<size_t>(kLdsStages)) {
            printf("UNEXPECTED stages n=%d %zu\n", n, rad.size());
            ++n_bad;
        }
    }
    printf("plans ok %d, rejected %d, unexpected %d\n", n_ok, n_err, n_bad);
    return n_bad ? 1 : 0;
}
