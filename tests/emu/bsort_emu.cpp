// Runs the bucket sort of the values (the kernels' own source, cut out of
// valuefit.hip by the test that builds this file) on the host, block by block,
// in the order the launcher issues them, and compares ranks and sorted values
// with a stable sort.  Every buffer is a heap allocation of exactly the size
// the plan gives, under AddressSanitizer and UBSan.
#include "hip/hip_runtime.h"
#include "dr_common.hpp"
#include "ranges.hpp"
#include <algorithm>
#include <functional>
#include <random>
#include <string>
#include <vector>

void emu_launch(uint32_t grid, uint32_t nt, const std::function<void()> &body);

namespace dr {
#include "ext_stile.inc"
#include "ext_bsort.inc"
}  // namespace dr
using namespace dr;

static float value(const std::string &kind, uint32_t i, uint32_t n, std::mt19937 &rng) {
    std::normal_distribution<float> normal;
    if (kind == "equal") return 0.25f;
    if (kind == "coarse") return (float)((int)(rng() % 19) - 9) * 0.25f;
    if (kind == "ulps") {  // neighbouring floats, each many times, and two far off
        if (i == 0 || i == n / 2) return i ? -1e30f : 1e30f;
        return __uint_as_float(__float_as_uint(1.5f) + rng() % 30);
    }
    if (kind == "nested") {  // clusters within clusters: too full after each cut but the last
        const uint32_t far[4] = {1u << 14, 1u << 6, 1u, 0u};
        return i == 7 ? -1e30f : __uint_as_float(__float_as_uint(1.0f) + (i < 4 ? far[i] : 0u));
    }
    if (kind == "signs") {  // two narrow clusters far apart
        const float x = 1.0f + 1e-6f * (float)(rng() % 16);
        return rng() & 1 ? x : -x;
    }
    return normal(rng);
}

// usage: kind planned nv ...: a tensor of nv values planned for `planned`
int main(int argc, char **argv) {
    const std::string kind = argv[1];
    const uint32_t T = (uint32_t)(argc - 2) / 2;
    std::vector<TDesc> td(T);
    memset(td.data(), 0, T * sizeof(TDesc));
    std::vector<uint32_t> plan(T), nv(T);
    uint64_t slots = 0, pairs = 0;
    uint32_t nb = 0, stiles = 0;
    bool multi = false;
    for (uint32_t t = 0; t < T; ++t) {
        plan[t] = atoi(argv[2 + 2 * t]);
        nv[t] = atoi(argv[3 + 2 * t]);
        TDesc &d = td[t];
        d.nv = nv[t];
        d.in.slot = slots;
        d.in.bs0 = nb;
        d.in.bsn = plan[t] <= BS_CAP ? 1 : (plan[t] + BS_AVG - 1) / BS_AVG;
        d.stile0 = stiles;
        d.sntiles = (nv[t] + TILE - 1) / TILE;
        multi |= d.in.bsn > 1;
        nb += d.in.bsn;
        stiles += d.sntiles;
        // as the selection's arrays give: 2 pairs a slot, the buckets within them
        const uint64_t need = std::max<uint64_t>(nv[t], (d.in.bsn > 1 ? (uint64_t)d.in.bsn * BS_CAP : 0) / 2);
        slots += (need + TILE - 1) / TILE * TILE;
    }
    pairs = 2 * slots;
    std::vector<uint32_t> keyA(slots), sig(slots, 0xAAAAAAAAu), cnt(nb, 0);
    std::vector<float> vs(slots, -7.0f), val(slots);
    std::vector<uint64_t> spl(nb, 0xDEADBEEFull), pr(pairs, 0xA5A5A5A5ull);
    std::mt19937 rng(3);
    for (uint32_t t = 0; t < T; ++t)
        for (uint32_t i = 0; i < nv[t]; ++i) {
            val[td[t].in.slot + i] = value(kind, i, nv[t], rng);
            keyA[td[t].in.slot + i] = ~order_key(val[td[t].in.slot + i]);
        }
    Glob glob{};
    glob.sort_tiles = stiles;
    Work w{};
    w.td = td.data();
    w.glob = &glob;
    w.ntensors = T;
    w.keyA = keyA.data();
    w.sig = sig.data();
    w.vsorted = vs.data();
    w.bscnt = cnt.data();
    w.bsspl = spl.data();
    w.bspair = pr.data();
    w.bstotal = nb;
    w.bsmulti = multi;
    if (multi) {
        emu_launch(T, BS_SPLIT_THREADS, [&] { k_bsort_split(w); });
        emu_launch(3, NTHREADS, [&] { k_bsort_deal(w); });
    }
    emu_launch(nb, BS_THREADS, [&] { k_bsort_bucket(w); });
    size_t bad = 0;
    for (uint32_t t = 0; t < T; ++t) {
        const uint64_t s = td[t].in.slot;
        std::vector<uint32_t> o(nv[t]);
        for (uint32_t i = 0; i < nv[t]; ++i) o[i] = i;
        std::stable_sort(o.begin(), o.end(), [&](uint32_t a, uint32_t b) { return keyA[s + a] < keyA[s + b]; });
        for (uint32_t r = 0; r < nv[t]; ++r) bad += sig[s + o[r]] != r || vs[s + r] != val[s + o[r]];
    }
    printf("%s: %zu values wrong\n", bad ? "FAIL" : "OK", bad);
    return bad ? 1 : 0;
}
