// Runs a wave of the probe pass (its own source, cut out of bloom.hip by the
// test that builds this file) on the host, 64 threads in step, over one window
// for every way of testing a filter's hashes, and compares the window's bitmap
// with a direct query.  The LDS part of the filter, the filter, the queue and
// the bitmap are heap allocations of exactly their sizes, under
// AddressSanitizer and UBSan.
#include "hip/hip_runtime.h"
#include "dr_common.hpp"
#include <functional>
#include <memory>
#include <random>

void emu_launch(uint32_t grid, uint32_t nt, const std::function<void()> &body);

namespace dr {
enum QueryMode { Q_ENCODE = 0, Q_PLAIN = 1, Q_DECODE = 2, Q_SUM = 3 };
__device__ inline uint32_t uni(uint32_t x) { return x; }
#include "ext_sizes.inc"
static void zero_step(float *dz, uint32_t s0, uint32_t nvalid) {
    for (uint32_t e = threadIdx.x; e < QWAVE; e += 64)
        if (s0 + e < nvalid) dz[s0 + e] = 0.0f;
}
#include "ext_groups.inc"
#include "ext_windows.inc"
}  // namespace dr
using namespace dr;

static uint32_t failures = 0, runs = 0;

template <int MODE>
static void one(uint32_t m, uint32_t k, uint32_t lds_words, bool part, uint32_t J, uint32_t nvalid, double fill) {
    std::mt19937 rng(m + k + J + nvalid);
    const uint32_t words = m / 32, fcw = std::min(words, lds_words), wbase = 4096 * (rng() % 50);
    std::unique_ptr<uint32_t[]> filt(new uint32_t[words]), fc(new uint32_t[fcw + 1]), mw(new uint32_t[64]);
    std::unique_ptr<uint16_t[]> me(new uint16_t[QCAP]);
    std::unique_ptr<float[]> dz(new float[nvalid]);
    uint32_t ps[33] = {}, sel[64];
    for (uint32_t j = 0; j <= k; ++j) ps[j] = (uint32_t)(((uint64_t)j * m) / k);
    for (uint32_t w = 0; w < words; ++w) {
        filt[w] = 0;
        for (uint32_t b = 0; b < 32; ++b) filt[w] |= (uint32_t)((rng() & 0xffff) < fill * 0x10000) << b;
    }
    std::copy(filt.get(), filt.get() + fcw, fc.get());
    fc[fcw] = 0xffffffffu;
    for (uint32_t w = 0; w < 64; ++w) {
        sel[w] = 0;  // the sender's selection, in range
        if (MODE == Q_ENCODE)
            for (uint32_t b = 0; b < 32; ++b) sel[w] |= (uint32_t)(32 * w + b < nvalid && rng() % 4 == 0) << b;
        mw[w] = sel[w];
    }
    std::fill(dz.get(), dz.get() + nvalid, 5.0f);
    const ProbeFilter f{fc.get(), ps, buffer_view(filt.get(), m / 8), m, k, fcw * 32, J};
    const bool all_lds = f.lim >= m;
    emu_launch(1, 64, [&] {
        // the choice of probe_take
        if (all_lds && !part && J != 0)
            probe_window<MODE, PK_LDS>(f, me.get(), mw.get(), wbase, nvalid, dz.get());
        else if (J != 0 && !part)
            probe_window<MODE, PK_STANDARD>(f, me.get(), mw.get(), wbase, nvalid, dz.get());
        else if (J != 0)
            probe_window<MODE, PK_PARTITIONED>(f, me.get(), mw.get(), wbase, nvalid, dz.get());
        else if (part)
            probe_single<MODE, PK_PARTITIONED>(f, me.get(), mw.get(), wbase, nvalid, dz.get());
        else
            probe_single<MODE, PK_STANDARD>(f, me.get(), mw.get(), wbase, nvalid, dz.get());
    });
    const PosMap pm{m, part ? ps : nullptr};
    uint32_t bad = 0, pos = 0;
    for (uint32_t e = 0; e < 2048; ++e) {
        bool all = e < nvalid;
        for (uint32_t j = 0; j < k && all; ++j) {
            const uint32_t p = pm(mm3_key(wbase + e), j);
            all = (filt[p >> 5] >> (p & 31)) & 1;
        }
        all |= (sel[e >> 5] >> (e & 31)) & 1;
        pos += all;
        bad += all != (bool)((mw[e >> 5] >> (e & 31)) & 1);
        bad += MODE == Q_DECODE && e < nvalid && dz[e] != 0.0f;
    }
    ++runs;
    if (bad) {
        ++failures;
        printf("FAIL mode %d m %u k %u lds %u part %d J %u nvalid %u: %u wrong (%u positives)\n", MODE, m, k, fcw, part, J,
               nvalid, bad, pos);
    }
}

// usage: k layout
int main(int, char **argv) {
    const uint32_t k = atoi(argv[1]);
    const bool part = atoi(argv[2]) != 0;
    const uint32_t m = 3 * 4096 + 32;
    const uint32_t lds[3] = {m / 32, m / 80, 16};
    for (uint32_t words : lds) {
        // a group of J hashes, 0 one at a time: what probe_hashes may give
        for (uint32_t J : {0u, 1u, 2u, 3u, 4u}) {
            const bool all = words * 32 >= m && !part;
            if (J > k || (J == 1 && !(all && k == 1)) || (J > 2 && (all || part))) continue;
            one<Q_DECODE>(m, k, words, part, J, 1200, 0.5);
            one<Q_DECODE>(m, k, words, part, J, 1025, 0.93);  // the queue overflows
            one<Q_ENCODE>(m, k, words, part, J, 513, 0.8);
            one<Q_PLAIN>(m, k, words, part, J, 1, 1.0);
        }
    }
    // the rule: a group of at most k, of two at least where memory is read
    for (uint32_t lim : {0u, 1u << 12, 1u << 18, 1u << 20, 1u << 22})
        for (uint32_t mm : {32u, 1u << 14, 1u << 20, (1u << 20) + 32, 1u << 23, 1u << 27, 0xffffffe0u})
            for (uint32_t d : {1u, 512u, 513u, 1u << 20, 0xffffffffu})
                for (uint32_t steps : {8u, 95u, 96u, 511u, 512u, 1u << 20}) {
                    const uint32_t l = std::min(lim, mm), J = probe_hashes(mm, k, l, part ? 1u : 0u, d, steps);
                    if (J > k || J > 4 || (part && J > 2) || (J == 1 && (k != 1 || l < mm || part))) {
                        ++failures;
                        printf("FAIL rule m %u k %u lim %u part %d d %u steps %u: %u\n", mm, k, l, part, d, steps, J);
                    }
                }
    printf("%s: %u of %u runs\n", failures ? "FAIL" : "OK", failures, runs);
    return failures ? 1 : 0;
}
