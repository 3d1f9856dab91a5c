// Host-side ABI checks run under AddressSanitizer and UndefinedBehaviorSanitizer:
// argument validation of every entry point (fake device pointers that are never
// dereferenced; the launch stubs abort if anything is launched) and the
// hybrid-aware partition, whose exact rounding runs big-integer arithmetic.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "launch_stubs.hpp"
#include "stateflow.h"

static int failures = 0;
#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) {                                                      \
            std::fprintf(stderr, "%s:%d: FAILED %s\n", __FILE__, __LINE__, #cond); \
            ++failures;                                                     \
        }                                                                   \
    } while (0)

static void *P(int i) { return (void *)(uintptr_t)(0x7F0000000000ull + (uint64_t)i * (1ull << 32)); }
static float *F(int i) { return (float *)P(i); }

static sf_shape shape(int64_t L = 1024) {
    sf_shape s;
    std::memset(&s, 0, sizeof s);
    s.B = 1, s.H = 2, s.Dk = 128, s.Dv = 128, s.L = L, s.chunk = 64, s.io_dtype = SF_BF16, s.gate = SF_GATE_SCALAR;
    return s;
}

// A chain of small segments goes out as one set of launches whose superchunks cover
// every segment's chunks in order, cross no segment's end and are no longer than
// those the segment would take in a call of its own.
static void check_merged(int B, int H, int D, int gate, const std::vector<int64_t> &len, int ts) {
    int64_t L = 0;
    for (int64_t x : len) L += x;
    sf_shape s = shape(L);
    s.B = B, s.H = H, s.Dk = s.Dv = D, s.gate = gate;
    sf_tuning t;
    std::memset(&t, 0, sizeof t);
    t.ts = ts;
    const int n = (int)len.size();
    sf::LaunchRecord rec, one;
    sf::launch_record = &rec;
    EXPECT(sf_chain_fwd(&s, n, len.data(), P(1), P(2), P(3), F(4), P(5), F(6), nullptr, 0, P(7), 1 << 30, &t, nullptr,
                        nullptr) == SF_OK);
    EXPECT(rec.seg.size() == 3);
    EXPECT(sf_chain_bwd(&s, n, len.data(), P(1), P(2), P(3), F(4), F(5), nullptr, 0, P(6), nullptr, P(8), P(9), P(10),
                        F(11), F(12), P(13), 1 << 30, &t, nullptr, nullptr) == SF_OK);
    EXPECT(rec.seg.size() == 7);
    sf::launch_record = &one;
    for (const auto &launch : rec.seg) {
        const sf::SegArgs &a = launch.second;
        EXPECT(a.n_seg == n && a.seg_sc[0] == 0 && a.seg_ck[0] == 0 && a.seg_sc[n] == a.n_super);
        for (int i = 0; i < n; ++i) {
            const int64_t nc = len[i] / 64, ns = a.seg_sc[i + 1] - a.seg_sc[i];
            EXPECT(a.seg_ck[i + 1] - a.seg_ck[i] == nc && a.seg_m[i] > 0);
            EXPECT(ns * a.seg_m[i] >= nc && (ns - 1) * a.seg_m[i] < nc);
            sf_shape si = s;
            si.L = len[i];
            EXPECT(sf_segment_fwd(&si, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) == SF_OK);
            const sf::SegArgs &b = one.seg.back().second;
            EXPECT(a.seg_m[i] * 64 <= (b.ts < len[i] ? b.ts : len[i]));
        }
    }
    sf::launch_record = nullptr;
}

// Launches of a chain's two directions, and the bytes it keeps.
static void check_form(int H, int D, int io, int gate, int n, int chunks, bool fwd_one, bool bwd_one) {
    const std::vector<int64_t> len(n, 64 * chunks);
    sf_shape s = shape((int64_t)n * 64 * chunks);
    s.B = 1, s.H = H, s.Dk = s.Dv = D, s.io_dtype = io, s.gate = gate;
    sf::LaunchRecord rec;
    sf::launch_record = &rec;
    EXPECT(sf_chain_fwd(&s, n, len.data(), P(1), P(2), P(3), F(4), P(5), F(6), nullptr, 0, P(7), 1ull << 40, nullptr, nullptr,
                        nullptr) == SF_OK);
    EXPECT(rec.seg.size() == (fwd_one ? 3 : (size_t)n));
    rec.seg.clear();
    EXPECT(sf_chain_bwd(&s, n, len.data(), P(1), P(2), P(3), F(4), F(5), nullptr, 0, P(6), nullptr, P(8), P(9), P(10),
                        F(11), F(12), P(13), 1ull << 40, nullptr, nullptr, nullptr) == SF_OK);
    EXPECT(rec.seg.size() == (bwd_one ? 4 : 2 * (size_t)n));
    sf::launch_record = nullptr;
    // segments of one superchunk, segment by segment: nothing to keep, and no states in the workspace
    const size_t state = (size_t)H * D * D * 4;
    EXPECT((sf_chain_ckpt_bytes(&s, n, len.data(), nullptr) == 0) == !fwd_one);
    EXPECT((sf_chain_workspace_bytes(&s, n, len.data(), nullptr) < 3 * state) == !bwd_one);
}

int main() {
    for (int gate : {SF_GATE_SCALAR, SF_GATE_VECTOR})
        for (int H : {1, 2, 6, 16}) {
            check_merged(1, H, 128, gate, {1984, 1088, 4160}, 0);
            check_merged(1, H, 64, gate, {1984, 1088, 4160}, 0);
            check_merged(1, H, 128, gate, {64, 8192, 192, 64, 2048}, 0);
            check_merged(2, H, 128, gate, std::vector<int64_t>(32, 512), 0);
            check_merged(1, H, 128, gate, {192, 64, 320, 128}, 64);
        }
    // segments of one superchunk each, on 256 CUs, either side of each line: in one (3
    // and 4 launches) or segment by segment (1 and 2 a segment)
    struct { int H, D, io, gate, n, chunks; bool one; } forms[] = {
        {112, 128, SF_BF16, SF_GATE_SCALAR, 16, 1, true},  {113, 128, SF_BF16, SF_GATE_SCALAR, 16, 1, false},
        {128, 128, SF_BF16, SF_GATE_SCALAR, 32, 8, false}, {128, 128, SF_BF16, SF_GATE_VECTOR, 16, 8, true},
        {129, 128, SF_BF16, SF_GATE_VECTOR, 16, 1, false}, {208, 64, SF_F32, SF_GATE_SCALAR, 8, 1, true},
        {209, 64, SF_F32, SF_GATE_SCALAR, 16, 1, false},   {160, 64, SF_F32, SF_GATE_SCALAR, 4, 1, true},
        {161, 64, SF_F32, SF_GATE_SCALAR, 4, 1, false},    {208, 64, SF_BF16, SF_GATE_VECTOR, 16, 1, true},
        {128, 64, SF_F32, SF_GATE_VECTOR, 16, 1, true},    {129, 64, SF_F32, SF_GATE_VECTOR, 16, 1, false},
        {129, 64, SF_F32, SF_GATE_SCALAR, 2, 1, false},    {100, 128, SF_BF16, SF_GATE_SCALAR, 2, 4, true},
        {33, 128, SF_BF16, SF_GATE_SCALAR, 33, 1, false}};
    for (const auto &f : forms)
        check_form(f.H, f.D, f.io, f.gate, f.n, f.chunks, f.one, f.one);
    // two of one chunk: forward segment by segment, backward in one
    for (int gate : {SF_GATE_SCALAR, SF_GATE_VECTOR}) check_form(5, 64, SF_F32, gate, 2, 1, false, true);

    sf_tuning t;
    std::memset(&t, 0, sizeof t);
    t.ts = 128;
    sf_shape s = shape();
    // segment forward
    EXPECT(sf_segment_fwd(nullptr, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) == SF_E_NULL);
    sf_shape bad = shape(100);
    EXPECT(sf_segment_fwd(&bad, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) == SF_E_SHAPE);
    bad = shape();
    bad.Dk = 96, bad.Dv = 96;
    EXPECT(sf_segment_fwd(&bad, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) ==
           SF_E_UNSUPPORTED);
    bad = shape();
    bad.io_dtype = 7;
    EXPECT(sf_segment_fwd(&bad, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) == SF_E_DTYPE);
    EXPECT(sf_segment_fwd(&s, (char *)P(1) + 2, P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) ==
           SF_E_ALIGN);
    EXPECT(sf_segment_fwd(&s, P(1), P(2), P(3), F(4), nullptr, P(1), F(6), P(7), 1 << 30, &t, nullptr) == SF_E_ALIAS);
    EXPECT(sf_segment_fwd(&s, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(5), 1 << 30, &t, nullptr) == SF_E_ALIAS);
    EXPECT(sf_segment_fwd(&s, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 16, &t, nullptr) == SF_E_WORKSPACE);
    EXPECT(std::strlen(sf_last_error()) > 0);
    // segment backward
    EXPECT(sf_segment_bwd(&s, P(1), P(2), P(3), F(4), nullptr, P(6), nullptr, P(8), P(9), P(10), F(11), F(12), P(8),
                          1 << 30, &t, nullptr) == SF_E_ALIAS);
    EXPECT(sf_segment_bwd(&s, P(1), P(2), P(3), F(4), nullptr, P(6), nullptr, P(8), P(9), P(10), F(11), nullptr,
                          P(13), 1 << 30, &t, nullptr) == SF_E_NULL);
    // chains
    const int64_t segs[2] = {512, 448};
    EXPECT(sf_chain_fwd(&s, 2, segs, P(1), P(2), P(3), F(4), P(5), F(6), nullptr, 0, P(7), 1 << 30, nullptr, nullptr, nullptr) ==
           SF_E_SHAPE);
    const int64_t segs2[2] = {512, 512};
    EXPECT(sf_chain_fwd(&s, 2, segs2, P(1), P(2), P(3), F(4), P(5), F(6), nullptr, 0, P(5), 1 << 30, nullptr, nullptr, nullptr) ==
           SF_E_ALIAS);
    EXPECT(sf_chain_bwd(&s, 2, segs2, P(1), P(2), P(3), F(4), F(5), nullptr, 0, P(6), nullptr, P(8), P(9), P(10), F(11), nullptr,
                        P(13), 1 << 30, nullptr, nullptr, nullptr) == SF_E_NULL);
    EXPECT(sf_chain_workspace_bytes(&s, 2, segs2, nullptr) > 0);
    EXPECT(sf_chain_workspace_bytes(&s, 2, segs, nullptr) == 0);
    // kept superchunk states
    sf_tuning t128;
    std::memset(&t128, 0, sizeof t128);
    t128.ts = 128;
    const size_t kneed = sf_chain_ckpt_bytes(&s, 2, segs2, &t128);
    EXPECT(kneed > 0);
    EXPECT(sf_chain_ckpt_bytes(&s, 2, segs, &t128) == 0 && std::strlen(sf_last_error()) > 0);
    EXPECT(sf_chain_fwd(&s, 2, segs2, P(1), P(2), P(3), F(4), P(5), F(6), P(8), kneed - 1, P(7), 1 << 30, &t128,
                        nullptr, nullptr) == SF_E_WORKSPACE);
    EXPECT(sf_chain_bwd(&s, 2, segs2, P(1), P(2), P(3), F(4), F(5), P(8), kneed, P(6), nullptr, P(8), P(9), P(10),
                        F(11), F(12), P(13), 1 << 30, &t128, nullptr, nullptr) == SF_E_ALIAS);
    // timing record
    sf_timing tm;
    std::memset(&tm, 0, sizeof tm);
    tm.capacity = 4, tm.count = 5;
    t.timing = &tm;
    EXPECT(sf_segment_fwd(&s, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) == SF_E_SHAPE);
    tm.count = 0;
    EXPECT(sf_segment_fwd(&s, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), P(7), 1 << 30, &t, nullptr) == SF_E_NULL);
    t.timing = nullptr;
    // allocation-free forward: oversized shapes are rejected before any launch
    sf_shape big = shape(65536);
    big.H = 40;
    sf_tuning t64;
    std::memset(&t64, 0, sizeof t64);
    t64.ts = 64;
    EXPECT(sf_segment_fwd_noalloc(&big, P(1), P(2), P(3), F(4), nullptr, P(5), F(6), &t64, nullptr) == SF_E_WORKSPACE);
    // short convolution
    sf_conv_shape c;
    std::memset(&c, 0, sizeof c);
    c.B = 2, c.C = 64, c.L = 1000, c.W = 4, c.io_dtype = SF_BF16, c.act = SF_ACT_SILU;
    EXPECT(sf_conv_fwd(&c, P(1), F(2), F(3), P(1), F(5), nullptr, nullptr) == SF_E_ALIAS);
    c.C = 12;
    EXPECT(sf_conv_fwd(&c, P(1), F(2), F(3), P(4), F(5), nullptr, nullptr) == SF_E_UNSUPPORTED);
    c.C = 64;
    EXPECT(sf_conv_bwd(&c, P(1), F(2), F(3), P(4), F(5), P(6), F(7), F(8), P(9), 16, nullptr, nullptr) ==
           SF_E_WORKSPACE);
    // few channels and many tokens: shortened runs may come in more than 65535 blocks,
    // whole ones (and so the call) may not
    for (int ch : {8, 16, 24}) {
        sf::LaunchRecord rec;
        sf::launch_record = &rec;
        c.B = 1, c.C = ch;
        for (int64_t L : {int64_t(524280), int64_t(524296), int64_t(1 << 20), int64_t(65535) * 256}) {
            c.L = L;
            EXPECT(sf_conv_fwd(&c, P(1), F(2), F(3), P(4), F(5), nullptr, nullptr) == SF_OK);
            const sf::ConvArgs &a = rec.conv.back();
            EXPECT(a.nTB * a.T >= L && (a.nTB - 1) * a.T < L);
            EXPECT(a.T == 256 ? a.nTB <= 65535 : a.T >= 8 && a.T < 256);
        }
        EXPECT(rec.conv.size() == 4);
        c.L = int64_t(65535) * 256 + 1;
        EXPECT(sf_conv_fwd(&c, P(1), F(2), F(3), P(4), F(5), nullptr, nullptr) == SF_E_UNSUPPORTED);
        sf::launch_record = nullptr;
    }
    // runs are shortened until the device at hand is full, and no further: an eighth
    // of the CUs need an eighth of the threads
    for (int cus : {32, 64, 256})
        for (int64_t L : {64, 1037, 4096, 65536}) {
            const int64_t groups = 1920 / 8;
            const int64_t T = sf::conv_fwd_run(1, 1920, L, cus), threads = groups * ((L + T - 1) / T);
            EXPECT(T == 256 || groups * ((L + 2 * T - 1) / (2 * T)) < 384 * cus);
            EXPECT(T == 8 || threads >= 384 * cus);
            for (bool b16 : {false, true}) {
                const int64_t whole = groups * ((L + 255) / 256), fill = (b16 ? 384 : 160) * cus;
                const int n = sf::conv_bwd_runs(whole, b16, cus);
                EXPECT((n == 1 || whole * n / 2 < fill) && (n == 32 || whole * n >= fill));
            }
        }
    // gated delta rule
    EXPECT(sf_gdn_fwd(&s, P(1), P(2), P(3), F(4), F(5), nullptr, P(1), F(7), nullptr, P(8), 1ull << 40, nullptr,
                      nullptr) == SF_E_ALIAS);
    EXPECT(sf_gdn_bwd(&s, P(1), P(2), P(3), F(4), F(5), nullptr, P(6), nullptr, P(7), P(8), P(9), F(10), F(11), F(12),
                      P(7), 1ull << 40, nullptr, nullptr) == SF_E_ALIAS);
    EXPECT(sf_gdn_chain_fwd(&s, 2, segs2, P(1), P(2), P(3), F(4), F(5), P(1), F(7), nullptr, 0, nullptr, P(8),
                            1ull << 40, nullptr, nullptr, nullptr) == SF_E_ALIAS);
    const size_t gk = sf_gdn_chain_ckpt_bytes(&s, 2, segs2, &t128);
    EXPECT(gk > 0);
    EXPECT(sf_gdn_chain_fwd(&s, 2, segs2, P(1), P(2), P(3), F(4), F(5), P(6), F(7), P(9), gk - 1, nullptr, P(8),
                            1ull << 40, &t128, nullptr, nullptr) == SF_E_WORKSPACE);
    EXPECT(sf_gdn_chain_bwd(&s, 2, segs2, P(1), P(2), P(3), F(4), F(5), F(7), P(9), gk, P(6), nullptr, P(9), P(10),
                            P(11), F(12), F(13), F(14), P(8), 1ull << 40, &t128, nullptr, nullptr) == SF_E_ALIAS);
    // partition: exact half-way cases round up, irrational boundaries, errors
    int64_t len[8];
    EXPECT(sf_partition_hybrid(384, 2, 0.0, 1.0, 1.0, 128, len) == SF_OK && len[0] == 256 && len[1] == 128);
    EXPECT(sf_partition_hybrid(384, 2, 1.25, 1.0, 0.0, 128, len) == SF_OK && len[0] == 256 && len[1] == 128);
    EXPECT(sf_partition_hybrid(1280, 4, 1.0, 0.0, 1.0, 128, len) == SF_OK && len[0] == 640 && len[1] == 256 &&
           len[2] == 256 && len[3] == 128);
    EXPECT(sf_partition_hybrid(640, 4, 1.0, 0.0, 1e-3, 128, len) == SF_E_SHAPE);
    EXPECT(sf_partition_hybrid(262144, 8, 1.0, 1e-300, 1e300, 128, len) == SF_OK);  // wide exponent gaps
    EXPECT(sf_partition_hybrid(262144, 8, 0.7, 7.5, 4.9e-324, 64, len) == SF_OK);   // a subnormal weight
    EXPECT(sf_partition_hybrid(int64_t(1) << 41, 8, 1.0, 1.0, 0.0, 128, len) == SF_E_SHAPE);
    EXPECT(sf_partition_hybrid(262144, 8, 1.0, 1.0, 1e-5, 128, nullptr) == SF_E_NULL);
    if (failures) std::fprintf(stderr, "%d check(s) failed\n", failures);
    else std::printf("abi checks passed\n");
    return failures ? 1 : 0;
}
