// Host build of the piece and list arithmetic of the packed FP16 tiles (csrc/lba_piece_index.h, lba_list_index.h) under the address and
// undefined-behaviour sanitizers: every address stays inside its operand and every piece holds the codes that the definition
// (64-bit indices, one byte at a time) gives.  Operands of 2 GiB and more are reserved address space of which only the rows
// under test are ever written.  tests/test_sanitizers_cpu.py compiles and runs it, one check at a time; nothing touches a GPU.
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include <vector>

#include "lba_list_index.h"
#include "lba_piece_index.h"

static int failures = 0;
#define CHECK(cond, ...) do { if (!(cond) && ++failures < 20) { std::printf("FAIL %s:%d: ", __FILE__, __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)

static uint64_t rng_state = 0x9E3779B97F4A7C15ull;
static uint32_t rnd32() {                                      // xorshift64*
    rng_state ^= rng_state >> 12; rng_state ^= rng_state << 25; rng_state ^= rng_state >> 27;
    return (uint32_t)((rng_state * 0x2545F4914F6CDD1Dull) >> 32);
}
static int below(int n) { return (int)(rnd32() % (uint32_t)n); }

struct Words { uint32_t x, y, z, w; };
static Words load(const uint8_t* a) { Words v; std::memcpy(&v, a, 16); return v; }

struct Operand {                                               // zero bytes until written; an access outside it faults
    uint8_t* base; size_t bytes, span;
    explicit Operand(size_t n) : bytes(n), span((n + 4095) / 4096 * 4096) {
        base = (uint8_t*)mmap(nullptr, span + 8192, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (base == MAP_FAILED || mprotect(base + 4096, span, PROT_READ | PROT_WRITE) != 0) { std::perror("mmap"); std::exit(3); }
        base += 4096;
    }
    ~Operand() { munmap(base - 4096, span + 8192); }
    Operand(const Operand&) = delete;
    void fill(size_t at, size_t n) { for (size_t i = at; i < at + n && i < bytes; ++i) base[i] = (uint8_t)(1 + below(255)); }
};

static const int kRows = 64;

// every piece of one row over the tiles [t0, t1): the matrix [rows][K] at op.base + off
static void check_row(const Operand& op, size_t off, int rows, int K, int r, int t0, int t1) {
    const uint8_t* G = op.base + off;
    const int ntiles = (int)(((int64_t)K + 63) / 64);
    for (int q = 0; q < 4; ++q) {
        const lba::RowPieces<kRows> s(G, rows, K, r / kRows * kRows, r % kRows + kRows * q);
        for (int t = t0; t < t1; ++t) {
            const uint8_t* a = s.address(lba::tile_start(t));
            const bool in = a >= G && a + 16 <= G + (int64_t)rows * K;
            CHECK(in, "rows %d K %d row %d tile %d of %d piece %d: loads at %lld", rows, K, r, t, ntiles, q, (long long)(a - G));
            if (!in || t >= ntiles) continue;                  // (a tile past the last one is fetched and dropped)
            const Words got = s.codes(load(a), t * 64);
            uint8_t want[16] = {};
            for (int j = 0; j < 16; ++j) {
                const int64_t k = (int64_t)t * 64 + 16 * q + j;
                if (r < rows && k < K) want[j] = G[(int64_t)r * K + k];
            }
            CHECK(std::memcmp(&got, want, 16) == 0, "rows %d K %d row %d tile %d piece %d: wrong codes", rows, K, r, t, q);
        }
    }
}

// rows at every distance from the operand's end, up to 4.5 GB
static void far_rows() {
    const int shapes[][2] = {{16000000, 147}, {33554435, 136}, {6, 3}, {1, 17}, {70, 64}, {300, 83}, {2, 1000}, {40000000, 113}};
    for (const auto& sh : shapes) {
        const int rows = sh[0], K = sh[1], ntiles = (K + 63) / 64;
        for (int off : {0, 5}) {
            Operand op((size_t)rows * K + off);
            std::vector<int> rs = {0, 1, 63, 64, rows / 2, rows - 2, rows - 1, rows};
            for (int64_t d : {1LL << 30, 1LL << 31, 3LL << 30, 1LL << 32})
                for (int e = -2; e <= 2; ++e) rs.push_back((int)(((int64_t)rows * K - d) / K + e));
            for (int i = 0; i < 60; ++i) rs.push_back(below(rows));
            for (int r : rs) {
                if (r < 0 || r > rows) continue;               // r == rows: a lane beyond the matrix
                op.fill((size_t)r * K + off, (size_t)K + 16);
                check_row(op, (size_t)off, rows, K, r, 0, ntiles + 2);
            }
        }
    }
}

// chains up to the longest, K = 2^31 - 64, that the planner gives to the packed tiles: the last tiles and the ones fetched ahead
// beyond them (the small lane blocks keep four tiles in flight: up to tile ntiles + 3).  M = N = 1 runs on those blocks.
static void long_chains() {
    int packed = 0, plain = 0;
    for (int d : {0, 1, 15, 16, 63, 64, 65, 127, 128, 190, 255, 256, 257, 300, 1000})
        for (int rows : {1, 2}) {
            const int K = 2147483584 - d, ntiles = (int)(((int64_t)K + 63) / 64);
            lba::Plan pl;
            const lba_qfmt qp = {5, 7, 12, 0}, qa = {4, 7, 7, 0};
            CHECK(lba::make_plan(rows, rows, K, qp, qa, LBA_ORDER_SEQ, 0, &pl) == LBA_OK && pl.kernel == lba::KERNEL_FAST, "plan of K = %d", K);
            ++(pl.kp.h_on ? packed : plain);
            if (!pl.kp.h_on) continue;
            Operand op((size_t)rows * K);
            for (int r = 0; r <= rows; ++r) {
                if (r < rows) { op.fill((size_t)r * K, 300); op.fill((size_t)(r + 1) * K - 300, 300); }
                check_row(op, 0, rows, K, r, 0, 6);
                check_row(op, 0, rows, K, r, ntiles - 3, ntiles + 4);
            }
        }
    CHECK(packed == 8 && plain == 22, "%d plans on packed carriers, %d not", packed, plain);
}

// im2col rows of an NHWC tensor: every piece of every row of the tile rows at r0
static void check_conv(const Operand& op, size_t off, int n, int h, int w, int c, int kh, int kw, int stride, int pad) {
    const uint8_t* X = op.base + off;
    const int64_t oh = ((int64_t)h + 2 * (int64_t)pad - kh) / stride + 1, ow = ((int64_t)w + 2 * (int64_t)pad - kw) / stride + 1;
    const int64_t total = (int64_t)n * h * w * c;
    lba::KParams p = {};
    p.M = (int32_t)(n * oh * ow); p.K = kh * kw * c;
    p.conv = 1; p.cv_h = h; p.cv_w = w; p.cv_c = c; p.cv_kw = kw; p.cv_stride = stride; p.cv_pad = pad; p.cv_oh = (int32_t)oh; p.cv_ow = (int32_t)ow;
    p.cv_vec = (c % 16 == 0 && (uintptr_t)X % 16 == 0) ? 1 : 0;
    p.cv_magic_c = (((uint64_t)1 << 40) + (uint64_t)c - 1) / (uint64_t)c;
    p.cv_magic_kw = (((uint64_t)1 << 40) + (uint64_t)kw - 1) / (uint64_t)kw;
    const int ntiles = (p.K + 63) / 64;
    for (int r = 0; r <= p.M; ++r) {
        if (r > 300 && r < p.M - 100) continue;
        for (int q = 0; q < 4; ++q) {
            const lba::ConvPieces s = lba::ConvPieces::make<kRows>(X, p, r / kRows * kRows, r % kRows + kRows * q);
            for (int t = 0; t < ntiles + 4; ++t) {
                if (t > 40 && t < ntiles - 3) continue;
                const int k0 = lba::tile_start(t);
                const uint8_t* a = s.first(p, k0);
                const uint8_t* b = p.cv_vec ? a : s.second(p, k0);
                const bool in = a >= X && a + 16 <= X + total && b >= X && b + 16 <= X + total;
                CHECK(in, "%dx%dx%dx%d kw %d stride %d pad %d row %d tile %d: loads at %lld and %lld", n, h, w, c, kw, stride, pad, r, t,
                      (long long)(a - X), (long long)(b - X));
                if (!in || t >= ntiles) continue;
                const Words got = s.codes(p, load(a), load(b), k0);
                uint8_t want[16] = {};
                for (int j = 0; j < 16; ++j) {
                    const int64_t k = (int64_t)t * 64 + 16 * q + j, tap = k / c;
                    if (r >= p.M || k >= p.K) continue;
                    const int64_t ih = r / ow % oh * stride - pad + tap / kw, iw = r % ow * stride - pad + tap % kw;
                    if (ih >= 0 && ih < h && iw >= 0 && iw < w) want[j] = X[((r / (oh * ow) * h + ih) * w + iw) * c + k % c];
                }
                CHECK(std::memcmp(&got, want, 16) == 0, "%dx%dx%dx%d kw %d stride %d pad %d row %d tile %d piece %d: wrong codes", n, h, w, c,
                      kw, stride, pad, r, t, q);
            }
        }
    }
}

// padding far beyond the image: distances in codes of 2^31 and more, output rows up to w + pad codes to the right of it
static void wide_padding() {
    for (int c : {1, 3, 5, 17, 1000, 16368, 16383})
        for (int kw : {1, 2, 3, 7})
            for (int64_t pad : {(1LL << 31) / c - 1, (1LL << 31) / c + 1, (1LL << 32) / c - 2, (1LL << 32) / c + 3, (1LL << 31) - 1}) {
                if (pad > 2147483647LL) continue;
                Operand op((size_t)2 * 3 * 4 * c + 32);
                op.fill(0, (size_t)2 * 3 * 4 * c + 32);
                for (int64_t stride : {pad, pad / 2 + 1, pad - 1})
                    for (int off : {0, 1}) check_conv(op, (size_t)off, 2, 3, 4, c, 2, kw, (int)stride, (int)pad);
            }
    Operand row((size_t)2147483647);                           // the widest image
    row.fill(0, 64);
    row.fill(2147483647u - 64, 64);
    for (int kw : {1, 3, 16, 20})
        for (int pad : {0, 1, 2147483647})
            for (int stride : {2147483647, 2147483646, 1 << 30}) check_conv(row, 0, 1, 1, 2147483647, 1, 1, kw, stride, pad);
}

// ordinary convolutions, some thousand
static void convolutions() {
    for (int i = 0; i < 3000; ++i) {
        const int n = 1 + below(3), h = 1 + below(12), w = 1 + below(12), kh = 1 + below(5), kw = 1 + below(8);
        const int c = (const int[]){1, 2, 3, 4, 5, 8, 15, 16, 17, 32, 48}[below(11)], pad = below(6), stride = 1 + below(3), off = below(2) * below(16);
        if (h + 2 * pad < kh || w + 2 * pad < kw || n * h * w * c < 16) continue;
        Operand op((size_t)n * h * w * c + off);
        op.fill(0, op.bytes);
        check_conv(op, (size_t)off, n, h, w, c, kh, kw, stride, pad);
    }
}

// lists of non-zero codes of every length over one row of a row tile, after a tile or a longer list whose words stay behind: every
// entry that serves as an address was written by the list or the pad, its row of B lies inside a stage, and no read leaves the row
template <int RW, int TN>
static void check_lists() {
    using T = lba::RowTile<RW, TN>;
    for (int len = 0; len <= 64; ++len) {
        std::vector<int64_t> row((size_t)T::PITCH, -1);        // -1: never written
        for (int l = 0; l < 4; ++l) lba::pad_row<T>(l, [&](int w) { CHECK(w >= 64 && w < T::PITCH, "pad word %d", w); row.at((size_t)w) = 0; });
        for (int w = 0; w < 64; ++w) row[(size_t)w] = (int64_t)((w < len ? 0x3C00 + w : 0) | (uint32_t)(T::B_WORDS * 4 + w * T::BROW * 4) << 16);
        const int n = (len + T::U - 1) & ~(T::U - 1);
        int next = 0;
        const auto round = [&](int i) {
            CHECK(i == next, "round at %d, not %d", i, next);
            for (int u = 0; u < T::U; ++u) {                   // the rows asked for: entries i + U ..., read two rounds ago
                const int64_t e = row.at((size_t)(i + T::U + u));
                CHECK(e >= 0 && (int)(e >> 16) % (T::BROW * 4) == 0 && (int)(e >> 16) + T::BROW * 4 <= 2 * T::B_WORDS * 4,
                      "list of %d: entry %d is an address and was never written", len, i + T::U + u);
            }
            CHECK(i + 3 * T::U <= T::PITCH, "list of %d: entries read up to %d", len, i + 3 * T::U);
            next += T::U;
        };
        lba::walk_list<T::U>(n, round, round);
        CHECK(next == n, "list of %d: %d entries taken", len, next);
    }
}
static void lists() { check_lists<16, 8>(); check_lists<12, 8>(); check_lists<8, 8>(); check_lists<8, 4>(); check_lists<8, 2>(); }

int main(int argc, char** argv) {
    if (argc != 2) { std::printf("usage: %s <check>\n", argv[0]); return 2; }
    if (!std::strcmp(argv[1], "far_rows")) far_rows();
    else if (!std::strcmp(argv[1], "long_chains")) long_chains();
    else if (!std::strcmp(argv[1], "convolutions")) convolutions();
    else if (!std::strcmp(argv[1], "wide_padding")) wide_padding();
    else if (!std::strcmp(argv[1], "lists")) lists();
    else { std::printf("no such check\n"); return 2; }
    if (failures) { std::printf("%d failures\n", failures); return 1; }
    std::printf("pieces ok\n");
    return 0;
}
