// The panel loads of the FP32 and 16-bit tiles and of the byte packs, run on the
// CPU over matrices in exactly sized buffers: the sanitizer sees every read, and
// what they deliver is checked element by element.  Built with MG_DEVICE as host
// code (see test_panel_loads_host.py); launches nothing.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "tile_bf16.h"
#include "tile_bytes.h"
#include "tile_f32.h"

static long checks = 0;

static void expect(bool ok, const char* what, long a, long b, long c, long d)
{
    ++checks;
    if (!ok) {
        std::fprintf(stderr, "%s: %ld %ld %ld %ld\n", what, a, b, c, d);
        std::exit(1);
    }
}

struct Matrix {
    int64_t ld;
    std::vector<float> x;
    Matrix(int64_t R, int64_t C, int64_t pad) : ld(C + pad), x(size_t((R - 1) * ld + C))
    {
        for (size_t i = 0; i < x.size(); ++i) x[i] = float(i + 1);
    }
};

// Every thread's panel at (mn0, k0), through the pack into LDS.
template <int B, int BK, int NT, bool KMAJOR>
static void fp32(int64_t MN, int64_t K, int64_t pad)
{
    const Matrix m(KMAJOR ? K : MN, KMAJOR ? MN : K, pad);
    const bool vec = (KMAJOR ? MN : K) >= 4;
    std::vector<float> lds(size_t(B) * BK);
    for (int64_t mn0 = 0; mn0 < MN; mn0 += B)
        for (int64_t k0 = 0; k0 < K; k0 += BK) {
            for (int t = 0; t < NT; ++t) {
                mg::PanelLoader<B, BK, NT, KMAJOR> p;
                p.load(m.x.data(), m.ld, mn0, k0, MN, K, vec, t);
                p.template store<B>(lds.data(), t);
            }
            for (int k = 0; k < BK; ++k)
                for (int i = 0; i < B; ++i) {
                    const float got = lds[size_t(k * B + (i ^ mg::panel_swizzle<BK, B>(k)))];
                    const int64_t r = KMAJOR ? k0 + k : mn0 + i, c = KMAJOR ? mn0 + i : k0 + k;
                    if (k0 + k >= K) expect(got == 0.f, "fp32 beyond K", MN, K, mn0 + i, k0 + k);
                    else if (mn0 + i < MN) expect(got == m.x[size_t(r * m.ld + c)], "fp32", MN, K, mn0 + i, k0 + k);
                }
        }
}

template <int ROWS, int BK, int NT, bool KSRC>
static void sixteen_bit(int64_t MN, int64_t K, int64_t pad)
{
    using P = mg::BfPanel<ROWS, BK, BK + 8, NT, KSRC, 1>;
    const Matrix m(KSRC ? MN : K, KSRC ? K : MN, pad);
    const bool vec = (KSRC ? K : MN) >= 4;
    for (int64_t mn0 = 0; mn0 < MN; mn0 += ROWS)
        for (int64_t k0 = 0; k0 < K; k0 += BK)
            for (int t = 0; t < NT; ++t) {
                P p;
                p.load(m.x.data(), m.ld, mn0, k0, MN, K, vec, P::offsets(m.ld, mn0, MN, t), t);
                for (int s = 0; s < P::LOADS; ++s)
                    for (int e = 0; e < 4; ++e) {
                        const int q = t + (KSRC ? s : s >> 2) * NT;
                        if (q >= (KSRC ? P::CHUNKS : P::BLOCKS)) continue;
                        const int64_t mn = mn0 + (KSRC ? mg::row_perm(q / (BK / 4)) : 4 * (q / (BK / 4)) + e);
                        const int64_t k = k0 + (KSRC ? 4 * (q % (BK / 4)) + e : 4 * (q % (BK / 4)) + (s & 3));
                        const float want = k < K && mn < MN ? m.x[size_t(KSRC ? mn * m.ld + k : k * m.ld + mn)] : 0.f;
                        if (k >= K || mn < MN) expect(p.v[s][e] == want, "16-bit", MN, K, mn, k);
                    }
            }
}

static void bytes(int64_t R, int64_t C, int64_t pad)
{
    const int64_t ld = C + pad;
    std::vector<uint8_t> x(size_t((R - 1) * ld + C));
    for (size_t i = 0; i < x.size(); ++i) x[i] = uint8_t(1 + i % 251);
    for (int64_t r0 = 0; r0 < R + 128; r0 += 128)
        for (int64_t c0 = 0; c0 < C + 128; c0 += 128) {
            const mg::Valid v = mg::valid_part(r0, c0, R, C, 16);
            for (int r = 0; r < 128; r += 3)
                for (int c = 0; c < 128; c += 16) {
                    const auto* at = reinterpret_cast<const uint8_t*>(reinterpret_cast<uintptr_t>(x.data()) + uintptr_t(r0 * ld + c0));
                    const mg::uintx4 w = mg::edge_fix_bytes(mg::edge_load_bytes(at, ld, r, c, v), r, c, v);
                    for (int e = 0; e < 16; ++e) {
                        const bool in = r0 + r < R && c0 + c + e < C;
                        const unsigned want = in ? x[size_t((r0 + r) * ld + c0 + c + e)] : 0u;
                        expect(((w[e >> 2] >> (8 * (e & 3))) & 255u) == want, "bytes", R, C, r0 + r, c0 + c + e);
                    }
                }
        }
}

int main()
{
    const int64_t mns[] = {1, 3, 4, 5, 31, 32, 33, 64, 65, 127, 130}, ks[] = {1, 3, 4, 15, 16, 17, 32, 33, 63, 64, 66};
    for (int64_t mn : mns)
        for (int64_t k : ks)
            for (int64_t pad = 0; pad < 3; ++pad) {
                fp32<32, 32, 64, true>(mn, k, pad);
                fp32<32, 32, 64, false>(mn, k, pad);
                fp32<64, 32, 256, true>(mn, k, pad);
                fp32<64, 32, 256, false>(mn, k, pad);
                fp32<128, 32, 512, true>(mn, k, pad);
                fp32<128, 32, 512, false>(mn, k, pad);
                fp32<256, 16, 512, true>(mn, k, pad);
                fp32<256, 16, 512, false>(mn, k, pad);
                sixteen_bit<64, 32, 256, true>(mn, k, pad);
                sixteen_bit<64, 32, 256, false>(mn, k, pad);
                sixteen_bit<128, 32, 512, true>(mn, k, pad);
                sixteen_bit<128, 32, 512, false>(mn, k, pad);
            }
    const int64_t rs[] = {1, 2, 5, 127, 128, 130}, cs[] = {1, 3, 15, 16, 17, 33, 127, 128, 129, 160};
    for (int64_t r : rs)
        for (int64_t c : cs)
            for (int64_t pad = 0; pad < 4; ++pad) bytes(r, c, pad);
    std::printf("%ld checks\n", checks);
    return 0;
}
