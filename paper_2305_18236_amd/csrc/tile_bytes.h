#pragma once
// Staging of one panel of a pre-packed 8-bit operand (FP8 codes or int8
// values): ROWS rows of a 128-deep K panel, k-contiguous in global memory
// (row stride ldq bytes, zero-padded so no bounds checks are needed), copied
// through registers into LDS rows of LDR bytes.  Eight lanes copy one
// 128-byte row with 16-byte accesses.
#include <type_traits>
#include <utility>

#include "common.h"

namespace mg {

// 16-byte access of bytes at any address.
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uintx4 uintx4u __attribute__((aligned(1)));

// The byte forms of edge_load and edge_fix (common.h): bytes c .. c+15 of row
// r of a block of a byte matrix (src: the block's first byte), where any may
// lie outside; those read 0.
MG_DEVICE uintx4 edge_load_bytes(const uint8_t* __restrict__ src, int64_t ld, int r, int c, Valid b)
{
    const uint8_t* __restrict__ p = src + min(r, b.rows - 1) * ld;
    if (b.wide) return *reinterpret_cast<const uintx4u*>(p + min(c, b.cols - 16));   // uniform
    uintx4 w = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e >> 2] |= uint32_t(p[min(c + e, b.cols - 1)]) << (8 * (e & 3));
    return w;
}

MG_DEVICE uintx4 edge_fix_bytes(uintx4 w, int r, int c, Valid v)
{
    const int left = max(0, min(16, v.cols - c));   // valid columns of the chunk
    const int keep = r < v.rows ? left : 0;
    const int sh = v.wide ? 16 - left : 0;          // how far the chunk was moved left
    uintx4 x = w;
    if (sh & 8) x = uintx4{x[2], x[3], 0, 0};
    if (sh & 4) x = uintx4{x[1], x[2], x[3], 0};
    const int b = 8 * (sh & 3);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint64_t pair = (uint64_t(d < 3 ? x[d + 1] : 0u) << 32) | x[d];
        const int n = keep - 4 * d;   // valid bytes of this word
        x[d] = uint32_t(pair >> b) & (n >= 4 ? 0xffffffffu : n <= 0 ? 0u : (1u << (8 * n)) - 1u);
    }
    return x;
}

template <int ROWS, int NT, int LDR>
struct BytePanel {
    static constexpr int CHUNKS = ROWS * 128 / 16;
    static constexpr int PER = CHUNKS / NT;
    static_assert(CHUNKS % NT == 0, "panels must split evenly");
    uint4 v[PER];

    MG_DEVICE void load(const uint8_t* __restrict__ q, int64_t ldq, int64_t row0, int64_t k0, int tid)
    {
        const uint8_t* __restrict__ base = q + row0 * ldq + k0;
        const uint32_t ld32 = uint32_t(ldq);
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            const uint32_t id = tid + s * NT;
            v[s] = load16u(base, (id / 8) * ld32 + 16 * (id % 8));
        }
    }

    MG_DEVICE void store(uint8_t* lds, int tid) const
    {
#pragma unroll
        for (int s = 0; s < PER; ++s) store_chunk(lds, tid, s);
    }

    // One of the PER 16-byte chunks, so that a caller can spread the LDS
    // writes of a panel between its matrix instructions.
    MG_DEVICE void store_chunk(uint8_t* lds, int tid, int s) const
    {
        const int id = tid + s * NT;
        *reinterpret_cast<uint4*>(&lds[(id / 8) * LDR + 16 * (id % 8)]) = v[s];
    }
};

// Direct form of the byte panels: packed 128-byte k rows copied from global
// memory straight into LDS (global_load_lds_dwordx4: each lane's 16 bytes land
// at the wave's LDS base + 16 * lane), with no register staging and no LDS
// write instructions.  LDS rows are unpadded; since the copy cannot scatter,
// the bank-conflict-free layout is made by choosing the source instead: LDS
// chunk c of row r holds global chunk c ^ direct_swz(r), so 16 consecutive
// rows read at one k fall on 16 distinct 16-byte bank groups.
MG_DEVICE int direct_swz(int r) { return (r >> 1) & 7; }

// Copy ROWS rows of 128 bytes (row stride ld32 from q, k offset k0) into
// `lds`; copy j of wave w fills LDS chunks (j*NW + w)*64 .. +63.
template <int ROWS, int NW>
MG_DEVICE void direct_copy(const uint8_t* __restrict__ q, uint32_t ld32, uint32_t k0, uint8_t* lds, int wave,
                           int lane)
{
    constexpr int J = ROWS * 8 / (NW * 64);
    static_assert(ROWS * 8 % (NW * 64) == 0, "panels must split evenly");
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int slot = (j * NW + wave) * 64 + lane, r = slot >> 3;
        const uint32_t off = uint32_t(r) * ld32 + k0 + 16u * uint32_t((slot & 7) ^ direct_swz(r));
        __builtin_amdgcn_global_load_lds(q + off, lds + (j * NW + wave) * 1024, 16, 0, 0);
    }
}

// The 16 bytes of global chunk g (k bytes 16g .. 16g+15) of LDS row `row`.
MG_DEVICE uint4 direct_chunk(const uint8_t* lds, int row, int g)
{
    return *reinterpret_cast<const uint4*>(lds + row * 128 + 16 * (g ^ direct_swz(row)));
}

// ---- Ring form of the direct copies: NS stages, NS - 1 panels ahead.  Where
// a launch gives a compute unit one workgroup only, nothing else runs while
// it waits for a panel, and the two-buffer form, whose copy has one panel's
// products (about 0.2 us on a 128 x 128 tile) to land in, waits out most of
// each copy's latency.  Here a copy has NS - 1 panels' time.
//
// One barrier per panel: past it every wave's share of panel kt has landed
// (each wave waited for its own copies, and only for those of this panel) and
// every wave is done reading panel kt - 1, whose stage takes the next copy.
template <int... I, class F>
MG_DEVICE void each_of(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// copy(stage, panel): issue this wave's PER copies of a panel into a stage;
// compute(stage, panel): multiply it.  stage: an integral_constant, so that
// each stage can be an array of its own (the compiler then tells the copies
// into one from the reads of another).
template <int NS, int PER, class Copy, class Compute>
MG_DEVICE void ring_loop(int nk, Copy copy, Compute compute)
{
    static_assert((NS - 2) * PER < 64, "the wait counts the copies in flight");
    auto turn = [&](auto stage, int kt, auto more) {
        constexpr bool MORE = decltype(more)::value;
        constexpr int S = decltype(stage)::value;
        constexpr int FLY = MORE ? (NS - 2) * PER : 0;   // copies of newer panels
        // vmcnt(FLY) lgkmcnt(0)
        __builtin_amdgcn_s_waitcnt(0x0070 | (FLY & 15) | (FLY >> 4 << 14));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (MORE) copy(std::integral_constant<int, (S + NS - 1) % NS>{}, kt + NS - 1);
        compute(stage, kt);
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    // (with fewer panels than stages the last one again, for the same reason)
    each_of(std::make_integer_sequence<int, NS - 1>{}, [&](auto s) { copy(s, min(decltype(s)::value, nk - 1)); });
    // NS panels at a time, so that each one's stage is a compile-time choice,
    // and without a branch while panels remain to be copied (with one the
    // compiler waits for every copy in flight)
    int kt = 0;
    for (; kt + 2 * NS - 2 < nk; kt += NS)
        each_of(std::make_integer_sequence<int, NS>{}, [&](auto s) { turn(s, kt + decltype(s)::value, Yes{}); });
    each_of(std::make_integer_sequence<int, 2 * NS - 2>{}, [&](auto t) {
        constexpr int T = decltype(t)::value;
        const std::integral_constant<int, T % NS> s{};
        if (kt + T + NS - 1 < nk) turn(s, kt + T, Yes{});
        else if (kt + T < nk) turn(s, kt + T, No{});
    });
}

// The LDS of a ring: one array per stage, picked by stage number.
#define MG_RING_STAGES(NS, BYTES)                                                       \
    __shared__ __attribute__((aligned(1024))) uint8_t ring0_[BYTES];                    \
    __shared__ __attribute__((aligned(1024))) uint8_t ring1_[BYTES];                    \
    __shared__ __attribute__((aligned(1024))) uint8_t ring2_[BYTES];                    \
    __shared__ __attribute__((aligned(1024))) uint8_t ring3_[(NS) > 3 ? (BYTES) : 16];  \
    __shared__ __attribute__((aligned(1024))) uint8_t ring4_[(NS) > 4 ? (BYTES) : 16];  \
    auto ring_stage = [&](auto s) -> uint8_t* {                                         \
        constexpr int S = decltype(s)::value;                                           \
        if constexpr (S == 0) return ring0_;                                            \
        else if constexpr (S == 1) return ring1_;                                       \
        else if constexpr (S == 2) return ring2_;                                       \
        else if constexpr (S == 3) return ring3_;                                       \
        else return ring4_;                                                             \
    }

// Global chunk g of row `row` of a stage's panel, as one 16-byte vector load (as
// a struct of words some of the reads lose what tells them from the copies in
// flight).
MG_DEVICE uintx4 ring_chunk(const uint8_t* lds, int row, int g)
{
    return *reinterpret_cast<const uintx4*>(lds + row * 128 + 16 * (g ^ direct_swz(row)));
}

// ---- K panels streamed by single waves: panels `wave`, wave + NW, ... of a
// tile go through this wave's own two-stage ring (S0, S1: its stages of (BM +
// BN) 128-byte rows), awaited by this wave alone, so that the K loop has no
// barrier.  A stage is read into registers whole and at once refilled, two
// panels ahead.  copy(stage, i): issue the copies of the wave's panel i;
// read(stage): its fragments into registers; multiply(slot): their products,
// slot = i modulo 60; batch(i): called at the first panel of each 60 (and with
// copies in flight, so its loads should be few).
template <int BM, int BN, class Copy, class Read, class Multiply, class Batch>
MG_DEVICE void stream_loop(uint8_t* S0, uint8_t* S1, int n, Copy copy, Read read, Multiply multiply, Batch batch)
{
    constexpr int COPIES = (BM + BN) / 8;   // copy instructions per stage
    static_assert(COPIES < 64, "the wait counts the copies in flight");
    // MORE: one newer panel is in flight and may stay so, and panel i + 2 exists
    auto step = [&](int i, int slot, uint8_t* S, auto more) {
        constexpr int FLY = decltype(more)::value ? COPIES : 0;
        __builtin_amdgcn_s_waitcnt(0x0f70 | (FLY & 15) | (FLY >> 4 << 14));   // vmcnt(FLY)
        read(S);
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the stage is read
        if constexpr (decltype(more)::value) copy(S, i + 2);
        multiply(slot);
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    // Two panels at a time, so that each one's stage is a compile-time choice,
    // and without a branch while panels remain to be copied (with one the
    // compiler waits for every copy in flight before each panel).
    int i = 0, at = 0;
    if (n <= 0) return;
    copy(S0, 0);
    copy(S1, min(1, n - 1));   // (a single panel again, rather than a branch)
    batch(0);
    for (;;) {
        const int lim = at + 60;
        for (; i < lim && i + 3 < n; i += 2) {
            step(i, i - at, S0, Yes{});
            step(i + 1, i + 1 - at, S1, Yes{});
        }
        if (i < lim) break;
        at = i;
        batch(at);
    }
    // the last panels, at most three, some of them not yet copied
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        uint8_t* S = t % 2 == 0 ? S0 : S1;
        if (i + 2 < n) step(i, i - at, S, Yes{});
        else if (i < n) step(i, i - at, S, No{});
        ++i;
    }
}

}  // namespace mg
