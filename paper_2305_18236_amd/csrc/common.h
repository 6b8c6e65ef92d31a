// Shared device-side helpers of the mgemm kernels (gfx950 / CDNA4 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int intx8 __attribute__((ext_vector_type(8)));

#ifndef MG_DEVICE   // (a CPU test compiles the panel loads as host code)
#define MG_DEVICE __device__ __forceinline__
#endif

namespace mg {

// Arguments of one GEMM, as the kernels see them.  Strides are row strides of
// the stored matrices in elements; trans flags say whether op(X) = X^T.
struct GemmArgs {
    const float* A;
    const float* B;
    float* C;
    int64_t M, N, K;
    int64_t lda, ldb, ldc;
    float alpha, beta;
    int tiles_m, tiles_n;
    int group_m;      // tile rows per raster group (L2 reuse of B panels)
    int remap;        // 1: give each XCD a contiguous range of tiles (see tile_of)
    // vec_a / vec_b: in-panel byte offsets fit 32 bits (ld < 2^22 - 64), which
    // lets panels address through a uniform base plus a 32-bit per-lane
    // offset, and stored rows hold at least one 4-float chunk.  No alignment
    // is asked for: 16-byte global accesses need 4-byte alignment only.
    int vec_a, vec_b;
    // Split-K (launched with gridDim.y > 1): workgroup row s of the grid
    // multiplies the K range [s*k_chunk, min(K, (s+1)*k_chunk)) and stores its
    // unscaled partial product at part + s*part_stride (row stride ldp, a
    // multiple of 4, 16-byte aligned); splitk_reduce_kernel then sums the
    // partials in order of s and applies alpha and beta.
    float* part;
    int64_t k_chunk, ldp, part_stride;
    // SYR2K: the panels of both products that sgemm_tile multiplies (set in
    // the kernel); the workgroups that a balanced split deals k_chunk panels
    // each (0: not balanced), and the most panels of one run of accumulators.
    int p0, p1, share, chain;
};

// The GEMM one workgroup of a split-K launch computes (see GemmArgs::part).
// PACKED: A and B are k-contiguous bf16 rows (the pre-packed planes).
template <bool TA, bool TB, bool PACKED>
MG_DEVICE void split_k_view(GemmArgs& g)
{
    if (gridDim.y == 1) return;
    const int64_t k0 = int64_t(blockIdx.y) * g.k_chunk;
    g.K = min(g.k_chunk, g.K - k0);
    if (PACKED) {
        g.A = reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(g.A) + k0);
        g.B = reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(g.B) + k0);
    } else {
        g.A += TA ? k0 * g.lda : k0;
        g.B += TB ? k0 : k0 * g.ldb;
    }
    g.C = g.part + int64_t(blockIdx.y) * g.part_stride;
    g.ldc = g.ldp;
    g.alpha = 1.f;
    g.beta = 0.f;
}

// Arguments of the FP8 GEMM on packed operands (see gemm_fp8.hip).
struct Fp8Args {
    const uint8_t* qA;   // Mp x Kp E4M3 codes of op(A), row stride ldq
    const uint8_t* qB;   // Np x Kp E4M3 codes of op(B)^T, row stride ldq
    const uint8_t* sA;   // (Mp/128) x (Kp/128) E8M0 scale bytes, row stride lds
    const uint8_t* sB;   // (Np/128) x (Kp/128)
    float* C;
    int64_t M, N, Kp;
    int64_t ldq, lds, ldc;
    float alpha, beta;
    int tiles_m, tiles_n, group_m, remap;
};

// Map a linear workgroup id to an output tile (tm, tn): a raster that walks
// groups of `group_m` tile rows column by column, so that tiles running at
// the same time share A row panels and B column panels.
//
// Hardware hands consecutive workgroup ids to the 8 XCDs round-robin.  With
// `remap` set the ids are first permuted so that each XCD owns a contiguous
// range of the raster (its resident tiles then form one compact block per
// XCD); without it each XCD takes every eighth tile of the raster.
MG_DEVICE void tile_of(int pid, int tiles_m, int tiles_n, int group_m, int remap, int& tm, int& tn)
{
    const int total = tiles_m * tiles_n;
    constexpr int XCDS = 8;
    if (remap && total % XCDS == 0) {
        const int per = total / XCDS;
        pid = (pid % XCDS) * per + pid / XCDS;
    }
    const int in_group = group_m * tiles_n;
    const int g = pid / in_group;
    const int first_m = g * group_m;
    const int rows = min(tiles_m - first_m, group_m);
    const int local = pid - g * in_group;
    tm = first_m + local % rows;
    tn = local / rows;
}

// 16-byte and 8-byte accesses of 4-byte aligned floats.  The global memory
// path takes them at any 4-byte address: an access that straddles two cache
// lines costs a second line, not a fault or a scalar sequence.
typedef floatx4 floatx4u __attribute__((aligned(4)));
typedef floatx2 floatx2u __attribute__((aligned(4)));

// The valid part of a block of a stored matrix whose first element is (r0, c0)
// of R x Cn valid entries: rows and columns from the block's first (not above
// zero where the block lies outside), and whether the matrix has a whole
// W-element chunk.
struct Valid {
    int rows, cols;
    bool wide;
};

MG_DEVICE Valid valid_part(int64_t r0, int64_t c0, int64_t R, int64_t Cn, int W)
{
    const int64_t big = 1 << 20;
    return {int(min(R - r0, big)), int(min(Cn - c0, big)), Cn >= W};
}

// Fetch of columns c .. c+3 of row r of a block where any of them may lie
// outside the matrix (src: the block's first element): those read 0.  Two
// halves without per-lane branches, so that a caller can put the loads of all
// its chunks in flight before the first is looked at: edge_load reads the
// chunk moved left and up until it is inside, edge_fix moves the values back
// and clears the rest.
MG_DEVICE floatx4 edge_load(const float* __restrict__ src, int64_t ld, int r, int c, Valid b)
{
    const float* __restrict__ p = src + min(r, b.rows - 1) * ld;
    if (b.wide) return *reinterpret_cast<const floatx4u*>(p + min(c, b.cols - 4));   // uniform
    return floatx4{p[min(c, b.cols - 1)], p[min(c + 1, b.cols - 1)], p[min(c + 2, b.cols - 1)],
                   p[min(c + 3, b.cols - 1)]};
}

MG_DEVICE floatx4 edge_fix(floatx4 w, int r, int c, Valid b)
{
    const int left = max(0, min(4, b.cols - c));   // valid columns of the chunk
    const int keep = r < b.rows ? left : 0;
    const int sh = b.wide ? 4 - left : 0;          // how far the chunk was moved left
    floatx4 x = w;
    if (sh & 1) x = floatx4{x[1], x[2], x[3], 0.f};
    if (sh & 2) x = floatx4{x[2], x[3], 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e >= keep) x[e] = 0.f;
    return x;
}

// 16-byte load at a uniform base plus a 32-bit per-lane BYTE offset: the
// form the global_load ... saddr instructions take (one VGPR per address).
MG_DEVICE floatx4 load16(const float* __restrict__ base, uint32_t byte_off)
{
    return *reinterpret_cast<const floatx4u*>(reinterpret_cast<const char*>(base) + byte_off);
}

MG_DEVICE uint4 load16u(const void* __restrict__ base, uint32_t byte_off)
{
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(base) + byte_off);
}

MG_DEVICE floatx16 mfma_f32_32x32x2(float a, float b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

}  // namespace mg
