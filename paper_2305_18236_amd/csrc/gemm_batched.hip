// Uneven batched GEMM in one persistent launch.
//
// Every problem of the batch is cut into output tiles of its own variant
// (tile shape chosen per problem by the tuning table or the default rule),
// the tiles of all problems form one work list, and a grid sized to fill the
// GPU once takes the items from that list one at a time through an atomic
// counter: whichever workgroup finishes first takes the next item.  The host
// orders the problems by the cost of one of their tiles, largest first, so
// this is greedy longest-processing-time-first scheduling, and the short
// tiles at the end fill the gaps the long ones leave.
//
// Each tile runs the same layered tile code as the single-GEMM kernels
// (tile_f32.h, tile_bf16.h): the blocked, packed, MFMA micro-kernel scheme of
// Algorithm 1 of Kuzma et al. (SPE 2023), with one LDS buffer sized for the
// largest variant shared by all of them.
#include "tile_f32.h"
#include "tile_bf16.h"
#include "kernels.h"

namespace mg {

const int kSgemmBatchedCfg[kSgemmBatchedVariants] = {3, 0};
const int kBf16BatchedCfg[kBf16BatchedVariants] = {4, 5, 2};
const BatchedTile kSgemmBatchedTile[kSgemmBatchedVariants] = {{64, 128}, {128, 128}};
const BatchedTile kBf16BatchedTile[kBf16BatchedVariants] = {{64, 64}, {128, 64}, {128, 128}};

// Index of the problem owning work item `item`: the last p with
// tile_begin <= item (problems with no tiles are skipped by the search).
MG_DEVICE int owner(const BatchProblem* __restrict__ P, int count, int64_t item)
{
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (P[mid].tile_begin <= item) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Eight waves, two register staging sets, waves outside C skipped: 64 x 128
// tiles of 32 x 32 waves for the small variant, 128 x 128 tiles of 64 x 32
// waves for the large one.  Every output adds its products in the order of
// configurations 3 and 0, so the results are theirs bit for bit.
template <bool TA, bool TB>
MG_DEVICE void f32_variant(const BatchProblem& p, int tm, int tn, float* smem)
{
    if (p.variant == 0) sgemm_tile<64, 128, 32, 32, 32, TA, TB, false, 0, true, 1, true>(p.g, tm, tn, smem);
    else sgemm_tile<128, 128, 32, 64, 32, TA, TB, false, 0, true, 1, true>(p.g, tm, tn, smem);
}

// Two workgroups share a compute unit (three of BF16's and FP16's), so that one's
// epilogue overlaps another's K loop: FP32's of 512 threads in 128 registers a
// lane, four waves per SIMD; bf16x3's of 256 threads in up to 256, two; BF16's
// and FP16's in up to 168, three.
//
// The next work item for the whole workgroup: thread 0 takes it from the
// counter and hands it to the others through the first 8 bytes of the panel
// buffer.  That buffer is free here: every tile ends its K loop with a
// workgroup barrier after its last LDS access (its epilogue touches no LDS),
// and the second barrier keeps the next tile's packing from overwriting the
// slot before every thread has read it.  (A separate __shared__ word would
// push the bf16x3 kernel's LDS past half a CU and halve its occupancy.)
MG_DEVICE int64_t next_item(unsigned long long* counter, void* smem)
{
    int64_t* slot = static_cast<int64_t*>(smem);
    if (threadIdx.x == 0) *slot = int64_t(atomicAdd(counter, 1ull));
    __syncthreads();
    // (through scalar registers, so that the problem's arguments, all indexed
    // by it, are loaded and kept in scalar registers too)
    const int64_t item = *slot;
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(item));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(item) >> 32));
    __syncthreads();
    return int64_t((uint64_t(hi) << 32) | lo);
}

// Optional timing of the launch: workgroup b writes the constant-rate wall
// clock at its start to stamps[2b] and after its last item to stamps[2b + 1]
// (one 8-byte vector store each, from thread 0), so the caller can measure
// how long workgroups idle at the end while the last tiles finish.
MG_DEVICE void stamp(unsigned long long* stamps, int which)
{
    if (stamps != nullptr && threadIdx.x == 0) stamps[2 * int64_t(blockIdx.x) + which] = wall_clock64();
}

// Problem `i` in scalar registers: loaded through the vector memory path (the
// compiler cannot show that no store to a C changes it) it would occupy a
// vector register per word.
MG_DEVICE BatchProblem problem(const BatchProblem* __restrict__ P, int i)
{
    constexpr int W = sizeof(BatchProblem) / 4;
    struct Words {
        uint32_t w[W];
    };
    Words x = __builtin_bit_cast(Words, P[i]);
#pragma unroll
    for (int k = 0; k < W; ++k) x.w[k] = __builtin_amdgcn_readfirstlane(x.w[k]);
    return __builtin_bit_cast(BatchProblem, x);
}

__global__ __launch_bounds__(512, 4) void sgemm_batched_kernel(const BatchProblem* __restrict__ P, int count,
                                                             int64_t total_tiles, unsigned long long* counter,
                                                             unsigned long long* stamps)
{
    __shared__ __attribute__((aligned(16))) float smem[sgemm_lds_floats<128, 128, 32>()];
    stamp(stamps, 0);
    for (int64_t item = next_item(counter, smem); item < total_tiles; item = next_item(counter, smem)) {
        const BatchProblem p = problem(P, owner(P, count, item));
        const int local = int(item - p.tile_begin);
        const int tm = local / p.g.tiles_n, tn = local % p.g.tiles_n;
        if (p.ta) {
            if (p.tb) f32_variant<true, true>(p, tm, tn, smem);
            else f32_variant<true, false>(p, tm, tn, smem);
        } else {
            if (p.tb) f32_variant<false, true>(p, tm, tn, smem);
            else f32_variant<false, false>(p, tm, tn, smem);
        }
    }
    stamp(stamps, 1);
}

template <int BM, int BN, int BK, int WM, int WN, int TERMS>
MG_DEVICE void bf16_variant(const BatchProblem& p, int tm, int tn, uint16_t* smem)
{
    if (p.ta) {
        if (p.tb) bf16_tile<BM, BN, BK, WM, WN, true, true, TERMS, false, true>(p.g, tm, tn, smem);
        else bf16_tile<BM, BN, BK, WM, WN, true, false, TERMS, false, true>(p.g, tm, tn, smem);
    } else {
        if (p.tb) bf16_tile<BM, BN, BK, WM, WN, false, true, TERMS, false, true>(p.g, tm, tn, smem);
        else bf16_tile<BM, BN, BK, WM, WN, false, false, TERMS, false, true>(p.g, tm, tn, smem);
    }
}

template <int TERMS>
__global__ __launch_bounds__(256, TERMS == 3 ? 2 : 3) void bf16_batched_kernel(const BatchProblem* __restrict__ P, int count,
                                                            int64_t total_tiles, unsigned long long* counter,
                                                            unsigned long long* stamps)
{
    __shared__ __attribute__((aligned(16))) uint16_t smem[bf16_lds_elems<128, 128, 32, TERMS>()];
    stamp(stamps, 0);
    for (int64_t item = next_item(counter, smem); item < total_tiles; item = next_item(counter, smem)) {
        const BatchProblem p = problem(P, owner(P, count, item));
        const int local = int(item - p.tile_begin);
        const int tm = local / p.g.tiles_n, tn = local % p.g.tiles_n;
        switch (p.variant) {
        case 0: bf16_variant<64, 64, 32, 32, 32, TERMS>(p, tm, tn, smem); break;
        case 1: bf16_variant<128, 64, 32, 64, 32, TERMS>(p, tm, tn, smem); break;
        default: bf16_variant<128, 128, 32, 64, 64, TERMS>(p, tm, tn, smem); break;
        }
    }
    stamp(stamps, 1);
}

static const void* batched_kernel(int path)
{
    switch (path) {
    case 0: return reinterpret_cast<const void*>(&sgemm_batched_kernel);
    case 1: return reinterpret_cast<const void*>(&bf16_batched_kernel<3>);
    case 2: return reinterpret_cast<const void*>(&bf16_batched_kernel<1>);
    case 4: return reinterpret_cast<const void*>(&bf16_batched_kernel<16>);
    default: return nullptr;
    }
}

static int batched_threads(int path) { return path == 0 ? 512 : 256; }

int batched_blocks_per_cu(int path)
{
    const void* k = batched_kernel(path);
    if (!k) return 0;
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k, batched_threads(path), 0) != hipSuccess || blocks < 1)
        blocks = 1;
    return blocks;
}

hipError_t launch_gemm_batched(int path, const BatchProblem* dev_problems, int count,
                               int64_t total_tiles, int grid, unsigned long long* counter,
                               unsigned long long* stamps, hipStream_t stream)
{
    const void* k = batched_kernel(path);
    if (!k) return hipErrorInvalidValue;
    void* args[] = {&dev_problems, &count, &total_tiles, &counter, &stamps};
    return hipLaunchKernel(k, dim3(grid), dim3(batched_threads(path)), args, 0, stream);
}

}  // namespace mg
