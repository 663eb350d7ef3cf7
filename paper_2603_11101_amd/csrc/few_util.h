// What the kernels for streams of few works share (fwd_few_bf16.hip, bwd_few_bf16.hip).
//
// The persistent kernels give a work of 128 rows to four waves that walk over the same tiles.  A small stream has
// fewer such works than the chip has CUs, and each is one serial walk.  Here a workgroup owns 32 rows, a
// quarter of a work, and its four waves share the walk instead: wave w takes the tiles w, w + 4, ... on its own
// (own LDS tiles, no barrier inside the loop) and the four partial sums meet in LDS at the end.  Four times
// the workgroups and a quarter of the serial chain, for four times the LDS traffic per product.
#pragma once

#include "kernels.h"
#include "mfma_util.h"

namespace va {

constexpr int kFewWaves = 4;

// Workgroup b runs part (b / 8) % 4, split (b / 32) % splits of work b / (32 splits) * 8 + b % 8: the parts of a
// work, and the works of one (sample, KV head) where the number of head chunks is a multiple of 8, share an
// XCD and its L2.  (Splits: dK/dV only, see bwd_few_bf16.hip.)
struct FewBlock {
    int work, part, split;
    VA_DEV explicit FewBlock(int splits = 1) {
        const int b = (int)(blockIdx.x / kXcds);
        part = b % kFewWaves;
        split = b / kFewWaves % splits;
        work = b / (kFewWaves * splits) * kXcds + (int)(blockIdx.x % kXcds);
    }
};
inline unsigned few_grid(int num_works, int splits = 1) {
    return (unsigned)((num_works + kXcds - 1) / kXcds * kXcds * kFewWaves * splits);
}
inline int rows_log2(int rows) {  // of a power of two
    int n = 0;
    while (rows >> (n + 1)) ++n;
    return n;
}

// A buffer of the given size, or, where there is nothing more to fetch, of none: loads through it then bring zeros
// from nowhere, and the loop around them needs no branch (at which the compiler would move every accumulator).
// The scalar offset of such loads must be 0: see AsyncTile::issue.
VA_DEV i32x4 rsrc_if(bool more, const void* base, unsigned bytes) { return make_rsrc(base, more ? bytes : 0u); }

// The end of a workgroup: four waves hold partial sums of one transposed 32 x DR block (accumulator layout: lane % 32
// is the row).  They leave them in LDS, 1 KiB per register quad, and take turns at strips of 16 columns, i.e.
// two quads: few_sum_strips calls out(strip, a, b) with the two summed quads.
// The region of a wave (DT * 4 KiB) starts wave * stride bytes into smem; nothing else may be using it.
template <int DT, typename Out>
VA_DEV void few_sum_strips(char* smem, int stride, int wave, int lane, const f32x16 (&acc)[DT], Out out) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[dt][4 * q], acc[dt][4 * q + 1], acc[dt][4 * q + 2], acc[dt][4 * q + 3]};
            *reinterpret_cast<f32x4*>(smem + wave * stride + (dt * 4 + q) * 1024 + lane * 16) = v;
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (2 * DT + kFewWaves - 1) / kFewWaves; ++i) {
        const int strip = wave + i * kFewWaves;
        if (strip >= 2 * DT) break;
        f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = a;
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) {
            a += *reinterpret_cast<const f32x4*>(smem + w * stride + (2 * strip) * 1024 + lane * 16);
            b += *reinterpret_cast<const f32x4*>(smem + w * stride + (2 * strip + 1) * 1024 + lane * 16);
        }
        out(strip, a, b);
    }
}

// Two summed quads of strip `strip`, times the factor of the lane's row, as bf16.  row_off: byte offset of the
// lane's row in the buffer, past its end if the row is not to be written.
template <int DR>
VA_DEV void few_store_strip(int strip, f32x4 a, f32x4 b, float factor, int lane, __amdgpu_buffer_rsrc_t rsrc, int row_off) {
    a *= factor;
    b *= factor;
    const u32x2 pa = __builtin_bit_cast(u32x2, __builtin_convertvector(a, bf16x4));
    const u32x2 pb = __builtin_bit_cast(u32x2, __builtin_convertvector(b, bf16x4));
    // a lane holds columns 4 hf .. + 3 of both groups of 8; after the swap the lower lanes hold all of the first
    // group of their row and the upper lanes all of the second
    const u32x2 s0 = __builtin_amdgcn_permlane32_swap(pa[0], pb[0], false, false);
    const u32x2 s1 = __builtin_amdgcn_permlane32_swap(pa[1], pb[1], false, false);
    const int col = 16 * strip + 8 * (lane >> 5);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{s0[0], s1[0], s0[1], s1[1]}, rsrc, col < DR ? row_off + 2 * col : 0x7ffffff0,
                                           0, 0);
}

template <int DR, int DT>
VA_DEV void few_merge_store(char* smem, int stride, int wave, int lane, const f32x16 (&acc)[DT], float factor,
                            __amdgpu_buffer_rsrc_t rsrc, int row_off) {
    few_sum_strips<DT>(smem, stride, wave, lane, acc, [&](int strip, f32x4 a, f32x4 b) {
        few_store_strip<DR>(strip, a, b, factor, lane, rsrc, row_off);
    });
}

// A tile's LDS offset, derived anew where it is used: known to be the same in every iteration, its sum with each of
// the fragment addresses would be kept in a register of its own across the loop.
VA_DEV int here(int tile) {
    asm volatile("" : "+s"(tile));
    return tile;
}

// Keeps a run of N MFMAs fed from LDS in the order it is written: AHEAD fragments (READS instructions each) read first,
// then one MFMA and the reads of a later one in turn.  Left alone, the compiler reads a fragment, waits and
// multiplies.  GROUP numbers the runs of one stretch of straight code.
template <int N, int AHEAD, int READS, int GROUP>
VA_DEV void pin_fed_by_lds() {
#pragma unroll
    for (int i = 0; i < AHEAD && i < N; ++i) __builtin_amdgcn_sched_group_barrier(0x100, READS, GROUP);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, GROUP);
        if (i + AHEAD < N) __builtin_amdgcn_sched_group_barrier(0x100, READS, GROUP);
    }
}

// LDS reads of a tile are over once their values have been used; said explicitly before the tile is refilled.
VA_DEV void lds_reads_done() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

}  // namespace va
