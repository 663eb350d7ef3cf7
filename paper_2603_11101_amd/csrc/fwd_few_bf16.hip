// Forward, bf16, for streams of few works: same arithmetic as fwd_bf16.hip, 32 rows per workgroup, the keys shared
// by its four waves (see few_util.h).
//
// A wave keeps the running softmax of its own tiles of 32 keys; at the end the four references meet, every wave
// scales its O and its row sum to the largest, and O is added up.  K and V of a wave have one LDS tile each: K of
// the next tile is requested once the scores are done, V once the second product is.
#include "few_util.h"

namespace va {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMaxLag = 8.0f;  // as in fwd_bf16.hip
constexpr int kPrefetch = 4;
constexpr int kKeys = 32;  // keys of a wave's tile

template <int D, int DR>
__global__ __launch_bounds__(256, D <= 128 ? 2 : 1) void fwd_few_kernel(AttnParams p, int bmt_log2) {
    constexpr int KSTEPS = DR / 16;
    constexpr int DT = (DR + 31) / 32;
    constexpr int TILE = kKeys * D * 2;
    using Loader = AsyncTile<D, kKeys, 1, DR>;
    extern __shared__ __attribute__((aligned(16))) char smem[];  // per wave a K and a V tile; then the row statistics

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    const FewBlock blk;
    if (blk.work >= p.num_items * p.works_per_item) return;
    // token rows and heads of a work (head counts are known here at run time only: they cost a few scalar operations)
    const int bmt = 1 << bmt_log2, hpb = kFwdBlockRows >> bmt_log2;
    const int hc = blk.work % p.works_per_item;
    const int G = p.Hq / p.Hkv, chunks = G / hpb, g = hc / chunks, h0 = g * G + hc % chunks * hpb;
    const WorkItem it = p.items[blk.work / p.works_per_item];
    const int q_row0 = it.w[0], q_rows = it.w[1], seq_row0 = it.w[2], L = it.w[7];

    // this workgroup's rows: stacked rows 32 part .. + 31, i.e. tokens tok0 .. tok1 - 1 of the item (of one or more heads)
    const int rr = 32 * blk.part + l32, tok = rr & (bmt - 1), head = rr >> bmt_log2;
    const int tok0 = 32 * blk.part & (bmt - 1) & ~31, tok1 = min(tok0 + min(32, bmt), q_rows);
    if (tok0 >= tok1) return;
    const bool valid = tok < q_rows;
    const int item_row = q_row0 - seq_row0;
    const MaskBounds mask(it.w[6], it.w[3], L, p.mask_mode);
    const int vis = mask.vis(item_row + tok), lo = mask.lo(item_row + tok);
    const int n_tiles = (mask.vis(item_row + tok1 - 1) + kKeys - 1) / kKeys;
    const int full_from = (mask.lo(item_row + tok1 - 1) + kKeys - 1) / kKeys;  // tiles without a hidden pair
    const int full_to = mask.vis(item_row + tok0) / kKeys;
    const int first = mask.lo(item_row + tok0) / kKeys;

    const int kv_row_bytes = p.Hkv * DR * 2;
    const size_t kv_off = ((size_t)seq_row0 * p.Hkv + g) * DR;
    const unsigned kv_bytes = (unsigned)(L - 1) * kv_row_bytes + DR * 2;
    const __bf16 *k_rows = static_cast<const __bf16*>(p.k) + kv_off, *v_rows = static_cast<const __bf16*>(p.v) + kv_off;
    const int k_tile = wave * 2 * TILE, v_tile = k_tile + TILE;
    const unsigned smem_lds = lds_addr(smem);
    Loader loader;
    loader.init(0, lane, kv_row_bytes);
    auto load_k = [&](int kt) {
        loader.issue(rsrc_if(kt < n_tiles, k_rows, kv_bytes), smem_lds + k_tile, kt < n_tiles ? kt * kKeys * kv_row_bytes : 0);
    };
    auto load_v = [&](int kt) {
        loader.issue(rsrc_if(kt < n_tiles, v_rows, kv_bytes), smem_lds + v_tile, kt < n_tiles ? kt * kKeys * kv_row_bytes : 0);
    };

    const int q_tok_bytes = p.Hq * DR * 2;
    const size_t q_off = ((size_t)q_row0 * p.Hq + h0) * DR;
    const unsigned q_bytes = (unsigned)(q_rows - 1) * q_tok_bytes + hpb * DR * 2;
    const int row_off = valid ? tok * q_tok_bytes + head * DR * 2 : 0x7fff0000;

    // tiles by their number in the sample, so that the result of a row does not depend on its neighbours
    int kt = first + ((wave - first) & (kFewWaves - 1));
    bf16x8 qf[KSTEPS];
    {
        const __amdgpu_buffer_rsrc_t rows = RowBlock<D, DR>::rows(static_cast<const __bf16*>(p.q) + q_off, q_bytes);
#pragma unroll
        for (int t = 0; t < KSTEPS; ++t)
            qf[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rows, row_off + 32 * t + 16 * hf, 0, 0));
    }
    load_k(kt);
    load_v(kt);
    const FragAddr<D> fa(lane);
    const float c = p.scale * kLog2e;

    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
    float m = -INFINITY, lsum = 0.0f;
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t) settle(qf[t]);

    for (; kt < n_tiles; kt += kFewWaves) {
        wait_async_loads_except<Loader::PER_WAVE>();  // K is here; V may still be on its way
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
        {
            const int tile = here(k_tile);
            bf16x8 ring[kPrefetch];
#pragma unroll
            for (int i = 0; i < kPrefetch && i < KSTEPS; ++i) ring[i] = fa.rowmajor(smem, tile, 0, i);
#pragma unroll
            for (int i = 0; i < KSTEPS; ++i) {
                const bf16x8 a = ring[i % kPrefetch];
                if (i + kPrefetch < KSTEPS) ring[i % kPrefetch] = fa.rowmajor(smem, tile, 0, i + kPrefetch);
                s = mfma32(a, qf[i], s);
            }
            pin_fed_by_lds<KSTEPS, kPrefetch, 1, 0>();
        }
        lds_reads_done();
        load_k(kt + kFewWaves);
        if (kt < full_from || kt >= full_to) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kt * kKeys + acc_row(r, hf);
                if (key >= vis || key < lo) s[r] = -INFINITY;
            }
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = pair_max(mx) * c;
        if (__builtin_amdgcn_ballot_w64(mx > m + kMaxLag) != 0) {
            asm volatile("");  // a branch, not selects
            const float m_new = fmaxf(m, mx);
            const float alpha = __builtin_amdgcn_exp2f(m - (m_new == -INFINITY ? 0.0f : m_new));
            m = m_new;
            lsum *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
        // a row may see no key of the wave's tiles: reference 0 until it does
        const float m_ref = m == -INFINITY ? 0.0f : m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -m_ref));
            lsum += s[r];
        }
        bf16x8 pf[2];
#pragma unroll
        for (int x = 0; x < 2; ++x)
            pf[x] = to_bf16x8(s[8 * x + 0], s[8 * x + 1], s[8 * x + 2], s[8 * x + 3], s[8 * x + 4], s[8 * x + 5],
                              s[8 * x + 6], s[8 * x + 7]);
        wait_async_loads_except<Loader::PER_WAVE>();  // V is here; the next K may be on its way
        {
            constexpr int NS = 2 * DT;  // step i: keys 16 (i / DT) .. + 15, O^T block i % DT
            const int tile = here(v_tile);
            bf16x8 ring[kPrefetch];
#pragma unroll
            for (int i = 0; i < kPrefetch && i < NS; ++i) ring[i] = fa.transposed(smem, tile, i / DT, i % DT);
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const bf16x8 a = ring[i % kPrefetch];
                if (i + kPrefetch < NS) ring[i % kPrefetch] = fa.transposed(smem, tile, (i + kPrefetch) / DT, (i + kPrefetch) % DT);
                o[i % DT] = mfma32(a, pf[i / DT], o[i % DT]);
            }
            pin_fed_by_lds<NS, kPrefetch, 2, 1>();
        }
        lds_reads_done();
        load_v(kt + kFewWaves);
    }

    wait_async_loads();  // of nothing, but they write: the tiles are about to be used otherwise
    // the four waves' references and sums, by row
    float* stats = reinterpret_cast<float*>(smem + kFewWaves * 2 * TILE);
    lsum = pair_sum(lsum);
    if (hf == 0) {
        stats[wave * 64 + l32] = m;
        stats[wave * 64 + 32 + l32] = lsum;
    }
    __syncthreads();
    float top = -INFINITY, total = 0.0f;
#pragma unroll
    for (int w = 0; w < kFewWaves; ++w) top = fmaxf(top, stats[w * 64 + l32]);
    const float ref = top == -INFINITY ? 0.0f : top;
#pragma unroll
    for (int w = 0; w < kFewWaves; ++w)
        total += stats[w * 64 + 32 + l32] * __builtin_amdgcn_exp2f(stats[w * 64 + l32] - ref);
    const float mine = __builtin_amdgcn_exp2f(m - ref);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= mine;
    few_merge_store<DR, DT>(smem, 2 * TILE, wave, lane, o, 1.0f / total,
                            RowBlock<D, DR>::rows(static_cast<__bf16*>(p.out) + q_off, q_bytes), row_off);
    if (wave == 0 && hf == 0 && valid)
        p.lse[(size_t)(h0 + head) * p.T + q_row0 + tok] = (top + __builtin_amdgcn_logf(total)) * kLn2;
}

template <int D, int DR = D>
hipError_t launch_d(const AttnParams& p, hipStream_t stream) {
    constexpr size_t smem = kFewWaves * 2 * kKeys * D * 2 + kFewWaves * 64 * sizeof(float);
    const hipError_t attr = VA_ALLOW_DYNAMIC_LDS((&fwd_few_kernel<D, DR>), smem);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((fwd_few_kernel<D, DR>), dim3(few_grid(p.num_items * p.works_per_item)), dim3(256), smem, stream, p,
                       rows_log2(kFwdBlockRows / heads_per_block(p.Hq, p.Hkv)));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_few(const AttnParams& p, hipStream_t stream) {
    switch (p.D) {
        case 48: return launch_d<64, 48>(p, stream);
        case 64: return launch_d<64>(p, stream);
        case 80: return launch_d<128, 80>(p, stream);
        case 96: return launch_d<128, 96>(p, stream);
        case 128: return launch_d<128>(p, stream);
        case 160: return launch_d<256, 160>(p, stream);
        case 192: return launch_d<256, 192>(p, stream);
        case 256: return launch_d<256>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace va
