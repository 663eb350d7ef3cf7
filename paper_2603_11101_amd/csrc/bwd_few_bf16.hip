// Backward, bf16, for streams of few works: the arithmetic of bwd_dq_bf16.hip and bwd_bf16.hip, 32 rows per
// workgroup, their tiles shared by its four waves (see few_util.h).
//
// The dQ kernel computes delta = rowsum(dO * O) and LSE * log2(e) of its rows at every head dimension and leaves
// them in the workspace, so it runs first and no separate pass over O and dO is launched.  (only_delta: it does that and
// ends; for a caller who asks for delta without dQ and gets the bits of the whole backward.)
#include "few_util.h"

namespace va {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kTileRows = 32;  // rows of a wave's tile (keys for dQ, queries for dK/dV)
constexpr int kPrefetch = 4;   // LDS fragment reads in flight ahead of the MFMA that uses them

template <int D, int DR>
__global__ __launch_bounds__(256, D <= 128 ? 2 : 1) void bwd_dq_few_kernel(AttnParams p, int bmt_log2, bool only_delta) {
    constexpr int KSTEPS = DR / 16;
    constexpr int DT = (DR + 31) / 32;
    constexpr int TILE = kTileRows * D * 2;
    using Loader = AsyncTile<D, kTileRows, 1, DR>;
    extern __shared__ __attribute__((aligned(16))) char smem[];  // per wave a K and a V tile

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    const FewBlock blk;
    if (blk.work >= p.num_items * p.works_per_item) return;
    // token rows and heads of a work (head counts are known here at run time only: they cost a few scalar operations)
    const int bmt = 1 << bmt_log2, hpb = kDqBlockRows >> bmt_log2;
    const int hc = blk.work % p.works_per_item;
    const int G = p.Hq / p.Hkv, chunks = G / hpb, g = hc / chunks, h0 = g * G + hc % chunks * hpb;
    const WorkItem it = p.items[blk.work / p.works_per_item];
    const int q_row0 = it.w[0], q_rows = it.w[1], seq_row0 = it.w[2], L = it.w[7];

    const int rr = 32 * blk.part + l32, tok = rr & (bmt - 1), head = rr >> bmt_log2;
    const int tok0 = 32 * blk.part & (bmt - 1) & ~31, tok1 = min(tok0 + min(32, bmt), q_rows);
    if (tok0 >= tok1) return;
    const bool valid = tok < q_rows;
    const int item_row = q_row0 - seq_row0;
    const MaskBounds mask(it.w[6], it.w[3], L, p.mask_mode);
    const int vis = mask.vis(item_row + tok), lo = mask.lo(item_row + tok);
    const int n_tiles = (mask.vis(item_row + tok1 - 1) + kTileRows - 1) / kTileRows;
    const int full_from = (mask.lo(item_row + tok1 - 1) + kTileRows - 1) / kTileRows;  // tiles without a hidden pair
    const int full_to = mask.vis(item_row + tok0) / kTileRows;
    const int first = mask.lo(item_row + tok0) / kTileRows;

    const int kv_row_bytes = p.Hkv * DR * 2;
    const size_t kv_off = ((size_t)seq_row0 * p.Hkv + g) * DR;
    const unsigned kv_bytes = (unsigned)(L - 1) * kv_row_bytes + DR * 2;
    const __bf16 *k_rows = static_cast<const __bf16*>(p.k) + kv_off, *v_rows = static_cast<const __bf16*>(p.v) + kv_off;
    const int k_tile = wave * 2 * TILE, v_tile = k_tile + TILE;
    const unsigned smem_lds = lds_addr(smem);
    Loader loader;
    loader.init(0, lane, kv_row_bytes);
    auto load_k = [&](int kt) {
        loader.issue(rsrc_if(kt < n_tiles, k_rows, kv_bytes), smem_lds + k_tile, kt < n_tiles ? kt * kTileRows * kv_row_bytes : 0);
    };
    auto load_v = [&](int kt) {
        loader.issue(rsrc_if(kt < n_tiles, v_rows, kv_bytes), smem_lds + v_tile, kt < n_tiles ? kt * kTileRows * kv_row_bytes : 0);
    };

    using Rows = RowBlock<D, DR>;
    const int q_tok_bytes = p.Hq * DR * 2;
    const size_t q_off = ((size_t)q_row0 * p.Hq + h0) * DR;
    const unsigned q_bytes = (unsigned)(q_rows - 1) * q_tok_bytes + hpb * DR * 2;
    const int row_off = valid ? tok * q_tok_bytes + head * DR * 2 : 0x7fff0000;
    auto load_rows = [&](bf16x8 (&f)[KSTEPS], const void* tensor) {
        const __amdgpu_buffer_rsrc_t rows = Rows::rows(static_cast<const __bf16*>(tensor) + q_off, q_bytes);
#pragma unroll
        for (int t = 0; t < KSTEPS; ++t)
            f[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rows, row_off + 32 * t + 16 * hf, 0, 0));
    };
    int kt = first + ((wave - first) & (kFewWaves - 1));
    bf16x8 qf[KSTEPS], dof[KSTEPS];
    const size_t stat = (size_t)(h0 + head) * p.T + q_row0 + tok;
    // rows past the item: Q = dO = 0 and LSE = delta = 0, so p = 1, dS = 0, and they are not stored
    float lse2 = valid ? p.lse[stat] * kLog2e : 0.0f, delta;
    {
        bf16x8 of[KSTEPS];
        load_rows(dof, p.dout);
        load_rows(of, p.out);
        load_rows(qf, p.q);
        load_v(kt);
        load_k(kt);
        // the diagonal of dO O^T, as in bwd_dq_bf16.hip
        f32x16 dd;
#pragma unroll
        for (int r = 0; r < 16; ++r) dd[r] = 0.0f;
#pragma unroll
        for (int t = 0; t < KSTEPS; ++t) dd = mfma32(dof[t], of[t], dd);
        const int want = l32 - 4 * hf;
        float acc = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc = (8 * (r / 4) + r % 4 == want) ? dd[r] : acc;
        delta = acc + __shfl_xor(acc, 32);
        if (wave == 0 && hf == 0 && valid) {
            p.delta[stat] = -delta;  // kept negated
            p.lse2[stat] = lse2;
        }
    }
    if (only_delta) {
        wait_async_loads();  // they write LDS: not after the workgroup has ended
        return;
    }
    const FragAddr<D> fa(lane);
    const float c = p.scale * kLog2e;

    f32x16 dq[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[dt][r] = 0.0f;
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t) settle(qf[t]);
    wait_async_loads();

    for (; kt < n_tiles; kt += kFewWaves) {
        auto product = [&](int tile, const bf16x8 (&rows)[KSTEPS]) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
            bf16x8 ring[kPrefetch];
#pragma unroll
            for (int i = 0; i < kPrefetch && i < KSTEPS; ++i) ring[i] = fa.rowmajor(smem, tile, 0, i);
#pragma unroll
            for (int i = 0; i < KSTEPS; ++i) {
                const bf16x8 a = ring[i % kPrefetch];
                if (i + kPrefetch < KSTEPS) ring[i % kPrefetch] = fa.rowmajor(smem, tile, 0, i + kPrefetch);
                acc = mfma32(a, rows[i], acc);
            }
            pin_fed_by_lds<KSTEPS, kPrefetch, 1, 0>();
            return acc;
        };
        wait_async_loads_except<Loader::PER_WAVE>();  // V is here; K may still be on its way
        f32x16 dp = product(here(v_tile), dof);
        lds_reads_done();
        load_v(kt + kFewWaves);
        wait_async_loads_except<Loader::PER_WAVE>();  // K is here
        const f32x16 s = product(here(k_tile), qf);
        const bool masked = kt < full_from || kt >= full_to;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -lse2));
            dp[r] = pv * (dp[r] - delta);
        }
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kt * kTileRows + acc_row(r, hf);
                if (key >= vis || key < lo) dp[r] = 0.0f;
            }
        }
        bf16x8 dsb[2];
#pragma unroll
        for (int x = 0; x < 2; ++x)
            dsb[x] = to_bf16x8(dp[8 * x], dp[8 * x + 1], dp[8 * x + 2], dp[8 * x + 3], dp[8 * x + 4], dp[8 * x + 5],
                               dp[8 * x + 6], dp[8 * x + 7]);
        {
            constexpr int NS = 2 * DT;  // step i: keys 16 (i / DT) .. + 15, dQ^T block i % DT
            const int tile = here(k_tile);
            bf16x8 ring[kPrefetch];
#pragma unroll
            for (int i = 0; i < kPrefetch && i < NS; ++i) ring[i] = fa.transposed(smem, tile, i / DT, i % DT);
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const bf16x8 a = ring[i % kPrefetch];
                if (i + kPrefetch < NS) ring[i % kPrefetch] = fa.transposed(smem, tile, (i + kPrefetch) / DT, (i + kPrefetch) % DT);
                dq[i % DT] = mfma32(a, dsb[i / DT], dq[i % DT]);
            }
            pin_fed_by_lds<NS, kPrefetch, 2, 1>();
        }
        lds_reads_done();
        load_k(kt + kFewWaves);
    }
    wait_async_loads();  // of nothing, but they write: the tiles are about to be used otherwise
    // a wave's partial takes exactly its own two tiles, which no other wave touches
    few_merge_store<DR, DT>(smem, 2 * TILE, wave, lane, dq, p.scale, Rows::rows(static_cast<__bf16*>(p.dq) + q_off, q_bytes),
                            row_off);
}

// One workgroup: 32 key rows of one KV head; the (query block, head) steps that see them go round its four waves.
// K fragments in registers, V in LDS (one tile for the workgroup), Q and dO of a step in the wave's own tiles:
// dO of the wave's next step is requested once dV is done, Q once dK is.
//
// Splits: one KV head that serves many query heads, or a long sample, can leave few workgroups with very many steps
// each.  The steps of a part are then dealt to `splits` workgroups, which leave float32 sums in the workspace
// (dK then dV, [register quad][lane] float4 as in LDS), and a merge kernel adds them in split order.
constexpr int kUnitFloats(int D) { return 2 * 32 * D; }  // partial sums of one (work, part, split)

// The 32 key rows of dK or dV a workgroup owns, as a buffer, and the lane's row in it.
template <int D, int DR>
struct KeyRows {
    size_t off;
    unsigned bytes;
    int row_off, keys;
    VA_DEV KeyRows(const AttnParams& p, const WorkItem& it, int part, int g, int l32) {
        keys = min(32, dkdv_item_rows(it.w[1]) - 32 * part);
        off = ((size_t)(it.w[0] + 32 * part) * p.Hkv + g) * DR;
        bytes = (unsigned)((max(keys, 1) - 1) * p.Hkv * DR * 2 + DR * 2);
        row_off = l32 < keys ? l32 * p.Hkv * DR * 2 : 0x7fff0000;
    }
    VA_DEV __amdgpu_buffer_rsrc_t of(const void* tensor) const {
        return RowBlock<D, DR>::rows(static_cast<const __bf16*>(tensor) + off, bytes);
    }
};

template <int D, int DR>
__global__ __launch_bounds__(256, D <= 128 ? 2 : 1) void bwd_dkdv_few_kernel(AttnParams p, int splits) {
    constexpr int KSTEPS = DR / 16;
    constexpr int DT = (DR + 31) / 32;
    constexpr int PF = D >= 128 ? 2 : kPrefetch;  // D >= 128 has no registers for more
    constexpr int TILE = kTileRows * D * 2;
    constexpr int STAGE = 2 * TILE + 512;  // Q, dO, then 64 floats each of LSE * log2(e) and -delta (the first 32 are used)
    constexpr int V_TILE = kFewWaves * STAGE;
    static_assert(STAGE % FragAddr<D>::kTileAlign == 0, "fragment addresses take tile offsets in multiples of the tile alignment");
    using Loader = AsyncTile<D, kTileRows, 1, DR>;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    const FewBlock blk(splits);
    if (blk.work >= p.num_items * p.works_per_item) return;
    const int g = blk.work % p.works_per_item;
    const WorkItem it = p.items[blk.work / p.works_per_item];
    const int seq_row0 = it.w[2], L = it.w[7];
    const int jw = it.w[0] - seq_row0 + 32 * blk.part;  // first key row of the workgroup, local to the sample
    const KeyRows<D, DR> own(p, it, blk.part, g, l32);
    if (own.keys <= 0) return;
    const MaskBounds mask(it.w[6], it.w[5], L, p.mask_mode);
    // query blocks of 32 rows that see one of the keys: the item's, less those that only see other parts of it
    int qb = it.w[3] * (dkdv_q_tile(D) / 32), qb_end = min((it.w[3] + it.w[4]) * (dkdv_q_tile(D) / 32), (L + 31) / 32);
    while (qb < qb_end && mask.vis(min(32 * qb + 31, L - 1)) <= jw) ++qb;
    while (qb < qb_end && mask.lo(32 * (qb_end - 1)) >= jw + 32) --qb_end;

    const int G = p.Hq / p.Hkv;
    const float c = p.scale * kLog2e;
    const int q_row_bytes = p.Hq * DR * 2, kv_row_bytes = p.Hkv * DR * 2;
    const int stage = wave * STAGE, q_tile = stage, do_tile = stage + TILE;
    const unsigned smem_lds = lds_addr(smem);
    Loader loader;
    loader.init(0, lane, q_row_bytes);
    // Step n: query block qb_end - 1 - n / G of head n % G of the group; with S splits the wave's
    // steps are 4 split + wave, + 4 S, ...
    const int n_steps = (qb_end - qb) * G;
    const unsigned q_bytes = (unsigned)(L - 1) * q_row_bytes + DR * 2;
    auto block_row = [&](int n) { return 32 * (qb_end - 1 - n / G); };
    // rows of one tensor and the statistic that goes with them
    auto load = [&](int n, const void* tensor, int tile, const float* per_row, int at) {
        const bool more = n < n_steps;
        const int i = min(n, n_steps - 1), h = g * G + i % G;
        loader.issue(rsrc_if(more, static_cast<const __bf16*>(tensor) + ((size_t)seq_row0 * p.Hq + h) * DR, q_bytes),
                     smem_lds + tile, more ? block_row(i) * q_row_bytes : 0);
        buffer_load_lds_4(smem_lds + at, lane * 4, rsrc_if(more, per_row + (size_t)h * p.T + seq_row0, (unsigned)L * 4),
                          more ? block_row(i) * 4 : 0);
    };
    auto load_q = [&](int n) { load(n, p.q, q_tile, p.lse2, stage + 2 * TILE); };
    auto load_do = [&](int n) { load(n, p.dout, do_tile, p.delta, stage + 2 * TILE + 256); };
    constexpr int kLoads = Loader::PER_WAVE + 1;
    {
        AsyncTile<D, kTileRows, kFewWaves, DR> v_loader;
        v_loader.init(wave, lane, kv_row_bytes);
        v_loader.issue(make_rsrc(static_cast<const __bf16*>(p.v) + ((size_t)seq_row0 * p.Hkv + g) * DR,
                                 (unsigned)(L - 1) * kv_row_bytes + DR * 2), smem_lds + V_TILE, jw * kv_row_bytes);
    }
    bf16x8 kf[KSTEPS];
    {
        const __amdgpu_buffer_rsrc_t rows = own.of(p.k);
#pragma unroll
        for (int t = 0; t < KSTEPS; ++t)
            kf[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rows, own.row_off + 32 * t + 16 * hf, 0, 0));
    }
    const int stride = kFewWaves * splits;
    int n = kFewWaves * blk.split + wave;
    load_do(n);
    load_q(n);
    // the query rows that see the lane's key
    const int first_row = mask.first_row(jw + l32);
    const unsigned rows_seeing = (unsigned)(mask.end_row(jw + l32) - first_row);
    const FragAddr<D> fa(lane);
    f32x16 dk[DT], dv[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            dk[dt][r] = 0.0f;
            dv[dt][r] = 0.0f;
        }
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t) settle(kf[t]);
    wait_async_loads();
    __syncthreads();  // the V tile is complete

    for (; n < n_steps; n += stride) {
        const int i0 = block_row(n);
        const float* lse_s = reinterpret_cast<const float*>(smem + stage + 2 * TILE);
        const float* delta_s = lse_s + 64;
        wait_async_loads_except<kLoads>();  // dO is here; Q may still be on its way
        // dP - delta: the sums start from -delta of their rows
        f32x16 dp, s;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 d4 = *reinterpret_cast<const f32x4*>(delta_s + 8 * r4 + 4 * hf);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dp[4 * r4 + e] = d4[e];
                s[4 * r4 + e] = 0.0f;
            }
        }
        {
            const int tile = here(do_tile), v_at = here(V_TILE);
            bf16x8 ring[PF], vring[PF];
            auto fetch = [&](int i) {
                ring[i % PF] = fa.rowmajor(smem, tile, 0, i);
                vring[i % PF] = fa.rowmajor(smem, v_at, 0, i);
            };
#pragma unroll
            for (int i = 0; i < PF && i < KSTEPS; ++i) fetch(i);
#pragma unroll
            for (int i = 0; i < KSTEPS; ++i) {
                const bf16x8 a = ring[i % PF], b = vring[i % PF];
                if (i + PF < KSTEPS) fetch(i + PF);
                dp = mfma32(a, b, dp);
            }
            pin_fed_by_lds<KSTEPS, PF, 2, 0>();
        }
        wait_async_loads();  // Q is here
        {
            const int tile = here(q_tile);
            bf16x8 ring[PF];
#pragma unroll
            for (int i = 0; i < PF && i < KSTEPS; ++i) ring[i] = fa.rowmajor(smem, tile, 0, i);
#pragma unroll
            for (int i = 0; i < KSTEPS; ++i) {
                const bf16x8 a = ring[i % PF];
                if (i + PF < KSTEPS) ring[i % PF] = fa.rowmajor(smem, tile, 0, i + PF);
                s = mfma32(a, kf[i], s);
            }
            pin_fed_by_lds<KSTEPS, PF, 1, 1>();
        }
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_s + 8 * r4 + 4 * hf);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 4 * r4 + e;
                s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -l4[e]));
                dp[r] *= s[r];
            }
        }
        if (mask.vis(i0) < jw + 32 || i0 + 32 > L || mask.lo(min(i0 + 31, L - 1)) > jw) {
            int base = i0 + 4 * hf - first_row;
            asm volatile("" : "+v"(base));  // a branch, not selects in every block
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((unsigned)(base + 8 * (r / 4) + r % 4) >= rows_seeing) {
                    s[r] = 0.0f;
                    dp[r] = 0.0f;
                }
        }
        bf16x8 pb[2], dsb[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            pb[x] = to_bf16x8(s[8 * x], s[8 * x + 1], s[8 * x + 2], s[8 * x + 3], s[8 * x + 4], s[8 * x + 5], s[8 * x + 6],
                              s[8 * x + 7]);
            dsb[x] = to_bf16x8(dp[8 * x], dp[8 * x + 1], dp[8 * x + 2], dp[8 * x + 3], dp[8 * x + 4], dp[8 * x + 5],
                               dp[8 * x + 6], dp[8 * x + 7]);
        }
        auto accumulate = [&](int tile, const bf16x8 (&b)[2], f32x16 (&acc)[DT]) {
            constexpr int NS = 2 * DT;
            bf16x8 ring[PF];
#pragma unroll
            for (int i = 0; i < PF && i < NS; ++i) ring[i] = fa.transposed(smem, tile, i / DT, i % DT);
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const bf16x8 a = ring[i % PF];
                if (i + PF < NS) ring[i % PF] = fa.transposed(smem, tile, (i + PF) / DT, (i + PF) % DT);
                acc[i % DT] = mfma32(a, b[i / DT], acc[i % DT]);
            }
            pin_fed_by_lds<NS, PF, 2, 2>();
        };
        accumulate(here(do_tile), pb, dv);
        lds_reads_done();
        load_do(n + stride);
        accumulate(here(q_tile), dsb, dk);
        lds_reads_done();
        load_q(n + stride);
    }

    wait_async_loads();  // of nothing, but they write: the tiles are about to be used otherwise
    // dK, then dV, through the waves' own tiles
    if (splits == 1) {
        few_merge_store<DR, DT>(smem, STAGE, wave, lane, dk, p.scale, own.of(p.dk), own.row_off);
        __syncthreads();
        few_merge_store<DR, DT>(smem, STAGE, wave, lane, dv, 1.0f, own.of(p.dv), own.row_off);
        return;
    }
    float* unit = p.partials + (size_t)((blk.work * kFewWaves + blk.part) * splits + blk.split) * kUnitFloats(D) + lane * 4;
    auto keep = [&](float* to) {
        return [=](int strip, f32x4 a, f32x4 b) {
            *reinterpret_cast<f32x4*>(to + strip * 512) = a;
            *reinterpret_cast<f32x4*>(to + strip * 512 + 256) = b;
        };
    };
    few_sum_strips<DT>(smem, STAGE, wave, lane, dk, keep(unit));
    __syncthreads();
    few_sum_strips<DT>(smem, STAGE, wave, lane, dv, keep(unit + kUnitFloats(D) / 2));
}

// One workgroup per (work, part, dK or dV) adds the splits: every wave the strips it would have summed there.
template <int D, int DR>
__global__ __launch_bounds__(256) void bwd_dkdv_few_merge_kernel(AttnParams p, int splits) {
    constexpr int DT = (DR + 31) / 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int which = (int)blockIdx.x & 1, part = (int)blockIdx.x / 2 % kFewWaves, work = (int)blockIdx.x / (2 * kFewWaves);
    const int g = work % p.works_per_item;
    const KeyRows<D, DR> own(p, p.items[work / p.works_per_item], part, g, lane & 31);
    if (own.keys <= 0) return;
    const float* unit = p.partials + (size_t)((work * kFewWaves + part) * splits) * kUnitFloats(D) +
                        which * (kUnitFloats(D) / 2) + lane * 4;
    for (int strip = wave; strip < 2 * DT; strip += kFewWaves) {
        f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = a;
#pragma unroll 4
        for (int i = 0; i < splits; ++i) {
            const float* src = unit + (size_t)i * kUnitFloats(D) + strip * 512;
            a += *reinterpret_cast<const f32x4*>(src);
            b += *reinterpret_cast<const f32x4*>(src + 256);
        }
        few_store_strip<DR>(strip, a, b, which ? 1.0f : p.scale, lane, own.of(which ? p.dv : p.dk), own.row_off);
    }
}

template <int D, int DR = D>
hipError_t launch_dq_d(const AttnParams& p, bool only_delta, hipStream_t stream) {
    constexpr size_t smem = kFewWaves * 2 * kTileRows * D * 2;
    const hipError_t attr = VA_ALLOW_DYNAMIC_LDS((&bwd_dq_few_kernel<D, DR>), smem);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((bwd_dq_few_kernel<D, DR>), dim3(few_grid(p.num_items * p.works_per_item)), dim3(256), smem, stream, p,
                       rows_log2(kDqBlockRows / heads_per_block(p.Hq, p.Hkv)), only_delta);
    return hipGetLastError();
}

template <int D, int DR = D>
hipError_t launch_dkdv_d(const AttnParams& p, hipStream_t stream) {
    constexpr size_t smem = kFewWaves * (2 * kTileRows * D * 2 + 512) + kTileRows * D * 2;
    const hipError_t attr = VA_ALLOW_DYNAMIC_LDS((&bwd_dkdv_few_kernel<D, DR>), smem);
    if (attr != hipSuccess) return attr;
    const int works = p.num_items * p.works_per_item;
    hipLaunchKernelGGL((bwd_dkdv_few_kernel<D, DR>), dim3(few_grid(works, p.few_splits)), dim3(256), smem, stream, p,
                       p.few_splits);
    if (p.few_splits > 1)
        hipLaunchKernelGGL((bwd_dkdv_few_merge_kernel<D, DR>), dim3((unsigned)(works * kFewWaves * 2)), dim3(256), 0, stream, p,
                           p.few_splits);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_dq_few(const AttnParams& p, bool only_delta, hipStream_t stream) {
    switch (p.D) {
        case 48: return launch_dq_d<64, 48>(p, only_delta, stream);
        case 64: return launch_dq_d<64>(p, only_delta, stream);
        case 80: return launch_dq_d<128, 80>(p, only_delta, stream);
        case 96: return launch_dq_d<128, 96>(p, only_delta, stream);
        case 128: return launch_dq_d<128>(p, only_delta, stream);
        case 160: return launch_dq_d<256, 160>(p, only_delta, stream);
        case 192: return launch_dq_d<256, 192>(p, only_delta, stream);
        case 256: return launch_dq_d<256>(p, only_delta, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_bwd_dkdv_few(const AttnParams& p, hipStream_t stream) {
    switch (p.D) {
        case 48: return launch_dkdv_d<64, 48>(p, stream);
        case 64: return launch_dkdv_d<64>(p, stream);
        case 80: return launch_dkdv_d<128, 80>(p, stream);
        case 96: return launch_dkdv_d<128, 96>(p, stream);
        case 128: return launch_dkdv_d<128>(p, stream);
        case 160: return launch_dkdv_d<256, 160>(p, stream);
        case 192: return launch_dkdv_d<256, 192>(p, stream);
        case 256: return launch_dkdv_d<256>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace va
