// Per-head OCP E4M3 quantisation on the device, bit-identical to the host
// routine va_quantize_e4m3_per_head: descale[h] = amax_h / 448 (1 for an
// all-zero head), code = round-to-nearest-even E4M3 of x / descale[h],
// saturating at +-448.  (The scaling vocabulary is that of section 2.2.3;
// applying it per attention head is this library's choice.)
//
// Two kernels on the caller's stream, no atomics on global memory and nothing to clear.  The rows are cut into
// R runs, one workgroup each.  The first kernel takes the per-head maxima of its run and leaves them in the
// code array, which nobody needs before the codes are written: once in the part of every one of the R
// workgroups.  In the second kernel a workgroup reads the R maxima of each head from its own part, and only
// then overwrites that part with codes, so no workgroup depends on another of the same launch.
//
// The block-wise quantiser (one scale per 128 tokens of one sample and one
// head, bit-identical to va_quantize_e4m3_blockwise) is one kernel further down.
#include "kernels.h"
#include "mfma_util.h"

namespace va {

namespace {

VA_DEV float bf16_bits_to_float(unsigned bits16) { return __builtin_bit_cast(float, bits16 << 16); }

typedef int i32x2 __attribute__((ext_vector_type(2)));

// |bf16| of the 8 values of a chunk as float bits, their maximum.  NaN patterns (above the bits of infinity)
// count as zero, as in the host routine, whose maximum drops them: a NaN in the input turns into the NaN
// code at its own place and leaves the scale of its head or block alone.
VA_DEV unsigned chunk_amax_bits(u32x4 raw) {
    unsigned m = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        // clear the sign, move the 16 bits to the top half
        const unsigned lo = (raw[w] & 0x7fffu) << 16, hi = raw[w] & 0x7fff0000u;
        m = max(m, lo > 0x7f800000u ? 0u : lo);
        m = max(m, hi > 0x7f800000u ? 0u : hi);
    }
    return m;
}

VA_DEV float descale_of(unsigned amax_bits) {
    const float s = __builtin_bit_cast(float, amax_bits) / 448.0f;
    return s > 0.0f ? s : 1.0f;
}

// A head's or block's descale with what the encoder needs beside it.
struct Scale {
    float d, r;    // descale and its reciprocal, both rounded once
    bool by_mult;  // d so far from the ends of the float32 range that no step of encode_chunk leaves the normal numbers
    VA_DEV explicit Scale(float descale) : d(descale), r(1.0f / descale), by_mult(descale > 0x1p-80f && descale < 0x1p120f) {}
};

// Eight bf16 values -> eight E4M3 codes of value / descale.  The quotient is the correctly rounded one in both
// branches: x * r is corrected once by its remainder.  (Both mantissas come from 8-bit numbers, so that was
// checked for every pair: the corrected product equals the division bit for bit, where x * r alone gives another
// code for some pairs on a rounding boundary.  The remainder is formed negated, q * d - x, which keeps the sign
// of a zero.)  A division is some ten instructions per value, and they, not memory, set the pace of these
// kernels.  |x| <= amax, so |quotient| rounds to at most 448 and needs no clamp.
VA_DEV i32x2 encode_chunk(u32x4 raw, const Scale& s) {
    float v[8];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        v[2 * w] = bf16_bits_to_float(raw[w] & 0xffffu);
        v[2 * w + 1] = __builtin_bit_cast(float, raw[w] & 0xffff0000u);
    }
    if (s.by_mult) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float q = v[e] * s.r;
            v[e] = __builtin_fmaf(-__builtin_fmaf(q, s.d, -v[e]), s.r, q);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] / s.d;
    }
    // The conversion instruction rounds to nearest even, subnormals included.  A NaN (the value itself, or
    // infinity over an infinite scale) becomes the NaN code with the sign it had: the host routine's is 0x7F,
    // so the sign goes wherever the other seven bits are all ones.
    i32x2 codes;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int word;  // the half the first conversion leaves alone is overwritten by the second: any old value serves
        asm volatile("" : "=v"(word));
        word = __builtin_amdgcn_cvt_pk_fp8_f32(v[4 * i], v[4 * i + 1], word, false);
        word = __builtin_amdgcn_cvt_pk_fp8_f32(v[4 * i + 2], v[4 * i + 3], word, true);
        const unsigned nan = ((unsigned)word & 0x7f7f7f7fu) + 0x01010101u;
        codes[i] = (int)((unsigned)word & ~(nan & 0x80808080u));
    }
    return codes;
}

// ---------------------------------------------------------------- per-head scales

constexpr int kQuantThreads = 1024;
constexpr int kQuantUnroll = 2;      // 16-byte loads a thread has in flight
constexpr int kMaxRuns = 256;        // one workgroup per CU; every run leaves its maxima in every other's part
constexpr int kHeadsPerGroup = 256;  // heads a workgroup handles (their maxima live in LDS)

// The share of workgroup (run i, head group y): token rows i, i + runs, i + 2 runs, ... and heads
// [h0, h0 + heads).  A thread stays on one column of 8 values, hence on one head, and walks down the rows.
struct QuantShare {
    int rows, h0, heads, columns, rows_at_once;
    size_t row_chunks;  // chunks of 8 values from one row of the run to the next
    VA_DEV QuantShare(int T, int H, int cpr, int runs) {
        rows = (T - 1 - (int)blockIdx.x) / runs + 1;
        h0 = (int)blockIdx.y * kHeadsPerGroup;
        heads = min(H - h0, kHeadsPerGroup);
        columns = heads * cpr;
        rows_at_once = max(1, kQuantThreads / columns);
        row_chunks = (size_t)runs * H * cpr;
    }
    // first chunk of the run
    VA_DEV size_t first(int H, int cpr) const { return ((size_t)blockIdx.x * H + h0) * cpr; }
    // f(row, chunk column, row step) for the thread's share; threads past the last whole row stay idle
    template <typename F>
    VA_DEV void for_columns(F f) const {
        if ((int)threadIdx.x >= columns * rows_at_once) return;
        for (int c = (int)threadIdx.x % columns; c < columns; c += kQuantThreads)
            f((int)threadIdx.x / columns % rows_at_once, c, rows_at_once);
    }
};

// Where word k of the maxima left for run r, head group [h0, h0 + heads) lies in the code array: in the rows of
// that run and the columns of those heads, row after row, so that only bytes the workgroup (r, y) will
// write itself are used.  The host chooses the number of runs so that R * heads words fit.
VA_DEV unsigned* partial_word(unsigned char* codes, int r, int k, int H, int D, int runs, int h0, int heads) {
    const int words_per_row = heads * D / 4;
    const size_t row = (size_t)(k / words_per_row) * runs + r;
    return reinterpret_cast<unsigned*>(codes + (row * H + h0) * D) + k % words_per_row;
}

// Mostly the read: the 67 MB of 16384 tokens x 16 heads x 128 take 14.1 us in a train of calls, 2.0 of them the maxima, which
// go a word at a time to every run (17.9 us behind other kernels).  A run is every R-th row, so that the workgroups
// sweep the tensor side by side: with runs of consecutive rows, which start at like addresses, it was 20.7 us instead
// of 17.9, and more loads in flight per thread made it worse (8 instead of 2: 24.8).
__global__ __launch_bounds__(kQuantThreads) void quant_partial_max_kernel(const u32x4* x, int T, int H, int D, int runs,
                                                                         unsigned char* codes) {
    __shared__ unsigned head_max[kHeadsPerGroup];
    const int cpr = D / 8;
    const QuantShare mine(T, H, cpr, runs);
    for (int h = threadIdx.x; h < mine.heads; h += kQuantThreads) head_max[h] = 0u;
    __syncthreads();
    mine.for_columns([&](int row, int c, int step) {
        const u32x4* col = x + mine.first(H, cpr) + c;
        unsigned m = 0u;
        for (; row < mine.rows; row += kQuantUnroll * step) {
            u32x4 raw[kQuantUnroll];
#pragma unroll
            for (int j = 0; j < kQuantUnroll; ++j)  // past the end: the last row again, which changes no maximum
                raw[j] = col[(size_t)min(row + j * step, mine.rows - 1) * mine.row_chunks];
#pragma unroll
            for (int j = 0; j < kQuantUnroll; ++j) m = max(m, chunk_amax_bits(raw[j]));
        }
        atomicMax(&head_max[c / cpr], m);
    });
    __syncthreads();
    for (int i = threadIdx.x; i < runs * mine.heads; i += kQuantThreads) {
        const int h = i % mine.heads;
        *partial_word(codes, i / mine.heads, (int)blockIdx.x * mine.heads + h, H, D, runs, mine.h0, mine.heads) = head_max[h];
    }
}

// Maxima of all runs from the workgroup's own part of the code array, then the codes over them.
__global__ __launch_bounds__(kQuantThreads) void quant_encode_kernel(const u32x4* x, int T, int H, int D, int runs,
                                                                    unsigned char* codes, float* descale) {
    __shared__ unsigned head_max[kHeadsPerGroup];
    const int cpr = D / 8;
    const QuantShare mine(T, H, cpr, runs);
    for (int h = threadIdx.x; h < mine.heads; h += kQuantThreads) head_max[h] = 0u;
    __syncthreads();
    for (int i = threadIdx.x; i < runs * mine.heads; i += kQuantThreads)
        atomicMax(&head_max[i % mine.heads],
                  *partial_word(codes, (int)blockIdx.x, i, H, D, runs, mine.h0, mine.heads));
    __syncthreads();  // every word has been read: the codes may overwrite them
    if (blockIdx.x == 0)
        for (int h = threadIdx.x; h < mine.heads; h += kQuantThreads) descale[mine.h0 + h] = descale_of(head_max[h]);
    mine.for_columns([&](int row, int c, int step) {
        const size_t col = mine.first(H, cpr) + c;
        const Scale s(descale_of(head_max[c / cpr]));
        for (; row < mine.rows; row += kQuantUnroll * step) {
            u32x4 raw[kQuantUnroll];
            size_t at[kQuantUnroll];
#pragma unroll
            for (int j = 0; j < kQuantUnroll; ++j) {
                at[j] = (size_t)min(row + j * step, mine.rows - 1) * mine.row_chunks + col;
                raw[j] = x[at[j]];
            }
#pragma unroll
            for (int j = 0; j < kQuantUnroll; ++j)  // past the end: the last row's codes again
                *reinterpret_cast<i32x2*>(codes + at[j] * 8) = encode_chunk(raw[j], s);
        }
    });
}

__global__ void quant_all_zero_kernel(float* descale, int H) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h < H) descale[h] = 1.0f;
}

// Block-wise variant: a block is up to kBlockTokens consecutive tokens of one sample, one head.
constexpr int kBlockTokens = 128;

// Rows [r0, r1) of block number b in sample order, found by a prefix sum over the samples' block counts,
// 64 samples at a time; every lane of the wave returns the same pair.  An empty range means "no such
// block".  The range is clipped to [0, T), whatever cu holds.
VA_DEV void find_block(const int* cu, int n, int T, int b, int lane, int* r0_out, int* r1_out) {
    int r0 = 0, r1 = 0;
    for (int base = 0; base < n; base += 64) {
        const int s = base + lane;
        int c0 = 0, c1 = 0;
        if (s < n) {
            c0 = cu[s];
            c1 = cu[s + 1];
        }
        const int nb = c1 > c0 ? (c1 - c0 + kBlockTokens - 1) / kBlockTokens : 0;
        int incl = nb;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d);
            if (lane >= d) incl += up;
        }
        const int total = __shfl(incl, 63);
        if (b < total) {
            const int src = __ffsll((unsigned long long)__ballot(b < incl)) - 1;  // the sample that holds block b
            const int first = __shfl(incl - nb, src);
            r0 = __shfl(c0, src) + (b - first) * kBlockTokens;
            r1 = min(__shfl(c1, src), r0 + kBlockTokens);
            break;
        }
        b -= total;
    }
    *r0_out = max(r0, 0);
    *r1_out = min(r1, T);
}

// Head dimensions up to 256.  A workgroup takes block number b in sample order and head h; wave w takes the
// rows 32 w .. 32 w + 31 of the block and keeps them in registers (J chunks of 8 values per lane), so x is
// read once: maximum per wave, the four maxima meet in LDS, then every wave encodes what it holds.
// Workgroup number (b / 8) 8 H + 8 h + b % 8: the heads of a block follow each other on one XCD, so that their
// scales, 4 bytes each of the same lines, meet in one L2 instead of reaching memory as partial lines.
template <int J>
__global__ __launch_bounds__(256) void quant_blockwise_kernel(const uint16_t* x, const int* cu, int n, int T, int H,
                                                              int chunks_per_row, unsigned char* codes,
                                                              float* descale_tok) {
    __shared__ unsigned wave_max[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = (int)(blockIdx.x / kXcds) % H;
    int r0, r1;
    find_block(cu, n, T, (int)(blockIdx.x / (kXcds * (unsigned)H) * kXcds + blockIdx.x % kXcds), lane, &r0, &r1);
    if (r0 >= r1) return;  // the same for the whole workgroup (the number of blocks is rounded up to the XCDs)
    const int w0 = r0 + 32 * wave;
    const int wrows = max(0, min(32, r1 - w0));  // rows of this wave
    const int chunks = wrows * chunks_per_row;
    const int row_bytes = H * chunks_per_row * 16;
    const size_t first = ((size_t)w0 * H + h) * chunks_per_row;  // first chunk of this wave, in chunks
    // the ranges end with the wave's last row of this head: nothing outside them can be touched
    const unsigned span = wrows > 0 ? (unsigned)(wrows - 1) * row_bytes + chunks_per_row * 16 : 0u;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(reinterpret_cast<const char*>(x)) + (wrows > 0 ? first * 16 : 0), 0, (int)span, 0x00020000);
    const __amdgpu_buffer_rsrc_t dst =
        __builtin_amdgcn_make_buffer_rsrc(codes + (wrows > 0 ? first * 8 : 0), 0, (int)(span / 2), 0x00020000);
    u32x4 raw[J];
    int at[J];  // byte offset of the lane's chunk j in x (half of it in codes), out of range where it has none
    unsigned m = 0u;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = lane + 64 * j;
        at[j] = i < chunks ? (i / chunks_per_row) * row_bytes + (i % chunks_per_row) * 16 : (int)0x7ffffff0;
        raw[j] = __builtin_amdgcn_raw_buffer_load_b128(src, at[j], 0, 0);  // zero where out of range
    }
#pragma unroll
    for (int j = 0; j < J; ++j) m = max(m, chunk_amax_bits(raw[j]));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d));
    if (lane == 0) wave_max[wave] = m;
    __syncthreads();
    const float descale = descale_of(max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3])));
    const Scale scale(descale);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        const int off = at[j] == (int)0x7ffffff0 ? at[j] : at[j] / 2;
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, encode_chunk(raw[j], scale)), dst, off, 0, 0);
    }
    const int r = r0 + 64 * (wave & 1) + lane;  // waves 0 and 1 write the scales of the block's rows
    if (wave < 2 && r < r1) descale_tok[(size_t)r * H + h] = descale;
}

// Any head dimension: workgroup (b, y), wave w takes head 4 y + w and the whole block, reads it twice
// (maximum, then encoding).  Waves do not interact.

__global__ __launch_bounds__(256) void quant_blockwise_two_pass_kernel(const uint16_t* x, const int* cu, int n, int T,
                                                                       int H, int chunks_per_row, unsigned char* codes,
                                                                       float* descale_tok) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = blockIdx.y * 4 + wave;
    if (h >= H) return;
    int r0, r1;
    find_block(cu, n, T, (int)blockIdx.x, lane, &r0, &r1);
    if (r0 >= r1) return;
    const int rows = r1 - r0, chunks = rows * chunks_per_row;
    const size_t row_chunks = (size_t)H * chunks_per_row;  // chunks from one token row to the next
    const uint16_t* xb = x + ((size_t)r0 * H + h) * chunks_per_row * 8;
    unsigned m = 0u;
    for (int i = lane; i < chunks; i += 64) {
        const size_t at = ((size_t)(i / chunks_per_row) * row_chunks + i % chunks_per_row) * 8;
        m = max(m, chunk_amax_bits(*reinterpret_cast<const u32x4*>(xb + at)));
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d));
    const float descale = descale_of(m);
    const Scale scale(descale);
    unsigned char* cb = codes + ((size_t)r0 * H + h) * chunks_per_row * 8;
    for (int i = lane; i < chunks; i += 64) {
        const size_t at = ((size_t)(i / chunks_per_row) * row_chunks + i % chunks_per_row) * 8;
        *reinterpret_cast<i32x2*>(cb + at) = encode_chunk(*reinterpret_cast<const u32x4*>(xb + at), scale);
    }
    for (int r = lane; r < rows; r += 64) descale_tok[(size_t)(r0 + r) * H + h] = descale;
}

}  // namespace

hipError_t launch_quantize_e4m3(const void* x, int32_t T, int32_t H, int32_t D, void* codes, float* descale,
                                hipStream_t stream) {
    if (T == 0) {
        hipLaunchKernelGGL(quant_all_zero_kernel, dim3((unsigned)((H + 255) / 256)), dim3(256), 0, stream, descale, H);
        return hipGetLastError();
    }
    // as many runs as CUs, unless their maxima would not fit the rows of one run: T / runs rows of D bytes
    // per head against one word per head from every run
    int32_t runs = std::min(T, kMaxRuns);
    while (runs > 1 && (int64_t)(T / runs) * D < (int64_t)4 * runs) --runs;
    const dim3 grid((unsigned)runs, (unsigned)((H + kHeadsPerGroup - 1) / kHeadsPerGroup));
    const u32x4* xs = static_cast<const u32x4*>(x);
    unsigned char* cs = static_cast<unsigned char*>(codes);
    hipLaunchKernelGGL(quant_partial_max_kernel, grid, dim3(kQuantThreads), 0, stream, xs, T, H, D, runs, cs);
    hipLaunchKernelGGL(quant_encode_kernel, grid, dim3(kQuantThreads), 0, stream, xs, T, H, D, runs, cs, descale);
    return hipGetLastError();
}

hipError_t launch_quantize_e4m3_blockwise(const void* x, const int32_t* cu_device, int32_t num_seqs, int32_t T,
                                          int32_t num_blocks, int32_t H, int32_t D, void* codes, float* descale_tok,
                                          hipStream_t stream) {
    if (num_blocks == 0) return hipSuccess;
    const uint16_t* xs = static_cast<const uint16_t*>(x);
    unsigned char* cs = static_cast<unsigned char*>(codes);
    const int cpr = D / 8;
    const int64_t wgs = (int64_t)((num_blocks + kXcds - 1) / kXcds * kXcds) * H;
    const dim3 grid((unsigned)wgs);
    const bool one_pass = wgs <= INT32_MAX / 256;
    // a wave holds 32 rows: 32 * cpr chunks over 64 lanes
    if (cpr <= 8 && one_pass)
        hipLaunchKernelGGL(quant_blockwise_kernel<4>, grid, dim3(256), 0, stream, xs, cu_device, num_seqs, T, H, cpr, cs, descale_tok);
    else if (cpr <= 16 && one_pass)
        hipLaunchKernelGGL(quant_blockwise_kernel<8>, grid, dim3(256), 0, stream, xs, cu_device, num_seqs, T, H, cpr, cs, descale_tok);
    else if (cpr <= 32 && one_pass)
        hipLaunchKernelGGL(quant_blockwise_kernel<16>, grid, dim3(256), 0, stream, xs, cu_device, num_seqs, T, H, cpr, cs, descale_tok);
    else
        hipLaunchKernelGGL(quant_blockwise_two_pass_kernel, dim3((unsigned)num_blocks, (unsigned)((H + 3) / 4)), dim3(256), 0,
                           stream, xs, cu_device, num_seqs, T, H, cpr, cs, descale_tok);
    return hipGetLastError();
}

}  // namespace va
