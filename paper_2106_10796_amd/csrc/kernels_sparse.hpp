// Sparse form of a packed stream: its geometry and the encoder.
#pragma once

namespace {

// ---------------------------------------------------------------------------
// Sparse form of a packed stream (this library's own wire format, see cdsgd.h)
// ---------------------------------------------------------------------------
// A segment is the 256 packed words of one chunk: 8 bitmap words (bit b of word m set iff packed
// word 32 m + b of the segment is non-zero), then the non-zero words in index order.  Segments
// sit at a fixed stride of 264 words.
constexpr unsigned kSegWords = 256;
constexpr unsigned kSegStride = 8 + kSegWords;
static_assert(kChunkQuads == 4 * kSegWords, "a segment of the sparse form is the packed stream of one chunk");

// One workgroup of 256 lanes per segment: lane i owns packed word i.
__global__ __launch_bounds__(256) void k_sparse_encode(const uint32_t *__restrict__ packed, unsigned long long nw,
                                                       uint32_t *__restrict__ sparse,
                                                       uint32_t *__restrict__ seg_words)
{
    __shared__ unsigned wave_count[4];
    const unsigned i = threadIdx.x, wave = i >> 6, lane = i & 63u;
    const unsigned long long w = (unsigned long long)blockIdx.x * kSegWords + i;
    const uint32_t v = w < nw ? packed[w] : 0u;
    const unsigned long long mask = __ballot(v != 0u);  // the wave's 64 words: two bitmap words
    if (lane == 0) wave_count[wave] = (unsigned)__builtin_popcountll(mask);
    __syncthreads();
    unsigned before = 0, total = 0;
#pragma unroll
    for (unsigned x = 0; x < 4; ++x) {
        if (x < wave) before += wave_count[x];
        total += wave_count[x];
    }
    uint32_t *seg = sparse + (size_t)blockIdx.x * kSegStride;
    if (lane == 0) {
        seg[2 * wave] = (uint32_t)mask;
        seg[2 * wave + 1] = (uint32_t)(mask >> 32);
    }
    if (v != 0u) seg[8u + before + (unsigned)__builtin_popcountll(mask & ((1ull << lane) - 1ull))] = v;
    if (i == 0 && seg_words) seg_words[blockIdx.x] = 8u + total;
}

}  // namespace
