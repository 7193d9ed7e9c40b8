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

// A wave per segment, four to a group: lane i holds packed words 4 i .. 4 i + 3, loaded at once (what lies past the end of the
// stream reads as 0).  Bound by HBM on long streams, by the launch on short ones: the words are staged in LDS in their order
// on the wire, so that whole runs of them are stored, and no wave waits for another.  Local update, quantise-and-pack and
// this call, a group of four waves per segment with a word per lane / so, us: one code in 16 3 M elements 14.1 / 13.6, 9.4 M
// 37.4 / 36.9, 25 M 92.4 / 90.9, 60 M 221.9 / 219.1;  one in 256 14.0 / 13.6, 37.2 / 36.8, 91.5 / 90.2, 221.0 / 217.9.
constexpr unsigned kEncodeWaves = 4;

__global__ __launch_bounds__(64 * kEncodeWaves) void k_sparse_encode(const uint32_t *__restrict__ packed, unsigned long long nw,
                                                                     uint32_t *__restrict__ sparse,
                                                                     uint32_t *__restrict__ seg_words, unsigned segments)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __shared__ unsigned staged[kEncodeWaves][kSegWords];
    const unsigned lane = threadIdx.x & 63u, wave = (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const unsigned s = blockIdx.x * kEncodeWaves + wave;
    if (s >= segments) return;
    const unsigned long long first = (unsigned long long)s * kSegWords, left = nw - first;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t *>(packed) + first, 0, (int)(4u * (left < kSegWords ? (unsigned)left : kSegWords)), kBufferFlags);
    const u4 v = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(16u * lane), 0, 0));
    unsigned nibble = 0u, at = 0u, total = 0u;
#pragma unroll
    for (unsigned c = 0; c < 4; ++c) {
        const unsigned long long sent = __ballot(v[c] != 0u);
        nibble |= (v[c] != 0u ? 1u : 0u) << c;
        at = __builtin_amdgcn_mbcnt_hi((unsigned)(sent >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)sent, at));
        total += (unsigned)__builtin_popcountll(sent);
    }
    // eight lanes' nibbles are a bitmap word
    unsigned bits = nibble << (4u * (lane & 7u));
    bits |= (unsigned)__builtin_amdgcn_mov_dpp((int)bits, 0xB1, 0xF, 0xF, true);   // quad_perm [1, 0, 3, 2]
    bits |= (unsigned)__builtin_amdgcn_mov_dpp((int)bits, 0x4E, 0xF, 0xF, true);   // quad_perm [2, 3, 0, 1]
    bits |= (unsigned)__builtin_amdgcn_mov_dpp((int)bits, 0x141, 0xF, 0xF, true);  // row_half_mirror
    uint32_t *seg = sparse + (size_t)s * kSegStride;
    if ((lane & 7u) == 0u) seg[lane >> 3] = bits;
    if (lane == 0u && seg_words) seg_words[s] = 8u + total;
#pragma unroll
    for (unsigned c = 0; c < 4; ++c)
        if (v[c] != 0u) staged[wave][at++] = v[c];
    // one wave's LDS operations run in order, only the compiler has to keep them so
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (unsigned i = lane; i < total; i += 64u) seg[8u + i] = staged[wave][i];
}

}  // namespace
