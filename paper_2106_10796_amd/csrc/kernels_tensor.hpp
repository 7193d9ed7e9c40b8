// Single-tensor kernels: quantise-and-pack (a1-a3), update (a5, a6).
#pragma once

namespace {

// How the caches are used, by the length of the tensor (one tensor of elements, several sets of buffers in turn; time
// over that of non-temporal loads and stores throughout).
//   kSmallTensor  up to 1.5 M elements: results are written through and stay in the 256 MB memory-side cache
//                 (0.1 M elements, local rule / global rule / both / quantise-and-pack: .93 / .92 / .94 / .96; 1 M 1.01 /
//                 .99 / .94 / .97)
//   kMidTensor    up to 24 M: they are written through and do not stay (2 M .98 / 1.04 / .97 / .94, 4 M .97 / 1.00 / .96 /
//                 .92, 16 M .98 / 1.01 / .99 / .95; staying costs 16 M 1.16 / .84 / 1.13 / 1.11, the weights that the
//                 global rule alone writes being in the cache still when it reads them next)
//   kLargeTensor  the same, and the gradient does not stay either (80 M .97 / 1.00 / 1.00 / .97)
// With decode-and-sum in front, which leaves the aggregate in the cache, the global rule gains as well (N = 32, 16 M,
// both calls: 64.4 us, 63.2 now; N = 12, 60 M: 163.8 and 161.6).
// Local update, quantise-and-pack and sparse encoding one after the other, before / now, us: 4 M 17.8 / 17.3, 9 M 39.2 /
// 37.3, 16 M 61.7 / 58.8, 90 M 333.9 / 327.6.
// The gradient of a worker's own tensor is read twice, by the update and by the quantiser: up to kKeepElems elements
// its loads take the default cache policy, and the second pass finds it in the memory-side cache.
// Update and quantise-and-pack one after the other, non-temporal / default policy: 4 M elements 18.2 / 16.9 us, 9 M
// 38.2 / 36.4, 16 M 65.1 / 62.3, 32 M 123.9 / 123.1, 64 M 241 / 241, 100 M 375 / 383.
constexpr int kSmallTensor = 0, kMidTensor = 1, kLargeTensor = 2;
constexpr size_t kSmallElems = (size_t)3 << 19, kKeepElems = (size_t)24 << 20;
template <int LEN>
constexpr int kTensorStore = LEN == kSmallTensor ? kThrough : kThroughStream;

// a5 + a6 (eq. 10, eq. 11) for one tensor, both from the weight that was loaded, in single-wave pieces of
// 64 quads (`ext` in pieces, as for k_quantize_pack; measured on 2^27 elements: 6.29 TB/s against 6.02 TB/s
// for 512-lane workgroups with two quads per lane).
template <bool G, bool LOCAL, bool GLOBAL, int LEN>
__device__ __forceinline__ void update_piece(float *__restrict__ wg, float *__restrict__ wl,
                                             const float *__restrict__ grad, const float *__restrict__ agg,
                                             unsigned rem_elems, float lr_local, float scale)
{
    const unsigned lane = threadIdx.x;
    const int cnt = quad_count<G>(rem_elems, lane);
    const f4 w = ld4g<G>(wg, lane, cnt);
    f4 g = {0.0f, 0.0f, 0.0f, 0.0f}, a = {0.0f, 0.0f, 0.0f, 0.0f};
    if (LOCAL) g = LEN != kLargeTensor && (!G || cnt == 4) ? ld4_kept(grad, lane) : ld4g<G>(grad, lane, cnt);
    if (GLOBAL) a = ld4g<G>(agg, lane, cnt);
    if (LOCAL) {
        f4 v;
#pragma unroll
        for (unsigned c = 0; c < 4; ++c) v[c] = __builtin_fmaf(-lr_local, g[c], w[c]);
        st4g<G, kTensorStore<LEN>>(wl, lane, cnt, v);
    }
    if (GLOBAL) {
        f4 v;
#pragma unroll
        for (unsigned c = 0; c < 4; ++c) v[c] = __builtin_fmaf(-scale, a[c], w[c]);
        st4g<G, kTensorStore<LEN>>(wg, lane, cnt, v);
    }
}

template <bool LOCAL, bool GLOBAL, int LEN>
__global__ __launch_bounds__(64) void k_update(float *__restrict__ wg, float *__restrict__ wl,
                                                     const float *__restrict__ grad, const float *__restrict__ agg,
                                                     Extent ext, float lr_local, float scale)
{
    const unsigned piece = blockIdx.x;
    const size_t quad0 = (size_t)piece * 64u;
    wg += 4 * quad0;
    if (LOCAL) {
        wl += 4 * quad0;
        grad += 4 * quad0;
    }
    if (GLOBAL) agg += 4 * quad0;
    if (piece < ext.full_chunks) update_piece<false, LOCAL, GLOBAL, LEN>(wg, wl, grad, agg, 256u, lr_local, scale);
    else update_piece<true, LOCAL, GLOBAL, LEN>(wg, wl, grad, agg, ext.tail_elems, lr_local, scale);
}

// a1-a3 for one tensor, one wave per piece of L = 64 quads (measured: 6.68 TB/s against 6.41 TB/s for
// 512-lane workgroups with two quads per lane).  `ext` describes the tensor in pieces: full_chunks whole pieces, then at most one
// ragged piece of tail_elems elements and tail_bytes packed bytes.
template <unsigned L, int LEN>
__global__ __launch_bounds__(L) void k_quantize_pack(const float *__restrict__ grad, float *__restrict__ resid,
                                                       uint8_t *__restrict__ packed, Extent ext, float t)
{
    const unsigned piece = blockIdx.x, lane = threadIdx.x;
    const size_t quad0 = (size_t)piece * L;
    grad += 4 * quad0;
    resid += 4 * quad0;
    packed += quad0;
    f4 sent;
    if (piece < ext.full_chunks) {
        const f4 g = LEN != kLargeTensor ? ld4_kept(grad, lane) : ld4(grad, lane);
        f4 r = ld4(resid, lane);
        const unsigned b = quantize_quad(g, r, t, sent);
        st4p<kTensorStore<LEN>>(resid, lane, r);
        packed[lane] = (uint8_t)b;
    } else {
        const int cnt = quad_count<true>(ext.tail_elems, lane);
        const f4 g = ld4g<true>(grad, lane, cnt);
        f4 r = ld4g<true>(resid, lane, cnt);
        const unsigned b = quantize_quad(g, r, t, sent);
        st4g<true, kTensorStore<LEN>>(resid, lane, cnt, r);
        if (lane < ext.tail_bytes) packed[lane] = (uint8_t)b;
    }
}

}  // namespace
