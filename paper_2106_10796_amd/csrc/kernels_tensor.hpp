// Single-tensor kernels: quantise-and-pack (a1-a3), update (a5, a6).
#pragma once

namespace {

// How the caches are used, by the length of the tensor (several sets of buffers in turn).
//   kSmallTensor  up to 7 M elements (the global rule: see weights_stay): results are written through and stay in the
//                 256 MB memory-side cache, but for the local weights (kLocalStore)
//   kMidTensor    up to 24 M: they are written through and do not stay
//   kLargeTensor  the same, and the gradient does not stay either
//   kDrainTensor  results are stored non-temporally (the global rule alone, see drains_results)
// Local update and quantise-and-pack, us, non-temporal stores / kMidTensor / kSmallTensor: 2 M elements 9.3 / 9.9 / 9.1, 3 M
// 13.2 / 13.1 / 11.8, 5 M 19.0 / 18.1 / 16.9, 7 M 26.4 / 26.8 / 26.2, 8 M 31.3 / 29.8 / 30.2, 9.4 M and encoding 39.5 / 37.6
// / 38.6, 13 M 48.6 / 46.6 / 52.2;  gradient kept or not, 90 M and encoding 333.9 / 327.6.
// Decode-and-sum, which leaves the aggregate in the cache, and the global rule: N = 24, 3 M 13.5 / 12.9 / 12.1, 7 M 26.4 /
// 24.7 / 24.1, 9 M 32.5 / 30.3 / 32.2, 12 M 42.0 / 40.9 / 43.6;  N = 8, 4 M 13.0 / 12.8 / 12.3, 9 M 26.8 / 25.5 / 24.7.
// The gradient of a worker's own tensor is read twice, by the update and by the quantiser: up to kKeepElems elements
// its loads take the default cache policy, and the second pass finds it in the memory-side cache.
// Update and quantise-and-pack one after the other, non-temporal / default policy: 4 M elements 18.2 / 16.9 us, 9 M
// 38.2 / 36.4, 16 M 65.1 / 62.3, 32 M 123.9 / 123.1, 64 M 241 / 241, 100 M 375 / 383.
constexpr int kSmallTensor = 0, kMidTensor = 1, kLargeTensor = 2, kDrainTensor = 3;
constexpr size_t kSmallElems = (size_t)7 << 20, kKeepElems = (size_t)24 << 20;
template <int LEN>
constexpr int kTensorStore = LEN == kSmallTensor ? kThrough : (LEN == kDrainTensor ? kStream : kThroughStream);
// ... of the local weights, which neither call reads again: they are left out of the cache at every length.  Local update and
// quantise-and-pack, time over that of non-temporal stores throughout, three sets of buffers in turn / 600 MB of sets / 1500 MB of
// sets, with the local weights staying, then so: 2 M .99 / 1.02 / .98, .99 / .95 / .97;  3 M .88 / 1.03 / 1.02, .90 / .95 / .98;  4 M .90 /
// 1.00 / .99, .91 / .91 / .99;  5 M .90 / 1.01 / 1.00, .91 / .94 / .99;  6 M .98 / 1.06 / 1.08, .91 / .97 / 1.02;  7 M 1.02 / 1.04 / 1.11, .92 /
// .95 / 1.04.
template <int LEN>
constexpr int kLocalStore = LEN == kSmallTensor ? kStream : kTensorStore<LEN>;

// a5 + a6 (eq. 10, eq. 11) for one tensor, both from the weight that was loaded, in single-wave pieces of
// 64 quads (`ext` in pieces, as for k_quantize_pack; measured on 2^27 elements: 6.29 TB/s against 6.02 TB/s
// for 512-lane workgroups with two quads per lane).
template <bool G, bool LOCAL, bool GLOBAL, int LEN>
__device__ __forceinline__ void update_piece(float *__restrict__ wg, float *__restrict__ wl,
                                             const float *__restrict__ grad, const float *__restrict__ agg,
                                             unsigned rem_elems, float lr_local, float scale)
{
    const unsigned lane = threadIdx.x;
    const f4 w = ld4g<G>(wg, lane, rem_elems);
    f4 g = {0.0f, 0.0f, 0.0f, 0.0f}, a = {0.0f, 0.0f, 0.0f, 0.0f};
    if (LOCAL) g = ld4g<G, LEN != kLargeTensor ? 0 : kLoad>(grad, lane, rem_elems);
    if (GLOBAL) a = ld4g<G>(agg, lane, rem_elems);
    if (LOCAL) {
        f4 v;
#pragma unroll
        for (unsigned c = 0; c < 4; ++c) v[c] = __builtin_fmaf(-lr_local, g[c], w[c]);
        st4g<G, kLocalStore<LEN>>(wl, lane, rem_elems, v);
    }
    if (GLOBAL) {
        f4 v;
#pragma unroll
        for (unsigned c = 0; c < 4; ++c) v[c] = __builtin_fmaf(-scale, a[c], w[c]);
        st4g<G, kTensorStore<LEN>>(wg, lane, rem_elems, v);
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

// The packed codes are written through and stay in the memory-side cache at every length, where the call that sends or encodes
// them reads them; at the default policy they are left to the flush of the L2s at the end of the kernel.  Local update and this
// call, packed codes at the default policy / so, us: 2 M elements 8.6 / 8.4, 3 M 11.5 / 11.3, 7 M 24.1 / 23.0, 9.4 M 34.6 / 34.4,
// 25 M 86.3 / 86.0, 60 M 213.7 / 211.6;  and encoding 2 M 10.9 / 10.6, 7 M 26.5 / 25.4, 25 M 91.2 / 90.9, 60 M 219.4 / 217.6;
// twelve sets of buffers in turn .98 to 1.00 (not staying: the encoder 1 % slower).
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
        st_code<kThrough>(packed, lane, b);
    } else {
        const f4 g = ld4g<true, LEN != kLargeTensor ? 0 : kLoad>(grad, lane, ext.tail_elems);
        f4 r = ld4g<true>(resid, lane, ext.tail_elems);
        const unsigned b = quantize_quad(g, r, t, sent);
        st4g<true, kTensorStore<LEN>>(resid, lane, ext.tail_elems, r);
        if (lane < ext.tail_bytes) st_code<kThrough>(packed, lane, b);
    }
}

}  // namespace
