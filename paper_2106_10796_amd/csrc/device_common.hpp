// What every kernel shares: the chunk geometry, 128-bit loads and stores with ragged ends,
// widening of 16-bit gradients, and the error-feedback quantiser (Sec. 2.3, Sec. 3.4.1).
#pragma once

namespace {

constexpr unsigned kChunkQuads = 1024;            // quads (= packed bytes) per chunk
constexpr unsigned kChunkElems = kChunkQuads * 4; // elements per chunk
static_assert(CDSGD_GRAD_F32 == 0 && CDSGD_GRAD_BF16 == 1 && CDSGD_GRAD_F16 == 2, "header and kernels agree");

typedef float f4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// 128-bit loads / stores, with the ragged end of a tensor handled per element
// ---------------------------------------------------------------------------
// Pointers that a kernel reads from a table are generic to the compiler, and it would access them with flat
// instructions, which count as LDS operations too: every wait for LDS, and every wait for some of the loads in
// flight, then becomes a wait for all of them.  All data buffers are global memory, and are accessed as that.
#define CDSGD_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ CDSGD_GLOBAL T *global_ptr(T *p)
{
    return (CDSGD_GLOBAL T *)p;
}

__device__ __forceinline__ f4 ld4(const float *base, unsigned qi)
{
    const CDSGD_GLOBAL f4 *p = global_ptr(reinterpret_cast<const f4 *>(base)) + qi;
#if CDSGD_NT_LOAD
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}

// The same with the default cache policy: for what the next call reads again.
__device__ __forceinline__ f4 ld4_kept(const float *base, unsigned qi)
{
    return *(global_ptr(reinterpret_cast<const f4 *>(base)) + qi);
}

__device__ __forceinline__ void st4(float *base, unsigned qi, f4 v)
{
    CDSGD_GLOBAL f4 *p = global_ptr(reinterpret_cast<f4 *>(base)) + qi;
#if CDSGD_NT_STORE
    __builtin_nontemporal_store(v, p);
#else
    *p = v;
#endif
}

// Stores that are written through the L2 of the compute die to memory, so that no dirty line is left for the flush at
// the end of the kernel (2.2 us after a kernel that writes at the default policy).  Non-temporal stores leave some: the
// lines that the flush wrote back were 33,000 of 383,000 in a compressed pass over 4 M elements, N = 16, 55,000 of 192,000
// over 2 M in bf16, and are none so (TCC_ALL_TC_OP_WB_WRITEBACK; TCC_WRITEBACK).
//   kThrough        the lines stay in the 256 MB memory-side cache: for what the next call reads
//   kThroughStream  they do not: for what is read again a training step later
// Policies of a buffer instruction: 1 and 16 are the scope bits sc0 and sc1, 2 is nt.
constexpr int kStream = 2, kThrough = 17, kThroughStream = 19;

constexpr unsigned kBufferFlags = 0x00027000;  // raw buffer, range checked in bytes

// A quad at most a chunk behind `base`, which is the same in all lanes.
template <int POLICY>
__device__ __forceinline__ void st4p(float *base, unsigned qi, f4 v)
{
    static_assert(POLICY == kStream || POLICY == kThrough || POLICY == kThroughStream, "policies in use");
    if constexpr (POLICY == kStream) {
        st4(base, qi, v);
    } else {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)(kChunkElems * sizeof(float)), kBufferFlags);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), rsrc, (int)(qi * 16u), 0, POLICY);
    }
}

// A lane's byte of the packed stream, at most a chunk behind `base`.  POLICY 0: the default.
template <int POLICY>
__device__ __forceinline__ void st_code(uint8_t *base, unsigned qi, unsigned byte)
{
    if constexpr (POLICY != 0) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)kChunkQuads, kBufferFlags);
        __builtin_amdgcn_raw_buffer_store_b8((unsigned char)byte, rsrc, (int)qi, 0, POLICY);
    } else {
        global_ptr(base)[qi] = (uint8_t)byte;
    }
}

// Ragged ends (G): a quad of a buffer of which `elems` elements are left from `base` on (the same in all lanes).  The range
// check of a buffer instruction, which works word by word, stands in for the tests: what lies past the end is loaded as 0 and
// not stored.  The loads of a ragged tile then wait for one another no more than those of a whole one; with a load per element
// behind a test of its own, and 16-bit elements widened behind each test, the last tile of a list ended several trips to
// memory after all others (16-bit gradients, an odd number of elements, us, before / now: compressed pass, N = 4, 0.7 M 5.1 / 4.0,
// 1 M 6.4 / 4.5, 2 M 9.7 / 8.7, 4 M 16.2 / 16.0;  correction pass with the kernel sum, N = 16, 0.25 M 12.1 / 6.3, 1 M 14.7 / 9.1,
// 4 M 31.3 / 28.5;  32-bit gradients the same within 1 %, update and quantise-and-pack of 2 M 9.2 / 8.8).
constexpr int kLoad = CDSGD_NT_LOAD ? kStream : 0;

// Elements left from `first` on, in a scalar register (a difference that saturates is a vector operation to the compiler).
__device__ __forceinline__ unsigned elems_from(unsigned first, unsigned elems)
{
    return (unsigned)__builtin_amdgcn_readfirstlane((int)(elems > first ? elems - first : 0u));
}

template <bool G, int POLICY = kLoad>
__device__ __forceinline__ f4 ld4g(const float *base, unsigned qi, unsigned elems)
{
    static_assert(POLICY == kStream || POLICY == 0, "policies in use");
    if constexpr (!G) {
        return POLICY == kStream ? ld4(base, qi) : ld4_kept(base, qi);
    } else {
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, (int)(elems * 4u), kBufferFlags);
        return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(qi * 16u), 0, POLICY));
    }
}

template <bool G, int POLICY = kStream>
__device__ __forceinline__ void st4g(float *base, unsigned qi, unsigned elems, f4 v)
{
    if constexpr (!G) {
        st4p<POLICY>(base, qi, v);
    } else {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)(elems * 4u), kBufferFlags);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), rsrc, (int)(qi * 16u), 0, POLICY);
    }
}

// Gradient element types: fp32, or bf16 / fp16 widened exactly to fp32 (everything downstream is the fp32 path).  A load
// and its widening are two steps, so that several loads can be asked for before the first is waited for.
constexpr int kGradF32 = 0, kGradBF16 = 1, kGradF16 = 2;

template <int GT>
__device__ __forceinline__ constexpr unsigned grad_bytes()
{
    return GT == kGradF32 ? 4u : 2u;
}

typedef unsigned u2 __attribute__((ext_vector_type(2)));

// A quad as it was loaded.  last: a ragged end's last element where its word is only half inside the buffer, else 0.
template <int GT>
struct GradQuad {
    u2 v;
    unsigned last;
};
template <>
struct GradQuad<kGradF32> {
    f4 v;
};

// One quad of a gradient buffer; `base` is the chunk's (or piece's) first element.
template <bool G, int GT>
__device__ __forceinline__ GradQuad<GT> load_grad(const void *base, unsigned qi, unsigned elems)
{
    GradQuad<GT> q;
    if constexpr (GT == kGradF32) {
        q.v = ld4g<G>(static_cast<const float *>(base), qi, elems);
    } else if constexpr (!G) {
        const CDSGD_GLOBAL u2 *p = global_ptr(static_cast<const u2 *>(base)) + qi;
#if CDSGD_NT_LOAD
        q.v = __builtin_nontemporal_load(p);
#else
        q.v = *p;
#endif
        q.last = 0u;
    } else {
        void *b = const_cast<void *>(base);
        const __amdgpu_buffer_rsrc_t words = __builtin_amdgcn_make_buffer_rsrc(b, 0, (int)(elems / 2u * 4u), kBufferFlags);
        const __amdgpu_buffer_rsrc_t halves = __builtin_amdgcn_make_buffer_rsrc(b, 0, (int)(elems * 2u), kBufferFlags);
        q.v = __builtin_bit_cast(u2, __builtin_amdgcn_raw_buffer_load_b64(words, (int)(qi * 8u), 0, kLoad));
        const bool mine = (elems & 1u) != 0u && qi == elems / 4u;
        q.last = __builtin_amdgcn_raw_buffer_load_b16(halves, mine ? (int)(elems * 2u - 2u) : 0x7FFFFFF0, 0, kLoad);
    }
    return q;
}

template <int GT>
__device__ __forceinline__ float widen16(unsigned h)  // h: the 16-bit pattern in the low half
{
    if (GT == kGradBF16) return __builtin_bit_cast(float, h << 16);
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

template <bool G, int GT>
__device__ __forceinline__ f4 widen(GradQuad<GT> q, unsigned elems)
{
    if constexpr (GT == kGradF32) {
        return q.v;
    } else {
        if constexpr (G) {  // (the word that it belongs to was loaded as 0)
            if ((elems & 2u) != 0u) q.v.y |= q.last;
            else q.v.x |= q.last;
        }
        return f4{widen16<GT>(q.v.x & 0xFFFFu), widen16<GT>(q.v.x >> 16), widen16<GT>(q.v.y & 0xFFFFu),
                  widen16<GT>(q.v.y >> 16)};
    }
}

template <int GT>
__device__ __forceinline__ const void *grad_at(const void *grad, size_t quad0)
{
    return static_cast<const char *>(grad) + quad0 * (4u * grad_bytes<GT>());
}

// ---------------------------------------------------------------------------
// a1 + a2: error-feedback threshold quantiser (Sec. 2.3, Sec. 3.4.1)
// ---------------------------------------------------------------------------
// a = r + g; |a| >= t sends sign(a)*t and keeps the rest.  `sent` is what the
// code stands for (+t, -t or +0); a - sent is bit-identical to a - t, a + t and
// a in the three cases.  Returns the 2-bit code (1 = +t, 2 = -t).
__device__ __forceinline__ unsigned quantize1(float g, float &r, float t, float &sent)
{
    const float a = r + g;
    const bool pos = a >= t;
    const bool neg = a <= -t;
    sent = pos ? t : (neg ? -t : 0.0f);
    r = a - sent;
    return pos ? 1u : (neg ? 2u : 0u);
}

// One quad: residual updated in place, returns the packed byte.
__device__ __forceinline__ unsigned quantize_quad(const f4 g, f4 &r, float t, f4 &sent)
{
    float s0, s1, s2, s3, r0 = r.x, r1 = r.y, r2 = r.z, r3 = r.w;
    const unsigned c0 = quantize1(g.x, r0, t, s0);
    const unsigned c1 = quantize1(g.y, r1, t, s1);
    const unsigned c2 = quantize1(g.z, r2, t, s2);
    const unsigned c3 = quantize1(g.w, r3, t, s3);
    r = f4{r0, r1, r2, r3};
    sent = f4{s0, s1, s2, s3};
    return c0 | (c1 << 2) | (c2 << 4) | (c3 << 6);
}

}  // namespace
