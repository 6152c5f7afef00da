// Layout packing, split-reduction epilogue and the small int8 network operators.
// All of them are bandwidth-bound permutations / elementwise passes.
#include <cstring>
#include <type_traits>

#include "unit_internal.h"

namespace unit {

// ------------------------------------------------------------------ pack_act
// NCHW -> [n][h*w][cp] with cp = channels padded to 16 bytes (zero filled): the graph
// level layout change of the paper (Section V-C; Section II-C.1 for the padding) done as
// one tiled transpose through LDS.  T = int8_t (16 channels per chunk) or uint16_t (8).
// With Q > 0 only the pixels (p*srow_step, q*scol_step) of each input image are packed
// (HW = P*Q output pixels, HWin = pixels per input channel): the input of a strided 1x1 conv.
template <typename T>
__device__ __forceinline__ void
pack_act_block(const T *__restrict__ x, uint8_t *__restrict__ xp, int C, int HW, int cp,
               int HWin, int Q, int srow, int scol, int bx, int by, int n)
{
    constexpr int CH = 16 / sizeof(T);            // channels per 16-byte chunk
    constexpr int TP = 64;                        // pixels per tile
    constexpr int TC = 64;                        // channels per tile
    __shared__ T tile[TC][TP + 4 / sizeof(T)];
    const int tid = threadIdx.x;
    const int hw0 = bx * TP, c0 = by * TC;
    const T *xn = x + (long)n * C * HWin;
    {
        const int px = tid & 63;
        int src = hw0 + px;
        if (Q > 0) {                               // subsampled source pixel
            const int p = src / Q;
            src = p * srow + (src - p * Q) * scol;
        }
        // every load is issued before the first LDS store: a masked element reads element 0 of
        // the image instead of branching around its load, and is zeroed afterwards
        const bool px_ok = hw0 + px < HW;
        T v[TC / 4];
#pragma unroll
        for (int i = 0; i < TC / 4; ++i) {
            const int c = (tid >> 6) + 4 * i;
            const bool ok = px_ok && c0 + c < C;
            v[i] = xn[ok ? (long)(c0 + c) * HWin + src : 0];
        }
#pragma unroll
        for (int i = 0; i < TC / 4; ++i) {
            const int c = (tid >> 6) + 4 * i;
            tile[c][px] = (px_ok && c0 + c < C) ? v[i] : (T)0;
        }
    }
    __syncthreads();
    constexpr int CHUNKS = TC / CH;               // chunks per pixel inside the tile
#pragma unroll
    for (int i = 0; i < TP * CHUNKS / 256; ++i) {
        int id = tid + i * 256;
        int px = id / CHUNKS, cc = id % CHUNKS;
        if (hw0 + px >= HW || c0 + cc * CH >= cp) continue;
        __attribute__((aligned(16))) T vals[CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) vals[e] = tile[cc * CH + e][px];
        *reinterpret_cast<v4i *>(xp + (((long)n * HW + hw0 + px) * cp + c0 + cc * CH) * sizeof(T)) =
            *reinterpret_cast<const v4i *>(vals);
    }
}

// The same transpose with the two mechanisms of the main kernel's direct 1x1 read: the 64-channel x TP-pixel tile
// comes into LDS with 16-byte global -> LDS loads (any byte offset; a row of pixels per channel, chunks XOR-swizzled
// by row), and gfx950's transposing LDS reads hand every lane the 16 bytes of consecutive channels of its pixel, i.e.
// one chunk of the packed tensor (see read_frags in igemm.hpp for the lane layout).  Lanes 16g..16g+15 of a wave hold
// chunk g of 16 consecutive pixels, so a wave's store covers whole 64-byte runs of the packed rows.  ES = element
// bytes; TP is chosen so that a channel row of the tile is a whole 128-byte line.  Needs rows that start on dword boundaries (the range check of those loads works per dword) and a tensor
// below 2 GiB; the byte-wise kernel above takes the rest.
template <int ES, int TP>
__device__ __forceinline__ void
pack_act_tr_block(const uint8_t *__restrict__ x, uint8_t *__restrict__ xp, int C, int HW, int cp, unsigned x_bytes,
                  int bx, int by, int n)
{
    constexpr int TC = 64;                        // channels per tile (TP pixels)
    constexpr int EPC = 16 / ES;                  // elements per 16-byte chunk
    constexpr int CPR = TP * ES / 16;             // chunks per channel row of the tile
    constexpr int CRPI = 64 / CPR;                // channel rows per wave-level load
    constexpr int NI = TC / CRPI / 4;             // loads per wave
    constexpr int RPR = (ES == 1) ? 8 : 4;        // channel rows per transposing read
    constexpr int SWZ_UNIT = (ES == 1) ? 2 : 4, SWZ_DIV = (16 / CPR > 1) ? 16 / CPR : 1;
    constexpr int SWZ_MOD = (CPR / SWZ_UNIT < RPR) ? CPR / SWZ_UNIT : RPR;
    static_assert(SWZ_DIV * SWZ_MOD == RPR, "the swizzle must repeat with the rows of one transposing read");
    auto swz = [](int r) { return SWZ_MOD > 1 ? SWZ_UNIT * ((r / SWZ_DIV) % SWZ_MOD) : 0; };
    __shared__ __attribute__((aligned(16))) uint8_t tile[TC * TP * ES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hw0 = bx * TP, c0 = by * TC;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(x, x_bytes);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int crow = (j * 4 + wave) * CRPI + lane / CPR;
        const int px = hw0 + ((lane % CPR) ^ swz(crow)) * EPC;
        const int c = c0 + crow;
        // (channels past C read as zeros: the padding of the packed rows; pixels past the image are never stored)
        const unsigned off = c < C ? (unsigned)((((long)n * C + c) * HW + px) * ES) : UNIT_OOB;
        dma16(rs, tile + (j * 4 + wave) * 1024, off);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int t16 = lane & 15;
    const int trow = (ES == 1) ? (t16 >> 1) : (t16 >> 2);      // channel row this lane points at
    const int tcol = (ES == 1) ? (t16 & 1) * 8 : (t16 & 3) * 4;
#pragma unroll
    for (int pg = wave; pg < TP / 16; pg += 4) {               // groups of 16 pixels of the tile, dealt to the waves
    const int cbyte = (pg * 16 + tcol) * ES;
    const int px = hw0 + pg * 16 + t16;
#pragma unroll
    for (int it = 0; it < TC / EPC / 4; ++it) {
        const int cc = it * 4 + (lane >> 4);                   // chunk of the tile's channels
        const uint8_t *src = tile + (cc * EPC + trow) * (TP * ES) + ((((cbyte >> 4) ^ swz(trow)) << 4) | (cbyte & 15));
        typedef __attribute__((address_space(3))) v2i lds_v2i;
        typedef __attribute__((address_space(3))) v4s lds_v4s;
        v2i r0, r1;
        if (ES == 1) {
            r0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)src);
            r1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(src + RPR * TP * ES));
        } else {
            r0 = __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)src));
            r1 = __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)(src + RPR * TP * ES)));
        }
        if (px < HW && c0 + cc * EPC < cp)
            *reinterpret_cast<v4i *>(xp + (((long)n * HW + px) * cp + c0 + cc * EPC) * ES) = v4i{r0[0], r0[1], r1[0], r1[1]};
    }
    }
}

// Images whose channels fit one 16-byte chunk (network inputs): one thread per pixel reads its
// CL >= C channel values (coalesced along the pixels; channels past C re-read channel 0 and are
// zeroed) and writes the pixel's chunk.  The tiled transpose above would spend a 64-channel tile
// on them.
template <typename T, int CL>
__device__ __forceinline__ void
pack_act_smallc_block(const T *__restrict__ x, uint8_t *__restrict__ xp, int C, int HW,
                      int HWin, int Q, int srow, int scol, int bx, int n)
{
    constexpr int CH = 16 / sizeof(T);
    const int px = bx * 256 + threadIdx.x;
    if (px >= HW) return;
    int src = px;
    if (Q > 0) {
        const int p = px / Q;
        src = p * srow + (px - p * Q) * scol;
    }
    const T *xn = x + (long)n * C * HWin + src;
    __attribute__((aligned(16))) T vals[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) vals[c] = 0;
    T v[CL];
#pragma unroll
    for (int c = 0; c < CL; ++c) v[c] = xn[(long)(c < C ? c : 0) * HWin];
#pragma unroll
    for (int c = 0; c < CL; ++c) vals[c] = c < C ? v[c] : (T)0;
    *reinterpret_cast<v4i *>(xp + ((long)n * HW + px) * 16) = *reinterpret_cast<const v4i *>(vals);
}

// ------------------------------------------------------------------ pack_weights
// OIHW -> [k][r][s][cp]: each output channel's reduction becomes one contiguous,
// zero-padded row (the "column-major B" of the implicit GEMM).  A thread gathers the 16 bytes of one chunk (consecutive
// channels of one tap, RS elements apart, which neighbouring threads find in the same cache lines) and stores them at
// once.  The chunks of all output channels are dealt out in one row, since a channel may have fewer than a workgroup has
// threads (a workgroup per channel: 100000 x 16 channels, one tap, int8, 31.8 us; 3.6 here, and 2.0 with the 16 bytes
// of a single tap as one load).  With SUMS (unsigned activations) a workgroup belongs to one output channel and sums its weights on the
// way: 128 times their sum corrects that channel's outputs.
struct PackW {
    const void *w;  uint8_t *wp;  int K, C, RS, cpc, chunks, total;     // cpc: chunks per tap, chunks = RS * cpc per row
    int per;                                        // chunks per workgroup (without sums): 256, or 64 where those fill the chip better
    DivU dv_cpc, dv_chunks;
    int32_t *sums;
};

// chunk i of output channel k; its 16 bytes
template <int ES>
__device__ __forceinline__ v4i pack_weights_chunk(const PackW &a, int k, int i)
{
    typedef typename std::conditional<ES == 1, uint8_t, uint16_t>::type T;
    constexpr int CH = 16 / ES;
    const int rs = divu(i, a.dv_cpc), c0 = (i - rs * a.cpc) * CH;
    const T *src = static_cast<const T *>(a.w) + ((size_t)k * a.C + c0) * a.RS + rs;
    v4i q;
    if (a.RS == 1 && c0 + CH <= a.C) {              // one tap: the chunk is contiguous (at any alignment)
        __builtin_memcpy(&q, src, 16);
    } else {
        T v[CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) v[e] = src[c0 + e < a.C ? (size_t)e * a.RS : 0];      // (past C: zeroed below)
        __attribute__((aligned(16))) T out[CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) out[e] = c0 + e < a.C ? v[e] : (T)0;
        q = *reinterpret_cast<const v4i *>(out);
    }
    *reinterpret_cast<v4i *>(a.wp + ((size_t)k * a.chunks + i) * 16) = q;
    return q;
}

template <int ES, bool SUMS>
__device__ __forceinline__ void pack_weights_block(const PackW &a, int blk, int blocks)
{
    if constexpr (SUMS) {
        __shared__ int part[4];
        for (int k = blk; k < a.K; k += blocks) {
            int sum = 0;
            for (int i = threadIdx.x; i < a.chunks; i += 256) {
                const v4i q = pack_weights_chunk<ES>(a, k, i);
#pragma unroll
                for (int d = 0; d < 4; ++d) { const int qd = q[d];  sum = __builtin_amdgcn_sdot4(qd, 0x01010101, sum, false); }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
            __syncthreads();                        // (the channel before has been read)
            if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
            __syncthreads();
            if (threadIdx.x == 0) a.sums[k] = 128 * (part[0] + part[1] + part[2] + part[3]);
        }
    } else {
        const long g = (long)blk * a.per + threadIdx.x;
        if ((int)threadIdx.x >= a.per || g >= a.total) return;
        const int k = divu((int)g, a.dv_chunks);
        pack_weights_chunk<ES>(a, k, (int)g - k * a.chunks);
    }
}

// ------------------------------------------------------------------ one launch for both
// The layout passes of a conv call: the first `wblocks` workgroups pack weights, the others activations.  Both are bound
// by their launch on all but large layers, and a call with plain operands needs both before its main kernel: one launch
// instead of two, or three with the weights' sums (3x3, 128 channels, 28x28, batch 8, u8 x i8, whole call: 15.2 -> 10.1 us;
// 3x3x3, 128 channels, 4x28x28, fp16: 17.9 -> 16.0).
// (ACT_SMALL + c: pixels of at most c channels, one chunk)
enum { ACT_TR = 0, ACT_TILE = 1, ACT_SMALL = 2, ACT_SMALL4 = ACT_SMALL + 4, ACT_SMALL8 = ACT_SMALL + 8, ACT_SMALL16 = ACT_SMALL + 16 };
struct PackA {
    const void *x;  uint8_t *xp;  int C, HW, cp, HWin, Q, srow, scol;  unsigned x_bytes;
    int gx, gy;  DivU dv_gx, dv_gy;                               // workgroups along the pixels and the channels of an image
};

template <int ES, int ACT>
__device__ __forceinline__ void pack_act_any(const PackA &a, int bx, int by, int n)
{
    typedef typename std::conditional<ES == 1, int8_t, uint16_t>::type T;
    const T *x = static_cast<const T *>(a.x);
    if constexpr (ACT == ACT_TR)
        pack_act_tr_block<ES, 128 / ES>(static_cast<const uint8_t *>(a.x), a.xp, a.C, a.HW, a.cp, a.x_bytes, bx, by, n);
    else if constexpr (ACT == ACT_TILE)
        pack_act_block<T>(x, a.xp, a.C, a.HW, a.cp, a.HWin, a.Q, a.srow, a.scol, bx, by, n);
    else
        pack_act_smallc_block<T, ACT - ACT_SMALL>(x, a.xp, a.C, a.HW, a.HWin, a.Q, a.srow, a.scol, bx, n);
}
// (each alone: the shared launch's dependent argument loads and divisions cost 0.5 us)
template <int ES, int ACT>
__global__ void __launch_bounds__(256) pack_act_kernel(const PackA a) { pack_act_any<ES, ACT>(a, blockIdx.x, blockIdx.y, blockIdx.z); }
template <int ES, bool SUMS>
__global__ void __launch_bounds__(256) pack_weights_kernel(const PackW w) { pack_weights_block<ES, SUMS>(w, blockIdx.x, gridDim.x); }
template <int ES, int ACT, bool SUMS>
__global__ void __launch_bounds__(256) pack_both_kernel(const PackW w, const PackA a, int wblocks)
{
    int blk = blockIdx.x;
    if (blk < wblocks) {
        pack_weights_block<ES, SUMS>(w, blk, wblocks);
        return;
    }
    blk -= wblocks;
    const int t = divu(blk, a.dv_gx), bx = blk - t * a.gx;
    const int n = divu(t, a.dv_gy), by = t - n * a.gy;
    pack_act_any<ES, ACT>(a, bx, by, n);
}

static DivU make_div(long d)
{
    DivU v;
    v.d = d > 1 ? (unsigned)d : 1u;
    v.m = d > 1 ? (unsigned)((1ULL << 32) / (unsigned long long)d) : 0xffffffffu;
    return v;
}

hipError_t launch_pack(int dtype, const PackWeights *w, const PackActs *x, hipStream_t st)
{
    const int es = (dtype == DT_I8) ? 1 : 2, ch = 16 / es;         // callers pass the storage type: one- or two-byte elements
    PackW pw;
    PackA pa;
    std::memset(&pw, 0, sizeof pw);
    std::memset(&pa, 0, sizeof pa);
    long wblocks = 0, ablocks = 0;
    int act = ACT_TILE;
    if (w) {
        pw.w = w->w;  pw.wp = static_cast<uint8_t *>(w->wp);  pw.K = w->k;  pw.C = w->c;  pw.RS = w->rs;
        pw.cpc = (w->c + ch - 1) / ch;
        const long chunks = (long)pw.cpc * pw.RS, total = chunks * w->k;
        if (total >= (1L << 31) || (w->sums && es != 1)) return hipErrorInvalidValue;
        pw.chunks = (int)chunks;
        pw.total = (int)total;
        pw.dv_cpc = make_div(pw.cpc);
        pw.dv_chunks = make_div(chunks);
        pw.sums = w->sums;
        // (layers of few chunks spread their waves over the chip: 256 x 256 channels, 3x3, int8, 2.60 -> 2.37 us)
        pw.per = total < 256 * 256 ? 64 : 256;
        wblocks = w->sums ? (w->k < (1 << 20) ? w->k : 1 << 20) : (total + pw.per - 1) / pw.per;
    }
    if (x) {
        const bool sub = x->p > 0;                                 // only the pixels (i * sh, j * sw), i < p, j < q
        pa.x = x->x;  pa.xp = static_cast<uint8_t *>(x->xp);  pa.C = x->c;
        pa.HWin = x->h * x->w;
        pa.HW = sub ? x->p * x->q : pa.HWin;
        pa.Q = sub ? x->q : 0;  pa.srow = x->sh * x->w;  pa.scol = x->sw;
        pa.cp = (x->c + ch - 1) / ch * ch;
        const long x_bytes = (long)x->n * x->c * pa.HWin * es;
        pa.gy = (pa.cp + 63) / 64;
        if (x->c <= ch) {
            act = x->c <= 4 ? ACT_SMALL4 : x->c <= 8 ? ACT_SMALL8 : ACT_SMALL16;
            pa.gx = (pa.HW + 255) / 256;
            pa.gy = 1;
        } else if (!sub && ((long)pa.HW * es) % 4 == 0 && (reinterpret_cast<uintptr_t>(x->x) & 15) == 0 && x_bytes < (1L << 31)) {
            act = ACT_TR;
            pa.gx = (pa.HW + 128 / es - 1) / (128 / es);           // tile pixels: one 128-byte line per channel row
            pa.x_bytes = (unsigned)x_bytes;
        } else {
            pa.gx = (pa.HW + 63) / 64;
        }
        pa.dv_gx = make_div(pa.gx);
        pa.dv_gy = make_div(pa.gy);
        ablocks = (long)pa.gx * pa.gy * x->n;
    }
    // a launch has fewer than 2^32 threads in a dimension: the flat grid holds 2^24 workgroups, the activations' own more
    if (w && x && wblocks + ablocks >= (1L << 24)) {
        const hipError_t e = launch_pack(dtype, w, nullptr, st);
        return e != hipSuccess ? e : launch_pack(dtype, nullptr, x, st);
    }
    const dim3 block(256), both((unsigned)(wblocks + ablocks)), acts(pa.gx, pa.gy, x ? x->n : 0);
    auto go = [&](auto es_c, auto act_c) {
        constexpr int ES = decltype(es_c)::value, ACT = decltype(act_c)::value;
        auto weights = [&](auto sums_c) {
            constexpr bool SUMS = decltype(sums_c)::value != 0;
            if (!x) hipLaunchKernelGGL((pack_weights_kernel<ES, SUMS>), both, block, 0, st, pw);
            else    hipLaunchKernelGGL((pack_both_kernel<ES, ACT, SUMS>), both, block, 0, st, pw, pa, (int)wblocks);
        };
        if (!w) {
            hipLaunchKernelGGL((pack_act_kernel<ES, ACT>), acts, block, 0, st, pa);
        } else if constexpr (ES == 1) {
            if (pw.sums) weights(IntC<1>{});
            else         weights(IntC<0>{});
        } else {
            weights(IntC<0>{});
        }
    };
    auto pick = [&](auto es_c) {
        if (act == ACT_TR)        go(es_c, IntC<ACT_TR>{});
        else if (act == ACT_TILE) go(es_c, IntC<ACT_TILE>{});
        else if (act == ACT_SMALL4) go(es_c, IntC<ACT_SMALL4>{});
        else if (act == ACT_SMALL8) go(es_c, IntC<ACT_SMALL8>{});
        else if constexpr (decltype(es_c)::value == 1) go(es_c, IntC<ACT_SMALL16>{});
    };
    if (es == 1) pick(IntC<1>{});
    else         pick(IntC<2>{});
    return hipGetLastError();
}

// packed int8 [n][hw][cp] -> NCHW
__global__ void unpack_act_i8_kernel(const int8_t *__restrict__ xp, int8_t *__restrict__ x,
                                     int C, int HW, int cp, long total)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    int px = i % HW;
    long nc = i / HW;
    int c = nc % C;
    long n = nc / C;
    x[i] = xp[(n * HW + px) * cp + c];
}

hipError_t launch_unpack_act_i8(int n, int c, int h, int w, const void *xp, int8_t *x, hipStream_t st)
{
    long total = (long)n * c * h * w;
    int cp = (c + 15) / 16 * 16;
    hipLaunchKernelGGL(unpack_act_i8_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const int8_t *)xp, x, c, h * w, cp, total);
    return hipGetLastError();
}

// ------------------------------------------------------------------ pad_rows
// Copies one or two [rows][row_bytes] matrices (row pitch ld_bytes, any alignment) into
// [rows][row_chunks * 16 bytes] ones of row pitch dst_ld, zero filling the tail: matmul operands that do not meet the
// 16-byte rule of the main kernel.  Bound by memory traffic and by the launch, so a thread moves a whole 16-byte
// chunk (the source needs no alignment), only the last chunk of a row, which may cross its end, is collected byte by
// byte, and both operands of a product go in one launch (grid.y).  Before, a thread moved one byte, after a 64-bit
// division of its own: 1533 x 2001 x 1777 in fp16, both operands copied, 25.4 us in two launches -> 8.7 us in one.
// (Both operands get the block count of the larger one, and the smaller one's spare workgroups leave at once; a few rows
// against a large matrix still gain: 32 x 4097 x 4095 in fp16, 63.8 -> 26.3 us as a whole.)
__global__ void __launch_bounds__(256)
pad_rows_kernel(const PadRows p0, const PadRows p1, int row_bytes, DivU row_chunks)
{
    const bool second = blockIdx.y != 0;
    const uint8_t *src = second ? p1.src : p0.src;
    uint8_t *dst = second ? p1.dst : p0.dst;
    const long ld_bytes = second ? p1.ld_bytes : p0.ld_bytes, dst_ld = second ? p1.dst_ld : p0.dst_ld;
    const long total = (long)(second ? p1.rows : p0.rows) * row_chunks.d;
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const long r = (total >> 31) ? i / row_chunks.d : (long)divu((int)i, row_chunks);
    const int b = (int)(i - r * row_chunks.d) * 16;
    const uint8_t *s = src + r * ld_bytes + b;
    uint4 w;
    if (b + 16 <= row_bytes) {
        __builtin_memcpy(&w, s, 16);                // (any byte alignment)
    } else {
        unsigned t[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 15; ++e)
            if (b + e < row_bytes) t[e >> 2] |= (unsigned)s[e] << (8 * (e & 3));
        w = make_uint4(t[0], t[1], t[2], t[3]);
    }
    *reinterpret_cast<uint4 *>(dst + r * dst_ld + b) = w;
}

hipError_t launch_pad_rows(const PadRows *ops, int nops, int row_bytes, int row_chunks, hipStream_t st)
{
    const PadRows &p0 = ops[0], &p1 = ops[nops - 1];
    const long rows = p0.rows > p1.rows ? p0.rows : p1.rows;
    hipLaunchKernelGGL(pad_rows_kernel, dim3((unsigned)((rows * row_chunks + 255) / 256), nops), dim3(256), 0, st,
                       p0, p1, row_bytes, make_div(row_chunks));
    return hipGetLastError();
}

// ------------------------------------------------------------------ split-K reduce + epilogue
// Sums the per-workgroup partial accumulators in slice order (fixed order: fp32 results
// are run-to-run identical), then applies the same epilogue as the main kernel.  The
// split reduction is the paper's "split reduction" tuning step (Section III-C.3) carried
// across workgroups; the in-group part lives in the main kernel.
//
// Each thread owns four consecutive outputs (the host keeps every slice a multiple of four
// elements long, so the 16-byte loads stay inside their slice) and reads the first eight slices
// at once: a slice index past the last one re-reads the last slice and is not added, which keeps
// the loads free of branches.  All loads of the requantise inputs go through buffer descriptors
// (an absent input has an empty range and reads as zero) and come before the first store.
template <typename E>
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const ReduceArgs a)
{
    typedef E v4e __attribute__((ext_vector_type(4)));
    const int total = (int)a.total;                  // < 2^29: the output stays below 2 GiB
    const int i = (int)(blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= total) return;
    const E *p = reinterpret_cast<const E *>(a.partials) + i;
    const int last = a.nsplit - 1;
    v4e head[8];
#pragma unroll
    for (int z = 0; z < 8; ++z)
        head[z] = *reinterpret_cast<const v4e *>(p + (long)(z < last ? z : last) * a.split_stride);
    v4e sum = head[0];
#pragma unroll
    for (int z = 1; z < 8; ++z) {                    // fixed order z = 1, 2, 3, ...: deterministic for fp32
        const v4e zero = {0, 0, 0, 0};
        sum += (z <= last) ? head[z] : zero;
    }
    for (int z = 8; z <= last; ++z) sum += *reinterpret_cast<const v4e *>(p + (long)z * a.split_stride);

    const bool full = i + 3 < total;
    if (a.out) {
        E *o = reinterpret_cast<E *>(a.out) + i;
        if (full) {
            *reinterpret_cast<v4e *>(o) = sum;       // (a global 16-byte store needs 4-byte alignment only)
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (i + e < total) o[e] = sum[e];
        }
    }
    if (a.epi != EPI_REQUANT) return;

    const __amdgpu_buffer_rsrc_t rsS = make_rsrc(a.scale, UNIT_OOB);
    const __amdgpu_buffer_rsrc_t rsB = make_rsrc(a.bias, a.bias ? UNIT_OOB : 0u);
    const __amdgpu_buffer_rsrc_t rsR = make_rsrc(a.residual, a.residual ? UNIT_OOB : 0u);
    const __amdgpu_buffer_rsrc_t rsP = make_rsrc(a.res_packed, a.res_packed ? UNIT_OOB : 0u);
    int t[4];  float sc[4];  unsigned pk[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = (i + e < total) ? i + e : i;              // a lane past the end repeats element i
        const int nk = div_any(idx, a.PQ);
        const int px = idx - nk * a.PQ;
        const int n = div_any(nk, a.K);
        const int k = nk - n * a.K;
        pk[e] = (unsigned)((n * a.PQ + px) * a.packed_ld + k);
        unsigned u = (unsigned)(int)sum[e];
        u += __builtin_amdgcn_raw_buffer_load_b32(rsB, (unsigned)k * 4u, 0, 0);
        u += __builtin_amdgcn_raw_buffer_load_b32(rsR, (unsigned)idx * 4u, 0, 0);
        const int r8 = (int)(int8_t)__builtin_amdgcn_raw_buffer_load_b8(rsP, pk[e], 0, 0);
        u += (unsigned)(r8 * a.res_mult);
        t[e] = (int)u;
        sc[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsS, (unsigned)k * 4u, 0, 0));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (i + e >= total) break;
        const int v = requant_elem(t[e], sc[e], a.relu);
        if (a.out_i8) a.out_i8[i + e] = (int8_t)v;
        if (a.out_packed) a.out_packed[pk[e]] = (int8_t)v;
    }
}

// zero the padding channels [K, packed_ld) of a packed int8 output
__global__ void zero_pad_channels_kernel(int8_t *yp, int K, int ld, long pixels)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    int npad = ld - K;
    if (i >= pixels * npad) return;
    yp[(i / npad) * ld + K + i % npad] = 0;
}

hipError_t launch_splitk_reduce(const ReduceArgs &a, hipStream_t st)
{
    // the requantise epilogue derives the channel from the element index
    if (a.total <= 0 || a.nsplit < 1 || (a.epi == EPI_REQUANT && (a.K <= 0 || a.PQ <= 0))) return hipErrorInvalidValue;
    dim3 grid((unsigned)((a.total + 1023) / 1024)), block(256);
    if (a.dtype == DT_I8) hipLaunchKernelGGL(splitk_reduce_kernel<int>, grid, block, 0, st, a);
    else                  hipLaunchKernelGGL(splitk_reduce_kernel<float>, grid, block, 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.epi == EPI_REQUANT && a.out_packed && a.packed_ld > a.K) {
        long pixels = a.total / a.K;
        long cnt = pixels * (a.packed_ld - a.K);
        hipLaunchKernelGGL(zero_pad_channels_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st,
                           a.out_packed, a.K, a.packed_ld, pixels);
        e = hipGetLastError();
    }
    return e;
}

// ------------------------------------------------------------------ unsigned-operand correction
// out[r] = 128 * (sum of the signed bytes of row r); rows are `ld` bytes apart, 16-byte
// aligned and `chunks` 16-byte chunks long.  One wave per row.
__global__ void __launch_bounds__(256)
rowsum128_i8_kernel(const uint8_t *__restrict__ m, long ld, int rows, int chunks, int32_t *__restrict__ out)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    const v4i *p = reinterpret_cast<const v4i *>(m + (long)row * ld);
    int sum = 0;
    for (int c = lane; c < chunks; c += 64) {
        v4i v = p[c];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            int w = v[d];
            sum += (int)(int8_t)(w & 0xff) + (int)(int8_t)((w >> 8) & 0xff) +
                   (int)(int8_t)((w >> 16) & 0xff) + (w >> 24);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (lane == 0) out[row] = sum * 128;
}

hipError_t launch_rowsum128_i8(const void *m, long ld, int rows, int chunks, int32_t *out, hipStream_t st)
{
    hipLaunchKernelGGL(rowsum128_i8_kernel, dim3((rows + 3) / 4), dim3(256), 0, st,
                       static_cast<const uint8_t *>(m), ld, rows, chunks, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ matmul with very few rows
// C[r][col] = sum_k A[r][k] * B[col][k] for a handful of rows (the fully connected layer of batch-1 inference: the paper's
// matmul with one row, Section II-A).  The matrix units would run 15/16 empty and, worse, a 16 x 64 tile leaves
// only n / 64 workgroups to stream B, the one operand of any size.  Here one wave owns one output column: it reads
// that column's reduction row of B once, 16 bytes per lane and load, multiplies each chunk with the same chunk of
// every row of A by the dot-product instructions of the vector ALU (v_dot4_i32_i8: four byte products added into an
// int32, exact; v_dot2_f32_f16: two half products added into an fp32) and adds the lanes' sums with a butterfly.
// n / 4 workgroups keep every compute unit streaming.  Rows of both operands start 16-byte aligned and are
// `kchunks` 16-byte chunks long (the caller pads otherwise).  MR = compiled number of rows (rows past m repeat row 0
// and are not stored).
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

template <int DT, int MR>
__global__ void __launch_bounds__(256)
gemv_kernel(const uint8_t *__restrict__ A, long lda, const uint8_t *__restrict__ B, long ldb,
            int m, int n, int kchunks, void *__restrict__ C, long ldc)
{
    typedef typename Mma<DT, 32>::elem_t elem_t;
    const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (col >= n) return;
    const v4i *b = reinterpret_cast<const v4i *>(B + (long)col * ldb);
    const v4i *a[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) a[r] = reinterpret_cast<const v4i *>(A + (long)(r < m ? r : 0) * lda);
    elem_t acc[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) acc[r] = 0;
    auto mac = [&](const v4i &bv, const v4i &av, elem_t &c) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int ai = av[d], bi = bv[d];       // (values, not vector-element lvalues: those do not bit_cast element-wise)
            if constexpr (DT == DT_I8) {
                c = __builtin_amdgcn_sdot4(ai, bi, c, false);
            } else {
                c = __builtin_amdgcn_fdot2(__builtin_bit_cast(v2h, ai), __builtin_bit_cast(v2h, bi), c, false);
            }
        }
    };
    // two chunks per lane and trip: all loads of a trip are issued before the first multiply
    int c = lane;
    for (; c + 64 < kchunks; c += 128) {
        const v4i b0 = b[c], b1 = b[c + 64];
        v4i a0[MR], a1[MR];
#pragma unroll
        for (int r = 0; r < MR; ++r) { a0[r] = a[r][c];  a1[r] = a[r][c + 64]; }
#pragma unroll
        for (int r = 0; r < MR; ++r) { mac(b0, a0[r], acc[r]);  mac(b1, a1[r], acc[r]); }
    }
    if (c < kchunks) {
        const v4i b0 = b[c];
#pragma unroll
        for (int r = 0; r < MR; ++r) mac(b0, a[r][c], acc[r]);
    }
#pragma unroll
    for (int r = 0; r < MR; ++r) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc[r] += __shfl_xor(acc[r], off, 64);
    }
    if (lane == 0) {
        elem_t *out = static_cast<elem_t *>(C);
#pragma unroll
        for (int r = 0; r < MR; ++r)
            if (r < m) out[(long)r * ldc + col] = acc[r];
    }
}

template <int DT>
static hipError_t launch_gemv_dt(const void *A, long lda, const void *B, long ldb, int m, int n, int kchunks,
                                 void *C, long ldc, hipStream_t st)
{
    const dim3 grid((n + 3) / 4), block(256);
    const uint8_t *a = static_cast<const uint8_t *>(A), *b = static_cast<const uint8_t *>(B);
    if (m == 1)      hipLaunchKernelGGL((gemv_kernel<DT, 1>), grid, block, 0, st, a, lda, b, ldb, m, n, kchunks, C, ldc);
    else if (m == 2) hipLaunchKernelGGL((gemv_kernel<DT, 2>), grid, block, 0, st, a, lda, b, ldb, m, n, kchunks, C, ldc);
    else if (m <= 4) hipLaunchKernelGGL((gemv_kernel<DT, 4>), grid, block, 0, st, a, lda, b, ldb, m, n, kchunks, C, ldc);
    else             hipLaunchKernelGGL((gemv_kernel<DT, 8>), grid, block, 0, st, a, lda, b, ldb, m, n, kchunks, C, ldc);
    return hipGetLastError();
}

// dtype: DT_I8 or DT_F16; m <= 8 (the API uses it up to GEMV_MAX_ROWS); lda, ldb in bytes
hipError_t launch_gemv(int dtype, const void *A, long lda, const void *B, long ldb, int m, int n, int kchunks,
                       void *C, long ldc, hipStream_t st)
{
    if (m < 1 || m > 8) return hipErrorInvalidValue;
    if (dtype == DT_I8) return launch_gemv_dt<DT_I8>(A, lda, B, ldb, m, n, kchunks, C, ldc, st);
    if (dtype == DT_F16) return launch_gemv_dt<DT_F16>(A, lda, B, ldb, m, n, kchunks, C, ldc, st);
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------ int8 network glue
// max-pool on packed int8: one thread per (n, p, q, 16-channel chunk).  With a compile-time
// window (WIN > 0) all window loads are issued at once through a buffer descriptor (taps in the
// padding get an out-of-range offset and are replaced by -128 afterwards); WIN == 0 walks a
// window of any size.
template <int WIN>
__global__ void __launch_bounds__(256)
maxpool_packed_i8_kernel(const int8_t *__restrict__ x, int8_t *__restrict__ y,
                         int cp, int H, int W, int P, int Q,
                         int window, int stride, int pad, int total, unsigned x_bytes)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= total) return;
    const int chunks = cp / 16;
    int t = div_any(i, chunks);
    const int cc = i - t * chunks;
    const int t2 = div_any(t, Q);
    const int q = t - t2 * Q;
    const int n = div_any(t2, P);
    const int p = t2 - n * P;
    int best[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) best[e] = -128;
    auto take = [&](const v4i &raw) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int b = (int)(int8_t)((unsigned)raw[e >> 2] >> (8 * (e & 3)));
            best[e] = (b > best[e]) ? b : best[e];
        }
    };
    if (WIN > 0) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(x, x_bytes);
        v4i raw[WIN > 0 ? WIN * WIN : 1];
#pragma unroll
        for (int r = 0; r < WIN; ++r)
#pragma unroll
            for (int s2 = 0; s2 < WIN; ++s2) {
                const int h = p * stride + r - pad, w = q * stride + s2 - pad;
                const bool ok = (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W;
                v4i v = buf_load16(rs, ok ? (unsigned)(((n * H + h) * W + w) * cp + cc * 16) : UNIT_OOB);
                const v4i lowest = {(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
                raw[r * WIN + s2] = ok ? v : lowest;
            }
#pragma unroll
        for (int k = 0; k < WIN * WIN; ++k) take(raw[k]);
    } else {
        for (int r = 0; r < window; ++r) {
            const int h = p * stride + r - pad;
            if (h < 0 || h >= H) continue;
            for (int s2 = 0; s2 < window; ++s2) {
                const int w = q * stride + s2 - pad;
                if (w < 0 || w >= W) continue;
                take(*reinterpret_cast<const v4i *>(x + ((long)(n * H + h) * W + w) * cp + cc * 16));
            }
        }
    }
    __attribute__((aligned(16))) int8_t outv[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) outv[e] = (int8_t)best[e];
    *reinterpret_cast<v4i *>(y + ((long)(n * P + p) * Q + q) * cp + cc * 16) = *reinterpret_cast<const v4i *>(outv);
}

hipError_t launch_maxpool_packed_i8(int n, int cp, int h, int w, int window, int stride, int pad,
                                    int p, int q, const void *x, void *y, hipStream_t st)
{
    const long total = (long)n * p * q * (cp / 16);
    const long x_bytes = (long)n * h * w * cp;
    if (total >= (1L << 31) || x_bytes >= (1L << 31)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    if (window == 3)
        hipLaunchKernelGGL(maxpool_packed_i8_kernel<3>, grid, block, 0, st, (const int8_t *)x, (int8_t *)y, cp, h, w,
                           p, q, window, stride, pad, (int)total, (unsigned)x_bytes);
    else if (window == 2)
        hipLaunchKernelGGL(maxpool_packed_i8_kernel<2>, grid, block, 0, st, (const int8_t *)x, (int8_t *)y, cp, h, w,
                           p, q, window, stride, pad, (int)total, (unsigned)x_bytes);
    else
        hipLaunchKernelGGL(maxpool_packed_i8_kernel<0>, grid, block, 0, st, (const int8_t *)x, (int8_t *)y, cp, h, w,
                           p, q, window, stride, pad, (int)total, (unsigned)x_bytes);
    return hipGetLastError();
}

// global average pool: integer sum then requantise.  One workgroup per (image, 64 channels):
// thread = (pixel slice, channel quad); every thread sums its slice of the pixels with 32-bit
// loads of four channels, the 16 slices are added through LDS, and 64 threads requantise.
__global__ void __launch_bounds__(256)
avgpool_packed_i8_kernel(const int8_t *__restrict__ x, const float *__restrict__ scale,
                         int8_t *__restrict__ y, int C, int cp, int HW, int groups)
{
    __shared__ int part[16][64];
    const int quad = threadIdx.x & 15, slice = threadIdx.x >> 4;
    const int grp = blockIdx.x % groups;
    const long n = blockIdx.x / groups;
    const int c0 = (grp * 16 + quad) * 4;               // first of this thread's four channels
    int s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    if (c0 < cp) {
        const int8_t *px = x + (n * HW + slice) * (long)cp + c0;
        for (int i = slice; i < HW; i += 16, px += 16L * cp) {
            const unsigned v = *reinterpret_cast<const unsigned *>(px);
            s0 += (int)(int8_t)v;  s1 += (int)(int8_t)(v >> 8);
            s2 += (int)(int8_t)(v >> 16);  s3 += (int)(int8_t)(v >> 24);
        }
    }
    part[slice][quad * 4 + 0] = s0;  part[slice][quad * 4 + 1] = s1;
    part[slice][quad * 4 + 2] = s2;  part[slice][quad * 4 + 3] = s3;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int c = grp * 64 + threadIdx.x;
        if (c < cp) {
            int sum = 0;
#pragma unroll
            for (int t = 0; t < 16; ++t) sum += part[t][threadIdx.x];
            y[n * cp + c] = c < C ? (int8_t)requant_elem(sum, scale[c], 0) : (int8_t)0;
        }
    }
}

hipError_t launch_avgpool_packed_i8(int n, int c, int cp, int hw, const void *x, const float *scale,
                                    int8_t *y, hipStream_t st)
{
    const int groups = (cp + 63) / 64;
    hipLaunchKernelGGL(avgpool_packed_i8_kernel, dim3((unsigned)((long)n * groups)), dim3(256), 0, st,
                       (const int8_t *)x, scale, y, c, cp, hw, groups);
    return hipGetLastError();
}

__global__ void widen_residual_i8_kernel(const int8_t *__restrict__ x, int32_t *__restrict__ res,
                                         int C, int cp, int HW, int mult, long total)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;   // NCHW index
    if (i >= total) return;
    int px = i % HW;
    long nc = i / HW;
    int c = nc % C;
    long n = nc / C;
    res[i] = (int)x[(n * HW + px) * cp + c] * mult;
}

hipError_t launch_widen_residual_i8(int n, int c, int cp, int hw, const void *x, int mult,
                                    int32_t *res, hipStream_t st)
{
    long total = (long)n * c * hw;
    hipLaunchKernelGGL(widen_residual_i8_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const int8_t *)x, res, c, cp, hw, mult, total);
    return hipGetLastError();
}

}  // namespace unit
