// Decoder forward pass for gfx950: kernels and their launcher.
//
// Every projection of a pass is a weight-streaming skinny GEMM Y[c][n] = sum_k W[n][k] X[c][k] with
// c < w <= 32 tokens.  bf16 weights are stored re-tiled in the order the MFMA consumes them, so a wave
// reads one contiguous 1 KiB block per (16 rows x 32 k) step; the activations are pre-split into
// bf16 hi + lo parts (x = hi + lo to 2^-17) in the matching B-operand order, so the product keeps
// fp32-like accuracy on the activation side and every output column depends on its own input column
// only: a token's result does not change with the width of the pass it is computed in.
// fp32 models (the tiny plumbing configuration) use plain VALU kernels.
#include "psd_device.h"
#include "psd_model.h"

#include <string.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace psd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

enum { EPI_RESID = 1, EPI_LOGITS = 2 };

// v combined over the four 16-lane rows of a wave, (row 0 with 1, 2 with 3), then the two results; every lane gets it.  The
// swaps of two equal registers leave a row and its partner side by side: no trip through LDS.
__device__ inline float rows_sum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ inline float rows_max(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// ---- operand packing ----------------------------------------------------------------------------
// GEMM input X[c][f] (c < 16 CT tokens, f < K features) of bf16 models: [K/32][CT col tiles][hi, lo][64 lanes][8]
// (CT = 2 for passes of up to 32 tokens, 32 for the passes of up to 512 tokens that ingest a prompt),
// lane = ((f % 32) / 8) * 16 + c % 16: exactly the B operand of v_mfma_f32_16x16x32_bf16.
// fp32 models: plain rows [c][K].
template <int CT>
__device__ inline void pack_store(void* xb, int c, int f, float v) {
    const int ks = f >> 5, g = (f & 31) >> 3, e = f & 7, t = c >> 4, cc = c & 15;
    uint16_t* p = (uint16_t*)xb;
    const size_t base = ((((size_t)ks * CT + t) * 2) * 64 + g * 16 + cc) * 8 + e;
    const uint16_t hi = f32_to_bf16(v);
    p[base] = hi;
    p[base + 64 * 8] = f32_to_bf16(v - bf16_to_f32(hi));
}

// ---- small kernels ------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void embed_rows(const float* embed, const PassDesc* desc, float* x, int d, int V) {
    const int c = blockIdx.x;
    if (c >= desc->w) return;
    int tok = desc->tok[c];
    tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);  // ids are validated on the host; never index outside the table
    for (int f = threadIdx.x; f < d; f += 256) x[(size_t)c * d + f] = embed[(size_t)tok * d + f];
}

__global__ void rope_table(float2* tab, int max_seq, int half, double theta) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= max_seq * half) return;
    const int pos = i / half, j = i % half;
    const double ang = (double)pos * pow(theta, -2.0 * j / (2.0 * half));
    tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}

__global__ void bf16_to_f32_vec(const uint16_t* in, float* out, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = bf16_to_f32(in[i]);
}

// row-major bf16 [N][K] -> MFMA A-operand tiles [Npad/16][K/32][64][8]; rows >= N become zeros.
// mode 1 (fused q/k/v projection): inside every head of `hd` rows, tile row 2e / 2e+1 of tile t holds the rotary
//   pair (j, j + hd/2), j = 8 t + e, so that one lane of the GEMM result owns both halves of a pair.
// mode 2 (fused gate/up projection, `hd` = F): tile row 2e / 2e+1 of tile t holds gate / up row 8 t + e.
__global__ __launch_bounds__(256) void tile_bf16(const uint4* src, uint4* dst, int N, int K, size_t n_chunks, int mode,
                                                 int hd) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_chunks) return;
    const int KS = K >> 5;
    const int lane = (int)(i & 63);
    const size_t t = i >> 6;
    const int ks = (int)(t % KS);
    const int tile = (int)(t / KS);
    int n = tile * 16 + (lane & 15);
    const int k = ks * 32 + (lane >> 4) * 8;
    if (mode == 1) {
        const int head = n / hd, within = n % hd, tt = within >> 4, tr = within & 15;
        n = head * hd + tt * 8 + (tr >> 1) + (tr & 1) * (hd >> 1);
    } else if (mode == 2) {
        const int tr = n & 15;
        n = (tr & 1) * hd + tile * 8 + (tr >> 1);
    }
    dst[i] = n < N ? src[((size_t)n * K + k) >> 3] : make_uint4(0, 0, 0, 0);
}

// ---- rotary embedding + KV append ------------------------------------------------------------------

// bf16 models keep every K and V element as a bf16 hi + lo pair (value = hi + lo to 2^-17) in four planes per
// (page, layer, kv head): K hi, K lo, V hi, V lo, each of kPage x hd elements.  One bf16 rounding of the
// cache alone would put ~0.1 % * sqrt(layers) of noise on the logits, which at 32 layers is past the tolerance.
__device__ inline size_t kv_plane(int page, int layer, int L, int g, int KV, int plane, int hd) {
    return ((((size_t)page * L + layer) * KV + g) * 4 + plane) * (size_t)kPage * hd;
}

// Inside a plane the elements sit in the order the attention MFMAs consume them, so that a wave's operand load is one
// contiguous block (1 KiB for K, 512 bytes for V) instead of sixteen strided pieces:
//   K planes: A-operand tiles of v_mfma_f32_16x16x32_bf16, [slot / 16][hd / 32][64 lanes][8], lane = (dim % 32) / 8 * 16 + slot % 16
//   V planes: half B-operand tiles of v_mfma_f32_16x16x32_bf16 (16 keys each), [hd / 16][slot / 16][64 lanes][4], lane = (slot % 16) / 4 * 16 + dim % 16
__device__ inline int kv_k_off(int slot, int dim, int hd) {
    return ((((slot >> 4) * (hd >> 5) + (dim >> 5)) * 64 + ((dim & 31) >> 3) * 16 + (slot & 15)) << 3) + (dim & 7);
}
__device__ inline int kv_v_off(int slot, int dim) {
    return ((((dim >> 4) * (kPage >> 4) + (slot >> 4)) * 64 + ((slot & 15) >> 2) * 16 + (dim & 15)) << 2) + (slot & 3);
}

__device__ inline size_t kv_base(int page, int layer, int L, int g, int KV, int which, int hd) {
    return ((((size_t)page * L + layer) * KV + g) * 2 + which) * (size_t)kPage * hd;
}

// sum over LP lanes (16 or 64), every lane gets it; fixed tree
template <int LP>
__device__ inline float lanes_sum(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
    v += dpp(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
    v += dpp(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
    v += dpp(v, std::integral_constant<int, 0x140>{});   // row_mirror
    if constexpr (LP == 64) v = rows_sum(v);
    return v;
}

__device__ inline float lanes_max(float v) {   // over a wave
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0xB1>{}));
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0x4E>{}));
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0x141>{}));
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0x140>{}));
    return rows_max(v);
}

// Arithmetic that the routes of an fp32 pass share, with every fusion written out: the same bits wherever the compiler puts it
__device__ inline float f32_squares(float4 v) { return fmaf(v.x, v.x, v.y * v.y) + fmaf(v.z, v.z, v.w * v.w); }
__device__ inline void f32_rotate(float& v1, float& v2, float2 cs) {
    const float r1 = fmaf(v1, cs.x, -(v2 * cs.y)), r2 = fmaf(v2, cs.x, v1 * cs.y);
    v1 = r1; v2 = r2;
}
__device__ inline float f32_silu_up(float g, float u) {
#pragma clang fp contract(off)
    return g / (1.f + expf(-g)) * u;
}
__device__ inline float f32_rms(float squares, float inv_k, float eps) { return rsqrtf(fmaf(squares, inv_k, eps)); }
__device__ inline float f32_score(float dot, float scale) {
#pragma clang fp contract(off)
    return dot * scale;
}

// ---- attention -------------------------------------------------------------------------------------
// grid (H, nsplit_max), 256 threads.  A workgroup owns one query head and one absolute key range
// [split * 128, split * 128 + 128); wave j takes the queries c = j, j + 4, ...  Partial result per
// (split, query, head): running max m, sum l and the un-normalised output, merged by attn_combine in
// split order.  The arithmetic for a query at a given position is the same whatever the pass width.
__global__ __launch_bounds__(256) void attn_partial(const float* qkv, const PassDesc* desc, const float* kv,
                                                    const int32_t* page_table, float* part, int layer, int L, int H,
                                                    int KV, int hd, int nqkv) {
    extern __shared__ float lds[];
    const int h = blockIdx.x, split = blockIdx.y;
    const int w = desc->w, pos0 = desc->pos0;
    const int key0 = split * kAttnSplit, kv_max = pos0 + w;
    if (key0 >= kv_max) return;
    const int nkeys = min(kAttnSplit, kv_max - key0);
    const int g = h / (H / KV), ld = hd + 1;
    float* Ks = lds;                       // [128][hd + 1]
    float* Vs = Ks + kAttnSplit * ld;      // [128][hd + 1]
    float* qs = Vs + kAttnSplit * ld;      // [4][hd]
    float* ps = qs + 4 * hd;               // [4][128]
    for (int idx = threadIdx.x; idx < nkeys * hd; idx += 256) {
        const int j = idx / hd, i = idx % hd, pos = key0 + j;
        const int page = page_table[pos / kPage], slot = pos % kPage;
        Ks[j * ld + i] = kv[kv_base(page, layer, L, g, KV, 0, hd) + (size_t)slot * hd + i];
        Vs[j * ld + i] = kv[kv_base(page, layer, L, g, KV, 1, hd) + (size_t)slot * hd + i];
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const float scale = rsqrtf((float)hd);
    float* q = qs + wave * hd;
    float* p = ps + wave * kAttnSplit;
    for (int c = wave; c < w; c += 4) {
        const int visible = min(nkeys, pos0 + c + 1 - key0);
        float* out = part + (((size_t)split * kCols + c) * H + h) * (hd + 2);
        if (visible <= 0) {
            if (lane == 0) { out[0] = -INFINITY; out[1] = 0.f; }
            continue;
        }
        for (int i = lane; i < hd; i += 64) q[i] = qkv[(size_t)c * nqkv + (size_t)h * hd + i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float s[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int j = lane + 64 * r;
            float acc = 0.f;
            if (j < visible)
                for (int i = 0; i < hd; ++i) acc += q[i] * Ks[j * ld + i];
            s[r] = j < visible ? f32_score(acc, scale) : -INFINITY;
        }
        const float m = lanes_max(fmaxf(s[0], s[1]));
        const float p0 = expf(s[0] - m), p1 = expf(s[1] - m);  // exp(-inf) = 0 for masked keys
        const float l = lanes_sum<64>(p0 + p1);
        p[lane] = p0;
        p[lane + 64] = p1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < hd; i += 64) {
            float acc = 0.f;
            for (int j = 0; j < visible; ++j) acc += p[j] * Vs[j * ld + i];
            out[2 + i] = acc;
        }
        if (lane == 0) { out[0] = m; out[1] = l; }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// grid (wmax, H), block hd: merges the split partials in order and writes the O-projection's input row
__global__ void attn_combine_f32(const float* part, const PassDesc* desc, float* out, int H, int hd) {
    const int c = blockIdx.x, h = blockIdx.y, i = threadIdx.x;
    if (c >= desc->w) return;
    const int nsp = (desc->pos0 + c + kAttnSplit) / kAttnSplit;  // splits holding keys <= pos0 + c
    float M = -INFINITY;
    for (int s = 0; s < nsp; ++s) M = fmaxf(M, part[(((size_t)s * kCols + c) * H + h) * (hd + 2)]);
    float Lsum = 0.f, o = 0.f;
    for (int s = 0; s < nsp; ++s) {
        const float* pr = part + (((size_t)s * kCols + c) * H + h) * (hd + 2);
        const float f = expf(pr[0] - M);
        Lsum += pr[1] * f;
        o += pr[2 + i] * f;
    }
    out[(size_t)c * H * hd + h * hd + i] = o / Lsum;
}

// Softmax of the bf16 models' attention works in base 2 (the query carries log2 e, exponentials are the hardware exp2).
// Key ranges are merged in order with a running maximum, the same arithmetic wherever it is done (attn_merge,
// attn_combine_long, attn_wide), so that a token's attention output has the same bits whichever kernel merges it:
// the state (M, Lsum, o) takes range (m, l, o_s) as
//   M' = max(M, m),  al = 2^(M - M'),  be = 2^(m - M'),  Lsum = Lsum al + l be,  o = o al + o_s be.
__device__ inline float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
struct MergeFac { float M, al, be; };
__device__ inline MergeFac merge_fac(float M, float m) {
    const float Mn = fmaxf(M, m);
    return MergeFac{Mn, M == -INFINITY ? 0.f : exp2_hw(M - Mn), m == -INFINITY ? 0.f : exp2_hw(m - Mn)};
}
__device__ inline float merge_add(float acc, float x, const MergeFac& f) { return fmaf(acc, f.al, x * f.be); }

// Merge of the split partials of one (token, head).  Returns the normalised output of head dims i .. i + N - 1.
template <int N>
__device__ inline void attn_merge(const float* part, int nsp, int c, int head, int H, int hd, int i, float out[N]) {
    const size_t stride = (size_t)kCols * H * (hd + 2);
    const float* p0 = part + ((size_t)c * H + head) * (hd + 2);
    float M = -INFINITY, Lsum = 0.f;
#pragma unroll
    for (int e = 0; e < N; ++e) out[e] = 0.f;
    for (int s0 = 0; s0 < nsp; s0 += 8) {   // eight partials in flight at a time
        float m[8], l[8], o[8][N];
#pragma unroll
        for (int s = 0; s < 8; ++s)
            if (s0 + s < nsp) {
                const float* pr = p0 + (size_t)(s0 + s) * stride;
                m[s] = pr[0];
                l[s] = pr[1];
#pragma unroll
                for (int e = 0; e < N; ++e) o[s][e] = pr[2 + i + e];
            }
#pragma unroll
        for (int s = 0; s < 8; ++s)
            if (s0 + s < nsp) {
                const MergeFac f = merge_fac(M, m[s]);
                M = f.M;
                Lsum = merge_add(Lsum, l[s], f);
#pragma unroll
                for (int e = 0; e < N; ++e) out[e] = merge_add(out[e], o[s][e], f);
            }
    }
#pragma unroll
    for (int e = 0; e < N; ++e) out[e] = out[e] / Lsum;
}

// ---- skinny GEMMs (bf16 weights, MFMA) ---------------------------------------------------------------
// Epilogues fused into the GEMM that produces the value:
//   EPI_QKV     rms scale, rotary embedding, q to the query buffer, k / v into the paged KV cache
//   EPI_RESID   x += y, then the next RMSNorm's operand (x * gain, bf16 hi/lo) and its sum-of-squares partials
//   EPI_SWIGLU  rms scale, silu(gate) * up, packed as the down projection's operand
//   EPI_LOGITS  rms scale, logits rows
// RMSNorm is split in two: the producer writes x * gain and per-tile partial sums of x^2, the consumer
// multiplies its result by rsqrt(mean x^2 + eps) (a per-token scalar commutes with the matrix product).
enum { EPI_QKV = 10, EPI_SWIGLU = 11 };

struct GemmArgs {
    const u32x4* Wt;       // tiled weights [Npad/16][KS][64] x 16 B
    const u32x4* XB;       // packed activations [KS][CT][2][64] x 16 B
    int N, KS;
    int wcap;              // widest pass this launch is meant for (its launch class): operand columns >= wcap are not loaded
    int lb_slots;          // LB kernels: 16-byte slots of a wave's staging area in LDS (64 per two K steps of its range)
    const PassDesc* desc;
    // rms scale of the input (EPI_QKV, EPI_SWIGLU, EPI_LOGITS): partial sums of squares [d/16][16 CT]
    const float* ss_in;
    int ss_tiles;
    float inv_d, eps;
    const float* rs_in;    // wide passes, EPI_SWIGLU: the columns' rms scales, from panel_scale
    // outputs
    float* Y;              // RESID: residual stream [32][ldy]; LOGITS: logits [rows][ldy]; QKV: query buffer [32][ldy]
    int ldy;
    void* xb_out;          // RESID / SWIGLU: operand of the next GEMM
    const float* gain_out; // RESID: gain of the RMSNorm that follows
    float* ss_out;         // RESID: [N/16][16 CT]
    // QKV only
    const float2* rope;
    uint16_t* kv;
    const int32_t* page_table;
    int layer, L, H, KV, hd;
};

// stores 4 (or 2) consecutive features of column c into a packed operand
template <int CT>
__device__ inline void pack4(void* xb, int c, int f0, const float v[4]) {
    const int ks = f0 >> 5, gq = (f0 & 31) >> 3, e = f0 & 7, t = c >> 4, cc = c & 15;
    uint16_t* p = (uint16_t*)xb + ((((size_t)ks * CT + t) * 2) * 64 + gq * 16 + cc) * 8 + e;
    uint32_t hi[2], lo[2];
    f32x2_split(v[0], v[1], hi[0], lo[0]);
    f32x2_split(v[2], v[3], hi[1], lo[1]);
    *reinterpret_cast<uint2*>(p) = make_uint2(hi[0], hi[1]);
    *reinterpret_cast<uint2*>(p + 512) = make_uint2(lo[0], lo[1]);
}
template <int CT>
__device__ inline void pack2(void* xb, int c, int f0, float v0, float v1) {
    const int ks = f0 >> 5, gq = (f0 & 31) >> 3, e = f0 & 7, t = c >> 4, cc = c & 15;
    uint16_t* p = (uint16_t*)xb + ((((size_t)ks * CT + t) * 2) * 64 + gq * 16 + cc) * 8 + e;
    uint32_t hi, lo;
    f32x2_split(v0, v1, hi, lo);
    *reinterpret_cast<uint32_t*>(p) = hi;
    *reinterpret_cast<uint32_t*>(p + 512) = lo;
}

// the pass descriptor's scalars, asked for when a kernel starts so that nothing waits for them at its end
struct DescVals { int w, pos0, n_logit, row0; };
__device__ inline DescVals load_desc(const PassDesc* d) { return DescVals{d->w, d->pos0, d->n_logit, d->logit_row0}; }

// What an epilogue reads from memory besides its own result.  The narrow kernels ask for it while the weights
// stream, so that the answers are there when the K loop ends; the arithmetic is the same either way.
template <int EPI> struct EpiPre {};
template <> struct EpiPre<EPI_RESID> { float4 x, gn; };
template <> struct EpiPre<EPI_QKV> { int page; float2 cs[2]; };

template <int EPI>
__device__ inline void epi_prefetch(const GemmArgs& a, const DescVals& dv, int tile, int g, int c, EpiPre<EPI>& p) {
    const int n = tile * 16 + g * 4;
    if constexpr (EPI == EPI_RESID) {
        p.x = *reinterpret_cast<const float4*>(a.Y + (size_t)c * a.ldy + n);
        p.gn = *reinterpret_cast<const float4*>(a.gain_out + n);
    } else if constexpr (EPI == EPI_QKV) {
        const int hd = a.hd, half = hd >> 1;
        const int head = (tile * 16) / hd, t_in = ((tile * 16) % hd) >> 4;
        const int pos = dv.pos0 + c;
        p.page = a.page_table[pos / kPage];
#pragma unroll
        for (int pr = 0; pr < 2; ++pr)
            if (head < a.H + a.KV) p.cs[pr] = a.rope[(size_t)pos * half + t_in * 8 + g * 2 + pr];
    }
}

// value tile of one lane: rows n0 + 4 g + r (r = 0..3) of column c
// PRE: `pre` was filled by epi_prefetch; otherwise the reads happen here
template <int EPI, int CT, bool PRE>
__device__ inline void epilogue(const GemmArgs& a, const DescVals& dv, int tile, int g, int c, f32x4 v, float rs,
                                const EpiPre<EPI>& pre) {
    const int n = tile * 16 + g * 4;
    const int w = dv.w;
    if constexpr (EPI == EPI_LOGITS) {
        const int first = w - dv.n_logit;
        if (c < first || n >= a.N) return;
        float* dst = a.Y + (size_t)(dv.row0 + c - first) * a.ldy + n;
        if ((a.ldy & 3) == 0 && n + 3 < a.N) {
            *reinterpret_cast<float4*>(dst) = make_float4(v[0] * rs, v[1] * rs, v[2] * rs, v[3] * rs);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (n + r < a.N) dst[r] = v[r] * rs;
        }
    } else if constexpr (EPI == EPI_RESID) {
        float* dst = a.Y + (size_t)c * a.ldy + n;
        float4 o, gn;
        if constexpr (PRE) { o = pre.x; gn = pre.gn; } else { o = *reinterpret_cast<const float4*>(dst); }
        o.x += v[0]; o.y += v[1]; o.z += v[2]; o.w += v[3];
        *reinterpret_cast<float4*>(dst) = o;
        if constexpr (!PRE) gn = *reinterpret_cast<const float4*>(a.gain_out + n);
        const float pk[4] = {o.x * gn.x, o.y * gn.y, o.z * gn.z, o.w * gn.w};
        pack4<CT>(a.xb_out, c, n, pk);
        float ss = o.x * o.x + o.y * o.y + o.z * o.z + o.w * o.w;
        ss = rows_sum(ss);
        if (g == 0) a.ss_out[tile * (16 * CT) + c] = ss;
    } else if constexpr (EPI == EPI_SWIGLU) {
        // weight rows are interleaved: tile row 2e = gate of feature 8 tile + e, tile row 2e + 1 = its up row
        const float g0 = v[0] * rs, u0 = v[1] * rs, g1 = v[2] * rs, u1 = v[3] * rs;
        pack2<CT>(a.xb_out, c, tile * 8 + g * 2, g0 / (1.f + expf(-g0)) * u0, g1 / (1.f + expf(-g1)) * u1);
    } else if constexpr (EPI == EPI_QKV) {
        // weight rows are permuted inside every head: tile row 2e, 2e + 1 = rotary pair (j, j + hd/2), j = 8 t + e;
        // a lane holds the pairs j0 and j0 + 1, so every store below covers two adjacent head dims
        const int hd = a.hd, half = hd >> 1;
        const int head = (tile * 16) / hd, t_in = ((tile * 16) % hd) >> 4;
        const int pos = dv.pos0 + c;
        int page;
        if constexpr (PRE) page = pre.page; else page = a.page_table[pos / kPage];
        const int slot = pos % kPage;
        const int j0 = t_in * 8 + g * 2;
        float x0[2], x1[2];
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
            x0[pr] = v[2 * pr] * rs;
            x1[pr] = v[2 * pr + 1] * rs;
            if (head < a.H + a.KV) {
                float2 cs;
                if constexpr (PRE) cs = pre.cs[pr]; else cs = a.rope[(size_t)pos * half + j0 + pr];
                const float r0 = x0[pr] * cs.x - x1[pr] * cs.y, r1 = x1[pr] * cs.x + x0[pr] * cs.y;
                x0[pr] = r0; x1[pr] = r1;
            }
        }
        if (head < a.H) {
            float* q = a.Y + (size_t)c * a.ldy + (size_t)head * hd;
            *reinterpret_cast<float2*>(q + j0) = make_float2(x0[0], x0[1]);
            *reinterpret_cast<float2*>(q + j0 + half) = make_float2(x1[0], x1[1]);
        } else if (head < a.H + a.KV) {   // K planes
            uint16_t* kh = a.kv + kv_plane(page, a.layer, a.L, head - a.H, a.KV, 0, hd);
            uint16_t* kl = kh + (size_t)kPage * hd;
            uint32_t h0, l0, h1, l1;
            f32x2_split(x0[0], x0[1], h0, l0);
            f32x2_split(x1[0], x1[1], h1, l1);
            const int o0 = kv_k_off(slot, j0, hd), o1 = kv_k_off(slot, j0 + half, hd);   // j0 is even: the pair stays together
            *reinterpret_cast<uint32_t*>(kh + o0) = h0;
            *reinterpret_cast<uint32_t*>(kh + o1) = h1;
            *reinterpret_cast<uint32_t*>(kl + o0) = l0;
            *reinterpret_cast<uint32_t*>(kl + o1) = l1;
        } else {                          // V planes
            uint16_t* vh = a.kv + kv_plane(page, a.layer, a.L, head - a.H - a.KV, a.KV, 2, hd);
            uint16_t* vl = vh + (size_t)kPage * hd;
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                const int j = j0 + pr;
                uint32_t hi, lo;
                f32x2_split(x0[pr], x1[pr], hi, lo);
                const int o0 = kv_v_off(slot, j), o1 = kv_v_off(slot, j + half);
                vh[o0] = (uint16_t)hi;
                vh[o1] = (uint16_t)(hi >> 16);
                vl[o0] = (uint16_t)lo;
                vl[o1] = (uint16_t)(lo >> 16);
            }
        }
    }
}

// 16-byte load from a wave-uniform base plus a 32-bit lane offset: the address arithmetic stays in scalar registers
__device__ inline u32x4 load16_at(const u32x4* uniform, uint32_t lane_bytes) {
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(uniform) + lane_bytes);
}

// Order of the sum over a projection's NW K ranges, the same for every pass width: the q/k/v, o and down projections
// (EPI_QKV, EPI_RESID) add the ranges of each quarter of K in order and then the four quarters in order, so that a wide
// pass can give a quarter to a workgroup of its own; the others add all ranges in order.
template <int EPI>
constexpr bool kGrouped = EPI == EPI_QKV || EPI == EPI_RESID;
template <int NW, int EPI, typename F>
__device__ inline f32x4 group_sum(F range) {
    constexpr int NG = kGrouped<EPI> ? 4 : 1, PER = NW / NG;
    static_assert(NW % NG == 0, "ranges per group");
    f32x4 sum;
#pragma unroll
    for (int j = 0; j < NG; ++j) {
        f32x4 gs = range(j * PER);
#pragma unroll
        for (int v = 1; v < PER; ++v) gs += range(j * PER + v);
        sum = j == 0 ? gs : sum + gs;
    }
    return sum;
}

// rms scale of a column in a wide pass: the narrow kernels' 4 NW strided partial sums of the input's sums of squares,
// folded as there: (0 + 1) + (2 + 3) within each group of four, the groups added in order
template <int NW>
__device__ inline float ss_slot(const GemmArgs& a, int slot, int col) {
    float sum = 0.f;
#pragma unroll 8
    for (int st = slot; st < a.ss_tiles; st += 4 * NW) sum += a.ss_in[st * (16 * kWideCT) + col];
    return sum;
}
template <int NW, int GC>
__device__ inline float ss_scale(const GemmArgs& a, const float (*ssp)[GC], int col) {
    float ssum = 0.f;
#pragma unroll
    for (int u = 0; u < NW; ++u) ssum += (ssp[4 * u][col] + ssp[4 * u + 1][col]) + (ssp[4 * u + 2][col] + ssp[4 * u + 3][col]);
    return rsqrtf(ssum * a.inv_d + a.eps);
}

// One workgroup of NW waves per RT tiles of 16 output rows; the waves split K and are summed in wave order.
// A wave multiplies RT row tiles by the same activation operand, which is loaded once per K step (the operand
// comes from L2 and would otherwise cost twice the weight bytes) and only by the lanes whose column is in use.
// Small projections get more waves and fewer tiles per workgroup so that enough loads are in flight.
// The rms scale of the input is gathered on the side: every thread loads a few sum-of-squares partials before
// the K loop and they are folded through LDS, in a fixed order, when the loop is done.
// LB (passes of at most 4 tokens, NT == 1): the few operand lanes that carry data are so little that a wave stages the
// operand of its whole K range in LDS before it asks for any weights: direct-to-LDS loads, 64 lanes x 16 bytes = the
// live blocks (4 columns x 4 k groups x hi, lo) of two K steps per instruction, no registers.  Loads return in order, so
// the staged blocks are there before the first weight block, and a K step then reads its operand from LDS (~100
// cycles) instead of L2 (~1400 cycles, of which a wave's two MFMAs per step hide nothing).
template <int NT, int NW, int RT, int EPI, bool LB = false, bool SK = false>
__global__ __launch_bounds__(64 * NW) void gemm_bf16(const GemmArgs a) {
    static_assert(!LB || NT == 1, "LDS staging of the operand is for one column tile");
    constexpr int CT = 2;   // column tiles of the operand
    extern __shared__ u32x4 lb_buf[];
    static_assert(RT <= NW, "one finishing wave per row tile");
    __shared__ f32x4 red[NW][RT][NT][64];
    constexpr bool kScaled = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LOGITS);
    __shared__ float ssp[kScaled ? NW : 1][16 * NT];
    const int tile0 = blockIdx.x * RT, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k0 = (int)(((long)a.KS * wave) / NW), k1 = (int)(((long)a.KS * (wave + 1)) / NW);
    const int g = lane >> 4, cc = lane & 15;
    const DescVals dv = load_desc(a.desc);
    // the epilogue's own reads: the finishing wave asks for them once its first weights are on the way
    EpiPre<EPI> pre[NT];   // wave r finishes row tile r
    float ss_mine[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) ss_mine[t] = 0.f;
    // Side reads (sum-of-squares partials for every wave, the epilogue's inputs for the finishing wave) are issued
    // right after a wave's first weight loads, never before them: the weight stream starts at once.
    bool want_pre = true;
    auto prefetch_all = [&]() {
        want_pre = false;
        if constexpr (kScaled) {
            const int gi = wave * 4 + g;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll 8
                for (int st = gi; st < a.ss_tiles; st += 4 * NW) ss_mine[t] += a.ss_in[st * (16 * CT) + t * 16 + cc];
            }
        }
        if (wave >= RT) return;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t * 16 + cc < dv.w) epi_prefetch<EPI>(a, dv, tile0 + wave, g, t * 16 + cc, pre[t]);
    };
    const u32x4* a_ptr = a.Wt + ((size_t)tile0 * a.KS + k0) * 64 + lane;
    const size_t tile_stride = (size_t)a.KS * 64;
    constexpr int kBStep = CT * 128;   // 16-byte words of the operand per K step
    const u32x4* b_ptr = a.XB + (size_t)k0 * kBStep + lane;
    const u32x4* const b_base = b_ptr;
    bool col_live[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) col_live[t] = t * 16 + cc < a.wcap;   // known at launch: nothing waits for the descriptor
    f32x4 acc[RT][NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // K steps per batch: about 16 weight loads of 16 bytes in flight per lane; 28 with seven row tiles per wave (one
    // workgroup per CU, so registers do not limit residency there; measured: 71 -> 67 ms per 1504 launches); for the
    // four-tile variant 24 or 32 in flight were slower than 16
    constexpr int U = RT == 7 ? 4 : 16 / RT;
    static_assert(U >= 1, "too many row tiles per wave");
    const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
    auto mfma_step = [&](const u32x4 (&wv)[RT], int t, const u32x4 bh, const u32x4 bl) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wv[r]),
                                                                __builtin_bit_cast(bf16x8, bh), acc[r][t], 0, 0, 0);
            acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wv[r]),
                                                                __builtin_bit_cast(bf16x8, bl), acc[r][t], 0, 0, 0);
        }
    };
    if constexpr (SK) {
        // Short K ranges (at most D steps per wave: the draft's q/k/v projection, the qualifier's o projection): a wave asks
        // for its whole range at once, weight blocks from memory and operand blocks from L2 side by side: one round of
        // loads instead of a weight batch followed by operand groups that each cost an exposed L2 round trip (draft q/k/v
        // 9.3 -> 8.6 us, qualifier o 9.8 -> 9.2 us between events).  A longer range would be walked D steps at a time; the
        // host does not pick this variant for one.  A window of D steps refilled step by step was measured for the long
        // ranges and loses to the batches below (target down 29.4 -> 31.1 us): loads return in order, so a window that
        // holds operand blocks next to the weight blocks has 7 instead of 16 weight blocks in flight.  Same K order, same bits.
        static_assert(NT == 1 && RT == 1 && !LB, "the short-range variant is for one tile per wave");
        constexpr int D = 7;
        for (int s0 = k0; s0 < k1; s0 += D) {
            const int n = min(D, k1 - s0);
            u32x4 wq[D], bq[D][2];
#pragma unroll
            for (int u = 0; u < D; ++u)
                if (u < n) {
                    wq[u] = __builtin_nontemporal_load(a_ptr + (size_t)u * 64);
                    bq[u][0] = zero; bq[u][1] = zero;
                    if (col_live[0]) {
                        const u32x4* bp = b_ptr + (size_t)u * kBStep;
                        bq[u][0] = bp[0]; bq[u][1] = bp[64];
                    }
                }
            if (want_pre) prefetch_all();
#pragma unroll
            for (int u = 0; u < D; ++u)
                if (u < n) {
                    const u32x4 w1[1] = {wq[u]};
                    mfma_step(w1, 0, bq[u][0], bq[u][1]);
                }
            a_ptr += (size_t)D * 64;
            b_ptr += (size_t)D * kBStep;
        }
    } else if constexpr (NT == 1 && RT == 4 && !LB) {
        // Four row tiles per wave (the qualifier's gate/up projection, one workgroup per CU, 12 K steps per wave): a step is
        // four weight blocks and one pair of operand blocks, and a window of D steps is on the way at all times: a step's
        // registers are asked for again, D steps ahead, as soon as its MFMAs are issued.  Loads return in the order they
        // were issued, which is the order the steps are used in.  Same K order, same bits as the batches that drain
        // (21.5 -> 20.4 us between events).  Measured and not kept: the same window for the seven-tile variant (4 steps are
        // all its registers hold: target gate/up 42.1 -> 42.6 us) and for the 8-wave q/k/v kernels (8 steps: qualifier 12.8
        // -> 13.9 us, target 16.3 -> 16.7 us).
        constexpr int D = 6;
        const int n = k1 - k0;
        u32x4 wq[D][RT], bq[D][2];
        auto fetch = [&](int slot, int st) {
#pragma unroll
            for (int r = 0; r < RT; ++r) wq[slot][r] = __builtin_nontemporal_load(a_ptr + r * tile_stride + (size_t)st * 64);
            bq[slot][0] = zero; bq[slot][1] = zero;
            if (col_live[0]) {
                const u32x4* bp = b_ptr + (size_t)st * kBStep;
                bq[slot][0] = bp[0]; bq[slot][1] = bp[64];
            }
        };
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < n) fetch(u, u);
        if (want_pre) prefetch_all();
        int st = 0;
        for (; st + 2 * D <= n; st += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                mfma_step(wq[u], 0, bq[u][0], bq[u][1]);
                fetch(u, st + D + u);
            }
        }
        // fewer than 2 D steps left, the first D of them (or all) on the way
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (st + u < n) {
                mfma_step(wq[u], 0, bq[u][0], bq[u][1]);
                if (st + D + u < n) fetch(u, st + D + u);
            }
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (st + D + u < n) mfma_step(wq[u], 0, bq[u][0], bq[u][1]);
    } else if constexpr (NT == 1) {
        // Operand blocks come from L2.  BG steps' worth of them is asked for at a time; the first group goes out with the
        // batch's weights and is there long before them, every later group costs one exposed L2 round trip.  The whole
        // batch at once (BG = U) takes up to 64 registers: on in the variants that run at most one workgroup per CU
        // anyway (qualifier q/k/v 39.8 -> 34.7 ms per 2632 launches); where it would cost residency (the draft's gate/up,
        // the LM heads: 17.6 -> 18.5 us) groups of 2 are used (17.6 -> 16.7 us).
        constexpr int BG = (U <= 8 && (RT >= 4 || EPI == EPI_QKV)) ? U : (U < 2 ? U : 2);
        static_assert(U % BG == 0, "operand groups must tile a batch");
        u32x4 bpre[BG][2];
        const u32x4* my_b = nullptr;   // LB: this wave's staged operand, [pair of steps][step parity][hi, lo][k group][column < 4]
        if constexpr (LB) {
            const int n = k1 - k0;
            u32x4* stage = lb_buf + __builtin_amdgcn_readfirstlane(wave) * a.lb_slots;
            const int par = lane >> 5, half = (lane >> 4) & 1, sg = (lane >> 2) & 3, sc = lane & 3;
            for (int i = 0; 2 * i < n; ++i) {
                // a range with an odd number of steps: the last instruction's upper lanes fetch the last step again, into
                // slots no step reads
                const int st = min(2 * i + par, n - 1);
                const u32x4* src = a.XB + (size_t)(k0 + st) * kBStep + half * 64 + sg * 16 + sc;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                 (__attribute__((address_space(3))) void*)(stage + i * 64), 16, 0, 0);
            }
            my_b = stage + g * 4 + cc;
            asm volatile("" ::: "memory");   // the staging loads stay ahead of every other load of the wave
        }
        bool staged_ready = !LB;
        // LB: called once, right after the first batch's weight loads (`later` of them, and nothing else, were issued after
        // the staging loads): when at most `later` loads are outstanding the staged operand is in LDS
        auto staged_wait = [&](bool full_batch) {
            if constexpr (LB) {
                if (staged_ready) return;
                staged_ready = true;
                // Counts on the loads issued since the staging loads: exactly the U * RT weight loads of the first full batch,
                // all unconditional (a predicated or split weight load would make the count, and with it this wait, wrong:
                // then wait for vmcnt(0) instead).  The narrow-against-wide bit-exactness tests guard this.
                static_assert(!LB || U * RT <= 63, "the vmcnt field holds at most 63");
                if (full_batch) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(U * RT < 63 ? U * RT : 63) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        };
        auto load_b = [&](int slot, const u32x4* bp) {
            bpre[slot][0] = zero; bpre[slot][1] = zero;
            if constexpr (LB) {
                // bp counts K steps in units of kBStep from the operand's start: recover the step within the wave's range
                const int s = (int)((bp - b_base) / kBStep);
                if (col_live[0]) {
                    const u32x4* q = my_b + (s >> 1) * 64 + (s & 1) * 32;
                    bpre[slot][0] = q[0]; bpre[slot][1] = q[16];
                }
            } else {
                if (col_live[0]) { bpre[slot][0] = bp[0]; bpre[slot][1] = bp[64]; }
            }
        };
        // batches of U K steps; the last batch of a range may be short (its loads still go out together)
        for (int ks = k0; ks < k1; ks += U) {
            u32x4 wv[U][RT];
            if (ks + U <= k1) {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r) wv[u][r] = __builtin_nontemporal_load(a_ptr + r * tile_stride + (size_t)u * 64);
                staged_wait(true);
#pragma unroll
                for (int u = 0; u < BG; ++u) load_b(u, b_ptr + (size_t)u * kBStep);
                if (want_pre) prefetch_all();
#pragma unroll
                for (int g0 = 0; g0 < U; g0 += BG) {
                    if (g0 > 0) {
#pragma unroll
                        for (int u = 0; u < BG; ++u) load_b(u, b_ptr + (size_t)(g0 + u) * kBStep);
                    }
#pragma unroll
                    for (int u = 0; u < BG; ++u) mfma_step(wv[g0 + u], 0, bpre[u][0], bpre[u][1]);
                }
            } else {
                const int cnt = k1 - ks;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u < cnt) {
#pragma unroll
                        for (int r = 0; r < RT; ++r) wv[u][r] = __builtin_nontemporal_load(a_ptr + r * tile_stride + (size_t)u * 64);
                    }
                staged_wait(false);
#pragma unroll
                for (int u = 0; u < BG; ++u)
                    if (u < cnt) load_b(u, b_ptr + (size_t)u * kBStep);
                if (want_pre) prefetch_all();
#pragma unroll
                for (int g0 = 0; g0 < U; g0 += BG) {
                    if (g0 > 0) {
#pragma unroll
                        for (int u = 0; u < BG; ++u)
                            if (g0 + u < cnt) load_b(u, b_ptr + (size_t)(g0 + u) * kBStep);
                    }
#pragma unroll
                    for (int u = 0; u < BG; ++u)
                        if (g0 + u < cnt) mfma_step(wv[g0 + u], 0, bpre[u][0], bpre[u][1]);
                }
            }
            a_ptr += (size_t)U * 64;
            b_ptr += (size_t)U * kBStep;
        }
    } else {
        // Several column tiles per wave: a step loads its operand blocks tile by tile right before it uses them (a group
        // of steps' blocks would not fit the registers: 302 spilled registers when tried)
        auto step = [&](const u32x4 (&wv)[RT], const u32x4* bp) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                u32x4 bh = zero, bl = zero;
                if (col_live[t]) { bh = bp[t * 128]; bl = bp[t * 128 + 64]; }
                mfma_step(wv, t, bh, bl);
            }
        };
        for (int ks = k0; ks < k1; ks += U) {
            u32x4 wv[U][RT];
            if (ks + U <= k1) {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r) wv[u][r] = __builtin_nontemporal_load(a_ptr + r * tile_stride + (size_t)u * 64);
                if (want_pre) prefetch_all();
#pragma unroll
                for (int u = 0; u < U; ++u) step(wv[u], b_ptr + (size_t)u * kBStep);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (ks + u < k1) {
#pragma unroll
                        for (int r = 0; r < RT; ++r) wv[u][r] = __builtin_nontemporal_load(a_ptr + r * tile_stride + (size_t)u * 64);
                    }
                if (want_pre) prefetch_all();
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (ks + u < k1) step(wv[u], b_ptr + (size_t)u * kBStep);
            }
            a_ptr += (size_t)U * 64;
            b_ptr += (size_t)U * kBStep;
        }
    }
    if (want_pre) prefetch_all();   // a wave without K steps
    if constexpr (kScaled) {
        // a wave's four strided partial sums are folded pairwise, (0 + 1) + (2 + 3); the waves' results are added in
        // wave order by whoever needs the scale
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float sw = rows_sum(ss_mine[t]);
            if (g == 0) ssp[wave][t * 16 + cc] = sw;
        }
    }
    // the waves' partial sums meet in LDS; wave r adds up row tile r in the order of group_sum and finishes it, so the RT
    // epilogues of a workgroup run side by side
    const int w = dv.w;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) red[wave][r][t][lane] = acc[r][t];
    __syncthreads();
    if (wave >= RT) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float rs = 1.f;
        if constexpr (kScaled) {
            float ssum = 0.f;
#pragma unroll
            for (int v = 0; v < NW; ++v) ssum += ssp[v][t * 16 + cc];
            rs = rsqrtf(ssum * a.inv_d + a.eps);
        }
        const int c = t * 16 + cc;
        const f32x4 sum = group_sum<NW, EPI>([&](int v) { return red[v][wave][t][lane]; });
        // whole 16-lane groups agree on c < w, and the shuffles inside the epilogue cross g only
        if (c < w) epilogue<EPI, CT, true>(a, dv, tile0 + wave, g, c, sum, rs, pre[t]);
    }
}

// rms scale of every column of a wide pass, once for all workgroups of the gate/up projection (each of them would
// otherwise read 128 KB of partial sums for its own columns: 16 us of a 95 us launch on the draft's shape).
// grid column tiles, 256 threads.
template <int NW>
__global__ __launch_bounds__(256) void panel_scale(const GemmArgs a, float* __restrict__ rs_out) {
    __shared__ float ssp[4 * NW][16];
    const int cc = threadIdx.x & 15;
#pragma unroll
    for (int s = threadIdx.x >> 4; s < 4 * NW; s += 16) ssp[s][cc] = ss_slot<NW>(a, s, blockIdx.x * 16 + cc);
    __syncthreads();
    if (threadIdx.x < 16) rs_out[blockIdx.x * 16 + cc] = ss_scale<NW, 16>(a, ssp, cc);
}

// Projections of a prompt-ingestion pass (33..512 tokens).  A workgroup of eight waves (two per SIMD) owns 8 RTW row
// tiles x TCW column tiles; every wave multiplies RTW row tiles of its own with all of the group's columns:
//   - weight blocks go from memory straight into the registers of the one wave that uses them, three chunks ahead
//     (they are stored in operand order, so nothing is gained by a detour through LDS);
//   - the group's operand (hi and lo halves) goes through three LDS buffers of one chunk, KB K steps, each: a chunk's blocks are
//     asked for six chunks ahead, written two ahead and read by all waves.  One barrier per chunk (two steps where a step is
//     few MFMAs), and the first blocks of the next chunk are read before it, so none begins with an LDS latency.
// Bound: the matrix cores.  A loop of these MFMAs alone settles at 1.42-1.48 PFLOP/s on this part (a plain library
// product of 8192^3 reaches 1.48); the draft's gate/up projection (16384 x 2048, 512 columns, hi + lo) runs at 1.11
// PFLOP/s, 62 us.  The rest is the launch, the first loads and the epilogue (14 us of it, by extrapolating the K loop
// to zero steps).  With the weights staged through LDS as well (4 x 4 tiles per wave) it took 75 us, with four waves of
// 4 x 8 tiles, one per SIMD, 78 us: nothing covers a wave's barriers and folds there.
// The arithmetic is that of gemm_bf16 with NW waves: K is cut at the same NW boundaries, each range is accumulated
// from zero by the same MFMA sequence, and the ranges are added in the same order, so the result has the same bits as
// the narrow kernels'.
// EPI_QKV and EPI_RESID have too few row tiles to fill the device: K is cut into the four groups of ranges that the
// narrow kernels add up separately (group_sum), a workgroup does one of them and leaves its sums in `part`
// ([group][row tile][column tile of the launch][64 lanes], fp32), and panel_finish adds the groups and runs the epilogue (target's
// down projection and o projection at 512 columns: 174 us on average as one launch, 74 + 12 us in two).
template <int NW, int EPI, int RTW, int TCW, int KB>
__global__ __launch_bounds__(512, 2) void gemm_panel(const GemmArgs a, const int tiles, const int ncg, const int cg0, f32x4* __restrict__ part) {
    constexpr int CT = kWideCT;
    constexpr bool kSplit = kGrouped<EPI>;
    constexpr bool kScaled = (EPI == EPI_SWIGLU);             // the grouped epilogues are scaled in panel_finish
    constexpr int GC = 16 * TCW, GW = 2 * TCW * 64;           // columns, and operand words per K step, of a column group
    constexpr int WV = 8, TH = 64 * WV, NB = KB * GW / TH;                             // operand words a thread stages per KB steps
    constexpr int kBStep = CT * 128;
    __shared__ float s_rs[kScaled ? GC : 1];
    __shared__ u32x4 sB[3][KB * GW];                          // [K step][column tile][hi, lo][lane]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, cc = lane & 15;
    // Workgroups go to the eight XCDs (one L2 each) round-robin in launch order.  The ncg column groups of a row
    // group take consecutive slots of one XCD, so they run side by side and its weights come from memory once.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int unit = (slot / ncg) * 8 + xcd, cg = slot % ncg, KS = a.KS;
    const int rgi = kSplit ? unit >> 2 : unit, grp = kSplit ? unit & 3 : 0;
    const int tile0 = (rgi * WV + wave) * RTW;
    if (rgi * WV * RTW >= tiles) return;
    // the K ranges of this workgroup: all of them, or those of one group
    int v = kSplit ? grp * (NW / 4) : 0;
    const int v_end = kSplit ? v + NW / 4 : NW;
    const int k0 = (int)(((long)KS * v) / NW), k1 = (int)(((long)KS * v_end) / NW);
    const u32x4* pa[RTW];
#pragma unroll
    for (int r = 0; r < RTW; ++r) pa[r] = a.Wt + (size_t)min(tile0 + r, tiles - 1) * KS * 64;
    const u32x4* pb = a.XB + (size_t)(cg0 + cg) * GW;
    const int k_last = min(max(k1 - 1, k0), KS - 1);   // loads past the range repeat its last step and are never used
    // chunk q: the KB steps from k0 + KB q on
    u32x4 wa[4][KB][RTW], sb[4][NB];
    auto fetch_a1 = [&](int st, int q, int e, int r) { wa[st][e][r] = load16_at(pa[r] + (size_t)min(k0 + q * KB + e, k_last) * 64, lane * 16); };
    auto fetch_b1 = [&](int st, int q, int i) {
        const int e = i * TH / GW;   // GW is a multiple of the threads' words or the other way round: a word's step is uniform
        sb[st][i] = load16_at(pb + (size_t)min(k0 + q * KB + e, k_last) * kBStep + (i * TH - e * GW), tid * 16);
    };
    auto fetch_a = [&](int st, int q) {
#pragma unroll
        for (int e = 0; e < KB; ++e)
#pragma unroll
            for (int r = 0; r < RTW; ++r) fetch_a1(st, q, e, r);
    };
    auto fetch_b = [&](int st, int q) {
#pragma unroll
        for (int i = 0; i < NB; ++i) fetch_b1(st, q, i);
    };
    auto put = [&](int st, int buf) {
#pragma unroll
        for (int i = 0; i < NB; ++i) sB[buf][tid + i * TH] = sb[st][i];
    };
    // in the order of use: the operand of the first two chunks first
    fetch_b(0, 0);
    fetch_b(1, 1);
    fetch_a(0, 0);
    fetch_b(2, 2);
    fetch_a(1, 1);
    fetch_b(3, 3);
    fetch_a(2, 2);
    if (kScaled && tid < GC) s_rs[tid] = a.rs_in[(cg0 + cg) * GC + tid];
    put(0, 0);
    put(1, 1);
    fetch_b(0, 4);
    fetch_b(1, 5);
    f32x4 cur[RTW][TCW], tot[RTW][TCW];
    const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < RTW; ++r)
#pragma unroll
        for (int t = 0; t < TCW; ++t) { cur[r][t] = zero4; tot[r][t] = zero4; }
    __syncthreads();
    u32x4 bh = sB[0][lane], bl = sB[0][64 + lane];
    int buf = 0, buf1 = 1, buf2 = 2;
    int nb = k0;   // where the current range began or ends: the first step of every range folds the one before it
    auto step = [&](int st, int q, int e) {
        constexpr int kSlots = KB * TCW;   // the chunk's writes and loads are spread over its column tiles: a burst of loads
                                           // would hold the wave up while the memory pipeline is full
#pragma unroll
        for (int t = 0; t < TCW; ++t) {
            const int slot = e * TCW + t;
#pragma unroll
            for (int i = slot; i < NB; i += kSlots) {
                sB[buf2][tid + i * TH] = sb[(st + 2) & 3][i];
                fetch_b1((st + 2) & 3, q + 6, i);
            }
#pragma unroll
            for (int x = 0; x < KB * RTW; ++x)
                if (slot == (NB + x) % kSlots) fetch_a1((st + 3) & 3, q + 3, x / RTW, x % RTW);
            const u32x4* nx = slot + 1 < kSlots ? &sB[buf][(slot + 1) * 128] : &sB[buf1][0];
            const u32x4 nh = nx[lane], nl = nx[64 + lane];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < RTW; ++r)
                cur[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[st][e][r]), __builtin_bit_cast(bf16x8, bh),
                                                                    cur[r][t], 0, 0, 0);
#pragma unroll
            for (int r = 0; r < RTW; ++r)
                cur[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[st][e][r]), __builtin_bit_cast(bf16x8, bl),
                                                                    cur[r][t], 0, 0, 0);
            bh = nh;
            bl = nl;
        }
    };
    auto next_chunk = [&]() {
        __syncthreads();
        const int b0 = buf;
        buf = buf1; buf1 = buf2; buf2 = b0;
    };
    // a finished range joins the total; empty ranges (fewer K steps than ranges) add nothing
    auto fold = [&](int ks) {
#pragma unroll
        for (int r = 0; r < RTW; ++r)
#pragma unroll
            for (int t = 0; t < TCW; ++t) {
                tot[r][t] += cur[r][t];
                cur[r][t] = zero4;
            }
        do { ++v; nb = (int)(((long)KS * v) / NW); } while (nb <= ks);
    };
    for (int q0 = 0, ks = k0; ks < k1; q0 += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (ks >= k1) break;
#pragma unroll
            for (int e = 0; e < KB; ++e) {
                if (KB > 1 && ks >= k1) break;   // a last chunk that is not full (nothing after it reads LDS)
                if (ks == nb) fold(ks);
                step(u, q0 + u, e);
                ++ks;
            }
            next_chunk();
        }
    }
    const DescVals dv = load_desc(a.desc);
#pragma unroll
    for (int t = 0; t < TCW; ++t) {
        const int c = (cg0 + cg) * GC + t * 16 + cc;
        const float rs = kScaled ? s_rs[kScaled ? t * 16 + cc : 0] : 1.f;
#pragma unroll
        for (int r = 0; r < RTW; ++r) {
            const f32x4 sum = tot[r][t] + cur[r][t];
            const int tile = tile0 + r;
            if constexpr (kSplit) {
                if (tile < tiles) part[(((size_t)grp * tiles + tile) * (ncg * TCW) + cg * TCW + t) * 64 + lane] = sum;
            } else {
                // whole 16-lane groups agree on c < w, and the shuffles inside the epilogue cross g only
                if (tile < tiles && c < dv.w) epilogue<EPI, CT, false>(a, dv, tile, g, c, sum, rs, EpiPre<EPI>{});
            }
        }
    }
}

// Second half of a grouped projection of a wide pass: adds the four groups' sums in order and runs the epilogue.
// grid (row tiles / 8, column tiles of the gemm_panel launch, the first of which is ct0), 256 threads: a wave finishes two row tiles of one column tile.  Latency: everything
// it reads is asked for at once, the epilogue's inputs beside the partial sums (512 columns of the draft's shape: q/k/v 12.5 ->
// 10.5 us, o and down 7.2 -> 6.4; 100 columns of the qualifier's: 10.0 -> 8.3, 5.6 -> 4.8).  Four row tiles per wave: 11.2 /
// 6.4 and 9.4 / 5.0, one: 10.6 / 6.3 and 8.2 / 4.9.
template <int NW, int EPI>
__global__ __launch_bounds__(256) void panel_finish(const GemmArgs a, const int tiles, const int ct0, const f32x4* __restrict__ part) {
    constexpr int CT = kWideCT;
    __shared__ float ssp[4 * NW][16];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, cc = lane & 15;
    const int ct = blockIdx.y, nct = gridDim.y, c = (ct0 + ct) * 16 + cc;
    const int tile0 = blockIdx.x * 8 + wave * 2;
    f32x4 p[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            p[i][j] = part[(((size_t)j * tiles + min(tile0 + i, tiles - 1)) * nct + ct) * 64 + lane];
    const DescVals dv = load_desc(a.desc);
    EpiPre<EPI> pre[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (c < dv.w && tile0 + i < tiles) epi_prefetch<EPI>(a, dv, tile0 + i, g, c, pre[i]);
    float rs = 1.f;
    if constexpr (EPI == EPI_QKV) {
#pragma unroll
        for (int s = tid >> 4; s < 4 * NW; s += 16) ssp[s][cc] = ss_slot<NW>(a, s, c);
        __syncthreads();
        rs = ss_scale<NW, 16>(a, ssp, cc);
    }
    if (c >= dv.w) return;   // whole 16-lane groups agree, and the shuffles inside the epilogue cross g only
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (tile0 + i >= tiles) break;
        const f32x4 sum = ((p[i][0] + p[i][1]) + p[i][2]) + p[i][3];
        epilogue<EPI, CT, true>(a, dv, tile0 + i, g, c, sum, rs, pre[i]);
    }
}

// o projection of a narrow pass (<= 4 tokens, K <= 2048, one row tile per workgroup): the merge of the attention
// split partials, otherwise a kernel of its own, is done here while the weight blocks are in flight; the merged
// rows go to LDS in B-operand order.  Same K split, MFMA order and reduction as gemm_bf16<1, 16, 1, EPI_RESID>, and
// the same merge arithmetic as attn_combine_bf16, so the result has the same bits as the two-kernel route.
__global__ __launch_bounds__(1024) void gemm_o_narrow(const GemmArgs a, const float* __restrict__ attn_part) {
    constexpr int NW = 16, KSMAX = 64;
    __shared__ f32x4 red[NW - 1][64];
    __shared__ u32x4 sB[KSMAX * 2 * 4 * 4];   // [k step][hi, lo][g][column < 4]
    const int tile = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k0 = (int)(((long)a.KS * wave) / NW), k1 = (int)(((long)a.KS * (wave + 1)) / NW);
    const int g = lane >> 4, cc = lane & 15;
    const u32x4* a_ptr = a.Wt + ((size_t)tile * a.KS + k0) * 64 + lane;
    u32x4 wv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (k0 + u < k1) wv[u] = __builtin_nontemporal_load(a_ptr + (size_t)u * 64);
    const DescVals dv = load_desc(a.desc);
    const int w = dv.w, pos0 = dv.pos0, K = a.KS * 32;
    EpiPre<EPI_RESID> pre;
    if (wave == 0 && cc < w) epi_prefetch<EPI_RESID>(a, dv, tile, g, cc, pre);   // answered while the partials are merged
    uint16_t* sB16 = reinterpret_cast<uint16_t*>(sB);
    // pairs of adjacent head dims: for one token that is exactly one pair per thread, i.e. one memory round trip
    for (int pidx = threadIdx.x; pidx < 2 * K; pidx += 1024) {
        const int c = pidx / (K >> 1), k = (pidx % (K >> 1)) * 2;
        float v[2] = {0.f, 0.f};
        if (c < w) attn_merge<2>(attn_part, (pos0 + c + kAttnSplit) / kAttnSplit, c, k / a.hd, a.H, a.hd, k % a.hd, v);
        uint32_t hi, lo;
        f32x2_split(v[0], v[1], hi, lo);
        const int ks = k >> 5, gq = (k & 31) >> 3, e = k & 7;
        *reinterpret_cast<uint32_t*>(sB16 + ((((ks * 2 + 0) * 4 + gq) * 4 + c) << 3) + e) = hi;
        *reinterpret_cast<uint32_t*>(sB16 + ((((ks * 2 + 1) * 4 + gq) * 4 + c) << 3) + e) = lo;
    }
    __syncthreads();
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
    auto step = [&](const u32x4 wblk, int ks) {
        u32x4 bh = zero, bl = zero;
        if (cc < 4) { bh = sB[((ks * 2 + 0) * 4 + g) * 4 + cc]; bl = sB[((ks * 2 + 1) * 4 + g) * 4 + cc]; }
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wblk), __builtin_bit_cast(bf16x8, bh), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wblk), __builtin_bit_cast(bf16x8, bl), acc, 0, 0, 0);
    };
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (k0 + u < k1) step(wv[u], k0 + u);
    for (int ks = k0 + 4; ks < k1; ++ks) step(__builtin_nontemporal_load(a_ptr + (size_t)(ks - k0) * 64), ks);
    if (wave > 0) red[wave - 1][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    acc = group_sum<NW, EPI_RESID>([&](int v) { return v == 0 ? acc : red[v - 1][lane]; });
    if (cc < w) epilogue<EPI_RESID, 2, true>(a, dv, tile, g, cc, acc, 1.f, pre);
}

// token embedding: x = E[token]; also the first RMSNorm's operand and sum-of-squares partials.  grid (d/16, column tiles),
// 64 threads
template <int CT>
__global__ __launch_bounds__(64) void embed_pack(const uint16_t* embed, const PassDesc* desc, float* x, void* xb,
                                                 const float* gain, float* ss_out, int d, int V) {
    const int tile = blockIdx.x, lane = threadIdx.x, g = lane >> 4, cc = lane & 15;
    const int w = desc->w, KS = d >> 5, c = blockIdx.y * 16 + cc;
    if (c >= w) return;   // whole 16-lane groups agree on it, and the shuffles below cross g only
    int tok = desc->tok[c];
    tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
    const int n = tile * 16 + g * 4;
    const size_t idx = ((((size_t)(tok >> 4) * KS + (n >> 5)) * 64) + ((n & 31) >> 3) * 16 + (tok & 15)) * 8 + (n & 7);
    const uint2 raw = *reinterpret_cast<const uint2*>(embed + idx);
    const float v[4] = {bf16_to_f32(raw.x & 0xffff), bf16_to_f32(raw.x >> 16), bf16_to_f32(raw.y & 0xffff), bf16_to_f32(raw.y >> 16)};
    *reinterpret_cast<float4*>(x + (size_t)c * d + n) = make_float4(v[0], v[1], v[2], v[3]);
    const float4 gn = *reinterpret_cast<const float4*>(gain + n);
    const float pk[4] = {v[0] * gn.x, v[1] * gn.y, v[2] * gn.z, v[3] * gn.w};
    pack4<CT>(xb, c, n, pk);
    float ss = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    ss = rows_sum(ss);
    if (g == 0) ss_out[tile * (16 * CT) + c] = ss;
}

// ---- attention, bf16 KV cache, MFMA ---------------------------------------------------------------------
// grid (KV heads, nsplit_max, query tiles), 256 threads.  A workgroup owns one KV head, the absolute key range
// [split * 128, +128) and 16 query rows rho = token * G + head_in_group; wave j owns the 32 keys
// [split * 128 + 32 j, +32):
//   S^T = K Q^T    v_mfma_f32_16x16x32_bf16, A = 16 keys x 32 head dims: one contiguous 1 KiB tile of the K planes
//                  (hi, lo), B = queries as bf16 hi + lo built in registers; result lane (g, c): keys 4g..4g+3 of query c
//   P   = 2^(S - max) per query over the wave's 32 keys (masked causally), kept in registers: the result
//         layout of S^T is an A operand layout of v_mfma_f32_16x16x32_bf16 (attn_probs)
//   O   = P V      B = 2 x 4 consecutive keys of one head dim: two contiguous 512-byte tiles of the V planes
// The four waves' (max, sum, O) are merged through LDS in wave order and written as one partial per split.
// Memory round trips on the critical path: the pass descriptor and the page-table entry travel together, then the
// queries (from L2), keys and values go out back to back; the kernel is latency-bound, so that is what counts.
// Two waves per SIMD are asked for (at head dim 128 the kernel would otherwise take 284 registers and run one workgroup
// per CU): with dozens of key ranges a launch has several workgroups per CU, and their round trips then overlap.
template <int HD>
__device__ inline float attn_scale() { return rsqrtf((float)HD) * 1.4426950408889634f; }   // scores come out in base 2

// Probabilities of one wave's 32 keys (two 16-key score tiles, lane (g, c): keys 4 g + r of query c) relative to `msafe`, as the
// A operand of v_mfma_f32_16x16x32_bf16 in hi and lo halves, and the query's sum over the 32 keys.  The instruction's k
// index is free as long as both operands agree on it: lane group g's eight entries are keys 4 g .. 4 g + 3 of the first tile,
// then of the second, which is how the scores lie already and how two 8-byte pieces of the V planes fit together.
__device__ inline void attn_probs(const f32x4 (&S)[2], float msafe, u32x4& Ph, u32x4& Pl, float& l) {
    l = 0.f;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = exp2_hw(S[kt][r] - msafe);   // 2^(-inf) = 0 for masked keys
            l += p[r];
        }
        uint32_t h0, l0, h1, l1;
        f32x2_split(p[0], p[1], h0, l0);
        f32x2_split(p[2], p[3], h1, l1);
        Ph[2 * kt] = h0; Ph[2 * kt + 1] = h1;
        Pl[2 * kt] = l0; Pl[2 * kt + 1] = l1;
    }
    l = rows_sum(l);
}
// (p_hi + p_lo)(v_hi + v_lo) without the lo * lo term, 16 queries x 16 JT head dims over 32 keys; the head dims' chains side
// by side
template <int JT>
__device__ inline void attn_pv(u32x4 Ph, u32x4 Pl, const u32x4 (&vh)[JT], const u32x4 (&vl)[JT], f32x4 (&O)[JT]) {
#pragma unroll
    for (int t3 = 0; t3 < 3; ++t3)
#pragma unroll
        for (int j = 0; j < JT; ++j)
            O[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, t3 == 1 ? Pl : Ph), __builtin_bit_cast(bf16x8, t3 < 2 ? vh[j] : vl[j]),
                                                           t3 == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : O[j], 0, 0, 0);
}

template <int HD>
__global__ __launch_bounds__(256, 2) void attn_mfma(const float* qkv, const PassDesc* desc, const uint16_t* kv,
                                                 const int32_t* page_table, int n_pages, float* part, int layer, int L, int H,
                                                 int KV, int nqkv, int qt_per_wg) {
    constexpr int KSQ = HD / 32, JT = HD / 16;
    __shared__ float mrg[4][16][HD + 2];
    const int gkv = blockIdx.x, split = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, cq = lane & 15;
    const int key0 = split * kAttnSplit, wkey0 = key0 + wave * 32;
    // asked for together with the descriptor: the entry exists for every key range a launch covers
    const int page = page_table[min(wkey0 / kPage, n_pages - 1)];
    const int w = desc->w, pos0 = desc->pos0;
    const int kv_max = pos0 + w;
    const int G = H / KV, R = w * G;
    if (key0 >= kv_max || (int)blockIdx.z * qt_per_wg * 16 >= R) return;
    const bool wave_live = wkey0 < kv_max;
    const float scale = attn_scale<HD>();
    // query rows of the first tile, as they come from the q/k/v projection (fp32); converted when they are used
    auto load_q = [&](int qt, float (&v)[KSQ][8]) {
        const int rho = qt * 16 + cq;
        const float* qrow = qkv + (size_t)(rho / G) * nqkv + (size_t)(gkv * G + rho % G) * HD;
#pragma unroll
        for (int ks = 0; ks < KSQ; ++ks) {
            if (rho < R) {
                const float4 a0 = *reinterpret_cast<const float4*>(qrow + ks * 32 + g * 8);
                const float4 a1 = *reinterpret_cast<const float4*>(qrow + ks * 32 + g * 8 + 4);
                v[ks][0] = a0.x; v[ks][1] = a0.y; v[ks][2] = a0.z; v[ks][3] = a0.w;
                v[ks][4] = a1.x; v[ks][5] = a1.y; v[ks][6] = a1.z; v[ks][7] = a1.w;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[ks][e] = 0.f;
            }
        }
    };
    float qraw[KSQ][8];
    if (wave_live) load_q(blockIdx.z * qt_per_wg, qraw);
    // the wave's keys and values stay in registers for all of the workgroup's query tiles
    u32x4 ka[2][KSQ], kb[2][KSQ];   // hi and lo halves
    uint2 vraw[JT][2], vlow[JT][2];
    if (wave_live) {
        // this wave's 32 keys are two 16-slot tiles of one page
        const int st0 = (wkey0 % kPage) >> 4;
        constexpr size_t kPlane = (size_t)kPage * HD;
        const uint16_t* Kp = kv + kv_plane(page, layer, L, gkv, KV, 0, HD);
        const uint16_t* Vp = Kp + 2 * kPlane;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int ks = 0; ks < KSQ; ++ks) {
                const uint16_t* p = Kp + ((size_t)((st0 + kt) * KSQ + ks) * 64 + lane) * 8;
                ka[kt][ks] = *reinterpret_cast<const u32x4*>(p);
                kb[kt][ks] = *reinterpret_cast<const u32x4*>(p + kPlane);
            }
#pragma unroll
        for (int j = 0; j < JT; ++j)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const uint16_t* p = Vp + ((size_t)(j * (kPage >> 4) + st0 + kt) * 64 + lane) * 4;
                vraw[j][kt] = *reinterpret_cast<const uint2*>(p);
                vlow[j][kt] = *reinterpret_cast<const uint2*>(p + kPlane);
            }
    }
    for (int qi = 0; qi < qt_per_wg; ++qi) {
    const int qt = blockIdx.z * qt_per_wg + qi;
    if (qt * 16 >= R) break;
    // every key of this split lies after the tile's last query: nothing to attend to, and the merge never reads it
    if (key0 > pos0 + ((qt * 16 + 15 < R ? qt * 16 + 15 : R - 1) / G)) {
        if (wave_live && qi + 1 < qt_per_wg) load_q(qt + 1, qraw);   // qraw always holds the queries of the tile about to be worked on
        continue;
    }
    const int rho = qt * 16 + cq;
    float m = -INFINITY, l = 0.f;
    f32x4 O[JT];
#pragma unroll
    for (int j = 0; j < JT; ++j) O[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave_live) {
        // query row rho as B operand: lane (g, c) holds head dims 32 ks + 8 g .. + 8 of row c, scaled by 1/sqrt(hd)
        u32x4 qh[KSQ], ql[KSQ];
#pragma unroll
        for (int ks = 0; ks < KSQ; ++ks) {
            uint32_t hw[4], lw[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f32x2_split(qraw[ks][2 * e] * scale, qraw[ks][2 * e + 1] * scale, hw[e], lw[e]);
            }
            qh[ks] = u32x4{hw[0], hw[1], hw[2], hw[3]};
            ql[ks] = u32x4{lw[0], lw[1], lw[2], lw[3]};
        }
        if (qi + 1 < qt_per_wg) load_q(qt + 1, qraw);   // the next tile's queries travel while this tile is worked on
        f32x4 Sx[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            Sx[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KSQ; ++ks) {
                // (k_hi + k_lo)(q_hi + q_lo) without the lo * lo term (2^-18 relative)
                Sx[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[kt][ks]), __builtin_bit_cast(bf16x8, qh[ks]), Sx[kt], 0, 0, 0);
                Sx[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[kt][ks]), __builtin_bit_cast(bf16x8, ql[ks]), Sx[kt], 0, 0, 0);
                Sx[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kb[kt][ks]), __builtin_bit_cast(bf16x8, qh[ks]), Sx[kt], 0, 0, 0);
            }
        }
        // causal mask: key position <= query position; rows beyond R see nothing
        const int qpos = rho < R ? pos0 + rho / G : -1;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int kp = wkey0 + kt * 16 + g * 4 + r;
                if (kp > qpos) Sx[kt][r] = -INFINITY;
                m = fmaxf(m, Sx[kt][r]);
            }
        m = rows_max(m);
        const float msafe = m == -INFINITY ? 0.f : m;
        u32x4 Ph, Pl;
        attn_probs(Sx, msafe, Ph, Pl, l);
        u32x4 vh[JT], vl[JT];
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            vh[j] = u32x4{vraw[j][0].x, vraw[j][0].y, vraw[j][1].x, vraw[j][1].y};
            vl[j] = u32x4{vlow[j][0].x, vlow[j][0].y, vlow[j][1].x, vlow[j][1].y};
        }
        attn_pv<JT>(Ph, Pl, vh, vl, O);
    }
    // merge the four waves: O lane (g, c) holds queries 4g + r, head dim 16 j + c
    if (g == 0) { mrg[wave][cq][0] = m; mrg[wave][cq][1] = l; }
#pragma unroll
    for (int j = 0; j < JT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) mrg[wave][g * 4 + r][2 + j * 16 + cq] = O[j][r];
    __syncthreads();
    // sixteen threads per query row: each works out the row's merged maximum and the four waves' rescaling factors for
    // itself (the same arithmetic in every thread), one of them stores (max, sum), and together they merge the row's
    // head dims, sixteen at a time
    {
        const int qr = threadIdx.x >> 4, i0 = threadIdx.x & 15, rr = qt * 16 + qr;
        if (rr < R) {
            float M = -INFINITY;
#pragma unroll
            for (int v = 0; v < 4; ++v) M = fmaxf(M, mrg[v][qr][0]);
            float fac[4], Ls = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                fac[v] = mrg[v][qr][0] == -INFINITY ? 0.f : exp2_hw(mrg[v][qr][0] - M);
                Ls = fmaf(mrg[v][qr][1], fac[v], Ls);
            }
            const int rh = (rr / G) * H + gkv * G + rr % G;
            float* out = part + ((size_t)split * kCols * H + rh) * (HD + 2);
            if (i0 == 0) { out[0] = M; out[1] = Ls; }
#pragma unroll
            for (int jj = 0; jj < JT; ++jj) {
                const int i = jj * 16 + i0;
                float o = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) o = fmaf(mrg[v][qr][2 + i], fac[v], o);
                out[2 + i] = o;
            }
        }
    }
    if (qi + 1 < qt_per_wg) __syncthreads();   // the merge buffer is reused by the next query tile
    }
}

// grid (wmax, H), block hd: merges the split partials and writes the O-projection's input operand (wide passes)
template <int CT>
__global__ void attn_combine_bf16(const float* part, const PassDesc* desc, void* xb, int H, int hd) {
    const int c = blockIdx.x, h = blockIdx.y, i = threadIdx.x;
    if (c >= desc->w) return;
    const int nsp = (desc->pos0 + c + kAttnSplit) / kAttnSplit;  // splits holding keys <= pos0 + c
    float o[1];
    attn_merge<1>(part, nsp, c, h, H, hd, i, o);
    pack_store<CT>(xb, c, h * hd + i, o[0]);
}

// The same merge for long contexts (more than eight key ranges): one workgroup per (token, head) brings the partials of
// all its ranges into LDS with one round of loads (the thread-per-head-dim form above walks them in dependent rounds of
// eight), works out every range's factors (a lane per range, from the maximum before it by a scan over the lanes) and
// then sums in range order: the arithmetic, hence the bits, of attn_merge.
// Latency, at thousands of tokens of context: 5.9 -> 4.45 us on average over the three models' passes at 4.1 K (32 ranges; the
// factors from a walk over all maxima before a range, single floats loaded with a division each: 5.9; the scan alone: 5.6).
// grid (wmax, H), 256 threads, dynamic LDS: nsplit * (hd + 4) floats.
template <int CT>
__global__ __launch_bounds__(256) void attn_combine_long(const float* part, const PassDesc* desc, void* xb, int H, int hd, int nsp_cap) {
    extern __shared__ __align__(16) float cmb[];
    const int c = blockIdx.x, h = blockIdx.y;
    if (c >= desc->w) return;
    // splits holding keys <= pos0 + c; never more than the launch covers (the LDS area is sized for those)
    const int nsp = min((desc->pos0 + c + kAttnSplit) / kAttnSplit, nsp_cap);
    const int row = hd + 2, hp = hd >> 1, nr = 256 / hp, tid = threadIdx.x, lane = tid & 63;
    const size_t stride = (size_t)kCols * H * row;
    const float* p0 = part + ((size_t)c * H + h) * row;   // even: pairs of floats are aligned
    float4* fac = reinterpret_cast<float4*>(cmb + nsp * hd);   // al, be, l be of every range
    auto max_sum = [&](int sp) { return sp < nsp ? *reinterpret_cast<const float2*>(p0 + (size_t)sp * stride) : make_float2(-INFINITY, 0.f); };
    float2 ml = make_float2(-INFINITY, 0.f);
    if (tid < 64) ml = max_sum(lane);
    // batches of 12 pairs per thread, all of a batch in flight together (one batch covers 48 ranges at head dim 128)
    constexpr int kBatch = 12;
    const int sub = tid / hp, pair = tid - sub * hp;
    for (int base = 0; base < nsp; base += kBatch * nr) {
        float2 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int sp = base + u * nr + sub;
            v[u] = sub < nr && sp < nsp ? *reinterpret_cast<const float2*>(p0 + (size_t)sp * stride + 2 + 2 * pair) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int sp = base + u * nr + sub;
            if (sub < nr && sp < nsp) *reinterpret_cast<float2*>(cmb + sp * hd + 2 * pair) = v[u];
        }
    }
    if (tid < 64) {   // the maximum before every range: an inclusive scan over the lanes, shifted by one
        float carry = -INFINITY;
        for (int s0 = 0; s0 < nsp; s0 += 64) {
            if (s0) ml = max_sum(s0 + lane);
            float run = ml.x;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const float up = __shfl_up(run, d);
                if (lane >= d) run = fmaxf(run, up);
            }
            run = fmaxf(run, carry);
            const float up = __shfl_up(run, 1);
            const MergeFac f = merge_fac(lane ? up : carry, ml.x);
            if (s0 + lane < nsp) fac[s0 + lane] = make_float4(f.al, f.be, ml.y * f.be, 0.f);
            carry = __shfl(run, 63);
        }
    }
    __syncthreads();
    if (tid < hd) {
        const int i = tid;
        float Lsum = 0.f, o = 0.f;
#pragma unroll 8
        for (int sp = 0; sp < nsp; ++sp) {
            const float4 f = fac[sp];
            Lsum = fmaf(Lsum, f.x, f.z);                                          // merge_add
            o = merge_add(o, cmb[sp * hd + i], MergeFac{0.f, f.x, f.y});
        }
        pack_store<CT>(xb, c, h * hd + i, o / Lsum);
    }
}

// ---- pieces of the sweeps over a tile's key ranges (attn_wide, attn_pair) ----
// one plane pair of a page in LDS: hi, then lo, HD / 8 * kPage words each
template <int HD>
constexpr int kPlaneWords = kPage * HD / 8;
// a tile's queries as B operand, scaled: lane (g, c) holds head dims 32 ks + 8 g .. + 8 of row c
template <int HD>
__device__ inline void sweep_queries(const float* __restrict__ qkv, int nqkv, int rho, int R, int G, int gkv, int g, u32x4 (&qh)[HD / 32], u32x4 (&ql)[HD / 32]) {
    const float scale = attn_scale<HD>();
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) {
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (rho < R) {
            const float* qrow = qkv + (size_t)(rho / G) * nqkv + (size_t)(gkv * G + rho % G) * HD + ks * 32 + g * 8;
            const float4 a0 = *reinterpret_cast<const float4*>(qrow), a1 = *reinterpret_cast<const float4*>(qrow + 4);
            v[0] = a0.x; v[1] = a0.y; v[2] = a0.z; v[3] = a0.w; v[4] = a1.x; v[5] = a1.y; v[6] = a1.z; v[7] = a1.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t hi, lo;
            f32x2_split(v[2 * e] * scale, v[2 * e + 1] * scale, hi, lo);
            qh[ks][e] = hi;
            ql[ks][e] = lo;
        }
    }
}
// scores of a range's four groups of 32 keys, masked, each group's maximum per query and the range's
template <int HD>
__device__ inline void sweep_scores(const u32x4* sK, const u32x4 (&qh)[HD / 32], const u32x4 (&ql)[HD / 32], int key0, int qpos, int qpos_first,
                                    f32x4 (&S)[4][2], float (&mv)[4], float& Ms) {
    constexpr int KSQ = HD / 32, PW = kPlaneWords<HD>;
    const int lane = threadIdx.x & 63, g = lane >> 4;
    // (k_hi + k_lo)(q_hi + q_lo) without the lo * lo term (2^-18 relative); eight independent chains side by side
#pragma unroll
    for (int kt = 0; kt < 8; ++kt) S[kt >> 1][kt & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KSQ; ++ks) {
        u32x4 kh[8], kl[8];
#pragma unroll
        for (int kt = 0; kt < 8; ++kt) {
            const u32x4* kp = sK + (kt >> 2) * 2 * PW + ((kt & 3) * KSQ + ks) * 64 + lane;
            kh[kt] = kp[0];
            kl[kt] = kp[PW];
        }
#pragma unroll
        for (int t3 = 0; t3 < 3; ++t3)
#pragma unroll
            for (int kt = 0; kt < 8; ++kt)
                S[kt >> 1][kt & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, t3 < 2 ? kh[kt] : kl[kt]), __builtin_bit_cast(bf16x8, t3 == 1 ? ql[ks] : qh[ks]),
                    S[kt >> 1][kt & 1], 0, 0, 0);
    }
    if (key0 + kAttnSplit - 1 > qpos_first) {   // causal mask: key position <= query position
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (key0 + v * 32 + k2 * 16 + g * 4 + r > qpos) S[v][k2][r] = -INFINITY;
    }
    Ms = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float m = -INFINITY;
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, S[v][k2][r]);
        mv[v] = rows_max(m);
        Ms = fmaxf(Ms, mv[v]);
    }
}
// a per-query value, held by the lanes of column c, for the four queries 4 g + r of the P V layout
__device__ inline void to_rows(float v, float (&out)[4]) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = __shfl(v, 4 * g + r, kWave);
}
// sum of exponentials and P V of a range, its groups added in order; probs(v, ...) as attn_probs for group v
template <int HD, typename Probs>
__device__ inline void sweep_values(const u32x4* sV, Probs probs, const float (&mv)[4], float Ms, float& Ls, f32x4 (&os)[HD / 16]) {
    constexpr int JT = HD / 16, PW = kPlaneWords<HD>;
    const int lane = threadIdx.x & 63;
    float fac[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) fac[v] = mv[v] == -INFINITY ? 0.f : exp2_hw(mv[v] - Ms);
    Ls = 0.f;
#pragma unroll
    for (int j = 0; j < JT; ++j) os[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        u32x4 Ph, Pl;
        float l, fr[4];
        probs(v, Ph, Pl, l);
        Ls = fmaf(l, fac[v], Ls);
        to_rows(fac[v], fr);
        const uint2* vp = reinterpret_cast<const uint2*>(sV + (v >> 1) * 2 * PW) + ((v & 1) * 2) * 64 + lane;
        u32x4 vh[JT], vl[JT];
        f32x4 O[JT];
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            const uint2 h0 = vp[j * 256], h1 = vp[j * 256 + 64], l0 = vp[2 * PW + j * 256], l1 = vp[2 * PW + j * 256 + 64];
            vh[j] = u32x4{h0.x, h0.y, h1.x, h1.y};
            vl[j] = u32x4{l0.x, l0.y, l1.x, l1.y};
        }
        attn_pv<JT>(Ph, Pl, vh, vl, O);
#pragma unroll
        for (int j = 0; j < JT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) os[j][r] = fmaf(O[j][r], fr[r], os[j][r]);
    }
}
// the running (M, Lsum, o) takes a range in
template <int JT>
__device__ inline void sweep_merge(float Ms, float Ls, const f32x4 (&os)[JT], float& M, float& Lsum, f32x4 (&o)[JT]) {
    const MergeFac f = merge_fac(M, Ms);
    M = f.M;
    Lsum = merge_add(Lsum, Ls, f);
    float al[4], be[4];
    to_rows(f.al, al);
    to_rows(f.be, be);
#pragma unroll
    for (int j = 0; j < JT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[j][r] = merge_add(o[j][r], os[j][r], MergeFac{0.f, al[r], be[r]});
}
// o projection's operand of the tile
template <int JT>
__device__ inline void sweep_store(void* xb, int row0, int R, int G, int gkv, float Lsum, const f32x4 (&o)[JT]) {
    const int lane = threadIdx.x & 63, g = lane >> 4, cq = lane & 15;
    float Lr[4];
    to_rows(Lsum, Lr);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int rr = row0 + 4 * g + r;
        if (rr >= R) continue;
        const int c = rr / G, f0 = (gkv * G + rr % G) * (16 * JT) + cq;
#pragma unroll
        for (int j = 0; j < JT; ++j) pack_store<kWideCT>(xb, c, f0 + 16 * j, o[j][r] / Lr[r]);
    }
}
// K (half 0) or V (half 1) planes of a range's two pages, hi and lo, by T threads through registers into LDS
template <int HD, int T>
struct SweepStage {
    static constexpr int PW = kPlaneWords<HD>, NS = 4 * PW / T;   // words per thread
    static_assert(kAttnSplit == 2 * kPage, "a key range is two pages");
    u32x4 st[NS];
    __device__ void load(const uint16_t* __restrict__ kv, const int32_t* __restrict__ page_table, int n_pages, int layer, int L, int gkv, int KV, int s, int half) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int page = page_table[min(2 * s + p, n_pages - 1)];
            const u32x4* src = reinterpret_cast<const u32x4*>(kv + kv_plane(page, layer, L, gkv, KV, 2 * half, HD));   // hi and lo planes are adjacent
#pragma unroll
            for (int i = 0; i < NS / 2; ++i) st[p * (NS / 2) + i] = src[threadIdx.x + i * T];
        }
    }
    __device__ void put(u32x4* dst) const {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < NS / 2; ++i) dst[p * 2 * PW + threadIdx.x + i * T] = st[p * (NS / 2) + i];
    }
};

// Attention of a prompt-ingestion pass in one sweep: a workgroup of four waves owns four consecutive 16-row query tiles of
// one kv head, one per wave, and walks the key ranges from the first to the last one its queries see.  A range's K planes
// (hi, lo), then its V planes, go through LDS for the four waves (K of the next range travels during P V, V during Q K^T);
// every wave keeps its tile's running (M, Lsum, o) in registers and writes the o projection's operand itself, so no
// partials go to memory and there is no merge kernel.  Within a range the arithmetic is that of attn_mfma: four groups of
// 32 keys (its four waves), each from its own maximum, added in order; ranges are merged as attn_merge does: same bits.
// With a workgroup per (kv head, range, four tiles) passes over a 3000-token prompt (head dim 64) spent 59 us per layer here and
// 30 us in the merge, waiting on loads and barriers per 16-row tile; this took 52 us (10 us worth of MFMAs and 19 us of vector
// instructions a wave, one wave per SIMD, so little of that overlaps: attn_pair overlaps them, and is taken where it fits).
// grid ceil(query tiles / 4) * KV; 128 KB of LDS at head dim 128 (one workgroup per CU).
template <int HD>
constexpr int kAttnWideLds = 8 * kPage * HD * 2;   // two pages x (K or V: hi, lo) each for K and V, bytes
template <int HD>
__global__ __launch_bounds__(256, 1) void attn_wide(const float* __restrict__ qkv, const PassDesc* desc, const uint16_t* __restrict__ kv,
                                                    const int32_t* __restrict__ page_table, int n_pages, void* xb, int layer, int L, int H,
                                                    int KV, int nqkv) {
    constexpr int JT = HD / 16;
    extern __shared__ u32x4 aw_lds[];
    u32x4* sK = aw_lds;            // [2 pages][hi, lo][plane]
    u32x4* sV = aw_lds + 4 * kPlaneWords<HD>;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, cq = lane & 15;
    // consecutive workgroups go round the eight XCDs: with eight kv heads each head's keys and values stay in one L2
    const int gkv = blockIdx.x % KV, grp = gridDim.x / KV - 1 - blockIdx.x / KV;   // the groups with the most ranges first
    const int w = desc->w, pos0 = desc->pos0, G = H / KV, R = w * G;
    if (grp * 64 >= R) return;
    const int tile = grp * 4 + wave, row0 = tile * 16;
    const int nsp = (pos0 + (min(R, grp * 64 + 64) - 1) / G) / kAttnSplit + 1;                        // ranges of the workgroup
    const int my_nsp = row0 < R ? (pos0 + (min(R, row0 + 16) - 1) / G) / kAttnSplit + 1 : 0;   // and of this wave's tile
    SweepStage<HD, 256> st;
    st.load(kv, page_table, n_pages, layer, L, gkv, KV, 0, 0);
    const int rho = row0 + cq;
    u32x4 qh[HD / 32], ql[HD / 32];
    sweep_queries<HD>(qkv, nqkv, rho, R, G, gkv, g, qh, ql);
    const int qpos = rho < R ? pos0 + rho / G : -1, qpos_first = pos0 + row0 / G;
    float M = -INFINITY, Lsum = 0.f;
    f32x4 o[JT];
#pragma unroll
    for (int j = 0; j < JT; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    st.put(sK);
    __syncthreads();
    for (int s = 0; s < nsp; ++s) {
        st.load(kv, page_table, n_pages, layer, L, gkv, KV, s, 1);
        const bool live = s < my_nsp;
        f32x4 S[4][2];
        float mv[4], Ms;
        if (live) sweep_scores<HD>(sK, qh, ql, s * kAttnSplit, qpos, qpos_first, S, mv, Ms);
        st.put(sV);
        __syncthreads();
        if (s + 1 < nsp) st.load(kv, page_table, n_pages, layer, L, gkv, KV, s + 1, 0);
        if (live) {
            float Ls;
            f32x4 os[JT];
            sweep_values<HD>(sV, [&](int v, u32x4& Ph, u32x4& Pl, float& l) { attn_probs(S[v], mv[v] == -INFINITY ? 0.f : mv[v], Ph, Pl, l); }, mv, Ms, Ls, os);
            sweep_merge<JT>(Ms, Ls, os, M, Lsum, o);
        }
        if (s + 1 < nsp) st.put(sK);   // everybody is past this range's K since the barrier above
        __syncthreads();
    }
    sweep_store<JT>(xb, row0, R, G, gkv, Lsum, o);
}

// planes of a range's pages straight into LDS, by T threads: lane l's 16 bytes land at the wave's destination + 16 l
template <int HD, int T>
__device__ inline void sweep_fetch(u32x4* dst, const uint16_t* __restrict__ kv, const int32_t* __restrict__ page_table, int n_pages, int layer, int L, int gkv,
                                   int KV, int s, int half) {
    constexpr int PW = kPlaneWords<HD>, NP = 2 * PW / T;   // words of a page per thread
    const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int page = page_table[min(2 * s + p, n_pages - 1)];
        const u32x4* src = reinterpret_cast<const u32x4*>(kv + kv_plane(page, layer, L, gkv, KV, 2 * half, HD)) + threadIdx.x;
#pragma unroll
        for (int i = 0; i < NP; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + i * T),
                                             (__attribute__((address_space(3))) void*)(dst + p * 2 * PW + w0 + i * T), 16, 0, 0);
    }
}
// One step's work on LDS.  The areas are told apart for the compiler: without that it waits for the fetches before the first read.
template <typename Fetch, typename Work>
__device__ __forceinline__ void apart(u32x4* __restrict__ to_k, u32x4* __restrict__ to_v, const u32x4* __restrict__ k, const u32x4* __restrict__ v,
                                      f32x4* __restrict__ o, float2* __restrict__ ml, Fetch fetch, Work work) {
    fetch(to_k, to_v);
    work(k, v, o, ml);
}
// The sweep of attn_wide with two waves per tile, for head dims up to 64: one takes the even key ranges, the other the odd ones, a step
// apart, so that on every SIMD one wave multiplies by keys and takes exponentials while the other multiplies by values.  In step p
// range p is scored and range p - 1 is summed; K of range p + 1 and V of range p come in meanwhile, straight into LDS (two
// buffers each, so one barrier a step).  The second wave hands its ranges' sums to the first, which merges all of them in
// order: same bits.  144.5 KB of LDS at head dim 64 (one workgroup per CU); at 128 the buffers do not fit.
// Bound: the two waves' vector and matrix instructions, 1.8 us a range if nothing waited, and LDS (1.1 us).  us a launch of 1024 tiles, one
// wave per tile / this, 4, 8, 12, 16, 20 ranges: 18.2 / 16.2, 31.6 / 27.0, 50.6 / 38.6, 66.5 / 50.9, 83.0 / 63.6.  On the way: two waves
// that split every range's keys 72.5 at 20 ranges, this with the buffers filled through registers 70.7-72.4 (with no loads at all
// 56), filled straight but with the exponentials beside the values' products, or with the fetches waited for at the first read, slower.
template <int HD>
constexpr int kAttnPairLds = 16 * kPage * HD * 2 + 4 * (HD / 16 * 64 * 16 + 2 * 16 * 4);
template <int HD>
__global__ __launch_bounds__(512, 1) void attn_pair(const float* __restrict__ qkv, const PassDesc* desc, const uint16_t* __restrict__ kv,
                                                    const int32_t* __restrict__ page_table, int n_pages, void* xb, int layer, int L, int H,
                                                    int KV, int nqkv) {
    constexpr int JT = HD / 16, PW = kPlaneWords<HD>;
    extern __shared__ u32x4 aw_lds[];
    u32x4* sK = aw_lds;            // [2 buffers][2 pages][hi, lo][plane]
    u32x4* sV = aw_lds + 8 * PW;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, cq = lane & 15;
    const int tw = wave & 3, odd = wave >> 2;   // the wave's tile in the workgroup, and whether it takes the odd ranges
    f32x4* sO = reinterpret_cast<f32x4*>(aw_lds + 16 * PW) + tw * JT * 64 + lane;                    // handed over: sums,
    float2* sML = reinterpret_cast<float2*>(aw_lds + 16 * PW + 4 * JT * 64) + tw * 16 + cq;   // maximum and sum of exponentials
    // consecutive workgroups go round the eight XCDs: with eight kv heads each head's keys and values stay in one L2
    const int gkv = blockIdx.x % KV, grp = gridDim.x / KV - 1 - blockIdx.x / KV;   // the groups with the most ranges first
    const int w = desc->w, pos0 = desc->pos0, G = H / KV, R = w * G;
    if (grp * 64 >= R) return;
    const int row0 = (grp * 4 + tw) * 16;
    const int nsp = (pos0 + (min(R, grp * 64 + 64) - 1) / G) / kAttnSplit + 1;                        // ranges of the workgroup
    const int my_nsp = row0 < R ? (pos0 + (min(R, row0 + 16) - 1) / G) / kAttnSplit + 1 : 0;   // and of this wave's tile
    auto fetch = [&](u32x4* dst, int r, int half) {   // K or V of range r
        sweep_fetch<HD, 512>(dst, kv, page_table, n_pages, layer, L, gkv, KV, r, half);
    };
    fetch(sK, 0, 0);
    const int rho = row0 + cq;
    u32x4 qh[HD / 32], ql[HD / 32];
    sweep_queries<HD>(qkv, nqkv, rho, R, G, gkv, g, qh, ql);
    const int qpos = rho < R ? pos0 + rho / G : -1, qpos_first = pos0 + row0 / G;
    float M = -INFINITY, Lsum = 0.f;
    f32x4 o[JT];
    u32x4 Ph[4], Pl[4];   // of the range that the wave scored last, as attn_probs
    float lv[4], mv[4], Ms = -INFINITY;
#pragma unroll
    for (int j = 0; j < JT; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 4; ++v) { Ph[v] = Pl[v] = u32x4{0u, 0u, 0u, 0u}; lv[v] = 0.f; mv[v] = -INFINITY; }
    auto take_odd = [&](const f32x4* sO, const float2* sML) {   // the other wave's range, handed over before the last barrier
        f32x4 os[JT];
#pragma unroll
        for (int j = 0; j < JT; ++j) os[j] = sO[j * 64];
        const float2 ml = *sML;
        sweep_merge<JT>(ml.x, ml.y, os, M, Lsum, o);
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    for (int p = 0; p <= nsp; ++p) {
        // into buffers that were read in the step before the last barrier
        auto next = [&](u32x4* to_k, u32x4* to_v) {
            if (p + 1 < nsp) fetch(to_k, p + 1, 0);
            if (p < nsp) fetch(to_v, p, 1);
        };
        auto work = [&](const u32x4* k, const u32x4* v, f32x4* sO, float2* sML) {
            if ((p & 1) == odd) {
                if (p >= my_nsp) return;
                f32x4 S[4][2];
                sweep_scores<HD>(k, qh, ql, p * kAttnSplit, qpos, qpos_first, S, mv, Ms);
#pragma unroll
                for (int u = 0; u < 4; ++u) attn_probs(S[u], mv[u] == -INFINITY ? 0.f : mv[u], Ph[u], Pl[u], lv[u]);
                return;
            }
            if (odd == 0 && p >= 3 && p - 2 < my_nsp) take_odd(sO, sML);
            if (p == 0 || p - 1 >= my_nsp) return;
            float Ls;
            f32x4 os[JT];
            sweep_values<HD>(v, [&](int u, u32x4& ph, u32x4& pl, float& l) { ph = Ph[u]; pl = Pl[u]; l = lv[u]; }, mv, Ms, Ls, os);
            if (odd) {
#pragma unroll
                for (int j = 0; j < JT; ++j) sO[j * 64] = os[j];
                if (g == 0) *sML = make_float2(Ms, Ls);
            } else {
                sweep_merge<JT>(Ms, Ls, os, M, Lsum, o);
            }
        };
        apart(sK + ((p + 1) & 1) * 4 * PW, sV + (p & 1) * 4 * PW, sK + (p & 1) * 4 * PW, sV + ((p + 1) & 1) * 4 * PW, sO, sML, next, work);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    if (odd) return;
    if ((nsp & 1) == 0 && nsp - 1 < my_nsp) take_odd(sO, sML);   // the last range, if it is the other wave's
    sweep_store<JT>(xb, row0, R, G, gkv, Lsum, o);
}

// ---- fp32 models -------------------------------------------------------------------------------------------
// Projection Y[c][n] = sum_k W[n][k] X[c][k] of a pass of up to 32 tokens, plain VALU, weights row-major [N][K].  These
// models are small, so a pass is a chain of launches of a few microseconds each and what counts is how many there are
// and how long a dependent chain each one holds: the norm in front and the rotation / cache append / SwiGLU / residual
// behind a projection are part of it (5 launches per layer; as kernels of their own they were 10).
// LP lanes share a pair of output rows (n1, n2): a rotary pair, a gate row and its up row, or two neighbours.  A lane
// takes 4 adjacent k of every 4 LP, its sums over NC columns stay in registers and are folded across the LP lanes at
// the end, so the weights are read 16 bytes per lane and the serial part is K / (4 LP) steps.  grid.y workgroups take the
// column groups in turn.  Every column's
// arithmetic is the same whatever NC and the pass width.
enum { F32_QKV, F32_RESID, F32_SWIGLU, F32_LOGITS };
struct F32Args {
    const float* W;
    const float* X;      // [32][K]
    const float* gain;   // RMSNorm of X in front (null: none)
    float* Y;            // QKV: query buffer [32][ldy]; RESID: residual stream; SWIGLU: [32][N / 2]; LOGITS: rows
    int N, K, ldy;
    float eps;
    const PassDesc* desc;
    const float2* rope;  // QKV only, from here
    float* kv;
    const int32_t* page_table;
    int layer, L, H, KV, hd;
};
constexpr int kF32Chunk = 1024;   // K entries of X staged in LDS at a time

template <int EPI, int LP, int NC>
__global__ __launch_bounds__(256) void proj_f32(const F32Args a) {
    __shared__ float xs[NC][kF32Chunk];
    __shared__ float gs[kF32Chunk];
    __shared__ float rsc[NC];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, sub = tid % LP;
    const int K = a.K, npairs = (a.N + 1) >> 1, pair = blockIdx.x * (256 / LP) + tid / LP, pc = min(pair, npairs - 1);
    int n1, n2;
    if constexpr (EPI == F32_QKV) {
        const int half = a.hd >> 1;
        n1 = (pc / half) * a.hd + pc % half;
        n2 = n1 + half;
    } else if constexpr (EPI == F32_SWIGLU) {
        n1 = pc;
        n2 = (a.N >> 1) + pc;
    } else {
        n1 = 2 * pc;
        n2 = min(n1 + 1, a.N - 1);
    }
    const float* w1 = a.W + (size_t)n1 * K;
    const float* w2 = a.W + (size_t)n2 * K;
    // nothing of this depends on the pass descriptor: the first steps' weights and the gains are asked for at once
    constexpr int U = 4;
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 p0[U], q0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = sub * 4 + u * 4 * LP;
        p0[u] = k < K ? *reinterpret_cast<const float4*>(w1 + k) : zero4;
        q0[u] = k < K ? *reinterpret_cast<const float4*>(w2 + k) : zero4;
    }
    const bool once = K <= kF32Chunk;   // X is staged once per column group
    if (a.gain && once)
        for (int k = tid * 4; k < K; k += 1024) *reinterpret_cast<float4*>(gs + k) = *reinterpret_cast<const float4*>(a.gain + k);
    const float inv_k = 1.f / (float)K;
    const int w = a.desc->w, pos0 = a.desc->pos0;
    const int first = EPI == F32_LOGITS ? w - a.desc->n_logit : 0, row0 = EPI == F32_LOGITS ? a.desc->logit_row0 : 0;
    for (int c0 = first + (int)blockIdx.y * NC; c0 < w; c0 += NC * (int)gridDim.y) {
        const int nc = min(NC, w - c0);
        const float* x0 = a.X + (size_t)c0 * K;
        auto square_sum = [&](const float* row) {   // one wave
            float ss = 0.f;
            for (int k = lane * 4; k < K; k += 256) {
                const float4 v = *reinterpret_cast<const float4*>(row + k);
                ss += f32_squares(v);
            }
            return lanes_sum<64>(ss);
        };
        if (a.gain && !once) {
            for (int c = wave; c < nc; c += 4) {
                const float ss = square_sum(x0 + (size_t)c * K);
                if (lane == 0) rsc[c] = f32_rms(ss, inv_k, a.eps);
            }
            __syncthreads();
        }
        float acc1[NC], acc2[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) { acc1[c] = 0.f; acc2[c] = 0.f; }
        auto step = [&](const float4 p, const float4 q, int k) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {   // columns past nc: whatever LDS holds, never stored
                const float4 x = *reinterpret_cast<const float4*>(&xs[c][k]);
                acc1[c] = fmaf(p.x, x.x, acc1[c]); acc1[c] = fmaf(p.y, x.y, acc1[c]);
                acc1[c] = fmaf(p.z, x.z, acc1[c]); acc1[c] = fmaf(p.w, x.w, acc1[c]);
                acc2[c] = fmaf(q.x, x.x, acc2[c]); acc2[c] = fmaf(q.y, x.y, acc2[c]);
                acc2[c] = fmaf(q.z, x.z, acc2[c]); acc2[c] = fmaf(q.w, x.w, acc2[c]);
            }
        };
        for (int kc = 0; kc < K; kc += kF32Chunk) {
            const int kn = min(kF32Chunk, K - kc), kq = kn >> 2;
            if (kc > 0) __syncthreads();   // the previous chunk has been read
            auto normalised = [&](float4 v, int c, int k) {
                const float r = rsc[c];
                const float4 gn = *reinterpret_cast<const float4*>(once ? gs + k : a.gain + kc + k);
                return make_float4(v.x * r * gn.x, v.y * r * gn.y, v.z * r * gn.z, v.w * r * gn.w);
            };
            for (int i = tid; i < nc * kq; i += 256) {
                const int c = i / kq, k = (i - c * kq) * 4;
                const float4 v = *reinterpret_cast<const float4*>(x0 + (size_t)c * K + kc + k);
                *reinterpret_cast<float4*>(&xs[c][k]) = a.gain && !once ? normalised(v, c, k) : v;
            }
            __syncthreads();
            if (a.gain && once) {   // squares and scaling out of LDS: X makes one trip from memory
                for (int c = wave; c < nc; c += 4) {
                    const float ss = square_sum(xs[c]);
                    if (lane == 0) rsc[c] = f32_rms(ss, inv_k, a.eps);
                }
                __syncthreads();
                for (int i = tid; i < nc * kq; i += 256) {
                    const int c = i / kq, k = (i - c * kq) * 4;
                    float4* x = reinterpret_cast<float4*>(&xs[c][k]);
                    *x = normalised(*x, c, k);
                }
                __syncthreads();
            }
            int k = sub * 4;
            if (kc == 0) {
#pragma unroll
                for (int u = 0; u < U; ++u, k += 4 * LP)
                    if (k < kn) step(p0[u], q0[u], k);
            }
#pragma unroll 4
            for (; k < kn; k += 4 * LP)
                step(*reinterpret_cast<const float4*>(w1 + kc + k), *reinterpret_cast<const float4*>(w2 + kc + k), k);
        }
        // lane c of a pair's LP lanes finishes column c
        float v1 = 0.f, v2 = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const float s1 = lanes_sum<LP>(acc1[c]), s2 = lanes_sum<LP>(acc2[c]);
            if (sub == c) { v1 = s1; v2 = s2; }
        }
        if (sub < nc && pair < npairs) {
            const int c = c0 + sub;
            if constexpr (EPI == F32_RESID) {
                float* y = a.Y + (size_t)c * a.ldy;
                y[n1] += v1;
                if (n2 != n1) y[n2] += v2;
            } else if constexpr (EPI == F32_SWIGLU) {
                a.Y[(size_t)c * a.ldy + n1] = f32_silu_up(v1, v2);
            } else if constexpr (EPI == F32_LOGITS) {
                float* y = a.Y + (size_t)(row0 + c - first) * a.ldy;
                y[n1] = v1;
                if (n2 != n1) y[n2] = v2;
            } else {
                const int hd = a.hd, head = n1 / hd, i = n1 % hd, pos = pos0 + c;
                if (head < a.H + a.KV) {
                    const float2 cs = a.rope[(size_t)pos * (hd >> 1) + i];
                    f32_rotate(v1, v2, cs);
                }
                float* y;
                if (head < a.H) {
                    y = a.Y + (size_t)c * a.ldy + (size_t)head * hd;
                } else {
                    const int g = head - a.H, which = g >= a.KV;
                    y = a.kv + kv_base(a.page_table[pos / kPage], a.layer, a.L, which ? g - a.KV : g, a.KV, which, hd) + (size_t)(pos % kPage) * hd;
                }
                y[i] = v1;
                y[i + (hd >> 1)] = v2;
            }
        }
        if (c0 + NC * (int)gridDim.y < w) __syncthreads();   // xs and rsc are written again
    }
}

// Attention of an fp32 model at contexts of at most kF32OneSplits key ranges: one workgroup per (head, query) takes all
// of them, wave v the ranges v, v + 4, and merges them in order; the arithmetic is that of attn_partial and
// attn_combine_f32, so a token's output does not depend on which route its launch takes.
// grid (H, wmax), 256 threads, writes the o projection's input [c][H hd].
constexpr int kF32OneSplits = 8;
__global__ __launch_bounds__(256) void attn_one_f32(const float* __restrict__ qkv, const PassDesc* desc, const float* __restrict__ kv,
                                                    const int32_t* __restrict__ page_table, int n_pages, float* __restrict__ out, int layer,
                                                    int L, int H, int KV, int hd, int nqkv) {
    __shared__ float s_q[128], s_p[4][kAttnSplit], s_m[kF32OneSplits], s_l[kF32OneSplits], s_o[kF32OneSplits][128];
    const int h = blockIdx.x, c = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = h / (H / KV);
    if ((int)threadIdx.x < hd) s_q[threadIdx.x] = qkv[(size_t)c * nqkv + (size_t)h * hd + threadIdx.x];
    __syncthreads();
    const float scale = rsqrtf((float)hd);
    // a key range is two pages; lane j takes keys j and j + 64 of it.  Any page of the table can be read (keys that are not
    // there are masked afterwards), so a wave's first range is on its way before the pass descriptor has arrived
    auto plane = [&](int sp, int half, int which) {
        return kv + kv_base(page_table[min(2 * sp + half, n_pages - 1)], layer, L, g, KV, which, hd);
    };
    auto dot = [&](int sp, int half) {
        const float* kr = plane(sp, half, 0) + (size_t)lane * hd;
        float acc = 0.f;
#pragma unroll 8
        for (int i = 0; i < hd; i += 4) {
            const float4 k4 = *reinterpret_cast<const float4*>(kr + i);
            acc = fmaf(s_q[i], k4.x, acc); acc = fmaf(s_q[i + 1], k4.y, acc);
            acc = fmaf(s_q[i + 2], k4.z, acc); acc = fmaf(s_q[i + 3], k4.w, acc);
        }
        return f32_score(acc, scale);
    };
    float v0[32];   // the first 32 values of head dim `lane` of the first range
    {
        const float* vp = plane(wave, 0, 1) + min(lane, hd - 1);
#pragma unroll
        for (int u = 0; u < 32; ++u) v0[u] = vp[(size_t)u * hd];
    }
    float s0 = dot(wave, 0), s1 = dot(wave, 1);
    if (c >= desc->w) return;
    const int nkeys = desc->pos0 + c + 1, nsp = min((nkeys + kAttnSplit - 1) / kAttnSplit, kF32OneSplits);
    float* p = s_p[wave];
    for (int sp = wave; sp < nsp; sp += 4) {
        const int visible = min(kAttnSplit, nkeys - sp * kAttnSplit);
        if (sp != wave) { s0 = dot(sp, 0); s1 = dot(sp, 1); }
        if (lane >= visible) s0 = -INFINITY;
        if (lane + 64 >= visible) s1 = -INFINITY;
        const float m = lanes_max(fmaxf(s0, s1));
        const float p0 = expf(s0 - m), p1 = expf(s1 - m);  // exp(-inf) = 0 for masked keys
        const float l = lanes_sum<64>(p0 + p1);
        p[lane] = p0;
        p[lane + 64] = p1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < hd; i += 64) {
            float acc = 0.f;
            for (int b = 0; b < visible; b += kPage) {
                const float* vp = plane(sp, b / kPage, 1) + i;
                const int n = min(kPage, visible - b);
#pragma unroll
                for (int j0 = 0; j0 < kPage; j0 += 32) {   // 32 loads in flight; keys past the last one add 0 * 0
                    if (j0 >= n) break;
                    const bool held = sp == wave && b == 0 && j0 == 0 && i == lane;
                    float vv[32];
#pragma unroll
                    for (int u = 0; u < 32; ++u) vv[u] = j0 + u >= n ? 0.f : held ? v0[u] : vp[(size_t)(j0 + u) * hd];
#pragma unroll
                    for (int u = 0; u < 32; ++u) acc = fmaf(p[b + j0 + u], vv[u], acc);
                }
            }
            s_o[sp][i] = acc;
        }
        if (lane == 0) { s_m[sp] = m; s_l[sp] = l; }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (i >= hd) return;
    float M = -INFINITY;
    for (int sp = 0; sp < nsp; ++sp) M = fmaxf(M, s_m[sp]);
    float Lsum = 0.f, o = 0.f;
    for (int sp = 0; sp < nsp; ++sp) {
        const float f = expf(s_m[sp] - M);
        Lsum = fmaf(s_l[sp], f, Lsum);
        o = fmaf(s_o[sp][i], f, o);
    }
    out[(size_t)c * H * hd + h * hd + i] = o / Lsum;
}

// A whole pass of a small fp32 model in one launch.  As a chain of launches (above) such a pass is 5 L + 2 of them at
// ~4.5 us each, of which the launch boundary itself is 1.7 us and the rest the trips to memory that every kernel starts and ends
// with; the arithmetic is next to nothing.  Here the workgroups stay and hand the activations to each other through memory: a
// value travels as a 64-bit slot (value, tag), written and polled with agent-scope accesses, so that the poll that finds the tag
// has the value (an all-gather of 512 slots among 32 workgroups: 1.1 us, on one die or across all eight).  A stage asks for its
// weights first and polls its input while they travel.  The pieces of work and the arithmetic are those of proj_f32 and
// attn_one_f32, so the results have the same bits.  Bound: the chain of exchanges and the instructions of one wave per SIMD between them, 2-4 us a
// stage: the exchange is 1.1 us of it among 32 workgroups and 2 to 2.5 among 192, the rest are instructions (350 to 400 spilled scalar
// registers that the stages read back are a part of them).  Tiny stack, us a pass between events: draft step with its sampling (2
// layers, d 64) 61 -> 30, qualifier (4, d 128, 5 tokens) 120 -> 68, target (6, d 256, 9 tokens) 201 -> 118.
// Tags are the pass's own, one per stage (tag0 + 5 l + 1 ..: q/k/v, attention, o, SwiGLU, down), and no slot is written again
// while somebody may still wait for its former tag:
//   X, Q, A, G hold one row per token and are handled in groups of NC tokens by every projection.  A group's slots of one buffer are
//   written again only by work that needs, through the all-to-all stages in between, the results of everybody who read them.
//   The new keys and values of a layer are read by the attention of later tokens too, whose groups may lag behind: they have
//   slots of their own for every layer.
// Every wait is bounded by the 100 MHz clock: a workgroup whose wait expires (the launch is not resident as a whole) says so in *gone
// and ends, the others follow, and the host runs the round again as chains of launches.  The draft steps behind such a pass get no
// tokens (chain_advance) and end at once: 30 of them would wait 1.5 s in turn.
typedef unsigned long long slot_t;
struct F32Pass {
    const float *embed, *final_norm;
    LayerW w;            // of layer 0; those of layer l lie l * layer_bytes further
    size_t layer_bytes;
    const PassDesc* desc;
    const float2* rope;
    float* kv;
    const int32_t* page_table;
    int n_pages;
    slot_t *X, *Q, *A, *G, *KVn;   // [32][d] residual stream, [32][d] queries, [32][d] attention output, [32][F] SwiGLU output, [L][32][2 KV hd] new keys and values
    float* logits;
    int32_t* gone;
    unsigned long long wait_ticks;
    float eps, inv_d;
    int L, d, H, KV, F, V, hd_log;
    int nux[6];          // per stage: workgroups of a group of columns (attention: heads)
};
constexpr int kF32PassK = 1024;   // largest K of a projection: 16 weights per lane of a row

__device__ inline void slot_store(slot_t* p, uint32_t tag, float v) {
    __hip_atomic_store(p, (slot_t)tag << 32 | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Pairs of slots in one 16-byte load that goes past the caches, as an agent-scope atomic load does; either half of it is as it was stored.  Buffer
// addressing: one register of offset per load, the base in scalar registers.
typedef __amdgpu_buffer_rsrc_t buf_t;
__device__ inline buf_t buf_of(const void* p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000); }
__device__ inline u32x4 pair_load(buf_t b, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 16 | (int)0x80000000); }   // sc1, volatile
// Bound of all the waiting that a stage does: lanes whose first wait ended well beside lanes whose wait expired do not wait once more
struct WaitBound {
    unsigned long long t0, ticks;
    __device__ bool over() const { return wall_clock64() - t0 >= ticks; }
};
// Waits for N pairs of slots at byte offsets off(u), until all of them carry `tag`; false when the bound was over
template <int N, typename O>
__device__ inline bool pairs_wait(buf_t b, O off, uint32_t tag, const WaitBound& bound, u32x4 (&v)[N]) {
    for (;;) {
        uint32_t diff = 0;
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = pair_load(b, off(u));
#pragma unroll
        for (int u = 0; u < N; ++u) diff |= (v[u].y ^ tag) | (v[u].w ^ tag);
        if (diff == 0) return true;
        if (bound.over()) return false;
    }
}
// n slots (even, at least two) from the start of b into LDS, by 256 threads
template <int N>
__device__ inline bool slots_gather_as(int tid, buf_t b, int n, uint32_t tag, const WaitBound& bound, float* dst) {
    u32x4 v[N];
    const bool ok = pairs_wait<N>(b, [&](int u) { return (uint32_t)min(2 * tid + 512 * u, n - 2) * 8; }, tag, bound, v);
#pragma unroll
    for (int u = 0; u < N; ++u)
        if (2 * tid + 512 * u < n) *reinterpret_cast<float2*>(dst + 2 * tid + 512 * u) = make_float2(__uint_as_float(v[u].x), __uint_as_float(v[u].z));
    return ok;
}
__device__ inline bool slots_gather(int tid, const slot_t* p, int n, uint32_t tag, const WaitBound& bound, float* dst) {
    if (2 * tid >= n) return true;
    const buf_t b = buf_of(p, n * 8);
    if (n <= 512) return slots_gather_as<1>(tid, b, n, tag, bound, dst);
    if (n <= 1024) return slots_gather_as<2>(tid, b, n, tag, bound, dst);
    bool ok = true;
    for (int i = 0; i < n && ok; i += 4096) {
        if (2 * tid >= n - i) break;
        ok = slots_gather_as<8>(tid, buf_of(p + i, (n - i) * 8), n - i, tag, bound, dst + i);
    }
    return ok;
}

// The thread's index, worked out anew: the compiler would otherwise keep what every stage derives from it in registers over the
// whole pass (190 spilled registers)
__device__ inline int fresh_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
struct F32PassVals { int w, pos0, n_logit, row0; uint32_t tag0; };
// The stages of a layer, and the logits.  Stage k of layer l takes its input with tag tag0 + 5 l + k and leaves its result with the next.
enum { kStQkv, kStAttn, kStO, kStGateUp, kStDown, kStLogits };

// what a projection reads besides its input: asked for as soon as the products of the stage before are done
struct F32Weights { float4 p[4], q[4], gain[4]; };   // of the lane's two rows; the norm's gains that the lane multiplies with

// This workgroup's part of stage K: row pairs 256 / LP bx .., columns NC cg ..  It has one part at most, the same in every layer.
template <int K_> struct F32Part { int bx, cg; bool mine; };
template <int K_, int NC>
__device__ inline F32Part<K_> f32_part(const F32Pass& a, const F32PassVals& dv) {
    const int b = blockIdx.x, cg = b / a.nux[K_], cols = K_ == kStLogits ? dv.n_logit : dv.w;
    return F32Part<K_>{b - cg * a.nux[K_], cg, K_ == kStAttn ? cg < dv.w : cg * NC < cols};
}
template <int K_>
__device__ inline const float* f32_matrix(const F32Pass& a, int layer) {
    const void* p = K_ == kStQkv ? a.w.wqkv : K_ == kStO ? a.w.wo : K_ == kStGateUp ? a.w.wgu : K_ == kStDown ? a.w.wd : a.embed;
    return reinterpret_cast<const float*>(static_cast<const char*>(p) + (K_ == kStLogits ? 0 : (size_t)layer * a.layer_bytes));
}
template <int K_> constexpr bool kStNorm = K_ == kStQkv || K_ == kStGateUp || K_ == kStLogits;   // an RMSNorm comes first
template <int K_> constexpr bool kStResid = K_ == kStO || K_ == kStDown;
template <int K_>
__device__ inline int f32_rows(const F32Pass& a) { return K_ == kStQkv ? a.d + (2 * a.KV << a.hd_log) : K_ == kStGateUp ? 2 * a.F : K_ == kStLogits ? a.V : a.d; }
// log2 of the lanes that share a row pair, as launch_proj_f32 picks them: 16 for K up to 256, 64 beyond
__device__ inline int f32_lp_log(int k) { return k > 256 ? 6 : 4; }
// the rows of this thread's pair; false: no pair of the matrix (the last one stands in)
template <int K_>
__device__ inline bool f32_pair(const F32Pass& a, const F32Part<K_>& part, int tid, int lp_log, int& n1, int& n2) {
    const int N = f32_rows<K_>(a), npairs = (N + 1) >> 1, pair = (part.bx << (8 - lp_log)) + (tid >> lp_log), pc = min(pair, npairs - 1);
    if constexpr (K_ == kStQkv) {
        const int half_log = a.hd_log - 1;
        n1 = ((pc >> half_log) << a.hd_log) + (pc & ((1 << half_log) - 1));
        n2 = n1 + (1 << half_log);
    } else if constexpr (K_ == kStGateUp) {
        n1 = pc;
        n2 = a.F + pc;
    } else {
        n1 = 2 * pc;
        n2 = K_ == kStLogits ? min(n1 + 1, N - 1) : n1 + 1;
    }
    return pair < npairs;
}
template <int K_>
__device__ inline void f32_fetch(const F32Pass& a, const F32Part<K_>& part, int layer, F32Weights& f) {
    if (!part.mine) return;
    const int K = K_ == kStDown ? a.F : a.d, lp_log = f32_lp_log(K), tid = fresh_tid(), sub = tid & ((1 << lp_log) - 1), lane = tid & 63;
    int n1, n2;
    f32_pair<K_>(a, part, tid, lp_log, n1, n2);
    const buf_t W = buf_of(f32_matrix<K_>(a, layer), (uint32_t)f32_rows<K_>(a) * K * 4);   // 8 MB at most
    const uint32_t o1 = ((uint32_t)n1 * K + sub * 4) * 4, o2 = ((uint32_t)n2 * K + sub * 4) * 4;
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = u << (lp_log + 2);
        f.p[u] = zero4; f.q[u] = zero4;
        if (sub * 4 + k < K) {
            f.p[u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(W, o1, k * 4, 0));
            f.q[u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(W, o2, k * 4, 0));
        }
    }
    if constexpr (kStNorm<K_>) {
        const float* G = K_ == kStLogits ? a.final_norm : reinterpret_cast<const float*>(reinterpret_cast<const char*>(K_ == kStQkv ? a.w.attn_norm : a.w.ffn_norm) + (size_t)layer * a.layer_bytes);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (lane * 4 + u * 256 < K) f.gain[u] = *reinterpret_cast<const float4*>(G + lane * 4 + u * 256);
    }
}

// One projection, K <= kF32PassK.  next() is called once the weights have been used.  rot, page: q/k/v, the rotation and the cache page of
// the column that this lane finishes.  False when a wait expired.
template <int K_, int NC, typename Next>
__device__ inline bool f32_project(const F32Pass& a, float* xs, const float* zeros, int& bad, const F32PassVals& dv, const F32Part<K_>& part, int layer, const F32Weights& f,
                                   float2 rot, int page, Next next) {
    const int K = K_ == kStDown ? a.F : a.d, lp_log = f32_lp_log(K);
    const int tid = fresh_tid(), wave = tid >> 6, lane = tid & 63, sub = tid & ((1 << lp_log) - 1);
    const int c0 = (K_ == kStLogits ? dv.w - dv.n_logit : 0) + part.cg * NC, nc = min(NC, dv.w - c0), c = c0 + sub;
    int n1, n2;
    const bool fin = f32_pair<K_>(a, part, tid, lp_log, n1, n2) && sub < nc;   // lane c of a pair finishes column c
    const uint32_t tag_in = dv.tag0 + 5 * layer + (K_ == kStLogits ? 0 : K_), tag = tag_in + 1;
    auto token_row = [&](int col) {
        const int tok = a.desc->tok[col];
        return a.embed + (size_t)(tok < 0 ? 0 : (tok >= a.V ? a.V - 1 : tok)) * a.d;
    };
    // the residual stream's values that the result is added to: as a rule there since two stages
    u32x4 r = u32x4{0u, 0u, 0u, 0u};
    float y1 = 0.f, y2 = 0.f;
    const buf_t res = buf_of(a.X, kMaxW * a.d * 8);
    const uint32_t res_off = (uint32_t)(c * a.d + n1) * 8;   // rows n1, n1 + 1
    const uint32_t old = K_ == kStDown ? tag_in - 1 : tag_in - 2;
    const bool embedded = K_ == kStO && layer == 0;
    if (kStResid<K_> && fin) {
        if (embedded) {
            const float* row = token_row(c);
            y1 = row[n1]; y2 = row[n2];
        } else {
            r = pair_load(res, res_off);
        }
    }
    __syncthreads();   // the last stage's LDS has been read
    const WaitBound bound{(unsigned long long)wall_clock64(), a.wait_ticks};
    bool ok = true;
    if (K_ == kStQkv && layer == 0) {
        for (int cc = 0; cc < nc; ++cc) {
            const float* row = token_row(c0 + cc);
            for (int k = tid; k < K; k += 256) xs[cc * K + k] = row[k];
        }
    } else {
        const slot_t* src = (K_ == kStO ? a.A : K_ == kStDown ? a.G : a.X) + c0 * K;
        ok = slots_gather(tid, src, nc * K, tag_in, bound, xs);
    }
    if (kStResid<K_> && fin && !embedded && ok) {
        if (r.y != old || r.w != old) {
            u32x4 again[1];
            ok = pairs_wait<1>(res, [&](int) { return res_off; }, old, bound, again);
            r = again[0];
        }
        y1 = __uint_as_float(r.x);
        y2 = __uint_as_float(r.z);
    }
    if (!ok) bad = 1;
    __syncthreads();
    if (bad) return false;
    if constexpr (kStNorm<K_>) {   // a wave sums and scales a column of its own
        for (int col = wave; col < nc; col += 4) {
            float ss = 0.f;
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (lane * 4 + u * 256 < K) {
                    v[u] = *reinterpret_cast<const float4*>(xs + col * K + lane * 4 + u * 256);
                    ss += f32_squares(v[u]);
                }
            const float r = f32_rms(lanes_sum<64>(ss), a.inv_d, a.eps);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float4 gn = f.gain[u];
                if (lane * 4 + u * 256 < K)
                    *reinterpret_cast<float4*>(xs + col * K + lane * 4 + u * 256) = make_float4(v[u].x * r * gn.x, v[u].y * r * gn.y, v[u].z * r * gn.z, v[u].w * r * gn.w);
            }
        }
        __syncthreads();
    }
    float acc1[NC], acc2[NC];
#pragma unroll
    for (int col = 0; col < NC; ++col) { acc1[col] = 0.f; acc2[col] = 0.f; }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if ((u << (lp_log + 2)) >= K) break;
        const int k = (sub + (u << lp_log)) * 4;
        const float4 p = f.p[u], q = f.q[u];
        const float* x0 = k < K ? xs + k : zeros;   // lanes past the row's end: 0 * 0
        const int step = k < K ? K : 0;
#pragma unroll
        for (int col = 0; col < NC; ++col) {   // columns past nc: whatever LDS holds, never stored
            const float4 x = *reinterpret_cast<const float4*>(x0 + col * step);
            acc1[col] = fmaf(p.x, x.x, acc1[col]); acc1[col] = fmaf(p.y, x.y, acc1[col]);
            acc1[col] = fmaf(p.z, x.z, acc1[col]); acc1[col] = fmaf(p.w, x.w, acc1[col]);
            acc2[col] = fmaf(q.x, x.x, acc2[col]); acc2[col] = fmaf(q.y, x.y, acc2[col]);
            acc2[col] = fmaf(q.z, x.z, acc2[col]); acc2[col] = fmaf(q.w, x.w, acc2[col]);
        }
    }
    next();
    float v1 = 0.f, v2 = 0.f;
#pragma unroll
    for (int col = 0; col < NC; ++col) {
        acc1[col] = lanes_sum<16>(acc1[col]);
        acc2[col] = lanes_sum<16>(acc2[col]);
    }
    if (lp_log == 6) {
#pragma unroll
        for (int col = 0; col < NC; ++col) {
            acc1[col] = rows_sum(acc1[col]);
            acc2[col] = rows_sum(acc2[col]);
        }
    }
#pragma unroll
    for (int col = 0; col < NC; ++col)
        if (sub == col) { v1 = acc1[col]; v2 = acc2[col]; }
    if (!fin) return true;
    if constexpr (kStResid<K_>) {
        slot_store(a.X + c * a.d + n1, tag, y1 + v1);
        slot_store(a.X + c * a.d + n2, tag, y2 + v2);
    } else if constexpr (K_ == kStGateUp) {
        slot_store(a.G + c * a.F + n1, tag, f32_silu_up(v1, v2));
    } else if constexpr (K_ == kStLogits) {
        float* y = a.logits + (size_t)(dv.row0 + part.cg * NC + sub) * a.V;
        y[n1] = v1;
        if (n2 != n1) y[n2] = v2;
    } else {
        const int half = 1 << (a.hd_log - 1), kvd = a.KV << a.hd_log;
        if (n1 < a.d + kvd) f32_rotate(v1, v2, rot);
        if (n1 < a.d) {
            slot_store(a.Q + c * a.d + n1, tag, v1);
            slot_store(a.Q + c * a.d + n1 + half, tag, v2);
        } else {
            const int at = n1 - a.d, which = at >= kvd;
            slot_t* s = a.KVn + ((size_t)layer * kMaxW + c) * 2 * kvd + at;
            slot_store(s, tag, v1);
            slot_store(s + half, tag, v2);
            float* y = a.kv + kv_base(page, layer, a.L, (at - which * kvd) >> a.hd_log, a.KV, which, 1 << a.hd_log) +
                       (size_t)(((dv.pos0 + c) % kPage) << a.hd_log) + (at & ((1 << a.hd_log) - 1));   // for later passes
            y[0] = v1;
            y[half] = v2;
        }
    }
    return true;
}

// Attention of the pass: per (head, token) what attn_one_f32 does.  Keys and values of earlier passes come from the cache (asked
// for before the queries are there), this pass's from their slots.
constexpr int f32_pass_attn_lds(int hd) { return hd + 4 * kAttnSplit + 2 * kF32OneSplits + kF32OneSplits * hd + 2 * kMaxW * hd; }   // floats
template <int HD, typename Next>
__device__ inline bool f32_attend(const F32Pass& a, float* lds, int& bad, const int* pages, const F32PassVals& dv, const F32Part<kStAttn>& part, int layer, Next next) {
    // a wave's first range waits in registers: its keys, the values of HELD of them (as many as the registers have room for)
    constexpr bool PRE = HD <= 32;
    constexpr int HELD = HD == 16 ? 64 : 32;
    float *s_q = lds, *s_p = s_q + HD, *s_m = s_p + 4 * kAttnSplit, *s_l = s_m + kF32OneSplits, *s_o = s_l + kF32OneSplits, *s_k = s_o + kF32OneSplits * HD, *s_v = s_k + kMaxW * HD;
    const int tid = fresh_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const uint32_t tag_in = dv.tag0 + 5 * layer + kStAttn, tag = tag_in + 1;
    const float scale = rsqrtf((float)HD);
    const int c = part.cg, h = part.bx, g = h * a.KV / a.H;
    const int nkeys = dv.pos0 + c + 1, nsp = min((nkeys + kAttnSplit - 1) / kAttnSplit, kF32OneSplits);
    auto plane = [&](int sp, int half, int which) {
        return a.kv + kv_base(__builtin_amdgcn_readfirstlane(pages[2 * sp + half]), layer, a.L, g, a.KV, which, HD);
    };
    float4 kr[2][PRE ? HD / 4 : 1];
    float vr[PRE ? HELD : 1];
    if constexpr (PRE) {
        if (wave < nsp) {
            const int old = dv.pos0 - wave * kAttnSplit;   // keys of the range that earlier passes left
#pragma unroll
            for (int half = 0; half < 2; ++half)
                if (half * 64 + lane < old) {
                    const float* p = plane(wave, half, 0) + (size_t)lane * HD;
#pragma unroll
                    for (int i = 0; i < HD / 4; ++i) kr[half][i] = *reinterpret_cast<const float4*>(p + 4 * i);
                }
            const float* p = plane(wave, 0, 1) + min(lane, HD - 1);
#pragma unroll
            for (int b = 0; b < HELD; b += 32) {
                if (b >= old) break;
#pragma unroll
                for (int u = 0; u < 32; ++u) vr[b + u] = p[(size_t)(b + u) * HD];
            }
        }
    }
    __syncthreads();   // the last piece's LDS has been read
    {
        // [token][K, V][hd] in pairs of slots; the query
        const int npairs = (c + 1) * HD, row = 2 * a.KV * HD * 8;   // bytes of a token's slots
        const buf_t kn = buf_of(a.KVn + ((size_t)layer * kMaxW * 2 * a.KV + g) * HD, row * (c + 1)), q = buf_of(a.Q + c * a.d + h * HD, HD * 8);
        u32x4 q0 = u32x4{0u, 0u, 0u, 0u};
        if (tid < HD / 2) q0 = pair_load(q, tid * 16);
        const WaitBound bound{(unsigned long long)wall_clock64(), a.wait_ticks};
        bool ok = true;
        auto gather = [&](auto n, int i0) {
            constexpr int N = decltype(n)::value;
            u32x4 v[N];
            if (!pairs_wait<N>(kn, [&](int u) {
                    const int i = min(i0 + 256 * u, npairs - 1);
                    return (uint32_t)((i / HD) * row + (i & (HD / 2) ? a.KV * HD * 8 : 0) + (i & (HD / 2 - 1)) * 16);
                }, tag_in, bound, v)) ok = false;
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int i = i0 + 256 * u;
                if (i < npairs) *reinterpret_cast<float2*>((i & (HD / 2) ? s_v : s_k) + (i / HD) * HD + 2 * (i & (HD / 2 - 1))) = make_float2(__uint_as_float(v[u].x), __uint_as_float(v[u].z));
            }
        };
        if (tid < npairs) {
            if (npairs <= 256) gather(std::integral_constant<int, 1>{}, tid);
            else for (int i = tid; i < npairs && ok; i += 1024) gather(std::integral_constant<int, 4>{}, i);
        }
        if (tid < HD / 2) {
            if (q0.y != tag_in || q0.w != tag_in) {
                u32x4 again[1];
                if (!pairs_wait<1>(q, [&](int) { return (uint32_t)tid * 16; }, tag_in, bound, again)) ok = false;
                q0 = again[0];
            }
            *reinterpret_cast<float2*>(s_q + 2 * tid) = make_float2(__uint_as_float(q0.x), __uint_as_float(q0.z));
        }
        if (!ok) bad = 1;
    }
    __syncthreads();
    if (bad) return false;
    next();
    for (int sp = wave; sp < nsp; sp += 4) {
        const int visible = min(kAttnSplit, nkeys - sp * kAttnSplit), old = dv.pos0 - sp * kAttnSplit;
        const bool held = PRE && sp == wave;
        float* p = s_p + wave * kAttnSplit;
        float s[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int j = half * 64 + lane;
            float acc = 0.f;
            auto dot4 = [&](int i, const float4 k4) {
                acc = fmaf(s_q[i], k4.x, acc); acc = fmaf(s_q[i + 1], k4.y, acc);
                acc = fmaf(s_q[i + 2], k4.z, acc); acc = fmaf(s_q[i + 3], k4.w, acc);
            };
            if (j < old) {
                if (held) {
                    if constexpr (PRE) {
#pragma unroll
                        for (int i = 0; i < HD / 4; ++i) dot4(4 * i, kr[half][i]);
                    }
                } else {
                    const float* k = plane(sp, half, 0) + (size_t)lane * HD;
#pragma unroll 8
                    for (int i = 0; i < HD; i += 4) dot4(i, *reinterpret_cast<const float4*>(k + i));
                }
            } else if (j < visible) {
                const float* k = s_k + (j - old) * HD;
#pragma unroll 4
                for (int i = 0; i < HD; i += 4) dot4(i, *reinterpret_cast<const float4*>(k + i));
            }
            s[half] = j < visible ? f32_score(acc, scale) : -INFINITY;
        }
        const float m = lanes_max(fmaxf(s[0], s[1]));
        const float p0 = expf(s[0] - m), p1 = expf(s[1] - m);  // exp(-inf) = 0 for masked keys
        const float l = lanes_sum<64>(p0 + p1);
        p[lane] = p0;
        p[lane + 64] = p1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < HD; i += 64) {
            float acc = 0.f;
            const int n = min(old, visible);   // keys past the last old one add p * 0
            auto add = [&](int b, const float* v) {
#pragma unroll
                for (int u = 0; u < 32; ++u) acc = fmaf(p[b + u], b + u < old ? v[u] : 0.f, acc);
            };
            int b = 0;
            if constexpr (PRE) {
                if (held) {
                    if (n > 0) { add(0, vr); b = 32; }
                    if (HELD > 32 && n > 32) { add(32, vr + (HELD - 32)); b = 64; }
                }
            }
#pragma unroll 1
            for (; b < n; b += 32) {
                const float* v = plane(sp, b / kPage, 1) + (size_t)(b % kPage) * HD + i;
                float vv[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) vv[u] = v[(size_t)u * HD];
                add(b, vv);
            }
#pragma unroll 8
            for (int j = max(old, 0); j < visible; ++j) acc = fmaf(p[j], s_v[(j - old) * HD + i], acc);
            if (nsp == 1) slot_store(a.A + c * a.d + h * HD + i, tag, acc / l);   // nothing to merge
            s_o[sp * HD + i] = acc;
        }
        if (lane == 0) { s_m[sp] = m; s_l[sp] = l; }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (nsp == 1) return true;
    __syncthreads();
    if (tid < HD) {
        float M = -INFINITY;
        for (int sp = 0; sp < nsp; ++sp) M = fmaxf(M, s_m[sp]);
        float Lsum = 0.f, o = 0.f;
        for (int sp = 0; sp < nsp; ++sp) {
            const float f = expf(s_m[sp] - M);
            Lsum = fmaf(s_l[sp], f, Lsum);
            o = fmaf(s_o[sp * HD + tid], f, o);
        }
        slot_store(a.A + (size_t)c * a.d + h * HD + tid, tag, o / Lsum);
    }
    return true;
}

template <int HD, int NC>
__global__ __launch_bounds__(256, 2) void pass_f32(const F32Pass a) {
    constexpr int kProj = NC * kF32PassK, kAttn = f32_pass_attn_lds(HD);
    __shared__ __align__(16) float lds[kProj > kAttn ? kProj : kAttn];
    __shared__ __align__(16) float zeros[4];
    __shared__ int bad, pages[2 * kF32OneSplits];
    if (threadIdx.x < 4) zeros[threadIdx.x] = 0.f;
    const F32PassVals dv{a.desc->w, a.desc->pos0, a.desc->n_logit, a.desc->logit_row0, a.desc->tag0};
    if (threadIdx.x == 0) bad = 0;
    if (threadIdx.x < 2 * kF32OneSplits) pages[threadIdx.x] = a.page_table[min((int)threadIdx.x, a.n_pages - 1)];
    const auto qkv = f32_part<kStQkv, NC>(a, dv);
    const auto attn = f32_part<kStAttn, 1>(a, dv);
    const auto o = f32_part<kStO, NC>(a, dv);
    const auto gu = f32_part<kStGateUp, NC>(a, dv);
    const auto down = f32_part<kStDown, NC>(a, dv);
    const auto lm = f32_part<kStLogits, NC>(a, dv);
    F32Weights f{};
    f32_fetch(a, qkv, 0, f);
    float2 rot = make_float2(1.f, 0.f);
    int page = 0;
    if (qkv.mine) {
        const int lp_log = f32_lp_log(a.d), c = min(qkv.cg * NC + ((int)threadIdx.x & ((1 << lp_log) - 1)), dv.w - 1), pos = dv.pos0 + c;
        int n1, n2;
        f32_pair<kStQkv>(a, qkv, threadIdx.x, lp_log, n1, n2);
        rot = a.rope[(size_t)pos * (HD / 2) + (n1 & (HD - 1))];   // read for the values as well, and not used
        page = a.page_table[pos / kPage];
    }
    __syncthreads();
    bool ok = true;
    for (int l = 0; l < a.L && ok; ++l) {
        if (qkv.mine) ok = f32_project<kStQkv, NC>(a, lds, zeros, bad, dv, qkv, l, f, rot, page, [] {});
        auto fetch_o = [&] { f32_fetch(a, o, l, f); };
        if (!attn.mine) fetch_o();
        else if (ok) ok = f32_attend<HD>(a, lds, bad, pages, dv, attn, l, fetch_o);
        auto fetch_gu = [&] { f32_fetch(a, gu, l, f); };
        if (!o.mine) fetch_gu();
        else if (ok) ok = f32_project<kStO, NC>(a, lds, zeros, bad, dv, o, l, f, rot, page, fetch_gu);
        auto fetch_down = [&] { f32_fetch(a, down, l, f); };
        if (!gu.mine) fetch_down();
        else if (ok) ok = f32_project<kStGateUp, NC>(a, lds, zeros, bad, dv, gu, l, f, rot, page, fetch_down);
        auto fetch_next = [&] { if (l + 1 < a.L) f32_fetch(a, qkv, l + 1, f); else f32_fetch(a, lm, 0, f); };
        if (!down.mine) fetch_next();
        else if (ok) ok = f32_project<kStDown, NC>(a, lds, zeros, bad, dv, down, l, f, rot, page, fetch_next);
    }
    if (lm.mine && ok) ok = f32_project<kStLogits, NC>(a, lds, zeros, bad, dv, lm, a.L, f, rot, page, [] {});
    if (!ok && threadIdx.x == 0) __hip_atomic_store(a.gone, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- profiler ---------------------------------------------------------------------------------------
int Profiler::row_of(const char* name) {
    for (size_t i = 0; i < rows.size(); ++i)
        if (!strncmp(rows[i].name, name, sizeof(rows[i].name))) return (int)i;
    KernelAcc r;
    memset(r.name, 0, sizeof(r.name));
    strncpy(r.name, name, sizeof(r.name) - 1);
    rows.push_back(r);
    return (int)rows.size() - 1;
}
hipEvent_t Profiler::get_event() {
    if (!free_events.empty()) { hipEvent_t e = free_events.back(); free_events.pop_back(); return e; }
    hipEvent_t e;
    (void)hipEventCreate(&e);
    return e;
}
void Profiler::begin(hipStream_t s, int row, double bytes) {
    Pending p{row, get_event(), get_event()};
    (void)hipEventRecord(p.a, s);
    pending.push_back(p);
    rows[row].launches++;
    rows[row].bytes += bytes;
}
void Profiler::end(hipStream_t s) { (void)hipEventRecord(pending.back().b, s); }
void Profiler::flush() {
    for (auto& p : pending) {
        (void)hipEventSynchronize(p.b);
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, p.a, p.b);
        rows[p.row].ms += ms;
        free_events.push_back(p.a);
        free_events.push_back(p.b);
    }
    pending.clear();
}
void Profiler::clear() { flush(); rows.clear(); }
Profiler::~Profiler() {
    flush();
    for (auto e : free_events) (void)hipEventDestroy(e);
}

// ---- sizing / init ----------------------------------------------------------------------------------
static size_t esize(int dtype) { return dtype == PSD_BF16 ? 2 : 4; }

static int round16(int n) { return (n + 15) & ~15; }

static int attn_lds_bytes(int hd) { return (2 * kAttnSplit * (hd + 1) + 4 * hd + 4 * kAttnSplit) * (int)sizeof(float); }

// most LDS a narrow GEMM may use for staging its operand (beside its 16 KB of partial sums)
constexpr size_t kLbMaxBytes = 128 * 1024;

template <int EPI>
static int lb_kernels_init(char* err) {
    PSD_HIP(hipFuncSetAttribute((const void*)gemm_bf16<1, 16, 1, EPI, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLbMaxBytes), err);
    PSD_HIP(hipFuncSetAttribute((const void*)gemm_bf16<1, 8, 2, EPI, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLbMaxBytes), err);
    PSD_HIP(hipFuncSetAttribute((const void*)gemm_bf16<1, 8, 1, EPI, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLbMaxBytes), err);
    return PSD_OK;
}

// Places for the workgroups of one-launch passes: three quarters of what the device holds of them, whatever the mix of
// instantiations (each takes at most 1 / n of a compute unit if n of the largest fit into one).  The last quarter is left to launches
// whose workgroups wait for a few neighbours only (a row of an ACCEPT sweep: 64): with room for those, everything else ends by itself.
constexpr int kMaxDevices = 64;   // devices beyond take the chains
struct DevicePlaces {
    Places places;
    int cus = 0;
};
static DevicePlaces g_pass_places[kMaxDevices];

template <int HD>
static hipError_t pass_f32_fit(int* least) {
    for (const void* f : {(const void*)pass_f32<HD, 1>, (const void*)pass_f32<HD, 4>, (const void*)pass_f32<HD, 8>}) {
        int n = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 256, 0);
        if (e != hipSuccess) return e;
        *least = std::min(*least, n);
    }
    return hipSuccess;
}
static int pass_places_init(char* err) {
    static std::mutex once;
    std::lock_guard<std::mutex> hold(once);
    int dev = 0, least = 1 << 20;
    PSD_HIP(hipGetDevice(&dev), err);
    if (dev >= kMaxDevices || g_pass_places[dev].cus > 0) return PSD_OK;
    DevicePlaces& d = g_pass_places[dev];
    PSD_HIP(pass_f32_fit<16>(&least), err);
    PSD_HIP(pass_f32_fit<32>(&least), err);
    PSD_HIP(pass_f32_fit<64>(&least), err);
    PSD_HIP(pass_f32_fit<128>(&least), err);
    int cus = 0;
    PSD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), err);
    d.places.open(cus * least * 3 / 4);
    d.cus = cus;
    return PSD_OK;
}

int model_kernels_init(char* err) {
    // attention stages two pages of K and V as fp32 in LDS: up to ~135 KB of the 160 KB a gfx950 CU has
    PSD_HIP(hipFuncSetAttribute((const void*)attn_partial, hipFuncAttributeMaxDynamicSharedMemorySize,
                                attn_lds_bytes(128)), err);
    PSD_HIP(hipFuncSetAttribute((const void*)attn_wide<128>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnWideLds<128>), err);
    PSD_HIP(hipFuncSetAttribute((const void*)attn_wide<64>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnWideLds<64>), err);
    PSD_HIP(hipFuncSetAttribute((const void*)attn_pair<64>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnPairLds<64>), err);
    PSD_HIP(hipFuncSetAttribute((const void*)attn_pair<32>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnPairLds<32>), err);
    int rc;
    if ((rc = lb_kernels_init<EPI_RESID>(err)) != PSD_OK) return rc;
    if ((rc = lb_kernels_init<EPI_LOGITS>(err)) != PSD_OK) return rc;
    return pass_places_init(err);
}

// bytes of the four K quarters' sums of one group of tcw column tiles
static size_t panel_group_bytes(int tiles, int tcw) { return (size_t)4 * tiles * tcw * 64 * sizeof(f32x4); }

constexpr size_t kDescBytes = (sizeof(PassDesc) + 255) / 256 * 256;

// walks the allocation sequence; with a dry pool this only measures.  roomy: with what wide passes need to run every projection
// in one launch
static int model_carve(Model& M, Pool& pool, bool roomy) {
    const size_t es = esize(M.dtype);
    const size_t q = (size_t)M.H * M.hd;
    bool ok = true;
    auto take = [&](size_t bytes) { void* p = pool.take(bytes); if (!p && !pool.dry) ok = false; return p; };
    M.embed = take((size_t)M.Vpad * M.d * es);
    M.layers.resize(M.L);
    for (int l = 0; l < M.L; ++l) {
        LayerW& w = M.layers[l];
        w.attn_norm = (const float*)take(M.d * sizeof(float));
        w.wqkv = take((size_t)M.nqkv * M.d * es);
        w.wo = take((size_t)M.d * q * es);
        w.ffn_norm = (const float*)take(M.d * sizeof(float));
        w.wgu = take((size_t)2 * M.F * M.d * es);
        w.wd = take((size_t)M.d * M.F * es);
    }
    M.final_norm = (const float*)take(M.d * sizeof(float));
    M.rope = (const float2*)take((size_t)M.max_seq * (M.hd / 2) * sizeof(float2));
    M.kv = take((size_t)M.n_pages * M.L * M.KV * 2 * kPage * M.hd * 4);   // fp32, or bf16 hi + lo
    const size_t kmax = std::max((size_t)M.d, (size_t)M.F);
    M.x = (float*)take((size_t)kCols * M.d * sizeof(float));
    M.xb = take(kmax * 128);
    if (M.dtype == PSD_BF16) {
        M.xb2 = take(kmax * 128);
        M.ss = (float*)take((size_t)(M.d / 16) * 32 * sizeof(float));
        M.xbw = take(kmax * 4 * kCols);
        M.ssw = (float*)take((size_t)(M.d / 16) * kCols * sizeof(float));
        M.xbw2 = take(kmax * 4 * kCols);
    }
    // The sums of a wide pass's K quarters lie in the attention partials, which hold nothing while a projection runs, at their end
    // first, and go on in a piece behind them where the cache is too short for that (under 770 to 1500 tokens; o and down always
    // fit).  Without that piece the q/k/v projection also has xbw2 in front, which the attention behind it writes, and runs in
    // as many launches as it then takes.  (Lines that every die's L2 has read shortly before, as xbw2's, take longer to write:
    // 512 columns, d 512, 4 heads and kv heads: q/k/v 16.5 us a launch, 20.1 from the start of xbw2 on.)  gemm_panel may
    // leave any bits in operand columns that the pass does not have; every column of a product is on its own, and no kernel
    // stores those.
    const size_t xbw2_at = pool.used - kmax * 4 * kCols, part_bytes = (size_t)M.nsplit_max * kCols * M.H * (M.hd + 2) * sizeof(float);
    M.attn_part = (float*)take(part_bytes);
    const size_t part_at = pool.used - part_bytes;
    if (M.dtype == PSD_BF16) {
        const int widest = std::min(M.ingest_max, M.nsplit_max * 128);
        const size_t sums = panel_group_bytes(round16(M.nqkv) / 16, widest / 16);
        if (roomy && sums > part_bytes) (void)take(sums - part_bytes);
        M.panel_qkv = PanelScratch{M.xbw2, pool.used - xbw2_at};
        M.panel_res = PanelScratch{M.attn_part, pool.used - part_at};
        M.panel_rs = M.attn_part;
    }
    M.qkv = (float*)take((size_t)kCols * M.nqkv * sizeof(float));
    if (M.dtype == PSD_F32) M.gu = (float*)take((size_t)kMaxW * M.F * sizeof(float));
    // the page table behind the pass descriptor, so that creation clears them in one go (70 us of the 1.4 ms of a tiny stack each)
    char* desc = (char*)take(kDescBytes + (size_t)M.n_pages * sizeof(int32_t));
    M.desc = (PassDesc*)desc;
    M.page_table = desc ? (int32_t*)(desc + kDescBytes) : nullptr;
    return ok ? PSD_OK : PSD_ENOMEM;
}

static void model_shape(Model& M, const psd_model_desc& m, int max_seq) {
    M.L = m.n_layers; M.d = m.d_model; M.H = m.n_heads; M.KV = m.n_kv_heads; M.hd = m.d_model / m.n_heads;
    M.F = m.d_ffn; M.V = m.vocab; M.Vpad = m.dtype == PSD_BF16 ? round16(m.vocab) : m.vocab;
    M.nqkv = (M.H + 2 * M.KV) * M.hd;
    M.dtype = m.dtype; M.theta = m.rope_theta; M.eps = m.rms_eps;
    M.max_seq = max_seq;
    M.n_pages = (max_seq + kPage - 1) / kPage;
    M.nsplit_max = (max_seq + kAttnSplit - 1) / kAttnSplit;
    // what the interface takes: 512 tokens per ingestion pass where no K range of any projection is empty, else 128
    auto ranges_ok = [](int n, int k) { return k / 32 >= (round16(n) / 16 <= 256 ? 16 : 8); };
    M.ingest_max = M.dtype != PSD_BF16 ? kMaxW
                   : (ranges_ok(M.nqkv, M.d) && ranges_ok(M.d, M.H * M.hd) && ranges_ok(2 * M.F, M.d) && ranges_ok(M.d, M.F)) ? kCols : 128;
}

// Slots of a one-launch pass lie in the rows of the residual stream and of the q/k/v buffer beyond the 32 that an fp32 pass can have:
// nothing else ever writes them, so what they hold is zero (from the creation on) or an older tag.
static bool f32_slots_fit(const Model& M) {
    const size_t rows = kCols - kMaxW, kv = (size_t)M.KV * M.hd;
    return (size_t)kMaxW * (3 * M.d + M.F) * sizeof(slot_t) <= rows * M.d * sizeof(float) &&
           (size_t)M.L * kMaxW * 2 * kv * sizeof(slot_t) <= rows * M.nqkv * sizeof(float);
}

// workgroups per group of columns of every stage (attention: heads per token)
static void f32_pass_parts(const Model& M, int nux[6]) {
    auto parts = [](int n, int k) { const int pw = k > 256 ? 4 : 16; return ((n + 1) / 2 + pw - 1) / pw; };
    nux[0] = parts(M.nqkv, M.d); nux[1] = M.H; nux[2] = parts(M.d, M.d);
    nux[3] = parts(2 * M.F, M.d); nux[4] = parts(M.d, M.F); nux[5] = parts(M.V, M.d);
}
// workgroups of a one-launch pass: one for every part of the largest stage
static int f32_pass_grid(const Model& M, int wcls) {
    int nux[6], most = 0;
    f32_pass_parts(M, nux);
    const int groups = wcls == 1 ? 1 : wcls <= 16 ? (wcls + 3) / 4 : (wcls + 7) / 8;
    for (int i = 0; i < 6; ++i) most = std::max(most, nux[i] * (i == 1 ? wcls : groups));
    return most;
}
// A pass in one launch, of a workgroup per CU at most (grid_max): models whose projections that many can hold (16 weights per lane of a
// row: d and d_ffn up to 1024; no more than the 2 M weights of a projection up to which proj_f32 gives every group of columns
// workgroups of its own) and whose slots fit (d_ffn up to 4.5 d, layers up to 3.75 (H / KV + 2)).  The LM head counts in the grid: on 256
// CUs the vocabulary may have 8192 entries (2048 where d > 256) in passes of up to four tokens, a quarter of that in passes of 13-16 and
// 25-32; one model's classes may go either way.  Nowhere slower than the chain as a graph, over 13 shapes up to these limits, 20 to 900
// tokens of context and 1 to 31 tokens a pass; us a draft step, one launch / chain: d 64, 2 layers 30 / 58; d 256, 6 layers 90 / 168; d 512, 4
// layers 78 / 111; d 1024 in 64 heads, 4 layers 82 / 126; d 256, 8 layers, head dim 128 behind 900 tokens 335 / 509.
static bool f32_one_launch(const Model& M) {
    const size_t most = (size_t)2 << 20;
    return M.dtype == PSD_F32 && M.d <= kF32PassK && M.F <= kF32PassK && (size_t)2 * M.F * M.d <= most && (size_t)M.nqkv * M.d <= most &&
           (size_t)M.V * M.d <= most && f32_slots_fit(M);
}

size_t model_pool_bytes(const psd_model_desc& m, int max_seq, bool roomy) {
    Model M;
    model_shape(M, m, max_seq);
    Pool p;
    p.dry = true;
    model_carve(M, p, roomy);
    return p.used + 256;
}

static size_t blob_elems(const psd_model_desc& m) {
    const size_t d = m.d_model, hd = d / m.n_heads, q = (size_t)m.n_heads * hd, kv = (size_t)m.n_kv_heads * hd, F = m.d_ffn;
    return (size_t)m.vocab * d + (size_t)m.n_layers * (d + q * d + 2 * kv * d + d * q + d + 2 * F * d + d * F) + d;
}

int model_init(Model& M, const psd_model_desc& m, const char* tag, int max_seq, bool scramble_pages, Pool& pool, bool roomy,
               hipStream_t stream, char* err) {
    if (!m.weights) PSD_FAIL(PSD_EINVAL, err, "%s: weights pointer is null", tag);
    if (m.dtype != PSD_F32 && m.dtype != PSD_BF16) PSD_FAIL(PSD_EINVAL, err, "%s: dtype %d", tag, m.dtype);
    if (m.n_layers < 1 || m.d_model < 32 || m.n_heads < 1 || m.n_kv_heads < 1 || m.d_ffn < 32 || m.vocab < 2)
        PSD_FAIL(PSD_EINVAL, err, "%s: bad shape", tag);
    if (m.d_model % m.n_heads || m.n_heads % m.n_kv_heads || m.d_model % 32 || m.d_ffn % 32)
        PSD_FAIL(PSD_EINVAL, err, "%s: d %% H, H %% KV, d %% 32 and F %% 32 must all be 0", tag);
    const int hd = m.d_model / m.n_heads;
    if (hd != 16 && hd != 32 && hd != 64 && hd != 128) PSD_FAIL(PSD_EINVAL, err, "%s: head dim %d not in {16,32,64,128}", tag, hd);
    if (m.dtype == PSD_BF16 && hd == 16) PSD_FAIL(PSD_EINVAL, err, "%s: bf16 models need a head dim of 32, 64 or 128", tag);
    if (!(m.rope_theta > 0.f) || !(m.rms_eps >= 0.f)) PSD_FAIL(PSD_EINVAL, err, "%s: rope_theta / rms_eps", tag);
    if (m.weights_bytes != blob_elems(m) * esize(m.dtype))
        PSD_FAIL(PSD_EINVAL, err, "%s: weights_bytes %zu, shape implies %zu", tag, m.weights_bytes, blob_elems(m) * esize(m.dtype));
    model_shape(M, m, max_seq);
    M.tag = tag;
    int rc = model_carve(M, pool, roomy);
    if (rc != PSD_OK) PSD_FAIL(PSD_ENOMEM, err, "%s: device pool too small (%zu bytes needed so far)", tag, pool.used);

    const bool bf = M.dtype == PSD_BF16;
    const size_t es = esize(M.dtype);
    const size_t q = (size_t)M.H * M.hd, d = M.d, F = M.F;
    const size_t biggest = std::max({(size_t)M.V * d, 2 * F * d, (size_t)M.nqkv * d});
    void* stage = nullptr;
    PSD_HIP(hipMalloc(&stage, biggest * es), err);
    struct Guard { void* p; ~Guard() { (void)hipFree(p); } } guard{stage};
    const char* src = (const char*)m.weights;
    // uploads `rows x cols` elements from the blob into dst, re-tiled when bf16
    auto put_matrix = [&](const void* dst, size_t rows, size_t cols, int mode = 0, int hd_arg = 0) -> int {
        const size_t bytes = rows * cols * es;
        if (bf) {
            PSD_HIP(hipMemcpyAsync(stage, src, bytes, hipMemcpyHostToDevice, stream), err);
            const size_t chunks = (size_t)round16((int)rows) / 16 * (cols / 32) * 64;
            tile_bf16<<<(unsigned)((chunks + 255) / 256), 256, 0, stream>>>((const uint4*)stage, (uint4*)dst, (int)rows, (int)cols, chunks, mode, hd_arg);
            PSD_HIP(hipStreamSynchronize(stream), err);  // the staging buffer is reused by the next tensor
        } else {
            PSD_HIP(hipMemcpyAsync((void*)dst, src, bytes, hipMemcpyHostToDevice, stream), err);
            PSD_HIP(hipStreamSynchronize(stream), err);
        }
        src += bytes;
        M.weight_bytes += bytes;
        return PSD_OK;
    };
    auto put_norm = [&](const float* dst) -> int {
        const size_t bytes = d * es;
        if (bf) {
            PSD_HIP(hipMemcpyAsync(stage, src, bytes, hipMemcpyHostToDevice, stream), err);
            bf16_to_f32_vec<<<(unsigned)((d + 255) / 256), 256, 0, stream>>>((const uint16_t*)stage, (float*)dst, (int)d);
            PSD_HIP(hipStreamSynchronize(stream), err);
        } else {
            PSD_HIP(hipMemcpyAsync((void*)dst, src, bytes, hipMemcpyHostToDevice, stream), err);
            PSD_HIP(hipStreamSynchronize(stream), err);
        }
        src += bytes;
        return PSD_OK;
    };
    M.weight_bytes = 0;
    if ((rc = put_matrix(M.embed, M.V, d)) != PSD_OK) return rc;
    for (int l = 0; l < M.L; ++l) {
        LayerW& w = M.layers[l];
        if ((rc = put_norm(w.attn_norm)) != PSD_OK) return rc;
        if ((rc = put_matrix(w.wqkv, M.nqkv, d, bf ? 1 : 0, M.hd)) != PSD_OK) return rc;  // wq, wk, wv are adjacent in the blob
        if ((rc = put_matrix(w.wo, d, q)) != PSD_OK) return rc;
        if ((rc = put_norm(w.ffn_norm)) != PSD_OK) return rc;
        if ((rc = put_matrix(w.wgu, 2 * F, d, bf ? 2 : 0, (int)F)) != PSD_OK) return rc;   // w_gate, w_up adjacent
        if ((rc = put_matrix(w.wd, d, F)) != PSD_OK) return rc;
    }
    if ((rc = put_norm(M.final_norm)) != PSD_OK) return rc;
    const int half = M.hd / 2, n_tab = M.max_seq * half;
    rope_table<<<(n_tab + 255) / 256, 256, 0, stream>>>((float2*)M.rope, M.max_seq, half, (double)M.theta);
    // scratch starts zeroed so that never-written operand columns hold finite values
    const size_t kmax = std::max(d, F);
    PSD_HIP(hipMemsetAsync(M.xb, 0, kmax * 128, stream), err);
    PSD_HIP(hipMemsetAsync(M.x, 0, (size_t)kCols * d * sizeof(float), stream), err);
    PSD_HIP(hipMemsetAsync(M.qkv, 0, (size_t)kCols * M.nqkv * sizeof(float), stream), err);
    // the descriptor and the page table: every entry is a valid page at all times (blocks without one name page 0), so that
    // attention kernels may read, and then mask, a block that is not mapped
    PSD_HIP(hipMemsetAsync(M.desc, 0, kDescBytes + (size_t)M.n_pages * sizeof(int32_t), stream), err);
    // KV pages start as zeros: attention may read (and mask) slots of a page that were never written
    PSD_HIP(hipMemsetAsync(M.kv, 0, (size_t)M.n_pages * M.L * M.KV * 2 * kPage * M.hd * 4, stream), err);
    if (bf) {
        PSD_HIP(hipMemsetAsync(M.xb2, 0, kmax * 128, stream), err);
        PSD_HIP(hipMemsetAsync(M.ss, 0, (size_t)(M.d / 16) * 32 * sizeof(float), stream), err);
        PSD_HIP(hipMemsetAsync(M.xbw, 0, kmax * 4 * kCols, stream), err);
        PSD_HIP(hipMemsetAsync(M.xbw2, 0, kmax * 4 * kCols, stream), err);
        PSD_HIP(hipMemsetAsync(M.ssw, 0, (size_t)(M.d / 16) * kCols * sizeof(float), stream), err);
    }
    // page bookkeeping: every logical block unmapped, free list in (optionally scrambled) order
    M.h_page_table.assign(M.n_pages, -1);
    M.free_pages.clear();
    for (int p = M.n_pages - 1; p >= 0; --p) M.free_pages.push_back(p);
    if (scramble_pages) {  // deterministic shuffle: physical pages no longer follow logical order
        uint64_t s = 0x9E3779B97F4A7C15ull;
        for (int i = M.n_pages - 1; i > 0; --i) {
            s = s * 6364136223846793005ull + 1442695040888963407ull;
            std::swap(M.free_pages[i], M.free_pages[(s >> 33) % (uint64_t)(i + 1)]);
        }
    }
    M.pages_mapped = 0;
    M.len = 0;
    int dev = 0;
    PSD_HIP(hipGetDevice(&dev), err);
    M.one_launch = f32_one_launch(M) && dev < kMaxDevices;
    if (M.one_launch) {
        M.places = &g_pass_places[dev].places;
        M.grid_max = std::min(g_pass_places[dev].cus, M.places->total());
    }
    M.tag_last = 0;
    PSD_HIP(hipStreamSynchronize(stream), err);
    PSD_HIP(hipGetLastError(), err);
    return PSD_OK;
}

int model_places(const Model& M, int wcls) {
    const int grid = M.one_launch ? f32_pass_grid(M, wcls) : 0;
    return grid <= M.grid_max ? Places::of(grid) : 0;
}

bool model_one_launch(const Model& M, int wcls, const float* logits) {
    return M.room && logits && model_places(M, wcls) > 0 && std::min(M.nsplit_max, kCtxBuckets[M.ctx_bucket]) <= kF32OneSplits;
}

int model_map_pages(Model& M, int keep, int upto, int* first_changed, int* n_changed, char* err) {
    *first_changed = 0;
    *n_changed = 0;
    if (upto > M.max_seq) PSD_FAIL(PSD_ESHAPE, err, "%s: position %d exceeds max_seq %d", M.tag, upto, M.max_seq);
    const int need = (upto + kPage - 1) / kPage, keep_pages = (keep + kPage - 1) / kPage;
    int lo = M.n_pages, hi = 0;
    // rollback: blocks wholly beyond the kept prefix go back to the free list (unless needed again right away)
    for (int b = M.pages_mapped - 1; b >= std::max(keep_pages, need); --b) {
        M.free_pages.push_back(M.h_page_table[b]);
        M.h_page_table[b] = -1;
        M.pages_mapped = b;
        lo = std::min(lo, b); hi = std::max(hi, b + 1);
    }
    for (int b = M.pages_mapped; b < need; ++b) {
        if (M.free_pages.empty()) PSD_FAIL(PSD_ENOMEM, err, "%s: out of KV pages", M.tag);
        M.h_page_table[b] = M.free_pages.back();
        M.free_pages.pop_back();
        M.pages_mapped = b + 1;
        lo = std::min(lo, b); hi = std::max(hi, b + 1);
    }
    if (hi > lo) { *first_changed = lo; *n_changed = hi - lo; }
    return PSD_OK;
}

// ---- forward ----------------------------------------------------------------------------------------
namespace {
struct Launch {
    Model& M;
    hipStream_t s;
    Profiler* prof;
    int wcls;  // launch class: one of kNarrowClasses, or a multiple of 128
    char name[48];
    void begin(const char* family, double bytes) {
        if (!prof || !prof->on) return;
        snprintf(name, sizeof(name), "%s %s w<=%d", family, M.tag, wcls);
        prof->begin(s, prof->row_of(name), bytes);
    }
    void end() {
        if (prof && prof->on) prof->end(s);
    }
};
}  // namespace

// fp32 models: five launches per layer
template <int EPI>
static void launch_proj_f32(Launch& L, const char* family, F32Args a) {
    const int npairs = (a.N + 1) / 2;
    a.desc = L.M.desc;
    L.begin(family, (double)a.N * a.K * 4);
    // Lanes per row pair: 64 where K feeds them (more workgroups and fewer serial steps), 16 for K up to 256; K decides the
    // summation order, the pass width does not.  Columns: a workgroup takes up to 4, the pass's others go to workgroups of
    // their own, which read the weights again; where that is more than L2 likes (over 2 M weights) 8 columns at a time
    // and one workgroup after the other.  (Tiny target, 9 tokens: 7.5 us with 8 columns in turn, 4.5 us side by side.)
    const bool big = (size_t)a.N * a.K > ((size_t)2 << 20);
    const dim3 grid16((npairs + 15) / 16, big || L.wcls <= 4 ? 1 : (L.wcls + 3) / 4), grid64((npairs + 3) / 4, grid16.y);
#define PSD_F32(LP_, NC_) proj_f32<EPI, LP_, NC_><<<LP_ == 16 ? grid16 : grid64, 256, 0, L.s>>>(a)
    if (a.K > 256) {
        if (L.wcls == 1) PSD_F32(64, 1); else if (L.wcls <= 4 || !big) PSD_F32(64, 4); else PSD_F32(64, 8);
    } else {
        if (L.wcls == 1) PSD_F32(16, 1); else if (L.wcls <= 4 || !big) PSD_F32(16, 4); else PSD_F32(16, 8);
    }
#undef PSD_F32
    L.end();
}

int model_near_last_tag(Model& M, int passes, hipStream_t stream, char* err) {
    if (!M.one_launch) return PSD_OK;
    PSD_HIP(hipMemsetD32Async(M.x + (size_t)kMaxW * M.d, 1, (size_t)(kCols - kMaxW) * M.d, stream), err);
    PSD_HIP(hipMemsetD32Async(M.qkv + (size_t)kMaxW * M.nqkv, 1, (size_t)(kCols - kMaxW) * M.nqkv, stream), err);
    M.tag_last = 0xffffffffu - (uint32_t)(passes * 5 * M.L);
    return PSD_OK;
}

int model_stamp(Model& M, PassDesc& d, int passes, hipStream_t stream, char* err) {
    if (!M.room) return PSD_OK;
    d.tag_step = 5 * M.L;
    const uint32_t span = (uint32_t)passes * d.tag_step;
    if (M.tag_last > 0xffffffffu - span) {   // used up: the slots forget them
        PSD_HIP(hipMemsetAsync(M.x + (size_t)kMaxW * M.d, 0, (size_t)(kCols - kMaxW) * M.d * sizeof(float), stream), err);
        PSD_HIP(hipMemsetAsync(M.qkv + (size_t)kMaxW * M.nqkv, 0, (size_t)(kCols - kMaxW) * M.nqkv * sizeof(float), stream), err);
        M.tag_last = 0;
    }
    d.tag0 = M.tag_last;
    M.tag_last += span;
    return PSD_OK;
}

template <int HD>
static void launch_pass_f32(Launch& L, float* logits) {
    Model& M = L.M;
    const int d = M.d, F = M.F;
    F32Pass a{};
    a.embed = (const float*)M.embed; a.final_norm = M.final_norm;
    a.w = M.layers[0];
    a.layer_bytes = M.L > 1 ? (const char*)M.layers[1].wqkv - (const char*)M.layers[0].wqkv : 0;   // the same for all: model_carve
    a.desc = M.desc; a.rope = M.rope; a.kv = (float*)M.kv; a.page_table = M.page_table; a.n_pages = M.n_pages;
    a.X = (slot_t*)(M.x + (size_t)kMaxW * d);
    a.Q = a.X + (size_t)kMaxW * d;
    a.A = a.Q + (size_t)kMaxW * d;
    a.G = a.A + (size_t)kMaxW * d;
    a.KVn = (slot_t*)(M.qkv + (size_t)kMaxW * M.nqkv);
    a.logits = logits;
    a.gone = M.gone;
    a.wait_ticks = wait_ticks();
    a.eps = M.eps;
    a.inv_d = 1.f / (float)d;
    a.L = M.L; a.d = d; a.H = M.H; a.KV = M.KV; a.F = F; a.V = M.V;
    a.hd_log = HD == 16 ? 4 : HD == 32 ? 5 : HD == 64 ? 6 : 7;
    f32_pass_parts(M, a.nux);
    const int grid = std::max(1, f32_pass_grid(M, L.wcls) - (M.short_passes ? 1 : 0));
    L.begin("pass_f32", (double)M.weight_bytes);
    if (L.wcls == 1) pass_f32<HD, 1><<<grid, 256, 0, L.s>>>(a);
    else if (L.wcls <= 16) pass_f32<HD, 4><<<grid, 256, 0, L.s>>>(a);
    else pass_f32<HD, 8><<<grid, 256, 0, L.s>>>(a);
    L.end();
}

static int forward_f32(Model& M, int wmax, float* logits, Launch& L) {
    hipStream_t stream = L.s;
    const int d = M.d, F = M.F, H = M.H, KV = M.KV, hd = M.hd;
    if (model_one_launch(M, wmax, logits)) {
        if (hd == 16) launch_pass_f32<16>(L, logits);
        else if (hd == 32) launch_pass_f32<32>(L, logits);
        else if (hd == 64) launch_pass_f32<64>(L, logits);
        else launch_pass_f32<128>(L, logits);
        return PSD_OK;
    }
    const double act = (double)wmax * d * 4;
    float* attn = (float*)M.xb;
    L.begin("embed", act);
    embed_rows<<<wmax, 256, 0, stream>>>((const float*)M.embed, M.desc, M.x, d, M.V);
    L.end();
    const int nsplit = std::min(M.nsplit_max, kCtxBuckets[M.ctx_bucket]);   // key ranges this launch covers
    F32Args base{};
    base.eps = M.eps;
    base.rope = M.rope; base.kv = (float*)M.kv; base.page_table = M.page_table;
    base.L = M.L; base.H = H; base.KV = KV; base.hd = hd;
    auto args = [&](const void* W, const float* X, const float* gain, float* Y, int N, int K, int ldy) {
        F32Args a = base;
        a.W = (const float*)W; a.X = X; a.gain = gain; a.Y = Y; a.N = N; a.K = K; a.ldy = ldy;
        return a;
    };
    for (int l = 0; l < M.L; ++l) {
        const LayerW& w = M.layers[l];
        base.layer = l;
        launch_proj_f32<F32_QKV>(L, "gemm_qkv", args(w.wqkv, M.x, w.attn_norm, M.qkv, M.nqkv, d, M.nqkv));
        L.begin("attn", (double)std::min(M.max_seq, M.len + wmax) * KV * hd * 2 * 4 + (double)wmax * H * hd * 4 * 2);
        // short contexts: one launch; longer ones spread the key ranges over workgroups and merge in a second
        if (nsplit <= kF32OneSplits) {
            attn_one_f32<<<dim3(H, wmax), 256, 0, stream>>>(M.qkv, M.desc, (const float*)M.kv, M.page_table, M.n_pages, attn, l, M.L, H, KV, hd, M.nqkv);
        } else {
            attn_partial<<<dim3(H, nsplit), 256, attn_lds_bytes(hd), stream>>>(M.qkv, M.desc, (const float*)M.kv, M.page_table, M.attn_part, l, M.L, H, KV, hd, M.nqkv);
            attn_combine_f32<<<dim3(wmax, H), hd, 0, stream>>>(M.attn_part, M.desc, attn, H, hd);
        }
        L.end();
        launch_proj_f32<F32_RESID>(L, "gemm_o", args(w.wo, attn, nullptr, M.x, d, H * hd, d));
        launch_proj_f32<F32_SWIGLU>(L, "gemm_gate_up", args(w.wgu, M.x, w.ffn_norm, M.gu, 2 * F, d, F));
        launch_proj_f32<F32_RESID>(L, "gemm_down", args(w.wd, M.gu, nullptr, M.x, d, F, d));
    }
    if (logits) launch_proj_f32<F32_LOGITS>(L, "gemm_lm_head", args(M.embed, M.x, M.final_norm, logits, M.V, d, M.V));
    return PSD_OK;
}

// Projection of a prompt-ingestion pass.  NW: the K split of the narrow kernels.
template <int NW, int EPI, int RTW, int TCW, int KB>
static void launch_panel_as(Launch& L, GemmArgs a, int tiles) {
    Model& M = L.M;
    const int ncg = L.wcls / (16 * TCW), units = (tiles + 8 * RTW - 1) / (8 * RTW) * (kGrouped<EPI> ? 4 : 1);
    if constexpr (kGrouped<EPI>) {
        // as many column groups per launch as the scratch has room for: all of them in a pool of the full size
        const PanelScratch& sc = EPI == EPI_QKV ? M.panel_qkv : M.panel_res;
        const int room = (int)std::min((size_t)ncg, sc.bytes / panel_group_bytes(tiles, TCW)), turns = (ncg + room - 1) / room;
        int n = (ncg + turns - 1) / turns;
        f32x4* part = (f32x4*)((char*)sc.mem + (sc.bytes - n * panel_group_bytes(tiles, TCW)) / 256 * 256);   // at its end
        for (int cg0 = 0; cg0 < ncg; cg0 += n) {
            n = std::min(n, ncg - cg0);
            gemm_panel<NW, EPI, RTW, TCW, KB><<<(units + 7) / 8 * 8 * n, 512, 0, L.s>>>(a, tiles, n, cg0, part);
            panel_finish<NW, EPI><<<dim3((tiles + 7) / 8, n * TCW), 256, 0, L.s>>>(a, tiles, cg0 * TCW, part);
        }
    } else {
        a.rs_in = M.panel_rs;
        panel_scale<NW><<<L.wcls / 16, 256, 0, L.s>>>(a, M.panel_rs);
        gemm_panel<NW, EPI, RTW, TCW, KB><<<(units + 7) / 8 * 8 * ncg, 512, 0, L.s>>>(a, tiles, ncg, 0, nullptr);
    }
}
template <int NW, int EPI>
static void launch_panel(Launch& L, const GemmArgs& a, int tiles) {
    // 256 x 128 outputs per workgroup move the fewest bytes per MFMA; smaller tiles where those would leave CUs idle.  us of a
    // projection with 256 x 128 / 256 x 64 / 128 x 64 tiles, over the number `full` of the first:
    //   160: 36.6 / 43.8 / 43.1    144: 30.0 / 32.5 / 33.7, 59.4 / 65.4 / 69.8    128: 58.2 / 41.9 / 50.3, 38.0 / 30.5 / 36.3
    //   112: 102 / 82 / 95          96: 38.3 / 32.5 / 35.8, 54.6 / 38.6 / 48.4      64: 55.8 / 38.4 / 31.0, 35.0 / 26.9 / 22.8
    const int full = (tiles + 15) / 16 * (kGrouped<EPI> ? 4 : 1) * (L.wcls / 128);
    // KB: a small tile's step is few MFMAs (64 x 64 outputs per SIMD: 128 cycles), so two of them share a barrier; where more
    // smallest tiles than CUs are launched (`full` from 64 to 96) two workgroups share a CU instead, which the second step's
    // registers would prevent (qualifier shape, 100 tokens: o + down 21.0 -> 18.6 us, gate/up 40.5 -> 36.8; q/k/v with 320 workgroups
    // 19.6 -> 21.2).  There the 256 x 64 tiles are no clear choice either: one step / two steps / those, 30.7 / 31.9 / 28.0 at 80,
    // 20.3 / 22.7 / 21.3 at 72
    // The scratch always has room for one group of 64 columns: q/k/v, 1024 nqkv <= 3072 d bytes of 2048 (max(d, F) +
    // nsplit_max (d + 2 H)); o and down, 1024 d of 2048 nsplit_max (d + 2 H).
    const size_t scratch = EPI == EPI_QKV ? L.M.panel_qkv.bytes : EPI == EPI_RESID ? L.M.panel_res.bytes : SIZE_MAX;
    if (full >= 144 && panel_group_bytes(tiles, 8) <= scratch) launch_panel_as<NW, EPI, 2, 8, 1>(L, a, tiles);
    else if (full >= 96) launch_panel_as<NW, EPI, 2, 4, 2>(L, a, tiles);
    else if ((tiles + 7) / 8 * (kGrouped<EPI> ? 4 : 1) * (L.wcls / 64) <= 256) launch_panel_as<NW, EPI, 1, 4, 2>(L, a, tiles);
    else launch_panel_as<NW, EPI, 1, 4, 1>(L, a, tiles);
}

// bf16 models: five or six launches per layer (q/k/v projection, attention, merge, o, gate/up, down)
template <int EPI>
static void launch_gemm_bf16(Launch& L, const char* family, GemmArgs a) {
    Model& M = L.M;
    const int tiles = round16(a.N) / 16;
    a.desc = M.desc;
    a.wcap = L.wcls;
    L.begin(family, (double)a.N * a.KS * 32 * 2);
    // Waves per workgroup (the K split, hence the summation order) follow from the number of row tiles only, never
    // from the pass width: a token's result must not depend on the width of the pass that computes it.  Row tiles
    // per wave do not change the arithmetic and are picked per width class.
#define PSD_GEMM(NT_, NW_, RT_) gemm_bf16<NT_, NW_, RT_, EPI><<<tiles / RT_, 64 * NW_, 0, L.s>>>(a)
    if (L.wcls > kMaxW) {   // prompt ingestion
        if constexpr (EPI != EPI_LOGITS) {
            if (tiles <= 256) launch_panel<16, EPI>(L, a, tiles);
            else launch_panel<8, EPI>(L, a, tiles);
        }
    } else {
        const bool wide = L.wcls > 16;
        bool done = false;
        if constexpr (EPI == EPI_SWIGLU) {   // shapes measured one by one; only the gate/up kernels have such variants
            if (tiles % 7 == 0 && tiles / 7 >= 256) {
                // one workgroup per CU for the target's gate/up projection (1792 tiles): 44 us against 47
                if (wide) PSD_GEMM(2, 8, 7); else PSD_GEMM(1, 8, 7);
                done = true;
            } else if (!wide && tiles == 1024 && a.KS >= 96) {
                PSD_GEMM(1, 8, 4);   // likewise the qualifier's (1024 tiles, K 3072): 20.2 us against 21.1; not for K 2048
                done = true;
            }
        }
        // passes of at most 4 tokens: the operand of a wave's whole K range is staged in LDS, 512 bytes per K step and wave
        const int nw = tiles <= 256 ? 16 : 8;
        const int lb_slots = 64 * (((a.KS + nw - 1) / nw + 1) / 2);
        const size_t lb_bytes = (size_t)nw * lb_slots * sizeof(u32x4);
        // Measured on the draft's shapes: long K ranges gain (down projection, 16 steps per wave: 14.3 -> 13.3 us) and
        // so does the LM head (89.6 -> 86.4 us); ranges of 4 or 8 steps lose 0.2 us to the wait for the staged blocks
        constexpr bool kHasLb = EPI == EPI_RESID || EPI == EPI_LOGITS;
        const bool lb = kHasLb && L.wcls <= 4 && lb_bytes <= kLbMaxBytes && (EPI == EPI_LOGITS || (a.KS + nw - 1) / nw >= 12);
        a.lb_slots = lb_slots;
#define PSD_GEMM_LB(NW_, RT_)                                                                                      \
    do {                                                                                                           \
        if constexpr (kHasLb) gemm_bf16<1, NW_, RT_, EPI, true><<<tiles / RT_, 64 * NW_, lb_bytes, L.s>>>(a);   \
    } while (0)
        // one column tile, at most 7 K steps per wave: the variant that asks for a wave's whole range at once
        const bool short_k = !wide && !lb && (a.KS + 15) / 16 <= 7 && (EPI == EPI_RESID || EPI == EPI_QKV);
        if (done) {
        } else if (tiles <= 256) {
            if (lb) PSD_GEMM_LB(16, 1);
            else if (wide) PSD_GEMM(2, 16, 1);
            else if (short_k) {
                if constexpr (EPI == EPI_RESID || EPI == EPI_QKV) gemm_bf16<1, 16, 1, EPI, false, true><<<tiles, 64 * 16, 0, L.s>>>(a);
            }
            else PSD_GEMM(1, 16, 1);
        } else if (tiles % 2 == 0) {
            if (lb) PSD_GEMM_LB(8, 2); else if (wide) PSD_GEMM(2, 8, 2); else PSD_GEMM(1, 8, 2);
        } else {
            if (lb) PSD_GEMM_LB(8, 1); else if (wide) PSD_GEMM(2, 8, 1); else PSD_GEMM(1, 8, 1);
        }
#undef PSD_GEMM_LB
    }
#undef PSD_GEMM
    L.end();
}

// Wide passes: one sweep per query tile (attn_wide, attn_pair) where there are enough tiles to fill the device or few key ranges to
// walk; few tiles over a long context keep a workgroup per key range and the merge kernel.  The most ranges for which a pass of
// `tiles` query tiles sweeps.  us a layer, ranges + merge / sweep, over the key ranges that the pass's last position has:
//   head dim 128 (attn_wide: 13 us and 5 for every range after the first)
//     64 tiles   1: 23 / 13    2: 23 / 19    3: 23 / 23    4: 23 / 28      384 tiles   5: 39 / 34    6: 44 / 39    7: 46 / 43    8: 46 / 48
//    256 tiles   3: 29 / 25    4: 29 / 30    5: 30 / 34    8: 32 / 50      512 tiles  14: 91 / 82   25: 137 / 138    768 tiles  27: 205 / 145
//   head dim 64 | 32 (attn_pair: 12 us and 2.3 for every range after the second)
//    128 tiles   4: 18 / 17 | 16 / 13      5: 18 / 20 | 16 / 15      6: 18 / 21 | 16 / 16      160 tiles   5: 21 / 19    6: 21 / 21    9: 23 / 28
//    192 tiles   5: 21 / 20                6: 21 / 22                256 tiles   5: 21 / 20 | 17 / 15    6: 22 / 21 | 18 / 16    7: 22 / 24 | 18 / 18
//    320 tiles  10: 35 / 30               14: 40 / 40               20: 51 / 53
//    384 tiles   7: 26 / 24 | 21 / 18     15: 45 / 42 | 36 / 31     21: 55 / 56 | 42 / 41     28: 66 / 72 | 48 / 52
//    480 tiles  28: 81 / 71               39: 97 / 97      512 tiles  29: 85 / 74 | 58 / 54    40: 105 / 99 | 67 / 71    67: 166 / 162 | 95 / 114
//    640 tiles  67: 200 / 160            768 tiles  66: 243 / 162
static int sweep_ranges(int hd, int tiles) {
    constexpr int all = 1 << 30;
    if (hd > 64) return tiles >= 512 ? all : tiles >= 384 ? 6 : tiles >= 256 ? 4 : 3;
    if (tiles >= (hd == 64 ? 512 : 640)) return all;
    return tiles >= 512 ? 39 : tiles >= 448 ? 32 : tiles >= 384 ? 19 : tiles >= 320 ? 13 : tiles >= 256 ? 6 : tiles >= 160 ? 5 : 4;
}

static int forward_bf16(Model& M, int wmax, float* logits, Launch& L) {
    hipStream_t stream = L.s;
    const int d = M.d, F = M.F, H = M.H, KV = M.KV, hd = M.hd, G = H / KV;
    const double act = (double)wmax * d * 4;
    const float inv_d = 1.0f / (float)d;
    const bool c128 = wmax > 32;   // prompt ingestion: operands with 32 column tiles in their own buffers
    void* xb = c128 ? M.xbw : M.xb;
    void* xb2 = c128 ? M.xbw2 : M.xb2;
    float* ss = c128 ? M.ssw : M.ss;
    L.begin("embed", act);
    const dim3 egrid(d / 16, (wmax + 15) / 16);
    if (c128) embed_pack<kWideCT><<<egrid, 64, 0, stream>>>((const uint16_t*)M.embed, M.desc, M.x, xb, M.layers[0].attn_norm, ss, d, M.V);
    else embed_pack<2><<<egrid, 64, 0, stream>>>((const uint16_t*)M.embed, M.desc, M.x, xb, M.layers[0].attn_norm, ss, d, M.V);
    L.end();
    // key ranges this launch covers: the bucket of the pass's last position (the caller's bound), never beyond the cache
    const int nsplit = std::min(M.nsplit_max, kCtxBuckets[M.ctx_bucket]);
    // prompt-ingestion passes: four query tiles share one load of the keys and values.  Narrow passes take one tile per
    // workgroup at every context length: since the key and value planes are tiled their loads are cheap enough that more
    // workgroups beat fewer loads (target pass at 4.6 K tokens of context: 3.99 ms with one tile per workgroup, 4.06 ms with
    // the pass's three tiles sharing one load; with the untiled planes it was the other way round beyond 16 key ranges)
    const int qt_per_wg = wmax > kMaxW ? 4 : 1;
    const int qt_max = ((wmax * G + 15) / 16 + qt_per_wg - 1) / qt_per_wg;
    // narrow passes of small models: the o projection merges the attention split partials itself (one launch less).
    // Every workgroup of it repeats the merge, so past a dozen key ranges the separate merge kernel is cheaper
    // (draft o projection at 36 ranges: 19.8 us against 4.2 + 6.5 us); both routes give the same bits.
    // algorithmic bytes of one layer's attention: K and V of every key the pass can see, as bf16 (the cache holds a hi and a
    // lo plane per value, so the kernels move twice that), plus the queries in and the outputs back
    const double kv_bytes = (double)std::min(M.max_seq, M.len + wmax) * KV * hd * 2 * 2 + (double)wmax * H * hd * 4 * 2;
    const int tiles = KV * ((wmax * G + 15) / 16), ranges = (std::min(M.max_seq, M.len + wmax) + kAttnSplit - 1) / kAttnSplit;
    const bool sweep = c128 && ranges <= sweep_ranges(hd, tiles);
    // head dims up to 64 sweep with two waves per tile where there is a second range for the second wave (attn_wide / attn_pair, us a
    // launch of 64 tiles: one range 7.7-8.3 / 8.3-8.9, two 11.0-11.6 / 10.8-11.3, three 14.2-14.5 / 13.4-13.6)
    const bool fold_merge = wmax <= 4 && d <= 2048 && d / 16 <= 256 && H * hd == d && nsplit <= kFoldSplits;
    GemmArgs base{};
    base.ss_in = ss; base.ss_tiles = d / 16; base.inv_d = inv_d; base.eps = M.eps;
    base.rope = M.rope; base.kv = (uint16_t*)M.kv; base.page_table = M.page_table;
    base.L = M.L; base.H = H; base.KV = KV; base.hd = hd;
    for (int l = 0; l < M.L; ++l) {
        const LayerW& w = M.layers[l];
        const float* next_gain = l + 1 < M.L ? M.layers[l + 1].attn_norm : M.final_norm;
        GemmArgs a = base;
        a.Wt = (const u32x4*)w.wqkv; a.XB = (const u32x4*)xb; a.N = M.nqkv; a.KS = d / 32;
        a.Y = M.qkv; a.ldy = M.nqkv; a.layer = l;
        launch_gemm_bf16<EPI_QKV>(L, "gemm_qkv", a);
        L.begin("attn", kv_bytes);
        const dim3 agrid(KV, nsplit, qt_max);
        const uint16_t* kvp = (const uint16_t*)M.kv;
#define PSD_ATTN(HD_)                                                                                                            \
    do {                                                                                                                         \
        if (sweep && HD_ <= 64 && ranges >= 2) attn_pair<HD_ <= 64 ? HD_ : 64><<<((wmax * G + 63) / 64) * KV, 512, kAttnPairLds<HD_>, stream>>>(M.qkv, M.desc, kvp, M.page_table, M.n_pages, xb2, l, M.L, H, KV, M.nqkv); \
        else if (sweep) attn_wide<HD_><<<((wmax * G + 63) / 64) * KV, 256, kAttnWideLds<HD_>, stream>>>(M.qkv, M.desc, kvp, M.page_table, M.n_pages, xb2, l, M.L, H, KV, M.nqkv); \
        else attn_mfma<HD_><<<agrid, 256, 0, stream>>>(M.qkv, M.desc, kvp, M.page_table, M.n_pages, M.attn_part, l, M.L, H, KV, M.nqkv, qt_per_wg); \
    } while (0)
        if (hd == 128) PSD_ATTN(128); else if (hd == 64) PSD_ATTN(64); else PSD_ATTN(32);
#undef PSD_ATTN
        L.end();
        a = base;
        a.Wt = (const u32x4*)w.wo; a.XB = (const u32x4*)xb2; a.N = d; a.KS = (H * hd) / 32;
        a.Y = M.x; a.ldy = d; a.xb_out = xb; a.gain_out = w.ffn_norm; a.ss_out = ss;
        if (fold_merge) {
            a.desc = M.desc; a.wcap = 4;
            L.begin("gemm_o", (double)d * d * 2);
            gemm_o_narrow<<<d / 16, 1024, 0, stream>>>(a, M.attn_part);
            L.end();
        } else {
            if (!sweep) {
                L.begin("attn_combine", act);
                // more than eight key ranges: the form that fetches a row's partials in one round (its LDS need grows with the
                // ranges; the dependent-rounds form takes over where that no longer fits)
                const size_t cmb_lds = ((size_t)nsplit * (hd + 4) + 1) * sizeof(float);
                if (nsplit > 8 && cmb_lds <= 64 * 1024) {
                    if (c128) attn_combine_long<kWideCT><<<dim3(wmax, H), 256, cmb_lds, stream>>>(M.attn_part, M.desc, xb2, H, hd, nsplit);
                    else attn_combine_long<2><<<dim3(wmax, H), 256, cmb_lds, stream>>>(M.attn_part, M.desc, xb2, H, hd, nsplit);
                } else if (c128) {
                    attn_combine_bf16<kWideCT><<<dim3(wmax, H), hd, 0, stream>>>(M.attn_part, M.desc, xb2, H, hd);
                } else {
                    attn_combine_bf16<2><<<dim3(wmax, H), hd, 0, stream>>>(M.attn_part, M.desc, xb2, H, hd);
                }
                L.end();
            }
            launch_gemm_bf16<EPI_RESID>(L, "gemm_o", a);
        }
        a = base;
        a.Wt = (const u32x4*)w.wgu; a.XB = (const u32x4*)xb; a.N = 2 * F; a.KS = d / 32; a.xb_out = xb2;
        launch_gemm_bf16<EPI_SWIGLU>(L, "gemm_gate_up", a);
        a = base;
        a.Wt = (const u32x4*)w.wd; a.XB = (const u32x4*)xb2; a.N = d; a.KS = F / 32;
        a.Y = M.x; a.ldy = d; a.xb_out = xb; a.gain_out = next_gain; a.ss_out = ss;
        launch_gemm_bf16<EPI_RESID>(L, "gemm_down", a);
    }
    if (logits) {
        GemmArgs a = base;
        a.Wt = (const u32x4*)M.embed; a.XB = (const u32x4*)xb; a.N = M.V; a.KS = d / 32; a.Y = logits; a.ldy = M.V;
        launch_gemm_bf16<EPI_LOGITS>(L, "gemm_lm_head", a);
    }
    return PSD_OK;
}

// what an event pair measures around a kernel that does nothing: the share of every profiled interval that is not kernel time
__global__ void empty_kernel() {}

int model_forward(Model& M, int wmax, float* logits, hipStream_t stream, Profiler* prof, char* err) {
    const bool ingest = wmax > kMaxW;
    if (ingest ? (wmax % 128 != 0 || wmax > M.ingest_max) : (narrow_class_index(wmax) < 0 || kNarrowClasses[narrow_class_index(wmax)] != wmax))
        PSD_FAIL(PSD_EINVAL, err, "forward: width class %d", wmax);
    if (ingest && (M.dtype != PSD_BF16 || logits)) PSD_FAIL(PSD_EINVAL, err, "forward: passes wider than %d tokens are for bf16 prompt ingestion only", kMaxW);
    Launch L{M, stream, prof, wmax, {0}};
    int rc = M.dtype == PSD_BF16 ? forward_bf16(M, wmax, logits, L) : forward_f32(M, wmax, logits, L);
    if (rc != PSD_OK) return rc;
    if (prof && prof->on) {
        prof->begin(stream, prof->row_of("empty kernel (event pair only)"), 0.0);
        empty_kernel<<<1, 64, 0, stream>>>();
        prof->end(stream);
    }
    PSD_HIP(hipGetLastError(), err);
    return PSD_OK;
}

}  // namespace psd
