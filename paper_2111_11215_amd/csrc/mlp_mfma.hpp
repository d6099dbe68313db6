// Colour network of the fine stage (paper Eq. fine_queries: two ReLU layers
// of 128 and a sigmoid RGB head) on CDNA4 matrix cores: the operand packing
// of both forms and the bfloat16 form (the float32 one is in mlp_split.hpp).
//
// Layout.  A 32x32 accumulator tile of v_mfma_f32_32x32x16_bf16 holds, in
// lane l and register r, row 8*(r/4) + 4*(l/32) + (r%4) and column l%32.
// Activations are kept transposed ("feature rows, sample columns").  In the
// forward a wave owns 32 samples (one per lane column) and each lane holds 16
// features per 32-feature tile; the next layer consumes those registers
// directly as its B operand; the K order this implies is folded into the
// packed weights (phi16 below), so a layer chain never leaves registers.  In
// the adjoint the weights stay and a block's samples pass: a wave owns 32
// features of every layer, and the activations go between the waves as
// [sample][feature] rows in LDS in the same K order.  Weight gradients need the
// sample index as the contraction dimension: they read those rows through the
// LDS transpose load, and each wave accumulates its own slice of dW in
// registers across the whole persistent loop; per-workgroup partials are
// summed afterwards.
#pragma once

#include "common.hpp"

namespace {

constexpr int kH = 128;                 // hidden width
constexpr int kC = 12;                  // feature channels
constexpr int kPE = 27;                 // PE(d) with 4 frequencies
constexpr int kIn = kC + kPE;           // first-layer input width
// Flat gradient layout of the colour network: w1, b1, w2, b2, w3, b3.
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kH * kIn;
constexpr int kOffW2 = kOffB1 + kH;
constexpr int kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH;
constexpr int kOffB3 = kOffW3 + 3 * kH;
constexpr int kMlpParams = kOffB3 + 3;
constexpr int kPStride = (kMlpParams + 63) / 64 * 64;
constexpr int kW2PackF32 = 4 * 16 * 64 * 4;
constexpr int kW2PackBF16 = 4 * 8 * 64 * 8;
constexpr int kW3PackBF16 = 8 * 64 * 8;    // layer 3 as a 32-row tile (rows >= 3 zero)
constexpr int kW3TPackBF16 = 4 * 64 * 8;   // W3^T, one K step (k >= 3 zero)
constexpr int kW1TPackBF16 = 8 * 64 * 8;   // W1[:, :12]^T as a 32-row tile (rows >= 12 zero)

// Layout of the network whose input also carries the encoded query
// position (Eq. fine_queries with k_x = KX frequencies): input [feat (12),
// PE_KX(u) (3 + 6 KX), PE(d) (27)], u the position in box coordinates.  The
// per-sample part of the first layer is [feat, PE_KX(u)] (kS values); the
// view part is evaluated once per ray as before.  KX = 0 is the 39-input
// network above.
template <int KX>
struct NetLayout {
    static constexpr int kXPE = KX ? 3 + 6 * KX : 0;
    static constexpr int kS = kC + kXPE;              // per-sample first-layer inputs
    static constexpr int kIn = kS + kPE;              // first-layer inputs
    static constexpr int kOffW1 = 0;
    static constexpr int kOffB1 = kOffW1 + kH * kIn;
    static constexpr int kOffW2 = kOffB1 + kH;
    static constexpr int kOffB2 = kOffW2 + kH * kH;
    static constexpr int kOffW3 = kOffB2 + kH;
    static constexpr int kOffB3 = kOffW3 + 3 * kH;
    static constexpr int kParams = kOffB3 + 3;
    static constexpr int kPStride = (kParams + 63) / 64 * 64;
    static constexpr int kQ1 = ((kS + 1) / 2 + 3) / 4;   // float4 groups of K = 2 layer-1 steps
    static constexpr int kS1 = (kS + 15) / 16;            // K = 16 layer-1 steps (bfloat16)
    static constexpr int kXT = (kIn + 1 + 31) / 32;      // 32-column tiles of x' = [input, 1]
};
static_assert(NetLayout<0>::kIn == kIn && NetLayout<0>::kParams == kMlpParams && NetLayout<0>::kQ1 == 2 &&
                  NetLayout<0>::kXT == 2,
              "the 39-input layout");
constexpr int kMaxKX = 5;                                          // the paper's k_x
constexpr int kW1PackF32Max = 4 * NetLayout<kMaxKX>::kQ1 * 64 * 4;   // packed W1 of either layout
constexpr int kW1PackBF16Max = 4 * NetLayout<kMaxKX>::kS1 * 64 * 8;
constexpr int kPStrideMax = NetLayout<kMaxKX>::kPStride;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Hides a uniform pointer's value from the optimiser.  Used once per
// persistent-loop iteration so weight loads are issued where they are
// consumed instead of being hoisted out of the loop into hundreds of
// registers.
// The pointer is passed through as a global-memory one, so that the loads
// through it stay global loads (a generic pointer would make them flat
// loads, which every LDS wait then has to include).
template <typename T>
__device__ __forceinline__ T* opaque(T* p) {
    typedef __attribute__((address_space(1))) T GT;
    GT* g = (GT*)p;
    asm volatile("" : "+s"(g));
    return (T*)g;
}

// Row within a 32-row accumulator tile of register r in lane half h.
__host__ __device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }
// Feature at step st (0..63), half h of the plain float32 chain's input order.
__host__ __device__ __forceinline__ int phi32(int st, int h) { return 32 * (st >> 4) + acc_row(st & 15, h); }
// Feature consumed at bfloat16 chain step st (0..7), element i (0..7), half h.
__host__ __device__ __forceinline__ int phi16(int st, int i, int h) {
    return 32 * (st >> 1) + acc_row(8 * (st & 1) + i, h);
}

__device__ __forceinline__ uint16_t f2bf(float f) {   // round to nearest even
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) return static_cast<uint16_t>((u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u));
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// The exact bfloat16 planes of a float32 value: hi = bf16(w), mid =
// bf16(w - hi), lo = w - hi - mid (both differences are exact, and lo fits
// bfloat16's 8 bits).  A finite w that rounds to infinity has the largest
// finite bfloat16 as hi.  The bfloat16 arithmetic uses plane 0 only.
__device__ __forceinline__ void store_planes(uint16_t* dst, int i, int stride, float w, int planes) {
    for (int p = 0; p < planes; ++p) {
        uint16_t b = f2bf(w);
        if (planes > 1 && (b & 0x7FFFu) == 0x7F80u && fabsf(w) < INFINITY) b -= 1;
        dst[p * stride + i] = b;
        w -= bf2f(b);
    }
}

struct PackArgs {
    const float* w1;
    const float* w2;
    const float* w3;
    const float* b2;
    float* b2p;   // b2 with kDeadBias for dead units (float32 form)
    uint16_t* w3pb;
    uint16_t* w3tpb;
    uint16_t* w1tpb;
    float* w1p;
    float* w2p;
    uint16_t* w1pb;
    uint16_t* w2pb;
    uint16_t* w2tpb;
    int bf16;
    int w1_in;   // first-layer input width (row stride of W1)
    int w1_ns;   // per-sample first-layer inputs (packed into w1p)
    int w1_q;    // float4 groups of w1p per output tile
    int w1_s1;   // K = 16 steps of w1pb per output tile
};

// Pack W1 (feature columns) and W2 / W2^T into matrix-core operand order.
// Operand packing of the network weights, one value per thread `gid` of
// kPackThreads (a device function so that it can share a launch).
constexpr int kPackThreads = kW2PackF32;

// The float32 form gives a unit without weights and bias this one: ReLU turns
// either into 0, but a pre-activation of exactly 0 in every sample would count
// as one near zero, whose branch is worth a second look (see add_live).
constexpr float kDeadBias = -1.0f;

__device__ __forceinline__ void pack_weights(const PackArgs& a, int gid) {
    const int planes = a.bf16 ? 1 : 3;
    if (!a.bf16 && gid < kH * 64) {   // a wavefront per unit of layer 2
        const int i = gid >> 6, lane = gid & 63;
        const bool any = __any(a.w2[i * kH + lane] != 0.0f || a.w2[i * kH + 64 + lane] != 0.0f);
        if (lane == 0) a.b2p[i] = any || a.b2[i] != 0.0f ? a.b2[i] : kDeadBias;
    }
    if (gid < kW2PackF32) {
        // float32: index ((mt*16 + q)*64 + lane)*4 + u, step st = 4q + u
        const int u = gid & 3, lane = (gid >> 2) & 63, q = (gid >> 8) & 15, mt = gid >> 12;
        const int st = 4 * q + u, m = lane & 31, h = lane >> 5;
        if (!a.bf16) a.w2p[gid] = a.w2[(32 * mt + m) * kH + phi32(st, h)];
        {
            // bfloat16 planes: index ((mt*8 + st)*64 + lane)*8 + i
            const int i = gid & 7, lane2 = (gid >> 3) & 63, st2 = (gid >> 9) & 7, mt2 = gid >> 12;
            const int m2 = lane2 & 31, h2 = lane2 >> 5;
            const int row2 = 32 * mt2 + m2, k2 = phi16(st2, i, h2);
            store_planes(a.w2pb, gid, kW2PackBF16, a.w2[row2 * kH + k2], planes);
            store_planes(a.w2tpb, gid, kW2PackBF16, a.w2[k2 * kH + row2], planes);
        }
    }
    if (!a.bf16 && gid < 4 * a.w1_q * 64 * 4) {
        // float32 layer 1: index ((mt*Q + q)*64 + lane)*4 + u, st = 4q+u, k = 2st + h (< w1_ns)
        const int u = gid & 3, lane = (gid >> 2) & 63, q = (gid >> 8) % a.w1_q, mt = (gid >> 8) / a.w1_q;
        const int st = 4 * q + u, m = lane & 31, h = lane >> 5;
        const int kk = 2 * st + h;
        a.w1p[gid] = kk < a.w1_ns ? a.w1[(32 * mt + m) * a.w1_in + kk] : 0.0f;
    }
    if (gid < kW3PackBF16) {
        // index (st*64 + lane)*8 + i; lane (m, h), element i
        const int i = gid & 7, lane = (gid >> 3) & 63, st = gid >> 9;
        const int m = lane & 31, h = lane >> 5;
        const int k = phi16(st, i, h);
        a.w3pb[gid] = m < 3 ? f2bf(a.w3[m * kH + k]) : static_cast<uint16_t>(0);
        store_planes(a.w1tpb, gid, kW1TPackBF16, m < kC ? a.w1[k * a.w1_in + m] : 0.0f, planes);
    }
    if (a.bf16 && gid < kW3TPackBF16) {
        // index (mt*64 + lane)*8 + i, k = 8h + i (< 3)
        const int i = gid & 7, lane = (gid >> 3) & 63, mt = gid >> 9;
        const int m = lane & 31, h = lane >> 5;
        const int k = 8 * h + i;
        a.w3tpb[gid] = k < 3 ? f2bf(a.w3[k * kH + 32 * mt + m]) : static_cast<uint16_t>(0);
    }
    if (gid < 4 * a.w1_s1 * 64 * 8) {
        // bfloat16 layer 1: index ((mt*S1 + st)*64 + lane)*8 + i, k = 16st + 8h + i (< w1_ns)
        const int i = gid & 7, lane = (gid >> 3) & 63, st = (gid >> 9) % a.w1_s1, mt = (gid >> 9) / a.w1_s1;
        const int m = lane & 31, h = lane >> 5;
        const int kk = 16 * st + 8 * h + i;
        store_planes(a.w1pb, gid, 4 * a.w1_s1 * 64 * 8, kk < a.w1_ns ? a.w1[(32 * mt + m) * a.w1_in + kk] : 0.0f,
                     planes);
    }
}


struct MlpArgs {
    const int* sample_ray;
    const int64_t* n_kept;
    int64_t cap;
    const float* w1;      // W1 and W2 as given, for plain_adjoint
    const float* w2;
    const float* b2;
    const float* w3;      // [3][128]
    const float* b3;
    const float* base;    // [B][128] per-ray first-layer part incl. b1
    const float* pe;      // [B][32]
    const float* w1p;
    const float* w2p;
    const uint16_t* w1pb;
    const uint16_t* w2pb;
    const uint16_t* w2tpb;
    const uint16_t* w3pb;
    const uint16_t* w3tpb;
    const uint16_t* w1tpb;
    float* feat;          // [cap][12]: gathered features in
    float* col;           // [cap][4]: colour out (forward) / dL/dc in (backward)
    float* partial;       // [blocks][kPStride] weight-gradient partials
    int bf16;
    // backward: each sample's record (head, dL/dfeat) goes to its binned slot
    const int2* cell_rank;    // [cap] (cell, rank within cell)
    const int* cell_start;    // [ncell + 1]
    const float4* rec_head;   // [cap] (fx, fy, fz, dL/draw)
    float4* rec;              // [cap][4] binned records
    uint32_t* live;           // [cap][8] ReLU branches (float32 form; NULL: not wanted)
    int* wide;                // float32 adjoint: not 0 where its values may leave the planes' range
};

// The query position of each sample, for the networks with an encoded
// position (a separate kernel argument, so that the other kernels' argument
// block stays as it is): x = o + t_k d in the sampler's float32 recipe,
// u = (x - pe_c) * pe_ih.
struct PosArgs {
    const float* rays_o;
    const float* rays_d;
    const float* jitter;
    const float* t_near;
    const int* sample_k;
    float step;
    float pe_c[3];
    float pe_ih[3];
};

__device__ __forceinline__ MlpArgs refresh(const MlpArgs& a) {
    MlpArgs l = a;
    l.b2 = opaque(a.b2);
    l.w3 = opaque(a.w3);
    l.b3 = opaque(a.b3);
    l.w1p = opaque(a.w1p);
    l.w2p = opaque(a.w2p);
    l.w1pb = opaque(a.w1pb);
    l.w2pb = opaque(a.w2pb);
    l.w2tpb = opaque(a.w2tpb);
    l.w3pb = opaque(a.w3pb);
    l.w3tpb = opaque(a.w3tpb);
    l.w1tpb = opaque(a.w1tpb);
    return l;
}

__device__ __forceinline__ void load_base(const float* base, int r, int h, f32x16 acc[4]) {
    const float* br = base + static_cast<int64_t>(r) * kH;
    #pragma unroll
    for (int mt = 0; mt < 4; ++mt)
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(br + 32 * mt + 8 * q + 4 * h);
            acc[mt][4 * q + 0] = v.x;
            acc[mt][4 * q + 1] = v.y;
            acc[mt][4 * q + 2] = v.z;
            acc[mt][4 * q + 3] = v.w;
        }
}

__device__ __forceinline__ void load_feat(const float* feat, int64_t s, float f[12]) {
    const float4* p = reinterpret_cast<const float4*>(feat + s * 12);
    const float4 q0 = p[0], q1 = p[1], q2 = p[2];
    f[0] = q0.x; f[1] = q0.y; f[2] = q0.z; f[3] = q0.w;
    f[4] = q1.x; f[5] = q1.y; f[6] = q1.z; f[7] = q1.w;
    f[8] = q2.x; f[9] = q2.y; f[10] = q2.z; f[11] = q2.w;
}

// Per-sample first-layer inputs of sample s on ray r: its 12 features,
// then (KX > 0) the encoded position [u, sin(2^j u), cos(2^j u)], j < KX
// (sine and cosine by pe_sincos: |2^j u| <= 16 for a sample in the box).
// (in two parts: the loads, then the arithmetic, so that a caller can place
// other work between them)
struct SampleIn {
    float f[kC];
    float o[3], d[3];
    float p, tn;
    int k;
};

template <int KX>
__device__ __forceinline__ void sample_loads(const PosArgs& a, const float* feat, int64_t s, int r, SampleIn& in) {
    load_feat(feat, s, in.f);
    if constexpr (KX > 0) {
        #pragma unroll
        for (int i = 0; i < 3; ++i) {
            in.o[i] = a.rays_o[3 * r + i];
            in.d[i] = a.rays_d[3 * r + i];
        }
        in.p = a.jitter ? a.jitter[r] : 0.0f;
        in.tn = a.t_near[r];
        in.k = a.sample_k[s];
    }
}

template <int KX>
__device__ __forceinline__ void sample_encode(const PosArgs& a, const SampleIn& in, float xs[NetLayout<KX>::kS]) {
    #pragma unroll
    for (int i = 0; i < kC; ++i) xs[i] = in.f[i];
    if constexpr (KX > 0) {
        float x[3];
        const float t = dvgo_dev::recipe_tk(in.tn, in.p, in.k, a.step);
        dvgo_dev::recipe_x(in.o, in.d, t, x);
        #pragma unroll
        for (int i = 0; i < 3; ++i) xs[kC + i] = (x[i] - a.pe_c[i]) * a.pe_ih[i];
        #pragma unroll
        for (int j = 0; j < KX; ++j)
            #pragma unroll
            for (int i = 0; i < 3; ++i) {
                float sv, cv;
                dvgo_dev::pe_sincos(xs[kC + i] * static_cast<float>(1 << j), &sv, &cv);
                xs[kC + 3 + 6 * j + i] = sv;
                xs[kC + 6 + 6 * j + i] = cv;
            }
    }
}

template <int KX>
__device__ __forceinline__ void sample_inputs(const PosArgs& a, const float* feat, int64_t s, int r,
                                              float xs[NetLayout<KX>::kS]) {
    SampleIn in;
    sample_loads<KX>(a, feat, s, r, in);
    sample_encode<KX>(a, in, xs);
}

// ---------------------------------------------------------------------------
// bfloat16 matrix cores (v_mfma_f32_32x32x16_bf16): K = 16 per step, 8
// consecutive K values per lane half; float32 accumulation.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Round-to-nearest-even bfloat16 pairs of accumulator values, as the packed
// 32-bit words of an 8-element operand (one v_cvt_pk_bf16_f32 per pair).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2 cvt_pair(const f32x16& v, int i) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 x = {v[i], v[i + 1]};
    return __builtin_bit_cast(u16x2, __builtin_convertvector(x, bf16x2));
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int g) {
    u32x4 w;
    #pragma unroll
    for (int p = 0; p < 4; ++p) w[p] = __builtin_bit_cast(unsigned int, cvt_pair(v, 8 * g + 2 * p));
    return __builtin_bit_cast(bf16x8, w);
}

// bf16(relu(x)) for 8 accumulator values: round first, then clamp the signed
// 16-bit patterns at 0 (two values per packed integer max).  Rounding is
// monotone and maps no positive float32 to a negative bfloat16, so this
// equals rounding relu(x) (a negative input gives +0 either way).
__device__ __forceinline__ bf16x8 relu_pack8(const f32x16& v, int g) {
    const s16x2 zero = {0, 0};
    u32x4 w;
    #pragma unroll
    for (int p = 0; p < 4; ++p) {
        const s16x2 q = __builtin_elementwise_max(__builtin_bit_cast(s16x2, cvt_pair(v, 8 * g + 2 * p)), zero);
        w[p] = __builtin_bit_cast(unsigned int, q);
    }
    return __builtin_bit_cast(bf16x8, w);
}

// bf16(d) where the activation (a bf16 relu output, so a non-negative
// pattern) is non-zero, else +0: the relu derivative applied after
// rounding, with packed 16-bit min(act, 1) as the 0/1 factor (written as
// the two packed instructions; the optimiser would otherwise split each
// pair into compares and selects).  The constant 1 goes in a register
// holding it in both halves: an inline constant of a packed instruction
// would give the high half 0.
__device__ __forceinline__ bf16x8 relu_grad_pack8(const f32x16& d, int g, const bf16x8& act) {
    const u32x4 aw = __builtin_bit_cast(u32x4, act);
    const unsigned int ones = 0x00010001u;
    u32x4 w;
    #pragma unroll
    for (int p = 0; p < 4; ++p) {
        unsigned int m, r;
        asm("v_pk_min_u16 %0, %1, %2" : "=v"(m) : "v"(aw[p]), "v"(ones));
        asm("v_pk_mul_lo_u16 %0, %1, %2" : "=v"(r) : "v"(__builtin_bit_cast(unsigned int, cvt_pair(d, 8 * g + 2 * p))),
            "v"(m));
        w[p] = r;
    }
    return __builtin_bit_cast(bf16x8, w);
}


// NT output tiles mt0 .. mt0+NT-1 of a chained 128-wide layer, K step
// outermost: the NT weight fragments of step st+1 are read from LDS while
// the NT matrix-core ops of step st run (the order is pinned with
// scheduling-group barriers: the register allocator would otherwise
// serialise every read with its consumer).
template <int NT>
__device__ __forceinline__ void chain_tiles_bf16(const bf16x8* w, int lane, int mt0, const bf16x8 in[8],
                                                 f32x16 acc[NT]) {
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 cur[NT];
    #pragma unroll
    for (int t = 0; t < NT; ++t) cur[t] = w[((mt0 + t) * 8) * 64 + lane];
    #pragma unroll
    for (int st = 0; st < 8; ++st) {
        bf16x8 nxt[NT];
        if (st < 7) {
            #pragma unroll
            for (int t = 0; t < NT; ++t) nxt[t] = w[((mt0 + t) * 8 + st + 1) * 64 + lane];
        }
        #pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mma_bf16(cur[t], in[st], acc[t]);
        if (st < 7) {
            #pragma unroll
            for (int t = 0; t < NT; ++t) cur[t] = nxt[t];
        }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);       // LDS reads of step 0
    #pragma unroll
    for (int st = 0; st < 7; ++st) {
        __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);   // LDS reads of step st+1
        __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);   // matrix-core ops of step st
    }
    __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
    __builtin_amdgcn_sched_barrier(0);
}

struct ChainBF16 {
    f32x16 z2[4];   // layer-2 pre-activation
    bf16x8 hb[8];   // bf16(relu(layer 1)) in chained operand order
};

// Operand of layer-1 K step st for lane half h: per-sample inputs
// 16st + 8h .. 16st + 8h + 7 (zero beyond kS), selected with constant
// indices.
template <int KX>
__device__ __forceinline__ bf16x8 layer1_operand(const float xs[NetLayout<KX>::kS], int st, int h) {
    constexpr int kS = NetLayout<KX>::kS;
    bf16x8 fb;
    #pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k0 = 16 * st + e, k1 = k0 + 8;
        const float v0 = k0 < kS ? xs[k0 < kS ? k0 : 0] : 0.0f;
        const float v1 = k1 < kS ? xs[k1 < kS ? k1 : 0] : 0.0f;
        fb[e] = static_cast<__bf16>(h ? v1 : v0);
    }
    return fb;
}

template <int KX>
__device__ __forceinline__ void forward_chain_bf16(const MlpArgs& a, const bf16x8* sW1, const bf16x8* sW2,
                                                   const float* sB2, int r, const float xs[NetLayout<KX>::kS],
                                                   int lane, ChainBF16& c) {
    constexpr int kS1 = NetLayout<KX>::kS1;
    const int h = lane >> 5;
    f32x16 h1[4];
    load_base(a.base, r, h, h1);
    #pragma unroll
    for (int st = 0; st < kS1; ++st) {
        const bf16x8 fb = layer1_operand<KX>(xs, st, h);
        #pragma unroll
        for (int mt = 0; mt < 4; ++mt) h1[mt] = mma_bf16(sW1[(mt * kS1 + st) * 64 + lane], fb, h1[mt]);
    }
    #pragma unroll
    for (int mt = 0; mt < 4; ++mt)
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 b = *reinterpret_cast<const float4*>(sB2 + 32 * mt + 8 * q + 4 * h);
            c.z2[mt][4 * q] = b.x;
            c.z2[mt][4 * q + 1] = b.y;
            c.z2[mt][4 * q + 2] = b.z;
            c.z2[mt][4 * q + 3] = b.w;
        }
    #pragma unroll
    for (int st = 0; st < 8; ++st) c.hb[st] = relu_pack8(h1[st >> 1], st & 1);
    chain_tiles_bf16<4>(sW2, lane, 0, c.hb, c.z2);
}

// Layer 3 on matrix cores: logits of sample m land in lane m (half 0),
// registers 0..2; bfloat16 relu(z2) and W3, float32 accumulation.
__device__ __forceinline__ f32x16 head_bf16(const MlpArgs& a, const f32x16 z2[4], int lane, float c[3],
                                            bf16x8 h2b[8]) {
    const int h = lane >> 5;
    f32x16 z3;
    #pragma unroll
    for (int rr = 0; rr < 16; ++rr) z3[rr] = (h == 0 && rr < 3) ? a.b3[rr] : 0.0f;
    const bf16x8* w3 = reinterpret_cast<const bf16x8*>(a.w3pb);
    #pragma unroll
    for (int st = 0; st < 8; ++st) {
        const bf16x8 hv = relu_pack8(z2[st >> 1], st & 1);
        h2b[st] = hv;
        z3 = mma_bf16(w3[st * 64 + lane], hv, z3);
    }
    c[0] = 1.0f / (1.0f + expf(-z3[0]));
    c[1] = 1.0f / (1.0f + expf(-z3[1]));
    c[2] = 1.0f / (1.0f + expf(-z3[2]));
    return z3;
}

// kN 16-byte operand fragments copied from global memory to LDS by a
// workgroup of kThreads, in two steps: load() issues a thread's loads into
// registers, store() writes them to LDS.  Trip counts are compile-time
// constants, so loads of several copies can all be issued before the first
// store (a runtime-bounded copy loop waits on each load in turn).
template <int kThreads, int kN>
struct Frags {
    static constexpr int kPer = (kN + kThreads - 1) / kThreads;
    bf16x8 t[kPer];
    __device__ __forceinline__ void load(const bf16x8* src) {
        #pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = static_cast<int>(threadIdx.x) + u * kThreads;
            if (kN % kThreads == 0 || i < kN) t[u] = src[i];
        }
    }
    __device__ __forceinline__ void store(bf16x8* dst) const {
        #pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = static_cast<int>(threadIdx.x) + u * kThreads;
            if (kN % kThreads == 0 || i < kN) dst[i] = t[u];
        }
    }
};

// The forward's operands: packed W1 (kW1 fragments), W2 and b2 (float32).
template <int kThreads, int kW1>
__device__ __forceinline__ void load_packed_bf16(const MlpArgs& a, bf16x8* sW1, bf16x8* sW2, float* sB2) {
    Frags<kThreads, kW2PackBF16 / 8> f2;
    Frags<kThreads, kW1> f1;
    f2.load(reinterpret_cast<const bf16x8*>(a.w2pb));
    f1.load(reinterpret_cast<const bf16x8*>(a.w1pb));
    const float b2 = threadIdx.x < kH ? a.b2[threadIdx.x] : 0.0f;
    f2.store(sW2);
    f1.store(sW1);
    if (threadIdx.x < kH) sB2[threadIdx.x] = b2;
}

template <int KX>
__global__ __launch_bounds__(256, 3) void mlp_fwd_bf16_kernel(MlpArgs a0, PosArgs pa) {
    constexpr int kW1 = 4 * NetLayout<KX>::kS1 * 64;   // layer-1 operand fragments
    __shared__ bf16x8 sW2[kW2PackBF16 / 8];
    __shared__ bf16x8 sW1[kW1];
    __shared__ __attribute__((aligned(16))) float sB2[kH];
    load_packed_bf16<256, kW1>(a0, sW1, sW2, sB2);
    __syncthreads();
    const int64_t n = *a0.n_kept < a0.cap ? *a0.n_kept : a0.cap;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 31, h = lane >> 5;
    for (int64_t tile = static_cast<int64_t>(blockIdx.x) * 4 + wave; tile * 32 < n;
         tile += static_cast<int64_t>(gridDim.x) * 4) {
        const MlpArgs a = refresh(a0);
        const int64_t s = tile * 32 + m;
        const bool ok = s < n;
        const int64_t sc = ok ? s : n - 1;
        const int r = a.sample_ray[sc];
        float xs[NetLayout<KX>::kS];
        sample_inputs<KX>(pa, a.feat, sc, r, xs);
        ChainBF16 c;
        forward_chain_bf16<KX>(a, sW1, sW2, sB2, r, xs, lane, c);
        float col[3];
        bf16x8 h2b[8];
        head_bf16(a, c.z2, lane, col, h2b);
        if (ok && h == 0) reinterpret_cast<float4*>(a.col)[s] = make_float4(col[0], col[1], col[2], 0.0f);
    }
}

constexpr int kSB = 64;   // samples per block

// Activation tile of one plane: kSB rows of 16 units of 16 bytes.  Unit
// 2st + h of a row holds the eight features phi16(st, 0..7, h) that one lane
// produces and, as the next layer's operand, reads: one 16-byte access each
// way.  The unit index is permuted by the row, so that eight consecutive rows
// (one phase of a 16-byte access) and the 4 rows x 2 units of a transpose
// read's 16 lanes cover all banks.
__device__ __forceinline__ int unit_swz(int r) { return ((r & 3) << 1) | ((r >> 2) & 1) | (r & 8); }

constexpr int kTile = kSB * kH;             // elements of one plane of an activation tile
constexpr uint32_t kPlaneB = 2 * kTile;     // its bytes
constexpr uint32_t kColB = 32 * kH * 2;     // bytes of one column tile's 32 rows

// LDS by byte address, so that one register serves every access that differs
// by a constant (the instruction's offset field): plane, column tile and K
// step of an activation tile.
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ uint32_t lds_addr(void* p) { return (uint32_t)(uintptr_t)(lds_char*)p; }
template <typename T>
__device__ __forceinline__ T lds_get(uint32_t a) { return *(__attribute__((address_space(3))) const T*)a; }
template <typename T>
__device__ __forceinline__ void lds_put(uint32_t a, const T& v) { *(__attribute__((address_space(3))) T*)a = v; }

// K-major operand from two LDS transpose reads: lane (m, h) receives feature
// c0 + m of samples s0 + 8h .. s0 + 8h + 7.  A read transposes a 16x4 block
// within each group of 16 lanes: lane t of group G addresses sample
// s0 + 8(G/2) + t/4 and features c0 + 16(G%2) + 4(t%4) .. + 3, and receives
// feature c0 + 16(G%2) + t of those four samples.  a: the first four samples'
// address, b: the same 4 rows on.
__device__ __forceinline__ bf16x8 tr_pair(uint32_t a, uint32_t b) {
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)a);
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)b);
    const s16x8 uv = __builtin_shufflevector(u, v, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, uv);
}

__device__ __forceinline__ float wave_total(float v) {
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ f32x16 zero_tile() {
    f32x16 z;
    #pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.0f;
    return z;
}

// ---------------------------------------------------------------------------
// bfloat16 adjoint: weights stationary.  Eight wavefronts per workgroup (two
// per SIMD) take a block of 128 samples.  Wavefront (w, q) owns the features
// 32w .. 32w + 31 of every layer for the 64 samples of half q (two column
// tiles), and of the weight gradients the rows 32w over all 128 samples: of
// dW2 the columns of tiles 2q and 2q + 1, of dW1 those of tile q.  Its rows of
// W2, then of W2^T, and its gradients stay in registers; a block's activations
// pass between the wavefronts as [sample][feature] rows in LDS: the operand of
// a layer is one 16-byte read per lane and K step for 32 x 32 outputs, that of
// a weight gradient the same rows through the LDS transpose load.
//
// Bound by the six phases between barriers, in which the two wavefronts of a
// SIMD do the same: their 160 matrix instructions per block are 5100 cycles,
// the vector instructions about 4800 (the head's sigmoid and the packing of
// rows), a block takes 14,800, of which 4400 are waits at the barriers.
// Reading the rows of the next K steps while a step's instructions run was
// worth 3,000 of them, dL/dz1 in rows of its own (one barrier less) 650.
// The layout before, 32 samples stationary per wavefront pair and the weights
// read from LDS, took 1.5 times the LDS bytes and eight barriers: 390k samples
// 93 -> 83 us, 7.1M samples 1610 -> 1383 us, with encoded positions (KX = 5,
// 153k samples) 80 -> 60 us.
// ---------------------------------------------------------------------------
template <int KX>
__global__ __launch_bounds__(512, 2) void mlp_bwd_bf16_kernel(MlpArgs a0, PosArgs pa) {
    using L = NetLayout<KX>;
    constexpr int kS1 = L::kS1;
    constexpr int kXP = KX > 0 ? 112 : 80;          // pitch of an x' row: 4 rows of a transpose read on distinct banks
    constexpr int kGroups = (L::kIn + 1 + 7) / 8;   // 8-column groups of x' = [inputs, PE(d), 1]
    constexpr int kXF = 8 * kGroups + 4;            // pitch of the float32 x' rows (KX > 0)
    constexpr int kCP = 72;                         // pitch of a dz3 row (samples)
    constexpr int kS = 128;                         // samples per block
    constexpr int kZB = kS * kH * 2, kDB = 4 * kS * kC * 4;
    __shared__ __attribute__((aligned(256))) __bf16 sH[kS * kH];    // h1
    __shared__ __attribute__((aligned(256))) __bf16 sG[kS * kH];    // dL/dz1
    // h2 (own rows and columns), then dL/dz2; the wavefronts' logits, then
    // their dL/dfeat; between two blocks the float32 x' rows share both
    __shared__ __attribute__((aligned(256))) char sU[kZB + kDB];
    __shared__ __attribute__((aligned(256))) __bf16 sX[kS * kXP];   // x'
    __shared__ __attribute__((aligned(16))) __bf16 sCs[8][4 * kCP]; // dL/dz3 [channel][sample], row 3 zero
    __shared__ __attribute__((aligned(16))) float sB2[kH];
    __shared__ float sRed[4];
    static_assert(kS * kXF * 4 <= kZB + kDB, "the float32 x' rows share sU");
    __bf16* sZ = reinterpret_cast<__bf16*>(sU);
    float (*sL)[kS][4] = reinterpret_cast<float (*)[kS][4]>(sU + kZB);
    float (*sD)[kS][kC] = reinterpret_cast<float (*)[kS][kC]>(sU + kZB);
    float* sXF = reinterpret_cast<float*>(sU);
    const int64_t n = *a0.n_kept < a0.cap ? *a0.n_kept : a0.cap;
    // The wavefront index in a scalar register: role branches are scalar
    // branches then.  Under a vector-masked branch a matrix instruction still
    // updates its accumulator in a wavefront whose mask is empty.
    const int t = static_cast<int>(threadIdx.x);
    const int lane = t & 63, wave8 = __builtin_amdgcn_readfirstlane(t >> 6);
    const int q = wave8 >> 2, wave = wave8 & 3;
    const int m = lane & 31, h = lane >> 5;
    __bf16* sC = sCs[wave8];
    // dW2, dW1: as above; over the half's own samples: dX (dW3 in columns
    // 0..2, db2 in column 3) and (KX > 0) dW1's third tile
    f32x16 dW2[2] = {zero_tile(), zero_tile()}, dW1 = zero_tile(), dW1c = zero_tile(), dX = zero_tile();
    float db3[3] = {0.0f, 0.0f, 0.0f};
    bf16x8 one3, zero8;   // a ones column 3
    #pragma unroll
    for (int e = 0; e < 8; ++e) {
        one3[e] = static_cast<__bf16>(m == 3 ? 1.0f : 0.0f);
        zero8[e] = static_cast<__bf16>(0.0f);
    }
    // the wavefront's rows of W2 (layer 2) or W2^T (its adjoint): one register
    // set, refilled from the L2 (both, and the smaller operands, did not fit:
    // 103 registers spilled)
    bf16x8 wf[8];
    auto load_w = [&](const uint16_t* w, int st) {
        wf[st] = (reinterpret_cast<const bf16x8*>(w) + wave * 512 + st * 64)[lane];
    };
    for (int i = t; i < kS * kXP / 8; i += 512) reinterpret_cast<bf16x8*>(sX)[i] = zero8;   // columns past the last group
    for (int i = lane; i < kCP; i += 64) sC[3 * kCP + i] = static_cast<__bf16>(0.0f);
    if (threadIdx.x < kH) sB2[threadIdx.x] = a0.b2[threadIdx.x];
    const float b3[3] = {a0.b3[0], a0.b3[1], a0.b3[2]};
    // |dL/dz2| stays below 2^120 where the sum of a sample's |dL/dz3| is below this
    float dz3_most = 0.0f;
    #pragma unroll
    for (int u = 0; u < 3 * kH / 64; ++u) dz3_most += fabsf(a0.w3[64 * u + lane]);
    dz3_most = 0x1p120f / wave_total(dz3_most);   // (an infinite or NaN weight: every block is mixed)
    __syncthreads();
    const int xrow = t >> 2, xq = t & 3;   // the x' row and first column group this thread stages
    // A block's samples by a scalar base and a 32-bit lane offset (the last
    // block's missing samples read its last one).
    const int nblocks = static_cast<int>((n + kS - 1) / kS);
    auto last_of = [&](int blk) {
        const int64_t left = n - static_cast<int64_t>(blk) * kS;
        return static_cast<int>(left < kS ? left : kS) - 1;
    };
    const int col0 = 64 * q + m;   // this lane's first column's sample (the second is 32 on)
    // the rays of the next block's samples (this lane's two columns, and this
    // thread's x' row), loaded a block ahead
    int r_n[2], xr_n;
    auto load_rays = [&](const MlpArgs& a, int blk) {
        const int* sr = a.sample_ray + static_cast<int64_t>(blk) * kS;
        const int last = last_of(blk);
        #pragma unroll
        for (int c = 0; c < 2; ++c) r_n[c] = sr[min(32 * c + col0, last)];
        xr_n = sr[min(xrow, last)];
    };
    // this thread's x' columns (KX == 0), loaded while the block before ends
    float4 xin[4];
    auto load_x = [&](const MlpArgs& a, int blk) {
        if constexpr (KX == 0) {
            // groups: f[0..7] | f[8..11], PE[0..3] | PE[4..11] | PE[12..19] | PE[20..26], 1
            const float* f = a.feat + static_cast<int64_t>(blk) * (kS * kC) + min(xrow, last_of(blk)) * kC;
            const float* pe = a.pe + static_cast<int64_t>(xr_n) * 32;
            xin[0] = *reinterpret_cast<const float4*>(xq < 2 ? f + 8 * xq : pe + 8 * xq - 12);
            xin[1] = *reinterpret_cast<const float4*>(xq < 1 ? f + 4 : pe + 8 * xq - 8);
            xin[2] = *reinterpret_cast<const float4*>(pe + 20);
            xin[3] = *reinterpret_cast<const float4*>(pe + 24);
        }
    };
    if (static_cast<int>(blockIdx.x) < nblocks) {
        load_rays(a0, blockIdx.x);
        load_x(a0, blockIdx.x);
        #pragma unroll
        for (int st = 0; st < 8; ++st) load_w(a0.w2pb, st);
    }
    // acc += wf * (rows of an activation tile); the rows of the next kAhead K
    // steps are on their way from LDS while a step's instructions run
    auto chain = [&](uint32_t row, f32x16 acc[2]) {
        constexpr int kAhead = 3;
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 B[kAhead + 1][2];
        auto rd = [&](int st) {
            #pragma unroll
            for (int c = 0; c < 2; ++c) B[st % (kAhead + 1)][c] = lds_get<bf16x8>((row ^ (32u * st)) + c * kColB);
        };
        #pragma unroll
        for (int st = 0; st < kAhead; ++st) rd(st);
        #pragma unroll
        for (int st = 0; st < 8; ++st) {
            if (st + kAhead < 8) rd(st + kAhead);
            #pragma unroll
            for (int c = 0; c < 2; ++c) acc[c] = mma_bf16(wf[st], B[st % (kAhead + 1)][c], acc[c]);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * kAhead, 0);
        #pragma unroll
        for (int st = 0; st < 8; ++st) {
            if (st + kAhead < 8) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // operand of a feature tile over samples 16st .. 16st + 15
    auto tr_unit = [&](uint32_t at, int st) {
        const uint32_t off = st * (16 * kH * 2);
        return tr_pair(at + off, (at ^ 16u) + 4 * kH * 2 + off);
    };
    for (int blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        const MlpArgs a = refresh(a0);
        // the next block of this workgroup, or (the last time) this one again
        const int next = blk + static_cast<int>(gridDim.x) < nblocks ? blk + static_cast<int>(gridDim.x) : blk;
        const int64_t s0 = static_cast<int64_t>(blk) * kS;
        const int last = last_of(blk);
        const int xi = min(xrow, last);   // this thread's x' and record sample
        // this lane's LDS addresses (hidden from the optimiser, which would
        // otherwise keep every sum of them in a register of its own):
        // its sample's row, unit h; the unit it stages; the first of its two
        // transpose reads of feature tile nt (the second is 4 rows on, where
        // the unit permutation differs in its lowest bit)
        const int tG = lane >> 4, tt = lane & 15, trow = 8 * (tG >> 1) + (tt >> 2);
        const uint32_t tsub = trow * 256 + 8 * ((tt & 3) >> 1), tu = 2 * (tG & 1) + (tt & 1);
        uint32_t rowH = lds_addr(sH) + col0 * 256 + 16 * (h ^ unit_swz(m));
        uint32_t rowZ = lds_addr(sZ) + col0 * 256 + 16 * (h ^ unit_swz(m));
        uint32_t putH = rowH ^ (64u * wave), putZ = rowZ ^ (64u * wave);
        uint32_t putG = lds_addr(sG) + (putH - lds_addr(sH));
        uint32_t trH = lds_addr(sH) + tsub + 16 * (tu ^ unit_swz(trow));
        uint32_t trZ = (lds_addr(sZ) + tsub + 16 * (tu ^ unit_swz(trow))) ^ (64u * wave);
        uint32_t trG = (lds_addr(sG) + tsub + 16 * (tu ^ unit_swz(trow))) ^ (64u * wave);
        uint32_t colX = lds_addr(sX) + (col0 * kXP + 8 * h) * 2;
        uint32_t trX = lds_addr(sX) + (trow * kXP + 16 * (tG & 1) + 4 * (tt & 3)) * 2;
        uint32_t putX = lds_addr(sX) + xrow * kXP * 2;
        asm volatile("" : "+v"(rowH), "+v"(rowZ), "+v"(putH), "+v"(putZ), "+v"(putG), "+v"(trH), "+v"(trZ), "+v"(trG),
                     "+v"(colX), "+v"(trX), "+v"(putX));
        // this block's loads, in the order of their use: the wavefront's rows
        // of the first layer's per-ray part, W1, inputs of the head and the
        // records
        float4 base4[2][4];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float4* br = reinterpret_cast<const float4*>(a.base + static_cast<int64_t>(r_n[c]) * kH) + 8 * wave + h;
            #pragma unroll
            for (int q = 0; q < 4; ++q) base4[c][q] = br[2 * q];
        }
        bf16x8 w1f[kS1];
        #pragma unroll
        for (int st = 0; st < kS1; ++st)
            w1f[st] = (reinterpret_cast<const bf16x8*>(a.w1pb) + (wave * kS1 + st) * 64)[lane];
        const int xr = xr_n;
        // ---- x' rows
        auto put_x = [&](int col, const float4& u, const float4& v) {
            const float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
            bf16x8 b;
            #pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = static_cast<__bf16>(x[e]);
            lds_put(putX + 2 * col, b);
        };
        if constexpr (KX == 0) {
            put_x(8 * xq, xin[0], xin[1]);
            if (xq == 0) put_x(32, xin[2], xin[3]);
        } else {
            // the four threads of a row evaluate the encoded position (thread
            // q frequency q, thread 3 also frequency 4) and copy the rest
            float* row = sXF + xrow * kXF;
            float x[3], u[3], o[3], d[3];
            #pragma unroll
            for (int i = 0; i < 3; ++i) {
                o[i] = pa.rays_o[3 * xr + i];
                d[i] = pa.rays_d[3 * xr + i];
            }
            const float tk = dvgo_dev::recipe_tk(pa.t_near[xr], pa.jitter ? pa.jitter[xr] : 0.0f,
                                                 (pa.sample_k + s0)[xi], pa.step);
            dvgo_dev::recipe_x(o, d, tk, x);
            #pragma unroll
            for (int i = 0; i < 3; ++i) u[i] = (x[i] - pa.pe_c[i]) * pa.pe_ih[i];
            const float* f = a.feat + s0 * kC + xi * kC;
            const float* pe = a.pe + static_cast<int64_t>(xr) * 32;
            // features by threads 0..2, the view encoding (32 values) by all
            if (xq < 3) *reinterpret_cast<float4*>(row + 4 * xq) = *reinterpret_cast<const float4*>(f + 4 * xq);
            const float4 e0 = *reinterpret_cast<const float4*>(pe + 8 * xq);
            const float4 e1 = *reinterpret_cast<const float4*>(pe + 8 * xq + 4);
            const float ev[8] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z, e1.w};
            #pragma unroll
            for (int e = 0; e < 8; ++e) row[L::kS + 8 * xq + e] = ev[e];
            if (xq == 0) {
                #pragma unroll
                for (int i = 0; i < 3; ++i) row[kC + i] = u[i];
            }
            for (int j = xq; j < KX; j += xq == 3 ? 1 : KX) {
                #pragma unroll
                for (int i = 0; i < 3; ++i) {
                    float sv, cv;
                    dvgo_dev::pe_sincos(u[i] * static_cast<float>(1 << j), &sv, &cv);
                    row[kC + 3 + 6 * j + i] = sv;
                    row[kC + 6 + 6 * j + i] = cv;
                }
            }
            // the four threads of a row are lanes of one wavefront: its LDS
            // accesses are in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int g = xq; g < kGroups; g += 4)
                put_x(8 * g, *reinterpret_cast<const float4*>(row + 8 * g),
                      *reinterpret_cast<const float4*>(row + 8 * g + 4));
        }
        f32x16 h1[2];
        #pragma unroll
        for (int c = 0; c < 2; ++c)
            #pragma unroll
            for (int q = 0; q < 4; ++q) {
                h1[c][4 * q] = base4[c][q].x;
                h1[c][4 * q + 1] = base4[c][q].y;
                h1[c][4 * q + 2] = base4[c][q].z;
                h1[c][4 * q + 3] = base4[c][q].w;
            }
        __syncthreads();   // x' rows complete
        // ---- layer 1 (columns past the per-sample inputs meet zero weights)
        #pragma unroll
        for (int st = 0; st < kS1; ++st)
            #pragma unroll
            for (int c = 0; c < 2; ++c)
                h1[c] = mma_bf16(w1f[st], lds_get<bf16x8>(colX + (32 * c * kXP + 16 * st) * 2), h1[c]);
        #pragma unroll
        for (int c = 0; c < 2; ++c)
            #pragma unroll
            for (int g = 0; g < 2; ++g) lds_put((g ? putH ^ 32u : putH) + c * kColB, relu_pack8(h1[c], g));
        // inputs of the later phases, and the next block's rays
        load_rays(a, next);
        bf16x8 w3[2];
        #pragma unroll
        for (int g = 0; g < 2; ++g) w3[g] = (reinterpret_cast<const bf16x8*>(a.w3pb) + (2 * wave + g) * 64)[lane];
        const bf16x8 w3t = (reinterpret_cast<const bf16x8*>(a.w3tpb) + wave * 64)[lane];
        float4 dc[2];
        #pragma unroll
        for (int c = 0; c < 2; ++c) dc[c] = (reinterpret_cast<const float4*>(a.col) + s0)[min(32 * c + col0, last)];
        const int2 cr = (a.cell_rank + s0)[xi];
        f32x16 z2[2];
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 b = *reinterpret_cast<const float4*>(sB2 + 32 * wave + 8 * q + 4 * h);
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                z2[c][4 * q] = b.x;
                z2[c][4 * q + 1] = b.y;
                z2[c][4 * q + 2] = b.z;
                z2[c][4 * q + 3] = b.w;
            }
        }
        __syncthreads();   // h1 rows complete
        // ---- layer 2, the wavefront's share of the logits, h2 into its own columns of sZ
        chain(rowH, z2);
        #pragma unroll
        for (int st = 0; st < 8; ++st) load_w(a.w2tpb, st);
        bf16x8 w1t[2];   // for dL/dfeat
        #pragma unroll
        for (int g = 0; g < 2; ++g) w1t[g] = (reinterpret_cast<const bf16x8*>(a.w1tpb) + (2 * wave + g) * 64)[lane];
        bf16x8 h2[2][2];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            f32x16 z3 = zero_tile();
            #pragma unroll
            for (int g = 0; g < 2; ++g) {
                h2[c][g] = relu_pack8(z2[c], g);
                lds_put((g ? putZ ^ 32u : putZ) + c * kColB, h2[c][g]);
                z3 = mma_bf16(w3[g], h2[c][g], z3);
            }
            if (h == 0) *reinterpret_cast<float4*>(sL[wave][32 * c + col0]) = make_float4(z3[0], z3[1], z3[2], 0.0f);
        }
        const int slot = a.cell_start[cr.x];
        const float4 rh = (a.rec_head + s0)[xi];
        __syncthreads();   // logits complete
        // ---- dz3 (lane half 0), dW3 over the block's samples, dz2 = (W3^T bf16(dz3)) * relu'(z2)
        // (lane half h takes the sample of column tile h; the operand of both
        // tiles is in lane half 0)
        // (mixed: h2 or dL/dz2 may be infinite or NaN, of which dW3's and db2's
        // products would leave NaN in each other's columns of dX: 0 x inf)
        bool mixed;
        bf16x8 dzb[2] = {zero8, zero8}, h2t[4];
        #pragma unroll
        for (int st = 0; st < 4; ++st) h2t[st] = tr_unit(trZ + q * (4 * 16 * kH * 2), st);   // the half's own samples
        {
            float z[3] = {b3[0], b3[1], b3[2]};
            #pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float4 v = *reinterpret_cast<const float4*>(sL[w][32 * h + col0]);
                z[0] += v.x;
                z[1] += v.y;
                z[2] += v.z;
            }
            const float g[3] = {h ? dc[1].x : dc[0].x, h ? dc[1].y : dc[0].y, h ? dc[1].z : dc[0].z};
            const float on = 32 * h + col0 <= last ? 1.0f : 0.0f;
            float size = 0.0f;
            #pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float cv = 1.0f / (1.0f + expf(-z[ch]));
                const float dz3 = on > 0.0f ? g[ch] * cv * (1.0f - cv) : 0.0f;
                db3[ch] += dz3;
                size += fabsf(dz3);
                const __bf16 b = static_cast<__bf16>(dz3);
                sC[ch * kCP + 32 * h + m] = b;
                const uint32_t own = __builtin_bit_cast(uint16_t, b), other = __shfl_xor(own, 32, 64);
                dzb[0][ch] = __builtin_bit_cast(__bf16, static_cast<uint16_t>(h ? 0u : own));
                dzb[1][ch] = __builtin_bit_cast(__bf16, static_cast<uint16_t>(h ? 0u : other));
            }
            mixed = __any(!(fabsf(z[0]) + fabsf(z[1]) + fabsf(z[2]) < INFINITY && size < dz3_most));
        }
        const int qx = mixed ? -1 : q;
        auto dz3_col = [&](int st) {
            return *reinterpret_cast<const bf16x8*>(sC + (m < 3 ? m : 3) * kCP + 16 * st + 8 * h);
        };
        if (__builtin_expect(mixed, 0)) {
            f32x16 d = zero_tile();
            #pragma unroll
            for (int st = 0; st < 4; ++st) d = mma_bf16(h2t[st], dz3_col(st), d);
            #pragma unroll
            for (int i = 0; i < 16; ++i) dX[i] += m < 3 ? d[i] : 0.0f;
        } else {
            #pragma unroll
            for (int st = 0; st < 4; ++st) dX = mma_bf16(h2t[st], dz3_col(st), dX);
        }
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            f32x16 dh = zero_tile();
            dh = mma_bf16(w3t, dzb[c], dh);
            #pragma unroll
            for (int g = 0; g < 2; ++g)
                lds_put((g ? putZ ^ 32u : putZ) + c * kColB, relu_grad_pack8(dh, g, h2[c][g]));
        }
        load_x(a, next);
        __syncthreads();   // dz2 rows complete
        // ---- dh1 = W2^T dz2, dz1 = dh1 * relu'(h1), this wavefront's share of dL/dfeat = W1[:, :12]^T dz1
        f32x16 dh1[2] = {zero_tile(), zero_tile()};
        chain(rowZ, dh1);
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            f32x16 df = zero_tile();
            #pragma unroll
            for (int g = 0; g < 2; ++g) {
                const bf16x8 d1 = relu_grad_pack8(dh1[c], g, lds_get<bf16x8>((g ? putH ^ 32u : putH) + c * kColB));
                lds_put((g ? putG ^ 32u : putG) + c * kColB, d1);
                df = mma_bf16(w1t[g], d1, df);
            }
            // rows 0..11 of the tile: registers 0..3 are channels 4h .. 4h + 3,
            // registers 4..7 (half 0) channels 8..11
            *reinterpret_cast<float4*>(&sD[wave][32 * c + col0][4 * h]) = make_float4(df[0], df[1], df[2], df[3]);
            if (h == 0) *reinterpret_cast<float4*>(&sD[wave][32 * c + col0][8]) = make_float4(df[4], df[5], df[6], df[7]);
        }
        // ---- dW2 rows 32w, tiles 2q and 2q + 1 over the block's samples, db2
        // (through the ones column) over the half's own
        {
            constexpr int kAhead = 2;
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t trB[2] = {trH ^ (128u * q), trH ^ (128u * q + 64u)};
            bf16x8 A[kAhead + 1], B[kAhead + 1][2];
            auto rd = [&](int st) {
                A[st % (kAhead + 1)] = tr_unit(trZ, st);
                #pragma unroll
                for (int c = 0; c < 2; ++c) B[st % (kAhead + 1)][c] = tr_unit(trB[c], st);
            };
            #pragma unroll
            for (int st = 0; st < kAhead; ++st) rd(st);
            #pragma unroll
            for (int st = 0; st < 8; ++st) {
                if (st + kAhead < 8) rd(st + kAhead);
                #pragma unroll
                for (int c = 0; c < 2; ++c) dW2[c] = mma_bf16(A[st % (kAhead + 1)], B[st % (kAhead + 1)][c], dW2[c]);
                if (st >> 2 == qx) dX = mma_bf16(A[st % (kAhead + 1)], one3, dX);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (__builtin_expect(mixed, 0)) {
                f32x16 d = zero_tile();
                #pragma unroll
                for (int st = 0; st < 4; ++st) d = mma_bf16(tr_unit(trZ + q * (4 * 16 * kH * 2), st), one3, d);
                #pragma unroll
                for (int i = 0; i < 16; ++i) dX[i] += m == 3 ? d[i] : 0.0f;
            }
        }
        __syncthreads();   // dz1 rows and dL/dfeat shares complete
        // the sample's record, one 16-byte word per thread of its row
        {
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            #pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float4 u = *reinterpret_cast<const float4*>(&sD[w][xrow][xq > 0 ? 4 * (xq - 1) : 0]);
                v.x += u.x;
                v.y += u.y;
                v.z += u.z;
                v.w += u.w;
            }
            v.x = xq > 0 ? v.x : rh.x;
            v.y = xq > 0 ? v.y : rh.y;
            v.z = xq > 0 ? v.z : rh.z;
            v.w = xq > 0 ? v.w : rh.w;
            if (xrow <= last) a.rec[(static_cast<int64_t>(slot) + cr.y) * 4 + xq] = v;
        }
        // dW1's third tile over the half's own dz1 rows
        if constexpr (KX > 0) {
            #pragma unroll
            for (int st = 0; st < 4; ++st) {
                const uint32_t at = trX + ((64 * q + 16 * st) * kXP + 64) * 2;
                dW1c = mma_bf16(tr_unit(trG + q * (4 * 16 * kH * 2), st),
                                tr_pair(at, at + 4 * kXP * 2), dW1c);
            }
        }
        // ---- dW1 rows 32w, tile q (column kIn: the bias) over the block's samples
        {
            constexpr int kAhead = 3;
            const uint32_t trQ = trX + 64u * q;
            bf16x8 A[kAhead + 1], B[kAhead + 1];
            auto rd = [&](int st) {
                const uint32_t at = trQ + 16 * st * kXP * 2;
                A[st % (kAhead + 1)] = tr_unit(trG, st);
                B[st % (kAhead + 1)] = tr_pair(at, at + 4 * kXP * 2);
            };
            __builtin_amdgcn_sched_barrier(0);
            #pragma unroll
            for (int st = 0; st < kAhead; ++st) rd(st);
            #pragma unroll
            for (int st = 0; st < 8; ++st) {
                load_w(a.w2pb, st);   // W2 for the next block's layer 2
                if (st + kAhead < 8) rd(st + kAhead);
                dW1 = mma_bf16(A[st % (kAhead + 1)], B[st % (kAhead + 1)], dW1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();   // x', sD and sG read before the next block's staging
    }
    // ---- epilogue: this workgroup's partial of the flat gradient.  Half 1's
    // sums over its own samples are added to half 0's through LDS.
    float* out = a0.partial + static_cast<int64_t>(blockIdx.x) * L::kPStride;
    float4* xch = reinterpret_cast<float4*>(sU);   // [2 tiles][4 words][256 threads]
    static_assert(kZB + kDB >= 2 * 4 * 256 * 16, "the exchange fits sU");
    const int t4 = t & 255;
    #pragma unroll
    for (int c = 0; c < 3; ++c) db3[c] = wave_total(db3[c]);
    if (q == 1) {
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            xch[i * 256 + t4] = make_float4(dX[4 * i], dX[4 * i + 1], dX[4 * i + 2], dX[4 * i + 3]);
            if (KX > 0) xch[(4 + i) * 256 + t4] = make_float4(dW1c[4 * i], dW1c[4 * i + 1], dW1c[4 * i + 2], dW1c[4 * i + 3]);
        }
        if (t4 == 0)
            for (int c = 0; c < 3; ++c) sRed[c] = db3[c];
    }
    __syncthreads();
    #pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 32 * wave + acc_row(i, h);
        #pragma unroll
        for (int c = 0; c < 2; ++c) out[L::kOffW2 + row * kH + 32 * (2 * q + c) + m] = dW2[c][i];
        const int col = 32 * q + m;
        if (col < L::kIn) out[L::kOffW1 + row * L::kIn + col] = dW1[i];
        else if (col == L::kIn) out[L::kOffB1 + row] = dW1[i];
    }
    if (q == 1) return;
    #pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 u = xch[i * 256 + t4];
        dX[4 * i] += u.x;
        dX[4 * i + 1] += u.y;
        dX[4 * i + 2] += u.z;
        dX[4 * i + 3] += u.w;
        if (KX > 0) {
            const float4 v = xch[(4 + i) * 256 + t4];
            dW1c[4 * i] += v.x;
            dW1c[4 * i + 1] += v.y;
            dW1c[4 * i + 2] += v.z;
            dW1c[4 * i + 3] += v.w;
        }
    }
    #pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 32 * wave + acc_row(i, h);
        if (m < 3) out[L::kOffW3 + m * kH + row] = dX[i];
        else if (m == 3) out[L::kOffB2 + row] = dX[i];
        if (KX > 0) {
            const int col = 64 + m;
            if (col < L::kIn) out[L::kOffW1 + row * L::kIn + col] = dW1c[i];
            else if (col == L::kIn) out[L::kOffB1 + row] = dW1c[i];
        }
    }
    if (t == 0)
        for (int c = 0; c < 3; ++c) out[L::kOffB3 + c] = db3[c] + sRed[c];
}

}  // namespace
