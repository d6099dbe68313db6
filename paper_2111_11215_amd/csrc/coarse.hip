// Coarse stage of the paper (Sec. 4.1, "Coarse geometry searching"): a
// density grid with post-activation and a view-invariant colour grid
// (Eq. coarse_queries, colour = sigmoid of the interpolated 3 channels),
// trained with the photometric loss, the per-point rgb loss and the
// background entropy loss, Adam with the view-count-based learning rate of
// Prior 2 on the density.
//   coarse_step_kernel  one wavefront per ray: the forward (gathers,
//                       prefix-scan compositing, the ray's loss terms),
//                       then the adjoint walked from the ray's end with the
//                       transmittance recomputed by prefix sums as in the
//                       forward.  The grid gradients leave it in one of two
//                       ways: as binned records (a counting sort by cell,
//                       then one thread per vertex gathers the records of
//                       its eight cells), or, where the workspace does not
//                       hold them, by float atomics
//   loss_reduce         the per-ray losses summed in a fixed order
//   view_count / scale  Prior 2: per-vertex view counts and n_j / n_max
//   adam_scaled         Adam with a per-element learning-rate factor
#include "adam.hpp"
#include "binning.hpp"
#include "common.hpp"
#include "scan.hpp"

using dvgo::GridArgs;
using namespace dvgo_dev;

namespace {

constexpr int kMaxSteps = 64;   // 64-sample steps per ray (4096 samples)

struct CoarseArgs {
    const float* rays_o;
    const float* rays_d;
    const float* jitter;
    const float* t_near;
    const int* perm;
    const int* ray_offset;
    const int* sample_k;
    const int64_t* n_kept;
    int64_t cap;
    int B;
    float step;
    GridArgs g;
    const float* density;
    const float* rgb;
    float act_shift;
    float bg[3];
    const float* target;
    float w_pt, w_bg;
    float* rgb_out;
    float* ray_loss;
    float* grad_density;
    float* grad_rgb;
    // binned form
    int* cell_count;     // [ncell + 1], zero on entry
    int2* cell_rank;     // [cap] (cell, rank within cell)
    float4* head;        // [cap][2] (fx, fy, fz, dL/draw), dL/dpre (3), 0
};

__device__ __forceinline__ float softplus_c(float x) { return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x))); }
__device__ __forceinline__ float sigmoid_c(float x) { return 1.0f / (1.0f + expf(-x)); }

// One sample's interpolated raw density and colour pre-activation, with the
// corner indices and weights for the scatter.
struct CSample {
    int64_t corner[8];   // corner[0] is the cell's base vertex
    float w[8];
    float f[3];          // position within the cell
    int cell;
    float raw, pre[3], t;
};

// Sum of v over the lanes from this one to the end of its run of equal
// keys (runs are contiguous: a ray's samples in one cell are consecutive,
// and a lane without a sample has a key of its own).
__device__ __forceinline__ float run_suffix_sum(float v, int64_t key, int lane) {
    #pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float ov = __shfl_down(v, off, 64);
        const int64_t ok = __shfl_down(key, off, 64);
        if (lane + off < 64 && ok == key) v += ov;
    }
    return v;
}

// kGather: with the grids' values; else its cell and position only.
template <bool kGather>
__device__ __forceinline__ void coarse_sample(const CoarseArgs& a, const float o[3], const float d[3], float tn, float p,
                                              int k, CSample& cs) {
    cs.t = recipe_tk(tn, p, k, a.step);
    float x[3];
    recipe_x(o, d, cs.t, x);
    int i0[3];
    float f[3];
    for (int i = 0; i < 3; ++i) {
        const float u = (x[i] - a.g.mn[i]) * a.g.scale[i];
        const float fl = fminf(fmaxf(floorf(u), 0.0f), static_cast<float>(a.g.n[i] - 2));
        i0[i] = static_cast<int>(fl);
        f[i] = fminf(fmaxf(u - fl, 0.0f), 1.0f);
    }
    const int64_t sx = static_cast<int64_t>(a.g.n[1]) * a.g.n[2], sy = a.g.n[2];
    const int64_t base = i0[0] * sx + i0[1] * sy + i0[2];
    for (int i = 0; i < 3; ++i) cs.f[i] = f[i];
    cs.cell = (i0[0] * (a.g.n[1] - 1) + i0[1]) * (a.g.n[2] - 1) + i0[2];
    if constexpr (!kGather) return;
    cs.raw = 0.0f;
    cs.pre[0] = cs.pre[1] = cs.pre[2] = 0.0f;
    #pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int bx = (c >> 2) & 1, by = (c >> 1) & 1, bz = c & 1;
        cs.w[c] = (bx ? f[0] : 1.0f - f[0]) * (by ? f[1] : 1.0f - f[1]) * (bz ? f[2] : 1.0f - f[2]);
        cs.corner[c] = base + bx * sx + by * sy + bz;
        cs.raw += cs.w[c] * a.density[cs.corner[c]];
        for (int ch = 0; ch < 3; ++ch) cs.pre[ch] += cs.w[c] * a.rgb[3 * cs.corner[c] + ch];
    }
}

// One ray per workgroup (a long ray holds only its own slot).  kBin: the
// gradients leave as binned records instead of float atomics.  A sample has 32
// grid entries and consecutive samples, half a voxel apart, share a cell only
// 1.25 at a time, so the atomics are about 25 per sample and bound the kernel:
// 574 us at 700k samples (8192 rays, 100^3).  The binned form takes 48 us here
// (70 without the cache), and the sort, the records' placement and the vertex
// gather 63 us; the whole training iteration 613 -> 145 us.
template <bool kBin>
__global__ __launch_bounds__(64) void coarse_step_kernel(CoarseArgs a) {
    // binned form: raw density and colour of the first kCached steps, for the
    // walk back (a ray across the 100^3 box has three)
    constexpr int kCached = 4;
    __shared__ float4 cache[kBin ? kCached : 1][64];
    const int lane = threadIdx.x;
    const int slot = blockIdx.x;
    const int64_t n = *a.n_kept < a.cap ? *a.n_kept : a.cap;
    const int r = a.perm[slot];
    int64_t s0 = a.ray_offset[slot], s1 = a.ray_offset[slot + 1];
    s0 = s0 < n ? s0 : n;
    s1 = s1 < n ? s1 : n;
    float o[3], d[3], tgt[3];
    for (int i = 0; i < 3; ++i) {
        o[i] = a.rays_o[3 * r + i];
        d[i] = a.rays_d[3 * r + i];
        tgt[i] = a.target[3 * r + i];
    }
    const float tn = a.t_near[r];
    const float p = a.jitter ? a.jitter[r] : 0.0f;
    const int64_t nsteps = (s1 - s0 + 63) / 64;
    // ---- forward: prefix-scan compositing; lane j keeps log T at the start of step j
    float logT = 0.0f, start = 0.0f, C[3] = {0.0f, 0.0f, 0.0f}, pt = 0.0f;
    for (int64_t it = 0; it < nsteps; ++it) {
        if (lane == static_cast<int>(it)) start = logT;
        const int64_t s = s0 + it * 64 + lane;
        const bool ok = s < s1;
        float sd = 0.0f, alpha = 0.0f, c[3] = {0.0f, 0.0f, 0.0f};
        if (ok) {
            CSample cs;
            coarse_sample<true>(a, o, d, tn, p, a.sample_k[s], cs);
            sd = softplus_c(cs.raw + a.act_shift) * a.step;
            alpha = -expm1f(-sd);
            for (int ch = 0; ch < 3; ++ch) c[ch] = sigmoid_c(cs.pre[ch]);
            if (kBin && it < kCached) cache[it][lane] = make_float4(cs.raw, c[0], c[1], c[2]);
        }
        const float incl = wave_incl_scan(sd, lane);
        const float excl = dpp_wave<0x138>(incl);
        const float w = ok ? expf(logT - excl) * alpha : 0.0f;
        float e2 = 0.0f;
        for (int ch = 0; ch < 3; ++ch) {
            C[ch] += w * c[ch];
            const float dd = c[ch] - tgt[ch];
            e2 += dd * dd;
        }
        pt += w * e2;
        logT -= lane_value(incl, 63);
    }
    for (int ch = 0; ch < 3; ++ch) C[ch] = wave_sum(C[ch]);
    pt = wave_sum(pt);
    const float Tend = expf(logT);
    const float invB = 1.0f / static_cast<float>(a.B);
    float gC[3], photo = 0.0f;
    for (int ch = 0; ch < 3; ++ch) {
        C[ch] += Tend * a.bg[ch];
        const float dd = C[ch] - tgt[ch];
        gC[ch] = 2.0f * dd * invB;
        photo += dd * dd;
    }
    // background entropy of T_end, clamped to [1e-6, 1 - 1e-6]
    const float pb = fminf(fmaxf(Tend, 1e-6f), 1.0f - 1e-6f);
    const float ent = -pb * logf(pb) - (1.0f - pb) * log1pf(-pb);
    const bool inside = Tend > 1e-6f && Tend < 1.0f - 1e-6f;
    const float gT = inside ? a.w_bg * (log1pf(-pb) - logf(pb)) * invB : 0.0f;
    if (lane == 0) {
        if (a.rgb_out)
            for (int ch = 0; ch < 3; ++ch) a.rgb_out[3 * r + ch] = C[ch];
        a.ray_loss[r] = photo + a.w_pt * pt + a.w_bg * ent;
    }
    // ---- adjoint: walk from the end, suffix sums S of w c (plus T_end bg)
    float S[3] = {Tend * a.bg[0], Tend * a.bg[1], Tend * a.bg[2]};
    const float ptk = 2.0f * a.w_pt * invB;
    for (int64_t it = nsteps - 1; it >= 0; --it) {
        const int64_t s = s0 + it * 64 + lane;
        const bool ok = s < s1;
        CSample cs;
        float sd = 0.0f, alpha = 0.0f, c[3] = {0.0f, 0.0f, 0.0f};
        if (ok) {
            if (kBin && it < kCached) {   // (each lane reads back its own entry)
                coarse_sample<false>(a, o, d, tn, p, a.sample_k[s], cs);
                const float4 v = cache[it][lane];
                cs.raw = v.x;
                c[0] = v.y;
                c[1] = v.z;
                c[2] = v.w;
            } else {
                coarse_sample<true>(a, o, d, tn, p, a.sample_k[s], cs);
                for (int ch = 0; ch < 3; ++ch) c[ch] = sigmoid_c(cs.pre[ch]);
            }
            sd = softplus_c(cs.raw + a.act_shift) * a.step;
            alpha = -expm1f(-sd);
        }
        const float logT0 = lane_value(start, static_cast<int>(it));
        const float incl = wave_incl_scan(sd, lane);
        const float excl = dpp_wave<0x138>(incl);
        const float Tafter = expf(logT0 - incl);
        const float w = ok ? expf(logT0 - excl) * alpha : 0.0f;
        float dsig = -Tend * gT;
        float tot[3];
        for (int ch = 0; ch < 3; ++ch) {
            const float sfx = wave_incl_suffix(w * c[ch], lane);
            const float sfx_ex = dpp_wave<0x130>(sfx);
            dsig += gC[ch] * (Tafter * c[ch] - (S[ch] + sfx_ex));
            tot[ch] = lane_value(sfx, 0);
        }
        {
            float draw = 0.0f, dpre[3] = {0.0f, 0.0f, 0.0f};
            if (ok) {
                draw = a.step * dsig * sigmoid_c(cs.raw + a.act_shift);
                for (int ch = 0; ch < 3; ++ch) {
                    const float dc = w * gC[ch] + ptk * w * (c[ch] - tgt[ch]);
                    dpre[ch] = dc * c[ch] * (1.0f - c[ch]);
                }
            }
            if constexpr (kBin) {
                const int rank = run_rank(ok ? cs.cell : -1, ok, lane, a.cell_count);
                if (ok) {
                    a.cell_rank[s] = make_int2(cs.cell, rank);
                    a.head[2 * s] = make_float4(cs.f[0], cs.f[1], cs.f[2], draw);
                    a.head[2 * s + 1] = make_float4(dpre[0], dpre[1], dpre[2], 0.0f);
                }
            } else {
            // every lane takes part in the shuffles; a lane without a sample
            // has a key of its own and contributes zeros
            const int64_t key = ok ? cs.corner[0] : -1 - static_cast<int64_t>(lane);
            const int64_t prev = __shfl_up(key, 1, 64);
            const bool head = ok && (lane == 0 || prev != key);
            #pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float wk = ok ? cs.w[k] : 0.0f;
                const float gd = run_suffix_sum(wk * draw, key, lane);
                float gr[3];
                for (int ch = 0; ch < 3; ++ch) gr[ch] = run_suffix_sum(wk * dpre[ch], key, lane);
                if (head) {
                    atomicAdd(a.grad_density + cs.corner[k], gd);
                    for (int ch = 0; ch < 3; ++ch) atomicAdd(a.grad_rgb + 3 * cs.corner[k] + ch, gr[ch]);
                }
            }
            }
        }
        for (int ch = 0; ch < 3; ++ch) S[ch] += tot[ch];
    }
}

// Records in cell order: each sample's two words at its cell's start + rank.
__global__ __launch_bounds__(256) void coarse_place_kernel(const int64_t* __restrict__ n_kept, int64_t cap,
                                                           const int2* __restrict__ cell_rank,
                                                           const int* __restrict__ cell_start,
                                                           const float4* __restrict__ head, float4* __restrict__ rec) {
    const int64_t n = *n_kept < cap ? *n_kept : cap;
    for (int64_t s = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; s < n;
         s += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int2 cr = cell_rank[s];
        const float4 h0 = head[2 * s], h1 = head[2 * s + 1];
        const int64_t pos = static_cast<int64_t>(cell_start[cr.x]) + cr.y;
        rec[2 * pos] = h0;
        rec[2 * pos + 1] = h1;
    }
}

// One thread per vertex: it is corner (dx, dy, dz) of cell (i-dx, j-dy, k-dz);
// for each (dx, dy) the records of cells k-1 and k are one run, split at the
// start of cell k.  Adds its gradient to the grids.
__global__ __launch_bounds__(256) void coarse_vertex_kernel(GridArgs g, const int* __restrict__ cell_start,
                                                            const float4* __restrict__ rec,
                                                            float* __restrict__ grad_density,
                                                            float* __restrict__ grad_rgb) {
    const int ny = g.n[1], nz = g.n[2], cy = ny - 1, cz = nz - 1;
    const int64_t nv = static_cast<int64_t>(g.n[0]) * ny * nz;
    const int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int k = static_cast<int>(v % nz), j = static_cast<int>((v / nz) % ny);
    const int i = static_cast<int>(v / (static_cast<int64_t>(nz) * ny));   // (beyond the grid for v >= nv: no cells)
    int p0[4], pm[4], p1[4];   // all in flight together
    #pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int ci = i - (c >> 1), cj = j - (c & 1);
        p0[c] = pm[c] = p1[c] = 0;
        if (v >= nv || ci < 0 || cj < 0 || ci >= g.n[0] - 1 || cj >= cy) continue;
        const int row = (ci * cy + cj) * cz;
        p0[c] = cell_start[row + (k > 0 ? k - 1 : 0)];
        pm[c] = cell_start[row + k];
        p1[c] = cell_start[row + (k < cz ? k + 1 : cz)];
    }
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    bool any = false;
    #pragma unroll
    for (int c = 0; c < 4; ++c) {
        const bool dx = c >> 1, dy = c & 1;
        #pragma unroll 2
        for (int p = p0[c]; p < p1[c]; ++p) {
            const float4 h = rec[2 * static_cast<int64_t>(p)], q = rec[2 * static_cast<int64_t>(p) + 1];
            const float w = (dx ? h.x : 1.0f - h.x) * (dy ? h.y : 1.0f - h.y) * (p < pm[c] ? h.z : 1.0f - h.z);
            acc[0] += w * h.w;
            acc[1] += w * q.x;
            acc[2] += w * q.y;
            acc[3] += w * q.z;
        }
        any |= p1[c] > p0[c];
    }
    const uint64_t touched = __ballot(any);
    if (touched == 0) return;
    // by atomics: calls on other streams may add to the same grids.  The 192
    // colour sums of the wavefront's vertices go out in address order: as fast
    // as plain additions (110 us for the whole call at 702k samples in 99^3
    // cells), where three strided atomics took 10 us more.
    __shared__ float col[4][64 * 3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (any) atomicAdd(grad_density + v, acc[0]);
    #pragma unroll
    for (int ch = 0; ch < 3; ++ch) col[wave][3 * lane + ch] = acc[1 + ch];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    #pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int e = 64 * u + lane;
        if (touched >> (e / 3) & 1) atomicAdd(grad_rgb + 3 * (v - lane) + e, col[wave][e]);
    }
}

// Single workgroup, fixed order: each thread adds every 1024th ray, eight
// loads in flight (a load at a time, 256 threads took 9.4 us for 8192 rays),
// then a fixed tree.
__global__ __launch_bounds__(1024) void ray_loss_reduce_kernel(const float* __restrict__ part, int n, float inv_n,
                                                               float* __restrict__ loss) {
    __shared__ float red[16];
    float s = 0.0f;
    for (int64_t k0 = threadIdx.x; k0 < n; k0 += 1024 * 8) {
        float v[8];
        #pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = k0 + 1024 * u < n ? part[k0 + 1024 * u] : 0.0f;
        #pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int w = 0; w < 16; ++w) t += red[w];
        *loss = t * inv_n;
    }
}

// Prior 2: vertex j at min + idx*((max-min)/(n-1)); visible to a camera
// (row-major camera-to-world R, centre c) when p = R^T (x - c) has p_z < 0
// and its projection (focal p_x/(-p_z) + W/2, -focal p_y/(-p_z) + H/2) lies
// in [0, W) x [0, H).
struct VcArgs {
    float mn[3], stepv[3];
    int n[3];
    const float* cams;   // [ncam][12]: R (9, row-major), centre (3)
    int ncam, H, W;
    float focal;
};

__global__ __launch_bounds__(256) void fill_zero_kernel(int* __restrict__ p) { *p = 0; }

__global__ __launch_bounds__(256) void view_count_kernel(VcArgs a, int* __restrict__ counts, int* __restrict__ nmax) {
    const int64_t nv = static_cast<int64_t>(a.n[0]) * a.n[1] * a.n[2];
    const int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (v >= nv) return;
    const int j2 = static_cast<int>(v % a.n[2]), j1 = static_cast<int>((v / a.n[2]) % a.n[1]);
    const int j0 = static_cast<int>(v / (static_cast<int64_t>(a.n[1]) * a.n[2]));
    const float x[3] = {a.mn[0] + j0 * a.stepv[0], a.mn[1] + j1 * a.stepv[1], a.mn[2] + j2 * a.stepv[2]};
    int cnt = 0;
    for (int c = 0; c < a.ncam; ++c) {
        const float* R = a.cams + 12 * c;
        const float dx = x[0] - R[9], dy = x[1] - R[10], dz = x[2] - R[11];
        const float px = R[0] * dx + R[3] * dy + R[6] * dz;
        const float py = R[1] * dx + R[4] * dy + R[7] * dz;
        const float pz = R[2] * dx + R[5] * dy + R[8] * dz;
        const float z = -pz;
        if (!(z > 0.0f)) continue;
        const float u = a.focal * px / z + 0.5f * a.W;
        const float vv = -a.focal * py / z + 0.5f * a.H;
        cnt += (u >= 0.0f && u < static_cast<float>(a.W) && vv >= 0.0f && vv < static_cast<float>(a.H)) ? 1 : 0;
    }
    counts[v] = cnt;
    atomicMax(nmax, cnt);
}

__global__ __launch_bounds__(256) void view_scale_kernel(const int* __restrict__ counts, int64_t nv,
                                                         const int* __restrict__ nmax, float* __restrict__ scale) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (v >= nv) return;
    const int m = *nmax;
    scale[v] = static_cast<float>(counts[v]) / static_cast<float>(m > 0 ? m : 1);
}

__global__ __launch_bounds__(256) void adam_scaled_kernel(float* __restrict__ p, float* __restrict__ g,
                                                          float* __restrict__ m, float* __restrict__ v,
                                                          const float* __restrict__ scale, int64_t n,
                                                          dvgo::AdamCoef c) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    dvgo::AdamCoef ci = c;
    ci.lr = c.lr * scale[i];
    float pi = p[i], mi = m[i], vi = v[i];
    dvgo::adam_update(ci, pi, g[i], mi, vi);
    p[i] = pi;
    m[i] = mi;
    v[i] = vi;
    g[i] = 0.0f;
}

}  // namespace

namespace {

// Workspace of the binned form: the per-ray losses first, as in the other.
struct CoarseWs {
    size_t cell_count, cell_start, scan, cell_rank, head, rec, total;
};

CoarseWs coarse_ws(int32_t B, int64_t cap, int64_t ncell) {
    CoarseWs L;
    size_t off = dvgo_coarse_workspace_bytes(B);
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = dvgo::align_up(off + bytes, 256);
        return o;
    };
    L.cell_count = take(static_cast<size_t>(ncell + 1) * 4);
    L.cell_start = take(static_cast<size_t>(ncell + 1) * 4);
    L.scan = take(cell_scan_bytes(ncell + 1));
    L.cell_rank = take(static_cast<size_t>(cap) * 8);
    L.head = take(static_cast<size_t>(cap) * 32);
    L.rec = take(static_cast<size_t>(cap) * 32);
    L.total = off;
    return L;
}

int64_t coarse_cells(const dvgo_box& b) {
    return static_cast<int64_t>(b.n[0] - 1) * (b.n[1] - 1) * (b.n[2] - 1);
}

}  // namespace

extern "C" {

size_t dvgo_coarse_workspace_bytes(int32_t B) {
    if (B < 0) return 0;
    return dvgo::align_up(static_cast<size_t>(B) * 4, 256) + 256;
}

// The binned form where it is faster, and its workspace (72 bytes a slot) at
// most 1 GiB.  It costs a fixed 35 us and 12 us per million cells, the atomics
// 0.8 us per thousand samples more than it: with capacities of four times the
// samples kept, 256 / 1024 rays in 39^3 cells take 36 / 36 us binned and 20 / 39
// by atomics, 256 / 512 / 1024 rays in 99^3 48 / 53 / 57 and 40 / 51 / 87, in
// 127^3 60 / 64 / 72 and 48 / 63 / 113.
size_t dvgo_coarse_step_workspace_bytes(int32_t B, int64_t capacity, const dvgo_box* grid) {
    if (B < 0 || capacity < 0 || !dvgo::box_ok(grid, 2)) return 0;
    const size_t small = dvgo_coarse_workspace_bytes(B);
    const int64_t ncell = coarse_cells(*grid);
    if (capacity < 100000 + ncell / 40 * 3 || capacity >= (1LL << 31)) return small;
    const size_t binned = coarse_ws(B, capacity, ncell).total;
    return binned - small <= (1ull << 30) ? binned : small;
}

int32_t dvgo_coarse_step(const dvgo_coarse_field* field, const float* rays_o, const float* rays_d,
                         const float* jitter, const float* t_near, const int32_t* perm, const int32_t* ray_offset,
                         const int32_t* sample_k, const int64_t* n_kept, int64_t capacity, int32_t B, int32_t max_samples,
                         float step, const float* bg, const float* target, float w_pt, float w_bg, float* rgb,
                         float* grad_density, float* grad_rgb, float* loss, void* workspace, size_t workspace_bytes,
                         void* stream) {
    if (!field || !field->density || !field->rgb || !dvgo::box_ok(&field->box, 2) || !bg || B < 0 || capacity < 0)
        return DVGO_E_ARG;
    if (!(step > 0.0f) || !(w_pt >= 0.0f) || !(w_bg >= 0.0f) || max_samples < 0) return DVGO_E_ARG;
    if (max_samples > 64 * kMaxSteps) return DVGO_E_UNSUPPORTED;
    if (static_cast<int64_t>(field->box.n[0]) * field->box.n[1] * field->box.n[2] >= (1LL << 31))
        return DVGO_E_UNSUPPORTED;
    if (B > 0 && (!rays_o || !rays_d || !t_near || !perm || !ray_offset || !n_kept || !target || !grad_density ||
                  !grad_rgb || !loss))
        return DVGO_E_ARG;
    if (capacity > 0 && !sample_k) return DVGO_E_ARG;
    if (workspace_bytes < dvgo_coarse_workspace_bytes(B) || (B > 0 && !workspace)) return DVGO_E_CAPACITY;
    if (B == 0) return DVGO_OK;
    CoarseArgs a;
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.jitter = jitter;
    a.t_near = t_near;
    a.perm = perm;
    a.ray_offset = ray_offset;
    a.sample_k = sample_k;
    a.n_kept = n_kept;
    a.cap = capacity;
    a.B = B;
    a.step = step;
    a.g = dvgo::make_grid(field->box);
    a.density = field->density;
    a.rgb = field->rgb;
    a.act_shift = field->act_shift;
    for (int i = 0; i < 3; ++i) a.bg[i] = bg[i];
    a.target = target;
    a.w_pt = w_pt;
    a.w_bg = w_bg;
    a.rgb_out = rgb;
    a.ray_loss = static_cast<float*>(workspace);
    a.grad_density = grad_density;
    a.grad_rgb = grad_rgb;
    a.cell_count = nullptr;
    a.cell_rank = nullptr;
    a.head = nullptr;
    hipStream_t s = dvgo::as_stream(stream);
    // the binned form wherever its workspace is given (16-byte aligned, for
    // its records; positions in the sorted list are 32-bit)
    const int64_t ncell = coarse_cells(field->box);
    const CoarseWs L = coarse_ws(B, capacity, ncell);
    if (workspace_bytes >= L.total && capacity < (1LL << 31) && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0) {
        char* ws = static_cast<char*>(workspace);
        int* start = reinterpret_cast<int*>(ws + L.cell_start);
        float4* rec = reinterpret_cast<float4*>(ws + L.rec);
        a.cell_count = reinterpret_cast<int*>(ws + L.cell_count);
        a.cell_rank = reinterpret_cast<int2*>(ws + L.cell_rank);
        a.head = reinterpret_cast<float4*>(ws + L.head);
        const int64_t cus = dvgo::device_cu_count();
        auto blocks = [&](int64_t work, int64_t most) {
            const int64_t b = (work + 255) / 256;
            return dim3(static_cast<unsigned>(b < 1 ? 1 : b > most ? most : b));
        };
        DVGO_LAUNCH(K_CELL_SCAN, fill_int_kernel, blocks(ncell + 1, cus * 8), dim3(256), 0, s, a.cell_count, ncell + 1, 0);
        if (int32_t st = dvgo::launch_status()) return st;
        DVGO_LAUNCH(K_COARSE_STEP, coarse_step_kernel<true>, dim3(B), dim3(64), 0, s, a);
        if (int32_t st = dvgo::launch_status()) return st;
        if (int32_t st = run_cell_scan(a.cell_count, ncell + 1, ws + L.scan, start, s)) return st;
        if (capacity > 0) {
            DVGO_LAUNCH(K_BIN_PLACE, coarse_place_kernel, blocks(capacity, cus * 16), dim3(256), 0, s, n_kept, capacity,
                        a.cell_rank, start, a.head, rec);
            if (int32_t st = dvgo::launch_status()) return st;
            const int64_t nv = static_cast<int64_t>(field->box.n[0]) * field->box.n[1] * field->box.n[2];
            DVGO_LAUNCH(K_SCATTER, coarse_vertex_kernel, dim3(static_cast<unsigned>((nv + 255) / 256)), dim3(256), 0, s,
                        a.g, start, rec, grad_density, grad_rgb);
            if (int32_t st = dvgo::launch_status()) return st;
        }
    } else {
        DVGO_LAUNCH(K_COARSE_STEP, coarse_step_kernel<false>, dim3(B), dim3(64), 0, s, a);
        if (int32_t st = dvgo::launch_status()) return st;
    }
    DVGO_LAUNCH(K_REDUCE, ray_loss_reduce_kernel, dim3(1), dim3(1024), 0, s, a.ray_loss, B,
                1.0f / static_cast<float>(B), loss);
    return dvgo::launch_status();
}

size_t dvgo_view_counts_workspace_bytes(void) { return 256; }

int32_t dvgo_view_counts(const dvgo_box* box, const float* cams, int32_t ncam, int32_t H, int32_t W, float focal,
                         int32_t* counts, float* lr_scale, void* workspace, size_t workspace_bytes, void* stream) {
    if (!dvgo::box_ok(box, 2) || ncam < 0 || (ncam > 0 && !cams) || H < 1 || W < 1 || !(focal > 0.0f) || !counts ||
        !lr_scale)
        return DVGO_E_ARG;
    if (!workspace || workspace_bytes < dvgo_view_counts_workspace_bytes()) return DVGO_E_CAPACITY;
    const int64_t nv = static_cast<int64_t>(box->n[0]) * box->n[1] * box->n[2];
    if (nv >= (1LL << 31)) return DVGO_E_UNSUPPORTED;
    VcArgs a;
    for (int i = 0; i < 3; ++i) {
        a.mn[i] = box->xyz_min[i];
        volatile float span = box->xyz_max[i] - box->xyz_min[i];
        volatile float nm1 = static_cast<float>(box->n[i] - 1);
        a.stepv[i] = span / nm1;
        a.n[i] = box->n[i];
    }
    a.cams = cams;
    a.ncam = ncam;
    a.H = H;
    a.W = W;
    a.focal = focal;
    int* nmax = static_cast<int*>(workspace);
    hipStream_t s = dvgo::as_stream(stream);
    const unsigned blocks = static_cast<unsigned>((nv + 255) / 256);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(1), 0, s, nmax);
    if (int32_t st = dvgo::launch_status()) return st;
    DVGO_LAUNCH(K_VIEW_COUNT, view_count_kernel, dim3(blocks), dim3(256), 0, s, a, counts, nmax);
    if (int32_t st = dvgo::launch_status()) return st;
    DVGO_LAUNCH(K_VIEW_COUNT, view_scale_kernel, dim3(blocks), dim3(256), 0, s, counts, nv, nmax, lr_scale);
    return dvgo::launch_status();
}

int32_t dvgo_adam_step_scaled(float* p, float* g, float* m, float* v, const float* lr_scale, int64_t n, float lr,
                              float beta1, float beta2, float eps, int32_t t, void* stream) {
    if (n < 0 || (n > 0 && (!p || !g || !m || !v || !lr_scale)) || !dvgo::adam_hyper_ok(beta1, beta2, eps, t))
        return DVGO_E_ARG;
    if (n == 0) return DVGO_OK;
    const dvgo::AdamCoef c = dvgo::adam_coef(lr, beta1, beta2, eps, t);
    DVGO_LAUNCH(K_ADAM, adam_scaled_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0,
                dvgo::as_stream(stream), p, g, m, v, lr_scale, n, c);
    return dvgo::launch_status();
}

}  // extern "C"
