// Final shading with the thesis's cone variants (Section 5.4.4, "Cone Tracing"):
// per G-buffer pixel, u diffuse cones (optionally stopping at the first
// sample whose alpha exceeds a threshold and returning its colour), one
// specular cone weighted per light by the angular-grace BRDF, and one
// occlusion cone per light (optionally with each sampled alpha scaled by a
// Hermite step of sqrt(distance) times a shadow strength), combined as
//   L = o_min * sum_q w_q C_diff,q + sum_s f_spec,s C_spec
//       + sum_s V_s (c_d i_d,s max(0, L_s.N) + c_s i_s,s max(0, R_s.w)^shininess),
// V_s = 1 - occlusion alpha, o_min = min_s V_s.  Output float4 (L.rgb, o_min).
//
// The specular cone is traced once: every light's specular cone has the same
// axis and aperture, so the per-light traces of the thesis are one trace
// weighted by the sum of the per-light BRDF values.
//
// Launch: the tiles, waves and XCD order of the forward trace.  With an
// anisotropic pyramid every cone samples its directional levels (Section 5.1.3).
#include "shade_pixel.h"

namespace {

using namespace vct;

// COUNT: instead of the shaded pixels, add the number of cone samples every
// march takes (diffuse, specular, one occlusion cone per light) to *count.
template <int DT, bool ANISO, bool COUNT>
__global__ __launch_bounds__(256) void k_shade(TraceArgs a, ShadeArgs s, float4* __restrict__ out,
                                               unsigned long long* __restrict__ count) {
    __shared__ LevelTable T;
    __shared__ DirSlot<ANISO> D;
    __shared__ unsigned long long s_cnt;
    load_level_table<kTapLog<DT>>(a, &T);
    load_dir_table<kTapLog<DT>>(a, &D);
    if (COUNT && threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    const int tile = xcd_tile(blockIdx.x, a.n_tiles);
    int view, y, x;
    tile_pixel(a, tile, threadIdx.x, view, y, x);
    const bool inb = x < a.w && y < a.h;
    const size_t pix = ((size_t)view * a.h + y) * a.w + x;
    unsigned int n = 0;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (inb) {
        const float4 nr = a.normal[pix];
        if (nr.w != 0.0f) v = shade_pixel<DT, ANISO>(a, T, dir_ptr(D), s, view, pix, nr, n);
    }
    if constexpr (COUNT) {
        if (n) atomicAdd(&s_cnt, (unsigned long long)n);
        __syncthreads();
        if (threadIdx.x == 0 && s_cnt) atomicAdd(count, s_cnt);
    } else {
        if (inb) out[pix] = v;
    }
}

// The shading of small frames (Tile8 in march.h): items are the specular cone,
// the lights' occlusion cones, then the diffuse cones.  First-hit cones and faded occlusion
// cones are shorter than a trace's, so the specular one soon is all the time, and
// frames gain up to 400 tiles only (64^3, float16, five cones and one light: 82 -> 73 us at
// 272 x 256, 93 -> 85 at 400 x 256, 93 -> 102 at 360 x 360, 529 tiles; four and three: 103 ->
// 74, 112 -> 96; 256^3, a cone and two lights, 400 x 256: 118 -> 122, 113 -> 113 in float16).  Directional
// float32 pyramids are marched slower from here, by half on some frames (64^3, 8 x 32 x 32,
// five and one: 163 -> 184 us; 256^3, 256 x 256: 202 -> 277), and keep one lane a pixel.
template <int DT, bool ANISO>
constexpr bool kShadeSplit = !(ANISO && (DT & ~VCT_WIDE) == VCT_F32);
constexpr int kShadeSplitTiles = 400;
template <int DT, bool ANISO>
__global__ __launch_bounds__(64 * kSplitWaves, 4) void k_shade_split(TraceArgs a, ShadeArgs s, float4* __restrict__ out) {
    __shared__ LevelTable T;
    __shared__ DirSlot<ANISO> D;
    __shared__ float s_col[VCT_MAX_DIFFUSE + 1][3][64];   // specular, diffuse
    __shared__ float s_occ[VCT_MAX_LIGHTS][64];
    __shared__ int s_next;
    load_level_table<kTapLog<DT>>(a, &T);
    load_dir_table<kTapLog<DT>>(a, &D);
    if (threadIdx.x == 0) s_next = 0;
    __syncthreads();
    const Tile8 tl = tiles8(a);
    const int lane = threadIdx.x & 63;
    int view, y, x;
    tile8_pixel(tl, xcd_tile(blockIdx.x, tl.n), lane, view, y, x);
    const bool inb = x < a.w && y < a.h;
    const size_t pix = inb ? ((size_t)view * a.h + y) * a.w + x : 0;
    const float4 nr = inb ? a.normal[pix] : make_float4(0.f, 0.f, 0.f, 0.f);
    const bool valid = nr.w != 0.0f;
    PixelSetup P;
    float3 cam = make_float3(0.f, 0.f, 0.f);
    if (valid) {
        P = pixel_setup(a, a.pos_rough[pix], nr);
        cam = make_float3(a.cam_pos[3 * view], a.cam_pos[3 * view + 1], a.cam_pos[3 * view + 2]);
    }
    take_items(&s_next, 1 + s.n_lights + a.n_diffuse, [&](int i) {
        if (!valid) return;
        unsigned int n = 0;
        if (i >= 1 && i <= s.n_lights) {
            s_occ[i - 1][lane] = shade_occlusion<DT, ANISO>(a, T, dir_ptr(D), s, P, i - 1, n);
            return;
        }
        float3 c;
        if (i == 0) {
            const MarchResult m = march<DT, ANISO, kShareFootprint<DT>>(a, T, cone_for_slot(a, P, a.n_diffuse, cam), dir_ptr(D));
            c = make_float3(m.r, m.g, m.b);
        } else {
            c = shade_diffuse<DT, ANISO>(a, T, dir_ptr(D), s, P, cam, i - 1 - s.n_lights, n);
        }
        const int at = i == 0 ? 0 : i - s.n_lights;
        s_col[at][0][lane] = c.x;
        s_col[at][1][lane] = c.y;
        s_col[at][2][lane] = c.z;
    });
    __syncthreads();
    if (threadIdx.x < 64 && inb) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (valid) {
            float3 d = make_float3(0.f, 0.f, 0.f);
            for (int q = 0; q < a.n_diffuse; ++q) {
                const float wq = a.weight[q];
                d.x = __builtin_fmaf(wq, s_col[1 + q][0][lane], d.x);
                d.y = __builtin_fmaf(wq, s_col[1 + q][1][lane], d.y);
                d.z = __builtin_fmaf(wq, s_col[1 + q][2][lane], d.z);
            }
            v = shade_combine(s, P, cam, s.material[pix], d,
                              make_float3(s_col[0][0][lane], s_col[0][1][lane], s_col[0][2][lane]),
                              [&](int l) { return s_occ[l][lane]; });
        }
        out[pix] = v;
    }
}

__global__ void k_zero_count(unsigned long long* p) { *p = 0ull; }

template <int DT, bool ANISO>
void launch_shade(const TraceArgs& a, const ShadeArgs& s, float* out, unsigned long long* count, hipStream_t st) {
    if (count)
        hipLaunchKernelGGL((k_shade<DT, ANISO, true>), dim3(a.n_tiles), dim3(256), 0, st, a, s, nullptr, count);
    else if (kShadeSplit<DT, ANISO> && a.n_tiles <= min(VCT_SPLIT_FORWARD_TILES, kShadeSplitTiles) &&
             s.n_lights + a.n_diffuse > 0) {
        if constexpr (kShadeSplit<DT, ANISO>)
            hipLaunchKernelGGL((k_shade_split<DT, ANISO>), dim3(tiles8(a).n), dim3(64 * kSplitWaves), 0, st, a, s,
                               reinterpret_cast<float4*>(out));
    } else
        hipLaunchKernelGGL((k_shade<DT, ANISO, false>), dim3(a.n_tiles), dim3(256), 0, st, a, s,
                           reinterpret_cast<float4*>(out), nullptr);
}

template <int DT>
hipError_t run_shade(const TraceArgs& a, const ShadeArgs& s, float* out, unsigned long long* count, hipStream_t st,
                     EventSink& es) {
    if (count) {
        es.mark(st);
        hipLaunchKernelGGL(k_zero_count, dim3(1), dim3(1), 0, st, count);
    }
    if (a.n_tiles > 0) {
        es.mark(st);
        if (a.aniso)
            launch_shade<DT, true>(a, s, out, count, st);
        else
            launch_shade<DT, false>(a, s, out, count, st);
    }
    es.mark(st);
    return hipGetLastError();
}

}  // namespace

hipError_t vct_launch_shade(const TraceArgs& a, int dtype, const vct_shade_params* p, const float* material,
                            float* out, unsigned long long* count, hipStream_t st, EventSink& es) {
    ShadeArgs s{};
    s.n_lights = p->n_lights;
    const double scale = (double)a.scale_hi + (double)a.scale_lo;
    for (int l = 0; l < p->n_lights; ++l)
        for (int i = 0; i < 3; ++i) {
            const double lt = ((double)p->light_pos[l][i] - (double)a.origin[i]) * scale;
            s.light_tex[l][i][0] = (float)lt;
            s.light_tex[l][i][1] = (float)(lt - (double)s.light_tex[l][i][0]);
            s.light_pos[l][i] = p->light_pos[l][i];
            s.light_diffuse[l][i] = p->light_diffuse[l][i];
            s.light_specular[l][i] = p->light_specular[l][i];
        }
    for (int i = 0; i < 3; ++i) s.specular_color[i] = p->specular_color[i];
    s.first_hit = p->diffuse_first_hit != 0;
    s.falloff = p->occlusion_falloff != 0;
    s.brdf = p->specular_brdf != 0;
    s.first_hit_alpha = p->first_hit_alpha;
    s.shadow_strength = p->shadow_strength;
    s.grace = p->grace_per_shininess;
    s.q = p->shininess_falloff;
    s.material = reinterpret_cast<const float4*>(material);
    return vct_dispatch_dt(dtype, a.wide != 0,
                           [&](auto dt) { return run_shade<decltype(dt)::value>(a, s, out, count, st, es); });
}
