// Forward cone trace: one lane per pixel, each lane marches all cones of its
// pixel (u diffuse, specular, occlusion) and writes the 8-float epilogue
// (D.rgb, D.a, S.rgb, O).  Sections 4.2, 4.3.2, 4.5 and 5.4.4; with an
// anisotropic pyramid the samples weight its directional levels by the cone
// axis (Section 5.1.3).
//
// Launch: 256-thread workgroups over 16x16-pixel tiles (a wave is an 8x8
// quadrant, so the 64 lanes of a wave start from neighbouring surface points
// and, for the fixed-aperture cones, step through the same LOD schedule),
// tiles ordered so that each XCD gets a contiguous run of the image.
#include "march.h"

namespace {

using namespace vct;

// COUNT: no output; count[0] += the cone samples taken, and with two
// counters count[1] += those that read two levels.
template <int DT, bool COUNT, bool ANISO>
__global__ __launch_bounds__(256) void k_trace(TraceArgs a, float4* __restrict__ out,
                                               unsigned long long* __restrict__ count, int n_counts) {
    __shared__ LevelTable T;
    __shared__ DirSlot<ANISO> D;
    __shared__ unsigned long long s_cnt[2];
    load_level_table<kTapLog<DT>>(a, &T);
    load_dir_table<kTapLog<DT>>(a, &D);
    if (COUNT && threadIdx.x < 2) s_cnt[threadIdx.x] = 0;
    __syncthreads();

    const int tile = xcd_tile(blockIdx.x, a.n_tiles);
    int view, y, x;
    tile_pixel(a, tile, threadIdx.x, view, y, x);
    const bool inb = x < a.w && y < a.h;
    unsigned int ksum = 0, k2sum = 0;
    float4 o0, o1;
    const size_t pix = ((size_t)view * a.h + y) * a.w + x;
    if (inb) trace_pixel<DT, ANISO>(a, T, view, pix, o0, o1, ksum, k2sum, dir_ptr(D));
    if constexpr (COUNT) {
        if (ksum) atomicAdd(&s_cnt[0], (unsigned long long)ksum);
        if (k2sum) atomicAdd(&s_cnt[1], (unsigned long long)k2sum);
        __syncthreads();
        if ((int)threadIdx.x < n_counts && s_cnt[threadIdx.x]) atomicAdd(&count[threadIdx.x], s_cnt[threadIdx.x]);
    } else {
        if (inb) {
            out[2 * pix] = o0;
            out[2 * pix + 1] = o1;
        }
    }
}

// The forward of small frames (Tile8).
template <int DT, bool ANISO>
__global__ __launch_bounds__(64 * kSplitWaves) void k_trace_split(TraceArgs a, float4* __restrict__ out) {
    __shared__ LevelTable T;
    __shared__ DirSlot<ANISO> D;
    __shared__ float4 s_end[VCT_MAX_DIFFUSE + 2][64];
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
    take_items(&s_next, a.n_diffuse + 2, [&](int i) {
        const int slot = item_slot(a, i);
        if (!valid || !slot_enabled(a, slot)) return;
        const MarchResult m = march<DT, ANISO, kShareFootprint<DT>>(a, T, cone_for_slot(a, P, slot, cam), dir_ptr(D));
        s_end[slot][lane] = make_float4(m.r, m.g, m.b, m.a);
    });
    __syncthreads();
    if (threadIdx.x < 64 && inb) {
        float4 o0 = make_float4(0.f, 0.f, 0.f, 0.f), o1 = o0;
        if (valid)
            for (int slot = 0; slot < a.n_diffuse + 2; ++slot)
                if (slot_enabled(a, slot)) {
                    const float4 m = s_end[slot][lane];
                    add_slot(a, slot, m.x, m.y, m.z, m.w, o0, o1);
                }
        out[2 * pix] = o0;
        out[2 * pix + 1] = o1;
    }
}

__global__ void k_zero_u64(unsigned long long* p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

template <int DT, bool ANISO>
hipError_t run_trace(const TraceArgs& a, float* out, unsigned long long* count, int n_counts, hipStream_t s,
                     EventSink& es) {
    dim3 grid(a.n_tiles), block(256);
    if (count) {
        es.mark(s);
        hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, s, count, n_counts);
        if (a.n_tiles > 0) {
            es.mark(s);
            hipLaunchKernelGGL((k_trace<DT, true, ANISO>), grid, block, 0, s, a, nullptr, count, n_counts);
        }
    } else if (a.n_tiles > 0) {
        es.mark(s);
        if (vct_split_forward(a))
            hipLaunchKernelGGL((k_trace_split<DT, ANISO>), dim3(tiles8(a).n), dim3(64 * kSplitWaves), 0, s, a,
                               reinterpret_cast<float4*>(out));
        else
            hipLaunchKernelGGL((k_trace<DT, false, ANISO>), grid, block, 0, s, a, reinterpret_cast<float4*>(out),
                               nullptr, 0);
    }
    es.mark(s);
    return hipGetLastError();
}

template <int DT>
hipError_t run_trace_any(const TraceArgs& a, float* out, unsigned long long* count, int n_counts, hipStream_t s,
                         EventSink& es) {
    return a.aniso ? run_trace<DT, true>(a, out, count, n_counts, s, es)
                   : run_trace<DT, false>(a, out, count, n_counts, s, es);
}

}  // namespace

hipError_t vct_launch_trace(const TraceArgs& a, int dtype, float* out, unsigned long long* count, int n_counts,
                            hipStream_t s, EventSink& es) {
    return vct_dispatch_dt(dtype, a.wide != 0, [&](auto dt) {
        return run_trace_any<decltype(dt)::value>(a, out, count, n_counts, s, es);
    });
}
