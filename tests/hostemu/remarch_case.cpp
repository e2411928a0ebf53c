// The cones of the scatter pass's re-march against those of the forward that keeps lane
// states, bit for bit, for random pixels; exits 1 if one differs.
#include "emu.h"
#include "bwd_pixel.h"

using namespace vct;

int main() {
    unsigned int s = 1;
    auto uni = [&](float lo, float hi) {
        s = s * 1664525u + 1013904223u;
        return lo + (hi - lo) * (float)(s >> 8) * 0x1p-24f;
    };
    TraceArgs a{};
    a.n = 64;
    a.scale_hi = 64.0f;
    a.voxel = 1.0f / 64;
    a.n_diffuse = 2;
    a.enable_spec = a.enable_occ = 1;
    const float dirs[2][3] = {{0.f, 0.f, 1.f}, {0.6f, -0.3f, 0.5f}};
    for (int q = 0; q < 2; ++q) {
        a.weight[q] = 0.5f;
        for (int i = 0; i < 3; ++i) a.dir[q][i] = dirs[q][i];
    }
    a.diffuse_aperture = a.spec_aperture_scale = a.occ_aperture = 1.0471976f;
    for (int i = 0; i < 3; ++i) a.light_tex[i][0] = 30.0f + 3.0f * i;
    a.normal_offset = a.max_dist = a.alpha_thresh = 1.0f;
    a.step_factor = 0.5f;
    a.max_steps = 130;
    int bad = 0;
    const int n = 20000;
    for (int k = 0; k < n; ++k) {
        const float4 pr = make_float4(uni(0, 1), uni(0, 1), uni(0, 1), uni(0.05f, 1));
        const float4 nr = make_float4(uni(-1, 1), uni(-1, 1), uni(-1, 1), 1.0f);
        const float3 cam = make_float3(uni(0, 1), uni(0, 1), uni(0, 1));
        const float4 g = make_float4(1, 1, 1, 1);
        const PixelSetup P = pixel_setup(a, pr, nr);
        for (int slot = 0; slot < a.n_diffuse + 2; ++slot) {
            const Cone f = cone_for_slot<true>(a, P, slot, cam);   // (as pass 1 and the saving forward call it)
            Pass2Lane L;
            pass2_init(a, P, cam, g, g, zero_lane_state(), slot, L);
            const float u[8] = {f.Wx, f.Wy, f.Wz, f.two_tan, f.tmax, f.Ox.hi, f.Oy.hi, f.Oz.hi};
            const float v[8] = {L.c.Wx, L.c.Wy, L.c.Wz, L.c.two_tan, L.c.tmax, L.c.Ox.hi, L.c.Oy.hi, L.c.Oz.hi};
            if (memcmp(u, v, sizeof u) != 0 && ++bad < 5)
                printf("pixel %d cone %d: axis %a %a %a, re-march %a %a %a\n", k, slot, u[0], u[1], u[2], v[0], v[1], v[2]);
        }
    }
    printf("%d of %d pixels have a cone that differs\n", bad, n);
    return bad != 0;
}
