// Voxelization with direct-light injection (Section 4.4 "Voxelization
// Process", Section 5.4.4 "Voxelization"): every triangle is rasterized once
// along its dominant axis onto an N x N viewport; every fragment (pixel centre
// inside the projected triangle) is the voxel (pixel, floor(depth)) and gets
// the Phong light of the surface point without its glossy term (ambient +
// diffuse with the triangle's own normal, distance attenuation) and alpha 1.
//
// Determinism: coverage and depth are decided on vertices snapped to 1/256
// voxel by exact integer edge functions and an exact floor division (a
// centre on an edge belongs to the triangle when the counter-clockwise edge
// runs upward or horizontally leftward, so shared edges are covered once);
// fragments falling into the same voxel are averaged through 64-bit
// fixed-point sums and a count, so the result does not depend on the order in
// which fragments arrive.
//
// Surface attributes (optional): per voxel the average of the fragments' unit
// triangle normals and of their triangle colours, through the same kind of
// fixed-point sums (a further 3D texture of surface normals is what more light
// bounces need, Section 6.2.2; deferred voxel cone tracing keeps albedo and
// normal textures from voxelization, Section 5.1.3).
//
// Launch: the first workgroups of the clearing pass set up the triangles (one thread
// each: the rasterization record and the pixel count of its bounding box, and the
// sums of 1024 counts); a scan turns the counts into offsets (one workgroup for
// up to 4096 triangles, else one workgroup over the sums, then the offsets
// inside each 1024, beside the clearing of the slots); the raster pass then walks the
// flattened pixel space, one lane per bounding-box pixel, each wave finding its
// triangles with a few wide probes of the offsets.  A wall-sized triangle spreads
// over many waves and a thousand one-pixel triangles fill a wave.
//
// Sparse accumulators: only voxels that a fragment reaches get one (most of a
// scene's grid is empty).  The output grids are zero-filled (base first;
// normal and albedo by workgroups of the raster launch of their own); while the
// raster pass runs, the alpha word of a reached voxel in `base` holds the
// index + 1 of its accumulator slot: that of the first fragment's pixel in the
// flattened pixel space, put there by a compare-and-swap.  Only when that space
// has more pixels than there are slots (one per voxel, less 1 in 257 for the
// bits below) are slots taken from a counter (a compare-and-swap to a claim mark, then the index is
// published; fragments that find the mark read the word again until the index
// appears, which follows the claim directly).  A slot is {int64
// r, g, b; uint32 count; uint32 voxel + 1} (32 bytes), and with surface
// attributes {int64 nx, ny, nz, r, g, b} (48 bytes) more.  Only as many slots
// as the triangles' bounding boxes hold pixels (at most one per voxel) are
// cleared, by fill kernels (no memset, so the path can be captured in a
// graph); the resolve pass writes the voxels of the used ones.  (Slots named by
// pixels have gaps, wide ones where triangles fill little of their boxes, so each
// wave of the raster pass leaves the bits of the slots that its 64 pixels claimed,
// and the resolve pass reads no others: 200 triangles
// thinner than a voxel along the diagonals of a 256^3 grid, 6465 of whose 12 million
// slots are used, 259 -> 214 us; with surface attributes 501 -> 443.)
// Which slot a voxel gets depends on arrival order; the integer sums in it do
// not, so the grids are the same bits whatever the order.
//
// (522000 triangles at 256^3, whose floor is the 43 us of clearing the base: 245 us
// with 64-bit coordinates in 152-byte records built in scratch memory, every slot from
// the counter, a binary search per lane and nine launches; 152 us with 32-bit ones and
// slots by pixel; 139 us with the wave's search and the passes side by side.  1102
// triangles with surface attributes: 337 -> 305 us, of which 125 clear the outputs.)
#include "vct_internal.h"

namespace {

constexpr int kSubLog = 8, kSub = 1 << kSubLog;   // subpixels per voxel
constexpr int kCoordLimit = 1 << 19;      // |snapped coordinate| bound of the exact arithmetic
constexpr float kFix = 4294967296.0f;     // 2^32: fixed-point scale of the colour sums
constexpr float kFixMax = 268435456.0f;   // 2^28: per-fragment colour bound of the fixed point

struct VoxArgs {
    int32_t n;
    float origin[3];
    float voxel;          // extent / N
    float snap_scale;     // 256 N / extent, float32
    int32_t n_lights;
    float light_pos[VCT_MAX_LIGHTS][3];
    float light_color[VCT_MAX_LIGHTS][3];
    float att[VCT_MAX_LIGHTS][3];
    float ambient, diffuse;
};

struct VoxAcc {
    unsigned long long r, g, b;
    unsigned int count, voxel;   // voxel: linear voxel index + 1 (0: slot unused)
};

constexpr unsigned int kClaimed = 0xffffffffu;   // alpha word of a voxel whose slot is being taken
constexpr int kMaxSpin = 1 << 24;                // bound of the wait for a claimed voxel's slot

struct SurfAcc {
    unsigned long long n[3], c[3];
};

// (coordinates are below 2^20 in absolute value, so differences fit 32 bits and one instruction multiplies them)
__device__ __forceinline__ long long mul(int32_t a, int32_t b) { return (long long)a * b; }

__device__ __forceinline__ bool top_left(int32_t dx, int32_t dy) { return dy > 0 || (dy == 0 && dx < 0); }

__device__ __forceinline__ unsigned long long to_fixed(float v) {
    v = fminf(fmaxf(v, -kFixMax), kFixMax);
    return (unsigned long long)(long long)rintf(v * kFix);
}

// Rasterization setup of one triangle: snapped, swizzled vertices (counter-
// clockwise), plane coefficients, pixel bounding box, the unit normal of the
// original triangle and its colour.
struct TriSetup {
    int32_t A[3], B[3], C[3];        // (X2, Y2, W) subpixel coordinates
    int32_t i0, j0, w;               // bounding box origin and width in pixels
    long long nx, ny, nw;            // plane: nw W = nw A.w - nx (X - A.x) - ny (Y - A.y), nw > 0
    float n[3], col[3];
    int32_t dom;                     // source axis of W (its X2, Y2 | W: z, y | x; x, z | y; x, y | z)
};
static_assert(sizeof(TriSetup) == 104);

constexpr int kScanBlock = 1024;     // counts per block of the offset scan (256 threads x 4)
constexpr int kScanThreads = 1024;   // threads of the one-workgroup scan of block sums

// Writes the record of triangle t and returns the pixel count of its bounding box
// (0: no record; the raster pass does not look at it).
__device__ __forceinline__ unsigned long long tri_setup(const VoxArgs& a, const float* __restrict__ tris,
                                                        const float* __restrict__ colors, long long t,
                                                        TriSetup* __restrict__ setup) {
    // snapped vertices (float32 arithmetic, round half to even)
    float vf[3][3];
    int32_t s[3][3];
    bool ok = true;
    for (int k = 0; k < 3; ++k)
        for (int i = 0; i < 3; ++i) {
            const float p = tris[t * 9 + k * 3 + i];
            vf[k][i] = p;
            const float u = rintf((p - a.origin[i]) * a.snap_scale);
            ok = ok && isfinite(p) && fabsf(u) <= (float)kCoordLimit;
            s[k][i] = ok ? (int32_t)u : 0;
        }
    if (!ok) return 0;
    // dominant axis of the snapped normal (ties to x, then y, then z)
    int32_t e1[3], e2[3];
    for (int i = 0; i < 3; ++i) {
        e1[i] = s[1][i] - s[0][i];
        e2[i] = s[2][i] - s[0][i];
    }
    const long long nrm[3] = {mul(e1[1], e2[2]) - mul(e1[2], e2[1]), mul(e1[2], e2[0]) - mul(e1[0], e2[2]),
                              mul(e1[0], e2[1]) - mul(e1[1], e2[0])};
    const long long ax = nrm[0] < 0 ? -nrm[0] : nrm[0], ay = nrm[1] < 0 ? -nrm[1] : nrm[1],
                    az = nrm[2] < 0 ? -nrm[2] : nrm[2];
    const int dom = (ax >= ay && ax >= az) ? 0 : (ay >= az ? 1 : 2);
    // projection frame (X2, Y2 | W): x-dominant (z, y | x), y-dominant (x, z | y), z-dominant (x, y | z)
    int32_t V[3][3];
    for (int k = 0; k < 3; ++k) {
        V[k][0] = dom == 0 ? s[k][2] : s[k][0];
        V[k][1] = dom == 1 ? s[k][2] : s[k][1];
        V[k][2] = dom == 0 ? s[k][0] : dom == 1 ? s[k][1] : s[k][2];
    }
    const long long area = mul(V[1][0] - V[0][0], V[2][1] - V[0][1]) - mul(V[1][1] - V[0][1], V[2][0] - V[0][0]);
    if (area == 0) return 0;
    TriSetup r;
    for (int i = 0; i < 3; ++i) {
        r.A[i] = V[0][i];
        r.B[i] = area < 0 ? V[2][i] : V[1][i];
        r.C[i] = area < 0 ? V[1][i] : V[2][i];
    }
    const int32_t h = kSub / 2;
    const int32_t minx = min(r.A[0], min(r.B[0], r.C[0])), maxx = max(r.A[0], max(r.B[0], r.C[0]));
    const int32_t miny = min(r.A[1], min(r.B[1], r.C[1])), maxy = max(r.A[1], max(r.B[1], r.C[1]));
    const int32_t i0 = max(0, -((h - minx) >> kSubLog)), i1 = min(a.n - 1, (maxx - h) >> kSubLog);
    const int32_t j0 = max(0, -((h - miny) >> kSubLog)), j1 = min(a.n - 1, (maxy - h) >> kSubLog);
    if (i1 < i0 || j1 < j0) return 0;
    const int32_t f1[3] = {r.B[0] - r.A[0], r.B[1] - r.A[1], r.B[2] - r.A[2]};
    const int32_t f2[3] = {r.C[0] - r.A[0], r.C[1] - r.A[1], r.C[2] - r.A[2]};
    r.nx = mul(f1[1], f2[2]) - mul(f1[2], f2[1]);
    r.ny = mul(f1[2], f2[0]) - mul(f1[0], f2[2]);
    r.nw = mul(f1[0], f2[1]) - mul(f1[1], f2[0]);
    r.i0 = i0;
    r.j0 = j0;
    r.w = i1 - i0 + 1;
    r.dom = dom;
    // lighting: unit normal of the original triangle as wound
    const float d1[3] = {vf[1][0] - vf[0][0], vf[1][1] - vf[0][1], vf[1][2] - vf[0][2]};
    const float d2[3] = {vf[2][0] - vf[0][0], vf[2][1] - vf[0][1], vf[2][2] - vf[0][2]};
    float tn[3] = {d1[1] * d2[2] - d1[2] * d2[1], d1[2] * d2[0] - d1[0] * d2[2], d1[0] * d2[1] - d1[1] * d2[0]};
    const float l = sqrtf(tn[0] * tn[0] + tn[1] * tn[1] + tn[2] * tn[2]);
    const float il = l > 0.f ? 1.0f / l : 0.f;
    for (int i = 0; i < 3; ++i) {
        r.n[i] = tn[i] * il;
        r.col[i] = colors[t * 3 + i];
    }
    setup[t] = r;
    return (unsigned long long)r.w * (unsigned)(j1 - j0 + 1);
}

// 16-byte stores of a thread of the clearing pass, 16 KB apart and with no loop: 4096
// workgroups in a loop took 65 us longer for a 512^3 base, 16384 of 256 threads 46.
constexpr int kFillStores = 4;

// Zeroes the output grids (n float4 each; normal and albedo may be null) and the slot
// counter, and with its first workgroups sets up the triangles and sums each block of
// kScanBlock pixel counts (offset scan, phase 1): the fill is bound by HBM, 43 us for
// the base of a 256^3 grid, and the set-up of 522000 triangles (17 us alone) runs beside it.
__global__ __launch_bounds__(kScanBlock) void k_begin(VoxArgs a, const float* __restrict__ tris,
                                                      const float* __restrict__ colors, long long n_tris, int tri_blocks,
                                                      TriSetup* __restrict__ setup, unsigned long long* __restrict__ counts,
                                                      unsigned long long* __restrict__ bsum, uint4* __restrict__ base,
                                                      uint4* __restrict__ normal, uint4* __restrict__ albedo, size_t n,
                                                      unsigned int* __restrict__ counter) {
    if ((int)blockIdx.x < tri_blocks) {
        __shared__ unsigned long long s[kScanBlock / 64];
        const long long t = (long long)blockIdx.x * kScanBlock + threadIdx.x;
        unsigned long long v = 0;
        if (t < n_tris) {
            v = tri_setup(a, tris, colors, t, setup);
            counts[t] = v;
        }
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            v = 0;
            for (int i = 0; i < kScanBlock / 64; ++i) v += s[i];
            bsum[blockIdx.x] = v;
        }
        return;
    }
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    const size_t first = (size_t)(blockIdx.x - tri_blocks) * (kFillStores * kScanBlock) + threadIdx.x;
    if (first == 0) *counter = 0u;
#pragma unroll
    for (int k = 0; k < kFillStores; ++k) {
        const size_t i = first + k * kScanBlock;
        if (i >= n) break;
        base[i] = z;
        if (normal) {
            normal[i] = z;
            albedo[i] = z;
        }
    }
}

// Phase 2, one workgroup: bsum[b] becomes the sum of bsum[0..b); *total the sum of all.
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(unsigned long long* __restrict__ bsum, long long nb,
                                                            unsigned long long* __restrict__ total) {
    __shared__ unsigned long long s[kScanThreads];
    const long long per = (nb + kScanThreads - 1) / kScanThreads;
    const long long b = threadIdx.x * per, e = min(b + per, nb);
    unsigned long long own = 0;
    for (long long i = b; i < e; ++i) own += bsum[i];
    s[threadIdx.x] = own;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {   // inclusive Hillis-Steele scan
        const unsigned long long add = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0ull;
        __syncthreads();
        s[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned long long run = s[threadIdx.x] - own;
    for (long long i = b; i < e; ++i) {
        const unsigned long long c = bsum[i];
        bsum[i] = run;
        run += c;
    }
    if (threadIdx.x == kScanThreads - 1) *total = s[kScanThreads - 1];
}

// Phase 3, the first nb workgroups: counts become exclusive offsets, in place (block
// base + prefix inside the block).  The others zero the first min(*total, cap) slots: no
// more can be taken than there are bounding-box pixels (each fragment claims at most
// one voxel) or voxels.
__global__ __launch_bounds__(256) void k_offsets_slots(unsigned long long* __restrict__ c, long long n,
                                                       const unsigned long long* __restrict__ bsum, int nb,
                                                       uint4* __restrict__ acc, uint4* __restrict__ surf,
                                                       const unsigned long long* total_p, unsigned long long cap) {
    if ((int)blockIdx.x >= nb) {
        const unsigned long long used = min(*total_p, cap);
        const uint4 z = make_uint4(0u, 0u, 0u, 0u);
        const size_t first = (size_t)(blockIdx.x - nb) * blockDim.x + threadIdx.x, stride = (size_t)(gridDim.x - nb) * blockDim.x;
        for (size_t i = first; i < used * 2; i += stride) acc[i] = z;
        if (surf)
            for (size_t i = first; i < used * 3; i += stride) surf[i] = z;
        return;
    }
    __shared__ unsigned long long s[256];
    const long long i0 = (long long)blockIdx.x * kScanBlock + threadIdx.x * 4;
    unsigned long long v[4], own = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = i0 + k < n ? c[i0 + k] : 0ull;
        own += v[k];
    }
    s[threadIdx.x] = own;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {   // inclusive Hillis-Steele scan of the thread sums
        const unsigned long long add = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0ull;
        __syncthreads();
        s[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned long long run = bsum[blockIdx.x] + s[threadIdx.x] - own;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i0 + k < n) {
            c[i0 + k] = run;
            run += v[k];
        }
}

// The whole offset scan in one workgroup, for meshes of at most kScanSmall
// triangles (1024 threads x 4 counts), with the same integer sums as the blocked
// scan of larger ones.
constexpr int kScanSmall = 4096;
__global__ __launch_bounds__(1024) void k_scan_small(unsigned long long* __restrict__ c, long long n,
                                                     unsigned long long* __restrict__ total) {
    __shared__ unsigned long long s[1024];
    const long long i0 = (long long)threadIdx.x * 4;
    unsigned long long v[4], own = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = i0 + k < n ? c[i0 + k] : 0ull;
        own += v[k];
    }
    s[threadIdx.x] = own;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {   // inclusive Hillis-Steele scan of the thread sums
        const unsigned long long add = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0ull;
        __syncthreads();
        s[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned long long run = s[threadIdx.x] - own;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i0 + k < n) {
            c[i0 + k] = run;
            run += v[k];
        }
    if (threadIdx.x == 1023) *total = s[1023];
}

// floor(a / b) for b > 0 from a float estimate corrected in exact int64 arithmetic
// (|a| < 2^63, quotients here are below 2^31).
__device__ __forceinline__ long long floor_div_est(long long a, long long b) {
    long long q = (long long)floorf((float)a / (float)b);
    while (q * b > a) --q;
    while ((q + 1) * b <= a) ++q;
    return q;
}

// Orders the LDS accesses of a wave's lanes around it (they execute in order;
// this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
#ifdef VCT_HOST_EMULATION
    (void)__ballot(true);
#else
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#endif
}

// The last t with offs[t] <= g for each lane's g = gw + lane (all lanes of the wave
// call; off: 64 words of LDS of its own).  A binary search is one load after another
// (19 for 522000 triangles); here the wave probes 64 places at a time until it has the
// triangle of its first pixel (4 loads), then holds the 64 offsets from there, in which
// nearly every lane finds its own; the others search on in memory.
__device__ __forceinline__ long long find_triangles(const unsigned long long* __restrict__ offs, long long n_tris,
                                                    unsigned long long gw, int lane, unsigned long long* off) {
    long long lo = 0, hi = n_tris - 1;
    for (long long step = 0; step != 1;) {
        step = (hi - lo + 64) >> 6;
        const long long t = lo + lane * step;
        const bool le = t <= hi && offs[t] <= gw;
        lo += (__popcll(__ballot(le)) - 1) * step;   // (lane 0's is always true)
        hi = min(hi, lo + step - 1);
    }
    const long long t = lo + lane;
    const unsigned long long g = gw + lane;
    wave_sync();   // (the last search's readers)
    off[lane] = t < n_tris ? offs[t] : ~0ull;
    wave_sync();
    int k = 0;
#pragma unroll
    for (int b = 32; b > 0; b >>= 1)
        if (off[k + b] <= g) k += b;
    lo += k;
    if (k == 63) {
        hi = n_tris - 1;
        while (lo < hi) {
            const long long mid = (lo + hi + 1) >> 1;
            if (offs[mid] <= g) lo = mid;
            else hi = mid - 1;
        }
    }
    return lo;
}

// Slots by pixel: one for each, and behind them one bit for each (whether it is used).
__device__ __forceinline__ bool slots_by_pixel(unsigned long long total, unsigned int cap) {
    static_assert(sizeof(VoxAcc) * 8 == 256);
    return total + (total + 255) / 256 <= cap;
}
__device__ __forceinline__ unsigned long long* claim_bits(VoxAcc* acc, unsigned long long total) {
    return reinterpret_cast<unsigned long long*>(acc + total);
}

// One lane per bounding-box pixel of the flattened pixel space (triangle t
// owns the pixels of its box from offs[t] on), in a grid-stride loop; a lane's triangle is
// the last t with offs[t] <= g (a triangle without pixels has offs[t] =
// offs[t + 1] and is passed over).
//
// With surface attributes the first kZeroBlocks workgroups instead zero the
// normal and albedo grids (n float4 each, walked as one index space), which
// nothing reads or writes before the resolve pass: their stores stream to HBM
// while the raster workgroups wait on their atomics.  (Cornell mesh at 256^3:
// 0.41 ms for the call with a separate fill, 0.33 ms with 256 such
// workgroups, 0.35 / 0.38 ms with 512 / 1024, 0.36 / 0.38 ms with 192 / 128.)
constexpr int kRasterBlocks = 2048;
constexpr int kZeroBlocks = 256;

template <bool SURF>
__global__ __launch_bounds__(256) void k_raster(VoxArgs a, const TriSetup* __restrict__ setup,
                                                const unsigned long long* __restrict__ offs, long long n_tris,
                                                const unsigned long long* __restrict__ total_p,
                                                VoxAcc* __restrict__ acc, SurfAcc* __restrict__ surf,
                                                unsigned int* __restrict__ base_words,
                                                unsigned int* __restrict__ counter, uint4* __restrict__ normal,
                                                uint4* __restrict__ albedo, size_t n) {
    int block = (int)blockIdx.x;
    if constexpr (SURF) {
        if (block < kZeroBlocks) {
            const uint4 z = make_uint4(0u, 0u, 0u, 0u);
            for (size_t i = (size_t)block * blockDim.x + threadIdx.x; i < 2 * n; i += (size_t)kZeroBlocks * blockDim.x)
                *(i < n ? normal + i : albedo + (i - n)) = z;
            return;
        }
        block -= kZeroBlocks;
    }
    const unsigned long long total = *total_p;
    const unsigned int cap = (unsigned int)a.n * a.n * a.n;
    const bool direct = slots_by_pixel(total, cap);
    const unsigned long long stride = (unsigned long long)kRasterBlocks * blockDim.x;
    const int32_t h = kSub / 2;
    const float sub_to_world = a.voxel / (float)kSub;
    __shared__ unsigned long long s_off[256];
    const int lane = threadIdx.x & 63;
    for (unsigned long long gw = (unsigned long long)block * blockDim.x + (threadIdx.x & ~63u); gw < total; gw += stride) {
        const long long lo = find_triangles(offs, n_tris, gw, lane, s_off + (threadIdx.x & ~63u));
        const unsigned long long g = gw + lane;
        bool claimed = false;
        if (g < total) do {
            const TriSetup& r = setup[lo];
            const int p = (int)(g - offs[lo]);
            const long long den = r.nw * kSub;
            const int pj_off = (int)((unsigned)p / (unsigned)r.w);
            const int32_t pi = r.i0 + (p - pj_off * r.w), pj = r.j0 + pj_off;
            const int32_t PX = pi * kSub + h, PY = pj * kSub + h;
            const long long ea = mul(r.B[0] - r.A[0], PY - r.A[1]) - mul(r.B[1] - r.A[1], PX - r.A[0]);
            const long long eb = mul(r.C[0] - r.B[0], PY - r.B[1]) - mul(r.C[1] - r.B[1], PX - r.B[0]);
            const long long ec = mul(r.A[0] - r.C[0], PY - r.C[1]) - mul(r.A[1] - r.C[1], PX - r.C[0]);
            const bool in = (ea > 0 || (ea == 0 && top_left(r.B[0] - r.A[0], r.B[1] - r.A[1]))) &&
                            (eb > 0 || (eb == 0 && top_left(r.C[0] - r.B[0], r.C[1] - r.B[1]))) &&
                            (ec > 0 || (ec == 0 && top_left(r.A[0] - r.C[0], r.A[1] - r.C[1])));
            if (!in) break;
            const long long wnum = r.nw * r.A[2] - r.nx * (PX - r.A[0]) - r.ny * (PY - r.A[1]);
            if (wnum < 0) break;                                  // depth below the grid
            const long long layer = floor_div_est(wnum, den);
            if (layer >= a.n) break;
            const int32_t lay = (int32_t)layer;
            const int32_t v[3] = {r.dom == 0 ? lay : pi, r.dom == 0 ? pj : r.dom == 1 ? lay : pj, r.dom == 0 ? pi : r.dom == 1 ? pj : lay};
            const float fx = (float)PX, fy = (float)PY, fw = (float)wnum / (float)r.nw;
            const float sub[3] = {r.dom == 0 ? fw : fx, r.dom == 0 ? fy : r.dom == 1 ? fw : fy, r.dom == 0 ? fx : r.dom == 1 ? fy : fw};
            const float pos[3] = {a.origin[0] + sub[0] * sub_to_world, a.origin[1] + sub[1] * sub_to_world,
                                  a.origin[2] + sub[2] * sub_to_world};
            float lr = 0.f, lg = 0.f, lb = 0.f;
            for (int l = 0; l < a.n_lights; ++l) {
                const float dx = a.light_pos[l][0] - pos[0], dy = a.light_pos[l][1] - pos[1],
                            dz = a.light_pos[l][2] - pos[2];
                const float dist = sqrtf(dx * dx + dy * dy + dz * dz);
                const float lam = dist > 0.f ? fmaxf((dx * r.n[0] + dy * r.n[1] + dz * r.n[2]) / dist, 0.0f) : 0.0f;
                const float at = 1.0f / (a.att[l][0] + a.att[l][1] * dist + a.att[l][2] * dist * dist);
                const float kk = (a.ambient + a.diffuse * lam) * at;
                lr += kk * a.light_color[l][0];
                lg += kk * a.light_color[l][1];
                lb += kk * a.light_color[l][2];
            }
            const unsigned int vi = ((unsigned)v[2] * a.n + v[1]) * a.n + v[0];   // (< 2^30)
            // the voxel's slot: its alpha word in base, claimed by the first fragment
            unsigned int* word = base_words + (size_t)vi * 4 + 3;
            unsigned int s = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // (a voxel is claimed once, so at most n^3 slots are taken; the
            // bound on s below only keeps a word that held anything else, were
            // base to alias another buffer, from indexing past the slots)
            if (s == 0u && direct) {
                s = atomicCAS(word, 0u, (unsigned int)g + 1u);
                if (s == 0u) {
                    s = (unsigned int)g + 1u;
                    claimed = true;
                    acc[g].voxel = vi + 1u;   // read by the resolve pass only
                }
            } else if (s == 0u) {
                s = atomicCAS(word, 0u, kClaimed);
                if (s == 0u) {
                    const unsigned int slot = atomicAdd(counter, 1u);
                    if (slot < cap) acc[slot].voxel = vi + 1u;
                    s = slot + 1u;
                    atomicExch(word, s);
                }
            }
            if (!direct)
                for (int spin = 0; s == kClaimed && spin < kMaxSpin; ++spin)
                    s = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (s > cap) break;   // (not reached: see above; a claim is published right away)
            VoxAcc* q = acc + (s - 1u);
            atomicAdd(&q->r, to_fixed(lr * r.col[0]));
            atomicAdd(&q->g, to_fixed(lg * r.col[1]));
            atomicAdd(&q->b, to_fixed(lb * r.col[2]));
            atomicAdd(&q->count, 1u);
            if constexpr (SURF) {
                SurfAcc* u = surf + (s - 1u);
                for (int i = 0; i < 3; ++i) {
                    atomicAdd(&u->n[i], to_fixed(r.n[i]));
                    atomicAdd(&u->c[i], to_fixed(r.col[i]));
                }
            }
        } while (false);
        if (direct) {
            const unsigned long long bits = __ballot(claimed);
            if (lane == 0) claim_bits(acc, total)[gw >> 6] = bits;
        }
    }
}

// One thread per slot: writes the voxels of the used ones in the output grids (the
// others keep the zeros of k_begin and of the raster launch's fill).
template <bool SURF>
__global__ __launch_bounds__(256) void k_resolve(VoxAcc* __restrict__ acc, const SurfAcc* __restrict__ surf,
                                                 const unsigned int* __restrict__ counter,
                                                 const unsigned long long* __restrict__ total_p, unsigned int cap,
                                                 float4* __restrict__ base,
                                                 float4* __restrict__ normal, float4* __restrict__ albedo) {
    const unsigned long long total = *total_p;
    const bool direct = slots_by_pixel(total, cap);
    const unsigned int used = direct ? (unsigned int)total : min(*counter, cap);
    const unsigned long long* bits = claim_bits(acc, total);
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    constexpr int kAhead = 4;   // slots whose bits a thread reads at a time
    for (size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i0 < used; i0 += kAhead * stride) {
        unsigned long long word[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) word[k] = !direct ? ~0ull : i0 + k * stride < used ? bits[(i0 + k * stride) >> 6] : 0ull;
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const size_t i = i0 + k * stride;
            if (i >= used || !(word[k] >> (i & 63) & 1ull)) continue;
            const VoxAcc q = acc[i];
            if (q.voxel == 0u) continue;
            const size_t v = (size_t)q.voxel - 1u;
            const float inv = 1.0f / ((float)q.count * kFix);
            base[v] = make_float4((float)(long long)q.r * inv, (float)(long long)q.g * inv, (float)(long long)q.b * inv,
                                  1.0f);
            if constexpr (SURF) {
                const SurfAcc u = surf[i];
                normal[v] = make_float4((float)(long long)u.n[0] * inv, (float)(long long)u.n[1] * inv,
                                        (float)(long long)u.n[2] * inv, 1.0f);
                albedo[v] = make_float4((float)(long long)u.c[0] * inv, (float)(long long)u.c[1] * inv,
                                        (float)(long long)u.c[2] * inv, 1.0f);
            }
        }
    }
}

}  // namespace

size_t vct_voxelize_acc_bytes(int n, bool surface) {
    return (size_t)n * n * n * (sizeof(VoxAcc) + (surface ? sizeof(SurfAcc) : 0));
}

size_t vct_voxelize_workspace_size(int n, long long n_tris, bool surface) {
    return vct_voxelize_acc_bytes(n, surface) + (size_t)n_tris * (sizeof(TriSetup) + 8) + 256 +
           (size_t)((n_tris + kScanBlock - 1) / kScanBlock) * 8;
}

namespace {

// Workspace: room for one accumulator slot per voxel (with surface attributes,
// the surface sums of every slot follow), then per-triangle setup records, the
// pixel offsets, the pixel total, the slot counter and the block sums of the
// offset scan.  The counter has a 128-byte line to itself: it lay beside the last
// offsets and the total, which every wave of the raster pass reads, unless n_tris was a
// multiple of 8, and each atomic took their line away from the other chips (401 thin
// triangles along a 256^3 grid's diagonal, more pixels than slots: 2237 us, now 744).
struct VoxWorkspace {
    VoxAcc* acc;
    SurfAcc* surf;
    TriSetup* setup;
    unsigned long long *offs, *total;
    unsigned int* counter;
    unsigned long long* bsum;
};

VoxWorkspace vox_workspace(void* ws, int n, long long n_tris, bool surface) {
    constexpr uintptr_t kLine = 128;
    const size_t nvox = (size_t)n * n * n;
    VoxWorkspace w;
    w.acc = static_cast<VoxAcc*>(ws);
    w.surf = surface ? reinterpret_cast<SurfAcc*>(w.acc + nvox) : nullptr;
    w.setup = reinterpret_cast<TriSetup*>(static_cast<char*>(ws) + vct_voxelize_acc_bytes(n, surface));
    w.offs = reinterpret_cast<unsigned long long*>(w.setup + n_tris);
    w.total = w.offs + n_tris;
    w.counter = reinterpret_cast<unsigned int*>(((uintptr_t)(w.total + 1) + kLine - 1) & ~(kLine - 1));
    w.bsum = w.total + 32;      // (the 256 bytes before it hold the total and the counter)
    return w;
}

}  // namespace

hipError_t vct_launch_voxelize(const vct_grid* g, const float* tris, const float* colors, long long n_tris,
                               const vct_voxelize_params* p, float* base, float* normal, float* albedo, void* ws,
                               hipStream_t st, EventSink& es) {
    const bool surface = normal != nullptr;
    VoxArgs a{};
    a.n = g->n;
    for (int i = 0; i < 3; ++i) a.origin[i] = g->origin[i];
    a.voxel = (float)((double)g->extent / g->n);
    a.snap_scale = (float)((double)kSub * g->n / (double)g->extent);
    a.n_lights = p->n_lights;
    for (int l = 0; l < p->n_lights; ++l)
        for (int i = 0; i < 3; ++i) {
            a.light_pos[l][i] = p->light_pos[l][i];
            a.light_color[l][i] = p->light_color[l][i];
            a.att[l][i] = p->attenuation[l][i];
        }
    a.ambient = p->ambient;
    a.diffuse = p->diffuse;
    const size_t nvox = (size_t)g->n * g->n * g->n;
    const auto [acc, surf, setup, offs, total, counter, bsum] = vox_workspace(ws, g->n, n_tris, surface);
    const long long nb = (n_tris + kScanBlock - 1) / kScanBlock;
    const int fill_blocks = (int)((nvox + kFillStores * kScanBlock - 1) / (kFillStores * kScanBlock));
    es.mark(st);
    // (with triangles, the raster pass zeroes the normal and albedo grids)
    hipLaunchKernelGGL(k_begin, dim3((unsigned)(nb + fill_blocks)), dim3(kScanBlock), 0, st, a, tris, colors, n_tris, (int)nb,
                       setup, offs, bsum, reinterpret_cast<uint4*>(base),
                       reinterpret_cast<uint4*>(n_tris > 0 ? nullptr : normal),
                       reinterpret_cast<uint4*>(n_tris > 0 ? nullptr : albedo), nvox, counter);
    es.mark(st);
    if (n_tris > 0) {
        const bool small = n_tris <= kScanSmall;
        if (small)
            hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, st, offs, n_tris, total);
        else
            hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanThreads), 0, st, bsum, nb, total);
        const int off_blocks = small ? 0 : (int)nb;
        hipLaunchKernelGGL(k_offsets_slots, dim3((unsigned)(off_blocks + 1024)), dim3(256), 0, st, offs, n_tris, bsum,
                           off_blocks, reinterpret_cast<uint4*>(acc), reinterpret_cast<uint4*>(surf), total,
                           (unsigned long long)nvox);
        unsigned int* words = reinterpret_cast<unsigned int*>(base);
        if (surface)
            hipLaunchKernelGGL(k_raster<true>, dim3(kZeroBlocks + kRasterBlocks), dim3(256), 0, st, a, setup, offs,
                               n_tris, total, acc, surf, words, counter, reinterpret_cast<uint4*>(normal),
                               reinterpret_cast<uint4*>(albedo), nvox);
        else
            hipLaunchKernelGGL(k_raster<false>, dim3(kRasterBlocks), dim3(256), 0, st, a, setup, offs, n_tris, total,
                               acc, surf, words, counter, nullptr, nullptr, nvox);
    }
    es.mark(st);
    if (n_tris > 0) {
        if (surface)
            hipLaunchKernelGGL(k_resolve<true>, dim3(1024), dim3(256), 0, st, acc, surf, counter, total, (unsigned)nvox,
                               reinterpret_cast<float4*>(base), reinterpret_cast<float4*>(normal),
                               reinterpret_cast<float4*>(albedo));
        else
            hipLaunchKernelGGL(k_resolve<false>, dim3(1024), dim3(256), 0, st, acc, surf, counter, total, (unsigned)nvox,
                               reinterpret_cast<float4*>(base), nullptr, nullptr);
    }
    es.mark(st);
    return hipGetLastError();
}
