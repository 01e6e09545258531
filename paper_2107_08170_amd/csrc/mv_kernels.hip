// HIP kernels (gfx950 / CDNA4) of the batched voxel-world renderer.
//
// Hot path (paper Sec. 3.2, Eq. 2: O = Render(S), all N*A views in one GPU request):
//   pack      : material ids -> occupancy "bit rows" along x and along y, and palette x face intensity ->
//               per-environment colour table (once per world upload)
//   cameras   : (x,y,z,yaw,pitch) -> 64-byte camera records (float64 trig, float32 result)
//   render    : a workgroup stages one environment's bit rows in LDS (plus mirrored copies, so that
//               every ray scans towards increasing bit positions); each wave renders 8x8-pixel
//               tiles, one pixel ray per lane.  The traversal is a DDA over the (v,z) rows the ray
//               passes through, where u is the ray's dominant horizontal axis: all cells the ray
//               covers inside one row are tested with a single 64-bit shift.  Colour and depth
//               leave as row-major dword stores.
// No MFMA anywhere: nothing on this path is a dense contraction.
#include "mv_internal.h"

#include <math.h>
#include <atomic>
#include <type_traits>

namespace mv {

// ------------------------------------------------------------------------------------------
// layout helpers (host)
// ------------------------------------------------------------------------------------------
GridLayout make_layout(int X, int Y, int Z)
{
    GridLayout g{};
    g.X = X; g.Y = Y; g.Z = Z;
    g.rowwords_x = (X + 63) / 64;
    g.rowwords_y = (Y + 63) / 64;
    g.xrow_words = Z * Y * g.rowwords_x;
    g.yrow_words = Z * X * g.rowwords_y;
    g.env_words = g.xrow_words + g.yrow_words;
    g.fast = (X <= 64 && Y <= 64) ? 1 : 0;
    return g;
}

constexpr int kScanClasses = 16;        // (dominant axis) x (direction along u, v, z)
// bytes between scan-class records in LDS (80 used, 16 more with the coarse level, 32 more for cameras outside): 28 dwords, so
// that the sixteen records start in sixteen different banks (a tile whose rays fall into several classes reads several records
// at once; 128 bytes apart they collided: render +0.6 %)
constexpr int kClassStride = 112;

static size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }

// LDS map (bytes):  [16 scan-class records, 112 B apart] | [sx: W floats][one RowRecord per image row] |
//                   [colour table 7*(M+1) dwords] | bit rows
// fast grids stage four row arrays (x, x mirrored, y, y mirrored) of `staged_layers` layers each.  With the coarse
// level, four more arrays follow: the OR of each pair of neighbouring rows of a layer.
// Grids wider than 64 voxels stage x and y rows of `staged_layers` layers for the window scan, which reads a row in
// either direction (mirrored copies would leave room for half as many workgroups); where those do not fit, all x rows
// for the per-cell tracer.
struct LdsMap {
    uint32_t scalars, classes, lut, rows;
    uint32_t total;
};

static LdsMap lds_map(const GridLayout& g, int W, int H, int materials_plus_one, int staged_layers, bool coarse, bool window)
{
    LdsMap m{};
    size_t off = 0;
    m.classes = (uint32_t)off; off += kScanClasses * kClassStride;
    m.scalars = (uint32_t)off; off = align16(off + (size_t)W * 4) + (size_t)H * 16;      // sx[W], then a 16-byte record per image row
    m.lut = (uint32_t)off;
    off = align16(off + (size_t)kNumFaces * materials_plus_one * 4);
    m.rows = (uint32_t)off;
    if (g.fast) off += 16 * (size_t)staged_layers * (size_t)(g.X + g.Y);
    else if (window) off += 8 * (size_t)staged_layers * ((size_t)g.Y * g.rowwords_x + (size_t)g.X * g.rowwords_y) + 16; // a window may end a dword behind its row
    else off += (size_t)g.xrow_words * 8;
    if (g.fast && coarse) off += 16 * (size_t)staged_layers * (size_t)((g.X + 1) / 2 + (g.Y + 1) / 2);
    m.total = (uint32_t)off;
    return m;
}

LdsPlan plan_lds(const GridLayout& g, int W, int H, int materials_plus_one, int staged_layers, bool coarse)
{
    LdsPlan plan{};
    plan.window = !g.fast;
    LdsMap m = lds_map(g, W, H, materials_plus_one, staged_layers, coarse, plan.window);
    // x and y rows are taken wherever they fit, also where they leave one workgroup per CU and x rows alone would leave two.
    // With the same reserve, per-cell -> window, us, 5 % of the columns filled to the top and, in brackets, worlds of four
    // layers: 128x128x24, 8 x 1 at 128x72 30 -> 21 (50 -> 22), 64 x 2 at 256x144 162 -> 148 (233 -> 89), 256 x 2 at 128x72
    // 181 -> 211 (233 -> 117); 128x128x36 35 -> 24 (50 -> 14), 173 -> 160 (239 -> 86), 224 -> 228 (296 -> 113); 200x200x12 48 -> 29,
    // 216 -> 148, 197 -> 192.  So large batches of worlds that are dense up there lose up to a sixth, at images of a few
    // tiles (17x17 pixels) up to a third, all others gain; the launch knows the tallest world only, not how many are.
    if (plan.window && m.total > kLdsBudget) {
        plan.window = false;
        m = lds_map(g, W, H, materials_plus_one, staged_layers, coarse, false);
    }
    if (m.total > kLdsBudget) return LdsPlan{};                             // bytes == 0: does not fit
    plan.bytes = m.total;
    // as many waves per workgroup as fill the CU's wave slots with the workgroups its LDS can hold
    // (measured: 64x64x32 grids, two workgroups per CU: 1024 threads render 9 % faster than 512)
    size_t per_cu = kLdsBudget / plan.bytes;
    size_t waves = 32 / (per_cu < 1 ? 1 : per_cu);          // 32 wave slots per CU
    waves &= ~(size_t)3;                                    // whole multiples of the 4 SIMDs: 5 or 6 waves per
    if (waves < 4) waves = 4;                               // workgroup load the SIMDs unevenly (-10 % measured)
    if (waves > 16) waves = 16;
    plan.threads = (int)(waves * 64);
    return plan;
}

// ------------------------------------------------------------------------------------------
// Work per camera, image row and column, and environment, microseconds in all: a launch of its own for each costs more
// (about 4.7 us between two others, most of it start and end of the launch) than the work.  Calls that know several of
// them at once run them together, in workgroups behind those of a launch the call makes anyway (SideWork).
//   pixel-centre scalars: sx[c] = (2c+1-W)/W, sy[r] = (H-2r-1)/H, one correctly rounded divide each
//   cameras: basis from yaw/pitch in float64, scaled, rounded once to float32.
//     forward F = (cos p cos y, cos p sin y, sin p), right = (sin y, -cos y, 0),
//     up = (-sin p cos y, -sin p sin y, cos p)
//   active[n] = (done[n] == 0)
// ------------------------------------------------------------------------------------------
constexpr int kSideThreads = 256;       // items a workgroup of any host kernel takes

__device__ __forceinline__ void write_camera(const SideWork& s, int o)
{
    const float* c = s.cams + 5 * (size_t)o;
    double yaw = (double)c[3], pitch = (double)c[4];
    double sy, cy, sp, cp;
    sincos(yaw, &sy, &cy);
    sincos(pitch, &sp, &cp);
    CameraRecord r;
    r.P[0] = c[0]; r.P[1] = c[1]; r.P[2] = c[2];
    r.F[0] = (float)(cp * cy); r.F[1] = (float)(cp * sy); r.F[2] = (float)sp;
    r.R[0] = (float)(s.tan_half_x * sy); r.R[1] = (float)(s.tan_half_x * -cy); r.R[2] = (float)(s.tan_half_x * 0.0);
    r.U[0] = (float)(s.tan_half_y * (-sp * cy)); r.U[1] = (float)(s.tan_half_y * (-sp * sy)); r.U[2] = (float)(s.tan_half_y * cp);
    const int body = s.self_voxel ? s.self_voxel[o] : -1;
    r.self_lo = body >= 0 ? body : -1;
    r.self_hi = body >= 0 ? body + s.X * s.Y : -1;
    // where the camera stands, once here instead of in every workgroup that renders for it
    const bool in_grid = r.P[0] >= 0.0f && r.P[0] <= (float)s.X && r.P[1] >= 0.0f && r.P[1] <= (float)s.Y &&
                         r.P[2] >= 0.0f && r.P[2] <= (float)s.Z;
    const bool near = fabsf(r.P[0]) <= kNearOutside && fabsf(r.P[1]) <= kNearOutside && fabsf(r.P[2]) <= kNearOutside;
    const bool hair = (r.P[0] < 0.0f && r.P[0] > -kHair) || (r.P[1] < 0.0f && r.P[1] > -kHair) || (r.P[2] < 0.0f && r.P[2] > -kHair);
    r.place = in_grid ? kPlaceInGrid : (near && !hair ? kPlaceOutside : kPlaceFarOutside);
    r.layer = min(max((int)floorf(r.P[2]), 0), s.Z - 1);
    s.rec[o] = r;
}

// item `i` of every kind the call has (the counts of the others are 0)
__device__ __forceinline__ void side_work(const SideWork& s, int i)
{
    if (i < s.W) s.sx[i] = __fdiv_rn((float)(2 * i + 1 - s.W), (float)s.W);
    if (i < s.H) s.sy[i] = __fdiv_rn((float)(s.H - 2 * i - 1), (float)s.H);
    if (i < s.num_done) s.active[i] = s.done[i] == 0 ? 1 : 0;
    if (i < s.num_obs) write_camera(s, i);
}

static int side_blocks(const SideWork& s)
{
    int n = s.num_obs;
    if (s.W > n) n = s.W;
    if (s.H > n) n = s.H;
    if (s.num_done > n) n = s.num_done;
    return (n + kSideThreads - 1) / kSideThreads;
}

__global__ void side_kernel(SideWork s) { side_work(s, blockIdx.x * blockDim.x + threadIdx.x); }

hipError_t launch_side(const SideWork& side, hipStream_t stream)
{
    // (workgroups of 128 spread few cameras over more compute units)
    hipLaunchKernelGGL(side_kernel, dim3(2 * side_blocks(side)), dim3(kSideThreads / 2), 0, stream, side);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// pack: one workgroup per environment, whole z layers per wave.  Two kernels, chosen by the host (launch_pack):
//   pack_kernel      grids of one word per row whose layers are whole 16-byte pieces at aligned addresses, or whole dwords
//                    and small: a layer is prefetched into registers one layer ahead, goes through LDS and leaves again
//                    as the batch's own copy; lane j turns x row j into bits dword by dword.
//   pack_any_kernel  every other size and alignment: a layer becomes a plain bit string in LDS (bit c = cell c of the
//                    layer) as it arrives, and the rows are cut out of that string at any bit offset.
// In both the y rows are the 64x64 bit transposes of the x rows, done across lanes without memory, and rows leave as
// one coalesced store per 64 rows.  A layer of air (no byte set) is written as zero rows without more work.
// ------------------------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPackThreads = 256;
constexpr int kPackAnyWaves = 16;       // most waves of a pack_any_kernel workgroup
constexpr int kPackAnyPieces = 3;       // 16-byte pieces of a layer each of its lanes keeps in flight

// Colour table entry (a6): round-to-nearest(palette value * face intensity) per channel as two
// separately rounded float32 operations (multiply, then add 0.5), floor, clamp to 255; r | g<<8 | b<<16.
struct Intensities { float v[kNumFaces]; };

__device__ __forceinline__ uint32_t shade_entry(const uint8_t* rgb, float intensity)
{
    uint32_t packed = 0;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        float q = floorf(__fadd_rn(__fmul_rn((float)rgb[ch], intensity), 0.5f));
        q = fminf(fmaxf(q, 0.0f), 255.0f);
        packed |= (uint32_t)q << (8 * ch);
    }
    return packed;
}

// The environment's palette: private copy, and the colour table lut[face][material].
__device__ __forceinline__ void pack_palette(const uint8_t* pal_src, uint8_t* pal_dst, uint32_t* lut_dst, int env,
                                             int materials_plus_one, const Intensities& I, int threads)
{
    const uint8_t* ps = pal_src + (size_t)env * materials_plus_one * 3;
    uint8_t* pd = pal_dst + (size_t)env * materials_plus_one * 3;
    uint32_t* lut = lut_dst + (size_t)env * kNumFaces * materials_plus_one;
    if (ps != pd)
        for (int i = threadIdx.x; i < materials_plus_one * 3; i += threads) pd[i] = ps[i];
    for (int i = threadIdx.x; i < kNumFaces * materials_plus_one; i += threads) {
        const int face = i / materials_plus_one, m = i - face * materials_plus_one;
        lut[i] = shade_entry(ps + 3 * m, I.v[face]);
    }
}

// The non-zero bytes of a dword as four bits (carry trick, then one dot product with weights 1,2,4,8).
__device__ __forceinline__ uint32_t nonzero_nibble(uint32_t x)
{
    const uint32_t flags = ((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) >> 7) & 0x01010101u;
    return __builtin_amdgcn_udot4(flags, 0x08040201u, 0u, false);
}

// 64x64 bit-matrix transpose across the wave: on entry lane j holds row j, on return lane i holds
// column i (bit j of the result = bit i of lane j's input).  Recursive block swap: at distance S
// lanes l and l^S exchange the off-diagonal SxS blocks.  The partner's word comes over the LDS
// crossbar (ds_swizzle / ds_bpermute, no memory), is rotated so that the wanted block lines up
// (the bits that wrap around fall on positions the mask discards) and is merged with one bit-select.
template <int S>
__device__ __forceinline__ uint32_t swap_blocks(uint32_t w, uint32_t keep, uint32_t rotate_right)
{
    const uint32_t partner = (uint32_t)__builtin_amdgcn_ds_swizzle((int)w, (S << 10) | 0x1f);    // lane ^ S
    const uint32_t lined_up = __builtin_amdgcn_alignbit(partner, partner, rotate_right);
    return (keep & w) | (~keep & lined_up);
}

__device__ __forceinline__ uint64_t transpose_bits_across_lanes(uint64_t row, int lane)
{
    uint32_t lo = (uint32_t)row, hi = (uint32_t)(row >> 32);
    {   // distance 32: whole words trade places
        const bool lower = (lane & 32) == 0;
        const uint32_t got = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(lower ? hi : lo));
        const uint32_t nlo = lower ? lo : got, nhi = lower ? got : hi;
        lo = nlo; hi = nhi;
    }
#define MV_SWAP_STAGE(S, MASK)                                                      \
    {                                                                               \
        const bool lower = (lane & S) == 0;                                         \
        const uint32_t keep = lower ? MASK : ~MASK;                                 \
        const uint32_t rot = lower ? 32 - S : S;                                    \
        lo = swap_blocks<S>(lo, keep, rot);                                         \
        hi = swap_blocks<S>(hi, keep, rot);                                         \
    }
    MV_SWAP_STAGE(16, 0x0000ffffu)
    MV_SWAP_STAGE(8, 0x00ff00ffu)
    MV_SWAP_STAGE(4, 0x0f0f0f0fu)
    MV_SWAP_STAGE(2, 0x33333333u)
    MV_SWAP_STAGE(1, 0x55555555u)
#undef MV_SWAP_STAGE
    return ((uint64_t)hi << 32) | lo;
}

// Called by one thread for a world (or a voxel) whose top is `top`: raises the batch's device word and, when
// it rose, the pinned host word (a system-scope atomic maximum, so that two risers cannot leave the smaller
// value behind).
__device__ __forceinline__ void report_height(const HeightFeedback& fb, int top)
{
    if (!fb.device_max) return;
    // thousands of worlds report per upload and almost none of them raises the word: look before the atomic
    if (top <= __hip_atomic_load(fb.device_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int old = atomicMax(fb.device_max, top);
    if (top > old) __hip_atomic_fetch_max(fb.host_max, top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Piece = what a lane moves at once: 16 bytes, or a dword where layers are not whole 16-byte pieces or start off their
// boundary.  kPieces = pieces of the next layer each lane keeps in flight, 2 KiB (40x40) or 4 KiB (64x64) of it in all: the
// deeper variant costs registers, so small layers keep the shallow one.  (Two layers in flight per wave change nothing, four are slower: the kernel moves its bytes at the rate of a plain
// device copy as it is.)  Other sizes and alignments have a kernel of their own: with their code in this one it
// needed a third more registers, and lost two of its eight waves per SIMD.
__device__ __forceinline__ uint32_t all_bits(uint32_t v) { return v; }
__device__ __forceinline__ uint32_t all_bits(u32x4 v) { return v.x | v.y | v.z | v.w; }

template <typename Piece, int kPieces, bool kSide>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ vox_dst,
                                                            uint64_t* __restrict__ bits_dst, int32_t* __restrict__ ztop_dst,
                                                            GridLayout g, const uint8_t* __restrict__ pal_src,
                                                            uint8_t* __restrict__ pal_dst, uint32_t* __restrict__ lut_dst,
                                                            int materials_plus_one, Intensities I, HeightFeedback heights,
                                                            int count, SideWork side)
{
    extern __shared__ __align__(16) uint8_t layer_lds[];   // one layer per wave
    __shared__ int top_lds;
    const int env = blockIdx.x;
    if (kSide && env >= count) {
        side_work(side, (env - count) * kSideThreads + (int)threadIdx.x);
        return;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int waves = kPackThreads / 64;
    const int X = g.X, Y = g.Y, Z = g.Z;
    const int XY = X * Y;
    uint8_t* mine = layer_lds + (size_t)wave * XY;
    const size_t env_vox = (size_t)env * XY * Z;
    const bool copy = (src != vox_dst);
    uint64_t* xrows = bits_dst + (size_t)env * g.env_words;
    uint64_t* yrows = xrows + g.xrow_words;
    int top = 0;
    const int pieces = XY / (int)sizeof(Piece);
    Piece pre[kPieces];
    auto fetch_layer = [&](int k) {
        const Piece* layer = reinterpret_cast<const Piece*>(src + env_vox + (size_t)k * XY);
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            Piece v = {};
            if (u * 64 + lane < pieces) v = __builtin_nontemporal_load(&layer[u * 64 + lane]);
            pre[u] = v;
        }
    };
    if (wave < Z) fetch_layer(wave);

    // (after the first layers have been requested, so that the palette's trip to memory runs beside theirs)
    if (pal_src) pack_palette(pal_src, pal_dst, lut_dst, env, materials_plus_one, I, kPackThreads);
    if (threadIdx.x == 0) top_lds = 0;
    __syncthreads();

    for (int k = wave; k < Z; k += waves) {
        // The private material copy is only ever read at voxels whose occupancy bit is set (the hit
        // voxel of a ray), so a layer without any solid voxel is not copied: its old bytes stay behind
        // bits that are all zero.
        uint32_t any = 0;
#pragma unroll
        for (int u = 0; u < kPieces; ++u) any |= all_bits(pre[u]);
        if (__ballot(any != 0) == 0) {
            // a layer of air: its rows are zero words, and neither LDS nor the transpose is needed for that
            if (k + waves < Z) fetch_layer(k + waves);
            if (lane < Y) xrows[(size_t)k * Y + lane] = 0ull;
            if (lane < X) yrows[(size_t)k * X + lane] = 0ull;
            continue;
        }
        top = k + 1;
        Piece* own_copy = reinterpret_cast<Piece*>(vox_dst + env_vox + (size_t)k * XY);
        Piece* in_lds = reinterpret_cast<Piece*>(mine);
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const int b = u * 64 + lane;
            if (b < pieces) {
                in_lds[b] = pre[u];
                if (copy) __builtin_nontemporal_store(pre[u], &own_copy[b]);
            }
        }
        // the next layer is requested as soon as the registers are free, and arrives while this one is packed
        if (k + waves < Z) fetch_layer(k + waves);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t lo = 0, hi = 0;
        const uint32_t* rowp = reinterpret_cast<const uint32_t*>(mine + min(lane, Y - 1) * X);
#pragma unroll
        for (int w4 = 0; w4 < 16; ++w4) {
            if (w4 * 4 < X) {
                const uint32_t nib = nonzero_nibble(rowp[w4]);
                if (w4 < 8) lo |= nib << (4 * w4); else hi |= nib << (4 * (w4 - 8));
            }
        }
        const uint64_t xbits = ((uint64_t)hi << 32) | lo;
        if (lane < Y) xrows[(size_t)k * Y + lane] = xbits;
        // y rows = the transpose of the 64x64 bit matrix whose row j is lane j's x row
        const uint64_t ybits = transpose_bits_across_lanes(lane < Y ? xbits : 0ull, lane);
        if (lane < X) yrows[(size_t)k * X + lane] = ybits;
        __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) atomicMax(&top_lds, top);
    __syncthreads();
    if (threadIdx.x == 0) {
        ztop_dst[env] = top_lds;
        report_height(heights, top_lds);
    }
}

// 16 bytes at any address (one unaligned vector access)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
// a dword of a bit string that is written 16 bits at a time
typedef uint32_t string_dword __attribute__((may_alias));

// Any grid size, any alignment.  What bounds it is memory, as for pack_kernel; a wave keeps 3 KiB in flight and the
// workgroup holds as many waves as the world has layers (up to 16), so that a CU with a single environment still has
// 48 KiB on its way.  A lane turns its 16 bytes into 16 bits where they arrive (the
// bytes never see LDS), and a row of the layer, wherever it starts in the bit string, costs two funnel shifts.
// The kernel before this one gathered rows cell by cell out of a byte copy in LDS (three instructions per
// cell and direction, four waves per environment).
template <bool kSide>
__global__ __launch_bounds__(kPackAnyWaves * 64) __attribute__((amdgpu_waves_per_eu(8, 8))) void pack_any_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ vox_dst,
                                                                      uint64_t* __restrict__ bits_dst, int32_t* __restrict__ ztop_dst,
                                                                      GridLayout g, const uint8_t* __restrict__ pal_src,
                                                                      uint8_t* __restrict__ pal_dst, uint32_t* __restrict__ lut_dst,
                                                                      int materials_plus_one, Intensities I, HeightFeedback heights,
                                                                      int bits_bytes, int waves, int count, SideWork side)
{
    extern __shared__ __align__(16) uint8_t bits_lds[];     // per wave: the bit string of one layer and two dwords more
    __shared__ int top_lds;
    const int env = blockIdx.x;
    if (kSide && env >= count) {
        if (threadIdx.x < kSideThreads) side_work(side, (env - count) * kSideThreads + (int)threadIdx.x);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int X = g.X, Y = g.Y, Z = g.Z;
    const int XY = X * Y, wx = g.rowwords_x, wy = g.rowwords_y;
    uint16_t* string16 = reinterpret_cast<uint16_t*>(bits_lds + (size_t)wave * bits_bytes);
    const string_dword* string32 = reinterpret_cast<const string_dword*>(string16);
    const size_t env_vox = (size_t)env * XY * Z;
    const bool copy = (src != vox_dst);
    uint64_t* xrows = bits_dst + (size_t)env * g.env_words;
    uint64_t* yrows = xrows + g.xrow_words;
    if (pal_src) pack_palette(pal_src, pal_dst, lut_dst, env, materials_plus_one, I, waves * 64);
    if (threadIdx.x == 0) top_lds = 0;
    __syncthreads();

    // word w of x row j, from the bit string (bits beyond the row's end cleared)
    auto row_word = [&](int j, int w) -> uint64_t {
        const uint32_t at = (uint32_t)(j * X + 64 * w), d = at >> 5;
        const uint32_t lo = __builtin_amdgcn_alignbit(string32[d + 1], string32[d], at);
        const uint32_t hi = __builtin_amdgcn_alignbit(string32[d + 2], string32[d + 1], at);
        const uint64_t both = ((uint64_t)hi << 32) | lo;
        const int n = X - 64 * w;
        return n >= 64 ? both : both & ((1ull << n) - 1ull);
    };
    int top = 0;
    for (int k = wave; k < Z; k += waves) {
        const uint8_t* layer = src + env_vox + (size_t)k * XY;
        uint8_t* dst = vox_dst + env_vox + (size_t)k * XY;
        uint64_t seen = 0;
        if (XY >= 16) {
            const int pieces = (XY + 15) >> 4;
            for (int b0 = 0; b0 < pieces; b0 += 64 * kPackAnyPieces) {
                u32x4 v[kPackAnyPieces];
#pragma unroll
                for (int u = 0; u < kPackAnyPieces; ++u) {
                    // the last piece is read 16 bytes from the layer's end (and shifted down below)
                    const int b = b0 + u * 64 + lane;
                    v[u] = u32x4{ 0u, 0u, 0u, 0u };
                    if (b < pieces) v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(layer + min(b * 16, XY - 16)));
                }
#pragma unroll
                for (int u = 0; u < kPackAnyPieces; ++u) {
                    const int b = b0 + u * 64 + lane, at = min(b * 16, XY - 16);
                    const uint32_t bits = nonzero_nibble(v[u].x) | (nonzero_nibble(v[u].y) << 4) | (nonzero_nibble(v[u].z) << 8) |
                                          (nonzero_nibble(v[u].w) << 12);
                    const uint64_t some = __ballot(bits != 0);
                    seen |= some;
                    if (b < pieces) {
                        string16[b] = (uint16_t)(bits >> (b * 16 - at));
                        // (the material copy is only read at solid voxels: 64 pieces that are all air are not copied)
                        if (copy && some) __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4_any*>(dst + at));
                    }
                }
            }
        } else {
            const uint8_t m = lane < XY ? layer[lane] : (uint8_t)0;
            seen = __ballot(m != 0);
            if (copy && lane < XY) dst[lane] = m;
            if (lane == 0) string16[0] = (uint16_t)seen;
        }
        if (seen == 0) {
            for (int r = lane; r < Y * wx; r += 64) xrows[(size_t)k * Y * wx + r] = 0ull;
            for (int r = lane; r < X * wy; r += 64) yrows[(size_t)k * X * wy + r] = 0ull;
            continue;
        }
        top = k + 1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // blocks of 64 rows x 64 cells: the x-row words as they are, the y-row words as the block's transpose
        for (int jb = 0; jb < wy; ++jb) {
            const int j = jb * 64 + lane;
            for (int w = 0; w < wx; ++w) {
                const uint64_t xbits = j < Y ? row_word(j, w) : 0ull;
                if (j < Y) xrows[((size_t)k * Y + j) * wx + w] = xbits;
                const uint64_t ybits = transpose_bits_across_lanes(xbits, lane);
                const int i = w * 64 + lane;
                if (i < X) yrows[((size_t)k * X + i) * wy + jb] = ybits;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) atomicMax(&top_lds, top);
    __syncthreads();
    if (threadIdx.x == 0) {
        ztop_dst[env] = top_lds;
        report_height(heights, top_lds);
    }
}

size_t pack_lds_bytes(const GridLayout& g)
{
    const size_t XY = (size_t)g.X * g.Y;
    return ((XY + 15) & ~(size_t)15) * (kPackThreads / 64);
}

hipError_t launch_pack(const uint8_t* src, uint8_t* vox_dst, uint64_t* bits_dst, int32_t* ztop_dst, int count,
                       const GridLayout& g, const uint8_t* pal_src, uint8_t* pal_dst, uint32_t* lut_dst,
                       int materials_plus_one, const float intensity[kNumFaces], const HeightFeedback& heights,
                       const SideWork* side, hipStream_t stream)
{
    static_assert(kPackThreads == kSideThreads, "a pack workgroup takes one workgroup's share of side work");
    const SideWork no_side{};
    const int blocks = count + (side ? side_blocks(*side) : 0);
    Intensities I;
    for (int f = 0; f < kNumFaces; ++f) I.v[f] = intensity[f];
    const size_t XY = (size_t)g.X * g.Y;
    const uintptr_t addresses = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(vox_dst);
    // (fast grids hold at most 64 x 64 cells, 4 KiB, per layer; rows are read as dwords)
    // Few worlds leave most of the chip idle: there the general kernel, a wave per layer instead of four layers one after
    // the other per wave, is the faster one (40x40x16, us: 64 worlds 6.8 -> 5.2, 256 7.2 -> 5.9, 512 8.3 and 7.9, 1024 11.7
    // and 14.3; 64x64x32: 64 worlds 11.8 -> 9.6, 256 13.7 -> 13.0, 512 21.5 and 21.9; 16x16x8 the same up to 512).
    const bool few = count <= 256;
    // Layers that are whole dwords but not whole 16-byte pieces, or start off a 16-byte boundary, move dword by dword while
    // that keeps eight waves per SIMD, up to 2 KiB (many worlds, general kernel -> dwords, us: 28x26x12 x 1024 10.6 -> 7.8, x
    // 4096 36.5 -> 20.0; 8x9x12 x 4096 31.4 -> 13.8; 36x30x16 x 4096 43.5 -> 29.6; 40x40x16 x 4096 at an odd dword 44.2 -> 35.3;
    // but 44x63x32, sixteen dwords per lane, x 300 12.3 -> 15.6, x 2048 54.7 -> 60.8).
    const bool whole = XY % 16 == 0 && (addresses & 15) == 0;
    const bool dwords = (addresses & 3) == 0 && XY <= 8 * 64 * 4;
    if (g.fast && (g.X & 3) == 0 && (whole || dwords) && !few) {
        const size_t lds = pack_lds_bytes(g);
#define MV_LAUNCH_PACK(PIECE, PIECES)                                                                                     \
    do {                                                                                                                  \
        if (side)                                                                                                         \
            hipLaunchKernelGGL((pack_kernel<PIECE, PIECES, true>), dim3(blocks), dim3(kPackThreads), lds, stream, src,      \
                               vox_dst, bits_dst, ztop_dst, g, pal_src, pal_dst, lut_dst, materials_plus_one, I, heights,  \
                               count, *side);                                                                             \
        else                                                                                                              \
            hipLaunchKernelGGL((pack_kernel<PIECE, PIECES, false>), dim3(blocks), dim3(kPackThreads), lds, stream, src,     \
                               vox_dst, bits_dst, ztop_dst, g, pal_src, pal_dst, lut_dst, materials_plus_one, I, heights,  \
                               count, no_side);                                                                           \
    } while (0)
        if (!whole) MV_LAUNCH_PACK(uint32_t, 8);
        else if (XY <= 2 * 64 * 16) MV_LAUNCH_PACK(u32x4, 2);
        else MV_LAUNCH_PACK(u32x4, 4);
#undef MV_LAUNCH_PACK
    } else {
        // (at least kSideThreads threads: what a workgroup takes of the side work)
        int waves = g.Z < kPackAnyWaves ? g.Z : kPackAnyWaves;
        if (waves < kSideThreads / 64) waves = kSideThreads / 64;
        // per wave: the layer's bit string, and the two dwords behind its last one that a row's last word may read
        const int bits_bytes = (int)(((XY + 31) / 32) * 4 + 8);
#define MV_LAUNCH_PACK_ANY(SIDE)                                                                                          \
    hipLaunchKernelGGL(pack_any_kernel<SIDE>, dim3(blocks), dim3(waves * 64), (size_t)waves * bits_bytes, stream, src,      \
                       vox_dst, bits_dst, ztop_dst, g, pal_src, pal_dst, lut_dst, materials_plus_one, I, heights,           \
                       bits_bytes, waves, count, side ? *side : no_side)
        if (side) MV_LAUNCH_PACK_ANY(true); else MV_LAUNCH_PACK_ANY(false);
#undef MV_LAUNCH_PACK_ANY
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// update: one thread per edited voxel.  The material byte is overwritten; the voxel's bit in its x row
// and in its y row is set or cleared with a 64-bit atomic (several edits of one call may share a row
// word); setting a voxel raises the environment's top-layer bound, clearing never lowers it.
// Two launches per call: kFill == false applies the edits that empty a voxel, kFill == true, after it in
// stream order, those that fill one -- so an object that moves into the voxel another one leaves in the
// same step ends up there whatever the order of the two edits in the list.
// ------------------------------------------------------------------------------------------
template <bool kFill, bool kSide>
__global__ void update_voxels_kernel(const int32_t* __restrict__ env, const int32_t* __restrict__ voxel_index,
                                     const uint8_t* __restrict__ material, int count, uint8_t* __restrict__ vox,
                                     uint64_t* __restrict__ bits, int32_t* __restrict__ ztop, int num_envs,
                                     int voxels_per_env, int num_materials, GridLayout g, HeightFeedback heights,
                                     int edit_blocks, SideWork side)
{
    if (kSide && (int)blockIdx.x >= edit_blocks) {
        side_work(side, ((int)blockIdx.x - edit_blocks) * kSideThreads + (int)threadIdx.x);
        return;
    }
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    const int n = env[e], idx = voxel_index[e];
    const int m = material ? material[e] : 0;           // no material array: every entry empties its voxel
    if ((m != 0) != kFill) return;
    if (n < 0 || n >= num_envs || idx < 0 || idx >= voxels_per_env || m > num_materials) return;
    const int XY = g.X * g.Y;
    const int k = idx / XY, rem = idx - k * XY, j = rem / g.X, i = rem - j * g.X;
    vox[(size_t)n * voxels_per_env + idx] = (uint8_t)m;
    unsigned long long* xrow = reinterpret_cast<unsigned long long*>(bits) + (size_t)n * g.env_words +
                               ((size_t)k * g.Y + j) * g.rowwords_x + (i >> 6);
    unsigned long long* yrow = reinterpret_cast<unsigned long long*>(bits) + (size_t)n * g.env_words + g.xrow_words +
                               ((size_t)k * g.X + i) * g.rowwords_y + (j >> 6);
    if (kFill) {
        atomicOr(xrow, 1ull << (i & 63));
        atomicOr(yrow, 1ull << (j & 63));
        // (the bound only grows while edits are applied, and hardly any edit raises it: look before the atomic)
        if (__hip_atomic_load(ztop + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < k + 1)
            if (atomicMax(ztop + n, k + 1) < k + 1) report_height(heights, k + 1);
    } else {
        atomicAnd(xrow, ~(1ull << (i & 63)));
        atomicAnd(yrow, ~(1ull << (j & 63)));
    }
}

constexpr int kEditThreads = kSideThreads;

// `side`, if any, runs in workgroups behind the first launch's
hipError_t launch_update_voxels(const int32_t* env, const int32_t* voxel_index, const uint8_t* material, int count,
                                uint8_t* vox, uint64_t* bits, int32_t* ztop, int num_envs, int voxels_per_env,
                                int num_materials, const GridLayout& g, const HeightFeedback& heights, const SideWork* side,
                                hipStream_t stream)
{
    const SideWork no_side{};
    const int blocks = (count + kEditThreads - 1) / kEditThreads;
    if (side)
        hipLaunchKernelGGL((update_voxels_kernel<false, true>), dim3(blocks + side_blocks(*side)), dim3(kEditThreads), 0,
                           stream, env, voxel_index, material, count, vox, bits, ztop, num_envs, voxels_per_env,
                           num_materials, g, heights, blocks, *side);
    else
        hipLaunchKernelGGL((update_voxels_kernel<false, false>), dim3(blocks), dim3(kEditThreads), 0, stream, env, voxel_index,
                           material, count, vox, bits, ztop, num_envs, voxels_per_env, num_materials, g, heights, blocks,
                           no_side);
    hipLaunchKernelGGL((update_voxels_kernel<true, false>), dim3(blocks), dim3(kEditThreads), 0, stream, env, voxel_index,
                       material, count, vox, bits, ztop, num_envs, voxels_per_env, num_materials, g, heights, blocks, no_side);
    return hipGetLastError();
}

// Objects that moved: every voxel an object left is emptied (first launch, no material array), then every voxel an
// object is in now is filled with the object's material (second launch); negative indices are skipped by the kernel.
hipError_t launch_move_voxels(const int32_t* env, const int32_t* from_voxel, const int32_t* to_voxel,
                              const uint8_t* material, int count, uint8_t* vox, uint64_t* bits, int32_t* ztop,
                              int num_envs, int voxels_per_env, int num_materials, const GridLayout& g,
                              const HeightFeedback& heights, hipStream_t stream)
{
    const SideWork no_side{};
    const int blocks = (count + kEditThreads - 1) / kEditThreads;
    hipLaunchKernelGGL((update_voxels_kernel<false, false>), dim3(blocks), dim3(kEditThreads), 0, stream, env, from_voxel,
                       static_cast<const uint8_t*>(nullptr), count, vox, bits, ztop, num_envs, voxels_per_env, num_materials,
                       g, heights, blocks, no_side);
    hipLaunchKernelGGL((update_voxels_kernel<true, false>), dim3(blocks), dim3(kEditThreads), 0, stream, env, to_voxel,
                       material, count, vox, bits, ztop, num_envs, voxels_per_env, num_materials, g, heights, blocks, no_side);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// render
// ------------------------------------------------------------------------------------------
struct Hit {
    int   idx;      // linear voxel index, negative = miss
    int   face;     // from trace_rows and trace_windows as FaceRows has it, from trace_generic 0..6, 255 = miss
    float t;        // planar depth
};

constexpr float kBig = 3.0e38f;            // stands in for 1/0: keeps every product finite or +inf, never NaN
constexpr float kSmallest = 0x1p-126f;      // smallest normal number
constexpr float kTinyDistance = 1e-30f;     // to a plane a camera is exactly on: nothing times |1/d|, or never if d is 0
constexpr float kNever = 0.5f * kBig;      // first crossing of an axis along which a ray does not move (below kBig, the
                                           // distance between two crossings: the one before the first lies behind the camera)

__device__ __forceinline__ float safe_rcp(float d)
{
    // v_rcp_f32 (1 ulp) then clamp: +-inf for d = +-0 becomes +-kBig
    return __builtin_amdgcn_fmed3f(__builtin_amdgcn_rcpf(d), -kBig, kBig);
}

// Small whole numbers as floats whose bits are the number (denormals): adding two of them, or multiplying one by a whole
// number, is integer arithmetic as long as the result stays below 2^23 (bits go on counting up to 2^24), exact and with any
// rounding.  The point is the instruction: a float add, multiply or fused multiply-add with its operands in vector registers
// issues in the shadow of the comparisons, selects, conversions and shifts other waves keep the vector pipeline busy with
// (0.5 cycles beside such an instruction, 4.4 for an integer add, shift or multiply-add, or for any operand in a scalar
// register; measured with streams of two instruction kinds).
__device__ __forceinline__ float tiny_int(uint32_t v) { return __uint_as_float(v); }
__device__ __forceinline__ float tiny_to_float(float t) { return (t * 0x1p127f) * 0x1p22f; }        // the number as a float
__device__ __forceinline__ float float_to_tiny(float v) { return (v * 0x1p-127f) * 0x1p-22f; }      // and back (whole numbers below 2^24)

// a value all lanes share, held in a vector register.  (The compiler often brings the scalar back from a spill with a
// v_readlane straight before, which needs two wait states between; it puts them in only in front of instructions of its own.)
__device__ __forceinline__ float in_vector(float v)
{
    float r;
    asm volatile("s_nop 1\n\tv_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}

// a value all lanes share, as a scalar
__device__ __forceinline__ float uniform(float v)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}

// What a tracer reports of the face a ray entered its voxel through: base + code * stride.  Launches with auxiliary outputs
// take the face code itself (0, 1); the others the LDS address of the face's row of the colour table, so that the colour of a
// pixel is one multiply-add away from its material.
struct FaceRows {
    int base, stride;
    __device__ __forceinline__ int of(int code) const { return base + code * stride; }
};

// Constants of one scan class of one camera.  A class is (dominant horizontal axis, direction along it,
// direction along the other horizontal axis, vertical direction): class = 8*(y dominant) + 4*(u negative) +
// 2*(v negative) + (z negative), so a ray picks every direction-dependent constant with one record load
// instead of selecting each per ray.  u is the scan axis, v the other horizontal axis.  For negative u
// the class works in mirrored coordinates u' = U - u against a bit-reversed copy of the rows, so that
// inside the traversal every ray runs towards increasing bit positions.  v and z crossings are counted
// without sign; the direction is folded into the address and index steps.
struct alignas(16) ScanClass {
    float Pu;           // camera coordinate along u (mirrored for negative u)
    float uexit;        // U - Pu: distance to the far side of the grid along u (window scan: to the first u plane)
    float Pu_err;       // what rounding took from the mirrored coordinate: (U - P) - Pu exactly, 0 if not mirrored
    int   addr0;        // LDS byte address of the camera's row in this class's row array
    float row_step_vz;  // row-address step of a v crossing minus that of a z crossing, and that of a z crossing, as floats
    float row_step_z;   // whose bits are the number of bytes (denormals; a sign bit for steps back): see the row loop
    float dist_v;       // distance from the camera to the first v plane in this direction (>= 0)
    float nv_max;       // v planes between the camera cell and the grid boundary in this direction
                        // (the z counterparts of these two depend on the image row: RowRecord holds them)
    int   i0;           // camera cell along u (mirrored)
    int   um1;          // U - 1
    // voxel index of the hit = idx0 + cell*stride_u + n_v*stride_v + n_z*stride_z, evaluated with three fused
    // multiply-adds: every term and partial sum is an integer below 2^24 in magnitude, so float32 is exact
    float idx0;         // voxel index of (mirrored cell 0, camera's v cell, camera's layer)
    float stride_u;     // voxel-index step per mirrored u cell: +-1 (x scans) or +-X (y scans)
    float stride_v;     // voxel-index step per v crossing: +-X (x scans) or +-1 (y scans)
    float stride_z;     // voxel-index step per z crossing: +-X*Y
    int   sv;           // row-address step per v crossing: +-8 bytes
    int   sz;           // row-address step per z crossing: +-8*V bytes
    int   face_u;       // face (see FaceRows) of a voxel found while scanning along the row
    int   face_v;       // of a voxel entered through a v crossing
    int   face_z;       // of a voxel entered through a z crossing
    int   pad;
};
static_assert(sizeof(ScanClass) == 80, "scan class record must be 80 bytes");

// What all pixels of one image row share.  The camera has no roll, so its right axis is horizontal and the vertical
// component of a pixel ray, d_z = F_z + sy*U_z, depends on the row alone: its clamped reciprocal, the parameter of
// the first z crossing and the parameter at which the ray leaves the grid along z are computed once per row when a
// workgroup starts, with the operations a ray would use, instead of once per ray.
struct alignas(16) RowRecord {
    float sy;           // pixel-centre scalar of the row, (H - 2r - 1) / H
    float rcp_z;        // 1 / d_z clamped to +-kBig; its sign is the ray's vertical direction (-0 counts as rising)
    float t0_z;         // parameter of the first z crossing: distance to the first z plane times |1 / d_z|
    float tend_z;       // parameter of the crossing that takes the ray out of the (cut) grid along z
};

// Coarse level (optional): the OR of each pair of neighbouring rows (2J, 2J+1) of a layer, one array per row
// array.  These constants of a scan class sit behind its record, in the same 128-byte slot.
struct alignas(16) PairClass {
    int addr0;          // LDS byte address of the camera's pair row in this class's pair array
    int sv;             // pair-address step when the ray crosses from one pair into the next: +-8 bytes
    int sz;             // pair-address step per z crossing: +-8 * (pairs per layer)
    int inner0;         // 1 if the first v plane ahead of the camera lies inside its pair, 0 if it bounds it
};
static_assert(sizeof(ScanClass) + sizeof(PairClass) <= kClassStride, "class slot too small");

// Where the rays of a camera outside the grid enter the box [0,X]x[0,Y]x[0,top] (row scan): these constants of a class sit
// behind its record, and in four words of the record that such cameras have no other use for (near_v: dist_v, far_v: nv_max,
// Pv: i0, last_v: pad).  Distances along u and v are those a ray has to go, so that times |1/d| they are its parameters.
struct alignas(16) EntryClass {
    float near_u, far_u;                    // to the near and to the far side of the box along u; near_v, far_v along v
                                            // Pv: camera coordinate along v, as it is; last_v: V - 1
    float ahead_v, ahead_z;                 // 0 or 1: from a cell's number to that of the plane a ray leaves it through
    float per_cell_v, per_cell_z;           // planes left behind a cell's = planes + per_cell * cell
    float planes_v, planes_z;
};
static_assert(sizeof(EntryClass) == 32 && sizeof(ScanClass) + sizeof(EntryClass) <= kClassStride, "class slot too small");

// Plain 3D-DDA through the x rows (any row width), in LDS or in global memory.  Used for grids whose x and y rows do not
// both fit into LDS, for cameras far outside the grid, and for workgroups whose world is taller than the layers staged.
// Crossing parameters are t = n*|1/d| + t_first (one fused op, error relative to t itself) rather than accumulated.
// self_lo / self_hi: voxels this camera must not see (-1 = none); callers that have already removed the body
// from their copy of the rows pass -1.
// Every cell it looks at lies in the grid, whatever the camera: no first crossing is NaN and every distance between two is
// finite, so an axis steps only while its parameter is the least of the three and below t_exit, which is at most that same
// expression at the axis's last plane.  A component below the smallest normal number counts as 0 (its reciprocal is infinite,
// and 0 times that not a number), and an axis whose first crossing is not a number (unchecked cameras) is never crossed: with
// NaN among them the comparisons fail one after the other, and z went on for ever.
__device__ __forceinline__ Hit trace_generic(const uint32_t* __restrict__ xrows32, int rowdwords, const float P[3],
                                             const float d[3], int X, int Y, int Z, bool origin_in_grid, int max_steps,
                                             int self_lo, int self_hi)
{
    const float kInf = __builtin_inff();
    const int dim[3] = { X, Y, Z };
    Hit miss = { -1, 255, 0.0f };
    float inv[3];
    bool pos[3], zero[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        zero[a] = fabsf(d[a]) < kSmallest;
        pos[a] = d[a] > 0.0f;
        inv[a] = zero[a] ? 0.0f : __builtin_amdgcn_rcpf(d[a]);
    }
    float t0 = 0.0f;
    int entry_axis = -1;
    if (!origin_in_grid) {
        float t_near = -kInf, t_far = kInf;
        bool dead = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (zero[a]) {
                dead |= (P[a] < 0.0f) | (P[a] > (float)dim[a]);
            } else {
                float ta = ((pos[a] ? 0.0f : (float)dim[a]) - P[a]) * inv[a];
                float tb = ((pos[a] ? (float)dim[a] : 0.0f) - P[a]) * inv[a];
                if (ta > t_near) { t_near = ta; entry_axis = a; }
                t_far = fminf(t_far, tb);
            }
        }
        if (dead || t_near > t_far || t_far < 0.0f) return miss;
        if (t_near > 0.0f) t0 = t_near; else entry_axis = -1;
    }
    int cell[3], step[3];
    float t_next[3], t_first[3], dt[3], n[3];
    float t_exit = kInf;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float q = floorf(fmaf(t0, d[a], P[a]));
        int c = (int)fminf(fmaxf(q, 0.0f), (float)(dim[a] - 1));
        if (a == entry_axis) c = pos[a] ? 0 : dim[a] - 1;
        cell[a] = c;
        step[a] = pos[a] ? 1 : -1;
        float plane = (float)(c + (pos[a] ? 1 : 0));
        t_first[a] = zero[a] ? kInf : (plane - P[a]) * inv[a];
        dt[a] = fabsf(inv[a]);
        if (!(t_first[a] == t_first[a])) { t_first[a] = kInf; dt[a] = 0.0f; }
        n[a] = 0.0f;
        t_next[a] = t_first[a];
        float planes_left = (float)(pos[a] ? dim[a] - 1 - c : c);
        float te = zero[a] ? kInf : fmaf(planes_left, dt[a], t_first[a]);
        t_exit = fminf(t_exit, te);
    }
    auto solid = [&](int i, int j, int k) -> bool {
        const int idx = (k * Y + j) * X + i;
        return ((xrows32[(k * Y + j) * rowdwords + (i >> 5)] >> (i & 31)) & 1u) && idx != self_lo && idx != self_hi;
    };
    int face = entry_axis >= 0 ? 2 * entry_axis + (pos[entry_axis] ? 0 : 1) : 6;
    if (solid(cell[0], cell[1], cell[2])) return Hit{ (cell[2] * Y + cell[1]) * X + cell[0], face, t0 };
    for (int it = 0; it < max_steps; ++it) {
        float tm = fminf(fminf(t_next[0], t_next[1]), t_next[2]);
        if (!(tm < t_exit)) return miss;
        bool cx = (t_next[0] <= t_next[1]) & (t_next[0] <= t_next[2]);
        bool cy = !cx & (t_next[1] <= t_next[2]);
        bool cz = !cx & !cy;
        n[0] += cx ? 1.0f : 0.0f;  cell[0] += cx ? step[0] : 0;
        n[1] += cy ? 1.0f : 0.0f;  cell[1] += cy ? step[1] : 0;
        n[2] += cz ? 1.0f : 0.0f;  cell[2] += cz ? step[2] : 0;
        t_next[0] = fmaf(n[0], dt[0], t_first[0]);
        t_next[1] = fmaf(n[1], dt[1], t_first[1]);
        t_next[2] = fmaf(n[2], dt[2], t_first[2]);
        if (solid(cell[0], cell[1], cell[2])) {
            int axis = cx ? 0 : (cy ? 1 : 2);
            bool p = cx ? pos[0] : (cy ? pos[1] : pos[2]);
            return Hit{ (cell[2] * Y + cell[1]) * X + cell[0], 2 * axis + (p ? 0 : 1), tm };
        }
    }
    return miss;
}

// three-operand forms of the same
__device__ __forceinline__ float vmax3(float a, float b, float c);
__device__ __forceinline__ float vmin3(float a, float b, float c);

// One-instruction min/max: fminf()/fmaxf() make the compiler quiet possible signalling NaNs first
// (an extra v_max per operand inside the loop); no operand here can be one.
__device__ __forceinline__ float vmin(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float vmax(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float vmax3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float vmed3(float a, float b, float c)
{
    float r;
    asm("v_med3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float vmin3(float a, float b, float c)
{
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// index of the lowest set bit; the result for 0 is unspecified (callers ignore it for rays that found nothing)
__device__ __forceinline__ int ctz64_nonzero(uint64_t v)
{
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    uint32_t flo, fhi;
    asm("v_ffbl_b32 %0, %1" : "=v"(flo) : "v"(lo));
    asm("v_ffbl_b32 %0, %1" : "=v"(fhi) : "v"(hi));
    // v_ffbl_b32 returns 0xffffffff for 0, so the unsigned minimum picks the low word whenever it has a bit
    return (int)min(flo, __float_as_uint(tiny_int(fhi) + tiny_int(32u)));      // (0xffffffff + 32 stays a NaN: all ones or nearly)
}

// v & 1 as a 32-bit operation of its own (the compiler otherwise widens the test back to the 64-bit row)
__device__ __forceinline__ uint32_t low_bit(uint32_t v)
{
    uint32_t b;
    asm("v_and_b32 %0, 1, %1" : "=v"(b) : "v"(v));
    return b;
}

typedef __attribute__((address_space(3))) const float* lds_f32_ptr;
typedef __attribute__((address_space(3))) const uint32_t* lds_u32_ptr;
typedef __attribute__((address_space(3))) const uint64_t* lds_u64_ptr;
typedef __attribute__((address_space(3))) const u32x4* lds_u32x4_ptr;

// A camera outside the grid, for the tracers below: its rays start where they enter the box [0,X]x[0,Y]x[0,top].
struct OutsideCamera {
    FaceRows faces;
    bool finite;        // the camera's directions are numbers (all rays of others miss)
    float P[3];
    float dz;           // vertical component of the ray
    int X, Y, top;      // top: layers that may hold a solid voxel, at least 1
};

// Where such a ray enters the box: the same slab test, entry cells and first crossings as trace_generic (window scan; the row
// scan gets the same values from an EntryClass).
struct BoxEntry {
    bool misses;
    float t;            // parameter of the entry point, >= 0
    int face;           // face code of a voxel found in the entry cell
    int i, j, k;        // entry cell along u, v and z
    float t0_u, t0_v, t0_z;     // parameters of the first crossing along each
    float left_u;
    float left_v, left_z;   // planes between the entry cell and the far side of the box along v and z
};

__device__ __forceinline__ BoxEntry enter_box(const OutsideCamera& o, float dx, float dy, bool xm, float rcp_z)
{
    const float kInf = __builtin_inff();
    const float d[3] = { dx, dy, o.dz };
    const float rcp[3] = { safe_rcp(dx + 0.0f), safe_rcp(dy + 0.0f), rcp_z };
    const int dim[3] = { o.X, o.Y, o.top };
    float t_near = -kInf, t_far = kInf;
    int axis = -1;
    // (a direction that is not a number misses, so that every comparison below means what it says)
    bool dead = !(fabsf(dx) + fabsf(dy) + fabsf(o.dz) < kBig);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = (0.0f - o.P[a]) * rcp[a], hi = ((float)dim[a] - o.P[a]) * rcp[a];
        const bool zero = d[a] == 0.0f;
        const float ta = zero ? -kInf : fminf(lo, hi), tb = zero ? kInf : fmaxf(lo, hi);
        dead |= zero && (o.P[a] < 0.0f || o.P[a] > (float)dim[a]);
        if (ta > t_near) { t_near = ta; axis = a; }
        t_far = fminf(t_far, tb);
    }
    BoxEntry e;
    e.misses = dead || t_near > t_far || t_far < 0.0f;
    e.t = fmaxf(t_near, 0.0f);
    if (!(t_near > 0.0f)) axis = -1;
    const float d_axis = axis == 0 ? dx : (axis == 1 ? dy : o.dz);
    e.face = o.faces.of(axis < 0 ? 6 : 2 * axis + (d_axis > 0.0f ? 0 : 1));
    auto along = [&](int a, float da, float pa, float ra, int n, int& cell, float& first, float& left) {
        const bool neg = da < 0.0f;
        int c = (int)fminf(fmaxf(floorf(fmaf(e.t, da, pa)), 0.0f), (float)(n - 1));
        if (a == axis) c = neg ? n - 1 : 0;
        cell = c;
        // (not before the entry point: what a ray crosses later it must also reach later, or the run of cells of its
        // first row would end before it begins)
        first = da == 0.0f ? kBig : fmaxf(((float)(neg ? c : c + 1) - pa) * ra, e.t);
        left = (float)(neg ? c : n - 1 - c);
    };
    if (xm) {
        along(0, dx, o.P[0], rcp[0], o.X, e.i, e.t0_u, e.left_u);
        along(1, dy, o.P[1], rcp[1], o.Y, e.j, e.t0_v, e.left_v);
    } else {
        along(1, dy, o.P[1], rcp[1], o.Y, e.i, e.t0_u, e.left_u);
        along(0, dx, o.P[0], rcp[0], o.X, e.j, e.t0_v, e.left_v);
    }
    along(2, o.dz, o.P[2], rcp_z, o.top, e.k, e.t0_z, e.left_z);
    return e;
}

// Row-scan traversal: DDA over the (v,z) rows the ray passes through, one 64-bit shift per row.
// The loop has one exit (row holds a solid cell in range, or the ray leaves the grid).  It ends for
// every input: each turn advances n_v or n_z, the crossing parameters n*dt + t0 never decrease, and
// t_end is that same expression at the last plane of each axis, so t_out reaches t_end after at most
// V + Z + 2 turns; a NaN anywhere makes the comparison false and ends it at once.
// n_v and n_z count crossings without sign: the cell is (v0 +- n_v, kc +- n_z), the signs sit in the class.
// kNarrow: both horizontal grid sizes are below 64.  The parameter at which a row is left is capped at
// t_end, which puts the last cell of the run at U at most (U only through rounding at the far boundary);
// with U <= 63 that still is a valid bit position of an always-empty cell, and the clamp to U - 1 that
// 64-cell rows need is left out.
// kOutside: the ray starts where it enters the grid's box instead of in the camera's cell (see EntryClass), and the
// class records hold row and voxel index of cell (0,0,0) of the class's array instead of the camera's.  The row loop
// is the same one; a ray that misses the box leaves it in its first turn.  No crossing parameter lies before the entry
// point, so the runs of cells are monotone here as well.  Bound by instruction issue like the inside scan (256 x 4 cameras
// around 40x40x16 worlds at 128x72, upload + cameras + render: 286 us with the per-cell tracer over rows in device memory,
// which still takes far ones; 77 us with the slab test worked out per ray and axis; 63 us with what a class and an image row
// know of it ready-made, and one reciprocal per ray and axis instead of two).  The last cell of a run is taken from the ray's
// position, as for cameras inside: a ray that passes exactly through a voxel edge may fall on the other side of it than with
// the per-cell tracer (45-degree views along cell middles: 6 of 10 000 pixels; views at random: one of 13 million).
template <bool kNarrow, bool kCoarse, bool kOutside = false>
__device__ __forceinline__ Hit trace_rows(uint32_t classes_addr, float dx, float dy, const RowRecord& rr, int fine_turns,
                                          const OutsideCamera* from_outside = nullptr)
{
    static_assert(!(kCoarse && kOutside), "the coarse level starts from the camera's own pair of rows");
    const bool xm = fabsf(dx) >= fabsf(dy);
    const float du = xm ? dx : dy;
    const float dv = xm ? dy : dx;
    // class = 8*(y dominant) + 4*(u negative) + 2*(v negative) + (z negative): each funnel shift moves the
    // index up one bit and brings in the sign bit of the next component.  Along v and z a component
    // of -0 counts as positive (the ray never crosses a plane of that axis, and the distance to the
    // upper plane is never 0 inside the cell): adding +0 turns -0 into +0 and changes nothing else.
    uint32_t q = xm ? 0u : 1u;
    q = __builtin_amdgcn_alignbit(q, __float_as_uint(du), 31);
    const float dv_ = dv + 0.0f;
    q = __builtin_amdgcn_alignbit(q, __float_as_uint(dv_), 31);
    q = __builtin_amdgcn_alignbit(q, __float_as_uint(rr.rcp_z), 31);        // the sign of 1/d_z is the sign of d_z
    const uint32_t record = __float_as_uint(tiny_int(q) * (float)kClassStride + tiny_int(classes_addr));
    ScanClass c;
    {
        lds_u32x4_ptr rec = (lds_u32x4_ptr)(uintptr_t)record;
        u32x4* dst = reinterpret_cast<u32x4*>(&c);
        dst[0] = rec[0]; dst[1] = rec[1]; dst[2] = rec[2]; dst[3] = rec[3]; dst[4] = rec[4];
    }

    // 1 / |d| of a component that may be 0: adding the smallest normal number to the magnitude keeps the reciprocal finite (at
    // most 8.5e37) and changes no component of 2^-101 or more.  (Added to the signed component it would take those just below
    // 0 to 0 or to a denormal number, whose reciprocal is infinite.)
    const float dua = fabsf(du);
    const float inv_u = __builtin_amdgcn_rcpf(dua + kSmallest);
    const float dt_v = __builtin_amdgcn_rcpf(fabsf(dv) + kSmallest), rcp_z = rr.rcp_z, dt_z = fabsf(rcp_z);
    // first crossing on an axis: the distance to the first plane in the ray's direction times |1/d| (along z: from
    // the image row's record, see RowRecord)
    float t0_v, t0_z, t_end;
    float t_in_box = 0.0f;
    int entry_face = 0;
    bool misses = false;
    if constexpr (kOutside) {
        // the slab test, the entry cell along v and z and the first crossings from there (see EntryClass; the row record holds
        // the parameters of the box's sides along z): the values of enter_box, in the order a class knows them
        EntryClass e;
        {
            lds_u32x4_ptr rec = (lds_u32x4_ptr)(uintptr_t)(record + (uint32_t)sizeof(ScanClass));
            u32x4* dst = reinterpret_cast<u32x4*>(&e);
            dst[0] = rec[0]; dst[1] = rec[1];
        }
        const float Pv = __int_as_float(c.i0), last_v = __int_as_float(c.pad), rcp_v = copysignf(dt_v, dv_);
        const float near_u = e.near_u * inv_u, near_v = c.dist_v * dt_v, near_z = rr.t0_z;
        const float t_far = vmin3(e.far_u * inv_u, c.nv_max * dt_v, rr.tend_z);
        const float t_near = vmax3(near_u, near_v, near_z);
        misses = !(t_near <= t_far) || !(t_far >= 0.0f) || !from_outside->finite;
        if (__ballot(!misses) == 0) return Hit{ -1, 0, 0.0f };               // no ray of the tile meets the box
        t_in_box = vmax(t_near, 0.0f);
        const bool by_v = xm ? near_v > near_u : near_v >= near_u;          // (x before y before z)
        const bool by_z = near_z > (by_v ? near_v : near_u);
        entry_face = by_z ? c.face_z : (by_v ? c.face_v : c.face_u);
        if (!(t_near > 0.0f)) entry_face = from_outside->faces.of(6);
        // (a cell number below 0 only from rounding; a ray that enters through a side of the axis stands in its first cell)
        const float dz = from_outside->dz, top_1 = (float)(from_outside->top - 1);
        float j = vmed3(floorf(fmaf(t_in_box, dv, Pv)), 0.0f, last_v), k = vmed3(floorf(fmaf(t_in_box, dz, from_outside->P[2])), 0.0f, top_1);
        const bool stands = t_near > 0.0f;
        if (stands && by_v && !by_z) j = last_v - e.planes_v;
        if (stands && by_z) k = top_1 - e.planes_z;
        // (the tiny distance stands for "never" where a component is 0 and the camera is exactly on the plane ahead)
        t0_v = vmax(((j + e.ahead_v) - Pv + kTinyDistance) * rcp_v, t_in_box);
        t0_z = vmax(((k + e.ahead_z) - from_outside->P[2] + kTinyDistance) * rcp_z, t_in_box);
        t_end = vmax(vmin3(c.uexit * inv_u, fmaf(fmaf(e.per_cell_v, j, e.planes_v), dt_v, t0_v), fmaf(fmaf(e.per_cell_z, k, e.planes_z), dt_z, t0_z)), t_in_box);
        // the record's address and index are those of cell (0,0,0)
        c.addr0 = __float_as_int(fmaf(k, fabsf(c.row_step_z), fmaf(j, tiny_int(8u), tiny_int((uint32_t)c.addr0))));
        c.idx0 = fmaf(k, fabsf(c.stride_z), fmaf(j, fabsf(c.stride_v), c.idx0));
        c.i0 = min(max((int)fmaf(t_in_box, dua, c.Pu), 0), c.um1);
        if (misses) t0_v = t0_z = t_end = 0.0f;
    } else {
        t0_v = c.dist_v * dt_v;
        t0_z = rr.t0_z;
        // leaving the grid: same n*dt + t0 expression as the crossings, so the comparison below is exact
        t_end = vmin3(c.uexit * inv_u, fmaf(c.nv_max, dt_v, t0_v), rr.tend_z);
    }

    // crossings made so far along v and z (without sign; the directions sit in the class), and the parameters
    // of the next ones: t_v = n_v*dt_v + t0_v, t_z likewise
    float t_v, t_z, n_v = 0.0f, n_z = 0.0f;
    uint32_t addr = (uint32_t)c.addr0;
    uint64_t r, in_range;
    int i_last;
    // One turn of the loop scans the current row from cell i_from up to the cell i_to where the ray leaves
    // it (parameter t_out = min(t_v, t_z), for narrow grids also capped at t_end): r = row >> i_from,
    // in_range = r << (63 - (i_to - i_from)), non-zero if a solid cell lies in the run; the loop ends there, or
    // when t_out reaches t_end (the ray leaves the grid); otherwise the ray crosses the nearer of the two planes
    // (v first at a tie), the counter of that axis and the row address step, and the crossing parameters are
    // recomputed.  The second shift count is 63 - (i_to - i_from) = (i_from + ~i_to) mod 64: one xor-add, the
    // shifter ignores the upper bits.  Nothing after the loop needs i_from: the hit cell follows from
    // the lowest set bit of in_range and i_to, and bit 0 of r tells whether it is the row's entry cell.
    // The next row is requested as soon as its address is known, at the end of the turn before (render -1 %).
    uint64_t row = 0;
    if constexpr (!kCoarse) row = *(lds_u64_ptr)(uintptr_t)addr;
    if constexpr (kOutside) row = misses ? 0ull : row;
    int i_a = c.i0, i_b;
    if constexpr (kCoarse) {
        // Coarse level: after `fine_turns` ordinary turns a ray first looks at the PAIR of rows it is in (the OR of
        // rows 2J and 2J+1 of its layer), over the whole run of cells it covers before it leaves the pair or the
        // layer.  An empty run takes it there in one turn (one or two v crossings, or one v crossing and the z
        // crossing, with the very comparisons the ordinary turns would make, so the state it arrives in is the
        // state they would arrive in); otherwise it takes one ordinary turn.  Every decision uses the same
        // crossing parameters as the ordinary scan: the result is the same bit for bit.
        PairClass pc;
        *reinterpret_cast<u32x4*>(&pc) = *(lds_u32x4_ptr)(uintptr_t)(record + (uint32_t)sizeof(ScanClass));
        t_v = t0_v; t_z = t0_z;
        uint32_t addr_p = (uint32_t)pc.addr0;
        int inner = pc.inner0;                  // the next v plane lies inside the current pair
        int i_from = i_a;
        r = 0; in_range = 0; i_last = i_from;
        for (int turn = 0;; ++turn) {
            if (turn >= fine_turns) {
                const float t_pair = inner ? fmaf(n_v + 1.0f, dt_v, t0_v) : t_v;     // where the ray leaves the pair along v
                const float t_out = kNarrow ? vmin3(t_pair, t_z, t_end) : vmin(t_pair, t_z);
                const float u_out = fmaf(t_out, dua, c.Pu);
                const int i_to = kNarrow ? (int)u_out : min((int)u_out, c.um1);
                const uint64_t pair_row = *(lds_u64_ptr)(uintptr_t)addr_p;
                const uint64_t pr = pair_row >> i_from;
                const uint64_t pin = pr << ((((i_to) ^ -1) + (i_from)) & 63);
                if (pin == 0) {
                    if (!(t_out < t_end)) { r = pr; in_range = 0; i_last = i_to; break; }   // leaves the grid: a miss
                    if (t_pair <= t_z) {
                        // out of the pair along v: the plane inside it (if it was still ahead) and the one behind it
                        n_v += inner ? 2.0f : 1.0f;
                        addr += (uint32_t)(inner ? 2 * c.sv : c.sv);
                        addr_p += (uint32_t)pc.sv;
                        inner = 1;
                    } else {
                        // the z crossing comes first; the plane inside the pair may still come before it
                        const bool mid = inner && t_v <= t_z;
                        n_v += mid ? 1.0f : 0.0f;
                        addr += (uint32_t)(mid ? c.sv : 0);
                        inner = mid ? 0 : inner;
                        n_z += 1.0f;
                        addr += (uint32_t)c.sz;
                        addr_p += (uint32_t)pc.sz;
                    }
                    t_v = fmaf(n_v, dt_v, t0_v);
                    t_z = fmaf(n_z, dt_z, t0_z);
                    i_from = i_to;
                    continue;
                }
            }
            // an ordinary turn on the row the ray is in
            const uint64_t fine_row = *(lds_u64_ptr)(uintptr_t)addr;
            const float t_out = kNarrow ? vmin3(t_v, t_z, t_end) : vmin(t_v, t_z);
            const float u_out = fmaf(t_out, dua, c.Pu);
            const int i_to = kNarrow ? (int)u_out : min((int)u_out, c.um1);
            r = fine_row >> i_from;
            in_range = r << ((((i_to) ^ -1) + (i_from)) & 63);
            i_last = i_to;
            if ((in_range != 0) | !(t_out < t_end)) break;
            const bool cv = t_v <= t_z;
            if (cv) {
                n_v += 1.0f;
                addr += (uint32_t)c.sv;
                if (!inner) addr_p += (uint32_t)pc.sv;      // that plane bounded the pair
                inner ^= 1;
            } else {
                n_z += 1.0f;
                addr += (uint32_t)c.sz;
                addr_p += (uint32_t)pc.sz;
            }
            t_v = fmaf(n_v, dt_v, t0_v);
            t_z = fmaf(n_z, dt_z, t0_z);
            i_from = i_to;
        }
    } else
    // The loop in assembly: the compiler's structured control flow spends about ten scalar instructions per turn
    // on lane masks (two breaks per trip); written out, a turn needs one, the branch: the two comparisons that
    // decide whether a lane goes on write the execution mask themselves.  Lanes that are done simply leave
    // the execution mask (it only ever shrinks; restored after the loop), so every register of a finished lane
    // keeps the values of its last turn.  The cell index alternates between i_a and i_b from turn to turn; the later cell
    // of a finished lane is the larger of the two.
    // The v-or-z decision of a turn is taken at its top (VCC), well ahead of the select that reads it (a vector instruction
    // may not read a lane mask within two instructions of the one that wrote it).
    // What bounds the loop is the issue of comparisons, selects, conversions and shifts, of which other waves' float adds and
    // multiply-adds run beside (see tiny_int); so the counters and the row address are float arithmetic with one select per
    // turn (two and an integer add before; 4096 x 2 of 40x40x16: step 304 -> 301 us, 2048 x 4 of 64x64x32 1085 -> 1070): the
    // row address as a number of bytes in a denormal, and for the first 13 turns, written out one by one, the z crossings as
    // the turns that are not v crossings (five turns written out: 64x64x32 +1.2 %).  A multiply-add whose three vector
    // registers all have even or all odd numbers takes twice the time: the temporaries, the counters and the address have
    // registers of their own (v48 to v55) that rule it out.
    {
        uint64_t exec_save, m_go, m_empty;
        int sh;
        float inc, row_addr = tiny_int(addr);
        // the run of cells [IFROM, ITO] of the current row: ITO from the parameter at which the ray leaves the row
        // (TOUT, NARROW: capped at the grid exit; else the cell is clamped to U - 1), then the two shifts
#define MV_ASM_TEST(TV, TZ, IFROM, ITO, CELL, WAIT)                                     \
            "v_cmp_le_f32_e32 vcc, " TV ", " TZ "\n\t"                                   \
            CELL(TV, TZ, ITO)                                                           \
            WAIT                                                                        \
            "v_lshrrev_b64 %[r], " IFROM ", %[row]\n\t"                                 \
            "v_xad_u32 %[sh], " ITO ", -1, " IFROM "\n\t"                               \
            "v_lshlrev_b64 %[inr], %[sh], %[r]\n\t"
#define MV_ASM_CELL_NARROW(TV, TZ, ITO)                                                 \
            "v_min3_f32 v51, " TV ", " TZ ", %[tend]\n\t"                                \
            "v_fma_f32 v53, v51, |%[du]|, %[pu]\n\t"                                    \
            "v_cvt_i32_f32_e32 " ITO ", v53\n\t"
#define MV_ASM_CELL_WIDE(TV, TZ, ITO)                                                   \
            "v_min_f32_e32 v51, " TV ", " TZ "\n\t"                                      \
            "v_fma_f32 v53, v51, |%[du]|, %[pu]\n\t"                                    \
            "v_cvt_i32_f32_e32 v53, v53\n\t"                                            \
            "v_min_i32_e32 " ITO ", v53, %[um1]\n\t"
        // lanes that found a solid cell leave first (their in_range stays non-zero), then the lanes whose ray leaves
        // the grid in this row (theirs is zero): each comparison writes the execution mask itself
#define MV_ASM_LEAVE                                                                    \
            "v_cmpx_eq_u64_e64 %[mempty], 0, %[inr]\n\t"                                \
            "v_cmpx_lt_f32_e64 %[mgo], v51, %[tend]\n\t"                                \
            "s_cbranch_execz 2f\n\t"
#define MV_ASM_NEXT_ROW                                                                 \
            "v_fma_f32 %[tv], %[nv], %[dtv], %[t0v]\n\t"                                \
            "v_fma_f32 %[tz], %[nz], |%[rz]|, %[t0z]\n\t"
#define MV_ASM_READ(INC)                                                                \
            "v_add_f32_e32 v55, v55, %[szd]\n\t"                                       \
            "v_cndmask_b32_e64 " INC ", 0, 1.0, vcc\n\t"                               \
            "v_fma_f32 v55, " INC ", %[svz], v55\n\t"                                  \
            "ds_read_b64 %[row], v55\n\t"
#define MV_ASM_FIRST_ADVANCE                                                            \
            MV_ASM_READ("%[nv]")                                                        \
            "v_sub_f32_e32 %[nz], 1.0, %[nv]\n\t"                                       \
            MV_ASM_NEXT_ROW
        // (after N turns the crossings along v and z add up to N)
#define MV_ASM_ADVANCE(N)                                                               \
            MV_ASM_READ("%[inc]")                                                       \
            "v_add_f32_e32 %[nv], %[nv], %[inc]\n\t"                                    \
            "v_sub_f32_e32 %[nz], " N ", %[nv]\n\t"                                     \
            MV_ASM_NEXT_ROW
#define MV_ASM_ADVANCE_ANY                                                              \
            MV_ASM_READ("%[inc]")                                                       \
            "v_add_f32_e32 %[nv], %[nv], %[inc]\n\t"                                    \
            "v_sub_f32_e32 %[inc], 1.0, %[inc]\n\t"                                     \
            "v_add_f32_e32 %[nz], %[nz], %[inc]\n\t"                                    \
            MV_ASM_NEXT_ROW
#define MV_ASM_WAIT "s_waitcnt lgkmcnt(0)\n\t"
#define MV_ASM_TO_A(CELL) MV_ASM_TEST("%[tv]", "%[tz]", "%[ib]", "%[ia]", CELL, MV_ASM_WAIT) MV_ASM_LEAVE
#define MV_ASM_TO_B(CELL) MV_ASM_TEST("%[tv]", "%[tz]", "%[ia]", "%[ib]", CELL, MV_ASM_WAIT) MV_ASM_LEAVE
#define MV_ASM_TWO(CELL, M, N) MV_ASM_TO_A(CELL) MV_ASM_ADVANCE(M) MV_ASM_TO_B(CELL) MV_ASM_ADVANCE(N)
        // (the first row has arrived when the statement starts: it is one of its inputs)
#define MV_ASM_LOOP(CELL)                                                               \
            "s_mov_b64 %[save], exec\n\t"                                               \
            "v_mov_b32_e32 %[nv], 0\n\t"                                                \
            "v_mov_b32_e32 %[nz], 0\n\t"                                                \
            MV_ASM_TEST("%[t0v]", "%[t0z]", "%[ia]", "%[ib]", CELL, "")                  \
            MV_ASM_LEAVE                                                                \
            MV_ASM_FIRST_ADVANCE                                                        \
            MV_ASM_TWO(CELL, "2.0", "0x40400000")                                       \
            MV_ASM_TWO(CELL, "4.0", "0x40a00000")                                       \
            MV_ASM_TWO(CELL, "0x40c00000", "0x40e00000")                                \
            MV_ASM_TWO(CELL, "0x41000000", "0x41100000")                                \
            MV_ASM_TWO(CELL, "0x41200000", "0x41300000")                                \
            MV_ASM_TWO(CELL, "0x41400000", "0x41500000")                                \
            "1:\n\t"                                                                    \
            MV_ASM_TO_A(CELL) MV_ASM_ADVANCE_ANY                                        \
            MV_ASM_TO_B(CELL) MV_ASM_ADVANCE_ANY                                        \
            "s_branch 1b\n"                                                             \
            "2:\n\t"                                                                    \
            "s_mov_b64 exec, %[save]\n\t"
#define MV_ASM_OPERANDS                                                                                              \
                : [save] "=&s"(exec_save), [mgo] "=&s"(m_go), [mempty] "=&s"(m_empty),                                \
                  [inc] "=&v"(inc), [sh] "=&v"(sh), [r] "=&v"(r), [inr] "=&v"(in_range), [ib] "=&v"(i_b),             \
                  [tv] "=&v"(t_v), [tz] "=&v"(t_z), [ia] "+&v"(i_a), [row] "+&v"(row), "+&{v55}"(row_addr),             \
                  [nv] "=&{v49}"(n_v), [nz] "=&{v48}"(n_z)                                                            \
                : [tend] "v"(t_end), [du] "v"(du), [pu] "v"(c.Pu), [svz] "v"(c.row_step_vz), [szd] "v"(c.row_step_z), \
                  [dtv] "v"(dt_v),                                                                                    \
                  [rz] "v"(rcp_z), [t0v] "{v50}"(t0_v), [t0z] "v"(t0_z), [um1] "v"(c.um1)                             \
                : "vcc", "scc", "memory", "v51", "v53"
        if (kNarrow) asm volatile(MV_ASM_LOOP(MV_ASM_CELL_NARROW) MV_ASM_OPERANDS);
        else         asm volatile(MV_ASM_LOOP(MV_ASM_CELL_WIDE) MV_ASM_OPERANDS);
#undef MV_ASM_OPERANDS
#undef MV_ASM_LOOP
#undef MV_ASM_TWO
#undef MV_ASM_ADVANCE_ANY
#undef MV_ASM_ADVANCE
#undef MV_ASM_FIRST_ADVANCE
#undef MV_ASM_READ
#undef MV_ASM_NEXT_ROW
#undef MV_ASM_WAIT
#undef MV_ASM_TO_A
#undef MV_ASM_TO_B
#undef MV_ASM_LEAVE
#undef MV_ASM_CELL_WIDE
#undef MV_ASM_CELL_NARROW
#undef MV_ASM_TEST
        i_last = max(i_a, i_b);
    }
    const bool found = in_range != 0;

    // in_range is r moved up so that cell i_last sits at bit 63: its lowest set bit p is cell i_last - (63 - p)
    // mirrored cell along u
    const float iu_f = tiny_to_float(tiny_int((uint32_t)i_last) + tiny_int((uint32_t)ctz64_nonzero(in_range))) - 63.0f;
    const bool along_row = low_bit((uint32_t)r) == 0u;                          // not the row's entry cell
    // the row was entered at the later of the last v crossing and the last z crossing (n-1; for n = 0
    // the expression is <= 0 because the first plane is at most one cell away).  Recomputed with one
    // fused operation each: "t_v - dt_v" would cancel badly for a camera that almost touches a plane.
    const float tv_last = fmaf(n_v - 1.0f, dt_v, t0_v);
    const float tz_last = fmaf(n_z - 1.0f, dt_z, t0_z);
    const bool via_z = tz_last >= tv_last;
    // A hit in the row's entry cell was entered through the later of the two crossings.  The camera's own
    // cell is never solid here (the caller handles that camera before tracing), so the only way to find
    // the entry cell of the first row solid is a camera exactly on a cell boundary looking into the
    // neighbour: both crossings are <= 0 then and the hit is at t = 0 on that boundary.
    const float t_in = vmax3(tv_last, tz_last, 0.0f);
    // distance along u to the near face of the hit cell: the mirrored camera coordinate was rounded once,
    // which matters when the camera almost touches that face; its exact rounding error comes with the class
    const float t_u = ((iu_f - c.Pu) - c.Pu_err) * inv_u;
    const int face_vz = via_z ? c.face_z : c.face_v;
    int face = along_row ? c.face_u : face_vz;
    float t = along_row ? t_u : t_in;
    if constexpr (kOutside) {
        // the voxel the ray meets as it enters the box
        const bool at_entry = !along_row && n_v + n_z == 0.0f;
        face = at_entry ? entry_face : face;
        t = at_entry ? t_in_box : t;
    }
    // voxel index: the class record holds the index of (mirrored cell 0, camera's v cell, camera's layer)
    // and the signed index steps per cell along u and per crossing along v and z
    const float idx_f = fmaf(n_z, c.stride_z, fmaf(n_v, c.stride_v, fmaf(iu_f, c.stride_u, c.idx0)));
    Hit h;
    // face and t are only meaningful for idx >= 0 (-1.0f becomes a negative number other than -1); the caller substitutes the
    // miss values
    h.idx = __float_as_int(float_to_tiny(found ? idx_f : -1.0f));
    h.face = face;
    h.t = t;
    return h;
}

// Row scan for grids of any width: the traversal of trace_rows, but a row is looked at through a window of 32 cells that
// starts wherever the ray is (two dwords of the row and one funnel shift); a run of more than 32 cells takes several
// windows.  There is one copy of the rows for both directions: for a ray that runs towards lower cells the window starts
// where its run ends, and the first cell it meets is the highest one.  The record's address and index steps are those of rows
// of several words; `pad` is -1 for mirrored classes, else 0.  Bits beyond a row's end belong to its neighbour in LDS and
// never count: runs end at cell U - 1.  Ends for every input as trace_rows does; a window that does not reach the end of the
// run advances it by 32 cells.  Bound by instruction issue (256 x 2 worlds of 96x96x16 at 128x72, upload + cameras + render:
// 184 us cell by cell; 97 us with the loop made by the compiler, a lane mask for every way out of it and every run's last cell
// checked against the u crossings; 69 us written out, with that check only where the position cannot tell the cell).
template <bool kOutside>
__device__ __forceinline__ Hit trace_windows(uint32_t classes_addr, float dx, float dy, const RowRecord& rr, float edge,
                                             const OutsideCamera* from_outside = nullptr)
{
    const bool xm = fabsf(dx) >= fabsf(dy);
    const float du = xm ? dx : dy;
    const float dv = xm ? dy : dx;
    uint32_t q = xm ? 0u : 1u;                      // the class index, as in trace_rows
    q = __builtin_amdgcn_alignbit(q, __float_as_uint(du), 31);
    q = __builtin_amdgcn_alignbit(q, __float_as_uint(dv + 0.0f), 31);
    q = __builtin_amdgcn_alignbit(q, __float_as_uint(rr.rcp_z), 31);
    ScanClass c;
    {
        lds_u32x4_ptr rec = (lds_u32x4_ptr)(uintptr_t)(classes_addr + q * (uint32_t)kClassStride);
        u32x4* dst = reinterpret_cast<u32x4*>(&c);
        dst[0] = rec[0]; dst[1] = rec[1]; dst[2] = rec[2]; dst[3] = rec[3]; dst[4] = rec[4];
    }
    const float dua = fabsf(du);
    const float inv_u = safe_rcp(dua);
    const float rcp_v = safe_rcp(dv);
    const float dt_v = fabsf(rcp_v), dt_z = fabsf(rr.rcp_z);
    float t0_u, t0_v, t0_z, t_end;
    BoxEntry in{};
    if constexpr (kOutside) {
        in = enter_box(*from_outside, dx, dy, xm, rr.rcp_z);
        if (__ballot(!in.misses) == 0) return Hit{ -1, 0, 0.0f };
        t0_u = in.t0_u; t0_v = in.t0_v; t0_z = in.t0_z;
        t_end = vmax(vmin3(fmaf(in.left_u, inv_u, t0_u), fmaf(in.left_v, dt_v, t0_v), fmaf(in.left_z, dt_z, t0_z)), in.t);
        const int V = xm ? from_outside->Y : from_outside->X;
        c.addr0 += abs(c.sv) * (in.k * V + in.j);
        c.idx0 += (float)((in.k * from_outside->Y) * from_outside->X + in.j * (xm ? from_outside->X : 1));
        c.i0 = du < 0.0f ? c.um1 - in.i : in.i;
    } else {
        // (an axis along which the ray does not move at all: its first plane is never reached, also from a camera exactly
        // on the far side of the grid, whose distance to it is 0)
        t0_u = du == 0.0f ? kNever : c.uexit * inv_u;
        t0_v = dv == 0.0f ? kNever : c.dist_v * dt_v;
        t0_z = rr.t0_z;
        t_end = vmin3(fmaf((float)(c.um1 - c.i0), inv_u, t0_u), fmaf(c.nv_max, dt_v, t0_v), rr.tend_z);
    }
    const int mirrored = c.pad;                     // -1 or 0
    const int origin = mirrored & (c.um1 + 1);      // mirrored cell i is cell ~i + U
    const uint64_t is_mirrored = __ballot(mirrored != 0), y_scan = __ballot(!xm);
    const uint64_t live = kOutside ? __ballot(!in.misses) : ~0ull;
    float t_v = t0_v, t_z = t0_z, n_v, n_z;
    uint32_t in_range = 0;
    int i_row = c.i0, i_win = c.i0, i_last;
    // A turn: the run of cells the ray covers in its row ends where the ray is at t_out; the window that starts (for a
    // mirrored class: ends) there is shifted so that only the cells of the run are left.
    // The last cell of the run is put right by the u crossings themselves wherever the ray's position is too close to a
    // voxel edge to tell: every choice of the next crossing is then the per-cell tracer's own comparison, ties included (x
    // before y before z, and none at or behind the far side), and so are the cells visited, for cameras inside the grid and
    // no higher than the solids.  From higher up the z crossings are counted from the top of the solids and not from the
    // camera's own layer (depths differ in the last bit), and a ray that leaves the solids' top plane exactly through
    // a voxel edge does not look at the voxel beside that edge, as one that leaves the grid.
    // How close is too close: the parameter of a u crossing has three roundings of at most 2^-23 and one reciprocal of one
    // unit (2^-23) in it, the position two roundings and the mirrored camera coordinate one, each relative to the largest
    // distance to a plane, D (the grid's size, for cameras outside plus theirs): less than 2^-20 D together.  `edge` is half
    // a voxel minus that.  Such a turn, about one in fifty, and one whose run is longer than a window, takes a path of its own
    // for the whole wave (3 below).
    // Registers: see trace_rows; lanes that are done leave the execution mask.  v40/v41 hold the two dwords of the window.
    {
        uint64_t exec_save, exec_turn, cv, m_a, m_b, m_c, strict;
        float t_out, u_out, u_prev = (float)c.i0, addr = tiny_int((uint32_t)c.addr0), tmp;
        int x, sh;
        asm volatile(
            "s_mov_b64 %[save], exec\n\t"
            "s_and_b64 exec, exec, %[live]\n\t"
            "v_mov_b32_e32 %[nv], 0\n\t"
            "v_mov_b32_e32 %[nz], 0\n"
            "1:\n\t"
            "v_cmp_le_f32_e64 %[cv], %[tv], %[tz]\n\t"
            "v_min3_f32 %[tout], %[tv], %[tz], %[tend]\n\t"
            "v_fma_f32 %[uout], %[tout], |%[du]|, %[pu]\n\t"
            "v_fract_f32_e32 %[tmp], %[uout]\n\t"
            "v_sub_f32_e32 %[up], %[uout], %[up]\n\t"
            "v_cvt_i32_f32_e32 %[ito], %[uout]\n\t"
            "v_add_f32_e32 %[tmp], -0.5, %[tmp]\n\t"
            "v_cmp_ngt_f32_e32 vcc, 0x41f00000, %[up]\n\t"                 // 30: a run of more than 31 cells, to be sure
            "v_cmp_nlt_f32_e64 %[ma], |%[tmp]|, %[edge]\n\t"
            "s_or_b64 vcc, vcc, %[ma]\n\t"
            "s_cbranch_vccnz 3f\n\t"
            "v_cndmask_b32_e64 %[x], %[irow], %[ito], %[mir]\n\t"
            "v_xad_u32 %[x], %[x], %[m], %[org]\n\t"
            "v_lshrrev_b32_e32 %[sh], 5, %[x]\n\t"
            "v_lshl_add_u32 %[sh], %[sh], 2, v45\n\t"
            "ds_read2_b32 v[40:41], %[sh] offset1:1\n\t"
            "v_xad_u32 %[sh], %[ito], -1, %[irow]\n\t"
            "s_waitcnt lgkmcnt(0)\n\t"
            "v_alignbit_b32 %[inr], v41, v40, %[x]\n\t"
            "v_lshlrev_b32_e32 %[inr], %[sh], %[inr]\n"
            "2:\n\t"
            "v_cmpx_eq_u32_e64 %[ma], 0, %[inr]\n\t"
            "v_cmpx_lt_f32_e64 %[mb], %[tout], %[tend]\n\t"
            "s_cbranch_execz 9f\n\t"
            "v_add_f32_e32 v45, v45, %[szd]\n\t"
            "v_cndmask_b32_e64 %[tmp], 0, 1.0, %[cv]\n\t"
            "v_fma_f32 v45, %[tmp], %[svz], v45\n\t"
            "v_add_f32_e32 %[nv], %[nv], %[tmp]\n\t"
            "v_sub_f32_e32 %[tmp], 1.0, %[tmp]\n\t"
            "v_add_f32_e32 %[nz], %[nz], %[tmp]\n\t"
            "v_fma_f32 %[tv], %[nv], |%[rv]|, %[t0v]\n\t"
            "v_fma_f32 %[tz], %[nz], |%[rz]|, %[t0z]\n\t"
            "v_mov_b32_e32 %[irow], %[ito]\n\t"
            "v_mov_b32_e32 %[iwin], %[ito]\n\t"
            "v_mov_b32_e32 %[up], %[uout]\n\t"
            "s_branch 1b\n"
            "3:\n\t"
            // the crossing that ends the run comes before (strict) or not after a u crossing at the same parameter
            "v_cmp_nlt_f32_e64 %[strict], %[tout], %[tend]\n\t"
            "s_and_b64 %[ma], %[yscan], %[cv]\n\t"
            "s_or_b64 %[strict], %[strict], %[ma]\n\t"
            "v_max_i32_e32 %[ito], %[ito], %[irow]\n\t"
            "v_min_i32_e32 %[ito], %[ito], %[um1]\n\t"
            "v_sub_u32_e32 %[tmp], %[ito], %[i0]\n\t"
            "v_cvt_f32_i32_e32 %[tmp], %[tmp]\n\t"
            "v_fma_f32 %[up], %[tmp], %[invu], %[t0u]\n\t"
            "v_cmp_lt_f32_e64 %[ma], %[up], %[tout]\n\t"
            "v_cmp_le_f32_e64 %[mb], %[up], %[tout]\n\t"
            "s_andn2_b64 %[mb], %[mb], %[strict]\n\t"
            "s_or_b64 %[ma], %[ma], %[mb]\n\t"                              // one cell further
            "v_add_f32_e32 %[tmp], -1.0, %[tmp]\n\t"
            "v_fma_f32 %[up], %[tmp], %[invu], %[t0u]\n\t"
            "v_cmp_lt_f32_e64 %[mc], %[up], %[tout]\n\t"
            "v_cmp_le_f32_e64 %[mb], %[up], %[tout]\n\t"
            "s_andn2_b64 %[mb], %[mb], %[strict]\n\t"
            "s_or_b64 %[mc], %[mc], %[mb]\n\t"
            "s_or_b64 %[mc], %[mc], %[ma]\n\t"
            "v_cmp_gt_i32_e64 %[mb], %[ito], %[irow]\n\t"
            "s_andn2_b64 %[mb], %[mb], %[mc]\n\t"                           // one cell less
            "v_cndmask_b32_e64 %[tmp], 0, 1, %[ma]\n\t"
            "v_add_u32_e32 %[tmp], %[tmp], %[ito]\n\t"
            "v_min_i32_e32 %[ito], %[tmp], %[um1]\n\t"
            "v_cndmask_b32_e64 %[tmp], 0, -1, %[mb]\n\t"
            "v_add_u32_e32 %[up], %[ito], %[tmp]\n\t"                       // the run's last cell
            "s_mov_b64 %[turn], exec\n"
            "4:\n\t"
            "v_add_u32_e32 %[ito], 31, %[iwin]\n\t"
            "v_min_i32_e32 %[ito], %[ito], %[up]\n\t"
            "v_cndmask_b32_e64 %[x], %[iwin], %[ito], %[mir]\n\t"
            "v_xad_u32 %[x], %[x], %[m], %[org]\n\t"
            "v_lshrrev_b32_e32 %[sh], 5, %[x]\n\t"
            "v_lshl_add_u32 %[sh], %[sh], 2, v45\n\t"
            "ds_read2_b32 v[40:41], %[sh] offset1:1\n\t"
            "v_xad_u32 %[sh], %[ito], -1, %[iwin]\n\t"
            "s_waitcnt lgkmcnt(0)\n\t"
            "v_alignbit_b32 %[inr], v41, v40, %[x]\n\t"
            "v_lshlrev_b32_e32 %[inr], %[sh], %[inr]\n\t"
            "v_cmpx_eq_u32_e64 %[ma], 0, %[inr]\n\t"
            "v_cmpx_lt_i32_e64 %[ma], %[ito], %[up]\n\t"
            "s_cbranch_execz 5f\n\t"
            "v_add_u32_e32 %[iwin], 1, %[ito]\n\t"
            "s_branch 4b\n"
            "5:\n\t"
            "s_mov_b64 exec, %[turn]\n\t"
            "s_branch 2b\n"
            "9:\n\t"
            "s_mov_b64 exec, %[save]\n\t"
            : [save] "=&s"(exec_save), [turn] "=&s"(exec_turn), [cv] "=&s"(cv), [ma] "=&s"(m_a), [mb] "=&s"(m_b), [mc] "=&s"(m_c),
              [strict] "=&s"(strict), [tout] "=&v"(t_out), [uout] "=&v"(u_out), [tmp] "=&v"(tmp), [x] "=&v"(x), [sh] "=&v"(sh),
              [inr] "+&v"(in_range), [ito] "=&v"(i_last), [irow] "+&v"(i_row), [iwin] "+&v"(i_win), [up] "+&v"(u_prev),
              [tv] "+&v"(t_v), [tz] "+&v"(t_z), "+&{v45}"(addr), [nv] "=&{v43}"(n_v), [nz] "=&{v42}"(n_z)
            : [live] "s"(live), [tend] "v"(t_end), [du] "v"(du), [pu] "v"(c.Pu), [edge] "s"(edge), [mir] "s"(is_mirrored), [yscan] "s"(y_scan),
              [m] "v"(mirrored), [org] "v"(origin), [rv] "v"(rcp_v), [rz] "v"(rr.rcp_z), [t0v] "v"(t0_v), [t0z] "v"(t0_z),
              [szd] "v"(c.row_step_z), [svz] "v"(c.row_step_vz), [um1] "v"(c.um1), [i0] "v"(c.i0),
              [invu] "v"(inv_u), [t0u] "v"(t0_u)
            : "vcc", "scc", "memory", "v40", "v41");
    }
    // as in trace_rows.  The first solid cell the ray meets: bit 31 of in_range is cell i_last and the lowest bit counts, for
    // mirrored classes bit 31 is the window's first cell and the highest one counts.
    const bool found = in_range != 0;
    uint32_t lowest, highest;
    asm("v_ffbl_b32 %0, %1" : "=v"(lowest) : "v"(in_range));
    asm("v_ffbh_u32 %0, %1" : "=v"(highest) : "v"(in_range));
    const int iu = mirrored ? i_win + (int)highest : i_last - 31 + (int)lowest;
    const bool along_row = iu != i_row;
    const float tv_last = fmaf(n_v - 1.0f, dt_v, t0_v);
    const float tz_last = fmaf(n_z - 1.0f, dt_z, t0_z);
    // (from a camera exactly on a z plane a rising ray has that plane one crossing behind it, at parameter 0)
    const bool via_z = tz_last >= tv_last && n_z > 0.0f;
    const float t_in = vmax3(tv_last, tz_last, 0.0f);
    const float iu_f = (float)iu;
    const float t_u = fmaf(iu_f - (float)c.i0 - 1.0f, inv_u, t0_u);
    int face = along_row ? c.face_u : (via_z ? c.face_z : c.face_v);
    float t = along_row ? t_u : t_in;
    if constexpr (kOutside) {
        const bool at_entry = !along_row && n_v + n_z == 0.0f;
        face = at_entry ? in.face : face;
        t = at_entry ? in.t : t;
    }
    const int idx = (int)fmaf(n_z, c.stride_z, fmaf(n_v, c.stride_v, fmaf(iu_f, c.stride_u, c.idx0)));
    return Hit{ found ? idx : -1, face, t };
}

// one dword or byte per lane at a scalar address plus a 32-bit offset of the lane
__device__ __forceinline__ void store_dword(uint32_t lane_offset, uint32_t v, const void* at)
{
    asm volatile("global_store_dword %0, %1, %2" :: "v"(lane_offset), "v"(v), "s"(at) : "memory");
}
__device__ __forceinline__ void store_byte(uint32_t lane_offset, uint32_t v, const void* at)
{
    asm volatile("global_store_byte %0, %1, %2" :: "v"(lane_offset), "v"(v), "s"(at) : "memory");
}

// filled columns of an indicator bar: one float32 multiply, one float32 add, floor, clamp
__device__ __forceinline__ int bar_columns(float fraction, int width)
{
    const float columns = floorf(__fadd_rn(__fmul_rn(fraction, (float)width), 0.5f));
    return (int)fminf(fmaxf(columns, 0.0f), (float)width);              // NaN falls to 0
}

// colour of lane+1 within each group of four lanes (lane 3 of the group keeps its own): DPP
// quad_perm [1,2,3,3]
__device__ __forceinline__ uint32_t next_in_quad(uint32_t v)
{
    // (every lane of a quad is named by the permutation, so no lane falls back on the first operand: with the
    // bound-control bit set the compiler need not initialise one)
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xF9, 0xF, 0xF, true);
}

// SCAN: which tracer a launch is for.  Each has a kernel of its own: in a kernel with the window scan the per-cell tracer kept
// 115 values in spill registers instead of 2 (256 x 2 of 128x128x40, full height:
// render 362 us in the shared kernel, 306 in its own), the window scan 115 instead of 32 (96x96x16: 108 -> 101 us).
// COARSE: with the optional second occupancy level (pairs of rows), row-scan grids only
template <bool AUX, bool PACKED, Scan SCAN, bool COARSE = false>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void render_kernel(RenderParams p)
{
    constexpr bool FAST = SCAN == Scan::kRows, scans = SCAN != Scan::kCells;
    extern __shared__ __align__(16) uint8_t lds[];
    // A workgroup that has just arrived runs its staging at a raised wave priority (the tile loop returns to the
    // default): its few instructions are issued ahead of the tracing waves it shares the SIMDs with, so its
    // loads are on their way sooner.
    __builtin_amdgcn_s_setprio(3);
    const int threads = p.threads;
    // LDS byte address of the dynamic segment: row addresses in the scan-class records are absolute
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;

    // XCD-aware mapping: hardware deals workgroup b to XCD b % 8; each XCD gets a contiguous range of
    // observations so that the workgroups sharing an environment also share an L2.  Within the range the
    // workgroups come strip by strip, observation by observation; the last observations are cut into
    // shorter strips (an XCD's work then ends with short workgroups instead of long ones: a shorter tail).
    const uint32_t b = blockIdx.x;
    const uint32_t xcd = b % kXcds, seq = b / kXcds;
    const uint32_t body = (uint32_t)p.obs_body_per_xcd * (uint32_t)p.blocks_per_obs;
    int obs, part, tiles_per_block, strips;
    if (seq < body) {
        const uint32_t local = p.by_blocks_per_obs.quotient(seq);
        obs = (int)(xcd * (uint32_t)p.obs_per_xcd + local);
        part = (int)(seq - local * (uint32_t)p.blocks_per_obs);
        tiles_per_block = p.tiles_per_block;
        strips = p.blocks_per_obs;
    } else {
        const uint32_t s2 = seq - body;
        const uint32_t t = p.by_blocks_per_obs_tail.quotient(s2);
        const uint32_t local = (uint32_t)p.obs_body_per_xcd + t;
        if (local >= (uint32_t)p.obs_per_xcd) return;
        obs = (int)(xcd * (uint32_t)p.obs_per_xcd + local);
        part = (int)(s2 - t * (uint32_t)p.blocks_per_obs_tail);
        tiles_per_block = p.tiles_per_block_tail;
        strips = p.blocks_per_obs_tail;
    }
    if (obs >= p.num_obs) return;
    // The hardware deals an XCD's consecutive workgroups to its four shader engines in turn: with an even
    // number of strips per observation the same engines would always get the top strips (mostly sky, the
    // slow ones).  Rotating the strips by a hash of the observation index breaks that pairing.
    if ((strips & 1) == 0) {
        const uint32_t turned = (uint32_t)part + (((uint32_t)obs * 2654435761u) >> 16);
        const uint32_t whole = (seq < body ? p.by_blocks_per_obs : p.by_blocks_per_obs_tail).quotient(turned);
        part = (int)(turned - whole * (uint32_t)strips);
    }
    const int env = (int)p.by_agents.quotient((uint32_t)obs);
    if (p.active && p.active[env] == 0) return;         // finished episode: its frame is never drawn
    const GridLayout& g = p.g;
    const int X = g.X, Y = g.Y, Z = g.Z;

    // LDS map, mirrors lds_map() on the host
    const uint32_t off_classes = 0;
    const uint32_t off_scalars = kScanClasses * kClassStride;
    const uint32_t off_rowrec = off_scalars + (uint32_t)((p.W * 4 + 15) & ~15);
    const uint32_t off_lut = off_rowrec + (uint32_t)p.H * 16u;
    const uint32_t off_rows = off_lut + (uint32_t)((kNumFaces * p.materials_plus_one * 4 + 15) & ~15);
    float* lds_sx = reinterpret_cast<float*>(lds + off_scalars);
    RowRecord* lds_rowrec = reinterpret_cast<RowRecord*>(lds + off_rowrec);
    uint64_t* lds_rows = reinterpret_cast<uint64_t*>(lds + off_rows);

    const FaceRows faces = AUX ? FaceRows{ 0, 1 } : FaceRows{ (int)(lds_base + off_lut), 4 * p.materials_plus_one };

    // the camera: uniform for the whole workgroup, read once
    const CameraRecord* __restrict__ recp = p.rec + obs;
    const float P[3] = { recp->P[0], recp->P[1], recp->P[2] };
    const float Fx = recp->F[0], Fy = recp->F[1], Fz = recp->F[2];
    const float Rx = recp->R[0], Ry = recp->R[1], Rz = recp->R[2];
    const float Ux = recp->U[0], Uy = recp->U[1], Uz = recp->U[2];
    const int self_lo = recp->self_lo;

    const int place = recp->place, k0 = recp->layer;
    const bool origin_in_grid = place == kPlaceInGrid;
    // Layers the rays of this camera can reach.  Above the highest solid layer of the environment a rising
    // ray can only miss, so the grid is cut there.  A camera that is itself above every solid sits, for the
    // row scan, in one tall empty layer that reaches from the top of the solids upwards: its layer index is
    // kc = ztop, the plane below it is z = ztop (however far down that is), and only layers 0 .. ztop are
    // ever read (layer ztop is empty by definition).
    const int ztop = p.ztop[env];
    const int kc = min(k0, ztop);
    const int zlim = kc + 1 > ztop ? kc + 1 : ztop;
    // Row scan: only if the launch reserved LDS for those layers (as many as the tallest world the host has heard of
    // needs).  A taller world is traced through the rows in global memory, cell by cell; the pack or the edit that made it
    // tall has told the host, so that a later launch reserves enough.
    const bool use_rows = scans && origin_in_grid && zlim <= p.staged_layers;
    // A camera outside the grid scans rows from where its rays enter it; far outside, by a hair, and for positions that are not
    // numbers, cell by cell.
    const int solid_layers = max(ztop, 1);
    const bool outside_rows = scans && place == kPlaceOutside && solid_layers <= p.staged_layers;
    // Layers copied: those this environment's rays can reach, whatever the launch has room for.  So a launch whose size was
    // fixed long before it runs (a replayed graph), or without knowledge of the worlds, copies no more than another.
    // (Copying as many as the tallest world of the whole batch needs, read from its device word, or all of them where there
    // is none, takes longer: 256 x 4 of 40x40x16 without a batch object 60.5 -> 56.8 us, with one 52.5 -> 52.2 us, 256 x 2
    // of 96x96x16 94.7 -> 81.7 us.)
    const int staged = __builtin_amdgcn_readfirstlane(!scans ? Z : (use_rows ? zlim : solid_layers));
    const bool stage_rows = use_rows || outside_rows;
    const int wx = FAST ? 1 : g.rowwords_x, wy = FAST ? 1 : g.rowwords_y;
    const int sxw = staged * Y * wx, syw = staged * X * wy;        // words of one staged x / y row array
    // Ends the basic block here: otherwise the compiler moves the address arithmetic of the staging into the wait for the
    // camera and the staging's loads start later (4096 x 2 of 40x40x16: render 259 -> 263 us, 2048 x 4 of 64x64x32 983 -> 998).
    if (scans && origin_in_grid && !use_rows) asm volatile("");
    {   // a3: stage pixel scalars, colour table and this environment's bit rows.
        // The first loads of every stream are issued before any of them is consumed (clamped indices
        // instead of branches keep them in one straight run, and a trip of the row loop fetches four
        // words per thread): the staging then waits for one or two memory round trips instead of five.
        const int tid = threadIdx.x;
        const uint32_t* gl = p.lut + (size_t)env * kNumFaces * p.materials_plus_one;
        uint32_t* ll = reinterpret_cast<uint32_t*>(lds + off_lut);
        const int lut_n = kNumFaces * p.materials_plus_one;
        const float first_sx = p.sx[min(tid, p.W - 1)], first_sy = p.sy[min(tid, p.H - 1)];
        const uint32_t first_lut = gl[min(tid, lut_n - 1)];
        const uint64_t* gb = p.bits + (size_t)env * g.env_words;
        if (FAST) {
            if (stage_rows) {
                // arrays: [x rows][x rows mirrored][y rows][y rows mirrored], layers 0 .. staged-1 of each
                uint64_t* ax = lds_rows;
                uint64_t* axm = ax + sxw;
                uint64_t* ay = axm + sxw;
                uint64_t* aym = ay + syw;
                const uint64_t* gy = gb + g.xrow_words;
                const int longest = sxw > syw ? sxw : syw;
                auto row_trip = [&](int base) {
                    const int w0 = base + tid, w1 = w0 + threads;
                    const uint64_t x0 = gb[min(w0, sxw - 1)], x1 = gb[min(w1, sxw - 1)];
                    const uint64_t y0 = gy[min(w0, syw - 1)], y1 = gy[min(w1, syw - 1)];
                    if (w0 < sxw) { ax[w0] = x0; axm[w0] = __brevll(x0) >> (64 - X); }
                    if (w1 < sxw) { ax[w1] = x1; axm[w1] = __brevll(x1) >> (64 - X); }
                    if (w0 < syw) { ay[w0] = y0; aym[w0] = __brevll(y0) >> (64 - Y); }
                    if (w1 < syw) { ay[w1] = y1; aym[w1] = __brevll(y1) >> (64 - Y); }
                };
                row_trip(0);                    // outside the loop: its loads join the three above
                for (int base = 2 * threads; base < longest; base += 2 * threads) row_trip(base);
            }
        } else {
            // x rows of the staged layers (all of them for the per-cell tracer), then y rows: word w is staged by thread
            // w modulo the workgroup size; four loads in flight per thread
            auto copy = [&](uint64_t* dst, const uint64_t* src, int n) {
                for (int base = tid; base < n; base += 4 * threads) {
                    uint64_t v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = src[min(base + u * threads, n - 1)];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (base + u * threads < n) dst[base + u * threads] = v[u];
                }
            };
            if (stage_rows || !scans) copy(lds_rows, gb, sxw);
            if (stage_rows) copy(lds_rows + sxw, gb + g.xrow_words, syw);
        }
        if (tid < p.W) lds_sx[tid] = first_sx;
        // image row records (see RowRecord); the z constants are those of the two vertical scan directions
        auto row_record = [&](float sy) {
            RowRecord rr;
            rr.sy = sy;
            const float dz = fmaf(sy, Uz, fmaf(first_sx, Rz, Fz));      // R_z = 0: the same for every column
            const bool zneg = (dz + 0.0f) < 0.0f;
            rr.rcp_z = safe_rcp(dz + 0.0f);
            const float dt_z = fabsf(rr.rcp_z);
            // (a rising ray of a camera above the solids leaves the cut grid at its first z plane: any positive
            // distance will do, the top of its real cell is one)
            const float dist_z = fabsf((float)(zneg ? kc : k0 + 1) - P[2]);
            const float nz_max = (float)(zneg ? kc : zlim - 1 - kc);
            rr.t0_z = !FAST && dz == 0.0f ? kNever : dist_z * dt_z;     // (see trace_windows)
            rr.tend_z = fmaf(nz_max, dt_z, rr.t0_z);
            return rr;
        };
        if (tid < p.H) lds_rowrec[tid] = row_record(first_sy);
        if (tid < lut_n) ll[tid] = first_lut;
        for (int i = tid + threads; i < p.W; i += threads) lds_sx[i] = p.sx[i];
        for (int i = tid + threads; i < p.H; i += threads) lds_rowrec[i] = row_record(p.sy[i]);
        for (int i = tid + threads; i < lut_n; i += threads) ll[i] = gl[i];
    }
    // This workgroup's copy of the rows is private to one camera: the camera's own body is removed from it
    // once, instead of being tested for at every step.  The thread that staged a word (word index modulo the
    // workgroup size) clears the body's bit in it straight after its own stores (one wave's LDS operations
    // keep their order), so the barrier below is the only one the staging needs.
    if (self_lo >= 0 && self_lo < X * Y * Z) {
        const int k = (int)p.by_plane.quotient((uint32_t)self_lo), rem = self_lo - k * X * Y;
        const int j = (int)p.by_x.quotient((uint32_t)rem), i = rem - j * X;
        auto staged_by_me = [&](int w) { return (int)threadIdx.x == w - (int)p.by_threads.quotient((uint32_t)w) * threads; };
#pragma unroll
        for (int up = 0; up < 2; ++up) {            // the voxel itself and the one above it
            const int kb = k + up;
            if (kb >= Z) continue;
            if (FAST) {
                if (stage_rows && kb < staged) {
                    uint64_t* ax = lds_rows;
                    uint64_t* axm = ax + sxw;
                    uint64_t* ay = axm + sxw;
                    uint64_t* aym = ay + syw;
                    if (staged_by_me(kb * Y + j)) {
                        ax[kb * Y + j] &= ~(1ull << i);
                        axm[kb * Y + j] &= ~(1ull << (X - 1 - i));
                    }
                    if (staged_by_me(kb * X + i)) {
                        ay[kb * X + i] &= ~(1ull << j);
                        aym[kb * X + i] &= ~(1ull << (Y - 1 - j));
                    }
                }
            } else if (kb < staged && (stage_rows || !scans)) {
                const int w = (kb * Y + j) * wx + (i >> 6);
                if (staged_by_me(w)) lds_rows[w] &= ~(1ull << (i & 63));
                const int wv = (kb * X + i) * wy + (j >> 6);
                if (stage_rows && staged_by_me(wv)) lds_rows[sxw + wv] &= ~(1ull << (j & 63));
            }
        }
    }
    // pair arrays (coarse level): [x pairs][x pairs mirrored][y pairs][y pairs mirrored] behind the row arrays
    const int vpx = (Y + 1) / 2, vpy = (X + 1) / 2;         // pairs per layer of the x / y arrays
    const int pxw = staged * vpx, pyw = staged * vpy;
    const uint32_t off_pairs = off_rows + 16u * (uint32_t)(sxw + syw);
    if (stage_rows && threadIdx.x >= 64 && threadIdx.x < 64 + kScanClasses) {
        const int q = threadIdx.x - 64;
        const bool xmaj = q < 8, neg = q & 4, vneg = q & 2, zneg = q & 1;
        const int U = xmaj ? X : Y, V = xmaj ? Y : X;
        const float pu = xmaj ? P[0] : P[1], pv = xmaj ? P[1] : P[0];
        ScanClass c;
        c.Pu = neg ? (float)U - pu : pu;
        c.Pu_err = 0.0f;
        c.pad = neg ? -1 : 0;
        if (neg) {                                         // exact error of the rounded difference (two-sum)
            const float a = (float)U, bneg = -pu;
            const float bb = __fsub_rn(c.Pu, a);
            c.Pu_err = __fadd_rn(__fsub_rn(a, __fsub_rn(c.Pu, bb)), __fsub_rn(bneg, bb));
        }
        c.uexit = (float)U - c.Pu;
        c.i0 = min(max((int)floorf(c.Pu), 0), U - 1);
        // A camera exactly on a u plane belongs to the cell on the + side (cell = floor(P)).  In mirrored
        // coordinates that cell is the one before floor(Pu): start the scan there, so that the neighbour
        // on the - side is found as an ordinary hit along the row (through its u face, at t = 0).
        if (neg && c.Pu == floorf(c.Pu) && c.i0 >= 1 && c.Pu < (float)U) c.i0 -= 1;
        if (!FAST) {
            // the window scan counts u crossings from the camera's cell: the cell itself (found in unmirrored coordinates,
            // where nothing is rounded) and the distance to its first u plane
            const int cell = min(max((int)floorf(pu), 0), U - 1);
            c.i0 = neg ? U - 1 - cell : cell;
            c.uexit = fabsf((float)(neg ? cell : cell + 1) - pu);
        }
        const int j0 = min(max((int)floorf(pv), 0), V - 1);
        // first plane along v: the upper plane of the camera's cell for rising v, the lower one otherwise
        c.dist_v = fabsf((float)(vneg ? j0 : j0 + 1) - pv);
        c.nv_max = (float)(vneg ? j0 : V - 1 - j0);
        const uint32_t array_off = off_rows + 8u * (uint32_t)(FAST ? (xmaj ? (neg ? sxw : 0) : 2 * sxw + (neg ? syw : 0))
                                                                   : (xmaj ? 0 : sxw));
        const int row_bytes = 8 * (xmaj ? wx : wy);
        // (for cameras outside: of cell (0,0,0), each ray adds its own entry cell)
        const int j_row = outside_rows ? 0 : j0, k_row = outside_rows ? 0 : kc;
        c.addr0 = (int)(lds_base + array_off) + row_bytes * (k_row * V + j_row);
        c.sv = vneg ? -row_bytes : row_bytes;
        c.sz = zneg ? -row_bytes * V : row_bytes * V;
        c.row_step_z = copysignf(tiny_int((uint32_t)(row_bytes * V)), zneg ? -1.0f : 1.0f);
        c.row_step_vz = copysignf(tiny_int((uint32_t)row_bytes), vneg ? -1.0f : 1.0f) - c.row_step_z;
        c.um1 = U - 1;
        c.face_u = faces.of(2 * (xmaj ? 0 : 1) + (neg ? 1 : 0));
        c.face_v = faces.of(2 * (xmaj ? 1 : 0) + (vneg ? 1 : 0));
        c.face_z = faces.of(zneg ? 5 : 4);
        const int su = xmaj ? 1 : X;                       // voxel-index step per original u cell
        const int sv_idx = xmaj ? X : 1;                   // and per v cell
        c.stride_u = (float)(neg ? -su : su);
        c.stride_v = (float)(vneg ? -sv_idx : sv_idx);
        c.stride_z = (float)(zneg ? -X * Y : X * Y);
        c.idx0 = (float)(k_row * X * Y + j_row * sv_idx + (neg ? (U - 1) * su : 0));
        *reinterpret_cast<ScanClass*>(lds + off_classes + q * kClassStride) = c;
        if (COARSE) {
            const int VP = xmaj ? vpx : vpy;
            PairClass pc;
            const uint32_t pair_off = off_pairs + 8u * (uint32_t)(xmaj ? (neg ? pxw : 0) : 2 * pxw + (neg ? pyw : 0));
            pc.addr0 = (int)(lds_base + pair_off + 8u * (uint32_t)(kc * VP + (j0 >> 1)));
            pc.sv = vneg ? -8 : 8;
            pc.sz = zneg ? -8 * VP : 8 * VP;
            // rising v: the plane above cell j0 lies inside its pair if j0 is even; falling v: the plane below it if j0 is odd
            pc.inner0 = ((j0 & 1) == (vneg ? 1 : 0)) ? 1 : 0;
            *reinterpret_cast<PairClass*>(lds + off_classes + q * kClassStride + sizeof(ScanClass)) = pc;
        }
    }
    if (FAST && outside_rows) {
        // what cameras outside know of the box (see EntryClass), by the threads that wrote the records
        for (int i = threadIdx.x; i < p.H; i += threads) {
            RowRecord& rr = lds_rowrec[i];
            const float dt_z = fabsf(rr.rcp_z);
            const bool zneg = rr.rcp_z < 0.0f;
            rr.t0_z = (zneg ? P[2] - (float)solid_layers : 0.0f - P[2]) * dt_z;
            rr.tend_z = ((zneg ? P[2] : (float)solid_layers - P[2]) + kTinyDistance) * dt_z;
        }
        if (threadIdx.x >= 64 && threadIdx.x < 64 + kScanClasses) {
            const int q = threadIdx.x - 64;
            const bool xmaj = q < 8, neg = q & 4, vneg = q & 2, zneg = q & 1;
            const float U = (float)(xmaj ? X : Y), V = (float)(xmaj ? Y : X), pu = xmaj ? P[0] : P[1], pv = xmaj ? P[1] : P[0];
            ScanClass& c = *reinterpret_cast<ScanClass*>(lds + off_classes + q * kClassStride);
            c.dist_v = vneg ? pv - V : 0.0f - pv;
            c.nv_max = (vneg ? pv : V - pv) + kTinyDistance;
            c.i0 = __float_as_int(pv);
            c.pad = __float_as_int(V - 1.0f);
            EntryClass e;
            e.near_u = neg ? pu - U : 0.0f - pu;
            e.far_u = (neg ? pu : U - pu) + kTinyDistance;
            e.ahead_v = vneg ? 0.0f : 1.0f;
            e.ahead_z = zneg ? 0.0f : 1.0f;
            e.per_cell_v = vneg ? 1.0f : -1.0f;
            e.per_cell_z = zneg ? 1.0f : -1.0f;
            e.planes_v = vneg ? 0.0f : V - 1.0f;
            e.planes_z = zneg ? 0.0f : (float)(solid_layers - 1);
            *reinterpret_cast<EntryClass*>(lds + off_classes + q * kClassStride + sizeof(ScanClass)) = e;
        }
    }
    __syncthreads();

    if (COARSE && use_rows) {
        const uint64_t* ax = lds_rows;
        const uint64_t* axm = ax + sxw;
        const uint64_t* ay = axm + sxw;
        const uint64_t* aym = ay + syw;
        uint64_t* px = reinterpret_cast<uint64_t*>(lds + off_pairs);
        uint64_t* pxm = px + pxw;
        uint64_t* py = pxm + pxw;
        uint64_t* pym = py + pyw;
        for (int w = threadIdx.x; w < pxw; w += threads) {
            const int k = w / vpx, J = w - k * vpx, a = k * Y + 2 * J;
            const bool two = 2 * J + 1 < Y;
            px[w] = ax[a] | (two ? ax[a + 1] : 0ull);
            pxm[w] = axm[a] | (two ? axm[a + 1] : 0ull);
        }
        for (int w = threadIdx.x; w < pyw; w += threads) {
            const int k = w / vpy, J = w - k * vpy, a = k * X + 2 * J;
            const bool two = 2 * J + 1 < X;
            py[w] = ay[a] | (two ? ay[a + 1] : 0ull);
            pym[w] = aym[a] | (two ? aym[a + 1] : 0ull);
        }
        __syncthreads();
    }

    // A camera inside a solid voxel (its own body is already gone) sees that voxel everywhere, at depth 0
    // with the "inside" face: one test per workgroup instead of one per ray.
    int cam_idx = -1;
    if (use_rows) {
        const int ic = min(max((int)floorf(P[0]), 0), X - 1), jc = min(max((int)floorf(P[1]), 0), Y - 1);
        const uint32_t bit = (uint32_t)(lds_rows[(kc * Y + jc) * wx + (FAST ? 0 : ic >> 6)] >> (ic & 63)) & 1u;
        if (__builtin_amdgcn_readfirstlane((int)bit)) cam_idx = (kc * Y + jc) * X + ic;
    }

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = threads >> 6;
    const int lane = threadIdx.x & 63;
    const int lx = lane % kTileW, ly = lane / kTileW, quad = lane & 3;
    const int lane_pix = ly * p.W + lx;
    const float* sx_lane = lds_sx + lx;
    const RowRecord* rowrec_lane = lds_rowrec + ly;
    const int tile_begin = part * tiles_per_block;
    const int tile_end = min(tile_begin + tiles_per_block, p.tiles_per_obs);
    // per-observation bases: everything inside one observation is addressed with 32-bit offsets
    const size_t obs_pix = (size_t)obs * p.H * p.W;
    float* __restrict__ depth_obs = p.depth + obs_pix;
    uint8_t* __restrict__ rgb_obs = p.rgb + obs_pix * 3;
    uint8_t* __restrict__ auxm_obs = AUX && p.aux_material ? p.aux_material + obs_pix : nullptr;
    int32_t* __restrict__ auxh_obs = AUX && p.aux_hit ? p.aux_hit + obs_pix : nullptr;
    uint8_t* __restrict__ auxf_obs = AUX && p.aux_face ? p.aux_face + obs_pix : nullptr;
    const uint8_t* __restrict__ vox_env = p.vox + (size_t)env * p.voxels_per_env;
    const uint32_t last_voxel = (uint32_t)p.voxels_per_env - 1u;
    const int last_material = p.materials_plus_one - 1;

    // a6 + a7 of a finished tile: material -> colour, then the stores.
    // Branch-free: lanes that found nothing look up a valid entry as well and then take the miss values.
    // `pix` is the wave-uniform pixel offset of the tile: the addresses of the stores are scalar, with a per-lane constant.
    // The store instructions are written out: the compiler adds the tile's offset per lane, in 64 bits.  Tiles that reach
    // beyond the image (PACKED launches have none) store what they have of it, colours byte by byte (256 x 4 cameras of 130x70
    // pixels: step 55.3 us when all tiles of such images did, 53.5 now).
    const uint32_t lane_depth_off = 4u * (uint32_t)lane_pix, lane_rgb_off = 3u * (uint32_t)lane_pix + (uint32_t)quad;
    // constants in vector registers (see tiny_int) where there are registers left for them (with the code of the tiles that
    // reach beyond the image they cost small images 1 % and gain large ones nothing)
    constexpr bool kVectors = FAST && PACKED && !AUX;
    const uint64_t three_of_four = 0x7777777777777777ull;
    // four consecutive lanes hold four consecutive pixels of one row = 12 bytes = three dwords, written by the first
    // three lanes of the quad: dword m holds the upper 3-m bytes of pixel m and the lower m+1 bytes of pixel m+1, one byte
    // permutation of the two (byte selectors 0..2: own pixel, 4..6: the next one)
    const uint32_t word_bytes = quad == 0 ? 0x04020100u : (quad == 1 ? 0x05040201u : 0x06050402u);
    const uint32_t sky = kVectors ? __float_as_uint(in_vector(__uint_as_float(p.sky_packed))) : p.sky_packed;
    auto shade_and_store = [&](int idx, int face, float t, uint32_t material, uint32_t pix, int columns_left, int rows_left) {
        const bool hit = idx >= 0;
        asm volatile("" : "+v"(material));          // (a whole register, not its low byte: no sub-dword operand below)
        material = min(material, (uint32_t)last_material);
        uint32_t shaded;
        if (AUX) {
            const float row = fmaf(tiny_int((uint32_t)face), (float)(4 * p.materials_plus_one), tiny_int(lds_base + off_lut));
            shaded = *(lds_u32_ptr)(uintptr_t)__float_as_uint(fmaf(tiny_int(material), 4.0f, row));
        } else shaded = *(lds_u32_ptr)(uintptr_t)__float_as_uint(fmaf(tiny_int(material), 4.0f, tiny_int((uint32_t)face)));
        asm volatile("" : "+v"(shaded));            // (read for every lane: a select costs less than a branch around the read)
        const uint32_t colour = hit ? shaded : sky;
        const float depth = hit ? t : 0.0f;
        if (PACKED || __builtin_expect(columns_left >= kTileW && rows_left >= kTileH, 1)) {
            store_dword(lane_depth_off, __float_as_uint(depth), reinterpret_cast<const uint8_t*>(depth_obs) + 4u * pix);
            if (AUX && auxm_obs) store_byte((uint32_t)lane_pix, hit ? material : 0u, auxm_obs + pix);
            if (AUX && auxh_obs) store_dword(lane_depth_off, (uint32_t)max(idx, -1), reinterpret_cast<const uint8_t*>(auxh_obs) + 4u * pix);
            if (AUX && auxf_obs) store_byte((uint32_t)lane_pix, (uint32_t)(hit ? face : 255), auxf_obs + pix);
            const uint32_t word = __builtin_amdgcn_perm(next_in_quad(colour), colour, word_bytes);
            // (all lanes of a wave are in the tile loop: the mask is set and reset without being read)
            asm volatile("s_mov_b64 exec, %0\n\tglobal_store_dword %1, %2, %3\n\ts_mov_b64 exec, -1"
                         :: "s"(three_of_four), "v"(lane_rgb_off), "v"(word), "s"(rgb_obs + 3u * pix) : "memory");
        } else {
            // (the lane's column and row are worked out again here: kept through the tile loop they cost it registers)
            const int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), row = l / kTileW, column = l % kTileW;
            if (column >= columns_left || row >= rows_left) return;
            const int lane_pix = row * p.W + column;
            const uint32_t lane_depth_off = 4u * (uint32_t)lane_pix;
            store_dword(lane_depth_off, __float_as_uint(depth), reinterpret_cast<const uint8_t*>(depth_obs) + 4u * pix);
            if (AUX && auxm_obs) store_byte((uint32_t)lane_pix, hit ? material : 0u, auxm_obs + pix);
            if (AUX && auxh_obs) store_dword(lane_depth_off, (uint32_t)max(idx, -1), reinterpret_cast<const uint8_t*>(auxh_obs) + 4u * pix);
            if (AUX && auxf_obs) store_byte((uint32_t)lane_pix, (uint32_t)(hit ? face : 255), auxf_obs + pix);
            uint8_t* out = rgb_obs + 3u * pix + 3u * (uint32_t)lane_pix;
            out[0] = (uint8_t)colour;
            out[1] = (uint8_t)(colour >> 8);
            out[2] = (uint8_t)(colour >> 16);
        }
    };

    // The tile loop is software-pipelined by one tile: a trip first requests the material bytes of the tile
    // traced in the previous trip, then traces its own tile, and only then shades and stores the previous
    // one, so that the global fetch hides behind a whole traversal.  (The request is issued in the trip that
    // consumes it: a value still in flight across the loop's back edge would be waited for there.)
    // The loop exists once for each of: the row scan alone (the common case), the row scan of cameras outside, the other
    // tracers, so that the values only one of them needs are not kept in registers through the others' loops.
    auto run_tiles = [&](auto rows_only_tag, auto narrow_tag, auto outside_tag) {
        constexpr bool kRowsOnly = decltype(rows_only_tag)::value;
        constexpr bool kOutside = decltype(outside_tag)::value;
        // What only the rarer loops need of the camera is read again for them (through a pointer the compiler cannot
        // match with the first read): kept in scalar registers from the prologue on, it costs the common loop spills.
        float Pc[3] = { 0.0f, 0.0f, 0.0f }, Fcz = 0.0f, Ucz = 0.0f;
        int body_lo = -1, body_hi = -1, top = 0;
        bool inside = true, finite = true;
        if constexpr (!scans) {
            // (one tile loop: nothing to keep out of another's registers)
            Pc[0] = P[0]; Pc[1] = P[1]; Pc[2] = P[2];
            Fcz = Fz; Ucz = Uz;
            inside = origin_in_grid;
        } else if constexpr (!kRowsOnly || kOutside) {
            const CameraRecord* again = p.rec + obs;
            const int32_t* tops = p.ztop;
            asm volatile("" : "+s"(again), "+s"(tops));
            Pc[0] = uniform(again->P[0]); Pc[1] = uniform(again->P[1]); Pc[2] = uniform(again->P[2]);
            Fcz = uniform(again->F[2]); Ucz = uniform(again->U[2]);         // R_z = 0: no roll
            body_lo = __builtin_amdgcn_readfirstlane(again->self_lo); body_hi = __builtin_amdgcn_readfirstlane(again->self_hi);
            top = __builtin_amdgcn_readfirstlane(tops[env]);
            inside = __builtin_amdgcn_readfirstlane(again->place) == kPlaceInGrid;
            float sum = 0.0f;           // (R_z is 0)
            for (int a = 0; a < 3; ++a) sum += fabsf(again->F[a]) + fabsf(again->R[a]) + fabsf(again->U[a]);
            finite = __builtin_amdgcn_readfirstlane(sum < kBig) != 0;
        }
        constexpr bool kNarrow = decltype(narrow_tag)::value;
        // (window scan) how far from the middle of a cell a position may be to tell the cell: see trace_windows
        const float edge = uniform(0.5f - 0x1p-20f * ((float)max(X, Y) + (kOutside ? fmaxf(fabsf(Pc[0]), fabsf(Pc[1])) : 0.0f)));
        int pend_idx = -1, pend_face = faces.base;
        float pend_t = 0.0f;
        uint32_t pend_pix = 0;
        int pend_columns = 0, pend_rows = 0;
        bool pending = false;
        // (in vector registers: see tiny_int)
        const float vFx = kVectors ? in_vector(Fx) : Fx, vFy = kVectors ? in_vector(Fy) : Fy, vRx = kVectors ? in_vector(Rx) : Rx, vRy = kVectors ? in_vector(Ry) : Ry,
                    vUx = kVectors ? in_vector(Ux) : Ux, vUy = kVectors ? in_vector(Uy) : Uy;
        // tile coordinates are carried along instead of divided out of the tile index every trip
        int ty = (int)p.by_tiles_x.quotient((uint32_t)(tile_begin + wave)), tx = (tile_begin + wave) - ty * p.tiles_x - waves;
        uint32_t tile_pix = (uint32_t)(ty * kTileH * p.W + tx * kTileW);
        const uint32_t pix_step = (uint32_t)(waves * kTileW), pix_wrap = (uint32_t)(kTileH * p.W - p.tiles_x * kTileW);
        for (int tile = tile_begin + wave; tile < tile_end; tile += waves) {
            // lanes without a hit (idx -1 = 0xffffffff) read the last voxel and drop it later: no branch
            const uint32_t pend_material = vox_env[min((uint32_t)pend_idx, last_voxel)];

            tx += waves;
            tile_pix += pix_step;
            while (tx >= p.tiles_x) { tx -= p.tiles_x; ++ty; tile_pix += pix_wrap; }
            float sx;
            RowRecord rr;
            if constexpr (PACKED) {
                sx = sx_lane[tx * kTileW];
                rr = rowrec_lane[ty * kTileH];
            } else {
                // (columns and rows of the last tiles that the image does not have repeat its last ones)
                const uint32_t first_sx = lds_base + off_scalars, first_row = lds_base + off_rowrec;
                const uint32_t at_sx = min(first_sx + 4u * (uint32_t)(tx * kTileW + lx), first_sx + 4u * (uint32_t)(p.W - 1));
                const uint32_t at_row = min(first_row + 16u * (uint32_t)(ty * kTileH + ly), first_row + 16u * (uint32_t)(p.H - 1));
                sx = *(lds_f32_ptr)(uintptr_t)at_sx;
                *reinterpret_cast<u32x4*>(&rr) = *(lds_u32x4_ptr)(uintptr_t)at_row;
            }

            // a4: ray through the pixel centre, two fused multiply-adds per axis (the row scan takes what it needs of
            // the vertical component from the row record)
            float d[3];
            d[0] = fmaf(rr.sy, vUx, fmaf(sx, vRx, vFx));
            d[1] = fmaf(rr.sy, vUy, fmaf(sx, vRy, vFy));
            if (!kRowsOnly || kOutside) d[2] = fmaf(rr.sy, Ucz, Fcz);

            // a5: traversal
            Hit h;
            if constexpr (kOutside) {
                const OutsideCamera from{ faces, finite, { Pc[0], Pc[1], Pc[2] }, d[2], X, Y, max(top, 1) };
                if constexpr (FAST) h = trace_rows<kNarrow, false, true>(lds_base + off_classes, d[0], d[1], rr, -1, &from);
                else h = trace_windows<true>(lds_base + off_classes, d[0], d[1], rr, edge, &from);
            } else if constexpr (kRowsOnly) {
                if constexpr (FAST) h = trace_rows<kNarrow, COARSE>(lds_base + off_classes, d[0], d[1], rr, p.coarse_after);
                else h = trace_windows<false>(lds_base + off_classes, d[0], d[1], rr, edge);
            } else if (use_rows) {
                h.idx = cam_idx; h.face = faces.of(6); h.t = 0.0f;
            } else if (scans) {
                // cameras far outside the grid, and worlds taller than the staged layers: the x rows in global
                // memory, own body skipped by index
                h = trace_generic(reinterpret_cast<const uint32_t*>(p.bits + (size_t)env * g.env_words), 2 * g.rowwords_x,
                                  Pc, d, X, Y, Z, inside, p.max_steps, body_lo, body_hi);
                h.face = faces.of(min(h.face, kNumFaces - 1));
            } else {
                h = trace_generic(reinterpret_cast<const uint32_t*>(lds_rows), 2 * g.rowwords_x, Pc, d, X, Y, Z,
                                  inside, p.max_steps, -1, -1);
                h.face = faces.of(min(h.face, kNumFaces - 1));
            }

            if (pending) shade_and_store(pend_idx, pend_face, pend_t, pend_material, pend_pix, pend_columns, pend_rows);
            pend_idx = h.idx; pend_face = h.face; pend_t = h.t;
            pend_pix = tile_pix;
            pend_columns = p.W - tx * kTileW; pend_rows = p.H - ty * kTileH;
            pending = true;
        }
        if (pending) {
            const uint32_t pend_material = vox_env[min((uint32_t)pend_idx, last_voxel)];
            shade_and_store(pend_idx, pend_face, pend_t, pend_material, pend_pix, pend_columns, pend_rows);
        }
    };
    __builtin_amdgcn_s_setprio(0);
    if (scans && use_rows && cam_idx < 0) {
        if (FAST && X < 64 && Y < 64) run_tiles(std::true_type{}, std::true_type{}, std::false_type{});
        else run_tiles(std::true_type{}, std::false_type{}, std::false_type{});
    } else if (scans && !use_rows && stage_rows) {
        run_tiles(std::true_type{}, std::false_type{}, std::true_type{});
    } else {
        run_tiles(std::false_type{}, std::false_type{}, std::false_type{});
    }

    // The indicator bar over the colours: each wave paints the bar's pixels in the tiles that it has rendered itself, behind
    // its own stores and without waiting for them (a wave's stores to one address keep their order).  Steps with bars of 9x3, us,
    // with a launch of its own -> so, in turn on one machine: 1024 x 4 cameras of 128x72 with edits 136.4 -> 135.0, 256 x 4 47.8 ->
    // 46.1, 64 x 2 20.9 -> 19.0.  The look for a bar costs launches without one nothing that stands out from the differences
    // between two builds: without this block 48.3 / 48.5 (256 x 4), 298.9 / 300.0 (4096 x 2), 51.3 / 51.2 (130x70 pixels), 47.0 /
    // 47.3 (no batch object), 62.6 / 63.2 (cameras outside), where builds that differ elsewhere only read 48.0 to 49.0 for the first.
    // (The bar is read here, through a pointer that the compiler cannot match with the argument: held in scalar registers through
    // the tile loop it costs spills.)
    typedef __attribute__((address_space(4))) const RenderParams* params_ptr;
    params_ptr again = (params_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(again));
    if (!AUX && again->bar_fraction) {
        const BarParams bar{ again->bar.x, again->bar.y, again->bar.width, again->bar.height, again->bar.fill_packed, again->bar.empty_packed };
        const float* fractions = again->bar_fraction;
        const int filled = bar_columns(fractions[obs], bar.width);
        const int first_row = max(bar.y, (int)p.by_tiles_x.quotient((uint32_t)tile_begin) * kTileH);
        const int end_row = min(bar.y + bar.height, ((int)p.by_tiles_x.quotient((uint32_t)(tile_end - 1)) + 1) * kTileH);
        const int pixels = max(end_row - first_row, 0) * bar.width;
        for (int i = (int)__lane_id(); i < pixels; i += 64) {
            const int r = i / bar.width, c = i - r * bar.width;
            const int y = first_row + r, x = bar.x + c;
            const int tile = (y / kTileH) * p.tiles_x + x / kTileW - tile_begin;
            if (tile < 0 || tile >= tile_end - tile_begin || tile % waves != wave) continue;
            const uint32_t colour = c < filled ? bar.fill_packed : bar.empty_packed;
            uint8_t* out = rgb_obs + 3u * (uint32_t)(y * p.W + x);
            out[0] = (uint8_t)colour;
            out[1] = (uint8_t)(colour >> 8);
            out[2] = (uint8_t)(colour >> 16);
        }
    }
}

// ------------------------------------------------------------------------------------------
// bars: one workgroup per observation paints the indicator bar over the rendered colours (small bars of mv_step: render_kernel).
// ------------------------------------------------------------------------------------------
__global__ void bars_kernel(uint8_t* __restrict__ rgb, const float* __restrict__ fraction,
                            const uint8_t* __restrict__ active, int A, int W, int H, BarParams bar)
{
    const int obs = blockIdx.x;
    if (active && active[obs / A] == 0) return;
    const int filled = bar_columns(fraction[obs], bar.width);
    uint8_t* img = rgb + (size_t)obs * H * W * 3;
    for (int p = threadIdx.x; p < bar.width * bar.height; p += blockDim.x) {
        const int r = p / bar.width, c = p - r * bar.width;
        const uint32_t colour = c < filled ? bar.fill_packed : bar.empty_packed;
        uint8_t* out = img + ((size_t)(bar.y + r) * W + (bar.x + c)) * 3;
        out[0] = (uint8_t)colour;
        out[1] = (uint8_t)(colour >> 8);
        out[2] = (uint8_t)(colour >> 16);
    }
}

hipError_t launch_bars(uint8_t* rgb, const float* fraction, const uint8_t* active, int num_obs, int A, int W, int H,
                       const BarParams& bar, hipStream_t stream)
{
    hipLaunchKernelGGL(bars_kernel, dim3(num_obs), dim3(128), 0, stream, rgb, fraction, active, A, W, H, bar);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// overlay: one workgroup per observation paints the primitives over the rendered colours, one after the
// other; the barrier between two primitives (it also waits for the workgroup's stores) keeps the list order
// where they overlap.
// ------------------------------------------------------------------------------------------
__global__ void overlay_kernel(uint8_t* __restrict__ rgb, const float* __restrict__ values, int values_per_obs,
                               const uint8_t* __restrict__ active, int A, int W, int H, OverlayParams overlay)
{
    const int obs = blockIdx.x;
    if (active && active[obs / A] == 0) return;
    uint8_t* img = rgb + (size_t)obs * H * W * 3;
    for (int k = 0; k < overlay.count; ++k) {
        const OverlayRect& q = overlay.rect[k];
        int filled = 0;
        if (q.kind != 0) {
            // filled columns or rows: one float32 multiply, one float32 add, floor, clamp (NaN falls to 0)
            const int extent = q.kind == 1 ? q.width : q.height;
            float n = floorf(__fadd_rn(__fmul_rn(values[(size_t)obs * values_per_obs + q.value_index], (float)extent), 0.5f));
            n = fminf(fmaxf(n, 0.0f), (float)extent);
            filled = (int)n;
        }
        for (int i = threadIdx.x; i < q.width * q.height; i += blockDim.x) {
            const int r = i / q.width, c = i - r * q.width;
            const bool front = q.kind == 0 || (q.kind == 1 ? c < filled : q.height - 1 - r < filled);
            const uint32_t colour = front ? q.front_packed : q.rest_packed;
            uint8_t* out = img + ((size_t)(q.y + r) * W + (q.x + c)) * 3;
            out[0] = (uint8_t)colour;
            out[1] = (uint8_t)(colour >> 8);
            out[2] = (uint8_t)(colour >> 16);
        }
        if (k + 1 < overlay.count) __syncthreads();
    }
}

hipError_t launch_overlay(uint8_t* rgb, const float* values, int values_per_obs, const uint8_t* active, int num_obs, int A,
                          int W, int H, const OverlayParams& overlay, hipStream_t stream)
{
    hipLaunchKernelGGL(overlay_kernel, dim3(num_obs), dim3(256), 0, stream, rgb, values, values_per_obs, active, A, W, H,
                       overlay);
    return hipGetLastError();
}

template <bool AUX, bool PACKED, Scan SCAN, bool COARSE = false>
static hipError_t set_lds_limit()
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&render_kernel<AUX, PACKED, SCAN, COARSE>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBudget);
}

// Workgroups of the render and pack kernels may ask for more dynamic LDS than the default limit: raise the limit
// of every instantiation to the whole LDS of a compute unit, once per device (the attribute belongs to the
// function on the current device, not to a batch: a value derived from one batch's plan would be wrong for
// the next batch).
hipError_t prepare_kernels()
{
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> done[kMaxDevices];
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    if (device >= 0 && device < kMaxDevices && done[device].load(std::memory_order_acquire)) return hipSuccess;
#define MV_SET(...)                                                          \
    if (e == hipSuccess) e = set_lds_limit<false, false, __VA_ARGS__>();     \
    if (e == hipSuccess) e = set_lds_limit<false, true, __VA_ARGS__>();      \
    if (e == hipSuccess) e = set_lds_limit<true, false, __VA_ARGS__>();      \
    if (e == hipSuccess) e = set_lds_limit<true, true, __VA_ARGS__>()
    MV_SET(Scan::kRows); MV_SET(Scan::kWindows); MV_SET(Scan::kCells); MV_SET(Scan::kRows, true);
#undef MV_SET
    // the pack kernel also has a few static words of LDS: its dynamic share must leave room for them
    const int pack_limit = (int)(kLdsBudget - kPackStaticLds);
    const void* pack_kernels[] = { reinterpret_cast<const void*>(&pack_kernel<u32x4, 2, false>), reinterpret_cast<const void*>(&pack_kernel<u32x4, 2, true>),
                                   reinterpret_cast<const void*>(&pack_kernel<u32x4, 4, false>), reinterpret_cast<const void*>(&pack_kernel<u32x4, 4, true>),
                                   reinterpret_cast<const void*>(&pack_kernel<uint32_t, 8, false>), reinterpret_cast<const void*>(&pack_kernel<uint32_t, 8, true>),
                                   reinterpret_cast<const void*>(&pack_any_kernel<false>), reinterpret_cast<const void*>(&pack_any_kernel<true>) };
    for (const void* k : pack_kernels)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, pack_limit);
    if (e == hipSuccess && device >= 0 && device < kMaxDevices) done[device].store(true, std::memory_order_release);
    return e;
}

hipError_t launch_render(const RenderParams& p, size_t lds_bytes, hipStream_t stream)
{
    const bool aux = p.aux_material || p.aux_hit || p.aux_face;
    // (images of whole 8x8 tiles whose colours start on a dword: no tile needs a second look, and no dword is split)
    const bool packed = (p.W % kTileW == 0) && (p.H % kTileH == 0) && ((reinterpret_cast<uintptr_t>(p.rgb) & 3) == 0);
    dim3 grid(p.blocks_per_xcd * kXcds), block(p.threads);
#define MV_LAUNCH(...)                                                                                                       \
    do {                                                                                                                     \
        if (aux) {                                                                                                           \
            if (packed) hipLaunchKernelGGL((render_kernel<true, true, __VA_ARGS__>), grid, block, lds_bytes, stream, p);       \
            else hipLaunchKernelGGL((render_kernel<true, false, __VA_ARGS__>), grid, block, lds_bytes, stream, p);             \
        } else {                                                                                                             \
            if (packed) hipLaunchKernelGGL((render_kernel<false, true, __VA_ARGS__>), grid, block, lds_bytes, stream, p);      \
            else hipLaunchKernelGGL((render_kernel<false, false, __VA_ARGS__>), grid, block, lds_bytes, stream, p);            \
        }                                                                                                                    \
    } while (0)
    if (p.g.fast && p.coarse_after >= 0) MV_LAUNCH(Scan::kRows, true);
    else if (p.g.fast) MV_LAUNCH(Scan::kRows);
    else if (p.window) MV_LAUNCH(Scan::kWindows);
    else MV_LAUNCH(Scan::kCells);
#undef MV_LAUNCH
    return hipGetLastError();
}

}  // namespace mv
