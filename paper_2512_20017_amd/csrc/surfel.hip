// 2D Gaussian surfels (the paper's 2DGS configuration: Sec. 5 "Applications"; Table 3b state of 20 floats; App. B
// "2DGS models [the projection] more accurately"): per-point projection and its derivative, raster record, and the
// per-tile compositing kernels with a ray-disk intersection per (pixel, splat) pair instead of a projected conic.
//
// A point is an oriented disk: centre, two raw tangent vectors made orthonormal by Gram-Schmidt, two scales, opacity,
// SH colour. ray_transform T = K [R s_u t_u | R s_v t_v | R mean + t] maps disk coordinates (u, v, 1) to homogeneous
// pixels. A pixel's ray meets the disk plane at (u, v) = (p_0, p_1) / p_2 with p = h_u x h_v, h_u = x T_2 - T_0,
// h_v = y T_2 - T_1 (rows of T); G = exp(-(u^2+v^2)/2), low-pass G^ = max(G, exp(-|pixel - mean2d|^2)),
// alpha = min(0.99, o G^); skip / stop / order rules as for 3D Gaussians.
//
// fp32 care: x T_2 - T_0 subtracts numbers of size (pixel x depth) to leave one of size (offset x depth). The raster
// record therefore stores rows centred on the projected centre, T_0' = T_0 - mx T_2 and T_1' = T_1 - my T_2 (one fused
// multiply-add each, so exactly rounded), and the kernels use h_u = dx T_2 - T_0' with dx = x - mx. The same value of
// mx is used on both sides, so this is the same number as x T_2 - T_0, without the cancellation.
#include "composite_common.h"
#include "pair_reduce.h"
#include "binning_common.h"
#include "sh_basis.h"

namespace pbdr {

// 64-byte raster record
struct __attribute__((aligned(16))) Packed2D {
    float t0x, t0y, t1x, t1y;      // centred rows T_0', T_1' (first two components)
    float t2x, t2y, t2z, o;        // T_2, opacity
    float mx, my, r, g;            // mean2d, red, green
    float b, radius_bits, t0z, t1z;  // blue, integer extent (bit-cast), third components of the centred rows (rounding residue)
};
static_assert(sizeof(Packed2D) == 64, "surfel raster record is 64 bytes");

struct Frame2D {
    float tu[3], tv[3], w[3], ainv, winv, btu, su, sv;
    float H[9];   // row-major; columns R s_u t_u, R s_v t_v, R mean + t
};

__device__ __forceinline__ void surfel_frame(const CamDev& cam, const float m[3], const float a[3], const float b[3],
                                             float ls0, float ls1, Frame2D& F)
{
    F.su = expf(ls0); F.sv = expf(ls1);
    F.ainv = 1.0f / sqrtf(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) F.tu[i] = a[i] * F.ainv;
    F.btu = b[0] * F.tu[0] + b[1] * F.tu[1] + b[2] * F.tu[2];
#pragma unroll
    for (int i = 0; i < 3; ++i) F.w[i] = b[i] - F.btu * F.tu[i];
    F.winv = 1.0f / sqrtf(F.w[0] * F.w[0] + F.w[1] * F.w[1] + F.w[2] * F.w[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) F.tv[i] = F.w[i] * F.winv;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        F.H[3 * i] = F.su * (cam.R[3 * i] * F.tu[0] + cam.R[3 * i + 1] * F.tu[1] + cam.R[3 * i + 2] * F.tu[2]);
        F.H[3 * i + 1] = F.sv * (cam.R[3 * i] * F.tv[0] + cam.R[3 * i + 1] * F.tv[1] + cam.R[3 * i + 2] * F.tv[2]);
        F.H[3 * i + 2] = cam.R[3 * i] * m[0] + cam.R[3 * i + 1] * m[1] + cam.R[3 * i + 2] * m[2] + cam.t[i];
    }
}

template <int kDeg>
__global__ __launch_bounds__(256) void k_preprocess2d(Scene2DDev sc, CamDev cam, Splats2DDev out)
{
    const int n = sc.n;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const size_t N = (size_t)n;
    const float m[3] = {sc.mean[i], sc.mean[N + i], sc.mean[2 * N + i]};
    const float pz = cam.R[6] * m[0] + cam.R[7] * m[1] + cam.R[8] * m[2] + cam.t[2];
    if (!(pz >= cam.near_p && pz <= cam.far_p)) { out.radius[i] = 0; return; }
    const float a[3] = {sc.tan_u[i], sc.tan_u[N + i], sc.tan_u[2 * N + i]};
    const float b[3] = {sc.tan_v[i], sc.tan_v[N + i], sc.tan_v[2 * N + i]};
    Frame2D F;
    surfel_frame(cam, m, a, b, sc.log_scale[i], sc.log_scale[N + i], F);
    float T[9];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T[k] = cam.fx * F.H[k] + cam.cx * F.H[6 + k];
        T[3 + k] = cam.fy * F.H[3 + k] + cam.cy * F.H[6 + k];
        T[6 + k] = F.H[6 + k];
    }
    const float aa = 9.f * (T[6] * T[6] + T[7] * T[7]) - T[8] * T[8];
    if (!(aa < 0.f)) { out.radius[i] = 0; return; }
    const float iz = 1.0f / T[8];
    // projected centre, formed from the camera-space columns so that cx, cy do not cancel
    const float mx = cam.fx * F.H[2] * iz + cam.cx, my = cam.fy * F.H[5] * iz + cam.cy;
    float reach = 0.f;
    {
        // Bounding box of the perspective image of the 3-sigma rim, in coordinates centred on the projected centre:
        // rows U_i = f_i (H_i - (H_i2 / H_22) H_2), whose third components vanish, so neither the principal point nor
        // the centre's own pixel coordinate enters (no cancellation of large numbers).
        const float ia = 1.0f / (9.f * (F.H[6] * F.H[6] + F.H[7] * F.H[7]) - F.H[8] * F.H[8]);
        const float f2[2] = {cam.fx, cam.fy};
#pragma unroll
        for (int ax = 0; ax < 2; ++ax) {
            const float* Hi = F.H + 3 * ax;
            const float sl = Hi[2] * iz;
            const float u0 = f2[ax] * (Hi[0] - sl * F.H[6]), u1 = f2[ax] * (Hi[1] - sl * F.H[7]);
            const float bb = 9.f * (u0 * F.H[6] + u1 * F.H[7]);
            const float cc = 9.f * (u0 * u0 + u1 * u1);
            const float c0 = bb * ia;
            const float half = sqrtf(fmaxf(1e-4f, c0 * c0 - cc * ia));
            reach = fmaxf(reach, fabsf(c0) + half);
        }
    }
    float ext = fmaxf(3.f, ceilf(reach));
    const int r = (ext < (float)kRadiusMax) ? (int)ext : kRadiusMax;
    if ((float)r <= cam.radius_clip) { out.radius[i] = 0; return; }
    {
        int x0, y0, x1, y1;
        tile_rect(cam, mx, my, r, x0, y0, x1, y1);
        if ((x1 - x0) * (y1 - y0) <= 0) { out.radius[i] = 0; return; }
    }
    const float vx = m[0] - cam.campos[0], vy = m[1] - cam.campos[1], vz = m[2] - cam.campos[2];
    const float vinv = 1.0f / sqrtf(vx * vx + vy * vy + vz * vz);
    float Y[16];
    sh_basis(kDeg, vx * vinv, vy * vinv, vz * vinv, Y);
    constexpr int K = (kDeg + 1) * (kDeg + 1);
    // all coefficients asked for before the first is used (written as one loop with the sums, every load was waited for
    // on its own: 48 round trips in a row per point)
    float coef[3 * K];
#pragma unroll
    for (int j = 0; j < 3 * K; ++j) coef[j] = __builtin_nontemporal_load(&sc.sh[(size_t)j * N + i]);
    const float lg = __builtin_nontemporal_load(&sc.logit[i]);
    float rgb[3] = {0.5f, 0.5f, 0.5f};
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int c = 0; c < 3; ++c) rgb[c] += Y[k] * coef[3 * k + c];
    }
    // normal = R (t_u x t_v), turned towards the camera
    float nw[3] = {F.tu[1] * F.tv[2] - F.tu[2] * F.tv[1], F.tu[2] * F.tv[0] - F.tu[0] * F.tv[2], F.tu[0] * F.tv[1] - F.tu[1] * F.tv[0]};
    float nc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) nc[k] = cam.R[3 * k] * nw[0] + cam.R[3 * k + 1] * nw[1] + cam.R[3 * k + 2] * nw[2];
    const float facing = nc[0] * F.H[2] + nc[1] * F.H[5] + nc[2] * F.H[8];
    const float sgn = facing > 0.f ? -1.f : 1.f;
    out.mean2d[i] = mx; out.mean2d[N + i] = my;
#pragma unroll
    for (int k = 0; k < 9; ++k) out.T[(size_t)k * N + i] = T[k];
    out.opacity[i] = 1.0f / (1.0f + expf(-lg));
#pragma unroll
    for (int c = 0; c < 3; ++c) { out.color[(size_t)c * N + i] = fmaxf(rgb[c], 0.f); out.normal[(size_t)c * N + i] = sgn * nc[c]; }
    out.radius[i] = r;
    out.depth[i] = T[8];
}

// kFirst, kFromRecords: see the 3D variant. With kFromRecords the splat-state gradient of a point is the 64-byte record
// the gather of the compositing backward left in the workspace (`rec`), and `radius` is the tiles-touched count.
template <int kDeg, bool kFirst, bool kFromRecords>
__global__ __launch_bounds__(256) void k_preprocess2d_bwd(Scene2DDev sc, CamDev cam, const int32_t* __restrict__ radius,
                                                          const float* __restrict__ Tst, Splat2DGradDev g2,
                                                          const float4* __restrict__ rec, CarryFold cf, Scene2DGradDev g)
{
    const int n = sc.n;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const size_t N = (size_t)n;
    if (radius[i] <= 0) {
        if (kFirst) {
            constexpr int K0 = (kDeg + 1) * (kDeg + 1);
            // zeros and SH / opacity reads: non-temporal, as in the 3D kernels (see preprocess.hip)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                __builtin_nontemporal_store(0.f, &g.mean[(size_t)k * N + i]);
                __builtin_nontemporal_store(0.f, &g.tan_u[(size_t)k * N + i]);
                __builtin_nontemporal_store(0.f, &g.tan_v[(size_t)k * N + i]);
            }
            __builtin_nontemporal_store(0.f, &g.log_scale[i]); __builtin_nontemporal_store(0.f, &g.log_scale[N + i]);
            __builtin_nontemporal_store(0.f, &g.logit[i]);
#pragma unroll
            for (int k = 0; k < 3 * K0; ++k) __builtin_nontemporal_store(0.f, &g.sh[(size_t)k * N + i]);
        }
        return;
    }
    // dL/d(splat state): T (nine), mean2d (two), opacity, colour (three), in the record's order
    float gs[15];
    if (kFromRecords) {
        const float4 ra = rec[(size_t)4 * i], rb = rec[(size_t)4 * i + 1], rc = rec[(size_t)4 * i + 2], rd = rec[(size_t)4 * i + 3];
        const float v[15] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w, rc.x, rc.y, rc.z, rc.w, rd.x, rd.y, rd.z};
#pragma unroll
        for (int k = 0; k < 15; ++k) gs[k] = v[k];
        // a point whose pairs are cut by a wavefront boundary of the gather: its record is still in pieces (this launch
        // puts it together, see pair_reduce.h)
        if (cf.carry != nullptr) (void)record_from_carries<15>(cf, cf.slot_base[i], (uint32_t)radius[i], gs);
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k) gs[k] = g2.T[(size_t)k * N + i];
        gs[9] = g2.mean2d[i]; gs[10] = g2.mean2d[N + i];
        gs[11] = g2.opacity[i];
        gs[12] = g2.color[i]; gs[13] = g2.color[N + i]; gs[14] = g2.color[2 * N + i];
    }
    const float m[3] = {sc.mean[i], sc.mean[N + i], sc.mean[2 * N + i]};
    const float a[3] = {sc.tan_u[i], sc.tan_u[N + i], sc.tan_u[2 * N + i]};
    const float b[3] = {sc.tan_v[i], sc.tan_v[N + i], sc.tan_v[2 * N + i]};
    Frame2D F;
    surfel_frame(cam, m, a, b, sc.log_scale[i], sc.log_scale[N + i], F);
    {
        const float o = 1.0f / (1.0f + expf(-__builtin_nontemporal_load(&sc.logit[i])));
        grad_out<kFirst>(&g.logit[i], gs[11] * o * (1.f - o));
    }
    float dmu[3] = {0.f, 0.f, 0.f};
    {
        const float vx = m[0] - cam.campos[0], vy = m[1] - cam.campos[1], vz = m[2] - cam.campos[2];
        const float vinv = 1.0f / sqrtf(vx * vx + vy * vy + vz * vz);
        const float dx = vx * vinv, dy = vy * vinv, dz = vz * vinv;
        float Y[16];
        float dY[16][3];
        sh_basis(kDeg, dx, dy, dz, Y);
        sh_basis_grad(kDeg, dx, dy, dz, dY);
        constexpr int K = (kDeg + 1) * (kDeg + 1);
        float gd0 = 0.f, gd1 = 0.f, gd2 = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float raw = 0.5f, t0 = 0.f, t1 = 0.f, t2 = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float co = __builtin_nontemporal_load(&sc.sh[(size_t)(3 * k + c) * N + i]);
                raw += Y[k] * co;
                t0 += dY[k][0] * co; t1 += dY[k][1] * co; t2 += dY[k][2] * co;
            }
            const float gc = raw > 0.f ? gs[12 + c] : 0.f;
            if (kFirst || gc != 0.f) {
#pragma unroll
                for (int k = 0; k < K; ++k) grad_out<kFirst>(&g.sh[(size_t)(3 * k + c) * N + i], Y[k] * gc);
            }
            gd0 += gc * t0; gd1 += gc * t1; gd2 += gc * t2;
        }
        const float dot = gd0 * dx + gd1 * dy + gd2 * dz;
        dmu[0] += (gd0 - dx * dot) * vinv; dmu[1] += (gd1 - dy * dot) * vinv; dmu[2] += (gd2 - dz * dot) * vinv;
    }
    // gradient w.r.t. the stored transform, plus mean2d_i = T_i2 / T_22
    float GT[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) GT[k] = gs[k];
    {
        const float T02 = Tst[2 * N + i], T12 = Tst[5 * N + i], T22 = Tst[8 * N + i];
        const float iz = 1.0f / T22, gmx = gs[9], gmy = gs[10];
        GT[2] += gmx * iz; GT[5] += gmy * iz;
        GT[8] -= (gmx * T02 + gmy * T12) * iz * iz;
    }
    float GH[9];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        GH[k] = cam.fx * GT[k];
        GH[3 + k] = cam.fy * GT[3 + k];
        GH[6 + k] = cam.cx * GT[k] + cam.cy * GT[3 + k] + GT[6 + k];
    }
    float gcol[3][3];   // world-space gradients of the three column vectors
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int r = 0; r < 3; ++r) gcol[k][r] = cam.R[r] * GH[k] + cam.R[3 + r] * GH[3 + k] + cam.R[6 + r] * GH[6 + k];
#pragma unroll
    for (int r = 0; r < 3; ++r) grad_out<kFirst>(&g.mean[(size_t)r * N + i], dmu[r] + gcol[2][r]);
    grad_out<kFirst>(&g.log_scale[i], F.su * (gcol[0][0] * F.tu[0] + gcol[0][1] * F.tu[1] + gcol[0][2] * F.tu[2]));
    grad_out<kFirst>(&g.log_scale[N + i], F.sv * (gcol[1][0] * F.tv[0] + gcol[1][1] * F.tv[1] + gcol[1][2] * F.tv[2]));
    {
        float gtu[3], gtv[3], gw[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) { gtu[r] = F.su * gcol[0][r]; gtv[r] = F.sv * gcol[1][r]; }
        float dot = gtv[0] * F.tv[0] + gtv[1] * F.tv[1] + gtv[2] * F.tv[2];
#pragma unroll
        for (int r = 0; r < 3; ++r) gw[r] = (gtv[r] - F.tv[r] * dot) * F.winv;
        const float gbtu = -(gw[0] * F.tu[0] + gw[1] * F.tu[1] + gw[2] * F.tu[2]);
        float gx[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            grad_out<kFirst>(&g.tan_v[(size_t)r * N + i], gw[r] + gbtu * F.tu[r]);
            gx[r] = gtu[r] - F.btu * gw[r] + gbtu * b[r];
        }
        dot = gx[0] * F.tu[0] + gx[1] * F.tu[1] + gx[2] * F.tu[2];
#pragma unroll
        for (int r = 0; r < 3; ++r) grad_out<kFirst>(&g.tan_u[(size_t)r * N + i], (gx[r] - F.tu[r] * dot) * F.ainv);
    }
}

// Surfels: the 64-byte raster record of a listed point, with centred rows (see binning_common.h for the rest of the
// block's work: compaction and pair emission as for 3D Gaussians).
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_pack2d(Splats2DDev sp, CamDev cam, BinArrays A, Packed2D* __restrict__ packed)
{
    const size_t N = (size_t)sp.n;
    struct Parts { float t[9], o, red, green, blue, mx, my; int radius; };
    pack_block<kThreads>(BinInput{sp.n, sp.mean2d, sp.radius}, cam, A, sp.depth,
        [&](int i, const PointExtent& e) {
            Parts p;
#pragma unroll
            for (int k = 0; k < 9; ++k) p.t[k] = sp.T[k * N + i];
            p.o = sp.opacity[i]; p.red = sp.color[i]; p.green = sp.color[N + i]; p.blue = sp.color[2 * N + i];
            p.mx = e.mx; p.my = e.my; p.radius = e.radius;
            return p;
        },
        [&](int i, const Parts& p) {
            float4* dst = reinterpret_cast<float4*>(packed + i);
            const float* t = p.t;
            const float mx = p.mx, my = p.my;
            dst[0] = make_float4(fmaf(-mx, t[6], t[0]), fmaf(-mx, t[7], t[1]), fmaf(-my, t[6], t[3]), fmaf(-my, t[7], t[4]));
            dst[1] = make_float4(t[6], t[7], t[8], p.o);
            dst[2] = make_float4(mx, my, p.red, p.green);
            dst[3] = make_float4(p.blue, __int_as_float(p.radius), fmaf(-mx, t[8], t[2]), fmaf(-my, t[8], t[5]));
        });
}

// Which of the sixteen 4x4 cells of the tile whose first pixel centre is (x0, y0) can the splat with raster record r0..r3 (L = log2
// of its opacity) touch with alpha >= 1/255? Four bits per quadrant (by_quadrant()). A cell is kept if the bounding box of the
// image of the disk rim where alpha falls to 1/255 (rho^2 = 2 ln(255 o)), or of the low-pass support around the centre, meets
// its pixel centres; taken conservatively, NaN keeps.
__device__ __forceinline__ uint32_t tile_cells2d(const float4& r0, const float4& r1, const float4& r2, const float4& r3, float L,
                                                 float x0, float y0)
{
    const float tau = (L + kLog2_255) * 0.6931471805599453f;      // ln(255 o): alpha >= 1/255 <=> -ln G^ <= tau
    if (tau < -0.02f) return 0u;
    const float rho2 = 2.f * fmaxf(tau, 0.f) + 0.05f;          // rim of the disk part, with margin
    const float lp = sqrtf(fmaxf(tau, 0.f)) + 0.05f;           // radius of the low-pass part, with margin
    // image of the rim u^2 + v^2 = rho2, relative to the projected centre: rows T_0', T_1', T_2
    const float aa = rho2 * (r1.x * r1.x + r1.y * r1.y) - r1.z * r1.z;
    if (!(aa < -0.02f * r1.z * r1.z)) return 0xffffu;   // the rim at this level comes (almost) to the camera plane: keep
    const float ia = 1.0f / aa;
    const float bx = rho2 * (r0.x * r1.x + r0.y * r1.y) - r3.z * r1.z, by = rho2 * (r0.z * r1.x + r0.w * r1.y) - r3.w * r1.z;
    const float cx = rho2 * (r0.x * r0.x + r0.y * r0.y) - r3.z * r3.z, cy = rho2 * (r0.z * r0.z + r0.w * r0.w) - r3.w * r3.w;
    const float c0x = bx * ia, c0y = by * ia;
    const float hx = sqrtf(fmaxf(0.f, c0x * c0x - cx * ia)) * 1.001f + 0.01f;
    const float hy = sqrtf(fmaxf(0.f, c0y * c0y - cy * ia)) * 1.001f + 0.01f;
    // a column or row of cells is out if it lies wholly beside it
    const float lo_x = fminf(-lp, c0x - hx), hi_x = fmaxf(lp, c0x + hx), lo_y = fminf(-lp, c0y - hy), hi_y = fmaxf(lp, c0y + hy);
    const float dx = x0 - r2.x, dy = y0 - r2.y;
    uint32_t cols = 0u, rows = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        cols |= !(hi_x < dx + 4.f * k || lo_x > dx + (4.f * k + 3.f)) ? 1u << k : 0u;
        rows |= !(hi_y < dy + 4.f * k || lo_y > dy + (4.f * k + 3.f)) ? 1u << k : 0u;
    }
    const auto half = [&](uint32_t r) { return by_quadrant(((r & 1u) ? cols : 0u) | ((r & 2u) ? cols << 4 : 0u)); };
    return half(rows) | (half(rows >> 2) << 8);
}

// per-pair evaluation shared by forward and backward: exponent of G^ in log2 units and the pieces the backward needs
struct Pair2D {
    float dx, dy, hu0, hu1, hu2, hv0, hv1, hv2, p2, ip2, u, v, e1, e2;
};

__device__ __forceinline__ void eval_pair2d(const float4& a, const float4& b, const float4& c, const float4& d, float fx, float fy,
                                            Pair2D& E)
{
    E.dx = fx - c.x; E.dy = fy - c.y;
    E.hu0 = E.dx * b.x - a.x; E.hu1 = E.dx * b.y - a.y; E.hu2 = E.dx * b.z - d.y;
    E.hv0 = E.dy * b.x - a.z; E.hv1 = E.dy * b.y - a.w; E.hv2 = E.dy * b.z - d.z;
    const float p0 = E.hu1 * E.hv2 - E.hu2 * E.hv1;
    const float p1 = E.hu2 * E.hv0 - E.hu0 * E.hv2;
    E.p2 = E.hu0 * E.hv1 - E.hu1 * E.hv0;
    E.ip2 = __builtin_amdgcn_rcpf(E.p2);
    E.u = p0 * E.ip2; E.v = p1 * E.ip2;
    E.e1 = (-0.5f * kLog2e) * (E.u * E.u + E.v * E.v);
    E.e2 = -kLog2e * (E.dx * E.dx + E.dy * E.dy);
}

// Forward. The tile's list is staged 256 surfels at a time by the whole workgroup, so that the rim test (over a hundred
// vector instructions) is made once per tile and splat. Independent wavefronts that stage and test for themselves make it
// four times: 344 against 333 us at 2M disks on 2600x1463, 169 against 163 at 1M on 1920x1080; they gain
// only where quadrants end far apart (390 against 424 us at 600k disks on 400x300).
//
// As in the 3D kernel each row of 16 lanes is a 4x4 cell and a visit is one entry of each of the four cells' lists: 64 positions
// that reach the quadrant at a time, LDS offsets of 16 bits, the entries behind a list's end name a record that reaches nothing.
//
// The walk also notes for the backward pass which cells blended which splats: lane i keeps the lane mask of visit i (two
// instructions a visit and two scalar ones), and after a window the lane that stands for a splat asks the lanes of its places in the four lists.
// Against one surfel a visit on the whole quadrant, 1M disks at 1920x1080 145.0 -> 131.0 us, 3,001 at 203x121 17.2 -> 15.4.
constexpr int kFwdBatch2D = 256;

__global__ __launch_bounds__(256, 6) void k_composite2d_fwd(CamDev cam, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                         const uint32_t* __restrict__ vals, const Packed2D* __restrict__ packed,
                                                         uint16_t* __restrict__ blend_words, float bg0, float bg1, float bg2,
                                                         float* __restrict__ image, float* __restrict__ final_T,
                                                         uint32_t* __restrict__ last_idx)
{
    constexpr int kPosBits = 12;
    static_assert(kFwdBatch2D == 256, "a position per thread");
    __shared__ float4 sA[kFwdBatch2D + 1];         // t0x, t0y, t1x, t1y (the last record of each part reaches nothing)
    __shared__ float4 sB[kFwdBatch2D + 1];         // t2x, t2y, t2z, log2(opacity)
    __shared__ float4 sC[kFwdBatch2D + 1];         // mx, my, red, green
    __shared__ float4 sD[kFwdBatch2D + 1];         // blue, t0z, t1z, -
    __shared__ uint16_t sHits[4][kFwdBatch2D];     // per quadrant: position in the batch | the quadrant's cells << kPosBits
    __shared__ __align__(8) uint16_t sList[4][4 * 64 + 4];
    __shared__ uint16_t sCells[kFwdBatch2D];
    __shared__ uint32_t sBlendedWords[kFwdBatch2D];      // as bytes [quadrant][position in the batch]: a bit per cell that blended it
    uint8_t* const sBlended = reinterpret_cast<uint8_t*>(sBlendedWords);
    const int tile = (int)tile_order[blockIdx.x];
    const int tiy = tile / cam.TX, tix = tile - tiy * cam.TX;
    const int tx0 = (cam.otx + tix) * kTile, ty0 = (cam.oty + tiy) * kTile;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = lane >> 4;
    const int px = tx0 + (wave & 1) * 8 + (group & 1) * 4 + (lane & 3), py = ty0 + (wave >> 1) * 8 + (group >> 1) * 4 + ((lane >> 2) & 3);
    const bool inside = px >= cam.rx0 && px < cam.rx1 && py >= cam.ry0 && py < cam.ry1;
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const float x0 = (float)tx0 + 0.5f, y0 = (float)ty0 + 0.5f;     // centre of the tile's first pixel
    constexpr uint32_t kNone = (uint32_t)kFwdBatch2D * 16u * 0x10001u;
    uint16_t* const list_w = sList[wave];
    uint16_t* const hits_w = sHits[wave];
    if (threadIdx.x == 0) {
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        sA[kFwdBatch2D] = zero; sB[kFwdBatch2D] = make_float4(0.f, 0.f, 0.f, -1e30f); sC[kFwdBatch2D] = zero; sD[kFwdBatch2D] = zero;
    }
    float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
    uint32_t last = 0;
    unsigned long long live = __ballot(inside);
    uint32_t id = start + threadIdx.x < end ? vals[start + threadIdx.x] : 0u;      // of this thread's position in the next batch
    for (uint32_t base = start; base < end; base += kFwdBatch2D) {
        const int cnt = (int)min((uint32_t)kFwdBatch2D, end - base);
        uint32_t reach = 0u;
        if ((int)threadIdx.x < cnt) {
            const float4* rec = reinterpret_cast<const float4*>(packed + id);
            const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3];
            id = base + kFwdBatch2D + threadIdx.x < end ? vals[base + kFwdBatch2D + threadIdx.x] : 0u;
            const float L = __log2f(r1.w);
            sA[threadIdx.x] = r0;
            sB[threadIdx.x] = make_float4(r1.x, r1.y, r1.z, L);
            sC[threadIdx.x] = r2;
            sD[threadIdx.x] = make_float4(r3.x, r3.z, r3.w, 0.f);
            reach = tile_cells2d(r0, r1, r2, r3, L, x0, y0);
        }
        sCells[threadIdx.x] = (uint16_t)reach;
        sBlendedWords[threadIdx.x] = 0u;
        __syncthreads();
        uint32_t last_off = ~0u;                     // 16 * place in the batch of the splat the lane blended last
        int nhit = 0;
#pragma unroll
        for (int r = 0; r < kFwdBatch2D; r += 64) {      // (positions past the end have no cells)
            const uint32_t m = ((uint32_t)sCells[r + lane] >> (4 * wave)) & 15u;
            const unsigned long long b = __ballot(m != 0u);
            if (m) hits_w[nhit + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = (uint16_t)((uint32_t)(r + lane) | (m << kPosBits));
            nhit += __builtin_popcountll(b);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int w0 = 0; w0 < nhit; w0 += 64) {
            if (live == 0ull) break;
            uint32_t m = 0u, at = 0u;
            *reinterpret_cast<uint2*>(list_w + 4 * lane) = make_uint2(kNone, kNone);
            if (w0 + lane < nhit) {
                const uint32_t h = hits_w[w0 + lane];
                m = h >> kPosBits;
                at = h & ((1u << kPosBits) - 1u);
            }
            int n = 0;
            uint32_t places = 0u;      // of this lane's splat in the four lists, a byte each
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const bool on = (m & (1u << g)) != 0u && ((live >> (16 * g)) & 0xffffull) != 0ull;
                const unsigned long long b = __ballot(on);
                const int place = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                if (on) list_w[g * 64 + place] = (uint16_t)(at * 16u);
                else m &= ~(1u << g);
                places |= (uint32_t)place << (8 * g);
                n = max(n, (int)__builtin_popcountll(b));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const uint16_t* const my_list = list_w + group * 64;
            int used_lo = 0, used_hi = 0;                // lane i: the lanes that blended in visit i
            // alpha of one visit: everything that does not depend on the pixel's running state. ok: lanes whose alpha counts
            auto eval = [&](uint32_t off, float& alpha, unsigned long long& ok, float& r, float& g, float& bl) {
                const auto from = [off](const float4* p) { return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(p) + off); };
                const float4 a = from(sA), b = from(sB), cc = from(sC), dd = from(sD);
                bl = dd.x; r = cc.z; g = cc.w;
                Pair2D E;
                eval_pair2d(a, b, cc, dd, fx, fy, E);
                alpha = fminf(kAlphaMax, __builtin_amdgcn_exp2f(b.w + fmaxf(E.e1, E.e2)));
                ok = __builtin_amdgcn_ballot_w64(E.p2 != 0.f) & __builtin_amdgcn_ballot_w64(alpha >= kAlphaMin);
            };
            auto blend_one = [&](uint32_t off, float alpha, unsigned long long ok, float r, float g, float bl, unsigned long long& blending_now) {
                const float aT = alpha * T;
                const float Tn = T - aT;            // T (1 - alpha), with the product the weight needs anyway
                const unsigned long long stop = __builtin_amdgcn_ballot_w64(Tn < kTStop);
                const unsigned long long blending = live & ok & ~stop;
                blending_now = blending;
                live &= ~(ok & stop);               // (a lane that is not live may be among these: it is not live anyway)
                const bool blend = __builtin_amdgcn_inverse_ballot_w64(blending);
                // (chosen, not weighted with zero: a colour that is not finite reaches only the pixels that blend it)
                C0 = blend ? fmaf(r, aT, C0) : C0; C1 = blend ? fmaf(g, aT, C1) : C1; C2 = blend ? fmaf(bl, aT, C2) : C2;
                T = blend ? Tn : T;
                last_off = blend ? off : last_off;
            };
            // two visits per trip (independent alphas, blends in list order)
            uint32_t next = *reinterpret_cast<const uint32_t*>(my_list);
            for (int i = 0; i < n; i += 2) {
                const uint32_t o0 = next & 0xffffu, o1 = next >> 16;
                next = *reinterpret_cast<const uint32_t*>(my_list + i + 2);      // (behind the last one: padding or the next list, not used)
                asm volatile("" ::: "memory");                                   // asked for here, a trip ahead
                float al0, red0, grn0, blu0, al1, red1, grn1, blu1;
                unsigned long long ok0, ok1;
                eval(o0, al0, ok0, red0, grn0, blu0);
                eval(o1, al1, ok1, red1, grn1, blu1);
                unsigned long long m0, m1;
                blend_one(o0, al0, ok0, red0, grn0, blu0, m0);
                blend_one(o1, al1, ok1, red1, grn1, blu1, m1);
                uint32_t keep;
                asm("s_mov_b32 %2, m0\n\ts_mov_b32 m0, %7\n\tv_writelane_b32 %0, %3, m0\n\tv_writelane_b32 %1, %4, m0\n\t"
                    "s_add_u32 m0, m0, 1\n\tv_writelane_b32 %0, %5, m0\n\tv_writelane_b32 %1, %6, m0\n\ts_mov_b32 m0, %2"
                    : "+v"(used_lo), "+v"(used_hi), "=&s"(keep)
                    : "s"((uint32_t)m0), "s"((uint32_t)(m0 >> 32)), "s"((uint32_t)m1), "s"((uint32_t)(m1 >> 32)), "s"(i) : "scc");
            }
            // visit i's cells, in lane i; then each splat's, from its places
            const uint32_t visit = ((uint32_t)used_lo & 0xffffu ? 1u : 0u) | ((uint32_t)used_lo >> 16 ? 2u : 0u) | ((uint32_t)used_hi & 0xffffu ? 4u : 0u) | ((uint32_t)used_hi >> 16 ? 8u : 0u);
            uint32_t blended = 0u;
#pragma unroll
            for (int g = 0; g < 4; ++g)
                blended |= (uint32_t)__builtin_amdgcn_ds_bpermute((int)((places >> (8 * g)) & 255u) << 2, (int)visit) & m & (1u << g);
            if (blended) sBlended[wave * kFwdBatch2D + at] = (uint8_t)blended;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();             // the next window overwrites the lists
        }
        if (last_off != ~0u) last = base - start + 1u + last_off / (uint32_t)sizeof(float4);
        const int open = __syncthreads_count(live != 0ull);
        if ((int)threadIdx.x < cnt) {
            uint32_t word = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) word |= (uint32_t)sBlended[q * kFwdBatch2D + threadIdx.x] << (4 * q);
            blend_words[base + threadIdx.x] = (uint16_t)word;
        }
        if (open == 0) break;                        // every pixel of the tile has ended
        __syncthreads();                             // (the blended bits have been read)
    }
    if (inside) {
        const size_t HW = (size_t)cam.W * cam.H;
        const size_t pix = (size_t)(py - cam.ry0) * (size_t)cam.W + (size_t)(px - cam.rx0);
        image[pix] = C0 + T * bg0;
        image[HW + pix] = C1 + T * bg1;
        image[2 * HW + pix] = C2 + T * bg2;
        final_T[pix] = T;
        last_idx[pix] = last;
    }
}

// Backward. With dp = dL/dp for p = h_u x h_v (three numbers per pair), the gradient of the transform is a lane sum of
// the moments S0 = sum dp, Sx = sum dx dp, Sy = sum dy dp (dx, dy from the projected centre):
//   sum dL/dh_u = T_2 x Sy - T_1' x S0,   sum dL/dh_v = Sx x T_2 - S0 x T_0',
//   dT_0 = -sum dL/dh_u, dT_1 = -sum dL/dh_v, dT_2 = mx sum dL/dh_u + my sum dL/dh_v - T_1' x Sx - Sy x T_0'.
// Together with 3 colour sums, sum G^ dL/dalpha (d opacity) and the 2 low-pass sums for mean2d: 15 sums per splat and one
// 64-byte record per (tile, splat) pair. dp and the low-pass sums leave out the factors o and, the latter, 2; the record
// has them.
//
// As in the 3D kernel a visit is one entry of each of the four cells' lists, and the sums over pixels are taken four visits at a
// time: a visit stores five numbers per pixel (dp, the blend weight, G^ dL/dalpha) as rows of 64 floats in LDS; after four visits
// each row of 16 lanes takes one of them and a quad of lanes each cell, a lane the numbers of four neighbouring pixels, a row of the
// cell, whose dx, dy and dL/dcolour give its 15 weighted sums, and two exchanges inside the quad finish sixteen (splat, cell)
// pairs at once. The sums are kept by visit and cell for kBwdVisits2D visits; then the lane that stands for a splat adds up those
// of its places in the four lists. Which pixels take the disk part is the sign of their weight, which is never negative itself:
// one instruction a visit (as a ballot kept in the lanes that need it, five). kRows2D rows, not six: the LDS then holds four
// workgroups per compute unit.
//
// Only the cells that blended a splat list it, and only the entries that some cell blended are staged, 64 of them at a time
// wherever they stand in the list.
// Against one surfel a visit on the whole quadrant, 27 % of whose lanes blended it: 1M disks at 1920x1080 296.6 -> 250.8 us, 3,001 at
// 203x121 36.8 -> 29.2; the errors against 64 bits are the same (mean2d 1.42e-7, opacity 1.75e-7, colour 1.78e-7, six scenes of 120k
// disks at 960x540).
constexpr int kBwdBatch2D = 64;    // surfels staged at a time by the backward kernel: one per lane
constexpr uint32_t kBwdChunk2D = 256;      // list positions that are searched for blended entries at a time, one per thread
constexpr int kSlots2D = 4;        // visits staged per reduction: one per row of 16 lanes
constexpr int kRows2D = 5;         // rows a visit stores: dp (3), signed w, G^ dL/dalpha
constexpr int kBwdVisits2D = 12;   // visits whose sums a wavefront keeps before it adds them up by splat (a multiple of kSlots2D)

__global__ __launch_bounds__(256, 4) void k_composite2d_bwd(CamDev cam, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                         const uint32_t* __restrict__ vals, const Packed2D* __restrict__ packed,
                                                         const uint16_t* __restrict__ blend_words, const uint32_t* __restrict__ slot_base,
                                                         float bg0, float bg1, float bg2,
                                                         const float* __restrict__ final_T, const uint32_t* __restrict__ last_idx,
                                                         const float* __restrict__ dL_dimage, uint32_t cap,
                                                         float4* __restrict__ partial)
{
    // the batch: t0x, t0y, t1x, t1y; t2x, t2y, t2z, log2(opacity); mx, my, red, green; blue, t0z, t1z, list position + 1. The last
    // record of each part reaches nothing.
    __shared__ float4 sA[kBwdBatch2D + 1], sB[kBwdBatch2D + 1], sC[kBwdBatch2D + 1], sD[kBwdBatch2D + 1];
    __shared__ uint16_t sCells[kBwdBatch2D];
    // per wavefront: visit slot s has rows kRows2D s ...; then, at the end of a batch, the wavefront's sums by splat, four parts of
    // [splat] float4
    __shared__ __align__(16) float sV[4][kRows2D * kSlots2D * 64];
    __shared__ __align__(16) float sSum[4][kBwdVisits2D * 64];        // per wavefront: [visit][cell][16 sums]
    __shared__ __align__(8) uint16_t sList[4][4 * kBwdBatch2D];
    __shared__ uint32_t sMax[4], sCount[4];
    __shared__ uint16_t sFound[kBwdBatch2D + kBwdChunk2D];
    static_assert(kRows2D * kSlots2D * 64 >= 16 * kBwdBatch2D && kBwdVisits2D % kSlots2D == 0, "the sums by splat fit where the rows were");
    const int tile = (int)tile_order[blockIdx.x];
    const int tile_y = tile / cam.TX, tile_x = tile - tile_y * cam.TX;
    const int tx0 = (cam.otx + tile_x) * kTile, ty0 = (cam.oty + tile_y) * kTile;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = lane >> 4;
    const int px = tx0 + (wave & 1) * 8 + (group & 1) * 4 + (lane & 3), py = ty0 + (wave >> 1) * 8 + (group >> 1) * 4 + ((lane >> 2) & 3);
    const bool inside = px >= cam.rx0 && px < cam.rx1 && py >= cam.ry0 && py < cam.ry1;
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const size_t HW = (size_t)cam.W * cam.H;
    float T = 1.f, g0 = 0.f, g1 = 0.f, g2c = 0.f;
    uint32_t last = 0;
    if (inside) {
        const uint32_t pix = (uint32_t)(py - cam.ry0) * (uint32_t)cam.W + (uint32_t)(px - cam.rx0);
        T = final_T[pix];
        last = min(last_idx[pix], end - start);
        g0 = dL_dimage[pix]; g1 = dL_dimage[HW + pix]; g2c = dL_dimage[2 * HW + pix];
    }
    float Sfx = T * (bg0 * g0 + bg1 * g1 + bg2 * g2c);
    uint32_t wmax = last;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) wmax = max(wmax, (uint32_t)__shfl_xor((int)wmax, d, 64));
    if (lane == 0) sMax[wave] = wmax;     // the last list position any pixel of the quadrant blended
    if (threadIdx.x == 0) {
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        sA[kBwdBatch2D] = zero; sB[kBwdBatch2D] = make_float4(0.f, 0.f, 0.f, -1e30f);
        sC[kBwdBatch2D] = zero; sD[kBwdBatch2D] = make_float4(0.f, 0.f, 0.f, __uint_as_float(0xffffffffu));
    }
    __syncthreads();
    const uint32_t tile_last = __builtin_amdgcn_readfirstlane(max(max(sMax[0], sMax[1]), max(sMax[2], sMax[3])));
    // Pairs that no pixel of the tile blended are never staged; the gather adds up the records of all pairs, so theirs are
    // written as zeros: those behind the last blended splat here, the others where the search below comes to them (every
    // pair is in exactly one tile's list: each record is written exactly once per call, and no fill of the whole array is
    // needed beforehand).
    const auto write_zeros = [&](uint32_t idz) {
        const float4* rz = reinterpret_cast<const float4*>(packed + idz);
        const float4 z2 = rz[2], z3 = rz[3];
        int x0, y0, x1, y1;
        tile_rect(cam, z2.x, z2.y, __float_as_int(z3.y), x0, y0, x1, y1);
        const uint32_t u = slot_base[idz] + (uint32_t)((tile_y - y0) * (x1 - x0) + (tile_x - x0));
        if (u < cap && tile_x >= x0 && tile_x < x1 && tile_y >= y0 && tile_y < y1) {
            float4* dst = partial + (size_t)4 * u;
            const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
            dst[0] = zero; dst[1] = zero; dst[2] = zero; dst[3] = zero;
        }
    };
    for (uint32_t p = tile_last + threadIdx.x; p < end - start; p += 256u) write_zeros(vals[start + p]);
    if (tile_last == 0) return;
    float* const sVw = sV[wave];
    float* const sSumW = sSum[wave];
    uint16_t* const list_w = sList[wave];
    // In a reduction lane l takes visit slot l / 16 and the four pixels held by the wavefront's lanes 4 pg .. 4 pg + 3,
    // pg = l % 16: a row of a 4x4 cell. Their dL/dcolour come from those lanes, through LDS.
    const int pg = lane & 15, cell = pg >> 2, quad_lane = lane & 3;
    float4 G0, G1, G2;
    {
        sVw[lane] = g0; sVw[64 + lane] = g1; sVw[128 + lane] = g2c;
        __builtin_amdgcn_wave_barrier();
        G0 = *reinterpret_cast<const float4*>(sVw + 4 * pg);
        G1 = *reinterpret_cast<const float4*>(sVw + 64 + 4 * pg);
        G2 = *reinterpret_cast<const float4*>(sVw + 128 + 4 * pg);
        __builtin_amdgcn_wave_barrier();
    }
    // centre of the first of the four pixels; the others follow on the same row
    const float rx = (float)(tx0 + (wave & 1) * 8 + (cell & 1) * 4) + 0.5f, ry = (float)(ty0 + (wave >> 1) * 8 + (cell >> 1) * 4 + quad_lane) + 0.5f;
    const float* const rd_row = sVw + kRows2D * 64 * (lane >> 4) + 4 * pg;
    float* const wr_row = sVw + lane;
    float* const wr_sum = sSumW + 64 * (lane >> 4) + 16 * cell + 2 * quad_lane;
    const uint16_t* const rd_list = list_w + cell * kBwdBatch2D + (lane >> 4);
    // Reduces the staged rows, visits at .. at + 3 of the lists: the sums of slot s go to place i + s of the run.
    auto reduce_slots = [&](int at, int i) {
        __builtin_amdgcn_wave_barrier();
        const float4 d0 = *reinterpret_cast<const float4*>(rd_row);
        const float4 d1 = *reinterpret_cast<const float4*>(rd_row + 64);
        const float4 d2 = *reinterpret_cast<const float4*>(rd_row + 128);
        const float4 w = *reinterpret_cast<const float4*>(rd_row + 192);
        const float4 e = *reinterpret_cast<const float4*>(rd_row + 256);
        const float2 centre = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(sC) + rd_list[at]);
        __builtin_amdgcn_wave_barrier();
        // each pixel's own offset (exact near the centre): dx of the first pixel times the sum, plus a ramp over the four,
        // cancels where the weight sits beside the centre
        const float dx0 = rx - centre.x, dx1 = rx + 1.f - centre.x, dx2 = rx + 2.f - centre.x, dx3 = rx + 3.f - centre.x, dy = ry - centre.y;
        const auto sum4 = [](const float4& v) { return (v.x + v.y) + (v.z + v.w); };
        const auto sum4x = [&](const float4& v) { return (v.x * dx0 + v.y * dx1) + (v.z * dx2 + v.w * dx3); };
        const float m0 = sum4(d0), m1 = sum4(d1), m2 = sum4(d2);
        const auto unless_disk = [](float ws, float v) { return __float_as_int(ws) < 0 ? 0.f : v; };
        const float4 l = make_float4(unless_disk(w.x, e.x), unless_disk(w.y, e.y), unless_disk(w.z, e.z), unless_disk(w.w, e.w));
        const auto sumw = [&](const float4& G) { return fabsf(w.x) * G.x + fabsf(w.y) * G.y + fabsf(w.z) * G.z + fabsf(w.w) * G.w; };
        const float va[8] = {m0, m1, m2, sum4x(d0), sum4x(d1), sum4x(d2), dy * m0, dy * m1};
        const float vb[8] = {dy * m2,
                             sumw(G0), sumw(G1), sumw(G2),
                             sum4(e), sum4x(l), dy * sum4(l), 0.f};
        float2 pa, pb;
        quad_sum8(va, quad_lane, pa);
        quad_sum8(vb, quad_lane, pb);
        *reinterpret_cast<float2*>(wr_sum + 64 * i) = pa;
        *reinterpret_cast<float2*>(wr_sum + 64 * i + 8) = pb;
    };
    // The list is searched from its end for the entries that some cell blended, a chunk of 256 positions at a time;
    // blend_words has four bits per quadrant, one per cell. The forward pass writes the words of
    // every position that its tile staged, and no pixel's last index lies behind those, so no word of an earlier call is
    // read here. What was found and not staged yet: sFound[head ..], nfound entries, positions falling. They are kept in
    // 16 bits, so that four workgroups still fit a compute unit; the upper 16 are `page`, and a chunk of another page
    // waits until the entries of this one are staged.
    uint32_t nfound = 0u, head = 0u, page = 0u, todo = tile_last;      // positions below `todo` are still to be searched
    uint32_t chunk_bits = 0u, chunk_id = 0u;                           // of this thread's position in the next chunk
    const auto ask_chunk = [&] {
        const uint32_t p = ((todo - 1u) & ~(kBwdChunk2D - 1u)) + (kBwdChunk2D - 1u) - threadIdx.x;
        chunk_bits = 0u;
        if (todo > 0u && p < todo) { chunk_bits = blend_words[start + p]; chunk_id = vals[start + p]; }
    };
    ask_chunk();
    for (;;) {
        while (nfound < (uint32_t)kBwdBatch2D && todo > 0u && (nfound == 0u || (todo - 1u) >> 16 == page)) {
            const uint32_t chunk = (todo - 1u) & ~(kBwdChunk2D - 1u);
            const uint32_t p = chunk + (kBwdChunk2D - 1u) - threadIdx.x;
            const bool blended = chunk_bits != 0u;
            const unsigned long long m = __ballot(blended);
            if (lane == 0) sCount[wave] = (uint32_t)__popcll(m);
            const uint16_t left = threadIdx.x < nfound ? sFound[head + threadIdx.x] : (uint16_t)0;
            __syncthreads();
            if (threadIdx.x < nfound) sFound[threadIdx.x] = left;
            uint32_t at = nfound, total = 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t n = sCount[k];
                if (k < wave) at += n;
                total += n;
            }
            if (blended) sFound[at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)p;
            else if (p < todo) write_zeros(chunk_id);
            nfound += __builtin_amdgcn_readfirstlane(total);
            head = 0u;
            page = chunk >> 16;
            todo = chunk;
            ask_chunk();
            __syncthreads();
        }
        if (nfound == 0u) break;      // (then nothing is left to search either)
        const int cnt = (int)min((uint32_t)kBwdBatch2D, nfound);
        // stage the batch, one entry per lane of the first wavefront, list positions rising with the lane
        uint32_t id = 0u;
        float opacity = 0.f, radius_bits = 0.f;
        if ((int)threadIdx.x < cnt) {
            const uint32_t p = (page << 16) | sFound[head + (uint32_t)cnt - 1u - threadIdx.x];
            id = vals[start + p];
            sCells[threadIdx.x] = blend_words[start + p];
            const float4* rec = reinterpret_cast<const float4*>(packed + id);
            const float4 q0 = rec[0], q1 = rec[1], q2 = rec[2], q3 = rec[3];
            opacity = q1.w; radius_bits = q3.y;
            sA[threadIdx.x] = q0;
            sB[threadIdx.x] = make_float4(q1.x, q1.y, q1.z, __log2f(q1.w));
            sC[threadIdx.x] = q2;
            sD[threadIdx.x] = make_float4(q3.x, q3.z, q3.w, __uint_as_float(p + 1u));
        }
        head += (uint32_t)cnt;
        nfound -= (uint32_t)cnt;
        __syncthreads();
        // the lists of the quadrant's cells, last splats first
        constexpr uint32_t kNone = (uint32_t)kBwdBatch2D * 16u * 0x10001u;
        *reinterpret_cast<uint2*>(list_w + 4 * lane) = make_uint2(kNone, kNone);
        const uint32_t cells = lane < cnt ? ((uint32_t)sCells[lane] >> (4 * wave)) & 15u : 0u;
        int n = 0;
        uint32_t places = 0u;             // of this lane's splat in the lists
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const unsigned long long b = __ballot((cells & (1u << g)) != 0u);
            const int c = __builtin_popcountll(b);
            const int place = c - 1 - (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
            const bool on = (cells & (1u << g)) != 0u;
            if (on) list_w[g * kBwdBatch2D + place] = (uint16_t)(lane * 16);
            places |= (on ? (uint32_t)place : 255u) << (8 * g);
            n = max(n, c);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // of the upper and of the lower two cells: two terms each, so that the sum does not depend on which run of visits has which
        float4 acc[2][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[0][k] = acc[1][k] = make_float4(0.f, 0.f, 0.f, 0.f);
        const uint16_t* const my_list = list_w + group * kBwdBatch2D;
        for (int first = 0; first < n; first += kBwdVisits2D) {
            const int count = min(kBwdVisits2D, n - first);
            const auto visit = [&](uint32_t off, float* rows) {
                const auto from = [off](const float4* p) { return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(p) + off); };
                const float4 a = from(sA), b = from(sB), cc = from(sC), dd = from(sD);
                const uint32_t pos = __float_as_uint(dd.w);      // list position + 1
                const float blue = dd.x;
                Pair2D E;
                eval_pair2d(a, b, cc, dd, fx, fy, E);
                const bool disk = E.e1 > E.e2;                         // which part of the max is active (false for NaN)
                const float ex = disk ? E.e1 : E.e2;
                const float araw = __builtin_amdgcn_exp2f(b.w + ex);   // o G^
                const float alpha = fminf(kAlphaMax, araw);
                const bool hit = (pos <= last) && (E.p2 != 0.f) && (alpha >= kAlphaMin);
                const float ioma = __builtin_amdgcn_rcpf(1.f - alpha);
                const float Tk = T * ioma;
                const float w = hit ? alpha * Tk : 0.f;
                const float cg = cc.z * g0 + cc.w * g1 + blue * g2c;
                const float dL_dalpha = Tk * cg - Sfx * ioma;
                const float da = (hit && araw < kAlphaMax) ? dL_dalpha : 0.f;     // zero where alpha was clamped
                T = hit ? Tk : T;
                Sfx += w * cg;
                // G^ by an exponential of its own: the opacity's gradient is the sum of G^ dL/dalpha, and o G^ over o
                // carries the rounding of log2(o). The sums below leave o out; the record multiplies them by it.
                const float d_o = __builtin_amdgcn_exp2f(ex) * da;       // zero unless hit
                // disk part: dL/du = -u o G dL/dalpha; low-pass part (the sums of the reduction): dL/dmx = 2 dx o G2 dL/dalpha.
                // u, v, 1/p2 are finite wherever the disk part is the active one; elsewhere they are replaced by 0
                // so that no 0 * inf reaches the sums.
                const float us = disk ? E.u : 0.f, vs = disk ? E.v : 0.f, ips = disk ? E.ip2 : 0.f;
                const float du = -us * d_o, dv = -vs * d_o;
                rows[0] = du * ips;
                rows[64] = dv * ips;
                rows[128] = -(du * us + dv * vs) * ips;
                rows[192] = disk ? -w : w;      // the sign marks the disk part
                rows[256] = d_o;
            };
            const uint16_t* const run = my_list + first;
            for (int i = 0; i < count; i += kSlots2D) {      // (behind the lists' ends: a record that reaches nothing)
                const uint2 o = *reinterpret_cast<const uint2*>(run + i);
                visit(o.x & 0xffffu, wr_row);
                if (i + 1 < count) visit(o.x >> 16, wr_row + kRows2D * 64);
                if (i + 2 < count) visit(o.y & 0xffffu, wr_row + 2 * kRows2D * 64);
                if (i + 3 < count) visit(o.y >> 16, wr_row + 3 * kRows2D * 64);
                reduce_slots(first + i, i);      // (what the rows of the slots behind the last visit hold goes to places that no splat has)
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint32_t at = ((places >> (8 * g)) & 255u) - (uint32_t)first;
                if (at < (uint32_t)kBwdVisits2D) {
                    const float4* v = reinterpret_cast<const float4*>(sSumW + 64 * at + 16 * g);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        float4& sum = acc[g >> 1][k];
                        sum.x += v[k].x; sum.y += v[k].y; sum.z += v[k].z; sum.w += v[k].w;
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            reinterpret_cast<float4*>(sVw)[k * kBwdBatch2D + lane] = make_float4(acc[0][k].x + acc[1][k].x, acc[0][k].y + acc[1][k].y, acc[0][k].z + acc[1][k].z, acc[0][k].w + acc[1][k].w);
        __syncthreads();
        if ((int)threadIdx.x < cnt) {
            const float4 q0 = sA[threadIdx.x], q1 = sB[threadIdx.x], q2 = sC[threadIdx.x];
            const float2 q3 = make_float2(sD[threadIdx.x].y, sD[threadIdx.x].z);
            int x0, y0, x1, y1;
            tile_rect(cam, q2.x, q2.y, __float_as_int(radius_bits), x0, y0, x1, y1);
            const uint32_t u = slot_base[id] + (uint32_t)((tile_y - y0) * (x1 - x0) + (tile_x - x0));
            if (u < cap && tile_x >= x0 && tile_x < x1 && tile_y >= y0 && tile_y < y1) {
                float acc[15];
#pragma unroll
                for (int k = 0; k < 15; ++k) {
                    const int e = 4 * ((k >> 2) * kBwdBatch2D + (int)threadIdx.x) + (k & 3);
                    acc[k] = (sV[0][e] + sV[1][e]) + (sV[2][e] + sV[3][e]);
                }
                const float o = opacity;
                const float s0[3] = {o * acc[0], o * acc[1], o * acc[2]};
                const float sx[3] = {o * acc[3], o * acc[4], o * acc[5]};
                const float sy[3] = {o * acc[6], o * acc[7], o * acc[8]};
                const float t0[3] = {q0.x, q0.y, q3.x}, t1[3] = {q0.z, q0.w, q3.y}, t2[3] = {q1.x, q1.y, q1.z};
                const float mx = q2.x, my = q2.y;
                float dhu[3], dhv[3], ex[3];
                // sum dL/dh_u = T2 x Sy - T1' x S0
                dhu[0] = (t2[1] * sy[2] - t2[2] * sy[1]) - (t1[1] * s0[2] - t1[2] * s0[1]);
                dhu[1] = (t2[2] * sy[0] - t2[0] * sy[2]) - (t1[2] * s0[0] - t1[0] * s0[2]);
                dhu[2] = (t2[0] * sy[1] - t2[1] * sy[0]) - (t1[0] * s0[1] - t1[1] * s0[0]);
                // sum dL/dh_v = Sx x T2 - S0 x T0'
                dhv[0] = (sx[1] * t2[2] - sx[2] * t2[1]) - (s0[1] * t0[2] - s0[2] * t0[1]);
                dhv[1] = (sx[2] * t2[0] - sx[0] * t2[2]) - (s0[2] * t0[0] - s0[0] * t0[2]);
                dhv[2] = (sx[0] * t2[1] - sx[1] * t2[0]) - (s0[0] * t0[1] - s0[1] * t0[0]);
                // - T1' x Sx - Sy x T0'
                ex[0] = -(t1[1] * sx[2] - t1[2] * sx[1]) - (sy[1] * t0[2] - sy[2] * t0[1]);
                ex[1] = -(t1[2] * sx[0] - t1[0] * sx[2]) - (sy[2] * t0[0] - sy[0] * t0[2]);
                ex[2] = -(t1[0] * sx[1] - t1[1] * sx[0]) - (sy[0] * t0[1] - sy[1] * t0[0]);
                float4* dst = partial + (size_t)4 * u;
                dst[0] = make_float4(-dhu[0], -dhu[1], -dhu[2], -dhv[0]);                                     // dT0, dT1.x
                dst[1] = make_float4(-dhv[1], -dhv[2], mx * dhu[0] + my * dhv[0] + ex[0], mx * dhu[1] + my * dhv[1] + ex[1]);
                dst[2] = make_float4(mx * dhu[2] + my * dhv[2] + ex[2], 2.f * o * acc[13], 2.f * o * acc[14],   // dT2.z, d mean2d
                                     acc[12]);                                                          // d opacity
                dst[3] = make_float4(acc[9], acc[10], acc[11], 0.f);        // d colour
            }
        }
        __syncthreads();
    }
}

// Per point: add up the 64-byte partial records of its pairs (balanced by pairs, see pair_reduce.h).
struct StoreSplat2DGrad {      // one 64-byte record per point, by point index (see the 3D variant)
    float4* rec;
    const uint32_t* order;
    __device__ __forceinline__ void operator()(uint32_t rank, const float (&v)[15]) const
    {
        float4* dst = rec + (size_t)4 * order[rank];
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
        dst[2] = make_float4(v[8], v[9], v[10], v[11]);
        dst[3] = make_float4(v[12], v[13], v[14], 0.f);
    }
};

__global__ __launch_bounds__(256) void k_gather2d(int n, const uint32_t* __restrict__ status, const uint32_t* __restrict__ order,
                                                  const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ chunk_rank,
                                                  const float4* __restrict__ partial, uint32_t cap, float* __restrict__ carry,
                                                  float4* __restrict__ rec)
{
    __shared__ uint32_t sEnd[4][64];
    const uint32_t w = blockIdx.x * 4u + (threadIdx.x >> 6);
    gather_wave<4, 15, false>(w, n, status, offsets, chunk_rank, partial, cap, carry, sEnd[threadIdx.x >> 6], StoreSplat2DGrad{rec, order});
}

__global__ __launch_bounds__(256) void k_grad_records_to_planes2d(int n, const uint32_t* __restrict__ tiles_touched,
                                                                  const float4* __restrict__ rec, CarryFold cf, Splat2DGradDev g2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t pairs = tiles_touched[i];
    if (pairs == 0) return;
    const size_t N = (size_t)n;
    const float4 a = rec[(size_t)4 * i], b = rec[(size_t)4 * i + 1], c = rec[(size_t)4 * i + 2], d = rec[(size_t)4 * i + 3];
    float v[15] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w, d.x, d.y, d.z};
    (void)record_from_carries<15>(cf, cf.slot_base[i], pairs, v);      // (see the 3D variant)
#pragma unroll
    for (int k = 0; k < 9; ++k) g2.T[(size_t)k * N + i] = v[k];
    g2.mean2d[i] = v[9]; g2.mean2d[N + i] = v[10];
    g2.opacity[i] = v[11];
    g2.color[i] = v[12]; g2.color[N + i] = v[13]; g2.color[2 * N + i] = v[14];
}

// Measurement aid: the forward walk with counters instead of colours (see the 3D variant).
__global__ __launch_bounds__(256) void k_render_stats2d(CamDev cam, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                        const uint32_t* __restrict__ vals, const Packed2D* __restrict__ packed,
                                                        unsigned long long* __restrict__ counters)
{
    __shared__ float4 sR[4][kBatch];
    __shared__ unsigned long long sCnt[2];
    const TileCtx c = tile_ctx(cam, ranges, tile_order);
    const float fx = (float)c.px + 0.5f, fy = (float)c.py + 0.5f;
    float T = 1.f;
    uint32_t examined = 0, blended = 0;
    bool done = !c.inside;
    if (threadIdx.x < 2) sCnt[threadIdx.x] = 0ull;
    for (uint32_t base = c.start; base < c.end; base += kBatch) {
        if (__syncthreads_count(!done) == 0) break;
        const uint32_t idx = base + threadIdx.x;
        if (idx < c.end) {
            const float4* rec = reinterpret_cast<const float4*>(packed + vals[idx]);
#pragma unroll
            for (int k = 0; k < 4; ++k) sR[k][threadIdx.x] = rec[k];
        }
        __syncthreads();
        const int cnt = (int)min((uint32_t)kBatch, c.end - base);
        if (!done) {
            for (int j = 0; j < cnt; ++j) {
                const float4 a = sR[0][j], b = sR[1][j], cc = sR[2][j], r3 = sR[3][j];
                Pair2D E;
                eval_pair2d(a, b, cc, make_float4(r3.x, r3.z, r3.w, 0.f), fx, fy, E);
                ++examined;
                if (E.p2 == 0.f) continue;
                const float alpha = fminf(kAlphaMax, b.w * __builtin_amdgcn_exp2f(fmaxf(E.e1, E.e2)));
                if (!(alpha >= kAlphaMin)) continue;
                const float Tn = T - alpha * T;     // as the forward kernel forms it
                if (Tn < kTStop) { done = true; break; }
                T = Tn;
                ++blended;
            }
        }
    }
    __syncthreads();
    atomicAdd(&sCnt[0], (unsigned long long)examined);
    atomicAdd(&sCnt[1], (unsigned long long)blended);
    __syncthreads();
    if (threadIdx.x < 2 && sCnt[threadIdx.x]) atomicAdd(&counters[threadIdx.x], sCnt[threadIdx.x]);
}

__global__ __launch_bounds__(64) void k_zero_counters2d(unsigned long long* __restrict__ counters)
{
    if (threadIdx.x < 2) counters[threadIdx.x] = 0ull;
}

// ---------------------------------------------------------------------------------------------------- launchers
hipError_t launch_preprocess2d(const Scene2DDev& sc, const CamDev& cam, const Splats2DDev& out, hipStream_t s)
{
    if (sc.n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((sc.n + 255) / 256);
    ProfScope prof(kKPreprocess, s);
    switch (sc.sh_degree) {
        case 0: hipLaunchKernelGGL(k_preprocess2d<0>, dim3(blocks), dim3(256), 0, s, sc, cam, out); break;
        case 1: hipLaunchKernelGGL(k_preprocess2d<1>, dim3(blocks), dim3(256), 0, s, sc, cam, out); break;
        case 2: hipLaunchKernelGGL(k_preprocess2d<2>, dim3(blocks), dim3(256), 0, s, sc, cam, out); break;
        default: hipLaunchKernelGGL(k_preprocess2d<3>, dim3(blocks), dim3(256), 0, s, sc, cam, out); break;
    }
    return hipGetLastError();
}

template <bool kFirst, bool kFromRecords>
static void launch_preprocess2d_bwd_t(const Scene2DDev& sc, const CamDev& cam, const int32_t* used, const float* Tst,
                                      const Splat2DGradDev& g2, const float4* rec, const CarryFold& cf, const Scene2DGradDev& g, unsigned blocks,
                                      hipStream_t s)
{
    switch (sc.sh_degree) {
        case 0: hipLaunchKernelGGL((k_preprocess2d_bwd<0, kFirst, kFromRecords>), dim3(blocks), dim3(256), 0, s, sc, cam, used, Tst, g2, rec, cf, g); break;
        case 1: hipLaunchKernelGGL((k_preprocess2d_bwd<1, kFirst, kFromRecords>), dim3(blocks), dim3(256), 0, s, sc, cam, used, Tst, g2, rec, cf, g); break;
        case 2: hipLaunchKernelGGL((k_preprocess2d_bwd<2, kFirst, kFromRecords>), dim3(blocks), dim3(256), 0, s, sc, cam, used, Tst, g2, rec, cf, g); break;
        default: hipLaunchKernelGGL((k_preprocess2d_bwd<3, kFirst, kFromRecords>), dim3(blocks), dim3(256), 0, s, sc, cam, used, Tst, g2, rec, cf, g); break;
    }
}

hipError_t launch_preprocess2d_bwd(const Scene2DDev& sc, const CamDev& cam, const Splats2DDev& sp, const Splat2DGradDev& g2,
                                   const Scene2DGradDev& g, bool first_view, hipStream_t s)
{
    if (sc.n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((sc.n + 255) / 256);
    ProfScope prof(kKPreprocessBwd, s);
    const CarryFold no_fold{nullptr, nullptr, nullptr, 0u};
    if (first_view) launch_preprocess2d_bwd_t<true, false>(sc, cam, sp.radius, sp.T, g2, nullptr, no_fold, g, blocks, s);
    else launch_preprocess2d_bwd_t<false, false>(sc, cam, sp.radius, sp.T, g2, nullptr, no_fold, g, blocks, s);
    return hipGetLastError();
}

// the same from the per-point gradient records in the workspace (see k_preprocess2d_bwd)
hipError_t launch_preprocess2d_bwd_records(const Scene2DDev& sc, const CamDev& cam, const Splats2DDev& sp, const uint32_t* tiles_touched,
                                           const float4* rec, const CarryFold& cf, const Scene2DGradDev& g, bool first_view, hipStream_t s)
{
    if (sc.n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((sc.n + 255) / 256);
    const int32_t* used = reinterpret_cast<const int32_t*>(tiles_touched);     // counts are far below 2^31
    const Splat2DGradDev none{nullptr, nullptr, nullptr, nullptr};
    ProfScope prof(kKPreprocessBwd, s);
    if (first_view) launch_preprocess2d_bwd_t<true, true>(sc, cam, used, sp.T, none, rec, cf, g, blocks, s);
    else launch_preprocess2d_bwd_t<false, true>(sc, cam, used, sp.T, none, rec, cf, g, blocks, s);
    return hipGetLastError();
}

hipError_t launch_bin_sort2d(const Splats2DDev& sp, const CamDev& cam, const Layout& L, char* ws, hipStream_t s)
{
    if (sp.n == 0) return launch_bin_begin(L, ws, s);      // nothing to count: only the cleared status words and ranges
    hipError_t e = launch_bin_count(BinInput{sp.n, sp.mean2d, sp.radius}, cam, L, ws, s);
    if (e != hipSuccess) return e;
    {
        ProfScope prof(kKPack, s);
        const unsigned nb = (unsigned)((sp.n + 255) / 256);
        Packed2D* packed = reinterpret_cast<Packed2D*>(ws + L.off_packed);
        if (block_threads(sp.n) == 256) hipLaunchKernelGGL(k_pack2d<256>, dim3(nb), dim3(256), 0, s, sp, cam, bin_arrays(L, ws), packed);
        else hipLaunchKernelGGL(k_pack2d<1024>, dim3(nb), dim3(1024), 0, s, sp, cam, bin_arrays(L, ws), packed);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_tile_depth_sort(cam, L, ws, s);
}

hipError_t launch_composite2d_fwd(const CamDev& cam, const Layout& L, char* ws, const float bg[3], float* image,
                                  float* final_T, uint32_t* last_idx, hipStream_t s)
{
    ProfScope prof(kKCompositeFwd, s);
    hipLaunchKernelGGL(k_composite2d_fwd, dim3((unsigned)(cam.TX * cam.TY)), dim3(256), 0, s, cam,
                       reinterpret_cast<const uint32_t*>(ws + L.off_ranges), reinterpret_cast<const uint32_t*>(ws + L.off_tile_order),
                       reinterpret_cast<const uint32_t*>(ws + L.off_vals),
                       reinterpret_cast<const Packed2D*>(ws + L.off_packed), reinterpret_cast<uint16_t*>(ws + L.off_reach),
                       bg[0], bg[1], bg[2], image, final_T, last_idx);
    return hipGetLastError();
}

hipError_t launch_composite2d_bwd(const CamDev& cam, const Layout& L, char* ws, int n, const float bg[3], const float* final_T,
                                  const uint32_t* last_idx, const float* dL_dimage, const Splat2DGradDev& g2, hipStream_t s)
{
    const uint32_t* status = reinterpret_cast<const uint32_t*>(ws + L.off_status);
    float4* partial = reinterpret_cast<float4*>(ws + L.off_partial);
    {
        ProfScope prof(kKCompositeBwd, s);
        hipLaunchKernelGGL(k_composite2d_bwd, dim3((unsigned)(cam.TX * cam.TY)), dim3(256), 0, s, cam,
                           reinterpret_cast<const uint32_t*>(ws + L.off_ranges), reinterpret_cast<const uint32_t*>(ws + L.off_tile_order),
                       reinterpret_cast<const uint32_t*>(ws + L.off_vals),
                           reinterpret_cast<const Packed2D*>(ws + L.off_packed), reinterpret_cast<const uint16_t*>(ws + L.off_reach),
                           reinterpret_cast<const uint32_t*>(ws + L.off_slot_base),
                           bg[0], bg[1], bg[2], final_T, last_idx, dL_dimage, L.cap, partial);
    }
    if (n > 0) {
        ProfScope prof(kKGather, s);
        const uint32_t* order = reinterpret_cast<const uint32_t*>(ws + L.off_order);
        const uint32_t* offsets = reinterpret_cast<const uint32_t*>(ws + L.off_offsets);
        const uint32_t* chunk_rank = reinterpret_cast<const uint32_t*>(ws + L.off_chunk_rank);
        float* carry = reinterpret_cast<float*>(ws + L.off_carry);
        const unsigned nwave = (unsigned)gather_chunks_max(L.cap);
        float4* rec = reinterpret_cast<float4*>(ws + L.off_grad_rec);
        hipLaunchKernelGGL(k_gather2d, dim3((nwave + 3) / 4), dim3(256), 0, s, n, status, order, offsets, chunk_rank, partial, L.cap, carry, rec);
        if (g2.mean2d != nullptr)      // else the caller goes on from the records, pieces included (launch_preprocess2d_bwd_records)
            hipLaunchKernelGGL(k_grad_records_to_planes2d, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n,
                               reinterpret_cast<const uint32_t*>(ws + L.off_touched), rec, carry_fold(L, ws), g2);
    }
    return hipGetLastError();
}

hipError_t launch_render_stats2d(const CamDev& cam, const Layout& L, char* ws, uint64_t* counters, hipStream_t s)
{
    ProfScope prof(kKStats, s);
    hipLaunchKernelGGL(k_zero_counters2d, dim3(1), dim3(64), 0, s, reinterpret_cast<unsigned long long*>(counters));
    hipLaunchKernelGGL(k_render_stats2d, dim3((unsigned)(cam.TX * cam.TY)), dim3(256), 0, s, cam,
                       reinterpret_cast<const uint32_t*>(ws + L.off_ranges), reinterpret_cast<const uint32_t*>(ws + L.off_tile_order),
                       reinterpret_cast<const uint32_t*>(ws + L.off_vals),
                       reinterpret_cast<const Packed2D*>(ws + L.off_packed), reinterpret_cast<unsigned long long*>(counters));
    return hipGetLastError();
}

}  // namespace pbdr
