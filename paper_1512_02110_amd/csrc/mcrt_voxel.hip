// Voxelised forward model of Sec. 3, deterministic part, in FP64: the
// transmittance T_c(k) from every voxel centre to every camera (Eqs.
// taoKtoc, Tck), the images i_c = Pi_c (j_c . beta . T_c) with n x n
// sub-pixel rays (Eqs. IcP, PIc, Icpixel), and the gradient of a loss of
// those images with j frozen (Eqs. Jaco1, TcofJaco1, DivTc):
//   grad(m) = sum_c [ T_c(m) j_c(m) B_c(m)
//                     - sum_k D_c(k, m) T_c(k) beta(k) j_c(k) B_c(k) ],
// B_c = Pi_c^T dL/di_c, D_c(k, m) the length in voxel m of the line of sight
// from the centre of voxel k to camera c.
//
// T (k_vox_transmittance) and the images (k_vox_project) are ray walks that
// gather.  B and the gradient scatter along rays that all meet at the camera:
// as device atomics (past the L2, one line at a time) they took 3.9 + 2.6 ms
// on the 64^3 grid with 9 cameras of 128^2 pixels and 2 x 2 rays.  So B is
// gathered instead: every voxel sums over the rays of its footprint on the
// image (k_vox_gather), except in a small box around each camera, where the
// footprints grow to the whole image and the rays are walked into an LDS copy
// of the box (k_vox_near); and the lines of sight are walked by tiles of
// voxels into an LDS copy of the beam from the tile to the camera
// (k_vox_los_adjoint).  Only voxels with j != 0 that some ray of the camera
// can cross take part: T, B and the adjoint lines of the others only ever
// multiply zero.
#include <algorithm>
#include <cmath>

#include "mcrt_internal.hpp"

namespace mcrt {
namespace {

constexpr int VOX_BLOCK = 256;

// One axis of a walk: the crossings are t0 + n dt for n = 0, 1, ... (one
// fused multiply-add, so that nothing accumulates), the last of them, the exit
// of the box, the same expression at its n: a walk ends at the box without
// testing its indices.
struct WalkAxis64 {
    double t0, dt, n;
    int i, s;
};

// Clip of [t0, t1] to the slab of faces lo, hi; false when a segment along the
// faces lies outside it.
__device__ __forceinline__ bool axis_clip(double p, double v, double iv, double d, int lo, int hi, double& t0,
                                          double& t1) {
    if (v == 0.0) return !(p < lo * d || p > hi * d);
    const double ta = __fma_rn((double)lo, d, -p) * iv, tb = __fma_rn((double)hi, d, -p) * iv;
    t0 = fmax(t0, fmin(ta, tb));
    t1 = fmin(t1, fmax(ta, tb));
    return true;
}

// The voxel of the entry point at t (a point on a face belongs to the voxel on
// the side the segment moves into) and the crossings from there; t1 becomes
// the exit of the box where that is earlier.
__device__ __forceinline__ void axis_begin(WalkAxis64& a, double p, double v, double iv, double d, double t, int lo,
                                           int hi, double& t1) {
    const double x = (p + t * v) / d;
    const double fl = floor(x);
    int i = (int)fl;
    if (v < 0.0 && x == fl) i -= 1;
    i = i < lo ? lo : (i > hi - 1 ? hi - 1 : i);
    a.i = i;
    a.s = v > 0.0 ? 1 : (v < 0.0 ? -1 : 0);
    a.n = 0.0;
    a.t0 = INFINITY;
    a.dt = 0.0;
    if (a.s != 0) {
        a.t0 = __fma_rn((double)(i + (a.s > 0 ? 1 : 0)), d, -p) * iv;
        a.dt = fabs(d * iv);
        t1 = fmin(t1, __fma_rn((double)(a.s > 0 ? hi - 1 - i : i - lo), a.dt, a.t0));
    }
}

struct Box {
    int x0, y0, z0, x1, y1, z1;  // voxels [x0, x1) x ...
};

// The voxels of a segment p + t v, t in [0, tmax] (v unit), that lie in a box,
// in order.  The segment is clipped to the box first; ties between axes go to
// the lowest axis.  Every choice between axes is a select of plain registers:
// the state as arrays indexed by the axis lives in scratch memory, and with it
// and a division per crossing the transmittances of 127 x 90 x 77 voxels to 16
// cameras took 5.2 ms.  About 25 instructions a step.
struct SegWalk {
    WalkAxis64 X, Y, Z;
    double t, t1, tx, ty, tz;
    int k, kx, ky, kz;

    // false: no voxel
    __device__ __forceinline__ bool begin(const VoxArgs& A, const Box& b, double px, double py, double pz, double vx,
                                          double vy, double vz, double tmax) {
        const double ivx = 1.0 / vx, ivy = 1.0 / vy, ivz = 1.0 / vz;
        double t0 = 0.0;
        t1 = tmax;
        if (!axis_clip(px, vx, ivx, A.dx, b.x0, b.x1, t0, t1)) return false;
        if (!axis_clip(py, vy, ivy, A.dy, b.y0, b.y1, t0, t1)) return false;
        if (!axis_clip(pz, vz, ivz, A.dz, b.z0, b.z1, t0, t1)) return false;
        if (!(t1 > t0)) return false;
        axis_begin(X, px, vx, ivx, A.dx, t0, b.x0, b.x1, t1);
        axis_begin(Y, py, vy, ivy, A.dy, t0, b.y0, b.y1, t1);
        axis_begin(Z, pz, vz, ivz, A.dz, t0, b.z0, b.z1, t1);
        const int nxy = A.nx * A.ny;
        k = X.i + A.nx * Y.i + nxy * Z.i;
        kx = X.s;
        ky = Y.s * A.nx;
        kz = Z.s * nxy;
        t = t0;
        tx = X.t0;
        ty = Y.t0;
        tz = Z.t0;
        return true;
    }
    // The length in voxel k, then k moves on; false when it was the last one.
    template <bool IJK>
    __device__ __forceinline__ bool step(int n_vox, double& l) {
        const double tn = fmin(tx, fmin(ty, tz));
        const double end = t1;  // values: a select of fields would select addresses
        const int dkx = kx, dky = ky, dkz = kz, sx = X.s, sy = Y.s, sz = Z.s;
        const bool last = !(tn < end);
        l = (last ? end : tn) - t;
        t = tn;
        const bool cx = tx == tn;
        const bool cy = !cx && ty == tn;
        const bool cz = !cx && !cy;
        k += cx ? dkx : (cy ? dky : dkz);
        if constexpr (IJK) {
            X.i += cx ? sx : 0;
            Y.i += cy ? sy : 0;
            Z.i += cz ? sz : 0;
        }
        X.n += cx ? 1.0 : 0.0;
        Y.n += cy ? 1.0 : 0.0;
        Z.n += cz ? 1.0 : 0.0;
        tx = __fma_rn(X.n, X.dt, X.t0);
        ty = __fma_rn(Y.n, Y.dt, Y.t0);
        tz = __fma_rn(Z.n, Z.dt, Z.t0);
        // (no crossing of the box's end comes before t1: the index test only
        // ends segments of non-finite numbers)
        return !last && (unsigned)k < (unsigned)n_vox;
    }
};

// f(linear index, ix, iy, iz, length inside) of the segment's voxels.
template <typename F>
__device__ __forceinline__ void seg_walk(const VoxArgs& A, const Box& b, double px, double py, double pz, double vx,
                                         double vy, double vz, double tmax, F&& f) {
    SegWalk W;
    if (!W.begin(A, b, px, py, pz, vx, vy, vz, tmax)) return;
    for (bool on = true; on;) {
        const int k = W.k, ix = W.X.i, iy = W.Y.i, iz = W.Z.i;
        double l;
        on = W.step<true>((int)A.n_vox, l);
        f(k, ix, iy, iz, l);
    }
}

// sum + the lengths of the segment's voxels times x[voxel], added in order.
// The fetches bound it, so the walk runs SEG_AHEAD voxels at a time: while
// the next ones are found, those of the last batch arrive (a batch's terms are
// added one batch later; the lanes whose segment has ended step on, reading
// voxel 0 and adding nothing).  Against one voxel ahead, with registers for
// six wavefronts a SIMD instead of four: images of 64^3, 9 cameras 70 us (91),
// of 127 x 90 x 77, 16 cameras 165 (188), transmittances 113 (114) and 335
// (354).  Two and four voxels ahead are within 3%.
constexpr int SEG_AHEAD = 3;

__device__ __forceinline__ double seg_sum(const VoxArgs& A, const Box& b, double px, double py, double pz, double vx,
                                          double vy, double vz, double tmax, const double* x, double sum) {
    SegWalk W;
    if (!W.begin(A, b, px, py, pz, vx, vy, vz, tmax)) return sum;
    double xa[SEG_AHEAD], la[SEG_AHEAD], xb[SEG_AHEAD], lb[SEG_AHEAD];
    bool on = true;
    auto fetch = [&](double (&xs)[SEG_AHEAD], double (&ls)[SEG_AHEAD]) {
        for (int i = 0; i < SEG_AHEAD; ++i) {
            const int k = W.k;
            xs[i] = x[on ? k : 0];
            const bool more = W.step<false>((int)A.n_vox, ls[i]);
            ls[i] = on ? ls[i] : -INFINITY;  // (no length of a voxel)
            on = on && more;
        }
    };
    auto add = [&](const double (&xs)[SEG_AHEAD], const double (&ls)[SEG_AHEAD]) {
        for (int i = 0; i < SEG_AHEAD; ++i) {
            const double s = sum + xs[i] * ls[i];
            sum = ls[i] == -INFINITY ? sum : s;
        }
    };
    fetch(xa, la);
    for (;;) {
        if (!on) {
            add(xa, la);
            return sum;
        }
        fetch(xb, lb);
        add(xa, la);
        if (!on) {
            add(xb, lb);
            return sum;
        }
        fetch(xa, la);
        add(xb, lb);
    }
}

__device__ __forceinline__ Box domain(const VoxArgs& A) { return Box{0, 0, 0, A.nx, A.ny, A.nz}; }

__device__ __forceinline__ int64_t voxel_index(const VoxArgs& A, int ix, int iy, int iz) {
    return ix + (int64_t)A.nx * (iy + (int64_t)A.ny * iz);
}

// Line of sight from the centre of voxel (ix, iy, iz) to the camera: its
// voxels in the domain (seg_walk), or their sum of beta times length.
template <typename F>
__device__ __forceinline__ void sight(const VoxArgs& A, const HostCam& cam, int ix, int iy, int iz, F&& f) {
    const double x = (ix + 0.5) * A.dx, y = (iy + 0.5) * A.dy, z = (iz + 0.5) * A.dz;
    const double Dx = cam.pos[0] - x, Dy = cam.pos[1] - y, Dz = cam.pos[2] - z;
    const double len = sqrt(Dx * Dx + Dy * Dy + Dz * Dz);
    if (len > 0.0) f(x, y, z, Dx / len, Dy / len, Dz / len, len);
}

template <typename F>
__device__ __forceinline__ void sight_walk(const VoxArgs& A, const HostCam& cam, int ix, int iy, int iz, F&& f) {
    sight(A, cam, ix, iy, iz, [&](double x, double y, double z, double vx, double vy, double vz, double len) {
        seg_walk(A, domain(A), x, y, z, vx, vy, vz, len, f);
    });
}

__device__ __forceinline__ double sight_depth(const VoxArgs& A, const HostCam& cam, int ix, int iy, int iz) {
    double tau = 0.0;
    sight(A, cam, ix, iy, iz, [&](double x, double y, double z, double vx, double vy, double vz, double len) {
        tau = seg_sum(A, domain(A), x, y, z, vx, vy, vz, len, A.beta, 0.0);
    });
    return tau;
}

// Camera of global pixel p (the last camera whose first pixel is <= p).
__device__ int camera_of_pixel(const VoxArgs& A, int64_t p) {
    int lo = 0, hi = A.n_cams - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (A.cams[mid].pix_off <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Direction (unnormalised) of the ray through the image point (u, v),
// back-projected (world = R^T camera).
__device__ __forceinline__ void image_dir(const HostCam& c, double u, double v, double& vx, double& vy, double& vz) {
    const double qx = (u - c.cx) / c.fx;
    const double qy = (v - c.cy) / c.fy;
    vx = c.R[0] * qx + c.R[3] * qy + c.R[6];
    vy = c.R[1] * qx + c.R[4] * qy + c.R[7];
    vz = c.R[2] * qx + c.R[5] * qy + c.R[8];
}

// Unit direction of sub-pixel ray (a, b) of pixel (row, col): through the
// image point (col + (a + 1/2)/n, row + (b + 1/2)/n).
__device__ __forceinline__ void subpixel_dir(const HostCam& c, int row, int col, int a, int b, int n, double& vx,
                                             double& vy, double& vz) {
    image_dir(c, (double)col + (a + 0.5) / n, (double)row + (b + 0.5) / n, vx, vy, vz);
    const double il = 1.0 / sqrt(vx * vx + vy * vy + vz * vz);
    vx *= il;
    vy *= il;
    vz *= il;
}

__global__ void k_vox_cams(CamChunk chunk, HostCam* dev, VoxRect* dl_box) {
    const int i = threadIdx.x;
    if (i >= chunk.n) return;
    dev[chunk.first + i] = chunk.c[i];
    if (dl_box) dl_box[chunk.first + i] = VoxRect{INFINITY, INFINITY, 0.0, 0.0};
}

// Extends the camera's rectangle of pixels with dl != 0 by block b of nb's
// share of its image: one atomic a side and block (with one a wavefront, and
// four pixels a thread, the last of them arrived 40 us after an image of 512^2
// was read).  Numbers that are not negative order like their bit patterns.
__device__ void vox_dl_box(const VoxArgs& A, int c, int b, int nb, int* s_box) {
    const HostCam& cam = A.cams[c];
    const int64_t n = (int64_t)cam.width * cam.height;
    const int64_t lo = n * b / nb, hi = n * (b + 1) / nb;
    if (threadIdx.x < 4) s_box[threadIdx.x] = threadIdx.x < 2 ? 0x7fffffff : -1;
    __syncthreads();
    int c0 = 0x7fffffff, r0 = 0x7fffffff, c1 = -1, r1 = -1;
#pragma unroll 4
    for (int64_t p = lo + threadIdx.x; p < hi; p += VOX_BLOCK) {
        const bool on = !(A.dl[cam.pix_off + p] == 0.0);
        const int row = (int)((uint32_t)p / (uint32_t)cam.width), col = (int)p - row * cam.width;
        c0 = on ? min(c0, col) : c0;
        r0 = on ? min(r0, row) : r0;
        c1 = on ? max(c1, col) : c1;
        r1 = on ? max(r1, row) : r1;
    }
    if (c1 >= 0) {
        atomicMin(s_box, c0);
        atomicMin(s_box + 1, r0);
        atomicMax(s_box + 2, c1);
        atomicMax(s_box + 3, r1);
    }
    __syncthreads();
    if (threadIdx.x < 4 && s_box[2] >= 0) {
        const double s = (double)A.n_side, x = s * s_box[threadIdx.x];
        unsigned long long* side = reinterpret_cast<unsigned long long*>(A.dl_box + c) + threadIdx.x;
        if (threadIdx.x < 2) atomicMin(side, (unsigned long long)__double_as_longlong(x));
        else atomicMax(side, (unsigned long long)__double_as_longlong(x + (s - 1.0)));
    }
    __syncthreads();
}

// What the gather needs of each camera: M, the map from world to camera axes
// that inverts the rays' back-projection R^T (R itself for a rotation), the
// longest ray direction of the image, and the near box.  A camera without
// such a map (a singular or badly conditioned R, which the rays do not need)
// has ok = 0 and an empty near box: its rays are walked with device atomics.
__global__ void k_vox_views(VoxArgs A, VoxView* views) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= A.n_cams) return;
    const HostCam& cam = A.cams[c];
    const double* R = cam.R;
    VoxView V;
    // cofactors: M = (R^T)^-1 = cof(R) / det(R)
    double C[9];
    C[0] = R[4] * R[8] - R[5] * R[7];
    C[1] = R[5] * R[6] - R[3] * R[8];
    C[2] = R[3] * R[7] - R[4] * R[6];
    C[3] = R[2] * R[7] - R[1] * R[8];
    C[4] = R[0] * R[8] - R[2] * R[6];
    C[5] = R[1] * R[6] - R[0] * R[7];
    C[6] = R[1] * R[5] - R[2] * R[4];
    C[7] = R[2] * R[3] - R[0] * R[5];
    C[8] = R[0] * R[4] - R[1] * R[3];
    const double det = R[0] * C[0] + R[1] * C[1] + R[2] * C[2];
    double off = 0.0;
    for (int i = 0; i < 9; ++i) V.M[i] = C[i] / det;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            // (M R^T)(i, j) = sum_k M(i, k) R(j, k)
            const double e = V.M[3 * i] * R[3 * j] + V.M[3 * i + 1] * R[3 * j + 1] + V.M[3 * i + 2] * R[3 * j + 2];
            off = fmax(off, fabs(e - (i == j ? 1.0 : 0.0)));
            if (!isfinite(e)) off = INFINITY;
        }
    // |v| is convex over the image: its largest value is at a corner
    double far2 = 0.0;
    for (int k = 0; k < 4; ++k) {
        double vx, vy, vz;
        image_dir(cam, k & 1 ? cam.width : 0, k & 2 ? cam.height : 0, vx, vy, vz);
        far2 = fmax(far2, vx * vx + vy * vy + vz * vz);
    }
    V.inv_far = 1.0 / sqrt(far2);
    V.ok = off < 1e-12 && far2 > 0.0 && isfinite(far2) && V.inv_far > 0.0;
    const double p[3] = {cam.pos[0] / A.dx, cam.pos[1] / A.dy, cam.pos[2] / A.dz};
    const int n[3] = {A.nx, A.ny, A.nz};
    for (int a = 0; a < 3; ++a) {
        const double lo = floor(p[a]) - VOX_NEAR, hi = floor(p[a]) + VOX_NEAR + 1;
        V.lo[a] = V.ok ? (int)fmin(fmax(lo, 0.0), (double)n[a]) : 0;
        V.hi[a] = V.ok ? (int)fmin(fmax(hi, 0.0), (double)n[a]) : 0;
    }
    for (int a = 0; a < 3; ++a) {
        // the walks' own reading of where the camera stands
        const double len = n[a] * (a == 0 ? A.dx : (a == 1 ? A.dy : A.dz)), fl = floor(p[a]);
        V.on_face[a] = p[a] == fl;
        V.at[a] = p[a];
        V.cell[a] = cam.pos[a] < 0.0 || cam.pos[a] > len ? -1 : (int)fmin(fmax(fl, 0.0), (double)(n[a] - 1));
    }
    for (int a = 0; a < 3; ++a)
        if (V.lo[a] >= V.hi[a]) V.lo[0] = V.hi[0] = V.lo[1] = V.hi[1] = V.lo[2] = V.hi[2] = 0;
    views[c] = V;
}

__device__ __forceinline__ bool in_near(const VoxView& V, int ix, int iy, int iz) {
    return ix >= V.lo[0] && ix < V.hi[0] && iy >= V.lo[1] && iy < V.hi[1] && iz >= V.lo[2] && iz < V.hi[2];
}

__device__ __forceinline__ VoxRect whole_image(const VoxArgs& A, const HostCam& cam) {
    return VoxRect{0.0, 0.0, (double)A.n_side * cam.width - 1.0, (double)A.n_side * cam.height - 1.0};
}

// Sub-pixel columns s0 .. s1 and rows r0 .. r1 (as whole doubles) of the
// rectangle F of the image whose rays can cross the voxel, which lies outside
// the near box; false when there are none.  The box of the voxel in camera axes, q = M X as intervals; a point of
// the view at distance r has qz >= r / |v|max, which keeps the ratios finite
// where the box reaches behind the camera.  (Conservative: a ray of the range
// that misses the voxel adds no length.)
__device__ __forceinline__ bool footprint(const VoxArgs& A, const HostCam& cam, const VoxView& V, const VoxRect& F,
                                          int ix, int iy, int iz, double& s0, double& s1, double& r0, double& r1) {
    const double hx = 0.5 * A.dx, hy = 0.5 * A.dy, hz = 0.5 * A.dz;
    const double x = (ix + 0.5) * A.dx - cam.pos[0], y = (iy + 0.5) * A.dy - cam.pos[1],
                 z = (iz + 0.5) * A.dz - cam.pos[2];
    const double ex = fmax(fabs(x) - hx, 0.0), ey = fmax(fabs(y) - hy, 0.0), ez = fmax(fabs(z) - hz, 0.0);
    const double zmin = sqrt(ex * ex + ey * ey + ez * ez) * V.inv_far * (1.0 - 1e-9);
    const double qz = V.M[6] * x + V.M[7] * y + V.M[8] * z;
    const double wz = fabs(V.M[6]) * hx + fabs(V.M[7]) * hy + fabs(V.M[8]) * hz;
    if (!(qz + wz > zmin)) return false;
    const double i0 = 1.0 / fmax(qz - wz, zmin), i1 = 1.0 / (qz + wz);
    const double n = (double)A.n_side;
    const double qx = V.M[0] * x + V.M[1] * y + V.M[2] * z;
    const double wx = fabs(V.M[0]) * hx + fabs(V.M[1]) * hy + fabs(V.M[2]) * hz;
    const double xa = qx - wx, xb = qx + wx;
    const double u0 = n * (cam.cx + cam.fx * (xa * (xa < 0.0 ? i0 : i1))) - 0.5;
    const double u1 = n * (cam.cx + cam.fx * (xb * (xb > 0.0 ? i0 : i1))) - 0.5;
    s0 = fmax(ceil(u0 - 1e-3 - 1e-9 * fabs(u0)), F.s0);
    s1 = fmin(floor(u1 + 1e-3 + 1e-9 * fabs(u1)), F.s1);
    if (!(s0 <= s1)) return false;
    const double qy = V.M[3] * x + V.M[4] * y + V.M[5] * z;
    const double wy = fabs(V.M[3]) * hx + fabs(V.M[4]) * hy + fabs(V.M[5]) * hz;
    const double ya = qy - wy, yb = qy + wy;
    const double v0 = n * (cam.cy + cam.fy * (ya * (ya < 0.0 ? i0 : i1))) - 0.5;
    const double v1 = n * (cam.cy + cam.fy * (yb * (yb > 0.0 ? i0 : i1))) - 0.5;
    r0 = fmax(ceil(v0 - 1e-3 - 1e-9 * fabs(v0)), F.r0);
    r1 = fmin(floor(v1 + 1e-3 + 1e-9 * fabs(v1)), F.r1);
    return r0 <= r1;
}

// A block takes VOX_CHUNK voxels of a camera, consecutive or (SPREAD) in runs
// of 64 spread over the whole grid: the voxels next to a camera hold most of
// its rays, and a block of consecutive ones there runs on alone.  (512 or 256
// voxels: the lists get too short, the gather 7-33% slower.)  Voxel of the
// block's offset o:
constexpr int VOX_CHUNK = 1024;

template <bool SPREAD>
__device__ __forceinline__ int64_t chunk_voxel(int o) {
    return SPREAD ? ((int64_t)(o >> 6) * gridDim.x + blockIdx.x) * 64 + (o & 63)
                  : (int64_t)blockIdx.x * VOX_CHUNK + o;
}

// The block's voxels that `take` accepts, as offsets in its LDS list (in no
// particular order): the lines that are walked are then dense in the lanes,
// where a third of the voxels hold cloud and a camera sees a part of them.
template <bool SPREAD, typename P>
__device__ __forceinline__ int list_voxels(const VoxArgs& A, uint16_t* s_list, int* s_n, P&& take) {
    if (threadIdx.x == 0) *s_n = 0;
    __syncthreads();
    for (int o = threadIdx.x; o < VOX_CHUNK; o += VOX_BLOCK) {
        const int64_t k = chunk_voxel<SPREAD>(o);
        const bool in = k < A.n_vox && take((int)k);
        const unsigned long long m = __ballot(in);
        int base = 0;
        if (m && __lane_id() == 0) base = atomicAdd(s_n, __popcll(m));
        base = __shfl(base, 0);
        if (in) s_list[base + __popcll(m & __lanemask_lt())] = (uint16_t)o;
    }
    __syncthreads();
    return *s_n;
}

__device__ __forceinline__ void voxel_of(const VoxArgs& A, int k, int& ix, int& iy, int& iz) {
    ix = k % A.nx;
    const int r = k / A.nx;
    iy = r % A.ny;
    iz = r / A.ny;
}

// Some ray of the camera can cross the voxel.
__device__ __forceinline__ bool visible(const VoxArgs& A, const HostCam& cam, const VoxView& V, int k) {
    int ix, iy, iz;
    double s0, s1, r0, r1;
    voxel_of(A, k, ix, iy, iz);
    return !V.ok || in_near(V, ix, iy, iz) ||
           footprint(A, cam, V, whole_image(A, cam), ix, iy, iz, s0, s1, r0, r1);
}

// T_c(k) (Eqs. taoKtoc, Tck) of the voxels with j != 0 that the camera's rays
// can cross, and for the images T j beta (src); the other voxels get 0, which
// is what they contribute.  Bound by the gathers of beta: the block's voxels
// are spread over the grid (shorter last lines) while beta fits an XCD's 4 MB
// of L2, and consecutive past it (64^3, 9 cameras: 113 us spread, 143
// consecutive; 127 x 90 x 77, 16 cameras: 480 and 335).
template <bool SPREAD>
__global__ void __launch_bounds__(VOX_BLOCK, 4) k_vox_transmittance(VoxArgs A) {
    __shared__ uint16_t s_list[VOX_CHUNK];
    __shared__ int s_n;
    for (int c = blockIdx.y; c < A.n_cams; c += gridDim.y) {
        const HostCam& cam = A.cams[c];
        const VoxView& V = A.views[c];
        const int64_t off = (int64_t)c * A.n_vox;
        const int n = list_voxels<SPREAD>(A, s_list, &s_n, [&](int k) {
            const bool on = A.j[off + k] != 0.0 && visible(A, cam, V, k);
            if (!on && A.T) A.T[off + k] = 0.0;
            if (!on && A.src) A.src[off + k] = 0.0;
            return on;
        });
        for (int e = threadIdx.x; e < n; e += VOX_BLOCK) {
            const int k = (int)chunk_voxel<SPREAD>(s_list[e]);
            int ix, iy, iz;
            voxel_of(A, k, ix, iy, iz);
            const double T = exp(-sight_depth(A, cam, ix, iy, iz));
            if (A.T) A.T[off + k] = T;
            if (A.src) A.src[off + k] = A.j[off + k] * A.beta[k] * T;
        }
        __syncthreads();
    }
}

// i_c(p) = 1/(n^2 V) sum_rho sum_k l_rho(k) src_c(k), src = j beta T.  One
// lane per sub-pixel ray (tpp lanes a pixel, at most a block's), summed in LDS:
// with one lane per pixel the images of 9 cameras of 128^2 pixels were two
// wavefronts a SIMD (64^3, 2 x 2 rays: 92 us, 270 before; 70 with seg_sum).
__global__ void __launch_bounds__(VOX_BLOCK, 4) k_vox_project(VoxArgs A) {
    __shared__ double s_acc[VOX_BLOCK];
    const double scale = 1.0 / ((double)A.n_side * A.n_side * A.dx * A.dy * A.dz);
    const int n2 = A.n_side * A.n_side;
    const int tpp = n2 < VOX_BLOCK ? n2 : VOX_BLOCK;
    const int per = VOX_BLOCK / tpp;
    const int slot = threadIdx.x / tpp, sub = threadIdx.x % tpp;
    for (int64_t p0 = (int64_t)blockIdx.x * per; p0 < A.n_pix; p0 += (int64_t)gridDim.x * per) {
        const int64_t p = p0 + slot;
        const bool in = slot < per && p < A.n_pix;
        double acc = 0.0;
        if (in) {
            const int c = camera_of_pixel(A, p);
            const HostCam& cam = A.cams[c];
            const int64_t lp = p - cam.pix_off;
            const int row = (int)(lp / cam.width), col = (int)(lp % cam.width);
            const double* src = A.src + (int64_t)c * A.n_vox;
            for (int r = sub; r < n2; r += tpp) {
                double vx, vy, vz;
                subpixel_dir(cam, row, col, r % A.n_side, r / A.n_side, A.n_side, vx, vy, vz);
                acc = seg_sum(A, domain(A), cam.pos[0], cam.pos[1], cam.pos[2], vx, vy, vz, INFINITY, src, acc);
            }
        }
        s_acc[threadIdx.x] = acc;
        __syncthreads();
        if (in && sub == 0) {
            for (int i = 1; i < tpp; ++i) acc += s_acc[threadIdx.x + i];
            A.images[p] = acc * scale;
        }
        __syncthreads();
    }
}

// Rays of the cameras inside their near boxes: B_c += g l (Pi^T dl), or, with
// COUNT, += 1 for every ray longer than eps in the voxel.  A block walks a
// range of one camera's rays and adds its LDS copy of the box at the end (the
// first voxels take every ray of the image, so device atomics would queue on
// them).  A camera without a view has its whole rays walked, with device
// atomics.  Blocks past the first n_near of a camera find the rectangle of its
// pixels with dl != 0 for the gather meanwhile (in the launch before this one
// they cost a gradient of 64^3 and 9 cameras 8 us).
template <bool COUNT>
__global__ void __launch_bounds__(VOX_BLOCK) k_vox_near(VoxArgs A, double* out, int n_near) {
    constexpr int W = 2 * VOX_NEAR + 1;
    __shared__ double s_b[W * W * W];
    __shared__ int s_box[4];
    const double scale = COUNT ? 1.0 : 1.0 / ((double)A.n_side * A.n_side * A.dx * A.dy * A.dz);
    const double eps = 1e-9 * fmin(A.dx, fmin(A.dy, A.dz));
    const int n = A.n_side, n2 = n * n;
    for (int c = blockIdx.y; c < A.n_cams; c += gridDim.y) {
        const HostCam& cam = A.cams[c];
        if (!COUNT && (int)blockIdx.x >= n_near) {
            vox_dl_box(A, c, (int)blockIdx.x - n_near, (int)gridDim.x - n_near, s_box);
            continue;
        }
        const VoxView V = A.views[c];
        double* Bc = out + (int64_t)c * A.n_vox;
        const Box box = V.ok ? Box{V.lo[0], V.lo[1], V.lo[2], V.hi[0], V.hi[1], V.hi[2]} : domain(A);
        if (box.x0 >= box.x1) continue;
        const int64_t rays = (int64_t)cam.width * cam.height * n2;
        if ((int64_t)blockIdx.x * VOX_BLOCK >= rays) continue;
        for (int i = threadIdx.x; i < W * W * W; i += VOX_BLOCK) s_b[i] = 0.0;
        __syncthreads();
        for (int64_t q = (int64_t)blockIdx.x * VOX_BLOCK + threadIdx.x; q < rays;
             q += (int64_t)n_near * VOX_BLOCK) {
            const int64_t lp = q / n2;
            const int r = (int)(q % n2);
            const double g = COUNT ? 1.0 : A.dl[cam.pix_off + lp] * scale;
            if (g == 0.0) continue;
            double vx, vy, vz;
            subpixel_dir(cam, (int)(lp / cam.width), (int)(lp % cam.width), r % n, r / n, n, vx, vy, vz);
            seg_walk(A, box, cam.pos[0], cam.pos[1], cam.pos[2], vx, vy, vz, INFINITY,
                           [&](int k, int ix, int iy, int iz, double l) {
                               if (COUNT && !(l > eps)) return;
                               const double x = COUNT ? 1.0 : g * l;
                               if (V.ok)
                                   atomicAdd(&s_b[(ix - box.x0) + W * ((iy - box.y0) + W * (iz - box.z0))], x);
                               else
                                   unsafeAtomicAdd(Bc + k, x);
                           });
        }
        __syncthreads();
        for (int i = threadIdx.x; V.ok && i < W * W * W; i += VOX_BLOCK) {
            const double x = s_b[i];
            if (x != 0.0)
                unsafeAtomicAdd(Bc + voxel_index(A, box.x0 + i % W, box.y0 + (i / W) % W, box.z0 + i / (W * W)), x);
        }
        __syncthreads();
    }
}

// A voxel's faces relative to the camera.  A ray along the faces of an axis
// runs through the voxels of one layer, the camera's (sx, sy, sz: this one).
// The faces of an axis on which the camera stands on a face are counted from
// that face, so that this one is at exactly 0 and a ray leaves it to the side
// that it moves into, as the walks have it, however small that motion is.
struct Slab {
    double x0, x1, y0, y1, z0, z1;
    bool sx, sy, sz;
};

__device__ __forceinline__ double face_from(const VoxView& V, int a, int i, double d, double p) {
    return V.on_face[a] ? ((double)i - V.at[a]) * d : __fma_rn((double)i, d, -p);
}

// 1/x to the last bit or two without the scaling of an IEEE division (x = 0
// is the callers').
__device__ __forceinline__ double fast_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __fma_rn(__fma_rn(-x, r, 1.0), r, r);
    return __fma_rn(__fma_rn(-x, r, 1.0), r, r);
}

__device__ __forceinline__ void slab_axis(double a0, double a1, bool same, double v, double& tin, double& tout) {
    const double iv = fast_rcp(v);
    const double ta = a0 * iv, tb = a1 * iv;
    const bool still = v == 0.0;
    tin = fmax(tin, still ? (same ? 0.0 : INFINITY) : fmin(ta, tb));
    tout = fmin(tout, still ? INFINITY : fmax(ta, tb));
}

// Length of the ray from the camera along (vx, vy, vz), not normalised, in the
// voxel: the overlap of its crossings of the three slabs.
__device__ __forceinline__ double slab_length(const Slab& B, double vx, double vy, double vz) {
    double tin = 0.0, tout = INFINITY;
    slab_axis(B.x0, B.x1, B.sx, vx, tin, tout);
    slab_axis(B.y0, B.y1, B.sy, vy, tin, tout);
    slab_axis(B.z0, B.z1, B.sz, vz, tin, tout);
    return tout > tin ? (tout - tin) * sqrt(vx * vx + vy * vy + vz * vz) : 0.0;
}

// B_c of the voxels outside the near box, gathered over the footprint of each
// on the image: a few rays a voxel far from the camera (one lane), hundreds
// next to the near box (a wavefront, 8 x 8 rays at a time).  No atomics, and
// the sum of a voxel does not depend on the launch.  Bound by instructions (the
// lanes' footprints differ) and the fetches of dl, each in flight while the
// next ray's length is found: 64^3, 9 cameras of 128^2, 2 x 2 rays 292 us (315
// with a wait for each) and the near pass's 58, against 3.86 ms of device
// atomics; 127 x 90 x 77, 16 cameras of 160 x 120 669 (757) + 84 us against
// 7.6 ms.  Wide images, whose voxels beside the camera see many rays that miss:
// gradients of 64^3 with 9 cameras of 110, 140, 160 and 175 degrees 0.88, 0.88,
// 0.90 and 0.94 ms, 7.5, 7.7, 6.6 and 4.8 with atomics.  (128 registers, for four
// wavefronts a SIMD, are ten too few: 44 bytes a lane spill.)
// COUNT: the number of rays longer than eps.  Otherwise B is used at once: grad(k) += q T j B, and B
// (scratch) becomes the weight w = T beta j B of the voxel's line of sight, and
// only the rays of the rectangle of the pixels with dl != 0 are looked at: a
// gradient of one pixel of 4 cameras of 512^2 (64^3 voxels) takes 0.19 ms, 1.39
// with every footprint and 0.47 with device atomics along that pixel's rays.
constexpr double VOX_LIGHT = 64.0;

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double x) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                            __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

template <bool COUNT>
__device__ __forceinline__ void voxel_done(const VoxArgs& A, double* out, int c, int k, double B) {
    const int64_t i = (int64_t)c * A.n_vox + k;
    if (COUNT) {
        out[i] = B;
        return;
    }
    const double bj = B * A.j[i];
    const double T = A.T[i];
    out[i] = bj == 0.0 ? 0.0 : T * A.beta[k] * bj;
    if (bj != 0.0) unsafeAtomicAdd(A.grad + k, (A.q ? A.q[i] : 1.0) * T * bj);
}

template <bool COUNT>
__global__ void __launch_bounds__(VOX_BLOCK, 4) k_vox_gather(VoxArgs A, double* out) {
    __shared__ uint16_t s_list[VOX_CHUNK], s_heavy[VOX_CHUNK];
    __shared__ double s_frac[64];
    __shared__ int s_n, s_nh;
    const double scale = 1.0 / ((double)A.n_side * A.n_side * A.dx * A.dy * A.dz);
    const double eps = 1e-9 * fmin(A.dx, fmin(A.dy, A.dz));
    const double n = (double)A.n_side, in = 1.0 / n;
    if (threadIdx.x < A.n_side) s_frac[threadIdx.x] = (threadIdx.x + 0.5) / n;
    for (int c = blockIdx.y; c < A.n_cams; c += gridDim.y) {
        const HostCam& cam = A.cams[c];
        const VoxView& V = A.views[c];
        const int64_t off = (int64_t)c * A.n_vox;
        const double* dl = A.dl + (COUNT ? 0 : cam.pix_off);
        const double ifx = 1.0 / cam.fx, ify = 1.0 / cam.fy;
        const VoxRect P = COUNT ? whole_image(A, cam) : A.dl_box[c];
        if (!COUNT && !(P.s0 <= P.s1)) continue;  // (dl is zero: so is B)
        const VoxRect F{uniform(P.s0), uniform(P.r0), uniform(P.s1), uniform(P.r1)};
        if (threadIdx.x == 0) s_nh = 0;
        const int n_list = list_voxels<true>(A, s_list, &s_n, [&](int k) {
            if (!COUNT && !(A.j[off + k] != 0.0)) {
                out[off + k] = 0.0;  // (the near pass may have added to it)
                return false;
            }
            int ix, iy, iz;
            voxel_of(A, k, ix, iy, iz);
            if (!V.ok || in_near(V, ix, iy, iz)) {
                // accumulated by the near pass
                if (!COUNT) voxel_done<COUNT>(A, out, c, k, out[off + k]);
                return false;
            }
            double s0, s1, r0, r1;
            return footprint(A, cam, V, F, ix, iy, iz, s0, s1, r0, r1);
        });
        auto slab = [&](int ix, int iy, int iz) {
            return Slab{face_from(V, 0, ix, A.dx, cam.pos[0]), face_from(V, 0, ix + 1, A.dx, cam.pos[0]),
                        face_from(V, 1, iy, A.dy, cam.pos[1]), face_from(V, 1, iy + 1, A.dy, cam.pos[1]),
                        face_from(V, 2, iz, A.dz, cam.pos[2]), face_from(V, 2, iz + 1, A.dz, cam.pos[2]),
                        ix == V.cell[0], iy == V.cell[1], iz == V.cell[2]};
        };
        // sum over the rays (s, r) of the range, strided
        auto gather = [&](const Slab& B, double s0, double s1, double r0, double r1, double step) {
            double acc = 0.0, dp = 0.0, lp = 0.0;
            for (double r = r0; r <= r1; r += step) {
                const double row = floor((r + 0.5) * in);
                const double qy = (row + s_frac[(int)(r - row * n)] - cam.cy) * ify;
                const double ox = __fma_rn(cam.R[3], qy, cam.R[6]), oy = __fma_rn(cam.R[4], qy, cam.R[7]),
                             oz = __fma_rn(cam.R[5], qy, cam.R[8]);
                for (double s = s0; s <= s1; s += step) {
                    const double col = floor((s + 0.5) * in);
                    const double qx = (col + s_frac[(int)(s - col * n)] - cam.cx) * ifx;
                    const double l = slab_length(B, __fma_rn(cam.R[0], qx, ox), __fma_rn(cam.R[1], qx, oy),
                                                 __fma_rn(cam.R[2], qx, oz));
                    if (COUNT) {
                        if (l > eps) acc += 1.0;
                    } else {
                        // (a ray's term is added when the next one's fetch is out)
                        const double x = acc + dp * scale * lp;
                        acc = lp > 0.0 ? x : acc;
                        dp = dl[(int)row * cam.width + (int)col];
                        lp = l;
                    }
                }
            }
            if (!COUNT && lp > 0.0) acc += dp * scale * lp;
            return acc;
        };
        for (int e = threadIdx.x; e < n_list; e += VOX_BLOCK) {
            const int k = (int)chunk_voxel<true>(s_list[e]);
            int ix, iy, iz;
            double s0, s1, r0, r1;
            voxel_of(A, k, ix, iy, iz);
            footprint(A, cam, V, F, ix, iy, iz, s0, s1, r0, r1);
            if ((s1 - s0 + 1.0) * (r1 - r0 + 1.0) > VOX_LIGHT) {
                s_heavy[atomicAdd(&s_nh, 1)] = s_list[e];
                continue;
            }
            voxel_done<COUNT>(A, out, c, k, gather(slab(ix, iy, iz), s0, s1, r0, r1, 1.0));
        }
        __syncthreads();
        const int lane = threadIdx.x & 63;
        for (int e = threadIdx.x >> 6; e < s_nh; e += VOX_BLOCK / 64) {
            const int k = (int)chunk_voxel<true>(s_heavy[e]);
            int ix, iy, iz;
            double s0, s1, r0, r1;
            voxel_of(A, k, ix, iy, iz);
            footprint(A, cam, V, F, ix, iy, iz, s0, s1, r0, r1);
            double acc = gather(slab(ix, iy, iz), s0 + (lane & 7), s1, r0 + (lane >> 3), r1, 8.0);
            for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
            if (lane == 0) voxel_done<COUNT>(A, out, c, k, acc);
        }
        __syncthreads();
    }
}

// The line of sight from the centre of k to the camera takes -w l (w = T beta
// j B of k, in A.B) in every voxel it crosses.  A block walks the lines of a
// tile of 8 x 8 x 8 voxels into an LDS copy of the beam from the tile to the
// camera: per slice of voxels along the beam's longest axis, the rectangle
// that the lines cross, which narrows from the tile to one voxel.  The beam
// is added to the gradient at the end, so that a device atomic stands for
// every voxel of the beam instead of every crossing of every line.  Bound by
// instructions and the blocks' barriers: 64^3, 9 cameras 240 us against 2.64 ms
// with an atomic per crossing, 127 x 90 x 77, 16 cameras 0.75 against 4.1 ms
// (275 us and 0.90 ms with a lane per rectangle and a division for each of its
// 16 ends, which all wavefronts of the block wait for).  Slices
// past the LDS copy's room, and a crossing that rounding puts outside its
// rectangle, go to the gradient directly.
constexpr int LOS_TILE = 8;
constexpr int LOS_BLOCK = LOS_TILE * LOS_TILE * LOS_TILE;
constexpr int LOS_SLICES = 256;
static_assert(2 * LOS_SLICES <= LOS_BLOCK, "two lanes a slice");
constexpr int LOS_CELLS = 4608;  // 36 KB: with the tables 41 KB, three blocks a CU (as many as 80 registers allow)

__global__ void __launch_bounds__(LOS_BLOCK, 6) k_vox_los_adjoint(VoxArgs A, int tx, int ty) {
    __shared__ double s_b[LOS_CELLS];
    __shared__ int4 s_sl[LOS_SLICES];  // a slice's rectangle: first u, first v, width (0: no room), first cell
    __shared__ int s_h[LOS_SLICES];    // and height
    __shared__ int s_any, s_cells;
    const int t = threadIdx.x;
    const int bx = (int)(blockIdx.x % tx) * LOS_TILE, by = (int)((blockIdx.x / tx) % ty) * LOS_TILE,
              bz = (int)(blockIdx.x / ((unsigned)tx * ty)) * LOS_TILE;
    const int l0 = t % LOS_TILE, l1 = (t / LOS_TILE) % LOS_TILE, l2 = t / (LOS_TILE * LOS_TILE);
    const int n[3] = {A.nx, A.ny, A.nz};
    const int lo[3] = {bx, by, bz};
    const int hi[3] = {min(bx + LOS_TILE, A.nx), min(by + LOS_TILE, A.ny), min(bz + LOS_TILE, A.nz)};
    for (int c = blockIdx.y; c < A.n_cams; c += gridDim.y) {
        const HostCam& cam = A.cams[c];
        // the camera in voxel units; the beam's axis a and the other two, u and v
        const double P[3] = {cam.pos[0] / A.dx, cam.pos[1] / A.dy, cam.pos[2] / A.dz};
        const double far_x = fabs(P[0] - 0.5 * (lo[0] + hi[0])), far_y = fabs(P[1] - 0.5 * (lo[1] + hi[1])),
                     far_z = fabs(P[2] - 0.5 * (lo[2] + hi[2]));
        const int a = far_z >= far_x && far_z >= far_y ? 2 : (far_y >= far_x ? 1 : 0);
        // the lanes of a wavefront span the beam's axis and one other, so that
        // at a step they stand in eight slices and fewer of them meet in one
        // voxel near the camera
        const int ix = bx + (a == 0 ? l0 : l1), iy = by + (a == 1 ? l0 : (a == 0 ? l1 : l2)),
                  iz = bz + (a == 2 ? l0 : l2);
        const bool in = ix < A.nx && iy < A.ny && iz < A.nz;
        const double w = in ? A.B[(int64_t)c * A.n_vox + voxel_index(A, ix, iy, iz)] : 0.0;
        if (t == 0) s_any = 0;
        __syncthreads();
        if (w != 0.0) s_any = 1;
        __syncthreads();
        if (!s_any) continue;
        // slices 0 .. n_s - 1: a0 + s, from the tile's first voxel or the
        // camera's, whichever is lower, nearest LOS_SLICES to the tile
        const double Pa = a == 0 ? P[0] : (a == 1 ? P[1] : P[2]);
        const int la = a == 0 ? lo[0] : (a == 1 ? lo[1] : lo[2]), ha = a == 0 ? hi[0] : (a == 1 ? hi[1] : hi[2]);
        const int na = a == 0 ? n[0] : (a == 1 ? n[1] : n[2]);
        const double fa = floor(Pa);
        int a0 = fa < la ? (int)fmax(fa, 0.0) : la;
        int a1 = fa >= ha ? (int)fmin(fa + 1.0, (double)na) : ha;
        if (a1 - a0 > LOS_SLICES) {
            if (a0 < la) a0 = a1 - LOS_SLICES;
            else a1 = a0 + LOS_SLICES;
        }
        const int n_s = a1 - a0;
        // two lanes a slice, one for each of the rectangle's sides (LOS_BLOCK
        // lanes for LOS_SLICES slices); the divisions by Pa - Xa once
        const bool level = Pa > la - 1.0 && Pa < ha + 1.0;
        const double X0 = la + 0.5, X1 = ha - 0.5;
        const double iv0 = level ? 0.0 : 1.0 / (Pa - X0), iv1 = level ? 0.0 : 1.0 / (Pa - X1);
        if (t < 2 * n_s) {
            const int s = t >> 1, d = t & 1;
            const int ax = d == 0 ? (a == 0 ? 1 : 0) : (a == 2 ? 1 : 2);
            const double Pd = ax == 0 ? P[0] : (ax == 1 ? P[1] : P[2]);
            const int ld = ax == 0 ? lo[0] : (ax == 1 ? lo[1] : lo[2]);
            const int hd = ax == 0 ? hi[0] : (ax == 1 ? hi[1] : hi[2]);
            const int nd = ax == 0 ? n[0] : (ax == 1 ? n[1] : n[2]);
            double m0 = INFINITY, m1 = -INFINITY;
            if (level) {
                // the camera is level with the tile: the hull of both
                m0 = fmin(ld + 0.5, Pd);
                m1 = fmax(hd - 0.5, Pd);
            } else {
                // the position X + (P - X)(z - Xa)/(Pa - Xa) is monotone
                // in X, Xa and z each: its extremes are at their ends
                for (int e = 0; e < 8; ++e) {
                    const double X = e & 1 ? hd - 0.5 : ld + 0.5;
                    const double z = a0 + s + (e & 4 ? 1 : 0);
                    const double f = fmin(fmax((z - (e & 2 ? X1 : X0)) * (e & 2 ? iv1 : iv0), 0.0), 1.0);
                    const double x = X + (Pd - X) * f;
                    m0 = fmin(m0, x);
                    m1 = fmax(m1, x);
                }
            }
            const int r0 = (int)fmin(fmax(floor(m0 - 1e-6), 0.0), (double)nd);
            const int r1 = (int)fmin(fmax(floor(m1 + 1e-6) + 1.0, 0.0), (double)nd);
            if (d == 0) {
                s_sl[s].x = r0;
                s_sl[s].z = max(r1 - r0, 0);
                s_sl[s].w = 0;
            } else {
                s_sl[s].y = r0;
                s_h[s] = max(r1 - r0, 0);
            }
        }
        __syncthreads();
        if (t < 64) {
            // first cells of the slices (four a lane): the slices in front of
            // the first one that does not fit get room
            int m[LOS_SLICES / 64], sum = 0;
            for (int i = 0; i < LOS_SLICES / 64; ++i) {
                const int s = t * (LOS_SLICES / 64) + i;
                m[i] = s < n_s ? (int)min((int64_t)s_sl[s].z * s_h[s], (int64_t)(LOS_CELLS + 1)) : 0;
                sum += m[i];
            }
            int end = sum;
            for (int o = 1; o < 64; o <<= 1) {
                const int x = __shfl_up(end, o);
                end += t >= o ? x : 0;
            }
            int o = end - sum, used = 0;
            for (int i = 0; i < LOS_SLICES / 64; ++i) {
                const int s = t * (LOS_SLICES / 64) + i;
                if (s < n_s) {
                    s_sl[s].w = o;
                    if (o + m[i] > LOS_CELLS) s_sl[s].z = s_h[s] = 0;
                    else used = o + m[i];
                }
                o += m[i];
            }
            for (int i = 32; i > 0; i >>= 1) used = max(used, __shfl_xor(used, i));
            if (t == 0) s_cells = used;
        }
        __syncthreads();
        const int cells = s_cells;
        for (int i = t; i < cells; i += LOS_BLOCK) s_b[i] = 0.0;
        __syncthreads();
        const double* qc = A.q ? A.q + (int64_t)c * A.n_vox : nullptr;
        if (w != 0.0)
            sight_walk(A, cam, ix, iy, iz, [&](int m, int jx, int jy, int jz, double l) {
                const int s = (a == 0 ? jx : (a == 1 ? jy : jz)) - a0;
                const int u = a == 0 ? jy : jx, v = a == 2 ? jy : jz;
                if ((unsigned)s < (unsigned)n_s) {
                    const int4 r = s_sl[s];
                    const int du = u - r.x, dv = v - r.y;
                    if ((unsigned)du < (unsigned)r.z && (unsigned)dv < (unsigned)s_h[s]) {
                        atomicAdd(&s_b[r.w + du + r.z * dv], w * l);
                        return;
                    }
                }
                unsafeAtomicAdd(A.grad + m, -(qc ? qc[m] : 1.0) * w * l);
            });
        __syncthreads();
        // a wavefront per slice: its cells in order of u
        for (int s = t >> 6; s < n_s; s += LOS_BLOCK / 64) {
            const int4 r = s_sl[s];
            const int m = r.z * s_h[s];
            for (int i = t & 63; i < m; i += 64) {
                const double x = s_b[r.w + i];
                if (x == 0.0) continue;
                const int u = r.x + i % r.z, v = r.y + i / r.z, z = a0 + s;
                const int64_t k = a == 0 ? voxel_index(A, z, u, v)
                                         : (a == 1 ? voxel_index(A, u, z, v) : voxel_index(A, u, v, z));
                unsafeAtomicAdd(A.grad + k, -(qc ? qc[k] : 1.0) * x);
            }
        }
        __syncthreads();
    }
}

// q = 1 / count where a ray passes, else 0 (in place).
__global__ void k_vox_invert(double* x, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = x[i] > 0.0 ? 1.0 / x[i] : 0.0;
}

// Block sum of v into *out (one device atomic per block).
__device__ void block_sum_add(double v, double* s_red, double* out) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) s_red[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += s_red[w];
        unsafeAtomicAdd(out, t);
    }
}

// 7-point Laplacian in voxel units at (ix, iy, iz); a neighbour outside the
// domain takes the centre's value (no flux through the boundary).
__device__ double lap_at(const double* f, int nx, int ny, int nz, int ix, int iy, int iz) {
    const int64_t nxy = (int64_t)nx * ny;
    const int64_t k = ix + (int64_t)nx * iy + nxy * iz;
    const double c = f[k];
    double s = -6.0 * c;
    s += ix > 0 ? f[k - 1] : c;
    s += ix < nx - 1 ? f[k + 1] : c;
    s += iy > 0 ? f[k - nx] : c;
    s += iy < ny - 1 ? f[k + nx] : c;
    s += iz > 0 ? f[k - nxy] : c;
    s += iz < nz - 1 ? f[k + nxy] : c;
    return s;
}

// Sec. 6, Psi = |W Lap beta|^2: r = W^2 Lap beta (scratch), *value += Psi.
__global__ void __launch_bounds__(VOX_BLOCK) k_reg_residual(int nx, int ny, int nz, const double* beta,
                                                            const double* w_layer, double* r, double* value) {
    __shared__ double s_red[VOX_BLOCK / 64];
    const int64_t n = (int64_t)nx * ny * nz, nxy = (int64_t)nx * ny;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const int ix = (int)(k % nx), iy = (int)((k / nx) % ny), iz = (int)(k / nxy);
        const double w = w_layer ? w_layer[iz] : 1.0;
        const double l = lap_at(beta, nx, ny, nz, ix, iy, iz);
        acc += (w * l) * (w * l);
        r[k] = w * w * l;
    }
    if (value) block_sum_add(acc, s_red, value);
}

// grad += eta * 2 Lap r (Lap is symmetric).
__global__ void __launch_bounds__(VOX_BLOCK) k_reg_grad(int nx, int ny, int nz, const double* r, double eta,
                                                        double* grad) {
    const int64_t n = (int64_t)nx * ny * nz, nxy = (int64_t)nx * ny;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const int ix = (int)(k % nx), iy = (int)((k / nx) % ny), iz = (int)(k / nxy);
        grad[k] += eta * 2.0 * lap_at(r, nx, ny, nz, ix, iy, iz);
    }
}

// Eq. (Cost) data term: r = M (i - measured); dl = 2 M r; *loss += sum r^2.
__global__ void __launch_bounds__(VOX_BLOCK) k_image_residual(int64_t n, const double* img, const double* meas,
                                                              const double* mask, double* dl, double* loss) {
    __shared__ double s_red[VOX_BLOCK / 64];
    double acc = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const double m = mask ? mask[p] : 1.0;
        const double r = m * (img[p] - meas[p]);
        acc += r * r;
        dl[p] = 2.0 * m * r;
    }
    if (loss) block_sum_add(acc, s_red, loss);
}

// Eq. (GD) projected on the non-negative set: beta = max(beta - delta g, 0).
__global__ void k_gd_step(int64_t n, double* beta, const double* g, double delta) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const double b = beta[k] - delta * g[k];
        beta[k] = b > 0.0 ? b : 0.0;
    }
}

// Largest masked pixel (values are >= 0: the bit pattern orders like the
// value, so an integer max does).
__global__ void __launch_bounds__(VOX_BLOCK) k_masked_max(int64_t n, const double* img, const double* mask,
                                                          unsigned long long* mx) {
    unsigned long long best = 0ull;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const double v = (mask ? mask[p] : 1.0) * img[p];
        if (v > 0.0) {
            const unsigned long long u = (unsigned long long)__double_as_longlong(v);
            best = u > best ? u : best;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long t = __shfl_down(best, o);
        best = t > best ? t : best;
    }
    if ((threadIdx.x & 63) == 0 && best) atomicMax(mx, best);
}

// Eq. (noise) with the caller's N(0,1) draws.
__global__ void k_camera_noise(int64_t n, const double* img, const double* normals,
                               const unsigned long long* mx, double* out, double* scale_out) {
    const double m = __longlong_as_double((long long)*mx);
    const double scale = m > 0.0 ? 1024.0 / m : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && scale_out) *scale_out = scale;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const double x = floor(img[p] * scale + 0.4 * normals[p] + 0.5);
        out[p] = x < 0.0 ? 0.0 : (x > 1024.0 ? 1024.0 : x);
    }
}

// Sec. 7: sums |b|, |t|, |b - t| into acc[0..2].
__global__ void __launch_bounds__(VOX_BLOCK) k_recovery_sums(int64_t n, const double* b, const double* t,
                                                             double* acc) {
    __shared__ double s_red[VOX_BLOCK / 64];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        a0 += fabs(b[k]);
        a1 += fabs(t[k]);
        a2 += fabs(b[k] - t[k]);
    }
    block_sum_add(a0, s_red, acc);
    __syncthreads();
    block_sum_add(a1, s_red, acc + 1);
    __syncthreads();
    block_sum_add(a2, s_red, acc + 2);
}

__global__ void k_d2f(int64_t n, const double* in, float* out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (float)in[i];
}

int grid_for(int64_t n) { return (int)((n + VOX_BLOCK - 1) / VOX_BLOCK < 65536 ? (n + VOX_BLOCK - 1) / VOX_BLOCK : 65536); }

}  // namespace

hipError_t launch_vox_cams(const CamChunk& chunk, HostCam* dev, VoxRect* dl_box, hipStream_t s) {
    hipLaunchKernelGGL(k_vox_cams, dim3(1), dim3(64), 0, s, chunk, dev, dl_box);
    return hipGetLastError();
}

// Grid of the kernels that take a range of voxels (or rays) and a camera.
static dim3 cam_grid(int64_t blocks, int n_cams) { return dim3((unsigned)(blocks > 0 ? blocks : 1), (unsigned)n_cams); }

static int64_t vox_chunks(const VoxArgs& a) { return (a.n_vox + VOX_CHUNK - 1) / VOX_CHUNK; }

hipError_t launch_vox_views(const VoxArgs& a, VoxView* views, hipStream_t s) {
    hipLaunchKernelGGL(k_vox_views, dim3((a.n_cams + 63) / 64), dim3(64), 0, s, a, views);
    return hipGetLastError();
}

hipError_t launch_vox_transmittance(const VoxArgs& a, hipStream_t s) {
    const dim3 grid = cam_grid(vox_chunks(a), a.n_cams);
    if (a.n_vox * (int64_t)sizeof(double) <= (int64_t)4 << 20)
        hipLaunchKernelGGL(k_vox_transmittance<true>, grid, dim3(VOX_BLOCK), 0, s, a);
    else
        hipLaunchKernelGGL(k_vox_transmittance<false>, grid, dim3(VOX_BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_vox_project(const VoxArgs& a, hipStream_t s) {
    const int64_t n2 = (int64_t)a.n_side * a.n_side;
    const int64_t per = VOX_BLOCK / (n2 < VOX_BLOCK ? n2 : VOX_BLOCK);
    if (a.n_pix > 0) {
        const int64_t blocks = (a.n_pix + per - 1) / per;
        hipLaunchKernelGGL(k_vox_project, dim3((unsigned)(blocks < 1048576 ? blocks : 1048576)), dim3(VOX_BLOCK), 0, s,
                           a);
    }
    return hipGetLastError();
}

// B (out, zeroed): near boxes, then the gather, which also turns B into the
// gradient's local term and the lines' weights (count: into the ray counts).
hipError_t launch_vox_backproject(const VoxArgs& a, double* out, bool count, int64_t max_pix, hipStream_t s) {
    // 8 rays a thread, so that a block's box is added once per 2048 rays, and 16 pixels a thread
    const auto blocks = [](int64_t n, int64_t per, int64_t most) { return std::min((n + per - 1) / per, most); };
    const int64_t near = blocks(max_pix * a.n_side * a.n_side, 8 * VOX_BLOCK, 4096);
    const int64_t n_box = blocks(max_pix, 16 * VOX_BLOCK, 1024);
    const dim3 g_far = cam_grid(vox_chunks(a), a.n_cams);
    if (count) {
        hipLaunchKernelGGL(k_vox_near<true>, cam_grid(near, a.n_cams), dim3(VOX_BLOCK), 0, s, a, out, (int)near);
        hipLaunchKernelGGL(k_vox_gather<true>, g_far, dim3(VOX_BLOCK), 0, s, a, out);
    } else {
        hipLaunchKernelGGL(k_vox_near<false>, cam_grid(near + n_box, a.n_cams), dim3(VOX_BLOCK), 0, s, a, out,
                           (int)near);
        hipLaunchKernelGGL(k_vox_gather<false>, g_far, dim3(VOX_BLOCK), 0, s, a, out);
    }
    return hipGetLastError();
}

hipError_t launch_vox_invert(double* x, int64_t n, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_vox_invert, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, x, n);
    return hipGetLastError();
}

hipError_t launch_reg(int nx, int ny, int nz, const double* beta, const double* w_layer, double eta, double* r,
                      double* grad, double* value, hipStream_t s) {
    const int64_t n = (int64_t)nx * ny * nz;
    hipLaunchKernelGGL(k_reg_residual, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, nx, ny, nz, beta, w_layer, r, value);
    if (grad) hipLaunchKernelGGL(k_reg_grad, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, nx, ny, nz, r, eta, grad);
    return hipGetLastError();
}

hipError_t launch_image_residual(int64_t n, const double* img, const double* meas, const double* mask, double* dl,
                                 double* loss, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_image_residual, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, n, img, meas, mask, dl, loss);
    return hipGetLastError();
}

hipError_t launch_gd_step(int64_t n, double* beta, const double* g, double delta, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_gd_step, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, n, beta, g, delta);
    return hipGetLastError();
}

hipError_t launch_camera_noise(int64_t n, const double* img, const double* mask, const double* normals,
                               unsigned long long* mx, double* out, double* scale_out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_masked_max, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, n, img, mask, mx);
    hipLaunchKernelGGL(k_camera_noise, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, n, img, normals, mx, out, scale_out);
    return hipGetLastError();
}

hipError_t launch_d2f(int64_t n, const double* in, float* out, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_d2f, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, n, in, out);
    return hipGetLastError();
}

hipError_t launch_recovery_sums(int64_t n, const double* b, const double* t, double* acc, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_recovery_sums, dim3(grid_for(n)), dim3(VOX_BLOCK), 0, s, n, b, t, acc);
    return hipGetLastError();
}

hipError_t launch_vox_los_adjoint(const VoxArgs& a, hipStream_t s) {
    const int tx = (a.nx + LOS_TILE - 1) / LOS_TILE, ty = (a.ny + LOS_TILE - 1) / LOS_TILE;
    const int64_t tiles = (int64_t)tx * ty * ((a.nz + LOS_TILE - 1) / LOS_TILE);
    hipLaunchKernelGGL(k_vox_los_adjoint, cam_grid(tiles, a.n_cams), dim3(LOS_BLOCK), 0, s, a, tx, ty);
    return hipGetLastError();
}

}  // namespace mcrt
