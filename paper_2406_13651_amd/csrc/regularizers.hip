// Comparison regularizers of Sec. V as prior agents of Alg. 2: the l_{2,1}
// agent (l2 over each range slice's cross-range plane, l1 over range) and
// the isotropic total-variation agent, each the proximal map of its
// regularizer on the prior agent's image.
//
// l_{2,1}: each range slice z is scaled by max(0, 1 - tau / ||v_z||_2): one
// pass of block partial sums of squares per slice, one pass that sums a
// slice's partials (fixed order, float64) and scales its voxels.
//
// TV: argmin_r lam TV(r) + ||r - v||^2 / 2 with TV the isotropic 3D total
// variation (forward differences, the difference leaving the volume zero),
// by `iters` steps of Chambolle's dual projection iteration from p = 0:
//   u = div p - v / lam;  g = grad u;  p <- (p + tau g) / (1 + tau |g|),
// then r = v - lam div p, with div the negative adjoint of grad and tau =
// 1/12 (the step that converges in three dimensions).  One launch per step:
// a block walks a tile of the (x, y) plane along z, keeps u of the current
// plane in LDS and forms the next plane's from p, so u never goes to memory,
// and writes the new p to a second buffer (its backward neighbours are still
// to be read).
#include "passes.hpp"

namespace clampk {

namespace {

constexpr int kL21Chunk = 16 * kBlock;  // voxels of a slice per partial-sum block

struct Vol {
    int nx, ny, nz;
};

__device__ __forceinline__ void voxel_coords(const Vol& d, unsigned i, int& x, int& y, int& z) {
    x = (int)(i % (unsigned)d.nx);
    const unsigned q = i / (unsigned)d.nx;
    y = (int)(q % (unsigned)d.ny);
    z = (int)(q / (unsigned)d.ny);
}

// Tile of a block of the TV kernels: LX lanes of four x-voxels each, kBlock /
// LX rows (64 x 16 voxels, or 32 x 32 where nx = 32).
template <int LX>
struct TvTile {
    static constexpr int kTX = 4 * LX, kTY = kBlock / LX;
};

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// The caller's images, which are only known to be float-aligned.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ld4u(const float* p) {
    const f4u v = *reinterpret_cast<const f4u*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

// What u of four x-voxels at one plane needs: pz, py there and one row back,
// px there and one voxel back, and v.  Off the low faces p is zero, and p is
// zero on the last index of its own axis (its difference there is zero and it
// starts at zero), so div p = p[i] - p[i - 1] holds on every voxel.
struct TvLoad {
    float4 c, b, by, a, w;
    float ax;
};

template <bool ZERO>
__device__ __forceinline__ void tv_load(TvLoad& t, const Vol& d, size_t n, const float* p, const float* v, unsigned i,
                                        int x, int y) {
    t.w = ld4u(v + i);
    if constexpr (!ZERO) {
        t.c = ld4(p + i);
        t.b = ld4(p + n + i);
        t.by = y > 0 ? ld4(p + n + i - (unsigned)d.nx) : make_float4(0.f, 0.f, 0.f, 0.f);
        t.a = ld4(p + 2 * n + i);
        t.ax = x > 0 ? p[2 * n + i - 1u] : 0.f;
    }
}

// div p (z, then y, then x component) of the loaded voxels; cprev = pz one
// plane back.
__device__ __forceinline__ float4 tv_div(const TvLoad& t, const float4& cprev) {
    return make_float4(t.c.x - cprev.x + (t.b.x - t.by.x) + (t.a.x - t.ax),
                       t.c.y - cprev.y + (t.b.y - t.by.y) + (t.a.y - t.a.x),
                       t.c.z - cprev.z + (t.b.z - t.by.z) + (t.a.z - t.a.y),
                       t.c.w - cprev.w + (t.b.w - t.by.w) + (t.a.w - t.a.z));
}

template <bool ZERO>
__device__ __forceinline__ float4 tv_u(const TvLoad& t, const float4& cprev, float inv_lam) {
    float4 u = make_float4(-t.w.x * inv_lam, -t.w.y * inv_lam, -t.w.z * inv_lam, -t.w.w * inv_lam);
    if constexpr (!ZERO) {
        const float4 q = tv_div(t, cprev);
        u = make_float4(q.x - t.w.x * inv_lam, q.y - t.w.y * inv_lam, q.z - t.w.z * inv_lam, q.w - t.w.w * inv_lam);
    }
    return u;
}

// The projection of one voxel: p <- (p + tau g) / (1 + tau |g|).  One
// reciprocal serves the three components; a residual step on each quotient
// keeps the division's rounding (left out for an overflowed denominator,
// where the quotient is 0 or NaN already).
__device__ __forceinline__ void tv_project(float gz, float gy, float gx, float tau, float& pz, float& py, float& px) {
    const float den = 1.f + tau * sqrtf(gz * gz + gy * gy + gx * gx);
    const float inv = 1.f / den;
    const float nz = pz + tau * gz, ny = py + tau * gy, nx = px + tau * gx;
    const float qz = nz * inv, qy = ny * inv, qx = nx * inv;
    const bool fin = den <= 3.402823466e38f;
    pz = fin ? fmaf(fmaf(-qz, den, nz), inv, qz) : qz;
    py = fin ? fmaf(fmaf(-qy, den, ny), inv, qy) : qy;
    px = fin ? fmaf(fmaf(-qx, den, nx), inv, qx) : qx;
}

}  // namespace

__global__ __launch_bounds__(kBlock) void k_l21_sums(int per, int chunks, const float* in, double* part) {
    const int z = blockIdx.y, c = blockIdx.x;
    const float* v = in + (size_t)z * per;
    const int end = (c + 1) * kL21Chunk < per ? (c + 1) * kL21Chunk : per;
    float f = 0.f;
    for (int i = c * kL21Chunk + (int)threadIdx.x; i < end; i += kBlock) f += v[i] * v[i];
    double acc[1] = {f};
    block_sum_store<1>(acc, part + (size_t)z * chunks + c);
}

__global__ __launch_bounds__(kBlock) void k_l21_shrink(int per, int chunks, float tau, const double* part,
                                                       const float* in, float* out) {
    const int z = blockIdx.y, c = blockIdx.x;
    __shared__ float scale;
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int k = 0; k < chunks; ++k) s += part[(size_t)z * chunks + k];
        const double nrm = sqrt(s);
        scale = nrm > 0.0 ? (float)fmax(0.0, 1.0 - (double)tau / nrm) : 0.f;
    }
    __syncthreads();
    const float sc = scale;
    const float* v = in + (size_t)z * per;
    float* o = out + (size_t)z * per;
    const int end = (c + 1) * kL21Chunk < per ? (c + 1) * kL21Chunk : per;
    for (int i = c * kL21Chunk + (int)threadIdx.x; i < end; i += kBlock) o[i] = sc * v[i];
}

// One step of the dual iteration, p in, q out (ZERO: p is zero and is not
// read).  Block (tile, z chunk): each thread owns four x-voxels of one row and
// walks `cz` planes.  u of plane z lies in LDS (with the row y0 + TY and the
// column x0 + TX past the tile, which the first wave's and the second wave's
// lanes compute beside their own voxels); the loads of plane z + 1 are issued
// before plane z is finished.  Two LDS planes, so one barrier per plane: it
// stands between the writes of plane z and its readers, and every reader of
// the plane that is overwritten next has passed it.
// Bound by memory (the images of a 256x256x64 volume stay in the 256 MB
// Infinity Cache): 28 bytes per voxel and step where separate divergence and
// projection passes move 48.  20 steps at 256x256x64: 410 us (5.6 TB/s of
// those bytes; the first step reads no p) against 940 us for the two passes; with the tiles dealt to the
// XCDs one by one instead of in runs, the halos of tiles on other XCDs made
// it 118 MB read per step instead of 67, and 523 us.
template <int LX, bool ZERO>
__global__ __launch_bounds__(kBlock) void k_tv_step(Vol d, size_t n, int cz, float inv_lam, float tau, const float* p,
                                                    const float* v, float* q) {
    constexpr int TX = TvTile<LX>::kTX, TY = TvTile<LX>::kTY;
    static_assert(LX <= 64 && TY <= 64, "the halo row and column fit one wave each");
    __shared__ __attribute__((aligned(16))) float su[2][TY + 1][TX + 4];
    const int tid = threadIdx.x, lx = tid % LX, ry = tid / LX;
    const int tiles_x = d.nx / TX;
    // blocks go to the eight XCDs in turn: each XCD gets a run of neighbouring
    // tiles, whose halos it then reads from its own L2
    const unsigned per_xcd = gridDim.x / 8u;
    const unsigned blk = blockIdx.x < 8u * per_xcd ? (blockIdx.x % 8u) * per_xcd + blockIdx.x / 8u : blockIdx.x;
    const int tiles = tiles_x * (d.ny / TY), tile = (int)(blk % tiles);
    const int x0 = tile % tiles_x * TX, y0 = tile / tiles_x * TY;
    const int z0 = (int)(blk / tiles) * cz, z1 = z0 + cz < d.nz ? z0 + cz : d.nz;
    const int x = x0 + 4 * lx, y = y0 + ry;
    const unsigned plane = (unsigned)d.nx * (unsigned)d.ny;
    const unsigned own = (unsigned)y * (unsigned)d.nx + (unsigned)x;
    // halo voxels: wave 0 the row y0 + TY, wave 1 the column x0 + TX
    const bool hrow = tid < LX, hcol = tid >= 64 && tid < 64 + TY;
    const int hx = hrow ? x : x0 + TX, hy = hrow ? y0 + TY : y0 + tid - 64;
    const bool halo = (hrow && hy < d.ny) || (hcol && hx < d.nx);
    const unsigned hown = halo ? (unsigned)hy * (unsigned)d.nx + (unsigned)hx : 0u;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);

    TvLoad t, th;
    float4 cprev = zero, hprev = zero;
    const unsigned i0 = (unsigned)z0 * plane;
    if (!ZERO && z0 > 0) {
        cprev = ld4(p + i0 - plane + own);
        if (halo) hprev = ld4(p + i0 - plane + hown);
    }
    tv_load<ZERO>(t, d, n, p, v, i0 + own, x, y);
    if (halo) tv_load<ZERO>(th, d, n, p, v, i0 + hown, hx, hy);
    auto put = [&](int s, const float4& u) {
        *reinterpret_cast<float4*>(&su[s][ry][4 * lx]) = u;
        if (halo) {
            const float4 uh = tv_u<ZERO>(th, hprev, inv_lam);
            if (hrow) *reinterpret_cast<float4*>(&su[s][TY][4 * lx]) = uh;
            else su[s][tid - 64][TX] = uh.x;
            if constexpr (!ZERO) hprev = th.c;
        }
    };
    float4 u = tv_u<ZERO>(t, cprev, inv_lam);
    put(0, u);
    float4 pz = zero, py = zero, px = zero;  // p of the plane being finished
    if constexpr (!ZERO) {
        pz = t.c;
        py = t.b;
        px = t.a;
        cprev = t.c;
    }
    int s = 0;
    for (int z = z0; z < z1; ++z, s ^= 1) {
        const unsigned i = (unsigned)z * plane;
        const bool up = z + 1 < d.nz;  // uniform: the plane above exists
        if (up) {
            tv_load<ZERO>(t, d, n, p, v, i + plane + own, x, y);
            if (halo) tv_load<ZERO>(th, d, n, p, v, i + plane + hown, hx, hy);
        }
        __syncthreads();
        const float4 uy = y + 1 < d.ny ? *reinterpret_cast<const float4*>(&su[s][ry + 1][4 * lx]) : u;
        const float ux = x + 4 < d.nx ? su[s][ry][4 * lx + 4] : u.w;
        const float4 un = up ? tv_u<ZERO>(t, cprev, inv_lam) : u;
        tv_project(un.x - u.x, uy.x - u.x, u.y - u.x, tau, pz.x, py.x, px.x);
        tv_project(un.y - u.y, uy.y - u.y, u.z - u.y, tau, pz.y, py.y, px.y);
        tv_project(un.z - u.z, uy.z - u.z, u.w - u.z, tau, pz.z, py.z, px.z);
        tv_project(un.w - u.w, uy.w - u.w, ux - u.w, tau, pz.w, py.w, px.w);
        *reinterpret_cast<float4*>(q + i + own) = pz;
        *reinterpret_cast<float4*>(q + n + i + own) = py;
        *reinterpret_cast<float4*>(q + 2 * n + i + own) = px;
        if (z + 1 < z1) put(s ^ 1, un);
        u = un;
        if constexpr (!ZERO) {
            pz = t.c;
            py = t.b;
            px = t.a;
            cprev = t.c;
        } else {
            pz = py = px = zero;
        }
    }
}

// r = v - lam div p, four x-voxels per thread (ZERO: p is zero)
template <bool ZERO>
__global__ __launch_bounds__(kBlock) void k_tv_out(Vol d, size_t n, float lam, const float* p, const float* v,
                                                   float* out) {
    const unsigned i = 4u * (blockIdx.x * kBlock + threadIdx.x);
    if (i >= n) return;
    float4 w = ld4u(v + i);
    if constexpr (!ZERO) {
        int x, y, z;
        voxel_coords(d, i, x, y, z);
        TvLoad t;
        tv_load<false>(t, d, n, p, v, i, x, y);
        const float4 cp = z > 0 ? ld4(p + i - (unsigned)d.nx * (unsigned)d.ny) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 q = tv_div(t, cp);
        w = make_float4(w.x - lam * q.x, w.y - lam * q.y, w.z - lam * q.z, w.w - lam * q.w);
    }
    *reinterpret_cast<f4u*>(out + i) = f4u{w.x, w.y, w.z, w.w};
}

int l21_chunks(int nx, int ny) { return (nx * ny + kL21Chunk - 1) / kL21Chunk; }

hipError_t launch_prior_l21(int nx, int ny, int nz, float tau, const float* in, float* out, double* part,
                            hipStream_t st) {
    const int per = nx * ny, chunks = l21_chunks(nx, ny);
    hipLaunchKernelGGL(k_l21_sums, dim3(chunks, nz), dim3(kBlock), 0, st, per, chunks, in, part);
    hipLaunchKernelGGL(k_l21_shrink, dim3(chunks, nz), dim3(kBlock), 0, st, per, chunks, tau, part, in, out);
    return hipGetLastError();
}

template <int LX>
static void launch_tv_steps(const Vol& d, size_t n, float lam, int iters, const float* in, float* p0, float* p1,
                            hipStream_t st) {
    const int tiles = (d.nx / TvTile<LX>::kTX) * (d.ny / TvTile<LX>::kTY);
    // Planes per block: a block forms u of one plane more than it finishes, so
    // long walks read least, but two blocks per CU are wanted to hide the
    // loads.  20 steps at 256x256x64: walks of 16, 8 and 4 planes (256, 512,
    // 1024 blocks) take 483, 410 and 429 us.
    int cz = 16;
    while (cz > 1 && (long)tiles * ((d.nz + cz - 1) / cz) < 512) cz /= 2;
    const dim3 grid((unsigned)tiles * (unsigned)((d.nz + cz - 1) / cz));
    const float inv_lam = 1.f / lam, tau = 1.f / 12.f;
    for (int k = 0; k < iters; ++k) {
        const float* src = (k & 1) ? p0 : p1;
        float* dst = (k & 1) ? p1 : p0;
        if (k == 0)
            hipLaunchKernelGGL((k_tv_step<LX, true>), grid, dim3(kBlock), 0, st, d, n, cz, inv_lam, tau, src, in, dst);
        else
            hipLaunchKernelGGL((k_tv_step<LX, false>), grid, dim3(kBlock), 0, st, d, n, cz, inv_lam, tau, src, in, dst);
    }
}

hipError_t launch_prior_tv(int nx, int ny, int nz, float lam, int iters, const float* in, float* out, float* p,
                           hipStream_t st) {
    const Vol d{nx, ny, nz};
    const size_t n = (size_t)nx * ny * nz;
    if (nx % 32 != 0 || ny % 32 != 0) return hipErrorInvalidValue;  // every supported length is a multiple of 32
    float* p1 = p + 3 * n;
    if (nx % 64 == 0) launch_tv_steps<16>(d, n, lam, iters, in, p, p1, st);
    else launch_tv_steps<8>(d, n, lam, iters, in, p, p1, st);
    const float* last = (iters & 1) ? p : p1;
    const dim3 grid((unsigned)((n / 4 + kBlock - 1) / kBlock));
    if (iters <= 0) hipLaunchKernelGGL(k_tv_out<true>, grid, dim3(kBlock), 0, st, d, n, lam, last, in, out);
    else hipLaunchKernelGGL(k_tv_out<false>, grid, dim3(kBlock), 0, st, d, n, lam, last, in, out);
    return hipGetLastError();
}

}  // namespace clampk
