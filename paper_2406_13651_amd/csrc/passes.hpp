// Work items of the forward-agent passes as device functions.  A work item
// is one unit that a block processes: a group of rows of one slice of one
// look (row passes), a tile of band columns of one slice of one look (column
// passes), or one look (step size and diagnostics).  The single-scene
// kernels map one block to one item; the batched kernels walk a queue of
// items of many scenes, choosing the FFT length of each item at run time.
// LDS buffers are passed in, so a batched kernel can share one allocation
// between items of different lengths.
#pragma once

#include <math.h>

#include <type_traits>

#include "fft.hpp"
#include "internal.h"

namespace clampk {

constexpr int kRowPad = 4;  // one float2 of LDS padding per 16 row samples

// Non-temporal loads and stores, for streams that do not fit the caches
// between their writer and reader anyway: the pointwise streams of the update
// pass and the Mann step, the residual update, and the band buffers between
// the column and row passes.  They then do not displace cached data that the
// other passes reuse (measured at 256x256x64, 16 looks: update pass 428 ->
// 355 us, whole iteration 1.30 -> 1.16 ms).
__device__ __forceinline__ float ld_stream(const float* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ float2 ld_stream(const float2* p) {
    return make_float2(__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y));
}
__device__ __forceinline__ void st_stream(float* p, float v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void st_stream(float2* p, float2 v) {
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
}

template <int N>
__host__ __device__ constexpr int row_lds_floats2() {
    return rows_per_block(N) * lds_len<N, kRowPad>();
}

// The other lane's double in a step of a reduction within rows of 16 lanes
// (DPP row rotation).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const long long b = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
// a + b after the upper half of a and the lower half of b (HALF = 32: of the
// wave; 16: of each half wave) have changed places: the lower half holds the
// sums of a's halves, the upper half those of b's.
template <int HALF>
__device__ __forceinline__ double swap_add_f64(double a, double b) {
    const unsigned long long ua = __builtin_bit_cast(unsigned long long, a);
    const unsigned long long ub = __builtin_bit_cast(unsigned long long, b);
    unsigned alo, ahi, blo, bhi;
    if constexpr (HALF == 32) {
        const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
        alo = lo[0], blo = lo[1], ahi = hi[0], bhi = hi[1];
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
        alo = lo[0], blo = lo[1], ahi = hi[0], bhi = hi[1];
    }
    return __builtin_bit_cast(double, ((unsigned long long)ahi << 32) | alo) +
           __builtin_bit_cast(double, ((unsigned long long)bhi << 32) | blo);
}
// Sums of up to four doubles over the wave: lane 16 i (and its row of 16
// lanes) returns the sum of value order(i) = {0, 2, 1, 3}.  The first two
// steps exchange registers and halve the number of values as they halve the
// lanes that hold them; the row steps are DPP moves.  No LDS instructions:
// three sums by shuffles were 36 of them and 18 additions, a tenth of the
// instructions of the gradient pass, which the vector unit bounds (74% busy;
// 256x256x64, 16 looks: 270 -> 244 us with these sums and slice_of_row).
template <int K>
__device__ __forceinline__ double wave_sums_f64(const double (&v)[K]) {
    static_assert(K >= 1 && K <= 4, "up to four values");
    const double a = swap_add_f64<32>(v[0], K > 1 ? v[K > 1 ? 1 : 0] : v[0]);
    double x;
    if constexpr (K > 2) x = swap_add_f64<16>(a, swap_add_f64<32>(v[2], K > 3 ? v[K > 3 ? 3 : 2] : v[2]));
    else x = swap_add_f64<16>(a, a);
    x += dpp_f64<0x128>(x);  // row_ror 8, 4, 2, 1
    x += dpp_f64<0x124>(x);
    x += dpp_f64<0x122>(x);
    x += dpp_f64<0x121>(x);
    return x;
}
// The value whose sum lane row i of wave_sums_f64 holds.
__host__ __device__ constexpr int wave_sums_slot(int i) { return i == 1 ? 2 : i == 2 ? 1 : i; }

// Each wave's sums of K doubles into red[.][wave] (W waves).
template <int K, int W>
__device__ __forceinline__ void wave_sums_store(const double (&v)[K], double (&red)[K][W]) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 4) {
        double s;
        if (k0 + 4 <= K) {
            double q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = v[k0 + k < K ? k0 + k : 0];
            s = wave_sums_f64<4>(q);
        } else {
            constexpr int KR = K % 4 > 0 ? K % 4 : 1;
            double q[KR];
#pragma unroll
            for (int k = 0; k < KR; ++k) q[k] = v[k0 + k < K ? k0 + k : 0];
            s = wave_sums_f64<KR>(q);
        }
        const int slot = k0 + wave_sums_slot(lane >> 4);
        if ((lane & 15) == 0 && slot < K) red[slot][wid] = s;
    }
}

// Sum of K doubles over the block, written by thread 0 to out[0..K).
template <int K>
__device__ __forceinline__ void block_sum_store(const double (&v)[K], double* out) {
    __shared__ double red[K][kBlock / 64];
    wave_sums_store(v, red);
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) s += red[k][w];
            out[k] = s;
        }
    }
    __syncthreads();  // red may be reused by the next item
}

// v[k] += p[i * stride + k] (k < K) for i = threadIdx.x, + kBlock, ... below
// count, with eight rows of loads in flight per thread (rows past count
// re-read the last one and are not added).  The order of the additions is
// fixed, so the sums are deterministic.
template <int K>
__device__ __forceinline__ void strided_sums(const double* p, int count, int stride, double* v) {
    for (int i0 = threadIdx.x; i0 < count; i0 += 8 * kBlock) {
        double x[8][K];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kBlock;
            const double* q = p + (size_t)(i < count ? i : count - 1) * stride;
#pragma unroll
            for (int k = 0; k < K; ++k) x[u][k] = q[k];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (i0 + u * kBlock < count) {
#pragma unroll
                for (int k = 0; k < K; ++k) v[k] += x[u][k];
            }
        }
    }
}

__device__ __forceinline__ void wave_or_fault(uint32_t bits, uint32_t* fault) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) bits |= __shfl_xor(bits, off);
    if ((threadIdx.x & 63) == 0 && bits != 0u && fault != nullptr) atomicOr(fault, bits);
}

// Read-only device tables (the batch's scene table and work queues) seen
// through the constant address space.  Nothing writes them while a kernel
// runs, so a read at a wave-uniform address is a scalar load that the
// compiler may issue again where a field is used instead of holding the
// whole block in registers -- as it does for kernel arguments.
// (The host pass of this file compiles the kernels' declarations only, and
// has no constant address space.)
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
using ConstAS = const __attribute__((address_space(4))) T;
#else
template <class T>
using ConstAS = const T;
#endif
template <class T>
__device__ __forceinline__ ConstAS<T>& const_ref(const T* p) {
    return *(ConstAS<T>*)p;
}

// Copy of a wave-uniform argument block from device memory into scalar
// registers: the private copy cannot alias the item's stores, and
// readfirstlane keeps it out of the vector register file.
template <class T>
__device__ __forceinline__ T load_uniform(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "argument blocks are whole dwords");
    T out;
    const int* src = reinterpret_cast<const int*>(p);
    int* dst = reinterpret_cast<int*>(&out);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) dst[i] = __builtin_amdgcn_readfirstlane(src[i]);
    return out;
}

// Interval factor and the derived constants of the surrogate r-update.
struct BetaVals {
    float beta, inv_beta, k_up, k_dn;
};
__host__ __device__ inline BetaVals beta_vals(double beta) {
    BetaVals b;
    b.beta = (float)beta;
    b.inv_beta = (float)(1.0 / beta);
    b.k_up = (float)((1.0 + beta) / (beta * beta));  // xi = beta r'
    b.k_dn = (float)(beta * (1.0 + beta));           // xi = r' / beta
    return b;
}

// Exact proximal map of the EM surrogate for one voxel (eq. surrogate-prox):
// argmin over r > 0 of log r + s/r + (r - v)^2 / (2 sigma^2).  Its stationary
// points are the positive roots of r^3 - v r^2 + sigma^2 r - sigma^2 s (the
// derivative times sigma^2 r^2, negative at r = 0, so a positive root exists).
// With r = t + v/3 the cubic is t^3 + p t + q; its roots come from the
// trigonometric form when it has three real roots and from Cardano's form
// (the cube root taken on the side without cancellation) when it has one,
// each polished by two Newton steps, all in float64.  The positive root with
// the smallest objective is returned (the objective is not convex for r > 2 s
// and can have two local minima).
__device__ __forceinline__ float exact_prox(float sf, float vf, float s2f) {
    const double s = sf, v = vf, q2 = s2f;
    const double sh = v / 3.0;
    const double p = q2 - v * v / 3.0;
    const double q = -2.0 * v * v * v / 27.0 + v * q2 / 3.0 - q2 * s;
    const double disc = 0.25 * q * q + p * p * p / 27.0;
    double root[3];
    int nr;
    if (disc > 0.0) {
        const double a = -0.5 * q;
        const double u = cbrt(a + copysign(sqrt(disc), a));
        root[0] = (u != 0.0 ? u - p / (3.0 * u) : 0.0) + sh;
        nr = 1;
    } else {
        const double m = 2.0 * sqrt(fmax(-p / 3.0, 0.0));
        const double c = m > 0.0 ? fmin(fmax(3.0 * q / (p * m), -1.0), 1.0) : 0.0;
        const double th = acos(c) / 3.0;
        const double third = 2.0943951023931954923;  // 2 pi / 3
        root[0] = m * cos(th) + sh;
        root[1] = m * cos(th - third) + sh;
        root[2] = m * cos(th - 2.0 * third) + sh;
        nr = 3;
    }
    double best = 0.0, best_phi = 0.0;
    bool found = false;
    for (int k = 0; k < nr; ++k) {
        double r = root[k];
        for (int it = 0; it < 2; ++it) {
            const double f = ((r - v) * r + q2) * r - q2 * s;
            const double df = (3.0 * r - 2.0 * v) * r + q2;
            if (df != 0.0) r -= f / df;
        }
        if (r > 0.0) {
            const double phi = log(r) + s / r + (r - v) * (r - v) / (2.0 * q2);
            if (!found || phi < best_phi) {
                best = r;
                best_phi = phi;
                found = true;
            }
        }
    }
    return (float)best;  // 0 (flagged by the caller) only if no positive root was found
}

// Surrogate r-update of one voxel at the anchor r0 and prox point v, with the
// updated mean m1: covariance diagonal c = sigma_w^2 r0 / (alpha r0 +
// sigma_w^2) (A^H A ~ alpha I), s = c + |m1|^2, then the quadratic surrogate
// of App. A (ROW_UPDATE) or the exact surrogate prox (ROW_UPDATE_EXACT).
// Fault bits: 1 for a non-finite result or mean, 2 for r <= 0.
template <int MODE, class A>
__device__ __forceinline__ float r_update_voxel(const A& a, const BetaVals& bv, float r0, float v, float2 m1,
                                                uint32_t& fb) {
    const float c = a.s2w * r0 / (a.alpha * r0 + a.s2w);
    const float sv = c + cabs2(m1);
    float rn;
    if constexpr (MODE == ROW_UPDATE_EXACT) {
        rn = exact_prox(sv, v, a.sigma2);
        if (!(rn == rn) || !isfinite(m1.x) || !isfinite(m1.y)) fb |= 1u;
    } else {
        // quadratic surrogate of r/r' + s/r, interpolating its derivative at
        // r' and xi; written with s/r' first so that small anchors stay in
        // float32 range
        const float inv = 1.f / r0;
        const float sr = sv * inv;
        const float dq = inv * (1.f - sr);                  // q'(r')
        const float D = dq + (r0 - v) * a.inv_sigma2;       // rho'(r')
        const bool down = D > 0.f;
        const float xi = down ? r0 * bv.inv_beta : r0 * bv.beta;
        const float qa = sr * inv * inv * (down ? bv.k_dn : bv.k_up);
        const float qb = dq - qa * r0;
        rn = (v - a.sigma2 * qb) / (1.f + a.sigma2 * qa);
        if (!(rn == rn) || !isfinite(m1.x) || !isfinite(m1.y)) fb |= 1u;
        rn = fminf(fmaxf(rn, fminf(r0, xi)), fmaxf(r0, xi));
    }
    if (!(rn > 0.f)) fb |= 2u;
    return rn;
}

// row / ny by the plan's reciprocal ny_mul = floor(2^32 / ny) + 1: with e = ny
// ny_mul - 2^32 <= ny the product's high word exceeds the quotient by at most
// row e / 2^32 / ny < 1 for any row below 2^31, so by one at most.
template <class T>
__device__ __forceinline__ int slice_of_row(const T& s, int row) {
    const int q = (int)__umulhi((unsigned)row, s.ny_mul);
    return q * s.ny > row ? q - 1 : q;
}

// LDS buffers of a row item: twiddles, band position and band column tables
// (length NX each; the band columns for the passes that write band rows) and
// the padded row buffers.
struct RowLds {
    float2* tw;
    int* bpos;
    int* bcol;
    float2* buf;
};

// How a row's first transform takes its samples: sample q of thread t is
// element t + q kStep.  Power-of-two rows go through fft_regs, whose first
// stage reads what the pointwise steps hold (t + k TR); 192- and 384-point rows
// through fft_split, whose first stage is one radix-8 butterfly on each of
// the threads t < kStep (384x192x37, 5 looks, against every stage through LDS:
// gradient pass 85 -> 70 us, update pass 118 -> 98 us).
template <int NX>
struct RowIn {
    static constexpr int TR = row_threads(NX);
    static constexpr int PX = NX / TR;  // row samples per thread
    static_assert(NX % TR == 0, "row samples divide among the threads");
    static constexpr bool kRegs = fft_regs_ok<NX, TR>();
    static constexpr int kStep = kRegs ? TR : NX / radix_at(NX, 0);
    static constexpr int kCount = kRegs ? PX : radix_at(NX, 0);
    __device__ __forceinline__ static bool has(int t) { return kRegs || t < kStep; }
};

// Row transform of in (the samples of RowIn) into h (h[k] = element t + k TR)
// or, without OUT_REGS, into rb in natural order, for gathers across the row
// by the row's own wave.
template <int NX, int S, bool OUT_REGS>
__device__ __forceinline__ void row_fft_in(float2 (&in)[RowIn<NX>::kCount], float2 (&h)[RowIn<NX>::PX], float2* rb,
                                           int t, const float2* tw) {
    using R = RowIn<NX>;
    if constexpr (R::kRegs) {
#pragma unroll
        for (int k = 0; k < R::PX; ++k) h[k] = in[k];
        fft_regs<NX, R::TR, S, kRowPad, true, OUT_REGS, true>(h, rb, 1, t, tw);
    } else {
        fft_split<NX, R::TR, S, kRowPad, OUT_REGS, true>(in, h, rb, t, tw);
    }
}

// Row transform of h (h[k] = element t + k TR of the row), to h or rb as above.
template <int NX, int S, bool OUT_REGS>
__device__ __forceinline__ void row_fft(float2 (&h)[RowIn<NX>::PX], float2* rb, int t, const float2* tw) {
    using R = RowIn<NX>;
    if constexpr (R::kRegs) {
        fft_regs<NX, R::TR, S, kRowPad, true, OUT_REGS, true>(h, rb, 1, t, tw);
    } else {
        group_sync<true>();
#pragma unroll
        for (int k = 0; k < R::PX; ++k) rb[lds_pos<kRowPad>(t + k * R::TR)] = h[k];
        group_sync<true>();
        float2 in[R::kCount];
        if (R::has(t)) {
#pragma unroll
            for (int q = 0; q < R::kCount; ++q) in[q] = rb[lds_pos<kRowPad>(t + q * R::kStep)];
        }
        fft_split<NX, R::TR, S, kRowPad, OUT_REGS, true>(in, h, rb, t, tw);
    }
}

// Pointwise step of the gradient pass on one row held in h (the inverse row
// FFT of the band already applied): d = A^H r / sigma_w^2 - omega mu with
// omega = 1 / (r' + sigma_w^2 / alpha), written back into h, plus the
// thread's shares of ||d||^2, sum omega |d|^2 and sum omega |mu|^2.
// SLICE (the slice pass): |mu|^2 is rounded as the compiler rounds it in the
// gradient row pass -- the square of x first, in the last sample that of y --
// so that both report the same sums.  The GPU tests compare a batch, which
// takes the row pass, with single scenes, which take the slice pass, and fail
// where a compiler rounds otherwise.
template <bool SLICE, int PX, class A>
__device__ __forceinline__ void row_grad_pointwise(const A& a, float2 (&h)[PX], const float2 (&m)[PX],
                                                   const float (&rp)[PX], float& dd, float& wd, float& wm) {
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        const float2 ahr = cscale(h[k], a.scale);
        const float om = 1.f / (rp[k] + a.floor_w);
        const float2 d = make_float2(ahr.x * a.inv_s2w - om * m[k].x, ahr.y * a.inv_s2w - om * m[k].y);
        h[k] = d;
        const float d2 = cabs2(d);
        dd += d2;
        wd += om * d2;
        if constexpr (SLICE) {
            const float x = k + 1 < PX ? m[k].x : m[k].y, y = k + 1 < PX ? m[k].y : m[k].x;
            wm = fmaf(om, fmaf(y, y, x * x), wm);
        } else {
            wm += om * cabs2(m[k]);
        }
    }
}

// ---------------------------------------------------------------------------
// Row pass over rows [rgroup * RPB, rgroup * RPB + RPB) of look `look`;
// `slot` indexes the look's partial-sum slots.  `load_tables` reloads the
// row tables (the caller skips it when the previous item had the same scene).
template <int NX, int MODE, class A>
__device__ __forceinline__ void row_item(const A& a, int look, int rgroup, size_t slot, const RowLds& L,
                                         bool load_tables, BetaVals bv) {
    constexpr int TR = row_threads(NX);
    constexpr int RPB = rows_per_block(NX);
    constexpr int PX = RowIn<NX>::PX;               // row samples per thread
    constexpr int PAD = kRowPad;
    constexpr int RS = lds_len<NX, PAD>();          // padded row length in LDS
    // ROW_UPDATE_EXACT is the update pass with the exact surrogate prox in
    // place of the quadratic surrogate (a separate instantiation, so that the
    // float64 root solve does not raise the register count of the other)
    constexpr bool UPD = (MODE == ROW_UPDATE || MODE == ROW_UPDATE_EXACT);
    constexpr bool FUSED = (MODE == ROW_GRAD || UPD);
    // Stream prefetch pays off for the gradient pass; the update pass already
    // runs near the read/write bandwidth ceiling and loads its streams late.
    constexpr bool PREFETCH = (MODE == ROW_GRAD);
    const auto& s = a.s;
    const int tid = threadIdx.x, t = tid % TR;
    // a row that fills its wave (384 and 512 points) has wave-uniform indices
    // and base addresses, held in scalar registers: 76 vector registers in the
    // 512-point gradient pass, where 80 were not enough at six waves and one
    // went to scratch (512x512x64, 8 looks: 486 -> 456 us)
    const int ri = TR == 64 ? __builtin_amdgcn_readfirstlane(tid / TR) : tid / TR;
    const int rows = s.nz * s.ny;
    const int row = rgroup * RPB + ri;
    const bool active = row < rows;
    const size_t img = ((size_t)look * rows + (active ? row : 0)) * NX;
    const int arow = active ? row : 0;
    const int slice = slice_of_row(s, arow);
    const size_t band = ((size_t)look * s.nz + slice) * s.ny * s.Bs + band_row_off(arow - slice * s.ny, s.ny);

    float2 m[FUSED ? PX : 1];
    float rp[FUSED ? PX : 1];
    float wv[UPD ? PX : 1];
    auto load_streams = [&]() {
        if (active) {
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                const int x = t + k * TR;
                if constexpr (UPD) {
                    m[k] = ld_stream(&a.mu[img + x]);
                    rp[k] = ld_stream(&a.r[img + x]);
                    wv[k] = ld_stream(&a.w[img + x]);
                } else {
                    m[k] = a.mu[img + x];
                    rp[k] = a.r[img + x];
                }
            }
        }
    };
    __syncthreads();  // the previous item's readers of the LDS buffers are done
    if (load_tables) {
        for (int i = tid; i < NX; i += kBlock) {
            // unconditional, and before the first store: one wait for all three tables
            const float2 w = s.tw_x[i];
            const int bp = s.band_pos[i], bc = s.band_cols[i < s.B ? i : 0];
            L.tw[i] = w;
            L.bpos[i] = bp;
            L.bcol[i] = i < s.B ? bc : 0;
        }
        __syncthreads();
    }
    float2* rb = L.buf + ri * RS;

    // the row's samples for the first transform (zero for inactive rows), and
    // the row in registers: h[k] = element t + k TR
    using In = RowIn<NX>;
    float2 in[In::kCount], h[PX];
    const bool has = active && In::has(t);
    if constexpr (MODE == ROW_FWD) {
        // all loads issued before the first is used (threads without samples
        // read the row's first ones, inactive rows row 0)
        const float2* row_in = a.img_in + img + (In::has(t) ? t : 0);
#pragma unroll
        for (int q = 0; q < In::kCount; ++q) in[q] = row_in[q * In::kStep];
#pragma unroll
        for (int q = 0; q < In::kCount; ++q)
            if (!has) in[q] = make_float2(0.f, 0.f);
    } else {
        // The row's band samples: all loads are issued before the first
        // is used (samples off the band read the row's first band sample and
        // are replaced by zero), then the pointwise streams are prefetched
        // behind them.
        float2 bin[In::kCount];
        int bp[In::kCount];
#pragma unroll
        for (int q = 0; q < In::kCount; ++q) {
            bp[q] = has ? L.bpos[t + q * In::kStep] : -1;
            bin[q] = ld_stream(a.band_in + band + (bp[q] >= 0 ? bp[q] : 0));  // inactive rows read row 0
        }
        if constexpr (PREFETCH) load_streams();
#pragma unroll
        for (int q = 0; q < In::kCount; ++q) in[q] = bp[q] >= 0 ? bin[q] : make_float2(0.f, 0.f);
    }

    if constexpr (MODE == ROW_INV) {
        row_fft_in<NX, +1, true>(in, h, rb, t, L.tw);
        if (active) {
#pragma unroll
            for (int k = 0; k < PX; ++k) a.img_out[img + t + k * TR] = cscale(h[k], a.scale);
        }
    } else if constexpr (MODE == ROW_FWD) {
        row_fft_in<NX, -1, false>(in, h, rb, t, L.tw);
        if (active)
            for (int b = t; b < s.B; b += TR)
                a.band_out[band + band_col_off(b, s.ny)] = cscale(rb[lds_pos<PAD>(L.bcol[b])], a.scale);
    } else if constexpr (MODE == ROW_GRAD) {
        row_fft_in<NX, +1, true>(in, h, rb, t, L.tw);
        float dd = 0.f, wd = 0.f, wm = 0.f;
        if (active) row_grad_pointwise<false>(a, h, m, rp, dd, wd, wm);
        row_fft<NX, -1, false>(h, rb, t, L.tw);
        if (active)
            for (int b = t; b < s.B; b += TR)
                st_stream(a.band_out + band + band_col_off(b, s.ny), cscale(rb[lds_pos<PAD>(L.bcol[b])], a.scale));
        double acc[3] = {dd, wd, wm};
        block_sum_store<3>(acc, a.part + slot * 3);
    } else {  // ROW_UPDATE
        row_fft_in<NX, +1, true>(in, h, rb, t, L.tw);
        if constexpr (!PREFETCH) load_streams();
        const float gamma = (float)a.diag[(size_t)look * kDiag];
        float wm1 = 0.f;
        uint32_t fb = 0u;
        if (active) {
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                const int x = t + k * TR;
                const float2 ahr = cscale(h[k], a.scale);
                const float r0 = rp[k];
                const float v = wv[k];
                const float om = 1.f / (r0 + a.floor_w);
                const float2 d = make_float2(ahr.x * a.inv_s2w - om * m[k].x, ahr.y * a.inv_s2w - om * m[k].y);
                const float2 m1 = make_float2(m[k].x + gamma * d.x, m[k].y + gamma * d.y);
                st_stream(&a.mu[img + x], m1);
                const float rn = r_update_voxel<MODE>(a, bv, r0, v, m1, fb);
                st_stream(&a.r[img + x], rn);
                wm1 += om * cabs2(m1);
            }
        }
        wave_or_fault(fb, a.fault);
        double acc[1] = {wm1};
        block_sum_store<1>(acc, a.part + slot);
    }
}

// ---------------------------------------------------------------------------
// Update pass with the Mann step of Alg. 1 fused in: every look of a group of
// rows passes through one block.  Per look it does what row_item's update
// does (recompute d, mu += gamma d, the r-update), with the prox point v =
// u_l + 2 rho xbar_old, and writes u_l' = v - 2 rho r_l; across looks it
// keeps, per voxel, sum_j upsilon_j r_j and sum_j (r_j - w_bar)^2, where
// w_bar = sum_j upsilon_j w_j is the average of the Mann state passed in
// (G(w)), which the previous call left in f.wbar.  After the last look it
// adds the prior agent (its w and H(w)) and writes x_bar = sum_j upsilon_j
// (2 r_j - w_j) = 2 sum_j upsilon_j r_j - w_bar, the new average w_bar +
// 2 rho (sum_j upsilon_j r_j - w_bar) and the prior's new w.
//
// A group is the 64 / TR rows of one wave.  `split` of the block's four waves
// (1, 2 or 4) share a group and take its looks in turn, so that the serial
// chain over the looks is that much shorter (mann_split).  After each turn the
// waves exchange their r_l through the row buffers, and each adds those of
// its share of the voxels in look order -- the same sums, rounding by
// rounding, as one wave walking every look -- and finishes that share.
// Partial sums per block: sum omega |mu'|^2 of each look into a.part, the
// convergence error's (sum_j (r_j - w_bar)^2, N w_bar^2) into f.part.
template <int NX>
__host__ __device__ constexpr int mann_lds_floats() {
    return 2 * kBlock * RowIn<NX>::PX;
}

// LDS: ups[64] holds the agent weights, keep[mann_lds_floats<NX>()] each
// group's x_bar and w_bar of the previous call ([k][group lane],
// conflict-free), read back at every look instead of held in registers.
template <int NX, int MODE, class A, class F>
__device__ __forceinline__ void row_update_mann(const A& a, const F& f, int split, int blk, int nblk,
                                                const RowLds& L, BetaVals bv, float* ups, float* keep) {
    __shared__ double wsum[64][4];                  // [look][wave], at most 64 looks
    constexpr int TR = row_threads(NX);
    constexpr int RPW = 64 / TR;                    // rows per wave
    constexpr int PX = RowIn<NX>::PX;
    constexpr int PAD = kRowPad;
    constexpr int RS = lds_len<NX, PAD>();
    const auto& s = a.s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gpb = 4 / split;                      // groups per block
    const int gi = wave / split, part = wave % split;
    const int t = lane % TR;
    const int rows = s.nz * s.ny;
    const int row = (blk * gpb + gi) * RPW + lane / TR;
    const bool active = row < rows;
    const size_t n = (size_t)rows * NX;
    const int arow = active ? row : 0;
    const int slice = slice_of_row(s, arow);
    const size_t pix = (size_t)arow * NX;
    const int kst = 64 * gpb, kl = gi * 64 + lane;  // keep's stride and this lane's slot
    for (int i = tid; i < NX; i += kBlock) {
        L.tw[i] = s.tw_x[i];
        L.bpos[i] = s.band_pos[i];
    }
    // the agent weights go to LDS with constant indices: indexing the
    // argument block by the look would make a private copy of it
    if (tid == 0) {
#pragma unroll
        for (int j = 0; j < 64; ++j) ups[j] = f.ups[j];
    }
    float2* rb = L.buf + (tid / TR) * RS;
    float* xo = keep;                  // xo[k * kst + kl]
    float* wb = keep + PX * kst;       // wb[k * kst + kl]
    float sr[PX], e2[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) sr[k] = e2[k] = 0.f;
    if (part == 0) {
        // all loads issued before the first is used (inactive rows read row 0)
        float a0[PX], a1[PX];
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            const int x = t + k * TR;
            const size_t i = pix + x;
            a0[k] = ld_stream(f.xbar + i);
            a1[k] = ld_stream(f.wbar + i);
        }
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            xo[k * kst + kl] = a0[k];
            wb[k * kst + kl] = a1[k];
        }
    }
    __syncthreads();
    uint32_t fb = 0u;
    // the block's waves stay on the same look, held there by its sum (mann_lockstep)
    const bool lockstep = split == 1 && (NX == 32 || NX == 512 || (NX <= 128 && f.lockstep));
    // the wave's row buffers, which also take its r_l (rx[k * 64 + lane])
    float* rx = reinterpret_cast<float*>(rb) - (lane / TR) * 2 * RS;
    static_assert(PX * 64 * sizeof(float) <= RPW * RS * sizeof(float2), "a wave's row buffers hold its r_l");
    for (int l0 = 0; l0 < a.looks; l0 += split) {
        const int l = l0 + part;
        if (l < a.looks) {
            const size_t img = (size_t)l * n + pix;
            const size_t band = ((size_t)l * s.nz + slice) * s.ny * s.Bs + band_row_off(arow - slice * s.ny, s.ny);
            using In = RowIn<NX>;
            float2 in[In::kCount], h[PX];
            {
                const bool has = active && In::has(t);
                float2 bin[In::kCount];
                int bp[In::kCount];
#pragma unroll
                for (int q = 0; q < In::kCount; ++q) {
                    bp[q] = has ? L.bpos[t + q * In::kStep] : -1;
                    bin[q] = ld_stream(a.band_in + band + (bp[q] >= 0 ? bp[q] : 0));
                }
#pragma unroll
                for (int q = 0; q < In::kCount; ++q) in[q] = bp[q] >= 0 ? bin[q] : make_float2(0.f, 0.f);
            }
            row_fft_in<NX, +1, true>(in, h, rb, t, L.tw);
            float2 m[PX];
            float rp[PX], uv[PX];
            if (active) {
#pragma unroll
                for (int k = 0; k < PX; ++k) {
                    const int x = t + k * TR;
                    m[k] = ld_stream(&a.mu[img + x]);
                    rp[k] = ld_stream(&a.r[img + x]);
                    uv[k] = ld_stream(&f.u[img + x]);
                }
            }
            const float gamma = (float)a.diag[(size_t)l * kDiag];
            const float ul = ups[l];
            float wm1 = 0.f;
            if (active) {
#pragma unroll
                for (int k = 0; k < PX; ++k) {
                    const int x = t + k * TR;
                    const float2 ahr = cscale(h[k], a.scale);
                    const float r0 = rp[k];
                    const float om = 1.f / (r0 + a.floor_w);
                    const float2 d = make_float2(ahr.x * a.inv_s2w - om * m[k].x, ahr.y * a.inv_s2w - om * m[k].y);
                    const float2 m1 = make_float2(m[k].x + gamma * d.x, m[k].y + gamma * d.y);
                    st_stream(&a.mu[img + x], m1);
                    const float v = uv[k] + f.two_rho * xo[k * kst + kl];
                    const float rn = r_update_voxel<MODE>(a, bv, r0, v, m1, fb);
                    st_stream(&a.r[img + x], rn);
                    st_stream(&f.u[img + x], v - f.two_rho * rn);
                    if (split == 1) {
                        sr[k] = fmaf(ul, rn, sr[k]);
                        const float e = rn - wb[k * kst + kl];
                        e2[k] = fmaf(e, e, e2[k]);
                    } else {
                        // over elements that other lanes of the wave took the transform's
                        // last inputs from: the transform synchronised after reading them
                        rx[k * 64 + lane] = rn;
                    }
                    wm1 += om * cabs2(m1);
                }
            }
            if (lockstep) {
                const double acc[1] = {wm1};
                block_sum_store<1>(acc, a.part + (size_t)l * nblk + blk);
            } else {
                // the wave's share of the look's sum omega |mu'|^2 (no wait for
                // the other waves here)
                const double acc = wave_sums_f64<1>({(double)wm1});
                if (lane == 0) wsum[l][wave] = acc;
            }
        }
        if (split > 1) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                if ((k & (split - 1)) != part) continue;
                for (int w = 0; w < split && l0 + w < a.looks; ++w) {
                    // the group's wave w: its buffers lie w - part waves from this one's
                    const float rn = rx[(w - part) * (2 * RPW * RS) + k * 64 + lane];
                    sr[k] = fmaf(ups[l0 + w], rn, sr[k]);
                    const float e = rn - wb[k * kst + kl];
                    e2[k] = fmaf(e, e, e2[k]);
                }
            }
            __syncthreads();  // the buffers are free for the next turn's transforms
        }
    }
    __syncthreads();
    if (!lockstep && tid < a.looks) {
        // in wave order; of a group's waves only one took this look
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (w % split == tid % split) acc += wsum[tid][w];
        a.part[(size_t)tid * nblk + blk] = acc;
    }
    const bool prior = f.wprior != nullptr;
    const float up = prior ? ups[a.looks] : 0.f;
    const float N = (float)f.n_agents;
    double num = 0.0, den = 0.0;
    // the prior agent's output and w, every load issued before the first is
    // used (without a prior the loads read x_bar, with weight 0, and nothing
    // of them is stored)
    float rpv[PX], wpv[PX];
    {
        const float* rsrc = prior ? f.rprior : f.xbar;
        const float* wsrc = prior ? f.wprior : f.xbar;
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            if ((k & (split - 1)) != part) continue;
            const int x = t + k * TR;
            const size_t i = pix + x;
            rpv[k] = rsrc[i];
            wpv[k] = ld_stream(wsrc + i);
        }
    }
    if (active) {
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            if ((k & (split - 1)) != part) continue;
            const int x = t + k * TR;
            const float wbk = wb[k * kst + kl];
            const float e = rpv[k] - wbk;
            const float s_r = prior ? sr[k] + up * rpv[k] : sr[k];
            const float nm = e2[k] + (prior ? e * e : 0.f);
            const float xb = 2.f * s_r - wbk;
            if (prior) st_stream(f.wprior + pix + x, wpv[k] + f.two_rho * (xb - rpv[k]));
            st_stream(f.xbar + pix + x, xb);
            st_stream(f.wbar + pix + x, wbk + f.two_rho * (s_r - wbk));
            num += (double)nm;
            den += (double)N * ((double)wbk * wbk);
        }
    }
    wave_or_fault(fb, a.fault);
    double acc2[2] = {num, den};
    block_sum_store<2>(acc2, f.part + (size_t)blk * 2);
}

// ---------------------------------------------------------------------------
// Inverse column pass of one tile from the column-major compact layout: the
// tile's columns are transformed and written as band columns.  `item` =
// zl * tiles + tile, which is also the partial-sum slot of the scene.
template <int NY, class A>
__device__ __forceinline__ void col_inv_item(const A& a, int item, float2* tw, float2* tile,
                                             bool load_tables) {
    constexpr int TC = col_tile_cols(NY);
    constexpr int TPC = kBlock / TC;
    const auto& s = a.s;
    const int tid = threadIdx.x;
    const int tile_i = item % s.tiles;
    const int zl = item / s.tiles;  // look * nz + z
    const int c0 = tile_i * TC;
    // the twiddles (when this block loads them) travel with the first loads,
    // not after the barrier
    constexpr int TWL = (NY + kBlock - 1) / kBlock;
    float2 twv[TWL];
    if (load_tables) {
#pragma unroll
        for (int j = 0; j < TWL; ++j) {
            const int i = tid + j * kBlock;
            twv[j] = s.tw_y[i < NY ? i : 0];
        }
    }
    const float2* src = a.cmp_in + (size_t)zl * s.P;
    const int co = tid % TC, bo = c0 + co;
    float2* dst = a.band_out + (size_t)zl * s.ny * s.Bs + (size_t)tile_i * s.ny * TC + co;  // the tile's block
    double acc[1] = {0.0};
    if constexpr (fft_regs_ok<NY, TPC>()) {
        // Each thread fetches its own transform inputs, rows tid / TC + k TPC
        // of band column bo, straight into registers: the compact index of
        // each from pidxb (-1 off the pupil), then the samples, every load
        // issued before the first is used.  No tile to clear, no scatter
        // through LDS.
        constexpr int PT = NY / TPC;
        const int yo = tid / TC;
        const bool col = bo < s.B;
        int pi[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) pi[k] = col ? s.pidxb[(size_t)(yo + k * TPC) * s.Bs + bo] : -1;
        float2 h[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) h[k] = src[pi[k] >= 0 ? pi[k] : 0];
        float f = 0.f;
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            if (pi[k] < 0) h[k] = make_float2(0.f, 0.f);
            f += cabs2(h[k]);
        }
        acc[0] = f;
        __syncthreads();  // the previous item's readers of the LDS buffers are done
        if (load_tables) {
#pragma unroll
            for (int j = 0; j < TWL; ++j) {
                const int i = tid + j * kBlock;
                if (i < NY) tw[i] = twv[j];
            }
        }
        // the transform opens with a block barrier (the twiddles are then in
        // place); its last stage leaves each thread rows yo + k TPC, which it
        // stores into the tile's block
        fft_regs<NY, TPC, +1, 0, true, true, false>(h, tile + co, TC, yo, tw);
        if (col) {
#pragma unroll
            for (int k = 0; k < PT; ++k) st_stream(dst + (size_t)(yo + k * TPC) * TC, cscale(h[k], a.scale));
        }
    } else {
        // Scatter of column bc's pupil samples p in [p0, p1): lane l takes
        // p0 + l, p0 + l + TPC, ..., all loads issued before the first is
        // used (positions past p1 re-read the column's last sample and are
        // dropped); a column holds at most NY = CH * TPC samples, so one
        // chunk, loaded before the tile is cleared, covers it.
        constexpr int CH = NY / TPC;
        const int c = tid / TPC, lane = tid % TPC, bc = c0 + c;
        int p0 = 0, p1 = 0;
        if (bc < s.B) {
            p0 = s.col_off[bc];
            p1 = s.col_off[bc + 1];
        }
        float2 v[CH];
        int ry[CH];
        const int base = p0 + lane;
        if (base < p1) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int p = base + k * TPC;
                const int pc = p < p1 ? p : p1 - 1;
                v[k] = src[pc];
                ry[k] = s.row_idx[pc];
            }
        }
        __syncthreads();  // the previous item's readers of the LDS buffers are done
        if (load_tables) {
#pragma unroll
            for (int j = 0; j < TWL; ++j) {
                const int i = tid + j * kBlock;
                if (i < NY) tw[i] = twv[j];
            }
        }
        for (int i = tid; i < NY * TC; i += kBlock) tile[i] = make_float2(0.f, 0.f);
        __syncthreads();
        float f = 0.f;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            if (base + k * TPC < p1) {
                tile[ry[k] * TC + c] = v[k];
                f += cabs2(v[k]);
            }
        }
        acc[0] = f;
        fft_lds<NY, TPC, +1>(tile + co, TC, tid / TC, tw);
        if (bo < s.B)
            for (int y = tid / TC; y < NY; y += TPC) st_stream(dst + (size_t)y * TC, cscale(tile[y * TC + co], a.scale));
    }
    if (a.part != nullptr) block_sum_store<1>(acc, a.part + item);
}

// Forward column pass over a stream of items (all of column length NY): the
// block walks items first, first + stride, ..., keeping the next item's band
// rows in registers, loaded while the current item's column FFTs run.
// `item_of(i)` returns the (ColArgs, scene item index) of stream position i.
// The twiddle table must already be in `tw` (it depends on NY only).
template <int NY, class ItemOf>
__device__ __forceinline__ void col_fwd_stream(int first, int count, int stride, ItemOf item_of, const float2* tw,
                                               float2* tile) {
    constexpr int TC = col_tile_cols(NY);
    constexpr int TPC = kBlock / TC;
    constexpr int PT = NY / TPC;
    static_assert(NY % TPC == 0, "column length must be a multiple of the threads per column");
    const int tid = threadIdx.x;
    const int c_ld = tid % TC, y_ld = tid / TC;
    float2 pre[PT];
    auto load = [&](int pos) {
        const auto ai = item_of(pos);
        const auto& a = ai.get();
        const auto& s = a.s;
        const int bc = (ai.item % s.tiles) * TC + c_ld;
        // the tile's contiguous block of the band buffer
        const float2* src = a.band_in + (size_t)(ai.item / s.tiles) * s.ny * s.Bs +
                            (size_t)(ai.item % s.tiles) * s.ny * TC + c_ld;
#pragma unroll
        for (int k = 0; k < PT; ++k)
            pre[k] = bc < s.B ? src[(size_t)(y_ld + k * TPC) * TC] : make_float2(0.f, 0.f);
    };
    int pos = first;
    if (pos < count) load(pos);
    for (; pos < count; pos += stride) {
        const auto ai = item_of(pos);
        const auto& a = ai.get();
        const auto& s = a.s;
        const int tile_i = ai.item % s.tiles;
        const int zl = ai.item / s.tiles;
        // the item's band rows move to h (rows y_ld + k TPC of column c_ld),
        // and pre is free for the next item's prefetch
        float2 h[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) h[k] = pre[k];
        // Rows of column bc's pupil samples p0 + lane + k TPC (at most NY =
        // PT * TPC of them), loaded before the next item's prefetch so that
        // waiting for them does not wait for it; positions past p1 re-read
        // the column's last row and are not stored.
        const int c = tid / TPC, lane = tid % TPC, bc = tile_i * TC + c;
        int p0 = 0, p1 = 0;
        int ry[PT];
        if (bc < s.B) {
            p0 = s.col_off[bc];
            p1 = s.col_off[bc + 1];
#pragma unroll
            for (int k = 0; k < PT; ++k) {
                const int p = p0 + lane + k * TPC;
                ry[k] = s.row_idx[p < p1 ? p : p1 - 1];
            }
        }
        if (pos + stride < count) load(pos + stride);
        // the transform's opening block barrier also orders it after the
        // previous item's readers of `tile`
        if constexpr (fft_regs_ok<NY, TPC>()) {
            fft_regs<NY, TPC, -1, 0, true, false, false>(h, tile + c_ld, TC, y_ld, tw);
        } else {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PT; ++k) tile[(y_ld + k * TPC) * TC + c_ld] = h[k];
            fft_lds<NY, TPC, -1>(tile + c_ld, TC, y_ld, tw);
        }
        double acc[1] = {0.0};
        if (bc < s.B) {
            float2* dst = a.cmp_out + (size_t)zl * s.P;
            float f = 0.f;
#pragma unroll
            for (int k = 0; k < PT; ++k) {
                const int p = p0 + lane + k * TPC;
                if (p < p1) {
                    const float2 val = cscale(tile[ry[k] * TC + c], a.scale);
                    dst[p] = val;
                    f += cabs2(val);
                }
            }
            acc[0] = f;
        }
        if (a.part != nullptr) block_sum_store<1>(acc, a.part + ai.item);
    }
}

// ---------------------------------------------------------------------------
// The three passes up to the step size on one slice of one look, for slices
// whose band fits in LDS: inverse column FFTs of the pupil samples, the
// gradient row pass, forward column FFTs back onto the pupil.  The band
// columns live in S (row y, band column b at slice_pos) from the first pass
// to the last, with the arithmetic and the float32 groups of the partial sums
// of the three passes; the only band traffic to memory is the copy the update
// pass reads.  NY / 8 threads hold a column, NX / 8 a row, both inside one
// wave, so block barriers stand only between the passes.  Small scenes are bound by
// the chain of dependent launches, about 4 us each: one iteration of 64x64x32
// with 8 looks and the Gaussian prior took 87 us and takes 54 us with this
// pass, the shared looks of row_update_mann and the joined final sums;
// 32x32x16 with 4 looks, forward agents only, 46 and 30 us.
template <int NX, int NY>
struct SliceGeo {
    static constexpr int TY = NY / 8, TR = NX / 8;      // threads per column, per row
    static constexpr int CPW = 64 / TY, RPW = 64 / TR;  // columns and rows per wave
    static constexpr int NT = NX * NY / 8 < 128 ? 128 : NX * NY / 8 > 1024 ? 1024 : NX * NY / 8;
    static constexpr int NW = NT / 64;
    static constexpr int RS = lds_len<NX, kRowPad>();
    static_assert(NY % (NW * RPW) == 0, "the block's waves share the rows evenly");
};

// Row stride of S: an odd multiple of the columns per wave, at least B, so
// that the 64 / TY columns of TY consecutive rows spread over the LDS banks;
// every eighth row shifts by as much again, for the autosort stores, whose
// rows are eight apart.
__host__ __device__ constexpr int slice_stride(int cpw, int B) {
    const int m = (B + cpw - 1) / cpw;
    return cpw * (m | 1);
}
__host__ __device__ constexpr int slice_pos(int y, int b, int stride, int cpw) {
    return y * stride + (y >> 3) * cpw + b;
}

// Dynamic LDS of the slice pass in bytes: S, the waves' row buffers, the two
// twiddle tables, the band column tables.
template <int NX, int NY>
__host__ __device__ constexpr size_t slice_lds_bytes(int B) {
    using G = SliceGeo<NX, NY>;
    const int st = slice_stride(G::CPW, B);
    return ((size_t)slice_pos(NY - 1, 0, st, G::CPW) + st + (size_t)G::NW * G::RPW * G::RS + NX + NY) * sizeof(float2) +
           2 * (size_t)NX * sizeof(int);
}

// Sums of K doubles over a block of NT threads, in a fixed order; thread 0
// gets them.
template <int K, int NT>
__device__ __forceinline__ void block_sums(double (&v)[K]) {
    __shared__ double red[K][NT / 64];
    wave_sums_store(v, red);
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NT / 64; ++w) s += red[k][w];
            v[k] = s;
        }
    }
}

// zl = look * nz + z.  Partial sums, one set per slice: prow (||d||^2, sum
// omega |d|^2, sum omega |mu|^2), pci (||resid||^2 of the slice), pcf
// (||A d||^2); pci and pcf may be NULL (3D operator: its range passes sum).
template <int NX, int NY, class A>
__device__ __forceinline__ void slice_grad_item(const A& a, int zl, float2* lds) {
    using G = SliceGeo<NX, NY>;
    constexpr int TY = G::TY, TR = G::TR, CPW = G::CPW, RPW = G::RPW, NT = G::NT, NW = G::NW, RS = G::RS;
    const auto& s = a.s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int B = s.B, st = slice_stride(CPW, B);
    float2* S = lds;
    float2* rbuf = S + slice_pos(NY - 1, 0, st, CPW) + st;
    float2* twx = rbuf + NW * RPW * RS;
    float2* twy = twx + NX;
    int* bidx = reinterpret_cast<int*>(twy + NY);  // band column of a column, -1 outside the band
    int* bcol = bidx + NX;
    for (int i = tid; i < NX; i += NT) {
        twx[i] = s.tw_x[i];
        const int off = s.band_pos[i];  // band_col_off of the column: tile * 16 ny + column in the tile
        bidx[i] = off < 0 ? -1 : off / (16 * NY) * 16 + (off & 15);
        const int bc = s.band_cols[i < B ? i : 0];
        bcol[i] = i < B ? bc : 0;
    }
    for (int i = tid; i < NY; i += NT) twy[i] = s.tw_y[i];

    // columns: lane (ct, cc) holds rows ct + k TY of column g CPW + cc
    const int cc = lane % CPW, ct = lane / CPW;
    const float2* src = a.cmp_in + (size_t)zl * s.P;
    double r2 = 0.0;
    // the pointwise streams of the wave's first rows, loaded behind the column pass
    const int ri = lane / TR, t = lane % TR;
    float2 m[8];
    float rp[8];
    auto load_streams = [&](int y) {
        const size_t img = ((size_t)zl * NY + y) * NX + t;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            m[k] = a.mu[img + k * TR];
            rp[k] = a.r[img + k * TR];
        }
    };
    load_streams(wave * RPW + ri);
    __syncthreads();
    for (int g = wave; g * CPW < B; g += NW) {
        const int c = g * CPW + cc;
        const bool ok = c < B;
        int pi[8];
        float2 h[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) pi[k] = ok ? s.pidxb[(size_t)(ct + k * TY) * s.Bs + c] : -1;
#pragma unroll
        for (int k = 0; k < 8; ++k) h[k] = src[pi[k] >= 0 ? pi[k] : 0];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (pi[k] < 0) h[k] = make_float2(0.f, 0.f);
        // ||resid||^2 of the column: samples p0 + lane + 16 k in float32 sums
        // per lane of 16, rounded as the inverse column pass rounds them
        if (c < B) {
            const int p0 = s.col_off[c], p1 = s.col_off[c + 1];
            for (int ln = ct; ln < 16; ln += TY) {
                float f = 0.f;
#pragma unroll
                for (int k = 0; k < NY / 16; ++k) {
                    const int p = p0 + ln + 16 * k;
                    if (p < p1) {
                        const float2 v = src[p];
                        f += fmaf(v.y, v.y, v.x * v.x);
                    }
                }
                r2 += f;
            }
        }
        // columns past the band transform zeros in the last column's place of
        // the row padding: st >= g CPW + CPW
        const auto pos = [c, st](int y) { return slice_pos(y, c, st, CPW); };
        fft_regs_at<NY, TY, +1, true, true, true>(h, S, pos, ct, twy);
        group_sync<true>();
#pragma unroll
        for (int k = 0; k < 8; ++k) S[pos(ct + k * TY)] = cscale(h[k], a.scale_y);
    }
    __syncthreads();

    // rows: RPW rows per wave and turn
    float2* rb = rbuf + (wave * RPW + ri) * RS;
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int y0 = wave * RPW; y0 < NY; y0 += NW * RPW) {
        const int y = y0 + ri;
        float2 h[8];
        float2* brow = a.band_out + (size_t)zl * NY * s.Bs + band_row_off(y, NY);
        float2* srow = S + slice_pos(y, 0, st, CPW);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int b = bidx[t + k * TR];
            h[k] = b >= 0 ? srow[b] : make_float2(0.f, 0.f);
            if (b >= 0) st_stream(brow + band_col_off(b, NY), h[k]);
        }
        row_fft<NX, +1, true>(h, rb, t, twx);
        float dd = 0.f, wd = 0.f, wm = 0.f;
        row_grad_pointwise<true>(a, h, m, rp, dd, wd, wm);
        acc[0] += dd;
        acc[1] += wd;
        acc[2] += wm;
        if (y0 + NW * RPW < NY) load_streams(y + NW * RPW);
        row_fft<NX, -1, false>(h, rb, t, twx);
        for (int b = t; b < B; b += TR) srow[b] = cscale(rb[lds_pos<kRowPad>(bcol[b])], a.scale);
    }
    __syncthreads();

    double ad = 0.0;
    float2* dst = a.cmp_out + (size_t)zl * s.P;
    for (int g = wave; g * CPW < B; g += NW) {
        const int c = g * CPW + cc;
        float2 h[8];
        const auto pos = [c, st](int y) { return slice_pos(y, c, st, CPW); };
#pragma unroll
        for (int k = 0; k < 8; ++k) h[k] = S[pos(ct + k * TY)];
        fft_regs_at<NY, TY, -1, true, false, true>(h, S, pos, ct, twy);
        // the column's pupil samples p0 + lane + 16 k, float32 sums per lane
        // of 16, as the forward column pass stores and sums them
        if (c < B) {
            const int p0 = s.col_off[c], p1 = s.col_off[c + 1];
            for (int ln = ct; ln < 16; ln += TY) {
                float f = 0.f;
#pragma unroll
                for (int k = 0; k < NY / 16; ++k) {
                    const int p = p0 + ln + 16 * k;
                    if (p < p1) {
                        const float2 v = cscale(S[pos(s.row_idx[p])], a.scale_y);
                        dst[p] = v;
                        f += cabs2(v);
                    }
                }
                ad += f;
            }
        }
    }
    acc[3] = ad;
    acc[4] = r2;
    block_sums<5, NT>(acc);
    if (tid == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) a.prow[(size_t)zl * 3 + k] = acc[k];
        if (a.pcf != nullptr) {
            a.pcf[zl] = acc[3];
            a.pci[zl] = acc[4];
        }
    }
}

// Column-pass item handles for col_fwd_stream: by pointer (kernel
// arguments) or by private copy (arguments read from device memory).
struct ColItemRef {
    const ColArgs* args;
    int item;
    __device__ const ColArgs& get() const { return *args; }
};
struct ColItemVal {
    ColArgs args;
    int item;
    __device__ const ColArgs& get() const { return args; }
};
struct ColItemConst {
    ConstAS<ColArgs>* args;
    int item;
    __device__ ConstAS<ColArgs>& get() const { return *args; }
};

// ---------------------------------------------------------------------------
// Exact step size of one look from the partial sums of the three passes, and
// h before the mu-step: h = ||resid||^2 / (2 sigma_w^2) + sum omega |mu|^2 / 2,
// which is eq. mu-objective less the constant ||(1 - a) y||^2 / (2 sigma_w^2)
// of the samples off the pupil.  Look 0 also zeroes the counter of looks the
// diagnostics pass has finished.
__device__ __forceinline__ void gamma_item(int look, const GammaArgs& a) {
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    strided_sums<3>(a.prow + (size_t)look * a.nrow * 3, a.nrow, 3, v);
    strided_sums<1>(a.pcf + (size_t)look * a.ncol, a.ncol, 1, v + 3);
    strided_sums<1>(a.pci + (size_t)look * a.ncol, a.ncol, 1, v + 4);
    __shared__ double tot[5];
    block_sum_store<5>(v, tot);
    if (threadIdx.x == 0) {
        const double dd = tot[0], wd = tot[1], wm = tot[2], ad = tot[3], r2 = tot[4];
        const double den = ad * a.inv_s2w + wd;
        const double g = dd > 0.0 ? dd / den : 0.0;
        double* o = a.diag + (size_t)look * kDiag;
        o[DG_GAMMA] = g;
        o[DG_DD] = dd;
        o[DG_AD] = ad;
        o[DG_H0] = 0.5 * (r2 * a.inv_s2w + wm);
        o[DG_WD] = wd;
        if (!(g >= 0.0) || !isfinite(g)) atomicOr(a.fault, 4u | 1u);
        if (look == 0) *a.counter = 0u;
    }
}

// resid -= gamma D(a) F d over entries [begin, end) of one look; returns the
// thread's share of ||resid||^2.
__device__ __forceinline__ float resid_range(float2* R, const float2* D, float g, size_t begin, size_t end,
                                             size_t stride) {
    float f = 0.f;
    for (size_t i = begin + threadIdx.x; i < end; i += stride) {
        float2 x = ld_stream(R + i);
        const float2 d = ld_stream(D + i);
        x.x -= g * d.x;
        x.y -= g * d.y;
        st_stream(R + i, x);
        f += cabs2(x);
    }
    return f;
}

// Diagnostics after the mu-step of one look: h after (the same omega as h
// before, so h before - h after = gamma ||d||^2 / 2 up to rounding), the
// look's mu-residual of eq. residual in its noise-floored form, ||d|| /
// ||A^H y / sigma_w^2|| with d the gradient the step used (0 without
// ||A^H y||^2), and ||resid||^2.  The block that finishes the last look of the
// call writes the summary row diag[looks]: the mu-residual averaged over looks
// (eq. residual), and the sums of h before and after, in look order.
__device__ __forceinline__ void diag_after_item(int look, const DiagArgs& a) {
    double v[2] = {0.0, 0.0};
    strided_sums<1>(a.pupd + (size_t)look * a.nrow, a.nrow, 1, v);
    strided_sums<1>(a.pres + (size_t)look * a.nres, a.nres, 1, v + 1);
    __shared__ double tot[2];
    block_sum_store<2>(v, tot);
    __shared__ int last;
    if (threadIdx.x == 0) {
        double* o = a.diag + (size_t)look * kDiag;
        o[DG_H1] = 0.5 * (tot[1] / a.s2w + tot[0]);
        o[DG_R2] = tot[1];
        double m2 = 0.0;
        if (a.ahy2 != nullptr) {
            const double y2 = a.ahy2[look];
            m2 = y2 > 0.0 ? a.s2w * sqrt(o[DG_DD] / y2) : 0.0;
        }
        o[DG_MURES] = m2;
        __threadfence();  // this look's row is visible before it is counted
        last = atomicAdd(a.counter, 1u) == (unsigned)(a.looks - 1);
    }
    __syncthreads();
    if (last) {
        // every look's row is written: one thread per look reads its row, and
        // thread 0 sums them in look order
        __shared__ double rows[3][kBlock];
        __threadfence();
        const volatile double* d = a.diag;
        for (int l0 = 0; l0 < a.looks; l0 += kBlock) {
            const int l = l0 + (int)threadIdx.x;
            if (l < a.looks) {
                rows[0][threadIdx.x] = d[(size_t)l * kDiag + DG_MURES];
                rows[1][threadIdx.x] = d[(size_t)l * kDiag + DG_H0];
                rows[2][threadIdx.x] = d[(size_t)l * kDiag + DG_H1];
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                double m = l0 == 0 ? 0.0 : a.diag[(size_t)a.looks * kDiag + 0];
                double h0 = l0 == 0 ? 0.0 : a.diag[(size_t)a.looks * kDiag + 1];
                double h1 = l0 == 0 ? 0.0 : a.diag[(size_t)a.looks * kDiag + 2];
                const int cnt = a.looks - l0 < kBlock ? a.looks - l0 : kBlock;
                for (int i = 0; i < cnt; ++i) {
                    m += rows[0][i];
                    h0 += rows[1][i];
                    h1 += rows[2][i];
                }
                double* srow = a.diag + (size_t)a.looks * kDiag;
                srow[0] = m;
                srow[1] = h0;
                srow[2] = h1;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            double* srow = a.diag + (size_t)a.looks * kDiag;
            srow[0] /= a.looks;
            for (int k = 3; k < kDiag; ++k) srow[k] = 0.0;
        }
    }
}

// Convergence error of the Mann step from its block partials.
__device__ __forceinline__ void mace_final_item(const double* part, int blocks, double* conv) {
    double v[2] = {0.0, 0.0};
    strided_sums<2>(part, blocks, 2, v);
    __shared__ double tot[2];
    block_sum_store<2>(v, tot);
    if (threadIdx.x == 0) conv[0] = tot[1] > 0.0 ? sqrt(tot[0] / tot[1]) : 0.0;
}

// Mann step of voxel i with every agent's w and r in registers (NA >=
// n_agents); returns (sum_j (r_j - w_bar)^2, n_agents w_bar^2).  The loads
// are unconditional so that all of them are in flight at once: padding agents
// re-read the last agent and carry weight 0 (ups[j] = 0 for j >= n_agents).
template <int NA>
__device__ __forceinline__ void mace_voxel(const MaceArgs& a, const float* ups, unsigned n, unsigned i, double& num,
                                           double& den) {
    float wv[NA], rv[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const size_t base = (size_t)(j < a.n_agents ? j : a.n_agents - 1) * n;
        wv[j] = ld_stream(a.w + base + i);
        rv[j] = ld_stream(a.r + base + i);
    }
    float wb = 0.f, rb = 0.f;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        wb += ups[j] * wv[j];
        rb += ups[j] * rv[j];
    }
    const float xb = 2.f * rb - wb;
    float wbn = 0.f, nm = 0.f;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        if (j < a.n_agents) {
            const float dr = rv[j] - wb;
            nm += dr * dr;
            const float wn = wv[j] + a.two_rho * (xb - rv[j]);
            st_stream(a.w + (size_t)j * n + i, wn);
            wbn += ups[j] * wn;
        }
    }
    st_stream(a.wbar + i, wbn);
    num += nm;
    den += (double)a.n_agents * wb * wb;
}

// Periodic 7-tap Gaussian smoothing along z, y and x in one pass over the
// volume: one call produces an output tile of kGaussTY rows x TX voxels over
// CZ range slices z0 .. z0 + CZ - 1.  Tiles are numbered z chunk fastest,
// then x, then y: tile t has bz = t % zc, bx = (t / zc) % (nx / TX),
// by = t / (zc nx / TX), so that consecutive tiles share their halos.  Every
// (kGaussTY + 6) x (TX + 6) window of the input slices z0 - 3 .. z0 +
// CZ + 2 is loaded into registers up front, so that the block waits
// for memory once, not once per slice, and is filtered along z there, each
// thread over its own window positions.  The z-filtered window goes to LDS and
// is filtered along x, then along y (the separable filter's three passes
// commute), as a pipeline: in phase o the block filters output slice o along
// z, slice o - 1 along x and slice o - 2 along y, with one barrier per phase
// and both LDS windows double-buffered.  A thread filters four adjacent x (ten
// LDS values in three 16-byte reads) and adjacent rows of one column, instead of
// seven values read per result: a tile's serial chain bounds the pass on small
// volumes (128^3: 17.7 -> 15.1 us, 384x192x37: 20.0 -> 18.3), the windows'
// traffic on large ones (gauss_slices).
// p holds nx, ny, nz (ny a multiple of kGaussTY, nx of TX), the taps g[7], in
// and out (not overlapping).
template <int TX>
__host__ __device__ constexpr int gauss_in_floats() { return (kGaussTY + 6) * (TX + 8); }  // one of two windows
template <int TX>
__host__ __device__ constexpr int gauss_xf_floats() { return (kGaussTY + 6) * TX; }

// f(0), ..., f(N - 1) with compile-time indices.
template <int N, int I = 0, class F>
__device__ __forceinline__ void for_each_index(F& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        for_each_index<N, I + 1>(f);
    }
}

template <int TX, int CZ, class P>
__device__ __forceinline__ void gauss3d_tile(const P& p, int tile, float (&tin)[2][gauss_in_floats<TX>()],
                                             float (&txf)[2][gauss_xf_floats<TX>()]) {
    constexpr int W = TX + 6, WS = TX + 8, H = kGaussTY + 6;  // window, its row stride in LDS
    constexpr int NIN = H * W;
    constexpr int LPT = (NIN + kBlock - 1) / kBlock;
    constexpr int NZW = CZ + 6;  // input slices of a chunk
    constexpr int XT = H * TX / 4;                                          // threads of the x filter
    constexpr int OPT = kGaussTY * TX / kBlock > 1 ? kGaussTY * TX / kBlock : 1;  // rows per thread of the y filter
    static_assert(XT <= kBlock && kGaussTY % OPT == 0 && kGaussTY / OPT * TX <= kBlock, "a tile divides among the threads");
    const int nx = p.nx, ny = p.ny, nz = p.nz;
    const float* in = p.in;
    float* out = p.out;
    float g[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) g[k] = p.g[k];
    const int tid = threadIdx.x;
    const int zc = (nz + CZ - 1) / CZ, tx = nx / TX;
    const int bz = tile % zc, bx = (tile / zc) % tx, by = tile / (zc * tx);
    const int x0 = bx * TX, y0 = by * kGaussTY, z0 = bz * CZ;
    const int slices = z0 + CZ < nz ? CZ : nz - z0;
    const unsigned slice = (unsigned)nx * (unsigned)ny;
    unsigned goff[LPT];
    int loff[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int e = tid + j * kBlock;
        const int r = (e < NIN ? e : 0) / W, c = (e < NIN ? e : 0) % W;
        int gy = y0 - 3 + r, gx = x0 - 3 + c;
        gy = gy < 0 ? gy + ny : (gy >= ny ? gy - ny : gy);
        gx = gx < 0 ? gx + nx : (gx >= nx ? gx - nx : gx);
        goff[j] = (unsigned)gy * nx + gx;
        loff[j] = r * WS + c;
    }
    // the chunk's input windows, all loads issued before the first is used
    // (in a chunk cut short by the end of the volume the slices past it wrap
    // periodically and are not used)
    float pre[NZW][LPT];
#pragma unroll
    for (int sl = 0; sl < NZW; ++sl) {
        int zz = (z0 - 3 + sl) % nz;
        zz = zz < 0 ? zz + nz : zz;
        const float* src = in + (size_t)zz * slice;
#pragma unroll
        for (int j = 0; j < LPT; ++j) pre[sl][j] = src[goff[j]];
    }
    const int xr = tid / (TX / 4), xc = tid % (TX / 4) * 4;  // x filter: row and first of four x
    const int yx = tid % TX, yr = tid / TX * OPT;            // y filter: column and first row
    __syncthreads();  // the previous tile's readers of the windows are done
    auto phase = [&](auto phase_index) {
        constexpr int o = decltype(phase_index)::value;
        if (o >= slices + 2) return;  // uniform over the block
        if constexpr (o < CZ) {
            if (o < slices) {
#pragma unroll
                for (int j = 0; j < LPT; ++j) {
                    float acc = 0.f;
#pragma unroll
                    for (int k = 0; k < 7; ++k) acc += g[k] * pre[o + k][j];
                    if (tid + j * kBlock < NIN) tin[o & 1][loff[j]] = acc;
                }
            }
        }
        if (o >= 1 && o - 1 < slices && tid < XT) {
            const float* row = &tin[(o - 1) & 1][xr * WS + xc];
            float v[12];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const float4 w = *reinterpret_cast<const float4*>(row + 4 * q);  // the last two are not used
                v[4 * q] = w.x, v[4 * q + 1] = w.y, v[4 * q + 2] = w.z, v[4 * q + 3] = w.w;
            }
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < 7; ++k) acc[i] += g[k] * v[i + k];
            *reinterpret_cast<float4*>(&txf[(o - 1) & 1][xr * TX + xc]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
        if (o >= 2 && tid < kGaussTY / OPT * TX) {
            float v[OPT + 6];
#pragma unroll
            for (int k = 0; k < OPT + 6; ++k) v[k] = txf[o & 1][(yr + k) * TX + yx];
            float* dst = out + (size_t)(z0 + o - 2) * slice + (size_t)(y0 + yr) * nx + x0 + yx;
#pragma unroll
            for (int q = 0; q < OPT; ++q) {
                float acc = 0.f;
#pragma unroll
                for (int k = 0; k < 7; ++k) acc += g[k] * v[q + k];
                dst[(size_t)q * nx] = acc;
            }
        }
        __syncthreads();
    };
    for_each_index<CZ + 2>(phase);
}

}  // namespace clampk
