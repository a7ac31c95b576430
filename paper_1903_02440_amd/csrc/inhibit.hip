// Pointwise inhibition and pooling of potentials (gfx950).
//
// Paper: section "functional Module" (pointwise inhibition: at each location
// only the neuron of the most salient feature -- the earliest spike, then the
// highest potential -- may spike) and section "snn Module" (pooling applied
// to a potentials tensor keeps the largest potential of each window).
#include <algorithm>

#include "common.hpp"

namespace {

constexpr int PW_THREADS = 512;
constexpr int PW_LOC = 1024;    // locations of a workgroup at most
constexpr int PW_SPLITS = 32;   // threads per 4 locations in the scan at most
constexpr int PW_U = 8;         // features per block of loads in the scan

// 4 values at any alignment, as one access where the hardware allows it.
struct __attribute__((packed, aligned(1))) Byte4u {
    uint32_t w;
};
struct __attribute__((packed, aligned(4))) Float4u {
    float v[4];
};

// Grid: (part, run of up to PW_LOC locations, image), from run u0 of all images' on.  The workgroup first finds
// the winner of each of its locations over the C features (the kWTA order:
// earlier spike, then larger potential, then lower feature index), 4 locations
// and every n-th feature per thread, the threads' findings joined in LDS.  Then
// it writes its part of the (feature, 4 locations) items: the surviving
// first-spike time and potential, and, when asked, the survivors' Eq.1 wave and
// zeros over the potentials of every feature that is no winner.  Nearly all of
// that is constant, so nothing is read again.  All inputs of the locations are
// read before any output is written and the parts of a run are only more than
// one when no output lies over an input, so the outputs may alias the inputs
// (the first-spike ones, or at one step the wave and the potentials).
// Bound by the writes (5 (1 + T) bytes a neuron with wave and potentials).  With
// one thread per 4 locations doing all of it (k_pointwise_each), 200 images of 250
// maps of 14x14 keep 39 workgroups busy and read the potentials: 1444 us; this form
// 245 us (833 MB, 3.4 TB/s).  256 or 1024 threads per workgroup 265 and 280 us;
// items in the inner loop, steps in the outer one 280 us.
//
// A potential that is no number never replaces another one, and is replaced by
// none at the same step when it comes first: the scan keeps the first feature of
// the earliest step and whether its potential is a number beside the best one.
struct PwBest {
    int t, c, first;  // step, best feature (-1: none), 2 * first feature + [its potential is no number]
    float v;
};
__device__ __forceinline__ void pw_join(PwBest &a, int t, int c, int first, float v) {
    if (first < 0 || t > a.t) return;
    if (t < a.t || a.first < 0) {
        a = PwBest{t, c, first, v};
        return;
    }
    a.first = min(a.first, first);
    if (c >= 0 && (a.c < 0 || v > a.v || (v == a.v && c < a.c))) {
        a.c = c;
        a.v = v;
    }
}

// I holds the bytes of an image's potentials.
template <typename I>
__global__ __launch_bounds__(PW_THREADS, 4) void k_pointwise(const uint8_t *tf, const float *vf, int T, int C, I HW,
                                                             int64_t u0, int64_t nrun, int parts, uint8_t *out_t,
                                                             float *out_v, uint8_t *wave, float *pot) {
    extern __shared__ uint4 pwsm[];  // [splits][4 nq] findings
    __shared__ __align__(16) int bc[PW_LOC];
    __shared__ float bv[PW_LOC];
    __shared__ uint8_t bt[PW_LOC];
    const int tid = threadIdx.x;
    const int part = blockIdx.x % parts;
    const int64_t u = u0 + blockIdx.x / parts, b = nrun == 1 ? u : u / nrun, p0 = (u - b * nrun) * PW_LOC;
    const int n = (int)min<int64_t>(PW_LOC, (int64_t)HW - p0), nq = (n + 3) / 4;
    const int splits = min(min(PW_SPLITS, PW_THREADS / nq), C);
    const int64_t plane = (int64_t)C * HW, base = b * plane + p0;
    tf += base;
    const char *vb = reinterpret_cast<const char *>(vf + base);
    PwBest *found = reinterpret_cast<PwBest *>(pwsm);
    if (tid < nq * splits) {
        const int sp = tid / nq, q = tid - sp * nq, nj = min(4, n - 4 * q);
        PwBest best[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) best[j] = PwBest{T, -1, -1, 0.0f};
        for (int c0 = sp; c0 < C; c0 += PW_U * splits) {
            uint32_t tw[PW_U];
            Float4u vw[PW_U];
            if (nj == 4) {
#pragma unroll
                for (int u = 0; u < PW_U; ++u) {  // (clamped: unconditional loads, all in flight)
                    const I o = (I)min(c0 + u * splits, C - 1) * HW + 4 * q;
                    tw[u] = reinterpret_cast<const Byte4u *>(tf + o)->w;
                    vw[u] = *reinterpret_cast<const Float4u *>(vb + 4 * o);
                }
            } else {
#pragma unroll
                for (int u = 0; u < PW_U; ++u) {
                    const I o = (I)min(c0 + u * splits, C - 1) * HW + 4 * q;
                    tw[u] = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const I oj = o + min(j, nj - 1);
                        tw[u] |= (uint32_t)tf[oj] << (8 * j);
                        vw[u].v[j] = *reinterpret_cast<const float *>(vb + 4 * oj);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < PW_U; ++u) {
                const int c = c0 + u * splits;
                if (c >= C) break;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = (int)((tw[u] >> (8 * j)) & 255u);
                    const float v = vw[u].v[j];
                    if (t < T) pw_join(best[j], t, v == v ? c : -1, 2 * c + (v == v ? 0 : 1), v);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) found[sp * 4 * nq + 4 * q + j] = best[j];
    }
    __syncthreads();
    for (int p = tid; p < 4 * nq; p += PW_THREADS) {
        PwBest a = found[p];
        for (int sp = 1; sp < splits; ++sp) {
            const PwBest o = found[sp * 4 * nq + p];
            pw_join(a, o.t, o.c, o.first, o.v);
        }
        const bool nan_first = p < n && a.first >= 0 && (a.first & 1);
        bc[p] = p < n ? (nan_first ? a.first >> 1 : a.c) : -1;
        bt[p] = (uint8_t)a.t;
        bv[p] = nan_first ? *reinterpret_cast<const float *>(vb + 4 * ((I)(a.first >> 1) * HW + p)) : a.v;  // (its own bits)
    }
    __syncthreads();
    // items (feature, 4 locations) of the part's features, PW_THREADS on each time
    const int c1 = (int)((int64_t)C * (part + 1) / parts), cs = PW_THREADS / nq, qs = PW_THREADS - cs * nq;
    int c = (int)((int64_t)C * part / parts) + tid / nq, q = tid % nq;
    for (; c < c1; c += cs + (q + qs >= nq ? 1 : 0), q = q + qs >= nq ? q + qs - nq : q + qs) {
        const int nj = min(4, n - 4 * q);
        const int4 w4 = *reinterpret_cast<const int4 *>(bc + 4 * q);
        const bool k[4] = {w4.x == c, w4.y == c, w4.z == c, w4.w == c};
        const int64_t e = (I)c * HW + 4 * q, o = base + e, ow = b * T * plane + p0 + e;
        uint32_t tw = 0;
        Float4u v;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            tw |= (uint32_t)(k[j] ? (int)bt[4 * q + j] : T) << (8 * j);
            v.v[j] = k[j] ? bv[4 * q + j] : 0.0f;
        }
        const bool any = k[0] || k[1] || k[2] || k[3];
        if (nj == 4) {
            reinterpret_cast<Byte4u *>(out_t + o)->w = tw;
            *reinterpret_cast<Float4u *>(out_v + o) = v;
            if (wave) {
                if (any)
                    for (int t = 0; t < T; ++t)
                        reinterpret_cast<Byte4u *>(wave + ow + t * plane)->w = spk::spikes4(tw, t, T);
                else
                    for (int t = 0; t < T; ++t) reinterpret_cast<Byte4u *>(wave + ow + t * plane)->w = 0;
            }
            if (pot) {
                if (any)
                    for (int t = 0; t < T; ++t)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if (!k[j]) pot[ow + t * plane + j] = 0.0f;
                        }
                else
                    for (int t = 0; t < T; ++t)
                        *reinterpret_cast<Float4u *>(pot + ow + t * plane) = Float4u{{0.0f, 0.0f, 0.0f, 0.0f}};
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= nj) continue;
                const int tj = (int)((tw >> (8 * j)) & 255u);
                out_t[o + j] = (uint8_t)tj;
                out_v[o + j] = v.v[j];
                if (wave)
                    for (int t = 0; t < T; ++t) wave[ow + t * plane + j] = (uint8_t)(t >= tj);
                if (pot && !k[j])
                    for (int t = 0; t < T; ++t) pot[ow + t * plane + j] = 0.0f;
            }
        }
    }
}

// One thread per location of one image (VEC: per 4 consecutive locations,
// with 4-byte / 16-byte accesses; the map size is then a multiple of 4): the
// winner over the C features, then every feature's surviving first-spike time
// and potential, and, when asked, the survivors' Eq.1 wave and the masked
// potentials.  All C features of the locations are read before any is written,
// so the outputs may alias the inputs.  Consecutive threads take consecutive
// locations, so every per-feature access of a wave is contiguous.
template <bool VEC>
__global__ __launch_bounds__(256) void k_pointwise_each(const uint8_t *tf, const float *vf, int64_t B, int T, int C,
                                                        int64_t HW, uint8_t *out_t, float *out_v, uint8_t *wave,
                                                        float *pot) {
    constexpr int L = VEC ? 4 : 1;
    const int64_t per_img = HW / L;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= B * per_img) return;
    const int64_t b = q / per_img, p = (q - b * per_img) * L;
    const int64_t base = b * C * HW + p;
    int best[L], bt[L];
    float bv[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
        best[j] = -1;
        bt[j] = T;
        bv[j] = 0.0f;
    }
    // features in blocks of PW_U, every load of a block issued before the
    // first is used (clamped feature indices keep them unconditional), in
    // increasing feature order so that strict comparisons keep the lower index
    for (int c0 = 0; c0 < C; c0 += PW_U) {
        uint32_t tw[PW_U];
        float4 vw[PW_U];
#pragma unroll
        for (int u = 0; u < PW_U; ++u) {
            const int64_t o = base + (int64_t)min(c0 + u, C - 1) * HW;
            if (VEC) {
                tw[u] = *reinterpret_cast<const uint32_t *>(tf + o);
                vw[u] = *reinterpret_cast<const float4 *>(vf + o);
            } else {
                tw[u] = tf[o];
                vw[u].x = vf[o];
            }
        }
#pragma unroll
        for (int u = 0; u < PW_U; ++u) {
            const int c = c0 + u;
            if (c >= C) break;
            int t[L];
            float v[L];
            t[0] = tw[u] & 255u;
            v[0] = vw[u].x;
            if (VEC) {
                t[L > 1 ? 1 : 0] = (tw[u] >> 8) & 255u;
                t[L > 2 ? 2 : 0] = (tw[u] >> 16) & 255u;
                t[L > 3 ? 3 : 0] = tw[u] >> 24;
                v[L > 1 ? 1 : 0] = vw[u].y; v[L > 2 ? 2 : 0] = vw[u].z; v[L > 3 ? 3 : 0] = vw[u].w;
            }
#pragma unroll
            for (int j = 0; j < L; ++j)
                if (t[j] < T && (best[j] < 0 || t[j] < bt[j] || (t[j] == bt[j] && v[j] > bv[j]))) {
                    best[j] = c;
                    bt[j] = t[j];
                    bv[j] = v[j];
                }
        }
    }
    // the surviving first-spike times of feature c, 4 to a word
    auto word = [&](int c) {
        uint32_t w = 0;
#pragma unroll
        for (int j = 0; j < L; ++j) w |= (uint32_t)(c == best[j] ? bt[j] : T) << (8 * j);
        return w;
    };
    for (int c = 0; c < C; ++c) {
        if (VEC) {
            *reinterpret_cast<uint32_t *>(out_t + base + c * HW) = word(c);
            *reinterpret_cast<float4 *>(out_v + base + c * HW) =
                float4{c == best[0] ? bv[0] : 0.0f, c == best[L > 1 ? 1 : 0] ? bv[L > 1 ? 1 : 0] : 0.0f,
                       c == best[L > 2 ? 2 : 0] ? bv[L > 2 ? 2 : 0] : 0.0f,
                       c == best[L > 3 ? 3 : 0] ? bv[L > 3 ? 3 : 0] : 0.0f};
        } else {
            out_t[base + c * HW] = (uint8_t)(c == best[0] ? bt[0] : T);
            out_v[base + c * HW] = c == best[0] ? bv[0] : 0.0f;
        }
    }
    const int64_t plane = (int64_t)C * HW;
    if (wave)  // feature by feature: its surviving times once, then its T steps
        for (int c = 0; c < C; ++c) {
            uint8_t *w = wave + b * T * plane + (int64_t)c * HW + p;
            if (VEC) {
                const uint32_t wc = word(c);
                for (int t = 0; t < T; ++t) *reinterpret_cast<uint32_t *>(w + t * plane) = spk::spikes4(wc, t, T);
            } else {
                const int tc = c == best[0] ? bt[0] : T;
                for (int t = 0; t < T; ++t) w[t * plane] = (uint8_t)(t >= tc);
            }
        }
    if (pot)
        for (int t = 0; t < T; ++t) {
            float *pp = pot + (b * T + t) * plane + p;
            if constexpr (VEC) {
                // blocks of PW_U features: the loads first (clamped), then the masked stores
                for (int c0 = 0; c0 < C; c0 += PW_U) {
                    float4 xw[PW_U];
#pragma unroll
                    for (int u = 0; u < PW_U; ++u)
                        xw[u] = *reinterpret_cast<const float4 *>(pp + (int64_t)min(c0 + u, C - 1) * HW);
#pragma unroll
                    for (int u = 0; u < PW_U; ++u) {
                        const int c = c0 + u;
                        if (c >= C) break;
                        if (c == best[0] && c == best[1] && c == best[2] && c == best[3])
                            continue;  // the feature survives at all four locations
                        float4 x = xw[u];
                        if (c != best[0]) x.x = 0.0f;
                        if (c != best[1]) x.y = 0.0f;
                        if (c != best[2]) x.z = 0.0f;
                        if (c != best[3]) x.w = 0.0f;
                        *reinterpret_cast<float4 *>(pp + (int64_t)c * HW) = x;
                    }
                }
            } else {
                for (int c = 0; c < C; ++c)
                    if (c != best[0]) pp[c * HW] = 0.0f;
            }
        }
}

// One thread per output value: the maximum over the window of the zero-padded
// input, taken in row-major window order keeping the first of equal values.
__global__ __launch_bounds__(256) void k_pool_potentials(const float *__restrict__ pot, int64_t total, int H, int W,
                                                         int P, int R, int D, int Ho, int Wo,
                                                         float *__restrict__ out) {
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= total) return;
    const int64_t pl = o / ((int64_t)Ho * Wo);
    const int r = (int)(o - pl * Ho * Wo), yo = r / Wo, xo = r - yo * Wo;
    const float *src = pot + pl * H * W;
    bool first = true;
    float m = 0.0f;
    for (int dy = 0; dy < P; ++dy)
        for (int dx = 0; dx < P; ++dx) {
            const int iy = yo * R + dy - D, ix = xo * R + dx - D;
            const float v = (iy >= 0 && iy < H && ix >= 0 && ix < W) ? src[(int64_t)iy * W + ix] : 0.0f;
            if (first || v > m) m = v;
            first = false;
        }
    out[o] = m;
}

// 2x2 windows, stride 2, no padding, W a multiple of 4, Wo even, aligned
// tensors: one thread per two adjacent outputs, from one 16-byte load of each
// of the two input rows; the same comparisons in the same window order.
__global__ __launch_bounds__(256) void k_pool_potentials_2x2(const float *__restrict__ pot, uint32_t pairs, int H,
                                                             int W, int Ho, int Wo, float *__restrict__ out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pairs) return;
    const uint32_t hw2 = (uint32_t)(Ho * Wo) / 2, wo2 = (uint32_t)Wo / 2;
    const uint32_t pl = i / hw2, r = i - pl * hw2, yo = r / wo2, x2 = r - yo * wo2;
    const float *src = pot + (size_t)pl * H * W + (size_t)(2 * yo) * W + 4 * x2;
    const float4 a = *reinterpret_cast<const float4 *>(src), c = *reinterpret_cast<const float4 *>(src + W);
    auto win = [](float v00, float v01, float v10, float v11) {
        float m = v00;
        if (v01 > m) m = v01;
        if (v10 > m) m = v10;
        if (v11 > m) m = v11;
        return m;
    };
    *reinterpret_cast<float2 *>(out + (size_t)pl * Ho * Wo + (size_t)yo * Wo + 2 * x2) =
        float2{win(a.x, a.y, c.x, c.y), win(a.z, a.w, c.z, c.w)};
}

// The same for even widths (8-byte aligned rows): one output per thread, from
// one 8-byte load of each of its two rows.  Single loads reach every other
// column of two rows at a time: 200 images of 250 maps of 14x14, T = 15, took
// 189 us; now 178 us (4.1 TB/s).
__global__ __launch_bounds__(256) void k_pool_potentials_2x2_even(const float *__restrict__ pot, uint32_t total, int H,
                                                                  int W, int Ho, int Wo, float *__restrict__ out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const uint32_t hw = (uint32_t)(Ho * Wo), pl = i / hw, r = i - pl * hw, yo = r / (uint32_t)Wo, xo = r - yo * Wo;
    const float *src = pot + (size_t)pl * H * W + (size_t)(2 * yo) * W + 2 * xo;
    const float2 a = *reinterpret_cast<const float2 *>(src), c = *reinterpret_cast<const float2 *>(src + W);
    float m = a.x;
    if (a.y > m) m = a.y;
    if (c.x > m) m = c.x;
    if (c.y > m) m = c.y;
    out[i] = m;
}

// Whether one thread per location does better than a workgroup per run.  That form
// takes about 0.3 us a feature (a quad of locations per thread; 0.15 one at a time) until
// the locations fill the chip, and T times that with the wave or the potentials; the
// workgroups share the features of a location, as far as its run leaves them threads,
// but are as many as there are images, however little each has to do.  Measured at
// T = 15 (each : runs, us): first spikes of 250 maps of 14x14, 200 images 91 : 81,
// 1000 images 135 : 162; of 28x28, 8 images 84 : 114; 30 maps of 28x28, 200 images
// 16 : 45; 200 of 4x4, 1000 images 73 : 30, 4096 77 : 107; 150 of 7x9, 64 images 25 : 20,
// 256 28 : 37.  With wave and potentials 64 maps of 14x14, 1000 images 507 : 363; 8 of
// 64x64, 16 images 36 : 24, 128 109 : 163; 12 of 7x7, 1000 images 20 : 28; 4 of 9x9, 100
// images 7.5 : 8.7; 10 of 1x1, 1000 images 42 : 10, 100,000 147 : 818.
bool pw_each(int64_t B, int64_t C, int64_t HW, int64_t nrun, bool vec, bool steps) {
    const int64_t loc = B * HW;
    if (steps) return C < 8 || loc > (vec ? 262144 : 40000) || B * nrun > std::max<int64_t>(4096, 64 * C);
    return C < (vec ? 32 : 100) || HW > 448 || loc > (vec ? std::max<int64_t>(12800, 200 * C) : 50 * C) || B > 2048;
}

}  // namespace

extern "C" int spk_pointwise_inhibition(const uint8_t *t_first, const float *v_first, int B, int T, int C, int H,
                                        int W, uint8_t *out_t_first, float *out_v_first, uint8_t *out_wave,
                                        float *potentials, void *stream) {
    SPK_REQUIRE(B >= 0 && T >= 1 && C >= 1 && H >= 1 && W >= 1, SPK_E_SHAPE, "spk_pointwise_inhibition: bad sizes");
    SPK_REQUIRE(T <= 255, SPK_E_RANGE, "spk_pointwise_inhibition: T=%d > 255", T);
    if (B == 0) return spk::ok();
    SPK_REQUIRE(t_first && v_first && out_t_first && out_v_first, SPK_E_ARG,
                "spk_pointwise_inhibition: t_first, v_first, out_t_first and out_v_first are required");
    const int64_t HW = (int64_t)H * W, total = (int64_t)B * HW;
    SPK_REQUIRE(spk::ceil_div(total, 256) < (1LL << 31), SPK_E_RANGE, "spk_pointwise_inhibition: too large");
    auto al = [](const void *q, uintptr_t a) { return ((uintptr_t)q & (a - 1)) == 0; };
    const bool vec = HW % 4 == 0 && al(t_first, 4) && al(out_t_first, 4) && al(out_wave, 4) && al(v_first, 16) &&
                     al(out_v_first, 16) && al(potentials, 16);
    hipStream_t st = spk::as_stream(stream);
    const int64_t nrun = spk::ceil_div(HW, PW_LOC);
    if (pw_each(B, C, HW, nrun, vec, out_wave || potentials)) {
        if (vec)
            hipLaunchKernelGGL(k_pointwise_each<true>, dim3((unsigned)spk::ceil_div(total / 4, 256)), dim3(256), 0, st,
                               t_first, v_first, (int64_t)B, T, C, HW, out_t_first, out_v_first, out_wave, potentials);
        else
            hipLaunchKernelGGL(k_pointwise_each<false>, dim3((unsigned)spk::ceil_div(total, 256)), dim3(256), 0, st,
                               t_first, v_first, (int64_t)B, T, C, HW, out_t_first, out_v_first, out_wave, potentials);
        return spk::check_launch("spk_pointwise_inhibition");
    }
    // more workgroups per run where the runs are few (each scans the run's inputs for
    // itself: 5 bytes a neuron, from L2 after the first), unless outputs are inputs
    const int64_t N = (int64_t)B * C * HW;
    auto overlap = [](const void *a, int64_t na, const void *b, int64_t nb) {
        const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
        return x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
    };
    auto on_inputs = [&](const void *out, int64_t bytes) {
        return out && (overlap(out, bytes, t_first, N) || overlap(out, bytes, v_first, 4 * N));
    };
    const bool alias = on_inputs(out_t_first, N) || on_inputs(out_v_first, 4 * N) || on_inputs(out_wave, T * N) ||
                       on_inputs(potentials, 4 * T * N);
    const int64_t per_run = spk::ceil_div((int64_t)C * spk::ceil_div(std::min<int64_t>(HW, PW_LOC), 4), PW_THREADS);
    const int64_t parts = alias ? 1 : std::max<int64_t>(1, std::min<int64_t>({1024 / (B * nrun), 8, per_run, C}));
    // a launch has fewer than 2^32 threads
    const int64_t most = ((1LL << 32) - 1) / PW_THREADS / parts;
    for (int64_t u0 = 0; u0 < B * nrun; u0 += most) {
        const dim3 grid((unsigned)(std::min(most, B * nrun - u0) * parts));
        const size_t lds = (size_t)PW_THREADS * 4 * sizeof(PwBest);
        if (C * HW <= 1LL << 30)
            hipLaunchKernelGGL(k_pointwise<uint32_t>, grid, dim3(PW_THREADS), lds, st, t_first, v_first, T, C,
                               (uint32_t)HW, u0, nrun, (int)parts, out_t_first, out_v_first, out_wave, potentials);
        else
            hipLaunchKernelGGL(k_pointwise<uint64_t>, grid, dim3(PW_THREADS), lds, st, t_first, v_first, T, C,
                               (uint64_t)HW, u0, nrun, (int)parts, out_t_first, out_v_first, out_wave, potentials);
    }
    return spk::check_launch("spk_pointwise_inhibition");
}

extern "C" int spk_pool_potentials(const float *potentials, int B, int T, int C, int H, int W, int kernel, int stride,
                                   int pad, float *out, void *stream) {
    SPK_REQUIRE(B >= 0 && T >= 1 && C >= 1 && H >= 1 && W >= 1, SPK_E_SHAPE, "spk_pool_potentials: bad sizes");
    SPK_REQUIRE(kernel >= 1 && stride >= 1 && pad >= 0, SPK_E_SHAPE,
                "spk_pool_potentials: bad window %d / stride %d / pad %d", kernel, stride, pad);
    SPK_REQUIRE(H + 2 * pad >= kernel && W + 2 * pad >= kernel, SPK_E_SHAPE,
                "spk_pool_potentials: window %d larger than the padded input", kernel);
    const int Ho = (H + 2 * pad - kernel) / stride + 1, Wo = (W + 2 * pad - kernel) / stride + 1;
    if (B == 0) return spk::ok();
    SPK_REQUIRE(potentials && out, SPK_E_ARG, "spk_pool_potentials: potentials and out are required");
    const int64_t total = (int64_t)B * T * C * Ho * Wo;
    SPK_REQUIRE(spk::ceil_div(total, 256) < (1LL << 31), SPK_E_RANGE, "spk_pool_potentials: too large");
    const bool al16 = ((uintptr_t)potentials & 15) == 0 && ((uintptr_t)out & 7) == 0;
    if (kernel == 2 && stride == 2 && pad == 0 && W % 4 == 0 && Wo % 2 == 0 && Ho == H / 2 && al16 &&
        total / 2 < (1LL << 32) && (int64_t)B * T * C * H * W < (1LL << 32)) {
        const int64_t pairs = total / 2;
        hipLaunchKernelGGL(k_pool_potentials_2x2, dim3((unsigned)spk::ceil_div(pairs, 256)), dim3(256), 0,
                           spk::as_stream(stream), potentials, (uint32_t)pairs, H, W, Ho, Wo, out);
        return spk::check_launch("spk_pool_potentials");
    }
    if (kernel == 2 && stride == 2 && pad == 0 && W % 2 == 0 && ((uintptr_t)potentials & 7) == 0 &&
        total < (1LL << 32) - 256) {
        hipLaunchKernelGGL(k_pool_potentials_2x2_even, dim3((unsigned)spk::ceil_div(total, 256)), dim3(256), 0,
                           spk::as_stream(stream), potentials, (uint32_t)total, H, W, Ho, Wo, out);
        return spk::check_launch("spk_pool_potentials");
    }
    hipLaunchKernelGGL(k_pool_potentials, dim3((unsigned)spk::ceil_div(total, 256)), dim3(256), 0,
                       spk::as_stream(stream), potentials, total, H, W, kernel, stride, pad, Ho, Wo, out);
    return spk::check_launch("spk_pool_potentials");
}
