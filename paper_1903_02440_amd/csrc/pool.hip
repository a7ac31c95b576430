// Spike max-pooling (gfx950).
//
// Paper: section "snn Module" (snn.Pooling / sf.pooling on spike waves: the
// output holds the earliest spike of each window; stride defaults to the
// window; zero padding) and Eq.3 for the output size, read as
// floor((H + 2D - P)/R) + 1 (equal to the printed form whenever P == R).
//
// Waves, in the general form, take one thread per output neuron (b, c, yo, xo):
// for every step t it ORs the window's bytes of plane t and stores one byte, so a
// wave reads and writes consecutive x positions of one plane; the first-spike map
// is T minus the number of steps at which the pooled neuron is on.  Larger batches
// of maps that fit go through LDS.
#include <algorithm>
#include <cstdint>

#include "common.hpp"

namespace {

// Grid: (image, chunk of 256 of the image's C*Ho*Wo outputs).
__global__ __launch_bounds__(256) void k_pool(const uint8_t *__restrict__ in, int T, int C, int H, int W, int P, int R,
                                              int D, int Ho, int Wo, uint8_t *__restrict__ out,
                                              uint8_t *__restrict__ out_tf) {
    const int per_img = C * Ho * Wo;
    const int i = blockIdx.y * 256 + threadIdx.x;
    if (i >= per_img) return;
    const int64_t b = blockIdx.x;
    const int hw = Ho * Wo;
    const int c = i / hw, pix = i - c * hw;
    const int yo = pix / Wo, xo = pix - yo * Wo;
    const int y0 = yo * R - D, x0 = xo * R - D;
    const int ya = max(y0, 0), yb = min(y0 + P, H), xa = max(x0, 0), xb = min(x0 + P, W);
    const int64_t in_plane = (int64_t)C * H * W, out_plane = (int64_t)per_img;
    const uint8_t *src = in + b * T * in_plane + (int64_t)c * H * W;
    uint8_t *dst = out + b * T * out_plane + i;
    int on = 0;
    for (int t = 0; t < T; ++t) {
        const uint8_t *pl = src + t * in_plane;
        int m = 0;
        for (int y = ya; y < yb; ++y)
            for (int x = xa; x < xb; ++x) m |= pl[y * W + x];
        m = m != 0;
        dst[t * out_plane] = (uint8_t)m;
        on += m;
    }
    if (out_tf) out_tf[b * per_img + i] = (uint8_t)(T - on);
}

// The same with the input staged in LDS: a workgroup takes CB whole maps of one
// image (contiguous in every step) and goes through the steps, copying the next
// step's bytes with 16-byte loads at any alignment while the current ones are
// pooled, 4 consecutive outputs per thread (at most WL_QUADS times) in one 4-byte
// store.  Bound by reading the wave: 256 images of 250 maps of 14x14, T = 15, 3x3
// windows, took 150 us with one output per thread from single byte loads, now 74 us
// (233 MB, 3.2 TB/s).
constexpr int WL_BYTES = 16384;  // input bytes of a step at most
constexpr int WL_QUADS = 2;      // quads of outputs per thread
constexpr int WL_LOADS = WL_BYTES / 16 / 256;
struct __attribute__((packed, aligned(1))) Bytes16 {
    uint32_t w[4];
};
struct __attribute__((packed, aligned(1))) Bytes4 {
    uint32_t w;
};
template <int PW, bool IN>  // IN: no padding, every window lies in its map
__global__ __launch_bounds__(256) void k_pool_lds(const uint8_t *__restrict__ in, int T, int C, int H, int W, int P,
                                                  int R, int D, int Ho, int Wo, int CB, uint8_t *__restrict__ out,
                                                  uint8_t *__restrict__ out_tf) {
    __shared__ uint4 lds[WL_BYTES / 16];
    uint8_t *lt = reinterpret_cast<uint8_t *>(lds);
    const int tid = threadIdx.x, nblk = (C + CB - 1) / CB;
    const int64_t b = blockIdx.x / nblk;
    const int c0 = (int)(blockIdx.x % nblk) * CB, cb = min(CB, C - c0), HW = H * W, hw = Ho * Wo;
    const int nbytes = cb * HW, nout = cb * hw;
    const int64_t in_plane = (int64_t)C * HW, out_plane = (int64_t)C * hw;
    const uint8_t *src = in + b * T * in_plane + (int64_t)c0 * HW;
    uint8_t *dst = out + b * T * out_plane + (int64_t)c0 * hw;
    const int n16 = nbytes / 16, rest = nbytes - 16 * n16;  // whole 16 bytes, then single ones
    uint4 v[WL_LOADS];
    uint8_t vb = 0;
    auto load = [&](int t) {
        const uint8_t *s = src + t * in_plane;
#pragma unroll
        for (int k = 0; k < WL_LOADS; ++k) {
            const int i = tid + k * 256;
            if (i < n16) {
                const Bytes16 x = *reinterpret_cast<const Bytes16 *>(s + 16 * i);
                v[k] = uint4{x.w[0], x.w[1], x.w[2], x.w[3]};
            }
        }
        if (tid < rest) vb = s[16 * n16 + tid];
    };
    uint32_t on[WL_QUADS];  // steps at which each output of a quad is on, a byte each
#pragma unroll
    for (int m = 0; m < WL_QUADS; ++m) on[m] = 0;
    int at[WL_QUADS][4];  // IN: each output's window corner in LDS (outputs past the block: the first's)
#pragma unroll
    for (int m = 0; m < WL_QUADS; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = (tid + m * 256) * 4 + q, jj = j < nout ? j : 0;
            const int c = jj / hw, yo = (jj - c * hw) / Wo, xo = jj - c * hw - yo * Wo;
            at[m][q] = IN ? c * HW + yo * R * W + xo * R : c << 20 | yo << 10 | xo;
        }
    load(0);
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int k = 0; k < WL_LOADS; ++k)
            if (tid + k * 256 < n16) lds[tid + k * 256] = v[k];
        if (tid < rest) lt[16 * n16 + tid] = vb;
        __syncthreads();
        if (t + 1 < T) load(t + 1);
#pragma unroll
        for (int m = 0; m < WL_QUADS; ++m) {
            const int j0 = (tid + m * 256) * 4;
            if (j0 >= nout) continue;
            uint32_t o4 = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t any = 0;
                if (IN) {
                    const uint8_t *w = lt + at[m][q];
                    if (PW > 0) {
#pragma unroll
                        for (int dy = 0; dy < PW; ++dy)
#pragma unroll
                            for (int dx = 0; dx < PW; ++dx) any |= w[dy * W + dx];
                    } else {
#pragma unroll 1
                        for (int dy = 0; dy < P; ++dy)
#pragma unroll 1
                            for (int dx = 0; dx < P; ++dx) any |= w[dy * W + dx];
                    }
                } else {
                    const int y0 = ((at[m][q] >> 10) & 1023) * R - D, x0 = (at[m][q] & 1023) * R - D;
                    const uint8_t *pl = lt + (at[m][q] >> 20) * HW;
                    for (int y = max(y0, 0); y < min(y0 + P, H); ++y)
                        for (int x = max(x0, 0); x < min(x0 + P, W); ++x) any |= pl[y * W + x];
                }
                o4 |= (any != 0 ? 1u : 0u) << (8 * q);
            }
            on[m] += o4;
            uint8_t *d = dst + t * out_plane + j0;
            if (j0 + 4 <= nout) {
                reinterpret_cast<Bytes4 *>(d)->w = o4;
            } else {
                for (int q = 0; j0 + q < nout; ++q) d[q] = (uint8_t)(o4 >> (8 * q));
            }
        }
        __syncthreads();
    }
    if (out_tf)
#pragma unroll
        for (int m = 0; m < WL_QUADS; ++m) {
            const int j0 = (tid + m * 256) * 4;
            if (j0 >= nout) continue;
            const uint32_t t4 = (uint32_t)T * 0x01010101u - on[m];
            uint8_t *d = out_tf + b * out_plane + (int64_t)c0 * hw + j0;
            for (int q = 0; q < 4 && j0 + q < nout; ++q) d[q] = (uint8_t)(t4 >> (8 * q));
        }
}

// Pooling of first-spike maps: the minimum over the window, then its T wave
// bytes.  Grid (image, chunk of the image's C*Ho*Wo outputs); with VEC (C*Ho*Wo
// a multiple of 4, 4-byte aligned outputs) each thread makes 4 consecutive
// outputs and stores them as one word per plane, else one output per thread.
// PW > 0 is the window size known at compile time: every window load is then
// issued before any is used.
template <bool VEC, int PW>
__global__ __launch_bounds__(256) void k_pool_first_spike(const uint8_t *__restrict__ tf, int T, int C, int H, int W,
                                                          int P, int R, int D, int Ho, int Wo,
                                                          uint8_t *__restrict__ out, uint8_t *__restrict__ out_tf) {
    constexpr int NQ = VEC ? 4 : 1;
    const int per_img = C * Ho * Wo;
    const int i0 = (blockIdx.y * 256 + threadIdx.x) * NQ;
    if (i0 >= per_img) return;
    const int64_t b = blockIdx.x;
    const int hw = Ho * Wo;
    uint32_t m4 = 0;
    // (c, yo, xo) of the first output, then stepped along x for the others
    int c = i0 / hw, yo = (i0 - c * hw) / Wo, xo = i0 - c * hw - yo * Wo;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q > 0 && ++xo == Wo) {
            xo = 0;
            if (++yo == Ho) {
                yo = 0;
                ++c;
            }
        }
        const int y0 = yo * R - D, x0 = xo * R - D;
        const int ya = max(y0, 0), yb = min(y0 + P, H), xa = max(x0, 0), xb = min(x0 + P, W);
        const uint8_t *src = tf + (b * C + c) * (int64_t)H * W;
        int m = T;
        if (PW > 0) {
#pragma unroll
            for (int dy = 0; dy < PW; ++dy)
#pragma unroll
                for (int dx = 0; dx < PW; ++dx) {
                    const int y = y0 + dy, x = x0 + dx;
                    const bool in = y >= 0 && y < H && x >= 0 && x < W;
                    m = min(m, in ? (int)src[y * W + x] : T);
                }
        } else {
            for (int y = ya; y < yb; ++y)
                for (int x = xa; x < xb; ++x) m = min(m, (int)src[y * W + x]);
        }
        m4 |= (uint32_t)m << (8 * q);
    }
    if (VEC) {
        if (out_tf) *reinterpret_cast<uint32_t *>(out_tf + b * per_img + i0) = m4;
        if (out) {
            uint8_t *dst = out + b * T * (int64_t)per_img + i0;
            for (int t = 0; t < T; ++t)
                *reinterpret_cast<uint32_t *>(dst + (int64_t)t * per_img) = spk::spikes4(m4, t, T);
        }
    } else {
        const int m = (int)m4;
        if (out_tf) out_tf[b * per_img + i0] = (uint8_t)m;
        if (out) {
            uint8_t *dst = out + b * T * (int64_t)per_img + i0;
            for (int t = 0; t < T; ++t) dst[(int64_t)t * per_img] = (uint8_t)(t >= m);
        }
    }
}

// The same pooling with the input staged in LDS: a workgroup takes CB whole
// input planes of one image (contiguous in memory), copies them with
// coalesced loads, and makes their outputs 4 consecutive ones per thread, so
// the window reads hit LDS instead of scattering bytes over many cache lines.
// Needs CB * Ho * Wo % 4 == 0 (quads never straddle blocks) and 4-byte
// aligned outputs.
template <int PW>
__global__ __launch_bounds__(256) void k_pool_first_spike_lds(const uint8_t *__restrict__ tf, int T, int C, int H,
                                                              int W, int P, int R, int D, int Ho, int Wo, int CB,
                                                              uint8_t *__restrict__ out, uint8_t *__restrict__ out_tf) {
    extern __shared__ uint32_t plsm[];
    uint8_t *lt = reinterpret_cast<uint8_t *>(plsm);
    const int64_t b = blockIdx.x;
    const int c0 = blockIdx.y * CB, cb = min(CB, C - c0);
    const int HW = H * W, hw = Ho * Wo;
    const uint8_t *src = tf + (b * C + c0) * (int64_t)HW;
    const int nbytes = cb * HW;
    if ((((uintptr_t)src) & 3) == 0) {
        // a thread issues up to 16 word loads before its first LDS store (clamped
        // indices keep the loads unconditional, so none waits for the one before)
        const int nw = nbytes >> 2;
        const uint32_t *s4 = reinterpret_cast<const uint32_t *>(src);
        for (int i0 = threadIdx.x; i0 < nw; i0 += 16 * 256) {
            uint32_t v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = s4[min(i0 + k * 256, nw - 1)];
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (i0 + k * 256 < nw) plsm[i0 + k * 256] = v[k];
        }
        for (int i = (nw << 2) + threadIdx.x; i < nbytes; i += 256) lt[i] = src[i];
    } else {
        for (int i = threadIdx.x; i < nbytes; i += 256) lt[i] = src[i];
    }
    __syncthreads();
    const int per_img = C * hw, nq = cb * hw / 4;
    for (int qd = threadIdx.x; qd < nq; qd += 256) {
        const int j0 = qd * 4;  // first output of the quad within the block
        int c = j0 / hw, yo = (j0 - c * hw) / Wo, xo = j0 - c * hw - yo * Wo;
        uint32_t m4 = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q > 0 && ++xo == Wo) {
                xo = 0;
                if (++yo == Ho) {
                    yo = 0;
                    ++c;
                }
            }
            const int y0 = yo * R - D, x0 = xo * R - D;
            const uint8_t *pl = lt + c * HW;
            int m = T;
            if (PW > 0) {
#pragma unroll
                for (int dy = 0; dy < PW; ++dy)
#pragma unroll
                    for (int dx = 0; dx < PW; ++dx) {
                        const int y = y0 + dy, x = x0 + dx;
                        const bool in = y >= 0 && y < H && x >= 0 && x < W;
                        m = min(m, in ? (int)pl[y * W + x] : T);
                    }
            } else {
                const int ya = max(y0, 0), yb = min(y0 + P, H), xa = max(x0, 0), xb = min(x0 + P, W);
                for (int y = ya; y < yb; ++y)
                    for (int x = xa; x < xb; ++x) m = min(m, (int)pl[y * W + x]);
            }
            m4 |= (uint32_t)m << (8 * q);
        }
        const int64_t i0 = (int64_t)c0 * hw + j0;
        if (out_tf) *reinterpret_cast<uint32_t *>(out_tf + b * per_img + i0) = m4;
        if (out) {
            uint8_t *dst = out + b * T * (int64_t)per_img + i0;
            for (int t = 0; t < T; ++t)
                *reinterpret_cast<uint32_t *>(dst + (int64_t)t * per_img) = spk::spikes4(m4, t, T);
        }
    }
}

}  // namespace

extern "C" int spk_pool_first_spike(const uint8_t *t_first, int B, int T, int C, int H, int W, int kernel,
                                    int stride, int pad, uint8_t *out_wave, uint8_t *out_t_first, void *stream) {
    SPK_REQUIRE(B >= 0 && T >= 1 && C >= 1 && H >= 1 && W >= 1, SPK_E_SHAPE, "spk_pool_first_spike: bad sizes");
    SPK_REQUIRE(T <= 255, SPK_E_RANGE, "spk_pool_first_spike: T=%d > 255", T);
    SPK_REQUIRE(kernel >= 1 && stride >= 1 && pad >= 0, SPK_E_SHAPE,
                "spk_pool_first_spike: bad window %d / stride %d / pad %d", kernel, stride, pad);
    const int Ho = (H + 2 * pad - kernel) / stride + 1, Wo = (W + 2 * pad - kernel) / stride + 1;
    SPK_REQUIRE(H + 2 * pad >= kernel && W + 2 * pad >= kernel && Ho >= 1 && Wo >= 1, SPK_E_SHAPE,
                "spk_pool_first_spike: window %d larger than the padded input", kernel);
    if (B == 0) return spk::ok();
    SPK_REQUIRE(t_first && (out_wave || out_t_first), SPK_E_ARG,
                "spk_pool_first_spike: t_first and an output are required");
    const int64_t per_img = (int64_t)C * Ho * Wo;
    SPK_REQUIRE(per_img <= 65535LL * 256 && (int64_t)C * H * W < (1LL << 31), SPK_E_RANGE,
                "spk_pool_first_spike: image too large");
    const bool vec = per_img % 4 == 0 && ((uintptr_t)out_wave & 3) == 0 && ((uintptr_t)out_t_first & 3) == 0;
    hipStream_t st = spk::as_stream(stream);
    // LDS-staged form: blocks of whole input planes (up to 16 KB), quads within a block
    const int64_t HW = (int64_t)H * W, hw = (int64_t)Ho * Wo;
    if (vec && HW <= 16384) {
        // about 1024 outputs (4 per thread) per workgroup, at most 16 KB of planes
        int CB = (int)std::min<int64_t>(std::min<int64_t>(C, 16384 / HW), std::max<int64_t>(1, (1024 + hw - 1) / hw));
        while (CB > 1 && (CB * hw) % 4 != 0) --CB;
        if ((CB * hw) % 4 == 0 && (C % CB == 0 || ((int64_t)(C % CB) * hw) % 4 == 0)) {
            const dim3 g2((unsigned)B, (unsigned)spk::ceil_div(C, CB));
            const size_t lds = spk::align_up((size_t)CB * HW, 4);
#define SPK_POOL_LDS(PW)                                                                                          \
    hipLaunchKernelGGL((k_pool_first_spike_lds<PW>), g2, dim3(256), lds, st, t_first, T, C, H, W, kernel, stride, pad, \
                       Ho, Wo, CB, out_wave, out_t_first)
            if (kernel == 2) SPK_POOL_LDS(2);
            else if (kernel == 3) SPK_POOL_LDS(3);
            else SPK_POOL_LDS(0);
#undef SPK_POOL_LDS
            return spk::check_launch("spk_pool_first_spike");
        }
    }
    const dim3 grid((unsigned)B, (unsigned)spk::ceil_div(per_img, vec ? 1024 : 256));
#define SPK_POOL(V, PW)                                                                                            \
    hipLaunchKernelGGL((k_pool_first_spike<V, PW>), grid, dim3(256), 0, st, t_first, T, C, H, W, kernel, stride, pad, \
                       Ho, Wo, out_wave, out_t_first)
    if (vec && kernel == 2) SPK_POOL(true, 2);
    else if (vec && kernel == 3) SPK_POOL(true, 3);
    else if (vec) SPK_POOL(true, 0);
    else SPK_POOL(false, 0);
#undef SPK_POOL
    return spk::check_launch("spk_pool_first_spike");
}

extern "C" int spk_pool(const uint8_t *wave, int B, int T, int C, int H, int W, int kernel, int stride, int pad,
                        uint8_t *out_wave, uint8_t *out_t_first, void *stream) {
    SPK_REQUIRE(B >= 0 && T >= 1 && C >= 1 && H >= 1 && W >= 1, SPK_E_SHAPE, "spk_pool: bad sizes");
    SPK_REQUIRE(T <= 255, SPK_E_RANGE, "spk_pool: T=%d > 255", T);
    SPK_REQUIRE(kernel >= 1 && stride >= 1 && pad >= 0, SPK_E_SHAPE,
                "spk_pool: bad window %d / stride %d / pad %d", kernel, stride, pad);
    const int Ho = (H + 2 * pad - kernel) / stride + 1, Wo = (W + 2 * pad - kernel) / stride + 1;
    SPK_REQUIRE(H + 2 * pad >= kernel && W + 2 * pad >= kernel && Ho >= 1 && Wo >= 1, SPK_E_SHAPE,
                "spk_pool: window %d larger than the padded input", kernel);
    if (B == 0) return spk::ok();
    SPK_REQUIRE(wave && out_wave, SPK_E_ARG, "spk_pool: wave and out_wave are required");
    const int64_t per_img = (int64_t)C * Ho * Wo;
    SPK_REQUIRE(per_img <= 65535LL * 256 && (int64_t)C * H * W < (1LL << 31), SPK_E_RANGE, "spk_pool: image too large");
    const int64_t HW = (int64_t)H * W, hw = (int64_t)Ho * Wo;
    if (HW <= WL_BYTES && hw <= WL_QUADS * 1024 && Ho < 1024 && Wo < 1024) {  // whole maps through LDS
        const int CB = (int)std::min<int64_t>({(int64_t)C, WL_BYTES / HW, WL_QUADS * 1024 / hw, (int64_t)2047});
        const int64_t blocks = (int64_t)B * spk::ceil_div(C, CB);
        // Its workgroups are few and walk all steps with two barriers each: it pays once they
        // are about as many as the CUs, with 2x2 and 3x3 windows of whole maps; the other windows'
        // loops are slower and need twice that, large ones more.  Measured at T = 15 (an output per
        // thread : LDS, us): 30 maps of 28x28, 2x2, 16 images (48 workgroups) 9.7 : 11.5, 64 (192) 15.1 : 12.0;
        // 250 of 14x14, 3x3, 16 images (64) 14.8 : 23.4, 64 (256) 33 : 24; 64 of 64x64, 2x2, 4
        // images (128) 12.2 : 13.0, 8 (256) 20.5 : 13.3; 32 of 64x64, 5x5, 16 images (128)
        // 40 : 73, 64 (512) 84 : 77; 30 of 28x28, 3x3 stride 2 padded, 64 images (192) 27 : 72,
        // 256 (768) 112 : 79; 4 of 100x120, 7x7 stride 6, T = 30, 128 images (512) 207 : 249,
        // 256 (1024) 343 : 255.  (A launch has fewer than 2^32 threads.)
        const bool few_taps = pad == 0 && (kernel == 2 || kernel == 3);
        if (blocks >= (few_taps ? 192 : kernel <= 5 ? 512 : 640) && blocks < (1LL << 24)) {
#define SPK_POOL_WAVE(PW, IN)                                                                                          \
    hipLaunchKernelGGL((k_pool_lds<PW, IN>), dim3((unsigned)blocks), dim3(256), 0, spk::as_stream(stream), wave, T, C, \
                       H, W, kernel, stride, pad, Ho, Wo, CB, out_wave, out_t_first)
            if (pad > 0) SPK_POOL_WAVE(0, false);
            else if (kernel == 2) SPK_POOL_WAVE(2, true);
            else if (kernel == 3) SPK_POOL_WAVE(3, true);
            else SPK_POOL_WAVE(0, true);
#undef SPK_POOL_WAVE
            return spk::check_launch("spk_pool");
        }
    }
    hipLaunchKernelGGL(k_pool, dim3((unsigned)B, (unsigned)spk::ceil_div(per_img, 256)), dim3(256), 0,
                       spk::as_stream(stream), wave, T, C, H, W, kernel, stride, pad, Ho, Wo, out_wave, out_t_first);
    return spk::check_launch("spk_pool");
}
