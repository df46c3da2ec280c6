// Shading of a pixel from its winning triangle: colour (vertex colours or
// texture), depth noise, and the write-out of a band of pixels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_util.h"

#pragma clang fp contract(off)

namespace habmi {

// Triangle t's N attribute words.
template <int N>
__device__ __forceinline__ void load_attr(const DView &v, uint32_t t, uint32_t (&q)[N])
{
    const auto *p = gmem(v.attr) + (uint64_t)N * t;
#pragma unroll
    for (int k = 0; k < N; ++k) q[k] = p[k];
}

__device__ __forceinline__ float f32(uint32_t x) { return __uint_as_float(x); }

// x / num for num > 0, correctly rounded as the division is: from r, the
// correctly rounded 1/num, by two steps of the exact remainder (Markstein: the
// second starts within an ulp of x / num).  Holds while no step under- or
// overflows: 2^-60 <= num <= 2^60, and x zero or of magnitude 2^-60 to 2^68.
// Callers with x below that range use it only where x / num < 2^-40 rounds away.
constexpr float kDivLo = 0x1p-60f, kDivHi = 0x1p60f;
__device__ __forceinline__ float div_by(float x, float num, float r)
{
    const float q = x * r;
    const float q1 = __builtin_fmaf(__builtin_fmaf(-q, num, x), r, q);
    return __builtin_fmaf(__builtin_fmaf(-q1, num, x), r, q1);
}

// Perspective-correct weights of pixel (i, j), which the triangle covers, for a
// triangle in front of the near plane (false: it is not, or leaves the
// fixed-point domain).  Vertices are snapped as the raster does; at a covered
// pixel the three edge functions have the sign of the area, so their magnitudes
// are those of the oriented triangle, and the orientation (swapped: vertices 1
// and 2 change places) is that sign.  w0, w1, w2 are in oriented order.
__device__ __forceinline__ bool pixel_weights(const DView &v, const float P[9], int i, int j, float &w0, float &w1,
                                              float &w2, bool &swapped)
{
    Vtx<0> c0, c1, c2;
    cam_xform(v, P[0], P[1], P[2], c0);
    cam_xform(v, P[3], P[4], P[5], c1);
    cam_xform(v, P[6], P[7], P[8], c2);
    if (!(c0.w >= v.zn && c1.w >= v.zn && c2.w >= v.zn)) return false;
    SVtx<0> a, b, c;
    bool ok = snap(v, c0, a);
    ok &= snap(v, c1, b);
    ok &= snap(v, c2, c);
    if (!ok) return false;
    const int px = 256 * i + 128, py = 256 * j + 128;
    const int ax = a.X - px, ay = a.Y - py, bx = b.X - px, by = b.Y - py, cx = c.X - px, cy = c.Y - py;
    constexpr int kNear = 1 << 14;
    float fa, fb, fc;
    if (abs(ax) < kNear && abs(ay) < kNear && abs(bx) < kNear && abs(by) < kNear && abs(cx) < kNear &&
        abs(cy) < kNear) {
        // within 64 px: 24-bit products, |E| < 2^30
        const int ea = __mul24(bx, cy) - __mul24(by, cx), eb = __mul24(cx, ay) - __mul24(cy, ax),
                  ec = __mul24(ax, by) - __mul24(ay, bx);
        swapped = (ea | eb | ec) < 0;
        fa = (float)abs(ea);
        fb = (float)abs(eb);
        fc = (float)abs(ec);
    } else {
        const long long ea = (long long)bx * cy - (long long)by * cx, eb = (long long)cx * ay - (long long)cy * ax,
                        ec = (long long)ax * by - (long long)ay * bx;
        swapped = (ea | eb | ec) < 0;
        fa = fabsf((float)ea);
        fb = fabsf((float)eb);
        fc = fabsf((float)ec);
    }
    w0 = fa * a.rw;
    const float ub = fb * b.rw, uc = fc * c.rw;
    w1 = swapped ? uc : ub;
    w2 = swapped ? ub : uc;
    return true;
}

// Colour of the winner at pixel (i, j): the triangle's setup rebuilt with the
// same arithmetic as the raster's, its three edge functions at the pixel
// centre give the perspective-correct weights (the depth comes from the
// winning key's 1/w, the same value).
__device__ __forceinline__ bool resolve(const DView &v, uint32_t key, int i, int j, uint32_t rgb[3])
{
    const uint32_t t = key >> 1;
    const int sub = (int)(key & 1u);
    float P[9];
    uint32_t q[3];
    load_pos(v, t, P);
    load_attr(v, t, q);
    const uint32_t k0 = q[0], k1 = q[1], k2 = q[2];
    float w0, w1, w2, x[3], num;
    bool swapped;
    if (sub == 0 && pixel_weights(v, P, i, j, w0, w1, w2, swapped)) {
        const uint32_t kb = swapped ? k2 : k1, kc = swapped ? k1 : k2;
        num = (w0 + w1) + w2;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch)
            x[ch] = (w0 * (float)unpack_rgb(k0, ch) + w1 * (float)unpack_rgb(kb, ch)) + w2 * (float)unpack_rgb(kc, ch);
    } else {
        Vtx<3> c0, c1, c2;
        cam_xform(v, P[0], P[1], P[2], c0);
        cam_xform(v, P[3], P[4], P[5], c1);
        cam_xform(v, P[6], P[7], P[8], c2);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            c0.a[ch] = (float)unpack_rgb(k0, ch);
            c1.a[ch] = (float)unpack_rgb(k1, ch);
            c2.a[ch] = (float)unpack_rgb(k2, ch);
        }
        SVtx<3> a = {}, b = {}, c = {};
        long long A = 1;
        bool rerr = false;
        if (!setup_sub(v, c0, c1, c2, sub, a, b, c, A, rerr)) {
            // unreachable: the key came from a successful setup of the same
            // arithmetic; report it as a device fault rather than guess
            rgb[0] = rgb[1] = rgb[2] = 0;
            return false;
        }
        const long long px = 256ll * i + 128, py = 256ll * j + 128;
        const long long E0 = edge_at(b.X, b.Y, c.X, c.Y, px, py);
        const long long E1 = edge_at(c.X, c.Y, a.X, a.Y, px, py);
        const long long E2 = edge_at(a.X, a.Y, b.X, b.Y, px, py);
        w0 = (float)E0 * a.rw;
        w1 = (float)E1 * b.rw;
        w2 = (float)E2 * c.rw;
        num = (w0 + w1) + w2;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) x[ch] = (w0 * a.a[ch] + w1 * b.a[ch]) + w2 * c.a[ch];
    }
    float val[3];
    if (__builtin_expect(num >= kDivLo && num <= kDivHi, 1)) {
        const float r = recip_rn(num);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) val[ch] = div_by(x[ch], num, r);
    } else {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) val[ch] = x[ch] / num;
    }
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) rgb[ch] = (uint32_t)fminf(fmaxf(rintf(val[ch]), 0.0f), 255.0f);
    return true;
}

// Textured colour: the texture coordinates ride through the clip and the
// perspective-correct interpolation exactly as colours do (same fp32
// sequence), then a bilinear fetch with texel centres at (k + 1/2) / size,
// coordinates repeating.  For a power-of-two size and |u| size < 2^22,
// u * size - 1/2 and its fraction are exact in fp32, so only the blend's
// rounding differs from an fp64 evaluation.
__device__ __forceinline__ void tex_bilinear(const DView &v, float u, float t, uint32_t rgb[3])
{
    const float x = u * (float)v.tex_w - 0.5f, y = t * (float)v.tex_h - 0.5f;
    const float xf = floorf(x), yf = floorf(y);
    const float fx = x - xf, fy = y - yf;
    const int xi = (int)xf, yi = (int)yf;
    const uint32_t wm = v.tex_w - 1u, hm = v.tex_h - 1u;
    const uint32_t i0 = (uint32_t)xi & wm, i1 = (uint32_t)(xi + 1) & wm;
    const uint32_t r0 = ((uint32_t)yi & hm) * v.tex_w, r1 = ((uint32_t)(yi + 1) & hm) * v.tex_w;
    const auto *tex = gmem(v.tex);
    const uint32_t t00 = tex[r0 + i0], t10 = tex[r0 + i1], t01 = tex[r1 + i0], t11 = tex[r1 + i1];
    const float gx = 1.0f - fx, gy = 1.0f - fy;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float c00 = (float)unpack_rgb(t00, ch), c10 = (float)unpack_rgb(t10, ch);
        const float c01 = (float)unpack_rgb(t01, ch), c11 = (float)unpack_rgb(t11, ch);
        float val = gy * (gx * c00 + fx * c10) + fy * (gx * c01 + fx * c11);
        val = rintf(val);
        rgb[ch] = (uint32_t)fminf(fmaxf(val, 0.0f), 255.0f);
    }
}

// resolve() for a textured scene: the same rebuild of the winner with the
// texture coordinates as its two attributes.
__device__ __forceinline__ bool resolve_tex(const DView &v, uint32_t key, int i, int j,
                                            uint32_t rgb[3])
{
    const uint32_t t = key >> 1;
    const int sub = (int)(key & 1u);
    float P[9];
    uint32_t q[6];
    load_pos(v, t, P);
    load_attr(v, t, q);
    const float a0[2] = {f32(q[0]), f32(q[1])}, a1[2] = {f32(q[2]), f32(q[3])}, a2[2] = {f32(q[4]), f32(q[5])};
    float w0, w1, w2, x[2], num;
    bool swapped;
    if (sub == 0 && pixel_weights(v, P, i, j, w0, w1, w2, swapped)) {
        num = (w0 + w1) + w2;
#pragma unroll
        for (int k = 0; k < 2; ++k)
            x[k] = (w0 * a0[k] + w1 * (swapped ? a2[k] : a1[k])) + w2 * (swapped ? a1[k] : a2[k]);
    } else {
        Vtx<2> c0, c1, c2;
        cam_xform(v, P[0], P[1], P[2], c0);
        cam_xform(v, P[3], P[4], P[5], c1);
        cam_xform(v, P[6], P[7], P[8], c2);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            c0.a[k] = a0[k];
            c1.a[k] = a1[k];
            c2.a[k] = a2[k];
        }
        SVtx<2> a = {}, b = {}, c = {};
        long long A = 1;
        bool rerr = false;
        if (!setup_sub(v, c0, c1, c2, sub, a, b, c, A, rerr)) {
            rgb[0] = rgb[1] = rgb[2] = 0;
            return false;
        }
        const long long px = 256ll * i + 128, py = 256ll * j + 128;
        const long long E0 = edge_at(b.X, b.Y, c.X, c.Y, px, py);
        const long long E1 = edge_at(c.X, c.Y, a.X, a.Y, px, py);
        const long long E2 = edge_at(a.X, a.Y, b.X, b.Y, px, py);
        w0 = (float)E0 * a.rw;
        w1 = (float)E1 * b.rw;
        w2 = (float)E2 * c.rw;
        num = (w0 + w1) + w2;
#pragma unroll
        for (int k = 0; k < 2; ++k) x[k] = (w0 * a.a[k] + w1 * b.a[k]) + w2 * c.a[k];
    }
    float uvp[2];
    const float m0 = fabsf(x[0]), m1 = fabsf(x[1]);
    if (__builtin_expect(num >= kDivLo && num <= kDivHi && (m0 == 0.0f || (m0 >= kDivLo && m0 <= kDivHi)) &&
                             (m1 == 0.0f || (m1 >= kDivLo && m1 <= kDivHi)),
                         1)) {
        const float r = recip_rn(num);
        uvp[0] = div_by(x[0], num, r);
        uvp[1] = div_by(x[1], num, r);
    } else {
        uvp[0] = x[0] / num;
        uvp[1] = x[1] / num;
    }
    tex_bilinear(v, uvp[0], uvp[1], rgb);
    return true;
}

// Depth noise (the appendix's noise study): a standard normal deviate per
// pixel, added to the inverse depth times the sensor's sigma.  Philox4x64
// with 10 rounds (Salmon, Moraes, Dror and Shaw, SC 2011) keyed by (view
// seed, stream tag), counter (pixel index, 0, 0, 0), so each pixel draws on
// its own, whatever thread renders it; the top 24 bits of the first two
// words feed the Box-Muller transform.
constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull;   // Weyl key increments
constexpr uint64_t kPhiloxW1 = 0xBB67AE8584CAA73Bull;
constexpr uint64_t kDepthNoiseTag = 0x6465707468ull;    // "depth"

__device__ __forceinline__ float depth_noise_normal(uint64_t seed, uint64_t pixel)
{
    uint64_t c0 = pixel, c1 = 0, c2 = 0, c3 = 0;
    uint64_t k0 = seed, k1 = kDepthNoiseTag;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t hi0 = __umul64hi(kPhiloxM0, c0), lo0 = kPhiloxM0 * c0;
        const uint64_t hi1 = __umul64hi(kPhiloxM1, c2), lo1 = kPhiloxM1 * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
    const float u1 = (float)((uint32_t)(c0 >> 40) + 1u) * 0x1p-24f;   // (0, 1]
    const float u2 = (float)(uint32_t)(c1 >> 40) * 0x1p-24f;          // [0, 1)
    return sqrtf(-2.0f * logf(u1)) * cospif(2.0f * u2);
}

// Bands: 32 x 2 pixels of one view per wave, one lane per pixel.  A band row
// is 96 bytes of RGB at a multiple of 96 (three whole 32-byte sectors) and
// 128 bytes of depth, index or instance (one whole line): the RGB bytes go
// through LDS so that the wave stores them as words, and every sector the
// band writes is written once and whole.
constexpr int kBandW = 32, kBandH = 2;
constexpr int kBandThreads = kBandW * kBandH;   // one wave
constexpr int kBandRgb = kBandH * kBandW * 3;   // bytes of LDS a band's colours take

// Shade and write one band, BW x BH pixels (this lane's pixel (pi, pj), `in` the view, of the
// band at (x0, y0)) from each pixel's winner (best_key, or kNone, with its
// 1/w best_rho).
template <int BW, int BH>
__device__ __forceinline__ void shade_band(const DView &v, uint32_t x0, uint32_t y0, int pi, int pj, bool in,
                                           float best_rho, uint32_t best_key, uint8_t *s_rgb,
                                           uint32_t *__restrict__ err)
{
    const uint32_t W = v.W, H = v.H, lane = lane_id();
    uint32_t rgb[3] = {0, 0, 0};
    if (in) {
        float depth = 0.0f;
        if (best_key != kNone) {
            // the depth is the reciprocal of the winning key's 1/w (the value
            // a rebuild of the triangle would compute again); colour needs
            // the rebuild
            depth = recip_rn(best_rho);
            if (v.rgb && !(v.tex ? resolve_tex(v, best_key, pi, pj, rgb) : resolve(v, best_key, pi, pj, rgb)))
                atomicOr(err, kErrResolve);
        }
        const size_t p = (size_t)pj * W + (size_t)pi;
        if (v.noise_sigma > 0.0f && best_key != kNone) {
            const float rp = best_rho + v.noise_sigma * depth_noise_normal(v.noise_seed, (uint64_t)p);
            depth = rp > 0.0f ? recip_rn(rp) : 0.0f;
        }
        if (v.depth) gmem_out(v.depth)[p] = depth;
        if (v.tri) gmem_out(v.tri)[p] = best_key == kNone ? kNone : (best_key >> 1);
        if (v.sem) gmem_out(v.sem)[p] = best_key == kNone ? kNone : gmem(v.inst)[best_key >> 1];
    }
    if (!v.rgb) return;
    auto *o = gmem_out(v.rgb);
    const uint32_t wpx = min((uint32_t)BW, W - x0), rows = min((uint32_t)BH, H - y0);
    if ((W % 4u) == 0 && (reinterpret_cast<uintptr_t>(v.rgb) % 4u) == 0) {
        // rows of 3 wpx bytes start on a word (the image does, W and x0 are
        // multiples of 4): stage the band's bytes, store words
        constexpr uint32_t kRowWords = BW * 3u / 4u;   // 24
        s_rgb[3 * lane] = (uint8_t)rgb[0];
        s_rgb[3 * lane + 1] = (uint8_t)rgb[1];
        s_rgb[3 * lane + 2] = (uint8_t)rgb[2];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t r = lane / kRowWords, d = lane % kRowWords;
        if (lane < BH * kRowWords && r < rows && d < wpx * 3u / 4u) {
            auto *dst = reinterpret_cast<__attribute__((address_space(1))) uint32_t *>(
                o + ((size_t)(y0 + r) * W + x0) * 3u);
            dst[d] = reinterpret_cast<const uint32_t *>(s_rgb)[lane];
        }
    } else if (in) {
        auto *q = o + 3 * ((size_t)pj * W + (size_t)pi);
        q[0] = (uint8_t)rgb[0];
        q[1] = (uint8_t)rgb[1];
        q[2] = (uint8_t)rgb[2];
    }
}

}  // namespace habmi
