// Shading of a pixel from its winning triangle: colour (vertex colours or
// texture), depth noise, and the write-out of a band of pixels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_util.h"

#pragma clang fp contract(off)

namespace habmi {

// Colour, depth and index of the winning sub-triangle at pixel (i, j):
// the winner's setup is rebuilt with colours, its three edge functions at
// the pixel centre give the perspective-correct weights.
// Colour of the winner at pixel (i, j): the triangle's setup rebuilt with
// the same arithmetic as the raster's (the depth comes from the winning
// key's 1/w, the same value).
__device__ __forceinline__ bool resolve(const DView &v, uint32_t key, int i, int j, uint32_t rgb[3])
{
    const uint32_t t = key >> 1;
    const int sub = (int)(key & 1u);
    float P[9];
    uint32_t vid[3];
    load_tri(v, t, P, vid);
    Vtx<3> c0, c1, c2;
    cam_xform(v, P[0], P[1], P[2], c0);
    cam_xform(v, P[3], P[4], P[5], c1);
    cam_xform(v, P[6], P[7], P[8], c2);
    const uint32_t k0 = v.col ? gmem(v.col)[vid[0]] : 0xFFFFFFu;
    const uint32_t k1 = v.col ? gmem(v.col)[vid[1]] : 0xFFFFFFu;
    const uint32_t k2 = v.col ? gmem(v.col)[vid[2]] : 0xFFFFFFu;
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
    const float w0 = (float)E0 * a.rw, w1 = (float)E1 * b.rw, w2 = (float)E2 * c.rw;
    const float num = (w0 + w1) + w2;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        float val = ((w0 * a.a[ch] + w1 * b.a[ch]) + w2 * c.a[ch]) / num;
        val = rintf(val);
        val = fminf(fmaxf(val, 0.0f), 255.0f);
        rgb[ch] = (uint32_t)val;
    }
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
    uint32_t vid[3];
    load_tri(v, t, P, vid);
    Vtx<2> c0, c1, c2;
    cam_xform(v, P[0], P[1], P[2], c0);
    cam_xform(v, P[3], P[4], P[5], c1);
    cam_xform(v, P[6], P[7], P[8], c2);
    const auto *uv = gmem(v.uv);
    c0.a[0] = uv[2u * vid[0]];
    c0.a[1] = uv[2u * vid[0] + 1u];
    c1.a[0] = uv[2u * vid[1]];
    c1.a[1] = uv[2u * vid[1] + 1u];
    c2.a[0] = uv[2u * vid[2]];
    c2.a[1] = uv[2u * vid[2] + 1u];
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
    const float w0 = (float)E0 * a.rw, w1 = (float)E1 * b.rw, w2 = (float)E2 * c.rw;
    const float num = (w0 + w1) + w2;
    const float u = ((w0 * a.a[0] + w1 * b.a[0]) + w2 * c.a[0]) / num;
    const float tv = ((w0 * a.a[1] + w1 * b.a[1]) + w2 * c.a[1]) / num;
    tex_bilinear(v, u, tv, rgb);
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
            depth = 1.0f / best_rho;
            if (v.rgb && !(v.tex ? resolve_tex(v, best_key, pi, pj, rgb) : resolve(v, best_key, pi, pj, rgb)))
                atomicOr(err, kErrResolve);
        }
        const size_t p = (size_t)pj * W + (size_t)pi;
        if (v.noise_sigma > 0.0f && best_key != kNone) {
            const float rp = best_rho + v.noise_sigma * depth_noise_normal(v.noise_seed, (uint64_t)p);
            depth = rp > 0.0f ? 1.0f / rp : 0.0f;
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
