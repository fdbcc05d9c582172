// gmc_device.hpp -- FP32 device building blocks of the gfx950 transport kernels:
// per-particle counter-based streams, log-grid table interpolation from LDS,
// voxel geometry, direction rotation and the interaction samplers.
//
// Every sampler consumes uniforms from the particle's own stream in a fixed
// order, so a particle's trajectory depends on its state and stream only,
// never on which lane, wavefront or pass runs it.
#pragma once
#include "gmc_internal.hpp"

namespace gmc {
namespace dev {

constexpr float kMc2 = 0.51099895f;                 // MeV
constexpr float kTwoPi = 6.28318530717958648f;
constexpr float kPi = 3.14159265358979324f;
constexpr float kLsbF = 7.450580596923828125e-09f;  // 2^-27 MeV per energy unit
constexpr float kInvLsbF = 134217728.0f;            // 2^27
constexpr float kU24 = 5.9604644775390625e-08f;     // 2^-24
constexpr float kInf = __builtin_huge_valf();
constexpr float kMaxLsbF = 4294967040.0f;           // largest float below 2^32
// Multiple scattering is drawn isotropically at or above this first moment.
constexpr float kG1Iso = 0.9999f;
constexpr float kLn2 = 0.693147180559945309f;
constexpr float kLog2e = 1.44269504088896341f;

// ---------------------------------------------------------------- fast FP32 forms
// Reciprocal, quotient, natural log and exponential of the transport as the
// hardware's v_rcp_f32, v_log_f32 (log2) and v_exp_f32 (exp2), each within
// about 1 ulp, and at most one multiply.  The general forms add range scaling
// for operands beyond 2^96 and an extended-precision ln 2 product; no operand
// here comes near such ranges (denormals are flushed, uniforms lie in
// [2^-24, 1), energies in [1 keV, 32 MeV], lengths and cross sections far
// inside), so those steps would only cost instructions.
__device__ __forceinline__ float frcp(float b) { return __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ float fdiv(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ float fln(float x) { return __builtin_amdgcn_logf(x) * kLn2; }
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

// ---------------------------------------------------------------- Philox4x32-10
struct Block { uint32_t w0, w1, w2, w3; };

__device__ __forceinline__ Block philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                        uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    // one 32x32->64 multiply each (a single v_mad_u64_u32)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    // three-input exclusive or as one gfx950 v_bitop3_b32 (truth table 0x96)
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
    c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
  }
  return Block{c0, c1, c2, c3};
}

// ---------------------------------------------------------------- lanes
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// The lanes with b set, straight from the comparison's mask (__ballot takes an
// integer: a select and a second comparison), and the number of set lanes of a
// mask below this one (two v_mbcnt, no mask of lower lanes kept).
__device__ __forceinline__ unsigned long long lanes_with(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool any_lane(bool b) { return __builtin_amdgcn_ballot_w64(b) != 0ull; }
__device__ __forceinline__ uint32_t rank_in(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ((w >> 8) | 1) 2^-24, formed without the shift: (w & ~255) | 256 is 256 times
// that integer, its conversion as exact and its scale a power of two.
__device__ __forceinline__ float to_uniform(uint32_t w) {
  return (float)((w & 0xffffff00u) | 0x100u) * (kU24 * 0.00390625f);
}

// Stream path of a child: splitmix64 finalizer of the parent path mixed with
// the parent's word counter at the spawning event and the child's index.
__device__ __forceinline__ void child_path(uint32_t plo, uint32_t phi, uint32_t n, uint32_t idx, uint32_t& olo,
                                           uint32_t& ohi) {
  uint64_t z = ((uint64_t)phi << 32) | (uint64_t)plo;
  z = (z ^ (((uint64_t)n << 2) | (uint64_t)idx)) + 0x9E3779B97F4A7C15ull;
  z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27; z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  olo = (uint32_t)z;
  ohi = (uint32_t)(z >> 32);
}

// A particle's stream: word n is word (n & 3) of Philox4x32-10 with counter
// (n >> 2, path lo, path hi, history) and key (seed lo, seed hi ^ beam id).
// Each event starts on a block boundary (align), so the block refresh falls on
// the same draw for every lane of a wavefront.
struct Stream {
  uint32_t k0, k1, plo, phi, hist, n;
  uint32_t b0, b1, b2, b3;

  __device__ __forceinline__ void align() { n = (n + 3u) & ~3u; }
  __device__ __forceinline__ uint32_t word() {
    const uint32_t j = n & 3u;
    if (j == 0) {
      const Block b = philox(n >> 2, plo, phi, hist, k0, k1);
      b0 = b.w0; b1 = b.w1; b2 = b.w2; b3 = b.w3;
    }
    const uint32_t wd = j == 0 ? b0 : (j == 1 ? b1 : (j == 2 ? b2 : b3));
    ++n;
    return wd;
  }
  __device__ __forceinline__ float uniform() { return to_uniform(word()); }
  // The same draw where n & 3 is known to be kPhase: no selection of the word,
  // and a block only where one begins.
  template <int kPhase>
  __device__ __forceinline__ float uniform_at() {
    if constexpr (kPhase == 0) {
      const Block b = philox(n >> 2, plo, phi, hist, k0, k1);
      b0 = b.w0; b1 = b.w1; b2 = b.w2; b3 = b.w3;
    }
    ++n;
    return to_uniform(kPhase == 0 ? b0 : kPhase == 1 ? b1 : kPhase == 2 ? b2 : b3);
  }
  // After a reload between two words of a block: recompute the cached block
  // the next draws come from (a particle stored at a block boundary needs
  // nothing).
  __device__ __forceinline__ void resume() {
    if (n & 3u) {
      const Block b = philox(n >> 2, plo, phi, hist, k0, k1);
      b0 = b.w0; b1 = b.w1; b2 = b.w2; b3 = b.w3;
    }
  }
};

// ---------------------------------------------------------------- tables
struct TPos { int i; float t; };

// Position of a transported particle's energy on the log-energy grid: node
// index i and fraction t.  Energies lie in [kEmin, 30 MeV], below the last
// node, so the position needs no upper limit and its fraction is one
// v_fract_f32 (the same bits as tpos below).
__device__ __forceinline__ TPos tpos_in(const DevTables& T, float e) {
  const float f = fmaxf((__log2f(e) - T.lg2_emin) * T.inv_h2, 0.0f);
  return TPos{(int)f, __builtin_amdgcn_fractf(f)};
}

// Position on the log-energy grid: node index i and fraction t in [0, 1].
__device__ __forceinline__ TPos tpos(const DevTables& T, float e) {
  float f = (__log2f(e) - T.lg2_emin) * T.inv_h2;
  f = fminf(fmaxf(f, 0.0f), (float)(kNE - 1));
  const int i = min((int)f, kNE - 2);
  return TPos{i, f - (float)i};
}

__device__ __forceinline__ float4 lerp4(const float4* tab, int base, TPos p) {
  const float4 a = tab[base + p.i];
  const float4 b = tab[base + p.i + 1];
  return make_float4(fmaf(p.t, b.x - a.x, a.x), fmaf(p.t, b.y - a.y, a.y), fmaf(p.t, b.z - a.z, a.z),
                     fmaf(p.t, b.w - a.w, a.w));
}

// The photon tables in LDS: kPhRow floats per node (the fourth of the node's
// float4 in memory is unused).
constexpr int kPhRow = 3;
__device__ __forceinline__ float3 lerp_ph(const float* tab, int base, TPos p) {
  const float* a = tab + (base + p.i) * kPhRow;
  return make_float3(fmaf(p.t, a[3] - a[0], a[0]), fmaf(p.t, a[4] - a[1], a[1]), fmaf(p.t, a[5] - a[2], a[2]));
}

__device__ __forceinline__ float lerp_x(const float4* tab, int base, TPos p) {
  const float a = tab[base + p.i].x;
  const float b = tab[base + p.i + 1].x;
  return fmaf(p.t, b - a, a);
}

__device__ __forceinline__ float lerp_w(const float4* tab, int base, TPos p) {
  const float a = tab[base + p.i].w;
  const float b = tab[base + p.i + 1].w;
  return fmaf(p.t, b - a, a);
}

// ---------------------------------------------------------------- geometry
__device__ __forceinline__ bool inside(const DevPhantom& P, float x, float y, float z) {
  return x >= 0.0f && x < P.lx && y >= 0.0f && y < P.ly && z >= 0.0f && z < P.lz;
}

// Number of voxel (ix, iy, iz) in tile order.
__device__ __forceinline__ uint32_t tiled(const DevTile& t, uint32_t ix, uint32_t iy, uint32_t iz) {
  const uint32_t tile = ((iz >> t.sz) * t.nby + (iy >> t.sy)) * t.nbx + (ix >> t.sx);
  const uint32_t lx = ix & ((1u << t.sx) - 1u), ly = iy & ((1u << t.sy) - 1u), lz = iz & ((1u << t.sz) - 1u);
  return (tile * kTallyBlock) | (ly << (t.sx + t.sz)) | (lz << t.sx) | lx;
}
// And back.
__device__ __forceinline__ void untiled(const DevTile& t, uint32_t v, uint32_t& ix, uint32_t& iy, uint32_t& iz) {
  const uint32_t w = v % kTallyBlock, tile = v / kTallyBlock;
  const uint32_t row = tile / t.nbx;
  ix = ((tile - row * t.nbx) << t.sx) | (w & ((1u << t.sx) - 1u));
  iz = ((row / t.nby) << t.sz) | ((w >> t.sx) & ((1u << t.sz) - 1u));
  iy = ((row % t.nby) << t.sy) | (w >> (t.sx + t.sz));
}

// Voxel of an inside point: floor(x / dx) per axis (a point on a face belongs
// to the voxel on its high side).
__device__ __forceinline__ uint32_t voxel(const DevPhantom& P, float x, float y, float z, int& ix, int& iy, int& iz) {
  ix = min((int)(x * P.idx), P.nx - 1);
  iy = min((int)(y * P.idy), P.ny - 1);
  iz = min((int)(z * P.idz), P.nz - 1);
  return tiled(P.tile, (uint32_t)ix, (uint32_t)iy, (uint32_t)iz);
}

// Voxel of an electron: each coordinate is advanced by the skin in the
// direction of travel before flooring, so a hinge endpoint left a hair short
// of the face it heads for counts as beyond it.  False when the advanced
// point is outside the phantom (the electron escapes); the voxel is then 0.
// No branch: a wavefront's electrons head all ways.  The advanced coordinate
// is never -0 (the skin and the spacing of the coordinates near it are far
// above the smallest float), so 0 <= q < l is one unsigned comparison.
__device__ __forceinline__ float skin_ahead(float x, float u, float sk) {
  return x + (u != 0.0f ? __builtin_copysignf(sk, u) : 0.0f);
}
__device__ __forceinline__ bool electron_voxel(const DevPhantom& P, float x, float y, float z, float u, float v,
                                               float w, int& ix, int& iy, int& iz, uint32_t& vox) {
  const float qx = skin_ahead(x, u, P.skin), qy = skin_ahead(y, v, P.skin), qz = skin_ahead(z, w, P.skin);
  const bool inx = __float_as_uint(qx) < __float_as_uint(P.lx), iny = __float_as_uint(qy) < __float_as_uint(P.ly),
             inz = __float_as_uint(qz) < __float_as_uint(P.lz);
  const bool in = (int)inx & (int)iny & (int)inz;
  const uint32_t v0 = voxel(P, qx, qy, qz, ix, iy, iz);
  vox = in ? v0 : 0u;
  return in;
}

// Distance along (u, v, w) to the boundary of voxel (ix, iy, iz): d_vox of
// Eq. 4.  An axis the direction does not move along has no boundary.
__device__ __forceinline__ float axis_distance(float x, float u, int i, float d) {
  const float t = fdiv((float)(i + (u > 0.0f ? 1 : 0)) * d - x, u);
  return u != 0.0f ? t : kInf;
}
__device__ __forceinline__ float dist_boundary(const DevPhantom& P, float x, float y, float z, float u, float v,
                                               float w, int ix, int iy, int iz) {
  const float t = fminf(fminf(axis_distance(x, u, ix, P.dx), axis_distance(y, v, iy, P.dy)),
                        axis_distance(z, w, iz, P.dz));
  return fmaxf(t, 0.0f);
}

// New direction at polar cosine cost and azimuth phi about (u, v, w),
// renormalised.
// Turn (u, v, w) by the polar angle with cosine cost and sine sint about the
// old direction, azimuth phi.
__device__ __forceinline__ void rotate_cs(float& u, float& v, float& w, float cost, float sint, float phi) {
  float sp, cp;
  __sincosf(phi, &sp, &cp);
  const float rho2 = u * u + v * v;
  const float r = sqrtf(rho2);
  const float ir = frcp(r);
  float nu = u * cost + sint * (u * w * cp - v * sp) * ir;
  float nv = v * cost + sint * (v * w * cp + u * sp) * ir;
  float nw = w * cost - r * sint * cp;
  const bool axis = !(rho2 > 1e-20f);   // along z: no azimuth of its own
  if (any_lane(axis)) {
    asm volatile("");   // rare: kept a scalar branch
    nu = axis ? sint * cp : nu;
    nv = axis ? sint * sp : nv;
    nw = axis ? (w >= 0.0f ? cost : -cost) : nw;
  }
  const float inv = rsqrtf(nu * nu + nv * nv + nw * nw);
  u = nu * inv; v = nv * inv; w = nw * inv;
}

__device__ __forceinline__ void rotate(float& u, float& v, float& w, float cost, float phi) {
  cost = fminf(fmaxf(cost, -1.0f), 1.0f);
  rotate_cs(u, v, w, cost, sqrtf((1.0f - cost) * (1.0f + cost)), phi);
}

// The same by om = 1 - cos(theta): for the small angles of a multiple-
// scattering step, cos(theta) rounded to FP32 keeps few digits of om, so the
// sine is formed from om itself, sin = sqrt(om (2 - om)).
__device__ __forceinline__ void rotate_om(float& u, float& v, float& w, float om, float phi) {
  om = fminf(fmaxf(om, 0.0f), 2.0f);
  rotate_cs(u, v, w, 1.0f - om, sqrtf(om * (2.0f - om)), phi);
}

__device__ __forceinline__ uint32_t to_lsb(float mev) {
  return (uint32_t)fminf(fmaxf(mev * kInvLsbF, 0.0f), kMaxLsbF);
}

// Rejection trials of three uniforms each until `trial` accepts.  Every lane
// that samples comes with the same stream phase (n & 3) of its first draw,
// kFirst, so each of the four trials that return to it knows its words: the
// selection of a word costs about ten instructions, and each draw had the code
// of a new block beside it.  With the draws of flights, hard events and
// absorptions alike: water job 25.46 -> 25.13 ms, 4e7 photons on 128^3 slabs
// 14.79 -> 14.48, 1e6 electrons 1.084 -> 1.052.
template <int kFirst, class F>
__device__ __forceinline__ void trials3(Stream& s, F&& trial) {
  for (;;) {
    float u1 = s.uniform_at<kFirst>(), u2 = s.uniform_at<(kFirst + 1) & 3>(), u3 = s.uniform_at<(kFirst + 2) & 3>();
    if (trial(u1, u2, u3)) return;
    u1 = s.uniform_at<(kFirst + 3) & 3>(), u2 = s.uniform_at<kFirst>(), u3 = s.uniform_at<(kFirst + 1) & 3>();
    if (trial(u1, u2, u3)) return;
    u1 = s.uniform_at<(kFirst + 2) & 3>(), u2 = s.uniform_at<(kFirst + 3) & 3>(), u3 = s.uniform_at<kFirst>();
    if (trial(u1, u2, u3)) return;
    u1 = s.uniform_at<(kFirst + 1) & 3>(), u2 = s.uniform_at<(kFirst + 2) & 3>(), u3 = s.uniform_at<(kFirst + 3) & 3>();
    if (trial(u1, u2, u3)) return;
  }
}

// ---------------------------------------------------------------- samplers
// Compton (Sec. II.A): Klein-Nishina epsilon = E'/E by composition-rejection,
// 1/eps with weight ln(1/eps0) and eps with weight (1 - eps0^2)/2, accepted
// with 1 - eps sin^2/(1 + eps^2).  Three uniforms per trial.
__device__ __forceinline__ void sample_kn(float k, Stream& s, float& eps, float& cost) {
  const float eps0 = frcp(1.0f + 2.0f * k);
  const float a1 = fln(1.0f + 2.0f * k);
  const float a2 = 0.5f * (1.0f - eps0 * eps0);
  const auto trial = [&](float u1, float u2, float u3) {
    const float e = (u1 * (a1 + a2) < a1) ? fexp(-a1 * u2) : sqrtf(eps0 * eps0 + (1.0f - eps0 * eps0) * u2);
    const float t = fdiv(1.0f - e, k * e);
    const float sin2 = t * (2.0f - t);
    const float g = 1.0f - fdiv(e * sin2, 1.0f + e * e);
    eps = e;
    cost = 1.0f - t;
    return u3 <= g;
  };
  trials3<2>(s, trial);
}

// Photoelectron polar cosine from the Sauter K-shell distribution (Sec. II.A):
// nu = 1 - cos from nu/(A+nu)^3 on [0, 2] by inversion, accepted with
// (2 - nu)(1/(A+nu) + B)/(2/A + 2 max(B, 0)).  Two uniforms per trial.
__device__ __forceinline__ float sample_sauter(float t, Stream& s) {
  const float g = 1.0f + t / kMc2;
  const float beta = fdiv(sqrtf(t * (t + 2.0f * kMc2)), t + kMc2);
  const float a = frcp(g * g * beta * (1.0f + beta));
  const float b = 0.5f * beta * g * (g - 1.0f) * (g - 2.0f);
  const float mx = fdiv(2.0f, a) + 2.0f * fmaxf(b, 0.0f);
  float nu;
  const auto trial = [&](float u1, float u2) {
    const float q = fdiv(2.0f * sqrtf(u1), a + 2.0f);
    nu = fdiv(q * a, 1.0f - q);
    const float f = (2.0f - nu) * (frcp(a + nu) + b);
    return u2 * mx <= f;
  };
  for (;;) {   // an absorption's first draw is word 2 of the flight's block
    float u1 = s.uniform_at<2>(), u2 = s.uniform_at<3>();
    if (trial(u1, u2)) break;
    u1 = s.uniform_at<0>();
    u2 = s.uniform_at<1>();
    if (trial(u1, u2)) break;
  }
  return 1.0f - nu;
}

// Pair electron polar cosine from (1 - beta cos)^-2 by inversion.
__device__ __forceinline__ float pair_cos(float t, float u) {
  const float g = 1.0f + t / kMc2;
  const float beta = fdiv(sqrtf(t * (t + 2.0f * kMc2)), t + kMc2);
  const float omb = frcp(g * g * (1.0f + beta));
  return fdiv(2.0f * u - 1.0f + beta, omb + 2.0f * beta * u);
}

// Moller energy fraction in [kcut/T, 1/2] (Sec. II.B.1): 1/eps^2 and flat
// components, accepted with h(eps)/(1 + 5 eps^2).  Three uniforms per trial.
__device__ __forceinline__ float sample_moller(float t, float kcut, Stream& s) {
  const float tau = t / kMc2, g = tau + 1.0f;
  const float e0 = fdiv(kcut, t);
  const float r2 = fdiv(tau, g) * fdiv(tau, g);
  const float c = fdiv(2.0f * tau + 1.0f, g * g);
  const float ie0 = frcp(e0);
  const float w1 = ie0 - 2.0f, w2 = 5.0f * (0.5f - e0);
  float eps;
  trials3<1>(s, [&](float u1, float u2, float u3) {
    eps = (u1 * (w1 + w2) < w1) ? frcp(ie0 - u2 * (ie0 - 2.0f)) : e0 + u2 * (0.5f - e0);
    const float q = fdiv(eps, 1.0f - eps);
    const float h = 1.0f + q * q + r2 * eps * eps - c * q;
    return u3 * (1.0f + 5.0f * eps * eps) <= h;
  });
  return eps;
}

// Bremsstrahlung photon energy in [kc, T] (Sec. II.B.1): log-uniform proposal
// accepted with (4/3 - 4y/3 + y^2)/(4/3), y = k/E.  Two uniforms per trial.
__device__ __forceinline__ float sample_brems(float t, float kc, Stream& s) {
  const float e = t + kMc2;
  const float lr = fln(fdiv(t, kc));
  const auto trial = [&](float u1, float u2, float& k) {
    k = kc * fexp(u1 * lr);
    const float y = fdiv(k, e);
    return u2 * (4.0f / 3.0f) <= 4.0f / 3.0f - (4.0f / 3.0f) * y + y * y;
  };
  float k;
  for (;;) {
    float u1 = s.uniform_at<1>(), u2 = s.uniform_at<2>();
    if (trial(u1, u2, k)) break;
    u1 = s.uniform_at<3>();
    u2 = s.uniform_at<0>();
    if (trial(u1, u2, k)) break;
  }
  return k;
}

// Screening parameter A of the step's screened-Rutherford angular shape for a
// first moment G1 (Sec. II.B.2), from the table of ln A at logit(G1); outside
// the table its end segments are extended.  Any G1 (0, 1) reads in bounds.
__device__ __forceinline__ float screening_A(const DevTables& T, const float* ms, float g1) {
  const float y = fln(fdiv(g1, 1.0f - g1));
  const float f = (y - T.ms_y0) * T.ms_inv_dy;
  const float fi = fminf(fmaxf(floorf(f), 0.0f), (float)(kNms - 2));
  const int i = (int)fi;
  return fexp(fmaf(f - fi, ms[i + 1] - ms[i], ms[i]));
}

// 1 - cos(theta) of a multiple-scattering step (Wentzel shape with screening
// A from G1): om = 2 A u / (1 + A - u); isotropic above the G1 limit, none at
// G1 = 0 (selected at the end: the lanes of a wavefront take all three).  The
// denominator is formed as (1 - u) + A: u is an odd multiple of 2^-24, so
// 1 - u is exact in FP32, whereas 1 + A rounds A away when A < 2^-24 (short
// steps, low density) and fattens the large-angle tail.
__device__ __forceinline__ float wentzel_om(const DevTables& T, const float* ms, float g1, float u) {
  const float a = screening_A(T, ms, g1);
  float om = fdiv(2.0f * a * u, (1.0f - u) + a);
  om = g1 >= kG1Iso ? 2.0f * u : om;
  return g1 > 0.0f ? om : 0.0f;
}

// ---------------------------------------------------------------- wave helpers
// Orders memory that a wavefront's lanes write and its other lanes read (or
// write again) later.  A wavefront's own vector memory operations on one
// address take effect in the order it issues them, so this only keeps the
// compiler from reordering them.
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// A wavefront's private segment of cap staging entries from p on, filled from
// the bottom (used entries, wave-uniform) and, with parked photons, from the
// top.  Each lane appends 0, 1 or 2 entries; the
// slots follow lane order, so no atomic is needed.
struct WaveSeg {
  uint4* p;
  uint32_t cap, used;
  struct Slots { uint32_t s0, s1; };
  __device__ __forceinline__ Slots append(bool want0, bool want1) {
    const unsigned long long m0 = lanes_with(want0);
    const unsigned long long m1 = lanes_with(want1);
    const uint32_t n0 = (uint32_t)__popcll(m0);
    Slots r;
    r.s0 = used + rank_in(m0);
    r.s1 = used + n0 + rank_in(m1);
    used += n0 + (uint32_t)__popcll(m1);
    return r;
  }
  // granule 0 of entry i (a segment is far smaller than 4 GB: 32-bit offsets
  // from a uniform base)
  __device__ __forceinline__ uint4* at(uint32_t i) const {
    return p + (uint32_t)((i / kQBlock) * (kQBlock * kStgGranules) + (i % kQBlock));
  }
};

// Granule 0 of entry i of a queue of G granules per entry (granule g is
// 64 g further on).
template <int G>
__device__ __forceinline__ const uint4* entry(const uint4* base, uint32_t i) {
  return base + (size_t)(i / kQBlock) * (kQBlock * G) + (i % kQBlock);
}
template <int G>
__device__ __forceinline__ uint4* entry(const DevQueue& q, uint32_t i) {
  return q.base + (size_t)(i / kQBlock) * (kQBlock * G) + (i % kQBlock);
}
// The segment of n entries from entry first (a multiple of kQBlock) of a staging queue.
__device__ __forceinline__ WaveSeg wave_seg(const DevQueue& q, uint32_t first, uint32_t n) {
  return WaveSeg{q.base + (size_t)first * kStgGranules, n, 0u};
}
// Index of the calling wavefront in the grid, as a scalar.
__device__ __forceinline__ uint32_t wave_index() {
  return __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
}

__device__ __forceinline__ void put(uint4* p, float x, float y, float z, float u, float v, float w, uint32_t e,
                                    uint32_t hist, uint32_t plo, uint32_t phi, uint32_t n, uint32_t beam) {
  p[QG_POS * kQBlock] = make_uint4(__float_as_uint(x), __float_as_uint(y), __float_as_uint(z), e);
  p[QG_DIR * kQBlock] = make_uint4(__float_as_uint(u), __float_as_uint(v), __float_as_uint(w), beam);
  p[QG_STREAM * kQBlock] = make_uint4(hist, plo, phi, n);
}

// Add to run counter `idx` in the slot of the calling wavefront.
__device__ __forceinline__ void ctr_add(unsigned long long* ctr, int idx, unsigned long long v) {
  const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  atomicAdd(&ctr[idx * kCtrSlots + (wave & (kCtrSlots - 1))], v);
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)v, off);
    const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), off);
    v += ((unsigned long long)hi << 32) | lo;
  }
  return v;
}

}  // namespace dev
}  // namespace gmc
