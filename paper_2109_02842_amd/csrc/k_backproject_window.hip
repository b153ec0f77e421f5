// Back-projection onto horizontal-plane pixels, eq. (8b) / (19b), on the
// matrix cores at FP32-class error (the whole-call form of the FP32 plans).
//
// For one channel c and a 4x4 pixel group every pixel's range lies in a short
// interval, so the profile at all sixteen pixels follows from the same eight
// range samples: q(x) = sum_s w_s(x) q[sr + s], w_s the least-squares weights
// over the band of k' (polynomials in the pixel's position x in the window,
// window_design in plan.cpp; no prefilter).  With B[s][p] = w_s(x_p) e^{j k_ref l_c(p)},
//   G[kz][p] += sum_s Q_c[kz][s] B_c[s][p]
// is a dense product: 32 k_z x (8 samples x (Re, Im)) by (8 x 2) x (16 pixels
// x (Re, Im)), K = 16 of v_mfma_f32_32x32x16_f16.  Both operands are FP16
// pairs hi + lo (22 significant bits; the profiles carry one power of two for
// the whole call) and each output part takes hi*hi + lo*hi + hi*lo,
// accumulated in FP32.
//
// The four-tap B-spline needs six times the Nyquist rate of range samples and
// 12 FMA per term; here half its error needs 2.5 to 5 times the rate.
//
// Workgroup: 16x16 pixels x 64 k_z rows, eight wavefronts, each 8x4 pixels
// (two groups) x all rows (64 accumulator registers, two workgroups per CU).
// The 64 rows of block b are k_z bins [32 b, 32 b + 32) and their mirrors
// n - 1 - kz: k_rho depends on k_z^2, so the block spans the band of 32 bins
// (one reference wavenumber) and B is formed once for 64 rows.  Row tiles of
// 32: bins 16 t .. 16 t + 15 and their mirrors.
//
// What bounds it: the matrix cores and the VALU of a SIMD hardly overlap (a
// few VALU instructions hide in a wavefront's own 32-cycle products, another
// wavefront's add to them).  Per (group, channel, 64 rows) the products take
// 6 x 32 = 192 cycles and the VALU, forming B for the most part, 235, of 400 in
// all (counters at 256 k_z x 320 channels x 200x200 pixels).  Measured there
// 0.72 ms where the pixel-per-lane gather takes 1.38, and at 512 x 896 x
// 256x256 6.5 ms (14.4).  16x16x32 products with four wavefronts
// took 0.80 ms, with eight 0.72 but more VGPRs than 32x32x16 leave; copies
// spread over the loop, or staged through registers, changed nothing.
//
// The window rows of a channel pair are copied into LDS by 16-byte direct
// loads one pair ahead (double buffer, one barrier per pair).  An LDS row
// holds the hi plane, the lo plane (WCH chunks of 16 bytes each) and one chunk
// of padding: an odd number of chunks, so that the rows of an operand read
// fall on distinct banks.
//
// Lane row r = lane / 16, pn = lane % 16: B is formed for pixel pn of group
// r & 1 and channel r >> 1 of the pair, all eight samples.  v_permlane32_swap
// then leaves samples 0..3 in lanes 0..31 and 4..7 in the upper ones, and
// v_permlane16_swap with the turned words (Im, Re) makes both groups' operands.
#include <algorithm>
#include <atomic>
#include <cstring>

#include "device.hpp"

namespace pl {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// window starts are any sample: 8-byte reads at 4-byte alignment
typedef unsigned int u32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kWaves = 8;
constexpr int kTile = 16;
constexpr int kRows = 2 * kWindowBins;   // 64 k_z rows per workgroup
constexpr int kDeg = kWindowDegree;
constexpr int kMaxThreads = 1024;        // per workgroup of the spectrum maximum

struct WinArgs {
    int n_ch, n_z, n_l, nx, ny, tiles_x, n_tiles, n_work, per_xcd;
    // as in the other matrix-core back-projection: items [0, n_whole) run
    // whole, each later one in n_part pieces over its channel pairs
    int n_whole, grid_whole, n_part, n_pair, per_xcd_tail;
    float dx, dy, inv_du, zscale, centre;   // centre: half the group span minus 3.5 samples
    float even[kDeg][4], odd[kDeg][4];
    int log2_gain;
};

// One call's arguments; pointers into its workspace.
struct WinCall {
    WinArgs a;
    const float* smax;   // parts of the largest |S| part (profile_exponent)
    float2* part;        // partial spectra of split items
    float kref_rev[kMaxBlocks / 2];
};

// One scan of a batch: its arguments, and byte offsets in the batch workspace.
struct WinScanDesc {
    WinArgs a;
    float kref_rev[kMaxBlocks / 2];
    unsigned long long q_off, tab_off, g_off, part_off, smax_off;
};

typedef __attribute__((address_space(3))) unsigned char* lds_bytes_t;
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) GatherTileEntry* const_tile_t;
#define PL_LDS_COPY16(RS, DST, VOFF) __builtin_amdgcn_raw_ptr_buffer_load_lds((RS), (DST), 16, (VOFF), 0, 0, 0)
#define PL_GLOBAL_LDS16(SRC, DST) __builtin_amdgcn_global_load_lds((SRC), (DST), 16, 0, 0)
__device__ __forceinline__ u32x2 swap16(unsigned a, unsigned b) {
    // odd rows of a exchanged with even rows of b (rows of 16 lanes)
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(a, b, false, false));
}
__device__ __forceinline__ u32x2 swap32(unsigned a, unsigned b) {
    // lanes 32..63 of a exchanged with lanes 0..31 of b
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(a, b, false, false));
}
__device__ __forceinline__ unsigned turned(unsigned v, unsigned sgn) {
    unsigned r;
    asm("v_pk_mul_f16 %0, %1, %2 op_sel:[1,0] op_sel_hi:[0,1]" : "=v"(r) : "v"(v), "s"(sgn));
    return r;
}
#else
// host pass: parsed only, never run (the builtins are device-only)
typedef const GatherTileEntry* const_tile_t;
#define PL_LDS_COPY16(RS, DST, VOFF) ((void)(RS), (void)(DST), (void)(VOFF))
#define PL_GLOBAL_LDS16(SRC, DST) ((void)(SRC), (void)(DST))
__device__ inline u32x2 swap16(unsigned a, unsigned b) { return u32x2{a, b}; }
__device__ inline u32x2 swap32(unsigned a, unsigned b) { return u32x2{a, b}; }
__device__ inline unsigned turned(unsigned v, unsigned) { return v; }
#endif

constexpr int kBufferFlags = 0x00020000;   // gfx9 raw-buffer descriptor word 3

__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const unsigned* p, unsigned bytes) {
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(a));
    const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(a >> 32));
    void* u = reinterpret_cast<void*>((static_cast<unsigned long long>(hi) << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(u, 0, __builtin_amdgcn_readfirstlane(bytes), kBufferFlags);
}

__device__ __forceinline__ unsigned pack_f16(float lo, float hi) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{lo, hi}), f16x2));
}
__device__ __forceinline__ float f16_lo(unsigned v) { return static_cast<float>(__builtin_bit_cast(f16x2, v)[0]); }
__device__ __forceinline__ float f16_hi(unsigned v) { return static_cast<float>(__builtin_bit_cast(f16x2, v)[1]); }

__device__ __forceinline__ f16x8 frag(const unsigned* v) {
    return __builtin_bit_cast(f16x8, u32x4{v[0], v[1], v[2], v[3]});
}
// a lane's four samples of a profile row; window starts on any sample (STEP
// 1) are 4-byte aligned, even ones 8-byte
template <int STEP>
__device__ __forceinline__ f16x8 read_quad(const unsigned char* p) {
    u32x2 h0, h1;
    if constexpr (STEP == 1) {
        h0 = *reinterpret_cast<const u32x2_a4*>(p);
        h1 = *reinterpret_cast<const u32x2_a4*>(p + 8);
    } else {
        h0 = *reinterpret_cast<const u32x2*>(p);
        asm volatile("" ::: "memory");   // kept apart: ds_read2_b64 serves fewer lanes per cycle
        h1 = *reinterpret_cast<const u32x2*>(p + 8);
        asm volatile("" ::: "memory");
    }
    return __builtin_bit_cast(f16x8, u32x4{h0[0], h0[1], h1[0], h1[1]});
}

// |X + d| - D for D = |X| and s = 2 X.d + d.d: s / (D + sqrt(D^2 + s)), then
// one Newton step on r (r + 2 D) = s, which halves the rounding error (the
// carrier takes r to a dozen revolutions over a 16x16 tile).
__device__ __forceinline__ float range_offset(float s, float D) {
    const float q = __builtin_amdgcn_rcpf(D + __builtin_amdgcn_sqrtf(fmaf(D, D, s)));
    const float r = s * q;
    return fmaf(fmaf(-r, fmaf(2.f, D, r), s), q, r);
}

// minimum over the 16 lanes of a row
template <int CTRL>
__device__ __forceinline__ int dpp_min(int v) {
    return min(v, __builtin_amdgcn_update_dpp(0x7fffffff, v, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_min(int v) {
    v = dpp_min<0x128>(v);   // row_ror:8, 4, 2, 1
    v = dpp_min<0x124>(v);
    v = dpp_min<0x122>(v);
    return static_cast<float>(dpp_min<0x121>(v));
}

// k_z bin of row r of block blk, or -1
__device__ __forceinline__ int row_bin(int blk, int r, int n_z) {
    const int m = kWindowBins * blk + (r >> 5) * 16 + (r & 15);
    if ((r >> 4) & 1) return m < n_z / 2 ? n_z - 1 - m : -1;
    return m < (n_z + 1) / 2 ? m : -1;
}

// One work item: channels [cb, ce) of (k_z block, tile); piece != nullptr
// receives the partial spectrum [pixel][row], else G the spectrum.  kr: the
// block's reference wavenumber in revolutions per metre.
template <int WCH, int STEP, bool MONO>
__device__ __forceinline__ void window_tile(const WinArgs& a, float kr, const float* __restrict__ smax,
                                            const unsigned* __restrict__ q,
                                            const GatherTileEntry* __restrict__ tab, float2* __restrict__ G,
                                            float2* __restrict__ piece, int blk, int tile, int cb, int ce,
                                            unsigned char* smem) {
    constexpr int RC = 2 * WCH + 1, RB = 16 * RC;
    constexpr unsigned kBuf = kRows * RB;
    constexpr int NI = kRows * RC / 64;                     // copy instructions per channel
    constexpr int NIW = (NI + kWaves - 1) / kWaves;
    static_assert((kRows * RC) % 64 == 0 && NI / kWaves == 2, "whole copy instructions, two for every wavefront");
    // with even window starts, the rows of mirrors (16..31 of a row tile) are
    // staged from two samples earlier: their 8-byte operand reads then take
    // the banks that those of rows 0..15 leave
    constexpr int kLead = STEP == 2 ? 2 : 0;
    constexpr float kLast = 4 * WCH - 8 - kLead;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pn = lane & 15;
    const int tx0 = (tile % a.tiles_x) * kTile, ty0 = (tile / a.tiles_x) * kTile;
    const int bx = 8 * (wave & 1), by = 4 * (wave >> 1);
    const bool active = tx0 + bx < a.nx && ty0 + by < a.ny;   // any pixel of this wavefront in the image

    const GatherTileEntry* tt = tab + static_cast<size_t>(tile) * a.n_ch;
    const float2* tc = reinterpret_cast<const float2*>(tab + static_cast<size_t>(a.n_tiles) * a.n_ch) +
                       (static_cast<size_t>(blk) * a.n_tiles + tile) * a.n_ch;
    // immutable during the launch: scalar loads through the constant address space
    const const_tile_t ttc = reinterpret_cast<const_tile_t>(reinterpret_cast<unsigned long long>(tt));

    unsigned doff[NIW];
#pragma unroll
    for (int j = 0; j < NIW; ++j) {
        const int g = (wave + kWaves * j) * 64 + lane;
        const int r = g / RC, jj = g - r * RC;
        const int kap = r < kRows ? row_bin(blk, r, a.n_z) : -1;
        const int plane = jj >= WCH ? 1 : 0, lead = (r >> 4) & 1 ? 0 : kLead;
        doff[j] = (kap >= 0 && jj < 2 * WCH)
                      ? 4u * static_cast<unsigned>((2 * kap + plane) * a.n_l + 4 * (jj - plane * WCH) + lead)
                      : 0x80000000u;
    }
    const size_t chan_words = 2 * static_cast<size_t>(a.n_z) * a.n_l;
    const unsigned chan_bytes = static_cast<unsigned>(4 * chan_words);
    // one copy instruction of a channel's rows (1 KiB of LDS): j < kEven for
    // every wavefront, the rest for the first NI % kWaves of them
    constexpr int kEven = NI / kWaves;
    auto rows = [&](int c, int win) {
        return uniform_rsrc(q + c * chan_words + (win - kLead), chan_bytes - 4u * (win - kLead));
    };
    auto copy = [&](__amdgpu_buffer_rsrc_t rs, int buf, int j) {
        PL_LDS_COPY16(rs, (lds_bytes_t)(smem + buf * kBuf) + (wave + kWaves * j) * 1024, doff[j]);
    };
    auto copy_all = [&](int c, int buf) {
        const __amdgpu_buffer_rsrc_t rs = rows(c, ttc[c].win);
#pragma unroll
        for (int j = 0; j < NIW; ++j)
            if (j < kEven || wave < NI % kWaves) copy(rs, buf, j);
    };
    // Tile-table entries and carriers of a channel pair, to slot p & 3 of the
    // entry ring (128 bytes each): lanes 0..5 the entries (48 bytes each),
    // lane 6 and 7 the carriers' 16 bytes.  Two pairs ahead of their use.
    unsigned char* ring = smem + 4 * kBuf;
    auto stage_entries = [&](int c) {
        if (wave == kWaves - 1 && lane < 8) {
            const int c0 = min(c, a.n_ch - 1), c1 = min(c + 1, a.n_ch - 1);
            const char* src = lane < 6 ? reinterpret_cast<const char*>(tt + (lane < 3 ? c0 : c1)) + 16 * (lane < 3 ? lane : lane - 3)
                                       : reinterpret_cast<const char*>(tc + (lane == 6 ? c0 : c1));
            PL_GLOBAL_LDS16(src, ring + (c >> 1 & 3) * 128);
        }
    };

    // this lane's pixel (group row & 1 of the wavefront's two) and channel of
    // the pair
    const int row = lane >> 4, cs = row >> 1;
    const float ox = (bx + 4 * (row & 1) + (pn & 3) - 7.5f) * a.dx, oy = (by + (pn >> 2) - 7.5f) * a.dy;
    const float oo = fmaf(ox, ox, oy * oy);
    const unsigned sgn = 0x3c00bc00u;   // (-1, 1) in FP16

    // byte offset of this lane's profile operand: k_z row lane % 32 of a row
    // tile, samples 4 (lane / 32) ..
    const unsigned adr = (lane & 31) * RB + (lane >> 5) * 16 + (STEP == 2 ? 8 * ((lane >> 4) & 1) : 0);

    f32x16 acc[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][t][v] = 0.f;

    __syncthreads();   // LDS free (the batch kernel reuses it per item)
    copy_all(cb, 0);
    copy_all(min(cb + 1, ce - 1), 1);
    stage_entries(cb);
    stage_entries(cb + 2);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    int buf = 0;
#pragma unroll 1
    for (int c = cb; c < ce; c += 2) {
        if (c + 2 < ce) {
            const int cz = min(c + 3, ce - 1), nb = 2 - 2 * buf;
            const unsigned char* en = ring + ((c >> 1) + 1 & 3) * 128 + 8;
            const int wa = __builtin_amdgcn_readfirstlane(*reinterpret_cast<const int*>(en));
            const int wz = __builtin_amdgcn_readfirstlane(*reinterpret_cast<const int*>(en + (cz & 1) * 48));
            const __amdgpu_buffer_rsrc_t ra = rows(c + 2, wa), rz = rows(cz, wz);
#pragma unroll
            for (int j = 0; j < NIW; ++j)
                if (j < kEven || wave < NI % kWaves) {
                    copy(ra, nb, j);
                    copy(rz, nb + 1, j);
                }
            stage_entries(c + 4);
        }
        if (active) {
            const unsigned char* en = ring + (c >> 1 & 3) * 128 + cs * 48;
            const float4 e1 = *reinterpret_cast<const float4*>(en + 16);   // uf, xt, yt, dt
            const float2 car = *reinterpret_cast<const float2*>(ring + (c >> 1 & 3) * 128 + 96 + cs * 16);
            const float base = static_cast<float>(*reinterpret_cast<const int*>(en + 12) + 1);
            // range from the tile centre's, position in the row, window start
            // (multiply-adds spelled out: the single and the batched kernel give
            // the same bits)
            const float sT = fmaf(2.f, fmaf(e1.y, ox, e1.z * oy), oo);
            float dl = range_offset(sT, e1.w);
            if (MONO) {
                dl += dl;
            } else {
                const float4 e2 = *reinterpret_cast<const float4*>(en + 32);   // xr, yr, dr
                const float sR = fmaf(2.f, fmaf(e2.x, ox, e2.y * oy), oo);
                dl += range_offset(sR, e2.z);
            }
            const float v = fmaf(dl, a.inv_du, e1.x);
            // lowest position of the group, to 1/64 sample
            const float low = fmaf(row_min(static_cast<int>(v * 64.f)), 1.f / 64, a.centre);
            // staged start of the group's window, a multiple of STEP; inside
            // the staged row by the planner's bound, the clamp holds every
            // read there
            const float st = fmaxf(0.f, fminf(rintf((base + low) * (1.f / STEP)) * STEP, kLast));
            const float x = v + (base - st) - 3.5f, z = fmaf(x * x, a.zscale, -1.f);
            const float2 c1 = cis_rev_f(kr * dl);
            const float on = c + cs < ce ? 1.f : 0.f;   // a missing second channel: B = 0
            const float cr = on * fmaf(car.x, c1.x, -(car.y * c1.y)), ci = -on * fmaf(car.x, c1.y, car.y * c1.x);   // conjugate
            // this lane's pixel's eight weights times the carrier, FP16 hi + lo
            unsigned xh[8], xl[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float ev = a.even[kDeg - 1][i], od = a.odd[kDeg - 1][i];
#pragma unroll
                for (int k = kDeg - 2; k >= 0; --k) {
                    ev = fmaf(ev, z, a.even[k][i]);
                    od = fmaf(od, z, a.odd[k][i]);
                }
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const float w = fmaf(m ? -x : x, od, ev), p = w * cr, s = w * ci;   // (Re B, -Im B)
                    const int j = m ? 7 - i : i;
                    xh[j] = pack_f16(p, s);
                    xl[j] = pack_f16(fmaf(w, cr, -f16_lo(xh[j])), fmaf(w, ci, -f16_hi(xh[j])));
                }
            }
            // halves of the wavefront exchanged: [0, 4) become channel c's
            // words (lanes 0..31 samples 0..3, 32..63 samples 4..7), [4, 8)
            // channel c + 1's
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u32x2 h = swap32(xh[j], xh[4 + j]), l = swap32(xl[j], xl[4 + j]);
                xh[j] = h[0];
                xh[4 + j] = h[1];
                xl[j] = l[0];
                xl[4 + j] = l[1];
            }
            const int so = 4 * static_cast<int>(st);
            const unsigned char* pb = smem + 2 * buf * kBuf + adr;
#pragma unroll
            for (int ch = 0; ch < 2; ++ch) {
                // operand words of the two groups: even rows of 16 lanes
                // (Re B, -Im B), odd ones (Im B, Re B)
                unsigned bh[2][4], bl[2][4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const u32x2 rh = swap16(xh[4 * ch + j], turned(xh[4 * ch + j], sgn));
                    const u32x2 rl = swap16(xl[4 * ch + j], turned(xl[4 * ch + j], sgn));
                    bh[0][j] = rh[0];
                    bh[1][j] = rh[1];
                    bl[0][j] = rl[0];
                    bl[1][j] = rl[1];
                }
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const f16x8 fh = frag(bh[g]), fl = frag(bl[g]);
                    const unsigned char* p = pb + ch * kBuf + __builtin_amdgcn_readlane(so, 32 * ch + 16 * g);
                    f16x8 ah[2], al[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        ah[t] = read_quad<STEP>(p + t * 32 * RB);
                        al[t] = read_quad<STEP>(p + t * 32 * RB + 16 * WCH);
                    }
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[g][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[t], fh, acc[g][t], 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[g][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[t], fh, acc[g][t], 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[g][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[t], fl, acc[g][t], 0, 0, 0);
                }
            }
        }
        buf ^= 1;
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }

    if (!active && !piece) return;   // no barrier follows in this item
    const int g_exp = profile_exponent(smax, a.log2_gain, lane);
    // result layout: column lane % 32 (pixel, Re below 16), rows
    // 8 (v / 4) + 4 (lane / 32) + v % 4; neighbouring rows are exchanged so
    // that a lane holds (Re, Im) of row v + lane / 16 % 2
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int lx = bx + 4 * g + (pn & 3), ly = by + (pn >> 2);
        const bool ok = tx0 + lx < a.nx && ty0 + ly < a.ny;
        float2* out = piece ? piece + (ly * kTile + lx) * kRows
                            : G + (static_cast<size_t>(ty0 + ly) * a.nx + tx0 + lx) * a.n_z;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                const u32x2 w = swap16(__float_as_uint(acc[g][t][v]), __float_as_uint(acc[g][t][v + 1]));
                const float2 val = make_float2(ldexpf(__uint_as_float(w[0]), g_exp), ldexpf(__uint_as_float(w[1]), g_exp));
                const int r = 32 * t + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3) + (row & 1);
                if (piece) {
                    out[r] = val;
                } else {
                    const int kap = row_bin(blk, r, a.n_z);
                    if (ok && kap >= 0) out[kap] = val;
                }
            }
    }
}

// The work item and channels of piece p of the split items.
__device__ __forceinline__ void split_item(const WinArgs& a, int p, int& work, int& cb, int& ce) {
    const int part = p % a.n_part;
    work = a.n_whole + p / a.n_part;
    cb = 2 * (part * a.n_pair / a.n_part);
    ce = min(a.n_ch, 2 * ((part + 1) * a.n_pair / a.n_part));
}

template <int WCH, int STEP, bool MONO>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(4)))
void backproject_window_kernel(const unsigned* __restrict__ q, const GatherTileEntry* __restrict__ tab, WinCall k,
                               float2* __restrict__ G) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const WinArgs& a = k.a;
    int work, cb = 0, ce = a.n_ch;
    float2* piece = nullptr;
    if (static_cast<int>(blockIdx.x) < a.grid_whole) {
        work = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
        if (work >= a.n_whole) return;   // workgroup-uniform, before any barrier
    } else {
        const int bt = blockIdx.x - a.grid_whole;
        const int p = (bt & 7) * a.per_xcd_tail + (bt >> 3);   // a contiguous share per XCD
        if (p >= (a.n_work - a.n_whole) * a.n_part) return;
        piece = k.part + static_cast<size_t>(p) * (kTile * kTile * kRows);
        split_item(a, p, work, cb, ce);
    }
    const int blk = work / a.n_tiles;
    window_tile<WCH, STEP, MONO>(a, k.kref_rev[blk], k.smax, q, tab, G, piece, blk, work - blk * a.n_tiles, cb, ce, smem);
}

// Persistent form for a batch of scans: eight work queues, one per XCD, of
// items (scan, work item or -1, piece) taken by atomic counters, the home
// XCD's first (as in the pixel-per-lane batch kernel).  wsr and ws are the
// same workspace: what is read (profiles, tables) and what is written.
template <int WCH, int STEP, bool MONO>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(4)))
void backproject_window_batch_kernel(const WinScanDesc* __restrict__ scans, const int4* __restrict__ items,
                                     const int* __restrict__ bounds, unsigned* __restrict__ counters,
                                     const char* __restrict__ wsr, char* __restrict__ ws) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int* next = reinterpret_cast<int*>(smem);   // the row buffers are free between items
    const int home = blockIdx.x & 7;
    for (int k = 0; k < 8; ++k) {
        const int x = (home + k) & 7;
        const int lo = bounds[x], hi = bounds[x + 1];
        for (;;) {
            if (threadIdx.x == 0) *next = lo + static_cast<int>(atomicAdd(counters + x, 1u));
            __syncthreads();
            const int it = __builtin_amdgcn_readfirstlane(*next);
            __syncthreads();   // every thread has read `next` before it is overwritten
            if (it >= hi) break;
            const int4 w = items[it];
            const WinScanDesc& d = scans[__builtin_amdgcn_readfirstlane(w.x)];
            const WinArgs a = d.a;
            int work = __builtin_amdgcn_readfirstlane(w.y), cb = 0, ce = a.n_ch;
            float2* piece = nullptr;
            if (work < 0) {
                const int p = __builtin_amdgcn_readfirstlane(w.z);
                piece = reinterpret_cast<float2*>(ws + d.part_off) + static_cast<size_t>(p) * (kTile * kTile * kRows);
                split_item(a, p, work, cb, ce);
            }
            const int blk = work / a.n_tiles;
            window_tile<WCH, STEP, MONO>(a, d.kref_rev[blk], reinterpret_cast<const float*>(wsr + d.smax_off),
                                         reinterpret_cast<const unsigned*>(wsr + d.q_off),
                                         reinterpret_cast<const GatherTileEntry*>(wsr + d.tab_off),
                                         reinterpret_cast<float2*>(ws + d.g_off), piece, blk, work - blk * a.n_tiles,
                                         cb, ce, smem);
            __syncthreads();   // LDS is reused by the next item
        }
    }
}

__global__ void reset_window_counters_kernel(unsigned* c) {
    if (threadIdx.x < 8) c[threadIdx.x] = 0u;
}

struct WinTailArgs {
    int n_whole, n_part, n_tiles, tiles_x, nx, ny, n_z;
    long long n_elems;   // tail items x elements per piece
};

// The pieces of every split item added in piece order into G.
__global__ void window_combine_kernel(const float2* __restrict__ part, WinTailArgs a, float2* __restrict__ G) {
    constexpr int tp = kTile * kTile * kRows;
    for (long long e = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; e < a.n_elems;
         e += static_cast<long long>(gridDim.x) * blockDim.x) {
        const int t = static_cast<int>(e / tp), r = static_cast<int>(e - static_cast<long long>(t) * tp);
        const int lp = r / kRows;
        const int work = a.n_whole + t;
        const int blk = work / a.n_tiles, tile = work - blk * a.n_tiles;
        const int gx = (tile % a.tiles_x) * kTile + lp % kTile, gy = (tile / a.tiles_x) * kTile + lp / kTile;
        const int kap = row_bin(blk, r - lp * kRows, a.n_z);
        if (gx >= a.nx || gy >= a.ny || kap < 0) continue;
        const float2* src = part + static_cast<size_t>(t) * a.n_part * tp + r;
        float2 acc = src[0];
        for (int k = 1; k < a.n_part; ++k) {
            const float2 v = src[static_cast<size_t>(k) * tp];
            acc.x += v.x;
            acc.y += v.y;
        }
        G[(static_cast<size_t>(gy) * a.nx + gx) * a.n_z + kap] = acc;
    }
}

WinArgs window_args(const HybridPlan& p) {
    WinArgs a{};
    a.n_ch = p.n_ch;
    a.n_z = p.n_z;
    a.n_l = p.n_l;
    a.nx = p.nx;
    a.ny = p.ny;
    a.tiles_x = p.tiles_x;
    a.n_tiles = p.tiles_x * p.tiles_y;
    a.n_work = a.n_tiles * p.n_blocks;
    a.n_pair = (p.n_ch + 1) / 2;
    a.dx = static_cast<float>(p.dx);
    a.dy = static_cast<float>(p.dy);
    a.inv_du = static_cast<float>(1.0 / p.du);
    a.zscale = static_cast<float>(p.win_z);
    a.centre = static_cast<float>(0.5 * p.win_span - 3.5);
    std::memcpy(a.even, p.win_even, sizeof(a.even));
    std::memcpy(a.odd, p.win_odd, sizeof(a.odd));
    a.log2_gain = p.log2_gain;
    return a;
}

// A plan's kernel variant: rows of 8 or 9 chunks, window starts on any or
// even samples, one antenna or two per channel.
#define PL_WIN_CLASSES(X) X(8, 1, true) X(9, 1, true) X(8, 2, true) X(9, 2, true) X(8, 1, false) X(9, 1, false) X(8, 2, false) X(9, 2, false)

const void* window_kernel(int wch, int step, bool mono, bool batch) {
#define PL_WIN(W_, S_, M_)                                                                              \
    if (wch == W_ && step == S_ && mono == M_)                                                          \
        return batch ? reinterpret_cast<const void*>(backproject_window_batch_kernel<W_, S_, M_>)       \
                     : reinterpret_cast<const void*>(backproject_window_kernel<W_, S_, M_>);
    PL_WIN_CLASSES(PL_WIN)
#undef PL_WIN
    return nullptr;
}

// Workgroups resident at once (the kernel's LDS size is set on first use).
int window_slots(int wch, int step, bool mono, bool batch, long long* slots) {
    const void* fn = window_kernel(wch, step, mono, batch);
    if (!fn) return fail(PL_EUNSUPPORTED, "no window back-projection for rows of %d chunks", wch);
    const size_t smem = backproject_window_lds_bytes(wch);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem)) != hipSuccess)
        return fail(PL_EDEVICE, "window back-projection: LDS of %zu bytes refused", smem);
    static std::atomic<int> cache[16];   // per CU, by variant; 0: not asked yet
    std::atomic<int>& slot = cache[(wch == 9) + 2 * (step == 2) + 4 * mono + 8 * batch];
    int per_cu = slot.load(std::memory_order_relaxed);
    if (per_cu == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * kWaves, smem) != hipSuccess || per_cu < 1)
            return fail(PL_EDEVICE, "window back-projection: occupancy query failed");
        slot.store(per_cu, std::memory_order_relaxed);
    }
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return fail(PL_EDEVICE, "window back-projection: device query failed");
    *slots = static_cast<long long>(per_cu) * cus;
    return PL_OK;
}

int check_window_plan(const HybridPlan& p) {
    if (!p.bp_window || p.window % 4 || p.window / 2 + 1 != p.window_pad || p.window + 4 > p.n_l ||
        p.n_blocks > kMaxBlocks / 2 || static_cast<unsigned long long>(p.n_z) * p.n_l * 8 >= (1ull << 31))
        return fail(PL_EUNSUPPORTED, "window back-projection: window %d, %d range samples", p.window, p.n_l);
    return PL_OK;
}

// Tail split, as in the other matrix-core back-projection: the items beyond
// the last full round of resident workgroups, if at most half a round, run
// in pieces over their channel pairs that fill it, as far as the workspace
// holds their partial spectra (planned for kWindowSlots workgroups).
int split_tail(const HybridPlan& p, WinArgs* a) {
    long long slots = 0;
    if (int rc = window_slots(p.window / 4, p.win_step, p.mode == PL_MONO, false, &slots)) return rc;
    a->n_whole = a->n_work;
    a->n_part = 1;
    const long long tail = a->n_work % slots;
    if (tail > 0 && 2 * tail <= slots) {
        const long long k =
            std::min({slots / tail, static_cast<long long>(a->n_pair), static_cast<long long>(p.part_pieces) / tail});
        if (k >= 2) {
            a->n_whole = static_cast<int>(a->n_work - tail);
            a->n_part = static_cast<int>(k);
        }
    }
    return PL_OK;
}

int launch_combine(const WinArgs& a, const float2* part, float2* G, hipStream_t s) {
    if (a.n_part == 1) return PL_OK;
    WinTailArgs t{};
    t.n_whole = a.n_whole;
    t.n_part = a.n_part;
    t.n_tiles = a.n_tiles;
    t.tiles_x = a.tiles_x;
    t.nx = a.nx;
    t.ny = a.ny;
    t.n_z = a.n_z;
    t.n_elems = static_cast<long long>(a.n_work - a.n_whole) * kTile * kTile * kRows;
    const unsigned cblocks = static_cast<unsigned>(std::min<long long>((t.n_elems + 255) / 256, 8192));
    hipLaunchKernelGGL(window_combine_kernel, dim3(cblocks), dim3(256), 0, s, part, t, G);
    return check_launch("back-projection (window) tail combine");
}

void set_kref(const HybridPlan& p, float* kref_rev) {
    for (int b = 0; b < p.n_blocks; ++b) kref_rev[b] = static_cast<float>(p.kref[b] * (0.5 / kPi));
}

// The largest |Re| or |Im| of the n spectrum values in kSpectrumMaxParts
// parts, one workgroup of sixteen wavefronts each with four loads in flight
// per lane: a plain read of the spectrum (470 MB in 100 us; with four
// wavefronts and one load 220).
__global__ __launch_bounds__(kMaxThreads) void spectrum_max_kernel(const float4* __restrict__ s, long long n,
                                                                   float* __restrict__ parts) {
    __shared__ float red[kMaxThreads / 64];
    const long long n4 = n / 2, step = static_cast<long long>(gridDim.x) * kMaxThreads;
    float m = 0.f;
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        const float2 v = reinterpret_cast<const float2*>(s)[n - 1];
        m = fmaxf(fabsf(v.x), fabsf(v.y));
    }
    auto take = [&](const float4& v) {
        m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    };
    long long i = blockIdx.x * static_cast<long long>(kMaxThreads) + threadIdx.x;
    for (; i + 3 * step < n4; i += 4 * step) {
        const float4 v0 = s[i], v1 = s[i + step], v2 = s[i + 2 * step], v3 = s[i + 3 * step];
        take(v0);
        take(v1);
        take(v2);
        take(v3);
    }
    for (; i < n4; i += step) take(s[i]);
    for (int d = 32; d; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kMaxThreads / 64; ++w) m = fmaxf(m, red[w]);
        parts[blockIdx.x] = m;
    }
}

}  // namespace

// two buffers of a channel pair's rows, and the entry ring
size_t backproject_window_lds_bytes(int chunks) { return 4ull * kRows * 16 * (2 * chunks + 1) + 4 * 128; }

int launch_spectrum_max(const HybridPlan& p, const float2* spec, char* ws, hipStream_t s) {
    const long long n = static_cast<long long>(p.n_ch) * p.n_z * p.n_f;
    hipLaunchKernelGGL(spectrum_max_kernel, dim3(kSpectrumMaxParts), dim3(kMaxThreads), 0, s,
                       reinterpret_cast<const float4*>(spec), n, reinterpret_cast<float*>(ws + p.off_smax));
    return check_launch("spectrum maximum");
}

int launch_backproject_window(const HybridPlan& p, const unsigned* q, char* ws, float2* G, hipStream_t s) {
    if (int rc = check_window_plan(p)) return rc;
    WinCall k{};
    k.a = window_args(p);
    WinArgs& a = k.a;
    if (int rc = split_tail(p, &a)) return rc;
    a.per_xcd = (a.n_whole + 7) / 8;
    a.grid_whole = 8 * a.per_xcd;
    a.per_xcd_tail = static_cast<int>((static_cast<long long>(a.n_work - a.n_whole) * a.n_part + 7) / 8);
    k.smax = reinterpret_cast<const float*>(ws + p.off_smax);
    k.part = reinterpret_cast<float2*>(ws + p.off_part);
    set_kref(p, k.kref_rev);
    const GatherTileEntry* tab = reinterpret_cast<const GatherTileEntry*>(ws + p.off_tiles);
    const unsigned blocks = static_cast<unsigned>(a.grid_whole + 8LL * a.per_xcd_tail);
    const size_t smem = backproject_window_lds_bytes(p.window / 4);
    int rc = fail(PL_EUNSUPPORTED, "no window back-projection for rows of %d samples", p.window);
#define PL_WIN(W_, S_, M_)                                                                                         \
    if (p.window == 4 * W_ && p.win_step == S_ && (p.mode == PL_MONO) == M_) {                                     \
        clear_error();                                                                                             \
        hipLaunchKernelGGL((backproject_window_kernel<W_, S_, M_>), dim3(blocks), dim3(64 * kWaves), smem, s, q,   \
                           tab, k, G);                                                                             \
        rc = check_launch("back-projection (window)");                                                             \
    }
    PL_WIN_CLASSES(PL_WIN)
#undef PL_WIN
    return rc ? rc : launch_combine(a, k.part, G, s);
}

size_t window_batch_desc_bytes() { return sizeof(WinScanDesc); }

int build_window_batch_desc(const HybridPlan& p, size_t ws_off, void* out, int* n_whole, int* n_pieces) {
    if (int rc = check_window_plan(p)) return rc;
    WinScanDesc d{};
    d.a = window_args(p);
    if (int rc = split_tail(p, &d.a)) return rc;
    set_kref(p, d.kref_rev);
    d.q_off = ws_off + p.off_q;
    d.tab_off = ws_off + p.off_tiles;
    d.g_off = ws_off + p.off_G;
    d.part_off = ws_off + p.off_part;
    d.smax_off = ws_off + p.off_smax;
    *n_whole = d.a.n_whole;
    *n_pieces = (d.a.n_work - d.a.n_whole) * d.a.n_part;
    std::memcpy(out, &d, sizeof(d));
    return PL_OK;
}

int window_batch_grid(int wch, int step, bool mono, int* blocks) {
    long long slots = 0;
    if (int rc = window_slots(wch, step, mono, true, &slots)) return rc;
    *blocks = static_cast<int>((slots + 7) & ~7LL);
    return PL_OK;
}

int launch_window_batch(const void* descs, const void* items, const int* bounds, unsigned* counters, char* ws, int wch,
                        int step, bool mono, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(reset_window_counters_kernel, dim3(1), dim3(64), 0, s, counters);
    if (int rc = check_launch("batch work counters")) return rc;
    const size_t smem = backproject_window_lds_bytes(wch);
#define PL_WIN(W_, S_, M_)                                                                                            \
    if (wch == W_ && step == S_ && mono == M_) {                                                                      \
        hipLaunchKernelGGL((backproject_window_batch_kernel<W_, S_, M_>), dim3(blocks), dim3(64 * kWaves), smem, s,   \
                           static_cast<const WinScanDesc*>(descs), static_cast<const int4*>(items), bounds, counters, \
                           ws, ws);                                                                                   \
        return check_launch("batched back-projection (window)");                                                      \
    }
    PL_WIN_CLASSES(PL_WIN)
#undef PL_WIN
    return fail(PL_EUNSUPPORTED, "no window back-projection for rows of %d chunks", wch);
}

int launch_window_combine(const HybridPlan& p, char* ws, hipStream_t s) {
    WinArgs a = window_args(p);
    if (int rc = split_tail(p, &a)) return rc;
    return launch_combine(a, reinterpret_cast<const float2*>(ws + p.off_part), reinterpret_cast<float2*>(ws + p.off_G), s);
}

}  // namespace pl
